"""The general kernels' matrix-core gauge and lane-parallel quantiser at the sizes where they can go
wrong: every group size that has a variant of its own and ones that stay on the vector ALU, heads
whose channel blocks do not divide evenly over the waves, blocks the lanes share and blocks one
thread takes, and batches around the 16 rows of an operand.

With the identity gauge z = x on both sides, so codes, side information and raw windows equal the
oracle's bit for bit; with a Haar gauge the fused-encoder criteria of tests/_parity.py apply."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2607_20538_amd import codec as cg
from paper_2607_20538_amd import synth

from _parity import bf16_dev, cache_to_dev, cache_to_host, check_fused_codes, to_cg, x_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cg.lib()


def _gauge(kind, L, H, d, g, seed=23):
    G = O.gauge_make(kind, L, H, d, g, seed=seed)
    shp = cg.shape(L, H, d, g)
    Gd = cg.alloc_gauge(shp)
    cg.gauge_make(cg.GAUGE_USER, shp, params=G, G_host=None, G_dev=Gd)
    return G, Gd, shp


def _workload(L, B, H, T, d, dtype):
    return synth.Workload("dims", L=L, B=B, H=H, T=T, d=d, dtype=dtype, g=0, backend="bu", bits=4, data_seed=0xD1)


# (d, g, bits, n, block_t or backend): matrix-core groups 16, 32, 64, 80, 96, 128, 192, 256, vector-ALU
# groups 8, 12, 48; blocks of 80 and 96 channels take one thread each
DIMS = [
    (32, 16, 4, 32, 1), (32, 32, 2, 16, 1), (48, 16, 4, 16, 1), (64, 64, 3, 32, 1), (64, 8, 6, 64, 1),
    (64, 32, 4, 32, 16), (80, 80, 4, 80, 1), (80, 16, 6, 16, 1), (96, 96, 4, 96, 1), (96, 48, 3, 32, 1),
    (96, 12, 8, 32, 1), (96, 32, 4, 32, 4), (128, 128, 6, 64, 1), (128, 64, 4, 128, 1), (192, 192, 4, 64, 1),
    (192, 64, 8, 32, 2), (256, 256, 3, 64, 1), (256, 128, 4, 256, 1), (256, 16, 2, 64, 32), (16, 16, 4, 16, 1),
]


@pytest.mark.parametrize("kind", [O.GAUGE_IDENTITY, O.GAUGE_HAAR], ids=["identity", "haar"])
@pytest.mark.parametrize("d,g,bits,n,bt", DIMS)
def test_append_over_head_widths(d, g, bits, n, bt, kind):
    """Rows at different positions, batches of 1 and 17 rows; the last tokens of tiles appended."""
    L, H, T_cap = 2, 2, 128
    dtype = "bf16" if bt > 1 or d % 64 else "f32"
    oc = O.Codec(backend=O.BLOCK_UNIFORM, bits=bits, block_c=n, block_t=bt)
    G, Gd, shp = _gauge(kind, L, H, d, g)
    for B in (1, 17):
        w = _workload(L, B, H, T_cap, d, dtype)
        X = [synth.kv_tensor(w, s) for s in (0, 1)]
        start = np.array([(32 if bt > 1 else 5) + (b % 3) * bt for b in range(B)])
        ref, dev = [], []
        for s in (0, 1):
            r, _ = O.kv_encode(oc, s, np.ascontiguousarray(X[s][:, :, :, :32]), G, T_cap=T_cap)
            ref.append(r)
            dev.append(cache_to_dev(r, oc, s, L, B, H, T_cap, d))
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        for i in range(bt):
            pos = start + i
            new = [np.ascontiguousarray(X[s][:, np.arange(B), :, pos].transpose(1, 0, 2, 3)) for s in (0, 1)]
            for s in (0, 1):
                O.kv_append(oc, s, new[s], G, ref[s], pos)
            cg.kv_append_step(0, L, x_dev(new[0][:, :, :, None, :]), x_dev(new[1][:, :, :, None, :]),
                              torch.tensor(pos, dtype=torch.int32, device="cuda"), Gd, shp, to_cg(oc), dev[0], dev[1],
                              err_flag=err)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        for s in (0, 1):
            got = cache_to_host(dev[s], oc, s)
            if kind == O.GAUGE_IDENTITY:
                for key in ("codes", "side", "residual"):
                    if got[key] is not None:
                        np.testing.assert_array_equal(got[key], ref[s][key], err_msg=key)
            else:
                # the appended tokens alone: token rows gathered per batch row
                z, _ = O.kv_encode(O.Codec(backend=O.PASSTHROUGH), s, X[s], G, T_cap=T_cap)
                pick = lambda a, u: np.stack([a[:, b, :, start[b] // u:start[b] // u + bt // u] for b in range(B)], 1)
                sub = lambda c: {"codes": pick(c["codes"], 1), "side": pick(c["side"], bt), "residual": None}
                check_fused_codes(sub(got), sub(ref[s]), pick(z["codes"], 1), oc, s, d, bt)


@pytest.mark.parametrize("g", [16, 128])
def test_append_kivi_flush_over_group_sizes(g):
    """The KIVI window flushed by the newest token: key groups of 16 and 64 tokens (32 runs elsewhere)."""
    L, B, H, d = 1, 2, 2, 128
    for kg, bits in ((16, 4), (64, 3)):
        oc = O.Codec(backend=O.KIVI, bits=bits, key_tokens=kg, val_channels=64, residual=kg)
        T_cap = 4 * kg
        w = _workload(L, B, H, T_cap, d, "bf16")
        G, Gd, shp = _gauge(O.GAUGE_IDENTITY, L, H, d, g)
        X = [synth.kv_tensor(w, s) for s in (0, 1)]
        T0 = 3 * kg - 1                      # the next token completes a group
        ref, dev = [], []
        for s in (0, 1):
            r, _ = O.kv_encode(oc, s, np.ascontiguousarray(X[s][:, :, :, :T0]), G, T_cap=T_cap)
            ref.append(r)
            dev.append(cache_to_dev(r, oc, s, L, B, H, T_cap, d, len_=T0))
        pos = np.array([T0, T0])
        new = [np.ascontiguousarray(X[s][:, :, :, T0]) for s in (0, 1)]
        for s in (0, 1):
            O.kv_append(oc, s, new[s], G, ref[s], pos)
        cg.kv_append_step(0, L, bf16_dev(new[0][:, :, :, None, :]), bf16_dev(new[1][:, :, :, None, :]),
                          torch.tensor(pos, dtype=torch.int32, device="cuda"), Gd, shp, to_cg(oc), dev[0], dev[1])
        torch.cuda.synchronize()
        for s in (0, 1):
            got = cache_to_host(dev[s], oc, s)
            for key in ("codes", "side", "residual"):
                np.testing.assert_array_equal(got[key], ref[s][key], err_msg=key)
