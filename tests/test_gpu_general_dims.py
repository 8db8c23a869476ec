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

from _parity import (GAUGE_TOL, bf16_dev, cache_to_dev, cache_to_host, check_bf16_within_ulp, check_fused_codes,
                     group_rel_err, out_host, to_cg, x_dev)

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


@pytest.mark.parametrize("kind", [O.GAUGE_IDENTITY, O.GAUGE_HAAR], ids=["identity", "haar"])
@pytest.mark.parametrize("g", [16, 128])
def test_append_kivi_flush_over_group_sizes(g, kind):
    """The KIVI window flushed by the newest token: key groups of 16 and 64 tokens (32 runs elsewhere)."""
    L, B, H, d = 1, 2, 2, 128
    for kg, bits in ((16, 4), (64, 3)):
        oc = O.Codec(backend=O.KIVI, bits=bits, key_tokens=kg, val_channels=64, residual=kg)
        T_cap = 4 * kg
        w = _workload(L, B, H, T_cap, d, "bf16")
        G, Gd, shp = _gauge(kind, L, H, d, g)
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
            if kind == O.GAUGE_IDENTITY:
                for key in ("codes", "side", "residual"):
                    np.testing.assert_array_equal(got[key], ref[s][key], err_msg=key)
            else:
                np.testing.assert_array_equal(got["residual"], ref[s]["residual"])
                z, _ = O.kv_encode(O.Codec(backend=O.PASSTHROUGH), s, X[s], G, T_cap=T_cap)
                pick = lambda a, u: a[:, :, :, kg // u:2 * kg // u]  # the flushed group's rows
                u = kg if s == 0 else 1
                sub = lambda c: {"codes": pick(c["codes"], u), "side": pick(c["side"], u), "residual": None}
                check_fused_codes(sub(got), sub(ref[s]), pick(z["codes"], 1), oc, s, d, kg)


# (backend, bits, n, block_t): every way the encoder stores a tile and the decoder fills one
STORES = [(O.BLOCK_UNIFORM, 4, 32, 1), (O.BLOCK_UNIFORM, 3, 32, 16), (O.KIVI, 2, 32, 1), (O.ZFP, 3, 32, 1),
          (O.PASSTHROUGH, 8, 32, 1)]


def _round_trip(oc, kind, L, B, H, T, d, g, dtype):
    """Encode and decode K and V, each against the oracle."""
    T_cap = (T + 31) // 32 * 32
    w = _workload(L, B, H, T, d, dtype)
    G, Gd, shp = _gauge(kind, L, H, d, g)
    for s in (0, 1):
        X = synth.kv_tensor(w, s)
        ref, flags = O.kv_encode(oc, s, X, G, T_cap=T_cap)
        dev = cg.Cache(to_cg(oc), s, L, B, H, T_cap, d)
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        cg.kv_encode(s, x_dev(X), Gd, shp, to_cg(oc), dev, err_flag=err)
        torch.cuda.synchronize()
        assert int(err.item()) == flags == 0
        got = cache_to_host(dev, oc, s)
        if kind == O.GAUGE_IDENTITY:
            for key in ("codes", "side", "residual"):
                if got[key] is not None:
                    np.testing.assert_array_equal(got[key], ref[key], err_msg=key)
        elif oc.backend == O.PASSTHROUGH:
            assert group_rel_err(ref["codes"], got["codes"], g) <= GAUGE_TOL
        elif oc.backend != O.ZFP:
            z, _ = O.kv_encode(O.Codec(backend=O.PASSTHROUGH), s, X, G, T_cap=T_cap)
            tq = O.kivi_tq(T, oc) if oc.backend == O.KIVI else O.tile_tq(T, oc)
            check_fused_codes(got, ref, z["codes"], oc, s, d, tq)
        # decode of the oracle's cache, from the start and from an offset
        cache = cache_to_dev(ref, oc, s, L, B, H, T_cap, d, len_=T)
        for t0 in (0, 36):
            want = O.kv_decode(oc, s, G, ref, t0, T - t0, lens=np.full(B, T, np.int32), out_bf16=False)
            for dt in (torch.float32, torch.bfloat16):
                Y = torch.zeros((L, B, H, T - t0, d), dtype=dt, device="cuda")
                cg.kv_decode(s, cache, Gd, shp, to_cg(oc), t0, Y, err_flag=err)
                torch.cuda.synchronize()
                if dt == torch.float32:
                    assert group_rel_err(want, Y.cpu().numpy(), g) <= GAUGE_TOL
                else:
                    check_bf16_within_ulp(want, out_host(Y), g)
        assert int(err.item()) == 0


@pytest.mark.parametrize("kind", [O.GAUGE_IDENTITY, O.GAUGE_HAAR], ids=["identity", "haar"])
@pytest.mark.parametrize("backend,bits,n,bt", STORES)
@pytest.mark.parametrize("d,g", [(32, 32), (64, 64), (64, 8), (96, 96), (96, 48), (192, 192), (256, 256)])
def test_round_trip_over_head_widths(d, g, backend, bits, n, bt, kind):
    """A ragged last tile, offsets inside a tile, window and staged rows."""
    oc = O.Codec(backend=backend, bits=bits, block_c=n, key_tokens=32, val_channels=n, residual=32, block_t=bt)
    T = 204 if backend == O.ZFP else 205
    _round_trip(oc, kind, 1, 2, 2, T, d, g, "bf16" if backend == O.KIVI or bt > 1 or d == 96 else "f32")


@pytest.mark.parametrize("kind", [O.GAUGE_IDENTITY, O.GAUGE_HAAR], ids=["identity", "haar"])
@pytest.mark.parametrize("d,g,bits,n", [(64, 64, 4, 32), (80, 80, 4, 80), (64, 16, 6, 16), (48, 16, 2, 16)])
def test_round_trip_with_several_tiles_per_workgroup(d, g, bits, n, kind):
    """Enough tokens that a workgroup runs several 64-token tiles, the next one fetched ahead."""
    oc = O.Codec(backend=O.BLOCK_UNIFORM, bits=bits, block_c=n)
    _round_trip(oc, kind, 2, 2, 16, 64 * 34 + 5, d, g, "bf16")


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d,g", [(64, 64), (96, 12), (192, 64)])
def test_strided_views(d, g, dt):
    """Views of tensors laid out [L][B][T][H][d] with padded rows (encode, decode, append) give the bytes that
    contiguous ones do, and nothing between their rows is written."""
    L, B, H, T = 2, 2, 3, 75
    _, Gd, shp = _gauge(O.GAUGE_HAAR, L, H, d, g)
    oc = cg.Codec(cg.BLOCK_UNIFORM, 4, 32)
    X = torch.randn((L, B, H, T, d), generator=torch.Generator().manual_seed(8)).to(dt).cuda()

    def strided(fill):
        return torch.full((L, B, T, H, d + 8), fill, dtype=dt, device="cuda").permute(0, 1, 3, 2, 4)[..., :d]

    Xs = strided(float("nan"))
    Xs.copy_(X)
    out = []
    for x in (X, Xs):
        k = [cg.Cache(oc, s, L, B, H, 96, d) for s in (0, 1)]
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        for s in (0, 1):
            cg.kv_encode(s, x, Gd, shp, oc, k[s], err_flag=err)
        Y = torch.full_like(X, 7.0) if x is X else strided(7.0)
        cg.kv_decode(0, k[0], Gd, shp, oc, 3, Y[:, :, :, : T - 3], err_flag=err)
        pos = torch.tensor([80, 81], dtype=torch.int32, device="cuda")
        cg.kv_append_step(0, L, x[:, :, :, 5:6], x[:, :, :, 6:7], pos, Gd, shp, oc, k[0], k[1], err_flag=err)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        out.append((k, Y))
    for s in (0, 1):
        assert torch.equal(out[0][0][s].codes, out[1][0][s].codes) and torch.equal(out[0][0][s].side, out[1][0][s].side)
    assert torch.equal(out[0][1], out[1][1]) and (out[1][1][:, :, :, T - 3:] == 7.0).all()
    base = out[1][1].as_strided((L, B, T, H, d + 8), (B * T * H * (d + 8), T * H * (d + 8), H * (d + 8), d + 8, 1))
    assert (base[..., d:] == 7.0).all()


def _half(v, up):
    """binary64 values rounded to binary16 upwards or downwards (no -0), as binary64."""
    h = v.to(torch.float16)
    off = h.double() < v if up else h.double() > v
    b = h.view(torch.int16).to(torch.int32)
    step = torch.where((b < 0) != (not up), -1, 1)        # away from zero: up the positive, down the negative
    h = torch.where(off, b + step, b).to(torch.int16).view(torch.float16).double()
    return torch.where(h == 0, torch.zeros_like(h), h)


@pytest.mark.parametrize("d,g,paged", [(128, 8, True), (128, 16, True), (128, 32, True), (128, 64, True), (128, 128, True),
                                       (64, 32, False), (64, 64, False), (96, 96, False), (256, 32, False)])
def test_three_planes_are_no_further_from_binary64_than_the_binary32_chain(d, g, paged):
    """bf16 tokens run the gauge as three bf16 planes of G, the same tokens in binary32 as a chain of binary32
    FMAs.  Side words and 8-bit codes that differ from those of z in binary64, over 2^23 values: an error of z
    moves each with a probability proportional to it, so the counts compare the errors.  They are near
    Poisson; the planes' may exceed the chain's by three standard deviations of the difference.  (Counted
    at 2^25 values: 2.3e-5 of the codes against 3.0e-5 at g = 128, 1.7e-5 against 1.7e-5 at g = 8.)"""
    H, T, n, P = 8, 1024, 16, 64
    B = max(1, 2 ** 23 // (H * T * d))
    oc = cg.Codec(cg.BLOCK_UNIFORM, 8, n)
    G, Gd, shp = _gauge(O.GAUGE_HAAR, 1, H, d, g)
    X = torch.randn((1, B, H, T, d), generator=torch.Generator().manual_seed(12)).to(torch.bfloat16).cuda()
    M = torch.from_numpy(G[0, 0]).cuda().double().transpose(-1, -2).contiguous()      # [H][R][g][g]
    x = X[0].double().reshape(B, H, T, d // g, g).permute(1, 3, 0, 2, 4).reshape(H * (d // g), B * T, g)
    z = torch.bmm(x.contiguous(), M.reshape(-1, g, g))
    z = z.reshape(H, d // g, B, T, g).permute(2, 0, 3, 1, 4).reshape(B, H, T, d // n, n)
    mn = _half(z.amin(-1), False)
    sc = _half((z.amax(-1) - mn) / 255.0, True)
    want = torch.clamp(torch.round((z - mn[..., None]) / sc[..., None]), 0, 255).to(torch.uint8)
    counts = []
    for xx in (X, X.float()):
        if paged:
            pages = torch.arange(B * T // P, dtype=torch.int32, device="cuda").reshape(B, T // P)
            k = cg.Cache(oc, 0, 1, B * T // P, H, P, d)
            cg.kv_encode_paged(0, xx, cg.page_table(pages, P), Gd, shp, oc, k, 0)
            rows = lambda t: t.view(B, T // P, H, P, -1).permute(0, 2, 1, 3, 4).reshape(B, H, T, -1)
        else:
            k = cg.Cache(oc, 0, 1, B, H, T, d)
            cg.kv_encode(0, xx, Gd, shp, oc, k)
            rows = lambda t: t.view(B, H, T, -1)
        torch.cuda.synchronize()
        side = rows(k.side.view(torch.float16)).reshape(B, H, T, d // n, 2).double()
        codes = rows(k.codes).reshape(B, H, T, d // n, n)
        assert (codes.int() - want.int()).abs().max() <= 1
        counts.append(int((side[..., 0] != mn).sum() + (side[..., 1] != sc).sum() + (codes != want).sum()))
    planes, chain = counts
    assert planes <= chain + 3 * (planes + chain) ** 0.5, counts
    assert 0 < chain < 2e-4 * z.numel(), counts           # the reference is the same arithmetic


def test_round_trip_of_64_token_key_groups():
    """Tiles of more granules than a thread fetches ahead (64 tokens of 256 channels)."""
    oc = O.Codec(backend=O.KIVI, bits=4, key_tokens=64, val_channels=64, residual=64)
    _round_trip(oc, O.GAUGE_IDENTITY, 1, 1, 2, 64 * 5 + 33, 256, 64, "bf16")


def test_general_encoder_flags_and_keeps_neighbouring_groups():
    """A non-finite channel sets NONFINITE and leaves every other group's codes alone."""
    d, g, T = 64, 16, 64
    oc = cg.Codec(cg.BLOCK_UNIFORM, 4, 16)
    _, Gd, shp = _gauge(O.GAUGE_HAAR, 1, 1, d, g)
    X = torch.randn((1, 1, 1, T, d), device="cuda")
    caches = []
    for bad in (None, float("nan"), float("inf")):
        x = X.clone()
        if bad is not None:
            x[0, 0, 0, 33, 20] = bad
        k = cg.Cache(oc, 0, 1, 1, 1, T, d)
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        cg.kv_encode(0, x, Gd, shp, oc, k, err_flag=err)
        torch.cuda.synchronize()
        assert bool(int(err.item()) & cg.CG_FLAG_NONFINITE) == (bad is not None)
        caches.append((k.codes.view(T, 4, 8).clone(), k.side.view(T, 4, 4).clone()))
    keep = torch.ones((T, 4), dtype=torch.bool, device="cuda")
    keep[33, 1] = False
    for codes, side in caches[1:]:
        assert torch.equal(codes[keep], caches[0][0][keep]) and torch.equal(side[keep], caches[0][1][keep])


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("d,g,n,backend", [(64, 64, 16, O.BLOCK_UNIFORM), (64, 32, 64, O.BLOCK_UNIFORM), (96, 32, 32, O.KIVI),
                                           (80, 16, 16, O.BLOCK_UNIFORM)])
def test_non_finite_bf16_tokens_as_binary32_ones(d, g, n, backend, bad):
    """Token rows of bf16 tensors (three gauge planes where g is a multiple of 32): with the identity gauge
    every byte and flag is that of the same tokens in binary32 (KIVI takes bf16 alone: of the
    block-uniform values), also where a channel, a group or a whole token is not finite."""
    T = 192
    shp = cg.shape(1, 1, d, g)
    Gd = cg.alloc_gauge(shp)
    cg.gauge_make(cg.GAUGE_IDENTITY, shp, G_host=None, G_dev=Gd)
    X = torch.randn((1, 1, 1, T, d), generator=torch.Generator().manual_seed(3)).to(torch.bfloat16).cuda()
    X[0, 0, 0, 33, g // 2] = bad
    X[0, 0, 0, 70, :g] = bad
    X[0, 0, 0, 5] = bad
    tq = 160 if backend == O.KIVI else T
    out = []
    for oc, x in ((cg.Codec(backend, 4, n, 32, n, 32), X), (cg.Codec(cg.BLOCK_UNIFORM, 4, n), X[:, :, :, :tq].float())):
        k = cg.Cache(oc, 1, 1, 1, 1, T, d)
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        cg.kv_encode(1, x, Gd, shp, oc, k, err_flag=err)
        torch.cuda.synchronize()
        out.append((k.codes.view(T, -1)[:tq].clone(), k.side.view(T, -1)[:tq].clone(), int(err.item())))
    assert out[0][2] == out[1][2] and out[1][2] & cg.CG_FLAG_NONFINITE
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("d,g", [(64, 32), (192, 64)])
def test_three_plane_encoder_keeps_neighbouring_groups(d, g, bad):
    """As above for bf16 token rows: the blocks of the other groups, and every other token, keep their bytes."""
    T, n = 160, 16
    oc = cg.Codec(cg.BLOCK_UNIFORM, 4, n)
    _, Gd, shp = _gauge(O.GAUGE_HAAR, 1, 1, d, g)
    X = torch.randn((1, 1, 1, T, d), generator=torch.Generator().manual_seed(4)).to(torch.bfloat16).cuda()
    spoilt = X.clone()
    spoilt[0, 0, 0, 33, 5] = bad
    out = []
    for x in (X, spoilt):
        k = cg.Cache(oc, 0, 1, 1, 1, T, d)
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        cg.kv_encode(0, x, Gd, shp, oc, k, err_flag=err)
        torch.cuda.synchronize()
        assert bool(int(err.item()) & cg.CG_FLAG_NONFINITE) == (x is spoilt)
        out.append((k.codes.view(T, d // n, -1), k.side.view(T, d // n, -1)))
    keep = torch.ones((T, d // n), dtype=torch.bool, device="cuda")
    keep[33, : g // n] = False
    for a, b in zip(*out):
        assert torch.equal(a[keep], b[keep])
