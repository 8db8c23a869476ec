"""Paged encode on the matrix cores (bf16, head dimension 128, block-uniform): every width and block
against the oracle in one-tile and multi-tile geometry, bit for bit against the contiguous encoder where
that takes three gauge planes too, and pages outside the pool."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2607_20538_amd import codec as cg
from paper_2607_20538_amd import synth

from _parity import cache_to_host, check_fused_codes, to_cg, x_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cg.lib()


def _setup(g, T, P, L=1, B=2, H=2, seed=5):
    G = O.gauge_make(O.GAUGE_HAAR, L, H, 128, g, seed=23)
    shp = cg.shape(L, H, 128, g)
    Gd = cg.alloc_gauge(shp)
    cg.gauge_make(cg.GAUGE_USER, shp, params=G, G_host=None, G_dev=Gd)
    w = synth.Workload("pe", L=L, B=B, H=H, T=T, d=128, dtype="bf16", g=g, backend="bu", bits=4, data_seed=0xE9)
    maxp = (T + P - 1) // P + 1
    order = np.random.default_rng(seed).permutation(B * maxp + 2).astype(np.int32)[: B * maxp].reshape(B, maxp)
    return G, Gd, shp, w, order, B * maxp + 2, maxp


def _rows(pool, oc, s, table, P):
    """The pool's rows in position order, as a contiguous cache."""
    host = cache_to_host(pool, oc, s)
    return {k: None if v is None else np.stack(
        [np.concatenate([v[:, p] for p in table[b]], axis=2) for b in range(table.shape[0])], axis=1)
        for k, v in host.items()}


@pytest.mark.parametrize("tiles", [None, 7])
@pytest.mark.parametrize("g,bits,n", [(128, 4, 64), (128, 2, 16), (64, 3, 32), (32, 3, 64), (8, 4, 32), (16, 6, 64),
                                      (128, 8, 16), (128, 6, 32)])
def test_paged_encode_over_widths(g, bits, n, tiles, monkeypatch):
    monkeypatch.delenv("CG_KERNELS", raising=False)
    monkeypatch.delenv("CG_TILES_PER_WG", raising=False)
    if tiles:
        monkeypatch.setenv("CG_TILES_PER_WG", str(tiles))
    P, T = 64, 32 * 17 + 13
    oc = O.Codec(backend=O.BLOCK_UNIFORM, bits=bits, block_c=n)
    G, Gd, shp, w, table, pool_pages, maxp = _setup(g, T, P)
    pt_pages = torch.from_numpy(table).cuda()
    pt = cg.page_table(pt_pages, P)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    for s in (0, 1):
        X = synth.kv_tensor(w, s)
        pool = cg.Cache(to_cg(oc), s, w.L, pool_pages, w.H, P, 128)
        cg.kv_encode_paged(s, x_dev(X), pt, Gd, shp, to_cg(oc), pool, 0, err)
        cont = cg.Cache(to_cg(oc), s, w.L, w.B, w.H, maxp * P, 128)
        cg.kv_encode(s, x_dev(X), Gd, shp, to_cg(oc), cont, 0, err)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        got, want = _rows(pool, oc, s, table, P), cache_to_host(cont, oc, s)
        if bits >= 6:
            for key in ("codes", "side"):
                np.testing.assert_array_equal(got[key], want[key], err_msg=key)   # rows past T stay zero
        else:
            assert not got["codes"][:, :, :, T:].any()
        ref, _ = O.kv_encode(oc, s, X, G, T_cap=maxp * P)
        z, _ = O.kv_encode(O.Codec(backend=O.PASSTHROUGH), s, X, G, T_cap=maxp * P)
        check_fused_codes(got, ref, z["codes"], oc, s, 128, T)
        # the rest of a prompt, from an offset inside a page
        part = cg.Cache(to_cg(oc), s, w.L, pool_pages, w.H, P, 128)
        cg.kv_encode_paged(s, x_dev(X)[:, :, :, :96], pt, Gd, shp, to_cg(oc), part, 0, err)
        cg.kv_encode_paged(s, x_dev(X)[:, :, :, 96:], pt, Gd, shp, to_cg(oc), part, 96, err)
        torch.cuda.synchronize()
        assert torch.equal(part.codes, pool.codes) and torch.equal(part.side, pool.side)


@pytest.mark.parametrize("tiles", [None, 9])
def test_pages_outside_the_pool_are_skipped(tiles, monkeypatch):
    """Flagged; the page's tiles write nothing (a NaN in them raises no flag of its own), the others do."""
    monkeypatch.delenv("CG_KERNELS", raising=False)
    monkeypatch.delenv("CG_TILES_PER_WG", raising=False)
    if tiles:
        monkeypatch.setenv("CG_TILES_PER_WG", str(tiles))
    P, T, g = 64, 320, 128
    oc = cg.Codec(cg.BLOCK_UNIFORM, 4, 64)
    _, Gd, shp, w, table, pool_pages, maxp = _setup(g, T, P)
    X = x_dev(synth.kv_tensor(w, 1))
    good = torch.from_numpy(table).cuda()
    bad_table = table.copy()
    bad_table[0, 1], bad_table[1, 3] = pool_pages, -1
    bad = torch.from_numpy(bad_table).cuda()
    pools, errs = [], []
    for pages in (good, bad):
        x = X.clone()
        if pages is bad:
            x[0, 0, :, P + 5, 3] = float("nan")
        pool = cg.Cache(oc, 1, w.L, pool_pages, w.H, P, 128)
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        cg.kv_encode_paged(1, x, cg.page_table(pages, P), Gd, shp, oc, pool, 0, err)
        torch.cuda.synchronize()
        pools.append(pool)
        errs.append(int(err.item()))
    assert errs == [0, cg.CG_FLAG_POS_RANGE]
    a, b = (p.codes.view(w.L, pool_pages, -1).clone() for p in pools)
    for r, i in ((0, 1), (1, 3)):
        assert not b[:, int(table[r, i])].any()
        a[:, int(table[r, i])] = 0
    assert torch.equal(a, b)


def _paged(X, table, P, Gd, shp, oc, pool_pages, w):
    pool = cg.Cache(oc, 0, w.L, pool_pages, w.H, P, 128)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    pt = torch.from_numpy(table).cuda()
    cg.kv_encode_paged(0, X, cg.page_table(pt, P), Gd, shp, oc, pool, 0, err)
    torch.cuda.synchronize()
    return pool.codes.clone(), pool.side.clone(), int(err.item())


BAD = [float("nan"), float("inf"), float("-inf"), "two"]


def _spoil(X, g, bad):
    """Three tokens with non-finite channels: one channel, one whole group, one whole token."""
    X = X.clone()
    v = float("inf") if bad == "two" else bad
    X[0, 0, 0, 33, g // 2] = v
    X[0, 1, 1, 70, 64:64 + g] = v
    X[0, 1, 0, 5] = v
    if bad == "two":                          # infinities of both signs in one group
        X[0, 0, 0, 33, g // 2 + 1] = -v
    return X


@pytest.mark.parametrize("tiles", [None, 4])
@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("g,bits,n", [(8, 4, 64), (16, 3, 32), (16, 8, 16), (32, 2, 64), (64, 6, 32), (128, 4, 64)])
def test_non_finite_tokens_as_the_general_kernel_codes_them(g, bits, n, bad, tiles, monkeypatch):
    """With the identity gauge z = x on both kernels, so every code and side word is the same, also of the
    blocks and groups that hold a non-finite channel (a side word that is no number: of either sign), and
    the flags are."""
    monkeypatch.delenv("CG_KERNELS", raising=False)
    monkeypatch.delenv("CG_TILES_PER_WG", raising=False)
    if tiles:
        monkeypatch.setenv("CG_TILES_PER_WG", str(tiles))
    P, T = 64, 160
    oc = cg.Codec(cg.BLOCK_UNIFORM, bits, n)
    _, _, _, w, table, pool_pages, _ = _setup(g, T, P)
    shp = cg.shape(w.L, w.H, 128, g)
    Gd = cg.alloc_gauge(shp)
    cg.gauge_make(cg.GAUGE_IDENTITY, shp, G_host=None, G_dev=Gd)
    # binary32 tokens take the general kernel's binary32 chain
    X = _spoil(x_dev(synth.kv_tensor(w, 0)), g, bad)
    want = _paged(X.float(), table, P, Gd, shp, oc, pool_pages, w)
    got = _paged(X, table, P, Gd, shp, oc, pool_pages, w)
    assert want[2] & cg.CG_FLAG_NONFINITE and got[2] == want[2]
    assert torch.equal(got[0], want[0])
    assert torch.allclose(got[1].view(torch.float16), want[1].view(torch.float16), rtol=0, atol=0, equal_nan=True)


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("g", [8, 16, 32])
def test_non_finite_channels_leave_other_groups_alone(g, bad):
    """Blocks of other groups keep the bytes that they have beside finite tokens."""
    P, T, n = 64, 160, 16
    oc = cg.Codec(cg.BLOCK_UNIFORM, 4, n)
    _, Gd, shp, w, table, pool_pages, _ = _setup(g, T, P)
    X = x_dev(synth.kv_tensor(w, 0))
    clean = _paged(X, table, P, Gd, shp, oc, pool_pages, w)
    got = _paged(_spoil(X, g, bad), table, P, Gd, shp, oc, pool_pages, w)
    assert clean[2] == 0 and got[2] & cg.CG_FLAG_NONFINITE
    keep = torch.ones((pool_pages, w.H, P, 128 // n), dtype=torch.bool, device="cuda")
    m = max(g, n)
    keep[int(table[0, 0]), 0, 33, : m // n] = False
    keep[int(table[1, 1]), 1, 70 - P, 64 // n:(64 + m) // n] = False
    keep[int(table[1, 0]), 0, 5] = False
    for a, b in zip(got[:2], clean[:2]):
        a, b = (t[: keep.numel() * (t.numel() // keep.numel())].view(*keep.shape, -1) for t in (a, b))
        assert torch.equal(a[keep], b[keep])
