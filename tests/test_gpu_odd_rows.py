"""Rows that no vector width divides, or that start anywhere, are cut into
chunks of four elements whose last begins inside the one before it: every
aggregation, the per-edge dots and the gradients at feature counts around the
edges of a chunk and of a 64-lane tile, tables and outputs shifted off their
alignment, strided tables, and degrees on both sides of the rule's.  Integer
features, weights and gradients: sums and dots are exact in any order."""
import sys

import numpy as np
import pytest
import torch

import paper_2507_16991_amd as mp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(autouse=True)
def _announce(request):
    sys.stderr.write(f"\n[gpu-case] {request.node.nodeid}\n")
    sys.stderr.flush()
    yield
    torch.cuda.synchronize()


def shifted(a, dtype, shift, ld=None):
    """a on the GPU, starting `shift` elements past an aligned address, rows
    ld elements apart, with NaN (or -1) all around."""
    n, f = a.shape
    ld = f if ld is None else ld
    fill = -1 if dtype == torch.int32 else float("nan")
    buf = torch.full((shift + n * ld + 16,), fill, dtype=dtype, device=DEV)
    view = buf[shift:shift + n * ld].view(n, ld)[:, :f]
    view.copy_(torch.from_numpy(a).to(dtype))
    return view, buf


@pytest.mark.parametrize("F", [4, 5, 7, 29, 31, 33, 50, 75, 253, 255, 257, 261])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("deg_hi", [9, 80, -24, -64])  # below 0: no row is longer, else one hub
@pytest.mark.parametrize("shift,pad", [(0, 0), (1, 0), (0, 3)])
def test_all_outputs(F, dtype, deg_hi, shift, pad):
    rng = np.random.default_rng(F + abs(deg_hi))
    n_dst, n_src = 61, 40
    deg = rng.integers(0, abs(deg_hi), n_dst)
    deg[[3, 7]] = [0, 700 if deg_hi > 0 else -deg_hi - 1]  # an empty row and a hub
    rp = np.concatenate([[0], np.cumsum(deg)])
    E = int(rp[-1])
    row = np.repeat(np.arange(n_dst), deg)
    col = rng.integers(0, n_src, E).astype(np.int32)
    x = rng.integers(-8, 9, (n_src, F)).astype(np.float32)
    w = rng.integers(-3, 4, E).astype(np.float32)
    g = rng.integers(-4, 5, (n_dst, F)).astype(np.float32)
    rp_d = torch.from_numpy(rp).to(DEV, torch.int32)
    col_d, w_d = torch.from_numpy(col).to(DEV), torch.from_numpy(w).to(DEV)
    x_d, _ = shifted(x, dtype, shift, F + pad if pad else None)
    zero = np.zeros((n_dst, F), np.float32)
    plan = mp.Plan(rp_d, E, F, dtype, opts=(0, 256, 64))
    for weight, wd in ((None, None), (w, w_d)):
        m = x[col] if weight is None else x[col] * weight[:, None]
        total = np.zeros((n_dst, F), np.float32)
        np.add.at(total, row, m)
        first = np.array([rp[v] + m[rp[v]:rp[v + 1]].argmax(0) if deg[v] else np.full(F, -1)
                          for v in range(n_dst)])
        best = np.where(first >= 0, m[np.maximum(first, 0), np.arange(F)], 0)
        for p in (plan, None):
            out, obuf = shifted(zero, torch.float32, shift)
            mx, mbuf = shifted(zero, torch.float32, shift)
            arg, abuf = shifted(zero, torch.int32, shift)
            mp.spmm(rp_d, col_d, x_d, mp.MP_SUM | mp.MP_MAX, w=wd, plan=p, out=out, out_max=mx,
                    argout=arg)
            assert np.array_equal(out.cpu().numpy(), total)
            assert np.array_equal(mx.cpu().numpy(), best)
            assert np.array_equal(arg.cpu().numpy(), first)
            for b in (obuf, mbuf):  # nothing written outside the rows
                assert torch.isnan(b[:shift]).all() and torch.isnan(b[shift + n_dst * F:]).all()
            assert (abuf[:shift] == -1).all() and (abuf[shift + n_dst * F:] == -1).all()
            only, _, _ = mp.spmm(rp_d, col_d, x_d, mp.MP_SUM, w=wd, plan=p)
            assert np.array_equal(only.cpu().numpy(), total)
            multi = mp.spmm_multi(rp_d, col_d, x_d, ["sum", "max", "min"], w=wd, plan=p)
            assert np.array_equal(multi["sum"].cpu().numpy(), total)
            assert np.array_equal(multi["max"].cpu().numpy(), best)
            assert np.array_equal(multi["argmax"].cpu().numpy(), first)
    if pad:
        return
    # gradients, and the dot of every edge
    g_d, _ = shifted(g, torch.float32, shift)
    dots = (g[row] * x[col]).sum(1)
    gw = mp.spmm_backward_w(rp_d, col_d, x_d, g_d, mp.MP_SUM)
    assert np.array_equal(gw.cpu().numpy(), dots)
    ed = mp.edge_dot(torch.from_numpy(g[row]).to(DEV), x_d, bidx=col_d)
    assert np.array_equal(ed.cpu().numpy(), dots)
    _, _, arg = mp.spmm(rp_d, col_d, x_d, mp.MP_MAX, plan=plan)
    hit = arg.cpu().numpy()[row] == np.arange(E)[:, None]
    gwm = mp.spmm_backward_w(rp_d, col_d, x_d, g_d, mp.MP_MAX, argout=arg)
    assert np.array_equal(gwm.cpu().numpy(), (g[row] * x[col] * hit).sum(1))
    rpT, colT, posT, _ = mp.csr_transpose(rp_d, col_d, n_src)
    for reduce, kept in ((mp.MP_SUM, 1.0), (mp.MP_MAX, hit)):
        want = np.zeros((n_src, F), np.float32)
        np.add.at(want, col, g[row] * kept)
        gx = mp.spmm_backward_x(rpT, colT, g_d, reduce, posT=posT, rowptr=rp_d, argout=arg)
        assert np.array_equal(gx.cpu().numpy(), want)


@pytest.mark.parametrize("F", [5, 6, 7, 75])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("back", [2, 3, 4])  # the infinite feature: F - back
@pytest.mark.parametrize("inf", [float("inf"), float("-inf")])
def test_infinite_features_in_two_chunks(F, dtype, back, inf):
    """An infinite feature in the elements that a row's last chunk shares with
    the one before it counts once, in the dots of sum, mean and max and in
    edge_dot.  All other features and all gradients are small positive integers,
    so that a dot is that infinity, or exact."""
    rng = np.random.default_rng(F + back)
    n_dst, n_src, deg = 20, 15, 40
    rp = np.arange(n_dst + 1) * deg
    E = n_dst * deg
    row = np.repeat(np.arange(n_dst), deg)
    col = rng.integers(0, n_src, E).astype(np.int32)
    x = rng.integers(1, 9, (n_src, F)).astype(np.float32)
    x[::2, F - back] = inf
    g = rng.integers(1, 5, (n_dst, F)).astype(np.float32)
    rp_d = torch.from_numpy(rp).to(DEV, torch.int32)
    col_d, x_d, g_d = torch.from_numpy(col).to(DEV), torch.from_numpy(x).to(DEV, dtype), torch.from_numpy(g).to(DEV)
    dots = (g[row] * x[col]).sum(1)
    assert np.isinf(dots).any() and not np.isnan(dots).any()
    assert np.array_equal(mp.spmm_backward_w(rp_d, col_d, x_d, g_d, mp.MP_SUM).cpu().numpy(), dots)
    mean = mp.spmm_backward_w(rp_d, col_d, x_d, g_d, mp.MP_MEAN).cpu().numpy()
    assert np.array_equal(mean, (dots / np.float32(deg)).astype(np.float32))
    ed = mp.edge_dot(torch.from_numpy(g[row]).to(DEV, dtype), x_d, bidx=col_d)
    assert np.array_equal(ed.cpu().numpy(), dots)
    arg = (rp[:-1, None] + rng.integers(0, deg, (n_dst, F))).astype(np.int32)
    arg[:, F - back] = rp[:-1] + np.array([np.isinf(x[col[rp[v]:rp[v + 1]], F - back]).argmax()
                                           for v in range(n_dst)])
    hit = arg[row] == np.arange(E)[:, None]
    won = np.where(hit, g[row] * np.where(hit, x[col], 0), 0).sum(1)
    got = mp.spmm_backward_w(rp_d, col_d, x_d, g_d, mp.MP_MAX, argout=torch.from_numpy(arg).to(DEV))
    assert np.isinf(won).any() and np.array_equal(got.cpu().numpy(), won.astype(np.float32))
