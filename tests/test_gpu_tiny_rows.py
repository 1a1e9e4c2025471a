"""Rows of at most seven edges: with the small rows while they make up to 8192
groups of a wavefront's rows, in their own kernel beyond, at the group counts
on both sides of that; and relations listed by one launch, more of them than
one launch takes.  Integer features: exact."""
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


@pytest.mark.parametrize("n", [16_384, 16_385, 16_401])  # two rows a wavefront at F = 128
@pytest.mark.parametrize("weighted", [False, True])
def test_tiny_rows(n, weighted):
    F = 128
    rng = np.random.default_rng(n)
    deg = rng.integers(0, 8, n)
    rp = np.concatenate([[0], np.cumsum(deg)])
    E = int(rp[-1])
    row = np.repeat(np.arange(n), deg)
    col = rng.integers(0, 500, E).astype(np.int32)
    x = rng.integers(-8, 9, (500, F)).astype(np.float32)
    w = rng.integers(-3, 4, E).astype(np.float32) if weighted else None
    m = x[col] if w is None else x[col] * w[:, None]
    total = np.zeros((n, F), np.float32)
    np.add.at(total, row, m)
    best = np.full((n, F), -np.inf, np.float32)
    np.maximum.at(best, row, m)
    rp_d, col_d = torch.from_numpy(rp).to(DEV, torch.int32), torch.from_numpy(col).to(DEV)
    x_d = torch.from_numpy(x).to(DEV)
    w_d = None if w is None else torch.from_numpy(w).to(DEV)
    plan = mp.Plan(rp_d, E, F)
    out, mx, arg = mp.spmm(rp_d, col_d, x_d, mp.MP_SUM | mp.MP_MAX, w=w_d, plan=plan)
    multi = mp.spmm_multi(rp_d, col_d, x_d, ["sum", "max"], w=w_d, plan=plan)
    some = deg > 0
    a = arg.cpu().numpy()
    for got, at in ((mx, a), (multi["max"], multi["argmax"].cpu().numpy())):
        assert np.array_equal(got.cpu().numpy(), np.where(some[:, None], best, 0))
        assert np.array_equal(at, a)
    assert (a[~some] == -1).all() and np.array_equal(m[a[some], np.arange(F)], best[some])
    assert np.array_equal(out.cpu().numpy(), total)
    assert np.array_equal(multi["sum"].cpu().numpy(), total)
    # gradient of max over a transpose whose rows are tiny: the same graph,
    # read as the transpose of another
    g = rng.integers(-4, 5, (500, F)).astype(np.float32)
    rp2, col2, pos2, w2 = mp.csr_transpose(rp_d, col_d, 500, val=w_d)
    rpT, colT, posT, wT = mp.csr_transpose(rp2, col2, n, val=w2)
    _, _, arg2 = mp.spmm(rp2, col2, torch.from_numpy(
        rng.integers(-8, 9, (n, F)).astype(np.float32)).to(DEV), mp.MP_MAX, w=w2)
    gx = mp.spmm_backward_x(rpT, colT, torch.from_numpy(g).to(DEV), mp.MP_MAX, posT=posT, wT=wT,
                            rowptr=rp2, argout=arg2, planT=mp.Plan(rpT, E, F))
    a2 = arg2.cpu().numpy()
    v, f = np.nonzero(a2 >= 0)
    want = np.zeros((n, F), np.float32)
    np.add.at(want, (col2.cpu().numpy()[a2[v, f]], f),
              g[v, f] * (1 if w is None else w2.cpu().numpy()[a2[v, f]]))
    assert np.array_equal(gx.cpu().numpy(), want)


@pytest.mark.parametrize("n_rel", [1, 32, 33, 70])
def test_many_relations(n_rel):
    rng = np.random.default_rng(n_rel)
    npt = [900, 1, 333]
    offs = np.concatenate([[0], np.cumsum(npt)])
    rels, src, dst = [], [], []
    for r in range(n_rel):
        s, d = int(rng.integers(0, 3)), int(rng.integers(0, 3))
        e = int(rng.integers(1, 5000)) if r % 5 else 2048 * (r % 3)  # whole and empty blocks
        e = max(e, 1) if r == 0 else e
        a, b = (rng.integers(0, npt[t], e).astype(np.int32) for t in (s, d))
        rels.append((s, d, torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV)))
        src.append(a + offs[s])
        dst.append(b + offs[d])
    src, dst = np.concatenate(src), np.concatenate(dst)
    rowptr, col = mp.hetero_build(npt, rels, mp.MP_ALL_TYPES)
    order = np.argsort(dst, kind="stable")
    assert np.array_equal(rowptr.cpu().numpy(), np.searchsorted(dst[order], np.arange(sum(npt) + 1)))
    assert np.array_equal(col.cpu().numpy(), src[order])
