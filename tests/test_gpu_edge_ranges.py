"""Kernels that cut the edge list into ranges, at the sizes where a range's ends
fall inside hub rows, on row ends and among empty rows: the row of every
position (256 or 1024 rows and positions per wavefront, in merged order) and the
gradient of materialized messages (a row's first 256 edges or more, then parts
of that many).  Integers and copies are exact; the mean's quotient is correctly
rounded."""
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


def degrees(name):
    rng = np.random.default_rng(3)
    if name == "one row":
        return np.array([5000])
    if name == "one edge":
        return np.array([0, 0, 1, 0])
    if name == "range ends":  # rows that end on and next to multiples of 1024 and 256
        return np.array([1024, 1023, 1, 1025, 255, 256, 257, 0, 511, 1, 2048, 3])
    if name == "hub among empty rows":
        d = np.zeros(200_000, dtype=np.int64)
        d[[7, 100_000, 100_001, 199_999]] = [3, 40_000, 1, 5]
        return d
    if name == "trailing empty rows":
        return np.concatenate([np.full(300, 4), np.zeros(70_000, dtype=np.int64)])
    if name == "more rows than edges":
        return np.bincount(rng.integers(0, 100_000, 5000), minlength=100_000)
    if name == "degree one":
        return np.ones(3000, dtype=np.int64)
    return np.minimum(rng.zipf(1.3, 20_000), 30_000)  # power law


NAMES = ["one row", "one edge", "range ends", "hub among empty rows", "trailing empty rows",
         "degree one", "power law", "more rows than edges"]


def rowptr_of(deg, dtype):
    rp = np.concatenate([[0], np.cumsum(deg)])
    return rp, torch.from_numpy(rp).to(DEV, dtype)


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("itype", [torch.int32, torch.int64])
@pytest.mark.parametrize("shift", [0, 1])  # ids stored four at a time, or one
def test_row_of_every_position(name, itype, shift):
    deg = degrees(name)
    rp, rp_d = rowptr_of(deg, itype)
    E, N = int(rp[-1]), len(deg)
    buf = torch.full((E + shift + 8,), -7, dtype=torch.int32, device=DEV)
    mp.mp_csr_rows(rp_d, mp.MP_I32 if itype == torch.int32 else mp.MP_I64, N, E,
                   buf[shift:shift + E])
    got = buf.cpu().numpy()
    assert np.array_equal(got[shift:shift + E], np.repeat(np.arange(N), deg))
    assert (got[:shift] == -7).all() and (got[shift + E:] == -7).all()


@pytest.mark.parametrize("name", ["range ends", "power law", "more rows than edges", "one row"])
@pytest.mark.parametrize("itype", [torch.int32, torch.int64])
@pytest.mark.parametrize("shift", [0, 1])
def test_row_of_every_position_in_long_ranges(name, itype, shift):
    """1024 rows and positions a wavefront, from 4M of them on."""
    deg = degrees(name)
    deg = np.tile(deg, -(-((1 << 22) + 5) // (len(deg) + int(deg.sum()))))
    rp, rp_d = rowptr_of(deg, itype)
    E, N = int(rp[-1]), len(deg)
    buf = torch.full((E + shift + 8,), -7, dtype=torch.int32, device=DEV)
    mp.mp_csr_rows(rp_d, mp.MP_I32 if itype == torch.int32 else mp.MP_I64, N, E,
                   buf[shift:shift + E])
    got = buf.cpu().numpy()
    assert np.array_equal(got[shift:shift + E], np.repeat(np.arange(N), deg))
    assert (got[:shift] == -7).all() and (got[shift + E:] == -7).all()


@pytest.mark.parametrize("e", [20_000, (1 << 22) + 5])  # short and long ranges
def test_row_of_every_position_ends_on_a_decreasing_rowptr(e):
    """A rowptr that jumps up and down (a caller's broken promise): the ids are
    unspecified but lie below the number of rows, and the call finishes."""
    n = 3000
    rp = np.where(np.arange(n + 1) % 64 == 0, 0, e)
    rp[-1] = e
    col = torch.zeros(e, dtype=torch.int32, device=DEV)  # one source row: positions stay in order
    _, colT, posT, _ = mp.csr_transpose(torch.from_numpy(rp).to(DEV, torch.int32), col, 1)
    rows = colT.cpu().numpy()
    assert rows.min() >= 0 and rows.max() < n
    assert np.array_equal(posT.cpu().numpy(), np.arange(e))


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("reduce", ["sum", "mean", "max"])
@pytest.mark.parametrize("F", [8, 7])
def test_message_gradient(name, reduce, F):
    deg = degrees(name)
    rp, rp_d = rowptr_of(deg, torch.int64 if F == 7 else torch.int32)
    E, N = int(rp[-1]), len(deg)
    rng = np.random.default_rng(5)
    g = rng.standard_normal((N, F)).astype(np.float32)
    row = np.repeat(np.arange(N), deg)
    arg = None
    want = g[row]
    if reduce == "mean":
        want = (want.astype(np.float64) / deg[row][:, None]).astype(np.float32)
    if reduce == "max":
        arg = np.where(deg[:, None] > 0,
                       rp[:-1, None] + rng.integers(0, 1 << 30, (N, F)) % np.maximum(deg, 1)[:, None],
                       -1).astype(np.int32)
        want = np.where(arg[row] == np.arange(E)[:, None], want, np.float32(0))
    got = mp.message_backward(rp_d, torch.from_numpy(g).to(DEV),
                              {"sum": mp.MP_SUM, "mean": mp.MP_MEAN, "max": mp.MP_MAX}[reduce], E=E,
                              argout=None if arg is None else torch.from_numpy(arg).to(DEV))
    assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("e", [(1 << 20) - 1, 1 << 20, (1 << 24) + 5])
@pytest.mark.parametrize("F,reduce", [(7, "max"), (8, "sum"), (130, "sum")])
def test_message_gradient_in_long_parts(e, F, reduce):
    """256 edges a part below 2^20 edges, then 256 to 4096 by the width, and four
    times that beyond 2^24: rows that end on and next to multiples of those, and
    a hub over several parts."""
    if e * F > 1 << 28:
        F = 5
    d = np.concatenate([degrees("range ends"), [4095, 4096, 4097, 16_383, 16_384, 16_385, 0, 1]])
    deg = np.tile(d, (e - 70_000) // int(d.sum()))
    deg = np.append(deg, e - int(deg.sum()))
    rp, rp_d = rowptr_of(deg, torch.int32)
    N = len(deg)
    g = torch.randn(N, F, device=DEV)
    row = torch.repeat_interleave(torch.arange(N, device=DEV), torch.from_numpy(deg).to(DEV))
    arg = None
    if reduce == "max":
        deg_d = torch.from_numpy(deg).to(DEV)[:, None]
        arg = (rp_d[:-1, None] + torch.randint(0, 1 << 30, (N, F), device=DEV) % deg_d.clamp(min=1)).int()
        arg = torch.where(deg_d > 0, arg, -1).int()
    got = mp.message_backward(rp_d, g, mp.MP_SUM if reduce == "sum" else mp.MP_MAX, E=e, argout=arg)
    want = g[row]
    if reduce == "max":
        want *= arg[row] == torch.arange(e, device=DEV)[:, None]
    assert torch.equal(got, want)


@pytest.mark.parametrize("F", [64, 70])  # one and two 64-feature tiles
@pytest.mark.parametrize("opts", [(1, 1, 1), (4, 9, 7)])  # and chunks that do not divide the rows
def test_hub_rows_of_few_and_many_chunks(F, opts):
    """Hub rows of one edge per chunk, their chunk counts on both sides of the
    16 (statistics) and 32 that one wavefront combines and at the 2048 of the
    longest rows; and rows cut evenly into chunks of up to seven edges.
    Integer features: sums are exact in any order."""
    deg = np.array([2, 16, 17, 32, 33, 63, 64, 65, 0, 66, 512, 2047, 2048, 5000, 1, 130])
    rp, rp_d = rowptr_of(deg, torch.int32)
    E, N = int(rp[-1]), len(deg)
    rng = np.random.default_rng(9)
    x = rng.integers(-8, 9, (40, F)).astype(np.float32)
    col = rng.integers(0, 40, E).astype(np.int32)
    plan = mp.Plan(rp_d, E, F, torch.float32, opts=opts)
    out, mx, arg = mp.spmm(rp_d, torch.from_numpy(col).to(DEV), torch.from_numpy(x).to(DEV),
                           mp.MP_SUM | mp.MP_MAX, plan=plan)
    multi = mp.spmm_multi(rp_d, torch.from_numpy(col).to(DEV), torch.from_numpy(x).to(DEV),
                          ["sum", "min", "max", "var"], plan=plan)
    m = x[col]
    for v in range(N):
        rows = m[rp[v]:rp[v + 1]]
        if not len(rows):
            assert (out[v] == 0).all() and (arg[v] == -1).all() and (multi["argmin"][v] == -1).all()
            continue
        assert np.array_equal(out[v].cpu().numpy(), rows.sum(0))
        assert np.array_equal(multi["sum"][v].cpu().numpy(), rows.sum(0))
        for got, at, first in ((mx, arg, rows.argmax(0)), (multi["max"], multi["argmax"], rows.argmax(0)),
                               (multi["min"], multi["argmin"], rows.argmin(0))):
            assert np.array_equal(at[v].cpu().numpy(), rp[v] + first)
            assert np.array_equal(got[v].cpu().numpy(), rows[first, np.arange(F)])
        var = rows.astype(np.float64).var(0)
        assert np.allclose(multi["var"][v].cpu().numpy(), var, rtol=1e-5, atol=0)
