"""COO->CSR and transpose where the sort's passes carry their elements in
different words: (key, src, id) packed whole, packed without the digit just
sorted by (up to exactly 64 bits), or too wide to pack; one to three passes,
digits of up to 8 and of 9 bits.  Destinations uniform, mostly one hub, already
sorted, and few (empty digit runs and rows).  Exact against numpy's stable
argsort."""
import sys

import numpy as np
import pytest
import torch

import paper_2507_16991_amd as mp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
BIG = 2 ** 31 - 1

# E, N, sources below: the words they give
SIZES = [
    (1, 1, 5), (64, 128, 9), (1_023, 129, 64), (1_025, 16_384, 300),  # one workgroup
    (5_000, 1, 17), (16_384, 1_000, BIG), (16_384, 16_384, BIG),
    (16_384, 16_385, BIG), (16_385, 16_384, BIG),  # just beyond
    (40_000, 300, BIG),        # one pass
    (16_385, 5_000, 1_000),    # two passes, packed whole (13 + 10 + 15 bits)
    (200_000, 200_000, 1 << 28),  # digits of 9 bits, whole (18 + 28 + 18 = 64)
    (40_000, 200_000, BIG),    # digits of 9 bits, too wide (18 + 31 + 16 = 65)
    (40_000, 1 << 22, BIG),    # three passes, one digit left out (15 + 31 + 16)
    (200_000, 1 << 22, BIG),   # the same, exactly 64 bits
    (300_000, 1 << 22, BIG),   # too wide by one bit
    (100_000, 20_000_000, 7),  # digits of 9 bits, three passes
    # edges enough for rowptr from the rows' starts rather than from the keys
    (300_000, 20_000, 1_000),      # two passes, packed whole (15 + 10 + 19)
    (300_000, 20_000, BIG),        # one digit left out (15 + 31 + 19)
    (1_100_000, 262_144, BIG),     # digits of 9 bits, too wide (18 + 31 + 21)
    (1_200_000, 270_000, 1 << 26),  # three passes, one digit left out (19 + 26 + 21)
    # ... and on both sides of where that begins
    (80_000, 20_000, 50), (80_001, 20_000, 50),
]


@pytest.fixture(autouse=True)
def _announce(request):
    sys.stderr.write(f"\n[gpu-case] {request.node.nodeid}\n")
    sys.stderr.flush()
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("E,N,src_max", SIZES)
@pytest.mark.parametrize("kind", ["uniform", "hub", "sorted", "few"])
def test_csr_and_transpose(E, N, src_max, kind):
    rng = np.random.default_rng(E + N)
    src = rng.integers(0, src_max, E).astype(np.int32)
    src[0] = src_max - 1  # every bit that the sources may have
    dst = rng.integers(0, N, E).astype(np.int32)
    if kind == "hub":
        dst[rng.random(E) < 0.7] = N - 1
    elif kind == "sorted":
        dst = np.sort(dst)
    elif kind == "few":
        dst = np.array([0, N // 3, N // 2, N - 1], dtype=np.int32)[dst % 4]
    order = np.argsort(dst, kind="stable")
    rp = np.searchsorted(dst[order], np.arange(N + 1))
    val = rng.standard_normal(E).astype(np.float32)
    src_d, dst_d = torch.from_numpy(src).to(DEV), torch.from_numpy(dst).to(DEV)
    for itype, perm, v in ((torch.int32, False, None), (torch.int64, True, None),
                           (torch.int32, True, torch.from_numpy(val).to(DEV))):
        rowptr, col, p, w = mp.coo_to_csr(src_d, dst_d, N, rowptr_dtype=itype, want_perm=perm, val=v)
        assert np.array_equal(rowptr.cpu().numpy(), rp)
        assert np.array_equal(col.cpu().numpy(), src[order])
        if perm:
            assert np.array_equal(p.cpu().numpy(), order)
        if v is not None:
            assert np.array_equal(w.cpu().numpy(), val[order])
    # the transpose of a CSR whose columns are these destinations
    n_rows = 777
    rp2 = np.sort(rng.integers(0, E + 1, n_rows + 1))
    rp2[0], rp2[-1] = 0, E
    row = np.repeat(np.arange(n_rows), np.diff(rp2))
    rpT, colT, posT, valT = mp.csr_transpose(torch.from_numpy(rp2).to(DEV, torch.int32), dst_d, N,
                                             val=torch.from_numpy(val).to(DEV))
    assert np.array_equal(rpT.cpu().numpy(), rp)
    assert np.array_equal(colT.cpu().numpy(), row[order])
    assert np.array_equal(posT.cpu().numpy(), order)
    assert np.array_equal(valT.cpu().numpy(), val[order])


@pytest.mark.parametrize("E,N", [(17_000_000, 8_388_607), (17_000_000, 8_388_608),  # 1024 and 1025 tiles
                                 (40_000_000, 18_000_000)])
@pytest.mark.parametrize("where", ["first rows", "last rows", "both ends"])
def test_rowptr_of_rows_beyond_the_last_edge(E, N, where):
    """All edges end in a few rows, and every other row's start is looked for in
    the tiles of rows after it."""
    dst = torch.randint(0, 5, (E,), dtype=torch.int32, device=DEV)
    if where == "last rows":
        dst += N - 5
    elif where == "both ends":
        dst[::2] += N - 5
    src = torch.zeros(E, dtype=torch.int32, device=DEV)
    rowptr, _, _, _ = mp.coo_to_csr(src, dst, N)
    want = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
    want[1:] = torch.bincount(dst, minlength=N).cumsum(0)
    assert torch.equal(rowptr.long(), want)
