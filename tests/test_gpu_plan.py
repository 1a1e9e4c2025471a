"""The plan's counting sort at the sizes where its launches change: one
workgroup up to 16384 rows, tiles of 4096 rows up to 4M, of 16384 beyond.
Every row must be aggregated exactly once, whatever its class: integer
features, so that sums are exact, against numpy's segment sums; and the hub
rows' chunks are counted through the workspace they need."""
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


@pytest.mark.parametrize("N", [1, 63, 1024, 1025, 16383, 16384, 16385, 20480, 300_001, 4_194_304,
                               4_194_305])
@pytest.mark.parametrize("itype", [torch.int32, torch.int64])
def test_every_row_once(N, itype):
    F = 4
    rng = np.random.default_rng(N)
    deg = np.minimum(rng.zipf(1.6 if N < 1_000_000 else 2.5, N) - 1, 3000)
    if N > 1000:
        deg[[0, N // 2, N - 1]] = [2500, 700, 4100]
    rp = np.concatenate([[0], np.cumsum(deg)])
    E = int(rp[-1])
    x = rng.integers(-3, 4, (64, F)).astype(np.float32)
    col = rng.integers(0, 64, E).astype(np.int32)
    rp_d = torch.from_numpy(rp).to(DEV, itype)
    small, hub, chunk = 32, 200, 64
    plan = mp.Plan(rp_d, E, F, opts=(small, hub, chunk))
    hubs = deg[deg > hub]
    size = np.maximum((hubs + 2047) // 2048, chunk)
    chunks = int(((hubs + size - 1) // size).sum())
    ws = plan.workspace(mp.MP_SUM)
    assert (0 if ws is None else ws.numel()) == (chunks * F * 4 + 255) // 256 * 256
    col_d = torch.from_numpy(col if E else np.zeros(1, np.int32)).to(DEV)
    out = torch.full((N, F), float("nan"), device=DEV)
    mp.spmm(rp_d, col_d, torch.from_numpy(x).to(DEV), mp.MP_SUM, plan=plan, out=out)
    sums = np.concatenate([np.zeros((1, F)), np.cumsum(x[col], axis=0, dtype=np.float64)])
    assert np.array_equal(out.cpu().numpy(), (sums[rp[1:]] - sums[rp[:-1]]).astype(np.float32))


@pytest.mark.parametrize("rows,deg,F", [(128, 2048, 2048), (1024, 257, 2048), (96, 1500, 4096),
                                        (128, 1024, 700)])
def test_short_chunks_fit_the_static_scratch(rows, deg, F):
    """Hub chunks are shortened on small graphs only as far as the partials of
    sum and max together stay within mp_spmm_noalloc's scratch."""
    E = rows * deg
    rp = torch.arange(rows + 1, dtype=torch.int32, device=DEV) * deg
    plan = mp.Plan(rp, E, F)
    need = mp.mp_spmm_workspace(plan.handle, mp.MP_SUM | mp.MP_MAX)
    assert 0 < need <= 64 << 20
    rng = np.random.default_rng(F)
    x = torch.from_numpy(rng.integers(-3, 4, (16, F)).astype(np.float32)).to(DEV)
    col = torch.from_numpy(rng.integers(0, 16, E).astype(np.int32)).to(DEV)
    out = torch.full((rows, F), float("nan"), device=DEV)
    mx = torch.full((rows, F), float("nan"), device=DEV)
    arg = torch.full((rows, F), -2, dtype=torch.int32, device=DEV)
    mp.mp_spmm_noalloc(plan.handle, rp, mp.MP_I32, col, None, x, mp.MP_F32, 16, rows, F, F,
                       mp.MP_SUM | mp.MP_MAX, out, mp.MP_F32, mx, mp.MP_F32, arg)
    counts = np.stack([np.bincount(c, minlength=16) for c in col.cpu().numpy().reshape(rows, deg)])
    xs = x.cpu().numpy().astype(np.float64)
    assert np.array_equal(out.cpu().numpy(), (counts @ xs).astype(np.float32))
    present = np.where(counts[:, :, None] > 0, xs[None], -np.inf)
    assert np.array_equal(mx.cpu().numpy(), present.max(1).astype(np.float32))


@pytest.mark.parametrize("N", [2000, 20_000])  # one launch, three
@pytest.mark.parametrize("longest", [1024, 1025])  # 32 wavefront steps of 32 edges, and more
def test_short_chunks_only_beside_long_rows(N, longest):
    """Rows of 16 to 32 steps on a small graph are cut into chunks of 8 steps
    only where there is a longer row, which is cut anyway."""
    F = 64
    deg = np.full(N, 4)
    deg[[5, N // 2, N - 1]] = [700, 513, 512]
    deg[77] = longest
    rp = np.concatenate([[0], np.cumsum(deg)])
    E = int(rp[-1])
    rng = np.random.default_rng(N)
    x = rng.integers(-3, 4, (50, F)).astype(np.float32)
    col = rng.integers(0, 50, E).astype(np.int32)
    rp_d = torch.from_numpy(rp).to(DEV, torch.int32)
    plan = mp.Plan(rp_d, E, F)
    chunks = 0 if longest <= 1024 else 3 + 3 + 5  # of 700, 513 and 1025 edges by 256
    assert mp.mp_spmm_workspace(plan.handle, mp.MP_SUM) == chunks * F * 4
    out, _, _ = mp.spmm(rp_d, torch.from_numpy(col).to(DEV), torch.from_numpy(x).to(DEV), mp.MP_SUM,
                        plan=plan)
    sums = np.concatenate([np.zeros((1, F)), np.cumsum(x[col], axis=0, dtype=np.float64)])
    assert np.array_equal(out.cpu().numpy(), (sums[rp[1:]] - sums[rp[:-1]]).astype(np.float32))
