"""Gradient of max by win records (graphs of at least 1.5M edges whose edges
win 0.6 to 3 features on average): records that hold no win, up to six, and
more (degree-one rows, whose edge wins every feature), hub rows on both sides,
empty rows, feature counts on both sides of a 64- and a 128-feature tile.  G
and the weights are small integers, so that every sum is exact in any order
and the gradient is compared bit for bit."""
import sys

import numpy as np
import pytest
import torch

import paper_2507_16991_amd as mp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
E_MIN = 3 << 19


@pytest.fixture(autouse=True)
def _announce(request):
    sys.stderr.write(f"\n[gpu-case] {request.node.nodeid}\n")
    sys.stderr.flush()
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("F,gdtype,weighted,plan,itype", [
    (7, torch.float32, False, "default", torch.int32),
    (64, torch.bfloat16, True, None, torch.int64),
    (100, torch.float32, True, "default", torch.int32),
    (128, torch.bfloat16, False, "hubs", torch.int32),
    (130, torch.float32, False, "default", torch.int64),
    (256, torch.float32, True, "hubs", torch.int32),
])
# bytes the workspace is off its alignment; or room for the win masks alone
@pytest.mark.parametrize("shift", [0, 4, "masks"])
def test_max_gradient_by_records(F, gdtype, weighted, plan, itype, shift):
    rng = np.random.default_rng(F)
    n_dst = 2 * E_MIN // F  # two wins an edge
    deg = np.minimum(rng.zipf(2.2, n_dst) - 1, 5_000)  # empty rows, degree one, hubs
    deg[:50] = 1
    deg[5] = 100_003
    missing = E_MIN + 77 - int(deg.sum())
    if missing > 0:
        deg += rng.multinomial(missing, np.full(n_dst, 1.0 / n_dst))
    E = int(deg.sum())
    assert E_MIN <= E and 0.6 * E <= n_dst * F <= 3 * E
    n_src = max(200, n_dst // 2)
    rp = np.concatenate([[0], np.cumsum(deg)])
    col = (n_src * rng.random(E) ** 3).astype(np.int32)  # some sources of many edges
    arg = np.where(deg[:, None] > 0, rp[:-1, None] + rng.integers(0, 1 << 40, (n_dst, F)) %
                   np.maximum(deg, 1)[:, None], -1).astype(np.int32)
    g = rng.integers(-8, 9, (n_dst, F)).astype(np.float32)
    w = rng.integers(-3, 4, E).astype(np.float32) if weighted else None
    want = np.zeros((n_src, F), dtype=np.float64)
    v, f = np.nonzero(arg >= 0)
    p = arg[v, f]
    np.add.at(want, (col[p], f), g[v, f] * (w[p] if weighted else 1.0))

    rp_d = torch.from_numpy(rp).to(DEV, itype)
    col_d = torch.from_numpy(col).to(DEV)
    rpT, colT, posT, wT = mp.csr_transpose(
        rp_d, col_d, n_src, val=None if w is None else torch.from_numpy(w).to(DEV))
    planT = None
    if plan:
        planT = mp.Plan(rpT, E, F, opts=(40, 200, 64) if plan == "hubs" else None)
    h = planT.handle if planT else None
    nb = mp.mp_spmm_backward_x_workspace(h, n_dst, E, F, mp.MP_MAX)
    part = mp.mp_spmm_backward_x_workspace(h, n_dst, E, F, mp.MP_SUM)
    assert nb == (part + 255) // 256 * 256 + (32 * E + 255) // 256 * 256  # records
    if shift == "masks":
        nb = (part + 255) // 256 * 256 + (E * ((F + 31) // 32) * 4 + 255) // 256 * 256
        shift = 0
    ws = torch.empty(nb + shift, dtype=torch.uint8, device=DEV)[shift:]
    g_d = torch.from_numpy(g).to(DEV, gdtype)
    out = torch.full((n_src, F), float("nan"), dtype=torch.float32, device=DEV)
    it = mp.MP_I32 if itype == torch.int32 else mp.MP_I64
    mp.mp_spmm_backward_x(h, rpT, mp.MP_I32, colT, posT, wT, rp_d, it, torch.from_numpy(arg).to(DEV),
                          g_d, mp.MP_F32 if gdtype == torch.float32 else mp.MP_BF16, n_dst, n_src,
                          E, F, mp.MP_MAX, out, mp.MP_F32, ws, nb)
    assert np.array_equal(out.cpu().numpy(), want.astype(np.float32))


def test_records_are_for_large_graphs_of_few_wins():
    size = lambda n, E, F: mp.mp_spmm_backward_x_workspace(None, n, E, F, mp.MP_MAX) // E
    E = E_MIN
    assert size(3 * E // 64, E, 64) == 32 and size(3 * E // 5 // 64 + 1, E, 64) == 32
    assert size(3 * E // 64 + 64, E, 64) == 8  # masks: two words per edge
    assert size(E // 2 // 64, E, 64) == 8 and size(3 * (E - 64) // 64, E - 64, 64) == 8
    assert size(E // 257, E, 257) == 36
    assert size(1 << 23, 1 << 28, 64) == 32 and size(1 << 23, (1 << 28) + 64, 64) == 8


@pytest.mark.parametrize("F", [7, 100])
def test_same_bits_wherever_the_workspace_begins(F):
    """The order of additions depends on the inputs and the workspace's size, not
    on its address: random G, whose sums differ with the order."""
    n, E = 2 * E_MIN // F, E_MIN
    gen = torch.Generator(device=DEV).manual_seed(F)
    dst = torch.randint(0, n, (E,), generator=gen, device=DEV, dtype=torch.int32)
    src = torch.randint(0, 500, (E,), generator=gen, device=DEV, dtype=torch.int32)
    rp, col, _, _ = mp.coo_to_csr(src, dst, n)
    x = torch.randn(500, F, generator=gen, device=DEV)
    g = torch.randn(n, F, generator=gen, device=DEV)
    _, _, arg = mp.spmm(rp, col, x, mp.MP_MAX)
    rpT, colT, posT, _ = mp.csr_transpose(rp, col, 500)
    plan = mp.Plan(rpT, E, F)
    nb = mp.mp_spmm_backward_x_workspace(plan.handle, n, E, F, mp.MP_MAX)
    got = []
    for shift in (0, 4, 12, 16):
        ws = torch.empty(nb + shift, dtype=torch.uint8, device=DEV)[shift:]
        out = torch.empty(500, F, device=DEV)
        mp.mp_spmm_backward_x(plan.handle, rpT, mp.MP_I32, colT, posT, None, rp, mp.MP_I32, arg, g,
                              mp.MP_F32, n, 500, E, F, mp.MP_MAX, out, mp.MP_F32, ws, nb)
        got.append(out)
    assert all(torch.equal(o, got[0]) for o in got[1:])


def test_masks_where_memory_does_not_hold_the_records(monkeypatch):
    """The binding's call goes on with the smaller workspace; integer G, so both
    ways give the same bits."""
    F, E = 40, E_MIN
    n = 2 * E // F
    dst = torch.randint(0, n, (E,), device=DEV, dtype=torch.int32)
    src = torch.randint(0, 300, (E,), device=DEV, dtype=torch.int32)
    rp, col, _, _ = mp.coo_to_csr(src, dst, n)
    _, _, arg = mp.spmm(rp, col, torch.randn(300, F, device=DEV), mp.MP_MAX)
    g = torch.randint(-8, 9, (n, F), device=DEV).float()
    rpT, colT, posT, _ = mp.csr_transpose(rp, col, 300)
    plan = mp.Plan(rpT, E, F)
    call = lambda: mp.spmm_backward_x(rpT, colT, g, mp.MP_MAX, posT=posT, rowptr=rp, argout=arg,
                                      planT=plan)
    want = call()
    full = mp.mp_spmm_backward_x_workspace(plan.handle, n, E, F, mp.MP_MAX)
    real, asked = mp._workspace, []

    def small_card(nbytes, device):
        asked.append(nbytes)
        if nbytes >= full:
            raise torch.OutOfMemoryError("no room")
        return real(nbytes, device)

    monkeypatch.setattr(mp, "_workspace", small_card)
    assert torch.equal(call(), want)
    assert len(asked) == 2 and asked[0] == full and asked[1] < full // 2
    monkeypatch.setattr(mp, "_workspace", lambda nbytes, device: small_card(full, device))
    with pytest.raises(torch.OutOfMemoryError):
        call()
