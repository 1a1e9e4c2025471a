"""Weight gradients whose segments have few and many 2048-row chunks, on both
sides of the 16 beyond which a workgroup shares an element's chunks, empty
segments among them; x and dout are small integers, so that every sum is exact
in any order."""
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


@pytest.mark.parametrize("sizes", [[16 * 2048], [16 * 2048 + 1], [5, 0, 17 * 2048 - 3, 2048],
                                   [30 * 2048 + 7, 0], [2048] * 5])
@pytest.mark.parametrize("F,Fo", [(8, 8), (24, 136)])
def test_weight_gradient(sizes, F, Fo):
    check(sizes, F, Fo)


@pytest.mark.parametrize("chunks", [17, 64, 65])  # elements enough: shared beyond 64 chunks
def test_weight_gradient_of_many_elements(chunks):
    check([chunks * 2048 - 5, 3], 264, 504)


def check(sizes, F, Fo):
    rng = np.random.default_rng(len(sizes) + F)
    seg = [0] + list(np.cumsum(sizes))
    n, T = seg[-1], len(sizes)
    x = rng.integers(-2, 3, (n, F)).astype(np.float32)
    d = rng.integers(-2, 3, (n, Fo)).astype(np.float32)
    W = torch.zeros(T, F, Fo, dtype=torch.bfloat16, device=DEV)
    _, dW = mp.segment_matmul_backward(seg, torch.from_numpy(x).to(DEV, torch.bfloat16), W,
                                       torch.from_numpy(d).to(DEV, torch.bfloat16), want_dx=False)
    for t in range(T):
        q = slice(seg[t], seg[t + 1])
        assert np.array_equal(dW[t].cpu().numpy(), x[q].T @ d[q])
