"""The library's calls inside a HIP graph (torch.cuda.CUDAGraph): they are
plain kernel launches on the caller's stream that allocate nothing and
record no memset, so a captured call replays as the same kernels.  Each
graph is replayed several times with the program's own eager work and
synchronizations between the replays (the output refilled with NaN by a
fill kernel, an eager call of the same product into another buffer), and
every replay must equal the eager result bit for bit (the kernels are
deterministic)."""
import numpy as np
import pytest
import torch

import paper_2308_15152_amd as pkg
import synth
from gpu_util import device, to_np

pytestmark = pytest.mark.gpu

# the tile kernel on whole tiles, on ragged ones and with four wave groups, the
# register flow (short k), the full-tile kernel (more than two rounds of tiles)
# and its persistent stream form
SHAPES = [(16, 64, 64, 64), (3, 100, 90, 70), (1, 65, 70, 2051), (3, 100, 90, 60),
          (520, 128, 128, 128), (300, 256, 256, 128)]
KERNELS = ["gemm_tile_kernel", "gemm_tile_kernel", "gemm_tile_kernel", "bgemm_reg_kernel",
           "bgemm_big_kernel", "bgemm_big_stream_kernel"]


def _capture(fn):
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            fn()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    return g


def _bits(x):
    return np.asarray(x, dtype=np.float32).view(np.uint32)


@pytest.mark.parametrize("shape,kernel", zip(SHAPES, KERNELS),
                         ids=["x".join(map(str, s)) for s in SHAPES])
def test_gemm_graph_replays_match_eager(shape, kernel):
    dev = device()
    A, B = synth.gemm_inputs(*shape, seed=500 + shape[1])
    Ad, Bd = A.to(dev), B.to(dev)
    eager = to_np(pkg.sgemm_emu_batched(Ad, Bd))
    C = torch.full(eager.shape, float("nan"), device=dev)
    assert pkg.sgemm_emu_launch_form(Ad, Bd, C)[0] == kernel
    g = _capture(lambda: pkg.sgemm_emu_batched(Ad, Bd, C))
    for _ in range(3):
        C.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(_bits(to_np(C)), _bits(eager))
        other = to_np(pkg.sgemm_emu_batched(Ad, Bd))
        assert np.array_equal(_bits(other), _bits(eager))


@pytest.mark.parametrize("rows,length", [(300, 2048), (5, 40000), (3000, 20)],
                         ids=["whole", "parts", "short"])
def test_scan_and_householder_graph_replays_match_eager(rows, length):
    """Whole rows, rows in parts (three launches) and short rows."""
    dev = device()
    X = synth.uniform((rows, length), synth.rng(510)).to(dev)
    u, B = synth.householder_inputs(40, 64, 64, seed=511)
    ud, Bd = u.to(dev), B.to(dev)
    y_eager = to_np(pkg.sgemm_emu_scan(X))
    h_eager = to_np(pkg.householder_emu_batched(ud, Bd))
    Y = torch.full(X.shape, float("nan"), device=dev)
    H = torch.full((40, 64, 64), float("nan"), device=dev)

    def step():
        pkg.sgemm_emu_scan(X, Y)
        pkg.householder_emu_batched(ud, Bd, H)

    g = _capture(step)
    for _ in range(3):
        Y.fill_(float("nan"))
        H.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(_bits(to_np(Y)), _bits(y_eager))
        assert np.array_equal(_bits(to_np(H)), _bits(h_eager))
        assert np.array_equal(_bits(to_np(pkg.sgemm_emu_scan(X))), _bits(y_eager))


def test_accumulate_graph_replays_match_eager():
    """D += A^T B in place: every replay adds once more."""
    dev = device()
    A, B = synth.gemm_inputs(4, 321, 70, 333, seed=512)
    Ad, Bd = A.transpose(1, 2).contiguous().to(dev), B.to(dev)
    C = synth.uniform((4, 321, 70), synth.rng(513)).to(dev)
    D = C.clone()
    g = _capture(lambda: pkg.sgemm_emu_batched_acc(Ad, Bd, D, D, op_a=pkg.OP_T))
    D.copy_(C)
    for _ in range(3):
        eager = to_np(pkg.sgemm_emu_batched_acc(Ad, Bd, D.clone(), op_a=pkg.OP_T))
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(_bits(to_np(D)), _bits(eager))
