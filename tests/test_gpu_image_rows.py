"""Images on both sides of the line that decides the height of their tiles: the launch that is made, and its results."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import test_gpu_image_tiles as tiles  # noqa: E402


class KernelNode(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint32 * 3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


# parts of 28 k-tiles and of 29, of 32; one of 32 and of 33; as many tiles as the chip has units, of 64 and of 65; grid: tiles of the height times parts
@pytest.mark.parametrize("m,d,k,grid", [(6144, 3584, 64, 96 * 2), (6144, 3712, 64, 48 * 5), (6100, 4096, 256, 48 * 5), (4096, 8192, 200, 32 * 8), (10240, 2048, 256, 160),
                                        (10240, 2112, 256, 80 * 3), (16384, 4096, 64, 256), (16384, 4160, 64, 128 * 2)])
def test_height(m, d, k, grid):
    from paper_2605_03109_amd import gsi

    W = torch.empty(m, d, dtype=torch.bfloat16, device="cuda")
    U, M = torch.empty(d, k, dtype=torch.bfloat16, device="cuda"), torch.empty(m, k, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(gsi.workspace_bytes(gsi.CALL_BUILD_IMAGE, m, d, k, 0), dtype=torch.uint8, device="cuda")
    print(f"case image height m={m} d={d} k={k}", flush=True)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        gsi.build_image(W, U, M, ws=ws)
    n = ctypes.c_size_t(0)
    vp = ctypes.c_void_p
    nodes, params = gsi.lib.hipGraphGetNodes, gsi.lib.hipGraphKernelNodeGetParams
    nodes.argtypes, params.argtypes = [vp, vp, ctypes.POINTER(ctypes.c_size_t)], [vp, ctypes.POINTER(KernelNode)]
    assert nodes(graph.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    found = (vp * n.value)()
    assert nodes(graph.raw_cuda_graph(), found, ctypes.byref(n)) == 0
    first = KernelNode()
    assert params(found[0], ctypes.byref(first)) == 0
    assert first.grid[0] == grid


@pytest.mark.parametrize("m,d,k", [(6144, 3712, 64), (6100, 4096, 256), (4096, 8192, 200), (10241, 2112, 260)])
def test_images(m, d, k):
    tiles.test_images(m, d, k, 0)
