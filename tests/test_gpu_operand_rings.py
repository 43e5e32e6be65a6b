"""Whole-tile products whose rings hold more tiles of one operand than the contraction has, as many, and more: all whole
tiles sum in the same order, so every depth is compared bit for bit with 256x256 tiles."""
import pytest

from test_gpu_forms import close, gpu
from test_gpu_kernels import dom      # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
TILE_256x128, TILE_256x256 = 1, 2


# 1 to 9 operand tiles of 64, ragged in the last; (M, N): a full tile and ragged edges; 192x256 tiles by the rule at every depth
DEPTHS = [8, 64, 72, 128, 192, 200, 256, 320, 328, 456, 520, 576]
TILES_192x256 = (4408, 1800)


@pytest.mark.parametrize("K", DEPTHS)
@pytest.mark.parametrize("tile,M,N", [(TILE_256x128, 264, 200), (TILE_256x128, 512, 128), (-1, *TILES_192x256)])
def test_every_depth_around_the_ring(dom, tile, M, N, K):
    torch.manual_seed(M + K)
    A, W = gpu((M, K)), gpu((K, N), 0.05)
    Wt, At = W.t().contiguous(), A.t().contiguous()
    for layout, a, lda, b, ldb, epi in ((dom.GEMM_NN, A, K, W, N, dom.EPI_STORE), (dom.GEMM_NT, A, K, Wt, K, dom.EPI_STORE),
                                        (dom.GEMM_TN, At, M, W, N, dom.EPI_ACC_F32)):
        got = [torch.full((M, N), 7.0, device="cuda", dtype=torch.float32 if epi == dom.EPI_ACC_F32 else torch.bfloat16) for _ in range(2)]
        for C, t in zip(got, (tile, TILE_256x256)):
            dom.domino_gemm(layout, epi, t, a, lda, b, ldb, C, N, M, N, K)
        torch.cuda.synchronize()
        assert close(got[1], A.float() @ W.float())
        assert torch.equal(*got), layout


# the longer rings of 256x128 tiles begin at a contraction of 2048: the line itself, one step under it, and behind it every remainder of
# tiles over the places of either operand
@pytest.mark.parametrize("K", [2040, 2048, 2056, 2112, 2184, 2240, 2312, 2368, 2440, 2496, 2568])
@pytest.mark.parametrize("M,N", [(264, 200), (512, 128)])
def test_deep_contractions(dom, M, N, K):
    test_every_depth_around_the_ring(dom, TILE_256x128, M, N, K)
