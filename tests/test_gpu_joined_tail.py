"""The Norm1 backward and the bias gradients in the launch of a small block's weight gradients: bit for bit what they are
as launches of their own, which the block's Norm1 part makes of them when it is a call by itself."""
import pytest

from paper_2409_15241_amd import synth
from test_gpu_parts import H, bwd_part      # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (hidden, heads, ranks, ffn, arch, batch, seq, p).  Rows of 1, 2 and 4 waves in workgroups of eight (64x64 tiles) and of four, and
# wider rows, which go out alone; odd numbers of rows, partial rows, row ranges and column blocks
BLOCKS = [(256, 4, 2, 1024, "gpt", 2, 128, 2), (2560, 32, 8, 1024, "gpt", 1, 131, 1), (2048, 32, 16, 1024, "gpt", 3, 43, 3),
          (4608, 36, 18, 1152, "gpt", 1, 64, 1), (1024, 8, 4, 5504, "llama", 2, 200, 1), (2048, 16, 4, 4096, "gpt", 4, 67, 4),
          (2560, 20, 4, 5120, "gpt", 2, 99, 2), (512, 8, 2, 1040, "gpt", 5, 13, 1)]


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("hidden,heads,tp,ffn,arch,batch,seq,p", BLOCKS)
def test_joined_as_alone(H, hidden, heads, tp, ffn, arch, batch, seq, p, accumulate):
    from paper_2409_15241_amd import domino as D
    sc = synth.WORKLOADS["tiny-llama" if arch == "llama" else "tiny"].replace(hidden=hidden, heads=heads, tp=tp, rank=0, ffn=ffn, batch=batch, seq=seq, p=p, q=1)
    params = synth.make_rank_params(sc, random_affine=True)
    x, dy = synth.make_activations(sc)
    bufs = [H.LayerBuffers(sc, params, x, dy, synth.make_others(sc)) for _ in range(2)]
    for b in bufs:
        for g in b.grads.values():
            if g is not None:
                g.fill_(0.25)
        b.dx.fill_(7.0)
        torch.cuda.synchronize()
        b.forward()
    whole, parts = bufs
    whole.backward(accumulate)
    bwd_part(D, parts, D.BWD_MLP | D.BWD_ATTN, accumulate)
    bwd_part(D, parts, D.BWD_NORM1, accumulate)
    torch.cuda.synchronize()
    assert torch.equal(whole.dx, parts.dx)
    for k, g in whole.grads.items():
        assert g is None or torch.equal(g, parts.grads[k]), k
