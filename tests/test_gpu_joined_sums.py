"""The bias gradients' column sums as further workgroups of the weight gradients' launch: bit for bit what they are as launches of their
own, which wgrad_per_slice keeps.  The weight gradients themselves are checked against their operands."""
import pytest

from paper_2409_15241_amd import synth
from test_gpu_parts import H      # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (hidden, heads, ranks, ffn, batch, seq, p): contraction ranges; whole tiles behind the chain, ragged; weight gradients beside the
# chain, one row group (one matrix a launch) and two (two sums a launch)
BLOCKS = [(512, 8, 1, 2048, 16, 1024, 1), (2560, 32, 8, 10240, 2, 501, 2), (5120, 40, 8, 20480, 2, 777, 2), (4096, 32, 8, 16384, 4, 2048, 4)]


@pytest.mark.parametrize("hidden,heads,tp,ffn,batch,seq,p", BLOCKS)
def test_joined_as_launches_of_their_own(H, hidden, heads, tp, ffn, batch, seq, p):
    sc = synth.WORKLOADS["tiny"].replace(hidden=hidden, heads=heads, tp=tp, rank=0, ffn=ffn, batch=batch, seq=seq, p=p, q=1)
    params = synth.make_rank_params(sc, random_affine=True)
    x, dy = synth.make_activations(sc)
    got = []
    for per_slice in (0, 1):
        b = H.LayerBuffers(sc.replace(wgrad_per_slice=per_slice), params, x, dy, synth.make_others(sc))
        b.forward()
        b.backward()
        torch.cuda.synchronize()
        got.append({k: g.clone() for k, g in b.grads.items()})
    for k in ("b_qkv", "b_up"):
        assert torch.equal(got[0][k], got[1][k]), k
    for k in ("w_down", "w_up", "w_o", "w_qkv"):      # fp32 sums over the rows in another order
        assert (got[0][k] - got[1][k]).norm() <= 1e-5 * got[1][k].norm(), k
