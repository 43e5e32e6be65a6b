"""The block output of blocks of 2^24 values and more, where a pass of its own moves it past the caches: exactly the rounded fp32 sum of what
the same call left of its terms, with and without the other ranks' sum, one row group and two."""
import pytest

from paper_2409_15241_amd import synth
from test_gpu_parts import H      # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("others", [True, False])
@pytest.mark.parametrize("hidden,heads,ffn,batch,seq,p", [(2560, 32, 10240, 7, 937, 1), (5120, 40, 20480, 4, 1283, 4)])
def test_sum_of_its_terms(H, hidden, heads, ffn, batch, seq, p, others):
    assert batch * seq * hidden >= 1 << 24
    sc = synth.WORKLOADS["tiny"].replace(hidden=hidden, heads=heads, tp=8, rank=0, ffn=ffn, batch=batch, seq=seq, p=p, q=1)
    x, dy = synth.make_activations(sc)
    b = H.LayerBuffers(sc, synth.make_rank_params(sc, random_affine=True), x, dy, synth.make_others(sc) if others else None)
    b.y.fill_(7.0)
    torch.cuda.synchronize()
    b.forward()
    torch.cuda.synchronize()
    want = b.saved_tensor("x1").view(b.y.shape).float() + b.mlp_partial.float()
    if others:
        want += b.mlp_others.float()
    assert torch.equal(b.y, (want + b.params["b_down"].float()).bfloat16())
