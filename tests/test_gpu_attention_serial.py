"""The attention forward that takes a tile's scores, softmax and output one after the other (lone tiles, heads of 64 in many workgroups,
heads of 128 of two tiles): against the same sums in 64 bits, and bit for bit what the form that works on two tiles at once gives for a
part of the batch."""
import pytest

from test_gpu_attention_tiles import dom, draw, forward      # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (head_dim, batch, seq, heads, batch elements that the other form takes, 0: none): the first and last number of workgroups of each range
# of the rule, one and two tiles and more, full and ragged, a lone position
SHAPES = [(64, 130, 1, 1, 0), (64, 33, 31, 4, 0), (64, 645, 64, 1, 0), (64, 513, 65, 1, 200), (64, 768, 100, 1, 250), (64, 129, 256, 1, 128), (64, 257, 129, 1, 100),
          (64, 205, 321, 2, 60), (64, 114, 1003, 3, 20), (80, 130, 64, 1, 0), (80, 70, 33, 2, 0), (128, 65, 64, 2, 0), (128, 131, 7, 1, 0),
          (128, 257, 128, 1, 200), (128, 128, 65, 4, 50)]


@pytest.mark.parametrize("d,b,s,nh,few", SHAPES)
def test_against_64_bits_and_the_other_form(dom, d, b, s, nh, few):
    qkv = draw(b, s, nh, d)
    ctx, lse = forward(dom, qkv, b, s, nh, d)
    for part in torch.arange(b, device="cuda").split(max(1, (1 << 24) // (nh * s * s))):      # the scores of a part in 64 bits: 128 MB at most
        rows = qkv.reshape(b, s, -1)[part].double()
        n = len(part)
        q, k, v = (t.reshape(n, s, nh, d).transpose(1, 2).reshape(n * nh, s, d).contiguous() for t in rows.split(nh * d, 2))
        scores = torch.bmm(q, k.transpose(1, 2).contiguous()) / d ** 0.5
        scores.masked_fill_(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
        want = torch.bmm(torch.softmax(scores, -1), v).reshape(n, nh, s, d).transpose(1, 2).reshape(n, s, nh * d)
        got = ctx.reshape(b, s, -1)[part].double()
        # as in test_gpu_attention_tiles: probabilities and results are rounded to bf16, the statistics are fp32
        assert (got - want).norm() <= 4e-3 * want.norm()
        assert (got - want).abs().max() <= 1e-2 * want.abs().max()
        assert (lse[part].double() - torch.logsumexp(scores, -1).reshape(n, nh, s)).abs().max() <= 2e-5
    if few:
        ctx2, lse2 = forward(dom, qkv[:few * s].contiguous(), few, s, nh, d)
        assert torch.equal(ctx2, ctx[:few * s]) and torch.equal(lse2, lse[:few])
