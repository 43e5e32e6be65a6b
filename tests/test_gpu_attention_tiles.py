"""The attention passes over 128 positions per workgroup, which work on two tiles at once: every count of tiles from one on,
sequences that end in any of a workgroup's waves, against the same sums in 64 bits; keys behind a query never reach it."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (batch, seq, heads): more than 128 workgroups, so that this form is taken; 1, 2, 3, 4, 5, 8 and 9 tiles of 64, ends in each wave
SHAPES = [(33, 1, 4), (44, 31, 3), (130, 64, 1), (65, 65, 2), (26, 97, 5), (33, 128, 4), (33, 129, 2), (22, 191, 3), (13, 225, 5),
          (33, 256, 2), (11, 300, 4), (9, 500, 4), (7, 513, 4)]


@pytest.fixture(scope="module")
def dom():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_15241_amd import domino
    domino.load()
    return domino


def forward(dom, qkv, b, s, nh, d):
    ctx = torch.full((b * s, nh * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((b, nh, s), float("nan"), device="cuda")
    dom.domino_attention_fwd(qkv, 3 * nh * d, b, s, nh, d, ctx, lse)
    return ctx, lse


def draw(b, s, nh, d):
    g = torch.Generator(device="cuda").manual_seed(b + 31 * s + 7 * nh + d)
    return torch.randn(b * s, 3 * nh * d, generator=g, device="cuda").to(torch.bfloat16)


@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("b,s,nh", SHAPES)
def test_forward(dom, d, b, s, nh):
    qkv = draw(b, s, nh, d)
    ctx, lse = forward(dom, qkv, b, s, nh, d)
    q, k, v = (t.double().reshape(b, s, nh, d).transpose(1, 2).reshape(b * nh, s, d).contiguous() for t in qkv.split(nh * d, 1))
    scores = torch.bmm(q, k.transpose(1, 2).contiguous()) / d ** 0.5
    scores.masked_fill_(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    want = torch.bmm(torch.softmax(scores, -1), v).reshape(b, nh, s, d).transpose(1, 2).reshape(b * s, nh * d)
    # probabilities and results are rounded to bf16 (2^-9 each): 2e-3 in the 2-norm; the statistics are fp32
    assert (ctx.double() - want).norm() <= 4e-3 * want.norm()
    assert (ctx.double() - want).abs().max() <= 1e-2 * want.abs().max()
    assert (lse.double() - torch.logsumexp(scores, -1).reshape(b, nh, s)).abs().max() <= 2e-5


@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_keys_behind_a_query_do_not_reach_it(dom, d, bad):
    b, s, nh = 13, 330, 5
    qkv = draw(b, s, nh, d)
    ctx, lse = forward(dom, qkv, b, s, nh, d)
    for first in (1, 64, 100, 257):
        spoiled = qkv.clone().reshape(b, s, 3, nh * d)
        spoiled[:, first:, 1] = bad
        ctx2, lse2 = forward(dom, spoiled.reshape(b * s, -1), b, s, nh, d)
        assert torch.equal(ctx2.reshape(b, s, -1)[:, :first], ctx.reshape(b, s, -1)[:, :first])
        assert torch.equal(lse2[:, :, :first], lse[:, :, :first])


@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("s,ld", [(1, (1 << 24) + 8), (5, (1 << 24) + 8), (3, (1 << 25) + 64), (7, 1 << 24)])
def test_rows_so_wide_that_a_tile_of_them_is_over_2_gib(dom, d, s, ld):
    """64 rows of such a matrix are more than 31 bits of bytes, the few that it has are not: same bits as from a narrow one."""
    qkv = draw(1, s, 1, d)
    ctx, lse = forward(dom, qkv, 1, s, 1, d)
    wide = torch.full((s, ld), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide[:, :3 * d] = qkv
    ctx2, lse2 = torch.zeros_like(ctx), torch.zeros_like(lse)
    dom.domino_attention_fwd(wide, ld, 1, s, 1, d, ctx2, lse2)
    assert torch.equal(ctx2, ctx) and torch.equal(lse2, lse)
