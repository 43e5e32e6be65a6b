"""The attention backward that forms D = rowsum(dctx * ctx) itself (at most 256 positions, few workgroups): against 64 bits, at the
edges of its tiles of 32 positions and of the rule, with a scratch that holds no D and still holds none afterwards, and with batch
elements whose next rows are anything but zero."""
import math

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# (batch, seq, heads): last tiles of 1, 31, 32 positions and between, rows of 3 to 8 tiles
OWN = [(1, 65, 1), (2, 95, 2), (3, 97, 1), (1, 127, 3), (2, 128, 2), (1, 129, 3), (2, 160, 1), (2, 255, 1), (2, 256, 2)]
# what the pass in front forms D for: too few positions for the form, and too many for its own D
PASS = [(1, 1, 1), (3, 31, 2), (2, 33, 1), (2, 257, 2)]


@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("b,s,nh", OWN + PASS)
def test_against_64_bits(d, b, s, nh):
    from paper_2409_15241_amd import domino as dom
    g = torch.Generator().manual_seed(1000 * d + s)
    hl = nh * d
    qkv = torch.randn((b * s, 3 * hl), generator=g).bfloat16()
    dctx = torch.randn((b * s, hl), generator=g).bfloat16()
    q, k, v = (t.reshape(b, s, nh, d).transpose(1, 2) for t in qkv.double().split(hl, dim=1))
    score = (q @ k.transpose(-1, -2) / math.sqrt(d)).masked_fill(torch.triu(torch.ones(s, s, dtype=torch.bool), 1), -math.inf)
    p = torch.softmax(score, -1)
    lse = torch.logsumexp(score, -1)
    ctx = (p @ v).transpose(1, 2).reshape(b * s, hl).bfloat16()         # what the forward leaves: rounded
    heads = lambda t: t.double().reshape(b, s, nh, d).transpose(1, 2)
    do = heads(dctx)
    ds = p * (do @ v.transpose(-1, -2) - (do * heads(ctx)).sum(-1, keepdim=True)) / math.sqrt(d)
    want = [(ds @ k), (ds.transpose(-1, -2) @ q), p.transpose(-1, -2) @ do]
    out = torch.full((b * s, 3 * hl), 7.0, dtype=torch.bfloat16, device="cuda")
    dot = torch.full((b, nh, s), math.nan, dtype=torch.float32, device="cuda")
    dom.domino_attention_bwd(qkv.cuda(), 3 * hl, ctx.cuda(), dctx.cuda(), lse.float().cuda(), out, dot, b, s, nh, d)
    torch.cuda.synchronize()
    assert bool(dot.isnan().all()) == ((b, s, nh) in OWN)         # nobody wrote a D where nobody reads one
    for got, ref in zip(out.cpu().double().split(hl, dim=1), want):
        ref = ref.transpose(1, 2).reshape(b * s, hl)
        # P and dS are rounded to bf16 before their products (2^-9 a term, of random sign), the results once more; one position: all zero but dV
        assert (got - ref).norm() <= 1e-2 * ref.norm() + 1e-6 * math.sqrt(ref.numel())
