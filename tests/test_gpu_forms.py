"""The forms that the launchers pick by size: products whose contraction is dealt over the waves of a workgroup, attention
with few and with many workgroups, weight gradients over several contraction ranges.  Shapes at the edges of tiles and of
the ranges in which a form is picked."""
import numpy as np
import pytest

from oracle import domino_oracle as O
from paper_2409_15241_amd import synth
from test_gpu_kernels import BF16_OUT, _attn_inputs, dev, dom, host, relerr, rnd      # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# 64x64 tiles, eight waves: fewer operand tiles than waves, one more than waves, a tail of the contraction, ragged edges
FEW = [(72, 136, 520), (200, 264, 200), (64, 64, 512), (400, 1032, 584)]
SHALLOW = [(200, 264, 72)]         # two operand tiles: dealt under GeLU', plain 128x128 tiles otherwise
# 128x128 tiles, four waves: deep products of more than two rounds of 64x64 tiles
DEEP = [(1032, 2568, 4104), (1024, 2688, 4096)]
# (M, ffn columns, K) of the gated and rotary products: dealt forms too
GATED = [(72, 96, 520), (400, 352, 584), (1032, 1376, 4104)]
# tiles of 192 and 320 rows or columns, products and (M, ffn columns, K): two operand tiles and more, ragged edges (fp32 sums
# that are added to what C holds take ADDING's)
WIDE = [(1976, 5944, 72), (3408, 2352, 328), (8104, 2552, 136), (4048, 5112, 264), (4776, 3376, 72), (2888, 5784, 264)]
WIDE_GATED = [(1160, 3392, 72), (2072, 3936, 200)]       # (the derivative takes 256x128 and 192x256 here; BY_TILE has it in all four)
# one tile of 192 or 320 each under every epilogue it can take, by GemmTile: products (also the gated derivative), (M, ffn
# columns, K) of the gated product, rotary products; the first of each row is one operand tile deep where such a shape takes it
BY_TILE = {6: [(7016, 1552, 64), (7352, 1056, 264)], 7: [(7208, 1032, 64), (1040, 7208, 264)],
           8: [(2896, 6488, 136), (2944, 6432, 264)], 9: [(7192, 2208, 64), (6184, 2584, 264)]}
# fp32 sums added to what C holds: 128x128, 256x256, and the tiles of 192 and 320 that the rule takes for them
ADDING = {0: (264, 3384, 64), 2: (3080, 3928, 264), 6: (2312, 3360, 520), 8: (3352, 4768, 520), 9: (2832, 6888, 2056)}
BY_TILE_GATED = {7: [(648, 5568, 64), (536, 6624, 264)], 9: [(2576, 3104, 64), (1576, 4736, 264)]}
BY_TILE_ROPE = {7: [(1184, 6784, 64), (1032, 7424, 200)], 9: [(2336, 6656, 64), (2080, 7296, 264)]}
# (hidden, ffn columns, local heads of 64, ranks, batch, seq) of blocks whose four weight gradients share a launch of such tiles
JOINED = {6: [(2688, 584, 7, 6, 2, 260), (3136, 376, 7, 7, 3, 67)], 7: [(3520, 464, 5, 11, 1, 130), (2560, 544, 8, 5, 3, 134)]}
# (batch, seq, heads): few workgroups, 32 positions each, and many, 128 positions each
ATTN_FEW = [(1, 129, 1), (2, 161, 3), (1, 1000, 2)]
ATTN_MANY = [(40, 200, 4), (35, 257, 2), (24, 63, 6)]
RANGE_SEQS = [1024, 1000]
# test_forms.py checks on the CPU that these shapes take these forms


def gpu(a, scale=1.0):
    return torch.randn(a, device="cuda").mul_(scale).to(torch.bfloat16)


def close(got, ref, bar=BF16_OUT):
    return float((got.float() - ref).abs().max() / ref.abs().max()) < bar


@pytest.mark.parametrize("M,N,K", FEW + SHALLOW + DEEP)
def test_products_with_a_dealt_contraction(dom, M, N, K):
    torch.manual_seed(M + N + K)
    A, W, bias = gpu((M, K)), gpu((K, N), 0.05), gpu(N, 0.5)
    ref = A.float() @ W.float()
    C, aux = torch.zeros((M, N), device="cuda", dtype=torch.bfloat16), torch.zeros((M, N), device="cuda", dtype=torch.bfloat16)
    dom.domino_gemm(dom.GEMM_NN, dom.EPI_STORE, -1, A, K, W, N, C, N, M, N, K, bias=bias)
    torch.cuda.synchronize()
    assert close(C, ref + bias.float())
    for tanh in (1, 0):
        dom.domino_gemm(dom.GEMM_NN, dom.EPI_BIAS_GELU, -1, A, K, W, N, C, N, M, N, K, bias=bias, aux=aux, ldaux=N, gelu_tanh=tanh)
        torch.cuda.synchronize()
        pre = ref + bias.float()
        assert close(aux, pre)
        assert close(C, torch.nn.functional.gelu(pre, approximate="tanh" if tanh else "none"))
    Wt = W.t().contiguous()                                        # [N][K]: the input-gradient layout
    dom.domino_gemm(dom.GEMM_NT, dom.EPI_STORE, -1, A, K, Wt, K, C, N, M, N, K)
    torch.cuda.synchronize()
    assert close(C, ref)
    pre = gpu((M, N), 1.5)
    x = pre.float().requires_grad_()
    for tanh in (1, 0):
        g, = torch.autograd.grad(torch.nn.functional.gelu(x, approximate="tanh" if tanh else "none").sum(), x)
        dom.domino_gemm(dom.GEMM_NT, dom.EPI_DGELU, -1, A, K, Wt, K, C, N, M, N, K, aux=pre, ldaux=N, gelu_tanh=tanh)
        torch.cuda.synchronize()
        assert close(C, ref * g)
    At = A.t().contiguous()                                        # [K][M]: the weight-gradient layout, summed onto what is there
    F = torch.ones((M, N), device="cuda")
    dom.domino_gemm(dom.GEMM_TN, dom.EPI_ACC_F32, -1, At, M, W, N, F, N, M, N, K, beta=1)
    torch.cuda.synchronize()
    assert close(F, ref + 1.0, 1e-4)


@pytest.mark.parametrize("M,fl,K", GATED)
def test_gated_and_rotary_products_with_a_dealt_contraction(dom, M, fl, K):
    torch.manual_seed(M + fl)
    A, W = gpu((M, K)), gpu((K, 2 * fl), 0.05)
    ref = A.float() @ W.float()
    act, gu = torch.zeros((M, fl), device="cuda", dtype=torch.bfloat16), torch.zeros((M, 2 * fl), device="cuda", dtype=torch.bfloat16)
    dom.domino_gemm(dom.GEMM_NN, dom.EPI_SWIGLU, -1, A, K, W, 2 * fl, act, fl, M, fl, K, aux=gu, ldaux=2 * fl, n_split=fl)
    torch.cuda.synchronize()
    assert close(gu, ref) and close(act, torch.nn.functional.silu(ref[:, :fl]) * ref[:, fl:])
    dact, Wd = gpu((M, K)), gpu((fl, K), 0.05)
    x = gu.float().requires_grad_()
    d = dact.float() @ Wd.float().t()
    g, = torch.autograd.grad((torch.nn.functional.silu(x[:, :fl]) * x[:, fl:] * d).sum(), x)
    out = torch.zeros_like(gu)
    dom.domino_gemm(dom.GEMM_NT, dom.EPI_DSWIGLU, -1, dact, K, Wd, K, out, 2 * fl, M, fl, K, aux=gu, ldaux=2 * fl, n_split=fl)
    torch.cuda.synchronize()
    assert close(out, g)
    for d_head in (64, 128):
        N = fl // 128 * 128 + 128
        Wr = gpu((K, N), 0.05)
        plain, turned = torch.zeros((M, N), device="cuda", dtype=torch.bfloat16), torch.zeros((M, N), device="cuda", dtype=torch.bfloat16)
        dom.domino_gemm(dom.GEMM_NN, dom.EPI_STORE, -1, A, K, Wr, N, plain, N, M, N, K)
        dom.domino_rope(plain, N, M, M, 0, 1, N // d_head, d_head, 10000.0, 0)
        dom.domino_gemm_rope(-1, A, K, Wr, N, turned, N, M, N, K, M, d_head, N, 10000.0)
        torch.cuda.synchronize()
        assert close(turned, plain.float(), 1.5e-2)


@pytest.mark.parametrize("M,N,K", WIDE)
def test_products_in_tiles_of_192_and_320(dom, M, N, K):
    test_products_with_a_dealt_contraction(dom, M, N, K)


@pytest.mark.parametrize("M,fl,K", WIDE_GATED)
def test_gated_and_rotary_products_in_tiles_of_192_and_320(dom, M, fl, K):
    test_gated_and_rotary_products_with_a_dealt_contraction(dom, M, fl, K)


TILE_256x256 = 2


def same_bits_by_rule_and_in_256x256(launch, *outs):
    """launch(tile) with the form picked by size and in 256x256 tiles: all whole tiles sum in the same order."""
    got = []
    for tile in (-1, TILE_256x256):
        for o in outs:
            o.fill_(7.0)
        launch(tile)
        torch.cuda.synchronize()
        got.append([o.clone() for o in outs])
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("M,N,K", [x for xs in BY_TILE.values() for x in xs])
def test_tiles_of_192_and_320_sum_as_256x256_does(dom, M, N, K):
    torch.manual_seed(M + N + K)
    A, W, bias = gpu((M, K)), gpu((K, N), 0.05), gpu(N, 0.5)
    Wt, At = W.t().contiguous(), A.t().contiguous()
    C, aux, pre = (torch.empty((M, N), device="cuda", dtype=torch.bfloat16) for _ in range(3))
    same_bits_by_rule_and_in_256x256(lambda t: dom.domino_gemm(dom.GEMM_NN, dom.EPI_STORE, t, A, K, W, N, C, N, M, N, K, bias=bias), C)
    same_bits_by_rule_and_in_256x256(lambda t: dom.domino_gemm(dom.GEMM_NN, dom.EPI_BIAS_GELU, t, A, K, W, N, C, N, M, N, K, bias=bias, aux=aux, ldaux=N), C, aux)
    same_bits_by_rule_and_in_256x256(lambda t: dom.domino_gemm(dom.GEMM_NT, dom.EPI_STORE, t, A, K, Wt, K, C, N, M, N, K), C)
    assert close(C, A.float() @ W.float())
    pre.normal_(0, 1.5)
    same_bits_by_rule_and_in_256x256(lambda t: dom.domino_gemm(dom.GEMM_NT, dom.EPI_DGELU, t, A, K, Wt, K, C, N, M, N, K, aux=pre, ldaux=N), C)
    gu, dgu = gpu((M, 2 * N)), torch.empty((M, 2 * N), device="cuda", dtype=torch.bfloat16)
    same_bits_by_rule_and_in_256x256(lambda t: dom.domino_gemm(dom.GEMM_NT, dom.EPI_DSWIGLU, t, A, K, Wt, K, dgu, 2 * N, M, N, K, aux=gu, ldaux=2 * N, n_split=N), dgu)
    F = torch.empty((M, N), device="cuda")
    same_bits_by_rule_and_in_256x256(lambda t: dom.domino_gemm(dom.GEMM_TN, dom.EPI_ACC_F32, t, At, M, W, N, F, N, M, N, K), F)


@pytest.mark.parametrize("M,N,K", ADDING.values())
def test_tiles_add_fp32_sums_as_256x256_does(dom, M, N, K):
    torch.manual_seed(M + N + K)
    A, W, F = gpu((K, M)), gpu((K, N), 0.05), torch.empty((M, N), device="cuda")
    same_bits_by_rule_and_in_256x256(lambda t: dom.domino_gemm(dom.GEMM_TN, dom.EPI_ACC_F32, t, A, M, W, N, F, N, M, N, K, beta=1), F)
    assert close(F, A.float().t() @ W.float() + 7.0, 1e-4)


@pytest.mark.parametrize("M,fl,K", [x for xs in BY_TILE_GATED.values() for x in xs])
def test_gated_products_in_tiles_of_192_and_320_rows_sum_as_256x256_does(dom, M, fl, K):
    torch.manual_seed(M + fl + K)
    A, W = gpu((M, K)), gpu((K, 2 * fl), 0.05)
    act, gu = torch.empty((M, fl), device="cuda", dtype=torch.bfloat16), torch.empty((M, 2 * fl), device="cuda", dtype=torch.bfloat16)
    same_bits_by_rule_and_in_256x256(
        lambda t: dom.domino_gemm(dom.GEMM_NN, dom.EPI_SWIGLU, t, A, K, W, 2 * fl, act, fl, M, fl, K, aux=gu, ldaux=2 * fl, n_split=fl), act, gu)
    assert close(gu, A.float() @ W.float())


@pytest.mark.parametrize("M,N,K", [x for xs in BY_TILE_ROPE.values() for x in xs])
def test_rotary_products_in_tiles_of_192_and_320_rows_sum_as_256x256_does(dom, M, N, K):
    torch.manual_seed(M + N + K)
    A, W, C = gpu((M, K)), gpu((K, N), 0.05), torch.empty((M, N), device="cuda", dtype=torch.bfloat16)
    for d in (64, 128):
        same_bits_by_rule_and_in_256x256(lambda t: dom.domino_gemm_rope(t, A, K, W, N, C, N, M, N, K, M // 2 + 1, d, N // 128 // 2 * 128, 10000.0), C)


@pytest.mark.parametrize("h,fl,nl,tp,b,s", [x for xs in JOINED.values() for x in xs])
def test_joined_weight_gradients_sum_as_single_ones_do(dom, h, fl, nl, tp, b, s):
    """All four in one launch against one launch each, both in whole tiles over the whole contraction."""
    from paper_2409_15241_amd import harness as H
    base = synth.ShardConfig(name="joined", hidden=h, heads=nl * tp, tp=tp, rank=0, ffn=fl * tp, batch=b, seq=s, p=1, q=1)
    params = synth.make_rank_params(base, random_affine=True)
    x, dy = synth.make_activations(base)
    grads = []
    for per_slice in (0, 1):
        buf = H.LayerBuffers(base.replace(wgrad_per_slice=per_slice), params, x, dy, None, nstreams=1)
        buf.forward()
        buf.backward(accumulate=False)
        buf.sync()
        grads.append({k: g.clone() for k, g in buf.grads.items() if k.startswith("w_")})
        if not per_slice:
            act, g = buf.saved_tensor("act").view(b * s, fl).float(), buf.dy.view(b * s, h).float()
            assert close(buf.grads["w_down"], act.t() @ g, 1e-4)
    for k in grads[0]:
        assert torch.equal(grads[0][k], grads[1][k]), k


@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("b,s,nh", ATTN_FEW + ATTN_MANY)
def test_attention_with_few_and_with_many_workgroups(dom, d, b, s, nh):
    rng = np.random.default_rng(d + s + nh)
    hl = nh * d
    qkv, q, k, v = _attn_inputs(rng, b, s, nh, d)
    dctx = rnd(rng, (b * s, hl))
    ctx = torch.zeros((b * s, hl), dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((b, nh, s), dtype=torch.float32, device="cuda")
    dqkv = torch.zeros((b * s, 3 * hl), dtype=torch.bfloat16, device="cuda")
    dot = torch.zeros((b, nh, s), dtype=torch.float32, device="cuda")
    qd = dev(qkv)
    dom.domino_attention_fwd(qd, 3 * hl, b, s, nh, d, ctx, lse)
    dom.domino_attention_bwd(qd, 3 * hl, ctx, dev(dctx), lse, dqkv, dot, b, s, nh, d)
    torch.cuda.synchronize()
    back = lambda m: m.transpose(0, 2, 1, 3).reshape(b * s, hl)
    rctx, rlse = O.attention_fwd(q, k, v)
    assert relerr(host(ctx), back(rctx)) < 1e-2
    assert np.max(np.abs(lse.cpu().numpy() - rlse)) < 2e-3
    refs = O.attention_bwd(dctx.reshape(b, s, nh, d).transpose(0, 2, 1, 3).astype(np.float64), q, k, v)
    got = host(dqkv)
    for i, ref in enumerate(refs):
        assert relerr(got[:, i * hl:(i + 1) * hl], back(ref)) < 1.5e-2


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("seq", RANGE_SEQS)
def test_weight_gradients_over_contraction_ranges(dom, seq, accumulate):
    """A narrow block with many tokens: one launch over all rows in ranges, against one launch per matrix without."""
    from paper_2409_15241_amd import harness as H
    base = synth.ShardConfig(name="narrow", hidden=512, heads=8, tp=1, rank=0, ffn=2048, batch=16, seq=seq, p=1, q=1)
    params = synth.make_rank_params(base, random_affine=True)
    x, dy = synth.make_activations(base)
    grads = []
    for per_slice in (0, 1):
        buf = H.LayerBuffers(base.replace(wgrad_per_slice=per_slice), params, x, dy, None, nstreams=2)
        buf.forward()
        buf.backward(accumulate=False)
        if accumulate:
            buf.backward(accumulate=True)
        buf.sync()
        grads.append({k: g.clone() for k, g in buf.grads.items() if g is not None})
    for k, g in grads[0].items():
        assert float((g - grads[1][k]).norm() / grads[1][k].norm()) < 1e-5, k


# (hidden, ffn, batch, seq, arch, other ranks' sum): 64x64 dealt (the first three) and 192x256 tiles, ragged rows
BLOCK_OUTPUT = [(256, 512, 2, 37, synth.ARCH_GPT, True), (512, 2048, 3, 333, synth.ARCH_GPT, False), (512, 1376, 3, 333, synth.ARCH_LLAMA, True),
                (1280, 320, 2, 4000, synth.ARCH_GPT, True), (2560, 320, 2, 4100, synth.ARCH_GPT, True)]
# (hidden, ffn columns, batch, seq, arch, other ranks' sum) of a shard with one head of 64, by GemmTile of the MLP-down product;
# ragged rows and columns.  256x320 tiles (8) leave the output to a pass of its own.
BLOCK_OUTPUT_BY_TILE = {0: (5568, 72, 1, 139, synth.ARCH_GPT, True), 1: (320, 352, 5, 2191, synth.ARCH_LLAMA, True),
                        2: (832, 1032, 5, 2697, synth.ARCH_GPT, False), 5: (320, 3080, 5, 1315, synth.ARCH_GPT, True),
                        6: (832, 352, 5, 1899, synth.ARCH_LLAMA, True), 7: (704, 352, 5, 2209, synth.ARCH_GPT, True),
                        8: (2112, 3080, 3, 2459, synth.ARCH_GPT, True), 9: (1088, 264, 5, 2921, synth.ARCH_GPT, True)}


@pytest.mark.parametrize("h,fl,b,s,arch,others", BLOCK_OUTPUT_BY_TILE.values())
def test_block_output_in_every_tile(dom, h, fl, b, s, arch, others):
    test_block_output_is_the_rounded_sum_of_what_the_block_stores(dom, h, fl * (h // 64), b, s, arch, others, tp=h // 64)


@pytest.mark.parametrize("h,f,b,s,arch,others", BLOCK_OUTPUT)
def test_block_output_is_the_rounded_sum_of_what_the_block_stores(dom, h, f, b, s, arch, others, tp=1):
    """y = ((x1 + mlp_partial) + others) + b_down in fp32 of the stored bf16 tensors, rounded once: bit for bit."""
    from paper_2409_15241_amd import harness as H
    sc = synth.ShardConfig(name="out", hidden=h, heads=h // 64, tp=tp, rank=0, ffn=f, batch=b, seq=s, p=1, q=1, arch=arch)
    params = synth.make_rank_params(sc, random_affine=True)
    x, dy = synth.make_activations(sc)
    buf = H.LayerBuffers(sc, params, x, dy, synth.make_others(sc) if others else None, nstreams=2)
    buf.forward()
    buf.sync()
    x1 = buf.saved_tensor("x1").view(b, s, h).float()
    y = x1 + buf.mlp_partial.float()
    if others:
        y = y + buf.mlp_others.float()
    if buf.params["b_down"] is not None:
        y = y + buf.params["b_down"].float()
    assert torch.equal(buf.y, y.to(torch.bfloat16))
    assert close(buf.mlp_partial.view(b * s, h), buf.saved_tensor("act").view(b * s, -1).float() @ buf.params["w_down"].float())
