"""The rules that pick a kernel's form by size, on the CPU: the shapes of the GPU tests take the forms that those tests are
about, and what decides the order of a sum does not look at the streams."""
import os
import random
import shutil
import subprocess

import pytest

import test_gpu_forms as F
from paper_2409_15241_amd import domino as D

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
pytestmark = pytest.mark.skipif(not os.path.exists(CLANG) and not shutil.which("g++"), reason="needs a C++ compiler")
TILE_64_DEALT, TILE_128_DEALT = 4, 5
EPI_ROPE, EPI_RESID = 6, 7       # of csrc/gemm.h: not among the single-kernel entry points' epilogues


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("forms") / "host_forms")
    cc = CLANG if os.path.exists(CLANG) else "g++"
    subprocess.run([cc, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "host_forms_main.cpp"), "-o", exe], check=True, capture_output=True)

    def ask(questions):
        text = "\n".join(" ".join(str(int(x)) if not isinstance(x, str) else x for x in q) for q in questions) + "\n"
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        out = [int(x) for x in r.stdout.split()]
        assert len(out) == len(questions)
        return out
    return ask


def test_shapes_of_the_gpu_tests_take_the_dealt_forms(ask):
    epis = (D.EPI_STORE, D.EPI_BIAS_GELU, D.EPI_DGELU, D.EPI_ACC_F32)
    for shapes, form in ((F.FEW, TILE_64_DEALT), (F.DEEP, TILE_128_DEALT)):
        for M, N, K in shapes:
            assert ask([("gemm", e, M, N, K, 1, 0) for e in epis]) == [form] * len(epis), (M, N, K)
    for M, N, K in F.SHALLOW:
        assert ask([("gemm", D.EPI_DGELU, M, N, K, 1, 0), ("gemm", D.EPI_STORE, M, N, K, 1, 0)]) == [TILE_64_DEALT, 0], (M, N, K)
    for M, fl, K in F.GATED:
        n = fl // 128 * 128 + 128
        forms = ask([("gemm", D.EPI_SWIGLU, M, fl, K, 1, 0), ("gemm", D.EPI_DSWIGLU, M, fl, K, 1, 0), ("gemm", EPI_ROPE, M, n, K, 1, 0)])
        assert all(f in (TILE_64_DEALT, TILE_128_DEALT) for f in forms), (M, fl, K, forms)


def test_shapes_of_the_gpu_tests_take_every_tile_of_192_and_320(ask):
    wide = {6: "256x192", 7: "192x256", 8: "256x320", 9: "320x256"}
    for e in (D.EPI_STORE, D.EPI_BIAS_GELU, D.EPI_DGELU, D.EPI_ACC_F32):
        assert set(ask([("gemm", e, M, N, K, 1, 0) for M, N, K in F.WIDE])) >= set(wide), e
    gated = ask([("gemm", D.EPI_SWIGLU, M, N, K, 1, 0) for M, N, K in F.WIDE_GATED])
    assert set(gated) == {7, 9}                   # pairs of columns 32 apart inside every 64 of a wave tile


def test_shapes_of_the_gpu_tests_take_the_tile_they_are_listed_under(ask):
    epis = (D.EPI_STORE, D.EPI_BIAS_GELU, D.EPI_DGELU, D.EPI_DSWIGLU, D.EPI_ACC_F32)
    for tile, shapes in F.BY_TILE.items():
        for shape in shapes:
            assert ask([("gemm", e, *shape, 1, 0) for e in epis]) == [tile] * len(epis), (tile, shape)
    for e, table in ((D.EPI_SWIGLU, F.BY_TILE_GATED), (EPI_ROPE, F.BY_TILE_ROPE)):
        for tile, shapes in table.items():
            assert ask([("gemm", e, *shape, 1, 0) for shape in shapes]) == [tile] * len(shapes), (e, tile)
    for tile, shape in F.ADDING.items():
        assert ask([("gemm", D.EPI_ACC_F32, *shape, 1, 0, 1)]) == [tile], (tile, shape)
    assert any(K == 64 for shapes in F.BY_TILE.values() for _, _, K in shapes)      # one operand tile


def test_blocks_of_the_gpu_tests_form_their_output_in_the_tile_they_are_listed_under(ask):
    def form(h, fl, b, s):       # (tile of the MLP-down product, whether it forms the block output)
        output, = ask([("output", b * s, h, fl)])
        return ask([("gemm", EPI_RESID if output else D.EPI_STORE, b * s, h, fl, 1, 0)])[0], output
    for tile, (h, fl, b, s, _, _) in F.BLOCK_OUTPUT_BY_TILE.items():
        assert form(h, fl, b, s) == (tile, tile != 8), (tile, h, fl, b, s)
    assert [form(h, f, b, s) for h, f, b, s, _, _ in F.BLOCK_OUTPUT] == [(TILE_64_DEALT, 1)] * 3 + [(7, 1)] * 2


def test_blocks_of_the_gpu_tests_join_their_weight_gradients_in_the_tile_they_are_listed_under(ask):
    for tile, blocks in F.JOINED.items():
        for h, fl, nl, _, b, s in blocks:
            hl, K = 64 * nl, b * s
            shapes = [(fl, h), (h, fl), (hl, h), (h, 3 * hl)]
            tiles = sum(-(-m // 256) * -(-n // 256) for m, n in shapes)
            assert tiles <= 200                                # on the chain's stream, all four in one launch
            assert ask([("ranges", tiles, K, h * (4 * hl + 2 * fl))]) == [1]
            assert ask([("joined", K, 1, 0, 1, *[x for s in shapes for x in s])]) == [tile], (tile, h, fl, nl)
            assert not {TILE_64_DEALT, TILE_128_DEALT} & set(ask([("gemm", D.EPI_ACC_F32, m, n, K, 1, 0) for m, n in shapes]))


def test_attention_shapes_of_the_gpu_tests_take_both_forms(ask):
    for shapes, form in ((F.ATTN_FEW, 1), (F.ATTN_MANY, 0)):
        for b, s, nh in shapes:
            assert ask([("attention", 0, b, s, nh), ("attention", 1, b, s, nh)]) == [form, form], (b, s, nh)


def test_ranges_of_the_gpu_test(ask):
    for seq in F.RANGE_SEQS:                                   # the narrow block of test_weight_gradients_over_contraction_ranges
        h, f = 512, 2048
        tiles = sum(-(-a // 256) * -(-b // 256) for a, b in ((f, h), (h, f), (h, h), (h, 3 * h)))
        assert ask([("ranges", tiles, 16 * seq, h * (4 * h + 2 * f))])[0] > 1


def test_shapes_of_the_other_gpu_tests_take_the_forms_that_these_name(ask):
    import test_gpu_attention_own_d as A
    import test_gpu_joined_sums as J
    import test_gpu_operand_rings as R
    for shapes, few in ((A.OWN, 1), (A.PASS[:-1], 0), (A.PASS[-1:], 1)):
        assert [ask([("attention", 1, *x)])[0] for x in shapes] == [few] * len(shapes)
    assert all(s <= 256 for _, s, _ in A.OWN) and A.PASS[-1][1] == 257         # attention_owns_d
    assert set(ask([("gemm", e, *R.TILES_192x256, K, 1, 0) for e in (D.EPI_STORE, D.EPI_ACC_F32) for K in R.DEPTHS])) == {7}
    ranges = []
    for h, _, tp, f, b, s, _ in J.BLOCKS:
        shapes = [(f // tp, h), (h, f // tp), (h // tp, h), (h, 3 * h // tp)]
        tiles = sum(-(-m // 256) * -(-n // 256) for m, n in shapes)
        ranges += ask([("ranges", tiles, b * s, sum(m * n for m, n in shapes))]) if tiles <= 200 else [1]      # beside the chain: one
    assert ranges == [5, 1, 1, 1]


# (hidden, ffn columns, batch, seq) of blocks whose MLP-down product was dealt with the block output in its epilogue and not
# without: 4 x 66 tokens of the Llama-2 7B shard, 16 x 257 of the smallest GPT block
ORDER_OF_BLOCK_OUTPUT = [(4096, 1376, 4, 66), (256, 512, 16, 257), (256, 48, 1, 233)]


def test_a_block_sums_alike_alone_and_in_a_stack(ask):
    """The last block of a stack, and a block alone, form the block output in the MLP-down product; the other blocks of a
    stack run the plain product.  Results are bitwise the same only if both deal the contraction in the same way."""
    rng = random.Random(5)
    order = lambda f: f if f in (TILE_64_DEALT, TILE_128_DEALT) else "whole"
    shapes = [(b * s, h, fl) for h, fl, b, s in ORDER_OF_BLOCK_OUTPUT]
    shapes += [(rng.randrange(60, 9000), rng.randrange(4, 129) * 64, rng.randrange(4, 400) * 8) for _ in range(4000)]
    for c in (1, 2, 4):
        plain, out = (ask([("gemm", e, *x, c, 0) for x in shapes]) for e in (D.EPI_STORE, EPI_RESID))
        assert [x for x, f, g in zip(shapes, plain, out) if order(f) != order(g)] == []


def test_weight_gradients_that_add_take_another_tile_and_the_same_order(ask):
    """Adding to what the gradients hold costs the forms differently, so it may move a launch to another whole tile (192 tokens
    of a 6144-wide shard, 256 of a 1536-wide one: back to 128x128), which sums alike.  It never decides whether the
    contraction is dealt: with gradients that hold zeros, adding and overwriting stay the same bit for bit."""
    four = lambda h, hl, fl: [fl, h, h, fl, hl, h, h, 3 * hl]
    for K, sizes, over in ((192, (6144, 768, 3072), 7), (256, (1536, 384, 1536), 1)):
        assert ask([("joined", K, 1, 0, 1, *four(*sizes), beta) for beta in (0, 1)]) == [over, 0], (K, sizes)
    rng = random.Random(9)
    order = lambda f: f if f in (TILE_64_DEALT, TILE_128_DEALT) else "whole"
    shapes = [(rng.randrange(64, 8000), [rng.randrange(8, 600) * 8 for _ in range(8)], c) for _ in range(1000) for c in (1, 2, 3)]
    over, adds = (ask([("joined", K, c, 0, 1, *mn, beta) for K, mn, c in shapes]) for beta in (0, 1))
    assert [s for s, f, g in zip(shapes, over, adds) if order(f) != order(g)] == []
    singles = [(rng.randrange(8, 900) * 8, rng.randrange(8, 900) * 8, rng.randrange(8, 900) * 8) for _ in range(2000)]
    over, adds = (ask([("gemm", D.EPI_ACC_F32, *s, 1, 0, beta) for s in singles]) for beta in (0, 1))
    assert [s for s, f, g in zip(singles, over, adds) if order(f) != order(g)] == []


def test_whether_a_contraction_is_dealt_does_not_depend_on_the_streams(ask):
    """The dealt forms sum in another order than the rest, which all sum alike: only whether one is taken may matter, and
    products that share the chip with others never take one."""
    rng = random.Random(2409)
    dealt = lambda f: f in (TILE_64_DEALT, TILE_128_DEALT)
    log = lambda lo, hi: int(lo * (hi / lo) ** rng.random()) // 8 * 8
    taken = 0
    for _ in range(300):
        e, M, N, K = rng.choice((0, 1, 2, 3, 4, 5, 6)), log(64, 32768), log(64, 32768), log(64, 32768)
        forms = ask([("gemm", e, M, N, K, c, 0) for c in (1, 2, 3, 4, 8)])
        assert len({dealt(f) for f in forms}) == 1, (e, M, N, K, forms)
        assert len({f for f in forms if dealt(f)}) <= 1, (e, M, N, K, forms)
        assert not dealt(ask([("gemm", e, M, N, K, 1, 1)])[0])
        taken += dealt(forms[0])
    assert 30 < taken < 270


def test_shapes_of_the_gpu_test_take_both_orders_of_a_tile(ask):
    """... of the 128-position attention forward, in whole and cut down to the batch elements that they are compared with."""
    import test_gpu_attention_serial as S
    for d, b, s, nh, few in S.SHAPES:
        assert ask([("attention", 0, b, s, nh), ("serial", d, b, s, nh)]) == [0, 1], (d, b, s, nh)
        if few:
            assert ask([("attention", 0, few, s, nh), ("serial", d, few, s, nh)]) == [0, 0], (d, few, s, nh)
    for d, b, s, nh in ((64, 128, 512, 1), (64, 256, 128, 1), (64, 104, 257, 1), (64, 8, 4096, 1), (64, 128, 1024, 1), (80, 640, 65, 1), (128, 256, 128, 1), (128, 513, 128, 1), (128, 400, 129, 1)):
        assert ask([("serial", d, b, s, nh)]) == [0], (d, b, s, nh)


def test_views_of_the_attention_forward_stay_inside_the_matrix(ask):
    """Any row pitch that the entry point takes (a matrix under 2 GiB), also one so wide that 64 rows of it are more than
    31 bits of bytes: no view begins before the matrix or ends behind the last row that is needed."""
    shapes = []
    for ld in (384, 3072, 24576, (1 << 24) - 8, 1 << 24, (1 << 24) + 8, 3 << 23, (1 << 25) + 8, (1 << 26) + 64, (1 << 29) - 8):
        most = ((1 << 30) - 1) // ld
        shapes += [(seq, ld, d) for seq in {1, 2, 3, 63, 64, 65, 200, most} if 1 <= seq <= most for d in (64, 80, 128)]
    reach = ask([("walk", seq, ld, d, (seq + 63) // 64) for seq, ld, d in shapes])
    for (seq, ld, d), end in zip(shapes, reach):
        assert end == ((seq - 1) * ld + d) * 2, (seq, ld, d)
