"""Norms of launches that outgrow the last-level cache (2^24 values and more), whose rows go past the caches: each row bit for
bit what a launch of few rows gives, whose parity test_gpu_kernels.py covers; column sums against 64 bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (rows, h): the line itself and one row under it (a power of two and not), the narrowest row, ragged rows, one row an iteration
SHAPES = [(4096, 4096), (4095, 4096), (2097152, 8), (6557, 2560), (6553, 2560), (2341, 7168), (2049, 8192)]


@pytest.fixture(scope="module")
def dom():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_15241_amd import domino
    domino.load()
    return domino


def draw(*shape, std=1.0, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed + shape[0] + 7 * shape[-1])
    return (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)


def some_rows(rows):
    """Rows of small launches: the first, the last and some between."""
    n = min(rows, 160)
    return [(a, n) for a in sorted({0, (rows - n) // 2, rows - n})]


@pytest.mark.parametrize("rms", [0, 1])
@pytest.mark.parametrize("rows,h", SHAPES)
def test_forward(dom, rms, rows, h):
    x, a1, a2 = draw(rows, h), draw(rows, h, std=0.5, seed=1), draw(rows, h, std=0.5, seed=2)
    vec, g, b = draw(h, std=0.1, seed=3), draw(h, seed=4), None if rms else draw(h, std=0.1, seed=5)

    def run(fused, a, n):
        y, xs = torch.empty(n, h, dtype=torch.bfloat16, device="cuda"), torch.zeros(n, h, dtype=torch.bfloat16, device="cuda")
        mean, rstd = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
        sl = lambda t: t[a:a + n] if fused else None
        dom.domino_norm_fwd(x[a:a + n], sl(a1), sl(a2), vec if fused else None, g, b, xs if fused else None, y, mean, rstd, n, h, rms, 1e-5)
        return y, xs, mean, rstd
    for fused in (False, True):
        whole = run(fused, 0, rows)
        for a, n in some_rows(rows):
            for got, want in zip(whole, run(fused, a, n)):
                assert torch.equal(got[a:a + n], want)


@pytest.mark.parametrize("rms", [0, 1])
@pytest.mark.parametrize("rows,h", SHAPES)
def test_backward(dom, rms, rows, h):
    x, ga, gb, dres = draw(rows, h), draw(rows, h, seed=1), draw(rows, h, std=0.5, seed=2), draw(rows, h, seed=3)
    g = draw(h, seed=4)
    mean, rstd = 0.1 * torch.randn(rows, device="cuda"), 0.5 + torch.rand(rows, device="cuda")

    def run(a, n):
        dx, dg, db = torch.empty(n, h, dtype=torch.bfloat16, device="cuda"), torch.zeros(h, device="cuda"), torch.zeros(h, device="cuda")
        scratch = torch.empty(dom.domino_norm_bwd_scratch_floats(n, h), device="cuda")
        dom.domino_norm_bwd(ga[a:a + n], gb[a:a + n], x[a:a + n], g, mean[a:a + n], rstd[a:a + n], dres[a:a + n], dx, dg,
                            None if rms else db, scratch, n, h, rms)
        return dx, dg, db
    dx, dg, db = run(0, rows)
    for a, n in some_rows(rows):
        assert torch.equal(dx[a:a + n], run(a, n)[0])
    # column sums of up to 2^21 rows in fp32, partial sums first: 1e-5 of their 2-norm
    rdg, rdb = torch.zeros(h, dtype=torch.float64, device="cuda"), torch.zeros(h, dtype=torch.float64, device="cuda")
    for a in range(0, rows, 1 << 17):
        s = slice(a, a + (1 << 17))
        gsum = ga[s].double() + gb[s].double()
        xh = (x[s].double() - (0 if rms else mean[s].double()[:, None])) * rstd[s].double()[:, None]
        rdg += (gsum * xh).sum(0)
        rdb += gsum.sum(0)
    assert (dg.double() - rdg).norm() <= 1e-5 * rdg.norm()
    if not rms:
        assert (db.double() - rdb).norm() <= 1e-5 * rdb.norm()
