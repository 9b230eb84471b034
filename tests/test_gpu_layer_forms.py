"""Linear-layer norms and clipped sums over every form of operand the entry
points accept: any sequence length, any width, rows of any alignment, both
dtypes, few examples and many. Every operand sits inside a larger buffer of
NaNs, so that a value used from outside the matrix shows in the result. The
reference is the per-example gradient in fp64.

Bounds: products of bf16 operands are exact in fp32 and products of fp32
operands round to 2^-24; a result is a sum of n <= 2^13 such terms accumulated
in fp32, whose relative error for random terms is about sqrt(n) * 2^-24
(5e-6); 1e-5 is the 2-norm bound below. Where clip factors scale bf16 rows
(the SCALED and ROWS forms, see sum_bound), each c_i A rounds to bf16: 2^-9 per
element at most, which the 2-norm of the sum keeps (5e-3 covers it).
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def matrix(g, B, T, w, ld, off, dtype, std=1.0):
    """[B, T, w] view, row stride ld, `off` elements into a NaN-filled buffer."""
    buf = torch.full((off + B * T * ld + 64,), float("nan"), device="cuda", dtype=dtype)
    v = buf[off:off + B * T * ld].view(B, T, ld)[:, :, :w]
    v.copy_((torch.randn(B, T, w, generator=g, device="cuda") * std).to(dtype))
    return v


def operands(seed, B, T, di, do, dtype, lda, ldg, off):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (matrix(g, B, T, di, lda, off, dtype), matrix(g, B, T, do, ldg, off, dtype, 0.1), g)


def per_example(A, G):
    return torch.stack([A[b].double().t() @ G[b].double() for b in range(A.shape[0])])


SHAPES = [
    # B, T, d_in, d_out
    (1, 1, 1, 1), (2, 7, 5, 9), (3, 16, 64, 64), (4, 31, 40, 257), (2, 33, 72, 130),
    (5, 64, 256, 96), (3, 100, 129, 511), (2, 128, 256, 320), (2, 130, 513, 64),
    (1, 200, 33, 700), (2, 257, 96, 264), (1, 300, 520, 48), (24, 40, 64, 200), (3, 96, 768, 1030),
]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows", ["aligned", "odd"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_norms_of_every_form(shape, rows, dtype):
    from paper_2609_40335_amd import dpghost as dp
    B, T, di, do = shape
    up = (lambda w: (w + 7) // 8 * 8) if rows == "aligned" else (lambda w: w + (1 - w % 2))
    off = 0 if rows == "aligned" else 3
    A, G, _ = operands(1, B, T, di, do, dtype, up(di), up(do), off)
    want = per_example(A, G).square().sum((1, 2))
    for algo in (dp.DP_NORM_GRAM, dp.DP_NORM_DIRECT):
        n2 = torch.full((B,), float("nan"), device="cuda")
        dp.dp_ghost_norm_linear(A, G, n2, algo=algo)
        torch.testing.assert_close(n2.double(), want, rtol=1e-5, atol=0, msg=lambda m: f"{algo}: {m}")
    # in a group with its bias: the same norm plus the bias's
    bias = torch.full((B, do), float("nan"), device="cuda")
    n2 = torch.full((B,), float("nan"), device="cuda")
    dp.dp_ghost_norm_linear_bias_grouped([(A, G, dp.DP_NORM_GRAM)], [bias], n2)
    bw = G.double().sum(1)
    torch.testing.assert_close(bias.double(), bw, rtol=1e-4, atol=1e-5 * float(bw.abs().max()) + 1e-6)
    torch.testing.assert_close(n2.double(), want + bw.square().sum(1), rtol=1e-5, atol=0)


def sum_bound(T, dtype):
    """2-norm bound of a clipped sum. bf16 rows are scaled where padding examples to whole
    stages of 32 rows would take more than 3/2 of their rows (sum_form, ROWS_NUM / ROWS_DEN);
    elsewhere the factors scale in fp32."""
    padded = -(-T // 32) * 32
    return 5e-3 if dtype == torch.bfloat16 and 2 * padded > 3 * T else 1e-5


def factors(B):
    c = torch.linspace(0.05, 1.0, B, device="cuda")
    if B > 2:
        c[1] = 0.0   # an example that is left out
    return c


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows", ["aligned", "odd"])
@pytest.mark.parametrize("shape", SHAPES + [(300, 3, 24, 40), (5000, 1, 16, 16), (4100, 32, 8, 24)],
                         ids=lambda s: "x".join(map(str, s)))
def test_clipped_sums_of_every_form(shape, rows, dtype):
    from paper_2609_40335_amd import dpghost as dp
    B, T, di, do = shape
    up = (lambda w: (w + 7) // 8 * 8) if rows == "aligned" else (lambda w: w + (1 - w % 2))
    off = 0 if rows == "aligned" else 3
    A, G, g = operands(2, B, T, di, do, dtype, up(di), up(do), off)
    c = factors(B)
    if B > 2:
        A[1] = float("inf")   # left out, whatever it holds
    Ac = torch.where(c.view(B, 1, 1) == 0, 0.0, A.double()) * c.double().view(B, 1, 1)
    want = torch.einsum("km,kn->mn", Ac.reshape(B * T, di), G.double().reshape(B * T, do))
    bound = sum_bound(T, dtype)
    prior = torch.randn(di, do, generator=g, device="cuda")
    for transpose in (False, True):
        w = want.t() if transpose else want
        out = torch.full(tuple(w.shape), float("nan"), device="cuda")
        dp.dp_clipped_grad_sum(A, G, c, out, transpose_out=transpose)
        rel = float((out.double() - w).norm() / w.norm())
        assert rel < bound, (transpose, rel)
        out.copy_(prior.t() if transpose else prior)
        dp.dp_clipped_grad_sum(A, G, c, out, transpose_out=transpose, accumulate=True)
        w2 = w + (prior.t() if transpose else prior).double()
        assert float((out.double() - w2).norm() / w2.norm()) < bound
    # the same with the noise fused, against the sum and the noise apart
    grp = dp.LinearGroup([(A, G)], [torch.full((di, do), float("nan"), device="cuda")])
    grp.clipped_sum_noised(c, [5], 0.5, 1.0, 3, 11, 2)
    z = torch.zeros(di, do, device="cuda")
    dp.dp_add_noise(z, 0.5, 1.0, 0, 11, 5, 2)
    w3 = (want + z.double()) / 3
    assert float((grp._outs[0].double() - w3).norm() / w3.norm()) < bound


@pytest.mark.parametrize("span", [0, 30], ids=["ordinary", "wide"])
def test_fp32_products_keep_their_bits(span):
    """One token, so that every output is one product of two fp32 values, over
    2 * span + 1 binary orders. A product of values cut into bf16 planes leaves out
    terms of at most 2^-22 of it (a plane kept too few would show as 2^-16);
    the norm is a product of two such sums over 300 and 260 features."""
    from paper_2609_40335_amd import dpghost as dp
    g = torch.Generator(device="cuda").manual_seed(9)

    def values(w):
        x = torch.randn(1, 1, w, generator=g, device="cuda")
        return x * torch.exp2(torch.randint(-span, span + 1, (1, 1, w), generator=g, device="cuda").float())

    A, G = values(300), values(260) * 2.0 ** -span   # (the norm must not overflow)
    out = torch.zeros(300, 260, device="cuda")
    dp.dp_clipped_grad_sum(A, G, torch.ones(1, device="cuda"), out)
    want = A.double().view(-1, 1) * G.double().view(1, -1)
    assert float(((out.double() - want) / want).abs().max()) <= 2.0 ** -21
    for algo in (dp.DP_NORM_GRAM, dp.DP_NORM_DIRECT):
        n2 = torch.zeros(1, device="cuda")
        dp.dp_ghost_norm_linear(A, G, n2, algo=algo)
        assert abs(float(n2) / float(want.square().sum()) - 1) <= 2.0 ** -19


# B, T, d_in, d_out: forms of the sum whose last round is split over K (a few tiles, long K;
# T a multiple of a stage or not; ranges that start inside an example)
SPLIT = [(6, 160, 300, 264), (5, 100, 264, 300), (150, 9, 64, 320), (3, 515, 512, 40)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows", ["aligned", "odd"])
@pytest.mark.parametrize("shape", SPLIT, ids=lambda s: "x".join(map(str, s)))
def test_split_sums_of_every_form(shape, rows, dtype):
    """LinearGroup and the single call split few tiles over K and add the parts (fp32: the
    same sum in another order, so the bound of the unsplit sum)."""
    from paper_2609_40335_amd import dpghost as dp
    B, T, di, do = shape
    up = (lambda w: (w + 7) // 8 * 8) if rows == "aligned" else (lambda w: w + (1 - w % 2))
    A, G, g = operands(3, B, T, di, do, dtype, up(di), up(do), 0 if rows == "aligned" else 3)
    c = factors(B)
    A[1] = float("inf")
    Ac = torch.where(c.view(B, 1, 1) == 0, 0.0, A.double()) * c.double().view(B, 1, 1)
    want = torch.einsum("km,kn->mn", Ac.reshape(B * T, di), G.double().reshape(B * T, do))
    bound = sum_bound(T, dtype)
    grp = dp.LinearGroup([(A, G)], [torch.full((di, do), float("nan"), device="cuda")])
    grp.clipped_sum(c)
    assert grp._split_ws is not None
    assert float((grp._outs[0].double() - want).norm() / want.norm()) < bound
    grp.clipped_sum_noised(c, [5], 0.5, 1.0, 3, 11, 2)
    z = torch.zeros(di, do, device="cuda")
    dp.dp_add_noise(z, 0.5, 1.0, 0, 11, 5, 2)
    w = (want + z.double()) / 3
    assert float((grp._outs[0].double() - w).norm() / w.norm()) < bound
    out = torch.randn(do, di, generator=g, device="cuda")
    w = want.t() + out.double()
    dp.dp_clipped_grad_sum(A, G, c, out, transpose_out=True, accumulate=True)
    assert float((out.double() - w).norm() / w.norm()) < bound


@pytest.mark.parametrize("B,T,di,do", [(600, 7, 40, 72), (40, 21, 264, 64), (64, 40, 64, 300)],
                         ids=lambda s: str(s))
def test_each_call_scales_by_its_own_factors(B, T, di, do):
    """Short bf16 sequences, whose rows are scaled from the factor table while they are
    staged: calls queued back to back, each with other factors, so that factors of an earlier
    call (or a table that is not yet filled) would show. One example of the first 64 rows is
    left out and holds inf. B = 600 takes two rounds of 512 threads to fill the table."""
    from paper_2609_40335_amd import dpghost as dp
    A, G, g = operands(4, B, T, di, do, torch.bfloat16, di, do, 0)
    cs, outs = [], []
    for i in range(12):
        c = torch.rand(B, device="cuda", generator=g) * 0.9 + 0.1
        c[i % 3] = 0.0
        cs.append(c)
        outs.append(torch.full((di, do), float("nan"), device="cuda"))
    inputs = []
    for i in range(3):
        Ai = A.clone()
        Ai[i] = float("inf")
        inputs.append(Ai)
    for i in range(12):
        dp.dp_clipped_grad_sum(inputs[i % 3], G, cs[i], outs[i])
    for i in range(12):
        c = cs[i].double().view(B, 1, 1)
        Ac = torch.where(c == 0, 0.0, A.double()) * c
        want = Ac.reshape(B * T, di).t() @ G.double().reshape(B * T, do)
        rel = float((outs[i].double() - want).norm() / want.norm())
        assert rel < 5e-3, (i, rel)


def test_split_sums_on_two_streams_and_in_a_graph():
    """Split sums queued on the current stream and, by `stream`, on another at the same time,
    then a captured one replayed on the second stream beside eager calls on the first: every
    call has partial tiles of its own, so each result keeps its bits."""
    from paper_2609_40335_amd import dpghost as dp
    B, T, di, do = 24, 128, 768, 768
    sets = []
    for seed in (5, 6):
        A, G, _ = operands(seed, B, T, di, do, torch.bfloat16, di, do, 0)
        sets.append((A, G, torch.linspace(0.05 * seed, 1.0, B, device="cuda")))
    grps = [dp.LinearGroup([(A, G)], [torch.zeros(di, do, device="cuda")]) for A, G, _ in sets]
    want = []
    for (A, G, c), grp in zip(sets, grps):
        grp.clipped_sum(c)
        assert grp._split_ws is not None
        want.append(grp._outs[0].clone())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    outs = [[torch.zeros(di, do, device="cuda") for _ in range(8)] for _ in sets]
    torch.cuda.synchronize()
    for i in range(8):
        for k, (A, G, c) in enumerate(sets):
            dp.dp_clipped_grad_sum(A, G, c, outs[k][i], stream=side if k else None)
    torch.cuda.synchronize()
    for k in range(2):
        for o in outs[k]:
            assert torch.equal(o, want[k])
    graph = torch.cuda.CUDAGraph()
    grps[1].clipped_sum(sets[1][2], stream=side)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        grps[1].clipped_sum(sets[1][2], stream=side)
    for i in range(4):
        for grp in grps:
            grp._outs[0].fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
        for _ in range(3):
            grps[0].clipped_sum(sets[0][2])
        torch.cuda.synchronize()
        for grp, w in zip(grps, want):
            assert torch.equal(grp._outs[0], w)


@pytest.mark.parametrize("exponent", [0, -100, -125], ids=["ordinary", "small", "near-denormal"])
def test_fp32_products_are_off_by_two_roundings(exponent):
    """One token and a factor of 1, so that every output is one product: the plane
    products that are left out are at most 2^-24 of it, and the kept ones are added with
    one rounding, 2^-24 again (what cutting the small ones' sum adds is below 2^-30).
    Values too small for exact bf16 planes (below 2^-110) keep the same bound, up to the
    outputs' own denormal spacing."""
    from paper_2609_40335_amd import dpghost as dp
    g = torch.Generator(device="cuda").manual_seed(10)
    A = torch.randn(1, 1, 300, generator=g, device="cuda")
    G = torch.randn(1, 1, 260, generator=g, device="cuda") * 2.0 ** exponent
    out = torch.zeros(300, 260, device="cuda")
    dp.dp_clipped_grad_sum(A, G, torch.ones(1, device="cuda"), out)
    want = A.double().view(-1, 1) * G.double().view(1, -1)
    err = (out.double() - want).abs() - 2.0 ** -149
    assert float((err / want.abs()).max()) <= 2.0 ** -23 * 1.02


ONE_SIGN = {
    "softmax": lambda r: torch.softmax(r, -1),
    "gelu": torch.nn.functional.gelu,
    "positive": torch.abs,
    "third": lambda r: torch.full_like(r, 1 / 3),
}


@pytest.mark.parametrize("T", [16, 128, 1024])
@pytest.mark.parametrize("kinds", [("gelu", "softmax"), ("third", "positive"), ("positive", "positive")],
                         ids="-".join)
def test_fp32_sums_of_one_sign(kinds, T):
    """Operands of one sign, where every cut of a partial sum adds up. A sum of T tokens is n =
    2 T / 16 additions, each off by at most 2^-24 of the running value, either way: 2^-24
    / sqrt(3) as a root mean square, times sqrt(n / 3) for a value that grows evenly; and each
    stage's products are cut one way, by 2^-24 of them at most. (Clipped sums add six times a
    stage, the small products among them: no more than twice as many roundings.) Over the matrix the
    additions' errors average out of a norm, which keeps twice that cut and the roundings of
    its own last additions: 1.5e-7 as a root mean square over the examples. (With the plane
    products on the running accumulator, direct norms were at 2e-7 to 7e-7 for T = 1024.)"""
    from paper_2609_40335_amd import dpghost as dp
    B, di, do = 64, 96, 80
    g = torch.Generator(device="cuda").manual_seed(12)
    A = ONE_SIGN[kinds[0]](torch.randn(B, T, di, generator=g, device="cuda"))
    G = ONE_SIGN[kinds[1]](torch.randn(B, T, do, generator=g, device="cuda"))
    P = per_example(A, G)
    want = P.square().sum((1, 2))
    for algo in (dp.DP_NORM_DIRECT,) + ((dp.DP_NORM_GRAM,) if T <= 128 else ()):
        n2 = torch.zeros(B, device="cuda")
        dp.dp_ghost_norm_linear(A, G, n2, algo=algo)
        assert float(((n2.double() - want) / want).square().mean().sqrt()) < 1.5e-7, algo
    bound = 2.0 ** -24 * (1 + (2 * T / 16 / 9) ** 0.5)
    for b in range(3):
        out = torch.zeros(di, do, device="cuda")
        dp.dp_clipped_grad_sum(A[b:b + 1], G[b:b + 1], torch.ones(1, device="cuda"), out)
        assert float((out.double() - P[b]).norm() / P[b].norm()) < bound


@pytest.mark.parametrize("shape", [(3, 1, 40, 50), (3, 5, 40, 300), (3, 100, 300, 72), (3, 130, 64, 64)],
                         ids=lambda s: "x".join(map(str, s)))
def test_fp32_infinities_and_overflow(shape):
    """What fp32 products and sums give: an infinite operand makes infinities of its products'
    signs, a product too large an infinity, NaN stays NaN, an example with c = 0 is left out;
    norms of overflowing examples are infinite, the other examples' untouched."""
    from paper_2609_40335_amd import dpghost as dp
    B, T, di, do = shape
    g = torch.Generator(device="cuda").manual_seed(13)
    A = torch.randn(B, T, di, generator=g, device="cuda")
    G = torch.randn(B, T, do, generator=g, device="cuda")
    c = torch.tensor([1.0, 0.5, 0.7], device="cuda")
    inf = float("inf")
    cases = {"inf": A.clone(), "overflow": A.clone(), "largest": A.clone(), "nan": A.clone()}
    cases["inf"][1, 0, 3] = inf
    cases["overflow"][1] = A[1].abs() * 1e25
    cases["largest"][1, 0, 5] = 3.4e38     # rounds to infinity in bf16
    cases["nan"][1, T - 1, 0] = float("nan")
    for name, X in cases.items():
        Y = G.clone()
        if name == "overflow":
            Y[1] = G[1].abs() * 1e14
        if name == "largest":
            Y[1] *= 1e-30
        want = (per_example(X, Y) * c.double().view(B, 1, 1)).sum(0).float()
        out = torch.zeros(di, do, device="cuda")
        dp.dp_clipped_grad_sum(X, Y, c, out)
        grp = dp.LinearGroup([(X, Y)], [torch.zeros(di, do, device="cuda")])
        grp.clipped_sum(c)
        for got in (out, grp._outs[0]):
            assert torch.equal(got == inf, want == inf), name
            assert torch.equal(got == -inf, want == -inf), name
            assert torch.equal(got.isnan(), want.isnan()), name
            ok = want.isfinite()
            if ok.any():
                assert float((got[ok].double() - want[ok].double()).norm()
                             / want[ok].double().norm()) < 1e-5, name
        c0 = torch.tensor([1.0, 0.0, 0.7], device="cuda")
        dp.dp_clipped_grad_sum(X, Y, c0, out)
        w0 = (per_example(A, G)[[0, 2]] * c0[[0, 2]].double().view(2, 1, 1)).sum(0)
        assert float((out.double() - w0).norm() / w0.norm()) < 1e-5, name
        n2w = per_example(A, G).square().sum((1, 2))
        for algo in (dp.DP_NORM_GRAM, dp.DP_NORM_DIRECT):
            n2 = torch.zeros(B, device="cuda")
            dp.dp_ghost_norm_linear(X, Y, n2, algo=algo)
            for b in (0, 2):
                assert abs(float(n2[b]) / float(n2w[b]) - 1) < 1e-5, name
            if name == "overflow":
                assert float(n2[1]) == inf, algo
            elif name == "nan":
                assert bool(n2[1].isnan()), algo
            elif name == "inf":
                assert not bool(n2[1].isfinite()), algo


def test_linear_form_leaves_its_workspace_alone():
    """dp_clipped_grad_sum's linear form takes no workspace: one that a caller passes
    (the argument serves the embedding form) is not written, whatever its size."""
    from paper_2609_40335_amd import dpghost as dp
    B, T, di, do = 6, 160, 300, 264
    A, G, _ = operands(7, B, T, di, do, torch.bfloat16, 304, 264, 0)
    c = factors(B)
    out = torch.zeros(di, do, device="cuda")
    desc = (dp.dp_linear_t * 1)(dp._layer(A, G))
    L = dp.lib()
    nbytes = L.dp_clipped_grad_sum_split_workspace(desc, 1, B, T, dp.DP_BF16, 0)
    assert nbytes > 0
    ws = torch.full((nbytes,), 0xAB, dtype=torch.uint8, device="cuda")
    d = desc[0]
    st = L.dp_clipped_grad_sum(d.A, d.lda, d.G, d.ldg, None, c.data_ptr(), B, T, di, do, dp.DP_BF16,
                               0, out.data_ptr(), 0, ws.data_ptr(), ws.numel(), dp._stream(None))
    assert st == 0
    assert bool((ws == 0xAB).all())
    want = (per_example(A, G) * c.double().view(B, 1, 1)).sum(0)
    assert float((out.double() - want).norm() / want.norm()) < 1e-5


@pytest.mark.parametrize("B,T,shapes,split", [
    (1, 256, [(768, 2304), (768, 768), (768, 3072), (3072, 768)], False),   # 108 tiles of 8 stages
    (10, 24, [(768, 2304), (768, 768), (768, 3072), (3072, 768)], False),   # short examples
    (24, 128, [(768, 3072)], True),                                         # 36 tiles of 96
], ids=["short-sums", "short-examples", "long-sums"])
def test_sums_are_split_only_where_that_pays(B, T, shapes, split):
    """Partial tiles cost their way to memory and back, so many tiles of short sums write
    none, whatever workspace they are given; few tiles of long sums do."""
    import ctypes
    from paper_2609_40335_amd import dpghost as dp
    L = dp.lib()
    layers = [operands(8 + i, B, T, a, b, torch.bfloat16, a, b, 0)[:2] for i, (a, b) in enumerate(shapes)]
    outs = [torch.zeros(a, b, device="cuda") for a, b in shapes]
    descs = (dp.dp_linear_t * len(shapes))(*[dp._layer(*l) for l in layers])
    ptrs = (ctypes.c_void_p * len(shapes))(*[o.data_ptr() for o in outs])
    c = torch.ones(B, device="cuda")
    ws = torch.full((256 * 256 * 256 * 4,), 0xAB, dtype=torch.uint8, device="cuda")
    st = L.dp_clipped_grad_sum_grouped_ws(descs, ptrs, len(shapes), c.data_ptr(), B, T, dp.DP_BF16, 0,
                                          0, ws.data_ptr(), ws.numel(), dp._stream(None))
    assert st == 0
    assert bool((ws == 0xAB).all()) != split
    for (A, G), o in zip(layers, outs):
        want = per_example(A, G).sum(0)
        assert float((o.double() - want).norm() / want.norm()) < 1e-5
