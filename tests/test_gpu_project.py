"""The projection kernel at the edges of its tiles and of its k-steps: every tile shape the launcher picks from,
rows and columns that end inside a tile, one k-step, half a k-step, and steps around the depth of its load ring."""
import pytest
import torch

from paper_2601_17818_amd import binding as vc

pytestmark = pytest.mark.gpu


def check(x, w, y, residual=None):
    """Within half a bf16 ulp (2^-8 of the value) of double precision, plus the fp32 sums' own error: at most one
    rounding of 2^-24 of the running sum per term, which sum |x w| bounds."""
    ref = x.double() @ w.double().T
    mass = x.double().abs() @ w.double().abs().T
    if residual is not None:
        ref += residual.double()
        mass += residual.double().abs()
    bound = 2.0 ** -8 * ref.abs() + x.shape[1] * 2.0 ** -24 * mass
    assert bool(((y.double() - ref).abs() <= bound).all())


def draw(M, N, K, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.empty((M, K), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    w = torch.empty((N, K), dtype=torch.bfloat16, device="cuda").normal_(0, K ** -0.5, generator=g)
    r = torch.empty((M, N), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    return x, w, r


@pytest.mark.parametrize("M,N", [(4096, 4096), (4001, 4016), (1537, 4096), (3000, 4096), (3100, 2064), (1500, 1040),
                                 (700, 2048), (260, 528), (5, 48)])
@pytest.mark.parametrize("K", [32, 64, 96, 128, 160, 224, 256, 288])
def test_tiles_and_k_steps(M, N, K):
    x, w, r = draw(M, N, K, M + K)
    y, _ = vc.vitcop_project(x, w, residual=r, scratch=False)
    check(x, w, y, r)
    y, parts = vc.vitcop_project(x, w, want_sumsq=True, scratch=False)
    check(x, w, y)
    sq = torch.nn.functional.pad(y.double() ** 2, (0, -N % 128)).reshape(M, -1, 128).sum(-1).T
    # fp32 sums of 128 squares
    assert bool(((parts.double() - sq).abs() <= 128 * 2.0 ** -24 * sq + 1e-30).all())


# (test_plan_cpu.py checks that these shapes are cut, and that the lists of this file reach every sliced tile)
SPLIT_K = [(257, 512, 4096), (317, 4096, 4064), (640, 4096, 4096), (1024, 1040, 4128), (500, 2064, 3008),
           (327, 3840, 2304), (390, 3840, 3584), (257, 8448, 4608), (327, 5632, 8448), (390, 5632, 8448)]


@pytest.mark.parametrize("M,N,K", SPLIT_K)
def test_split_k(M, N, K):
    assert vc.lib.vitcop_project_workspace_bytes(M, N, K) > 0
    x, w, r = draw(M, N, K, M)
    y, _ = vc.vitcop_project(x, w, residual=r)
    check(x, w, y, r)


SPLIT_TALL = [(1025, 512, 4096), (1500, 3584, 14336), (1300, 1040, 4128), (1536, 2048, 5632), (1500, 272, 2048)]


@pytest.mark.parametrize("M,N,K", SPLIT_TALL)
def test_slices_of_tall_launches(M, N, K):
    x, w, r = draw(M, N, K, M)
    y, _ = vc.vitcop_project(x, w, residual=r)
    check(x, w, y, r)
    y, parts = vc.vitcop_project(x, w, want_sumsq=True)
    check(x, w, y)
    sq = torch.nn.functional.pad(y.double() ** 2, (0, -N % 128)).reshape(M, -1, 128).sum(-1).T
    assert bool(((parts.double() - sq).abs() <= 128 * 2.0 ** -24 * sq + 1e-30).all())


# slices of 32 k-steps and more start at different k and wrap around with one or two tile rows, and stay in step with more;
# a last step of half a step in the middle of the walk (test_plan_cpu.py checks their length and their tile rows)
SPREAD_SLICES = [(20, 4096, 8192), (64, 4096, 12288), (100, 8192, 8192), (250, 8192, 8192), (300, 4096, 8224), (300, 8192, 8224),
                 (380, 4144, 8224), (420, 8448, 8448)]
LONG_SLICES = SPREAD_SLICES + [(700, 4096, 12320), (1000, 4096, 8224), (640, 4096, 4128)]


@pytest.mark.parametrize("M,N,K", LONG_SLICES)
def test_long_slices(M, N, K):
    x, w, r = draw(M, N, K, M)
    y, _ = vc.vitcop_project(x, w, residual=r)
    check(x, w, y, r)


@pytest.mark.parametrize("M,D,Hq,Hkv,d,F", [(120, 2048, 2, 2, 128, 8320), (250, 2112, 1, 1, 128, 8320), (300, 2080, 2, 2, 128, 8320)])
def test_long_gate_up(M, D, Hq, Hkv, d, F):
    """The same walk in whole tiles of gate and up."""
    test_matrices_side_by_side(M, D, Hq, Hkv, d, F)


# (slices of two tile rows that the XCDs' ranges cut inside a column, on tiles of 160, 192 and 256 rows; few rows, three
# tile rows and more, whole tiles)
@pytest.mark.parametrize("M,N,K", [(300, 4144, 8224), (380, 4608, 11008), (420, 8448, 8448), (300, 5632, 11008), (120, 4096, 8192),
                                   (250, 8192, 8192), (1000, 4112, 8224), (1300, 1040, 4128), (2600, 4096, 1024)])
def test_equal_rows_get_equal_sums(M, N, K):
    """Wherever a row stands in a launch, its sums are added in the same order: equal samples of a batch stay equal."""
    x, w, r = draw(M // 2, N, K, M)
    y, _ = vc.vitcop_project(torch.cat([x, x]), w, residual=torch.cat([r, r]))
    assert torch.equal(y[:M // 2], y[M // 2:])


@pytest.mark.parametrize("T", [60, 150, 190, 250, 600])
@pytest.mark.parametrize("D,F", [(2080, 8320), (2048, 11008)])
def test_equal_samples_of_a_batch_stay_equal(T, D, F):
    """The same over a decoder layer that prunes: K, Q and V, gate and up in whole tiles, the kept tokens."""
    Hq, Hkv, d, keep = 4, 4, 128, T - 20
    g = torch.Generator(device="cuda").manual_seed(T + F)

    def t(*shape, std=1.0):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    w = {"ln1": t(D), "ln2": t(D), "wq": t(Hq * d, D, std=D ** -0.5), "wk": t(Hkv * d, D, std=D ** -0.5),
         "wv": t(Hkv * d, D, std=D ** -0.5), "wo": t(D, Hq * d, std=D ** -0.5), "wg": t(F, D, std=D ** -0.5),
         "wu": t(F, D, std=D ** -0.5), "wd": t(D, F, std=F ** -0.5)}
    h = t(1, T + 10, D).repeat(2, 1, 1)
    pos = torch.arange(T + 10, dtype=torch.int32, device="cuda").repeat(2, 1)
    out = vc.vitcop_decoder_layer_prefill(h, pos, w, Hq, Hkv, d, 5, T, keep)
    assert torch.equal(out["keep_idx"][0], out["keep_idx"][1])
    assert torch.equal(out["y"][0], out["y"][1])


def test_rows_past_the_end_do_not_leak_in():
    """What lies behind the last row of x in memory (here infinities) is never multiplied."""
    x, w, r = draw(300, 512, 96, 3)
    big = torch.full((400, 96), float("inf"), dtype=torch.bfloat16, device="cuda")
    big[:300] = x
    y, _ = vc.vitcop_project(big[:300], w, residual=r, scratch=False)
    check(x, w, y, r)


FEW_ROWS = [5, 32, 33, 64, 65, 100, 128, 129, 161, 193, 225, 256]
FEW_ROWS_NK = [(528, 128), (4096, 192), (1552, 2048), (16400, 256), (8256, 1152), (12352, 2048), (8320, 3456)]


@pytest.mark.parametrize("M", FEW_ROWS)
@pytest.mark.parametrize("N,K", FEW_ROWS_NK)
def test_few_rows(M, N, K):
    assert vc.lib.vitcop_project_workspace_bytes(M, N, K) > 0
    x, w, r = draw(M, N, K, M + N)
    y, _ = vc.vitcop_project(x, w, residual=r)
    check(x, w, y, r)
    y, parts = vc.vitcop_project(x, w, want_sumsq=True)
    check(x, w, y)
    sq = torch.nn.functional.pad(y.double() ** 2, (0, -N % 128)).reshape(M, -1, 128).sum(-1).T
    assert bool(((parts.double() - sq).abs() <= 128 * 2.0 ** -24 * sq + 1e-30).all())


@pytest.mark.parametrize("M", [1, 2, 3, 4])
@pytest.mark.parametrize("N,K", [(48, 512), (4096, 2048), (1040, 2080), (3008, 4128), (2064, 11008), (512, 12288)])
def test_one_to_four_rows(M, N, K):
    """Pieces of a row pair in rotated order: one to six of them, the last one short, pairs cut between wavefronts."""
    x, w, r = draw(M, N, K, M + K)
    y, _ = vc.vitcop_project(x, w, residual=r)
    check(x, w, y, r)


SIDE_BY_SIDE = ([(M, *layer) for layer in ((512, 4, 2, 64, 1408), (640, 5, 1, 128, 896), (1024, 16, 4, 64, 2816))
                 for M in (7, 40, 115, 200, 300, 700, 1100, 2900)] +
                # K, Q and V as one launch of k-slices on each of its tiles
                [(257, 512, 2, 2, 128, 256), (257, 512, 44, 11, 128, 256), (327, 512, 22, 11, 128, 256),
                 (327, 512, 44, 11, 128, 256), (481, 512, 40, 5, 128, 256)] +
                # K in k-slices of its own, Q and V as a pair in slices of 256 columns
                [(257, 5888, 36, 36, 128, 512)] +
                # gate and up of few rows in tiles of 32 + 32, 48 + 48 and 64 + 64 columns, and in k-slices
                [(M, *layer) for M, D in ((20, 7168), (50, 2048), (80, 1536), (120, 1280), (150, 1024), (180, 1024),
                                          (210, 1024), (250, 1024))
                 for layer in ((512, 1, 1, 128, 256), (256, 1, 1, 128, 8320), (256, 1, 1, 128, 12928), (D, 1, 1, 128, 128))])


@pytest.mark.parametrize("M,D,Hq,Hkv,d,F", SIDE_BY_SIDE)
def test_matrices_side_by_side(M, D, Hq, Hkv, d, F):
    """K, Q and V as one launch and gate and up as one launch: a decoder layer that keeps every token gives the values
    of its pieces called one by one (tiles that hold the end of one matrix and the start of the next)."""
    g = torch.Generator(device="cuda").manual_seed(M)

    def t(*shape, std=1.0):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    w = {"ln1": t(D), "ln2": t(D), "wq": t(Hq * d, D, std=D ** -0.5), "wk": t(Hkv * d, D, std=D ** -0.5),
         "wv": t(Hkv * d, D, std=D ** -0.5), "wo": t(D, Hq * d, std=D ** -0.5), "wg": t(F, D, std=D ** -0.5),
         "wu": t(F, D, std=D ** -0.5), "wd": t(D, F, std=F ** -0.5)}
    h, pos = t(1, M, D), torch.arange(M, dtype=torch.int32, device="cuda")[None]
    out = vc.vitcop_decoder_layer_prefill(h, pos, w, Hq, Hkv, d, 0, M, M)
    x = vc.vitcop_rmsnorm(h[0], w["ln1"])
    q, k, v = (vc.vitcop_project(x, w[n], scratch=False)[0].reshape(1, M, -1, d) for n in ("wq", "wk", "wv"))
    for name, ref in (("wq", q), ("wk", k), ("wv", v)):
        check(x, w[name], ref.reshape(M, -1))
    vc.vitcop_rope(q, k, pos)
    a = vc.vitcop_prefill_attn(q, k, v)[0].reshape(M, -1)
    h1, _ = vc.vitcop_project(a, w["wo"], residual=h[0], scratch=False)
    x2 = vc.vitcop_rmsnorm(h1, w["ln2"])
    act = vc.vitcop_silu_mul(vc.vitcop_project(x2, w["wg"], scratch=False)[0], vc.vitcop_project(x2, w["wu"], scratch=False)[0])
    y, _ = vc.vitcop_project(act, w["wd"], residual=h1, scratch=False)
    got = out["y"].reshape(M, D).double()
    # the same sums in another order: now and then a bf16 rounding falls the other way (2^-8 of an intermediate value)
    # and travels on; the two agree to a small part of that on average, and a wrong column would be off by its size
    err = (got - y.double()).abs()
    assert float(err.mean()) <= 2.0 ** -9 * float(y.double().abs().mean())
    assert float(err.max()) <= 2.0 ** -4 * max(1.0, float(y.double().abs().max()))


@pytest.mark.parametrize("B,n_vis,keep", [(1, 1500, 700), (1, 300, 120), (2, 900, 330), (1, 600, 290), (4, 3000, 720)])
def test_query_and_value_of_unequal_width(B, n_vis, keep):
    """Q and V of a pruned layer as one launch: grouped-query widths (896 + 128, 1536 + 512, 512 + 256), in every range of rows."""
    g = torch.Generator(device="cuda").manual_seed(n_vis)
    for D, Hq, Hkv, d in ((896, 7, 1, 128), (768, 12, 4, 128), (512, 8, 4, 64)):
        def t(*shape, std=1.0):
            return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
        T = n_vis + 30
        x, wq, wk, wv, wo = t(B, T, D), *(t(n, D, std=D ** -0.5) for n in (Hq * d, Hkv * d, Hkv * d)), t(D, Hq * d, std=D ** -0.5)
        r = vc.vitcop_layer_prefill(x, wq, wk, wv, wo, Hq, Hkv, d, 10, n_vis, keep)
        idx = r["keep_idx"].long()
        xs = torch.gather(x, 1, idx[:, :, None].expand(-1, -1, D))
        Tp = keep + 30
        q, k, v = (vc.vitcop_project(xs.reshape(B * Tp, D), w, scratch=False)[0].reshape(B, Tp, -1, d) for w in (wq, wk, wv))
        check(xs.reshape(-1, D), wq, q.reshape(B * Tp, -1))
        check(xs.reshape(-1, D), wv, v.reshape(B * Tp, -1))
        a = vc.vitcop_prefill_attn(q, k, v)[0]
        y, _ = vc.vitcop_project(a.reshape(B * Tp, -1), wo, scratch=False)
        got, want = r["y"].reshape(B * Tp, D).double(), y.double()
        # (another order of the fp32 sums: a bf16 rounding of q, k or v falls the other way now and then)
        assert float((got - want).norm() / want.norm()) <= 2.0 ** -7


# slices of 256 columns of 160, 192 and 256 rows, then of 128 columns
PAIRS = [(8192, 64, 8, 300), (8192, 64, 2, 257), (12288, 48, 8, 350), (12288, 48, 8, 640),
         (3328, 2, 2, 257), (2304, 28, 4, 327), (3584, 28, 4, 390)]


@pytest.mark.parametrize("D,Hq,Hkv,keep", PAIRS)
def test_query_and_value_pair_in_slices(D, Hq, Hkv, keep):
    """Q and V of pruned layers as k-slices over both matrices: the layer's output and its caches are those of Q and V
    projected one by one in whole tiles."""
    d, T = 128, keep + 100
    g = torch.Generator(device="cuda").manual_seed(keep)

    def t(*shape, std=1.0):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    x, wq, wk, wv, wo = t(1, T, D), *(t(n, D, std=D ** -0.5) for n in (Hq * d, Hkv * d, Hkv * d)), t(D, Hq * d, std=D ** -0.5)
    pos = torch.arange(T, dtype=torch.int32, device="cuda")[None]

    def pieces(xs, at):
        q, k, v = (vc.vitcop_project(xs, w, scratch=False)[0].reshape(1, keep, -1, d) for w in (wq, wk, wv))
        for w, y in ((wq, q), (wk, k), (wv, v)):
            check(xs, w, y.reshape(keep, -1))
        if at is not None:
            vc.vitcop_rope(q, k, at)
        return vc.vitcop_prefill_attn(q, k, v)[0].reshape(keep, -1), k, v
    r = vc.vitcop_layer_prefill(x, wq, wk, wv, wo, Hq, Hkv, d, 0, T, keep)
    xs = x[0, r["keep_idx"][0].long()]
    want = vc.vitcop_project(pieces(xs, None)[0], wo, scratch=False)[0].double()
    # (another order of the fp32 sums: a bf16 rounding of q, k or v falls the other way now and then)
    assert float((r["y"][0].double() - want).norm() / want.norm()) <= 2.0 ** -7

    F = 512
    w = {"ln1": t(D), "ln2": t(D), "wq": wq, "wk": wk, "wv": wv, "wo": wo, "wg": t(F, D, std=D ** -0.5),
         "wu": t(F, D, std=D ** -0.5), "wd": t(D, F, std=F ** -0.5)}
    caches = [torch.zeros((1, keep, Hkv, d), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    r = vc.vitcop_decoder_layer_prefill(x, pos, w, Hq, Hkv, d, 0, T, keep, caches=caches)
    idx = r["keep_idx"][0].long()
    a, k, v = pieces(vc.vitcop_rmsnorm(x[0], w["ln1"])[idx], pos[:, idx].contiguous())
    # one rounding to bf16 of sums in another order: at most an ulp apart (2^-7 of the value), and the rotary embedding
    # keeps the length of the pairs that it turns
    for got, ref in zip(caches, (k, v)):
        assert float((got.double() - ref.double()).norm() / ref.double().norm()) <= 2.0 ** -7
    h1 = vc.vitcop_project(a, wo, residual=x[0, idx].contiguous(), scratch=False)[0]
    x2 = vc.vitcop_rmsnorm(h1, w["ln2"])
    act = vc.vitcop_silu_mul(vc.vitcop_project(x2, w["wg"], scratch=False)[0], vc.vitcop_project(x2, w["wu"], scratch=False)[0])
    want = vc.vitcop_project(act, w["wd"], residual=h1, scratch=False)[0].double()
    assert float((r["y"][0].double() - want).norm() / want.norm()) <= 2.0 ** -7
