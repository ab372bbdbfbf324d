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


@pytest.mark.parametrize("M,N,K", [(257, 512, 4096), (317, 4096, 4064), (640, 4096, 4096), (1024, 1040, 4128), (500, 2064, 3008)])
def test_split_k(M, N, K):
    assert vc.lib.vitcop_project_workspace_bytes(M, N, K) > 0
    x, w, r = draw(M, N, K, M)
    y, _ = vc.vitcop_project(x, w, residual=r)
    check(x, w, y, r)


def test_rows_past_the_end_do_not_leak_in():
    """What lies behind the last row of x in memory (here infinities) is never multiplied."""
    x, w, r = draw(300, 512, 96, 3)
    big = torch.full((400, 96), float("inf"), dtype=torch.bfloat16, device="cuda")
    big[:300] = x
    y, _ = vc.vitcop_project(big[:300], w, residual=r, scratch=False)
    check(x, w, y, r)
