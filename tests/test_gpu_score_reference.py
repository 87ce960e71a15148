"""What sweep 1 takes its exponentials against: the error of the scores where key ranges are long, and keys without any weight."""
import numpy as np
import pytest
import torch

from test_gpu_score_ranges import _reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import paper_2604_06694_amd as A
    return A


def _continuous(x):
    """First-order autoregression (0.95) along the tokens of white noise [heads, L, d]."""
    step, decay = 1, 0.95
    while step < x.shape[1] and decay > 1e-3:
        x = torch.cat([x[:, :step], x[:, step:] + decay * x[:, :-step]], dim=1)
        step, decay = 2 * step, decay * decay
    return x


def _spread(n, lo, hi):
    return [int(lo * (hi / lo) ** ((i * 7 % n) / (n - 1))) for i in range(n)]


# most: the mean error of these inputs with ranges as short as equal lengths have and one reference for each, which these calls' longer
# ranges need not exceed
@pytest.mark.parametrize("H_q,H_kv,d,W,lens,most", [
    (32, 4, 128, 16, _spread(12, 500, 16000), 4.2e-7), (28, 4, 128, 32, _spread(12, 500, 16000), 3.6e-7),
    (28, 4, 128, 64, _spread(12, 500, 16000), 2.9e-7), (8, 2, 64, 32, _spread(12, 500, 16000), 3.5e-7),
    (14, 2, 256, 32, _spread(12, 500, 16000), 4.3e-7), (32, 4, 128, 16, _spread(70, 300, 2500), 3.2e-7),
    (16, 2, 64, 32, [8192] * 4, 4.4e-7)], ids=lambda v: str(v) if isinstance(v, (int, float)) else f"{len(v)}x{max(v)}")
def test_error_of_long_ranges(A, H_q, H_kv, d, W, lens, most):
    errors = []
    for seed in range(4):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        q = torch.randn(len(lens) * H_q * W * d, generator=gen, device="cuda").to(torch.bfloat16)
        k = torch.cat([_continuous(torch.randn((H_kv, L, d), generator=gen, device="cuda")).reshape(-1) for L in lens]).to(torch.bfloat16)
        ref, _ = _reference(q, k, H_q, H_kv, d, W, lens, True)
        got = A.score(A.Params(H_q, H_kv, d, W, pool_kernel=1), q, k, lens)
        errors.append(float((got.double() - ref).norm() / ref.norm()))
    print(f"\nerror {np.mean(errors):.3e}")
    assert np.mean(errors) <= most


# ragged items in ranges of one size; a call of 256 rows with one row tile per wave; two and three row tiles
@pytest.mark.parametrize("H_q,H_kv,d,W,lens", [(14, 2, 128, 32, _spread(12, 500, 12000)), (8, 2, 256, 32, _spread(8, 500, 12000)),
                                               (8, 2, 64, 16, _spread(70, 300, 2500)), (14, 2, 128, 64, _spread(12, 500, 12000)),
                                               (16, 2, 128, 32, [4096] * 2), (7, 1, 128, 32, [5000]), (18, 2, 128, 64, [3000])],
                         ids=lambda v: str(v) if isinstance(v, int) else f"{len(v)}x{max(v)}")
@pytest.mark.parametrize("first,n", [(0, 40), (0, 300), (64, 65), (200, 400), (255, 2000)])
def test_keys_whose_logits_are_minus_infinity(A, H_q, H_kv, d, W, lens, first, n):
    """Whole blocks of such keys, from the first of a range or later: they have no weight, and the others' weights are as without them."""
    gen = torch.Generator(device="cuda").manual_seed(3)
    q = (torch.rand(len(lens) * H_q * W * d, generator=gen, device="cuda") + 0.1).to(torch.bfloat16)
    k = torch.randn(sum(lens) * H_kv * d, generator=gen, device="cuda").to(torch.bfloat16)
    at = 0
    for L in lens:
        k[at:at + L * H_kv * d].view(H_kv, L, d)[:, first:min(first + n, L - W - 1)] = -torch.inf
        at += L * H_kv * d
    ref, _ = _reference(q, k, H_q, H_kv, d, W, lens, True)
    assert bool(ref.isfinite().all()) and bool((ref == 0).any())
    got = A.score(A.Params(H_q, H_kv, d, W, pool_kernel=1), q, k, lens)
    # (the bound of test_scores_for_every_division_into_ranges)
    assert ((got.double() - ref).abs() <= 3e-5 * ref + 1e-30).all()
