"""Calls whose workgroups outnumber what one launch holds, or whose heads outlast the workgroups that a launch gives them."""
import numpy as np
import pytest
import torch

from workloads import f64_to_bf16_bits

from gpu_util import bf16_tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import paper_2604_06694_amd as A
    return A


def test_evict_300000_heads_with_a_wide_pooling_kernel(A):
    """Beyond 2^18 heads, sixty-four workgroups of 256 threads each are more than a launch holds."""
    n, L, d, W = 300_000, 24, 64, 2
    gen = torch.Generator(device="cuda").manual_seed(0)
    k = torch.randn(n * L * d, generator=gen, device="cuda").to(torch.bfloat16)
    q = torch.randn(n * W * d, generator=gen, device="cuda").to(torch.bfloat16)
    w = torch.ones(n, device="cuda")
    p = A.Params(1, 1, d, W, pool_kernel=15)
    out = A.evict(p, q, k, k, w, [L] * n, 0.5, 0.25, 1.0, alloc_scope=A.SCOPE_ITEM)
    torch.cuda.synchronize()
    rows = out["total_rows"] // n
    for i in (0, 1, 131_071, 262_143, 262_144, n - 1):
        one = A.evict(p, q.view(n, -1)[i].contiguous(), k.view(n, -1)[i].contiguous(), k.view(n, -1)[i].contiguous(), w[:1], [L], 0.5,
                      0.25, 1.0, alloc_scope=A.SCOPE_ITEM)
        assert torch.equal(out["indices"].view(-1)[i * rows:(i + 1) * rows], one["indices"].view(-1)[:rows])


@pytest.mark.parametrize("kernel,mode", [(7, 0), (7, 1), (5, 0), (9, 1), (15, 0)])
def test_pooling_of_a_head_longer_than_its_workgroups(A, kernel, mode):
    """2.2 million tokens: more than 1024 workgroups of eight outputs per thread cover in one go."""
    L, d, W = 2_200_003, 64, 4
    rng = np.random.default_rng(1)
    q = bf16_tensor(f64_to_bf16_bits(rng.standard_normal(W * d)))
    k = torch.randn(L * d, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda").to(torch.bfloat16)
    raw = A.score(A.Params(1, 1, d, W, pool_kernel=1), q, k, [L])
    got = A.score(A.Params(1, 1, d, W, pool_kernel=kernel, pool_mode=mode), q, k, [L])
    pad = kernel // 2
    ref = torch.nn.functional.pad(raw.double(), (pad, pad), value=0.0 if mode == 0 else -np.inf).unfold(0, kernel, 1)
    ref = ref.mean(1) if mode == 0 else ref.max(1).values
    if mode == 1:
        assert torch.equal(got.double(), ref)
    else:
        assert ((got.double() - ref).abs() <= 1e-6 * ref).all()       # up to fifteen fp32 additions of positive scores


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("megabytes", [100, 260])          # of K, V and the kept rows: what the memory-side cache holds, and more
def test_gather_on_either_side_of_the_cache(A, d, megabytes):
    H, L = 2, megabytes * (1 << 20) * 5 // 7 // (2 * 2 * d * 2)      # 0.4 of the rows kept
    gen = torch.Generator(device="cuda").manual_seed(d)
    k = torch.randn(H * L * d, generator=gen, device="cuda").to(torch.bfloat16)
    v = torch.randn(H * L * d, generator=gen, device="cuda").to(torch.bfloat16)
    keep = [torch.sort(torch.randperm(L, generator=gen, device="cuda")[:int(0.4 * L) + h])[0] for h in range(H)]
    cu_b = torch.tensor(np.concatenate([[0], np.cumsum([len(x) for x in keep])]), dtype=torch.int32, device="cuda")
    ko, vo = A.compact(A.Params(H, H, d, 1), k, v, torch.cat(keep).to(torch.int32), cu_b, [L], int(cu_b[-1]))
    for got, src in ((ko, k), (vo, v)):
        assert torch.equal(got, torch.cat([src.view(H, L, d)[h][keep[h]] for h in range(H)]))


def test_scores_of_keys_that_do_not_fit_the_cache(A):
    """Beyond 256 MB of keys the second sweep takes the heads from the last to the first, whole groups of eight; here 17 of them."""
    n, L, d, W = 17, 130_000, 64, 4
    gen = torch.Generator(device="cuda").manual_seed(3)
    k = torch.randn(n * L * d, generator=gen, device="cuda").to(torch.bfloat16)
    q = torch.randn(n * W * d, generator=gen, device="cuda").to(torch.bfloat16)
    p = A.Params(1, 1, d, W)
    got = A.score(p, q, k, [L] * n).view(n, L)
    for i in (0, 7, 8, 15, 16):
        one = A.score(p, q.view(n, -1)[i].contiguous(), k.view(n, -1)[i].contiguous(), [L])
        # the same logits; the row sums are added over other ranges
        assert ((got[i] - one).abs() <= 2e-6 * one).all()
