"""Sweep 2 merges the row statistics of the key ranges for itself: every number of ranges that its batches divide differently,
ranges in which a row sees nothing, one to nine heads (which take different XCDs), and what rides along with the sweeps."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import paper_2604_06694_amd as A
    return A


def _inputs(H_q, H_kv, d, W, lens, seed=0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q = torch.randn(len(lens) * H_q * W * d, generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn(sum(lens) * H_kv * d, generator=gen, device="cuda").to(torch.bfloat16)
    return q, k


def _reference(q, k, H_q, H_kv, d, W, lens, causal):
    """Column sums of the softmax rows, and the rows' log-sum-exp, in float64."""
    G, at, sums, lse = H_q // H_kv, 0, [], []
    for i, L in enumerate(lens):
        qi = q.view(len(lens), H_kv, G * W, d)[i].double()
        ki = k[at:at + L * H_kv * d].view(H_kv, L, d).double()
        at += L * H_kv * d
        z = torch.matmul(qi, ki.transpose(1, 2).contiguous()) / d ** 0.5
        if causal:
            last = (L - W + torch.arange(W, device="cuda")).repeat(G)
            z = z.masked_fill(torch.arange(L, device="cuda")[None, None] > last[None, :, None], -torch.inf)
        lse.append(torch.logsumexp(z, 2).reshape(-1))
        sums.append(torch.softmax(z, 2).sum(1).reshape(-1))
    return torch.cat(sums), torch.cat(lse)


# query heads, KV heads, head_dim, window: one, two and three row tiles per wave, rows beyond one launch of sweep 2
@pytest.mark.parametrize("H_q,H_kv,d,W", [(7, 1, 128, 32), (28, 4, 128, 64), (16, 2, 128, 32), (24, 3, 64, 16), (20, 5, 256, 32),
                                          (36, 9, 128, 16), (8, 1, 128, 64), (1, 1, 64, 1)])
@pytest.mark.parametrize("lens", [[70], [1056], [2016], [2112], [4097], [9000, 300], [700] * 5])
@pytest.mark.parametrize("causal", [1, 0])
def test_scores_for_every_division_into_ranges(A, H_q, H_kv, d, W, lens, causal):
    q, k = _inputs(H_q, H_kv, d, W, lens)
    ref, lse = _reference(q, k, H_q, H_kv, d, W, lens, causal)
    p = A.Params(H_q, H_kv, d, W, pool_kernel=1, causal=causal)
    # exp2 of arguments of up to about 64 in magnitude, a logit and a constant each rounded a few times to 24 bits:
    # 2 * 64 * 3 * 2^-24 * ln 2 = 1.6e-5, and as much again for the fp32 sums of products
    for got in (A.score(p, q, k, lens), A.score(p, q, k, lens, lse=lse.float())):
        assert ((got.double() - ref).abs() <= 3e-5 * ref + 1e-30).all()


@pytest.mark.parametrize("n_items", [1, 3, 9, 40])
@pytest.mark.parametrize("with_lse", [False, True])
def test_allocation_and_taps_that_ride_along(A, n_items, with_lse):
    H_q, H_kv, d, W = 8, 2, 64, 16
    lens = [500 + 37 * i for i in range(n_items)]                    # no powers of two: taps for every length
    q, k = _inputs(H_q, H_kv, d, W, lens)
    w = torch.rand(n_items * H_kv, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    p = A.Params(H_q, H_kv, d, W)
    lse = _reference(q, k, H_q, H_kv, d, W, lens, True)[1].float() if with_lse else None
    out = A.evict(p, q, k, k, w, lens, 0.4, 0.125, 1.0, alloc_scope=A.SCOPE_ITEM, lse=lse)
    budgets, cu = A.allocate(p, w, n_items, H_kv, lens, 0.4)
    assert torch.equal(out["budgets"], budgets) and torch.equal(out["cu_budgets"], cu)
    smoothed = A.smooth(p, A.score(p, q, k, lens, lse=lse), lens, 0.125, 1.0)
    assert torch.equal(out["indices"], A.select(p, smoothed, budgets, cu, lens, out["total_rows"]))


@pytest.mark.parametrize("n_items", [10, 30, 33])                    # pools of 40, 120 and 132 heads: one wave, one wave, 256 threads
def test_pools_of_a_call_that_may_not_use_another_stream(A, n_items):
    H_q, H_kv, d, W, L = 4, 4, 64, 8, 256
    q, k = _inputs(H_q, H_kv, d, W, [L] * n_items)
    w = torch.rand(n_items * H_kv, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    p = A.Params(H_q, H_kv, d, W)
    ref = A.evict(p, q, k, k, w, [L] * n_items, 0.4, 0.125, 1.0)
    cu = torch.tensor(np.arange(n_items + 1) * L, dtype=torch.int32, device="cuda")
    out = {key: torch.zeros_like(t) for key, t in ref.items() if torch.is_tensor(t) and key != "workspace"}
    A.evict_noalloc(p, q, k, k, w, [L] * n_items, 0.4, 0.125, 1.0, out, cu_seqlens=cu)
    for key in out:
        assert torch.equal(out[key], ref[key]), key
