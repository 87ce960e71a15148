"""Scores of items of different lengths: key ranges of one size, in which a workgroup finds its item among up to 64, as many ranges for
every head (more items, many heads, a K beyond the memory-side cache, calls that fit the chip at once), sweeps of one call that divide the
heads differently."""
import numpy as np
import pytest
import torch

from test_gpu_score_ranges import _inputs, _reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import paper_2604_06694_amd as A
    return A


def _spread(n, lo, hi):
    return [int(lo * (hi / lo) ** ((i * 7 % n) / max(1, n - 1))) for i in range(n)]


# query heads, KV heads, head_dim, window; the last ones cover 576 rows, in which the second launch of sweep 2 holds twice the workgroups
@pytest.mark.parametrize("H_q,H_kv,d,W", [(28, 4, 128, 32), (8, 1, 128, 32), (14, 2, 128, 64), (8, 2, 256, 32), (8, 2, 64, 16), (9, 1, 128, 64)])
@pytest.mark.parametrize("lens", [[100, 70], [64, 65, 63 + 64, 2048], [9000, 300], [300, 20011], [4000, 3900, 500, 2000, 4096], _spread(12, 90, 6000),
                                  _spread(64, 64, 700), _spread(65, 64, 700), [5000] + [64] * 130],
                         ids=lambda v: f"{len(v)}x{min(v)}-{max(v)}")
def test_scores_of_ragged_items(A, H_q, H_kv, d, W, lens):
    q, k = _inputs(H_q, H_kv, d, W, lens)
    ref, lse = _reference(q, k, H_q, H_kv, d, W, lens, True)
    p = A.Params(H_q, H_kv, d, W, pool_kernel=1)
    # (the bound of test_scores_for_every_division_into_ranges)
    for got in (A.score(p, q, k, lens), A.score(p, q, k, lens, lse=lse.float())):
        assert ((got.double() - ref).abs() <= 3e-5 * ref + 1e-30).all()


@pytest.mark.parametrize("n_items", [3, 70])
def test_items_score_as_they_do_alone(A, n_items):
    """The same item twice, and by itself: a range belongs to the right item and head in either order."""
    H_q, H_kv, d, W = 8, 2, 64, 16
    lens = _spread(n_items, 200, 9000)
    q, k = _inputs(H_q, H_kv, d, W, lens)
    p = A.Params(H_q, H_kv, d, W)
    got = A.score(p, q, k, lens).cpu().numpy()
    cu = np.concatenate([[0], np.cumsum(lens)])
    for i in (0, n_items // 2, n_items - 1):
        a, b = cu[i] * H_kv, cu[i + 1] * H_kv
        alone = A.score(p, q.view(n_items, -1)[i].contiguous(), k[a * d:b * d].contiguous(), [lens[i]]).cpu().numpy()
        # the statistics are added up over other ranges: a few roundings of sums of up to 9000 terms around 1
        assert np.allclose(got[a:b], alone, rtol=1e-5, atol=0)


# ranges of some 300 to 900 keys, in which sweep 1 raises its reference tile by tile: one and two row tiles per wave, every head dimension, and
# the uniform call of 256 rows that raises it as well
@pytest.mark.parametrize("H_q,H_kv,d,W,lens", [(14, 2, 128, 32, _spread(12, 3000, 24000)), (14, 2, 128, 64, _spread(12, 3000, 24000)),
                                               (8, 2, 256, 32, _spread(8, 3000, 24000)), (8, 2, 64, 16, _spread(12, 3000, 24000)),
                                               (32, 4, 128, 32, [16384, 16384])], ids=lambda v: str(v) if isinstance(v, int) else f"{len(v)}")
@pytest.mark.parametrize("shape", ["ramp", "step", "sawtooth"])
def test_logits_that_drift_past_each_new_reference(A, H_q, H_kv, d, W, lens, shape):
    """Logits that climb, fall (every third query sees them the other way round) and jump by hundreds of octaves along an item."""
    q, k = _inputs(H_q, H_kv, d, W, lens, 5)
    q = (0.25 * q.view(-1, d).float() + 1.0)
    q[::3] *= -1.0
    q = q.to(torch.bfloat16).reshape(-1)
    steps = []
    for L in lens:
        x = torch.linspace(-1, 1, L, device="cuda")
        steps.append({"ramp": x, "step": torch.sign(x), "sawtooth": torch.remainder(x * 20, 2) - 1}[shape].repeat(H_kv))
    k = (0.25 * k.view(-1, d).float() + 6.0 * torch.cat(steps)[:, None]).to(torch.bfloat16).reshape(-1)
    ref, _ = _reference(q, k, H_q, H_kv, d, W, lens, True)
    got = A.score(A.Params(H_q, H_kv, d, W, pool_kernel=1), q, k, lens)
    # logits of up to 150 octaves, rounded in each of d / 16 products and sums, and the row's constant likewise: 2 * 16 * 150 * 2^-24 * ln 2
    assert ((got.double() - ref).abs() <= 2e-4 * ref + 1e-30).all()


# as many ranges for every head, which sweep 2 takes from the last to the first: K of some 300 MB at d = 256, and 129 heads of short items
@pytest.mark.parametrize("H_q,H_kv,d,W,lens", [(2, 2, 256, 16, _spread(41, 2000, 18000)), (3, 1, 128, 32, _spread(129, 64, 2500))],
                         ids=lambda v: str(v) if isinstance(v, int) else f"{len(v)}x{max(v)}")
def test_items_that_get_as_many_ranges_for_every_head(A, H_q, H_kv, d, W, lens):
    q, k = _inputs(H_q, H_kv, d, W, lens)
    ref, lse = _reference(q, k, H_q, H_kv, d, W, lens, True)
    p = A.Params(H_q, H_kv, d, W, pool_kernel=1)
    # (the bound of test_scores_for_every_division_into_ranges)
    for got in (A.score(p, q, k, lens), A.score(p, q, k, lens, lse=lse.float())):
        assert ((got.double() - ref).abs() <= 3e-5 * ref + 1e-30).all()
