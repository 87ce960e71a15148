"""Batches whose workspace is just what the static scratch of audiokv_evict_noalloc holds: a division into more key ranges that is a
little faster does not keep them from it."""
import numpy as np
import pytest

import paper_2604_06694_amd as A

# query heads, KV heads, head_dim, window; items, shortest, longest: with as many ranges for every head 6.1 to 8.4 MB (8 MiB are 8.39),
# with ranges of one size for all of them, and 256 rows planned for one workgroup per CU, 8.4 to 10.3
BATCHES = [(28, 4, 128, 64, 98, 118, 475), (28, 4, 128, 32, 106, 208, 417), (36, 4, 128, 64, 45, 268, 1075), (8, 2, 64, 16, 21, 2867, 5734),
           (32, 4, 128, 32, 97, 213, 426), (7, 1, 128, 32, 54, 504, 2018), (16, 1, 256, 16, 108, 626, 939), (7, 1, 128, 32, 27, 1623, 3246),
           (28, 4, 128, 64, 50, 555, 1111), (8, 2, 256, 32, 81, 755, 1133), (32, 4, 128, 16, 114, 168, 673), (32, 4, 128, 32, 101, 428, 642),
           (32, 8, 128, 32, 34, 828, 911), (36, 4, 128, 64, 106, 211, 233), (28, 4, 128, 32, 15, 693, 2773), (28, 4, 128, 64, 24, 1206, 1810),
           (32, 4, 128, 32, 95, 602, 602), (32, 4, 128, 32, 90, 668, 668)]


def _lengths(n, lo, hi):
    return [int(lo * (hi / lo) ** ((i * 7 % n) / (n - 1))) for i in range(n)]


@pytest.mark.parametrize("H_q,H_kv,d,W,n,lo,hi", BATCHES)
def test_fits_the_static_scratch(H_q, H_kv, d, W, n, lo, hi):
    assert A.workspace_bytes(A.Params(H_q, H_kv, d, W), _lengths(n, lo, hi)) <= A.NOALLOC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("H_q,H_kv,d,W,n,lo,hi", [(28, 4, 128, 64, 24, 1206, 1810), (28, 4, 128, 32, 15, 693, 2773), (32, 4, 128, 32, 95, 602, 602),
                                                  (8, 2, 64, 16, 21, 2867, 5734)])
def test_scores_with_the_ranges_that_fit(H_q, H_kv, d, W, n, lo, hi):
    from test_gpu_score_ranges import _inputs, _reference
    lens = _lengths(n, lo, hi)
    q, k = _inputs(H_q, H_kv, d, W, lens)
    ref, _ = _reference(q, k, H_q, H_kv, d, W, lens, True)
    got = A.score(A.Params(H_q, H_kv, d, W, pool_kernel=1), q, k, lens)
    # (the bound of test_scores_for_every_division_into_ranges)
    assert ((got.double() - ref).abs() <= 3e-5 * ref + 1e-30).all()


@pytest.mark.gpu
def test_the_static_scratch_takes_them():
    from test_zz_no_alloc import _case
    _case(A, np.random.default_rng(9), 28, 4, 128, 64, _lengths(24, 1206, 1810), 0.4, 0.125)
