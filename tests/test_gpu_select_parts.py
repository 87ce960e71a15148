"""Selection where its division of the scores' range can go wrong: budgets of a few tokens and of nearly all, parts that hold too
many, scores that share values, that lie close together far from zero, drift along the head, or are not finite; all register counts."""
import numpy as np
import pytest
import torch

from oracle import audiokv_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import paper_2604_06694_amd as A
    return A


def _scores(kind, rng, L):
    x = rng.standard_normal(L)
    if kind == "normal":     return x
    if kind == "skewed":     return np.exp(2.0 * x) - 0.5
    if kind == "outlier":    return np.where(np.arange(L) == L // 3, 1e6, x)
    if kind == "clusters":   return np.where(rng.random(L) < 0.55, 1e-3 * x, 5.0 + 1e-4 * x)
    if kind == "close":      return 1000.0 + 1e-4 * x
    if kind == "levels":     return np.floor(4 * np.abs(x)) / 4
    if kind == "zeros":      return np.where(rng.random(L) < 0.5, np.where(rng.random(L) < 0.5, -0.0, 0.0), x)
    if kind == "equal":      return np.full(L, 0.25)
    if kind == "drift":      return np.cumsum(x)
    if kind == "tiny":       return 1e-42 * x
    if kind == "huge":       return 1e30 * x
    if kind == "infinite":   return np.where(rng.random(L) < 0.02, np.inf, np.where(rng.random(L) < 0.02, -np.inf, x))
    raise ValueError(kind)


KINDS = ["normal", "skewed", "outlier", "clusters", "close", "levels", "zeros", "equal", "drift", "tiny", "huge", "infinite"]


@pytest.mark.parametrize("L", [17, 80, 81, 500, 2048, 2049, 4096, 5000, 8208, 16384, 16400, 20001, 32768])
@pytest.mark.parametrize("kind", KINDS)
def test_selection_is_exact(A, kind, L):
    W, shares = 16, [0.0, 0.002, 0.07, 0.09, 0.4, 0.9, 0.93, 0.999, 1.0]
    rng = np.random.default_rng(L + KINDS.index(kind))
    s = np.stack([_scores(kind, rng, L) for _ in shares]).astype(np.float32)
    b = np.array([W + int(r * (L - W)) for r in shares], dtype=np.int32)
    cu = np.concatenate([[0], np.cumsum(b)]).astype(np.int32)
    p = A.Params(len(shares), len(shares), 64, W)
    got = A.select(p, torch.from_numpy(s).cuda().reshape(-1), torch.from_numpy(b).cuda(), torch.from_numpy(cu).cuda(), [L], int(cu[-1]))
    got = got.cpu().numpy()
    for h in range(len(shares)):
        order = np.lexsort((np.arange(L - W), -s[h, :L - W].astype(np.float64)))
        want = np.concatenate([np.sort(order[:b[h] - W]), np.arange(L - W, L)])
        assert np.array_equal(got[cu[h]:cu[h + 1]], want), (kind, L, shares[h])


def test_scores_that_are_no_numbers_keep_their_place(A):
    """NaN of either sign among ordinary scores: positive ones first of all, negative ones last."""
    L, W = 3000, 8
    rng = np.random.default_rng(5)
    s = rng.standard_normal(L).astype(np.float32)
    s[[10, 700, 2900]] = np.nan
    s[[11, 1500]] = -np.nan
    b = np.array([W + 1000], dtype=np.int32)
    got = A.select(A.Params(1, 1, 64, W), torch.from_numpy(s).cuda(), torch.from_numpy(b).cuda(),
                   torch.from_numpy(np.array([0, b[0]], dtype=np.int32)).cuda(), [L], int(b[0])).cpu().numpy()
    key = s.view(np.uint32).astype(np.int64)
    key = np.where(key & 0x80000000, 0xffffffff - key, key | 0x80000000)
    want = np.sort(np.lexsort((np.arange(L - W), -key[:L - W]))[:1000])
    assert np.array_equal(got, np.concatenate([want, np.arange(L - W, L)]))


@pytest.mark.parametrize("lens", [[4097], [5000, 700], [8191, 4096], [9001, 2048], [16001], [16385, 32768, 600], [32767, 5001], [40000, 9000]])
@pytest.mark.parametrize("alpha,kernel,mode", [(1.0, 7, 0), (0.5, 7, 0), (0.5, 1, 0), (0.75, 15, 1), (1.0, 5, 1)])
def test_selection_combines_the_chunks_of_a_convolution(A, lens, alpha, kernel, mode):
    """evict, whose selection reads heads of several chunks uncombined, against its stages one by one."""
    H, d, W = 2, 64, 8
    gen = torch.Generator(device="cuda").manual_seed(sum(lens))
    q = torch.randn(len(lens) * H * W * d, generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn(sum(lens) * H * d, generator=gen, device="cuda").to(torch.bfloat16)
    w = torch.rand(len(lens) * H, generator=gen, device="cuda")
    p = A.Params(H, H, d, W, pool_kernel=kernel, pool_mode=mode)
    out = A.evict(p, q, k, k, w, lens, 0.3, 0.125, alpha, alloc_scope=A.SCOPE_ITEM)
    smoothed = A.smooth(p, A.score(p, q, k, lens), lens, 0.125, alpha)
    staged = A.select(p, smoothed, out["budgets"], out["cu_budgets"], lens, out["total_rows"])
    assert torch.equal(out["indices"], staged)


@pytest.mark.parametrize("lens", [[4097], [8193], [5000, 700], [8193, 600, 4099, 1025], [12289, 4096, 333]])
@pytest.mark.parametrize("weights", [[1.0], [0.0, 1.0], [1.0, 0.0]])
def test_combining_chunks_stays_inside_the_head(A, lens, weights):
    """The combined scores that evict leaves in its workspace: those of every head what smooth gives, whole batches through, also
    of heads that keep no more than the window, and the bytes between the last head's and the next region (regions start at
    multiples of 256 bytes) as they were."""
    H, d, W = len(weights), 64, 8
    gen = torch.Generator(device="cuda").manual_seed(sum(lens))
    q = torch.randn(len(lens) * H * W * d, generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn(sum(lens) * H * d, generator=gen, device="cuda").to(torch.bfloat16)
    w = torch.tensor(weights * len(lens), dtype=torch.float32, device="cuda")
    p = A.Params(H, H, d, W, floor_frac=0.0)
    smoothed = A.smooth(p, A.score(p, q, k, lens), lens, 0.125, 1.0).view(torch.int32)
    n, poison = smoothed.numel(), 0x7f7f7f7f
    ws = torch.full((A.workspace_bytes(p, lens),), 0x7f, dtype=torch.uint8, device="cuda")
    out = A.evict(p, q, k, k, w, lens, 0.3, 0.125, 1.0, alloc_scope=A.SCOPE_ITEM, workspace=ws)
    if H > 1:
        assert (out["budgets"].view(-1, H)[:, weights.index(0.0)] == W).all()
    words = ws[:ws.numel() // 4 * 4].view(torch.int32)
    at = [64 * i for i in (words[:words.numel() - n + 1:64] == smoothed[0]).nonzero().view(-1).tolist()]
    at = [i for i in at if torch.equal(words[i:i + n], smoothed)]
    assert len(at) == 1
    gap = words[at[0] + n:(at[0] + n + 63) // 64 * 64]
    assert bool((gap == poison).all())


def _ties(kind, rng, L):
    if kind == "one value":   return np.full(L, -0.75)
    if kind == "two values":  return np.where(rng.random(L) < 0.5, 1.0, 1.0 + 2.0**-23)
    if kind == "ten values":  return np.floor(5 * rng.standard_normal(L)) / 8
    if kind == "few above":   return np.where(np.arange(L) % 97 == 5, 3.0, np.where(np.arange(L) % 3 == 0, 1.0, -1.0))
    if kind == "last":        return np.where(np.arange(L) < L - 70, -2.0, rng.standard_normal(L))
    if kind == "infinite":    return np.where(rng.random(L) < 0.4, np.inf, np.where(rng.random(L) < 0.5, -np.inf, 0.5))
    if kind == "no numbers":  return np.where(rng.random(L) < 0.4, np.nan, np.where(rng.random(L) < 0.5, -np.nan, 0.5))
    raise ValueError(kind)


@pytest.mark.parametrize("W", [0, 5])
@pytest.mark.parametrize("L", [40, 64, 65, 71, 513, 2048, 4095, 8192, 8193, 16384, 16385, 24577, 32768])
@pytest.mark.parametrize("kind", ["one value", "two values", "ten values", "few above", "last", "infinite", "no numbers"])
def test_equal_scores_are_kept_in_index_order(A, kind, L, W):
    """Thresholds that many tokens share, up to all of the longest head's, with none, some and all of them kept."""
    shares = [0.0, 0.03, 0.2, 0.4, 0.5, 0.71, 0.95, 1.0]
    rng = np.random.default_rng(L)
    s = np.stack([_ties(kind, rng, L) for _ in shares]).astype(np.float32)
    b = np.array([W + int(r * (L - W)) for r in shares], dtype=np.int32)
    cu = np.concatenate([[0], np.cumsum(b)]).astype(np.int32)
    p = A.Params(len(shares), len(shares), 64, W)
    got = A.select(p, torch.from_numpy(s).cuda().reshape(-1), torch.from_numpy(b).cuda(), torch.from_numpy(cu).cuda(), [L], int(cu[-1]))
    got = got.cpu().numpy()
    key = (s + np.float32(0)).view(np.uint32).astype(np.int64)
    key = np.where(key & 0x80000000, 0xffffffff - key, key | 0x80000000)
    for h in range(len(shares)):
        order = np.lexsort((np.arange(L - W), -key[h, :L - W]))
        want = np.concatenate([np.sort(order[:b[h] - W]), np.arange(L - W, L)])
        assert np.array_equal(got[cu[h]:cu[h + 1]], want), (kind, L, W, shares[h])
