"""Smoothing of lengths that are not powers of two as a convolution with the mask's taps: the edges of its transforms (one
chunk, several, the longest), of the sequences inside them and of the pooling windows, masks with a taper and at the
Nyquist bin, filters shared by many heads or formed by every workgroup, against a float64 library transform with the
mask applied (itself pinned to the oracle on a short sequence)."""
import numpy as np
import pytest
import torch

from oracle import audiokv_oracle as O
from workloads import f64_to_bf16_bits

from gpu_util import SCORE_RTOL, bf16_tensor, rel_err

pytestmark = pytest.mark.gpu

# fp32 transforms of up to 2^17 points: about log2(N) roundings of 6e-8 of the sequence's largest value, both ways
ATOL = 4e-6


@pytest.fixture(scope="module")
def A():
    import paper_2604_06694_amd as A
    return A


def reference(x, cutoff, alpha, T):
    L = len(x)
    ks = int(np.floor(cutoff * (L // 2)))
    k = np.arange(L // 2 + 1)
    w = np.where(k <= ks, 1.0, np.where(k <= ks + T, 0.5 * (1 + np.cos(np.pi * (k - ks) / (T + 1))), 0.0))
    return (1 - alpha) * x + alpha * np.fft.irfft(np.fft.rfft(x) * w, n=L)


def sequences(rng, n, L):
    x = np.exp(np.cumsum(rng.standard_normal((n, L)) * 0.05, axis=1) % 2.0)
    x[:, rng.integers(0, L, 3)] *= 20.0
    return x.astype(np.float32)


def check(A, rng, lens, H, cutoff, alpha=1.0, T=0):
    s = [sequences(rng, H, L) for L in lens]
    out = A.smooth(A.Params(H, H, 128, 1, taper_bins=T), torch.from_numpy(np.concatenate([x.reshape(-1) for x in s])).cuda(), lens,
                   cutoff, alpha).cpu().numpy()
    at = 0
    for x in s:
        for h in range(H):
            ref = reference(x[h].astype(np.float64), cutoff, alpha, T)
            got = out[at:at + x.shape[1]]
            assert np.abs(got - ref).max() <= ATOL * np.abs(x[h]).max(), (x.shape, h, np.abs(got - ref).max() / np.abs(x[h]).max())
            at += x.shape[1]
    return out


def test_reference_is_the_oracle():
    x = sequences(np.random.default_rng(1), 1, 101)[0].astype(np.float64)
    for T in (0, 4, 60):
        np.testing.assert_allclose(reference(x, 0.3, 0.7, T), O.smooth(x, 0.3, 0.7, taper_bins=T), rtol=0, atol=1e-12 * np.abs(x).max())


@pytest.mark.parametrize("L", [3, 5, 7, 9, 11, 15, 17, 1023, 1025, 2047, 2049, 4095, 4097, 8191, 8193, 16383, 16385, 32767, 32769,
                               65535, 65537, 131071])
def test_lengths_around_the_transform_sizes(A, L):
    check(A, np.random.default_rng(L), [L], 2, 0.5 if L < 100 else 0.125)


@pytest.mark.parametrize("L", [12, 999, 1000, 4500, 9001])
@pytest.mark.parametrize("cutoff,alpha,T", [(0.125, 0.5, 0), (0.25, 1.0, 1), (0.0, 1.0, 7), (0.5, 0.25, 300), (0.95, 1.0, 40),
                                            (0.999, 1.0, 1_000_000)])
def test_masks(A, L, cutoff, alpha, T):
    check(A, np.random.default_rng(L + T), [L], 3, cutoff, alpha, T)


@pytest.mark.parametrize("L", [5, 64, 999, 1024, 5000, 32768, 40000])
@pytest.mark.parametrize("T", [2**30, 2**31 - 1])
def test_tapers_as_long_as_the_argument_allows(A, L, T):
    check(A, np.random.default_rng(L), [L], 2, 0.3, 1.0, T)
    check(A, np.random.default_rng(L), [L] * 40, 2, 0.3, 1.0, T)


def test_ragged_batch_with_equal_and_short_lengths(A):
    check(A, np.random.default_rng(2), [5000, 30, 1024, 5000, 20000, 700, 9, 4097, 20000], 2, 0.2)


@pytest.mark.parametrize("L", [700, 3000, 5000, 17000])
def test_filter_shared_by_many_heads_gives_the_same_bits(A, L):
    rng = np.random.default_rng(L)
    x = sequences(rng, 4, L)
    p = A.Params(4, 4, 128, 1)
    t = torch.from_numpy(x.reshape(-1)).cuda()
    few = A.smooth(p, t, [L], 0.125, 1.0)                       # 4 heads: every workgroup transforms the filter
    many = A.smooth(p, t.repeat(5), [L] * 5, 0.125, 1.0)        # 20 heads of one length: a launch of its own does
    assert torch.equal(many, few.repeat(5))
    inplace = t.clone()
    A.smooth(p, inplace, [L], 0.125, 1.0, out=inplace)
    assert torch.equal(inplace, few)


@pytest.mark.parametrize("lens", [[300], [1100, 517], [5003], [70, 4099, 70, 9000, 70]])
@pytest.mark.parametrize("kernel,mode", [(1, 0), (3, 0), (5, 1), (7, 0), (7, 1), (9, 0), (11, 0), (31, 1)])
def test_pooling_on_load_equals_the_stages_composed(A, lens, kernel, mode):
    rng = np.random.default_rng(sum(lens) + kernel)
    H_q, H_kv, d, W = 4, 2, 64, 8
    q = bf16_tensor(f64_to_bf16_bits(rng.standard_normal(len(lens) * H_q * W * d)))
    k = bf16_tensor(f64_to_bf16_bits(rng.standard_normal(sum(lens) * H_kv * d)))
    v = bf16_tensor(f64_to_bf16_bits(rng.standard_normal(sum(lens) * H_kv * d)))
    w = torch.rand(len(lens) * H_kv, device="cuda") + 0.1
    p = A.Params(H_q, H_kv, d, W, pool_kernel=kernel, pool_mode=mode)
    for alpha in (1.0, 0.5):
        out = A.evict(p, q, k, v, w, lens, 0.4, 0.25, alpha, alloc_scope=A.SCOPE_ITEM)
        b, cu = A.allocate(p, w, len(lens), H_kv, lens, 0.4)
        idx = A.select(p, A.smooth(p, A.score(p, q, k, lens), lens, 0.25, alpha), b, cu, lens, out["total_rows"])
        assert torch.equal(idx, out["indices"][:out["total_rows"]])


def found(ws, close_to):
    """The run of floats in a workspace that lies within 1e-6 of the sequence `close_to`, as bits; runs start at multiples of 256
    bytes."""
    w, x = ws[:ws.numel() // 4 * 4].view(torch.float32), torch.from_numpy(close_to).cuda()
    head = w[:w.numel() - x.numel() + 1][::64]
    for i in ((head - x[0]).abs() <= 1e-6).nonzero().view(-1).tolist():
        if bool(((w[64 * i:64 * i + x.numel()] - x).abs() <= 1e-6).all()):
            return w[64 * i:64 * i + x.numel()].view(torch.int32).clone()
    raise AssertionError("no such run of floats")


@pytest.mark.parametrize("T", [0, 1, 1000])
@pytest.mark.parametrize("lens,H_kv", [([13577], 2), ([5003] * 20, 2), ([3000, 700], 2)])
def test_taps_are_the_same_bits_wherever_they_are_evaluated(A, T, lens, H_kv):
    """The filter's taps are evaluated in extra workgroups of the first sweep, on the helper stream, or by smooth itself; evict
    equals the calls composed only if they are the same bits from all of them, with a taper as well."""
    rng = np.random.default_rng(T + len(lens))
    H_q, d, W, n, L, cutoff = 2 * H_kv, 64, 8, len(lens), lens[0], 0.25
    q = bf16_tensor(f64_to_bf16_bits(rng.standard_normal(n * H_q * W * d)))
    k = bf16_tensor(f64_to_bf16_bits(rng.standard_normal(sum(lens) * H_kv * d)))
    w = torch.rand(n * H_kv, device="cuda") + 0.1
    p = A.Params(H_q, H_kv, d, W, taper_bins=T)
    impulse = np.zeros(L)
    impulse[0] = 1.0
    taps = reference(impulse, cutoff, 1.0, T).astype(np.float32)
    ws = torch.zeros(A.workspace_bytes(p, lens), dtype=torch.uint8, device="cuda")
    smoothed = A.smooth(p, A.score(p, q, k, lens), lens, cutoff, 1.0, workspace=ws)
    h = found(ws, taps)
    for scope in (A.SCOPE_ITEM, A.SCOPE_GLOBAL):
        if scope == A.SCOPE_GLOBAL and len(set(lens)) > 1:
            continue
        for timed in (False, True):
            ws.zero_()
            A.profile_enable(timed)
            try:
                A.evict(p, q, k, k, w, lens, 0.4, cutoff, 1.0, alloc_scope=scope, workspace=ws)
            finally:
                A.profile_enable(False)
            assert torch.equal(found(ws, taps), h)
            assert torch.equal(found(ws, smoothed.cpu().numpy()), smoothed.view(torch.int32))


def test_smoothed_scores_meet_the_oracle(A):
    L = 2500
    x = sequences(np.random.default_rng(3), 2, L)
    out = A.smooth(A.Params(2, 2, 128, 1), torch.from_numpy(x.reshape(-1)).cuda(), [L], 0.125, 1.0).cpu().numpy().reshape(2, L)
    for h in range(2):
        assert rel_err(out[h], O.smooth(x[h].astype(np.float64), 0.125, 1.0)) <= SCORE_RTOL


def test_smooth_more_heads_than_a_grid_dimension_holds(A):
    """70000 short sequences of one head each: beyond 65535, where the second dimension of a grid ends; the first and the
    last ones are what they are on their own, bit for bit."""
    L, n = 21, 70000
    s = torch.rand(n * L, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    p = A.Params(1, 1, 64, 1)
    out = A.smooth(p, s, [L] * n, 0.25, 1.0).view(n, L)
    some = [0, 1, 65534, 65535, 65536, n - 1]
    alone = torch.stack([A.smooth(p, s.view(n, L)[i].contiguous(), [L], 0.25, 1.0) for i in some])
    torch.cuda.synchronize()
    assert torch.equal(out[some], alone)
    spectrum = torch.fft.rfft(s.view(n, L).double(), dim=1)
    spectrum[:, int(0.25 * (L // 2)) + 1:] = 0
    ref = torch.fft.irfft(spectrum, n=L, dim=1)
    # fp32 transforms of 32 points and 21 taps: a few ulps of the mean-1/2 sequence
    assert (out.double() - ref).abs().max().item() < 5e-6


@pytest.mark.parametrize("lens", [[9001] * 3, [9001, 9003, 16000], [9001, 1500, 30011], [40000, 70000], [70000, 70001], [2048, 9001, 9001]])
@pytest.mark.parametrize("H", [2, 5])
def test_heads_of_as_many_chunks_and_of_fewer(A, lens, H):
    """The residues of a head in their order, and turned from head to head where some heads have fewer."""
    check(A, np.random.default_rng(len(lens) + H), lens, H, 0.125)
