"""Power-of-two lengths, one workgroup per head, every transform size: masks at both ends of the spectrum and with a taper,
the energy-adaptive cutoff, in place, fused pooling against the staged calls, several lengths in one call."""
import numpy as np
import pytest
import torch

from workloads import f64_to_bf16_bits

from gpu_util import bf16_tensor
from test_gpu_conv import ATOL, reference, sequences

pytestmark = pytest.mark.gpu

LENGTHS = [512, 1024, 2048, 4096, 8192, 16384, 32768]      # 512: the first length of the kernel for shorter heads


@pytest.fixture(scope="module")
def A():
    import paper_2604_06694_amd as A
    return A


def smooth(A, x, cutoff, alpha, heads, **params):
    """`x` [n, L] in a call of `heads` heads (more than 64: no head is spread over several workgroups)."""
    n, L = x.shape
    reps = -(-heads // n)
    t = torch.from_numpy(x.reshape(-1)).cuda().repeat(reps)
    out = A.smooth(A.Params(n, n, 128, 1, **params), t, [L] * reps, cutoff, alpha)
    assert torch.equal(out, out[:n * L].repeat(reps))
    A.smooth(A.Params(n, n, 128, 1, **params), t, [L] * reps, cutoff, alpha, out=t)
    assert torch.equal(t, out)
    return out[:n * L].cpu().numpy().reshape(n, L)


@pytest.mark.parametrize("L", LENGTHS)
@pytest.mark.parametrize("cutoff,alpha,T", [(0.125, 1.0, 0), (0.0, 1.0, 0), (0.0, 0.5, 3), (0.5, 1.0, 100), (0.999, 0.25, 0),
                                            (0.97, 1.0, 1_000_000)])
def test_every_transform_size(A, L, cutoff, alpha, T):
    x = sequences(np.random.default_rng(L + T), 2, L)
    got = smooth(A, x, cutoff, alpha, 66, taper_bins=T)
    for h in range(2):
        ref = reference(x[h].astype(np.float64), cutoff, alpha, T)
        assert np.abs(got[h] - ref).max() <= ATOL * np.abs(x[h]).max()
        if cutoff == 0.0 and T == 0:
            assert np.all(got[h] == got[h, 0])              # the mean, everywhere the same


@pytest.mark.parametrize("lens", [[1024, 2048], [2048, 16384, 1024], [32768, 1024, 4096], [1024, 2048, 4096, 8192, 16384, 32768],
                                  [512, 1024], [8, 16384, 1024], [4, 256, 8192, 32768], [2048, 3000, 1024, 31], [16384, 32768, 700]])
@pytest.mark.parametrize("H", [2, 40])
@pytest.mark.parametrize("mode,cutoff,T,alpha", [(0, 0.125, 0, 1.0), (0, 0.4, 9, 0.5), (0, 1.0, 0, 1.0), (2, 0.9, 0, 1.0)])
def test_several_lengths_in_one_call(A, lens, H, mode, cutoff, T, alpha):
    """Every head of a call with power-of-two lengths of different paths is smoothed, once, as the mask says: up to 80 heads share
    launches, 40 heads of a length are too many to be spread over workgroups."""
    rng = np.random.default_rng(sum(lens) + H)
    s = [sequences(rng, 2, L) for L in lens]
    flat = torch.from_numpy(np.concatenate([np.tile(x, (H // 2, 1)).reshape(-1) for x in s])).cuda()
    p = A.Params(H, H, 128, 1, taper_bins=T, cutoff_mode=mode)
    out = A.smooth(p, flat, lens, cutoff, alpha).cpu().numpy()
    ks = A.smooth_cutoffs(p, flat, lens, cutoff).cpu().numpy()
    at = 0
    for i, x in enumerate(s):
        L = x.shape[1]
        got = out[at:at + H * L].reshape(H, L)
        at += H * L
        for h in range(2):
            assert np.all(got[h::2] == got[h])
            k = int(ks[i * H + h])
            if mode == 0:
                assert k == int(np.floor(cutoff * (L // 2)))
            bins = np.arange(L // 2 + 1)
            w = np.where(bins <= k, 1.0, np.where(bins <= k + T, 0.5 * (1 + np.cos(np.pi * (bins - k) / (T + 1))), 0.0))
            x64 = x[h].astype(np.float64)
            ref = (1 - alpha) * x64 + alpha * np.fft.irfft(np.fft.rfft(x64) * w, n=L)
            assert np.abs(got[h] - ref).max() <= ATOL * np.abs(x[h]).max(), (L, h)


@pytest.mark.parametrize("L", LENGTHS)
@pytest.mark.parametrize("rho", [0.2, 0.9, 0.999])
@pytest.mark.parametrize("no_dc", [False, True])
def test_energy_cutoff(A, L, rho, no_dc):
    x = sequences(np.random.default_rng(L), 3, L)
    x -= x.mean(axis=1, keepdims=True) * np.float32(0.8)     # little enough DC for the rule to look beyond it
    mode = A.CUTOFF_ENERGY_NO_DC if no_dc else A.CUTOFF_ENERGY
    p = A.Params(3, 3, 128, 1, cutoff_mode=mode)
    t = torch.from_numpy(x.reshape(-1)).cuda()
    ks = A.smooth_cutoffs(p, t, [L], rho).cpu().numpy()
    out = A.smooth(p, t, [L], rho, 1.0).cpu().numpy().reshape(3, L)
    for h in range(3):
        f = np.fft.rfft(x[h].astype(np.float64))
        e = np.abs(f) ** 2
        if no_dc:
            e[0] = 0.0
        c, k = np.cumsum(e), int(ks[h])
        tol = 2e-5 * c[-1]                                  # fp32 bin energies: either neighbour of a near tie is right
        assert k >= int(no_dc) and c[k] >= rho * c[-1] - tol and (k == int(no_dc) or c[k - 1] < rho * c[-1] + tol)
        f[k + 1:] = 0
        assert np.abs(out[h] - np.fft.irfft(f, n=L)).max() <= ATOL * np.abs(x[h]).max()


@pytest.mark.parametrize("L", [256, 512, 1000, 1024, 2048, 5003, 16384, 32768])
@pytest.mark.parametrize("no_dc", [False, True])
def test_energy_cutoff_keeps_everything_at_rho_one(A, L, no_dc):
    """rho = 1 is allowed: k* captures the whole energy up to what fp32 energies resolve, and the result is the input. Smooth
    and peaked sequences: the bins at the end hold next to nothing, so that the last prefix sums are all about the total."""
    rng = np.random.default_rng(L)
    n = 96 if L <= 5003 else 24
    t = np.arange(L) / L
    x = np.empty((n, L))
    for i in range(n):
        if i % 3 == 0:
            x[i] = np.convolve(rng.random(L + 40), np.hanning(41) / 20, "valid")
        elif i % 3 == 1:
            x[i] = 0.1 + np.exp(-0.5 * ((t - rng.random()) / rng.uniform(0.002, 0.2)) ** 2)
        else:
            x[i] = 1 + sum(rng.standard_normal() / k ** 2 * np.cos(2 * np.pi * k * t + rng.random() * 6) for k in range(1, 40))
    x = x.astype(np.float32)
    mode = A.CUTOFF_ENERGY_NO_DC if no_dc else A.CUTOFF_ENERGY
    p = A.Params(n, n, 128, 1, cutoff_mode=mode)
    f = torch.from_numpy(x.reshape(-1)).cuda()
    ks = A.smooth_cutoffs(p, f, [L], 1.0).cpu().numpy()
    out = A.smooth(p, f, [L], 1.0, 1.0).cpu().numpy().reshape(n, L)
    e = np.abs(np.fft.rfft(x.astype(np.float64), axis=1)) ** 2
    e[:, 0] *= not no_dc
    c = np.cumsum(e, axis=1)
    kept = c[np.arange(n), ks] / c[:, -1]
    assert kept.min() >= 1 - 1e-6, (kept.min(), int((kept < 1 - 1e-6).sum()))     # what fp32 bin energies can hide
    assert np.abs(out - x).max() <= 2e-3 * np.abs(x).max()                       # sqrt(1e-6), plus fp32 transforms


@pytest.mark.parametrize("kernel,mode", [(3, 0), (5, 1), (7, 0), (7, 1), (9, 1), (11, 0), (21, 0), (255, 1), (1025, 0)])
def test_pooling_on_load_equals_the_stages_composed(A, kernel, mode):
    rng = np.random.default_rng(kernel)
    lens, H_q, H_kv, d, W = [1024, 8192, 512, 1024, 700, 16384, 32768], 4, 10, 64, 8
    H_q = 20
    q = bf16_tensor(f64_to_bf16_bits(rng.standard_normal(len(lens) * H_q * W * d)))
    k = bf16_tensor(f64_to_bf16_bits(rng.standard_normal(sum(lens) * H_kv * d)))
    w = torch.rand(len(lens) * H_kv, device="cuda") + 0.1
    for cutoff_mode, cutoff in ((A.CUTOFF_FRACTION, 0.2), (A.CUTOFF_ENERGY_NO_DC, 0.9)):
        p = A.Params(H_q, H_kv, d, W, pool_kernel=kernel, pool_mode=mode, cutoff_mode=cutoff_mode)
        for alpha in (1.0, 0.5):
            out = A.evict(p, q, k, k, w, lens, 0.4, cutoff, alpha, alloc_scope=A.SCOPE_ITEM)
            b, cu = A.allocate(p, w, len(lens), H_kv, lens, 0.4)
            idx = A.select(p, A.smooth(p, A.score(p, q, k, lens), lens, cutoff, alpha), b, cu, lens, out["total_rows"])
            assert torch.equal(idx, out["indices"][:out["total_rows"]])
