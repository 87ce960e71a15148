"""Combining a head's chunks in a decoding step with 256 and 1024 threads: caches on either side of the line between them, every head
dimension, heads of very different sizes, against attention in float64."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import paper_2604_06694_amd as A
    return A


# one head, two of which one is nearly empty, five: three rounds of 1024 / D chunks of 128 rows per head, one row fewer, many more
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("H", [1, 2, 5])
@pytest.mark.parametrize("rows", [0, -1, 1, 20000])
def test_merge_threads(A, D, H, rows):
    total = 3 * (1024 // D) * 128 * H + rows
    counts = np.full(H, total // H)
    counts[0] += total - counts.sum()
    if H == 2:
        counts = np.array([1, total - 1])
    cu = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(total)
    G = 7 if D == 128 else 3
    q = torch.randn(H * G, D, generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn(total, D, generator=gen, device="cuda").to(torch.bfloat16)
    v = torch.randn(total, D, generator=gen, device="cuda").to(torch.bfloat16)
    p = A.Params(H * G, H, D, 1)
    got = A.decode_attend(p, q.reshape(-1), k, v, cu, 1, total).view(H, G, D).double()
    at = cu.cpu().tolist()
    for h in range(H):
        z = q.view(H, G, D)[h].double() @ k[at[h]:at[h + 1]].double().t().contiguous() / D ** 0.5
        ref = torch.softmax(z, dim=1) @ v[at[h]:at[h + 1]].double()
        # fp32 logits of up to about 5 in size, weights and sums over up to 20000 rows in a few hundred partial sums: 1e-5 of the largest
        assert (got[h] - ref).abs().max() <= 1e-5 * ref.abs().max() + 1e-7
