"""Combining a head's chunks in a decoding step with 256 and 1024 threads: caches on either side of the line between them at d = 128 and
256 (d = 64 always takes 256), heads of very different sizes, against attention in float64."""
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


@pytest.mark.parametrize("n", [32, 33])
def test_merge_of_many_caches(A, n):
    """512 workgroups and a few more, either side of the other line between the two."""
    D, G, rows = 128, 16, 24 * 128 + 5
    cu = torch.arange(n + 1, dtype=torch.int32, device="cuda") * rows
    gen = torch.Generator(device="cuda").manual_seed(n)
    q = torch.randn(n, G, D, generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn(n, rows, D, generator=gen, device="cuda").to(torch.bfloat16)
    v = torch.randn(n, rows, D, generator=gen, device="cuda").to(torch.bfloat16)
    got = A.decode_attend(A.Params(G, 1, D, 1), q.reshape(-1), k.view(-1, D), v.view(-1, D), cu, n, n * rows).view(n, G, D).double()
    z = torch.matmul(q.double(), k.double().transpose(1, 2).contiguous()) / D ** 0.5
    ref = torch.matmul(torch.softmax(z, dim=2), v.double())
    # (the bound of test_merge_threads)
    assert (got - ref).abs().max() <= 1e-5 * ref.abs().max() + 1e-7
