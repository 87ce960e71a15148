"""GPU parity of the decode-side consumer (single-query attention over the
packed, per-head-ragged compacted cache) against the float64 oracle, through
the C ABI. Tolerance: the floored relative error used for the scores (2e-3),
plus a much tighter absolute guard, since the arithmetic is fp32 throughout."""
import numpy as np
import pytest
import torch

from oracle import audiokv_oracle as O
from workloads import bf16_bits_to_f64, f64_to_bf16_bits, gen_item, gen_weights, get_config

from gpu_util import SCORE_RTOL, bf16_bits, bf16_tensor, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import paper_2604_06694_amd as A
    return A


def run_case(A, rng, H_q, H_kv, d, budgets, n_items, *, k_scale=1.0, total_rows=None, scale=0.0):
    n_heads = n_items * H_kv
    assert len(budgets) == n_heads
    cu = np.concatenate([[0], np.cumsum(budgets)]).astype(np.int32)
    rows = int(cu[-1])
    kb = f64_to_bf16_bits(k_scale * rng.standard_normal((rows, d)))
    vb = f64_to_bf16_bits(rng.standard_normal((rows, d)))
    qb = f64_to_bf16_bits(rng.standard_normal((n_items, H_q, d)))
    p = A.Params(H_q, H_kv, d, 1, softmax_scale=scale)
    tr = rows if total_rows is None else total_rows
    out = A.decode_attend(p, bf16_tensor(qb.reshape(-1)), bf16_tensor(kb.reshape(-1)), bf16_tensor(vb.reshape(-1)),
                          torch.from_numpy(cu).cuda(), n_items, tr)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    kf, vf, qf = bf16_bits_to_f64(kb), bf16_bits_to_f64(vb), bf16_bits_to_f64(qb)
    sc = None if scale == 0.0 else float(np.float32(scale))
    for i in range(n_items):
        kr = [kf[cu[i * H_kv + h]:min(cu[i * H_kv + h + 1], tr)] for h in range(H_kv)]
        vr = [vf[cu[i * H_kv + h]:min(cu[i * H_kv + h + 1], tr)] for h in range(H_kv)]
        ref = O.decode_attend(qf[i], kr, vr, scale=sc)
        assert rel_err(out[i], ref) <= SCORE_RTOL, (i, rel_err(out[i], ref))
        assert np.abs(out[i] - ref).max() <= 1e-4 * max(np.abs(ref).max(), 1e-3)
    return out


@pytest.mark.parametrize("H_q,H_kv,d", [(28, 4, 128), (8, 8, 64), (8, 2, 256), (32, 2, 128), (32, 4, 128), (6, 2, 64),
                                         (32, 2, 256)])
def test_decode_ragged_budgets(A, H_q, H_kv, d):
    rng = np.random.default_rng(H_q * 1000 + d)
    n_items = 2
    pool = [1, 5, 16, 17, 511, 512, 513, 1500, 64, 1024]
    budgets = [int(pool[(3 * g + H_q) % len(pool)]) for g in range(n_items * H_kv)]
    run_case(A, rng, H_q, H_kv, d, budgets, n_items)


def test_decode_long_heads_and_peaked_softmax(A):
    rng = np.random.default_rng(5)
    # many chunks per head; large keys make the softmax sharp (logits up to ~ +-60)
    run_case(A, rng, 28, 4, 128, [32768, 13107, 6554, 700], 1, k_scale=4.0)
    run_case(A, rng, 8, 2, 256, [9000, 3000], 1, k_scale=0.05, scale=0.5)


def test_decode_one_very_long_head(A):
    # about a thousand chunks in one head, several per thread of the merge
    rng = np.random.default_rng(8)
    run_case(A, rng, 1, 1, 64, [1024 * 256 + 300], 1, k_scale=0.5)
    run_case(A, rng, 9, 1, 64, [512 * 256 + 7], 1, k_scale=0.5)          # 16-wide group padding: 512-row chunks


def test_decode_total_rows_bounds_the_reads_and_errors(A):
    rng = np.random.default_rng(6)
    run_case(A, rng, 8, 2, 128, [2000, 300], 1, total_rows=2100)      # rows at or past total_rows are not read
    p = A.Params(8, 2, 128, 1)
    q = torch.zeros(8 * 128, dtype=torch.bfloat16, device="cuda")
    kv = torch.zeros(10 * 128, dtype=torch.bfloat16, device="cuda")
    cu = torch.tensor([0, 5, 10], dtype=torch.int32, device="cuda")
    with pytest.raises(A.AudioKVError) as e:
        A.decode_attend(p, q, kv, kv, cu, 1, 10, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    assert e.value.code == -3
    with pytest.raises(A.AudioKVError) as e:
        A.decode_attend(A.Params(34, 2, 128, 1), q, kv, kv, cu, 1, 10)
    assert e.value.code == -2
    with pytest.raises(A.AudioKVError) as e:
        A.decode_attend(p, q, kv, kv, cu, 1, -1)
    assert e.value.code == -1
    # zero query: the mean of the retained rows; an empty head gives zeros
    v = torch.arange(10 * 128, dtype=torch.float32, device="cuda").remainder(7).to(torch.bfloat16)
    cu0 = torch.tensor([0, 10, 10], dtype=torch.int32, device="cuda")
    out = A.decode_attend(p, q, kv, v, cu0, 1, 10).cpu().numpy()
    want = v.float().view(10, 128).mean(0).cpu().numpy()
    np.testing.assert_allclose(out[0, :4], np.tile(want, (4, 1)), rtol=1e-6)
    assert np.all(out[0, 4:] == 0.0)


def test_decode_consumes_the_output_of_evict(A):
    cfg = get_config(1, n_items=2)
    items = [gen_item(cfg, i) for i in range(cfg.n_items)]
    L = cfg.seqlen
    q = bf16_tensor(np.concatenate([it["q_win"].reshape(-1) for it in items]))
    k = bf16_tensor(np.concatenate([it["k"].reshape(-1) for it in items]))
    v = bf16_tensor(np.concatenate([it["v"].reshape(-1) for it in items]))
    w = torch.from_numpy(gen_weights(cfg)).cuda()
    p = A.Params(cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.window, pool_kernel=cfg.pool_kernel,
                 floor_frac=cfg.floor_frac)
    ev = A.evict(p, q, k, v, w, [L] * cfg.n_items, cfg.ratio, cfg.cutoff, cfg.alpha, alloc_scope=A.SCOPE_GLOBAL)
    # the next query: the last window row of every query head stands in for the first generated token's query
    qn_bits = np.stack([it["q_win"][:, -1, :] for it in items])              # [items, H_q, d]
    out = A.decode_attend(p, bf16_tensor(qn_bits.reshape(-1)), ev["k_out"], ev["v_out"], ev["cu_budgets"],
                          cfg.n_items, ev["total_rows"])
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    cu = ev["cu_budgets"].cpu().numpy(); idx = ev["indices"].cpu().numpy()
    for i, it in enumerate(items):
        kr, vr = [], []
        for h in range(cfg.n_kv_heads):
            g = i * cfg.n_kv_heads + h
            mine = idx[cu[g]:cu[g + 1]]
            kr.append(bf16_bits_to_f64(it["k"][h][mine])); vr.append(bf16_bits_to_f64(it["v"][h][mine]))
        ref = O.decode_attend(bf16_bits_to_f64(qn_bits[i]), kr, vr)
        assert rel_err(out[i], ref) <= SCORE_RTOL
        assert np.abs(out[i] - ref).max() <= 1e-4 * np.abs(ref).max()


@pytest.mark.parametrize("H_q,H_kv,d,n_items,budgets", [
    (4, 2, 64, 35, lambda g: (2, 1, 127, 128, 129, 300)[g % 6]),       # more than 64 heads: two rounds of the head search
    (14, 2, 128, 2, lambda g: (128, 256, 128, 257)[g]),                # chunk starts that fall on multiples of the chunk
    (10, 1, 256, 3, lambda g: (1, 513, 127)[g]),
    (8, 1, 128, 1, lambda g: 128 * 2048 - 1),                          # the longest call of 128-row chunks, 2048 for one head
    (8, 1, 128, 1, lambda g: 128 * 2048),                              # the shortest of 256-row chunks
    (3, 1, 256, 2, lambda g: (1024 * 512 - 5, 5)[g]),                  # the same edge one chunk size up, ending in a short head
])
def test_decode_chunk_edges(A, H_q, H_kv, d, n_items, budgets):
    run_case(A, np.random.default_rng(n_items * d), H_q, H_kv, d, [budgets(g) for g in range(n_items * H_kv)], n_items,
             k_scale=0.5)


def test_decode_more_chunks_than_weights_fit_on_chip(A):
    # 16-wide group padding: chunks of at most 512 rows, 2051 of them in one head
    run_case(A, np.random.default_rng(9), 9, 1, 64, [2050 * 512 + 9], 1, k_scale=0.5)


def test_decode_empty_heads_between_full_ones(A):
    # zero queries: every head's output is the mean of its own rows, zeros for the heads that kept none
    n, d, pool = 130, 64, (0, 0, 128, 1, 0, 129, 256)
    budgets = np.array([pool[g % 7] for g in range(n)])
    cu = np.concatenate([[0], np.cumsum(budgets)]).astype(np.int32)
    v = torch.arange(int(cu[-1]), dtype=torch.float32).remainder(251).repeat_interleave(d).to(torch.bfloat16).cuda()
    q = torch.zeros(n * d, dtype=torch.bfloat16, device="cuda")
    out = A.decode_attend(A.Params(1, 1, d, 1), q, v, v, torch.from_numpy(cu).cuda(), n, int(cu[-1])).cpu().numpy()
    want = [(np.arange(cu[g], cu[g + 1]) % 251).mean() if budgets[g] else 0.0 for g in range(n)]
    np.testing.assert_allclose(out[:, 0], np.repeat(np.array(want)[:, None], d, 1), rtol=2e-6)     # fp32 sums of <= 256 terms


@pytest.mark.parametrize("d,groups", [(64, 16), (128, 8), (256, 4)])
def test_decode_merge_around_the_accumulators_requested_early(A, d, groups):
    """Chunks per head on either side of what a thread of the merge requests before it knows the statistics (four per
    thread, `groups` threads on a channel), of one thread's share and of nothing. Chunks hold 128 rows at these sizes."""
    rng = np.random.default_rng(d)
    edge = 4 * groups * 128
    run_case(A, rng, 8, 4, d, [edge, edge + 1, edge - 127, 129], 1)
    run_case(A, rng, 4, 4, d, [groups * 128, groups * 128 + 1, 1, edge + groups * 128 + 1], 1)


@pytest.mark.parametrize("H_q,d", [(2, 64), (7, 128), (3, 256), (12, 64), (16, 256)])
def test_decode_infinity_in_the_last_row_of_a_head(A, H_q, d):
    """An infinite value is what its channel becomes, whatever the budget (the rows that fill up a trip carry weight 0 and
    must not turn it into NaN); the other channels and heads are the means of their rows (zero queries)."""
    budgets = [1, 5, 16, 17, 127, 128, 129, 300]
    n = len(budgets)
    cu = np.concatenate([[0], np.cumsum(budgets)]).astype(np.int32)
    v = (np.arange(int(cu[-1])) % 7).astype(np.float32)[:, None].repeat(d, 1)
    last = cu[1:] - 1
    want = np.array([v[cu[g]:cu[g + 1], 0].mean() for g in range(n)])
    v[last, 3] = np.inf
    v[last, d - 1] = -np.inf
    vt = torch.from_numpy(v).to(torch.bfloat16).cuda()
    kt = torch.zeros_like(vt)
    q = torch.zeros(n * H_q * d, dtype=torch.bfloat16, device="cuda")
    out = A.decode_attend(A.Params(H_q, 1, d, 1), q, kt.view(-1), vt.view(-1), torch.from_numpy(cu).cuda(), n, int(cu[-1]))
    out = out.cpu().numpy().reshape(n, H_q, d)
    assert np.all(out[:, :, 3] == np.inf) and np.all(out[:, :, d - 1] == -np.inf)
    rest = np.delete(out, [3, d - 1], axis=2)
    np.testing.assert_allclose(rest, np.broadcast_to(want[:, None, None], rest.shape), rtol=2e-6)    # fp32 sums of <= 300 terms


def test_decode_workspace_of_the_largest_call_serves_smaller_ones(A):
    """One workspace sized for the largest cache, calls on either side of the sizes at which the chunks double; the bytes
    behind what such a call asks for stay untouched."""
    H_q, H_kv, d, n = 4, 4, 64, 1
    p = A.Params(H_q, H_kv, d, 1)
    most = 600_000
    ws = torch.empty(A.decode_workspace_bytes(p, n, most), dtype=torch.uint8, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(1)
    k, v = (torch.randn(most * d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    q = torch.randn(H_q * d, generator=gen, device="cuda").to(torch.bfloat16)
    for rows in (most, 524_288, 524_287, 262_144, 262_143, 200_000, 1000, 3):
        cu = torch.tensor([0, rows // 3, rows // 2, rows - 1, rows], dtype=torch.int32, device="cuda")
        need = A.decode_workspace_bytes(p, n, rows)
        ws.fill_(7)
        got = A.decode_attend(p, q, k, v, cu, n, rows, workspace=ws)
        assert torch.equal(got, A.decode_attend(p, q, k, v, cu, n, rows))
        assert bool((ws[need:] == 7).all())


@pytest.mark.parametrize("H_q,H_kv,d", [(8, 2, 64), (28, 4, 128), (8, 2, 256), (32, 2, 128)])
def test_decode_takes_a_cache_at_any_element(A, H_q, H_kv, d):
    """Queries and cache that start at any bf16 element, as slices of larger buffers do, give the bits of aligned copies."""
    rows, n = 1003, 1
    gen = torch.Generator(device="cuda").manual_seed(d)
    bufs = [torch.randn(m + 8, generator=gen, device="cuda").to(torch.bfloat16) for m in (H_q * d, rows * d, rows * d)]
    cu = torch.tensor([rows * i // H_kv for i in range(H_kv + 1)], dtype=torch.int32, device="cuda")
    p = A.Params(H_q, H_kv, d, 1)
    for off in (0, 1, 2, 3, 4, 7):
        parts = [b[off:b.numel() - 8 + off] for b in bufs]
        got = A.decode_attend(p, *parts, cu, n, rows)
        assert torch.equal(got, A.decode_attend(p, *[x.clone() for x in parts], cu, n, rows))
