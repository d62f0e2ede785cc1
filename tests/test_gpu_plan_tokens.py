"""GPU parity of the token-granular plan (kap_compile_plan_masked, bit-exact
on every output including the token masks) and of decode over such a view
(kap_selected_decode_masked, within the attention tolerances)."""
import numpy as np
import pytest
import torch

from oracle import kap_oracle as O
from paper_2607_24260_amd import kap as K
from paper_2607_24260_amd.workloads import make_workload

from kap_testlib import (LSE_TOL, O_TOL, assert_close, assert_plan_equal, dev_i32, kv_of,
                         oracle_pool)

pytestmark = pytest.mark.gpu


def assert_masks_equal(gpu, plans):
    m = gpu["view_token_mask"].cpu().numpy().astype(np.int64) & 0xFFFFFFFF
    for b, p in enumerate(plans):
        if p.status == O.PLAN_OK:
            assert np.array_equal(m[b, :p.num_blocks], np.asarray(p.token_masks, np.int64)), b


def run_both(seq_lens, fbt, spans_per_seq, prefix, suffix, budget, policy=0, capacity=None,
             num_pages=None, offsets=None):
    B = len(seq_lens)
    fbt = np.asarray(fbt, dtype=np.int32).reshape(B, -1)
    st, ln, pr, offs = [], [], [], [0]
    for sp in spans_per_seq:
        for s in sp:
            st.append(s[0]); ln.append(s[1]); pr.append(s[2])
        offs.append(len(st))
    if offsets is not None:
        offs = offsets
    st = np.asarray(st, dtype=np.int32)
    ln = np.asarray(ln, dtype=np.int32)
    pr = np.asarray(pr, dtype=np.float32)
    cap = fbt.shape[1] if capacity is None else capacity
    npages = int(fbt.max()) + 1 if num_pages is None else num_pages
    gpu = K.compile_plan(
        dev_i32(seq_lens), dev_i32(fbt), dev_i32(offs), dev_i32(st), dev_i32(ln),
        torch.as_tensor(pr).cuda(), dev_i32(prefix), dev_i32(suffix), dev_i32(budget),
        num_pages=npages, view_capacity=cap, policy=policy, token_granular=True)
    torch.cuda.synchronize()
    plans = O.compile_plan(seq_lens, fbt, offs, st, ln, pr, prefix, suffix, budget, policy,
                           npages, cap, token_granular=True)
    assert_plan_equal(gpu, plans, offs)
    assert_masks_equal(gpu, plans)
    return gpu, plans


C1_FBT = [7, 3, 9, 0, 5, 2, 8]
C1_SPANS = [(20, 10, 0.5), (40, 30, 0.9), (90, 5, 0.9), (0, 5, 0.1)]


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("budget", [10, 24, 54, 56, 60, 66, 100, 1000])
def test_hand_vector(policy, budget):
    _, plans = run_both([100], C1_FBT, [C1_SPANS], [16], [8], [budget], policy=policy)
    if budget == 60:
        assert plans[0].token_masks == [0xFFFF, 0xFF00, 0xFFFF, 0x003F, 0xFC00, 0x000F]


def test_error_statuses_match():
    fbt = np.array([C1_FBT + [0], [1, 2, 3, 4, 5, 6, 7, 99]], dtype=np.int32)
    _, p = run_both([100, 100], fbt, [C1_SPANS, C1_SPANS], [16, 16], [8, 8], [60, 60],
                    capacity=3, num_pages=50)
    assert [x.status for x in p] == [O.PLAN_OVER_CAPACITY, O.PLAN_OVER_CAPACITY]
    _, p = run_both([100, 128], fbt, [C1_SPANS, [(0, 128, 1.0)]], [16, 0], [8, 1], [60, 128],
                    capacity=8, num_pages=50)
    assert [x.status for x in p] == [O.PLAN_OK, O.PLAN_BAD_PAGE]
    nan = [(20, 10, float("nan"))] + C1_SPANS[1:]
    run_both([100, 100], [C1_FBT, C1_FBT], [nan, C1_SPANS], [16, 16], [8, 8], [60, 60])
    _, p = run_both([0, 145], [C1_FBT + [0, 0], C1_FBT + [0, 0]], [C1_SPANS, C1_SPANS],
                    [16, 16], [8, 8], [60, 60])
    assert [x.status for x in p] == [O.PLAN_BAD_LENGTH, O.PLAN_BAD_LENGTH]
    _, p = run_both([100, 100], [C1_FBT, C1_FBT], [C1_SPANS, C1_SPANS], [16, 16], [8, 8],
                    [60, 60], offsets=[0, 4, 99])
    assert [x.status for x in p] == [O.PLAN_OK, O.PLAN_BAD_SPANS]


@pytest.mark.parametrize("seed", range(30))
def test_random_small(seed):
    # lengths across word and page boundaries, spans that overlap, touch the
    # ends, or are empty after clipping; +-0, +-inf priors
    rng = np.random.default_rng(2000 + seed)
    B = int(rng.integers(1, 6))
    seq_lens = rng.integers(1, 900, B)
    stride = int(-(-seq_lens.max() // 16))
    fbt = np.stack([rng.permutation(stride * B)[:stride] for _ in range(B)])
    spans = []
    for b in range(B):
        n = int(rng.integers(0, 40))
        L = int(seq_lens[b])
        spans.append([(int(rng.integers(-50, L + 30)), int(rng.integers(-5, 120)),
                       float(rng.choice([0.0, -0.0, 0.5, rng.random(), np.inf, -np.inf])))
                      for _ in range(n)])
    prefix = rng.integers(-10, 100, B)
    suffix = rng.integers(-10, 100, B)
    budget = rng.integers(-5, 900, B)
    cap = int(rng.integers(1, stride + 1))
    run_both(seq_lens, fbt, spans, prefix, suffix, budget, policy=int(seed % 2), capacity=cap,
             num_pages=stride * B)


def test_long_spans_and_many_spans():
    # one 65536-token sequence, 3000 spans (exact ties); spans longer than 64
    # bitmap words (2048 tokens) take several wavefront passes
    rng = np.random.default_rng(6)
    L = 65536
    stride = L // 16
    spans = [(int(rng.integers(0, L)), int(rng.integers(1, 600)), float(rng.random()))
             for _ in range(3000)]
    spans += [(int(rng.integers(0, L)), int(rng.integers(2048, 9000)), 0.97) for _ in range(6)]
    for s in range(0, 3000, 7):
        spans[s] = (spans[s][0], spans[s][1], 0.25)
    for budget in (3000, 20000):
        run_both([L], [rng.permutation(stride)], [spans], [500], [250], [budget])


def test_largest_supported_stride():
    # fbt_stride = 16384 pages (262144 tokens), one full-length sequence
    L = 16384 * 16
    rng = np.random.default_rng(8)
    spans = [(int(rng.integers(0, L)), int(rng.integers(1, 5000)), float(rng.random()))
             for _ in range(200)]
    run_both([L], [np.arange(16384)], [spans], [1000], [300], [60000])


@pytest.mark.parametrize("L", [16384 * 16, 16384 * 16 - 5])
@pytest.mark.parametrize("policy", [0, 1])
def test_spans_reaching_the_last_bitmap_word(L, policy):
    # Spans that end at L or are clipped there, single-token spans and spans
    # on word boundaries in the last words of the largest token bitmap: a
    # span's price counts the clear bits of its range eight words at a time
    # past its last word, and the end words by their bits inside the range.
    # With the mandatory last token, the hand-picked spans cost 39, 0, 255,
    # 0, 0, 33 and 160 tokens in rank order (488 in all), so a budget one
    # below that total rejects exactly the last of them.
    hand = [(L - 40, 40, 0.99), (L - 3, 10, 0.98), (L - 32 * 9 - 7, 300, 0.97),
            (L - 1, 1, 0.96), (L - 64, 1, 0.95), (L - 700, 33, 0.94),
            (L - 32 * 20, 32 * 5, 0.93)]
    rng = np.random.default_rng(11)
    rand = [(int(rng.integers(L - 3000, L)), int(rng.integers(1, 600)), float(rng.random()) * 0.9)
            for _ in range(60)]
    fbt = [np.arange(16384)]
    for budget in (488, 487, 489):
        gpu, plans = run_both([L], fbt, [hand], [0], [1], [budget], policy=policy)
        assert plans[0].view_tokens == (488 if budget >= 488 else 328)
    for budget in (100, 400, 1200, 2500):
        run_both([L], fbt, [hand + rand], [0], [1], [budget], policy=policy)


@pytest.mark.parametrize("config", [2, 4])
def test_workload_plans(config):
    w = make_workload(config, device="cuda", n_decode=1, n_verify=1, with_kv=False)
    gpu = K.compile_plan(
        dev_i32(w.seq_lens), dev_i32(w.full_block_table), dev_i32(w.span_offsets),
        dev_i32(w.span_start), dev_i32(w.span_len),
        torch.as_tensor(np.asarray(w.span_prior, dtype=np.float32)).cuda(), dev_i32(w.prefix),
        dev_i32(w.suffix), dev_i32(w.budget), num_pages=w.num_pages,
        view_capacity=w.max_pages_per_seq, token_granular=True)
    torch.cuda.synchronize()
    plans = O.compile_plan(w.seq_lens, w.full_block_table, w.span_offsets, w.span_start,
                           w.span_len, w.span_prior, w.prefix, w.suffix, w.budget, 0,
                           w.num_pages, w.max_pages_per_seq, token_granular=True)
    assert_plan_equal(gpu, plans, w.span_offsets)
    assert_masks_equal(gpu, plans)
    assert all(p.status == O.PLAN_OK for p in plans)
    # every visible token is within budget (the mandatory part fits these budgets)
    assert all(p.view_tokens <= int(bud) for p, bud in zip(plans, w.budget))


def token_plan(w, capacity=None):
    cap = w.max_pages_per_seq if capacity is None else capacity
    gpu = K.compile_plan(
        dev_i32(w.seq_lens), dev_i32(w.full_block_table), dev_i32(w.span_offsets),
        dev_i32(w.span_start), dev_i32(w.span_len),
        torch.as_tensor(np.asarray(w.span_prior, dtype=np.float32)).cuda(), dev_i32(w.prefix),
        dev_i32(w.suffix), dev_i32(w.budget), num_pages=w.num_pages, view_capacity=cap,
        token_granular=True)
    plans = O.compile_plan(w.seq_lens, w.full_block_table, w.span_offsets, w.span_start,
                           w.span_len, w.span_prior, w.prefix, w.suffix, w.budget, 0,
                           w.num_pages, cap, token_granular=True)
    torch.cuda.synchronize()
    return gpu, plans


@pytest.mark.parametrize("config,kw,num_splits", [
    (1, {}, 0),                                         # fp32: wide path
    (1, {}, 3),
    (2, dict(batch=3, seq_len=6000), 0),                # bf16: tuned, balanced map
    (2, dict(batch=3, seq_len=6000), 2),                # bf16: tuned, uniform splits
    (5, dict(batch=8, seq_len=20000), 0),               # fp8, ragged
])
def test_masked_decode_matches_oracle(config, kw, num_splits):
    w = make_workload(config, device="cuda", n_decode=1, n_verify=1, **kw)
    kv = kv_of(w)
    gpu, plans = token_plan(w)
    assert all(p.status == O.PLAN_OK for p in plans)
    q = w.q_decode[0]
    o, lse = K.selected_decode(kv, q, dev_i32(w.seq_lens), gpu["view_block_table"],
                               gpu["view_logical_block"], gpu["view_num_blocks"],
                               w.max_pages_per_seq, w.sm_scale, num_splits=num_splits,
                               view_token_mask=gpu["view_token_mask"])
    torch.cuda.synchronize()
    cap = w.max_pages_per_seq
    B = w.batch
    vbt = np.zeros((B, cap), np.int64)
    vlb = np.zeros((B, cap), np.int64)
    msk = np.zeros((B, cap), np.int64)
    for b, p in enumerate(plans):
        vbt[b, :p.num_blocks] = p.block_table
        vlb[b, :p.num_blocks] = p.logical_blocks
        msk[b, :p.num_blocks] = p.token_masks
    nb = [p.num_blocks for p in plans]
    eo, el = O.selected_decode(oracle_pool(w), q.float().cpu().numpy(), w.seq_lens, vbt, vlb,
                               nb, w.sm_scale, view_token_mask=msk)
    assert_close("masked decode O", o.cpu().numpy(), eo, O_TOL)
    assert_close("masked decode LSE", lse.cpu().numpy(), el, LSE_TOL)


def test_masked_decode_differs_from_page_view_and_full_masks_match_it():
    # partial masks change the result; all-ones masks give exactly the
    # page-granular call's result (same kernels, same order)
    w = make_workload(2, device="cuda", n_decode=1, n_verify=1, batch=4, seq_len=8000)
    kv = kv_of(w)
    gpu, _ = token_plan(w)
    args = (kv, w.q_decode[0], dev_i32(w.seq_lens), gpu["view_block_table"],
            gpu["view_logical_block"], gpu["view_num_blocks"], w.max_pages_per_seq, w.sm_scale)
    o_page, l_page = K.selected_decode(*args)
    ones = torch.full_like(gpu["view_token_mask"], 0xFFFF)
    o_ones, l_ones = K.selected_decode(*args, view_token_mask=ones)
    o_tok, _ = K.selected_decode(*args, view_token_mask=gpu["view_token_mask"])
    torch.cuda.synchronize()
    assert torch.equal(o_page, o_ones) and torch.equal(l_page, l_ones)
    assert not torch.equal(o_page, o_tok)


def test_empty_masks_see_no_key():
    w = make_workload(2, device="cuda", n_decode=1, n_verify=1, batch=2, seq_len=3000)
    kv = kv_of(w)
    gpu, _ = token_plan(w)
    zero = torch.zeros_like(gpu["view_token_mask"])
    o, lse = K.selected_decode(kv, w.q_decode[0], dev_i32(w.seq_lens), gpu["view_block_table"],
                               gpu["view_logical_block"], gpu["view_num_blocks"],
                               w.max_pages_per_seq, w.sm_scale, view_token_mask=zero)
    torch.cuda.synchronize()
    assert bool((o == 0).all()) and bool(torch.isinf(lse).all()) and bool((lse < 0).all())


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("n,longest", [(129, 1024), (700, 40), (2048, 1024), (150, 60000)])
def test_rankings_and_late_fits(n, longest, policy):
    # bucket ranking, the filter after the first rejection, spans of one or two
    # bitmap words (set by a lane each), of up to 33 and of up to 1875 (set by
    # all lanes together)
    from test_gpu_plan import ranked_spans
    rng = np.random.default_rng(n)
    lens = [65536, 9001]
    spans = [ranked_spans(n, "spread", L, rng, longest) for L in lens]
    spans[0] += [(int(s), 3, -5.0) for s in rng.integers(0, 65536, 30)]
    fbt = np.stack([rng.permutation(4096 * 2)[:4096] for _ in lens])
    run_both(lens, fbt, spans, [100, 0], [50, 1], [9000, 700], policy=policy, num_pages=8192)
