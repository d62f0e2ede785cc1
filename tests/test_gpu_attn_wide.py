"""The wide attention kernel (every geometry and dtype outside the tuned ones)
at the edges of its row tiles, row blocks and split merge, and with infinities
and NaNs in V, against the fp64 oracle.

Tolerance: float32 weights, sums and outputs. Over at most 700 keys of N(0, 1)
logits and values, each output is a weighted mean of unit values; 700 float32
roundings of relative size 2^-24 bound its error by 700 * 6e-8 = 4.2e-5, and
fp8 page scales by the same relative amount.
"""
import numpy as np
import pytest
import torch

from oracle import kap_oracle as O
from paper_2607_24260_amd import kap as K

from kap_testlib import assert_close, dev_i32

pytestmark = pytest.mark.gpu

TOL = 5e-5


def _inputs(kv_dtype, D, Hkv, lens, seed):
    r = np.random.default_rng(seed)
    npg = [-(-L // 16) for L in lens]
    P = sum(npg) + 3
    perm, at = r.permutation(P).astype(np.int32), 0
    fbt = np.full((len(lens), max(npg)), -1, np.int32)
    for b, n in enumerate(npg):
        fbt[b, :n] = perm[at:at + n]
        at += n
    x = [torch.as_tensor(r.standard_normal(s, dtype=np.float32))
         for s in ((P, Hkv, D // 8, 16, 8), (P, Hkv, D, 16))]
    sc = None
    if kv_dtype == "f32":
        k, v = (t.cuda() for t in x)
    elif kv_dtype == "bf16":
        k, v = (t.to(torch.bfloat16).cuda() for t in x)
    else:
        s = [t.abs().flatten(1).amax(1) / 448.0 for t in x]
        k, v = ((t / u.view(-1, *[1] * (t.dim() - 1))).to(torch.float8_e4m3fn)
                .view(torch.uint8).cuda() for t, u in zip(x, s))
        sc = torch.stack(s, 1).contiguous().cuda()
    return r, k, v, sc, fbt


def _pool(kv_dtype, k, v, sc):
    host = lambda t: (t.view(torch.int16) if t.dtype == torch.bfloat16 else t).cpu().numpy()
    hk, hv = host(k), host(v)
    if kv_dtype == "bf16":
        hk, hv = hk.view(np.uint16), hv.view(np.uint16)
    return O.KVPool(hk, hv, kv_dtype, None if sc is None else sc.cpu().numpy())


def _query(r, shape, kv_dtype):
    q = torch.as_tensor(r.standard_normal(shape, dtype=np.float32) / np.sqrt(shape[-1]))
    return q.to(torch.float32 if kv_dtype == "f32" else torch.bfloat16).cuda()


# (D, G, window): rows 1, 15 / 16 / 17, 32 / 33, 48, 64 / 65 (one to four tiles
# and the first split into row blocks), and 272 (17 float32 row blocks: more
# than the 16 arrival counters of a KV head)
ROWS = [(64, 1, 1), (128, 3, 5), (64, 2, 8), (128, 17, 1), (64, 2, 16), (128, 11, 3),
        (128, 6, 8), (64, 8, 8), (128, 13, 5), (128, 17, 16), (256, 1, 3), (256, 8, 4),
        (256, 3, 11)]


@pytest.mark.parametrize("kv_dtype", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("D,G,W", ROWS)
def test_rows_and_splits(kv_dtype, D, G, W):
    lens = [700, 33, 5]                     # 44, 3 and 1 pages; windows longer than 5 tokens
    Hkv = 2
    r, k, v, sc, fbt = _inputs(kv_dtype, D, Hkv, lens, D + 31 * G + W)
    pool = _pool(kv_dtype, k, v, sc)
    kv = K.KVCache(k, v, Hkv * G, _query(r, (1, 1), kv_dtype).dtype, sc)
    q = _query(r, (len(lens), W, Hkv * G, D), kv_dtype)
    eo, el = O.verify(pool, q.float().cpu().numpy(), np.asarray(lens), fbt, 1.0)
    seq = dev_i32(lens)
    for ns in (0, 1, 3, 100):
        print(f"verify {kv_dtype} D={D} G={G} W={W} splits={ns}", flush=True)
        o, lse = K.verify(kv, q, seq, dev_i32(fbt), 700, 1.0, num_splits=ns)
        torch.cuda.synchronize()
        assert_close(f"verify O ({ns} splits)", o.cpu().numpy(), eo, TOL)
        assert_close(f"verify LSE ({ns} splits)", lse.cpu().numpy(), el, TOL)
    # decode: a view in descending page order, every page's odd tokens hidden
    nb = [-(-L // 16) for L in lens]
    vbt, vlb = np.zeros_like(fbt), np.zeros_like(fbt)
    for b, n in enumerate(nb):
        vbt[b, :n], vlb[b, :n] = fbt[b, :n][::-1], np.arange(n)[::-1]
    mask = np.full(fbt.shape, 0x5555, np.int32)
    for mk in (None, mask):
        eo, el = O.selected_decode(pool, q[:, 0].float().cpu().numpy(), np.asarray(lens), vbt,
                                   vlb, nb, 1.0, view_token_mask=mk)
        for ns in (0, 3):
            print(f"decode {kv_dtype} D={D} G={G} masked={mk is not None} splits={ns}", flush=True)
            o, lse = K.selected_decode(kv, q[:, 0].contiguous(), seq, dev_i32(vbt), dev_i32(vlb),
                                       dev_i32(nb), fbt.shape[1], 1.0, num_splits=ns,
                                       view_token_mask=None if mk is None else dev_i32(mk))
            torch.cuda.synchronize()
            assert_close("decode O", o.cpu().numpy(), eo, TOL)
            assert_close("decode LSE", lse.cpu().numpy(), el, TOL)


@pytest.mark.parametrize("kv_dtype", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("num_splits", [0, 1, 3])
def test_infinities_and_nans_in_v_reach_only_the_rows_that_see_them(kv_dtype, num_splits):
    # a window of 4 over 70 tokens: V of token 67 is +inf in dim 3, of token 68
    # -inf in dim 5, of token 69 NaN in dim 7 (rows 1.., 2.. and 3 see them);
    # the slots past the end hold NaN, K included (fp8 has no infinities: NaN)
    D, G, W, L = 64, 3, 4, 70
    fp8 = kv_dtype == "fp8"
    nan = 0x7F if fp8 else np.nan
    r, k, v, sc, fbt = _inputs(kv_dtype, D, 1, [L], 5)
    clean_k, clean = k.clone(), v.clone()
    for tok, dim, x in ((67, 3, np.inf), (68, 5, -np.inf), (69, 7, np.nan)):
        v[int(fbt[0, tok // 16]), 0, dim, tok % 16] = nan if fp8 else x
        clean[int(fbt[0, tok // 16]), 0, dim, tok % 16] = 0
    last = int(fbt[0, L // 16])
    k[last, 0, :, L % 16:] = nan
    v[last, 0, :, L % 16:] = nan
    clean_k[last, 0, :, L % 16:] = 0
    clean[last, 0, :, L % 16:] = 0
    kv = K.KVCache(k, v, G, _query(r, (1, 1), kv_dtype).dtype, sc)
    q = _query(r, (1, W, G, D), kv_dtype)
    eo, el = O.verify(_pool(kv_dtype, clean_k, clean, sc),
                      q.float().cpu().numpy(), np.asarray([L]), fbt, 1.0)
    inf = np.nan if fp8 else np.inf
    eo[:, 1:, :, 3], eo[:, 2:, :, 5], eo[:, 3:, :, 7] = inf, -inf, np.nan
    o, lse = K.verify(kv, q, dev_i32([L]), dev_i32(fbt), L, 1.0, num_splits=num_splits)
    torch.cuda.synchronize()
    o = o.cpu().numpy()
    assert np.array_equal(np.isnan(o), np.isnan(eo))
    assert_close("O", np.nan_to_num(o, nan=0.0, posinf=np.inf, neginf=-np.inf),
                 np.nan_to_num(eo, nan=0.0, posinf=np.inf, neginf=-np.inf), TOL)
    assert_close("LSE", lse.cpu().numpy(), el, TOL)


@pytest.mark.parametrize("kv_dtype,D,G", [("bf16", 128, 4), ("fp8", 128, 4), ("bf16", 64, 3),
                                          ("fp8", 256, 4), ("f32", 128, 4)])
@pytest.mark.parametrize("step", [0.3, 0.7, -0.7, 3.5, -3.5, 7.0])
def test_logits_that_climb_from_page_to_page(kv_dtype, D, G, step):
    # every key of page p has the logit step * (p - 30). A wavefront's pages are
    # four apart (eight with two-page steps, more with splits): with 0.3 and 0.7
    # it climbs by 1.7 to 8 powers of two a step, so that several steps weigh up
    # to 2^8 against an older reference before it moves; with 3.5 and 7 (20 and
    # more) it moves at every step, upwards from -105; downwards it stays. fp8
    # page scales carry the value, negative ones included. Weights of the
    # tuned kernels are rounded to 2^-16 (of values up to about 4: 6e-5), LSEs
    # of up to 210 to a few 2^-23 of that.
    L = 44 * 16 - 3
    r, k, v, sc, fbt = _inputs(kv_dtype, D, 2, [L], 11)
    k.zero_()
    val = torch.zeros(k.shape[0], device="cuda")
    val[torch.as_tensor(fbt[0].astype(np.int64)).cuda()] = \
        step * (torch.arange(44, device="cuda") - 30).float()
    if kv_dtype == "fp8":
        k[:, :, 0, :, 0] = 0x38                                     # 1.0
        sc[:, 0] = val
    else:
        k[:, :, 0, :, 0] = val[:, None, None].to(k.dtype)
    qd = torch.float32 if kv_dtype == "f32" else torch.bfloat16
    kv = K.KVCache(k, v, 2 * G, qd, sc)
    q = torch.zeros((1, 5, 2 * G, D), dtype=qd, device="cuda")
    q[..., 0] = 1
    pool = _pool(kv_dtype, k, v, sc)
    lens, table = np.asarray([L]), dev_i32(np.arange(44)[None])
    for ns in (0, 1, 4):
        o, lse = K.verify(kv, q, dev_i32([L]), dev_i32(fbt), L, 1.0, num_splits=ns)
        od, ld = K.selected_decode(kv, q[:, 0].contiguous(), dev_i32([L]), dev_i32(fbt), table,
                                   dev_i32([44]), 44, 1.0, num_splits=ns)
        torch.cuda.synchronize()
        eo, el = O.verify(pool, q.float().cpu().numpy(), lens, fbt, 1.0)
        assert_close("verify O", o.cpu().numpy(), eo, 1e-4)
        assert_close("verify LSE", lse.cpu().numpy(), el, 1e-4)
        eo, el = O.selected_decode(pool, q[:, 0].float().cpu().numpy(), lens, fbt,
                                   np.arange(44)[None], [44], 1.0)
        assert_close("decode O", od.cpu().numpy(), eo, 1e-4)
        assert_close("decode LSE", ld.cpu().numpy(), el, 1e-4)


@pytest.mark.parametrize("kv_dtype,D,G", [("f32", 64, 3), ("bf16", 64, 3), ("fp8", 64, 3),
                                          ("f32", 128, 4), ("bf16", 128, 2), ("fp8", 256, 5),
                                          ("bf16", 128, 4), ("fp8", 128, 4)])
@pytest.mark.parametrize("where", ["k", "q"])
@pytest.mark.parametrize("num_splits", [0, 1])
def test_a_nan_logit_reaches_the_rows_that_see_it(kv_dtype, D, G, where, num_splits):
    # 700 tokens: with the automatic splits a wavefront has one step, so the
    # one that meets the NaN has no other logit; with one split it has several.
    # K: tokens 100 and 698 (seen by the last two rows of the window of 4) of KV
    # head 0. Q: window token 1 of the last query head.
    L, W, Hkv = 700, 4, 2
    r, k, v, sc, fbt = _inputs(kv_dtype, D, Hkv, [L], 17)
    kv = K.KVCache(k, v, Hkv * G, _query(r, (1, 1), kv_dtype).dtype, sc)
    q = _query(r, (1, W, Hkv * G, D), kv_dtype)
    pool = _pool(kv_dtype, k, v, sc)
    nan = 0x7F if kv_dtype == "fp8" else np.nan
    for toks in ((698,), (100, 698)) if where == "k" else ((),):
        eo, el = (x.copy() for x in O.verify(pool, q.float().cpu().numpy(), np.asarray([L]), fbt,
                                             1.0))
        kn, qn = k.clone(), q.clone()
        for tok in toks:
            kn[int(fbt[0, tok // 16]), 0, 1, tok % 16, 3] = nan
            first = max(0, tok - (L - W))            # rows first.. see the token
            eo[:, first:, :G], el[:, first:, :G] = np.nan, np.nan
        if where == "q":
            qn[0, 1, -1, 5] = np.nan
            eo[0, 1, -1], el[0, 1, -1] = np.nan, np.nan
        kv = K.KVCache(kn, v, Hkv * G, q.dtype, sc)
        calls = [("verify", K.verify(kv, qn, dev_i32([L]), dev_i32(fbt), L, 1.0,
                                     num_splits=num_splits), eo, el)]
        if 100 in toks or where == "q":
            # decode of the window's last (Q: second) row over the whole context:
            # the last row sees every key, the second one every key but two
            i = 1 if where == "q" else W - 1
            do, dl = (x.copy() for x in O.selected_decode(
                pool, q[:, i].float().cpu().numpy(), np.asarray([L]), fbt,
                np.arange(fbt.shape[1])[None], [fbt.shape[1]], 1.0))
            if where == "q":
                do[0, -1], dl[0, -1] = np.nan, np.nan
            else:
                do[:, :G], dl[:, :G] = np.nan, np.nan
            calls.append(("decode", K.selected_decode(
                kv, qn[:, i].contiguous(), dev_i32([L]), dev_i32(fbt),
                dev_i32(np.arange(fbt.shape[1])[None]), dev_i32([fbt.shape[1]]), fbt.shape[1], 1.0,
                num_splits=num_splits), do, dl))
        torch.cuda.synchronize()
        # tuned kernels (128 dims, four heads): weights rounded to 2^-16
        tol = 1e-4 if (D, G) == (128, 4) and kv_dtype != "f32" else TOL
        for name, (o, lse), xo, xl in calls:
            for part, got, want in (("O", o, xo), ("LSE", lse, xl)):
                got = got.cpu().numpy()
                assert np.array_equal(np.isnan(got), np.isnan(want)), f"{name} {part}: NaN rows"
                assert_close(f"{name} {part}", np.nan_to_num(got), np.nan_to_num(want), tol)


@pytest.mark.parametrize("kv_dtype,D,G,W", [("bf16", 128, 4, 5), ("bf16", 128, 4, 12),
                                            ("fp8", 128, 4, 9), ("fp8", 128, 4, 16),
                                            ("f32", 64, 3, 5), ("bf16", 64, 3, 5),
                                            ("fp8", 256, 4, 5), ("bf16", 128, 8, 8)])
@pytest.mark.parametrize("num_splits", [0, 1])
def test_values_near_the_largest_float(kv_dtype, D, G, W, num_splits):
    # |V| up to 2^120 under logits that climb by 0.3 (0.43 powers of two) a page:
    # with weights of at most 1 a wavefront's sums stay below 2^120 * 16 * 2 *
    # sum(2^(-0.43 k)) < 2^127; with weights of 2^7 against an older reference
    # they would not. Tolerances relative to 2^120.
    L, big = 44 * 16, 2.0 ** 120
    r, k, v, sc, fbt = _inputs(kv_dtype, D, 2, [L], 23)
    k.zero_()
    val = torch.zeros(k.shape[0], device="cuda")
    val[torch.as_tensor(fbt[0].astype(np.int64)).cuda()] = \
        0.3 * (torch.arange(44, device="cuda") + 1).float()
    if kv_dtype == "fp8":
        k[:, :, 0, :, 0] = 0x38                                     # 1.0
        sc[:, 0] = val
        sc[:, 1] = big / 448
    else:
        k[:, :, 0, :, 0] = val[:, None, None].to(k.dtype)
        v = (v.float() / v.float().abs().max() * big).to(v.dtype)
    qd = torch.float32 if kv_dtype == "f32" else torch.bfloat16
    kv = K.KVCache(k, v, 2 * G, qd, sc)
    q = torch.zeros((1, W, 2 * G, D), dtype=qd, device="cuda")
    q[..., 0] = 1
    pool = _pool(kv_dtype, k, v, sc)
    lens, table = np.asarray([L]), np.arange(44)[None]
    print(f"verify, decode {kv_dtype} D={D} G={G} W={W} splits={num_splits}", flush=True)
    o, lse = K.verify(kv, q, dev_i32([L]), dev_i32(fbt), L, 1.0, num_splits=num_splits)
    od, ld = K.selected_decode(kv, q[:, 0].contiguous(), dev_i32([L]), dev_i32(fbt),
                               dev_i32(table), dev_i32([44]), 44, 1.0, num_splits=num_splits)
    torch.cuda.synchronize()
    eo, el = O.verify(pool, q.float().cpu().numpy(), lens, fbt, 1.0)
    assert_close("verify O", o.cpu().numpy() / big, eo / big, 1e-4)
    assert_close("verify LSE", lse.cpu().numpy(), el, 1e-4)
    eo, el = O.selected_decode(pool, q[:, 0].float().cpu().numpy(), lens, fbt, table, [44], 1.0)
    assert_close("decode O", od.cpu().numpy() / big, eo / big, 1e-4)
    assert_close("decode LSE", ld.cpu().numpy(), el, 1e-4)


@pytest.mark.parametrize("batch", [64, 70])
@pytest.mark.parametrize("op", ["decode", "verify"])
def test_a_long_sequence_among_many_short_ones_is_split(batch, op):
    # 16 KV heads: with 64 and more sequences every (sequence, KV head) gets a
    # workgroup four times over; up to 64 sequences the balanced map splits,
    # above that every sequence by its own length (1030 pages: four pieces of
    # 258, 300 pages: two). Tolerance: 16480 keys of near-equal weight, whose
    # float32 sums' errors grow with the square root: 130 * 6e-8, fourfold.
    D, Hkv, W = 128, 16, 2
    lens = [1030 * 16, 300 * 16 - 5] + [1 + (7 * i) % 40 for i in range(batch - 2)]
    r, k, v, sc, fbt = _inputs("bf16", D, Hkv, lens, 31)
    kv = K.KVCache(k, v, Hkv, torch.bfloat16, sc)
    q = _query(r, (batch, W, Hkv, D), "bf16")
    pool = _pool("bf16", k, v, sc)
    seq, M = dev_i32(lens), fbt.shape[1]
    heads = (0, 7, 15)
    for ns in (0, 1):                       # 1: pieces of at most 64 pages (17 for the longest)
        print(f"{op} batch={batch} splits={ns}", flush=True)
        if op == "verify":
            assert K.verify_workspace_bytes(kv, batch, W, max(lens), ns) > 0
            o, lse = K.verify(kv, q, seq, dev_i32(fbt), max(lens), 1.0, num_splits=ns)
            eo, el = O.verify(pool, q.float().cpu().numpy(), np.asarray(lens), fbt, 1.0,
                              kv_heads=heads)
        else:
            assert K.selected_decode_workspace_bytes(kv, batch, M, ns) > 0
            nb = [-(-L // 16) for L in lens]
            vlb = np.tile(np.arange(M, dtype=np.int32), (batch, 1))
            args = (kv, q[:, 0].contiguous(), seq, dev_i32(fbt), dev_i32(vlb), dev_i32(nb), M, 1.0)
            o, lse = K.selected_decode(*args, num_splits=ns)
            eo, el = (x[:, 0] for x in O.verify(pool, q[:, :1].float().cpu().numpy(),
                                                np.asarray(lens), fbt, 1.0, kv_heads=heads))
        torch.cuda.synchronize()
        at = (..., list(heads), slice(None))
        assert_close("O", o.cpu().numpy()[at], eo[at], TOL)
        assert_close("LSE", lse.cpu().numpy()[at[:-1]], el[at[:-1]], TOL)


def test_a_split_count_is_a_least_count_outside_the_tuned_geometry():
    # pieces of at most 64 pages, whatever count is asked for
    k = torch.zeros((4, 2, 8, 16, 8), device="cuda")
    v = torch.zeros((4, 2, 64, 16), device="cuda")
    kv = K.KVCache(k, v, 4, torch.float32)
    size = lambda ns, pages=256: K.selected_decode_workspace_bytes(kv, 1, pages, ns)
    assert size(1) == size(2) == size(4) > 0 and size(8) > size(4)
    assert size(1, 64) == 0
    size = lambda ns: K.verify_workspace_bytes(kv, 1, 3, 256 * 16, ns)
    assert size(1) == size(4) > 0
