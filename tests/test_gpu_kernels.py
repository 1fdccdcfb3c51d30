"""Kernels at the sizes where their tiling can go wrong, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_helpers import check_close, i32_dev, mask_from_bits, to_dev, to_host, vt_layout
from paper_2510_21270_amd import binding as pbs
from paper_2510_21270_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _qkv(seed, Hq, Hkv, n, d, dtype):
    rng = np.random.default_rng(seed)
    x = [rng.standard_normal((1, h, n, d)).astype(np.float32) for h in (Hq, Hkv, Hkv)]
    return [wl.round_to_bf16(a) for a in x] if dtype == "bf16" else x


# n: one query, one query past a 16-query tile, one short of a block, several blocks and a ragged tail; few workgroups and
# (34 heads) several to a compute unit
@pytest.mark.parametrize("n", [1, 17, 127, 700])
@pytest.mark.parametrize("dtype,d,block,Hq,Hkv", [("f32", 64, 16, 2, 1), ("f32", 64, 64, 34, 2), ("f32", 128, 32, 3, 3),
                                                   ("f32", 128, 128, 34, 34), ("bf16", 64, 32, 2, 2),
                                                   ("bf16", 128, 16, 34, 2)])
def test_fp32_attention_over_given_lists(oracle, dtype, d, block, Hq, Hkv, n):
    Q, K, V = _qkv(n + d, Hq, Hkv, n, d, dtype)
    T, seg = -(-n // block), 2 * block
    kidx = wl.random_segment_perm(3, Hkv, n, seg).reshape(1, Hkv, n)
    Kp, Vp = oracle.gather_rows(K, kidx), oracle.gather_rows(V, kidx)
    cnt, cols = wl.random_block_lists(5, 1, Hq, T, 0.5)
    p = pbs.problem(1, Hq, Hkv, n, d, block, seg, dtype)
    want, want_lse = oracle.attn_fwd(Q, Kp, Vp, None, kidx, cnt, cols, block, want_lse=True)
    got, lse = pbs.attn_fwd(p, to_dev(Q, dtype), to_dev(Kp, dtype), to_dev(vt_layout(Vp, block), dtype), None,
                            i32_dev(kidx), i32_dev(cnt), i32_dev(cols), want_lse=True)
    torch.cuda.synchronize()
    lse = lse.cpu().numpy()
    fin = np.isfinite(want_lse)                            # a query that sees no listed key: zeros and -inf
    assert np.isneginf(lse[~fin]).all()
    check_close(to_host(got), np.where(fin[..., None], want, 0.0), dtype, "fp32 kernel")
    np.testing.assert_allclose(lse[fin], want_lse[fin], atol=1e-4, rtol=0)


# ... and the d = 64 kernel, 64 queries to a tile: short of one, one past it, ragged blocks, a T of its own; four waves
# share a list (all of them, or fewer entries than waves) up to 4096 tiles, one wave has it to itself from there on
@pytest.mark.parametrize("block,Hq,Hkv,n,rho", [(b, hq, hkv, n, 0.5) for b, hq, hkv in [(64, 4, 2), (128, 3, 1), (64, 7, 7)]
                                                for n in (1, 65, 190, 900)] + [(64, 64, 2, 16410, 0.02)])
def test_d64_attention_over_given_lists(oracle, block, Hq, Hkv, n, rho):
    Q, K, V = _qkv(n + block, Hq, Hkv, n, 64, "bf16")
    Q[0, :, n // 2:] *= 8.0                                # scores that outgrow the first reference
    T, seg = -(-n // block), 2 * block
    kidx = wl.random_segment_perm(3, Hkv, n, seg).reshape(1, Hkv, n)
    qidx = wl.random_segment_perm(4, Hq, n, seg).reshape(1, Hq, n)
    Qp, Kp, Vp = oracle.gather_rows(Q, qidx), oracle.gather_rows(K, kidx), oracle.gather_rows(V, kidx)
    cnt, cols = wl.random_block_lists(5, 1, Hq, T, rho)
    p = pbs.problem(1, Hq, Hkv, n, 64, block, seg, "bf16")
    want, want_lse = oracle.attn_fwd(Qp, Kp, Vp, qidx, kidx, cnt, cols, block, want_lse=True)
    got, lse = pbs.attn_fwd(p, to_dev(Qp, "bf16"), to_dev(Kp, "bf16"), to_dev(vt_layout(Vp, block), "bf16"),
                            i32_dev(qidx), i32_dev(kidx), i32_dev(cnt), i32_dev(cols), want_lse=True)
    torch.cuda.synchronize()
    lse = lse.cpu().numpy()
    fin = np.isfinite(want_lse)
    assert np.isneginf(lse[~fin]).all()
    check_close(to_host(got), np.where(fin[..., None], want, 0.0), "bf16", "d = 64 kernel")
    np.testing.assert_allclose(lse[fin], want_lse[fin], atol=1e-4, rtol=0)


# (float32, d = 128, blocks of 32 and more: sub-tiles are halves of a group of 32 keys; later: the key in the second half)
@pytest.mark.parametrize("dtype,d,block,later", [("f32", 64, 64, 0), ("f32", 128, 16, 0), ("bf16", 64, 32, 0), ("bf16", 64, 64, 0),
                                                 ("bf16", 64, 128, 0), ("f32", 128, 32, 3), ("f32", 128, 128, 19)])
def test_values_that_are_not_finite_reach_only_the_queries_that_see_them(oracle, dtype, d, block, later):
    n, at = 3 * block - 5, block + block // 2 + later
    Q, K, V = _qkv(7, 2, 1, n, d, dtype)
    kidx = np.arange(n, dtype=np.int32).reshape(1, 1, n)
    p = pbs.problem(1, 2, 1, n, d, block, block, dtype)
    cnt, cols = pbs.admitted_lists(p)

    def run(v):
        return to_host(pbs.attn_fwd(p, to_dev(Q, dtype), to_dev(K, dtype), to_dev(vt_layout(v, block), dtype), None,
                                    i32_dev(kidx), cnt, cols))
    clean = run(V)
    bad = V.copy()
    bad[0, 0, at, 3], bad[0, 0, at, d - 1], bad[0, 0, n - 1, 5] = np.inf, np.nan, -np.inf
    got = run(bad)
    torch.cuda.synchronize()
    want = clean.copy()
    want[0, :, at:, 3], want[0, :, at:, d - 1], want[0, :, n - 1, 5] = np.inf, np.nan, -np.inf
    # (the d = 64 kernel sums such a query tile in another order, with probabilities that are not split: sums that differ
    # by less than 2^-17 of the weights times |v| < 4, then one bf16 rounding of either side)
    np.testing.assert_allclose(got, want, rtol=2.0 ** -7, atol=2.0 ** -15, equal_nan=True)


# key tiles of 16, chunks of at least 16, 32 and 64 keys, one to eight row tiles shared by four waves; 140001 keys: long ranges in
# both sweeps, the statistics running on into the average-query region of the workspace
@pytest.mark.parametrize("n", [1, 15, 63, 65, 1000, 140001])
@pytest.mark.parametrize("dtype,d,block", [("f32", 64, 64), ("f32", 128, 128), ("bf16", 64, 64), ("bf16", 64, 128)])
def test_fp64_key_scores(oracle, dtype, d, block, n):
    Hq, Hkv = (2, 1) if n > 100000 else (6, 3)
    Q, K, _ = _qkv(n + d, Hq, Hkv, n, d, dtype)
    p = pbs.problem(1, Hq, Hkv, n, d, block, block, dtype)
    got = pbs.key_scores(p, to_dev(Q, dtype), to_dev(K, dtype))
    # sums in fp64 on both sides, one rounding to float32
    np.testing.assert_allclose(got.cpu().numpy(), oracle.key_scores(Q, K, block), rtol=2.0 ** -23, atol=1e-37)


@pytest.mark.parametrize("m", [1, 16, 17, 33, 48, 128])
@pytest.mark.parametrize("dtype,d,block", [("f32", 64, 16), ("bf16", 64, 32), ("f32", 128, 16)])
def test_fp64_key_scores_from_listed_rows(oracle_variants, dtype, d, block, m):
    Q, K, _ = _qkv(m, 4, 2, 777, d, dtype)
    rows = wl.random_query_rows(m, 777, m)
    p = pbs.problem(1, 4, 2, 777, d, block, block, dtype)
    got = pbs.key_scores_proxy(p, pbs.PROXY_QUERY_ROWS, i32_dev(rows), to_dev(Q, dtype), to_dev(K, dtype))
    want = oracle_variants.key_scores_proxy(Q, K, rows)
    np.testing.assert_allclose(got.cpu().numpy(), want, rtol=2.0 ** -23, atol=1e-37)


def test_rows_from_queues_and_lists_of_every_length(oracle):
    # 4400 rows: workgroups take rows from queues and prepare the next one under the current one.  Lists too short for
    # that, empty ones, and ones that end around the 1024 entries that are staged at a time, with and without the own
    # segment that token order replaces at their end.
    block, d, T, Hq, Hkv, seg = 128, 128, 1100, 4, 2, 1024
    n, R = T * block - 77, seg // block
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    Q, K, V = (torch.randn((1, h, n, d), generator=g, device="cuda").to(torch.bfloat16) for h in (Hq, Hkv, Hkv))
    p = pbs.problem(1, Hq, Hkv, n, d, block, seg, "bf16", flags=pbs.FLAG_TOKEN_ORDER_COPY)
    kidx, Kp, Vt = pbs.segment_permute(p, None, K, V)
    rng = np.random.default_rng(12)
    lens = [0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 40, 1015, 1016, 1020, 1021, 1022, 1023, 1024, 1025, 1026, 1027, 1040]
    cnt = np.zeros((1, Hq, T), dtype=np.int32)
    cols = np.full((1, Hq, T, T), -1, dtype=np.int32)
    rows = []
    for h in range(Hq):
        for i in range(T):
            seg_lo, full = i // R * R, (i // R + 1) * seg <= n
            want = lens[(i * Hq + h) % len(lens)]
            own = list(range(seg_lo, seg_lo + R)) if full and i % 3 else [i]
            below = seg_lo if full else i
            take = min(max(0, want - len(own)), below)
            lst = ([] if want == 0 else sorted(rng.choice(below, take, replace=False).tolist()) + own)
            cnt[0, h, i] = len(lst)
            cols[0, h, i, :len(lst)] = lst
            if i >= T - 60 and (h + i) % 3 == 0 or i < 40 and h == 1:
                rows.append([0, h, i])
    rows = np.asarray(rows, dtype=np.int32)
    got, lse = pbs.attn_fwd(p, Q, Kp, Vt, None, kidx, i32_dev(cnt), i32_dev(cols), want_lse=True)
    torch.cuda.synchronize()
    host = [x.float().cpu().numpy() for x in (Q, K, V)]
    kh = np.tile(np.arange(n, dtype=np.int32), (1, Hkv, 1))
    want = oracle.attn_rows(*host, None, kh, cnt, cols, block, rows)
    got = to_host(got)
    for k, (_, h, i) in enumerate(rows):
        lo, hi = i * block, min(n, (i + 1) * block)
        if cnt[0, h, i] == 0:
            assert (got[0, h, lo:hi] == 0).all() and torch.isneginf(lse[0, h, lo:hi]).all()
        else:
            check_close(got[0, h, lo:hi], want[k][:hi - lo], "bf16", "row %d of head %d" % (i, h))


@pytest.mark.parametrize("token_copy", [False, True])
@pytest.mark.parametrize("Hq,Hkv,T,tail", [(2, 1, 1, 77), (4, 4, 2, 0), (2, 2, 9, 127), (4, 2, 41, 1)])
def test_rows_in_two_halves(oracle, Hq, Hkv, T, tail, token_copy):
    # calls with few rows give each half of a list two waves of its own: lists of 0, 1, 2, 3 .. entries, halves that differ
    # by a block, halves without a key some queries may see, and references that rise along the list by up to 25 nats
    # (no probability outgrows the first one's reference by 2^64) and fall by as much in every other head
    block, d, seg = 128, 128, 256
    n, R = T * block - tail, seg // block
    g = torch.Generator(device="cuda")
    g.manual_seed(31 + T)
    Q, K, V = (torch.randn((1, h, n, d), generator=g, device="cuda") for h in (Hq, Hkv, Hkv))
    u = torch.nn.functional.normalize(torch.randn(d, generator=g, device="cuda"), dim=0)
    rise = torch.linspace(0.0, 1.0, n, device="cuda")
    Q += 8.0 * u
    for h in range(Hkv):
        K[0, h] += 25.0 * d ** 0.5 / 8.0 * (rise if h % 2 == 0 else 1.0 - rise)[:, None] * u
    Q, K, V = (x.to(torch.bfloat16) for x in (Q, K, V))
    p = pbs.problem(1, Hq, Hkv, n, d, block, seg, "bf16", flags=pbs.FLAG_TOKEN_ORDER_COPY if token_copy else 0)
    scores = torch.softmax(torch.randn((1, Hkv, n), generator=g, device="cuda"), dim=-1)
    kidx, Kp, Vt = pbs.segment_permute(p, scores, K, V)
    rng = np.random.default_rng(T)
    cnt = np.zeros((1, Hq, T), dtype=np.int32)
    cols = np.full((1, Hq, T, T), -1, dtype=np.int32)
    for h in range(Hq):
        for i in range(T):
            seg_lo, full = i // R * R, (i // R + 1) * seg <= n
            own = list(range(seg_lo, seg_lo + R)) if full else [i]
            below = seg_lo if full else i
            lst = [] if (i + h) % 7 == 3 else sorted(rng.choice(below, min(below, (3 * i + h) % (T + 1)), replace=False).tolist()) + own
            if i % 5 == 4:
                lst = lst[::-1]
            cnt[0, h, i] = len(lst)
            cols[0, h, i, :len(lst)] = lst
    got, lse = pbs.attn_fwd(p, Q, Kp, Vt, None, kidx, i32_dev(cnt), i32_dev(cols), want_lse=True)
    torch.cuda.synchronize()
    host = [x.float().cpu().numpy() for x in (Q, K, V)]
    kg = kidx.cpu().numpy()
    want, want_lse = oracle.attn_fwd(host[0], oracle.gather_rows(host[1], kg), oracle.gather_rows(host[2], kg), None, kg, cnt,
                                     cols, block, want_lse=True)
    got, lse = to_host(got), lse.cpu().numpy()
    empty = np.repeat(cnt == 0, block, axis=-1)[..., :n]
    assert (got[empty] == 0).all() and np.isneginf(lse[empty]).all()
    check_close(got, np.where(empty[..., None], 0.0, want), "bf16", "rows in two halves")
    # fp32 logits of up to 40 and sums of a thousand terms: 2^-24 * 40 * log2(1000) is 2.4e-5; bf16 products are exact
    np.testing.assert_allclose(lse[~empty], want_lse[~empty], atol=1e-4)


def test_flagged_rows_from_queues_go_to_the_second_pass(oracle):
    # 4096 rows, the fewest that come from queues: their flags share the workspace with the queue heads.  Logits rise by
    # 60 nats along a sequence in the first head of each group only, so that it alone is flagged.
    block, d, T, Hq, Hkv = 128, 128, 512, 8, 4
    n = T * block
    rng = np.random.default_rng(31)
    Q = 0.05 * rng.standard_normal((1, Hq, n, d)).astype(np.float32)
    K = 0.05 * rng.standard_normal((1, Hkv, n, d)).astype(np.float32)
    Q[0, ::2, :, 0] += 16.0
    K[0, :, :, 0] += np.linspace(0.0, 60.0 * np.sqrt(d) / 16.0, n, dtype=np.float32)
    Q, K = wl.round_to_bf16(Q), wl.round_to_bf16(K)
    V = wl.round_to_bf16(rng.standard_normal((1, Hkv, n, d)).astype(np.float32))
    p = pbs.problem(1, Hq, Hkv, n, d, block, block, "bf16")
    Qd, Kd, Vd = (to_dev(x, "bf16") for x in (Q, K, V))
    kidx, Kp, Vt = pbs.segment_permute(p, None, Kd, Vd)
    cnt = np.tile(np.minimum(np.arange(T) + 1, 6).astype(np.int32), (1, Hq, 1))
    cols = np.zeros((1, Hq, T, T), dtype=np.int32)
    for i in range(T):
        cols[0, :, i, :cnt[0, 0, i]] = np.unique(np.linspace(0, i, 6).astype(np.int32)) if i > 5 else np.arange(i + 1)
    ws = pbs.alloc_workspace(p, pbs.STAGE_ATTN_FWD)
    ws.fill_(0x55)
    got, lse = pbs.attn_fwd(p, Qd, Kp, Vt, None, kidx, i32_dev(cnt), i32_dev(cols), want_lse=True, ws=ws)
    torch.cuda.synchronize()
    flags = ws[:Hq * T * 2].view(torch.int16).view(Hq, T).cpu().numpy() != 0
    assert flags[::2, T - 60:].all() and not flags[1::2].any()
    rows = np.asarray([[0, h, i] for h in range(Hq) for i in (0, 5, 6, 300, T - 2, T - 1)], dtype=np.int32)
    kh = np.tile(np.arange(n, dtype=np.int32), (1, Hkv, 1))
    want = oracle.attn_rows(Q, K, V, None, kh, cnt, cols, block, rows)
    got = to_host(got)
    for k, (_, h, i) in enumerate(rows):
        check_close(got[0, h, i * block:(i + 1) * block], want[k], "bf16", "row %d of head %d" % (i, h))


# four keys to a lane, 64 lanes to a wave: segments inside a lane row, a wave, two waves, sixteen; sizes
# that are no power of two; ties, both zeros, infinities
@pytest.mark.parametrize("block,segment", [(16, 16), (16, 48), (32, 256), (16, 272), (128, 512), (128, 1024), (64, 1088),
                                           (128, 2048), (128, 3968), (128, 4096)])
def test_segment_argsort_of_ragged_lengths_with_ties(oracle, block, segment):
    n = 3 * segment + segment // 2 + 3
    rng = np.random.default_rng(segment)
    s = rng.standard_normal((1, 3, n)).astype(np.float32)
    s[0, 1] = np.round(s[0, 1])                            # mostly ties, -0.0 among them
    s[0, 2, ::7], s[0, 2, ::11] = np.inf, -np.inf
    p = pbs.problem(1, 3, 3, n, 64, block, segment, "f32", flags=pbs.FLAG_TOKEN_ORDER_COPY)
    kidx, _, _ = pbs.segment_permute(p, torch.from_numpy(s).cuda(), None, None, indices_only=True)
    np.testing.assert_array_equal(kidx.cpu().numpy(), oracle.segment_argsort(s, segment))
    assert (pbs.token_copy(p, kidx, 1).cpu().numpy() == np.arange(n)).all()


# up to 32768 keys in segments of 256 and more are placed by counting: both sides of that line, a buffer shared by scores
# and indices (never by counting)
@pytest.mark.parametrize("heads,segment,segments", [(8, 1024, 4), (8, 1024, 5), (1, 256, 128), (1, 256, 129), (2, 240, 3),
                                                    (1, 4096, 8), (3, 1040, 2), (1, 4096, 0)])
def test_segment_argsort_by_counting(oracle, heads, segment, segments):
    n = max(segments * segment + 37, 300)
    rng = np.random.default_rng(heads * segment + segments)
    s = np.round(rng.standard_normal((1, heads, n)) * 8).astype(np.float32) / 8
    s[0, 0, ::5] = -0.0
    p = pbs.problem(1, heads, heads, n, 64, 16, segment, "f32", flags=pbs.FLAG_TOKEN_ORDER_COPY)
    want = oracle.segment_argsort(s, segment)
    kidx, _, _ = pbs.segment_permute(p, torch.from_numpy(s).cuda(), None, None, indices_only=True)
    np.testing.assert_array_equal(kidx.cpu().numpy(), want)
    assert (pbs.token_copy(p, kidx, 1).cpu().numpy() == np.arange(n)).all()
    p = pbs.problem(1, heads, heads, n, 64, 16, segment, "f32")
    both = torch.from_numpy(s).cuda()
    kidx, _, _ = pbs.segment_permute(p, both, None, None, kidx=both.view(torch.int32), indices_only=True)
    np.testing.assert_array_equal(kidx.cpu().numpy(), want)


# A value that is not finite in a block that every later query sees in full, the later blocks' own values finite: what
# p * v gives must come out, also where p enters the product as several terms of either sign.  The long case has more than 4096
# query tiles: there a wave has its list to itself.
@pytest.mark.parametrize("dtype,d,block,Hq,Hkv,n,later", [("bf16", 64, 64, 4, 2, 500, 0), ("bf16", 64, 128, 2, 1, 700, 0),
                                                          ("bf16", 64, 64, 64, 2, 16410, 0), ("bf16", 64, 32, 2, 1, 300, 0),
                                                          ("f32", 64, 64, 2, 1, 300, 0), ("f32", 128, 32, 2, 1, 300, 3),
                                                          ("f32", 128, 128, 2, 1, 700, 19)])
def test_values_of_an_earlier_segment_that_are_not_finite(dtype, d, block, Hq, Hkv, n, later):
    Q, K, V = (to_dev(x, dtype) for x in _qkv(9, Hq, Hkv, n, d, dtype))
    T, at = -(-n // block), block // 2 + later
    p = pbs.problem(1, Hq, Hkv, n, d, block, block, dtype)
    i = torch.arange(T, dtype=torch.int32, device="cuda")
    cnt = torch.clamp(i + 1, max=2).repeat(1, Hq, 1).contiguous()
    cols = torch.zeros((T, T), dtype=torch.int32, device="cuda")
    cols[1:, 1] = i[1:]                                    # every query block sees block 0 and itself
    cols = cols.repeat(1, Hq, 1, 1).contiguous()

    def run(v):
        kidx, kp, vt = pbs.segment_permute(p, None, K, v)
        return pbs.attn_fwd(p, Q, kp, vt, None, kidx, cnt, cols, want_lse=True)
    want, want_lse = run(V)
    bad = V.clone()
    bad[0, :, at, 3], bad[0, :, at, 5], bad[0, :, at, d - 1] = np.inf, -np.inf, np.nan
    bad[0, :, at, 7], bad[0, :, at + 1, 7] = np.inf, -np.inf
    got, lse = run(bad)
    torch.cuda.synchronize()
    want = want.clone()
    want[0, :, at:, 3], want[0, :, at:, 5], want[0, :, at:, d - 1] = np.inf, -np.inf, np.nan
    want[0, :, at, 7], want[0, :, at + 1:, 7] = np.inf, np.nan
    # two bf16 roundings of sums of which one may be formed relative to another reference: as above
    torch.testing.assert_close(got.float(), want.float(), rtol=2.0 ** -7, atol=2.0 ** -15, equal_nan=True)
    assert torch.equal(lse, want_lse)


# a key that is not a number makes every score of its head one, wherever it stands: alone in its chunk, in its key share,
# in its lane's part of a tile
@pytest.mark.parametrize("dtype,d,block,n", [("f32", 64, 16, 17), ("f32", 128, 128, 65), ("bf16", 64, 32, 33),
                                             ("bf16", 64, 128, 257), ("f32", 64, 64, 1)])
def test_fp64_key_scores_of_a_key_that_is_not_a_number(oracle, dtype, d, block, n):
    Q, K, _ = _qkv(n, 4, 2, n, d, dtype)
    K[0, 1, n - 1] = np.nan
    p = pbs.problem(1, 4, 2, n, d, block, block, dtype)
    got = pbs.key_scores(p, to_dev(Q, dtype), to_dev(K, dtype)).cpu().numpy()
    assert np.isnan(got[0, 1]).all()
    np.testing.assert_allclose(got[0, 0], oracle.key_scores(Q, K, block)[0, 0], rtol=2.0 ** -23, atol=1e-37)


def test_calls_on_two_streams_may_share_a_workspace():
    # 4096 rows each, so that both calls hand their rows out from queues at the same time.  On ordinary inputs the flags that
    # either call leaves in the workspace are all zero, so nothing else in it can disturb the other.
    block, d, T, Hq, Hkv = 128, 128, 512, 8, 4
    n = T * block
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    K, V = (torch.randn((1, Hkv, n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    Q = [torch.randn((1, Hq, n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2)]
    p = pbs.problem(1, Hq, Hkv, n, d, block, block, "bf16")
    kidx, Kp, Vt = pbs.segment_permute(p, None, K, V)
    i = torch.arange(T, dtype=torch.int32, device="cuda")
    cnt = torch.clamp(i + 1, max=8).repeat(1, Hq, 1).contiguous()
    cols = torch.zeros((T, T), dtype=torch.int32, device="cuda")
    for k in range(8):                                     # the last eight blocks, ascending
        cols[:, k] = torch.clamp(i - 7, min=0) + k
    cols = cols.repeat(1, Hq, 1, 1).contiguous()
    want = [pbs.attn_fwd(p, q, Kp, Vt, None, kidx, cnt, cols) for q in Q]
    ws, streams = pbs.alloc_workspace(p, pbs.STAGE_ATTN_FWD), [torch.cuda.Stream() for _ in range(2)]
    got = [torch.empty_like(q) for q in Q]
    for _ in range(4):
        for o in got:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        for _ in range(3):
            for q, o, s in zip(Q, got, streams):
                with torch.cuda.stream(s):
                    pbs.attn_fwd(p, q, Kp, Vt, None, kidx, cnt, cols, o, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def _rows_that_outgrow_their_reference(seed, Hq, Hkv, T, last):
    """Inputs, lists of up to 64 blocks each and a workspace: keys from block T - last on stand 80 nats above the others for
    the query heads that the caller gives a first feature of 16."""
    block = d = 128
    n = T * block
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    Q = 0.05 * torch.randn((1, Hq, n, d), generator=g, device="cuda")
    K = 0.05 * torch.randn((1, Hkv, n, d), generator=g, device="cuda")
    K[0, :, (T - last) * block:, 0] += 80.0 * d ** 0.5 / 16.0
    V = torch.randn((1, Hkv, n, d), generator=g, device="cuda")
    p = pbs.problem(1, Hq, Hkv, n, d, block, block, "bf16")
    kidx, Kp, Vt = pbs.segment_permute(p, None, K.to(torch.bfloat16), V.to(torch.bfloat16))
    i = torch.arange(T, device="cuda")
    cnt = torch.clamp(i + 1, max=64)
    k = torch.arange(T, device="cuda")
    cols = torch.where(k[None] < cnt[:, None], (k[None] * i[:, None]) // torch.clamp(cnt[:, None] - 1, min=1), 0).to(torch.int32)
    return p, Q, Kp, Vt, kidx, cnt.to(torch.int32).repeat(1, Hq, 1).contiguous(), cols.repeat(1, Hq, 1, 1).contiguous()


# 4400 rows (more than the 4096 ids that are looked at together), 840 and 21: all of the late rows flagged, those of one
# head, of some heads, none
@pytest.mark.parametrize("Hq,Hkv,T,last", [(44, 4, 100, 40), (44, 4, 100, 1), (28, 4, 30, 12), (3, 3, 7, 3)])
@pytest.mark.parametrize("heads", ["all", "one", "some", "none"])
def test_second_pass_takes_exactly_the_flagged_rows(Hq, Hkv, T, last, heads):
    p, Q, Kp, Vt, kidx, cnt, cols = _rows_that_outgrow_their_reference(Hq + T, Hq, Hkv, T, last)
    on = {"all": list(range(Hq)), "one": [Hq // 2], "some": [h for h in range(Hq) if h % 5 in (1, 2)], "none": []}[heads]
    Q[0, on, :, 0] += 16.0
    Q = Q.to(torch.bfloat16)
    got, lse = pbs.attn_fwd(p, Q, Kp, Vt, None, kidx, cnt, cols, want_lse=True)
    plain = pbs.problem(1, Hq, Hkv, p.n, 128, 128, 128, "bf16", flags=pbs.FLAG_RUNNING_MAX_ONLY)
    want, want_lse = pbs.attn_fwd(plain, Q, Kp, Vt, None, kidx, cnt, cols, want_lse=True)
    # flagged rows went through the kernel that the plain call uses for all of them: the same bits
    late = torch.zeros((Hq, T), dtype=torch.bool, device="cuda")
    late[on, T - last:] = True
    rows = late.repeat_interleave(128, 1)[None]
    assert torch.equal(got[rows], want[rows]) and torch.equal(lse[rows], want_lse[rows])
    err = (got.float() - want.float()).abs()
    assert err.max() < 4e-2 and err.mean() < 2e-3          # twice the bound against the oracle: each side has its own


def test_second_pass_of_some_rows_takes_its_share_of_the_time():
    # 8192 rows of equally long lists (but for the first 64 blocks), the last quarter of each head flagged: as long as a quarter
    # of the same kernel over all rows, give or take the end of the launch.  Dealt out by row number it took twice that.
    p, Q, Kp, Vt, kidx, cnt, cols = _rows_that_outgrow_their_reference(3, 32, 8, 256, 64)
    flat, steep = Q.to(torch.bfloat16), Q.clone()
    steep[0, :, :, 0] += 16.0
    steep = steep.to(torch.bfloat16)
    plain = pbs.problem(1, 32, 8, p.n, 128, 128, 128, "bf16", flags=pbs.FLAG_RUNNING_MAX_ONLY)
    ws, out = pbs.alloc_workspace(p, pbs.STAGE_ATTN_FWD), torch.empty_like(flat)

    def best(problem, q):
        times = []
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            pbs.attn_fwd(problem, q, Kp, Vt, None, kidx, cnt, cols, out, ws=ws)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times[2:])
    first, both, alone = best(p, flat), best(p, steep), best(plain, steep)
    assert both - first < 1.5 * alone * 2048 / 8192, (first, both, alone)


@pytest.mark.parametrize("d,block,flags", [(128, 128, 0), (128, 128, pbs.FLAG_TOKEN_ORDER_COPY), (64, 128, 0)])
def test_v_prime_may_take_the_place_of_k(d, block, flags):
    # K is not needed once K' and the block means are there, and 16 heads x 8192 rows are far more than the chip moves at a time
    Hkv, n, seg = 16, 8192, 1024
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    K, V = (torch.randn((1, Hkv, n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    scores = torch.rand((1, Hkv, n), generator=g, device="cuda")
    p = pbs.problem(1, Hkv, Hkv, n, d, block, seg, "bf16", flags=flags)
    ws = pbs.alloc_workspace(p, pbs.STAGE_BLOCK_MASK).zero_()
    want = pbs.segment_permute(p, scores, K, V, ws=ws)
    Vt, ws2 = pbs.alloc_vt(p), torch.zeros_like(ws)
    place = torch.as_strided(Vt, K.shape, K.stride(), Vt.storage_offset())       # K lies where V' goes
    place.copy_(K)
    got = pbs.segment_permute(p, scores, place, V, Vt=Vt, ws=ws2)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    assert torch.equal(ws, ws2)
    if flags:
        assert torch.equal(pbs.token_copy(p, got[1], d), K)
        assert torch.equal(pbs.token_copy(p, got[2], d), pbs.token_copy(p, want[2], d))


@pytest.mark.parametrize("dtype,d,block", [("bf16", 64, 64), ("bf16", 64, 128), ("bf16", 64, 32), ("f32", 64, 64)])
def test_probabilities_keep_their_32_bits(dtype, d, block):
    # Three keys whose weighted values all but cancel: V[1] undoes V[0] up to its rounding, V[2] what is left up to its own, so the
    # sum is about 2^-16 of its terms and shows a probability's error of 2^-18 (two bf16 terms) plainly.  Bound: 2^-20 of the
    # terms for the weights (scores within 2, so that fp32 sums and exp2 are good to about 2^-22) and the output's rounding.
    H, n = 64, 3
    Q, K, V = _qkv(77, H, H, n, d, "bf16")
    Q = wl.round_to_bf16(0.25 * Q)
    w = np.exp((K.astype(np.float64) @ Q[..., 2, :, None].astype(np.float64))[..., 0] / np.sqrt(d))   # of the last query
    w /= w.sum(-1, keepdims=True)

    def cancel(k):
        V[:, :, k] = 0.0
        V[:, :, k] = wl.round_to_bf16((-(w[..., None] * V).sum(2) / w[..., k, None]).astype(np.float32))
    V[:, :, 2] = 0.0
    cancel(1)
    cancel(2)
    want, size = (w[..., None] * V).sum(2), (w[..., None] * np.abs(V)).sum(2)
    assert np.median(np.abs(want) / size) < 2.0 ** -16
    p = pbs.problem(1, H, H, n, d, block, block, dtype)
    cnt, cols = pbs.admitted_lists(p)
    kidx, Kp, Vt = pbs.segment_permute(p, None, to_dev(K, dtype), to_dev(V, dtype))
    got = to_host(pbs.attn_fwd(p, to_dev(Q, dtype), Kp, Vt, None, kidx, cnt, cols))[0, :, 2]
    err = np.abs(got - want[0])
    assert (err <= 2.0 ** -20 * size[0] + 2.0 ** -8 * np.abs(want[0])).all(), (err / size[0]).max() * 2.0 ** 20


def test_selection_time_follows_the_number_of_columns():
    # 4096 query blocks against 1024: sixteen times the probabilities (and four times the pooling).  With the long rows in LDS
    # it took 34 times as long.
    def best(n):
        Q, K = (torch.randn((1, h, n, 128), device="cuda").to(torch.bfloat16) for h in (8, 4))
        p = pbs.problem(1, 8, 4, n, 128, 32, 1024, "bf16")
        out = pbs.block_mask(p, Q, K)
        kbar = pbs.alloc_workspace(p, pbs.STAGE_BLOCK_MASK)
        times = []
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            pbs.block_mask(p, Q, K, *out, ws=kbar)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times)
    short, long = best(32768), best(131072)
    assert long < 22.0 * short, (short, long)


# rows of 2048 and 4096 columns and one more or less, with query heads in groups of one, two, three and five
@pytest.mark.parametrize("n,block,Hq,Hkv,dtype", [(32767, 16, 1, 1, "f32"), (32785, 16, 4, 2, "bf16"), (65519, 16, 3, 1, "bf16"),
                                                  (65536, 16, 5, 1, "f32")])
def test_selection_of_long_rows(oracle, n, block, Hq, Hkv, dtype):
    Q, K, _ = _qkv(n, Hq, Hkv, n, 64, dtype)
    p = pbs.problem(1, Hq, Hkv, n, 64, block, 64 * block, dtype, tau=0.9, flags=pbs.FLAG_FORCE_FIRST_BLOCK)
    mask, cnt, cols = pbs.block_mask(p, to_dev(Q, dtype), to_dev(K, dtype))
    want, want_cnt, want_cols = oracle.block_mask(Q, K, block, 64 * block, float(np.float32(0.9)), flags=pbs.FLAG_FORCE_FIRST_BLOCK)
    np.testing.assert_array_equal(mask_from_bits(mask, pbs.T_of(p)), want)
    np.testing.assert_array_equal(cnt.cpu().numpy(), want_cnt)
    listed = np.arange(pbs.T_of(p)) < want_cnt[..., None]
    np.testing.assert_array_equal(cols.cpu().numpy()[listed], want_cols[listed])


# segments of at most 128 keys lie side by side in a wave: numbers that fill it and that do not, one segment, none
@pytest.mark.parametrize("block,segment", [(16, 16), (32, 32), (16, 48), (64, 64), (16, 80), (32, 128), (16, 144)])
@pytest.mark.parametrize("segments", [0, 1, 2, 15, 16, 17, 53])
def test_segment_argsort_of_short_segments(oracle, block, segment, segments):
    n = segments * segment + segment - 5
    s = np.round(np.random.default_rng(n).standard_normal((1, 3, n)) * 8).astype(np.float32) / 8
    s[0, 1, ::3], s[0, 2, ::5], s[0, 2, 1::5] = -0.0, np.inf, -np.inf
    p = pbs.problem(1, 3, 3, n, 64, block, segment, "f32", flags=pbs.FLAG_TOKEN_ORDER_COPY)
    want = oracle.segment_argsort(s, segment)
    kidx, _, _ = pbs.segment_permute(p, torch.from_numpy(s).cuda(), None, None, indices_only=True)
    np.testing.assert_array_equal(kidx.cpu().numpy(), want)
    assert (pbs.token_copy(p, kidx, 1).cpu().numpy() == np.arange(n)).all()
    p = pbs.problem(1, 3, 3, n, 64, block, segment, "f32")
    both = torch.from_numpy(s).cuda()
    kidx, _, _ = pbs.segment_permute(p, both, None, None, kidx=both.view(torch.int32), indices_only=True)
    np.testing.assert_array_equal(kidx.cpu().numpy(), want)


def test_short_segments_sort_as_fast_as_long_ones():
    # the same 524288 keys in segments of 16 and of 256: with a wave to a segment of 16 it took more than five times as long
    def best(block, segment):
        p = pbs.problem(1, 8, 8, 65536, 64, block, segment, "f32")
        s, kidx = torch.rand((1, 8, 65536), device="cuda"), pbs.alloc_kidx(p)
        times = []
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                pbs.segment_permute(p, s, None, None, kidx=kidx, indices_only=True)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times)
    short, long = best(16, 16), best(64, 256)
    assert short < 2.5 * long, (short, long)


# one and two query heads to a kv head: four query blocks to a workgroup in rows of more than 64 columns, or from 256
# workgroups on, two otherwise; the last workgroup with one to four of them
@pytest.mark.parametrize("T", [62, 64, 65, 124, 125, 126, 127])
@pytest.mark.parametrize("Hq,Hkv,d,dtype", [(8, 8, 64, "bf16"), (16, 8, 128, "bf16"), (8, 8, 128, "f32"), (16, 8, 64, "f32")])
def test_selection_with_few_query_heads_to_a_kv_head(oracle, Hq, Hkv, d, dtype, T):
    n, block, seg = T * 16 - 5, 16, 128
    Q, K, _ = _qkv(T + d, Hq, Hkv, n, d, dtype)
    p = pbs.problem(1, Hq, Hkv, n, d, block, seg, dtype, tau=0.9)
    mask, cnt, cols = pbs.block_mask(p, to_dev(Q, dtype), to_dev(K, dtype))
    want, want_cnt, want_cols = oracle.block_mask(Q, K, block, seg, float(np.float32(0.9)))
    np.testing.assert_array_equal(mask_from_bits(mask, T), want)
    np.testing.assert_array_equal(cnt.cpu().numpy(), want_cnt)
    listed = np.arange(T) < want_cnt[..., None]
    np.testing.assert_array_equal(cols.cpu().numpy()[listed], want_cols[listed])


def test_selection_time_with_a_kv_head_to_every_query_head():
    # the same rows, four times the pooled keys: 1.3 times the time of a shared kv head (1.8 times with two rows to a workgroup,
    # which leave half of a matrix instruction empty)
    def best(hkv):
        Q, K = (torch.randn((1, h, 65536, 128), device="cuda").to(torch.bfloat16) for h in (32, hkv))
        p = pbs.problem(1, 32, hkv, 65536, 128, 128, 1024, "bf16", flags=pbs.FLAG_KBAR_IN_WS)
        ws = pbs.alloc_workspace(p, pbs.STAGE_BLOCK_MASK)
        ws.view(torch.float64).normal_()                   # block means of some keys
        out, times = pbs.block_mask(p, Q, K, ws=ws), []
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(5):
                pbs.block_mask(p, Q, K, *out, ws=ws)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times)
    own, shared = best(32), best(8)
    assert own < 1.55 * shared, (own, shared)


# long inputs, two waves of 64 rows to a workgroup: the last tile of one key, shares of a head that end inside a range, one
# head, heads of two sequences; whole shares of one and of three ranges, which the workgroups start at different tiles.  Qhat's two bf16 terms leave 2^-18 of each product, 128 fp32 additions 2^-17 of their sum,
# and sum |q k| / sqrt(d) < 8 for these inputs: within 1e-4 of a score.
@pytest.mark.parametrize("batch,h_kv,n", [(1, 32, 10273), (2, 33, 5001), (1, 1, 327701), (1, 8, 41000),
                                          (1, 8, 65536), (1, 3, 524288)])
def test_key_scores_of_long_inputs(batch, h_kv, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    Q = torch.randn((batch, h_kv, n, 128), generator=g, device="cuda").bfloat16()
    K = torch.randn((batch, h_kv, n, 128), generator=g, device="cuda").bfloat16()
    got = pbs.key_scores(pbs.problem(batch, h_kv, h_kv, n, 128, 128, 1024, "bf16"), Q, K)
    for b in range(batch):
        for h in range(h_kv):
            want = torch.softmax(Q[b, h, -128:].double() @ K[b, h].double().T / 128 ** 0.5, -1).mean(0)
            torch.testing.assert_close(got[b, h].double(), want, rtol=1e-4, atol=0)


# five heads take the long form, four of them the short one, with ranges of 512 keys both; eight heads and seven of them both
# the long form, with shares of three and two ranges: a head's scores do not depend on the others
# short inputs: ranges of 64, 128 and 256 keys, of which a workgroup takes one, two or four
@pytest.mark.parametrize("h_kv,fewer,n", [(5, 4, 65536), (5, 4, 65555), (8, 7, 140000), (8, 7, 147456), (40, 1, 40), (17, 16, 1100),
                                          (100, 3, 2048), (17, 8, 2050), (40, 7, 4100), (16, 5, 8192), (17, 4, 8193), (9, 2, 20001)])
def test_key_scores_of_a_head_do_not_depend_on_the_others(h_kv, fewer, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    Q = torch.randn((1, h_kv, n, 128), generator=g, device="cuda", dtype=torch.bfloat16)
    K = torch.randn((1, h_kv, n, 128), generator=g, device="cuda", dtype=torch.bfloat16)
    got = [pbs.key_scores(pbs.problem(1, h, h, n, 128, 128, 1024, "bf16"), Q[:, :h].contiguous(), K[:, :h].contiguous())
           for h in (h_kv, fewer)]
    assert torch.equal(got[0][:, :fewer], got[1])


# the fp64 sweeps: chunks of 16, 32 and 64 keys, of which a workgroup takes one to four.  Another order of sums shows in few results
# after their rounding to float32, so the rows' maxima and sums are compared too, which a call leaves in its workspace behind Qhat
@pytest.mark.parametrize("dtype,d,block,heads,fewer,n", [("f32", 64, 64, 40, 2, 1024), ("f32", 64, 64, 33, 2, 4096), ("bf16", 64, 128, 12, 1, 2048),
                                                         ("f32", 128, 16, 70, 3, 700), ("f32", 64, 32, 24, 4, 4097)])
def test_fp64_key_scores_of_a_head_do_not_depend_on_the_others(dtype, d, block, heads, fewer, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K = (torch.randn((1, heads, n, d), generator=g, device="cuda").to(kind) for _ in range(2))

    def run(lo, hi):
        p = pbs.problem(1, hi - lo, hi - lo, n, d, block, 128, dtype)
        ws = pbs.alloc_workspace(p, pbs.STAGE_KEY_SCORES)
        scores = pbs.key_scores(p, Q[:, lo:hi].contiguous(), K[:, lo:hi].contiguous(), ws=ws)
        stats = ws[(hi - lo) * 128 * d * 8:].view(torch.int64)[:(hi - lo) * block * 2].clone()
        return scores, stats.view(hi - lo, block, 2)
    scores, stats = run(0, heads)
    for lo in range(0, heads - fewer + 1, fewer):
        one, own = run(lo, lo + fewer)
        assert torch.equal(scores[:, lo:lo + fewer], one) and torch.equal(stats[lo:lo + fewer], own)


def test_block_64_attention_time_with_five_kv_heads():
    # sparse lists share tiles in an XCD's L2, which rows of all five heads on every XCD would crowd (5 / 5 heads x 40000, an
    # eighth of the blocks: 386 us against 498; a head's time 1.11 .. 1.18 and 1.41 .. 1.44 of that with four heads, two XCDs
    # to each)
    n, block, rho = 40000, 64, 0.12
    T = -(-n // block)

    def best(heads):
        g = torch.Generator(device="cuda")
        g.manual_seed(heads)
        Q, K, V = (torch.randn((1, heads, n, 128), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
        on = torch.tril(torch.rand((1, heads, T, T), generator=g, device="cuda") < rho, -1) | torch.eye(T, dtype=torch.bool, device="cuda")
        cnt = on.sum(-1, dtype=torch.int32)
        cols = torch.argsort(on.to(torch.uint8), dim=-1, descending=True, stable=True).to(torch.int32)
        p = pbs.problem(1, heads, heads, n, 128, block, 1024, "bf16")
        kidx, kp, vt = pbs.segment_permute(p, None, K, V)
        O, times = torch.empty_like(Q), []
        for _ in range(9):
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            pbs.attn_fwd(p, Q, kp, vt, None, kidx, cnt, cols, O)
            stop.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(stop))
        return min(times) / heads
    four, five = best(4), best(5)
    assert five < 1.3 * four, (four, five)


# K', V' and the block means of K' out of one launch (float32 storage; bf16 blocks of fewer than 1024 pieces of 16 bytes), against
# the launches that a call without a workspace and pbs_block_mask make: the same bytes.  One key, ragged blocks, whole ones.
@pytest.mark.parametrize("copy", [False, True])
@pytest.mark.parametrize("dtype,d,block", [("f32", 64, 16), ("f32", 64, 64), ("f32", 128, 128), ("bf16", 64, 16),
                                           ("bf16", 64, 64), ("bf16", 128, 32)])
def test_gather_with_means_in_one_launch(dtype, d, block, copy):
    for n in (1, block + 1, 5 * block - 3, 6 * block):
        flags = pbs.FLAG_TOKEN_ORDER_COPY if copy else 0
        p = pbs.problem(2, 3, 3, n, d, block, 2 * block, dtype, flags=flags)
        rng = np.random.default_rng(n)
        K, V = (to_dev(rng.standard_normal((2, 3, n, d)) * 2.0 ** rng.integers(-12, 13, (2, 3, n, 1)), dtype) for _ in range(2))
        scores = torch.from_numpy(rng.random((2, 3, n)).astype(np.float32)).cuda()
        ws = pbs.alloc_workspace(p, pbs.STAGE_BLOCK_MASK)
        kidx, Kp, Vt = pbs.segment_permute(p, scores, K, V, ws=ws)
        kidx0, Kp0, Vt0 = pbs.segment_permute(p, scores, K, V)
        assert torch.equal(kidx, kidx0) and torch.equal(Kp, Kp0) and torch.equal(Vt, Vt0)
        if copy:
            for x, x0, e in ((kidx, kidx0, 1), (Kp, Kp0, d), (Vt, Vt0, d)):
                assert torch.equal(pbs.token_copy(p, x, e), pbs.token_copy(p, x0, e))
        ws0 = pbs.alloc_workspace(p, pbs.STAGE_BLOCK_MASK)
        pbs.block_mask(p, K, Kp0, ws=ws0)
        T = pbs.T_of(p)
        stride = -(-T // 4) * 4
        means, means0 = (w[:6 * d * stride * 8].view(torch.float64).view(6, d, stride)[..., :T] for w in (ws, ws0))
        assert torch.equal(means, means0)
        if n % block == 0 and not copy:                    # V' in the place of K
            pbs.segment_permute(p, scores, K, V, kidx, Kp, K.view(Vt.shape), ws=ws)
            assert torch.equal(Kp, Kp0) and torch.equal(K.view(Vt.shape), Vt0)


# Qhat formed by the sweeps themselves (one or two query heads) and by a launch of its own, against the oracle: fp64 sums, a float
# result (2^-24), exponentials good to an ulp of fp64
@pytest.mark.parametrize("r", [1, 2, 3, 8])
@pytest.mark.parametrize("dtype,d,block,n", [("f32", 64, 64, 700), ("f32", 128, 128, 130), ("bf16", 64, 16, 9), ("f32", 64, 32, 1)])
def test_fp64_key_scores_of_query_groups(oracle, dtype, d, block, n, r):
    Q, K, _ = _qkv(r + n, 2 * r, 2, n, d, dtype)
    p = pbs.problem(1, 2 * r, 2, n, d, block, 2 * block, dtype)
    got = pbs.key_scores(p, to_dev(Q, dtype), to_dev(K, dtype))
    want = oracle.key_scores(Q, K, block)
    np.testing.assert_allclose(got.cpu().numpy(), want, rtol=2.0 ** -23, atol=1e-37)       # as in test_fp64_key_scores


# Ranges of 64, 128 and 256 keys, whole and ragged ones, up to 16 kv heads and beyond: 16 bits of Qhat in two terms, sums in fp32
@pytest.mark.parametrize("Hq,Hkv,n", [(2, 2, 1), (2, 1, 63), (4, 2, 129), (8, 8, 2050), (4, 2, 8193), (16, 16, 1100), (17, 17, 1100)])
def test_key_scores_in_short_ranges(oracle, Hq, Hkv, n):
    Q, K, _ = _qkv(n, Hq, Hkv, n, 128, "bf16")
    p = pbs.problem(1, Hq, Hkv, n, 128, 128, 1024, "bf16")
    got = pbs.key_scores(p, to_dev(Q, "bf16"), to_dev(K, "bf16"))
    np.testing.assert_allclose(got.cpu().numpy(), oracle.key_scores(Q, K, 128), rtol=1e-4, atol=0)


# Selection with a compute unit to every workgroup (whole query blocks loaded at a time) and with more workgroups than that, ragged
# last blocks, 3 and 4 query heads in a chunk; four query blocks to a workgroup with one query head to a kv head (more than 64
# blocks) and with two (256 workgroups): the masks and lists of the oracle, bit for bit
@pytest.mark.parametrize("Hq,Hkv,n,segment", [(4, 4, 5, 256), (3, 1, 130, 256), (7, 1, 2000, 512), (2, 1, 8200, 1024),
                                               (8, 2, 8191, 1024), (8, 2, 33000, 1024), (2, 2, 8200, 1024), (1, 1, 16389, 1024),
                                               (16, 8, 16300, 1024), (16, 8, 16400, 1024)])
def test_selection_with_few_workgroups(oracle, Hq, Hkv, n, segment):
    Q, K, _ = _qkv(n, Hq, Hkv, n, 128, "bf16")
    p = pbs.problem(1, Hq, Hkv, n, 128, 128, segment, "bf16", tau=0.9)
    bits, cnt, cols = pbs.block_mask(p, to_dev(Q, "bf16"), to_dev(K, "bf16"))
    want, want_cnt, want_cols = oracle.block_mask(Q, K, 128, segment, float(np.float32(0.9)))
    mask = mask_from_bits(bits, pbs.T_of(p))
    assert np.array_equal(mask, want) and np.array_equal(cnt.cpu().numpy(), want.sum(-1))
    listed = np.arange(pbs.T_of(p)) < want_cnt[..., None]
    assert np.array_equal(cols.cpu().numpy()[listed], want_cols[listed])


# d = 64: a row of probabilities that outgrows its reference in a sub-tile under the token-level mask, whose queries have met keys
# before: its scores are formed again from memory and masked again.  In either sub-tile of a pair and for either query tile a
# visible key stands 30 nats above all others, and a hidden one 45.  Four waves to a list, and one (4096 query tiles).
@pytest.mark.parametrize("heads", [3, 512])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("part", [0, 1])
@pytest.mark.parametrize("tile", [0, 1])
def test_d64_probabilities_that_outgrow_their_reference_under_the_mask(tile, part, block, heads):
    n, d, seg = 8 * block if block == 64 else 6 * block, 64, 2 * block
    g = torch.Generator(device="cuda")
    g.manual_seed(block + 2 * part + tile)
    Q, K, V = (torch.randn((1, heads, n, d), generator=g, device="cuda") for _ in range(3))
    Q[..., 0] = 0.0
    K[..., 0] = 0.0
    kidx = torch.arange(n, dtype=torch.int32, device="cuda")
    first = n - seg                                        # the last segment: keys of its own slots are masked
    seen, hidden = first + block + 32 * part + 5, first + block + 32 * part + 9      # slots, both in one sub-tile
    for slot, pos in ((seen, first), (hidden, n - 1)):     # exchanged: the segment's first key and its last one
        other = int((kidx == pos).nonzero())
        kidx[other], kidx[slot] = kidx[slot].clone(), pos
    queries = first + block + 32 * tile                    # of the segment's second block
    Q[0, :, queries:queries + 32, 0] = 8.0
    K[0, :, seen, 0], K[0, :, hidden, 0] = 30.0, 45.0      # (K as permuted: row = slot)
    Q, K, V = (x.to(torch.bfloat16) for x in (Q, K, V))
    p = pbs.problem(1, heads, heads, n, d, block, seg, "bf16")
    cnt, cols = pbs.admitted_lists(p)
    _, _, vt = pbs.segment_permute(p, None, K, V)
    got, lse = pbs.attn_fwd(p, Q, K, vt, None, kidx.repeat(1, heads, 1).contiguous(), cnt, cols, want_lse=True)
    see = kidx[None].long() <= torch.arange(n, device="cuda")[:, None]
    for h in range(0, heads, 64):
        at = slice(h, min(heads, h + 64))
        s = (Q[0, at].double() @ K[0, at].double().transpose(1, 2).contiguous() / 8.0).masked_fill(~see, -np.inf)
        torch.testing.assert_close(lse[0, at].double(), torch.logsumexp(s, -1), rtol=0, atol=1e-4)
        err = (got[0, at].double() - torch.softmax(s, -1) @ V[0, at].double()).abs()
        assert err.max() <= 2e-2 and err.mean() <= 2e-3
    top = see[queries:queries + 32, seen].all() and not see[queries:queries + 31, hidden].any()
    assert bool(top)
