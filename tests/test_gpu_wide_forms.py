"""The three forms of the block-128 attention kernel on the same kinds of lists: up to 256 rows (query blocks of all heads) a
row has two pairs of waves, from 4096 rows on workgroups take rows from queues, in between each row has a workgroup."""
import numpy as np
import pytest
import torch

from gpu_helpers import check_close, i32_dev, to_host
from paper_2510_21270_amd import binding as pbs
from paper_2510_21270_amd import workloads as wl

pytestmark = pytest.mark.gpu

BLOCK, D, R = 128, 128, 4
# batch, query heads, kv heads, blocks, keys missing in the last block
FORMS = {"two_halves": (1, 4, 2, 12, 9), "workgroup_per_row": (2, 6, 3, 50, 77), "rows_from_queues": (1, 32, 8, 130, 1)}


def _rows(form):
    batch, Hq, _, T, _ = FORMS[form]
    return batch * Hq * T


def test_the_forms_are_told_apart_by_their_rows():
    assert _rows("two_halves") <= 256 < _rows("workgroup_per_row") < 4096 <= _rows("rows_from_queues")


def _qkv(seed, batch, Hq, Hkv, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [torch.randn((batch, h, n, D), generator=g, device="cuda").to(torch.bfloat16) for h in (Hq, Hkv, Hkv)]


def _host(x):
    return x.float().cpu().numpy()


# keys in random order, own segments from a token-order copy where a list ends with one; keys reversed in every segment, so
# that early queries see nothing in the blocks they visit first; queries permuted too
@pytest.mark.parametrize("order,sigma,token_copy", [("random", False, True), ("reversed", False, False), ("random", True, False)])
@pytest.mark.parametrize("form", list(FORMS))
def test_lists_of_any_order_with_empty_rows_and_entries_out_of_range(oracle, form, order, sigma, token_copy):
    batch, Hq, Hkv, T, tail = FORMS[form]
    n, seg = T * BLOCK - tail, R * BLOCK
    Q, K, V = _qkv(T, batch, Hq, Hkv, n)
    p = pbs.problem(batch, Hq, Hkv, n, D, BLOCK, seg, "bf16", flags=pbs.FLAG_TOKEN_ORDER_COPY if token_copy else 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    scores = (torch.rand((batch, Hkv, n), generator=g, device="cuda") if order == "random"
              else torch.linspace(0.0, 1.0, n, device="cuda").expand(batch, Hkv, n).contiguous())
    kidx, Kp, Vt = pbs.segment_permute(p, scores, K, V)
    qidx = None
    if sigma:
        qidx = i32_dev(wl.random_segment_perm(4, batch * Hq, n, seg).reshape(batch, Hq, n))
        Q = torch.gather(Q, 2, qidx.long()[..., None].expand(-1, -1, -1, D)).contiguous()
    rng = np.random.default_rng(T)
    cnt, clean_cnt = np.zeros((2, batch, Hq, T), dtype=np.int32)
    cols, clean = np.full((2, batch, Hq, T, T), -1, dtype=np.int32)
    for b in range(batch):
        for h in range(Hq):
            for i in range(T):
                lo, full = i // R * R, (i // R + 1) * seg <= n
                ni = lo + R if full else i + 1
                own = list(range(lo, lo + R)) if full else [i]
                lst = rng.choice(lo if full else i, min(lo if full else i, rng.integers(0, 6)), replace=False).tolist()
                how = rng.integers(0, 6)
                if how == 0:
                    lst = []
                elif how == 1:                             # the own segment ends it, ascending
                    lst = sorted(lst) + own
                elif how == 2:
                    lst = sorted(lst + own, reverse=True)
                elif how == 3:
                    lst = rng.permutation(lst + own).tolist()
                elif how == 4:
                    lst = sorted(lst + [i])
                else:                                      # no block of its own segment
                    lst = sorted(lst)
                clean_cnt[b, h, i] = len(lst)
                clean[b, h, i, :len(lst)] = lst
                if rng.integers(0, 3) == 0:
                    for junk in (-1, ni, -2 ** 31, T + 5, 2 ** 20 + 3):
                        if len(lst) < T:
                            lst.insert(int(rng.integers(0, len(lst) + 1)), junk)
                cnt[b, h, i] = len(lst)
                cols[b, h, i, :len(lst)] = lst
    got, lse = pbs.attn_fwd(p, Q, Kp, Vt, qidx, kidx, i32_dev(cnt), i32_dev(cols), want_lse=True)
    torch.cuda.synchronize()
    rows = np.argwhere(np.ones((batch, Hq, T), dtype=bool))
    if len(rows) > 700:
        rows = rows[rng.choice(len(rows), 400, replace=False)]
    kh = kidx.cpu().numpy()
    want, want_lse = oracle.attn_rows(_host(Q), oracle.gather_rows(_host(K), kh), oracle.gather_rows(_host(V), kh),
                                      None if qidx is None else qidx.cpu().numpy(), kh, clean_cnt, clean, BLOCK, rows,
                                      want_lse=True)
    got, lse = to_host(got), lse.cpu().numpy()
    err_got, err_want = [], []
    for k, (b, h, i) in enumerate(rows):
        lo, hi = i * BLOCK, min(n, (i + 1) * BLOCK)
        fin = np.isfinite(want_lse[k][:hi - lo])           # queries that see a listed key
        if clean_cnt[b, h, i] == 0:
            fin[:] = False
        assert (got[b, h, lo:hi][~fin] == 0).all() and np.isneginf(lse[b, h, lo:hi][~fin]).all(), (b, h, i)
        # fp32 logits within 8 and sums of at most ten thousand terms: 2^-24 * (8 + 14) is 1.3e-6
        np.testing.assert_allclose(lse[b, h, lo:hi][fin], want_lse[k][:hi - lo][fin], atol=2e-5)
        err_got.append(got[b, h, lo:hi][fin])
        err_want.append(want[k][:hi - lo][fin])
    check_close(np.concatenate(err_got), np.concatenate(err_want), "bf16", form)


@pytest.mark.parametrize("form", list(FORMS))
def test_values_that_are_not_finite_stay_with_the_rows_that_list_them(form):
    batch, Hq, Hkv, T, tail = FORMS[form]
    n, at = T * BLOCK - tail, BLOCK + 3
    Q, K, V = _qkv(T + 1, batch, Hq, Hkv, n)
    p = pbs.problem(batch, Hq, Hkv, n, D, BLOCK, BLOCK, "bf16")
    rng = np.random.default_rng(3)
    cnt = np.zeros((batch, Hq, T), dtype=np.int32)
    cols = np.full((batch, Hq, T, T), -1, dtype=np.int32)
    listed = np.zeros((batch, Hq, T), dtype=bool)
    for b, h, i in np.ndindex(batch, Hq, T):
        lst = rng.permutation(i)[:rng.integers(0, 9)].tolist() + [i]
        if rng.integers(0, 2):
            lst = lst[::-1]
        listed[b, h, i] = 1 in lst
        cnt[b, h, i] = len(lst)
        cols[b, h, i, :len(lst)] = lst
    cnt, cols = i32_dev(cnt), i32_dev(cols)

    def run(v):
        kidx, kp, vt = pbs.segment_permute(p, None, K, v)
        return pbs.attn_fwd(p, Q, kp, vt, None, kidx, cnt, cols, want_lse=True)
    want, want_lse = run(V)
    bad = V.clone()
    bad[:, :, at, 3], bad[:, :, at, 5], bad[:, :, at, D - 1] = np.inf, -np.inf, np.nan
    bad[:, :, at, 7], bad[:, :, at + 1, 7] = np.inf, -np.inf
    got, lse = run(bad)
    torch.cuda.synchronize()
    assert listed.any() and not listed[:, :, 2:].all()
    # the queries of later blocks whose lists hold block 1 see the key; those of block 1 itself may also meet it with weight 0,
    # which is NaN
    lists_it = torch.from_numpy(np.repeat(listed, BLOCK, axis=-1)[..., :n]).cuda()
    behind = lists_it.clone()
    behind[..., :2 * BLOCK] = False
    want = want.clone()
    for e, value in ((3, np.inf), (5, -np.inf), (D - 1, np.nan), (7, np.nan)):
        want[..., e][behind] = value
        got[..., BLOCK:2 * BLOCK, e] = want[..., BLOCK:2 * BLOCK, e]
    torch.testing.assert_close(got, want, rtol=0, atol=0, equal_nan=True)
    assert torch.equal(lse, want_lse)


def test_lists_longer_than_a_staged_chunk_with_a_workgroup_per_row(oracle):
    # 2200 rows; lists that end around the 1024 entries that are staged at a time, with and without the own segment that
    # token order replaces at their end
    T, Hq, Hkv, seg = 1100, 2, 1, 1024
    n, own = T * BLOCK - 77, seg // BLOCK
    Q, K, V = _qkv(5, 1, Hq, Hkv, n)
    p = pbs.problem(1, Hq, Hkv, n, D, BLOCK, seg, "bf16", flags=pbs.FLAG_TOKEN_ORDER_COPY)
    kidx, Kp, Vt = pbs.segment_permute(p, None, K, V)
    rng = np.random.default_rng(12)
    lens = [1015, 1020, 1021, 1022, 1023, 1024, 1025, 1026, 1027, 1028, 1032, 1040]
    cnt = np.ones((1, Hq, T), dtype=np.int32)
    cols = np.full((1, Hq, T, T), -1, dtype=np.int32)
    cols[..., 0] = np.arange(T)
    rows = []
    for k, m in enumerate(lens):
        h, i = k % Hq, T - 1 - 3 * k
        lo, full = i // own * own, (i // own + 1) * seg <= n
        end = list(range(lo, lo + own)) if full and k % 3 else [i]
        lst = sorted(rng.choice(lo if full else i, m - len(end), replace=False).tolist()) + end
        cnt[0, h, i] = m
        cols[0, h, i, :m] = lst
        rows.append([0, h, i])
    got = to_host(pbs.attn_fwd(p, Q, Kp, Vt, None, kidx, i32_dev(cnt), i32_dev(cols)))
    torch.cuda.synchronize()
    want = oracle.attn_rows(_host(Q), _host(K), _host(V), None, kidx.cpu().numpy(), cnt, cols, BLOCK, np.asarray(rows))
    for k, (_, h, i) in enumerate(rows):
        lo, hi = i * BLOCK, min(n, (i + 1) * BLOCK)
        check_close(got[0, h, lo:hi], want[k][:hi - lo], "bf16", "%d entries" % lens[k])


def test_time_of_one_row_to_a_head_is_that_of_eight_rows_to_a_head():
    # 256 rows of a block each: 17 and 18 us; 81 where workgroups without a row wait for a compute unit between those that
    # have one
    def best(Hq, Hkv, T):
        n = T * BLOCK
        Q, K, V = _qkv(1, 1, Hq, Hkv, n)
        p = pbs.problem(1, Hq, Hkv, n, D, BLOCK, BLOCK, "bf16")
        kidx, kp, vt = pbs.segment_permute(p, None, K, V)
        cnt = torch.ones((1, Hq, T), dtype=torch.int32, device="cuda")
        cols = torch.arange(T, dtype=torch.int32, device="cuda").view(1, 1, T, 1).expand(1, Hq, T, T).contiguous()
        O, ws, times = torch.empty_like(Q), pbs.alloc_workspace(p, pbs.STAGE_ATTN_FWD), []
        for _ in range(7):
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            start.record()
            for _ in range(20):
                pbs.attn_fwd(p, Q, kp, vt, None, kidx, cnt, cols, O, ws=ws)
            stop.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(stop))
        return min(times)
    many, few = best(256, 256, 1), best(32, 8, 8)
    assert many < 1.5 * few, (many, few)
