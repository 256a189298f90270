"""GPU parity of the query-block kernels where a tile, a mask or the dealing of heads to the XCDs begins or ends."""
import pytest
import torch

import oracle
import workloads as W
from gpu_util import (check_attention, check_lse, check_rows, default_scale, dev, kernel_names, make_attention_case, nan_outputs,
                      oracle_attention_rows_parallel, template_arguments)

pytestmark = pytest.mark.gpu


# nuggets and local rows on both sides of a 32-key block and a 64-key tile; heads in blocks of H / 8 per XCD (the 8-wavefront
# kernel, and grouped heads), in turn otherwise; one or two query blocks per workgroup
@pytest.mark.parametrize("q_lens,H,H_kv,d_h", [
    ([129, 257, 130], 8, 8, 128), ([129, 257, 130], 16, 16, 64), ([200, 129], 24, 8, 128),
    ([16, 128, 65], 16, 2, 128), ([128, 31, 64], 12, 12, 64), ([257, 300] * 8, 16, 16, 64),
])
@pytest.mark.parametrize("k0", [31, 63, 96])
def test_edges_of_tiles_masks_and_head_blocks(q_lens, H, H_kv, d_h, k0):
    import paper_2310_02409_amd as D
    k_lens = [k0 + i % 3 for i in range(len(q_lens))]
    m_lens = [q + 30 + i % 4 for i, q in enumerate(q_lens)]
    host, t = make_attention_case(431 + k0, q_lens, k_lens, m_lens, H, H_kv, d_h, torch.bfloat16, dev())
    scale = default_scale(d_h)
    want, lse_want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"],
                                      host["cu_nuggets"], host["cu_local"], scale)
    O, lse = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"],
                                     max(q_lens), max(k_lens), max(m_lens), scale, want_lse=True)
    check_attention(O, want, torch.bfloat16)
    check_lse(lse, lse_want, torch.bfloat16)


# grouped heads and small query blocks, one split each: rows requested with the non-temporal hint (the host bounds promise
# more than half of the last-level cache) and without, the same bits; the longest block of one pass, the next of two
@pytest.mark.parametrize("q,H,H_kv,d_h", [(1, 64, 8, 128), (1, 32, 8, 64), (4, 32, 32, 128), (8, 32, 8, 64), (9, 32, 8, 128)])
def test_streamed_rows_of_grouped_heads(q, H, H_kv, d_h):
    import paper_2310_02409_amd as D
    B = 70
    k_lens, m_lens = [i % 67 for i in range(B)], [q + i % 35 for i in range(B)]
    host, t = make_attention_case(470 + q, [q] * B, k_lens, m_lens, H, H_kv, d_h, torch.bfloat16, dev())
    scale = default_scale(d_h)
    want, lse_want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"],
                                      host["cu_nuggets"], host["cu_local"], scale)
    got = [D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], q, max_k,
                                   max(m_lens), scale, want_lse=True, ws=torch.zeros(16, dtype=torch.uint8, device=dev()))
           for max_k in (max(k_lens), 20000)]
    for O, lse in got:
        check_attention(O, want, torch.bfloat16)
        check_lse(lse, lse_want, torch.bfloat16)
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


# the same with the keys of a (sequence, K/V head) pair shared by several workgroups, whose records and flags the last one reads:
# plain call, head-major cache and cached form, twice on one workspace
@pytest.mark.parametrize("q,H,H_kv,d_h", [(1, 64, 8, 128), (2, 32, 8, 128), (1, 32, 4, 64), (4, 16, 16, 64)])
def test_streamed_rows_in_several_splits(q, H, H_kv, d_h):
    import paper_2310_02409_amd as D
    k_lens, m_lens, big = [3001, 1500], [700, 513], 1 << 16
    host, t = make_attention_case(480 + q, [q] * 2, k_lens, m_lens, H, H_kv, d_h, torch.bfloat16, dev())
    scale = default_scale(d_h)
    want, lse_want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"],
                                      host["cu_nuggets"], host["cu_local"], scale)
    need = D.dodo_nugget_attention_workspace_bytes_grouped(2, H, H_kv, d_h, q, max(k_lens), max(m_lens), D.BF16)
    assert need > 2 * (2 * q * H * (d_h + 3) * 4) and 2 * big * H_kv * d_h * 4 >= 128 << 20
    ws = torch.zeros(need, dtype=torch.uint8, device=dev())
    Kh, Vh = (t[n].transpose(0, 1).contiguous() for n in ("Kn", "Vn"))
    start, length = t["cu_nuggets"][:2].contiguous(), torch.tensor(k_lens, dtype=torch.int32, device=dev())
    loc = (t["Kl"], t["Vl"], t["cu_q"])
    kw = dict(want_lse=True, ws=ws)
    calls = [lambda mk: D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], *loc, t["cu_nuggets"], t["cu_local"], q, mk, max(m_lens), scale, **kw),
             lambda mk: D.dodo_nugget_attention(t["Q"], Kh, Vh, *loc, t["cu_nuggets"], t["cu_local"], q, mk, max(m_lens), scale, D.HEAD_MAJOR, **kw),
             lambda mk: D.dodo_nugget_attention_cached(t["Q"], t["Kn"], t["Vn"], *loc, start, length, t["cu_local"], q, mk, max(m_lens), scale, **kw)]
    for call in calls:
        for _ in range(2):
            O, lse = call(big)
            check_attention(O, want, torch.bfloat16)
            check_lse(lse, lse_want, torch.bfloat16)


def _split_case(q_lens, k_lens, m_lens, H, H_kv, d_h):
    host, t = make_attention_case(520 + len(q_lens) + H, q_lens, k_lens, m_lens, H, H_kv, d_h, torch.bfloat16, dev())
    scale = default_scale(d_h)
    want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"], host["cu_nuggets"],
                            host["cu_local"], scale)
    return t, scale, want


# few rows over many keys: the keys of a query block shared by several workgroups, with the workspace that this would like,
# with one for two splits, and without; rows and blocks that see nothing, splits without a tile, blocks of 128 rows of what the
# 8-wavefront kernel would take whole
@pytest.mark.parametrize("q_lens,k_lens,m_lens,H,H_kv,d_h", [
    ([20], [1500], [33], 4, 4, 128), ([16, 128, 31], [1100, 0, 64], [16, 700, 20], 8, 2, 128), ([130, 257], [1300, 900], [130, 300], 2, 2, 64),
    ([64, 40], [1999, 1], [10, 40], 3, 1, 128), ([129], [2113], [0], 4, 4, 64),
])
def test_keys_shared_by_workgroups(q_lens, k_lens, m_lens, H, H_kv, d_h):
    import paper_2310_02409_amd as D
    t, scale, (want, lse_want) = _split_case(q_lens, k_lens, m_lens, H, H_kv, d_h)
    B, mq, mk, mm = len(q_lens), max(q_lens), max(k_lens), max(m_lens)
    need = D.dodo_nugget_attention_workspace_bytes(B, H, d_h, mq, mk, mm, D.BF16)
    two = B * mq * H * 2 * (d_h + 2) * 4
    assert need >= two
    a = (t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], mq, mk, mm, scale)
    results = []
    for size in (need, two, 16, None):
        ws = None if size is None else torch.full((size,), 255, dtype=torch.uint8, device=dev())
        O, lse = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], *a, want_lse=True, ws=ws)
        check_attention(O, want, torch.bfloat16)
        check_lse(lse, lse_want, torch.bfloat16)
        results.append((O, lse))
    assert torch.equal(results[0][0], results[3][0]) and torch.equal(results[0][1], results[3][1])  # (None: the binding allocates)
    O = torch.empty_like(t["Q"])
    D.dodo_nugget_attention_noalloc(t["Q"], t["Kn"], t["Vn"], *a, 0, O)
    assert torch.equal(O, results[2][0])
    hm = D.dodo_nugget_attention(t["Q"], t["Kn"].transpose(0, 1).contiguous(), t["Vn"].transpose(0, 1).contiguous(), *a, D.HEAD_MAJOR)[0]
    assert torch.equal(hm, results[0][0])


# More than 128 rows over many keys: shared out in blocks of 128 rows where blocks of 64 would be more than the compute units, and not
# left to the 8-wavefront kernel, whose fixed exponent offset costs precision; with the workspace for it and with one for two shares.
@pytest.mark.parametrize("B,q,k,m,H,H_kv,d_h", [(8, 525, 2768, 574, 4, 4, 128), (2, 214, 2312, 214, 40, 40, 128), (1, 570, 2674, 697, 32, 8, 128),
                                                (1, 1195, 4537, 1423, 16, 16, 64)])
@pytest.mark.parametrize("room", ["whole", "two shares"])
def test_blocks_of_128_rows_share_their_keys(B, q, k, m, H, H_kv, d_h, room):
    import paper_2310_02409_amd as D
    q_lens, k_lens, m_lens = [q - 9 * b for b in range(B)], [k - 70 * b for b in range(B)], [m - 5 * b for b in range(B)]
    host, t = make_attention_case(530, q_lens, k_lens, m_lens, H, H_kv, d_h, torch.bfloat16, dev())
    scale = default_scale(d_h)
    two = B * q * H * 2 * (d_h + 2) * 4
    need = D.dodo_nugget_attention_workspace_bytes_grouped(B, H, H_kv, d_h, q, k, m, D.BF16)
    assert need >= two
    O, lse = nan_outputs(t["Q"], H)
    ws = torch.full((two if room != "whole" else need,), 255, dtype=torch.uint8, device=dev())
    names = kernel_names(lambda: D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], q, k, m,
                                                         scale, O=O, lse=lse, ws=ws), "block_attention_kernel")
    assert len(names) == 1 and template_arguments(names[0])[0] == "4", names
    assert bool(torch.isfinite(O.float()).all())
    rows = [(b, (3 * b + h) % H, i) for b in range(B) for h in (0, 1) for i in (0, 1, 127, 128, q_lens[b] // 2, q_lens[b] - 1)]
    want = oracle_attention_rows_parallel(host, host["Kn"], host["Vn"], host["cu_nuggets"], scale, rows)
    check_rows(O, lse, host["cu_q"], rows, *want, torch.bfloat16)


def test_shared_keys_through_an_index_list_and_a_workspace_used_by_a_decode_call_next():
    import paper_2310_02409_amd as D
    import workloads as W
    H, q, n, k = 4, 48, 3000, 1200
    g = torch.Generator().manual_seed(9)
    r = lambda *s: torch.randn(s, generator=g).to(torch.bfloat16).to(dev())
    K, V, Q, Kl, Vl = r(n, H, 128), r(n, H, 128), r(q, H, 128), r(60, H, 128), r(60, H, 128)
    idx = torch.randperm(n, generator=g)[:k].sort().values.int().to(dev())
    cu = lambda v: W.cumulative([v], dev())
    Kn, Vn = D.dodo_gather_nuggets(K, V, idx, cu(n), cu(k), k)
    ws = torch.zeros(D.dodo_nugget_attention_workspace_bytes(1, H, 128, q, k, 60, D.BF16), dtype=torch.uint8, device=dev())
    args = (Kl, Vl, cu(q), cu(k), cu(60), q, k, 60)
    O, lse = D.dodo_nugget_attention(Q, Kn, Vn, *args, want_lse=True, ws=ws)
    Oi, lse_i = D.dodo_nugget_attention_indexed(Q, K, V, idx, cu(n), *args, n, want_lse=True, ws=ws)
    assert torch.equal(O, Oi) and torch.equal(lse, lse_i)
    one = (Q[:1].contiguous(), Kn, Vn, Kl, Vl, cu(1), cu(k), cu(60), 1, k, 60)
    fresh = D.dodo_nugget_attention(*one, ws=torch.zeros_like(ws))[0]
    assert torch.equal(D.dodo_nugget_attention(*one, ws=ws)[0], fresh)


def _finite(x):
    return torch.isfinite(x.float())


# A NaN or an infinity in K or V reaches the rows that see it, whether the keys are shared out or not: the same rows finite with
# a workspace and without, and those as if the others were not there.  Nuggets of the middle of the keys; every query row of
# their K/V head sees them.  (lse of a row without a sum is -inf.)
@pytest.mark.parametrize("d_h", [64, 128])
@pytest.mark.parametrize("tensor,value", [("Kn", float("nan")), ("Kn", float("inf")), ("Vn", float("nan")), ("Vn", float("-inf"))])
def test_shared_keys_that_are_not_finite(tensor, value, d_h):
    import paper_2310_02409_amd as D
    q_lens, k_lens, m_lens, H, H_kv = [20, 40], [1500, 1100], [33, 64], 4, 2
    host, t = make_attention_case(540, q_lens, k_lens, m_lens, H, H_kv, d_h, torch.bfloat16, dev())
    t["Q"][..., 3] = t["Q"][..., 3].abs() + 0.5  # an infinite channel of K makes an infinite logit, of one sign
    t[tensor][700, 1, 3] = value                 # sequence 0, K/V head 1: query heads 2 and 3
    scale = default_scale(d_h)
    a = (t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], 40, 1500, 64, scale)
    need = D.dodo_nugget_attention_workspace_bytes(2, H, d_h, 40, 1500, 64, D.BF16)
    two = 2 * 40 * H * 2 * (d_h + 2) * 4
    assert need > two
    got = []
    for size in (16, two, need):
        O, lse = (torch.full_like(t["Q"], float("nan")), torch.full((60, H), float("nan"), device=dev()))
        D.dodo_nugget_attention(*a, O=O, lse=lse, ws=torch.full((size,), 255, dtype=torch.uint8, device=dev()))
        got.append((O, lse))
    hit = torch.zeros(60, H, dtype=torch.bool, device=dev())
    hit[:20, 2:] = True
    for O, lse in got:
        assert torch.equal(_finite(O), _finite(got[0][0])) and torch.equal(_finite(lse), _finite(got[0][1]))
        assert torch.equal(_finite(O).all(-1), ~hit) and not (torch.isnan(lse)).any()
        fine = _finite(got[0][0])
        assert (O[fine].float() - got[0][0][fine].float()).abs().max() <= 2e-2
        ok = _finite(lse)
        assert (lse[ok] - got[0][1][ok]).abs().max() <= 2e-2


# A first tile whose logits are all -inf (nuggets that a caller rules out so): the rest decides, also where it lies far from zero.  (Few
# heads, which halves of tiles take; the 8-wavefront kernel, whose offsets come from the first tile, further down.)
@pytest.mark.parametrize("far", [0.0, -300.0, 300.0])
def test_first_tile_without_a_finite_logit(far):
    import paper_2310_02409_amd as D
    q, k, m, H, d_h = 160, 100, 160, 2, 128
    host, t = make_attention_case(550, [q], [k], [m], H, H, d_h, torch.bfloat16, "cpu")
    scale = default_scale(d_h)
    t["Q"][..., 0], t["Q"][..., 1] = 1.0, 16.0
    for x in (t["Kn"], t["Kl"]):
        x[..., 0], x[..., 1] = 0.0, far / (16.0 * scale)
    t["Kn"][:64, :, 0] = float("-inf")
    host = {n: W.to_numpy(v) for n, v in t.items()}
    want, lse_want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"], host["cu_nuggets"],
                                      host["cu_local"], scale)
    g = {n: v.to(dev()) for n, v in t.items()}
    O, lse = D.dodo_nugget_attention(g["Q"], g["Kn"], g["Vn"], g["Kl"], g["Vl"], g["cu_q"], g["cu_nuggets"], g["cu_local"], q, k, m, scale,
                                     want_lse=True, ws=torch.zeros(16, dtype=torch.uint8, device=dev()))
    check_attention(O, want, torch.bfloat16)
    check_lse(lse, lse_want, torch.bfloat16)


# Rows past the sequence's last one in a query block (they read as zeros, so that a ruled-out nugget's logits are NaN there) have
# no say in the others' results: the same bits as in a block that is full.  (Few heads; the 8-wavefront kernel further down.)
def test_rows_past_the_last_do_not_count():
    import paper_2310_02409_amd as D
    q, k, H, d_h = 160, 300, 2, 128
    _, t = make_attention_case(560, [q], [k], [0], H, H, d_h, torch.bfloat16, dev())
    t["Q"][..., 0] = 1.0
    t["Kn"][7, :, 0] = float("-inf")
    got = []
    for rows in (160, 150):
        cu = torch.tensor([0, rows], dtype=torch.int32, device=dev())
        got.append(D.dodo_nugget_attention(t["Q"][:rows].contiguous(), t["Kn"], t["Vn"], t["Kl"], t["Vl"], cu, t["cu_nuggets"], t["cu_local"], rows, k,
                                           0, want_lse=True, ws=torch.zeros(16, dtype=torch.uint8, device=dev())))
    assert _finite(got[1][0]).all() and _finite(got[1][1]).all()
    assert torch.equal(got[0][0][:150], got[1][0]) and torch.equal(got[0][1][:150], got[1][1])


def _kernels(call):
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA], acc_events=True) as prof:
        call()
        torch.cuda.synchronize()
    return [e.name for e in prof.events() if "group_attention_kernel" in e.name]


# Segments of a text share its nuggets and overlap in its local rows: they are asked for without the non-temporal hint however
# large the bounds, where a plain call with the same bounds has it.
def test_rows_of_segments_are_not_streamed():
    import paper_2310_02409_amd as D
    n, seg, H, d_h, k = 64, 8, 16, 128, 40
    host, t = make_attention_case(570, [n], [k], [n], H, H, d_h, torch.bfloat16, dev())
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device=dev())
    starts = list(range(0, n, seg))
    scale, big = default_scale(d_h), 1 << 20
    kv = (t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"])
    ws = torch.zeros(16, dtype=torch.uint8, device=dev())
    seg_args = (i32(starts + [n]), i32([0] * len(starts)), i32([s * k // n for s in starts]), i32([max(0, s - 16) for s in starts]),
                i32([s + seg - max(0, s - 16) for s in starts]))
    names = _kernels(lambda: D.dodo_nugget_attention_segments(*kv, *seg_args, seg, big, seg + 16, scale, ws=ws))
    assert len(names) == 1 and "false" in names[0] and "true" not in names[0]
    cu = i32(starts + [n])
    names = _kernels(lambda: D.dodo_nugget_attention(*kv, cu, i32([s * k // n for s in starts] + [k]), cu, seg, big, seg, scale, ws=ws))
    assert len(names) == 1 and "true" in names[0]


# A bound on the query rows that is too small leaves rows without a place for their shares: nothing is written past the workspace,
# and the rows within the bound are whole.
@pytest.mark.parametrize("q,said", [(25, 20), (200, 130)])
def test_more_rows_than_said_stay_inside_the_workspace(q, said):
    import paper_2310_02409_amd as D
    H, d_h, k, m = 2, 128, 2500, 300
    t, scale, (want, lse_want) = _split_case([q], [k], [m], H, H, d_h)
    need = D.dodo_nugget_attention_workspace_bytes(1, H, d_h, said, k, m, D.BF16)
    assert need > 0
    room = torch.full((need + (1 << 22),), 255, dtype=torch.uint8, device=dev())
    O, lse = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], said, k, m, scale,
                                     want_lse=True, ws=room[:need])
    assert torch.all(room[need:] == 255)
    check_attention(O[:said], want[:said], torch.bfloat16)
    check_lse(lse[:said], lse_want[:said], torch.bfloat16)


# A workspace that is anything but zero, though free of the ready value, serves calls that share keys out and decode calls in turn:
# a ragged batch leaves words of it alone, and none that it writes is a flag to the next call.
def test_workspace_of_shared_keys_serves_a_decode_call():
    import paper_2310_02409_amd as D
    q_lens, k_lens, m_lens, H, d_h = [48, 17, 33], [2900, 1, 2000], [60, 20, 33], 4, 128
    t, scale, (want, _) = _split_case(q_lens, k_lens, m_lens, H, H, d_h)
    mq, mk, mm = max(q_lens), max(k_lens), max(m_lens)
    one = dict(cu_q=torch.arange(4, dtype=torch.int32, device=dev()), Q=t["Q"][:3].contiguous())
    decode = lambda ws: D.dodo_nugget_attention(one["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], one["cu_q"], t["cu_nuggets"], t["cu_local"], 1, mk, mm,
                                                scale, want_lse=True, ws=ws)
    size = max(D.dodo_nugget_attention_workspace_bytes(3, H, d_h, n, mk, mm, D.BF16) for n in (1, mq))
    fresh = decode(torch.zeros(size, dtype=torch.uint8, device=dev()))
    ws = torch.full((size,), 0x5A, dtype=torch.uint8, device=dev())
    for _ in range(2):
        O = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], mq, mk, mm, scale, ws=ws)[0]
        check_attention(O, want, torch.bfloat16)
        got = decode(ws)
        assert torch.equal(got[0], fresh[0]) and torch.equal(got[1], fresh[1])


# What one (sequence, head) holds stays there: tiles that are not full leave nothing of an earlier tile, block or head in LDS (rows
# past a tile's last one arrive as zeros).  NaN in all K and V of two of 256 pairs; every other row has the bits of a run without.
@pytest.mark.parametrize("q,k", [(300, 70), (100, 70), (129, 3)])
def test_nan_stays_in_its_head(q, k):
    import paper_2310_02409_amd as D
    B, H, d_h, m = 8, 32, 128, q + 5
    _, t = make_attention_case(580 + q, [q] * B, [k] * B, [m] * B, H, H, d_h, torch.bfloat16, dev())
    run = lambda: D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], q, k, m, want_lse=True)
    O, lse = run()
    bad = torch.zeros(B * q, H, dtype=torch.bool, device=dev())
    for b, h in ((2, 3), (5, 17)):
        for n, rows in (("Kn", k), ("Vn", k), ("Kl", m), ("Vl", m)):
            t[n][b * rows:(b + 1) * rows, h] = float("nan")
        bad[b * q:(b + 1) * q, h] = True
    O2, lse2 = run()
    assert torch.equal(O2[~bad], O[~bad]) and torch.equal(lse2[~bad], lse[~bad])
    assert torch.isnan(O2[bad]).all()


# Grouped heads whose rows go through the tiles together: blocks of 128 and 256 rows, 2, 3, 4 and 8 heads (a block begins at any head
# of a query row), rows left over, sequences of fewer rows than the bound, several blocks per sequence with the heavy ones first, and
# keys shared by several workgroups in blocks of 64 and of 128 rows; the same rows through an index list.
@pytest.mark.parametrize("B,q,k,H,H_kv,d_h", [
    (40, 16, 70, 16, 2, 128), (40, 17, 33, 16, 2, 128), (40, 21, 64, 16, 2, 64), (24, 43, 40, 24, 8, 128), (20, 33, 65, 32, 8, 64),
    (70, 130, 20, 16, 8, 128), (12, 546, 30, 16, 2, 128), (5, 16, 2000, 64, 8, 128), (9, 40, 1500, 32, 8, 64),
    (6, 33, 1960, 16, 4, 128), (6, 71, 905, 16, 4, 128), (3, 91, 1081, 16, 4, 128), (2, 139, 560, 16, 2, 128),
])
def test_rows_of_grouped_heads_together(B, q, k, H, H_kv, d_h):
    import paper_2310_02409_amd as D
    q_lens = [max(1, q - (3 * b) % 11) for b in range(B)]
    k_lens = [k - b % 5 for b in range(B)]
    m_lens = [n + (7 * b) % 30 - (b % 3 == 2) * 9 for b, n in enumerate(q_lens)]
    m_lens = [max(0, m) for m in m_lens]
    host, t = make_attention_case(900 + q, q_lens, k_lens, m_lens, H, H_kv, d_h, torch.bfloat16, dev())
    scale = default_scale(d_h)
    want, lse_want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"], host["cu_nuggets"],
                                      host["cu_local"], scale)
    a = (t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], max(q_lens), max(k_lens), max(m_lens))
    O, lse = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], *a, scale, want_lse=True)
    check_attention(O, want, torch.bfloat16)
    check_lse(lse, lse_want, torch.bfloat16)
    idx = torch.cat([torch.arange(n, dtype=torch.int32) for n in k_lens]).to(dev())
    Oi, lse_i = D.dodo_nugget_attention_indexed(t["Q"], t["Kn"], t["Vn"], idx, t["cu_nuggets"], *a, max(k_lens), scale, want_lse=True)
    assert torch.equal(O, Oi) and torch.equal(lse, lse_i)


# Two wavefronts per 32 rows, each half of a tile's keys: rows that see keys of one half only, none at all, or one key more; one and two
# workgroups per compute unit (more than 256 blocks), blocks of 64 rows with one left over, and the whole-tile form beside it.
@pytest.mark.parametrize("B,q,k,H,H_kv,d_h", [
    (2, 40, 31, 4, 4, 128), (3, 65, 33, 4, 4, 128), (2, 64, 0, 8, 8, 64), (3, 129, 64, 2, 2, 64), (20, 64, 95, 16, 16, 128),
    (20, 33, 32, 16, 16, 64), (20, 100, 97, 16, 16, 128), (1, 16, 1100, 4, 4, 128), (2, 70, 900, 6, 3, 64),
])
def test_halves_of_a_tile(B, q, k, H, H_kv, d_h):
    import paper_2310_02409_amd as D
    q_lens = [max(1, q - b % 7) for b in range(B)]
    k_lens = [max(0, k - b % 3) for b in range(B)]
    m_lens = [max(0, n - (5 if b % 2 else -35)) for b, n in enumerate(q_lens)]  # (some rows see no local row, or the first only)
    host, t = make_attention_case(950 + q, q_lens, k_lens, m_lens, H, H_kv, d_h, torch.bfloat16, dev())
    scale = default_scale(d_h)
    want, lse_want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"], host["cu_nuggets"],
                                      host["cu_local"], scale)
    a = (t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], max(q_lens), max(k_lens), max(m_lens))
    O, lse = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], *a, scale, want_lse=True)
    check_attention(O, want, torch.bfloat16)
    check_lse(lse, lse_want, torch.bfloat16)


# A NaN or an infinity in either half of a tile reaches the rows and channels that it reaches when a wavefront takes the whole tile.
@pytest.mark.parametrize("key", [3, 40])
def test_halves_of_a_tile_that_are_not_finite(key):
    import paper_2310_02409_amd as D
    B, q, k, H, d_h = 2, 20, 64, 4, 128
    host, t = make_attention_case(970, [q] * B, [k] * B, [q] * B, H, H, d_h, torch.bfloat16, dev())
    run = lambda: D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], q, k, q)[0]
    clean = run()
    t["Vn"][key, 1, 7] = float("inf")
    t["Vn"][k + key, 2, 9] = float("nan")
    O, want = run(), clean.clone()
    want[:q, 1, 7], want[q:, 2, 9] = float("inf"), float("nan")
    assert torch.equal(torch.nan_to_num(O.float(), nan=-7.0), torch.nan_to_num(want.float(), nan=-7.0))
    t["Kn"][key, 3, 5] = float("nan")
    bad = run()
    assert torch.isnan(bad[:q, 3].float()).all() and torch.equal(bad[q:, 3], clean[q:, 3]) and torch.equal(bad[:, 0], clean[:, 0])


# ---- the 8-wavefront kernel, by its name: it takes calls whose blocks of 64 rows are more than the compute units ----
def _eight(host, t, q_lens, k_lens, m_lens, scale, rows, grouped=False):
    """The call's (O, lse), checked against the oracle at `rows`, and that the 8-wavefront kernel made them."""
    import paper_2310_02409_amd as D
    O, lse = nan_outputs(t["Q"], t["Q"].shape[1])
    names = kernel_names(lambda: D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"],
                                                         max(q_lens), max(k_lens), max(m_lens), scale, O=O, lse=lse), "block_attention_kernel")
    assert len(names) == 1, names
    args = template_arguments(names[0])
    assert args[:2] == ["8", "1"] and args[-1] == ("true" if grouped else "false"), names
    assert bool(torch.isfinite(O.float()).all())
    want = oracle_attention_rows_parallel(host, host["Kn"], host["Vn"], host["cu_nuggets"], scale, rows)
    check_rows(O, lse, host["cu_q"], rows, *want, torch.bfloat16)
    return O, lse


# A huge scale spreads the logits far beyond the fixed exponent offset of a row, so that the block is done again with the running maximum;
# scales that are not positive take that loop from the start.  Blocks of 256 rows and the rest of them, sequences without nuggets.
@pytest.mark.parametrize("q_lens,H,H_kv,d_h", [([300, 160, 257], 32, 32, 128), ([300, 160, 257], 32, 32, 64), ([336, 300, 129, 330, 336, 257, 312, 336], 64, 8, 128)])
@pytest.mark.parametrize("scale", [8.0, -0.09, 0.0])
def test_eight_wavefronts_without_a_fixed_offset(q_lens, H, H_kv, d_h, scale):
    B = len(q_lens)
    k_lens, m_lens = [(60, 0, 30)[b % 3] for b in range(B)], [q + (64, 0, 11)[b % 3] for b, q in enumerate(q_lens)]
    host, t = make_attention_case(1100, q_lens, k_lens, m_lens, H, H_kv, d_h, torch.bfloat16, dev())
    rows = [(b, (5 * b + 3 * i) % H, i) for b, q in enumerate(q_lens) for i in [*range(0, q, 17), 255, 256, q - 1] if i < q]
    _eight(host, t, q_lens, k_lens, m_lens, scale, rows, grouped=H != H_kv)


# The row's exponent offset comes from its first tile: one whose logits are all -inf leaves it none, and the block is done again.
@pytest.mark.parametrize("d_h", [64, 128])
@pytest.mark.parametrize("far", [0.0, -300.0, 300.0])
def test_eight_wavefronts_with_a_first_tile_without_a_finite_logit(far, d_h):
    q_lens, k_lens, m_lens, H = [160, 300, 150], [100, 65, 70], [160, 290, 170], 32
    host, t = make_attention_case(1110, q_lens, k_lens, m_lens, H, H, d_h, torch.bfloat16, "cpu")
    scale = default_scale(d_h)
    t["Q"][..., 0], t["Q"][..., 1] = 1.0, 16.0
    for x in (t["Kn"], t["Kl"]):
        x[..., 0], x[..., 1] = 0.0, far / (16.0 * scale)
    for b, first in enumerate((0, 100, 165)):
        if b != 1:  # (sequence 1 keeps its offsets)
            t["Kn"][first:first + 64, :, 0] = float("-inf")
    host = {n: W.to_numpy(v) for n, v in t.items()}
    rows = [(b, (5 * b + 3 * i) % H, i) for b, q in enumerate(q_lens) for i in [*range(0, q, 11), q - 1]]
    _eight(host, {n: v.to(dev()) for n, v in t.items()}, q_lens, k_lens, m_lens, scale, rows)


# One key far above a row's fixed offset: its weight 2^e times values of 3 overflows (e = 127) before the row sum does (e = 128), and either has
# the block done again; below 2^64 it is not.
@pytest.mark.parametrize("e", [60, 100, 126, 127, 128])
def test_eight_wavefronts_with_a_key_far_above_the_offset(e):
    B, q, k, H, d_h = 3, 160, 130, 32, 128
    host, t = make_attention_case(1115, [q] * B, [k] * B, [0] * B, H, H, d_h, torch.bfloat16, "cpu")
    scale = default_scale(d_h)
    t["Q"][..., 0] = 16.0
    t["Kn"][..., 0] = 0.0
    t["Kn"][[70, k + 129, 2 * k + 64], :, 0] = e / (16.0 * scale * 1.4426950408889634)
    t["Vn"][[70, k + 129, 2 * k + 64]] = 3.0
    host = {n: W.to_numpy(v) for n, v in t.items()}
    rows = [(b, (5 * b + 3 * i) % H, i) for b in range(B) for i in range(0, q, 9)]
    _eight(host, {n: v.to(dev()) for n, v in t.items()}, [q] * B, [k] * B, [0] * B, scale, rows)


# Spare rows of a block have no say in the others' results: a ruled-out nugget, whose logit a row of zeros would make NaN, leaves the rest its
# bits, and the block its fixed offsets.
@pytest.mark.parametrize("d_h", [64, 128])
def test_eight_wavefronts_rows_past_the_last_do_not_count(d_h):
    B, q, k, H = 3, 160, 300, 32
    host, t = make_attention_case(1120, [q] * B, [k] * B, [0] * B, H, H, d_h, torch.bfloat16, dev())
    t["Q"][..., 0] = 1.0
    t["Kn"][[7, k + 70, 2 * k + 299], :, 0] = float("-inf")
    got = []
    for n in (160, 150):
        part = dict(t, Q=t["Q"].view(B, q, H, d_h)[:, :n].reshape(B * n, H, d_h).contiguous(), cu_q=W.cumulative([n] * B, dev()))
        rows = [(b, (5 * b + 3 * i) % H, i) for b in range(B) for i in [*range(0, n, 17), n - 1]]
        got.append(_eight({x: W.to_numpy(v) for x, v in part.items()}, part, [n] * B, [k] * B, [0] * B, default_scale(d_h), rows))
    whole = [x.view(B, q, *x.shape[1:])[:, :150].reshape(B * 150, *x.shape[1:]) for x in got[0]]
    assert torch.equal(whole[0], got[1][0]) and torch.equal(whole[1], got[1][1])
