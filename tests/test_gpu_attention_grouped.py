"""GPU parity: the matrix-core kernel for a few query vectors per K/V row (grouped-query heads and small query
blocks, bf16, d_h = 128 or 64) against the oracle, through dodo_nugget_attention and its variants."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import check_attention, check_lse, default_scale, dev, kernel_names, make_attention_case, nan_outputs

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.fixture(scope="module")
def D():
    import paper_2310_02409_amd as D
    return D


def _check(D, seed, q_lens, k_lens, m_lens, H, H_kv, layout=0, ws="wanted", scale=None, d_h=128):
    host, t = make_attention_case(seed, q_lens, k_lens, m_lens, H, H_kv, d_h, BF, dev())
    scale = default_scale(d_h) if scale is None else scale
    B, mq, mk, mm = len(q_lens), max(q_lens), max(k_lens), max(m_lens)
    O_ref, lse_ref = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"],
                                      host["cu_nuggets"], host["cu_local"], scale)
    Kn, Vn = t["Kn"], t["Vn"]
    if layout == D.HEAD_MAJOR:
        Kn, Vn = Kn.transpose(0, 1).contiguous(), Vn.transpose(0, 1).contiguous()
    O, lse = nan_outputs(t["Q"], H)
    if ws == "wanted":  # as much as the kernel would like to have
        need = D.dodo_nugget_attention_workspace_bytes_grouped(B, H, H_kv, d_h, mq, mk, mm, D.BF16)
    elif ws == "plain":  # what the query without H_kv asks for: fewer splits, same result to the tolerance
        need = D.dodo_nugget_attention_workspace_bytes(B, H, d_h, mq, mk, mm, D.BF16)
    else:
        need = int(ws)
    buf = torch.zeros(max(need, 16), dtype=torch.uint8, device=dev()) if need else None
    for _ in range(2):  # the second call finds the workspace as the first left it
        D.dodo_nugget_attention(t["Q"], Kn, Vn, t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], mq, mk, mm,
                                scale, layout, O=O, lse=lse, ws=buf)
        check_attention(O, O_ref, BF)
        check_lse(lse, lse_ref, BF)
    return O, lse, need


@pytest.mark.parametrize("H,H_kv", [(32, 8), (64, 8), (40, 8), (32, 4), (32, 1)])
def test_grouped_heads_decode_large_batch(D, H, H_kv):
    # one workgroup of two wavefronts per (sequence, KV head): group sizes 4, 8, 5 (not a power of two), 32
    rng = np.random.default_rng(H * 100 + H_kv)
    B = 70
    k_lens = [int(v) for v in rng.integers(0, 150, B)]
    m_lens = [int(v) for v in rng.integers(1, 70, B)]
    k_lens[3], m_lens[3] = 0, 1
    k_lens[4], m_lens[4] = 31, 33   # one ragged tile each
    k_lens[5], m_lens[5] = 64, 32   # whole tiles only
    _check(D, 700 + H_kv, [1] * B, k_lens, m_lens, H, H_kv)


def test_grouped_heads_decode_splits_over_workgroups(D):
    # few (sequence, KV head) pairs and long caches: the keys of a pair are split over workgroups, whose partial
    # records the last one merges; with the larger workspace more splits than with the plain one
    q, k, m = [1, 1], [3277, 1500], [1089, 1025]
    _, _, wanted = _check(D, 710, q, k, m, 64, 8)
    _, _, plain = _check(D, 710, q, k, m, 64, 8, ws="plain")
    assert wanted > plain
    _check(D, 711, q, k, m, 32, 8, layout=1)
    # four wavefronts per workgroup (fewer than two workgroups per compute unit in all), ragged split ends
    _check(D, 712, [1] * 5, [205, 410, 333, 1, 0], [257, 257, 40, 3, 5], 64, 8)
    _check(D, 713, [1] * 3, [2000, 37, 900], [300, 700, 31], 40, 8)


def test_small_query_blocks_share_their_keys(D):
    # 2 <= q <= 8 rows: vector (row, head); every row stops at its own causal limit (also m_b < q_b: early rows see
    # no local row at all), ragged q_b, sequences without queries
    rng = np.random.default_rng(9)
    B = 48
    q_lens = [int(v) for v in rng.integers(0, 5, B)]
    q_lens[0], q_lens[1] = 4, 0
    k_lens = [int(v) for v in rng.integers(0, 120, B)]
    m_lens = [int(v) for v in rng.integers(0, 40, B)]
    m_lens[0] = 2
    _check(D, 720, q_lens, k_lens, m_lens, 32, 4)    # 8 heads x up to 4 rows = 32 vectors
    _check(D, 721, q_lens, k_lens, m_lens, 40, 8)    # 5 heads x 4 rows
    q8 = [int(v) for v in rng.integers(1, 9, B)]
    _check(D, 722, q8, k_lens, m_lens, 32, 32)       # multi-head attention: 8 rows of one head
    _check(D, 723, q8, k_lens, [0] * B, 16, 4)       # nuggets only
    _check(D, 724, q8, [0] * B, [max(m, 1) for m in m_lens], 16, 4)  # local rows only


def test_more_than_32_vectors_take_several_passes(D):
    # rows x heads beyond one tile: the rows are dealt out to up to four launches, each with its own causal limits
    rng = np.random.default_rng(13)
    B = 40
    q_lens = [int(v) for v in rng.integers(0, 16, B)]
    q_lens[0], q_lens[1], q_lens[2] = 15, 0, 4        # all passes, none, exactly the first
    k_lens = [int(v) for v in rng.integers(0, 120, B)]
    m_lens = [int(v) for v in rng.integers(0, 40, B)]
    m_lens[0] = 7                                       # fewer local rows than query rows: early rows see none
    _check(D, 780, q_lens, k_lens, m_lens, 64, 8)      # 8 heads x 15 rows: four passes of 4 rows
    _check(D, 781, q_lens, k_lens, m_lens, 16, 4)      # 4 heads x 15 rows: two passes of 8 rows
    _check(D, 782, [min(q, 8) for q in q_lens], k_lens, m_lens, 32, 2, d_h=64)   # 16 heads x 8 rows: four passes of 2
    _check(D, 783, [min(q, 6) for q in q_lens], k_lens, m_lens, 20, 4)           # 5 heads x 6 rows: one pass of 6
    # few sequences and long caches: every pass splits the keys over workgroups, all on one workspace
    _check(D, 784, [15, 9], [3277, 1500], [1089, 1025], 64, 8)
    _check(D, 785, [7, 7, 2], [2000, 37, 900], [300, 700, 31], 40, 8, layout=1)


def test_heads_of_64_channels(D):
    # the same kernel with half the channels: other tile sizes, LDS swizzles and fragment counts
    rng = np.random.default_rng(12)
    B = 70
    k_lens = [int(v) for v in rng.integers(0, 150, B)]
    m_lens = [int(v) for v in rng.integers(1, 70, B)]
    k_lens[3], m_lens[3] = 0, 1
    k_lens[4], m_lens[4] = 31, 33
    _check(D, 770, [1] * B, k_lens, m_lens, 32, 8, d_h=64)
    _check(D, 771, [1] * B, k_lens, m_lens, 40, 8, d_h=64, layout=1)
    q_lens = [int(v) for v in rng.integers(0, 5, B)]
    _check(D, 772, q_lens, k_lens, m_lens, 32, 4, d_h=64)
    _check(D, 773, [int(v) for v in rng.integers(1, 9, B)], k_lens, m_lens, 16, 16, d_h=64)
    # split over workgroups (two and four wavefronts each)
    _check(D, 774, [1, 1], [3277, 1500], [1089, 1025], 64, 8, d_h=64)
    _check(D, 775, [1] * 5, [205, 410, 333, 1, 0], [257, 257, 40, 3, 5], 64, 8, d_h=64)
    _check(D, 776, [2] * 3, [2000, 37, 900], [300, 700, 31], 40, 8, d_h=64)


def test_softmax_scale_and_large_logits(D):
    # a scale that makes single keys dominate: the running maximum moves from tile to tile
    _check(D, 730, [1] * 40, [100] * 40, [64] * 40, 32, 8, scale=1.5)


def test_run_to_run_deterministic(D):
    host, t = make_attention_case(740, [1, 1], [3277, 1500], [1089, 1025], 64, 8, 128, BF, dev())
    need = D.dodo_nugget_attention_workspace_bytes_grouped(2, 64, 8, 128, 1, 3277, 1089, D.BF16)
    ws = torch.zeros(need, dtype=torch.uint8, device=dev())
    outs = []
    for _ in range(4):
        O, lse = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"],
                                         t["cu_local"], 1, 3277, 1089, default_scale(128), 0, want_lse=True, ws=ws)
        outs.append((O.clone(), lse.clone()))
    for O, lse in outs[1:]:
        assert torch.equal(O, outs[0][0]) and torch.equal(lse, outs[0][1])
    n_slots = need // ((128 + 3) * 4)
    assert not bool(ws.view(torch.int32)[-n_slots:].any())  # the flags of the largest layout are left cleared


def test_workspace_needs_no_zero_fill_and_is_reusable(D):
    # bytes that are not the "ready" value are as good as zeros, and a workspace serves call after call
    q, k, m, H, H_kv = [1, 1], [3000, 1234], [700, 1025], 64, 8
    need = D.dodo_nugget_attention_workspace_bytes_grouped(2, H, H_kv, 128, 1, max(k), max(m), D.BF16)
    assert need > D.dodo_nugget_attention_workspace_bytes(2, H, 128, 1, max(k), max(m), D.BF16)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=dev())
    for seed in (790, 791, 792):
        host, t = make_attention_case(seed, q, k, m, H, H_kv, 128, BF, dev())
        O_ref, lse_ref = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"],
                                          host["cu_nuggets"], host["cu_local"], default_scale(128))
        O, lse = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"],
                                         t["cu_local"], 1, max(k), max(m), default_scale(128), 0, want_lse=True, ws=ws)
        check_attention(O, O_ref, BF)
        check_lse(lse, lse_ref, BF)


def test_caches_with_room_to_grow_and_segment_ranges(D):
    # start + length ranges for the nuggets (cached form) and for both kinds of rows (segment form)
    rng = np.random.default_rng(11)
    B, H, H_kv, cap = 40, 32, 8, 96
    lens = [int(v) for v in rng.integers(0, cap, B)]
    m_lens = [int(v) for v in rng.integers(1, 50, B)]
    mk = lambda tid, n, h: W.normal(750, tid, (n, h, 128), 1.0, BF, "cpu")
    Q, Kc, Vc = mk(0, B, H), mk(1, B * cap, H_kv), mk(2, B * cap, H_kv)
    Kl, Vl = mk(3, sum(m_lens), H_kv), mk(4, sum(m_lens), H_kv)
    start = np.arange(B, dtype=np.int32) * cap
    cu_q, cu_l = W.cumulative([1] * B), W.cumulative(m_lens)
    scale = default_scale(128)
    # oracle on the packed equivalent
    rows = np.concatenate([np.arange(s, s + n) for s, n in zip(start, lens)]).astype(np.int64)
    Kn_p, Vn_p = Kc[torch.from_numpy(rows)], Vc[torch.from_numpy(rows)]
    O_ref, lse_ref = oracle.attention(W.to_numpy(Q), W.to_numpy(Kn_p), W.to_numpy(Vn_p), W.to_numpy(Kl), W.to_numpy(Vl),
                                      W.to_numpy(cu_q), oracle.cu_from_lengths(lens), W.to_numpy(cu_l), scale)
    d = dev()
    O, lse = D.dodo_nugget_attention_cached(Q.to(d), Kc.to(d), Vc.to(d), Kl.to(d), Vl.to(d), cu_q.to(d),
                                            torch.from_numpy(start).to(d), torch.tensor(lens, dtype=torch.int32, device=d),
                                            cu_l.to(d), 1, cap, max(m_lens), scale, want_lse=True)
    check_attention(O, O_ref, BF)
    check_lse(lse, lse_ref, BF)
    loc_start = W.to_numpy(cu_l)[:-1].astype(np.int32)
    O2, lse2 = D.dodo_nugget_attention_segments(Q.to(d), Kc.to(d), Vc.to(d), Kl.to(d), Vl.to(d), cu_q.to(d),
                                                torch.from_numpy(start).to(d),
                                                torch.tensor(lens, dtype=torch.int32, device=d),
                                                torch.from_numpy(loc_start).to(d),
                                                torch.tensor(m_lens, dtype=torch.int32, device=d), 1, cap, max(m_lens),
                                                scale, want_lse=True)
    check_attention(O2, O_ref, BF)
    check_lse(lse2, lse_ref, BF)


def test_entry_point_that_allocates_nothing(D):
    # the library's own buffer bounds the number of splits; same results to the tolerance, twice in a row, the
    # second call smaller
    for seed, q, k, m, H, H_kv in ((760, [1, 1], [3277, 1500], [1089, 1025], 64, 8), (761, [1], [1200], [300], 32, 8),
                                   (762, [1] * 70, [90] * 70, [33] * 70, 32, 8)):
        host, t = make_attention_case(seed, q, k, m, H, H_kv, 128, BF, dev())
        scale = default_scale(128)
        O_ref, lse_ref = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"],
                                          host["cu_nuggets"], host["cu_local"], scale)
        O, lse = nan_outputs(t["Q"], H)
        D.dodo_nugget_attention_noalloc(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"],
                                        t["cu_local"], max(q), max(k), max(m), scale, D.TOKEN_MAJOR, O, lse)
        check_attention(O, O_ref, BF)
        check_lse(lse, lse_ref, BF)


# Tiles 16 (up to 16 query vectors per KV head) and 32 wide, at 4, 16, 17 and 32 vectors: nuggets and local rows at the edges of
# the 32-key tiles and of the wavefronts' turns, and the weights' precision -- in two bf16 parts they leave O the error of its own
# rounding (2^-9 relative: 2-norm 1.66e-3), where weights rounded to bf16 would show 2.1e-3 or more.
@pytest.mark.parametrize("G,q", [(4, 1), (16, 1), (17, 1), (32, 1), (1, 4), (1, 15), (2, 8), (3, 10)])
@pytest.mark.parametrize("d_h", [64, 128])
def test_widths_of_the_tiles(D, G, q, d_h):
    B, H_kv = 34, 8
    edges = [0, 1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 160, 255, 300]
    k_lens = [edges[i % 14] for i in range(B)]
    m_lens = [max(q, edges[(5 * i + 3) % 14]) for i in range(B)]
    host, t = make_attention_case(800 + G, [q] * B, k_lens, m_lens, G * H_kv, H_kv, d_h, BF, dev())
    scale = default_scale(d_h)
    want, lse_want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"], host["cu_nuggets"],
                                      host["cu_local"], scale)
    O, lse = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], q, max(k_lens),
                                     max(m_lens), scale, want_lse=True)
    check_attention(O, want, BF)
    check_lse(lse, lse_want, BF)
    err = O.float().cpu().double().numpy().reshape(want.shape) - want
    assert np.linalg.norm(err) <= 1.9e-3 * np.linalg.norm(want)


# An infinity in a visible row of V is the row's result, as with a weight in one piece; other rows and channels are not touched.
def test_infinite_value_in_a_visible_row(D):
    B, H, H_kv, d_h = 40, 32, 8, 128
    host, t = make_attention_case(830, [1] * B, [90] * B, [40] * B, H, H_kv, d_h, BF, dev())
    clean = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], 1, 90, 40)[0]
    t["Vn"][90 * 3 + 50, 2, 7] = float("inf")
    t["Vl"][40 * 5 + 11, 0, 64] = float("-inf")
    O = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], 1, 90, 40)[0]
    want = clean.clone()
    want[3, 8:12, 7] = float("inf")
    want[5, 0:4, 64] = float("-inf")
    assert torch.equal(O, want)


# A small batch with one query row each goes from the split-K kernel to this one where its vectors and rows are many (128 Ki of their
# products) and this one is the faster.  Both sides have the same precision.
@pytest.mark.parametrize("k", [200, 480, 500, 1500])
def test_small_batches_on_either_side_of_the_line(D, k):
    B, H, H_kv, d_h = 4, 64, 8, 128
    k_lens, m_lens = [k - 7 * b for b in range(B)], [10 + b for b in range(B)]
    host, t = make_attention_case(840, [1] * B, k_lens, m_lens, H, H_kv, d_h, BF, dev())
    want, lse_want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"], host["cu_nuggets"],
                                      host["cu_local"], default_scale(d_h))
    O, lse = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], 1, max(k_lens),
                                     max(m_lens), want_lse=True)
    check_lse(lse, lse_want, BF)
    err = O.float().cpu().double().numpy().reshape(want.shape) - want
    assert np.linalg.norm(err) <= 1.9e-3 * np.linalg.norm(want)


# Which kernel takes a small batch with one query row each: this one where the split-K kernel's workgroups are more than the compute units
# or its shares long, that one where its workgroups come out even or this one would merge many splits.
@pytest.mark.parametrize("B,rows,H,H_kv,d_h,kernel", [
    (4, 357, 64, 8, 128, "splitk"), (6, 357, 64, 8, 128, "group"), (4, 667, 64, 8, 128, "splitk"), (5, 454, 64, 8, 128, "group"),
    (2, 1887, 40, 8, 128, "splitk"), (2, 1099, 64, 8, 128, "group"), (7, 687, 32, 8, 128, "splitk"), (2, 3168, 32, 4, 64, "splitk"),
    (9, 1508, 16, 2, 64, "group"),
])
def test_kernel_of_a_small_batch(D, B, rows, H, H_kv, d_h, kernel):
    k, m = rows - 20, 20
    host, t = make_attention_case(850, [1] * B, [k] * B, [m] * B, H, H_kv, d_h, BF, dev())
    out = []
    names = kernel_names(lambda: out.extend(D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"],
                                                                    1, k, m, want_lse=True)), "attention_kernel")
    assert len(names) == 1 and kernel + "_attention_kernel" in names[0], names
    want, lse_want = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"], host["cu_nuggets"],
                                      host["cu_local"], default_scale(d_h))
    check_attention(out[0], want, BF)
    check_lse(out[1], lse_want, BF)


# Small batches that come here from the split-K kernel keep weights of 24 bits.  O is then off by a few 1e-7 of itself before it is rounded
# to bf16, whose neighbours are 2^-8 to 2^-7 apart: about one value in 5000 rounds to another neighbour than the 64-bit result (1.2e-4 to
# 3.3e-4 in the split-K kernel too); with weights of 16 bits, off by up to 2^-17, it is one in 250.
@pytest.mark.parametrize("B,k,m,H,H_kv,d_h", [(6, 300, 57, 64, 8, 128), (13, 200, 40, 64, 8, 128), (2, 1000, 99, 64, 8, 128), (9, 1450, 50, 16, 2, 64),
                                              (10, 500, 5, 32, 4, 64)])
def test_weights_of_a_small_batch_are_whole(D, B, k, m, H, H_kv, d_h):
    host, t = make_attention_case(860, [1] * B, [k] * B, [m] * B, H, H_kv, d_h, BF, dev())
    want, _ = oracle.attention(host["Q"], host["Kn"], host["Vn"], host["Kl"], host["Vl"], host["cu_q"], host["cu_nuggets"],
                               host["cu_local"], default_scale(d_h))
    O = D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], 1, k, m)[0]
    check_attention(O, want, BF)
    other = (O.cpu() != torch.from_numpy(want).to(BF).reshape(O.shape)).double().mean().item()
    assert other <= 1e-3, other


# An infinity in V with weights in three parts, one of them far below the others.
def test_infinite_value_in_a_visible_row_of_a_small_batch(D):
    B, k, m, H, H_kv, d_h = 6, 300, 57, 64, 8, 128
    host, t = make_attention_case(861, [1] * B, [k] * B, [m] * B, H, H_kv, d_h, BF, dev())
    t["Kn"][k * 3 + 50, 2] = -8 * t["Q"][3, 2 * 8]  # a logit far below the rest, for the first of the heads
    run = lambda: D.dodo_nugget_attention(t["Q"], t["Kn"], t["Vn"], t["Kl"], t["Vl"], t["cu_q"], t["cu_nuggets"], t["cu_local"], 1, k, m)[0]
    want = run()
    t["Vn"][k * 3 + 50, 2, 7] = float("inf")
    t["Vl"][m * 5 + 11, 0, 64] = float("-inf")
    O = run()
    want[3, 17:24, 7] = float("inf")
    want[5, 0:8, 64] = float("-inf")
    O[3, 16, 7] = want[3, 16, 7]  # (its weight may have underflowed to zero: 0 x inf)
    assert torch.equal(O, want)


# Query rows further than 2^31 bytes from the launch's first one (the heads of a row take 157 MB): the last one has its own result.
def test_query_rows_far_apart(D):
    q, G, H_kv, d_h = 15, 2, 307200, 128
    g = torch.Generator(device=dev()).manual_seed(5)
    r = lambda n, h: torch.randn((n, h, d_h), generator=g, dtype=BF, device=dev())
    Q, Kl, Vl = r(q, G * H_kv), r(q, H_kv), r(q, H_kv)
    cu = W.cumulative([q], dev())
    none = torch.empty((0, H_kv, d_h), dtype=BF, device=dev())
    O = D.dodo_nugget_attention(Q, none, none, Kl, Vl, cu, W.cumulative([0], dev()), cu, q, 0, q, ws=torch.zeros(16, dtype=torch.uint8, device=dev()))[0]
    for h0 in (0, H_kv - 500):
        K, V = Kl[:, h0:h0 + 500].float(), Vl[:, h0:h0 + 500].float()
        last = Q[q - 1].view(H_kv, G, d_h)[h0:h0 + 500].float()
        P = torch.softmax((K.unsqueeze(2) * last).sum(-1) * default_scale(d_h), 0)  # [key, K/V head, head of the group]
        want = (P.unsqueeze(-1) * V.unsqueeze(2)).sum(0)
        got = O[q - 1].view(H_kv, G, d_h)[h0:h0 + 500].float()
        assert (got - want).abs().max().item() <= 2e-2
