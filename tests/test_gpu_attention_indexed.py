"""GPU parity: dodo_nugget_attention_indexed (nuggets read in place through the index list) against the
oracle, and bit for bit against the HIP gather followed by the HIP attention."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import check_attention, check_lse, default_scale, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    import paper_2310_02409_amd as D
    return D


def _case(seed, n_lens, k_lens, q_lens, m_lens, H, H_kv, d_h, dtype, pad_heads=0):
    N, Sq, Sm = sum(n_lens), sum(q_lens), sum(m_lens)
    mk = lambda tid, n, h: W.normal(seed, tid, (n, h, d_h), 1.0, dtype, "cpu")
    K, V = mk(0, N, H_kv + pad_heads), mk(1, N, H_kv + pad_heads)
    t = dict(Q=mk(2, Sq, H), Kl=mk(3, Sm, H_kv), Vl=mk(4, Sm, H_kv))
    s = W.normal(seed, 5, (N,), 1.0, torch.float32).numpy()
    cu_s, cu_k = oracle.cu_from_lengths(n_lens), oracle.cu_from_lengths(k_lens)
    idx = oracle.select_topk(s, cu_s, cu_k)
    cu = dict(cu_s=cu_s, cu_k=cu_k, cu_q=oracle.cu_from_lengths(q_lens), cu_l=oracle.cu_from_lengths(m_lens), idx=idx)
    host = {k: W.to_numpy(v) for k, v in t.items()}
    host.update(K=W.to_numpy(K[:, :H_kv].contiguous()), V=W.to_numpy(V[:, :H_kv].contiguous()), **cu)
    devt = {k: v.to(dev()) for k, v in t.items()}
    devt.update({k: torch.from_numpy(v).to(dev()) for k, v in cu.items()})
    devt.update(K=K.to(dev())[:, :H_kv], V=V.to(dev())[:, :H_kv])  # views: token stride (H_kv + pad_heads) d_h
    return host, devt


def _check(D, seed, n_lens, k_lens, q_lens, m_lens, H, H_kv, d_h, dtype, pad_heads=0):
    host, d = _case(seed, n_lens, k_lens, q_lens, m_lens, H, H_kv, d_h, dtype, pad_heads)
    scale = default_scale(d_h)
    O_ref, lse_ref = oracle.attention_indexed(host["Q"], host["K"], host["V"], host["idx"], host["cu_s"], host["Kl"],
                                              host["Vl"], host["cu_q"], host["cu_k"], host["cu_l"], scale)
    O, lse = D.dodo_nugget_attention_indexed(d["Q"], d["K"], d["V"], d["idx"], d["cu_s"], d["Kl"], d["Vl"], d["cu_q"],
                                             d["cu_k"], d["cu_l"], max(q_lens), max(k_lens), max(m_lens), max(n_lens),
                                             scale, want_lse=True)
    check_attention(O, O_ref, dtype)
    check_lse(lse, lse_ref, dtype)
    # the same arithmetic in the same order as the packed form: identical bits
    Kn, Vn = D.dodo_gather_nuggets(d["K"].contiguous(), d["V"].contiguous(), d["idx"], d["cu_s"], d["cu_k"],
                                   int(host["cu_k"][-1]))
    O2, lse2 = D.dodo_nugget_attention(d["Q"], Kn, Vn, d["Kl"], d["Vl"], d["cu_q"], d["cu_k"], d["cu_l"], max(q_lens),
                                       max(k_lens), max(m_lens), scale, want_lse=True)
    assert torch.equal(O, O2) and torch.equal(lse, lse2)


@pytest.mark.parametrize("dtype,H,H_kv,d_h", [(torch.float32, 4, 4, 64), (torch.bfloat16, 8, 2, 128),
                                              (torch.bfloat16, 4, 4, 64), (torch.float32, 4, 2, 128)])
def test_decode_ragged(D, dtype, H, H_kv, d_h):
    n_lens = [2050, 4100, 999, 1, 7]
    k_lens = [205, 410, 333, 1, 0]
    _check(D, 500, n_lens, k_lens, [1] * 5, [257, 257, 40, 3, 5], H, H_kv, d_h, dtype)


def test_decode_split_k_and_padded_token_stride(D):
    _check(D, 501, [9000, 4000], [3277, 1500], [1, 1], [1089, 1025], 2, 2, 128, torch.bfloat16, pad_heads=1)


@pytest.mark.parametrize("n_lens,k_lens,q_lens,m_lens,H,H_kv", [
    ([700], [64], [128], [128], 2, 2),                                       # 4-wavefront kernel
    ([4096, 4096], [410, 410], [512, 512], [640, 640], 4, 4),                # workload-2 shape, fewer heads
    ([130, 2000, 5, 800], [13, 200, 0, 77], [100, 37, 256, 16], [150, 37, 300, 16], 4, 2),  # ragged, GQA, partial tiles
    ([1030], [103], [300], [300], 3, 1),                                     # compressor mode
    ([5000, 90], [500, 9], [64, 200], [0, 100], 2, 2),                       # nuggets only; short local buffer
])
def test_block_kernel_bf16(D, n_lens, k_lens, q_lens, m_lens, H, H_kv):
    _check(D, 502, n_lens, k_lens, q_lens, m_lens, H, H_kv, 128, torch.bfloat16)
    _check(D, 505, n_lens, k_lens, q_lens, m_lens, H, H_kv, 64, torch.bfloat16)


# Blocks of 64 rows whose wavefronts take half of a tile's keys each, more of them than compute units: two workgroups share a unit's LDS,
# the stages, index lists and merges of both.
@pytest.mark.parametrize("q,k,d_h", [(64, 150, 128), (33, 65, 128), (64, 200, 64)])
def test_halves_of_a_tile_through_the_index_list(D, q, k, d_h):
    B, H = 20, 16
    k_lens, q_lens = [k - b % 5 for b in range(B)], [q - b % 3 for b in range(B)]
    _check(D, 506, [3 * k] * B, k_lens, q_lens, [n + 20 - b % 40 for b, n in enumerate(q_lens)], H, H, d_h, torch.bfloat16)


def test_block_kernel_padded_token_stride_and_long_index_list(D):
    _check(D, 503, [20000], [4000], [256], [256], 2, 1, 128, torch.bfloat16, pad_heads=1)


# Lists of more entries than two workgroups of a compute unit have room for: the plan, and with it the bits, of the packed form, whether
# the keys are shared out, halves of tiles, whole tiles of grouped heads, or the 8-wavefront kernel's
@pytest.mark.parametrize("B,q,k,H,H_kv,d_h,room", [(1, 160, 4500, 2, 2, 128, True), (1, 160, 4500, 2, 2, 128, False), (1, 200, 7680, 4, 4, 64, True),
                                                   (11, 160, 4200, 32, 8, 128, False), (2, 300, 4097, 32, 32, 128, False)])
def test_long_index_lists_have_the_packed_plan(D, B, q, k, H, H_kv, d_h, room):
    g = torch.Generator().manual_seed(k + q)
    r = lambda *s: torch.randn(s, generator=g).to(torch.bfloat16).to(dev())
    n, m, cu = k + 300, q + 40, lambda v: W.cumulative([v] * B, dev())
    K, V, Q, Kl, Vl = r(B * n, H_kv, d_h), r(B * n, H_kv, d_h), r(B * q, H, d_h), r(B * m, H_kv, d_h), r(B * m, H_kv, d_h)
    idx = torch.cat([torch.randperm(n, generator=g)[:k].sort().values for _ in range(B)]).int().to(dev())
    Kn, Vn = D.dodo_gather_nuggets(K, V, idx, cu(n), cu(k), B * k)
    size = D.dodo_nugget_attention_workspace_bytes(B, H, d_h, q, k, m, D.BF16) if room else 16
    ws = torch.zeros(size, dtype=torch.uint8, device=dev())
    a = (Kl, Vl, cu(q), cu(k), cu(m), q, k, m)
    O, lse = D.dodo_nugget_attention(Q, Kn, Vn, *a, want_lse=True, ws=ws)
    Oi, lse_i = D.dodo_nugget_attention_indexed(Q, K, V, idx, cu(n), *a, n, want_lse=True, ws=ws)
    assert bool(torch.isfinite(O.float()).all()) and torch.equal(O, Oi) and torch.equal(lse, lse_i)


def test_limits_are_reported(D):
    # more nuggets in a sequence than the query-block kernel keeps in LDS: refused, not wrong
    host, d = _case(504, [9000], [7681], [256], [256], 1, 1, 128, torch.bfloat16)
    with pytest.raises(D.DodoError) as e:
        D.dodo_nugget_attention_indexed(d["Q"], d["K"], d["V"], d["idx"], d["cu_s"], d["Kl"], d["Vl"], d["cu_q"],
                                        d["cu_k"], d["cu_l"], 256, 7681, 256, 9000)
    assert e.value.status == -2
    host, d = _case(504, [9000], [4097], [128], [128], 1, 1, 128, torch.bfloat16)  # (up to 128 query rows)
    with pytest.raises(D.DodoError) as e:
        D.dodo_nugget_attention_indexed(d["Q"], d["K"], d["V"], d["idx"], d["cu_s"], d["Kl"], d["Vl"], d["cu_q"],
                                        d["cu_k"], d["cu_l"], 128, 4097, 128, 9000)
    assert e.value.status == -2
