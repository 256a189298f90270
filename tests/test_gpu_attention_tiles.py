"""GPU parity of the query-block kernels where a tile, a mask or the dealing of heads to the XCDs begins or ends."""
import pytest
import torch

import oracle
from gpu_util import check_attention, check_lse, default_scale, dev, make_attention_case

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
