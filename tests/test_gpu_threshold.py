"""GPU parity of the autoregressive mode's selection (Sec. 2.4, Eq. 8) against the oracle: threshold
calibration, threshold selection, streaming append and attention over caches with room to grow."""
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


def _cu(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


@pytest.mark.parametrize("n,num,den,kind", [
    (1, 1, 10, "gauss"), (37, 1, 10, "gauss"), (5000, 1, 10, "gauss"), (100000, 1, 20, "gauss"),
    (70000, 1, 10, "quant"), (4096, 1, 1, "gauss"), (3000, 3, 4, "specials"),
])
def test_threshold_from_sample_is_bit_exact(D, n, num, den, kind):
    s = W.normal(500 + n, 0, (n,), 1.0, torch.float32)
    if kind == "quant":
        s = W.quantise16(s)
    if kind == "specials":
        s[::7] = float("nan")
        s[1::11] = -0.0
        s[2::13] = float("inf")
        s[3::17] = float("-inf")
    want = np.float32(oracle.threshold_from_sample(s.numpy(), num, den))
    got = D.dodo_threshold_from_sample(s.to(dev()), num, den).cpu().numpy()[0]
    assert got.tobytes() == want.tobytes(), (got, want)


@pytest.mark.parametrize("n,num,den,kind", [(40000, 1, 10, "gauss"), (410000, 1, 20, "gauss"), (65536, 1, 10, "quant"),
                                            (100001, 1, 10, "specials"), (33000, 9, 10, "specials")])
def test_threshold_from_large_samples_over_many_workgroups(D, n, num, den, kind):
    # beyond 16384 scores, given the workspace, one launch per radix pass over many workgroups: the same bits as
    # the oracle, and as the one-workgroup form (no workspace)
    assert D.dodo_threshold_from_sample_workspace_bytes(n) > 0
    s = W.normal(600 + n, 0, (n,), 1.0, torch.float32)
    if kind == "quant":
        s = W.quantise16(s)
    if kind == "specials":
        s[::7] = float("nan")
        s[1::11] = -0.0
        s[2::13] = float("inf")
        s[3::17] = float("-inf")
    want = np.float32(oracle.threshold_from_sample(s.numpy(), num, den))
    sd = s.to(dev())
    ws = torch.full((D.dodo_threshold_from_sample_workspace_bytes(n),), 0xAB, dtype=torch.uint8, device=dev())
    got = D.dodo_threshold_from_sample(sd, num, den, ws=ws).cpu().numpy()[0]
    assert got.tobytes() == want.tobytes(), (got, want)
    one = D.dodo_threshold_from_sample(sd, num, den, ws=torch.zeros(16, dtype=torch.uint8, device=dev())).cpu().numpy()[0]
    assert one.tobytes() == want.tobytes()


# sizes at the edges of the forms of the kernel (scores in registers, in LDS, in memory)
@pytest.mark.parametrize("n", [2, 64, 4096, 4097, 15000, 33792, 33793, 34816, 34817])
@pytest.mark.parametrize("kind", ["gauss", "ties", "exponents", "rising", "specials", "constant"])
def test_threshold_from_sample_in_one_workgroup(D, n, kind):
    g = np.random.default_rng(n)
    s = g.standard_normal(n).astype(np.float32)
    if kind == "ties":
        s = W.quantise16(torch.from_numpy(s)).numpy()
    elif kind == "exponents":
        s = (s * np.exp(20 * g.standard_normal(n))).astype(np.float32)
    elif kind == "rising":
        s = np.arange(n, dtype=np.float32)
    elif kind == "specials":
        s[::3], s[1::11], s[2::13], s[4::17] = np.nan, np.inf, -np.inf, -0.0
    elif kind == "constant":
        s[:] = -2.5
    for num, den in ((1, 10), (9, 10), (1, n)):
        want = np.float32(oracle.threshold_from_sample(s, num, den))
        got = D.dodo_threshold_from_sample(torch.from_numpy(s).to(dev()), num, den).cpu().numpy()[0]
        assert got.tobytes() == want.tobytes(), (num, den, got, want)


def test_threshold_from_sample_when_the_rank_falls_on_nan(D):
    s = torch.tensor([float("nan"), 5.0, float("nan"), 1.0, -0.0, 7.0], dtype=torch.float32)
    for num, den in [(1, 3), (1, 2), (4, 6)]:
        want = np.float32(oracle.threshold_from_sample(s.numpy(), num, den))
        got = D.dodo_threshold_from_sample(s.to(dev()), num, den).cpu().numpy()[0]
        assert got.tobytes() == want.tobytes()


@pytest.mark.parametrize("lens", [[4096] * 8, [200, 0, 300, 1, 4097, 33], [32768, 32768], [5]])
def test_select_threshold_matches_oracle(D, lens):
    N = sum(lens)
    s = W.normal(600 + len(lens), 0, (N,), 1.0, torch.float32)
    s[::97] = float("nan")
    lam = np.float32(0.4)
    s[5 % N] = float(lam)  # a score equal to the threshold is dropped
    counts_ref, cu_ref, idx_ref = oracle.select_threshold_indices(s.numpy(), _cu(lens), float(lam))
    counts, cu_k, idx = D.dodo_select_threshold(s.to(dev()), torch.from_numpy(_cu(lens)).to(dev()),
                                                torch.tensor([lam], dtype=torch.float32, device=dev()))
    assert np.array_equal(counts.cpu().numpy(), counts_ref)
    assert np.array_equal(cu_k.cpu().numpy(), cu_ref)
    assert np.array_equal(idx.cpu().numpy()[: cu_ref[-1]], idx_ref)


def test_calibrate_select_gather_chain_without_host_readback(D):
    # Lambda stays on the device; gather takes an upper bound of the nugget count
    lens, H_kv, d_h = [700, 1300, 64], 2, 64
    N = sum(lens)
    s = W.normal(610, 0, (N,), 1.0, torch.float32)
    K = W.normal(610, 1, (N, H_kv, d_h), 1.0, torch.bfloat16, "cpu")
    V = W.normal(610, 2, (N, H_kv, d_h), 1.0, torch.bfloat16, "cpu")
    cu = _cu(lens)
    lam_ref = oracle.threshold_from_sample(s.numpy(), 1, 10)
    counts_ref, cu_ref, idx_ref = oracle.select_threshold_indices(s.numpy(), cu, lam_ref)
    Kn_ref, Vn_ref = oracle.gather(W.to_numpy(K), W.to_numpy(V), idx_ref, cu, cu_ref)
    sd, cud = s.to(dev()), torch.from_numpy(cu).to(dev())
    lam = D.dodo_threshold_from_sample(sd, 1, 10)
    counts, cu_k, idx = D.dodo_select_threshold(sd, cud, lam)
    bound = N  # no read-back: every token could have been kept
    Kn = torch.zeros((bound, H_kv, d_h), dtype=torch.bfloat16, device=dev())
    Vn = torch.zeros_like(Kn)
    D.dodo_gather_nuggets(K.to(dev()), V.to(dev()), idx, cud, cu_k, bound, D.TOKEN_MAJOR, Kn, Vn)
    kt = int(cu_ref[-1])
    assert kt == int(counts_ref.sum()) > 0
    assert np.array_equal(W.to_numpy(Kn.cpu())[:kt], Kn_ref) and np.array_equal(W.to_numpy(Vn.cpu())[:kt], Vn_ref)
    assert not W.to_numpy(Kn.cpu())[kt:].any()  # rows past the end are left untouched


@pytest.mark.parametrize("dtype,H,H_kv,d_h", [(torch.bfloat16, 8, 8, 128), (torch.float32, 4, 2, 64)])
def test_decode_loop_append_then_attend(D, dtype, H, H_kv, d_h):
    """Autoregressive mode end to end: at every step one token per sequence leaves the window and is
    appended to its cache if kept; the new token then attends over [its nuggets ; the window]."""
    B, steps, cap, tau = 3, 40, 24, 16
    lam_v = np.float32(-0.2)  # keeps a good half, so that the cache of some sequence fills up
    lam = torch.tensor([lam_v], dtype=torch.float32, device=dev())
    Kn = torch.zeros((B, cap, H_kv, d_h), dtype=dtype, device=dev())
    Vn = torch.zeros_like(Kn)
    counts = torch.zeros(B, dtype=torch.int32, device=dev())
    dropped = torch.zeros(1, dtype=torch.int32, device=dev())
    Kn_ref = np.zeros((B, cap, H_kv, d_h), dtype=W.to_numpy(Kn.cpu()).dtype)
    Vn_ref = np.zeros_like(Kn_ref)
    counts_ref = np.zeros(B, dtype=np.int32)
    dropped_ref = 0
    start = (torch.arange(B, dtype=torch.int32) * cap).to(dev())
    cu_q = torch.from_numpy(_cu([1] * B)).to(dev())
    cu_l = torch.from_numpy(_cu([tau + 1] * B)).to(dev())
    scale = default_scale(d_h)
    for t in range(steps):
        sc = W.normal(700, 10 + t, (B,), 1.0, torch.float32)
        Kr = W.normal(700, 1000 + t, (B, H_kv, d_h), 1.0, dtype, "cpu")
        Vr = W.normal(700, 2000 + t, (B, H_kv, d_h), 1.0, dtype, "cpu")
        D.dodo_stream_append(sc.to(dev()), lam, Kr.to(dev()), Vr.to(dev()), counts, Kn, Vn, dropped)
        dropped_ref += oracle.stream_append(sc.numpy(), float(lam_v), W.to_numpy(Kr), W.to_numpy(Vr), counts_ref, Kn_ref,
                                            Vn_ref)
        if t % 13 == 12 or t == steps - 1:
            assert np.array_equal(counts.cpu().numpy(), counts_ref)
            assert np.array_equal(W.to_numpy(Kn.cpu()), Kn_ref) and np.array_equal(W.to_numpy(Vn.cpu()), Vn_ref)
            # the new token's attention: oracle on the packed form of the caches
            Q = W.normal(700, 3000 + t, (B, H, d_h), 1.0, dtype, "cpu")
            Kl = W.normal(700, 4000 + t, (B * (tau + 1), H_kv, d_h), 1.0, dtype, "cpu")
            Vl = W.normal(700, 5000 + t, (B * (tau + 1), H_kv, d_h), 1.0, dtype, "cpu")
            packK = np.concatenate([Kn_ref[b, :counts_ref[b]] for b in range(B)])
            packV = np.concatenate([Vn_ref[b, :counts_ref[b]] for b in range(B)])
            O_ref, lse_ref = oracle.attention(W.to_numpy(Q), packK, packV, W.to_numpy(Kl), W.to_numpy(Vl), _cu([1] * B),
                                              _cu(counts_ref), _cu([tau + 1] * B), scale)
            O, lse = D.dodo_nugget_attention_cached(Q.to(dev()), Kn.view(B * cap, H_kv, d_h), Vn.view(B * cap, H_kv, d_h),
                                                    Kl.to(dev()), Vl.to(dev()), cu_q, start, counts, cu_l, 1, cap, tau + 1,
                                                    scale, want_lse=True)
            check_attention(O, O_ref, dtype)
            check_lse(lse, lse_ref, dtype)
    assert int(dropped.cpu()[0]) == dropped_ref > 0 and counts_ref.max() == cap


def test_cached_attention_block_kernel_reads_start_and_length(D):
    # query blocks (MFMA kernel) over caches with gaps between the sequences
    B, H, d_h, cap, q, m = 2, 2, 128, 300, 160, 200
    lens = [257, 31]
    Kc = W.normal(710, 1, (B * cap, H, d_h), 1.0, torch.bfloat16, "cpu")
    Vc = W.normal(710, 2, (B * cap, H, d_h), 1.0, torch.bfloat16, "cpu")
    Q = W.normal(710, 3, (B * q, H, d_h), 1.0, torch.bfloat16, "cpu")
    Kl = W.normal(710, 4, (B * m, H, d_h), 1.0, torch.bfloat16, "cpu")
    Vl = W.normal(710, 5, (B * m, H, d_h), 1.0, torch.bfloat16, "cpu")
    Kc_h, Vc_h = W.to_numpy(Kc), W.to_numpy(Vc)
    packK = np.concatenate([Kc_h[b * cap: b * cap + lens[b]] for b in range(B)])
    packV = np.concatenate([Vc_h[b * cap: b * cap + lens[b]] for b in range(B)])
    scale = default_scale(d_h)
    O_ref, lse_ref = oracle.attention(W.to_numpy(Q), packK, packV, W.to_numpy(Kl), W.to_numpy(Vl), _cu([q] * B), _cu(lens),
                                      _cu([m] * B), scale)
    to = lambda a: a.to(dev())
    O, lse = D.dodo_nugget_attention_cached(to(Q), to(Kc), to(Vc), to(Kl), to(Vl), to(torch.from_numpy(_cu([q] * B))),
                                            to(torch.tensor([0, cap], dtype=torch.int32)),
                                            to(torch.tensor(lens, dtype=torch.int32)),
                                            to(torch.from_numpy(_cu([m] * B))), q, cap, m, scale, want_lse=True)
    check_attention(O, O_ref, torch.bfloat16)
    check_lse(lse, lse_ref, torch.bfloat16)
