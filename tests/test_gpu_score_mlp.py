"""GPU parity of dodo_score_mlp (2-layer scorer of App. B) against the oracle.

Tolerance: |s - s_ref| <= 1e-4 (1 + |s_ref|).  bf16 products are exact in fp32; the d-term sums inside the
MFMA and the d_hid-term sum of w2 * act(h) are fp32 in an order that differs from the oracle's: with
d = d_hid = 4096, O(1) pre-activations and scores, the accumulated rounding is a few 1e-6 (observed),
erff / tanhf add about 1e-7 relative per term."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import dev, kernel_names, template_arguments

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    import paper_2310_02409_amd as D
    return D


def _case(seed, N, d, dh, dtype):
    x = W.normal(seed, 0, (N, d), 1.0, dtype)
    W1 = W.normal(seed, 1, (dh, d), d ** -0.5, dtype)
    b1 = W.normal(seed, 2, (dh,), 0.5, torch.float32)
    w2 = W.normal(seed, 3, (dh,), dh ** -0.5, dtype)
    return x, W1, b1, w2


def _check(got, want):
    err = np.abs(got - want)
    assert np.all(err <= 1e-4 * (1 + np.abs(want))), f"max err {err.max():.3e}"
    return float(err.max())


@pytest.mark.parametrize("N,d,dh", [(300, 64, 256), (257, 128, 512), (1000, 256, 768), (5, 64, 256), (700, 192, 256),
                                    (300, 64, 1280)])  # 5 hidden tiles over 4 splits: one split has none
@pytest.mark.parametrize("act", [0, 1, 2])
def test_mfma_path_small_shapes(D, N, d, dh, act):
    x, W1, b1, w2 = _case(900 + N, N, d, dh, torch.bfloat16)
    want = oracle.score_mlp(W.to_numpy(x), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.25, act)
    got = D.dodo_score_mlp(x.to(dev()), W1.to(dev()), b1.to(dev()), w2.to(dev()), 0.25, act).cpu().numpy()
    _check(got, want)


# few tokens: blocks of 16 tokens, runs of 64 channels over 8 wavefronts (1, 9 and 130 of them), equal shares of the
# hidden units per compute unit (a single one, an incomplete second block of 16, two full blocks with a short last share)
@pytest.mark.parametrize("N", [1, 15, 16, 17, 32, 33, 64, 65])
@pytest.mark.parametrize("d,dh", [(64, 256), (576, 5376), (128, 8448), (8320, 256)])
def test_few_tokens(D, N, d, dh):
    x, W1, b1, w2 = _case(970 + N, N, d, dh, torch.bfloat16)
    want = oracle.score_mlp(W.to_numpy(x), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.25, 1)
    padded = torch.full((N, d + 8), float("nan"), dtype=torch.bfloat16)  # rows further apart than d: nothing between them is read
    padded[:, :d] = x
    got = D.dodo_score_mlp(padded.to(dev())[:, :d], W1.to(dev()), b1.to(dev()), w2.to(dev()), 0.25, 1).cpu().numpy()
    _check(got, want)


# The kernel for few tokens and tiles of 64 tokens on either side of the line between them: 28 tokens where the tiles are at most half as many as
# the compute units and W1 has 2048 channels or more, 20 elsewhere.
@pytest.mark.parametrize("d,dh,line", [(2048, 2048, 28), (4096, 4096, 28), (1024, 1024, 20), (2048, 4352, 20)])
def test_line_between_few_tokens_and_tiles_of_64(D, d, dh, line):
    x, W1, b1, w2 = _case(975, line + 1, d, dh, torch.bfloat16)
    t = [v.to(dev()) for v in (x, W1, b1, w2)]
    want = oracle.score_mlp(W.to_numpy(x), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.25, 1)
    for N, kernel in ((line, "score_mlp_few_kernel"), (line + 1, "score_mlp_some_kernel")):
        out = []
        names = kernel_names(lambda: out.append(D.dodo_score_mlp(t[0][:N], *t[1:], 0.25, 1)), "score_mlp_")
        assert any(kernel in n for n in names), names
        _check(out[0].cpu().numpy(), want[:N])


# small tiles alone (edges of 128 tokens), whole rounds of big tiles followed by small ones, big tiles alone
@pytest.mark.parametrize("N,d,dh", [(65, 64, 512), (127, 128, 256), (128, 64, 256), (129, 64, 768), (2049, 64, 1280),
                                    (4096, 64, 4096), (4097, 64, 4096), (4500, 128, 4096), (66000, 64, 256)])
def test_shares_of_big_and_small_tiles(D, N, d, dh):
    x, W1, b1, w2 = _case(980 + N, N, d, dh, torch.bfloat16)
    rows = np.arange(N) if N * dh < 2e6 else np.unique(np.r_[0:130, N - 600:N, 4090:min(N, 4110)] % N)
    want = oracle.score_mlp(W.to_numpy(x[rows]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.25, 1)
    got = D.dodo_score_mlp(x.to(dev()), W1.to(dev()), b1.to(dev()), w2.to(dev()), 0.25, 1).cpu().numpy()
    _check(got[rows], want)


# one buffer for calls with fewer and with more tokens: the least that a call needs is a float per token and split of
# the big tiles, and a buffer below that is refused
@pytest.mark.parametrize("N,least", [(40, 16), (64, 16), (100, 16), (4500, 16), (8200, 8)])
def test_workspace_sized_for_another_call(D, N, least):
    d, dh = 64, 4096
    x, W1, b1, w2 = _case(990, N, d, dh, torch.bfloat16)
    t = [v.to(dev()) for v in (x, W1, b1, w2)]
    rows = np.r_[0:20, N - 20:N]
    want = oracle.score_mlp(W.to_numpy(x[rows]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.0, 0)
    ws = torch.full((least * N * 4 + 64,), 255, dtype=torch.uint8, device=dev())
    got = D.dodo_score_mlp(*t, ws=ws[:least * N * 4]).cpu().numpy()
    _check(got[rows], want)
    assert torch.all(ws[least * N * 4:] == 255)
    with pytest.raises(D.DodoError):
        D.dodo_score_mlp(*t, ws=ws[:least * N * 4 - 4])


# one buffer, sized once for the most tokens, while their number falls
@pytest.mark.parametrize("most", [65536, 32768, 300])
def test_workspace_kept_for_fewer_tokens(D, most):
    d, dh = 64, 4096
    x, W1, b1, w2 = _case(991, most, d, dh, torch.bfloat16)
    t = [v.to(dev()) for v in (x, W1, b1, w2)]
    ws = torch.full((max(1, D.dodo_score_mlp_workspace_bytes(D.BF16, most, d, dh)),), 255, dtype=torch.uint8, device=dev())
    for N in (most, 63488, 30720, 16128, 8200, 4097, 300, 65, 64, 1):
        if N <= most:
            rows = np.unique(np.r_[0:min(N, 20), max(0, N - 20):N])
            got = D.dodo_score_mlp(t[0][:N], *t[1:], ws=ws).cpu().numpy()
            _check(got[rows], oracle.score_mlp(W.to_numpy(x[rows]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.0, 0))


# a buffer sized for more tokens may be too small for the plan with tiles of 64 tokens: the plan without them is next (big tiles in eight
# splits, which fill whole rounds), and not big tiles in as many splits as there are hidden tiles
@pytest.mark.parametrize("most,N", [(6987, 6165), (8054, 6226)])
def test_workspace_too_small_for_tiles_of_64_tokens(D, most, N):
    d, dh = 2048, 4096
    x, W1, b1, w2 = _case(992, N, d, dh, torch.bfloat16)
    t = [v.to(dev()) for v in (x, W1, b1, w2)]
    ws = torch.full((D.dodo_score_mlp_workspace_bytes(D.BF16, most, d, dh),), 255, dtype=torch.uint8, device=dev())
    got = D.dodo_score_mlp(*t, ws=ws).cpu().numpy()
    rows = np.unique(np.r_[0:20, 4090:4100, N - 20:N])
    _check(got[rows], oracle.score_mlp(W.to_numpy(x[rows]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.0, 0))
    assert not torch.all(ws[7 * N * 4:8 * N * 4] == 255) and torch.all(ws[8 * N * 4:] == 255)


@pytest.mark.parametrize("N,dh", [(1, 256), (16, 256), (40, 5120), (70, 256)])
def test_infinite_channel_saturates(D, N, dh):
    # tanh of an infinite hidden unit is 1 or -1: the score stays finite, also where a workgroup's share of the hidden units
    # is no whole block
    x, W1, b1, w2 = _case(996, N, 64, dh, torch.bfloat16)
    x[N // 2, 9], x[0, 5] = float("-inf"), float("inf")
    x[0, 9] = 0.0
    got = D.dodo_score_mlp(*[v.to(dev()) for v in (x, W1, b1, w2)], act=D.TANH).cpu().numpy()
    _check(got, oracle.score_mlp(W.to_numpy(x), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.0, 2))


@pytest.mark.parametrize("dtype,N,d,dh", [(torch.float32, 512, 256, 256), (torch.bfloat16, 37, 40, 100),
                                          (torch.float32, 9, 24, 7)])
def test_plain_path_any_shape(D, dtype, N, d, dh):
    x, W1, b1, w2 = _case(950 + N, N, d, dh, dtype)
    for act in (0, 1, 2):
        want = oracle.score_mlp(W.to_numpy(x), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), -0.5, act)
        got = D.dodo_score_mlp(x.to(dev()), W1.to(dev()), b1.to(dev()), w2.to(dev()), -0.5, act).cpu().numpy()
        _check(got, want)


def test_row_stride_and_determinism(D):
    N, d, dh = 600, 64, 256
    x, W1, b1, w2 = _case(960, N, d, dh, torch.bfloat16)
    wide = torch.zeros((N, d + 24), dtype=torch.bfloat16)
    wide[:, :d] = x
    want = oracle.score_mlp(W.to_numpy(x), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.0, 1)
    a = D.dodo_score_mlp(wide.to(dev())[:, :d], W1.to(dev()), b1.to(dev()), w2.to(dev()), 0.0, 1)
    b = D.dodo_score_mlp(wide.to(dev())[:, :d], W1.to(dev()), b1.to(dev()), w2.to(dev()), 0.0, 1)
    _check(a.cpu().numpy(), want)
    assert torch.equal(a, b)


def test_llama7b_shape_sampled_tokens(D):
    # the paper's scorer size: d = d_hid = 4096 (16.8 M parameters) on the prefill workload's 32768 tokens
    wl = W.config(2)
    N, d = wl.N, wl.d_model
    x = W.make_inputs(wl, dev(), which=["hidden"])["hidden"]
    W1 = W.normal(wl.seed, 40, (d, d), d ** -0.5, torch.bfloat16, dev())
    b1 = W.normal(wl.seed, 41, (d,), 0.5, torch.float32, dev())
    w2 = W.normal(wl.seed, 42, (d,), d ** -0.5, torch.bfloat16, dev())
    got = D.dodo_score_mlp(x, W1, b1, w2, 0.125, 1)
    rows = [0, 1, 255, 256, 4095, 4096, 17000, 32767] + [int(v) for v in np.random.default_rng(1).integers(0, N, 8)]
    want = oracle.score_mlp(W.to_numpy(x[rows].cpu()), W.to_numpy(W1.cpu()), b1.cpu().numpy(), W.to_numpy(w2.cpu()), 0.125, 1)
    _check(got[rows].cpu().numpy(), want)


# channels shared by two groups of wavefronts, in small tiles (1024 tokens the most of them, 1025 too many) and, up to a few hundred
# tokens, in tiles of 64: one, two and an odd number of steps each
@pytest.mark.parametrize("N,d,dh", [(65, 128, 256), (129, 256, 512), (128, 384, 256), (1024, 128, 4096), (1025, 128, 4096),
                                    (130, 192, 512), (200, 1024, 512)])
@pytest.mark.parametrize("act", [0, 2])
def test_channels_shared_by_two_groups(D, N, d, dh, act):
    x, W1, b1, w2 = _case(1000 + N, N, d, dh, torch.bfloat16)
    rows = np.unique(np.r_[0:min(N, 140), N - 20:N])
    want = oracle.score_mlp(W.to_numpy(x[rows]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.25, act)
    got = D.dodo_score_mlp(x.to(dev()), W1.to(dev()), b1.to(dev()), w2.to(dev()), 0.25, act).cpu().numpy()
    _check(got[rows], want)


# Infinite and NaN channels in either half of the channels (tiles of 64 tokens; small tiles below): tanh of an infinite hidden unit is 1 or -1, a NaN channel makes its token's score
# NaN and no other one's.
@pytest.mark.parametrize("N,d,dh", [(65, 128, 256), (130, 128, 512), (200, 384, 256)])
def test_channels_shared_by_two_groups_that_are_not_finite(D, N, d, dh):
    x, W1, b1, w2 = _case(1010 + N, N, d, dh, torch.bfloat16)
    x[N // 2, 9], x[3, d - 5], x[N - 1, d // 2] = float("-inf"), float("inf"), float("inf")
    nan = [1, 40, N - 2]
    x[1, 0], x[40, d // 2 - 1], x[N - 2, d - 1] = float("nan"), float("nan"), float("nan")
    got = D.dodo_score_mlp(*[v.to(dev()) for v in (x, W1, b1, w2)], act=D.TANH).cpu().numpy()
    assert np.isnan(got[nan]).all()
    rest = np.setdiff1d(np.arange(N), nan)
    _check(got[rest], oracle.score_mlp(W.to_numpy(x[rest]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.0, 2))


# Tiles of 64 tokens: 32 hidden units per tile (a tile per compute unit at most), 64 with one and with two tiles per unit; tokens around
# a tile's end, fewer steps than there are stages, one more than are folded, and an even number; beside them a call of few tokens and one of
# big and small tiles.  (What whole rounds of other tiles leave: further down.)
@pytest.mark.parametrize("N,d,dh", [(17, 128, 256), (63, 1152, 512), (64, 128, 8192), (65, 256, 4096), (129, 384, 4096), (256, 2048, 1024),
                                    (300, 512, 4096), (512, 128, 4096), (577, 1152, 2048), (2100, 4096, 512), (9000, 1152, 4096)])
@pytest.mark.parametrize("act", [0, 1, 2])
def test_tiles_of_64_tokens(D, N, d, dh, act):
    x, W1, b1, w2 = _case(1020 + N, N, d, dh, torch.bfloat16)
    rows = np.unique(np.r_[0:min(N, 20), 60:min(N, 70), max(0, N - 70):N])
    want = oracle.score_mlp(W.to_numpy(x[rows]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.25, act)
    padded = torch.full((N, d + 8), float("nan"), dtype=torch.bfloat16)
    padded[:, :d] = x
    t = [v.to(dev()) for v in (padded, W1, b1, w2)]
    ws = torch.full((D.dodo_score_mlp_workspace_bytes(D.BF16, N, d, dh) + 64,), 255, dtype=torch.uint8, device=dev())
    got = D.dodo_score_mlp(t[0][:, :d], *t[1:], 0.25, act, ws=ws[:-64]).cpu().numpy()
    _check(got[rows], want)
    assert torch.all(ws[-64:] == 255)


@pytest.mark.parametrize("N,d,dh", [(40, 256, 4096), (150, 256, 4096), (300, 128, 4096)])
def test_tiles_of_64_tokens_that_are_not_finite(D, N, d, dh):
    x, W1, b1, w2 = _case(1040 + N, N, d, dh, torch.bfloat16)
    x[N // 2, 9], x[3, d - 5], x[N - 1, d // 2] = float("-inf"), float("inf"), float("inf")
    nan = [1, 30, N - 2]
    x[1, 0], x[30, d // 2 - 1], x[N - 2, d - 1] = float("nan"), float("nan"), float("nan")
    got = D.dodo_score_mlp(*[v.to(dev()) for v in (x, W1, b1, w2)], act=D.TANH).cpu().numpy()
    assert np.isnan(got[nan]).all()
    rest = np.setdiff1d(np.arange(N), nan)
    _check(got[rest], oracle.score_mlp(W.to_numpy(x[rest]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.0, 2))


# Small tiles whose channels two groups of wavefronts share, by the kernel's name: one, three, two, five and one (odd) steps each, tokens at a
# tile's edges; then with NaN and infinite channels in either group's half.
@pytest.mark.parametrize("N,d,dh", [(808, 128, 4096), (1010, 384, 4096), (700, 256, 4096), (1024, 640, 4096), (600, 128, 5120)])
@pytest.mark.parametrize("finite", [True, False])
def test_small_tiles_in_two_groups(D, N, d, dh, finite):
    x, W1, b1, w2 = _case(1060 + N, N, d, dh, torch.bfloat16)
    nan = [] if finite else [1, 140, N - 2]
    if not finite:
        x[N // 2, 9], x[3, d - 5], x[N - 1, d // 2] = float("-inf"), float("inf"), float("inf")
        x[1, 0], x[140, d // 2 - 1], x[N - 2, d - 1] = float("nan"), float("nan"), float("nan")
    rows = np.setdiff1d(np.r_[0:8, 124:150, 250:260, N // 2, N - 30:N], nan)
    want = oracle.score_mlp(W.to_numpy(x[rows]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.25, 2)
    t, out = [v.to(dev()) for v in (x, W1, b1, w2)], []
    names = [n for n in kernel_names(lambda: out.append(D.dodo_score_mlp(*t, 0.25, D.TANH)), "score_mlp_") if "combine" not in n]
    assert len(names) == 1 and "score_mlp_mfma_kernel" in names[0] and template_arguments(names[0])[3] == "2", names
    got = out[0].cpu().numpy()
    _check(got[rows], want)
    assert np.isnan(got[nan]).all() and np.isfinite(np.delete(got, nan)).all()


# Several kinds of tiles in one call: whole rounds of big or of small tiles and, for what they leave, tiles of 64 tokens, whose partial
# scores have a region and a part of the last kernel of their own; tokens on both sides of the boundary, rows further apart than d.
@pytest.mark.parametrize("N,first,d,dh", [(2322, 2048, 4096, 4096), (2100, 2048, 1920, 4096), (4121, 4096, 2048, 4096), (4121, 4096, 2048, 2048),
                                          (6165, 6144, 2048, 4096)])
@pytest.mark.parametrize("act", [0, 2])
def test_tiles_of_64_tokens_after_whole_rounds(D, N, first, d, dh, act):
    x, W1, b1, w2 = _case(1070 + N, N, d, dh, torch.bfloat16)
    rows = np.unique(np.r_[0:4, 4094:min(N, 4098), first - 12:first + 20, first + 60:min(N, first + 68), N - 6:N] % N)
    want = oracle.score_mlp(W.to_numpy(x[rows]), W.to_numpy(W1), b1.numpy(), W.to_numpy(w2), 0.25, act)
    padded = torch.full((N, d + 8), float("nan"), dtype=torch.bfloat16)
    padded[:, :d] = x
    t = [v.to(dev()) for v in (padded, W1, b1, w2)]
    ws = torch.full((D.dodo_score_mlp_workspace_bytes(D.BF16, N, d, dh) + 64,), 255, dtype=torch.uint8, device=dev())
    out = torch.full((N + 16,), float("nan"), device=dev())
    names = kernel_names(lambda: D.dodo_score_mlp(t[0][:, :d], *t[1:], 0.25, act, out=out[:N], ws=ws[:-64]), "score_mlp_")
    assert any("some_kernel" in n for n in names) and any("mfma_kernel" in n for n in names), names
    got = out.cpu().numpy()
    _check(got[rows], want)
    assert np.isfinite(got[:N]).all() and np.isnan(got[N:]).all() and torch.all(ws[-64:] == 255)
