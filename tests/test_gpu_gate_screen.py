"""The gate's kernels in weight mode: ids and weights must be the bits that the
float64 logits of every expert give.

A call that asks for the logits forms all of them in float64 (one token per
block for few tokens, else on the matrix cores); the same call without them
screens the experts on the matrix cores first. Inputs where
the screen says little (large terms that cancel, equal experts, equal logits
at the k-th place, overflowing magnitudes, denormals) are among them.
"""
import numpy as np
import pytest
import torch

from oracle import moe_ew as O
from paper_2601_01310_amd import synth, tg
from tests import _gate_cases as C
from tests._util import host, u16
from tests.test_gpu_logits_topk import check_without_nan

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _run(x, w, k, want_logits):
    T, d = x.shape
    E = w.shape[0]
    logits = torch.empty((T, E), dtype=torch.float32, device=DEV) if want_logits else None
    ids = torch.full((T, k), -7, dtype=torch.int32, device=DEV)
    tw = torch.full((T, k), -7.0, dtype=torch.float32, device=DEV)
    tg.tg_gate_topk(x, w, None, T, d, E, k, logits, ids, tw)
    torch.cuda.synchronize()
    return (None if logits is None else host(logits)), host(ids), host(tw)


def _same(x, w, k):
    logits, ids, tw = _run(x, w, k, True)
    _, ids2, tw2 = _run(x, w, k, False)
    assert np.array_equal(ids, O.topk(logits, k))
    assert np.array_equal(ids2, ids)
    assert np.array_equal(tw2.view(np.uint32), tw.view(np.uint32))


def _normal(T, d, E, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.randn((T, d), generator=g, device=DEV).to(torch.bfloat16)
    w = (torch.randn((E, d), generator=g, device=DEV) * 0.02).to(torch.bfloat16)
    return x, w


# Up to 256 tokens (512 with at most 16 experts, 1024 with 8) a block per
# token; beyond, up to 16 experts by one dense block per 16 tokens, else the
# screen in every number of pieces and groups (E <= 64, 128, 256, 512,
# 1024), tiles of 16 experts that are partial, token tails, row lengths off
# the stages' 64 to 256 elements, the largest E and k.
@pytest.mark.parametrize("T,d,E,k", [
    (1, 7168, 256, 8), (3, 128, 5, 5), (256, 448, 40, 5), (1024, 192, 8, 4), (512, 192, 16, 4),
    (257, 7168, 256, 8), (1025, 4096, 16, 1), (1030, 256, 8, 2), (1033, 320, 3, 3), (513, 7168, 16, 8),
    (299, 3136, 17, 17), (276, 1856, 64, 6), (321, 960, 65, 3), (287, 4160, 128, 32),
    (274, 448, 129, 8), (273, 1024, 160, 6), (296, 2112, 257, 9), (291, 192, 512, 32),
    (306, 128, 1000, 8), (289, 7168, 1024, 32)])
def test_screen_gives_the_bits_of_all_float64_logits(T, d, E, k):
    print(f"[gpu] gate screen T={T} d={d} E={E} k={k}", flush=True)
    x, w = _normal(T, d, E, T * 7 + d + E)
    _same(x, w, k)


@pytest.mark.parametrize("T,E,I", [(300, 64, 128), (1030, 17, 192), (700, 256, 128)])
def test_the_forward_gates_as_the_gate_does(T, E, I):
    """The forward may form the logits in its workspace first."""
    print(f"[gpu] gate in the forward T={T} E={E}", flush=True)
    wl = synth.make_custom(T=T, d=256, E=E, k=2, I=I, n_local=2, shadow_experts=[0],
                           gate="weights", seed=T, device=DEV)
    f = tg.EwForward(wl)
    f()
    _, ids, tw = _run(wl.x, wl.wg, 2, False)
    logits = O.gate_logits(u16(wl.x), u16(wl.wg))
    assert np.array_equal(ids, O.topk(logits, 2))
    assert np.array_equal(host(f.topk_ids), ids)
    assert np.array_equal(host(f.topk_w).view(np.uint32), tw.view(np.uint32))


@pytest.mark.parametrize("E,k", [(64, 4), (100, 8), (256, 8)])
def test_equal_experts_and_ties(E, k):
    """Copies of one gate row tie exactly: the lower ids win."""
    print(f"[gpu] gate screen ties E={E}", flush=True)
    x, w = _normal(293, 2048, E, 5)
    w[E // 2:] = w[:E - E // 2]      # every expert twice
    w[3:E:9] = w[3]                  # and one of them many times
    _same(x, w, k)
    w[:] = w[0]                      # all of them: every expert is a candidate
    _same(x, w, k)


def test_cancelling_terms_at_float32_midpoints():
    """Rows whose exact logits lie at float32 midpoints behind a +1024 / -1024
    pair, which a float32 sum cannot tell apart."""
    print("[gpu] gate screen midpoints", flush=True)
    xb, wb, expected, _ = C.engineered(40, 32, 4096, seed=11)
    xb, expected = np.tile(xb, (8, 1)), np.tile(expected, (8, 1))  # 320 tokens
    x = torch.from_numpy(xb.view(np.int16)).view(torch.bfloat16).to(DEV)
    w = torch.from_numpy(wb.view(np.int16)).view(torch.bfloat16).to(DEV)
    logits, _, _ = _run(x, w, 6, True)
    assert np.array_equal(logits.view(np.uint32), expected.view(np.uint32))
    _, ids, tw = _run(x, w, 6, False)
    r_ids = O.topk(expected, 6)
    assert np.array_equal(ids, r_ids)
    assert np.abs(tw - O.gate_weights(expected, r_ids)).max() <= 1e-6


@pytest.mark.parametrize("what", ["zero", "denormal", "huge", "overflow", "one_sided"])
def test_extreme_magnitudes(what):
    print(f"[gpu] gate screen {what}", flush=True)
    x, w = _normal(280, 1024, 96, 3)
    if what == "zero":
        x[::2] = 0
    elif what == "denormal":        # products near and below the smallest float32
        x *= 2.0 ** -120
        w[:, ::2] *= 2.0 ** -20
        w[:, 1::2] = (w[:, 1::2].float() * 2.0 ** -125).to(torch.bfloat16)
    elif what == "huge":            # near float32's end, finite sums
        x *= 2.0 ** 100
        w *= 2.0 ** 15
    elif what == "overflow":        # products past float32 that cancel in float64
        # (no small values: every float64 sum is exact, multiples of 2^82 below 2^132)
        x[x.abs() < 2.0 ** -4] = 0
        w[w.abs() < 2.0 ** -10] = 0
        x, w = x * 2.0 ** 55, w * 2.0 ** 55
        x[:, 0] = x[:, 1] = w[:, 0] = 2.0 ** 65
        w[:, 1] = -(2.0 ** 65)
    else:                           # all products of one sign
        x, w = x.abs(), w.abs()
    _same(x, w, 8)


def test_screen_matches_the_oracle():
    print("[gpu] gate screen oracle", flush=True)
    x, w = _normal(300, 7168, 256, 77)
    _, ids, tw = _run(x, w, 8, False)
    logits = O.gate_logits(u16(x), u16(w))
    r = O.topk(logits, 8)
    assert np.array_equal(ids, r)
    assert np.abs(tw - O.gate_weights(logits, r)).max() <= 1e-6


def _lane_order_logits(x, w):
    """Float64 sums in the kernels' one order: lane l of 64 adds the products of
    the 8-element chunks l, l + 64, ... (exact in float64) one after the other,
    then neighbouring lanes are added pairwise up to sixteen, and the four
    sixteens in order."""
    x, w = x.astype(np.float64), w.astype(np.float64)
    T, d = x.shape
    lanes = np.zeros((T, len(w), 64))
    for c in range(0, d, 512):
        n = min(512, d - c) // 8
        for i in range(8):
            lanes[:, :, :n] += x[:, None, c + i:c + 8 * n:8] * w[None, :, c + i:c + 8 * n:8]
    for _ in range(4):
        lanes = lanes[..., 0::2] + lanes[..., 1::2]
    s = ((lanes[..., 0] + lanes[..., 1]) + lanes[..., 2]) + lanes[..., 3]
    return s.astype(np.float32)


# Few tokens (a block per token), and a batch that takes the dense kernel with
# its top-k (16 experts), the dense kernel (the logits wanted, or in the
# forward's workspace), or the screen.
@pytest.mark.parametrize("T,E,d", [(600, 16, 1088), (1030, 8, 256), (300, 40, 1088), (300, 200, 7168),
                                   (270, 300, 192)])
def test_a_token_gates_alike_in_every_batch(T, E, d):
    """Terms of 2^40 that cancel leave a logit that depends on the order of the
    float64 additions: it has to be one order in every kernel."""
    print(f"[gpu] gate order T={T} E={E} d={d}", flush=True)
    k = 6
    x, w = _normal(T, d, E, T + d)
    w *= 50.0
    for a, b in ((5, d - 3), (70, 131), (33, 34)):
        x[:, a] = x[:, b] = 2.0 ** 20
        w[:, a], w[:, b] = 2.0 ** 20, -(2.0 ** 20)
    few = 4
    expected = _lane_order_logits(x[:few].float().cpu().numpy(), w.float().cpu().numpy())
    exact = x[:few].double().cpu().numpy() @ w.double().cpu().numpy().T
    assert (exact.astype(np.float32) != expected).any()  # the order shows
    logits, ids, tw = _run(x[:few].contiguous(), w, k, True)
    assert np.array_equal(logits.view(np.uint32), expected.view(np.uint32))
    for want in (True, False):
        l2, ids2, tw2 = _run(x, w, k, want)
        if want:
            assert np.array_equal(l2[:few].view(np.uint32), expected.view(np.uint32))
        assert np.array_equal(ids2[:few], ids)
        assert np.array_equal(tw2[:few].view(np.uint32), tw.view(np.uint32))
    wl = synth.make_custom(T=T, d=d, E=E, k=k, I=1024, n_local=2, shadow_experts=[0], gate="weights",
                           seed=T, device=DEV)
    wl.x.copy_(x)
    wl.wg.copy_(w)
    f = tg.EwForward(wl)
    f()
    torch.cuda.synchronize()
    assert np.array_equal(host(f.topk_ids)[:few], ids)
    assert np.array_equal(host(f.topk_w)[:few].view(np.uint32), tw.view(np.uint32))


# token (4 tokens), dense with its top-k (16 experts) and after it (logits
# wanted), screen.
@pytest.mark.parametrize("T,E", [(4, 40), (600, 16), (300, 200), (300, 300)])
def test_nan_is_not_chosen(T, E):
    """Gate rows that hold a NaN are passed over; a token that holds one has
    no choice at all."""
    print(f"[gpu] gate NaN T={T} E={E}", flush=True)
    d, k = 256, 8
    x, w = _normal(T, d, E, T + E)
    w[1::7, 5] = float("nan")
    x[2] = float("nan")
    x[3, :] = 0
    logits = O.gate_logits(u16(x), u16(w))
    assert np.isnan(logits[:, 1]).all()
    for want in (False, True):
        _, ids, tw = _run(x, w, k, want)
        check_without_nan(logits, k, ids, tw)
    w[k - 2:, 5] = float("nan")  # fewer than k experts are left
    w[:k - 2] = w[0]
    logits = O.gate_logits(u16(x), u16(w))
    for want in (False, True):
        _, ids, tw = _run(x, w, k, want)
        check_without_nan(logits, k, ids, tw)
