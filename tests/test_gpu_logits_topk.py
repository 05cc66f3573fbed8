"""Top-k over given logits: winners and weights against the oracle, at sizes
around the kernels' rows and blocks, with ties, equal logits, masks of -inf and
of the lowest float32, and signed zeros."""
import numpy as np
import pytest
import torch

from oracle import moe_ew as O
from paper_2601_01310_amd import tg
from tests._util import host

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _check(lg, k):
    T, E = lg.shape
    ids = torch.full((T, k), -7, dtype=torch.int32, device=DEV)
    w = torch.full((T, k), -7.0, dtype=torch.float32, device=DEV)
    tg.tg_gate_topk(None, None, lg, T, 0, E, k, None, ids, w)
    torch.cuda.synchronize()
    l = host(lg)
    # larger first, equal logits (also -0 and +0) by lower id
    r = np.argsort(-(l.astype(np.float64) + 0.0), axis=1, kind="stable")[:, :k]
    assert np.array_equal(host(ids), r)
    top = np.take_along_axis(l, r, 1).astype(np.float64)
    e = np.exp(top - top[:, :1])
    assert np.abs(host(w) - e / e.sum(1, keepdims=True)).max() <= 1e-6


@pytest.mark.parametrize("T,E,k", [
    (1, 256, 8), (3, 256, 16), (5, 7, 7), (63, 16, 4), (130, 64, 6), (257, 65, 8), (511, 128, 8),
    (1000, 129, 3), (4095, 256, 8), (4097, 255, 8), (4100, 8, 2), (9, 256, 17), (6, 300, 8),
    (4099, 1, 1), (37, 33, 1)])
def test_random_logits(T, E, k):
    print(f"[gpu] logits topk T={T} E={E} k={k}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + E)
    _check(torch.randn((T, E), generator=g, device=DEV), k)


# At the limits between the kernels: one token per wave (under 4096 tokens, more
# than 64 experts, 2 or 3 choices), rounds, and a few candidates (from 3 to 5
# choices on, up to 9 to 12 of more than 32 experts).
@pytest.mark.parametrize("T,E,k", [
    (700, 64, 2), (700, 65, 2), (700, 65, 3), (700, 128, 3), (700, 128, 4), (700, 129, 3), (700, 129, 4), (4095, 200, 1),
    (4096, 200, 1), (4096, 200, 3), (700, 64, 4), (700, 64, 5), (700, 32, 16), (700, 33, 10),
    (700, 33, 11), (700, 65, 9), (700, 65, 10), (700, 250, 16), (8192, 100, 10), (8193, 100, 11),
    (8193, 100, 12), (32768, 129, 2), (32769, 129, 1), (32769, 129, 12), (32769, 40, 13), (32769, 8, 4)])
def test_limits_between_the_kernels(T, E, k):
    print(f"[gpu] logits topk limits T={T} E={E} k={k}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + E + k)
    lg = torch.randn((T, E), generator=g, device=DEV)
    lg[0::7] = torch.round(lg[0::7])
    lg[1::7] = 0.5
    lg[2::7, k:] = -float("inf")
    _check(lg, k)


@pytest.mark.parametrize("E,k", [(40, 8), (100, 8), (256, 8), (256, 16)])
def test_ties_and_masks(E, k):
    print(f"[gpu] logits topk ties E={E} k={k}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(E)
    lg = torch.randn((4104, E), generator=g, device=DEV)
    lg[0::9] = torch.round(lg[0::9])                # few distinct values
    lg[1::9] = 0.25                                 # all equal
    lg[2::9, ::2] = -0.0                            # signed zeros tie
    lg[2::9, 1::2] = 0.0
    lg[3::9, k:] = -float("inf")                    # just k experts left
    lg[4::9, k + 3:] = torch.finfo(torch.float32).min
    lg[5::9] = torch.sort(lg[5::9], dim=1)[0]       # increasing
    lg[6::9, : E // 2] += 40.0                      # one half far above
    lg[7::9, 5::16] += 40.0                         # the winners in one lane's column
    _check(lg, k)


# NaN logits are never chosen by batches under 4096 tokens or beyond 256
# experts; where fewer than k are left, the id is 0x7fffffff, the weight 0 (NaN
# without any).
@pytest.mark.parametrize("T,E,k", [(5, 40, 8), (70, 256, 8), (4095, 128, 16), (4100, 300, 4),
                                   (70, 64, 3), (70, 200, 3), (700, 256, 12)])
def test_nan_is_not_chosen(T, E, k):
    print(f"[gpu] logits topk NaN T={T} E={E} k={k}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + E)
    lg = torch.randn((T, E), generator=g, device=DEV)
    lg[0::5, 3] = float("nan")
    lg[1::5, : E - k] = float("nan")      # just k are left
    lg[2::5, 2:] = float("nan")           # two
    lg[3::5] = 0.5                        # more than 16 candidates
    lg[3::5, ::2] = float("nan")
    lg[4::5, 1::2] = -float("nan")
    lg[4] = float("nan")
    ids = torch.full((T, k), -7, dtype=torch.int32, device=DEV)
    w = torch.full((T, k), -7.0, dtype=torch.float32, device=DEV)
    tg.tg_gate_topk(None, None, lg, T, 0, E, k, None, ids, w)
    torch.cuda.synchronize()
    check_without_nan(host(lg), k, host(ids), host(w))


def check_without_nan(l, k, ids, w):
    nan = np.isnan(l)
    r = np.argsort(np.where(nan, np.inf, -l.astype(np.float64)), axis=1, kind="stable")[:, :k]
    left = ~np.take_along_axis(nan, r, 1)
    assert np.array_equal(ids, np.where(left, r, 0x7FFFFFFF))
    some = left[:, 0]
    assert np.isnan(w[~some]).all()
    top = np.where(left, np.take_along_axis(l, r, 1).astype(np.float64), -np.inf)[some]
    e = np.exp(top - top[:, :1])
    assert np.abs(w[some] - e / e.sum(1, keepdims=True)).max() <= 1e-6


@pytest.mark.parametrize("k", [3, 5])
def test_nan_is_ordered_in_large_batches_by_either_kernel(k):
    """As below, by rounds and among a few candidates, down to the negative NaN."""
    print(f"[gpu] logits topk NaN order k={k}", flush=True)
    T = 4100
    lg = torch.full((T, 40), -float("inf"), device=DEV)
    lg[:, 11] = float("nan")
    lg.view(torch.int32)[:, :37] = torch.where(lg[:, :37].isnan(), lg.view(torch.int32)[:, :37], -4194304)
    lg[:, 38] = 2.0
    ids = torch.full((T, k), -7, dtype=torch.int32, device=DEV)
    w = torch.empty((T, k), dtype=torch.float32, device=DEV)
    tg.tg_gate_topk(None, None, lg, T, 0, 40, k, None, ids, w)
    torch.cuda.synchronize()
    assert (host(ids) == np.array([11, 38, 37, 39, 0][:k])).all()


def test_nan_is_ordered_in_large_batches():
    """From 4096 tokens on a positive NaN ranks above +inf, a negative one below -inf."""
    print("[gpu] logits topk NaN order", flush=True)
    lg = torch.arange(4096 * 64, device=DEV, dtype=torch.float32).reshape(4096, 64) % 61
    lg[:, 7], lg[:, 9] = float("nan"), float("inf")
    lg.view(torch.int32)[:, 60] = -4194304  # 0xffc00000, a negative NaN
    ids = torch.full((4096, 3), -7, dtype=torch.int32, device=DEV)
    w = torch.empty((4096, 3), dtype=torch.float32, device=DEV)
    tg.tg_gate_topk(None, None, lg, 4096, 0, 64, 3, None, ids, w)
    torch.cuda.synchronize()
    l = host(lg).copy()
    l[:, [7, 9, 60]] = -1.0
    third = l.argmax(axis=1)
    assert np.array_equal(host(ids), np.stack([np.full(4096, 7), np.full(4096, 9), third], 1))
