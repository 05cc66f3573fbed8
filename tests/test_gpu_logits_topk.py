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
