"""The grouped GEMMs' middle tile shapes: every launch gives the bits of the
256-row walk, whichever shape its slot counts select.

The cases reach each shape of both projections (named per case) with row tails, empty slots and widths that leave partial panels; the
256-row walk itself is held against the oracle by the parity tests, and one
case here is too.
"""
import numpy as np
import pytest
import torch

from oracle import moe_ew as O
from paper_2601_01310_amd import synth, tg
from tests._gpu import assert_close_bf16
from tests._util import u16

pytestmark = pytest.mark.gpu
DEV = "cuda"

# d, I, rows per slot, and the shapes that a grid of 256 blocks takes for them: a
# CPU test holds the names to the kernels' choice.
CASES = [
    (320, 192, [30, 30, 30], "32x32", "32x32"),
    (192, 320, [0, 32, 0], "32x32", "32x32"),
    (1088, 320, [127, 127], "32x32", "32x64"),
    (2112, 512, [70, 139, 0], "32x32", "64x64"),
    (320, 192, [129, 0, 129, 129, 129, 126, 129, 128], "32x64", "32"),
    (192, 704, [62, 33, 64], "32x64", "32x32"),
    (512, 1472, [124], "32x64", "32x32"),
    (1088, 128, [400, 400, 399], "32x64", "128x64"),
    (1088, 512, [513], "64x64", "64x64"),
    (1024, 1472, [129, 128], "64x64", "32x64"),
    (1088, 192, [300, 0, 0, 150, 300, 297, 297, 300], "64x64", "64x128"),
    (2112, 192, [513, 513, 513], "64x64", "128x128"),
    (576, 2304, [399], "64x128", "32x32"),
    (576, 704, [257, 129, 257, 257, 254], "64x128", "64x64"),
    (320, 2048, [30, 59, 57, 30, 60, 60, 60, 0], "64x128", "32x32"),
    (320, 704, [0, 399, 397], "128x64", "32x64"),
    (2112, 512, [400, 397, 0, 400, 400], "128x64", "128x256"),
    (1024, 1472, [200, 399, 200], "128x128", "64x64"),
    (128, 704, [510, 513, 513], "128x128", "32x32"),
    (576, 2304, [513, 510, 0], "128x256", "64x64"),
    (192, 2304, [400, 397], "128x256", "32x32"),
]
# One block dispatches up to 4096 pairs, and a second one chooses the shapes;
# beyond, the scatter plans the GEMMs in a block of its own, from the histogram
# in each of its forms.
FORWARDS = CASES[::4] + [CASES[9], CASES[10], CASES[17]] + [
    (128, 192, [241] * 18, "128x64", "64x64"),
    (128, 128, [0] * 20 + [97, 96, 31, 1] * 22, "32", "128x64"),
    (192, 128, [33] * 130, "256", "256"),
    (128, 128, [5] * 900, "32", "32"),
    (128, 128, [400] * 60, "128x256", "128x128"),
    (192, 128, [1, 0, 70, 500] * 70, "128x256", "256"),
]


def _weights(S, d, I, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    w13 = (torch.randn((S, 2 * I, d), generator=g, device=DEV) * 0.05).to(torch.bfloat16)
    w2 = (torch.randn((S, d, I), generator=g, device=DEV) * 0.05).to(torch.bfloat16)
    return w13, w2, g


def _bits(t):
    return t.view(torch.int16)


def test_the_grid_is_the_one_the_shapes_are_named_for():
    assert torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8 == 256


@pytest.mark.parametrize("i", range(len(CASES)))
def test_every_shape_gives_the_bits_of_the_full_tiles(i):
    d, I, counts = CASES[i][:3]
    print(f"[gpu] gemm shapes d={d} I={I} counts={counts}", flush=True)
    S, P = len(counts), sum(counts)
    w13, w2, g = _weights(S, d, I, i)
    x = torch.randn((P, d), generator=g, device=DEV).to(torch.bfloat16)
    off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device=DEV)
    spare = 40  # rows past P must not be written
    outs = []
    for policy in (tg.TILES_AUTO, tg.TILES_FULL):
        h = torch.full((P + spare, I), -7.0, dtype=torch.bfloat16, device=DEV)
        y = torch.full((P + spare, d), -7.0, dtype=torch.bfloat16, device=DEV)
        with tg.tile_policy(policy):
            tg.tg_expert_ffn_grouped(x, off, S, P + spare, w13, w2, d, I, h, y)
        torch.cuda.synchronize()
        outs.append((h, y))
    for a, b in zip(*outs):
        assert torch.equal(_bits(a), _bits(b))
        assert (a[P:] == -7.0).all()
    if i == 13:
        at = 0
        for s, c in enumerate(counts):
            h, y = O.expert_ffn(u16(x[at:at + c]), u16(w13[s]), u16(w2[s]))
            assert_close_bf16(u16(outs[0][1][at:at + c]), y, f"slot {s}")
            at += c


@pytest.mark.parametrize("d,I,counts", [c[:3] for c in FORWARDS])
def test_the_forward_plans_its_gemms_as_the_full_tiles(d, I, counts):
    print(f"[gpu] gemm shapes in the forward d={d} I={I} S={len(counts)} P={sum(counts)}", flush=True)
    E, T = len(counts), sum(counts)
    wl = synth.make_custom(T=T, d=d, E=E, k=1, I=I, n_local=E, shadow_experts=[], gate="logits",
                           seed=d + I + E, device=DEV)
    expert = np.random.default_rng(3).permutation(np.repeat(np.arange(E), counts))
    wl.logits.fill_(-1.0)
    wl.logits[torch.arange(T, device=DEV), torch.from_numpy(expert).to(DEV)] = 1.0
    outs = []
    for policy in (tg.TILES_AUTO, tg.TILES_FULL):
        f = tg.EwForward(wl, keep_y=True)
        f.y.fill_(-7.0)
        with tg.tile_policy(policy):
            f()
        torch.cuda.synchronize()
        assert f.slot_counts.tolist() == counts
        outs.append(f)
    assert torch.equal(_bits(outs[0].y), _bits(outs[1].y))
    assert torch.equal(_bits(outs[0].out), _bits(outs[1].out))
    assert not (outs[0].y == -7.0).all(dim=1).any()
