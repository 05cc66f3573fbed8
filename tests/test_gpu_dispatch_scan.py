"""Dispatch in chunks (beyond 4096 pairs; chunks of 256 pairs, at most 256 of
them), where every scatter block scans the histogram: as it lies (up to 1024
entries and 32 chunks), or one, two or four chunks per lane, slots in groups of
64, 32 or 16. Routing, counts, offsets and rows bit
for bit against the oracle."""
import numpy as np
import pytest
import torch

from oracle import moe_ew as O
from paper_2601_01310_amd import tg
from tests._util import host

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("T,k,S", [(8192, 8, 64), (8192, 8, 65), (8190, 8, 3), (2731, 6, 250),
                                   (2731, 6, 256), (4097, 1, 1), (4097, 1, 1000), (700, 7, 40),
                                   (16384, 8, 40),
                                   # 64 | 65, 128 | 129 chunks
                                   (2048, 8, 63), (2048, 8, 1000), (16385, 1, 129), (4096, 8, 33),
                                   (4096, 8, 1024), (32769, 1, 17), (5462, 6, 1000), (13107, 5, 256),
                                   # 32 | 33 chunks, 1024 | more entries
                                   (1024, 8, 32), (1024, 8, 33), (8193, 1, 31), (4352, 1, 60), (4352, 1, 61)])
def test_dispatch_matches_the_oracle(T, k, S):
    print(f"[gpu] dispatch scan T={T} k={k} S={S}", flush=True)
    rng = np.random.default_rng(T + S)
    E = max(S, 8)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32) if E <= 300 else \
        rng.integers(0, E, (T, k)).astype(np.int32)
    ert = np.full((E, 2), -1, np.int32)
    ert[:S, 0] = rng.permutation(S)
    ert[:S // 2, 1] = rng.integers(0, S, S // 2)
    alive = (rng.random(S) > 0.2).astype(np.uint8)
    dev = {n: torch.from_numpy(v).to(DEV) for n, v in dict(ids=ids, ert=ert, alive=alive).items()}
    i32 = dict(dtype=torch.int32, device=DEV)
    slot, row = torch.empty((T, k), **i32), torch.empty((T, k), **i32)
    counts, offsets, nu = torch.empty(S, **i32), torch.empty(S + 1, **i32), torch.empty(1, **i32)
    perm = torch.full((T * k,), -7, **i32)
    nbytes = tg.tg_remap_dispatch_workspace(T, k, S)
    ws = tg.workspace(nbytes, DEV)
    tg.tg_remap_dispatch(dev["ids"], T, k, dev["ert"], E, 2, dev["alive"], S, None, 64, slot, counts,
                         offsets, perm, row, None, nu, ws, nbytes)
    torch.cuda.synchronize()
    r_slot, r_nu = O.remap(ids, ert, alive)
    r_counts, r_offsets, r_perm, r_row = O.dispatch(r_slot, S)
    assert np.array_equal(host(slot), r_slot) and int(nu[0]) == r_nu
    assert np.array_equal(host(counts), r_counts) and np.array_equal(host(offsets), r_offsets)
    P = int(r_offsets[-1])
    assert np.array_equal(host(perm)[:P], r_perm) and (host(perm)[P:] == -7).all()
    assert np.array_equal(host(row), r_row)
