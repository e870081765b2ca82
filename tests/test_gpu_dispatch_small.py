"""Dispatch around the route count (2048) up to which every block counts all the
routes itself instead of reading an earlier launch's histograms: exact against
the oracle, ghost routes and out-of-range ids included."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2606_19025_amd import binding as B

from .parity_helpers import canary, host, say

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (5, 8, 3), (33, 2, 256), (256, 8, 16), (257, 8, 16), (2048, 1, 256),
          (2049, 1, 7), (682, 3, 4), (683, 3, 4), (300, 6, 0)]


@pytest.mark.parametrize("T,k,E_r", SHAPES)
def test_dispatch_small(gpu_lib, T, k, E_r):
    say(f"[dispatch] T={T} k={k} E_r={E_r}")
    g = np.random.default_rng([T, k, E_r])
    E, d = max(2 * E_r, k + 1), 72
    idx = np.argsort(g.random((T, E)), axis=1)[:, :k]
    local = np.where(idx < E_r, idx, -1).astype(np.int32)
    x = g.standard_normal((T, d)).astype(np.float32)
    cap = T * min(k, E_r)
    i32 = torch.int32
    counts = torch.full((max(E_r, 1),), -7, dtype=i32, device="cuda")
    offsets = torch.full((E_r + 1,), -7, dtype=i32, device="cuda")
    perm = torch.full((max(cap, 1),), -7, dtype=i32, device="cuda")
    inv = torch.full((T, k), -7, dtype=i32, device="cuda")
    xp = canary(max(cap, 1), d, dtype=torch.float32)
    n_ws = B.moe_dispatch_workspace_size(T, k, E_r)
    ws = torch.full((n_ws,), 0xFF, dtype=torch.uint8, device="cuda")
    B.moe_dispatch(torch.from_numpy(x).cuda(), B.MOE_F32, T, d, k, E_r, torch.from_numpy(local).cuda(),
                   counts, offsets, perm, inv, xp, ws, n_ws)
    torch.cuda.synchronize()
    ref = O.dispatch_plan(local, E_r)
    n = int(ref["offsets"][-1])
    assert np.array_equal(host(offsets), ref["offsets"])
    assert np.array_equal(host(counts)[:E_r], ref["counts"])
    assert np.array_equal(host(perm)[:n], ref["perm"][:n])
    assert np.array_equal(host(inv), ref["inv_perm"])
    assert np.array_equal(xp[:n].cpu().numpy(), x[ref["perm"][:n] // k])
    assert torch.isnan(xp[n:]).all() and (perm[n:] == -7).all()
