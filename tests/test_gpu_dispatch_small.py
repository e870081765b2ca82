"""Dispatch around the route count (2048) up to which every block counts all the
routes itself instead of reading an earlier launch's histograms: exact against
the oracle, ghost routes included, and ids outside [0, E_r), which count as ghosts."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2606_19025_amd import binding as B

from .parity_helpers import canary, host, say

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (5, 8, 3), (33, 2, 256), (256, 8, 16), (257, 8, 16), (2048, 1, 256),
          (2049, 1, 7), (682, 3, 4), (683, 3, 4), (300, 6, 0)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,k,E_r", SHAPES)
def test_dispatch_small(gpu_lib, T, k, E_r, dtype):
    say(f"[dispatch] T={T} k={k} E_r={E_r} {dtype}")
    g = np.random.default_rng([T, k, E_r])
    E, d = max(2 * E_r, k + 1), 72
    idx = np.argsort(g.random((T, E)), axis=1)[:, :k]
    ghost = g.choice([-1, -1, -7, -2 ** 31, E_r, E_r + 1, 256, 300, 2 ** 31 - 1], size=idx.shape)
    local = np.where(idx < E_r, idx, np.where((ghost >= 0) & (ghost < E_r), -1, ghost)).astype(np.int32)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.from_numpy(g.standard_normal((T, d)).astype(np.float32)).to(dt)
    cap = T * min(k, E_r)
    i32 = torch.int32
    counts = torch.full((max(E_r, 1),), -7, dtype=i32, device="cuda")
    offsets = torch.full((E_r + 1,), -7, dtype=i32, device="cuda")
    perm = torch.full((max(cap, 1),), -7, dtype=i32, device="cuda")
    inv = torch.full((T, k), -7, dtype=i32, device="cuda")
    xp = canary(max(cap, 1), d, dtype=dt)
    n_ws = B.moe_dispatch_workspace_size(T, k, E_r)
    ws = torch.full((n_ws,), 0xFF, dtype=torch.uint8, device="cuda")
    B.moe_dispatch(x.cuda(), B.MOE_BF16 if dtype == "bf16" else B.MOE_F32, T, d, k, E_r, torch.from_numpy(local).cuda(),
                   counts, offsets, perm, inv, xp, ws, n_ws)
    torch.cuda.synchronize()
    ref = O.dispatch_plan(np.where(local < E_r, np.maximum(local, -1), -1), E_r)
    n = int(ref["offsets"][-1])
    assert np.array_equal(host(offsets), ref["offsets"])
    assert np.array_equal(host(counts)[:E_r], ref["counts"])
    assert np.array_equal(host(perm)[:n], ref["perm"][:n])
    assert np.array_equal(host(inv), ref["inv_perm"])
    assert torch.equal(xp[:n].cpu(), x[torch.from_numpy(ref["perm"][:n] // k).long()])
    assert torch.isnan(xp[n:]).all() and (perm[n:] == -7).all()
