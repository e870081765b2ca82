"""Grouped expert FFN of fp32 layers (forward and backward) against the oracle,
with group sizes at the edges of the GEMM's 32- and 64-row tiles.

The kernel takes one of two tile sizes by the number of tiles; each is
reached here in every GEMM kind, with widths that leave partial column tiles,
K extents that are no multiple of its 32-deep k-steps, empty groups, both
expert forms, one and two sets per call, and accumulated weight gradients.
The tolerance is the fp32 layers' own (1e-5 normwise): products and sums are
fp32, over at most 4096 terms here.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2606_19025_amd import binding as B

from .parity_helpers import TOL, assert_close, canary, host, record_errors, say

pytestmark = pytest.mark.gpu

F32 = torch.float32
# name: (group sizes of each set, d, H of each set, expert, accumulate_dw)
CASES = {
    "small-tiles": ([[0, 1, 31, 32, 33, 0]], 8, [64], "swiglu", 0),
    "small-tiles-silu-two-sets": ([[5, 0, 40], [45]], 72, [64, 128], "silu", 1),
    "middle-tiles": ([[63, 64, 65, 0, 127, 129, 700, 1]], 520, [448], "swiglu", 1),
    "middle-tiles-silu": ([[300, 0, 511]], 264, [960], "silu", 0),
    # enough 64 x 128 tiles in GU, dHh + dW_d / in the down projection, dX + dW_gu
    "large-tiles-wide-hidden": ([[2047, 0, 129, 1601]], 72, [4096], "swiglu", 0),
    "large-tiles-wide-model": ([[1900, 127, 1801]], 4104, [64], "swiglu", 1),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_grouped_ffn_f32_tiles(gpu_lib, name):
    set_sizes, d, Hs, expert, acc = CASES[name]
    say(f"[grouped-ffn-f32] {name}")
    g = np.random.default_rng([29, d, Hs[0]])
    r1 = 2 if expert == "swiglu" else 1
    act = B.ACTIVATIONS[expert]

    def draw(*shape, std=1.0):
        return (g.standard_normal(shape) * std).astype(np.float32)

    def dev(a):
        return torch.from_numpy(a).cuda()

    sets, state = [], []
    for sizes, H in zip(set_sizes, Hs):
        G, n = len(sizes), sum(sizes)
        cap = n + 70  # rows past the groups stay untouched
        s = dict(sizes=sizes, H=H, n=n, off=np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32),
                 xp=draw(cap, d), dyp=draw(cap, d), w1=draw(G, r1 * H, d, std=d ** -0.5),
                 w2=draw(G, d, H, std=H ** -0.5))
        s["dw1_0"] = draw(G, r1 * H, d, std=0.01) if acc else None
        s["dw2_0"] = draw(G, d, H, std=0.01) if acc else None
        t = {k: dev(s[k]) for k in ("off", "xp", "dyp", "w1", "w2")}
        t.update(gu=canary(cap, r1 * H, dtype=F32), h=canary(cap, H, dtype=F32),
                 yp=canary(cap, d, dtype=F32), dgu=canary(cap, r1 * H, dtype=F32),
                 dxp=canary(cap, d, dtype=F32),
                 dw1=dev(s["dw1_0"]) if acc else canary(G, r1 * H, d, dtype=F32),
                 dw2=dev(s["dw2_0"]) if acc else canary(G, d, H, dtype=F32))
        sets.append(B.ffn_set(t["xp"], t["w1"], t["w2"], t["off"], cap, H, G, t["gu"], t["h"],
                              yp=t["yp"], dyp=t["dyp"], dgu=t["dgu"], dxp=t["dxp"],
                              dw_gate_up=t["dw1"], dw_down=t["dw2"], activation=act))
        state.append((s, t))
    B.moe_grouped_ffn_fwd_sets(sets, B.MOE_F32, d)
    B.moe_grouped_ffn_bwd_sets(sets, B.MOE_F32, d, acc)
    torch.cuda.synchronize()

    tol, errs = TOL["f32"], {}
    for i, (s, t) in enumerate(state):
        n, H = s["n"], s["H"]
        f = O.grouped_ffn_fwd(s["xp"][:n], s["off"], s["w1"], s["w2"], expert)
        b = O.grouped_ffn_bwd(s["dyp"][:n], s["xp"][:n], f["G"], f["U"], f["Hh"], s["off"],
                              s["w1"], s["w2"], expert)
        gu, dgu = host(t["gu"]), host(t["dgu"])
        pairs = [("G", gu[:n, :H], f["G"]), ("h", host(t["h"])[:n], f["Hh"]),
                 ("yp", host(t["yp"])[:n], f["Y"]), ("dG", dgu[:n, :H], b["dG"]),
                 ("dxp", host(t["dxp"])[:n], b["dXp"])]
        if expert == "swiglu":
            pairs += [("U", gu[:n, H:], f["U"]), ("dU", dgu[:n, H:], b["dU"])]
        for name_, got, want in pairs:
            errs[f"{name_}{i}"] = assert_close(name_, got, want, tol)
        for key in ("gu", "h", "yp", "dgu", "dxp"):
            assert torch.isnan(t[key][n:]).all(), f"{key}: a row past the groups was written"
        for key, want, first in (("dw1", b["dW_gate_up"], s["dw1_0"]),
                                 ("dw2", b["dW_down"], s["dw2_0"])):
            got = host(t[key])
            for r, sz in enumerate(s["sizes"]):
                w = want[r] + (first[r] if acc else 0.0)
                if sz == 0:
                    assert np.array_equal(got[r], w), f"{key} of empty group {r}"
                else:
                    errs[f"{key}.{i}.{r}"] = assert_close(f"{key}[{r}]", got[r], w, tol)
    record_errors(f"grouped_ffn_f32[{name}]", errs)
