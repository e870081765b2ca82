"""The bf16 grouped FFN in each of its tile sizes against the oracle.

A launch takes 256 x 256, 64 x 128, 64 x 64 or 32 x 64 tiles by an estimate of
its time.  The timing names tell the large tiles from the small ones; the
shapes here reach every kind in both, with group sizes at the edges of the
tile heights (empty, 1, 31..33, 63..65, 127..129, 255..257, 511, 513 rows),
partial column tiles, ragged K of the weight gradients, both expert forms, one
and two sets, with and without a workspace, accumulated gradients, reductions cut
into parts (by rows, by K) and a first group that does not start at row 0.  The
tolerance is the bf16 layers' own, normwise.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2606_19025_amd import binding as B
from paper_2606_19025_amd import inputs as I

from .parity_helpers import TOL, assert_close, canary, host, record_errors, say

pytestmark = pytest.mark.gpu

F32 = torch.float32
LARGE = [0, 1, 127, 128, 129, 0, 255, 256, 257, 383, 511, 513, 1300, 2001, 0]
# name: (group sizes of each set, d, H of each set, expert, workspace, accumulate_dw, large launches)
CASES = {
    "all-large": ([LARGE], 2240, [1984], "swiglu", True, 1, "1111"),
    "all-large-silu": ([LARGE], 2240, [1984], "silu", False, 0, "1111"),
    "rows-32": ([[0, 1, 31, 32, 33, 2, 0]], 192, [320], "swiglu", True, 0, "0000"),
    "rows-32-silu-shared": ([[7, 0, 30, 5], [42]], 128, [192, 448], "silu", False, 1, "0000"),
    "rows-64": ([[63, 64, 65, 0, 127, 129, 1, 200]], 320, [704], "swiglu", True, 0, "0000"),
    "rows-64-silu": ([[500, 3, 65, 0, 129]], 1088, [192], "silu", True, 1, "0000"),
    "rows-64-shared": ([[260, 90, 0, 511], [861]], 448, [576, 1152], "swiglu", True, 0, "0000"),
    # more than eight uneven groups, whose weight-gradient tiles each XCD shares
    "many-uneven-groups": ([[5 * (i % 17) if i % 9 else 300 for i in range(70)]], 192, [192],
                           "swiglu", True, 1, "0000"),
    "many-groups": ([[5 * (i % 17) for i in range(70)]], 64, [64], "swiglu", True, 0, "0000"),
    # the same in the large tiles, whose uneven groups are shared out by time
    "many-uneven-groups-large": ([[600 if i % 9 == 0 else 190 + i for i in range(70)]], 704, [832],
                                 "swiglu", True, 0, "1111"),
    # one group's weight gradients cut by rows into parts, and their sum
    "one-group-split": ([[8532]], 256, [256], "swiglu", True, 0, "0010"),
    "one-group-split-silu-acc": ([[8626]], 192, [192], "silu", True, 1, "0011"),
    # few tiles with a long reduction: dX in K parts
    "k-parts": ([[300, 0, 109]], 192, [3328], "swiglu", True, 0, "0001"),
    "k-parts-shared": ([[100, 0, 270, 10], [132]], 256, [2432, 4864], "swiglu", True, 1, "0001"),
    # the down projection too
    "k-parts-down": ([[60, 0, 30, 9], [962]], 512, [4224, 8448], "silu", True, 0, "1110"),
    # the first group does not start at row 0
    "lead-small": ([[63, 64, 0, 129, 144]], 320, [704], "silu", True, 0, "0000"),
    "lead-large": ([LARGE], 2240, [1984], "swiglu", True, 0, "1111"),
    "lead-k-parts": ([[300, 0, 109]], 192, [3328], "swiglu", True, 1, "0001"),
}
LEAD = {"lead-small": 40, "lead-large": 37, "lead-k-parts": 5}  # rows before the first group
# other kernels that have to run
ALSO = {"one-group-split": "splitk_reduce", "one-group-split-silu-acc": "splitk_reduce",
        "k-parts": "splitk_rows_reduce", "k-parts-shared": "splitk_rows_reduce",
        "k-parts-down": "splitk_rows_reduce", "lead-k-parts": "splitk_rows_reduce"}


@pytest.mark.parametrize("name", sorted(CASES))
def test_ffn_tile_sizes(gpu_lib, name):
    set_sizes, d, Hs, expert, use_ws, acc, large = CASES[name]
    say(f"[gemm-tiles] {name}")
    g = np.random.default_rng([31, d, Hs[0]])
    r1 = 2 if expert == "swiglu" else 1
    act = B.ACTIVATIONS[expert]

    def draw(*shape, std=1.0):
        return I.bf16_round(g.standard_normal(shape, dtype=np.float32) * np.float32(std))

    def dev(a, dt=torch.bfloat16):
        return torch.from_numpy(a).cuda().to(dt)

    sets, state = [], []
    for sizes, H in zip(set_sizes, Hs):
        G, n = len(sizes), sum(sizes)
        lead = LEAD.get(name, 0)
        cap = lead + n + 70 if len(sizes) > 1 else n  # rows outside the groups stay untouched
        off = (lead + np.concatenate([[0], np.cumsum(sizes)])).astype(np.int32)
        s = dict(sizes=sizes, H=H, n=n, off=off, xp=draw(cap, d), dyp=draw(cap, d),
                 w1=draw(G, r1 * H, d, std=d ** -0.5), w2=draw(G, d, H, std=H ** -0.5))
        for key, shape in (("dw1", (G, r1 * H, d)), ("dw2", (G, d, H))):
            s[key] = (g.standard_normal(shape) * 0.01).astype(np.float32) if acc else None
        t = {k: dev(s[k]) for k in ("xp", "dyp", "w1", "w2")}
        t.update(off=torch.from_numpy(off).cuda(), gu=canary(cap, r1 * H), h=canary(cap, H),
                 yp=canary(cap, d), dgu=canary(cap, r1 * H), dxp=canary(cap, d),
                 dw1=dev(s["dw1"], F32) if acc else canary(G, r1 * H, d, dtype=F32),
                 dw2=dev(s["dw2"], F32) if acc else canary(G, d, H, dtype=F32))
        sets.append(B.ffn_set(t["xp"], t["w1"], t["w2"], t["off"], cap, H, G, t["gu"], t["h"],
                              yp=t["yp"], dyp=t["dyp"], dgu=t["dgu"], dxp=t["dxp"],
                              dw_gate_up=t["dw1"], dw_down=t["dw2"], activation=act))
        state.append((s, t))
    ws = {}
    for way, size in (("fwd", B.moe_grouped_ffn_fwd_workspace_size),
                      ("bwd", B.moe_grouped_ffn_bwd_workspace_size)):
        n = size(sets, B.MOE_BF16, d) if use_ws else 0
        ws[way] = (torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda") if n else None, n)
    B.moe_timing_enable(64)
    try:
        B.moe_grouped_ffn_fwd_sets(sets, B.MOE_BF16, d, *ws["fwd"])
        B.moe_grouped_ffn_bwd_sets(sets, B.MOE_BF16, d, acc, *ws["bwd"])
        ran = set(B.moe_timing_collect())
    finally:
        B.moe_timing_enable(0)
    kinds = (("gemm_gu_fwd", "gemm_down_fwd", "gemm_dhh_dwd", "gemm_dx_dwgu") if expert == "swiglu"
             else ("gemm_up_fwd", "gemm_down_fwd", "gemm_dh_dwd", "gemm_dx_dwgu"))
    got = "".join("1" if k in ran else "0" for k in kinds)
    assert all((k in ran) != (k + "_tile" in ran) for k in kinds), ran
    assert got == large, f"large tiles in {got}, expected {large}"
    assert name not in ALSO or ALSO[name] in ran, ran

    tol, errs = TOL["bf16"], {}
    for i, (s, t) in enumerate(state):
        H, lead = s["H"], int(s["off"][0])
        at, off = slice(lead, lead + s["n"]), s["off"] - lead  # the groups' rows
        f = O.grouped_ffn_fwd(s["xp"][at], off, s["w1"], s["w2"], expert)
        b = O.grouped_ffn_bwd(s["dyp"][at], s["xp"][at], f["G"], f["U"], f["Hh"], off,
                              s["w1"], s["w2"], expert)
        gu, dgu = host(t["gu"]), host(t["dgu"])
        pairs = [("G", gu[at, :H], f["G"]), ("h", host(t["h"])[at], f["Hh"]),
                 ("yp", host(t["yp"])[at], f["Y"]), ("dG", dgu[at, :H], b["dG"]),
                 ("dxp", host(t["dxp"])[at], b["dXp"])]
        if expert == "swiglu":
            pairs += [("U", gu[at, H:], f["U"]), ("dU", dgu[at, H:], b["dU"])]
        for key, value, want in pairs:
            errs[f"{key}{i}"] = assert_close(key, value, want, tol)
        for key in ("gu", "h", "yp", "dgu", "dxp"):
            assert torch.isnan(t[key][at.stop:]).all(), f"{key}: a row past the groups was written"
            assert torch.isnan(t[key][:lead]).all(), f"{key}: a row before the groups was written"
        for key, want in (("dw1", b["dW_gate_up"]), ("dw2", b["dW_down"])):
            value = host(t[key])
            for r, sz in enumerate(s["sizes"]):
                w = want[r] + (s[key][r] if acc else 0.0)
                if sz == 0:
                    assert np.array_equal(value[r], w), f"{key} of empty group {r}"
                else:
                    errs[f"{key}.{i}.{r}"] = assert_close(f"{key}[{r}]", value[r], w, tol)
    record_errors(f"gemm_tiles[{name}]", errs)


# groups, rows of each, d, H, direction, kernels that must run and must not: where
# the wrong size took a fifth to four fifths longer than the right one
CHOICES = [
    (16, 200, 2048, 1408, "fwd", {"gemm_gu_fwd"}, {"gemm_gu_fwd_tile"}),
    (8, 300, 4096, 2048, "fwd", {"gemm_gu_fwd", "gemm_down_fwd"}, {"gemm_gu_fwd_tile", "gemm_down_fwd_tile"}),
    (8, 32, 1024, 2816, "bwd", {"gemm_dx_dwgu", "splitk_rows_reduce"}, {"gemm_dx_dwgu_tile"}),
    (12, 80, 768, 704, "fwd", {"gemm_gu_fwd_tile", "gemm_down_fwd_tile"}, {"gemm_gu_fwd", "gemm_down_fwd"}),
    (12, 80, 768, 704, "bwd", {"gemm_dhh_dwd_tile", "gemm_dx_dwgu_tile"}, {"gemm_dhh_dwd", "gemm_dx_dwgu"}),
]


@pytest.mark.parametrize("G,rows,d,H,way,runs,not_", CHOICES)
def test_choice_where_every_row_is_present(gpu_lib, G, rows, d, H, way, runs, not_):
    """A direct call fills the bound on its rows: the estimate has to hold there too."""
    say(f"[gemm-choice] {G} x {rows} rows d={d} H={H} {way}")
    n, bf = G * rows, torch.bfloat16

    def new(*shape, dt=bf):
        return torch.zeros(shape, dtype=dt, device="cuda")

    off = (torch.arange(G + 1, dtype=torch.int32) * rows).cuda()
    t = dict(yp=new(n, d))  # (a set holds addresses only)
    if way == "bwd":
        t.update(dyp=new(n, d), dgu=new(n, 2 * H), dxp=new(n, d), dw_gate_up=new(G, 2 * H, d, dt=F32),
                 dw_down=new(G, d, H, dt=F32))
    xp, w1, w2, gu, h = new(n, d), new(G, 2 * H, d), new(G, d, H), new(n, 2 * H), new(n, H)
    s = B.ffn_set(xp, w1, w2, off, n, H, G, gu, h, **t)
    size = B.moe_grouped_ffn_fwd_workspace_size if way == "fwd" else B.moe_grouped_ffn_bwd_workspace_size
    n_ws = size([s], B.MOE_BF16, d)
    ws = new(max(1, n_ws), dt=torch.uint8)
    B.moe_timing_enable(64)
    try:
        if way == "fwd":
            B.moe_grouped_ffn_fwd_sets([s], B.MOE_BF16, d, ws if n_ws else None, n_ws)
        else:
            B.moe_grouped_ffn_bwd_sets([s], B.MOE_BF16, d, 0, ws, n_ws)
        ran = set(B.moe_timing_collect())
    finally:
        B.moe_timing_enable(0)
    assert runs <= ran and not (not_ & ran), ran
