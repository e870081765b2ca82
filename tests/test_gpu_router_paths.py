"""Router forward and backward through the C ABI against the oracle, at the
shapes that select each kernel path: fp32 with 16-byte aligned rows and
without (odd d, or a base that is only 4-byte aligned), bf16 with more than 64
experts, one to eight 32-expert groups, last slices and column blocks cut
short, one chunk of tokens (whose sums are the results) and several, more than
64 routes per token, d_bias not wanted, an unaligned dW.

Logits, dz, dW and d_bias are fp32 sums (1e-5 normwise, as the fp32 layers); a
bf16 dx adds its own rounding (2^-9 of each value, 2^-8 accumulated).
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2606_19025_amd import binding as B
from paper_2606_19025_amd import inputs as I

from .parity_helpers import TOL, assert_close, dev, host, record_errors, say

pytestmark = pytest.mark.gpu

F32, I32 = torch.float32, torch.int32


def _unaligned(a):
    """a on the GPU at an address that is a multiple of 4 but not of 16."""
    buf = torch.full((a.size + 1,), float("nan"), dtype=F32, device="cuda")
    buf[1:] = dev(a.reshape(-1), F32)
    return buf[1:].view(a.shape)


def _inputs(T, d, E, dtype):
    g = np.random.default_rng([T, d, E])
    x, w = g.standard_normal((T, d)).astype(np.float32), (g.standard_normal((E, d)) * 0.05).astype(np.float32)
    if dtype == "bf16":
        x, w = I.bf16_round(x), I.bf16_round(w)
    return g, x, w


# dtype, T, d, E, k, base aligned
FWD = [("f32", 70, 72, 10, 3, True), ("f32", 33, 37, 40, 2, True), ("f32", 64, 160, 64, 6, False),
       ("f32", 31, 1096, 65, 8, True), ("f32", 5, 1, 200, 9, False), ("f32", 40, 260, 256, 8, True),
       ("bf16", 70, 8, 65, 4, True), ("bf16", 100, 1544, 128, 8, True), ("bf16", 45, 200, 130, 5, True),
       ("bf16", 33, 2056, 256, 70, True)]


@pytest.mark.parametrize("dtype,T,d,E,k,aligned", FWD)
def test_router_forward(gpu_lib, dtype, T, d, E, k, aligned):
    say(f"[router-fwd] {dtype} T={T} d={d} E={E} k={k} aligned={aligned}")
    g, x, w = _inputs(T, d, E, dtype)
    bias = (g.standard_normal(E) * 0.1).astype(np.float32)
    res = np.zeros(E, np.uint8)
    res[g.choice(E, max(1, E // 2), replace=False)] = 1
    dt = torch.bfloat16 if dtype == "bf16" else F32
    tx, tw_ = (dev(x, dt), dev(w, dt)) if aligned else (_unaligned(x), _unaligned(w))
    logits = torch.full((T, E), float("nan"), dtype=F32, device="cuda")
    idx = torch.full((T, k), -7, dtype=I32, device="cuda")
    loc = torch.full_like(idx, -7)
    wts = torch.full((T, k), float("nan"), dtype=F32, device="cuda")
    B.moe_route_mask(tx, tw_, dev(bias, F32), B.MOE_BF16 if dtype == "bf16" else B.MOE_F32, T, d, E,
                     k, 0.8, B.GATES["softmax"], torch.from_numpy(res).cuda(), logits, idx, wts, loc)
    torch.cuda.synchronize()
    z = host(logits)
    e = assert_close("logits", z, O.router_logits(x, w, 0.8, bias), TOL["f32"])
    record_errors(f"router_fwd[{dtype} {T} {d} {E}]", {"logits": e})
    ref = O.topk_select(z, k)
    assert np.array_equal(host(idx), ref)
    rank = np.cumsum(res.astype(np.int64)) - 1
    assert np.array_equal(host(loc), np.where(res[ref] == 1, rank[ref], -1))
    np.testing.assert_allclose(host(wts), O.gate_weights(z, ref, "softmax"), rtol=2e-6, atol=1e-7)


def _chain(x, w):
    """x w^T in fp32, each logit one chain of fused multiply-adds in the order of d.
    (A product and its sum in 64 mantissa bits, then rounded to 24: the fused
    result, but for one step in some 2^40.)"""
    x, w = x.astype(np.longdouble), w.astype(np.longdouble)
    s = np.zeros((x.shape[0], w.shape[0]), np.float32)
    for c in range(x.shape[1]):
        s = (x[:, c, None] * w[None, :, c] + s).astype(np.float32)
    return s


# as FWD's, and one and two tiles of 16 experts, more stages than the ring holds
@pytest.mark.parametrize("T,d,E,aligned", [(f[1], f[2], f[3], f[5]) for f in FWD if f[0] == "f32"]
                         + [(50, 64, 8, True), (96, 516, 32, True), (33, 1030, 17, True),
                            (40, 132, 128, False), (17, 900, 129, True)])
def test_f32_logits_are_bitwise_a_serial_chain(gpu_lib, T, d, E, aligned):
    """Another order of the sum moves logits by a rounding, and two of one token
    that lie that close then change ranks: selections, gates and whole rows of the
    gradients would depend on the kernel's split of d."""
    say(f"[router-chain] T={T} d={d} E={E} aligned={aligned}")
    g, x, w = _inputs(T, d, E, "f32")
    bias = (g.standard_normal(E) * 0.1).astype(np.float32)
    tx, tw_ = (dev(x, F32), dev(w, F32)) if aligned else (_unaligned(x), _unaligned(w))
    z = _logits(tx, tw_, dev(bias, F32), 0.8)
    want = (_chain(x, w) + bias) * np.float32(0.8)
    assert np.array_equal(z.cpu().numpy(), want)


@pytest.mark.parametrize("T,d,E", [(70, 8, 65), (45, 200, 130), (33, 1544, 128), (20, 2056, 256),
                                   (9, 4160, 100)])
def test_bf16_logits_do_not_depend_on_the_number_of_experts(gpu_lib, T, d, E):
    """More than 64 experts take another kernel path; it adds in the same order (see
    above), so each 40 experts by themselves have bitwise the same logits."""
    say(f"[router-experts] T={T} d={d} E={E}")
    _, x, w = _inputs(T, d, E, "bf16")
    tx, tw_ = dev(x, torch.bfloat16), dev(w, torch.bfloat16)
    z = _logits(tx, tw_, None, 1.0)
    for e in range(0, E, 40):
        some = tw_[e:e + 40]
        assert torch.equal(_logits(tx, some, None, 1.0), z[:, e:e + 40]), e


def _logits(x, w, bias, tau):
    (T, d), E = x.shape, w.shape[0]
    z = torch.full((T, E), float("nan"), dtype=F32, device="cuda")
    idx, loc = (torch.empty((T, 1), dtype=I32, device="cuda") for _ in range(2))
    B.moe_route_mask(x, w, bias, B.dtype_code(x), T, d, E, 1, tau, B.GATES["softmax_topk"],
                     torch.ones(E, dtype=torch.uint8, device="cuda"), z, idx,
                     torch.empty((T, 1), dtype=F32, device="cuda"), loc)
    torch.cuda.synchronize()
    return z


# dtype, T, d, E, k, gate, accumulate_dx, d_bias wanted, dW aligned
BWD = [("f32", 70, 72, 10, 3, "softmax_topk", 1, True, True), ("f32", 256, 8, 16, 2, "sigmoid", 0, True, True),
       ("f32", 300, 200, 50, 4, "softmax", 0, True, True), ("f32", 600, 136, 100, 8, "softmax_topk", 1, True, False),
       ("f32", 65, 320, 256, 70, "softmax", 0, True, True), ("f32", 200, 64, 7, 2, "softmax_topk", 1, False, True),
       ("bf16", 70, 72, 10, 3, "softmax_topk", 1, True, True), ("bf16", 700, 200, 64, 6, "softmax", 0, True, True),
       ("bf16", 300, 256, 33, 4, "sigmoid", 1, True, True), ("bf16", 90, 256, 64, 4, "softmax_topk", 0, False, False),
       ("bf16", 300, 136, 65, 4, "softmax_topk", 1, True, True), ("bf16", 64, 64, 128, 8, "softmax", 0, True, True),
       ("bf16", 1000, 584, 255, 8, "softmax", 1, True, True), ("bf16", 129, 72, 256, 66, "sigmoid", 0, False, True)]


@pytest.mark.parametrize("dtype,T,d,E,k,gate,acc,want_bias,aligned", BWD)
def test_router_backward(gpu_lib, dtype, T, d, E, k, gate, acc, want_bias, aligned):
    say(f"[router-bwd] {dtype} T={T} d={d} E={E} k={k} {gate} acc={acc}")
    g, x, w = _inputs(T, d, E, dtype)
    tau = 0.7
    z = O.router_logits(x, w, tau).astype(np.float32)
    idx = O.topk_select(z, k)
    wts = O.gate_weights(z, idx, gate).astype(np.float32)
    dtw = g.standard_normal((T, k)).astype(np.float32)
    dx0 = g.standard_normal((T, d)).astype(np.float32)
    dt = torch.bfloat16 if dtype == "bf16" else F32
    if dtype == "bf16":
        dx0 = I.bf16_round(dx0)
    ws_bytes = B.moe_route_bwd_workspace_size(T, d, E)
    ws = torch.full((ws_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    dz = torch.full((T, E), float("nan"), dtype=F32, device="cuda")
    dw = torch.full((E, d), float("nan"), dtype=F32, device="cuda")
    if not aligned:
        dw = _unaligned(np.full((E, d), np.nan, np.float32))
    db = torch.full((E,), float("nan"), dtype=F32, device="cuda")
    dx = dev(dx0, dt) if acc else torch.full((T, d), float("nan"), dtype=dt, device="cuda")
    B.moe_route_bwd(dev(x, dt), dev(w, dt), B.MOE_BF16 if dtype == "bf16" else B.MOE_F32, T, d, E, k,
                    tau, B.GATES[gate], torch.from_numpy(idx.astype(np.int32)).cuda(), dev(wts, F32),
                    dev(z, F32), dev(dtw, F32), dz, dw, db if want_bias else None, dx, acc, ws, ws_bytes)
    torch.cuda.synchronize()
    ref = O.route_bwd(x, w, idx, wts, z, dtw, tau, gate)
    errs = {"dz": assert_close("dz", host(dz), ref["dz"], TOL["f32"]),
            "dW": assert_close("dW", host(dw), ref["dW_router"], TOL["f32"])}
    if want_bias:
        errs["db"] = assert_close("d_bias", host(db), ref["d_bias"], TOL["f32"])
    else:
        assert torch.isnan(db).all()
    want = ref["dx"] + (dx0 if acc else 0.0)
    errs["dx"] = assert_close("dx", host(dx), want, TOL["f32"] if dtype == "f32" else 2.0 ** -8)
    record_errors(f"router_bwd[{dtype} {T} {d} {E} {gate}]", errs)


@pytest.mark.parametrize("gate", ["sigmoid", "softmax"])
@pytest.mark.parametrize("T,d,E", [(70, 72, 10), (300, 136, 64), (300, 136, 65), (129, 72, 256)])
def test_router_backward_keeps_infinities(gpu_lib, T, d, E, gate):
    """bf16 layers that take dz in three parts: an infinite upstream gradient, x or
    W_r gives the infinities and NaNs of plain sums of products, and no others."""
    say(f"[router-inf] T={T} d={d} E={E} {gate}")
    g, x, w = _inputs(T, d, E, "bf16")
    k, inf = 3, np.inf
    z = O.router_logits(x, w, 1.0).astype(np.float32)
    idx = O.topk_select(z, k)
    wts = O.gate_weights(z, idx, gate).astype(np.float32)
    dtw = g.standard_normal((T, k)).astype(np.float32)
    if gate == "sigmoid":  # (the others' dz of such a token is infinite or NaN throughout)
        dtw[T // 2, 1], dtw[T - 1, 0] = inf, -inf
    x[3, 5], x[T - 2, d - 1], w[E - 1, 9], w[E // 2, d - 7] = inf, -inf, inf, -inf
    bf = torch.bfloat16
    n_ws = B.moe_route_bwd_workspace_size(T, d, E)
    dz, dw, db = (torch.empty(s, dtype=F32, device="cuda") for s in ((T, E), (E, d), (E,)))
    dx = torch.empty((T, d), dtype=bf, device="cuda")
    B.moe_route_bwd(dev(x, bf), dev(w, bf), B.MOE_BF16, T, d, E, k, 1.0, B.GATES[gate],
                    torch.from_numpy(idx.astype(np.int32)).cuda(), dev(wts, F32), dev(z, F32),
                    dev(dtw, F32), dz, dw, db, dx, 0, torch.empty(n_ws, dtype=torch.uint8, device="cuda"), n_ws)
    torch.cuda.synchronize()
    # (dz itself is elementwise and fp32: the sums are checked on the call's own)
    z64 = host(dz)
    assert np.isinf(z64).any() == (gate == "sigmoid")
    with np.errstate(invalid="ignore"):
        want = {"dW": (dw, z64.T @ x.astype(np.float64), TOL["f32"]), "d_bias": (db, z64.sum(0), TOL["f32"]),
                "dx": (dx, z64 @ w.astype(np.float64), 2.0 ** -8)}
    for name, (got, ref, tol) in want.items():
        got = host(got)
        assert np.array_equal(np.isnan(got), np.isnan(ref)), name
        fin = np.isfinite(ref)
        assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]), name
        assert name == "d_bias" or (fin.any() and np.isinf(ref).any()), name
        if fin.any():
            assert_close(name, got[fin], ref[fin], tol)
