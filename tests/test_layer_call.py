"""moe_layer_fwd / moe_layer_bwd: a failed check is reported as the entry point's
own (CPU), and the results are those of the entry points called one by one (GPU)."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2606_19025_amd import binding as B


def _status(fn, layer):
    if torch.cuda.device_count() > 0:
        pytest.skip("host-only rejection test: runs where no GPU is visible")
    where = C.c_char_p()
    status = fn(None if layer is None else C.byref(layer), C.byref(where), None)
    return status, where.value.decode()


def test_layer_calls_report_the_failing_entry_point():
    lib = B.lib()
    for fn, first in ((lib.moe_layer_fwd, "moe_route_mask"), (lib.moe_layer_bwd, "moe_combine_bwd")):
        assert _status(fn, None) == (-1, fn.__name__)
        assert _status(fn, B.moe_layer(dtype=7)) == (-2, first)
        assert "dtype 7" in B.moe_last_error()
    # the forward's second entry point: its first launches nothing at T = 0
    p = 256  # a fake, never dereferenced address
    layer = B.moe_layer(dtype=B.MOE_F32, T=0, d=8, E=4, k=2, E_r=300, inv_tau=1.0, n_sets=1,
                        w_router=p, resident=p)
    assert _status(lib.moe_layer_fwd, layer) == (-1, "moe_dispatch")
    layer.E_r, layer.offsets, layer.counts = 2, p, p
    layer.ws_dispatch, layer.ws_dispatch_bytes = p, 0
    assert _status(lib.moe_layer_fwd, layer) == (-1, "moe_dispatch")
    assert "workspace" in B.moe_last_error()
    with pytest.raises(B.MoeError, match="moe_route_mask returned -2"):
        B.moe_layer_fwd(B.moe_layer(dtype=7), stream=0)


@pytest.mark.gpu
@pytest.mark.parametrize("shared", [0, 64])
def test_layer_call_equals_the_single_calls(gpu_lib, shared):
    from .parity_helpers import gpu_outputs, make_layer, run_gpu_layer
    from .test_gpu_parity import synth_inputs
    inp = synth_inputs(300, 128, 12, 3, 128, [0, 3, 5, 8], "bf16", seed=7, shared_hidden=shared)
    L, d_in = run_gpu_layer(inp)
    whole = gpu_outputs(L)
    M = make_layer(inp)
    args = [d_in[n] for n in ("x", "w_router", "w_gate_up", "w_down")]
    extra = {n: d_in.get(n) for n in ("shared_gate_up", "shared_down")}
    calls = []
    M.forward(*args, router_bias=d_in["router_bias"], hook=lambda: calls.append(0), **extra)
    M.backward(d_in["dy"], *args, hook=lambda: calls.append(0), **extra)
    torch.cuda.synchronize()
    assert len(calls) == 8
    single = gpu_outputs(M)
    for key in whole:
        assert np.array_equal(whole[key], single[key]), key
