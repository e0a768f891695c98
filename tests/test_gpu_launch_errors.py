"""A call that reads results back reports a launch error of its thread instead of
returning what its result memory held before.  The error is one that the runtime
keeps from a host call it refuses (a device number that does not exist): nothing
is launched wrongly, and the same calls succeed afterwards."""
import ctypes as C

import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["stress", "explicit step", "implicit step", "training epoch"])
def test_pending_launch_error_is_reported(call):
    import torch
    from paper_2603_12550_amd import _vds as vds

    print(f"pending error: {call}", flush=True)
    if call == "training epoch":
        m = vds.Mlp(5, 8, 4, 16)
        m.set_params(torch.zeros(5 * 8 + 8 + 64 + 8 + 32 + 4, device="cuda"))
        X, T = torch.randn(32, 5, device="cuda"), torch.randn(32, 4, device="cuda")
        loss = C.c_double()
        order = torch.arange(32, dtype=torch.int32, device="cuda")
        go = lambda: vds._lib.vds_mlp_train_epoch(m.m, vds._ptr(X), vds._ptr(T), 32, 16, 1e-3, vds._ptr(order),
                                                  C.byref(loss))
    else:
        ctx = vds.Context(2, 300, 0.5, scheme=call.split()[0] if "step" in call else "explicit")
        q = torch.from_numpy(wl.to_f32(wl.gaussian_bonds(3, 2, 300, 0.5))).cuda()
        d, tau = vds.vds_diag(), (C.c_double * 9)()
        if call == "stress":
            go = lambda: vds._lib.vds_stress(ctx.ctx, vds._ptr(q), None, tau)
        else:
            go = lambda: vds._lib.vds_step(ctx.ctx, vds._ptr(q), None, 1, C.byref(d))
    assert go() == vds.VDS_OK
    torch.cuda.synchronize()
    lib = vds._lib
    lib.hipSetDevice.restype = lib.hipPeekAtLastError.restype = lib.hipGetLastError.restype = C.c_int
    assert lib.hipSetDevice(C.c_int(1 << 20)) != 0  # refused by the runtime, on the host
    if lib.hipPeekAtLastError() == 0:
        pytest.skip("this runtime keeps no error of a refused host call")
    st = go()
    lib.hipGetLastError()  # clears it also where the call did not
    assert st == 2, st  # VDS_ERR_HIP
    assert go() == vds.VDS_OK
