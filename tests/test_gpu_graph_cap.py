"""A captured pass holds the secular sweep cap (max_sweeps) by value, so calls
on the same buffers with different caps are different graphs: a call never
replays another call's cap, in either order and again on later replays."""
import numpy as np
import pytest

import oracle
import tdgen

pytestmark = pytest.mark.gpu

GATE = 2e-11


@pytest.fixture(scope="module")
def tde():
    import torch

    import paper_2605_26599_amd as m

    assert torch.cuda.is_available()
    m.lib()
    return m


@pytest.mark.parametrize("call", ["eigvals", "eigvals_batched", "eigvals_ckpt", "eigvals_rows"])
@pytest.mark.parametrize("caps", [(1, None, 1, None), (None, 1, None, 1), (96, 1, 1, 96)], ids=str)
def test_cap_belongs_to_the_call(tde, call, caps):
    import ctypes

    import torch

    n = 3000
    d, e = tdgen.tridiag("uniform", n)
    tol = GATE * tdgen.tnorm1(d, e)
    exact = oracle.eigvals(d, e)
    dv = torch.from_numpy(d).cuda()
    ev = torch.from_numpy(np.append(e, 0.0)).cuda()
    out, q0, q1 = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(3))
    ws = torch.empty(tde.workspace_bytes(n), dtype=torch.uint8, device="cuda")
    ckpt = torch.empty(tde.checkpoint_bytes(n), dtype=torch.uint8, device="cuda")
    offs = (ctypes.c_int64 * 2)(0, n)

    def solve(cap):
        if call == "eigvals_rows":
            opts = tde.tde_opts(max_sweeps=cap or 0)
            stream = torch.cuda.current_stream().cuda_stream
            assert tde.lib().tde_eigvals_rows(dv.data_ptr(), ev.data_ptr(), offs, 1, out.data_ptr(), q0.data_ptr(),
                                              q1.data_ptr(), ws.data_ptr(), ws.numel(), stream,
                                              ctypes.byref(opts)) == tde.TDE_OK
            st = tde.last_status(ws)
            if st != tde.TDE_OK:
                raise tde.TDEError(st)
            return
        tde.set_defaults(max_sweeps=cap)
        try:
            if call == "eigvals":
                tde.eigvals(dv, ev, out=out, workspace=ws)
            elif call == "eigvals_batched":
                tde.eigvals_batched(dv, ev, [0, n], out=out, workspace=ws)
            else:
                tde.eigvals_ckpt(dv, ev, out=out, ckpt=ckpt, workspace=ws)
        finally:
            tde.set_defaults()

    for cap in caps:
        print(f"[gpu-cap] {call} cap={cap}", flush=True)
        if cap == 1:
            with pytest.raises(tde.TDEError) as ex:
                solve(cap)
            assert ex.value.code == tde.TDE_ENOCONV
        else:
            solve(cap)
            assert np.abs(out.cpu().numpy() - exact).max() <= tol
