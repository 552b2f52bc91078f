"""CPU build: a kept checkpointed forward whose gradient is taken after a change of the fusion mode, for every
ordered pair of modes, in workspaces that hold NaN before the call (EMU_FILL=255), under AddressSanitizer.  The
windows are odd and, for 128-column tiles, many, so that steps of one mode read FP32 slots by column pairs that
steps of another wrote column by column.  Every result is bitwise that of one level per launch throughout.
Prints one JSON line."""
import json
import os

import numpy as np

import driver as D
from paper_2304_05592_amd import binding as B
import workloads as W


def main():
    lib = D.EmuLib(os.environ["AWE_EMU_SO"])
    lib.L.awe_backward.argtypes = [D.ctypes.c_void_p] * 7 + [D.ctypes.c_size_t, D.ctypes.c_void_p]
    widths = [int(w) for w in os.environ["CASE_WIDTHS"].split(",")] * int(os.environ["CASE_COPIES"])
    wl = W.small_2d(nz=18, nbl=4, windows=widths, T_per_shot=[6.0 + (s % 2) for s in range(len(widths))], nrec=5)
    dds = [W.synthetic_residual(s.nt, len(s.rec), wl.dt, wl.f0, 3 + i) for i, s in enumerate(wl.shots)]

    def grad(fwd_mode, bwd_mode):
        plan = D.EmuPlan(lib, wl, storage=B.Storage(B.STORE_CHECKPOINT, 2))
        plan.set_checks(4)
        m, q = plan.pack([wl.m(w) for w in range(wl.nwindow)]), plan.pack([wl.q(i) for i in range(wl.nshot)])
        dd, ws, lay = plan.pack(dds), plan.workspace(), plan.layout
        g, v = D._guarded(lay.m_size * 8).view(np.float64), D._guarded(lay.q_size * 4).view(np.float32)
        plan.set_fusion(fwd_mode)
        lib.check(lib.L.awe_forward(plan.h, D._p(m), D._p(q), None, 1, D._p(ws), ws.nbytes, None))
        plan.set_fusion(bwd_mode)
        lib.check(lib.L.awe_backward(plan.h, D._p(m), D._p(q), D._p(dd), D._p(g), D._p(v), D._p(ws), ws.nbytes, None))
        return g.copy(), v.copy()

    ref = grad(0, 0)
    res = {"nt": sorted({s.nt for s in wl.shots}), "finite": bool(np.isfinite(ref[0]).all()),
           "nonzero": bool(np.abs(ref[0]).max() > 0), "bitwise": {}}
    for a in (0, 1, 2, 3):
        for b in (0, 1, 2, 3):
            if (a, b) != (0, 0):
                res["bitwise"][f"{a} {b}"] = all(np.array_equal(x, y) for x, y in zip(ref, grad(a, b)))
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
