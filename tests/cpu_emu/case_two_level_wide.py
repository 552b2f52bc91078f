"""CPU build: the two-level kernels on 128-column tiles (many shots of windows whose widths fill such tiles
but for an odd remainder; FP32, BF16 and FP16 stores), under AddressSanitizer with the host launch checks on: gradient, F^T dd, traces
(FULL storage) and Born traces bitwise those of the one-level kernels.  Prints one JSON line."""
import json
import os

import numpy as np

import driver as D
from paper_2304_05592_amd import binding as B
import workloads as W


def main():
    lib = D.EmuLib(os.environ["AWE_EMU_SO"])
    widths = [117] * 56 + [241] * 28     # computational widths 125 and 249: 220 tiles of 24 rows
    wl = W.small_2d(nz=22, nbl=4, windows=widths, T_per_shot=[7.0 + (s % 3) for s in range(len(widths))], nrec=7)
    dds = [W.synthetic_residual(s.nt, len(s.rec), wl.dt, wl.f0, 3 + i) for i, s in enumerate(wl.shots)]
    dms = [W.random_field(wl.comp_shape(w), 40 + w) * 0.01 for w in range(wl.nwindow)]
    res = {"nt": sorted({s.nt for s in wl.shots}), "bitwise": [], "nonzero": []}
    for prec in (B.PREC_FP32, B.PREC_BF16, B.PREC_FP16):
        got = []
        for tz, fusion in ((16, 0), (24, 3)):
            plan = D.EmuPlan(lib, wl, storage=B.Storage(B.STORE_FULL, prec=prec))
            plan.set_checks(4)
            plan.set_tiles(tz, 8, 0)
            plan.set_fusion(fusion)
            m, q = plan.pack([wl.m(w) for w in range(wl.nwindow)]), plan.pack([wl.q(i) for i in range(wl.nshot)])
            got.append(plan.gradient(m, q, plan.pack(dds), v=True, d=True) + (plan.born(m, q, plan.pack(dms)),))
            del plan
        res["bitwise"] += [bool(np.array_equal(a, b)) for a, b in zip(*got)]
        res["nonzero"] += [bool(np.abs(a).max() > 0) for a in got[0]]
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
