"""CPU build: small forward solves, which default plans advance several levels per launch, under
AddressSanitizer with the host launch checks on: traces and gradient (FULL FP32) of batches with per-shot nt
and every remainder of the step count are bitwise those of one level per launch.  Prints one JSON line."""
import json
import os

import numpy as np

import driver as D
from paper_2304_05592_amd import binding as B
import workloads as W


def main():
    lib = D.EmuLib(os.environ["AWE_EMU_SO"])
    out = {}
    for widths, T in (([40, 57], [9.0, 4.0]), ([33], [6.0]), ([33], [7.0]), ([33], [8.0]), ([33], [1.0]),
                      ([119, 52, 40], [14.0, 2.0, 11.0]), ([40] * 60, [5.0, 4.0]), ([40] * 120, [4.0])):
        wl = W.small_2d(nz=30, nbl=6, windows=widths, T_per_shot=[T[s % len(T)] for s in range(len(widths))], nrec=9)
        dds = [W.synthetic_residual(s.nt, len(s.rec), wl.dt, wl.f0, 3 + i) for i, s in enumerate(wl.shots)]
        got = []
        for fusion in (None, 0):
            plan = D.EmuPlan(lib, wl, storage=B.Storage(B.STORE_FULL))
            plan.set_checks(4)
            if fusion is not None:
                plan.set_fusion(fusion)
            m, q = plan.pack([wl.m(w) for w in range(wl.nwindow)]), plan.pack([wl.q(i) for i in range(wl.nshot)])
            got.append(plan.gradient(m, q, plan.pack(dds), v=True, d=True) + (plan.forward(m, q),))
        out[f"{len(widths)} shots, nt {[s.nt for s in wl.shots[:3]]}"] = all(np.array_equal(a, b) for a, b in zip(*got))
    print(json.dumps({"bitwise": out, "nonzero": bool(np.abs(got[0][0]).max() > 0)}), flush=True)


if __name__ == "__main__":
    main()
