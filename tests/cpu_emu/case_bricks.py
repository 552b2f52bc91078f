"""CPU build: 3D steps on bricks (shape ty = 8, bz = 8) against the z-march, under AddressSanitizer with the
host launch checks on, on a grid whose bricks have remainders on every axis: gradient, F^T dd and traces with
FULL FP32 / BF16 storage, the probed gradient and F^T dd alone, all bitwise.  Prints one JSON line."""
import json
import os

import numpy as np

import driver as D
from paper_2304_05592_amd import binding as B
import workloads as W


def main():
    lib = D.EmuLib(os.environ["AWE_EMU_SO"])
    wl = W.small_3d(n=(13, 10, 59), nbl=4, T=16.0, nrec_side=5, nshot=2)
    dds = [W.synthetic_residual(s.nt, len(s.rec), wl.dt, wl.f0, 3 + i) for i, s in enumerate(wl.shots)]
    nt = wl.shots[0].nt
    C, s = W.probe_table("rademacher", nt, r=3, seed=1)
    out = {"grid": wl.comp_shape(0), "nt": nt, "bitwise": {}}
    for tag, st in (("fp32", B.Storage(B.STORE_FULL)), ("bf16", B.Storage(B.STORE_FULL, 0, B.PREC_BF16)),
                    ("probed", B.Storage(B.STORE_PROBED, 3)), ("adjoint", B.Storage())):
        got = []
        for ty, bz in ((16, 32), (8, 8)):
            plan = D.EmuPlan(lib, wl, storage=st)
            plan.set_checks(4)
            plan.set_tiles(32, ty, bz)
            m, q, dd = plan.pack([wl.m(0)]), plan.pack([wl.q(i) for i in range(wl.nshot)]), plan.pack(dds)
            if tag == "probed":
                got.append(plan.gradient_probed(m, q, dd, C, s, v=True, d=True))
            elif tag == "adjoint":
                got.append((plan.adjoint(m, dd), plan.forward(m, q)))
            else:
                got.append(plan.gradient(m, q, dd, v=True, d=True))
        out["bitwise"][tag] = all(np.array_equal(a, b) for a, b in zip(*got))
        out["bitwise"][tag + "_nonzero"] = all(bool(np.abs(a).max() > 0) for a in got[0])
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
