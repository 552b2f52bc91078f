"""CPU build: default tile rows of many small windows (plans are created, nothing runs).  Prints one JSON line:
per window and count, the forward and adjoint rows."""
import json
import os

import driver as D
from paper_2304_05592_amd import binding as B
import workloads as W


def main():
    lib = D.EmuLib(os.environ["AWE_EMU_SO"])
    res = {}
    for nz, nx, n in ((41, 45, 450), (70, 64, 500), (33, 64, 800), (25, 64, 900), (97, 190, 150), (12, 250, 800),
                      (26, 250, 400), (49, 250, 300)):
        wl = W.small_2d(nz=nz - 8, nbl=4, windows=[nx - 8] * n, T_per_shot=[4.0] * n, nrec=1)
        plan = D.EmuPlan(lib, wl, storage=B.Storage(B.STORE_FULL))
        fw, rv, fusion = plan.get_tiles()
        res[f"{nz} {nx} {n}"] = [fw[0], rv[0], fusion]
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
