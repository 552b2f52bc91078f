"""CPU build: awe_plan_set_fusion and the plan's device tables.  A HIP graph captured in one mode holds the
addresses of that mode's tables, so a change of mode must give none back; switching back must build none again;
and a change that fails for want of memory must leave the mode before in effect.  Prints one JSON line."""
import json
import os

import numpy as np

import driver as D
from paper_2304_05592_amd import binding as B
import workloads as W


def main():
    lib = D.EmuLib(os.environ["AWE_EMU_SO"])
    count = {k: getattr(lib.L, f"emu_{k}_count") for k in ("malloc", "free")}
    for f in count.values():
        f.restype = D.ctypes.c_longlong
    res = {"freed": {}, "rebuilt": {}}
    small = W.small_2d(nz=30, windows=[40, 33], T_per_shot=[12.0, 9.0])
    wide = W.small_2d(nz=22, nbl=4, windows=[249] * 80, T_per_shot=[7.0] * 80, nrec=5)   # Born has tables of its own
    for name, wl, tiles in (("small", small, None), ("wide", wide, None), ("16 rows", small, 16), ("64 rows", small, 64)):
        plan = D.EmuPlan(lib, wl, storage=B.Storage(B.STORE_FULL))
        if tiles:
            plan.set_tiles(tiles)
        modes = (0, 1, 2, 3) if tiles != 64 else (0,)   # 64 rows: another mode sets rows it has kernels for
        free0 = count["free"]()
        for mode in modes:
            plan.set_fusion(mode)
        n0 = count["malloc"]()
        for mode in modes[::-1] + modes:
            plan.set_fusion(mode)
            assert plan.get_tiles()[2] == mode
        res["freed"][name] = count["free"]() - free0
        res["rebuilt"][name] = count["malloc"]() - n0

    dds = [W.synthetic_residual(s.nt, len(s.rec), small.dt, small.f0, 3 + i) for i, s in enumerate(small.shots)]
    dms = [W.random_field(small.comp_shape(w), 40 + w) * 0.01 for w in range(small.nwindow)]
    plan = D.EmuPlan(lib, small, storage=B.Storage(B.STORE_FULL))
    plan.set_checks(4)
    m, q = plan.pack([small.m(w) for w in range(small.nwindow)]), plan.pack([small.q(i) for i in range(small.nshot)])
    calls = lambda: plan.gradient(m, q, plan.pack(dds), v=True, d=True) + (plan.born(m, q, plan.pack(dms)),)
    ref, shapes = calls(), plan.get_tiles()
    os.environ["EMU_FAIL_MALLOC"] = "1"
    try:
        plan.set_fusion(0)
        res["refused"] = False
    except B.AweError:
        res["refused"] = True
    del os.environ["EMU_FAIL_MALLOC"]
    res["unchanged"] = plan.get_tiles() == shapes and all(np.array_equal(a, b) for a, b in zip(ref, calls()))
    res["bitwise"] = []
    for mode in (0, 3, 1, 0, 2, 3):
        plan.set_fusion(mode)
        res["bitwise"].append(all(np.array_equal(a, b) for a, b in zip(ref, calls())))
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
