"""CPU build: what awe_profile_read counts.  A plan whose fusion mode is the default counts time levels, whatever
its storage and the call; one whose mode was set, by the caller or the autotuner, counts launches.  Prints one JSON
line: counts per storage and mode, and the levels of a sweep."""
import ctypes
import json
import os

import driver as D
from paper_2304_05592_amd import binding as B
import workloads as W


def main():
    lib = D.EmuLib(os.environ["AWE_EMU_SO"])
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    lib.L.awe_profile_enable.argtypes = [vp, i64, ctypes.c_int32]
    lib.L.awe_profile_read.argtypes = [vp, ctypes.POINTER(i64), ctypes.POINTER(ctypes.c_double)]
    wl = W.small_2d(nz=30, windows=[40, 33], T_per_shot=[16.0, 12.0])
    dds = [W.synthetic_residual(s.nt, len(s.rec), wl.dt, wl.f0, 3 + i) for i, s in enumerate(wl.shots)]
    dms = [W.random_field(wl.comp_shape(w), 40 + w) * 0.01 for w in range(wl.nwindow)]
    res = {"levels": max(s.nt for s in wl.shots) - 1, "counts": {}}
    for name, storage in (("full", B.Storage(B.STORE_FULL)), ("bf16", B.Storage(B.STORE_FULL, prec=B.PREC_BF16)),
                          ("checkpoint", B.Storage(B.STORE_CHECKPOINT, 3))):
        for mode in ("default", "tiles", 0, 3, "tuned"):
            plan = D.EmuPlan(lib, wl, storage=storage)
            m, q = plan.pack([wl.m(w) for w in range(wl.nwindow)]), plan.pack([wl.q(i) for i in range(wl.nshot)])
            if mode == "tuned":
                plan.autotune(m, q, None, probe_steps=4)
            elif mode == "tiles":
                plan.set_tiles(16)
            elif mode != "default":
                plan.set_fusion(mode)
            counts, ms = (i64 * 3)(), (ctypes.c_double * 3)()
            got = []
            for call in (lambda: plan.gradient(m, q, plan.pack(dds)), lambda: plan.born(m, q, plan.pack(dms))):
                lib.check(lib.L.awe_profile_enable(plan.h, 1000, 1))
                call()
                lib.check(lib.L.awe_profile_read(plan.h, counts, ms))
                got += list(counts)
            res["counts"][f"{name} {mode}"] = [got[0], got[1], got[5]]
    res["advances"] = int(sum(b - a for op, a, b in schedule(lib, res["levels"], 3) if op == 0))
    print(json.dumps(res), flush=True)


def schedule(lib, n, slots):
    cnt = ctypes.c_int64()
    buf = (ctypes.c_int32 * 3000)()
    lib.L.awe_checkpoint_schedule.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p]
    lib.check(lib.L.awe_checkpoint_schedule(n, slots, buf, 1000, ctypes.byref(cnt)))
    return [tuple(buf[3 * i:3 * i + 3]) for i in range(cnt.value)]


if __name__ == "__main__":
    main()
