"""CPU build, where a launch takes a millisecond: a tuned plan's forward solves of few tiles take no more launches
than a default plan's (three levels each), whatever the storage and the probe length, also from the tuner's cache,
and give the same bits.  Prints one JSON line."""
import json
import os
import tempfile

import numpy as np

import driver as D
from paper_2304_05592_amd import binding as B
import workloads as W


def main():
    lib = D.EmuLib(os.environ["AWE_EMU_SO"])
    wl = W.small_2d(nz=30, windows=[40, 33], T_per_shot=[20.0, 14.0])
    dds = [W.synthetic_residual(s.nt, len(s.rec), wl.dt, wl.f0, 3 + i) for i, s in enumerate(wl.shots)]
    res = {"nt": [s.nt for s in wl.shots], "launches": {}, "bitwise": []}

    def forward(storage, probe=None):
        """(launches of a forward solve, its traces) of a plan, tuned where probe is given."""
        plan = D.EmuPlan(lib, wl, storage=storage)
        plan.set_checks(4)
        m, q = plan.pack([wl.m(w) for w in range(wl.nwindow)]), plan.pack([wl.q(i) for i in range(wl.nshot)])
        if probe is not None:
            plan.autotune(m, q, plan.pack(dds), probe_steps=probe)
        n0 = lib.L.emu_launch_count()
        d = plan.forward(m, q)
        return lib.L.emu_launch_count() - n0, d

    ref = None
    for name, storage in (("none", B.Storage()), ("full", B.Storage(B.STORE_FULL)),
                          ("bf16", B.Storage(B.STORE_FULL, prec=B.PREC_BF16)),
                          ("checkpoint", B.Storage(B.STORE_CHECKPOINT, 3)), ("probed", B.Storage(B.STORE_PROBED, 2))):
        default, d = forward(storage)
        ref = d if ref is None else ref
        res["bitwise"].append(bool(np.array_equal(d, ref)))
        res["launches"][name] = [default]
        for probe in (1, 2, 5, 12, 1000):
            n, d = forward(storage, probe)
            res["launches"][name].append(n)
            res["bitwise"].append(bool(np.array_equal(d, ref)))
    with tempfile.TemporaryDirectory() as tmp:
        path = os.environ["AWE_TUNE_CACHE"] = os.path.join(tmp, "tune.json")
        n1, _ = forward(B.Storage(), 12)
        n2, d = forward(B.Storage(), 12)          # from the file
        res["cache"] = [n1, n2, len(json.load(open(path)))]
        res["bitwise"].append(bool(np.array_equal(d, ref)))
        del os.environ["AWE_TUNE_CACHE"]
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
