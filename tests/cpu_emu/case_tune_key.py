"""CPU build: an autotuner cache entry written before the kernels changed (its key names no tuner version) is left
in the file but not applied.  Prints one JSON line."""
import json
import os
import re
import tempfile

import driver as D
from paper_2304_05592_amd import binding as B
import workloads as W


def main():
    lib = D.EmuLib(os.environ["AWE_EMU_SO"])
    wl = W.small_2d(nz=30, windows=[40, 33], T_per_shot=[8.0, 6.0])

    def tune():
        plan = D.EmuPlan(lib, wl, storage=B.Storage(B.STORE_FULL))
        m, q = plan.pack([wl.m(w) for w in range(wl.nwindow)]), plan.pack([wl.q(i) for i in range(wl.nshot)])
        return plan.autotune(m, q, None, probe_steps=4)

    with tempfile.TemporaryDirectory() as tmp:
        path = os.environ["AWE_TUNE_CACHE"] = os.path.join(tmp, "tune.json")
        tiles, _ = tune()
        key = next(iter(json.load(open(path))))
        old = re.sub(r"^v(\d+)(\.\d+)?/", r"v\1/", key)
        with open(path, "w") as f:
            f.write('{\n  "%s": {"fw": [64, 8, 0], "rv": [64, 8, 0], "fusion": 0, "ms": 42.500000}\n}\n' % old)
        again, ms = tune()
        res = {"applied": ms == 42.5, "same": again == tiles, "entries": sorted(json.load(open(path))) == sorted([old, key])}
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
