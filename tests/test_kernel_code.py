"""Properties of the compiled kernels that no run can show (CPU:
cross-compiles for gfx950)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1811_04156_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not shutil.which(HIPCC) and not os.path.exists(HIPCC), reason="hipcc not available")


def _functions(src, tmp_path):
    """The functions of a unit as the front end emits them (no optimisation),
    name -> lines."""
    from paper_1811_04156_amd.build import HIPCC_FLAGS
    out = tmp_path / "unit.ll"
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared",)]
    cmd = [HIPCC, *flags, "-I", os.path.join(ROOT, "include"), "--cuda-device-only", "-S", "-emit-llvm", "-Xclang",
           "-disable-llvm-passes", "-o", str(out), os.path.join(CSRC, src)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    fns, cur = {}, None
    for line in out.read_text().splitlines():
        m = re.match(r"define .*@(\w+)\(", line)
        if m:
            cur = fns.setdefault(m.group(1), [])
        elif line == "}":
            cur = None
        elif cur is not None:
            cur.append(line)
    return fns


@pytest.mark.parametrize("src", ["rj_run_f32_tree.hip", "rj_run_f64_mala.hip"])
def test_shared_shift_loads_a_window_before_it_stores(src, tmp_path):
    """The lanes of a window of the shared vertex shift store to slots that
    other lanes of it load.  The order is the source's, not the compiler's: a
    fence and a wave barrier stand between the window's loads and stores, on
    every way from the ones to the others."""
    fns = _functions(src, tmp_path)
    ordered = [n for n, body in fns.items() if any("@llvm.amdgcn.wave.barrier()" in x for x in body)
               and any(re.match(r"\s*fence .*acq_rel", x) for x in body)]
    shifts = {n: b for n, b in fns.items() if "shift_shared" in n}
    assert len(shifts) == 1
    for name, body in shifts.items():
        # the slots in LDS, which is where one branch of the loads and of the stores goes
        loads = [i for i, x in enumerate(body) if re.search(r"= load <4 x (float|double)>, ptr addrspace\(3\)", x)]
        stores = [i for i, x in enumerate(body) if re.search(r"store <4 x (float|double)> .*, ptr addrspace\(3\)", x)]
        order = [i for i, x in enumerate(body) if any(f"@{n}(" in x for n in ordered)]
        assert len(loads) == 1 and len(stores) == 1
        assert any(loads[0] < i < stores[0] for i in order), (name, loads, stores, order)
        # and in a block that both the loads' branches and the lanes without an item reach
        block = {}
        at = "entry"
        for i, x in enumerate(body):
            m = re.match(r"(\w+):", x)
            at = m.group(1) if m else at
            block[i] = at
        mid = [i for i in order if loads[0] < i < stores[0]]
        preds = next(x for x in body if x.startswith(block[mid[0]] + ":")).split("preds =")[1].split(",")
        assert len(preds) == 2, preds
