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


def _resources(src):
    from paper_1811_04156_amd.build import HIPCC_FLAGS
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared",)]
    cmd = [HIPCC, *flags, "-I", os.path.join(ROOT, "include"), "--cuda-device-only", "-c", "-o", os.devnull,
           "-Rpass-analysis=kernel-resource-usage", os.path.join(CSRC, src)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out, cur = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        m = re.search(r"(VGPRs|AGPRs|ScratchSize \[bytes/lane\]): (\d+)", line)
        if m and cur is not None:
            cur[m.group(1).split()[0]] = int(m.group(2))
    return out


# Registers (VGPRs and AGPRs together) and scratch bytes per lane that each
# kernel may use, by its mangled name; a kernel that no line names fails.
#
# 256 registers are two waves per SIMD, 168 three.  The FP32 step kernels of
# evenly layered media are held to two by their launch bounds and spill what
# that takes: without the bound they keep everything in registers and one wave,
# and 50,001 chains of joint Langevin moves take 5.1 ms instead of 3.1, 262,144
# of tree moves 7.2 instead of 4.4.  The other step kernels' budgets of FP32 are
# tests/test_kernel_resources.py's.  FP64 step kernels run one wave per SIMD.
# The score pass is held to three waves in FP32 (two with the media tables read
# from memory: 315 us instead of 205 for 2^20 chains), the bridge to two.
ONE, TWO, THREE = 512, 256, 168
BUDGETS = {
    "rj_run_f32.hip": [(r"run_kernelIf", ONE, 16), (r"even_layers_kernelIfLi2ELi0ELb0E", TWO, 0),
                       (r"even_layers_kernelIfLi2ELi0ELb1E", TWO, 16)],
    "rj_run_f32_mala.hip": [(r"run_kernelIf", TWO, 16), (r"even_layers_kernelIfLi2ELi1ELb0E", TWO, 40),
                            (r"even_layers_kernelIfLi2ELi1ELb1E", TWO, 88)],
    "rj_run_f32_lmala.hip": [(r"run_kernelIf", ONE, 16), (r"even_layers_kernelIfLi2ELi2ELb0E", TWO, 0),
                             (r"even_layers_kernelIfLi2ELi2ELb1E", TWO, 48)],
    "rj_run_f32_tree.hip": [(r"run_kernelIf", ONE, 16), (r"even_layers_kernelIfLi2ELi3ELb0E", TWO, 16),
                            (r"even_layers_kernelIfLi2ELi3ELb1E", TWO, 88)],
    "rj_run_f64.hip": [(r"(run_kernel|even_layers_kernel)IdLi\dELi0ELb0E", ONE, 0),
                       (r"(run_kernel|even_layers_kernel)IdLi\dELi0ELb1E", ONE, 32)],
    "rj_run_f64_mala.hip": [(r"(run_kernel|even_layers_kernel)IdLi\dELi1ELb0E", ONE, 0),
                            (r"(run_kernel|even_layers_kernel)IdLi\dELi1ELb1E", ONE, 32)],
    "rj_run_f64_lmala.hip": [(r"(run_kernel|even_layers_kernel)IdLi\dELi2ELb0E", ONE, 0),
                             (r"(run_kernel|even_layers_kernel)IdLi\dELi2ELb1E", ONE, 32)],
    "rj_run_f64_tree.hip": [(r"(run_kernel|even_layers_kernel)IdLi\dELi3ELb0E", ONE, 0),
                            (r"(run_kernel|even_layers_kernel)IdLi\dELi3ELb1E", ONE, 32)],
    # grad_kernel<R, DV, KIND (0 any, 1 even layers, 2 homogeneous), SCORE>
    "rj_sampler.hip": [(r"grad_kernelIfLb[01]ELi[12]ELb0E", THREE, 0), (r"grad_kernelIfLb[01]ELi0ELb0E", THREE, 24),
                       (r"grad_kernelIfLb[01]ELi2ELb1E", THREE, 0), (r"grad_kernelIfLb0ELi1ELb1E", THREE, 40),
                       (r"grad_kernelIfLb0ELi0ELb1E", THREE, 80), (r"grad_kernelIfLb1ELi[01]ELb1E", THREE, 144),
                       (r"grad_kernelIdLb[01]ELi[12]ELb[01]E", TWO, 0), (r"grad_kernelIdLb[01]ELi0ELb[01]E", ONE, 48),
                       (r"advance_kernel", 64, 0)],
    "rj_observe.hip": [(r"yield_kernelIf", TWO, 112), (r"yield_kernelId", ONE, 24), (r"lhist_kernelI[fd]", 64, 0)],
    "rj_anchor.hip": [(r"anchor_(lean_|direct_)?kernel", TWO, 0), (r"anchor_sum_kernel", 64, 0)],
    "rj_order.hip": [(r"(weight|order|clear)_kernel", 64, 0)],
}


@pytest.mark.slow
@pytest.mark.parametrize("src", sorted(BUDGETS))
def test_registers_and_scratch_of_every_kernel(src):
    res = _resources(src)
    assert res
    unused = {b[0] for b in BUDGETS[src]}
    for name, r in res.items():
        budget = [b for b in BUDGETS[src] if re.search(b[0], name)]
        assert len(budget) == 1, (name, budget)
        pattern, registers, scratch = budget[0]
        unused.discard(pattern)
        assert r["VGPRs"] + r.get("AGPRs", 0) <= registers, (name, r)
        assert r["ScratchSize"] <= scratch, (name, r)
    assert not unused, unused
