"""The kernel instances that bench.py names are those the library launches for
the calls it times (read from csrc/wilson.hip)."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def _body(src, name):
    i = src.index(f"void {name}(")
    return src[i:src.index("\n}\n", i)]


def test_stencil_leg_names_its_kernels():
    import bench

    with open(os.path.join(ROOT, "paper_0704_3486_amd", "csrc", "wilson.hip")) as f:
        src = f.read()
    with open(os.path.join(ROOT, "bench.py")) as f:
        leg = f.read().split("def stencil_leg")[1].split("\ndef ")[0]
    # sgn_matvec launches wilson_apply_abi's instance
    args = re.search(r"hw_launch_as<([^>]*)>", _body(src, "wilson_apply_abi")).group(1)
    assert bench.STENCIL_KERNELS["matvec"] == f"wilson_hw_dir_kernel<{args}>"
    assert 'STENCIL_KERNELS["matvec"]' in leg and "sg.sgn_matvec(" in leg
    # an apply launches the component-major form without further terms, split by the workgroups
    terms = re.search(r"hw_launch<double2, (\d)>", _body(src, "wilson_apply")).group(1)
    below = int(re.search(r"kSplitBelow = (\d+);", src).group(1))
    V = 1
    for d in bench.STENCIL_DIMS:
        V *= d
    sites = 16 if (V + 31) // 32 < below else 32
    assert bench.STENCIL_KERNELS["apply"] == f"wilson_hw_dir_kernel<double2, {sites}, {terms}, false>"
    # the 6^4 legs
    V = 6**4
    assert (V + 31) // 32 * bench.BATCH < below
    assert bench.HBM_KERNELS["wilson_hw"] == "wilson_hw_dir_kernel<double2, 16, 0, false>"
    assert bench.HBM_KERNELS_BLOCK["wilson_hw"] == "wilson_hw_dir_kernel<double2, 16, 1, false>"
