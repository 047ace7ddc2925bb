"""Register and scratch budgets of the push kernels that the FP32 check of
test_abi does not cover, read from the built library (no GPU needed)."""
import re
import subprocess

from tests.test_abi import P, _code_objects  # noqa: F401 (P: the fixture)


def _kernels(lib_path, tmp_path, prefix):
    """{name: metadata} of the library's kernels whose mangled name starts so."""
    out = {}
    for co in _code_objects(lib_path, tmp_path):
        notes = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", str(co)], capture_output=True,
                               text=True).stdout
        for block in notes.split("  - .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", block).group(1)
            if name.startswith(prefix):
                out[name] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)", block)}
    return out


def test_fp64_push_kernels_keep_their_register_budget(P, tmp_path):  # noqa: F811
    # three waves per SIMD: at most 168 VGPRs, none spilled; only the wall
    # variants have scratch, the per-lane array that the wall's axis indexes
    found = _kernels(P.LIB_PATH, tmp_path, "_ZN3pic11push_kernelId")
    assert len(found) == 6
    for name, m in found.items():
        walls = re.match(r"_ZN3pic11push_kernelIdLi\dELi(\d)E", name).group(1) == "1"
        assert m["vgpr_count"] <= 168 and m["vgpr_spill_count"] == 0, (name, m)
        assert m["private_segment_fixed_size"] <= (32 if walls else 0), (name, m)


def test_other_push_kernels_keep_the_budgets(P, tmp_path):  # noqa: F811
    # the variants with 64-bit slots as the plain ones; those with 512 or 1024
    # threads per tile at most 128 VGPRs (1024 threads are four waves per SIMD);
    # all within the static LDS that pic_plan keeps back
    far = _kernels(P.LIB_PATH, tmp_path, "_ZN3pic15far_push_kernel")
    wide = _kernels(P.LIB_PATH, tmp_path, "_ZN3pic16wide_push_kernel")
    assert len(far) == 6 and len(wide) == 6
    for name, m in far.items():
        form, walls = re.match(r"_ZN3pic15far_push_kernelI([fd])Li(\d)E", name).groups()
        scratch = 0 if walls == "0" else (16 if form == "f" else 32)
        assert m["vgpr_count"] <= (128 if form == "f" else 168) and m["vgpr_spill_count"] == 0, (name, m)
        assert m["private_segment_fixed_size"] <= scratch, (name, m)
    for name, m in wide.items():
        assert m["vgpr_count"] <= 128 and m["vgpr_spill_count"] == 0, (name, m)
        assert m["private_segment_fixed_size"] == 0, (name, m)
    for name, m in {**far, **wide}.items():
        assert m["group_segment_fixed_size"] <= 2176, (name, m)
