"""The device flags of the kernel files (no GPU needed)."""
import os

import pytest

from paper_1407_1309_amd import build


def test_only_the_fused_2d_kernel_assumes_finite_data():
    """mpdata_diag promises that a NaN or an infinity in psi or in the advector
    reaches the next step's psi.  Under -fno-honor-nans the compiler may give a
    NaN operand any result, so the promise would rest on what it happens to
    emit."""
    relaxed = {f for f, flags in build.FILE_FLAGS.items()
               if any("no-honor" in x or "fast-math" in x or "finite-math" in x for x in flags)}
    assert relaxed <= {"fused2d_f32.hip", "fused2d_f64.hip"}
    assert not any("fast-math" in x or "no-honor" in x for x in build.CFLAGS)


def _tree(tmp_path, monkeypatch):
    import shutil
    csrc = str(tmp_path / "csrc")
    shutil.copytree(build.CSRC, csrc)
    monkeypatch.setattr(build, "CSRC", csrc)
    return csrc


# the files a kernel is written, instantiated and given its launch shape in
PARTS = {"k_resident1d": ["line1d.hpp", "resident1d.hip", "resident1d_f32.hip"],
         "k_pass2d": ["pass2d.hpp", "pass2d.hip", "pass2d_f64_donor.hip", "pass2d_f32_pass.hip",
                      "chunks.hpp"],
         "k_fused2d": ["fused2d.hpp", "fused2d_f64.hip", "fused2d_f32.hip", "chunks.hpp"],
         "k_step3d": ["step3d.hip"], "k_donor3d": ["fused3d.hip"]}


@pytest.mark.parametrize("kernel", sorted(PARTS))
def test_source_hash_covers_what_a_kernel_is_made_of(kernel, tmp_path, monkeypatch):
    """Stored counter readings hold for a kernel only while its source, its
    launch rules and its device flags are those they were taken with."""
    csrc = _tree(tmp_path, monkeypatch)
    base = build.source_hash(kernel)
    for f in PARTS[kernel] + ["common.hpp"]:
        with open(os.path.join(csrc, f), "a") as out:
            out.write("// changed\n")
        changed = build.source_hash(kernel)
        assert changed != base, f
        base = changed
    for f in PARTS[kernel]:
        if f.endswith(".hip"):
            monkeypatch.setitem(build.FILE_FLAGS, f, build.FILE_FLAGS.get(f, []) + ["-DX"])
            changed = build.source_hash(kernel)
            assert changed != base, f
            base = changed
    # and another kernel's file changes nothing
    with open(os.path.join(csrc, "adjoint.hip"), "a") as out:
        out.write("// changed\n")
    assert build.source_hash(kernel) == base
