"""The device flags of the kernel files (no GPU needed)."""
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
