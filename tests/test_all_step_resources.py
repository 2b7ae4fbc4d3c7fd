"""Resource use of every kernel that runs a time step, read from the compiler's
gfx950 output (no GPU needed): no instance may appear, grow scratch or spill
beyond what is written here. Four of them do today: the bricks of eight FP32 and
four FP64 cells a thread, whose state and operator (some 20 values a cell) do not
fit 256 registers beside the step's own, the deep fixed-K kernel of 16 cells a thread,
which has 168 registers, and the traced fixed-K step. They are faster all the same
than the kernel that would take their grids: 12 steps of 256x128x32 take 7.9 ms
on bricks of eight cells a thread, 12.8 on the resident kernel."""
import re

import pytest

from test_kernel_resources import asm, kernel_body, kernel_meta  # noqa: F401  (asm: fixture)

# (scratch bytes, VGPR spills) where not (0, 0)
BUDGET = {
    "brick_steps_kernelIfLi8ELi512E": (184, 45),
    "brick_steps_kernelIdLi4ELi512E": (48, 11),
    "jacobi_deep_kernelILi16ELi2ELi4E": (208, 60),
    "jacobi_step_kernelILi2E": (20, 0),
}
KERNELS = {
    *(f"brick_steps_kernelI{r}Li{zc}ELi{nt}E" for r in "fd" for zc, nt in ((1, 512), (2, 512), (4, 512), (8, 256))),
    "brick_steps_kernelIfLi8ELi512E",
    *(f"{k}ILi{iy}E" for k in ("jacobi_steps_kernel", "jacobi_step_kernel") for iy in (2, 4, 8)),
    *(f"jacobi_deep_kernelILi{h}ELi{p}ELi{iy}E" for h, p, iy in ((12, 2, 2), (8, 3, 4), (16, 2, 2), (16, 2, 4))),
    "step_kernelIf", "step_kernelId", "resident_step_kernelILi64E", "resident_full_kernelILi64E",
    "batch_run_kernel", "batch_resident_kernel",
}

def short(sym):
    for k in KERNELS:
        if re.match(r"_ZN2nh\d+" + re.escape(k), sym):
            return k
    return None


def test_the_step_kernels_are_the_ones_listed(asm):  # noqa: F811
    found = [s for s in kernel_meta(asm)
             if re.match(r"_ZN2nh\d+(brick_|jacobi_|resident_|batch_|step_)\w*kernel", s)]
    assert {short(s) for s in found} == KERNELS, [s for s in found if short(s) is None]


@pytest.mark.parametrize("kernel", sorted(KERNELS))
def test_step_kernel_stays_within_its_registers(asm, kernel):  # noqa: F811
    meta = kernel_meta(asm)
    sym, = (s for s in meta if short(s) == kernel)
    private, spills = BUDGET.get(kernel, (0, 0))
    assert meta[sym]["private"] <= private and meta[sym]["vgpr_spill"] <= spills, meta[sym]
    assert "s_swappc" not in kernel_body(asm, sym)
