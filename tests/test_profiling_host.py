"""Names of kernels in the profiles: every whole-step kernel of the library has a kind, and the
bench looks a kernel's counters up under the kind that the profile summary writes."""
import os
import re

import pytest

from paper_2411_18341_amd import build, profiling

KERNELS = {
    "void phx::rk4_step_kernel<float, true, false, false, 8, 4>(phx::StepArgs<float>)": ("rk4_step", (8, 4)),
    "void phx::rk4_stream_step_kernel<float, 2, true, false, false, false, true, false, false, true, 3>(phx::StepArgs<float>)":
        ("rk4_step", (2, 0)),
    "void phx::rk4_stream_step_kernel<double, 1, false, true, true, true, false, true, false, false, 3>(phx::StepArgs<double>)":
        ("rk4_step", (1, 40)),
    "void phx::rk4_stream_pair_kernel<float, 2, true, false, false, false, 2, true, false>(phx::StepArgs<float>)":
        ("rk4_step_pair", (2, 0)),
    "void phx::rk4_stage_kernel<float, 1, true, false, 2>(phx::Rk4Args<float>)": ("rk4_stage2", (4, 16)),
}


@pytest.mark.parametrize("name", KERNELS)
def test_the_bench_finds_what_the_summary_writes(name):
    timing_kind, shape = KERNELS[name]
    assert profiling.step_kernel_kind(timing_kind, *shape) == profiling.kernel_kind(name)


def test_every_named_kernel_exists():
    """The summary names every rk4 kernel that the library has, and of those that it no longer
    has only the ones that older profiles hold."""
    sources = "".join(open(os.path.join(build.CSRC, f)).read() for f in os.listdir(build.CSRC))
    have = set(re.findall(r"(?<!\w)((?:rk4|dp|batch|conv|wiener)_\w*kernel)(?=\(|<)", sources))
    with open(profiling.__file__) as f:
        named = set(re.findall(r"(?:rk4|dp|batch|conv|wiener)_\w*kernel(?=\W)", f.read()))
    assert named <= have | {"rk4_stream_wide_kernel"}
    assert {k for k in have if k.startswith("rk4_")} <= named
