"""The tracing variant (-DMOE_SCHED_TRACE) of the register-stationary weight-gradient kernel times the kernel that ships: its
source differs by the clock reads alone.  CPU only: both variants are preprocessed and compared."""
import os
import subprocess

import pytest

from paper_2605_23764_amd.build import SOURCES

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _sweep(*flags):
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "--cuda-device-only", "-E", "-P", *flags, *SOURCES],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    src = res.stdout
    start = src.index("void wp_item(")
    return src[start:src.index("grouped_wgrad_panel_bf16_kernel(", start)]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_traced_sweep_is_the_shipped_sweep():
    def squeezed(text):   # statement by statement
        return [" ".join(x.split()) for x in text.replace("{", "{;").replace("}", "};").split(";") if x.strip()]
    shipped, traced = squeezed(_sweep()), squeezed(_sweep("-DMOE_SCHED_TRACE"))
    assert not any("trace_" in x for x in shipped)
    assert sum("s_memtime" in x for x in traced) >= 5
    assert [x for x in traced if "trace_" not in x] == shipped
