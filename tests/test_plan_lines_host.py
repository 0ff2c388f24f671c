"""Where the built-in plan leaves the fused schedule (host-only C code): FP32 at
two rounds of 16-atom tiles on the 256 compute units, BF16 at 16384 atoms."""
import pytest

from paper_2505_22168_amd import _capi as A
from test_plan_host import _Sys, _model, _resolve


@pytest.mark.parametrize("hidden", [64, 256])
def test_fused_line(hidden):
    m = _model(hidden=hidden)
    fused, split = (A.GMNN_SCHEDULE_FUSED, 64), (A.GMNN_SCHEDULE_SPLIT, 16)
    assert _resolve(m, _Sys([8192]), 0)[1] == fused
    assert _resolve(m, _Sys([8193]), 0)[1] == split
    assert _resolve(m, _Sys([100] * 90), 0)[1] == split
    assert _resolve(m, _Sys([16383]), A.GMNN_PREC_BF16)[1] == fused
    assert _resolve(m, _Sys([16384]), A.GMNN_PREC_BF16)[1] == split
    # an explicit plan is taken as it is
    assert _resolve(m, _Sys([16384]), 0, A.GMNN_SCHEDULE_FUSED, 64)[1] == fused
