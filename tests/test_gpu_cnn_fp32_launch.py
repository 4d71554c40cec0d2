"""FP32 first passes of the fused CNN on both sides of the rule that launches the width classes together or one
by one (16 frames a workgroup): ids and written-order counts against the oracle."""
import numpy as np
import pytest

from oracle import hydro_oracle as ho
from tests.gpu_util import case, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402


@pytest.mark.parametrize("order", [(0, 1, 2), (2, 0, 1)])
@pytest.mark.parametrize("off", [None, 0, 1])
def test_fp32_first_pass_around_the_rule(order, off):
    c = case(2, 6144)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    n = 100 if off is None else min(c.n, 16 * cu + off)
    pol = hydro.make_policy("fixed", order=list(order), precision="fp32", cost_source="static", wave=n)
    ids, stats = hydro.query(c.device_frames()[:n], c.cfg.dtype, c.specs(), c.pt.thresholds, c.seg_len, pol)
    log(f"[gpu] FP32 first pass, {n} frames, order {order}: {ids.size} ids")
    assert np.array_equal(ids, ho.result_ids(c.P[:n]))
    _, ev, ps = ho.short_circuit_eval(c.P[:n], list(order))
    assert [st["evaluated"] for st in stats] == list(ev) and [st["passed"] for st in stats] == list(ps)
