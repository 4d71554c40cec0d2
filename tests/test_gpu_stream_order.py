"""Scores and bands of frames that work on the default stream is still writing when the call is made: they
are those of the finished frames (the session's own stream does not wait for the default stream by itself)."""
import numpy as np
import pytest

import hydro_synth as hs
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402


def _late(dst, src):
    """src copied to dst behind some tens of milliseconds of other work on the default stream."""
    a = torch.full((8192, 8192), 1e-3, device="cuda")
    for _ in range(8):
        a = a @ a
    dst.copy_(src, non_blocking=True)


@pytest.mark.parametrize("wl,hw", [(1, 32), (2, 64), (5, 128)])
def test_logits_and_bands_wait_for_the_frames(wl, hw):
    n = 256
    cfg = hs.workload(wl)
    pt = hs.load_predicates(cfg)
    first, then = (torch.from_numpy(hs.make_frames(cfg, lo, n)).cuda() for lo in (0, n))
    spec = hydro.ModelSpec.from_weights(hs.make_model(cfg.models[0]), pt.class_masks[0])
    s = hydro.Session([spec], hydro.make_policy("score", precision="bf16"), hw, n)
    want = [s.logits(0, tier, then, cfg.dtype) for tier in (0, 1, 2)]
    bands = s.calibrate(then, cfg.dtype, 2.0)
    buf = first.clone()
    other = s.logits(0, 1, buf, cfg.dtype)
    assert not np.array_equal(other, want[1])
    for tier in (0, 1, 2):
        buf.copy_(first)
        torch.cuda.synchronize()
        _late(buf, then)
        got = s.logits(0, tier, buf, cfg.dtype)
        log(f"[gpu] late frames, workload {wl}, tier {tier}: equal {np.array_equal(got, want[tier])}")
        assert np.array_equal(got, want[tier])
    buf.copy_(first)
    torch.cuda.synchronize()
    _late(buf, then)
    got = s.calibrate(buf, cfg.dtype, 2.0)
    assert all(np.array_equal(g, b) for g, b in zip(got, bands))
    s.close()
