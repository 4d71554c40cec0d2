"""Crop predicates of few channels, whose products are packed one after the other and whose activations take
no more room than whole pairs of channels: against the FP64 oracle, with crops on both sides of the limit up to
which activations stay in LDS, and on frames so large that padding to whole tiles would not fit the GPU."""
import numpy as np
import pytest

import hydro_synth as hs
from oracle import hydro_oracle as ho
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402

MASK = 0b0000011111


def _frames(hw, n):
    cfg = hs.WorkloadConfig(name="t", index=0, n=n, hw=hw, dtype="u8", data_seed=33, models=[], targets=[(0.5,)])
    return hs.make_frames(cfg, 0, n)


# widths (16, 32, 64): 24x24 and 25x24 crops take 3,456 and 3,840 of LDS's 4,096 doubles, 24x25 ones 4,224
@pytest.mark.parametrize("widths", [(1,), (1, 1, 1, 1), (2, 2, 2), (3, 5, 7, 9), (4, 4), (15, 16), (14, 17, 2), (16, 8, 8),
                                    (13, 64), (1, 130), (16, 32, 64)])
@pytest.mark.parametrize("balance", [0, 1])
def test_few_channels_equal_the_oracle(widths, balance):
    hw, n = 40, 120
    frames = _frames(hw, n)
    rng = np.random.default_rng(6)
    sides = [(1, 1), (1, 2), (2, 1), (1, hw), (hw, 1), (hw, hw), (hw, hw - 1), (24, 24), (24, 25), (25, 24), (25, 25), (3, 3)]
    hh = np.array([s[0] for s in sides] + rng.integers(1, hw + 1, n - len(sides)).tolist(), dtype=np.int32)
    ww = np.array([s[1] for s in sides] + rng.integers(1, hw + 1, n - len(sides)).tolist(), dtype=np.int32)
    crops = np.stack([(rng.random(n) * (hw - hh + 1)).astype(np.int32),
                      (rng.random(n) * (hw - ww + 1)).astype(np.int32), hh, ww], axis=1).astype(np.int32)
    w = hs.make_model(hs.ModelDesc(arch="cnn", seed=79, in_hw=hw, widths=widths))
    d = ho.predicate_margin(ho.crop_logits(w, frames, "u8", crops), MASK)
    u = np.unique(d)
    theta = np.float32((u[u.size // 2 - 1] + u[u.size // 2]) / 2.0) if u.size > 1 else np.float32(u[0] - 1.0)
    assert np.abs(d - float(theta)).min() > 1e-9
    s = hydro.Session([hydro.ModelSpec.from_weights(w, MASK, on_crop=True, in_hw=hw)],
                      hydro.make_policy("score", wave=64, balance=balance), hw, n)
    log(f"[gpu] crops, widths {widths}, balance {balance}")
    s.push(torch.from_numpy(frames).cuda(), "u8", np.array([[theta]], dtype=np.float32), n, crops=crops)
    ids, _ = s.finish()
    s.close()
    assert np.array_equal(ids, np.nonzero(d > float(theta))[0])


def test_two_channels_on_a_large_frame():
    """Two channels of 1,152 x 1,152 activations for each workgroup are 43 GB, sixteen would be 348."""
    hw = 2304
    frames = np.random.default_rng(7).integers(0, 256, (1, hw, hw, 3), dtype=np.uint8)
    w = hs.make_model(hs.ModelDesc(arch="cnn", seed=80, in_hw=hw, widths=(2,)))
    crops = np.array([[1000, 900, 30, 41]], dtype=np.int32)
    d = float(ho.predicate_margin(ho.crop_logits(w, frames, "u8", crops), MASK)[0])
    for off, want in ((-0.01, 1), (0.01, 0)):
        s = hydro.Session([hydro.ModelSpec.from_weights(w, MASK, on_crop=True, in_hw=hw)], hydro.make_policy("score"), hw, 1)
        s.push(torch.from_numpy(frames).cuda(), "u8", np.array([[d + off]], dtype=np.float32), 1, crops=crops)
        ids, _ = s.finish()
        s.close()
        assert ids.size == want
