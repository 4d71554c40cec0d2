"""FP64 convolutions on matrix instructions at the edges of their tiles: crops from 1 x 1 to the whole
frame (in LDS and beyond it), channel counts that do not fill a tile, position counts that do not,
and escalated entries on both sides of the layer-parallel limit, against the FP64 oracle."""
import numpy as np
import pytest

import hydro_synth as hs
from oracle import hydro_oracle as ho
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402

MASK = 0b0000011111


def frames_of(hw, dtype, n, seed):
    cfg = hs.WorkloadConfig(name="t", index=0, n=n, hw=hw, dtype=dtype, data_seed=seed, models=[], targets=[(0.5,)])
    return hs.make_frames(cfg, 0, n)


@pytest.mark.parametrize("widths", [(16, 32, 64), (12, 20, 40), (1, 130), (256,), (16, 16, 16, 32)])
@pytest.mark.parametrize("balance", [0, 1])
def test_crop_edges_ids_equal_the_oracle(widths, balance):
    hw, n = 48, 160
    frames = frames_of(hw, "u8", n, 31)
    rng = np.random.default_rng(5)
    sides = [(1, 1), (1, 2), (2, 1), (1, hw), (hw, 1), (hw, hw), (hw, hw - 1), (25, 25), (26, 26), (27, 26), (33, 31)]
    hh = np.array([s[0] for s in sides] + rng.integers(1, hw + 1, n - len(sides)).tolist(), dtype=np.int32)
    ww = np.array([s[1] for s in sides] + rng.integers(1, hw + 1, n - len(sides)).tolist(), dtype=np.int32)
    crops = np.stack([(rng.random(n) * (hw - hh + 1)).astype(np.int32),
                      (rng.random(n) * (hw - ww + 1)).astype(np.int32), hh, ww], axis=1).astype(np.int32)
    w = hs.make_model(hs.ModelDesc(arch="cnn", seed=77, in_hw=hw, widths=widths))
    d = ho.predicate_margin(ho.crop_logits(w, frames, "u8", crops), MASK)
    u = np.unique(d)
    theta = np.float32((u[u.size // 2 - 1] + u[u.size // 2]) / 2.0)
    assert np.abs(d - float(theta)).min() > 1e-9
    spec = hydro.ModelSpec.from_weights(w, MASK, on_crop=True, in_hw=hw)
    s = hydro.Session([spec], hydro.make_policy("score", wave=64, balance=balance), hw, n)
    log(f"[gpu] crops, widths {widths}, balance {balance}")
    s.push(torch.from_numpy(frames).cuda(), "u8", np.array([[theta]], dtype=np.float32), n, crops=crops)
    ids, _ = s.finish()
    s.close()
    assert np.array_equal(ids, np.nonzero(d > float(theta))[0])


# both sides sum at most 9 x 48 products per output in FP64: a few 1e-16 relative each (the same
# tolerance as the other FP64 tier tests)
@pytest.mark.parametrize("hw,widths,n", [(8, (16,), 33), (24, (16, 48), 40), (40, (32, 16, 80), 5), (128, (32, 64, 128, 256), 34)])
@pytest.mark.parametrize("dtype", ["u8", "bf16"])
def test_f64_tier_logits(hw, widths, n, dtype):
    frames = frames_of(hw, dtype, n, 32)
    w = hs.make_model(hs.ModelDesc(arch="cnn", seed=78, in_hw=hw, widths=widths))
    z64 = ho.model_logits(w, frames, dtype)
    s = hydro.Session([hydro.ModelSpec.from_weights(w, MASK)], hydro.make_policy("score"), hw, n)
    z = s.logits(0, 2, torch.from_numpy(frames).cuda(), dtype)
    s.close()
    err = np.abs(z - z64).max()
    log(f"[gpu] FP64 tier hw {hw} widths {widths} {dtype}: max |z - z64| = {err:.3e}")
    assert err <= 1e-13
