"""4-layer CNN launches that hold few frames (bands of a frame shared among workgroups, 64-position
tiles in layers 3 and 4): a frame's logits are bit for bit those of a launch that fills the large
tiles, at the edges of every rule, in each tier and with several predicates in one launch."""
import numpy as np
import pytest

import hydro_synth as hs
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402

BIG = 640          # more than every few-frame rule takes


@pytest.mark.parametrize("dtype", ["u8", "bf16"])
def test_few_frame_logits_equal_the_large_tiles(dtype):
    cfg = hs.workload(5)
    pt = hs.load_predicates(cfg)
    frames = hs.make_frames(cfg, 0, BIG)
    if dtype == "bf16":
        frames = hs.f64_to_bf16_bits(frames.astype(np.float64) / 255.0)
    dev = torch.from_numpy(frames.view(np.int16) if dtype == "bf16" else frames).cuda()
    specs = [hydro.ModelSpec.from_weights(hs.make_model(d), m) for d, m in zip(cfg.models[:2], pt.class_masks)]
    s = hydro.Session(specs, hydro.make_policy("score", precision="bf16", rescore3=1), 128, BIG)
    for tier in (0, 1, 3):
        z = s.logits(1, tier, dev, dtype)
        for n in (1, 2, 31, 32, 33, 64, 65, 127, 128, 129, 255, 256, 257, 513):
            log(f"[gpu] few frames: {dtype} tier {tier} n {n}")
            assert np.array_equal(s.logits(1, tier, dev[BIG - n:], dtype), z[BIG - n:])
    s.close()
