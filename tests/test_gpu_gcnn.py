"""The layer-wise CNN path over the shapes its dispatch tells apart: every frame size of the row-staged
first layer and others, channel counts of every tile width and mixtures of them in one launch,
k-blocks that span two taps, frames at addresses that are not 16-byte aligned, queues that do not
fill a tile; logits against the FP64 oracle at the tolerances of the other CNN tests."""
import numpy as np
import pytest

import hydro_synth as hs
from oracle import hydro_oracle as ho
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402

MASK = 0b0000011111


@pytest.mark.parametrize("hw,widths", [
    (32, ((16, 32, 64), (64, 16))),
    (64, ((16, 48), (32, 128, 80))),
    (128, ((48, 16, 32), (32, 64, 128))),
    (256, ((16, 16, 256),)),
    (40, ((16, 32), (80, 64))),            # first layer: any size, more than 64 channels
    (8, ((32, 16, 512),)),
])
@pytest.mark.parametrize("dtype,offset", [("u8", 0), ("u8", 1), ("bf16", 0), ("bf16", 1)])
def test_layerwise_logits(hw, widths, dtype, offset):
    n = 5
    cfg = hs.WorkloadConfig(name="t", index=0, n=n, hw=hw, dtype=dtype, data_seed=41, models=[], targets=[(0.5,)])
    frames = hs.make_frames(cfg, 0, n)
    weights = [hs.make_model(hs.ModelDesc(arch="cnn", seed=80 + i, in_hw=hw, widths=w)) for i, w in enumerate(widths)]
    specs = [hydro.ModelSpec.from_weights(w, MASK) for w in weights]
    flat = torch.empty(frames.size + 16, dtype=torch.uint8 if dtype == "u8" else torch.int16, device="cuda")
    flat[offset:offset + frames.size] = torch.from_numpy(frames.view(np.uint8 if dtype == "u8" else np.int16).ravel()).cuda()
    dev = flat[offset:offset + frames.size].view(frames.shape)
    s = hydro.Session(specs, hydro.make_policy("score", precision="bf16"), hw, n)
    for k, w in enumerate(weights):
        z64 = ho.model_logits(w, frames, dtype)
        for tier, tol in ((0, 0.05), (1, 5e-6)):
            err = np.abs(s.logits(k, tier, dev, dtype) - z64).max()
            log(f"[gpu] layer-wise {hw} {widths[k]} {dtype}+{offset} tier {tier}: max |z - z64| = {err:.3e}")
            assert err <= tol
    s.close()


def test_layerwise_grouped_query():
    """Predicates of different tile widths and depths grouped in each launch: ids and written-order
    counts against the oracle."""
    hw, n = 32, 700
    cfg = hs.WorkloadConfig(name="t", index=0, n=n, hw=hw, dtype="u8", data_seed=42, models=[], targets=[(0.5,)])
    frames = hs.make_frames(cfg, 0, n)
    weights = [hs.make_model(hs.ModelDesc(arch="cnn", seed=90 + i, in_hw=hw, widths=w))
               for i, w in enumerate([(16, 32, 64), (64, 16), (32, 128, 48)])]
    D = np.stack([ho.predicate_margin(ho.model_logits(w, frames, "u8"), MASK) for w in weights], axis=1)
    th = np.zeros((1, 3), dtype=np.float32)
    for j in range(3):
        u = np.unique(D[:, j])
        m = np.searchsorted(u, np.quantile(D[:, j], 0.3))
        th[0, j] = np.float32((u[m - 1] + u[m]) / 2.0)
    theta = ho.tuple_thresholds(th, n, np.arange(n))
    assert np.abs(D - theta).min() > 1e-9
    P = ho.decide(D, theta)
    specs = [hydro.ModelSpec.from_weights(w, MASK) for w in weights]
    s = hydro.Session(specs, hydro.make_policy("fixed", order=[1, 0, 2], precision="bf16", wave=128), hw, n)
    s.push(torch.from_numpy(frames).cuda(), "u8", th, n)
    ids, stats = s.finish()
    s.close()
    assert np.array_equal(ids, ho.result_ids(P))
    _, ev, ps = ho.short_circuit_eval(P, [1, 0, 2])
    assert [st["evaluated"] for st in stats] == list(ev)
    assert [st["passed"] for st in stats] == list(ps)
