"""The layer-wise CNN path's FP32 tier on values that its bf16 terms do not hold: infinite, undefined and very
large pixels, weights near the largest fp32.  What fp32 arithmetic makes of them is what the FP64 tier
does (ReLU turns an undefined sum into zero in both), so the tiers' logits agree to the tolerance that the
FP32 tier has on ordinary frames, relative to a frame's largest logit."""
import numpy as np
import pytest

import hydro_synth as hs
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402

TOL = 5e-6


def _spec(hw, widths):
    w = hs.make_model(hs.ModelDesc(arch="cnn", seed=7, in_hw=hw, widths=widths))
    return hydro.ModelSpec.from_weights(w, 0b0000011111)


def _frames(hw, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    return torch.rand((n, hw, hw, 3), generator=g, device="cuda").to(torch.bfloat16)


def _agree(z, z64):
    scale = np.maximum(1.0, np.where(np.isfinite(z64), np.abs(z64), 0.0).max(axis=1, keepdims=True))
    return np.isclose(z / scale, z64 / scale, rtol=0.0, atol=TOL, equal_nan=True).all(axis=1)


@pytest.mark.parametrize("hw,widths", [(32, (16, 32, 64)), (64, (48, 16, 128)), (128, (16, 32, 64)), (40, (80, 64)),
                                       (8, (32,)), (8, (32, 16, 512))])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 1e30])
def test_fp32_logits_of_wide_pixels(hw, widths, value):
    n = 40
    plain = _frames(hw, n)
    odd = plain.clone()
    for i in range(0, n, 2):
        odd[i, (3 * i) % hw, (5 * i) % hw, i % 3] = value
    s = hydro.Session([_spec(hw, widths)], hydro.make_policy("score", precision="bf16"), hw, n)
    want = s.logits(0, 1, plain, "bf16")
    ok = _agree(s.logits(0, 1, odd, "bf16"), s.logits(0, 2, odd, "bf16"))
    log(f"[gpu] layer-wise {hw} {widths}, pixels of {value}: {int((~ok).sum())} of {n} frames differ")
    assert ok.all()
    # nothing of it is left for the next launch
    assert np.array_equal(s.logits(0, 1, plain, "bf16"), want)
    s.close()


@pytest.mark.parametrize("layer", [0, 1])
def test_fp32_logits_with_wide_weights(layer):
    """Layer 1: a channel of weights 2^40, which layer 2 ignores.  Layer 2: weights near the largest fp32 on a
    channel that layer 1 leaves at zero."""
    hw, n = 32, 20
    spec = _spec(hw, (16, 32))
    frames = _frames(hw, n)
    convs = spec.t["convs"] = [(w.copy(), b.copy()) for w, b in spec.t["convs"]]
    if layer == 0:
        convs[0][0][3] = 2.0**40
        convs[1][0][:, 3] = 0.0
    else:
        convs[0][0][5] = 0.0
        convs[0][1][5] = 0.0
        convs[1][0][:, 5] = 3.4e38
    s = hydro.Session([spec], hydro.make_policy("score", precision="bf16"), hw, n)
    ok = _agree(s.logits(0, 1, frames, "bf16"), s.logits(0, 2, frames, "bf16"))
    s.close()
    log(f"[gpu] layer-wise, wide weights in layer {layer}: {int((~ok).sum())} of {n} frames differ")
    assert ok.all()
