"""Launches that hold the queues of several predicates at once, at sizes where a workgroup takes several items,
predicates change under it, few-frame tiles of several predicates share a launch or a split falls inside a later
predicate: every decision is that of the logits which each predicate has alone.

Each tuple has thresholds of its own, set from those logits: a float below the margin where the predicate is to
pass, a float above where it is to fail (MLPs, whose K parts follow the queue lengths, 1e-4 away), with bands far
narrower than that, so every decision is the first pass's."""
import numpy as np
import pytest

import hydro_synth as hs
from oracle import hydro_oracle as ho
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402

MASK = 0b0000011111


def _frames(hw, dtype, n, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.rand((n, hw, hw, 3), generator=g, device="cuda")
    return torch.round(x * 255).to(torch.uint8) if dtype == "u8" else x.to(torch.bfloat16)


def _margins(z):
    z = z.astype(np.float32)
    inside = np.array([(MASK >> c) & 1 for c in range(10)], dtype=bool)
    return z[:, inside].max(axis=1) - z[:, ~inside].max(axis=1)


def _check(models, hw, dtype, n, batch, precision, off, **kw):
    k = len(models)
    specs = [hydro.ModelSpec.from_weights(w, MASK) for w in models]
    frames = _frames(hw, dtype, n, 17)
    pol = hydro.make_policy("score", precision=precision, cost_source="static", tau=1e-30, tau32=1e-30, wave=n,
                            routing_batch=batch, log_routes=1, **kw)
    s = hydro.Session(specs, pol, hw, n)
    d = np.stack([_margins(s.logits(j, 0, frames, dtype)) for j in range(k)], axis=1)
    P = np.random.default_rng(18).random((n, k)) < 0.6
    if off:
        th = (d + np.where(P, -off, off)).astype(np.float32)
    else:
        th = np.where(P, np.nextafter(d, np.float32(-np.inf)), np.nextafter(d, np.float32(np.inf)))
    s.push(frames, dtype, th, 1)
    ids, stats = s.finish()
    rounds = s.round_log(0, 2)
    ok, _, _, _, msg = ho.replay_route(P, hydro.decode_routes(s.routes(0, n)))
    s.close()
    first = rounds[1]["folded_evaluated"] if len(rounds) > 1 else None
    log(f"[gpu] {k} predicates, {n} frames {hw}x{hw} {dtype} {precision}: first launch {first}, {ids.size} ids")
    assert ok, msg
    assert np.array_equal(ids, np.nonzero(P.all(axis=1))[0])
    assert first is None or min(first) > 0            # the first launch did hold every predicate's queue


@pytest.mark.parametrize("precision", ["bf16", "fp32"])
@pytest.mark.parametrize("hw,dtype,n", [(128, "u8", 420), (32, "bf16", 10400), (64, "u8", 900)])
def test_layerwise_streams(hw, dtype, n, precision):
    """More first-layer tiles than 1,280 workgroups and, at 32x32, more evaluations than 4,096 head waves."""
    models = [hs.make_model(hs.ModelDesc(arch="cnn", seed=60 + i, in_hw=hw, widths=w))
              for i, w in enumerate([(16, 32, 64), (48, 16), (32, 64, 128)])]
    if hw == 64:                                      # (three layers of 16 m there are the fused kernel's)
        models = models[1:2] + [hs.make_model(hs.ModelDesc(arch="cnn", seed=63, in_hw=hw, widths=(32, 32)))]
    _check(models, hw, dtype, n, n // len(models), precision, 0.0)


@pytest.mark.parametrize("precision", ["bf16", "fp32"])
@pytest.mark.parametrize("n", [9, 60, 120, 240, 390])
def test_few_frame_tiles_of_several_predicates(n, precision):
    cfg = hs.workload(5)
    _check([hs.make_model(m) for m in cfg.models[:3]], 128, "u8", n, max(1, n // 6), precision, 0.0, warmup_batches=2)


def test_few_fp8_frames_equal_many():
    cfg = hs.workload(5)
    frames = _frames(128, "u8", 640, 19)
    s = hydro.Session([hydro.ModelSpec.from_weights(hs.make_model(cfg.models[1]), MASK)],
                      hydro.make_policy("score", precision="fp8"), 128, 640)
    s.calibrate(frames[:64], "u8", 2.0)
    z = s.logits(0, 0, frames, "u8")
    for n in (1, 31, 33, 64, 65, 128, 129, 257):
        assert np.array_equal(s.logits(0, 0, frames[640 - n:], "u8"), z[640 - n:])
    s.close()


@pytest.mark.parametrize("precision,n", [("fp32", 6000), ("bf16", 12000)])
@pytest.mark.parametrize("dtype", ["bf16", "u8"])
def test_mlp_split_inside_a_later_predicate(precision, n, dtype):
    """Two predicates of 1,024 hidden units, half of the tuples each: on 256 CUs 192 tiles of 128 (256) rows each,
    so that the tiles which are split start within the second (bf16 frames)."""
    models = [hs.make_model(hs.ModelDesc(arch="mlp", seed=70 + i, d_in=768, hidden=1024)) for i in range(2)]
    _check(models, 16, dtype, n, n // 2, precision, 1e-4)


@pytest.mark.parametrize("precision,tier", [("fp32", 0), ("bf16", 0)])
def test_left_over_tiles_are_split(monkeypatch, precision, tier):
    """With splitting switched off the sums run in another order: the logits differ in the last bits and no more."""
    w = hs.make_model(hs.ModelDesc(arch="mlp", seed=72, d_in=3072, hidden=256))
    frames = _frames(32, "bf16", 300, 20)
    z = {}
    for below in ("0", ""):
        monkeypatch.setenv("HYDRO_SPLITK_BELOW", below)
        s = hydro.Session([hydro.ModelSpec.from_weights(w, MASK)], hydro.make_policy("score", precision=precision), 32, 300)
        z[below] = s.logits(0, tier, frames, "bf16")
        s.close()
    assert not np.array_equal(z["0"], z[""])
    assert np.abs(z["0"] - z[""]).max() < 1e-4
