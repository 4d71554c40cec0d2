"""Rounding errors of the FP32 tiers against FP64, over long sums: no larger than those of fp32 arithmetic that
rounds its sum after every four products, as an fp32 MFMA does, or after each of three products of bf16 terms
(emulated on the CPU), in a given number of parts."""
import numpy as np
import pytest

import hydro_synth as hs
from oracle import hydro_oracle as ho
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402

MASK = 0b0000011111


def _sum4(x, w, start=0):
    """x @ w, the sum rounded to fp32 after every four products (each product and the four's sum exact)."""
    acc = np.zeros((x.shape[0], w.shape[1]), dtype=np.float32)
    x, w = x.astype(np.float64), w.astype(np.float64)
    for k in range(start, x.shape[1], 4):
        acc = (acc + x[:, k:k + 4] @ w[k:k + 4]).astype(np.float32)
    return acc


def _columns(x):
    """[n][h][w][c] padded with zeros -> [n * h/2 * w/2][9 c] of a 3x3 stride-2 convolution, (tap, channel)."""
    n, h, w, c = x.shape
    p = np.zeros((n, h + 1, w + 1, c), dtype=x.dtype)
    p[:, 1:, 1:] = x
    cols = [p[:, u:u + h - 1:2, v:v + w - 1:2] for u in range(3) for v in range(3)]
    return np.concatenate([q[:, :h // 2, :w // 2] for q in cols], axis=3).reshape(-1, 9 * c)


def _cnn_fp32(weights, frames, dtype):
    x = ((ho.frames_to_f64(frames, dtype) - 0.5) * 4.0).astype(np.float32)
    for w, b in weights.tensors["convs"]:
        n, h = x.shape[0], x.shape[1]
        wk = np.transpose(w, (2, 3, 1, 0)).reshape(-1, w.shape[0])
        x = np.maximum(_sum4(_columns(x), wk) + b, np.float32(0)).reshape(n, h // 2, h // 2, -1)
    return x.astype(np.float64).mean(axis=(1, 2)) @ weights.tensors["Wfc"].astype(np.float64) + weights.tensors["bfc"]


@pytest.mark.parametrize("hw,widths", [(16, (1024, 1024)), (16, (256, 512)), (16, (128, 128, 128, 128)), (4, (1024, 16))])
def test_layerwise_fp32_error(hw, widths):
    n = 32
    cfg = hs.WorkloadConfig(name="t", index=0, n=n, hw=hw, dtype="bf16", data_seed=43, models=[], targets=[(0.5,)])
    frames = hs.make_frames(cfg, 0, n)
    w = hs.make_model(hs.ModelDesc(arch="cnn", seed=7, in_hw=hw, widths=widths))
    s = hydro.Session([hydro.ModelSpec.from_weights(w, MASK)], hydro.make_policy("score"), hw, n)
    z = s.logits(0, 1, torch.from_numpy(frames).cuda(), "bf16")
    s.close()
    z64 = ho.model_logits(w, frames, "bf16")
    got, bound = (np.sqrt(((v - z64) ** 2).mean()) for v in (z, _cnn_fp32(w, frames, "bf16")))
    log(f"[gpu] layer-wise {hw} {widths}: FP32 rms error {got:.3e}, fp32 sums of four products {bound:.3e}")
    assert got <= bound


def _bf16(x):
    u = x.astype(np.float32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)


def _sum_terms(x, w):
    """x @ w from three bf16 terms of w, the sum rounded to fp32 after 32 products of each, smallest first."""
    hi = _bf16(w)
    mid = _bf16(w - hi)
    terms = [t.astype(np.float64) for t in ((w - hi) - mid, mid, hi)]
    acc = np.zeros((x.shape[0], w.shape[1]), dtype=np.float32)
    x = x.astype(np.float64)
    for k in range(0, x.shape[1], 32):
        for t in terms:
            acc = (acc + x[:, k:k + 32] @ t[k:k + 32]).astype(np.float32)
    return acc


@pytest.mark.parametrize("hw,hidden,dtype,n,parts,block", [
    (64, 512, "bf16", 2048, 8, 64),        # three bf16 terms
    (64, 2048, "bf16", 600, 7, 64),
    (32, 256, "bf16", 5000, 7, 64),
    (32, 256, "f32", 5000, 7, 16),         # fp32 MFMAs
    (64, 2048, "u8", 600, 7, 16),
])
def test_mlp_fp32_error(hw, hidden, dtype, n, parts, block):
    rows, d_in = 64, hw * hw * 3
    cfg = hs.WorkloadConfig(name="t", index=0, n=n, hw=hw, dtype=dtype, data_seed=44, models=[], targets=[(0.5,)])
    some = hs.make_frames(cfg, 0, rows)
    w = hs.make_model(hs.ModelDesc(arch="mlp", seed=5, d_in=d_in, hidden=hidden))
    frames = torch.from_numpy(some).cuda().repeat(-(-n // rows), 1, 1, 1)[:n].contiguous()
    s = hydro.Session([hydro.ModelSpec.from_weights(w, MASK)], hydro.make_policy("score"), hw, n)
    z = s.logits(0, 1, frames, dtype)[:rows]
    s.close()
    z64 = ho.model_logits(w, some, dtype)
    # the folded form: raw values times s W1, the normalisation in the bias
    scale = 4.0 / 255.0 if dtype == "u8" else 4.0
    t = {k: v.astype(np.float64) for k, v in w.tensors.items()}
    wf = (t["W1"] * scale).astype(np.float32)
    raw = (ho.frames_to_f64(some, dtype) * (255.0 if dtype == "u8" else 1.0)).reshape(rows, -1)
    cuts = [d_in // block * p // parts * block for p in range(parts + 1)]
    pre = np.zeros((rows, hidden), dtype=np.float32)
    for lo, hi in zip(cuts, cuts[1:]):
        pre += (_sum_terms if block == 64 else _sum4)(raw[:, lo:hi], wf[lo:hi])
    h = np.maximum(pre + (t["b1"] - 2.0 * t["W1"].sum(axis=0)).astype(np.float32), np.float32(0))
    got, bound = (np.sqrt(((v - z64) ** 2).mean()) for v in (z, h.astype(np.float64) @ t["W2"] + t["b2"]))
    log(f"[gpu] MLP {d_in}-{hidden} {dtype}, {n} rows: FP32 rms error {got:.3e}, fp32 sums in {parts} parts {bound:.3e}")
    assert got <= bound


# rms errors over these frames with the taps of layers 3 and 4 in row order and every product added to the running
# sum, measured: the limits for any other order
ROW_ORDER_RMS = {"u8": (1.3801e-7, 1.3577e-7, 1.0567e-7, 1.7617e-7),
                 "bf16": (1.3124e-7, 1.1968e-7, 1.0091e-7, 1.5069e-7)}


@pytest.mark.parametrize("dtype", ["u8", "bf16"])
@pytest.mark.parametrize("model", range(4))
def test_cnn4_fp32_error(model, dtype):
    n = 512
    cfg = hs.workload(5)
    frames = hs.make_frames(cfg, 0, n)
    if dtype == "bf16":
        frames = hs.f64_to_bf16_bits(frames.astype(np.float64) / 255.0)
    dev = torch.from_numpy(frames.view(np.int16) if dtype == "bf16" else frames).cuda()
    s = hydro.Session([hydro.ModelSpec.from_weights(hs.make_model(cfg.models[model]), MASK)], hydro.make_policy("score"),
                      128, n)
    z64 = s.logits(0, 2, dev, dtype)
    for part in (n, 100):                   # large tiles, few-frame tiles
        e = np.sqrt(((s.logits(0, 1, dev[:part], dtype) - z64[:part]) ** 2).mean())
        log(f"[gpu] 4-layer CNN {model} {dtype}, {part} frames: FP32 rms error {e:.4e}")
        if part == n:
            assert e <= ROW_ORDER_RMS[dtype][model]
    s.close()
