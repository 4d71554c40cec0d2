"""GPU parity of the batched MLP workload (64x64x3 bf16 frames, six MLP 12288-h-10 predicates,
h = 256 ... 2048, grouped into one launch per tier) against the FP64 oracle."""
import numpy as np
import pytest

import hydro_synth as hs
from oracle import hydro_oracle as ho
from tests.gpu_util import case, check_stats, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402


@pytest.fixture(scope="module")
def c3():
    return case(3, 4096)


@pytest.fixture(scope="module")
def c3z():
    return case(3, 512, logits=True)


@pytest.fixture(scope="module")
def calib_frames():
    cfg = hs.workload(3)
    return torch.from_numpy(hs.make_frames(cfg, 0, 1024, data_seed=cfg.data_seed + 101)).cuda()


def test_mlp6_logits_each_tier(c3z):
    s = hydro.Session(c3z.specs(), hydro.make_policy("score", precision="bf16"), 64, c3z.n)
    dev = c3z.device_frames()
    for k in range(c3z.cfg.k):
        for tier, tol in ((0, 0.06), (1, 4e-5), (2, 1e-12)):      # measured 2.3e-2, 8.3e-6, 4.9e-15
            err = np.abs(s.logits(k, tier, dev, "bf16") - c3z.Z[k]).max()
            log(f"[gpu] mlp6 predicate {k} (h={c3z.cfg.models[k].hidden}) tier {tier}: max |z - z64| = {err:.3e}")
            assert err <= tol
    s.close()


@pytest.mark.parametrize("route", ["score", "fixed", "learned"])
def test_mlp6_calibrated_query(c3, calib_frames, route):
    pol = hydro.make_policy(route, precision="bf16", wave=1024, log_routes=1)
    s = hydro.Session(c3.specs(), pol, 64, c3.n)
    tau, tau32 = s.calibrate(calib_frames, "bf16", safety=3.0)
    log(f"[gpu] mlp6 calibrated tau={np.round(tau, 5).tolist()} tau32={tau32.tolist()}")
    s.push(c3.device_frames(), "bf16", c3.pt.thresholds, c3.seg_len)
    ids, stats = s.finish()
    log(f"  |R|={ids.size} evaluated={[st['evaluated'] for st in stats]} rescored={[st['rescored'] for st in stats]}")
    assert np.array_equal(ids, c3.expect)
    check_stats(stats, c3.n, ids.size)
    ok, rev, rps, out, msg = ho.replay_route(c3.P, hydro.decode_routes(s.routes(0, c3.n)))
    assert ok, msg
    if route == "fixed":
        _, ev, ps = ho.short_circuit_eval(c3.P, list(range(6)))
        assert [st["evaluated"] for st in stats] == list(ev)
    s.close()


def test_mlp6_ungrouped_matches(c3):
    """One launch per predicate (the plain form) against the grouped launch, written order: the
    same ids, evaluations and FP64 escalations (each predicate must run its own weights: with
    another predicate's, its FP32 margins would land in the FP64 band far more often)."""
    order = list(range(c3.cfg.k))
    out = {}
    for grouped in (0, 1):
        pol = hydro.make_policy("fixed", order=order, precision="fp32", wave=2048, grouped=grouped, tau32=1e-4)
        ids, stats = hydro.query(c3.device_frames(), "bf16", c3.specs(), c3.pt.thresholds, c3.seg_len, pol)
        assert np.array_equal(ids, c3.expect)
        out[grouped] = [(st["evaluated"], st["escalated"]) for st in stats]
    log(f"[gpu] mlp6 fp32 (evaluated, escalated) ungrouped {out[0]} grouped {out[1]}")
    assert [v for v, _ in out[0]] == [v for v, _ in out[1]]
    # split-K may split the two launches' K ranges differently (last-bit differences at the band
    # edge), so the escalations agree to a few tuples, and stay a small fraction
    assert all(abs(a[1] - b[1]) <= 3 for a, b in zip(out[0], out[1]))
    assert sum(e for _, e in out[0]) <= 0.01 * sum(v for v, _ in out[0])


@pytest.mark.parametrize("n", [1, 17, 256, 257, 2048 + 1, 9000])
@pytest.mark.parametrize("tier", [0, 1])
def test_mlp_whole_and_split_tiles(n, tier):
    """Queues whose tiles all split along K (few rows), fill the GPU exactly or leave a split rest
    behind whole tiles, rows that do not fill a tile: logits against FP64 numpy.  Rounding errors are
    independent: a bf16 weight's has a standard deviation below 2^-9 of it, each of 768 fp32 sums
    one below 2^-24 of a partial sum (within four standard deviations of the products' sum);
    eight of the logit's standard deviation bound every row (a lost or doubled part is about 1)."""
    d_in, hidden = 768, 2048
    rng = np.random.default_rng(n)
    frames = hs.f64_to_bf16_bits(rng.random((n, 16, 16, 3)))
    w = hs.make_model(hs.ModelDesc(arch="mlp", seed=910, d_in=d_in, hidden=hidden))
    s = hydro.Session([hydro.ModelSpec.from_weights(w, 0b0000011111)], hydro.make_policy("score", precision="bf16"), 16, n)
    z = s.logits(0, tier, torch.from_numpy(frames).cuda(), "bf16")
    s.close()
    x = (ho.frames_to_f64(frames, "bf16").reshape(n, -1) - 0.5) * 4.0
    t = {k: v.astype(np.float64) for k, v in w.tensors.items()}
    pre = x @ t["W1"] + t["b1"]
    z64 = np.maximum(pre, 0.0) @ t["W2"] + t["b2"]
    # the folded form multiplies the raw frame (at most 1) by 4 W1
    size = 4.0 * np.sqrt((t["W1"] ** 2).sum(axis=0))
    sigma = size * 2.0**-9 if tier == 0 else 4.0 * size * np.sqrt(d_in) * 2.0**-24
    bound = 8.0 * np.sqrt((sigma**2) @ (t["W2"] ** 2))
    err = np.abs(z - z64).max(axis=0)
    log(f"[gpu] mlp {n} rows tier {tier}: max |z - z64| {err.max():.3e}, bound {bound.min():.3e}")
    assert np.all(err <= bound)


# both sides sum at most 4,800 and 384 products in FP64, a few 1e-16 relative each (the same tolerance as the
# other FP64 tier tests)
@pytest.mark.parametrize("cap", ["2", "128"])
@pytest.mark.parametrize("hw,n", [(8, 1), (16, 5), (24, 7), (16, 17), (40, 23), (16, 130), (8, 260)])
def test_f64_tier_splits(monkeypatch, cap, hw, n):
    """FP64 tier: groups of 8 entries that are not full, whole and cut 256-long parts of the input, two
    blocks of hidden units with the second half full, and more entries than esc_cap (longer chunks)
    and than its room (one group per block)."""
    monkeypatch.setenv("HYDRO_ESC_CAP", cap)
    d_in, hidden = hw * hw * 3, 384
    frames = hs.f64_to_bf16_bits(np.random.default_rng(n).random((n, hw, hw, 3)))
    w = hs.make_model(hs.ModelDesc(arch="mlp", seed=911, d_in=d_in, hidden=hidden))
    s = hydro.Session([hydro.ModelSpec.from_weights(w, 0b0000011111)], hydro.make_policy("score", precision="bf16"), hw, n)
    z = s.logits(0, 2, torch.from_numpy(frames).cuda(), "bf16")
    s.close()
    z64 = ho.model_logits(w, frames, "bf16")
    err = np.abs(z - z64).max()
    log(f"[gpu] FP64 mlp {hw}x{hw}, {n} entries, cap {cap}: max |z - z64| = {err:.3e}")
    assert err <= 1e-12


# fp32 sums of 192 or 768 products: the tolerance of the other fp32 MLP tests, 3e-5
@pytest.mark.parametrize("dtype", ["u8", "bf16", "f32"])
@pytest.mark.parametrize("hw,hidden", [(8, 128), (8, 384), (16, 256)])
def test_folded_weights(dtype, hw, hidden):
    """The folded weights and biases that a session makes on the device, in the forms of the tiers and of
    each frame type's scale."""
    n = 70
    cfg = hs.WorkloadConfig(name="t", index=0, n=n, hw=hw, dtype=dtype, data_seed=5, models=[], targets=[(0.5,)])
    frames = hs.make_frames(cfg, 0, n)
    w = hs.make_model(hs.ModelDesc(arch="mlp", seed=912, d_in=hw * hw * 3, hidden=hidden))
    z64 = ho.model_logits(w, frames, dtype)
    s = hydro.Session([hydro.ModelSpec.from_weights(w, 0b0000011111)], hydro.make_policy("score", precision="bf16"), hw, n)
    dev = torch.from_numpy(frames).cuda()
    err = [np.abs(s.logits(0, t, dev, dtype) - z64).max() for t in (0, 1)]
    s.close()
    log(f"[gpu] folded weights {hw}x{hw} {dtype} {hidden}: max |z - z64| {err[0]:.3e}, {err[1]:.3e}")
    assert err[0] <= 0.08 and err[1] <= 3e-5
