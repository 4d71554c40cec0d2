"""The allocation-free query's limit is the size that the header states, whatever the library's array takes beyond
it: a query whose buffers need more is refused, one that needs less runs."""
import numpy as np
import pytest

import hydro_synth as hs
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402

LIMIT = 128 << 20         # HYDRO_NOALLOC_BYTES


def test_queries_beyond_the_stated_size_are_refused():
    k, d_in, hidden = 2, 3072, 256
    # what two MLPs cannot do without there, a tuple and in all: partial logits of 32 hidden units, live lists, three
    # tiers' queues, result bit and id; fp32 weights twice, bf16 weights, 128 tiles of split sums, 8 entries of
    # 256-long chunks in fp64
    per_tuple = k * (hidden // 32) * 10 * 4 + 2 * 4 + 3 * k * 4 + 1 / 8 + 8
    fixed = k * d_in * hidden * 10 + 128 * 128 * 128 * 4 + k * (d_in // 256) * 8 * hidden * 8
    n = int((LIMIT - fixed) / per_tuple) + 1
    weights = [hs.make_model(hs.ModelDesc(arch="mlp", seed=5 + i, d_in=d_in, hidden=hidden)) for i in range(k)]
    specs = [hydro.ModelSpec.from_weights(w, 0b0000011111) for w in weights]
    frames = torch.zeros((n, 32, 32, 3), dtype=torch.int16, device="cuda")
    th = np.full((1, k), 1e9, dtype=np.float32)
    pol = hydro.make_policy("score", tau=1e-3, tau32=1e-6)
    log(f"[gpu] allocation-free query: {n} tuples are more than {LIMIT} bytes")
    with pytest.raises(hydro.HydroError) as e:
        hydro.query_noalloc(frames, "bf16", specs, th, n, pol, out_cap=n)
    assert e.value.code == hydro.ECAPACITY and str(LIMIT) in str(e.value)
    m = n - 1000              # (state, thresholds and the rounding of each buffer to 256 bytes: far below 680,000)
    ids, _ = hydro.query_noalloc(frames[:m], "bf16", specs, th, m, pol, out_cap=m)
    assert ids.size == 0
