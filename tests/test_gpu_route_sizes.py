"""Queries whose rounds fall on both sides of the router's chunk lengths (a thread takes one to eight
tuples) and whose result bitmap is one launch's or three launches' work, against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import case, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2403_14902_amd import hydro  # noqa: E402


# 32 tuples a bitmap word, 1,024 words a launch; 64 chunks of 256 threads x 1 .. 8 tuples
@pytest.mark.parametrize("n", [1, 33, 257, 16385, 32768, 32769])
@pytest.mark.parametrize("reuse", [0, 2])
def test_ids_at_chunk_and_bitmap_edges(n, reuse):
    c = case(1, n)
    s = hydro.Session(c.specs(), hydro.make_policy("score", precision="bf16", wave=1 << 17, reuse=reuse), 32, n)
    for turn in range(2):        # (with reuse, the second query takes its decisions from the cache)
        s.push(c.device_frames(), c.cfg.dtype, c.pt.thresholds, c.seg_len)
        ids, _ = s.finish()
        assert np.array_equal(ids, c.expect), turn
        s.reset()
    s.close()
    log(f"[gpu] {n} tuples, reuse {reuse}: |R| = {c.expect.size}")


@pytest.mark.parametrize("wave", [64, 256, 16384, 32768, 262144])
def test_compaction_waves_at_chunk_lengths(wave):
    # 300,000 tuples through three predicates of random decisions: the survivors in ascending order
    n, k = 300_000 if wave >= 16384 else 3_000, 3
    rng = np.random.default_rng(wave)
    bits = rng.random((k, n)) < 0.7
    packed = np.zeros((k, (n + 31) // 32), dtype=np.uint32)
    for j in range(k):
        b = np.zeros(packed.shape[1] * 32, dtype=np.uint8)
        b[:n] = bits[j]
        packed[j] = np.packbits(b.reshape(-1, 32), axis=1, bitorder="little").view(np.uint32).ravel()
    out = torch.zeros(n, dtype=torch.int64, device="cuda")
    cnt, _, _ = hydro.compaction_debug(k, n, torch.from_numpy(packed.view(np.int32)).cuda(), out, route="score", wave=wave)
    assert np.array_equal(out[:cnt].cpu().numpy(), np.nonzero(bits.all(axis=0))[0])
