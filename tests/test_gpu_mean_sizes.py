"""Aligned mean at sizes and frame counts where its kernels split the work
differently, against the FP64 oracle: frames that fit LDS, passes, and both in
one call; sums shorter and longer than a thread's loads in flight."""
import numpy as np
import pytest
import torch

from oracle import ccpt_oracle as O
from tests.test_gpu_reference import rel_err, results_with
from tests.test_gpu_window import spots, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,count", [(16, 1), (24, 33), (54, 32), (64, 65), (108, 31), (128, 2), (144, 40),
                                     (162, 258), (192, 129), (192, 5), (256, 34), (324, 3)])
@pytest.mark.parametrize("dtype", ["u16", "f32", "f64"])
def test_mean_aligned(n, count, dtype):
    print(f"case: aligned mean of {count} {dtype} frames of {n}x{n}", flush=True)
    from paper_2310_08770_amd import Tracker
    fr, _ = spots(4, n, n, 1.9 if n < 32 else 3.0, 900.0, 30.0, 7 * n)
    fr = np.round(fr).astype({"u16": np.uint16, "f32": np.float32, "f64": np.float64}[dtype])
    frames = fr[np.arange(count) % 4]
    rng = np.random.Generator(np.random.PCG64(n + count))
    ds = rng.uniform(-2, 2, (4, 2))[np.arange(count) % 4]
    st = np.zeros(count, np.uint32)
    st[count // 2 + 1:count // 2 + 2] = O.FLAT
    if dtype != "u16" and count > 1:
        frames = frames.copy()
        frames[count // 2 + 1:count // 2 + 2] = np.nan
    pad = 1 if n % 16 else 0  # a pitch with pixels to spare
    buf = np.zeros((count, n, n + pad), frames.dtype)
    buf[:, :, :n] = frames
    tr = Tracker(upsample=20)
    got = tr.mean_aligned(t(buf)[:, :, :n], results_with(ds, st)).cpu().numpy()
    tr.close()
    # the oracle's mean of the distinct frames, weighted by how often each counts
    used = np.flatnonzero(st == 0)
    want = sum(O.mean_aligned([fr[k]], [ds[k]]) * np.sum(used % 4 == k)
               for k in range(min(4, count))) / used.size
    # 2e-6: the FP32 transforms; 2^-24 an addition: the sum in frame order
    assert rel_err(got, want) <= 2e-6 + count * 2.0 ** -24
