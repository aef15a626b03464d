"""Real-time updates (Eq. 9) at sizes where the update's kernels split rows and
columns differently, wide and tall frames, with a frame that does not track,
against the FP64 oracle."""
import numpy as np
import pytest

from oracle import ccpt_oracle as O
from tests.test_gpu_window import spots, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx", [(16, 16), (18, 18), (54, 54), (64, 64), (108, 108), (162, 162), (324, 324),
                                   (512, 512), (512, 256), (256, 512), (128, 1024)])
@pytest.mark.parametrize("mode", ["ccu", "ccsn"])
def test_updates_match_the_oracle(ny, nx, mode):
    print(f"case: {ny}x{nx}, {mode}, four frames with a0 = 0.25", flush=True)
    from paper_2310_08770_amd import Tracker, decode
    from paper_2310_08770_amd.reference import realtime_track
    fr, _ = spots(4, ny, nx, 1.9 if ny < 32 else 3.0, 900.0, 30.0, ny + nx)
    frames = [np.round(f).astype(np.float32) for f in fr]
    om = O.MODE_CCU if mode == "ccu" else O.MODE_CCSN
    want = O.realtime_track(frames, 37, 0.25, om, 200.0)
    bad = frames[:2] + [np.full_like(frames[0], np.nan)] + frames[2:]  # leaves the reference as it is
    tr = Tracker(upsample=37, mode=mode, eps=200.0)
    got = decode(realtime_track(tr, t(np.stack(bad)), 0.25))
    tr.close()
    assert got["status"][2] & O.NONFINITE
    keep = [0, 1, 3, 4]
    assert np.array_equal(got["p"][keep], np.array([x["p"] for x in want]))
    # the bound of the other real-time tests
    assert np.max(np.abs(got["d"][keep] - np.array([x["d"] for x in want]))) <= 1e-3
