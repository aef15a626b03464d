"""Frames that the one-kernel correlation in LDS takes (csrc/xcorr_lds.hip)
against the three passes, which timed launches take: the whole result records
are equal, bit for bit."""
import numpy as np
import pytest
import torch

from tests.test_gpu_window import spots, t

pytestmark = pytest.mark.gpu

SHAPES = [(n, n) for n in (16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192)] + [(256, 128), (128, 256)]


@pytest.mark.parametrize("ny,nx", SHAPES)
def test_same_bits_as_the_passes(ny, nx):
    from paper_2310_08770_amd import Tracker, decode
    fr, ref = spots(5, ny, nx, max(1.2, min(ny, nx) / 40), 900.0, 30.0, 8)
    fr = np.maximum(np.round(fr), 0.0)
    # below and above 128 frames, and (sizes that have a CU each) past a round of 256
    counts = (3, 130) if ny * (nx // 2 + 1) <= 8320 else (130, 300)
    for mode in ("ccu", "ccsn"):
        lds, passes = (Tracker(upsample=37, mode=mode, profile=p) for p in (False, True))
        for tr in (lds, passes):
            tr.set_reference(t(np.maximum(ref, 0.0)))
        for dtype in (np.int16, np.float32, np.float64):  # (int16: uint16 bits)
            x = t(fr.astype(dtype))
            for count in counts:
                print(f"case: {count} frames of {ny}x{nx}, {mode}, {np.dtype(dtype).name}", flush=True)
                frames = [x[i % 5] for i in range(count)]
                got, want = (decode(tr.track(frames, [0] * count)) for tr in (lds, passes))
                torch.cuda.synchronize()
                assert got.tobytes() == want.tobytes()
        lds.close()
        passes.close()
