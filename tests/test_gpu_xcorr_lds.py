"""The one-kernel correlation of small frames (csrc/xcorr_lds.hip) against the
three passes, which keep the same order of operations: the same integer peak
and status, displacements equal to the rounding of the FP64 sums that follow
(their order changes with the launch size: 1e-12 px)."""
import numpy as np
import pytest
import torch

from oracle import ccpt_oracle as O
from tests.test_gpu_window import spots, t

pytestmark = pytest.mark.gpu


def frames_as(fr, kind):
    """The frames with a dtype and row pitch that select each way of reading."""
    n, ny, nx = fr.shape
    dt, pad = {"u16": (np.uint16, 0), "u16_odd": (np.uint16, 3), "f32": (np.float32, 4),
               "f32_odd": (np.float32, 1), "f64": (np.float64, 0)}[kind]
    buf = np.full((n, ny, nx + pad), 9, dt)
    buf[:, :, :nx] = fr
    return t(buf)[:, :, :nx]


@pytest.mark.parametrize("kind", ["u16", "u16_odd", "f32", "f32_odd", "f64"])
@pytest.mark.parametrize("ny,nx", [(144, 144), (162, 162), (192, 192), (256, 128), (128, 256)])
def test_rounds_and_rest_match_the_three_passes(ny, nx, kind):
    """300 frames: one round of 256 in the one kernel, 44 in three passes; 100
    at a time: three passes; 128: one kernel; CC-SN."""
    from paper_2310_08770_amd import Tracker, decode
    print(f"case: {ny}x{nx} {kind}", flush=True)
    few, ref = spots(20, ny, nx, 3.0, 900.0, 20.0, ny * 7 + nx)
    fr = np.concatenate([few] * 15)
    fr[3] = 11.0  # flat
    x = frames_as(fr, kind)
    if kind[0] == "f":
        x[280, 5, 7] = float("nan")
        x[7, ny - 1, nx - 1] = float("inf")
    tr = Tracker(mode="ccsn", upsample=20)
    tr.set_reference(t(ref.astype(np.float32)))
    whole = decode(tr.track(x))
    parts = np.concatenate([decode(tr.track(x[i:i + 100])) for i in (0, 100, 200)])
    mid = decode(tr.track(x[100:228]))
    tr.close()
    assert whole["status"][3] == O.FLAT
    for a, b in ((whole, parts), (whole[100:228], mid)):
        assert np.array_equal(a["p"], b["p"]) and np.array_equal(a["status"], b["status"])
        ok = (a["status"] & (O.NONFINITE | O.FLAT)) == 0
        assert np.max(np.abs(a["d"][ok] - b["d"][ok])) <= 1e-12
        assert np.all(np.isnan(a["d"]) == np.isnan(b["d"]))


@pytest.mark.parametrize("kind", ["u16", "u16_odd", "f32", "f64"])
@pytest.mark.parametrize("N", [16, 18, 24, 36, 48, 72, 96, 108, 128])
def test_small_frames_vs_oracle(N, kind):
    """Every size class (powers of two padded in LDS, factors of three not) and
    way of reading against the oracle: integer peak and status exact, 1e-3 px."""
    from paper_2310_08770_amd import Tracker, decode
    print(f"case: {N}x{N} {kind}", flush=True)
    fr, ref = spots(5, N, N, 1.9 if N < 32 else 3.0, 900.0, 20.0, N)
    ref = ref.astype(np.float32)
    tr = Tracker(upsample=20)
    tr.set_reference(t(ref))
    res = decode(tr.track(frames_as(fr, kind)))
    tr.close()
    for i in range(5):
        o = O.track(fr[i], ref.astype(np.float64), 20)
        assert tuple(res["p"][i]) == tuple(o["p"])
        assert int(res["status"][i]) & O.NEAR_TIE == o["status"] & O.NEAR_TIE
        if not o["status"] & (O.NEWTON_FALLBACK | O.WINDOW_EXIT):
            assert np.max(np.abs(res["d"][i] - o["d"])) <= 1e-3
