"""The expansion of the correlation on the window (csrc/refine.hip): the grid
maximum, C and its Hessian against direct FP64 sums over the spectrum, at the
edges of its tiles (16 columns, 4 row pairs, 32 grid points), for odd and even
M, the widest window, launches that spread a frame over blocks, and iterates
that leave the window."""
import numpy as np
import pytest
import torch

from oracle import ccpt_oracle as O
from synth import frames as S

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def t(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def spots(n, ny, nx, sigma, peak, bg, seed, spread=1.5):
    rng = np.random.Generator(np.random.PCG64(seed))
    y, x = np.arange(ny) - ny / 2, np.arange(nx) - nx / 2
    spot = S.zero_nyquist(peak * np.exp(-0.5 * (y[:, None] ** 2 + x[None, :] ** 2) / sigma ** 2))
    d = rng.uniform(-spread, spread, (n, 2))
    fr = np.stack([S.noisy(S.phase_ramp_shift(spot, e) + bg, rng) for e in d])
    return fr, spot + bg


def grid(X, p, u, window):
    """U on the M x M grid of a window of any side (the oracle's own is 1.5 px)."""
    M = int(np.ceil(window * u - 1e-9))
    off = (np.arange(M) - M // 2) / u
    ny, nx = X.shape
    Ky = np.stack([O.phi(ny, p[0] + o) for o in off])
    Kx = np.stack([O.phi(nx, p[1] + o) for o in off])
    return (Ky @ X @ Kx.T).real / (ny * nx), off


def check(res, fr, ref, u, window, mode, tol_grid, tol_c, idx):
    for i in idx:
        A, B = O.weights(fr[i].astype(np.float64), ref, mode, 200.0)
        X = O.cross_power(A, B)
        r = res[i]
        U, off = grid(X, r["p"], u, window)
        my, mx = [int(np.argmin(np.abs(off - (r["d_grid"][a] - r["p"][a])))) for a in range(2)]
        ac = abs(U.max() - X[0, 0].real / X.size)
        # the grid value at the reported point lies within rounding of the maximum
        assert U.max() - U[my, mx] <= tol_grid * ac, (i, U.max() - U[my, mx], ac)
        if r["status"] & (O.NEWTON_FALLBACK | O.WINDOW_EXIT):
            continue
        c, _, H = O.gradient_hessian(X, r["d"])
        h = np.array([H[0, 0], H[0, 1], H[1, 1]])
        assert abs(r["peak"] - c) <= tol_c * abs(c)
        assert np.max(np.abs(r["hess"] - h)) <= tol_c * max(np.max(np.abs(h)), ac)


# FP64: the series stops below FP64 rounding (2 J_24(pi B) < 1e-17 at B = 1.05),
# 1e3 roundings for the sums; the grid maximum exact but for such rounding.
# FP32: the FP32 spectrum's 2^-20 of AC per grid value (tests/_parity.py), and
# 1e-5 for sums over FP32 spectra (a few 2^-24 sqrt(NX NY) of the largest terms).
TOL = {"fp64": (1e-12, 2e-13), "fp32": (2.0 ** -20, 1e-5)}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("N,u,window", [
    (16, 1, 1.5), (18, 20, 1.5), (32, 21, 1.0), (36, 64, 2.0), (54, 43, 1.5), (162, 10, 2.0),
    (162, 85, 0.5), (256, 22, 1.5), (216, 2, 1.9), (486, 33, 1.5)])
def test_window_expansion_square(N, u, window, prec):
    """M = 2 .. 128: one strip, exactly one, one more than whole strips; 8 to
    243 columns; 9 to 244 row pairs; odd M and M even."""
    from paper_2310_08770_amd import Tracker, decode
    print(f"case: {N}x{N} u={u} window={window} {prec}", flush=True)
    fr, ref = spots(4, N, N, 1.8 if N < 32 else 3.0, 900.0, 20.0, 1000 * N + u)
    tr = Tracker(upsample=u, window=window, precision=prec)
    tr.set_reference(t(ref))  # float64: both sides use the same values
    res = decode(tr.track(t(fr if prec == "fp64" else fr.astype(np.float32))))
    r64 = ref if prec == "fp64" else ref.astype(np.float32).astype(np.float64)
    check(res, fr, r64, u, window, O.MODE_CCU, *TOL[prec], range(4))
    tr.close()


@pytest.mark.parametrize("count", [1, 63, 64, 127, 128, 130])
@pytest.mark.parametrize("ny,nx,u", [(64, 64, 43), (128, 256, 150)])
def test_window_expansion_launch_sizes(ny, nx, u, count):
    """A frame on one block, on four and on one per column tile, its grid on
    one block and on several: the same frames give the same results to FP64
    rounding of the sums (1e-12 px), grid points within FP32 rounding."""
    from paper_2310_08770_amd import Tracker, decode
    print(f"case: {ny}x{nx} u={u}, {count} frames per launch", flush=True)
    fr, ref = spots(130, ny, nx, 3.0, 900.0, 20.0, ny + nx + u)
    frt, reft = t(fr.astype(np.uint16)), t(ref.astype(np.float32))
    tr = Tracker(upsample=u)
    tr.set_reference(reft)
    whole = decode(tr.track(frt))
    part = decode(tr.track(frt[:count]))
    tr.close()
    assert np.array_equal(part["p"], whole["p"][:count])
    assert np.array_equal(part["status"], whole["status"][:count])
    assert np.max(np.abs(part["d"] - whole["d"][:count])) <= 1e-12
    assert np.max(np.abs(part["d_grid"] - whole["d_grid"][:count])) <= 1.0 / u + 1e-6
    check(part, fr, ref.astype(np.float32).astype(np.float64), u, 1.5, O.MODE_CCU, *TOL["fp32"],
          [0, count - 1])


def test_iterates_outside_the_window():
    """A narrow window on a broad spot with the integer peak displaced by
    noise: Newton's first steps leave the series' interval and are evaluated
    from the spectrum; the decisions follow the definition (step limit 0.75 px
    for windows under 1.5 px is half the window, never under a grid step)."""
    from paper_2310_08770_amd import Tracker, decode
    print("case: 64x64, window 0.25, u = 4: steps past the window", flush=True)
    fr, ref = spots(40, 64, 64, 6.0, 60.0, 5.0, 77)
    tr = Tracker(upsample=4, window=0.25, newton_iters=6)  # M = 1, B = 0.175 px, steps up to 0.25
    tr.set_reference(t(ref.astype(np.float32)))
    res = decode(tr.track(t(fr.astype(np.uint16))))
    tr.close()
    r64 = ref.astype(np.float32).astype(np.float64)
    exits = 0
    for i in range(40):
        X = O.cross_power(fr[i], r64)
        s = np.asarray(res["p"][i], np.float64)
        seed, status = s.copy(), 0
        centre, passes = s.copy(), 0
        for it in range(6):
            _, g, H = O.gradient_hessian(X, s)
            step = -np.linalg.solve(H, g)
            if not (H[0, 0] < 0 and np.linalg.det(H) > 0) or np.max(np.abs(step)) > 0.25:
                status, s = status | O.NEWTON_FALLBACK, seed.copy()
                break
            s = s + step
            if it < 5 and np.max(np.abs(s - centre)) > 0.02:
                if passes >= 2:
                    break
                passes, centre = passes + 1, s.copy()
        exits += bool(np.max(np.abs(s - seed)) > 0.175)
        if np.max(np.abs(s - seed)) > 0.125:
            status, s = status | O.WINDOW_EXIT, seed.copy()
        near = abs(np.max(np.abs(s - seed)) - 0.125) < 1e-5
        if not near:
            assert (int(res["status"][i]) & 24) == status, (i, int(res["status"][i]), status)
            assert np.max(np.abs(res["d"][i] - s)) <= 1e-4
    assert exits >= 3, exits  # the case is what it says
