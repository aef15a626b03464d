"""A graph captured for frames that the one-kernel correlation reads, then the
same call (count, output, stream) with frames of another pixel layout: each
result is the eager one's."""
import numpy as np
import pytest
import torch

from tests.test_gpu_window import spots, t

pytestmark = pytest.mark.gpu


def test_graphs_of_other_pixel_layouts():
    n = 130
    print(f"case: {n} frames of 256x256 by graph: uint16, float64, odd pitch, uint16", flush=True)
    from paper_2310_08770_amd import Tracker, decode
    fr, ref = spots(5, 256, 256, 3.0, 900.0, 30.0, 6)
    u16 = t(np.round(fr).astype(np.int16))[[i % 5 for i in range(n)]].contiguous()  # (uint16 bits)
    wide = torch.zeros(n, 256, 257, dtype=torch.int16, device=u16.device)
    wide[:, :, :256] = u16
    f64 = u16.to(torch.float64)
    eager, graph = Tracker(upsample=50), Tracker(upsample=50, graph=True)
    for tr in (eager, graph):
        tr.set_reference(t(ref))
    out = torch.empty(n, 72, dtype=torch.uint8, device=u16.device)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for frames in (u16, f64, wide[:, :, :256], u16):
        want = decode(eager.track(frames))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            out.zero_()
            graph.track(frames, out=out, stream=side)
        side.synchronize()
        assert decode(out).tobytes() == want.tobytes()
    eager.close()
    graph.close()
