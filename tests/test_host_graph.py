"""Captured launches are replayed only for calls that would launch the same."""
import torch

from tests._host import host, host_lib  # noqa: F401

STREAM = 1  # (a stream of its own: the default stream is not captured)


def test_a_graph_serves_only_frames_of_its_pixel_layout(host):
    n = 130  # enough for the one-kernel correlation, which reads pixel pairs
    tr = host.tracker(graph=True)
    tr.set_reference(torch.ones(256, 256), stream=STREAM)
    out = torch.empty(n, 72, dtype=torch.uint8)
    pixels = torch.zeros(256 * 257 * n + 1)
    pairs = pixels[:256 * 256 * n].view(n, 256, 256)
    odd = pixels[:256 * 257 * n].view(n, 256, 257)[:, :, :256]  # odd pitch
    doubles = torch.zeros(n, 256, 256, dtype=torch.float64)
    for frames, ok in ((pairs, 1), (doubles, 0), (pairs, 1), (odd, 0), (doubles, 0)):
        tr.track(frames, out=out, stream=STREAM)
        assert host.launches() == [(256, 256, n, 1, ok)]
