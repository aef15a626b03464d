"""Launch plans and the tuners, by the launches that they lead to."""
import json
from types import SimpleNamespace

import pytest
import torch

from tests._host import host, host_lib  # noqa: F401


def run(host, tr, count, n, dtype=torch.float32):
    frame = torch.zeros(n, n, dtype=dtype)
    tr.track([frame] * count, [0] * count, stream=0)
    return host.launches()


@pytest.mark.parametrize("n", [16, 64, 256, 512])
@pytest.mark.parametrize("precision", ["fp32", "bf16x2", "fp64"])
def test_a_plan_that_is_read_and_written_back_changes_nothing(host, n, precision):
    tr = host.tracker(precision=precision)
    tr.set_reference(torch.ones(n, n), stream=0)
    counts = (1, 100, 481, 762, 961, 1500, 6000)  # 481 frames of 256 x 256: 381 in one kernel, 100 in passes
    want = [run(host, tr, c, n) for c in counts]
    plan = tr.plan(n)
    for write in (lambda: tr.set_plan(n, **plan), lambda: tr.set_chunk(n, tr.chunk(n)), lambda: tr.set_plan(n)):
        write()
        assert tr.plan(n) == plan
        assert [run(host, tr, c, n) for c in counts] == want
    # any other chunk is taken as it is
    tr.set_plan(n, chunk=48)
    assert tr.plan(n)["chunk"] == 48
    assert [l[2] for l in run(host, tr, 100, n)] == [48, 48, 4]


def test_autotune_keeps_the_default_unless_it_is_beaten(host):
    # (in the model a launch takes the same time whatever its size, and 900 frames
    # are one default launch, a quarter over 768: every chunk makes two or more)
    tr = host.tracker()
    tr.set_reference(torch.ones(256, 256), stream=0)
    plan = tr.plan(256)
    assert tr.autotune(256, 900, stream=0) == plan["chunk"]
    assert tr.plan(256) == plan
    host.launches()
    assert len(run(host, tr, 900, 256)) == 1
    # two launches beat the three of the default (the first chunk that makes two)
    tr.autotune(256, 2000, stream=0)
    assert tr.plan(256)["chunk"] == 1024


def test_cached_plans_are_whole_and_of_these_kernels(host, monkeypatch, tmp_path):
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: SimpleNamespace(gcnArchName="gfx950", name=""))
    cache = str(tmp_path / "plans.json")
    # a chunk kept for other kernels is not applied, and is left in the file
    old = {"gfx950|N=256|batch=900|u=100|prec=0|mode=0": 16}
    with open(cache, "w") as fh:
        json.dump(old, fh)

    def tracker():
        tr = host.tracker()
        tr.set_reference(torch.ones(256, 256), stream=0)
        return tr

    a = tracker()
    chunk = a.autotune(256, 900, stream=0, cache=cache)
    assert chunk == a.chunk(256) != 16
    table = json.load(open(cache))
    key, = set(table) - set(old)
    assert table[key] == a.plan(256) and old.items() <= table.items()
    # every field of a kept plan is applied, without timing anything
    table[key] = dict(chunk=512, split_blocks=512, fused_min=1)
    with open(cache, "w") as fh:
        json.dump(table, fh)
    b = tracker()
    host.launches()
    assert b.autotune(256, 900, stream=0, cache=cache) == 512
    assert b.plan(256) == table[key] and host.launches() == []
