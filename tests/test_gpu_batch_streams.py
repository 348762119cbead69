"""GPU checks of how vktApplyFilterBatched launches its classes: on streams that
fork from the caller's and join it again.  A result equals the single-volume
call's bit for bit, so all comparisons are exact:

- on a stream of the caller's, between its work before (which fills the sources)
  and after (which copies the results), with no synchronisation in between;
- captured into a graph and replayed, also after the cache has dropped the plan;
- with a class deep enough for 64-plane slabs, at and about a slab's edge.

They run in a process of their own, so that the plans that they make are not
added to those of the other tests."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SPECS = [((40, 37, 90), "uint16", 5), ((17, 70, 33), "uint16", 7), ((33, 64, 64), "uint8", 3),
         ((12, 30, 50), "float32", 5), ((6, 96, 70), "float32", 9), ((25, 25, 26), "uint16", 3)]


def test_ordered_with_the_callers_stream():
    run_child("order")


def test_captured_plan_outlives_the_cache():
    run_child("capture")


def test_deep_slabs():
    run_child("depth")


def run_child(what):
    r = subprocess.run([sys.executable, "-u", os.path.abspath(__file__), what], cwd=ROOT,
                       env=dict(os.environ, PYTHONPATH=ROOT), capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and "all equal" in r.stdout, r.stdout + r.stderr


class Batch:
    def __init__(self, torch, vkt, specs=SPECS):
        self.torch, self.vkt = torch, vkt
        self.src, self.dst, self.want = [], [], []
        self.f = []
        for i, (shape, fmt, k) in enumerate(specs):
            dtype = getattr(torch, fmt)
            for out in (self.src, self.dst, self.want):
                out.append(torch.zeros(shape, dtype=torch.uint8 if fmt == "uint8" else torch.int16
                                       if fmt == "uint16" else torch.float32,
                                       device="cuda").view(dtype))
            w = np.abs(np.random.default_rng(k + i).standard_normal((k, k, k))) + 0.1
            self.f.append(vkt.vktFilterCreate((w / w.sum()).astype(np.float32)))
        self.hs, self.hd, self.hw = ([vkt.volume_from_tensor(t) for t in ts]
                                     for ts in (self.src, self.dst, self.want))

    def fill(self, seed):
        """New sources and cleared results, on the current stream."""
        g = self.torch.Generator(device="cuda").manual_seed(seed)
        for s, d in zip(self.src, self.dst):
            v = s.view(self.torch.int16) if s.dtype == self.torch.uint16 else s
            if v.dtype == self.torch.float32:
                v.normal_(generator=g)
            else:
                v.random_(0, 200 if v.dtype == self.torch.uint8 else 30000, generator=g)
            d.view(self.torch.uint8).fill_(0xA5)

    def run(self):
        self.vkt.vktApplyFilterBatched(self.hd, self.hs, self.f, "mirror")

    def copies(self):
        return [d.view(self.torch.uint8).clone() for d in self.dst]

    def singles(self):
        for h, s, f in zip(self.hw, self.hs, self.f):
            self.vkt.vktApplyFilter(h, s, f, "mirror")
        return [w.view(self.torch.uint8).clone() for w in self.want]


def check(torch, got, want, what):
    print(what, flush=True)
    for i, (a, b) in enumerate(zip(got, want)):
        assert torch.equal(a, b), (what, i)


def order(torch, vkt):
    s = torch.cuda.Stream()
    b = Batch(torch, vkt)
    torch.cuda.synchronize()
    vkt.vktSetStream(s)
    with torch.cuda.stream(s):
        busy = torch.ones(1 << 26, device="cuda")
        got, want = [], []
        for rep in range(4):
            for _ in range(20):
                busy.mul_(1.0)  # (the sources are written some ms later)
            b.fill(rep)
            b.run()
            got.append(b.copies())
            want.append(b.singles())
    torch.cuda.synchronize()
    for rep in range(4):
        check(torch, got[rep], want[rep], f"call {rep}")


def capture(torch, vkt):
    s = torch.cuda.Stream()
    b = Batch(torch, vkt)
    others = [Batch(torch, vkt) for _ in range(17)]  # more than the cache holds
    torch.cuda.synchronize()
    vkt.vktSetStream(s)
    with torch.cuda.stream(s):
        b.fill(1)
        b.run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        b.run()
    for rep in range(6):
        with torch.cuda.stream(s):
            if rep == 3:
                for o in others:
                    vkt.vktApplyFilterBatched(o.hd[:1], o.hs[:1], o.f[:1], "mirror")
            b.fill(10 + rep)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            got, want = b.copies(), b.singles()
        torch.cuda.synchronize()
        check(torch, got, want, f"replay {rep}")


def depth(torch, vkt):
    b = Batch(torch, vkt, [((z, 513, 390), fmt, k) for z, fmt, k in
                           ((63, "uint16", 5), (64, "uint16", 5), (65, "uint16", 5),
                            (129, "uint16", 5), (1, "float32", 7), (64, "float32", 7),
                            (67, "float32", 7), (130, "float32", 7))])
    vkt.vktSetStream(torch.cuda.current_stream())
    b.fill(1)
    b.run()
    got, want = b.copies(), b.singles()
    torch.cuda.synchronize()
    check(torch, got, want, "depths")


if __name__ == "__main__":
    import torch as _torch
    from paper_2203_10213_amd import vkt as _vkt
    {"order": order, "capture": capture, "depth": depth}[sys.argv[1]](_torch, _vkt)
    print("all equal", flush=True)
