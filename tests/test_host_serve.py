"""The render server's open loop on the CPU: launches and the GPU replaced by
stubs, time by a clock that moves 5 us per reading."""
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")

from paper_2405_13943_amd import serve  # noqa: E402

CAM = SimpleNamespace(width=64, height=48)


class Clock:
    """perf_counter moves 5 us a reading, so that a loop that only waits ends."""

    def __init__(self):
        self.t = 0.0

    def perf_counter(self):
        self.t += 5e-6
        return self.t

    def sleep(self, s):
        self.t += s


class Server(serve.RenderServer):
    def __init__(self, clock, n_slots, max_batch, service):
        self.clock, self.service = clock, service
        arena = SimpleNamespace(max_pixels=1 << 30, capacity=1 << 30, counters_host=torch.zeros(4, dtype=torch.int32))
        self.slots = [SimpleNamespace(arena=arena, event=None, batch=None) for _ in range(n_slots)]
        self.max_batch, self.pairs_per_px = max_batch, 1.0
        self.queue, self.finished, self.pool = [], [], {}
        self.retries = self.largest_batch = self.most_in_flight = 0
        self.launches = []          # (time, batch size, requests waiting)

    def _launch(self, slot, batch, now):
        self.launches.append((self.clock.t, len(batch), len(self.queue) + len(batch)))
        end = self.clock.t + self.service
        slot.batch, slot.event = batch, SimpleNamespace(query=lambda: self.clock.t >= end)
        for r in batch:
            r.started = now


def serve_all(monkeypatch, arrivals, n_slots=3, max_batch=16, service=1e-3):
    clock = Clock()
    monkeypatch.setattr(serve, "time", clock)
    srv = Server(clock, n_slots, max_batch, service)
    stats, reqs = srv.run_open_loop([CAM] * len(arrivals), arrivals)
    assert stats["requests"] == len(arrivals) and all(r.done is not None for r in reqs)
    return srv, reqs


@pytest.mark.parametrize("gap", [50e-6, 20e-6, 1e-6])
def test_launches_are_not_held_by_a_run_of_arrivals(monkeypatch, gap):
    """Arrivals closer together than the gather window, for many windows: the
    first launch comes one window after the first arrival (and one step of the
    loop, which here costs below 200 us), not after the last."""
    arrivals = [1e-3 + gap * k for k in range(2000)]
    srv, _ = serve_all(monkeypatch, arrivals)
    assert srv.launches[0][0] <= 1e-3 + srv.GATHER + 200e-6
    assert srv.launches[0][0] < arrivals[-1]


def test_a_full_batch_is_not_held(monkeypatch):
    """With room for four requests in a batch and arrivals 10 us apart, every
    launch that finds a free slot takes a batch as soon as four wait."""
    srv, _ = serve_all(monkeypatch, [1e-3 + 10e-6 * k for k in range(400)], n_slots=200, max_batch=4)
    assert max(q for _, _, q in srv.launches) <= 8


def test_images_are_retired_while_a_launch_is_held(monkeypatch):
    """A batch that ends while the next is gathered is stamped done then, not
    after the window."""
    arrivals = [1e-3, 2e-3, 2e-3 + 90e-6]
    srv, reqs = serve_all(monkeypatch, arrivals, service=1.03e-3)
    first_end = srv.launches[0][0] + 1.03e-3
    assert arrivals[1] < first_end < arrivals[2]          # the case the test is about
    assert reqs[0].done <= first_end + 40e-6
    assert [n for _, n, _ in srv.launches] == [1, 2]      # and the two arrivals shared a launch


def test_a_lone_arrival_is_launched_at_once(monkeypatch):
    srv, reqs = serve_all(monkeypatch, [1e-3, 5e-3])
    assert [n for _, n, _ in srv.launches] == [1, 1]
    assert all(r.started - a <= 60e-6 for r, a in zip(reqs, (1e-3, 5e-3)))
