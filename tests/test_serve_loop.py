"""The request loop's order of work, without a GPU: problems and launches are stand-ins, time is the
test's own."""
import numpy as np
import pytest

import meshgen


class Clock:
    def __init__(self):
        self.t = 0.0

    def perf_counter(self):
        self.t += 1e-6
        return self.t

    def sleep(self, s):
        self.t += max(s, 1e-6)


def run(monkeypatch, arrivals, launch_s=1.5e-3, admit_s=2e-4):
    """Serves requests that arrive at these times; the launches as (time, how many) and the
    statistics."""
    import torch

    import paper_2407_20026_amd as sso
    from paper_2407_20026_amd import serve
    clock, launches = Clock(), []

    class Stand:
        """A begun problem, or the batch that launches some."""

        def __init__(self, *args, **kw):
            pass

        def solve_begin(self):
            clock.t += admit_s

        def solve_ready(self):
            return True

        def launch(self, problems, n_iter):
            launches.append((clock.t - start, len(problems)))

        def wait(self, problems):
            clock.t += launch_s
            return [True] * len(problems)

        def set_stream(self, stream):
            pass

        def close(self):
            pass

    monkeypatch.setattr(sso, "Batch", Stand)
    monkeypatch.setattr(serve, "Problem", Stand)
    monkeypatch.setattr(serve, "time", clock)
    monkeypatch.setattr(serve, "streams_overlap", lambda a, b: True)
    monkeypatch.setattr(serve, "finish_one", lambda p, req: (0.0, None, None, 0, 0, 0.0, 0, 0.0))
    monkeypatch.setattr(torch.cuda, "Stream", lambda device=None: object())
    mesh = meshgen.gridshell(4)
    start = clock.t
    stats = serve.BatchedServer().run([serve.Request(i, mesh, float(t))
                                       for i, t in enumerate(arrivals)])
    assert stats.n == len(arrivals)
    return launches, stats


def streams():
    rng = np.random.default_rng(1)
    out = [0.002 * np.arange(9), 0.0007 * np.arange(12), np.zeros(5), 0.004 * np.arange(6)]
    out += [np.cumsum(rng.exponential(1.0 / r, 30)) for r in (200.0, 500.0, 1000.0)]
    pairs = 0.02 * (np.arange(8) // 2) + 0.001 * (np.arange(8) % 2)
    return out + [pairs]


@pytest.mark.parametrize("k", range(8))
def test_the_loop_knows_nothing_of_requests_to_come(monkeypatch, k):
    """What is launched before a request arrives is launched at the same times, and in the same
    company, whether that request comes or not."""
    arrivals = streams()[k]
    whole, _ = run(monkeypatch, arrivals)
    for n in range(1, len(arrivals)):
        if arrivals[n] > arrivals[n - 1]:
            part, _ = run(monkeypatch, arrivals[:n])
            early = [x for x in part if x[0] < arrivals[n]]
            assert early == [x for x in whole if x[0] < arrivals[n]][:len(early)]
            assert len(early) == len([x for x in whole if x[0] < arrivals[n]])


def test_only_requests_at_a_steady_interval_are_held(monkeypatch):
    """Pairs, and requests further apart than a launch takes, are launched as they come; at a steady
    interval they gather, and the last are not held longer than a quarter of it past the next."""
    _, stats = run(monkeypatch, streams()[7])
    assert all(r.latency < 4e-3 for r in stats.results)
    launches, stats = run(monkeypatch, 0.004 * np.arange(6))
    assert [n for _, n in launches] == [1] * 6
    launches, stats = run(monkeypatch, 0.002 * np.arange(9))
    assert max(n for _, n in launches) == 4 and stats.peak_inflight >= 4
    assert launches[-1][0] <= 0.016 + 1.25 * 0.002 + 5e-4
