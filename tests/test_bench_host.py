"""bench.py's bookkeeping, on the CPU with a clock that settles while it measures."""
import types

import pytest

import bench


@pytest.mark.parametrize("slow", [2.0, 0.5])
def test_main_kernels_are_part_of_their_calls_while_the_clock_settles(slow, monkeypatch):
    """A step's durations drift from `slow` times the final ones to those over the first two hundred steps; a main kernel takes 0.97 of
    its call at any time, and so it does in the figures, whichever way the clock drifts."""
    state = {"step": 0, "mask": set(), "ms": {}}

    def step(S, st):
        scale = 1.0 + (slow - 1.0) * max(0.0, 1.0 - state["step"] / 200)
        state["step"] += 1
        for c, ms in ((0, 0.97), (1, 2.91), (2, 1.0), (3, 3.0)):
            if c in state["mask"]:
                state["ms"].setdefault(c, []).append(ms * scale)

    def enable(on, channels=None):
        state["mask"] = set(channels if channels is not None else range(4)) if on else set()
        state["ms"] = {}

    def read(backward, whole_call=False):
        ms = state["ms"].get(int(backward) + 2 * int(whole_call), [])
        return len(ms), sum(ms)

    monkeypatch.setattr(bench, "step", step)
    S = types.SimpleNamespace(sig_profile_enable=enable, sig_profile_read=read)
    torch = types.SimpleNamespace(cuda=types.SimpleNamespace(synchronize=lambda: None))
    _, kf, kb, cf, cb, (which, timed) = bench.time_steps(S, torch, None, 20, 5)
    assert which == 1 and timed == pytest.approx(2.91 * (1 + (slow - 1) * (1 - 14.5 / 200)))
    assert kf / cf == pytest.approx(0.97) and kb / cb == pytest.approx(0.97)
