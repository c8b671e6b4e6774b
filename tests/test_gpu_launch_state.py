"""What a launch of the persistent kernel finds and leaves in the dependency counters.

Calls on one handle (or on the static array) must not overlap.  Where they did all the same, the counters may
hold anything; the next step must be right again, and a step that was not run must not be reported
as done.  The tests write such leftovers from the host, into counters that nobody is using.
"""
import numpy as np
import pytest
import torch

import paper_2604_15379_amd as F
import synth_inputs as si
from gpu_common import Model

pytestmark = pytest.mark.gpu

# words of a counter set: abort word, workers of an XCD, start-up words, first event counter
ABORT, ROSTER, READY, EVENTS = 32, 64, 320, 832
LEFTOVERS = [(ABORT, 1), (ABORT + 1, 0xFFFFFFFC), (ROSTER, 3), (ROSTER + 32 * 7, 40), (READY, 7), (READY + 32 * 15, 300),
             (EVENTS, 5), (EVENTS + 1, 1), (EVENTS + 9, 77)]


class _Steps:
    """One model and handle; ``run`` makes a step through an entry point and returns its status code and output."""

    def __init__(self, batch, entry):
        sh = si.reduced_shape(max_batch=batch, max_seq=96, n_layers=2, vocab=512)
        self.m = Model(sh, seed=5, batch=batch, positions=np.random.default_rng(batch).integers(0, 96, batch).astype(np.int32))
        self.f = F.fleet_create(sh.asdict(), self.m.w, 0, 0, 0)
        self.static = entry == "static"
        self.call = F.fleet_decode_step_static if self.static else F.fleet_decode_step
        self.hout = torch.empty((batch, sh.hidden), device="cuda")
        self.logits = torch.empty((batch, sh.vocab), device="cuda")
        self.kc, self.vc = self.m.kc.clone(), self.m.vc.clone()   # (a step writes the same entries every time)

    def launch(self, stream):
        self.call(self.f, self.m.batch, self.m.hidden, None, self.kc, self.vc, self.m.pos, self.hout, self.logits, stream.cuda_stream)

    def clear(self):
        self.hout.fill_(float("nan"))
        self.logits.fill_(float("nan"))
        torch.cuda.synchronize()

    def run(self, stream):
        self.clear()
        self.launch(stream)
        code = F.fleet_last_status(self.f)["code"]
        return code, self.hout.clone(), self.logits.clone()

    def leave(self, sets=(0, 1)):
        for s in sets:
            for word, value in LEFTOVERS:
                F.fleet_test_counter(self.f, self.static, s, word, value)


@pytest.fixture(params=[(1, "step"), (3, "step"), (20, "step"), (3, "static")], ids=lambda p: f"b{p[0]}-{p[1]}")
def steps(request):
    s = _Steps(*request.param)
    yield s
    F.fleet_destroy(s.f)


def _same(got, ref):
    assert got[0] == 0 and torch.equal(got[1], ref[1]) and torch.equal(got[2], ref[2])


def test_leftover_counters_are_reported_and_cleaned_by_the_status_call(steps):
    """A handle that has been used on the default stream only (the static array: unless another test came first)."""
    default = torch.cuda.default_stream()
    ref = steps.run(default)
    assert ref[0] == 0 and torch.isfinite(ref[1]).all()
    print("leftovers in the counters of the next step", flush=True)
    steps.leave(sets=(0,))
    for _ in range(2):       # reported, and again
        assert F.fleet_last_status(steps.f)["code"] != 0
    for _ in range(3):
        _same(steps.run(default), ref)


def test_a_step_on_another_stream_is_right_after_any_leftovers(steps):
    """From the first call on another stream on, every call clears the counters in front, also on the default stream."""
    default, side = torch.cuda.default_stream(), torch.cuda.Stream()
    ref = steps.run(default)
    assert ref[0] == 0 and torch.isfinite(ref[1]).all()
    for stream in (side, side, default, default):
        print(f"leftovers, then a step on {'the default stream' if stream == default else 'a side stream'}", flush=True)
        steps.leave()
        _same(steps.run(stream), ref)
        _same(steps.run(stream), ref)


def test_replays_of_a_captured_step_are_right_after_any_leftovers(steps):
    side = torch.cuda.Stream()
    ref = steps.run(side)
    assert ref[0] == 0 and torch.isfinite(ref[1]).all()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        steps.launch(torch.cuda.current_stream())
    for replay in range(4):
        print(f"replay {replay}", flush=True)
        if replay % 2:
            steps.leave()
        steps.clear()
        g.replay()
        code = F.fleet_last_status(steps.f)["code"]
        _same((code, steps.hout, steps.logits), ref)
        _same(steps.run(torch.cuda.default_stream()), ref)      # eager steps in between


@pytest.mark.parametrize("expect", [[33, 31] + [32] * 6, [0, 64] + [32] * 6, [256] + [0] * 7, [1, 63, 16, 48, 30, 34, 32, 32]],
                         ids=lambda e: "-".join(map(str, e)))
def test_steps_do_not_depend_on_the_expected_workers(steps, expect):
    """Start-up is told how many workers to expect on each XCD; where that is wrong it adds up the rosters instead."""
    default = torch.cuda.default_stream()
    ref = steps.run(default)
    status = F.fleet_last_status(steps.f)
    if status["workers"] != [32] * 8:
        pytest.skip(f"the numbers are for 32 workers on each of eight XCDs, not {status['workers']}")
    print(f"expected workers {expect}", flush=True)
    F.fleet_test_expect_workers(steps.f, expect)
    for _ in range(3):
        _same(steps.run(default), ref)
        assert F.fleet_last_status(steps.f)["workers"] == status["workers"]
    for bad in ([32] * 7 + [31], [-1, 65] + [32] * 6):
        with pytest.raises(F.FleetError):
            F.fleet_test_expect_workers(steps.f, bad)
