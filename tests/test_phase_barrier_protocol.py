"""CPU model of the batches' barrier between phases: a count that only grows
and a published number of completed barriers.  Random interleavings of the
work-groups' steps, with polls that may return any older value per-location
coherence still allows, over several launches that share the words.  A model
of the steps, not of the kernel: it pins the protocol the kernel implements."""
import random

import pytest


class Words:
    def __init__(self):
        self.count = 0
        self.gen = [0]     # every value the published word has held, in store order


def run_launch(words, units, barriers, rng, timeouts=0.0):
    """One launch of `units` work-groups over `barriers` barriers.  A poll that
    does not hold gives up with probability `timeouts` (the spin limit) and
    the work-group goes on.  Returns the number of waits that gave up."""
    start = len(words.gen) - 1       # a launch sees everything stored before it
    wgs = [dict(b=0, g=None, seen=start, step="arrive") for _ in range(units)]
    arrived = [0] * barriers
    gave_up = steps = 0
    while any(w["b"] < barriers for w in wgs):
        steps += 1
        assert steps < 60_000, "no progress"
        w = rng.choice([x for x in wgs if x["b"] < barriers])
        if w["step"] == "arrive":
            old = words.count
            words.count += 1
            arrived[w["b"]] += 1
            if w["g"] is None:
                w["g"] = old // units
            w["g"] += 1
            w["step"] = "publish" if old + 1 == w["g"] * units else "wait"
        elif w["step"] == "publish":
            words.gen.append(w["g"])
            w["seen"] = len(words.gen) - 1
            w["b"], w["step"] = w["b"] + 1, "arrive"
            if not timeouts:
                assert arrived[w["b"] - 1] == units
        else:
            w["seen"] = rng.randint(w["seen"], len(words.gen) - 1)
            held = words.gen[w["seen"]] >= w["g"]
            if held and not timeouts:
                assert arrived[w["b"]] == units, "left before every arrival"
            late = not held and rng.random() < timeouts
            if held or late:
                gave_up += late
                w["b"], w["step"] = w["b"] + 1, "arrive"
    return gave_up


@pytest.mark.parametrize("seed", range(40))
def test_phases_hold_over_launches_that_share_the_words(seed):
    rng = random.Random(seed)
    units = rng.choice([1, 2, 3, 5, 8])
    words, total = Words(), 0
    for _ in range(4):
        barriers = rng.randint(1, 9)
        assert run_launch(words, units, barriers, rng) == 0
        total += barriers
        assert words.count == total * units and words.gen[-1] == total


@pytest.mark.parametrize("cleared", [False, True])
@pytest.mark.parametrize("seed", range(40))
def test_a_launch_with_timeouts_ends_and_leaves_usable_words(seed, cleared):
    """Work-groups that give up waiting still arrive at every later barrier, so
    the launch ends with a whole number of barriers in the count, and the next
    launch's barriers hold, whether or not the host cleared the words between."""
    rng = random.Random(500 + seed)
    units, barriers = rng.choice([2, 3, 5, 8]), rng.randint(1, 8)
    words = Words()
    run_launch(words, units, 2, rng)
    run_launch(words, units, barriers, rng, timeouts=0.3)
    assert words.count == (2 + barriers) * units and max(words.gen) <= 2 + barriers
    if cleared:
        words = Words()
    for _ in range(2):
        assert run_launch(words, units, rng.randint(1, 8), rng) == 0


def test_the_model_sees_a_wrong_number_of_work_groups():
    """Launches of different sizes on one set of words must fail in the model
    (the kernel's caller fixes the size for the words' life)."""
    failed = 0
    for seed in range(20):
        rng, words = random.Random(900 + seed), Words()
        run_launch(words, 3, 1, rng)
        try:
            run_launch(words, 4, 3, rng, timeouts=0.0)
        except AssertionError:
            failed += 1
    assert failed == 20
