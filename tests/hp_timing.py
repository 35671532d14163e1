"""Times of GPU work for the tests that compare two ways to do the same."""
from __future__ import annotations


def times_in_turn(runs, reps=16, inner=4):
    """The shortest time (us) of each of `runs` over `reps` rounds, all of them
    timed in turn in every round (a change of clocks or a neighbour's load meets
    them alike), `inner` calls at a time."""
    import torch
    best = [float("inf")] * len(runs)
    for run in runs:
        run()
    for _ in range(reps):
        for i, run in enumerate(runs):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(inner):
                run()
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 1e3 / inner)
    return best
