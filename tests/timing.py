"""Device time of calls, for tests that compare calls on one GPU."""
import torch


def least_us(calls, passes=40, rounds=7):
    """For each call the least mean time of `passes` in a row over the rounds, in us; the
    calls take turns, so that the clock and the host treat them alike."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    least = [float("inf")] * len(calls)
    for call in calls:
        for _ in range(5):
            call()
    for _ in range(rounds):
        for i, call in enumerate(calls):
            a.record()
            for _ in range(passes):
                call()
            b.record()
            torch.cuda.synchronize()
            least[i] = min(least[i], a.elapsed_time(b) / passes * 1e3)
    return least
