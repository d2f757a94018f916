"""Device time of a call, for tests that compare two calls on one GPU."""
import torch


def median_us(call, passes=40, rounds=5):
    """Median over rounds of the mean time of `passes` calls in a row, in us."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(5):
        call()
    times = []
    for _ in range(rounds):
        a.record()
        for _ in range(passes):
            call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) / passes * 1e3)
    return sorted(times)[rounds // 2]
