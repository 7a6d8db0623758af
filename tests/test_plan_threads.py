"""A plan answers several threads at once: the passes of an evolution depend on its
own step count only, whatever other threads ask the same plan."""
import threading

import paper_1208_2407_amd as tsq


def test_passes_from_several_threads():
    plan = tsq.Plan(256, 256, 0.05, "c64")
    counts = [1, 2, 7, 20, 100, 333]
    want = {n: plan.passes(n) for n in counts}
    wrong = []

    def ask(k):
        for i in range(4000):
            n = counts[(i * (k + 1) + k) % len(counts)]
            if plan.passes(n) != want[n]:
                wrong.append(n)

    threads = [threading.Thread(target=ask, args=(k,)) for k in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
