"""GPU: the pinned result blocks, shared out of slabs of 64 over the process's
contexts: more contexts than a slab holds, destroyed in any order and from
several threads, never share one, and results do not depend on which block a
context got."""
import random
import threading

import pytest

from pairs import gpu_for

pytestmark = pytest.mark.gpu

KW = dict(dtype="fp64", n=0.8, Da=1e-2, Ra=1e5, Pr=10.0, eps=0.6)


@pytest.mark.parametrize("count", [63, 64, 65, 150])
def test_contexts_over_several_slabs(count):
    sides = (20, 33, 47)
    ref = [gpu_for(n, n, **KW).step(6).nu() for n in sides]
    rng = random.Random(count)
    cs = [gpu_for(sides[i % 3], **KW).step(6) for i in range(count)]
    live = dict(enumerate(cs))
    del cs
    for i in rng.sample(sorted(live), count // 2):
        live.pop(i).close()
    for i in range(count, count + 20):
        live[i] = gpu_for(sides[i % 3], **KW).step(6)
    assert [live[i].nu() for i in live] == [ref[i % 3] for i in live]
    for i in rng.sample(sorted(live), len(live)):
        live.pop(i).close()


def test_threads_create_use_and_destroy():
    ref = gpu_for(24, **KW).step(4).nu()
    bad = []

    def work(seed):
        rng, held = random.Random(seed), []
        for _ in range(40):
            held.append(gpu_for(24, **KW).step(4))
            if held[rng.randrange(len(held))].nu() != ref:
                bad.append(seed)
            if rng.random() < 0.4:
                held.pop(rng.randrange(len(held))).close()
        for c in held:
            c.close()

    ts = [threading.Thread(target=work, args=(s,)) for s in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
