"""How many threads an encode starts: as many as its work is worth, up to the
caller's count.  A few large or noisy bricks take as many as there are bricks,
small smooth ones none."""
import os
import threading

import numpy as np
import pytest


@pytest.fixture(scope="module")
def P():
    import paper_2609_36898_amd  # (not at collection: GPU tests import torch first)
    return paper_2609_36898_amd


def _most_threads(fn):
    """Largest number of threads besides those that were there while fn runs."""
    base, most, stop = None, 0, threading.Event()
    ready = threading.Event()

    def watch():
        nonlocal base, most
        base = len(os.listdir("/proc/self/task"))
        ready.set()
        while not stop.is_set():
            most = max(most, len(os.listdir("/proc/self/task")) - base)

    t = threading.Thread(target=watch)
    t.start()
    ready.wait()
    fn()
    stop.set()
    t.join()
    return most


def _encode(P, v, l2, n_threads, streamed):
    n = len(v)
    if not streamed:
        return P.csgv_encode_bricks(v.reshape(-1), [l2] * n, 8, origins=np.zeros((n, 3), np.uint32), n_threads=n_threads)
    e = P.csgv.csgv_encoder(8, n_threads=n_threads)
    e.add(v.reshape(-1), [l2] * n)
    return e.finish()


@pytest.mark.parametrize("streamed", [False, True])
@pytest.mark.parametrize("side,n", [(64, 2), (64, 4), (32, 8)])
def test_few_hard_bricks_use_the_threads_asked_for(P, side, n, streamed):
    rng = np.random.default_rng(side + n)
    v = rng.integers(1, 1 << 60, (n, side ** 3)).astype(np.uint64)
    l2 = side.bit_length() - 1
    assert max(_most_threads(lambda: _encode(P, v, l2, 4, streamed)) for _ in range(3)) == min(n, 4) - 1
    assert _most_threads(lambda: _encode(P, v, l2, 1, streamed)) == 0
    assert _encode(P, v, l2, 4, streamed) == _encode(P, v, l2, 1, streamed)


def test_little_work_starts_no_thread(P):
    v = np.broadcast_to((np.arange(16) // 5).astype(np.uint64), (4, 16, 16, 16)).reshape(4, -1)
    assert max(_most_threads(lambda: [_encode(P, v, 4, 8, False) for _ in range(200)]) for _ in range(3)) == 0


def test_record_buffer_follows_the_lanes():
    # one 64^3 brick of few labels at random, half a million symbols and more: encoded with one lane it
    # takes no more memory than with 256 (a buffer of 64 lanes' room would take 64 bytes a symbol more)
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = ("import numpy as np, resource, paper_2609_36898_amd as P\n"
            "v = np.random.default_rng(0).integers(1, 17, 64 ** 3).astype(np.uint32)\n"
            "go = lambda s: P.csgv_encode_bricks(v, [6], 4, coder_policy=2, lane_syms=s, n_threads=1)\n"
            "go(64)\n"
            "a = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss\n"
            "go(1 << 20)\n"
            "print(resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - a)")
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, check=True)
    assert int(r.stdout.split()[-1]) < 8192, "KiB more"
