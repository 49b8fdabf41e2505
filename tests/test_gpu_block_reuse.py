"""Device blocks that freed hierarchies leave for the next ones: the same
results in reused memory, from several threads and streams, and a bound on
what is kept."""

import threading

import numpy as np
import pytest

from gpu_helpers import setup, to_dev

pytestmark = pytest.mark.gpu


def solve_once(N, precision, stream=None):
    import torch

    from paper_2006_16147_amd import amg, inputs

    stream = stream or torch.cuda.current_stream()
    with torch.cuda.stream(stream):
        A = inputs.laplacian7(N)
        h = setup(A, precision=precision, stream=stream)
        b = to_dev(np.random.default_rng(N).uniform(-1, 1, A.n))
        x = torch.zeros_like(b)
        amg.amg_pcg_solve(h, b, x, rtol=1e-8)
        out = x.cpu().numpy()
        h.close()
    return out


def test_reused_blocks_give_the_same_solutions():
    first = {N: solve_once(N, 0) for N in (12, 33, 40)}
    for N in (40, 12, 33, 12, 40):
        np.testing.assert_array_equal(solve_once(N, 0), first[N])


def test_threads_and_streams_share_the_blocks():
    import torch

    want = {(N, p): solve_once(N, p) for N in (16, 24, 32) for p in (0, 1)}
    errors = []

    def work(i):
        try:
            torch.cuda.set_device(0)
            stream = torch.cuda.Stream()
            for r in range(6):
                key = sorted(want)[(i + r) % len(want)]
                np.testing.assert_array_equal(solve_once(*key, stream=stream), want[key])
        except BaseException as e:  # noqa: BLE001 - reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_what_is_kept_is_bounded():
    import torch

    from paper_2006_16147_amd import amg, inputs

    A = inputs.constant_diffusion7_arrays(144, 1.0, 1.0, 1.0, torch, "cuda:0")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    held = [amg.amg_setup(*A) for _ in range(8)]  # about 1.5 GB each, and the setups' own
    total = sum(h.footprint_bytes() for h in held)
    assert total > 9 << 30
    for h in held:
        h.close()
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] < (8 << 30) + (1 << 30)
