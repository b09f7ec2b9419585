"""Blocks that a context or a call returns serve the next one: nothing of the last owner shows, the kept memory is
bounded, and threads on streams of their own do not disturb each other."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scd():
    from paper_2410_01799_amd import scd as mod

    mod.lib()
    return mod


def gauss(shape, seed, dtype=torch.float32):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float64).to(dtype)


CALLS = [
    lambda s, k: s.scd_decompose(gauss((256, 256), k), 6, k)["c"],
    lambda s, k: s.scd_decompose(gauss((301, 257), k, torch.float64), 6, k)["c"],
    lambda s, k: s.scd_decompose(gauss((40, 30, 7), k), 4, k)["c"],
    lambda s, k: s.scd_decompose_scalars(gauss((40, 30, 3), k), 4, k)["c"],
    lambda s, k: s.scd_lsq_decompose(gauss((96, 130), k), 5, k)["c"],
    lambda s, k: s.scd_col_signed_sum(gauss((300, 200), k), s.scd_rng_signs(k, 0, 0, 300))[0],
    lambda s, k: s.scd_decompose(gauss((2048, 1024), k), 4, k, options={"resident": 0, "sparse_min_mib": 0})["c"],
]


def test_reused_blocks_do_not_show(scd):
    first = [[f(scd, k).clone() for k in (1, 2)] for f in CALLS]
    for f, ref in zip(CALLS, first):   # every block now comes from another owner, with other contents
        for k in (2, 1):
            assert torch.equal(f(scd, k), ref[k - 1])


def test_kept_memory_is_bounded(scd):
    A = gauss((4096, 4096), 3)
    scd.scd_decompose(A, 1, 1, options={"resident": 0, "sparse_min_mib": 0})
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for i in range(12):                # a new shape each time: 100 MB and more a context
        scd.scd_decompose(gauss((3000 + 64 * i, 4096), i), 1, 1, options={"resident": 0, "sparse_min_mib": 0})
    torch.cuda.empty_cache()
    assert free0 - torch.cuda.mem_get_info()[0] <= (1 << 30) + (64 << 20)


def test_threads_with_streams_of_their_own(scd):
    ref = [[f(scd, k).clone() for k in (1, 2)] for f in CALLS]
    bad = []

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for r in range(3):
                j = (i + r) % len(CALLS)
                k = 1 + (i + r) % 2
                if not torch.equal(CALLS[j](scd, k), ref[j][k - 1]):
                    bad.append((i, j, k))
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
