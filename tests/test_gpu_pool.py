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


def device_free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()           # (what torch keeps would hide what the library keeps)
    return torch.cuda.mem_get_info()[0]


def test_kept_memory_is_bounded_and_given_back(scd):
    opts = {"resident": 0, "sparse_min_mib": 0}
    scd.scd_decompose(gauss((512, 512), 3), 1, 1, options=opts)
    scd.scd_release_memory()
    free0 = device_free()
    for i in range(40):                # a new shape each time, 100 MB and more a context: 5 GB in all
        scd.scd_decompose(torch.full((3000 + 64 * i, 4096), 1.0 + i, device="cuda"), 1, 1, options=opts)
    kept = free0 - device_free()
    assert 0 < kept <= (1 << 30) + (64 << 20)
    released = scd.scd_release_memory()
    assert kept - (64 << 20) <= released <= 1 << 30
    assert free0 - device_free() <= 16 << 20
    assert scd.scd_release_memory() == 0
    # blocks in use are not touched
    with scd.ScdContext(gauss((301, 257), 4), 6, 4) as ctx:
        ctx.run(2)
        scd.scd_release_memory()
        ctx.run(4)
        c = ctx.results()["c"]
    assert torch.equal(c, scd.scd_decompose(gauss((301, 257), 4), 6, 4)["c"])


def test_threads_with_streams_of_their_own(scd):
    ref = [[f(scd, k).clone() for k in (1, 2)] for f in CALLS]
    bad = []

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for r in range(3):
                if i == 5:
                    scd.scd_release_memory()   # (waits for the others and takes what they have returned)
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


AFTER_RESET = """
import ctypes as C, sys
hip, scd = C.CDLL("libamdhip64.so"), C.CDLL(sys.argv[1])
def malloc(n):
    p = C.c_void_p()
    assert hip.hipMalloc(C.byref(p), C.c_size_t(n)) == 0
    return p
def known(p):
    v = C.c_uint64()
    return hip.hipPointerGetAttribute(C.byref(v), 7, p) == 0     # HIP_POINTER_ATTRIBUTE_BUFFER_ID
m, n = 640, 512
A, S, T, c, tr = malloc(4 * m * n), malloc(8 * 10), malloc(8 * 8), malloc(4), malloc(16)
assert hip.hipMemset(A, 0, C.c_size_t(4 * m * n)) == 0
scd.scd_release_memory.restype = C.c_size_t
scd.scd_decompose.argtypes = [C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_int64, C.c_uint64, C.c_void_p, C.c_void_p] + 3 * [C.c_void_p]
dims, signs = (C.c_int64 * 2)(m, n), (C.c_void_p * 2)(S.value, T.value)
assert scd.scd_decompose(A, 0, 2, dims, 1, 3, None, signs, c, tr, None) == 0
assert hip.hipDeviceSynchronize() == 0 and known(A)
assert hip.hipDeviceReset() == 0 and not known(A)
mine = [malloc(k) for k in (4 * m * n, 4 * m * n, 1 << 20, 4096, 4096, 80, 64, 16, 8, 8, 4)]
assert scd.scd_release_memory() == 0
assert all(known(p) for p in mine)
print("whole")
"""


def test_blocks_of_before_a_device_reset_are_forgotten(scd, tmp_path):
    # the addresses belong to the program's own allocations now; no kernel runs after the reset
    import subprocess
    import sys

    prog = tmp_path / "after_reset.py"
    prog.write_text(AFTER_RESET)
    run = subprocess.run([sys.executable, str(prog), str(scd.LIB_PATH)], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0 and run.stdout.strip() == "whole", run.stderr[-2000:]
