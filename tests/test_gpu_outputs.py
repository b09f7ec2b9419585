"""Every call that succeeds writes its outputs whole, padding bits included: the binding allocates them without clearing, so
the same call on outputs that held other values before gives the same bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scd():
    from paper_2410_01799_amd import scd as mod

    mod.lib()
    return mod


def gauss(shape, seed, dtype=np.float32):
    return torch.from_numpy(np.random.Generator(np.random.PCG64(seed)).standard_normal(shape).astype(dtype)).cuda()


def run_context(scd, shape, dtype, opts):
    with scd.ScdContext(gauss(shape, 1, dtype), 5, 3, options=opts) as ctx:
        ctx.run(2)
        ctx.step()
        return ctx.results(), ctx.remainder()


def expand(scd, shape, w, dtype):
    signs = [torch.stack([scd.scd_rng_signs(7, j, i, d) for j in range(w)]) for i, d in enumerate(shape)]
    return scd.scd_expand(signs, gauss(w, 2, dtype), shape)


def apply(scd, m, n, w, dtype, nvec, transpose):
    S = torch.stack([scd.scd_rng_signs(7, j, 0, m) for j in range(w)])
    T = torch.stack([scd.scd_rng_signs(7, j, 1, n) for j in range(w)])
    return scd.scd_apply(S, T, gauss(w, 2, dtype), m, n, gauss((nvec, m if transpose else n), 3, dtype), transpose)


STREAM = {"resident": 0, "sparse": 0, "persistent_stream": 0}
CASES = {}
for sh, dt in (((256, 256), np.float32), ((61, 67), np.float32), ((300, 520), np.float32), ((301, 257), np.float32), ((3, 5), np.float32),
               ((130, 101), np.float64), ((600, 401), np.float64), ((40, 30, 3), np.float32), ((9, 70, 5, 2), np.float32),
               ((130, 1, 3), np.float64), ((40, 3), np.float32), ((70, 5000), np.float32)):
    CASES[f"decompose-{sh}-{dt.__name__}"] = lambda s, sh=sh, dt=dt: s.scd_decompose(gauss(sh, 1, dt), 3, 5)
for name, o in (("sparse", {"resident": 0, "sparse_min_mib": 0}), ("persistent-stream", {"resident": 0, "sparse": 0}), ("stream", STREAM)):
    CASES[f"context-{name}"] = lambda s, o=o: run_context(s, (328, 264), np.float32, o)
CASES["context-odd-stream"] = lambda s: run_context(s, (97, 131), np.float64, STREAM)
for sh, dt in (((40, 30, 3), np.float32), ((90, 70, 3), np.float64), ((9, 70, 5, 2), np.float32), ((70, 33), np.float32)):
    CASES[f"scalars-{sh}-{dt.__name__}"] = lambda s, sh=sh, dt=dt: s.scd_decompose_scalars(gauss(sh, 1, dt), 3, 5)
for sh, dt, cuts in (((100, 76), np.float32, 0), ((300, 521), np.float64, 0), ((100, 76), np.float32, 1), ((65, 131), np.float64, 1), ((70, 4100), np.float32, 0)):
    CASES[f"lsq-{sh}-{dt.__name__}-{cuts}"] = lambda s, sh=sh, dt=dt, cuts=cuts: s.scd_lsq_decompose_form(gauss(sh, 1, dt), 3, 5, cuts=cuts)
CASES["lsq-matrix"] = lambda s: s.scd_lsq_decompose(gauss((100, 76), 1), 3, 5)
CASES["lsq-tensor"] = lambda s: s.scd_lsq_decompose(gauss((40, 30, 7), 1), 3, 5)
for sh, w, dt in (((70, 130), 7, np.float32), ((129, 65), 70, np.float32), ((129, 65), 460, np.float32),
                  ((129, 65), 70, np.float64), ((33, 10, 3), 60, np.float32), ((6, 5, 4, 3), 25, np.float64)):
    CASES[f"expand-{sh}-{w}-{dt.__name__}"] = lambda s, sh=sh, w=w, dt=dt: expand(s, sh, w, dt)
for dt in (np.float32, np.float64):
    for nvec in (1, 3, 5):
        for tr in (False, True):
            CASES[f"apply-{dt.__name__}-{nvec}-{tr}"] = lambda s, dt=dt, nvec=nvec, tr=tr: apply(s, 130, 77, 70, dt, nvec, tr)
    for m, n in ((100, 77), (130, 8200), (3, 5), (2049, 64), (300, 260)):
        CASES[f"row-{m}-{n}-{dt.__name__}"] = lambda s, m=m, n=n, dt=dt: s.scd_row_signed_sum(gauss((m, n), 1, dt), s.scd_rng_signs(1, 2, 1, n))
        CASES[f"col-{m}-{n}-{dt.__name__}"] = lambda s, m=m, n=n, dt=dt: s.scd_col_signed_sum(gauss((m, n), 1, dt), s.scd_rng_signs(1, 2, 0, m))
    CASES[f"pack-{dt.__name__}"] = lambda s, dt=dt: [s.scd_pack(gauss(n, 1, dt)) for n in (1, 63, 64, 65, 1000, 70001)]
CASES["unpack"] = lambda s: [s.scd_unpack(s.scd_rng_signs(1, 2, 0, n), n) for n in (1, 63, 64, 65, 1000)]


def tensors(x):
    if isinstance(x, torch.Tensor):
        return [x]
    if isinstance(x, dict):
        return [t for k in sorted(x) for t in tensors(x[k])]
    return [t for e in x for t in tensors(e)] if isinstance(x, (list, tuple)) else []


@pytest.mark.parametrize("name", CASES)
def test_outputs_are_written_whole(scd, monkeypatch, name):
    empty = torch.empty
    got = []
    for word in (-1, 0x2B5A17C93D5E6F01):                 # (all bits set: NaN in the real types)
        def held(*size, word=word, **kw):
            t = empty(*size, **kw)
            raw = t.view(torch.uint8).reshape(-1) if t.dim() else t.reshape(1).view(torch.uint8)
            pattern = torch.tensor([word], dtype=torch.int64).view(torch.uint8).to(t.device)
            raw.copy_(pattern.repeat((raw.numel() + 7) // 8)[: raw.numel()])
            return t

        with monkeypatch.context() as mp:
            mp.setattr(torch, "empty", held)
            got.append([t.cpu() for t in tensors(CASES[name](scd))])
    assert len(got[0]) == len(got[1]) > 0
    for a, b in zip(*got):
        assert a.numel() > 0 and torch.equal(a.reshape(-1).view(torch.uint8), b.reshape(-1).view(torch.uint8))
