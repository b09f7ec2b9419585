"""The calls whose speed is tracked: what users of this library have it do, through its public entry points.

The cases follow the workloads of bench.py and of the tests (the 256x256 and 4096x4096 Gaussian matrices, the
matrices of a Mistral-7B-shaped decoder layer, the image-like tensor, the least squares refit, products with and
expansion of packed factors) with widths cut so that a pass takes milliseconds; `draw` spreads the same kinds of
calls over odd and ragged sizes, both data types, both directions and all variants.

What a run returns.  The greedy loop decides signs: an f32 sum that differs in its last bits can take a near tie
the other way (measured: about one term in a hundred at 4096x4096), and every later term of the run then lands in
another local maximum of the same quality.  Runs on f64 inputs have no such ties and return everything (signs,
coefficients, norms, alternations).  Runs on f32 inputs return the numbers that describe the approximation (the
coefficients and the norm after every term).  The signs that f32 sums decide are returned by the half-step case.
"""
import math

import torch

from paper_2410_01799_amd import scd

DEV = "cuda"


# --------------------------------------------------------------------------- cases


def listed():
    return [
        # a small matrix to full width: launches and exchange latency are all there is (256x256, width 64)
        dict(name="decompose_256_f32", kind="matrix", law="gauss", m=256, n=256, dtype="f32", w=64, share=0),
        # the headline matrix, the first terms of its run
        dict(name="decompose_4096_f32", kind="matrix", law="gauss", m=4096, n=4096, dtype="f32", w=64, share=0),
        # its f64 copy
        dict(name="decompose_4096_f64", kind="matrix", law="gauss", m=4096, n=4096, dtype="f64", w=32, share=0),
        # the largest matrix of a decoder layer (gate and up projection)
        dict(name="decompose_14336x4096_f32", kind="matrix", law="weights", m=14336, n=4096, dtype="f32", w=24, share=0),
        # a matrix of a decoder layer on its share of the device, as the model run drives it
        dict(name="share32_1024x4096_f32", kind="matrix", law="weights", m=1024, n=4096, dtype="f32", w=64, share=32),
        # rows of an odd length: nothing is aligned, nothing fills a tile
        dict(name="decompose_1501x999_f32", kind="matrix", law="gauss", m=1501, n=999, dtype="f32", w=16, share=0),
        # the image-like tensor, sign vectors in all modes
        dict(name="image_4000x3000x3_f32", kind="image", m=4000, n=3000, q=3, dtype="f32", w=24, scalars=0),
        # all coefficients refitted after every term
        dict(name="lsq_1024_f32", kind="lsq", m=1024, n=1024, q=0, dtype="f32", w=32),
        # one decode step with a packed 4096x4096 projection at half its bf16 size, and the transposed product of
        # the largest one with a few vectors
        dict(name="apply_4096_f32", kind="apply", m=4096, n=4096, w=16320, nvec=1, transpose=0, dtype="f32"),
        dict(name="apply_t_14336x4096_f32", kind="apply", m=14336, n=4096, w=25442, nvec=4, transpose=1, dtype="f32"),
        # a packed key projection back to a dense matrix when a model is loaded
        dict(name="expand_1024x4096_f32", kind="expand", m=1024, n=4096, q=0, w=6512, dtype="f32"),
        # one alternation driven by the caller: start vector, row half step, column half step
        dict(name="halfsteps_4096_f32", kind="halfsteps", m=4096, n=4096, dtype="f32"),
    ]


def _size(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    # half of the sizes as they come (odd ones among them), half rounded to what layouts like
    return max(lo, n if rng.random() < 0.5 else n // 64 * 64) if n >= 128 else n


def draw(rng):
    kind = rng.choice(["matrix", "matrix", "matrix", "image", "tensor", "lsq", "apply", "apply", "expand", "halfsteps"])
    dtype = rng.choice(["f32", "f32", "f64"])
    if kind == "matrix":
        m, n = _size(rng, 64, 14336), _size(rng, 64, 8192)
        if min(m, n) <= 256:  # a small matrix is small both ways
            m, n = min(m, 512), min(n, 512)
        share = rng.choice([0, 0, 0, 32, 64])
        case = dict(kind=kind, law=rng.choice(["gauss", "weights"]), m=m, n=n, dtype=dtype, share=share)
        cap = 2.0e8 if dtype == "f32" else 1.0e8  # entries times terms
        case["w"] = max(4, min(rng.randint(8, 96), int(cap / (m * n))))
        return case
    if kind == "image":
        m, n = _size(rng, 200, 4000), _size(rng, 200, 3000)
        return dict(kind=kind, m=m, n=n, q=rng.choice([1, 3, 3, 4]), dtype="f32", w=rng.randint(8, 32), scalars=rng.choice([0, 1]))
    if kind == "tensor":
        # several modes of middling length (a stack of frames, a convolution kernel)
        m, n = _size(rng, 16, 400), _size(rng, 16, 300)
        return dict(kind="image", m=m, n=n, q=rng.randint(5, 40), dtype=dtype, w=rng.randint(4, 12), scalars=rng.choice([0, 0, 1]))
    if kind == "lsq":
        return dict(kind=kind, m=_size(rng, 64, 2048), n=_size(rng, 64, 2048), q=rng.choice([0, 0, 3]) if rng.random() < 0.5 else 0,
                    dtype=dtype, w=rng.randint(8, 40))
    if kind == "apply":
        m, n = _size(rng, 256, 14336), _size(rng, 256, 8192)
        w = max(64, int(8 * m * n / (m + n + 32) * rng.choice([0.5, 0.75, 1.0])))
        return dict(kind=kind, m=m, n=n, w=w, nvec=rng.choice([1, 1, 2, 4, 8]), transpose=rng.choice([0, 1]), dtype=dtype)
    if kind == "expand":
        m, n = _size(rng, 64, 4096), _size(rng, 64, 4096)
        q = rng.choice([0, 0, 3])
        cap = 2.5e10 / (m * n * max(1, q))  # entries times terms
        return dict(kind=kind, m=m, n=n, q=q, w=max(8, min(int(8 * m * n / (m + n + 32)), int(cap))), dtype=dtype)
    return dict(kind=kind, m=_size(rng, 64, 14336), n=_size(rng, 64, 8192), dtype=dtype)


# --------------------------------------------------------------------------- inputs


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _dims(case):
    return (case["m"], case["n"]) + ((case["q"],) if case.get("q") else ())


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _gauss(dims, g, dtype):
    return torch.randn(dims, generator=g, device=DEV, dtype=torch.float64).to(dtype)


def _weights(m, n, g, dtype):
    """Noise, a rank-16 part with a tenth of the energy, one column in a hundred eight times as large, bf16 values."""
    a = torch.randn((m, n), generator=g, device=DEV) * 0.02
    low = torch.randn((m, 16), generator=g, device=DEV) @ torch.randn((16, n), generator=g, device=DEV)
    a += low * float(a.norm() / low.norm() / 3.0)
    cols = torch.randperm(n, generator=g, device=DEV)[: n // 100]
    a[:, cols] *= 8.0
    return a.to(torch.bfloat16).to(dtype).contiguous()


def _image(dims, g, dtype):
    """Per channel a gradient and smooth blobs of many sizes around a mean grey, integers 0..255."""
    m, n, q = dims
    y = torch.arange(m, device=DEV, dtype=torch.float32)[:, None] / m
    x = torch.arange(n, device=DEV, dtype=torch.float32)[None, :] / n
    out = torch.empty(dims, device=DEV, dtype=torch.float32)
    for ch in range(q):
        p = torch.rand((60, 5), generator=g, device=DEV).cpu()
        img = 128.0 + 40.0 * (float(p[0, 0]) - 0.5) * y + 40.0 * (float(p[0, 1]) - 0.5) * x
        sy = torch.exp(-5.0 + 3.7 * p[:, 2])
        sx = torch.exp(-5.0 + 3.7 * p[:, 3])
        # separable blobs: rows (m x blobs) times columns (blobs x n)
        by = torch.exp(-0.5 * ((y - p[:, 0].to(DEV)) / sy.to(DEV)) ** 2) * (160.0 * (p[:, 4].to(DEV) - 0.5))
        bx = torch.exp(-0.5 * ((x.T - p[:, 1].to(DEV)) / sx.to(DEV)) ** 2)
        out[:, :, ch] = (img + by @ bx.T).round().clamp(0, 255)
    return out.to(dtype).contiguous()


def _bitset(w, n, g):
    """w random sign vectors of length n, packed, padding bits clear."""
    words = scd.words(n)
    b = torch.randint(-(2 ** 63), 2 ** 63 - 1, (w, words), generator=g, device=DEV, dtype=torch.int64)
    if n % 64:
        b[:, -1] &= (1 << (n % 64)) - 1
    return b


def prepare(case, seed):
    g = _gen(seed)
    kind, dtype = case["kind"], _dtype(case)
    st = dict(case=case, seed=int(seed))
    if kind == "matrix":
        st["A"] = _weights(case["m"], case["n"], g, dtype) if case["law"] == "weights" else _gauss(_dims(case), g, dtype)
    elif kind == "image":
        st["A"] = _image(_dims(case), g, dtype)
    elif kind == "lsq":
        st["A"] = _gauss(_dims(case), g, dtype)
    elif kind == "halfsteps":
        st["A"] = _gauss(_dims(case), g, dtype)
    elif kind in ("apply", "expand"):
        st["signs"] = [_bitset(case["w"], d, g) for d in _dims(case)]
        # coefficients fall off exponentially, as those of a greedy decomposition do
        k = torch.arange(case["w"], device=DEV, dtype=torch.float64)
        st["c"] = (0.02 * torch.exp(-3.7 * k / case["w"]) * (1 + 0.05 * torch.rand(case["w"], generator=g, device=DEV))).to(dtype)
        if kind == "apply":
            nin = case["m"] if case["transpose"] else case["n"]
            x = _gauss((case["nvec"], nin), g, dtype)
            st["x"] = x[0].contiguous() if case["nvec"] == 1 else x
            need = scd.lib().scd_apply_workspace_bytes(case["m"], case["n"], case["w"])
            st["workspace"] = torch.empty((need + 7) // 8, dtype=torch.float64, device=DEV)
    return st


# --------------------------------------------------------------------------- one pass


def _numbers(res, case):
    if case["dtype"] == "f64":
        return dict(signs=list(res["signs"]), c=res["c"], trace=res["trace"], iters=res["iters"])
    return dict(c=res["c"], trace=res["trace"])


def run(st):
    case, seed = st["case"], st["seed"]
    kind = case["kind"]
    if kind == "matrix":
        if not case["share"]:
            return _numbers(scd.scd_decompose(st["A"], case["w"], seed), case)
        with scd.ScdContext(st["A"], case["w"], seed) as ctx:
            ctx.set_workgroups(case["share"])
            ctx.run(case["w"])
            return _numbers(ctx.results(), case)
    if kind == "image":
        call = scd.scd_decompose_scalars if case["scalars"] else scd.scd_decompose
        return _numbers(call(st["A"], case["w"], seed), case)
    if kind == "lsq":
        return _numbers(scd.scd_lsq_decompose(st["A"], case["w"], seed), case)
    if kind == "apply":
        return scd.scd_apply(st["signs"][0], st["signs"][1], st["c"], case["m"], case["n"], st["x"],
                             transpose=bool(case["transpose"]), workspace=st["workspace"])
    if kind == "expand":
        return scd.scd_expand(st["signs"], st["c"], _dims(case))
    t0 = scd.scd_rng_signs(seed, 0, 1, case["n"])
    u, s = scd.scd_row_signed_sum(st["A"], t0)
    v, t, c = scd.scd_col_signed_sum(st["A"], s)
    return dict(t0=t0, u=u, s=s, v=v, t=t, c=c)


# --------------------------------------------------------------------------- what a pass cannot do without


def _alternations(case):
    """Alternations a term takes on these inputs (a fit to measured runs: 70 at 4096x4096, 39 at 14336x4096, 21 at
    1024x4096; 8 sweeps on the image-like tensor)."""
    if case["kind"] == "image":
        return 8.0
    lo, hi = sorted((case["m"], case["n"]))
    return 4.0 + lo / math.sqrt(hi)


def work(case):
    dims = _dims(case)
    total = math.prod(dims)
    es = 4 if case["dtype"] == "f32" else 8
    kind, w = case["kind"], case.get("w", 1)
    packed = sum(scd.words(d) * 8 for d in dims)  # sign bits of one term
    if kind in ("matrix", "image", "lsq"):
        # the input once, the packed terms once; an addition per entry and half step, the update of every term
        return dict(bytes=float(total * es + w * (packed + es + 12)), flops=float(total) * w * (2.0 * _alternations(case) + 3.0))
    if kind == "apply":
        nv = case["nvec"]
        return dict(bytes=float(w * (packed + es) + nv * es * sum(dims)), flops=2.0 * nv * w * sum(dims))
    if kind == "expand":
        return dict(bytes=float(w * (packed + es) + total * es), flops=2.0 * total * w)
    # each half step is a call of its own on the whole matrix
    return dict(bytes=float(2 * total * es + 2 * packed + 8 * sum(dims)), flops=2.0 * total)


def tolerance(case):
    kind, f32 = case["kind"], case["dtype"] == "f32"
    if kind == "expand":
        return "exact"  # the terms are added in their order into one f64 sum per entry
    if kind == "halfsteps":
        return {"rel": 6e-7} if f32 else {"rel": 1e-14}  # measured against 64 bits: 1.5e-7
    if kind == "apply":
        return {"rel": 1.2e-7} if f32 else {"rel": 1e-14}  # measured: 2.7e-8
    if not f32:
        return {"rel": 1e-10, "max": 1e-9}
    # another way out of one near tie: the coefficients of the later terms differ by as much as local maxima do
    # (measured between engines at 4096x4096: 5e-3, the largest entry 2.1e-2; without a near tie 2e-8)
    return {"rel": 0.02, "max": 0.1}


# --------------------------------------------------------------------------- 64-bit reference


_G, _H, _K = 0x9E3779B97F4A7C15, 0xD1B54A32D192ED03, 0x8CB92BA72F3D8DD7
_M64 = (1 << 64) - 1


def _mix(z):
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _M64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _M64
    return z ^ (z >> 31)


def _start_words(seed, term, mode, n):
    base = _mix(_mix((seed & _M64) ^ (_G * (term + 1) & _M64)) + _H * (mode + 1) & _M64)
    out = [_mix(base + _K * (p + 1) & _M64) for p in range(scd.words(n))]
    if n % 64:
        out[-1] &= (1 << (n % 64)) - 1
    return torch.tensor([x - (1 << 64) if x >> 63 else x for x in out], dtype=torch.int64)


def _dense(bits, n):
    """+-1 in f64 from packed signs (last dimension words)."""
    q = torch.arange(64, device=bits.device)
    b = (bits.unsqueeze(-1) >> q) & 1
    return 1.0 - 2.0 * b.reshape(*bits.shape[:-1], -1)[..., :n].double()


def _pack(v):
    """Packed signs (1 where v < 0) of a vector."""
    n = v.numel()
    b = torch.zeros(scd.words(n) * 64, dtype=torch.int64, device=v.device)
    b[:n] = (v < 0).to(torch.int64)
    b = b.reshape(-1, 64) << torch.arange(64, device=v.device)
    return b.sum(-1)  # distinct bits: the sum is their union (bit 63 wraps to the sign)


def _cut(R, t):
    """Greedy signed cut: alternate s = sgn(R t), t = sgn(R^T s) until <s, R t> stops growing."""
    prev, j = -math.inf, 0
    while True:
        s = 1.0 - 2.0 * (R.mv(t) < 0).double()
        v = R.t().mv(s)
        t = 1.0 - 2.0 * (v < 0).double()
        cut = float(v.abs().sum())
        j += 1
        if cut <= prev:
            return s, t, cut, j
        prev = cut


def _exact_matrix(case, seed):
    A = prepare(case, seed)["A"].double()
    m, n = A.shape
    R, S, T, c, trace, iters = A.clone(), [], [], [], [float(A.norm())], []
    lsq = case["kind"] == "lsq"
    Sd, Td = [], []
    for k in range(case["w"]):
        s, t, cut, j = _cut(R, _dense(_start_words(seed, k, 1, n).to(DEV), n))
        S.append(_pack(-1.0 * (s < 0).double()))
        T.append(_pack(-1.0 * (t < 0).double()))
        iters.append(j)
        if lsq:
            Sd.append(s)
            Td.append(t)
            sm, tm = torch.stack(Sd), torch.stack(Td)
            coef = torch.linalg.solve((sm @ sm.t()) * (tm @ tm.t()), ((sm @ A) * tm).sum(1))
            R = A - (sm * coef[:, None]).t() @ tm
            c = [coef]
        else:
            c.append(torch.tensor([cut / (m * n)], device=DEV, dtype=torch.float64))
            R = R - c[-1] * torch.outer(s, t)
        trace.append(float(R.norm()))
    return dict(signs=[torch.stack(S), torch.stack(T)], c=torch.cat(c), trace=torch.tensor(trace, dtype=torch.float64),
                iters=torch.tensor(iters, dtype=torch.int32))


def exact(case, seed):
    kind = case["kind"]
    dims = _dims(case)
    if kind in ("matrix", "lsq"):
        # f32 runs have no single answer (near ties)
        if case["dtype"] != "f64" or len(dims) != 2:
            return None
        return _exact_matrix(case, seed)
    if kind == "image":
        return None
    st = prepare(case, seed)
    if kind == "halfsteps":
        A = st["A"].double()
        t0 = _start_words(seed, 0, 1, case["n"]).to(DEV)
        u = (A * _dense(t0, case["n"])).sum(1)
        s = _pack(u)
        v = (A * _dense(s, case["m"])[:, None]).sum(0)
        return dict(t0=t0, u=u, s=s, v=v, t=_pack(v), c=v.abs().sum().reshape(1))
    c = st["c"].double()
    if kind == "apply":
        S, T = st["signs"]
        ib, ob = (S, T) if case["transpose"] else (T, S)
        nin, nout = (case["m"], case["n"]) if case["transpose"] else (case["n"], case["m"])
        x = st["x"].double().reshape(-1, nin)
        y = torch.zeros((x.shape[0], nout), dtype=torch.float64, device=DEV)
        for a in range(0, case["w"], 1024):
            z = x @ _dense(ib[a:a + 1024], nin).t() * c[a:a + 1024]
            y += z @ _dense(ob[a:a + 1024], nout)
        return y[0] if case["nvec"] == 1 else y
    out = torch.zeros((dims[0], math.prod(dims[1:])), dtype=torch.float64, device=DEV)
    for a in range(0, case["w"], 512):
        right = _dense(st["signs"][1][a:a + 512], dims[1])
        if len(dims) == 3:
            right = (right[:, :, None] * _dense(st["signs"][2][a:a + 512], dims[2])[:, None, :]).reshape(right.shape[0], -1)
        out += (_dense(st["signs"][0][a:a + 512], dims[0]) * c[a:a + 512, None]).t() @ right
    return out.reshape(dims)
