"""Timed cases of the batched GEMM library: what its callers have it do, through
the Python binding, over the sizes, layouts, element types and precision modes
it serves.

A case is a dict of plain values; ``kind`` selects the entry point:

``gemm``   uniform binary64 batch (``Handle.batched``) or, with ``mode``, the
           same batch in a precision mode (``Handle.batched_mode``);
``vgemm``  variable sizes (``Handle.vbatched``);
``zgemm``  uniform complex batch (``Handle.zbatched``);
``gate``   two-spin gates on a batch of states (``Handle.zgate2``);
``serve``  the request loop draining a backlog (``serve.Server``).

Matrices are column-major, stored as (batch, cols, ld) tensors.
"""
import math

import numpy as np
import torch

from paper_2203_09353_amd import bgemm, serve

DEV = "cuda"


def _gemm(name, batch, m, n, k, ta="N", tb="N", alpha=1.0, beta=1.0, pad=0, mode="fp64", slices=0):
    return {"name": name, "kind": "gemm", "batch": batch, "m": m, "n": n, "k": k, "ta": ta,
            "tb": tb, "alpha": alpha, "beta": beta, "pad": pad, "mode": mode, "slices": slices}


def listed():
    return [
        # the smallest call in use: a thousand 32^3 products, bound by the
        # launch and by one trip to memory
        _gemm("uniform_32", 1000, 32, 32, 32, beta=0.0),
        # a very large batch of small products, accumulated in place
        _gemm("uniform_64", 200_000, 64, 64, 64),
        # the ordinary batch: 256^3, accumulated in place
        _gemm("uniform_256", 20_000, 256, 256, 256),
        # the largest matrices of the benchmark
        _gemm("uniform_512", 5_000, 512, 512, 512),
        # odd extents off every tile edge, a transposed operand, padded
        # leading dimensions and general scalars
        _gemm("odd_transposed", 3_000, 129, 513, 257, ta="T", alpha=1.5, beta=-0.5, pad=2),
        # a variable-size batch: m, n, k independently 2^j + {-1, 0, 1},
        # j in 3..9
        {"name": "variable_7_513", "kind": "vgemm", "batch": 100_000, "lo": 3, "hi": 9, "ta": "N",
         "tb": "N", "alpha": 1.0, "beta": 0.5, "pad": 0, "mix": 4},
        # the entropy step of a 15-spin chain: Hermitian Gram products
        # Psi Psi^H of 256 x 128 complex states
        {"name": "gram_256x128", "kind": "zgemm", "batch": 10_000, "m": 256, "n": 256, "k": 128,
         "ta": "N", "tb": "C", "beta": 0.0, "pad": 0, "gram": True},
        # the step before it at the largest chain: one two-spin gate on each
        # of 64 states of 21 spins, in place
        {"name": "gate_21", "kind": "gate", "spins": 21, "batch": 64},
        # callers that trade accuracy for speed: binary32 arithmetic
        _gemm("fp32_256", 20_000, 256, 256, 256, beta=0.0, mode="fp32"),
        # ... bfloat16 inputs with binary32 sums
        _gemm("bf16_256", 20_000, 256, 256, 256, beta=0.0, mode="bf16"),
        # ... and binary64 emulated with seven int8 digits per operand
        _gemm("int8x7_256", 20_000, 256, 256, 256, beta=0.0, mode="i8emu", slices=7),
        # the request loop: 32 clients with states of 32..512, a backlog of
        # 2000 requests of 1..16 products each, then every state read back
        {"name": "serve_backlog", "kind": "serve", "clients": 32, "kmin": 5, "kmax": 9,
         "requests": 2000, "max_len": 16},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "vgemm", "zgemm", "gate", "mode", "mode", "serve"])
    if kind == "gate":
        spins = rng.randint(6, 21)
        return {"kind": "gate", "spins": spins,
                "batch": min(_log_int(rng, 1, 2000), (1 << 27) >> spins) or 1}
    if kind == "serve":
        kmin = rng.randint(5, 8)
        return {"kind": "serve", "clients": rng.randint(4, 32), "kmin": kmin,
                "kmax": rng.randint(kmin, 9), "requests": _log_int(rng, 50, 1500),
                "max_len": rng.randint(1, 16)}
    if kind == "vgemm":
        lo = rng.randint(3, 6)
        hi = rng.randint(lo, 9)
        return {"kind": "vgemm", "batch": _log_int(rng, 500, 30_000), "lo": lo, "hi": hi,
                "ta": rng.choice("NT"), "tb": rng.choice("NT"), "alpha": 1.0,
                "beta": rng.choice([0.0, 0.5, 1.0]), "pad": rng.choice([0, 0, 1, 8]),
                "mix": rng.randint(5, 10 ** 6)}
    if kind == "zgemm":
        m, n, k = (_log_int(rng, 8, 400) for _ in range(3))
        ta, tb = rng.choice("NTC"), rng.choice("NTC")
        most = min(4e11 / (8.0 * m * n * k), 4e9 / (16.0 * (m * k + k * n + m * n)))
        return {"kind": "zgemm", "batch": _log_int(rng, 20, max(20, min(20_000, most))), "m": m,
                "n": n, "k": k, "ta": ta, "tb": tb, "beta": rng.choice([0.0, 1.0]),
                "pad": rng.choice([0, 0, 1, 3]), "gram": False}
    m, n, k = (_log_int(rng, 7, 513) for _ in range(3))
    if rng.random() < 0.5:  # whole tiles as often as odd extents
        m, n, k = (max(8, 8 * (x // 8)) for x in (m, n, k))
    most = min(4e11 / (2.0 * m * n * k), 6e9 / (8.0 * (m * k + k * n + 2 * m * n)))
    batch = _log_int(rng, 50, max(50, min(100_000, most)))
    alpha, beta = rng.choice([1.0, 1.0, -0.75]), rng.choice([0.0, 1.0, 0.5])
    pad = rng.choice([0, 0, 1, 2, 5])
    if kind == "mode":
        mode, slices = rng.choice([("fp32", 0), ("bf16", 0), ("i8emu", 5), ("i8emu", 6),
                                   ("i8emu", 7), ("i8emu", 8)])
        c = _gemm("", batch, m, n, k, "N", "N", alpha, beta, pad, mode, slices)
    else:
        c = _gemm("", batch, m, n, k, rng.choice("NT"), rng.choice("NT"), alpha, beta, pad)
    del c["name"]
    return c


# ---- inputs -------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _uniform(shape, gen, dtype=torch.float64):
    """Entries uniform in [-1, 1) (each part of a complex one)."""
    x = torch.empty(shape + ((2,) if dtype.is_complex else ()), dtype=torch.float64, device=DEV)
    x.uniform_(-1.0, 1.0, generator=gen)
    return torch.view_as_complex(x) if dtype.is_complex else x


def _wide(shape, gen):
    """Entries spread over magnitudes 2^-20..2^20, as the precision modes are
    studied on."""
    x = _uniform(shape, gen)
    e = torch.empty(shape, dtype=torch.float64, device=DEV).uniform_(-20.0, 20.0, generator=gen)
    return x.mul_(torch.exp2(e.round_()))


def _stored(rows, cols, trans):
    return (cols, rows) if trans == "N" else (rows, cols)   # (cols, rows) as stored


def _sizes(c):
    """Sizes of a variable-size batch: fixed by the case, so that every seed
    gives a batch of the same shape."""
    r = np.random.RandomState(c["mix"])
    j = r.randint(c["lo"], c["hi"] + 1, size=(3, c["batch"]))
    return (1 << j) + r.randint(-1, 2, size=(3, c["batch"]))


def _vb_layout(c):
    m, n, k = _sizes(c)
    rows = [m if c["ta"] == "N" else k, k if c["tb"] == "N" else n, m]
    cols = [k if c["ta"] == "N" else m, n if c["tb"] == "N" else k, n]
    lds = [r + c["pad"] for r in rows]
    offs = [np.concatenate([[0], np.cumsum(ld.astype(np.int64) * cl)]) for ld, cl in zip(lds, cols)]
    return (m, n, k), lds, cols, offs


def prepare(case, seed):
    c, gen = case, _generator(seed)
    if c["kind"] == "serve":
        h = bgemm.Handle()
        r = np.random.RandomState(c["clients"])
        sizes = 1 << r.randint(c["kmin"], c["kmax"] + 1, size=c["clients"])
        clients = r.randint(0, c["clients"], size=c["requests"])
        lengths = r.randint(1, c["max_len"] + 1, size=c["requests"])
        return {"c": c, "h": h, "server": serve.Server(h, sizes, seed), "clients": clients,
                "lengths": lengths, "arrivals": np.zeros(c["requests"])}
    h = bgemm.Handle()
    if c["kind"] == "gate":
        r = np.random.RandomState(seed % (1 << 32))
        b, s = c["batch"], c["spins"]
        z = r.normal(size=(b, 4, 4)) + 1j * r.normal(size=(b, 4, 4))
        q, t = np.linalg.qr(z)
        d = np.einsum("bii->bi", t)
        U = torch.from_numpy(np.ascontiguousarray(q * (d / np.abs(d))[:, None, :])).to(DEV)
        sites = torch.from_numpy(r.randint(0, s - 1, size=b).astype(np.int32)).to(DEV)
        psi = _uniform((b, 1 << s), gen, torch.complex128)
        psi *= math.sqrt(1.5 / (1 << s))
        return {"c": c, "h": h, "U": U, "sites": sites, "psi": psi}
    if c["kind"] == "vgemm":
        (m, n, k), lds, _, offs = _vb_layout(c)
        slabs = [_uniform((int(o[-1]),), gen) for o in offs]
        ptrs = tuple(torch.from_numpy(o[:-1] * 8 + s.data_ptr()).to(DEV) for o, s in zip(offs, slabs))
        i32 = [torch.from_numpy(x.astype(np.int32)).to(DEV) for x in (m, n, k, *lds)]
        info = torch.empty(c["batch"], dtype=torch.int32, device=DEV)
        return {"c": c, "h": h, "slabs": slabs, "ptrs": ptrs, "dims": i32, "info": info}
    dtype = torch.complex128 if c["kind"] == "zgemm" else torch.float64
    m, n, k, pad, b = c["m"], c["n"], c["k"], c["pad"], c["batch"]
    fill = (lambda shape: _wide(shape, gen)) if c.get("mode", "fp64") != "fp64" else (
        lambda shape: _uniform(shape, gen, dtype))
    (ca, ra), (cb, rb) = _stored(m, k, c["ta"]), _stored(k, n, c["tb"])
    A = fill((b, ca, ra + pad))
    B = A if c.get("gram") else fill((b, cb, rb + pad))
    C = (_uniform((b, n, m + pad), gen, dtype) if c["beta"] != 0.0 else
         torch.zeros((b, n, m + pad), dtype=dtype, device=DEV))
    ptrs = (bgemm.pointer_array(A), bgemm.pointer_array(B), bgemm.pointer_array(C))
    return {"c": c, "h": h, "A": A, "B": B, "C": C, "ptrs": ptrs}


# ---- one pass -----------------------------------------------------------------

def run(state):
    c, h = state["c"], state["h"]
    if c["kind"] == "serve":
        s = state["server"]
        s.reset()
        s.run(state["arrivals"], state["clients"], state["lengths"])
        return [s.state(i)[0] for i in range(c["clients"])]
    if c["kind"] == "gate":
        info = h.zgate2(c["spins"], state["sites"], state["U"], state["psi"])
        return {"psi": state["psi"], "info": info}
    if c["kind"] == "vgemm":
        m, n, k, lda, ldb, ldc = state["dims"]
        info = h.vbatched(None, None, None, m, n, k, c["alpha"], c["beta"], c["ta"], c["tb"],
                          ldas=lda, ldbs=ldb, ldcs=ldc, info=state["info"], ptrs=state["ptrs"])
        return {"C": state["slabs"][2], "info": info}
    A, B, C, ptrs = state["A"], state["B"], state["C"], state["ptrs"]
    m, n, k = c["m"], c["n"], c["k"]
    if c["kind"] == "zgemm":
        h.zbatched(A, B, C, m, n, k, 1.0, c["beta"], c["ta"], c["tb"], ptrs=ptrs)
    elif c["mode"] != "fp64":
        h.batched_mode(c["mode"], A, B, C, m, n, k, c["alpha"], c["beta"], c["slices"], ptrs=ptrs)
    else:
        h.batched(A, B, C, m, n, k, c["alpha"], c["beta"], c["ta"], c["tb"], ptrs=ptrs)
    return C


# ---- what a pass cannot do without ------------------------------------------------

def work(case):
    c = case
    if c["kind"] == "serve":
        r = np.random.RandomState(c["clients"])
        n = (1 << r.randint(c["kmin"], c["kmax"] + 1, size=c["clients"])).astype(np.float64)
        cl = r.randint(0, c["clients"], size=c["requests"])
        ln = r.randint(1, c["max_len"] + 1, size=c["requests"])
        # each product reads a state and writes one; factors need not leave
        # the chip's caches; every state is read back once
        return {"bytes": float((ln * 16 * n[cl] ** 2).sum() + (16 * n ** 2).sum()),
                "flops": float((ln * 2 * n[cl] ** 3).sum())}
    if c["kind"] == "gate":
        amps = float(c["batch"]) * (1 << c["spins"])
        return {"bytes": amps * 32 + c["batch"] * 256, "flops": amps * 32}
    if c["kind"] == "vgemm":
        m, n, k = (x.astype(np.float64) for x in _sizes(c))
        cw = 1 + (c["beta"] != 0.0)
        return {"bytes": float(8 * (m * k + k * n + cw * m * n).sum()) + 48.0 * c["batch"],
                "flops": float((2 * m * n * k).sum())}
    m, n, k, b = (float(c[x]) for x in ("m", "n", "k", "batch"))
    cw = 1 + (c["beta"] != 0.0)
    z = c["kind"] == "zgemm"
    operands = m * k if c.get("gram") else m * k + k * n
    return {"bytes": b * ((16 if z else 8) * (operands + cw * m * n) + 24),
            "flops": (8 if z else 2) * b * m * n * k}


# ---- the same in plain torch --------------------------------------------------

def _op_t(x, rows, trans):
    """op(X)^T, row-major, of a stored (batch, cols, ld) operand."""
    x = x[..., :rows]
    if trans == "N":
        return x.contiguous()
    x = x.transpose(-1, -2)
    return (x.conj() if trans == "C" else x).resolve_conj().contiguous()


def exact(case, seed):
    c = case
    if c["kind"] == "serve":
        return None
    s = prepare(case, seed)
    if c["kind"] == "gate":
        out = s["psi"].clone()
        for i in range(c["batch"]):
            j = int(s["sites"][i])
            v = s["psi"][i].view(-1, 4, 1 << j)
            out[i] = sum(s["U"][i][:, q].view(1, 4, 1) * v[:, q:q + 1, :] for q in range(4)).reshape(-1)
        return {"psi": out, "info": None}
    if c["kind"] == "vgemm":
        (m, n, k), lds, cols, offs = _vb_layout(c)
        A, B, C = s["slabs"]
        out = C.clone()
        for i in range(c["batch"]):
            a, b, d = (x[int(o[i]):int(o[i + 1])].view(int(cl[i]), int(ld[i])) for x, o, cl, ld in
                       zip((A, B, out), offs, cols, lds))
            a = a[:, :m[i]] if c["ta"] == "N" else a[:, :k[i]].t()
            b = b[:, :k[i]] if c["tb"] == "N" else b[:, :n[i]].t()
            d = d[:, :m[i]]
            d.copy_(torch.addmm(d, b, a, beta=c["beta"], alpha=c["alpha"]))
        return {"C": out, "info": None}
    m, n, k, alpha = c["m"], c["n"], c["k"], c.get("alpha", 1.0)
    ra = m if c["ta"] == "N" else k
    rb = k if c["tb"] == "N" else n
    out = s["C"].clone()
    step = max(1, int(2e8 / (m * k + k * n + m * n)))
    for i in range(0, c["batch"], step):
        at = _op_t(s["A"][i:i + step], ra, c["ta"])
        bt = _op_t(s["B"][i:i + step], rb, c["tb"])
        x = alpha * torch.matmul(bt, at)
        if c["beta"] != 0.0:
            x = x + c["beta"] * out[i:i + step, :, :m]
        out[i:i + step, :, :m] = x
    return out
