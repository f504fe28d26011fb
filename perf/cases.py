"""Timed workloads of the block-Toeplitz operator, through its public calls.

A case is a dict of plain values: ``kind`` names the work, the rest its
sizes.  Kinds and what they stand for:

* ``gradient``: one objective evaluation of an optimiser, misfit and gradient
  (forward and adjoint product with the misfit between them);
* ``gauss_newton``: Gauss-Newton Hessian products F* F v for several vectors
  (a block Krylov or randomised method), forward then adjoint;
* ``ragged``: a batch of event windows of different lengths, forward products
  of parameter series and adjoint products of data series;
* ``columns``: columns F F* e_j of the data-space operator (assembly of K);
* ``load``: a new operator from its time-domain blocks, up to its first
  product;
* ``factor``: K from the blocks and its Cholesky factor (offline phase);
* ``online``: the MAP point of new observations and the QoI prediction Q d;
* ``qoi``: rows of the data-to-QoI map, all of them (offline phase).

The online and QoI phases use FP64 plans, as they subtract nearly equal
numbers through K^-1.  The misfit of a plan with FP32 series is returned in
FP32, as a program that logs it beside its FP32 gradient keeps it.
"""
import math

import torch

from paper_2501_14911_amd import (P2OOperator, assemble_K_from_blocks, cholesky, d2q_apply)

CHUNK = 4096                    # columns per block chunk (the loader's scale block)
DEV = "cuda"
QOIS, QOI_STEP = 16, 10        # QoIs, observed every 10th step
ELEM = {"fp64": 16, "fp32": 8, "bf16": 4, "fp16": 4}


def listed():
    return [
        # the smallest call: a 4-sensor toy problem in an optimiser's loop, launches and latency only
        dict(name="gradient_tiny_fp64", kind="gradient", Nd=4, Nm=64, Nt=16, prec="fp64", nrhs=1),
        # one gradient at the time-dependent benchmark's size: the spectrum is streamed twice
        dict(name="gradient_600_fp16", kind="gradient", Nd=600, Nm=16384, Nt=420, prec="fp16", nrhs=1),
        # block Krylov on the medium problem, in the precision the paper uses
        dict(name="gauss_newton_64_fp64", kind="gauss_newton", Nd=64, Nm=4096, Nt=128, prec="fp64", nrhs=8),
        # the same in single precision on a year of daily steps (transform length 750), odd sizes
        dict(name="gauss_newton_101_fp32", kind="gauss_newton", Nd=101, Nm=10007, Nt=365, prec="fp32", nrhs=4),
        # event windows on a small BF16 operator, nothing a multiple of anything
        dict(name="ragged_37_bf16", kind="ragged", Nd=37, Nm=5003, Nt=241, prec="bf16", nrhs=5),
        # 32 windows of 64..420 steps at the benchmark's size
        dict(name="ragged_600_fp16", kind="ragged", Nd=600, Nm=16384, Nt=420, prec="fp16", nrhs=32),
        # 64 data-space columns at the benchmark's size
        dict(name="columns_600_fp16", kind="columns", Nd=600, Nm=16384, Nt=420, prec="fp16", nrhs=64),
        # 32 data-space columns at the paper's size: few sensors, a 513 x 513 parameter grid
        dict(name="columns_49_fp16", kind="columns", Nd=49, Nm=513 * 513, Nt=500, prec="fp16", nrhs=32),
        # a new medium operator: loading and the first product
        dict(name="load_64_fp16", kind="load", Nd=64, Nm=16384, Nt=128, prec="fp16", nrhs=1),
        # K and its factor for the medium problem (8192 data)
        dict(name="factor_64", kind="factor", Nd=64, Nm=4096, Nt=128, prec="fp64", nrhs=1),
        # the warning centre's call: one set of observations in, the MAP point and the QoIs out (12250 data)
        dict(name="online_49_fp64", kind="online", Nd=49, Nm=16384, Nt=250, prec="fp64", nrhs=1),
        # the data-to-QoI map of a smaller network (4000 data, 16 QoIs every 10th step)
        dict(name="qoi_16_fp64", kind="qoi", Nd=16, Nm=16384, Nt=250, prec="fp64", nrhs=32),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["gradient", "gauss_newton", "gauss_newton", "ragged", "ragged", "columns", "columns", "load",
                       "factor", "online", "qoi"])
    while True:
        c = dict(kind=kind, Nd=_log(rng, 4, 600), Nm=_log(rng, 64, 65536), Nt=_log(rng, 16, 500), prec="fp64", nrhs=1)
        if kind == "gradient":
            c.update(prec=rng.choice(["fp64", "fp32", "bf16", "fp16"]))
        elif kind == "gauss_newton":
            c.update(prec=rng.choice(["fp64", "fp32", "bf16", "fp16"]), nrhs=_log(rng, 2, 16))
        elif kind == "ragged":
            c.update(prec=rng.choice(["fp64", "fp32", "bf16", "fp16"]), nrhs=_log(rng, 2, 32))
        elif kind == "columns":
            c.update(prec=rng.choice(["fp64", "fp32", "fp16", "fp16"]), nrhs=_log(rng, 8, 64))
        elif kind == "load":
            c.update(prec=rng.choice(["fp64", "fp32", "bf16", "fp16"]))
        elif kind == "qoi":
            c.update(nrhs=_log(rng, 8, 32))
        if kind in ("online", "qoi"):
            c.update(Nt=10 * max(2, c["Nt"] // 10))         # QoIs every 10th step
        N = c["Nd"] * c["Nt"]
        spectrum = c["Nd"] * c["Nm"] * (c["Nt"] + 1) * ELEM[c["prec"]]
        series = c["nrhs"] * c["Nm"] * (c["Nt"] + 1) * (16 if c["prec"] == "fp64" else 8)
        if spectrum > 5e9 or series > 4e9 or (kind in ("gauss_newton", "columns") and spectrum * c["nrhs"] > 6e10):
            continue
        if kind in ("factor", "online", "qoi") and (N > 12000 or N < 200 or N * N * c["Nm"] > 1e12):
            continue
        return c


# ------------------------------------------------------------------ inputs
def _seed(seed, *more):
    s = seed
    for v in more:
        s = (s * 1000003 + v + 1) % (1 << 62)
    return s


def _blocks(c, seed, which, c0, n, Nd=None):
    """F_k[:, c0:c0+n] for all k: Gaussian with an exponential decay over the lags, [Nt, Nd, n] float32."""
    g = torch.Generator(device=DEV).manual_seed(_seed(seed, which, c0))
    Nt = c["Nt"]
    F = torch.randn((Nt, Nd or c["Nd"], n), generator=g, device=DEV, dtype=torch.float32)
    k = torch.arange(Nt, device=DEV, dtype=torch.float32)
    return F.mul_(torch.exp(-k / max(Nt / 4, 1.0))[:, None, None] / math.sqrt(c["Nm"]))


def _series(c, seed, which, nrhs, last):
    g = torch.Generator(device=DEV).manual_seed(_seed(seed, 100 + which))
    dt = torch.float64 if c["prec"] == "fp64" else torch.float32
    return torch.randn((nrhs, c["Nt"], last), generator=g, device=DEV, dtype=dt)


def _lengths(c, seed):
    g = torch.Generator().manual_seed(_seed(seed, 200))
    return torch.randint(max(1, c["Nt"] * 64 // 420), c["Nt"] + 1, (c["nrhs"],), generator=g, dtype=torch.int32)


def _units(c, seed):
    N = c["Nd"] * c["Nt"]
    g = torch.Generator().manual_seed(_seed(seed, 300))
    j = torch.randint(0, N, (c["nrhs"],), generator=g)
    j[0] = j[0] % c["Nd"]                                   # one at the first step
    e = torch.zeros((c["nrhs"], N), device=DEV, dtype=torch.float64 if c["prec"] == "fp64" else torch.float32)
    e[torch.arange(c["nrhs"], device=DEV), j.to(DEV)] = 1.0
    return e.reshape(c["nrhs"], c["Nt"], c["Nd"])


def _noise(c):
    """One variance per sensor around 1e-2."""
    return 1e-2 * (1.0 + 0.5 * torch.cos(torch.arange(c["Nd"], device=DEV, dtype=torch.float64)))


def _operator(c, seed, which=0, Nd=None):
    op = P2OOperator(Nd or c["Nd"], c["Nm"], c["Nt"], c["prec"], max_rhs=c["nrhs"])
    op.load(lambda c0, n: _blocks(c, seed, which, c0, n, Nd), chunk_cols=CHUNK)
    return op


def _all_blocks(c, seed):
    return torch.cat([_blocks(c, seed, 0, c0, min(CHUNK, c["Nm"] - c0)) for c0 in range(0, c["Nm"], CHUNK)], dim=2)


def _factor(c, seed):
    K = assemble_K_from_blocks(lambda c0, n: _blocks(c, seed, 0, c0, n), c["Nd"], c["Nm"], c["Nt"], _noise(c),
                               chunk_cols=CHUNK)
    return cholesky(K)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = dict(c=c)
    if kind == "load":
        s["op"] = P2OOperator(c["Nd"], c["Nm"], c["Nt"], c["prec"], max_rhs=c["nrhs"])
        s["blocks"] = _all_blocks(c, seed)
        s["m"] = _series(c, seed, 0, c["nrhs"], c["Nm"])
        return s
    if kind == "factor":
        s["blocks"] = _all_blocks(c, seed).double()
        s["var"] = _noise(c)
        return s
    s["op"] = _operator(c, seed)
    if kind == "gradient":
        s["m"] = _series(c, seed, 0, c["nrhs"], c["Nm"])
        s["d"] = _series(c, seed, 1, c["nrhs"], c["Nd"])
        s["var"] = _noise(c)
    elif kind == "gauss_newton":
        s["m"] = _series(c, seed, 0, c["nrhs"], c["Nm"])
    elif kind == "ragged":
        s["m"] = _series(c, seed, 0, c["nrhs"], c["Nm"])
        s["d"] = _series(c, seed, 1, c["nrhs"], c["Nd"])
        s["nt"] = _lengths(c, seed).to(DEV)
    elif kind == "columns":
        s["e"] = _units(c, seed)
    elif kind == "online":
        s["L"] = _factor(c, seed)
        s["var"] = _noise(c)
        s["d"] = 0.1 * _series(c, seed, 1, 1, c["Nd"])[0]
        fq = P2OOperator(QOIS, c["Nm"], c["Nt"], c["prec"], max_rhs=16)
        fq.load(lambda c0, n: _blocks(c, seed, 1, c0, n, QOIS), chunk_cols=CHUNK)
        fq.set_output_stride(QOI_STEP)
        f16 = P2OOperator(c["Nd"], c["Nm"], c["Nt"], c["prec"], max_rhs=16)
        f16.load(lambda c0, n: _blocks(c, seed, 0, c0, n), chunk_cols=CHUNK)
        s["Q"] = f16.d2q_map(fq, s["L"], s["var"])
        fq.close()
        f16.close()
    elif kind == "qoi":
        s["L"] = _factor(c, seed)
        s["var"] = _noise(c)
        s["fq"] = _operator(c, seed, 1, QOIS)
        s["fq"].set_output_stride(QOI_STEP)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    c, kind = s["c"], s["c"]["kind"]
    if kind == "load":
        B = s["blocks"]
        s["op"].load(lambda c0, n: B[:, :, c0:c0 + n], chunk_cols=CHUNK)
        return {"d": s["op"].apply_F(s["m"])}
    if kind == "factor":
        B = s["blocks"]
        K = assemble_K_from_blocks(lambda c0, n: B[:, :, c0:c0 + n], c["Nd"], c["Nm"], c["Nt"], s["var"])
        return {"L": cholesky(K)}
    op = s["op"]
    if kind == "gradient":
        phi, grad = op.misfit_grad(s["m"], s["d"], s["var"])
        return {"phi": phi.to(grad.dtype), "grad": grad}
    if kind == "gauss_newton":
        d = op.apply_F(s["m"])
        return {"d": d, "g": op.apply_Ft(d)}
    if kind == "ragged":
        return {"d": op.apply_F(s["m"], s["nt"]), "m": op.apply_Ft(s["d"], s["nt"])}
    if kind == "columns":
        return {"h": op.apply_FFt(s["e"])}
    if kind == "online":
        m = op.map_point(s["d"], s["L"], s["var"])
        return {"m": m, "q": d2q_apply(s["Q"], s["d"].reshape(-1))}
    return {"Q": op.d2q_map(s["fq"], s["L"], s["var"])}


def work(case):
    """Bytes: the spectrum (or blocks, factor) once per product that has to follow another, inputs and outputs once.
    Flops: 8 per complex multiply-add of the products, the dense algebra's usual counts, 5 L/2 log2(L/2) per transform."""
    c, kind = case, case["kind"]
    Nd, Nm, Nt, B = c["Nd"], c["Nm"], c["Nt"], c["nrhs"]
    io = 8 if c["prec"] == "fp64" else 4
    N = Nd * Nt
    spec = (Nt + 1) * Nd * Nm * ELEM[c["prec"]]
    mv = 8 * (Nt + 1) * Nd * Nm                              # flops of one product with one right-hand side
    fft = 5 * Nt * math.log2(max(Nt, 2))
    ms, ds = io * Nt * Nm, io * N                            # bytes of one parameter or data series
    nq = QOIS * (Nt // QOI_STEP)
    if kind == "gradient":
        return dict(bytes=2 * spec + B * (2 * ms + ds), flops=B * (2 * mv + 2 * fft * (Nm + Nd)))
    if kind == "gauss_newton":
        return dict(bytes=2 * spec + B * (2 * ms + ds), flops=B * (2 * mv + 2 * fft * (Nm + Nd)))
    if kind == "ragged":
        return dict(bytes=2 * spec + 2 * B * (ms + ds), flops=B * (2 * mv + 2 * fft * (Nm + Nd)))
    if kind == "columns":
        return dict(bytes=2 * spec + 2 * B * ds, flops=B * (2 * mv + 2 * fft * (Nm + Nd)))
    if kind == "load":
        return dict(bytes=4 * N * Nm + spec + spec + ms + ds, flops=Nd * Nm * fft + mv + fft * (Nm + Nd))
    if kind == "factor":
        return dict(bytes=8 * N * Nm + 8 * N * N, flops=N * N * Nm + N ** 3 / 3)
    if kind == "online":
        return dict(bytes=3 * spec + 2 * 4 * N * N + ms + ds + 8 * nq * N,
                    flops=3 * mv + 2 * 2 * N * N / 2 + 3 * fft * (Nm + Nd) + 2 * nq * N)
    spq = (Nt + 1) * QOIS * Nm * ELEM[c["prec"]]
    return dict(bytes=spq + 3 * spec + 8 * N * N + 8 * nq * N,
                flops=nq * (3 * mv + 8 * (Nt + 1) * QOIS * Nm + 2 * N * N + 4 * fft * Nm))


# ------------------------------------------------------------------ the same results in 64 bits
def _chunks(c, nrhs):
    per = (2 * c["Nt"]) * 16 * (c["Nd"] + 3 * nrhs)
    n = max(64, min(CHUNK, int(2e9 / per) // 64 * 64))
    for b0 in range(0, c["Nm"], CHUNK):
        width = min(CHUNK, c["Nm"] - b0)
        for c0 in range(0, width, n):
            yield b0, width, c0, min(n, width - c0)


def _spectra(c, seed, nrhs, which=0, Nd=None):
    """Half spectra of the blocks, column chunk by column chunk: (first column, columns, [bins, Nd, columns])."""
    have, F = None, None
    for b0, width, c0, n in _chunks(c, nrhs):
        if have != b0:
            have, F = b0, _blocks(c, seed, which, b0, width, Nd)
        yield b0 + c0, n, torch.fft.rfft(F[:, :, c0:c0 + n].double(), n=2 * c["Nt"], dim=0)


def _mask(c, nt):
    return 1.0 if nt is None else (torch.arange(c["Nt"], device=DEV)[None, :] < nt[:, None]).double()[:, :, None]


def _hat(c, x):
    """[nrhs, Nt, n] -> [bins, n, nrhs]."""
    return torch.fft.rfft(x, n=2 * c["Nt"], dim=1).permute(1, 2, 0).contiguous()


def _unhat(c, X):
    return torch.fft.irfft(X.permute(2, 0, 1).contiguous(), n=2 * c["Nt"], dim=1)[:, :c["Nt"]].contiguous()


def _forward(c, seed, m, nt=None, which=0, Nd=None):
    m, y = m.double(), 0
    for c0, n, F in _spectra(c, seed, m.shape[0], which, Nd):
        y = y + torch.bmm(F, _hat(c, m[:, :, c0:c0 + n] * _mask(c, nt)))
    return _unhat(c, y) * _mask(c, nt)


def _adjoint(c, seed, d, nt=None, out=None, which=0, Nd=None):
    y = _hat(c, d.double() * _mask(c, nt))
    m = torch.empty((d.shape[0], c["Nt"], c["Nm"]), dtype=torch.float64, device=DEV)
    for c0, n, F in _spectra(c, seed, d.shape[0], which, Nd):
        Fh = F.conj().transpose(1, 2).resolve_conj().contiguous()
        m[:, :, c0:c0 + n] = _unhat(c, torch.bmm(Fh, y)) * _mask(c, nt)
    return m


def _columns(c, seed, e, which=0, Nd=None):
    """F G* e, G the map with Nd sensors drawn as ``which`` (F itself by default)."""
    y, h = _hat(c, e.double()), 0
    other = _spectra(c, seed, e.shape[0], which, Nd)
    for c0, n, F in _spectra(c, seed, e.shape[0]):
        G = F if which == 0 else next(other)[2]
        Gh = G.conj().transpose(1, 2).resolve_conj().contiguous()
        h = h + torch.bmm(F, _hat(c, _unhat(c, torch.bmm(Gh, y))))
    return _unhat(c, h)


def _K(c, seed):
    Nt, Nd, N = c["Nt"], c["Nd"], c["Nt"] * c["Nd"]
    G = torch.zeros((N, N), dtype=torch.float64, device=DEV)
    for c0 in range(0, c["Nm"], CHUNK):
        A = _blocks(c, seed, 0, c0, min(CHUNK, c["Nm"] - c0)).double().reshape(N, -1)
        G.addmm_(A, A.T)
    for t in range(1, Nt):
        G[t * Nd:(t + 1) * Nd, Nd:] += G[(t - 1) * Nd:t * Nd, :-Nd]
    G.diagonal().add_(_noise(c).repeat(Nt))
    return G


def _solve(K, x):
    """K^-1 x for rows x."""
    L = torch.linalg.cholesky(K)
    return torch.cholesky_solve(x.T.contiguous(), L).T.contiguous()


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "load":
        return {"d": _forward(c, seed, _series(c, seed, 0, c["nrhs"], c["Nm"]))}
    if kind == "factor":
        # row j of the result is column j: L below (transposed) and L^T above the diagonal
        L = torch.linalg.cholesky(_K(c, seed))
        return {"L": L + L.T - torch.diag(L.diagonal())}
    if kind == "gradient":
        var = _noise(c)
        r = _forward(c, seed, _series(c, seed, 0, c["nrhs"], c["Nm"])) - _series(c, seed, 1, c["nrhs"], c["Nd"]).double()
        return {"phi": 0.5 * (r * r / var).sum(dim=(1, 2)), "grad": _adjoint(c, seed, r / var)}
    if kind == "gauss_newton":
        d = _forward(c, seed, _series(c, seed, 0, c["nrhs"], c["Nm"]))
        return {"d": d, "g": _adjoint(c, seed, d)}
    if kind == "ragged":
        nt = _lengths(c, seed).to(DEV)
        return {"d": _forward(c, seed, _series(c, seed, 0, c["nrhs"], c["Nm"]), nt),
                "m": _adjoint(c, seed, _series(c, seed, 1, c["nrhs"], c["Nd"]), nt)}
    if kind == "columns":
        return {"h": _columns(c, seed, _units(c, seed))}
    K, N = _K(c, seed), c["Nt"] * c["Nd"]
    if kind == "online":
        # m = F* K^-1 d (the Woodbury form with unit prior variance), q = F_q m at the QoI steps
        d = 0.1 * _series(c, seed, 1, 1, c["Nd"])
        m = _adjoint(c, seed, _solve(K, d.reshape(1, N)).reshape(1, c["Nt"], c["Nd"]))
        r = QOI_STEP
        return {"m": m[0], "q": _forward(c, seed, m, which=1, Nd=QOIS)[0, r - 1::r].reshape(-1)}
    # Q = F_q F* K^-1: row i is K^-1 F F_q* e_i
    r, nq = QOI_STEP, QOIS * (c["Nt"] // QOI_STEP)
    rows = []
    for i0 in range(0, nq, 64):
        b = min(64, nq - i0)
        e = torch.zeros((b, c["Nt"], QOIS), dtype=torch.float64, device=DEV)
        i = torch.arange(i0, i0 + b, device=DEV)
        e[torch.arange(b, device=DEV), r * (i // QOIS + 1) - 1, i % QOIS] = 1.0
        rows.append(_columns(c, seed, e, which=1, Nd=QOIS).reshape(b, N))
    return {"Q": _solve(K, torch.cat(rows))}
