"""Performance cases of the library: the calls that programs using it make.

`listed()` names the cases, `draw(rng)` gives further ones from the same
ranges.  A case is a dict of plain values; `prepare` builds what a program
holds before the call (device buffers, plan, launch layout), `run` is one pass
through the public calls, `work` the bytes and operations a pass cannot do
without, and `exact` the same results in 64 bits from plain torch.

Kinds:
  stencil2d   one 2D stencil application (fixed weights or point function)
  set         the eight applications of the benchmark's stencil set
  fn          a stencil with a user function over two inputs
  ragged1d    a 1D stencil over uneven signals stored back to back
  solve       cyclic tri- or pentadiagonal solves (uneven lines, rows, columns)
  weno        the WENO advection term
  ch          steps of one Cahn-Hilliard grid
  ensemble    steps of many Cahn-Hilliard grids advanced together
  run         Cahn-Hilliard steps, then mass and coarsening diagnostics, as a
              long run does at every sample
"""
import math

import numpy as np
import torch

from paper_1902_09931_amd import binding as mxs

DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
WORD = {"f64": 8, "f32": 4, "bf16": 2}

# Windows (weights per unit spacing): second derivative of order 2, 4 and 8
# along one axis, the 9-point cross derivative, the 5-point Laplacian and the
# 13-point biharmonic.
D2_2ND = (1.0, -2.0, 1.0)
D2_4TH = (-1.0 / 12, 16.0 / 12, -30.0 / 12, 16.0 / 12, -1.0 / 12)
D2_8TH = (-1.0 / 560, 8.0 / 315, -1.0 / 5, 8.0 / 5, -205.0 / 72, 8.0 / 5, -1.0 / 5, 8.0 / 315, -1.0 / 560)
CROSS = (1.0, -2.0, 1.0, -2.0, 4.0, -2.0, 1.0, -2.0, 1.0)
LAPLACE = (0.0, 1.0, 0.0, 1.0, -4.0, 1.0, 0.0, 1.0, 0.0)
BIHARMONIC = (0.0, 0.0, 1.0, 0.0, 0.0,
              0.0, 2.0, -8.0, 2.0, 0.0,
              1.0, -8.0, 20.0, -8.0, 1.0,
              0.0, 2.0, -8.0, 2.0, 0.0,
              0.0, 0.0, 1.0, 0.0, 0.0)
CUBIC_MINUS_LINEAR = (0.0, -1.0, 0.0, 1.0)
D1_4TH = (1.0 / 12, -8.0 / 12, 0.0, 8.0 / 12, -1.0 / 12)

# name -> (direction, half width in x, half width in y, weights, coefficients)
STENCILS = {
    "x_d2_2nd": ("X", 1, 0, D2_2ND, None),
    "x_d2_4th": ("X", 2, 0, D2_4TH, None),
    "x_d2_8th": ("X", 4, 0, D2_8TH, None),
    "y_d2_2nd": ("Y", 0, 1, D2_2ND, None),
    "y_d2_4th": ("Y", 0, 2, D2_4TH, None),
    "y_d2_8th": ("Y", 0, 4, D2_8TH, None),
    "xy_cross": ("XY", 1, 1, CROSS, None),
    "xy_lap_cubic": ("XY", 1, 1, LAPLACE, CUBIC_MINUS_LINEAR),
    "xy_biharmonic": ("XY", 2, 2, BIHARMONIC, None),
}
SET = ("x_d2_4th", "y_d2_4th", "xy_cross", "xy_lap_cubic")

# A user function over two inputs: the Laplacian of the first window times the
# centre of the second.
FN_SOURCE = """
__device__ mxs_real flux(const mxs_real *const *w, const mxs_real *coe, int loc) {
    const mxs_real lap = w[0][loc - 3] + w[0][loc - 1] + w[0][loc + 1] + w[0][loc + 3] - coe[0] * w[0][loc];
    return lap * w[1][loc];
}
"""

D_COEF, GAMMA = 1.0, 0.01


def listed():
    return [
        # the smallest call: one derivative of a small grid, as in a first script
        {"name": "x_256_f64", "kind": "stencil2d", "stencil": "x_d2_4th", "nx": 256, "ny": 256, "pad": 0,
         "periodic": True, "dtype": "f64", "tuned": False},
        # an ordinary grid of odd sides with a padded pitch and a wide window
        {"name": "y_8th_odd_f32", "kind": "stencil2d", "stencil": "y_d2_8th", "nx": 3001, "ny": 2003, "pad": 7,
         "periodic": False, "dtype": "f32", "tuned": False},
        # the benchmark's stencil set on its large grid
        {"name": "set_8192_f64", "kind": "set", "n": 8192, "dtype": "f64", "tuned": True},
        # the nonlinear term on a large grid stored in 16 bits
        {"name": "lap_cubic_8192_bf16", "kind": "stencil2d", "stencil": "xy_lap_cubic", "nx": 8192, "ny": 8192,
         "pad": 0, "periodic": False, "dtype": "bf16", "tuned": True},
        # the benchmark's batch of uneven signals
        {"name": "ragged1d_65536_f32", "kind": "ragged1d", "count": 65536, "lo": 64, "hi": 4096, "periodic": True,
         "dtype": "f32"},
        # the benchmark's batch of uneven tridiagonal lines
        {"name": "tri_65536_f64", "kind": "solve", "geometry": "ragged", "bw": 1, "count": 65536, "lo": 64,
         "hi": 4096, "dtype": "f64", "tuned": True},
        # one implicit sweep along y on a rectangular grid
        {"name": "penta_cols_f64", "kind": "solve", "geometry": "cols", "bw": 2, "nx": 2051, "ny": 3000, "pad": 1,
         "dtype": "f64", "tuned": False},
        # a sample interval of a long physics run: steps, then its diagnostics
        {"name": "run_512_f64", "kind": "run", "nx": 512, "ny": 512, "steps": 20, "dtype": "f64", "tuned": True},
        # the Cahn-Hilliard configurations of the benchmark
        {"name": "ch_1024_f64", "kind": "ch", "nx": 1024, "ny": 1024, "steps": 10, "dtype": "f64", "tuned": True},
        {"name": "ch_4096_f64", "kind": "ch", "nx": 4096, "ny": 4096, "steps": 10, "dtype": "f64", "tuned": True},
        # many grids advanced together
        {"name": "ensemble_64_f32", "kind": "ensemble", "count": 64, "lo": 256, "hi": 1024, "steps": 10,
         "dtype": "f32", "tuned": True},
        # the advection term of a level-set step on a large grid
        {"name": "weno_8192_f64", "kind": "weno", "nx": 8192, "ny": 8192, "tuned": True},
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("stencil2d", "stencil2d", "stencil2d", "fn", "ragged1d", "ragged1d", "solve", "solve",
                       "solve", "run", "ch", "ch", "ensemble", "weno"))
    dtype = rng.choice(("f64", "f64", "f32", "bf16"))
    tuned = rng.random() < 0.5
    if kind == "stencil2d":
        return {"kind": kind, "stencil": rng.choice(sorted(STENCILS)), "nx": _log(rng, 64, 8192),
                "ny": _log(rng, 64, 8192), "pad": rng.choice((0, 0, 1, 8, 13)), "periodic": rng.random() < 0.5,
                "dtype": dtype, "tuned": tuned}
    if kind == "fn":
        return {"kind": kind, "nx": _log(rng, 64, 4096), "ny": _log(rng, 64, 4096), "dtype": dtype}
    if kind == "ragged1d":
        lo = _log(rng, 16, 512)
        return {"kind": kind, "count": _log(rng, 8, 65536), "lo": lo, "hi": _log(rng, 2 * lo, 4096),
                "periodic": rng.random() < 0.5, "dtype": dtype}
    if kind == "solve":
        geometry, bw = rng.choice(("ragged", "rows", "cols")), rng.choice((1, 2))
        if geometry == "ragged":
            lo = _log(rng, 16, 512)
            return {"kind": kind, "geometry": geometry, "bw": bw, "count": _log(rng, 8, 65536 // bw), "lo": lo,
                    "hi": _log(rng, 2 * lo, 4096), "dtype": dtype, "tuned": tuned}
        return {"kind": kind, "geometry": geometry, "bw": bw, "nx": _log(rng, 64, 8192), "ny": _log(rng, 64, 8192),
                "pad": rng.choice((0, 0, 1, 8)), "dtype": dtype, "tuned": tuned}
    if kind == "weno":
        return {"kind": kind, "nx": _log(rng, 64, 8192), "ny": _log(rng, 64, 8192), "tuned": tuned}
    if kind == "run":
        return {"kind": kind, "nx": 1 << rng.randint(6, 11), "ny": 1 << rng.randint(6, 11),
                "steps": rng.randint(1, 20), "dtype": "f64", "tuned": tuned}
    if kind == "ch":
        return {"kind": kind, "nx": _log(rng, 64, 4096), "ny": _log(rng, 64, 4096), "steps": rng.randint(1, 10),
                "dtype": dtype, "tuned": tuned}
    return {"kind": "ensemble", "count": _log(rng, 2, 64), "lo": 32 * rng.randint(2, 8),
            "hi": 32 * rng.randint(9, 32), "steps": rng.randint(1, 10), "dtype": rng.choice(("f32", "bf16")),
            "tuned": tuned}


# --- inputs ------------------------------------------------------------------

class _Plan:
    """A plan handle that is destroyed with its owner."""

    def __init__(self, handle, tune=False):
        self.handle = handle
        if tune:
            mxs.mxs_autotune(handle)

    def __del__(self):
        if self.handle is not None:
            mxs.mxs_destroy(self.handle)
            self.handle = None


def _uniform(shape, dtype, seed, amplitude=1.0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.empty(shape, dtype=torch.float64, device="cuda").uniform_(-amplitude, amplitude, generator=gen)
    return v.to(DTYPES[dtype])


def _lengths(case):
    """Uneven lengths: the shape of the batch belongs to the case, not to the seed."""
    n = np.random.default_rng(3).integers(case["lo"], case["hi"] + 1, case["count"], dtype=np.int64)
    return np.concatenate([[0], np.cumsum(n)])


def _sides(case):
    """Ensemble grid sides: multiples of 32 in [lo, hi]."""
    return [int(v) for v in np.random.default_rng(6).choice(np.arange(case["lo"], case["hi"] + 1, 32), case["count"])]


def _weights(name, scale=1.0):
    return [w * scale for w in STENCILS[name][3]]


def _penta(case):
    """I + a d_xxxx for the time steps of the Cahn-Hilliard runs, or circ(-1, 2.5, -1)."""
    return [2.5, -1.0] if case["bw"] == 1 else [1.0 + 6.0 * 20.0, -4.0 * 20.0, 20.0]


def _code(case):
    return mxs.dtype_code(DTYPES[case["dtype"]])


def _stencil_plan(name, nx, ny, ld, periodic, code, src, dst, tuned):
    direction, hx, hy, _, coe = STENCILS[name]
    return _Plan(mxs.mxs_create_2d(nx, ny, ld, {"X": mxs.MXS_X, "Y": mxs.MXS_Y, "XY": mxs.MXS_XY}[direction],
                                   mxs.MXS_P if periodic else mxs.MXS_NP, code, hx, hx, hy, hy, _weights(name), coe,
                                   src, dst), tuned)


def _grids(case):
    """(nx, ny, dx, dy, dt) of every grid of a Cahn-Hilliard case."""
    sizes = [(n, n) for n in _sides(case)] if case["kind"] == "ensemble" else [(case["nx"], case["ny"])]
    out = []
    for nx, ny in sizes:
        dx, dy = 2.0 * math.pi / nx, 2.0 * math.pi / ny
        out.append((nx, ny, dx, dy, 0.1 * min(dx, dy) ** 2))
    return out


def _ch_start(case, seed):
    """C^0 of every grid, stored back to back."""
    return _uniform(sum(g[0] * g[1] for g in _grids(case)), case["dtype"], seed, 0.1)


def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind}
    if kind == "stencil2d":
        ld = case["nx"] + case["pad"]
        src = _uniform((case["ny"], ld), case["dtype"], seed)
        dst = torch.zeros_like(src)
        state.update(src=src, out=dst, plan=_stencil_plan(case["stencil"], case["nx"], case["ny"], ld,
                                                          case["periodic"], _code(case), src, dst, case["tuned"]))
    elif kind == "set":
        n = case["n"]
        src = _uniform((n, n), case["dtype"], seed)
        state.update(src=src, out=[], plans=[])
        for name in SET:
            for periodic in (True, False):
                dst = torch.zeros_like(src)
                state["out"].append(dst)
                state["plans"].append(_stencil_plan(name, n, n, n, periodic, _code(case), src, dst, case["tuned"]))
    elif kind == "fn":
        nx, ny = case["nx"], case["ny"]
        both = _uniform((2, ny, nx), case["dtype"], seed)
        dst = torch.zeros_like(both[0])
        state.update(src=both, out=dst, plan=_Plan(mxs.mxs_create_2d_fn(
            nx, ny, nx, mxs.MXS_XY, mxs.MXS_P, _code(case), 1, 1, 1, 1, [both[0], both[1]], dst, [4.0], FN_SOURCE,
            "flux")))
    elif kind == "ragged1d":
        offsets = _lengths(case)
        src = _uniform(int(offsets[-1]), case["dtype"], seed)
        dst = torch.zeros_like(src)
        state.update(src=src, out=dst, plan=_Plan(mxs.mxs_create_1d_batch(
            offsets, mxs.MXS_P if case["periodic"] else mxs.MXS_NP, _code(case), 2, 2, D1_4TH, None, src, dst)))
    elif kind == "solve":
        if case["geometry"] == "ragged":
            offsets = _lengths(case)
            src = _uniform(int(offsets[-1]), case["dtype"], seed)
            shape = (mxs.MXS_LINES_RAGGED, 0, 0, 0, offsets)
        else:
            ld = case["nx"] + case["pad"]
            src = _uniform((case["ny"], ld), case["dtype"], seed)
            shape = (mxs.MXS_LINES_ROWS if case["geometry"] == "rows" else mxs.MXS_LINES_COLS, case["nx"],
                     case["ny"], ld, None)
        dst = torch.zeros_like(src)
        state.update(src=src, out=dst, plan=_Plan(mxs.mxs_create_cyclic_solve(
            case["bw"], _penta(case), *shape, _code(case), src, dst), case["tuned"]))
    elif kind == "weno":
        nx, ny = case["nx"], case["ny"]
        src = _uniform((3, ny, nx), "f64", seed)
        dst = torch.zeros_like(src[0])
        state.update(src=src, out=dst, plan=_Plan(mxs.mxs_create_weno_adv(
            nx, ny, nx, 1.0 / nx, 1.0 / ny, mxs.MXS_F64, src[0], src[1], src[2], dst), case["tuned"]))
    else:
        start = _ch_start(case, seed)
        levels = [start, start.clone(), torch.zeros_like(start)]
        grids = _grids(case)
        if kind == "ensemble":
            at = np.concatenate([[0], np.cumsum([g[0] * g[1] for g in grids])])
            nx, ny, dx, dy, dt = (list(v) for v in zip(*grids))
            plan = mxs.mxs_ch_ensemble_create(nx, ny, dx, dy, dt, D_COEF, GAMMA, _code(case),
                                              *[[v[at[k]:] for k in range(len(grids))] for v in levels])
        else:
            plan = mxs.mxs_ch_create(*grids[0], D_COEF, GAMMA, _code(case), *levels)
        state.update(levels=levels, steps=case["steps"], plan=_Plan(plan, case["tuned"]))
    return state


# --- one pass ----------------------------------------------------------------

def run(state):
    kind = state["kind"]
    if kind == "set":
        for plan in state["plans"]:
            mxs.mxs_compute(plan.handle)
        return state["out"]
    plan = state["plan"].handle
    if kind not in ("ch", "ensemble", "run"):
        mxs.mxs_compute(plan)
        return state["out"]
    mxs.mxs_ch_step(plan, state["steps"], True)
    prev, cur = mxs.mxs_ch_state(plan)
    by_address = {v.data_ptr(): v for v in state["levels"]}
    out = {"prev": by_address[prev], "cur": by_address[cur]}
    if kind == "run":
        out["mass"] = mxs.mxs_ch_mass(plan)[0]
        out["s"], out["k1"] = mxs.mxs_ch_coarsening(plan)
    return out


# --- work --------------------------------------------------------------------

def _points(case):
    if case["kind"] in ("stencil2d", "fn", "weno"):
        return case["nx"] * case["ny"]
    if case["kind"] == "set":
        return case["n"] ** 2
    if case["kind"] == "ragged1d" or case.get("geometry") == "ragged":
        return int(_lengths(case)[-1])
    if case["kind"] == "solve":
        return case["nx"] * case["ny"]
    return sum(g[0] * g[1] for g in _grids(case))


def _stencil_flops(name):
    _, _, _, weights, coe = STENCILS[name]
    return 2 * sum(1 for w in weights if w != 0.0) + (2 * len(coe) if coe else 0)


def work(case):
    kind, n = case["kind"], _points(case)
    if kind == "stencil2d":
        return {"bytes": 2 * n * WORD[case["dtype"]], "flops": n * _stencil_flops(case["stencil"])}
    if kind == "set":
        # eight calls, each of which reads the grid and writes its output
        return {"bytes": 16 * n * WORD[case["dtype"]], "flops": 2 * n * sum(_stencil_flops(s) for s in SET)}
    if kind == "fn":
        return {"bytes": 3 * n * WORD[case["dtype"]], "flops": 7 * n}
    if kind == "ragged1d":
        return {"bytes": 2 * n * WORD[case["dtype"]], "flops": 8 * n}
    if kind == "solve":
        return {"bytes": 2 * n * WORD[case["dtype"]], "flops": n * (4 * case["bw"] + 1)}
    if kind == "weno":
        return {"bytes": 4 * n * 8, "flops": 150 * n}
    # one step reads C^{n-1} and C^n and writes C^{n+1}: 13- and 5-point
    # windows, the nonlinear term and two pentadiagonal solves per point
    per_step = {"bytes": 3 * n * WORD[case["dtype"]], "flops": 64 * n}
    total = {k: v * case["steps"] for k, v in per_step.items()}
    if kind == "run":
        # mass and diagnostics read the state once; two real FFTs' operations
        total["bytes"] += n * WORD[case["dtype"]]
        total["flops"] += int(2.5 * n * math.log2(n)) + 10 * n
    return total


# --- the same results in 64 bits ----------------------------------------------

def _shifted(u, a, b):
    """u[j + b][i + a] with wrap."""
    return torch.roll(u, (-b, -a), (0, 1))


def _stencil_exact(u, name, periodic, nx):
    direction, hx, hy, weights, coe = STENCILS[name]
    c = u[:, :nx].double()
    if coe:
        f = torch.zeros_like(c)
        for m in reversed(coe):
            f = f * c + m
        c = f
    out = torch.zeros_like(c)
    for k, w in enumerate(weights):
        if w != 0.0:
            out += w * _shifted(c, k % (2 * hx + 1) - hx, k // (2 * hx + 1) - hy)
    ny = c.shape[0]
    whole = torch.zeros(u.shape, dtype=torch.float64, device=u.device)
    if periodic:
        whole[:, :nx] = out
    else:
        whole[hy:ny - hy, hx:nx - hx] = out[hy:ny - hy, hx:nx - hx]
    return whole


def _cyclic_exact(r, coef, dim):
    """circ(coef) x = r along `dim`, by the discrete Fourier transform."""
    n = r.shape[dim]
    theta = torch.arange(n // 2 + 1, dtype=torch.float64, device=r.device) * (2.0 * math.pi / n)
    symbol = coef[0] + sum(2.0 * c * torch.cos((d + 1) * theta) for d, c in enumerate(coef[1:]))
    shape = [1, 1]
    shape[dim] = n // 2 + 1
    return torch.fft.irfft(torch.fft.rfft(r, dim=dim) / symbol.reshape(shape), n=n, dim=dim)


def _ragged_exact(r, coef, offsets):
    """circ(coef) x = r on every line: the circulant is K prod (1 - p S)(1 - p S^-1)
    over the roots p of its symbol inside the unit circle, and the inverse of
    each factor is the product of (1 + (p S)^(2^k))."""
    bw = len(coef) - 1
    roots = np.roots(np.concatenate([coef[::-1], coef[1:]]))
    inside = sorted(roots[np.abs(roots) < 1.0], key=lambda p: (p.real, p.imag))
    scale = coef[bw] / np.prod([-p for p in inside])
    lengths = torch.as_tensor(np.diff(offsets), device=r.device)
    start = torch.repeat_interleave(torch.as_tensor(offsets[:-1], device=r.device), lengths)
    n = torch.repeat_interleave(lengths, lengths)
    pos = torch.arange(r.numel(), device=r.device) - start
    real = all(abs(p.imag) < 1e-14 for p in inside)
    x = r.clone() if real else r.to(torch.complex128)
    for p in inside:
        for sign in (1, -1):
            k, q = 1, float(p.real) if real else complex(p)
            while abs(q) > 1e-20:
                x = x + q * x[start + torch.remainder(pos - sign * k, n)]
                k, q = 2 * k, q * q
    return (x if real else x.real) / float(np.real(scale))


def _weno_derivative(v):
    """Fifth-order Hamilton-Jacobi WENO from five one-sided differences."""
    a, b, c, d, e = v
    p1 = a / 3 - 7 * b / 6 + 11 * c / 6
    p2 = -b / 6 + 5 * c / 6 + d / 3
    p3 = c / 3 + 5 * d / 6 - e / 6
    s1 = 13 / 12 * (a - 2 * b + c) ** 2 + (a - 4 * b + 3 * c) ** 2 / 4
    s2 = 13 / 12 * (b - 2 * c + d) ** 2 + (b - d) ** 2 / 4
    s3 = 13 / 12 * (c - 2 * d + e) ** 2 + (3 * c - 4 * d + e) ** 2 / 4
    eps = 1e-6 * torch.maximum(torch.maximum(torch.maximum(a * a, b * b), torch.maximum(c * c, d * d)), e * e) + 1e-99
    w1, w2, w3 = 0.1 / (s1 + eps) ** 2, 0.6 / (s2 + eps) ** 2, 0.3 / (s3 + eps) ** 2
    return (w1 * p1 + w2 * p2 + w3 * p3) / (w1 + w2 + w3)


def _weno_exact(phi, u, v, dx, dy):
    out = torch.zeros_like(phi)
    for vel, h, dim in ((u, dx, 1), (v, dy, 0)):
        back = (phi - torch.roll(phi, 1, dim)) / h          # backward difference at i
        at = lambda k: torch.roll(back, -k, dim)            # noqa: E731  the one at i + k
        minus = _weno_derivative([at(k) for k in (-2, -1, 0, 1, 2)])
        plus = _weno_derivative([at(k) for k in (3, 2, 1, 0, -1)])
        out += vel * torch.where(vel > 0, minus, plus)
    return out


def _ch_exact(c0, grid, steps):
    nx, ny, dx, dy, dt = grid

    def lap(f):
        return ((_shifted(f, 1, 0) - f) - (f - _shifted(f, -1, 0))) / dx ** 2 + \
               ((_shifted(f, 0, 1) - f) - (f - _shifted(f, 0, -1))) / dy ** 2

    def solve(r, h, dim):
        n = r.shape[dim]
        theta = torch.arange(n // 2 + 1, dtype=torch.float64, device=r.device) * (math.pi / n)
        shape = [1, 1]
        shape[dim] = n // 2 + 1
        symbol = 1.0 + 2.0 / 3.0 * D_COEF * GAMMA * dt * (2.0 * torch.sin(theta) / h) ** 4
        return torch.fft.irfft(torch.fft.rfft(r, dim=dim) / symbol.reshape(shape), n=n, dim=dim)

    prev, cur = c0.clone(), c0
    for _ in range(steps):
        bar = 2.0 * cur - prev
        r = -2.0 / 3.0 * (cur - prev) - 2.0 / 3.0 * D_COEF * GAMMA * dt * lap(lap(bar)) \
            + 2.0 / 3.0 * D_COEF * dt * lap(cur ** 3 - cur)
        prev, cur = cur, bar + solve(solve(r, dx, 1), dy, 0)
    return prev, cur


def _diagnostics_exact(c, dx, dy):
    ny, nx = c.shape
    ax = torch.where(torch.arange(nx, device=c.device) % 2 == 0, 2.0 / 3.0, 4.0 / 3.0).double()
    ay = torch.where(torch.arange(ny, device=c.device) % 2 == 0, 2.0 / 3.0, 4.0 / 3.0).double()
    mean = float((ay[:, None] * ax[None, :] * c * c).sum()) / (nx * ny)
    power = torch.fft.fft2(c).abs() ** 2
    kx = 2.0 * math.pi / (nx * dx) * torch.fft.fftfreq(nx, 1.0 / nx, dtype=torch.float64, device=c.device)
    ky = 2.0 * math.pi / (ny * dy) * torch.fft.fftfreq(ny, 1.0 / ny, dtype=torch.float64, device=c.device)
    k = torch.sqrt(kx[None, :] ** 2 + ky[:, None] ** 2)
    power[0, 0], k[0, 0] = 0.0, 1.0
    return float(c.sum()), 1.0 / (1.0 - mean), float(power.sum() / (power / k).sum())


def exact(case, seed):
    kind = case["kind"]
    if kind == "stencil2d":
        src = _uniform((case["ny"], case["nx"] + case["pad"]), case["dtype"], seed)
        return _stencil_exact(src, case["stencil"], case["periodic"], case["nx"])
    if kind == "set":
        src = _uniform((case["n"], case["n"]), case["dtype"], seed)
        return [_stencil_exact(src, name, periodic, case["n"]) for name in SET for periodic in (True, False)]
    if kind == "fn":
        u, v = _uniform((2, case["ny"], case["nx"]), case["dtype"], seed).double()
        lap = _shifted(u, 0, -1) + _shifted(u, -1, 0) + _shifted(u, 1, 0) + _shifted(u, 0, 1) - 4.0 * u
        return lap * v
    if kind == "ragged1d":
        offsets = _lengths(case)
        u = _uniform(int(offsets[-1]), case["dtype"], seed).double()
        lengths = torch.as_tensor(np.diff(offsets), device=u.device)
        start = torch.repeat_interleave(torch.as_tensor(offsets[:-1], device=u.device), lengths)
        n = torch.repeat_interleave(lengths, lengths)
        pos = torch.arange(u.numel(), device=u.device) - start
        out = torch.zeros_like(u)
        for k, w in enumerate(D1_4TH):
            if w != 0.0:
                out += w * u[start + torch.remainder(pos + k - 2, n)]
        return out if case["periodic"] else torch.where((pos >= 2) & (pos < n - 2), out, 0.0)
    if kind == "solve":
        if case["geometry"] == "ragged":
            offsets = _lengths(case)
            return _ragged_exact(_uniform(int(offsets[-1]), case["dtype"], seed).double(), _penta(case), offsets)
        src = _uniform((case["ny"], case["nx"] + case["pad"]), case["dtype"], seed).double()
        whole = torch.zeros_like(src)
        whole[:, :case["nx"]] = _cyclic_exact(src[:, :case["nx"]].contiguous(), _penta(case),
                                              1 if case["geometry"] == "rows" else 0)
        return whole
    if kind == "weno":
        phi, u, v = _uniform((3, case["ny"], case["nx"]), "f64", seed)
        return _weno_exact(phi, u, v, 1.0 / case["nx"], 1.0 / case["ny"])
    grids, start = _grids(case), _ch_start(case, seed).double()
    prev, cur, at = [], [], 0
    for g in grids:
        p, c = _ch_exact(start[at:at + g[0] * g[1]].reshape(g[1], g[0]), g, case["steps"])
        prev.append(p.reshape(-1))
        cur.append(c.reshape(-1))
        at += g[0] * g[1]
    out = {"prev": torch.cat(prev), "cur": torch.cat(cur)}
    if kind == "run":
        g = grids[0]
        out["mass"], out["s"], out["k1"] = _diagnostics_exact(out["cur"].reshape(g[1], g[0]), g[2], g[3])
    return out
