"""Performance cases: what users of this package have it compute.

Each case is one pass through the public entry points with inputs resident on
the GPU, as in an imaging run: predictions of a component model (direct sum,
wavelet tree, FFT + degridding), residual images and gradients, a batched
major cycle over several channels, and a whole clean run.  listed() holds fixed
cases, draw() gives more of the same ranges, prepare() makes a case's inputs
from a seed, run() is the pass, work() what it cannot do without and exact()
the same outputs in plain 64-bit torch / numpy.

Rows are Earth-rotation tracks of random arrays (all antenna pairs, time
major, u, v, w in wavelengths); components are Gaussian blobs plus a uniform
field with lognormal fluxes, or sphere pixels for the tree cases.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1909_03956_amd as swv
from paper_1909_03956_amd import autograd

LAT = math.radians(34.08)
C_LIGHT = 299792458.0
# antennas, disk radius (m), declination (deg), frequency (Hz), hours: a large
# L-band array, and a 27-antenna array at 10 MHz (wide fields, strong w term)
ARRAYS = {"wide": (256, 20e3, 30.0, 1.4e9, 8.0),
          "mid": (64, 5e3, 45.0, 1.4e9, 2.0),
          "low": (27, 1.7e3, 45.0, 1.0e7, 1.0)}
LOW_CELL = math.radians(42.0 + 40.0 / 60.0) / 256.0


# ------------------------------------------------------------------ cases --
def listed():
    return [
        # one integration of a 27-antenna array against a handful of sources:
        # calibration-style calls, where launches and latency are everything
        {"name": "snapshot_7", "kind": "direct", "array": "low", "rows": 351, "comps": 7,
         "field": 20.0, "prec": "fp64", "sign": -1},
        # two hours of a 64-antenna array, 200 components
        {"name": "direct_120k_200", "kind": "direct", "array": "mid", "rows": 120960,
         "comps": 200, "field": 2.0, "prec": "fp64", "sign": -1},
        # a full eight-hour observation of 256 antennas against a deep model
        {"name": "direct_8M_2000", "kind": "direct", "array": "wide", "rows": 8355840,
         "comps": 2000, "field": 4.0, "prec": "fp64", "sign": -1},
        # the FP32-compensated form on one odd-sized hour
        {"name": "direct_f32c_1M_1999", "kind": "direct", "array": "wide", "rows": 1263601,
         "comps": 1999, "field": 3.0, "prec": "f32c", "sign": 1},
        # wavelet prediction at the measured level of a wide field
        {"name": "tree_J10_8M", "kind": "tree", "array": "wide", "rows": 8355840, "J": 10,
         "level": 5, "comps": 2000, "prec": "fp64"},
        # deep tree over a short list of distinct components
        {"name": "tree_J20_1M", "kind": "tree", "array": "low", "rows": 1263600, "J": 20,
         "level": 3, "comps": 140, "prec": "fp64"},
        # residual image on the sphere pixels of a 4 degree disk (and its size)
        {"name": "adjoint_8M_955", "kind": "adjoint", "array": "wide", "rows": 8355840,
         "pixels": 955, "field": 8.0, "prec": "fp64"},
        # residual image on a regular grid in the FP32-compensated form
        {"name": "image_f32c_256", "kind": "image", "array": "low", "rows": 176904, "nx": 256,
         "ny": 256, "prec": "f32c"},
        # one optimisation step through autograd: prediction, then gradients
        {"name": "autograd_261k_1000", "kind": "autograd", "array": "wide", "rows": 261120,
         "comps": 1000, "field": 4.0},
        # a major cycle over four channels of uneven size
        {"name": "cycle_4_channels", "kind": "cycle", "array": "wide", "rows": 195840,
         "channels": 4, "comps": 600, "pixels": 501},
        # a whole wide-field clean run: beam, images, minor cycles, tree model
        {"name": "clean_256_2x300", "kind": "clean", "array": "low", "rows": 176904, "nx": 256,
         "ny": 256, "J": 11, "minor": 300, "major": 2},
        # the conventional predictor on the same field
        {"name": "degrid_256_W10", "kind": "degrid", "array": "low", "rows": 707616, "nx": 256,
         "ny": 256, "support": 10, "comps": 140},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["direct", "direct", "direct", "tree", "tree", "adjoint", "adjoint", "image",
                       "autograd", "cycle", "clean", "degrid"])
    if kind == "direct":
        rows, comps = _log(rng, 351, 8355840), _log(rng, 1, 20000)
        comps = max(1, min(comps, int(1.6e10 / rows)))
        return {"kind": kind, "array": rng.choice(["wide", "mid", "low"]), "rows": rows,
                "comps": comps, "field": rng.uniform(1.0, 10.0),
                "prec": rng.choice(["fp64", "fp64", "f32c"]), "sign": rng.choice([-1, 1])}
    if kind == "tree":
        deep = rng.random() < 0.5
        J = rng.randint(11, 25) if deep else rng.randint(6, 10)
        comps = _log(rng, 5, 140) if deep else _log(rng, 50, 2000)
        return {"kind": kind, "array": "low" if deep else "wide",
                "rows": _log(rng, 1000, 1200000 if deep else 8000000), "J": J,
                "level": 3 if deep else rng.randint(3, 5), "comps": comps,
                "prec": rng.choice(["fp64", "f32c"])}
    if kind == "adjoint":
        rows, pixels = _log(rng, 1000, 8000000), _log(rng, 20, 60000)
        pixels = max(1, min(pixels, int(7.5e9 / rows)))
        return {"kind": kind, "array": rng.choice(["wide", "mid"]), "rows": rows,
                "pixels": pixels, "field": rng.uniform(2.0, 8.0),
                "prec": rng.choice(["fp64", "f32c"])}
    if kind == "image":
        nx, ny = _log(rng, 20, 300), _log(rng, 20, 300)
        return {"kind": kind, "array": "low", "rows": min(_log(rng, 2000, 170000), 11 * 10 ** 9 // (nx * ny)),
                "nx": nx, "ny": ny, "prec": rng.choice(["fp64", "f32c"])}
    if kind == "autograd":
        rows = _log(rng, 5000, 250000)
        return {"kind": kind, "array": rng.choice(["wide", "mid"]), "rows": rows,
                "comps": _log(rng, 10, 1000), "field": rng.uniform(1.0, 4.0)}
    if kind == "cycle":
        return {"kind": kind, "array": "wide", "rows": _log(rng, 10000, 150000),
                "channels": rng.randint(2, 4), "comps": _log(rng, 50, 600),
                "pixels": _log(rng, 50, 500)}
    if kind == "clean":
        n = rng.randint(33, 200)
        return {"kind": kind, "array": "low", "rows": _log(rng, 8424, 150000), "nx": n,
                "ny": n + rng.randint(-3, 3), "J": rng.randint(9, 12),
                "minor": rng.randint(20, 200), "major": rng.randint(1, 2)}
    n = rng.randint(64, 256)
    return {"kind": kind, "array": "low", "rows": _log(rng, 20000, 700000), "nx": n,
            "ny": rng.randint(64, 256), "support": rng.choice([6, 8, 10]), "comps": _log(rng, 10, 140)}


# ----------------------------------------------------------------- inputs --
def _gen(seed, salt):
    return np.random.default_rng([int(seed), salt])


def _tracks(array, rows, seed, salt=1, scale=1.0):
    """u, v, w of the first `rows` (time, baseline) rows on the GPU."""
    n, radius, dec, freq, hours = ARRAYS[array]
    rng = _gen(seed, salt)
    r, th = radius * np.sqrt(rng.random(n)), 2 * np.pi * rng.random(n)
    e, no, up = r * np.cos(th), r * np.sin(th), 10.0 * rng.standard_normal(n)
    p, q = np.triu_indices(n, 1)
    e, no, up = e[q] - e[p], no[q] - no[p], up[q] - up[p]
    X = -no * math.sin(LAT) + up * math.cos(LAT)
    Z = no * math.cos(LAT) + up * math.sin(LAT)
    to = lambda a: torch.as_tensor(a * (freq * scale / C_LIGHT), device="cuda")[None, :]
    X, Y, Z = to(X), to(e), to(Z)
    nt = -(-rows // len(p))
    H = ((torch.arange(nt, dtype=torch.float64, device="cuda") + 0.5) / nt - 0.5)[:, None]
    H = H * (hours * 2.0 * math.pi / 23.934469)
    s, c, sd, cd = torch.sin(H), torch.cos(H), math.sin(math.radians(dec)), math.cos(math.radians(dec))
    out = (s * X + c * Y, -sd * c * X + sd * s * Y + cd * Z, cd * c * X - cd * s * Y + sd * Z)
    return tuple(t.reshape(-1)[:rows].contiguous() for t in out)


def _model(comps, field_deg, seed, salt=2):
    """(l, m, flux): 70 % in five blobs of 0.1 degrees, the rest uniform."""
    rng = _gen(seed, salt)
    h = math.sin(math.radians(0.5 * field_deg))
    nb = int(0.7 * comps) if comps >= 20 else 0
    cen = rng.uniform(-0.75 * h, 0.75 * h, (5, 2))
    lm = np.concatenate([cen[rng.integers(0, 5, nb)] + rng.normal(0, math.radians(0.1), (nb, 2)),
                         rng.uniform(-h, h, (comps - nb, 2))])
    return lm[:, 0].copy(), lm[:, 1].copy(), rng.lognormal(-3.0, 1.0, comps)


def _dev(*arrays):
    return tuple(torch.as_tensor(np.ascontiguousarray(a), device="cuda") for a in arrays)


def _nm1(l, m):
    l, m = np.asarray(l, np.longdouble), np.asarray(m, np.longdouble)
    r2 = l * l + m * m
    return (-r2 / (1 + np.sqrt(1 - r2))).astype(np.float64)


def _noise(n, seed, sigma=1.0):
    g = torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 62))
    return torch.complex(*(sigma * torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
                           for _ in range(2)))


def _pixels(case, seed):
    """Nested sphere pixels of the tree cases: blobs and single pixels under one
    pixel of a coarser level; the phase centre is that pixel's centre."""
    rng = _gen(seed, 3)
    J, lv, n = case["J"], min(case["level"], case["J"]), case["comps"]
    top = int(rng.integers(4 * 4 ** (lv - 1), 8 * 4 ** (lv - 1)))      # equatorial faces
    span = 4 ** (J - lv)
    blob = min(span, 256)
    nb = int(0.7 * n) if case["array"] == "wide" else 0
    cen = rng.integers(0, span // blob, 5)
    pix = np.concatenate([cen[rng.integers(0, 5, nb)] * blob + rng.integers(0, blob, nb),
                          rng.integers(0, span, n - nb)]) + top * span
    x = _centres(lv, np.array([top]))
    ra, dec = float(np.arctan2(x[1], x[0])[0]), float(np.arcsin(x[2])[0])
    return pix.astype(np.int64), rng.lognormal(-3.0, 1.0, n), ra, dec


def _centres(level, pix):
    """Unit vectors (long double) of HEALPix nested pixels at nside 2^(level-1)."""
    ld = np.longdouble
    nside = 1 << (level - 1)
    face, k = pix >> (2 * (level - 1)), pix & (nside * nside - 1)
    ix, iy = np.zeros_like(pix), np.zeros_like(pix)
    for b in range(level - 1):
        ix |= ((k >> (2 * b)) & 1) << b
        iy |= ((k >> (2 * b + 1)) & 1) << b
    ring_of = np.array([2, 2, 2, 2, 3, 3, 3, 3, 4, 4, 4, 4])[face]
    phi_of = np.array([1, 3, 5, 7, 0, 2, 4, 6, 1, 3, 5, 7])[face]
    jr = ring_of * nside - ix - iy - 1
    nr = np.where(jr < nside, jr, np.where(jr > 3 * nside, 4 * nside - jr, nside)).astype(ld)
    cap = nr * nr / (3 * ld(nside) * nside)
    z = np.where(jr < nside, 1 - cap, np.where(jr > 3 * nside, cap - 1,
                                               ld(2) * (2 * nside - jr) / (3 * ld(nside))))
    polar = (jr < nside) | (jr > 3 * nside)
    st = np.where(polar, np.sqrt(cap * (2 - cap)), np.sqrt(np.maximum(1 - z * z, 0)))
    quarter = ld("0.785398163397448309615660845819875721")
    phi = quarter * (phi_of * nr + (ix - iy)) / nr
    return np.stack([st * np.cos(phi), st * np.sin(phi), z])


def _project(x, ra, dec):
    """(l, m, n - 1) of unit vectors about the phase centre, rounded to doubles."""
    ld = np.longdouble
    sa, ca, sd, cd = np.sin(ld(ra)), np.cos(ld(ra)), np.sin(ld(dec)), np.cos(ld(dec))
    l = -sa * x[0] + ca * x[1]
    m = -sd * ca * x[0] - sd * sa * x[1] + cd * x[2]
    return l.astype(np.float64), m.astype(np.float64), _nm1(l, m)


def _grid(nx, ny, cx, cy):
    l, m = (np.arange(nx) - cx) * LOW_CELL, (np.arange(ny) - cy) * LOW_CELL
    return tuple(a.ravel() for a in np.meshgrid(l, m))


def _sky(case, seed, u, v, w):
    """Noisy visibilities of seven 1 Jy sources over 30 degrees."""
    l, m = _gen(seed, 4).uniform(-0.25, 0.25, (2, 7))
    V = _noise(u.numel(), seed, 0.01)
    for a, b, c in zip(l, m, _nm1(l, m)):
        V += torch.polar(torch.ones_like(u), -2 * math.pi * (u * a + v * b + w * c))
    return V


def _degrid_image(case, seed):
    rng = _gen(seed, 5)
    nx, ny = case["nx"], case["ny"]
    img = np.zeros((ny, nx))
    iy, ix = rng.integers(ny // 6, ny - ny // 6, case["comps"]), rng.integers(nx // 6, nx - nx // 6, case["comps"])
    np.add.at(img, (iy, ix), rng.lognormal(-3.0, 1.0, case["comps"]))
    return img


def _channels(case, seed):
    """Per channel: route, tracks, model, observed visibilities, pixels."""
    out = []
    for k in range(case["channels"]):
        rows = max(300, int(case["rows"] * (1.0 - 0.13 * k)) - 7 * k)
        uvw = _tracks(case["array"], rows, seed, 10 + k, 1.0 + 0.1 * k)
        d = {"rows": rows, "uvw": uvw, "route": "direct" if k % 2 == 0 else "tree",
             "obs": _noise(rows, seed * 8 + k, 1.0)}
        pl, pm, _ = _model(case["pixels"], 6.0, seed, 30 + k)
        d["pix"] = (pl, pm, _nm1(pl, pm))
        if d["route"] == "direct":
            d["model"] = _model(case["comps"] + k, 4.0, seed, 20 + k)
        else:
            d["tree"] = _pixels({"J": 8 + k % 2, "level": 4, "comps": case["comps"], "array": "wide"},
                                seed * 8 + k)
            d["J"] = 8 + k % 2
        out.append(d)
    return out


# --------------------------------------------------------- prepare and run --
def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "cycle":
        spec = _channels(case, seed)
        inst = []
        for k, d in enumerate(spec):
            u, v, w = d["uvw"]
            e = {"route": d["route"], "u": u, "v": v, "w": w, "vis_obs": d["obs"],
                 "inv_sigma2": 1.0, "pixels": _dev(*d["pix"]), "comp_cap": case["comps"] + k}
            if d["route"] == "direct":
                e["grads"] = True
            else:
                e["tree_level_cap"] = 9
            inst.append(e)
        cy = swv.MajorCycle(inst)
        for k, d in enumerate(spec):
            if d["route"] == "direct":
                cy.set_components(k, *_dev(*d["model"]))
            else:
                pix, flux, ra, dec = d["tree"]
                cy.set_tree(k, swv.Tree.from_pixels(d["J"], ra, dec, pix, flux))
        st["cycle"] = cy
        return st
    u, v, w = st["uvw"] = _tracks(case["array"], case["rows"], seed)
    if kind in ("direct", "autograd"):
        st["model"] = _dev(*_model(case["comps"], case["field"], seed))
        if kind == "autograd":
            st["model"] = tuple(t.requires_grad_(True) for t in st["model"])
            st["obs"] = _noise(case["rows"], seed)
    elif kind == "tree":
        pix, flux, ra, dec = _pixels(case, seed)
        st["tree"] = swv.Tree.from_pixels(case["J"], ra, dec, pix, flux)
    elif kind == "adjoint":
        l, m, _ = _model(case["pixels"], case["field"], seed, 6)
        st["pix"] = _dev(l, m, _nm1(l, m))
        st["y"] = _noise(case["rows"], seed)
    elif kind in ("image", "clean"):
        st["y"] = _sky(case, seed, u, v, w)
    elif kind == "degrid":
        st["image"] = _dev(_degrid_image(case, seed))[0]
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "cycle":
        st["cycle"].run()
        return [[o["vis_model"], o["resid"], o["chi2"], o["image"]] + list(o.get("grads", []))
                for o in st["cycle"].out]
    u, v, w = st["uvw"]
    if kind == "direct":
        return swv.predict_direct(u, v, w, *st["model"], sign=case["sign"], prec=case["prec"])
    if kind == "tree":
        return st["tree"].predict(u, v, w, prec=case["prec"])
    if kind == "adjoint":
        return swv.adjoint(u, v, w, st["y"], *st["pix"], prec=case["prec"])
    if kind == "image":
        return swv.dirty_image(u, v, w, st["y"], case["nx"], case["ny"], LOW_CELL, prec=case["prec"])
    if kind == "autograd":
        l, m, flux = st["model"]
        V = autograd.predict_direct(u, v, w, l, m, flux)
        return [V.detach()] + list(torch.autograd.grad(V, (l, m, flux), V.detach() - st["obs"]))
    if kind == "clean":
        d = swv.wavelet_clean(u, v, w, st["y"], case["nx"], case["ny"], LOW_CELL, case["J"],
                              math.pi, math.radians(ARRAYS[case["array"]][2]), gain=0.1,
                              minor_iter=case["minor"], n_major=case["major"])
        return [d["beam"], d["residual"], d["vis_model"], d["pix"], d["val"]]
    return swv.predict_degrid(st["image"], u, v, w, LOW_CELL, support=case["support"])[0]


# ------------------------------------------------------------------- work --
# Operations one (row, term) cannot do without: phase 5, its reduction 1, a
# sine and a cosine 2; then the multiply-adds of what is summed.
PHASOR = 8


def work(case):
    kind, N = case["kind"], case.get("rows", 0)
    wide = 8 if case.get("prec") == "f32c" else 16
    if kind == "direct":
        return {"bytes": N * (24 + wide) + 24 * case["comps"], "flops": N * case["comps"] * (PHASOR + 4)}
    if kind == "tree":
        leaves = len(set(_pixels(case, 0)[0].tolist()))
        return {"bytes": N * (24 + wide) + 24 * leaves, "flops": N * leaves * (PHASOR + 4)}
    if kind == "adjoint":
        return {"bytes": N * 40 + 40 * case["pixels"], "flops": N * case["pixels"] * (PHASOR + 8)}
    if kind == "image":
        P = case["nx"] * case["ny"]
        return {"bytes": N * 40 + 8 * P, "flops": N * P * (PHASOR + 4)}
    if kind == "autograd":
        return {"bytes": N * (40 + 16 + 40) + 72 * case["comps"],
                "flops": N * case["comps"] * (2 * PHASOR + 4 + 14)}
    if kind == "cycle":
        b = f = 0
        for k in range(case["channels"]):
            n = max(300, int(N * (1.0 - 0.13 * k)) - 7 * k)
            b += n * (24 + 16 + 16 + 16 + 16) + 40 * case["pixels"]
            f += n * (case["comps"] * (PHASOR + 4) + case["pixels"] * (PHASOR + 8))
            if k % 2 == 0:
                f += n * case["comps"] * (PHASOR + 14)
        return {"bytes": b, "flops": f}
    if kind == "clean":
        P, B = case["nx"] * case["ny"], (2 * case["nx"] - 1) * (2 * case["ny"] - 1)
        it = case["minor"] * case["major"]
        return {"bytes": N * 40 * (2 + 2 * case["major"]) + 24 * P * it,
                "flops": N * (B + P * (1 + case["major"])) * (PHASOR + 4) + 3 * P * it}
    T = case["support"]
    return {"bytes": N * 40 + 8 * case["nx"] * case["ny"],
            "flops": N * (4 * T ** 3 + 60 * T) + 0.0}


# ------------------------------------------------------------------ exact --
def _split(a):
    c = 134217729.0 * a
    hi = c - (c - a)
    return hi, a - hi


def _turns(rows, terms):
    """u l + v m + w (n - 1) modulo 1 of every (row, term): each product with its
    rounding error, so that only the reduced sum rounds."""
    r = None
    for a, b in zip(rows, terms):
        (ah, al), (bh, bl) = _split(a[:, None]), _split(b[None, :])
        p = a[:, None] * b[None, :]
        e = ((ah * bh - p) + ah * bl + al * bh) + al * bl
        p -= torch.round(p)
        p += e
        r = p if r is None else r.add_(p)
    return r.sub_(torch.round(r)).mul_(2 * math.pi)


def _blocks(n, terms):
    step = max(1, (1 << 24) // max(1, terms))
    return range(0, n, step), step


def _sum_terms(uvw, lmn, amp, sign=-1):
    """V_j = sum_k amp_k exp(sign 2 pi i phi_jk)."""
    n, K = uvw[0].numel(), lmn[0].numel()
    V = torch.zeros(n, dtype=torch.complex128, device="cuda")
    starts, step = _blocks(n, K)
    for i in starts:
        x = _turns([t[i:i + step] for t in uvw], lmn)
        V[i:i + step] = torch.complex(torch.cos(x) @ amp, sign * (torch.sin(x) @ amp))
    return V


def _sum_rows(uvw, y, lmn, sign=-1):
    """x_p = sum_j conj(e_jp) y_j."""
    n, P = uvw[0].numel(), lmn[0].numel()
    out = torch.zeros(2, P, dtype=torch.float64, device="cuda")
    starts, step = _blocks(n, P)
    yr, yi = y.real.contiguous(), y.imag.contiguous()
    for i in starts:
        x = _turns([t[i:i + step] for t in uvw], lmn)
        a, b = yr[i:i + step], yi[i:i + step]
        c = torch.cos(x)
        s = torch.sin(x).mul_(sign)
        out[0] += a @ c + b @ s
        out[1] += b @ c - a @ s
    return torch.complex(out[0], out[1])


def _gradients(uvw, y, l, m, flux, sign=-1):
    """Gradients of Re sum_j conj(y_j) V_j with respect to (l, m, flux)."""
    lmn = _dev(l, m, _nm1(l, m))
    n, K = uvw[0].numel(), len(l)
    S = torch.zeros(4, K, dtype=torch.float64, device="cuda")
    starts, step = _blocks(n, K)
    yr, yi = y.real.contiguous(), y.imag.contiguous()
    for i in starts:
        rows = [t[i:i + step] for t in uvw]
        x = _turns(rows, lmn)
        a, b = yr[i:i + step], yi[i:i + step]
        c = torch.cos(x)
        s = torch.sin(x).mul_(sign)
        S[0] += a @ c + b @ s
        for q, t in enumerate(rows):
            S[1 + q] += (a * t) @ s - (b * t) @ c
    I, L, M = _dev(flux, l, m)
    f = -I * sign * 2 * math.pi
    nn = 1.0 + lmn[2]
    return [f * (S[1] - L / nn * S[3]), f * (S[2] - M / nn * S[3]), S[0]]


def exact(case, seed):
    kind = case["kind"]
    if kind == "clean":
        return None
    if kind == "cycle":
        out = []
        for d in _channels(case, seed):
            if d["route"] == "direct":
                l, m, flux = d["model"]
                lmn = (l, m, _nm1(l, m))
            else:
                pix, flux, ra, dec = d["tree"]
                lmn = _project(_centres(d["J"], pix), ra, dec)
            V = _sum_terms(d["uvw"], _dev(*lmn), _dev(flux)[0])
            r = d["obs"] - V
            o = [V, r, (r.real ** 2 + r.imag ** 2).sum().reshape(1),
                 _sum_rows(d["uvw"], r, _dev(*d["pix"]))]
            if d["route"] == "direct":
                gl, gm, gf = _gradients(d["uvw"], -2.0 * r, l, m, flux)
                o += [gf, gl, gm]
            out.append(o)
        return out
    uvw = _tracks(case["array"], case["rows"], seed)
    if kind == "direct":
        l, m, flux = _model(case["comps"], case["field"], seed)
        V = _sum_terms(uvw, _dev(l, m, _nm1(l, m)), _dev(flux)[0], case["sign"])
        return V.to(torch.complex64) if case["prec"] == "f32c" else V
    if kind == "tree":
        pix, flux, ra, dec = _pixels(case, seed)
        pix, inv = np.unique(pix, return_inverse=True)
        flux = np.bincount(inv, flux)
        V = _sum_terms(uvw, _dev(*_project(_centres(case["J"], pix), ra, dec)), _dev(flux)[0])
        return V.to(torch.complex64) if case["prec"] == "f32c" else V
    if kind == "adjoint":
        l, m, _ = _model(case["pixels"], case["field"], seed, 6)
        return _sum_rows(uvw, _noise(case["rows"], seed), _dev(l, m, _nm1(l, m)))
    if kind == "image":
        nx, ny = case["nx"], case["ny"]
        l, m = _grid(nx, ny, nx // 2, ny // 2)
        x = _sum_rows(uvw, _sky(case, seed, *uvw), _dev(l, m, _nm1(l, m)))
        return (x.real / case["rows"]).reshape(ny, nx).contiguous()
    if kind == "autograd":
        l, m, flux = _model(case["comps"], case["field"], seed)
        V = _sum_terms(uvw, _dev(l, m, _nm1(l, m)), _dev(flux)[0])
        return [V] + _gradients(uvw, V - _noise(case["rows"], seed), l, m, flux)
    img = _degrid_image(case, seed)
    l, m = _grid(case["nx"], case["ny"], case["nx"] // 2, case["ny"] // 2)
    on = img.ravel() != 0.0
    return _sum_terms(uvw, _dev(l[on], m[on], _nm1(l[on], m[on])), _dev(img.ravel()[on])[0])
