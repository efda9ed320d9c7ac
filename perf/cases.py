"""Workloads whose speed matters to users of the MOFF imager, one dict per case.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs on the GPU (from the seed) and the plan
    run(state)           one pass through the public entry points; its outputs
    work(case)           bytes and flops one pass cannot do without
    exact(case, seed)    the same outputs in 64 bits, in plain torch

A case is an antenna array (layout, illumination tables, grid), a band, an
integration length, an input format, and what is done with it (`op`):

    image      time-averaged image cube of one integration
    stream     the integration arrives in `chunks` pieces: running sums, then
               the image (returned with the sums)
    calibrate  one step of gain calibration: image, L2 loss against a model sky
               and its gradient with respect to the complex gains
    fx         the visibility-route image of the integration
    fields     per-sample gridded apertures and complex image fields

The array belongs to the case; samples and gains come from the seed.  Plans
are kept from one integration to the next, as a program that images a stream
of integrations of one array keeps them.
"""
import math

import numpy as np
import torch

import paper_1510_08318_amd as moff

_DEVICE = 0
_C_LIGHT = 299792458.0
_LAYOUT_SEED = 1510
_PRECISION_FLAG = {"f32": 0, "f16": moff.MOFF_MFMA_F16, "bf16": moff.MOFF_MFMA_BF16}
_AUTOCORR_FLAG = {"exact": 0, "none": moff.MOFF_AUTOCORR_NONE, "uv": moff.MOFF_AUTOCORR_UV}
_BAND = {"low": (40e6, 80e6), "high": (100e6, 200e6)}


def _case(op, layout, ant, extent, tables, grid, chan, time, fmt, band="high", gains=False, precision="f32",
          autocorr="exact", pairs=False, tuned=False, chunks=1):
    return dict(op=op, layout=layout, ant=ant, extent=extent, tables=tables, grid=grid, chan=chan, time=time, fmt=fmt,
                band=band, gains=gains, precision=precision, autocorr=autocorr, pairs=pairs, tuned=tuned, chunks=chunks)


def listed():
    cases = {
        # A small array's quick look: one channel, a few samples; latency and launches.
        "quick look": _case("image", "square", 16, 8.0, "tophat2", 32, 1, 64, "c64", "low"),
        # A full LWA-shaped integration of raw 4+4-bit samples.
        "lwa integration": _case("image", "disc", 256, 100.0, "dipole3", 128, 128, 1000, "ci4", "low", tuned=True),
        # A full HERA-shaped integration, all channels of the band in one call (the benchmark's workload).
        "hera integration": _case("image", "hex", 350, 14.6, "airy7", 256, 1024, 256, "ci4", tuned=True),
        # One step of a gain calibration on a heterogeneous array: forward, loss, backward.
        "calibration step": _case("calibrate", "disc", 1024, 400.0, "mixed", 256, 256, 128, "c64", gains=True,
                                  tuned=True),
        # Calibration of a small array with few channels: a ragged call, complex illumination tables.
        "small calibration": _case("calibrate", "square", 61, 40.0, "complex", 64, 12, 75, "c64", gains=True),
        # Real-time imaging: an LWA-shaped integration arrives in pieces, calibrated, on a part of the band.
        "stream in pieces": _case("stream", "disc", 256, 100.0, "dipole3", 128, 37, 200, "ci4", "low", gains=True,
                                  chunks=4),
        # A mid-sized heterogeneous array with complex tables, pair-normalised, odd sizes, default launch.
        "mixed array": _case("image", "disc", 203, 60.0, "complex", 64, 33, 257, "c64", gains=True, autocorr="uv",
                             pairs=True),
        # The LWA-shaped integration at reduced precision.
        "lwa binary16": _case("image", "disc", 256, 100.0, "dipole3", 128, 128, 1000, "c64", "low", precision="f16",
                              tuned=True),
        # The same layout on the coarser grid in bfloat16, raw samples.
        "lwa bfloat16 coarse": _case("image", "disc", 256, 100.0, "dipole3", 64, 128, 1000, "ci4", "low",
                                     precision="bf16", tuned=True),
        # Visibility-route image of a HERA-shaped band for comparison with the direct image.
        "hera visibilities": _case("fx", "hex", 350, 14.6, "airy7", 256, 256, 256, "ci4"),
        # The same for a large calibrated heterogeneous array.
        "calibrated visibilities": _case("fx", "disc", 1024, 400.0, "mixed", 256, 64, 128, "c64", gains=True),
        # Per-sample image fields (transient search): gridding and the padded transform, every frame written out.
        "sample fields": _case("fields", "disc", 256, 100.0, "dipole3", 128, 32, 24, "ci4", "low"),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_MAX_COST = 262144 * 256 * 256 * 16.0   # the benchmark workload: frames x N^2 log2 N^2


def _cost(c):
    per_frame = c["grid"] ** 2 * 2.0 * math.log2(c["grid"])
    cost = per_frame * c["time"] * c["chan"]
    if c["op"] == "calibrate":
        cost *= 4
    if c["op"] == "fx":
        cost = c["chan"] * (0.5 * c["time"] * c["ant"] ** 2 + 60.0 * c["ant"] ** 2 + 400.0 * c["grid"] ** 2)
    if c["op"] == "fields":
        cost *= 16
    return cost


def draw(rng):
    op = rng.choice(["image", "image", "image", "stream", "calibrate", "fx", "fields"])
    grid = rng.choice([32, 64, 64, 128, 128, 128, 256, 256])
    layout = rng.choice(["square", "disc", "hex"])
    tables = rng.choice(["tophat2", "dipole3", "airy7", "mixed", "complex"])
    extent = 14.6 if layout == "hex" else round(rng.uniform(8.0, 400.0), 1)
    ant = _log_int(rng, 12, 1024 if grid >= 64 else 200)
    c = _case(op, layout, ant, extent, tables, grid, _log_int(rng, 1, 1024), _log_int(rng, 8, 1000),
              rng.choice(["c64", "ci4"]), rng.choice(["low", "high"]), gains=op == "calibrate" or rng.random() < 0.5)
    if op == "image":
        c["autocorr"] = rng.choice(["exact", "exact", "exact", "none", "uv"])
        c["pairs"] = rng.random() < 0.3
        if grid in (64, 128) and rng.random() < 0.3:
            c["precision"] = rng.choice(["f16", "bf16"])
    if op == "stream":
        c["chunks"] = rng.randint(2, 5)
    # no more than a quarter of the largest listed case, and inputs of at most 400 MB
    while _cost(c) > _MAX_COST / 4 or c["time"] * c["chan"] * c["ant"] * 8 > 4e8 or (
            op == "fields" and c["time"] * c["chan"] * c["grid"] ** 2 * 10 > 4e8):
        if c["chan"] > 1 and (c["time"] <= 16 or rng.random() < 0.5):
            c["chan"] = max(1, c["chan"] * 2 // 3)
        else:
            c["time"] = max(1, c["time"] * 2 // 3)
    c["chunks"] = min(c["chunks"], c["time"])
    return c


# ---- the array: part of the case ---------------------------------------------

def _layout(case):
    rng = np.random.default_rng(_LAYOUT_SEED)
    n = case["ant"]
    if case["layout"] == "square":
        return rng.uniform(0.0, case["extent"], size=(n, 2))
    if case["layout"] == "disc":
        r = 0.5 * case["extent"] * np.sqrt(rng.uniform(size=n))
        th = rng.uniform(0.0, 2 * np.pi, size=n)
        return np.stack([r * np.cos(th), r * np.sin(th)], axis=1)
    span = int(math.sqrt(n)) + 4    # hexagonal packing of the given pitch, nearest points first
    j, i = np.meshgrid(np.arange(-span, span + 1), np.arange(-span, span + 1), indexing="ij")
    pts = np.stack([(i + 0.5 * j).ravel(), (j * math.sqrt(3.0) / 2).ravel()], axis=1)
    order = np.lexsort((np.round(np.arctan2(pts[:, 1], pts[:, 0]), 9), np.round(np.hypot(pts[:, 0], pts[:, 1]), 9)))
    return pts[order[:n]] * case["extent"]


def _tables(case):
    dipole = np.outer([0.5, 1.0, 0.5], [0.5, 1.0, 0.5])
    h = np.arange(7) - 3.0
    airy = np.maximum(0.0, 1.0 - (np.hypot(h[:, None], h[None, :]) / 3.5) ** 2)
    rng = np.random.default_rng(_LAYOUT_SEED + 1)
    n = case["ant"]
    types = np.zeros(n, np.int32)
    if case["tables"] == "mixed":
        tabs = [dipole, airy]
        types[rng.permutation(n)[: (3 * n) // 10]] = 1
    elif case["tables"] == "complex":
        tabs = [rng.uniform(-1, 1, (k, k)) + 1j * rng.uniform(-1, 1, (k, k)) for k in (3, 5)]
        types = rng.integers(0, 2, n).astype(np.int32)
    else:
        tabs = [{"tophat2": np.ones((2, 2)), "dipole3": dipole, "airy7": airy}[case["tables"]]]
    return [t.astype(np.complex64) for t in tabs], types


def _freqs(case):
    lo, hi = _BAND[case["band"]]
    return lo + (np.arange(case["chan"]) + 0.5) * (hi - lo) / case["chan"]


def _flags(case):
    return ((moff.MOFF_IN_CI4 if case["fmt"] == "ci4" else moff.MOFF_IN_C64) | _PRECISION_FLAG[case["precision"]]
            | _AUTOCORR_FLAG[case["autocorr"]] | (moff.MOFF_NORM_PAIRS if case["pairs"] else 0))


_kept = {}   # the plans of the two arrays in use


def _plan(case, E, gains):
    key = tuple(sorted((k, v) for k, v in case.items() if k != "name"))
    if key not in _kept:
        while len(_kept) >= 2:
            del _kept[next(iter(_kept))]
        tabs, types = _tables(case)
        plan = moff.Plan(_layout(case), [t.shape[0] for t in tabs], tabs, types, _freqs(case), case["grid"], 0.0,
                         _flags(case), _DEVICE)
        if case["tuned"]:
            plan.autotune(E, gains)
        _kept[key] = plan
    return _kept[key]


# ---- samples and gains: from the seed ----------------------------------------

def _inputs(case, seed):
    """Samples E (point sources of random phase, spatially coherent, plus
    receiver noise), gains that undo the antennas' own, and the model sky."""
    dev = f"cuda:{_DEVICE}"
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    T, C, Na, N = case["time"], case["chan"], case["ant"], case["grid"]
    S = 3 if Na < 32 else 20
    noise = 0.1 if case["op"] == "calibrate" or Na < 32 else 1.0
    xy = torch.tensor(_layout(case), device=dev)
    k0 = 2 * math.pi * torch.tensor(_freqs(case), device=dev) / _C_LIGHT
    u = torch.rand((3, S), generator=gen, device=dev, dtype=torch.float64)
    r, th, flux = 0.9 * torch.sqrt(u[0]), 2 * math.pi * u[1], 1.0 + 9.0 * u[2]
    l, m = r * torch.cos(th), r * torch.sin(th)
    path = l[:, None] * xy[None, :, 0] + m[:, None] * xy[None, :, 1]          # [S, Na]
    geo = torch.sqrt(flux)[None, :, None] * torch.exp(-1j * k0[:, None, None] * path[None])
    geo = geo.to(torch.complex64).contiguous()
    phi = torch.rand((C, T, S), generator=gen, device=dev) * (2 * math.pi)
    E = torch.matmul(torch.polar(torch.ones_like(phi), phi), geo)             # [C, T, Na]
    E = E.permute(1, 0, 2).contiguous()
    E += math.sqrt(noise) * torch.randn((T, C, Na), generator=gen, device=dev, dtype=torch.complex64)
    gains = None
    if case["gains"]:
        amp = 0.8 + 0.4 * torch.rand((C, Na), generator=gen, device=dev)
        true = torch.polar(amp, 2 * math.pi * torch.rand((C, Na), generator=gen, device=dev) - math.pi)
        E *= true[None]
        gains = (1.0 / true).contiguous()
    if case["fmt"] == "ci4":
        q = torch.view_as_real(E)
        q = torch.clamp(torch.round(q * (2.0 / torch.sqrt(torch.mean(q * q)))), -8, 7).to(torch.int16)
        E = (((q[..., 0] & 15) << 4) | (q[..., 1] & 15)).to(torch.uint8).contiguous()
    model = None
    if case["op"] == "calibrate":
        # model sky: a two-pixel beam at each source's direction, at the array's total power
        step = _C_LIGHT / torch.tensor(_freqs(case), device=dev) / (N * _cell_m(case))
        pix = torch.arange(N, device=dev, dtype=torch.float64) - N // 2
        tabs, types = _tables(case)
        peak = float(sum(abs(tabs[t].sum()) for t in types)) ** 2
        model = torch.zeros((C, N, N), device=dev)
        for s in range(S):
            bx = torch.exp(-0.125 * (pix[None] - l[s] / step[:, None]) ** 2)
            by = torch.exp(-0.125 * (pix[None] - m[s] / step[:, None]) ** 2)
            model += (float(flux[s]) * peak * by[:, :, None] * bx[:, None, :]).float()
    return E, gains, model


def prepare(case, seed):
    E, gains, model = _inputs(case, seed)
    plan = _plan(case, E, gains)
    state = dict(op=case["op"], plan=plan, E=E, gains=gains, model=model)
    if case["op"] == "stream":
        C, N, T = case["chan"], case["grid"], case["time"]
        cuts = [T * i // case["chunks"] for i in range(case["chunks"] + 1)]
        state["pieces"] = [E[a:b] for a, b in zip(cuts, cuts[1:])]
        state["S"] = torch.zeros((C, N, N), device=E.device)
        state["A"] = torch.zeros((C, plan.n_ktypes), device=E.device, dtype=torch.float64)
    return state


def run(state):
    op, plan, E, gains = state["op"], state["plan"], state["E"], state["gains"]
    if op == "image":
        return plan.image(E, gains)
    if op == "fx":
        return plan.image_fx(E, gains)
    if op == "fields":
        grid = plan.grid(E, gains)
        return grid, plan.fft2(grid)
    if op == "stream":
        S, A = state["S"].zero_(), state["A"].zero_()
        for piece in state["pieces"]:
            plan.accumulate(piece, S, A, gains)
        return plan.finalize(S, A, E.shape[0]), S, A
    g = gains.detach().requires_grad_()
    image = moff.moff_image_autograd(plan, E, g)
    loss = torch.sum((image - state["model"]) ** 2)
    loss.backward()
    return image.detach(), g.grad


def work(case):
    T, C, Na, N = case["time"], case["chan"], case["ant"], case["grid"]
    tabs, types = _tables(case)
    nnz = sum(int(np.count_nonzero(tabs[t])) for t in types)
    sample = 1 if case["fmt"] == "ci4" else 8
    image_bytes = 4.0 * C * N * N
    read = float(T) * C * Na * sample + (8.0 * C * Na if case["gains"] else 0.0)
    transform = 5.0 * N * N * 2 * math.log2(N)
    frame = transform + 8.0 * nnz
    if case["op"] == "fields":
        return {"bytes": read + 8.0 * T * C * (N * N + N * N / 4), "flops": T * C * frame}
    if case["op"] == "fx":
        return {"bytes": read + image_bytes, "flops": C * (4.0 * T * Na * Na + 2.0 * Na * Na + transform)}
    flops = T * C * (frame + 4.0 * N * N)
    if case["op"] == "calibrate":   # forward, then the recomputed field, its adjoint and the model sky
        return {"bytes": read + 2 * image_bytes + 8.0 * C * Na,
                "flops": flops + T * C * (2 * transform + 16.0 * nnz + 2.0 * N * N)}
    return {"bytes": read + image_bytes, "flops": flops}


# ---- the same outputs in 64 bits ---------------------------------------------

def _cell_m(case):
    xy = _layout(case)
    tabs, types = _tables(case)
    room = case["grid"] // 2 - max(tabs[t].shape[0] for t in types) - 1
    span = max(np.ptp(xy[:, 0]), np.ptp(xy[:, 1]))
    return max(_C_LIGHT / float(np.max(_freqs(case))) / 2, float(span) / room)


def _cells(case):
    xy, (tabs, types), cell = _layout(case), _tables(case), _cell_m(case)
    half = (np.array([tabs[t].shape[0] for t in types], np.float64) - 1.0) / 2.0
    ix = np.floor(xy[:, 0] / cell - half + 0.5).astype(np.int64)
    iy = np.floor(xy[:, 1] / cell - half + 0.5).astype(np.int64)
    return ix - ix.min(), iy - iy.min()


def _decoded(case, E):
    if case["fmt"] == "c64":
        return E.to(torch.complex128)
    b = E.to(torch.int16)
    nib = torch.stack([b >> 4, b & 15], dim=-1)
    return torch.view_as_complex(torch.where(nib >= 8, nib - 16, nib).to(torch.float64))


def _taps(case, dev):
    """(antennas, flat aperture cells, table value) of every table entry."""
    tabs, types = _tables(case)
    ix, iy = _cells(case)
    L = case["grid"] // 2
    for p, tab in enumerate(tabs):
        a = np.nonzero(types == p)[0]
        for u in range(tab.shape[0]):
            for v in range(tab.shape[1]):
                if tab[u, v] != 0 and len(a):
                    yield (torch.tensor(a, device=dev), torch.tensor((iy[a] + u) * L + ix[a] + v, device=dev),
                           complex(tab[u, v]))


def exact(case, seed):
    E, gains, model = _inputs(case, seed)
    dev = E.device
    T, C, Na, N = case["time"], case["chan"], case["ant"], case["grid"]
    L = N // 2
    ph = torch.remainder((torch.arange(N, device=dev)[:, None] - L) * torch.arange(L, device=dev)[None, :], N)
    A = torch.polar(torch.ones((N, L), device=dev, dtype=torch.float64), ph.double() * (2 * math.pi / N))   # [N, L]
    tabs, types = _tables(case)
    P = []
    for tab in tabs:
        k = tab.shape[0]
        t = torch.tensor(tab, device=dev).to(torch.complex128)
        P.append((A[:, :k] @ t @ A[:, :k].T).abs() ** 2)
    taps = list(_taps(case, dev))
    kinds = [torch.tensor(np.nonzero(types == p)[0], device=dev) for p in range(len(tabs))]
    scale = 1.0 / (Na * (Na - 1)) if case["pairs"] else 1.0
    fields = case["op"] == "fields"
    grids = torch.empty((T, C, L, L), device=dev, dtype=torch.complex128) if fields else None
    images = torch.empty((T, C, N, N), device=dev, dtype=torch.complex128) if fields else None
    out = torch.empty((C, N, N), device=dev, dtype=torch.float64)
    grad = torch.empty((C, Na), device=dev, dtype=torch.complex128)
    sums = torch.empty((C, N, N), device=dev, dtype=torch.float64)
    powers = torch.empty((C, len(tabs)), device=dev, dtype=torch.float64)
    step = max(1, int(64e6 / (N * N)))     # frames in hand at a time
    for c in range(C):
        raw = _decoded(case, E[:, c])                                          # [T, Na]
        e = raw if gains is None else raw * gains[c].to(torch.complex128)
        S = torch.zeros((N, N), device=dev, dtype=torch.float64)
        kept = []
        for t0 in range(0, T, step):
            ec = e[t0:t0 + step]
            g = torch.zeros((L * L, ec.shape[0]), device=dev, dtype=torch.complex128)
            gr = torch.view_as_real(g)
            for a, cell, w in taps:
                gr.index_add_(0, cell, torch.view_as_real((ec[:, a] * w).T.contiguous()))
            g = g.T.reshape(-1, L, L)
            Y = torch.matmul(torch.matmul(A, g), A.T.contiguous())
            if fields:
                grids[t0:t0 + step, c], images[t0:t0 + step, c] = g, Y
                continue
            S += (Y.real ** 2 + Y.imag ** 2).sum(0)
            if case["op"] == "calibrate":
                kept.append(Y)
        if fields:
            continue
        power = (e.real ** 2 + e.imag ** 2).sum(0)
        sums[c], powers[c] = S, torch.stack([power[k].sum() for k in kinds])
        if case["autocorr"] == "uv":
            Pn = sum(len(kinds[p]) * P[p] for p in range(len(tabs)))
            a0 = sum(len(kinds[p]) * float(np.sum(np.abs(tabs[p].astype(np.complex128)) ** 2))
                     for p in range(len(tabs)))
            I = S - S.sum() / (N * N * a0) * Pn
        elif case["autocorr"] == "none":
            I = S
        else:
            I = S - sum(powers[c, p] * P[p] for p in range(len(tabs)))
        out[c] = I * (scale / T)
        if case["op"] == "calibrate":
            R = 2.0 * (out[c] - model[c].double())
            D = torch.zeros((T, Na), device=dev, dtype=torch.complex128)
            for n, Y in enumerate(kept):
                Z = torch.matmul(torch.matmul(A.conj().T.contiguous(), R * Y), A.conj().resolve_conj())
                Z = Z.reshape(Z.shape[0], L * L)
                for a, cell, w in taps:
                    D[n * step:n * step + Z.shape[0], a] += Z[:, cell] * w.conjugate()
            rho = torch.zeros(Na, device=dev, dtype=torch.float64)
            for p in range(len(tabs)):
                rho[kinds[p]] = (R * P[p]).sum()
            grad[c] = (2.0 * scale / T) * (raw.conj() * (D - e * rho)).sum(0)
    if fields:
        return grids, images
    if case["op"] == "stream":
        return out, sums, powers
    return (out, grad) if case["op"] == "calibrate" else out
