"""Workloads of the registration library, from its smallest call to its largest.

A case is a dict of plain values.  `listed()` names the fixed ones, `draw(rng)`
gives more of the same ranges, `prepare` makes what a program holds before the
call (scans of one phantom, a displacement field, the pair with its pyramid),
`run` is one pass through the public entry points, `work` the bytes and
operations that pass cannot do without, and `exact` the same outputs computed
by torch in 64 bits.

Kinds:
  eval      Pair.eval: the objective and its gradient of one pair at its finest
            level (what every step of a registration calls)
  batch     objective(...).sum().backward(): several pairs behind autograd
  multi     Multi.eval: four scans (two orthogonal pairs) evaluated jointly
  ingest    Pair(...) from volumes, and the first evaluation of every coarser
            level at zero displacement (how each registration begins)
  register  Pair.register with a short schedule, merged volumes included
  merge     Pair.merge of the OCT and OCTA volumes with a given field
  enface    enface_project of one scan
  axial     resample_axial of one volume
"""
import math

import numpy as np
import torch

import paper_2010_06931_amd as octmc

DEV = "cuda"
ALPHA, DELTA0, EPS, EPS_R, FLYBACK, KAPPA, TAU = 1.0, 0.5, 1e-3, 0.1, 0.25, 1.0, 0.05
STORE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def listed():
    return [
        # one small pair, or a coarse pyramid level of a large one: launches and latency
        dict(name="eval 64x128 f32", kind="eval", n=64, d=128, dtype="f32"),
        # a ragged mid-size scan of odd depth (the second level of a 500 x 465 pair)
        dict(name="eval 251x233 bf16", kind="eval", n=251, d=233, dtype="bf16"),
        # a clinical scan in full precision
        dict(name="eval 300x640 f32", kind="eval", n=300, d=640, dtype="f32"),
        # the paper's scan size
        dict(name="eval 500x465 f16", kind="eval", n=500, d=465, dtype="f16"),
        # the dense workload of the benchmark
        dict(name="eval 500x800 bf16", kind="eval", n=500, d=800, dtype="bf16"),
        # a batch behind autograd, forward and backward
        dict(name="batch 8 200x512 f32", kind="batch", n=200, d=512, dtype="f32", count=8),
        # two orthogonal pairs registered jointly
        dict(name="multi 300x640 bf16", kind="multi", n=300, d=640, dtype="bf16"),
        # the start of a registration: volumes to a pair with its pyramid, and
        # the coarser levels' first evaluations
        dict(name="ingest 300x640 f32", kind="ingest", n=300, d=640, dtype="f32"),
        # a whole call: solve with a short schedule and merge
        dict(name="register 64x128 f32", kind="register", n=64, d=128, dtype="f32", levels=3, iters=4),
        # the outputs of a registration at the paper's scan size
        dict(name="merge 500x465 bf16", kind="merge", n=500, d=465, dtype="bf16"),
        # the OCTA image of one scan at the paper's scan size
        dict(name="enface 500x465 f32", kind="enface", n=500, d=465, dtype="f32", scan=1),
        # one prealigned volume of the dense workload
        dict(name="axial 500x800 f32", kind="axial", n=500, d=800, dtype="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval"] * 5 + ["batch", "multi", "ingest", "register", "merge", "enface", "axial"])
    dtype = rng.choice(["f32", "bf16", "f16"])
    n, d = _log(rng, 40, 500), _log(rng, 96, 800)
    if kind == "eval":
        return dict(kind=kind, n=n, d=d, dtype=dtype)
    if kind == "batch":
        return dict(kind=kind, n=min(n, 200), d=min(d, 512), dtype=dtype, count=rng.randint(2, 8))
    if kind == "multi":
        return dict(kind=kind, n=min(n, 300), d=min(d, 640), dtype=dtype)
    if kind == "ingest":
        return dict(kind=kind, n=min(n, 400), d=d, dtype="f32")
    if kind == "register":
        return dict(kind=kind, n=_log(rng, 40, 120), d=_log(rng, 96, 256), dtype=dtype, levels=rng.randint(2, 3),
                    iters=4)
    if kind == "merge":
        return dict(kind=kind, n=n, d=min(d, 465), dtype=dtype)
    if kind == "enface":
        return dict(kind=kind, n=n, d=min(d, 465), dtype="f32", scan=rng.randint(0, 1))
    return dict(kind=kind, n=n, d=d, dtype="f32")


# ---------------------------------------------------------------------------
# scans of one phantom


def _walk(rng, n, amp, orient):
    """Eye motion at every A-scan [n][n][3] (pixels): a drift over acquisition
    time and a few saccades; B-scans along x (orient 0) or y (1)."""
    fly = int(math.floor(FLYBACK * n + 0.5))
    t = n * (n + fly)
    step = rng.normal(0.0, 0.03, (t, 3))
    for q in rng.integers(1, t, 6):
        step[q] += rng.uniform(-amp, amp, 3)
    m = np.cumsum(step, axis=0).reshape(n, n + fly, 3)[:, :n]
    m = m - m.mean(axis=(0, 1))
    m = m * min(1.0, 8.0 / max(1e-9, np.abs(m).max()))
    return m if orient == 0 else m.transpose(1, 0, 2).copy()


def _pull(m):
    """The field that undoes the motion: d(p) = -m(p + d(p))."""
    n = m.shape[0]
    j, i = np.meshgrid(np.arange(n), np.arange(n), indexing="ij")
    d = -m
    for _ in range(6):
        x = np.clip(np.rint(i + d[..., 0]).astype(np.int64), 0, n - 1)
        y = np.clip(np.rint(j + d[..., 1]).astype(np.int64), 0, n - 1)
        d = -m[y, x]
    return d


def _smooth(v, dim):
    n = v.shape[dim]
    out = 0.5 * v
    out.narrow(dim, 1, n - 1).add_(v.narrow(dim, 0, n - 1), alpha=0.25)
    out.narrow(dim, 0, n - 1).add_(v.narrow(dim, 1, n - 1), alpha=0.25)
    return out


def _acquire(truth, m, margin, n, d):
    """One scan: trilinear samples of the phantom at the moved positions."""
    out = torch.empty((n, n, d), device=DEV)
    m = torch.as_tensor(m, dtype=torch.float32, device=DEV) + margin
    k = torch.arange(d, device=DEV)
    rows = max(1, 2 ** 23 // (n * d))
    g = truth.shape[0]
    for j0 in range(0, n, rows):
        q = m[j0:j0 + rows]
        jj = torch.arange(j0, j0 + q.shape[0], device=DEV)[:, None]
        ii = torch.arange(n, device=DEV)[None, :]
        f = torch.floor(q)
        t = q - f
        f = f.long()
        acc = 0.0
        for b in (0, 1):
            for a in (0, 1):
                y, x = (jj + f[..., 1] + b).clamp(0, g - 1), (ii + f[..., 0] + a).clamp(0, g - 1)
                wgt = (t[..., 1] if b else 1 - t[..., 1]) * (t[..., 0] if a else 1 - t[..., 0])
                acc = acc + wgt[..., None] * truth[y, x]
        z = k + f[..., 2:3]
        top = truth.shape[2] - 1
        out[j0:j0 + rows] = (1 - t[..., 2:3]) * acc.gather(2, z.clamp(0, top)) + \
            t[..., 2:3] * acc.gather(2, (z + 1).clamp(0, top))
    return out


def _scans(n, d, seed, orients=(0, 1), octa=False):
    """Structural volumes, OCTA volumes (or None), en face images, validity and
    an estimate of the displacement field (0.2 px off the truth)."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed + 1)
    margin = 9
    g, gd = n + 2 * margin, d + 2 * margin
    u = torch.arange(g, device=DEV) / g - 0.5
    z = (torch.arange(gd, device=DEV) - margin).float()
    refl = [0.05, 0.7, 0.35, 0.6, 0.25, 0.95, 0.4]
    noise = torch.randn((g, g, gd), generator=gen, device=DEV)
    for dim in (0, 1, 2):
        noise = _smooth(noise, dim)
    noise /= noise.std()
    truth = torch.empty_like(noise)
    slab = torch.empty_like(noise) if octa else None
    c = rng.normal(0, 0.03, (6, 4))
    for r in range(0, g, 32):
        ur = u[r:r + 32, None]
        val = torch.full((ur.shape[0], g, gd), refl[0], device=DEV)
        for b in range(6):
            edge = d * (0.25 + 0.09 * b + c[b, 0] + c[b, 1] * ur + c[b, 2] * u + c[b, 3] * ur * u)
            s = torch.sigmoid((z - edge[..., None]) * 1.5)
            val += (refl[b + 1] - refl[b]) * s
            if octa and b in (1, 3):
                slab[r:r + 32] = s if b == 1 else slab[r:r + 32] * (1 - s)
        truth[r:r + 32] = val * torch.exp(0.5 * noise[r:r + 32] - 0.125)
    del noise
    vessel = torch.randn((g, g), generator=gen, device=DEV)
    for _ in range(6):
        vessel = _smooth(_smooth(vessel, 0), 1)
    vessel = torch.sigmoid((vessel / vessel.std()).abs().sub(0.3).mul(-12.0))
    mot = [_walk(rng, n, 4.0, o) for o in orients]
    centre = np.mean([m.mean(axis=(0, 1)) for m in mot], axis=0)
    mot = [m - centre for m in mot]
    S = [_acquire(truth, m, margin, n, d) for m in mot]
    peak = [s.reshape(-1)[::97].quantile(0.99) for s in S]
    for s, p in zip(S, peak):
        s /= p
    O = None
    if octa:
        slab *= vessel[:, :, None]
        slab += 0.5 * torch.exp(-truth / 0.1)
        O = [_acquire(slab, m, margin, n, d) for m in mot]
        for o in O:
            o += 0.1 * torch.sqrt(-2.0 * torch.log(torch.rand(o.shape, generator=gen, device=DEV).clamp_min_(1e-12)))
        A = [o.mean(dim=2) for o in O]
    else:
        A = [_acquire(vessel[:, :, None].contiguous(), m, margin, n, 1)[..., 0] for m in mot]
        A = [a + 0.05 * torch.randn(a.shape, generator=gen, device=DEV) for a in A]
    V = []
    for _ in orients:
        v = torch.ones(n, device=DEV)
        b = int(rng.integers(3, n - 3))
        v[b - 2:b + 3] = 0.0
        V.append(v)
    D = np.stack([_pull(m) for m in mot])
    D = torch.as_tensor(D + rng.normal(0.0, 0.2, D.shape), dtype=torch.float32, device=DEV)
    return S, O, A, V, D.contiguous()


# ---------------------------------------------------------------------------


def prepare(case, seed):
    kind, n, d = case["kind"], case["n"], case["d"]
    st = dict(case=case, seed=seed)
    if kind == "eval":
        S, _, A, V, D = _scans(n, d, seed)
        st["pair"] = octmc.Pair(S[0], S[1], ax=A[0], ay=A[1], vx=V[0], vy=V[1], dtype=case["dtype"])
        st["pair"].eval(0, D, eta_mode=0)
        st["disp"] = D
    elif kind == "batch":
        st["pairs"], D = [], []
        for b in range(case["count"]):
            S, _, A, V, Db = _scans(n, d, seed * 64 + b)
            st["pairs"].append(octmc.Pair(S[0], S[1], ax=A[0], ay=A[1], vx=V[0], vy=V[1], dtype=case["dtype"],
                                          levels=3))
            D.append(Db)
        D = torch.stack(D)
        octmc.eval_batched(st["pairs"], 0, D, eta_mode=0)
        st["disp"] = D.requires_grad_(True)
    elif kind == "multi":
        S, _, A, V, D = _scans(n, d, seed, (0, 1, 0, 1))
        st["multi"] = octmc.Multi(S, (0, 1, 0, 1), enface=A, valid=V, dtype=case["dtype"], levels=4)
        st["multi"].eval(0, D, eta_mode=0)
        st["disp"] = D
    elif kind in ("ingest", "register", "merge"):
        S, O, _, V, D = _scans(n, d, seed, octa=True)
        st.update(S=S, O=O, V=V)
        if kind == "ingest":
            st["zero"] = []
            while n >= 32:
                n = (n + 1) // 2
                st["zero"].append(torch.zeros((2, n, n, 3), device=DEV))
        else:
            st["pair"] = octmc.Pair(S[0], S[1], ox=O[0], oy=O[1], vx=V[0], vy=V[1], dtype=case["dtype"],
                                    levels=case.get("levels", 0), iters_per_level=case.get("iters", 100))
            st["disp"] = D
    elif kind == "enface":
        S, O, _, V, _ = _scans(n, d, seed, (case["scan"],), octa=True)
        st.update(S=S, O=O, V=V, work=torch.empty(octmc.enface_workspace_size(n, n, d), dtype=torch.uint8, device=DEV))
    else:
        S, _, _, _, D = _scans(n, d, seed, (0,))
        st.update(S=S, dz=D[0, :, :, 2].contiguous())
    return st


def run(st):
    kind = st["case"]["kind"]
    if kind == "eval":
        return st["pair"].eval(0, st["disp"])
    if kind == "batch":
        st["disp"].grad = None
        F = octmc.objective(st["disp"], st["pairs"], 0)
        F.sum().backward()
        return F.detach(), st["disp"].grad
    if kind == "multi":
        return st["multi"].eval(0, st["disp"])
    if kind == "ingest":
        S, O, V = st["S"], st["O"], st["V"]
        pair = octmc.Pair(S[0], S[1], ox=O[0], oy=O[1], vx=V[0], vy=V[1], dtype=st["case"]["dtype"])
        out = [pair.eval(1 + q, z, eta_mode=0) for q, z in enumerate(st["zero"]) if 1 + q < pair.levels]
        pair.close()
        return out
    if kind == "register":
        disp, oct_, octa, _ = st["pair"].register(merged=True)
        return disp, oct_, octa
    if kind == "merge":
        return st["pair"].merge(st["disp"], octa=True)
    if kind == "enface":
        return octmc.enface_project(st["S"][0], st["O"][0], st["case"]["scan"], st["V"][0], workspace=st["work"])
    return octmc.resample_axial(st["S"][0], st["dz"])


def work(case):
    """Volumes read once in their storage type, fields and images once each;
    operations: the separable resampling of every voxel and its adjoint."""
    kind, na, d = case["kind"], case["n"] ** 2, case["d"]
    b = 4 if case["dtype"] == "f32" else 2
    vox = float(na) * d
    if kind == "eval":
        return dict(bytes=2 * vox * b + 56 * na, flops=192 * vox)
    if kind == "batch":
        return dict(bytes=case["count"] * (2 * vox * b + 56 * na), flops=case["count"] * 192 * vox)
    if kind == "multi":
        return dict(bytes=4 * vox * b + 112 * na, flops=4 * 104 * vox + 6 * 24 * vox)
    if kind == "ingest":
        return dict(bytes=4 * vox * 4 + 2 * vox * 4 * 8 / 7, flops=4 * vox + 192 * vox / 7)
    if kind == "register":
        evals = case["iters"] + 2
        return dict(bytes=evals * (2 * vox * b + 56 * na) + 2 * vox * (b + 4) + 8 * vox,
                    flops=evals * 192 * vox * 8 / 7 + 160 * vox)
    if kind == "merge":
        return dict(bytes=2 * vox * b + 2 * vox * 4 + 8 * vox + 24 * na, flops=160 * vox)
    if kind == "enface":
        return dict(bytes=8 * vox + 4 * na, flops=84 * vox)
    return dict(bytes=8 * vox + 4 * na, flops=8 * vox)


# ---------------------------------------------------------------------------
# the same outputs in 64 bits

F64 = torch.float64


def _taps(t):
    t2, t3 = t * t, t * t * t
    w = [(-t3 + 2 * t2 - t) / 2, (3 * t3 - 5 * t2 + 2) / 2, (-3 * t3 + 4 * t2 + t) / 2, (t3 - t2) / 2]
    dw = [(-3 * t2 + 4 * t - 1) / 2, (9 * t2 - 10 * t) / 2, (-9 * t2 + 8 * t + 1) / 2, (3 * t2 - 2 * t) / 2]
    return w, dw


def _split(x):
    f = torch.floor(x)
    return f.long(), x - f


def _resample(vol, D, r0, r1, grad=True):
    """Values (and x, y, z derivatives) of vol [h][w][d] resampled with the
    field D [h][w][3] at the A-scans of rows r0 .. r1."""
    h, w, d = vol.shape
    flat = vol.reshape(h * w, d)
    q = D[r0:r1].to(F64)
    jj = torch.arange(r0, r1, device=DEV)[:, None]
    ii = torch.arange(w, device=DEV)[None, :]
    (nx, tx), (ny, ty), (nz, tz) = (_split(q[..., c].reshape(r1 - r0, w)) for c in range(3))
    (wx, dwx), (wy, dwy), (wz, dwz) = _taps(tx), _taps(ty), _taps(tz)
    lat = [0.0, 0.0, 0.0]
    for b in range(4):
        for a in range(4):
            y, x = (jj + ny - 1 + b).clamp(0, h - 1), (ii + nx - 1 + a).clamp(0, w - 1)
            col = flat[(y * w + x).reshape(-1)].to(F64)
            lat[0] = lat[0] + (wx[a] * wy[b]).reshape(-1, 1) * col
            if grad:
                lat[1] = lat[1] + (dwx[a] * wy[b]).reshape(-1, 1) * col
                lat[2] = lat[2] + (wx[a] * dwy[b]).reshape(-1, 1) * col
    k = torch.arange(d, device=DEV)
    out = [0.0, 0.0, 0.0, 0.0]
    for c in range(4):
        z = (k + nz.reshape(-1, 1) - 1 + c).clamp(0, d - 1)
        v = lat[0].gather(1, z)
        out[0] = out[0] + wz[c].reshape(-1, 1) * v
        if grad:
            out[3] = out[3] + dwz[c].reshape(-1, 1) * v
            out[1] = out[1] + wz[c].reshape(-1, 1) * lat[1].gather(1, z)
            out[2] = out[2] + wz[c].reshape(-1, 1) * lat[2].gather(1, z)
    return out


def _image(img, D):
    """A 2-D image sampled at (i + dx, j + dy): value, d/dx, d/dy."""
    h, w = img.shape
    D = D.to(F64)
    jj, ii = torch.arange(h, device=DEV)[:, None], torch.arange(w, device=DEV)[None, :]
    (nx, tx), (ny, ty) = _split(D[..., 0]), _split(D[..., 1])
    (wx, dwx), (wy, dwy) = _taps(tx), _taps(ty)
    v = gx = gy = 0.0
    for b in range(4):
        for a in range(4):
            s = img[(jj + ny - 1 + b).clamp(0, h - 1), (ii + nx - 1 + a).clamp(0, w - 1)].to(F64)
            v, gx, gy = v + wx[a] * wy[b] * s, gx + dwx[a] * wy[b] * s, gy + wx[a] * dwy[b] * s
    return v, gx, gy


def _valid(vec, D, orient):
    """The validity resampled along the slow axis, clamped, and its derivative."""
    n = vec.numel()
    idx = torch.arange(n, device=DEV)
    idx = idx[:, None] if orient == 0 else idx[None, :]
    f, t = _split(D[..., 1 if orient == 0 else 0].to(F64))
    w, dw = _taps(t)
    v = g = 0.0
    for a in range(4):
        s = vec[(idx + f - 1 + a).clamp(0, n - 1)].to(F64)
        v, g = v + w[a] * s, g + dw[a] * s
    return v.clamp(0, 1), g * ((v > 0) & (v < 1))


def _huber(x, eps):
    u = x / eps
    s = torch.sqrt(1 + u * u)
    return eps * u * u / (s + 1), u / s


def _objective(S, A, V, orients, D):
    """Terms and gradient of n scans [n][h][w][3], every pair with the eta of
    this field."""
    n, h, w, _ = D.shape
    d = S[0].shape[2]
    pairs = [(p, q) for p in range(n) for q in range(p + 1, n)]
    lam = {pq: torch.zeros((h, w), dtype=F64, device=DEV) for pq in pairs}
    gam = {pq: torch.zeros((2, h, w, 3), dtype=F64, device=DEV) for pq in pairs}
    rows = max(1, 2 ** 24 // (w * d))
    for r0 in range(0, h, rows):
        r1 = min(h, r0 + rows)
        R = [_resample(S[v], D[v], r0, r1) for v in range(n)]
        for p, q in pairs:
            L, dL = _huber(R[p][0] - R[q][0], EPS)
            lam[p, q][r0:r1] = L.sum(1).reshape(r1 - r0, w)
            for s, v in enumerate((p, q)):
                for c in range(3):
                    gam[p, q][s, r0:r1, :, c] = (dL * R[v][1 + c]).sum(1).reshape(r1 - r0, w)
        del R
    t = [0.0] * 10
    G = torch.zeros((n, h, w, 3), dtype=F64, device=DEV)
    for p, q in pairs:
        jp, jq = _image(A[p], D[p]), _image(A[q], D[q])
        LA, dLA = _huber(jp[0] - jq[0], EPS)
        (vp, dvp), (vq, dvq) = _valid(V[p], D[p], orients[p]), _valid(V[q], D[q], orients[q])
        l = lam[p, q]
        s05, a05 = ((1 - 0.5 * vp * vq) * l).sum(), (0.5 * vp * vq * d * LA).sum()
        eta = torch.sqrt(a05 / s05) if s05 > 1e-300 and a05 > 1e-300 else torch.ones((), dtype=F64, device=DEV)
        delta = DELTA0 * vp * vq
        s, a = ((1 - delta) * l).sum(), (delta * d * LA).sum()
        dpd = -eta * l + d / eta * LA
        ws, wa = eta * (1 - delta), d / eta * delta * dLA
        for sgn, v, j, g in ((1, p, jp, gam[p, q][0]), (-1, q, jq, gam[p, q][1])):
            G[v] += sgn * ws[..., None] * g
            G[v, ..., 0] += sgn * wa * j[1]
            G[v, ..., 1] += sgn * wa * j[2]
        G[p, ..., 1 if orients[p] == 0 else 0] += dpd * DELTA0 * vq * dvp
        G[q, ..., 1 if orients[q] == 0 else 0] += dpd * DELTA0 * vp * dvq
        for k, x in ((1, eta * s + a / eta), (2, s), (3, a), (6, s05), (7, a05)):
            t[k] = t[k] + x
        if (p, q) == pairs[0]:
            t[8] = eta
    om = 1 / math.sqrt(1 + math.floor(FLYBACK * w + 0.5))
    for v in range(n):
        X = D[v].to(F64)
        X = (X if orients[v] == 0 else X.transpose(0, 1)).reshape(-1, 3)
        wt = torch.ones(h * w - 1, dtype=F64, device=DEV)
        wt[w - 1::w] = om
        L, dL = _huber(X[1:] - X[:-1], EPS_R)
        t[4] = t[4] + d * (wt[:, None] * L).sum()
        g = torch.zeros_like(X)
        g[1:] += ALPHA * d * wt[:, None] * dL
        g[:-1] -= ALPHA * d * wt[:, None] * dL
        g = g.reshape(h, w, 3)
        G[v] += g if orients[v] == 0 else g.transpose(0, 1)
    sums = D.to(F64).sum(dim=(0, 1, 2))
    t[5] = d * (sums * sums).sum() / (n * h * w)
    G += 2 * d * sums / (n * h * w)
    t[0] = t[1] + ALPHA * t[4] + t[5]
    return torch.stack([torch.as_tensor(x, dtype=F64, device=DEV) for x in t]), G


def _half(x, dims):
    for dim in dims:
        n = x.shape[dim]
        i = torch.arange((n + 1) // 2, device=DEV)
        x = (x.index_select(dim, 2 * i) + x.index_select(dim, (2 * i + 1).clamp(max=n - 1))) / 2
    return x


def _weights(D, V):
    """Normalised merge weights (OCT and OCTA) of the two scans."""
    _, h, w, _ = D.shape
    jj, ii = torch.arange(h, device=DEV)[:, None], torch.arange(w, device=DEV)[None, :]
    rho = []
    for v in range(2):
        x = (ii + D[v, ..., 0]).clamp(0, w - 1).to(F64)
        y = (jj + D[v, ..., 1]).clamp(0, h - 1).to(F64)
        (x0, fx), (y0, fy) = _split(x), _split(y)
        x1, y1 = (x0 + 1).clamp(max=w - 1), (y0 + 1).clamp(max=h - 1)
        c = [(y0 * w + x0, (1 - fx) * (1 - fy)), (y0 * w + x1, fx * (1 - fy)), (y1 * w + x0, (1 - fx) * fy),
             (y1 * w + x1, fx * fy)]
        grid = torch.zeros(h * w, dtype=F64, device=DEV)
        for at, wt in c:
            grid.index_add_(0, at.reshape(-1), wt.reshape(-1))
        rho.append(sum(wt * grid[at] for at, wt in c))
    wt = [torch.exp(-KAPPA * (r - 1).clamp(min=0)) for r in rho]
    wt = [torch.where(x < TAU, torch.zeros_like(x), x) for x in wt]
    s = wt[0] + wt[1]
    first = (rho[0] <= rho[1]).to(F64)
    oct_ = [torch.where(s > 0, wt[0] / s, first), torch.where(s > 0, wt[1] / s, 1 - first)]
    va = [wt[v] * _valid(V[v], D[v], v)[0] for v in range(2)]
    sa = va[0] + va[1]
    octa = [torch.where(sa > 0, x / sa, torch.zeros_like(x)) for x in va]
    return oct_, octa


def _fill(O, V, orient):
    """Invalid B-scans replaced by their nearest valid one (the lower on a tie)."""
    good = torch.nonzero(V > 0.5).reshape(-1).tolist()
    src = [min(good, key=lambda g: (abs(g - b), g)) for b in range(V.numel())]
    return O.index_select(0 if orient == 0 else 1, torch.tensor(src, device=DEV))


def _projection(oct_, octa, scan, valid):
    h, w, d = octa.shape

    def window(v, dim, r):
        n = v.shape[dim]
        return [v.index_select(dim, (torch.arange(n, device=DEV) + o).clamp(0, n - 1)) for o in range(-r, r + 1)]

    med = torch.empty_like(octa)
    rows = max(1, 2 ** 23 // (w * d))
    for r0 in range(0, h, rows):
        j = torch.arange(r0, min(h, r0 + rows), device=DEV)
        s = [q for o in (-1, 0, 1) for x in window(octa[(j + o).clamp(0, h - 1)], 1, 1) for q in window(x, 2, 1)]
        med[r0:r0 + rows] = torch.stack(s).kthvalue(14, dim=0).values
    for dim in ((1, 0) if scan == 0 else (0, 1)):
        out = torch.empty_like(med)
        cut = max(1, 2 ** 23 // (w * d))
        other = 1 - dim
        for r0 in range(0, med.shape[other], cut):
            m = min(cut, med.shape[other] - r0)
            out.narrow(other, r0, m).copy_(torch.stack(window(med.narrow(other, r0, m), dim, 7)).kthvalue(3, dim=0).values)
        med = out
    pool = (med[valid > 0.5] if scan == 0 else med[:, valid > 0.5]).reshape(-1).sort().values
    p = []
    for q in (0.05, 0.95):
        x = q * (pool.numel() - 1)
        lo = int(math.floor(x))
        a, b = float(pool[lo]), float(pool[min(lo + 1, pool.numel() - 1)])
        p.append(a + (x - lo) * (b - a))
    top = oct_[:, :, :max(1, int(round(0.05 * d)))].to(F64)
    thr = float(top.mean() + 2 * top.std(unbiased=False))
    mask = (med.to(F64) < p[0] + 0.1 * (p[1] - p[0])) & (oct_.to(F64) > thr)
    cnt = mask.sum(2)
    img = torch.where(cnt > 0, (octa.to(F64) * mask).sum(2) / cnt.clamp(min=1), torch.zeros((), dtype=F64, device=DEV))
    lines = img if scan == 0 else img.T
    srt = lines.sort(dim=1).values
    n = lines.shape[1]
    img = lines - (srt[:, (n - 1) // 2] + srt[:, n // 2])[:, None] / 2
    img = img if scan == 0 else img.T
    return _fill(img, valid, scan)


def exact(case, seed):
    kind, n, d = case["kind"], case["n"], case["d"]
    if kind == "register":
        return None  # an iterative solve
    store = STORE[case["dtype"]]
    if kind == "eval":
        S, _, A, V, D = _scans(n, d, seed)
        return _objective([s.to(store) for s in S], A, V, (0, 1), D)
    if kind == "batch":
        F, G = [], []
        for b in range(case["count"]):
            S, _, A, V, D = _scans(n, d, seed * 64 + b)
            t, g = _objective([s.to(store) for s in S], A, V, (0, 1), D)
            F.append(t[0])
            G.append(g)
        return torch.stack(F), torch.stack(G)
    if kind == "multi":
        S, _, A, V, D = _scans(n, d, seed, (0, 1, 0, 1))
        return _objective([s.to(store) for s in S], A, V, (0, 1, 0, 1), D)
    if kind == "ingest":
        S, O, _, V, _ = _scans(n, d, seed, octa=True)
        S, A = [s.to(F64) for s in S], [_fill(O[v], V[v], v).to(F64).mean(2) for v in range(2)]
        out = []
        while n >= 32:
            n = (n + 1) // 2
            S, A, V = [_half(s, (0, 1, 2)) for s in S], [_half(a, (0, 1)) for a in A], [_half(v, (0,)) for v in V]
            out.append(_objective(S, A, V, (0, 1), torch.zeros((2, n, n, 3), device=DEV)))
        return out
    if kind == "merge":
        S, O, _, V, D = _scans(n, d, seed, octa=True)
        wo, wa = _weights(D, V)
        out = [torch.empty((n, n, d), dtype=F64, device=DEV) for _ in range(2)]
        O = [_fill(O[v], V[v], v) for v in range(2)]
        rows = max(1, 2 ** 24 // (n * d))
        for r0 in range(0, n, rows):
            r1 = min(n, r0 + rows)
            for o, vols, wt in ((out[0], [s.to(store) for s in S], wo), (out[1], O, wa)):
                o[r0:r1] = sum(wt[v][r0:r1, :, None] * _resample(vols[v], D[v], r0, r1, False)[0].reshape(r1 - r0, n, d)
                               for v in range(2))
        return out[0], out[1]
    if kind == "enface":
        S, O, _, V, _ = _scans(n, d, seed, (case["scan"],), octa=True)
        return _projection(S[0], O[0], case["scan"], V[0])
    S, _, _, _, D = _scans(n, d, seed, (0,))
    dz = torch.zeros((n, n, 3), device=DEV)
    dz[..., 2] = D[0, :, :, 2]
    out = torch.empty((n, n, d), dtype=F64, device=DEV)
    rows = max(1, 2 ** 24 // (n * d))
    for r0 in range(0, n, rows):
        r1 = min(n, r0 + rows)
        out[r0:r1] = _resample(S[0], dz, r0, r1, False)[0].reshape(r1 - r0, n, d)
    return out
