"""Performance cases of the permutohedral-lattice filter.

A case is one use of the public entry points of ``paper_1907_00641_amd`` at
one size; ``listed()`` holds the named ones, ``draw(rng)`` gives further ones
of the same ranges.  ``prepare`` makes the inputs on the GPU (from the seed
alone) and the lattice handle a program keeps between steps, ``run`` is one
pass, ``work`` the traffic and arithmetic the pass cannot do without,
``exact`` the same results in 64 bits from plain torch.

Kinds of pass:

* ``train``  rebuild the lattice on the handle (features change every step),
             forward, backward (value and feature gradients)
* ``infer``  rebuild, forward
* ``apply``  forward on a lattice built once (fixed features, new values)
* ``cross``  rebuild over keys and queries, asymmetric forward and backward
* ``block``  the permutohedral block: prologue (1x1x1 convolutions), batched
             build over the channel groups, forward, backward, prologue
             backward

Embeddings are voxel coordinates divided by a spatial scale plus channels
that look learned: ``mix`` (blobs with a mean each, plus noise per voxel) or
``smooth`` (one slowly varying intensity channel).  Values and upstream
gradients are i.i.d. N(0, 1).
"""
import torch

import paper_1907_00641_amd as P


def _volume(name, kind, w, h, z, extent, mix, smooth, c, mode="raw", batch=1):
    case = {"kind": kind, "w": w, "h": h, "z": z, "extent": extent, "mix": mix, "smooth": smooth, "c": c,
            "mode": mode, "batch": batch}
    return dict(case, name=name) if name else case


def _block(name, w, h, z, c_in, groups, d, c):
    case = {"kind": "block", "w": w, "h": h, "z": z, "c_in": c_in, "groups": groups, "d": d, "c": c}
    return dict(case, name=name) if name else case


def listed():
    return [
        # smallest: a 32^3 patch filtered by its coordinates alone, at inference
        _volume("infer 32^3 d3 C8", "infer", 32, 32, 32, 8.0, 0, False, 8),
        # an attention module on a small feature map, training step
        _volume("train 64^3 d5 C16", "train", 64, 64, 64, 8.0, 2, False, 16),
        # the headline: a training step on a 128^3 volume
        _volume("train 128^3 d5 C32", "train", 128, 128, 128, 8.0, 2, False, 32),
        # the same as normalised non-local means
        _volume("train 128^3 d5 C32 norm", "train", 128, 128, 128, 8.0, 2, False, 32, "norm"),
        # the same with the augmented-channel feature gradient
        _volume("train 128^3 d5 C32 aug", "train", 128, 128, 128, 8.0, 2, False, 32, "aug"),
        # a batch of two 160x160x96 patches with eight learned features, one batched build
        _volume("train 2x160x160x96 d8 C16", "train", 160, 160, 96, 10.0, 5, False, 16, "raw", 2),
        # largest: many channels on a large volume, few features
        _volume("train 192^3 d4 C64", "train", 192, 192, 192, 8.0, 0, True, 64),
        # a cropped, ragged volume whose channel count is no multiple of 4 (scalar rows)
        _volume("train 75x53x41 d5 C7", "train", 75, 53, 41, 8.0, 2, False, 7),
        # many learned features: a lattice of high dimension on a coarse map
        _volume("train 40x36x28 d12 C24", "train", 40, 36, 28, 8.0, 9, False, 24),
        # asymmetric attention: the voxels as keys, the same voxels moved by half a voxel as queries
        _volume("cross 96^3 d5 C32", "cross", 96, 96, 96, 8.0, 2, False, 32),
        # smoothing with fixed features: new values on a lattice built once, normalised
        _volume("apply 100x100x60 d4 C12 norm", "apply", 100, 100, 60, 8.0, 0, True, 12, "norm"),
        # the permutohedral block at half resolution of a 160x160x96 patch: 18 input channels, two groups
        _block("block 80x80x48 2x(d5 C8)", 80, 80, 48, 18, 2, 5, 8),
    ]


def _spread(rng, lo, hi):
    """A whole number spread over [lo, hi] by its logarithm."""
    return int(round(lo * (hi / lo) ** rng.random()))


def _sides(rng, n):
    """Ragged sides of a volume of about n voxels."""
    a, b = 0.75 + 0.5 * rng.random(), 0.75 + 0.5 * rng.random()
    side = n ** (1.0 / 3.0)
    w, h = max(4, round(side * a)), max(4, round(side * b))
    return w, h, max(4, round(n / (w * h)))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "train", "infer", "apply", "cross", "block", "high"])
    if kind == "block":
        w, h, z = _sides(rng, _spread(rng, 20000, 400000))
        return _block(None, w, h, z, rng.randint(8, 32), rng.choice([1, 2, 4]), rng.randint(3, 6),
                      rng.choice([4, 6, 8, 12]))
    if kind == "high":  # many features: few points
        w, h, z = _sides(rng, _spread(rng, 4000, 60000))
        return _volume(None, "train", w, h, z, 8.0, rng.randint(6, 11), False, rng.randint(4, 40))
    w, h, z = _sides(rng, _spread(rng, 12000, 2200000))
    smooth = rng.random() < 0.25
    mix = 0 if smooth else rng.randint(0, 5)
    c = rng.choice([rng.randint(1, 64), 4 * rng.randint(1, 16), 4 * rng.randint(1, 16)])
    mode, batch = "raw", 1
    if kind == "cross":
        w, h, z = _sides(rng, _spread(rng, 8000, 900000))
    elif kind == "train":
        mode = rng.choice(["raw", "raw", "raw", "norm", "aug"])
        if mode == "aug":
            w, h, z = _sides(rng, _spread(rng, 12000, 500000))
            c = min(c, 32)
        elif rng.random() < 0.25:
            batch = rng.choice([2, 3])
            w, h, z = _sides(rng, _spread(rng, 8000, 1500000 // batch))
    else:
        mode = rng.choice(["raw", "norm"])
    return _volume(None, kind, w, h, z, 6.0 + 4.0 * rng.random(), mix, smooth, c, mode, batch)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _coords(case, dev, shift=0.0):
    w, h, z = case["w"], case["h"], case["z"]
    i = torch.arange(w * h * z, device=dev)
    xyz = torch.stack([i % w, (i // w) % h, i // (w * h)], 1).float()
    return xyz, (xyz + shift) * (case["extent"] / max(w, h, z))


def _extras(case, gen, dev, xyz):
    """Learned-like channels of one volume (n x (mix + smooth))."""
    w, h, z = case["w"], case["h"], case["z"]
    parts = []
    if case["mix"]:
        blobs = 6 if case["mix"] <= 2 else 10
        size = torch.tensor([w, h, z], device=dev, dtype=torch.float32)
        centres = torch.rand(blobs, 3, generator=gen, device=dev) * size
        means = torch.rand(blobs, case["mix"], generator=gen, device=dev) * 6 - 3
        best = None
        for b in range(blobs):
            dist = ((xyz - centres[b]) ** 2).sum(1)
            if best is None:
                best, comp = dist, torch.zeros_like(dist, dtype=torch.long)
            else:
                near = dist < best
                best, comp = torch.where(near, dist, best), torch.where(near, b, comp)
        std = 0.5 if case["mix"] <= 2 else 0.4
        parts.append(means[comp] + std * torch.randn(xyz.shape[0], case["mix"], generator=gen, device=dev))
    if case["smooth"]:
        coarse = torch.randn(1, 1, z // 6 + 2, h // 6 + 2, w // 6 + 2, generator=gen, device=dev)
        vol = torch.nn.functional.interpolate(coarse, size=(z, h, w), mode="trilinear", align_corners=True).reshape(-1, 1)
        parts.append(3.0 * (vol - vol.mean()) / vol.std())
    return parts


def _features(case, gen, dev):
    parts = []
    for _ in range(case["batch"]):
        xyz, f = _coords(case, dev)
        ex = _extras(case, gen, dev, xyz)
        parts.append(torch.cat([f] + ex, 1))
        if case["kind"] == "cross":  # queries: the keys' voxels moved by half a voxel
            parts.append(torch.cat([_coords(case, dev, 0.5)[1]] + ex, 1))
    return torch.cat(parts, 0).contiguous()


def _inputs(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev)

    n = case["w"] * case["h"] * case["z"]
    if case["kind"] == "block":
        ci, G = case["c_in"], case["groups"]
        d_tot, c_tot = G * case["d"], G * case["c"]
        return {"x": normal(n, ci), "wf": normal(d_tot, ci + 3) / (ci + 3) ** 0.5, "bf": 0.1 * normal(d_tot),
                "wv": normal(c_tot, ci) / ci ** 0.5, "bv": 0.1 * normal(c_tot), "gout": normal(G * n, case["c"])}
    f = _features(case, gen, dev)
    rows = n * case["batch"]
    data = {"f": f, "v": normal(rows, case["c"])}
    if case["kind"] in ("train", "cross"):
        data["g"] = normal(rows, case["c"])
    return data


_FLAGS = {"raw": 0, "norm": P.PAM_NORMALIZE, "aug": 0}
_MESH, _SLOPE = 1.0 / 8.0, 0.01


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    n = case["w"] * case["h"] * case["z"]
    if case["kind"] == "block":
        G = case["groups"]
        s["desc"] = P.block_desc(case["c_in"], G * case["d"], G * case["c"], G, (case["w"], case["h"], case["z"]),
                                 _MESH, _SLOPE)
        s["groups"] = [g * n for g in range(G + 1)] if G > 1 else None
        feat, _ = P.pam_block_fwd(s["desc"], s["x"], s["wf"], s["bf"], s["wv"], s["bv"])
        s["lat"] = P.pam_lattice_build(feat, group_start=s["groups"])
        return s
    s["flags"] = _FLAGS[case["mode"]]
    s["groups"] = [b * n for b in range(case["batch"] + 1)] if case["batch"] > 1 else None
    s["lat"] = P.pam_lattice_build(s["f"], group_start=s["groups"])
    return s


def run(s):
    case, kind, lat = s["case"], s["case"]["kind"], s["lat"]
    if kind == "block":
        feat, val = P.pam_block_fwd(s["desc"], s["x"], s["wf"], s["bf"], s["wv"], s["bv"])
        P.pam_lattice_build(feat, lat=lat, group_start=s["groups"])
        out = P.pam_filter_fwd(lat, val)
        dv, df = P.pam_filter_bwd(lat, val, s["gout"])
        dx, dwf, dbf, dwv, dbv = P.pam_block_bwd(s["desc"], s["x"], s["wf"], s["bf"], s["wv"], df, dv)
        return {"out": out, "dx": dx, "dwf": dwf, "dbf": dbf, "dwv": dwv, "dbv": dbv}
    if kind != "apply":
        P.pam_lattice_build(s["f"], lat=lat, group_start=s["groups"])
    if kind == "cross":
        nk = s["v"].shape[0]
        out = P.pam_filter_fwd_asym(lat, nk, s["v"])
        dv, df = P.pam_filter_bwd_asym(lat, nk, s["v"], s["g"])
        return {"out": out, "dv": dv, "df": df}
    out = P.pam_filter_fwd(lat, s["v"], s["flags"])
    if kind != "train":
        return {"out": out}
    flags = P.PAM_EGRAD_AUGMENTED if case["mode"] == "aug" else s["flags"]
    dv, df = P.pam_filter_bwd(lat, s["v"], s["g"], flags)
    return {"out": out, "dv": dv, "df": df}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Bytes: every input read once, every output written once (the lattice
    is internal).  Operations: the elevation of a point, and two per channel
    and simplex vertex for a splat, a slice and each of eq. 8's two products
    (the blur's depend on the vertex count and are left out)."""
    n = case["w"] * case["h"] * case["z"] * case.get("batch", 1)
    if case["kind"] == "block":
        ci, G, d, c = case["c_in"], case["groups"], case["d"], case["c"]
        wts = G * d * (ci + 4) + G * c * (ci + 1)
        return {"bytes": 4 * (n * (2 * ci + 2 * G * c) + 2 * wts),
                "flops": 3 * 2 * n * G * (d * (ci + 3) + c * ci) + n * G * (2 * (d + 1) ** 2 + 12 * (d + 1) * c)}
    d, c = 3 + case["mix"] + int(case["smooth"]), case["c"]
    pts = 2 * n if case["kind"] == "cross" else n
    elevate, side = 2 * (d + 1) ** 2, 2 * (d + 1) * c
    if case["kind"] == "apply":
        return {"bytes": 4 * n * 2 * c, "flops": 2 * n * side}
    if case["kind"] == "infer":
        return {"bytes": 4 * n * (d + 2 * c), "flops": n * (elevate + 2 * side)}
    flops = pts * elevate + n * 6 * side
    if case["mode"] == "aug":
        flops += n * 4 * d * side
    return {"bytes": 4 * (2 * pts * d + n * 4 * c), "flops": flops}


def tolerance(case):
    """32-bit sums in any order.  Measured against exact() over the listed
    cases and six drawn ones: at most 2.8e-7 (df), 7e-7 between two runs of
    the block (dwf, a sum over all voxels), 1.7e-6 for the augmented-channel
    gradient, whose terms f (x) v - f W v cancel; largest single values 6e-6,
    2e-5 for the augmented gradient."""
    if case["kind"] == "block":
        return {"rel": 4e-6, "max": 1e-3}
    if case["mode"] == "aug":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 2e-6, "max": 2e-4}


# ---------------------------------------------------------------------------
# 64-bit results in plain torch
# ---------------------------------------------------------------------------

def _embedding(d):
    """E = alpha Q: column j has alpha / sqrt((j+1)(j+2)) on rows 0..j and
    -(j+1) times that on row j+1, alpha = (d+1) sqrt(2/3)."""
    E = torch.zeros(d + 1, d, dtype=torch.float64)
    for j in range(d):
        s = (d + 1) * (2.0 / 3.0) ** 0.5 / ((j + 1) * (j + 2)) ** 0.5
        E[:j + 1, j] = s
        E[j + 1, j] = -(j + 1) * s
    return E


class _Lattice:
    """The lattice of n x d 32-bit features.  Which simplex a point lies in
    is decided in 32 bits (elevation summed in ascending input order, ties
    of the rounding to even, equal residuals by index), everything else is
    64-bit.  A vertex key is the sum of its d first coordinates times random
    64-bit factors, so that a step along a direction adds a constant."""

    def __init__(self, f, group):
        n, d = f.shape
        dev = f.device
        self.d = d
        E = _embedding(d).to(dev)
        self.E = E
        E32 = E.float().double()
        p = f.double()
        x = []
        for c in range(d + 1):
            acc = torch.zeros(n, dtype=torch.float32, device=dev)
            for j in ([c - 1] if c else []) + list(range(c, d)):
                acc = (E32[c, j] * p[:, j] + acc.double()).float()
            x.append(acc)
        x = torch.stack(x, 1)
        inv = torch.tensor(1.0 / (d + 1), dtype=torch.float64).float().to(dev)
        q = torch.round(x * inv).long()
        delta = x - (q * (d + 1)).float()
        order = torch.sort(delta, dim=1, descending=True, stable=True)[1]
        rank = torch.empty_like(order)
        rank.scatter_(1, order, torch.arange(d + 1, device=dev).expand(n, -1).contiguous())
        off = q.sum(1, keepdim=True)
        up, down = (off > 0) & (rank >= d + 1 - off), (off < 0) & (rank < -off)
        q = q - up.long() + down.long()
        rank = rank + off + (d + 1) * (down.long() - up.long())
        self.rank = rank
        y = (p @ E.T - (q * (d + 1)).double()) / (d + 1)
        ys = torch.empty_like(y).scatter_(1, rank, y)
        b = torch.empty_like(y)
        b[:, 0] = 1 + ys[:, d] - ys[:, 0]
        for k in range(1, d + 1):
            b[:, k] = ys[:, d - k] - ys[:, d + 1 - k]
        self.b = b
        gen = torch.Generator()
        gen.manual_seed(1907)
        R = torch.randint(-(1 << 62), 1 << 62, (d + 1,), generator=gen).to(dev)
        keys = []
        for k in range(d + 1):
            t = q[:, :d] - (rank[:, :d] > d - k).long()
            keys.append(((k + (d + 1) * t) * R[:d]).sum(1) + group * R[d])
        key, inverse = torch.unique(torch.stack(keys, 1), return_inverse=True)
        self.v = inverse
        self.M = M = key.numel()
        self.nbr = []
        for j in range(d + 1):
            step = -R[:d].sum() + ((d + 1) * R[j] if j < d else 0)
            both = []
            for sgn in (-1, 1):
                want = key + sgn * step
                at = torch.searchsorted(key, want).clamp_(max=M - 1)
                both.append(torch.where(key[at] == want, at, M))
            self.nbr.append(both)
        G = 4.0 ** (d + 1) * (3 / (4 * torch.pi)) ** (d / 2) / (d + 1) ** 0.5
        self.scale = 1.0 / G

    def splat(self, x):
        L = torch.zeros(self.M, x.shape[1], dtype=torch.float64, device=x.device)
        for k in range(self.d + 1):
            L.index_add_(0, self.v[:, k], self.b[:, k:k + 1] * x)
        return L

    def blur(self, L, reverse=False):
        zero = torch.zeros(1, L.shape[1], dtype=torch.float64, device=L.device)
        for lo, hi in (self.nbr[::-1] if reverse else self.nbr):
            pad = torch.cat([L, zero])
            L = 2 * L + pad[lo] + pad[hi]
        return L

    def slice(self, L):
        return sum(self.b[:, k:k + 1] * L[self.v[:, k]] for k in range(self.d + 1))

    def at_vertices(self, x, L):
        """<x_i, L[m_ik]> for every point and vertex."""
        return torch.stack([(x * L[self.v[:, k]]).sum(1) for k in range(self.d + 1)], 1)

    def feature_gradient(self, h):
        """Eq. 8: from the derivatives with respect to the weights."""
        d = self.d
        r = self.rank
        gx = (h.gather(1, d - r) - h.gather(1, (d + 1 - r) % (d + 1))) / (d + 1)
        return gx @ self.E


def _filter(lat, v, g, mode):
    """(out, dv, df); dv and df None without g."""
    s = lat.scale
    if mode == "norm":
        one = torch.ones(v.shape[0], 1, dtype=torch.float64, device=v.device)
        A = lat.blur(lat.splat(torch.cat([v, one], 1)))
        sl = lat.slice(A)
        z = sl[:, -1:]
        out = sl[:, :-1] / z
        if g is None:
            return out, None, None
        gz, gam = g / z, -(g * out).sum(1, keepdim=True) / z
        At = lat.blur(lat.splat(torch.cat([gz, gam], 1)), True)
        dv = lat.slice(At)[:, :-1]
        h = lat.at_vertices(torch.cat([gz, gam], 1), A) + lat.at_vertices(torch.cat([v, one], 1), At)
        return out, dv, lat.feature_gradient(h)
    A = lat.blur(lat.splat(v))
    out = s * lat.slice(A)
    if g is None:
        return out, None, None
    At = lat.blur(lat.splat(g), True)
    dv = s * lat.slice(At)
    return out, dv, lat.feature_gradient(s * (lat.at_vertices(g, A) + lat.at_vertices(v, At)))


def _augmented_gradient(lat, f, v, g, out, dv):
    """dL/df_iq = sum_c g_ic (W(f_q v)_ic - f_iq out_ic) + v_ic (W^T(f_q g)_ic - f_iq dv_ic)."""
    cols = []
    for q in range(f.shape[1]):
        fq = f[:, q:q + 1].double()
        W = lat.scale * lat.slice(lat.blur(lat.splat(fq * v)))
        Wt = lat.scale * lat.slice(lat.blur(lat.splat(fq * g), True))
        cols.append((g * (W - fq * out) + v * (Wt - fq * dv)).sum(1))
    return torch.stack(cols, 1)


def exact(case, seed):
    s = _inputs(case, seed)
    n = case["w"] * case["h"] * case["z"]
    dev = torch.device("cuda")
    if case["kind"] == "block":
        return _exact_block(case, s, n, dev)
    f, v = s["f"], s["v"].double()
    g = s["g"].double() if "g" in s else None
    if case["kind"] == "cross":
        lat = _Lattice(f, torch.zeros(2 * n, dtype=torch.long, device=dev))
        none = torch.zeros_like(v)
        out, dv, df = _filter(lat, torch.cat([v, none]), torch.cat([none, g]), "raw")
        return {"out": out[n:].clone(), "dv": dv[:n].clone(), "df": df}
    lat = _Lattice(f, torch.arange(f.shape[0], device=dev) // n)
    out, dv, df = _filter(lat, v, g, case["mode"])
    if case["kind"] != "train":
        return {"out": out}
    if case["mode"] == "aug":
        df = _augmented_gradient(lat, f, v, g, out, dv)
    return {"out": out, "dv": dv, "df": df}


def _exact_block(case, s, n, dev):
    G = case["groups"]
    x, wf, wv = s["x"].double(), s["wf"].double(), s["wv"].double()
    w, h = case["w"], case["h"]
    i = torch.arange(n, device=dev)
    xm = torch.cat([x, _MESH * torch.stack([i % w, (i // w) % h, i // (w * h)], 1).double()], 1)
    pre = xm @ wf.T + s["bf"].double()
    f, v = torch.where(pre > 0, pre, _SLOPE * pre), x @ wv.T + s["bv"].double()

    def split(a):
        return torch.cat(a.chunk(G, 1), 0)

    def join(a):
        return torch.cat(a.chunk(G, 0), 1)

    lat = _Lattice(split(f).float(), torch.arange(G * n, device=dev) // n)
    out, dv, df = _filter(lat, split(v), s["gout"].double(), "raw")
    dz, dv = join(df) * torch.where(pre > 0, 1.0, _SLOPE), join(dv)
    return {"out": out, "dx": dz @ wf[:, :case["c_in"]] + dv @ wv, "dwf": dz.T @ xm, "dbf": dz.sum(0),
            "dwv": dv.T @ x, "dbv": dv.sum(0)}
