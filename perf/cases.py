"""The work that programs built on this library have it do, as measurable cases.

An integrator with the P3T split evaluates the long-range force once per long
step: radii, tree, force with neighbour lists, the second neighbour stage,
clusters and groups, and, where binaries are handled as groups, the set with
artificial particles and its post-fit. Between long steps it evaluates the
fitted tidal field at the members. Sizes run from a thousand stars to the ten
million of the largest benchmark model; opening angles from 0.3 to 0.8.

A case is a dict of plain values; `kind` names the call sequence:

  step      petar_tree_build + petar_force_long, lists unless nb is False
  graph     the same as one replayed graph (petar_step_graph)
  batch     the same on n_sys clusters of uneven size (petar_step_graph)
  cycle     radii, build, force with the kick, filter, clusters, groups
  close     second neighbour stage, clusters and groups on candidate lists
  binaries  artificial set, its force on the target subset, fit and kick
  eval      fitted tidal field at the members of binaries
"""

import math

import torch

import paper_2006_16560_amd as pt

DEV = "cuda:0"
F64 = torch.float64


def listed():
    def case(name, kind, n, **kw):
        c = dict(name=name, kind=kind, n=n, theta=0.5, leaf=8, group=64, ipl=2, precision="mixed",
                 binaries=0.5, imf=True, nb=True)
        c.update(kw)
        return c

    return [
        # members of a thousand binaries between two long steps: the call
        # that is made most often, all launch and read-back
        case("eval_2k", "eval", 2000, order=3),
        # a young or dissolving cluster of a thousand stars, eager
        case("step_1k", "step", 1000, binaries=0.1),
        # the equal-mass 4k cluster, captured and replayed every long step
        case("graph_4k", "graph", 4096, binaries=0.0, imf=False),
        # 64k stars with half of them in binaries, eager
        case("step_64k", "step", 65536),
        # the same in FP64 pair arithmetic (validation runs, close accounting)
        case("fp64_64k", "step", 65536, precision="fp64"),
        # a whole long step of a 100k cluster (an odd size): radii to groups
        case("cycle_100k", "cycle", 100003, binaries=0.2),
        # tidal tensors of the binaries of the 64k cluster, third order
        case("binaries_64k", "binaries", 65536, order=3),
        # narrow opening angle, a size off every power of two, no lists
        case("step_300k_t03", "step", 300007, theta=0.3, binaries=0.1, nb=False),
        # a million stars, all in binaries: the benchmark's step
        case("step_1m", "step", 1048576, leaf=4, binaries=1.0),
        # second neighbour stage, clusters and groups of that cluster at the
        # benchmark's radii (the core is one percolating cluster)
        case("close_1m", "close", 1048576, leaf=4, binaries=1.0, radii=1.0),
        # a parameter study: 128 clusters of 1k to 128k stars in one launch
        case("batch_128", "batch", 0, binaries=0.2, n_sys=128, n_lo=1024, n_hi=131072),
        # the largest model: ten million stars
        case("step_10m", "step", 10485760, binaries=0.1),
    ]


def draw(rng):
    """A case of the same ranges: sizes over their logarithm, mostly odd."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "step", "step", "graph", "batch", "cycle", "close",
                       "binaries", "eval"])
    c = dict(kind=kind, n=size(1000, 2000000), theta=round(rng.uniform(0.3, 0.8), 3),
             leaf=rng.choice([4, 8, 16]), group=rng.choice([32, 64, 64, 128]),
             ipl=rng.choice([1, 2, 2, 4]), precision="mixed",
             binaries=round(rng.uniform(0.0, 1.0), 2), imf=rng.random() < 0.9, nb=True)
    if kind in ("step", "graph"):
        c["nb"] = rng.random() < 0.8
        if rng.random() < 0.25:
            c.update(precision="fp64", n=size(1000, 300000))
    elif kind == "batch":
        c.update(n=0, n_sys=size(2, 128), n_lo=1024, n_hi=size(4096, 131072), leaf=8, group=64)
    elif kind == "cycle":
        c["n"] = size(1000, 500000)
    elif kind == "close":
        c["radii"] = rng.choice([0.25, 1.0])  # the paper's own radii are a quarter
    elif kind == "binaries":
        c.update(n=size(1000, 300000), order=rng.choice([2, 3]),
                 binaries=round(rng.uniform(0.1, 1.0), 2))
    elif kind == "eval":
        c.update(n=size(2, 400000), order=rng.choice([2, 3]))
    return c


# --------------------------------------------------------------- inputs
def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV, dtype=F64)


def _isotropic(g, n):
    z = 2.0 * _rand(g, n) - 1.0
    phi = 2.0 * math.pi * _rand(g, n)
    s = torch.sqrt(1.0 - z * z)
    return torch.stack([s * torch.cos(phi), s * torch.sin(phi), z])


def _plummer(g, n):
    """Positions and velocities (3, n) of a Plummer sphere, G = M = 1, virial radius 1."""
    x = 0.999 * _rand(g, n) + 1e-12
    r = 1.0 / torch.sqrt(x ** (-2.0 / 3.0) - 1.0)
    q = torch.linspace(0.0, 1.0, 4097, device=DEV, dtype=F64)  # v/v_esc, g(q) = q^2 (1-q^2)^3.5
    cdf = torch.cumsum(q * q * (1.0 - q * q) ** 3.5, 0)
    cdf = cdf / cdf[-1].clone()
    u = _rand(g, n)
    k = torch.searchsorted(cdf, u).clamp(1, 4096)
    f = (u - cdf[k - 1]) / (cdf[k] - cdf[k - 1]).clamp_min(1e-300)
    v = (q[k - 1] + f.clamp(0.0, 1.0) / 4096.0) * math.sqrt(2.0) * (1.0 + r * r) ** -0.25
    scale = 3.0 * math.pi / 16.0
    return r * _isotropic(g, n) * scale, v * _isotropic(g, n) / math.sqrt(scale)


def _masses(g, n, imf):
    """Kroupa masses in [0.08, 150] (slopes 1.3 and 2.3, break at 0.5), sum 1."""
    if not imf:
        return torch.full((n,), 1.0 / n, device=DEV, dtype=F64)

    def power(a, lo, hi):
        p, q = lo ** (1.0 - a), hi ** (1.0 - a)
        return p, q - p, 1.0 / (1.0 - a)

    lo, hi = power(1.3, 0.08, 0.5), power(2.3, 0.5, 150.0)
    w1, w2 = lo[1] * lo[2], 0.5 * hi[1] * hi[2]
    u, pick = _rand(g, n), _rand(g, n) < w1 / (w1 + w2)
    m = torch.where(pick, (lo[0] + u * lo[1]) ** lo[2], (hi[0] + u * hi[1]) ** hi[2])
    return m / m.sum()


def _cluster(n, seed, binaries, imf, a_max=1e-2):
    """pos, vel (3, n), mass (n,) and the members (2, n_bin) of the binaries."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    n_bin = min(int(round(0.5 * binaries * n)), n // 2)
    n_single = n - 2 * n_bin
    m = _masses(g, n, imf)
    cpos, cvel = _plummer(g, n - n_bin)
    pos, vel = cpos[:, :n_single], cvel[:, :n_single]
    if n_bin:
        m1, m2 = m[n_single:n_single + n_bin], m[n_single + n_bin:]
        mt = m1 + m2
        a = torch.exp(math.log(1e-5) + (math.log(a_max) - math.log(1e-5)) * _rand(g, n_bin))
        e = 0.999 * torch.sqrt(_rand(g, n_bin))
        anom = 2.0 * math.pi * _rand(g, n_bin)
        E = anom + e * torch.sin(anom)
        for _ in range(30):  # Kepler's equation
            E = E - (E - e * torch.sin(E) - anom) / (1.0 - e * torch.cos(E))
        c, s, b = torch.cos(E), torch.sin(E), a * torch.sqrt(1.0 - e * e)
        w = torch.sqrt(mt / a ** 3) / (1.0 - e * c)
        x = _isotropic(g, n_bin)
        y = torch.linalg.cross(x, _isotropic(g, n_bin), dim=0)
        y = y / torch.linalg.norm(y, dim=0)
        dr, dv = a * (c - e) * x + b * s * y, w * (b * c * y - a * s * x)
        p, v = cpos[:, n_single:], cvel[:, n_single:]
        f1, f2 = m2 / mt, m1 / mt
        pos = torch.cat([pos, p - f1 * dr, p + f2 * dr], 1)
        vel = torch.cat([vel, v - f1 * dv, v + f2 * dv], 1)
    perm = torch.randperm(n, generator=g, device=DEV)
    where = torch.empty_like(perm)
    where[perm] = torch.arange(n, device=DEV)
    pairs = torch.stack([where[n_single:n_single + n_bin], where[n_single + n_bin:]])
    return (pos[:, perm].contiguous(), vel[:, perm].contiguous(), m[perm].contiguous(),
            pairs.to(torch.int32).contiguous())


def _r_out_ref(n):
    return 0.02 * (65536.0 / n) ** (1.0 / 3.0)


def _radii(mass, r_out_ref, vel=None, cr_dt=0.0):
    s = (mass / mass.mean()).clamp_min(1.0) ** (1.0 / 3.0)
    r_out = s * r_out_ref
    r_s = 1.2 * r_out if vel is None else r_out + cr_dt * torch.linalg.norm(vel, dim=0)
    return (0.1 * r_out).contiguous(), r_out.contiguous(), r_s.contiguous()


def _sizes(case):
    """System sizes of a batch, log-uniform; the same for every seed (buffers keep their shapes)."""
    g = torch.Generator()
    g.manual_seed(7919 + case["n_sys"])
    lo, hi = math.log(case["n_lo"]), math.log(case["n_hi"])
    u = torch.rand(case["n_sys"], generator=g, dtype=F64).tolist()
    return [int(round(math.exp(lo + (hi - lo) * x))) for x in u]


def _inputs(case, seed):
    """The particles (and, for a batch, the system offsets) of a case."""
    if case["kind"] == "batch":
        offs, parts = [0], []
        for k, n in enumerate(_sizes(case)):
            p, v, m, _ = _cluster(n, seed * 1009 + k, case["binaries"], case["imf"])
            parts.append((p, v, m) + _radii(m, _r_out_ref(n)))
            offs.append(offs[-1] + n)
        cols = [torch.cat(c, -1).contiguous() for c in zip(*parts)]
        return dict(pos=cols[0], vel=cols[1], mass=cols[2], radii=tuple(cols[3:]), offs=offs)
    n = case["n"]
    ro = _r_out_ref(n)
    a_max = 0.05 * ro if case["kind"] == "binaries" else 1e-2
    pos, vel, mass, pairs = _cluster(n, seed, case["binaries"], case["imf"], a_max)
    if case["kind"] == "close":  # eq. rnb: C_r = 3, dt = r_out/(10 sigma), sigma = 0.41
        ro *= case["radii"]
        radii = _radii(mass, ro, vel, 3.0 * ro / 4.1)
    else:
        radii = _radii(mass, ro)
    return dict(pos=pos, vel=vel, mass=mass, pairs=pairs, radii=radii, r_out_ref=ro, offs=None)


def _eval_inputs(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    n, k = case["n"], 6 if case["order"] == 2 else 16
    n_pair = max(1, n // 2)
    frame = torch.cat([_plummer(g, n_pair)[0], (1e-4 * (1.0 + _rand(g, n_pair)))[None]])
    tensor = 2.0 * _rand(g, 4 + k, n_pair) - 1.0
    pair_of = (torch.arange(n, device=DEV) // 2).clamp_max(n_pair - 1).to(torch.int32)
    pos = frame[:3, pair_of.long()] + 1e-4 * (2.0 * _rand(g, 3, n) - 1.0)
    return tensor.contiguous(), frame.contiguous(), pair_of, pos.contiguous()


# ---------------------------------------------------------------- cases
def _context(case):
    ctx = pt.petar_create(0)
    prec = pt.PETAR_FP64 if case["precision"] == "fp64" else pt.PETAR_MIXED
    pt.petar_set_params(ctx, precision=prec, i_per_lane=case["ipl"])
    return ctx


def prepare(case, seed):
    ctx = _context(case)
    kind, st = case["kind"], {"case": case, "ctx": ctx}
    if kind == "eval":
        tensor, frame, pair_of, pos = _eval_inputs(case, seed)
        n = case["n"]
        st.update(tensor=tensor, frame=frame, pair_of=pair_of, pos=pos,
                  acc=torch.zeros((3, n), dtype=F64, device=DEV),
                  pot=torch.zeros(n, dtype=F64, device=DEV))
        return st
    st.update(_inputs(case, seed))
    n = st["mass"].shape[0]
    if case["nb"] and kind in ("step", "cycle", "close"):
        st["idx"] = torch.zeros(64 * n, dtype=torch.int32, device=DEV)
    if kind in ("cycle", "close"):
        for name in ("clusters", "groups"):
            st[name + "_offsets"] = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        st["groups_pairs"] = torch.zeros((n, 2), dtype=torch.int32, device=DEV)
    if kind == "close":
        pt.petar_tree_build(ctx, st["pos"], st["mass"], case["theta"], case["leaf"])
        _, _, st["lists"] = pt.force_long_with_retry(ctx, case["group"], *st["radii"],
                                                     nb_capacity=64 * n)
    elif kind in ("graph", "batch"):  # a replayed step keeps its output buffers
        st.update(acc=torch.empty((3, n), dtype=F64, device=DEV),
                  pot=torch.empty(n, dtype=F64, device=DEV))
        if case["nb"]:
            st["out_nb"] = (torch.empty(n + 1, dtype=torch.int64, device=DEV),
                            torch.zeros(64 * n, dtype=torch.int32, device=DEV))
    return st


def _keep(st, name, x):
    """An output whose length varies (a list, cluster offsets, pairs), at the front of the
    program's own array for it."""
    st[name][:x.shape[0]].copy_(x)
    return st[name]


def _components(st, name, out):
    """Label, offsets and members of clusters or groups (and the bound pairs of the latter)."""
    got = {name + "_label": out[0], name + "_offsets": _keep(st, name + "_offsets", out[1]),
           name + "_members": out[2]}
    if len(out) > 3:
        got[name + "_pairs"] = _keep(st, name + "_pairs", out[3].T)
    return got


def run(st):
    case, ctx, kind = st["case"], st["ctx"], st["case"]["kind"]
    if kind == "eval":
        return pt.petar_tidal_eval(ctx, case["order"], st["tensor"], st["frame"], st["pair_of"],
                                   st["pos"], st["acc"], st["pot"])
    pos, mass, n = st["pos"], st["mass"], st["mass"].shape[0]
    if kind == "step":
        pt.petar_tree_build(ctx, pos, mass, case["theta"], case["leaf"])
        if not case["nb"]:
            acc, pot = pt.petar_force_long(ctx, case["group"], *st["radii"])
            return {"acc": acc, "pot": pot}
        acc, pot, lists = pt.petar_force_long(ctx, case["group"], *st["radii"],
                                              nb_capacity=64 * n)
        return {"acc": acc, "pot": pot, "offsets": lists[0],
                "idx": _keep(st, "idx", lists[1])}
    if kind in ("graph", "batch"):
        nb = st.get("out_nb")
        pt.petar_step_graph(ctx, pos, mass, case["theta"], case["leaf"], case["group"],
                            *st["radii"], st["acc"], st["pot"], sys_offsets=st["offs"], nb=nb)
        out = {"acc": st["acc"], "pot": st["pot"]}
        if nb is not None:
            out.update(offsets=nb[0], idx=nb[1])
        return out
    if kind == "cycle":
        radii = pt.petar_changeover_radii(ctx, mass, 0.1 * st["r_out_ref"], st["r_out_ref"])
        pt.petar_tree_build(ctx, pos, mass, case["theta"], case["leaf"])
        vel = st["vel"].clone()  # the state before the kick is kept for the step's retry
        acc, pot, lists = pt.petar_force_long(ctx, case["group"], *radii, nb_capacity=64 * n,
                                              kick=(vel, 1.0 / 4096.0))
        kept = pt.petar_nb_filter(ctx, pos, st["vel"], mass, radii[2], 1.5, *lists)
        out = {"acc": acc, "pot": pot, "vel": vel, "r_in": radii[0], "r_out": radii[1],
               "r_search": radii[2]}
    elif kind == "close":
        out, radii, lists = {}, st["radii"], st["lists"]
        kept = pt.petar_nb_filter(ctx, pos, st["vel"], mass, radii[2], 1.5, *lists)
    if kind in ("cycle", "close"):
        out.update(offsets=kept[0], idx=_keep(st, "idx", kept[1]))
        out.update(_components(st, "clusters", pt.petar_clusters(ctx, *kept)))
        out.update(_components(st, "groups", pt.petar_groups(
            ctx, pos, st["vel"], mass, radii[0], case["theta"], *lists)))
        return out
    # binaries: the set in place of the pairs, the field on its targets, the
    # fit, and the kick of every star
    art = pt.petar_artificial_make(ctx, pos, st["vel"], mass, *st["radii"], st["pairs"],
                                   case["order"])
    pt.petar_tree_build(ctx, art["pos"], art["mass"], case["theta"], case["leaf"])
    pt.petar_set_targets(ctx, art["target"])
    acc_set, pot_set = pt.petar_force_long(ctx, case["group"], art["r_in"], art["r_out"],
                                           art["r_search"])
    tensor, acc, pot = pt.petar_tidal_fit(ctx, art, st["pairs"], acc_set, pot_set, pos)
    vel = pt.petar_kick(ctx, st["vel"].clone(), acc, 1.0 / 4096.0)
    return {"set_pos": art["pos"], "set_mass": art["mass"], "set_src": art["src"],
            "frame": art["frame"], "acc_set": acc_set, "pot_set": pot_set, "tensor": tensor,
            "acc": acc, "pot": pot, "vel": vel}


# ----------------------------------------------------------------- work
def _interactions(n, theta):
    """Cells and particles that act on one target: counted 1340 (theta 0.7), 2940 (0.5) and
    9900 (0.3) at a million stars, 3550 (0.5) at ten million."""
    return min(float(n), max(200.0, 190.0 * math.log2(n) - 860.0) * (0.5 / theta) ** 2.35)


def work(case):
    kind = case["kind"]
    if kind == "eval":
        n, k = case["n"], 6 if case["order"] == 2 else 16
        return {"bytes": 8.0 * (8 + 4 + k / 2) * n, "flops": 60.0 * n}
    if kind == "batch":
        sizes = _sizes(case)
    else:
        sizes = [case["n"]]
    n = sum(sizes)
    flops = 23.0 * sum(s * _interactions(s, case["theta"]) for s in sizes)
    lists = 8.0 * n + 4.0 * 4.0 * n if case["nb"] else 0.0
    if kind == "close":  # lists read twice and written once, stars read, labels and members
        return {"bytes": (64.0 + 3 * 24.0 + 2 * 16.0) * n, "flops": 60.0 * 4.0 * n}
    if kind == "binaries":
        p = 4 if case["order"] == 2 else 8
        n_out = n * (1.0 + 0.5 * case["binaries"] * (p + 2))
        targets = n_out - 1.5 * case["binaries"] * n
        return {"bytes": 80.0 * n + 88.0 * n_out,
                "flops": 23.0 * targets * _interactions(n_out, case["theta"])}
    more = 24.0 * n * 2 + lists + 48.0 * n if kind == "cycle" else 0.0
    return {"bytes": 88.0 * n + lists + more, "flops": flops}


# ---------------------------------------------------------------- exact
_MOST_PAIRS = 2.5e10  # direct sums above this take too long


def _direct(tpos, tr_in, tr_out, spos, smass, sr_in, sr_out, self_at=None):
    """Long-range field and potential at the targets by the direct sum: (3, t), (t,). self_at:
    each target's own place among the sources, -1 for none."""
    n_t, n_s = tpos.shape[1], spos.shape[1]
    acc = torch.empty((3, n_t), dtype=F64, device=DEV)
    pot = torch.empty(n_t, dtype=F64, device=DEV)
    step = max(1, (1 << 25) // n_s)
    for a in range(0, n_t, step):
        b = min(n_t, a + step)
        d = [spos[k][None, :] - tpos[k, a:b, None] for k in range(3)]
        r = torch.sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2])
        ri = torch.maximum(tr_in[a:b, None], sr_in[None, :])
        ro = torch.maximum(tr_out[a:b, None], sr_out[None, :])
        lam = (ro - ri) / (ro + ri)
        x = ((r - ri) / (ro - ri)).clamp(0.0, 1.0)
        x4, y = x ** 4, 1.0 - x
        f = x4 * (35.0 - 84.0 * x + 70.0 * x * x - 20.0 * x ** 3 - 35.0 * lam * y ** 4)
        inside = 2.0 / (ro + ri) - lam * x4 * x * (14.0 - 28.0 * x + 20.0 * x * x
                                                   - 5.0 * x ** 3) / r
        p = torch.where(r >= ro, 1.0 / r, torch.where(r > 0.0, inside, 2.0 / (ro + ri)))
        f = torch.where(r > 0.0, f / r ** 3, torch.zeros_like(r))
        if self_at is not None:
            own = self_at[a:b]
            rows = torch.nonzero(own >= 0)[:, 0]
            f[rows, own[rows]] = 0.0
            p[rows, own[rows]] = 0.0
        f, p = f * smass, p * smass
        for k in range(3):
            acc[k, a:b] = (f * d[k]).sum(1)
        pot[a:b] = -p.sum(1)
    return acc, pot


def _field(pos, mass, radii):
    return _direct(pos, radii[0], radii[1], pos, mass, radii[0], radii[1],
                   torch.arange(mass.shape[0], device=DEV))


def _units(order):
    """Measure points in units of d_c, (P, 3)."""
    if order == 2:
        h = math.sqrt(0.5)
        u = [[1, 0, -h], [-1, 0, -h], [0, 1, h], [0, -1, h]]
    else:
        u = [[x, y, z] for z in (-1, 1) for x, y in ((1, 0), (0, 1), (-1, 0), (0, -1))]
    return torch.tensor(u, dtype=F64, device=DEV)


def _model(order, r):
    """Rows of the tensor model at offsets r (..., 3): (..., 3, K) of first and second order."""
    x, y, z = r[..., 0], r[..., 1], r[..., 2]
    o = torch.zeros_like(x)
    first = [[x, y, z, o, o, o], [o, x, o, y, z, o], [o, o, x, o, y, z]]
    if order == 2:
        return torch.stack([torch.stack(row, -1) for row in first], -2), None
    xx, yy, zz, xy, xz, yz = x * x, y * y, z * z, 2 * x * y, 2 * x * z, 2 * y * z
    second = [[xx, xy, xz, yy, yz, zz, o, o, o, o], [o, xx, o, xy, xz, o, yy, yz, zz, o],
              [o, o, xx, o, xy, xz, o, yy, yz, zz]]
    pad = [o] * 6
    one = torch.stack([torch.stack(row + [o] * 10, -1) for row in first], -2)
    return one, torch.stack([torch.stack(pad + row, -1) for row in second], -2)


def _tidal(order, tensor, r):
    """Model field (3, n) and potential (n,) at offsets r (n, 3); tensor (4 + K, n)."""
    one, two = _model(order, r)
    t = tensor[4:].T[:, :, None]
    a0 = tensor[1:4].T
    a1 = (one @ t)[..., 0]
    a2 = (two @ t)[..., 0] if two is not None else torch.zeros_like(a1)
    return (a0 + a1 + a2).T, tensor[0] - (r * (a0 + a1 / 2 + a2 / 3)).sum(1)


def _exact_binaries(case, s):
    order, pos, vel, mass, pairs = case["order"], s["pos"], s["vel"], s["mass"], s["pairs"].long()
    n, n_pair, u = mass.shape[0], pairs.shape[1], _units(case["order"])
    i, j = pairs[0], pairs[1]
    single = torch.ones(n, dtype=torch.bool, device=DEV)
    single[pairs.reshape(-1)] = False
    single = torch.nonzero(single)[:, 0]
    n_p = u.shape[0]
    sources = single.shape[0] + 3 * n_pair
    if (single.shape[0] + (n_p + 1) * n_pair) * sources > _MOST_PAIRS:
        return None
    m = mass[i] + mass[j]
    r, v = pos[:, j] - pos[:, i], vel[:, j] - vel[:, i]
    cm = (mass[i] * pos[:, i] + mass[j] * pos[:, j]) / m
    rr = torch.linalg.norm(r, dim=0)
    a = -m / (2.0 * (0.5 * (v * v).sum(0) - m / rr))
    h = torch.linalg.cross(r, v, dim=0)
    ev = torch.linalg.cross(v, h, dim=0) / m - r / rr
    e = torch.linalg.norm(ev, dim=0)
    ex = ev / e
    ey = torch.linalg.cross(h / torch.linalg.norm(h, dim=0), ex, dim=0)
    d_c = a * (1.0 + e)
    scale = a * torch.sqrt(mass[i] * mass[j]) / m
    b, c = torch.sqrt(3.0 * e * e + 0.75), torch.sqrt(1.0 - e * e)
    pseudo = [cm + scale * (px * ex + py * ey)
              for px, py in ((0.0 * b, c), (b, -0.5 * c), (-b, -0.5 * c))]
    points = [cm] + [cm + d_c * u[k][:, None] for k in range(n_p)]
    block = torch.stack(points + pseudo, -1).reshape(3, -1)
    third, zero = m / 3.0, torch.zeros_like(m)
    set_pos = torch.cat([pos[:, single], block], 1)
    set_mass = torch.cat([mass[single],
                          torch.stack([zero] * (n_p + 1) + [third] * 3, -1).reshape(-1)])
    rad = []
    for q in s["radii"][:2]:
        big = torch.maximum(q[i], q[j])
        rad.append(torch.cat([q[single], big[:, None].expand(-1, n_p + 4).reshape(-1)]))
    n_s = single.shape[0]
    at = torch.arange(set_mass.shape[0], device=DEV)
    is_target = (at < n_s) | ((at - n_s) % (n_p + 4) <= n_p)
    is_source = set_mass > 0.0
    place = torch.cumsum(is_source, 0) - 1
    place[~is_source] = -1
    ta, tp = _direct(set_pos[:, is_target], rad[0][is_target], rad[1][is_target],
                     set_pos[:, is_source], set_mass[is_source], rad[0][is_source],
                     rad[1][is_source], place[is_target])
    acc_set = torch.zeros_like(set_pos)
    pot_set = torch.zeros_like(set_mass)
    acc_set[:, is_target] = ta
    pot_set[is_target] = tp
    at_p = acc_set[:, n_s:].reshape(3, n_pair, n_p + 4)
    a0 = at_p[:, :, 0]
    diff = (at_p[:, :, 1:n_p + 1] - a0[:, :, None]).permute(1, 2, 0).reshape(n_pair, -1)
    one, two = _model(order, u)
    design = (one if two is None else one + two).reshape(3 * n_p, -1)
    coef = torch.linalg.pinv(design) @ diff.T
    coef[:6] /= d_c
    coef[6:] /= d_c * d_c
    tensor = torch.cat([pot_set[n_s:].reshape(n_pair, -1)[:, 0][None], a0, coef])
    acc, pot = torch.empty_like(pos), torch.empty_like(mass)
    acc[:, single], pot[single] = acc_set[:, :n_s], pot_set[:n_s]
    for mem in (i, j):
        acc[:, mem], pot[mem] = _tidal(order, tensor, (pos[:, mem] - cm).T)
    # the tensor's coefficients divide the field's differences by d_c and d_c^2, which magnifies
    # the tree's truncation past any use of the direct sum as their reference
    return {"set_pos": set_pos, "set_mass": set_mass, "set_src": None,
            "frame": torch.cat([cm, d_c[None]]), "acc_set": acc_set, "pot_set": pot_set,
            "tensor": None, "acc": acc, "pot": pot, "vel": vel + acc / 4096.0}


def exact(case, seed):
    kind = case["kind"]
    if kind == "eval":
        tensor, frame, pair_of, pos = _eval_inputs(case, seed)
        k = pair_of.long()
        return _tidal(case["order"], tensor[:, k], (pos - frame[:3, k]).T)
    if kind == "close":
        return None  # lists, labels and members: whole numbers only
    if kind != "batch" and kind != "binaries" and case["n"] ** 2 > _MOST_PAIRS:
        return None
    if kind == "batch" and sum(float(n) ** 2 for n in _sizes(case)) > _MOST_PAIRS:
        return None
    s = _inputs(case, seed)
    if kind == "binaries":
        return _exact_binaries(case, s)
    offs = s["offs"] or [0, case["n"]]
    parts = [_field(s["pos"][:, a:b], s["mass"][a:b], [q[a:b] for q in s["radii"]])
             for a, b in zip(offs[:-1], offs[1:])]
    out = {"acc": torch.cat([p[0] for p in parts], 1), "pot": torch.cat([p[1] for p in parts])}
    if kind == "cycle":
        out.update(vel=s["vel"] + out["acc"] / 4096.0, r_in=s["radii"][0], r_out=s["radii"][1],
                   r_search=s["radii"][2])
    return out
