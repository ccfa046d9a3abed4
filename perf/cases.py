"""The evaluations whose speed and accuracy this framework is held to.

A case is a dict of plain values: a way of calling the library (`call`), the
sizes, the point distribution and the options that go into the call.

  plan     geometry fixed once (`Plan`), charges change from call to call: the
           matrix-vector product of an iterative solver or of a fixed grid
  oneshot  `potential`: the particles have moved, so trees, lists and potentials
           are all made in the call (one step of a particle simulation)
  direct   `direct`: all pairs, for a sample of targets (how the error of a
           treecode run is checked) or for systems too small for a tree
  batch    `Batch`: many independent systems with 16 charge vectors each

`listed()` gives the fixed cases, `draw()` more of the same ranges, `prepare()`
what a program holds before the call, `run()` one call, `work()` the bytes and
operations that a call cannot do without and `exact()` the potentials by the
direct sum in 64 bits.
"""
import math

import torch

import paper_2003_01836_amd as bltc

DEVICE = "cuda:0"

# Pairs of the direct sum that exact() forms (about 130 bytes of memory traffic
# each): beyond this many it gives no value.
EXACT_PAIRS = 1.8e11


def _case(call, **kw):
    case = dict(call=call, nt=0, ns=10000, m=1, dist="cube", kernel="coulomb", kappa=0.0,
                delta=0.0, precision="fp64", method="bltc", degree=8, theta=0.7, leaf=2000,
                threads=1, systems=1)
    case.update(kw)
    return case


def listed():
    return [
        # a few hundred to a few thousand bodies: the launches and their gaps are the time
        _case("plan", name="plan-1500", ns=1500, degree=4, leaf=200),
        # ten thousand moving bodies, everything rebuilt: the size of a small simulation
        _case("oneshot", name="oneshot-10k", ns=10007, degree=4, leaf=500),
        # an ordinary solver iteration in mixed precision, threads per target as tuned there
        _case("plan", name="plan-100k-mixed", ns=100003, degree=6, leaf=1000,
              precision="fp32_mixed", threads=4),
        # the headline: 10^6 uniform particles, FP64
        _case("plan", name="plan-1M-fp64", ns=1000000, threads=4),
        # a million moving particles in mixed precision: setup and evaluation of the headline
        _case("oneshot", name="oneshot-1M-mixed", ns=1000000, precision="fp32_mixed"),
        # three charge vectors on the same points (the components of a vector potential)
        _case("plan", name="vectors-3", ns=150001, m=3),
        # screened interaction on a centrally condensed distribution
        _case("plan", name="yukawa-plummer", ns=200003, dist="plummer", kernel="yukawa",
              kappa=0.5, degree=6),
        # targets of their own, fewer than the sources, softened kernel: field at probe points
        _case("plan", name="probes-softened", nt=30011, ns=400009, kernel="regularized",
              delta=0.02, degree=6, leaf=1500),
        # both sides interpolated
        _case("plan", name="cluster-cluster", ns=300007, method="cc"),
        # Hermite interpolation, mixed precision
        _case("plan", name="hermite-mixed", ns=200003, method="hermite", degree=4,
              precision="fp32_mixed"),
        # several systems of different sizes, 16 charge vectors each, one queue
        _case("batch", name="batch-16", ns=100000, m=16, systems=8, leaf=1000, degree=6,
              precision="fp32_mixed"),
        # reference potentials at a thousand sampled targets of a large run
        _case("direct", name="direct-sample", nt=1000, ns=2000003),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tree_options(rng, case):
    """Degree, leaf capacity and MAC parameter in the ranges of the tests and the benchmark."""
    if case["method"] == "hermite":
        case["degree"] = rng.randint(2, 4)
        least = 8 * (case["degree"] + 1) ** 3
    else:
        case["degree"] = rng.randint(3, 9)
        least = (case["degree"] + 1) ** 3
    case["leaf"] = max(200, min(4000, int(least * rng.uniform(1.1, 3.0))))
    case["theta"] = rng.choice([0.6, 0.7, 0.8])
    return case


def _kernel_options(rng, case):
    case["kernel"] = rng.choice(["coulomb", "coulomb", "coulomb", "yukawa", "regularized"])
    if case["kernel"] == "yukawa":
        case["kappa"] = rng.choice([0.1, 0.5, 2.0])
    if case["kernel"] == "regularized":
        case["delta"] = rng.choice([0.005, 0.02])
    return case


def draw(rng):
    call = rng.choice(["plan", "plan", "plan", "vectors", "oneshot", "oneshot", "batch", "direct"])
    dist = rng.choice(["cube", "cube", "plummer"])
    precision = rng.choice(["fp64", "fp64", "fp32_mixed"])
    if call == "direct":
        case = _case("direct", nt=_log_uniform(rng, 100, 20000), ns=_log_uniform(rng, 1000, 1000000),
                     m=rng.choice([1, 1, 2, 3]), dist=dist)
        return _kernel_options(rng, case)
    if call == "batch":
        case = _case("batch", ns=_log_uniform(rng, 10000, 60000), m=rng.choice([2, 4, 16]),
                     systems=rng.randint(2, 8), dist=dist, precision=precision)
        return _kernel_options(rng, _tree_options(rng, case))
    if call == "vectors":
        case = _case("plan", ns=_log_uniform(rng, 2000, 100000), m=rng.randint(2, 16), dist=dist,
                     precision=precision)
        return _kernel_options(rng, _tree_options(rng, case))
    method = rng.choice(["bltc", "bltc", "bltc", "cp", "cc", "hermite"])
    case = _case(call, ns=_log_uniform(rng, 1000, 200000), dist=dist, precision=precision,
                 method=method)
    case = _kernel_options(rng, _tree_options(rng, case))
    if case["kernel"] == "yukawa":
        case["ns"] = min(case["ns"], 100000 + case["ns"] % 1000)
    if rng.random() < 0.25:
        case["nt"] = _log_uniform(rng, 500, 50000)
    if method in ("bltc", "hermite"):
        case["threads"] = rng.choice([1, 2, 4])
    return case


def _points(gen, n, dist):
    """(3, n) positions: uniform in [-1, 1]^3, or a Plummer sphere (scale 1, cut at r = 10)."""
    u = torch.rand((3, n), dtype=torch.float64, device=DEVICE, generator=gen)
    if dist == "cube":
        return (u * 2.0 - 1.0).contiguous()
    mass = (u[0] * (1000.0 / 101.0 ** 1.5)).clamp_min(1e-300)
    r = 1.0 / torch.sqrt(mass ** (-2.0 / 3.0) - 1.0)
    cos_t = u[1] * 2.0 - 1.0
    sin_t = torch.sqrt((1.0 - cos_t * cos_t).clamp_min(0.0))
    az = u[2] * (2.0 * math.pi)
    return torch.stack([r * sin_t * torch.cos(az), r * sin_t * torch.sin(az), r * cos_t]).contiguous()


def _sizes(case):
    """System sizes of a batch: from ns / 8 to ns, evenly spread over their logarithm, odd."""
    k = case["systems"]
    return [int(case["ns"] * 8.0 ** (i / max(1, k - 1) - 1.0)) | 1 for i in range(k)]


def _inputs(case, seed):
    """One (targets, sources, charges) per system; targets is sources where they coincide."""
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    systems = []
    for n in _sizes(case) if case["call"] == "batch" else [case["ns"]]:
        s = _points(gen, n, case["dist"])
        t = _points(gen, case["nt"], case["dist"]) if case["nt"] else s
        shape = (n,) if case["m"] == 1 else (case["m"], n)
        q = torch.rand(shape, dtype=torch.float64, device=DEVICE, generator=gen) * 2.0 - 1.0
        systems.append((t, s, q))
    return systems


def _kernel(case):
    return dict(kernel=case["kernel"], kappa=case["kappa"], delta=case["delta"])


def _options(case):
    return dict(theta=case["theta"], degree=case["degree"], leaf_size=case["leaf"],
                batch_size=case["leaf"], precision=case["precision"], method=case["method"],
                threads_per_target=case["threads"], **_kernel(case))


def _out(case, t):
    n = t.shape[1]
    return torch.empty((n,) if case["m"] == 1 else (case["m"], n), dtype=torch.float64, device=DEVICE)


def prepare(case, seed):
    systems = _inputs(case, seed)
    state = {"case": case, "systems": systems, "out": [_out(case, t) for t, _, _ in systems]}
    if case["call"] in ("plan", "batch"):
        max_q = case["m"] if case["call"] == "plan" else 16
        state["plans"] = [bltc.Plan(t, s, max_q=max_q, **_options(case)) for t, s, _ in systems]
    if case["call"] == "batch":
        state["batch"] = bltc.Batch(state["plans"])
    return state


def run(state):
    case, systems, out = state["case"], state["systems"], state["out"]
    t, s, q = systems[0]
    if case["call"] == "plan":
        return state["plans"][0].execute(q, out=out[0])
    if case["call"] == "oneshot":
        return bltc.potential(t, s, q, out=out[0], **_options(case))
    if case["call"] == "direct":
        return bltc.direct(t, s, q, out=out[0], **_kernel(case))
    return state["batch"].execute([x[2] for x in systems], out)


def work(case):
    """Each coordinate a call takes, each charge and each potential once; the kernel values of the
    method's lists (a value of two leaves that see each other directly serves both), each with its
    multiply-adds, and the modified charges."""
    per_value = {"coulomb": 10, "yukawa": 13, "regularized": 11}[case["kernel"]]
    m = case["m"]
    total_bytes, flops = 0.0, 0.0
    for t, s, _ in _inputs(case, 0):
        nt, ns = t.shape[1], s.shape[1]
        total_bytes += 8.0 * (3 * ns + m * ns + m * nt + (3 * nt if t is not s else 0))
        if case["call"] == "direct":
            flops += float(nt) * ns * (per_value + 2 * (m - 1))
            continue
        plan = bltc.Plan(t, s, max_q=max(m, 16 if case["call"] == "batch" else 1), **_options(case))
        st = plan.stats()
        plan.close()
        far = float(st["far_evals"])
        if case["method"] == "hermite":
            flops += far / 8 * 37
        else:
            flops += far * (per_value + 2 * (m - 1))
        once = float(st["near_evals"] - st["mutual_pair_evals"])
        flops += once * per_value + 2.0 * st["mutual_pair_evals"] + once * 2 * (m - 1)
        flops += 2.0 * m * st["upward_terms"]
    return {"bytes": total_bytes, "flops": flops}


def _direct_sum(case, t, s, q):
    """Potentials of the charges q (vectors by rows) by the direct sum in 64 bits, pairs at zero
    distance left out."""
    n = s.shape[1]
    q2 = (q if q.dim() == 2 else q.unsqueeze(0)).t().contiguous()
    phi = torch.empty((t.shape[1], q2.shape[1]), dtype=torch.float64, device=DEVICE)
    step = max(1, (1 << 28) // max(1, n))
    for i in range(0, t.shape[1], step):
        x = t[:, i:i + step]
        r2 = x[0][:, None] - s[0][None, :]
        r2.mul_(r2)
        for l in (1, 2):
            d = x[l][:, None] - s[l][None, :]
            r2.addcmul_(d, d)
        r2.masked_fill_(r2 == 0.0, math.inf)
        if case["kernel"] == "regularized":
            g = r2.add_(case["delta"] ** 2).rsqrt_()
        elif case["kernel"] == "yukawa":
            g = torch.exp(-case["kappa"] * r2.sqrt()).mul_(r2.rsqrt_())
        else:
            g = r2.rsqrt_()
        phi[i:i + step] = g @ q2
    phi = phi.t().contiguous()
    return phi if q.dim() == 2 else phi[0]


def exact(case, seed):
    systems = _inputs(case, seed)
    if sum(float(t.shape[1]) * s.shape[1] for t, s, _ in systems) > EXACT_PAIRS:
        return None
    got = [_direct_sum(case, *x) for x in systems]
    return got if case["call"] == "batch" else got[0]
