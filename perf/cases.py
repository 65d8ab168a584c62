"""The work that programs have this library do, as measurable cases.

A case is one pass through the public calls of `paper_1802_04434_amd`: an optimisation step over a
d-parameter model held by M workers (in one call, or as pack / vote / apply), the server's side
alone, or the gradient statistics.  Sizes are those of the repository's five workloads, of a
gradient bucket, and everything between; the arithmetic is fixed to the last bit by the library's
header, so nearly every case is compared exactly.
"""
import math

import torch

import paper_1802_04434_amd as ss

BETA, DELTA, TAU, QUORUM = 0.9, 1e-4, 0.05, 2
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(name, kind, d, M, dtype="f32", momentum=True, packed=False, scheme="majority"):
    return {"name": name, "kind": kind, "d": d, "M": M, "dtype": dtype, "momentum": momentum, "packed": packed,
            "scheme": scheme}


def listed():
    return [
        # the smallest model of the repository (ResNet-20 sized), 7 workers: launches and latency count
        _case("step_tiny_f32", "step", 272_474, 7),
        # one 25 MB bucket of a larger model, stepped on its own; bf16 gradients, odd length
        _case("step_bucket_bf16", "step", 6_553_613, 8, dtype="bf16"),
        # the headline workload: Signum with majority vote over a ResNet-50 sized model
        _case("step_resnet50_f32", "step", 25_557_032, 7),
        # many workers and a vector beyond every cache (VGG sized)
        _case("step_16_workers_f32", "step", 138_357_544, 16),
        # the largest: bf16 gradients with fp32 momentum and master parameters, ragged end
        _case("step_large_bf16", "step", 400_000_017, 8, dtype="bf16"),
        # Algorithm 1: signSGD on one worker
        _case("signsgd_one_worker_f32", "step", 25_557_032, 1, momentum=False),
        # Algorithm 3 literally: vote over the signs of the gradients, no momentum
        _case("signsgd_vote_bf16", "step", 25_557_032, 8, dtype="bf16", momentum=False),
        # the same step by the paper's roles: every worker packs, the server votes, the worker applies
        _case("calls_resnet50_f32", "calls", 25_557_032, 7),
        # the step for a caller that also wants every worker's sign bits
        _case("step_packed_f32", "step", 25_557_032, 7, packed=True),
        # vote with abstention, one call
        _case("ternary_step_f32", "ternary_step", 25_557_032, 7),
        # the server alone: 16 packed sign vectors in, one out
        _case("server_vote_16", "server", 138_357_544, 16),
        # gradient statistics of Figure 1: running mean / variance, sigma, and the density of both
        _case("statistics_f32", "stats", 25_557_032, 1),
    ]


MOST_BYTES = 27e9


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "calls", "sum_step", "ternary_step", "server", "server", "stats"])
    d = int(math.exp(rng.uniform(math.log(3_000), math.log(400_000_000))))
    d += rng.choice([0, 1, 3, 17]) if rng.random() < 0.7 else -(d % 1024)
    M = 1 if kind == "stats" else rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 15, 16, 24])
    case = {"kind": kind, "d": max(d, 1), "M": M, "dtype": rng.choice(["f32", "bf16"]),
            "momentum": kind == "stats" or rng.random() < 0.75, "packed": kind == "step" and rng.random() < 0.3,
            "scheme": rng.choice(["majority", "sum", "quorum"]) if kind == "server" else "majority"}
    most = MOST_BYTES / (work(case)["bytes"] / case["d"])
    if case["d"] > most:
        case["d"] = int(most) - rng.randrange(1000)
    return case


def _bytes_per_coordinate(case):
    M, kind = case["M"], case["kind"]
    grad = 4 if case["dtype"] == "f32" else 2
    if kind == "stats":
        return grad + 16 + 8 + 4 + 4                 # g, mean, m2 in; mean, m2, sigma out; two densities
    if kind == "server":
        return {"majority": (M + 1) / 8, "sum": M / 8 + 1, "quorum": (2 * M + 2) / 8}[case["scheme"]]
    step = M * (grad + (8 if case["momentum"] else 0)) + 8 + 0.125
    if case["packed"] or kind == "calls":
        step += M / 8
    return step + {"sum_step": 1, "ternary_step": 0.125}.get(kind, 0)


def work(case):
    d, M = case["d"], case["M"]
    flops = {"stats": 12, "server": 0.2 * M}.get(case["kind"], M * (4 if case["momentum"] else 1) + 2)
    return {"bytes": _bytes_per_coordinate(case) * d, "flops": flops * d}


def tolerance(case):
    # every rounding is fixed by the header; the density's fp64 sums may be added in another order
    return {"rel": 1e-11} if case["kind"] == "stats" else "exact"


# ------------------------------------------------------------------ inputs ----

def _planes(case, gen):
    """packed words of random votes with the unused bits at zero; about a quarter of them abstentions"""
    d, n = case["d"], ss.packed_bytes(case["d"]) // 4

    def words():
        w = torch.randint(-2**31, 2**31, (n,), dtype=torch.int32, device="cuda", generator=gen)
        w[(d + 31) // 32:] = 0
        if d % 32:
            w[d // 32] &= (1 << (d % 32)) - 1
        return w

    neg = [words() for _ in range(case["M"])]
    if case["scheme"] != "quorum":
        return neg, None
    zero = [words().bitwise_and_(words()) for _ in range(case["M"])]
    for n_, z in zip(neg, zero):
        n_.bitwise_and_(z.bitwise_not())
    return neg, zero


def prepare(case, seed):
    d, M, kind = case["d"], case["M"], case["kind"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1_000_003 + d * 67 + M)

    def normal(scale):
        return torch.randn(d, device="cuda", generator=gen).mul_(scale)

    def bits():
        return torch.zeros(ss.packed_bytes(d) // 4, dtype=torch.int32, device="cuda")

    s = {"case": case}
    if kind == "server":
        s["neg"], s["zero"] = _planes(case, gen)
        s["voted"] = bits()
        if case["scheme"] == "sum":
            s["sums"] = torch.zeros(d, dtype=torch.int8, device="cuda")
        if case["scheme"] == "quorum":
            s["voted_zero"] = bits()
        return s
    mu = normal(0.1)
    if kind == "stats":
        s["g"] = normal(0.5).add_(mu).to(DTYPES[case["dtype"]])
        s["mean"] = normal(0.2).add_(mu)
        s["m2"] = normal(0.5).square_().mul_(6)
        s["sigma"] = torch.zeros(d, device="cuda")
        s["n"] = 7
        s["out"] = [torch.zeros(3, dtype=torch.float64, device="cuda") for _ in range(2)]
        s["workspace"] = ss.new_density_workspace("cuda")
        return s
    # gradients around a common mean; about 5 % exact zeros where there is no momentum to spread them
    s["g"], s["m"] = [], [] if case["momentum"] else None
    for _ in range(M):
        g = normal(0.5).add_(mu)
        if not case["momentum"]:
            g.mul_(g.abs() > 0.03)
        s["g"].append(g.to(DTYPES[case["dtype"]]))
        if case["momentum"]:
            s["m"].append(normal(0.115).add_(mu))
    s["x"] = normal(0.05)
    s["voted"] = bits()
    if case["packed"] or kind == "calls":
        s["packed"] = [bits() for _ in range(M)]
    if kind == "sum_step":
        s["sums"] = torch.zeros(d, dtype=torch.int8, device="cuda")
    if kind == "ternary_step":
        s["voted_zero"] = bits()
    return s


# -------------------------------------------------------------------- pass ----

def run(state):
    s, case = state, state["case"]
    kind, d = case["kind"], case["d"]
    if kind == "server":
        if case["scheme"] == "sum":
            return {"sums": ss.vote_sum(s["neg"], s["sums"], d)}
        if case["scheme"] == "quorum":
            ss.quorum_vote(s["neg"], s["zero"], QUORUM, s["voted"], s["voted_zero"], d)
            return {"voted": s["voted"], "voted_zero": s["voted_zero"]}
        return {"voted": ss.majority_vote(s["neg"], s["voted"], d)}
    if kind == "stats":
        ss.welford_update(s["g"], s["mean"], s["m2"], s["n"])
        ss.welford_sigma(s["m2"], s["n"], s["sigma"])
        ss.density(s["mean"], s["out"][0], s["workspace"])
        ss.density(s["sigma"], s["out"][1], s["workspace"])
        s["n"] += 1
        return {"mean": s["mean"], "m2": s["m2"], "sigma": s["sigma"], "density": s["out"]}
    out = {"m": s["m"], "x": s["x"], "voted": s["voted"]}
    if kind == "calls":
        for w, g in enumerate(s["g"]):
            ss.signum_pack(g, s["m"][w] if s["m"] is not None else None, BETA, s["packed"][w])
        ss.majority_vote(s["packed"], s["voted"], d)
        ss.sign_apply(s["x"], s["voted"], DELTA)
        out["packed"] = s["packed"]
    elif kind == "sum_step":
        ss.signum_vote_step_ex(s["g"], s["m"], BETA, DELTA, s["x"], s["voted"], sums_out=s["sums"],
                               flags=ss.STEP_SUM_UPDATE)
        out["sums"] = s["sums"]
    elif kind == "ternary_step":
        ss.signum_vote_step_ternary(s["g"], s["m"], BETA, TAU, QUORUM, DELTA, s["x"], s["voted"], s["voted_zero"])
        out["voted_zero"] = s["voted_zero"]
    else:
        ss.signum_vote_step(s["g"], s["m"], BETA, DELTA, s["x"], s["voted"], s.get("packed"))
        if case["packed"]:
            out["packed"] = s["packed"]
    return out


# ----------------------------------------------------- the same in 64 bits ----

def _f32(v):
    return float(torch.tensor(v, dtype=torch.float32))


def _pack(neg):
    """bool per coordinate -> words, 32 coordinates each, least significant bit first"""
    d = neg.numel()
    words = torch.zeros(ss.packed_bytes(d) * 8, dtype=torch.bool, device=neg.device)
    words[:d] = neg
    words = words.view(-1, 32)
    out = torch.zeros(words.shape[0], dtype=torch.int32, device=neg.device)
    for k in range(32):
        out |= words[:, k].to(torch.int32) << k
    return out


def _unpack(words, d):
    out = torch.empty(words.numel(), 32, dtype=torch.bool, device=words.device)
    for k in range(32):
        out[:, k] = ((words >> k) & 1).bool()
    return out.view(-1)[:d]


def _density(v):
    l1, l2 = v.abs().sum(), v.square().sum()
    return torch.stack([l1, l2, l1 * l1 / (v.numel() * l2)])


def exact(case, seed):
    s = prepare(case, seed)
    kind, d, M = case["kind"], case["d"], case["M"]
    if kind == "server":
        minus = torch.zeros(d, dtype=torch.int32, device="cuda")
        silent = torch.zeros(d, dtype=torch.int32, device="cuda")
        for w in range(M):
            minus += _unpack(s["neg"][w], d)
            if s["zero"] is not None:
                silent += _unpack(s["zero"][w], d)
        total = M - silent - 2 * minus
        if case["scheme"] == "sum":
            return {"sums": total.to(torch.int8)}
        if case["scheme"] == "quorum":
            return {"voted": _pack(total <= -QUORUM), "voted_zero": _pack(total.abs() < QUORUM)}
        return {"voted": _pack(total < 0)}
    if kind == "stats":
        g, n = s["g"].double(), s["n"]
        delta = g - s["mean"].double()
        mean = s["mean"].double() + delta / n
        m2 = s["m2"].double() + delta * (g - mean)
        sigma = (m2 / n).sqrt()
        return {"mean": mean, "m2": m2, "sigma": sigma, "density": [_density(mean), _density(sigma)]}
    beta, delta, tau = _f32(BETA), _f32(DELTA), _f32(TAU)
    total = torch.zeros(d, dtype=torch.int32, device="cuda")
    ms, packed = [] if case["momentum"] else None, []
    for w in range(M):
        v = s["g"][w].double()
        if case["momentum"]:
            v = beta * s["m"][w].double() + (1 - beta) * v
            ms.append(v)
        vote = 1 - 2 * (v < 0).to(torch.int32)
        if kind == "ternary_step":
            vote *= v.abs() >= tau
        total += vote
        if "packed" in s:
            packed.append(_pack(v < 0))
        s["g"][w] = None
        if case["momentum"]:
            s["m"][w] = None
    out = {"m": ms}
    if kind == "ternary_step":
        answer = total.sign() * (total.abs() >= QUORUM)
        out.update(voted=_pack(answer < 0), voted_zero=_pack(answer == 0))
    else:
        answer = 1 - 2 * (total < 0).to(torch.int32)
        out["voted"] = _pack(answer < 0)
        if kind == "sum_step":
            answer = total
            out["sums"] = total.to(torch.int8)
    out["x"] = s["x"].double() - delta * answer.double()
    if packed:
        out["packed"] = packed
    return out
