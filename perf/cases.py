"""The routing calls whose speed counts, as a program that serves a mixture-of-experts model
makes them: sizes, inputs, one pass, the work it cannot do without, and how far two correct
results may be apart.

Inputs follow the seeded recipe of the benchmark's workloads, drawn on the GPU: a gate matrix
W ~ N(0, 0.02^2), hidden rows sigma_t g_t + pinv(W) b_t with g_t ~ N(0, I), so that a row's
logits are a chosen bias b_t plus natural noise.  What the bias is ("gate" of a case):

  zipf     expert popularity falls like rank^-1.1, a rank map per layer (a skewed gate)
  decode   the same with a temperature per token out of {0.3, 1, 3}
  peaked   half of the rows have one random expert far ahead, the others have none
  mixed    rank^-1.3 popularity, a share `flat` of the rows with nearly equal scores

How many tokens depend on the load counters follows from the gate and the thresholds
(eps_high, t_fix), which are those of the paper's table for the two kinds of model, or, where
every token is to take the load-aware branch, eps_high = 2 with t_fix = 1e-30.

Outputs are the call's own buffers, whole: expert ids, weights, permutation, offsets and the
counters after the last token.
"""
import math

import torch

from paper_2510_03293_amd import binding as B

ALL_TOKENS = (2.0, 1e-30)   # thresholds that make every token load-dependent


def listed():
    return [
        # One decode step of one layer: 64 sequences, counters carried from step to step.  The
        # smallest call, bound by latency and launches.
        dict(name="decode", kind="call", T=64, H=2048, E=64, k=6, c=8, layers=1, gate="decode",
             flat=0.0, eps=0.40, tfix=0.80, carry=True),
        # The same step through all layers of the model, replayed from a HIP graph, which is how
        # a serving loop runs it.
        dict(name="decode_graph", kind="graph", T=64, H=2048, E=64, k=6, c=8, layers=27, gate="decode",
             flat=0.0, eps=0.40, tfix=0.80, carry=True),
        # Sixteen decode-sized problems that are at hand together (micro-batches in flight at
        # different layers) in one batched call.
        dict(name="batched_decode", kind="batched", T=64, H=2048, E=64, k=6, c=8, layers=16, gate="decode",
             flat=0.0, eps=0.40, tfix=0.80, carry=True),
        # A chunk of a prompt: an odd number of rows, a tenth of them load-dependent, counters
        # carried from chunk to chunk.
        dict(name="chunk", kind="call", T=3001, H=2048, E=64, k=6, c=8, layers=1, gate="mixed",
             flat=0.10, eps=0.40, tfix=0.80, carry=True),
        # The benchmark's headline: a 16K-token batch through all 27 layers of the 64-expert
        # model, counters cleared before the pass.  Nearly every token keeps its top-k.
        dict(name="layers_64_experts", kind="call", T=16384, H=2048, E=64, k=6, c=8, layers=27, gate="zipf",
             flat=0.0, eps=0.40, tfix=0.80, carry=False),
        # The 8-expert model, four layers: about a tenth of the tokens is load-dependent, and
        # they compete for the same few experts.
        dict(name="layers_8_experts", kind="call", T=16384, H=4096, E=8, k=2, c=4, layers=4, gate="peaked",
             flat=0.0, eps=0.6419, tfix=0.60, carry=False),
        # A long prefill, one layer of 1 GiB of hidden states.
        dict(name="prefill", kind="call", T=131072, H=4096, E=64, k=6, c=8, layers=1, gate="mixed",
             flat=0.10, eps=0.40, tfix=0.80, carry=False),
        # Calibration: the per-token statistics of the gate scores beside the routing.
        dict(name="calibration", kind="stats", T=16384, H=2048, E=64, k=6, c=8, layers=1, gate="zipf",
             flat=0.0, eps=0.40, tfix=0.80, carry=False),
        # A program with a gate of its own hands over logits; trimming is randomized, thresholds
        # are those of the table's reasoning rows, and a tenth of the tokens is sampled.
        dict(name="logits_random", kind="logits", T=12345, H=0, E=64, k=6, c=8, layers=1, gate="mixed",
             flat=0.10, eps=0.30, tfix=0.55, carry=False, random=True),
        # Balance before everything: every token takes the load-aware branch with a full working
        # set (the longest chain of decisions that depend on one another).
        dict(name="balance_all", kind="call", T=16384, H=2048, E=64, k=6, c=8, layers=1, gate="zipf",
             flat=0.0, eps=ALL_TOKENS[0], tfix=ALL_TOKENS[1], carry=False),
        # The load-only baseline of the paper's evaluation: all experts are candidates.
        dict(name="load_only", kind="call", T=8192, H=2048, E=64, k=6, c=64, layers=1, gate="zipf",
             flat=0.0, eps=ALL_TOKENS[0], tfix=ALL_TOKENS[1], carry=False),
        # Routers kept in single precision.
        dict(name="fp32", kind="call", T=2048, H=2048, E=64, k=6, c=8, layers=1, gate="zipf",
             flat=0.0, eps=0.40, tfix=0.80, carry=False, fp32=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice([c["name"] for c in listed()])
    E, k, c = rng.choice([(64, 6, 8), (64, 6, 8), (64, 6, 10), (8, 2, 4), (8, 2, 3), (32, 4, 8), (16, 4, 12),
                          (33, 3, 9)])
    H = rng.choice([2048, 2048, 4096, 4096, 1024, 3000, 1536])
    case = dict(kind="call", T=0, H=H, E=E, k=k, c=c, layers=1, gate="mixed",
                flat=round(rng.choice([0.0, rng.uniform(0.01, 0.3)]), 3), eps=0.40, tfix=0.80, carry=False)
    if what == "decode":
        case.update(T=_log(rng, 1, 256), carry=True, gate=rng.choice(["decode", "mixed"]))
    elif what == "decode_graph":
        case.update(kind="graph", T=_log(rng, 1, 256), layers=rng.randint(8, 32), carry=True,
                    gate=rng.choice(["decode", "mixed"]))
    elif what == "batched_decode":
        case.update(kind="batched", T=_log(rng, 1, 256), layers=rng.randint(2, 32), carry=True,
                    gate=rng.choice(["decode", "mixed"]))
    elif what == "chunk":
        case.update(T=_log(rng, 257, 8192), carry=True, gate=rng.choice(["mixed", "zipf"]))
    elif what == "layers_64_experts":
        case.update(T=_log(rng, 4096, 32768), gate="zipf", E=64, k=6, c=rng.choice([8, 10]), flat=0.0)
        case["layers"] = max(1, min(27, 442368 * 2048 // (case["T"] * case["H"]) - 1))
    elif what == "layers_8_experts":
        case.update(T=_log(rng, 4096, 32768), gate="peaked", E=8, k=2, c=rng.choice([3, 4]), flat=0.0,
                    eps=rng.choice([0.7159, 0.6419, 0.6285, 0.75]), tfix=0.60, layers=rng.randint(1, 4))
    elif what == "prefill":
        case.update(T=_log(rng, 40000, 131072))
    elif what == "calibration":
        case.update(kind="stats", T=_log(rng, 2048, 32768), gate=rng.choice(["zipf", "mixed"]))
    elif what == "logits_random":
        case.update(kind="logits", H=0, T=_log(rng, 1000, 65536), random=rng.random() < 0.6)
        if case["random"]:
            case.update(eps=0.30, tfix=rng.choice([0.25, 0.45, 0.55]))
    elif what == "balance_all":
        case.update(T=_log(rng, 1024, 16384), gate=rng.choice(["zipf", "mixed"]), eps=ALL_TOKENS[0],
                    tfix=ALL_TOKENS[1])
    elif what == "load_only":
        E, k = rng.choice([(64, 6), (64, 6), (32, 4), (40, 3)])
        case.update(T=_log(rng, 512, 8192), E=E, k=k, c=E, gate=rng.choice(["zipf", "mixed"]),
                    eps=ALL_TOKENS[0], tfix=ALL_TOKENS[1])
    else:
        case.update(T=_log(rng, 64, 2048), H=rng.choice([128, 512, 1000, 2048]), fp32=True,
                    gate=rng.choice(["zipf", "mixed"]))
    return case


def _gate_bias(case, gen, cpu_gen):
    """(bias [E] or [T,E], sigma None or [T]) of one layer, see the recipe above."""
    T, E = case["T"], case["E"]
    ranks = (torch.randperm(E, generator=cpu_gen) + 1).float().cuda()
    gate = case["gate"]
    if gate == "zipf":
        return -1.1 * torch.log(ranks), None
    if gate == "decode":
        levels = torch.tensor([1 / 0.3, 1.0, 1 / 3.0], device="cuda")
        sigma = levels[torch.randint(0, 3, (T,), generator=gen, device="cuda")]
        return (-1.1 * torch.log(ranks))[None, :] * sigma[:, None], sigma
    if gate == "peaked":
        bias = torch.zeros((T, E), device="cuda")
        rows = torch.randperm(T, generator=cpu_gen)[: T // 2].cuda()
        bias[rows, torch.randint(0, E, (rows.numel(),), generator=gen, device="cuda")] = 3.0
        return bias, None
    natural = 0.02 * math.sqrt(case["H"]) if case["H"] else 1.0
    flat = torch.rand(T, generator=gen, device="cuda") < case["flat"]
    bias = torch.where(flat[:, None], torch.zeros((), device="cuda"), (-1.3 * torch.log(ranks))[None, :])
    return bias, torch.where(flat, 0.05 / natural, 1.0).float()


def _layer(case, gen, cpu_gen, hidden):
    """Fills hidden [T,H] and returns the gate matrix [E,H] of one layer."""
    T, H, E = case["T"], case["H"], case["E"]
    w = (torch.randn((E, H), generator=cpu_gen) * 0.02).to(hidden.dtype)
    w64 = w.double()
    pinv_t = torch.linalg.solve(w64 @ w64.T, w64).float().cuda()        # (W W^T)^-1 W, [E,H]
    bias, sigma = _gate_bias(case, gen, cpu_gen)
    g = torch.randn((T, H), generator=gen, device="cuda")
    if sigma is not None:
        g *= sigma[:, None]
    g += bias @ pinv_t if bias.dim() == 2 else (bias[None, :] @ pinv_t)
    hidden.copy_(g)
    return w.cuda()


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(1000003 * (seed % 1000003) + 17)
    cpu_gen = torch.Generator().manual_seed(1000033 * (seed % 1000003) + 5)
    kind, T, H, E, k, n = case["kind"], case["T"], case["H"], case["E"], case["k"], case["layers"]
    fp32, random = bool(case.get("fp32")), bool(case.get("random"))
    s = {"case": case, "stream": torch.cuda.current_stream()}
    s["params"] = B.make_params(
        k, case["c"], case["eps"], case["tfix"], dtype=B.DTYPE_F32 if fp32 else B.DTYPE_BF16,
        trim_mode=B.TRIM_RANDOM if random else B.TRIM_TOP, seed=seed)
    if kind == "logits":
        bias, sigma = _gate_bias(case, gen, cpu_gen)
        z = torch.randn((T, E), generator=gen, device="cuda")
        s["logits"] = (z * sigma[:, None] if sigma is not None else z) + bias
    else:
        s["hidden"] = torch.empty((n, T, H), dtype=torch.float32 if fp32 else torch.bfloat16, device="cuda")
        s["w"] = torch.stack([_layer(case, gen, cpu_gen, s["hidden"][i]) for i in range(n)])
    # outputs of every layer, one workspace (the layers run one after the other), the counters
    s["ids"] = torch.empty((n, T, k), dtype=torch.int32, device="cuda")
    s["weights"] = torch.empty((n, T, k), dtype=torch.float32, device="cuda")
    s["perm"] = torch.empty((n, T * k), dtype=torch.int32, device="cuda")
    s["offsets"] = torch.empty((n, E + 1), dtype=torch.int32, device="cuda")
    s["loads"] = torch.zeros((n, E), dtype=torch.int32, device="cuda")
    one = B.laser_workspace_bytes(T, H, E, s["params"])
    s["workspace"] = torch.empty(one * (n if kind == "batched" else 1), dtype=torch.uint8, device="cuda")
    s["out"] = {x: s[x] for x in ("ids", "weights", "perm", "offsets", "loads")}
    if kind == "stats":
        s["mass"] = torch.empty(T, dtype=torch.float32, device="cuda")
        s["entropy"] = torch.empty(T, dtype=torch.float32, device="cuda")
        s["pool"] = torch.empty(T, dtype=torch.int32, device="cuda")
        s["out"].update({x: s[x] for x in ("mass", "entropy", "pool")})
    if kind != "batched":
        s["layer"] = [tuple(s[x][i] for x in ("loads", "ids", "weights", "perm", "offsets")) for i in range(n)]
        if kind != "logits":
            s["inputs"] = [(s["hidden"][i], s["w"][i]) for i in range(n)]
    if kind == "graph":
        _layers(s, s["stream"])           # once outside: first launches are not captured
        torch.cuda.synchronize()
        s["loads"].zero_()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _layers(s, None)              # on the capture stream
    return s


def _layers(s, stream):
    c, p, ws = s["case"], s["params"], s["workspace"]
    T, H, E = c["T"], c["H"], c["E"]
    for (hidden, w), (loads, ids, weights, perm, offsets) in zip(s["inputs"], s["layer"]):
        B.laser_route(hidden, w, T, H, E, p, loads, ids, weights, perm, offsets, None, ws, stream)


def run(state):
    s, c = state, state["case"]
    kind, p, stream = c["kind"], s["params"], s["stream"]
    if not c["carry"]:
        s["loads"].zero_()                # a new batch starts from empty counters
    if kind == "graph":
        s["graph"].replay()
    elif kind == "call":
        _layers(s, stream)
    elif kind == "batched":
        B.laser_route_batched(s["hidden"], s["w"], c["layers"], c["T"], c["H"], c["E"], p, s["loads"], s["ids"],
                              s["weights"], s["perm"], s["offsets"], None, s["workspace"], stream)
    elif kind == "stats":
        (hidden, w), (loads, ids, weights, perm, offsets) = s["inputs"][0], s["layer"][0]
        B.laser_route_stats(hidden, w, c["T"], c["H"], c["E"], p, loads, ids, weights, perm, offsets, None,
                            s["mass"], s["entropy"], s["pool"], s["workspace"], stream)
    else:
        loads, ids, weights, perm, offsets = s["layer"][0]
        B.laser_route_from_logits(s["logits"], c["T"], c["E"], p, loads, ids, weights, perm, offsets,
                                  s["workspace"], stream)
    return s["out"]


def work(case):
    T, H, E, k = case["T"], case["H"], case["E"], case["k"]
    size = 4 if case.get("fp32") else 2
    read = T * E * 4 if case["kind"] == "logits" else (T + E) * H * size
    # ids, weights and permutation out, offsets out, counters in and out
    per_layer = read + T * k * 12 + (E + 1) * 4 + 2 * E * 4 + (T * 12 if case["kind"] == "stats" else 0)
    return {"bytes": per_layer * case["layers"], "flops": 2 * T * H * E * case["layers"]}


def tolerance(case):
    # ids, permutation, offsets and counters are decided in one specified order of binary32
    # operations: whole values are equal.  Weights, and the statistics, are quotients of sums
    # of such numbers: against the same formulas in 64 bits they are 4e-8 .. 8e-8 (2-norm) and
    # at most 4e-7 (largest) off; four times that.
    return {"rel": 3e-7, "max": 1.6e-6, "differ": 0.0}
