"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the
same seeded inputs.  Integer outputs bit-exact; logits and weights within 2e-3
(bf16 inputs) / 1e-5 (fp32 inputs) max abs error."""
import json
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from synth import workloads as wl  # noqa: E402

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "hand_cases.json")


def _util():
    from tests import gpu_util
    return gpu_util


def _hand_cases():
    with open(GOLDEN) as f:
        return json.load(f)["cases"]


@pytest.mark.parametrize("case", _hand_cases(), ids=lambda c: c["name"])
def test_hand_cases_on_gpu(case):
    u = _util()
    logits = np.log(np.array(case["p"], dtype=np.float64)).astype(np.float32)
    gpu = u.run_route_from_logits(logits, case["k"], case["c"], case["eps_high"], case["t_fix"],
                                  np.array(case["loads_in"], np.int32))
    assert gpu["expert_ids"].tolist() == case["expert_ids"]
    assert gpu["loads"].tolist() == case["loads_out"]
    np.testing.assert_allclose(gpu["weights"], np.array(case["weights"]), atol=1e-5)


@pytest.mark.parametrize("preset", ["paper", "stress", "topk", "gsm8k"])
def test_tiny_fp32_config(preset):
    u = _util()
    inp = wl.layer_inputs("tiny")
    s = inp["shape"]
    eps, tfix = wl.thresholds("tiny", 0, preset)
    gpu, ref = u.check_route(inp["hidden"], inp["w_gate"], s.dtype, s.k, s.c, eps, tfix,
                             inp["loads_in"], label=f"tiny/{preset}")
    assert gpu["loads"].sum() == s.T * s.k


SHAPES_FROM_LOGITS = [
    # T, E, k, c, eps, tfix, kind
    (1, 8, 2, 4, 0.9, 0.3, "normal"),
    (63, 8, 2, 4, 0.7, 0.6, "normal"),
    (64, 8, 2, 8, 2.0, 1e-30, "normal"),
    (65, 64, 6, 8, 0.4, 0.8, "normal"),
    (130, 64, 6, 8, 2.0, 1e-30, "normal"),
    (1000, 64, 6, 16, 2.0, 0.05, "normal"),
    (777, 5, 1, 5, 0.9, 0.2, "normal"),
    (500, 33, 4, 7, 0.8, 0.3, "normal"),
    (500, 2, 1, 2, 0.99, 0.1, "normal"),
    (500, 2, 2, 2, 0.99, 0.1, "normal"),
    (300, 16, 16, 16, 2.0, 0.5, "normal"),
    (900, 6, 2, 4, 0.999, 0.37, "ties"),
    (900, 64, 6, 10, 0.999, 0.37, "ties"),
    (4096, 8, 2, 3, 0.6419, 0.6, "normal"),
    (3000, 48, 8, 12, 0.5, 0.4, "normal"),
]


@pytest.mark.parametrize("T,E,k,c,eps,tfix,kind", SHAPES_FROM_LOGITS)
@pytest.mark.parametrize("renorm", [True, False])
def test_route_from_logits(T, E, k, c, eps, tfix, kind, renorm):
    u = _util()
    rng = np.random.default_rng(T * 131 + E)
    logits = wl.random_logits(T + E + k, T, E, kind=kind, tie_levels=3,
                              scale=float(rng.uniform(0.3, 2.0)))
    loads_in = rng.integers(0, 7, size=E).astype(np.int32)
    u.check_from_logits(logits, k, c, eps, tfix, loads_in, renormalize=renorm,
                        label=f"T{T} E{E} k{k} c{c} {kind}")


# The chain decides flexible tokens a window at a time where that pays and one by one
# otherwise, switching over at an arbitrary token.  Two window evaluations exist: 64
# tokens in one wavefront, data staged in segments of 192 through a ring of 576; and
# (many experts per candidate) 128 tokens in two wavefronts, data staged in batches of
# 128 through a ring of 512, output words of 32 tokens.  Every token here is flexible
# (eps_high = 2, tiny t_fix), so T is the number of flexible tokens.
WINDOW_SIZES = [191, 192, 193, 255, 256, 257, 287, 288, 289, 383, 384, 385, 511, 512, 513, 575, 576, 577,
                639, 640, 641, 1023, 1024, 1025, 1151, 1153, 2000, 4097]


@pytest.mark.parametrize("T", WINDOW_SIZES)
@pytest.mark.parametrize("E,k,c", [(64, 6, 8), (8, 2, 4), (40, 3, 16), (64, 2, 4), (33, 5, 8), (64, 9, 16)])
def test_window_chain_sizes(T, E, k, c):
    u = _util()
    rng = np.random.default_rng(T * 7 + E)
    logits = wl.random_logits(T + 3 * E + c, T, E, kind="normal", scale=0.3)
    loads_in = rng.integers(0, 1000, size=E).astype(np.int32)
    u.check_from_logits(logits, k, c, 2.0, 1e-30, loads_in, label=f"window T{T} E{E} k{k} c{c}")


@pytest.mark.parametrize("T", [257, 577, 2000])
@pytest.mark.parametrize("E,k,c", [(64, 2, 4), (64, 3, 4), (64, 5, 8), (64, 6, 16), (16, 6, 8), (15, 2, 4)])
def test_window_chain_variants(T, E, k, c):
    """The window evaluation exists with and without first guesses (chosen by the number
    of experts per candidate) and for 4, 8 and 16 candidates, k fixed at compile time or
    not: every variant, with unrelated candidate sets (windows retire whole) and with
    scores flat enough that neighbours compete."""
    u = _util()
    rng = np.random.default_rng(T * 11 + E + c)
    for scale in (1.0, 0.05):
        logits = wl.random_logits(T + E + c, T, E, kind="normal", scale=scale)
        loads_in = rng.integers(0, 30, size=E).astype(np.int32)
        u.check_from_logits(logits, k, c, 2.0, 1e-30, loads_in, label=f"window variant T{T} E{E} k{k} c{c} s{scale}")


# The sequential walks stage their tokens in batches: of 48 with 9 to 16 candidates, of 21 with
# more, of 16 with up to 8, of 96 where there are no more than 8 experts; a producer wave's share of the
# first two in two halves (of 8, and of 4 and 3); output words of 32 tokens.
@pytest.mark.parametrize("T", [1, 2, 3, 7, 20, 21, 22, 31, 32, 33, 41, 42, 43, 47, 48, 49, 62, 63, 64, 65, 95, 96, 97,
                               191, 192, 193, 250])
@pytest.mark.parametrize("E,k,c", [(64, 6, 8), (8, 2, 4), (64, 9, 16), (16, 4, 12), (9, 8, 9), (64, 6, 64), (20, 3, 18)])
def test_sequential_walk_sizes(T, E, k, c):
    """Every token load-dependent, fewer than the window evaluation takes: counters equal,
    slightly apart and far apart (the wide walk goes level by level of the counters)."""
    u = _util()
    rng = np.random.default_rng(T * 13 + E + c)
    for hi in (1, 3, 100):
        logits = wl.random_logits(T + E + c + hi, T, E, kind="normal", scale=0.3)
        loads_in = rng.integers(0, hi, size=E).astype(np.int32)
        u.check_from_logits(logits, k, c, 2.0, 1e-30, loads_in, label=f"walk T{T} E{E} k{k} c{c} loads<{hi}")


@pytest.mark.parametrize("E,k,c,T1,T2", [(64, 6, 8, 3001, 3000), (8, 2, 4, 1237, 5000),
                                         (64, 6, 12, 700, 2500), (16, 4, 8, 5000, 0)])
def test_window_chain_gives_way_to_sequential(E, k, c, T1, T2):
    """First T1 tokens with unrelated candidate sets (decided side by side), then T2
    identical tokens that all compete for the same experts at equal loads (one by
    one): the hand-over happens wherever progress drops, mid word and mid tile.  (Up to 8
    experts there is no window to give way: one walk through both kinds of tokens.)"""
    u = _util()
    rng = np.random.default_rng(E * 1000 + T1)
    a = wl.random_logits(E + T1, T1, E, kind="normal", scale=1.0)
    row = wl.random_logits(E + T2 + 1, 1, E, kind="normal", scale=1.0)
    logits = np.concatenate([a, np.repeat(row, T2, axis=0)], axis=0)
    loads_in = rng.integers(0, 50, size=E).astype(np.int32)
    u.check_from_logits(logits, k, c, 2.0, 1e-30, loads_in, label=f"handover E{E} c{c} {T1}+{T2}")


@pytest.mark.parametrize("scale,loads_hi", [(3.0, 1), (1.0, 50), (0.3, 1000), (0.02, 3)])
@pytest.mark.parametrize("E,k,c", [(64, 6, 8), (64, 2, 4), (64, 4, 16)])
def test_wide_window_regimes(E, k, c, scale, loads_hi):
    """The 128-token window from windows that retire whole (peaked scores, unrelated
    candidate sets) down to neighbours that all compete (flat scores: it gives up and the
    sequential walk finishes), flexible tokens dense and sparse inside their tiles."""
    u = _util()
    T = 6000
    rng = np.random.default_rng(int(scale * 100) + E + c)
    z = wl.random_logits(17 + c, T, E, kind="normal", scale=scale)
    loads_in = rng.integers(0, loads_hi, size=E).astype(np.int32)
    gpu, ref = u.check_from_logits(z, k, c, 2.0, 1e-30, loads_in, label=f"wide window dense s{scale} c{c}")
    peaked = wl.random_logits(5, T, E, kind="normal", scale=4.0)
    pick = rng.random(T) < 0.15
    flat = wl.random_logits(6, T, E, kind="normal", scale=min(scale, 0.2))
    mixed = np.where(pick[:, None], flat, peaked).astype(np.float32)
    gpu, ref = u.check_from_logits(mixed, k, c, 0.6, 0.5, loads_in, label=f"wide window sparse s{scale} c{c}")
    assert int((ref["cstar"] > k).sum()) > 256


def test_window_chain_long_run():
    """Many segments: the ring wraps dozens of times; flexible tokens are sparse inside
    their tiles (about one in ten), as in the prefill-shaped workload."""
    u = _util()
    T, E, k, c = 40000, 64, 6, 8
    rng = np.random.default_rng(4242)
    peaked = wl.random_logits(1, T, E, kind="normal", scale=3.0)
    flat = wl.random_logits(2, T, E, kind="normal", scale=0.05)
    pick = rng.random(T) < 0.1
    logits = np.where(pick[:, None], flat, peaked).astype(np.float32)
    loads_in = np.zeros(E, np.int32)
    gpu, ref = u.check_from_logits(logits, k, c, 0.4, 0.8, loads_in, label="window long run")
    assert int((ref["cstar"] > k).sum()) > 2000


@pytest.mark.parametrize("E,k,c", [(33, 5, 8), (64, 6, 8), (64, 2, 4), (16, 2, 4), (64, 9, 16)])
def test_window_whose_first_guesses_hold(E, k, c):
    """Counters far apart at the start: nearly every first guess of the window evaluation
    is right, so whole windows retire in the sweep in which their tokens entered -- except
    where two candidates are close, and there a token must have seen the choices of all
    tokens before it, also of those that entered in the same sweep in the other half of
    the window.  Many seeds, several windows each."""
    u = _util()
    for seed in range(24):
        rng = np.random.default_rng(1000 * E + seed)
        T = int(rng.choice([300, 641, 1151, 2500]))
        logits = wl.random_logits(seed + E, T, E, kind="normal", scale=0.3)
        # a few groups of experts with nearly equal counters, the groups far apart
        groups = rng.integers(0, 6, size=E)
        loads_in = (groups * 400 + rng.integers(0, 3, size=E)).astype(np.int32)
        u.check_from_logits(logits, k, c, 2.0, 1e-30, loads_in, label=f"guesses hold E{E} seed{seed}")


def _random_case(seed):
    rng = np.random.default_rng(seed)
    E = int(rng.choice([2, 3, 5, 8, 8, 8, 16, 24, 33, 48, 64, 64, 64]))
    k = int(rng.integers(1, min(E, 8) + 1))
    c = int(rng.integers(k, min(E, 16) + 1))
    T = int(rng.choice([1, 17, 64, 100, 257, 700, 1500, 4000, 9000]))
    kind = rng.choice(["normal", "flat", "mixed", "ties", "same", "blocks"])
    scale = float(rng.choice([0.02, 0.1, 0.5, 1.0, 3.0]))
    if kind == "normal":
        z = rng.standard_normal((T, E)) * scale
    elif kind == "flat":
        z = rng.standard_normal((T, E)) * 0.01
    elif kind == "mixed":
        z = rng.standard_normal((T, E)) * scale
        pick = rng.random(T) < rng.uniform(0.02, 0.6)
        z[pick] = rng.standard_normal((int(pick.sum()), E)) * 0.01
    elif kind == "ties":
        z = (rng.standard_normal(3) * scale)[rng.integers(0, 3, size=(T, E))]
    elif kind == "same":
        z = np.repeat(rng.standard_normal((1, E)) * scale, T, axis=0)
    else:  # runs of identical tokens inside random stretches
        z = rng.standard_normal((T, E)) * scale
        for _ in range(int(rng.integers(1, 6))):
            a = int(rng.integers(0, T))
            z[a:min(T, a + int(rng.integers(1, 600)))] = z[a]
    eps = float(rng.choice([2.0, 0.999, 0.9, 0.7, 0.5, 0.3]))
    tfix = float(rng.choice([1e-30, 0.01, 0.2, 0.5, 0.8, 1.0]))
    loads = rng.integers(0, int(rng.choice([1, 10, 1000, 100000])), size=E).astype(np.int32)
    return z.astype(np.float32), k, c, eps, tfix, loads, bool(rng.integers(0, 2)), f"{kind} T{T} E{E} k{k} c{c}"


def test_random_cases_against_oracle():
    """Seeded random shapes, thresholds, load offsets and logit structures (flat,
    peaked, mixed, exact ties, identical tokens, runs of identical tokens)."""
    u = _util()
    flexible = 0
    for seed in range(5000, 5400):
        z, k, c, eps, tfix, loads, renorm, label = _random_case(seed)
        gpu, ref = u.check_from_logits(z, k, c, eps, tfix, loads, renormalize=renorm,
                                       label=f"seed {seed} {label}")
        flexible += int((ref["cstar"] > k).sum())
    assert flexible > 100000


# ------------------------------------------------------------- RANDOM trimming ----

RANDOM_SHAPES = [
    # T, E, k, c, eps, tfix, kind
    (1, 8, 2, 4, 2.0, 1e-30, "normal"),
    (63, 8, 2, 4, 0.9, 0.05, "normal"),
    (500, 8, 2, 3, 2.0, 1e-30, "normal"),        # every token sampled, c = k + 1
    (500, 8, 2, 2, 2.0, 1e-30, "normal"),        # c = k: a random k of the pool, no load dependence
    (1000, 64, 6, 8, 2.0, 0.02, "normal"),
    (3000, 64, 6, 16, 0.9, 0.1, "normal"),       # more than four draws per token
    (700, 33, 4, 7, 0.8, 0.3, "normal"),
    (900, 12, 3, 5, 0.999, 0.01, "ties"),
    (5000, 16, 2, 4, 0.7, 0.2, "normal"),
    (257, 64, 1, 16, 2.0, 1e-30, "normal"),
]


@pytest.mark.parametrize("T,E,k,c,eps,tfix,kind", RANDOM_SHAPES)
def test_random_trimming_from_logits(T, E, k, c, eps, tfix, kind):
    u = _util()
    rng = np.random.default_rng(T * 17 + E)
    logits = wl.random_logits(T + 2 * E + c, T, E, kind=kind, tie_levels=3, scale=0.5)
    loads_in = rng.integers(0, 9, size=E).astype(np.int32)
    for renorm in (True, False):
        u.check_random_from_logits(logits, k, c, eps, tfix, loads_in, seed=2 ** 40 + 12345 + T,
                                   stream=E, token_offset=2 ** 33 + 5, renormalize=renorm,
                                   label=f"random T{T} E{E} k{k} c{c}")


def test_random_trimming_equals_top_when_nothing_is_trimmed():
    """With c as large as any pool the sampling never happens: the RANDOM analysis
    kernel must then reproduce the deterministic path bit for bit."""
    u = _util()
    for T, E, k, c, eps, tfix in [(2000, 16, 2, 16, 0.9, 0.2), (1500, 64, 6, 16, 0.5, 0.6),
                                  (700, 8, 2, 8, 2.0, 1e-30)]:
        logits = wl.random_logits(T + E, T, E, scale=1.0)
        loads_in = (np.arange(E) % 3).astype(np.int32)
        top = u.run_route_from_logits(logits, k, c, eps, tfix, loads_in)
        rnd = u.run_random_from_logits(logits, k, c, eps, tfix, loads_in, seed=99)
        for key in ("expert_ids", "permutation", "expert_offsets", "loads"):
            assert np.array_equal(top[key], rnd[key]), key
        assert np.abs(top["weights"] - rnd["weights"]).max() <= 1e-6


def test_random_trimming_full_path_and_split_calls():
    """From hidden states (bf16 gate), and the same tokens in two calls with
    token_offset carried: identical choices."""
    import oracle
    u = _util()
    import torch
    from paper_2510_03293_amd import binding as B
    rng = np.random.default_rng(321)
    T, H, E, k, c = 900, 512, 32, 4, 6
    hidden, w = wl.make_gate(rng, T, H, E, wl.DTYPE_BF16)
    kw = dict(dtype=wl.DTYPE_BF16, trim_mode=B.TRIM_RANDOM, seed=7, stream=3)
    hd, wd = u.to_device(hidden), u.to_device(w)

    def run(rows, loads, off):
        params = B.make_params(k, c, 2.0, 0.05, token_offset=off, **kw)
        buf = B.route(hd[rows], wd, params, loads, want_logits=True)
        torch.cuda.synchronize()
        return buf
    loads = torch.zeros(E, dtype=torch.int32, device="cuda")
    whole = run(slice(0, T), loads, 100)
    z = whole.logits.cpu().numpy()
    assert np.abs(z - oracle.gate(hidden, w, wl.DTYPE_BF16)).max() <= 2e-3
    ref = oracle.route_random(z, k, c, 2.0, 0.05, np.zeros(E, np.int32), 7, 3, 100)
    assert np.array_equal(whole.expert_ids.cpu().numpy(), ref["expert_ids"])
    assert np.array_equal(whole.permutation.cpu().numpy(), ref["permutation"])
    assert np.array_equal(loads.cpu().numpy(), ref["loads"])
    l2 = torch.zeros(E, dtype=torch.int32, device="cuda")
    a = run(slice(0, 333), l2, 100)
    ids_a = a.expert_ids.cpu().numpy().copy()
    b = run(slice(333, T), l2, 433)
    assert np.array_equal(np.vstack([ids_a, b.expert_ids.cpu().numpy()]), ref["expert_ids"])
    assert np.array_equal(l2.cpu().numpy(), ref["loads"])


# A handful of flexible tokens among many fixed ones: the finishing workgroups resolve
# them without the chain workgroup (at most 8 tokens in at most 4 tiles, at most 256
# tiles); one more token or tile and the call goes the general way.
FEW_FLEX = [
    # T, E, k, c, positions of the flexible tokens
    (16384, 64, 6, 8, [9500]),
    (16384, 64, 6, 8, [0]),
    (16384, 64, 6, 8, [16383]),
    (16384, 64, 6, 8, [64, 65, 66, 127, 4000, 4001, 9000, 16320]),      # 8 tokens, 4 tiles
    (16384, 64, 6, 8, [64, 65, 66, 127, 4000, 4001, 9000, 16320, 16321]),  # 9 tokens: general path
    (16384, 64, 6, 8, [10, 1000, 5000, 9000, 13000]),                   # 5 tiles: general path
    (3000, 8, 2, 4, [5, 6, 7, 8, 9, 10, 11, 12]),                       # all in one tile, E = 8
    (3000, 8, 2, 4, [2990, 2999]),                                      # in the ragged last tile
    (1000, 33, 4, 12, [100, 500, 501, 900]),
    (200, 16, 3, 16, [0, 63, 64, 199]),
]


@pytest.mark.parametrize("T,E,k,c,where", FEW_FLEX)
def test_few_flexible_tokens(T, E, k, c, where):
    u = _util()
    rng = np.random.default_rng(T + E + len(where))
    logits = wl.random_logits(T + E, T, E, kind="normal", scale=1.0)
    hot = rng.integers(0, E, size=T)
    logits[np.arange(T), hot] += 30.0                    # peaked: the top-k mass test passes
    logits[where] = wl.random_logits(7, len(where), E, kind="normal", scale=0.01)   # flat
    loads_in = rng.integers(0, 50, size=E).astype(np.int32)
    gpu, ref = u.check_from_logits(logits, k, c, 0.9, 0.5, loads_in, label=f"few flex {where}")
    assert np.array_equal(np.where(ref["cstar"] > k)[0], np.array(sorted(where)))


@pytest.mark.parametrize("T,E,k,c", [(1, 1, 1, 1), (100, 1, 1, 1), (300, 2, 2, 2), (64, 16, 16, 16),
                                     (1000, 16, 15, 16), (129, 64, 16, 16), (5000, 64, 1, 16), (70, 3, 3, 3)])
def test_limits_of_the_parameters(T, E, k, c):
    """One expert, every expert chosen, the largest k and c, counters near the 2^27
    limit -- from logits and through the bf16 gate."""
    u = _util()
    rng = np.random.default_rng(T + 100 * E + k)
    for eps, tfix in [(2.0, 1e-30), (0.5, 0.5)]:
        z = (rng.standard_normal((T, E)) * 0.5).astype(np.float32)
        loads = rng.integers(0, 2 ** 26, size=E).astype(np.int32)
        label = f"limits T{T} E{E} k{k} c{c} eps{eps}"
        u.check_from_logits(z, k, c, eps, tfix, loads, label=label)
        h, w = wl.make_gate(rng, T, 64, E, wl.DTYPE_BF16)
        u.check_route(h, w, wl.DTYPE_BF16, k, c, eps, tfix, loads, label="bf16 " + label)


def test_extreme_logits():
    """Scores that underflow the clamp, huge spreads, and all-equal rows."""
    u = _util()
    T, E = 200, 64
    logits = wl.random_logits(5, T, E, scale=40.0)
    logits[::7] = 1.25
    logits[3] = -300.0
    logits[3, 10] = 300.0
    u.check_from_logits(logits, 6, 8, 0.9, 0.01, np.zeros(E, np.int32), label="extreme")


def test_empty_batch():
    u = _util()
    E = 8
    loads_in = np.arange(E, dtype=np.int32)
    gpu = u.run_route_from_logits(np.zeros((0, E), np.float32), 2, 4, 0.5, 0.5, loads_in)
    assert np.array_equal(gpu["loads"], loads_in)
    assert np.array_equal(gpu["expert_offsets"], np.zeros(E + 1, np.int32))
    assert gpu["expert_ids"].shape == (0, 2)


BF16_SHAPES = [
    # T, H, E, k, c
    (200, 2048, 64, 6, 8),
    (130, 4096, 8, 2, 4),
    (65, 1000, 5, 2, 3),      # H not a multiple of the 64-value chunk, E < 8
    (64, 8, 33, 4, 6),        # H smaller than a chunk
    (1, 2048, 64, 6, 8),
    (333, 512, 17, 3, 9),
]


@pytest.mark.parametrize("T,H,E,k,c", BF16_SHAPES)
def test_bf16_gate_and_route(T, H, E, k, c):
    u = _util()
    rng = np.random.default_rng(T + H + E)
    hidden, w = wl.make_gate(rng, T, H, E, wl.DTYPE_BF16, bias=np.linspace(-1.0, 1.0, E))
    if H < 64:
        w = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(w) * 8.0)   # keep the logits spread
    u.check_route(hidden, w, wl.DTYPE_BF16, k, c, 0.6, 0.3, rng.integers(0, 5, E).astype(np.int32),
                  label=f"bf16 T{T} H{H} E{E}")


STATS_SHAPES = [
    # T, H, E, k, c, dtype
    (300, 2048, 64, 6, 8, wl.DTYPE_BF16),
    (130, 4096, 8, 2, 4, wl.DTYPE_BF16),
    (65, 1000, 5, 2, 3, wl.DTYPE_BF16),
    (700, 512, 33, 4, 12, wl.DTYPE_BF16),
    (256, 128, 8, 2, 4, wl.DTYPE_F32),
]


@pytest.mark.parametrize("T,H,E,k,c,dtype", STATS_SHAPES)
def test_token_statistics(T, H, E, k, c, dtype):
    """Top-k mass, entropy and pool size written alongside the routing step, against
    the oracle on the GPU's own logits; the routing outputs are those of laser_route."""
    import oracle
    u = _util()
    rng = np.random.default_rng(T + H + E + 1)
    hidden, w = wl.make_gate(rng, T, H, E, dtype, bias=np.linspace(-1.5, 1.5, E))
    if dtype == wl.DTYPE_F32:
        w = (w * 20).astype(np.float32)
    loads_in = rng.integers(0, 5, E).astype(np.int32)
    eps, tfix = 0.6, 0.3
    plain = u.run_route(hidden, w, dtype, k, c, eps, tfix, loads_in)
    got = u.run_route_stats(hidden, w, dtype, k, c, eps, tfix, loads_in)
    for key in ("expert_ids", "permutation", "expert_offsets", "loads"):
        assert np.array_equal(plain[key], got[key]), key
    assert np.abs(plain["logits"] - got["logits"]).max() <= 1e-6
    ref = oracle.token_stats(got["logits"], k, tfix)
    assert np.abs(got["topk_mass"] - ref["topk_mass"]).max() <= 1e-5
    assert np.abs(got["entropy"] - ref["entropy"]).max() <= 1e-4
    assert np.array_equal(got["pool_size"], ref["pool_size"])
    # any subset of the three may be asked for
    only = u.run_route_stats(hidden, w, dtype, k, c, eps, tfix, loads_in, which=(False, True, False))
    assert only["topk_mass"] is None and only["pool_size"] is None
    assert np.array_equal(only["entropy"], got["entropy"])


@pytest.mark.parametrize("L,E,G", [(1, 8, 0), (27, 64, 8), (5, 64, 64), (3, 1000, 7), (4, 5, 3), (0, 8, 0)])
def test_imbalance_metrics(L, E, G):
    import torch
    import oracle
    from paper_2510_03293_amd import binding as B
    rng = np.random.default_rng(L * 100 + E + G)
    n = rng.integers(0, 3000, size=(L, E)).astype(np.int32)
    if L > 1:
        n[1] = 0                                     # a layer without assignments
    A = w = None
    if G:
        A = rng.random((G, E)).astype(np.float32)
        A /= A.sum(0, keepdims=True)
        A = A.astype(np.float32)
        w = rng.random(L).astype(np.float32)
    out = B.laser_imbalance(torch.from_numpy(n).cuda(),
                            None if A is None else torch.from_numpy(A).cuda(),
                            None if w is None else torch.from_numpy(w).cuda())
    torch.cuda.synchronize()
    ref = oracle.imbalance(n, None if A is None else A.astype(np.float64),
                           None if w is None else w.astype(np.float64))
    np.testing.assert_allclose(out["I"].cpu().numpy(), ref["I"], rtol=1e-14)
    np.testing.assert_allclose(out["MV"].cpu().numpy(), ref["MV"], rtol=1e-12, atol=1e-14)
    if G:
        np.testing.assert_allclose(out["I_gpu"].cpu().numpy(), ref["I_gpu"], rtol=1e-12)
    np.testing.assert_allclose(out["agg"].cpu().numpy(), ref["agg"] if L else [0.0, 0.0], rtol=1e-12)


BATCHED = [
    # B, T, H, E, k, c, dtype, eps_high, t_fix
    (3, 200, 2048, 64, 6, 8, wl.DTYPE_BF16, 0.6, 0.3),
    (5, 65, 1000, 5, 2, 3, wl.DTYPE_BF16, 0.6, 0.3),
    (2, 1500, 512, 16, 2, 6, wl.DTYPE_BF16, 2.0, 0.01),     # every token flexible: window evaluation
    (7, 64, 2048, 64, 6, 8, wl.DTYPE_BF16, 0.4, 0.8),       # decode-sized problems
    (4, 256, 128, 8, 2, 4, wl.DTYPE_F32, 0.6, 0.3),
    (1, 130, 4096, 8, 2, 4, wl.DTYPE_BF16, 0.6, 0.3),
]


@pytest.mark.parametrize("nb,T,H,E,k,c,dtype,eps,tfix", BATCHED)
def test_batched_call_equals_single_calls(nb, T, H, E, k, c, dtype, eps, tfix):
    """Every problem of a batched call: logits against the fp64 gate, decisions and
    tables against the oracle on those logits, and everything bit for bit what a call
    of its own gives."""
    import oracle
    u = _util()
    rng = np.random.default_rng(nb * 1000 + T + H + E)
    hs, ws_, ls = [], [], []
    for b in range(nb):
        h, w = wl.make_gate(rng, T, H, E, dtype, bias=np.linspace(-1.0, 1.0, E) * (b % 3))
        hs.append(h)
        ws_.append(w)
        ls.append(rng.integers(0, 5 + 40 * b, E).astype(np.int32))
    got = u.run_route_batched(hs, ws_, dtype, k, c, eps, tfix, ls)
    tol = u.TOL_LOGIT[dtype]
    for b in range(nb):
        label = f"batched problem {b} of {nb}"
        z = oracle.gate(hs[b], ws_[b], dtype)
        assert np.abs(got[b]["logits"].astype(np.float64) - z).max() <= tol, label
        ref = oracle.route(got[b]["logits"], k, c, eps, tfix, ls[b])
        u.assert_discrete_equal(got[b], ref, label)
        assert np.abs(got[b]["weights"].astype(np.float64) - ref["weights"]).max() <= tol, label
        single = u.run_route(hs[b], ws_[b], dtype, k, c, eps, tfix, ls[b])
        for key in ("logits", "expert_ids", "weights", "permutation", "expert_offsets", "loads"):
            assert np.array_equal(got[b][key], single[key]), f"{label}: {key} differs from the single call"
    blind = u.run_route_batched(hs, ws_, dtype, k, c, eps, tfix, ls, want_logits=False)   # no logits buffer
    for b in range(nb):
        for key in ("expert_ids", "weights", "permutation", "expert_offsets", "loads"):
            assert np.array_equal(got[b][key], blind[b][key]), f"problem {b}: {key} differs without a logits buffer"


def test_batched_call_random_trimming_and_no_logits():
    """RANDOM trimming in a batch: problem b draws with stream id stream + b.  Without
    a logits buffer the results are the same."""
    import oracle
    from paper_2510_03293_amd import binding as B
    u = _util()
    nb, T, H, E, k, c = 3, 300, 512, 32, 2, 5
    rng = np.random.default_rng(77)
    hs, ws_, ls = [], [], []
    for b in range(nb):
        h, w = wl.make_gate(rng, T, H, E, wl.DTYPE_BF16)
        hs.append(h)
        ws_.append(wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(w) * 0.25))    # flat scores: big pools
        ls.append(rng.integers(0, 9, E).astype(np.int32))
    got = u.run_route_batched(hs, ws_, wl.DTYPE_BF16, k, c, 0.9, 0.05, ls, trim_mode=B.TRIM_RANDOM,
                              seed=1234, stream=5)
    blind = u.run_route_batched(hs, ws_, wl.DTYPE_BF16, k, c, 0.9, 0.05, ls, trim_mode=B.TRIM_RANDOM,
                                seed=1234, stream=5, want_logits=False)
    sampled = 0
    for b in range(nb):
        ref = oracle.route_random(got[b]["logits"], k, c, 0.9, 0.05, ls[b], 1234, 5 + b, 0)
        u.assert_discrete_equal(got[b], ref, f"batched random problem {b}")
        assert np.abs(got[b]["weights"].astype(np.float64) - ref["weights"]).max() <= 1e-5
        for key in ("expert_ids", "weights", "permutation", "expert_offsets", "loads"):
            assert np.array_equal(got[b][key], blind[b][key]), key
        pool = oracle.token_stats(got[b]["logits"], k, 0.05)["pool_size"]
        sampled += int(((pool > c) & (ref["expanded"] == 1)).sum())
    assert sampled > 0


def test_random_trimming_with_statistics_in_one_call():
    """laser_route_stats in RANDOM mode: the pool sizes the caller asked for are the ones
    the resampling pass works from (no copy in the workspace then)."""
    import torch
    import oracle
    from paper_2510_03293_amd import binding as B
    u = _util()
    T, H, E, k, c = 500, 512, 32, 2, 5
    rng = np.random.default_rng(5)
    h, w = wl.make_gate(rng, T, H, E, wl.DTYPE_BF16)
    w = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(w) * 0.25)
    loads_in = rng.integers(0, 9, E).astype(np.int32)
    params = B.make_params(k, c, 0.9, 0.05, dtype=wl.DTYPE_BF16, trim_mode=B.TRIM_RANDOM, seed=99, stream=3)
    hd, wd = u.to_device(h), u.to_device(w)
    loads = torch.from_numpy(loads_in.copy()).cuda()
    buf = B.RouteBuffers(T, H, E, params, want_logits=True)
    pool = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    B.laser_route_stats(hd, wd, T, H, E, params, loads, buf.expert_ids, buf.weights, buf.permutation,
                        buf.expert_offsets, buf.logits, None, None, pool, buf.workspace)
    torch.cuda.synchronize()
    z = buf.logits.cpu().numpy()
    ref = oracle.route_random(z, k, c, 0.9, 0.05, loads_in, 99, 3, 0)
    got = {"expert_ids": buf.expert_ids.cpu().numpy(), "weights": buf.weights.cpu().numpy(),
           "permutation": buf.permutation.cpu().numpy(), "expert_offsets": buf.expert_offsets.cpu().numpy(),
           "loads": loads.cpu().numpy()}
    u.assert_discrete_equal(got, ref, "random + stats")
    st = oracle.token_stats(z, k, 0.05)
    assert np.array_equal(pool.cpu().numpy(), st["pool_size"])
    assert int(((st["pool_size"] > c) & (ref["expanded"] == 1)).sum()) > 0


def test_batched_call_argument_errors_and_empty():
    import torch
    from paper_2510_03293_amd import binding as B
    p = B.make_params(2, 4, 0.5, 0.5)
    dummy = torch.zeros(1024, dtype=torch.uint8, device="cuda")
    B.laser_route_batched(None, None, 0, 64, 64, 8, p, None, None, None, None, None, None, None)  # B = 0
    # three problems without tokens: offsets zeroed, loads untouched
    E = 8
    loads = torch.arange(3 * E, dtype=torch.int32, device="cuda").reshape(3, E).contiguous()
    offs = torch.full((3, E + 1), -1, dtype=torch.int32, device="cuda")
    wg = torch.zeros((3, E, 64), dtype=torch.bfloat16, device="cuda")
    ws0 = torch.zeros(3 * B.laser_workspace_bytes(0, 64, E, p), dtype=torch.uint8, device="cuda")
    B.laser_route_batched(None, wg, 3, 0, 64, E, p, loads, None, None, None, offs, None, ws0)
    torch.cuda.synchronize()
    assert torch.equal(offs, torch.zeros_like(offs))
    assert torch.equal(loads.cpu(), torch.arange(3 * E, dtype=torch.int32).reshape(3, E))
    with pytest.raises(B.LaserError):
        B.laser_route_batched(dummy, dummy, -1, 64, 64, 8, p, dummy, dummy, dummy, dummy, dummy, None, dummy)
    with pytest.raises(B.LaserError):      # workspace for one problem only
        one = B.laser_workspace_bytes(64, 64, 8, p)
        ws = torch.zeros(one, dtype=torch.uint8, device="cuda")
        big = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
        B.laser_route_batched(big, big, 2, 64, 64, 8, p, big, big, big, big, big, None, ws)


@pytest.mark.parametrize("n", [1, 2, 5, 100, 1001, 4096])
def test_percentiles_on_device(n):
    """Percentiles over batches: the device result against the oracle (same fp64
    operations, so equal to the last bit), with repeated values in the list."""
    import torch
    import oracle
    from paper_2510_03293_amd import binding as B
    rng = np.random.default_rng(n)
    x = np.round(rng.random(n) * 9 + 1, 2)               # rounding makes ties
    q = [0, 1, 33.3, 50, 95, 99.9, 100]
    got = B.laser_percentiles(torch.from_numpy(x).cuda(), q).cpu().numpy()
    assert np.array_equal(got, oracle.percentiles(x, q))
    with pytest.raises(B.LaserError):
        B.laser_percentiles(torch.zeros(4097, dtype=torch.float64, device="cuda"), [50])
    with pytest.raises(B.LaserError):
        B.laser_percentiles(torch.zeros(4, dtype=torch.float64, device="cuda"), [101.0])


@pytest.mark.parametrize("n", [1, 2, 63, 1000, 16384, 100001])
def test_layer_summary_on_device(n):
    """Mean and percentiles of a layer's per-token statistic: order statistics exact
    (equal to the oracle's percentiles of the same values, bit for bit), the mean to
    fp64 rounding.  Negative values, repeated values, both zeros."""
    import torch
    import oracle
    from paper_2510_03293_amd import binding as B
    rng = np.random.default_rng(n)
    x = np.round(rng.standard_normal(n) * 3, 1).astype(np.float32)
    if n > 2:
        x[0], x[1] = 0.0, -0.0
    q = [0, 5, 25, 50, 75, 95, 99.9, 100]
    mean, got = B.laser_summary_f32(torch.from_numpy(x).cuda(), q)
    ref = oracle.percentiles(x.astype(np.float64), q)
    assert np.array_equal(np.abs(got.cpu().numpy()), np.abs(ref))      # (-0 and +0 are one value)
    assert abs(float(mean) - float(x.astype(np.float64).mean())) <= 1e-12 * max(1.0, float(np.abs(x).max()))


def test_fp32_gate_ragged():
    u = _util()
    rng = np.random.default_rng(17)
    hidden, w = wl.make_gate(rng, 300, 132, 12, wl.DTYPE_F32)
    w = (w * 20).astype(np.float32)
    u.check_route(hidden, w, wl.DTYPE_F32, 3, 6, 0.5, 0.2, np.zeros(12, np.int32), label="fp32 ragged")


def test_split_call_carries_loads():
    u = _util()
    E, k, c, T = 64, 6, 8, 700
    logits = wl.random_logits(9, T, E, scale=0.8)
    L0 = (np.arange(E) % 5).astype(np.int32)
    whole = u.run_route_from_logits(logits, k, c, 0.6, 0.5, L0)
    a = 233
    first = u.run_route_from_logits(logits[:a], k, c, 0.6, 0.5, L0)
    second = u.run_route_from_logits(logits[a:], k, c, 0.6, 0.5, first["loads"])
    assert np.array_equal(np.vstack([first["expert_ids"], second["expert_ids"]]), whole["expert_ids"])
    assert np.array_equal(second["loads"], whole["loads"])


@pytest.mark.parametrize("T", [1, 37, 64])
@pytest.mark.parametrize("H,E,k,c", [(2048, 64, 6, 8), (4096, 33, 2, 4), (512, 64, 4, 16), (1000, 40, 6, 8)])
def test_single_tile_calls(T, H, E, k, c):
    """Calls of at most 64 tokens (one tile; one chain and one finishing workgroup):
    every regime of the chain -- no flexible token, a few, all of them -- with loads
    carried over, for each variant of the gate kernel's main loop."""
    u = _util()
    rng = np.random.default_rng(T + H + E)
    loads = rng.integers(0, 40, size=E).astype(np.int32)
    for eps, tfix in [(1e-6, 1.0), (0.6, 0.3), (2.0, 1e-30)]:
        hidden, w = wl.make_gate(rng, T, H, E, wl.DTYPE_BF16, bias=np.linspace(-1.0, 1.0, E))
        gpu, ref = u.check_route(hidden, w, wl.DTYPE_BF16, k, c, eps, tfix, loads,
                                 label=f"single tile T{T} H{H} E{E} eps{eps}")
        loads = ref["loads"].astype(np.int32)


def test_calls_replayed_from_a_hip_graph():
    """The entry points allocate nothing, never synchronise and clear their own flags
    with kernels, so a sequence of calls can be captured into a HIP graph (a decode loop
    does that).  Three decode-sized calls with carried loads are captured once and
    replayed on new inputs several times, with eager work in between; every replay must
    give exactly what the eager calls give."""
    import torch
    from paper_2510_03293_amd import binding as B
    u = _util()
    s = wl.SHAPES["decode"]
    w = wl.decode_gate_weight()
    wd = u.to_device(w)
    eps, tfix = wl.thresholds("decode", 0, "paper")
    params = B.make_params(s.k, s.c, eps, tfix, dtype=s.dtype)
    steps = 3
    hid = [torch.empty((s.T, s.H), dtype=torch.bfloat16, device="cuda") for _ in range(steps)]
    bufs = [B.RouteBuffers(s.T, s.H, s.E, params) for _ in range(steps)]
    loads = torch.zeros(s.E, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()

    def enqueue(stream):
        for i in range(steps):
            B.laser_route(hid[i], wd, s.T, s.H, s.E, params, loads, bufs[i].expert_ids, bufs[i].weights,
                          bufs[i].permutation, bufs[i].expert_offsets, None, bufs[i].workspace, stream)

    def fill(rep):
        for i in range(steps):
            hid[i].copy_(u.to_device(wl.layer_inputs("decode", 10 * rep + i, w=w)["hidden"]))
        loads.zero_()

    fill(0)
    with torch.cuda.stream(side):
        enqueue(side)                       # warm-up outside the capture (per-kernel set-up happens here)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    fill(0)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        enqueue(side)
    torch.cuda.synchronize()
    for rep in range(1, 5):
        fill(rep)
        torch.cuda.synchronize()
        enqueue(torch.cuda.current_stream())
        torch.cuda.synchronize()
        want = [(b.expert_ids.clone(), b.weights.clone(), b.permutation.clone(), b.expert_offsets.clone())
                for b in bufs]
        want_loads = loads.clone()
        for b in bufs:                      # eager work between the replays; outputs wiped
            b.expert_ids.fill_(-1)
            b.permutation.fill_(-1)
        fill(rep)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for b, (ids, wts, perm, offs) in zip(bufs, want):
            assert torch.equal(b.expert_ids, ids) and torch.equal(b.permutation, perm)
            assert torch.equal(b.weights.view(torch.int32), wts.view(torch.int32))
            assert torch.equal(b.expert_offsets, offs)
        assert torch.equal(loads, want_loads), f"replay {rep}"
    assert int(loads.sum()) == steps * s.T * s.k


def test_calls_side_by_side_on_two_streams():
    """Calls with their own workspaces and outputs share nothing: two streams, each
    running its own sequence of layers at the same time, give what one stream gives."""
    import torch
    from paper_2510_03293_amd import binding as B
    u = _util()
    T, H, E, k, c = 3000, 512, 64, 6, 8
    rng = np.random.default_rng(31)
    params = B.make_params(k, c, 2.0, 1e-30, dtype=wl.DTYPE_BF16)      # every token on the chain
    prob = []
    for i in range(4):
        h, w = wl.make_gate(rng, T, H, E, wl.DTYPE_BF16, bias=np.linspace(-1.0, 1.0, E))
        prob.append((u.to_device(h), u.to_device(w)))

    def run(streams):
        bufs = [B.RouteBuffers(T, H, E, params) for _ in prob]
        loads = [torch.zeros(E, dtype=torch.int32, device="cuda") for _ in prob]
        torch.cuda.synchronize()
        for rep in range(3):
            for i, (hd, wd) in enumerate(prob):
                st = streams[i % len(streams)]
                B.laser_route(hd, wd, T, H, E, params, loads[i], bufs[i].expert_ids, bufs[i].weights,
                              bufs[i].permutation, bufs[i].expert_offsets, None, bufs[i].workspace, st)
        torch.cuda.synchronize()
        return [(b.expert_ids.clone(), b.permutation.clone(), l.clone()) for b, l in zip(bufs, loads)]

    one = run([torch.cuda.current_stream()])
    two = run([torch.cuda.Stream(), torch.cuda.Stream()])
    for (i1, p1, l1), (i2, p2, l2) in zip(one, two):
        assert torch.equal(i1, i2) and torch.equal(p1, p2) and torch.equal(l1, l2)


def test_run_to_run_determinism():
    u = _util()
    inp = wl.layer_inputs("deepseek", 1, T=2048)
    s = inp["shape"]
    outs = [u.run_route(inp["hidden"], inp["w_gate"], s.dtype, s.k, s.c, 2.0, 1e-30, inp["loads_in"])
            for _ in range(3)]
    for o in outs[1:]:
        for key in outs[0]:
            assert np.array_equal(o[key], outs[0][key]), key


@pytest.mark.parametrize("name,layer,preset,T", [
    ("mixtral", 0, "paper", 4096),
    ("mixtral", 15, "paper", 4096),
    ("mixtral", 3, "stress", 2048),
    ("deepseek", 0, "paper", 4096),
    ("deepseek", 2, "stress", 4096),
    ("decode", 0, "gsm8k", None),
    ("prefill", 0, "paper", 4096),
])
def test_benchmark_shapes_reduced_tokens(name, layer, preset, T):
    u = _util()
    inp = wl.layer_inputs(name, layer, T=T)
    s = inp["shape"]
    eps, tfix = wl.thresholds(name, layer, preset)
    gpu, ref = u.check_route(inp["hidden"], inp["w_gate"], s.dtype, s.k, s.c, eps, tfix,
                             inp["loads_in"], label=f"{name}/{preset}")
    if preset == "stress":
        assert ref["expanded"].all() and (ref["cstar"] == s.c).all()


# ---------------------------------------------------------------- full sizes --

@pytest.mark.parametrize("name,layer,preset", [
    ("deepseek", 0, "paper"), ("deepseek", 13, "stress"), ("deepseek", 26, "gsm8k"),
    ("mixtral", 0, "paper"), ("mixtral", 31, "paper"),
])
def test_full_size_layers(name, layer, preset):
    """One whole layer of the benchmark configurations, every output checked."""
    u = _util()
    inp = wl.layer_inputs(name, layer)
    s = inp["shape"]
    eps, tfix = wl.thresholds(name, layer, preset)
    gpu, ref = u.check_route(inp["hidden"], inp["w_gate"], s.dtype, s.k, s.c, eps, tfix,
                             inp["loads_in"], label=f"{name}[{layer}]/{preset} full")
    assert gpu["loads"].sum() == s.T * s.k


def test_full_size_prefill():
    """131072 tokens, H=4096, E=64: logits checked on a sample of rows (the fp64 gate
    of all rows would take minutes), routing and dispatch checked in full against the
    oracle fed with the GPU's logits."""
    u = _util()
    inp = wl.layer_inputs("prefill", 0)
    s = inp["shape"]
    eps, tfix = wl.thresholds("prefill", 0, "paper")
    rows = np.random.default_rng(1).choice(s.T, size=1536, replace=False)
    rows = np.concatenate([rows, [0, 63, 64, s.T - 65, s.T - 1]])
    gpu, ref = u.check_route(inp["hidden"], inp["w_gate"], s.dtype, s.k, s.c, eps, tfix,
                             inp["loads_in"], label="prefill full", logit_rows=rows)
    assert 0.05 < ref["expanded"].mean() < 0.2
    # properties that hold at any size
    perm = gpu["permutation"]
    assert np.array_equal(np.sort(perm), np.arange(s.T * s.k, dtype=np.int32))
    flat = gpu["expert_ids"].ravel()[perm]
    assert np.all(np.diff(flat) >= 0)


def test_decode_steps_carry_loads():
    """64 tokens per step, loads persist across steps (a sample of the 512 steps of
    the decode configuration is enough to cross several preset boundaries)."""
    import torch
    from paper_2510_03293_amd import binding as B
    import oracle
    u = _util()
    s = wl.SHAPES["decode"]
    w = wl.decode_gate_weight()
    wd = u.to_device(w)
    eps, tfix = wl.thresholds("decode", 0, "gsm8k")
    params = B.make_params(s.k, s.c, eps, tfix, dtype=s.dtype)
    loads = torch.zeros(s.E, dtype=torch.int32, device="cuda")
    buf = B.RouteBuffers(s.T, s.H, s.E, params, want_logits=True)
    ref_loads = np.zeros(s.E, dtype=np.int32)
    flexible = 0
    for step in range(96):
        inp = wl.layer_inputs("decode", step, w=w)
        hd = u.to_device(inp["hidden"])
        B.route(hd, wd, params, loads, buffers=buf)
        torch.cuda.synchronize()
        z = buf.logits.cpu().numpy()
        ref = oracle.route(z, s.k, s.c, eps, tfix, ref_loads)
        assert np.array_equal(buf.expert_ids.cpu().numpy(), ref["expert_ids"]), step
        assert np.array_equal(buf.permutation.cpu().numpy(), ref["permutation"]), step
        assert np.array_equal(buf.expert_offsets.cpu().numpy(), ref["expert_offsets"]), step
        ref_loads = ref["loads"]
        assert np.array_equal(loads.cpu().numpy(), ref_loads), step
        flexible += int((ref["cstar"] > s.k).sum())
        if step % 32 == 0:
            zz = oracle.gate(inp["hidden"], w, s.dtype)
            assert np.abs(z - zz).max() <= 2e-3
    assert flexible > 100          # the load-aware branch was really exercised
    assert ref_loads.sum() == 96 * s.T * s.k
