"""The walks over load-dependent tokens with up to 8 candidates against the oracle, integers bit for
bit: batches of 16 and 96 tokens, output words of 32, fixed tokens in between, counters that are
equal, far apart, or as large as they may be."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from synth import workloads as wl

pytestmark = pytest.mark.gpu


def _check(T, E, k, c, logits, loads_in, eps, label):
    from tests import gpu_util as u
    u.check_from_logits(logits, k, c, eps, 1e-30, loads_in, label=label)


def _sweeps(T, E, k, c, logits, loads_in, label):
    """_check with every token load-dependent; the sweeps of the window evaluation (the fourth of
    the workspace's status words)."""
    import oracle
    from paper_2510_03293_amd import binding as B
    from tests import gpu_util as u
    loads = torch.from_numpy(np.ascontiguousarray(loads_in, dtype=np.int32)).cuda()
    buf = B.route_from_logits(torch.from_numpy(logits).cuda(), B.make_params(k, c, 2.0, 1e-30), loads)
    torch.cuda.synchronize()
    u.assert_discrete_equal(u._collect(buf, loads, None), oracle.route(logits, k, c, 2.0, 1e-30, loads_in), label)
    return int(buf.workspace[:16].view(torch.int32)[3])


@pytest.mark.parametrize("T", [1, 15, 16, 17, 32, 33, 48, 95, 96, 97, 128, 193, 255, 256, 257, 700])
@pytest.mark.parametrize("E,k,c", [(8, 2, 4), (8, 7, 8), (3, 1, 2), (9, 2, 3), (16, 4, 8), (33, 5, 7), (64, 1, 8), (64, 7, 8)])
def test_walks_of_up_to_eight_candidates(T, E, k, c):
    rng = np.random.default_rng(T * 31 + E + k)
    for hi in (1, 3, 50):
        logits = wl.random_logits(T + E + c + hi, T, E, kind="normal", scale=0.3)
        _check(T, E, k, c, logits, rng.integers(0, hi, size=E).astype(np.int32), 2.0, f"T{T} E{E} k{k} c{c} loads<{hi}")
    # a third of the tokens keeps its top-k whatever the loads
    logits[rng.random(T) < 0.33, 0] += 30.0
    _check(T, E, k, c, logits, np.zeros(E, np.int32), 0.999, f"T{T} E{E} k{k} c{c} mixed")


@pytest.mark.parametrize("E,k,c", [(8, 2, 4), (16, 4, 8), (64, 6, 8)])
def test_counters_at_their_limit(E, k, c):
    """loads + T < 2^27 is what a call may hold: keys just below 2^31 and differences as large."""
    T = 400
    logits = wl.random_logits(77 + E, T, E, kind="normal", scale=0.3)
    loads = np.where(np.arange(E) % 3 == 0, 0, (1 << 27) - 1 - T).astype(np.int32)
    _check(T, E, k, c, logits, loads, 2.0, f"E{E} loads at the limit")


def test_walk_takes_over_inside_a_word():
    """Tokens that all compete: the window evaluation gives up after a few sweeps, and the walk goes
    on from a token that is in general no multiple of a batch or of an output word."""
    for T, E, k, c in ((900, 64, 6, 8), (2000, 64, 6, 8), (1500, 32, 4, 8), (1300, 16, 2, 4)):
        base = wl.random_logits(T, 1, E, kind="normal", scale=1.0)
        logits = (base + wl.random_logits(T + 1, T, E, kind="normal", scale=0.05)).astype(np.float32)
        _check(T, E, k, c, logits, np.zeros(E, np.int32), 2.0, f"handover T{T} E{E}")


# (9 to 31 experts: the window of 64 tokens, for up to 4, 8 and 16 candidates, k fixed at compile time or not)
WINDOW_64 = [(9, 2, 3), (15, 2, 4), (12, 3, 4), (12, 3, 6), (16, 4, 8), (24, 4, 8), (31, 6, 8), (31, 4, 12)]


@pytest.mark.parametrize("E,k,c", WINDOW_64)
def test_window_where_tokens_do_not_compete(E, k, c):
    """Counters so far apart that no choice changes the order of the candidates: the window
    decides every token, 32 per sweep."""
    T = 2000
    loads = (np.random.default_rng(E).permutation(E) * 10 * T).astype(np.int32)
    n = _sweeps(T, E, k, c, wl.random_logits(E, T, E, kind="normal", scale=1.0), loads, f"far E{E} c{c}")
    assert T // 32 <= n <= T // 32 + 4


@pytest.mark.parametrize("T", [256, 300, 321, 2000])
@pytest.mark.parametrize("E,k,c", [x for x in WINDOW_64 if x[2] <= 8])
def test_window_is_given_up_where_tokens_compete(T, E, k, c):
    """One row for all tokens, equal counters: a token or a few per sweep, so that the walk takes
    over at the first look, after four sweeps that are not judged and eight that are."""
    logits = np.repeat(wl.random_logits(E + T, 1, E, kind="normal", scale=1.0), T, axis=0)
    n = _sweeps(T, E, k, c, logits, np.zeros(E, np.int32), f"competing E{E} c{c}")
    assert n == 12


@pytest.mark.parametrize("E,k,c", [(64, 6, 8), (64, 2, 4), (64, 9, 16), (40, 3, 16)] + WINDOW_64)
def test_window_gives_way_inside_a_word(E, k, c):
    """Tokens with unrelated candidates at counters far apart, then one row for all tokens at
    counters that have come close: the window is entered, given up, and the walk goes on from wherever
    that was."""
    for T1 in (333, 901):
        T = T1 + 1500
        rng = np.random.default_rng(E + T1)
        row = wl.random_logits(E + c, 1, E, kind="normal", scale=1.0)
        far = wl.random_logits(E + T1, T1, E, kind="normal", scale=1.0)
        loads = np.zeros(E, np.int32)
        best = np.argsort(-row[0])[:c]          # the row's candidates: equal counters, the others behind
        loads[np.setdiff1d(np.arange(E), best)] = rng.permutation(E - c) * 4000 + 20000
        far[:, best] -= 50.0                    # (the first tokens do not have them, where there are others)
        n = _sweeps(T, E, k, c, np.concatenate([far, np.repeat(row, T - T1, axis=0)]).astype(np.float32), loads,
                    f"hand-over E{E} c{c} T1 {T1}")
        assert 0 < n < T - 200                  # (fewer sweeps than tokens by far: the walk took the rest)


# (the window of 256 tokens: rings of 768 tokens, 512 with more than 8 candidates, staged 256 at a time)
@pytest.mark.parametrize("T", [256, 257, 511, 512, 513, 767, 768, 769, 1024, 1025, 1281, 3071])
@pytest.mark.parametrize("E,k,c", [(64, 6, 8), (64, 2, 4), (33, 3, 8), (16, 3, 4), (64, 9, 16), (64, 6, 9)])
def test_window_of_256_tokens(T, E, k, c):
    """Counters far apart, where the first guesses hold and a sweep retires the whole window, and groups of
    experts at nearly equal counters, where tokens of the window change one another's choices."""
    rng = np.random.default_rng(T + E + c)
    logits = wl.random_logits(T + c, T, E, kind="normal", scale=1.0)
    n = _sweeps(T, E, k, c, logits, rng.permutation(E) * 10 * T, f"far T{T} E{E} c{c}")
    assert n <= T // 256 + 12
    _check(T, E, k, c, logits, (rng.integers(0, 4, size=E) * 5 * T).astype(np.int32), 2.0, f"groups T{T} E{E} c{c}")


# (above 512 tiles four wavefronts share a tile instead of sixteen)
@pytest.mark.parametrize("T", [1, 15, 16, 17, 49, 64, 65, 127, 512 * 64, 512 * 64 + 21])
@pytest.mark.parametrize("E,k,c", [(64, 6, 8), (8, 2, 4), (33, 3, 16)])
def test_resampling_of_a_whole_tile(T, E, k, c):
    """Every token's pool is larger than c: a wavefront draws for up to four tokens of a tile at once."""
    from tests import gpu_util as u
    logits = wl.random_logits(T + E, T, E, kind="normal", scale=0.3)
    _, ref = u.check_random_from_logits(logits, k, c, 2.0, 1e-30, np.zeros(E, np.int32), seed=77 + T, stream=3,
                                        token_offset=(1 << 32) - 5, label=f"resample T{T} E{E}")
    assert (ref["cstar"] == c).all()


def _rounded(seed, T, E, step):
    """Normal logits rounded to multiples of `step`, zeros of either sign: many are equal."""
    rng = np.random.default_rng(seed)
    z = (np.round(wl.random_logits(seed, T, E, kind="normal", scale=0.9) / step) * step).astype(np.float32)
    return np.where(z == 0, np.where(rng.random(z.shape) < 0.5, np.float32(-0.0), np.float32(0.0)), z)


@pytest.mark.parametrize("E,k,c", [(64, 6, 6), (64, 6, 8), (33, 3, 3), (9, 2, 2), (40, 3, 5)])
@pytest.mark.parametrize("step", [0.25, 4.0])
def test_equal_logits_are_ranked_by_expert(E, k, c, step):
    """The ranks by counting, where counts are equal too: samples, weights and dispatch."""
    from tests import gpu_util as u
    for T in (65, 1000):
        u.check_random_from_logits(_rounded(T + E, T, E, step), k, c, 0.4, 0.3, np.zeros(E, np.int32), seed=7, stream=1,
                                   label=f"equal E{E} c{c} step {step}")


def test_equal_logits_take_no_longer():
    """Logits that were rounded to bf16 have equal ones in nearly every token: the ranks were then counted
    twice, the second time with double keys, and the call took 1.6 times as long (1.3 times what it took
    when it only counted with keys)."""
    from paper_2510_03293_amd import binding as B
    T, E, k = 40000, 64, 6
    z = torch.from_numpy(wl.random_logits(3, T, E, kind="normal", scale=0.9)).cuda()
    params = B.make_params(k, k, 0.4, 0.55, trim_mode=B.TRIM_RANDOM, seed=3)
    loads = torch.zeros(E, dtype=torch.int32, device="cuda")
    took = {}
    for name, logits in (("distinct", z), ("equal", z.bfloat16().float())) * 2:
        buf = B.RouteBuffers(T, 0, E, params)
        us = []
        for _ in range(9):
            loads.zero_()
            torch.cuda.synchronize()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            B.route_from_logits(logits, params, loads, buf)
            b.record()
            torch.cuda.synchronize()
            us.append(1e3 * a.elapsed_time(b))
        took[name] = min(took.get(name, 1e9), float(np.median(us)))
    print(took, flush=True)
    assert took["equal"] < 1.25 * took["distinct"]
