"""The walks over load-dependent tokens with up to 8 candidates against the oracle, integers bit for
bit: batches of 16 and 96 tokens, output words of 32, fixed tokens in between, counters that are
equal, far apart, or as large as they may be."""
from __future__ import annotations

import numpy as np
import pytest

from synth import workloads as wl

pytestmark = pytest.mark.gpu


def _check(T, E, k, c, logits, loads_in, eps, label):
    from tests import gpu_util as u
    u.check_from_logits(logits, k, c, eps, 1e-30, loads_in, label=label)


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
