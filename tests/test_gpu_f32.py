"""The single-precision gate projection: a logit is one chain of fused multiply-adds in the
order of the contraction axis, so the logits are compared bit for bit with the C library's fmaf."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2510_03293_amd import binding as B

pytestmark = pytest.mark.gpu

_fmaf = ctypes.CDLL("libm.so.6").fmaf
_fmaf.restype = ctypes.c_float
_fmaf.argtypes = [ctypes.c_float] * 3


def chains(hidden, w):
    z = np.zeros((hidden.shape[0], w.shape[0]), dtype=np.float32)
    for t, x in enumerate(hidden.tolist()):
        for e, y in enumerate(w.tolist()):
            acc = 0.0
            for a, b in zip(x, y):
                acc = _fmaf(a, b, acc)
            z[t, e] = acc
    return z


# (edges: one chunk of 128 columns and its remainders, more chunks than are in flight, blocks of 16
# tokens and experts, one or two blocks of experts per workgroup)
@pytest.mark.parametrize("values", ["normal", "exponents", "cancelling", "subnormal"])
@pytest.mark.parametrize("T,E,H", [(1, 1, 4), (17, 9, 132), (33, 16, 128), (2, 17, 124), (19, 33, 60), (16, 64, 640),
                                   (5, 64, 604)])
def test_logits_are_chains_of_fused_multiply_adds(T, E, H, values):
    rng = np.random.default_rng(1000 * T + E + H)
    hidden = rng.standard_normal((T, H)).astype(np.float32)
    w = rng.standard_normal((E, H)).astype(np.float32)
    if values == "exponents":
        hidden = np.ldexp(hidden, rng.integers(-30, 30, (T, H))).astype(np.float32)
        w = np.ldexp(w, rng.integers(-30, 30, (E, H))).astype(np.float32)
    elif values == "cancelling":   # every other product takes the one before it back, nearly
        hidden[:, 1::2] = -hidden[:, ::2][:, : hidden[:, 1::2].shape[1]]
        w[:, 1::2] = w[:, ::2][:, : w[:, 1::2].shape[1]] * np.float32(1 + 2 ** -20)
    elif values == "subnormal":
        hidden = np.ldexp(hidden, rng.integers(-75, -65, (T, H))).astype(np.float32)
        w = np.ldexp(w, rng.integers(-75, -65, (E, H))).astype(np.float32)
    k = min(2, E)
    params = B.make_params(k, k, 0.4, 0.8, dtype=B.DTYPE_F32)
    loads = torch.zeros(E, dtype=torch.int32, device="cuda")
    buf = B.route(torch.from_numpy(hidden).cuda(), torch.from_numpy(w).cuda(), params, loads, want_logits=True)
    torch.cuda.synchronize()
    got, want = buf.logits.cpu().numpy(), chains(hidden, w)
    assert np.array_equal(got.view(np.int32), want.view(np.int32))
