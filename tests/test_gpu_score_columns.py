"""Scoring at the widths and sizes where its reads change: rows of one to nine
columns of 64 16-byte chunks, whole and partial last chunks, X and the states of
different widths, rows below one chunk; and launches large enough to be paced,
which must give each row the bits it gets in a small one."""
import math

import numpy as np
import pytest
import torch

import oracle
import parity

pytestmark = pytest.mark.gpu

DEV = "cuda"
BF, F4 = torch.bfloat16, torch.float32


def rows_of(g, rows, D, dtype):
    """Token-like rows: magnitudes vary, some low-variance, one zero, one one-hot."""
    x = torch.randn(rows, D, generator=g) * torch.exp(0.5 * torch.randn(rows, 1, generator=g))
    x[::7] = 1.0 + 0.05 * torch.randn(x[::7].shape, generator=g)
    x[3] = 0
    x[5] = 0
    x[5, D // 2] = -3.0
    return x.to(dtype)


def check(D, Dc, dtype, shannon):
    import paper_2607_13500_amd as tr
    print("[case] score", D, Dc, dtype, "shannon" if shannon else "", flush=True)
    rows = 40
    g = torch.Generator().manual_seed(D * 7 + Dc)
    X, P = rows_of(g, rows, D, dtype), rows_of(g, rows, Dc, dtype)
    Q = (0.4 * P.float() + torch.randn(rows, Dc, generator=g)).to(dtype)
    r = tr.Reducer(D, Dc, dtype, max_images=1, max_tokens=rows, max_N=rows, shannon=shannon)
    Xd, Pd, Qd = X.to(DEV), P.to(DEV), Q.to(DEV)
    key, s, h = r.score(Xd, Pd, Qd, want_h2=True)
    keya, _, ha = r.score(Xd, None, None, want_h2=True)
    _, sb, _ = r.score(None, Pd, Qd)
    assert torch.equal(key, keya) and torch.equal(h, ha) and torch.equal(s, sb)
    href, sref = oracle.scores(X, P, Q, entropy=1 if shannon else 2)
    kref = parity.stage1_key(href, D, 1 if shannon else 2)
    h, key, s = (t.double().cpu().numpy() for t in (h, key, s))
    # the kernel forms h as log D less a function of the key, so a key held to TOL of
    # itself leaves h TOL max(key, 1) off (one-hot row, Shannon: key = log D, h = 0)
    assert np.all(np.abs(h - href) <= parity.TOL * np.maximum(np.abs(kref) if shannon else 1, np.maximum(1, np.abs(href))))
    assert np.all(np.abs(key - kref) <= parity.TOL * np.abs(kref) + parity.KEY_FLOOR[1 if shannon else 2])
    assert np.all(np.abs(s - sref) <= parity.TOL * np.maximum(parity.S_FLOOR, np.abs(sref)))
    r.close()


@pytest.mark.parametrize("shannon", [False, True])
@pytest.mark.parametrize("dtype", [BF, F4])
def test_every_number_of_columns(dtype, shannon):
    col = 512 if dtype == BF else 256
    for c in range(1, 10):
        for D in (col * c - 1, col * c, col * c + 1, col * (c - 1) + 8):
            check(D, D, dtype, shannon)
    for D, Dc in ((1, 1), (2, 7), (7, 2), (3, 4 * col), (4 * col, 5), (col, 8 * col), (8 * col, col), (3 * col + 8, 5 * col),
                  (6 * col, 2 * col + 1), (2 * col + 1, 6 * col), (9 * col, 4 * col + 3), (4, 4), (8, 8), (9, 17)):
        check(D, Dc, dtype, shannon)
