"""Scoring at the widths and sizes where its reads change: rows of one to nine
columns of 64 16-byte chunks, whole and partial last chunks, X and the states of
different widths, rows below one chunk; and launches large enough to be paced,
which must give each row the bits it gets in a small one."""
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


# launches that each rule paces: rows, D (and Dc), dtype, what is read
PACED = [(61000, (1024, 4096), BF, "xc"), (61008, (3584, 3072), F4, "xch"), (36864, 4096, BF, "xc"), (130000, 1536, BF, "xc"), (98304, 4096, BF, "xc"), (12400, 16384, F4, "xc"), (150016, 1024, BF, "xc"),
         (49152, 2560, BF, "xch"), (98304, 4096, BF, "xch"), (66000, 2048, F4, "xch"), (49160, 6144, BF, "x"), (41000, 1024, BF, "xh"),
         (41000, 2048, F4, "xh"), (36864, 4096, BF, "c"), (151000, 512, F4, "c")]


@pytest.mark.parametrize("rows,D,dtype,read", PACED)
def test_a_row_scores_alike_in_launches_of_any_size(rows, D, dtype, read):
    """The bits of a row's scores in a large (paced) launch are those it gets in a
    launch of 300 rows, and those of the launches that read X or the states alone."""
    import paper_2607_13500_amd as tr
    print("[case] paced", rows, D, dtype, read, flush=True)
    D, Dc = D if isinstance(D, tuple) else (D, D)
    g = torch.Generator(device=DEV).manual_seed(rows + D)
    T = [torch.empty(rows, d, dtype=dtype, device=DEV) if k in read else None for k, d in zip("xcc", (D, Dc, Dc))]
    for t in T:
        if t is not None:
            for part in t.split(8192):
                part.copy_(torch.randn(part.shape, generator=g, device=DEV))
            t[5], t[rows - 2], t[rows // 2] = 0, t[rows - 2] * 2.0 ** -70, t[rows // 2] * 2.0 ** 66
    r = tr.Reducer(D, Dc, dtype, max_images=1, max_tokens=rows, max_N=1, shannon="h" in read)
    whole = r.score(*T, want_h2=True)
    for at in (0, rows // 2 - 150, rows - 300):
        some = [None if t is None else t[at:at + 300] for t in T]
        got = [r.score(*some, want_h2=True)]
        if "x" in read and "c" in read:
            got.append(r.score(some[0], None, None, want_h2=True))
            got.append(r.score(None, some[1], some[2]))
        for res in got:
            for w, v in zip(whole, res):
                assert v is None or torch.equal(w[at:at + 300], v)
    if "x" in read and "c" in read:
        for alone in (r.score(T[0], None, None, want_h2=True), r.score(None, T[1], T[2])):
            for w, v in zip(whole, alone):
                assert v is None or torch.equal(w, v)
    r.close()
