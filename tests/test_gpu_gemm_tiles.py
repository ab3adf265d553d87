"""The GEMM's tiles at their edges: one to five k-tiles (the pipeline's first
and last steps), rows and columns just below, at and above a tile, every tile
height, plain, with gathered rows and with the cosine epilogue, against the
oracle's float64 product (bounds of tests/test_gpu_gemm.py)."""
import numpy as np
import pytest
import torch

import oracle
import parity
from test_gpu_gemm import DEV, check_gemm, randn_bf16, reducer, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_rows", [128, 192, 256])
@pytest.mark.parametrize("M,N,K", [(1, 128, 64), (129, 256, 128), (191, 384, 192), (257, 128, 256), (193, 640, 320)])
def test_tile_edges(M, N, K, tile_rows, monkeypatch):
    monkeypatch.setenv("TR_GEMM_TILE_ROWS", str(tile_rows))
    say("gemm tile edges", M, N, K, "tile rows", tile_rows)
    g = torch.Generator().manual_seed(M * 7 + N + K)
    A, B, P = randn_bf16(g, M, K), randn_bf16(g, N, K), randn_bf16(g, M, N)
    rows = torch.randint(-1, M + 1, (M + 3,), generator=g, dtype=torch.int32)
    r = reducer(D=N, Dc=N, max_tokens=M)
    wide = torch.zeros(M + 3, N + 9, dtype=torch.bfloat16, device=DEV)      # rows at odd places, a border around
    plain, gathered = r.gemm(A.to(DEV), B.to(DEV)), r.gemm(A.to(DEV), B.to(DEV), rows=rows.to(DEV), out=wide[:, 1:N + 1])
    post, s = r.mlp_out_cos(A.to(DEV), B.to(DEV), P.to(DEV))
    torch.cuda.synchronize()
    check_gemm(plain, A, B)
    Ag = torch.zeros(M + 3, K, dtype=torch.bfloat16)
    ok = (rows >= 0) & (rows < M)
    Ag[ok] = A[rows[ok].long()]
    check_gemm(gathered.contiguous(), Ag, B)
    assert not wide[:, 0].any() and not wide[:, N + 1:].any()
    assert torch.equal(post.view(torch.int16), plain.view(torch.int16))
    p, q = oracle.as_f64(P), oracle.as_f64(post.cpu())
    ref = np.array([oracle.cosine(p[m], q[m]) for m in range(M)])
    assert np.all(np.abs(s.double().cpu().numpy() - ref) <= parity.TOL * np.maximum(parity.S_FLOOR, np.abs(ref)))
    r.close()
