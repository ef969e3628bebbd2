"""GPU parity of the many-token float32 compress / projection (operands split
into three bf16 planes): both block sizes, ragged token counts, every width
class of the basis, an odd number of chunks, and infinities and NaN.

Tolerance: the parity, design and per-element bounds of helpers.check.
"""
import numpy as np
import pytest
import torch

from helpers import check, mag_compress, mag_project, sample_rows
from oracle import ssn_oracle as O
from paper_2607_13332_amd import inputs as I
from paper_2607_13332_amd import ssn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# 128-token blocks from 256 of them on, 64-token blocks below (and the d-split
# kernel only for d % 512 == 0 with few tokens, k > 64: d % 256 == 0)
@pytest.mark.parametrize("N,d,k", [(32700, 128, 1), (32701, 192, 16), (40000, 64, 17), (12401, 320, 33),
                                   (13000, 576, 51), (12500, 192, 64), (33000, 128, 80), (100, 192, 99),
                                   (1, 64, 40), (32800, 192, 113), (12600, 320, 128)])
def test_many_token_compress(N, d, k):
    print(f"[case] compress f32 N={N} d={d} k={k}", flush=True)
    V = 60
    k = min(k, d)
    r = np.random.default_rng(N + d + k)
    Uh = I.store(I.gaussian_orthonormal_basis(d, k, d + k), "f32")
    Eh = I.store(0.02 * r.standard_normal((V, d)), "f32")
    ids_h = r.integers(0, V, size=N).astype(np.int32)
    Xh = I.store(r.standard_normal((N, d)), "f32")
    X, E, U = (I.to_device(a, "f32", DEV) for a in (Xh, Eh, Uh))
    ids = torch.from_numpy(ids_h).to(DEV)
    rows = sample_rows(N, 400, 3)
    Xs, loc = Xh[rows], ids_h[rows]
    host = lambda t: I.to_host(t)[rows]  # noqa: E731
    check("compress", host(ssn.compress(X, ids, E, U)), O.compress(Xs, loc, Eh, Uh), "f32", "f32out",
          mag_compress(Xs, loc, Eh, Uh))
    check("project_grad", host(ssn.project_grad(X, U)), O.project_grad(Xs, Uh), "f32", "f32out",
          mag_project(Xs, Uh))
    P = ssn.project_table(E, U)
    check("compress_projected", host(ssn.compress_projected(X, ids, P, U)), O.compress(Xs, loc, Eh, Uh),
          "f32", "f32out", mag_compress(Xs, loc, Eh, Uh))
    if k % 16:
        # a zero-padded basis gives the stored basis's bits
        assert torch.equal(ssn.project_grad(X, ssn.pad_basis(U), k=k), ssn.project_grad(X, U))


# 64-token blocks with float32 instructions (widths of whole tiles, or up to
# 16): one token, edges of a block, one block per compute unit and one more,
# and the last widths of each line
@pytest.mark.parametrize("N,d,k", [(1, 64, 16), (1, 192, 1), (65, 320, 9), (1024, 64, 15), (1025, 64, 15), (63, 192, 32), (65, 320, 48), (12300, 128, 80),
                                   (16384, 64, 64), (16385, 64, 32), (16400, 128, 16), (16385, 64, 48)])
def test_float32_blocks(N, d, k):
    test_many_token_compress(N, d, k)


def test_many_token_infinities_propagate():
    N, d, k = 33000, 128, 33
    U = I.to_device(I.store(I.gaussian_orthonormal_basis(d, k, 3), "f32"), "f32", DEV)
    X = torch.from_numpy(np.random.default_rng(1).standard_normal((N, d)).astype(np.float32)).to(DEV)
    clean = I.to_host(ssn.project_grad(X, U))
    X[5, 3], X[300, 127], X[N - 1, 0], X[N - 1, 1] = float("inf"), float("nan"), float("inf"), -float("inf")
    got = I.to_host(ssn.project_grad(X, U)).astype(np.float64)
    bad = [5, 300, N - 1]
    x, u = I.to_host(X)[bad].astype(np.float64), I.to_host(U).astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = (x[:, :, None] * u[None]).sum(1)
    assert np.array_equal(np.isnan(got[bad]), np.isnan(ref))
    assert np.array_equal(got[bad][np.isinf(ref)], ref[np.isinf(ref)])
    keep = np.setdiff1d(np.arange(N), bad)
    assert np.allclose(got[keep], clean[keep], rtol=1e-5, atol=1e-5)
