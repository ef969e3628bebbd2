"""GPU parity of the decompress / expansion kernels at the edges of their
launches: both splits of a block's waves (over columns, over tokens), waves
past the last column, one tile and ragged tiles, widths whose last group of
eight is a window that overlaps the one before, widths below eight, padded
bases, float32 and bf16 coordinates, gathered coordinates.

Tolerance: the parity, design and per-element bounds of helpers.check.
"""
import numpy as np
import pytest
import torch

from helpers import check, mag_decompress, rand_coords, sample_rows
from oracle import ssn_oracle as O
from paper_2607_13332_amd import inputs as I
from paper_2607_13332_amd import ssn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# (N, d, k): one tile, ragged tiles; few tokens (waves split the tokens), many
# tokens (d = 640 and 2176 leave three of a block's four waves without
# columns), k on both sides of every K step
SHAPES = [(1, 128, 1), (15, 256, 7), (17, 640, 9), (100, 1024, 31), (700, 384, 40), (1030, 2048, 51),
          (12400, 640, 33), (24700, 128, 3), (5003, 2176, 63), (4990, 2176, 64), (1, 128, 65),
          (333, 640, 80), (2100, 2176, 93), (700, 512, 101), (4100, 1152, 128)]


@pytest.mark.parametrize("N,d,k", SHAPES)
@pytest.mark.parametrize("wire", ["f32", "bf16"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_decompress_shapes(N, d, k, wire, dtype):
    print(f"[case] decompress {dtype} N={N} d={d} k={k} wire={wire}", flush=True)
    t, kind = (torch.bfloat16, "bf16out") if dtype == "bf16" else (torch.float32, "f32out_dec")

    def mag(Zs, ids_s, Es):
        M, L, _ = mag_decompress(Zs, ids_s, Es, Uh)
        return M, L, dtype == "bf16"       # float32 operands lose no bits
    V = 50
    r = np.random.default_rng(N + d + k)
    Uh = I.store(I.gaussian_orthonormal_basis(d, k, d + k), dtype)
    Eh = I.store(0.02 * r.standard_normal((V, d)), dtype)
    ids_h = r.integers(0, V, size=N).astype(np.int32)
    Zh = rand_coords(N, k, N + k)
    if wire == "bf16":
        Zh = O.f64(I.store(Zh, "bf16")).astype(np.float32)
    U, E = I.to_device(Uh, dtype, DEV), I.to_device(Eh, dtype, DEV)
    Z = torch.from_numpy(Zh).to(DEV).to(torch.bfloat16 if wire == "bf16" else torch.float32)
    ids = torch.from_numpy(ids_h).to(DEV)
    rows = sample_rows(N, 400, 3)
    bases = [("", U)]
    if k % 16:
        bases.append((" padded", ssn.pad_basis(U)))
    for label, B in bases:
        # rows after the output's end must stay untouched
        out = torch.full((N + 1, d), 7.0, dtype=t, device=DEV)
        Y = ssn.decompress(Z, ids, E, B, out=out[:N])
        check("decompress" + label, I.to_host(Y)[rows], O.decompress(Zh[rows], ids_h[rows], Eh, Uh),
              dtype, kind, mag(Zh[rows], ids_h[rows], Eh))
        assert torch.all(out[N] == 7.0)
        G = ssn.expand_grad(Z, B, out=out[:N])
        check("expand_grad" + label, I.to_host(G)[rows], O.expand_grad(Zh[rows], Uh), dtype, kind,
              mag(Zh[rows], None, None))
        assert torch.all(out[N] == 7.0)
    if wire == "f32":
        T = torch.from_numpy(rand_coords(V, k, 5)).to(DEV)
        X0 = ssn.factored_embedding(ids, T, U)
        assert torch.equal(X0, ssn.expand_grad(T[ids.long()].contiguous(), U))


# float32, narrow bases: both sides of the lines between the chunk-staged and
# the column kernel (2^21, 2^23, 5 x 2^21 and 2^25 output elements, a full round
# of blocks or not), whole and odd widths, and about one tile to a range
@pytest.mark.parametrize("N,d,k", [(1, 128, 16), (129, 640, 31), (2048, 1024, 17), (2049, 1024, 24),
                                   (4096, 1024, 24), (8192, 1024, 16), (8193, 1024, 8), (4096, 2560, 8),
                                   (4224, 2560, 16), (1300, 640, 48), (1500, 640, 100)])
@pytest.mark.parametrize("wire", ["f32", "bf16"])
def test_float32_narrow_bases(N, d, k, wire):
    test_decompress_shapes(N, d, k, wire, "f32")


# bf16, the chunk-staged kernel: wide bases of whole pieces up to its last
# output sizes (k = 72: 2^24, k = 128: 5308416, twice with a full round), one
# round of blocks for k <= 64, odd widths with long rows
@pytest.mark.parametrize("N,d,k", [(1, 128, 72), (130, 256, 96), (300, 640, 120), (5184, 1024, 128),
                                   (5185, 1024, 128), (4096, 2560, 128), (4096, 2560, 40), (4096, 2560, 51),
                                   (2048, 5120, 64), (1024, 18432, 51)])
@pytest.mark.parametrize("wire", ["f32", "bf16"])
def test_chunk_staged_bf16(N, d, k, wire):
    test_decompress_shapes(N, d, k, wire, "bf16")


# gathered coordinates from 2^27 elements on, in the expansion's bits
def test_gathered_coordinates_of_a_full_round():
    N, d, k = 32700, 4224, 64
    U = I.to_device(I.store(I.gaussian_orthonormal_basis(d, k, 3), "bf16"), "bf16", DEV)
    T = torch.from_numpy(rand_coords(40, k, 5)).to(DEV)
    ids = torch.from_numpy(np.random.default_rng(6).integers(0, 40, size=N).astype(np.int32)).to(DEV)
    X0 = ssn.factored_embedding(ids, T, U)
    rows = sample_rows(N, 400, 3)
    assert torch.equal(X0, ssn.expand_grad(T[ids.long()].contiguous(), U))
    check("factored", I.to_host(X0)[rows], O.expand_grad(I.to_host(T)[I.to_host(ids)[rows]], I.to_host(U)),
          "bf16", "bf16out")


@pytest.mark.parametrize("N,d,k", [(200, 256, 51), (13000, 640, 33), (200, 256, 100)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_non_finite_coordinates_stay_in_their_token(N, d, k, dtype):
    U = I.to_device(I.store(I.gaussian_orthonormal_basis(d, k, 3), dtype), dtype, DEV)
    Z = torch.from_numpy(rand_coords(N, k, 4)).to(DEV)
    clean = ssn.expand_grad(Z, U)
    bad = [0, 17, N // 2, N - 2]
    Z[bad] = torch.tensor([float("inf"), float("nan"), -float("inf"), float("nan")], device=DEV)[:, None]
    got = ssn.expand_grad(Z, U)
    keep = torch.ones(N, dtype=torch.bool, device=DEV)
    keep[bad] = False
    # (float32 recomputes the tiles that hold them in plain float32)
    assert torch.allclose(got[keep].float(), clean[keep].float(), rtol=1e-5, atol=1e-5)
    assert not torch.isfinite(got[bad].float()).any()


@pytest.mark.parametrize("k", [8, 51, 128])
def test_float32_infinities_propagate(k):
    """A coordinate or basis row that is infinite gives the infinities and
    NaN of float32 arithmetic."""
    N, d = 40, 256
    U = I.to_device(I.store(I.gaussian_orthonormal_basis(d, k, 3), "f32"), "f32", DEV)
    Z = torch.from_numpy(rand_coords(N, k, 4)).to(DEV)
    Z[3, 1], Z[20, k - 1], Z[30, 0], Z[30, 1] = float("inf"), -float("inf"), float("inf"), float("nan")
    U[7, 2] = float("inf")
    got = I.to_host(ssn.expand_grad(Z, U)).astype(np.float64)
    z, u = I.to_host(Z).astype(np.float64), I.to_host(U).astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = (z[:, None, :] * u[None, :, :]).sum(-1)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    ok = np.isfinite(ref)
    assert np.allclose(got[ok], ref[ok], rtol=1e-5, atol=1e-5)
