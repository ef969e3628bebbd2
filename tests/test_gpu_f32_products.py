"""GPU float32 products on the bf16 matrix cores (operands split into three
bf16 planes): no product is left short, whatever its operands.  Random sums
hide what a single product loses, so these use sums of one product, operands
whose parts would all be cut the same way, and operands near the lower end of
float32.

Bounds: the six plane pairs leave out at most 2^-24 of a product, of either
sign, and the sum and its last addition round once each (2^-24 each): one
product is within 3 x 2^-24, and the mean of many is not off zero (each is off
by 3 x 2^-24 at most, so the mean of a million independent ones by 2^-32).
"""
import numpy as np
import pytest
import torch

from paper_2607_13332_amd import ssn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
ONE = 3 * 2.0 ** -24
MEAN = 2.0 ** -27


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


# Each takes float32 x [n] and y [m] and returns products x_i y_j [n, m]:
# k = 1 or one nonzero row, so that a sum holds one product.
def expand(x, y):
    return ssn.expand_grad(gpu(x[:, None]), gpu(y[:, None])).cpu().numpy()


def decompress(x, y):
    ids = torch.zeros(len(x), dtype=torch.int32, device=DEV)
    return ssn.decompress(gpu(x[:, None]), ids, torch.zeros((1, len(y)), device=DEV), gpu(y[:, None])).cpu().numpy()


def project(x, y):
    G, U = np.zeros((len(x), 64), np.float32), np.zeros((64, len(y)), np.float32)
    G[:, 5], U[5] = x, y
    return ssn.project_grad(gpu(G), gpu(U)).cpu().numpy()


def factor_grad(x, y):
    # dZp = H^T (G U), U = the unit basis: one token
    d = max(64, len(y))
    G = np.zeros((1, d), np.float32)
    G[0, :len(y)] = y
    _, _, GZ = ssn.reparam_backward(gpu(x[None]), gpu(np.zeros((len(x), len(y)))), gpu(np.eye(d, len(y))), gpu(G))
    return GZ.cpu().numpy()


def strips(x, y):
    # W = U (U^T W): U one column with a single 1, so that T = x, and a row of
    # y's below it
    d = 32 * ((len(y) + 33) // 32)
    U, W = np.zeros((d, 1), np.float32), np.zeros((d, len(x)), np.float32)
    U[0], U[1:1 + len(y), 0], W[0] = 1.0, y, x
    w = gpu(W)
    ssn.project_weights(w, gpu(U))
    return w.cpu().numpy()[1:1 + len(y)].T


OPS = {"expand": (expand, 40000, 1024), "decompress": (decompress, 40000, 1024), "project": (project, 33000, 33),
       "project_aligned": (project, 33000, 16), "factor_grad": (factor_grad, 20036, 40), "weights": (strips, 20036, 62)}


@pytest.mark.parametrize("op", OPS)
def test_one_product(op):
    fn, n, m = OPS[op]
    r = np.random.default_rng(7)
    x = (1.0 + r.random(n)).astype(np.float32)
    y = (1.0 + r.random(m)).astype(np.float32)
    # every bit below the first plane set: what truncation cuts most of
    x[:4] = np.array([0x3F80FFFF, 0x3F80FFFE, 0x3FFFFFFF, 0x3F817FFF], np.uint32).view(np.float32)
    y[:4] = x[:4]
    got = fn(x, y).astype(np.float64)
    ref = x[:, None].astype(np.float64) * y[None, :].astype(np.float64)
    err = got / ref - 1.0
    print(f"[products] {op}: worst {np.abs(err).max():.2e} mean {err.mean():+.1e}", flush=True)
    assert np.abs(err).max() <= ONE
    assert abs(err.mean()) <= MEAN


# 2^-100 is above the range of the lowest plane, 2^-126 float32's last normal
@pytest.mark.parametrize("scale", [2.0 ** -100, 2.0 ** -115, 2.0 ** -126])
@pytest.mark.parametrize("op", OPS)
def test_one_product_of_a_tiny_operand(op, scale):
    fn, n, m = OPS[op]
    r = np.random.default_rng(8)
    x = ((1.0 + r.random(n)) * scale).astype(np.float32)
    y = (1.0 + r.random(m)).astype(np.float32)
    ref = x[:, None].astype(np.float64) * y[None, :].astype(np.float64)
    assert np.abs(fn(x, y).astype(np.float64) / ref - 1.0).max() <= ONE


# results from where float32's last place is 2^-149 on are within one of it
@pytest.mark.parametrize("op", ["expand", "decompress"])
def test_subnormal_coordinates(op):
    fn, n, m = OPS[op]
    r = np.random.default_rng(9)
    x = ((1.0 + r.random(n)) * 2.0 ** -138).astype(np.float32)
    y = (1.0 + r.random(m)).astype(np.float32)
    ref = x[:, None].astype(np.float64) * y[None, :].astype(np.float64)
    assert np.abs(fn(x, y).astype(np.float64) - ref).max() <= 2.0 ** -149


@pytest.mark.parametrize("scale", [2.0 ** 108, 2.0 ** 118])
@pytest.mark.parametrize("op", OPS)
def test_one_product_of_a_large_operand(op, scale):
    fn, n, m = OPS[op]
    r = np.random.default_rng(10)
    n = min(n, 2000)
    x = ((1.0 + r.random(n)) * scale).astype(np.float32)
    y = (1.0 + r.random(m)).astype(np.float32)
    ref = x[:, None].astype(np.float64) * y[None, :].astype(np.float64)
    assert np.abs(fn(x, y).astype(np.float64) / ref - 1.0).max() <= ONE


# A running sum of L random terms that is rounded once per product errs by
# 0.425 x 2^-24 sqrt(L / 2) of the result: a rounding is off by 2^-24 / (sqrt(3)
# m) of a value of mantissa m, and the mean of 1 / m^2 over log-uniform m is 3 / (8
# ln 2); the i-th partial sum has sqrt(i / L) of the last one's size.  n chains
# divide that by sqrt(n): 8 chains (and the planes) stay below half of it, the
# few chains of a short sum below three quarters.
@pytest.mark.parametrize("op,N,d,k,part", [
    ("project", 512, 256, 8, 0.5), ("compress", 512, 256, 8, 0.5), ("project", 900, 576, 16, 0.5),
    ("compress", 20000, 1024, 16, 0.5), ("project", 4096, 576, 80, 0.5), ("project", 12300, 4096, 32, 0.5),
    ("project", 16384, 2048, 64, 0.5), ("project", 20000, 1024, 32, 0.5), ("expand", 3000, 576, 24, 0.75),
    ("expand", 1500, 1024, 31, 0.75)])
def test_rounding_of_sums(op, N, d, k, part):
    r = np.random.default_rng(11)
    U = r.standard_normal((d, k)).astype(np.float32)
    if op == "expand":
        L, A, B = k, r.standard_normal((N, k)).astype(np.float32), U.T
        out = ssn.expand_grad(gpu(A), gpu(U))
    else:
        L, A, B = d, r.standard_normal((N, d)).astype(np.float32), U
        if op == "compress":
            ids = torch.zeros(N, dtype=torch.int32, device=DEV)
            out = ssn.compress(gpu(A), ids, torch.zeros((1, d), device=DEV), gpu(U))
        else:
            out = ssn.project_grad(gpu(A), gpu(U))
    rows = np.arange(0, N, max(1, N // 2000))
    ref = A[rows].astype(np.float64) @ B.astype(np.float64)
    err = out.cpu().numpy()[rows].astype(np.float64) - ref
    assert np.sqrt((err ** 2).mean() / (ref ** 2).mean()) <= part * 0.425 * 2.0 ** -24 * np.sqrt(L / 2)
