"""GPU parity of the float32 kernels that multiply on the bf16 matrix cores
(each float32 operand split exactly into three bf16 planes): every shape of
their launches at its edges against the float64 oracle, and infinities and
NaN against float64 arithmetic.

Tolerance: no operand loses bits and the dropped plane pairs stay below 2^-24
of a product, so every element keeps the bound of a float32 sum of L products
(helpers.elementwise_bound with split False): one ulp of the result plus
2 L 2^-23 times the sum of |terms|.
"""
import numpy as np
import pytest
import torch

from helpers import check_elementwise, mag_reparam_grad_factor, mag_weights, sample_rows
from oracle import ssn_oracle as O
from paper_2607_13332_amd import inputs as I
from paper_2607_13332_amd import ssn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def dev(a):
    return I.to_device(a, "f32", DEV)


# columns of a launch on 256 compute units -> the strip shapes: one wave per
# strip of 64 columns, rows shared by 2 and 4 waves, 32- and 16-column strips
# with 4 and 8 waves (k > 64: 32 columns with 1 and 2 waves, 16 with 2 and 4);
# every last strip is partial, d is an odd number of 32-row steps
STRIPS = [(160, n, k) for k in (5, 16, 51, 64) for n in (66004, 40052, 20036, 10004, 5012, 260)]
STRIPS += [(160, n, k) for k in (80, 101, 128) for n in (40052, 20036, 10004, 260)]
STRIPS += [(32, 4, 1), (32, 4, 32), (2048, 36, 64), (1056, 20036, 33)]


@pytest.mark.parametrize("d,n,k", STRIPS)
def test_weight_strips(d, n, k):
    print(f"[case] weights strips d={d} n={n} k={k}", flush=True)
    Uh = I.store(I.gaussian_orthonormal_basis(d, k, d + k), "f32")
    Wh = I.weights_host(d, n, n + k, "f32")
    W = dev(Wh)
    ssn.project_weights(W, dev(Uh))
    cols = np.unique(np.concatenate([sample_rows(n, 300, 1), np.arange(max(0, n - 70), n)]))
    M, L, _ = mag_weights(Wh[:, cols], Uh)
    check_elementwise("strips", I.to_host(W)[:, cols], O.project_weights(Wh[:, cols], Uh), M, L,
                      False, False)


@pytest.mark.parametrize("n", [66004, 20036, 260])
def test_weight_strips_propagate_non_finite(n):
    d, k = 160, 16
    Uh = I.store(I.gaussian_orthonormal_basis(d, k, 3), "f32")
    Wh = I.weights_host(d, n, 4, "f32")
    W0 = dev(Wh)
    ssn.project_weights(W0, dev(Uh))
    bad = {7: np.inf, 130: -np.inf, 199: np.nan, n - 1: np.inf}
    Wb = Wh.copy()
    for j, v in bad.items():
        Wb[j % d, j] = v
    W = dev(Wb)
    ssn.project_weights(W, dev(Uh))
    got, clean = I.to_host(W), I.to_host(W0)
    js = sorted(bad)
    with np.errstate(invalid="ignore"):
        ref = Uh.astype(np.float64) @ (Uh.T.astype(np.float64) @ Wb[:, js].astype(np.float64))
    assert np.array_equal(np.isnan(got[:, js]), np.isnan(ref))
    assert np.array_equal(got[:, js][np.isinf(ref)], ref[np.isinf(ref)])
    # columns of other 64-column strips keep their bits, those of the same
    # strip (recomputed in float32) their bound
    far = np.array([j for j in range(n) if all(j // 64 != b // 64 for b in js)])
    assert np.array_equal(got[:, far], clean[:, far])
    near = np.array([j for j in range(n) if j not in bad and j not in set(far.tolist())])
    M, L, _ = mag_weights(Wh[:, near], Uh)
    check_elementwise("same strip", got[:, near], O.project_weights(Wh[:, near], Uh), M, L, False, False)


# widths that fill no tile, both widths of strips and both passes' chunk sizes;
# a basis of one sign, so that an infinity gives infinities and not NaN
@pytest.mark.parametrize("n", [66004, 20036, 260])
@pytest.mark.parametrize("k", [1, 3, 16, 33, 51, 101])
def test_weight_strips_infinities_at_any_width(k, n):
    d = 160
    r = np.random.default_rng(k)
    Uh = ((0.1 + r.random((d, k))) / d ** 0.5).astype(np.float32)
    Wh = I.weights_host(d, n, 4, "f32")
    js = [7, 130, 199, n - 1]
    for j, v in zip(js, (np.inf, -np.inf, np.nan, np.inf)):
        Wh[j % d, j] = v
    W = dev(Wh)
    ssn.project_weights(W, dev(Uh))
    got = I.to_host(W)[:, js]
    with np.errstate(invalid="ignore"):
        ref = Uh.astype(np.float64) @ (Uh.T.astype(np.float64) @ Wh[:, js].astype(np.float64))
    assert np.isinf(ref).sum() == 3 * d
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])


@pytest.mark.parametrize("N,din,k", [(1, 64, 3), (33, 20036, 51), (95, 10004, 64), (160, 5012, 16),
                                     (1000, 260, 40), (70, 40052, 100), (129, 10004, 128),
                                     (257, 260, 80)])
def test_factor_gradient_strips(N, din, k):
    d = max(64, k)
    print(f"[case] factor gradient N={N} din={din} k={k}", flush=True)
    r = np.random.default_rng(N + din)
    Uh = I.store(I.gaussian_orthonormal_basis(d, k, 9), "f32")
    Hh = r.standard_normal((N, din)).astype(np.float32)
    Gh = r.standard_normal((N, d)).astype(np.float32)
    Zh = (0.02 * r.standard_normal((din, k))).astype(np.float32)
    _, _, GZ = ssn.reparam_backward(dev(Hh), dev(Zh), dev(Uh), dev(Gh))
    M, L, _ = mag_reparam_grad_factor(Hh, Gh, Uh)
    check_elementwise("dZp", I.to_host(GZ), O.reparam_grad_factor(Hh, Gh, Uh), M, L, False, False)
