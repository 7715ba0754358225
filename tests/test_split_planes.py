"""What the accuracy bound of the GPU kernels that contract three bf16 planes of
each fp32 operand (tests/test_gpu_split.py) can see: the same contraction in
numpy, with every plane product in place and with one of them lost or taken from
the wrong plane."""
import numpy as np
import pytest

BOUND = 5e-7                      # of tests/test_gpu_split.py
PRODUCTS = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]


def bf16(x):
    """Round to nearest even bf16, as float32."""
    bits = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    bits = (bits + 0x7FFF + ((bits >> 16) & 1)) & 0xFFFF0000
    return bits.astype(np.uint32).view(np.float32)


def planes(x):
    out, rest = [], np.asarray(x, dtype=np.float32)
    for _ in range(3):
        p = bf16(rest)
        out.append(p)
        rest = rest - p
    return out


def hidden_state_error(products, K, seed=0):
    """Relative 2-norm error of tanh(W x) against 64 bits, plane products in fp64
    (their own rounding in fp32 accumulators is below them)."""
    rng = np.random.default_rng(seed)
    x = np.tanh(rng.standard_normal((64, K))).astype(np.float32)
    w = rng.uniform(-0.05, 0.05, (48, K)).astype(np.float32)
    a, b = planes(x), planes(w)
    z = sum(a[i].astype(np.float64) @ b[j].astype(np.float64).T for i, j in products)
    exact = np.tanh(x.astype(np.float64) @ w.astype(np.float64).T)
    return float(np.linalg.norm(np.tanh(z) - exact) / np.linalg.norm(exact))


@pytest.mark.parametrize("K", [256, 512, 1536])
def test_planes_hold_an_fp32_value(K):
    x = np.random.default_rng(K).standard_normal(K).astype(np.float32)
    assert np.array_equal(sum(p.astype(np.float64) for p in planes(x)), x.astype(np.float64))
    assert hidden_state_error(PRODUCTS, K) <= BOUND / 10


@pytest.mark.parametrize("K", [256, 512, 1536])
@pytest.mark.parametrize("lost", range(6))
def test_bound_finds_a_lost_product(lost, K):
    assert hidden_state_error([p for i, p in enumerate(PRODUCTS) if i != lost], K) > 2 * BOUND


@pytest.mark.parametrize("K", [256, 512, 1536])
@pytest.mark.parametrize("right,wrong", [((0, 2), (0, 1)), ((2, 0), (1, 0)), ((1, 1), (1, 2)), ((0, 1), (0, 2)), ((1, 0), (2, 0))])
def test_bound_finds_a_misplaced_plane(right, wrong, K):
    assert hidden_state_error([wrong if p == right else p for p in PRODUCTS], K) > 2 * BOUND
