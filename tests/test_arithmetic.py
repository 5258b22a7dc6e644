"""Identities of arithmetic that the kernels rely on, checked with numpy."""
import numpy as np


def test_quotient_by_reciprocal():
    """The encoder's quotient: an fp64 product with the fp64 reciprocal, rounded once, is the fp32 division."""
    rng = np.random.default_rng(1)
    a = rng.integers(1 << 23, 1 << 24, 4_000_000).astype(np.float32) * np.exp2(rng.integers(-30, 30, 4_000_000)).astype(np.float32)
    b = rng.integers(1 << 23, 1 << 24, 4_000_000).astype(np.float32)
    assert ((a.astype(np.float64) * (1.0 / b.astype(np.float64))).astype(np.float32) == a / b).all()
    # quotients next to the middle between two floats
    q = (rng.integers(1 << 23, 1 << 24, 1_000_000) * 2 + 1).astype(np.float64) / 2
    near = (q * b[:q.size]).astype(np.float32)
    assert ((near.astype(np.float64) * (1.0 / b[:q.size].astype(np.float64))).astype(np.float32) == near / b[:q.size]).all()
