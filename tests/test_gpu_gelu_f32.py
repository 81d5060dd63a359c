"""fp32 GELU against the definition in more than 64 bits: both tails, tiny and huge inputs, zeros, infinities and NaN, and inputs
whose result lies so close to the middle of two fp32 values that an error of 5e-15 turns it."""
import numpy as np
import pytest
from scipy.special import erfc

import paper_2503_19779_amd as pg  # noqa: F401
from gpu_util import Harness
from paper_2503_19779_amd.binding import to_device
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT

pytestmark = pytest.mark.gpu

# (input, a * Phi(a) in 113 bits, rounded to fp32): all within 2e-15 of the middle, relative
CLOSE = """
0x1.a0e308p-10 0x1.a16a74p-11
0x1.5be652p-7 0x1.5ed8c6p-8
0x1.8332fp-7 0x1.86d976p-8
0x1.f82964p-7 0x1.fe59cp-8
0x1.4e2deap-6 0x1.539e14p-7
0x1.92798cp-3 0x1.d12deap-4
0x1.c16d0ep-3 0x1.07bebep-3
0x1.5b4488p-2 0x1.b7767cp-3
-0x1.a0e308p-10 -0x1.a05b9cp-11
-0x1.5be652p-7 -0x1.58f3dep-8
-0x1.8332fp-7 -0x1.7f8c6ap-8
-0x1.f82964p-7 -0x1.f1f908p-8
-0x1.92798cp-3 -0x1.53c52ep-4
-0x1.4e2deap-6 -0x1.48bdcp-7
"""


def _gelu(x):
    spec = ChainSpec("gelu_f32", [KernelSpec("gelu", "f32", 0, (Ref(EXT, 0),), x.size)], [TensorSpec("f32", x.size)], [TensorSpec("f32", x.size)], [], [0], 1)
    h = Harness(spec)
    got = h.run("eager", [to_device(x)])[0]
    h.close()
    return got


def test_results_next_to_the_middle_of_two_fp32_values():
    pairs = np.array([[float.fromhex(v) for v in line.split()] for line in CLOSE.split("\n") if line])
    assert np.array_equal(_gelu(pairs[:, 0].astype(np.float32)).astype(np.float64), pairs[:, 1])


def test_gelu_f32_is_the_rounded_definition():
    rng = np.random.default_rng(5)
    a = np.concatenate([-np.logspace(-44, np.log10(40), 300000), np.logspace(-44, 3, 100000), rng.normal(0, 1, 400000), rng.normal(0, 5, 200000),
                        [0.0, -0.0, 3e38, -3e38, -14.1, -14.2, -37.5, -39.6, -39.7, 1e-38, -1e-38]]).astype(np.float32)
    special = np.array([np.inf, -np.inf, np.nan], dtype=np.float32)
    x = np.concatenate([a, special])
    got = _gelu(x)
    # erfc at the rounded argument, and the argument's rounding error to first order
    d = a.astype(np.float64)
    z = d * -0.70710678118654752440
    err_z = (-a.astype(np.longdouble) / np.sqrt(np.longdouble(2)) - z).astype(np.float64)
    want = 0.5 * d * (erfc(z) - 2 / np.sqrt(np.pi) * np.exp(-np.minimum(z * z, 1e4)) * err_z)
    err = np.abs(got[:a.size].astype(np.float64) - want)
    # half a unit in the last place of the result (2^-24 relative, 2^-150 among the subnormals) and what the reference's erfc is off in the far tail
    assert np.all(err <= np.maximum(np.abs(want) * (2.0 ** -24 * (1 + 1e-5)), 2.0 ** -149))
    assert np.all(np.mean(got[:a.size] != want.astype(np.float32)) <= 1e-5)
    assert got[a.size] == np.inf and np.isnan(got[a.size + 1]) and np.isnan(got[a.size + 2])
