"""fp32 GELU against the definition in 64 bits: both tails, tiny and huge inputs, zeros, infinities and NaN."""
import numpy as np
import pytest
from scipy.special import erfc

import paper_2503_19779_amd as pg  # noqa: F401
from gpu_util import Harness
from paper_2503_19779_amd.binding import to_device
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT

pytestmark = pytest.mark.gpu


def test_gelu_f32_is_the_rounded_definition():
    rng = np.random.default_rng(5)
    a = np.concatenate([-np.logspace(-44, np.log10(40), 300000), np.logspace(-44, 3, 100000), rng.normal(0, 1, 400000), rng.normal(0, 5, 200000),
                        [0.0, -0.0, 3e38, -3e38, -14.1, -14.2, -37.5, -39.6, -39.7, 1e-38, -1e-38]]).astype(np.float32)
    special = np.array([np.inf, -np.inf, np.nan], dtype=np.float32)
    x = np.concatenate([a, special])
    spec = ChainSpec("gelu_f32", [KernelSpec("gelu", "f32", 0, (Ref(EXT, 0),), x.size)], [TensorSpec("f32", x.size)], [TensorSpec("f32", x.size)], [], [0], 1)
    h = Harness(spec)
    got = h.run("eager", [to_device(x)])[0]
    h.close()
    d = a.astype(np.float64)
    want = 0.5 * d * erfc(d * -0.70710678118654752440)
    err = np.abs(got[:a.size].astype(np.float64) - want)
    # half a unit in the last place of the result (2^-24 relative, 2^-150 among the subnormals) and the 1e-13 the formula may add
    assert np.all(err <= np.maximum(np.abs(want) * (2.0 ** -24 * (1 + 1e-5)), 2.0 ** -149))
    assert np.all(np.mean(got[:a.size] != want.astype(np.float32)) <= 1e-5)
    assert got[a.size] == np.inf and np.isnan(got[a.size + 1]) and np.isnan(got[a.size + 2])
