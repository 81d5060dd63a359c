"""Runs of scale + bias + ReLU kernels in one dispatch: the same bits as kernel by kernel, both buffers of a chain that
alternates between two (what no later kernel of a run overwrites is stored), at vectors that straddle two channels, a
partial last vector, one channel, as many channels as a run takes and one more, runs longer than one dispatch holds."""
import pytest

import paper_2503_19779_amd as pg  # noqa: F401
from gpu_util import Harness, same_bits, stepwise_check
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT, INT, WEIGHT

pytestmark = pytest.mark.gpu


def _chain(dtype, batch, channels, inner, kernels, seed=7100):
    n = batch * channels * inner
    ks = []
    for k in range(kernels):
        # kernel 2 takes its scale from an external, kernel 4 its bias from an internal buffer that is no part of the chain
        s = Ref(EXT, 1) if k == 2 else Ref(WEIGHT, 2 * (k % 3))
        b = Ref(INT, 2) if k == 4 else Ref(WEIGHT, 2 * (k % 3) + 1)
        ks.append(KernelSpec("scale_bias_relu", dtype, k % 2, (Ref(EXT, 0) if k == 0 else Ref(INT, (k - 1) % 2), s, b), n,
                             inner=inner, channels=channels))
    ks.insert(0, KernelSpec("add", dtype, 2, (Ref(EXT, 1), Ref(WEIGHT, 1)), channels, m=channels))
    ks.append(KernelSpec("scale_bias_relu", dtype, (kernels - 1) % 2, (Ref(INT, (kernels - 1) % 2), Ref(WEIGHT, 0), Ref(INT, 2)), n,
                         inner=inner, channels=channels))                        # in place
    return ChainSpec(f"sbr_run_{dtype}_{batch}x{channels}x{inner}_{kernels}", ks,
                     [TensorSpec(dtype, n), TensorSpec(dtype, channels, ("normal", 1.0, 0.1))],
                     [TensorSpec(dtype, n), TensorSpec(dtype, n), TensorSpec(dtype, channels)],
                     [TensorSpec(dtype, channels, ("normal", float(i % 2 == 0), 0.1)) for i in range(6)], [0, 1, 2], seed)


@pytest.mark.parametrize("dtype,batch,channels,inner,kernels,nodes", [
    ("f32", 2, 3, 16, 6, 2), ("f32", 3, 5, 7, 6, 2), ("f32", 1, 1, 4, 3, 2), ("f32", 2, 128, 9, 5, 2), ("f32", 2, 129, 9, 5, 7), ("f32", 2, 7, 3, 5, 7),
    ("f32", 1, 3, 4099, 20, 3), ("f32", 3, 63, 6000, 4, 2), ("f32", 5, 33, 6643, 4, 2), ("bf16", 2, 3, 16, 6, 2), ("bf16", 3, 5, 11, 16, 3), ("bf16", 1, 1, 9, 2, 2),
    ("bf16", 3, 5, 139811, 3, 2)])
def test_runs_of_scale_bias_relu(dtype, batch, channels, inner, kernels, nodes):
    h = Harness(_chain(dtype, batch, channels, inner, kernels), capture=False)
    assert h.chain.graph_dispatches() == (nodes, kernels + 2)
    h.chain.capture(h.stream)
    for t in range(3):
        x_np, x_dev = h.inputs(t)
        h.scrub()
        want = h.run("eager", x_dev)
        for mode in ("copy", "indirect", "copy"):
            h.scrub()
            got = h.run(mode, x_dev)
            for o in range(3):
                assert same_bits(want[o], got[o]), (mode, t, o)
    if batch * channels * inner < 100000:
        h.scrub()
        stepwise_check(h, x_np, x_dev)
    h.close()


@pytest.mark.parametrize("kernels", [8, 9, 16])
@pytest.mark.parametrize("dtype,batch,channels,inner", [("f32", 17, 128, 512), ("f32", 17, 64, 1027), ("f32", 1700, 128, 5), ("f32", 3, 7, 256), ("f32", 4, 8, 260), ("f32", 9, 3, 509),
                                                        ("bf16", 33, 64, 1024), ("bf16", 17, 125, 1001), ("bf16", 5, 3, 516), ("bf16", 40, 11, 9)])
def test_stretches_of_one_two_and_many_channels(dtype, batch, channels, inner, kernels):
    """A wave's stretch that ends where a channel does, just before and behind, or holds many channels, one and two vectors per lane, up to the
    longest run; scales and biases from weights and from externals."""
    n = batch * channels * inner
    ks = [KernelSpec("scale_bias_relu", dtype, k % 2, (Ref(INT, (k - 1) % 2) if k else Ref(EXT, 0), Ref(EXT, 1) if k % 3 == 0 else Ref(WEIGHT, 0),
                                                       Ref(EXT, 2) if k % 4 == 1 else Ref(WEIGHT, 1)), n, inner=inner, channels=channels) for k in range(kernels)]
    spec = ChainSpec(f"stretch_{dtype}_{batch}x{channels}x{inner}_{kernels}", ks,
                     [TensorSpec(dtype, n), TensorSpec(dtype, channels, ("normal", 1.0, 0.1)), TensorSpec(dtype, channels, ("normal", 0.0, 0.1))],
                     [TensorSpec(dtype, n), TensorSpec(dtype, n)],
                     [TensorSpec(dtype, channels, ("normal", 1.0, 0.1)), TensorSpec(dtype, channels, ("normal", 0.0, 0.1))], [0, 1], 8600)
    h = Harness(spec)
    assert h.chain.graph_dispatches() == (1, kernels)
    for t in range(2):
        _, x_dev = h.inputs(t)
        h.scrub()
        want = h.run("eager", x_dev)
        for mode in ("copy", "indirect"):
            h.scrub()
            got = h.run(mode, x_dev)
            assert all(same_bits(a, b) for a, b in zip(want, got)), (mode, t)
    h.close()
