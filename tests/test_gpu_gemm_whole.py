"""GEMVs of 17 rows and more with kernels behind them, up to 2048 columns: one workgroup per CU, all of its loads at once.  Around the edges of the tiles (16 and 32 rows
and outputs), of the grid (256 workgroups), of a wave's blocks of 64 columns (512, 1024, 1536), with rows that end inside a vector; tails of every form."""
import numpy as np
import pytest

from gpu_util import Harness, same_bits, stepwise_check
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT, INT, WEIGHT, make_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tail", ["gelu add add", "mul gelu"])
@pytest.mark.parametrize("rows,n,cols", [(33, 16, 8), (33, 1, 64), (40, 300, 511), (64, 1024, 512), (64, 1025, 513), (49, 1023, 1024), (128, 512, 1025), (127, 513, 1000), (65, 1700, 1536),
                                         (64, 2048, 1537), (64, 2049, 2048), (80, 2048, 2048), (72, 2730, 1984), (79, 700, 2047), (100, 2048, 2048), (200, 300, 72), (2000, 20, 130),
                                         # tiles of two rows of tiles by one: where neither 1 x 1 nor 1 x 2 fits, from 81 rows on
                                         (96, 1360, 512), (81, 1345, 1001), (96, 1352, 1352), (145, 801, 1536), (150, 816, 2047), (150, 810, 1024), (4100, 16, 72)])
def test_shapes_and_tails(rows, n, cols, tail):
    N, K = rows * n, rows * cols
    ks = [KernelSpec("rmsnorm", "bf16", 0, (Ref(EXT, 0), Ref(WEIGHT, 1)), cols, rows=rows, cols=cols, eps=1e-6),
          KernelSpec("gemv", "bf16", 1, (Ref(WEIGHT, 0), Ref(INT, 0)), n, rows=rows, cols=cols)]
    for op in tail.split():
        src = Ref(INT, ks[-1].out)
        ks.append(KernelSpec("gelu", "bf16", ks[-1].out + 1, (src,), N) if op == "gelu" else KernelSpec(op, "bf16", ks[-1].out + 1, (Ref(EXT, 1), src), N, m=N))
    spec = ChainSpec(f"whole_{rows}x{n}x{cols}", ks, [TensorSpec("bf16", K), TensorSpec("bf16", N)], [TensorSpec("bf16", K)] + [TensorSpec("bf16", N) for _ in range(4)],
                     [TensorSpec("bf16", n * cols, ("normal", 0.0, 0.05)), TensorSpec("bf16", cols, ("normal", 1.0, 0.1))], sorted({k.out for k in ks}), 7600)
    h = Harness(spec)
    assert h.chain.graph_dispatches()[0] == 2
    x_np, x_dev = h.inputs(3)
    ref = h.run("eager", x_dev)
    for mode in ("copy", "indirect"):
        h.scrub()
        got = h.run(mode, x_dev)
        assert all(same_bits(a, b) for a, b in zip(ref, got)), mode
    h.scrub()
    stepwise_check(h, x_np, x_dev, rtol=2.0 ** -7)      # one bf16 ulp, every kernel
    h.close()


@pytest.mark.parametrize("rows,n,cols", [(33, 17, 8), (49, 33, 66), (64, 1024, 513), (40, 1030, 1000), (40, 2730, 1023), (72, 1640, 511), (80, 2049, 777), (64, 2047, 513), (64, 1300, 200),
                                         (96, 1360, 512), (150, 810, 1024), (145, 801, 1536), (150, 816, 2048)])
def test_in_a_chain_beyond_the_cache(rows, n, cols):
    """A GEMV of 269 MB elsewhere in the chain makes these take the weights by non-temporal loads: up to 80 rows and 1024 columns whose rows share cache lines,
    tiles of 1 x 1, 1 x 2 and 2 x 2, one and two blocks a wave; tiles of 2 x 1 whose rows share none, one to four blocks."""
    big, N, K = 65600, rows * n, rows * cols
    ks = [KernelSpec("gemv", "bf16", 3, (Ref(WEIGHT, 1), Ref(EXT, 2)), big, rows=5, cols=2048),
          KernelSpec("gemv", "bf16", 0, (Ref(WEIGHT, 0), Ref(EXT, 0)), n, rows=rows, cols=cols),
          KernelSpec("gelu", "bf16", 1, (Ref(INT, 0),), N),
          KernelSpec("add", "bf16", 2, (Ref(EXT, 1), Ref(INT, 1)), N, m=N)]
    spec = ChainSpec(f"whole_beyond_{rows}x{n}x{cols}", ks, [TensorSpec("bf16", K), TensorSpec("bf16", N), TensorSpec("bf16", 5 * 2048)],
                     [TensorSpec("bf16", N) for _ in range(3)] + [TensorSpec("bf16", 5 * big)],
                     [TensorSpec("bf16", n * cols, ("normal", 0.0, 0.05)), TensorSpec("bf16", big * 2048)], [0, 1, 2], 7610)
    small = make_weights(ChainSpec(spec.name, [], [], [], spec.weights[:1], [], spec.seed))
    h = Harness(spec, weights_np=small + [np.zeros(big * 2048, np.uint16)])
    assert h.chain.graph_dispatches()[0] == 2
    x_np, x_dev = h.inputs(0)
    ref = h.run("eager", x_dev)
    for mode in ("copy", "indirect"):
        h.scrub()
        got = h.run(mode, x_dev)
        assert all(same_bits(a, b) for a, b in zip(ref, got)), mode
    h.scrub()
    stepwise_check(h, x_np, x_dev, rtol=2.0 ** -7, kernels=range(1, len(ks)))
    h.close()
