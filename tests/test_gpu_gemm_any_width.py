"""Matrix-core GEMV dispatches at five rows and more of any width, around the edges of their forms: rows that end inside a
vector, inside a K-block of 64 columns, on and around 1024 and 2048 columns (K-steps per wave; the prologue's limit),
fewer K-blocks than waves, ragged column blocks, one and several tiles of rows, every tile size.  Graphs equal eager bit
for bit and every kernel matches the oracle."""
import numpy as np
import pytest

from gpu_util import Harness, same_bits, say, stepwise_check
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT, INT, WEIGHT, decode_chain, make_weights

pytestmark = pytest.mark.gpu


def _check(h, rows=None):
    for t in range(2):
        x_np, x_dev = h.inputs(t)
        outs = {}
        for mode in ("eager", "copy", "indirect"):
            h.scrub()
            outs[mode] = h.run(mode, x_dev)
        for o in range(len(h.spec.outputs)):
            assert same_bits(outs["eager"][o], outs["copy"][o]) and same_bits(outs["eager"][o], outs["indirect"][o]), (t, o)
    h.scrub()
    stepwise_check(h, x_np, x_dev, rows=rows, rtol=2.0 ** -7)      # one bf16 ulp, every kernel
    h.close()


@pytest.mark.parametrize("rows,hidden", [(r, h) for h in (16, 31, 72, 520, 1023, 1024, 1030, 2047, 2056) for r in (5, 9, 16, 17, 32, 33, 64, 81, 100)] +
                         [(r, h) for h in (127, 1016, 2041, 4096, 4107) for r in (8, 13, 25, 80, 130)])
def test_square_chains(rows, hidden):
    spec = decode_chain(batch=rows, layers=3, blocks_per_layer=1, hidden=hidden, n_ext=3)
    h = Harness(spec, capture=False)
    assert h.chain.graph_dispatches()[0] == (3 if rows <= 32 and hidden <= 2048 else 6)
    h.chain.capture(h.stream)
    _check(h, rows=sorted({0, rows // 2, rows - 1}))


@pytest.mark.parametrize("rows,n,cols", [(6, 17, 40), (17, 4097, 33), (33, 8195, 136), (64, 8192, 200), (77, 8192, 71), (128, 8196, 64), (40, 4096, 72), (20, 8193, 1024),
                                         (200, 40, 300), (96, 2050, 56), (11, 15, 64), (5, 300, 8),
                                         (6, 1, 40), (9, 2, 1030), (33, 5, 136), (64, 12, 4096), (81, 7, 2056), (128, 8, 2048), (70, 3, 33), (200, 16, 1030), (6, 8201, 40),
                                         (65, 2050, 2304), (80, 2304, 2601), (70, 40, 2304), (18, 4112, 2056)])
def test_other_output_widths(rows, n, cols):
    """RMSNorm -> GEMV -> GELU -> add -> add with a broadcast operand, n outputs per row; h then comes straight from
    an external, at an address that is no multiple of 16 bytes."""
    N, K = rows * n, rows * cols
    ks = [KernelSpec("rmsnorm", "bf16", 0, (Ref(EXT, 0), Ref(WEIGHT, 1)), cols, rows=rows, cols=cols, eps=1e-6),
          KernelSpec("gemv", "bf16", 1, (Ref(WEIGHT, 0), Ref(INT, 0)), n, rows=rows, cols=cols),
          KernelSpec("gelu", "bf16", 1, (Ref(INT, 1),), N),
          KernelSpec("add", "bf16", 2, (Ref(EXT, 1), Ref(INT, 1)), N, m=N),
          KernelSpec("add", "bf16", 2, (Ref(INT, 2), Ref(WEIGHT, 2)), N, m=n),
          KernelSpec("gemv", "bf16", 1, (Ref(WEIGHT, 0), Ref(EXT, 0)), n, rows=rows, cols=cols),
          KernelSpec("mul", "bf16", 3, (Ref(INT, 1), Ref(INT, 2)), N, m=N)]
    spec = ChainSpec(f"gemm_{rows}x{n}x{cols}", ks, [TensorSpec("bf16", K), TensorSpec("bf16", N)],
                     [TensorSpec("bf16", K)] + [TensorSpec("bf16", N) for _ in range(3)],
                     [TensorSpec("bf16", n * cols, ("normal", 0.0, 0.05)), TensorSpec("bf16", cols, ("normal", 1.0, 0.1)), TensorSpec("bf16", n)], [0, 1, 2, 3], 7200)
    h = Harness(spec)
    say(f"{spec.name}: {h.chain.graph_dispatches()}")
    x_np, x_dev = h.inputs(5)
    ref = h.run("eager", x_dev)
    import torch
    moved = []
    for x in x_dev:
        big = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)
        big[1:1 + x.numel()].copy_(x)
        moved.append(big[1:1 + x.numel()])
    torch.cuda.synchronize()
    for mode in ("eager", "copy", "indirect"):
        h.scrub()
        got = h.run(mode, moved)
        for o in range(4):
            assert same_bits(ref[o], got[o]), (mode, o)
    _check(h)


def test_rows_of_sixteen_million_columns():
    rows, n, cols = 5, 3, (1 << 24) + 8
    k = KernelSpec("gemv", "bf16", 0, (Ref(WEIGHT, 0), Ref(EXT, 0)), n, rows=rows, cols=cols)
    h = Harness(ChainSpec("gemm_long", [k], [TensorSpec("bf16", rows * cols)], [TensorSpec("bf16", rows * n)], [TensorSpec("bf16", n * cols)], [0], 7201))
    _check(h)


@pytest.mark.parametrize("rows,n,cols", [(1, 1030, 2048), (1, 5, 61), (2, 2056, 1024), (4, 2046, 520), (5, 2048, 2048), (16, 40, 1030), (20, 33, 520), (40, 48, 1024), (72, 2304, 2304),
                                         (81, 37, 2048), (128, 2048, 256), (130, 8192, 136)])
@pytest.mark.parametrize("tail", ["gelu", "add", "mul", "gelu mul", "add gelu"])
def test_short_tails(rows, n, cols, tail):
    """One or two kernels behind the GEMV, GELU alone, in front and last, out of place, with and without the RMSNorm in front."""
    N = rows * n
    ks = [KernelSpec("rmsnorm", "bf16", 0, (Ref(EXT, 0), Ref(WEIGHT, 1)), cols, rows=rows, cols=cols, eps=1e-6)]
    for h in (Ref(INT, 0), Ref(EXT, 0)):
        ks.append(KernelSpec("gemv", "bf16", 1, (Ref(WEIGHT, 0), h), n, rows=rows, cols=cols))
        for op in tail.split():
            src = Ref(INT, ks[-1].out)
            ks.append(KernelSpec("gelu", "bf16", ks[-1].out + 1, (src,), N) if op == "gelu" else KernelSpec(op, "bf16", ks[-1].out + 1, (Ref(EXT, 1), src), N, m=N))
    spec = ChainSpec(f"tail_{rows}x{n}x{cols}", ks, [TensorSpec("bf16", rows * cols), TensorSpec("bf16", N)],
                     [TensorSpec("bf16", rows * cols)] + [TensorSpec("bf16", N) for _ in range(3)],
                     [TensorSpec("bf16", n * cols, ("normal", 0.0, 0.05)), TensorSpec("bf16", cols, ("normal", 1.0, 0.1))], [], 7300)
    spec.outputs[:] = sorted({k.out for k in spec.kernels})
    h = Harness(spec)
    merged, unmerged = h.chain.graph_dispatches()
    assert merged < unmerged
    _check(h)


@pytest.mark.parametrize("rows", [40, 100])
def test_weights_beyond_the_cache(rows):
    """More than 256 MB of weights in one chain: the forms that take them by non-temporal loads, same results."""
    spec = decode_chain(batch=rows, layers=33, blocks_per_layer=1, hidden=2048, n_ext=2)
    h = Harness(spec)
    x_np, x_dev = h.inputs(0)
    ref = h.run("eager", x_dev)
    for mode in ("copy", "indirect"):
        h.scrub()
        assert same_bits(h.run(mode, x_dev)[0], ref[0]), mode
    h.scrub()
    stepwise_check(h, x_np, x_dev, rows=[0, rows - 1], rtol=2.0 ** -7)
    h.close()


@pytest.mark.parametrize("rows,n,cols", [(17, 40, 1088), (40, 1030, 1536), (64, 2049, 1984), (80, 33, 1600), (72, 15, 1152), (33, 1030, 1544),
                                         (81, 37, 64), (81, 300, 64), (100, 1990, 1024), (128, 1990, 1088), (97, 2050, 2048), (128, 24, 4160), (66, 2310, 2304), (100, 1030, 1544), (81, 50, 1601)])
def test_shapes_in_a_chain_beyond_the_cache(rows, n, cols):
    """One GEMV of 269 MB makes the rest of the chain use the forms for weights beyond the cache: ragged outputs, K tails, widths without such
    a form; behind an RMSNorm of its own, with kernels that ride and alone."""
    big, N, K = 65600, rows * n, rows * cols
    ks = [KernelSpec("gemv", "bf16", 4, (Ref(WEIGHT, 2), Ref(EXT, 2)), big, rows=5, cols=2048),
          KernelSpec("rmsnorm", "bf16", 0, (Ref(EXT, 0), Ref(WEIGHT, 1)), cols, rows=rows, cols=cols, eps=1e-6),
          KernelSpec("gemv", "bf16", 1, (Ref(WEIGHT, 0), Ref(INT, 0)), n, rows=rows, cols=cols),
          KernelSpec("gelu", "bf16", 1, (Ref(INT, 1),), N),
          KernelSpec("add", "bf16", 2, (Ref(EXT, 1), Ref(INT, 1)), N, m=N),
          KernelSpec("gemv", "bf16", 3, (Ref(WEIGHT, 0), Ref(EXT, 0)), n, rows=rows, cols=cols),
          KernelSpec("rmsnorm", "bf16", 0, (Ref(EXT, 0), Ref(WEIGHT, 1)), cols, rows=rows, cols=cols, eps=1e-6)]
    spec = ChainSpec(f"beyond_{rows}x{n}x{cols}", ks, [TensorSpec("bf16", K), TensorSpec("bf16", N), TensorSpec("bf16", 5 * 2048)],
                     [TensorSpec("bf16", K)] + [TensorSpec("bf16", N) for _ in range(3)] + [TensorSpec("bf16", 5 * big)],
                     [TensorSpec("bf16", n * cols, ("normal", 0.0, 0.05)), TensorSpec("bf16", cols, ("normal", 1.0, 0.1)), TensorSpec("bf16", big * 2048)], [0, 1, 2, 3], 7400)
    small = make_weights(ChainSpec(spec.name, [], [], [], spec.weights[:2], [], spec.seed))
    h = Harness(spec, weights_np=small + [np.zeros(big * 2048, np.uint16)])
    x_np, x_dev = h.inputs(0)
    ref = h.run("eager", x_dev)
    for mode in ("copy", "indirect"):
        h.scrub()
        got = h.run(mode, x_dev)
        assert all(same_bits(a, b) for a, b in zip(ref, got)), mode
    h.scrub()
    stepwise_check(h, x_np, x_dev, rtol=2.0 ** -7, kernels=range(1, len(ks)))
    h.close()
