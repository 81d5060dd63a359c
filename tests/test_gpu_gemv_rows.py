"""GEMV dispatches with prologue and epilogue at one to four rows of any width: around every edge of the
kernel's forms (rows that end inside a vector, inside a chunk of 2048 columns, on it; one and two weight rows
per wave; one to four chunks), graphs equal eager bit for bit and every kernel matches the oracle."""
import pytest

from gpu_util import Harness, same_bits, say, stepwise_check
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT, INT, WEIGHT, decode_chain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,hidden", [(r, h) for h in (7, 8, 9, 61, 520, 1023, 1024, 1030, 2047, 2049, 2056, 4091, 4096) for r in (1, 2, 3, 4)] +
                         [(r, h) for h in (4104, 5000, 6142, 6151, 6144, 7000, 8191, 8192, 8200) for r in (1, 4)])
def test_rows_of_any_width(rows, hidden):
    spec = decode_chain(batch=rows, layers=3, blocks_per_layer=1, hidden=hidden, n_ext=3)
    h = Harness(spec, capture=False)
    merged, unmerged = h.chain.graph_dispatches()
    say(f"{spec.name}: {unmerged} kernels in {merged} dispatches")
    # sub-block 0 reads an external, the other two rename the stream: one dispatch each; three and four rows of more than 4096
    # columns leave the RMSNorm in a dispatch of its own (more than 256 workgroups: it is dearer in front of each)
    assert merged == (6 if rows > 2 and hidden > 4096 else 3) if 8 <= hidden <= 8192 else merged > 3
    h.chain.capture(h.stream)
    for t in range(2):
        x_np, x_dev = h.inputs(t)
        outs = {}
        for mode in ("eager", "copy", "indirect"):
            h.scrub()
            outs[mode] = h.run(mode, x_dev)[0]
        assert same_bits(outs["eager"], outs["copy"]) and same_bits(outs["eager"], outs["indirect"]), t
    h.scrub()
    stepwise_check(h, x_np, x_dev, rtol=2.0 ** -7)      # one bf16 ulp, every kernel
    h.close()


@pytest.mark.parametrize("cols", [8, 61, 256, 511, 512, 513, 1000, 1023])
@pytest.mark.parametrize("rows,n", [(1, 1024), (1, 2053), (2, 1030), (3, 1024), (3, 1031), (4, 1027), (4, 4096)])
def test_short_rows_of_many_outputs(rows, n, cols):
    """More outputs than columns, two weight rows per wave: rows of one and two pieces of 512 columns, with the RMSNorm in front, with kernels that
    ride and alone; h also straight from an external."""
    N, K = rows * n, rows * cols
    ks = [KernelSpec("rmsnorm", "bf16", 0, (Ref(EXT, 0), Ref(WEIGHT, 1)), cols, rows=rows, cols=cols, eps=1e-6),
          KernelSpec("gemv", "bf16", 1, (Ref(WEIGHT, 0), Ref(INT, 0)), n, rows=rows, cols=cols),
          KernelSpec("gelu", "bf16", 1, (Ref(INT, 1),), N),
          KernelSpec("gemv", "bf16", 2, (Ref(WEIGHT, 0), Ref(EXT, 0)), n, rows=rows, cols=cols),
          KernelSpec("add", "bf16", 2, (Ref(INT, 2), Ref(EXT, 1)), N, m=N),
          KernelSpec("gemv", "bf16", 3, (Ref(WEIGHT, 0), Ref(EXT, 0)), n, rows=rows, cols=cols),
          KernelSpec("rmsnorm", "bf16", 0, (Ref(EXT, 0), Ref(WEIGHT, 1)), cols, rows=rows, cols=cols, eps=1e-6)]
    spec = ChainSpec(f"short_rows_{rows}x{n}x{cols}", ks, [TensorSpec("bf16", K), TensorSpec("bf16", N)], [TensorSpec("bf16", K)] + [TensorSpec("bf16", N) for _ in range(3)],
                     [TensorSpec("bf16", n * cols, ("normal", 0.0, 0.05)), TensorSpec("bf16", cols, ("normal", 1.0, 0.1))], [0, 1, 2, 3], 7410)
    h = Harness(spec)
    assert h.chain.graph_dispatches()[0] == 4
    for t in range(2):
        x_np, x_dev = h.inputs(t)
        ref = h.run("eager", x_dev)
        for mode in ("copy", "indirect"):
            h.scrub()
            got = h.run(mode, x_dev)
            assert all(same_bits(a, b) for a, b in zip(ref, got)), (mode, t)
    h.scrub()
    stepwise_check(h, x_np, x_dev, rtol=2.0 ** -7)      # one bf16 ulp, every kernel
    h.close()
