"""k_gemm_tile with kernels behind it: outputs and operands that no 4-byte word reaches (an odd number of outputs, externals at an odd element), rows that 16-byte
loads reach and rows that they do not (columns no multiple of 8, h at an odd element), in each of its tiles.  Operands wait in LDS, as pairs or one by one, or in registers."""
import pytest
import torch

from gpu_util import Harness, same_bits, stepwise_check
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT, INT, WEIGHT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tail", ["gelu add add", "add gelu add", "gelu"])
@pytest.mark.parametrize("rows,n,cols", [(6, 33, 2056), (6, 34, 2056), (6, 33, 2060), (17, 1, 2056), (40, 47, 2061), (16, 4095, 2064),        # 16 x 16
                                         (81, 1501, 136), (81, 1502, 136), (81, 1501, 132), (96, 35, 2056), (96, 36, 2061),                   # 32 x 32
                                         (100, 4097, 72), (100, 4098, 72), (100, 4100, 72), (100, 4097, 71)])                                 # 64 x 32
def test_layouts(rows, n, cols, tail):
    N, K = rows * n, rows * cols
    ks = [KernelSpec("gemv", "bf16", 0, (Ref(WEIGHT, 0), Ref(EXT, 0)), n, rows=rows, cols=cols)]
    for i, op in enumerate(tail.split()):
        src = Ref(INT, i)
        ks.append(KernelSpec("gelu", "bf16", i + 1, (src,), N) if op == "gelu"
                  else KernelSpec("add", "bf16", i + 1, (src, Ref(EXT, 1)) if i == 1 else (Ref(EXT, 2), src), N, m=N))
    spec = ChainSpec(f"layout_{rows}x{n}x{cols}", ks, [TensorSpec("bf16", K), TensorSpec("bf16", N), TensorSpec("bf16", N)], [TensorSpec("bf16", N) for _ in ks],
                     [TensorSpec("bf16", n * cols, ("normal", 0.0, 0.05))], list(range(len(ks))), 7700)
    h = Harness(spec)
    assert h.chain.graph_dispatches()[0] == 1
    x_np, x_dev = h.inputs(1)

    def moved(which):
        out = []
        for i, x in enumerate(x_dev):
            big = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)
            at = 1 if i in which else 0
            big[at:at + x.numel()].copy_(x)
            out.append(big[at:at + x.numel()])
        torch.cuda.synchronize()
        return out

    ref = h.run("eager", x_dev)
    for ext in (x_dev, moved((1,)), moved((2,)), moved((0,)), moved((0, 1, 2))):
        for mode in ("copy", "indirect"):
            h.scrub()
            got = h.run(mode, ext)
            assert all(same_bits(a, b) for a, b in zip(ref, got)), mode
    h.scrub()
    stepwise_check(h, x_np, x_dev, rtol=2.0 ** -7)      # one bf16 ulp, every kernel
    h.close()
