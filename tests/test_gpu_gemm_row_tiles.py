"""GEMVs of 5 to 32 rows with the RMSNorm in front, one dispatch: tiles of 4, 8 and 16 rows by 8 and 16 outputs, around the lines between them
(256 workgroups), with last tiles of one row and one output, rows of one wave sum (512 columns), two and four."""
import pytest

from gpu_util import Harness, same_bits, stepwise_check
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT, INT, WEIGHT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,n,cols", [(5, 1024, 512), (5, 1025, 511), (8, 1024, 1024), (9, 680, 513), (9, 681, 256), (13, 1023, 1000), (16, 1024, 520), (16, 1025, 520), (16, 2048, 512),
                                         (12, 2056, 264), (17, 816, 65), (17, 1365, 1024), (25, 585, 1023), (32, 512, 128), (32, 1024, 1024), (32, 1040, 1024), (32, 2064, 40),
                                         (8, 1024, 1032), (8, 2048, 2048), (8, 2056, 1100), (12, 1360, 2047), (16, 2048, 1536), (16, 2064, 2048), (17, 1361, 1025), (17, 2048, 2041), (32, 33, 2048),
                                         # 8 x 8: where none of the tiles fits, and at 21 to 24 rows
                                         (8, 4104, 512), (5, 8192, 1000), (8, 4100, 1024), (7, 4097, 2041), (24, 680, 512), (22, 673, 1001)])
def test_tiles_of_rows(rows, n, cols):
    N, K = rows * n, rows * cols
    ks = [KernelSpec("rmsnorm", "bf16", 0, (Ref(EXT, 0), Ref(WEIGHT, 1)), cols, rows=rows, cols=cols, eps=1e-6),
          KernelSpec("gemv", "bf16", 1, (Ref(WEIGHT, 0), Ref(INT, 0)), n, rows=rows, cols=cols),
          KernelSpec("gelu", "bf16", 1, (Ref(INT, 1),), N),
          KernelSpec("add", "bf16", 1, (Ref(INT, 1), Ref(EXT, 1)), N, m=N),
          KernelSpec("add", "bf16", 1, (Ref(INT, 1), Ref(WEIGHT, 2)), N, m=n)]
    spec = ChainSpec(f"tiles_{rows}x{n}x{cols}", ks, [TensorSpec("bf16", K), TensorSpec("bf16", N)], [TensorSpec("bf16", K), TensorSpec("bf16", N)],
                     [TensorSpec("bf16", n * cols, ("normal", 0.0, 0.05)), TensorSpec("bf16", cols, ("normal", 1.0, 0.1)), TensorSpec("bf16", n)], [0, 1], 7500)
    h = Harness(spec)
    assert h.chain.graph_dispatches()[0] == 1
    x_np, x_dev = h.inputs(3)
    ref = h.run("eager", x_dev)
    for mode in ("copy", "indirect"):
        h.scrub()
        got = h.run(mode, x_dev)
        assert all(same_bits(a, b) for a, b in zip(ref, got)), mode
    h.scrub()
    stepwise_check(h, x_np, x_dev, rtol=2.0 ** -7)      # one bf16 ulp, every kernel
    h.close()
