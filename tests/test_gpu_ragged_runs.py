"""Runs of bf16 elementwise kernels over tensors whose length is no multiple of a 16-byte vector: the workgroup that owns
the partial vector works it out element by element; in place, out of place, with broadcast operands, from externals at any
element boundary, up to eight kernels per dispatch from 16384 elements on."""
import pytest
import torch

from gpu_util import Harness, same_bits, stepwise_check
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT, INT, WEIGHT, elementwise_chain

pytestmark = pytest.mark.gpu


def _moved(x_dev):
    out = []
    for x in x_dev:
        big = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)
        big[3:3 + x.numel()].copy_(x)
        out.append(big[3:3 + x.numel()])
    torch.cuda.synchronize()
    return out


def _check(h):
    for t in range(2):
        x_np, x_dev = h.inputs(t)
        h.scrub()
        want = h.run("eager", x_dev)
        moved = _moved(x_dev)
        for mode, x in (("copy", x_dev), ("indirect", x_dev), ("indirect", moved), ("copy", moved)):
            h.scrub()
            got = h.run(mode, x)
            for o in range(len(want)):
                assert same_bits(want[o], got[o]), (t, mode, o)
    h.scrub()
    stepwise_check(h, x_np, x_dev)
    h.close()


@pytest.mark.parametrize("numel", [1, 7, 9, 511, 2047, 2049, 2048 * 3 + 1, 16383, 16384, 16385, 20479, 100003])
def test_chains(numel):
    h = Harness(elementwise_chain(n_kernels=19, numel=numel, dtype="bf16"))
    assert h.chain.graph_dispatches()[0] == (3 if numel >= 16384 else 5)
    _check(h)


@pytest.mark.parametrize("n", [13, 2051, 6151, 20491, 18432])
def test_general_runs(n):
    ks = [KernelSpec("add", "bf16", 0, (Ref(EXT, 0), Ref(EXT, 1)), n, m=n),
          KernelSpec("mul", "bf16", 1, (Ref(INT, 0), Ref(WEIGHT, 0)), n, m=5),
          KernelSpec("add", "bf16", 2, (Ref(INT, 1), Ref(INT, 0)), n, m=n),
          KernelSpec("gelu", "bf16", 2, (Ref(INT, 2),), n),
          KernelSpec("mul", "bf16", 0, (Ref(INT, 0), Ref(WEIGHT, 0)), n, m=8),
          KernelSpec("add", "bf16", 1, (Ref(EXT, 1), Ref(INT, 2)), n, m=n),
          KernelSpec("add", "bf16", 3, (Ref(INT, 1), Ref(INT, 0)), n, m=n),
          KernelSpec("mul", "bf16", 3, (Ref(INT, 3), Ref(EXT, 0)), n, m=n),
          KernelSpec("add", "bf16", 2, (Ref(INT, 2), Ref(INT, 3)), n, m=1)]
    spec = ChainSpec(f"ragged_{n}", ks, [TensorSpec("bf16", n) for _ in range(2)], [TensorSpec("bf16", n) for _ in range(4)],
                     [TensorSpec("bf16", 8, ("normal", 1.0, 0.3))], [0, 1, 2, 3], 8100)
    h = Harness(spec)
    assert h.chain.graph_dispatches()[0] < len(ks)
    _check(h)


@pytest.mark.parametrize("dtype,n,kernels", [("bf16", 5, 3), ("bf16", 512, 2), ("bf16", 513, 7), ("bf16", 16391, 8), ("bf16", (1 << 20) - 1, 5), ("bf16", (1 << 20) + 1, 3), ("bf16", (1 << 20) + 2056, 8),
                                             ("f32", 3, 4), ("f32", 257, 3), ("f32", 16384, 4), ("f32", 16388, 2), ("f32", 1 << 20, 2), ("f32", (1 << 20) + 4, 2)])
def test_chains_with_periods(dtype, n, kernels):
    """One run of kernels that each take the result of the one before, out of place, every output kept; second operands whole, with a
    period that holds whole vectors and with ones that a vector wraps around."""
    ks, seconds = [], [(Ref(EXT, 1), n), (Ref(WEIGHT, 0), 1), (Ref(WEIGHT, 0), 3), (Ref(WEIGHT, 0), 24)]
    for i in range(kernels):
        a = Ref(INT, i - 1) if i else Ref(EXT, 0)
        if i % 3 == 2 and (dtype == "bf16" or n <= 16384):
            ks.append(KernelSpec("gelu", dtype, i, (a,), n))
        else:
            b, m = seconds[i % 4]
            ks.append(KernelSpec("mul" if i % 2 else "add", dtype, i, (a, b), n, m=m))
    spec = ChainSpec(f"periods_{dtype}_{n}", ks, [TensorSpec(dtype, n) for _ in range(2)], [TensorSpec(dtype, n) for _ in range(kernels)],
                     [TensorSpec(dtype, 24, ("normal", 1.0, 0.3))], list(range(kernels)), 8400)
    h = Harness(spec)
    assert h.chain.graph_dispatches()[0] == -(-kernels // (8 if dtype == "bf16" and n >= 16384 else 4))
    _check(h)


@pytest.mark.parametrize("dtype,n", [("bf16", 1000), ("bf16", 1021), ("bf16", 20000), ("f32", 1021), ("f32", 20000)])
@pytest.mark.parametrize("more", [1, 8, 5000])
def test_periods_longer_than_the_tensor(dtype, n, more):
    """Second operands that are longer than what a kernel takes of them: alone (behind a kernel of another length), in a chain and in a run with two
    live buffers."""
    b = (Ref(EXT, 1),)
    ks = [KernelSpec("add", dtype, 0, (Ref(EXT, 0),) + b, n, m=n + more),
          KernelSpec("mul", dtype, 0, (Ref(INT, 0),) + b, n, m=n + more),
          KernelSpec("add", dtype, 3, (Ref(EXT, 0),) + b, n - 5, m=n + more),
          KernelSpec("mul", dtype, 1, (Ref(EXT, 0),) + b, n, m=n + more),
          KernelSpec("add", dtype, 2, (Ref(INT, 1), Ref(INT, 0)), n, m=n),
          KernelSpec("add", dtype, 1, (Ref(INT, 1),) + b, n, m=n + more)]
    spec = ChainSpec(f"long_periods_{dtype}_{n}_{more}", ks, [TensorSpec(dtype, n), TensorSpec(dtype, n + more)], [TensorSpec(dtype, n)] * 4, [], [0, 1, 2], 8420)
    h = Harness(spec)
    _check(h)
