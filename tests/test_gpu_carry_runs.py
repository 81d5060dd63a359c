"""Runs of bf16 kernels that take the head of the previous kernel's output as a short-period operand: one dispatch, the same
bits as kernel by kernel in both buffers, everywhere (what a later kernel of a run overwrites only in part keeps its
rest), with tensors shorter and longer than each other, than a unit and than four units per workgroup, with every
period, and where a run has to end: a tensor shorter than the period, a first operand that the run writes, another
period."""
import random

import pytest

from gpu_util import Harness, same_bits, stepwise_check
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT, INT, WEIGHT, refresh_stress_chain

pytestmark = pytest.mark.gpu


def _check(h, step=True):
    for t in range(3):
        x_np, x_dev = h.inputs(t)
        h.scrub()
        want = h.run("eager", x_dev)
        for mode in ("copy", "indirect", "indirect"):
            h.scrub()
            got = h.run(mode, x_dev)
            for o in range(len(want)):
                assert same_bits(want[o], got[o]), (t, mode, o)
    if step:
        h.scrub()
        stepwise_check(h, x_np, x_dev)
    h.close()


@pytest.mark.parametrize("tensors,log2_max,seed", [(1, 12.0, 3), (2, 12.0, 1), (9, 11.0, 2), (24, 16.0, 3), (40, 14.0, 4), (33, 23.5, 5)])
def test_refresh_chains(tensors, log2_max, seed):
    spec = refresh_stress_chain(n_tensors=tensors, log2_max=log2_max, seed=seed)
    spec.outputs[:] = [0, 1]
    h = Harness(spec)
    assert h.chain.graph_dispatches()[0] == (tensors + 7) // 8
    _check(h, step=log2_max < 20)


@pytest.mark.parametrize("n,kernels", [(8, 3), (256, 4), (512, 6), (512, 13)])
def test_carries_that_are_whole_tensors(n, kernels):
    """Every kernel takes what the one before wrote, whole, as its second operand -- and every fourth as its first."""
    ks = [KernelSpec("gelu", "bf16", 0, (Ref(EXT, 0),), n)]
    for i in range(1, kernels):
        prev, own = Ref(INT, ks[-1].out), Ref(EXT, i % 3)
        ks.append(KernelSpec("add" if i % 2 else "mul", "bf16", i % 2, (prev, own) if i % 4 == 2 else (own, prev), n, m=n))
    spec = ChainSpec(f"whole_{n}_{kernels}", ks, [TensorSpec("bf16", n)] * 3, [TensorSpec("bf16", n)] * 2, [], [0, 1], 8200 + kernels)
    h = Harness(spec)
    assert h.chain.graph_dispatches()[0] <= -(-kernels // 4)
    _check(h)


@pytest.mark.parametrize("period", [8, 64, 256, 512])
@pytest.mark.parametrize("seed", [1, 2, 3, 4])
def test_random_runs(period, seed):
    rng = random.Random(1000 * period + seed)
    sizes = [8 * rng.choice([rng.randint(1, 40), rng.randint(period // 8, 600), rng.randint(1, 3000)]) for _ in range(26)]
    big = max(sizes + [512])
    ks, ext = [], []
    for k, n in enumerate(sizes):
        out = rng.choice([0, 1, 2])
        if k and out == ks[-1].out:
            out = (out + 1) % 3
        prev = Ref(INT, ks[-1].out) if k and ks[-1].n >= period else Ref(WEIGHT, 0)
        if rng.random() < 0.1:
            prev = Ref(WEIGHT, 0)                         # no carry: a run ends here
        a = Ref(EXT, len(ext))
        ext.append(TensorSpec("bf16", n))
        op = rng.choice(["add", "mul", "gelu", "add"])
        if k > 3 and rng.random() < 0.15 and ks[-1].n >= n and ks[-1].out != out:
            a = Ref(INT, ks[-1].out)                      # the whole of the previous output: not in one run with it
        if op == "gelu":
            ks.append(KernelSpec("gelu", "bf16", out, (a,), n))
        else:
            m = period if rng.random() < 0.9 else 8
            ks.append(KernelSpec(op, "bf16", out, (a, prev), n, m=m))
    spec = ChainSpec(f"carry_{period}_{seed}", ks, ext, [TensorSpec("bf16", big) for _ in range(3)], [TensorSpec("bf16", 512)], [], 8000 + seed)
    spec.outputs[:] = sorted({k.out for k in ks})
    h = Harness(spec)
    merged, unmerged = h.chain.graph_dispatches()
    assert merged < unmerged
    _check(h)


@pytest.mark.parametrize("period", [8, 512])
@pytest.mark.parametrize("sizes", [[512, 520, 1024, 512, 2056, 512, 1528, 512, 1032], [(1 << 19) + 8, 2048, 1 << 19, 2056, 4104, (1 << 19) + 2056, 512, 4096, 2040]])
def test_no_gelu_cuts_the_carry(period, sizes):
    """Adds and muls alone: the last kernel of a run depends on the head of every one before it; tensors that end within a
    workgroup's unit, at its edge and behind it, on 4 and on 16 bytes a lane."""
    ks = [KernelSpec("mul" if i % 3 == 1 else "add", "bf16", i % 2, (Ref(EXT, i), Ref(INT, (i - 1) % 2) if i else Ref(WEIGHT, 0)), n, m=period) for i, n in enumerate(sizes)]
    spec = ChainSpec(f"no_gelu_{period}_{max(sizes)}", ks, [TensorSpec("bf16", n) for n in sizes], [TensorSpec("bf16", max(sizes))] * 2, [TensorSpec("bf16", 512)], [0, 1], 8300)
    h = Harness(spec)
    assert h.chain.graph_dispatches()[0] == 2
    _check(h)
