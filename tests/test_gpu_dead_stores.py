"""Outputs of runs that are overwritten before anything reads them from memory are not stored: what is read later, in the same
segment or another one, in whatever mode that one is replayed, must be there all the same, and so must every buffer's last version."""
import dataclasses
import itertools

import pytest

import paper_2503_19779_amd as pg
from gpu_util import Harness, same_bits
from pg_workloads import ChainSpec, KernelSpec, TensorSpec, Ref, EXT, INT, WEIGHT, decode_chain

pytestmark = pytest.mark.gpu


def _check(spec):
    """Every output after every combination of modes, bit for bit what eager launches leave."""
    spec.outputs[:] = range(len(spec.ints))
    h = Harness(spec)
    for t in range(2):
        _, x = h.inputs(t)
        h.scrub()
        want = h.run("eager", x)
        for mode in ("copy", "indirect", "copy"):
            h.scrub()
            got = h.run(mode, x)
            assert all(same_bits(a, b) for a, b in zip(want, got)), (mode, t)
        has_ext = [any(r.kind == EXT for k in spec.kernels if k.segment == s for r in k.ins) for s in range(spec.n_segments)]
        if spec.n_segments > 1:
            for modes in itertools.product(*[(pg.EAGER, pg.GRAPH_COPY, pg.GRAPH_INDIRECT) if e else (pg.EAGER, pg.GRAPH_COPY) for e in has_ext]):
                h.scrub()
                got = h.run("selected", x, list(modes))
                assert all(same_bits(a, b) for a, b in zip(want, got)), (modes, t)
    h.close()


@pytest.mark.parametrize("cut", [0, 9, 17])
@pytest.mark.parametrize("reader", [None, 512, 2040, 4096])
def test_carry_runs(reader, cut):
    """Three runs over two buffers, the longest tensors first: what the shorter ones behind leave of them stays.  `reader`: between the second and
    the third run a kernel of its own reads that many elements.  `cut`: a new segment from that kernel on."""
    sizes = [512, 4096, 2048, 1024, 8192, 520, 1032, 512, 2048, 2056, 512, 512, 1024, 3000, 512, 4104, 512, 1024, 512, 2048]
    ks, ext = [], []
    for i, n in enumerate(sizes):
        op = ("add", "mul", "gelu")[i % 3]
        a = (Ref(EXT, i),)
        ks.append(KernelSpec(op, "bf16", i % 2, a if op == "gelu" else a + (Ref(INT, (i - 1) % 2) if i else Ref(WEIGHT, 0),), n, m=512 if op != "gelu" else 0))
        ext.append(TensorSpec("bf16", n))
    if reader:
        ks.insert(16, KernelSpec("gelu", "bf16", 2, (Ref(INT, 0),), reader))
    ks = [dataclasses.replace(k, segment=int(bool(cut) and i >= cut)) for i, k in enumerate(ks)]
    spec = ChainSpec(f"dead_carry_{reader}_{cut}", ks, ext, [TensorSpec("bf16", 8192)] * 3, [TensorSpec("bf16", 512)], [], 8500)
    _check(spec)


@pytest.mark.parametrize("sizes", [[4096, 2048, 1024, 512, 4104, 520], [(1 << 19) + 4096, 2048, 8192, 512, 4104, 520]])
@pytest.mark.parametrize("writer", [1, 515, 2043, 4099, 4103])
def test_carry_runs_behind_which_a_vector_is_cut(writer, sizes):
    """A kernel behind the run, on its own, overwrites a number of elements that is no whole number of vectors, of 4 or of 16 bytes: the rest of the
    vector it ends in stays what the run left there."""
    ks = [KernelSpec(("add", "mul")[i % 2], "bf16", i % 2, (Ref(EXT, i), Ref(INT, (i - 1) % 2) if i else Ref(WEIGHT, 0)), n, m=512) for i, n in enumerate(sizes)]
    ks += [KernelSpec("add", "bf16", b, (Ref(EXT, len(sizes)), Ref(WEIGHT, 0)), writer, m=512) for b in (0, 1) if b == 0 or writer <= 2048]
    spec = ChainSpec(f"dead_cut_{writer}_{max(sizes)}", ks, [TensorSpec("bf16", n) for n in sizes] + [TensorSpec("bf16", writer)], [TensorSpec("bf16", max(sizes))] * 2,
                     [TensorSpec("bf16", 512)], [], 8520)
    _check(spec)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("reader", [None, 0, 1])
def test_scale_bias_relu_segments(dtype, reader):
    """Three segments of five kernels over two buffers.  `reader`: the second segment begins with a kernel that reads buffer 0 or 1."""
    n, inner, ch = 2 * 6 * 40, 40, 6
    ks = []
    for i in range(15):
        if i == 5 and reader is not None:
            ks.append(KernelSpec("add", dtype, 2, (Ref(INT, reader), Ref(EXT, 0)), n - 8, m=n - 8, segment=1))
        ks.append(KernelSpec("scale_bias_relu", dtype, i % 2, (Ref(INT, (i - 1) % 2) if i else Ref(EXT, 0), Ref(WEIGHT, 2 * (i % 3)), Ref(WEIGHT, 2 * (i % 3) + 1)), n,
                             segment=i // 5, inner=inner, channels=ch))
    spec = ChainSpec(f"dead_sbr_{dtype}_{reader}", ks, [TensorSpec(dtype, n)], [TensorSpec(dtype, n)] * 3,
                     [TensorSpec(dtype, ch, ("normal", float(i % 2 == 0), 0.1)) for i in range(6)], [], 8510)
    _check(spec)


@pytest.mark.parametrize("batch", [1, 3, 16, 24, 40, 100])
@pytest.mark.parametrize("reader", [None, 1, 2])
@pytest.mark.parametrize("hidden", [256, 520])
def test_decoder_blocks(batch, reader, hidden):
    """Normalised rows (buffer 1) and GEMV results (buffer 2) that the next block overwrites.  `reader`: a kernel behind the second of four blocks, and
    one at the chain's end in a segment of its own, read one of them."""
    spec = decode_chain(batch=batch, layers=4, blocks_per_layer=1, hidden=hidden, n_ext=1)
    n = batch * hidden
    ks = list(spec.kernels)
    if reader is not None:
        ks.insert(8, KernelSpec("add", "bf16", 3, (Ref(INT, reader), Ref(EXT, 0)), n, m=n))
        ks.append(KernelSpec("add", "bf16", 3, (Ref(INT, 3), Ref(INT, reader)), n, m=n, segment=1))
    spec = dataclasses.replace(spec, name=f"{spec.name}_dead_{reader}", kernels=ks, ints=spec.ints + [TensorSpec("bf16", n)], outputs=[])
    if reader is None:
        spec.ints.pop()
    _check(spec)


def _check_inside(spec, inside):
    """External `e` of inside = {e: buffer} is that internal buffer.  Indirect replays and every combination of modes leave the bits of eager
    launches, with each way of moving the table; each iteration starts from the same contents."""
    spec.outputs[:] = range(len(spec.ints))
    h = Harness(spec, graphs=False)
    has_ext = [any(r.kind == EXT for k in spec.kernels if k.segment == s for r in k.ins) for s in range(spec.n_segments)]
    for t in range(2):
        _, x = h.inputs(t)
        x = [h.chain.int_buffer(inside[e]) if e in inside else a for e, a in enumerate(x)]
        h.scrub()
        want = h.run("eager", x)
        for how in (pg.TABLE_KERNARG, pg.TABLE_MEMCPY, pg.TABLE_GRAPH_MEMCPY, pg.TABLE_HOST):
            h.chain.set_table_refresh(how)
            h.scrub()
            got = h.run("indirect", x)
            assert all(same_bits(a, b) for a, b in zip(want, got)), (how, t)
        h.chain.set_table_refresh(pg.TABLE_KERNARG)
        for modes in itertools.product(*[(pg.EAGER, pg.GRAPH_COPY, pg.GRAPH_INDIRECT) if e else (pg.EAGER, pg.GRAPH_COPY) for e in has_ext]):
            h.scrub()
            got = h.run("selected", x, list(modes))
            assert all(same_bits(a, b) for a, b in zip(want, got)), (modes, t)
        # replays with other memory in between are as before
        _, y = h.inputs(t + 2)
        h.scrub()
        want = h.run("eager", y)
        for mode in ("indirect", "copy"):
            h.scrub()
            assert all(same_bits(a, b) for a, b in zip(want, h.run(mode, y))), (mode, t)
    h.close()


@pytest.mark.parametrize("buffer", [0, 1])
def test_external_in_a_buffer_of_scale_bias_relu_segments(buffer):
    """What the first segment leaves in either buffer, read at the head of the second: the last version in one, in the other one that the
    second segment overwrites and no kernel of the chain reads."""
    n, inner, ch = 2 * 6 * 40, 40, 6
    ks = []
    for i in range(15):
        if i == 5:
            ks.append(KernelSpec("add", "f32", 2, (Ref(EXT, 1), Ref(EXT, 0)), n, m=n, segment=1))
        ks.append(KernelSpec("scale_bias_relu", "f32", i % 2, (Ref(INT, (i - 1) % 2) if i else Ref(EXT, 0), Ref(WEIGHT, 0), Ref(WEIGHT, 1)), n, segment=i // 5, inner=inner, channels=ch))
    spec = ChainSpec(f"inside_sbr_{buffer}", ks, [TensorSpec("f32", n)] * 2, [TensorSpec("f32", n)] * 3,
                     [TensorSpec("f32", ch, ("normal", 1.0, 0.1)), TensorSpec("f32", ch, ("normal", 0.0, 0.1))], [], 8600)
    _check_inside(spec, {1: buffer})


@pytest.mark.parametrize("reader", [4100, 2040])
@pytest.mark.parametrize("buffer", [0, 1])
def test_external_in_a_buffer_of_carry_runs(buffer, reader):
    """A kernel between runs (4100 elements: it joins none), and one that is part of a run whose other kernels write the buffer."""
    sizes = [512, 4104, 2048, 4112, 8192, 520, 1032, 512, 2048, 2056, 512, 512, 1024, 3000, 512, 4104, 512, 1024, 512, 2048]
    ks, ext = [], []
    for i, n in enumerate(sizes):
        op = ("add", "mul", "gelu")[i % 3]
        a = (Ref(EXT, i),)
        ks.append(KernelSpec(op, "bf16", i % 2, a if op == "gelu" else a + (Ref(INT, (i - 1) % 2) if i else Ref(WEIGHT, 0),), n, m=512 if op != "gelu" else 0))
        ext.append(TensorSpec("bf16", n))
    ks.insert(14, KernelSpec("gelu", "bf16", 2, (Ref(EXT, len(sizes)),), reader))
    ks = [dataclasses.replace(k, segment=int(i >= 14)) for i, k in enumerate(ks)]
    spec = ChainSpec(f"inside_carry_{reader}", ks, ext + [TensorSpec("bf16", reader)], [TensorSpec("bf16", 8192)] * 3, [TensorSpec("bf16", 512)], [], 8610)
    _check_inside(spec, {len(sizes): buffer})


@pytest.mark.parametrize("batch", [1, 16, 40])
@pytest.mark.parametrize("buffer", [1, 2])
def test_external_in_a_buffer_of_decoder_blocks(batch, buffer):
    """Normalised rows or the GEMV's result of the third of five blocks, read at the head of the next segment."""
    spec = decode_chain(batch=batch, layers=5, blocks_per_layer=1, hidden=256, n_ext=1)
    n = batch * 256
    ks = [dataclasses.replace(k, segment=int(i >= 12)) for i, k in enumerate(spec.kernels)]
    ks.insert(12, KernelSpec("add", "bf16", 3, (Ref(EXT, 1), Ref(EXT, 0)), n, m=n, segment=1))
    spec = dataclasses.replace(spec, name=f"{spec.name}_inside_{buffer}", kernels=ks, ext=spec.ext + [TensorSpec("bf16", n)], ints=spec.ints + [TensorSpec("bf16", n)], outputs=[])
    _check_inside(spec, {1: buffer})
