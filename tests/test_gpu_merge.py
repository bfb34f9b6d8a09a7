"""Operators that the fused executor runs as one kernel, at the edges of what that kernel takes:
against the oracle, every operator's result, and refused where buffers overlap."""
import numpy as np
import pytest
import torch

from oracle import executor
from workloads import Builder
from paper_2312_10351_amd import binding as B
from paper_2312_10351_amd.runtime import Session
from util import compare_all, mismatch

pytestmark = pytest.mark.gpu


def run_fused(wl, launches, reps=2):
    """Replays the fused executor on clean buffers; it must launch `launches` kernels."""
    ref = executor.run_dag(wl)
    s = Session(wl)
    try:
        exe = s.capture(B.FUSED)
        assert B.opara_exec_info(exe) == (launches, launches - 1)
        node_of, n = B.opara_fused_plan(exe, len(wl.ops))
        assert n == B.opara_wave_of(s.dag)[1]
        us = B.opara_fused_time_nodes(exe, s.make_streams(1).handles[0], 2)
        assert sum(u > 0 for u in us) == launches
        for _ in range(reps):
            for t in s.out_dev:
                t.fill_(float("nan"))
            torch.cuda.synchronize()                         # the session replays on a stream of its own
            s.replay(exe)
            assert not compare_all(s, ref)
    finally:
        s.close()


def attention(heads, seq, d, dtype):
    b = Builder("attention", dtype)
    q, k, v = (b.ext((seq, heads * d)) for _ in range(3))
    att = dict(heads=heads, seq=seq, dhead=d)
    s = b.add("bgemm", [q, k], [(seq, heads * d)] * 2, (heads, seq, seq), dict(mode="qk", alpha=1.0 / d ** 0.5, **att))
    p = b.rowwise("softmax", [s], heads * seq, seq)
    b.add("bgemm", [p, v], [(heads, seq, seq), (seq, heads * d)], (seq, heads * d), dict(mode="pv", alpha=1.0, **att))
    return b.build(23)


@pytest.mark.parametrize("heads,seq,d", [(1, 1, 8), (2, 15, 64), (12, 16, 64), (3, 33, 24), (12, 128, 64), (3, 77, 64), (2, 129, 56),
                                         (5, 256, 40), (2, 300, 64), (1, 511, 8), (4, 512, 64)])
def test_attention(heads, seq, d):
    run_fused(attention(heads, seq, d, "f16"), 1)


@pytest.mark.parametrize("heads,seq,d,dtype", [(2, 520, 64, "f16"), (2, 64, 72, "f16"), (3, 48, 20, "f16"), (2, 64, 64, "f32")])
def test_attention_outside_its_range_stays_three_launches(heads, seq, d, dtype):
    run_fused(attention(heads, seq, d, dtype), 3)


def masked_attention(seq):
    """Rows 1 and 16 of the first head: keys at the ends of the kernels' lane groups have scores of
    minus infinity and key 5 the lowest finite one; the same rows of the second head: all keys do."""
    wl = attention(2, seq, 64, "f16")
    q, k = wl.ext_inputs[:2]
    q[:, [0, 64]] = 0
    q[[1, 16], 0] = q[[1, 16], 64] = 65504
    k[:, 0] = 0
    k[[i for i in (0, 15, 16, 63, 127, 128, 255, 256, seq - 1) if i < seq], 0] = -60000
    k[5, 0] = -8                                             # 65504 * -8 / sqrt(64), and a little
    k[:, 64] = -60000
    return wl


@pytest.mark.parametrize("seq", [18, 64, 129, 300, 512])
def test_attention_with_masked_scores(seq):
    """Rows that hold minus infinity and the type's lowest value beside other scores, and nothing but
    minus infinity."""
    s = Session(masked_attention(seq))
    try:
        got = []
        for mode in (B.SEQUENTIAL, B.FUSED):
            s.clear_outputs()
            s.replay(s.capture(mode))
            got.append([s.output(v).astype(np.float64) for v in range(3)])
        scores, probs = got[0][:2]
        for row in (1, 16):
            r = scores.reshape(2, seq, seq)[0, row]
            assert np.isneginf(r).sum() >= 4 and r.min(where=np.isfinite(r), initial=0) == -65504 and not (r == np.inf).any()
            assert np.isfinite(r).sum() > 8 and np.isfinite(probs.reshape(2, seq, seq)[0, row]).all()
            assert np.isneginf(scores.reshape(2, seq, seq)[1, row]).all()
        for a, b in zip(*got):
            assert (np.isnan(a) == np.isnan(b)).all() and (np.isinf(a) == np.isinf(b)).all()
            ok = np.isfinite(a)
            assert np.allclose(a[ok], b[ok], rtol=2e-3, atol=2e-3)
    finally:
        s.close()


# (m, k, n): every tile shape a contraction of its own takes, rows and columns past the tiles' end
TAIL_SHAPES = [(17, 520, 36), (83, 1192, 60), (300, 2056, 700), (1150, 288, 312), (256, 400, 2068), (1938, 360, 260), (1517, 328, 1348),
               (1122, 280, 1592)]


def tail(shape, kind, place, dtype, extras=0):
    """A product and an element-wise operator that takes its result as input number `place`."""
    m, k, n = shape
    b = Builder("tail", dtype)
    u = b.gemm(b.ext((m, k)), m, k, n, extras=[b.ext((m, n)) for _ in range(extras)], relu=extras > 0)
    ins = [b.ext((m, n)) for _ in range(3 if kind == "add3" else 2 if kind == "add" else 1)]
    ins[place] = u
    b.rowwise("add" if kind.startswith("add") else kind, ins, m, n)
    return b.build(29, random_bias=True, he_init=True)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("shape", TAIL_SHAPES)
def test_element_wise_tail(shape, dtype):
    for i, (kind, place) in enumerate((("gelu", 0), ("add", 0), ("add", 1))):
        run_fused(tail(shape, kind, place, dtype, extras=i % 2), 1, reps=1)


@pytest.mark.parametrize("kind,place", [("add3", 0), ("add3", 1), ("add3", 2), ("relu", 0)])
def test_element_wise_tail_of_several_inputs(kind, place):
    run_fused(tail((83, 520, 72), kind, place, "f16"), 1)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_element_wise_tail_of_a_convolution(dtype):
    b = Builder("tail", dtype, 2)
    x = b.ext((64, 13, 11))
    b.add_images([b.ext((36, 13, 11)), b.conv(x, 36, 3, pad=1, relu=False)])
    run_fused(b.build(31, random_bias=True, he_init=True), 1)


def test_element_wise_operators_that_stay_on_their_own():
    run_fused(tail((83, 520, 71), "gelu", 0, "f16"), 2)              # rows that are no whole vectors
    run_fused(tail((83, 72, 72), "gelu", 0, "f16"), 2)               # shallow product: fragment-loading kernel
    b = Builder("tail", "f16")                                       # a view of part of the result
    u = b.gemm(b.ext((64, 520)), 64, 520, 64)
    b.rowwise("gelu", [u], 32, 64)
    run_fused(b.build(1, he_init=True), 2)
    b = Builder("tail", "f16")                                       # the result twice
    u = b.gemm(b.ext((64, 520)), 64, 520, 64)
    b.rowwise("add", [u, u], 64, 64)
    run_fused(b.build(1, he_init=True), 2)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("rows,parts", [(1, (8,)), (7, (8, 40, 16)), (33, (72, 8, 8, 264)), (129, (16, 16))])
def test_concatenation_of_element_wise_results(rows, parts, dtype):
    b = Builder("concat", dtype)
    us = [b.rowwise(("add", "gelu", "relu")[i % 3], [b.ext((rows, c)) for _ in range(2 if i % 3 == 0 else 1)], rows, c)
          for i, c in enumerate(parts)]
    b.add("concat", us, [(rows, c) for c in parts], (rows, sum(parts)), {"axis": 1})
    run_fused(b.build(41), 1)


def test_concatenations_that_stay_on_their_own():
    for case in range(4):
        b = Builder("concat", "f16")
        n = 20 if case == 0 else 16                                  # parts that are no whole chunks
        u, v = b.rowwise("add", [b.ext((9, 16))] * 2, 9, 16), b.rowwise("relu", [b.ext((9, n))], 9, n)
        if case == 1:
            v = u                                                    # one result twice
        if case == 2:
            v = b.ext((9, n))                                        # a part nobody computes
        if case == 3:
            v = b.rowwise("softmax", [b.ext((9, n))], 9, n)
        b.add("concat", [u, v], [(9, 16), (9, n)], (9, 16 + n), {"axis": 1})
        wl = b.build(43)
        ref = executor.run_dag(wl)
        s = Session(wl)
        try:
            exe = s.capture(B.FUSED)
            assert B.opara_exec_info(exe)[0] == 2
            s.replay(exe)
            assert not compare_all(s, ref)
        finally:
            s.close()


def test_overlapping_buffers_are_not_merged():
    wl = attention(2, 64, 64, "f16")
    ref = executor.run_dag(wl)
    s = Session(wl)
    try:
        s.descs[2].out = s.ext_dev[0].data_ptr()         # the context replaces the queries
        dag = B.opara_build_dag(s.descs, [t.data_ptr() for t in s.ext_dev])
        B.opara_order_launch(dag)
        exe = B.opara_capture(dag, s.make_streams(1).handles[:1], B.FUSED)
        assert B.opara_exec_info(exe) == (3, 2)
        s.replay(exe)
        got = s.ext_dev[0].cpu().numpy().astype(np.float64)
        assert np.abs(got - ref[2].astype(np.float64)).max() < 1e-2
        B.opara_exec_destroy(exe)
        B.opara_dag_destroy(dag)
    finally:
        s.close()


def run_with(wl, rebind, launches):
    """Fused executor of `wl` with buffers that `rebind(session, descs, ext)` has changed: it must
    launch `launches` kernels.  Returns the session (its `descs` and `ext_dev` hold the results)."""
    s = Session(wl)
    ext = [t.data_ptr() for t in s.ext_dev]
    rebind(s, s.descs, ext)
    dag = B.opara_build_dag(s.descs, ext)
    B.opara_order_launch(dag)
    exe = B.opara_capture(dag, s.make_streams(1).handles[:1], B.FUSED)
    try:
        assert B.opara_exec_info(exe)[0] == launches
        torch.cuda.synchronize()
        s.replay(exe)
    finally:
        B.opara_exec_destroy(exe)
        B.opara_dag_destroy(dag)
    return s


@pytest.mark.parametrize("where", ["operand", "extra", "other input"])
def test_overlapping_buffers_are_not_merged_with_a_tail(where):
    b = Builder("tail", "f16")
    x, e, z = (b.ext((83, 520)) for _ in range(3))
    b.rowwise("add", [b.gemm(x, 83, 520, 520, extras=[e]), z], 83, 520)
    wl = b.build(37, random_bias=True, he_init=True)
    ref = executor.run_dag(wl)
    slot = {"operand": 0, "extra": 1, "other input": 2}[where]

    def rebind(s, descs, ext):
        descs[1].out = ext[slot]

    run_with(wl, lambda *a: None, 1).close()
    s = run_with(wl, rebind, 2)
    try:
        assert mismatch(s.output(0), ref[0], "f16") is None
        assert mismatch(s.ext_dev[slot].cpu().numpy().reshape(83, 520), ref[1], "f16") is None
    finally:
        s.close()


@pytest.mark.parametrize("kind", ["conv", "conv 1x1", "gemm", "bgemm", "pool", "gavgpool", "softmax", "add", "concat"])
def test_a_concatenation_over_what_an_earlier_operator_reads_is_not_written_in_place(kind):
    b = Builder("concat", "f16")
    image = (16, 9, 9)
    if kind in ("conv", "conv 1x1"):
        x = b.ext(image)
        o = b.conv(x, 16, 3 if kind == "conv" else 1, pad=1 if kind == "conv" else 0)
    elif kind == "pool":
        o = b.pool("maxpool", b.ext(image), 3, 1, 1)
    elif kind == "gavgpool":
        o = b.gavgpool(b.ext(image))
    elif kind == "gemm":
        o = b.gemm(b.ext((9, 520)), 9, 520, 16)
    elif kind == "bgemm":
        o = b.add("bgemm", [b.ext((16, 64)), b.ext((16, 64))], [(16, 64)] * 2, (2, 16, 16), dict(mode="qk", alpha=0.125, heads=2, seq=16, dhead=32))
    elif kind == "concat":
        o = b.add("concat", [b.ext((9, 16)), b.ext((9, 8))], [(9, 16), (9, 8)], (9, 24), {"axis": 1})
    else:
        o = b.rowwise(kind, [b.ext((9, 16))] * (2 if kind == "add" else 1), 9, 16)
    shape = b.shape(o)
    if len(shape) == 3 and kind != "bgemm":
        part, whole, axis = shape, (2 * shape[0],) + tuple(shape[1:]), 0
    else:
        part, whole, axis = (int(np.prod(shape)) // 8, 8), (int(np.prod(shape)) // 8, 16), 1
    n = int(np.prod(part))
    u = b.add("relu", [b.ext(part)], [part], part)
    v = b.add("gelu", [o], [part], part)
    c = b.add("concat", [u, v], [part] * 2, whole, {"axis": axis})
    wl = b.build(47, random_bias=True, he_init=True)
    ref = executor.run_dag(wl)
    keep = []

    def rebind(s, descs, ext):                               # the concatenation's buffer begins with what `o` reads
        keep.append(torch.zeros(max(2 * n, s.ext_dev[0].numel()), dtype=torch.float16, device=s.device))
        keep[0][:s.ext_dev[0].numel()] = s.ext_dev[0].reshape(-1)
        ext[0] = descs[c].out = keep[0].data_ptr()

    run_with(wl, lambda *a: None, 2).close()
    s = run_with(wl, rebind, 3)
    try:
        s.out_dev[c] = keep[0][:2 * n]
        assert not compare_all(s, ref)
    finally:
        s.close()
