"""The LDS-fed contraction kernels at the edges of their tiles: every tile shape, GEMM-shaped
and gathered operands, partial last K steps, rows and columns past the end, padding taps,
strides; alone and with the tile shapes a fused wave gives its members together."""
import pytest
import torch

from oracle import executor
from workloads import Builder
from paper_2312_10351_amd import binding as B
from paper_2312_10351_amd.runtime import Session
from util import compare_all

pytestmark = pytest.mark.gpu

# ("g", m, k, n) or ("c", cin, h, w, cout, stride); 3 x 3 convolutions with padding 1
SHAPES = [("g", 17, 520, 33), ("g", 83, 1192, 60), ("g", 300, 2056, 702), ("g", 1150, 288, 311), ("g", 256, 400, 2066),
          ("g", 1938, 360, 257), ("g", 1517, 328, 1345), ("g", 1122, 280, 1591),
          ("c", 40, 31, 23, 22, 2), ("c", 32, 23, 129, 189, 2), ("c", 32, 110, 126, 67, 2), ("c", 48, 156, 84, 42, 1),
          ("c", 32, 82, 29, 201, 1), ("c", 24, 98, 158, 151, 1), ("c", 40, 113, 66, 215, 1)]


def add(b, case, x=None):
    if case[0] == "g":
        _, m, k, n = case
        return b.gemm(b.ext((m, k)), m, k, n, extras=[b.ext((m, n))] if n % 2 else [], relu=bool(m % 2))
    _, c, h, w, cout, s = case
    return b.conv(b.ext((c, h, w)), cout, 3, stride=s, pad=1, relu=bool(h % 2))


def kernel_of(case, dtype):
    b = Builder("one", dtype)
    add(b, case)
    s = Session(b.build(1), device=None)
    try:
        return B.opara_kernel_info(B.opara_get_demands(s.dag)[0].kernel_id)[0].split("_")[-1]
    finally:
        s.close()


def test_the_shapes_reach_every_tile_shape():
    reached = {kernel_of(c, dt) for c in SHAPES for dt in ("f16", "f32")}
    assert {"quad4s", "quad4", "quad64x4", "quad64x64", "tile64x64", "t128x64", "tile128x128"} <= reached


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("case", SHAPES)
def test_alone(case, dtype):
    b = Builder("one", dtype)
    add(b, case)
    wl = b.build(31, random_bias=True, he_init=True)
    s = Session(wl)
    try:
        exe = s.capture(B.SEQUENTIAL)
        for t in s.out_dev:
            t.fill_(float("nan"))
        torch.cuda.synchronize()                         # the session replays on a stream of its own
        s.replay(exe)
        assert not compare_all(s, executor.run_dag(wl))
    finally:
        s.close()


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("cases", [SHAPES[:2] + SHAPES[8:10], SHAPES[2:8], SHAPES[10:]])
def test_together_in_one_wave(cases, dtype):
    b = Builder("wave", dtype)
    for c in cases:
        add(b, c)
    wl = b.build(32, random_bias=True, he_init=True)
    ref = executor.run_dag(wl)
    s = Session(wl)
    try:
        for exe in (s.capture(B.FUSED), s.capture_chained()):
            for t in s.out_dev:
                t.fill_(float("nan"))
            torch.cuda.synchronize()                         # the session replays on a stream of its own
            s.replay(exe)
            assert not compare_all(s, ref)
    finally:
        s.close()


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("heads,seq,d", [(3, 17, 264), (5, 70, 320), (2, 200, 520), (2, 610, 264)])
def test_batched(heads, seq, d, dtype):
    """Batched products, the operands interleaved head by head in their rows."""
    b = Builder("batched", dtype)
    q, k = b.ext((seq, heads * d)), b.ext((seq, heads * d))
    b.add("bgemm", [q, k], [(seq, heads * d)] * 2, (heads, seq, seq), dict(mode="qk", alpha=d ** -0.5, heads=heads, seq=seq, dhead=d))
    b.add("bgemm", [k, q], [(seq, heads * d)] * 2, (heads, seq, seq), dict(mode="qk", alpha=d ** -0.5, heads=heads, seq=seq, dhead=d))
    wl = b.build(33)
    ref = executor.run_dag(wl)
    s = Session(wl)
    try:
        for dem in B.opara_get_demands(s.dag):
            assert "quad" in B.opara_kernel_info(dem.kernel_id)[0] or "tile" in B.opara_kernel_info(dem.kernel_id)[0]
        for exe in (s.capture(B.SEQUENTIAL), s.capture(B.FUSED), s.capture_chained()):
            for t in s.out_dev:
                t.fill_(float("nan"))
            torch.cuda.synchronize()                         # the session replays on a stream of its own
            s.replay(exe)
            assert not compare_all(s, ref)
    finally:
        s.close()


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("hw,couts", [((9, 11), (7, 33, 22)), ((31, 23), (40, 3, 66)), ((70, 67), (101, 130, 5))])
def test_convolutions_into_slices(hw, couts, dtype):
    """Branches that write their channels into the concatenated tensor, at offsets of any parity."""
    b = Builder("slices", dtype)
    x = b.ext((72,) + hw)
    b.concat_c([b.conv(x, c, 3 if i % 2 == 0 else 1, pad=1 - i % 2) for i, c in enumerate(couts)])
    wl = b.build(34, random_bias=True, he_init=True)
    ref = executor.run_dag(wl)
    s = Session(wl, zero_copy_concat=True)
    try:
        assert s.elided
        for exe in (s.capture(B.SEQUENTIAL), s.capture(B.FUSED), s.capture_chained()):
            s.out_dev[len(couts)].fill_(float("nan"))
            torch.cuda.synchronize()
            s.replay(exe)
            assert not compare_all(s, ref)
    finally:
        s.close()
