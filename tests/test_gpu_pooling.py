"""Pooling windows and global averages where their index arithmetic can go wrong: windows that
hang over every edge, strides and windows of other sizes than 3 x 3, channel counts with and
without 16-byte chunks, several images, pixel counts around the rounds of the global average."""
import numpy as np
import pytest
import torch

from oracle import executor
from workloads import Builder
from paper_2312_10351_amd import binding as B
from paper_2312_10351_amd.runtime import Session
from util import compare_all

pytestmark = pytest.mark.gpu


def check(wl):
    ref = executor.run_dag(wl)
    s = Session(wl)
    try:
        for exe in (s.capture(B.SEQUENTIAL), s.capture(B.FUSED)):
            for t in s.out_dev:
                t.fill_(float("nan"))
            torch.cuda.synchronize()                         # the session replays on a stream of its own
            s.replay(exe)
            assert not compare_all(s, ref)
    finally:
        s.close()


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("c,h,w,batch", [(8, 1, 1, 1), (8, 2, 5, 3), (24, 7, 6, 2), (5, 9, 4, 1), (160, 17, 35, 2), (264, 3, 70, 1)])
def test_windows(c, h, w, batch, dtype):
    b = Builder("pool", dtype, batch)
    x = b.ext((c, h, w))
    for kind in ("maxpool", "avgpool"):
        for k, s, p in ((3, 1, 1), (3, 2, 1), (3, 2, 2), (2, 2, 1), (5, 3, 2), (1, 2, 0)):
            b.pool(kind, x, k, s, p)
    check(b.build(17))


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("c,hw", [(8, (1, 1)), (40, (3, 3)), (72, (11, 12)), (160, (28, 28)), (7, (13, 5)), (1032, (8, 16)), (20, (43, 3))])
def test_global_average(c, hw, dtype):
    for batch in (1, 3):
        b = Builder("gap", dtype, batch)
        x = b.ext((c,) + hw)
        b.gavgpool(x)
        b.gavgpool(b.pool("maxpool", x, 3, 1, 1))
        check(b.build(19))


def test_maximum_of_infinities_and_not_a_numbers():
    """A maximum skips values that are not numbers; padding never wins over minus infinity."""
    b = Builder("pool", "f16")
    x = b.ext((16, 6, 6))
    b.pool("maxpool", x, 3, 1, 1)
    wl = b.build(3)
    a = wl.ext_inputs[0]
    a[0] = -np.inf
    a[1, ::2] = np.nan
    a[2, 1::3] = np.inf
    s = Session(wl)
    try:
        s.replay(s.capture(B.SEQUENTIAL))
        got = s.output(0).astype(np.float64)
    finally:
        s.close()
    pad = np.pad(np.where(np.isnan(a), -np.inf, a.astype(np.float64)), ((0, 0), (1, 1), (1, 1)), constant_values=-np.inf)
    want = np.max([pad[:, i:i + 6, j:j + 6] for i in range(3) for j in range(3)], axis=0)
    assert (got == want).all()
