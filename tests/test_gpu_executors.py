"""Executors that live side by side: of different workloads, element types and needs of workgroup
memory, replayed in turn, with executors destroyed and made in between, each pass on clean buffers
and every operator against the oracle."""
import pytest
import torch

from oracle import executor
from workloads import Builder, googlenet_like, inception_block, random_small_dag
from paper_2312_10351_amd import binding as B
from paper_2312_10351_amd.runtime import Session
from util import compare_all

pytestmark = pytest.mark.gpu


def contractions(dtype):
    """A wave of products that take the largest tiles, then one of small ones."""
    b = Builder("contractions", dtype)
    for m, k, n in ((300, 2056, 700), (1517, 328, 1345), (1150, 288, 311), (256, 400, 2066)):
        u = b.gemm(b.ext((m, k)), m, k, n)
        b.rowwise("relu", [u], m, n)
        b.gemm(u, 16, 64, 24)
    return b.build(51, random_bias=True, he_init=True)


class Alive:
    def __init__(self, wl, mode):
        self.ref = executor.run_dag(wl)
        self.s = Session(wl, zero_copy_concat=True)
        self.exe = self.s.capture(mode)
        self.mode = mode

    def check(self):
        for t in self.s.out_dev:
            t.fill_(float("nan"))
        torch.cuda.synchronize()                             # the session replays on a stream of its own
        self.s.replay(self.exe)
        assert not compare_all(self.s, self.ref)

    def close(self):
        self.s.close()


def test_executors_replayed_in_turn():
    make = [lambda: Alive(contractions("f32"), B.FUSED), lambda: Alive(inception_block(dtype="f32"), B.FUSED),
            lambda: Alive(contractions("f16"), B.FUSED), lambda: Alive(random_small_dag(7), B.FUSED),
            lambda: Alive(googlenet_like(he_init=True), B.PARALLEL), lambda: Alive(inception_block(dtype="f16", batch=3), B.FUSED),
            lambda: Alive(random_small_dag(11, dtype="f32"), B.SEQUENTIAL)]
    alive = [m() for m in make]
    try:
        for turn in range(3):
            for a in alive:
                a.check()
            # nodes by themselves, after executors that need less workgroup memory were captured
            for a in alive:
                if a.mode == B.FUSED:
                    B.opara_fused_time_nodes(a.exe, a.s.make_streams(1).handles[0], 1)
            for i in (turn, turn + 3):                       # gone, and another in its place
                alive[i].close()
                torch.cuda.empty_cache()
                alive[i] = make[i]()
                alive[i].check()
    finally:
        for a in alive:
            a.close()
