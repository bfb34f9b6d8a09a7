"""Operands around the reach of 32-bit offsets: which kernel takes a contraction on either side of
each limit (planned on made-up addresses), and on the GPU the results past it."""
import pytest
import torch

from paper_2312_10351_amd import binding as B


def desc(kind, dtype=B.F16, **params):
    d = B.OpDesc()
    d.op_type, d.op_class, d.dtype = kind, B.CLASS_DEFAULT, dtype
    d.n_inputs = 2 if kind == B.BGEMM else 1
    d.inputs[0], d.inputs[1] = -1, -2
    for k, v in params.items():
        setattr(d.params, k, v)
    d.weight, d.out = 0x100000, 0x200000
    return d


def planned(d):
    dag = B.opara_build_dag([d], [0x300000, 0x400000])
    try:
        return B.opara_kernel_info(B.opara_get_demands(dag)[0].kernel_id)[0]
    finally:
        B.opara_dag_destroy(dag)


def conv(h, w, c, batch, stride):
    return desc(B.CONV2D, h_in=h, w_in=w, c_in=c, c_out=64, kh=3, kw=3, sh=stride, sw=stride, ph=1, pw=1,
                h_out=(h - 1) // stride + 1, w_out=(w - 1) // stride + 1, batch=batch)


LIMIT = 0xc0000000
ROWS = 128                                                   # of the largest tile


def largest_row(es):
    """Elements, in whole vectors, of the longest row of which a tile's worth is within reach."""
    ve = 16 // es
    return ((LIMIT - 1) // es // (ROWS + 1)) // ve * ve


@pytest.mark.parametrize("case,fed", [
    (desc(B.GEMM, m=LIMIT // 8192 - 1, n=64, k=4096), True), (desc(B.GEMM, m=LIMIT // 8192, n=64, k=4096), True),
    (desc(B.GEMM, m=64, n=LIMIT // 8192, k=4096), True), (desc(B.GEMM, B.F32, m=LIMIT // 4096, n=1000, k=1024), True),
    (desc(B.GEMM, m=1000, n=64, k=largest_row(2)), True), (desc(B.GEMM, m=1000, n=64, k=largest_row(2) + 8), False),
    (desc(B.GEMM, B.F32, m=1000, n=64, k=largest_row(4)), True), (desc(B.GEMM, B.F32, m=1000, n=64, k=largest_row(4) + 4), False),
    (desc(B.GEMM, m=5, n=5, k=(1 << 28) - 8), True), (desc(B.GEMM, m=5, n=5, k=1 << 28), False),     # a row's own limit
    (conv(2048, 2048, 192, 1, 4), True), (conv(2048, 2048, 184, 3, 4), True), (conv(2048, 2048, 192, 3, 4), False),   # images a tile touches
    (conv(40, 40, 848, 1200, 1), True), (conv(8, 8, 4096, 4096, 1), True),
    (conv(3, 5592400, 8, 1, 1), True), (conv(3, 5592408, 8, 1, 1), False),                           # a window's positions
    (desc(B.BGEMM, m=2000, n=2000, k=512, batch=2, a_row_stride=1000000, b_row_stride=512, c_row_stride=2000, a_batch_stride=8,
          b_batch_stride=8, c_batch_stride=4000000, alpha=1.0), True),
])
def test_which_kernel_takes_them(case, fed):
    name = planned(case)
    assert ("t64x64" not in name) == fed, name


def launch(d, ext):
    dag = B.opara_build_dag([d], [t.data_ptr() for t in ext])
    try:
        torch.cuda.synchronize()
        stream = torch.cuda.Stream()
        B.opara_launch_op(dag, 0, stream.cuda_stream)
        torch.cuda.synchronize()
    finally:
        B.opara_dag_destroy(dag)
        torch.cuda.empty_cache()


def close(got, want):
    """fp16 results of sums of about unit size: the tolerance of the operator tests."""
    return bool(((got.float() - want).abs() <= 2e-2 * want.abs() + 1e-2 * want.square().mean().sqrt()).all())


def half(*shape, std=1.0):
    return torch.empty(shape, dtype=torch.float16, device="cuda").normal_(0, std)


@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n", [(394000, 4096, 40), (72, 4096, 394000)])
def test_gemm_past_the_reach(m, k, n):
    x, w, y = half(m, k), half(n, k, std=k ** -0.5), torch.full((m, n), float("nan"), dtype=torch.float16, device="cuda")
    d = desc(B.GEMM, m=m, n=n, k=k)
    d.weight, d.out = w.data_ptr(), y.data_ptr()
    launch(d, [x])
    for rows, cols in ((slice(0, 700), slice(0, 700)), (slice(m // 2, m // 2 + 700), slice(n // 2, n // 2 + 700)), (slice(-700, None), slice(-700, None))):
        assert close(y[rows, cols], x[rows].float() @ w[cols].float().t())
    assert not torch.isnan(y).any()


@pytest.mark.gpu
def test_executors_past_the_reach():
    """A product past the reach beside a small one: as members of a group, and in the executors whose
    kernel does not hold the body that counts from its tile."""
    m, k, n = 394000, 4096, 40
    x, w = half(m, k), half(n, k, std=k ** -0.5)
    ys = [torch.empty(rows, n, dtype=torch.float16, device="cuda") for rows in (m, 64)]
    descs = []
    for rows, y in zip((m, 64), ys):
        d = desc(B.GEMM, m=rows, n=n, k=k)
        d.weight, d.out = w.data_ptr(), y.data_ptr()
        descs.append(d)
    dag = B.opara_build_dag(descs, [x.data_ptr()])
    B.opara_order_launch(dag)
    stream = torch.cuda.Stream()
    spaces = [torch.zeros(f(dag) + 256, dtype=torch.uint8, device="cuda") for f in (B.opara_chained_workspace_bytes, B.opara_persistent_workspace_bytes)]
    at = [(s.data_ptr() + 255) // 256 * 256 for s in spaces]
    torch.cuda.synchronize()
    execs = [B.opara_capture(dag, [stream.cuda_stream], B.FUSED), B.opara_capture_chained(dag, at[0], B.opara_chained_workspace_bytes(dag)),
             B.opara_capture_persistent(dag, at[1], B.opara_persistent_workspace_bytes(dag), 0)]
    try:
        for exe in execs:
            for y in ys:
                y.fill_(float("nan"))
            torch.cuda.synchronize()
            B.opara_replay(exe, stream.cuda_stream)
            torch.cuda.synchronize()
            assert close(ys[1], x[:64].float() @ w.float().t()) and close(ys[0][-700:], x[-700:].float() @ w.float().t())
            assert not torch.isnan(ys[0]).any()
    finally:
        for exe in execs:
            B.opara_exec_destroy(exe)
        B.opara_dag_destroy(dag)
        torch.cuda.empty_cache()


@pytest.mark.gpu
def test_convolution_past_the_reach():
    b, h, w, c, n = 1200, 40, 40, 848, 24
    x, wt, y = half(b, h, w, c), half(n, 3, 3, c, std=(9 * c) ** -0.5), torch.full((b, h, w, n), float("nan"), dtype=torch.float16, device="cuda")
    d = conv(h, w, c, b, 1)
    d.params.c_out = n
    d.weight, d.out = wt.data_ptr(), y.data_ptr()
    launch(d, [x])
    assert not torch.isnan(y).any()
    for img in (0, b // 2, b - 2, b - 1):
        want = torch.zeros(h, w, n, device="cuda")
        pad = torch.nn.functional.pad(x[img].float(), (0, 0, 1, 1, 1, 1))
        for i in range(3):
            for j in range(3):
                want += (pad[i:i + h, j:j + w].reshape(-1, c) @ wt[:, i, j].float().t()).reshape(h, w, n)
        assert close(y[img], want)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", [B.MAXPOOL, B.AVGPOOL])
def test_pooling_past_the_reach(kind):
    b, h, w, c = 3, 2100, 2100, 88                           # 2.3 GB: offsets of more than 31 bits
    x, y = half(b, h, w, c), torch.full((b, 1050, 1050, c), float("nan"), dtype=torch.float16, device="cuda")
    d = desc(kind, h_in=h, w_in=w, c_in=c, c_out=c, kh=3, kw=3, sh=2, sw=2, ph=1, pw=1, h_out=1050, w_out=1050, batch=b)
    d.out = y.data_ptr()
    launch(d, [x])
    pool = torch.nn.functional.max_pool2d if kind == B.MAXPOOL else torch.nn.functional.avg_pool2d
    for img in (0, b - 1):
        want = pool(x[img, :, :, :8].float().permute(2, 0, 1)[None], 3, 2, 1)[0].permute(1, 2, 0)
        assert close(y[img, :, :, :8], want)
    assert not torch.isnan(y).any()
