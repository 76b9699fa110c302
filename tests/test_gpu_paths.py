"""The sizes at which a kernel with a narrow domain can go wrong: edges of its tiles, remainders, the ends of its range."""
import ctypes as ct

import numpy as np
import pytest
import torch

from gpu_harness import GpuStage, compare_minibatch, gpu_minibatch, stage_io, to_dev
from oracle.stage import OracleStage, one_f_one_b_order
from paper_2012_12544_amd import binding as B
from stage_inputs import configs as C
from stage_inputs import gen
from test_gpu_stage import single

pytestmark = pytest.mark.gpu


# ------------------------------------------------------------------------------ LSTM recurrence in one launch
@pytest.mark.parametrize("cin,hidden,T,mb", [
    (16, 128, 1, 1),         # no recurrent product, one block column of the smallest matrix
    (24, 128, 2, 17),        # a second group of sequences with one member
    (128, 384, 5, 16),       # four pieces of K for each half of the rows, not eight for all
    (64, 640, 3, 3),
    (128, 1024, 4, 33),      # the widest matrix, a ragged third group
])
@pytest.mark.parametrize("need_dx", [1, 0])
def test_lstm_sequence_kernels(cin, hidden, T, mb, need_dx):
    st = single(lambda b: b.lstm(cin, hidden, src=-1), cin, (T, 1), C.BF16, micro_batch=mb, need_input_grad=need_dx)
    compare_minibatch(st, verbose="lstm %d->%d T=%d N=%d" % (cin, hidden, T, mb))


def test_lstm_sequence_kernels_twice_are_bit_identical():
    """Blocks hand their slices to each other inside the launch: a missing wait would show as a difference."""
    st = C.gnmt_lstm_stage(hidden=256, seq=30, n_layers=2, micro_batch=40, n_micro=3)
    a, b = gpu_minibatch(st), gpu_minibatch(st)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


def _lstm_seq(direction, signature):
    f = getattr(B.load(), "_ZN6bapipe12lstm_seq_%sE%s" % (direction, signature))
    f.restype = ct.c_int
    return f


def _lstm_layer(n, t, h, polls, spoil=None, given_up=None):
    """Both directions of one layer's recurrence on seeded operands: every tensor they write, as integers.  `given_up` receives, for
    each direction, whether a block of a group of 16 sequences gave up: the first word of the groups' lines of 64."""
    g = torch.Generator("cuda")
    g.manual_seed(n + t + h)
    bf16 = dict(device="cuda", dtype=torch.bfloat16)
    rand = lambda *shape: (torch.rand(shape, device="cuda", generator=g) * 2 - 1).bfloat16()
    p, dy, w = rand(n, t, 4 * h), rand(n, t, h), rand(4 * h, h) / h ** 0.5
    wt = w.t().contiguous()
    if spoil:
        spoil(p, dy)
    gates, cells = torch.empty(n, t, 4 * h, device="cuda"), torch.empty(n, t, h, device="cuda")
    y, ys, d = torch.empty(n, t, h, **bf16), torch.empty(n, t, h, **bf16), torch.empty(n, t, 4 * h, **bf16)
    carry = torch.empty(n, h, device="cuda")
    size = getattr(B.load(), "_ZN6bapipe18lstm_seq_workspaceEii")
    size.restype, size.argtypes = ct.c_size_t, [ct.c_int] * 2
    work = torch.empty(size(n, h), device="cuda", dtype=torch.uint8)
    ptr = lambda x: ct.c_void_p(x.data_ptr())
    stream = ct.c_void_p(torch.cuda.current_stream().cuda_stream)
    dims = (ct.c_int(n), ct.c_int(t), ct.c_int(h), ptr(work), stream, ct.c_uint(polls))
    lines = lambda: work.view(torch.int32)[64:64 * (1 + (n + 15) // 16):64].tolist()
    assert _lstm_seq("fwd", "PKvS1_PfS2_PvS3_iiiS3_P12ihipStream_tj")(ptr(p), ptr(w), ptr(gates), ptr(cells), ptr(y), ptr(ys), *dims) == 0
    if given_up is not None:
        given_up.append(lines())
    assert _lstm_seq("bwd", "PKvS1_PKfS3_PfPviiiS5_P12ihipStream_tj")(ptr(dy), ptr(wt), ptr(gates), ptr(cells), ptr(carry), ptr(d), *dims) == 0
    if given_up is not None:
        given_up.append(lines())
    torch.cuda.synchronize()
    return [x.view(torch.int16 if x.dtype == torch.bfloat16 else torch.int32).clone() for x in (gates, cells, y, ys, d)]


@pytest.mark.parametrize("h,t,n", [(128, 2, 3), (256, 7, 33), (640, 3, 16), (1024, 5, 40)])
def test_lstm_sequence_kernels_finish_without_their_neighbours(h, t, n):
    """A block that does not wait, or hardly, leaves its group of sequences to one block that computes it alone: the
    same bits, whichever step the group was left at."""
    want = _lstm_layer(n, t, h, 1 << 16)
    for polls in (0, 1, 8, 64):
        for a, b in zip(_lstm_layer(n, t, h, polls), want):
            assert torch.equal(a, b), polls


def test_lstm_sequence_kernels_pass_nan_on():
    """Values that are not numbers travel between blocks too, whatever their bits: the sequence they are in has them from
    its first on, in forward to the end, in backward to the start; the others do not, and nobody gives up."""
    n, t, h = 20, 6, 256
    want = _lstm_layer(n, t, h, 1 << 14)
    spoil = lambda p, dy: (p[3, 2].view(torch.int16).fill_(-1), dy[17, 4].view(torch.int16).fill_(-1))
    waited, left = [], []
    got, alone = _lstm_layer(n, t, h, 1 << 14, spoil, waited), _lstm_layer(n, t, h, 0, spoil, left)
    assert waited == [[0, 0]] * 2 and left == [[1, 1]] * 2
    for bits in (got[2][3, 2:], got[4][17, :5]):               # pairs of values that would read as a slice not yet sent
        assert (bits.reshape(-1, 2) == -1).all(dim=1).any()
    as_float = lambda x: x.view(torch.bfloat16 if x.dtype == torch.int16 else torch.float32).float()
    y, d = as_float(got[2]), as_float(got[4])
    assert torch.isnan(y[3, 2:]).all() and not torch.isnan(y[3, :2]).any()
    assert torch.isnan(d[17, :5]).all() and not torch.isnan(d[17, 5]).any()
    for a, b, c in zip(got, want, alone):
        rest = [i for i in range(n) if i not in (3, 17)]
        assert torch.equal(a[rest], b[rest])
        assert torch.equal(torch.isnan(as_float(a)), torch.isnan(as_float(c)))


class _ConvShape(ct.Structure):
    _fields_ = [(f, ct.c_int) for f in "N H W C P Q K R S stride pad".split()]


class _WgradJob(ct.Structure):
    _fields_ = [("x", ct.c_void_p), ("dy", ct.c_void_p), ("dw", ct.c_void_p), ("db", ct.c_void_p), ("c", _ConvShape), ("x2", ct.c_void_p), ("dw2", ct.c_void_p)]


def _wgrad_workspace(shape):
    f = getattr(B.load(), "_ZN6bapipe25conv_wgrad_mfma_workspaceERKNS_9ConvShapeE")
    f.restype = ct.c_size_t
    return f(ct.byref(shape))


def _wgrad_jobs(jobs, work, room):
    f = getattr(B.load(), "_ZN6bapipe20conv_wgrad_mfma_jobsEPKNS_8WgradJobEiPvmP12ihipStream_tb")
    f.restype = ct.c_int
    assert f((_WgradJob * len(jobs))(*jobs), ct.c_int(len(jobs)), ct.c_void_p(work.data_ptr()), ct.c_size_t(room),
             ct.c_void_p(torch.cuda.current_stream().cuda_stream), ct.c_bool(False)) == 0


@pytest.mark.parametrize("products", [1, 2])     # whose partial sums the workspace holds
@pytest.mark.parametrize("c,k,rows,bias", [
    (1024, 4096, 1043, True),     # 256 x 128, 33 tiles of rows, the last of 19: four parts and a short one
    (896, 3584, 1024, False),     # ... 14 x 7 of them, twice
    (512, 2048, 700, True),       # no pair: 128 x 64, two groups of waves
    (128, 512, 333, True),        # 64 x 64
    (1024, 4096, 40, False),      # a step of rows and a short one
    (72, 40, 9, True),
    (128, 512, 3200, True),       # partial sums
    (64, 256, 2560, True),
    (256, 1024, 6400, False),
])
def test_weight_gradients_of_a_pair(c, k, rows, bias, products):
    """dw += dy^T x and dw2 += dy^T x2: against float64, a rounding of 2^-24 for each term of the sum and each of the additions."""
    g = torch.Generator("cuda")
    g.manual_seed(c + rows)
    rand = lambda *shape: torch.randn(shape, device="cuda", generator=g)
    x, x2, dy = rand(rows, c).bfloat16(), rand(rows, c).bfloat16(), rand(rows, k).bfloat16()
    dw, dw2, db = rand(k, c), rand(k, c), rand(k)
    want = [dw.double() + dy.double().t() @ x.double(), dw2.double() + dy.double().t() @ x2.double(), db.double() + dy.double().sum(0)]
    terms = [dw.abs() + dy.float().abs().t() @ x.float().abs(), dw2.abs() + dy.float().abs().t() @ x2.float().abs(), db.abs() + dy.float().abs().sum(0)]
    shape = _ConvShape(rows, 1, 1, c, 1, 1, k, 1, 1, 1, 0)
    room = products * (_wgrad_workspace(shape) + 255) // 256 * 256
    work = torch.full((room + (1 << 20),), 0xA5, device="cuda", dtype=torch.uint8)         # behind it nothing may be written
    _wgrad_jobs([_WgradJob(x.data_ptr(), dy.data_ptr(), dw.data_ptr(), db.data_ptr() if bias else None, shape, x2.data_ptr(), dw2.data_ptr())], work, room)
    torch.cuda.synchronize()
    assert (work[room:] == 0xA5).all()
    for got, ref, t in list(zip((dw, dw2, db), want, terms))[:3 if bias else 2]:
        assert ((got.double() - ref).abs() <= (rows + 8) * 2.0 ** -24 * t).all()


@pytest.mark.parametrize("c,rows", [(128, 1024), (128, 1600), (256, 3200), (512, 12800), (1024, 3200), (1024, 12800)])
def test_weight_gradients_of_a_pair_are_as_exact_as_one_by_one(c, rows):
    """Operands of one sign.  P parts of n sums of 16 products, each rounded by 2.4e-8 of the sum so far on average, added up in double (splits of a
    few parts, or the parts of a tile) and rounded twice more at most: sqrt(n / (3 P) + 2) times that, with n = 16 and P = 4 at the least 4.4e-8.  Parts
    added up in float, as many as there are without splits, are 4.5e-8 to 6.2e-8 off here."""
    g = torch.Generator("cuda")
    g.manual_seed(c + rows)
    rand = lambda *shape: torch.rand(shape, device="cuda", generator=g).bfloat16()
    x, x2, dy = rand(rows, c), rand(rows, c), rand(rows, 4 * c)
    dw, dw2, db = torch.zeros(4 * c, c, device="cuda"), torch.zeros(4 * c, c, device="cuda"), torch.zeros(4 * c, device="cuda")
    shape = _ConvShape(rows, 1, 1, c, 1, 1, 4 * c, 1, 1, 1, 0)
    room = 2 * (_wgrad_workspace(shape) + 256)
    _wgrad_jobs([_WgradJob(x.data_ptr(), dy.data_ptr(), dw.data_ptr(), db.data_ptr(), shape, x2.data_ptr(), dw2.data_ptr())],
                torch.empty(room, device="cuda", dtype=torch.uint8), room)
    torch.cuda.synchronize()
    dyt = dy.double().t().contiguous()
    off = lambda got, exact: float((got.double() - exact).norm() / exact.norm())
    e = off(dw, dyt @ x.double()), off(dw2, dyt @ x2.double()), off(db, dy.double().sum(0))
    assert max(e) < 4.4e-8, e


@pytest.mark.parametrize("room", [1 << 30, 0])      # of the workspace: for all partial sums, or for those of one product at a time
def test_weight_gradients_that_share_launches(room):
    """The same bits as one by one: products of both tile shapes, more than a launch takes, some with partial sums, one that
    fills the chip by itself, one on patches."""
    shapes = [(2, 9, 9, 64, 64, 3), (1, 20, 20, 128, 128, 3), (3, 14, 14, 256, 64, 1), (2, 14, 14, 128, 256, 3), (5, 7, 7, 512, 512, 1),
              (4, 64, 64, 128, 128, 3), (1, 4, 4, 2048, 4096, 1), (2, 30, 30, 72, 40, 3), (4, 28, 28, 256, 256, 3), (1, 5, 5, 8, 64, 3), (2, 11, 13, 64, 192, 3)]
    g = torch.Generator("cuda")
    g.manual_seed(5)
    rand = lambda *shape: torch.randn(shape, device="cuda", generator=g)
    keep, jobs, most = [], [], 0
    for n, h, w, c, k, r in shapes:
        t = [rand(n, h, w, c).bfloat16(), rand(n, h, w, k).bfloat16(), rand(k, r, r, c), rand(k)]
        keep.append(t)
        shape = _ConvShape(n, h, w, c, h, w, k, r, r, 1, r // 2)
        most = max(most, _wgrad_workspace(shape))
        jobs.append(_WgradJob(t[0].data_ptr(), t[1].data_ptr(), t[2].data_ptr(), t[3].data_ptr(), shape, None, None))
    start = [[a.clone() for a in t[2:]] for t in keep]
    room = max(room, most) if room == 0 else 4 * most
    work = torch.empty(room + 4096, device="cuda", dtype=torch.uint8)

    def run(batches):
        for t, s0 in zip(keep, start):
            for a, b in zip(t[2:], s0):
                a.copy_(b)
        for b in batches:
            _wgrad_jobs(b, work, room)
        torch.cuda.synchronize()
        return [a.clone() for t in keep for a in t[2:]]
    for a, b in zip(run([jobs]), run([[j] for j in jobs])):
        assert torch.equal(a, b)


@pytest.mark.parametrize("hidden,reads", [(128, 1), (64, 5)])       # the recurrent matrix: kept for the launch, read each step
def test_lstm_traffic_is_what_the_layer_moves(hidden, reads):
    cin, t, n, g = 24, 6, 5, 4 * hidden
    st = single(lambda b: b.lstm(cin, hidden, src=-1), cin, (t, 1), C.BF16, micro_batch=n, n_micro=1)
    gpu = GpuStage(st, gen.all_params(st))
    xs, gs = stage_io(st)
    B.bapipe_stage_kernel_timing(gpu.h, 0)
    gpu.forward(0, xs[0])
    fwd = B.bapipe_stage_kernel_timing_read(gpu.h)
    gpu.backward(0, gs[0])
    bwd = B.bapipe_stage_kernel_timing_read(gpu.h)
    gpu.close()
    floats = 4 * n * t * (g + hidden)                             # gates and cells
    assert fwd["bytes"] == 2 * (n * t * (cin + 2 * g + 2 * hidden) + g * cin + reads * g * hidden) + floats
    assert bwd["bytes"] == 2 * (n * t * (hidden + 2 * g + cin) + g * cin + reads * g * hidden) + floats


@pytest.mark.parametrize("streams", [1, 3])
def test_tap_counts_every_weight_gradient(streams):
    """... also of those that share a launch."""
    def build(b):
        b.conv(64, 64, 3, relu=1, src=-1)
        b.conv(64, 128, 1, pad=0, relu=1)
        b.conv(128, 64, 3)
    st = single(build, 64, (14, 14), C.BF16, micro_batch=4, n_micro=2)
    gpu = GpuStage(st, gen.all_params(st), backward_stream=streams == 3)
    xs, gs = stage_io(st)
    B.bapipe_stage_kernel_timing(gpu.h, B.KC_CONV_WGRAD_MFMA)
    for m in range(2):
        gpu.forward(m, xs[m])
        gpu.backward(m, gs[m])
    tap = B.bapipe_stage_kernel_timing_read(gpu.h)
    gpu.close()
    assert tap["launches"] == 6 and tap["flop"] == 2 * 2.0 * 4 * 196 * (9 * 64 * 64 + 64 * 128 + 9 * 128 * 64)


# ------------------------------------------------------------------------------ direct weight gradients that share launches
def test_direct_weight_gradients_that_share_launches():
    """More float layers of a pass than a launch takes, of different shapes, in one order of streams and in another."""
    def build(b):
        b.conv(5, 8, 3, relu=1, src=-1)
        for k in (1, 3, 5, 3, 1, 3, 3, 1, 3):
            b.conv(8, 8, k, relu=1)
        b.conv(8, 3, 3, stride=2)
    st = single(build, 5, (9, 11), C.FP32, micro_batch=3, n_micro=3)
    compare_minibatch(st, verbose="shared direct weight gradients")
    a, b = gpu_minibatch(st), gpu_minibatch(st, backward_stream=True, wgrad_stream=True)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


# ------------------------------------------------------------------------------ input gradient of a strided convolution
@pytest.mark.parametrize("k,stride,pad,cin,cout,hw,mb", [
    (3, 2, 1, 64, 32, (21, 19), 3),      # classes of unequal size, one K-tile a tap
    (3, 2, 1, 72, 64, (8, 7), 2),        # a ragged channel tile
    (3, 2, 1, 136, 96, (2, 3), 1),       # smaller than a tile in every class
    (3, 2, 0, 256, 32, (17, 16), 5),     # no padding: class 0 sits on the even pixels
    (5, 3, 2, 64, 32, (16, 14), 2),      # nine classes of 1, 2 and 4 taps
    (2, 3, 0, 64, 64, (13, 14), 2),      # stride beyond the filter: classes without taps
    (3, 2, 1, 128, 128, (56, 56), 3),    # many tiles
    (1, 2, 0, 72, 64, (15, 15), 2),      # 1x1: one class with a tap, three with their epilogue only
    (1, 3, 0, 136, 32, (7, 8), 2),
    (1, 2, 0, 64, 40, (15, 14), 3),      # 1x1 with a ragged K-tile of channels: 32 + 8
    (1, 2, 0, 136, 8, (9, 9), 2),        # ... of 8 alone
    (1, 3, 0, 256, 520, (20, 22), 5),    # ... 16 whole ones and 8, many tiles
    (2, 5, 1, 64, 32, (3, 4), 2),        # stride beyond the image: fewer classes than stride^2
    (3, 300, 1, 16, 32, (7, 9), 2),
    (1, 300, 0, 8, 32, (301, 301), 1),   # more classes than a grid axis holds
    (1, 40, 0, 16, 32, (41, 83), 2),     # 1600 classes of 12 pixels: taken together
    (3, 40, 1, 16, 32, (41, 83), 3),     # ... of 18: apart
])
def test_strided_conv_gradient(k, stride, pad, cin, cout, hw, mb):
    st = single(lambda b: b.conv(cin, cout, k, stride=stride, pad=pad, relu=1, src=-1), cin, hw, C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="strided conv k%d s%d p%d %d->%d %s" % (k, stride, pad, cin, cout, hw))


@pytest.mark.parametrize("k,stride,cin,mid,cout,hw,mb", [
    (1, 2, 72, 72, 64, (15, 13), 3),     # ragged tiles in every class, three of them with gate and sum only
    (3, 2, 64, 136, 96, (9, 10), 2),
    (1, 3, 64, 64, 32, (7, 8), 2),
    (1, 2, 64, 72, 40, (15, 13), 3),     # a ragged K-tile of channels
])
def test_strided_conv_gradient_behind_a_gate_and_a_sum(k, stride, cin, mid, cout, hw, mb):
    """The strided layer's input is a ReLU output that a second layer reads too: its gradient is added to and gated, also
    at the pixels that no tap reaches."""
    def build(b):
        t = b.conv(cin, mid, 3, relu=1, src=-1)
        s = b.conv(mid, cout, k, stride=stride, pad=k // 2, src=t)
        u = b.conv(mid, cout, 3, stride=stride, pad=1, src=t)
        b.addl(s, u, relu=0)
    st = single(build, cin, hw, C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="strided conv k%d s%d %d->%d %s, gate and sum" % (k, stride, mid, cout, hw))


def test_strided_conv_gradient_takes_a_residual_share():
    """A tensor read by a strided 1x1 layer and by an ADD: the ADD's share comes in with the strided gradient."""
    def build(b):
        t = b.conv(64, 72, 3, relu=1, src=-1)
        s = b.conv(72, 64, 1, stride=2, pad=0, src=t)
        u = b.conv(64, 72, 3, src=-1)
        a = b.addl(t, u, relu=1)
        v = b.conv(72, 64, 3, stride=2, pad=1, src=a)
        b.addl(s, v, relu=0)
    compare_minibatch(single(build, 64, (11, 14), C.BF16), verbose="strided 1x1 and residual share")


@pytest.mark.parametrize("k,cin,c,cout,hw,mb,relu", [
    (1, 64, 72, 64, (25, 23), 4, 1),     # sums of dy and dy*xhat per class tile, ragged channel tile
    (1, 64, 128, 32, (48, 45), 2, 1),
    (3, 64, 64, 64, (29, 27), 3, 1),
    (1, 64, 72, 24, (25, 23), 4, 1),
])
def test_strided_conv_gradient_with_batch_norm_sums(k, cin, c, cout, hw, mb, relu):
    def build(b):
        b.conv(cin, c, 1, pad=0, bias=0, src=-1)
        b.bn(c, relu=relu)
        b.conv(c, cout, k, stride=2, pad=k // 2)
    st = single(build, cin, hw, C.BF16, micro_batch=mb)
    assert mb * hw[0] * hw[1] > 2048             # below that the batch-norm reads its input itself
    compare_minibatch(st, verbose="batch-norm and strided conv k%d %d->%d %s" % (k, c, cout, hw))


@pytest.mark.parametrize("dtype,cin,cout", [(C.FP32, 8, 12), (C.BF16, 9, 7), (C.BF16, 16, 32)])
@pytest.mark.parametrize("k,stride,pad", [(3, 2 ** 31 - 1, 1), (3, 2 ** 31 - 3, 2), (1, 2 ** 31 - 1, 0), (3, 70000, 0)])
def test_strides_of_one_output(dtype, cin, cout, k, stride, pad):
    st = single(lambda b: b.conv(cin, cout, k, stride=stride, pad=pad, relu=1, src=-1), cin, (5, 6), dtype)
    compare_minibatch(st, verbose="conv k%d s%d p%d" % (k, stride, pad))


# ------------------------------------------------------------------------------ 64-channel K-tiles of the 64-pixel gather tile
@pytest.mark.parametrize("k,cin,cout,hw,mb", [
    (1, 64, 136, (9, 11), 2),        # one K-tile (an odd count: the second half of the trip is skipped), ragged tiles
    (3, 192, 64, (7, 7), 3),         # 27 K-tiles; the gradient has 9 of them
    (1, 2048, 128, (5, 5), 2),       # few tiles: K split over blocks, every split ending inside the tensor
    (3, 128, 256, (14, 14), 5),      # 36 or 18 K-tiles, whole channel tiles
])
def test_conv_wide_k_tiles(k, cin, cout, hw, mb):
    st = single(lambda b: b.conv(cin, cout, k, relu=1, src=-1), cin, hw, C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="wide K tiles k%d %d->%d %s" % (k, cin, cout, hw))


# ------------------------------------------------------------------------------ gather tiles whose K is split over wave groups
@pytest.mark.parametrize("k,cin,cout,hw,mb", [
    (1, 512, 40, (5, 5), 2),         # 32 x 32: two K-tiles a group, ragged both ways
    (3, 64, 72, (9, 8), 1),          # 18 K-tiles: two groups have one more than the rest
    (1, 520, 64, (6, 5), 3),         # a ragged K-tile, flattened order of K
    (3, 72, 24, (7, 7), 2),          # K-tiles that straddle taps
    (1, 512, 520, (10, 10), 5),      # 32 x 64, ragged channel tile
    (3, 96, 320, (20, 13), 6),
    (1, 256, 1024, (14, 14), 4),     # 64 x 64, two groups
    (1, 264, 1000, (14, 13), 4),     # ... of 32-channel K-tiles
    (3, 128, 64, (45, 45), 3),
])
def test_conv_groups_of_waves(k, cin, cout, hw, mb):
    st = single(lambda b: b.conv(cin, cout, k, relu=1, src=-1), cin, hw, C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="gather groups k%d %d->%d %s x %d" % (k, cin, cout, hw, mb))


@pytest.mark.parametrize("cin,cout,mb", [
    (4992, 4104, 40),      # a large matrix, one row of tiles: groups and splits
    (4992, 4104, 32),      # ... few rows: groups alone
    (4992, 4104, 65),      # ... more rows: splits alone
    (1024, 1000, 1),
])
def test_linear_groups_of_waves(cin, cout, mb):
    st = single(lambda b: b.linear(cin, cout, relu=1, src=-1), cin, (1, 1), C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="linear groups %d->%d x %d" % (cin, cout, mb))


@pytest.mark.parametrize("cin,cout,mb", [
    (32, 32, 1),           # one panel either way
    (96, 160, 70),         # panels and a half of 64 columns, ragged tiles of rows
    (64, 40, 3),           # panels forward, rows backward
    (1088, 4128, 64),      # deep ring of the gradient: K-tiles of 64, channels that end inside a tile
    (1056, 4128, 64),      # K-tiles of 32
    (4096, 4096, 61),      # K split over four blocks a tile, the last of which adds, in both directions
    (64, 128, 4200),       # 256 x 128
    (1024, 512, 19000),    # 256 x 256
])
def test_linear_filters_in_panels(cin, cout, mb):
    """Matrices whose copies are kept in panels of 32 columns, before and after an update.  (No ReLU: of the gates of 10^7 outputs a
    few would differ, and a row of dx with each.)"""
    b = C._Builder()
    b.linear(cin, cout, src=-1)
    st = C._stage("panels", b.layers, C.BF16, (cin, 1, 1), mb, 2, 1, 2, 1, C.BASE_SEED + 79, "kaiming")
    compare_minibatch(st, verbose="linear %d->%d x %d" % (cin, cout, mb))
    _copies_after_an_update_are_those_of_its_weights(st)


def _copies_after_an_update_are_those_of_its_weights(st):
    xs, gs = stage_io(st)
    one = GpuStage(st, gen.all_params(st, perturb=True))
    _mini_batch(one, st, xs, gs)
    B.bapipe_stage_step(one.h, 0.05)
    other = GpuStage(st, [one.get_params(i) for i in range(len(st["layers"]))])
    for u, v in zip(_mini_batch(one, st, xs, gs), _mini_batch(other, st, xs, gs)):
        assert np.array_equal(u, v)
    one.close()
    other.close()


@pytest.mark.parametrize("layer", ["lstm", "conv", "norm"])
def test_filters_in_panels_that_are_streamed(layer):
    """The input block of an LSTM, beside a recurrent block in rows; a 1x1 convolution of a map; two around a batch-norm, whose sums they leave."""
    b = C._Builder()
    if layer == "lstm":
        b.lstm(8224, 512, src=-1)
        st = C._stage("streamed", b.layers, C.BF16, (8224, 7, 1), 5, 2, 1, 2, 1, C.BASE_SEED + 81, "kaiming")
    else:
        b.conv(1024, 16416, 1, bias=layer == "conv", src=-1)
        if layer == "norm":
            b.bn(16416, relu=1)
            b.conv(16416, 1024, 1)
        st = C._stage("streamed", b.layers, C.BF16, (1024, 7, 7), 1, 2, 1, 2, 1, C.BASE_SEED + 82, "kaiming")
    compare_minibatch(st, verbose="streamed %s" % layer)
    _copies_after_an_update_are_those_of_its_weights(st)


def test_strided_convolutions_to_single_pixels_add_their_gradients():
    """Two 1x1 / 2 convolutions read one 2x2 map: the second gradient, of four pixel classes, is added to the first."""
    st = single(lambda b: (b.conv(4096, 4096, 1, stride=2, src=-1), b.conv(4096, 4096, 1, stride=2, src=-1), b.addl(0, 1, relu=0)), 4096, (2, 2), C.BF16,
                micro_batch=10)
    compare_minibatch(st, verbose="two 1x1 / 2 of one 2x2 map")


@pytest.mark.parametrize("layer,cout,mb", [
    ("linear", 4096, 40),        # four blocks share a tile's K
    ("linear", 4608, 64),        # three
    ("conv", 4096, 33),          # and add what the sum's gradient left, from where it lies
    ("linear", 8192, 48),        # two
])
def test_last_block_of_a_tile_runs_every_epilogue(layer, cout, mb):
    """Bias and ReLU forward; behind a ReLU and beside a residual sum, a gate and the gradient that is already there."""
    make = (lambda b, *c, **kw: b.conv(*c, 1, **kw)) if layer == "conv" else (lambda b, *c, **kw: b.linear(*c, **kw))
    cin = 4096 if cout < 8192 else 2048
    st = single(lambda b: (make(b, 64, cin, relu=1, src=-1), make(b, cin, cout, relu=1), make(b, cout, cin), b.addl(0, 2, relu=0)), 64, (1, 1), C.BF16,
                micro_batch=mb)
    compare_minibatch(st, verbose="%s %d->%d->%d x %d, added" % (layer, cin, cout, cin, mb))


def test_blocks_of_a_tile_count_themselves_on_every_stream():
    """Passes that overlap, the static workspace, one stream: the same bits."""
    b = C._Builder()
    b.linear(4096, 4096, src=-1)
    b.linear(4096, 4608)
    b.linear(4608, 4096)
    st = C._stage("shared K", b.layers, C.BF16, (4096, 1, 1), 48, 3, 1, 2, 1, C.BASE_SEED + 80, "kaiming")
    ref = gpu_minibatch(st)
    for kw in (dict(backward_stream=True, eager_sync=False), dict(backward_stream="no wgrad stream", eager_sync=False), dict(static=True),
               dict(static=True, backward_stream=True, eager_sync=False)):
        got = gpu_minibatch(st, **kw)
        for k in ref:
            assert np.array_equal(got[k], ref[k]), (kw, k)


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("cin,cout,mb", [(96, 64, 5), (4096, 4096, 40)])
def test_conv_of_single_pixels(cin, cout, mb, stride):
    """A 1x1 convolution of 1x1 maps is a linear layer."""
    st = single(lambda b: b.conv(cin, cout, 1, stride=stride, src=-1), cin, (1, 1), C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="1x1 / %d of 1x1 maps %d->%d x %d" % (stride, cin, cout, mb))


@pytest.mark.parametrize("cin,mid,hw,mb", [(512, 64, (7, 7), 3), (512, 72, (10, 9), 2)])
def test_groups_of_waves_in_a_bottleneck(cin, mid, hw, mb):
    """Every epilogue on tiles of wave groups: statistics, sums of dy and dy*xhat behind a gate, a residual share.  Small
    enough that no gate flips: of 1024/264 channels, 14x14, 8 samples, tiles without groups were off by up to 7.5e-2 of the
    largest element and these by 7.7e-2, both beyond what an element-wise 2e-2 can tell from a mistake."""
    def build(b):
        t = b.conv(cin, cin, 1, pad=0, relu=1, src=-1)
        b.conv(cin, mid, 1, pad=0, bias=0)
        b.bn(mid, relu=1)
        b.conv(mid, mid, 3, bias=0)
        b.bn(mid, relu=1)
        b.conv(mid, cin, 1, pad=0, bias=0)
        u = b.bn(cin)
        b.addl(u, t, relu=1)
    st = single(build, cin, hw, C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="bottleneck %d/%d %s x %d" % (cin, mid, hw, mb))


@pytest.mark.parametrize("k,cin,cout,hw,mb", [
    (3, 512, 512, 7, 32),       # 64 x 64, two groups: 36 K-tiles of 64 each
    (1, 4096, 1000, 1, 64),     # 32 x 32, eight
    (7, 1024, 32, 15, 4),       # 49 taps, flattened order of K
    (3, 256, 64, 28, 32),       # 128 x 64, no groups
    (3, 1024, 32, 47, 13),
    (3, 64, 64, 90, 5),         # patches of ragged images: 18 steps of 32
    (3, 128, 64, 45, 40),       # ... 36
    (3, 192, 64, 40, 45),       # ... 54, the last part half as long
    (3, 256, 64, 28, 110),      # ... 72
])
def test_conv_sums_are_short(k, cin, cout, hw, mb):
    """Terms of one sign on an image that is the same everywhere, and a bias that takes the exact sum away: what is left away from
    the border is the error of the sum.  Each of the 24 sums of a part of 384 terms is rounded by at most 2^-24/sqrt(3) of itself
    on average, the k-th of 24 being k/24 of the part: 1e-7 for a part, less for several; adding up to 24 parts the same."""
    st = single(lambda b: b.conv(cin, cout, k, src=-1), cin, (hw, hw), C.BF16, micro_batch=mb, n_micro=1)
    rng = np.random.default_rng(k + cin)
    bf16 = lambda a: torch.from_numpy(a.astype(np.float32)).bfloat16().float().numpy()
    w, x = bf16(np.abs(rng.standard_normal((cout, cin, k, k))) / (cin * k * k) ** 0.5), bf16(rng.random(cin))
    exact = np.einsum("ocrs,c->o", w.astype(np.float64), x.astype(np.float64))
    bias = -exact.astype(np.float32)
    g = GpuStage(st, [(w, bias)])
    y = g.forward(0, np.broadcast_to(x[None, :, None, None], (mb, cin, hw, hw)))
    g.close()
    p = k // 2
    left = y[:, :, p:hw - p, p:hw - p] - (exact + bias)[None, :, None, None]
    rms = float(np.sqrt(np.mean(left ** 2) / np.mean(exact ** 2)))
    assert rms < 1e-7


# ------------------------------------------------------------------------------ batch-norm passes that add the partial sums
@pytest.mark.parametrize("dtype", [C.FP32, C.BF16])
@pytest.mark.parametrize("c,hw,mb", [
    (64, (29, 25), 3),       # one slice of 64 channels, a last row block of a few rows
    (72, (29, 25), 3),       # a second slice of 8
    (8, (33, 32), 2),        # less than a slice
    (136, (50, 49), 5),      # several rows a thread
    (12, (29, 25), 3),       # bf16: channels that no 16-byte access holds, two launches
])
def test_batch_norm_adds_partial_sums(dtype, c, hw, mb):
    """More than 2048 rows and up to 64 chunks of partial sums, from passes of their own."""
    def build(b):
        u = b.bn(c, relu=1, src=-1)
        v = b.bn(c)
        b.addl(v, u, relu=1)
    st = single(build, c, hw, dtype, micro_batch=mb)
    compare_minibatch(st, verbose="batch-norm sums c%d %s x %d" % (c, hw, mb))


@pytest.mark.parametrize("c,hw,mb", [(1024, 14, 4), (512, 7, 32), (256, 14, 10)])
def test_batch_norm_sums_of_a_neighbouring_conv_are_exact(c, hw, mb):
    """Between two convolutions that pass everything on, up to 2048 rows: the second one's gradient leaves the sums of dy and
    dy*xhat.  Random terms: each carries three roundings (difference, product, product), is added up in eights (three levels),
    the eights' total is rounded once per tile and the total once: a relative error of sqrt(8) 2^-24/sqrt(3) = 1e-7 if every
    rounding were of the worst mantissa, 8e-8 on average; one after the other in float it is 1.2e-7."""
    def build(b):
        b.conv(c, c, 1, bias=0, src=-1)
        b.bn(c, relu=1)
        b.conv(c, c, 1, bias=0)
    st = single(build, c, (hw, hw), C.BF16, micro_batch=mb, n_micro=1)
    eye = np.eye(c, dtype=np.float32).reshape(c, c, 1, 1)
    g = GpuStage(st, [(eye, None), (np.ones(c, np.float32), np.zeros(c, np.float32)), (eye, None)])
    xs, gs = stage_io(st)
    y = g.forward(0, xs[0])
    g.backward(0, gs[0])
    dgamma, dbeta = g.grads(1)
    g.close()
    x, dy = (torch.from_numpy(a[0]).bfloat16().double().numpy() for a in (xs, gs))
    mean, var = (f(x, axis=(0, 2, 3), keepdims=True) for f in (np.mean, np.var))
    dy = dy * (y > 0)
    off = lambda got, exact: float(np.linalg.norm(got - exact) / np.linalg.norm(exact))
    eps = float(np.float32(st["layers"][1]["eps"]))
    e = (off(dgamma, (dy * (x - mean) / np.sqrt(var + eps)).sum(axis=(0, 2, 3))), off(dbeta, dy.sum(axis=(0, 2, 3))))
    assert max(e) < 1e-7


# ------------------------------------------------------------------------------ a stage's output, stored by its last pass or copied
@pytest.mark.parametrize("dtype", [C.FP32, C.BF16])
@pytest.mark.parametrize("kind,c,hw", [("bn", 64, (9, 7)), ("bn", 128, (32, 33)), ("bn", 20, (48, 50)), ("sum", 64, (9, 7)),
                                       ("sum", 128, (64, 33)), ("loss", 1000, (1, 1)), ("loss", 1500, (1, 1))])
def test_output_wherever_it_lies(dtype, kind, c, hw):
    """An address that no 16-byte access takes gets a copy; both are the stashed tensor bit for bit."""
    b = C._Builder()
    if kind == "loss":
        b.linear(64, c, src=-1)
        b.xent()
    else:
        u = b.bn(c, relu=kind == "bn", src=-1)
        if kind == "sum":
            b.addl(b.bn(c), u, relu=1)
    cin = 64 if kind == "loss" else c
    st = C._stage("out", b.layers, dtype, (cin,) + hw, 2, 1, 1, 1, 1, C.BASE_SEED + 79, "kaiming")
    x = to_dev(st, stage_io(st)[0][0], B.NHWC)
    t = torch.float32 if kind == "loss" or dtype == C.FP32 else torch.bfloat16
    n = 2 * c * (1 if kind == "loss" else hw[0] * hw[1])
    out = []
    for at in (0, 8 // t.itemsize):
        g = GpuStage(st, gen.all_params(st, perturb=True))
        y = torch.full((n + 16,), float("nan"), device="cuda", dtype=t)
        torch.cuda.synchronize()
        B.bapipe_stage_forward(g.h, 0, x.data_ptr(), y[at:].data_ptr())
        torch.cuda.synchronize()
        assert torch.isnan(y[at + n:]).all() and torch.isnan(y[:at]).all()
        out.append(y[at:at + n].clone())
        g.close()
    assert torch.equal(out[0], out[1]) and not torch.isnan(out[0]).any()


@pytest.mark.parametrize("dtype", [C.FP32, C.BF16])
@pytest.mark.parametrize("kind,shift", [("loss", 0), ("loss", 3), ("sum", 0), ("sum", 1)])
def test_output_that_overlaps_the_input(dtype, kind, shift):
    """Layers may read the caller's x in place until the last of them has run; only then is y stored over it."""
    c, hw, mb = (1500, (1, 1), 300) if kind == "loss" else (64, (40, 40), 4)
    b = C._Builder()
    if kind == "loss":
        b.xent(src=-1)
    else:
        b.relu(src=-1)
        b.addl(b.bn(c), -1, relu=0)
    st = C._stage("over", b.layers, dtype, (c,) + hw, mb, 1, 1, 1, 1, C.BASE_SEED + 80, "kaiming")
    x = to_dev(st, stage_io(st)[0][0], B.NHWC).reshape(-1)
    row = shift * c * x.element_size()                       # bytes from x to y
    n = x.numel() * (4 if kind == "loss" else x.element_size())
    out = []
    for apart in (True, False):
        g = GpuStage(st, gen.all_params(st, perturb=True))
        buf = torch.zeros(n + row + 256, device="cuda", dtype=torch.uint8)
        buf[:x.numel() * x.element_size()] = x.view(torch.uint8)
        y = torch.zeros_like(buf) if apart else buf
        torch.cuda.synchronize()
        B.bapipe_stage_forward(g.h, 0, buf.data_ptr(), y.data_ptr() + row)
        torch.cuda.synchronize()
        out.append(y[row:row + n].clone())
        g.close()
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("kind,streams", [("plain", 1), ("sum", 1), ("linear", 1), ("plain", 3)])
@pytest.mark.parametrize("shift", [0, 2])
def test_gradient_that_overlaps_the_upstream_gradient(kind, streams, shift, static):
    """dx may be stored over dy: whatever still reads dy has run by then."""
    c, hw, mb = (512, (1, 1), 300) if kind == "linear" else (64, (14, 14), 4)
    b = C._Builder()
    if kind == "linear":
        b.linear(c, c, relu=1, src=-1)
        b.linear(c, c)
    else:
        u = b.conv(c, c, 3, relu=1, src=-1)
        v = b.conv(c, c, 3)
        if kind == "sum":
            b.addl(v, u)
    st = C._stage("over", b.layers, C.BF16, (c,) + hw, mb, 1, 1, 1, 1, C.BASE_SEED + 81, "kaiming")
    xs, gs = stage_io(st)
    dy = to_dev(st, gs[0], B.NHWC).reshape(-1)
    n, at = dy.numel(), shift * c
    entry = B.bapipe_stage_backward_static if static else B.bapipe_stage_backward
    out = []
    for apart in (True, False):
        g = GpuStage(st, gen.all_params(st, perturb=True), backward_stream=streams == 3)
        g.forward(0, xs[0])
        buf = torch.zeros(n + at, device="cuda", dtype=dy.dtype)
        buf[:n] = dy
        dx = torch.zeros_like(buf) if apart else buf
        torch.cuda.synchronize()
        entry(g.h, 0, buf.data_ptr(), dx[at:].data_ptr())
        torch.cuda.synchronize()
        out.append([dx[at:at + n].float().cpu().numpy()] + [a for i, (w, _) in enumerate(g.params) if w is not None for a in g.grads(i)])
        g.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b) and np.any(a)


# ------------------------------------------------------------------------------ direct convolution (fp32 stages)
@pytest.mark.parametrize("k,stride,pad,cin,cout,hw,mb", [
    (3, 1, 1, 16, 64, (9, 33), 2),       # four outputs a tile and channel, the last tile one column
    (3, 1, 1, 64, 12, (6, 50), 1),       # 21 columns a tile, which their input does not allow
    (3, 1, 1, 3, 12, (5, 8), 1),         # one channel at a time; fewer columns than a tile
    (5, 2, 2, 8, 20, (11, 13), 2),       # every other column, taps outside on all sides
    (1, 1, 0, 60, 60, (5, 7), 1),
    (7, 1, 3, 4, 4, (6, 5), 1),          # a filter larger than the image
    (3, 1, 0, 12, 8, (40, 64), 60),      # more tiles than blocks, several image rows a chunk
    (3, 1, 1, 32, 32, (4, 80), 2),
    (3, 1, 1, 20, 64, (8, 9), 2),        # a filter that LDS does not take
])
def test_direct_conv_tiles(k, stride, pad, cin, cout, hw, mb):
    st = single(lambda b: b.conv(cin, cout, k, stride=stride, pad=pad, relu=1, src=-1), cin, hw, C.FP32, micro_batch=mb)
    compare_minibatch(st, verbose="direct conv tiles k%d s%d p%d %d->%d %s" % (k, stride, pad, cin, cout, hw))


@pytest.mark.parametrize("k,stride,pad,cin,cout,hw,mb", [
    (3, 1, 1, 3, 64, (9, 33), 6),        # one channel at a time; two blocks for the weights of a row
    (3, 1, 1, 16, 64, (9, 33), 5),
    (5, 2, 2, 8, 20, (11, 61), 30),      # every other column
    (1, 1, 0, 60, 60, (5, 70), 18),
    (3, 1, 1, 32, 32, (4, 80), 11),      # three times the threads of a block for the weights of a row
    (7, 1, 3, 4, 4, (6, 45), 80),        # rows outside the image on both sides at once
])
def test_direct_weight_gradient_tiles(k, stride, pad, cin, cout, hw, mb):
    st = single(lambda b: b.conv(cin, cout, k, stride=stride, pad=pad, src=-1), cin, hw, C.FP32, micro_batch=mb)
    compare_minibatch(st, verbose="direct weight gradient tiles k%d s%d p%d %d->%d %s" % (k, stride, pad, cin, cout, hw))


@pytest.mark.parametrize("k,stride,pad,cin,cout,hw,mb", [
    (3, 1, 1, 20, 12, (9, 11), 3),       # a last trip of one vector of channels
    (3, 2, 2, 4, 8, (8, 7), 2),          # fewer channels than a trip, two columns of padding
    (1, 3, 0, 36, 5, (10, 10), 2),       # gradient operand with an odd channel count: one channel at a time
    (5, 3, 1, 16, 16, (7, 19), 1),       # columns at the right edge that no output reads
    (3, 2, 1, 7, 6, (9, 8), 2),          # three and two channels left of a group, two classes of taps a side
    (5, 3, 2, 9, 13, (16, 14), 2),       # one channel left
    (2, 5, 1, 20, 28, (13, 12), 2),      # stride beyond the filter: pixels that no tap reaches
    (4, 2, 3, 24, 8, (7, 6), 3),         # padding: taps before the first row
])
def test_direct_conv(k, stride, pad, cin, cout, hw, mb):
    st = single(lambda b: b.conv(cin, cout, k, stride=stride, pad=pad, relu=1, src=-1), cin, hw, C.FP32, micro_batch=mb)
    compare_minibatch(st, verbose="direct conv k%d s%d p%d %d->%d %s" % (k, stride, pad, cin, cout, hw))


@pytest.mark.parametrize("k,stride,pad,cin,cout,hw,mb", [
    (3, 2, 1, 9, 22, (9, 8), 2),
    (5, 3, 2, 30, 13, (16, 14), 2),
])
def test_direct_conv_bf16(k, stride, pad, cin, cout, hw, mb):
    st = single(lambda b: b.conv(cin, cout, k, stride=stride, pad=pad, relu=1, src=-1), cin, hw, C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="direct conv bf16 k%d s%d p%d %d->%d %s" % (k, stride, pad, cin, cout, hw))


@pytest.mark.parametrize("cin,cout,mb", [
    (16384, 16384, 1),      # 2^28 weights: more threads than a grid holds if several share one of them
    (1, 1 << 24, 2),        # 2^24 bias gradients: the same for the column sums
])
def test_gradients_of_the_largest_linear_layers(cin, cout, mb):
    """One or two samples: the sums are single products, and sums of two floats, which have one rounding."""
    st = single(lambda b: b.linear(cin, cout, src=-1), cin, (1, 1), C.FP32, micro_batch=mb, n_micro=1, need_input_grad=0)
    g = GpuStage(st, [(None, None)])
    rng = np.random.default_rng(cin)
    x = rng.standard_normal((mb, cin, 1, 1), dtype=np.float32)
    dy = rng.standard_normal((mb, cout, 1, 1), dtype=np.float32)
    g.forward(0, x)
    g.backward(0, dy)
    dw, db = B.bapipe_stage_get_grads(g.h, 0, (cout, cin), (cout,))
    g.close()
    dy = dy.reshape(mb, cout)
    assert np.array_equal(db, dy.sum(axis=0, dtype=np.float64).astype(np.float32))
    for k in range(0, cout, 997):              # terms below 16: two roundings of 2^-21 at most
        assert np.allclose(dw[k], dy[:, k].astype(np.float64) @ x.reshape(mb, cin), rtol=0, atol=2.0 ** -20)


@pytest.mark.parametrize("dtype,k,cin,cout,hw,mb", [
    (C.FP32, 3, 512, 512, 28, 8),      # seven chunks of 896 pixels
    (C.FP32, 3, 12, 20, 224, 2),       # one image row a chunk
    (C.FP32, 1, 8, 2048, 31, 30),      # 930 image rows: the bias gradient would cost the filter chunks, column sums
    (C.FP32, 1, 2048, 4096, 8, 1),     # two chunks; the same
    (C.BF16, 3, 252, 252, 28, 2),      # channels that the matrix kernels do not take
])
def test_direct_bias_gradient_of_wide_layers(dtype, k, cin, cout, hw, mb):
    """Gradients of one sign, so a rounding is at most 2^-24 of the result.  Riding along: three levels of an eight, the chunk's sum,
    the total.  Column sums of these shapes: a run of up to 57 floats (the k-th of its sums is k/57 of it: 29 in all), the total."""
    st = single(lambda b: b.conv(cin, cout, k, src=-1), cin, (hw, hw), dtype, micro_batch=mb, n_micro=1, need_input_grad=0)
    g = GpuStage(st, [(None, None)])
    rng = np.random.default_rng(cout)
    dy = rng.random((mb, cout, hw, hw), dtype=np.float32)
    if dtype == C.BF16:
        dy = torch.from_numpy(dy).bfloat16().float().numpy()
    g.forward(0, np.ones((mb, cin, hw, hw), np.float32))
    g.backward(0, dy)
    dw, db = B.bapipe_stage_get_grads(g.h, 0, (cout, cin, k, k), (cout,))
    g.close()
    exact = dy.sum(axis=(0, 2, 3), dtype=np.float64)
    roundings = 30 if k == 1 else 5
    worst = float(np.max(np.abs(db - exact) / exact))
    assert worst <= roundings * 2.0 ** -24


# ------------------------------------------------------------------------------ 2x2 pools that store and read NCHW
@pytest.mark.parametrize("dtype", [C.FP32, C.BF16])
@pytest.mark.parametrize("relu", [0, 1])
@pytest.mark.parametrize("c,hw,mb", [
    (64, (16, 16), 3),       # whole tiles of 64 channels and of positions
    (72, (15, 9), 2),        # a second tile of 8 channels, the last row and column in no window
    (8, (2, 3), 1), (136, (33, 2), 2), (16, (32, 32), 4),
    (12, (7, 10), 3),        # bf16: channels that no 16-byte access holds, launches of their own
    (8, (130, 129), 9),      # more positions than few channels share a launch for
])
def test_pool_at_the_end_of_a_stage_in_either_layout(dtype, relu, c, hw, mb):
    """The pooled tensor leaves, and its gradient comes, in the layout of the boundary."""
    st = single(lambda b: (b.conv(c, c, 1, relu=relu, src=-1), b.pool()), c, hw, dtype, micro_batch=mb)
    compare_minibatch(st, verbose="pool at the end c%d %s x %d" % (c, hw, mb), layout=B.NCHW)
    a, b = gpu_minibatch(st, layout=B.NCHW), gpu_minibatch(st, layout=B.NHWC)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


# ------------------------------------------------------------------------------ average pooling: batches of 8, 4 and 1 positions
@pytest.mark.parametrize("dtype", [C.FP32, C.BF16])
@pytest.mark.parametrize("k,c,hw", [(1, 8, (3, 4)), (2, 24, (7, 4)), (3, 5, (10, 9)), (5, 16, (5, 11)), (6, 8, (13, 6))])
def test_avgpool_windows(dtype, k, c, hw):
    st = single(lambda b: b.avgpool(k, src=-1), c, hw, dtype)
    compare_minibatch(st, verbose="avgpool %d of %s" % (k, hw))


# ------------------------------------------------------------------------------ max-pool gradient by cells of 2 x 2 positions
CELLS = [
    (2, 1, 8, (5, 6), 2),         # windows that do not overlap: position by position
    (3, 0, 16, (8, 6), 3),        # the last row and column belong to no window
    (3, 2, 8, (3, 1), 2),         # cells wholly in the padding, one column
    (4, 0, 24, (4, 4), 1),        # one window
    (4, 1, 5, (9, 10), 2),        # elements one by one in fp32
    (4, 3, 8, (7, 2), 3),
    (5, 2, 8, (9, 7), 2),         # wider than a cell's windows reach: so too
]


@pytest.mark.parametrize("dtype", [C.FP32, C.BF16])
@pytest.mark.parametrize("k,pad,c,hw,mb", CELLS)
def test_pool_gradient_at_stride_two(dtype, k, pad, c, hw, mb):
    """Identical inputs on both sides; a position takes up to nine gradients, added in one order and rounded once."""
    st = single(lambda b: b.pool(src=-1, k=k, stride=2, pad=pad), c, hw, dtype, micro_batch=mb, n_micro=1)
    xs, gs = stage_io(st)
    orc, gpu = OracleStage(st, gen.all_params(st)), GpuStage(st, gen.all_params(st))
    assert np.array_equal(orc.forward(0, xs[0]), gpu.forward(0, xs[0]))
    ref, dx = orc.backward(0, gs[0]), gpu.backward(0, gs[0])
    gpu.close()
    # fp32: eight additions of terms up to the largest |dy|, each within 2^-24 of a sum up to nine times that; bf16: one rounding, half an
    # ulp of the result, on either side
    top = float(np.max(np.abs(gs[0])))
    assert np.allclose(ref, dx, rtol=2.0 ** -7 if dtype == C.BF16 else 0, atol=72 * 2.0 ** -24 * top)


@pytest.mark.parametrize("k,pad,c,hw,mb", CELLS)
def test_pool_gradient_at_stride_two_behind_a_gate_and_a_sum(k, pad, c, hw, mb):
    def build(b):
        t = b.conv(c, c, 1, relu=1, src=-1)
        p = b.pool(src=t, k=k, stride=2, pad=pad)
        u = b.conv(c, c, k, stride=2, pad=pad, src=t)
        b.addl(p, u, relu=0)
    compare_minibatch(single(build, c, hw, C.FP32, micro_batch=mb), verbose="pool k%d p%d of %s, gate and sum" % (k, pad, hw))


# ------------------------------------------------------------------------------ weight gradient: steps of 32 pixels through small images
@pytest.mark.parametrize("k,stride,cin,cout,hw,mb", [
    (3, 1, 64, 72, (2, 3), 23),          # 32 pixels are five images and two pixels
    (3, 1, 16, 64, (1, 5), 17),          # ... six rows, each an image
    (3, 2, 64, 64, (9, 13), 5),          # the columns wrap in a step, with a stride
    (3, 1, 64, 128, (40, 1), 3),         # rows of one pixel
    (1, 1, 136, 64, (5, 7), 9),          # 1x1: a plain list of rows, ragged tiles
    (1, 2, 64, 64, (5, 4), 9),           # 1x1 with a stride keeps its image
])
def test_wgrad_small_images(k, stride, cin, cout, hw, mb):
    st = single(lambda b: b.conv(cin, cout, k, stride=stride, relu=1, src=-1), cin, hw, C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="wgrad k%d s%d %d->%d %s x %d" % (k, stride, cin, cout, hw, mb))


@pytest.mark.parametrize("k,cin,cout,hw,mb", [
    (3, 320, 320, 28, 4),       # one split: 49 tiles a group of waves
    (1, 1024, 1024, 51, 1),     # 41 of them, ragged
    (1, 1024, 4096, 40, 2),     # the wider of the two tiles
    (1, 64, 64, 56, 32),        # many splits
])
def test_wgrad_sums_are_short(k, cin, cout, hw, mb):
    """Operands of one sign.  A part of 384 pixels is 24 sums of 16 products, each rounded to half a unit, 2^-24/sqrt(3) of the sum so
    far on average: sqrt(24/3) of that for the part, independent parts of a group added up the same way, a split's partial and
    the total rounded once more: 6e-8 at most for the shapes here.  Twice that is allowed; one sum of 1568 pixels is at 1.5e-7."""
    assert max(_wgrad_errors(k, cin, cout, hw, mb)) < 1.2e-7


@pytest.mark.parametrize("cin,cout,hw,mb", [
    (64, 64, 16, 2),            # one split, two groups of two parts
    (256, 256, 16, 8),          # four splits
    (128, 512, 32, 2),
    (256, 256, 48, 1),          # parts of 96 pixels
    (768, 768, 16, 1),          # too many tiles for wave groups: units
])
def test_wgrad_sums_of_small_whole_maps_are_as_short_as_units(cin, cout, hw, mb):
    """Operands of one sign.  P parts of 8 sums of 16 products, rounded to 2^-24/sqrt(3) of the sum so far: 8/(3 P) of that squared, two parts
    of a group added up 2/P, two groups of a split 2 (2/P), and the total 1, P = 4 at the least, where the groups' sum is the total: sqrt(8/12 + 1/2 + 1)
    times 3.4e-8.  Parts of 384 pixels are 5.3e-8 to 6.4e-8 off here."""
    assert _wgrad_errors(3, cin, cout, hw, mb)[0] < 5.1e-8


def _wgrad_errors(k, cin, cout, hw, mb):
    """Of dw and db against float64, operands of one sign."""
    st = single(lambda b: b.conv(cin, cout, k, src=-1), cin, (hw, hw), C.BF16, micro_batch=mb, n_micro=1, need_input_grad=0)
    g = GpuStage(st, [(None, None)])
    rng = np.random.default_rng(cin + cout)
    x, dy = (torch.from_numpy(rng.random((mb, c, hw, hw), dtype=np.float32)).bfloat16().double() for c in (cin, cout))
    g.forward(0, x.float().numpy())
    g.backward(0, dy.float().numpy())
    dw, db = B.bapipe_stage_get_grads(g.h, 0, (cout, cin, k, k), (cout,))
    g.close()
    cols = torch.nn.functional.unfold(x, k, padding=k // 2).permute(1, 0, 2).reshape(cin * k * k, -1)
    rows = dy.permute(1, 0, 2, 3).reshape(cout, -1)
    off = lambda got, exact: float(np.linalg.norm(got - exact) / np.linalg.norm(exact))
    return off(dw.reshape(cout, -1), (rows @ cols.t().contiguous()).numpy()), off(db, rows.sum(dim=1).numpy())


@pytest.mark.parametrize("k,stride,cin,cout,hw,mb", [
    (1, 1, 64, 64, (5, 6), 1),           # 30 pixels: the second group of waves has none
    (3, 1, 72, 136, (7, 9), 1),          # 63 pixels: one short of a step of both groups; ragged tiles both ways
    (3, 1, 8, 40, (13, 20), 1),          # 260 pixels: a step of four, over several splits
    (3, 2, 128, 64, (31, 29), 5),        # splits that end inside an image
    (1, 1, 256, 1024, (11, 9), 2),       # one split, added to the gradient
    (3, 1, 520, 264, (30, 31), 3),       # 128-row tiles, the last of them ragged
    (1, 1, 24, 2056, (40, 40), 20),      # ... of a layer narrower than a tile
    (3, 1, 256, 256, (56, 57), 8),       # 256 x 256 in one group, splits that end inside an image
])
def test_wgrad_groups_of_waves(k, stride, cin, cout, hw, mb):
    st = single(lambda b: b.conv(cin, cout, k, stride=stride, relu=1, src=-1), cin, hw, C.BF16, micro_batch=mb)
    compare_minibatch(st, verbose="wgrad groups k%d s%d %d->%d %s x %d" % (k, stride, cin, cout, hw, mb))


# ------------------------------------------------------------------------------ gradients read in the middle of a mini-batch
@pytest.mark.parametrize("cin,cout,mb,n_micro,at", [
    (128, 1000, 100, 16, (13,)),      # 13 micro-batches take seven copies of the partial sums, 16 take five
    (256, 256, 128, 16, (15,)),
    (64, 72, 9, 5, (1, 2, 4)),
])
def test_gradients_read_in_the_middle_of_a_mini_batch(monkeypatch, cin, cout, mb, n_micro, at):
    """The deferred product over the micro-batches so far, then over the rest; what lies behind each block of the stage's
    memory stays as it is."""
    guard = 1 << 21

    class Guarded(B.TorchAllocator):
        def _alloc(self, nbytes, ctx):
            p = super()._alloc(nbytes + guard, ctx)
            t = self.live[p]
            self.behind = getattr(self, "behind", []) + [t[p - t.data_ptr() + nbytes:][:guard].fill_(0xA5)]
            torch.cuda.synchronize()
            return p

    monkeypatch.setattr(B, "TorchAllocator", Guarded)
    st = single(lambda b: b.linear(cin, cout, src=-1), cin, (1, 1), C.BF16, micro_batch=mb, n_micro=n_micro)
    g = GpuStage(st, gen.all_params(st))
    xs, gs = stage_io(st)
    bf16 = lambda a: torch.from_numpy(a.reshape(mb, -1)).bfloat16().double().numpy()
    dw, db = np.zeros((cout, cin)), np.zeros(cout)
    for m in range(n_micro):
        g.forward(m, xs[m])
        g.backward(m, gs[m])
        dw += bf16(gs[m]).T @ bf16(xs[m])
        db += bf16(gs[m]).sum(axis=0)
        if m + 1 in at or m + 1 == n_micro:
            got = g.grads(0)
            # fp32 sums of up to 2048 products: the error of a random order is about sqrt(2048) 2^-24 = 3e-6
            assert np.linalg.norm(got[0] - dw) < 1e-5 * np.linalg.norm(dw), m
            assert np.linalg.norm(got[1] - db) < 1e-5 * np.linalg.norm(db), m
    assert len(g.alloc.behind) >= 6 and all(bool((t == 0xA5).all()) for t in g.alloc.behind)
    g.close()


# ------------------------------------------------------------------------------ weight gradients on a stream of their own
def _wide_chain(micro_batch=3, n_micro=4):
    """Seven 1x1 convolutions of 1024 channels with batch-norms and residual sums, no gates: the filters alone are worth a
    hand-over after four of them in a backward pass, the other three are left for its end.  (No batch-norm behind the second
    of each pair: it would take away what a shift of the first one's output changes, and with it that gradient.)"""
    b = C._Builder()
    b.conv(1024, 1024, 1, bias=0, src=-1)
    t = b.bn(1024)
    for _ in range(3):
        b.conv(1024, 1024, 1, bias=0)
        b.bn(1024)
        t = b.addl(b.conv(1024, 1024, 1, bias=0), t, relu=0)
    return C._stage("wide chain", b.layers, C.BF16, (1024, 3, 3), micro_batch, n_micro, 1, 2, 1, C.BASE_SEED + 81, "kaiming")


HANDED_OVER = [
    ("bottlenecks", lambda: C.resnet50_stage(cin=128, mid3=64, mid4=128, hw=29, n3=2, n4=2, micro_batch=24, n_micro=5)),
    ("wide chain", _wide_chain),
    ("3x3", lambda: single(lambda b: (b.conv(256, 256, 3, relu=1, src=-1), b.conv(256, 256, 3, relu=1)), 256, (20, 20), C.BF16, micro_batch=16, n_micro=3)),
]


@pytest.mark.parametrize("name,make", HANDED_OVER)
def test_weight_gradients_reach_their_stream(name, make):
    """A backward pass ends behind what its weight-gradient stream was given before, so kernels of it run there."""
    st = make()
    g = GpuStage(st, gen.all_params(st), wgrad_stream=True)
    xs, gs = stage_io(st)
    g.forward(0, xs[0])
    dy, dx = to_dev(st, gs[0], B.NHWC), to_dev(st, xs[0], B.NHWC)
    a = torch.randn(8192, 8192, device="cuda")
    busy, done = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    with torch.cuda.stream(g.wstream):
        for _ in range(4):
            a @ a
    busy.record(g.wstream)
    B.bapipe_stage_backward(g.h, 0, dy.data_ptr(), dx.data_ptr())
    done.record(g.stream)
    torch.cuda.synchronize()
    g.close()
    assert busy.elapsed_time(done) > 0


@pytest.mark.parametrize("name,make", HANDED_OVER)
def test_handed_over_weight_gradients_give_the_same_results_bit_for_bit(name, make):
    ref = gpu_minibatch(make())
    for kw in (dict(backward_stream=True), dict(backward_stream=True, static=True), dict(backward_stream="no wgrad stream"),
               dict(wgrad_stream=True)):
        got = gpu_minibatch(make(), eager_sync=False, **kw)
        assert sorted(got) == sorted(ref)
        for k in ref:
            assert np.array_equal(got[k], ref[k]), (kw, k)


def test_handed_over_weight_gradients_against_the_oracle():
    compare_minibatch(_wide_chain(), backward_stream=True, verbose="three streams, wide chain")


# ------------------------------------------------------------------------------ pixel tiles that depend on other streams
def test_pixel_tiles_beside_other_streams_same_bits():
    """144 tiles of 256 x 128 stay whole beside other streams and are halved alone on the chip."""
    def build(b):
        b.conv(512, 512, 3, relu=1, src=-1)
        b.conv(512, 512, 3, relu=1)
    st = single(build, 512, (14, 14), C.BF16, micro_batch=46, n_micro=3)
    ref, got = gpu_minibatch(st), gpu_minibatch(st, eager_sync=False, backward_stream=True)
    assert sorted(got) == sorted(ref)
    for k in ref:
        assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("mb", [46, 60])
def test_large_tiles_beside_other_streams_same_bits(mb):
    """Alone tiles of 128 x 256; beside other streams, 144 halves of 256 x 128 and 184, which are 92 tiles of 256 x 256."""
    def build(b):
        b.conv(512, 512, 3, relu=1, src=-1)
        b.conv(512, 512, 3, relu=1)
    st = single(build, 512, (14, 14), C.BF16, micro_batch=mb, n_micro=2)
    ref, got = gpu_minibatch(st), gpu_minibatch(st, eager_sync=False, backward_stream=True)
    assert sorted(got) == sorted(ref)
    for k in ref:
        assert np.array_equal(got[k], ref[k]), k


def _conv_in_doubles(x, w, pad):
    """The convolution and the sum of its terms' magnitudes, float64, on the GPU."""
    x, w = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda").double() for a in (x, w))
    n, _, h, wd = x.shape
    cols = torch.nn.functional.unfold(x, w.shape[2:], padding=pad).transpose(1, 2).reshape(n * h * wd, -1).contiguous()
    m = w.reshape(w.shape[0], -1).t().contiguous()
    back = lambda t: t.reshape(n, h, wd, -1).permute(0, 3, 1, 2).cpu().numpy()
    return back(cols @ m), back(cols.abs() @ m.abs())


@pytest.mark.parametrize("k,cin,cout,hw,mb", [
    (3, 128, 2048, (13, 17), 10),      # 128 x 256: 144 halves, pixels end inside a tile
    (1, 1088, 2048, (11, 19), 10),     # ... 17 K-tiles
    (3, 128, 2048, (13, 17), 13),      # 256 x 128: 192 halves
    (3, 192, 1112, (15, 11), 24),      # ... 144 of a width that ends inside a tile; 27 K-tiles
    (3, 128, 2048, (13, 17), 19),      # 256 x 256: 272 halves
    (1, 1024, 4352, (9, 8), 29),       # ... one tap; 17 channel tiles
])
def test_conv_tiles_of_eight_waves(k, cin, cout, hw, mb):
    _conv_against_doubles(k, cin, cout, hw, mb)


@pytest.mark.parametrize("cin,cout,mb", [(1088, 16400, 33), (1024, 16640, 64)])
def test_conv_tiles_that_start_anywhere_in_k(cin, cout, mb):
    """One row of 129 and 130 tiles over a filter of 35 MB: every block at another of the 17 and 16 K-tiles."""
    _conv_against_doubles(1, cin, cout, (1, 1), mb)


@pytest.mark.parametrize("cin,cout,hw,mb", [
    (64, 64, (83, 81), 5),             # 180 patches, cut on both sides
    (64, 64, (17, 145), 10),           # one row of pixels in the last patch, one column
    (128, 64, (35, 47), 36),           # two slices of channels; gradient 64->128
    (256, 256, (30, 31), 32),          # ... four
    (64, 72, (90, 90), 5),             # an output width that the patches do not take
    (8, 64, (45, 33), 2),              # first layer
    (8, 128, (17, 31), 1),             # ... a last patch of one row
])
def test_conv_patches_of_ragged_images(cin, cout, hw, mb):
    _conv_against_doubles(3, cin, cout, hw, mb)


@pytest.mark.parametrize("cin,cout,hw,mb", [
    (64, 64, (32, 64), 16),       # 128 patches, the fewest; weight gradient by 64 x 64 tiles
    (128, 128, (64, 64), 4),      # ... and 2.4 GMAC, the least for units of 8 x 16 pixels
    (256, 256, (16, 16), 32),     # ... one patch an image
    (128, 192, (32, 16), 24),     # ... 192 = 3 x 64 output channels
    (64, 64, (16, 16), 7),        # neither
    (8, 64, (160, 160), 16),      # first layer, with the fewest pixels for its own weight gradient
])
def test_conv_patches_of_whole_images(cin, cout, hw, mb):
    _conv_against_doubles(3, cin, cout, hw, mb)


@pytest.mark.parametrize("hw", [(83, 81), (82, 95), (90, 84)])
def test_ragged_patches_with_pool_and_gate(hw):
    """Against the same layers without the pool, which is done here: odd sides lose their last row or column.  The ReLU gate of
    the input gradient against float64 sums: two bf16 roundings of 2^-9 on the way, three of them allowed."""
    def build(pool):
        def layers(b):
            b.conv(64, 64, 3, relu=1, src=-1)
            b.conv(64, 64, 3, relu=1)
            if pool:
                b.pool()
        return single(layers, 64, hw, C.BF16, micro_batch=6, n_micro=1)
    params = gen.all_params(build(True))
    rng = np.random.default_rng(hw[1])
    bf16 = lambda a: torch.from_numpy(a.astype(np.float32)).bfloat16().float().numpy()
    x = bf16(rng.standard_normal((6, 64) + hw))
    h, w = hw[0] // 2, hw[1] // 2
    dy = bf16(rng.standard_normal((6, 64, h, w)))
    g = GpuStage(build(True), params)
    y, idx, dx = g.forward(0, x), g.pool_indices(2, 0), g.backward(0, dy)
    g.close()
    plain = GpuStage(build(False), params)
    full = plain.forward(0, x)
    windows = np.stack([full[:, :, i:2 * h:2, j:2 * w:2] for i in (0, 1) for j in (0, 1)])
    at = np.argmax(windows, 0)                                     # the first of equals
    assert np.array_equal(idx, at) and np.array_equal(y, np.take_along_axis(windows, at[None], 0)[0])
    spread = np.zeros_like(full)
    for k in range(4):
        spread[:, :, k // 2:2 * h:2, k % 2:2 * w:2] = np.where(at == k, dy, 0)
    assert np.array_equal(plain.backward(0, spread), dx)
    plain.close()
    first = GpuStage(single(lambda b: b.conv(64, 64, 3, relu=1, src=-1), 64, hw, C.BF16, micro_batch=6, n_micro=1), params[:1])
    gate = first.forward(0, x) > 0
    first.close()
    turned = lambda p: np.flip(bf16(p[0]), (2, 3)).transpose(1, 0, 2, 3)
    ref, _ = _conv_in_doubles(bf16(np.where(gate, _conv_in_doubles(spread * (full > 0), turned(params[1]), 1)[0], 0)), turned(params[0]), 1)
    assert np.linalg.norm(dx - ref) <= 3 * 2.0 ** -9 * np.linalg.norm(ref)


def _conv_against_doubles(k, cin, cout, hw, mb):
    """Against float64: half a bf16 step of the result and a rounding of 2^-24 for each term of the sum."""
    st = single(lambda b: b.conv(cin, cout, k, src=-1), cin, hw, C.BF16, micro_batch=mb, n_micro=1)
    params = gen.all_params(st)
    g = GpuStage(st, params)
    rng = np.random.default_rng(cout + mb)
    bf16 = lambda a: torch.from_numpy(a.astype(np.float32)).bfloat16().float().numpy()
    x, dy = bf16(rng.standard_normal((mb, cin) + hw)), bf16(rng.standard_normal((mb, cout) + hw))
    y = g.forward(0, x)
    dx = g.backward(0, dy)
    dw, _ = g.grads(0)
    g.close()
    w, b = params[0]
    w = bf16(w)
    pixels = mb * hw[0] * hw[1]
    xs, gs = (torch.from_numpy(a).to("cuda").double() for a in (x, dy))
    cols = torch.nn.functional.unfold(xs, (k, k), padding=k // 2).transpose(0, 1).reshape(-1, pixels)
    rows = gs.permute(0, 2, 3, 1).reshape(pixels, cout)
    ref, terms = (a.t().reshape(dw.shape).cpu().numpy() for a in (cols @ rows, cols.abs() @ rows.abs()))
    assert np.all(np.abs(dw - ref) <= (pixels + 1) * 2.0 ** -24 * terms)
    ref, terms = _conv_in_doubles(x, w, k // 2)
    ref += 0.0 if b is None else b.reshape(1, -1, 1, 1)
    assert np.all(np.abs(y - ref) <= 2.0 ** -8 * np.abs(ref) + (k * k * cin + 1) * 2.0 ** -24 * (terms + np.abs(ref)))
    ref, terms = _conv_in_doubles(dy, np.flip(w, (2, 3)).transpose(1, 0, 2, 3), k // 2)
    assert np.all(np.abs(dx - ref) <= 2.0 ** -8 * np.abs(ref) + (k * k * cout + 1) * 2.0 ** -24 * (terms + np.abs(ref)))


# ------------------------------------------------------------------------------ weight update: ragged tiles, both access widths, both copies
def _mini_batch(gpu, stage, xs, gs):
    out = []
    for t, m in one_f_one_b_order(stage["n_micro"], B.bapipe_stage_stash_bytes(gpu.h)[1]):
        out.append(gpu.forward(m, xs[m]) if t == "F" else gpu.backward(m, gs[m]))
    return out


@pytest.mark.parametrize("dtype", [C.FP32, C.BF16])
@pytest.mark.parametrize("kind,cin,cout", [("conv", 72, 136), ("conv", 3, 20), ("conv", 7, 5), ("linear", 136, 72),
                                           ("linear", 24, 8), ("lstm", 24, 40), ("lstm", 128, 128)])
def test_update_leaves_the_copies_that_setting_the_weights_makes(dtype, kind, cin, cout):
    """The mini-batch after an update runs on the copies that the update wrote; the same weights set from the host are
    copied by other kernels.  Outputs and input gradients (working and transposed copies) agree bit for bit."""
    b = C._Builder()
    if kind == "conv":
        b.conv(cin, cout, 3, relu=1, src=-1)
        b.conv(cout, cin, 3, relu=0)
    elif kind == "linear":
        b.linear(cin, cout, relu=1, src=-1)
        b.linear(cout, cin, relu=0)
    else:
        b.lstm(cin, cout, src=-1)
    hw = {"conv": (6, 5), "linear": (1, 1), "lstm": (4, 1)}[kind]
    st = C._stage("update", b.layers, dtype, (cin,) + hw, 3, 2, 1, 2, 1, C.BASE_SEED + 78, "lstm" if kind == "lstm" else "kaiming")
    xs, gs = stage_io(st)
    one = GpuStage(st, gen.all_params(st, perturb=True))
    _mini_batch(one, st, xs, gs)
    B.bapipe_stage_step(one.h, 0.05)
    other = GpuStage(st, [one.get_params(i) if w is not None else (None, None)
                          for i, (w, _) in enumerate(gen.all_params(st, perturb=True))])
    for u, v in zip(_mini_batch(one, st, xs, gs), _mini_batch(other, st, xs, gs)):
        assert np.array_equal(u, v)
    one.close()
    other.close()
