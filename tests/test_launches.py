"""Which kernels a call launches and on what grids, asked without a GPU: tests/launch_recorder.c takes the place of the runtime."""
import ctypes as ct
import json
import os
import re
import shutil
import struct
import subprocess
import sys

import pytest

from oracle.stage import one_f_one_b_order
from paper_2012_12544_amd import binding as B
from stage_inputs import configs as C

HERE = os.path.dirname(os.path.abspath(__file__))
SOMEWHERE = 1 << 40          # an address; nothing is read or written there


class _GatherConv(ct.Structure):
    _fields_ = [(f, ct.c_int) for f in "N Hi Wi Ci Ho Wo Co R S s_out s_in pad_h pad_w beside by_norm wt_panels".split()]


class _GradEpi(ct.Structure):
    _fields_ = [("gate", ct.c_void_p), ("accum", ct.c_int), ("accum_from", ct.c_void_p)]


def _gather(lib, case, rec):
    f = getattr(lib, "_ZN6bapipe16conv_gather_mfmaEPKvS1_PKfPviNS_7GradEpiERKNS_10GatherConvES4_PjP12ihipStream_tPfS1_S3_")
    at = ct.c_void_p(SOMEWHERE)
    return f(at, at, None, at, ct.c_int(0), _GradEpi(None, case.get("accum", 0), None), ct.byref(_GatherConv(*case["g"])), at, at, None, None, None, None)


def _pool(lib, case, rec):
    """2x2 pool that ends a stage of NCHW neighbours: forward, then the gradient.  Returns whether either takes that layout."""
    at, dt, shape, stored = ct.c_void_p(SOMEWHERE), ct.c_int(case["dtype"]), [ct.c_int(v) for v in case["shape"]], ct.c_bool(False)
    assert lib._ZN6bapipe14maxpool2x2_fwdEiPKvPvPhiiiiP12ihipStream_tS2_Pb(dt, at, at, at, *shape, None, at, ct.byref(stored)) == 0
    takes = lib._ZN6bapipe25maxpool2x2_bwd_takes_nchwEiPKvPKhS1_S1_iiii
    takes.restype = ct.c_bool
    return [stored.value, takes(dt, at, at, at, None, *shape)]


STREAMS = dict(own=1 << 20, backward=2 << 20, wgrad=3 << 20)


def _mini_batch(lib, case, rec):
    """One mini-batch in 1F1B order and the update.  Returns how often the update allocated; the blocks that the stage asked its allocator
    for are left in case["blocks"]."""
    blocks = case["blocks"] = []

    def alloc(nbytes, ctx):
        blocks.append((SOMEWHERE + (sum(n for _, n in blocks) + 4095) // 4096 * 4096 + 4096 * len(blocks), nbytes))
        return blocks[-1][0]

    b = C._Builder()
    for kind, args in case["layers"]:
        getattr(b, kind)(*args[0], **args[1])
    st = C._stage("recorded", b.layers, C.BF16, tuple(case["input"]), case["micro_batch"], case["n_micro"], 1, case["in_flight"], 1, 0, "kaiming")
    o = B.make_opts(st, stream=STREAMS["own"])
    o.mem.alloc, o.mem.free = B.ALLOC_FN(alloc), B.FREE_FN(lambda ptr, ctx: None)
    h = B.bapipe_stage_create(b.layers, case["micro_batch"], case["n_micro"], o)
    if case["streams"] > 1:
        B.bapipe_stage_set_streams(h, STREAMS["backward"], STREAMS["wgrad"] if case["streams"] == 3 else None)
    backward = B.bapipe_stage_backward_static if case.get("static") else B.bapipe_stage_backward
    for what, m in one_f_one_b_order(case["n_micro"], B.bapipe_stage_stash_bytes(h)[1]):
        if what == "F":
            B.bapipe_stage_forward(h, m, SOMEWHERE >> 1, SOMEWHERE >> 2)
        else:
            backward(h, m, SOMEWHERE >> 3, SOMEWHERE >> 4)
    news = rec.recorder_news()
    assert B.load().bapipe_stage_step(h, 0.1) == 0
    news = rec.recorder_news() - news
    B.bapipe_stage_destroy(h)
    return news


def _record(recorder, library, cases):
    """In a process of its own: for each case what the call returned and (kernel, template arguments, grid, stream, tickets, LDS) of every launch."""
    rec, lib = ct.CDLL(recorder, mode=ct.RTLD_GLOBAL), ct.CDLL(library)
    B.LIB_PATH = library
    rec.recorder_launch.restype = ct.c_char_p
    out = []
    for case in cases:
        rec.recorder_clear()
        rc = globals()["_" + case["call"]](lib, case, rec)
        launches = []
        for i in range(rec.recorder_launches()):
            grid, stream, tickets, lds = (ct.c_uint * 3)(), ct.c_size_t(), ct.c_size_t(), ct.c_size_t()
            name = rec.recorder_launch(i, grid, ct.byref(stream), ct.byref(tickets), ct.byref(lds)).decode()
            m = re.search(r"\d(k_[a-z0-9_]+?)(?:I((?:L[ib]\d+E)+)E|E?v|E?P|I)", name)
            launches.append((m.group(1) if m else name, [int(a) for a in re.findall(r"L[ib](\d+)E", m.group(2) or "")] if m else [], list(grid),
                             stream.value, tickets.value, lds.value))
        out.append(dict(rc=rc, launches=launches, blocks=case.get("blocks")))
    return out


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    if shutil.which("gcc") is None:
        pytest.skip("needs gcc")
    B.load()
    so = str(tmp_path_factory.mktemp("recorder") / "recorder.so")
    subprocess.check_call(["gcc", "-O1", "-std=c11", "-shared", "-fPIC", "-Wall", "-o", so, os.path.join(HERE, "launch_recorder.c")])

    def run(cases):
        r = subprocess.run([sys.executable, os.path.abspath(__file__), so, B.LIB_PATH], input=json.dumps(cases), capture_output=True, text=True, timeout=120,
                           env=dict(os.environ, PYTHONPATH=os.path.dirname(HERE)))
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout)
    return run


# ------------------------------------------------------------------------------ gather convolution
# Template arguments of k_gather_mfma: BP, BC, WP, WC, BK, STAGES, KG, S1, TAPS_INNER, PHASED, PANELS
KG, PHASED, PANELS = 6, 9, 10


def _strided_gradient(n, c, k, side, r, stride):
    """Input gradient of an r x r convolution c -> k at that stride, no padding, of `side` x `side` maps."""
    out = (side - r) // stride + 1
    return [n, out, out, k, side, side, c, r, r, 1, stride, r - 1, r - 1, 0, 0, 0]


def test_a_launch_of_pixel_classes_is_of_a_kernel_that_knows_them(record):
    """The classes of a strided gradient are the grid's z axis.  A kernel that does not look at it stores each tile once per class,
    and where it adds to what is stored, adds that often."""
    cases = [dict(call="gather", accum=accum, g=_strided_gradient(n, c, k, side, r, stride))
             for c, k in ((4096, 4096), (6144, 3072), (2048, 9216), (4096, 4608), (1024, 256), (64, 64), (256, 72))
             for side, r, stride in ((2, 1, 2), (3, 1, 2), (3, 1, 3), (7, 1, 2), (3, 3, 2), (8, 3, 2), (5, 2, 4))
             for n in (1, 5, 9, 12, 16, 40) for accum in (0, 1)]
    classes = 0
    for case, got in zip(cases, record(cases)):
        assert got["rc"] == 0, case
        name, args, grid = got["launches"][0][:3]
        assert name == "k_gather_mfma", got
        assert grid[2] == 1 or (args[PHASED] and args[KG] == 1), (case, got)
        classes += grid[2] > 1
    assert classes > len(cases) // 2           # otherwise nothing was asked


def _flat(rows, cin, cout, panels):
    return [rows, 1, 1, cin, 1, 1, cout, 1, 1, 1, 1, 0, 0, 0, 0, panels]


BAND = [(2048, 8192), (2560, 6144), (3072, 5120), (4096, 4096), (4608, 4096), (6144, 3072), (9216, 2048)]       # 15 to 20 M weights


@pytest.mark.parametrize("panels", [0, 1])
@pytest.mark.parametrize("rows,shares", [(32, False), (33, True), (64, True), (65, False)])
def test_few_rows_share_k(record, rows, shares, panels):
    """Of a filter in panels up to four splits are added by their tile's last block, others by a launch (the input product of an LSTM of one
    step, strided convolutions of single pixels)."""
    cases = [dict(call="gather", g=_flat(rows, cin, cout, panels)) for cin, cout in BAND]
    if not panels:               # the gradient of a 1x1 / 2 convolution of 1x1 maps: one class of pixels
        cases += [dict(call="gather", g=_strided_gradient(rows, cout, cin, 1, 1, 2)) for cin, cout in BAND]
    for case, (cin, cout), got in zip(cases, BAND * 2, record(cases)):
        name, args, grid = got["launches"][0][:3]
        assert got["rc"] == 0 and name == "k_gather_mfma", got
        if shares:
            assert args[KG] == 2 and grid == [cout // 64, min(256 // (cout // 64), cin // 512), 1], (case, got)
            adds = not panels or grid[1] > 4
            assert [launch[0] for launch in got["launches"][1:]] == (["k_gather_splitk_reduce"] if adds else []), (case, got)
        elif case["g"][10] == 1:
            assert grid[1] == 1 and len(got["launches"]) == 1, (case, got)


@pytest.mark.parametrize("layer,input,mb,panels", [
    (("lstm", [[8224, 512], {}]), (8224, 4, 1), 16, 2),              # 33.7 MB of filter, 64 rows, in either direction
    (("lstm", [[8224, 512], {}]), (8224, 5, 1), 13, 0),              # 65 rows
    (("lstm", [[8192, 512], {}]), (8192, 4, 1), 16, 0),              # 32 MiB
    (("conv", [[1024, 16416, 1], {}]), (1024, 7, 7), 1, 2),
    (("conv", [[1024, 16416, 1], {}]), (1024, 7, 7), 2, 0),
    (("conv", [[1024, 16416, 1], dict(stride=2)]), (1024, 14, 14), 1, 1),      # its gradient has classes of pixels
])
def test_a_filter_that_is_streamed_is_kept_in_panels(record, layer, input, mb, panels):
    """The input product of a wide LSTM, 1x1 convolutions of small maps: more than the L2s hold, for one row of tiles."""
    kind, (args, kw) = layer
    case = dict(call="mini_batch", layers=[(kind, [args, dict(kw, src=-1)])], input=input, micro_batch=mb, n_micro=1, in_flight=1, streams=1)
    got = record([case])[0]
    in_panels = [a[PANELS] for name, a, *_ in got["launches"] if name == "k_gather_mfma"]
    assert got["rc"] == 0 and len(in_panels) >= 2 and sum(in_panels) == panels, got


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("streams", [1, 2, 3])
def test_passes_that_may_run_at_once_have_tickets_of_their_own(record, streams, static):
    """A block that counts itself among another launch's would add sums that are not there yet."""
    linear = lambda cin, cout: ("linear", [[cin, cout], {}])
    case = dict(call="mini_batch", layers=[("linear", [[4096, 4096], dict(src=-1)]), linear(4096, 4608), linear(4608, 4096)], input=[4096, 1, 1],
                micro_batch=48, n_micro=3, in_flight=2, streams=streams, static=static)
    got = record([case])[0]
    words = {}
    for name, args, grid, stream, tickets, _ in got["launches"]:
        if name == "k_gather_mfma" and 1 < grid[1] <= 4:
            assert tickets and grid[0] <= 128, got
            words.setdefault(stream, set()).add(tickets)
    assert set(words) == {STREAMS[s] for s in ("own", "backward")[:min(streams, 2)]}
    assert sum(len(w) for w in words.values()) == len(set().union(*words.values())) == len(words), words
    assert all(any(at <= t and t + 128 * 4 <= at + n for at, n in got["blocks"]) for w in words.values() for t in w)
    starts = sorted(set().union(*words.values()))
    assert all(b - a >= 128 * 4 for a, b in zip(starts, starts[1:]))


def test_an_update_allocates_nothing(record):
    """What is enqueued in a mini-batch's rhythm does not fail for want of host memory, where an exception would cross the C ABI."""
    conv = lambda cin, cout, k: ("conv", [[cin, cout, k], {}])
    case = dict(call="mini_batch", layers=[("conv", [[64, 64, 3], dict(src=-1)])] + [conv(64, 64, 1)] * 20 + [("flatten", [[], {}]), ("linear", [[64 * 8 * 8, 64], {}])],
                input=[64, 8, 8], micro_batch=2, n_micro=2, in_flight=2, streams=1)
    got = record([case])[0]
    assert got["rc"] == 0 and got["launches"][-1][0] == "k_sgd_group"


# ------------------------------------------------------------------------------ pools that store and read NCHW
def test_pools_of_few_channels_leave_large_maps_to_the_conversion(record):
    """Most lanes of the kernel that does both would idle."""
    shapes = [(C.FP32, n, hw, c) for c in (4, 8, 12, 16) for n, hw in ((4, 64), (32, 64), (33, 64), (32, 224))]
    shapes += [(C.BF16, n, hw, c) for c in (8, 16, 64) for n, hw in ((1, 2), (32, 64), (33, 65), (32, 224))]
    cases = [dict(call="pool", dtype=int(dt == C.BF16), shape=[n, hw, hw, c]) for dt, n, hw, c in shapes]
    for (_, n, hw, c), got in zip(shapes, record(cases)):
        both = c >= 12 or n * (hw // 2) ** 2 <= 32768
        assert got["rc"] == [both, both], (n, hw, c)
        assert [launch[0] for launch in got["launches"]] == ["k_pool_fwd_nchw" if both else "k_pool_fwd"], (got, n, hw, c)


# ------------------------------------------------------------------------------ blocks of a kernel that fit a compute unit
def _kernels_of_the_library():
    """What the code objects of the built library say of each kernel: name -> its metadata."""
    msgpack = pytest.importorskip("msgpack")
    B.load()
    data, out, at = open(B.LIB_PATH, "rb").read(), {}, 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            first, size, n = struct.unpack_from("<3Q", data, entry)
            elf = data[at + first:at + first + size]
            if data[entry + 24:entry + 24 + n].endswith(b"gfx950"):
                sections, = struct.unpack_from("<Q", elf, 40)
                for i in range(struct.unpack_from("<H", elf, 60)[0]):
                    kind, where, length = struct.unpack_from("<I", elf, sections + 64 * i + 4)[0], *struct.unpack_from("<2Q", elf, sections + 64 * i + 24)
                    if kind == 7 and struct.unpack_from("<3I", elf, where)[2] == 32:          # a note with AMDGPU metadata
                        owner, desc, _ = struct.unpack_from("<3I", elf, where)
                        start = where + 12 + (owner + 3) // 4 * 4
                        out.update((k[".name"], k) for k in msgpack.unpackb(elf[start:start + desc])["amdhsa.kernels"])
            entry += 24 + n
        at += 1
    return out


def _wgrad_halo(lib, case, rec):
    at = ct.c_void_p(SOMEWHERE)
    shape = (ct.c_int * 11)(*case["shape"])
    return getattr(lib, "_ZN6bapipe18wgrad3x3_halo_mfmaEPKvS1_PfS2_PvRKNS_9ConvShapeEP12ihipStream_t")(at, at, at, at, at, shape, None)


def test_blocks_of_the_halo_weight_gradient_are_one_round(record):
    """A block for every unit is rounded up to whole splits of a tile, so that a unit may be handed a second block: one that has to wait for
    the first would take the launch as long again.  Where there is one for each unit none takes two."""
    shapes = [(96, 32, 32, c, 32, 32, k, 3, 3, 1, 1) for c, k in ((64, 64), (64, 192), (192, 192), (320, 320), (448, 448), (704, 704))]
    most = 0
    for got in record([dict(call="wgrad_halo", shape=s) for s in shapes]):
        name, _, grid, _, _, lds = got["launches"][0]
        assert got["rc"] == 0 and name == "k_wgrad3x3_halo"
        most = max(most, grid[0] * grid[1])
        assert (2 * lds <= 160 << 10) == (grid[0] * grid[1] > 256), got
    kernel, = [k for name, k in _kernels_of_the_library().items() if "k_wgrad3x3_halo" in name]
    assert 256 < most <= 512
    # a block has a wave on each SIMD, of whose 512 registers a lane a wave of two has half
    assert kernel[".vgpr_count"] <= 256 and kernel[".vgpr_spill_count"] == 0 and kernel[".max_flat_workgroup_size"] == 256


if __name__ == "__main__":
    print(json.dumps(_record(sys.argv[1], sys.argv[2], json.load(sys.stdin))))
