"""Where the partial sums of weight gradients lie, asked without a GPU: tests/launch_recorder.c takes the place of the runtime."""
import ctypes as ct
import json
import os
import shutil
import subprocess
import sys

import pytest

from paper_2012_12544_amd import binding as B
from stage_inputs import configs as C

HERE = os.path.dirname(os.path.abspath(__file__))
WORK, ELSEWHERE = 1 << 40, 1 << 20          # addresses; nothing is read or written there


class _ConvShape(ct.Structure):
    _fields_ = [(f, ct.c_int) for f in "N H W C P Q K R S stride pad".split()]


class _WgradJob(ct.Structure):
    _fields_ = [("x", ct.c_void_p), ("dy", ct.c_void_p), ("dw", ct.c_void_p), ("db", ct.c_void_p), ("c", _ConvShape), ("x2", ct.c_void_p), ("dw2", ct.c_void_p)]


def _record(recorder, library, cases):
    """In a process of its own: for each case the workspace it is given, and (offset, bytes) of every product's partial sums."""
    rec, lib = ct.CDLL(recorder, mode=ct.RTLD_GLOBAL), ct.CDLL(library)
    size = getattr(lib, "_ZN6bapipe25conv_wgrad_mfma_workspaceERKNS_9ConvShapeE")
    size.restype = ct.c_size_t
    many = getattr(lib, "_ZN6bapipe20conv_wgrad_mfma_jobsEPKNS_8WgradJobEiPvmP12ihipStream_tb")
    out = []
    for case in cases:
        shapes = [_ConvShape(*s) for s in case["shapes"]]
        room = max(size(ct.byref(s)) for s in shapes) + case.get("more", 0)
        rec.recorder_clear()
        jobs = (_WgradJob * len(shapes))(*[_WgradJob(ELSEWHERE, ELSEWHERE, ELSEWHERE, ELSEWHERE, s, *([ELSEWHERE] * 2 if case["pair"] else [None] * 2))
                                           for s in shapes])
        rc = many(jobs, ct.c_int(len(shapes)), ct.c_void_p(WORK), ct.c_size_t(room), None, ct.c_bool(case["beside"]))
        parts = []
        for i in range(rec.recorder_count()):
            first, nbytes = ct.c_size_t(), ct.c_size_t()
            rec.recorder_get(i, ct.byref(first), ct.byref(nbytes))
            parts.append((first.value - WORK, nbytes.value))
        out.append(dict(rc=rc, room=room, parts=parts, launches=rec.recorder_launches()))
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


def _in_turn_or_side_by_side(case, got):
    """Partial sums of one launch after another from the start of the workspace on, those of one launch side by side."""
    assert got["rc"] == 0
    end = 0
    for first, nbytes in got["parts"]:
        assert first == 0 or first >= end
        end = first + nbytes
        assert end <= got["room"], (case, got)


@pytest.mark.parametrize("more", [0, 1 << 20, 64 << 20])
def test_partial_sums_of_a_pair_stay_in_the_workspace(record, more):
    """The two weight gradients of an LSTM layer whose input is as wide as its output, given what either of them asks for and some more."""
    cases = [dict(shapes=[(rows, 1, 1, h, 1, 1, 4 * h, 1, 1, 1, 0)], pair=True, beside=False, more=more)
             for h in (8, 64, 72, 128, 192, 256, 384, 512, 640, 768, 896, 1000, 1024, 2048)
             for rows in (1, 40, 64, 333, 1000, 1024, 2560, 3200, 4096, 6400, 12800, 51200)]
    results = record(cases)
    for case, got in zip(cases, results):
        _in_turn_or_side_by_side(case, got)
    assert sum(len(got["parts"]) == 2 for got in results) >= 20           # otherwise nothing was asked


@pytest.mark.parametrize("beside", [False, True])
@pytest.mark.parametrize("more", [0, 1 << 20, 64 << 20])
def test_partial_sums_of_shared_launches_stay_in_the_workspace(record, beside, more):
    """Products of a pass, given what the largest of them asks for and some more: partial sums of one launch do not overlap."""
    conv = lambda n, hw, c, k, r: (n, hw, hw, c, hw, hw, k, r, r, 1, r // 2)
    passes = [[conv(4, 14, 256, 256, 3), conv(4, 14, 1024, 256, 1), conv(4, 14, 256, 1024, 1)],
              [conv(5, 90, 64, 64, 3), conv(5, 45, 64, 128, 3), conv(5, 45, 128, 128, 3), conv(5, 90, 8, 64, 3)],
              [conv(n, hw, c, k, r) for n in (1, 8) for hw in (7, 16) for c, k in ((64, 64), (128, 512), (512, 72)) for r in (1, 3)]]
    cases = [dict(shapes=p, pair=False, beside=beside, more=more) for p in passes]
    for case, got in zip(cases, record(cases)):
        _in_turn_or_side_by_side(case, got)


@pytest.mark.parametrize("hidden,steps,samples", [(128, 50, 64), (256, 50, 64), (256, 50, 128), (512, 50, 256), (64, 40, 64), (1024, 50, 64)])
def test_an_lstm_stage_brings_the_workspace_of_its_weight_gradients(hidden, steps, samples):
    sizes = []

    def alloc(nbytes, ctx):
        sizes.append(nbytes)
        return 256 * len(sizes) if len(sizes) <= 5 else None

    b = C._Builder()
    b.lstm(hidden, hidden, src=-1)
    st = C._stage("lstm", b.layers, C.BF16, (hidden, steps, 1), samples, 1, 1, 1, 1, 0, "xavier")
    o = B.make_opts(st)
    o.mem.alloc, o.mem.free = B.ALLOC_FN(alloc), B.FREE_FN(lambda ptr, ctx: None)
    with pytest.raises(B.BapipeError):
        B.bapipe_stage_create(b.layers, samples, 1, o)
    f = getattr(B.load(), "_ZN6bapipe25conv_wgrad_mfma_workspaceERKNS_9ConvShapeE")
    f.restype = ct.c_size_t
    one = f(ct.byref(_ConvShape(samples, steps, 1, hidden, steps, 1, 4 * hidden, 1, 1, 1, 0)))
    assert sizes[4] >= one and (sizes[4] >= 2 * one or 2 * one + 512 > 24 << 20)


if __name__ == "__main__":
    print(json.dumps(_record(sys.argv[1], sys.argv[2], json.load(sys.stdin))))
