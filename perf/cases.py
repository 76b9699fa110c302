"""What a user has the stage engine do: mini-batches of one pipeline stage, through the C ABI's binding.

One pass is one mini-batch as a pipeline worker runs it: M forward and M backward passes in 1F1B order (warm-up
forwards, one backward and one forward in turn, drain), then the weight update.  What comes back: the stage's output
of every micro-batch, the gradient handed to the previous stage (where the stage has one), the accumulated gradients
as they stand before the update, and the updated master weights.

The stages are the slices of the networks that this repository is configured for (stage_inputs/configs.py), cut so
that a mini-batch can be compared between two correct implementations: every ReLU and max-pool takes a decision on a
bf16 value, two orders of summation disagree about a few of those decisions, and each one that flips moves the
gradients upstream of it.  Over the ten bottlenecks of the full residual stage that is 47 % of the input gradient
(2-norm), over the six convolutions of the deep VGG stage 10 %, over one bottleneck or three convolutions 1 to 2 %,
so the residual stage appears as its single bottlenecks and the deep stage as its two halves, at their full sizes.
For the same reason the weights are what a bf16 checkpoint holds (masters on bf16 values: an update of LR does not push
them over a rounding boundary in one implementation and not in the other), and weights and upstream gradients are
uniform (no single flipped gate outweighs the rest of an element's sum).
"""
import math

import torch

from paper_2012_12544_amd import binding as B
from stage_inputs import configs as C

LR = 2e-5


# ---------------------------------------------------------------------------------------------- the stages
def _identity_bottleneck(channels, mid, hw, micro_batch, n_micro):
    """One bottleneck whose shortcut is its input: the second block of a residual group, as a stage of its own.  The
    layers below are frozen, so nothing is handed back: behind an identity shortcut a flipped output gate would be the
    whole of a dx element."""
    two = C.resnet50_stage(cin=channels, mid3=mid, hw=2 * hw, n3=2, n4=0, micro_batch=micro_batch, n_micro=n_micro)
    first = 1 + [L["kind"] for L in two["layers"]].index(C.ADD)
    layers = [dict(L, src0=max(L["src0"] - first, -1), src1=max(L["src1"] - first, -1)) for L in two["layers"][first:]]
    return dict(two, layers=layers, in_c=4 * mid, in_h=hw, in_w=hw, need_input_grad=0)


def _stage(case):
    """The workload description (stage_inputs/configs.py) of a case."""
    mb, M, c, hw = case["micro_batch"], case["n_micro"], case["width"], case["hw"]
    k = case["kind"]
    if k == "tiny":
        st = C.tiny_stage(c=c, hw=hw, micro_batch=mb, n_micro=M)
    elif k == "vgg_stage1":
        st = C.vgg16_stage1(c1=c, c2=2 * c, hw=hw, micro_batch=mb, n_micro=M)
    elif k == "vgg_block":
        st = C.vgg16_conv3(cin=case["cin"], c=c, hw=hw, micro_batch=mb, n_micro=M)
    elif k == "classifier":
        st = C.vgg16_classifier(c=case["cin"], hw=hw, hidden=c, micro_batch=mb, n_micro=M)
    elif k == "projection":
        st = C.resnet50_stage(cin=case["cin"], mid3=c, hw=hw, n3=1, n4=0, micro_batch=mb, n_micro=M)
    elif k == "identity":
        st = _identity_bottleneck(4 * c, c, hw, mb, M)
    elif k == "stem":
        st = C.resnet50_stem(c=c, hw=hw, n2=1, micro_batch=mb, n_micro=M)
    elif k == "tail":
        st = C.resnet50_tail(cin=case["cin"], mid=c, hw=hw, n5=1, micro_batch=mb, n_micro=M)
    elif k == "lstm":
        st = C.gnmt_lstm_stage(hidden=c, seq=hw, micro_batch=mb, n_micro=M)
    else:
        raise ValueError(k)
    # the stage's place in the pipeline: N-i+1 micro-batches are in flight
    return dict(st, stage_index=9 - case["in_flight"], n_stages=8)


def _case(name, kind, width, hw, micro_batch, n_micro, in_flight, cin=0, streams=3, layout="NHWC"):
    return dict(name=name, kind=kind, width=width, hw=hw, cin=cin, micro_batch=micro_batch, n_micro=n_micro,
                in_flight=in_flight, streams=streams, layout=layout)


def listed():
    return [
        # the smallest stage the repository is configured for, in float: launches and latency
        _case("tiny fp32", "tiny", 16, 32, 4, 4, 2, streams=1, layout="NCHW"),
        # VGG-16 stage 1 of four, the benchmark's headline workload
        _case("vgg stage 1", "vgg_stage1", 64, 224, 32, 8, 4),
        # the same layers on ragged images in small micro-batches, from a neighbour that sends NCHW
        _case("vgg stage 1 ragged", "vgg_stage1", 64, 90, 5, 3, 2, streams=1, layout="NCHW"),
        # the halves of the deep VGG stage: conv4_1..4_3 + pool, conv5_1..5_3 + pool (the first: the largest product)
        _case("vgg conv4", "vgg_block", 512, 28, 64, 8, 2, cin=256),
        _case("vgg conv5", "vgg_block", 512, 14, 64, 8, 2, cin=512),
        # the end of VGG-16: three linear layers and the loss, one micro-batch in flight, weights dominate
        _case("vgg classifier", "classifier", 4096, 7, 64, 16, 1, cin=512, streams=1),
        # bottlenecks of the residual stage: the first of conv3_x (stride 2, projection), one of conv4_x (identity)
        _case("resnet conv3 first", "projection", 128, 56, 32, 8, 3, cin=256),
        _case("resnet conv4 block", "identity", 256, 14, 32, 8, 3),
        # the same identity block fed four samples at a time: a deep pipeline's fine split, launches count
        _case("resnet conv4 small", "identity", 256, 14, 4, 8, 4, streams=1),
        # the head of ResNet-50 (7x7 conv, overlapping max-pool) and its end (conv5_x, average pool, loss)
        _case("resnet stem", "stem", 64, 224, 32, 8, 4),
        _case("resnet tail", "tail", 512, 14, 32, 8, 1, cin=1024, streams=1),
        # two LSTM layers of GNMT: 50 dependent steps per layer and direction
        _case("gnmt lstm", "lstm", 1024, 50, 64, 8, 3),
    ]


# ranges that the listed cases stand for: kind -> widths, map sizes, micro-batch range, input widths per width
_RANGES = {
    "tiny": ([8, 12, 16, 24, 32], (16, 64), (1, 16), None),
    "vgg_stage1": ([32, 48, 64], (32, 224), (1, 32), None),
    "vgg_block": ([128, 192, 256, 320, 512], (8, 56), (2, 64), (0.5, 1)),
    "classifier": ([1024, 2048, 4096], (3, 7), (1, 64), (0.125,)),
    "projection": ([64, 96, 128, 256], (14, 56), (2, 32), (2, 4)),
    "identity": ([64, 96, 128, 256], (7, 28), (2, 32), None),
    "stem": ([32, 64], (64, 224), (1, 32), None),
    "tail": ([256, 384, 512], (8, 14), (4, 32), (2,)),
    "lstm": ([256, 512, 1024], (2, 50), (1, 64), None),
}


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    # no dearer than the largest listed case: by its arithmetic here, by the size of its feature maps and the number of
    # dependent steps through the ranges
    most = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(sorted(_RANGES))
        widths, (hlo, hhi), (blo, bhi), ratio = _RANGES[kind]
        width = rng.choice(widths)
        case = dict(kind=kind, width=width, hw=_log_int(rng, hlo, hhi), cin=int(width * rng.choice(ratio)) if ratio else 0,
                    micro_batch=_log_int(rng, blo, bhi), n_micro=rng.randint(1, 8), in_flight=rng.randint(1, 4),
                    streams=rng.choice([1, 3]), layout=rng.choice(["NHWC", "NHWC", "NCHW"]))
        if work(case)["flops"] <= most:
            return case


# ---------------------------------------------------------------------------------------------- inputs
_side = []


def _side_streams():
    """The program's two further streams (backward passes, weight gradients): one pair, whatever stages it runs."""
    if not _side:
        _side.extend(torch.cuda.Stream() for _ in range(2))
    return _side


def _uniform(shape, bound, g):
    return (torch.rand(shape, device="cuda", generator=g) * 2 - 1) * bound


def _parameters(stage, g):
    """(w, b) per layer, on the GPU: Kaiming- / Xavier-uniform, gamma 1, biases and beta 0."""
    out = []
    for L in stage["layers"]:
        w = b = None
        if L["kind"] == C.CONV2D:
            w = _uniform((L["cout"], L["cin"], L["kh"], L["kw"]), math.sqrt(6.0 / (L["cin"] * L["kh"] * L["kw"])), g)
            if L["has_bias"]:
                b = torch.zeros(L["cout"], device="cuda")
        elif L["kind"] == C.LINEAR:
            w = _uniform((L["cout"], L["cin"]), math.sqrt(6.0 / (L["cin"] + L["cout"])), g)
            b = torch.zeros(L["cout"], device="cuda")
        elif L["kind"] == C.LSTM:
            w = _uniform((4 * L["cout"], L["cin"] + L["cout"]), 1.0 / math.sqrt(L["cout"]), g)
            b = torch.zeros(4 * L["cout"], device="cuda")
        elif L["kind"] == C.BATCHNORM2D:
            w, b = torch.ones(L["cout"], device="cuda"), torch.zeros(L["cout"], device="cuda")
        if w is not None and stage["dtype"] == C.BF16:
            w = w.bfloat16().float()
        out.append((w, b))
    return out


def _ends_in_loss(stage):
    return stage["layers"][-1]["kind"] == C.SOFTMAX_XENT


def _order(M, depth):
    """1F1B: `depth` forwards, one backward and one forward in turn, drain."""
    W = min(M, depth)
    order = [("F", m) for m in range(W)]
    for m in range(M - W):
        order += [("B", m), ("F", m + W)]
    return order + [("B", m) for m in range(M - W, M)]


class _Program:
    """What a worker holds: the stage's handle, the tensors its neighbours fill and read, and the memory it gave the stage."""

    def __init__(self, case, seed):
        self.handle = None
        stage = _stage(case)
        g = torch.Generator("cuda")
        g.manual_seed(int(seed))
        bf16 = stage["dtype"] == C.BF16
        dtype = torch.bfloat16 if bf16 else torch.float32
        nhwc = case["layout"] == "NHWC"
        self.M, mb = stage["n_micro"], stage["micro_batch"]
        shapes = C.infer_shapes(stage)
        oc, oh, ow = shapes[-1]

        def io(c, h, w):
            return (mb, h, w, c) if nhwc else (mb, c, h, w)

        # N(0,1) activations; upstream gradients with the size a mean over samples and positions gives them
        self.x = [torch.randn(io(stage["in_c"], stage["in_h"], stage["in_w"]), device="cuda", generator=g).to(dtype) for _ in range(self.M)]
        self.loss = _ends_in_loss(stage)
        if self.loss:
            self.g = [torch.randint(0, oc, (mb,), device="cuda", generator=g, dtype=torch.int32) for _ in range(self.M)]
        else:
            self.g = [_uniform(io(oc, oh, ow), math.sqrt(3.0) / (mb * self.M * oh * ow), g).to(dtype) for _ in range(self.M)]
        out_shape = io(oc, oh, ow)
        self.y = torch.zeros((self.M,) + out_shape, device="cuda", dtype=torch.float32 if self.loss else dtype)
        self.dx = torch.zeros((self.M,) + tuple(self.x[0].shape), device="cuda", dtype=dtype) if stage["need_input_grad"] else None

        self.memory = B.TorchAllocator("cuda:0")
        opts = B.make_opts(stage, io_layout=B.NHWC if nhwc else B.NCHW, stream=torch.cuda.current_stream().cuda_stream,
                           allocator=self.memory)
        self.handle = B.bapipe_stage_create(stage["layers"], mb, self.M, opts)
        ptr, block = next(iter(self.memory.live.items()))
        # The first block the stage asks for holds its parameters: the float masters of all layers in order, every
        # vector padded to 256 bytes, then the gradient accumulators in the same order.  (The first convolution of
        # a bf16 stage reads its image padded to a multiple of 8 channels.)
        nbytes = 0
        for i, (L, (w, b)) in enumerate(zip(stage["layers"], _parameters(stage, g))):
            if w is None:
                continue
            B.bapipe_stage_set_params(self.handle, i, w.cpu().numpy(), None if b is None else b.cpu().numpy())
            n = w.numel()
            if bf16 and L["kind"] == C.CONV2D and L["src0"] < 0:
                n = n // L["cin"] * ((L["cin"] + 7) // 8 * 8)
            nbytes += sum((4 * k + 255) // 256 * 256 for k in (n, 0 if b is None else b.numel()))
        at = ptr - block.data_ptr()
        self.weights = block[at:at + nbytes].view(torch.float32)
        self.accumulators = block[at + nbytes:at + 2 * nbytes].view(torch.float32)
        self.gradients = torch.zeros_like(self.accumulators)

        self.order = _order(self.M, B.bapipe_stage_stash_bytes(self.handle)[1])
        self.backward_stream = None
        if case["streams"] == 3:
            self.backward_stream, wgrad_stream = _side_streams()
            B.bapipe_stage_set_streams(self.handle, self.backward_stream.cuda_stream, wgrad_stream.cuda_stream)

    def __del__(self):
        if self.handle is not None:
            B.bapipe_stage_destroy(self.handle)
            self.handle = None


def prepare(case, seed):
    return _Program(case, seed)


def run(p):
    for what, m in p.order:
        if what == "F":
            B.bapipe_stage_forward(p.handle, m, p.x[m].data_ptr(), p.y[m].data_ptr())
        else:
            B.bapipe_stage_backward(p.handle, m, p.g[m].data_ptr(), None if p.dx is None else p.dx[m].data_ptr())
    if p.backward_stream is not None:
        torch.cuda.current_stream().wait_stream(p.backward_stream)
    p.gradients.copy_(p.accumulators)      # the update clears them
    B.bapipe_stage_step(p.handle, LR)
    out = {"y": p.y, "gradients": p.gradients, "weights": p.weights}
    if p.dx is not None:
        out["dx"] = p.dx
    return out


# ---------------------------------------------------------------------------------------------- work and tolerance
def work(case):
    """The mini-batch's multiply-adds (forward, input gradient, weight gradient of every conv / linear / LSTM layer) and
    the boundary tensors and parameters, each once: x, y, dy, dx; masters read and written, gradients written."""
    stage = _stage(case)
    es = 2 if stage["dtype"] == C.BF16 else 4
    samples = stage["micro_batch"] * stage["n_micro"]
    oc, oh, ow = C.infer_shapes(stage)[-1]
    x = samples * stage["in_c"] * stage["in_h"] * stage["in_w"] * es
    y = samples * oc * oh * ow * (4 if _ends_in_loss(stage) else es)
    dy = samples * 4 if _ends_in_loss(stage) else y
    params = 0
    for L in stage["layers"]:
        if L["kind"] == C.CONV2D:
            params += L["cout"] * L["cin"] * L["kh"] * L["kw"]
        elif L["kind"] == C.LINEAR:
            params += L["cout"] * L["cin"]
        elif L["kind"] == C.LSTM:
            params += 4 * L["cout"] * (L["cin"] + L["cout"])
    return {"bytes": x + y + dy + (x if stage["need_input_grad"] else 0) + 12 * params, "flops": C.flops_per_minibatch(stage)}


def tolerance(case):
    """Measured by running each stage a second time with the channels of every tensor permuted (the same sums in another
    order), over the listed cases and drawn ones, first and second mini-batch: the relative 2-norm of the difference, the
    worst of y, dx and the accumulated gradients, was

        tiny 3e-7;  vgg_stage1 6.5e-3;  vgg_block 2.1e-2;  classifier 3.8e-3;  projection 5e-3 (2.6e-2 at the smallest sizes);
        identity 1.3e-2;  stem 7e-3 (1.4e-2);  tail 1.6e-2;  lstm 1.2e-3

    and single elements of dx behind a flipped decision were off by up to 0.7 of their size (of the root mean square
    where that is larger); 0.17 in the classifier, 0.02 in the LSTM."""
    if case["kind"] == "tiny":
        return {"rel": 1e-5, "max": 1e-3}
    rel = {"vgg_stage1": 0.026, "classifier": 0.015, "lstm": 0.005}
    return {"rel": rel.get(case["kind"], 0.03), "max": {"classifier": 0.7, "lstm": 0.1}.get(case["kind"], 0.99)}
