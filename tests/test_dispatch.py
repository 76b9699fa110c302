"""Rules of the dispatch that can be asked without a GPU."""
import ctypes as ct

import pytest

from paper_2012_12544_amd import binding as B
from stage_inputs import configs as C


def _lstm_seq_supported(n, hidden, compute_units, steps=50):
    f = getattr(B.load(), "_ZN6bapipe18lstm_seq_supportedEiiii")
    f.restype, f.argtypes = ct.c_bool, [ct.c_int] * 4
    return f(n, steps, hidden, compute_units)


@pytest.mark.parametrize("hidden", [128, 256, 512, 640, 1024])
@pytest.mark.parametrize("units", [0, 8, 32, 64, 128, 256])
def test_one_launch_recurrence_needs_room_for_eight_launches(hidden, units):
    """Blocks of a launch wait for each other.  At one block per compute unit, eight launches that each miss the last
    block of a group must leave a unit free; a partition of fewer units takes two launches per step."""
    blocks_per_group = hidden // 32
    assert _lstm_seq_supported(64, hidden, units) == (8 * (blocks_per_group - 1) < units)


def test_one_launch_recurrence_takes_the_hidden_sizes_it_has_kernels_for():
    assert _lstm_seq_supported(1, 128, 256) and _lstm_seq_supported(512, 1024, 256)
    for n, hidden in ((64, 64), (64, 192), (64, 1152), (528, 1024), (0, 128)):
        assert not _lstm_seq_supported(n, hidden, 256)


@pytest.mark.parametrize("n,hidden,least", [
    (1, 128, 2), (64, 256, 2), (64, 1024, 2),       # a single step has no recurrent product
    (256, 1024, 4), (512, 1024, 8),                 # two and four rounds of the chip, each of which loads the matrix
    (1024, 512, 8), (2048, 256, 4), (4096, 128, 3),
])
def test_one_launch_recurrence_needs_two_steps_a_round(n, hidden, least):
    assert not _lstm_seq_supported(n, hidden, 256, least - 1)
    assert _lstm_seq_supported(n, hidden, 256, least)


class _GatherConv(ct.Structure):
    _fields_ = [(f, ct.c_int) for f in "N Hi Wi Ci Ho Wo Co R S s_out s_in pad_h pad_w beside by_norm wt_panels".split()]


def _pixel_tiles(rows, cin, cout, k=1, hw=1, beside=0):
    """(pixel tiles of the product where K is not split, bytes of partial sums where it is)"""
    lib, g = B.load(), _GatherConv(rows, hw, hw, cin, hw, hw, cout, k, k, 1, 1, k // 2, k // 2, beside)
    chunks = getattr(lib, "_ZN6bapipe28conv_gather_mfma_stat_chunksERKNS_10GatherConvE")
    work = getattr(lib, "_ZN6bapipe26conv_gather_mfma_workspaceERKNS_10GatherConvE")
    work.restype = ct.c_size_t
    return chunks(ct.byref(g)), work(ct.byref(g))


@pytest.mark.parametrize("rows,cin,cout,k,hw,tile", [
    (900, 4096, 4096, 1, 1, 128),     # two blocks of 64 rows per unit would stream 34 MB of weights each
    (600, 6144, 3072, 1, 1, 64),      # one block of 64 rows per unit
    (512, 4096, 4096, 1, 1, 64),
    (3200, 4096, 1024, 1, 1, 64),     # weights that stay in the L2s
    (32, 512, 512, 3, 14, 64),        # a 3x3 filter reads the tile's pixels again
])
def test_pixel_tile_of_products_of_8_to_16_gmac(rows, cin, cout, k, hw, tile):
    assert _pixel_tiles(rows, cin, cout, k, hw) == ((rows * hw * hw + tile - 1) // tile, 0)


@pytest.mark.parametrize("mb,beside,tile", [
    (40, 1, 128), (41, 1, 256),        # 124 and 128 tiles of 256 x 128 beside other streams
    (61, 0, 128), (62, 0, 256),        # 188 and 192 alone on the chip
    (130, 0, 256), (131, 0, 256), (131, 1, 256),        # 400, 404 (from there 256 x 256)
])
def test_pixel_tile_of_few_large_tiles(mb, beside, tile):
    """3x3, 512->512 at 14x14."""
    assert _pixel_tiles(mb, 512, 512, 3, 14, beside) == ((mb * 196 + tile - 1) // tile, 0)


@pytest.mark.parametrize("rows,cin,cout,tile", [
    (1024, 512, 256, 32),      # 256 tiles of 32 x 32
    (1024, 504, 256, 64),      # K too short for them
    (2048, 512, 256, 32),      # 512 of them, 256 of 32 x 64
    (2049, 512, 256, 64),      # 260
    (100352, 64, 64, 128),     # up to 64 channels: 128 x 64
    (100352, 64, 72, 64),
])
def test_pixel_tile_of_few_small_tiles(rows, cin, cout, tile):
    assert _pixel_tiles(rows, cin, cout) == ((rows + tile - 1) // tile, 0)


@pytest.mark.parametrize("rows,splits", [(32, 2), (33, 4), (64, 4), (65, 8)])
def test_splits_of_a_large_matrix_for_few_rows(rows, splits):
    """Two rows of 32 x 32 tiles would fetch it twice, so 33 to 64 rows are one of 64 x 64; above, no groups of waves."""
    assert _pixel_tiles(rows, 25088, 4096) == (0, splits * rows * 4096 * 4)


def test_large_weights_are_not_streamed_by_more_rows_of_tiles_than_before():
    assert _pixel_tiles(128, 25088, 4096) == (0, 16 * 128 * 4096 * 4)


@pytest.mark.parametrize("c,hw,least,beside_norm", [
    (64, 32, 32, 128), (128, 32, 16, 64), (256, 16, 32, 128),       # whole patches: blocks of 64 channels x 256 pixels
    (64, 90, 5, None), (128, 28, 38, None),                          # patches cut at the border: more than 160 and 300 of them
])
def test_3x3_layers_take_patches_from_so_many_samples_on(c, hw, least, beside_norm):
    """Next to a batch-norm, whose sums the gather kernel leaves, later or not at all."""
    f = getattr(B.load(), "_ZN6bapipe22conv3x3_halo_supportedERKNS_10GatherConvE")
    f.restype = ct.c_bool
    takes = lambda n, by_norm: f(ct.byref(_GatherConv(n, hw, hw, c, hw, hw, c, 3, 3, 1, 1, 1, 1, 0, by_norm)))
    for by_norm, n in ((0, least), (1, beside_norm)):
        if n is None:
            assert not takes(1 << 10, by_norm)
        else:
            assert takes(n, by_norm) and not takes(n - 1, by_norm)


# ------------------------------------------------------------------------------ workspace of the deferred weight gradients
class _ConvShape(ct.Structure):
    _fields_ = [(f, ct.c_int) for f in "N H W C P Q K R S stride pad".split()]


def _wgrad_workspace(rows, cin, cout):
    f = getattr(B.load(), "_ZN6bapipe25conv_wgrad_mfma_workspaceERKNS_9ConvShapeE")
    f.restype = ct.c_size_t
    return f(ct.byref(_ConvShape(rows, 1, 1, cin, 1, 1, cout, 1, 1, 1, 0)))


def _blocks_of_a_linear_stage(cin, cout, micro_batch, n_micro):
    """Sizes a stage of one linear layer asks its allocator for: parameters, stash, transient, gradients, workspace.  The next
    request is refused, so that nothing reaches a device."""
    sizes = []

    def alloc(nbytes, ctx):
        sizes.append(nbytes)
        return 256 * len(sizes) if len(sizes) <= 5 else None

    b = C._Builder()
    b.linear(cin, cout, src=-1)
    st = C._stage("linear", b.layers, C.BF16, (cin, 1, 1), micro_batch, n_micro, 1, 1, 1, 0, "kaiming")
    o = B.make_opts(st)
    o.mem.alloc, o.mem.free = B.ALLOC_FN(alloc), B.FREE_FN(lambda ptr, ctx: None)
    with pytest.raises(B.BapipeError) as e:
        B.bapipe_stage_create(b.layers, micro_batch, n_micro, o)
    assert e.value.status == B.E_OOM
    return sizes[:5]


@pytest.mark.parametrize("cin,cout,micro_batch,n_micro", [
    (128, 1000, 100, 16),          # 13 micro-batches want more partial sums than 16
    (256, 512, 100, 16), (256, 256, 128, 16), (512, 512, 96, 24), (64, 64, 50, 40), (1024, 1000, 64, 16), (4096, 4096, 100, 40),
])
def test_workspace_holds_the_weight_gradient_of_any_part_of_a_mini_batch(cin, cout, micro_batch, n_micro):
    """Reading the gradients in the middle of a mini-batch runs the deferred product over the micro-batches so far, the update
    runs it over the rest."""
    have = _blocks_of_a_linear_stage(cin, cout, micro_batch, n_micro)[4]
    assert have >= max(_wgrad_workspace(micro_batch * n, cin, cout) for n in range(1, n_micro + 1))
