"""GPU parity at the sizes where a kernel's work split changes: edges of tiles, passes and parts, remainders, the smallest
and largest of a range.  Integer and binary layers bit-exact, bf16 within the bound of the other parity tests."""
import pytest
import torch

import rrm_synth as S
from gpu_util import run_sequence

pytestmark = pytest.mark.gpu


# One channel block and 1, 2, 4 or 8 sub-tiles per workgroup (a layer of few sub-tiles): the consumers split the K steps, of
# layers of few K steps in the dense launch only (the delta launch then has eight).
# (map, c_in, c_out, k, stride, pad, groups, n): K steps fewer than the parts, one slab and several, channel counts off
# the blocks of 32 and off the fours, groups, several units per workgroup.
FEW_SUBTILES = [
    (4, 16, 16, 1, 1, 0, 1, 1), (13, 384, 384, 3, 1, 1, 1, 1), (13, 256, 384, 3, 1, 1, 1, 2), (27, 96, 256, 5, 1, 2, 2, 1),
    (20, 48, 130, 3, 1, 1, 1, 1), (29, 32, 33, 3, 2, 1, 1, 2), (55, 16, 64, 3, 1, 1, 1, 1), (7, 512, 512, 3, 1, 1, 1, 1),
    (31, 16, 7, 3, 1, 1, 1, 9), (40, 16, 32, 5, 1, 2, 1, 10), (20, 112, 130, 3, 1, 1, 1, 1), (29, 128, 33, 3, 2, 1, 1, 2),
]


@pytest.mark.parametrize("shp", FEW_SUBTILES)
@pytest.mark.parametrize("dt", [S.I8, S.BF16])
def test_window_tile_kernel_with_few_subtiles(shp, dt):
    m, ci, co, k, st, pad, g, n = shp
    seq = S.random_layer(9100 + m, S.conv_shape(m, m, ci, co, k, st, pad, g, n=n), dt, T=4, frac=0.2, block=3)
    run_sequence(seq, check_dense=(0, 3), path=1, conv_kernel=1)


# int8 layers whose windows leave room for 12 slots and not for 16, with more sub-tiles than one pass of eight over the grid:
# six of the eight consumers have a pair.  (map, c_in, c_out, k, stride, pad, groups, n): one slab of K and several (the last
# one short), channel runs off 16 bytes, channel counts off the blocks of 32 and off the fours, groups, units of an odd
# number of sub-tiles, one unit per workgroup and several.
TWELVE_SLOTS = [
    (27, 96, 256, 5, 1, 2, 2, 13), (27, 96, 256, 5, 1, 2, 2, 22), (32, 128, 70, 2, 2, 0, 1, 66), (33, 80, 96, 2, 2, 0, 1, 66),
    (56, 16, 128, 4, 4, 0, 1, 66), (33, 48, 66, 3, 2, 1, 1, 42), (33, 40, 130, 5, 1, 2, 1, 9), (33, 32, 96, 6, 1, 2, 1, 17),
    (30, 16, 96, 9, 1, 4, 1, 17),
]


@pytest.mark.parametrize("shp", TWELVE_SLOTS)
def test_window_tile_kernel_with_twelve_slots(shp):
    m, ci, co, k, st, pad, g, n = shp
    seq = S.random_layer(9500 + m + n, S.conv_shape(m, m, ci, co, k, st, pad, g, n=n), S.I8, T=4, frac=0.2, block=3)
    run_sequence(seq, check_dense=(0, 3), path=1, conv_kernel=1)
    run_sequence(seq, check_dense=(), check_frames=(3,), dense_switch_pct=1, conv_kernel=1)


# The binary band kernel: 64 output channels per workgroup in two blocks of 32, passes of 64 listed positions in two tiles
# of 32, K steps of two words in four parts for each tile, a few in flight at a time.
@pytest.mark.parametrize("ci,co,k,m,n,frac", [
    (32, 1, 1, 5, 1, 0.5), (128, 31, 3, 8, 1, 0.3), (128, 32, 3, 8, 2, 0.6), (128, 33, 3, 9, 1, 0.95), (256, 64, 3, 12, 3, 0.1),
    (256, 65, 1, 16, 1, 0.95), (512, 130, 3, 7, 2, 0.2), (128, 96, 5, 17, 1, 0.9), (640, 48, 3, 10, 1, 0.4), (96, 20, 3, 11, 2, 0.3),
])
def test_binary_band_kernel_edges(ci, co, k, m, n, frac):
    seq = S.random_layer(9200 + ci + co, S.conv_shape(m, m + 1, ci, co, k, 1, k // 2, 1, n=n), S.BIN, T=4, frac=frac, block=2)
    run_sequence(seq, check_dense=(0, 3))
    run_sequence(seq, check_dense=(), bin_single_launch=0)


# Forms of the band kernel: bands of a tile or less and of several, one workgroup per compute unit and more; K steps of a wavefront
# fewer than, equal to and beyond the weights in its registers, one block of 32 channels and two; the dense layer with a tile per
# wavefront, with one per wavefront and block, with two tiles per wavefront; filters wider than a word of flags; a step with taller
# bands than the dense launch (fewer than 32 K steps) and not.
@pytest.mark.parametrize("h,w,ci,co,k,st,pad,g,n,frac", [
    (14, 14, 512, 130, 3, 1, 1, 1, 1, 0.3), (5, 7, 128, 40, 3, 1, 1, 1, 1, 0.9), (11, 40, 32, 20, 3, 1, 1, 1, 1, 0.2), (12, 12, 128, 96, 3, 1, 1, 1, 130, 0.2),
    (9, 9, 256, 65, 3, 2, 1, 1, 150, 0.5), (20, 20, 64, 34, 5, 1, 2, 2, 12, 0.3), (24, 30, 128, 30, 3, 1, 1, 1, 90, 0.1), (40, 13, 640, 64, 1, 1, 0, 1, 5, 0.4),
    (36, 39, 32, 8, 33, 1, 2, 1, 1, 0.02), (16, 16, 384, 70, 3, 1, 1, 1, 140, 0.05),
    (20, 9, 128, 70, 4, 1, 1, 1, 2, 0.1), (20, 9, 96, 70, 5, 1, 2, 1, 2, 0.1), (28, 28, 256, 80, 1, 1, 0, 1, 2, 0.1),
])
def test_binary_band_kernel_forms(h, w, ci, co, k, st, pad, g, n, frac):
    seq = S.random_layer(9250 + h + ci + co, S.conv_shape(h, w, ci, co, k, st, pad, g, n=n), S.BIN, T=3, frac=frac, block=2)
    run_sequence(seq, check_dense=(0, 2), check_frames=(0, 2))


# Lists that every wavefront makes for itself (bands of up to 64 outputs: one, a tile, a tile and more, 64) and not (65); blocks of 32
# channels (few workgroups: channels below, at, off and beyond them, an odd count of them, groups), in the step and the dense launch;
# wavefronts of more than 64 K steps, whose places come in turns (words of 2048 and of 4096 channels).
@pytest.mark.parametrize("h,w,ci,co,k,st,pad,g,n,frac", [
    (1, 1, 128, 7, 1, 1, 0, 1, 1, 1.0), (4, 8, 256, 32, 3, 1, 1, 1, 1, 0.5), (6, 16, 128, 33, 3, 1, 1, 1, 2, 0.5), (4, 64, 128, 64, 3, 1, 1, 1, 1, 0.3),
    (4, 65, 128, 65, 3, 1, 1, 1, 1, 0.3), (14, 14, 256, 96, 3, 1, 1, 2, 1, 0.3), (14, 13, 512, 160, 3, 1, 1, 1, 1, 0.4), (9, 9, 256, 31, 3, 2, 1, 1, 3, 0.5),
    (4, 7, 2048, 40, 3, 1, 1, 1, 1, 0.5), (2, 4, 4096, 33, 3, 1, 1, 1, 1, 0.6), (6, 40, 2048, 70, 3, 1, 1, 1, 2, 0.3),
])
def test_binary_bands_of_short_lists_and_narrow_blocks(h, w, ci, co, k, st, pad, g, n, frac):
    seq = S.random_layer(9450 + h + w + co, S.conv_shape(h, w, ci, co, k, st, pad, g, n=n), S.BIN, T=3, frac=frac, block=2)
    run_sequence(seq, check_dense=(0, 2))
    run_sequence(seq, check_dense=(), check_frames=(2,), bin_single_launch=0)


# A band fewer where bands make a few workgroups over two per compute unit: in the step and the dense launch, in one of them (many
# bands; one band left), with strides and words off the 16-byte vectors (two launches).
@pytest.mark.parametrize("h,w,ci,co,k,st,pad,g,n,frac", [
    (12, 7, 128, 8, 3, 1, 1, 1, 180, 0.1), (20, 5, 32, 8, 3, 1, 1, 1, 110, 0.1), (8, 9, 128, 5, 3, 1, 1, 1, 350, 0.1),
    (23, 9, 128, 66, 3, 2, 1, 1, 88, 0.2), (13, 6, 96, 8, 5, 1, 2, 1, 176, 0.1), (14, 5, 256, 18, 3, 1, 1, 2, 65, 0.2),
])
def test_binary_bands_over_two_workgroups_per_compute_unit(h, w, ci, co, k, st, pad, g, n, frac):
    seq = S.random_layer(9350 + h + w + n, S.conv_shape(h, w, ci, co, k, st, pad, g, n=n), S.BIN, T=3, frac=frac, block=2)
    run_sequence(seq, check_dense=(0, 2), check_frames=(0, 2))


# Wide binary layers: one output row fits LDS only without the padding of the staged positions.  (h, w, c_in, c_out, k,
# stride, pad, groups, n): one row and several per band, whole 16-byte vectors and not, columns that no window reads
# (difference kernel in front), several channel blocks, groups; the dense layer takes the tile kernel.
@pytest.mark.parametrize("h,w,ci,co,k,st,pad,g,n,frac", [
    (2, 350, 128, 33, 3, 1, 1, 1, 2, 0.1), (4, 365, 128, 64, 3, 1, 1, 1, 1, 0.6), (3, 345, 64, 70, 3, 1, 1, 1, 1, 0.3),
    (4, 340, 128, 16, 3, 1, 1, 1, 140, 0.05), (2, 1100, 128, 5, 1, 1, 0, 1, 3, 0.2), (3, 1100, 128, 8, 1, 2, 0, 1, 1, 0.2),
    (2, 470, 512, 65, 1, 1, 0, 1, 1, 0.9), (2, 350, 256, 24, 3, 1, 1, 2, 2, 0.1),
])
def test_binary_wide_layer_on_bands(h, w, ci, co, k, st, pad, g, n, frac):
    seq = S.random_layer(9300 + w + co, S.conv_shape(h, w, ci, co, k, st, pad, g, n=n), S.BIN, T=4, frac=frac, block=2)
    stats, _ = run_sequence(seq, check_dense=(0, 3))
    assert stats["tile_positions"] == 1  # (listed positions: the band kernel)
    run_sequence(seq, check_dense=(), bin_single_launch=0)


# The dense launch of 1 x 1 binary layers: on tiles up to 256 channels a group, on bands above and where these fill the chip and
# the map leaves its tiles empty.  (h, w, c_in, c_out, stride, groups, n): words off the 16-byte vectors, maps off the tiles.
@pytest.mark.parametrize("h,w,ci,co,st,g,n", [
    (1, 1, 32, 1, 1, 1, 1), (9, 17, 96, 33, 1, 1, 2), (13, 13, 128, 65, 2, 1, 1), (16, 24, 256, 70, 1, 1, 3), (7, 9, 288, 16, 1, 1, 2),
    (9, 8, 512, 24, 1, 2, 2), (13, 13, 128, 8, 1, 1, 172), (12, 13, 256, 5, 1, 1, 171), (13, 13, 96, 8, 1, 1, 172),
])
def test_binary_dense_layer_of_1x1_filters(h, w, ci, co, st, g, n):
    seq = S.random_layer(9600 + w + co + n, S.conv_shape(h, w, ci, co, 1, st, 0, g, n=n), S.BIN, T=3, frac=0.2, block=2)
    run_sequence(seq, check_dense=(0, 2), check_frames=(0, 2))


# The FC step fills the caller's copy itself where every output has one owner, and by a copy otherwise; rows off the 16-byte
# units (also the last bytes of the array); frame 2 repeats frame 1.
@pytest.mark.parametrize("ci,co,n", [(64, 5, 1), (300, 33, 2), (301, 7, 3), (2049, 40, 2), (4096, 64, 1), (9216, 48, 1), (8192, 16, 3)])
@pytest.mark.parametrize("dt", [S.I8, S.BF16])
def test_fc_step_fills_the_callers_copy(ci, co, n, dt):
    seq = S.random_layer(9400 + ci, S.fc_shape(ci, co, n=n), dt, T=4, frac=0.2)
    seq.frames[2] = seq.frames[1].copy()
    run_sequence(seq, check_dense=(0,), y_out_frames=(0, 1, 2, 3), fc_batched=0)


# Compare rounds of the FC step: int8 rows around 8192 inputs (two workgroups on a list from there), bf16 rows around 4096 and,
# of the larger form, 5632 and 11264; rows off the 16-byte units; channels off the 64 bytes of a workgroup; int8 differences of nine bits;
# and more streams than leave a bf16 workgroup a compute unit of its own.
@pytest.mark.parametrize("ci,co,n", [(4097, 40, 1), (7160, 5, 2), (7169, 72, 1), (8191, 64, 1), (8193, 100, 2), (14337, 33, 1), (16385, 20, 1), (5000, 2100, 5)])
@pytest.mark.parametrize("dt", [S.I8, S.BF16])
def test_fc_step_compare_rounds(ci, co, n, dt):
    seq = S.random_layer(9900 + ci, S.fc_shape(ci, co, n=n), dt, T=3, frac=0.4)
    if dt == S.I8:  # the last entries: from the lowest value to the highest and back
        for t, frame in enumerate(seq.frames):
            frame[..., -40:] = (-128, 127)[t % 2]
    run_sequence(seq, check_dense=(), fc_batched=0)


# Rounds of two units per thread (int8 up to 12288 entries, bf16 of the larger form up to 11264) and their neighbours: the second
# unit's first and last thread, a second round of one unit, two full rounds, ragged rows.  One workgroup per
# compute unit (the wavefront that announces it) and more (many channels and streams: thread 0 does; int8 up to 8192 entries in a form of
# one unit).
@pytest.mark.parametrize("ci,co,n", [
    (8192, 64, 1), (8208, 48, 1), (12288, 64, 2), (12304, 32, 1), (24576, 32, 1), (4096, 64, 1), (4104, 32, 2), (5632, 32, 1), (5640, 64, 1),
    (11264, 32, 1), (11272, 32, 1), (9217, 32, 1), (12289, 16, 2), (9216, 8256, 3), (4112, 208, 70), (8192, 208, 70), (8208, 208, 70),
])
@pytest.mark.parametrize("dt", [S.I8, S.BF16])
def test_fc_step_rounds_of_two_units(ci, co, n, dt):
    seq = S.random_layer(9990 + ci, S.fc_shape(ci, co, n=n), dt, T=3, frac=0.3)
    st, _ = run_sequence(seq, check_dense=(), y_out_frames=(1, 2), fc_batched=0)
    import numpy as np
    before = [np.zeros_like(seq.frames[0])] + list(seq.frames[:-1])
    assert st["changed_elems"] == sum(int((a != b).sum()) for a, b in zip(before, seq.frames)) and st["delta_steps"] == 3


# Ragged rows, read and committed 16 bytes at a time at any alignment: arrays of fewer than 16 bytes, of 16 and just over (the
# array's last unit is read from its last 16 bytes), rows one entry off whole units, many streams (a row's last unit beside the next
# row's first), second units of a thread that end with the row.
@pytest.mark.parametrize("ci,co,n", [
    (1, 3, 1), (3, 5, 2), (7, 16, 1), (5, 4, 3), (9, 8, 1), (15, 20, 1), (17, 20, 1), (25, 9, 7), (127, 33, 15), (4103, 20, 3), (8195, 24, 2), (5633, 40, 2),
    (11263, 16, 1), (12287, 33, 2),
])
@pytest.mark.parametrize("dt", [S.I8, S.BF16])
def test_fc_step_of_ragged_rows(ci, co, n, dt):
    import numpy as np
    from gpu_util import make_layer, to_device, x_bytes
    seq = S.random_layer(9940 + ci, S.fc_shape(ci, co, n=n), dt, T=4, frac=0.5)
    run_sequence(seq, check_dense=(), fc_batched=0)
    layer = make_layer(seq, fc_batched=0)
    for t, x in enumerate(seq.frames):
        layer.step(to_device(x, dt))
        assert np.array_equal(layer.x_snapshot_bytes().cpu().numpy(), x_bytes(x, dt)), f"stored input after frame {t}"
    layer.destroy()


# Channel runs that are not whole units: a unit of x within one run, across two (of a position's groups, of two positions), a run
# of just over a unit and of a unit less than two, runs shorter than a unit, arrays of fewer than 16 bytes, the array's last unit cut
# short.  Changes come and go, so that the padded differences are written and wiped; the dense launch re-lays the whole frame.
@pytest.mark.parametrize("h,w,ci,co,k,g,n", [
    (1, 1, 5, 4, 1, 1, 1), (1, 2, 3, 8, 1, 1, 1), (5, 7, 17, 8, 3, 1, 1), (9, 6, 31, 16, 3, 1, 2), (4, 5, 100, 33, 3, 1, 3), (7, 5, 154, 20, 5, 2, 2),
    (3, 3, 66, 12, 3, 3, 1), (6, 6, 40, 16, 3, 1, 2), (8, 9, 505, 24, 1, 1, 1), (6, 5, 36, 8, 3, 4, 2), (11, 13, 23, 9, 3, 1, 5),
])
@pytest.mark.parametrize("dt,eps", [(S.I8, 0.0), (S.BF16, 0.0), (S.BF16, 0.25)])
def test_ragged_channel_runs(h, w, ci, co, k, g, n, dt, eps):
    import numpy as np
    import oracle
    from gpu_util import assert_matches, make_layer, to_device
    seq = S.random_layer(9860 + h + ci, S.conv_shape(h, w, ci, co, k, 1, k // 2, g, n=n), dt, T=5, frac=0.3, block=2)
    seq.frames[3] = seq.frames[2].copy()
    run_sequence(seq, check_dense=(0, 1, 4), dense_switch_pct=100)
    if eps:
        layer = make_layer(seq, dense_switch_pct=100)
        layer.set_threshold(eps)
        stored = np.zeros_like(seq.frames[0])
        f32 = lambda a: (a.astype(np.uint32) << 16).view(np.float32)
        for t, x in enumerate(seq.frames):
            layer.step(to_device(x, dt))
            stored = np.where(np.abs(f32(x) - f32(stored)) < np.float32(eps), stored, x)
            assert_matches(layer.y_snapshot().cpu().numpy(), oracle.dense(seq.shape, dt, seq.weights, seq.bias, stored), dt, f"frame {t}")
        layer.destroy()


# The product of layers that are padded for it, steps and dense: rows of one entry over a step and one short of it, of whole 16-byte
# units, with whole units of padding; outputs one over a block of 16, off the fours that a thread sums, one short of a block, and
# outputs alone padded (rows of whole steps); every count of 16-stream tiles, groups of streams; the stored input, the counts and
# the caller's copy; rounding as the walk's (sums of short chains).
@pytest.mark.parametrize("ci,co,n", [
    (65, 33, 704), (63, 64, 704), (2049, 1001, 44), (4095, 1007, 64), (2048, 1001, 33), (100, 130, 300), (999, 2002, 23), (2064, 1601, 28),
    (3001, 1030, 90), (4100, 4001, 16), (2999, 513, 128), (2300, 7000, 9),
])
@pytest.mark.parametrize("dt", [S.I8, S.BF16])
def test_fc_padded_product(ci, co, n, dt):
    import numpy as np
    from gpu_util import make_layer, to_device, x_bytes
    seq = S.random_layer(9930 + ci, S.fc_shape(ci, co, n=n), dt, T=3, frac=0.3)
    st, _ = run_sequence(seq, check_dense=(0, 2), y_out_frames=(1, 2), rel=1e-5)
    before = [np.zeros_like(seq.frames[0])] + list(seq.frames[:-1])
    assert st["changed_elems"] == sum(int((a != b).sum()) for a, b in zip(before, seq.frames)) and st["delta_steps"] == 3
    layer, walk = make_layer(seq), make_layer(seq, fc_batched=0)
    for x in seq.frames:
        xd = to_device(x, dt)
        layer.step(xd)
        walk.step(xd)
        assert np.array_equal(layer.x_snapshot_bytes().cpu().numpy(), x_bytes(x, dt))
    if dt == S.BF16:  # against 64 bits; the walk's own sums too
        f64 = lambda a: (a.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        want = f64(seq.frames[-1]).reshape(n, ci) @ f64(seq.weights).reshape(co, ci).T + (0 if seq.bias is None else seq.bias.astype(np.float64))
        err = [np.linalg.norm(l.y_snapshot().cpu().numpy().reshape(n, co) - want) / np.linalg.norm(want) for l in (layer, walk)]
        assert err[0] <= max(err[1], 1.0e-7), err
    layer.destroy()
    walk.destroy()


# Output channels off the fours that a lane holds: one, two and three of a last four, fewer than four in all, whole blocks of 32 and one
# more, two blocks, groups whose channels start at any offset; maps off the 4 x 4 sub-tiles; few sub-tiles (K in parts) and
# many; changed sub-tiles alone, and everything recomputed.
@pytest.mark.parametrize("h,w,ci,co,k,st,g,n", [
    (5, 6, 16, 1, 3, 1, 1, 1), (9, 7, 32, 3, 3, 1, 1, 2), (8, 8, 64, 33, 3, 1, 1, 1), (13, 13, 128, 66, 3, 1, 2, 3), (14, 10, 48, 101, 1, 1, 1, 9),
    (20, 20, 32, 62, 5, 2, 1, 8), (28, 28, 64, 67, 3, 1, 1, 24), (30, 29, 32, 130, 3, 1, 1, 40), (40, 40, 48, 18, 3, 1, 3, 20), (17, 17, 256, 5, 3, 1, 1, 40),
])
@pytest.mark.parametrize("dt,opts", [(S.I8, {}), (S.BF16, {}), (S.BF16, {"bf16_terms": 1}), (S.I8, {"dense_switch_pct": 1}), (S.BF16, {"dense_switch_pct": 1})])
def test_output_channels_off_the_fours(h, w, ci, co, k, st, g, n, dt, opts):
    seq = S.random_layer(9840 + h + co, S.conv_shape(h, w, ci, co, k, st, k // 2, g, n=n), dt, T=3, frac=0.1, block=2)
    run_sequence(seq, check_dense=(0, 2), rel=5e-3 if opts.get("bf16_terms") else 1e-4, path=1, **opts)


# ... and their fp32 sums round once, when they meet the projection or the bias.  Inputs and weights are multiples of 1/64 and of 1/256 and
# the sums below 2^7, so that sums of products among themselves are exact in fp32 in any order; projections of 4096 and more are
# multiples of 2^-11, which every addition rounds to.  Sixteen slots of two terms (one channel block, two, groups, 1 x 1) and eight.
@pytest.mark.parametrize("h,w,ci,co,k,g,n", [(40, 40, 16, 18, 3, 1, 11), (40, 40, 16, 66, 3, 1, 11), (40, 40, 48, 18, 3, 3, 11), (40, 40, 48, 18, 1, 1, 11), (28, 28, 128, 101, 3, 1, 8)])
def test_output_channels_off_the_fours_round_once(h, w, ci, co, k, g, n):
    import numpy as np
    import oracle
    from gpu_util import make_layer, to_device
    seq = S.random_layer(9830 + co + k, S.conv_shape(h, w, ci, co, k, 1, k // 2, g, n=n), S.BF16, T=2, frac=0.1, block=2)
    rng = np.random.default_rng(9831 + co + k)
    bf16 = lambda a: (a.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    seq.weights = bf16(rng.integers(-16, 17, seq.weights.shape) / 256.0)
    seq.bias = rng.uniform(4200.0, 8000.0, co).astype(np.float32)
    changed = (seq.frames[1] != seq.frames[0]).any(axis=-1, keepdims=True)
    seq.frames[0] = bf16(rng.integers(0, 65, seq.frames[0].shape) / 64.0)
    seq.frames[1] = np.where(changed, bf16(rng.integers(0, 65, seq.frames[1].shape) / 64.0), seq.frames[0])
    sums = [oracle.dense(seq.shape, S.BF16, seq.weights, None, x) for x in seq.frames]
    assert max(abs(s).max() for s in sums) < 128.0
    full = [(seq.bias.astype(np.float64) + s).astype(np.float32) for s in sums]
    stepped = (full[0].astype(np.float64) + (sums[1] - sums[0])).astype(np.float32)
    frames = [to_device(x, S.BF16) for x in seq.frames]
    for opts, want in (({"path": 1}, stepped), ({"dense_switch_pct": 1}, full[1])):
        layer = make_layer(seq, conv_kernel=1, **opts)
        for x, y in zip(frames, (full[0], want)):
            layer.step(x)
            assert np.array_equal(layer.y_snapshot().cpu().numpy(), y), opts
        y = torch.empty(layer.y_shape, dtype=torch.float32, device="cuda")
        layer.dense(frames[1], y)
        assert np.array_equal(y.cpu().numpy(), full[1])
        layer.destroy()


# The single-launch scatter path: blocks of 8 .. 64 positions (the last one short), one workgroup per block and several, one
# tile of 32 listed positions and two, units off the pairs of a K step, several parts of K, channels off the blocks of 32,
# strides that skip positions, groups; a few positions change, then all of them, then none.
@pytest.mark.parametrize("h,w,ci,co,k,st,pad,g,n", [
    (8, 8, 16, 16, 3, 1, 1, 1, 1), (5, 13, 48, 33, 3, 1, 1, 1, 1), (13, 5, 80, 31, 3, 2, 1, 1, 3), (9, 7, 144, 70, 1, 1, 0, 1, 2), (9, 9, 288, 40, 3, 1, 1, 2, 1),
    (6, 6, 512, 64, 3, 1, 1, 1, 1), (4, 4, 1024, 20, 3, 3, 2, 1, 1), (40, 37, 16, 16, 5, 1, 2, 1, 1), (61, 3, 64, 96, 3, 2, 0, 4, 7),
])
@pytest.mark.parametrize("dt", [S.I8, S.BF16])
def test_scatter_path_edges(h, w, ci, co, k, st, pad, g, n, dt):
    seq = S.random_layer(9800 + h + ci, S.conv_shape(h, w, ci, co, k, st, pad, g, n=n), dt, T=5, frac=0.1, block=2)
    seq.frames[2] = S.random_layer(9850 + h + ci, seq.shape, dt, T=1, frac=0.1, block=2).frames[0]
    seq.frames[3] = seq.frames[2].copy()
    run_sequence(seq, check_dense=(), path=3)


# Forms of the scatter kernel: one, two, four and eight units per thread, and one beyond a whole number of them; the commit by the
# wavefront that announces the workgroup (few workgroups; 1024 units, the most that it takes), by all threads (more units, many
# workgroups that share blocks of one, two and four units a thread, one workgroup per block); blocks halved to those 1024 units and not (few
# blocks, and many; shared by few workgroups, and by many).  With and without a threshold
# (bf16): the stored input holds the entries that differ by it or more, the projection is that input's.
@pytest.mark.parametrize("h,w,ci,co,k,n", [
    (9, 7, 16, 16, 3, 1), (16, 16, 64, 32, 3, 1), (12, 11, 144, 40, 3, 1), (14, 14, 256, 64, 3, 1), (14, 14, 512, 32, 1, 1), (8, 8, 1024, 33, 1, 1),
    (40, 40, 512, 16, 1, 2), (31, 33, 256, 96, 3, 1), (24, 24, 16, 8, 1, 9), (24, 27, 32, 48, 3, 10), (28, 28, 96, 96, 3, 4), (20, 20, 256, 96, 3, 8),
    (13, 13, 384, 256, 3, 2), (24, 7, 400, 112, 3, 5),
])
@pytest.mark.parametrize("dt,eps", [(S.I8, 0.0), (S.BF16, 0.0), (S.BF16, 0.25)])
def test_scatter_kernel_forms(h, w, ci, co, k, n, dt, eps):
    import numpy as np
    import oracle
    from gpu_util import assert_matches, make_layer, to_device, x_bytes
    seq = S.random_layer(9880 + h + ci, S.conv_shape(h, w, ci, co, k, 1, k // 2, 1, n=n), dt, T=5, frac=0.15, block=3)
    seq.frames[3] = seq.frames[2].copy()
    layer = make_layer(seq, path=3)
    if eps:
        layer.set_threshold(eps)
    stored = np.zeros_like(seq.frames[0])
    for t, x in enumerate(seq.frames):
        layer.step(to_device(x, dt))
        if dt == S.BF16:
            f32 = lambda a: (a.astype(np.uint32) << 16).view(np.float32)
            keep = np.abs(f32(x) - f32(stored)) < np.float32(eps)
            stored = np.where(keep, stored, x)
        else:
            stored = x
        assert np.array_equal(layer.x_snapshot_bytes().cpu().numpy(), x_bytes(stored, dt)), f"stored input after frame {t}"
        want = oracle.dense(seq.shape, dt, seq.weights, seq.bias, stored)
        assert_matches(layer.y_snapshot().cpu().numpy(), want, dt, f"frame {t}")
    layer.destroy()


# The differences without a threshold are made by another loop than with one.  Denormal, huge and infinite entries that change, and
# infinite ones that stay beside entries that change: with a threshold that truncates nothing the projections are the same bits
# (1 x 1 and one part of the channels: one add an output), and an infinity that stays adds nothing.
def test_scatter_differences_of_special_values():
    import numpy as np
    import torch
    from gpu_util import make_layer, to_device
    seq = S.random_layer(9891, S.conv_shape(9, 11, 128, 40, 1, 1, 0, 1), S.BF16, T=4, frac=0.3, block=2)
    for t, x in enumerate(seq.frames):
        x[..., 3, 4, 5] = 0x7F80
        x[..., 7, 2, 0] = 0xFF80
        x[..., 5, 5, :] = [(0x0001, 0x8003, 0x7F7F, 0x0080)[(c + t) % 4] for c in range(128)]
        x[..., 6, 6, :] = 0x7F7F if t % 2 else 0xFF7F
        x[..., 8, 8, 17:19] = (0x7F80, 0x4000) if t == 2 else (0x4000, 0x7F80)
        x[..., 3, 4, 6] = x[..., 7, 2, 9] = 0x3F80 + t
    exact, other = make_layer(seq, path=3), make_layer(seq, path=3)
    other.set_threshold(2.0 ** -149)
    for t, x in enumerate(seq.frames):
        got = []
        for layer in (exact, other):
            layer.step(to_device(x, S.BF16))
            got.append(layer.y_snapshot().cpu().numpy())
        assert np.array_equal(got[0], got[1], equal_nan=True), f"frame {t}"
        if t == 0:  # (an infinity's tail is not a number: the projections that the first frame left start again from zero)
            for layer in (exact, other):
                state = type("State", (), {"__cuda_array_interface__": {
                    "shape": (9 * 11 * 40,), "typestr": "<f4", "data": (layer.snapshot_ptrs()[1], False), "version": 2}})()
                torch.as_tensor(state, device="cuda").zero_()
            torch.cuda.synchronize()
        else:
            y = got[0].reshape(9, 11, 40)
            assert np.isfinite(y[3, 4]).all() and np.isfinite(y[7, 2]).all() and y[3, 4].any() and y[7, 2].any(), f"frame {t}"
    exact.destroy()
    other.destroy()


# ... and the bf16 blocks whose planes and lists together are beyond 64 KB of LDS.
@pytest.mark.parametrize("ci", [496, 1000])
def test_scatter_path_with_the_largest_blocks(ci):
    seq = S.random_layer(9870 + ci, S.conv_shape(6, 7, ci, 24, 3, 1, 1, 1, n=2), S.BF16, T=3, frac=0.2, block=2)
    run_sequence(seq, check_dense=(), path=3)


# A layer of few adds behind another one: its products are the scatter kernel's, of the difference that the scan has left, and
# the launch leaves flags, statistics and words as the tile kernel does ("path" = 1), in turn with plain steps of either path;
# what reads the flags then sees all that was written.  (map, c, c_out, k, stride, pad, groups, streams)
@pytest.mark.parametrize("m,ci,co,k,st,pad,g,n", [
    (13, 32, 48, 3, 1, 1, 1, 1), (9, 64, 36, 5, 2, 2, 1, 3), (27, 48, 72, 3, 1, 1, 1, 2), (6, 160, 64, 1, 1, 0, 2, 5), (40, 16, 16, 3, 1, 1, 1, 9),
])
def test_scatter_of_a_scans_difference(m, ci, co, k, st, pad, g, n):
    import numpy as np
    import oracle
    import paper_1802_09723_amd as rrm
    import torch
    from gpu_util import assert_matches, to_device
    first = S.random_layer(9950 + m, S.conv_shape(m, m, 16, ci, 3, 1, 1, 1, n=n), S.I8, T=8, frac=0.1, block=3)
    first.frames[4] = first.frames[3].copy()
    nxt = S.random_layer(9960 + m, S.conv_shape(m, m, ci, co, k, st, pad, g, n=n), S.I8, T=1, frac=0.1, block=3)
    A = rrm.Layer(first.shape, S.I8, first.weights, first.bias)
    B, T = (rrm.Layer(nxt.shape, S.I8, nxt.weights, nxt.bias) for _ in range(2))
    T.set_option("path", 1)
    shift = oracle.calibrate_shift(oracle.dense(first.shape, S.I8, first.weights, first.bias, first.frames[0]))
    out = [torch.full(B.y_shape, -1, dtype=torch.int8, device="cuda") for _ in range(2)]
    for t, x in enumerate(first.frames):
        A.step(to_device(x, S.I8))
        f = oracle.relu_requant_pool(oracle.dense(first.shape, S.I8, first.weights, first.bias, x), shift, False)
        for layer in (B, T):
            if t == 5:
                layer.step(to_device(f, S.I8))
            else:
                layer.step_from_projection(A, shift, False)
        want = oracle.dense(nxt.shape, S.I8, nxt.weights, nxt.bias, f)
        for layer, o in zip((B, T), out):
            assert_matches(layer.y_snapshot().cpu().numpy(), want, S.I8, f"frame {t}")
            layer.relu_requant_pool_changed(o, 4, False)
            assert np.array_equal(o.cpu().numpy(), oracle.relu_requant_pool(want, 4, False)), f"frame {t}: what was written"
        if t < 5:  # (a plain scatter step counts positions)
            assert B.stats() == T.stats(), f"frame {t}"
    for layer in (A, B, T):
        layer.destroy()


def fc_step_is_product(dt, ci, co, n):
    """Which way a step of an FC layer runs where both are possible: one product for all streams, or a column walk per stream."""
    if dt == S.BF16 and n >= 16:
        return True
    es = 1 if dt == S.I8 else 2
    walks = n * ((co * es + 63) // 64)
    if walks >= (640 if ci * es > 16384 else 512):
        return True
    return dt == S.I8 and n <= 64 and ci * co <= 40 << 20 and walks * 64 * ci >= 200 << 20


# int8 steps as one product: every stream-tile count and group count, on the shortest layer of whole 64-row groups and off them that
# takes the product; k ranges with a ragged last chunk, one split and several.
@pytest.mark.parametrize("n", [4, 9, 15, 16, 17, 32, 33, 48, 64, 65, 90, 100, 128, 129, 190, 300, 520])
def test_fc_int8_product_step_at_every_stream_count(n):
    co, ci = 64 * ((511 + n) // n) - 48 * (n % 2), 64 * (1, 2, 5, 7, 13, 24)[n % 6]
    assert fc_step_is_product(S.I8, ci, co, n) and not fc_step_is_product(S.I8, ci, 64 * (511 // n), n)
    seq = S.random_layer(9950 + n, S.fc_shape(ci, co, n=n), S.I8, T=3, frac=0.2)
    st, _ = run_sequence(seq, check_dense=(0, 2), y_out_frames=(1, 2))
    walk, _ = run_sequence(seq, check_dense=(2,), fc_batched=0)
    assert st["delta_steps"] == 3 and st["changed_elems"] == walk["changed_elems"]


# Sixteen splits and around: the sums' launch reads five at a time behind the first.  (c_in, c_out, streams), int8 in bytes: 16, 12, 11
# and 6 splits of four-step chunks, 16 and 9 of two-step ones; the dense layer, and the step of bf16 layers.
@pytest.mark.parametrize("ci,co,n", [(16384, 64, 16), (12288, 48, 20), (11264, 112, 33), (6144, 64, 16), (8192, 80, 70), (4608, 64, 128)])
@pytest.mark.parametrize("dt", [S.I8, S.BF16])
def test_fc_product_of_many_splits(ci, co, n, dt):
    seq = S.random_layer(9960 + n, S.fc_shape(ci // (1 if dt == S.I8 else 2), co, n=n), dt, T=2, frac=0.2)
    run_sequence(seq, check_dense=(0, 1), rel=1e-4)


# int8 layers whose walks would read more than 200 MiB: on both sides of that line, of the 64 streams and of a W of 40 MiB.
@pytest.mark.parametrize("ci,co,n,product", [
    (9216, 1040, 22, True), (9216, 1040, 20, False), (16384, 192, 50, False), (16384, 208, 50, True), (8192, 368, 64, False), (8192, 400, 64, True),
    (8256, 400, 65, False), (16384, 2576, 5, False), (16384, 2560, 5, True),
])
def test_fc_step_of_long_rows(ci, co, n, product):
    assert fc_step_is_product(S.I8, ci, co, n) == product
    seq = S.random_layer(9940 + n, S.fc_shape(ci, co, n=n), S.I8, T=3, frac=0.1)
    st, _ = run_sequence(seq, check_frames=(1, 2), y_out_frames=(1, 2), check_dense=())
    assert st["delta_steps"] == 3


# Many streams: the launch that sums the splits commits and counts the frame and fills the caller's copy; one group of streams and
# several, a frame that repeats; few streams of many channels, on both sides of the line.
@pytest.mark.parametrize("ci,co,n", [(64, 16, 16), (192, 48, 33), (1024, 80, 129), (320, 272, 300), (128, 4096, 4), (64, 4096, 8), (192, 2048, 7), (128, 2064, 15)])
@pytest.mark.parametrize("dt", [S.I8, S.BF16])
def test_fc_step_of_many_streams(ci, co, n, dt):
    import numpy as np
    seq = S.random_layer(9930 + n, S.fc_shape(ci, co, n=n), dt, T=4, frac=0.1)
    seq.frames[2] = seq.frames[1].copy()
    st, _ = run_sequence(seq, check_dense=(0,), y_out_frames=(0, 1, 2, 3))
    before = [np.zeros_like(seq.frames[0])] + list(seq.frames[:-1])
    assert st["changed_elems"] == sum(int((a != b).sum()) for a, b in zip(before, seq.frames)) and st["delta_steps"] == 4


# The rounding error of a bf16 layer as one product, norm over norm against 64 bits: dense, and the step where it takes the product.
# Up to 16 streams: chains of four matrix instructions (each adds about 0.26e-7, independent roundings: 0.52e-7), a rounding per
# split and one of the result (0.35e-7 each, the mean of 2^-24 over a binade): 0.72e-7.  More streams: chains of at most 20 or, from
# 65 streams on, 32 instructions, 1.3e-7 and 1.6e-7.  The bounds leave a third.  Rows where the split cap binds, few outputs and many.
@pytest.mark.parametrize("ci,co,n,bound", [
    (4096, 4096, 4, 1e-7), (4096, 4096, 15, 1e-7), (9216, 256, 16, 1e-7), (65536, 64, 4, 1e-7), (608, 48, 5, 1e-7),
    (65536, 64, 17, 1.7e-7), (65536, 64, 33, 1.7e-7), (24576, 192, 64, 1.7e-7), (65536, 64, 65, 2.1e-7), (65536, 48, 129, 2.1e-7),
])
def test_fc_product_rounding(ci, co, n, bound):
    import numpy as np
    import paper_1802_09723_amd as rrm
    import torch
    gen = torch.Generator(device="cuda").manual_seed(ci + n)
    w = (torch.randn((co, ci), generator=gen, device="cuda") * 0.05).to(torch.bfloat16)
    bias = torch.randn((co,), generator=gen, device="cuda") * 0.1
    layer = rrm.Layer(S.fc_shape(ci, co, n=n), S.BF16, w.view(torch.int16).cpu().numpy().view(np.uint16), bias.cpu().numpy())
    y = torch.empty(layer.y_shape, dtype=torch.float32, device="cuda")
    for t in range(2):
        x = torch.randn((n, ci), generator=gen, device="cuda").clamp_(min=0).to(torch.bfloat16)
        want = x.double() @ w.double().T + bias.double()
        layer.dense(x, y)
        layer.step(x)
        torch.cuda.synchronize()
        error = float((y.double() - want).norm() / want.norm())
        assert error <= bound, f"frame {t}: {error:.2e}"
        if fc_step_is_product(S.BF16, ci, co, n):
            assert torch.equal(layer.y_snapshot(), y), f"frame {t}: the step's projection is not the dense one"
    layer.destroy()


# Any two int8 inputs are in range for an FC layer, whichever way its step runs: frames from the lowest value to the highest and
# back are exact and raise no range error.  (c_out, streams): the column walk and the product, one group of streams and several.
@pytest.mark.parametrize("co,n,product", [(48, 1, False), (48, 20, False), (4096, 8, True), (2048, 33, True), (272, 300, True)])
def test_fc_step_of_full_range_differences(co, n, product):
    assert fc_step_is_product(S.I8, 192, co, n) == product
    seq = S.random_layer(9970 + n, S.fc_shape(192, co, n=n), S.I8, T=4, frac=0.3)
    for t, frame in enumerate(seq.frames):
        frame[..., -40:] = (-128, 127)[t % 2]
    st, _ = run_sequence(seq, check_dense=())
    assert st["range_error"] == 0


# What a step counts and the unit that the statistics name go together: input positions on the single-launch scatter path (automatic
# for layers of few adds, asked for otherwise), 4 x 4 blocks of output positions on the tile kernel.
@pytest.mark.parametrize("m,ci,co,n,dt,path", [(20, 16, 24, 4, S.I8, 0), (9, 32, 40, 1, S.BF16, 0), (40, 96, 96, 8, S.I8, 3)])
def test_units_of_the_step_counters(m, ci, co, n, dt, path):
    from gpu_util import make_layer, to_device
    seq = S.random_layer(9980 + m, S.conv_shape(m, m, ci, co, 3, 1, 1, 1, n=n), dt, T=3, frac=0.1, block=3)
    layer = make_layer(seq, path=path)
    changed, last = 0, 0
    for x in seq.frames:
        layer.step(to_device(x, dt))
        changed += int((x != last).any(axis=3).sum())
        last = x
    st = layer.stats()
    assert (st["tile_positions"], st["active_tiles"], st["total_tiles"]) == (1, changed, 3 * n * m * m)
    layer.set_option("path", 1)
    layer.reset()
    layer.step(to_device(seq.frames[0], dt))
    st = layer.stats()
    assert (st["tile_positions"], st["active_tiles"], st["total_tiles"]) == (16,) + 2 * (n * ((m + 3) // 4) ** 2,)
    layer.destroy()


# The sub-tile flags carry the step's own value and are wiped a step later: what a step counts as active is what its own frame
# changed, whatever the steps before marked.  (map, streams): flag arrays off the words of four and the vectors of 16, one
# workgroup per flag group, one round of vectors in the work list, several, and more than stay in registers; the frames
# change, stay, change elsewhere.
@pytest.mark.parametrize("m,n", [(9, 1), (29, 3), (31, 15), (31, 40), (64, 17), (63, 67), (63, 150)])
def test_active_subtiles_of_consecutive_steps(m, n):
    import numpy as np
    import oracle
    from gpu_util import assert_matches, make_layer, to_device
    seq = S.random_layer(9700 + m, S.conv_shape(m, m, 16, 40, 3, 1, 1, 1, n=n), S.I8, T=2, frac=0.1, block=3)
    layer = make_layer(seq, path=1, conv_kernel=1)
    rng = np.random.default_rng(m)
    x = np.array(seq.frames[0])
    layer.step(to_device(x, S.I8))
    seen = layer.stats()["active_tiles"]
    sub = (m + 3) // 4
    for t in range(6):
        changed = np.zeros((n, m, m), bool)
        if t % 3:
            for b in range(0, n, 1 + t):
                y0, x0 = rng.integers(0, m - 2, 2)
                changed[b, y0:y0 + 2, x0:x0 + 3] = True
        x[changed] ^= 1
        layer.step(to_device(x, S.I8))
        grown = np.zeros((n, m + 2, m + 2), bool)
        for dy in range(3):
            for dx in range(3):
                grown[:, dy:dy + m, dx:dx + m] |= changed
        tiles = np.zeros((n, 4 * sub, 4 * sub), bool)
        tiles[:, :m, :m] = grown[:, 1:-1, 1:-1]
        want = int(tiles.reshape(n, sub, 4, sub, 4).any(axis=(2, 4)).sum())
        now = layer.stats()["active_tiles"]
        assert now - seen == want, f"step {t}: {now - seen} active sub-tiles, not {want}"
        seen = now
    want = oracle.dense(seq.shape, S.I8, seq.weights, seq.bias, x)
    assert_matches(layer.y_snapshot().cpu().numpy(), want, S.I8, "last frame")
    layer.destroy()


# The scan of a layer fed by the layer before, pooled and not: one group of 16 units per wavefront, and four where the input is
# large (pooled); loads ahead of the flags where it is small.  (producer's map, channels, streams): units off the 16s, the 64s and
# the workgroups, both sides of the lines, one unit in all.
# The producer's frame changes, stays (the difference buffer is cleared) and changes elsewhere; every count is the frame's own.
@pytest.mark.parametrize("m,c,n,pool", [
    (3, 16, 1, True), (11, 48, 3, True), (55, 16, 2, True), (29, 32, 40, True), (29, 48, 40, True), (55, 16, 180, True),
    (1, 16, 1, False), (11, 48, 3, False), (29, 32, 9, False), (29, 32, 12, False),
])
def test_scan_of_a_fused_step(m, c, n, pool):
    import numpy as np
    import oracle
    import paper_1802_09723_amd as rrm
    from gpu_util import assert_matches, to_device
    rng = np.random.default_rng(m + n)
    s1, q = S.conv_shape(m, m, 16, c, 3, 1, 1, 1, n=n), (m - 3) // 2 + 1 if pool else m
    s2 = S.conv_shape(q, q, c, 24, 3 if q > 1 else 1, 1, 1 if q > 1 else 0, 1, n=n)
    w1, w2 = (rng.integers(-127, 128, (s.c_out, s.kh, s.kw, s.c_in), dtype=np.int8) for s in (s1, s2))
    b1, b2 = (rng.integers(-1000, 1001, s.c_out).astype(np.int32) for s in (s1, s2))
    A, B = rrm.Layer(s1, S.I8, w1, b1), rrm.Layer(s2, S.I8, w2, b2)
    x = S.draw_i8_relu(rng, s1.x_shape)
    old, shift, seen = np.zeros(s2.x_shape, np.int8), None, (0, 0)
    for t in range(4):
        if t in (1, 3):
            y0 = int(rng.integers(0, max(1, m - 4)))
            x[::1 + t, y0:y0 + 4, :1 + m // 2] = S.draw_i8_relu(rng, x[::1 + t, y0:y0 + 4, :1 + m // 2].shape)
        A.step(to_device(x, S.I8))
        ya = oracle.dense(s1, S.I8, w1, b1, x) if t != 2 else ya
        if shift is None:
            shift = oracle.calibrate_shift(ya)
        B.step_from_projection(A, shift, pool)
        f = oracle.relu_requant_pool(ya, shift, pool)
        st = B.stats()
        units = int((f != old).reshape(-1, 16).any(axis=1).sum())
        assert (st["changed_elems"] - seen[0], st["changed_units"] - seen[1]) == (int((f != old).sum()), units), f"step {t}"
        assert np.array_equal(B.x_snapshot_bytes().cpu().numpy(), f.view(np.uint8).reshape(-1)), f"step {t}"
        seen, old = (st["changed_elems"], st["changed_units"]), f
    assert_matches(B.y_snapshot().cpu().numpy(), oracle.dense(s2, S.I8, w2, b2, old), S.I8, "last frame")
    A.destroy()
    B.destroy()


# Few channels: a 16-byte unit covers several positions, which are marked a run at a time.  Strides beyond the filter leave
# columns that no window reads; units cross rows; what counts as active is exact.
@pytest.mark.parametrize("h,w,c,k,st,pad,n", [(9, 5, 3, 3, 1, 1, 2), (40, 33, 3, 11, 4, 0, 2), (12, 50, 2, 1, 3, 0, 1), (31, 30, 1, 2, 5, 1, 3), (7, 3, 5, 3, 2, 1, 2)])
def test_active_subtiles_of_few_channels(h, w, c, k, st, pad, n):
    import numpy as np
    import oracle
    from gpu_util import assert_matches, make_layer, to_device
    seq = S.random_layer(9800 + w, S.conv_shape(h, w, c, 16, k, st, pad, 1, n=n), S.I8, T=2, frac=0.1, block=3)
    layer = make_layer(seq, path=1, conv_kernel=1)
    rng = np.random.default_rng(w)
    x = np.array(seq.frames[0])
    layer.step(to_device(x, S.I8))
    seen = layer.stats()["active_tiles"]
    ho, wo = (h + 2 * pad - k) // st + 1, (w + 2 * pad - k) // st + 1
    for t in range(5):
        x[rng.integers(0, n), rng.integers(0, h), rng.integers(0, w), rng.integers(0, c)] ^= 1
        units = (x.reshape(-1) != np.array(seq.frames[0]).reshape(-1)) if t == 0 else (x.reshape(-1) != last.reshape(-1))
        flat = np.zeros((units.size + 15) // 16 * 16, bool)
        flat[:units.size] = units
        flat = np.repeat(flat.reshape(-1, 16).any(axis=1), 16)[:units.size]  # (a position is marked with its whole unit)
        pos = flat.reshape(n, h, w, c).any(axis=3)
        want = np.zeros((n, (ho + 3) // 4, (wo + 3) // 4), bool)
        for b, iy, ix in zip(*np.nonzero(pos)):
            ys = [oy for oy in range(ho) if 0 <= iy + pad - oy * st < k]
            xs = [ox for ox in range(wo) if 0 <= ix + pad - ox * st < k]
            for oy in ys:
                for ox in xs:
                    want[b, oy // 4, ox // 4] = True
        last = x.copy()
        layer.step(to_device(x, S.I8))
        now = layer.stats()["active_tiles"]
        assert now - seen == int(want.sum()), f"step {t}"
        seen = now
    assert_matches(layer.y_snapshot().cpu().numpy(), oracle.dense(seq.shape, S.I8, seq.weights, seq.bias, x), S.I8, "last frame")
    layer.destroy()


def test_default_stream_is_the_current_one():
    """A call without a stream goes to torch's current stream, inside and outside of a stream context."""
    from paper_1802_09723_amd import binding
    assert (binding._stream_ptr(None) or 0) == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert binding._stream_ptr(None) == s.cuda_stream == binding._stream_ptr(s)
    assert (binding._stream_ptr(None) or 0) == torch.cuda.current_stream().cuda_stream
