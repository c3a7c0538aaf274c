// Geometry of the binary (XNOR / popcount) convolution and the choice of the band kernel's bands.  Plain host C++
// (no HIP types): the kernels, the dispatcher and a host-only test include it.
#pragma once
#include <stddef.h>

#include "rrm.h"

namespace rrm {

constexpr int BIN_TILE = 8;        // output tile edge of the tile kernel
constexpr long long BIN_TILE_MAX_LDS = 152 * 1024;  // both window copies of one tile (160 KB per workgroup, less static use)
constexpr int BAND_WAVES = 8;      // wavefronts of a band-kernel workgroup
constexpr int BAND_RP = 65;        // row pitch (words) of the sums of a pass (at most 64 x 64)
constexpr int BAND_SUMS = 64 * BAND_RP * 4;    // bytes of them
constexpr long long BAND_LDS = 79 * 1024;      // LDS of a band-kernel workgroup (two per compute unit)
constexpr long long BAND_WIDE_FRAME = 128 * 1024;  // a stream's frame up to which a wide layer has bands
constexpr int BIN_NUM_CU = 256;    // compute units of the MI355X

struct BinGeom {
    int n, h, w, c_out, kh, kw, stride, pad, groups;
    int wpp;             // 32-bit words per input position (all groups)
    int wg;              // words per position per group
    int og;              // output channels per group
    int ho, wo, tiles_y, tiles_x;
    int th_in, tw_in;
    int pitch;           // LDS words per staged position
    int nslab;           // word slabs of 4 per group
    int nob8;            // packed 8-channel filter blocks per group (og padded to 16)
    unsigned int magic_wg4;    // floor(2^32/d)+1 for d = 4*nslab
    unsigned int magic_tw;     // same for d = tw_in
    // band kernel: bands of band_rows output rows over the full width; 0 rows = the layer has no bands (they do not fit
    // LDS, or it is a wide layer with large frames) and runs the tile kernel
    int band_rows, nbands, bth_in, btw_in;
    unsigned int magic_btw;    // same for d = btw_in
    unsigned int magic_nslab;  // same for d = nslab
    int vec4;                  // 1: a group's words per position are whole 16-byte vectors (wg % 4 == 0, wpp % 4 == 0)
    int fused_ok;              // 1: the band kernel can run the whole step (compare and commit included)
    // (Nothing.  The same instructions take 6.10 us a step with the fields after it here and 6.23 eight bytes lower: 14 x 14, 512 -> 512, one
    // stream, 10 %; 256 -> 256, two, 5.90 and 6.00.  Only their places among the kernel's arguments differ; the cause is not known.)
    int gap[2];
    int bpitch;                // LDS words per staged position of the band kernel: `pitch`, or without its padding
    unsigned int magic_nbands, magic_nblk, magic_nblk32, magic_wo;  // same for d = nbands, blocks of 64 and of 32 channels per group, wo
    const int* steps;          // (device memory) a K step's place in a position's window, in pairs of words: see bin_step_at
    int nsplit;                // (set by the launcher) workgroups that share a band's list
};


inline unsigned int bin_magic_for(int d) { return d <= 1 ? 0u : (unsigned int)((1ull << 32) / (unsigned long long)d + 1ull); }

// dynamic LDS of a band-kernel workgroup with bands of band_rows output rows: the A and B words of the band's input
// window, its flags (a byte per window position, or less), the list of active output positions (16 bits each), and the sums of
// a pass
#ifdef __HIPCC__
__host__ __device__
#endif
inline size_t bin_band_list_offset(const BinGeom& g) {
    const size_t npos = (size_t)g.bth_in * (size_t)g.btw_in;
    return 2 * npos * g.bpitch * 4 + ((npos + 15) & ~(size_t)15);
}
inline size_t bin_band_lds_bytes(const BinGeom& g, int band_rows) {
    const size_t npos = (size_t)((band_rows - 1) * g.stride + g.kh) * (size_t)((g.wo - 1) * g.stride + g.kw);
    return 2 * npos * g.bpitch * 4 + ((npos + 15) & ~(size_t)15) + (((size_t)band_rows * g.wo * 2 + 15) & ~(size_t)15) + BAND_SUMS;
}

// Pairs of staged words per input position, at an odd pitch except in wide layers; where a K step (a tap, two words of its channels)
// starts in the window of an output position
#ifdef __HIPCC__
__host__ __device__
#endif
inline int bin_pair_pitch(const BinGeom& g) { return g.bpitch < g.pitch ? g.nslab * 4 : g.nslab * 4 + 1; }
inline int bin_step_at(const BinGeom& g, int k) {
    const int nkt = 2 * g.nslab, tap = k / nkt;
    return (tap / g.kw * g.btw_in + tap % g.kw) * bin_pair_pitch(g) + 2 * (k - tap * nkt);
}

// Does the dense layer run the tile kernel: without bands; wide layers (us, tile and band: 4 x 1100, 128 -> 1024 channels 1 x 1, 11.8
// and 31.0; 3 x 3, one stream, 4 x 350, 128 -> 64, 7.5 and 14.5; 24 x 350, 128 -> 512, 20.8 and 19.9; four streams of 8 x 350, 128 -> 256,
// 14.8 and 17.1; but many streams gain on bands: 16 of 16 x 350, 128 -> 64, 21.8 and 18.5, 64 of 2 x 350, 128 -> 128, 58.8 and 18.4); and 1 x 1
// filters of few words, whose products are too short for what a band costs beside them (16 x 320, 256 -> 256, 2 streams, 8.7
// and 13.0; 112 x 112, 64 -> 64, 64 streams, 65.5 and 85.5; 20 x 33, 224 -> 112, 30 streams, 8.4 and 10.1; 14 x 14, 256 -> 512, 8
// streams, 7.2 and 7.5; but 28 x 28, 256 -> 256, 16 streams, 10.3 and 9.3; 512 channels are level or behind: 7 x 7, 512 -> 512, 64
// streams, 9.0 and 7.8).  Not where bands fill the chip and their words are read whole, but the map leaves more than a fifth of its
// 8 x 8 tiles empty (28 x 28, 128 -> 512, 64 streams, 45.2 and 41.3; 13 x 13, 256 -> 256, 128, 18.3 and 13.0).
inline bool bin_dense_on_tiles(const BinGeom& g) {
    if (g.band_rows == 0 || g.bpitch < g.pitch) return true;
    if (g.kh * g.kw != 1 || g.wg > 8) return false;
    const bool fills = (long long)g.n * g.nbands * g.groups * ((g.og + 63) / 64) >= 2 * BIN_NUM_CU;
    const bool empty = 5ll * g.ho * g.wo < 4ll * BIN_TILE * BIN_TILE * g.tiles_y * g.tiles_x;
    return !(fills && empty && g.vec4);
}

// Fill the geometry of a binary layer, for its steps or for its dense launches (only the bands differ).  False: the input
// window of one 8x8 output tile does not fit LDS (the layer cannot be created).
inline bool bin_choose_shape(const rrm_shape& s, BinGeom& g, bool dense = false) {
    g.n = s.n; g.h = s.h; g.w = s.w; g.c_out = s.c_out; g.kh = s.kh; g.kw = s.kw;
    g.stride = s.stride; g.pad = s.pad; g.groups = s.groups;
    g.wpp = s.c_in / 32;
    g.wg = g.wpp / s.groups;
    g.og = s.c_out / s.groups;
    g.ho = (s.h + 2 * s.pad - s.kh) / s.stride + 1;
    g.wo = (s.w + 2 * s.pad - s.kw) / s.stride + 1;
    g.tiles_y = (g.ho + BIN_TILE - 1) / BIN_TILE;
    g.tiles_x = (g.wo + BIN_TILE - 1) / BIN_TILE;
    g.th_in = (BIN_TILE - 1) * s.stride + s.kh;
    g.tw_in = (BIN_TILE - 1) * s.stride + s.kw;
    g.nslab = (g.wg + 3) / 4;
    g.pitch = g.nslab * 4 + 4;
    g.nob8 = 2 * ((g.og + 15) / 16);
    g.magic_wg4 = bin_magic_for(g.nslab * 4);
    g.magic_tw = bin_magic_for(g.tw_in);
    if ((long long)2 * g.th_in * g.tw_in * g.pitch * 4 > BIN_TILE_MAX_LDS) return false;
    // delta step: bands of output rows whose window, flags and list fit the LDS budget (two workgroups per compute
    // unit); as tall as fits when the streams alone fill the chip (a tall band wastes least on its halo rows and
    // fills its 64-lane chunks best), shorter -- down to 4 rows -- while there are fewer than two workgroups per
    // compute unit; no band at all = the tile kernel
    // Wide layers, of which one output row fits that budget without the sums of a pass but not with them, stage their
    // window without the padding: still two workgroups per compute unit.  (3 x 3, 5 % of the values flipping: 2 x 350, 128
    // -> 128 channels, 64 streams, 37.1 us on the tile kernel and 12.5 on bands; 4 x 350, 128 -> 256, 50.6 and 21.0; 16 x
    // 350, 128 -> 512, one stream, 17.4 and 11.7.)  Not where a stream's frame is large: its last workgroup copies it
    // alone (350 x 350, 128 -> 64, one stream: 27 and 80 us; 64 x 350, 128 -> 128, 8 streams, 1 %: 26 and 32).
    g.bpitch = g.pitch;
    g.band_rows = 0;
    const long long row_lds = (long long)bin_band_lds_bytes(g, 1);
    const bool wide = row_lds > BAND_LDS;
    if (wide && row_lds <= BAND_LDS + BAND_SUMS && (long long)g.h * g.w * g.wpp * 4 <= BAND_WIDE_FRAME) g.bpitch = 4 * g.nslab;
    for (int r = g.ho; r >= 1 && (!wide || g.bpitch < g.pitch); --r)
        if ((long long)bin_band_lds_bytes(g, r) <= BAND_LDS && (long long)r * g.wo <= 65535) {
            g.band_rows = r;
            break;
        }
    if (g.band_rows == 0) g.bpitch = g.pitch;
    const int tallest = g.band_rows;
    g.vec4 = (g.wg % 4 == 0 && g.wpp % 4 == 0) ? 1 : 0;
    auto set_rows = [&](int rows) {
        g.band_rows = rows;
        g.nbands = (g.ho + g.band_rows - 1) / g.band_rows;
        g.bth_in = (g.band_rows - 1) * s.stride + s.kh;
        g.btw_in = (g.wo - 1) * s.stride + s.kw;
        // The band kernel can run the whole step in one launch when every input position lies inside the window of
        // the band that owns its row (band k owns input rows k*R*stride .. (k+1)*R*stride - 1, the last band the rest):
        // then each position is compared and counted exactly once, and whole 16-byte vectors are compared.
        const bool cols = g.btw_in - s.pad >= s.w;
        const bool rows_mid = g.nbands == 1 || s.stride <= s.kh - s.pad;
        const bool rows_last = (g.nbands - 1) * g.band_rows * s.stride - s.pad + g.bth_in >= s.h;
        g.fused_ok = g.vec4 && cols && rows_mid && rows_last ? 1 : 0;
    };
    const long long per_band = (long long)g.n * g.groups * ((g.og + 63) / 64);
    // Bands of at most `tallest` rows: more of them while there are fewer than `want` workgroups and the next count's bands
    // still have `min_rows` rows and `min_out` outputs.
    auto cut = [&](long long want, int min_rows, int min_out) {
        g.nbands = (g.ho + tallest - 1) / tallest;
        for (; per_band * g.nbands < want && g.nbands < g.ho; ++g.nbands) {
            const int next = (g.ho + g.nbands) / (g.nbands + 1);
            if (next < min_rows || (long long)next * g.wo < min_out) break;
        }
        set_rows((g.ho + g.nbands - 1) / g.nbands);
    };
    g.nbands = 1;
    g.fused_ok = 0;
    if (tallest > 0) {
        // (a row of a wide layer holds several passes: down to one row)
        cut(2 * BIN_NUM_CU, wide ? 1 : 4, 0);
        // A few workgroups over two per compute unit wait for the first ones to end: a band fewer then, as long as two thirds of
        // those places are taken.  (us without and so, dense: 26 streams of 60 x 13, 448 -> 72, ten bands, 29.3 and 21.5; 54 of 40 x
        // 40, 128 -> 128, 5 x 5, five, 47.9 and 36.7; 50 of 20 x 20, 256 -> 256, three, 25.0 and 19.8; but 64 of 28 x 28, 128 -> 384,
        // two, 42.1 and 44.9.  A step, 5 % of the values flipping: 43 streams of 14 x 14, 256 -> 512, two bands, 16.0 and 11.3; the
        // third dense layer 17.2 and 15.3; but the second 33.7 and 34.5: of many bands some are short and make room early.)  1 x 1
        // filters keep theirs: bin_dense_on_tiles goes by the count.
        const int fewer = g.nbands - 1;
        if (s.kh * s.kw > 1 && per_band * g.nbands > 2 * BIN_NUM_CU && 3 * per_band * fewer >= 4 * BIN_NUM_CU &&
            (dense ? fewer >= 2 : fewer <= 3) && (g.ho + fewer - 1) / fewer <= tallest) {
            const BinGeom before = g;
            set_rows((g.ho + fewer - 1) / fewer);
            if (g.fused_ok < before.fused_ok) g = before;
        }
        // Layers that leave compute units empty even so: bands of down to half a tile of 32 positions, as long as that does not
        // cost the single launch.  A step stages and lists as much again for it, which few K steps do not repay.  (us a step, 2 / 5 / 10
        // % of the values flipping, without and so: 72 K steps, one stream of 14 x 14, 512 -> 512, 8.9 / 8.8 / 10.2 and 7.4 / 7.3 / 7.6; two
        // of 28 x 28, 512 -> 256, 10.4 / 10.7 / 11.2 and 9.8 / 9.9 / 10.1; 36, one of 28 x 28, 256 -> 256, 7.1 / 7.8 / 8.1 and 7.1 / 7.3 / 7.4,
        // but two 7.9 / 8.2 / 8.3 and 8.5 / 8.7 / 8.8; 18, two of 28 x 28, 128 -> 256, 7.3 / 7.4 / 7.6 and 8.1 / 8.3 / 8.3; 4, 256 -> 256 1 x
        // 1, 7.3 / 7.3 / 7.4 and 8.0 / 8.1 / 8.2.  Dense: 14 x 14, 512 -> 512, 9.1 and 7.4; 56 x 56, 128 -> 256, 10.2 and 7.5)
        if (per_band * g.nbands < BIN_NUM_CU && (dense || s.kh * s.kw * 2 * g.nslab >= 32)) {
            const BinGeom before = g;
            cut(BIN_NUM_CU, 1, 16);
            if (g.fused_ok < before.fused_ok) g = before;
        }
    }
    if ((long long)g.n * g.nbands > 65535) g.band_rows = 0;  // (stream x band is the grid's z dimension)
    g.magic_nslab = bin_magic_for(g.nslab);
    g.bth_in = ((g.band_rows > 1 ? g.band_rows : 1) - 1) * s.stride + s.kh;
    g.btw_in = (g.wo - 1) * s.stride + s.kw;
    if (g.band_rows == 0) g.fused_ok = 0;
    g.magic_btw = bin_magic_for(g.btw_in);
    g.magic_nbands = bin_magic_for(g.nbands);
    g.magic_nblk = bin_magic_for((g.og + 63) / 64);
    g.magic_nblk32 = bin_magic_for((g.og + 31) / 32);
    g.magic_wo = bin_magic_for(g.wo);
    return true;
}

}  // namespace rrm
