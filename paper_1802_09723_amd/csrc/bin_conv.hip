// Binary (XNOR / popcount) convolution for +1/-1 weights and activations bit-packed along channels.
//
// Sec. 4.3 (XNOR-Net paragraph): after the difference of two +1/-1 frames the surviving entries are
// all +2 or -2, so the delta convolution keeps the binary form up to a constant factor.  With
// m = x_t XOR x_{t-1} (the flip mask) and bit 1 = +1, a flipped input contributes w * 2*x_t, i.e.
//      dP = 2 * ( popc(m) - 2 * popc( m & (w XOR x_t) ) )          summed over the window's words.
// The dense layer (Eq. 3) is the same expression with m = "tap inside the image" and factor 1:
//      P  = b + popc(m) - 2 * popc( m & (w XOR x) ).
// Per lane and 32 inputs this is one v_bfi_b32 ((w & B) | (~w & A) with A = m & x, B = m & ~x, which
// equals m & (w XOR x)) and one v_bcnt_u32_b32 with accumulate: plain vector ALU work, no matrix core (the tile
// kernel).  The band kernel multiplies on the matrix cores instead (see there).
//
// Mapping of the tile kernel (layers without bands, and the dense layer of some that have them, see bin_shape.h): one
// workgroup = one 8x8 output tile (lane = output position) x 4*CW output channels (wavefront w owns CW of
// them); the filter words of an output channel are wave-uniform and come through scalar loads.  A/B words of
// the tile's input window are staged in LDS once; (slab, tap) pairs in which no lane of the wavefront has a
// flipped bit are skipped.
//
// Mapping of the band kernel (the delta step, and the dense layer): one workgroup = a band of output rows of one stream x 64 output
// channels.  It stages the band's input window (the flip mask m and the flips to -1, m & ~x, see pack_e2m1), notes in bits which
// input positions hold a flip, lists the output positions whose window sees one (ballot compaction into LDS) and multiplies that
// list 32 or 64 entries at a time: every column of the product is an output position with work to do, wherever in the band it
// lies, so the work follows the changed positions instead of the 8x8 tiles they fall into.
#include <algorithm>
#include <mutex>

#include "rrm_internal.h"

namespace rrm {

namespace {

constexpr int BAND_THREADS = 64 * BAND_WAVES;  // the band kernel's workgroup

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// Workgroup barrier that publishes LDS contents only (__syncthreads() would also wait for the filter fragments)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// t + popcount(v) in one instruction (v_bcnt_u32_b32 adds its second operand; the compiler otherwise counts
// into a fresh register and adds pairs of counts with a third instruction)
__device__ __forceinline__ int popc_acc(unsigned int v, int t) {
    int r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(v), "v"(t));
    return r;
}

template <int MODE, int CW>
__global__ __launch_bounds__(256) void bin_conv_kernel(const unsigned int* __restrict__ xsrc,
                                                       const unsigned int* __restrict__ flip,
                                                       unsigned int* tileflag,
                                                       const uint4* __restrict__ wpack, const int* __restrict__ bias,
                                                       int* y, BinGeom g, DevStats* __restrict__ stats) {
    extern __shared__ uint4 smem[];
    unsigned int* A = reinterpret_cast<unsigned int*>(smem);
    const int npos = g.th_in * g.tw_in;
    unsigned int* B = A + npos * g.pitch;
    __shared__ unsigned int s_flag;

    const int tile = blockIdx.x;
    if (MODE == MODE_DELTA) {
        // the stamp counts the workgroups that still have to consume this tile (see scan.hip)
        if (threadIdx.x == 0) {
            const unsigned int f = tileflag[tile];
            if (f) {
                atomicSub(&tileflag[tile], 1u);
                if (blockIdx.y == 0) atomicAdd(&stats[tile & (STAT_SLOTS - 1)].active_tiles, 1ull);
            }
            s_flag = f;
        }
        __syncthreads();
        if (s_flag == 0) return;
    }
    const int tiles_per_img = g.tiles_y * g.tiles_x;
    const int b = tile / tiles_per_img;
    const int trem = tile - b * tiles_per_img;
    const int ty = trem / g.tiles_x, tx = trem - ty * g.tiles_x;
    const int nblk = (g.og + 4 * CW - 1) / (4 * CW);
    const int grp = blockIdx.y / nblk;
    const int blk = blockIdx.y - grp * nblk;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int iy0 = ty * TILE * g.stride - g.pad, ix0 = tx * TILE * g.stride - g.pad;
    const int wg4 = g.nslab * 4;

    // ---- stage A = m & x and B = m & ~x of the input window -------------------------------------
    const int units = npos * wg4;
    for (int u = tid; u < units; u += 256) {
        const int hp = (int)(g.magic_wg4 ? __umulhi((unsigned int)u, g.magic_wg4) : (unsigned int)u), wd = u - hp * wg4;
        const int hy = (int)(g.magic_tw ? __umulhi((unsigned int)hp, g.magic_tw) : (unsigned int)hp), hx = hp - hy * g.tw_in;
        const int iy = iy0 + hy, ix = ix0 + hx;
        unsigned int m = 0, xv = 0;
        if (wd < g.wg && iy >= 0 && iy < g.h && ix >= 0 && ix < g.w) {
            const long long wi = (((long long)b * g.h + iy) * g.w + ix) * g.wpp + (long long)grp * g.wg + wd;
            m = MODE == MODE_DELTA ? flip[wi] : 0xFFFFFFFFu;  // the flip buffer is zero where nothing changed
            if (m) xv = xsrc[wi];
        }
        A[hp * g.pitch + wd] = m & xv;
        B[hp * g.pitch + wd] = m & ~xv;
    }
    __syncthreads();

    const int py = lane >> 3, px = lane & 7;
    const int lbase = ((py * g.stride) * g.tw_in + px * g.stride) * g.pitch;
    const int co_w = blk * 4 * CW + wave * CW;  // first output channel of this wavefront in the group
    if (co_w >= g.og) return;
    const int ntaps = g.kh * g.kw;
    int tot[CW];
#pragma unroll
    for (int o = 0; o < CW; ++o) tot[o] = 0;
    int popm = 0;
    // filter words: [group][co/8][slab][tap][co%8] uint4, co padded to a multiple of 16 per group
    const long long ob8 = (long long)grp * g.nob8 + co_w / 8;
    for (int slab = 0; slab < g.nslab; ++slab) {
        for (int tap = 0; tap < ntaps; ++tap) {
            const int ky = tap / g.kw, kx = tap - ky * g.kw;
            const int off = lbase + (ky * g.tw_in + kx) * g.pitch + slab * 4;
            const uint4 a = *reinterpret_cast<const uint4*>(A + off);
            const uint4 bb = *reinterpret_cast<const uint4*>(B + off);
            const unsigned int any = a.x | a.y | a.z | a.w | bb.x | bb.y | bb.z | bb.w;
            if (__ballot(any != 0u) == 0ull) continue;  // wave-uniform: nothing flipped under this tap
            popm += __popc(a.x | bb.x) + __popc(a.y | bb.y) + __popc(a.z | bb.z) + __popc(a.w | bb.w);
#pragma unroll
            for (int o8 = 0; o8 < CW / 8; ++o8) {
                const uint4* wp = wpack + (((ob8 + o8) * g.nslab + slab) * ntaps + tap) * 8;
#pragma unroll
                for (int o = 0; o < 8; ++o) {
                    const uint4 w = wp[o];
                    int t = tot[o8 * 8 + o];
                    t = popc_acc((w.x & bb.x) | (~w.x & a.x), t);
                    t = popc_acc((w.y & bb.y) | (~w.y & a.y), t);
                    t = popc_acc((w.z & bb.z) | (~w.z & a.z), t);
                    t = popc_acc((w.w & bb.w) | (~w.w & a.w), t);
                    tot[o8 * 8 + o] = t;
                }
            }
        }
    }
    // ---- epilogue ---------------------------------------------------------------------------------
    const int oy = ty * TILE + py, ox = tx * TILE + px;
    if (oy >= g.ho || ox >= g.wo) return;
    if (MODE == MODE_DELTA && popm == 0) return;
    const long long ybase = (((long long)b * g.ho + oy) * g.wo + ox) * g.c_out + (long long)grp * g.og + co_w;
    const bool vec = (g.c_out & 3) == 0 && (g.og & 3) == 0;
#pragma unroll
    for (int o4 = 0; o4 < CW / 4; ++o4) {
        int r[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int v = popm - 2 * tot[o4 * 4 + k];
            r[k] = MODE == MODE_DELTA ? 2 * v : v;
        }
        const int co = co_w + o4 * 4;
        if (co >= g.og) break;
        if (vec && co + 3 < g.og) {
            int4* p = reinterpret_cast<int4*>(y + ybase + o4 * 4);
            int4 o;
            if (MODE == MODE_DELTA) {
                o = *p;
                o.x += r[0]; o.y += r[1]; o.z += r[2]; o.w += r[3];
            } else {
                const int bo = grp * g.og + co;
                o.x = r[0] + (bias ? bias[bo] : 0);
                o.y = r[1] + (bias ? bias[bo + 1] : 0);
                o.z = r[2] + (bias ? bias[bo + 2] : 0);
                o.w = r[3] + (bias ? bias[bo + 3] : 0);
            }
            *p = o;
        } else {
            for (int k = 0; k < 4 && co + k < g.og; ++k) {
                if (MODE == MODE_DELTA)
                    y[ybase + o4 * 4 + k] += r[k];
                else
                    y[ybase + o4 * 4 + k] = r[k] + (bias ? bias[grp * g.og + co + k] : 0);
            }
        }
    }
}

// ---- the band kernel's product ------------------------------------------------------------------------------------
// Half of a difference of two +1/-1 frames is -1, 0 or +1, which the 4-bit float format of the matrix cores (E2M1)
// holds exactly, like the weights; the products are summed in fp32, exact below 2^24 terms (a band's window in LDS
// holds far fewer).  v_mfma_f32_32x32x64_f8f6f4 multiplies 32 output channels x 32 listed positions x 64 input
// channels of one tap in 32 cycles, where the popcount form takes 256 vector cycles.
// Measured (28 x 28, 256 -> 256 channels, 64 streams, 5 % of the values flipping): 36.8 us a step with popcounts, 23.0 with weights
// fetched as nibbles (16 bytes a lane, K step and 32 channels: what the vector cache delivers per clock was the bound), 21.0 so, 19.3 with
// the steps' table;
// one stream of 14 x 14, 512 -> 512 channels, 10 %: 16.8, 10.3 and 7.4 (6.3 with shorter lists and the steps' table).
//
// 32 values of a word are 4 registers of E2M1 nibbles; nibble j of register i is value 4 j + (1, 0, 3, 2)[i].  Of a difference
// (0x2 = +1, 0xA = -1, 0x0 = unchanged) only the bits 1 and 3 are ever set, so two registers lie in one word of LDS, the second one
// a bit lower, as the flip mask m and the flips to -1, q, give them in two instructions each; of a weight (0x2 or 0xA) one bit is
// kept, and a wavefront holds all of its steps' in registers.
__device__ __forceinline__ uint2 pack_e2m1(unsigned int m, unsigned int q) {
    const unsigned int M = 0x33333333u;
    return make_uint2((m & M) | (q << 2 & ~M), (m >> 2 & M) | (q & ~M));
}
__device__ __forceinline__ v8i difference_e2m1(const uint2& p) {
    const unsigned int K = 0xAAAAAAAAu;
    return v8i{(int)(p.x & K), (int)(p.x << 1 & K), (int)(p.y & K), (int)(p.y << 1 & K), 0, 0, 0, 0};
}
__device__ __forceinline__ v8i weights_e2m1(unsigned int minus) {  // `minus`: a bit per value of -1
    const unsigned int P = 0x22222222u, N = 0x88888888u;
    return v8i{(int)((minus << 2 & N) | P), (int)((minus << 3 & N) | P), (int)((minus & N) | P), (int)((minus << 1 & N) | P), 0, 0, 0, 0};
}

__device__ __forceinline__ v16f mma_e2m1(const v8i& a, const v8i& b, v16f c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 4, 4, 0, 0, 0, 0);  // E2M1 x E2M1, unscaled
}

// FUSED: the whole step in this one launch.  `xsrc` is the new frame x_t and `flip` the stored input: the flip
// mask is their XOR, formed while the window is staged (no difference kernel, no flip buffer); the change counts
// are taken over the input rows a band owns; and the workgroup of a stream that finishes staging last (arrival
// counter) copies the frame into the stored input, when nobody reads the old one any more, and rearms the counter.
//
// DENSE: the layer itself (Eq. 3) with the same product: m = "tap inside the image", every output position is listed, and
// the result is the bias plus the sums.  (`flip` and `stats` are not touched.)  60 x 13, 448 -> 72 channels, 26 streams: 40.9 us on the tile
// kernel, 28.6 here.
//
// TILES > 0: a pass is 32 * TILES listed positions x 64 channels.  The wavefronts of a tile of 32 positions split the K steps (a
// tap, 64 channels): a wavefront takes steps kpart, kpart + KPARTS, ... and adds its sums in LDS.  The weights of KU of its steps
// are in registers at a time (they do not depend on the list: they are fetched ahead of it) and are replaced one by one as they
// are used; if that is all of them, they stay for every pass.
// TILES = 0: no pass and no sums in LDS; a wavefront takes tiles with all of their K steps.  For long lists, where there are
// tiles for all wavefronts.
template <bool FUSED, bool DENSE, int TILES, int KU, int CB>
__global__ __launch_bounds__(BAND_THREADS, 4) void bin_band_kernel(const unsigned int* __restrict__ xsrc,
                                                       const unsigned int* flip, unsigned int* snap,
                                                       unsigned int* arrive,
                                                       const uint2* __restrict__ wband, const int* __restrict__ bias,
                                                       int* y, BinGeom g, DevStats* __restrict__ stats) {
    // (Not where two workgroups share a compute unit: 12 x 43, 256 -> 480, 13 streams, 10.9 us a step without and 11.1 so, 8 x 22, 64 -> 164, 56
    // streams, 10.65 and 10.8; 35 x 35, 384 -> 144 5 x 5 dense, two streams, 11.65 and 11.8)
    if (TILES == 1) fetch_args<7 * sizeof(void*) + sizeof(BinGeom) + sizeof(void*)>();
    constexpr int KPARTS = TILES > 0 ? BAND_WAVES / TILES : 1, PASS = 32 * TILES;
    constexpr int CPT = 4 * TILES;  // channels per thread of a pass' results (CB = 1: half of the threads have none)
    extern __shared__ uint4 smem[];
    const int npos = g.bth_in * g.btw_in;
    // The mask m and the flips to -1, m & ~x, of a word lie side by side, and a position's words at an odd pitch of such pairs
    // (except in wide layers, without padding): the 32 lanes of a read are 32 positions and meet no bank twice.
    const int ip = bin_pair_pitch(g);
    uint2* AB = reinterpret_cast<uint2*>(smem);
    // a bit per input position that holds a flip, rows of whole words (with the padding saved above they take no more than a
    // byte per position)
    const int bw = (g.btw_in + 31) >> 5;
    unsigned int* bits = reinterpret_cast<unsigned int*>(AB + npos * ip);
    unsigned short* list = reinterpret_cast<unsigned short*>(reinterpret_cast<unsigned char*>(smem) + bin_band_list_offset(g));  // active output positions
    // sums of a pass: PASS positions x 64 channels, rows padded by one word
    int* red = reinterpret_cast<int*>(reinterpret_cast<unsigned char*>(list) + (((size_t)g.band_rows * g.wo * 2 + 15) & ~(size_t)15));
    __shared__ unsigned int s_wc[BAND_WAVES], s_prev;

    // grid: x = list split (fastest, so the workgroups that share a band start together), y = channel block,
    // z = stream x band
    const int sb = (int)blockIdx.z, zsplit = (int)blockIdx.x, nsplit = g.nsplit;
    const int b = (int)udiv_magic((unsigned int)sb, (unsigned int)g.nbands, g.magic_nbands), band = sb - b * g.nbands;
    const int nblk = (g.og + 32 * CB - 1) / (32 * CB);
    const int grp = (int)udiv_magic(blockIdx.y, (unsigned int)nblk, CB == 2 ? g.magic_nblk : g.magic_nblk32);
    const int blk = blockIdx.y - grp * nblk;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int oy0 = band * g.band_rows;
    const int rows = min(g.band_rows, g.ho - oy0);
    const int iy0 = oy0 * g.stride - g.pad, ix0 = -g.pad;
    const int wg4 = g.nslab * 4;

    const int ntaps = g.kh * g.kw, nkt = 2 * g.nslab, nk = ntaps * nkt;  // K steps per tap, in all
    const int n = lane & 31, khalf = lane >> 5;
    // (the weights are packed for blocks of 64)
    const uint2* wfrag = wband + (long long)(CB == 2 ? grp * nblk + blk : grp * ((g.og + 63) >> 6) + (blk >> 1)) * nk * 64 + lane;
    const int kpart = TILES > 0 ? wave & (KPARTS - 1) : 0, tile = wave / KPARTS;
    unsigned int w[KU][CB];  // of a step: the lane's word of the block's channels 0 .. 31 and 32 .. 63
    auto fetch_w = [&](unsigned int (&f)[CB], int k) __attribute__((always_inline)) {
        if constexpr (CB == 2) {
            const uint2 v = wfrag[(long long)k * 64];
            f[0] = v.x;
            f[1] = v.y;
        } else {
            f[0] = reinterpret_cast<const unsigned int*>(wfrag + (long long)k * 64)[blk & 1];
        }
    };
    // (FUSED) input rows whose changes this band counts, by the workgroup of the band's first channel block
    const int own_lo = oy0 * g.stride, own_hi = band == g.nbands - 1 ? g.h : (oy0 + g.band_rows) * g.stride;
    const bool count_here = FUSED && blk == 0 && zsplit == 0;
    unsigned int nbits = 0, nunits = 0, arrived_before = 0;
    auto clear_lds = [&]() __attribute__((always_inline)) {
        for (int i = tid; i < g.bth_in * bw; i += BAND_THREADS) bits[i] = 0;
        for (int i = tid; i < PASS * BAND_RP; i += BAND_THREADS) red[i] = 0;
    };
    // Where the wavefront's K steps lie in a window, from a table, a lane each (up to 64 of them).  Worked out, it was a chain of some
    // twenty scalar instructions a step that every pass waited for (a dependent instruction takes 8 cycles): with the table, 14 x 14, 512 ->
    // 512, 10 %, 64 streams, 24.6 -> 21.7 us a step, one stream 7.5 -> 6.9; 28 x 28, 448 -> 256 dense, 8 streams, 16.6 -> 14.5.
    int at0 = 0;
    auto first_frags = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < KU; ++i) fetch_w(w[i], min(kpart + i * KPARTS, nk - 1));
    };
    // What does not depend on the staged window, while its loads are on their way.  The weights and the table too where a compute unit
    // has one workgroup.  Where two share it they are fetched after the window, which they would hold up: the weights 28 x 28, 256 -> 256, 8
    // streams, 10.1 us and 10.9 so; the table, a load on its way through the loop that stages, 36 x 36, 256 -> 184 1 x 1, 59 streams, 16.9 and
    // 18.0 (17.0 before there was a table), 28 x 28, 128 -> 109, 30 streams, 14.2 and 15.1, 28 x 28, 256 -> 256, 64 streams, 19.3 and 20.5.
    auto fetch_first = [&]() __attribute__((always_inline)) {
        at0 = g.steps[min(kpart + lane * KPARTS, nk - 1)];
        first_frags();
    };
    auto ahead = [&]() __attribute__((always_inline)) {
        clear_lds();
        if (TILES == 1) fetch_first();
        lds_barrier();
    };
    // ---- stage m and m & ~x of the band's input window ----------------------------------------
    if (g.vec4) {
        // four words at a time, BATCH of them in flight per thread
        constexpr int BATCH = 4;
        const int units = npos * g.nslab;
        for (int u0 = 0; u0 < units; u0 += BATCH * BAND_THREADS) {
            uint4 m[BATCH], xv[BATCH];
            int hy[BATCH], hx[BATCH];
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                m[i] = xv[i] = make_uint4(0, 0, 0, 0);
                if (u0 + i * BAND_THREADS >= units) continue;
                const int u = u0 + i * BAND_THREADS + tid;
                const int hp = (int)udiv_magic((unsigned int)u, (unsigned int)g.nslab, g.magic_nslab), sl = u - hp * g.nslab;
                hy[i] = (int)udiv_magic((unsigned int)hp, (unsigned int)g.btw_in, g.magic_btw);
                hx[i] = hp - hy[i] * g.btw_in;
                const int iy = iy0 + hy[i], ix = ix0 + hx[i];
                if (u < units && iy >= 0 && iy < g.h && ix >= 0 && ix < g.w) {
                    const long long wi = (((long long)b * g.h + iy) * g.w + ix) * g.wpp + (long long)grp * g.wg + sl * 4;
                    m[i] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
                    if (!DENSE) m[i] = *reinterpret_cast<const uint4*>(flip + wi);  // the flip buffer is zero where nothing changed
                    xv[i] = *reinterpret_cast<const uint4*>(xsrc + wi);
                }
            }
            if (u0 == 0) ahead();
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int u = u0 + i * BAND_THREADS + tid;
                if (u >= units) break;
                const int hp = hy[i] * g.btw_in + hx[i], sl = u - hp * g.nslab, iy = iy0 + hy[i];
                uint4 f = m[i];
                const uint4 x = xv[i];
                if (FUSED) {  // (outside of the frame both are zero)
                    f = make_uint4(f.x ^ x.x, f.y ^ x.y, f.z ^ x.z, f.w ^ x.w);
                    if (count_here && iy >= own_lo && iy < own_hi && (f.x | f.y | f.z | f.w)) {
                        nbits += __popc(f.x) + __popc(f.y) + __popc(f.z) + __popc(f.w);
                        ++nunits;
                    }
                }
                if (!DENSE && (f.x | f.y | f.z | f.w)) atomicOr(&bits[hy[i] * bw + (hx[i] >> 5)], 1u << (hx[i] & 31));
                uint2* d = AB + hp * ip + sl * 4;
                d[0] = pack_e2m1(f.x, f.x & ~x.x);
                d[1] = pack_e2m1(f.y, f.y & ~x.y);
                d[2] = pack_e2m1(f.z, f.z & ~x.z);
                d[3] = pack_e2m1(f.w, f.w & ~x.w);
            }
        }
    } else {
        // a word at a time, BATCH of them in flight per thread
        constexpr int BATCH = 4;
        const int units = npos * wg4;
        for (int u0 = 0; u0 < units; u0 += BATCH * BAND_THREADS) {
            unsigned int m[BATCH], xv[BATCH], at[BATCH];  // at: input position (row, column) of the word
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                m[i] = xv[i] = at[i] = 0;
                if (u0 + i * BAND_THREADS >= units) continue;
                const int u = u0 + i * BAND_THREADS + tid;
                const int hp = (int)udiv_magic((unsigned int)u, (unsigned int)wg4, g.magic_wg4), wd = u - hp * wg4;
                const int hy = (int)udiv_magic((unsigned int)hp, (unsigned int)g.btw_in, g.magic_btw), hx = hp - hy * g.btw_in;
                const int iy = iy0 + hy, ix = ix0 + hx;
                at[i] = (unsigned int)hy << 16 | (unsigned int)hx;
                if (u < units && wd < g.wg && iy >= 0 && iy < g.h && ix >= 0 && ix < g.w) {
                    const long long wi = (((long long)b * g.h + iy) * g.w + ix) * g.wpp + (long long)grp * g.wg + wd;
                    m[i] = DENSE ? 0xFFFFFFFFu : flip[wi];  // the flip buffer is zero where nothing changed
                    xv[i] = xsrc[wi];
                }
            }
            if (u0 == 0) ahead();
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int u = u0 + i * BAND_THREADS + tid;
                if (u >= units) break;
                const int hy = (int)(at[i] >> 16), hx = (int)(at[i] & 0xFFFFu), hp = hy * g.btw_in + hx;
                if (!DENSE && m[i]) atomicOr(&bits[hy * bw + (hx >> 5)], 1u << (hx & 31));
                AB[hp * ip + u - hp * wg4] = pack_e2m1(m[i], m[i] & ~xv[i]);
            }
        }
    }
    lds_barrier();
    if (TILES > 1) fetch_first();
    // this workgroup has read the stored input for the last time
    // (thread 0 keeps the answer to the end: stored at once, it would hold up the list by a memory round trip)
    if (FUSED && tid == 0) arrived_before = atomicAdd(&arrive[b], 1u);
    // ---- list the output positions of the band whose window holds a flip ------------------------
    const int nout = rows * g.wo;
    int cnt = 0;
    if (DENSE) {
        for (int q = tid; q < nout; q += BAND_THREADS) list[q] = (unsigned short)q;
        cnt = nout;
        lds_barrier();
    }
    // (up to 64 outputs: every wavefront makes the list for itself, and all of them the same one, so that none waits for another: 14 x
    // 14, 512 -> 512, one stream, 1.0 -> 0.55 us from the staged window to the list)
    const bool short_list = nout <= 64;
    for (int base = 0; !DENSE && base < nout; base += BAND_THREADS) {
        const int q = short_list ? lane : base + tid;
        bool act = false;
        if (q < nout) {
            const int oyl = (int)udiv_magic((unsigned int)q, (unsigned int)g.wo, g.magic_wo), x0 = (q - oyl * g.wo) * g.stride;
            const unsigned int* row = bits + (oyl * g.stride) * bw;
            if (g.kw <= 32) {
                // the window's columns lie in one or two words of a row; four rows in flight
                const int i0 = x0 >> 5, i1 = min(i0 + 1, bw - 1), sh = x0 & 31;
                unsigned long long any = 0;
                for (int ky = 0; ky < g.kh; ky += 4) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const unsigned int* r = row + min(ky + k, g.kh - 1) * bw;
                        any |= (unsigned long long)r[i1] << 32 | r[i0];
                    }
                }
                act = ((unsigned int)(any >> sh) << (32 - g.kw)) != 0;
            } else {
                for (int ky = 0; ky < g.kh; ++ky)
                    for (int kx = x0; kx < x0 + g.kw; ++kx) act |= (row[ky * bw + (kx >> 5)] >> (kx & 31) & 1u) != 0;
            }
        }
        // (the same order in every workgroup of the band: the workgroups of a list split deal its chunks among them)
        const unsigned long long mask = __ballot(act);
        if (short_list) {
            if (act) list[__popcll(mask & ((1ull << lane) - 1ull))] = (unsigned short)q;
            cnt = (int)__popcll(mask);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // LDS operations of one wavefront execute in order
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            break;
        }
        if (lane == 0) s_wc[wave] = (unsigned int)__popcll(mask);
        lds_barrier();
        unsigned int wbase = (unsigned int)cnt, all = 0;
#pragma unroll
        for (int k = 0; k < BAND_WAVES; ++k) {
            const unsigned int c = s_wc[k];
            if (k < wave) wbase += c;
            all += c;
        }
        if (act) list[wbase + __popcll(mask & ((1ull << lane) - 1ull))] = (unsigned short)q;
        cnt += (int)all;
        lds_barrier();  // (the counts are overwritten in the next round; after the last one: the list is complete)
    }

    const bool vec = (g.c_out & 3) == 0 && (g.og & 3) == 0;
    // y[0 .. 3] of a position and four channels that start at channel `ch` of the group
    auto load4 = [&](const int* yp, int ch) __attribute__((always_inline)) {
        if (vec) return *reinterpret_cast<const int4*>(yp);
        return make_int4(yp[0], ch + 1 < g.og ? yp[1] : 0, ch + 2 < g.og ? yp[2] : 0, ch + 3 < g.og ? yp[3] : 0);
    };
    auto store4 = [&](int* yp, int ch, const int4& v) __attribute__((always_inline)) {
        if (vec) {
            *reinterpret_cast<int4*>(yp) = v;
            return;
        }
        yp[0] = v.x;
        if (ch + 1 < g.og) yp[1] = v.y;
        if (ch + 2 < g.og) yp[2] = v.z;
        if (ch + 3 < g.og) yp[3] = v.w;
    };
    const int bch = blk * 32 * CB;  // the block's first channel of the group
    auto y_at = [&](int q) __attribute__((always_inline)) {  // ... at a listed position
        const int oyl = (int)udiv_magic((unsigned int)q, (unsigned int)g.wo, g.magic_wo);
        return y + ((((long long)b * g.ho + oy0 + oyl) * g.wo + (q - oyl * g.wo)) * g.c_out + (long long)grp * g.og + bch);
    };
    auto window_at = [&](int q) __attribute__((always_inline)) {
        const int oyl = (int)udiv_magic((unsigned int)q, (unsigned int)g.wo, g.magic_wo);
        return AB + ((oyl * g.stride) * g.btw_in + (q - oyl * g.wo) * g.stride) * ip + khalf;
    };
    if constexpr (TILES > 0) {
        // The list in passes of PASS entries, dealt to the workgroups of a list split.
        constexpr int PT = 32 * CB / CPT;  // threads per position of the results
        const int el = tid / PT, j4 = (tid & (PT - 1)) * TILES;
        const bool mine = CB == 2 || el < PASS;
        for (int first = zsplit * PASS; first < cnt; first += nsplit * PASS) {
            const bool more = first + nsplit * PASS < cnt;
            // this thread's part of the pass' results: one position, CPT channels; fetched now, needed at the end
            const int e = first + el;
            const bool out = mine && e < cnt;
            int* yp = y_at(list[out ? e : 0]) + 4 * j4;
            int4 yv[TILES];
#pragma unroll
            for (int h = 0; h < TILES; ++h) {
                const int ch = bch + 4 * (j4 + h);
                yv[h] = make_int4(0, 0, 0, 0);
                const int* add = DENSE ? (bias ? bias + grp * g.og + ch : nullptr) : yp + 4 * h;
                if (add && out && ch < g.og) yv[h] = load4(add, ch);
            }
            // this lane's column: the window of its listed position (an entry beyond the list repeats its first; its sums are
            // not read)
            const bool work = first + 32 * tile < cnt && kpart < nk;  // (the same in every lane)
            const int ent = first + 32 * tile + n;
            const uint2* lp = window_at(list[ent < cnt ? ent : 0]);
            v16f acc[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[c][r] = 0.f;
            int first_of = 0, at = at0;  // the K step whose place lane 0 holds, past kpart
#pragma unroll 1
            for (int k0 = kpart; work && k0 < nk; k0 += KU * KPARTS) {
                const int i0 = (k0 - kpart) / KPARTS;  // (a power of two)
                if (i0 - first_of + KU > 64) {  // (more than 64 steps a wavefront)
                    first_of = i0;
                    at = g.steps[min(k0 + lane * KPARTS, nk - 1)];
                }
                uint2 ab[KU];
#pragma unroll
                for (int i = 0; i < KU; ++i) ab[i] = lp[__builtin_amdgcn_readlane(at, i0 - first_of + i)];
#pragma unroll
                for (int i = 0; i < KU; ++i) {
                    const int k = k0 + i * KPARTS;
                    if (k < nk) {
                        const v8i d = difference_e2m1(ab[i]);
#pragma unroll
                        for (int c = 0; c < CB; ++c) acc[c] = mma_e2m1(weights_e2m1(w[i][c]), d, acc[c]);
                    }
                    if (nk > KU * KPARTS) {  // the step that comes in this place next, or in the next pass
                        const int kn = k + KU * KPARTS;
                        if (kn < nk || more) fetch_w(w[i], kn < nk ? kn : min(kpart + i * KPARTS, nk - 1));
                    }
                }
            }
            if (work) {
                // columns of a row: [khalf][c][r / 4][r % 4], so that the halves of the wavefront, 32 rows each, meet no bank twice
#pragma unroll
                for (int c = 0; c < CB; ++c)
#pragma unroll
                    for (int r = 0; r < 16; ++r) atomicAdd(&red[(32 * tile + n) * BAND_RP + 32 * khalf + 16 * c + r], (int)acc[c][r]);
            }
            lds_barrier();
#pragma unroll
            for (int h = 0; h < TILES && mine; ++h) {
                const int c4 = j4 + h;  // channels 4 c4 .. of the block: 32 * (c4 / 8) + 8 * (c4 / 2 % 4) + 4 * (c4 % 2)
                int* r = red + el * BAND_RP + 32 * (c4 & 1) + 16 * (c4 >> 3) + 4 * (c4 >> 1 & 3);
                constexpr int F = DENSE ? 1 : 2;
                const int4 v = make_int4(yv[h].x + F * r[0], yv[h].y + F * r[1], yv[h].z + F * r[2], yv[h].w + F * r[3]);
#pragma unroll
                for (int k = 0; k < 4; ++k) r[k] = 0;
                if (out && bch + 4 * c4 < g.og) store4(yp + 4 * h, bch + 4 * c4, v);
            }
            if (more) lds_barrier();  // (the sums are cleared)
        }
    } else {
        // Every wavefront for itself: NT tiles of 32 listed positions x NB blocks of 32 channels, all K steps.
        auto item = [&]<int NT, int NB>(int tile0, int c0) __attribute__((always_inline)) {
            const unsigned int* wf = reinterpret_cast<const unsigned int*>(wfrag) + c0;
            unsigned int w[KU][NB];
            auto fetch_w = [&](unsigned int (&f)[NB], int k) __attribute__((always_inline)) {
                if constexpr (NB == 2) {
                    const uint2 v = wfrag[(long long)k * 64];
                    f[0] = v.x;
                    f[1] = v.y;
                } else {
                    f[0] = wf[(long long)k * 128];
                }
            };
#pragma unroll
            for (int i = 0; i < KU; ++i) fetch_w(w[i], min(i, nk - 1));
            int q[NT];
            const uint2* lp[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int ent = (tile0 + t) * 32 + n;
                q[t] = list[ent < cnt ? ent : 0];
                lp[t] = window_at(q[t]);
            }
            v16f acc[NT][NB];
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int c = 0; c < NB; ++c)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[t][c][r] = 0.f;
            int off = 0, st = 0, kx = 0;  // of the next step to read
#pragma unroll 1
            for (int k0 = 0; k0 < nk; k0 += KU) {
#pragma unroll
                for (int j = 0; j < KU; j += 3) {
                    uint2 ab[3][NT];
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
#pragma unroll
                        for (int t = 0; t < NT; ++t) ab[i][t] = lp[t][off];
                        if (k0 + j + i + 1 < nk) {
                            off += 2;
                            if (++st == nkt) {
                                st = 0;
                                off += ip - 2 * nkt;
                                if (++kx == g.kw) {
                                    kx = 0;
                                    off += (g.btw_in - g.kw) * ip;
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const int k = k0 + j + i;
                        if (k >= nk) break;
                        v8i wc[NB];
#pragma unroll
                        for (int c = 0; c < NB; ++c) wc[c] = weights_e2m1(w[j + i][c]);
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            const v8i d = difference_e2m1(ab[i][t]);
#pragma unroll
                            for (int c = 0; c < NB; ++c) acc[t][c] = mma_e2m1(wc[c], d, acc[t][c]);
                        }
                        if (k + KU < nk) fetch_w(w[j + i], k + KU);
                    }
                }
            }
            // a lane holds channels 8 * (r / 4) + 4 * khalf + r % 4 of each block, at one position of each tile
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if ((tile0 + t) * 32 + n >= cnt) continue;
                int* yp = y_at(q[t]);
                int4 yv[NB][4];
#pragma unroll
                for (int c = 0; c < NB; ++c)
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        const int ch = 32 * (c0 + c) + 8 * h + 4 * khalf;
                        yv[c][h] = make_int4(0, 0, 0, 0);
                        const int* add = DENSE ? (bias ? bias + grp * g.og + bch + ch : nullptr) : yp + ch;
                        if (add && bch + ch < g.og) yv[c][h] = load4(add, bch + ch);
                    }
#pragma unroll
                for (int c = 0; c < NB; ++c)
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        const int ch = 32 * (c0 + c) + 8 * h + 4 * khalf;
                        constexpr int F = DENSE ? 1 : 2;
                        const v16f& s = acc[t][c];
                        if (bch + ch < g.og)
                            store4(yp + ch, bch + ch, make_int4(yv[c][h].x + F * (int)s[4 * h], yv[c][h].y + F * (int)s[4 * h + 1],
                                                                yv[c][h].z + F * (int)s[4 * h + 2], yv[c][h].w + F * (int)s[4 * h + 3]));
                    }
            }
        };
        const int ntile = (cnt + 31) >> 5, nb = g.og - bch > 32 ? 2 : 1;
        if (nb == 1 || 2 * ntile <= BAND_WAVES) {
            for (int i = wave; i < nb * ntile; i += BAND_WAVES) item.template operator()<1, 1>(nb == 1 ? i : i >> 1, nb == 1 ? 0 : i & 1);
        } else if (ntile <= BAND_WAVES) {
            if (wave < ntile) item.template operator()<1, 2>(wave, 0);
        } else {
            for (int i = wave; 2 * i < ntile; i += BAND_WAVES) item.template operator()<2, 2>(2 * i, 0);
        }
    }
    if (FUSED) {
        if (tid == 0) s_prev = arrived_before;
        if (count_here && __any(nunits != 0)) {
            nbits = wave_scan(nbits);
            nunits = wave_scan(nunits);
            if (lane == 63) {
                atomicAdd(&stats[sb & (STAT_SLOTS - 1)].changed_elems, (unsigned long long)nbits);
                atomicAdd(&stats[sb & (STAT_SLOTS - 1)].changed_units, (unsigned long long)nunits);
            }
        }
        if (sb == 0 && blockIdx.y == 0 && zsplit == 0 && tid == 0) {  // one launch = one delta step
            atomicAdd(&stats[0].delta_steps, 1ull);
            atomicAdd(&stats[0].total_tiles, (unsigned long long)g.n * g.ho * g.wo);
        }
    }
    if (!DENSE && cnt > 0 && blockIdx.y == 0 && zsplit == 0 && tid == 0)
        atomicAdd(&stats[sb & (STAT_SLOTS - 1)].active_tiles, (unsigned long long)cnt);
    if (FUSED) {
        // commit: the stream's last workgroup to finish staging
        lds_barrier();
        if (s_prev == (unsigned int)(g.nbands * g.groups * nblk * nsplit) - 1u) {
            const long long words = (long long)g.h * g.w * g.wpp;  // (a multiple of four: whole 16-byte vectors)
            const uint4* src = reinterpret_cast<const uint4*>(xsrc + (long long)b * words);
            uint4* dst = reinterpret_cast<uint4*>(snap + (long long)b * words);
            for (long long i = tid; i < words / 4; i += BAND_THREADS) dst[i] = src[i];
            if (tid == 0) arrive[b] = 0u;
        }
    }
}

template <int MODE, int CW>
hipError_t launch_one(const void* xsrc, const void* flip, unsigned int* tileflag, const void* wpack,
                      const void* bias, void* y, const BinGeom& g, DevStats* stats, hipStream_t s) {
    const int nblk = (g.og + 4 * CW - 1) / (4 * CW);
    dim3 grid((unsigned int)(g.n * g.tiles_y * g.tiles_x), (unsigned int)(g.groups * nblk));
    const size_t lds = (size_t)2 * g.th_in * g.tw_in * g.pitch * sizeof(unsigned int);
    auto kern = bin_conv_kernel<MODE, CW>;
    if (lds > 64 * 1024) {  // (large strided windows; at most BIN_TILE_MAX_LDS, checked at create)
        static std::mutex mu;
        static size_t granted = 0;
        std::lock_guard<std::mutex> lock(mu);
        if (lds > granted) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            granted = lds;
        }
    }
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, s, static_cast<const unsigned int*>(xsrc),
                       static_cast<const unsigned int*>(flip), tileflag,
                       static_cast<const uint4*>(wpack), static_cast<const int*>(bias), static_cast<int*>(y), g,
                       stats);
    return hipGetLastError();
}

}  // namespace

int bin_consumers(int cw, const BinGeom& g) { return g.groups * ((g.og + 4 * cw - 1) / (4 * cw)); }

template <bool FUSED, bool DENSE, int TILES, int KU, int CB = 2>
hipError_t launch_band_form(int z, const void* xsrc, const void* flip, void* snap, unsigned int* arrive, const void* wband, const void* bias,
                            void* y, const BinGeom& geom, DevStats* stats, hipStream_t s) {
    BinGeom g = geom;
    g.nsplit = z;
    dim3 grid((unsigned int)z, (unsigned int)(g.groups * ((g.og + 32 * CB - 1) / (32 * CB))), (unsigned int)(g.n * g.nbands));
    const size_t lds = bin_band_lds_bytes(g, g.band_rows);
    auto kern = bin_band_kernel<FUSED, DENSE, TILES, KU, CB>;
    if (lds > 64 * 1024) {
        static std::mutex mu;
        static size_t granted = 0;
        std::lock_guard<std::mutex> lock(mu);
        if (lds > granted) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            granted = lds;
        }
    }
    hipLaunchKernelGGL(kern, grid, dim3(BAND_THREADS), lds, s, static_cast<const unsigned int*>(xsrc),
                       static_cast<const unsigned int*>(flip), static_cast<unsigned int*>(snap), arrive,
                       static_cast<const uint2*>(wband), static_cast<const int*>(bias), static_cast<int*>(y), g, stats);
    return hipGetLastError();
}

template <bool FUSED, bool DENSE = false>
hipError_t launch_band(const void* xsrc, const void* flip, void* snap, unsigned int* arrive, const void* wband, const void* bias, void* y,
                       const BinGeom& g, DevStats* stats, hipStream_t s) {
    const int nblk = (g.og + 63) / 64;
    const long long wgs = (long long)g.n * g.nbands * g.groups * nblk;
    const int nout = g.band_rows * g.wo;
    // A band of at most 32 outputs (see bin_choose_shape): one tile, its K steps over all eight wavefronts.
    // Where such bands leave compute units empty, blocks of 32 channels: half of the products' and the sums' instructions per wavefront,
    // twice the workgroups that stage, list and count up the stream's arrival word (us a step with 64 and with 32 channels: 14 x 14, one
    // stream, 512 -> 512, 56 workgroups of 64, 6.8 and 6.3; two, 256 -> 256, 56, 6.25 and 6.05; but 28 x 28, 256 -> 256, 112, 7.1 and 7.5; 24 x
    // 24, 256 -> 128, two streams, 96, 7.0 and 7.3.  Dense, no list and no count: 28 x 28 5.35 and 5.05).
    if (nout <= 32 && (DENSE ? 2 : 4) * wgs <= NUM_CU) return launch_band_form<FUSED, DENSE, 1, 9, 1>(1, xsrc, flip, snap, arrive, wband, bias, y, g, stats, s);
    if (nout <= 32 && wgs <= NUM_CU) return launch_band_form<FUSED, DENSE, 1, 9>(1, xsrc, flip, snap, arrive, wband, bias, y, g, stats, s);
    // The dense layer lists all positions: a wavefront has tiles of its own (us with the K steps split and so: 28 x 28, 256 -> 256, 3 x
    // 3, 64 streams, 45.4 and 34.5; 56 x 56, 64 -> 64, 32 streams, 23.3 and 17.8; 112 x 112, 128 -> 128, 5 x 5, 2 streams, 25.1 and
    // 17.8).  Not in a step, whose lists are short and uneven (the first layer, 5 / 20 % changed, 21.0 / 36.3 split and 22.6 / 39.9 so).
    // Nor where workgroups have compute units to spare and a tile alone is a long chain (8 streams, 28 x 28, 448 -> 256,
    // 72 steps, 16.4 split and 17.0; two of 55 x 55, 384 -> 480, 54 steps, 22.6 and 18.5).
    const int nk = g.kh * g.kw * 2 * g.nslab;
    if constexpr (DENSE)
        if (nout > 64 && (wgs > NUM_CU || nk <= 64)) return launch_band_form<FUSED, DENSE, 0, 9>(1, xsrc, flip, snap, arrive, wband, bias, y, g, stats, s);
    // Few streams: deal the band's list over several workgroups, as long as every one has a compute unit to itself: each stages the
    // window and makes the list again, which a second one per compute unit does not repay.
    const int z = std::max(1, (int)std::min((long long)(nout + 63) / 64, (DENSE ? 2 : 1) * NUM_CU / wgs));
    // Weights of five, seven or nine of a wavefront's steps at a time, whichever fetches least that is not used (us with nine and with
    // five, 5 % of the values flipping: 9 steps, the layer above, 21.0 and 22.3; 5 steps, 128 -> 256 channels in two groups, 22.0 and
    // 20.1; 25 steps, 14 x 14, 256 -> 256, 5 x 5, 64 streams, 19.0 and 17.8; with five and with seven: 14 steps, 55 x 55, 384 -> 480, two
    // streams, 18.2 and 17.8.  Eighteen, with a compute unit per workgroup: the last one 20.2).
    const int steps = (nk + 3) / 4;
    auto fetched = [&](int ku) { return (steps + ku - 1) / ku * ku; };
    if (fetched(9) <= std::min(fetched(7), fetched(5)))
        return launch_band_form<FUSED, DENSE, 2, 9>(z, xsrc, flip, snap, arrive, wband, bias, y, g, stats, s);
    if (fetched(7) <= fetched(5)) return launch_band_form<FUSED, DENSE, 2, 7>(z, xsrc, flip, snap, arrive, wband, bias, y, g, stats, s);
    return launch_band_form<FUSED, DENSE, 2, 5>(z, xsrc, flip, snap, arrive, wband, bias, y, g, stats, s);
}

// two launches: xsrc = the stored input after the difference kernel, flip = its flip buffer
hipError_t launch_bin_band(const void* xsrc, const void* flip, const void* wband, void* y, const BinGeom& g,
                           DevStats* stats, hipStream_t s) {
    if (g.band_rows < 1 || g.band_rows * g.wo > 65535) return hipErrorInvalidValue;  // (list entries are 16 bits)
    return launch_band<false>(xsrc, flip, nullptr, nullptr, wband, nullptr, y, g, stats, s);
}

// the dense layer: xsrc = x
hipError_t launch_bin_band_dense(const void* x, const void* wband, const void* bias, void* y, const BinGeom& g, hipStream_t s) {
    if (g.band_rows < 1 || g.band_rows * g.wo > 65535) return hipErrorInvalidValue;  // (list entries are 16 bits)
    return launch_band<false, true>(x, nullptr, nullptr, nullptr, wband, bias, y, g, nullptr, s);
}

// one launch: the whole step (needs g.fused_ok: every input position lies in the window of the band that owns it,
// and a group's words per position are whole 16-byte vectors)
hipError_t launch_bin_band_fused(const void* x_t, void* x_snap, unsigned int* arrive, const void* wband, void* y,
                                 const BinGeom& g, DevStats* stats, hipStream_t s) {
    if (g.band_rows < 1 || g.band_rows * g.wo > 65535 || !g.fused_ok || !arrive) return hipErrorInvalidValue;
    return launch_band<true>(x_t, x_snap, x_snap, arrive, wband, nullptr, y, g, stats, s);
}

hipError_t launch_bin_conv(int mode, int cw, const void* xsrc, const void* flip, unsigned int* tileflag,
                           const void* wpack, const void* bias, void* y, const BinGeom& g, DevStats* stats,
                           hipStream_t s) {
    if (mode == MODE_DELTA) {
        if (cw == 16) return launch_one<MODE_DELTA, 16>(xsrc, flip, tileflag, wpack, bias, y, g, stats, s);
        return launch_one<MODE_DELTA, 8>(xsrc, flip, tileflag, wpack, bias, y, g, stats, s);
    }
    if (cw == 16) return launch_one<MODE_DENSE, 16>(xsrc, flip, tileflag, wpack, bias, y, g, stats, s);
    return launch_one<MODE_DENSE, 8>(xsrc, flip, tileflag, wpack, bias, y, g, stats, s);
}

}  // namespace rrm
