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
// channels.  It stages the band's input window (the flip mask m, and the flips to -1, m & ~x), notes which input positions hold a
// flip, lists
// the output positions whose window sees one (ballot compaction into LDS) and multiplies that list 64 entries
// at a time: every column of the product is an output position with work to do, wherever in the band it lies, so
// the work follows the changed positions instead of the 8x8 tiles they fall into.
#include <algorithm>
#include <mutex>

#include "rrm_internal.h"

namespace rrm {

namespace {

constexpr int BAND_THREADS = 64 * BAND_WAVES;  // the band kernel's workgroup

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

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
// channels of one tap in 32 cycles, where the popcount form takes 256 vector cycles, and a lane makes its 32 entries
// of the difference out of two LDS words with 16 instructions.
// Measured (28 x 28, 256 -> 256 channels, 64 streams, 5 % of the values flipping): 36.8 -> 23.0 us a step; one stream
// of 14 x 14, 512 -> 512 channels, 10 %: 16.8 -> 10.3.

// 32 differences as E2M1 nibbles: m = flip mask, q = flips to -1.  Nibble j of register i is bit 4j + i of the word
// (the weights are packed in the same order): 0x2 = +1, 0xA = -1, 0x0 = unchanged.
__device__ __forceinline__ v8i expand_e2m1(unsigned int m, unsigned int q) {
    const unsigned int P = 0x22222222u, N = 0x88888888u;
    return v8i{(int)(((m << 1) & P) | ((q << 3) & N)), (int)((m & P) | ((q << 2) & N)),
               (int)(((m >> 1) & P) | ((q << 1) & N)), (int)(((m >> 2) & P) | (q & N)), 0, 0, 0, 0};
}

__device__ __forceinline__ v16f mma_e2m1(const uint4& a, const v8i& b, v16f c) {
    const v8i av{(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, b, c, 4, 4, 0, 0, 0, 0);  // E2M1 x E2M1, unscaled
}

// FUSED: the whole step in this one launch.  `xsrc` is the new frame x_t and `flip` the stored input: the flip
// mask is their XOR, formed while the window is staged (no difference kernel, no flip buffer); the change counts
// are taken over the input rows a band owns; and the workgroup of a stream that finishes staging last (arrival
// counter) copies the frame into the stored input, when nobody reads the old one any more, and rearms the counter.
//
// DENSE: the layer itself (Eq. 3) with the same product: m = "tap inside the image", every output position is listed, and
// the result is the bias plus the sums.  (`flip` and `stats` are not touched.)  60 x 13, 448 -> 72 channels, 26 streams: 40.9 us on the tile
// kernel, 28.6 here.
template <bool FUSED, bool DENSE>
__global__ __launch_bounds__(BAND_THREADS, 4) void bin_band_kernel(const unsigned int* __restrict__ xsrc,
                                                       const unsigned int* flip, unsigned int* snap,
                                                       unsigned int* arrive,
                                                       const uint4* __restrict__ wband, const int* __restrict__ bias,
                                                       int* y, BinGeom g, DevStats* __restrict__ stats) {
    extern __shared__ uint4 smem[];
    const int npos = g.bth_in * g.btw_in;
    unsigned int* A = reinterpret_cast<unsigned int*>(smem);
    unsigned int* B = A + npos * g.bpitch;
    unsigned char* posany = reinterpret_cast<unsigned char*>(B + npos * g.bpitch);     // input position holds a flip
    unsigned short* list = reinterpret_cast<unsigned short*>(posany + ((npos + 15) & ~15));  // active output positions
    // sums of a pass: 64 positions x 64 channels, rows padded by one word (the lanes of an add are 32 positions)
    int* red = reinterpret_cast<int*>(reinterpret_cast<unsigned char*>(list) + (((size_t)g.band_rows * g.wo * 2 + 15) & ~(size_t)15));
    __shared__ unsigned int s_wc[BAND_THREADS / 64], s_prev;

    // grid: x = list split (fastest, so the workgroups that share a band start together), y = channel block,
    // z = stream x band
    const int sb = (int)blockIdx.z, zsplit = (int)blockIdx.x, nsplit = (int)gridDim.x;
    const int b = sb / g.nbands, band = sb - b * g.nbands;
    const int nblk = (g.og + 63) / 64;
    const int grp = blockIdx.y / nblk;
    const int blk = blockIdx.y - grp * nblk;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int oy0 = band * g.band_rows;
    const int rows = min(g.band_rows, g.ho - oy0);
    const int iy0 = oy0 * g.stride - g.pad, ix0 = -g.pad;
    const int wg4 = g.nslab * 4;

    // A pass is 64 listed positions x 64 channels.  Each half of the wavefronts takes one of its two tiles of 32 positions,
    // and the four of a half split the K steps (a tap, 64 channels): a wavefront takes steps w, w + 4, ... and adds its
    // sums in LDS.  Filter fragments go from memory straight into registers, BAND_KU steps in flight; the first ones do
    // not depend on the list: they are fetched ahead of it (and stay for every pass if they are all).  (Eight parts of both
    // tiles: twice the adds, and registers for fewer steps in flight.)
    const int ntaps = g.kh * g.kw, nkt = 2 * g.nslab, nk = ntaps * nkt;  // K steps per tap, in all
    const int n = lane & 31, khalf = lane >> 5;
    const uint4* wfrag = wband + ((long long)(grp * 2 * nblk + 2 * blk) * nk) * 64;
    const int kpart = wave & 3, tile = wave >> 2;
    uint4 w[BAND_KU][2];
    auto load_frags = [&](int k0) {
#pragma unroll
        for (int i = 0; i < BAND_KU; ++i) {
            const int k = min(k0 + i * 4, nk - 1);
#pragma unroll
            for (int c = 0; c < 2; ++c) w[i][c] = (wfrag + (long long)(c * nk + k) * 64)[(unsigned int)lane];
        }
    };
    for (int i = tid; i < npos; i += BAND_THREADS) posany[i] = 0;
    for (int i = tid; i < 64 * BAND_RP; i += BAND_THREADS) red[i] = 0;
    __syncthreads();
    // (FUSED) input rows whose changes this band counts, by the workgroup of the band's first channel block
    const int own_lo = oy0 * g.stride, own_hi = band == g.nbands - 1 ? g.h : (oy0 + g.band_rows) * g.stride;
    const bool count_here = FUSED && blk == 0 && zsplit == 0;
    unsigned int nbits = 0, nunits = 0, arrived_before = 0;
    // ---- stage A = m and B = m & ~x of the band's input window ------------------------------
    if (g.vec4) {
        // four words at a time, both loads issued whatever the mask holds (independent loads, several in flight)
        const int units = npos * g.nslab;
#pragma unroll 4
        for (int u = tid; u < units; u += BAND_THREADS) {
            const int hp = (int)(g.magic_nslab ? __umulhi((unsigned int)u, g.magic_nslab) : (unsigned int)u), sl = u - hp * g.nslab;
            const int hy = (int)(g.magic_btw ? __umulhi((unsigned int)hp, g.magic_btw) : (unsigned int)hp), hx = hp - hy * g.btw_in;
            const int iy = iy0 + hy, ix = ix0 + hx;
            uint4 m = make_uint4(0, 0, 0, 0), xv = make_uint4(0, 0, 0, 0);
            if (iy >= 0 && iy < g.h && ix >= 0 && ix < g.w) {
                const long long wi = (((long long)b * g.h + iy) * g.w + ix) * g.wpp + (long long)grp * g.wg + sl * 4;
                m = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
                if (!DENSE) m = *reinterpret_cast<const uint4*>(flip + wi);  // the flip buffer is zero where nothing changed
                xv = *reinterpret_cast<const uint4*>(xsrc + wi);
                if (FUSED) {
                    m = make_uint4(m.x ^ xv.x, m.y ^ xv.y, m.z ^ xv.z, m.w ^ xv.w);
                    if (count_here && iy >= own_lo && iy < own_hi && (m.x | m.y | m.z | m.w)) {
                        nbits += __popc(m.x) + __popc(m.y) + __popc(m.z) + __popc(m.w);
                        ++nunits;
                    }
                }
            }
            if (m.x | m.y | m.z | m.w) posany[hp] = 1;
            *reinterpret_cast<uint4*>(A + hp * g.bpitch + sl * 4) = m;
            *reinterpret_cast<uint4*>(B + hp * g.bpitch + sl * 4) = make_uint4(m.x & ~xv.x, m.y & ~xv.y, m.z & ~xv.z, m.w & ~xv.w);
        }
    } else {
        const int units = npos * wg4;
        for (int u = tid; u < units; u += BAND_THREADS) {
            const int hp = (int)(g.magic_wg4 ? __umulhi((unsigned int)u, g.magic_wg4) : (unsigned int)u), wd = u - hp * wg4;
            const int hy = (int)(g.magic_btw ? __umulhi((unsigned int)hp, g.magic_btw) : (unsigned int)hp), hx = hp - hy * g.btw_in;
            const int iy = iy0 + hy, ix = ix0 + hx;
            unsigned int m = 0, xv = 0;
            if (wd < g.wg && iy >= 0 && iy < g.h && ix >= 0 && ix < g.w) {
                const long long wi = (((long long)b * g.h + iy) * g.w + ix) * g.wpp + (long long)grp * g.wg + wd;
                m = DENSE ? 0xFFFFFFFFu : flip[wi];  // the flip buffer is zero where nothing changed
                if (m) {
                    xv = xsrc[wi];
                    posany[hp] = 1;
                }
            }
            A[hp * g.bpitch + wd] = m;
            B[hp * g.bpitch + wd] = m & ~xv;
        }
    }
    __syncthreads();
    load_frags(kpart);
    if (FUSED) {
        // this workgroup has read the stored input for the last time
        // (thread 0 keeps the answer to the end: stored at once, it would hold up the list by a memory round trip)
        if (tid == 0) arrived_before = atomicAdd(&arrive[b], 1u);
        if (count_here) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                nbits += __shfl_xor(nbits, o);
                nunits += __shfl_xor(nunits, o);
            }
            if (lane == 0 && nunits) {
                atomicAdd(&stats[sb & (STAT_SLOTS - 1)].changed_elems, (unsigned long long)nbits);
                atomicAdd(&stats[sb & (STAT_SLOTS - 1)].changed_units, (unsigned long long)nunits);
            }
        }
        if (sb == 0 && blockIdx.y == 0 && zsplit == 0 && tid == 0) {  // one launch = one delta step
            atomicAdd(&stats[0].delta_steps, 1ull);
            atomicAdd(&stats[0].total_tiles, (unsigned long long)g.n * g.ho * g.wo);
        }
    }
    // ---- list the output positions of the band whose window holds a flip ------------------------
    const int nout = rows * g.wo;
    int cnt = 0;
    if (DENSE) {
        for (int q = tid; q < nout; q += BAND_THREADS) list[q] = (unsigned short)q;
        cnt = nout;
        __syncthreads();
    }
    for (int base = 0; !DENSE && base < nout; base += BAND_THREADS) {
        const int q = base + tid;
        bool act = false;
        if (q < nout) {
            const int oyl = q / g.wo, ox = q - oyl * g.wo;
            const unsigned char* pa = posany + (oyl * g.stride) * g.btw_in + ox * g.stride;
            for (int ky = 0; ky < g.kh; ++ky)
                for (int kx = 0; kx < g.kw; ++kx) act |= pa[ky * g.btw_in + kx] != 0;
        }
        // (the same order in every workgroup of the band: the workgroups of a list split deal its chunks among them)
        const unsigned long long mask = __ballot(act);
        if (lane == 0) s_wc[wave] = (unsigned int)__popcll(mask);
        __syncthreads();
        unsigned int wbase = (unsigned int)cnt, all = 0;
#pragma unroll
        for (int w = 0; w < BAND_THREADS / 64; ++w) {
            const unsigned int c = s_wc[w];
            if (w < wave) wbase += c;
            all += c;
        }
        if (act) list[wbase + __popcll(mask & ((1ull << lane) - 1ull))] = (unsigned short)q;
        cnt += (int)all;
        __syncthreads();  // (the counts are overwritten in the next round; after the last one: the list is complete)
    }
    if (!DENSE && cnt > 0 && blockIdx.y == 0 && zsplit == 0 && tid == 0)
        atomicAdd(&stats[sb & (STAT_SLOTS - 1)].active_tiles, (unsigned long long)cnt);

    // The list in passes of 64 entries, dealt to the workgroups of a list split.
    const bool vec = (g.c_out & 3) == 0 && (g.og & 3) == 0;
    for (int first = zsplit * 64; first < cnt; first += nsplit * 64) {
        // this thread's part of the pass' results: one position, eight channels; fetched now, needed at the end
        const int e = first + (tid >> 3), c8 = (tid & 7) * 8, co = blk * 64 + c8;
        const int qe = list[e < cnt ? e : 0], oye = qe / g.wo;
        int* yp = y + ((((long long)b * g.ho + oy0 + oye) * g.wo + (qe - oye * g.wo)) * g.c_out + (long long)grp * g.og + co);
        int yv[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int4 t = make_int4(0, 0, 0, 0);
            const int* add = DENSE ? (bias ? bias + grp * g.og + co : nullptr) : yp;
            if (add && e < cnt && co + 4 * h < g.og) {
                if (vec) {
                    t = reinterpret_cast<const int4*>(add)[h];
                } else {
                    t.x = add[4 * h];
                    t.y = co + 4 * h + 1 < g.og ? add[4 * h + 1] : 0;
                    t.z = co + 4 * h + 2 < g.og ? add[4 * h + 2] : 0;
                    t.w = co + 4 * h + 3 < g.og ? add[4 * h + 3] : 0;
                }
            }
            yv[4 * h] = t.x;
            yv[4 * h + 1] = t.y;
            yv[4 * h + 2] = t.z;
            yv[4 * h + 3] = t.w;
        }
        // this lane's column: the window offset of its listed position (an entry beyond the list repeats its first; its
        // sums are not read)
        const bool work = first + 32 * tile < cnt && kpart < nk;  // (the same in every lane)
        const int ent = first + 32 * tile + n;
        const int q = list[ent < cnt ? ent : 0], oyl = q / g.wo;
        const int lbase = ((oyl * g.stride) * g.btw_in + (q - oyl * g.wo) * g.stride) * g.bpitch + khalf;
        v16f acc[2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[c][r] = 0.f;
#pragma unroll 1
        for (int k0 = kpart; work && k0 < nk; k0 += BAND_KU * 4) {
            if (k0 != kpart) load_frags(k0);
#pragma unroll
            for (int i = 0; i < BAND_KU; ++i) {
                const int k = k0 + i * 4;
                if (k >= nk) break;
                const int tap = (int)udiv_magic((unsigned int)k, (unsigned int)nkt, g.magic_nkt), st = k - tap * nkt;
                const int ky = (int)udiv_magic((unsigned int)tap, (unsigned int)g.kw, g.magic_kw), kx = tap - ky * g.kw;
                const int off = (ky * g.btw_in + kx) * g.bpitch + 2 * st;
                const v8i d = expand_e2m1(A[lbase + off], B[lbase + off]);
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[c] = mma_e2m1(w[i][c], d, acc[c]);
            }
        }
        if (nk > BAND_KU * 4 && first + nsplit * 64 < cnt) load_frags(kpart);  // (the next pass')
        if (work) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    atomicAdd(&red[(32 * tile + n) * BAND_RP + 32 * c + 8 * (r >> 2) + 4 * khalf + (r & 3)], (int)acc[c][r]);
        }
        __syncthreads();
        int v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            v[k] = yv[k] + (DENSE ? 1 : 2) * red[(tid >> 3) * BAND_RP + c8 + k];
            red[(tid >> 3) * BAND_RP + c8 + k] = 0;
        }
        if (e < cnt) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (vec) {
                    if (co + 4 * h < g.og)
                        reinterpret_cast<int4*>(yp)[h] = make_int4(v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]);
                } else {
#pragma unroll
                    for (int k = 4 * h; k < 4 * h + 4; ++k)
                        if (co + k < g.og) yp[k] = v[k];
                }
            }
        }
        __syncthreads();  // (the sums are cleared for the next pass)
    }
    if (FUSED) {
        // commit: the stream's last workgroup to finish staging
        if (tid == 0) s_prev = arrived_before;
        __syncthreads();
        if (s_prev == (unsigned int)g.nbands * gridDim.y * (unsigned int)nsplit - 1u) {
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

template <bool FUSED, bool DENSE = false>
hipError_t launch_band(const void* xsrc, const void* flip, void* snap, unsigned int* arrive, const void* wband, const void* bias, void* y,
                       const BinGeom& g, DevStats* stats, hipStream_t s) {
    const int nblk = (g.og + 63) / 64;
    // few streams: deal the band's list over several workgroups.  In a step as long as every one has a compute unit to itself: each
    // stages the window and makes the list again, which a second one per compute unit does not repay (us with two and with one, 5 %
    // of the values flipping: 28 x 28, 256 -> 256 channels 3 x 3, 8 streams, 13.6 and 10.8, no change 9.6 and 7.3; 4 x 350, 128 ->
    // 256, 16 streams, 15.8 and 10.8).  Long lists of many taps lose (kernel us, 20 % of the positions: 5 x 5, 56 x 56, 128 -> 128,
    // 8 streams, 23.8 and 26.4; 112 x 112, 64 -> 64, 4 streams, 30.1 and 32.9; no change 10.4 and 7.4, 10.5 and 8.9), and some of 1
    // x 1 (64 x 500, 128 -> 128, 22.9 and 25.0).  The dense layer makes no list and has all positions: two per compute unit (5 x 5,
    // 112 x 112, 128 -> 128, 2 streams, 20.0 and 24.1; 3 x 3, 56 x 56, 64 -> 64, 16 streams, 14.8 and 16.4).
    const long long wgs = (long long)g.n * g.nbands * g.groups * nblk;
    const int chunks = (g.band_rows * g.wo + 63) / 64;  // (a workgroup takes the list 64 entries at a time)
    int z = (int)((DENSE ? 2 : 1) * NUM_CU / wgs);
    z = z < 1 ? 1 : (z > chunks ? chunks : z);
    dim3 grid((unsigned int)z, (unsigned int)(g.groups * nblk), (unsigned int)(g.n * g.nbands));
    const size_t lds = bin_band_lds_bytes(g, g.band_rows);
    auto kern = bin_band_kernel<FUSED, DENSE>;
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
                       static_cast<const uint4*>(wband), static_cast<const int*>(bias), static_cast<int*>(y), g, stats);
    return hipGetLastError();
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
