// Fused delta + change-map kernel for convolution layers (int8, bf16, binary).
//
// Algorithm 1, first statement of the inner loop: the difference of this frame's input with the
// stored input.  The GPU form of "skip the zero elements" (Sec. 3.1, Sec. 3.5: the engine scans
// the activation vector for its non-zero entries) is a change map: x is scanned once as a flat
// array of 16-byte units; each wavefront turns its 64 compare results into one 64-bit mask
// (ballot), which is the bitmap word of those units; changed units write their difference, are
// committed to the snapshot, and mark the output blocks whose receptive field contains them: one byte
// flag per 4x4 output sub-tile for the MFMA path (the gather kernel ranks these flags into its work
// list), one stamp per 8x8 output tile for the binary path.
//
// The difference buffer keeps the invariant "zero wherever the bitmap bit is clear": a unit that
// changed in the previous step but not in this one is written back to zero, so the tile kernel can
// stage its input window with plain loads.  A stamped 8x8 tile holds the number of workgroups that
// will consume it; each consumer takes one off, so the stamps are all zero again after the binary
// kernel; the sub-tile flags hold the step's own value and are wiped by the next step's tile kernel (see StepEpoch).
// Nothing on the host has to change between steps (graph replay safe).
//
// HBM traffic per step: 2|x| read, plus (difference + snapshot) written only where x changed.
#include "rrm_internal.h"

namespace rrm {

namespace {

__device__ __forceinline__ float bf16_to_f32(unsigned int h) { return __uint_as_float(h << 16); }

// round-to-nearest-even float -> bf16 pattern (finite inputs)
__device__ __forceinline__ unsigned int f32_to_bf16(float f) {
    unsigned int u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

// floor(u / d) for u < 2^31 through the reciprocal rd = 1.0 / d: (u + 0.5) / d is at least 0.5 / d away
// from an integer, far more than the rounding error of the product, so the truncation is exact.
__device__ __forceinline__ unsigned int udiv_big(unsigned int u, double rd) {
    return (unsigned int)(((double)u + 0.5) * rd);
}
// floor(u / d) for u * d < 2^32 through magic = floor(2^32 / d) + 1 (0 encodes d == 1)
__device__ __forceinline__ int udiv_small(int u, unsigned int magic) {
    return magic ? (int)__umulhi((unsigned int)u, magic) : u;
}

__device__ __forceinline__ uint4 load_x_guarded(const unsigned char* x, long long off, long long total_bytes) {
    if (off + 16 <= total_bytes) return *reinterpret_cast<const uint4*>(x + off);
    unsigned int w[4] = {0u, 0u, 0u, 0u};
    for (int i = 0; i < 16; ++i)
        if (off + i < total_bytes) w[i >> 2] |= (unsigned int)x[off + i] << (8 * (i & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

__device__ __forceinline__ void mark_tiles(const ScanGeom& g, int pos, unsigned int* tileflag,
                                           unsigned int stamp) {
    const int hw = g.h * g.w;
    const int b = (int)udiv_big((unsigned int)pos, g.r_hw);
    const int r = pos - b * hw;
    const int iy = (int)udiv_big((unsigned int)r, g.r_w), ix = r - iy * g.w;
    const int ty0 = iy + g.pad - (g.kh - 1), tx0 = ix + g.pad - (g.kw - 1);
    const int oy_lo = ty0 <= 0 ? 0 : udiv_small(ty0 + g.stride - 1, g.magic_stride);
    const int ox_lo = tx0 <= 0 ? 0 : udiv_small(tx0 + g.stride - 1, g.magic_stride);
    int oy_hi = udiv_small(iy + g.pad, g.magic_stride), ox_hi = udiv_small(ix + g.pad, g.magic_stride);
    if (oy_hi > g.ho - 1) oy_hi = g.ho - 1;
    if (ox_hi > g.wo - 1) ox_hi = g.wo - 1;
    if (oy_lo > oy_hi || ox_lo > ox_hi) return;
    for (int ty = oy_lo / TILE; ty <= oy_hi / TILE; ++ty)
        for (int tx = ox_lo / TILE; tx <= ox_hi / TILE; ++tx)
            tileflag[(b * g.tiles_y + ty) * g.tiles_x + tx] = stamp;
}

// Mark the 4x4 output sub-tiles that see the input positions pos .. last (of a unit of few channels: several): one byte flag
// each, plain stores (every writer stores the same value, so no atomics and no same-address serialisation).  A run of
// positions in a row is marked at once -- the outputs whose windows meet it are those between its ends', at any stride (227 x 227
// x 3, one stream, the scan 9.1 -> 8.0 us).
__device__ __forceinline__ void mark_subtiles(const ScanGeom& g, unsigned int pos, unsigned int last, unsigned char* flags, unsigned char mark) {
    const unsigned int hw = (unsigned int)(g.h * g.w);
    while (pos <= last) {
        const int b = (int)udiv_big(pos, g.r_hw);
        const int r = (int)(pos - (unsigned int)b * hw);
        const int iy = (int)udiv_big((unsigned int)r, g.r_w), ix = r - iy * g.w;
        const int more = min((int)(last - pos), g.w - 1 - ix);
        pos += (unsigned int)more + 1u;
        const int ty0 = iy + g.pad - (g.kh - 1), tx0 = ix + g.pad - (g.kw - 1);
        const int oy_lo = ty0 <= 0 ? 0 : udiv_small(ty0 + g.stride - 1, g.magic_stride);
        const int ox_lo = tx0 <= 0 ? 0 : udiv_small(tx0 + g.stride - 1, g.magic_stride);
        const int oy_hi = min(udiv_small(iy + g.pad, g.magic_stride), g.ho - 1);
        const int ox_hi = min(udiv_small(ix + more + g.pad, g.magic_stride), g.wo - 1);
        if (oy_lo > oy_hi || ox_lo > ox_hi) continue;
        for (int sy = oy_lo >> 2; sy <= (oy_hi >> 2); ++sy)
            for (int sx = ox_lo >> 2; sx <= (ox_hi >> 2); ++sx) flags[(b * g.sty + sy) * g.stx + sx] = mark;
    }
}

// Element index of x element e in the padded / folded difference layout (see ScanGeom).
// (tensors are below 2^30 elements, so 32-bit arithmetic is exact)
__device__ __forceinline__ unsigned int scatter_index(const ScanGeom& g, unsigned int e) {
    const unsigned int p = e / (unsigned int)g.c;
    const unsigned int c = e - p * (unsigned int)g.c;
    const unsigned int r = p / (unsigned int)g.w;
    const unsigned int ix = p - r * (unsigned int)g.w;
    const unsigned int grp = c / (unsigned int)g.cg;
    return ((r * g.wp + ix) * g.groups + grp) * g.cp + (c - grp * g.cg);
}

// Write the 16 bytes of unit v (already computed difference words) into the padded / folded layout; where runs are shorter than
// a unit element by element, the (row, column, channel) of the first one divided out once and then stepped.
template <int DT>
__device__ __forceinline__ void scatter_unit(const ScanGeom& g, unsigned int v, uint4 w0, uint4 w1, uint4* d0, uint4* d1) {
    constexpr int PV = DT == RRM_I8_I32 ? 16 : 8, ESIZE = 16 / PV;
    const unsigned int e0 = v * PV;
    const unsigned int total = (unsigned int)g.total_elems;
    if (g.cg >= PV) {
        // Runs (one group's channels of a position) of a unit or more, padded one by one to whole units and never folded: the unit
        // lies in one run, one store at whatever alignment that gives, or ends one and begins the next, two pieces of 8, 4, 2 and 1
        // bytes.  (Element by element, 16 stores:
        // 28 x 28 x 100 int8, one stream, the scan 6.4 us and 3.8 so; 40 x 40 x 200, 40 streams, 12.5 and 9.0.)
        const unsigned int run = udiv_big(e0, g.r_cg), at = e0 - run * (unsigned int)g.cg;
        const unsigned int n = min((unsigned int)PV, total - e0), n0 = min(n, (unsigned int)g.cg - at);
        const unsigned int o0 = (run * (unsigned int)g.cp + at) * ESIZE, o1 = (run + 1u) * (unsigned int)g.cp * ESIZE;
        auto put = [&](uint4 w, uint4* d) __attribute__((always_inline)) {
            unsigned char* const b = reinterpret_cast<unsigned char*>(d);
            if (n0 == (unsigned int)PV) {
                __builtin_memcpy(b + o0, &w, 16);
                return;
            }
            const unsigned __int128 u = __builtin_bit_cast(unsigned __int128, w);
            store_piece(b + o0, u, n0 * ESIZE);
            store_piece(b + o1, u >> (8 * n0 * ESIZE), (n - n0) * ESIZE);
        };
        put(w0, d0);
        if (DT == RRM_BF16_F32) put(w1, d1);
        return;
    }
    const unsigned int p = udiv_big(e0, g.r_c);
    int c = (int)(e0 - p * (unsigned int)g.c);
    const unsigned int r0 = udiv_big(p, g.r_w);
    int ix = (int)(p - r0 * (unsigned int)g.w);
    unsigned int rowbase = r0 * (unsigned int)g.wp;
    if (DT == RRM_I8_I32 && g.groups == 1 && g.cp == 4) {
        // Few int8 channels padded to one 32-bit word per position (e.g. RGB -> RGBX): a position that lies
        // wholly inside the unit is one word store (its pad byte is zero anyway); the cut positions at the
        // unit's ends go byte by byte.
        const unsigned long long lo = (unsigned long long)w0.x | (unsigned long long)w0.y << 32;
        const unsigned long long hi = (unsigned long long)w0.z | (unsigned long long)w0.w << 32;
        const unsigned int keep = g.c >= 4 ? 0xFFFFFFFFu : (1u << (8 * g.c)) - 1u;
        unsigned int* dw = reinterpret_cast<unsigned int*>(d0);
        unsigned char* db = reinterpret_cast<unsigned char*>(d0);
        int k = 0;
        while (k < 16 && e0 + (unsigned int)k < total) {
            // the four bytes of the unit starting at byte k (zeros beyond its end)
            const unsigned int four = k < 8 ? (unsigned int)(lo >> (8 * k)) | (k ? (unsigned int)(hi << (64 - 8 * k)) : 0u)
                                            : (unsigned int)(hi >> (8 * (k - 8)));
            if (c == 0 && k + g.c <= 16 && e0 + (unsigned int)(k + g.c) <= total) {
                dw[rowbase + ix] = four & keep;
                k += g.c;
                c = g.c;
            } else {
                db[(rowbase + ix) * 4u + (unsigned int)c] = (unsigned char)four;
                ++k;
                ++c;
            }
            if (c == g.c) {
                c = 0;
                if (++ix == g.w) {
                    ix = 0;
                    rowbase += (unsigned int)g.wp;
                }
            }
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < PV; ++k) {
        if (e0 + k >= total) break;
        const int grp = g.groups == 1 ? 0 : c / g.cg;
        const unsigned int dst = ((rowbase + ix) * g.groups + grp) * g.cp + (c - grp * g.cg);
        if (DT == RRM_I8_I32) {
            const unsigned int word = k < 4 ? w0.x : (k < 8 ? w0.y : (k < 12 ? w0.z : w0.w));
            reinterpret_cast<unsigned char*>(d0)[dst] = (unsigned char)(word >> (8 * (k & 3)));
        } else if (DT == RRM_BF16_F32) {
            const unsigned int a = k < 2 ? w0.x : (k < 4 ? w0.y : (k < 6 ? w0.z : w0.w));
            const unsigned int b = k < 2 ? w1.x : (k < 4 ? w1.y : (k < 6 ? w1.z : w1.w));
            reinterpret_cast<unsigned short*>(d0)[dst] = (unsigned short)(a >> (16 * (k & 1)));
            reinterpret_cast<unsigned short*>(d1)[dst] = (unsigned short)(b >> (16 * (k & 1)));
        }
        if (++c == g.c) {
            c = 0;
            if (++ix == g.w) {
                ix = 0;
                rowbase += (unsigned int)g.wp;
            }
        }
    }
}

template <int ESIZE>
__global__ void repack_kernel(const unsigned char* __restrict__ x, unsigned char* __restrict__ dst, ScanGeom g) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= g.total_elems) return;
    const unsigned int d = scatter_index(g, (unsigned int)e);
    if (ESIZE == 1)
        dst[d] = x[e];
    else
        reinterpret_cast<unsigned short*>(dst)[d] = reinterpret_cast<const unsigned short*>(x)[e];
}

// The same re-layout where runs (one group's channels of a position) are padded to whole units and columns are not folded: one
// thread per unit of the padded layout, one load at whatever alignment the run has and one store.  (A thread per element: 40 x 40
// x 200 int8, 40 streams, 26.5 us and 8.5 so; 202 bf16 27.6 and 10.4.)
template <int ESIZE>
__global__ __launch_bounds__(256) void repack_unit_kernel(const unsigned char* __restrict__ x, uint4* __restrict__ dst, ScanGeom g,
                                                          unsigned int n_units, unsigned int per_run, unsigned int magic_per_run) {
    const unsigned int v = blockIdx.x * 256u + threadIdx.x;
    if (v >= n_units) return;
    const unsigned int run = udiv_magic(v, per_run, magic_per_run), u = v - run * per_run;
    const long long off = (long long)run * (g.cg * ESIZE) + 16 * u;
    dst[v] = load_unit_at<ESIZE>(x, off, g.total_elems * ESIZE, g.cg * ESIZE - 16 * (int)u);
}

// The same re-layout for few int8 channels padded to one 32-bit word per position (e.g. RGB -> RGBX): one
// thread per position, one word store.
__global__ void repack_word_kernel(const unsigned char* __restrict__ x, unsigned int* __restrict__ dst, ScanGeom g,
                                   unsigned int n_pos) {
    const unsigned int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_pos) return;
    const unsigned int r = udiv_big(p, g.r_w), ix = p - r * (unsigned int)g.w;
    const unsigned char* src = x + (size_t)p * (unsigned int)g.c;
    unsigned int word = 0;
    for (int c = 0; c < g.c; ++c) word |= (unsigned int)src[c] << (8 * c);
    dst[r * (unsigned int)g.wp + ix] = word;
}

// Fused scans of up to this many units read the producer's projection without waiting for the flags that say whether they have to:
// one round trip less, for reads that are mostly not needed.  (us a step of a five-layer stack with and without, 1 / 2 / 4 streams:
// 52.1 / 60.3 / 70.4 and 54.0 / 61.8 / 71.7; up to 65536 units, 8 streams: 87.1 and 87.4)
constexpr long long SCAN_SPEC_UNITS = 16384;

// Workgroup barrier that publishes LDS contents only (__syncthreads() would also wait for the stores)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// FUSED: the unit's input is computed from the producer's projection (see FusedSrc; no pooling); a unit none of whose
// source blocks was written by the producer's last step cannot have changed and is not even loaded.
// SPEC (fused, small launches): the projection is read without waiting for the flags that say whether it has to be.
template <int DT, bool SCATTER, bool FUSED, bool SPEC>
__device__ __forceinline__ void scan_body(const unsigned char* __restrict__ x_t, uint4* __restrict__ x_snap,
                                          uint4* __restrict__ d0, uint4* __restrict__ d1,
                                          unsigned long long* __restrict__ bitmap, unsigned int* __restrict__ tileflag,
                                          unsigned int stamp, const ScanGeom& g, unsigned int nvec, unsigned int total_bytes,
                                          DevStats* __restrict__ stats_base, const FusedSrc& fs) {
    fetch_args<6 * sizeof(void*) + 8 + sizeof(ScanGeom) + 16 + (FUSED ? sizeof(FusedSrc) : 0)>();
    // FUSED: neighbouring workgroups read overlapping rows of the producer's projection (pooling windows), and
    // consecutive workgroup ids go to different XCDs, each with an L2 of its own: the grid is a multiple of 8
    // and workgroup id i works on block (i % 8) * (grid / 8) + i / 8, so that an XCD gets a contiguous range.
    const unsigned int blk = FUSED ? (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    const unsigned int v = blk * 256u + threadIdx.x;
    DevStats* __restrict__ stats = stats_base + (blockIdx.x & (STAT_SLOTS - 1));
    // Every lane loads, those beyond the end unit 0, so that the first thing a wavefront does is to get its loads under way, and
    // what they all wait for is one round of the arguments.  The step's value comes through a vector load (of an address that
    // only looks different per lane): a scalar load would be waited for ahead of the units.
    const bool in = v < nvec;
    const unsigned int vc = in ? v : 0u;
    const unsigned long long prev_mask = bitmap[vc >> 6];  // (used where in)
    uint4 a = make_uint4(0, 0, 0, 0), b = a;
    if (!FUSED) {
        const bool whole = in && v * 16u + 16u <= total_bytes;
        a = *(whole ? reinterpret_cast<const uint4*>(x_t) + v : static_cast<const uint4*>(x_snap));
        b = x_snap[vc];
        if (in && !whole) a = load_x_guarded(x_t, (long long)v * 16, total_bytes);
    }
    const unsigned int epoch = DT == RRM_BIN_I32 ? 0u : g.epoch[EPOCH_SCAN + (threadIdx.x >> 8)];
    bool changed = false;
    int p0 = 0, p1 = -1;  // input positions of this unit, when it changed
    unsigned int nelem = 0, ntrunc = 0;
    float tsq = 0.f;  // truncated entries of this unit: count and sum of squares (bf16 with a threshold)
    bool compare = in;
    if (FUSED) {
        // (c_in is a multiple of 16: the unit is 16 channels of one position)
        const unsigned int e0 = vc * 16u;
        const unsigned int p = udiv_big(e0, g.r_c), c0 = e0 - p * (unsigned int)g.c;
        const unsigned int bb = udiv_big(p, g.r_hw), r = p - bb * (unsigned int)(g.h * g.w);
        const int iy = (int)udiv_big(r, g.r_w), ix = (int)r - iy * g.w;
        const unsigned char* t = fs.touched + (size_t)bb * fs.sty * fs.stx;
        const int4* yb = reinterpret_cast<const int4*>(fs.y + (((size_t)bb * fs.hy + iy) * fs.wy + ix) * g.c + c0);
        const unsigned int any = t[(iy >> fs.tshift) * fs.stx + (ix >> fs.tshift)];
        int4 w[4];
        if (SPEC) {
            b = x_snap[vc];
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q] = yb[q];
        }
        compare = in && (fs.fresh[0] != 0u || fs.touched_all[0] != 0u || (any & fs.epoch[0]) != 0u);
        if (compare) {
            if (!SPEC) {
                b = x_snap[v];  // in flight together with the projection's loads
#pragma unroll
                for (int q = 0; q < 4; ++q) w[q] = yb[q];
            }
            auto f = [&](int x) __attribute__((always_inline)) { return (unsigned int)min(127, max(0, x) >> fs.shift); };
            unsigned int wds[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) wds[q] = f(w[q].x) | f(w[q].y) << 8 | f(w[q].z) << 16 | f(w[q].w) << 24;
            a = make_uint4(wds[0], wds[1], wds[2], wds[3]);
        }
    }
    if (in) {
      if (compare) {
        const unsigned int za = a.x ^ b.x, zb = a.y ^ b.y, zc = a.z ^ b.z, zd = a.w ^ b.w;
        changed = (za | zb | zc | zd) != 0u;
        if (changed) {
            const unsigned int aw[4] = {a.x, a.y, a.z, a.w};
            const unsigned int bw[4] = {b.x, b.y, b.z, b.w};
            unsigned int dw[4], lw[4] = {0u, 0u, 0u, 0u};
            unsigned int sw[4] = {a.x, a.y, a.z, a.w};  // the unit's new snapshot (bf16: entry by entry)
            if (DT == RRM_I8_I32) {
                const unsigned int H = 0x80808080u;
                unsigned int ovf = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // byte-wise wrapping subtraction and its signed-overflow mask
                    const unsigned int d = ((aw[i] | H) - (bw[i] & ~H)) ^ ((aw[i] ^ ~bw[i]) & H);
                    ovf |= (aw[i] ^ bw[i]) & (aw[i] ^ d) & H;
                    dw[i] = d;
                    const unsigned int z = aw[i] ^ bw[i];
                    nelem += __popc((((z & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | z) & H);
                }
                if (ovf) atomicOr(&stats->range_error, 1u);
            } else if (DT == RRM_BF16_F32) {
                // Truncation threshold (Sec. 3.4, "Improving sparsity"): an entry whose difference is below
                // g.eps in magnitude is not applied and not committed (its snapshot entry keeps the old
                // value), so the stored projection stays the projection of the stored input.  eps = 0: exact.
                bool any_pass = false;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    unsigned int hi2 = 0, lo2 = 0, sn2 = 0;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const unsigned int xa = (aw[i] >> (16 * k)) & 0xFFFFu, xb = (bw[i] >> (16 * k)) & 0xFFFFu;
                        // difference in fp32 (exact unless the operands are > 2^15 apart in magnitude),
                        // then split into a bf16 head and a bf16 tail; equal inputs give 0 and 0 (no
                        // branch: the lanes of a wavefront would diverge on it)
                        const float d = bf16_to_f32(xa) - bf16_to_f32(xb);
                        const bool differ = xa != xb;
                        const bool trunc = differ && fabsf(d) < g.eps;
                        const bool pass = differ && !trunc;
                        any_pass |= pass;
                        nelem += pass ? 1u : 0u;
                        ntrunc += trunc ? 1u : 0u;
                        tsq += trunc ? d * d : 0.f;
                        const unsigned int hi = pass ? f32_to_bf16(d) : 0u;
                        const unsigned int lo = pass ? f32_to_bf16(d - bf16_to_f32(hi)) : 0u;
                        hi2 |= hi << (16 * k);
                        lo2 |= lo << (16 * k);
                        sn2 |= (pass ? xa : xb) << (16 * k);
                    }
                    dw[i] = hi2;
                    lw[i] = lo2;
                    sw[i] = sn2;
                }
                changed = any_pass;
            } else {  // binary: the flip mask
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    dw[i] = aw[i] ^ bw[i];
                    nelem += __popc(dw[i]);
                }
            }
            if (changed) {  // (bf16: every differing entry of the unit may have been truncated)
                if (!SCATTER) {
                    d0[v] = make_uint4(dw[0], dw[1], dw[2], dw[3]);
                    if (DT == RRM_BF16_F32) d1[v] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
                } else {
                    scatter_unit<DT>(g, v, make_uint4(dw[0], dw[1], dw[2], dw[3]), make_uint4(lw[0], lw[1], lw[2], lw[3]), d0, d1);
                }
                x_snap[v] = make_uint4(sw[0], sw[1], sw[2], sw[3]);  // snapshot of the input, only where it changed
                // input positions covered by this unit
                const unsigned int e0 = (unsigned int)v * g.per_vec;
                unsigned int e1 = e0 + g.per_vec - 1;
                if (e1 > (unsigned int)g.total_elems - 1) e1 = (unsigned int)g.total_elems - 1;
                p0 = (int)udiv_big(e0, g.r_c);
                p1 = (int)udiv_big(e1, g.r_c);
            }
        }
      }  // compare
        if (!changed && ((prev_mask >> (threadIdx.x & 63)) & 1ull)) {
            // changed last step, unchanged now: restore the zero of the difference buffer
            if (!SCATTER) {
                d0[v] = make_uint4(0, 0, 0, 0);
                if (DT == RRM_BF16_F32) d1[v] = make_uint4(0, 0, 0, 0);
            } else {
                scatter_unit<DT>(g, v, make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0), d0, d1);
            }
        }
    }
    // mark the output blocks that see the changed positions
    if (DT == RRM_BIN_I32) {
        if (stamp)  // (stamp 0: the layer's delta kernel reads the flip words itself)
            for (int p = p0; p <= p1; ++p) mark_tiles(g, p, tileflag, stamp);
    } else if (g.sty > 0) {  // (layers on the position-gather kernel read the bitmap instead: no flags)
        if (p0 <= p1) mark_subtiles(g, (unsigned int)p0, (unsigned int)p1, reinterpret_cast<unsigned char*>(tileflag), (unsigned char)epoch);
    }
    const unsigned long long mask = __ballot(changed);
    if ((threadIdx.x & 63) == 0 && in) bitmap[v >> 6] = mask;
    // change counts: summed over the wavefront, then over the workgroup, one pair of atomics per workgroup
    // (atomics on one address serialise: a pair per wavefront was the slowest part of a busy scan)
    __shared__ unsigned int s_ne[4], s_nu[4], s_nt[4];
    __shared__ float s_tq[4];
    if (mask) nelem = (unsigned int)__builtin_amdgcn_readlane((int)wave_scan(nelem), 63);
    if (DT == RRM_BF16_F32 && __any(ntrunc != 0u)) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            ntrunc += __shfl_xor(ntrunc, o);
            tsq += __shfl_xor(tsq, o);
        }
    }
    if ((threadIdx.x & 63) == 0) {
        s_ne[threadIdx.x >> 6] = nelem;
        s_nu[threadIdx.x >> 6] = (unsigned int)__popcll(mask);
        s_nt[threadIdx.x >> 6] = ntrunc;
        s_tq[threadIdx.x >> 6] = tsq;
    }
    lds_barrier();
    if (threadIdx.x == 0) {
        const unsigned int ne = s_ne[0] + s_ne[1] + s_ne[2] + s_ne[3], nu = s_nu[0] + s_nu[1] + s_nu[2] + s_nu[3];
        if (nu) {
            atomicAdd(&stats->changed_elems, (unsigned long long)ne);
            atomicAdd(&stats->changed_units, (unsigned long long)nu);
        }
        const unsigned int nt = s_nt[0] + s_nt[1] + s_nt[2] + s_nt[3];
        if (DT == RRM_BF16_F32 && nt) {
            atomicAdd(&stats->truncated_elems, (unsigned long long)nt);
            atomicAdd(&stats->truncated_sumsq, (double)s_tq[0] + (double)s_tq[1] + (double)s_tq[2] + (double)s_tq[3]);
        }
        if (blockIdx.x == 0) {  // one scan launch = one delta step
            atomicAdd(&stats_base->delta_steps, 1ull);
            atomicAdd(&stats_base->total_tiles, g.tiles_per_step);
            if (DT != RRM_BIN_I32) g.epoch[EPOCH_TILE] = epoch;
        }
    }
}

template <int DT, bool SCATTER, bool FUSED, bool SPEC = false>
__global__ __launch_bounds__(256) void scan_kernel(const unsigned char* __restrict__ x_t, uint4* __restrict__ x_snap,
                                                   uint4* __restrict__ d0, uint4* __restrict__ d1,
                                                   unsigned long long* __restrict__ bitmap,
                                                   unsigned int* __restrict__ tileflag, unsigned int stamp,
                                                   ScanGeom g, unsigned int nvec, unsigned int total_bytes,
                                                   DevStats* __restrict__ stats_base, FusedSrc fs) {
    scan_body<DT, SCATTER, FUSED, SPEC>(x_t, x_snap, d0, d1, bitmap, tileflag, stamp, g, nvec, total_bytes, stats_base, fs);
}

// The pooled fused form: every unit is the largest of nine positions of the producer's projection, nine times 64 bytes.  Four
// lanes share a unit, four channels each, so that a load instruction reads 16 whole units' 1 KiB and all nine loads of a unit
// are in flight.  (A lane that reads all 64 bytes of its unit touches four times as many cache lines per instruction and had
// three rows of loads one after the other: 27 x 27 x 96 and 13 x 13 x 256 consumers, 512 streams, 41.4 and 41.2 -> 29.7 and
// 34.0 us, one stream 6.3 -> 5.1 each.  More rows in flight in that form: 48 us.)  A wavefront takes ITER groups of 16 units;
// with ITER = 4 the lanes first look after a unit each -- its place, whether it can have changed -- and hand that to the four
// that compute it, and groups with nothing to do are skipped.  The unpooled form, one 64-byte read per unit, is at the rate of
// the memory as it is: 25.1 us a launch in scan_body's form, 27.4 in this one (13 x 13 x 384, 512 streams).
template <int ITER, bool SPEC>
__global__ __launch_bounds__(256) void scan_pooled_kernel(unsigned int* __restrict__ x_snap, unsigned int* __restrict__ d0,
                                                          unsigned long long* __restrict__ bitmap, unsigned char* __restrict__ flags,
                                                          ScanGeom g, unsigned int nvec, DevStats* __restrict__ stats_base, FusedSrc fs) {
    fetch_args<4 * sizeof(void*) + sizeof(ScanGeom) + 16 + sizeof(FusedSrc)>();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // (contiguous ranges of units per XCD: see scan_body)
    const unsigned int blk = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const unsigned int v0 = (blk * 4u + (unsigned int)wave) * (16u * ITER);  // the wavefront's first unit
    const unsigned int epoch = g.epoch[EPOCH_SCAN];
    const unsigned int prev16 = v0 < nvec ? (unsigned int)(bitmap[v0 >> 6] >> (v0 & 63u)) : 0u;  // (ITER = 1)
    const unsigned long long prev = ITER == 1 ? prev16 & 0xFFFFu : v0 < nvec ? bitmap[v0 >> 6] : 0ull;
    // this lane's unit: 16 channels of one position (c_in is a multiple of 16)
    const unsigned int v = v0 + (unsigned int)(ITER == 1 ? lane >> 2 : lane);
    unsigned int p = 0, off = 0;
    bool compare = v < nvec;
    unsigned int b_early = 0;
    int4 w_early[3][3];
    if (compare) {
        const unsigned int e0 = v * 16u;
        p = udiv_big(e0, g.r_c);
        const unsigned int c0 = e0 - p * (unsigned int)g.c, bb = udiv_big(p, g.r_hw), r = p - bb * (unsigned int)(g.h * g.w);
        const int iy = (int)udiv_big(r, g.r_w), ix = (int)r - iy * g.w, y0 = 2 * iy, x0 = 2 * ix;
        off = ((bb * (unsigned int)fs.hy + (unsigned int)y0) * (unsigned int)fs.wy + (unsigned int)x0) * (unsigned int)g.c + c0;
        if (SPEC) {
            b_early = x_snap[4u * v0 + (unsigned int)lane];
            const int* yb = fs.y + off + 4u * (unsigned int)(lane & 3);
#pragma unroll
            for (int k = 0; k < 9; ++k) w_early[k / 3][k % 3] = *reinterpret_cast<const int4*>(yb + (size_t)(k / 3 * fs.wy + k % 3) * (unsigned int)g.c);
        }
        const unsigned char* t = fs.touched + (size_t)bb * fs.sty * fs.stx;
        const int sy0 = y0 >> fs.tshift, sy1 = (y0 + 2) >> fs.tshift, sx0 = x0 >> fs.tshift, sx1 = (x0 + 2) >> fs.tshift;
        unsigned int any = 0;
        for (int sy = sy0; sy <= sy1; ++sy)
            for (int sx = sx0; sx <= sx1; ++sx) any |= t[sy * fs.stx + sx];
        compare = fs.fresh[0] != 0u || fs.touched_all[0] != 0u || (any & fs.epoch[0]) != 0u;
    }
    const unsigned long long todo = __ballot(compare);
    unsigned long long mask = 0;
    unsigned int nelem = 0;
#pragma unroll 1
    for (int i = 0; i < ITER; ++i) {
        const unsigned long long here = ITER == 1 ? todo : todo >> 16 * i & 0xFFFFull;
        const unsigned int was = (unsigned int)(prev >> 16 * i) & 0xFFFFu;
        if (!here && !was) continue;  // (the same in every lane)
        const unsigned int dw = 4u * (v0 + 16u * (unsigned int)i) + (unsigned int)lane;  // this lane's word of x
        unsigned int o = off;
        bool act = compare;
        if (ITER > 1) {
            o = __shfl(off, 16 * i + (lane >> 2));
            act = here >> (lane >> 2) & 1ull;
        }
        unsigned int a = 0, b = 0;
        if (act) {
            if (!SPEC) b = x_snap[dw];
            const char* yb = reinterpret_cast<const char*>(fs.y);
            const unsigned int vo = (o + 4u * (unsigned int)(lane & 3)) * 4u;
            int4 w[3][3];
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    w[dy][dx] = SPEC ? w_early[dy][dx] : *reinterpret_cast<const int4*>(yb + (size_t)(dy * fs.wy + dx) * (unsigned int)g.c * 4u + vo);
            if (SPEC) b = b_early;
            int best[4] = {0, 0, 0, 0};
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    best[0] = max(best[0], w[dy][dx].x);
                    best[1] = max(best[1], w[dy][dx].y);
                    best[2] = max(best[2], w[dy][dx].z);
                    best[3] = max(best[3], w[dy][dx].w);
                }
            // max commutes with the monotone map v -> min(127, max(0, v) >> shift)
#pragma unroll
            for (int k = 0; k < 4; ++k) a |= (unsigned int)min(127, best[k] >> fs.shift) << (8 * k);
        }
        const unsigned int z = a ^ b;
        unsigned int zz = z;  // ... of the unit
        zz |= (unsigned int)__builtin_amdgcn_mov_dpp((int)zz, 0xB1, 0xF, 0xF, true);  // quad_perm 1, 0, 3, 2
        zz |= (unsigned int)__builtin_amdgcn_mov_dpp((int)zz, 0x4E, 0xF, 0xF, true);  // quad_perm 2, 3, 0, 1
        const bool changed = zz != 0u;  // (not compared: a == b)
        if (changed) {
            // byte-wise wrapping subtraction and its signed-overflow mask
            const unsigned int H = 0x80808080u, d = ((a | H) - (b & ~H)) ^ ((a ^ ~b) & H);
            if (z & (a ^ d) & H) atomicOr(&stats_base[blockIdx.x & (STAT_SLOTS - 1)].range_error, 1u);
            nelem += __popc((((z & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | z) & H);
            d0[dw] = d;
            x_snap[dw] = a;
        } else if (was >> (lane >> 2) & 1u) {
            d0[dw] = 0u;  // changed last step, unchanged now: the zero of the difference buffer is restored
        }
        // one bit per unit: lanes 0 .. 15 take the word of theirs
        const unsigned int c16 = (unsigned int)__ballot(__shfl(changed ? 1 : 0, 4 * (lane & 15)) != 0) & 0xFFFFu;
        mask |= (unsigned long long)c16 << 16 * i;
    }
    // mark the sub-tiles that see the changed positions
    if (ITER == 1 ? (lane & 3) == 0 && (mask >> (lane >> 2) & 1ull) : (mask >> lane & 1ull) != 0ull)
        if (g.sty > 0) mark_subtiles(g, p, p, flags, (unsigned char)epoch);  // (the position-gather kernel reads the bitmap)
    __shared__ unsigned int s_ne[4];
    __shared__ unsigned long long s_mask[4];
    if (mask) nelem = (unsigned int)__builtin_amdgcn_readlane((int)wave_scan(nelem), 63);
    if (lane == 0) {
        s_ne[wave] = nelem;
        s_mask[wave] = mask;
        if (ITER == 4 && v0 < nvec) bitmap[v0 >> 6] = mask;
    }
    lds_barrier();
    if (threadIdx.x == 0) {
        DevStats* stats = stats_base + (blockIdx.x & (STAT_SLOTS - 1));
        if (ITER == 1 && v0 < nvec) bitmap[v0 >> 6] = s_mask[0] | s_mask[1] << 16 | s_mask[2] << 32 | s_mask[3] << 48;
        const unsigned int nu = (unsigned int)(__popcll(s_mask[0]) + __popcll(s_mask[1]) + __popcll(s_mask[2]) + __popcll(s_mask[3]));
        if (nu) {
            atomicAdd(&stats->changed_elems, (unsigned long long)(s_ne[0] + s_ne[1] + s_ne[2] + s_ne[3]));
            atomicAdd(&stats->changed_units, (unsigned long long)nu);
        }
        if (blockIdx.x == 0) {  // one scan launch = one delta step
            atomicAdd(&stats_base->delta_steps, 1ull);
            atomicAdd(&stats_base->total_tiles, g.tiles_per_step);
            g.epoch[EPOCH_TILE] = epoch;
        }
    }
}

}  // namespace

hipError_t launch_repack(int esize, const void* x, void* dst, const ScanGeom& g, hipStream_t s) {
    const long long blocks = (g.total_elems + 255) / 256;
    if (blocks <= 0) return hipSuccess;
    if (esize == 1 && g.groups == 1 && g.cp == 4 && g.c <= 4) {
        const long long n_pos = g.total_elems / g.c;
        hipLaunchKernelGGL(repack_word_kernel, dim3((unsigned int)((n_pos + 255) / 256)), dim3(256), 0, s,
                           (const unsigned char*)x, (unsigned int*)dst, g, (unsigned int)n_pos);
        return hipGetLastError();
    }
    if (g.wp == g.w && g.cp * esize % 16 == 0) {
        const int per_run = g.cp * esize / 16;
        const unsigned int units = (unsigned int)(g.total_elems / g.cg) * (unsigned int)per_run;
        const dim3 grid((units + 255u) / 256u), block(256);
        if (esize == 1)
            hipLaunchKernelGGL(repack_unit_kernel<1>, grid, block, 0, s, (const unsigned char*)x, (uint4*)dst, g, units,
                               (unsigned int)per_run, magic_of(per_run));
        else
            hipLaunchKernelGGL(repack_unit_kernel<2>, grid, block, 0, s, (const unsigned char*)x, (uint4*)dst, g, units,
                               (unsigned int)per_run, magic_of(per_run));
        return hipGetLastError();
    }
    if (esize == 1)
        hipLaunchKernelGGL(repack_kernel<1>, dim3((unsigned int)blocks), dim3(256), 0, s, (const unsigned char*)x,
                           (unsigned char*)dst, g);
    else
        hipLaunchKernelGGL(repack_kernel<2>, dim3((unsigned int)blocks), dim3(256), 0, s, (const unsigned char*)x,
                           (unsigned char*)dst, g);
    return hipGetLastError();
}

hipError_t launch_scan(int dtype, const void* x_t, void* x_snap, void* d0, void* d1, unsigned long long* bitmap,
                       unsigned int* tileflag, unsigned int stamp, const ScanGeom& g, DevStats* stats,
                       hipStream_t s) {
    const int esize = dtype == RRM_I8_I32 ? 1 : (dtype == RRM_BF16_F32 ? 2 : 4);
    const long long total_bytes = g.total_elems * esize;
    const long long nvec = (total_bytes + 15) / 16;
    const long long blocks = (nvec + 255) / 256;
    if (blocks <= 0) return hipSuccess;
    dim3 grid((unsigned int)blocks), block(256);
    const unsigned char* xt = static_cast<const unsigned char*>(x_t);
    const FusedSrc none{};
#define RRM_SCAN(DTV, SC)                                                                                               \
    hipLaunchKernelGGL((scan_kernel<DTV, SC, false>), grid, block, 0, s, xt, (uint4*)x_snap, (uint4*)d0, (uint4*)d1, bitmap, \
                       tileflag, stamp, g, (unsigned int)nvec, (unsigned int)total_bytes, stats, none)
    if (dtype == RRM_I8_I32) {
        if (g.scatter) RRM_SCAN(RRM_I8_I32, true); else RRM_SCAN(RRM_I8_I32, false);
    } else if (dtype == RRM_BF16_F32) {
        if (g.scatter) RRM_SCAN(RRM_BF16_F32, true); else RRM_SCAN(RRM_BF16_F32, false);
    } else {
        RRM_SCAN(RRM_BIN_I32, false);
    }
#undef RRM_SCAN
    return hipGetLastError();
}

hipError_t launch_scan_fused(const FusedSrc& src, void* x_snap, void* d0, unsigned long long* bitmap, unsigned int* marks,
                             const ScanGeom& g, DevStats* stats, hipStream_t s) {
    if (g.scatter || g.c % 16 != 0) return hipErrorInvalidValue;
    const long long total_bytes = g.total_elems;
    const long long nvec = total_bytes / 16;
    if (nvec <= 0) return hipSuccess;
    if (src.pool) {
        // Small inputs: a group per wavefront, four times the wavefronts.  Stack steps with one and four groups: 66.2 and 69.7 us at
        // one stream, 101.9 and 104.7 at 16 (70 and 43 thousand units), 136.1 and 135.4 at 64, 635 and 603 at 512.
        const bool small = nvec <= 131072;
        const unsigned int units = small ? 64u : 256u;  // of a workgroup
        const dim3 grid(((unsigned int)nvec + units * 8 - 1) / (units * 8) * 8);
        auto kern = nvec <= SCAN_SPEC_UNITS ? scan_pooled_kernel<1, true> : small ? scan_pooled_kernel<1, false> : scan_pooled_kernel<4, false>;
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, (unsigned int*)x_snap, (unsigned int*)d0, bitmap, (unsigned char*)marks, g,
                           (unsigned int)nvec, stats, src);
    } else {
        const long long blocks = ((nvec + 255) / 256 + 7) / 8 * 8;  // a multiple of the 8 XCDs (see the kernel)
        auto kern = nvec <= SCAN_SPEC_UNITS ? scan_kernel<RRM_I8_I32, false, true, true> : scan_kernel<RRM_I8_I32, false, true, false>;
        hipLaunchKernelGGL(kern, dim3((unsigned int)blocks), dim3(256), 0, s, (const unsigned char*)nullptr, (uint4*)x_snap, (uint4*)d0,
                           (uint4*)nullptr, bitmap, marks, 0u, g, (unsigned int)nvec, (unsigned int)total_bytes, stats, src);
    }
    return hipGetLastError();
}

}  // namespace rrm
