// Input-stationary ("scatter") delta convolution in ONE launch per step, for low change densities and for layers
// with too few positions to fill the chip otherwise (int8 -> int32, bf16 -> fp32).
//
// Algorithm 1's inner loop as the sparse engine of Sec. 3.5 walks it: the activations are scanned for non-zero
// entries of the difference, and every such entry multiplies the weights that see it and is summed into the
// outputs it touches.  Here a workgroup owns a block of consecutive input positions (and a share of the output
// channels).  It compares x_t with the stored input for its positions (first statement of the loop), keeps the
// difference in LDS, compacts the changed positions with one ballot, and multiplies them, as the rows of a
// matrix product per filter tap,
//     Z_tap [changed positions x c_out] = dI [changed positions x c_in] * W_tap^T [c_in x c_out]
// (v_mfma_i32_32x32x32_i8 / v_mfma_f32_32x32x16_bf16; weight fragments straight from memory in per-lane order, each
// used once per workgroup), and adds row p of Z_tap into the stored projection at the output position that sees
// input position p under that tap, with atomic adds: several input positions meet in one output, and integer adds
// commute (bit-exact); fp32 adds are applied in arrival order (within the layer's tolerance, not bit-reproducible).
// The work is exactly proportional to the number of changed input positions (Table 1 / Eq. 6 at position
// granularity), there is no change map, no work list in memory and no second launch.
//
// The stored input is committed by the workgroup's own threads from registers; when several workgroups share a
// position block (output-channel splits) the one that finishes its compare last does it (arrival counter per block,
// rearmed by that workgroup), because the others still read the old values until then.
//
// A step of few changes is bound by its serial chain, not by bytes or matrix rate: arguments (0.25 us a line), the units, the
// compare, a list, weights, products, adds, commit, each waiting for the one before.  So the arguments are fetched together,
// the arrival and the commit have a wavefront of their own beside the products, blocks of 1, 2, 4 and 8 units a thread have
// forms of their own (UPT; one form of 8 with its loops cut short in the others cost 0.3 us: it is the registers and the code to
// step over), and the compiler is held to registers for 2 wavefronts a SIMD, which is what a chip of two workgroups a compute
// unit needs, instead of spilling for more (waves_per_eu).  32 x 32, 16 -> 16 int8, 5 %, 4.4 us a step before and 4.2 now; 28 x 28, 512
// -> 128 1 x 1 int8 6.8 and 5.3; 14 x 14 x 256 bf16 7.1 and 5.9.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "rrm_internal.h"

namespace rrm {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

__device__ __forceinline__ v16i mma(const uint4& a, const uint4& b, v16i c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(v4i, a), __builtin_bit_cast(v4i, b), c, 0, 0, 0);
}
__device__ __forceinline__ v16f mma(const uint4& a, const uint4& b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0,
                                                   0);
}

__device__ __forceinline__ float bf16_to_f32(unsigned int h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ unsigned int f32_to_bf16(float f) {  // round to nearest even (finite inputs)
    unsigned int u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

constexpr int ST = 256;          // threads that compare and multiply
constexpr int SCAT_BOOKS = 64;   // ... and of the wavefront that announces the workgroup to the others of its block
constexpr size_t SCAT_STATIC_LDS = 4 * 1024;  // room for the static arrays of a workgroup

// The differences of two entries each (fp32), as bf16 heads and tails, rounded to nearest even
__device__ __forceinline__ unsigned int pack_bf16(float a, float b) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned int, __builtin_convertvector(v2f{a, b}, v2bf));
}
__device__ __forceinline__ void split_pair(unsigned int a, unsigned int b, unsigned int& hi, unsigned int& lo) {
    const float d0 = __uint_as_float(a << 16) - __uint_as_float(b << 16), d1 = __uint_as_float(a & 0xFFFF0000u) - __uint_as_float(b & 0xFFFF0000u);
    hi = pack_bf16(d0, d1);
    lo = pack_bf16(d0 - __uint_as_float(hi << 16), d1 - __uint_as_float(hi & 0xFFFF0000u));
}

// Workgroup barrier that publishes LDS contents only (__syncthreads() would also wait for the answer of the arrival counter)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A uniform value that stays in a scalar register from here on
template <typename T>
__device__ __forceinline__ T kept(T v) {
    asm volatile("" : "+s"(v));
    return v;
}

// difference planes in LDS (bf16 with one term: the second one holds the stored input until the difference is formed)
constexpr int scat_planes(int dtype) { return dtype == RRM_BF16_F32 ? 2 : 1; }

// DIFF (int8): the compare is a scan's (one that computed the input from another layer's projection, in a launch of its own); x_t is
// the difference it left, zero wherever nothing changed.  The launch keeps the sub-tile flags as the tile kernel does, in a
// row of workgroups of its own behind the position blocks.
template <int DT, int TERMS, bool DIFF, int UPT, bool BOOKS>
__global__ __launch_bounds__(ST + (BOOKS ? SCAT_BOOKS : 0)) __attribute__((amdgpu_waves_per_eu(2, 3))) void conv_scatter_kernel(const uint4* __restrict__ x_t, uint4* x_snap,
                                                          const uint4* __restrict__ wsc, void* y_v, ScatGeom g,
                                                          DevStats* __restrict__ stats_base) {
    typedef typename std::conditional<DT == RRM_I8_I32, v16i, v16f>::type acc_t;
    typedef typename std::conditional<DT == RRM_I8_I32, int, float>::type sc_t;
    // (14 x 14, 512 -> 512 int8, six streams, eight units a thread, 14.65 us a step without and 14.75 so)
    if (DIFF || UPT < SCAT_UPT) fetch_args<4 * sizeof(void*) + sizeof(ScatGeom) + sizeof(void*)>();
    // LDS: difference planes [scat_planes][PB][U] x 16 bytes, then one 16-byte block of zeros
    extern __shared__ uint4 smem[];
    uint4* dl = smem;
    const int plane = g.PB * g.U;  // units per plane
    uint4* zero_unit = dl + scat_planes(DT) * plane;
    __shared__ unsigned int s_flag[64];
    __shared__ int s_list[ST / 64 + (BOOKS ? 1 : 0)][64];  // (every wavefront makes its own list: nothing to wait for)
    __shared__ unsigned int s_prev;
    __shared__ __align__(16) int s_out[ST / 64][2][32];  // output offsets of an item's rows, or -1
    static_assert(sizeof(s_flag) + sizeof(s_list) + sizeof(s_prev) + sizeof(s_out) + 64 <= SCAT_STATIC_LDS, "see scatter_lds");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned int p0 = blockIdx.x * (unsigned int)g.PB;                     // first position of the block
    const int npos = min(g.PB, (int)((unsigned int)g.npos_total - p0));          // positions in it
    const int nunits = npos * g.U;
    const size_t u0 = (size_t)p0 * g.U;  // first 16-byte unit of the block (positions are contiguous in x)
    DevStats* stats = stats_base + (blockIdx.x & (STAT_SLOTS - 1));
    sc_t* y = static_cast<sc_t*>(y_v);
    if (DIFF && p0 >= (unsigned int)g.npos_total) {
        const unsigned int eshift = g.epoch[EPOCH_TILE] - 1u, bits = 0x01010101u << eshift;
        const int per = (g.n_words + g.cs - 1) / g.cs, w1 = min(g.n_words, ((int)blockIdx.y + 1) * per);
        unsigned int active = 0;
        for (int w = (int)blockIdx.y * per + tid; w < w1; w += ST) {
            const unsigned int f = g.flags[w], now = f & bits;
            active += __popc(now);
            if (f != now) g.flags[w] = now;  // the step before's marks
        }
        if (__any(active != 0)) {
            active = wave_scan(active);
            if (lane == 63) atomicAdd(&stats->active_tiles, (unsigned long long)active);
        }
        if (blockIdx.y == 0 && tid == 0) {
            g.epoch[EPOCH_SCAN] = 2u - eshift;
            g.fresh[0] = 0u;        // the stored input holds this step's input
            g.touched_all[0] = 0u;  // the flags describe this step
        }
        return;
    }

    // A block's workgroups count up one word, and the answer (0.7 us on an idle chip, 1.7 among the 36 of 14 x 14 x 256 bf16) must
    // not be waited for by a wavefront that has products to make: one more wavefront asks for it, and commits the stored input
    // if its workgroup was the last of the block to compare.  (BOOKS: see launch_conv_scatter.  Always set then, but read from the
    // arguments: known to the compiler, it waits for the weights ahead of the list, 28 x 28, 512 -> 128 1 x 1, 5.2 -> 5.4 us.)
    static_assert(!BOOKS || (!DIFF && UPT * ST <= SCAT_BOOKS_UNITS), "one wavefront commits a block's units");
    const bool books = BOOKS && g.books != 0;
    if (books && wave == ST / 64) {
        const int U = kept(g.U);
        const unsigned int magic_U = kept(g.magic_U);
        lds_barrier();
        lds_barrier();
        const bool flag = lane < npos && s_flag[lane] != 0u;
        const unsigned long long found = __ballot(flag);
        // (the workgroups that share a block see the same list, and without a changed position there is nothing to commit: they
        // don't count)
        if (!found) return;
        unsigned int before = 0;
        if (lane == 0) before = atomicAdd(&g.arrive[blockIdx.x], 1u);
        int* const mine = s_list[ST / 64];
        if (flag) mine[__popcll(found & ((1ull << lane) - 1ull))] = lane * U;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // LDS operations of one wavefront execute in order
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // The units of the changed positions, all in flight, and on their way before it is known whether they are needed: this
        // commit is what a launch ends with (32 x 32, 16 -> 16 int8, 4.7 us without and 4.2 so; 14 x 14 x 256 bf16, 5 %, 6.65 and
        // 6.2).
        constexpr int BATCH = SCAT_BOOKS_UNITS / 64;
        const int total = (int)__popcll(found) * U;
        uint4 x[BATCH];
        auto place = [&](int v) __attribute__((always_inline)) {
            const unsigned int c = (unsigned int)min(v + lane, total - 1), i = udiv_magic(c, (unsigned int)U, magic_U);
            return (unsigned int)(mine[i] + (int)(c - i * (unsigned int)U));
        };
        auto keep = [&](unsigned int x, unsigned int o) __attribute__((always_inline)) {  // entries whose difference was truncated keep the stored value
            const float d0 = __uint_as_float(x << 16) - __uint_as_float(o << 16), d1 = __uint_as_float(x & 0xFFFF0000u) - __uint_as_float(o & 0xFFFF0000u);
            const unsigned int old = (fabsf(d0) < g.eps ? 0xFFFFu : 0u) | (fabsf(d1) < g.eps ? 0xFFFF0000u : 0u);
            return (x & ~old) | (o & old);
        };
#pragma unroll
        for (int k = 0; k < BATCH; ++k)
            if (64 * k < total) x[k] = x_t[u0 + place(64 * k)];
        if (__builtin_amdgcn_readfirstlane((int)before) != g.cs - 1) return;
#pragma unroll
        for (int k = 0; k < BATCH; ++k)
            if (64 * k < total) {
                uint4* const p = x_snap + u0 + place(64 * k);
                uint4 n = x[k];
                if (DT == RRM_BF16_F32 && g.eps != 0.f) {
                    const uint4 o = *p;
                    n = make_uint4(keep(n.x, o.x), keep(n.y, o.y), keep(n.z, o.z), keep(n.w, o.w));
                }
                if (64 * k + lane < total) *p = n;
            }
        if (lane == 0) g.arrive[blockIdx.x] = 0u;
        return;
    }

    // ---- both frames' units, all in flight together ------------------------------------------------------------------
    uint4 a[UPT], b[UPT];
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        if (ST * i >= nunits) break;
        const int v = min(tid + ST * i, nunits - 1);
        a[i] = x_t[u0 + v];
        if (!DIFF) b[i] = x_snap[u0 + v];
    }
    if (tid < 64) s_flag[tid] = 0u;
    if (tid == 0) *zero_unit = make_uint4(0, 0, 0, 0);
    const bool counts = !DIFF && blockIdx.y == 0;  // statistics: one workgroup per position block
    // what the rest of the kernel needs of its arguments arrives while the units do
    const int U = kept(g.U), ug = kept(g.ug), nk = kept(g.nk), nkp = kept(g.nkp), ntaps = kept(g.ntaps), ncb = kept(g.ncb), kw = kept(g.kw),
              og = kept(g.og), c_out = kept(g.c_out), nitems = kept(g.npair * g.ntaps * g.nkp), cs = kept(g.cs), pad = kept(g.pad),
              stride = kept(g.stride), ho = kept(g.ho), wo = kept(g.wo), w_in = kept(g.w), hw = kept(g.h * g.w);
    const unsigned int magic_U = kept(g.magic_U), magic_hw = kept(g.magic_hw), magic_w = kept(g.magic_w), magic_nkp = kept(g.magic_nkp),
                       magic_taps = kept(g.magic_taps), magic_ncb = kept(g.magic_ncb), magic_kw = kept(g.magic_kw),
                       magic_stride = kept(g.magic_stride);
    lds_barrier();

    // ---- difference with the stored input (Algorithm 1), into LDS -------------------------------------------------------
    unsigned int keep_mask = 0;        // units to commit
    unsigned long long trunc_mask = 0;  // bf16: their entries that keep the stored value, eight bits a unit
    unsigned int nelem = 0, nunit = 0, ntrunc = 0;
    float tsq = 0.f;
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        if (ST * i >= nunits) break;
        const int v = tid + ST * i;
        if (DIFF) {
            if (v < nunits) {
                dl[v] = a[i];
                if (a[i].x | a[i].y | a[i].z | a[i].w) s_flag[udiv_magic(v, U, magic_U)] = 1u;
            }
            continue;
        }
        const unsigned int aw[4] = {a[i].x, a[i].y, a[i].z, a[i].w}, bw[4] = {b[i].x, b[i].y, b[i].z, b[i].w};
        const bool changed = v < nunits && ((aw[0] ^ bw[0]) | (aw[1] ^ bw[1]) | (aw[2] ^ bw[2]) | (aw[3] ^ bw[3])) != 0u;
        if (DT == RRM_I8_I32) {
            const unsigned int H = 0x80808080u;
            unsigned int dw[4], ovf = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // byte-wise wrapping subtraction and its signed-overflow mask
                const unsigned int d = ((aw[k] | H) - (bw[k] & ~H)) ^ ((aw[k] ^ ~bw[k]) & H);
                ovf |= (aw[k] ^ bw[k]) & (aw[k] ^ d) & H;
                dw[k] = d;
            }
            if (v < nunits) dl[v] = make_uint4(dw[0], dw[1], dw[2], dw[3]);
            if (changed) {
                if (ovf) atomicOr(&stats->range_error, 1u);
                if (counts)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const unsigned int z = aw[k] ^ bw[k];
                        nelem += __popc((((z & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | z) & H);
                    }
                s_flag[udiv_magic(v, U, magic_U)] = 1u;  // (every writer stores the same value)
                keep_mask |= 1u << i;
            }
        } else {
            // a unit that differs lies in the planes as it is until this thread forms its difference, below
            if (v < nunits) {
                dl[v] = changed ? a[i] : make_uint4(0, 0, 0, 0);
                dl[plane + v] = changed ? b[i] : make_uint4(0, 0, 0, 0);
            }
            keep_mask |= changed ? 1u << i : 0u;
        }
    }
    if (DT == RRM_BF16_F32) {
        // (truncation threshold, Sec. 3.4 "Improving sparsity": an entry whose difference is below g.eps is neither applied
        // nor committed; eps = 0 is the exact method.)  The difference is formed in fp32 and carried as a bf16 head and a
        // bf16 tail.  A loop over the thread's units that differ: unrolled over all of them it was 2400 instructions, most of
        // them fetched for nothing, and the units' loads waited for each other (7 x 7 x 512, one stream, 5 %: 13.3 us a step,
        // and 9.6 with this loop, one list per wavefront, no integer division and the commit ahead of the products).
        if (g.eps == 0.f) {
            // (nothing is truncated.  Two entries at a time, a third of the instructions; the planes of an entry that is equal are
            // cleared, because an infinity less itself is not 0)
            for (unsigned int m = keep_mask; m; m &= m - 1) {
                const int i = __ffs(m) - 1, v = tid + ST * i;
                const uint4 ua = dl[v], ub = dl[plane + v];
                const unsigned int aw[4] = {ua.x, ua.y, ua.z, ua.w}, bw[4] = {ub.x, ub.y, ub.z, ub.w};
                unsigned int hw[4], lw[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const unsigned int z = aw[k] ^ bw[k], d = (((z & 0x7FFF7FFFu) + 0x7FFF7FFFu) | z) & 0x80008000u;
                    const unsigned int differ = d | (d - (d >> 15));
                    split_pair(aw[k], bw[k], hw[k], lw[k]);
                    hw[k] &= differ;
                    lw[k] &= differ;
                    nelem += __popc(d);
                }
                dl[v] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
                if (TERMS == 2) dl[plane + v] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
                s_flag[udiv_magic(v, U, magic_U)] = 1u;
            }
        }
        for (unsigned int m = g.eps == 0.f ? 0u : keep_mask; m; m &= m - 1) {
            const int i = __ffs(m) - 1, v = tid + ST * i;
            const uint4 ua = dl[v], ub = dl[plane + v];
            const unsigned int aw[4] = {ua.x, ua.y, ua.z, ua.w}, bw[4] = {ub.x, ub.y, ub.z, ub.w};
            unsigned int dw[4], lw[4], passed = 0, tmask = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                unsigned int hi2 = 0, lo2 = 0;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const unsigned int xa = (aw[k] >> (16 * e)) & 0xFFFFu, xb = (bw[k] >> (16 * e)) & 0xFFFFu;
                    const float d = bf16_to_f32(xa) - bf16_to_f32(xb);
                    const bool differ = xa != xb;
                    const bool trunc = differ && fabsf(d) < g.eps;
                    const bool pass = differ && !trunc;
                    passed += pass ? 1u : 0u;
                    tmask |= trunc ? 1u << (2 * k + e) : 0u;
                    tsq += trunc ? d * d : 0.f;
                    const unsigned int hi = pass ? f32_to_bf16(d) : 0u;
                    const unsigned int lo = pass && TERMS == 2 ? f32_to_bf16(d - bf16_to_f32(hi)) : 0u;
                    hi2 |= hi << (16 * e);
                    lo2 |= lo << (16 * e);
                }
                dw[k] = hi2;
                lw[k] = lo2;
            }
            dl[v] = make_uint4(dw[0], dw[1], dw[2], dw[3]);
            if (TERMS == 2) dl[plane + v] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
            nelem += passed;
            ntrunc += __popc(tmask);
            trunc_mask |= (unsigned long long)tmask << (8 * i);
            if (passed)
                s_flag[udiv_magic(v, U, magic_U)] = 1u;
            else
                keep_mask &= ~(1u << i);
        }
    }
    if (DT == RRM_BF16_F32 && g.eps != 0.f) {  // what will be stored: truncated entries keep their value
#pragma unroll
        for (int i = 0; i < UPT; ++i) {
            if (ST * i >= nunits) break;
            const unsigned int tm = (unsigned int)(trunc_mask >> (8 * i)) & 0xFFu;
            auto pick = [&](unsigned int x, unsigned int sn, int k) __attribute__((always_inline)) {
                const unsigned int old = (tm >> (2 * k) & 1u ? 0xFFFFu : 0u) | (tm >> (2 * k + 1) & 1u ? 0xFFFF0000u : 0u);
                return (x & ~old) | (sn & old);
            };
            if (tm) a[i] = make_uint4(pick(a[i].x, b[i].x, 0), pick(a[i].y, b[i].y, 1), pick(a[i].z, b[i].z, 2), pick(a[i].w, b[i].w, 3));
        }
    }
    nunit = __popc(keep_mask);
    // the wavefront's first item, decoded while others compare
    int item = (int)blockIdx.y + wave * cs;
    int grp = 0, cb = 0, ky = 0, kx = 0, k0 = 0;
    const uint4* wp = wsc;
    auto decode = [&]() __attribute__((always_inline)) {
        const int pt = (int)udiv_magic(item, nkp, magic_nkp), pair = (int)udiv_magic(pt, ntaps, magic_taps), tap = pt - pair * ntaps;
        k0 = (item - pt * nkp) * 8;
        grp = (int)udiv_magic(pair, ncb, magic_ncb);
        cb = pair - grp * ncb;
        ky = (int)udiv_magic(tap, kw, magic_kw);
        kx = tap - ky * kw;
        wp = wsc + ((size_t)pt * nk + k0) * 64 + lane;
    };
    decode();
    lds_barrier();

    // ---- changed positions of the block (at most 64): the wavefront's list -----------------------------------------
    const bool flag = lane < npos && s_flag[lane] != 0u;
    const unsigned long long found = __ballot(flag);
    const int cnt = (int)__popcll(found);
    if (cnt > 0) {
        // (blocks of more units than the books' wavefront commits at once: every read of the stored input by this workgroup is done)
        const bool count_here = !DIFF && !books && cs > 1;
        unsigned int arrived_before = 0;
        if (count_here && tid == 0) arrived_before = atomicAdd(&g.arrive[blockIdx.x], 1u);
        if (flag) s_list[wave][__popcll(found & ((1ull << lane) - 1ull))] = lane;

        // ---- the products: work items (channel block of a group, tap, part of the K range of at most 8 steps).  A
        // workgroup takes items blockIdx.y, + cs, ... and deals them to its wavefronts; a wavefront has an item's
        // (at most 8) weight fragments in flight together, multiplies, and adds its rows.
        uint4 wv[8];
        auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k0 + k < nk) wv[k] = wp[(size_t)k * 64];
        };
        if (item < nitems) fetch();
        const int n = lane & 31, khalf = lane >> 5;
        const int ntile = (cnt + 31) >> 5;  // 1 or 2
        // this lane's positions: block-local position, stream, image coordinates
        int pl[2], cbs[2], ciy[2], cix[2];
        bool cok[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int ci = t * 32 + n;
            cok[t] = t < ntile && ci < cnt;
            pl[t] = cok[t] ? s_list[wave][ci] : 0;
            const unsigned int P = p0 + pl[t];
            cbs[t] = (int)udiv_magic(P, hw, magic_hw);
            const unsigned int r = P - (unsigned int)cbs[t] * hw;
            ciy[t] = (int)udiv_magic(r, w_in, magic_w);
            cix[t] = (int)r - ciy[t] * w_in;
        }
        // ---- commit the stored input (only where a difference was applied), while the weights arrive: at the end the answer of
        // the arrival counter would be waited for behind all of the outputs' atomic adds
        bool last = !DIFF && !books;
        if (count_here) {
            if (tid == 0) s_prev = arrived_before;
            lds_barrier();
            last = s_prev == (unsigned int)cs - 1u;
            if (last && tid == 0) g.arrive[blockIdx.x] = 0u;
        }
        if (last) {
#pragma unroll
            for (int i = 0; i < UPT; ++i) {
                if (ST * i >= nunits) break;
                if (keep_mask & (1u << i)) x_snap[u0 + tid + ST * i] = a[i];
            }
        }
        while (item < nitems) {
            acc_t acc[2];
            const int ub = grp * ug;  // first unit of the group within a position
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (t >= ntile) break;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][r] = 0;
                // the tile's operands, in flight together (a read ahead of each product was waited for each time)
                uint4 op[TERMS][8];
                const uint4* bp = dl + (pl[t] * U + ub + 2 * k0 + khalf);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const bool ok = 2 * (k0 + k) + khalf < ug;  // (units that are not there: zeros)
                    op[0][k] = *(ok ? bp + 2 * k : zero_unit);
                    if (TERMS == 2) op[TERMS - 1][k] = *(ok ? bp + plane + 2 * k : zero_unit);
                }
#pragma unroll
                for (int k = 0; k < 8; ++k)
#pragma unroll
                    for (int e = 0; e < TERMS; ++e) asm volatile("" : "+v"(op[e][k].x), "+v"(op[e][k].y), "+v"(op[e][k].z), "+v"(op[e][k].w));
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (k0 + k >= nk) break;
                    acc[t] = mma(op[0][k], wv[k], acc[t]);
                    if (TERMS == 2) acc[t] = mma(op[TERMS - 1][k], wv[k], acc[t]);
                }
            }
            // Row p of this tap's product belongs to the output position that sees input position p under the tap: the lanes work
            // out one position each, and read the four of a register group together.  The lanes of an add are 32 channels of
            // two positions, whole cache lines.  (With the operands the other way round, 32 positions and two channels: bf16
            // 3 x 3, one stream, 14 x 14 x 256, 5 / 25 % changed, 9.2 / 13.7 us instead of 7.4 / 8.4; 10 x 10 x 320, four
            // streams, 10 %, 23.8 instead of 11.4; int8 5 x 5, 27 x 27, 96 -> 256, 10 %, 15.3 instead of 7.2.)
            const int c = cb * 32 + n;
            // An address from a scalar base and a 32-bit offset (an output has at most 2^30 entries) takes half of the instructions,
            // where there are scalar registers for the base: next to the books they are short, and it would be fetched back from a
            // vector register's lane at every add (us a step with it and without: 14 x 14, 512 -> 256 int8, half changed, 9.15 and 8.3;
            // 28 x 28, 256 -> 64 bf16, 8.3 and 7.75; without books 24 x 27, 32 -> 48, ten streams, 4.6 and 5.0, 64 x 64, 512 -> 64
            // 1 x 1, 8 streams, 10.05 and 10.3; the five-layer stack 50.3 -> 48.5).
            constexpr bool SADDR = !BOOKS;
            const int least = c < og ? 0 : 0x7FFFFFFF;  // (no row is that large: a channel that is not there adds nothing)
            char* const yb = reinterpret_cast<char*>(y);
            const unsigned int ch = (unsigned int)(grp * og + c);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (t >= ntile) break;
                const int ty = ciy[t] + pad - ky, tx = cix[t] + pad - kx;
                const int oy = (int)udiv_magic(ty, stride, magic_stride), ox = (int)udiv_magic(tx, stride, magic_stride);
                const bool hit = cok[t] && ty >= 0 && tx >= 0 && oy * stride == ty && ox * stride == tx && oy < ho && ox < wo;
                if (khalf == 0) s_out[wave][t][n] = hit ? ((cbs[t] * ho + oy) * wo + ox) * c_out : -1;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (t >= ntile) break;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int4 o4 = *reinterpret_cast<const int4*>(&s_out[wave][t][8 * q + 4 * khalf]);
                    const int o[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if constexpr (SADDR) {
                            if (o[r] >= least) atomicAdd(reinterpret_cast<sc_t*>(yb + ((unsigned int)o[r] + ch) * 4u), acc[t][4 * q + r]);
                        } else {
                            const sc_t v = acc[t][4 * q + r];
                            if (o[r] >= 0 && c < og && v != (sc_t)0) atomicAdd(y + grp * og + c + o[r], v);
                        }
                    }
                }
            }
            item += (ST / 64) * cs;
            if (item < nitems) {
                decode();
                fetch();
            }
        }
    }

    // ---- statistics ---------------------------------------------------------------------------------------------------
    if (!counts) return;
    if (__any(nunit != 0)) {
        const unsigned int both = wave_scan(nelem | nunit << 16);  // (at most 8192 and 512 a wavefront)
        if (lane == 63) {
            atomicAdd(&stats->changed_elems, (unsigned long long)(both & 0xFFFFu));
            atomicAdd(&stats->changed_units, (unsigned long long)(both >> 16));
        }
    }
    if (DT == RRM_BF16_F32 && __any(ntrunc != 0)) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            ntrunc += __shfl_xor(ntrunc, o);
            tsq += __shfl_xor(tsq, o);
        }
        if (lane == 0) {
            atomicAdd(&stats->truncated_elems, (unsigned long long)ntrunc);
            atomicAdd(&stats->truncated_sumsq, (double)tsq);
        }
    }
    if (tid == 0) {
        if (cnt) atomicAdd(&stats->active_tiles, (unsigned long long)cnt);
        if (blockIdx.x == 0) {  // one launch = one delta step
            atomicAdd(&stats_base->delta_steps, 1ull);
            atomicAdd(&stats_base->total_tiles, (unsigned long long)g.npos_total);
            if (g.touched_all) g.touched_all[0] = 1u;  // this path keeps no flags of what it wrote: "everything"
        }
    }
}

}  // namespace

// A workgroup's LDS beyond 64 KB, dynamic and static (the lists and flags, 2.6 KB at most): for every form of the kernel, once per process
static hipError_t scatter_lds(size_t lds) {
    if (lds + SCAT_STATIC_LDS <= 64 * 1024) return hipSuccess;
    static std::once_flag once;
    static hipError_t attr = hipSuccess;
    std::call_once(once, [] {
        auto all = [&]<int UPT, bool BOOKS>() {
            for (const void* f : {reinterpret_cast<const void*>(&conv_scatter_kernel<RRM_I8_I32, 1, false, UPT, BOOKS>),
                                  reinterpret_cast<const void*>(&conv_scatter_kernel<RRM_I8_I32, 1, !BOOKS, UPT, BOOKS>),
                                  reinterpret_cast<const void*>(&conv_scatter_kernel<RRM_BF16_F32, 1, false, UPT, BOOKS>),
                                  reinterpret_cast<const void*>(&conv_scatter_kernel<RRM_BF16_F32, 2, false, UPT, BOOKS>)})
                if (attr == hipSuccess) attr = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
        };
        all.template operator()<1, false>();
        all.template operator()<2, false>();
        all.template operator()<4, false>();
        all.template operator()<8, false>();
        all.template operator()<1, true>();
        all.template operator()<2, true>();
        all.template operator()<4, true>();
    });
    return attr;
}

// the form of the kernel for blocks of PB * U units: see UPT there
template <int DT, int TERMS, bool DIFF, bool BOOKS>
static auto scatter_form(const ScatGeom& g) {
    const int upt = (g.PB * g.U + ST - 1) / ST;
    if constexpr (!BOOKS)
        if (upt > 4) return conv_scatter_kernel<DT, TERMS, DIFF, 8, false>;
    return upt <= 1 ? conv_scatter_kernel<DT, TERMS, DIFF, 1, BOOKS> : upt <= 2 ? conv_scatter_kernel<DT, TERMS, DIFF, 2, BOOKS>
                                                                                : conv_scatter_kernel<DT, TERMS, DIFF, 4, BOOKS>;
}

hipError_t launch_conv_scatter(int dtype, int terms, const void* x_t, void* x_snap, const void* wsc, void* y,
                               const ScatGeom& g0, DevStats* stats, hipStream_t s) {
    ScatGeom g = g0;
    const long long nblk = (g.npos_total + g.PB - 1) / g.PB;
    dim3 grid((unsigned int)nblk, (unsigned int)g.cs);
    const size_t lds = ((size_t)scat_planes(dtype) * g.PB * g.U + 1) * 16;
    const hipError_t e = scatter_lds(lds);
    if (e != hipSuccess) return e;
    // The wavefront of the books costs a compute unit that holds two workgroups more than it saves the one that is last: int8 up to a
    // few workgroups more than there are compute units, bf16, with more registers, up to that.  (us a step with and without, int8,
    // 5 / 25 % changed: 280 workgroups, 11 x 19, 368 -> 96, three streams, 5.55 / 6.7 and 5.85 / 7.15; 294, 18 x 18, 352 -> 96, two, 5.5
    // / 6.95 and 5.4 / 7.0; 343, 28 x 28 x 96, four, 4.95 / 7.25 and 4.85 / 6.85; 510, 24 x 27, 32 -> 48, ten, 5.2 / 6.85 and 4.6 / 6.65)
    const bool books = g.books = g.cs > 1 && g.PB * g.U <= SCAT_BOOKS_UNITS && nblk * g.cs <= (dtype == RRM_I8_I32 ? 9 * NUM_CU / 8 : NUM_CU);
    auto form = [&]<bool BOOKS>() {
        return dtype == RRM_I8_I32 ? scatter_form<RRM_I8_I32, 1, false, BOOKS>(g)
               : terms == 2        ? scatter_form<RRM_BF16_F32, 2, false, BOOKS>(g)
                                   : scatter_form<RRM_BF16_F32, 1, false, BOOKS>(g);
    };
    const auto kernel = books ? form.template operator()<true>() : form.template operator()<false>();
    hipLaunchKernelGGL(kernel, grid, dim3(ST + (books ? SCAT_BOOKS : 0)), lds, s, static_cast<const uint4*>(x_t), static_cast<uint4*>(x_snap),
                       static_cast<const uint4*>(wsc), y, g, stats);
    return hipGetLastError();
}

hipError_t launch_conv_scatter_diff(const void* d0, const void* wsc, void* y, const ScatGeom& g, DevStats* stats, hipStream_t s) {
    const long long nblk = (g.npos_total + g.PB - 1) / g.PB;
    dim3 grid((unsigned int)nblk + 1u, (unsigned int)g.cs);
    const size_t lds = ((size_t)g.PB * g.U + 1) * 16;
    const hipError_t e = scatter_lds(lds);
    if (e != hipSuccess) return e;
    const auto kernel = scatter_form<RRM_I8_I32, 1, true, false>(g);
    hipLaunchKernelGGL(kernel, grid, dim3(ST), lds, s, static_cast<const uint4*>(d0), static_cast<uint4*>(nullptr),
                       static_cast<const uint4*>(wsc), y, g, stats);
    return hipGetLastError();
}

}  // namespace rrm
