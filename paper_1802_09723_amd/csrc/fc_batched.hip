// Fully-connected layers with many streams: the layer is a skinny matrix product, W [c_out x c_in] times the
// streams' vectors [c_in x n], and it runs on the matrix cores with W read once for all streams.
//
// Dense layer (Eq. 3, FC form):      Y = b + W X^T
// Delta step (Algorithm 1, FC branch): with tens of streams the union of the changed columns is most of the matrix (64
// streams at 1 % each already touch half of the columns), so a product of the differences would run over all of W: its
// cost is one pass over W whatever the density, a tenth of what n separate column walks cost at 64 streams -- and the
// layer itself takes the same pass (a bf16 difference, which needs two bf16 terms, two).  The step therefore recomputes
// Y = b + W X_t^T, which for integers is the same sum and for bf16 free of the step-to-step rounding of an accumulated one,
// and commits and counts the frame.
// Shapes: v_mfma_i32_16x16x64_i8 / v_mfma_f32_16x16x32_bf16.  Lane l of a wavefront supplies 16 bytes of A (row
// l % 16 of a 16-row block of W, k-group l / 16: contiguous in W's own row-major layout) and 16 bytes of B (stream
// l % 16 of a 16-stream tile, same k-group: contiguous in a stream's vector), and receives rows 4 (l / 16) .. + 3
// of column l % 16: four consecutive output channels of one stream, one 16-byte store.
// The k range is split over workgroups (fc_bt_kernel, partial sums per split) and a second launch adds the splits
// in a fixed order (fc_bt_reduce_kernel: bit-reproducible fp32).  (Adding them in the product kernel, by the last
// split to arrive, needs device-scope fences around the arrival count; with those the kernel measured 28 us
// slower on the 9216 x 4096 layer -- the second launch costs 4.)
#include <algorithm>
#include <type_traits>

#include "rrm_internal.h"

namespace rrm {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int BT_CHAIN_TILES = 1;  // bf16 products of up to so many 16-stream tiles sum short chains (see fc_bt_kernel)

// x_snap <- x_t for every stream, change counts.  One thread per 16-byte unit.  (No difference is formed: any two int8 inputs
// are in range, as they are for the column walk with its nine-bit differences.)
struct FcCommit {
    const uint4* x_t;
    uint4* x_snap;
    long long nvec;
    unsigned long long n_cin;
    DevStats* stats;
};
__device__ __forceinline__ void fc_count(unsigned int block, unsigned int nchanged, const FcCommit& c) {
    // counts: wavefront, then workgroup, then one set of atomics
    __shared__ unsigned int s_n[4];
    if (__any(nchanged != 0u)) nchanged = (unsigned int)__builtin_amdgcn_readlane((int)wave_scan(nchanged), 63);
    if ((threadIdx.x & 63) == 0) s_n[threadIdx.x >> 6] = nchanged;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned int tot = s_n[0] + s_n[1] + s_n[2] + s_n[3];
        if (tot) {
            DevStats* slot = c.stats + (block & (STAT_SLOTS - 1));
            atomicAdd(&slot->changed_elems, (unsigned long long)tot);
            atomicAdd(&slot->changed_units, (unsigned long long)tot);
            atomicAdd(&slot->active_tiles, (unsigned long long)tot);
        }
        if (block == 0) {  // one launch = one delta step
            atomicAdd(&c.stats->delta_steps, 1ull);
            atomicAdd(&c.stats->total_tiles, c.n_cin);
        }
    }
}
template <int DT>
__device__ __forceinline__ unsigned int fc_changes(const uint4& a, const uint4& s) {  // entries of a unit that differ
    unsigned int nchanged = 0;
    const unsigned int zw[4] = {a.x ^ s.x, a.y ^ s.y, a.z ^ s.z, a.w ^ s.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned int z = zw[i];
        if (DT == RRM_I8_I32)
            nchanged += __popc((((z & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | z) & 0x80808080u);
        else
            nchanged += ((z & 0xFFFFu) != 0u) + (z > 0xFFFFu);
    }
    return nchanged;
}
template <int DT>
__device__ __forceinline__ void fc_commit(unsigned int block, const FcCommit& c) {
    const long long v = (long long)block * 256 + threadIdx.x;
    unsigned int nchanged = 0;
    if (v < c.nvec) {
        const uint4 a = c.x_t[v], s = c.x_snap[v];
        if ((a.x ^ s.x) | (a.y ^ s.y) | (a.z ^ s.z) | (a.w ^ s.w)) {
            nchanged = fc_changes<DT>(a, s);
            c.x_snap[v] = a;
        }
    }
    fc_count(block, nchanged, c);
}
// Vectors whose entries do not fill whole 64-byte steps, ahead of the product: their copy with every row padded by zeros to whole
// steps, a thread per 16 bytes of it, and (COMMIT) x_snap <- x_t with the change counts on the way.  It costs a launch, 2.5 us;
// without it such layers walk (steps) and read W once a stream (dense): 8999 -> 4000 bf16, 64 streams, a step of 2 % 144 us and 40.5, dense
// 200 and 39.5 (see fc_step_batched and fc_dense_batched).
template <int DT, bool COMMIT>
__global__ __launch_bounds__(256) void fc_pad_kernel(const unsigned char* __restrict__ x, uint4* __restrict__ padded, int row_bytes,
                                                     unsigned int per_row, unsigned int magic_per_row, unsigned int n_units,
                                                     long long total, FcCommit c) {
    constexpr int ESIZE = DT == RRM_I8_I32 ? 1 : 2;
    const unsigned int v = blockIdx.x * 256u + threadIdx.x;
    unsigned int nchanged = 0;
    if (v < n_units) {
        const unsigned int row = udiv_magic(v, per_row, magic_per_row), u = v - row * per_row;
        const int valid = row_bytes - 16 * (int)u;
        uint4 a = make_uint4(0, 0, 0, 0), s = a;
        if (valid > 0) {
            const long long off = (long long)row * row_bytes + 16 * u;
            if (COMMIT) {
                unsigned char* const snap = reinterpret_cast<unsigned char*>(c.x_snap);
                load_units_at<ESIZE>(x, snap, off, total, valid, a, s);
                if ((a.x ^ s.x) | (a.y ^ s.y) | (a.z ^ s.z) | (a.w ^ s.w)) {
                    nchanged = fc_changes<DT>(a, s);
                    if (valid >= 16)
                        __builtin_memcpy(snap + off, &a, 16);
                    else
                        store_piece(snap + off, __builtin_bit_cast(unsigned __int128, a), (unsigned int)valid);
                }
            } else {
                a = load_unit_at<ESIZE>(x, off, total, valid);
            }
        }
        padded[v] = a;
    }
    if (COMMIT) fc_count(blockIdx.x, nchanged, c);
}

// Partial products P[split] = W[:, k range of the split] B[:, k range]^T.  w: [c_out][c_in] row-major; b: [n][c_in]
// (the streams' vectors, or their differences); part: [splits][n][c_out] 4-byte sums.
// Workgroup (blockIdx.x, blockIdx.y) = (64-row group of W, split of the k range); wavefront v of its four takes the
// 16-row block v of the group.  The k range is walked in chunks of CK steps (a step = 64 bytes of a row and of every
// stream's vector).  Per chunk the workgroup copies the streams' bytes into LDS once -- all four wavefronts multiply
// the same streams, and read from memory they would cost four times the bytes of W -- while every lane reads its own
// 16 bytes of W per step straight into registers.  Loads run four chunks ahead of the matrix instructions, LDS is
// double-buffered, one barrier per chunk.
// LDS layout: (step of the chunk, stream) -> 80 bytes (64 used): the 16 streams that a group of 16 lanes reads for
// one k-group start 20 banks apart and fall on 16 different 4-bank groups.
template <int DT, int TMAX, int CK, bool CHAINS>
__global__ __launch_bounds__(256) void fc_bt_kernel(const unsigned char* __restrict__ w, const unsigned char* __restrict__ b,
                                                    void* __restrict__ part_v, FcGeom g, int cps) {
    constexpr int ESIZE = DT == RRM_I8_I32 ? 1 : 2;
    constexpr int KSTEP = 64 / ESIZE;  // elements per step: 64 int8 / 32 bf16
    constexpr int NS = 16 * TMAX;      // stream slots of the LDS layout
    constexpr int UPT = (NS * CK * 4 + 255) / 256;  // 16-byte units of the streams' chunk per thread
    constexpr int SPP = 256 / (CK * 4);             // streams covered by one pass of the 256 threads
    static_assert(256 % (CK * 4) == 0, "a pass of the threads covers whole streams");
    typedef typename std::conditional<DT == RRM_I8_I32, int, float>::type val_t;
    typedef typename std::conditional<DT == RRM_I8_I32, v4i, v4f>::type acc_t;
    __shared__ uint4 xs[2][CK * NS * 5];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4;  // k-group: bytes 16 kg .. 16 kg + 15 of a step
    const long long row_bytes = (long long)g.c_in * ESIZE;
    const int nsteps = g.c_in / KSTEP;
    const int kbeg = (int)blockIdx.y * cps * CK;
    const int kend = min(kbeg + cps * CK, nsteps);
    const int nch = (kend - kbeg + CK - 1) / CK;  // (>= 1: the host launches no empty split)
    // W: row of this lane (blocks beyond c_out read the last row; their sums are not stored)
    const int o0 = (int)blockIdx.x * 64 + wave * 16;
    const int row = min(o0 + (lane & 15), g.c_out - 1);
    // (byte offsets in 32 bits from the uniform bases: W and the streams' vectors are below 4 GB, checked at create)
    const unsigned int aoff = (unsigned int)row * (unsigned int)row_bytes + kg * 16;
    // streams' chunk: unit tid + 256 i = (stream tid / (4 CK) + SPP i, step (tid / 4) % CK, k-group tid % 4)
    const int xc = (tid >> 2) % CK;
    unsigned int xp[UPT], xm[UPT];
    int xoff[UPT];
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        const int s = tid / (CK * 4) + i * SPP;
        xm[i] = (unsigned int)-(int)(s < g.n);  // (a stream beyond n reads offset 0: never stored)
        xp[i] = (unsigned int)min(s, g.n - 1) * (unsigned int)row_bytes + (tid & 3) * 16;  // (streams beyond n: the last one's bytes, unused)
        xoff[i] = (xc * NS + s) * 5 + (tid & 3);
    }
    // A matrix instruction rounds its fp32 sum more than once, and the error of a chain of them grows as the square root of its
    // length.  Up to BT_CHAIN_TILES tiles a chain therefore has a chunk's CK instructions, and the chains are summed in 64 bits, behind
    // the loads of a chunk to come (relative error of 9216 -> 4096, 4 .. 15 streams, whose chains are 72 instructions long without:
    // 2.3e-7 and 0.6e-7, the column walk's 0.9e-7; us dense, 8 streams, 18.3 and 18.9).  More tiles' sums would cost more than they are
    // worth (32 streams of 9216 -> 256, 12.9 and 13.9, 64 of 9216 -> 4096 22.2 and 27.6): there the splits bound the chains, see bt_splits.
    acc_t acc[TMAX];
    v4d total[CHAINS ? TMAX : 1];
#pragma unroll
    for (int t = 0; t < TMAX; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[t][i] = 0;
            if constexpr (CHAINS) total[t][i] = 0;
        }
    auto join = [&]() __attribute__((always_inline)) {
        if constexpr (CHAINS)
#pragma unroll
            for (int t = 0; t < TMAX; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    total[t][i] += (double)acc[t][i];
                    acc[t][i] = 0;
                }
    };
    auto mma = [&](const uint4& a, const uint4& bb, acc_t c) {
        if constexpr (DT == RRM_I8_I32)
            return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, a), __builtin_bit_cast(v4i, bb), c, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, bb), c, 0, 0, 0);
    };
    struct Set {
        uint4 a[CK], x[UPT];
    };
    // Loads and LDS stores are unconditional and free of branches, so that the counted waits stay exact (a wait
    // placed after a branch would be for all outstanding loads, the newest included, and the prefetch would be
    // worth nothing): a chunk beyond the split, or a stream slot beyond the tiles in use, reads offset 0 -- one
    // cached line for the whole wavefront -- and the bytes it stores to LDS are never multiplied.  A step beyond
    // the range re-reads the last step: loaded, never multiplied.
    auto issue = [&](int chunk, Set& s) __attribute__((always_inline)) {
        const int k0 = kbeg + chunk * CK;
        const unsigned int lm = (unsigned int)-(int)(chunk < nch);
#pragma unroll
        for (int c = 0; c < CK; ++c)
            s.a[c] = *reinterpret_cast<const uint4*>(w + (size_t)((aoff + (unsigned int)min(k0 + c, nsteps - 1) * 64u) & lm));
#pragma unroll
        for (int i = 0; i < UPT; ++i)
            s.x[i] = *reinterpret_cast<const uint4*>(b + (size_t)((xp[i] + (unsigned int)min(k0 + xc, nsteps - 1) * 64u) & lm & xm[i]));
    };
    auto stage = [&](const Set& s, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < UPT; ++i) xs[buf][xoff[i]] = s.x[i];
    };
    const int boff = (lane & 15) * 5 + kg;
    // (TMAX is the number of 16-stream tiles in use or the next instantiated count: a tile beyond the streams
    // multiplies the bytes that the masked loads brought -- its sums are not stored -- so the products of a chunk
    // are one straight line of LDS reads and matrix instructions)
    auto compute = [&](const uint4(&a)[CK], int buf, int chunk) __attribute__((always_inline)) {
        const int k0 = kbeg + chunk * CK;
        if (k0 + CK <= kend) {
#pragma unroll
            for (int c = 0; c < CK; ++c)
#pragma unroll
                for (int t = 0; t < TMAX; ++t) acc[t] = mma(a[c], xs[buf][(c * NS + 16 * t) * 5 + boff], acc[t]);
            // issue order: the LDS reads of a step ahead of the matrix instructions of the step before it (one
            // wavefront per SIMD: nothing else hides the LDS latency)
            __builtin_amdgcn_sched_group_barrier(0x100, TMAX, 0);
#pragma unroll
            for (int c = 0; c + 1 < CK; ++c) {
                __builtin_amdgcn_sched_group_barrier(0x100, TMAX, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, TMAX, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, TMAX, 0);
        } else {  // the ragged last chunk of the range
#pragma unroll
            for (int c = 0; c < CK; ++c) {
                if (k0 + c >= kend) break;
#pragma unroll
                for (int t = 0; t < TMAX; ++t) acc[t] = mma(a[c], xs[buf][(c * NS + 16 * t) * 5 + boff], acc[t]);
            }
        }
    };
    // Four register sets in a ring: while chunk j is multiplied, chunks j + 1 .. j + 4 are in flight (one workgroup
    // per compute unit: the depth in registers is what keeps enough bytes in flight).  Per chunk: multiply; the next
    // chunk's streams go to the other LDS buffer (every wavefront finished reading it before the last barrier) and
    // its rows of W to `acur`; the freed set is refilled with the chunk four further on; one barrier.
    Set s0, s1, s2, s3;
    uint4 acur[CK];
    auto take = [&](const Set& s) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CK; ++c) acur[c] = s.a[c];
    };
    auto phase = [&](int j, int buf, Set& nxt) __attribute__((always_inline)) {
        if (j < nch) compute(acur, buf, j);
        stage(nxt, buf ^ 1);
        take(nxt);
        issue(j + 5, nxt);
        join();
        __syncthreads();
    };
    issue(0, s0);
    issue(1, s1);
    issue(2, s2);
    issue(3, s3);
    stage(s0, 0);
    take(s0);
    issue(4, s0);
    __syncthreads();
    for (int j = 0; j < nch; j += 4) {
        phase(j, 0, s1);
        phase(j + 1, 1, s2);
        phase(j + 2, 0, s3);
        phase(j + 3, 1, s0);
    }
    // this split's sums: rows 4 (lane / 16) .. + 3 of the block for stream lane % 16 of every tile
    if (o0 < g.c_out) {
        val_t* part = static_cast<val_t*>(part_v) + (long long)blockIdx.y * g.n * g.c_out;
        const int oc = o0 + 4 * kg;
#pragma unroll
        for (int t = 0; t < TMAX; ++t) {
            const int s = 16 * t + (lane & 15);
            if constexpr (CHAINS)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[t][i] = (float)total[t][i];
            if (s < g.n) *reinterpret_cast<acc_t*>(part + (long long)s * g.c_out + oc) = acc[t];
        }
    }
}

// y = bias + the splits' sums, added in the order of the splits (bit-reproducible fp32).  One thread per four consecutive
// output channels of one stream.  y_out: the caller's copy, or nullptr.  COMMIT: the workgroups behind the `blocks` of the
// reduction commit and count the frame.  (In a launch of its own ahead of the product: a step of 9216 -> 4096 bf16, 64 streams,
// 24.9 -> 22.5 us; int8, where that launch also wrote the differences and the sums went onto y, 18.7 -> 16.0.)
// WIDE (bf16): the splits are summed in 64 bits, where the product kernel sums its chains so or there are many splits (64 streams of
// 9216 -> 4096, whose four splits gain nothing by it, would take 0.2 us longer).
template <int DT, bool COMMIT, bool WIDE, bool RAGGED>
__global__ __launch_bounds__(256) void fc_bt_reduce_kernel(const void* __restrict__ part_v, const void* __restrict__ bias_v,
                                                           void* y_v, void* y_out, long long nvec, int c_out4, int c_out, int splits,
                                                           unsigned int blocks, FcCommit cm) {
    if (COMMIT && blockIdx.x >= blocks) {
        fc_commit<DT>(blockIdx.x - blocks, cm);
        return;
    }
    typedef typename std::conditional<DT == RRM_I8_I32, v4i, v4f>::type acc_t;
    const long long v = (long long)blockIdx.x * 256 + threadIdx.x;
    if (v >= nvec) return;
    typedef typename std::conditional<WIDE, v4d, acc_t>::type sum_t;
    const acc_t* part = static_cast<const acc_t*>(part_v);
    sum_t sum = __builtin_convertvector(part[v], sum_t);
    auto add = [&](const acc_t& a) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] += a[i];
    };
    for (int s0 = 1; s0 < splits; s0 += 5) {  // (five in flight)
        acc_t o[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) o[k] = part[(long long)min(s0 + k, splits - 1) * nvec + v];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            if (s0 + k >= splits) break;
            add(o[k]);
        }
    }
    if constexpr (RAGGED) {  // c_out is not whole 16-row blocks: the sums' rows are c_out4 vectors, y's c_out entries
        typedef typename std::conditional<DT == RRM_I8_I32, int, float>::type val_t;
        const long long row = v / c_out4;
        const int o0 = 4 * (int)(v - row * c_out4);
        const val_t* const bias = static_cast<const val_t*>(bias_v);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (o0 + i >= c_out) break;
            if (bias) sum[i] += bias[o0 + i];
            const val_t r = (val_t)sum[i];
            static_cast<val_t*>(y_v)[row * c_out + o0 + i] = r;
            if (y_out) static_cast<val_t*>(y_out)[row * c_out + o0 + i] = r;
        }
        return;
    }
    if (bias_v) add(static_cast<const acc_t*>(bias_v)[v % c_out4]);
    const acc_t out = __builtin_convertvector(sum, acc_t);
    acc_t* y = static_cast<acc_t*>(y_v);
    y[v] = out;
    if (y_out) static_cast<acc_t*>(y_out)[v] = out;
}

int bt_chunk(int ntiles) { return ntiles <= 4 ? 4 : 2; }

// streams per launch of the product kernel: more than 128 go in equal groups (a launch for 256 streams would walk the
// k range in single steps with a barrier each and far fewer splits: two launches of 128 take half its time, W is read
// twice)
constexpr int BT_MAX_STREAMS = 128;
constexpr int BT_MAX_SPLITS = 16;
int bt_group(int n) {
    const int ngroups = (n + BT_MAX_STREAMS - 1) / BT_MAX_STREAMS;
    return std::min(n, ((n + ngroups - 1) / ngroups + 15) / 16 * 16);
}

// Splits of the k range of one launch of n streams: about one workgroup per compute unit, about four chunks per split (what a
// workgroup has in flight) and at most sixteen, which the sums' launch reads.  The partial sums' bytes are no bound, they stay in
// the caches.  (us a step, held to half of W's bytes and three chunks, and so: int8 2048 -> 1024, 100 streams, 15.7 and 10.0; 300
// streams, 45.8 and 27.8; 4096 -> 4096, 128 streams, 18.7 and 16.6; bf16 1024 -> 512, 128 streams, 15.8 and 10.0.  Dense with at
// most 8 / 12 / 16 splits: bf16 9216 -> 256, 100 streams, 18.3 / 16.5 / 16.8; 9216 -> 1024, 100, 19.7 / 18.3 / 18.9; 4096 -> 256, 100,
// 12.8 / 13.0 / 12.6; 65536 -> 64, 16, 28.2 with twelve, 23.9 with sixteen; int8 9216 -> 1024, 100, 15.2 / 14.9 / 16.2.  Twelve are
// often a little faster, and eight for 4096 -> 1024, 100, 14.1 / 14.8 / 15.3, but longer chains cost bf16 precision: relative error of
// 9216 -> 256, 100 streams, 1.39e-7 with twelve and 1.31e-7 with sixteen.)
// More where a bf16 split's chain of matrix instructions would be longer than 20, or, with more than 64 streams, 32: the
// rounding error of long rows is then no larger than that of short ones (see fc_bt_kernel).
int bt_splits(int dtype, const FcGeom& g, int n) {
    const int esize = dtype == RRM_I8_I32 ? 1 : 2;
    const int ntiles = (n + 15) / 16, ck = bt_chunk(ntiles);
    const int chunks = (g.c_in * esize / 64 + ck - 1) / ck;
    const int groups = (g.c_out + 63) / 64;
    int most = BT_MAX_SPLITS;
    if (dtype == RRM_BF16_F32 && ntiles > BT_CHAIN_TILES) most = std::max(most, ck == 4 ? (chunks + 4) / 5 : (chunks + 15) / 16);
    return std::max(1, std::min(std::min((NUM_CU + groups - 1) / groups, most), (chunks + 3) / 4));
}

template <int DT>
void launch_batched(const void* w_rm, const void* x_t, void* padded, void* part, const void* bias, void* y, void* y_out, const FcGeom& real,
                    const FcCommit* commit, hipStream_t s) {
    constexpr int esize = DT == RRM_I8_I32 ? 1 : 2;
    constexpr bool BF = DT == RRM_BF16_F32;
    const FcGeom g = fc_product_geom(DT, real);
    const bool ragged = g.c_out != real.c_out;
    const void* b0 = x_t;
    if (g.c_in != real.c_in) {
        const unsigned int per_row = (unsigned int)(g.c_in * esize / 16), units = (unsigned int)g.n * per_row;
        const auto pad = commit ? fc_pad_kernel<DT, true> : fc_pad_kernel<DT, false>;
        hipLaunchKernelGGL(pad, dim3((units + 255u) / 256u), dim3(256), 0, s, static_cast<const unsigned char*>(x_t), static_cast<uint4*>(padded),
                           real.c_in * esize, per_row, magic_of((int)per_row), units, (long long)real.n * real.c_in * esize,
                           commit ? *commit : FcCommit{});
        b0 = padded;
        commit = nullptr;
    }
    const int nsteps = g.c_in * esize / 64;
    const int per = bt_group(g.n);
    const unsigned char* w = static_cast<const unsigned char*>(w_rm);
    for (int s0 = 0; s0 < g.n; s0 += per) {
        FcGeom gg = g;
        gg.n = std::min(per, g.n - s0);
        const int ntiles = (gg.n + 15) / 16;
        const int ck = bt_chunk(ntiles);
        const int chunks = (nsteps + ck - 1) / ck;
        const int want = bt_splits(DT, g, gg.n);
        const int cps = (chunks + want - 1) / want;
        const int splits = (chunks + cps - 1) / cps;  // (no empty split)
        dim3 grid((unsigned int)((g.c_out + 63) / 64), (unsigned int)splits);
        const unsigned char* p0 = static_cast<const unsigned char*>(b0) + (size_t)s0 * g.c_in * esize;
        unsigned char* yg = static_cast<unsigned char*>(y) + (size_t)s0 * real.c_out * 4;
        unsigned char* og = y_out ? static_cast<unsigned char*>(y_out) + (size_t)s0 * real.c_out * 4 : nullptr;
        // (padded layers took a walk, or sums of a few rows each, whose error is that of short chains)
        const bool chains = BF && (ntiles <= BT_CHAIN_TILES || ragged || g.c_in != real.c_in);
#define RRM_BT(T, C)                                                                                                  \
    if (ntiles <= T) {                                                                                                \
        const auto product = chains ? fc_bt_kernel<DT, T, C, BF> : fc_bt_kernel<DT, T, C, BF && T <= BT_CHAIN_TILES>; \
        hipLaunchKernelGGL(product, grid, dim3(256), 0, s, w, p0, part, gg, cps);                                     \
    } else
        RRM_BT(1, 4) RRM_BT(2, 4) RRM_BT(3, 4) RRM_BT(4, 4) RRM_BT(6, 2) RRM_BT(8, 2) {}
#undef RRM_BT
        const long long nvec = (long long)gg.n * g.c_out / 4;
        const unsigned int blocks = (unsigned int)((nvec + 255) / 256);
        const bool last = commit && s0 + per >= g.n, wide = BF && (chains || splits > BT_MAX_SPLITS);
        auto form = [&]<bool RAGGED>() {
            return last ? (wide ? fc_bt_reduce_kernel<DT, true, BF, RAGGED> : fc_bt_reduce_kernel<DT, true, false, RAGGED>)
                        : (wide ? fc_bt_reduce_kernel<DT, false, BF, RAGGED> : fc_bt_reduce_kernel<DT, false, false, RAGGED>);
        };
        const auto reduce = ragged ? form.template operator()<true>() : form.template operator()<false>();
        const FcCommit cm = last ? *commit : FcCommit{};
        hipLaunchKernelGGL(reduce, dim3(blocks + (last ? (unsigned int)((cm.nvec + 255) / 256) : 0u)), dim3(256), 0, s, part, bias, yg, og,
                           nvec, g.c_out / 4, real.c_out, splits, blocks, cm);
    }
}

}  // namespace

FcGeom fc_product_geom(int dtype, const FcGeom& g) {
    const int step = dtype == RRM_I8_I32 ? 64 : 32;
    FcGeom p = g;
    p.c_in = (g.c_in + step - 1) / step * step;
    p.c_out = (g.c_out + 15) / 16 * 16;
    return p;
}

// bytes of the partial sums (the groups of streams of one call use them one after the other; the last group can be smaller and
// have more splits)
size_t fc_batched_part_bytes(int dtype, const FcGeom& real) {
    const FcGeom g = fc_product_geom(dtype, real);
    const int per = bt_group(g.n), last = g.n - (g.n - 1) / per * per;
    const auto sums = [&](int n) { return (size_t)bt_splits(dtype, g, n) * (size_t)n; };
    return std::max(sums(per), sums(last)) * (size_t)g.c_out * 4;
}

// padded for the product: rows off the 64-byte steps (its vectors, in a launch of their own) or outputs off the blocks of 16
static bool fc_rows_padded(int dtype, const FcGeom& g) { return fc_product_geom(dtype, g).c_in != g.c_in; }
static bool fc_padded(int dtype, const FcGeom& g) { return fc_rows_padded(dtype, g) || fc_product_geom(dtype, g).c_out != g.c_out; }

bool fc_batched_ok(int dtype, const FcGeom& g) {
    const int esize = dtype == RRM_I8_I32 ? 1 : 2;
    // (byte offsets into W and the vectors in 32 bits)
    const FcGeom p = fc_product_geom(dtype, g);
    if (g.n < FC_BATCH_MIN_STREAMS || g.n > FC_BATCH_MAX_STREAMS || (long long)p.c_in * esize * std::max(p.c_out, p.n) > 0xFFFFFFFFll) return false;
    return !fc_padded(dtype, g) || fc_dense_batched(dtype, g) || fc_step_batched(dtype, g);  // (no copy of W for what never runs so)
}

// Does the dense layer run as one product?  Otherwise it reads W once a stream, from the caches.  Padded layers: us a call without
// and with it (with the launch that pads the vectors, but for the last row of a type):
//   int8  8999 -> 4000   4 streams  17.5 / 13.7   64 streams 163 / 21.6      8999 -> 1001   4  10.0 / 11.0    8  12.1 / 11.4   64  48.3 / 14.1
//   int8  4100 -> 1001   8           9.6 / 10.4   16          11.8 / 10.0    4099 ->  270  16  10.9 / 10.1   32  15.5 / 10.7   64  24.2 / 11.7
//   int8  1001 ->  500  64          10.8 / 10.9  128          15.4 / 11.3     523 ->  270 128  11.1 / 10.5
//   int8  4096 -> 1001   4           8.6 /  7.6   16          11.8 /  7.6
//   bf16  8999 -> 4000   4          21.6 / 23.2    8          34.5 / 23.4    8999 -> 1001   8  13.2 / 15.0   16  19.3 / 15.0   64  58.4 / 21.0
//   bf16  4100 -> 1001  16          12.0 / 11.8   32          17.6 / 12.9    4099 ->  270  32  11.6 / 12.4   64  17.0 / 14.8
//   bf16  1001 ->  500 128          13.0 / 13.8                              2050 -> 1001  32  12.1 / 11.4   64  18.9 / 13.6
//   bf16  4096 -> 1001   4           7.7 /  9.2   16          12.1 /  9.2
// (bf16: a stream's own read of W adds 0.045 us a MB of it; the product takes what about two and a half of them add, and 5 us beyond
// that path's fixed part, 4 without the launch that pads: level at (n - 2.5) w of 128 and 96 MiB, a fit to the rows above.  int8 products
// are level from a smaller n w on, and with many streams from the bytes of the vectors.)
bool fc_dense_batched(int dtype, const FcGeom& g) {
    if (!fc_padded(dtype, g)) return true;
    const long long w = (long long)g.c_in * g.c_out * (dtype == RRM_I8_I32 ? 1 : 2), rows = fc_rows_padded(dtype, g) ? 1 : 0;
    if (dtype == RRM_I8_I32) return g.n * w >= (rows ? 56ll : 16ll) * 1000000 || (g.n >= 16 && (long long)g.n * g.c_in >= 100000);
    return (2ll * g.n - 5) * w >= (rows ? 256ll : 192ll) << 20;
}

// Does a step run as one product?  Its cost is a pass over W, the streams' own column walks cost by the number of their workgroups
// (64 bytes of a stream's channels each), all of which compare their stream's row.  us a step walking, 1 / 5 / 25 % changed, and as
// a product (its step where it runs so, its dense layer, 0.1 .. 0.4 us less, elsewhere):
//   int8  9216 -> 4096   4 streams   256 workgroups    7.1 /  7.7 / 13.7   11.8      8 streams   512   11.0 / 12.3 / 21.6   12.1
//   int8  4096 -> 4096   4           256               6.3 /  6.8 /  7.1    7.4      8           512   10.0 / 10.7 / 10.9    7.2
//   int8  2048 -> 1024  24           384               7.5 /  8.3 /  8.6    7.5     32           512    8.6 /  9.1 /  9.6    7.9
//   int8  1024 ->  512  64           512               7.3 /  7.7 /  8.0    8.5    100           800   10.7 / 11.2 / 11.3    8.4
//   bf16  9216 -> 4096   4           512              14.0 / 15.4 / 25.2   18.2      6           768   20.9 / 23.7 / 38.3   18.5
//   bf16  4096 -> 4096   2           256               6.5 /  6.7 /  8.5    9.6      4           512    9.9 / 10.3 / 12.4   10.4
//   bf16  2048 -> 2048   6           384               8.5 /  8.5 /  8.7    7.5      8           512    9.8 /  9.9 / 10.2    7.6
// Rows of more than 16 KB: the product is dearer, the line is a quarter later.
// int8 layers below that line whose walks would read more than 200 MiB of W if everything changed, of a W that the caches hold: level
// while next to nothing changes, and dear soon.  us a step walking, 1 / 5 / 25 / 50 / 100 % changed, and as a product:
//   9216 -> 1024  24 streams  216 MiB    8.9 /  9.4 / 14.1 / 18.2 / 26.9   10.0      9216 -> 4096   7   252   10.3 / 11.5 / 20.6 / 30.2 / 39.5   12.1
//   9216 -> 2048  15          270       10.7 / 11.7 / 16.9 / 22.5 / 31.8    9.5      9216 ->  512  63   284    8.6 /  9.4 / 13.9 / 18.6 / 28.0   10.6
// and on the other side of it, where a walk is ahead, or level, up to a quarter and the product from half on:
//   9216 -> 1024  16          144        7.2 /  7.5 /  9.9 / 12.3 / 16.7    8.8      4096 -> 1024  31   124    8.6 /  9.2 /  9.6 / 12.0 / 16.5    8.0
//   4096 -> 4096   7          112        9.3 / 10.0 / 10.1 / 12.7 / 17.2    7.2      9216 ->  256  64   144    7.5 /  8.1 / 10.2 / 12.5 / 17.4   10.5
//   2048 -> 1024  31           62        8.6 /  8.9 /  9.4 /  9.5 / 11.8    7.6      1024 ->  512  63    32    7.2 /  7.6 /  7.9 /  8.1 /  8.0    8.1
// (more than 64 streams, whose product is dearer: 9216 -> 256, 127, 286 MiB, 10.0 / 10.6 / 13.6 / 17.9 / 26.7 and 14.0).
// Both sides have become faster since the line was laid, the product of short rows by more: rows of up to 4096 with a few hundred workgroups
// are level or ahead as products now, at any change.
// bf16 layers of 16 and more streams always.
// Padded layers, whose product is a launch dearer and whose bf16 sums are all of short chains, as exact as the walk's: us a step
// walking, 2 / 25 % changed, and as a product:
//   int8  8999 -> 4000   8 streams   504 workgroups   13.3 / 28.6   14.4     64 streams  4032   79.8 / 178   22.5
//   int8  4099 -> 4000   8           504              10.7 / 16.4   11.3     16          1008   19.5 / 27.9  11.6
//   int8  4100 -> 1001  32           512               9.6 / 12.4   11.6     48           768   13.8 / 16.6  12.0
//   int8  1001 ->  500  64           512               7.8 /  8.7   11.6     96           768   11.8 / 12.3  11.5
//   int8  4099 ->  270 128           640              10.7 / 13.8   14.2    523 -> 270  128  640  11.2 / 11.3  11.2
//   bf16  8999 -> 4000   4           500              15.3 / 27.8   23.7      8          1000   25.2 / 48.1  24.0
//   bf16  4100 -> 1001  16           512              11.4 / 13.4   12.3     32          1024   18.6 / 22.7  13.4
//   bf16  2050 -> 1001  16           512              10.1 / 10.4   11.0     64          2048   24.2 / 28.0  14.2
//   bf16  1001 ->  500  64          1024              13.2 / 13.3   13.2    128          2048   20.8 / 21.3  14.3
//   bf16  4099 ->  270  64           576              11.5 / 14.4   15.4    128          1152   17.2 / 21.3  20.2
//   rows of whole 64 bytes: int8 4096 -> 1001, 16, 256, 7.0 / 7.5 and 7.7, 64, 1024, 13.8 / 15.6 and 9.8; bf16 16, 512, 10.3 / 11.0 and 9.4
// (Rounding, 9216 -> 4096: a recomputed sum 0.6e-7 up to 16 streams and 2.3e-7 beyond, whatever ran before; a walked one 0.9e-7
// after the first step, 1.2e-7 after the sixth.)
bool fc_step_batched(int dtype, const FcGeom& g) {
    const int esize = dtype == RRM_I8_I32 ? 1 : 2;
    const long long workgroups = (long long)g.n * ((g.c_out_p * esize + 63) / 64);
    if (fc_padded(dtype, g)) {
        const bool rows = fc_rows_padded(dtype, g);
        if (dtype == RRM_I8_I32) return workgroups >= (rows ? 704 : 512);
        return workgroups >= (g.n > 64 ? 1280 : !rows ? 512 : g.c_in * esize > 16384 ? 1000 : 896);
    }
    if (dtype == RRM_BF16_F32 && g.n >= 16) return true;
    if (workgroups >= (g.c_in * esize > 16384 ? 640 : 512)) return true;
    return dtype == RRM_I8_I32 && g.n <= 64 && (long long)g.c_in * g.c_out <= 40ll << 20 && workgroups * 64 * g.c_in >= 200ll << 20;
}

hipError_t launch_fc_batched_dense(int dtype, const void* w_rm, const void* x, void* padded, void* part, const void* bias, void* y,
                                   const FcGeom& g, hipStream_t s) {
    if (!fc_batched_ok(dtype, g)) return hipErrorInvalidValue;
    if (dtype == RRM_I8_I32)
        launch_batched<RRM_I8_I32>(w_rm, x, padded, part, bias, y, nullptr, g, nullptr, s);
    else
        launch_batched<RRM_BF16_F32>(w_rm, x, padded, part, bias, y, nullptr, g, nullptr, s);
    return hipGetLastError();
}

hipError_t launch_fc_batched_delta(int dtype, const void* w_rm, const void* x_t, void* x_snap, void* padded, void* part,
                                   const void* bias, void* y, void* y_out, const FcGeom& g, DevStats* stats, hipStream_t s) {
    if (!fc_batched_ok(dtype, g) || g.eps != 0.0f) return hipErrorInvalidValue;
    const int esize = dtype == RRM_I8_I32 ? 1 : 2;
    const long long nvec = (long long)g.n * g.c_in * esize / 16;
    const unsigned long long n_cin = (unsigned long long)g.n * (unsigned long long)g.c_in;
    const FcCommit commit{static_cast<const uint4*>(x_t), static_cast<uint4*>(x_snap), nvec, n_cin, stats};
    if (dtype == RRM_I8_I32)
        launch_batched<RRM_I8_I32>(w_rm, x_t, padded, part, bias, y, y_out, g, &commit, s);
    else
        launch_batched<RRM_BF16_F32>(w_rm, x_t, padded, part, bias, y, y_out, g, &commit, s);
    return hipGetLastError();
}

}  // namespace rrm
