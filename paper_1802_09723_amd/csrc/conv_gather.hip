// Gather-tile implicit-GEMM convolution on the gfx950 matrix cores (int8 -> int32, bf16 -> fp32).
//
// Delta mode computes the second term of Eq. 5, F * (I_t - I_{t-1}), only where it is non-zero, and
// adds it in place into the stored projection (Algorithm 1: P_t = P_{t-1} + F * dI).  Dense mode
// computes Eq. 3, y = b + F * x, everywhere.
//
// Unit of work: a 4x4 block of output positions (a "sub-tile", 16 positions = one MFMA column
// block).  The scan kernel sets one byte flag per sub-tile whose receptive field contains a changed
// input.  Every workgroup of this kernel reads that flag array (a few KB at most), ranks the set flags
// with a popcount prefix sum, and takes its share of the ranked list: up to NT active sub-tiles from
// anywhere in the batch.  They become the N dimension of one GEMM per workgroup:
//     M = NCB blocks of 32 output channels
//     N = 16 x (gathered sub-tiles), two sub-tiles per MFMA
//     K = (filter tap, 16-byte channel chunk) pairs, two per MFMA
//         (v_mfma_i32_32x32x32_i8 / v_mfma_f32_32x32x16_bf16; lane l supplies row/column l%32 and the
//          16 bytes of pair 2k + l/32).  The 32x32 shapes are used because one wavefront per SIMD issues
//         them back to back at the full rate, which the 16x16 shapes only reach with two wavefronts.
// Both operands go through LDS, one slab of channel chunks at a time:
//   * weights: the filters are packed at create time in per-lane MFMA order, K pairs ordered chunk by
//     chunk, so a slab is a contiguous run of 1 KiB fragments per channel block; wavefronts copy them
//     with LDS-direct loads (global_load_lds_dwordx4, no registers), double-buffered across slabs;
//   * activations: the gathered sub-tiles' input windows, gathered 16 bytes per lane with the same
//     LDS-direct loads (chunk index rotated by position against bank conflicts; units outside the
//     image read a block of zeros), also double-buffered.  In delta mode the source is the difference
//     buffer, zero where nothing changed.
// The source is always in a 16-byte-chunk layout [stream][row][column][group][chunk]: the caller's x
// when its channel runs are 16-byte multiples, otherwise the padded (or column-folded) copy that the
// scan / repack kernels write (see scan.hip); the kernel itself only sees "source positions" of
// pos_bytes bytes with their own strides and window size.
// A workgroup's wavefronts have two roles.  Wavefronts 0-3 ("producers") own the work list and
// the copies into LDS; the others ("consumers", one per pair of gathered sub-tiles: eight of the 16-slot shape, four of
// the 8-slot one) only multiply and write results.  A consumer owns its pair and all NCB channel blocks.  While
// the consumers multiply slab k, the producers stage slab k+1 -- or the first slab of the workgroup's next
// work unit, including its list and address work -- into the other buffer; the two roles meet at one
// barrier per slab.  The producers' address arithmetic and load issue thus run in the shadow of the matrix
// instructions of another wavefront on the same SIMD.
// Two consumers per SIMD with one pair each read half as much again from LDS as one with two pairs, which costs
// nothing (the LDS is not what bounds the kernel), and leave registers to fetch the stored projection ahead of its use
// (see LATE_BASE): the five-layer stack at 512 streams 674 -> 626 us, the eight consumers alone 674 -> 668.
// The number of sub-tiles per workgroup adapts on the device: few active sub-tiles are spread one per
// workgroup (latency), many are packed NT per workgroup (operand reuse).
// Every output element has exactly one owner: no atomics on y, results reproducible run to run.
// The grid holds no more workgroups than the chip runs at once; a workgroup takes work units
// blockIdx.x, blockIdx.x + gridDim.x, ... of the ranked list.
// Every workgroup wipes its share of the flag array of the step before's marks (see StepEpoch), so nothing on the host
// changes between steps (HIP-graph replay safe).
#include <algorithm>
#include <mutex>

#include "rrm_internal.h"
#include "subtile_list.h"

namespace rrm {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

template <int DT>
struct Acc;
template <>
struct Acc<RRM_I8_I32> {
    typedef v16i type;
    typedef int4 vec;
    typedef int scalar;
};
template <>
struct Acc<RRM_BF16_F32> {
    typedef v16f type;
    typedef float4 vec;
    typedef float scalar;
};

// D (32x32) += A (32 x K) * B (K x 32); lane l holds row / column l%32 of A / B and 16 bytes of K
// (half l/32), and of D the column l%32 with rows 8*(r/4) + 4*(l/32) + r%4 in register r.
__device__ __forceinline__ v16i mma(const uint4& a, const uint4& b, v16i c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(v4i, a), __builtin_bit_cast(v4i, b), c, 0, 0, 0);
}
__device__ __forceinline__ v16f mma(const uint4& a, const uint4& b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0,
                                                   0);
}

// Issue order of a K step for the instruction scheduler: N_MFMA matrix instructions with N_READ LDS reads
// spread evenly between them.
template <int I, int N_MFMA, int N_READ>
__device__ __forceinline__ void sched_interleave() {
    if constexpr (I < N_MFMA) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
        constexpr int R = (N_READ * (I + 1)) / N_MFMA - (N_READ * I) / N_MFMA;
        if constexpr (R > 0) __builtin_amdgcn_sched_group_barrier(0x100, R, 0);  // R LDS reads
        sched_interleave<I + 1, N_MFMA, N_READ>();
    }
}

// Workgroup barrier that publishes LDS contents only: it waits for this wavefront's LDS operations, not for its
// outstanding global loads (__syncthreads() would also wait for the copies into LDS that were started early).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

typedef const void __attribute__((address_space(1))) * gptr_t;
typedef void __attribute__((address_space(3))) * lptr_t;

constexpr int wg_threads(int nt) { return CONV_THREADS + nt / 2 * WAVE; }  // 4 producer + nt / 2 consumer wavefronts
constexpr int LIST_CAP = 1024;                // ranked sub-tile ids held in LDS per ranking round

// The kernel's one argument.  It is read through the kernel argument segment, by a pointer that each role of the kernel hides
// from the compiler once: a field is then loaded where a role uses it instead of all of them at the kernel's start, where they
// took two hundred scalar registers, most of them spilled into the lanes of vector registers.  (With the reciprocals in ConvGeom
// and the list of subtile_list.h, a step: 56 x 56, 64 -> 64 bf16, 64 streams, 10 %, 36.05 -> 34.6 us; 35 x 29, 80 -> 112, 9 streams,
// 18.4 -> 16.95; the five-layer int8 stack at one stream 74.2 -> 70.1; 27 x 27, 96 -> 256 dense, 16 streams, 12.8 -> 12.3.)
struct ConvArgs {
    const unsigned char *src0, *src1, *zero16;
    unsigned int* flags;
    const uint4* wpack;
    const int* offtab;
    const void* bias;
    void* y;
    DevStats* stats;
    ConvGeom g;
};
typedef const ConvArgs __attribute__((address_space(4))) * args_t;
__device__ __forceinline__ args_t hidden(args_t a) {
    asm volatile("" : "+s"(a));
    return a;
}

// A uniform value that stays in a scalar register from here on (what a role's loops use: loaded anew in a loop, a field is a
// scalar round trip that the loop waits for, with its LDS reads).  Not for pointers: a hidden one is no longer known to be global.
template <typename T>
__device__ __forceinline__ T kept(T v) {
    asm volatile("" : "+s"(v));
    return v;
}

// CUT: a group's channels are not a multiple of four.  A form of its own: the scalar registers that the cut quads' conditions take cost
// the others 4 to 10 % (the five-layer stack, 512 streams, 571 -> 604 us).
template <int DT, int MODE, int NCB, int NT, int TERMS, bool CUT>
__global__ __launch_bounds__(wg_threads(NT)) void conv_gather_kernel(ConvArgs) {
    const args_t args = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
    fetch_args<sizeof(ConvArgs)>();
    const auto& g = args->g;
    unsigned int* const flags = args->flags;
    const int* const offtab = args->offtab;
    DevStats* const stats = args->stats;
    typedef typename Acc<DT>::type acc_t;
    typedef typename Acc<DT>::vec vec_t;
    typedef typename Acc<DT>::scalar sc_t;
    constexpr int WG_THREADS = wg_threads(NT);
    constexpr int MAXU = CONV_MAX_STAGE_UNITS;  // staged 16-byte units per producer thread and slab (host guarantees)
    static_assert(NT % 8 == 0 && NT <= 16, "NT: two sub-tiles per consumer wavefront, at most twelve wavefronts");
    // Few slots per workgroup (g.ksh > 0): the consumers of a pair split its K steps, and each finishes its share of the
    // channels from the other parts' sums (`owned`: the register quads that this part finishes and initialises).
    constexpr bool KSPLIT = NCB == 1 && NT == 8;
    const int ksh = KSPLIT ? g.ksh : 0;
    static_assert(LIST_CAP >= 2 * NT, "a ranking round holds at least two work units");

    // LDS: [weights x nbuf_a][windows (TERMS planes) x 2][window offset table][K parts' sums: g.ksh > 0]
    extern __shared__ uint4 smem[];
    unsigned char* lds = reinterpret_cast<unsigned char*>(smem);
    const int nbuf_a = g.nslab > 1 ? 2 : 1;  // a single slab of weights is staged once and serves every unit
    const int nq2 = 2 * g.nq;  // MFMA steps (two K pairs each) per slab; a K step is two of them
    const int a_bytes = NCB * nq2 * 1024;
    const int plane_bytes = g.nt * g.slot_bytes;  // one term's windows (g.nt <= NT slots: large windows get fewer)
    const int b_bytes = TERMS * plane_bytes;
    unsigned char* bbase = lds + nbuf_a * a_bytes;
    int2* tab = reinterpret_cast<int2*>(bbase + 2 * b_bytes);
    __shared__ int s_list[LIST_CAP];         // ranked sub-tile ids of this workgroup's units of a round
    __shared__ unsigned int s_base[4][NT];   // per producer wavefront: source byte offset of the window origin
    __shared__ int s_iy0[4][NT];             //   (wraps when the origin is in the padding) and the origin itself
    __shared__ int s_ix0[4][NT];
    __shared__ int s_scan[CONV_THREADS / WAVE];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool producer = wave < 4;
    const int cw = (wave - 4) & ((NT / 2 >> ksh) - 1);   // consumer: pair of slots
    const int kpart = KSPLIT ? (wave - 4) >> (2 - ksh) & 3 : 0;  // ... and part of the K steps
    auto owned = [&](int gq) { return !KSPLIT || (gq >> (2 - ksh)) == kpart; };  // register quad finished by this part
    // Workgroup coordinates: BX of GX unit lanes (a lane takes work units BX, BX + GX, ...), BY of GY channel-block
    // groups.  With g.xcd_deal set the grid is one-dimensional and the coordinates are dealt so that the GY
    // workgroups of a lane, which gather the same input windows, sit on the same XCD (workgroups go to the
    // eight XCDs round-robin by their linear index) and find each other's windows in that XCD's L2.
    const int GX = g.gx, GY = g.gy;
    int BX = (int)blockIdx.x, BY = (int)blockIdx.y;
    if (g.xcd_deal) {
        const int lin = (int)blockIdx.x, dealt = (GX >> 3) * 8 * GY;  // workgroups of the lanes that are dealt XCD by XCD
        // (the few lanes beyond a multiple of eight: wherever they fall)
        const int slot = lin < dealt ? lin >> 3 : lin - dealt, lane0 = (int)udiv_magic((unsigned int)slot, (unsigned int)GY, g.magic_gy);
        BY = slot - lane0 * GY;
        BX = lin < dealt ? lane0 * 8 + (lin & 7) : (GX >> 3) * 8 + lane0;
    }

    const int ncbg = g.gyg;  // channel-block groups per filter group
    const int grp = (int)udiv_magic((unsigned int)BY, (unsigned int)ncbg, g.magic_gyg);
    const int cbg = BY - grp * ncbg;
    // packed weights: [group][32-channel block (padded to ncbg*NCB)][MFMA step][lane]; a slab is MFMA steps
    // slab*nq2 .. slab*nq2 + nq2 - 1 of each of this workgroup's NCB blocks
    const int kall = g.nslab * nq2;
    const uint4* wbase = args->wpack + ((size_t)(grp * ncbg + cbg) * NCB) * kall * 64 + lane;
    auto stage_weights = [&](int slab, int buf) {  // producers
        unsigned char* dst = lds + buf * a_bytes;
#pragma unroll
        for (int c = 0; c < NCB; ++c) {
            const uint4* src = wbase + (size_t)(c * kall + slab * nq2) * 64;
            for (int q = wave; q < nq2; q += 4)
                __builtin_amdgcn_global_load_lds((gptr_t)(src + (size_t)q * 64), (lptr_t)(dst + (c * nq2 + q) * 1024), 16,
                                                 0, 0);
        }
    };
    // This thread's rows of the staging table and the first weight slab, which serve every unit, do not depend on the work
    // list.  A dense launch starts their loads at once; a delta launch when it knows that it has a unit, ahead of making the list
    // (behind the loads of the flags: loads return in order).
    const int2* utab = reinterpret_cast<const int2*>(offtab + conv_tab_words(g));
    int2 ut[MAXU];
    auto load_rows = [&]() {
#pragma unroll
        for (int i = 0; i < MAXU; ++i) {
            if (i * CONV_THREADS >= g.nt * g.wpos * g.sc) break;  // (the same in every thread: the table is padded)
            ut[i] = utab[tid + i * CONV_THREADS];
        }
    };
    if (MODE == MODE_DENSE && producer) {
        stage_weights(0, 0);
        load_rows();
    }
    if (!producer)
        for (int e = tid - CONV_THREADS; e < conv_tab_words(g) / 2; e += WG_THREADS - CONV_THREADS)
            tab[e] = reinterpret_cast<const int2*>(offtab)[e];  // window offset table, the same for every slab

    // ---- how many sub-tiles are active? -------------------------------------------------------------
    constexpr unsigned int LOW = 0x01010101u;
    unsigned int eshift = 0;  // this step's bit of a flag
    SubtileList ranks;
    int count;
    // Few sub-tiles in all (one stream of a small map: at most 256, and every group of nt consecutive sub-tiles
    // has a workgroup of its own in the grid): the launch is latency bound, so there is no global list.  A workgroup reads
    // the flags of its own group only, compacts them with one ballot, and is done after one barrier.
    const bool own_group = MODE == MODE_DELTA && g.n_sub <= GX * g.nt && g.n_sub <= CONV_THREADS;
    if (own_group) {
        eshift = g.epoch[EPOCH_TILE] - 1u;
        if (wave == 0) {
            const int id = BX * g.nt + lane;
            const bool f = lane < g.nt && id < g.n_sub && (reinterpret_cast<const unsigned char*>(flags)[id] >> eshift & 1u);
            const unsigned long long m = __ballot(f);
            if (f) s_list[__popcll(m & ((1ull << lane) - 1ull))] = id;
            if (lane < 4) s_scan[lane] = lane == 0 ? (int)__popcll(m) : 0;
        }
        lds_barrier();
        count = s_scan[0];
    } else if (MODE == MODE_DELTA) {
        if (producer) {
            const int mine = ranks.count(flags, g.n_words, g.epoch, wave, lane, eshift);
            if (lane == 0) s_scan[wave] = mine;
        } else {
            eshift = g.epoch[EPOCH_TILE] - 1u;
        }
        lds_barrier();
        count = s_scan[0] + s_scan[1] + s_scan[2] + s_scan[3];
    } else {
        count = g.n_sub;
    }
    // Above a density of active sub-tiles where reading and re-writing the stored projection costs more than
    // recomputing it, a delta launch recomputes everything instead (Eq. 3): all sub-tiles, the committed
    // input x_t (the scan has made the snapshot equal to it) as the source, one term, accumulators from the
    // bias.  The switch is the same in every workgroup (same count).
    const int n_flagged = count;
    const bool full = MODE == MODE_DELTA && !own_group && g.xfull != nullptr &&
                      (long long)count * 100 > (long long)g.n_sub * g.full_pct;
    if (full) count = g.n_sub;
    const bool listed = MODE == MODE_DELTA && !full;  // sub-tile ids come from the ranked list (else: all, in order)
    const bool from_y = listed;                        // accumulators start from the stored projection (else: bias)
    // The active sub-tiles are cut into work units of `per` sub-tiles: few sub-tiles are spread thinly (a
    // unit's latency grows with its size), many are packed NT per unit (operand reuse).
    // (a workgroup with a sub-tile group of its own: one unit, the group's active sub-tiles)
    const int gx = own_group ? 1 : GX;
    const int bx = own_group ? 0 : BX;
    // (several units per workgroup: as many as full-size units would need, but of equal size, so that the
    // last pass over the grid is not a nearly empty one of full-size units)
    const unsigned int mgx = own_group ? 0u : g.magic_gx;
    const int passes = max(1, (int)udiv_magic(udiv_magic((unsigned int)(count + gx * g.nt - 1), (unsigned int)gx, mgx),
                                              (unsigned int)g.nt, g.magic_per[g.nt]));
    int per = (int)udiv_magic((unsigned int)(count + gx * passes - 1), (unsigned int)gx, mgx);
    if (passes > 1) per = passes <= 16 ? (int)udiv_magic((unsigned int)per, (unsigned int)passes, g.magic_per[passes]) : per / passes;
    per = min(max(per, 1), g.nt);
    int my_nunits = passes;  // this workgroup's units: bx + i * gx, i = 0 .. my_nunits - 1, as far as they hold a sub-tile
    while (my_nunits > 0 && (bx + (my_nunits - 1) * gx) * per >= count) --my_nunits;

    // What a delta launch leaves for the steps and consumers to come (nothing that a workgroup of this launch reads).
    if (MODE == MODE_DELTA && !producer) {
        const int nwg = GX * GY, me = BY * GX + BX, share = (g.n_words + nwg - 1) / nwg;
        const int w1 = min(g.n_words, (me + 1) * share);
        for (int w = me * share + tid - CONV_THREADS; w < w1; w += WG_THREADS - CONV_THREADS) {
            const unsigned int v = flags[w], now = v & LOW << eshift;
            if (v != now) flags[w] = now;  // the step before's marks
        }
        if (me == 0 && tid == CONV_THREADS) {
            g.epoch[EPOCH_SCAN] = 2u - eshift;
            g.fresh[0] = 0u;  // the stored input holds this step's input
            g.touched_all[0] = full ? 1u : 0u;  // the flags describe this step, or it writes everything
            if (n_flagged && !own_group) atomicAdd(&stats[0].active_tiles, (unsigned long long)n_flagged);
        }
        // (each workgroup counted only its own group's flags)
        if (own_group && tid == CONV_THREADS && n_flagged && BY == 0)
            atomicAdd(&stats[(unsigned int)BX & (STAT_SLOTS - 1)].active_tiles, (unsigned long long)n_flagged);
    }
    if (my_nunits == 0) {
        __builtin_amdgcn_s_waitcnt(0);  // let a dense launch's early weight copy land before the LDS is released
        return;
    }
    constexpr int ur = LIST_CAP / NT;  // units ranked in one round

    // lane roles of a consumer: position j of sub-tile `half` of a pair (MFMA column l%32), K pair `khalf` of
    // an MFMA step; of the result it holds channels 8*gq + 4*khalf + (0..3), gq = 0..3, of each 32-channel block
    const int j = lane & 15, half = (lane >> 4) & 1, khalf = lane >> 5;
    // lane-constant window position of its output position (tap 0,0)
    const int off_lane = (((j >> 2) * g.str_y) * g.ww + (j & 3) * g.str_x) * g.sc * 16;
    // this lane's rows of the window offset table: its position's share of the chunk rotation, its K pairs
    const int2* tp = tab + (((g.rot_a * (j >> 2) + g.rot_b * (j & 3)) & (g.rot_p - 1)) * 2 + khalf) * g.nq;
    // channel (within the filter group) of register 4*gq of block c; the 4 registers are 4 consecutive channels
    auto chan = [&](int c, int gq) { return (cbg * NCB + c) * 32 + 8 * gq + 4 * khalf; };
    const unsigned int slab_src_bytes = (unsigned int)(g.sc * 16);  // source bytes between consecutive slabs

    int gs = 0;  // stages (slabs) done so far: the window buffer, and the weight buffer if there are two, alternate

    // The two roles run the same loops (ranking rounds, units, slabs) and meet at the same barriers, but
    // each in its own copy of the loops: what one role keeps in registers across iterations is not live
    // in the other's code.
    if (producer) {
    const args_t pargs = hidden(args);
    const auto& g = pargs->g;
    const unsigned char *const src0 = full ? g.xfull : pargs->src0, *const src1 = pargs->src1, *const zero16 = pargs->zero16;
    const int nslab = kept(g.nslab), src_h = kept(g.src_h), src_w = kept(g.src_w);
    if (MODE == MODE_DELTA) {
        load_rows();
        stage_weights(0, 0);
    }
    for (int r0 = 0; r0 < my_nunits; r0 += ur) {
    const int r1 = min(r0 + ur, my_nunits);
    // ---- ranking round: the sub-tile ids of units r0 .. r1-1 of this workgroup go to s_list ------------
    if (MODE == MODE_DELTA) {
        if (r0 > 0) __syncthreads();  // the previous round's list is no longer in use
        if (listed && !own_group) {  // (own_group: the list was made with the count)
            // The rank of a set flag is the number of set flags before it; this workgroup owns the ranks
            // unit*per .. unit*per + per - 1 of its units.
            int before = 0;
            for (int w = 0; w < wave; ++w) before += s_scan[w];
            ranks.fill(s_list, before, eshift, per, g.magic_per[per], BX, GX, g.magic_gx, r0, r1);
        }
        lds_barrier();  // the list is published
    } else if (r0 == 0) {
        lds_barrier();  // (the window offset table is published)
    }


    for (int iu = r0; iu < r1; ++iu) {
    const int unit = bx + iu * gx;
    const int first = unit * per;
    int mycount = count - first;
    if (mycount > per) mycount = per;
    {
        // ---- window origins of the unit's sub-tiles (each producer wavefront keeps its own copy: no barrier) --
        if (lane < mycount) {
            const int id = listed ? s_list[(iu - r0) * per + lane] : first + lane;
            const int b = (int)udiv_magic((unsigned int)id, (unsigned int)(g.sty * g.stx), g.magic_sub);
            const int r = id - b * (g.sty * g.stx);
            const int sy = (int)udiv_magic((unsigned int)r, (unsigned int)g.stx, g.magic_stx), sx = r - sy * g.stx;
            const int iy0 = 4 * sy * g.str_y - g.pad_y, ix0 = 4 * sx * g.str_x - g.pad_x;
            s_iy0[wave][lane] = iy0;
            s_ix0[wave][lane] = ix0;
            s_base[wave][lane] = (unsigned int)((b * src_h + iy0) * src_w + ix0) * (unsigned int)g.pos_bytes +
                                 (unsigned int)(grp * g.grp_bytes);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // LDS operations of one wavefront execute in order
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // ---- window staging ----------------------------------------------------------------------------
        // A staged unit is 16 bytes of one (sub-tile, window position, chunk-in-slab).  Unit v lives at LDS
        // byte 16*v of its plane, v = (slot*wpos + hp)*sc + cs, where slot cs of a position holds chunk
        // (cs - rotation(position)) mod rot_p, so that the MFMA operand reads of a sub-tile's 16 positions
        // fall into different banks.  Consecutive lanes own consecutive units, which is what the LDS-direct
        // gather (per-lane global address, LDS address = wave base + 16*lane) needs.  The decomposition
        // does not depend on the slab or on the sub-tiles, so it comes from a table made at create time; a
        // thread adds the window origins of its units' sub-tiles once per work unit, and a slab only adds
        // its channel offset.  Units outside the image, or whose chunk does not exist in the last slab,
        // read a 16-byte block of zeros instead.
        const int units = mycount * g.wpos * g.sc;
        const int my_units = units > tid ? (units - tid + CONV_THREADS - 1) / CONV_THREADS : 0;  // this thread's share
        unsigned int uoff[MAXU];   // source byte offset at slab 0, 0xFFFFFFFF = zeros
        unsigned int ulast = 0;    // bit i: unit i's chunk does not exist in the last slab
#pragma unroll
        for (int i = 0; i < MAXU; ++i) {
            uoff[i] = 0xFFFFFFFFu;
            if (i < my_units) {
                const int2 u = ut[i];
                const int slot = u.x & 31, hy = (u.x >> 5) & 255, hx = (u.x >> 13) & 255;
                const int iy = s_iy0[wave][slot] + hy, ix = s_ix0[wave][slot] + hx;
                ulast |= (unsigned int)((u.x >> 21) & 1) << i;
                if (iy >= 0 && iy < src_h && ix >= 0 && ix < src_w) uoff[i] = s_base[wave][slot] + (unsigned int)u.y;
            }
        }
        auto stage_windows = [&](int slab, int buf) {
            unsigned char* dst = bbase + buf * b_bytes;
            const bool last = slab == nslab - 1;
#pragma unroll
            for (int i = 0; i < MAXU; ++i) {
                if (i >= my_units) break;
                const bool real = uoff[i] != 0xFFFFFFFFu && !(last && ((ulast >> i) & 1u));
                const unsigned int o = uoff[i] + (unsigned int)slab * slab_src_bytes;
                unsigned char* d = dst + (i * CONV_THREADS + wave * 64) * 16;  // wave-uniform; lane adds 16*lane
                const unsigned char* p0 = real ? src0 + o : zero16;
                __builtin_amdgcn_global_load_lds((gptr_t)p0, (lptr_t)d, 16, 0, 0);
                if (TERMS == 2 && !full) {
                    const unsigned char* p1 = real ? src1 + o : zero16;
                    __builtin_amdgcn_global_load_lds((gptr_t)p1, (lptr_t)(d + plane_bytes), 16, 0, 0);
                }
            }
        };
        // Stage by stage: slab k of this unit goes into the buffers of parity gs + k.  Slab 0 is staged
        // while the consumers still multiply the previous unit's last slab (other parity).
        if (nbuf_a == 2 && iu > 0) stage_weights(0, gs & 1);  // (the very first slab was started at kernel entry)
        stage_windows(0, gs & 1);
        for (int k = 0; k < nslab; ++k) {
            __builtin_amdgcn_s_waitcnt(0);  // this wavefront's copies for slab k have landed in LDS
            __syncthreads();                // slab k is published; the consumers are done with slab k-1
            ++gs;
            if (k + 1 < nslab) {
                stage_weights(k + 1, gs & 1);
                stage_windows(k + 1, gs & 1);
            }
        }
        if (KSPLIT && ksh) lds_barrier();  // (the consumers exchange their parts' sums)
    }
    }  // units of the round
    }  // rounds
    } else {
    const args_t cargs = hidden(args);
    const auto& g = cargs->g;
    sc_t* const y = static_cast<sc_t*>(cargs->y);
    const sc_t* const bias = static_cast<const sc_t*>(cargs->bias);
    const int nslab = kept(g.nslab), nq = kept(g.nq), nt = kept(g.nt), slot_bytes = kept(g.slot_bytes), tiles = kept(g.sty * g.stx),
              stx = kept(g.stx), ho = kept(g.ho), wo = kept(g.wo), c_out = kept(g.c_out), og = kept(g.og);
    const unsigned int magic_sub = kept(g.magic_sub), magic_stx = kept(g.magic_stx);
    // Consumer state of a unit: this lane's output position of its sub-tile, the accumulators, and what the result is
    // added to -- the stored projection (delta: Algorithm 1, P_t = P_{t-1} + F * dI) or the bias (dense: Eq. 3).
    // `base` is fetched as soon as the previous unit's results are stored (the sub-tile ids come from the ranked
    // list, not from the producers) and is needed only after the unit's last slab: accumulators that start from it
    // would hold up the unit's first product until these loads, and the previous unit's stores before them (memory
    // operations of a wavefront are waited for in order), are done.  A dense launch, and the two-term 16-slot shape,
    // which have no registers to spare for it, start the accumulators from `base`.
    // Four outputs at the alignment of one (a position's channels need not be multiples of 4), fewer at the end of a group's channels.
    // (All of
    // such a layer's outputs entry by entry, added to the stored ones at the end: 28 x 28, 128 -> 101, 16 streams, int8 step 25.8 us and 14.6 so,
    // bf16 26.5 and 19.3, bf16 dense 17.5 and 11.6; 59 x 59, 64 -> 469 1 x 1, nine streams, int8 dense 61.9 and 33.0.)
    struct __attribute__((packed, aligned(CUT ? 4 : 16))) quad {
        vec_t v;
    };
    auto load4 = [](const sc_t* p) __attribute__((always_inline)) { return reinterpret_cast<const quad*>(p)->v; };
    auto store4 = [&](sc_t* p, const vec_t& v, int n) __attribute__((always_inline)) {
        if (!CUT || n >= 4) {
            reinterpret_cast<quad*>(p)->v = v;
        } else {
            p[0] = v.x;
            if (n > 1) p[1] = v.y;
            if (n > 2) p[2] = v.z;
        }
    };
    unsigned int ybase;
    bool pos_ok;
    acc_t acc[NCB];
    // fp32 sums of CUT layers always meet it at the end, in the two-term shape of 16 slots and two blocks fetched only then (END_BASE):
    // accumulators that start from it round every product at its magnitude (relative error of 40 x 40, 48 -> 18 1 x 1, 40 streams,
    // 3.75e-8 so and 3.57e-8, of 56 x 56, 24 -> 101, 20 streams, 5 % changed, 6.67e-8 and 6.53e-8, whose step takes 17.5 and 18.6 us).
    constexpr bool CUT_SUMS = CUT && DT == RRM_BF16_F32;
    constexpr bool LATE_BASE = TERMS == 2 && NT == 16 ? CUT_SUMS && NCB == 1 : MODE == MODE_DELTA || CUT_SUMS;
    constexpr bool END_BASE = CUT_SUMS && !LATE_BASE;
    vec_t base[NCB][LATE_BASE ? 4 : 1];
    auto base_quad = [&](int c, int gq) __attribute__((always_inline)) {
        const int co = chan(c, gq);
        const bool ch_ok = (CUT ? co + 3 : co) < og && owned(gq);
        vec_t v = vec_t{0, 0, 0, 0};
        if (!from_y && ch_ok && bias) v = load4(bias + grp * og + co);
        if (from_y && ch_ok && pos_ok) v = load4(y + (ybase + (unsigned int)co));
        if (CUT && co < og && co + 3 >= og && owned(gq) && (from_y ? pos_ok : bias != nullptr)) {
            const sc_t* const p = from_y ? y + (ybase + (unsigned int)co) : bias + grp * og + co;
            v.x = p[0];
            if (co + 1 < og) v.y = p[1];
            if (co + 2 < og) v.z = p[2];
        }
        return v;
    };
    auto begin_unit = [&](int iu2, int r0) {
        const int first2 = (bx + iu2 * gx) * per;
        const int mycount2 = min(per, count - first2);
        const int slot = 2 * cw + half;
        pos_ok = false;
        ybase = 0;
        if (slot < mycount2) {
            const int id = listed ? s_list[(iu2 - r0) * per + slot] : first2 + slot;
            const int b = (int)udiv_magic((unsigned int)id, (unsigned int)tiles, magic_sub);
            const int r = id - b * tiles;
            const int sy = (int)udiv_magic((unsigned int)r, (unsigned int)stx, magic_stx), sx = r - sy * stx;
            const int oy = 4 * sy + (j >> 2), ox = 4 * sx + (j & 3);
            pos_ok = ox < wo && oy < ho;
            ybase = (unsigned int)((b * ho + oy) * wo + ox) * (unsigned int)c_out + (unsigned int)(grp * og);
        }
#pragma unroll
        for (int c = 0; c < NCB; ++c)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                vec_t v = vec_t{0, 0, 0, 0};
                if constexpr (LATE_BASE)
                    base[c][gq] = base_quad(c, gq);
                else if constexpr (!END_BASE)
                    v = base_quad(c, gq);
                acc[c][4 * gq + 0] = v.x;
                acc[c][4 * gq + 1] = v.y;
                acc[c][4 * gq + 2] = v.z;
                acc[c][4 * gq + 3] = v.w;
            }
    };
    for (int r0 = 0; r0 < my_nunits; r0 += ur) {
    const int r1 = min(r0 + ur, my_nunits);
    // the barriers of the ranking round
    if (MODE == MODE_DELTA) {
        if (r0 > 0) __syncthreads();
        lds_barrier();
    } else if (r0 == 0) {
        lds_barrier();
    }
    begin_unit(r0, r0);
    for (int iu = r0; iu < r1; ++iu) {
    const int unit = bx + iu * gx;
    const int first = unit * per;
    int mycount = count - first;
    if (mycount > per) mycount = per;
    const bool active = mycount > 2 * cw;  // (slots 2*cw, 2*cw + 1)
    {
        // ---- consumers ---------------------------------------------------------------------------------
        // K loop of one slab (an unused second slot reads stale LDS and its results are dropped).  A K step is four K pairs,
        // i.e. two MFMA steps.  Software pipeline: while K step q multiplies, the operands of step q+1 are
        // read from LDS into a second register set (the sets swap roles every step, nothing is copied) and
        // the table entries of step q+2 are fetched, so that no address waits for a table read.  The reads
        // are issued one by one between the MFMAs: a wavefront that issues them in a batch leaves the
        // matrix pipeline idle meanwhile.  What is not a matrix
        // instruction or an operand read is kept off this loop: a pair's window offset comes ready from the table
        // (one add per operand), the weights' addresses are one base per channel block with immediate offsets (67
        // instead of 91 instructions per two K steps of 16 matrix instructions; the five-layer stack 687 -> 674 us at
        // 512 streams, 84.2 -> 80.3 us at one).
        auto k_loop = [&]<int T>(unsigned int aw, unsigned int bw) {  // LDS offsets; T: terms multiplied
            const unsigned int ap = aw + lane * 16;
            // (slots beyond the allocated ones are never in use; their lanes read slot 0 instead of running
            // off the buffer)
            const unsigned int bp = bw + (2 * cw + half < nt ? 2 * cw + half : 0) * slot_bytes + off_lane;
            struct Ops {
                uint4 a[2][NCB], b0[2], b1[2];
            };
            constexpr int N_MFMA = 2 * NCB * T;
            constexpr int N_READ = 2 * (NCB + T);
            auto fetch = [&](int q, const int2& t, Ops& o) {
#pragma unroll
                for (int c = 0; c < NCB; ++c) {
                    unsigned int ao = ap + (unsigned int)(c * nq2 + 2 * q) * 1024u;
                    asm("" : "+v"(ao));  // (one base register for the step's two fragments)
#pragma unroll
                    for (int h = 0; h < 2; ++h) o.a[h][c] = *reinterpret_cast<const uint4*>(lds + ao + h * 1024);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const unsigned int off = bp + (unsigned int)(h ? t.y : t.x);
                    o.b0[h] = *reinterpret_cast<const uint4*>(lds + off);
                    if (T == 2) o.b1[h] = *reinterpret_cast<const uint4*>(lds + plane_bytes + off);
                }
            };
            auto multiply = [&](const Ops& o) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int c = 0; c < NCB; ++c) {
                        acc[c] = mma(o.a[h][c], o.b0[h], acc[c]);
                        if (T == 2) acc[c] = mma(o.a[h][c], o.b1[h], acc[c]);
                    }
            };
            // one K step: multiply `cur`, read step q1 (table entries `t`) into `nxt`, fetch the table entries
            // of step q2 into `tn`; operand sets and table registers swap roles every step, nothing is copied
            auto step = [&](const Ops& cur, Ops& nxt, const int2& t, int2& tn, int q1, int q2) {
                tn = tp[q2];
                fetch(q1, t, nxt);
                multiply(cur);
                // issue order: the table read, then MFMAs with the operand reads spread between them
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                sched_interleave<0, N_MFMA, N_READ>();
            };
            Ops o0, o1;
            int2 ta, tb;
            const int q0 = KSPLIT ? (nq * kpart) >> ksh : 0, q1 = KSPLIT ? (nq * (kpart + 1)) >> ksh : nq;
            if (KSPLIT && q0 >= q1) return;
            const int qmax = q1 - 1;
            // (scalar loads and LDS reads share a counter: with none of the former under way the loop's waits are counted ones)
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
            tb = tp[q0];
            fetch(q0, tb, o0);
            ta = tp[min(q0 + 1, qmax)];
            // Two matrix instructions a step do not hide where the loop lies in the 32-byte lines that instructions are fetched in: it
            // begins eight bytes into one, the fastest of the eight places.  (us a call over them, long windows that leave short
            // slabs, five streams of 46 x 25, 456 -> 144, 5 x 5 bf16: half changed, recomputed, 71.4 .. 74.9, dense 57.2 .. 60.9; 448 ->
            // 144 int8 dense 38.3 .. 41.2.  The other shapes' times are within 1 % of each other.)
            if constexpr (KSPLIT && T == 1) asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0");
            for (int q = q0; q < q1; q += 2) {
                step(o0, o1, ta, tb, min(q + 1, qmax), min(q + 2, qmax));
                if (q + 1 < q1) step(o1, o0, tb, ta, min(q + 2, qmax), min(q + 3, qmax));
            }
        };

        for (int k = 0; k < nslab; ++k) {
            // slab k is staged.  A bare barrier: the producers waited for their copies before they arrived,
            // and this wavefront's own stores and loads of stored projections (previous / this unit) need not
            // have completed -- __syncthreads() would wait for all of them.
            asm volatile("s_barrier" ::: "memory");
            const unsigned int aw = (unsigned int)((nbuf_a == 2 ? (gs & 1) : 0) * a_bytes);
            const unsigned int bw = (unsigned int)(nbuf_a * a_bytes + (gs & 1) * b_bytes);
            ++gs;
            if (TERMS == 2 && !full) {
                if constexpr (TERMS == 2)
                    if (active) k_loop.template operator()<2>(aw, bw);
            } else if (active) {
                k_loop.template operator()<1>(aw, bw);
            }
        }

        if (KSPLIT && ksh) {
            // the K parts' sums: every part leaves the quads that it does not finish in LDS and adds the others' to its own,
            // in the order of the parts
            vec_t* part = reinterpret_cast<vec_t*>(lds + nbuf_a * a_bytes + 2 * b_bytes + conv_tab_words(g) * (int)sizeof(int));
            const int prow = cw << ksh;  // rows of this pair: [part][quad][lane]
#pragma unroll
            for (int gq = 0; gq < 4; ++gq)
                if (active && !owned(gq))
                    part[((prow + kpart) * 4 + gq) * WAVE + lane] =
                        vec_t{acc[0][4 * gq + 0], acc[0][4 * gq + 1], acc[0][4 * gq + 2], acc[0][4 * gq + 3]};
            lds_barrier();
            if (active)
                for (int o = 0; o < (1 << ksh); ++o) {
                    if (o == kpart) continue;
#pragma unroll
                    for (int gq = 0; gq < 4; ++gq)
                        if (owned(gq)) {
                            const vec_t v = part[((prow + o) * 4 + gq) * WAVE + lane];
                            acc[0][4 * gq + 0] += v.x;
                            acc[0][4 * gq + 1] += v.y;
                            acc[0][4 * gq + 2] += v.z;
                            acc[0][4 * gq + 3] += v.w;
                        }
                }
        }

        // ---- epilogue ----------------------------------------------------------------------------------
        if constexpr (LATE_BASE || END_BASE)
#pragma unroll
            for (int c = 0; c < NCB; ++c)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    vec_t v;
                    if constexpr (LATE_BASE)
                        v = base[c][gq];
                    else
                        v = base_quad(c, gq);
                    acc[c][4 * gq + 0] += v.x;
                    acc[c][4 * gq + 1] += v.y;
                    acc[c][4 * gq + 2] += v.z;
                    acc[c][4 * gq + 3] += v.w;
                }
        // (the store addresses are rebuilt from ybase here: kept across the K loops they would cost two
        // registers per store)
        asm volatile("" : "+v"(ybase));
        // The MFMA layout gives a lane 4 consecutive channels of ONE position, so a store instruction writes
        // 32-byte pieces of 32 different rows of y; measured, read-modify-writing an output tile that way runs at
        // 5.9 TB/s against 8 TB/s when the stores are whole 128-byte rows.  So each result block (32 positions x
        // 32 channels) is turned through LDS first: written in the MFMA layout, read back with 8 lanes along the
        // channels of a position, 8 positions per store.  The scratch is the window area of this wavefront's own
        // two slots in the buffer of the slab just finished: only this wavefront reads those windows, and
        // the producers are filling the other buffer.
        constexpr int RP = 36;  // words per position row of the scratch (16-byte aligned, spreads the banks)
        if (!active) {
            // (no pair in this unit, perhaps no slots at all: a 12-slot layer on the 16-slot shape)
        } else if (nt >= 8 && 2 * slot_bytes >= 32 * RP * 4) {
            vec_t* scr = reinterpret_cast<vec_t*>(bbase + ((gs - 1) & 1) * b_bytes + (2 * cw) * slot_bytes);
            const int posl = lane & 31;
            // the two sub-tiles of the pair (the same in every lane)
            unsigned int corner[2];
            int ny[2], nx[2];
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                const int slot = 2 * cw + sl;
                corner[sl] = 0;
                ny[sl] = nx[sl] = 0;
                if (slot < mycount) {
                    const int id = listed ? s_list[(iu - r0) * per + slot] : first + slot;
                    const int b = (int)udiv_magic((unsigned int)id, (unsigned int)tiles, magic_sub);
                    const int r = id - b * tiles;
                    const int sy = (int)udiv_magic((unsigned int)r, (unsigned int)stx, magic_stx), sx = r - sy * stx;
                    ny[sl] = ho - 4 * sy;
                    nx[sl] = wo - 4 * sx;
                    corner[sl] = (unsigned int)((b * ho + 4 * sy) * wo + 4 * sx) * (unsigned int)c_out +
                                 (unsigned int)(grp * og);
                }
            }
#pragma unroll
            for (int c = 0; c < NCB; ++c) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // (the previous block's reads are done)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    vec_t o;
                    o.x = acc[c][4 * gq + 0];
                    o.y = acc[c][4 * gq + 1];
                    o.z = acc[c][4 * gq + 2];
                    o.w = acc[c][4 * gq + 3];
                    scr[(posl * RP + 8 * gq + 4 * khalf) >> 2] = o;
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // LDS operations of a wavefront execute in order
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const int ch = (cbg * NCB + c) * 32 + 4 * (lane & 7);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int q = 8 * i + (lane >> 3);  // position of the pair: sub-tile q / 16, position q % 16
                    const vec_t o = scr[(q * RP + 4 * (lane & 7)) >> 2];
                    const int sl = i >> 1, py = 2 * (i & 1) + (lane >> 5), px = (lane >> 3) & 3;
                    if (py < ny[sl] && px < nx[sl] && ch < og) store4(y + (corner[sl] + (unsigned int)((py * wo + px) * c_out + ch)), o, og - ch);
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < NCB; ++c)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const int co = chan(c, gq);
                    if (co >= og || !pos_ok || !owned(gq)) continue;
                    vec_t o;
                    o.x = acc[c][4 * gq + 0];
                    o.y = acc[c][4 * gq + 1];
                    o.z = acc[c][4 * gq + 2];
                    o.w = acc[c][4 * gq + 3];
                    store4(y + (ybase + (unsigned int)co), o, og - co);
                }
        }
        if (iu + 1 < r1) begin_unit(iu + 1, r0);  // (a new round's first unit waits for its ranking)
    }
    }  // units of the round
    }  // rounds
    }
}

template <int DT, int MODE, int NCB, int NT, int TERMS, bool CUT>
hipError_t launch_one(const void* src0, const void* src1, const void* zero16, unsigned int* flags,
                      const void* wpack, const int* offtab, const void* bias, void* y,
                      const ConvGeom& g, DevStats* stats, hipStream_t s) {
    const int ncbg = (g.ncb + NCB - 1) / NCB;
    const size_t lds = conv_lds_bytes(g, NCB, g.nt, TERMS);
    // no more workgroups than are resident at once (the kernel loops over its work units)
    const int gy = g.groups * ncbg;
    const int resident = NUM_CU;  // eight wavefronts with up to 256 registers each fill a compute unit
    int gx = std::min((g.n_sub + g.nt - 1) / g.nt, std::max(1, resident / gy));
    dim3 grid((unsigned int)gx, (unsigned int)gy);
    // A full grid (more units than lanes): one-dimensional, with the channel-block groups of a lane on one XCD
    // (see the kernel).
    ConvGeom gg = g;
    gg.gx = gx;
    gg.gy = gy;
    gg.gyg = ncbg;
    gg.magic_gx = magic_of(gx);
    gg.magic_gy = magic_of(gy);
    gg.magic_gyg = magic_of(ncbg);
    gg.xcd_deal = gx >= 8 && gx == resident / gy;
    if (gg.xcd_deal) grid = dim3((unsigned int)(gx * gy), 1u);
    auto kern = conv_gather_kernel<DT, MODE, NCB, NT, TERMS, CUT>;
    if (lds > 64 * 1024) {
        // one per instantiation, shared by every handle and thread of the process: guarded, so that
        // distinct handles stay independent
        static std::mutex mu;
        static size_t granted = 0;
        std::lock_guard<std::mutex> lock(mu);
        if (lds > granted) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            granted = lds;
        }
    }
    const ConvArgs args{static_cast<const unsigned char*>(src0), static_cast<const unsigned char*>(src1),
                        static_cast<const unsigned char*>(zero16), flags, static_cast<const uint4*>(wpack), offtab, bias, y, stats, gg};
    hipLaunchKernelGGL(kern, grid, dim3(wg_threads(NT)), lds, s, args);
    return hipGetLastError();
}

template <int DT, int MODE, int TERMS>
hipError_t launch_shape(int ncb, int nt, const void* src0, const void* src1, const void* zero16,
                        unsigned int* flags, const void* wpack, const int* offtab, const void* bias, void* y,
                        const ConvGeom& g, DevStats* stats, hipStream_t s) {
#define RRM_CASE(CBV, NTV)                                                                                          \
    if (ncb == CBV && nt == NTV)                                                                                     \
        return g.og % 4 ? launch_one<DT, MODE, CBV, NTV, TERMS, true>(src0, src1, zero16, flags, wpack, offtab, bias, y, g, stats, s) \
                        : launch_one<DT, MODE, CBV, NTV, TERMS, false>(src0, src1, zero16, flags, wpack, offtab, bias, y, g, stats, s);
    nt = nt <= 8 ? 8 : 16;  // fewer slots than the shape has: same code, the slot count is in g.nt
    RRM_CASE(2, 16) RRM_CASE(2, 8) RRM_CASE(1, 16) RRM_CASE(1, 8)
#undef RRM_CASE
    return hipErrorInvalidValue;
}

}  // namespace

size_t conv_lds_bytes(const ConvGeom& g, int ncb, int nt, int terms) {
    return (size_t)(g.nslab > 1 ? 2 : 1) * (size_t)ncb * 2 * g.nq * 1024 + 2 * (size_t)terms * nt * g.slot_bytes +
           (size_t)conv_tab_words(g) * sizeof(int) + (g.ksh ? CONV_PART_BYTES : 0);
}

hipError_t launch_conv(int dtype, int mode, int ncb, int nt, int terms, const void* src0, const void* src1,
                       const void* zero16, unsigned int* flags, const void* wpack, const int* offtab,
                       const void* bias, void* y, const ConvGeom& g, DevStats* stats, hipStream_t s) {
    if (dtype == RRM_I8_I32) {
        if (mode == MODE_DELTA)
            return launch_shape<RRM_I8_I32, MODE_DELTA, 1>(ncb, nt, src0, src1, zero16, flags, wpack, offtab, bias, y, g, stats, s);
        return launch_shape<RRM_I8_I32, MODE_DENSE, 1>(ncb, nt, src0, src1, zero16, flags, wpack, offtab, bias, y, g, stats, s);
    }
    if (mode == MODE_DENSE)
        return launch_shape<RRM_BF16_F32, MODE_DENSE, 1>(ncb, nt, src0, src1, zero16, flags, wpack, offtab, bias, y, g, stats, s);
    if (terms == 2)
        return launch_shape<RRM_BF16_F32, MODE_DELTA, 2>(ncb, nt, src0, src1, zero16, flags, wpack, offtab, bias, y, g, stats, s);
    return launch_shape<RRM_BF16_F32, MODE_DELTA, 1>(ncb, nt, src0, src1, zero16, flags, wpack, offtab, bias, y, g, stats, s);
}

}  // namespace rrm
