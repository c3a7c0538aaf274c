// The flagged sub-tiles of a delta launch, ranked: how many there are, and which of them a workgroup's share of the ranks are.
//
// A launch is over in a few microseconds and every workgroup makes its list for itself, so the list is a chain of round trips
// and cross-lane steps that nothing hides.  16 flags (one 16-byte vector) per lane and round, neighbouring lanes reading
// neighbouring vectors, eight rounds in flight together; the first eight rounds' masks stay in registers.  The
// vectors that hold a flag of the workgroup's units are few; they go to the list one after the other, a lane per flag.
// (Clocks from the count to the finished list, 227 x 227 -> 55 x 55, 512 streams, 60 % of 100352 sub-tiles flagged: 46 k with a
// binary search per rank over 64-flag masks, 27 k so; 784 sub-tiles, half of them flagged: 8.3 k and 6.2 k, the first loads of
// weights and tables included.)
#pragma once
#include "rrm_internal.h"

namespace rrm {

#ifdef __HIPCC__

// Four wavefronts (`wave` 0 .. 3), each with a contiguous quarter of the flag array.
struct SubtileList {
    static constexpr int BATCH = 8;  // rounds read together; the first batch stays in registers (32768 sub-tiles)
    const uint4* fv;
    int n_vec, rounds, wave, lane;
    unsigned int m[BATCH / 2];  // masks of rounds 2 i (low half) and 2 i + 1

    __device__ __forceinline__ int vec_at(int r) const { return (wave * rounds + r) * WAVE + lane; }
    // byte flags with the bit 1 << eshift of a vector -> 16 bits (a dot product sums its four bytes, weighted by their places)
    static __device__ __forceinline__ unsigned int squeeze(const uint4& v, unsigned int eshift) {
        const unsigned int bit = 0x01010101u << eshift;
        const unsigned int lo = __builtin_amdgcn_udot4(v.y & bit, 0x80402010u, __builtin_amdgcn_udot4(v.x & bit, 0x08040201u, 0u, false), false);
        const unsigned int hi = __builtin_amdgcn_udot4(v.w & bit, 0x80402010u, __builtin_amdgcn_udot4(v.z & bit, 0x08040201u, 0u, false), false);
        return (lo | hi << 8) >> eshift;
    }
    // the masks of rounds r0 .. r0 + BATCH - 1 (every lane reads something: a round or vector that is not there counts as zero)
    template <typename F>
    __device__ __forceinline__ void masks(int r0, unsigned int (&mm)[BATCH / 2], F eshift) const {
        uint4 v[BATCH];
        auto at = [&](int k) __attribute__((always_inline)) { return (unsigned int)min(vec_at(r0 + k), n_vec - 1); };
        v[0] = fv[at(0)];
        if (rounds > 1) {
#pragma unroll
            for (int k = 1; k < BATCH; ++k) v[k] = fv[at(k)];
        } else {
#pragma unroll
            for (int k = 1; k < BATCH; ++k) v[k] = uint4{0u, 0u, 0u, 0u};
        }
        const unsigned int e = eshift();
#pragma unroll
        for (int k = 0; k < BATCH; k += 2) {
            auto one = [&](int kk) __attribute__((always_inline)) {
                const unsigned int q = squeeze(v[kk], e);
                return ((r0 + kk < rounds) & (vec_at(r0 + kk) < n_vec)) ? q : 0u;
            };
            mm[k / 2] = one(k) | one(k + 1) << 16;
        }
    }

    // Reads the flags; returns the wavefront's count.  `epoch`: the device words of StepEpoch.
    __device__ __forceinline__ int count(const unsigned int* flags, int n_words, const unsigned int* epoch, int wave_, int lane_,
                                         unsigned int& eshift) {
        fv = reinterpret_cast<const uint4*>(flags);
        n_vec = (n_words + 3) >> 2;
        rounds = (n_vec + 4 * WAVE - 1) / (4 * WAVE);
        wave = wave_;
        lane = lane_;
        masks(0, m, [&]() __attribute__((always_inline)) { return eshift = epoch[EPOCH_TILE] - 1u; });
        int n = 0;
#pragma unroll
        for (int k = 0; k < BATCH / 2; ++k) n += __popc(m[k]);
        for (int r0 = BATCH; r0 < rounds; r0 += BATCH) {
            unsigned int mm[BATCH / 2];
            masks(r0, mm, [&]() __attribute__((always_inline)) { return eshift; });
#pragma unroll
            for (int k = 0; k < BATCH / 2; ++k) n += __popc(mm[k]);
        }
        return __builtin_amdgcn_readlane((int)wave_scan((unsigned int)n), 63);
    }

    // The ids of ranks lo .. lo + per - 1 of the units first + i * step, i = i0 .. i1 - 1 (lo = unit * per), go to
    // list[(i - i0) * per ..]; `before`: flags of the wavefronts before this one; mper, mstep: reciprocals of per, step.
    __device__ __forceinline__ void fill(int* list, int before, unsigned int eshift, int per, unsigned int mper, int first, int step,
                                         unsigned int mstep, int i0, int i1) const {
        unsigned int mm[BATCH / 2];
#pragma unroll
        for (int k = 0; k < BATCH / 2; ++k) mm[k] = m[k];
        for (int r0 = 0;;) {
#pragma unroll 1
            for (int r = r0; r < r0 + BATCH && r < rounds; r += 2) {
                // two rounds' counts are summed at once (at most 1024 each)
                const unsigned int two = mm[0];
#pragma unroll
                for (int k = 0; k + 1 < BATCH / 2; ++k) mm[k] = mm[k + 1];
                const unsigned int pc = (unsigned int)__popc(two & 0xFFFFu) | (unsigned int)__popc(two >> 16) << 16;
                const unsigned int incl = wave_scan(pc), ex = incl - pc;
                const unsigned int all = (unsigned int)__builtin_amdgcn_readlane((int)incl, 63);
#pragma unroll 1
                for (int h = 0; h < 2; ++h) {
                    const unsigned int mask = two >> 16 * h & 0xFFFFu;
                    const int b = before + (int)(ex >> 16 * h & 0xFFFFu);  // rank of the vector's first flag
                    // the workgroup's first unit that ends behind rank b
                    const int over = (int)udiv_magic((unsigned int)b, (unsigned int)per, mper) - first;
                    int i = over <= 0 ? 0 : (int)udiv_magic((unsigned int)(over + step - 1), (unsigned int)step, mstep);
                    if (i < i0) i = i0;
                    // vectors with a flag of such a unit, one after the other: a lane per flag
                    unsigned long long todo = __ballot(mask && i < i1 && (first + i * step) * per < b + __popc(mask));
                    while (todo) {
                        const int l = __ffsll((long long)todo) - 1;
                        todo &= todo - 1ull;
                        const unsigned int vm = (unsigned int)__builtin_amdgcn_readlane((int)mask, l);
                        const int vb = __builtin_amdgcn_readlane(b, l), ve = vb + __popc(vm);
                        const int t = vb + __popc(vm & ((1u << (lane & 15)) - 1u));
                        const bool mine = lane < 16 && (vm >> (lane & 15) & 1u);
                        for (int u = __builtin_amdgcn_readlane(i, l); u < i1; ++u) {
                            const int lo = (first + u * step) * per;
                            if (lo >= ve) break;
                            if (mine && t >= lo && t < lo + per) list[(u - i0) * per + t - lo] = ((wave * rounds + r + h) * WAVE + l) * 16 + lane;
                        }
                    }
                    before += (int)(all >> 16 * h & 0xFFFFu);
                }
            }
            r0 += BATCH;
            if (r0 >= rounds) break;
            masks(r0, mm, [&]() __attribute__((always_inline)) { return eshift; });
        }
    }
};

#endif

}  // namespace rrm
