// postab.h -- the column -> position hash table of one row held in LDS,
// shared by the numeric and adjoint kernels.
#pragma once

#include "common.h"

namespace mls {

// Column -> position table of one row of C, in one of two layouts:
//   wide  : int2 slots (column, position), any column count;
//   packed: one uint32 per slot, column << PB | position, with PB bits for the
//           position (positions < CAP/2). Usable when every column index of C
//           fits in the remaining bits; halves the bytes of every lookup.
// Empty slots hold -1 (all ones); a packed key never equals it because the
// column range excludes the all-ones column field.
template <int CAP>
struct PackBits {
    static constexpr int PB = CAP == 64 ? 5 : (CAP == 256 ? 7 : (CAP == 1024 ? 9 : (CAP == 2048 ? 10 : 11)));
    static_assert(CAP == 64 || CAP == 256 || CAP == 1024 || CAP == 2048 || CAP == 4096, "table class");
    static constexpr uint32_t kMaxCols = (1u << (32 - PB)) - 1u;   // columns < this fit
};

// Bucket words of a packed table: BK = 2 or 4 slots read in one LDS access.
template <int BK> struct BucketT;
template <> struct BucketT<2> {
    using T = uint2;
    __device__ __forceinline__ static uint32_t minx(T w, uint32_t k) { return min(w.x ^ k, w.y ^ k); }
    __device__ __forceinline__ static uint32_t last(T w) { return w.y; }
    __device__ __forceinline__ static int first_empty(T w, uint32_t e) { return w.x == e ? 0 : (w.y == e ? 1 : 2); }
};
template <> struct BucketT<4> {
    using T = uint4;
    __device__ __forceinline__ static uint32_t minx(T w, uint32_t k)
    {
        return min(min(w.x ^ k, w.y ^ k), min(w.z ^ k, w.w ^ k));
    }
    __device__ __forceinline__ static uint32_t last(T w) { return w.w; }
    __device__ __forceinline__ static int first_empty(T w, uint32_t e)
    {
        return w.x == e ? 0 : (w.y == e ? 1 : (w.z == e ? 2 : (w.w == e ? 3 : 4)));
    }
};

template <int CAP, bool PACK, int BK = 4>
struct PosTab {
    static_assert(BK == 2 || BK == 4, "bucket of 2 or 4 slots");
    using BT = BucketT<BK>;
    using BW = typename BT::T;
    static constexpr int LB = BK == 2 ? 1 : 2;   // log2 of the bucket width
    static constexpr int PB = PackBits<CAP>::PB;
    // a lookup's result is a position when it is at most kMaxPos
    static constexpr uint32_t kMaxPos = PACK ? (1u << PB) - 1u : 0x7fffffffu;
    static constexpr uint32_t kEmpty = 0xffffffffu;
    uint32_t *t;             // CAP words (packed) or 2*CAP words (wide)
    int logcap = 0;          // slots of the current row's table: 2^logcap
    uint32_t sh = 0, bm = 0; // packed: home bucket of a column, as a byte offset: (hash >> sh) & bm

    // The current row's table: at least twice its n columns, at least 32 slots.
    __device__ __forceinline__ void open(int n, int lane, int G)
    {
        logcap = ilog2_ceil(2 * n);
        if (logcap < 5) logcap = 5;
        const int cap = 1 << logcap;
        if (PACK) {
            sh = (uint32_t)(22 - logcap);
            bm = 4u * (uint32_t)cap - (4u << LB);
            if (cap >= 4 * G) {
                for (int h = 4 * lane; h < cap; h += 4 * G)
                    *(uint4 *)(t + h) = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
            } else {
                for (int h = lane; h < cap; h += G) t[h] = kEmpty;
            }
        } else {
            for (int h = lane; h < cap; h += G) ((int2 *)t)[h] = make_int2(-1, 0);
        }
    }

    // Packed tables are probed a bucket (BK slots, one LDS read) at a time: a key
    // takes the first empty slot at or after the start of its home bucket, so
    // the filled slots of every bucket are a prefix of it (a lane only claims
    // a slot after seeing every earlier one taken, and slots are never
    // emptied), and a bucket whose last slot is empty ends a search. Buckets
    // are addressed by byte offset; bm, all ones but a bucket's own bits, also
    // wraps the offset of the next one.
    __device__ __forceinline__ uint32_t home(int j) const { return (__umul24((uint32_t)j, kHashMul) >> sh) & bm; }
    __device__ __forceinline__ BW bucket(uint32_t h) const { return *(const BW *)((const char *)t + h); }

    __device__ __forceinline__ void insert(int j, int pos)
    {
        const uint32_t cap = 1u << logcap;
        if (PACK) {
            const uint32_t v = ((uint32_t)j << PB) | (uint32_t)pos;
            uint32_t h = home(j);
            for (uint32_t probe = 0; probe < cap; probe += BK) {
                int sl = BT::first_empty(bucket(h), kEmpty);
                for (; sl < BK; ++sl)
                    if (atomicCAS(t + (h >> 2) + sl, kEmpty, v) == kEmpty) return;
                h = (h + (4u << LB)) & bm;
            }
        } else {
            uint32_t h = hslot32((uint32_t)j, logcap);
            int2 *tab = (int2 *)t;
            for (uint32_t probe = 0; probe < cap; ++probe) {
                int old = atomicCAS(&tab[h].x, -1, j);
                if (old == -1) { tab[h].y = pos; return; }
                h = (h + 1u) & (cap - 1u);
            }
        }
    }

    // Packed: a slot holds column j iff its word XOR (j << PB) is at most
    // kMaxPos, and that value is then the position; at most one slot of a
    // bucket holds j, so the minimum over the bucket decides.

    // the search past a full home bucket h (rarely needed)
    __device__ __forceinline__ uint32_t find_more(uint32_t key, uint32_t h) const
    {
        const uint32_t cap = 1u << logcap;
        for (uint32_t probe = BK; probe < cap; probe += BK) {
            h = (h + (4u << LB)) & bm;
            const BW v = bucket(h);
            const uint32_t mv = BT::minx(v, key);
            if (mv <= kMaxPos || BT::last(v) == kEmpty) return mv;
        }
        return kEmpty;
    }

    // position of column j (j >= 0), or more than kMaxPos when it is not in the row
    __device__ __forceinline__ uint32_t lookup(int j) const
    {
        if (PACK) {
            const uint32_t h = home(j), key = (uint32_t)j << PB;
            const BW w = bucket(h);
            const uint32_t m = BT::minx(w, key);
            return m <= kMaxPos || BT::last(w) == kEmpty ? m : find_more(key, h);
        } else {
            const uint32_t cap = 1u << logcap;
            uint32_t h = hslot32((uint32_t)j, logcap);
            const int2 *tab = (const int2 *)t;
            for (uint32_t probe = 0; probe < cap; ++probe) {
                const int2 v = tab[h];
                if (v.x == j) return (uint32_t)v.y;
                if (v.x == -1) return kEmpty;
                h = (h + 1u) & (cap - 1u);
            }
        }
        return kEmpty;
    }

    // positions of D columns (meaningless where ok is false): the home buckets
    // of two are read before either is searched (four buckets in registers
    // would cost 16 VGPRs)
    template <int D>
    __device__ __forceinline__ void lookup_n(const int (&jv)[D], const bool (&ok)[D], uint32_t (&pos)[D]) const
    {
        static_assert(D % 2 == 0, "looked up in pairs");
        if (PACK) {
#pragma unroll
            for (int d0 = 0; d0 < D; d0 += 2) {
                uint32_t hv[2];
                BW wv[2];
#pragma unroll
                for (int d = 0; d < 2; ++d) hv[d] = home(jv[d0 + d]);
#pragma unroll
                for (int d = 0; d < 2; ++d) wv[d] = bucket(hv[d]);
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const uint32_t key = (uint32_t)jv[d0 + d] << PB;
                    uint32_t m = BT::minx(wv[d], key);
                    if (ok[d0 + d] && m > kMaxPos && BT::last(wv[d]) != kEmpty) m = find_more(key, hv[d]);
                    pos[d0 + d] = m;
                }
            }
        } else {
#pragma unroll
            for (int d = 0; d < D; ++d) pos[d] = ok[d] ? lookup(jv[d]) : kEmpty;
        }
    }
};

}  // namespace mls
