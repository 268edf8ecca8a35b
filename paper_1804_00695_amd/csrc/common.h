// common.h -- device-side descriptors and helpers shared by the gfx950 kernels.
//
// Every kernel works on a *batch* of independent products C_t = A_t * B_t
// (a single product is a batch of one). Rows of all A_t are numbered in one
// global row space: product t owns global rows [abase[t], abase[t+1]).
// The same holds for the rows of all B_t (bbase). A row-range restriction
// (k_lo, k_hi) and array offsets let the same kernels run on chunk parts
// (the row-range fused multiply-add kernel of the chunking algorithms).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mls {

constexpr int kWG = 256;          // threads per workgroup
constexpr int kWave = 64;         // gfx950 wavefront
constexpr int kXcd = 8;           // MI355X: 8 accelerator complex dies, 32 CUs each
constexpr int kNumClasses = 5;    // LDS classes
constexpr int kNumBins = 7;       // 5 LDS classes, spill, empty
constexpr int kBinSpill = 5;
constexpr int kBinEmpty = 6;

// Error bits (device flag).
constexpr uint32_t kErrBadCsr = 1u;
constexpr uint32_t kErrOverflow = 2u;
constexpr uint32_t kErrStructure = 4u;
constexpr uint32_t kErrTable = 8u;

// LDS capacities (hash slots) of the five classes, per phase. A row goes to
// the first class whose threshold holds; beyond class 3 it spills. The
// smallest class keeps many short rows in flight (small tables, 8 lanes).
//   count  : threshold on the word upper bound u, table = u slots at most
//   fill / numeric : threshold on the exact size n, table >= 2n slots
// (triangle counting keeps a table of its own, on the same rule)
constexpr int kCountCap[kNumClasses] = {64, 256, 512, 2048, 8192};
constexpr int kFillCap[kNumClasses] = {64, 256, 1024, 2048, 4096};

struct Prob {
    // A (or an A/C row part): row pointers hold global entry offsets; the
    // local entry index is row_ptr value - a_off.
    const int32_t *arp;
    const int32_t *aci;
    const double *aval;
    // B (or a B row part): local row = k - k_lo; local entry = brp - b_off.
    const int32_t *brp;
    const int32_t *bci;
    const double *bval;
    // Compressed B pattern, padded layout: row k's words at bw[brp[k]-b_off ...].
    uint2 *bw;
    int32_t *bwc;
    // C: row pointers with offset c_off.
    int32_t *crp;
    int32_t *cci;
    double *cval;
    int32_t nrows;   // rows of A / C
    int32_t ncols;   // columns of B / C
    int32_t krows;   // rows of B held (k_hi - k_lo)
    int32_t a_off, b_off, c_off;
    int32_t k_lo, k_hi;     // A columns outside [k_lo, k_hi) are skipped
    int32_t accumulate;     // numeric: 1 = add onto the values already in C
    int32_t ranged;         // numeric: [k_lo, k_hi) is part of B's rows; a row of at most one
                            // chunk with no entry in it is skipped (its values stay, or are
                            // set to 0 when not accumulating)
};

static_assert(sizeof(Prob) % 16 == 0, "Prob is copied in 16-byte words");

struct Batch {
    const Prob *probs;      // device array [nprob] (used when nprob > 1)
    Prob p0;                // the product when nprob == 1
    const int32_t *abase;   // device [nprob + 1]
    const int32_t *bbase;   // device [nprob + 1]
    int32_t nprob;
    int32_t na;             // total A rows
    int32_t nb;             // total B rows
    int32_t max_ncols;      // largest column count of C over the products (0 = unknown)
};

// Per-phase device state inside the workspace.
enum { kSeenSmall = 0, kSeenMid = 1, kSeenLarge = 2, kSeenMore = 3, kNumSeen = 4 };   // up to 16, 32, 64 words, more

struct Sched {
    uint32_t *err;
    int32_t *bin_count;     // [kNumBins]
    int32_t *blk_cnt;       // [kNumBins * nblk]: rows of each bin per block of kBinRowsPerWG rows,
                            // then (after the bin scan) where those rows start in perm
    int32_t nblk;
    int32_t *task_cursor;   // [kNumBins * kXcd]
    int32_t *val;           // per global row: size used for binning / result
    uint8_t *cls;           // per global row: bin
    int32_t *perm;          // rows grouped by bin
    // symbolic scratch: the count pass leaves each row's compacted (set, mask)
    // words here (up to kScratchWords per row; scnt = -1 when a row has more)
    // and the fill pass expands them instead of recomputing the union
    uint2 *scr;             // nullptr when the workspace has no room for it
    int32_t *scnt;
    // set by the count pass where any row has that many words (kSeen*): which
    // launches the fill pass needs, read back with the counts
    uint32_t *seen;
    // numeric / adjoint spill path: first task of each spill row (position in
    // the spill bin), then the total; per-row scratch of na + 1 entries
    int32_t *wstart;
};

constexpr int kScratchWords = 64;

static_assert(kBinSpill == kNumClasses, "the spill bin follows the classes");

// Rows per binning block: every binning kernel assigns rows [b * kBinRowsPerWG,
// (b + 1) * kBinRowsPerWG) to workgroup b and leaves the block's row count per
// bin in blk_cnt, so that the bin scan and the scatter need no global atomics.
constexpr int kBinRowsPerWG = 1024;

// Pointers read out of descriptors are generic; loads through them compile
// to flat instructions, which make the compiler wait on LDS and vector memory
// together. Every kernel therefore casts them to the global address space.
#define MLS_G __attribute__((address_space(1)))
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <class T>
__device__ __forceinline__ const MLS_G T *gp(const T *p)
{
    return (const MLS_G T *)(p);
}

template <class T>
__device__ __forceinline__ MLS_G T *gpw(T *p)
{
    return (MLS_G T *)(p);
}

// Whether the CSR check that ran before on this stream refused the operands:
// every kernel queued behind it that follows their indices, or that works on
// what such a kernel would have written, returns at once then, so the host
// reads the verdict back once, with the result. err may be NULL (no check).
__device__ __forceinline__ bool bad_csr(const uint32_t *err)
{
    return err && (*gp(err) & kErrBadCsr) != 0u;
}

__device__ __forceinline__ int find_prob(const int32_t *base, int nprob, int g)
{
    // largest t with base[t] <= g
    int lo = 0, hi = nprob - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (gp(base)[mid] <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// find_prob for a g that is the same in every lane of the wave, all lanes
// active: 64 candidates per step, so one or two dependent loads (up to 4096
// products) in place of log2(nprob).
__device__ __forceinline__ int find_prob_wave(const int32_t *base, int nprob, int g)
{
    if (nprob > 4096) return find_prob(base, nprob, g);
    const int lane = (int)(threadIdx.x & 63);
    const MLS_G int32_t *bs = gp(base);
    int t = 0;
    if (nprob > 64) {
        const int c = lane * 64;
        const int v = bs[c < nprob ? c : 0];
        const unsigned long long m = __ballot(c < nprob && v <= g);   // lane 0 always: base[0] = 0
        t = (63 - __clzll(m)) * 64;
    }
    const int c = t + lane;
    const int v = bs[c < nprob ? c : 0];
    const unsigned long long m = __ballot(c < nprob && v <= g);
    return t + (63 - __clzll(m));
}

// Largest r in [0, n) with at[r] <= u (at ascending, at[0] <= u, n >= 1), for a
// u that is the same in every lane, all lanes active: 64 candidates per step,
// three dependent loads for n = 20000 in place of fifteen.
__device__ __forceinline__ int find_last_wave(const MLS_G int32_t *at, int n, int u)
{
    const int lane = (int)(threadIdx.x & 63);
    int lo = 0;
    while (n > 1) {
        const int step = (n + kWave - 1) / kWave;
        const int c = lane * step;
        const int v = at[lo + (c < n ? c : 0)];
        const int k = 63 - __clzll((long long)__ballot(c < n && v <= u));   // lane 0 always holds
        lo += k * step;
        n = min(step, n - k * step);
    }
    return lo;
}

// Product of row g when consecutive rows are spread over a wave (g = g_w +
// lane, g_w uniform): the product of the wave's first row serves every lane
// whose row lies before that product's end, the others search on their own.
// Call with every lane of the wave active.
__device__ __forceinline__ int find_prob_rows(const int32_t *base, int nprob, int g_w, int g)
{
    const int t = find_prob_wave(base, nprob, g_w);
    if (g < gp(base)[t + 1]) return t;
    return find_prob(base, nprob, g);
}

// Product lookup with a per-lane memory of the last product found: rows a
// lane takes in a row usually belong to the same product of a batch, and then
// two compares replace the binary search.
struct ProbCache {
    int t = 0, lo = 0, hi = 0;   // rows [lo, hi) belong to product t
};

__device__ __forceinline__ int find_prob_cached(const int32_t *base, int nprob, int g, ProbCache &c)
{
    if (g >= c.lo && g < c.hi) return c.t;
    c.t = find_prob(base, nprob, g);
    c.lo = gp(base)[c.t];
    c.hi = gp(base)[c.t + 1];
    return c.t;
}

// The descriptor of product t by value: from the kernel arguments for a
// single product, from global memory for a batch.
__device__ __forceinline__ Prob get_prob(const Batch &b, int t)
{
    if (b.nprob == 1) return b.p0;
    Prob P;
    const MLS_G u32x4 *src = (const MLS_G u32x4 *)(b.probs + t);
    u32x4 *dst = (u32x4 *)&P;
#pragma unroll
    for (int w = 0; w < (int)(sizeof(Prob) / 16); ++w) dst[w] = src[w];
    return P;
}

// get_prob for kernels specialised for batches: when every active lane of
// the wave asks for the same product (the rows of a wave are consecutive, so
// almost always), the descriptor is read once through the scalar cache
// (constant address space: the descriptors do not change while a kernel
// runs) and waits only on the scalar counter; otherwise each lane reads its
// own, and that wait stays inside its branch.
typedef const __attribute__((address_space(4))) u32x4 *MLS_K_u32x4p;

__device__ __forceinline__ Prob get_prob_batch(const Batch &b, int t)
{
    Prob P;
    u32x4 *dst = (u32x4 *)&P;
    const int t0 = __builtin_amdgcn_readfirstlane(t);
    if (__ballot(t != t0) == 0ull) {
        const MLS_K_u32x4p src = (MLS_K_u32x4p)(b.probs + t0);
#pragma unroll
        for (int w = 0; w < (int)(sizeof(Prob) / 16); ++w) dst[w] = src[w];
    } else {
        const MLS_G u32x4 *src = (const MLS_G u32x4 *)(b.probs + t);
#pragma unroll
        for (int w = 0; w < (int)(sizeof(Prob) / 16); ++w) dst[w] = src[w];
#pragma unroll
        for (int w = 0; w < (int)(sizeof(Prob) / 16); ++w) asm volatile("" ::"v"(dst[w]));
    }
    return P;
}

// get_prob_batch for kernels that serve both (the choice is made at run time).
__device__ __forceinline__ Prob get_prob_any(const Batch &b, int t)
{
    if (b.nprob == 1) return b.p0;
    return get_prob_batch(b, t);
}

// Multiplicative (Fibonacci) hashing of a key's low 24 bits (a column, or a set
// of 32): the product modulo 2^24 spreads consecutive keys by the golden
// ratio, its top bits are the slot. The 24-bit multiply runs at full rate, the
// 32-bit one at a quarter of it. Keys that differ above bit 24 alone share
// their home slot: at most 4 sets, and 2 to 8 columns of a packed table.
constexpr uint32_t kHashMul = 0x9E3779u;

__device__ __forceinline__ uint32_t hslot(uint32_t key, int logcap)
{
    return __builtin_amdgcn_ubfe(__umul24(key, kHashMul), 24 - logcap, logcap);
}

// The same of all 32 bits, for columns of wide tables: up to 128 may differ above
// bit 24 alone (100 columns 2^24 apart per row of B, 40000 rows of 3: numeric
// phase 2590 us with hslot, 136 us; adjoint 1959, 289; 2^20 apart 268 and 412, 136
// and 293; neighbours 136 and 295, 135 and 293).
__device__ __forceinline__ uint32_t hslot32(uint32_t key, int logcap) { return (key * 0x9E3779B1u) >> (32 - logcap); }

__device__ __forceinline__ int ilog2_ceil(int x)
{
    return x <= 1 ? 0 : 32 - __clz(x - 1);
}

// Cross-lane sums and scans over the G consecutive lanes of a group (G a
// power of two <= 64, groups aligned to G). Groups of at most 16 lanes lie in
// one 16-lane DPP row, where DPP moves read a neighbour's register directly
// (no LDS round trip): quad permutations and (half-)row mirrors for sums,
// row shifts for scans; every read stays inside the group (or is masked
// off). Wider groups use shuffles. All lanes of a group must be active.
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}

// DPP broadcasts of the last lane of a 16-lane row to the next row (row_bcast:15,
// written to rows 1 and 3) and of lane 31 to the upper half (row_bcast:31):
// they carry a row's prefix into the rows after it.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_bcast(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false);
}

template <int G, typename T>
__device__ __forceinline__ T group_sum(T v)
{
    if constexpr (sizeof(T) == 4 && T(-1) < T(0)) {
        if constexpr (G >= 2) v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]: lane ^ 1
        if constexpr (G >= 4) v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]: lane ^ 2
        if constexpr (G >= 8) v += dpp_move<0x141>(v);   // row_half_mirror: the other quad of 8
        if constexpr (G >= 16) v += dpp_move<0x140>(v);  // row_mirror: the other half of 16
        if constexpr (G >= 32) v += __shfl_xor(v, 16, G);
        if constexpr (G >= 64) v += __shfl_xor(v, 32, G);
        return v;
    } else {
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, G);
        return v;
    }
}

// the group's total, given a lane's value v and its inclusive prefix incl
template <int G>
__device__ __forceinline__ int group_total(int v, int incl)
{
    if constexpr (G <= 16) return group_sum<G>(v);
    else if constexpr (G == 64) return __builtin_amdgcn_readlane(incl, 63);
    else return __shfl(incl, G - 1, G);
}

// at, or last where !ok (ok: at <= last). Written as a select on an opaque copy:
// as a plain minimum, the compiler would redo the comparison where ok is used
// next, behind the loads, and keep both operands in registers until then
// (which spilled).
__device__ __forceinline__ int or_last(bool ok, int at, int last)
{
    asm("" : "+v"(at));
    return ok ? at : last;
}

// OR over the 8 lanes of a group
__device__ __forceinline__ uint32_t group_or8(uint32_t v)
{
    v |= (uint32_t)dpp_move<0xB1>((int)v);    // quad_perm [1,0,3,2]: lane ^ 1
    v |= (uint32_t)dpp_move<0x4E>((int)v);    // quad_perm [2,3,0,1]: lane ^ 2
    v |= (uint32_t)dpp_move<0x141>((int)v);   // row_half_mirror: the other quad of 8
    return v;
}

// OR over the group of G consecutive lanes
template <int G>
__device__ __forceinline__ uint32_t group_or(uint32_t v)
{
    static_assert(G == 8 || G == 16 || G == 32 || G == 64, "group size");
    v = group_or8(v);
    if constexpr (G >= 16) v |= (uint32_t)dpp_move<0x140>((int)v);   // row_mirror: the other 8 of 16
    if constexpr (G >= 32) {
        // the other row of 16 of a pair: each takes the odd row of one copy for the even row of the other
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = r[0] | r[1];
    }
    if constexpr (G == 64)
        v = (uint32_t)__builtin_amdgcn_readlane((int)v, 0) | (uint32_t)__builtin_amdgcn_readlane((int)v, 32);
    return v;
}

// inclusive prefix sum over the group; lane = position in the group
template <int G>
__device__ __forceinline__ int group_scan_incl(int v, int lane)
{
    int y;
    const int l16 = lane & 15;
    if constexpr (G >= 2) { y = dpp_move<0x111>(v); if (l16 >= 1) v += y; }   // row_shr:1
    if constexpr (G >= 4) { y = dpp_move<0x112>(v); if (l16 >= 2) v += y; }   // row_shr:2
    if constexpr (G >= 8) { y = dpp_move<0x114>(v); if (l16 >= 4) v += y; }   // row_shr:4
    if constexpr (G >= 16) { y = dpp_move<0x118>(v); if (l16 >= 8) v += y; }  // row_shr:8
    if constexpr (G >= 32) v += dpp_bcast<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    if constexpr (G >= 64) v += dpp_bcast<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

// The elements of a group's entries (entry l of lane l: a run of a row of B)
// laid end to end in one sequence. seq_compact: the first element of every
// entry that has any, less its place in the sequence (q), in lane r of the
// group for the r-th such entry.
template <int G>
__device__ __forceinline__ int seq_compact(bool nonempty, int q, int slot, int lane)
{
    const unsigned long long lt = (1ull << lane) - 1ull;
    constexpr unsigned long long kAll = G == kWave ? ~0ull : (1ull << (G & 63)) - 1ull;
    const unsigned long long ne = (__ballot(nonempty) >> (slot * G)) & kAll;
    const int rank = nonempty ? __popcll(ne & lt) : __popcll(ne) + __popcll(~ne & kAll & lt);
    return __builtin_amdgcn_ds_permute((slot * G + rank) * 4, q);
}

// Starts in a wave's tile handed over by compares (2 to 3 instructions per step
// each, no cross-lane chain) rather than by start bits: the dense-bitmap count and
// fill of the R-MAT 16 square with every row of more than 64 entries set aside,
// those rows 492 and 657 us, with bits always 719 and 876 us; the short ones 230
// and 523, with compares always 230 and 578 us.
constexpr int kSeqFew = 6;

// One tile of that sequence, SB elements per lane, loads in flight together:
// lane l of the group takes elements base + d * G + l. A bit per element tells
// where an entry starts (OR-ed over the group without LDS), so an element's
// entry is the count of the bits up to it; eb is the lane (of the wave) of the
// last entry that started before the tile. Elements past the sequence (ok
// false) load its last one.
template <int G, int SB, typename T>
__device__ __forceinline__ void seq_tile(const MLS_G T *src, int lane, int base, int total, int first, bool nonempty,
                                         int qd, int &eb, T (&v)[SB], bool (&ok)[SB])
{
    static_assert(SB * G % 32 == 0, "whole 32-bit words of start bits");
    constexpr int SW = G < 32 ? 32 / G : 1;   // steps per word of start bits
    constexpr int WS = G > 32 ? G / 32 : 1;   // words of start bits per step
    if constexpr (G == kWave) {
        unsigned long long st = __ballot(nonempty && (uint32_t)(first - base) < (uint32_t)(SB * kWave));
        if (__popcll(st) <= kSeqFew) {
            int qv[SB];
            const int q = __builtin_amdgcn_readlane(qd, eb > 0 ? eb : 0);
#pragma unroll
            for (int d = 0; d < SB; ++d) qv[d] = q;
            for (; st; st &= st - 1ull) {
                const int f = __builtin_amdgcn_readlane(first, __ffsll((long long)st) - 1);
                const int qn = __builtin_amdgcn_readlane(qd, ++eb);
#pragma unroll
                for (int d = 0; d < SB; ++d) qv[d] = base + d * kWave + lane >= f ? qn : qv[d];
            }
#pragma unroll
            for (int d = 0; d < SB; ++d) {
                const int pp = base + d * kWave + lane;
                ok[d] = pp < total;
                v[d] = src[qv[d] + min(pp, total - 1)];
            }
            return;
        }
    }
#pragma unroll
    for (int h = 0; h < SB / SW; ++h) {
        uint32_t m[WS];
#pragma unroll
        for (int x = 0; x < WS; ++x) {
            const int at = first - base - 32 * (WS * h + x);
            m[x] = group_or<G>(nonempty && (uint32_t)at < 32u ? 1u << at : 0u);
        }
#pragma unroll
        for (int d4 = 0; d4 < SW; ++d4) {
            const int d = SW * h + d4;
            int en = eb;
            if constexpr (WS == 1) {
                en += __popc(m[0] & ((2u << (G * d4 + lane)) - 1u));
            } else {
                en += __popc(m[0] & (lane < 31 ? (2u << lane) - 1u : ~0u));
                en += lane >= 32 ? __popc(m[1] & ((2u << (lane - 32)) - 1u)) : 0;
            }
            const int pp = base + d * G + lane;
            ok[d] = pp < total;
            const int q = __builtin_amdgcn_ds_bpermute(en * 4, qd) + min(pp, total - 1);
            v[d] = src[q];
        }
#pragma unroll
        for (int x = 0; x < WS; ++x) eb += __popc(m[x]);
    }
}

// Row at position pos of perm, or -1 (and an error bit) when the position or
// the row lies outside the batch -- which consistent bins never produce; the
// kernels then skip the row instead of dereferencing a bad index.
__device__ __forceinline__ int bin_row(const int32_t *perm, uint32_t *err, int na, int pos)
{
    if ((unsigned)pos >= (unsigned)na) { atomicOr(err, kErrTable); return -1; }
    const int g = gp(perm)[pos];
    if ((unsigned)g >= (unsigned)na) { atomicOr(err, kErrTable); return -1; }
    return g;
}

// Constant words read in place of an entry a lane does not need, so that a
// load needs no branch around it (a branch would make the wave wait for the
// load where the branches join): all ones (a column or row -1) and zeros.
static __device__ __attribute__((aligned(16))) int32_t k_ones4[4] = {-1, -1, -1, -1};
static __device__ __attribute__((aligned(16))) int32_t k_zeros4[4] = {0, 0, 0, 0};

// Pipelined form of bin_row: the perm load is only issued (a lane that wants
// no row reads -1), and bin_row_checked validates the value where it is first
// used, a row or more later. A position outside the batch never comes from
// consistent bins and is flagged at once.
__device__ __forceinline__ int bin_row_issue(const int32_t *perm, uint32_t *err, int na, int pos, bool want)
{
    const bool ok = want && (unsigned)pos < (unsigned)na;
    if (want && !ok) atomicOr(err, kErrTable);
    return *(ok ? gp(perm) + pos : (const MLS_G int32_t *)k_ones4);
}

__device__ __forceinline__ int bin_row_checked(uint32_t *err, int na, int g, bool want)
{
    if (!want) return -1;
    if ((unsigned)g >= (unsigned)na) { atomicOr(err, kErrTable); return -1; }
    return g;
}

// Bin start = exclusive prefix of the bin counts.
__device__ __forceinline__ int bin_start(const int32_t *bin_count, int bin)
{
    int s = 0;
    for (int c = 0; c < bin; ++c) s += bin_count[c];
    return s;
}

// Windows of a spill row that a wave of the numeric phase takes in turn: where
// one window ends in a row of B the next one starts (kept for kWinCarry
// entries of A), which saves it a search; rows of more entries take one window
// at a time, as theirs are long and have to spread over all waves. R-MAT 16
// square, windows of rows of up to 64 and 448 entries: 4 and 2 in turn 2.78 ms,
// 2 and 2 2.92 ms, 8 and 4 2.75 ms; R-MAT 15 with 12 entries per row: 1.61,
// 1.69 and 1.65 ms. Up to kWinSpread windows in all, one for each wave that stays
// resident, every window is a task of its own: larger ones would leave waves idle
// (16, 250 and 1000 rows of 6000 outputs, 60 entries of A each: 134, 148 and 186
// us with tasks of 4 windows, 92, 127 and 246 with tasks of one).
constexpr int kWinCarry = 448;
constexpr int kWinSpread = 4096;
__device__ __forceinline__ int win_block(int entries) { return entries <= kWave ? 4 : (entries <= kWinCarry ? 2 : 1); }

// One launch for every class of the numeric (or adjoint) phase: which part
// (class 0..4, or kNumClasses for the spill windows) this workgroup serves, -1
// for none, with its index and the number of workgroups of that part. The
// launch's workgroups are divided in proportion to the parts' rows over `per`,
// the rows (windows) a workgroup of the part takes at once; every part with
// rows gets at least one.
__device__ __forceinline__ int part_of_block(const Sched &sc, const int (&per)[kNumClasses + 1], int &vblk, int &vgrid)
{
    int want[kNumClasses + 1], all = 0, parts = 0, at = 0;
    for (int c = 0; c <= kNumClasses; ++c) {
        int n = gp(sc.bin_count)[c];
        if (c == kBinSpill && n > 0) n = gp(sc.wstart)[n];
        want[c] = (n + per[c] - 1) / per[c];
        all += want[c];
        parts += n > 0;
    }
    const int grid = (int)gridDim.x, blk = (int)blockIdx.x;
    const int share = grid > parts ? grid - parts : 0;   // beyond one each
    int sum = 0;
    for (int c = 0; c <= kNumClasses; ++c) {
        if (want[c] == 0) continue;
        const int lo = at + (int)((int64_t)share * sum / all);
        sum += want[c];
        ++at;
        const int hi = at + (int)((int64_t)share * sum / all);
        if (blk >= lo && blk < hi) {
            vblk = blk - lo;
            vgrid = hi - lo;
            return c;
        }
    }
    return -1;
}

// Per-wave task schedule. Tasks of a bin are split into one contiguous slab
// per XCD (workgroup w runs on XCD w % 8, and the CUs of an XCD share one L2).
// Inside a slab, waves take blocks of kTaskBlock tasks from a per-XCD counter;
// block b holds the tasks base + c, base + c + S, ..., c = b mod S, base set
// by b div S, with S the number of waves the grid places on the XCD. While
// every wave is busy, the rows in flight on an XCD therefore form a narrow
// window of about S consecutive tasks (neighbouring rows share most of their
// rows of B, and a narrow window keeps that shared working set in the L2).
// A wave's first block is the one of its own index on the XCD (the grid is
// sized to be resident at once), so a launch does not start with every wave
// queued on the same counter; only the blocks after the first S are taken
// from the counter, and a slab that the first blocks cover takes none.
constexpr int kTaskBlock = 16;

//
// With log_chunk >= 0 the tasks are instead cut into chunks of 2^log_chunk
// consecutive tasks, dealt to the XCDs round-robin: each XCD then holds a
// uniform sample of the bin, for bins whose work per task drifts with the
// row index (the degree-ordered rows of a power-law graph), where contiguous
// slabs leave some XCDs idle while others still work.
struct TaskIter {
    int lo, hi, S, cur, left, x, lc, wid;
    bool first;
};

// vblk, vgrid: the workgroup's index among those of its bin and their number
// (the launch's own, unless one launch serves several bins: FEW, when they may
// be fewer than the XCDs and cut as many slabs).
template <bool FEW>
__device__ __forceinline__ TaskIter task_iter(int ntasks, int waves_per_wg, int log_chunk, int vblk, int vgrid)
{
    const int nx = FEW && vgrid < kXcd ? vgrid : kXcd;
    const int x = vblk % nx;
    TaskIter it;
    it.x = x;
    it.lc = log_chunk;
    if (log_chunk < 0) {
        it.lo = (int)(((int64_t)ntasks * x) / nx);
        it.hi = (int)(((int64_t)ntasks * (x + 1)) / nx);
    } else {
        // local tasks of XCD x: the full chunks x, x + 8, ... and the
        // partial last chunk when it falls on x
        const int nch = ntasks >> log_chunk;
        const int rem = ntasks & ((1 << log_chunk) - 1);
        const int full = nch > x ? (nch - x + kXcd - 1) / kXcd : 0;
        it.lo = 0;
        it.hi = (full << log_chunk) + (nch % kXcd == x ? rem : 0);
    }
    const int wgs_x = (vgrid - x + nx - 1) / nx;   // workgroups on this XCD
    it.S = wgs_x * waves_per_wg;
    if (it.S < 1) it.S = 1;
    it.cur = 0;
    it.left = 0;
    // in [0, S); read from the first lane so that the compiler keeps it, and
    // every task index derived from it, in scalar registers
    it.wid = (vblk / nx) * waves_per_wg + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    it.first = true;
    return it;
}

__device__ __forceinline__ TaskIter task_iter(int ntasks, int waves_per_wg, int log_chunk = -1)
{
    return task_iter<false>(ntasks, waves_per_wg, log_chunk, (int)blockIdx.x, (int)gridDim.x);
}

__device__ __forceinline__ int task_global(const TaskIter &it, int t)
{
    if (it.lc < 0) return t;
    return ((((t >> it.lc) * kXcd) + it.x) << it.lc) + (t & ((1 << it.lc) - 1));
}

// Next task of this wave, or -1. Uniform across the wave; call with all lanes
// active. cursor: the bin's kXcd counters, zero before the launch.
__device__ __forceinline__ int next_task_wave(int32_t *cursor, int ntasks, TaskIter &it)
{
    (void)ntasks;
    if (it.lo >= it.hi) return -1;   // empty slab: no counter traffic
    for (;;) {
        if (it.left > 0) {
            const int t = it.cur;
            it.cur += it.S;
            --it.left;
            if (t < it.hi) return task_global(it, t);
            it.left = 0;
        }
        int blk = 0;
        if (it.first) {
            blk = it.wid;
            it.first = false;
        } else {
            if ((int64_t)it.lo + (int64_t)it.S * kTaskBlock >= it.hi) return -1;   // no block past the first S
            if ((threadIdx.x & 63) == 0) blk = atomicAdd(cursor + it.x, 1);
            blk = __builtin_amdgcn_readlane(blk, 0) + it.S;
        }
        const int64_t base = (int64_t)it.lo + (int64_t)(blk / it.S) * it.S * kTaskBlock + blk % it.S;
        if (base >= it.hi) return -1;
        it.cur = (int)base;
        it.left = kTaskBlock;
    }
}

}  // namespace mls
