// k_symbit.hip -- symbolic phase (Sec. 2.1) of products whose C has few
// columns: the union of the rows B_k, k in row i of A, as a dense bitmap over
// C's columns in LDS, one wave per row, straight from B's column indices or,
// where rows are long, from compressed B. No binning and no hash tables: the
// count pass is one launch over the rows and one over the rows set aside, the
// fill pass the same two, and columns come out of the bitmap in ascending order.
//
// What bounds it: latency for small products (each launch of the binned path
// costs its 2-20 us run or at least 4.7 us of stream time, and there are 14
// in a count pass), the issue of the pairs' instructions and LDS atomics for
// large ones. Whole products, binned path
// against this one: 64x64 Laplacian square 273 / 143 us, 3000 x 2000 x 2500
// random rows 372 / 144 us, R-MAT 16 square 12.9 / 9.6 ms.
#include <cstdio>

#include "common.h"
#include "launch.h"
#include "profile.h"

namespace mls {

constexpr int kBitTile = 4 * kWave;        // words a wave reads per step of a bitmap scan (16 bytes per lane)
constexpr int kBitRowWork = 4096;          // multiply-adds of a row one wave takes; longer rows are set aside
constexpr int kBitLongWG = 512;            // threads per set-aside row
constexpr int kBitDepth = 4;               // columns of B in flight per lane
constexpr int kBitStage = 32;              // words of a bitmap written out per step of a wave

__device__ __forceinline__ void bit_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// What is OR-ed into a bitmap of `words` words: B's columns, or (WORDS) the
// (set, mask) words of compressed B, where rows of B are long: a stencil's
// columns share words, and random ones cost little more as words.
template <bool WORDS> struct BitSrc {
    using T = int32_t;
    __device__ __forceinline__ static const MLS_G T *base(const Prob &P) { return gp(P.bci); }
    __device__ __forceinline__ static void set(uint32_t *bm, int words, T j, bool ok, bool &bad)
    {
        if (!ok) return;
        if ((uint32_t)j < 32u * (uint32_t)words) atomicOr(bm + (j >> 5), 1u << (j & 31));
        else bad = true;
    }
};
template <> struct BitSrc<true> {
    using T = u32x2;
    __device__ __forceinline__ static const MLS_G T *base(const Prob &P) { return (const MLS_G T *)P.bw; }
    __device__ __forceinline__ static void set(uint32_t *bm, int words, T w, bool ok, bool &bad)
    {
        if (!ok) return;
        if (w.x < (uint32_t)words) atomicOr(bm + w.x, w.y);
        else bad = true;
    }
};

// Rows of at most kBitRowWork multiply-adds (and entries of A), one per wave (dealt
// round-robin: their sizes vary), 64 entries of A at a time; the others go to
// the list in sc.perm, counted in the spill bin's count, up to 64 of a wave's with
// one atomic. R-MAT 16 square, count and fill: 297 and 525 us with a bisection
// per pair and no row in flight, 231 and 467 us with the pairs as a sequence and
// an atomic per row set aside, 104 and 323 us; 60000 random rows of 64 outputs
// (none set aside) 85 and 175, 61 and 128, 66 and 120 us.
template <bool FILL, bool WORDS>
__global__ __launch_bounds__(kWG) void k_bit_rows(Batch b, Sched sc, int words)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t s_bm[];   // words per wave, a multiple of kBitTile
    if (bad_csr(sc.err)) return;
    const int lane = threadIdx.x & 63, wave = (int)(threadIdx.x >> 6);
    uint32_t *bm = s_bm + wave * words;
    const Prob &P = b.p0;
    const MLS_G int32_t *__restrict__ arp = gp(P.arp);
    const MLS_G int32_t *__restrict__ aci = gp(P.aci);
    const MLS_G int32_t *__restrict__ brp = gp(P.brp);
    using Src = BitSrc<WORDS>;
    const MLS_G typename Src::T *__restrict__ src = Src::base(P);
    const MLS_G int32_t *__restrict__ bwc = gp(P.bwc);   // (WORDS)
    const MLS_G int32_t *__restrict__ crp = gp(P.crp);
    MLS_G int32_t *__restrict__ cci = gpw(P.cci);
    for (int x = 4 * lane; x < words; x += kBitTile) *(uint4 *)(bm + x) = make_uint4(0u, 0u, 0u, 0u);
    bit_sync();
    bool bad = false;
    const int stride = (int)gridDim.x * (kWG / kWave);
    int g = __builtin_amdgcn_readfirstlane((int)blockIdx.x * (kWG / kWave) + wave);
    // three rows in flight: this one's rows of B are located, the next one's
    // entries of A load during its pairs and their rows of B before its bitmap
    // is read (and so before its stores, which a later load's wait would cover),
    // the one after has its row pointers loading
    int s1 = 0, e1 = 0, cs1 = 0, ce1 = 0, s2 = 0, e2 = 0, cs2 = 0, ce2 = 0;
    int k1 = -1, q1 = 0, n1 = 0;
    auto row_ptrs = [&](int at, int &s, int &e, int &cs, int &ce) {
        const int r = (uint32_t)at < (uint32_t)b.na ? at : b.na - 1;   // (past the rows, or past an int)
        s = arp[r];
        e = arp[r + 1];
        if (FILL) { cs = crp[r]; ce = crp[r + 1]; }
    };
    auto entries = [&](int s, int e) {
        const int x = s - P.a_off + lane;
        k1 = *(x < e - P.a_off ? aci + x : (const MLS_G int32_t *)k_ones4);
    };
    // row k of B (none for k < 0): its start before b_off, and its elements
    auto row_b = [&](int k, int &q, int &n) {
        const bool in = k >= P.k_lo && k < P.k_hi;
        const MLS_G int32_t *zero = (const MLS_G int32_t *)k_zeros4;
        const MLS_G int32_t *pb = in ? brp + (k - P.k_lo) : zero;
        q = pb[0];
        if (WORDS) n = *(in ? bwc + (k - P.k_lo) : zero);
        else n = in ? pb[1] - q : 0;
    };
    auto rows_b = [&]() {
        row_b(k1, q1, n1);
    };
    if (g < b.na) {
        row_ptrs(g, s1, e1, cs1, ce1);
        row_ptrs(g + stride, s2, e2, cs2, ce2);
        entries(s1, e1);
        rows_b();
    }
    int aside = 0, n_aside = 0;   // lane l: the l-th row set aside and not yet listed
    auto list = [&]() {
        int at = 0;
        if (lane == 0) at = atomicAdd(sc.bin_count + kBinSpill, n_aside);
        at = __builtin_amdgcn_readlane(at, 0) + lane;
        if (lane < n_aside && at < b.na) gpw(sc.perm)[at] = aside;
        n_aside = 0;
    };
    for (; g < b.na; g = g < b.na - stride ? g + stride : b.na) {
        const int len = e1 - s1, ps = s1 - P.a_off;
        const int cs = FILL ? cs1 - P.c_off : 0, ce = FILL ? ce1 - P.c_off : 0;
        int q0 = q1 - P.b_off, n = n1;
        s1 = s2; e1 = e2; cs1 = cs2; ce1 = ce2;
        entries(s1, e1);
        row_ptrs((int)((uint32_t)g + 2u * (uint32_t)stride), s2, e2, cs2, ce2);
        // the (entry, position in B_k) pairs of 64 entries of A as one sequence, four
        // per lane in flight
        auto set_columns = [&](int total, int incl) {
            const int first = incl - n;
            const int qd = seq_compact<kWave>(n > 0, q0 - first, 0, lane);
            int eb = -1;
            for (int base = 0; base < total; base += kBitDepth * kWave) {
                typename Src::T v[kBitDepth];
                bool ok[kBitDepth];
                seq_tile<kWave, kBitDepth>(src, lane, base, total, first, n > 0, qd, eb, v, ok);
#pragma unroll
                for (int u = 0; u < kBitDepth; ++u) Src::set(bm, words, v[u], ok[u], bad);
            }
        };
        const int incl = group_scan_incl<kWave>(n, lane);
        int work = group_total<kWave>(n, incl);
        bool over = work > kBitRowWork || len > kBitRowWork;   // (entries of empty rows of B take time too)
        if (!over) set_columns(work, incl);
        for (int pc = kWave; !over && pc < len; pc += kWave) {   // a longer row's other entries
            const int k = *(lane < len - pc ? aci + ps + pc + lane : (const MLS_G int32_t *)k_ones4);
            row_b(k, q0, n);
            q0 -= P.b_off;
            const int more = group_scan_incl<kWave>(n, lane);
            const int total = group_total<kWave>(n, more);
            work += total;
            over = work > kBitRowWork;
            if (!over) set_columns(total, more);
        }
        if (over) {
            if (len > kWave) {   // (the chunks before have set columns)
                bit_sync();
                for (int x = 4 * lane; x < words; x += kBitTile) *(uint4 *)(bm + x) = make_uint4(0u, 0u, 0u, 0u);
            }
            if (lane == n_aside) aside = g;
            if (++n_aside == kWave) list();
            rows_b();
            bit_sync();
            continue;
        }
        rows_b();
        bit_sync();
        // the bitmap in column order, cleared for the next row as it is read
        int c = 0, at = cs;
        for (int x0 = 0; x0 < words; x0 += kBitTile) {
            const int x = x0 + 4 * lane;
            const uint4 w = *(const uint4 *)(bm + x);
            const bool any = (w.x | w.y | w.z | w.w) != 0u;
            if (!__ballot(any)) continue;
            if (any) *(uint4 *)(bm + x) = make_uint4(0u, 0u, 0u, 0u);
            const int pc = __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
            if constexpr (!FILL) {
                c += pc;
            } else {
                const int in = group_scan_incl<kWave>(pc, lane);
                int pos = at + in - pc;
                at += group_total<kWave>(pc, in);
                const uint64_t wv[2] = {((uint64_t)w.y << 32) | w.x, ((uint64_t)w.w << 32) | w.z};
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    uint64_t m = wv[d];
                    while (m) {
                        if (pos < ce) cci[pos] = x * 32 + d * 64 + (__ffsll((unsigned long long)m) - 1);
                        else bad = true;
                        ++pos;
                        m &= m - 1u;
                    }
                }
            }
        }
        if constexpr (FILL) {
            if (at != ce) bad = true;
        } else {
            c = group_sum<kWave>(c);
            if (lane == 0) gpw(sc.val)[g] = c;
        }
        bit_sync();
    }
    if (n_aside) list();
    if (bad) atomicOr(sc.err, kErrStructure);
}

// The rows set aside, a workgroup each: the columns of their rows of B as one
// sequence, an equal share of it per wave. R-MAT 16 square, count and fill: 750
// and 1011 us with 64-column pieces found by bisection and a thread writing a
// run of columns, 488 and 653 us so, 450 and 638 us with rows of up to
// kBitRowWork multiply-adds left to the waves.
template <bool FILL, bool WORDS>
__global__ __launch_bounds__(kBitLongWG) void k_bit_long(Batch b, Sched sc, int words)
{
    constexpr int NT = kBitLongWG, NWV = NT / kWave;
    extern __shared__ __attribute__((aligned(16))) uint32_t s_bm[];   // words
    __shared__ int s_first[NT + 1], s_qd[NT], s_red[NWV];
    __shared__ uint16_t s_col[NWV][kBitStage * 32];
    __shared__ int s_row;
    const int n_rows = min(gp(sc.bin_count)[kBinSpill], b.na);
    if ((int)blockIdx.x >= n_rows) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const Prob &P = b.p0;
    const MLS_G int32_t *__restrict__ aci = gp(P.aci);
    const MLS_G int32_t *__restrict__ brp = gp(P.brp);
    using Src = BitSrc<WORDS>;
    const MLS_G typename Src::T *__restrict__ src = Src::base(P);
    const MLS_G int32_t *__restrict__ bwc = gp(P.bwc);   // (WORDS)
    MLS_G int32_t *__restrict__ cci = gpw(P.cci);
    // exclusive scan over the workgroup; returns the thread's prefix, all = the total
    auto scan = [&](int v, int &all) -> int {
        const int incl = group_scan_incl<kWave>(v, lane);
        if (lane == kWave - 1) s_red[wave] = incl;
        __syncthreads();
        int before = 0;
        all = 0;
#pragma unroll
        for (int x = 0; x < NWV; ++x) {
            before += x < wave ? s_red[x] : 0;
            all += s_red[x];
        }
        __syncthreads();
        return before + incl - v;
    };
    bool bad = false;
    // the first row by the workgroup's index, the others from a counter
    for (int r = (int)blockIdx.x; r < n_rows;) {
        const int g = bin_row(sc.perm, sc.err, b.na, r);
        for (int x = tid; x < words; x += NT) s_bm[x] = 0u;
        const int s = g >= 0 ? gp(P.arp)[g] - P.a_off : 0, e = g >= 0 ? gp(P.arp)[g + 1] - P.a_off : 0;
        for (int pb = s; pb < e; pb += NT) {
            int q0 = 0, n = 0;
            if (pb + tid < e) {
                const int k = aci[pb + tid];
                if (k >= P.k_lo && k < P.k_hi) {
                    q0 = brp[k - P.k_lo] - P.b_off;
                    n = WORDS ? bwc[k - P.k_lo] : brp[k - P.k_lo + 1] - P.b_off - q0;
                }
            }
            int all;
            const int first = scan(n, all);
            s_first[tid] = first;
            s_qd[tid] = q0 - first;
            if (tid == 0) s_first[NT] = all;
            __syncthreads();
            // the chunk's columns as one sequence, an equal share of it per wave
            const int share = ((all + NWV - 1) / NWV + kWave - 1) / kWave * kWave;
            int base = wave * share;
            const int end = min(all, base + share);
            if (base < end) {
                int lo = 0, hi = NT - 1;   // largest entry that starts at or before base
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (s_first[mid] <= base) lo = mid; else hi = mid - 1;
                }
                for (int e0 = lo; base < end; e0 += kWave) {
                    const int f = s_first[min(e0 + lane, NT)], fn = s_first[min(e0 + lane + 1, NT)];
                    const int stop = min(end, s_first[min(e0 + kWave, NT)]);
                    const bool any = fn > f;
                    const int qd = seq_compact<kWave>(any, s_qd[min(e0 + lane, NT - 1)], 0, lane);
                    int eb = __builtin_amdgcn_readlane(f, 0) < base ? 0 : -1;
                    for (; base < stop; base += kBitDepth * kWave) {
                        typename Src::T v[kBitDepth];
                        bool ok[kBitDepth];
                        seq_tile<kWave, kBitDepth>(src, lane, base, stop, f, any, qd, eb, v, ok);
#pragma unroll
                        for (int u = 0; u < kBitDepth; ++u) Src::set(s_bm, words, v[u], ok[u], bad);
                    }
                    base = stop;
                }
            }
            __syncthreads();
        }
        if (s >= e) __syncthreads();   // (the bitmap is cleared)
        // wave w owns a run of consecutive words
        const int run = (words / kBitStage + NWV - 1) / NWV * kBitStage;
        const int x0 = wave * run, x1 = min(x0 + run, words);
        int c = 0;
        for (int x = x0 + lane; x < x1; x += kWave) c += __popc(s_bm[x]);
        int all;
        const int mine = scan(c, all);
        if constexpr (FILL) {
            const int cs = g >= 0 ? gp(P.crp)[g] - P.c_off : 0, ce = g >= 0 ? gp(P.crp)[g + 1] - P.c_off : 0;
            int pos = cs + __builtin_amdgcn_readlane(mine, 0);
            // kBitStage words per step, half a word per lane: the lanes place their
            // columns in LDS, then the wave writes them out in order
            for (int x = x0; x < x1; x += kBitStage) {
                uint32_t m = (s_bm[x + (lane >> 1)] >> ((lane & 1) * 16)) & 0xffffu;
                const int pc = __popc(m);
                const int in = group_scan_incl<kWave>(pc, lane);
                const int tot = group_total<kWave>(pc, in);
                if (tot == 0) continue;
                int at = in - pc;
                while (m) {
                    s_col[wave][at++] = (uint16_t)(lane * 16 + (__ffs(m) - 1));
                    m &= m - 1u;
                }
                bit_sync();
                for (int o = lane; o < tot; o += kWave) {
                    if (pos + o < ce) cci[pos + o] = x * 32 + (int)s_col[wave][o];
                    else bad = true;
                }
                pos += tot;
                bit_sync();
            }
            if (cs + all != ce) bad = true;
        } else if (tid == 0 && g >= 0) {
            gpw(sc.val)[g] = all;
        }
        if (n_rows <= (int)gridDim.x) break;
        if (tid == 0) s_row = (int)gridDim.x + atomicAdd(sc.task_cursor + kBinSpill * kXcd, 1);
        __syncthreads();
        r = s_row;
    }
    if (bad) atomicOr(sc.err, kErrStructure);
}

// Row pointers and nnz(C) of one product of few rows from the rows' counts,
// one workgroup, 8 rows per thread and step (four launches otherwise).
constexpr int kRowptrWG = 1024;
constexpr int kRowptrPer = 8;

__global__ __launch_bounds__(kRowptrWG) void k_rowptr_small(Batch b, const int32_t *val, int64_t *total, uint32_t *err)
{
    __shared__ int64_t s_red[kRowptrWG / kWave];
    if (bad_csr(err)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    MLS_G int32_t *crp = gpw(b.p0.crp);
    int64_t carry = 0;
    for (int r0 = 0; r0 < b.na; r0 += kRowptrWG * kRowptrPer) {
        const int r = r0 + (int)threadIdx.x * kRowptrPer;
        int v[kRowptrPer];
        int sum = 0;   // at most 8 rows of at most 65536 columns
#pragma unroll
        for (int d = 0; d < kRowptrPer; ++d) {
            v[d] = r + d < b.na ? gp(val)[r + d] : 0;
            sum += v[d];
        }
        const int incl = group_scan_incl<kWave>(sum, lane);
        if (lane == kWave - 1) s_red[wave] = incl;
        __syncthreads();
        int64_t off = carry + incl - sum, all = 0;
        for (int w = 0; w < kRowptrWG / kWave; ++w) {
            off += w < wave ? s_red[w] : 0;
            all += s_red[w];
        }
#pragma unroll
        for (int d = 0; d < kRowptrPer; ++d) {
            off += v[d];
            if (r + d < b.na) {
                if (off >= 0x7fffffffLL) atomicOr(err, kErrOverflow);
                crp[r + d + 1] = (int32_t)(off >= 0x7fffffffLL ? 0x7fffffffLL : off);
            }
        }
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        crp[0] = 0;
        *gpw(total) = carry;
    }
}

// ---------------------------------------------------------------------------

// Bitmaps or hash tables, by the product's rows and its multiply-adds per row (the
// mean row of A times the mean row of B). Symbolic phase in us, binned / columns
// / words; random: uniform columns, the others on grids; A P: the operator
// times a multigrid prolongator.
//   More than kBitRowWork multiply-adds: words. Stencils' columns share words
//   (elasticity, 27 neighbours of 3 unknowns, 59049 rows squared: 1166 / 1590 /
//   450; 6 unknowns, 63888 rows: 1994 / 5143 / 864), random ones do not and cost
//   little more as words (40000 rows, 100 times 100 in 60000 columns: 2912 / 1522
//   / 1669).
//   Up to kBitFewRows rows: columns. The launches decide (20000 rows in 16384
//   columns, 2 times 2: 113 / 89, 20 times 20: 338 / 108).
//   Fewer than 1024 columns: the adds of a step meet in few words, and compressed
//   rows are short (200000 rows, 20 times 20 in 256 columns: 308 / 825; 60000,
//   30 times 30 in 512: 280 / 364; 30000, 60 times 60: 672 / 318).
//   Few multiply-adds leave most of a wave idle, a group of lanes less so, and
//   the more the more rows there are: 64000 rows of the 5-point Laplacian's
//   square, 25: 111 / 158; 80000 random rows, 36 in 16384 columns: 211 / 151;
//   200000, 36: 273 / 276, 64: 424 / 310, and 64 in 65536 columns, where LDS
//   leaves 20 waves per CU: 448 / 605, 144: 1144 / 650; 2 million rows, 9: 545 /
//   1912. 27-point A P, 262144 rows, 32768 columns, 102: 320 / 411, 493039 rows,
//   64000 columns, 104: 439 / 1106.
//   Rows of A past a wave's 64 entries, many of them: 81-point A P, 331776 rows:
//   662 / 924 (59049 rows: 206 / 209; 40000 random rows of 100 times 4: 588 / 238).
constexpr int kBitFewRows = 32768, kBitManyRows = 131072;

SymBits symbit_choose(const Batch &b, double avg_a, double avg_b)
{
    if (b.nprob != 1 || b.p0.ncols > kBitMaxCols) return kBitsNone;
    const int ncols = b.p0.ncols;
    const double work = avg_a * avg_b;
    if (work > kBitRowWork) return kBitsWords;
    if (b.na <= kBitFewRows) return kBitsColumns;
    bool bits;
    if (ncols < 1024) bits = work >= 2048.0;
    else if (b.na <= kBitManyRows) bits = work >= 32.0;
    else bits = avg_a <= kWave && work >= (ncols <= 32768 ? 48.0 : 128.0);
    return bits ? kBitsColumns : kBitsNone;
}

template <bool FILL, bool WORDS>
static void launch_bits(const Batch &b, const Sched &sc, hipStream_t s)
{
    int words = (b.p0.ncols + 31) / 32;
    words = (words + kBitTile - 1) / kBitTile * kBitTile;
    if (words < kBitTile) words = kBitTile;
    const size_t wave_bytes = (size_t)words * 4;
    static int cus = device_cu_count();
    const int nw = kWG / kWave;
    // as many workgroups as stay resident (160 KB of LDS, 32 waves per CU)
    int per_cu = (int)(163840 / (nw * wave_bytes));
    per_cu = per_cu > 8 ? 8 : (per_cu < 1 ? 1 : per_cu);
    const int want = (b.na + nw - 1) / nw;
    const int grid = want < cus * per_cu ? want : cus * per_cu;
    int long_per_cu = (int)(163840 / (wave_bytes + (FILL ? 21504 : 4608)));
    long_per_cu = long_per_cu > 4 ? 4 : (long_per_cu < 1 ? 1 : long_per_cu);
    const int long_grid = b.na < cus * long_per_cu ? b.na : cus * long_per_cu;
    ProfScope ps(FILL ? "sym_bit_fill" : "sym_bit_count", s);
    hipLaunchKernelGGL((k_bit_rows<FILL, WORDS>), dim3(grid), dim3(kWG), nw * wave_bytes, s, b, sc, words);
    hipLaunchKernelGGL((k_bit_long<FILL, WORDS>), dim3(long_grid), dim3(kBitLongWG), wave_bytes, s, b, sc, words);
}

void launch_symbit(const Batch &b, const Sched &sc, int fill, bool words, hipStream_t s)
{
    if (b.na <= 0) return;
    if (words) {
        if (fill) launch_bits<true, true>(b, sc, s);
        else launch_bits<false, true>(b, sc, s);
    } else {
        if (fill) launch_bits<true, false>(b, sc, s);
        else launch_bits<false, false>(b, sc, s);
    }
}

void launch_rowptr_small(const Batch &b, const int32_t *val, int64_t *total, uint32_t *err, hipStream_t s)
{
    ProfScope ps("rowptr_small", s);
    hipLaunchKernelGGL(k_rowptr_small, dim3(1), dim3(kRowptrWG), 0, s, b, val, total, err);
}

}  // namespace mls
