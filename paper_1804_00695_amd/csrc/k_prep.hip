// k_prep.hip -- kernels around the two phases: CSR checks, column compression
// of B, per-row work estimate and binning, the row-pointer scan.
#include "common.h"
#include "launch.h"
#include "profile.h"

namespace mls {

// ---------------------------------------------------------------------------
// state reset (a fill kernel instead of hipMemsetAsync so that a captured
// graph replays it faithfully)

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

__global__ void k_fill_f64(double *p, double v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

__global__ void k_zero2_f64(double *p, int64_t n, double *q, int64_t m)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n + m; i += stride) *(i < n ? p + i : q + (i - n)) = 0.0;
}

// ---------------------------------------------------------------------------
// Entry streams: the rows of a wave (rw consecutive ones, rw a power of two up
// to 64) hold one contiguous run of entries, which the wave walks 64 at a time
// whatever the rows' lengths, with the loads of a tile of kTileSteps steps in
// flight. A bit per entry of the tile tells where a (non-empty) row starts.
// Positions in the stream are unsigned: a tile's end, and a lane's position behind
// the run's end, may lie past the largest int (the entry limit).
constexpr int kTileSteps = 8;
constexpr int kTileEntries = kTileSteps * kWave;

__device__ __forceinline__ void prep_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Row starts of the tile [tb, tb + kTileEntries) from the lanes' rows [s, e),
// as a bitmap in flags (kTileEntries bits).
__device__ __forceinline__ void tile_starts(uint32_t *flags, int lane, uint32_t tb, int s, int e)
{
    static_assert(kTileEntries / 32 <= kWave, "one word per lane");
    if (lane < kTileEntries / 32) flags[lane] = 0u;
    prep_sync();
    const uint32_t at = (uint32_t)s - tb;
    if (s < e && at < (uint32_t)kTileEntries) atomicOr(flags + (at >> 5), 1u << (at & 31));
    prep_sync();
}

// Lane l's value from lane l - 1; lane 0 gets `first` (DPP wave shift).
__device__ __forceinline__ int lane_before(int v, int first)
{
    return __builtin_amdgcn_update_dpp(first, v, 0x138, 0xF, 0xF, false);
}

// CSR checks over the A rows (which = 0) or B rows (which = 1) of a batch:
// row_ptr[0] == 0, non-decreasing, row_ptr[n] == nnz, columns in range and
// strictly increasing. Column indices outside [0, nnz) are never read: a wave
// whose row pointers fail reads no entries.
// which = 2: the A rows by the first a_blocks workgroups, the B rows by the
// others. Bound by the reads of the columns: 27-point stencil 128^3 54 us (223
// MB, 4.1 TB/s), R-MAT 18's L 21 us. (112 and 74 us with rows dealt to 1, 16,
// 32 or 64 lanes by length, rows of more than 32 entries one after the other.)
__global__ __launch_bounds__(kWG) void k_validate(Batch b, int which, const int64_t *nnz_tab, int64_t nnz_a,
                                                  int64_t nnz_b, int a_blocks, int rw_a, int rw_b, uint32_t *err)
{
    __shared__ uint32_t s_flags[kWG / kWave][kTileEntries / 32];
    const int lane = threadIdx.x & 63;
    uint32_t *flags = s_flags[threadIdx.x >> 6];
    int blk = (int)blockIdx.x;
    if (which == 2) {
        which = blk < a_blocks ? 0 : 1;
        if (which) blk -= a_blocks;
    }
    const int total = which == 0 ? b.na : b.nb;
    const int rw = which == 0 ? rw_a : rw_b;
    const int g0 = (blk * (kWG / kWave) + (int)(threadIdx.x >> 6)) * rw, g = g0 + lane;
    const int32_t *base = which == 0 ? b.abase : b.bbase;
    const bool row = lane < rw && g < total;
    const int gw = g0 < total ? g0 : total - 1;
    const int t = b.nprob == 1 ? 0 : find_prob_rows(base, b.nprob, gw, row ? g : gw);
    bool bad = false;
    const int32_t *ci = nullptr;
    int s = 0, e = 0, ncols = 0;
    if (row) {
        const Prob P = get_prob_any(b, t);
        const int i = g - (b.nprob == 1 ? 0 : gp(base)[t]);
        const MLS_G int32_t *rp = gp(which == 0 ? P.arp : P.brp);
        const int off = which == 0 ? P.a_off : P.b_off;
        ci = which == 0 ? P.aci : P.bci;
        ncols = which == 0 ? P.k_hi : P.ncols;
        const int nrows = which == 0 ? P.nrows : P.krows;
        const int64_t nnz = nnz_tab ? gp(nnz_tab)[2 * t + which] : (which == 0 ? nnz_a : nnz_b);
        s = rp[i];
        e = rp[i + 1];
        if (i == 0 && s != off) bad = true;
        if (i == nrows - 1 && (int64_t)e - off != nnz) bad = true;
        if (e < s || s < off || (int64_t)e - off > nnz) bad = true;
        s -= off;
        e -= off;
    }
    if (__ballot(bad)) {
        if (lane == 0) atomicOr(err, kErrBadCsr);
        return;
    }
    // the wave's rows of one product at a time (almost always all of them):
    // their pointers are consistent, so their entries are contiguous
    unsigned long long todo = __ballot(row);
    while (todo) {
        const int l0 = __ffsll((long long)todo) - 1;
        const int t0 = __builtin_amdgcn_readlane(t, l0);
        const unsigned long long seg = __ballot(row && t == t0);
        const int l1 = 63 - __clzll((long long)seg);
        todo &= ~seg;
        const bool mine = row && t == t0;
        const int nc = __builtin_amdgcn_readlane(ncols, l0);
        const uint32_t q0 = (uint32_t)__builtin_amdgcn_readlane(s, l0), q1 = (uint32_t)__builtin_amdgcn_readlane(e, l1);
        const uint64_t pa = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)((uint64_t)ci >> 32), l0) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint64_t)ci, l0);
        const MLS_G int32_t *c = (const MLS_G int32_t *)pa;
        int carry = -1;
        for (uint32_t tb = q0; tb < q1; tb += kTileEntries) {
            const MLS_G int32_t *ct = c + tb;
            const uint32_t left = q1 - tb;
            int cv[kTileSteps];
#pragma unroll
            for (int u = 0; u < kTileSteps; ++u) {
                const uint32_t x = (uint32_t)(u * kWave + lane);
                cv[u] = *(x < left ? ct + x : (const MLS_G int32_t *)k_zeros4);
            }
            tile_starts(flags, lane, tb, mine ? s : 0, mine ? e : 0);
#pragma unroll
            for (int u = 0; u < kTileSteps; ++u) {
                const bool start = ((flags[2 * u + (lane >> 5)] >> (lane & 31)) & 1u) != 0u;
                const int prev = lane_before(cv[u], carry);
                bad |= (uint32_t)(u * kWave + lane) < left && (cv[u] < 0 || cv[u] >= nc || (!start && cv[u] <= prev));
                carry = __builtin_amdgcn_readlane(cv[u], 63);
            }
            prep_sync();
        }
    }
    if (__ballot(bad) && lane == 0) atomicOr(err, kErrBadCsr);
}

// Column compression of every B row (set = col >> 5, mask bit = col & 31),
// padded layout: the words of row k start at B's entry offset of row k. An
// entry starts a word (is a head) where a row starts or its set differs from
// the entry before; the masks of a step's words are OR-ed in LDS, and the last
// word of a step stays open (it may continue in the next one). With H the
// heads of the wave's stream before a head, its word goes to q - H of the
// latest row start, plus H. Bound by reads and writes: 27-point stencil 128^3
// 136 us (about 0.39 GB); R-MAT 18's L, whose long rows are neighbours, 77 us,
// by its waves' longest runs. (179 and 199 us row by row as above; 155 and 186
// us as a stream of 64 rows per wave and one LDS exchange per step.)
__global__ __launch_bounds__(kWG) void k_compress(Batch b, int rw, const uint32_t *err)
{
    if (bad_csr(err)) return;
    constexpr int NWV = kWG / kWave;
    __shared__ uint32_t s_flags[NWV][kTileEntries / 32];
    __shared__ uint32_t s_msk[NWV][kTileEntries + kWave];   // masks of a tile's words, 0 the one left open
    __shared__ int s_heads[NWV][kWave + 1];   // heads before the k-th non-empty row
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t *flags = s_flags[wave], *wmsk = s_msk[wave];
    int *heads = s_heads[wave];
    constexpr uint32_t kNone = 0xffffffffu;
    const int g0 = ((int)blockIdx.x * NWV + wave) * rw, g = g0 + lane;
    const bool row = lane < rw && g < b.nb;
    const int gw = g0 < b.nb ? g0 : b.nb - 1;
    const int t = b.nprob == 1 ? 0 : find_prob_rows(b.bbase, b.nprob, gw, row ? g : gw);
    const int32_t *ci = nullptr;
    uint2 *bw = nullptr;
    int32_t *cnt = nullptr;
    int s = 0, e = 0;
    if (row) {
        const Prob P = get_prob_any(b, t);
        const int k = g - (b.nprob == 1 ? 0 : gp(b.bbase)[t]);
        s = gp(P.brp)[k] - P.b_off;
        e = gp(P.brp)[k + 1] - P.b_off;
        ci = P.bci;
        bw = P.bw;
        cnt = P.bwc + k;
    }
    for (int x = lane; x < kTileEntries + kWave; x += kWave) wmsk[x] = 0u;
    const unsigned long long upto = lane == 63 ? ~0ull : (2ull << lane) - 1ull;   // lanes 0 .. lane
    unsigned long long todo = __ballot(row);
    while (todo) {
        const int l0 = __ffsll((long long)todo) - 1;
        const int t0 = __builtin_amdgcn_readlane(t, l0);
        const bool mine = row && t == t0;
        const unsigned long long seg = __ballot(mine);
        const int l1 = 63 - __clzll((long long)seg);
        todo &= ~seg;
        auto rl64 = [&](const void *p) {
            const uint64_t v = (uint64_t)p;
            return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l0) << 32) |
                   (uint32_t)__builtin_amdgcn_readlane((int)v, l0);
        };
        const MLS_G int32_t *c = (const MLS_G int32_t *)rl64(ci);
        MLS_G u32x2 *out = (MLS_G u32x2 *)rl64(bw);
        const uint32_t q0 = (uint32_t)__builtin_amdgcn_readlane(s, l0), q1 = (uint32_t)__builtin_amdgcn_readlane(e, l1);
        const unsigned long long full = __ballot(mine && s < e);
        // the open word (set, mask, its place), the latest row start's q - H,
        // and the heads and row starts of the stream so far
        uint32_t open_set = kNone, open_msk = 0u;
        int open_pos = 0, shift = 0, nheads = 0, nrows = 0;
        for (uint32_t tb = q0; tb < q1; tb += kTileEntries) {
            const MLS_G int32_t *ct = c + tb;
            const uint32_t left = q1 - tb;
            uint32_t cv[kTileSteps];
#pragma unroll
            for (int u = 0; u < kTileSteps; ++u) {
                const uint32_t x = (uint32_t)(u * kWave + lane);
                cv[u] = (uint32_t)*(x < left ? ct + x : (const MLS_G int32_t *)k_zeros4);
            }
            tile_starts(flags, lane, tb, mine ? s : 0, mine ? e : 0);
            // the tile's heads and their words' masks: every step's ORs before
            // any of their results is read
            int lw[kTileSteps], at[kTileSteps];   // at < 0: no head
            int th = 0;                           // heads of the tile so far
            uint32_t carry = open_set, last_set = open_set;
            int last_pos = open_pos;
#pragma unroll
            for (int u = 0; u < kTileSteps; ++u) {
                lw[u] = 0;
                at[u] = -1;
                if ((uint32_t)(u * kWave) >= left) continue;
                const int q = (int)(tb + (uint32_t)(u * kWave + lane));
                const bool valid = (uint32_t)(u * kWave + lane) < left;
                const bool start = valid && ((flags[2 * u + (lane >> 5)] >> (lane & 31)) & 1u) != 0u;
                const uint32_t set = valid ? cv[u] >> 5 : kNone;
                const uint32_t prev = (uint32_t)lane_before((int)set, (int)carry);
                const bool head = valid && (start || set != prev);
                const unsigned long long hm = __ballot(head), sm = __ballot(start);
                lw[u] = th + __popcll(hm & upto);     // the entry's word in the tile
                const int h = nheads + lw[u] - 1;     // heads before the entry's own
                if (start) heads[nrows + __popcll(sm & upto) - 1] = h;
                // q - H of the latest row start at or before this lane
                const unsigned long long sb = sm & upto;
                const int sh = __shfl(q - h, sb ? 63 - __clzll((long long)sb) : 0, kWave);
                const int place = (sb ? sh : shift) + h;
                if (head) at[u] = place;
                if (valid) atomicOr(&wmsk[lw[u]], 1u << (cv[u] & 31u));
                if (hm) {
                    const int lh = 63 - __clzll((long long)hm);
                    last_set = (uint32_t)__builtin_amdgcn_readlane((int)set, lh);
                    last_pos = __builtin_amdgcn_readlane(place, lh);
                }
                if (sm) shift = __builtin_amdgcn_readlane(q - h, 63 - __clzll((long long)sm));
                carry = (uint32_t)__builtin_amdgcn_readlane((int)set, 63);
                th += __popcll(hm);
                nrows += __popcll(sm);
            }
            prep_sync();
            // word 0 continues the open word, words 1 .. th - 1 are complete,
            // word th stays open
            if (th > 0 && open_set != kNone && lane == 0) {
                u32x2 w; w.x = open_set; w.y = open_msk | wmsk[0];
                out[open_pos] = w;
            }
            if (th == 0) open_msk |= (uint32_t)__builtin_amdgcn_readfirstlane((int)wmsk[0]);
            else open_msk = (uint32_t)__builtin_amdgcn_readfirstlane((int)wmsk[th]);
            open_set = last_set;
            open_pos = last_pos;
            nheads += th;
#pragma unroll
            for (int u = 0; u < kTileSteps; ++u)
                if (at[u] >= 0 && lw[u] < th) {
                    u32x2 w; w.x = cv[u] >> 5; w.y = wmsk[lw[u]];
                    out[at[u]] = w;
                }
            prep_sync();
            for (int x = lane; x <= th; x += kWave) wmsk[x] = 0u;
            prep_sync();
        }
        if (open_set != kNone && lane == 0) {
            u32x2 w; w.x = open_set; w.y = open_msk;
            out[open_pos] = w;
        }
        if (lane == 0) heads[nrows] = nheads;
        prep_sync();
        if (mine) {
            const int o = __popcll(full & upto) - 1;   // this row's rank among the non-empty ones
            gpw(cnt)[0] = s < e ? heads[o + 1] - heads[o] : 0;
        }
        prep_sync();
    }
}

// ---------------------------------------------------------------------------
// Row sizes and bins.
//   kModeCount  : size = sum over in-range k of the word count of B_k (an
//                 upper bound of the distinct column sets of row i of C)
//   kModeFill   : size = min(that bound, nnz(C_i))
//   kModeNumeric: size = nnz(C_i)
//   kModeWork   : size = sum over in-range k of nnz(B_k) (multiply-adds)
//   kModeSized  : kModeCount with the sizes in val (k_work)
// Threshold classes: kCountCap for count, kFillCap/2 for fill and numeric.

// force < 0: natural class; force = kBinSpill: every non-empty row spills;
// 0 <= force < kNumClasses: rows of a smaller natural class move up to class
// `force` (a larger table always holds a row; test knob).
__device__ __forceinline__ int class_of(int mode, int64_t size, int force)
{
    if (size == 0) return kBinEmpty;
    if (force == kBinSpill) return kBinSpill;
    int cls = kBinSpill;
    if (mode == kModeCount) {
        for (int c = 0; c < kNumClasses; ++c)
            if (size <= kCountCap[c]) { cls = c; break; }
    } else {
        for (int c = 0; c < kNumClasses; ++c)
            if (size <= kFillCap[c] / 2) { cls = c; break; }
    }
    if (force >= 0 && cls < force) cls = force;
    return cls;
}

constexpr int kBinRG = 4;                    // lanes per row where the size is gathered (measured: 2-16)
constexpr int kBinSlots = kWG / kBinRG;      // rows in flight per workgroup
constexpr int kBinLongRow = 512;             // rows of A longer than this are gathered by the workgroup
constexpr int kBinMaxLong = 64;              // such rows deferred per block (more are gathered in place)

// Per-block bin counts (LDS) written to blk_cnt[c * nblk + block].
__device__ __forceinline__ void bin_write_counts(const Sched &sc, const int *cnt)
{
    if (threadIdx.x < kNumBins) gpw(sc.blk_cnt)[threadIdx.x * sc.nblk + (int)blockIdx.x] = cnt[threadIdx.x];
}

// Bin of a row of known size (count, fill and work modes), by one thread.
__device__ __forceinline__ void bin_place(int mode, const Sched &sc, int force, const Prob &P, int g, int i,
                                          bool from_scratch, int64_t size, int *cnt, unsigned long long *tsum)
{
    int c;
    if (from_scratch) {
        c = kBinEmpty;
    } else {
        if (mode == kModeFill) {
            const int64_t nc = gp(P.crp)[i + 1] - gp(P.crp)[i];
            size = size < nc ? size : nc;
        }
        if (mode == kModeWork) {
            c = kBinEmpty;
            if (size >= 0x7fffffffLL) atomicOr(sc.err, kErrOverflow);
            atomicAdd(tsum, (unsigned long long)size);
        } else {
            c = class_of(mode, size, force);
            // a large row whose dense bitmap over C's columns is at most half
            // its class table takes the spill path's LDS bitmap instead
            if (c >= 3 && c < kNumClasses &&
                (int64_t)P.ncols <= 32 * (int64_t)(mode == kModeCount ? kCountCap[c] : kFillCap[c]))
                c = kBinSpill;
            // rows without work get no symbolic kernel: their scratch is empty
            if (mode == kModeCount && sc.scr && c == kBinEmpty) gpw(sc.scnt)[g] = 0;
        }
    }
    if (size >= 0x7fffffffLL) size = 0x7fffffff;
    gpw(sc.val)[g] = (int32_t)size;
    gpw(sc.cls)[g] = (uint8_t)c;
    atomicAdd(&cnt[c], 1);
}

// Sizes of the rows of A for the count pass (kModeCount) as an entry stream:
// the word counts of the entries' rows of B, their running sum over a tile in
// LDS, of which every row takes the difference at its ends. Words of a row past
// kWorkMax, which no class holds, count as kWorkMax, so that a tile's sum fits.
// Bound by the gathers. 27-point stencil 128^3, sizes and bins: 158 us with 4
// lanes per row, 113 us; 20 Galerkin setups 104 and 52 us.
constexpr int kWorkMax = 1 << 22;
static_assert(kWorkMax > kCountCap[kNumClasses - 1] && (int64_t)kTileEntries * kWorkMax <= (1ll << 31), "tile sums");

__global__ __launch_bounds__(kWG) void k_work(Batch b, int rw, Sched sc)
{
    if (bad_csr(sc.err)) return;
    constexpr int NWV = kWG / kWave;
    __shared__ uint32_t s_sum[NWV][kTileEntries];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t *sum = s_sum[wave];
    const int g0 = ((int)blockIdx.x * NWV + wave) * rw, g = g0 + lane;
    const bool row = lane < rw && g < b.na;
    const int gw = g0 < b.na ? g0 : b.na - 1;
    const int t = b.nprob == 1 ? 0 : find_prob_rows(b.abase, b.nprob, gw, row ? g : gw);
    int s = 0, e = 0;
    if (row) {
        const Prob P = get_prob_any(b, t);
        const int i = g - (b.nprob == 1 ? 0 : gp(b.abase)[t]);
        s = gp(P.arp)[i] - P.a_off;
        e = gp(P.arp)[i + 1] - P.a_off;
    }
    int64_t size = 0;
    unsigned long long todo = __ballot(row);
    while (todo) {
        const int l0 = __ffsll((long long)todo) - 1;
        const int t0 = __builtin_amdgcn_readlane(t, l0);
        const bool mine = row && t == t0;
        const unsigned long long seg = __ballot(mine);
        const int l1 = 63 - __clzll((long long)seg);
        todo &= ~seg;
        const Prob P = get_prob_any(b, t0);
        const MLS_G int32_t *aci = gp(P.aci), *bwc = gp(P.bwc);
        const int k_lo = P.k_lo, k_hi = P.k_hi;
        const uint32_t q0 = (uint32_t)__builtin_amdgcn_readlane(s, l0), q1 = (uint32_t)__builtin_amdgcn_readlane(e, l1);
        for (uint32_t tb = q0; tb < q1; tb += kTileEntries) {
            int cv[kTileSteps];
#pragma unroll
            for (int u = 0; u < kTileSteps; ++u) {
                const uint32_t q = tb + (uint32_t)(u * kWave + lane);
                cv[u] = *(q < q1 ? aci + q : (const MLS_G int32_t *)k_ones4);
            }
#pragma unroll
            for (int u = 0; u < kTileSteps; ++u)
                cv[u] = *(cv[u] >= k_lo && cv[u] < k_hi ? bwc + (cv[u] - k_lo) : (const MLS_G int32_t *)k_zeros4);
            uint32_t before = 0;
#pragma unroll
            for (int u = 0; u < kTileSteps; ++u) {
                const int incl = group_scan_incl<kWave>(min(cv[u], kWorkMax), lane);
                sum[u * kWave + lane] = before + (uint32_t)incl;
                before += (uint32_t)__builtin_amdgcn_readlane(incl, 63);
            }
            prep_sync();
            const int lo = max(s - (int)tb, 0), hi = min(e - (int)tb, kTileEntries);   // (tb < q1 is an int)
            if (mine && lo < hi) size += (int64_t)(sum[hi - 1] - (lo > 0 ? sum[lo - 1] : 0u));
            prep_sync();
        }
    }
    if (row) gpw(sc.val)[g] = size >= 0x7fffffffLL ? 0x7fffffff : (int32_t)size;
}

__global__ __launch_bounds__(kWG) void k_bin(Batch b, int mode, Sched sc, int force,
                                             unsigned long long *total)
{
    __shared__ int cnt[kNumBins];
    __shared__ unsigned long long tsum;
    __shared__ int s_long[kBinMaxLong];
    __shared__ int s_nlong;
    __shared__ uint16_t s_todo[kBinRowsPerWG];   // fill pass: rows without scratch words
    __shared__ int s_ntodo;
    __shared__ int64_t s_red[kWG / kWave];
    if (bad_csr(sc.err)) return;
    if (threadIdx.x < kNumBins) cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) { tsum = 0; s_nlong = 0; s_ntodo = 0; }
    __syncthreads();
    const int g0 = blockIdx.x * kBinRowsPerWG;
    ProbCache pc;
    if (b.nprob > 1) {
        // the product of the block's first row, searched once per wave: the
        // block's rows almost always belong to it
        pc.t = find_prob_wave(b.abase, b.nprob, g0);
        pc.lo = gp(b.abase)[pc.t];
        pc.hi = gp(b.abase)[pc.t + 1];
    }
    if (mode == kModeSized) {   // size left in val by k_work: one thread per row
        for (int r = threadIdx.x; r < kBinRowsPerWG; r += kWG) {
            const int g = g0 + r;
            if (g >= b.na) break;
            const int t = b.nprob == 1 ? 0 : find_prob_cached(b.abase, b.nprob, g, pc);
            const Prob P = get_prob_any(b, t);
            bin_place(kModeCount, sc, force, P, g, g - (b.nprob == 1 ? 0 : pc.lo), false, gp(sc.val)[g], cnt, &tsum);
        }
        __syncthreads();
        bin_write_counts(sc, cnt);
        return;
    }
    if (mode == kModeNumeric) {   // size = nnz(C_i): one thread per row
        for (int r = threadIdx.x; r < kBinRowsPerWG; r += kWG) {
            const int g = g0 + r;
            if (g >= b.na) break;
            const int t = b.nprob == 1 ? 0 : find_prob_cached(b.abase, b.nprob, g, pc);
            const Prob P = get_prob_any(b, t);
            const int i = g - (b.nprob == 1 ? 0 : pc.lo);
            const int nc = gp(P.crp)[i + 1] - gp(P.crp)[i];
            const int c = class_of(mode, nc, force);
            gpw(sc.val)[g] = nc;
            gpw(sc.cls)[g] = (uint8_t)c;
            atomicAdd(&cnt[c], 1);
        }
        __syncthreads();
        bin_write_counts(sc, cnt);
        return;
    }
    // fill pass: rows whose words the count pass kept are expanded, not binned,
    // a thread each (with 4 lanes each 28 us of 2.1M rows, 13 us)
    const bool scratch = mode == kModeFill && sc.scr;
    int nrows = min(kBinRowsPerWG, b.na - g0);
    if (scratch) {
        const int all = nrows;
        for (int r = threadIdx.x; r < all; r += kWG) {
            const int g = g0 + r;
            if (gp(sc.scnt)[g] < 0) { s_todo[atomicAdd(&s_ntodo, 1)] = (uint16_t)r; continue; }
            const int t = b.nprob == 1 ? 0 : find_prob_cached(b.abase, b.nprob, g, pc);
            bin_place(mode, sc, force, get_prob_any(b, t), g, g - (b.nprob == 1 ? 0 : pc.lo), true, 0, cnt, &tsum);
        }
        __syncthreads();
        nrows = s_ntodo;
    }
    const int slot = threadIdx.x / kBinRG, lane = threadIdx.x % kBinRG;
    for (int x = slot; x < nrows; x += kBinSlots) {   // uniform per row group
        const int r = scratch ? (int)s_todo[x] : x;
        const int g = g0 + r;
        const int t = b.nprob == 1 ? 0 : find_prob_cached(b.abase, b.nprob, g, pc);
        const Prob P = get_prob_any(b, t);
        const int i = g - (b.nprob == 1 ? 0 : pc.lo);
        int64_t size = 0;
        const int s = gp(P.arp)[i] - P.a_off, e = gp(P.arp)[i + 1] - P.a_off;
        if (e - s > kBinLongRow) {
            // long row: gathered below by the whole workgroup, unless the list is full
            int at = 0;
            if (lane == 0) {
                at = atomicAdd(&s_nlong, 1);
                if (at < kBinMaxLong) s_long[at] = r;
            }
            at = __shfl(at, 0, kBinRG);
            if (at < kBinMaxLong) continue;
        }
        const MLS_G int32_t *__restrict__ aci = gp(P.aci);
        const MLS_G int32_t *__restrict__ brp = gp(P.brp);
        const MLS_G int32_t *__restrict__ bwc = gp(P.bwc);
        const int k_lo = P.k_lo, k_hi = P.k_hi;
        // four entries per lane in flight: their columns, then the gathers
        for (int p0 = s + lane; p0 < e; p0 += 4 * kBinRG) {
            int kv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = p0 + u * kBinRG;
                kv[u] = p < e ? aci[p] : -1;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (kv[u] < k_lo || kv[u] >= k_hi) continue;
                const int kl = kv[u] - k_lo;
                size += mode == kModeWork ? (int64_t)(brp[kl + 1] - brp[kl]) : (int64_t)bwc[kl];
            }
        }
        size = group_sum<kBinRG>(size);
        if (lane == 0) bin_place(mode, sc, force, P, g, i, false, size, cnt, &tsum);
    }
    __syncthreads();
    // the deferred long rows, one at a time across the workgroup
    const int nlong = s_nlong < kBinMaxLong ? s_nlong : kBinMaxLong;
    for (int x = 0; x < nlong; ++x) {
        const int g = g0 + s_long[x];
        const int t = b.nprob == 1 ? 0 : find_prob_cached(b.abase, b.nprob, g, pc);
        const Prob P = get_prob_any(b, t);
        const int i = g - (b.nprob == 1 ? 0 : pc.lo);
        const MLS_G int32_t *__restrict__ aci = gp(P.aci);
        const MLS_G int32_t *__restrict__ brp = gp(P.brp);
        const MLS_G int32_t *__restrict__ bwc = gp(P.bwc);
        const int s = gp(P.arp)[i] - P.a_off, e = gp(P.arp)[i + 1] - P.a_off;
        int64_t size = 0;
        for (int p = s + (int)threadIdx.x; p < e; p += kWG) {
            const int k = aci[p];
            if (k < P.k_lo || k >= P.k_hi) continue;
            const int kl = k - P.k_lo;
            size += mode == kModeWork ? (int64_t)(brp[kl + 1] - brp[kl]) : (int64_t)bwc[kl];
        }
        size = group_sum<kWave>(size);
        if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = size;
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t tot = 0;
            for (int w = 0; w < kWG / kWave; ++w) tot += s_red[w];
            bin_place(mode, sc, force, P, g, i, false, tot, cnt, &tsum);
        }
        __syncthreads();
    }
    bin_write_counts(sc, cnt);
    if (threadIdx.x == 0 && total && tsum) atomicAdd(total, tsum);
}

// One workgroup: bin totals into bin_count, and every block's count per bin
// replaced by the position in perm where that block's rows of the bin start
// (bins in order, blocks in order inside a bin). Only the nb blocks of this
// launch count: a launch over fewer rows than the workspace was laid out for
// (a chunk part) leaves the counts of later blocks from earlier launches.
// Bound by latency (one workgroup, no reuse): two waves per bin, each over
// half of the blocks, first sum their counts (all loads independent), then
// rescan them from the positions the sums give; one barrier, against three
// per bin with all threads on one bin at a time (2048 blocks: 20.9 us).
constexpr int kScanWG = 1024;
constexpr int kScanHalves = 2;   // waves per bin
constexpr int kScanPer = 8;      // consecutive blocks per lane and step

__global__ __launch_bounds__(kScanWG) void k_bin_scan(Sched sc, int nb)
{
    static_assert(kNumBins * kScanHalves <= kScanWG / kWave, "a wave per bin and half");
    __shared__ int s_tot[kNumBins * kScanHalves];
    if (bad_csr(sc.err)) return;
    MLS_G int32_t *blk = gpw(sc.blk_cnt);
    const int stride = sc.nblk;
    const int nblk = nb < stride ? nb : stride;
    const int lane = threadIdx.x & 63, wave = (int)(threadIdx.x >> 6);
    const int c = wave / kScanHalves, h = wave % kScanHalves;
    const int half = (nblk + kScanHalves - 1) / kScanHalves;
    const int x_lo = h * half, x_hi = min(nblk, x_lo + half);
    MLS_G int32_t *row = blk + (int64_t)c * stride;   // used by the waves that hold a bin
    if (c < kNumBins) {
        int sum = 0;
#pragma unroll 4
        for (int x = x_lo + lane; x < x_hi; x += kWave) sum += row[x];
        sum = group_sum<kWave>(sum);
        if (lane == 0) s_tot[wave] = sum;
    }
    __syncthreads();
    if (c >= kNumBins) return;
    int at = 0;
    for (int w = 0; w < wave; ++w) at += s_tot[w];
    if (h == 0 && lane == 0) {
        int tot = 0;
        for (int w = 0; w < kScanHalves; ++w) tot += s_tot[wave + w];
        gpw(sc.bin_count)[c] = tot;
    }
    for (int x0 = x_lo; x0 < x_hi; x0 += kWave * kScanPer) {
        const int xb = x0 + lane * kScanPer;
        int v[kScanPer], sum = 0;
#pragma unroll
        for (int d = 0; d < kScanPer; ++d) {
            v[d] = xb + d < x_hi ? row[xb + d] : 0;
            sum += v[d];
        }
        const int incl = group_scan_incl<kWave>(sum, lane);
        int off = at + incl - sum;
#pragma unroll
        for (int d = 0; d < kScanPer; ++d) {
            if (xb + d < x_hi) row[xb + d] = off;
            off += v[d];
        }
        at += group_total<kWave>(sum, incl);
    }
}

// Group the rows by bin: perm[start of bin c ...] = global rows of bin c in
// ascending order (ranks by wave ballots, so the order is deterministic).
// With fold (at most kFoldBlocks blocks) blk_cnt still holds the blocks'
// counts: every workgroup sums them for itself, wave w the bins w, w + 4, and
// the first one writes the bin totals, which saves the scan's launch (4.7 us
// of stream time and its 15 us run on a product of 4096 rows).
constexpr int kFoldBlocks = 256;

__global__ __launch_bounds__(kWG) void k_scatter(int na, Sched sc, int nb, int fold)
{
    __shared__ int s_wcnt[kWG / kWave][kNumBins];
    __shared__ int s_base[kNumBins];
    __shared__ int s_tot[kNumBins];
    if (bad_csr(sc.err)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int me = (int)blockIdx.x;
    if (fold) {
        for (int c = wave; c < kNumBins; c += kWG / kWave) {
            const MLS_G int32_t *row = gp(sc.blk_cnt) + (int64_t)c * sc.nblk;
            int v[kFoldBlocks / kWave], before = 0, tot = 0;
#pragma unroll
            for (int d = 0; d < kFoldBlocks / kWave; ++d) {
                const int x = d * kWave + lane;
                v[d] = x < nb ? row[x] : 0;
            }
#pragma unroll
            for (int d = 0; d < kFoldBlocks / kWave; ++d) {
                before += d * kWave + lane < me ? v[d] : 0;
                tot += v[d];
            }
            before = group_sum<kWave>(before);
            tot = group_sum<kWave>(tot);
            if (lane == 0) { s_base[c] = before; s_tot[c] = tot; }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int at = 0;
            for (int c = 0; c < kNumBins; ++c) {
                s_base[c] += at;
                at += s_tot[c];
            }
        }
        if (me == 0 && threadIdx.x < kNumBins) gpw(sc.bin_count)[threadIdx.x] = s_tot[threadIdx.x];
    } else if (threadIdx.x < kNumBins) {
        s_base[threadIdx.x] = gp(sc.blk_cnt)[threadIdx.x * sc.nblk + me];
    }
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int r0 = 0; r0 < kBinRowsPerWG; r0 += kWG) {
        const int g = me * kBinRowsPerWG + r0 + (int)threadIdx.x;
        const int c = g < na ? (int)gp(sc.cls)[g] : -1;
        int rank = 0;
#pragma unroll
        for (int cc = 0; cc < kNumBins; ++cc) {
            const unsigned long long m = __ballot(c == cc);
            if (c == cc) rank = __popcll(m & below);
            if (lane == 0) s_wcnt[wave][cc] = __popcll(m);
        }
        __syncthreads();
        if (c >= 0) {
            int off = s_base[c];
            for (int w = 0; w < wave; ++w) off += s_wcnt[w][c];
            gpw(sc.perm)[off + rank] = g;
        }
        __syncthreads();
        if (threadIdx.x < kNumBins) {
            int t = 0;
            for (int w = 0; w < kWG / kWave; ++w) t += s_wcnt[w][threadIdx.x];
            s_base[threadIdx.x] += t;
        }
        __syncthreads();
    }
}

// Numeric binning of one product of few rows by one workgroup, in place of the
// header fill, the binning, the scatter and the window scan: sizes from C's
// row pointers, counts per bin and wave, then each wave's rows placed in
// ascending order (wave w takes the rows [w * span, (w + 1) * span), read
// again from the cache: classes kept in registers spilled). The launch that
// follows has no part for the largest class: its rows join the spill bin.
// Latency bound: 4096 rows take 4 iterations, 20480 take 20.
constexpr int kSmallWG = 1024;

__device__ __forceinline__ int small_class(int nc)
{
    const int c = class_of(kModeNumeric, nc, -1);
    return c == kNumClasses - 1 ? kBinSpill : c;
}

__global__ __launch_bounds__(kSmallWG) void k_bin_small(Batch b, Sched sc, int m, int blocks)
{
    constexpr int NW = kSmallWG / kWave;
    __shared__ int s_cnt[NW][kNumBins];
    __shared__ int s_red[NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const MLS_G int32_t *crp = gp(b.p0.crp);
    if (tid == 0) *gpw(sc.err) = 0u;
    if (tid < kNumBins * kXcd) gpw(sc.task_cursor)[tid] = 0;
    const int span = ((b.na + NW - 1) / NW + kWave - 1) / kWave * kWave;
    const int r0 = wave * span, r1 = min(b.na, r0 + span);
    const unsigned long long below = (1ull << lane) - 1ull;
    int n[kNumBins];
#pragma unroll
    for (int c = 0; c < kNumBins; ++c) n[c] = 0;
#pragma unroll 4
    for (int r = r0; r < r1; r += kWave) {
        const int i = r + lane;
        const int nc = i < r1 ? crp[i + 1] - crp[i] : 0;
        const int cls = i < r1 ? small_class(nc) : -1;
        if (i < r1) gpw(sc.val)[i] = nc;
#pragma unroll
        for (int c = 0; c < kNumBins; ++c) n[c] += __popcll(__ballot(cls == c));
    }
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < kNumBins; ++c) s_cnt[wave][c] = n[c];
    }
    __syncthreads();
    int at[kNumBins], before = 0, spill0 = 0, nspill = 0;
#pragma unroll
    for (int c = 0; c < kNumBins; ++c) {
        int mine = 0, all = 0;
        for (int w = 0; w < NW; ++w) {
            mine += w < wave ? s_cnt[w][c] : 0;
            all += s_cnt[w][c];
        }
        at[c] = before + mine;
        if (c == kBinSpill) { spill0 = before; nspill = all; }
        before += all;
        if (tid == 0) gpw(sc.bin_count)[c] = all;
    }
#pragma unroll 4
    for (int r = r0; r < r1; r += kWave) {
        const int i = r + lane;
        const int cls = i < r1 ? small_class(crp[i + 1] - crp[i]) : -1;
#pragma unroll
        for (int c = 0; c < kNumBins; ++c) {
            const unsigned long long mm = __ballot(cls == c);
            if (cls == c) gpw(sc.perm)[at[c] + __popcll(mm & below)] = i;
            at[c] += __popcll(mm);
        }
    }
    if (nspill == 0) return;
    __threadfence_block();
    __syncthreads();
    // tasks of the spill rows, as k_win_scan numbers them
    MLS_G int32_t *ws = gpw(sc.wstart);
    int carry = 0;
    if (blocks) {
        int w = 0;
        for (int q = tid; q < nspill; q += kSmallWG) {
            const int i = __hip_atomic_load(sc.perm + spill0 + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            w += (crp[i + 1] - crp[i] + m - 1) / m;
        }
        w = group_sum<kWave>(w);
        if (lane == 0) s_red[wave] = w;
        __syncthreads();
        int all = 0;
        for (int x = 0; x < NW; ++x) all += s_red[x];
        blocks = all > kWinSpread;
        __syncthreads();
    }
    for (int q0 = 0; q0 < nspill; q0 += kSmallWG) {
        const int q = q0 + tid;
        int c = 0;
        if (q < nspill) {
            const int i = __hip_atomic_load(sc.perm + spill0 + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            c = (crp[i + 1] - crp[i] + m - 1) / m;
            if (blocks) {
                const int per = win_block(gp(b.p0.arp)[i + 1] - gp(b.p0.arp)[i]);
                c = (c + per - 1) / per;
            }
        }
        const int incl = group_scan_incl<kWave>(c, lane);
        if (lane == kWave - 1) s_red[wave] = incl;
        __syncthreads();
        int off = carry, all = 0;
        for (int w = 0; w < NW; ++w) {
            off += w < wave ? s_red[w] : 0;
            all += s_red[w];
        }
        if (q < nspill) ws[q] = off + incl - c;
        carry += all;
        __syncthreads();
    }
    if (tid == 0) ws[nspill] = carry;
}

// ---------------------------------------------------------------------------
// Exclusive scan of the per-row counts into int64 prefixes, then the int32
// row pointers of each product.

constexpr int kScanTile = 2048;   // rows per workgroup (8 per thread)

__global__ void k_scan_tiles(const int32_t *val, int n, int64_t *tile_sum)
{
    __shared__ int64_t red[kWG / kWave];
    int64_t s = 0;
    int base = blockIdx.x * kScanTile;
    for (int r = threadIdx.x; r < kScanTile; r += kWG) {
        int g = base + r;
        if (g < n) s += val[g];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w = 0; w < kWG / kWave; ++w) t += red[w];
        tile_sum[blockIdx.x] = t;
    }
}

// One workgroup: exclusive scan of the tile sums in place.
__global__ void k_scan_sums(int64_t *tile_sum, int ntiles)
{
    __shared__ int64_t part[kWG];
    int per = (ntiles + kWG - 1) / kWG;
    int lo = threadIdx.x * per, hi = min(ntiles, lo + per);
    int64_t s = 0;
    for (int i = lo; i < hi; ++i) s += tile_sum[i];
    part[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t run = 0;
        for (int w = 0; w < kWG; ++w) { int64_t v = part[w]; part[w] = run; run += v; }
    }
    __syncthreads();
    int64_t run = part[threadIdx.x];
    for (int i = lo; i < hi; ++i) { int64_t v = tile_sum[i]; tile_sum[i] = run; run += v; }
}

__global__ void k_scan_apply(const int32_t *val, int n, const int64_t *tile_off, int64_t *prefix)
{
    // 256 threads x 8 consecutive rows
    __shared__ int64_t wsum[kWG / kWave];
    int base = blockIdx.x * kScanTile + threadIdx.x * 8;
    int64_t v[8];
    int64_t s = 0;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        int g = base + r;
        v[r] = g < n ? val[g] : 0;
        s += v[r];
    }
    // inclusive scan of s across the wave
    int lane = threadIdx.x & 63;
    int64_t incl = s;
    for (int o = 1; o < 64; o <<= 1) {
        int64_t y = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[threadIdx.x >> 6] = incl;
    __syncthreads();
    int64_t off = tile_off[blockIdx.x];
    for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) off += wsum[w];
    int64_t run = off + incl - s;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        int g = base + r;
        if (g < n) prefix[g] = run;
        run += v[r];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kWG - 1) prefix[n] = run;
    if (base + 8 >= n && base < n) prefix[n] = run;
}

// Row pointers of every product from the global prefix; totals[t] = nnz(C_t).
__global__ void k_write_rowptr(Batch b, const int64_t *prefix, int64_t *totals, uint32_t *err)
{
    if (bad_csr(err)) return;
    int g = blockIdx.x * blockDim.x + threadIdx.x;
    const int t = b.nprob == 1 ? 0 : find_prob_rows(b.abase, b.nprob, g - (int)(threadIdx.x & 63), g);
    if (g >= b.na) return;
    const Prob P = get_prob_any(b, t);
    int r0 = b.nprob == 1 ? 0 : gp(b.abase)[t];
    int i = g - r0;
    int64_t v = prefix[g + 1] - prefix[r0];
    if (v >= 0x7fffffffLL) { atomicOr(err, kErrOverflow); v = 0x7fffffff; }
    gpw(P.crp)[i + 1] = (int32_t)v;
    if (i == 0) gpw(P.crp)[0] = 0;
    if (i == P.nrows - 1) totals[t] = prefix[g + 1] - prefix[r0];
}

// ---------------------------------------------------------------------------
// launchers

static inline int nblk(int64_t n, int per) { return (int)((n + per - 1) / per); }

void launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s)
{
    if (n <= 0) return;
    int grid = nblk(n, kWG);
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid), dim3(kWG), 0, s, p, v, n);
}

void launch_fill_f64(double *p, double v, int64_t n, hipStream_t s)
{
    if (n <= 0) return;
    int grid = nblk(n, kWG);
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(k_fill_f64, dim3(grid), dim3(kWG), 0, s, p, v, n);
}

void launch_zero2_f64(double *p, int64_t n, double *q, int64_t m, hipStream_t s)
{
    if (!p) n = 0;
    if (!q) m = 0;
    if (n + m <= 0) return;
    int grid = nblk(n + m, kWG);
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(k_zero2_f64, dim3(grid), dim3(kWG), 0, s, p, n, q, m);
}

// Rows per wave of the entry streams: about a tile of entries (512) on
// average, at least 8 rows. Few rows also bound the run of entries that falls
// to one wave where long rows lie next to each other.
static int stream_rows(int64_t rows, int64_t nnz)
{
    int rw = 64;
    while (rw > 8 && (int64_t)rw * nnz > kTileEntries * rows) rw >>= 1;
    return rw;
}

void launch_validate(const Batch &b, int which, const int64_t *nnz_tab, int64_t nnz_a, int64_t nnz_b, uint32_t *err,
                     hipStream_t s)
{
    constexpr int nw = kWG / kWave;
    const int rw_a = stream_rows(b.na, nnz_a), rw_b = stream_rows(b.nb, nnz_b);
    const int a_blocks = which == 1 ? 0 : nblk(b.na, nw * rw_a), b_blocks = which == 0 ? 0 : nblk(b.nb, nw * rw_b);
    if (a_blocks + b_blocks <= 0) return;
    ProfScope ps("validate", s);
    hipLaunchKernelGGL(k_validate, dim3(a_blocks + b_blocks), dim3(kWG), 0, s, b, which, nnz_tab, nnz_a, nnz_b,
                       a_blocks, rw_a, rw_b, err);
}

void launch_compress(const Batch &b, int64_t nnz_b, const uint32_t *err, hipStream_t s)
{
    if (b.nb <= 0) return;
    ProfScope ps("compress", s);
    const int rw = stream_rows(b.nb, nnz_b);
    hipLaunchKernelGGL(k_compress, dim3(nblk(b.nb, kWG / kWave * rw)), dim3(kWG), 0, s, b, rw, err);
}

void launch_bin_count(const Batch &b, int64_t nnz_a, const Sched &sc, int force, hipStream_t s)
{
    if (b.na <= 0) return;
    {
        ProfScope ps("work", s);
        const int rw = stream_rows(b.na, nnz_a);
        hipLaunchKernelGGL(k_work, dim3(nblk(b.na, kWG / kWave * rw)), dim3(kWG), 0, s, b, rw, sc);
    }
    launch_bin(b, kModeSized, sc, force, nullptr, s);
}

void launch_bin(const Batch &b, int mode, const Sched &sc, int force, unsigned long long *total,
                hipStream_t s)
{
    if (b.na <= 0) return;
    {
        ProfScope ps("bin", s);
        hipLaunchKernelGGL(k_bin, dim3(nblk(b.na, kBinRowsPerWG)), dim3(kWG), 0, s, b, mode, sc, force, total);
    }
    launch_scatter(b.na, sc, s);
}

// Bin scan and scatter after a binning kernel (blocks of kBinRowsPerWG rows).
void launch_scatter(int na, const Sched &sc, hipStream_t s)
{
    if (na <= 0) return;
    ProfScope ps("scatter", s);
    const int nb = nblk(na, kBinRowsPerWG);
    const int fold = nb <= kFoldBlocks;
    if (!fold) hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(kScanWG), 0, s, sc, nb);
    hipLaunchKernelGGL(k_scatter, dim3(nb), dim3(kWG), 0, s, na, sc, nb, fold);
}

void launch_bin_small(const Batch &b, const Sched &sc, int m, int blocks, hipStream_t s)
{
    ProfScope ps("bin_small", s);
    hipLaunchKernelGGL(k_bin_small, dim3(1), dim3(kSmallWG), 0, s, b, sc, m, blocks);
}

int scan_tiles(int n) { return nblk(n > 0 ? n : 1, kScanTile); }

void launch_scan(const int32_t *val, int n, int64_t *tile_sum, int64_t *prefix, hipStream_t s)
{
    int nt = scan_tiles(n);
    ProfScope ps("scan", s);
    hipLaunchKernelGGL(k_scan_tiles, dim3(nt), dim3(kWG), 0, s, val, n, tile_sum);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kWG), 0, s, tile_sum, nt);
    hipLaunchKernelGGL(k_scan_apply, dim3(nt), dim3(kWG), 0, s, val, n, tile_sum, prefix);
}

void launch_write_rowptr(const Batch &b, const int64_t *prefix, int64_t *totals, uint32_t *err, hipStream_t s)
{
    if (b.na <= 0) return;
    ProfScope ps("write_rowptr", s);
    hipLaunchKernelGGL(k_write_rowptr, dim3(nblk(b.na, kWG)), dim3(kWG), 0, s, b, prefix, totals, err);
}

}  // namespace mls
