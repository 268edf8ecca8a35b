// launch.h -- host-side launchers of the gfx950 kernels (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace mls {

enum { kModeCount = 0, kModeFill = 1, kModeNumeric = 2, kModeWork = 3, kModeSized = 4 };

void launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s);
void launch_fill_f64(double *p, double v, int64_t n, hipStream_t s);
// Both arrays in one launch (either may be NULL or empty).
void launch_zero2_f64(double *p, int64_t n, double *q, int64_t m, hipStream_t s);
// CSR checks: which = 0 A, 1 B, 2 both in one launch. The entry counts come
// from nnz_tab (device, two per product), or, when it is NULL (one product),
// from nnz_a and nnz_b (which are the batch's totals otherwise).
void launch_validate(const Batch &b, int which, const int64_t *nnz_tab, int64_t nnz_a, int64_t nnz_b, uint32_t *err,
                     hipStream_t s);
// nnz_b: entries of all B. err (may be NULL): the error word of a CSR check
// queued before.
void launch_compress(const Batch &b, int64_t nnz_b, const uint32_t *err, hipStream_t s);
// Binning of a count pass; nnz_a: entries of all A.
void launch_bin_count(const Batch &b, int64_t nnz_a, const Sched &sc, int force, hipStream_t s);
void launch_bin(const Batch &b, int mode, const Sched &sc, int force, unsigned long long *total,
                hipStream_t s);
int scan_tiles(int n);
void launch_scan(const int32_t *val, int n, int64_t *tile_sum, int64_t *prefix, hipStream_t s);
void launch_write_rowptr(const Batch &b, const int64_t *prefix, int64_t *totals, uint32_t *err, hipStream_t s);

// Symbolic phase: count (fill == 0) or fill (fill == 1) over the binned rows.
// G = lanes per row for the LDS classes.
void launch_symbolic(const Batch &b, const Sched &sc, int fill, int G, hipStream_t s);

// Symbolic phase by dense bitmaps, of B's columns or of compressed B's words: one
// product of at most kBitMaxCols columns. A wave's bitmap then takes at most 8
// KB of LDS, which leaves 20 waves per CU resident; each doubling halves them
// (60000 random rows of 30 times 30, binned / bitmaps: 1573 / 349 us in 8192
// columns, 1606 / 305 in 32768, 1598 / 443 in 65536).
constexpr int kBitMaxCols = 65536;
enum SymBits { kBitsNone, kBitsColumns, kBitsWords };
SymBits symbit_choose(const Batch &b, double avg_a, double avg_b);
void launch_symbit(const Batch &b, const Sched &sc, int fill, bool words, hipStream_t s);
// Row pointers and nnz(C) of one product of few rows in one launch of one
// workgroup (17 us for 16384 rows, 30 for 30000, 61 for 65536; the four
// launches that take more rows, 20 us for all of these).
constexpr int kRowptrSmallRows = 16384;
void launch_rowptr_small(const Batch &b, const int32_t *val, int64_t *total, uint32_t *err, hipStream_t s);

// Fill pass from the count pass's scratch words (rows with scnt >= 0); seen: the
// sizes that any row has (bits kSeen*).
void launch_sym_expand(const Batch &b, const Sched &sc, unsigned seen, hipStream_t s);

// Tasks of the spill bin's rows, ceil(size / m) windows per row, one per task
// or (blocks) win_block of the row's entries: sc.wstart[r] = the first task of
// the r-th spill row, sc.wstart[n] = their total (one workgroup).
constexpr int kWinScanWG = 1024;
__global__ void k_win_scan(Batch b, Sched sc, int m, int blocks);

// Products of at most kSmallRows rows (one product, columns that fit the
// packed tables): the numeric phase as two launches, one workgroup that bins
// the rows (those of the largest class with the spill rows), clears the
// scheduling counters (and the error word, which it owns) and numbers the
// windows of `m` positions, and one launch for every class. Up to 20480 rows:
// beyond, the one workgroup that bins takes longer than the launches it saves
// (random rows of 36 outputs, numeric / adjoint in us by class and in two
// launches: 12000 rows 55/57 and 32/39, 20000 rows 50/58 and 46/55, 32000
// rows 66/77 and 67/80).
// Its workgroups hold few waves where rows are long, so products with many outputs
// go by class: thresholds and figures at num_small_fit and bwd_small_fit
// (outputs: entries of C, or of W).
constexpr int kSmallRows = 20480;
// Five workgroups per CU; four stay resident (104 and 112 vector registers).
// Compiled for five, with 4 and 36 registers spilled, the kernels take as long
// (20000 rows of 36 to 450 outputs within 1 %); 1024 workgroups, 1280: numeric
// 20000 rows of 36 outputs 39, 44 us, of 100 61, 70, of 250 113, 101, of 450 149, 131.
constexpr int kSmallGrid = 1280;
bool num_small_fit(const Batch &b, int64_t outputs);
bool bwd_small_fit(const Batch &b, int64_t outputs);
bool small_rows_fit(const Batch &b);
int small_rows_grid(int na, int64_t outputs);
void launch_bin_small(const Batch &b, const Sched &sc, int m, int blocks, hipStream_t s);
void launch_numeric_small(const Batch &b, const Sched &sc, int64_t outputs, hipStream_t s);
void launch_backward_small(const Batch &b, const Sched &sc, double *dA, double *dB, int64_t outputs, hipStream_t s);

// Numeric phase (row-range fused multiply-add) over the binned rows.
void launch_numeric(const Batch &b, const Sched &sc, int G, hipStream_t s);
// The same with the lanes per row of the first (G1) and second (G2) LDS classes
// given, and, where the caller knows them, the rows of every bin (n_bin, host):
// bins without rows are not launched.
void launch_numeric_groups(const Batch &b, const Sched &sc, int G1, int G2, const int32_t *n_bin, hipStream_t s);

// Triangle counting over the binned rows of L (A = B = L in the batch).
void launch_tc(const Batch &b, const Sched &sc, int64_t *counts, unsigned long long *total,
               uint32_t *spill_bitmaps, int spill_slots, int64_t spill_words, hipStream_t s);
void launch_tc_bin(const Batch &b, const Sched &sc, int force, hipStream_t s);
void launch_scatter(int na, const Sched &sc, hipStream_t s);

// Backward (adjoint) over the binned rows of W (= pattern of C).
void launch_backward(const Batch &b, const Sched &sc, const double *wval, double *dA, double *dB, int G,
                     hipStream_t s);

// Deterministic adjoint (one lane per output entry, sequential sums; W_ij by
// binary search in W_i). trp/tci/tv: the transpose of A with its values.
void launch_backward_det(int32_t m, int32_t kb, int64_t nnz_b, int64_t nnz_w, const int32_t *arp, const int32_t *aci,
                         const int32_t *brp, const int32_t *bci, const double *bval, const int32_t *wrp,
                         const int32_t *wci, const double *wval, const int32_t *trp, const int32_t *tci,
                         const double *tv, double *dA, double *dB, uint32_t *err, hipStream_t s);

// Transpose and masked gather helpers. cursor: ncols words somewhere behind cnt
// in the same allocation (both, and what lies between, are cleared).
void launch_transpose(int32_t nrows, int32_t ncols, int64_t nnz, const int32_t *rp, const int32_t *ci, const double *v,
                      int32_t *trp, int32_t *tci, double *tv, int32_t *cursor, int64_t *tile_sum,
                      int64_t *prefix, int32_t *cnt, hipStream_t s);
void launch_mask_gather(int32_t nrows, const int32_t *xrp, const int32_t *xci, const double *xv,
                        const int32_t *prp, const int32_t *pci, double *out, hipStream_t s);

// Persistent grid sizes (workgroups) per kernel shape.
int device_cu_count();
int device_max_lds();   // LDS bytes one workgroup may allocate

// Workgroups of a persistent grid: resident workgroups per CU times the CUs,
// for a kernel of kWG threads with `smem` bytes of dynamic LDS.
template <typename K>
inline int spill_grid(K kernel, int smem)
{
    static int cus = device_cu_count();
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kWG, (size_t)smem) != hipSuccess || per_cu < 1)
        per_cu = 1;
    return cus * per_cu;
}

}  // namespace mls
