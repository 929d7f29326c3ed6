// Device kernels of the hierarchy setup (Section 2, amg_setup: strength ->
// C/F split -> interpolation -> Galerkin product) for gfx950.
//
// Every step reproduces the host setup's arithmetic bit for bit: per-row
// sums run in ascending column order in one thread, and each entry of the
// Galerkin products adds its terms in the canonical order (ascending inner
// index, first term assigned), whether row by row in LDS or listed, sorted
// stably by (row, column) and summed.  The C/F split is either the
// Ruge-Stueben first pass (computed elsewhere) or PMIS, the parallel
// aggressive coarsening Section 1 cites, in rounds on the device.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace amg355 {

// point states of the C/F split
constexpr int32_t kPtUndecided = 0, kPtC = 1, kPtF = 2;

// error bits of the input check and of the symmetrization
enum SetupError : int {
    kErrRowPtr = 1,          // row_ptr not 0-based, decreasing or not ending at nnz
    kErrColRange = 2,        // column index out of range
    kErrColOrder = 4,        // columns not strictly ascending in a row
    kErrNonFinite = 8,       // NaN or infinite value
    kErrNoDiag = 16,         // no stored diagonal
    kErrDiagSign = 32,       // diagonal not positive
    kErrAsymmetric = 64,     // (j,i) missing or a_ji != a_ij bitwise
    kErrPattern = 128,       // coarse product pattern not structurally symmetric
};

// err[0] |= error bits, err[1] = min offending row (init INT32_MAX)
void launch_validate_csr(int n, int64_t nnz, const int32_t* rp, const int32_t* ci, const double* v,
                         int* err, hipStream_t st);

// strength (negative couplings, -a_ij >= fl(theta max_{k!=i}(-a_ik))): the
// strong columns of row i from sci[rp[i]] on, their number cnt[i], and
// lambda_j = #{i : S_ij} (lam zeroed by the caller)
void launch_strength(int n, int64_t nnz, const int32_t* rp, const int32_t* ci, const double* v, double theta,
                     int32_t* cnt, int32_t* sci, int32_t* lam, hipStream_t st);

// PMIS: weights w_i = lambda_i + u_i with u_i the top 53 bits of output i+1
// of the SplitMix64 stream `seed`; lambda_i = 0 points start as F
void launch_pmis_init(int n, const int32_t* lam, uint64_t seed, double* w, int32_t* state, int32_t* mark,
                      hipStream_t st);
// one round: local maxima among undecided points become C, then undecided
// points depending strongly on a C point become F; *undecided receives the
// number left (a round without undecided points changes nothing)
void launch_pmis_round(int n, const int32_t* rp, const int32_t* cnt, const int32_t* sci, const double* w,
                       int32_t* state, int32_t* mark, int round, int32_t* undecided, hipStream_t st);

// flag[i] = 1 for C points, pcnt[i] the entries of P's row i; after the scans
// c_points[cidx[i]] = i, code[i] = cidx[i] for C points and -1 for F points
void launch_split_counts(int n, const int32_t* rp, const int32_t* cnt, const int32_t* sci, const int32_t* state,
                         int32_t* flag, int32_t* pcnt, hipStream_t st);
void launch_c_points(int n, const int32_t* state, const int32_t* cidx, int32_t* c_points, int32_t* code,
                     hipStream_t st);

// direct interpolation: the entries of P
void launch_interp_fill(int n, int64_t nnz, const int32_t* rp, const int32_t* ci, const double* v, double theta,
                        const int32_t* code, const int32_t* prp, int32_t* pci, double* pv, hipStream_t st);

// ---- products and transposes row by row (product_kernels.hip) --------------
// out = X Y: X in CSR, Y in CSR (yrp) or loose rows (row l from yoff[l] on,
// ylen[l] entries); out's rows loose, row i from off[i] on
struct ProductArgs {
    int rows;
    const int32_t *xrp, *xci;
    const double* xv;
    const int32_t* yrp;
    const int64_t *yoff, *ylen;
    const int32_t* yci;
    const double* yv;
    const int64_t* off;
    int32_t* oci;
    double* ov;
    int64_t* olen;
};
// The row kernels take products whose largest row has at most kProductRowTerms
// terms (the steps of a row follow each other, about 0.4 us each) and whose mean
// row kProductMeanTerms: beyond, most rows have more columns than a table holds.
// Sorted, the terms of all rows go in parallel.
constexpr int kProductRowTerms = 8192;
constexpr double kProductMeanTerms = 1024.0;
// most entries of a row of a transpose that is ordered by rank (each entry is
// compared with all)
constexpr int kOrderedRow = 2048;
// terms[i] of every row (terms[rows] = 0), the largest raised in *most
void launch_product_terms(const ProductArgs& a, int64_t* terms, int32_t* most, hipStream_t st);
// mean_row: mean length of the rows of Y that are read; mean_terms: of the
// product's rows; list: 2 rows entries; counts[0..1] zero on entry, counts[1] >
// 0 on exit: rows with more columns than a table holds, whose result is missing
void launch_row_product(const ProductArgs& a, double mean_row, double mean_terms, int32_t* list, int32_t* counts,
                        hipStream_t st);
// (c_ij + c_ji) / 2 of loose rows in CSR (start: scanned lengths); err |=
// kErrPattern where (j,i) is missing
void launch_pack_symmetrized(int n, const int64_t* off, const int64_t* len, const int32_t* lci, const double* lv,
                             const int64_t* start, int32_t* rp, int32_t* ci, double* v, int* err, hipStream_t st);
// transpose: places of the entries in their columns (cnt zeroed by the caller,
// the largest count raised in *most), the entries at their places, the rows in
// ascending order
void launch_column_places(int64_t nnz, const int32_t* ci, int32_t* cnt, int32_t* place, int32_t* most, hipStream_t st);
void launch_column_fill(int rows, const int32_t* rp, const int32_t* ci, const double* v, const int32_t* place,
                        const int32_t* trp, int32_t* tci, double* tv, hipStream_t st);
void launch_order_rows(int rows, const int32_t* rp, const int32_t* uci, const double* uv, int32_t* ci, double* v,
                       hipStream_t st);

// values of up to four device words (int32 or int64 each), then a sequence
// number, to host-coherent memory
struct PublishWords {
    const void* src[4];
    int bytes[4];
    int count;
};
void launch_publish_words(const PublishWords& w, int64_t* host, uint32_t* flag, uint32_t seq, hipStream_t st);

// ---- the same through sorted terms: rows of any length ----------------------
// keys (column << row_bits | row) of every entry of a CSR matrix, with values
void launch_transpose_keys(int rows, const int32_t* rp, const int32_t* ci, const double* v, int row_bits,
                           uint64_t* keys, double* vals, hipStream_t st);

// the terms of each of X's nnz entries (terms[nnz] = 0), then the m terms of a
// product, row by row in order, entry p's from start[p] (the scan) on
void launch_entry_terms(const ProductArgs& a, int64_t nnz, int64_t* terms, hipStream_t st);
void launch_expand_terms(const ProductArgs& a, int64_t nnz, int64_t m, const int64_t* start, int col_bits,
                         uint64_t* keys, double* vals, hipStream_t st);
// a CSR row pointer as starts and lengths (rows + 1 entries each, the last
// length 0)
void launch_loose_rows(int rows, const int32_t* rp, int64_t* off, int64_t* len, hipStream_t st);

// sorted (key, value) list -> head flags of equal-key runs
void launch_run_heads(int64_t m, const uint64_t* keys, int64_t* flags, hipStream_t st);
// every run summed in list order (first term assigned): column and value of
// output entry head_index[q] for each head q; the run's key is copied to
// out_keys
void launch_run_sums(int64_t m, const uint64_t* keys, const double* vals, const int64_t* head_index,
                     int col_bits, int32_t* out_ci, double* out_v, uint64_t* out_keys, hipStream_t st);
// row pointer (rows + 1 entries) of m entries whose sorted keys hold the row
// above col_bits
void launch_rowptr_from_keys(int64_t m, const uint64_t* keys, int col_bits, int rows, int32_t* rp,
                             hipStream_t st);
// column and value of each sorted (key, value) pair
void launch_unpack_keys(int64_t m, const uint64_t* keys, const double* vals, int col_bits, int32_t* ci,
                        double* v, hipStream_t st);

// stable ascending sort of (key, value) pairs on bits [0, bits) (keys and
// vals are double buffers; returns which buffer holds the result) and
// exclusive scan of int64 counts (out[m] = total: in has m + 1 entries, the
// last 0); temp == nullptr queries the scratch size
hipError_t sort_pairs(void* temp, size_t& temp_bytes, uint64_t* keys[2], double* vals[2], int64_t m, int bits,
                      int& result, hipStream_t st);
hipError_t scan_counts(void* temp, size_t& temp_bytes, const int64_t* in, int64_t* out, int64_t m,
                       hipStream_t st);

}  // namespace amg355
