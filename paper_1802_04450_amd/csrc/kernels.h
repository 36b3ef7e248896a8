// Launch wrappers of the gfx950 kernels.  All pointers are device pointers unless said otherwise;
// every wrapper only enqueues work on `st` and returns hipGetLastError().
//
// Dense blocks are row-major: element (i, c) of a block with leading dimension ld is p[i*ld + c].
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sceig {

constexpr int kMaxBlock = 32;      // largest Lanczos block size
constexpr int kLongRow = 128;      // rows with more entries than this are "long" for the wide sparse products
constexpr int kPartialPad = 32;    // column stride of partial / coefficient blocks (>= kMaxBlock)
constexpr int kPairPad = 64;       // the same for two blocks side by side of more than kMaxBlock columns together

// ---- setup ---------------------------------------------------------------------------------
// host[0] = *wide, host[1] = *a, host[2] = *b (what is null is left out), and then host[3] = 1, in coherent host memory: what the
// host waits for comes without a copy and without waiting for the stream (a word to the host 12 us sooner).
hipError_t launch_report(const int64_t* wide, const int32_t* a, const int32_t* b, int64_t* host, hipStream_t st);
// Host: until *word = value, which a kernel on st writes to coherent host memory.  An error where the stream has come to its end
// without that: what the word stands for is then whatever the memory held.
hipError_t wait_for_word(const int64_t* word, int64_t value, hipStream_t st);
hipError_t wait_for_word(const int32_t* word, int32_t value, hipStream_t st);
// nnz < 0: it is read from rowptr[n].
// flag[0] |= 1 if rowptr is not monotone / rowptr[0] != 0, |= 2 if a column is out of range.
hipError_t launch_validate_csr(const int64_t* rowptr, const int32_t* col, int64_t n, int64_t nnz, int* flag,
                               hipStream_t st);
// flag[0] |= 8 if W is not symmetric (for some entry (i, j) the weights listed in row i under column j and in row j
// under column i add up to different values), |= 16 if a weight is negative or not finite.  Only for a CSR that
// launch_validate_csr has accepted (columns are used as row indices).
hipError_t launch_validate_symmetry(const int64_t* rowptr, const int32_t* col, const double* val, int64_t n, int* flag,
                                    hipStream_t st);
// d_i = sum of row i, s_i = d_i^-1/2; flag[0] |= 4 if some d_i is <= 0 or not finite, |= kBelowZero if some weight is below
// zero.  d may be null.
constexpr int kBelowZero = 32;
hipError_t launch_degree_scaling(const int64_t* rowptr, const double* val, int64_t n, double* d, double* s, int* flag,
                                 hipStream_t st);

// ---- sparse product ------------------------------------------------------------------------
// z[i*b + t] = s[i] * x[i*ldx + t]   (packed scaled copy of an n x b block)
hipError_t launch_pack_scaled(const double* x, int64_t ldx, const double* s, int64_t n, int b, double* z,
                              hipStream_t st);
// y[i*ldy + t] = s[i] * sum_e val[e] * z[col[e]*b + t]  over the entries e of row i; b in {1,2,4,8,16,32}.
// s == null: no row scaling (the values are the scaled operator S_ij and z = x).
// avg_deg steers the lanes-per-row choice of the b <= 4 kernels.
hipError_t launch_spmm(const int64_t* rowptr, const int32_t* col, const double* val, const double* s, int64_t n,
                       const double* z, int b, double* y, int64_t ldy, double avg_deg, hipStream_t st);

// Single-vector product inside a chain of products: z = s o x (the operand, scaled by the call that produced x),
// y = s o (W z), zout = s o y (the operand of the next product), one launch.
hipError_t launch_spmv_chain(const int64_t* rowptr, const int32_t* col, const double* val, const double* s, int64_t n,
                             const double* z, double* y, double* zout, double avg_deg, hipStream_t st);

// ---- tall-skinny projections (fp64 MFMA) ---------------------------------------------------
struct ProjectPlan {
  int rows_per_panel;  // multiple of 4
  int nwc;             // waves of a workgroup laid along the columns (1, 2 or 4)
  int npart;           // number of partial blocks produced = row panels (one per workgroup: waves that share a
                       // column tile add their sums inside the workgroup)
};
// max_partials: partial blocks of kPartialPad columns that there is room for.
ProjectPlan plan_project(int64_t n, int ja, int max_partials, int b = 1);
// part[p][c][t] (c < ja, t < kPartialPad) = sum over the rows of partial p of A[i, acol0 + c] * B[i, bcol0 + t]
// with A and B both columns of `basis` (row-major n x ld); t >= b entries are written as 0.  b <= 2 kMaxBlock, with the plan
// for that b; kPairPad takes the place of kPartialPad, here and in launch_reduce_partials, where b > kMaxBlock.
// skip (here and below; may be null): device int; if *skip != 0 when the kernel starts, the launch does nothing.
hipError_t launch_project(const double* basis, int64_t n, int64_t ld, int acol0, int ja, int bcol0, int b,
                          const ProjectPlan& plan, double* part, hipStream_t st, const int* skip = nullptr);
// h[c*kPartialPad + t] = sum_p part[p][c][t] in the fixed order p = 0..npart-1 (t < b, else 0);
// if hsum != null: hsum = (accumulate ? hsum : 0) + h.
// if slot != null: rows [slot_row0, ja) of the resulting hsum (or h) are copied to slot[(c-slot_row0)*kPartialPad + t].
hipError_t launch_reduce_partials(const double* part, int npart, int ja, int b, double* h, double* hsum,
                                  int accumulate, double* slot, int slot_row0, hipStream_t st,
                                  const int* skip = nullptr);
// skip[0] = 1 when no column of the block needs a second Gram-Schmidt pass: for every column t < b the squared norm
// the first pass removed, the sum of the squares of the t-th column of h (rows x b, row stride pad) and of h2, is at most ratio2
// times the squared norm it kept, gram[t*kPartialPad + t]; else skip[0] = 0.
struct Removed {
  const double* h = nullptr;
  int rows = 0, pad = kPartialPad;
};
hipError_t launch_second_pass_test(Removed h, Removed h2, int b, const double* gram, double ratio2, int* skip,
                                   hipStream_t st);

// C = A * B row GEMM:  A = basis[:, acol0 : acol0+kdim] (n x kdim), B = bmat (kdim x ncols, row-major, ldb).
// mode 0: basis[:, ccol0 + t] -= C[:, t]          (in place update, ncols <= 64, out unused)
// mode 1: out[i*ldo + t]  = C[i, t]                (row-major)
// mode 2: out[t*ldo + r(i)] = C[i, t]             (column-major; r(i) = rowmap[i] if rowmap != null, else i)
// mode 3: basis[:, ccol0 + t] = C[:, t]           (ncols <= 64, out unused; the columns written may be among the
//         columns read: one wave owns all ncols entries of its rows and stores them after its last read of those rows)
hipError_t launch_row_gemm(double* basis, int64_t n, int64_t ld, int acol0, int kdim, const double* bmat, int ldb,
                           int ncols, int mode, int ccol0, double* out, int64_t ldo, const int32_t* rowmap,
                           hipStream_t st, const int* skip = nullptr);

// ---- block orthonormalization --------------------------------------------------------------
// One Cholesky-QR pass bookkeeping on the Gram matrix g_in (b x b, stride kPartialPad; single workgroup):
//   Cholesky g = r^T r with dependent columns dropped (zero row in r, zero row+column in rinv);
//   rinv = r^-1 on the kept columns; g_out = symmetrised copy of g_in.
//   If rprev != null: rout = r * rprev (composition of two passes) else rout = r.  Any output may be null.
hipError_t launch_gram_cholesky(const double* g_in, int b, double* g_out, double* rinv, double* rout,
                                const double* rprev, double abs_tol2, double rel_tol, hipStream_t st);
// The same on the sum of nparts partial Gram blocks (as launch_project and launch_update_gram leave them), as the first
// part of the launch that applies rinv, where gram_cholesky_takes_parts says that this is the cheaper way.
struct GramParts {
  const double* parts = nullptr;
  int nparts = 0;
  double *g_out = nullptr, *r_out = nullptr;  // may be null
  const double* rprev = nullptr;
  double abs_tol2 = 0.0, rel_tol = 0.0;
};
bool gram_cholesky_takes_parts(int npart, int b);
// W <- W rinv for W = basis[:, col : col+b]; gpart: the partial Gram matrices of the new block (see launch_update_gram),
// another buffer than f.parts
hipError_t launch_factor_update_gram(double* basis, int64_t n, int64_t ld, int col, int b, const GramParts& f, double* gpart,
                                     hipStream_t st);
// as launch_apply_rinv
hipError_t launch_factor_apply_rinv(double* basis, int64_t n, int64_t ld, int col0, int b, const GramParts& f, double* z,
                                    const double* s, hipStream_t st);
// basis[:, col0 : col0+b] = basis[:, col0 : col0+b] * rinv  (rinv b x b row-major stride kPartialPad);
// if z != null also z[i*b + t] = s[i] * new value.
hipError_t launch_apply_rinv(double* basis, int64_t n, int64_t ld, int col0, int b, const double* rinv, double* z,
                             const double* s, hipStream_t st);

// One block step, or the QR of a block, as one launch whose workgroups exchange partial sums while it runs: for few rows,
// where the launches of a step are each as long as a launch takes at least.
//   launch_fused_step: columns [j, j + kFusedStepBlock) of the basis become the product of the operator (rowptr, col, val) with
//     z, orthogonalized against columns [from1, j) and once more against [from2, j) (from >= j: not), and then as below.  slot_a:
//     the sum of both passes' coefficients of columns [j - kFusedStepBlock, j).
//   launch_fused_qr: columns [j, j + b) are made orthonormal by two Cholesky QRs as launch_gram_cholesky does, and z becomes a
//     packed copy of them.  slot_g: the Gram matrix before the first factorization; slot_r: the factor of both.
// Rows of the slots are slot_ld long; z and, but for launch_fused_step, the slots may be null.
// The workgroups wait for one another.  If, after `polls` looks, one has not started yet (other work holds the compute units), the
// launch leaves without having done anything, and so do all further ones with this sync, and the caller takes the step by other
// launches.  Slots and *done may be in coherent host memory: *done becomes `number` when all workgroups are through and the slots
// are written (-number: they had all started, but did not come to an end); it is not touched else.  base: the workgroups of all
// launches with this sync so far. exchange: fused_exchange() doubles of all ones, which the launch writes; the first `clear`
// doubles of used, those of the launch before, become all ones again (two such areas take turns).
constexpr int kFusedStepBlock = 8;
constexpr int kFusedGroups = 256;   // workgroups at most
constexpr int kFusedColumns = 256;  // j of launch_fused_step at most
constexpr int kSyncWord = 16, kSyncDone = 48, kSyncWords = 64;  // the words that count, on cache lines of their own; 0 .. 15 are the caller's
struct FusedStep {
  const int64_t* rowptr = nullptr;
  const int32_t* col = nullptr;
  const double* val = nullptr;
  double *basis = nullptr, *z = nullptr;
  int64_t n = 0, ld = 0;
  int j = 0, from1 = 0, from2 = 0;
  int rows = 0;  // rows a workgroup: fused_step_rows, fused_qr_rows
  double *slot_a = nullptr, *slot_g = nullptr, *slot_r = nullptr;
  int slot_ld = kPartialPad;
  int* done = nullptr;
  int number = 1;
  uint32_t* sync = nullptr;
  uint32_t base = 0;
  int polls = 0;
  double *exchange = nullptr, *used = nullptr;
  int64_t clear = 0;
  double abs_tol2[2] = {0.0, 0.0}, rel_tol[2] = {0.0, 0.0};
};
// Rows that a workgroup takes; 0: the call is not for this kernel (too many rows, or columns, for the workgroups' LDS).
int fused_step_rows(int64_t n, int j, size_t lds_limit);
int fused_qr_rows(int64_t n, int b, size_t lds_limit);
inline int fused_groups(int64_t n, int rows) { return (int)((n + rows - 1) / rows); }
// Sums of j1 and j2 x b coefficients and two Gram matrices, with the workgroups' shares of them.
inline int64_t fused_exchange(int groups, int j1, int j2, int b) { return (int64_t)(groups + 1) * b * (j1 + j2 + 2 * b); }
// Before the first launch with this sync (kSyncWords) and these areas; stopped: as after a launch that has left.
hipError_t launch_fused_prepare(double* exchange, int64_t len, uint32_t* sync, bool stopped, hipStream_t st);
// For tests: from here on as after a launch that has left.
hipError_t launch_fused_stop(uint32_t* sync, hipStream_t st);
hipError_t launch_fused_step(const FusedStep& a, size_t lds_limit, hipStream_t st);
hipError_t launch_fused_qr(const FusedStep& a, int b, size_t lds_limit, hipStream_t st);

// Fused variant used inside the block step (same arithmetic as the separate kernels):
//   update_gram: basis[:, ccol0 : ccol0+b] -= basis[:, acol0 : acol0+kdim] * bmat (bmat kdim x b, row stride
//                kPartialPad) and
//                gpart[p] (b x b, row stride kPartialPad, p < plan_update_gram(n)) = partial Gram matrices of the
//                updated block, to be summed with launch_reduce_partials(gpart, npart, b, b, ...).
int plan_update_gram(int64_t n);
// overwrite = 1: the block is replaced by the product instead of having it subtracted (W <- W R^-1 with
// acol0 = ccol0, kdim = b, bmat = R^-1); overwrite = 2: the product is subtracted for the Gram matrix only, the block
// in memory stays as it is
hipError_t launch_update_gram(double* basis, int64_t n, int64_t ld, int acol0, int kdim, const double* bmat, int b,
                              int ccol0, int overwrite, double* gpart, hipStream_t st, const int* skip = nullptr);
// ---- Chebyshev filter with the iterates resident in LDS (resident.hip) -------------------------------
// A work item is a diagonal block (or a 16-column slice of it) worked on by lane groups of cl = 4 lanes (32 columns)
// or cl = 2 lanes (16 columns).  Its rows are cut into chunks of 8 cl entries; `extra` = chunks beyond the first,
// summed over its rows.  LDS bytes of an item, and the largest number of chunks (rows + extra) one may have:
constexpr int kItemInts = 5;
size_t resident_item_lds_bytes(int nrows, int cl, int extra);
int resident_max_chunks(int cl);
// Diagonal blocks of a CSR matrix with a symmetric pattern: starts[0 .. *count) = the rows p (ascending) such that no
// row before p has an entry in column p or beyond; starts has room for n entries, count is a device int32.
// work: device scratch of diagonal_blocks_workspace(n) bytes.  n <= INT32_MAX.
size_t diagonal_blocks_workspace(int64_t n);
hipError_t diagonal_blocks(const int64_t* rowptr, const int32_t* col, int64_t n, void* work, size_t work_bytes,
                           int32_t* starts, int32_t* count, hipStream_t st);
// extra[kBlockCounts t ..] (device int32) = extra chunks of block t for chunks of 32 and of 16 entries, the extra rows of the
// sliced form in pieces of sliced_piece() entries, the block's entries, and the least that its rows' first pieces take in the
// sliced form with their padding (both at most INT32_MAX)
constexpr int kBlockCounts = 5;
hipError_t launch_block_extra_chunks(const int64_t* rowptr, const int32_t* starts, int nblk, int64_t n, int32_t* extra,
                                     hipStream_t st);
// y (n x b, leading dimension ldy >= b) = the recurrence applied to x (packed n x b): u_0 = x, u_1 = alpha_first (A u_0 - shift u_0),
// u_{i+1} = alpha_rest (A u_i - shift u_i) - u_{i-1}; y = u_d.  A = the CSR matrix, whose rows [row0, row0 + nrows) of
// every item form a diagonal block.  items: device int32[kItemInts * nitems] = (row0, nrows, col0, cl | extra << 4, 0) per
// workgroup, covering columns [col0, col0 + 8 cl); every (block, column) pair must be covered exactly once, extra must
// be the block's extra-chunk count for chunks of 8 cl entries and nrows + extra <= resident_max_chunks(cl).
// lds_bytes = the largest resident_item_lds_bytes over the items.  y must not alias x.
// A sliced item (cl = sliced_shape(cols); the word's upper bits carry the item's first slot, the last word the block's extra rows)
// covers `cols` = 16, 8 or 4 columns of a block for which resident_sliced_lds_bytes is within the limit, and reads its entries from the
// sliced copy (scol, sval, slice_base, slice_len, slice_first, row_extra; null when no item is sliced) made for that many columns.
// d32 (0 <= d32 < d): the first d32 steps of the items with cl = 2 or 4 run in single precision (iterates and entries
// rounded to float), the rest in double; sliced items take all steps in double.  0 gives the recurrence in double.
// use_rnd != 0: x is not read; the operand is the random block of key rnd_key (random_block_key), entry by entry as
// launch_random_block would have written it into a packed n x b buffer.
// copies = 2 (use_rnd only): the same for the random block of key rnd_key2, whose result goes to the b columns behind y's.
hipError_t launch_cheb_resident(const int64_t* rowptr, const int32_t* col, const double* val, const double* x, double* y,
                                int64_t ldy, int b, int d, double alpha_first, double alpha_rest, double shift, const int32_t* items,
                                int nitems, size_t lds_bytes, const uint16_t* scol, const double* sval,
                                const int64_t* slice_base, const int32_t* slice_len, const int32_t* slice_first,
                                const int32_t* row_extra, hipStream_t st, int d32 = 0, uint64_t rnd_key = 0, int use_rnd = 0,
                                int copies = 1, uint64_t rnd_key2 = 0);
// key of random block number `stream_id` under `seed`: entry i * b + t of the block launch_random_block writes is
// 2 u - 1 with u the top 53 bits of mix(key + i * b + t)
uint64_t random_block_key(uint64_t seed, uint64_t stream_id);
// Sliced copy of diagonal blocks for the sliced form.  A block whose rows are cut into pieces has `extra` extra rows (the third
// count of launch_block_extra_chunks for pieces of sliced_piece() entries, 0 for pieces of INT32_MAX) and sliced_block_slots
// slots for slices; blocks: device, for every sliced block (first row, rows, place of its first extra row in a list for all
// blocks, extra rows, columns of its items, first slot, entries of a piece).  sliced_extra_rows
// makes that list and row_extra (int32[n]).  sliced_copy_layout fills, per slot, desc (sliced_desc_bytes of scratch),
// slice_len, slice_first, slice_entries (int64[nslots + 1]: entries the slice takes in the copy, padding included) and
// slice_base (int64[nslots + 1]: exclusive prefix sums; the last one is the size of the copy).  sliced_copy_fill writes the
// copy: scol (8-byte aligned) and sval (16-byte aligned) with room for slice_base[nslots] entries.
constexpr int kSliceBlockInts = 7;
int sliced_piece();
int sliced_shape(int cols);
size_t resident_sliced_lds_bytes(int nrows, int extra, int cols);
int sliced_block_slots(int nrows, int extra, int cols);
size_t sliced_desc_bytes(int nslots);
size_t sliced_scan_workspace(int nslots);
hipError_t sliced_extra_rows(const int64_t* rowptr, const int32_t* blocks, int nblocks, int32_t* list, int32_t* row_extra,
                             hipStream_t st);
hipError_t sliced_copy_layout(const int64_t* rowptr, const int32_t* blocks, int nblocks, const int32_t* list,
                              const int32_t* row_extra, int nslots, void* desc, int32_t* slice_len, int32_t* slice_first,
                              int64_t* slice_entries, int64_t* slice_base, void* work, size_t work_bytes, hipStream_t st);
hipError_t sliced_copy_fill(const int64_t* rowptr, const int32_t* col, const double* val, const void* desc,
                            const int32_t* list, const int32_t* row_extra, int nslots, const int64_t* slice_base,
                            const int64_t* slice_entries, uint16_t* scol, double* sval, hipStream_t st);

// Block steps of b random columns after which the check phase of a solve (driver.hip), whose largest Ritz value is theta, has
// shown but for a chance of 1e-20 that nothing above kappa is left, on n rows and for a spectrum in [-1, 1]; its block went
// through a filter of degree d on [lo, a] (d = 0: none).  2^30: never.
int check_steps_needed(double theta, double kappa, int d, double lo, double a, int64_t n, int b);

// Host part of the filter's plan alone (driver.hip), for tests: what a step is modelled to take, in seconds, for diagonal blocks of
// rows starts[t] .. starts[t + 1] with the counts of launch_block_extra_chunks and b = 16 or 32 columns in a filter of `steps`
// steps; *nitems = the work items.  Negative: there is no plan.
double resident_items_model(const int32_t* starts, const int32_t* counts, int nblk, int b, int64_t nnz, double steps,
                            int64_t lds_limit, int64_t* nitems);

// ---- connected components and locality reordering (setup) --------------------------------------
// Renumbering from the component labels (label[i] = smallest node index of i's component), on the device:
//   old_of_new[p] = original index of new row p (components contiguous, ordered by their smallest node; inside a
//   component by three levels of neighbourhood min-hash, ties in original order), new_of_old = its inverse,
//   rowptr_new (n+1) = row pointers of the permuted matrix, comp_of_new[p] = component index of new row p.
// work: device scratch of order_by_component_workspace(n) bytes.  All outputs are device arrays; n <= INT32_MAX.
size_t order_by_component_workspace(int64_t n);
// by_length != 0: on a graph with hubs (longest row > 3 average rows) the rows of a component are ordered by decreasing
// length first (for the wide sparse products), then by the min-hash levels.  big_rows > 0: the components with more
// nodes than that come after all the others (in the order of their smallest node among themselves).
hipError_t order_by_component(const int64_t* rowptr, const int32_t* col, const int32_t* label, int64_t n, int by_length,
                              int big_rows, void* work,
                              size_t work_bytes, int32_t* old_of_new, int32_t* new_of_old, int64_t* rowptr_new,
                              int32_t* comp_of_new, hipStream_t st);
// list[0 .. *count) = the rows with more than kLongRow entries, ascending; list has room for n entries; count: device
// int32.  work: device scratch of long_row_list_workspace(n) bytes.
size_t long_row_list_workspace(int64_t n);
hipError_t long_row_list(const int64_t* rowptr, int64_t n, void* work, size_t work_bytes, int32_t* list, int32_t* count,
                         hipStream_t st);
// label[i] = i
hipError_t launch_iota(int32_t* label, int64_t n, hipStream_t st);
// one round of minimum-label propagation with pointer jumping; *changed = 1 if a label moved
hipError_t launch_cc_round(const int64_t* rowptr, const int32_t* col, const double* val, int32_t* label, int64_t n,
                           const int* before, int* changed, hipStream_t st);
// permuted CSR: row p = input row old_of_new[p], column c renamed new_of_old[c]; rowptr_new precomputed
hipError_t launch_permute_csr(const int64_t* rowptr, const int32_t* col, const double* val, const int32_t* old_of_new,
                              const int32_t* new_of_old, const int64_t* rowptr_new, int32_t* col_new, double* val_new,
                              int64_t n, hipStream_t st);
// basis[i, col0 + t] = comp[i] == t ? coef[i] : 0  for t < ncols (closed-form null vectors of the components)
hipError_t launch_nullspace_fill(double* basis, int64_t n, int64_t ld, int col0, int ncols, const int32_t* comp,
                                 const double* coef, hipStream_t st);

// ---- misc ----------------------------------------------------------------------------------
// dst[i*ldd + dcol0 + t] -= src[i*lds + scol0 + t], t < w (regions must not overlap)
hipError_t launch_sub_cols(const double* src, int64_t lds, int scol0, double* dst, int64_t ldd, int dcol0, int w,
                           int64_t n, hipStream_t st);
// basis[i*ld + col] = v[rowmap ? rowmap[i] : i]
hipError_t launch_set_column(double* basis, int64_t n, int64_t ld, int col, const double* v, const int32_t* rowmap,
                             hipStream_t st);
// basis[i, col0 + t] = uniform(-1, 1) from a counter-based hash of (seed, stream_id, i, t)
hipError_t launch_random_block(double* basis, int64_t n, int64_t ld, int col0, int b, uint64_t seed,
                               uint64_t stream_id, hipStream_t st);
// dst[i*ldd + dcol0 + t] = src[i*lds + scol0 + t], t < w (regions must not overlap)
// out[pos[c]*n + o] = basis[r(o)*ld + c] for c < ncols with pos[c] >= 0 (pos: device int32[ncols], the output column
// of basis column c or -1; r(o) = inv[o], the internal row of original row o, if inv is given, else o); factor (may be
// null): row r of the basis is multiplied by factor[r] on the way
hipError_t launch_gather_cols_colmajor(const double* basis, int64_t n, int64_t ld, const int32_t* pos, int ncols,
                                       double* out, const int32_t* inv, const double* factor, hipStream_t st);
// factor[i] = 1 / 2-norm of the entries of row i that the gather copies (1 if they are all zero)
hipError_t launch_row_factor(const double* basis, int64_t n, int64_t ld, const int32_t* pos, int ncols, double* factor,
                             hipStream_t st);
// The solver's own operator copy for wide blocks (b = 8, 16, 32) holds S_ij = s_i W_ij s_j multiplied out:
// val_out[e] = s_i * val[e] * s_j (val_out may be val).
hipError_t launch_scale_values(const int64_t* rowptr, const int32_t* col, const double* val, const double* s,
                               double* val_out, int64_t n, hipStream_t st);
// y = A x with the values as stored (the scaled copy); x packed n x b (b = 8, 16, 32; 16-byte aligned), y row-major
// with leading dimension ldy.
// longrows (may be null): device list of the nlong rows with more than kLongRow entries, ascending (long_row_list);
// those rows are then computed by a workgroup each instead of a lane group.
hipError_t launch_spmm_vals(const int64_t* rowptr, const int32_t* col, const double* val, int64_t n, const double* x,
                            int b, double* y, int64_t ldy, double avg_deg, const int32_t* longrows, int nlong,
                            hipStream_t st);
// One Chebyshev recurrence step on packed blocks:  unext = alpha * (A ucur - shift * ucur) - beta * uprev
// (uprev is not read when beta == 0; unext must not be ucur).  row_begin > 0: only the rows [row_begin, n) are computed
// and written (the rows before it belong to a caller that computes them another way).
hipError_t launch_spmm_vals_cheb(const int64_t* rowptr, const int32_t* col, const double* val, int64_t n,
                                 const double* ucur, int b, const double* uprev, double* unext, double alpha,
                                 double shift, double beta, double avg_deg, const int32_t* longrows, int nlong,
                                 hipStream_t st, int64_t row_begin = 0);
// out[t*n + o] *= s[r(o)], t < k (column-major vectors in the caller's numbering; s in the internal numbering)
hipError_t launch_scale_rows_colmajor(double* out, int64_t n, int k, const double* s, const int32_t* inv, hipStream_t st);
// every row of the n x k column-major matrix scaled to unit 2-norm (zero rows stay zero)
hipError_t launch_normalize_rows_colmajor(double* out, int64_t n, int k, hipStream_t st);
// ynext = alpha (w - shift ycur) - beta yprev and znext = s o ynext on packed n x b blocks (Chebyshev recurrence step)
hipError_t launch_cheb_combine(const double* w, const double* ycur, const double* yprev, const double* s, double alpha,
                               double shift, double beta, double* ynext, double* znext, int64_t n, int b,
                               hipStream_t st);
hipError_t launch_copy_cols(const double* src, int64_t lds, int scol0, double* dst, int64_t ldd, int dcol0, int w,
                            int64_t n, hipStream_t st);

// ---- k-means on the embedding (Section IV-C, Algorithms 4-5; kmeans.hip) ------------------------
// x (n x ldx row-major, zero padded beyond d) from the caller's points (column-major v[t*ldv + i] or row-major)
hipError_t launch_points_to_rowmajor(const double* v, int64_t ldv, int colmajor, int64_t n, int d, double* x, int64_t ldx,
                                     hipStream_t st);
// The count of changed labels is the sum of kChangeSlots device ints, kChangeStride apart.
constexpr int kChangeSlots = 64, kChangeStride = 32, kChangeInts = kChangeSlots * kChangeStride;
// ct (dpad x ldc row-major) = transpose of the k x ldx centre array, cnorm[j] = |c_j|^2, changes = 0
hipError_t launch_centroid_operand(const double* c, int64_t ldx, int k, int d, int dpad, double* ct, int64_t ldc,
                                   double* cnorm, int* changes, hipStream_t st);
// label[i] = arg-min_j cnorm[j] - 2 (x ct)[i, j] (first on ties); changes += number of labels that changed.  x: 32-byte
// aligned, ldx % 4 == 0, zero padded; ct: ldx rows; work: label_workspace bytes
size_t label_workspace(int64_t n, int64_t ldx, int k);
hipError_t launch_label(const double* x, int64_t ldx, int64_t n, const double* ct, int64_t ldc, int k, const double* cnorm,
                        void* work, size_t work_bytes, int32_t* label, int* changes, hipStream_t st);
// the same for the points rows[0 .. *listed) (device) alone, *listed <= n
hipError_t launch_label_listed(const double* x, int64_t ldx, int64_t n, const int32_t* rows, const int* listed,
                               const double* ct, int64_t ldc, int k, const double* cnorm, int32_t* label, int* changes,
                               hipStream_t st);
// Labelling screened in bf16 (kmeans.hip): the same labels.  It pays from label_screen_steps labelling steps on (INT32_MAX:
// never); 0 bytes where it is not made.  launch_label_copy makes the
// reduced copy of the points, once (centring: ldx + 1 doubles, the points' mean and scale; centred: launch_kmeanspp has left them
// there for the same points, else they are made: 100,000 x 100 43 us); launch_label_screened does a labelling step and leaves the
// number of points that the screen could not decide, which were labelled in fp64, at changes[kChangeUndecided].
constexpr int kChangeUndecided = 1, kChangeSum = 2;
int label_screen_steps(int64_t n, int64_t ldx, int k);
size_t label_screen_workspace(int64_t n, int64_t ldx, int k);
hipError_t launch_label_copy(const double* x, int64_t ldx, int d, int64_t n, int k, void* work, double* centring, bool centred,
                             hipStream_t st);
hipError_t launch_label_screened(const double* x, int64_t ldx, int d, int64_t n, const double* c, const double* ct,
                                 int64_t ldc, int k, const double* cnorm, void* work, const double* centring, int32_t* label, int* changes,
                                 hipStream_t st);
hipError_t launch_fill_int32(int32_t* a, int64_t n, int32_t value, int use_iota, hipStream_t st);
// centres = means of their points (grouped by label, fixed summation order); empty clusters keep their centre.  ct, cnorm
// and changes as launch_centroid_operand would then make them.  work: kmeans_update_workspace(n, ldx, k) bytes; start:
// device int32[k+1] (first grouped position of every cluster).  The labelling's counts, which the caller decides by whether to
// go on, are in report.host (coherent host memory) once report.host[2] = report.number, long before the update is done: [0] labels
// changed, [1] points that the screen could not decide.  If no label has changed the centres come out as they are.
// which: the launch that reports, the ones behind it, or both.
constexpr int kUpdateReport = 1, kUpdateCentres = 2;
struct LabelReport {
  int* host;
  int number;
};
size_t kmeans_update_workspace(int64_t n, int64_t ldx, int k);
hipError_t launch_centroid_update(const double* x, int64_t ldx, int d, int64_t n, const int32_t* label, int k, void* work,
                                  size_t work_bytes, int32_t* start, double* c, double* ct, int64_t ldc, double* cnorm,
                                  int* changes, const LabelReport& report, int which, hipStream_t st);
// Algorithm 5, launch_kmeanspp below; chosen: device int32[k].  screen = 0: without the reduced copy of the points, which
// makes the draws faster and takes a quarter of their bytes.  centring: ldx + 1 doubles; *centred: whether the reduced copy has left
// there what launch_label_copy takes
size_t kmeans_seed_workspace(int64_t n, int64_t ldx, int d, int k, int screen);
// Uniform number `index` in [0, 1) of the seeding draws, made where it is used: top 53 bits of mix(key + index),
// key = seed_key(seed).
__host__ __device__ inline uint64_t seed_mix(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}
inline uint64_t seed_key(uint64_t seed) { return seed_mix(seed); }
__host__ __device__ inline double seed_uniform(uint64_t key, uint64_t index) {
  return (double)(seed_mix(key + index) >> 11) * (1.0 / 9007199254740992.0);
}
constexpr int kNeverFused = -2;
struct SeedFused {
  size_t lds_limit = 0;
  int polls = kNeverFused;  // as for launch_fused_step
  int groups = 0;           // out: workgroups of the one launch, 0: there is none
  int* done = nullptr;      // out: device, in work
};
hipError_t launch_kmeanspp(const double* x, int64_t ldx, int d, int64_t n, int k, uint64_t key, int screen, void* work,
                           size_t work_bytes, int32_t* chosen, double* centring, bool* centred, SeedFused& f, hipStream_t st);
hipError_t launch_gather_rows(const double* x, int64_t ldx, const int32_t* index, int k, double* c, hipStream_t st);
// part[p], p < kmeans_objective_parts(): partial sums of |x_i - c_label(i)|^2 (add them in order on the host); NaN for a
// point whose label is not in [0, k)
int kmeans_objective_parts();
hipError_t launch_objective(const double* x, int64_t ldx, int d, int64_t n, const int32_t* label, int k, const double* c,
                            double* part, hipStream_t st);
hipError_t launch_copy_rows(const double* src, int64_t lds, double* dst, int64_t ldd, int rows, int cols, hipStream_t st);

// ---- similarity graph (Section IV-A, Algorithm 1; Algorithm 2 step 4; similarity.hip) ----------------------------
// mean[i] = row mean (0 if centre == 0), norm[i] = 2-norm of the row minus that mean; x row-major n x ldx
hipError_t launch_row_stats(const double* x, int64_t ldx, int64_t n, int d, int centre, double* mean, double* norm,
                            hipStream_t st);
// measure 0 cross correlation, 1 cosine (both with mean/norm from launch_row_stats), 2 exp(-|xu-xv|^2 / (2 sigma^2));
// *bad |= 1 and val[e] = NaN for an edge with an index outside [0, n)
hipError_t launch_edge_similarity(const double* x, int64_t ldx, int d, const int32_t* eu, const int32_t* ev,
                                  int64_t nedges, int measure, double sigma, const double* mean, const double* norm,
                                  int64_t n, int* bad, double* val, hipStream_t st);
// The same through buckets of rows: 0 bytes of work where that does not pay.  nrest: device int, 0 on entry, the number of
// pairs that had no room in their bucket or an index out of range afterwards (they are done like the others).
size_t edge_buckets_workspace(int64_t n, int d, int64_t nedges);
hipError_t launch_edge_similarity_buckets(const double* x, int64_t ldx, int d, const int32_t* eu, const int32_t* ev,
                                          int64_t nedges, int measure, double sigma, const double* mean,
                                          const double* norm, int64_t n, void* work, size_t work_bytes, int* bad,
                                          int32_t* nrest, double* val, hipStream_t st);
// ---- k-nearest-neighbour graph (Section III-A; knn.hip) -------------------------------------------------------
// Exact Euclidean k nearest neighbours of every row of x (n x d, leading dimension ldx) other than the row itself:
// idx_out[i*k + a] / dist_out[i*k + a] = index / distance of the a-th nearest, nearest first, equal distances by
// index.  xp: device scratch of n * (knn_padded_dim(d) + 1) doubles, which launch_knn_pad fills with the rows, zero
// padded.  2 <= n <= INT32_MAX, 1 <= k <= n - 1, and knn_search_lds_bytes(d, k) must not exceed the LDS a workgroup may
// have (else hipErrorInvalidValue).
int knn_padded_dim(int d);
size_t knn_search_lds_bytes(int d, int k);
hipError_t launch_knn_pad(const double* x, int64_t ldx, int64_t n, int d, double* xp, hipStream_t st);
// The bf16 screen: bytes of scratch it needs, 0 where it is not used.  It leaves device pointers to a list of tiles of
// 64 queries that it could not settle, to their number and to an upper bound of every query's k-th squared distance;
// launch_knn_search does those (tiles, ntiles, bound), or every query when tiles is null (all that there is to do without
// the screen; bound may be null then).  host: kLostInts pinned ints that launches write to; the call waits for their words
// (once per round of queries, and up to twice more, once a round, where the points are grouped).
constexpr int kLostSlots = 64, kLostStride = 32, kLostInts = kLostSlots * kLostStride;
size_t knn_screen_workspace(int64_t n, int d, int k);
// Scratch of the screen's grouped form, which passes over the tiles of points that cannot hold a neighbour; 0 where it is
// not used.  group_work may be null: the screen then looks at every pair.  *grouped_out: whether it took the grouped form.
size_t knn_group_workspace(int64_t n, int d, int k);
hipError_t launch_knn_screen(const double* xp, int64_t n, int d, int k, void* work, void* group_work, int32_t* host,
                             int32_t** tiles, int32_t** ntiles, double** bound, bool* grouped_out, int32_t* idx_out,
                             double* dist_out, hipStream_t st);
hipError_t launch_knn_search(int64_t n, int d, int k, double* xp, const int32_t* tiles, int64_t ntiles,
                             const double* bound, int32_t* idx_out, double* dist_out, hipStream_t st);
// The undirected edges {i, j} (j in i's list or i in j's) once each as eu < ev, in row order of the emitting list;
// val = the listed distance, or exp(-dist^2 / (2 sigma^2)) if sigma > 0.  eu, ev, val have room for n * k entries;
// host (4 words of coherent host memory): host[1] + host[2] is the pair count once st is idle.  work: knn_pairs_workspace(n, k) bytes.
size_t knn_pairs_workspace(int64_t n, int k);
hipError_t launch_knn_union_pairs(const int32_t* idx, const double* dist, int64_t n, int k, double sigma, void* work,
                                  size_t work_bytes, int32_t* eu, int32_t* ev, double* val, int64_t* host,
                                  hipStream_t st);
size_t coo_to_csr_workspace(int64_t total, int64_t n, int radix);
hipError_t coo_to_csr(const int32_t* row, const int32_t* col, const double* val, int64_t nnz_in, int64_t n,
                      int symmetrize, int radix, void* work, size_t work_bytes, int64_t* rowptr_out, int32_t* col_out,
                      double* val_out, int* bad, hipStream_t st);

// Measurement aid: `workgroups` workgroups of four waves, each wave issuing iters * 8 fp64 matrix instructions and
// nothing else; shape 16: 16x16x4 (2,048 flops each), shape 4: 4x4x4 (512 flops each); sink: device, workgroups * 256
// doubles.
hipError_t launch_mfma_rate(double* sink, int shape, int workgroups, int iters, hipStream_t st);

}  // namespace sceig
