// Internal declarations shared by the HIP sources of liblilac.so.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <mutex>
#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "lilac.h"

namespace lilac {

// Row classes by row length.  C_W<n>: n lanes of a wavefront share one row
// (n = 1 is one lane per row, n = 64 a whole wavefront per row).  C_WG: one
// 256-lane workgroup per row.  C_SPLIT: the row is cut into chunks of
// `chunk` non-zeros, one workgroup per chunk, partial sums combined by a
// finaliser in chunk order.
enum RowClass : int32_t {
    C_W1 = 0, C_W2, C_W4, C_W8, C_W16, C_W32, C_W64, C_WG, C_SPLIT, NCLASS
};

constexpr int kBlock = 256;       // threads per workgroup (4 wave64)
constexpr int kWaves = kBlock / 64;
constexpr int kPad = 64;          // device arrays of nnz are padded to this
constexpr int kDotParts = 1024;   // partials of a standalone dot
// Partial sums of a solve: r.r and r.w, two parities each.
constexpr size_t kCgParts = 4 * kDotParts;
// Pieces of each vector in flight per thread: 2^26 float64 elements, 2, 4 and 8
// of them 163, 158 and 159 us (one element at a time 171; float32 145 -> 79).
constexpr int kDotAhead = 4;
// Vectors up to here take one workgroup and one launch: 16,000 float64 elements
// 10.1 -> 7.0 us a call; 40,000 by one workgroup 11.1 against 10.1.
constexpr int64_t kDotSmall = 16384;

// One unit of work of a product: `count` rows of class `cls`, taken from the
// class-ordered row list at `first` (for C_SPLIT: chunk index `first`).
// When the tile's rows are consecutive matrix rows, cls carries
// kTileContig and `first` is the first row itself.
constexpr int32_t kTileClassMask = 0xFF;
constexpr int32_t kTileContig = 0x100;
struct Tile {
    int32_t cls;
    int32_t mat;
    int32_t first;
    int32_t count;
};

// Everything a kernel needs to know about one matrix of a product.
struct MatDesc {
    const int32_t *row_ptr;
    const int32_t *col;
    const void *vals;
    const int32_t *bin_rows;  // rows ordered by class, ascending per class
    const int32_t *c_k0;      // chunk table: first non-zero of each chunk
    const int32_t *c_k1;      //              one past the last
    const int32_t *s_first;   // per split row: first chunk (nsplit+1 entries)
    const int32_t *c_row;     // chunk table: row of each chunk
    const void *x;
    void *y;
    const void *w;            // second operand of the fused dot (or null)
    double *chunk_part;       // one partial sum per chunk
    int32_t split_begin;      // position of the first split row in bin_rows
    int32_t nsplit;
    const Tile *tiles;        // the matrix's own tile list (segment launches)
    int32_t ntiles;
    int32_t pad;
};

enum EpiMode : int32_t { EPI_NONE = 0, EPI_PAGERANK = 1 };

// Epilogue applied when a row's sum s is stored:
//   EPI_NONE:      y = s
//   EPI_PAGERANK:  y = d * s + tele
struct Epi {
    int32_t mode;
    int32_t pad;
    double d;
    double tele;
};

struct Thresholds {
    int32_t upper[NCLASS];  // inclusive upper row length per class
};

// Per-matrix launch plan (row classes and tile shapes).
struct Plan {
    int32_t upper[NCLASS];
    int32_t rpg[NCLASS];    // rows per lane group per tile
    int32_t chunk;          // non-zeros per split-row chunk
    int32_t grid_per_cu;    // persistent workgroups per compute unit
    int32_t layout;         // LAYOUT_AUTO, _ROWS, _PANELS, _HOT or _BAND
};

// Device layouts of a matrix for the product: the row-class tiles over the
// CSR arrays, or column panels (x staged in LDS one panel at a time).
enum : int32_t { LAYOUT_AUTO = -1, LAYOUT_ROWS = 0, LAYOUT_PANELS = 1, LAYOUT_HOT = 2,
                 LAYOUT_BAND = 3 };

// Column-panel layout: the columns are cut into panels of `pw` (a panel of
// x fits the LDS), the rows into blocks of `rb`.  Within row block b and
// panel p the entries are stored row by row (each row's entries in their
// CSR order), with the row inside the block and the column inside the panel
// packed into 32 bits, (row << 16) | col.  Each of the sixteen wavefronts of
// a workgroup owns `rw` consecutive rows of the block; wptr[(b*np + p)*17 + w]
// is where wavefront w's entries of panel p start (entry 16: the end).
struct PanelDesc {
    const void *vals;
    const uint32_t *rc;
    const int32_t *wptr;
    int32_t rows, cols;
    int32_t pw, np, rb, nblk, rw;
    int32_t per;    // row blocks to a workgroup of a grouped launch (1, 2, 4)
    int32_t gper;   // the same where the groups of panels have a workgroup each (1, 2)
    // lane form (col0 != null; see below): vals, words and start
    const uint16_t *words;
    const uint8_t *start;
    const int32_t *col0;
    // the panels in ng groups of pg: a row's sum is the groups' sums added in
    // order, whether one workgroup forms them all or one each
    int32_t ng, pg;
};
// Lane form of the column-panel layout.  A run is what one wavefront holds of
// one (row block, panel): the entries of its rows in order, with a filler for
// every row without an entry between two that have one.  The run is cut into
// 64 equal pieces of K consecutive entries, one per lane, stored column by
// column: run q = (b * np + p) * 16 + wave holds the columns col0[q] ..
// col0[q + 1] (64 entries each), two together (entry j of lane l at column
// col0[q] + (j & ~1), place l * 2 + (j & 1)), an odd last one alone (place l).
// An entry is its value and a 16-bit word: its column in the panel, and
// kLaneEnd on the last entry of its row, the run's last row excepted (so a
// lane never steps past it).  Fillers and the padding of the last
// pieces have value 0 and column pw, where the LDS holds a zero.
// start[q * 64 + l]: row (from the wavefront's first) of the lane's first entry.
constexpr uint32_t kLaneEnd = 0x8000u;
constexpr int kLaneMaxWidth = 32752;           // panel columns: 15 bits, pw itself too
constexpr int kLanePairs = 3;                  // pairs of columns in flight
// Vectors of one matrix in a grouped panel launch.
// dot: when set (float64 only), the blocks also write the partial sums of
// x_i * y_i over their rows (square matrices), one per row block, the
// product's fused dot of the single-matrix launch.
struct PanelIO {
    const void *x;
    void *y;
    double *dot = nullptr;
};
constexpr int kPanelThreads = 1024;            // 16 wave64: one workgroup per CU
constexpr int kPanelWaves = kPanelThreads / 64;
constexpr int kPanelMaxRb = 4096;              // rows per block (sums in LDS)
constexpr int kPanelLds = 160 * 1024;          // LDS of one workgroup
constexpr int kPanelChunks = 2;                // 128-entry chunks in flight
constexpr int kPanelMaxPanels = 64;            // one lane per panel in the build
constexpr int kPanelRotateBlocks = 128;        // blocks from which panel order rotates
// LDS bytes of the row sums of a block of rb rows (the x panel follows)
constexpr int panel_sum_bytes(int rb)
{
    return (rb * 8 + 15) & ~15;
}
// widest panel (elements) for a value size and rb rows per block
constexpr int panel_width(int vsize, int rb)
{
    return (kPanelLds - panel_sum_bytes(rb)) / vsize;
}
// The row blocks to a workgroup of a grouped launch that holds `total` of them: a
// matrix's own number, but not so many that CUs are left idle (with four
// workgroups for each CU instead of one, 160 matrices 246 us, 239; 16: the same).
inline int32_t panel_per(const PanelDesc &pd, int64_t total, int32_t cu)
{
    int32_t per = pd.per;
    while (per > 1 && total < (int64_t)cu * per)
        per /= 2;
    return per;
}
// workgroups of a matrix in a grouped launch
inline int32_t panel_groups_of(const PanelDesc &pd) { return (pd.nblk + pd.per - 1) / pd.per; }
// the same for the lane form: 16 bytes for the zero after the panel
constexpr int lane_panel_width(int vsize, int rb)
{
    return (kPanelLds - panel_sum_bytes(rb) - 16) / vsize < kLaneMaxWidth
               ? (kPanelLds - panel_sum_bytes(rb) - 16) / vsize
               : kLaneMaxWidth;
}

// Hot-column layout, for matrices whose most referenced columns come first
// (a graph relabelled by decreasing out-degree).  Columns [0, hot) are
// copied into LDS once per workgroup; the others are read from x in global
// memory.  Rows are cut into blocks of at most kHotRows non-empty rows and
// about the same number of entries; block b holds rows [brow[b], brow[b+1])
// and the entries [bent[b], bent[b+1]), its hot entries first (up to
// bsplit[b]), then its cold ones, each part row by row.  A row's key is its
// number among the non-empty rows of its block (rmap[row]; kHotEmpty for an
// empty row), so empty rows take no row sum.  A hot entry's word packs the
// key and the column, (key << 16) | col; a cold entry's word is its column
// and key[] holds its key.
struct HotDesc {
    const void *vals;
    const uint32_t *rc;
    const uint16_t *key;
    const uint16_t *rmap;    // [rows]: key of the row, kHotEmpty if it has no entries
    const int32_t *brow;     // [nblk + 1]
    const int32_t *bent;     // [nblk + 1]
    const int32_t *bsplit;   // [nblk]
    const int32_t *gptr;     // [grid + 1]: workgroup g takes blocks gblk[gptr[g] .. gptr[g+1])
    const int32_t *gblk;     // [nblk]
    const int32_t *newid;    // [cols]: number of the caller's column, or null (the same)
    const int32_t *old;      // [hot]: the caller's columns of the hot ones
    const uint32_t *cold;    // [nnz]: with newid, the caller's columns of the cold entries
    int32_t rows, cols, nblk, hot, grid, pad;
};
constexpr int kHotRows = 1536;                        // non-empty rows per block
constexpr uint16_t kHotEmpty = 0xFFFF;                // rmap of an empty row
constexpr int kHotSpan = 16 * kHotRows;               // rows per block, empty ones too
constexpr int kHotLdsHead = 2 * kHotRows * 8 + 1024;  // hot and cold row sums + carries
// hot columns (elements) for a value size
constexpr int hot_width(int vsize)
{
    return ((kPanelLds - kHotLdsHead) / vsize) & ~63;
}

// Band layout, for matrices whose rows reach only nearby columns: the CSR
// order and values are kept, and each entry gets a 32-bit word
// (row inside its block << 16) | (column - cbase[b]).  Rows are cut into
// blocks of at most kBandRows rows, about the same number of entries, and
// a column span below 65536; block b holds rows [brow[b], brow[b+1]) and
// the entries [bent[b], bent[b+1]).
struct BandDesc {
    const void *vals;        // the CSR values
    const uint32_t *rc;      // [nnz + pad]
    const int32_t *brow;     // [nblk + 1]
    const int32_t *bent;     // [nblk + 1]
    const int32_t *cbase;    // [nblk]
    int32_t rows, cols, nblk;
    // sliced form (nslice > 0): vals, off and slice replace the arrays above
    int32_t nslice, spb;     // slices, slices per workgroup
    const int32_t *row_ptr;
    const uint16_t *off;
    const struct SellSlice *slice;   // [nslice]
};
// Sliced form of the band layout, for rows of nearly one length: rows are cut
// into slices of 64 (one lane each), a slice is as wide as its longest row,
// and its entries are stored column by column of the slice, so that the 64
// lanes read consecutive memory: four columns together, then a pair, then a
// single one, each lane's entries of a group side by side.  Entry j of lane
// l in a slice at column `at` of width w:
//   groups of four (j < w & ~3): column at + (j & ~3), place l * 4 + (j & 3)
//     (float64 values: two pairs, column at + (j & ~1), place l * 2 + (j & 1))
//   pair (w & 2): column at + (w & ~3), place l * 2 + (j & 1)
//   last (w & 1): column at + w - 1, place l
// A column holds 64 values and 64 16-bit column offsets from `base`.  Rows
// shorter than the slice are padded; lanes stop at their row's length.
struct SellSlice {
    int32_t at, base;        // first column, smallest column index
    int32_t wmin, wmax;      // shortest and longest row (wmin 0 in a short slice)
};
constexpr int kBandThreads = 256;
constexpr int kBandWaves = kBandThreads / 64;
constexpr int kBandRows = 2048;                            // rows per block
constexpr int kBandLds = kBandRows * 8 + kBandWaves * 12 + 16;

Plan default_plan();

struct CgState;      // device buffers + graph cache of a CG solve
struct PrState;      // graph cache of PageRank

enum : int32_t { kBuildAuto = 0, kBuildOnce = 1, kBuildHot = 2 };

struct CsrHandle {
    int32_t rows = 0, cols = 0;
    int32_t cols_given = -1;   // as passed at creation (-1: derived)
    int64_t nnz = 0;
    int32_t max_len = 0;         // longest row (set when constructed)
    lilac_dtype dt = LILAC_F64;
    unsigned flags = 0;
    // device copies
    int32_t *d_row_ptr = nullptr;
    int32_t *d_col = nullptr;
    void *d_vals = nullptr;
    // analysis
    int32_t *d_bin_rows = nullptr;
    int32_t *d_c_row = nullptr, *d_c_k0 = nullptr, *d_c_k1 = nullptr;
    int32_t *d_s_first = nullptr;
    double *d_chunk_part = nullptr;
    Tile *d_tiles = nullptr;
    double *d_dot_part = nullptr;   // one per persistent workgroup + finaliser
    // distinct 128-byte lines of x per non-zero in sampled groups of 64
    // rows (near 1: scattered columns; -1: not measured)
    double line_ratio = -1.0;
    double line_group = 0.0;     // distinct lines per sampled group
    // column-panel layout (when use_panels)
    bool use_panels = false;
    PanelDesc pan{};
    void *d_pv = nullptr;
    uint32_t *d_prc = nullptr;
    int32_t *d_pw = nullptr;
    int32_t *d_ppos = nullptr;      // places of each row's entries in each panel, or null
    int64_t lane_cols = 0;          // lane form: columns of 64 entries it holds
    // hot-column layout (when use_hot)
    bool use_hot = false;
    HotDesc hot{};
    void *d_hv = nullptr;           // values | words | keys | own columns | row keys
    uint32_t *d_hrc = nullptr;
    uint16_t *d_hkey = nullptr;
    uint16_t *d_hrmap = nullptr;    // rows: key of each row in its block
    int32_t *d_hb = nullptr;        // brow | bent | bsplit
    int32_t *d_hold = nullptr;      // renamed columns: newid | old
    uint32_t *d_hcold = nullptr;    // the caller's columns of the cold entries
    // band layout (when use_band)
    bool use_band = false;
    BandDesc band{};
    uint32_t *d_brc = nullptr;
    int32_t *d_bb = nullptr;        // brow | bent | cbase
    void *d_sv = nullptr;           // sliced form: values | offsets | slices
    uint16_t *d_so = nullptr;       // the offsets in it
    int64_t sell_cols = 0;          // columns of 64 entries it holds
    int32_t sell_wide = 0;          // longest row
    // working memory of the products (product_space), or null; space_done: the
    // end of the last one that uses it.  space_mu: from the wait for that event
    // to the launch that sets it again
    void *d_space = nullptr;
    hipEvent_t space_done = nullptr;
    mutable std::mutex space_mu;
    std::vector<int32_t> bin_off;   // NCLASS+1
    int64_t nchunks = 0;
    int32_t nsplit = 0;
    int32_t ntiles = 0;
    int32_t grid = 0;               // workgroups of the tile kernel
    int32_t fin_blocks = 0;         // workgroups of the finaliser
    Plan plan;
    int32_t build = 0;              // kBuildAuto, _Once or _Hot
    // remembered host arrays (LILAC_KEEP_HOST or raw-call cache)
    const int32_t *h_row_ptr = nullptr, *h_col = nullptr;
    const void *h_vals = nullptr;
    bool dirty_struct = false, dirty_vals = false;
    int64_t dev_bytes = 0;
    CgState *cg = nullptr;
    PrState *pr = nullptr;
};

size_t dtype_size(lilac_dtype dt);

// Whether the product runs on a layout of its own (column panels or hot
// columns) rather than on the row-class tiles.
inline bool own_layout(const CsrHandle &h)
{
    return h.use_panels || h.use_hot || h.use_band;
}

// ---- errors ---------------------------------------------------------------
struct Error {
    int code;
    std::string msg;
};
[[noreturn]] void fail(int code, const std::string &msg);
void hip_check(hipError_t e, const char *what, const char *file, int line);
#define HIPC(x) ::lilac::hip_check((x), #x, __FILE__, __LINE__)

// ---- device memory with a byte budget -----------------------------------
// Every device allocation of the library goes through dev_alloc, which
// charges it to the library-wide budget (LILAC_HBM_BUDGET) and, when the
// calling thread has an account set, to that account and each of its
// parents; an allocation that would take any of them past its limit fails
// with LILAC_ERR_BUDGET and allocates nothing.  dev_free returns the bytes
// to the accounts charged at allocation, whichever thread frees.  Accounts
// are read and changed only under lib_mutex().
struct Account {
    int64_t limit = INT64_MAX;
    int64_t in_use = 0;
    int64_t peak = 0;
    Account *parent = nullptr;
};
// The calling thread's current account (nullptr: none).
Account *&thread_account();
void *dev_alloc(size_t bytes);
void dev_free(void *p);

// Temporaries of a handle build (freed before the build returns).  A thread
// that installs a TmpCache takes them from one grow-only buffer of at most
// `limit` bytes, charged to `acct`, so that its builds call no hipFree
// (which waits for every stream of the device); without one, or for a
// larger or second temporary, they are ordinary allocations.
struct TmpCache {
    void *p = nullptr;
    size_t cap = 0, limit = 0;
    bool busy = false;
    Account *acct = nullptr;
};
TmpCache *&thread_tmp_cache();
void *tmp_alloc(size_t bytes);
void tmp_free(void *p);
void tmp_cache_release(TmpCache &t);   // frees the buffer
int device_cu_count();

// ---- kernel launchers (kernels.hip) --------------------------------------
void launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s);
void launch_fill_bytes_zero(void *p, int64_t bytes, hipStream_t s);
void launch_fill_f64(double *p, int64_t n, double v, hipStream_t s);
// HBM stream ceiling (read, or copy when dst is set) over bytes/16 pieces.
void launch_stream(const void *src, void *dst, int64_t bytes, int32_t groups,
                   uint32_t *sink, hipStream_t s);
void launch_validate(int32_t rows, const int32_t *rp, int64_t nnz,
                     const int32_t *col, int32_t cols_given, int32_t *status,
                     hipStream_t s);
void launch_bin_count(int32_t rows, const int32_t *rp, const Thresholds &th,
                      int32_t *hist, int32_t nblk, hipStream_t s);
// Exclusive prefix sum of a[0..n) in place; *total (if non-null) receives
// the sum.  Beyond 65536 elements it takes a temporary buffer and waits for
// the stream: analysis only, never inside a captured graph.
void launch_scan_excl(int32_t *a, int64_t n, int32_t *total, hipStream_t s);
void launch_bin_scatter(int32_t rows, const int32_t *rp, const Thresholds &th,
                        const int32_t *hist, int32_t nblk, int32_t *bin_rows,
                        hipStream_t s);
void launch_chunk_count(int32_t nsplit, const int32_t *split_rows,
                        const int32_t *rp, int32_t chunk, int32_t *cnt,
                        hipStream_t s);
void launch_chunk_fill(int32_t nsplit, const int32_t *split_rows,
                       const int32_t *rp, int32_t chunk, const int32_t *s_first,
                       int32_t *c_row, int32_t *c_k0, int32_t *c_k1,
                       hipStream_t s);

// Product over the tiles of one matrix (GROUPED = false, desc passed by
// value) or of many (desc table in device memory).  With dot_part non-null,
// workgroup g also writes dot_part[g] = sum over its rows of w[i]*y[i] and
// the finaliser writes dot_part[grid + b].
void launch_spmv_tiles(lilac_dtype dt, const Tile *tiles, int32_t ntiles,
                       int32_t grid, const MatDesc &single,
                       const MatDesc *mats, const Epi &epi, double *dot_part,
                       hipStream_t s);
// Column-panel product (see PanelDesc); dot_part (or null) receives one
// partial of sum w[i]*y[i] per workgroup.
void launch_spmv_panels(lilac_dtype dt, const PanelDesc &pd, const void *x,
                        void *y, const Epi &epi, const void *w, double *dot_part,
                        hipStream_t s);
// The lane form with a workgroup for each row block and group of panels: part
// (pd.ng * pd.rows doubles) receives the groups' sums, a second kernel adds
// them up.  Same results as launch_spmv_panels.  done (or null): an event for the
// last launch's end, here and in launch_spmv_hot.
void launch_spmv_lane_groups(lilac_dtype dt, const PanelDesc &pd, const void *x, void *y,
                             const Epi &epi, const void *w, double *dot_part, double *part,
                             hipStream_t s, hipEvent_t done);
void launch_panel_count(const PanelDesc &pd, const int32_t *rp,
                        const int32_t *col, int32_t *cnt, hipStream_t s);
void launch_panel_scatter(lilac_dtype dt, const PanelDesc &pd, const int32_t *rp,
                          const int32_t *col, const void *vals, const int32_t *ptr,
                          void *pv, uint32_t *prc, hipStream_t s);
// Lane form: row counts get the fillers (in place), kc[run] the columns of a
// run; then, with cnt and kc scanned, col0 = kc: padding, fillers and start
// rows of every run, and the entries.
void launch_lane_runs(const PanelDesc &pd, int32_t *cnt, int32_t *kc, hipStream_t s);
void launch_lane_fill(lilac_dtype dt, const PanelDesc &pd, const int32_t *pos, void *vals,
                      uint16_t *words, uint8_t *start, hipStream_t s);
void launch_lane_scatter(lilac_dtype dt, const PanelDesc &pd, const int32_t *rp,
                         const int32_t *col, const void *src, const int32_t *pos,
                         void *vals, uint16_t *words, hipStream_t s);
void launch_panel_wptr(const PanelDesc &pd, const int32_t *ptr, int32_t *wptr,
                       hipStream_t s);
// Column-panel products of nmat matrices in one launch of nblocks
// workgroups: matrix j owns workgroups [prefix[j], prefix[j+1]).  Each
// result equals the single-matrix launch bit for bit.
void launch_spmv_panels_grouped(lilac_dtype dt, const PanelDesc *descs,
                                const PanelIO *io, const int32_t *prefix,
                                int32_t nmat, int32_t nblocks, hipStream_t s);
// Band product (see BandDesc): one workgroup per row block; dot_part (or
// null) receives one partial per block.
void launch_spmv_band(lilac_dtype dt, const BandDesc &bd, const void *x, void *y,
                      const Epi &epi, const void *w, double *dot_part, hipStream_t s);
// Band products of nmat matrices in one launch (as for column panels).
void launch_spmv_band_grouped(lilac_dtype dt, const BandDesc *descs, const PanelIO *io,
                              const int32_t *prefix, int32_t nmat, int32_t nblocks,
                              hipStream_t s);
// lo[i], hi[i] = smallest and largest column of row i (INT_MAX, -1 if empty).
void launch_row_span(int32_t rows, const int32_t *rp, const int32_t *col, int32_t *lo,
                     int32_t *hi, hipStream_t s);
void launch_band_pack(const BandDesc &bd, const int32_t *rp, const int32_t *col,
                      uint32_t *rc, hipStream_t s);
// Per slice of 64 rows (see SellSlice): {smallest column, largest column,
// shortest row, longest row}; INT_MAX, -1 for a slice with no entries.
void launch_slice_span(int32_t rows, const int32_t *rp, const int32_t *col, int32_t nslice,
                       int32_t *out, hipStream_t s);
void launch_sell_pack(lilac_dtype dt, const BandDesc &bd, const int32_t *col,
                      const void *vals, void *sv, uint16_t *so, hipStream_t s);
// For ngroups groups of 64 consecutive rows spread over the matrix:
// out[2g] = non-zeros looked at (at most 8192), out[2g+1] = distinct
// (col >> shift) among them, hashed into 16384 bins.
void launch_line_reuse(int32_t rows, const int32_t *rp, const int32_t *col,
                       int32_t ngroups, int32_t shift, int32_t *out, hipStream_t s);
// Lets the panel kernels use the whole LDS of a CU (once per process).
void panels_prepare();
// Hot-column product (see HotDesc): hd.grid persistent workgroups take the
// row blocks in turn; dot_part (or null) receives one partial per workgroup.
// Where the layout renames columns (hd.old), xp (cols elements) receives x in
// its order first; without xp the kernel reads x as it is (same results).
void launch_spmv_hot(lilac_dtype dt, const HotDesc &hd, const void *x, void *y,
                     const Epi &epi, const void *w, double *dot_part, void *xp,
                     hipStream_t s, hipEvent_t done);
// cnt[r] = entries of row r with a column below hd.hot (as hd.newid numbers
// them).  list: the nlist rows of more than `most` entries.
void launch_hot_count(const HotDesc &hd, const int32_t *rp, const int32_t *col,
                      const int32_t *list, int32_t nlist, int32_t most, int32_t *cnt,
                      hipStream_t s);
// bsplit from the block bounds and the exclusive scan hx of the hot counts.
void launch_hot_split(const HotDesc &hd, const int32_t *hx, int32_t *bsplit,
                      hipStream_t s);
void launch_hot_scatter(lilac_dtype dt, const HotDesc &hd, const int32_t *rp,
                        const int32_t *col, const void *vals, const int32_t *list,
                        int32_t nlist, int32_t most, const int32_t *hx, void *hv, uint32_t *hrc,
                        uint16_t *hkey, uint32_t *hcold, hipStream_t s);
// out[0..rows]: 1 for a row with entries, else 0; row keys from its exclusive
// scan and the block bounds.
void launch_row_filled(int32_t rows, const int32_t *rp, int32_t *out, hipStream_t s);
// Block bounds by up to kHotTries rules of keys and entries at once: `cap` words for
// each of the parts of `part` rows, one rule after the other.
constexpr int kHotTries = 8;
struct HotTries {
    int32_t n, keys[kHotTries], target[kHotTries];
};
void launch_hot_blocks(int32_t rows, const int32_t *rp, const int32_t *filled, int32_t part,
                       const HotTries &tries, int32_t cap, int32_t *out, hipStream_t s);
void launch_hot_rmap(const HotDesc &hd, const int32_t *filled, uint16_t *rmap, hipStream_t s);
// *out += entries 0, step, 2 step, ... whose column has a newid below hot.
void launch_hot_share(int64_t nnz, int32_t step, const int32_t *col, const int32_t *newid,
                      int32_t hot, int32_t *out, hipStream_t s);
// flag[0..n]: 1 for a column with a newid below hot; from its exclusive scan, those
// columns renumbered in the caller's order, and the inverse of that.
void launch_hot_flag(int32_t n, const int32_t *newid, int32_t hot, int32_t *flag,
                     hipStream_t s);
void launch_hot_order(int32_t n, int32_t hot, const int32_t *before, int32_t *newid,
                      int32_t *old, hipStream_t s);
// Finaliser for split rows: single matrix (items == null, n = nsplit) or a
// list of (matrix, split row) items for grouped launches.
void launch_split_finalize(lilac_dtype dt, const int32_t *items, int32_t n,
                           const MatDesc &single, const MatDesc *mats,
                           const Epi &epi, double *dot_part, hipStream_t s);

// Product over several matrices whose own tile lists are concatenated
// virtually: tile v belongs to matrix j with prefix[j] <= v < prefix[j+1].
void launch_spmv_segments(lilac_dtype dt, const MatDesc *mats,
                          const int32_t *prefix, int32_t nseg, int32_t total,
                          int32_t grid, hipStream_t s);

// Many CG solves advanced together, one iteration per call sequence, in
// the Chronopoulos-Gear arrangement of the single-matrix solve: init once
// (x = 0, r = b, p = s = 0), then after each product w = A r the partial
// sums of r.w (rw) and one step that forms beta, alpha and updates
// p = r + beta p, s = w + beta s, x += alpha p, r -= alpha s.
struct CgSeg {
    const double *b;
    double *x, *r, *p, *w, *s;
    double *rw_part;    // nb partial sums of r.w
    double *rr_part;    // 2*nb partial sums of r.r (by iteration parity)
    double *sc;         // gamma[2], alpha[2] (by iteration parity)
    int32_t *done;      // set once the solve stopped (gamma or p.Ap zero)
    int64_t n;
    int32_t nb;         // workgroups of this solve (fixed by n)
    int32_t iter;       // iteration index k of this step
    int32_t blk0;       // first workgroup of this solve in the launch
    int32_t nrw;        // r.w partials the product wrote (0: k_cgb_rw writes nb)
};
int32_t cg_seg_blocks(int64_t n);
void launch_cgb_init(const CgSeg *segs, int32_t nseg, int32_t blocks, hipStream_t s);
void launch_cgb_rw(const CgSeg *segs, int32_t nseg, int32_t blocks, hipStream_t s);
void launch_cgb_step(const CgSeg *segs, int32_t nseg, int32_t blocks, hipStream_t s);

// *out = a . b (part: kDotParts doubles of scratch); a float32 result is the
// binary64 total rounded once.
template <typename T, typename TOut>
void launch_dot(int64_t n, const T *a, const T *b, double *part, TOut *out, hipStream_t s);

// Breadth-first search by Boolean products.  bits: three frontier bitmaps of
// `words` words (bfs_words of the rows), todo: a 64-bit word for each 64 rows,
// last: the deepest level given out so far.  A step gives level depth + 1 to
// every row without a level that has a column of level depth, and does nothing
// when no row has level depth; the report hands `last` to the host (pinned
// memory).  The nchunk chunks of the split rows and the nlong rows before the
// split ones in the class order hold every row of more than kBfsShort entries.
constexpr int kBfsThreads = 1024;
constexpr int32_t kBfsShort = 128;
inline int32_t bfs_words(int32_t rows)
{
    return (int32_t)((((int64_t)rows + 31) / 32 + 3) & ~(int64_t)3);   // 16-byte pieces
}
void launch_bfs_init(int32_t rows, int32_t source, const int32_t *rp, int32_t *level,
                     uint32_t *bits, int32_t words, uint64_t *todo, int32_t *last,
                     hipStream_t s);
void launch_bfs_step(const MatDesc &m, int32_t nchunk, int32_t nlong, int32_t rows,
                     int32_t *level, int32_t depth, uint32_t *bits, int32_t words,
                     uint64_t *todo, int32_t *last, hipStream_t s);
void launch_bfs_report(const int32_t *last, int32_t *host, hipStream_t s);

// Relabelling of a graph's vertices by decreasing out-degree (locality of the
// gathered vector): deg[u] = entries in column u (of every step-th); key = bucket of deg
// (powers of two, largest first); newid = stable position by key.
void launch_count_cols(int64_t nnz, int32_t step, const int32_t *col, int32_t *deg,
                       hipStream_t s);
void launch_degree_keys(int32_t n, const int32_t *deg, int32_t *key, hipStream_t s);
constexpr int kDegKeys = 33;
void launch_key_hist(int32_t n, const int32_t *key, int32_t *hist, int32_t nblk,
                     hipStream_t s);
void launch_key_scatter(int32_t n, const int32_t *key, const int32_t *hist,
                        int32_t nblk, int32_t *newid, hipStream_t s);
// Permuted copy: row newid[v] of the output is row v of the input with its
// columns renamed by newid (entries keep their order).
void launch_perm_lengths(int32_t rows, const int32_t *rp, const int32_t *newid,
                         int32_t *len2, hipStream_t s);
void launch_perm_entries(lilac_dtype dt, int32_t rows, int64_t nnz, const int32_t *rp,
                         const int32_t *col, const void *vals, const int32_t *newid,
                         const int32_t *rp2, int32_t *col2, void *vals2, hipStream_t s);
// out[newid[v]] = in[v] (to = true) or out[v] = in[newid[v]] (to = false)
void launch_permute_f32(int32_t n, const int32_t *newid, const float *in, float *out,
                        bool to, hipStream_t s);

// Jagged Diagonal Storage product, every sum in diagonal order without
// contraction (bitwise equal to the sequential definition).  The check inverts
// perm into iperm and sets bits of status[0] (0 before); the product stores
// nothing if any is set and copies status[0] to host_status (pinned).
void launch_jds_check(int32_t rows, int32_t max_len, const int32_t *perm,
                      const int32_t *jd_ptr, const int32_t *jd_col, int32_t *iperm,
                      int32_t *status, hipStream_t s);
void launch_spmv_jds(int32_t rows, int32_t max_len, const int32_t *perm,
                     const int32_t *iperm, const int32_t *nzcnt, const int32_t *jd_ptr,
                     const int32_t *jd_col, const double *jd_val, const double *x, double *y,
                     const int32_t *status, int32_t *host_status, hipStream_t s);
void launch_sum_parts(const double *part, int32_t nparts, double *out,
                      hipStream_t s);
// Bytes between device and pinned host memory, both 16-byte aligned and with
// room for whole 16-byte pieces.
void launch_copy_bytes(const void *src, void *dst, int64_t bytes, hipStream_t s);
void launch_copy_f32(int64_t n, const float *src, float *dst, hipStream_t s);

// CG building blocks (device scalars in `CgScalars`)
struct CgScalars {
    double rho;                 // r.r (of the final residual, or at the stop)
    double gamma[2], alpha[2];  // r.r and alpha of the last two iterations
    int32_t done, iters;
};
// A conjugate gradient solve is k_cg_init, then per iteration the product
// w = A r with the w.r partials fused into it and k_cg_step, then
// k_cg_final (see kernels.hip).  rr holds r.r partials for two parities
// (kDotParts each), so no partial is written by one workgroup while others
// read it.
void launch_cg_init(int64_t n, const double *b, double *x, double *r, double *p,
                    double *sv, double *rr, int32_t nparts, CgScalars *sc, hipStream_t s);
void launch_cg_step(int64_t n, CgScalars *sc, const double *w, double *p, double *sv,
                    double *x, double *r, const double *dot_part, int32_t ndot, double *rr,
                    int32_t nparts, int32_t k, hipStream_t s);
// Iteration k of a sliced band matrix, the step and the next product in one
// kernel: vectors by parity of the iteration, nrr partials of r.r and bd.nblk
// of r.w in, bd.nblk of each out (last: no product).
struct CgFused {
    double *r[2], *s[2], *w[2], *p, *x;
};
void launch_cg_sell(const BandDesc &bd, const CgFused &f, CgScalars *sc, const double *rr,
                    int32_t nrr, const double *rw, double *rr1, double *rw1, int32_t k,
                    bool last, hipStream_t s);
void launch_cg_final(CgScalars *sc, const double *rr, int32_t nparts, int32_t par,
                     hipStream_t s);
int32_t blas1_parts(int64_t n);
// Workgroups of the tile kernel resident per compute unit.
int occupancy_tiles(lilac_dtype dt);
bool is_device_ptr(const void *p);

// ---- runtime services shared with the request server ----------------------
std::recursive_mutex &lib_mutex();
void set_last_error(const std::string &msg);
int lib_device();
// build: kBuildOnce for a handle of one product (no renamed columns: they take
// many products to pay for), kBuildHot for the hot-column layout whatever is tuned.
// inputs_ready: device inputs are complete (the caller synchronised the
// stream that wrote them), so no device-wide wait is needed.
CsrHandle *create_handle(int rows, int cols, int64_t nnz, const int32_t *rp,
                         const int32_t *col, const void *vals, lilac_dtype dt,
                         unsigned flags, bool inputs_ready = false,
                         int32_t build = kBuildAuto);
// A handle that takes over device arrays allocated with dev_alloc and
// already holding the matrix: rp[rows+1], col and vals with room for
// padded_nnz(nnz) entries.  They belong to the handle from the call on
// (freed with it, also when the call fails).  Blocking.
int64_t padded_nnz(int64_t nnz);
// The checks and the analysis run on stream s (null: the library's stream).
CsrHandle *create_handle_adopt(int rows, int cols, int64_t nnz, int32_t *rp,
                               int32_t *col, void *vals, lilac_dtype dt,
                               hipStream_t s = nullptr);
void destroy_handle(CsrHandle *h);
MatDesc make_desc(const CsrHandle &h, const void *x, void *y, const void *w,
                  double *chunk_part);
// part: space for the product (see product_space), or null to take the
// handle's own.  done: an event for the end of a product that uses it.
void spmv_enqueue(const CsrHandle &h, const void *x, void *y, const Epi &epi,
                  const void *w, bool dot, hipStream_t s, void *part = nullptr,
                  hipEvent_t done = nullptr);
void run_cg(CsrHandle &h, const double *b, double *x, int iters,
            unsigned flags, hipStream_t s, double *rho_out, int *iters_done);
// Allocates the handle's CG state now (otherwise done on the first solve).
void handle_cg_prepare(CsrHandle &h);
int tile_grid(lilac_dtype dt);   // persistent workgroups for a grouped launch

// ---- CSR -> JDS (jds.hip) ---------------------------------------------------
// Longest row of the handle's matrix (d_tmp: one device int of scratch).
// Blocking.
int32_t jds_max_len(const CsrHandle &h, int32_t *d_tmp, hipStream_t s);
// The JDS arrays of the handle's matrix into device outputs perm[rows],
// nzcnt[rows], jd_ptr[max_len+1], jd_col[nnz], jd_val[nnz] (handle's dtype).
// Blocking.
void jds_convert(const CsrHandle &h, int32_t max_len, int32_t *perm, int32_t *nzcnt,
                 int32_t *jd_ptr, int32_t *jd_col, void *jd_val, hipStream_t s);

}  // namespace lilac
