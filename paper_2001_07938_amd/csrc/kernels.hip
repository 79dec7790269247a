// Device code of liblilac.so for gfx950 (CDNA4, wave64): CSR analysis and
// the layout builds, the CSR product in its four storage layouts (row-class
// tiles with the split-row finaliser, column panels, hot columns, band) and
// their grouped launches, dot products, the conjugate-gradient vector
// kernels (single and batched), PageRank relabelling, JDS and BFS.
//
// Every reduction here has a fixed shape (lane groups reduce with DPP moves
// in a fixed pattern, segmented scans run over lanes in order, workgroups
// combine their wavefronts in index order, split rows add their chunk sums
// in chunk order, carries between wavefronts are added in slot order, and a
// row sum held in LDS takes its additions from the one wavefront that owns
// the row, whose LDS operations complete in program order), so a given
// matrix, layout and plan always give bitwise identical results, whatever
// else runs on the GPU.
#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>

#include "lilac_internal.h"

namespace lilac {
namespace {

// Streaming loads for data read exactly once per product (vals, col_idx):
// non-temporal, so they do not push the gathered vector out of the caches.
template <typename T>
__device__ __forceinline__ T ld_stream(const T *p)
{
    return __builtin_nontemporal_load((const __attribute__((address_space(1))) T *)p);
}

// Loads and stores of device memory through a global (address space 1)
// pointer.  Pointers read from a descriptor table (grouped launches) are
// otherwise generic to the compiler, which then emits flat instructions;
// those also count against the LDS wait counter and so stall LDS work.
template <typename T>
__device__ __forceinline__ T gld(const T *p)
{
    return *(const __attribute__((address_space(1))) T *)p;
}

template <typename T>
__device__ __forceinline__ void gst(T *p, T v)
{
    *(__attribute__((address_space(1))) T *)p = v;
}

// Set bits of a wavefront mask in the lanes below this one.
__device__ __forceinline__ int32_t lanes_below(uint64_t m)
{
    return (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ int32_t wave_sum_i32(int32_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}

// Cross-lane move of a double with a DPP pattern (two 32-bit halves); a
// lane with no source lane gets 0 (bound_ctrl), so no old value has to be
// set up first.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const int lo = __double2loint(v);
    const int hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, CTRL, 0xF, 0xF, true),
                            __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xF, 0xF, true));
}

// The same for a 32-bit integer.
template <int CTRL>
__device__ __forceinline__ int32_t dpp_i32z(int32_t v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}

// DPP move with a row mask; lanes of masked rows (or with no source) get
// `old`.
template <int CTRL, int ROWS>
__device__ __forceinline__ int32_t dpp_i32(int32_t v, int32_t old)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xF, false);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64m(double v, double old)
{
    return __hiloint2double(
        __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), CTRL, ROWS, 0xF, false),
        __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), CTRL, ROWS, 0xF, false));
}

// One step of a segmented inclusive scan over a wavefront whose keys
// ascend along the lanes: add the partial of the source lane when it has
// the same key (monotone keys: the whole span between has that key).
// Shifts inside rows (all rows enabled) read 0 and key 0 where there is no
// source lane: a false key match then adds 0.  Broadcasts into some rows
// keep the lane's own key -1 / value 0 in the other rows.
// MASKED: the addition runs under an execution mask (the empty asm keeps
// the compiler from turning it into a select), one vector instruction
// instead of an addition and two 32-bit selects; it pays in the
// column-panel product, whose instruction stream bounds it.
template <int CTRL, int ROWS, bool MASKED = false>
__device__ __forceinline__ void seg_step(double &val, int32_t key)
{
    double t;
    int32_t tk;
    if (ROWS == 0xF) {
        t = dpp_f64<CTRL>(val);
        tk = dpp_i32z<CTRL>(key);
    } else {
        t = dpp_f64m<CTRL, ROWS>(val, 0.0);
        tk = dpp_i32<CTRL, ROWS>(key, -1);
    }
    if (tk == key) {
        val += t;
        if (MASKED)
            __asm__ volatile("" : "+v"(val));
    }
}

// acc += v on a double in LDS, no value returned (ds_add_f64: the wave
// does not wait for it).
__device__ __forceinline__ void lds_add_f64(double *acc, double v)
{
    (void)__hip_atomic_fetch_add(acc, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Segmented inclusive scan by key over the 64 lanes (keys ascending): row
// shifts by 1, 2, 4, 8 inside each row of 16, then the last lane of row 0
// (and of row 2) into rows 1 (and 3), then lane 31 into rows 2 and 3.
template <bool MASKED = false>
__device__ __forceinline__ double seg_scan64(double val, int32_t key)
{
    seg_step<0x111, 0xF, MASKED>(val, key);  // row_shr:1
    seg_step<0x112, 0xF, MASKED>(val, key);  // row_shr:2
    seg_step<0x114, 0xF, MASKED>(val, key);  // row_shr:4
    seg_step<0x118, 0xF, MASKED>(val, key);  // row_shr:8
    seg_step<0x142, 0xA, MASKED>(val, key);  // row_bcast:15 into rows 1 and 3
    seg_step<0x143, 0xC, MASKED>(val, key);  // row_bcast:31 into rows 2 and 3
    return val;
}

// Key of the next lane (wave_shl:1); the last lane gets -1.
__device__ __forceinline__ int32_t next_lane_key(int32_t key)
{
    return __builtin_amdgcn_update_dpp(-1, key, 0x130, 0xF, 0xF, false);
}

__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum over aligned groups of W lanes (W a power of two <= 64).  Inside a
// row of 16 lanes: neighbours (quad_perm 1,0,3,2), pairs (2,3,0,1), then the
// half-row and row mirrors, each adding the partner's partial; across rows
// the four row sums are read as uniform values and added in lane order.
// All lanes of a group end with the same value (x + y == y + x bitwise).
template <int W>
__device__ __forceinline__ double lane_group_sum(double v)
{
    if (W >= 2)
        v += dpp_f64<0xB1>(v);
    if (W >= 4)
        v += dpp_f64<0x4E>(v);
    if (W >= 8)
        v += dpp_f64<0x141>(v);
    if (W >= 16)
        v += dpp_f64<0x140>(v);
    if (W >= 32) {
        const double r0 = readlane_f64(v, 0), r1 = readlane_f64(v, 16);
        const double r2 = readlane_f64(v, 32), r3 = readlane_f64(v, 48);
        if (W == 32)
            v = (threadIdx.x & 32) ? r2 + r3 : r0 + r1;
        else
            v = (r0 + r1) + (r2 + r3);
    }
    return v;
}

template <int W>
__device__ __forceinline__ int32_t lane_group_or(int32_t v)
{
#pragma unroll
    for (int off = W / 2; off >= 1; off >>= 1)
        v |= __shfl_xor(v, off, 64);
    return v;
}

template <int W>
__device__ __forceinline__ int32_t lane_group_max(int32_t v)
{
#pragma unroll
    for (int off = W / 2; off >= 1; off >>= 1)
        v = max(v, __shfl_xor(v, off, 64));
    return v;
}

// Sum over a workgroup of NW wavefronts; every thread must call it and every
// thread receives the total.  lds holds NW doubles.
template <int NW>
__device__ __forceinline__ double block_sum(double v, double *lds)
{
    v = lane_group_sum<64>(v);
    __syncthreads();  // earlier readers of lds are done
    if ((threadIdx.x & 63) == 0)
        lds[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = lds[0];
#pragma unroll
    for (int i = 1; i < NW; ++i)
        t += lds[i];
    return t;
}

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));

// VEC consecutive values / column indices in one 16-byte (8-byte for the
// float64 indices) streaming load.  `p` is VEC-element aligned.
template <typename V, int VEC> struct Lanes;
template <typename V> struct Lanes<V, 1> {
    V v[1];
    int32_t c[1];
    __device__ __forceinline__ void load(const V *vp, const int32_t *cp)
    {
        v[0] = ld_stream(vp);
        c[0] = ld_stream(cp);
    }
};
template <> struct Lanes<double, 2> {
    double v[2];
    int32_t c[2];
    __device__ __forceinline__ void load(const double *vp, const int32_t *cp)
    {
        const f64x2 a = ld_stream((const f64x2 *)vp);
        const i32x2 b = ld_stream((const i32x2 *)cp);
        v[0] = a.x;
        v[1] = a.y;
        c[0] = b.x;
        c[1] = b.y;
    }
};
template <> struct Lanes<float, 4> {
    float v[4];
    int32_t c[4];
    __device__ __forceinline__ void load(const float *vp, const int32_t *cp)
    {
        const f32x4 a = ld_stream((const f32x4 *)vp);
        const i32x4 b = ld_stream((const i32x4 *)cp);
        v[0] = a.x;
        v[1] = a.y;
        v[2] = a.z;
        v[3] = a.w;
        c[0] = b.x;
        c[1] = b.y;
        c[2] = b.z;
        c[3] = b.w;
    }
};

// One lane's share of sum_{k in [k0,k1)} vals[k] * x[col[k]] when W lanes
// split the range.  The range is walked in passes over an aligned window
// starting at k0 rounded down to VEC: in a pass, lane l loads the VEC-element
// vectors at base + (j*W + l)*VEC for j < U, all issued before any is used
// (so U*VEC elements per lane are in flight), then gathers x for the
// elements that belong to the row.  Elements of a loaded vector outside
// [k0, k1) belong to neighbouring rows (or the array padding) and are
// skipped.  Products are formed and accumulated in binary64 (float32 data is
// widened exactly), in the order j, then element within the vector.
template <typename V, int W, int VEC, int U>
__device__ __forceinline__ double row_partial(const int32_t *__restrict__ col,
                                              const V *__restrict__ vals,
                                              const V *__restrict__ x,
                                              int32_t k0, int32_t k1, int lane)
{
    double acc = 0.0;
    const int32_t kb = k0 & ~(VEC - 1);
    for (int32_t base = kb; base < k1; base += U * W * VEC) {
        // every load is issued unconditionally (vectors past the row end
        // re-read the first one), so all U loads are in flight together
        Lanes<V, VEC> d[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int32_t e0 = base + (j * W + lane) * VEC;
            const int32_t ea = (e0 < k1) ? e0 : kb;
            d[j].load(vals + ea, col + ea);
        }
        // column indices of loaded vectors are all valid (real entries of
        // some row or the zero padding), so the gathers need no guard
        double xv[U][VEC];
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int t = 0; t < VEC; ++t)
                xv[j][t] = (double)gld(x + d[j].c[t]);
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int t = 0; t < VEC; ++t) {
                const int32_t e = base + (j * W + lane) * VEC + t;
                if (e >= k0 && e < k1)
                    acc = fma((double)d[j].v[t], xv[j][t], acc);
            }
    }
    return acc;
}

// Vector width used by a class: 16-byte value loads for groups of 8 lanes
// or more, single elements for narrower groups (rows of a few non-zeros).
template <typename V, int W>
struct VecOf {
    static constexpr int value = (W >= 8) ? (int)(16 / sizeof(V)) : 1;
};
constexpr int kUnroll = 2;

template <typename V>
__device__ __forceinline__ V epilogue(double s, const Epi &e)
{
    if (e.mode == EPI_PAGERANK)
        s = e.d * s + e.tele;
    return (V)s;
}

// Row number of position p of a tile: contiguous tiles store the first row
// itself, others index the class-ordered row list.
__device__ __forceinline__ int32_t tile_row(const MatDesc &m, const Tile &t,
                                            int32_t p)
{
    return (t.cls & kTileContig) ? t.first + p : gld(m.bin_rows + t.first + p);
}

// Rows of a tile, W lanes per row (W <= 64).  Group g of the workgroup takes
// rows g, g+G, g+2G, ... of the tile, so consecutive groups read consecutive
// rows.  Each wavefront first loads the row numbers and bounds of all the
// rows its groups will handle (one lane per row) and hands them to the
// groups with lane shuffles, so no row waits on its own pointer loads.
template <typename V, int W, bool DOT>
__device__ __forceinline__ void rows_by_lanes(const MatDesc &m, const Tile &t,
                                              const Epi &epi, double &dacc)
{
    constexpr int G = kBlock / W;   // groups per workgroup
    constexpr int GPW = 64 / W;     // groups per wavefront
    const int wave = threadIdx.x >> 6;
    const int wl = threadIdx.x & 63;
    const int q = wl / W;           // group within the wavefront
    const int lane = wl % W;
    const int g = wave * GPW + q;
    const V *vals = (const V *)m.vals;
    const V *x = (const V *)m.x;
    V *y = (V *)m.y;
    const int32_t count = t.count;
    // prefetch: lane wl holds row i_p*G + wave*GPW + (wl % GPW)
    const int32_t jp = (wl / GPW) * G + wave * GPW + (wl % GPW);
    int32_t pr = 0, pk0 = 0, pk1 = 0;
    if (jp < count) {
        pr = tile_row(m, t, jp);
        pk0 = gld(m.row_ptr + pr);
        pk1 = gld(m.row_ptr + pr + 1);
    }
    const int32_t g0 = wave * GPW;
    const int32_t iters = (count > g0) ? (count - g0 + G - 1) / G : 0;
    for (int32_t i = 0; i < iters; ++i) {
        const int src = i * GPW + q;
        const int32_t row = __shfl(pr, src, 64);
        const int32_t k0 = __shfl(pk0, src, 64);
        const int32_t k1 = __shfl(pk1, src, 64);
        if (g + i * G < count) {
            const double s = lane_group_sum<W>(
                row_partial<V, W, VecOf<V, W>::value, kUnroll>(m.col, vals, x,
                                                                k0, k1, lane));
            if (lane == 0) {
                const V out = epilogue<V>(s, epi);
                gst(y + row, out);
                if (DOT)
                    dacc = fma((double)gld((const V *)m.w + row), (double)out, dacc);
            }
        }
    }
}

// Rows of a tile, one whole workgroup per row.
template <typename V, bool DOT>
__device__ __forceinline__ void rows_by_block(const MatDesc &m, const Tile &t,
                                              const Epi &epi, double &dacc,
                                              double *lds)
{
    const V *vals = (const V *)m.vals;
    const V *x = (const V *)m.x;
    V *y = (V *)m.y;
    for (int j = 0; j < t.count; ++j) {
        const int32_t row = tile_row(m, t, j);
        const int32_t k0 = gld(m.row_ptr + row);
        const int32_t k1 = gld(m.row_ptr + row + 1);
        const double s = block_sum<kWaves>(
            row_partial<V, kBlock, VecOf<V, kBlock>::value, kUnroll>(
                m.col, vals, x, k0, k1, threadIdx.x),
            lds);
        if (threadIdx.x == 0) {
            const V out = epilogue<V>(s, epi);
            gst(y + row, out);
            if (DOT)
                dacc = fma((double)gld((const V *)m.w + row), (double)out, dacc);
        }
    }
}

// One chunk of a split row: the workgroup's sum goes to chunk_part.
template <typename V>
__device__ __forceinline__ void split_chunk(const MatDesc &m, const Tile &t,
                                            double *lds)
{
    const int32_t c = t.first;
    const int32_t k0 = gld(m.c_k0 + c);
    const int32_t k1 = gld(m.c_k1 + c);
    const double s = block_sum<kWaves>(
        row_partial<V, kBlock, VecOf<V, kBlock>::value, kUnroll>(
            m.col, (const V *)m.vals, (const V *)m.x, k0, k1, threadIdx.x),
        lds);
    if (threadIdx.x == 0)
        gst(m.chunk_part + c, s);
}

// Persistent tile loop: workgroup b takes tiles b, b+grid, b+2*grid, ...
// (a static assignment, so the optional fused dot is summed in a fixed
// order).  Tiles are ordered longest work first.
template <typename V, bool GROUPED, bool DOT>
__global__ __launch_bounds__(kBlock) void k_spmv_tiles(
    const Tile *__restrict__ tiles, int32_t ntiles, MatDesc single,
    const MatDesc *__restrict__ mats, Epi epi, double *__restrict__ dot_part)
{
    __shared__ double lds[kWaves];
    double dacc = 0.0;
    for (int32_t ti = blockIdx.x; ti < ntiles; ti += gridDim.x) {
        const Tile t = tiles[ti];
        const MatDesc m = GROUPED ? mats[t.mat] : single;
        switch (t.cls & kTileClassMask) {
        case C_W1: rows_by_lanes<V, 1, DOT>(m, t, epi, dacc); break;
        case C_W2: rows_by_lanes<V, 2, DOT>(m, t, epi, dacc); break;
        case C_W4: rows_by_lanes<V, 4, DOT>(m, t, epi, dacc); break;
        case C_W8: rows_by_lanes<V, 8, DOT>(m, t, epi, dacc); break;
        case C_W16: rows_by_lanes<V, 16, DOT>(m, t, epi, dacc); break;
        case C_W32: rows_by_lanes<V, 32, DOT>(m, t, epi, dacc); break;
        case C_W64: rows_by_lanes<V, 64, DOT>(m, t, epi, dacc); break;
        case C_WG: rows_by_block<V, DOT>(m, t, epi, dacc, lds); break;
        default: split_chunk<V>(m, t, lds); break;
        }
    }
    if (DOT) {
        const double tot = block_sum<kWaves>(dacc, lds);
        if (threadIdx.x == 0)
            dot_part[blockIdx.x] = tot;
    }
}

// Split rows: add the chunk sums of each split row in chunk order, apply the
// epilogue and store.  One thread per split row.
template <typename V, bool GROUPED, bool DOT>
__global__ __launch_bounds__(kBlock) void k_split_finalize(
    const int32_t *__restrict__ items, int32_t n, MatDesc single,
    const MatDesc *__restrict__ mats, Epi epi, double *__restrict__ dot_part)
{
    __shared__ double lds[kWaves];
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    double dacc = 0.0;
    if (i < n) {
        const int32_t mi = GROUPED ? items[2 * i] : 0;
        const int32_t j = GROUPED ? items[2 * i + 1] : i;
        const MatDesc m = GROUPED ? mats[mi] : single;
        const int32_t row = m.bin_rows[m.split_begin + j];
        double s = 0.0;
        for (int32_t c = m.s_first[j]; c < m.s_first[j + 1]; ++c)
            s += m.chunk_part[c];
        const V out = epilogue<V>(s, epi);
        ((V *)m.y)[row] = out;
        if (DOT)
            dacc = (double)((const V *)m.w)[row] * (double)out;
    }
    if (DOT) {
        const double tot = block_sum<kWaves>(dacc, lds);
        if (threadIdx.x == 0)
            dot_part[blockIdx.x] = tot;
    }
}

// Several matrices in one launch, each with its own tile list; workgroup b
// takes virtual tiles b, b+grid, ...; virtual tile v is tile v - prefix[j]
// of matrix j (binary search over the prefix).
template <typename V>
__global__ __launch_bounds__(kBlock) void k_spmv_segments(
    const MatDesc *__restrict__ mats, const int32_t *__restrict__ prefix,
    int32_t nseg, int32_t total)
{
    __shared__ double lds[kWaves];
    const Epi epi{EPI_NONE, 0, 0.0, 0.0};
    double dacc = 0.0;
    for (int32_t v = blockIdx.x; v < total; v += gridDim.x) {
        int32_t lo = 0, hi = nseg;
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (prefix[mid] <= v)
                lo = mid;
            else
                hi = mid;
        }
        const MatDesc m = mats[lo];
        const i32x4 tv = gld((const i32x4 *)(m.tiles + (v - prefix[lo])));
        const Tile t{tv.x, tv.y, tv.z, tv.w};
        switch (t.cls & kTileClassMask) {
        case C_W1: rows_by_lanes<V, 1, false>(m, t, epi, dacc); break;
        case C_W2: rows_by_lanes<V, 2, false>(m, t, epi, dacc); break;
        case C_W4: rows_by_lanes<V, 4, false>(m, t, epi, dacc); break;
        case C_W8: rows_by_lanes<V, 8, false>(m, t, epi, dacc); break;
        case C_W16: rows_by_lanes<V, 16, false>(m, t, epi, dacc); break;
        case C_W32: rows_by_lanes<V, 32, false>(m, t, epi, dacc); break;
        case C_W64: rows_by_lanes<V, 64, false>(m, t, epi, dacc); break;
        case C_WG: rows_by_block<V, false>(m, t, epi, dacc, lds); break;
        default: split_chunk<V>(m, t, lds); break;
        }
    }
}

// ------------------------------------------------------- column panels

// Product over the column-panel layout.  Workgroup b (one per CU, 16
// wavefronts) owns row block b; for each panel it copies that slice of x into
// LDS, and each wavefront streams its own entries of the panel in coalesced
// chunks: lane j forms vals[k] * x[col] from LDS for two consecutive
// entries, a segmented scan over the lanes (rows ascend along the chunk) adds
// up each row's run, and the last lane of a run adds it to the row's sum in
// LDS.  Rows belong to one wavefront, chunks follow in order, panels follow
// in an order fixed for the block: the additions are in a fixed order given
// by the matrix and the layout.
template <typename V, bool DOT>
__device__ __forceinline__ void panel_block(const PanelDesc &pd, int32_t b,
                                            const V *__restrict__ x,
                                            V *__restrict__ y, const Epi &epi,
                                            const V *__restrict__ w,
                                            double *__restrict__ dot_part,
                                            unsigned char *smem)
{
    double *acc = (double *)smem;                                 // row sums
    V *xs = (V *)(smem + panel_sum_bytes(pd.rb));                 // x panel
    constexpr int VV = 16 / sizeof(V);
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int32_t r0 = b * pd.rb;
    const int32_t nr = min(pd.rb, pd.rows - r0);
    const V *pv = (const V *)pd.vals;
    for (int i = threadIdx.x; i < pd.rb; i += kPanelThreads)
        acc[i] = 0.0;
    // the dot operand of this thread's row (rows <= threads), read now so
    // the epilogue does not wait for it
    double wrow = 0.0;
    if (DOT && (int32_t)threadIdx.x < nr)
        wrow = (double)gld(w + r0 + threadIdx.x);
    const bool aligned = (((uintptr_t)x) & 15) == 0;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    typedef V pair_t __attribute__((ext_vector_type(2)));
    typedef uint32_t upair_t __attribute__((ext_vector_type(2)));
    // entry range of this wavefront in panel q; uniform over the wavefront
    // (scalar registers, scalar branches)
    // (scalar loads: the table is read-only while the kernel runs)
    auto range = [&](int32_t q, int32_t &rs, int32_t &re) {
        typedef const __attribute__((address_space(4))) int32_t *cptr;
        const cptr wp = (cptr)(pd.wptr + ((int64_t)b * pd.np + q) * (kPanelWaves + 1));
        rs = wp[wv];
        re = wp[wv + 1];
    };
    // chunks of 128 entries from an even start: lane j holds the two
    // consecutive entries at + 2j and at + 2j + 1 (one 16-byte value load,
    // one 8-byte index load).  The entries of the next step are requested
    // before this step's arithmetic (the first step of the next panel before
    // that panel is copied), so loads stay in flight while the wavefront
    // computes or waits.
    pair_t nv[kPanelChunks];
    upair_t nrc[kPanelChunks];
    auto request = [&](int32_t at, int32_t rb, int32_t re) {
#pragma unroll
        for (int u = 0; u < kPanelChunks; ++u) {
            const int32_t e = at + u * 128 + 2 * lane;
            const int32_t ea = (e < re) ? e : rb;
            nv[u] = ld_stream((const pair_t *)(pv + ea));
            nrc[u] = ld_stream((const upair_t *)(pd.rc + ea));
        }
    };
    int32_t ks = 0, ke = 0;
    // One step: chunks of 128 entries at base, base + 128, ..., all in
    // lockstep (independent scans interleave); the sums reach the rows chunk
    // by chunk, in order.  FULL: every entry of the step lies in [ks, ke)
    // (most steps), so the bound checks are compiled out; the two cases are
    // separate code, with no merge of their values.
    auto body = [&](auto fullc, const pair_t (&v)[kPanelChunks],
                    const upair_t (&rc)[kPanelChunks], int32_t base) {
        constexpr bool FULL = decltype(fullc)::value;
        int32_t k0[kPanelChunks], k1[kPanelChunks];
        double p0[kPanelChunks], incl[kPanelChunks];
        // the x values of all entries first, every LDS read in flight at
        // once.  Entries outside [ks, ke) are read too: each is some entry
        // of the matrix, whose column in its panel is below pw, so the read
        // stays inside the panel buffer; its product is dropped.
        V xa[kPanelChunks], xb[kPanelChunks];
#pragma unroll
        for (int u = 0; u < kPanelChunks; ++u) {
            xa[u] = xs[rc[u].x & 0xFFFFu];
            xb[u] = xs[rc[u].y & 0xFFFFu];
        }
#pragma unroll
        for (int u = 0; u < kPanelChunks; ++u) {
            const int32_t e = base + u * 128 + 2 * lane;
            // keys ascend along the wavefront: entries before ks belong to
            // the previous wavefront (-1), entries past ke to nobody (max)
            double p1;
            if (FULL) {
                k0[u] = (int32_t)(rc[u].x >> 16);
                k1[u] = (int32_t)(rc[u].y >> 16);
                p0[u] = (double)v[u].x * (double)xa[u];
                p1 = (double)v[u].y * (double)xb[u];
            } else {
                k0[u] = (e < ks) ? -1 : (e < ke) ? (int32_t)(rc[u].x >> 16) : kPanelMaxRb;
                k1[u] = (e + 1 < ks) ? -1
                        : (e + 1 < ke) ? (int32_t)(rc[u].y >> 16)
                                       : kPanelMaxRb;
                const bool ok0 = e >= ks && e < ke, ok1 = e + 1 >= ks && e + 1 < ke;
                p0[u] = ok0 ? (double)v[u].x * (double)xa[u] : 0.0;
                p1 = ok1 ? (double)v[u].y * (double)xb[u] : 0.0;
            }
            // this lane's part of the run of its last key (a run that
            // starts inside a lane breaks the scan because keys ascend)
            incl[u] = (k0[u] == k1[u]) ? p0[u] + p1 : p1;
        }
#pragma unroll
        for (int u = 0; u < kPanelChunks; ++u)
            incl[u] = seg_scan64<true>(incl[u], k1[u]);
#pragma unroll
        for (int u = 0; u < kPanelChunks; ++u) {
            // the previous lane's scan value and key (wave_shr:1; lane 0
            // reads 0 and key 0, which adds 0 if it matches)
            const double prev_incl = dpp_f64<0x138>(incl[u]);
            const int32_t prev_k1 = dpp_i32z<0x138>(k1[u]);
            const int32_t next_k0 = next_lane_key(k0[u]);
            // a run of k0 that ends on this lane's first entry.  A row's run
            // ends on one lane of a chunk, and a row belongs to one
            // wavefront, whose LDS operations complete in order: the
            // additions (no-return LDS adds, nothing to wait for) reach each
            // row in a fixed order.  Keys of a full step are all rows.
            if (k0[u] != k1[u] && (FULL || (k0[u] >= 0 && k0[u] < kPanelMaxRb)))
                lds_add_f64(&acc[k0[u]], (prev_k1 == k0[u]) ? prev_incl + p0[u] : p0[u]);
            // the run of k1 ends on this lane
            if (next_k0 != k1[u] && (FULL || (k1[u] >= 0 && k1[u] < kPanelMaxRb)))
                lds_add_f64(&acc[k1[u]], incl[u]);
        }
    };
    typedef std::integral_constant<bool, true> full_t;
    typedef std::integral_constant<bool, false> edge_t;
    // A matrix with many row blocks takes its panels in a rotated order:
    // the workgroups that share an XCD (b, b + 8, ...) start at different
    // panels, so their copies of x from that XCD's L2 spread over the run
    // instead of all coming at once.  The order depends only on the matrix
    // and the block, so a block sums its rows the same way in every launch.
    const int32_t rot =
        (pd.np > 1 && pd.nblk >= kPanelRotateBlocks) ? (int32_t)((b >> 3) % pd.np) : 0;
    auto panel_at = [&](int32_t i) { return (i + rot < pd.np) ? i + rot : i + rot - pd.np; };
    if (pd.np > 0)
        range(panel_at(0), ks, ke);
    if ((ks & ~1) < ke)
        request(ks & ~1, ks & ~1, ke);
    for (int32_t pk = 0; pk < pd.np; ++pk) {   // the block's pk-th panel
        const int32_t p = panel_at(pk);
        const int32_t c0 = p * pd.pw;
        const int32_t width = min(pd.pw, pd.cols - c0);
        int32_t nks = 0, nke = 0;  // the next panel's range
        if (pk + 1 < pd.np)
            range(panel_at(pk + 1), nks, nke);
        __syncthreads();  // the previous panel is no longer read
        // 16-byte pieces straight from memory into LDS (no registers): each
        // wavefront instruction fills 1 KiB at a uniform LDS address
        const int32_t nvec = aligned ? width / VV : 0;
        for (int32_t c = wv; c * 64 < nvec; c += kPanelWaves) {
            const int32_t i = c * 64 + lane;
            if (i < nvec)
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void *)(x + c0 + i * VV),
                    (__attribute__((address_space(3))) void *)(xs + c * 64 * VV), 16, 0, 0);
        }
        for (int32_t e = nvec * VV + threadIdx.x; e < width; e += kPanelThreads)
            xs[e] = gld(x + c0 + e);
        __builtin_amdgcn_s_waitcnt(0);  // the direct loads have landed
        __syncthreads();                 // the panel is in LDS
        const int32_t kb = ks & ~1;
        const int32_t nkb = nks & ~1;
        if (kb >= ke && nkb < nke)
            request(nkb, nkb, nke);  // nothing here: the next panel's first step
        for (int32_t base = kb; base < ke; base += 128 * kPanelChunks) {
            pair_t v[kPanelChunks];
            upair_t rc[kPanelChunks];
#pragma unroll
            for (int u = 0; u < kPanelChunks; ++u) {
                v[u] = nv[u];
                rc[u] = nrc[u];
            }
            if (base + 128 * kPanelChunks < ke)
                request(base + 128 * kPanelChunks, kb, ke);
            else if (nkb < nke)
                request(nkb, nkb, nke);
            if (base >= ks && base + 128 * kPanelChunks <= ke)
                body(full_t(), v, rc, base);
            else
                body(edge_t(), v, rc, base);
        }
        ks = nks;
        ke = nke;
    }
    __syncthreads();
    double dacc = 0.0;
    for (int32_t i = threadIdx.x; i < nr; i += kPanelThreads) {
        const V out = epilogue<V>(acc[i], epi);
        gst(y + r0 + i, out);
        if (DOT)
            dacc = fma(i == (int32_t)threadIdx.x ? wrow : (double)gld(w + r0 + i),
                       (double)out, dacc);
    }
    if (DOT) {
        const double tot = block_sum<kPanelWaves>(dacc, (double *)xs);
        if (threadIdx.x == 0)
            dot_part[b] = tot;
    }
}

// Product over the lane form of the column-panel layout: as panel_block, but
// each lane walks its own piece of the wavefront's run, entry after entry:
// value times the LDS copy of x, added up in a register, and at a row's last
// entry one LDS add to the row's sum.  Only what a lane holds of a row that
// goes on in the next lane takes the scan across the wavefront, once a run.
// Bound by the stream of entries (10 bytes each, 12 in the scan form): 150,000
// rows of 241 random columns, float64, 74.5 -> 61.3 us a product (6.28 TB/s of
// the 385 MB it moves; at 63.5 us, 60.5 with one panel copied instead of eight,
// 62.6 without the scan).  Three pairs of columns in flight: two and four took 1% longer, six
// 5% (registers).
// PART: panel group `grp` only, its sums to part[grp * rows + row]; else all.
// Blocks b .. b + NB - 1 by one workgroup (grouped launches): each panel is
// copied once for them; every block's sums are formed as it would alone.
template <typename V, bool DOT, bool PART = false, int NB = 1>
__device__ __forceinline__ void lane_block(const PanelDesc &pd, int32_t b,
                                           const V *__restrict__ x,
                                           V *__restrict__ y, const Epi &epi,
                                           const V *__restrict__ w,
                                           double *__restrict__ dot_part,
                                           unsigned char *smem, int32_t grp = 0,
                                           double *__restrict__ part = nullptr)
{
    constexpr int B = kLanePairs;
    constexpr int VV = 16 / sizeof(V);
    typedef V pair_t __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(4))) int32_t *cptr;
    double *acc = (double *)smem;                                 // row sums
    V *xs = (V *)(smem + panel_sum_bytes(NB * pd.rb));            // x panel
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int32_t r0 = b * pd.rb;
    const V *pv = (const V *)pd.vals;
    for (int i = threadIdx.x; i < NB * pd.rb; i += kPanelThreads)
        acc[i] = 0.0;
    if (threadIdx.x == 0)
        xs[pd.pw] = (V)0;
    // this lane's rows of block b + j: mine, mine + 64, ... below end(j)
    const int32_t mine = wv * pd.rw + lane;
    auto end = [&](int32_t j) {
        return min((wv + 1) * pd.rw, min(pd.rb, pd.rows - r0 - j * pd.rb));
    };
    double wrow = 0.0;
    if (DOT && mine < end(0))
        wrow = (double)gld(w + r0 + mine);
    const bool aligned = (((uintptr_t)x) & 15) == 0;
    // (groups are only formed where there are few blocks: no rotation then)
    const int32_t rot =
        (pd.np > 1 && pd.nblk >= kPanelRotateBlocks) ? (int32_t)((b >> 3) % pd.np) : 0;
    const int32_t p0 = PART ? grp * pd.pg : 0;
    const int32_t p1 = PART ? min(p0 + pd.pg, pd.np) : pd.np;
    constexpr int T = kPanelMaxRb / kPanelThreads / NB;   // rows of a lane in a block
    double tot[NB][T] = {};                               // sums of the groups so far
    auto panel_at = [&](int32_t i) { return (i + rot < pd.np) ? i + rot : i + rot - pd.np; };
    // a run: its first column, its pairs, whether a single column follows
    struct Run {
        int32_t at, pairs, odd;
    };
    auto run_of = [&](int32_t p, int32_t j) {
        if (NB > 1 && b + j >= pd.nblk)
            return Run{0, 0, 0};
        const int32_t q = ((b + j) * pd.np + p) * kPanelWaves + wv;
        const int32_t c0 = ((cptr)pd.col0)[q], k = ((cptr)pd.col0)[q + 1] - c0;
        return Run{c0, k >> 1, k & 1};
    };
    pair_t nv[B];
    u16x2 nw[B];
    V nv1 = (V)0;
    uint16_t nw1 = 0;
    int32_t nstart = 0;
    auto request = [&](const Run &r, int32_t k) {
        const V *v = pv + ((int64_t)r.at + 2 * k) * 64;
        const uint16_t *o = pd.words + ((int64_t)r.at + 2 * k) * 64;
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (k + u < r.pairs) {
                nv[u] = ld_stream((const pair_t *)(v + u * 128) + lane);
                nw[u] = ld_stream((const u16x2 *)(o + u * 128) + lane);
            }
    };
    auto request_first = [&](const Run &r, int32_t p, int32_t j) {
        if (NB > 1 && r.pairs + r.odd == 0)
            return;
        request(r, 0);
        if (r.odd) {
            const int64_t at = ((int64_t)r.at + 2 * r.pairs) * 64 + lane;
            nv1 = ld_stream(pv + at);
            nw1 = ld_stream(pd.words + at);
        }
        nstart = gld(pd.start + ((int64_t)((b + j) * pd.np + p) * kPanelWaves + wv) * 64 + lane);
    };
    Run cur{0, 0, 0}, next{0, 0, 0};
    if (p0 < p1) {
        next = run_of(panel_at(p0), 0);
        request_first(next, panel_at(p0), 0);
    }
    for (int32_t pk = p0; pk < p1; ++pk) {
        const int32_t c0 = panel_at(pk) * pd.pw;
        const int32_t width = min(pd.pw, pd.cols - c0);
        __syncthreads();  // the previous panel is no longer read
        const int32_t nvec = aligned ? width / VV : 0;
        for (int32_t c = wv; c * 64 < nvec; c += kPanelWaves) {
            const int32_t i = c * 64 + lane;
            if (i < nvec)
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void *)(x + c0 + i * VV),
                    (__attribute__((address_space(3))) void *)(xs + c * 64 * VV), 16, 0, 0);
        }
        for (int32_t e = nvec * VV + threadIdx.x; e < width; e += kPanelThreads)
            xs[e] = gld(x + c0 + e);
        __builtin_amdgcn_s_waitcnt(0);  // the direct loads have landed
        __syncthreads();                 // the panel is in LDS
        // the blocks' runs of this panel, each while the next one's first
        // entries are on their way
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            cur = next;
            const bool more = j + 1 < NB || pk + 1 < p1;
            const int32_t jn = j + 1 < NB ? j + 1 : 0;
            const int32_t pn = !more ? 0 : panel_at(j + 1 < NB ? pk : pk + 1);
            if (more)
                next = run_of(pn, jn);
            double *const sums = acc + j * pd.rb;
            int32_t row = wv * pd.rw + nstart;
            const V v1 = nv1;
            const uint32_t w1 = nw1;
            double sum = 0.0;
            auto step = [&](V v, V xv, uint32_t word) {
                sum = fma((double)v, (double)xv, sum);
                if (word & kLaneEnd) {
                    lds_add_f64(&sums[row], sum);
                    ++row;
                    sum = 0.0;
                }
            };
            for (int32_t k = 0; k < cur.pairs; k += B) {
                pair_t v[B];
                u16x2 o[B];
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    v[u] = nv[u];
                    o[u] = nw[u];
                }
                if (k + B < cur.pairs)
                    request(cur, k + B);
                else if (more)
                    request_first(next, pn, jn);
                if (k + B <= cur.pairs) {
                    V xa[B], xb[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        xa[u] = xs[o[u].x & 0x7FFFu];
                        xb[u] = xs[o[u].y & 0x7FFFu];
                    }
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        step(v[u].x, xa[u], o[u].x);
                        step(v[u].y, xb[u], o[u].y);
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < B - 1; ++u)
                        if (k + u < cur.pairs) {
                            const V xa = xs[o[u].x & 0x7FFFu], xb = xs[o[u].y & 0x7FFFu];
                            step(v[u].x, xa, o[u].x);
                            step(v[u].y, xb, o[u].y);
                        }
                }
            }
            if (cur.pairs == 0 && more)
                request_first(next, pn, jn);
            if (cur.odd)
                step(v1, xs[w1 & 0x7FFFu], w1);
            // rows that go on in the next lane, and the run's last row: rows ascend
            // along the lanes, the last lane of a row adds what they hold of it
            if (cur.pairs + cur.odd > 0) {
                const double left = seg_scan64<true>(sum, row);
                if (next_lane_key(row) != row)
                    lds_add_f64(&sums[row], left);
            }
            // a group ends: its sums of the wavefront's own rows (no other adds to
            // them) move to the totals
            if (!PART && pd.ng > 1 && ((pk + 1) % pd.pg == 0 || pk + 1 == p1)) {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const int32_t i = mine + t * 64;
                    if (i < end(j)) {
                        tot[j][t] += sums[i];
                        sums[i] = 0.0;
                    }
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int32_t rj = r0 + j * pd.rb;
        const double *const sums = acc + j * pd.rb;
        double dacc = 0.0;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int32_t i = mine + t * 64;
            if (i >= end(j))
                break;
            if (PART) {
                gst(part + (int64_t)grp * pd.rows + rj + i, sums[i]);
                continue;
            }
            const V out = epilogue<V>(pd.ng > 1 ? tot[j][t] : sums[i], epi);
            gst(y + rj + i, out);
            if (DOT)
                dacc = fma(t == 0 && j == 0 ? wrow : (double)gld(w + rj + i), (double)out, dacc);
        }
        if (DOT && b + j < pd.nblk) {
            const double whole = block_sum<kPanelWaves>(dacc, (double *)xs);
            if (threadIdx.x == 0)
                dot_part[b + j] = whole;
        }
    }
}

template <typename V, bool DOT>
__global__ __launch_bounds__(kPanelThreads) void k_spmv_lanes(
    PanelDesc pd, const V *__restrict__ x, V *__restrict__ y, Epi epi,
    const V *__restrict__ w, double *__restrict__ dot_part)
{
    extern __shared__ __align__(16) unsigned char smem[];
    lane_block<V, DOT>(pd, blockIdx.x, x, y, epi, w, dot_part, smem);
}

// One workgroup for each row block and group of panels: a matrix of few row
// blocks would leave most compute units idle (200k rows: 49 blocks).
// NB row blocks to each of them (pd.gper).
template <typename V, int NB>
__global__ __launch_bounds__(kPanelThreads) void k_spmv_lane_groups(
    PanelDesc pd, const V *__restrict__ x, double *__restrict__ part)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const Epi epi{EPI_NONE, 0, 0.0, 0.0};
    const int32_t nb = (pd.nblk + NB - 1) / NB;
    const int32_t grp = blockIdx.x / nb;
    lane_block<V, false, true, NB>(pd, (blockIdx.x - grp * nb) * NB, x, nullptr, epi, nullptr,
                                   nullptr, smem, grp, part);
}

// The groups' sums of a row block added up in order, with the epilogue and the
// fused dot of lane_block (the same additions in the same order).
template <typename V, bool DOT>
__global__ __launch_bounds__(kPanelThreads) void k_lane_total(
    PanelDesc pd, const double *__restrict__ part, V *__restrict__ y, Epi epi,
    const V *__restrict__ w, double *__restrict__ dot_part)
{
    __shared__ double lds[kPanelWaves];
    // with the dot a row block each, every lane the rows lane_block gives it
    // (its partial's additions in the same order); else a row for each thread
    const int32_t b = blockIdx.x;
    const int32_t wv = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)b * (DOT ? pd.rb : kPanelThreads);
    const int32_t nr = (int32_t)min((int64_t)(DOT ? pd.rb : kPanelThreads), pd.rows - r0);
    const int32_t rw = DOT ? pd.rw : 64;
    const int32_t end = min((wv + 1) * rw, nr);
    double dacc = 0.0;
    for (int32_t i = wv * rw + (threadIdx.x & 63); i < end; i += 64) {
        double sum = 0.0;
#pragma unroll 4
        for (int32_t g = 0; g < pd.ng; ++g)
            sum += gld(part + (int64_t)g * pd.rows + r0 + i);
        const V out = epilogue<V>(sum, epi);
        gst(y + r0 + i, out);
        if (DOT)
            dacc = fma((double)gld(w + r0 + i), (double)out, dacc);
    }
    if (DOT) {
        const double tot = block_sum<kPanelWaves>(dacc, lds);
        if (threadIdx.x == 0)
            dot_part[b] = tot;
    }
}

template <typename V, bool DOT>
__global__ __launch_bounds__(kPanelThreads) void k_spmv_panels(
    PanelDesc pd, const V *__restrict__ x, V *__restrict__ y, Epi epi,
    const V *__restrict__ w, double *__restrict__ dot_part)
{
    extern __shared__ __align__(16) unsigned char smem[];
    panel_block<V, DOT>(pd, blockIdx.x, x, y, epi, w, dot_part, smem);
}

// Column-panel products of many matrices in one launch: workgroup g takes
// the (g - prefix[j])-th row block of matrix j (prefix[j] <= g < prefix[j + 1]),
// or its (g - prefix[j])-th two or four (per).  Each block's sums are formed exactly as in
// the single-matrix kernel.
template <typename V>
__global__ __launch_bounds__(kPanelThreads) void k_spmv_panels_grouped(
    const PanelDesc *__restrict__ descs, const PanelIO *__restrict__ io,
    const int32_t *__restrict__ prefix, int32_t nmat)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int32_t g = blockIdx.x;
    int32_t lo = 0, hi = nmat - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= g)
            lo = mid;
        else
            hi = mid - 1;
    }
    const PanelDesc pd = descs[lo];
    const Epi epi{EPI_NONE, 0, 0.0, 0.0};
    const PanelIO pio = io[lo];
    if (pd.col0) {
        const int32_t b = (g - prefix[lo]) * pd.per;
        const V *x = (const V *)pio.x;
        V *y = (V *)pio.y;
        if constexpr (sizeof(V) == 8) {
            if (pio.dot && pd.per == 4)
                lane_block<V, true, false, 4>(pd, b, x, y, epi, x, pio.dot, smem);
            else if (pio.dot && pd.per == 2)
                lane_block<V, true, false, 2>(pd, b, x, y, epi, x, pio.dot, smem);
            else if (pio.dot)
                lane_block<V, true>(pd, b, x, y, epi, x, pio.dot, smem);
            if (pio.dot)
                return;
        }
        if (pd.per == 4)
            lane_block<V, false, false, 4>(pd, b, x, y, epi, nullptr, nullptr, smem);
        else if (pd.per == 2)
            lane_block<V, false, false, 2>(pd, b, x, y, epi, nullptr, nullptr, smem);
        else
            lane_block<V, false>(pd, b, x, y, epi, nullptr, nullptr, smem);
        return;
    }
    if constexpr (sizeof(V) == 8) {
        if (pio.dot) {
            panel_block<V, true>(pd, g - prefix[lo], (const V *)pio.x, (V *)pio.y, epi,
                                 (const V *)pio.x, pio.dot, smem);
            return;
        }
    }
    panel_block<V, false>(pd, g - prefix[lo], (const V *)pio.x, (V *)pio.y,
                          epi, nullptr, nullptr, smem);
}

// Distinct x cache lines among the non-zeros of sampled row groups (see
// launch_line_reuse).  The count is a union of bits, so it does not depend
// on the order of the atomic updates.
__global__ __launch_bounds__(kBlock) void k_line_reuse(int32_t rows,
                                                       const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ col,
                                                       int32_t ngroups, int32_t shift,
                                                       int32_t *__restrict__ out)
{
    __shared__ uint32_t bits[512];
    __shared__ int32_t red[kWaves];
    for (int i = threadIdx.x; i < 512; i += kBlock)
        bits[i] = 0u;
    __syncthreads();
    const int64_t groups = ((int64_t)rows + 63) / 64;
    const int32_t grp = (int32_t)((int64_t)blockIdx.x * groups / ngroups);
    const int32_t r0 = grp * 64;
    const int32_t r1 = min(rows, r0 + 64);
    const int32_t k0 = rp[r0];
    const int32_t k1 = min(rp[r1], k0 + 8192);
    for (int32_t k = k0 + threadIdx.x; k < k1; k += kBlock) {
        const uint32_t line = (uint32_t)col[k] >> shift;
        atomicOr(&bits[(line >> 5) & 511u], 1u << (line & 31u));
    }
    __syncthreads();
    int32_t cnt = 0;
    for (int i = threadIdx.x; i < 512; i += kBlock)
        cnt += __popc(bits[i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        cnt += __shfl_down(cnt, off, 64);
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int i = 0; i < kWaves; ++i)
            t += red[i];
        out[2 * blockIdx.x] = k1 - k0;
        out[2 * blockIdx.x + 1] = t;
    }
}

// Entries of each row per panel: one wavefront per row, 64 entries at a
// time, one ballot per panel (cnt pre-zeroed).
__global__ __launch_bounds__(kBlock) void k_panel_count(PanelDesc pd,
                                                        const int32_t *__restrict__ rp,
                                                        const int32_t *__restrict__ col,
                                                        int32_t *__restrict__ cnt)
{
    const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (i >= pd.rows)
        return;  // whole wavefronts
    const int32_t b = (int32_t)(i / pd.rb), rl = (int32_t)(i - (int64_t)b * pd.rb);
    const int32_t a = rp[i], e = rp[i + 1];
    int32_t mine = 0;  // lane p < np counts panel p
    for (int32_t base = a; base < e; base += 64) {
        const int32_t k = base + lane;
        const int32_t pan = (k < e) ? col[k] / pd.pw : -1;
        for (int32_t p = 0; p < pd.np; ++p) {
            const int32_t n = __popcll(__ballot(pan == p));
            if (lane == p)
                mine += n;
        }
    }
    if (lane < pd.np)
        cnt[(int64_t)(b * pd.np + lane) * (pd.rb + 1) + rl] = mine;
}

// Move each row's entries to their panels, keeping their order inside a
// row: one wavefront per row, 64 entries at a time, positions from ballots.
template <typename V>
__global__ __launch_bounds__(kBlock) void k_panel_scatter(
    PanelDesc pd, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const V *__restrict__ vals, const int32_t *__restrict__ ptr,
    V *__restrict__ pv, uint32_t *__restrict__ prc)
{
    const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (i >= pd.rows)
        return;  // whole wavefronts
    const int32_t b = (int32_t)(i / pd.rb), rl = (int32_t)(i - (int64_t)b * pd.rb);
    const int32_t a = rp[i], e = rp[i + 1];
    // lane p < np holds the next free position of panel p
    int32_t next = (lane < pd.np) ? ptr[(int64_t)(b * pd.np + lane) * (pd.rb + 1) + rl] : 0;
    for (int32_t base = a; base < e; base += 64) {
        const int32_t k = base + lane;
        const int32_t c = (k < e) ? col[k] : 0;
        const int32_t pan = (k < e) ? c / pd.pw : -1;
        int32_t pos = 0;
        for (int32_t p = 0; p < pd.np; ++p) {
            const uint64_t m = __ballot(pan == p);
            const int32_t start = __shfl(next, p, 64);
            if (pan == p)
                pos = start + lanes_below(m);
            if (lane == p)
                next += __popcll(m);
        }
        if (k < e) {
            pv[pos] = vals[k];
            if (prc)
                prc[pos] = ((uint32_t)rl << 16) | (uint32_t)(c - pan * pd.pw);
        }
    }
}

// Lane form, per run (one wavefront each): rows without an entry between the
// run's first and last row that have one get a filler (count 1), and the run
// as many columns as 64 equal pieces of it take.
__global__ __launch_bounds__(kBlock) void k_lane_runs(PanelDesc pd, int32_t *__restrict__ cnt,
                                                      int32_t *__restrict__ kc)
{
    const int64_t q = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (q >= (int64_t)pd.nblk * pd.np * kPanelWaves)
        return;  // whole wavefronts
    const int64_t seg = q / kPanelWaves;
    const int32_t a = min((int32_t)(q - seg * kPanelWaves) * pd.rw, pd.rb);
    const int32_t z = min(a + pd.rw, pd.rb);
    int32_t *c = cnt + seg * (pd.rb + 1);
    int32_t first = INT_MAX, last = -1;
    for (int32_t r = a + lane; r < z; r += 64)
        if (c[r] > 0) {
            first = min(first, r);
            last = r;
        }
    first = -lane_group_max<64>(-first);
    last = lane_group_max<64>(last);
    int32_t n = 0;
    for (int32_t r = a + lane; r < z; r += 64) {
        int32_t m = c[r];
        if (m == 0 && r > first && r < last) {
            m = 1;
            c[r] = 1;
        }
        n += m;
    }
    n = wave_sum_i32(n);
    if (lane == 0)
        kc[q] = (n + 63) / 64;
}

// Place of entry j of lane l of a run of k columns from column at.
__device__ __forceinline__ int64_t lane_place(int32_t at, int32_t k, int32_t j, int32_t l)
{
    return (j < (k & ~1)) ? ((int64_t)at + (j & ~1)) * 64 + l * 2 + (j & 1)
                          : ((int64_t)at + j) * 64 + l;
}

// Padding, fillers and start rows (the entries are written afterwards; a row
// of count 1 is written as a filler here, whatever it is).  pos: exclusive
// scan of the counts.  One wavefront per run.
template <typename V>
__global__ __launch_bounds__(kBlock) void k_lane_fill(PanelDesc pd,
                                                      const int32_t *__restrict__ pos,
                                                      V *__restrict__ vals,
                                                      uint16_t *__restrict__ words,
                                                      uint8_t *__restrict__ start)
{
    const int64_t q = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (q >= (int64_t)pd.nblk * pd.np * kPanelWaves)
        return;  // whole wavefronts
    const int64_t seg = q / kPanelWaves;
    const int32_t a = min((int32_t)(q - seg * kPanelWaves) * pd.rw, pd.rb);
    const int32_t z = min(a + pd.rw, pd.rb);
    const int32_t *P = pos + seg * (pd.rb + 1);
    const int32_t base = P[a], n = P[z] - base;
    const int32_t at = pd.col0[q], k = pd.col0[q + 1] - at;
    for (int32_t i = n + lane; i < k * 64; i += 64) {
        const int32_t l = i / k;
        const int64_t e = lane_place(at, k, i - l * k, l);
        vals[e] = (V)0;
        words[e] = (uint16_t)pd.pw;
    }
    for (int32_t r = a + lane; r < z; r += 64)
        if (P[r + 1] - P[r] == 1) {
            const int32_t i = P[r] - base, l = i / k;
            const int64_t e = lane_place(at, k, i - l * k, l);
            vals[e] = (V)0;
            words[e] = (uint16_t)(pd.pw | kLaneEnd);
        }
    // row of the lane's first entry: the last row that starts at or before
    // it and is not empty; lanes past the end take the last row
    int32_t lo = a, hi = max(a, z - 1);
    const int32_t want = base + min(lane * k, max(n - 1, 0));
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (P[mid] <= want)
            lo = mid;
        else
            hi = mid - 1;
    }
    start[q * 64 + lane] = (uint8_t)(lo - a);
}

// The entries (words null: their values alone): one wavefront per row, 64 entries
// at a time, positions from ballots as in k_panel_scatter.
template <typename V>
__global__ __launch_bounds__(kBlock) void k_lane_scatter(
    PanelDesc pd, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const V *__restrict__ src, const int32_t *__restrict__ pos, V *__restrict__ vals,
    uint16_t *__restrict__ words)
{
    const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (i >= pd.rows)
        return;  // whole wavefronts
    const int32_t b = (int32_t)(i / pd.rb), rl = (int32_t)(i - (int64_t)b * pd.rb);
    const int32_t wv = rl / pd.rw;
    const int32_t a = rp[i], e = rp[i + 1];
    // lane p < np: panel p's next position in the run, the row's last one
    // (-1 on the run's last row, which takes no end mark), the run's first
    // column and columns
    int32_t next = 0, last = 0, at = 0, k = 1;
    if (lane < pd.np) {
        const int64_t seg = (int64_t)b * pd.np + lane;
        const int32_t *P = pos + seg * (pd.rb + 1);
        const int32_t base = P[wv * pd.rw];
        next = P[rl] - base;
        last = (P[rl + 1] < P[min((wv + 1) * pd.rw, pd.rb)]) ? P[rl + 1] - base - 1 : -1;
        at = pd.col0[seg * kPanelWaves + wv];
        k = max(1, pd.col0[seg * kPanelWaves + wv + 1] - at);
    }
    for (int32_t s = a; s < e; s += 64) {
        const int32_t n = s + lane;
        const int32_t c = (n < e) ? col[n] : 0;
        const int32_t pan = (n < e) ? c / pd.pw : -1;
        int32_t j = 0, end = 0, pat = 0, pk = 1;
        for (int32_t p = 0; p < pd.np; ++p) {
            const uint64_t m = __ballot(pan == p);
            if (!m)
                continue;   // uniform
            const int32_t from = __shfl(next, p, 64), to = __shfl(last, p, 64);
            const int32_t fat = __shfl(at, p, 64), fk = __shfl(k, p, 64);
            if (pan == p) {
                j = from + lanes_below(m);
                end = to;
                pat = fat;
                pk = fk;
            }
            if (lane == p)
                next += __popcll(m);
        }
        if (n < e) {
            const int32_t l = j / pk;
            const int64_t place = lane_place(pat, pk, j - l * pk, l);
            vals[place] = src[n];
            if (words)
                words[place] = (uint16_t)((c - pan * pd.pw) | (j == end ? kLaneEnd : 0u));
        }
    }
}

// Where each wavefront's rows start, for every (row block, panel).
__global__ __launch_bounds__(kBlock) void k_panel_wptr(PanelDesc pd,
                                                       const int32_t *__restrict__ ptr,
                                                       int32_t *__restrict__ wptr)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t nseg = (int64_t)pd.nblk * pd.np;
    if (t >= nseg * (kPanelWaves + 1))
        return;
    const int64_t seg = t / (kPanelWaves + 1);
    const int32_t wv = (int32_t)(t - seg * (kPanelWaves + 1));
    wptr[t] = ptr[seg * (pd.rb + 1) + min(wv * pd.rw, pd.rb)];
}

// ------------------------------------------------------- hot columns

// Row keys inside a block are below 2^16; this one is past every row.
constexpr int32_t kKeyEnd = 1 << 16;

// The first chunk of a wavefront's share of a block part, requested ahead.
template <typename V>
struct HotChunk {
    typedef V pair_t __attribute__((ext_vector_type(2)));
    typedef uint32_t upair_t __attribute__((ext_vector_type(2)));
    typedef uint16_t kpair_t __attribute__((ext_vector_type(2)));
    pair_t v;
    upair_t rc;
    kpair_t kk;
};

// This wavefront's share [ks, ke) of a part [s, e) split evenly between NW.
template <int NW>
__device__ __forceinline__ void hot_share(int32_t s, int32_t e, int wave, int32_t &ks,
                                          int32_t &ke)
{
    const int64_t n = (int64_t)e - s;
    ks = __builtin_amdgcn_readfirstlane(s + (int32_t)(n * wave / NW));
    ke = __builtin_amdgcn_readfirstlane(s + (int32_t)(n * (wave + 1) / NW));
}

// Requests the first chunk of this wavefront's share of a part (nothing if
// the share is empty).
template <typename V, bool HOT, int NW = kPanelWaves>
__device__ __forceinline__ void hot_first(const V *__restrict__ pv,
                                          const uint32_t *__restrict__ prc,
                                          const uint16_t *__restrict__ pkey, int32_t s,
                                          int32_t e, int wave, int lane, HotChunk<V> &c)
{
    typedef typename HotChunk<V>::pair_t pair_t;
    typedef typename HotChunk<V>::upair_t upair_t;
    typedef typename HotChunk<V>::kpair_t kpair_t;
    int32_t ks, ke;
    hot_share<NW>(s, e, wave, ks, ke);
    const int32_t kb = ks & ~1;
    if (kb < ke) {
        const int32_t en = kb + 2 * lane;
        const int32_t ea = (en < ke) ? en : kb;
        c.v = ld_stream((const pair_t *)(pv + ea));
        c.rc = ld_stream((const upair_t *)(prc + ea));
        if (!HOT)
            c.kk = ld_stream((const kpair_t *)(pkey + ea));
    }
}

// One wavefront's share of a block part [s, e) of the hot-column layout.
// The part is split evenly by entries, so a row can span wavefronts: the
// run of the wavefront's first row goes to its carry slot (added after the
// block, in slot order), every other run is added to the row sum in LDS by
// the one wavefront where it ends.  A row is named by its key (its number
// among the block's non-empty rows in the hot-column layout, its offset in
// the block in the band layout).  HOT: the entry's word packs (key << 16)
// | column offset and the gather reads xsrc[offset] (the LDS copy of the
// hot columns, or x from a block's first column in the band layout);
// otherwise the word is the column of x and the key comes from key[].  The
// entries of the next chunk are requested before the gathers of the
// current one are used; with gathers from device memory the next chunk's
// gathers are requested too.  NW wavefronts share the part; XG: xsrc is in
// device memory (else in LDS).  PRE: the first chunk was requested earlier
// into *pre (hot_first, same part and wavefront).
template <typename V, bool HOT, int NW = kPanelWaves, bool XG = !HOT, bool PRE = false>
__device__ __forceinline__ void hot_part(const V *__restrict__ pv,
                                         const uint32_t *__restrict__ prc,
                                         const uint16_t *__restrict__ pkey,
                                         int32_t s, int32_t e, const V *xsrc,
                                         double *acc, int32_t *ckey, double *csum,
                                         int wave, int lane,
                                         const HotChunk<V> *pre = nullptr)
{
    typedef typename HotChunk<V>::pair_t pair_t;
    typedef typename HotChunk<V>::upair_t upair_t;
    typedef typename HotChunk<V>::kpair_t kpair_t;
    int32_t ks, ke;
    hot_share<NW>(s, e, wave, ks, ke);
    const int32_t kb = ks & ~1;
    pair_t v;
    upair_t rc;
    kpair_t kk;
    int32_t first = -1;
    if (kb < ke) {
        if (PRE) {
            v = pre->v;
            rc = pre->rc;
            if (!HOT)
                kk = pre->kk;
        } else {
            const int32_t en = kb + 2 * lane;
            const int32_t ea = (en < ke) ? en : kb;
            v = ld_stream((const pair_t *)(pv + ea));
            rc = ld_stream((const upair_t *)(prc + ea));
            if (!HOT)
                kk = ld_stream((const kpair_t *)(pkey + ea));
        }
        // the share's first entry is entry 0 or 1 of lane 0
        const int32_t f0 = HOT ? (int32_t)(rc.x >> 16) : (int32_t)kk.x;
        const int32_t f1 = HOT ? (int32_t)(rc.y >> 16) : (int32_t)kk.y;
        first = __builtin_amdgcn_readfirstlane((ks == kb) ? f0 : f1);
    }
    if (lane == 0) {
        *ckey = first;
        *csum = 0.0;
    }
    // whether entry j of the chunk at `base` lies in the share, and the
    // column it gathers (entries outside the share may belong to the other
    // part, another packing: they gather element 0, which always exists)
    auto in_share = [&](int32_t base, int j) {
        const int32_t en = base + 2 * lane + j;
        return (base >= ks && base + 128 <= ke) || (en >= ks && en < ke);
    };
    auto column = [&](uint32_t w, bool ok) {
        return ok ? (HOT ? (w & 0xFFFFu) : w) : 0u;
    };
    auto request = [&](int32_t at, pair_t &rv, upair_t &rr, kpair_t &rk) {
        const int32_t nn = at + 2 * lane;
        const int32_t ea = (nn < ke) ? nn : kb;
        rv = ld_stream((const pair_t *)(pv + ea));
        rr = ld_stream((const upair_t *)(prc + ea));
        if (!HOT)
            rk = ld_stream((const kpair_t *)(pkey + ea));
    };
    // gathers from device memory: the next chunk's entries are in hand and
    // its gathers requested before this chunk's arithmetic, with the entries
    // of the chunk after it on the way (two memory round trips per chunk,
    // the second depending on the first, kept in flight together)
    V gx0 = 0, gx1 = 0;     // gathers of the current chunk
    pair_t v2;              // entries of the next chunk
    upair_t rc2;
    kpair_t kk2;
    if (XG && kb < ke) {
        gx0 = gld(xsrc + column(rc.x, in_share(kb, 0)));
        gx1 = gld(xsrc + column(rc.y, in_share(kb, 1)));
        if (kb + 128 < ke)
            request(kb + 128, v2, rc2, kk2);
    }
    for (int32_t base = kb; base < ke; base += 128) {
        const int32_t en = base + 2 * lane;
        // chunks wholly inside [ks, ke) (most of them) need no bound checks
        const bool full = base >= ks && base + 128 <= ke;
        const bool ok0 = full || (en >= ks && en < ke);
        const bool ok1 = full || (en + 1 >= ks && en + 1 < ke);
        const int32_t r0 = HOT ? (int32_t)(rc.x >> 16) : (int32_t)kk.x;
        const int32_t r1 = HOT ? (int32_t)(rc.y >> 16) : (int32_t)kk.y;
        // keys ascend along the wavefront: entries before ks belong to the
        // previous wavefront (-1), entries past ke to nobody (kKeyEnd)
        const int32_t k0 = full ? r0 : (en < ks) ? -1 : ok0 ? r0 : kKeyEnd;
        const int32_t k1 = full ? r1 : (en + 1 < ks) ? -1 : ok1 ? r1 : kKeyEnd;
        const pair_t cv = v;
        const int32_t nb = base + 128;
        V x0, x1;
        if (XG) {
            x0 = gx0;
            x1 = gx1;
            if (nb < ke) {
                v = v2;
                rc = rc2;
                if (!HOT)
                    kk = kk2;
                gx0 = gld(xsrc + column(rc.x, in_share(nb, 0)));
                gx1 = gld(xsrc + column(rc.y, in_share(nb, 1)));
                if (nb + 128 < ke)
                    request(nb + 128, v2, rc2, kk2);
            }
        } else {
            x0 = xsrc[column(rc.x, ok0)];
            x1 = xsrc[column(rc.y, ok1)];
            if (nb < ke)
                request(nb, v, rc, kk);
        }
        const double p0 = ok0 ? (double)cv.x * (double)x0 : 0.0;
        const double p1 = ok1 ? (double)cv.y * (double)x1 : 0.0;
        // this lane's part of the run of its last key (a run that starts
        // inside a lane breaks the scan because keys ascend)
        double incl = (k0 == k1) ? p0 + p1 : p1;
        incl = seg_scan64(incl, k1);
        // previous lane's scan value and key (wave_shr:1; lane 0 reads 0)
        const double prev_incl = dpp_f64<0x138>(incl);
        const int32_t prev_k1 = dpp_i32z<0x138>(k1);
        const int32_t next_k0 = next_lane_key(k0);
        // no-return LDS adds: a row's runs end in this wavefront only (its
        // first row goes to the carry slot), in program order
        if (k0 != k1 && k0 >= 0 && k0 < kKeyEnd) {
            double *t = (k0 == first) ? csum : acc + k0;
            lds_add_f64(t, (prev_k1 == k0) ? prev_incl + p0 : p0);
        }
        if (next_k0 != k1 && k1 >= 0 && k1 < kKeyEnd) {
            double *t = (k1 == first) ? csum : acc + k1;
            lds_add_f64(t, incl);
        }
    }
}


// The same for four entries per lane (float32 values: 16-byte loads).
struct HotChunk4 {
    typedef float quad_t __attribute__((ext_vector_type(4)));
    typedef uint32_t uquad_t __attribute__((ext_vector_type(4)));
    typedef uint16_t kquad_t __attribute__((ext_vector_type(4)));
    quad_t v;
    uquad_t rc;
    kquad_t kk;
};

template <bool HOT, int NW = kPanelWaves>
__device__ __forceinline__ void hot_first4(const float *__restrict__ pv,
                                           const uint32_t *__restrict__ prc,
                                           const uint16_t *__restrict__ pkey, int32_t s,
                                           int32_t e, int wave, int lane, HotChunk4 &c)
{
    int32_t ks, ke;
    hot_share<NW>(s, e, wave, ks, ke);
    const int32_t kb = ks & ~3;
    if (kb < ke) {
        const int32_t en = kb + 4 * lane;
        const int32_t ea = (en < ke) ? en : kb;
        c.v = ld_stream((const HotChunk4::quad_t *)(pv + ea));
        c.rc = ld_stream((const HotChunk4::uquad_t *)(prc + ea));
        if (!HOT)
            c.kk = ld_stream((const HotChunk4::kquad_t *)(pkey + ea));
    }
}

// hot_part with four consecutive entries per lane and chunks of 256 from a
// multiple of four: the runs that start and end inside a lane are added
// directly, the lane's first run joins the previous lane's scan value, its
// last run enters a segmented scan over the wavefront.  Each row still
// gets one addition per chunk, from the lane where its run ends, so the
// order of the additions is fixed by the matrix and the layout.
template <bool HOT, int NW = kPanelWaves, bool XG = !HOT, bool PRE = false>
__device__ __forceinline__ void hot_part4(const float *__restrict__ pv,
                                          const uint32_t *__restrict__ prc,
                                          const uint16_t *__restrict__ pkey,
                                          int32_t s, int32_t e, const float *xsrc,
                                          double *acc, int32_t *ckey, double *csum,
                                          int wave, int lane,
                                          const HotChunk4 *pre = nullptr)
{
    typedef HotChunk4::quad_t quad_t;
    typedef HotChunk4::uquad_t uquad_t;
    typedef HotChunk4::kquad_t kquad_t;
    constexpr int32_t CH = 256;
    int32_t ks, ke;
    hot_share<NW>(s, e, wave, ks, ke);
    const int32_t kb = ks & ~3;
    quad_t v;
    uquad_t rc;
    kquad_t kk;
    int32_t first = -1;
    if (kb < ke) {
        if (PRE) {
            v = pre->v;
            rc = pre->rc;
            if (!HOT)
                kk = pre->kk;
        } else {
            const int32_t en = kb + 4 * lane;
            const int32_t ea = (en < ke) ? en : kb;
            v = ld_stream((const quad_t *)(pv + ea));
            rc = ld_stream((const uquad_t *)(prc + ea));
            if (!HOT)
                kk = ld_stream((const kquad_t *)(pkey + ea));
        }
        // the share's first entry is entry ks - kb of lane 0
        const int32_t d = ks - kb;
        const uint32_t w0 = d == 0 ? rc.x : d == 1 ? rc.y : d == 2 ? rc.z : rc.w;
        const uint32_t q0 = d == 0 ? kk.x : d == 1 ? kk.y : d == 2 ? kk.z : kk.w;
        first = __builtin_amdgcn_readfirstlane(HOT ? (int32_t)(w0 >> 16) : (int32_t)q0);
    }
    if (lane == 0) {
        *ckey = first;
        *csum = 0.0;
    }
    auto in_share = [&](int32_t base, int j) {
        const int32_t en = base + 4 * lane + j;
        return (base >= ks && base + CH <= ke) || (en >= ks && en < ke);
    };
    auto column = [&](uint32_t w, bool ok) {
        return ok ? (HOT ? (w & 0xFFFFu) : w) : 0u;
    };
    auto request = [&](int32_t at, quad_t &rv, uquad_t &rr, kquad_t &rk) {
        const int32_t nn = at + 4 * lane;
        const int32_t ea = (nn < ke) ? nn : kb;
        rv = ld_stream((const quad_t *)(pv + ea));
        rr = ld_stream((const uquad_t *)(prc + ea));
        if (!HOT)
            rk = ld_stream((const kquad_t *)(pkey + ea));
    };
    auto add = [&](int32_t k, double t) {
        lds_add_f64((k == first) ? csum : acc + k, t);
    };
    float g[4] = {0.f, 0.f, 0.f, 0.f};   // gathers of the current chunk
    quad_t v2;                           // entries of the next chunk
    uquad_t rc2;
    kquad_t kk2;
    if (XG && kb < ke) {
        g[0] = gld(xsrc + column(rc.x, in_share(kb, 0)));
        g[1] = gld(xsrc + column(rc.y, in_share(kb, 1)));
        g[2] = gld(xsrc + column(rc.z, in_share(kb, 2)));
        g[3] = gld(xsrc + column(rc.w, in_share(kb, 3)));
        if (kb + CH < ke)
            request(kb + CH, v2, rc2, kk2);
    }
    // one chunk; FULL: every entry lies in [ks, ke) (most chunks), so the
    // bound checks are compiled out (full and edge chunks are separate code)
    auto body = [&](int32_t base, auto fullc) {
        const int32_t en = base + 4 * lane;
        constexpr bool full = decltype(fullc)::value;
        const uint32_t wv[4] = {rc.x, rc.y, rc.z, rc.w};
        const int32_t rw[4] = {HOT ? (int32_t)(rc.x >> 16) : (int32_t)kk.x,
                               HOT ? (int32_t)(rc.y >> 16) : (int32_t)kk.y,
                               HOT ? (int32_t)(rc.z >> 16) : (int32_t)kk.z,
                               HOT ? (int32_t)(rc.w >> 16) : (int32_t)kk.w};
        const float cv[4] = {v.x, v.y, v.z, v.w};
        bool ok[4];
        int32_t k[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            ok[t] = full || (en + t >= ks && en + t < ke);
            k[t] = full ? rw[t] : (en + t < ks) ? -1 : ok[t] ? rw[t] : kKeyEnd;
        }
        float xv[4];
        const int32_t nb = base + CH;
        if (XG) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                xv[t] = g[t];
            if (nb < ke) {
                v = v2;
                rc = rc2;
                if (!HOT)
                    kk = kk2;
                g[0] = gld(xsrc + column(rc.x, in_share(nb, 0)));
                g[1] = gld(xsrc + column(rc.y, in_share(nb, 1)));
                g[2] = gld(xsrc + column(rc.z, in_share(nb, 2)));
                g[3] = gld(xsrc + column(rc.w, in_share(nb, 3)));
                if (nb + CH < ke)
                    request(nb + CH, v2, rc2, kk2);
            }
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                xv[t] = xsrc[column(wv[t], ok[t])];
            if (nb < ke)
                request(nb, v, rc, kk);
        }
        double pr[4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            pr[t] = ok[t] ? (double)cv[t] * (double)xv[t] : 0.0;
        // runs inside the lane (keys ascend)
        double run = pr[0], head = 0.0;
        int32_t rk = k[0];
        bool split = false;
#pragma unroll
        for (int t = 1; t < 4; ++t) {
            if (k[t] == rk) {
                run += pr[t];
            } else {
                if (!split) {
                    head = run;
                    split = true;
                } else if (full || (rk >= 0 && rk < kKeyEnd)) {
                    add(rk, run);   // a run wholly inside this lane
                }
                rk = k[t];
                run = pr[t];
            }
        }
        const double incl = seg_scan64(run, k[3]);
        const double prev_incl = dpp_f64<0x138>(incl);
        const int32_t prev_kl = dpp_i32z<0x138>(k[3]);
        const int32_t next_kf = next_lane_key(k[0]);
        if (split && (full || (k[0] >= 0 && k[0] < kKeyEnd)))
            add(k[0], (prev_kl == k[0]) ? prev_incl + head : head);
        if (next_kf != k[3] && (full || (k[3] >= 0 && k[3] < kKeyEnd)))
            add(k[3], incl);
    };
    for (int32_t base = kb; base < ke; base += CH) {
        if (base >= ks && base + CH <= ke)
            body(base, std::true_type());
        else
            body(base, std::false_type());
    }
}

// Product over the hot-column layout.  Persistent: workgroup g copies the
// hot columns of x into LDS once, then takes its own list of row blocks
// (assigned on the host, balanced by work).
// Each wavefront streams its share of the block's hot part and of its cold
// part (odd wavefronts cold first, so LDS and global gathers overlap); the
// two parts add into separate row sums, so no wavefront waits for another
// between them.  The carries are then summed in slot order by one lane per
// row, and each row's result is its hot sum plus its cold sum: every sum is
// formed in an order fixed by the matrix and the layout.  float32 matrices
// take four entries per lane (hot_part4), float64 two (hot_part).
// DIRECT: x is in the caller's column order; hd.old places the hot columns in
// it, and the cold entries' words are the caller's columns.  For where no memory
// may be used for x in the layout's order, as under capture: the same sums, but
// the cold gathers meet x as it lies.  R-MAT, 16 entries a row, x copied first,
// direct, and row-class tiles: float32 2^18 24, 26 and 39 us, 2^20 70, 86 and 149,
// 2^22 292, 495 and 771; float64 32, 37 and 48; 97, 114 and 180; 406, 695 and 910.
template <typename V, bool DOT, bool DIRECT = false>
__global__ __launch_bounds__(kPanelThreads) void k_spmv_hot(
    HotDesc hd, const V *__restrict__ x, V *__restrict__ y, Epi epi,
    const V *__restrict__ w, double *__restrict__ dot_part)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double *acc_h = (double *)smem;                                    // hot row sums
    double *acc_c = (double *)(smem + kHotRows * 8);                   // cold row sums
    double *csum = (double *)(smem + 2 * kHotRows * 8);                // 32 carries
    int32_t *ckey = (int32_t *)(smem + 2 * kHotRows * 8 + 32 * 8);     // their rows
    V *xs = (V *)(smem + kHotLdsHead);                                 // hot columns
    constexpr int VV = 16 / sizeof(V);
    typedef V vec_t __attribute__((ext_vector_type(VV)));
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const V *pv = (const V *)hd.vals;
    const uint32_t *cold = DIRECT ? hd.cold : hd.rc;   // words of the cold entries
    const int32_t width = hd.hot;
    const bool aligned = (((uintptr_t)x) & 15) == 0;
    const int32_t nvec = aligned ? width / VV : 0;
    if (DIRECT) {
        for (int32_t e = threadIdx.x; e < width; e += kPanelThreads)
            xs[e] = gld(x + gld(hd.old + e));
    } else {
        for (int32_t i = threadIdx.x; i < nvec; i += kPanelThreads)
            *(vec_t *)(xs + i * VV) = gld((const vec_t *)(x + i * VV));
        for (int32_t e = nvec * VV + threadIdx.x; e < width; e += kPanelThreads)
            xs[e] = gld(x + e);
    }
    for (int i = threadIdx.x; i < 2 * kHotRows; i += kPanelThreads)
        acc_h[i] = 0.0;  // both sum arrays
    double dacc = 0.0;
    // the first chunk of the wavefront's first part of block bb is requested
    // before the barriers that end the previous block
    typedef const __attribute__((address_space(4))) int32_t *cptr;
    constexpr bool Q = sizeof(V) == 4;   // float32: four entries per lane
    HotChunk<V> pre;
    HotChunk4 pre4;
    auto prefetch = [&](int32_t bb) {
        const int32_t pe0 = ((cptr)hd.bent)[bb], pes = ((cptr)hd.bsplit)[bb];
        const int32_t pe1 = ((cptr)hd.bent)[bb + 1];
        if constexpr (Q) {
            if (wave & 1)
                hot_first4<false>((const float *)pv, cold, hd.key, pes, pe1, wave, lane, pre4);
            else
                hot_first4<true>((const float *)pv, hd.rc, hd.key, pe0, pes, wave, lane, pre4);
        } else {
            if (wave & 1)
                hot_first<V, false>(pv, cold, hd.key, pes, pe1, wave, lane, pre);
            else
                hot_first<V, true>(pv, hd.rc, hd.key, pe0, pes, wave, lane, pre);
        }
    };
    // this workgroup's blocks (a static assignment balanced by work)
    const int32_t i0 = ((cptr)hd.gptr)[blockIdx.x];
    const int32_t i1 = ((cptr)hd.gptr)[blockIdx.x + 1];
    if (i0 < i1)
        prefetch(((cptr)hd.gblk)[i0]);
    for (int32_t i = i0; i < i1; ++i) {
        const int32_t b = ((cptr)hd.gblk)[i];
        const int32_t r0 = ((cptr)hd.brow)[b];
        const int32_t nr = ((cptr)hd.brow)[b + 1] - r0;
        const int32_t e0 = ((cptr)hd.bent)[b], es = ((cptr)hd.bsplit)[b];
        const int32_t e1 = ((cptr)hd.bent)[b + 1];
        __syncthreads();  // hot columns staged, sums of the last block cleared
        if constexpr (Q) {
            const float *fv = (const float *)pv;
            const float *fx = (const float *)x;
            const float *fs = (const float *)xs;
            if (wave & 1) {
                hot_part4<false, kPanelWaves, true, true>(
                    fv, cold, hd.key, es, e1, fx, acc_c, ckey + kPanelWaves + wave,
                    csum + kPanelWaves + wave, wave, lane, &pre4);
                hot_part4<true>(fv, hd.rc, hd.key, e0, es, fs, acc_h, ckey + wave,
                                csum + wave, wave, lane);
            } else {
                hot_part4<true, kPanelWaves, false, true>(fv, hd.rc, hd.key, e0, es, fs,
                                                          acc_h, ckey + wave, csum + wave,
                                                          wave, lane, &pre4);
                hot_part4<false>(fv, cold, hd.key, es, e1, fx, acc_c,
                                 ckey + kPanelWaves + wave, csum + kPanelWaves + wave,
                                 wave, lane);
            }
        } else {
            if (wave & 1) {
                hot_part<V, false, kPanelWaves, true, true>(
                    pv, cold, hd.key, es, e1, x, acc_c, ckey + kPanelWaves + wave,
                    csum + kPanelWaves + wave, wave, lane, &pre);
                hot_part<V, true>(pv, hd.rc, hd.key, e0, es, xs, acc_h, ckey + wave,
                                  csum + wave, wave, lane);
            } else {
                hot_part<V, true, kPanelWaves, false, true>(pv, hd.rc, hd.key, e0, es, xs,
                                                            acc_h, ckey + wave, csum + wave,
                                                            wave, lane, &pre);
                hot_part<V, false>(pv, cold, hd.key, es, e1, x, acc_c,
                                   ckey + kPanelWaves + wave, csum + kPanelWaves + wave,
                                   wave, lane);
            }
        }
        if (i + 1 < i1)
            prefetch(((cptr)hd.gblk)[i + 1]);
        __syncthreads();  // all runs are in
        if (wave == 0) {
            // lanes 0-15: hot slots, 16-31: cold slots.  A slot leads its
            // row if no earlier slot of its part has it; the leader adds the
            // row's carries of that part in slot order (distinct rows per part)
            const int32_t k = (lane < 2 * kPanelWaves) ? ckey[lane] : -1;
            const double c = (lane < 2 * kPanelWaves) ? csum[lane] : 0.0;
            const bool cold = lane >= kPanelWaves;
            bool lead = k >= 0;
            double t = 0.0;
            for (int j = 0; j < 2 * kPanelWaves; ++j) {
                const int32_t kj = __builtin_amdgcn_readlane(k, j);
                const double cj = readlane_f64(c, j);
                if ((j >= kPanelWaves) == cold && kj == k) {
                    if (j < lane)
                        lead = false;
                    else
                        t += cj;
                }
            }
            if (lead)
                (cold ? acc_c : acc_h)[k] += t;
        }
        __syncthreads();  // carries are in
        for (int32_t r = threadIdx.x; r < nr; r += kPanelThreads) {
            const uint16_t k = gld(hd.rmap + r0 + r);
            double sum = 0.0;
            if (k != kHotEmpty) {
                sum = acc_h[k] + acc_c[k];
                acc_h[k] = 0.0;  // the thread that reads a sum clears it
                acc_c[k] = 0.0;
            }
            const V out = epilogue<V>(sum, epi);
            gst(y + r0 + r, out);
            if (DOT)
                dacc = fma((double)gld(w + r0 + r), (double)out, dacc);
        }
    }
    if (DOT) {
        const double tot = block_sum<kPanelWaves>(dacc, csum);
        if (threadIdx.x == 0)
            dot_part[blockIdx.x] = tot;
    }
}

// xp[newid[c]] = x[c]: x in the column order of a layout.  Columns of one power
// of two of entries keep their order, so the stores of a wavefront fall on a
// few ascending streams (2^20 float32: 3 us; reading x through the inverse
// instead took 7.4).
template <typename V>
__global__ __launch_bounds__(kBlock) void k_place_cols(int32_t n,
                                                       const int32_t *__restrict__ newid,
                                                       const V *__restrict__ x,
                                                       V *__restrict__ xp)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n)
        xp[newid[i]] = gld(x + i);
}

// ------------------------------------------------------------- band

// Product over the band layout (see BandDesc): one workgroup per row block,
// its wavefronts share the block's entries evenly (a row can span them),
// gather from x starting at the block's first column, and the carries of
// rows split between wavefronts are added in slot order by one lane each.
template <typename V, bool DOT>
__device__ __forceinline__ void band_block(const BandDesc &bd, int32_t b,
                                           const V *__restrict__ x,
                                           V *__restrict__ y, const Epi &epi,
                                           const V *__restrict__ w,
                                           double *__restrict__ dot_part,
                                           unsigned char *smem)
{
    double *acc = (double *)smem;                                  // row sums
    double *csum = (double *)(smem + kBandRows * 8);               // carries
    int32_t *ckey = (int32_t *)(smem + kBandRows * 8 + kBandWaves * 8);
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int32_t r0 = gld(bd.brow + b);
    const int32_t nr = gld(bd.brow + b + 1) - r0;
    for (int32_t i = threadIdx.x; i < nr; i += kBandThreads)
        acc[i] = 0.0;
    __syncthreads();
    hot_part<V, true, kBandWaves, true>((const V *)bd.vals, bd.rc, nullptr,
                                  gld(bd.bent + b), gld(bd.bent + b + 1),
                                  x + gld(bd.cbase + b), acc, ckey + wave,
                                  csum + wave, wave, lane);
    __syncthreads();
    if (wave == 0) {
        const int32_t k = (lane < kBandWaves) ? ckey[lane] : -1;
        const double c = (lane < kBandWaves) ? csum[lane] : 0.0;
        bool lead = k >= 0;
        double t = 0.0;
        for (int j = 0; j < kBandWaves; ++j) {
            const int32_t kj = __builtin_amdgcn_readlane(k, j);
            const double cj = readlane_f64(c, j);
            if (kj == k) {
                if (j < lane)
                    lead = false;
                else
                    t += cj;
            }
        }
        if (lead)
            acc[k] += t;
    }
    __syncthreads();
    double dacc = 0.0;
    for (int32_t i = threadIdx.x; i < nr; i += kBandThreads) {
        const V out = epilogue<V>(acc[i], epi);
        gst(y + r0 + i, out);
        if (DOT)
            dacc = fma((double)gld(w + r0 + i), (double)out, dacc);
    }
    if (DOT) {
        const double tot = block_sum<kBandWaves>(dacc, csum);
        if (threadIdx.x == 0)
            dot_part[b] = tot;
    }
}

// One group of a lane's entries in a sliced block (see SellSlice): N values
// and N 16-bit column offsets, by 16-byte (8-byte) streaming loads.
template <typename V, int N> struct SellGroup;
template <> struct SellGroup<double, 4> {
    f64x2 a, b;
    u16x4 o;
    __device__ __forceinline__ void load(const double *v, const uint16_t *off, int lane)
    {
        a = ld_stream((const f64x2 *)v + lane);
        b = ld_stream((const f64x2 *)v + 64 + lane);
        o = ld_stream((const u16x4 *)off + lane);
    }
    __device__ __forceinline__ double val(int t) const
    {
        return t == 0 ? a.x : t == 1 ? a.y : t == 2 ? b.x : b.y;
    }
};
template <> struct SellGroup<float, 4> {
    f32x4 a;
    u16x4 o;
    __device__ __forceinline__ void load(const float *v, const uint16_t *off, int lane)
    {
        a = ld_stream((const f32x4 *)v + lane);
        o = ld_stream((const u16x4 *)off + lane);
    }
    __device__ __forceinline__ double val(int t) const { return (double)a[t]; }
};
template <typename V> struct SellGroup<V, 2> {
    typedef V pair_t __attribute__((ext_vector_type(2)));
    pair_t a;
    u16x2 o;
    __device__ __forceinline__ void load(const V *v, const uint16_t *off, int lane)
    {
        a = ld_stream((const pair_t *)v + lane);
        o = ld_stream((const u16x2 *)off + lane);
    }
    __device__ __forceinline__ double val(int t) const { return (double)a[t]; }
};

// The sums of a row's entries j, j + 4, ... of up to eight, together.
__device__ __forceinline__ double total4(const double (&sum)[4])
{
    return (sum[0] + sum[1]) + (sum[2] + sum[3]);
}

// Row blocks of the sliced form: a workgroup takes `spb` consecutive slices,
// its wavefronts in turn; one lane per row adds the row up in order.  No
// scan, no LDS, and neighbouring lanes gather neighbouring entries of x
// where neighbouring rows reach shifted columns (stencils), so the product
// is bound by the 10 (float32: 6) bytes per entry it streams: 27-point
// stencil of 128^3 (55.7 M entries) 105 us float64 = 5.9 TB/s of its own
// bytes (scan form: 146 us), 60.5 us float32.  Two groups of four in flight:
// one took 107 us, four 105 but 40 against 36 us on the 7-point rows (more
// registers, fewer wavefronts); ordinary loads instead of non-temporal 113.
// A row is added up eight entries at a time, in four sums each, float64 rows four
// such parts at a time: root mean square errors against exact sums of random values,
// over sum |a x|, this way, one entry after the other, and in the scan form: 27
// points 3.1e-17, 4.5e-17 and 3.3e-17, 60 entries 2.2e-17, 4.5e-17 and 2.3e-17, 200
// entries 1.5e-17, 4.5e-17 and 1.4e-17; the times are the same.
template <typename V, bool DOT>
__device__ __forceinline__ void sell_block(const BandDesc &bd, int32_t b,
                                           const V *__restrict__ x,
                                           V *__restrict__ y, const Epi &epi,
                                           const V *__restrict__ w,
                                           double *__restrict__ dot_part, double *lds)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int32_t s1 = min((b + 1) * bd.spb, bd.nslice);
    double dacc = 0.0;
    for (int32_t s = b * bd.spb + wave; s < s1; s += kBandWaves) {
        const i32x4 sl = *(const __attribute__((address_space(4))) i32x4 *)(bd.slice + s);
        const int32_t wmin = sl.z, wmax = sl.w;
        const int32_t row = s * 64 + lane;
        const V *pv = (const V *)bd.vals + (int64_t)sl.x * 64;
        const uint16_t *po = bd.off + (int64_t)sl.x * 64;
        const V *xb = x + sl.y;
        const int32_t nq = wmax >> 2;
        // the entries past the groups of four are requested first
        SellGroup<V, 2> pr;
        V v1 = (V)0;
        uint16_t o1 = 0;
        const int32_t tail = wmax & ~3;
        if (wmax & 2)
            pr.load(pv + tail * 64, po + tail * 64, lane);
        if (wmax & 1) {
            v1 = ld_stream(pv + (wmax - 1) * 64 + lane);
            o1 = ld_stream(po + (wmax - 1) * 64 + lane);
        }
        int32_t len = wmax;
        if (wmin < wmax)
            len = (row < bd.rows) ? gld(bd.row_ptr + row + 1) - gld(bd.row_ptr + row) : 0;
        double acc = 0.0, all = 0.0;   // of 32 entries, of those before them
        double sum[4];
        auto clear = [&]() { sum[0] = sum[1] = sum[2] = sum[3] = 0.0; };
        auto add = [&](int32_t j, int u, double v, double xv) {
            if (j < len)
                sum[u] = fma(v, xv, sum[u]);
        };
        int32_t q = 0;
        for (; q + 2 <= nq; q += 2) {
            SellGroup<V, 4> g[2];
            V xv[8];
#pragma unroll
            for (int u = 0; u < 2; ++u)
                g[u].load(pv + (q + u) * 256, po + (q + u) * 256, lane);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    xv[u * 4 + t] = gld(xb + g[u].o[t]);
            clear();
            if (q * 4 + 8 <= wmin) {
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    sum[t & 3] = fma(g[t >> 2].val(t & 3), (double)xv[t], sum[t & 3]);
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    add(q * 4 + t, t & 3, g[t >> 2].val(t & 3), (double)xv[t]);
            }
            acc += total4(sum);
            if (sizeof(V) == 8 && (q & 6) == 6) {
                all += acc;
                acc = 0.0;
            }
        }
        clear();
        if (q < nq) {
            SellGroup<V, 4> g;
            V xv[4];
            g.load(pv + q * 256, po + q * 256, lane);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                xv[t] = gld(xb + g.o[t]);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                add(q * 4 + t, t, g.val(t), (double)xv[t]);
        }
        if (wmax & 2) {
            const V xa = gld(xb + pr.o.x), xc = gld(xb + pr.o.y);
            add(tail, 0, pr.val(0), (double)xa);
            add(tail + 1, 1, pr.val(1), (double)xc);
        }
        if (wmax & 1)
            add(wmax - 1, 2, (double)v1, (double)gld(xb + o1));
        if (row < bd.rows) {
            const V out = epilogue<V>(all + (acc + total4(sum)), epi);
            gst(y + row, out);
            if (DOT)
                dacc = fma((double)gld(w + row), (double)out, dacc);
        }
    }
    if (DOT) {
        const double tot = block_sum<kBandWaves>(dacc, lds);
        if (threadIdx.x == 0)
            dot_part[b] = tot;
    }
}

// Row block of the i-th of n workgroups: the workgroups i, i + 8, ... share
// an XCD and take neighbouring blocks, so that the x a block shares with its
// neighbours is read into that XCD's L2 once.
__device__ __forceinline__ int32_t xcd_block(int32_t i, int32_t n)
{
    const int32_t per = n >> 3;
    return (i < per * 8) ? (i & 7) * per + (i >> 3) : i;
}

template <typename V, bool DOT>
__global__ __launch_bounds__(kBandThreads) void k_spmv_sell(
    BandDesc bd, const V *__restrict__ x, V *__restrict__ y, Epi epi,
    const V *__restrict__ w, double *__restrict__ dot_part)
{
    __shared__ double lds[kBandWaves];
    sell_block<V, DOT>(bd, xcd_block(blockIdx.x, bd.nblk), x, y, epi, w, dot_part, lds);
}

template <typename V, bool DOT>
__global__ __launch_bounds__(kBandThreads) void k_spmv_band(
    BandDesc bd, const V *__restrict__ x, V *__restrict__ y, Epi epi,
    const V *__restrict__ w, double *__restrict__ dot_part)
{
    __shared__ __align__(16) unsigned char smem[kBandLds];
    band_block<V, DOT>(bd, blockIdx.x, x, y, epi, w, dot_part, smem);
}

// Band products of many matrices in one launch: workgroup g takes row
// block g - prefix[j] of matrix j, exactly as its single launch does.
template <typename V>
__global__ __launch_bounds__(kBandThreads) void k_spmv_band_grouped(
    const BandDesc *__restrict__ descs, const PanelIO *__restrict__ io,
    const int32_t *__restrict__ prefix, int32_t nmat)
{
    __shared__ __align__(16) unsigned char smem[kBandLds];
    const int32_t g = blockIdx.x;
    int32_t lo = 0, hi = nmat - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= g)
            lo = mid;
        else
            hi = mid - 1;
    }
    const BandDesc bd = descs[lo];
    const Epi epi{EPI_NONE, 0, 0.0, 0.0};
    const PanelIO bio = io[lo];
    if (bd.nslice > 0) {
        const int32_t b = g - prefix[lo];
        if constexpr (sizeof(V) == 8) {
            if (bio.dot) {
                sell_block<V, true>(bd, b, (const V *)bio.x, (V *)bio.y, epi,
                                    (const V *)bio.x, bio.dot, (double *)smem);
                return;
            }
        }
        sell_block<V, false>(bd, b, (const V *)bio.x, (V *)bio.y, epi, nullptr, nullptr,
                             (double *)smem);
        return;
    }
    if constexpr (sizeof(V) == 8) {
        if (bio.dot) {
            band_block<V, true>(bd, g - prefix[lo], (const V *)bio.x, (V *)bio.y, epi,
                                (const V *)bio.x, bio.dot, smem);
            return;
        }
    }
    band_block<V, false>(bd, g - prefix[lo], (const V *)bio.x, (V *)bio.y, epi,
                         nullptr, nullptr, smem);
}

// Smallest and largest column of every row (INT_MAX / -1 for empty rows).
__global__ __launch_bounds__(kBlock) void k_row_span(int32_t rows,
                                                     const int32_t *__restrict__ rp,
                                                     const int32_t *__restrict__ col,
                                                     int32_t *__restrict__ lo,
                                                     int32_t *__restrict__ hi)
{
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= rows)
        return;
    int32_t a = INT_MAX, z = -1;
    for (int32_t k = rp[i]; k < rp[i + 1]; ++k) {
        a = min(a, col[k]);
        z = max(z, col[k]);
    }
    lo[i] = a;
    hi[i] = z;
}

// Band words of every entry: (row in block << 16) | (col - block's base).
__global__ __launch_bounds__(kBlock) void k_band_pack(BandDesc bd,
                                                      const int32_t *__restrict__ rp,
                                                      const int32_t *__restrict__ col,
                                                      uint32_t *__restrict__ rc)
{
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= bd.rows)
        return;
    int32_t lo = 0, hi = bd.nblk - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (bd.brow[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    const uint32_t rl = (uint32_t)(i - bd.brow[lo]);
    const int32_t base = bd.cbase[lo];
    for (int32_t k = rp[i]; k < rp[i + 1]; ++k)
        rc[k] = (rl << 16) | (uint32_t)(col[k] - base);
}

// Column span and row lengths of every slice of 64 rows: one wavefront per
// slice, its entries read in order.
__global__ __launch_bounds__(kBlock) void k_slice_span(int32_t rows,
                                                       const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ col,
                                                       int32_t nslice,
                                                       i32x4 *__restrict__ out)
{
    const int32_t s = blockIdx.x * kWaves + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (s >= nslice)
        return;  // whole wavefronts
    const int64_t row = (int64_t)s * 64 + lane;
    const int32_t a = rp[min(row, (int64_t)rows)], z = rp[min(row + 1, (int64_t)rows)];
    const int32_t k0 = __shfl(a, 0, 64), k1 = __shfl(z, 63, 64);
    int32_t lo = INT_MAX, hi = -1;
    constexpr int U = 8;   // loads in flight
    for (int64_t k = (int64_t)k0 + lane; k < k1; k += 64 * U) {
        int32_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            c[u] = col[min(k + 64 * u, (int64_t)k1 - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lo = min(lo, c[u]);
            hi = max(hi, c[u]);
        }
    }
    const int32_t wmax = lane_group_max<64>(z - a);
    const int32_t wmin = -lane_group_max<64>(a - z);
    lo = -lane_group_max<64>(-lo);
    hi = lane_group_max<64>(hi);
    if (lane == 0)
        out[s] = i32x4{lo, hi, wmin, wmax};
}

// Place of entry j of lane l in a slice (see SellSlice): values (VV to a
// 16-byte load) and offsets.
template <int VV>
__device__ __forceinline__ int64_t sell_value_at(const i32x4 &sl, int32_t j, int32_t l)
{
    const int32_t w = sl.w, full = w & ~3;
    if (j < full)
        return VV == 4 ? ((int64_t)sl.x + (j & ~3)) * 64 + l * 4 + (j & 3)
                       : ((int64_t)sl.x + (j & ~1)) * 64 + l * 2 + (j & 1);
    if ((w & 2) && j < full + 2)
        return ((int64_t)sl.x + full) * 64 + l * 2 + (j - full);
    return ((int64_t)sl.x + j) * 64 + l;
}

// Fills the sliced form: one wavefront per slice reads its entries in order
// and writes each to its place; then every lane pads its row.
template <typename V>
__global__ __launch_bounds__(kBlock) void k_sell_pack(BandDesc bd,
                                                      const int32_t *__restrict__ col,
                                                      const V *__restrict__ vals,
                                                      V *__restrict__ sv,
                                                      uint16_t *__restrict__ so)
{
    __shared__ int32_t starts[kWaves][65];
    constexpr int VV = 16 / sizeof(V);
    const int wave = threadIdx.x >> 6;
    const int32_t s = blockIdx.x * kWaves + wave;
    const int lane = threadIdx.x & 63;
    const bool on = s < bd.nslice;
    const int64_t row = (int64_t)s * 64 + lane;
    const int64_t rows = bd.rows;
    const int32_t a = on ? bd.row_ptr[min(row, rows)] : 0;
    const int32_t z = on ? bd.row_ptr[min(row + 1, rows)] : 0;
    int32_t *st = starts[wave];
    st[lane] = a;
    if (lane == 63)
        st[64] = z;
    __syncthreads();
    if (!on)
        return;
    const i32x4 sl = *(const i32x4 *)(bd.slice + s);
    const int32_t k0 = st[0], k1 = st[64];
    constexpr int U = 8;   // loads in flight
    for (int64_t kb = (int64_t)k0 + lane; kb < k1; kb += 64 * U) {
        V v[U];
        int32_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = min(kb + 64 * u, (int64_t)k1 - 1);
            v[u] = vals[k];
            c[u] = col[k];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = kb + 64 * u;
            if (k >= k1)
                break;
            int32_t lo = 0, hi = 63;   // the last row that starts at or before k
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) >> 1;
                if (st[mid] <= k)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            const int32_t j = (int32_t)(k - st[lo]);
            sv[sell_value_at<VV>(sl, j, lo)] = v[u];
            so[sell_value_at<4>(sl, j, lo)] = (uint16_t)(c[u] - sl.y);
        }
    }
    for (int32_t j = z - a; j < sl.w; ++j) {
        sv[sell_value_at<VV>(sl, j, lane)] = (V)0;
        so[sell_value_at<4>(sl, j, lane)] = 0;
    }
}

// The rows of a workgroup of the two kernels below: 64 consecutive ones, whose
// entries follow one another, less those of more than `most` entries; or (long
// rows, `list` given) one such row alone, so that no workgroup has much more
// than the others.
struct HotRows {
    int64_t row;      // this lane's row (rows: none)
    int32_t a, z;     // its entries
    __device__ __forceinline__ HotRows(int32_t rows, const int32_t *__restrict__ rp,
                                       const int32_t *__restrict__ list)
    {
        const int lane = threadIdx.x & 63;
        row = list ? (int64_t)list[blockIdx.x] + (lane ? rows : 0)
                   : (int64_t)blockIdx.x * 64 + lane;
        row = min(row, (int64_t)rows);
        if (list && lane) {
            a = z = rp[list[blockIdx.x] + 1];
        } else {
            a = rp[row];
            z = rp[min(row + 1, (int64_t)rows)];
        }
    }
};

// Hot entries of each row, 64 entries to a wavefront at a time; lane l counts
// the hot ones among those that are its row's.
__global__ __launch_bounds__(kBlock) void k_hot_count(HotDesc hd,
                                                      const int32_t *__restrict__ rp,
                                                      const int32_t *__restrict__ col,
                                                      const int32_t *__restrict__ list,
                                                      int32_t most, int32_t *__restrict__ cnt)
{
    __shared__ int32_t sum[64];
    constexpr int U = 4;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const HotRows R(hd.rows, rp, list);
    if (threadIdx.x < 64)
        sum[threadIdx.x] = 0;
    __syncthreads();
    const int32_t *newid = hd.newid;
    uint64_t skip = list ? 0ull : __ballot(R.z - R.a > most);   // the long rows
    int32_t n = 0;
    int64_t k0 = __builtin_amdgcn_readlane(R.a, 0);
    const int64_t last = __builtin_amdgcn_readlane(R.z, 63);
    for (;;) {
        // entries up to the next long row
        const int l = skip ? __builtin_ctzll(skip) : 64;
        const int64_t k1 = l < 64 ? __builtin_amdgcn_readlane(R.a, l & 63) : last;
        for (int64_t kb = k0 + wave * 64 * U; kb < k1; kb += kBlock * U) {
            int32_t c[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                c[u] = col[min(kb + u * 64 + lane, k1 - 1)];
            if (newid) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    c[u] = newid[c[u]];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t base = kb + u * 64;
                const uint64_t m = __ballot(base + lane < k1 && c[u] < hd.hot);
                const int64_t lo = max(R.a - base, (int64_t)0), hi = min(R.z - base, (int64_t)64);
                if (lo < hi) {
                    const uint64_t upto = hi == 64 ? ~0ull : (1ull << hi) - 1ull;
                    n += __popcll(m & upto & ~((1ull << lo) - 1ull));
                }
            }
        }
        if (l == 64)
            break;
        k0 = __builtin_amdgcn_readlane(R.z, l & 63);
        skip &= skip - 1;
    }
    if (n)
        atomicAdd(&sum[lane], n);
    __syncthreads();
    if (threadIdx.x < 64 && R.row < hd.rows && (list ? lane == 0 : R.z - R.a <= most))
        cnt[R.row] = sum[threadIdx.x];
}

// 1 for a row with entries, 0 for an empty one (and past the last row).
__global__ __launch_bounds__(kBlock) void k_row_filled(int32_t rows,
                                                       const int32_t *__restrict__ rp,
                                                       int32_t *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i <= rows)
        out[i] = (i < rows && rp[i + 1] > rp[i]) ? 1 : 0;
}

// Block bounds of the hot-column layout.  Wavefront g cuts rows [g * part, (g +
// 1) * part): a block ends before the row that would be its keys + 1st
// non-empty one, or where it has `target` entries or kHotSpan rows.  Each test,
// once true, stays true along the rows, so the end is found in three steps of
// up to 64 rows each.  out[g * cap]: the number of blocks, then first row and
// first entry of each.  A chain of loads, 0.2 ms: several rules (blockIdx.y) are
// tried at once.
__global__ __launch_bounds__(64) void k_hot_blocks(int32_t rows, const int32_t *__restrict__ rp,
                                                   const int32_t *__restrict__ filled,
                                                   int32_t part, HotTries tries, int32_t cap,
                                                   int32_t *__restrict__ out)
{
    constexpr int32_t S1 = kHotSpan / 64, S2 = S1 / 64;
    static_assert(S2 * 64 * 64 == kHotSpan && S2 <= 64, "steps of the search");
    const int lane = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * part;
    const int32_t end = (int32_t)min(r0 + part, (int64_t)rows);
    const int32_t keys = tries.keys[blockIdx.y], target = tries.target[blockIdx.y];
    int32_t *o = out + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * cap;
    int32_t start = (int32_t)r0, n = 0;
    while (start < end) {
        const int32_t f0 = filled[start], e0 = rp[start];
        if (lane == 0 && 2 * n + 2 < cap) {
            o[1 + 2 * n] = start;
            o[2 + 2 * n] = e0;
        }
        ++n;
        // the first lane whose row r ends a block that starts here
        auto first = [&](int64_t r) {
            const bool ends = r >= end || r - start >= kHotSpan || filled[r + 1] - f0 > keys ||
                              (int64_t)rp[r] - e0 >= target;
            return (int64_t)__builtin_ctzll(__ballot(ends) | 1ull << 63);
        };
        int64_t at = start;
        at += first(at + (int64_t)(lane + 1) * S1) * S1;
        at += first(at + (int64_t)(lane + 1) * S2) * S2;
        at += first(at + min(lane, S2 - 1) + 1) + 1;
        start = (int32_t)min(at, (int64_t)end);
    }
    if (lane == 0)
        o[0] = n;
}

// Keys: the number of a row among the non-empty rows of its block.  filled:
// exclusive scan of k_row_filled.
__global__ __launch_bounds__(kBlock) void k_hot_rmap(HotDesc hd,
                                                     const int32_t *__restrict__ filled,
                                                     uint16_t *__restrict__ rmap)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= hd.rows)
        return;
    int32_t lo = 0, hi = hd.nblk - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (hd.brow[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    rmap[i] = filled[i + 1] > filled[i] ? (uint16_t)(filled[i] - filled[hd.brow[lo]])
                                        : kHotEmpty;
}

// out[0] += entries k = 0, step, 2 step, ... whose column's newid is below hot.
__global__ __launch_bounds__(kBlock) void k_hot_share(int64_t nnz, int32_t step,
                                                      const int32_t *__restrict__ col,
                                                      const int32_t *__restrict__ newid,
                                                      int32_t hot, int32_t *__restrict__ out)
{
    int32_t n = 0;
    for (int64_t k = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * step; k < nnz;
         k += (int64_t)gridDim.x * kBlock * step)
        n += newid[col[k]] < hot ? 1 : 0;
    n = wave_sum_i32(n);
    __shared__ int32_t red[kWaves];
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kWaves; ++i)
            n += red[i];
        atomicAdd(out, n);
    }
}

// 1 for a column below hot, else 0 (and past the last one).
__global__ __launch_bounds__(kBlock) void k_hot_flag(int32_t n, const int32_t *__restrict__ newid,
                                                     int32_t hot, int32_t *__restrict__ flag)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i <= n)
        flag[i] = (i < n && newid[i] < hot) ? 1 : 0;
}

// The columns below hot renumbered in the caller's order, from the exclusive scan
// of their flags: 64 consecutive ones then lie near each other in x (and the
// order inside the LDS does not matter).  old: the inverse of that part.
__global__ __launch_bounds__(kBlock) void k_hot_order(int32_t n, int32_t hot,
                                                      const int32_t *__restrict__ before,
                                                      int32_t *__restrict__ newid,
                                                      int32_t *__restrict__ old)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n && newid[i] < hot) {
        newid[i] = before[i];
        old[before[i]] = (int32_t)i;
    }
}

__global__ __launch_bounds__(kBlock) void k_hot_split(HotDesc hd,
                                                      const int32_t *__restrict__ hx,
                                                      int32_t *__restrict__ bsplit)
{
    const int32_t b = blockIdx.x * kBlock + threadIdx.x;
    if (b >= hd.nblk)
        return;
    bsplit[b] = hd.bent[b] + (hx[hd.brow[b + 1]] - hx[hd.brow[b]]);
}

// Moves the entries to the hot or cold part of their row's block, in their
// order, 256 entries at a time; an entry's place follows from the hot entries
// before it in the matrix: hx (the exclusive scan of the rows' counts) where
// the workgroup's entries begin, plus those it has met.
template <typename V>
__global__ __launch_bounds__(kBlock) void k_hot_scatter(
    HotDesc hd, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const V *__restrict__ vals, const int32_t *__restrict__ list, int32_t most,
    const int32_t *__restrict__ hx, V *__restrict__ hv, uint32_t *__restrict__ hrc,
    uint16_t *__restrict__ hkey, uint32_t *__restrict__ hcold)
{
    // per row: first entry, what a hot (cold) entry's place adds to the hot
    // (cold) entries before it in the matrix, key
    __shared__ int32_t st[64], to_hot[64], to_cold[64];
    __shared__ uint16_t key[64];
    constexpr int U = 4;
    __shared__ int32_t tot[U * kWaves];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const HotRows R(hd.rows, rp, list);
    if (wave == 0) {
        st[lane] = R.a;
        if (R.row < hd.rows) {
            int32_t lo = 0, hi = hd.nblk - 1;   // the last block that starts at or before it
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) >> 1;
                if (hd.brow[mid] <= R.row)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            const int32_t before = hd.bent[lo] - hx[hd.brow[lo]];   // cold ones before it
            to_hot[lane] = before;
            to_cold[lane] = hd.bsplit[lo] - before;
            key[lane] = hd.rmap[R.row];
        }
    }
    __syncthreads();
    const int32_t *newid = hd.newid;
    const int32_t hot_at = hx[R.row];   // hot entries before this lane's row
    uint64_t skip = list ? 0ull : __ballot(R.z - R.a > most);   // the long rows
    int64_t k0 = __builtin_amdgcn_readlane(R.a, 0);
    int32_t done = __builtin_amdgcn_readlane(hot_at, 0);   // hot entries before kb
    const int64_t last = __builtin_amdgcn_readlane(R.z, list ? 0 : 63);
    for (;;) {
        // entries up to the next long row
        const int l = skip ? __builtin_ctzll(skip) : 64;
        const int64_t k1 = l < 64 ? __builtin_amdgcn_readlane(R.a, l & 63) : last;
        for (int64_t kb = k0; kb < k1; kb += kBlock * U) {
            int32_t own[U], c[U];   // the caller's column, the layout's
            V v[U];
            uint64_t m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t k = min(kb + u * kBlock + threadIdx.x, k1 - 1);
                c[u] = own[u] = col[k];
                v[u] = vals[k];
            }
            if (newid) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    c[u] = newid[c[u]];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                m[u] = __ballot(kb + u * kBlock + threadIdx.x < k1 && c[u] < hd.hot);
                if (lane == 0)
                    tot[u * kWaves + wave] = __popcll(m[u]);
            }
            __syncthreads();
            int32_t before = done;
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    if (w == wave) {
                        const int64_t k = kb + u * kBlock + threadIdx.x;
                        const int32_t hot = before + lanes_below(m[u]);
                        if (k < k1) {
                            int32_t lo = 0, hi = 63;   // the last row that starts at or before k
                            while (lo < hi) {
                                const int32_t mid = (lo + hi + 1) >> 1;
                                if (st[mid] <= k)
                                    lo = mid;
                                else
                                    hi = mid - 1;
                            }
                            if (c[u] < hd.hot) {
                                const int64_t at = (int64_t)to_hot[lo] + hot;
                                hv[at] = v[u];
                                hrc[at] = ((uint32_t)key[lo] << 16) | (uint32_t)c[u];
                            } else {
                                const int64_t at = (int64_t)to_cold[lo] + (k - hot);
                                hv[at] = v[u];
                                hrc[at] = (uint32_t)c[u];
                                hkey[at] = key[lo];
                                if (hcold)
                                    hcold[at] = (uint32_t)own[u];
                            }
                        }
                    }
                    before += tot[u * kWaves + w];
                }
            }
            done = before;
            __syncthreads();   // tot is read
        }
        if (l == 64)
            break;
        k0 = __builtin_amdgcn_readlane(R.z, l & 63);
        done = l < 63 ? __builtin_amdgcn_readlane(hot_at, (l + 1) & 63) : done;
        skip &= skip - 1;
    }
}

// ------------------------------------------------------------------ BFS

// Start: level -1 but 0 at the source, the first two frontier bitmaps, last =
// 0, and the rows still to decide: a bit for every row of 1 to kBfsShort
// entries but the source.
__global__ __launch_bounds__(kBlock) void k_bfs_init(int32_t rows, int32_t source,
                                                     const int32_t *__restrict__ rp,
                                                     int32_t *__restrict__ level,
                                                     uint32_t *__restrict__ bits, int32_t words,
                                                     uint64_t *__restrict__ todo,
                                                     int32_t *__restrict__ last)
{
    const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    // whole wavefronts: 64 consecutive rows to a word
    for (int64_t i = tid; i < (((int64_t)rows + 63) & ~(int64_t)63); i += stride) {
        const bool in = i < rows;
        const int32_t n = in ? rp[i + 1] - rp[i] : 0;
        if (in)
            level[i] = (i == source) ? 0 : -1;
        const uint64_t m = __ballot(n > 0 && n <= kBfsShort && i != source);
        if ((threadIdx.x & 63) == 0)
            todo[i >> 6] = m;
    }
    for (int64_t i = tid; i < 2 * (int64_t)words; i += stride)
        bits[i] = (i == (source >> 5)) ? 1u << (source & 31) : 0u;
    if (tid == 0)
        *last = 0;
}

// The frontier as a wavefront sees it: a bit per vertex, in LDS or (LDS = false)
// in device memory.
template <bool LDS>
struct Frontier {
    const uint32_t *bits;
    __device__ __forceinline__ bool has(int32_t v) const
    {
        const uint32_t i = (uint32_t)v;
        return ((LDS ? bits[i >> 5] : gld(bits + (i >> 5))) >> (i & 31)) & 1u;
    }
};

// Whether entries [k0, k1) hold a column of the frontier, W lanes for each row
// (all with the row's bounds), U * W entries at a time; true in every lane of a
// row that has one.  All 64 lanes call it.
template <int W, int U, bool LDS>
__device__ __forceinline__ bool bfs_hit(const int32_t *__restrict__ col, int32_t k0, int32_t k1,
                                        const Frontier<LDS> &f)
{
    const int wl = threadIdx.x & 63;
    constexpr uint64_t ones = W == 64 ? ~0ull : (1ull << (W & 63)) - 1ull;
    const uint64_t group = ones << (wl / W * W);
    bool hit = false, on = k0 < k1;
    // the trips of the wavefront's longest row; a row stops at its own end
    for (int32_t k = k0; __ballot(on); k += U * W) {
        int32_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            c[u] = on ? gld(col + min(k + wl % W + u * W, k1 - 1)) : 0;
        if (on) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                hit = f.has(c[u]) || hit;
        }
        hit = (__ballot(hit) & group) != 0;
        on = on && !hit && k + U * W < k1;
    }
    return hit;
}

// The rows of a wavefront's 64 that `want` names (lane l holds the bounds of
// the l-th), 64 / W at a time; returns the mask of those with a hit.
template <int W, int U, bool LDS>
__device__ __forceinline__ uint64_t bfs_rows(const int32_t *__restrict__ col, int32_t k0,
                                             int32_t k1, uint64_t want,
                                             const Frontier<LDS> &f)
{
    if (!want)
        return 0;
    const int wl = threadIdx.x & 63;
    const bool on = (want >> wl) & 1u;
    if (W == 1)
        return __ballot(bfs_hit<W, U, LDS>(col, k0, on ? k1 : k0, f));
    const int32_t n = __popcll(want);
    // wanted rows to the first lanes (the others go where nobody looks)
    const int32_t rank = on ? lanes_below(want) : n + lanes_below(~want);
    const int32_t a = __builtin_amdgcn_ds_permute(rank * 4, k0);
    const int32_t z = __builtin_amdgcn_ds_permute(rank * 4, k1);
    bool mine = false;
    for (int32_t i = 0; i < n; i += 64 / W) {
        const int src = min(i + wl / W, 63);
        // by all lanes: the lane that is read has to take part
        const int32_t ra = __shfl(a, src, 64), rz = __shfl(z, src, 64);
        const int hit = bfs_hit<W, U, LDS>(col, ra, i + wl / W < n ? rz : ra, f);
        // back to the row's own lane
        const int32_t at = rank - i;
        const int h = __shfl(hit, (at >= 0 && at < 64 / W) ? at * W : wl, 64);
        mine = mine || (at >= 0 && at < 64 / W && h);
    }
    return __ballot(on && mine);
}

// One level: every row without a level that has a column in the frontier
// (bitmap depth % 3) gets depth + 1 and its bit in bitmap (depth + 1) % 3; the
// third one is cleared for the level after.  Nothing is done once a level
// found nothing (last < depth), so several levels can be enqueued at once.
// Columns are tested against a copy of the frontier in LDS where it fits (1.3M
// vertices), else in device memory: a bit per vertex instead of a gather of a
// 4-byte level, which the caches serve at one line per 4.7 clocks and CU.  Larger
// frontiers by one LDS part after the other read every column again for each
// part: 2^21 vertices, 32M edges, 413 us by two parts and 360 from memory; 2^22
// with 16M edges, four parts, 1068 and 357; a 7-point stencil of 160^3 (478
// levels) 83.5 and 16.2 ms.
// The chunks of split rows and the nlong rows before them in the class order
// (all of more than kBfsShort entries) go 64 to a wavefront.  The others go 64 consecutive rows to a
// wavefront, which owns their word of `todo`: what is decided or empty costs a
// bit.  R-MAT 2^20, 16 M entries: 47 + 37 us for the two levels that look at
// every entry and 15 us for each late one with tiles for all rows; 43 + 36 and
// 8 to 12 us with the words (140 us for the call of six levels).
template <bool LDS>
__global__ __launch_bounds__(kBfsThreads) void k_bfs_step(
    MatDesc m, int32_t nchunk, int32_t nlong, int32_t rows,
    int32_t *__restrict__ level, int32_t depth, uint32_t *__restrict__ bits, int32_t words,
    uint64_t *__restrict__ todo, int32_t *__restrict__ last)
{
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *fb = (uint32_t *)smem;
    if (__hip_atomic_load(last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < depth)
        return;
    const uint32_t *cur = bits + (int64_t)(depth % 3) * words;
    uint32_t *next = bits + (int64_t)((depth + 1) % 3) * words;
    uint32_t *clear = bits + (int64_t)((depth + 2) % 3) * words;
    const int64_t tid = (int64_t)blockIdx.x * kBfsThreads + threadIdx.x;
    for (int64_t i = tid; i < words; i += (int64_t)gridDim.x * kBfsThreads)
        clear[i] = 0u;
    const int lane = threadIdx.x & 63;
    const int32_t waves = (int32_t)gridDim.x * (kBfsThreads / 64);
    // wavefronts of one workgroup take rows far apart (longest come first)
    const int32_t w0 = __builtin_amdgcn_readfirstlane(
        (int32_t)(threadIdx.x >> 6) * (int32_t)gridDim.x + (int32_t)blockIdx.x);
    const int32_t groups = (int32_t)(((int64_t)rows + 63) >> 6);
    bool any = false;
    if (LDS) {
        for (int32_t i = threadIdx.x * 4; i < words; i += kBfsThreads * 4)
            *(i32x4 *)(fb + i) = gld((const i32x4 *)(cur + i));
        __syncthreads();
    }
    const Frontier<LDS> f{LDS ? fb : cur};
    for (int32_t i0 = w0; i0 < nchunk + nlong; i0 += waves * 64) {
        // row and bounds of this wavefront's next 64 long rows and chunks
        const int64_t i = (int64_t)i0 + (int64_t)lane * waves;
        int32_t row = 0, k0 = 0, k1 = 0;
        if (i < nchunk) {
            row = gld(m.c_row + i);
            k0 = gld(m.c_k0 + i);
            k1 = gld(m.c_k1 + i);
        } else if (i < nchunk + nlong) {
            row = gld(m.bin_rows + m.split_begin - 1 - (i - nchunk));
            k0 = gld(m.row_ptr + row);
            k1 = gld(m.row_ptr + row + 1);
            if (k1 - k0 <= kBfsShort)
                k1 = k0;   // its class reaches below: the row is in todo
        }
        const int32_t n = (k0 < k1 && gld(level + row) == -1) ? k1 - k0 : 0;
        uint64_t found = bfs_rows<32, 8, LDS>(m.col, k0, k1, __ballot(n > 0 && n <= 512), f);
        found |= bfs_rows<64, 8, LDS>(m.col, k0, k1, __ballot(n > 512), f);
        if (found) {
            any = true;
            if ((found >> lane) & 1u) {
                level[row] = depth + 1;
                atomicOr(&next[row >> 5], 1u << (row & 31));
            }
        }
    }
    for (int32_t g0 = w0; g0 < groups; g0 += waves * 64) {
        // the words of this wavefront's next 64 groups
        const int64_t gl = (int64_t)g0 + (int64_t)lane * waves;
        const uint64_t word = gl < groups ? todo[gl] : 0;
        uint64_t live = __ballot(word != 0);
        // bounds of the next group's rows, asked for one group ahead
        int32_t nk0 = 0, nk1 = 0;
        auto request = [&]() {
            const int64_t g = (int64_t)g0 + (int64_t)__builtin_ctzll(live) * waves;
            const int64_t row = min(g * 64 + lane, (int64_t)rows - 1);
            nk0 = gld(m.row_ptr + row);
            nk1 = gld(m.row_ptr + row + 1);
        };
        if (live)
            request();
        while (live) {
            const int l = __builtin_ctzll(live);
            live &= live - 1;
            const int32_t g = g0 + l * waves;
            const int32_t k0 = nk0, k1 = nk1;
            if (live)
                request();
            const uint64_t want =
                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(word >> 32), l) << 32) |
                (uint32_t)__builtin_amdgcn_readlane((int)word, l);
            const int32_t row = g * 64 + lane;   // of this matrix where `want` says so
            const bool on = (want >> lane) & 1u;
            const int32_t n = on ? k1 - k0 : 0;
            uint64_t found = bfs_rows<1, 4, LDS>(m.col, k0, k1, __ballot(n > 0 && n <= 4), f);
            found |= bfs_rows<4, 8, LDS>(m.col, k0, k1, __ballot(n > 4 && n <= 32), f);
            found |= bfs_rows<16, 8, LDS>(m.col, k0, k1, __ballot(n > 32), f);
            if (found) {
                any = true;
                if ((found >> lane) & 1u)
                    level[row] = depth + 1;
                if (lane == 0) {
                    atomicAnd((unsigned long long *)&todo[g], ~(unsigned long long)found);
                    // its two words of the frontier hold long rows too
                    if ((uint32_t)found)
                        atomicOr(&next[2 * g], (uint32_t)found);
                    if (found >> 32)
                        atomicOr(&next[2 * g + 1], (uint32_t)(found >> 32));
                }
            }
        }
    }
    if (any && lane == 0)
        *last = depth + 1;
}

// The deepest level found so far, to the host.
__global__ void k_bfs_report(const int32_t *__restrict__ last, int32_t *host)
{
    *host = *last;
}

// --------------------------------------------------- graph relabelling

__global__ __launch_bounds__(kBlock) void k_count_cols(int64_t nnz, int32_t step,
                                                       const int32_t *__restrict__ col,
                                                       int32_t *__restrict__ deg)
{
    for (int64_t k = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * step; k < nnz;
         k += (int64_t)gridDim.x * kBlock * step)
        atomicAdd(&deg[col[k]], 1);
}

// key 0 holds the largest degrees (2^31..), key 31 degree 1, key 32 degree 0
__global__ __launch_bounds__(kBlock) void k_degree_keys(int32_t n,
                                                        const int32_t *__restrict__ deg,
                                                        int32_t *__restrict__ key)
{
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) {
        const int32_t d = deg[i];
        key[i] = (d <= 0) ? 32 : __clz(d);
    }
}

__global__ __launch_bounds__(kBlock) void k_key_hist(int32_t n,
                                                     const int32_t *__restrict__ key,
                                                     int32_t *__restrict__ hist,
                                                     int32_t nblk)
{
    __shared__ int32_t cnt[kDegKeys];
    if (threadIdx.x < kDegKeys)
        cnt[threadIdx.x] = 0;
    __syncthreads();
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n)
        atomicAdd(&cnt[key[i]], 1);
    __syncthreads();
    if (threadIdx.x < kDegKeys)
        hist[threadIdx.x * nblk + blockIdx.x] = cnt[threadIdx.x];
}

// Stable placement by key (same scheme as the row-class scatter).
__global__ __launch_bounds__(kBlock) void k_key_scatter(int32_t n,
                                                        const int32_t *__restrict__ key,
                                                        const int32_t *__restrict__ hist,
                                                        int32_t nblk,
                                                        int32_t *__restrict__ newid)
{
    __shared__ int32_t wcnt[kWaves][kDegKeys];
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int32_t c = (i < n) ? key[i] : -1;
    const unsigned long long below = (lane == 0) ? 0ull : ((1ull << lane) - 1ull);
    int32_t rank = 0;
    for (int b = 0; b < kDegKeys; ++b) {
        const unsigned long long m = __ballot(c == b);
        if (lane == 0)
            wcnt[wave][b] = __popcll(m);
        if (c == b)
            rank = __popcll(m & below);
    }
    __syncthreads();
    if (c >= 0) {
        int32_t off = hist[c * nblk + blockIdx.x];
        for (int w = 0; w < wave; ++w)
            off += wcnt[w][c];
        newid[i] = off + rank;
    }
}

__global__ __launch_bounds__(kBlock) void k_perm_lengths(int32_t rows,
                                                         const int32_t *__restrict__ rp,
                                                         const int32_t *__restrict__ newid,
                                                         int32_t *__restrict__ len2)
{
    const int32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v < rows)
        len2[newid[v]] = rp[v + 1] - rp[v];
    else if (v == rows)
        len2[rows] = 0;
}

// One thread per entry: its row by binary search in row_ptr.
template <typename V>
__global__ __launch_bounds__(kBlock) void k_perm_entries(
    int32_t rows, int64_t nnz, const int32_t *__restrict__ rp,
    const int32_t *__restrict__ col, const V *__restrict__ vals,
    const int32_t *__restrict__ newid, const int32_t *__restrict__ rp2,
    int32_t *__restrict__ col2, V *__restrict__ vals2)
{
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < nnz;
         k += (int64_t)gridDim.x * kBlock) {
        int32_t lo = 0, hi = rows;  // rp[lo] <= k < rp[hi]
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (rp[mid] <= k)
                lo = mid;
            else
                hi = mid;
        }
        const int64_t dst = (int64_t)rp2[newid[lo]] + (k - rp[lo]);
        col2[dst] = newid[col[k]];
        vals2[dst] = vals[k];
    }
}

__global__ __launch_bounds__(kBlock) void k_permute_f32(int32_t n,
                                                        const int32_t *__restrict__ newid,
                                                        const float *__restrict__ in,
                                                        float *__restrict__ out, int to)
{
    const int32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v < n) {
        if (to)
            out[newid[v]] = in[v];
        else
            out[v] = in[newid[v]];
    }
}

// ------------------------------------------------------------------ JDS

// Before the product: iperm[q] = i for perm[i] = q (positions that perm does
// not name keep what they hold; the product looks at perm again), and
// status[0] gets 8 if a column index is negative and 16 if the entry count
// jd_ptr[max_len] is.
__global__ __launch_bounds__(kBlock) void k_jds_check(
    int32_t rows, int32_t max_len, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ jd_ptr, const int32_t *__restrict__ jd_col,
    int32_t *__restrict__ iperm, int32_t *__restrict__ status)
{
    const int32_t nnz = jd_ptr[max_len];
    int32_t flags = (nnz < 0) ? 16 : 0;
    const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = tid; i < rows; i += stride) {
        const int32_t q = perm[i];
        if (q >= 0 && q < rows)
            iperm[q] = (int32_t)i;
    }
    if (jd_col) {
        int32_t any = 0;   // the sign bit of any index
        int64_t k = tid;
        for (; k + 3 * stride < nnz; k += 4 * stride)
            any |= jd_col[k] | jd_col[k + stride] | jd_col[k + 2 * stride] |
                   jd_col[k + 3 * stride];
        for (; k < nnz; k += stride)
            any |= jd_col[k];
        flags |= (any < 0) ? 8 : 0;
    }
    flags = lane_group_or<64>(flags);
    if (flags && (threadIdx.x & 63) == 0)
        atomicOr(&status[0], flags);
}

// Thread p handles the row at JDS position p: diagonal j holds its j-th
// entry at jd_ptr[j] + p, so consecutive threads read consecutive entries.
// Each sum is taken in diagonal order without contraction.  The loads of
// kJdsAhead diagonals are in flight together: rows differ little along a
// wavefront, and one thread per row leaves few wavefronts to hide a chain of
// a load and a gather per diagonal (5,000 rows of 2 to 100 entries: the call
// 52 us with one, 44.6 with eight).  Large matrices are bound by the gathers
// (200k rows of 5 to 60 entries, 6.5 M gathers: 47 us at any depth).  A
// wavefront's part of a diagonal starts anywhere in a cache line, so the loads
// are ordinary ones: non-temporal, each line was fetched twice (65 us).
// Entries outside [0, nnz) and diagonals past max_len are never touched,
// whatever the arrays hold; a position whose original row is unknown (perm
// not a permutation) is not stored.  Nothing is stored if k_jds_check found
// the arrays at fault; workgroup 0 hands what it found to the host.
constexpr int kJdsAhead = 8;
__global__ __launch_bounds__(kBlock) void k_spmv_jds(
    int32_t rows, int32_t max_len, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ iperm, const int32_t *__restrict__ nzcnt,
    const int32_t *__restrict__ jd_ptr, const int32_t *__restrict__ jd_col,
    const double *__restrict__ jd_val, const double *__restrict__ x,
    double *__restrict__ y, const int32_t *__restrict__ status, int32_t *host_status)
{
#pragma clang fp contract(off)
    typedef const __attribute__((address_space(4))) int32_t *cptr;
    const int32_t fault = status[0];
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *host_status = fault;
    if (fault)
        return;
    const int32_t p = blockIdx.x * kBlock + threadIdx.x;
    const int32_t nnz = ((cptr)jd_ptr)[max_len];
    const int32_t n = (p < rows) ? min(nzcnt[p], max_len) : 0;
    const int32_t nmax = __builtin_amdgcn_readfirstlane(lane_group_max<64>(n));
    double s = 0.0;
    bool on = true;
    for (int32_t j0 = 0; j0 < nmax; j0 += kJdsAhead) {
        int32_t k[kJdsAhead], c[kJdsAhead];
        bool ok[kJdsAhead];
        double v[kJdsAhead];
#pragma unroll
        for (int u = 0; u < kJdsAhead; ++u) {
            const int32_t j = j0 + u;
            const uint32_t first = (uint32_t)((cptr)jd_ptr)[min(j, max_len)];
            k[u] = (int32_t)(first + (uint32_t)p);
            on = on && (j >= n || (k[u] >= 0 && k[u] < nnz));
            ok[u] = on && j < n;
        }
#pragma unroll
        for (int u = 0; u < kJdsAhead; ++u) {
            v[u] = ok[u] ? gld(jd_val + k[u]) : 0.0;
            c[u] = ok[u] ? gld(jd_col + k[u]) : 0;
        }
        double xv[kJdsAhead];
#pragma unroll
        for (int u = 0; u < kJdsAhead; ++u)
            xv[u] = ok[u] ? gld(x + c[u]) : 0.0;
#pragma unroll
        for (int u = 0; u < kJdsAhead; ++u) {
            const double prod = v[u] * xv[u];
            const double t = s + prod;
            s = ok[u] ? t : s;
        }
    }
    if (p >= rows)
        return;
    const int32_t i = iperm[p];
    if (i >= 0 && i < rows && perm[i] == p)
        y[i] = s;
}

// ---------------------------------------------------------- batched CG

// Segment of workgroup blockIdx.x (segments ordered by blk0).
__device__ __forceinline__ int32_t cg_seg_of(const CgSeg *__restrict__ segs,
                                             int32_t nseg)
{
    int32_t lo = 0, hi = nseg;
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (segs[mid].blk0 <= (int32_t)blockIdx.x)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Sum of part[0..n) (n <= kBlock) by one workgroup, the same in every
// workgroup that calls it.
__device__ __forceinline__ double sum_small(const double *__restrict__ part,
                                            int32_t n, double *lds)
{
    const double v = ((int32_t)threadIdx.x < n) ? part[threadIdx.x] : 0.0;
    return block_sum<kWaves>(v, lds);
}

__global__ __launch_bounds__(kBlock) void k_cgb_init(const CgSeg *__restrict__ segs,
                                                     int32_t nseg)
{
    __shared__ double lds[kWaves];
    const CgSeg sg = segs[cg_seg_of(segs, nseg)];
    const int32_t lb = blockIdx.x - sg.blk0;
    double acc = 0.0;
    for (int64_t i = (int64_t)lb * kBlock + threadIdx.x; i < sg.n;
         i += (int64_t)sg.nb * kBlock) {
        const double bi = sg.b[i];
        sg.x[i] = 0.0;
        sg.r[i] = bi;
        sg.p[i] = 0.0;
        sg.s[i] = 0.0;
        acc = fma(bi, bi, acc);
    }
    const double t = block_sum<kWaves>(acc, lds);
    if (threadIdx.x == 0) {
        sg.rr_part[lb] = t;  // parity of iteration 0
        if (lb == 0)
            *sg.done = 0;
    }
}

// Partial sums of r.w after the product w = A r (segments whose product
// wrote them, nrw > 0, are skipped).
__global__ __launch_bounds__(kBlock) void k_cgb_rw(const CgSeg *__restrict__ segs,
                                                   int32_t nseg)
{
    __shared__ double lds[kWaves];
    const CgSeg sg = segs[cg_seg_of(segs, nseg)];
    if (sg.nrw > 0)
        return;   // the product wrote them
    const int32_t lb = blockIdx.x - sg.blk0;
    double acc = 0.0;
    for (int64_t i = (int64_t)lb * kBlock + threadIdx.x; i < sg.n;
         i += (int64_t)sg.nb * kBlock)
        acc = fma(sg.r[i], sg.w[i], acc);
    const double t = block_sum<kWaves>(acc, lds);
    if (threadIdx.x == 0)
        sg.rw_part[lb] = t;
}

// gamma = r.r, delta = r.w; beta = gamma / gamma_old (0 at k = 0),
// p.Ap = delta - beta gamma / alpha_old, alpha = gamma / p.Ap; then
// p = r + beta p, s = w + beta s, x += alpha p, r -= alpha s and the
// partial sums of the new r.r.
__global__ __launch_bounds__(kBlock) void k_cgb_step(const CgSeg *__restrict__ segs,
                                                     int32_t nseg)
{
    __shared__ double lds[kWaves];
    const CgSeg sg = segs[cg_seg_of(segs, nseg)];
    if (*sg.done)
        return;
    const int32_t lb = blockIdx.x - sg.blk0;
    const int par = sg.iter & 1;
    const double g = sum_small(sg.rr_part + par * sg.nb, sg.nb, lds);
    const double d = sum_small(sg.rw_part, sg.nrw > 0 ? sg.nrw : sg.nb, lds);
    const double beta = (sg.iter > 0) ? g / sg.sc[par ^ 1] : 0.0;
    const double pap = (sg.iter > 0) ? d - beta * g / sg.sc[2 + (par ^ 1)] : d;
    if (g == 0.0 || pap == 0.0) {
        if (lb == 0 && threadIdx.x == 0)
            *sg.done = 1;
        return;
    }
    const double alpha = g / pap;
    double acc = 0.0;
    for (int64_t i = (int64_t)lb * kBlock + threadIdx.x; i < sg.n;
         i += (int64_t)sg.nb * kBlock) {
        const double ri = sg.r[i];
        const double pi = fma(beta, sg.p[i], ri);
        const double si = fma(beta, sg.s[i], sg.w[i]);
        sg.p[i] = pi;
        sg.s[i] = si;
        sg.x[i] = fma(alpha, pi, sg.x[i]);
        const double rn = fma(-alpha, si, ri);
        sg.r[i] = rn;
        acc = fma(rn, rn, acc);
    }
    const double t = block_sum<kWaves>(acc, lds);
    if (threadIdx.x == 0) {
        sg.rr_part[(par ^ 1) * sg.nb + lb] = t;
        if (lb == 0) {
            sg.sc[par] = g;
            sg.sc[2 + par] = alpha;
        }
    }
}

// ---------------------------------------------------------------- analysis

// status (zeroed before): [0] faults found, [1] largest column + 1, [2] longest
// row.
__global__ __launch_bounds__(kBlock) void k_validate(
    int32_t rows, const int32_t *__restrict__ rp, int64_t nnz,
    const int32_t *__restrict__ col, int32_t cols_given,
    int32_t *__restrict__ status)
{
    int32_t flags = 0, mx = 0, len = 0;
    const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = tid; i < rows; i += stride) {
        const int32_t n = rp[i + 1] - rp[i];
        if (rp[i + 1] < rp[i])
            flags |= 2;
        else
            len = max(len, n);
    }
    if (tid == 0) {
        if (rp[0] != 0)
            flags |= 1;
        if ((int64_t)rp[rows] != nnz)
            flags |= 4;
    }
    for (int64_t k = tid; k < nnz; k += stride) {
        const int32_t c = col[k];
        if (c < 0 || (cols_given >= 0 && c >= cols_given))
            flags |= 8;
        mx = max(mx, (int32_t)min((uint32_t)c + 1u, (uint32_t)INT_MAX));
    }
    // one update per workgroup, and none where the maximum is there already:
    // an update of one word takes some 12 ns, so one of each wavefront of
    // 4096 workgroups took 190 us whatever the matrix
    __shared__ int32_t fl[kWaves], top[kWaves], most[kWaves];
    flags = lane_group_or<64>(flags);
    mx = lane_group_max<64>(mx);
    len = lane_group_max<64>(len);
    if ((threadIdx.x & 63) == 0) {
        fl[threadIdx.x >> 6] = flags;
        top[threadIdx.x >> 6] = mx;
        most[threadIdx.x >> 6] = len;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kWaves; ++i) {
            flags |= fl[i];
            mx = max(mx, top[i]);
            len = max(len, most[i]);
        }
        if (flags)
            atomicOr(&status[0], flags);
        if (mx > __hip_atomic_load(&status[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(&status[1], mx);
        if (len > __hip_atomic_load(&status[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(&status[2], len);
    }
}

// Class of a row = number of class bounds it exceeds (bounds ascending), i.e.
// the first class whose inclusive upper bound holds it.
__device__ __forceinline__ int32_t row_class(int32_t len, const Thresholds &th)
{
    int32_t c = 0;
#pragma unroll
    for (int b = 0; b < NCLASS - 1; ++b)
        c += (len > th.upper[b]) ? 1 : 0;
    return c;
}

// hist is class-major: hist[c * nblk + block] = rows of class c in block.
__global__ __launch_bounds__(kBlock) void k_bin_count(
    int32_t rows, const int32_t *__restrict__ rp, Thresholds th,
    int32_t *__restrict__ hist, int32_t nblk)
{
    __shared__ int32_t cnt[NCLASS];
    if (threadIdx.x < NCLASS)
        cnt[threadIdx.x] = 0;
    __syncthreads();
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < rows)
        atomicAdd(&cnt[row_class(rp[i + 1] - rp[i], th)], 1);
    __syncthreads();
    if (threadIdx.x < NCLASS)
        hist[threadIdx.x * nblk + blockIdx.x] = cnt[threadIdx.x];
}

// Stable scatter: after the exclusive scan, hist[c*nblk+b] is where block
// b's rows of class c start; inside the block rows keep ascending order
// (wave by wave, lane by lane, ranks from ballots).
__global__ __launch_bounds__(kBlock) void k_bin_scatter(
    int32_t rows, const int32_t *__restrict__ rp, Thresholds th,
    const int32_t *__restrict__ hist, int32_t nblk,
    int32_t *__restrict__ bin_rows)
{
    __shared__ int32_t wcnt[kWaves][NCLASS];
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int32_t c = (i < rows) ? row_class(rp[i + 1] - rp[i], th) : -1;
    const unsigned long long below = (lane == 0) ? 0ull : ((1ull << lane) - 1ull);
    int32_t rank = 0;
#pragma unroll
    for (int b = 0; b < NCLASS; ++b) {
        const unsigned long long m = __ballot(c == b);
        if (lane == 0)
            wcnt[wave][b] = __popcll(m);
        if (c == b)
            rank = __popcll(m & below);
    }
    __syncthreads();
    if (c >= 0) {
        int32_t off = hist[c * nblk + blockIdx.x];
        for (int w = 0; w < wave; ++w)
            off += wcnt[w][c];
        bin_rows[off + rank] = i;
    }
}

// Exclusive prefix sum of a[0..n) in place by one 1024-thread workgroup;
// *total (if non-null) receives the sum.
__global__ __launch_bounds__(1024) void k_scan_excl(int32_t *__restrict__ a,
                                                    int64_t n,
                                                    int32_t *__restrict__ total)
{
    __shared__ int32_t s[1024];
    int32_t carry = 0;
    for (int64_t base = 0; base < n; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const int32_t v = (i < n) ? a[i] : 0;
        s[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const int32_t t = ((int)threadIdx.x >= off) ? s[threadIdx.x - off] : 0;
            __syncthreads();
            s[threadIdx.x] += t;
            __syncthreads();
        }
        if (i < n)
            a[i] = carry + s[threadIdx.x] - v;
        carry += s[1023];
        __syncthreads();
    }
    if (threadIdx.x == 0 && total)
        *total = carry;
}

// Exclusive scan of 8192-element tiles of a (8 consecutive per thread); the
// tile totals go to aux[tile].
__global__ __launch_bounds__(1024) void k_scan_tiles(int32_t *__restrict__ a,
                                                     int64_t n,
                                                     int32_t *__restrict__ aux)
{
    __shared__ int32_t ws[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * 8192 + (int64_t)threadIdx.x * 8;
    int32_t v[8];
    int32_t t = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = (base + j < n) ? a[base + j] : 0;
        t += v[j];
    }
    int32_t inc = t;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t u = __shfl_up(inc, o, 64);
        if (lane >= o)
            inc += u;
    }
    if (lane == 63)
        ws[wave] = inc;
    __syncthreads();
    int32_t run = inc - t;
    for (int i = 0; i < wave; ++i)
        run += ws[i];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (base + j < n)
            a[base + j] = run;
        run += v[j];
    }
    if (threadIdx.x == 1023)
        aux[blockIdx.x] = run;
}

// Adds the scanned tile totals to every element of the tile.
__global__ __launch_bounds__(1024) void k_scan_add(int32_t *__restrict__ a,
                                                   int64_t n,
                                                   const int32_t *__restrict__ aux)
{
    const int32_t add = aux[blockIdx.x];
    const int64_t base = (int64_t)blockIdx.x * 8192;
    for (int j = threadIdx.x; j < 8192; j += 1024)
        if (base + j < n)
            a[base + j] += add;
}

__global__ __launch_bounds__(kBlock) void k_chunk_count(
    int32_t nsplit, const int32_t *__restrict__ split_rows,
    const int32_t *__restrict__ rp, int32_t chunk, int32_t *__restrict__ cnt)
{
    const int32_t j = blockIdx.x * kBlock + threadIdx.x;
    if (j < nsplit) {
        const int32_t r = split_rows[j];
        const int64_t len = (int64_t)rp[r + 1] - rp[r];
        cnt[j] = (int32_t)((len + chunk - 1) / chunk);
    } else if (j == nsplit) {
        cnt[j] = 0;
    }
}

__global__ __launch_bounds__(kBlock) void k_chunk_fill(
    int32_t nsplit, const int32_t *__restrict__ split_rows,
    const int32_t *__restrict__ rp, int32_t chunk,
    const int32_t *__restrict__ s_first, int32_t *__restrict__ c_row,
    int32_t *__restrict__ c_k0, int32_t *__restrict__ c_k1)
{
    const int32_t j = blockIdx.x * kBlock + threadIdx.x;
    if (j >= nsplit)
        return;
    const int32_t r = split_rows[j];
    const int64_t a = rp[r], e = rp[r + 1];
    int32_t c = s_first[j];
    for (int64_t k = a; k < e; k += chunk, ++c) {
        c_row[c] = r;
        c_k0[c] = (int32_t)k;
        c_k1[c] = (int32_t)((e - k > chunk) ? k + chunk : e);
    }
}

__global__ __launch_bounds__(kBlock) void k_fill_i32(int32_t *__restrict__ p,
                                                     int64_t n, int32_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        p[i] = v;
}

__global__ __launch_bounds__(kBlock) void k_fill_f64(double *__restrict__ p, int64_t n,
                                                     double v)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        p[i] = v;
}

__global__ __launch_bounds__(kBlock) void k_zero_bytes(
    unsigned char *__restrict__ p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        p[i] = 0;
}

// ---------------------------------------------------------------- BLAS-1

// Sum of part[0..n) by a 1024-thread workgroup in a fixed order.
__device__ __forceinline__ double sum_parts_1024(const double *__restrict__ part,
                                                 int32_t n, double *lds)
{
    double acc = 0.0;
    for (int32_t i = threadIdx.x; i < n; i += 1024)
        acc += part[i];
    return block_sum<16>(acc, lds);
}

// This thread's part of sum a_i * b_i (float32 data is widened exactly, sums
// are binary64): THREADS threads to a workgroup, kDotAhead pieces of each
// vector requested together.  The pieces are 16 bytes, one load each where
// both vectors start on 16 bytes (WIDE), else one load per element; the sum
// is the same either way.  Bound by memory: 2^26 float64 elements, with the sum
// of the partials, in 158 us (6.8 TB/s); with ordinary loads 174 us.
template <typename T, bool WIDE, int THREADS>
__device__ __forceinline__ double dot_range(int64_t n, const T *__restrict__ a,
                                            const T *__restrict__ b)
{
    constexpr int U = kDotAhead, VV = 16 / sizeof(T);
    typedef T vec_t __attribute__((ext_vector_type(VV)));
    const int64_t nv = n / VV;
    auto piece = [](const T *p, int64_t i) {
        vec_t v;
        if constexpr (WIDE) {
            v = ld_stream((const vec_t *)p + i);
        } else {
#pragma unroll
            for (int j = 0; j < VV; ++j)
                v[j] = gld(p + i * VV + j);
        }
        return v;
    };
    double acc[VV] = {};
    for (int64_t i0 = (int64_t)blockIdx.x * THREADS * U; i0 < nv;
         i0 += (int64_t)gridDim.x * THREADS * U) {
        vec_t p[U], q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = min(i0 + u * THREADS + threadIdx.x, nv - 1);
            p[u] = piece(a, i);
            q[u] = piece(b, i);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + u * THREADS + threadIdx.x < nv) {
#pragma unroll
                for (int j = 0; j < VV; ++j)
                    acc[j] = fma((double)p[u][j], (double)q[u][j], acc[j]);
            }
        }
    }
    const int64_t rest = nv * VV + threadIdx.x;
    if (blockIdx.x == 0 && rest < n)
        acc[0] = fma((double)a[rest], (double)b[rest], acc[0]);
#pragma unroll
    for (int j = 1; j < VV; ++j)
        acc[0] += acc[j];
    return acc[0];
}

// Partial dot products, one per workgroup.
template <typename T, bool WIDE>
__global__ __launch_bounds__(kBlock) void k_dot_parts(
    int64_t n, const T *__restrict__ a, const T *__restrict__ b,
    double *__restrict__ part)
{
    __shared__ double lds[kWaves];
    const double t = block_sum<kWaves>(dot_range<T, WIDE, kBlock>(n, a, b), lds);
    if (threadIdx.x == 0)
        part[blockIdx.x] = t;
}

// The whole dot product of short vectors by one workgroup.
template <typename T, bool WIDE, typename TOut>
__global__ __launch_bounds__(1024) void k_dot_small(int64_t n, const T *__restrict__ a,
                                                    const T *__restrict__ b,
                                                    TOut *__restrict__ out)
{
    __shared__ double lds[16];
    const double t = block_sum<16>(dot_range<T, WIDE, 1024>(n, a, b), lds);
    if (threadIdx.x == 0)
        *out = (TOut)t;
}

// The total of the partials, stored as TOut: a float32 result is the
// binary64 total rounded once.
template <typename TOut>
__global__ __launch_bounds__(1024) void k_sum_parts(
    const double *__restrict__ part, int32_t n, TOut *__restrict__ out)
{
    __shared__ double lds[16];
    const double t = sum_parts_1024(part, n, lds);
    if (threadIdx.x == 0)
        *out = (TOut)t;
}

// HBM stream ceiling: every 16-byte piece of src read once with
// non-temporal loads, U pieces per thread in flight; with dst, each piece is
// also stored there (a copy).  The read-only form folds the data into a
// value that is stored only if it equals a constant nothing in practice
// produces, so the loads stay.  Workgroup g streams the contiguous range of
// pieces [g * per, (g + 1) * per).
template <int U, bool COPY>
__global__ __launch_bounds__(kBlock) void k_stream(const i32x4 *__restrict__ src,
                                                   i32x4 *__restrict__ dst, int64_t n,
                                                   int64_t per, uint32_t *__restrict__ sink)
{
    const int64_t lo = (int64_t)blockIdx.x * per;
    const int64_t hi = min(n, lo + per);
    int32_t fold = 0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += (int64_t)U * kBlock) {
        i32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = i + (int64_t)u * kBlock;
            v[u] = (k < hi) ? ld_stream(src + k) : i32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = i + (int64_t)u * kBlock;
            if (COPY) {
                if (k < hi)
                    __builtin_nontemporal_store(
                        v[u], (__attribute__((address_space(1))) i32x4 *)(dst + k));
            } else {
                fold ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
            }
        }
    }
    if (!COPY && fold == (int32_t)0x9E3779B9)
        sink[0] = (uint32_t)fold;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_copy(int64_t n,
                                                 const T *__restrict__ src,
                                                 T *__restrict__ dst)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock)
        dst[i] = src[i];
}

// Conjugate gradient in the arrangement of Chronopoulos and Gear (1989):
// the same iterates as the textbook loop in exact arithmetic, with both
// inner products of an iteration (r.r and r.Ar) available together, so an
// iteration is one product w = A r (with the partials of w.r fused into it)
// and one vector kernel.  Recurrences (s = A p kept alongside p):
//   gamma = r.r, delta = w.r, beta = gamma / gamma_old (0 at first),
//   p.Ap = delta - beta * gamma / alpha_old, alpha = gamma / p.Ap,
//   p = r + beta p, s = w + beta s, x += alpha p, r -= alpha s.
// The scalars of iteration k go to slot k & 1 of gamma[] and alpha[], so an
// iteration reads the previous slot while it writes its own.

// Start: x = 0, r = b, p = s = 0, partial sums of b.b into rr (parity 0).
__global__ __launch_bounds__(kBlock) void k_cg_init(
    int64_t n, const double *__restrict__ b, double *__restrict__ x,
    double *__restrict__ r, double *__restrict__ p, double *__restrict__ sv,
    double *__restrict__ rr, CgScalars *__restrict__ sc)
{
    __shared__ double lds[kWaves];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        const double bi = b[i];
        x[i] = 0.0;
        r[i] = bi;
        p[i] = 0.0;
        sv[i] = 0.0;
        acc = fma(bi, bi, acc);
    }
    const double t = block_sum<kWaves>(acc, lds);
    if (threadIdx.x == 0) {
        rr[blockIdx.x] = t;
        if (blockIdx.x == 0) {
            sc->rho = 0.0;
            sc->gamma[0] = sc->gamma[1] = 1.0;
            sc->alpha[0] = sc->alpha[1] = 1.0;
            sc->done = 0;
            sc->iters = 0;
        }
    }
}

// Sums of two values over the workgroup at once, each in the order of
// block_sum (so each equals block_sum of that value).
__device__ __forceinline__ void block_sum2(double &a, double &b, double *lds)
{
    a = lane_group_sum<64>(a);
    b = lane_group_sum<64>(b);
    __syncthreads();  // earlier readers of lds are done
    if ((threadIdx.x & 63) == 0) {
        lds[threadIdx.x >> 6] = a;
        lds[kWaves + (threadIdx.x >> 6)] = b;
    }
    __syncthreads();
    double ta = lds[0], tb = lds[kWaves];
#pragma unroll
    for (int i = 1; i < kWaves; ++i) {
        ta += lds[i];
        tb += lds[kWaves + i];
    }
    a = ta;
    b = tb;
}

// This thread's share of the sum of part[0..n): kPartsAhead of them requested
// together (a product of many workgroups leaves up to 8192).
constexpr int kPartsAhead = 8;
__device__ __forceinline__ double parts_share(const double *__restrict__ part, int32_t n)
{
    if (n <= kBlock)
        return (int32_t)threadIdx.x < n ? part[threadIdx.x] : 0.0;
    double acc = 0.0;
    for (int32_t i = threadIdx.x; i < n; i += kBlock * kPartsAhead) {
        double v[kPartsAhead];
#pragma unroll
        for (int u = 0; u < kPartsAhead; ++u)
            v[u] = (i + u * kBlock < n) ? part[i + u * kBlock] : 0.0;
#pragma unroll
        for (int u = 0; u < kPartsAhead; ++u)
            acc += v[u];
    }
    return acc;
}

// Iteration k (slot par = k & 1), after w = A r with the w.r partials in
// dot_part: every workgroup forms gamma, delta, beta and alpha itself, in
// the same order; the solve stops (x kept) when gamma or p.Ap is exactly 0.
// Each thread's first U pieces of VV elements are read before the sums, so
// their loads overlap; the partials of the new r.r go to rr[par ^ 1].  A piece
// is one load where every vector starts on it (WIDE), else one per element;
// the sums are the same either way.
// Bound by the latency of its two grid-wide dependences up to 262,144 rows, by
// L2 and the memory-side cache above: 7-point stencil of 100^3, 75 iterations
// of product and step, one element per thread and turn 3203 us, pairs with one
// piece in flight 2772, two 2653, four 2717 (two partials in flight instead of
// eight: 2750).
template <int VV, int U, bool WIDE>
__global__ __launch_bounds__(kBlock) void k_cg_step(
    int64_t n, CgScalars *__restrict__ sc, const double *__restrict__ w,
    double *__restrict__ p, double *__restrict__ sv, double *__restrict__ x,
    double *__restrict__ r, const double *__restrict__ dot_part, int32_t ndot,
    double *__restrict__ rr, int32_t nparts, int32_t k)
{
    struct Piece {
        double e[VV];
    };
    __shared__ double lds[2 * kWaves];
    const int32_t par = k & 1;
    const int64_t nv = n / VV;
    const int64_t step = (int64_t)gridDim.x * kBlock;
    auto read = [](const double *v, int64_t i) {
        Piece q;
        if constexpr (WIDE && VV == 2) {
            const f64x2 t = gld((const f64x2 *)v + i);
            q.e[0] = t.x;
            q.e[1] = t.y;
        } else {
#pragma unroll
            for (int j = 0; j < VV; ++j)
                q.e[j] = gld(v + i * VV + j);
        }
        return q;
    };
    auto write = [](double *v, int64_t i, const Piece &q) {
        if constexpr (WIDE && VV == 2) {
            gst((f64x2 *)v + i, f64x2{q.e[0], q.e[1]});
        } else {
#pragma unroll
            for (int j = 0; j < VV; ++j)
                gst(v + i * VV + j, q.e[j]);
        }
    };
    Piece wv[U], pv[U], ss[U], xv[U], rv[U];
    auto fetch = [&](int64_t i) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + u * step < nv) {
                wv[u] = read(w, i + u * step);
                pv[u] = read(p, i + u * step);
                ss[u] = read(sv, i + u * step);
                xv[u] = read(x, i + u * step);
                rv[u] = read(r, i + u * step);
            }
        }
    };
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    fetch(i);
    const int32_t done = sc->done;
    const double g_old = sc->gamma[par ^ 1], a_old = sc->alpha[par ^ 1];
    double g = parts_share(rr + par * kDotParts, nparts);
    double d = parts_share(dot_part, ndot);
    if (done)
        return;
    block_sum2(g, d, lds);
    const double beta = (k > 0) ? g / g_old : 0.0;
    const double pap = d - beta * g / a_old;
    if (g == 0.0 || pap == 0.0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            sc->done = 1;
            sc->rho = g;
        }
        return;
    }
    const double alpha = g / pap;
    double acc = 0.0;
    auto update = [&](double &pe, double &se, double &xe, double &re, double we) {
        pe = fma(beta, pe, re);
        se = fma(beta, se, we);
        xe = fma(alpha, pe, xe);
        re = fma(-alpha, se, re);
        acc = fma(re, re, acc);
    };
    for (;;) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t at = i + u * step;
            if (at < nv) {
#pragma unroll
                for (int j = 0; j < VV; ++j)
                    update(pv[u].e[j], ss[u].e[j], xv[u].e[j], rv[u].e[j], wv[u].e[j]);
                write(p, at, pv[u]);
                write(sv, at, ss[u]);
                write(x, at, xv[u]);
                write(r, at, rv[u]);
            }
        }
        i += U * step;
        if (i >= nv)
            break;
        fetch(i);
    }
    if (VV > 1 && (n & (VV - 1)) && blockIdx.x == 0 && threadIdx.x == 0) {
        double pe = p[n - 1], se = sv[n - 1], xe = x[n - 1], re = r[n - 1];
        update(pe, se, xe, re, w[n - 1]);
        p[n - 1] = pe;
        sv[n - 1] = se;
        x[n - 1] = xe;
        r[n - 1] = re;
    }
    const double t = block_sum<kWaves>(acc, lds);
    if (threadIdx.x == 0) {
        rr[(par ^ 1) * kDotParts + blockIdx.x] = t;
        if (blockIdx.x == 0) {
            sc->gamma[par] = g;
            sc->alpha[par] = alpha;
            sc->iters = k + 1;
        }
    }
}

// Iterations of a small sliced band matrix in one kernel each: a step and the
// next product together, which leaves one launch and one grid-wide dependence
// per iteration instead of two.  Iteration k reads r, s and w = A r (index 0)
// with the partials of r.r and r.w, updates p and x of its own rows, and
// writes the new r, s (index 1) and the new w = A r: the r of a gathered column
// is formed again from that column's old r, s and w, by the operations its own
// row uses, so no workgroup waits for another's update.  Three gathers for
// one, so only where launches, not entries, are the cost.  What does not need
// the scalars (own vectors, the slice's first entries and their gathers) is
// read before they are summed.
struct CgVecs {
    const double *r0, *s0, *w0;
    double *r1, *s1, *w1, *p, *x;
};

__global__ __launch_bounds__(kBandThreads) void k_cg_sell(
    BandDesc bd, CgVecs v, CgScalars *__restrict__ sc, const double *__restrict__ rr,
    int32_t nrr, const double *__restrict__ rw, double *__restrict__ rr1,
    double *__restrict__ rw1, int32_t k, int32_t last)
{
    __shared__ double lds[2 * kWaves];
    typedef SellGroup<double, 4> Quad;
    const int32_t par = k & 1;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int32_t b = xcd_block(blockIdx.x, bd.nblk);
    const int32_t done = sc->done;
    const double g_old = sc->gamma[par ^ 1], a_old = sc->alpha[par ^ 1];
    double g = 0.0, d = 0.0;
    for (int32_t i = threadIdx.x; i < nrr; i += kBandThreads)
        g += rr[i];
    for (int32_t i = threadIdx.x; i < bd.nblk; i += kBandThreads)
        d += rw[i];
    // a column's r, s and w as they are gathered
    struct Old {
        double r, s, w;
    };
    auto gather = [&](int32_t base, uint16_t off) {
        const int32_t c = base + off;
        return Old{gld(v.r0 + c), gld(v.s0 + c), gld(v.w0 + c)};
    };
    double alpha = 0.0, beta = 0.0;
    auto now = [&](const Old &o) { return fma(-alpha, fma(beta, o.s, o.w), o.r); };
    bool first = true;
    double arr = 0.0, arw = 0.0;
    const int32_t send = min((b + 1) * bd.spb, bd.nslice);
    for (int32_t s = b * bd.spb + wave; first || s < send; s += kBandWaves) {
        // (a wavefront without a slice takes part in the sums)
        const bool have = s < send;
        i32x4 sl{0, 0, 0, 0};
        if (have)
            sl = *(const __attribute__((address_space(4))) i32x4 *)(bd.slice + s);
        const int32_t row = s * 64 + lane;
        const bool mine = have && row < bd.rows;
        const double *pv = (const double *)bd.vals + (int64_t)sl.x * 64;
        const uint16_t *po = bd.off + (int64_t)sl.x * 64;
        const int32_t width = last ? 0 : sl.w;   // the last iteration needs no product
        const int32_t nq = width >> 2, tail = width & ~3;
        Old own{0.0, 0.0, 0.0};
        double p = 0.0, x = 0.0;
        int32_t len = width;
        if (mine) {
            own = Old{gld(v.r0 + row), gld(v.s0 + row), gld(v.w0 + row)};
            p = gld(v.p + row);
            x = gld(v.x + row);
        }
        if (sl.z < width)
            len = mine ? gld(bd.row_ptr + row + 1) - gld(bd.row_ptr + row) : 0;
        Quad q0, q1;
        SellGroup<double, 2> pr;
        double v1 = 0.0;
        uint16_t o1 = 0;
        if (nq > 0)
            q0.load(pv, po, lane);
        if (nq > 1)
            q1.load(pv + 256, po + 256, lane);
        if (width & 2)
            pr.load(pv + tail * 64, po + tail * 64, lane);
        if (width & 1) {
            v1 = ld_stream(pv + (width - 1) * 64 + lane);
            o1 = ld_stream(po + (width - 1) * 64 + lane);
        }
        Old g0[4], g1[4], gp[2], gl{0.0, 0.0, 0.0};
        if (nq > 0)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                g0[t] = gather(sl.y, q0.o[t]);
        if (nq > 1)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                g1[t] = gather(sl.y, q1.o[t]);
        if (width & 2) {
            gp[0] = gather(sl.y, pr.o.x);
            gp[1] = gather(sl.y, pr.o.y);
        }
        if (width & 1)
            gl = gather(sl.y, o1);
        if (first) {
            first = false;
            if (done)
                return;   // every wavefront of the launch
            block_sum2(g, d, lds);
            beta = (k > 0) ? g / g_old : 0.0;
            const double pap = d - beta * g / a_old;
            if (g == 0.0 || pap == 0.0) {
                if (blockIdx.x == 0 && threadIdx.x == 0) {
                    sc->done = 1;
                    sc->rho = g;
                }
                return;
            }
            alpha = g / pap;
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                sc->gamma[par] = g;
                sc->alpha[par] = alpha;
                sc->iters = k + 1;
            }
        }
        if (!have)
            break;
        double sum[4] = {};   // as in sell_block
        auto add = [&](int32_t j, int u, double val, const Old &o) {
            if (j < len)
                sum[u] = fma(val, now(o), sum[u]);
        };
        if (nq > 0)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                add(t, t, q0.val(t), g0[t]);
        if (nq > 1)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                add(4 + t, t, q1.val(t), g1[t]);
        if (width & 2) {
            add(tail, 0, pr.val(0), gp[0]);
            add(tail + 1, 1, pr.val(1), gp[1]);
        }
        if (width & 1)
            add(width - 1, 2, v1, gl);
        const double acc = total4(sum);
        if (mine) {
            const double si = fma(beta, own.s, own.w);
            const double pi = fma(beta, p, own.r);
            const double ri = fma(-alpha, si, own.r);
            v.p[row] = pi;
            v.x[row] = fma(alpha, pi, x);
            v.s1[row] = si;
            v.r1[row] = ri;
            v.w1[row] = acc;
            arr = fma(ri, ri, arr);
            arw = fma(ri, acc, arw);
        }
    }
    block_sum2(arr, arw, lds);
    if (threadIdx.x == 0) {
        rr1[b] = arr;
        rw1[b] = arw;
    }
}

// After the last iteration: rho = r.r of the final residual (partials in
// rr[par]), unless the solve stopped early (rho was set then).
__global__ __launch_bounds__(1024) void k_cg_final(CgScalars *__restrict__ sc,
                                                   const double *__restrict__ rr,
                                                   int32_t nparts, int32_t par)
{
    __shared__ double lds[16];
    const double t = sum_parts_1024(rr + par * kDotParts, nparts, lds);
    if (threadIdx.x == 0 && !sc->done)
        sc->rho = t;
}

inline int32_t grid_for(int64_t n, int32_t per_block, int32_t cap)
{
    int64_t g = (n + per_block - 1) / per_block;
    if (g < 1)
        g = 1;
    if (g > cap)
        g = cap;
    return (int32_t)g;
}

inline void check_launch(const char *what)
{
    hip_check(hipGetLastError(), what, __FILE__, __LINE__);
}

}  // namespace

// ------------------------------------------------------------- launchers

int32_t blas1_parts(int64_t n) { return grid_for(n, kBlock, kDotParts); }

int occupancy_tiles(lilac_dtype dt)
{
    int n = 0;
    hipError_t e = (dt == LILAC_F64)
        ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
              &n, k_spmv_tiles<double, true, false>, kBlock, 0)
        : hipOccupancyMaxActiveBlocksPerMultiprocessor(
              &n, k_spmv_tiles<float, true, false>, kBlock, 0);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return n;
}

void launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s)
{
    if (n <= 0)
        return;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, kBlock, 4096)),
                       dim3(kBlock), 0, s, p, n, v);
    check_launch("k_fill_i32");
}

void launch_fill_f64(double *p, int64_t n, double v, hipStream_t s)
{
    if (n <= 0)
        return;
    hipLaunchKernelGGL(k_fill_f64, dim3(grid_for(n, kBlock, 4096)), dim3(kBlock), 0, s, p,
                       n, v);
    check_launch("k_fill_f64");
}

void launch_fill_bytes_zero(void *p, int64_t bytes, hipStream_t s)
{
    if (bytes <= 0)
        return;
    hipLaunchKernelGGL(k_zero_bytes, dim3(grid_for(bytes, kBlock, 4096)),
                       dim3(kBlock), 0, s, (unsigned char *)p, bytes);
    check_launch("k_zero_bytes");
}

void launch_validate(int32_t rows, const int32_t *rp, int64_t nnz,
                     const int32_t *col, int32_t cols_given, int32_t *status,
                     hipStream_t s)
{
    const int64_t work = nnz > rows ? nnz : (int64_t)rows + 1;
    hipLaunchKernelGGL(k_validate, dim3(grid_for(work, kBlock * 4, 2048)),
                       dim3(kBlock), 0, s, rows, rp, nnz, col, cols_given,
                       status);
    check_launch("k_validate");
}

void launch_bin_count(int32_t rows, const int32_t *rp, const Thresholds &th,
                      int32_t *hist, int32_t nblk, hipStream_t s)
{
    hipLaunchKernelGGL(k_bin_count, dim3(nblk), dim3(kBlock), 0, s, rows, rp,
                       th, hist, nblk);
    check_launch("k_bin_count");
}

void launch_scan_excl(int32_t *a, int64_t n, int32_t *total, hipStream_t s)
{
    if (n <= 65536) {
        hipLaunchKernelGGL(k_scan_excl, dim3(1), dim3(1024), 0, s, a, n, total);
        check_launch("k_scan_excl");
        return;
    }
    // tiles of 8192, then the tile totals, then the offsets back into the tiles
    const int64_t nt = (n + 8191) / 8192;
    if (nt > INT32_MAX)
        fail(LILAC_ERR_ARG, "scan too long");
    int32_t *aux = (int32_t *)dev_alloc((size_t)nt * 4);
    hipLaunchKernelGGL(k_scan_tiles, dim3((uint32_t)nt), dim3(1024), 0, s, a, n, aux);
    check_launch("k_scan_tiles");
    hipLaunchKernelGGL(k_scan_excl, dim3(1), dim3(1024), 0, s, aux, nt, total);
    check_launch("k_scan_excl");
    hipLaunchKernelGGL(k_scan_add, dim3((uint32_t)nt), dim3(1024), 0, s, a, n,
                       (const int32_t *)aux);
    check_launch("k_scan_add");
    HIPC(hipStreamSynchronize(s));
    dev_free(aux);
}

void launch_bin_scatter(int32_t rows, const int32_t *rp, const Thresholds &th,
                        const int32_t *hist, int32_t nblk, int32_t *bin_rows,
                        hipStream_t s)
{
    hipLaunchKernelGGL(k_bin_scatter, dim3(nblk), dim3(kBlock), 0, s, rows, rp,
                       th, hist, nblk, bin_rows);
    check_launch("k_bin_scatter");
}

void launch_chunk_count(int32_t nsplit, const int32_t *split_rows,
                        const int32_t *rp, int32_t chunk, int32_t *cnt,
                        hipStream_t s)
{
    hipLaunchKernelGGL(k_chunk_count, dim3(grid_for((int64_t)nsplit + 1, kBlock, INT_MAX)),
                       dim3(kBlock), 0, s, nsplit, split_rows, rp, chunk, cnt);
    check_launch("k_chunk_count");
}

void launch_chunk_fill(int32_t nsplit, const int32_t *split_rows,
                       const int32_t *rp, int32_t chunk, const int32_t *s_first,
                       int32_t *c_row, int32_t *c_k0, int32_t *c_k1,
                       hipStream_t s)
{
    if (nsplit <= 0)
        return;
    hipLaunchKernelGGL(k_chunk_fill, dim3(grid_for(nsplit, kBlock, INT_MAX)),
                       dim3(kBlock), 0, s, nsplit, split_rows, rp, chunk,
                       s_first, c_row, c_k0, c_k1);
    check_launch("k_chunk_fill");
}

void launch_spmv_tiles(lilac_dtype dt, const Tile *tiles, int32_t ntiles,
                       int32_t grid, const MatDesc &single,
                       const MatDesc *mats, const Epi &epi, double *dot_part,
                       hipStream_t s)
{
    if (ntiles <= 0 || grid <= 0)
        return;
    const bool grouped = mats != nullptr;
    const bool dot = dot_part != nullptr;
    dim3 g(grid), b(kBlock);
    if (dt == LILAC_F64) {
        if (grouped && dot)
            hipLaunchKernelGGL((k_spmv_tiles<double, true, true>), g, b, 0, s, tiles, ntiles, single, mats, epi, dot_part);
        else if (grouped)
            hipLaunchKernelGGL((k_spmv_tiles<double, true, false>), g, b, 0, s, tiles, ntiles, single, mats, epi, dot_part);
        else if (dot)
            hipLaunchKernelGGL((k_spmv_tiles<double, false, true>), g, b, 0, s, tiles, ntiles, single, mats, epi, dot_part);
        else
            hipLaunchKernelGGL((k_spmv_tiles<double, false, false>), g, b, 0, s, tiles, ntiles, single, mats, epi, dot_part);
    } else {
        if (dot)
            fail(LILAC_ERR_UNSUPPORTED, "fused dot is only provided for float64");
        if (grouped)
            hipLaunchKernelGGL((k_spmv_tiles<float, true, false>), g, b, 0, s, tiles, ntiles, single, mats, epi, dot_part);
        else
            hipLaunchKernelGGL((k_spmv_tiles<float, false, false>), g, b, 0, s, tiles, ntiles, single, mats, epi, dot_part);
    }
    check_launch("k_spmv_tiles");
}

void launch_split_finalize(lilac_dtype dt, const int32_t *items, int32_t n,
                           const MatDesc &single, const MatDesc *mats,
                           const Epi &epi, double *dot_part, hipStream_t s)
{
    if (n <= 0)
        return;
    const bool grouped = mats != nullptr;
    const bool dot = dot_part != nullptr;
    dim3 g(grid_for(n, kBlock, INT_MAX)), b(kBlock);
    if (dt == LILAC_F64) {
        if (grouped)
            hipLaunchKernelGGL((k_split_finalize<double, true, false>), g, b, 0, s, items, n, single, mats, epi, dot_part);
        else if (dot)
            hipLaunchKernelGGL((k_split_finalize<double, false, true>), g, b, 0, s, items, n, single, mats, epi, dot_part);
        else
            hipLaunchKernelGGL((k_split_finalize<double, false, false>), g, b, 0, s, items, n, single, mats, epi, dot_part);
    } else {
        if (grouped)
            hipLaunchKernelGGL((k_split_finalize<float, true, false>), g, b, 0, s, items, n, single, mats, epi, dot_part);
        else
            hipLaunchKernelGGL((k_split_finalize<float, false, false>), g, b, 0, s, items, n, single, mats, epi, dot_part);
    }
    check_launch("k_split_finalize");
}

void launch_spmv_segments(lilac_dtype dt, const MatDesc *mats,
                          const int32_t *prefix, int32_t nseg, int32_t total,
                          int32_t grid, hipStream_t s)
{
    if (total <= 0 || nseg <= 0)
        return;
    grid = std::min(grid, total);
    if (dt == LILAC_F64)
        hipLaunchKernelGGL(k_spmv_segments<double>, dim3(grid), dim3(kBlock), 0, s,
                           mats, prefix, nseg, total);
    else
        hipLaunchKernelGGL(k_spmv_segments<float>, dim3(grid), dim3(kBlock), 0, s,
                           mats, prefix, nseg, total);
    check_launch("k_spmv_segments");
}

// A launch whose end `done` (or null) stands for: the event rides on the kernel's
// own packet, where recording it behind the kernel is a packet more (products of
// 100,000 random rows one after the other 15.7 and 16.7 us).
template <typename F, typename... Args>
static void launch_done(F kernel, dim3 g, dim3 b, int lds, hipStream_t s, hipEvent_t done,
                        Args... args)
{
    if (done)
        hipExtLaunchKernelGGL(kernel, g, b, lds, s, nullptr, done, 0, args...);
    else
        hipLaunchKernelGGL(kernel, g, b, lds, s, args...);
}

void launch_spmv_panels(lilac_dtype dt, const PanelDesc &pd, const void *x,
                        void *y, const Epi &epi, const void *w, double *dot_part,
                        hipStream_t s)
{
    if (pd.nblk <= 0)
        return;
    dim3 g(pd.nblk), b(kPanelThreads);
    if (pd.col0) {
        if (dt == LILAC_F32 && dot_part)
            fail(LILAC_ERR_UNSUPPORTED, "fused dot is only provided for float64");
        if (dt == LILAC_F32)
            hipLaunchKernelGGL((k_spmv_lanes<float, false>), g, b, kPanelLds, s, pd,
                               (const float *)x, (float *)y, epi, (const float *)w, dot_part);
        else if (dot_part)
            hipLaunchKernelGGL((k_spmv_lanes<double, true>), g, b, kPanelLds, s, pd,
                               (const double *)x, (double *)y, epi, (const double *)w, dot_part);
        else
            hipLaunchKernelGGL((k_spmv_lanes<double, false>), g, b, kPanelLds, s, pd,
                               (const double *)x, (double *)y, epi, (const double *)w, dot_part);
        check_launch("k_spmv_lanes");
        return;
    }
    if (dt == LILAC_F64) {
        if (dot_part)
            hipLaunchKernelGGL((k_spmv_panels<double, true>), g, b, kPanelLds, s, pd,
                               (const double *)x, (double *)y, epi, (const double *)w, dot_part);
        else
            hipLaunchKernelGGL((k_spmv_panels<double, false>), g, b, kPanelLds, s, pd,
                               (const double *)x, (double *)y, epi, (const double *)w, dot_part);
    } else {
        if (dot_part)
            fail(LILAC_ERR_UNSUPPORTED, "fused dot is only provided for float64");
        hipLaunchKernelGGL((k_spmv_panels<float, false>), g, b, kPanelLds, s, pd,
                           (const float *)x, (float *)y, epi, (const float *)w, dot_part);
    }
    check_launch("k_spmv_panels");
}

void launch_spmv_lane_groups(lilac_dtype dt, const PanelDesc &pd, const void *x, void *y,
                             const Epi &epi, const void *w, double *dot_part, double *part,
                             hipStream_t s, hipEvent_t done)
{
    if (pd.nblk <= 0)
        return;
    dim3 g((pd.nblk + pd.gper - 1) / pd.gper * pd.ng), b(kPanelThreads);
    dim3 t(dot_part ? pd.nblk : grid_for(pd.rows, kPanelThreads, INT_MAX));
    if (dt == LILAC_F64) {
        if (pd.gper == 2)
            hipLaunchKernelGGL((k_spmv_lane_groups<double, 2>), g, b, kPanelLds, s, pd,
                               (const double *)x, part);
        else
            hipLaunchKernelGGL((k_spmv_lane_groups<double, 1>), g, b, kPanelLds, s, pd,
                               (const double *)x, part);
        if (dot_part)
            launch_done(k_lane_total<double, true>, t, b, 0, s, done, pd, part, (double *)y, epi,
                        (const double *)w, dot_part);
        else
            launch_done(k_lane_total<double, false>, t, b, 0, s, done, pd, part, (double *)y, epi,
                        (const double *)w, dot_part);
    } else {
        if (dot_part)
            fail(LILAC_ERR_UNSUPPORTED, "fused dot is only provided for float64");
        if (pd.gper == 2)
            hipLaunchKernelGGL((k_spmv_lane_groups<float, 2>), g, b, kPanelLds, s, pd,
                               (const float *)x, part);
        else
            hipLaunchKernelGGL((k_spmv_lane_groups<float, 1>), g, b, kPanelLds, s, pd,
                               (const float *)x, part);
        launch_done(k_lane_total<float, false>, t, b, 0, s, done, pd, part, (float *)y, epi,
                    (const float *)w, dot_part);
    }
    check_launch("k_spmv_lane_groups");
}

void launch_spmv_panels_grouped(lilac_dtype dt, const PanelDesc *descs,
                                const PanelIO *io, const int32_t *prefix,
                                int32_t nmat, int32_t nblocks, hipStream_t s)
{
    if (nmat <= 0 || nblocks <= 0)
        return;
    dim3 g(nblocks), b(kPanelThreads);
    if (dt == LILAC_F64)
        hipLaunchKernelGGL(k_spmv_panels_grouped<double>, g, b, kPanelLds, s, descs,
                           io, prefix, nmat);
    else
        hipLaunchKernelGGL(k_spmv_panels_grouped<float>, g, b, kPanelLds, s, descs,
                           io, prefix, nmat);
    check_launch("k_spmv_panels_grouped");
}

void launch_spmv_band(lilac_dtype dt, const BandDesc &bd, const void *x, void *y,
                      const Epi &epi, const void *w, double *dot_part, hipStream_t s)
{
    if (bd.nblk <= 0)
        return;
    dim3 g(bd.nblk), b(kBandThreads);
    if (bd.nslice > 0) {
        if (dt == LILAC_F32 && dot_part)
            fail(LILAC_ERR_UNSUPPORTED, "fused dot is only provided for float64");
        if (dt == LILAC_F32)
            hipLaunchKernelGGL((k_spmv_sell<float, false>), g, b, 0, s, bd,
                               (const float *)x, (float *)y, epi, (const float *)w, dot_part);
        else if (dot_part)
            hipLaunchKernelGGL((k_spmv_sell<double, true>), g, b, 0, s, bd,
                               (const double *)x, (double *)y, epi, (const double *)w, dot_part);
        else
            hipLaunchKernelGGL((k_spmv_sell<double, false>), g, b, 0, s, bd,
                               (const double *)x, (double *)y, epi, (const double *)w, dot_part);
        check_launch("k_spmv_sell");
        return;
    }
    if (dt == LILAC_F64) {
        if (dot_part)
            hipLaunchKernelGGL((k_spmv_band<double, true>), g, b, 0, s, bd,
                               (const double *)x, (double *)y, epi, (const double *)w, dot_part);
        else
            hipLaunchKernelGGL((k_spmv_band<double, false>), g, b, 0, s, bd,
                               (const double *)x, (double *)y, epi, (const double *)w, dot_part);
    } else {
        if (dot_part)
            fail(LILAC_ERR_UNSUPPORTED, "fused dot is only provided for float64");
        hipLaunchKernelGGL((k_spmv_band<float, false>), g, b, 0, s, bd,
                           (const float *)x, (float *)y, epi, (const float *)w, dot_part);
    }
    check_launch("k_spmv_band");
}

void launch_spmv_band_grouped(lilac_dtype dt, const BandDesc *descs, const PanelIO *io,
                              const int32_t *prefix, int32_t nmat, int32_t nblocks,
                              hipStream_t s)
{
    if (nmat <= 0 || nblocks <= 0)
        return;
    dim3 g(nblocks), b(kBandThreads);
    if (dt == LILAC_F64)
        hipLaunchKernelGGL(k_spmv_band_grouped<double>, g, b, 0, s, descs, io, prefix, nmat);
    else
        hipLaunchKernelGGL(k_spmv_band_grouped<float>, g, b, 0, s, descs, io, prefix, nmat);
    check_launch("k_spmv_band_grouped");
}

void launch_row_span(int32_t rows, const int32_t *rp, const int32_t *col, int32_t *lo,
                     int32_t *hi, hipStream_t s)
{
    if (rows <= 0)
        return;
    hipLaunchKernelGGL(k_row_span, dim3(grid_for(rows, kBlock, INT_MAX)), dim3(kBlock), 0,
                       s, rows, rp, col, lo, hi);
    check_launch("k_row_span");
}

void launch_band_pack(const BandDesc &bd, const int32_t *rp, const int32_t *col,
                      uint32_t *rc, hipStream_t s)
{
    hipLaunchKernelGGL(k_band_pack, dim3(grid_for(bd.rows, kBlock, INT_MAX)), dim3(kBlock),
                       0, s, bd, rp, col, rc);
    check_launch("k_band_pack");
}

void launch_slice_span(int32_t rows, const int32_t *rp, const int32_t *col, int32_t nslice,
                       int32_t *out, hipStream_t s)
{
    if (nslice <= 0)
        return;
    hipLaunchKernelGGL(k_slice_span, dim3(grid_for(nslice, kWaves, INT_MAX)), dim3(kBlock), 0,
                       s, rows, rp, col, nslice, (i32x4 *)out);
    check_launch("k_slice_span");
}

void launch_sell_pack(lilac_dtype dt, const BandDesc &bd, const int32_t *col,
                      const void *vals, void *sv, uint16_t *so, hipStream_t s)
{
    if (bd.nslice <= 0)
        return;
    dim3 g(grid_for(bd.nslice, kWaves, INT_MAX)), b(kBlock);
    if (dt == LILAC_F64)
        hipLaunchKernelGGL(k_sell_pack<double>, g, b, 0, s, bd, col, (const double *)vals,
                           (double *)sv, so);
    else
        hipLaunchKernelGGL(k_sell_pack<float>, g, b, 0, s, bd, col, (const float *)vals,
                           (float *)sv, so);
    check_launch("k_sell_pack");
}

void launch_line_reuse(int32_t rows, const int32_t *rp, const int32_t *col,
                       int32_t ngroups, int32_t shift, int32_t *out, hipStream_t s)
{
    if (rows <= 0 || ngroups <= 0)
        return;
    hipLaunchKernelGGL(k_line_reuse, dim3(ngroups), dim3(kBlock), 0, s, rows, rp, col,
                       ngroups, shift, out);
    check_launch("k_line_reuse");
}

template <bool DIRECT>
static void launch_hot(lilac_dtype dt, const HotDesc &hd, const void *x, void *y,
                       const Epi &epi, const void *w, double *dot_part, hipStream_t s,
                       hipEvent_t done)
{
    dim3 g(hd.grid), b(kPanelThreads);
    if (dt == LILAC_F64) {
        if (dot_part)
            launch_done(k_spmv_hot<double, true, DIRECT>, g, b, kPanelLds, s, done, hd,
                        (const double *)x, (double *)y, epi, (const double *)w, dot_part);
        else
            launch_done(k_spmv_hot<double, false, DIRECT>, g, b, kPanelLds, s, done, hd,
                        (const double *)x, (double *)y, epi, (const double *)w, dot_part);
    } else {
        if (dot_part)
            fail(LILAC_ERR_UNSUPPORTED, "fused dot is only provided for float64");
        launch_done(k_spmv_hot<float, false, DIRECT>, g, b, kPanelLds, s, done, hd,
                    (const float *)x, (float *)y, epi, (const float *)w, dot_part);
    }
    check_launch("k_spmv_hot");
}

void launch_spmv_hot(lilac_dtype dt, const HotDesc &hd, const void *x, void *y,
                     const Epi &epi, const void *w, double *dot_part, void *xp, hipStream_t s,
                     hipEvent_t done)
{
    if (hd.nblk <= 0 || hd.grid <= 0)
        return;
    if (hd.old && !xp) {
        launch_hot<true>(dt, hd, x, y, epi, w, dot_part, s, done);
        return;
    }
    if (hd.old) {
        dim3 g(grid_for(hd.cols, kBlock, INT_MAX)), b(kBlock);
        if (dt == LILAC_F64)
            hipLaunchKernelGGL(k_place_cols<double>, g, b, 0, s, hd.cols, hd.newid,
                               (const double *)x, (double *)xp);
        else
            hipLaunchKernelGGL(k_place_cols<float>, g, b, 0, s, hd.cols, hd.newid,
                               (const float *)x, (float *)xp);
        check_launch("k_place_cols");
        x = xp;
    }
    launch_hot<false>(dt, hd, x, y, epi, w, dot_part, s, done);
}

void launch_hot_count(const HotDesc &hd, const int32_t *rp, const int32_t *col,
                      const int32_t *list, int32_t nlist, int32_t most, int32_t *cnt,
                      hipStream_t s)
{
    hipLaunchKernelGGL(k_hot_count, dim3(grid_for(hd.rows, 64, INT_MAX)), dim3(kBlock), 0, s,
                       hd, rp, col, (const int32_t *)nullptr, most, cnt);
    check_launch("k_hot_count");
    if (nlist > 0)
        hipLaunchKernelGGL(k_hot_count, dim3(nlist), dim3(kBlock), 0, s, hd, rp, col, list, most,
                           cnt);
    check_launch("k_hot_count");
}

void launch_row_filled(int32_t rows, const int32_t *rp, int32_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_row_filled, dim3(grid_for((int64_t)rows + 1, kBlock, INT_MAX)),
                       dim3(kBlock), 0, s, rows, rp, out);
    check_launch("k_row_filled");
}

void launch_hot_blocks(int32_t rows, const int32_t *rp, const int32_t *filled, int32_t part,
                       const HotTries &tries, int32_t cap, int32_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_hot_blocks, dim3(grid_for(rows, part, INT_MAX), tries.n), dim3(64), 0,
                       s, rows, rp, filled, part, tries, cap, out);
    check_launch("k_hot_blocks");
}

void launch_hot_rmap(const HotDesc &hd, const int32_t *filled, uint16_t *rmap, hipStream_t s)
{
    hipLaunchKernelGGL(k_hot_rmap, dim3(grid_for(hd.rows, kBlock, INT_MAX)), dim3(kBlock), 0,
                       s, hd, filled, rmap);
    check_launch("k_hot_rmap");
}

void launch_hot_share(int64_t nnz, int32_t step, const int32_t *col, const int32_t *newid,
                      int32_t hot, int32_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_hot_share, dim3(grid_for(nnz / step, kBlock * 8, 1024)), dim3(kBlock),
                       0, s, nnz, step, col, newid, hot, out);
    check_launch("k_hot_share");
}

void launch_hot_flag(int32_t n, const int32_t *newid, int32_t hot, int32_t *flag,
                     hipStream_t s)
{
    hipLaunchKernelGGL(k_hot_flag, dim3(grid_for((int64_t)n + 1, kBlock, INT_MAX)), dim3(kBlock),
                       0, s, n, newid, hot, flag);
    check_launch("k_hot_flag");
}

void launch_hot_order(int32_t n, int32_t hot, const int32_t *before, int32_t *newid,
                      int32_t *old, hipStream_t s)
{
    hipLaunchKernelGGL(k_hot_order, dim3(grid_for(n, kBlock, INT_MAX)), dim3(kBlock), 0, s, n,
                       hot, before, newid, old);
    check_launch("k_hot_order");
}

void launch_hot_split(const HotDesc &hd, const int32_t *hx, int32_t *bsplit,
                      hipStream_t s)
{
    hipLaunchKernelGGL(k_hot_split, dim3(grid_for(hd.nblk, kBlock, INT_MAX)),
                       dim3(kBlock), 0, s, hd, hx, bsplit);
    check_launch("k_hot_split");
}

void launch_hot_scatter(lilac_dtype dt, const HotDesc &hd, const int32_t *rp,
                        const int32_t *col, const void *vals, const int32_t *list,
                        int32_t nlist, int32_t most, const int32_t *hx, void *hv, uint32_t *hrc,
                        uint16_t *hkey, uint32_t *hcold, hipStream_t s)
{
    auto go = [&](dim3 g, const int32_t *l) {
        if (dt == LILAC_F64)
            hipLaunchKernelGGL(k_hot_scatter<double>, g, dim3(kBlock), 0, s, hd, rp, col,
                               (const double *)vals, l, most, hx, (double *)hv, hrc, hkey, hcold);
        else
            hipLaunchKernelGGL(k_hot_scatter<float>, g, dim3(kBlock), 0, s, hd, rp, col,
                               (const float *)vals, l, most, hx, (float *)hv, hrc, hkey, hcold);
        check_launch("k_hot_scatter");
    };
    go(dim3(grid_for(hd.rows, 64, INT_MAX)), nullptr);
    if (nlist > 0)
        go(dim3(nlist), list);
}

void panels_prepare()
{
    static bool done = false;
    if (done)
        return;
    HIPC(hipFuncSetAttribute((const void *)k_spmv_panels_grouped<double>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_panels_grouped<float>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_hot<double, true, true>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_hot<double, true>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_hot<double, false, true>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_hot<double, false>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_hot<float, false, true>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_hot<float, false>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_panels<double, true>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_panels<double, false>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_panels<float, false>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_lane_groups<double, 1>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_lane_groups<double, 2>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_lane_groups<float, 1>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_lane_groups<float, 2>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_lanes<double, true>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_lanes<double, false>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    HIPC(hipFuncSetAttribute((const void *)k_spmv_lanes<float, false>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
    done = true;
}

void launch_panel_count(const PanelDesc &pd, const int32_t *rp,
                        const int32_t *col, int32_t *cnt, hipStream_t s)
{
    hipLaunchKernelGGL(k_panel_count, dim3(grid_for((int64_t)pd.rows * 64, kBlock, INT_MAX)),
                       dim3(kBlock), 0, s, pd, rp, col, cnt);
    check_launch("k_panel_count");
}

void launch_panel_scatter(lilac_dtype dt, const PanelDesc &pd, const int32_t *rp,
                          const int32_t *col, const void *vals, const int32_t *ptr,
                          void *pv, uint32_t *prc, hipStream_t s)
{
    dim3 g(grid_for((int64_t)pd.rows * 64, kBlock, INT_MAX)), b(kBlock);
    if (dt == LILAC_F64)
        hipLaunchKernelGGL(k_panel_scatter<double>, g, b, 0, s, pd, rp, col,
                           (const double *)vals, ptr, (double *)pv, prc);
    else
        hipLaunchKernelGGL(k_panel_scatter<float>, g, b, 0, s, pd, rp, col,
                           (const float *)vals, ptr, (float *)pv, prc);
    check_launch("k_panel_scatter");
}

void launch_lane_runs(const PanelDesc &pd, int32_t *cnt, int32_t *kc, hipStream_t s)
{
    const int64_t n = (int64_t)pd.nblk * pd.np * kPanelWaves * 64;
    hipLaunchKernelGGL(k_lane_runs, dim3(grid_for(n, kBlock, INT_MAX)), dim3(kBlock), 0, s, pd,
                       cnt, kc);
    check_launch("k_lane_runs");
}

void launch_lane_fill(lilac_dtype dt, const PanelDesc &pd, const int32_t *pos, void *vals,
                      uint16_t *words, uint8_t *start, hipStream_t s)
{
    const int64_t n = (int64_t)pd.nblk * pd.np * kPanelWaves * 64;
    dim3 g(grid_for(n, kBlock, INT_MAX)), b(kBlock);
    if (dt == LILAC_F64)
        hipLaunchKernelGGL(k_lane_fill<double>, g, b, 0, s, pd, pos, (double *)vals, words,
                           start);
    else
        hipLaunchKernelGGL(k_lane_fill<float>, g, b, 0, s, pd, pos, (float *)vals, words,
                           start);
    check_launch("k_lane_fill");
}

void launch_lane_scatter(lilac_dtype dt, const PanelDesc &pd, const int32_t *rp,
                         const int32_t *col, const void *src, const int32_t *pos,
                         void *vals, uint16_t *words, hipStream_t s)
{
    dim3 g(grid_for((int64_t)pd.rows * 64, kBlock, INT_MAX)), b(kBlock);
    if (dt == LILAC_F64)
        hipLaunchKernelGGL(k_lane_scatter<double>, g, b, 0, s, pd, rp, col,
                           (const double *)src, pos, (double *)vals, words);
    else
        hipLaunchKernelGGL(k_lane_scatter<float>, g, b, 0, s, pd, rp, col,
                           (const float *)src, pos, (float *)vals, words);
    check_launch("k_lane_scatter");
}

void launch_panel_wptr(const PanelDesc &pd, const int32_t *ptr, int32_t *wptr,
                       hipStream_t s)
{
    const int64_t n = (int64_t)pd.nblk * pd.np * (kPanelWaves + 1);
    hipLaunchKernelGGL(k_panel_wptr, dim3(grid_for(n, kBlock, INT_MAX)), dim3(kBlock),
                       0, s, pd, ptr, wptr);
    check_launch("k_panel_wptr");
}

void launch_bfs_init(int32_t rows, int32_t source, const int32_t *rp, int32_t *level,
                     uint32_t *bits, int32_t words, uint64_t *todo, int32_t *last,
                     hipStream_t s)
{
    hipLaunchKernelGGL(k_bfs_init, dim3(grid_for(rows, kBlock, 2048)), dim3(kBlock), 0, s,
                       rows, source, rp, level, bits, words, todo, last);
    check_launch("k_bfs_init");
}

void launch_bfs_step(const MatDesc &m, int32_t nchunk, int32_t nlong, int32_t rows,
                     int32_t *level, int32_t depth, uint32_t *bits, int32_t words,
                     uint64_t *todo, int32_t *last, hipStream_t s)
{
    static bool ready = false;
    if (!ready) {
        HIPC(hipFuncSetAttribute((const void *)k_bfs_step<true>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, kPanelLds));
        ready = true;
    }
    if (rows <= 0)
        return;
    const int32_t cu = device_cu_count();
    const int64_t work = (int64_t)nchunk + nlong + ((int64_t)rows + 63) / 64;
    const int32_t full = grid_for(work, kBfsThreads / 64, cu * 2);
    if (words * 4 <= kPanelLds) {
        const int32_t per_cu = std::max(1, std::min(2, kPanelLds / (words * 4)));
        hipLaunchKernelGGL(k_bfs_step<true>, dim3(std::min(full, cu * per_cu)),
                           dim3(kBfsThreads), words * 4, s, m, nchunk, nlong, rows, level,
                           depth, bits, words, todo, last);
    } else {
        hipLaunchKernelGGL(k_bfs_step<false>, dim3(full), dim3(kBfsThreads), 0, s, m, nchunk,
                           nlong, rows, level, depth, bits, words, todo, last);
    }
    check_launch("k_bfs_step");
}

void launch_bfs_report(const int32_t *last, int32_t *host, hipStream_t s)
{
    hipLaunchKernelGGL(k_bfs_report, dim3(1), dim3(1), 0, s, last, host);
    check_launch("k_bfs_report");
}

void launch_jds_check(int32_t rows, int32_t max_len, const int32_t *perm,
                      const int32_t *jd_ptr, const int32_t *jd_col, int32_t *iperm,
                      int32_t *status, hipStream_t s)
{
    hipLaunchKernelGGL(k_jds_check, dim3(1024), dim3(kBlock), 0, s, rows, max_len, perm,
                       jd_ptr, jd_col, iperm, status);
    check_launch("k_jds_check");
}

void launch_spmv_jds(int32_t rows, int32_t max_len, const int32_t *perm,
                     const int32_t *iperm, const int32_t *nzcnt, const int32_t *jd_ptr,
                     const int32_t *jd_col, const double *jd_val, const double *x, double *y,
                     const int32_t *status, int32_t *host_status, hipStream_t s)
{
    hipLaunchKernelGGL(k_spmv_jds, dim3(grid_for(rows, kBlock, INT_MAX)), dim3(kBlock),
                       0, s, rows, max_len, perm, iperm, nzcnt, jd_ptr, jd_col, jd_val, x, y,
                       status, host_status);
    check_launch("k_spmv_jds");
}

void launch_count_cols(int64_t nnz, int32_t step, const int32_t *col, int32_t *deg,
                       hipStream_t s)
{
    if (nnz <= 0)
        return;
    hipLaunchKernelGGL(k_count_cols, dim3(grid_for(nnz / step, kBlock * 8, 8192)), dim3(kBlock),
                       0, s, nnz, step, col, deg);
    check_launch("k_count_cols");
}

void launch_degree_keys(int32_t n, const int32_t *deg, int32_t *key, hipStream_t s)
{
    hipLaunchKernelGGL(k_degree_keys, dim3(grid_for(n, kBlock, INT_MAX)), dim3(kBlock),
                       0, s, n, deg, key);
    check_launch("k_degree_keys");
}

void launch_key_hist(int32_t n, const int32_t *key, int32_t *hist, int32_t nblk,
                     hipStream_t s)
{
    hipLaunchKernelGGL(k_key_hist, dim3(nblk), dim3(kBlock), 0, s, n, key, hist, nblk);
    check_launch("k_key_hist");
}

void launch_key_scatter(int32_t n, const int32_t *key, const int32_t *hist,
                        int32_t nblk, int32_t *newid, hipStream_t s)
{
    hipLaunchKernelGGL(k_key_scatter, dim3(nblk), dim3(kBlock), 0, s, n, key, hist,
                       nblk, newid);
    check_launch("k_key_scatter");
}

void launch_perm_lengths(int32_t rows, const int32_t *rp, const int32_t *newid,
                         int32_t *len2, hipStream_t s)
{
    hipLaunchKernelGGL(k_perm_lengths, dim3(grid_for((int64_t)rows + 1, kBlock, INT_MAX)),
                       dim3(kBlock), 0, s, rows, rp, newid, len2);
    check_launch("k_perm_lengths");
}

void launch_perm_entries(lilac_dtype dt, int32_t rows, int64_t nnz, const int32_t *rp,
                         const int32_t *col, const void *vals, const int32_t *newid,
                         const int32_t *rp2, int32_t *col2, void *vals2, hipStream_t s)
{
    if (nnz <= 0)
        return;
    dim3 g(grid_for(nnz, kBlock, 65536)), b(kBlock);
    if (dt == LILAC_F64)
        hipLaunchKernelGGL(k_perm_entries<double>, g, b, 0, s, rows, nnz, rp, col,
                           (const double *)vals, newid, rp2, col2, (double *)vals2);
    else
        hipLaunchKernelGGL(k_perm_entries<float>, g, b, 0, s, rows, nnz, rp, col,
                           (const float *)vals, newid, rp2, col2, (float *)vals2);
    check_launch("k_perm_entries");
}

void launch_permute_f32(int32_t n, const int32_t *newid, const float *in, float *out,
                        bool to, hipStream_t s)
{
    if (n <= 0)
        return;
    hipLaunchKernelGGL(k_permute_f32, dim3(grid_for(n, kBlock, INT_MAX)), dim3(kBlock), 0,
                       s, n, newid, in, out, to ? 1 : 0);
    check_launch("k_permute_f32");
}

int32_t cg_seg_blocks(int64_t n) { return grid_for(n, kBlock, kBlock); }

void launch_cgb_init(const CgSeg *segs, int32_t nseg, int32_t blocks, hipStream_t s)
{
    if (blocks <= 0)
        return;
    hipLaunchKernelGGL(k_cgb_init, dim3(blocks), dim3(kBlock), 0, s, segs, nseg);
    check_launch("k_cgb_init");
}

void launch_cgb_rw(const CgSeg *segs, int32_t nseg, int32_t blocks, hipStream_t s)
{
    if (blocks <= 0)
        return;
    hipLaunchKernelGGL(k_cgb_rw, dim3(blocks), dim3(kBlock), 0, s, segs, nseg);
    check_launch("k_cgb_rw");
}

void launch_cgb_step(const CgSeg *segs, int32_t nseg, int32_t blocks, hipStream_t s)
{
    if (blocks <= 0)
        return;
    hipLaunchKernelGGL(k_cgb_step, dim3(blocks), dim3(kBlock), 0, s, segs, nseg);
    check_launch("k_cgb_step");
}

template <bool WIDE, typename T, typename TOut>
static void launch_dot_as(int64_t n, const T *a, const T *b, double *part, TOut *out,
                          hipStream_t s)
{
    if (n <= kDotSmall) {
        hipLaunchKernelGGL((k_dot_small<T, WIDE, TOut>), dim3(1), dim3(1024), 0, s, n, a, b, out);
        check_launch("k_dot_small");
        return;
    }
    const int32_t np = grid_for(n, kBlock * (int)(16 / sizeof(T)), kDotParts);
    hipLaunchKernelGGL((k_dot_parts<T, WIDE>), dim3(np), dim3(kBlock), 0, s, n, a, b, part);
    check_launch("k_dot_parts");
    hipLaunchKernelGGL(k_sum_parts<TOut>, dim3(1), dim3(1024), 0, s, part, np, out);
    check_launch("k_sum_parts");
}

template <typename T, typename TOut>
void launch_dot(int64_t n, const T *a, const T *b, double *part, TOut *out, hipStream_t s)
{
    if ((((uintptr_t)a | (uintptr_t)b) & 15) == 0)
        launch_dot_as<true>(n, a, b, part, out, s);
    else
        launch_dot_as<false>(n, a, b, part, out, s);
}
template void launch_dot<double, double>(int64_t, const double *, const double *, double *,
                                         double *, hipStream_t);
template void launch_dot<float, float>(int64_t, const float *, const float *, double *, float *,
                                       hipStream_t);
template void launch_dot<float, double>(int64_t, const float *, const float *, double *,
                                        double *, hipStream_t);

void launch_sum_parts(const double *part, int32_t nparts, double *out,
                      hipStream_t s)
{
    hipLaunchKernelGGL(k_sum_parts<double>, dim3(1), dim3(1024), 0, s, part, nparts,
                       out);
    check_launch("k_sum_parts");
}

void launch_stream(const void *src, void *dst, int64_t bytes, int32_t groups,
                   uint32_t *sink, hipStream_t s)
{
    const int64_t n = bytes / 16;
    if (n <= 0)
        return;
    const int64_t per = (n + groups - 1) / groups;
    if (dst)
        hipLaunchKernelGGL((k_stream<4, true>), dim3(groups), dim3(kBlock), 0, s,
                           (const i32x4 *)src, (i32x4 *)dst, n, per, sink);
    else
        hipLaunchKernelGGL((k_stream<8, false>), dim3(groups), dim3(kBlock), 0, s,
                           (const i32x4 *)src, (i32x4 *)nullptr, n, per, sink);
    check_launch("k_stream");
}

void launch_copy_bytes(const void *src, void *dst, int64_t bytes, hipStream_t s)
{
    const int64_t n = (bytes + 15) / 16;
    if (n <= 0)
        return;
    hipLaunchKernelGGL(k_copy<i32x4>, dim3(grid_for(n, kBlock, 8192)), dim3(kBlock), 0, s, n,
                       (const i32x4 *)src, (i32x4 *)dst);
    check_launch("k_copy");
}

void launch_copy_f32(int64_t n, const float *src, float *dst, hipStream_t s)
{
    if (n <= 0)
        return;
    hipLaunchKernelGGL(k_copy<float>, dim3(grid_for(n, kBlock, 8192)),
                       dim3(kBlock), 0, s, n, src, dst);
    check_launch("k_copy");
}

void launch_cg_init(int64_t n, const double *b, double *x, double *r, double *p,
                    double *sv, double *rr, int32_t nparts, CgScalars *sc, hipStream_t s)
{
    hipLaunchKernelGGL(k_cg_init, dim3(nparts), dim3(kBlock), 0, s, n, b, x, r, p, sv, rr,
                       sc);
    check_launch("k_cg_init");
}

void launch_cg_step(int64_t n, CgScalars *sc, const double *w, double *p, double *sv,
                    double *x, double *r, const double *dot_part, int32_t ndot, double *rr,
                    int32_t nparts, int32_t k, hipStream_t s)
{
    dim3 g(nparts), b(kBlock);
    // one element per thread up to one round of the workgroups, then pairs
    if (n <= (int64_t)kDotParts * kBlock)
        hipLaunchKernelGGL((k_cg_step<1, 1, false>), g, b, 0, s, n, sc, w, p, sv, x, r, dot_part,
                           ndot, rr, nparts, k);
    else if ((((uintptr_t)w | (uintptr_t)p | (uintptr_t)sv | (uintptr_t)x | (uintptr_t)r) & 15) ==
             0)
        hipLaunchKernelGGL((k_cg_step<2, 2, true>), g, b, 0, s, n, sc, w, p, sv, x, r, dot_part,
                           ndot, rr, nparts, k);
    else
        hipLaunchKernelGGL((k_cg_step<2, 2, false>), g, b, 0, s, n, sc, w, p, sv, x, r, dot_part,
                           ndot, rr, nparts, k);
    check_launch("k_cg_step");
}

void launch_cg_sell(const BandDesc &bd, const CgFused &f, CgScalars *sc, const double *rr,
                    int32_t nrr, const double *rw, double *rr1, double *rw1, int32_t k,
                    bool last, hipStream_t s)
{
    const int i = k & 1;
    const CgVecs v{f.r[i], f.s[i], f.w[i], f.r[i ^ 1], f.s[i ^ 1], f.w[i ^ 1], f.p, f.x};
    hipLaunchKernelGGL(k_cg_sell, dim3(bd.nblk), dim3(kBandThreads), 0, s, bd, v, sc, rr, nrr,
                       rw, rr1, rw1, k, last ? 1 : 0);
    check_launch("k_cg_sell");
}

void launch_cg_final(CgScalars *sc, const double *rr, int32_t nparts, int32_t par,
                     hipStream_t s)
{
    hipLaunchKernelGGL(k_cg_final, dim3(1), dim3(1024), 0, s, sc, rr, nparts, par);
    check_launch("k_cg_final");
}

}  // namespace lilac
