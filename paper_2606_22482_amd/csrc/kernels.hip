// kernels.hip -- gfx950 kernels of the hybrid SpMM: one kernel per item kind
// (segments, vector items, windows, window partials) launched in dependency
// order, the batched persistent kernels, and the copy kernel.  The items
// themselves are in items.hpp.
#include "items.hpp"
namespace spmm {

template <int VT, int BT, int E, int CPL, bool POL, bool HOLD>
__global__ __launch_bounds__(256) void segment_kernel(DevPlan P, RunArgs a) {
    const int wid = logical_block(a.xcd) * 4 + wave_id();
    if (wid < P.n_seg * a.n_panels) segment_item<VT, BT, E, CPL, POL, false, HOLD>(P, a, wid);
}


template <int VT, int BT, int E, int CPL, int VAR, bool HOLD>
__global__ __launch_bounds__(256, (vector_waves<BT, CPL, VAR, unroll_of<E, CPL>(), HOLD>())) void vector_kernel(
    DevPlan P, RunArgs a) {
    const int wid = logical_block(a.xcd) * 4 + wave_id();
    if (wid < P.n_vitems * a.n_panels) vector_item_var<VT, BT, E, CPL, VAR, false, unroll_of<E, CPL>(), HOLD>(P, a, wid);
}


template <int VT, int BT, int TT, int MB, int MBW, int CW, bool BUF, int RG>
__global__ __launch_bounds__(256, (window_waves<MBW, CW>())) void window_kernel(DevPlan P, RunArgs a, int partial) {
    const int wid = logical_block(a.xcd) * 4 + wave_id();
    if (wid < (partial ? P.n_wpart : P.n_win) * a.win_panels * a.win_subs)
        window_item<VT, BT, TT, MB, MBW, CW, BUF, RG>(P, a, wid, partial != 0);
}


// ------------------------------------------------------------------------------------------
// Batched persistent kernels: a fixed grid walks the global item space of a
// descriptor table with a static stride, so the item -> matrix lookup only
// moves forward.  Each matrix's items run exactly the code of a single run, so
// a matrix's result is bitwise the same alone and in a batch.

// Persistent walk over one XCD's items of one kind: item ids g of XCD x are
// [xb[x], xb[x+1]); entries of XCD x start at x_entry[x]; `end` gives an
// entry's exclusive item prefix (global over the table), `base` the matrix
// item index of its first item.
#define SPMM_XCD_WALK(XB, END, BASE, PER_WG, BODY)                                     \
    do {                                                                               \
        const int x = blockIdx.x & 7, local = blockIdx.x >> 3, nloc = gridDim.x >> 3;   \
        const int lo = hdr->XB[x], hi = hdr->XB[x + 1];                                \
        int d = hdr->x_entry[x];                                                       \
        for (int g = lo + local * PER_WG + sub; g < hi; g += nloc * PER_WG) {          \
            while (g >= tab[d].END) ++d;                                               \
            const int item = g - (d ? tab[d - 1].END : 0) + tab[d].BASE;               \
            BODY;                                                                      \
        }                                                                              \
    } while (0)

template <int VT, int BT, int E, int CPL, bool POL>
__global__ __launch_bounds__(256) void batch_segment_kernel(const BatchHeader *__restrict__ hdr,
                                                            const BatchEntry *__restrict__ tab) {
    const int sub = wave_id();
    SPMM_XCD_WALK(x_seg, seg_end, seg_base, 4, (segment_item<VT, BT, E, CPL, POL, false, !POL>(tab[d].P, tab[d].a, item)));
}

// Entries per group and step of the batched vector kernel: 4 for 16-bit B in
// one chunk per lane (the persistent walk over many matrices holds more
// registers, and half the step brings the kernel from 4 to 5 waves per SIMD:
// measured 10.78 -> 10.01 ms on 512 uneven f16 matrices, where single runs
// are faster with 8); a row's sum does not depend on it, so a batched result
// stays bitwise equal to the same plan run alone.
template <int E, int CPL>
constexpr int batch_unroll() { return (E == 8 && CPL == 1) ? 4 : unroll_of<E, CPL>(); }

// The batch's rows of f32 B load their own entries: the small matrices of a
// serving batch are bound by latency, and held entries add a hand-out to it (16
// matrices of 1,000 to 20,000 rows: 164 us, held 174).
template <int BT>
constexpr bool batch_hold() { return BT != DT_F32; }

template <int VT, int BT, int E, int CPL, int VAR>
__global__ __launch_bounds__(256, (vector_waves<BT, CPL, VAR, batch_unroll<E, CPL>(), batch_hold<BT>()>())) void batch_vector_kernel(const BatchHeader *__restrict__ hdr,
                                                           const BatchEntry *__restrict__ tab) {
    const int sub = wave_id();
    SPMM_XCD_WALK(x_vec, vec_end, vec_base, 4,
                  (vector_item_var<VT, BT, E, CPL, VAR, false, batch_unroll<E, CPL>(), batch_hold<BT>()>(tab[d].P, tab[d].a, item)));
}

// An item of a batch: one 16-row block a wave, two (of 64-row windows of 16-bit
// B), or one row a lane group; 172 registers without the last two, and with them
// 237, which the same 2 waves per SIMD hold.
template <int VT, int BT, int TT, int MB, int MBW, int CW, int RG>
__device__ __forceinline__ void batch_window_shape(const BatchEntry &e, int wid, bool partial) {
    if (e.a.b_rec) window_item<VT, BT, TT, MB, MBW, CW, true, RG>(e.P, e.a, wid, partial);
    else window_item<VT, BT, TT, MB, MBW, CW, false, RG>(e.P, e.a, wid, partial);
}

template <int VT, int BT, int TT, bool PARTIAL>
__device__ __forceinline__ void batch_window_item(const BatchEntry &e, int wid) {
    const int np = e.a.win_np;
    if (e.a.win_rows == 1) {
        if constexpr (BT != DT_F32)
            if (np == 128) return batch_window_shape<VT, BT, TT, 0, 1, 8, 1>(e, wid, PARTIAL);
        if (np == 64) return batch_window_shape<VT, BT, TT, 0, 1, 4, 1>(e, wid, PARTIAL);
        return batch_window_shape<VT, BT, TT, 0, 1, 2, 1>(e, wid, PARTIAL);
    }
    if constexpr (BT != DT_F32) {
        if (16 * e.a.win_subs < e.P.H)
            return np == 128 ? batch_window_shape<VT, BT, TT, 4, 2, 8, 4>(e, wid, PARTIAL)
                             : batch_window_shape<VT, BT, TT, 4, 2, 4, 4>(e, wid, PARTIAL);
        if (np == 128) return batch_window_shape<VT, BT, TT, 0, 1, 8, 4>(e, wid, PARTIAL);
    }
    if (np == 64) return batch_window_shape<VT, BT, TT, 0, 1, 4, 4>(e, wid, PARTIAL);
    if (np == 32) return batch_window_shape<VT, BT, TT, 0, 1, 2, 4>(e, wid, PARTIAL);
    window_item<VT, BT, TT, 0, 1, 1, false, 4>(e.P, e.a, wid, PARTIAL);
}

template <int VT, int BT, int TT, bool PARTIAL>
__global__ __launch_bounds__(256, 2) void batch_window_kernel(const BatchHeader *__restrict__ hdr,
                                                           const BatchEntry *__restrict__ tab) {
    const int sub = wave_id();
    if (PARTIAL) SPMM_XCD_WALK(x_wpart, wpart_end, wpart_base, 4, (batch_window_item<VT, BT, TT, true>(tab[d], item)));
    else SPMM_XCD_WALK(x_win, win_end, win_base, 4, (batch_window_item<VT, BT, TT, false>(tab[d], item)));
}

// One tile a wavefront (up to 64 rows of 32 slots): the rows' value counts are
// summed over the lanes, then two rows a step are written side by side.
__global__ __launch_bounds__(256) void spread_tiles_kernel(int64_t tiles, int32_t H, const uint32_t *__restrict__ bitmap,
                                                           const int32_t *__restrict__ val_ptr,
                                                           const uint16_t *__restrict__ vals,
                                                           uint16_t *__restrict__ dense) {
    const int64_t t = (int64_t)blockIdx.x * 4 + wave_id();
    if (t >= tiles) return;
    const int lane = threadIdx.x & 63;
    const uint32_t w = lane < H ? bitmap[t * H + lane] : 0u;
    const int before = wave_inclusive_scan(__popc(w)) - __popc(w);
    const int64_t v0 = val_ptr[t];
    for (int r0 = 0; r0 < H; r0 += 2) {
        const int r = r0 + (lane >> 5), j = lane & 31;
        const uint32_t m = (uint32_t)__shfl((int)w, r, 64);
        const int64_t at = v0 + __shfl(before, r, 64) + __popc(m & ((1u << j) - 1u));
        dense[(t * H + r) * 32 + j] = (m >> j) & 1u ? vals[at] : (uint16_t)0;
    }
}

// Streaming copy used as the achievable-bandwidth reference: one 16-byte
// load and store per lane per round over a large grid (measured on gfx950:
// 5.4 TB/s read + write over 1 GiB; four loads in flight per lane over an
// eight-workgroups-per-CU grid reached only 4.5 TB/s).
__global__ __launch_bounds__(256) void copy_kernel(const f32x4 *__restrict__ src,
                                                   f32x4 *__restrict__ dst, int64_t n4) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// ------------------------------------------------------------------------------------------
// launchers

static inline unsigned grid_for_waves(int64_t waves) { return (unsigned)((waves + 3) / 4); }

template <int VT, int BT, bool POL, bool HOLD>
static hipError_t seg_dispatch_pol(const DevPlan &P, const RunArgs &a, hipStream_t s) {
    const int64_t waves = (int64_t)P.n_seg * a.n_panels;
    if (waves == 0) return hipSuccess;
    constexpr int EV = BT == DT_F32 ? 4 : 8;
    const int chunks = a.vec_ok ? (a.np + EV - 1) / EV : a.np;
    dim3 grid(grid_for_waves(waves)), block(256);
    if (a.vec_ok) {
        if (chunks <= 64) launch_kernel((segment_kernel<VT, BT, EV, 1, POL, HOLD>), grid, block, 0, s, P, a);
        else launch_kernel((segment_kernel<VT, BT, EV, 2, POL, HOLD>), grid, block, 0, s, P, a);
    } else {
        launch_kernel((segment_kernel<VT, BT, 1, 2, POL, false>), grid, block, 0, s, P, a);
    }
    return hipGetLastError();
}

template <int VT, int BT>
static hipError_t seg_dispatch(const DevPlan &P, const RunArgs &a, hipStream_t s) {
    // the per-entry cache-policy choice only for plans with a cold policy
    if (a.cold_aux >= 0) return seg_dispatch_pol<VT, BT, true, false>(P, a, s);
    return a.hold ? seg_dispatch_pol<VT, BT, false, true>(P, a, s) : seg_dispatch_pol<VT, BT, false, false>(P, a, s);
}

template <int VT, int BT, int VAR, bool HOLD>
static hipError_t vec_dispatch_var(const DevPlan &P, const RunArgs &a, hipStream_t s) {
    const int64_t waves = (int64_t)P.n_vitems * a.n_panels;
    if (waves == 0) return hipSuccess;
    constexpr int EV = BT == DT_F32 ? 4 : 8;
    const int chunks = a.vec_ok ? (a.np + EV - 1) / EV : a.np;
    dim3 grid(grid_for_waves(waves)), block(256);
    if (a.vec_ok) {
        if (chunks <= 64) launch_kernel((vector_kernel<VT, BT, EV, 1, VAR, HOLD>), grid, block, 0, s, P, a);
        else launch_kernel((vector_kernel<VT, BT, EV, 2, VAR, HOLD>), grid, block, 0, s, P, a);
    } else {
        launch_kernel((vector_kernel<VT, BT, 1, 2, VAR, false>), grid, block, 0, s, P, a);
    }
    return hipGetLastError();
}

template <int VT, int BT>
static hipError_t vec_dispatch(const DevPlan &P, const RunArgs &a, hipStream_t s) {
    if (a.pipeline == 3) return vec_dispatch_var<VT, BT, 3, false>(P, a, s);
    if (a.pipeline == 2)  // (the others' rows load their own entries)
        return a.hold ? vec_dispatch_var<VT, BT, 2, true>(P, a, s) : vec_dispatch_var<VT, BT, 2, false>(P, a, s);
    if (a.pipeline == 1) return vec_dispatch_var<VT, BT, 1, false>(P, a, s);
    return vec_dispatch_var<VT, BT, 0, false>(P, a, s);
}

template <int VT, int BT, int TT>
static hipError_t win_dispatch(const DevPlan &P, const RunArgs &a, hipStream_t s, bool partial) {
    const int64_t waves = (int64_t)(partial ? P.n_wpart : P.n_win) * a.win_panels * a.win_subs;
    if (waves == 0) return hipSuccess;
    return window_shape<BT>(P, a, [&](auto mb, auto mbw, auto cw, auto buf, auto rg) {
        launch_kernel((window_kernel<VT, BT, TT, decltype(mb)::value, decltype(mbw)::value, decltype(cw)::value,
                                     decltype(buf)::value, decltype(rg)::value>),
                      dim3(grid_for_waves(waves)), dim3(256), 0, s, P, a, partial ? 1 : 0);
        return hipGetLastError();
    });
}

hipError_t launch_segment(const DevPlan &P, int32_t vt, int32_t bt, const RunArgs &a, hipStream_t s) {
    if (vt == DT_F32 && bt == DT_F32) return seg_dispatch<DT_F32, DT_F32>(P, a, s);
    if (vt == DT_F32 && bt == DT_BF16) return seg_dispatch<DT_F32, DT_BF16>(P, a, s);
    if (vt == DT_BF16 && bt == DT_BF16) return seg_dispatch<DT_BF16, DT_BF16>(P, a, s);
    if (vt == DT_F16 && bt == DT_F16) return seg_dispatch<DT_F16, DT_F16>(P, a, s);
    return hipErrorInvalidValue;
}

hipError_t launch_vector(const DevPlan &P, int32_t vt, int32_t bt, const RunArgs &a, hipStream_t s) {
    if (vt == DT_F32 && bt == DT_F32) return vec_dispatch<DT_F32, DT_F32>(P, a, s);
    if (vt == DT_F32 && bt == DT_BF16) return vec_dispatch<DT_F32, DT_BF16>(P, a, s);
    if (vt == DT_BF16 && bt == DT_BF16) return vec_dispatch<DT_BF16, DT_BF16>(P, a, s);
    if (vt == DT_F16 && bt == DT_F16) return vec_dispatch<DT_F16, DT_F16>(P, a, s);
    return hipErrorInvalidValue;
}

hipError_t launch_window(const DevPlan &P, int32_t vt, int32_t bt, int32_t tt, const RunArgs &a,
                         hipStream_t s, bool partial) {
    if (vt == DT_F32 && bt == DT_F32 && tt == DT_BF16) return win_dispatch<DT_F32, DT_F32, DT_BF16>(P, a, s, partial);
    if (vt == DT_F32 && bt == DT_BF16 && tt == DT_BF16) return win_dispatch<DT_F32, DT_BF16, DT_BF16>(P, a, s, partial);
    if (vt == DT_BF16 && bt == DT_BF16 && tt == DT_BF16) return win_dispatch<DT_BF16, DT_BF16, DT_BF16>(P, a, s, partial);
    if (vt == DT_F16 && bt == DT_F16 && tt == DT_F16) return win_dispatch<DT_F16, DT_F16, DT_F16>(P, a, s, partial);
    return hipErrorInvalidValue;
}

template <int VT, int BT, int TT, int E, int CPL, int VAR>
static hipError_t batch_variant(const BatchHeader *hdr, const BatchEntry *tab, const BatchGrids &g,
                                hipStream_t s, BatchGrids *occ) {
    if (occ) {
        int o = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &o, batch_segment_kernel<VT, BT, E, CPL, VAR == 0>, 256, 0);
        if (e != hipSuccess) return e;
        occ->seg = (unsigned)o;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, batch_vector_kernel<VT, BT, E, CPL, VAR>, 256, 0);
        if (e != hipSuccess) return e;
        occ->vec = (unsigned)o;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &o, batch_window_kernel<VT, BT, TT, false>, 256, 0);
        occ->win = (unsigned)o;
        return e;
    }
    // phase 1: partial sums (segments, window tile chunks); phase 2: owners
    hipLaunchKernelGGL((batch_segment_kernel<VT, BT, E, CPL, VAR == 0>), dim3(g.seg), dim3(256), 0, s, hdr, tab);
    hipLaunchKernelGGL((batch_window_kernel<VT, BT, TT, true>), dim3(g.win), dim3(256), 0, s,
                       hdr, tab);
    hipLaunchKernelGGL((batch_vector_kernel<VT, BT, E, CPL, VAR>), dim3(g.vec), dim3(256), 0, s, hdr, tab);
    hipLaunchKernelGGL((batch_window_kernel<VT, BT, TT, false>), dim3(g.win), dim3(256), 0,
                       s, hdr, tab);
    return hipGetLastError();
}

template <int VT, int BT, int TT, int VAR>
static hipError_t batch_types_var(const BatchHeader *hdr, const BatchEntry *tab, int vec_ok,
                                  int cpl, const BatchGrids &g, hipStream_t s, BatchGrids *occ) {
    constexpr int EV = BT == DT_F32 ? 4 : 8;
    if (!vec_ok) return batch_variant<VT, BT, TT, 1, 2, VAR>(hdr, tab, g, s, occ);
    if (cpl == 1) return batch_variant<VT, BT, TT, EV, 1, VAR>(hdr, tab, g, s, occ);
    return batch_variant<VT, BT, TT, EV, 2, VAR>(hdr, tab, g, s, occ);
}

template <int VT, int BT, int TT>
static hipError_t batch_types(const BatchHeader *hdr, const BatchEntry *tab, int vec_ok, int cpl,
                              int var, const BatchGrids &g, hipStream_t s, BatchGrids *occ) {
    if (var == 3) return batch_types_var<VT, BT, TT, 3>(hdr, tab, vec_ok, cpl, g, s, occ);
    if (var == 2) return batch_types_var<VT, BT, TT, 2>(hdr, tab, vec_ok, cpl, g, s, occ);
    if (var == 1) return batch_types_var<VT, BT, TT, 1>(hdr, tab, vec_ok, cpl, g, s, occ);
    return batch_types_var<VT, BT, TT, 0>(hdr, tab, vec_ok, cpl, g, s, occ);
}

static hipError_t batch_any(const BatchHeader *hdr, const BatchEntry *tab, int32_t vt, int32_t bt,
                            int32_t tt, int vec_ok, int cpl, int var, const BatchGrids &g,
                            hipStream_t s, BatchGrids *occ) {
    if (vt == DT_F32 && bt == DT_F32 && tt == DT_BF16)
        return batch_types<DT_F32, DT_F32, DT_BF16>(hdr, tab, vec_ok, cpl, var, g, s, occ);
    if (vt == DT_F32 && bt == DT_BF16 && tt == DT_BF16)
        return batch_types<DT_F32, DT_BF16, DT_BF16>(hdr, tab, vec_ok, cpl, var, g, s, occ);
    if (vt == DT_BF16 && bt == DT_BF16 && tt == DT_BF16)
        return batch_types<DT_BF16, DT_BF16, DT_BF16>(hdr, tab, vec_ok, cpl, var, g, s, occ);
    if (vt == DT_F16 && bt == DT_F16 && tt == DT_F16)
        return batch_types<DT_F16, DT_F16, DT_F16>(hdr, tab, vec_ok, cpl, var, g, s, occ);
    return hipErrorInvalidValue;
}

hipError_t launch_batch(const BatchHeader *hdr, const BatchEntry *tab, int32_t vt, int32_t bt,
                        int32_t tt, int vec_ok, int cpl, int var, const BatchGrids &grids,
                        hipStream_t s) {
    return batch_any(hdr, tab, vt, bt, tt, vec_ok, cpl, var, grids, s, nullptr);
}

hipError_t batch_occupancy(int32_t vt, int32_t bt, int32_t tt, int vec_ok, int cpl, int var,
                           BatchGrids *per_cu) {
    return batch_any(nullptr, nullptr, vt, bt, tt, vec_ok, cpl, var, BatchGrids{}, nullptr, per_cu);
}

hipError_t launch_spread_tiles(int64_t tiles, int32_t H, const uint32_t *bitmap, const int32_t *val_ptr,
                               const uint16_t *vals, uint16_t *dense, hipStream_t s) {
    if (tiles <= 0) return hipSuccess;
    if (H < 2 || H > 64 || H % 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(spread_tiles_kernel, dim3(grid_for_waves(tiles)), dim3(256), 0, s, tiles, H, bitmap, val_ptr,
                       vals, dense);
    return hipGetLastError();
}

hipError_t launch_copy(const float4 *src, float4 *dst, int64_t n4, hipStream_t s) {
    if (n4 <= 0) return hipSuccess;
    int64_t blocks = (n4 + 255) / 256;
    if (blocks > 256 * 64) blocks = 256 * 64;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                       reinterpret_cast<const f32x4 *>(src), reinterpret_cast<f32x4 *>(dst), n4);
    return hipGetLastError();
}

}  // namespace spmm

