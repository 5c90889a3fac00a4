// items.hpp -- device functions of one work item of each kind (gfx950).
//
// The kernels that execute a plan (NeutronSparse Sec. 5.1 execution models,
// adapted to CDNA4 where the matrix cores and the vector ALUs share a CU) are
// built from three items:
//
//   segment  -- one wavefront per segment of a long remainder row: FP32
//               gather-FMA partial sum into a per-run workspace.
//   vector   -- one wavefront per vector work item (consecutive rows): FP32
//               gather-FMA over each row's remainder (Sec. 5.1, gather then
//               accumulate), or the fixed-order sum of its segment partials,
//               then one write of the C row.
//   window   -- one wavefront per (row window or a share of its rows, column
//               panel of 128, 64, 32 or 16): the B rows of each tile's
//               compacted columns are loaded straight into MFMA operand order
//               (Sec. 5.1, matrix-engine execution), each tile's dense values
//               are the other operand (bf16 / f16 in, f32 accumulate), then
//               each row adds its remainder and is written once.
//
// Summation order of a remainder segment (identical in every kernel that
// computes one, so a row's bits depend only on the plan and N, never on the
// schedule): the wavefront is split into G groups of LPR lanes; entry i of the
// segment is accumulated by group i mod G with fmaf, in increasing i; the
// groups are then combined by an xor butterfly.  Segments of a split row are
// added in segment order.  No floating-point atomics are used anywhere.
#pragma once

#include <type_traits>

#include "devplan.hpp"
namespace spmm {

enum { DT_F32 = 0, DT_BF16 = 1, DT_F16 = 2 };

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes at element alignment: a row of N columns with any leading dimension
// starts anywhere, and gfx950 reads and writes 16 bytes at such an address in
// one instruction (two cache lines where it straddles them)
typedef float f32x4e __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u32x4e __attribute__((ext_vector_type(4), aligned(2)));

// First column of chunk q of a panel of ncols >= E columns: a last chunk that
// would run past the panel starts at its last E columns instead, so every
// chunk is whole and in bounds; the columns it shares with the chunk before it
// are computed twice from the same operands in the same order, so both lanes
// store the same values.
template <int E>
__device__ __forceinline__ int chunk_col(int q, int ncols) {
    return E == 1 ? q : min(q * E, ncols - E);
}

// First column of panel p of width np: the last panel is widened to the left
// to hold a whole chunk.
template <int E>
__device__ __forceinline__ int panel_col(int p, int np, int n) {
    return E == 1 ? p * np : min(p * np, n - E);
}

__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ float f16_to_f32(uint32_t h) {
    return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}

template <int DT>
__device__ __forceinline__ float load_val(const void *base, int idx) {
    if constexpr (DT == DT_F32) {
        return __builtin_nontemporal_load(static_cast<const float *>(base) + idx);
    } else {
        uint32_t b = __builtin_nontemporal_load(static_cast<const unsigned short *>(base) + idx);
        return DT == DT_BF16 ? bf16_to_f32(b) : f16_to_f32(b);
    }
}

// NT selects the non-temporal cache policy (the line is streamed through L2
// and is the first to be evicted), used for B rows outside the hot set.
template <bool NT, class T>
__device__ __forceinline__ T ld(const T *p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT>
__device__ __forceinline__ f32x4 ld16(const float *p) {
    const f32x4e *q = reinterpret_cast<const f32x4e *>(p);
    if constexpr (NT) return __builtin_nontemporal_load(q);
    else return *q;
}
template <bool NT>
__device__ __forceinline__ u32x4 ld16(const unsigned short *p) {
    const u32x4e *q = reinterpret_cast<const u32x4e *>(p);
    if constexpr (NT) return __builtin_nontemporal_load(q);
    else return *q;
}

// A gathered chunk kept in its stored form until it is consumed, so that 16-bit
// B rows hold 4 registers per 8 elements while loads are in flight.
template <int BT, int E>
struct Raw {
    using T = typename std::conditional<E == 1, uint32_t,
                                        typename std::conditional<BT == DT_F32, f32x4, u32x4>::type>::type;
    T x;
};

template <int BT, int E, bool NT>
__device__ __forceinline__ void load_raw(const void *B, int64_t off, Raw<BT, E> &r) {
    if constexpr (E == 1) {
        if constexpr (BT == DT_F32)
            r.x = __float_as_uint(ld<NT>(static_cast<const float *>(B) + off));
        else
            r.x = ld<NT>(static_cast<const unsigned short *>(B) + off);
    } else if constexpr (BT == DT_F32) {
        r.x = ld16<NT>(static_cast<const float *>(B) + off);
    } else {
        r.x = ld16<NT>(static_cast<const unsigned short *>(B) + off);
    }
}

template <int BT, int E>
__device__ __forceinline__ void zero_raw(Raw<BT, E> &r) {
    if constexpr (E == 1) r.x = 0u;
    else if constexpr (BT == DT_F32) r.x = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    else r.x = u32x4{0u, 0u, 0u, 0u};
}

// acc[e] = fma(v, chunk[e], acc[e]) for the E elements of a raw chunk.
template <int BT, int E>
__device__ __forceinline__ void fma_raw(float v, const Raw<BT, E> &r, float (&acc)[E]) {
    if constexpr (E == 1) {
        const float b = BT == DT_F32 ? __uint_as_float(r.x)
                                     : (BT == DT_BF16 ? bf16_to_f32(r.x) : f16_to_f32(r.x));
        acc[0] = __builtin_fmaf(v, b, acc[0]);
    } else if constexpr (BT == DT_F32) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(v, r.x[e], acc[e]);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float lo, hi;
            if constexpr (BT == DT_BF16) {
                lo = __uint_as_float(r.x[i] << 16);
                hi = __uint_as_float(r.x[i] & 0xFFFF0000u);
            } else {
                lo = f16_to_f32(r.x[i] & 0xFFFFu);
                hi = f16_to_f32(r.x[i] >> 16);
            }
            acc[2 * i] = __builtin_fmaf(v, lo, acc[2 * i]);
            acc[2 * i + 1] = __builtin_fmaf(v, hi, acc[2 * i + 1]);
        }
    }
}

// The same chunk through a raw buffer load whose cache-policy bits are `aux`
// (gfx950: bit 0 sc0, bit 1 nt, bit 4 sc1).  A distinct intrinsic, so the
// compiler never merges it with the default-policy load of a hot row.
template <int AUX>
__device__ __forceinline__ u32x4 buf16(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, AUX);
}
template <int AUX>
__device__ __forceinline__ uint32_t buf4(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, AUX);
}
template <int AUX>
__device__ __forceinline__ uint32_t buf2(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, AUX);
}

template <int BT, int E>
__device__ __forceinline__ void load_raw_policy(__amdgpu_buffer_rsrc_t rs, int64_t off, int aux,
                                                Raw<BT, E> &r) {
    constexpr int SB = BT == DT_F32 ? 4 : 2;
    const uint32_t boff = (uint32_t)(off * SB);
    if constexpr (E == 1) {
        if constexpr (SB == 4) {
            switch (aux) {
            case 2: r.x = buf4<2>(rs, boff); break;
            case 16: r.x = buf4<16>(rs, boff); break;
            case 18: r.x = buf4<18>(rs, boff); break;
            default: r.x = buf4<0>(rs, boff); break;
            }
        } else {
            switch (aux) {
            case 2: r.x = buf2<2>(rs, boff); break;
            case 16: r.x = buf2<16>(rs, boff); break;
            case 18: r.x = buf2<18>(rs, boff); break;
            default: r.x = buf2<0>(rs, boff); break;
            }
        }
    } else {
        u32x4 x;
        switch (aux) {
        case 2: x = buf16<2>(rs, boff); break;
        case 16: x = buf16<16>(rs, boff); break;
        case 18: x = buf16<18>(rs, boff); break;
        default: x = buf16<0>(rs, boff); break;
        }
        if constexpr (BT == DT_F32) r.x = __builtin_bit_cast(f32x4, x);
        else r.x = x;
    }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t b_resource(const void *B, uint32_t rec) {
    // raw buffer over B: stride 0, `rec` bytes addressable (all 2^32-1 when 0),
    // gfx9 word-3 flags; a load at or beyond `rec` returns zeros and moves no data
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(B), (short)0,
                                             rec ? (int)rec : (int)0xFFFFFFFF, 0x00020000);
}

// A raw chunk through the default-policy buffer load at byte offset `off`.
template <int BT, int E>
__device__ __forceinline__ void load_raw_buf(__amdgpu_buffer_rsrc_t rs, uint32_t off, Raw<BT, E> &r) {
    if constexpr (E == 1) {
        if constexpr (BT == DT_F32) r.x = buf4<0>(rs, off);
        else r.x = buf2<0>(rs, off);
    } else {
        const u32x4 x = buf16<0>(rs, off);
        if constexpr (BT == DT_F32) r.x = __builtin_bit_cast(f32x4, x);
        else r.x = x;
    }
}

template <int E>
__device__ __forceinline__ void store_chunk(float *C, int64_t off, const float (&v)[E]) {
    if constexpr (E == 1) {
        __builtin_nontemporal_store(v[0], C + off);
    } else {
#pragma unroll
        for (int i = 0; i < E; i += 4) {
            f32x4e x = {v[i], v[i + 1], v[i + 2], v[i + 3]};
            __builtin_nontemporal_store(x, reinterpret_cast<f32x4e *>(C + off + i));
        }
    }
}

template <int E>
__device__ __forceinline__ void load_f32_chunk(const float *W, int64_t off, float (&v)[E]) {
    if constexpr (E == 1) {
        v[0] = W[off];
    } else {
#pragma unroll
        for (int i = 0; i < E; i += 4) {
            f32x4 x = *reinterpret_cast<const f32x4e *>(W + off + i);
            v[i] = x[0]; v[i + 1] = x[1]; v[i + 2] = x[2]; v[i + 3] = x[3];
        }
    }
}

// Workgroup id after the optional XCD remap: workgroups are dispatched
// round-robin over the 8 XCDs, so id b runs on XCD b % 8.  The remap gives
// each XCD one contiguous range of logical ids, so neighbouring items (which
// tend to share rows of B) share that XCD's L2.
// Logical id of workgroup b of a range of nwg workgroups whose first one runs
// on XCD 0 (ranges of a fused launch start at multiples of 8).
__device__ __forceinline__ int remap_block(int b, int nwg) {
    const int full = nwg >> 3, rem = nwg & 7, x = b & 7, local = b >> 3;
    return (x < rem ? x * (full + 1) : rem * (full + 1) + (x - rem) * full) + local;
}

__device__ __forceinline__ int logical_block(int xcd) {
    const int b = blockIdx.x;
    if (!xcd) return b;
    return remap_block(b, gridDim.x);
}

// This wave's index in its workgroup, as a wave-uniform (scalar) value, so
// that the item and descriptor loads that depend on it are scalar loads.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Lane layout of the gather-FMA: lane = group * LPR + li; lane li of a group
// owns chunks q = c * LPR + li (c < CPL), i.e. columns q*E .. q*E+E-1 of the
// panel.
struct Lanes {
    int lpr_log2, lpr, groups, group, li;
    __device__ __forceinline__ Lanes() = default;
    __device__ __forceinline__ explicit Lanes(int lg) {
        const int lane = threadIdx.x & 63;
        lpr_log2 = lg;
        lpr = 1 << lg;
        groups = 64 >> lg;
        group = lane >> lg;
        li = lane & (lpr - 1);
    }
    // the same lane position with entry stride 1: the group walks a row alone
    __device__ __forceinline__ Lanes single() const {
        Lanes o = *this;
        o.groups = 1;
        return o;
    }
};

// Entries p, p + G, ..., p + (U-1)G of a group (masked at p1): columns and values.
// CLAMP: every load is issued, at an index clamped into [0, p1 - 1], with no
// branch around it (a branch can make the compiler wait for each load before
// issuing the next); a masked entry gets value 0 and the column of the
// clamped entry, which is a real column when p < p1 (the plan arrays carry a
// zero tail for the empty case).  Otherwise masked entries are not loaded, so
// a step whose entries are all masked issues nothing.  Measured: clamping
// pays where gathers are small and latency-bound (16-bit B), predication
// where they are large and bandwidth-bound (f32 B).
template <int VT, int U, bool CLAMP>
__device__ __forceinline__ void load_entries(const int32_t *__restrict__ rcol,
                                             const void *__restrict__ rval, int p, int p1,
                                             const Lanes &L, int (&col)[U], float (&v)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int pp = p + u * L.groups;
        if constexpr (CLAMP) {
            const int q = max(min(pp, p1 - 1), 0);
            col[u] = __builtin_nontemporal_load(rcol + q);
            const float x = load_val<VT>(rval, q);
            v[u] = pp < p1 ? x : 0.0f;
        } else {
            const bool ok = pp < p1;
            col[u] = ok ? __builtin_nontemporal_load(rcol + pp) : 0;
            v[u] = ok ? load_val<VT>(rval, pp) : 0.0f;
        }
    }
}

// Gathers the B rows of U loaded entries (hot rows cacheable, the others with
// the cold policy) and accumulates them in entry order.
// POL: the per-entry cache-policy choice is compiled in (row-by-row variant
// and segments of plans with a cold policy); without it every gather uses the
// default policy and the loop carries no per-entry branches.
template <int BT, int E, int CPL, int U, bool POL = false>
__device__ __forceinline__ void gather_fma(const int (&col)[U], const float (&v)[U], int p, int p1,
                                           const void *__restrict__ B,
                                           __amdgpu_buffer_rsrc_t rs, int64_t ldb, uint32_t brec,
                                           const bool (&cok)[CPL], const int64_t (&coff)[CPL],
                                           const Lanes &L, int cold_aux, float (&acc)[CPL][E]) {
    constexpr int SB = BT == DT_F32 ? 4 : 2;
    Raw<BT, E> b[U][CPL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool ok = p + u * L.groups < p1;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            // bit 31 of a column marks a hot B row (cacheable gather)
            const int64_t boff = (int64_t)(col[u] & 0x7FFFFFFF) * ldb + coff[c];
            if constexpr (POL) {
                if (ok && cok[c] && (col[u] < 0 || cold_aux < 0)) {
                    load_raw<BT, E, false>(B, boff, b[u][c]);
                } else if (ok && cok[c]) {
                    // (rows not aligned to 4 bytes: plain loads, which know nt only)
                    if (brec != 0) load_raw_policy<BT, E>(rs, boff, cold_aux, b[u][c]);
                    else if (cold_aux & 2) load_raw<BT, E, true>(B, boff, b[u][c]);
                    else load_raw<BT, E, false>(B, boff, b[u][c]);
                } else {
                    zero_raw<BT, E>(b[u][c]);
                }
            } else {
                // No branch around a load when B is addressable by a buffer
                // resource (a branch makes the compiler wait for each load
                // before issuing the next): a masked entry or a chunk outside
                // the panel loads at offset brec, out of the buffer's range,
                // which returns zeros without a memory access.  Without one:
                // f32 B (spanning 4 GiB or more) takes predicated plain loads;
                // 16-bit B (that, or rows not aligned to 4 bytes) plain loads
                // throughout, a masked entry's from the row its clamped entry
                // names (a row of B), whose value is not used.
                (void)cold_aux;
                if (brec != 0) {
                    load_raw_buf<BT, E>(rs, ok && cok[c] ? (uint32_t)(boff * SB) : brec, b[u][c]);
                } else if (BT != DT_F32 || (ok && cok[c])) {
                    load_raw<BT, E, false>(B, boff, b[u][c]);
                } else {
                    zero_raw<BT, E>(b[u][c]);
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (p + u * L.groups < p1) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) fma_raw<BT, E>(v[u], b[u][c], acc[c]);
        }
    }
}

template <int E, int CPL>
__device__ __forceinline__ void chunk_layout(int ncol0, int ncols, const Lanes &L, bool (&cok)[CPL],
                                             int64_t (&coff)[CPL]) {
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int q = c * L.lpr + L.li;
        cok[c] = q * E < ncols;
        coff[c] = ncol0 + (cok[c] ? chunk_col<E>(q, ncols) : 0);  // a valid chunk when outside the panel
    }
}

// Entries of a row (or segment) held by the lanes that sum it: a block of
// `groups` lane groups, whose lane l of `span` holds entries l and span + l of
// those from the hold's first on (at clamped indices: a real entry of the row).
// Two coalesced loads of each array serve as many steps as the hold spans,
// where every lane loading its own group's entries takes 2 U loads a step, each
// of one entry per group.  A run whose gathers fill the card is bound by loads in
// flight, and the entry loads took half of its load slots (graphs, us, own loads
// / held: 2^20 rows, N = 128 of f32 956 / 884; 500,000, N = 256 of f16 558 / 479;
// 200,000, N = 47 of f32 102 / 89; 64 uneven f16 matrices in a batch
// 1183 / 1002).  Smaller and narrower runs get slower (the rule and both sides:
// make_run_args).  Also loading the next hold or the next rows' entries ahead
// costs registers and gained nothing (2^20 rows: 934 and 1052 us).
struct Hold {
    int c[2];
    float v[2];
};
template <int VT>
__device__ __forceinline__ void load_hold(const int32_t *__restrict__ rcol, const void *__restrict__ rval, int p,
                                          int p1, int l, int span, Hold &h) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int q = max(min(p + k * span + l, p1 - 1), 0);
        h.c[k] = __builtin_nontemporal_load(rcol + q);
        h.v[k] = load_val<VT>(rval, q);
    }
}

// acc += sum over entries [p0, p1) of v_p * B[col_p][panel columns], entry
// p0 + i taken by group i mod L.groups of the block, in increasing i (see the
// file comment); `local` is this lane's group in the block, which starts at
// lane `first`.
template <int VT, int BT, int E, int CPL, int U, bool POL, bool HOLD>
__device__ __forceinline__ void accumulate(const int32_t *__restrict__ rcol, const void *__restrict__ rval, int p0,
                                           int p1, const void *__restrict__ B, int64_t ldb, uint32_t brec,
                                           const bool (&cok)[CPL], const int64_t (&coff)[CPL], const Lanes &L,
                                           int first, int local, int cold_aux, float (&acc)[CPL][E]) {
    const __amdgpu_buffer_rsrc_t rs = b_resource(B, brec);
    const int S = L.groups, step = S * U;
    // A batch's kernels hold entries at any width (single runs: make_run_args);
    // narrow rows load their own: a hold of theirs is no longer than a step, or
    // (f32, fewer than 16 lanes a row) the hand-out costs more than the loads.
    if (!HOLD || (BT == DT_F32 ? L.lpr < 2 * U : 2 * L.lpr < U)) {
        for (int p = p0 + local; p < p1; p += step) {
            int col[U];
            float v[U];
            load_entries<VT, U, BT != DT_F32>(rcol, rval, p, p1, L, col, v);
            gather_fma<BT, E, CPL, U, POL>(col, v, p, p1, B, rs, ldb, brec, cok, coff, L, cold_aux, acc);
        }
        return;
    }
    const int span = S * L.lpr, l = (int)(threadIdx.x & 63) - first;
    for (int pb = p0; pb < p1; pb += 2 * span) {
        Hold h;
        load_hold<VT>(rcol, rval, pb, p1, l, span, h);
        for (int t = 0; t < 2 * L.lpr && pb + t * S < p1; t += U) {
            const int p = pb + t * S + local;
            auto from = [&](int u, int lo, int hi) {  // entry u of this group
                const int src = (first + ((t + u) & (L.lpr - 1)) * S + local) << 2;
                return __builtin_amdgcn_ds_bpermute(src, t + u >= L.lpr ? hi : lo);
            };
            int col[U];
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) col[u] = from(u, h.c[0], h.c[1]);
            if constexpr (BT == DT_F32 || POL) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    v[u] = __int_as_float(from(u, __float_as_int(h.v[0]), __float_as_int(h.v[1])));
                gather_fma<BT, E, CPL, U, POL>(col, v, p, p1, B, rs, ldb, brec, cok, coff, L, cold_aux, acc);
            } else {
                // 16-bit rows: the values behind the gathers, in the columns'
                // registers (batched kernel 104 -> 90)
                Raw<BT, E> b[U][CPL];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        const int64_t boff = (int64_t)(col[u] & 0x7FFFFFFF) * ldb + coff[c];
                        const bool ok = p + u * S < p1 && cok[c];
                        if (brec != 0) load_raw_buf<BT, E>(rs, ok ? (uint32_t)(boff * 2) : brec, b[u][c]);
                        else load_raw<BT, E, false>(B, boff, b[u][c]);
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    v[u] = __int_as_float(from(u, __float_as_int(h.v[0]), __float_as_int(h.v[1])));
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (p + u * S < p1) {
#pragma unroll
                        for (int c = 0; c < CPL; ++c) fma_raw<BT, E>(v[u], b[u][c], acc[c]);
                    }
            }
        }
    }
}

// The same for one row on the whole wavefront.
template <int VT, int BT, int E, int CPL, int U, bool POL, bool HOLD>
__device__ __forceinline__ void seg_accumulate(const int32_t *__restrict__ rcol,
                                               const void *__restrict__ rval, int p0, int p1,
                                               const void *__restrict__ B, int64_t ldb, uint32_t brec,
                                               int ncol0, int ncols, const Lanes &L, int cold_aux,
                                               float (&acc)[CPL][E]) {
    bool cok[CPL];
    int64_t coff[CPL];
    chunk_layout<E, CPL>(ncol0, ncols, L, cok, coff);
    accumulate<VT, BT, E, CPL, U, POL, HOLD>(rcol, rval, p0, p1, B, ldb, brec, cok, coff, L, 0, L.group, cold_aux, acc);
}

// acc += sum over entries [p0, p1) of one row, all taken by this lane's group
// in increasing order (each group works on its own row).
template <int VT, int BT, int E, int CPL, int U, bool POL, bool HOLD>
__device__ __forceinline__ void row_accumulate_group(const int32_t *__restrict__ rcol,
                                                     const void *__restrict__ rval, int p0, int p1,
                                                     const void *__restrict__ B, int64_t ldb,
                                                     uint32_t brec, int ncol0, int ncols,
                                                     const Lanes &L, int cold_aux,
                                                     float (&acc)[CPL][E]) {
    bool cok[CPL];
    int64_t coff[CPL];
    chunk_layout<E, CPL>(ncol0, ncols, L, cok, coff);
    accumulate<VT, BT, E, CPL, U, POL, HOLD>(rcol, rval, p0, p1, B, ldb, brec, cok, coff, L.single(), L.group * L.lpr, 0,
                                       cold_aux, acc);
}

template <int E, int CPL>
__device__ __forceinline__ void group_reduce(float (&acc)[CPL][E], const Lanes &L) {
    for (int off = 32; off >= L.lpr; off >>= 1) {
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int e = 0; e < E; ++e) acc[c][e] += __shfl_xor(acc[c][e], off, 64);
    }
}

// Stores and loads of parts exchanged between the workgroups of one launch
// (co-scheduled execution) go through the workspace as a raw buffer with the
// device-scope cache policy (sc1): stores write through an XCD's L2 (each XCD
// has its own) and loads read past it, so a part stored on one XCD is read
// intact on another once its store has completed.  Offsets are in floats from
// the workspace base (a co-scheduled run keeps its workspace below 4 GiB).
constexpr int kDevScope = 16;  // gfx950 buffer cache-policy bits: sc1

__device__ __forceinline__ __amdgpu_buffer_rsrc_t ws_resource(const RunArgs &a) {
    return b_resource(a.work, a.ws_rec);
}
__device__ __forceinline__ void st_dev1(__amdgpu_buffer_rsrc_t rs, int64_t off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, (uint32_t)(off * 4), 0, kDevScope);
}
__device__ __forceinline__ f32x4 ld_dev4(__amdgpu_buffer_rsrc_t rs, int64_t off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (uint32_t)(off * 4), 0, kDevScope));
}
template <int E>
__device__ __forceinline__ void st_dev_chunk(__amdgpu_buffer_rsrc_t rs, int64_t off, const float (&v)[E]) {
    if constexpr (E == 1) {
        st_dev1(rs, off, v[0]);
    } else {
#pragma unroll
        for (int i = 0; i < E; i += 4)
            __builtin_amdgcn_raw_buffer_store_b128(
                __builtin_bit_cast(u32x4, f32x4{v[i], v[i + 1], v[i + 2], v[i + 3]}), rs,
                (uint32_t)((off + i) * 4), 0, kDevScope);
    }
}
template <int E>
__device__ __forceinline__ void ld_dev_chunk(__amdgpu_buffer_rsrc_t rs, int64_t off, float (&v)[E]) {
    if constexpr (E == 1) {
        v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (uint32_t)(off * 4), 0, kDevScope));
    } else {
#pragma unroll
        for (int i = 0; i < E; i += 4) {
            const f32x4 x = ld_dev4(rs, off + i);
            v[i] = x[0]; v[i + 1] = x[1]; v[i + 2] = x[2]; v[i + 3] = x[3];
        }
    }
}

// acc = P[sid] + P[sid+1] + ... + P[sid+ns-1] (panel columns), in that order.
// DEV: the partials were stored by other workgroups of this launch (rs: the
// workspace); loads go out four segments at a time.
template <int E, int CPL, bool DEV = false>
__device__ __forceinline__ void sum_partials(const float *__restrict__ work, int64_t ld, int sid,
                                             int ns, int ncol0, int ncols, const Lanes &L,
                                             float (&acc)[CPL][E],
                                             __amdgpu_buffer_rsrc_t rs = b_resource(nullptr, 0u)) {
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int q = c * L.lpr + L.li;
        if (q * E >= ncols) continue;
        const int64_t off = ncol0 + chunk_col<E>(q, ncols);
        if constexpr (DEV) {
            (void)work;
            ld_dev_chunk<E>(rs, (int64_t)sid * ld + off, acc[c]);
            for (int j0 = 1; j0 < ns; j0 += 4) {
                float t[4][E];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    ld_dev_chunk<E>(rs, (int64_t)(sid + min(j0 + u, ns - 1)) * ld + off, t[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (j0 + u < ns) {
#pragma unroll
                        for (int e = 0; e < E; ++e) acc[c][e] += t[u][e];
                    }
            }
        } else {
            load_f32_chunk<E>(work, (int64_t)sid * ld + off, acc[c]);
            for (int j = 1; j < ns; ++j) {
                float t[E];
                load_f32_chunk<E>(work, (int64_t)(sid + j) * ld + off, t);
#pragma unroll
                for (int e = 0; e < E; ++e) acc[c][e] += t[e];
            }
        }
    }
}

template <int E, int CPL>
__device__ __forceinline__ void store_row(float *C, int64_t row_off, int ncol0, int ncols,
                                          const Lanes &L, const float (&acc)[CPL][E]) {
    if (L.group != 0) return;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int q = c * L.lpr + L.li;
        if (q * E < ncols) store_chunk<E>(C, row_off + ncol0 + chunk_col<E>(q, ncols), acc[c]);
    }
}

template <int E, int CPL>
constexpr int unroll_of() { return E == 1 ? 4 : (CPL == 1 ? 8 : 4); }

// ------------------------------------------------------------------------------------------
// Co-scheduled execution.  Segments, vector items, window owners and window
// partial items run side by side, so no item waits for a kernel boundary.  A
// result made of several items' parts (a split row's segment partials; a
// window's MFMA result, its partial tiles and its split rows) is finished by
// whichever contributor comes last: each contributor stores its part with
// device-coherent stores (st_dev), waits until they have completed, then adds
// 1 to the result's integer counter in global memory with a device-scope
// atomic; the one whose increment reaches the target reads every part with
// device-coherent loads (ld_dev), sums them in the same fixed order as the
// serial kernels, writes C, and clears the counter for the next run.  No
// contributor ever waits for another, so any schedule completes, and C is
// bitwise the same as with one kernel per item kind.  (A full device-scope
// fence instead writes back the whole XCD L2 at every arrival: measured 4x
// slower on the 2^20-vertex graph's 62,629 segments.)

// Waits until this wave's stores have completed.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// One wavefront arrives at a counter; true on every lane of the last arrival.
__device__ __forceinline__ bool wave_arrive(int32_t *cnt, int target) {
    stores_done();
    int old = 0;
    if ((threadIdx.x & 63) == 0) {
        old = atomicAdd(cnt, 1);
        if (old == target - 1) atomicExch(cnt, 0);
    }
    old = __shfl(old, 0, 64);
    return old == target - 1;
}

// Counter of window slot `dep` in window panel q (win_np columns) and row
// share `sub` (one of the win_subs waves of a window item).
__device__ __forceinline__ int32_t *win_counter(const DevPlan &P, const RunArgs &a, int q, int dep, int sub) {
    return a.cnt + (int64_t)a.n_panels * P.n_seg + ((int64_t)q * P.n_dep + dep) * a.win_subs + sub;
}

// Arrivals each row share of a window panel waits for: its owner, its partial
// items, and every segment panel (width np) overlapping the window panel for
// each segment of the window's split rows (a segment arrives at every share).
__device__ __forceinline__ int win_target(const DevPlan &P, const RunArgs &a, int w, int q) {
    const int c0 = q * a.win_np, c1 = min(P.n, c0 + a.win_np) - 1;
    return 1 + (P.win_part[w + 1] - P.win_part[w]) + P.win_nsseg[w] * (c1 / a.np - c0 / a.np + 1);
}

// The last arrival of window w, panel q, row share `sub`: for each of its
// rows, the MFMA result plus the partial tiles' results in tile order, plus
// the remainder (the owner's sum, or the row's segment partials in segment
// order), written to C.  Lane t takes 4-column chunks t, t + 64, ... of the
// rows x panel columns (the workspace rows are padded to a multiple of 4
// columns, so a chunk load stays in its row).
// UN: chunks whose loads a lane has in flight together (the parts come past
// L2, some microseconds each way).
template <int UN>
__device__ __forceinline__ void window_combine(const DevPlan &P, const RunArgs &a, int w, int q, int dep,
                                               int sub) {
    const int H = P.H, rows = H / a.win_subs;  // (win_rows 1: rows sub % 4, + 4, + 8, + 12 of block sub / 4)
    const int first = a.win_rows == 1 ? (sub >> 2) * 16 + (sub & 3) : sub * rows, step = a.win_rows == 1 ? 4 : 1;
    const int ncol0 = q * a.win_np, ncols = min(a.win_np, P.n - ncol0), nch = (ncols + 3) >> 2;
    const int pa = P.win_part[w], pb = P.win_part[w + 1];
    const int64_t ld = a.work_ld;
    const __amdgpu_buffer_rsrc_t rs = ws_resource(a);
    const int64_t wp0 = (int64_t)P.n_seg * ld;                                // window partials
    const int64_t cs0 = wp0 + ((int64_t)H * P.n_wpart + (int64_t)dep * 2 * H) * ld;  // slot: MFMA result
    const int64_t rm0 = cs0 + (int64_t)H * ld;                                // slot: remainders
    const int total = rows * nch;
    for (int u0 = threadIdx.x & 63; u0 < total; u0 += 64 * UN) {
        int r[UN], sid[UN], s[UN], c[UN];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const int u = min(u0 + 64 * i, total - 1);
            s[i] = first + u / nch * step;
            c[i] = u % nch;
            r[i] = P.windows[(int64_t)w * H + s[i]];
            sid[i] = P.win_row_sid[(int64_t)w * H + s[i]];
        }
        f32x4 v[UN], y[UN];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const int64_t col = ncol0 + 4 * c[i];
            v[i] = ld_dev4(rs, cs0 + (int64_t)s[i] * ld + col);
            // (of a split row: its first segment's partial)
            y[i] = ld_dev4(rs, (sid[i] >= 0 ? (int64_t)sid[i] * ld : rm0 + (int64_t)s[i] * ld) + col);
        }
        for (int k0 = pa; k0 < pb; k0 += 4) {
            f32x4 x[UN][4];
#pragma unroll
            for (int i = 0; i < UN; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    x[i][k] = ld_dev4(rs, wp0 + ((int64_t)min(k0 + k, pb - 1) * H + s[i]) * ld + ncol0 + 4 * c[i]);
#pragma unroll
            for (int i = 0; i < UN; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k0 + k < pb) v[i] += x[i][k];
        }
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            if (u0 + 64 * i >= total || r[i] < 0) continue;
            const int64_t col = ncol0 + 4 * c[i];
            if (sid[i] >= 0) {
                const int len = P.rem_ptr[r[i] + 1] - P.rem_ptr[r[i]];
                const int ns = (len + P.seg_len - 1) / P.seg_len;
                for (int j0 = 1; j0 < ns; j0 += 4) {
                    f32x4 x[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) x[k] = ld_dev4(rs, (int64_t)(sid[i] + min(j0 + k, ns - 1)) * ld + col);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (j0 + k < ns) y[i] += x[k];
                }
            }
            const f32x4 z = v[i] + y[i];
            float *dst = a.C + (int64_t)r[i] * a.ldc + col;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * c[i] + e < ncols) dst[e] = z[e];
        }
    }
}

// ------------------------------------------------------------------------------------------
// One segment (of one panel) per wavefront: wid in [0, n_seg * n_panels).
// FUSED: the segment then arrives at its row's counter (a vector row) or its
// window's counters (a window row), and the last arrival finishes the result.
template <int VT, int BT, int E, int CPL, bool POL, bool FUSED, bool HOLD>
__device__ __forceinline__ void segment_item(const DevPlan &P, const RunArgs &a, int wid) {
    const int panel = wid / P.n_seg, li = wid - panel * P.n_seg;
    const int sid = P.seg_order ? P.seg_order[li] : li;  // the partial's slot
    const int ncol0 = panel_col<E>(panel, a.np, P.n), ncols = min(a.np, P.n - ncol0);
    const Lanes L(a.lpr_log2);
    float acc[CPL][E];
#pragma unroll
    for (int c = 0; c < CPL; ++c)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[c][e] = 0.0f;
    seg_accumulate<VT, BT, E, CPL, unroll_of<E, CPL>(), POL, HOLD>(P.rem_col, P.rem_val, P.seg_begin[sid],
                                                              P.seg_end[sid], a.B, a.ldb, a.b_rec, ncol0, ncols,
                                                              L, a.cold_aux, acc);
    group_reduce<E, CPL>(acc, L);
    if (L.group == 0) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int q = c * L.lpr + L.li;
            if (q * E < ncols) {
                const int64_t off = (int64_t)sid * a.work_ld + ncol0 + chunk_col<E>(q, ncols);
                float *dst = a.work + off;
                if constexpr (FUSED) {
                    st_dev_chunk<E>(ws_resource(a), off, acc[c]);
                } else if constexpr (E == 1) {
                    dst[0] = acc[c][0];
                } else {
#pragma unroll
                    for (int i = 0; i < E; i += 4)
                        *reinterpret_cast<f32x4e *>(dst + i) =
                            f32x4e{acc[c][i], acc[c][i + 1], acc[c][i + 2], acc[c][i + 3]};
                }
            }
        }
    }
    if constexpr (FUSED) {
        // segments of a row have consecutive ids, segment j starting j * seg_len
        // entries into the row's remainder
        const int r = P.seg_row[sid];
        const int rb = P.rem_ptr[r], re = P.rem_ptr[r + 1];
        const int ns = (re - rb + P.seg_len - 1) / P.seg_len;
        const int sid0 = sid - (P.seg_begin[sid] - rb) / P.seg_len;
        const int w = P.seg_win ? P.seg_win[sid] : -1;
        if (w < 0) {
            if (wave_arrive(a.cnt + (int64_t)panel * P.n_seg + sid0, ns)) {
                // the vector items' sum of a split row, in segment order
                sum_partials<E, CPL, true>(a.work, a.work_ld, sid0, ns, ncol0, ncols, L, acc, ws_resource(a));
                store_row<E, CPL>(a.C, (int64_t)r * a.ldc, ncol0, ncols, L, acc);
            }
        } else {
            const int dep = P.win_dep[w];
            // (the panel's own columns, without those it was widened by: win_target)
            for (int q = panel * a.np / a.win_np; q <= (ncol0 + ncols - 1) / a.win_np; ++q)
                for (int sub = 0; sub < a.win_subs; ++sub)
                    if (wave_arrive(win_counter(P, a, q, dep, sub), win_target(P, a, w, q)))
                        window_combine<1>(P, a, w, q, dep, sub);
        }
    }
}

// One vector work item (of one panel) per wavefront: wid in [0, n_vitems * n_panels).
// FUSED (every variant): a split row is finished by its last segment, so the
// item skips it.
template <int VT, int BT, int E, int CPL, bool FUSED = false>
__device__ __forceinline__ void vector_item(const DevPlan &P, const RunArgs &a, int wid) {
    const int panel = wid / P.n_vitems, item = wid - panel * P.n_vitems;
    const int ncol0 = panel_col<E>(panel, a.np, P.n), ncols = min(a.np, P.n - ncol0);
    const Lanes L(a.lpr_log2);
    int sid = P.vitem_seg[item];
    const int i0 = P.vitem_ptr[item], i1 = P.vitem_ptr[item + 1];
    for (int i = i0; i < i1; ++i) {
        const int r = P.vec_rows ? P.vec_rows[i] : i;
        const int b = P.rem_ptr[r], e = P.rem_ptr[r + 1];
        float acc[CPL][E];
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int x = 0; x < E; ++x) acc[c][x] = 0.0f;
        if (e - b <= P.seg_len) {
            seg_accumulate<VT, BT, E, CPL, unroll_of<E, CPL>(), true, false>(P.rem_col, P.rem_val, b, e, a.B,
                                                                       a.ldb, a.b_rec, ncol0, ncols, L,
                                                                       a.cold_aux, acc);
            group_reduce<E, CPL>(acc, L);
        } else {
            if constexpr (FUSED) continue;
            const int ns = (e - b + P.seg_len - 1) / P.seg_len;
            sum_partials<E, CPL>(a.work, a.work_ld, sid, ns, ncol0, ncols, L, acc);
            sid += ns;
        }
        store_row<E, CPL>(a.C, (int64_t)r * a.ldc, ncol0, ncols, L, acc);
    }
}

// Vector work item with a software pipeline across its rows: while a row's
// B rows are being gathered, the next row's pointers and first batch of
// (column, value) are already in flight.  Each row's entries are consumed in
// exactly the order of vector_item, so the results are bitwise identical.
template <int VT, int BT, int E, int CPL, bool FUSED = false>
__device__ __forceinline__ void vector_item_pipelined(const DevPlan &P, const RunArgs &a, int wid) {
    constexpr int U = unroll_of<E, CPL>();
    const int panel = wid / P.n_vitems, item = wid - panel * P.n_vitems;
    const int ncol0 = panel_col<E>(panel, a.np, P.n), ncols = min(a.np, P.n - ncol0);
    const Lanes L(a.lpr_log2);
    const int step = L.groups * U;
    const __amdgpu_buffer_rsrc_t rs = b_resource(a.B, a.b_rec);
    bool cok[CPL];
    int64_t coff[CPL];
    chunk_layout<E, CPL>(ncol0, ncols, L, cok, coff);
    int sid = P.vitem_seg[item];
    const int i0 = P.vitem_ptr[item], i1 = P.vitem_ptr[item + 1];

    int r = P.vec_rows ? P.vec_rows[i0] : i0;
    int b = P.rem_ptr[r], e = P.rem_ptr[r + 1];
    int col[U];
    float v[U];
    load_entries<VT, U, BT != DT_F32>(P.rem_col, P.rem_val, b + L.group, e - b <= P.seg_len ? e : b, L, col, v);
    for (int i = i0; i < i1; ++i) {
        int nr = r, nb = 0, ne = 0;
        if (i + 1 < i1) {
            nr = P.vec_rows ? P.vec_rows[i + 1] : i + 1;
            nb = P.rem_ptr[nr];
            ne = P.rem_ptr[nr + 1];
        }
        float acc[CPL][E];
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int x = 0; x < E; ++x) acc[c][x] = 0.0f;
        int ncl[U];
        float nv[U];
        if (e - b <= P.seg_len) {
            Raw<BT, E> bv[U][CPL];
            // gathers of this row's first batch
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool ok = b + L.group + u * L.groups < e;
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    const int64_t boff = (int64_t)(col[u] & 0x7FFFFFFF) * a.ldb + coff[c];
                    if (ok && cok[c]) load_raw<BT, E, false>(a.B, boff, bv[u][c]);
                    else zero_raw<BT, E>(bv[u][c]);
                }
            }
            // the next row's first batch, in flight behind the gathers
            load_entries<VT, U, BT != DT_F32>(P.rem_col, P.rem_val, nb + L.group, ne - nb <= P.seg_len ? ne : nb,
                                L, ncl, nv);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (b + L.group + u * L.groups < e) {
#pragma unroll
                    for (int c = 0; c < CPL; ++c) fma_raw<BT, E>(v[u], bv[u][c], acc[c]);
                }
            }
            // the rest of a row longer than one batch, continuing the same order
            for (int p = b + step + L.group; p < e; p += step) {
                int c2[U];
                float v2[U];
                load_entries<VT, U, BT != DT_F32>(P.rem_col, P.rem_val, p, e, L, c2, v2);
                gather_fma<BT, E, CPL, U>(c2, v2, p, e, a.B, rs, a.ldb, a.b_rec, cok, coff, L, a.cold_aux,
                                          acc);
            }
            group_reduce<E, CPL>(acc, L);
        } else {
            load_entries<VT, U, BT != DT_F32>(P.rem_col, P.rem_val, nb + L.group, ne - nb <= P.seg_len ? ne : nb,
                                L, ncl, nv);
            if constexpr (!FUSED) {
                const int ns = (e - b + P.seg_len - 1) / P.seg_len;
                sum_partials<E, CPL>(a.work, a.work_ld, sid, ns, ncol0, ncols, L, acc);
                sid += ns;
            }
        }
        if (!FUSED || e - b <= P.seg_len) store_row<E, CPL>(a.C, (int64_t)r * a.ldc, ncol0, ncols, L, acc);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            col[u] = ncl[u];
            v[u] = nv[u];
        }
        r = nr;
        b = nb;
        e = ne;
    }
}

// Inclusive prefix sum over the 64 lanes of a wavefront.
__device__ __forceinline__ int wave_inclusive_scan(int x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int t = __shfl_up(x, d, 64);
        if (lane >= d) x += t;
    }
    return x;
}

// Vector work item with short rows packed one per lane group: a row whose
// remainder has at most 2U entries is summed in entry order by one group, and
// up to G such consecutive rows are gathered at once; longer rows take the
// whole wavefront as in vector_item.  The rule depends only on a row's length.
// The row ids and remainder ranges of the next 64 rows are loaded once, one
// row per lane, and handed to the groups by lane shuffles as the rows are
// taken, so a batch of short rows starts with its entry loads.
// UL: entries per group and step; the short-row bound stays 2 unroll_of, so
// the summation order (which depends only on a row's length) is the same for
// any UL.
template <int VT, int BT, int E, int CPL, bool FUSED, int UL, bool HOLD>
__device__ __forceinline__ void vector_item_packed(const DevPlan &P, const RunArgs &a, int wid) {
    constexpr int U = UL;
    constexpr int SHORT = 2 * unroll_of<E, CPL>();
    const int panel = wid / P.n_vitems, item = wid - panel * P.n_vitems;
    const int ncol0 = panel_col<E>(panel, a.np, P.n), ncols = min(a.np, P.n - ncol0);
    const Lanes L(a.lpr_log2);
    const int lane = threadIdx.x & 63;
    int sid = P.vitem_seg[item];
    const int i0 = P.vitem_ptr[item], i1 = P.vitem_ptr[item + 1];
    for (int i = i0; i < i1; i += 64) {
        // the next (up to 64) rows, one per lane: id and remainder range
        const int li_row = i + lane;
        int rr = 0, rb = 0, re = 0, len = 0x7FFFFFFF;
        if (li_row < i1) {
            rr = P.vec_rows ? P.vec_rows[li_row] : li_row;
            rb = P.rem_ptr[rr];
            re = P.rem_ptr[rr + 1];
            len = re - rb;
        }
        const uint64_t longmask = __ballot(len > SHORT || len > P.seg_len || li_row >= i1);
        const int avail = min(64, i1 - i);
        int j = 0;
        while (j < avail) {
            // k = consecutive short rows from j, at most G
            const uint64_t lm = longmask >> j;
            int k = lm ? __builtin_ctzll(lm) : 64 - j;
            k = min(k, L.groups);
            if (k > 0) {
                const int src = min(j + L.group, 63);
                const int r = __shfl(rr, src, 64), b = __shfl(rb, src, 64), e = __shfl(re, src, 64);
                float acc[CPL][E];
#pragma unroll
                for (int c = 0; c < CPL; ++c)
#pragma unroll
                    for (int x = 0; x < E; ++x) acc[c][x] = 0.0f;
                if (L.group < k) {
                    row_accumulate_group<VT, BT, E, CPL, U, false, HOLD>(P.rem_col, P.rem_val, b, e, a.B, a.ldb, a.b_rec,
                                                            ncol0, ncols, L, a.cold_aux, acc);
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        const int q = c * L.lpr + L.li;
                        if (q * E < ncols)
                            store_chunk<E>(a.C, (int64_t)r * a.ldc + ncol0 + chunk_col<E>(q, ncols), acc[c]);
                    }
                }
                j += k;
                continue;
            }
            // a long row: the whole wavefront, as in vector_item
            const int r = __shfl(rr, j, 64), b = __shfl(rb, j, 64), e = __shfl(re, j, 64);
            ++j;
            float acc[CPL][E];
#pragma unroll
            for (int c = 0; c < CPL; ++c)
#pragma unroll
                for (int x = 0; x < E; ++x) acc[c][x] = 0.0f;
            if (e - b <= P.seg_len) {
                seg_accumulate<VT, BT, E, CPL, U, false, HOLD>(P.rem_col, P.rem_val, b, e, a.B, a.ldb, a.b_rec, ncol0, ncols,
                                                  L, a.cold_aux, acc);
                group_reduce<E, CPL>(acc, L);
            } else {
                if constexpr (FUSED) continue;
                const int ns = (e - b + P.seg_len - 1) / P.seg_len;
                sum_partials<E, CPL>(a.work, a.work_ld, sid, ns, ncol0, ncols, L, acc);
                sid += ns;
            }
            store_row<E, CPL>(a.C, (int64_t)r * a.ldc, ncol0, ncols, L, acc);
        }
    }
}

// Size class of a row: the least power of two S of lane groups with
// len <= u2 * S, at most every group of the wavefront (grow: log2 of the step
// from one class to the next).
__device__ __forceinline__ int size_class(int len, int u2, int groups, int grow) {
    int s = 1;
    while (s < groups && len > u2 * s) s <<= grow;
    return s;
}

__device__ __forceinline__ uint64_t wave_or64(uint64_t x) {
    uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        lo |= __shfl_xor(lo, off, 64);
        hi |= __shfl_xor(hi, off, 64);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Vector work item with rows packed by size class: a row of class S is summed
// by an aligned block of S lane groups (entry p of the row by group p mod S,
// each group in entry order, then the groups' sums by an xor butterfly inside
// the block), so the order depends only on the row's length.  One pass takes
// consecutive rows while their classes do not grow and the blocks fit in the
// wavefront; with rows ordered longest first every block is aligned.  Split
// rows (class 1) sum their segment partials in segment order.
// UL: entries per group and step; size classes are counted in units of
// 2 unroll_of entries for any UL, and a class-S row's entry p goes to group
// p mod S in entry order whatever the step, so the result does not depend on UL.
template <int VT, int BT, int E, int CPL, bool FUSED = false, int UL = unroll_of<E, CPL>()>
__device__ __forceinline__ void vector_item_classed(const DevPlan &P, const RunArgs &a, int wid) {
    constexpr int U = UL;
    const int panel = wid / P.n_vitems, item = wid - panel * P.n_vitems;
    const int ncol0 = panel_col<E>(panel, a.np, P.n), ncols = min(a.np, P.n - ncol0);
    const Lanes L(a.lpr_log2);
    const int lane = threadIdx.x & 63;
    const __amdgpu_buffer_rsrc_t rs = b_resource(a.B, a.b_rec);
    bool cok[CPL];
    int64_t coff[CPL];
    chunk_layout<E, CPL>(ncol0, ncols, L, cok, coff);
    int sid = P.vitem_seg[item];
    const int i0 = P.vitem_ptr[item], i1 = P.vitem_ptr[item + 1];
    // f32 rows of more than 32 columns that are not whole chunks are of class 1
    // or all groups, which is the packed variant's order: at such widths the two
    // variants give the same bits (as when a lane took one column of them, and a
    // row of more than 32 all lanes).
    const int grow = BT == DT_F32 && E > 1 && P.n > 32 && P.n % E != 0 ? 6 - L.lpr_log2 : 1;
    // id, remainder range, class and segments of rows base .. base + 63, one
    // per lane, loaded again only when fewer rows than a full pass takes
    // (L.groups) remain loaded
    int base = i0 - 64;
    int wr = -1, wb = 0, we = 0, wcls = 1, wns = 0;
    for (int i = i0; i < i1;) {
        if (i - base + L.groups > 64) {
            base = i;
            const int l_row = i + lane;
            wr = -1; wb = 0; we = 0; wcls = 1; wns = 0;
            if (l_row < i1) {
                wr = P.vec_rows ? P.vec_rows[l_row] : l_row;
                wb = P.rem_ptr[wr];
                we = P.rem_ptr[wr + 1];
                if (we - wb > P.seg_len) {
                    wns = (we - wb + P.seg_len - 1) / P.seg_len;
                    we = wb;  // the entries were summed by the segment kernel
                } else {
                    wcls = size_class(we - wb, 2 * unroll_of<E, CPL>(), L.groups, grow);
                }
            }
        }
        // row i + lane, from the loaded rows (a lane past them ends the pass)
        const int j_row = i + lane, off = i - base;
        const bool have = lane + off < 64;
        const int srcl = min(lane + off, 63);
        int r = __shfl(wr, srcl, 64), b = __shfl(wb, srcl, 64), e = __shfl(we, srcl, 64);
        int cls = __shfl(wcls, srcl, 64), ns = __shfl(wns, srcl, 64);
        if (!have) {
            r = -1; b = 0; e = 0; cls = 1; ns = 0;
        }
        // the pass: rows before the first class increase whose blocks fit
        const int prev = __shfl_up(cls, 1, 64);
        const uint64_t cut = __ballot(j_row >= i1 || !have || (lane > 0 && cls > prev));
        const int kmax = cut ? __builtin_ctzll(cut) : 64;
        const int cin = lane < kmax ? cls : 0;
        const int incl = wave_inclusive_scan(cin);
        const uint64_t fits = __ballot(lane < kmax && incl <= L.groups);
        const int k = __popcll(fits);  // >= 1: row i always fits
        const int excl = incl - cin;
        // this lane group's row: the last block start at or below the group
        const uint64_t starts = wave_or64(lane < k ? (1ull << excl) : 0ull);
        const int g = L.group;
        const uint64_t upto = g >= 63 ? ~0ull : ((2ull << g) - 1ull);
        const int jr = (g < __shfl(incl, k - 1, 64)) ? __popcll(starts & upto) - 1 : -1;
        const int src = jr < 0 ? 0 : jr;
        int my_r = __shfl(r, src, 64), my_b = __shfl(b, src, 64), my_e = __shfl(e, src, 64);
        const int my_s = __shfl(cls, src, 64), my_ns = __shfl(ns, src, 64);
        const int local = g - __shfl(excl, src, 64);
        int my_sid = sid;
        if (__ballot(lane < k && ns > 0)) {
            const int nin = lane < k ? ns : 0;
            const int nincl = wave_inclusive_scan(nin);
            my_sid = sid + __shfl(nincl - nin, src, 64);
            sid += __shfl(nincl, k - 1, 64);
        }
        if (jr < 0) my_b = my_e = 0;
        const int smax = __builtin_amdgcn_readfirstlane(cls);  // the pass's largest class (lane 0)
        // the first group of a row's block stores it (fused: not a split row,
        // which its last segment stores)
        const bool writes = jr >= 0 && local == 0 && !(FUSED && my_ns > 0);

        float acc[CPL][E];
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int x = 0; x < E; ++x) acc[c][x] = 0.0f;
        // split rows (no entries left to gather) start from their segment sums
        if (!FUSED && jr >= 0 && my_ns > 0)
            sum_partials<E, CPL>(a.work, a.work_ld, my_sid, my_ns, ncol0, ncols, L, acc);
        Lanes Ls = L;
        Ls.groups = my_s;
        if constexpr (U < unroll_of<E, CPL>()) {
            accumulate<VT, BT, E, CPL, U, false, true>(P.rem_col, P.rem_val, my_b, my_e, a.B, a.ldb, a.b_rec, cok, coff, Ls,
                                          (g - local) * L.lpr, local, a.cold_aux, acc);
        } else {
            // (single runs, which hold 8 entries a step beside the pass's
            // layout, keep their own loads: 100,000 rows, N = 128 of f16 75 us,
            // held 78; 20,000 rows 25.2 / 26.8)
            for (int p = my_b + local; p < my_e; p += my_s * U) {
                int col[U];
                float v[U];
                load_entries<VT, U, BT != DT_F32>(P.rem_col, P.rem_val, p, my_e, Ls, col, v);
                gather_fma<BT, E, CPL, U>(col, v, p, my_e, a.B, rs, a.ldb, a.b_rec, cok, coff, Ls, a.cold_aux,
                                          acc);
            }
        }
        // butterfly inside each block, from the pass's largest class down
        for (int off = (smax * L.lpr) >> 1; off >= L.lpr; off >>= 1) {
            const bool take = off < my_s * L.lpr;
#pragma unroll
            for (int c = 0; c < CPL; ++c)
#pragma unroll
                for (int x = 0; x < E; ++x) {
                    const float t = __shfl_xor(acc[c][x], off, 64);
                    if (take) acc[c][x] += t;
                }
        }
        if (writes) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int q = c * L.lpr + L.li;
                if (q * E < ncols) store_chunk<E>(a.C, (int64_t)my_r * a.ldc + ncol0 + chunk_col<E>(q, ncols), acc[c]);
            }
        }
        i += k;
    }
}
// Waves per SIMD the kernels of vector items are compiled for, without which
// held entries cost one (f32 B 88 registers for 80: graph of 2^20 rows, N = 128,
// 925 us, bounded 891; more spills: 997 and up) or, in the batch's 16-bit
// kernel, two (64 uneven f16 matrices: 1086 us, bounded 1015).  Size classes
// hold entries in the batch's half steps only (UL < 8); full steps need 92 to 97
// registers, of which 5 waves have 96, and a bound of 80 spills 9 of them (f32,
// 200,000 rows, N = 128: 202 us, at 5 waves 184).
template <int BT, int CPL, int VAR, int UL, bool HOLD>
constexpr int vector_waves() {
    if (CPL != 1 || VAR < 2) return 1;
    if (VAR == 3 && UL >= 8) return 5;
    if (!HOLD) return 1;
    return BT == DT_F32 ? 6 : UL < 8 ? 5 : 1;
}

template <int VT, int BT, int E, int CPL, int VAR, bool FUSED, int UL, bool HOLD>
__device__ __forceinline__ void vector_item_var(const DevPlan &P, const RunArgs &a, int wid) {
    if constexpr (VAR == 3) vector_item_classed<VT, BT, E, CPL, FUSED, UL>(P, a, wid);
    else if constexpr (VAR == 2) vector_item_packed<VT, BT, E, CPL, FUSED, UL, HOLD>(P, a, wid);
    else if constexpr (VAR == 1) vector_item_pipelined<VT, BT, E, CPL, FUSED>(P, a, wid);
    else vector_item<VT, BT, E, CPL, FUSED>(P, a, wid);
}

template <int TT>
__device__ __forceinline__ f32x4 mfma_16x16x32(const u32x4 &a, const u32x4 &b, const f32x4 &c) {
    if constexpr (TT == DT_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Two f32 as bf16 (round to nearest even), the first in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// CW consecutive elements of a B row, as stored (DW dwords; a lone one in a
// pair, so that the type is a vector in every case).
template <int BT, int CW>
struct Chunk {
    static constexpr int BYTES = CW * (BT == DT_F32 ? 4 : 2), DW = (BYTES + 3) / 4;
    typedef uint32_t V __attribute__((ext_vector_type(DW < 2 ? 2 : DW)));
    V w;
    // at element alignment
    __device__ __forceinline__ void load(const void *p) {
        typedef V Ve __attribute__((aligned(2)));
        typedef uint32_t u32e __attribute__((aligned(2)));
        if constexpr (BYTES == 2) w[0] = *static_cast<const unsigned short *>(p);
        else if constexpr (BYTES == 4) w[0] = *static_cast<const u32e *>(p);
        else w = *static_cast<const Ve *>(p);
    }
    // through a buffer resource (an offset at its size or beyond gives zeros)
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
        if constexpr (BYTES == 2) w[0] = buf2<0>(rs, off);
        else if constexpr (BYTES == 4) w[0] = buf4<0>(rs, off);
        else if constexpr (BYTES == 8) w = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
        else w = buf16<0>(rs, off);
    }
    __device__ __forceinline__ float f32(int i) const {
        if constexpr (BT == DT_F32) return __uint_as_float(w[i]);
        else if constexpr (BT == DT_BF16)
            return __uint_as_float(i & 1 ? w[i >> 1] & 0xFFFF0000u : w[i >> 1] << 16);
        else return f16_to_f32(i & 1 ? w[i >> 1] >> 16 : w[i >> 1] & 0xFFFFu);
    }
};

// x of lane I of each 16-lane row (DPP row_newbcast), on all its lanes.
template <int I>
__device__ __forceinline__ int row16_broadcast(int x) {
    return __builtin_amdgcn_update_dpp(0, x, 0x150 + I, 0xf, 0xf, true);
}

// One wavefront's share of a window item: (window, panel of 16 CW columns) and
// MBW 16-row blocks of the window, MB in all (MB = 0: the plan's, MBW = 1);
// wid = item * (MB / MBW) + share, panel innermost, so a window's waves run
// side by side and share its tiles and B rows in L1 and L2.
// RG: rows of the block that each of the wave's 4 lane groups takes: all four of
// its MFMA results', or (1: four shares a block, one wave each) row 4g + share %
// 4 alone, 8 or 16 of whose remainder entries are in flight instead of 2 or 4.
// Every share of a block multiplies its tiles.  (A row's sum is the same: its
// entries are added one after the other.)
//
// A wave needs no LDS and no barrier: lane (g, c) = (lane / 16, lane % 16)
// loads CW consecutive elements of the B rows 8g .. 8g+7 of a tile, which is
// 16 CW columns of 32 rows for the wave.  MFMA operand i takes element i of
// each lane's chunk, i.e. the 16 columns {c CW + i}: the lane holds rows
// 8g .. 8g+7 of column c CW + i, as the operand wants it, after one v_perm per
// pair of rows (16-bit B) or one conversion of the pair (f32 B to bf16).  Its
// results are rows 4g .. 4g+3 of CW consecutive columns: C is written from
// the accumulators, and the lane group's rows are those whose remainder
// entries it gathers, in the same chunks.  The A operand (lane (g, c): row c,
// columns 8g .. 8g+7) is one aligned 16-byte load: the plan holds its tiles
// dense on the device (packed values behind a bitmap cost a misaligned load,
// 64 and more cache accesses where this one takes 16, and 64 instructions to
// spread them, per row block and tile).
//
// NBUF tiles' B rows and values are in flight while one is multiplied, and
// the tile columns NBUF tiles beyond those.  Loads sit behind no branch inside
// the loop (a branch makes the compiler wait for all of them): past the last
// tile they are of no column, which moves no data, and of a tile of zeros
// behind the plan's own.  A chunk at the end of a ragged panel starts at its last CW columns,
// and computes the columns it shares with its neighbour twice, from the same
// operands in the same order.
//
// FUSED: partial items and owners of windows with a slot (win_dep) store
// their parts in the workspace and arrive at the counter of (panel, slot,
// share); the last arrival combines these rows (window_combine).  Owners skip
// split rows, which the combine takes from the segments' partials.
// BUF: B is reached through a buffer resource (a.b_rec; else plain loads).
//
// Bound by B rows arriving from L2 and beyond (latency at small grids).  One
// workgroup per (window, panel of 128) with B in LDS, a barrier per 4 tiles
// and tile values expanded from the bitmap took (us, before / now): a 32,768-row attention mask
// (H = 64) at N = 256 of bf16 230 / 114 (1.0 GB of B rows, 0.57 PFLOP/s with
// the tiles' zeros), 16,384 rows at N = 64 of f32 89 / 48, 3,001 rows at
// N = 128 30 / 13; blocks of 262,144 rows (H = 16) at N = 256 of bf16 202 / 189.
//
// Waves per SIMD a kernel of window items is compiled for: 128 accumulators
// (in AGPRs) leave room for one, a single block fits three.
template <int MBW, int CW>
constexpr int window_waves() { return MBW * CW == 32 ? 1 : MBW == 1 ? 3 : 2; }

template <int VT, int BT, int TT, int MB, int MBW, int CW, bool BUF, int RG, bool FUSED = false>
__device__ __forceinline__ void window_item(const DevPlan &P, const RunArgs &a, int wid, bool partial) {
    static_assert(MB == 0 ? MBW == 1 : MB % MBW == 0, "a wave takes whole 16-row blocks");
    static_assert(RG == 4 || (RG == 1 && MB == 0), "rows of a lane group");
    constexpr int NBUF = 2;
    constexpr bool ACC = MBW * CW == 32;
    constexpr int NPW = 16 * CW, SB = BT == DT_F32 ? 4 : 2;
    constexpr bool PRE = MBW == 1;  // the rows' remainder ranges are loaded with the first tiles
    const int H = MB ? MB * 16 : P.H;
    const int subs_log2 = (MB ? (MB / MBW == 4 ? 2 : MB / MBW == 2 ? 1 : 0) : (H >> 5))  // H 16, 32, 64
                          + (RG == 1 ? 2 : 0);
    const int item = wid >> subs_log2, sub = wid & ((1 << subs_log2) - 1);
    const int j_item = item / a.win_panels, panel = item - j_item * a.win_panels;
    const int wi = partial ? P.wpart_win[j_item] : (P.win_order ? P.win_order[j_item] : j_item);
    const int ncol0 = panel_col<CW>(panel, NPW, P.n), ncols = min(NPW, P.n - ncol0);
    const int lane = threadIdx.x & 63, g = lane >> 4, l16 = lane & 15;
    const int t0 = partial ? P.wpart_t0[j_item] : P.win_tile_ptr[wi];
    const int t1 = partial ? P.wpart_t1[j_item] : min(P.win_tile_ptr[wi + 1], t0 + P.win_tmax);
    const int start = ncol0 + min(l16 * CW, ncols - CW);  // this lane's columns start .. start + CW - 1
    const bool own = l16 * CW < ncols;
    const int rb0 = (RG == 1 ? sub >> 2 : sub) * MBW;  // first block
    const int rq = RG == 1 ? sub & 3 : 0;              // first row of a lane group's (4g + rq ..)
    const __amdgpu_buffer_rsrc_t rs = b_resource(a.B, a.b_rec);
    const uint32_t ldbs = (uint32_t)(a.ldb * SB), sbyte = (uint32_t)(start * SB);
    const int64_t zoff = reinterpret_cast<const char *>(P.zeros) - static_cast<const char *>(a.B);

    // chunks of 8 B rows at this lane's columns; zeros where col < 0
    auto load_rows = [&](const int (&col)[8], Chunk<BT, CW> (&x)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (BUF) {
                x[i].load(rs, (uint32_t)col[i] * ldbs + sbyte);  // -1: wraps to beyond the resource
            } else {
                const int64_t off = ((int64_t)col[i] * a.ldb + start) * SB;
                x[i].load(static_cast<const char *>(a.B) + (col[i] >= 0 ? off : zoff));
            }
        }
    };

    typedef int i32x4 __attribute__((ext_vector_type(4)));
    // rows 16 (rb0 + mb) + 4g + rq .. + RG - 1 of the window: id and remainder range
    struct Rows {
        int r[RG], b[RG], e[RG];
    };
    auto row_ids = [&](int mb, Rows &R) {
        const int32_t *w = P.windows + (int64_t)wi * H + (rb0 + mb) * 16 + 4 * g + rq;
        if constexpr (RG == 4) {
            const i32x4 r = *reinterpret_cast<const i32x4 *>(w);
#pragma unroll
            for (int x = 0; x < 4; ++x) R.r[x] = r[x];
        } else {
            R.r[0] = *w;
        }
    };
    auto row_ranges = [&](Rows &R) {
#pragma unroll
        for (int x = 0; x < RG; ++x) {
            R.b[x] = P.rem_ptr[max(R.r[x], 0)];
            R.e[x] = P.rem_ptr[max(R.r[x], 0) + 1];
        }
    };
    auto split = [&](const Rows &R, int x) { return R.r[x] >= 0 && R.e[x] - R.b[x] > P.seg_len; };
    // end of the entries gathered here: none of a missing or a split row
    auto end = [&](const Rows &R, int x) { return R.r[x] < 0 || R.e[x] - R.b[x] > P.seg_len ? R.b[x] : R.e[x]; };
    // entries u .. u + 15 of each of the rows, one a lane of the row's group
    // (at clamped indices: the plan's arrays end in zeros)
    struct Entries {
        int col[RG];
        float v[RG];
    };
    auto entries = [&](const Rows &R, int u, Entries &q) {
#pragma unroll
        for (int x = 0; x < RG; ++x) {
            const int p = max(min(R.b[x] + u + l16, end(R, x) - 1), 0);
            q.col[x] = __builtin_nontemporal_load(P.rem_col + p) & 0x7FFFFFFF;
            q.v[x] = load_val<VT>(P.rem_val, p);
        }
    };
    // whether row x has an entry u, and its column (-1 without it) and value,
    // from lane u % 16 of the group
    auto has = [&](const Rows &R, int x, int u) { return R.b[x] + u < end(R, x); };
    auto from = [&](int v, int u) { return __builtin_amdgcn_ds_bpermute(((lane & 48) | (u & 15)) << 2, v); };
    // entries 0 .. PE - 1 of every row, in the place of a tile's 8 rows a lane group
    constexpr int PE = 8 / RG;
    auto first8 = [&](const int (&q)[RG], int (&c)[8]) {
        if constexpr (RG == 4) {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                c[2 * x] = row16_broadcast<0>(q[x]);
                c[2 * x + 1] = row16_broadcast<1>(q[x]);
            }
        } else {
            c[0] = row16_broadcast<0>(q[0]); c[1] = row16_broadcast<1>(q[0]);
            c[2] = row16_broadcast<2>(q[0]); c[3] = row16_broadcast<3>(q[0]);
            c[4] = row16_broadcast<4>(q[0]); c[5] = row16_broadcast<5>(q[0]);
            c[6] = row16_broadcast<6>(q[0]); c[7] = row16_broadcast<7>(q[0]);
        }
    };

    Rows R;
    Entries q0;
    bool some = false;  // any of the rows has an entry to gather

    struct Buf {
        Chunk<BT, CW> b[8];
        u32x4 a[MBW];
    };
    // tile column 8g + lane % 8 of tile t (of the last past the end)
    auto fetch = [&](int t) { return (P.tile_cols + (int64_t)min(t, t1 - 1) * 32)[8 * g + (lane & 7)]; };
    // (the scheduling barriers keep a buffer's loads behind the multiplication
    // that frees it: moved up, they take another buffer's registers)
    // (REM: past the last tile the remainder's rows instead)
    auto issue = [&](int t, int c, Buf &x, auto rem_tag) {
        constexpr bool REM = decltype(rem_tag)::value;
        __builtin_amdgcn_sched_barrier(0);
        if (!REM && t >= t1) c = -1;
        const uint16_t *v = P.tile_dense + ((int64_t)(t < t1 ? t : P.n_tiles) * H + rb0 * 16) * 32;
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) x.a[mb] = *reinterpret_cast<const u32x4 *>(v + (mb * 16 + l16) * 32 + 8 * g);
        int col[8] = {row16_broadcast<0>(c), row16_broadcast<1>(c), row16_broadcast<2>(c), row16_broadcast<3>(c),
                      row16_broadcast<4>(c), row16_broadcast<5>(c), row16_broadcast<6>(c), row16_broadcast<7>(c)};
        if constexpr (REM) {
            int rc[8];
            first8(q0.col, rc);
#pragma unroll
            for (int i = 0; i < 8; ++i) col[i] = t < t1 ? col[i] : some && has(R, i / PE, i % PE) ? rc[i] : -1;
        }
        load_rows(col, x.b);
        __builtin_amdgcn_sched_barrier(0);
    };

    f32x4 acc[MBW][CW];
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
        for (int i = 0; i < CW; ++i) acc[mb][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto multiply = [&](const Buf &x) {
#pragma unroll
        for (int i = 0; i < CW; ++i) {
            u32x4 bf;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const Chunk<BT, CW> &lo = x.b[2 * p], &hi = x.b[2 * p + 1];
                if constexpr (BT == DT_F32) bf[p] = pack_bf16(lo.f32(i), hi.f32(i));
                else bf[p] = __builtin_amdgcn_perm(hi.w[i >> 1], lo.w[i >> 1], i & 1 ? 0x07060302u : 0x05040100u);
            }
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb) {
                if constexpr (ACC) {
                    if constexpr (TT == DT_BF16)
                        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[mb][i]) : "v"(x.a[mb]), "v"(bf));
                    else
                        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc[mb][i]) : "v"(x.a[mb]), "v"(bf));
                } else {
                    acc[mb][i] = mfma_16x16x32<TT>(x.a[mb], bf, acc[mb][i]);
                }
            }
            if (i & 1) __builtin_amdgcn_sched_barrier(0);  // two operands at a time
        }
    };

    const std::false_type tiles;
    int m[NBUF];
    Buf x[NBUF];
    if (PRE && !partial) row_ids(0, R);
#pragma unroll
    for (int i = 0; i < NBUF; ++i) m[i] = fetch(t0 + i);
    if (PRE && !partial) row_ranges(R);
#pragma unroll
    for (int i = 0; i < NBUF; ++i) {
        issue(t0 + i, m[i], x[i], tiles);
        m[i] = fetch(t0 + NBUF + i);
    }
    if constexpr (PRE) {
        bool any = false;
#pragma unroll
        for (int x = 0; x < RG; ++x) any |= !partial && has(R, x, 0);
        some = __any(any);
        if (some) entries(R, 0, q0);
    }
    for (int t = t0; t < t1; t += NBUF) {
        // (the first buffer's last issue is not multiplied any more)
        multiply(x[0]);
        issue(t + NBUF, m[0], x[0], std::integral_constant<bool, PRE>{});
        m[0] = fetch(t + 2 * NBUF);
#pragma unroll
        for (int i = 1; i < NBUF; ++i) {
            multiply(x[i]);
            issue(t + NBUF + i, m[i], x[i], tiles);
            m[i] = fetch(t + 2 * NBUF + i);
        }
    }
    if constexpr (ACC) {
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
            for (int i = 0; i < CW; ++i) asm volatile("s_nop 15\n\ts_nop 7" : "+a"(acc[mb][i]));
    }

    const int64_t ld = a.work_ld;
    const __amdgpu_buffer_rsrc_t ws = ws_resource(a);
    const int dep = FUSED ? P.win_dep[wi] : -1;
    // CW columns of a workspace row that other workgroups of this launch read
    auto st_ws = [&](int64_t off, const float (&z)[CW]) {
#pragma unroll
        for (int c = 0; c < CW; c += CW >= 4 ? 4 : 1) {
            if constexpr (CW >= 4) st_dev_chunk<4>(ws, off + c, *reinterpret_cast<const float(*)[4]>(&z[c]));
            else st_dev1(ws, off + c, z[c]);
        }
    };
    // the MFMA result of row x of this lane group
    auto result = [&](int mb, int x, float (&z)[CW]) {
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const f32x4 &v = acc[mb][c];
            if constexpr (RG == 4) z[c] = v[x];
            else z[c] = rq == 0 ? v[0] : rq == 1 ? v[1] : rq == 2 ? v[2] : v[3];
        }
    };
    if (partial || dep >= 0) {
        // the MFMA result of these tiles: for the owner item (or the last
        // arrival) to add, or the owner's own, kept in the window's slot
        const int64_t dst = partial ? (int64_t)P.n_seg * ld + (int64_t)j_item * H * ld
                                    : (a.dep - a.work) + (int64_t)dep * 2 * H * ld;
        if (own) {
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
                for (int x = 0; x < RG; ++x) {
                    float z[CW];
                    result(mb, x, z);
                    const int64_t off = dst + (int64_t)((rb0 + mb) * 16 + 4 * g + rq + x) * ld + start;
                    if constexpr (FUSED) {
                        st_ws(off, z);
                    } else {
#pragma unroll
                        for (int c = 0; c < CW; ++c) a.work[off + c] = z[c];
                    }
                }
        }
        if (partial) {
            if constexpr (FUSED) {
                if (wave_arrive(win_counter(P, a, panel, dep, sub), win_target(P, a, wi, panel)))
                    window_combine<MBW == 1 ? 4 : 8>(P, a, wi, panel, dep, sub);
            }
            return;
        }
    }

#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
        float v[RG][CW];
#pragma unroll
        for (int x = 0; x < RG; ++x)
#pragma unroll
            for (int c = 0; c < CW; ++c) v[x][c] = 0.0f;
        int u = 0;
        if constexpr (PRE) {
            if (some) {
                int q[RG], val[8];
#pragma unroll
                for (int r = 0; r < RG; ++r) q[r] = __float_as_int(q0.v[r]);
                first8(q, val);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int r = i / PE;
                    if (has(R, r, i % PE)) {
#pragma unroll
                        for (int c = 0; c < CW; ++c)
                            v[r][c] = __builtin_fmaf(__int_as_float(val[i]), x[0].b[i].f32(c), v[r][c]);
                    }
                }
                u = PE;
            }
        } else {
            row_ids(mb, R);
            row_ranges(R);
        }
        auto more = [&] {
            bool any = false;
#pragma unroll
            for (int r = 0; r < RG; ++r) any |= has(R, r, u);
            return __any(any);
        };
        // the rest, RE entries of every row at a time, the next 16 entries in
        // flight with the last of these.  4 entries, 2 where their chunks would
        // spill: 64 registers of chunks for any width (16 entries at 32 columns)
        // cost 38,624 rows in blocks (2.2 entries a row), N = 32, 18.8 us for 8.1.
        constexpr int CH = MBW == 1 && CW == 8 && RG == 4 ? 8 : 16, RE = CH / RG;
        if (more()) {
            if (!PRE) entries(R, 0, q0);
            do {
                Chunk<BT, CW> rows[CH / 8][8];
                float val[CH];
                const int u0 = u;
#pragma unroll
                for (int i = 0; i < CH / 8; ++i) {
                    int col[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int r = (8 * i + k) / RE, w = u0 + (8 * i + k) % RE;
                        const int c = from(q0.col[r], w);
                        col[k] = has(R, r, w) && w < (u0 | 15) + 1 ? c : -1;
                        val[8 * i + k] = __int_as_float(from(__float_as_int(q0.v[r]), w));
                    }
                    load_rows(col, rows[i]);
                }
                const int u1 = min(u0 + RE, (u0 | 15) + 1);  // (not past the 16 entries held)
                u = u1;
                if ((u1 & 15) == 0) entries(R, u1, q0);
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const int r = i / RE, w = u0 + i % RE;
                    if (w < u1 && has(R, r, w)) {
#pragma unroll
                        for (int c = 0; c < CW; ++c)
                            v[r][c] = __builtin_fmaf(val[i], rows[i >> 3][i & 7].f32(c), v[r][c]);
                    }
                }
            } while (more());
        }
#pragma unroll
        for (int x = 0; x < RG; ++x) {
            const int s = (rb0 + mb) * 16 + 4 * g + rq + x;
            if (R.r[x] < 0 || !own) continue;
            if (dep >= 0) {
                // the row's remainder, for the combine (a split row's is
                // summed there from its segments' partials)
                if (!split(R, x)) st_ws((a.dep - a.work) + ((int64_t)dep * 2 + 1) * H * ld + (int64_t)s * ld + start, v[x]);
                continue;
            }
            float z[CW];
            result(mb, x, z);
            if constexpr (!FUSED) {
                // the window's other tiles' partial results, in tile order
                // (fused: a window with partial items has a slot)
                for (int k = P.win_part[wi]; k < P.win_part[wi + 1]; ++k) {
                    const float *w = a.work + ((int64_t)P.n_seg + (int64_t)k * H + s) * ld + start;
#pragma unroll
                    for (int c = 0; c < CW; ++c) z[c] += w[c];
                }
                if (split(R, x)) {  // its segments' partials, in segment order
                    const int sid = P.win_row_sid[(int64_t)wi * H + s];
                    const int ns = (R.e[x] - R.b[x] + P.seg_len - 1) / P.seg_len;
                    for (int k = 0; k < ns; ++k) {
                        const float *w = a.work + (int64_t)(sid + k) * ld + start;
#pragma unroll
                        for (int c = 0; c < CW; ++c) v[x][c] = k ? v[x][c] + w[c] : w[c];
                    }
                }
            }
            float *dst = a.C + (int64_t)R.r[x] * a.ldc + start;
#pragma unroll
            for (int c = 0; c < CW; ++c) z[c] = z[c] + v[x][c];
            if constexpr (CW >= 4) {
#pragma unroll
                for (int c = 0; c < CW; c += 4)
                    __builtin_nontemporal_store(f32x4e{z[c], z[c + 1], z[c + 2], z[c + 3]},
                                                reinterpret_cast<f32x4e *>(dst + c));
            } else {
#pragma unroll
                for (int c = 0; c < CW; ++c) __builtin_nontemporal_store(z[c], dst + c);
            }
        }
    }
    if constexpr (FUSED) {
        if (dep >= 0 && wave_arrive(win_counter(P, a, panel, dep, sub), win_target(P, a, wi, panel)))
            window_combine<MBW == 1 ? 4 : 8>(P, a, wi, panel, dep, sub);
    }
}
}  // namespace spmm
