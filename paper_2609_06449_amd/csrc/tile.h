// Device code of the direct form (direct.hip) and of the batched kernel
// (batch.hip): transforms whose data fit one workgroup, and the two column
// passes of the others.  FP32 arithmetic, the stages of stages.h.
//
// A tile is 2^LT transforms of n = 2^L points.  Every thread holds
// E = min(16, n) items of each of the H groups the tile's columns are dealt
// into (H = 2: column 2 t + h is column t of group h, so that one 16-byte
// access moves both; the groups take turns in an exchange buffer of one
// group).  Two orders of the butterflies over the threads:
//   column fastest (JF = false): neighbouring lanes own neighbouring columns
//     of a matrix, whose items are adjacent in HBM;
//   index fastest (JF = true): neighbouring lanes own neighbouring indices of
//     one transform, for transforms that lie contiguous in HBM.
// The result of an item does not depend on LT, H or JF: the same stages run on
// it in the same order, so the single and the batched kernels give the same
// bits with tiles of different widths.
//
// The two column passes of N = M1 M2 (x[j1 M2 + c], y[k1 + M1 k2]):
//   pass A: A[k1, c] = sum_j1 x[j1, c] w_M1^{-k1 j1}, stored blocked,
//           ws[((k1 >> lb) M2 + c) 2^lb + (k1 mod 2^lb)];
//   pass B: y[k1 + M1 k2] = sum_c (A[k1, c] w_N^{-k1 c}) w_M2^{-k2 c}
// with 2^lb the column count of a pass-B tile: pass B reads one contiguous
// piece of ws per tile, and pass A writes runs of 2^(lb + LT) items.
#pragma once

#include "stages.h"

namespace paco {
namespace {

// Stages S.. of a tile: v holds the operands of stage S (v[h E + i R + r]:
// operand r of butterfly g = tid + i NT of group h); store(t, j, u, R, LNS) is
// called once per butterfly of the last stage with its R outputs
// k = j + r 2^LNS at u[r] (group h: u[h E + r]).  The exchange buffer may be
// written from the call on; slower threads may still read it after the return.
// PREC: the radix-16 butterflies' arithmetic; the split MFMA forms use the
// exchange buffer as the waves' scratch (full waves only).
template <int L, int S, int LTG, int H, bool JF, int PREC = kPrecFP32, typename Store>
__device__ __forceinline__ void tile_stage(float2 (&v)[H * tile_items(L)], float2 *lds, const float2 *twl, int tid,
                                           const Store &store)
{
    constexpr int E = tile_items(L), LR = stage_log2radix(L, S), R = 1 << LR, LNS = stage_log2ns(L, S), NB = E / R;
    constexpr int NT = (1 << (L + LTG)) / E, LJ = L - LR;
    constexpr bool MF = PREC != kPrecFP32 && LR == 4;
    static_assert(!MF || (NT % 64 == 0 && NB == 1), "MFMA butterflies run on full waves");
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if constexpr (LNS > 0) {
            const int k = tile_idx<LTG, LJ, JF>(tid + i * NT) & ((1 << LNS) - 1);
            constexpr int LOW = stage_lo_width(L, S), HIW = stage_hi_width(L, S), OFF = stage_tw_offset(L, S);
            const float2 *tlo = twl + OFF + (k & (LOW - 1));
            const float2 *thi = twl + OFF + (R - 1) * LOW + (k >> 4);
#pragma unroll
            for (int r = 1; r < R; ++r) {
                float2 w = tlo[(r - 1) * LOW];
                if constexpr (HIW > 0) w = cmul(w, thi[(r - 1) * HIW]);
#pragma unroll
                for (int h = 0; h < H; ++h) v[h * E + i * R + r] = cmul(v[h * E + i * R + r], w);
            }
        }
        if constexpr (!MF) {
#pragma unroll
            for (int h = 0; h < H; ++h) dft_regs<LR>(&v[h * E + i * R]);
        }
    }
    if constexpr (MF) {
        if constexpr (S > 0) __syncthreads();  // every wave has read its operands out of the buffer
#pragma unroll
        for (int h = 0; h < H; ++h) mfma_dft16<PREC>(&v[h * E], lds + ((tid >> 6) << 10), tid & 63);
    }
    if constexpr (S + 1 < stage_count(L)) {
        constexpr int LR2 = stage_log2radix(L, S + 1), R2 = 1 << LR2, NB2 = E / R2, LNR2 = L - LR2;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            if (S > 0 || h > 0 || MF) __syncthreads();  // the previous contents were consumed
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int g = tid + i * NT;
                const int t = tile_col<LTG, LJ, JF>(g), j = tile_idx<LTG, LJ, JF>(g);
                const int d = stage_dest<LNS, LR>(j);
#pragma unroll
                for (int r = 0; r < R; ++r) lds[tile_slot<L, LTG, JF>(d + (r << LNS), t)] = v[h * E + i * R + r];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NB2; ++i) {
                const int g = tid + i * NT;
                const int t = tile_col<LTG, LNR2, JF>(g), j = tile_idx<LTG, LNR2, JF>(g);
#pragma unroll
                for (int r = 0; r < R2; ++r) v[h * E + i * R2 + r] = lds[tile_slot<L, LTG, JF>(j + (r << LNR2), t)];
            }
        }
        tile_stage<L, S + 1, LTG, H, JF, PREC>(v, lds, twl, tid, store);
    } else {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int g = tid + i * NT;
            store(tile_col<LTG, LJ, JF>(g), tile_idx<LTG, LJ, JF>(g), &v[i * R], std::integral_constant<int, R>(),
                  std::integral_constant<int, LNS>());
        }
    }
}

// First-stage operands: load(t, j, u, R, LJ) fills u[r] (and u[E + r] with
// H = 2) with row j + r 2^LJ of column t, r < R.
template <int L, int LTG, int H, bool JF, typename Load>
__device__ __forceinline__ void tile_load(float2 (&v)[H * tile_items(L)], int tid, const Load &load)
{
    constexpr int E = tile_items(L), LR = stage_log2radix(L, 0), R = 1 << LR, NB = E / R, LJ = L - LR;
    constexpr int NT = (1 << (L + LTG)) / E;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int g = tid + i * NT;
        load(tile_col<LTG, LJ, JF>(g), tile_idx<LTG, LJ, JF>(g), &v[i * R], std::integral_constant<int, R>(),
             std::integral_constant<int, LJ>());
    }
}

template <int N>
__device__ __forceinline__ void tile_conj(float2 (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) v[i].y = -v[i].y;
}

// ---- transforms of one workgroup ----------------------------------------------

// 2^LT transforms of 2^L points, transform t at item base(t) of src and dst
// (base(t) < 0: none).
template <int L, int LT, typename Base>
__device__ __forceinline__ void chip_tile(const float2 *src, float2 *dst, const Base &base, const float2 *stw,
                                          float2 *smem, int tid, bool conj_in, float oscale)
{
    float2 v[tile_items(L)];
    tile_load<L, LT, 1, true>(v, tid, [&](int t, int j, float2 *u, auto R, auto LJ) {
        const int64_t b = base(t);
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = b < 0 ? make_float2(0.f, 0.f) : src[b + j + (r << LJ)];
    });
    copy_twiddles(smem, stw, stage_tw_total(L), tid, tile_threads(L, LT, 1));
    if (conj_in) tile_conj(v);
    tile_stage<L, 0, LT, 1, true>(v, smem + tile_tw(L), smem, tid, [&](int t, int j, const float2 *u, auto R, auto LNS) {
        const int64_t b = base(t);
        if (b < 0) return;
        float2 *d = dst + b + j;
#pragma unroll
        for (int r = 0; r < R; ++r) d[r << LNS] = oscale != 0.f ? conj_scale(u[r], oscale) : u[r];
    });
}

// One transform of 2^14 points: the even and the odd items are the two groups
// of a 2^13-point tile, joined by a last radix-2 step with w_2^14^{-k} (hi, lo:
// its two-level table, split at 2^7).  Butterfly i of a thread's last stage
// (radix 2) has k = tid + 512 i and k + 4096: w^{-k} = w^{-tid} w_32^{-i}.
__device__ __forceinline__ void chip14_tile(const float2 *src, float2 *dst, const float2 *stw, const float2 *hi,
                                            const float2 *lo, float2 *smem, int tid, bool conj_in, float oscale)
{
    constexpr int L = 13, E = 16;
    float2 v[2 * E];
    tile_load<L, 0, 2, true>(v, tid, [&](int, int j, float2 *u, auto R, auto LJ) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float4 a = *reinterpret_cast<const float4 *>(src + 2 * (j + (r << LJ)));
            u[r] = make_float2(a.x, a.y);
            u[E + r] = make_float2(a.z, a.w);
        }
    });
    copy_twiddles(smem, stw, stage_tw_total(L), tid, 512);
    const float2 a = cmul(hi[tid >> 7], lo[tid & 127]);
    if (conj_in) tile_conj(v);
    tile_stage<L, 0, 0, 2, true>(v, smem + tile_tw(L), smem, tid, [&](int, int j, const float2 *u, auto R, auto LNS) {
        static_assert(R == 2 && LNS == 12, "the last stage of 2^13 points");
        const float2 w = cmul(a, hi[4 * (j >> 9)]);
        const float2 o0 = cmul(u[E], w), o1 = cmul(u[E + 1], w);
        float2 y[4] = {cadd(u[0], o0), cadd(u[1], make_float2(o1.y, -o1.x)),  // w^{-4096} = -i
                       csub(u[0], o0), csub(u[1], make_float2(o1.y, -o1.x))};
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[j + 4096 * q] = oscale != 0.f ? conj_scale(y[q], oscale) : y[q];
    });
}

// The same by 1024 threads, for one transform alone: the groups are two
// columns, and a thread's last-stage butterflies of column 1 are those of
// column 0 with the same j, so the radix-2 step stays in registers.  The same
// operations on every item as above.
__device__ __forceinline__ void chip14_wide_tile(const float2 *src, float2 *dst, const float2 *stw,
                                                 const float2 *__restrict__ hi, const float2 *__restrict__ lo,
                                                 float2 *smem, int tid, bool conj_in, float oscale)
{
    constexpr int L = 13;
    __builtin_assume(tid >= 0 && tid < 1024);
    float2 v[16];
    tile_load<L, 1, 1, true>(v, tid, [&](int t, int j, float2 *u, auto R, auto LJ) {
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = src[2 * (j + (r << LJ)) + t];
    });
    copy_twiddles(smem, stw, stage_tw_total(L), tid, 1024);
    if (conj_in) tile_conj(v);
    float2 even[8];
    tile_stage<L, 0, 1, 1, true>(v, smem + tile_tw(L), smem, tid, [&](int t, int j, const float2 *u, auto R, auto LNS) {
        static_assert(R == 2 && LNS == 12, "the last stage of 2^13 points");
        const int i = (j >> 10) & 3;  // j = tid + 1024 i
        if (t == 0) {
            even[2 * i] = u[0];
            even[2 * i + 1] = u[1];
            return;
        }
        const float2 w = cmul(cmul(hi[(j & 511) >> 7], lo[j & 127]), hi[4 * (j >> 9)]);
        const float2 o0 = cmul(u[0], w), o1 = cmul(u[1], w);
        const float2 y[4] = {cadd(even[2 * i], o0), cadd(even[2 * i + 1], make_float2(o1.y, -o1.x)),
                             csub(even[2 * i], o0), csub(even[2 * i + 1], make_float2(o1.y, -o1.x))};
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[j + 4096 * q] = oscale != 0.f ? conj_scale(y[q], oscale) : y[q];
    });
}

// ---- the two column passes -----------------------------------------------------

// Pass A: columns col0 .. of x (M1 = 2^L rows of M2 = 2^l2 items).  The wide
// tiles (H = 2) read x and write y with non-temporal accesses: both are used
// once, and the buffer between the passes then stays in the caches (batch of
// 4096 transforms 2^8..2^20 3.80 -> 3.63 ms, 128 of 2^20 812 -> 778 us, that
// is 5.5 TB/s over its two passes, a large copy's rate; pass A of 2^23, whose
// transform takes 72 us, another 7 to 10 us of that).
template <int L, int LT, int H, bool COH, int PREC = kPrecFP32>
__device__ __forceinline__ void pass_a_tile(const float2 *src, float2 *dst, int l2, int lb, uint32_t col0,
                                            const float2 *stw, float2 *smem, int tid, bool conj_in)
{
    constexpr int E = tile_items(L), LTG = LT - (H == 2 ? 1 : 0);
    float2 v[H * E];
    src += col0;
    tile_load<L, LTG, H, false>(v, tid, [&](int t, int j, float2 *u, auto R, auto LJ) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float2 *p = off32(src, addr::pass_a_load(uint32_t(j + (r << LJ)), uint32_t(t * H), l2));
            if constexpr (H == 2) {
                const float4 a = ld4_last(p);
                u[r] = make_float2(a.x, a.y);
                u[E + r] = make_float2(a.z, a.w);
            } else {
                u[r] = *p;
            }
        }
    });
    copy_twiddles(smem, stw, stage_tw_total(L), tid, tile_threads(L, LT, H));
    if (conj_in) tile_conj(v);
    tile_stage<L, 0, LTG, H, false, PREC>(v, smem + tile_tw(L), smem, tid, [&](int t, int j, const float2 *u, auto R, auto LNS) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t k = uint32_t(j + (r << LNS));
            const uint32_t at = addr::pass_a_store(k, col0 + uint32_t(t * H), l2, lb);
#pragma unroll
            for (int h = 0; h < H; ++h)
                st2<COH>(reinterpret_cast<char *>(off32(dst, at + (uint32_t(h) << lb))), u[h * E + r]);
        }
    });
}

// Pass B: columns v = col0 .. (k1), M2 = 2^L rows (c); 2^l1 columns in all.
// The top-level twiddle w_N^{-v c}, c = j + r 2^(L-4), is w_N^{-v j} (two-level
// table, one product per thread and column) times w_{16 M1}^{-v r} (cw),
// the latter for the tile's 2^LT columns through LDS (the exchange buffer's
// place, before the first exchange).
struct TopRoots {
    const float2 *hi, *lo, *cw;  // w_N^{-e} = hi[e >> log2Lo] lo[e mod 2^log2Lo]; cw[k] = w_{16 M1}^{-k}, k < 16 M1
    int log2N, log2Lo;
};
template <int L, int LT, int H, int PREC = kPrecFP32>
__device__ __forceinline__ void pass_b_tile(const float2 *src, float2 *dst, int l1, uint32_t col0, const TopRoots &T,
                                            const float2 *stw, float2 *smem, int tid, float oscale)
{
    static_assert(L >= 4, "the first stage is radix 16");
    constexpr int E = 16, LTG = LT - (H == 2 ? 1 : 0), NT = tile_threads(L, LT, H);
    float2 v[H * E];
    const float2 *s = src + (size_t(col0) << L);
    tile_load<L, LTG, H, false>(v, tid, [&](int t, int j, float2 *u, auto R, auto LJ) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float2 *p = off32(s, addr::pass_b_load(uint32_t(j + (r << LJ)), uint32_t(t * H), LT));
            if constexpr (H == 2) {
                const float4 a = ld4_last(p);
                u[r] = make_float2(a.x, a.y);
                u[E + r] = make_float2(a.z, a.w);
            } else {
                u[r] = ld2_last(p);
            }
        }
    });
    float2 *cwt = smem + tile_tw(L);  // [r][column]
    constexpr int CW = 16 << LT;
#pragma unroll
    for (int i = 0; i < (CW + NT - 1) / NT; ++i) {
        const int e = tid + i * NT;
        if (CW % NT == 0 || e < CW)
            cwt[e] = T.cw[addr::pass_b_cw(col0 + uint32_t(e & ((1 << LT) - 1)), uint32_t(e >> LT), l1)];
    }
    copy_twiddles(smem, stw, stage_tw_total(L), tid, NT);
    const int t0 = (tid & ((1 << LTG) - 1)) * H, j0 = tid >> LTG;
    const uint32_t lomask = (1u << T.log2Lo) - 1u;
    float2 a[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const uint32_t e = addr::pass_b_top(col0 + uint32_t(t0 + h), uint32_t(j0), T.log2N);
        a[h] = cmul(T.hi[e >> T.log2Lo], T.lo[e & lomask]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int h = 0; h < H; ++h) v[h * E + r] = cmul(v[h * E + r], cmul(a[h], cwt[(r << LT) + t0 + h]));
    __syncthreads();  // the factors are read: the exchange buffer is free
    dst += col0;
    tile_stage<L, 0, LTG, H, false, PREC>(v, cwt, smem, tid, [&](int t, int j, const float2 *u, auto R, auto LNS) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float2 *p = off32(dst, addr::pass_b_store(uint32_t(j + (r << LNS)), uint32_t(t * H), l1));
            const float2 y0 = oscale != 0.f ? conj_scale(u[r], oscale) : u[r];
            if constexpr (H == 2) {
                const float2 y1 = oscale != 0.f ? conj_scale(u[E + r], oscale) : u[E + r];
                __builtin_nontemporal_store(nt_f4{y0.x, y0.y, y1.x, y1.y}, reinterpret_cast<nt_f4 *>(p));
            } else {
                *p = y0;
            }
        }
    });
}

}  // namespace
}  // namespace paco
