// Row-per-lane helpers of the 16 x 16 tile routines (leaf.hip, trsm_stream.hip): multiply-adds whose
// second operand is a DPP row broadcast, and the inverse of a lower-triangular tile in registers.
#pragma once
#include "common.hpp"

namespace la {

constexpr int LT = 16;  // tile edge

// acc -= (value of src in lane K of the 16-lane row) * other, one instruction.  The hardware
// needs two wait states between a VALU write of src and this read of it; callers keep that.
template <int K>
__device__ __forceinline__ void fnmac_row(float &acc, float src, float other)
{
    asm volatile("v_fmac_f32_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                 : "+v"(acc)
                 : "v"(src), "v"(other), "n"(K));
}
template <int K>
__device__ __forceinline__ void fnmac_row(double &acc, double src, double other)
{
    asm volatile("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                 : "+v"(acc)
                 : "v"(src), "v"(other), "n"(K));
}
// acc -= (value of acc in lane K of the row) * other
template <int K>
__device__ __forceinline__ void fnmac_row_self(float &acc, float other)
{
    asm volatile("v_fmac_f32_dpp %0, -%0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(other), "n"(K));
}
template <int K>
__device__ __forceinline__ void fnmac_row_self(double &acc, double other)
{
    asm volatile("v_fmac_f64_dpp %0, -%0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(other), "n"(K));
}
// (value of src in lane K of the row) * other
template <int K>
__device__ __forceinline__ float mul_row(float src, float other)
{
    float d = 0.0f;
    asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                 : "+v"(d)
                 : "v"(src), "v"(other), "n"(K));
    return d;
}
template <int K>
__device__ __forceinline__ double mul_row(double src, double other)
{
    double d = 0.0;
    asm volatile("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                 : "+v"(d)
                 : "v"(src), "v"(other), "n"(K));
    return d;
}
// acc += (value of src in lane K of the row) * other
template <int K>
__device__ __forceinline__ void fmac_row(float &acc, float src, float other)
{
    asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                 : "+v"(acc)
                 : "v"(src), "v"(other), "n"(K));
}
template <int K>
__device__ __forceinline__ void fmac_row(double &acc, double src, double other)
{
    asm volatile("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                 : "+v"(acc)
                 : "v"(src), "v"(other), "n"(K));
}
// two wait states, with v routed through the statement so that whatever computes it stays before
template <typename T>
__device__ __forceinline__ void settle(T &v)
{
    asm volatile("s_nop 1" : "+v"(v));
}

// what one lane of the wavefront wrote to LDS is there for the others: the barrier alone keeps the lanes together but lets the compiler move
// accesses across it whose addresses it can tell apart
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float rcp_newton(float x) { return __builtin_amdgcn_rcpf(x); }
// seed good to 2^-24, one third-order step r (1 + e + e^2), e = 1 - x r: three dependent multiply-adds
__device__ __forceinline__ double rcp_newton(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// x = row r of the inverse of a 16 x 16 lower-triangular tile (a[c] = row r of the tile, dr its
// diagonal entry), columns shared out over the lane rows as in diag_factor_invert.  With
// m_rk = l_rk / l_kk the unit-triangular factor M = L diag(l)^-1 is inverted by
//   y_r. -= m_rk y_k.  (r > k),   k = 0, 1, ...   and   L^-1 = diag(l)^-1 M^-1.
template <typename T>
__device__ __forceinline__ void diag_invert(const T (&a)[LT], T dr, T (&x)[4], int r, int g)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        x[j] = (4 * j + g == r) ? T(1) : T(0);
        settle(x[j]);  // inside a loop the start values are copies made right here: keep them two wait states away
    }
    T rinv = rcp_newton(dr);
    settle(rinv);
    static_for<0, LT - 1>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        const T am = (r > k) ? a[k] : T(0);
        const T t = mul_row<k>(rinv, am);
        static_for<0, k / 4 + 1>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            fnmac_row_self<k>(x[j], t);
        });
    });
#pragma unroll
    for (int j = 0; j < 4; ++j)
        x[j] *= rinv;
}

// Factor and invert one 16 x 16 tile held one row per lane.  All four 16-lane rows of the
// wavefront factor copies of the same tile; the inverse is shared out between them: in lane row
// g register x[j] is column 4 j + g of the inverse.
// In: a[c] = A(r, c) for c <= r (what lies above the diagonal is never looked at).
// Out: a[c] = L(r, c) for c <= r, x[j] = L^-1(r, 4 j + g) (entries above the diagonal hold
// leftovers, respectively zero) and the return value is the 1-based index of the first pivot that
// is not > 0, or 0.
//
// The pivots run on the unscaled matrix,   a_rc -= a_rk a_ck / a_kk,   x_rc -= a_rk x_kc / a_kk,
// which needs only a reciprocal on the critical path (started as soon as the next pivot is final);
// the square roots are taken for all 16 pivots at once afterwards:
// L = A_raw diag(d)^-1/2,  L^-1 = diag(d)^-1/2 X_raw.
// SKIP: rows and columns from nk on are those of the identity; their pivots are left out, four at a time.
template <typename T, bool SKIP = false>
__device__ __forceinline__ int diag_factor_invert(T (&a)[LT], T (&x)[4], int r, int g, int nk = LT)
{
    T d = T(1);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        x[j] = (4 * j + g == r) ? T(1) : T(0);
    T rinv = rcp_newton(a[0]);  // meaningful in the pivot's lane only
    static_for<0, LT / 4>([&](auto bc) {
        constexpr int k0 = 4 * decltype(bc)::value;
        if constexpr (SKIP) {
            if (k0 >= nk)
                return;
            // a branch can leave copies of the operands right here: two wait states behind them
#pragma unroll
            for (int c = 0; c < LT; ++c)
                asm volatile("" : "+v"(a[c]));
#pragma unroll
            for (int j = 0; j < 4; ++j)
                asm volatile("" : "+v"(x[j]));
            asm volatile("s_nop 1");
        }
        static_for<k0, k0 + 4>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            const T am = (r > k) ? a[k] : T(0);
            d = (r == k) ? a[k] : d;
            settle(rinv);
            const T t = mul_row<k>(rinv, am);  // a_rk / a_kk below the pivot, zero elsewhere
            if constexpr (k + 1 < LT) {
                fnmac_row<k + 1>(a[k + 1], a[k], t);
                rinv = rcp_newton(a[k + 1]);  // overlaps the rest of this pivot's updates
            }
            static_for<k + 2, LT>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                fnmac_row<c>(a[c], a[k], t);  // a_rc -= a_ck t_r
            });
            static_for<0, k / 4 + 1>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                fnmac_row_self<k>(x[j], t);  // x_rc -= x_kc t_r (a no-op where column c > k)
        });
    });
    });
    const unsigned long long bad = __ballot(!(d > T(0)));
    T rs = rsqrt_acc(d);
    settle(rs);
    static_for<0, LT>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        a[c] = mul_row<c>(rs, a[c]);  // column c times d_c^-1/2
    });
#pragma unroll
    for (int j = 0; j < 4; ++j)
        x[j] *= rs;  // row r times d_r^-1/2
    const unsigned first = (unsigned)(bad & 0xffffu);
    return first ? __builtin_ctz(first) + 1 : 0;
}

// acc += (value of acc in lane K of the row) * other
template <int K>
__device__ __forceinline__ void fmac_row_self(float &acc, float other)
{
    asm volatile("v_fmac_f32_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(other), "n"(K));
}
template <int K>
__device__ __forceinline__ void fmac_row_self(double &acc, double other)
{
    asm volatile("v_fmac_f64_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(other), "n"(K));
}

// ---------------------------------------------------------------------------------------
// Factor and invert one 16 x 16 tile that a wavefront holds as a matrix-core accumulator.
//
// A single wavefront issues one instruction per 6 to 9 cycles whatever it is, so the chain of pivots is bound by their number.
// The symmetric tile S is therefore shared out over the four lane groups: register v of group g (g = lane / 16) is column
// 4 v + g, lane = row, which is the accumulator layout of the matrix cores.  A rank-1 update of the whole tile is then four multiply-adds
// at most, whose second factor a_kc is the tile's own row k, a row broadcast of the register that is updated (S is symmetric,
// so both triangles are kept up).  Only the first factor, column k, has to be known to all groups: four columns at a time go through
// LDS, and the pivots of those four run on the copies.
//
// Rows and columns are numbered by chain_nat: the row of the tile that lane position l (of 16) stands for.  In fp64 it is l
// itself; the fp32 accumulator holds rows 4 g + v instead of g + 4 v, so there the positions are relabelled,
// which turns one layout into the other (the map is its own inverse).
// ---------------------------------------------------------------------------------------
template <typename T>
__host__ __device__ constexpr int chain_nat(int l)
{
    return sizeof(T) == 8 ? l : 4 * (l % 4) + l / 4;
}

// The inverse of a tile with a pivot that is not > 0, once more for the rows before it.  A zero or NaN there has reached their x as
// 0 * inf or 0 * NaN, and the columns of the factor before that pivot are still asked for.  Out of line of the chain of pivots: only such a tile
// comes here (the question after the last pivot: potrf of 32 x 128^2 12.5 -> 12.6 us in fp32, 16.5 -> 16.4 in fp64).
// row = row r of the tile in LDS, its columns before `first` final and divided by anything that is the same down a
// column; p = element r of that row; x as elsewhere, scaled so that its diagonal is one.  at(k) = the lane (of 16) that has row k.
template <typename T, typename F>
__device__ __forceinline__ void inverse_before(const T *row, T p, T (&x)[4], int r, int g, int first, F &&at)
{
    T y[4];
#pragma unroll
    for (int v = 0; v < 4; ++v)
        y[v] = (4 * v + g == r) ? T(1) : T(0);
    for (int k = 0; k + 1 < first; ++k) {
        const T pk = __shfl(p, at(k), WAVE);
        const T t = (k < r && r < first) ? row[k] / pk : T(0);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            y[v] = fma(-t, __shfl(y[v], 16 * g + at(k), WAVE), y[v]);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
        x[v] = r < first ? y[v] : x[v];
}
// the first of the rows whose lanes (of 16) are set in `bad`, LT if none
template <typename T>
__device__ __forceinline__ int first_row(unsigned bad)
{
    int f = LT;
    for (int q = LT - 1; q >= 0; --q)
        f = (bad >> chain_nat<T>(q)) & 1 ? q : f;
    return f;
}

// t where keep, otherwise zero or (fp64, whose lower half is left alone) a number below the normal range: as good as zero
// beside multipliers of order one, for one instruction
__device__ __forceinline__ float keep_if(float t, bool keep) { return keep ? t : 0.0f; }
__device__ __forceinline__ double keep_if(double t, bool keep)
{
    uint2 w = __builtin_bit_cast(uint2, t);
    w.y = keep ? w.y : 0u;
    return __builtin_bit_cast(double, w);
}

// In: S as above, both triangles.  r = chain_nat(lane % 16), g = lane / 16; row = row r of a tile in LDS (16-byte aligned, the
// rows of different lanes apart).
// Out: the tile's row r holds the columns of the factor times the square roots of their pivots (what lies above the diagonal is
// left over), d = pivot r, X[v] = element (r, 4 v + g) of the inverse of the factor times the square root of pivot r (zero or as good
// as zero above the diagonal).  Returns the lanes of lane group 0 whose pivot is not > 0; the rows before the first of those are right.
//
// The pivots run on the unscaled matrix,   a_rc -= t_r a_kc,   x_rc -= t_r x_kc (r > k),   t_r = a_rk / a_kk.
template <typename T>
__device__ __forceinline__ unsigned chain_diag(T (&S)[4], T *row, T &d, T (&X)[4], int r, int g)
{
    using V = typename Mfma<T>::vec_t;
    constexpr int VW = Mfma<T>::VW;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        X[v] = (4 * v + g == r) ? T(1) : T(0);
        asm volatile("" : "+v"(S[v]), "+v"(X[v]));  // their own registers from here on: no copies next to the broadcasts below
    }
    asm volatile("s_nop 1");
    static_for<0, 4>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        T c[4];
        row[4 * p + g] = S[p];
        wave_sync();
#pragma unroll
        for (int h = 0; h < 4; h += VW) {
            const V w = *reinterpret_cast<const V *>(row + 4 * p + h);
            c[h] = w.x;
            c[h + 1] = w.y;
            if constexpr (VW == 4) {
                c[2] = w.z;
                c[3] = w.w;
            }
        }
        wave_sync();
        T rinv = rcp_newton(c[0]);  // meaningful in the pivot's lane only
        static_for<0, 4>([&](auto qc) {
            constexpr int q = decltype(qc)::value, k = 4 * p + q, K = chain_nat<T>(k);
            T nt = T(0);  // -t
            settle(rinv);
            fnmac_row<K>(nt, rinv, c[q]);
            if constexpr (q < 3) {
                fmac_row<chain_nat<T>(k + 1)>(c[q + 1], c[q], nt);
                rinv = rcp_newton(c[q + 1]);  // overlaps the rest of this pivot's updates
            }
            if constexpr (q < 2)
                fmac_row<chain_nat<T>(k + 2)>(c[q + 2], c[q], nt);
            if constexpr (q < 1)
                fmac_row<chain_nat<T>(k + 3)>(c[q + 3], c[q], nt);
            static_for<p + 1, 4>([&](auto vc) { fmac_row_self<K>(S[decltype(vc)::value], nt); });
            if constexpr (k + 1 < LT) {
                const T tm = keep_if(nt, r > k);
                static_for<0, p + 1>([&](auto vc) { fmac_row_self<K>(X[decltype(vc)::value], tm); });
            }
        });
#pragma unroll
        for (int h = 0; h < 4; h += VW) {
            V w;
            w.x = c[h];
            w.y = c[h + 1];
            if constexpr (VW == 4) {
                w.z = c[2];
                w.w = c[3];
            }
            *reinterpret_cast<V *>(row + 4 * p + h) = w;
        }
    });
    wave_sync();
    d = row[r];
    const unsigned bad = (unsigned)(__ballot(!(d > T(0))) & 0xffffu);
    if (__builtin_expect(bad != 0, 0))
        inverse_before<T>(row, d, X, r, g, first_row<T>(bad), chain_nat<T>);
    return bad;
}

}  // namespace la
