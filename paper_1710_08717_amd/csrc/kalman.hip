// Kalman filter over a batch of sequences (section 3.4, "Kalman Filtering"): every matrix of
// the recursion is at most 16 x 16, so one sequence lives in D = 16 lanes for its whole length --
// lane r holds row r of each matrix in registers (zero padded to D columns), vectors have one
// element per lane -- and a wavefront carries four sequences; with all dimensions <= 4 the same
// code runs with D = 4 and sixteen sequences per wavefront.  Nothing but the observation v_t
// is read and nothing but f_t, F_t is written per step.
//
// With rows in lanes, both product shapes of the recursion are chains of one instruction, a
// multiply-add whose second factor is broadcast from one lane of the group (DPP row_newbcast for
// 16 lanes, DPP quad_perm for 4):
//   C = X Y    C[r][j] += X[r][k] * (Y[k][j]: register j of lane k)
//   C = X Y^T  C[r][j] += X[r][k] * (Y[j][k]: register k of lane j)
// and the right-side triangular solves of the gain matrix work on rows, i.e. inside a lane.
// The parameters (A, B, S_h, S_v) wait in LDS and a lane fetches its row before each use.
//
// That is k_kalman.  Where one model is filtered over all sequences, the covariance recursion --
// F_t, the gain, the factor of S_vv -- does not depend on the observations and is the same for
// every sequence: k_kalman_shared runs it once per workgroup and only the means and the
// likelihood per sequence.  (In fp32 with dimensions up to 4 that saves little; there k_kalman
// takes one model as well, for the batches where it is the faster one.)
#include "common.hpp"
#include "leaf_dpp.hpp"

namespace la {

template <typename T, int D>  // D: lanes per sequence = padded dimension (16, 8 or 4)
struct KfLds {
    static constexpr int GROUPS = 64 / D;                // sequences per workgroup (one wavefront)
    static constexpr int PS = D + 16 / (int)sizeof(T);   // row stride: 16-byte row reads of 16 lanes hit all banks
    static constexpr int MAT = D * PS;
    static constexpr int GROUP = 4 * MAT;  // A, B, S_h, S_v
    static constexpr size_t BYTES = (size_t)GROUPS * GROUP * sizeof(T);
};

// acc <- acc +- other * (src of lane K of the D-lane group)
template <int K>
__device__ __forceinline__ void fmac_quad(float &acc, float src, float other, bool neg)
{
    if (neg)
        asm volatile("v_fmac_f32_dpp %0, -%1, %2 quad_perm:[%3,%3,%3,%3] row_mask:0xf bank_mask:0xf"
                     : "+v"(acc)
                     : "v"(src), "v"(other), "n"(K));
    else
        asm volatile("v_fmac_f32_dpp %0, %1, %2 quad_perm:[%3,%3,%3,%3] row_mask:0xf bank_mask:0xf"
                     : "+v"(acc)
                     : "v"(src), "v"(other), "n"(K));
}
template <int K>
__device__ __forceinline__ void fmac_quad(double &acc, double src, double other, bool neg)
{
    // 64-bit DPP has no quad_perm: two 32-bit lane moves, then a plain multiply-add
    constexpr int ctrl = K | (K << 2) | (K << 4) | (K << 6);
    const long long v = __builtin_bit_cast(long long, src);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(v & 0xffffffffll), ctrl, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), ctrl, 0xf, 0xf, false);
    const double b = __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
    acc = fma(neg ? -other : other, b, acc);
}
template <int D, int K, typename T>
__device__ __forceinline__ void kf_fma(T &acc, T src, T other, bool neg)
{
    if constexpr (D == 16 || D == 8)  // D == 8: two sequences per 16-lane row, the instruction once per half
        fma_bcast<D, K>(acc, src, other, neg);
    else
        fmac_quad<K>(acc, src, other, neg);
}
// two wait states between a vector write of a register and a DPP read of it inside inline asm
template <typename T, int N>
__device__ __forceinline__ void kf_settle(T (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i)
        asm volatile("" : "+v"(v[i]));
    asm volatile("s_nop 1");
}
template <typename T>
__device__ __forceinline__ void kf_settle1(T &v)
{
    asm volatile("s_nop 1" : "+v"(v));
}

template <typename T>
struct KfArgs {
    const T *A, *B, *Sh, *Sv, *mu0, *S0, *v;
    T *f, *F, *nll;
    int32_t *info;
    int64_t batch;
    int T_, dh, dv, shared;  // shared: one model for all sequences
};

// f(k) for k = 0 .. D-1 in ascending (or descending) order, in blocks of four; a block is skipped
// when all of it lies at or beyond `dim`.  (One uniform branch per block: a branch per index
// costs more scalar registers than there are.)  Indices between dim and the end of its block
// see the zero / identity padding.
template <int D, class Fn>
__device__ __forceinline__ void kf_upto(int dim, Fn &&fn)
{
    static_for<0, D / 4>([&](auto bc) {
        constexpr int b0 = 4 * decltype(bc)::value;
        if (b0 < dim) {
            static_for<0, 4>([&](auto ic) { fn(std::integral_constant<int, b0 + decltype(ic)::value>{}); });
        }
    });
}
template <int D, class Fn>
__device__ __forceinline__ void kf_downfrom(int dim, Fn &&fn)
{
    static_for<0, D / 4>([&](auto bc) {
        constexpr int b0 = D - 4 - 4 * decltype(bc)::value;
        if (b0 < dim) {
            static_for<0, 4>([&](auto ic) { fn(std::integral_constant<int, b0 + 3 - decltype(ic)::value>{}); });
        }
    });
}

// C[r][j] += sum_{k < kdim} X[r][k] Y[k][j]   (neg: subtract)
template <typename T, int D>
__device__ __forceinline__ void kf_nn(T (&C)[D], const T (&X)[D], T (&Y)[D], int kdim, bool neg = false)
{
    kf_settle(Y);
    kf_upto<D>(kdim, [&](auto kc) {
        constexpr int k = decltype(kc)::value;
        static_for<0, D>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            kf_fma<D, k>(C[j], Y[j], X[k], neg);
        });
    });
}

// C[r][j] += sum_k X[r][k] Y[j][k] for j < jdim
template <typename T, int D>
__device__ __forceinline__ void kf_nt(T (&C)[D], const T (&X)[D], T (&Y)[D], int jdim)
{
    kf_settle(Y);
    static_for<0, D / 4>([&](auto bc) {  // four columns at a time: their chains of multiply-adds interleave
        constexpr int b0 = 4 * decltype(bc)::value;
        if (b0 < jdim) {
            static_for<0, D>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                static_for<0, 4>([&](auto ic) {
                    constexpr int j = b0 + decltype(ic)::value;
                    kf_fma<D, j>(C[j], Y[k], X[k], false);
                });
            });
        }
    });
}

// c[r] += sum_{k < kdim} X[r][k] y[k]
template <typename T, int D>
__device__ __forceinline__ void kf_mv(T &c, const T (&X)[D], T &y, int kdim)
{
    kf_settle1(y);
    kf_upto<D>(kdim, [&](auto kc) {
        constexpr int k = decltype(kc)::value;
        kf_fma<D, k>(c, y, X[k], false);
    });
}

template <typename T, int D>
__device__ __forceinline__ void kf_zero(T (&x)[D])
{
#pragma unroll
    for (int j = 0; j < D; ++j)
        x[j] = T(0);
}

template <typename T, int D>
__device__ __forceinline__ void kf_row(T (&x)[D], const T *row)
{
#pragma unroll
    for (int j = 0; j < D; ++j)
        x[j] = row[j];
}

template <typename T, int D>
__global__ __launch_bounds__(64) void k_kalman(KfArgs<T> a)
{
    using Lds = KfLds<T, D>;
    constexpr int KF_D = D, KF_GROUPS = Lds::GROUPS;
    extern __shared__ __align__(16) unsigned char kf_smem[];
    const int lane = threadIdx.x, g = lane / D, r = lane % D;
    const int dh = a.dh, dv = a.dv, steps = a.T_;
    const int64_t b_raw = (int64_t)blockIdx.x * KF_GROUPS + g;
    const bool live = b_raw < a.batch;
    const int64_t b = live ? b_raw : a.batch - 1;  // a spare group repeats the last sequence and stores nothing
    const int64_t pb = a.shared ? 0 : b;

    // one copy of the parameters per sequence, or one for the workgroup
    T *sA = reinterpret_cast<T *>(kf_smem) + (a.shared ? 0 : g * Lds::GROUP), *sB = sA + Lds::MAT, *sSh = sB + Lds::MAT,
      *sSv = sSh + Lds::MAT;
    if (!a.shared || g == 0) {   // zero padded (S_v: identity padded, so that the padded S_vv keeps a unit pivot)
        const T *Ap = a.A + pb * dh * dh, *Bp = a.B + pb * dv * dh, *Shp = a.Sh + pb * dh * dh, *Svp = a.Sv + pb * dv * dv;
#pragma unroll
        for (int j = 0; j < KF_D; ++j) {
            sA[r * Lds::PS + j] = (r < dh && j < dh) ? Ap[r * dh + j] : T(0);
            sB[r * Lds::PS + j] = (r < dv && j < dh) ? Bp[r * dh + j] : T(0);
            sSh[r * Lds::PS + j] = (r < dh && j < dh) ? Shp[r * dh + j] : T(0);
            sSv[r * Lds::PS + j] = (r < dv && j < dv) ? Svp[r * dv + j] : (r == j ? T(1) : T(0));
        }
    }
    __syncthreads();

    T F[KF_D];  // filtered covariance, row r
    T f = (r < dh) ? a.mu0[pb * dh + r] : T(0);
#pragma unroll
    for (int j = 0; j < KF_D; ++j)
        F[j] = (r < dh && j < dh) ? a.S0[pb * dh * dh + r * dh + j] : T(0);

    const T *vp = a.v + b * (int64_t)steps * dv;
    T vnext = (steps > 0 && r < dv) ? vp[r] : T(0);
    double nll_acc = 0.0;
    int32_t bad = 0;
    const T one = T(1);

    for (int t = 0; t < steps; ++t) {
        const T vt = vnext;
        if (t + 1 < steps && r < dv)
            vnext = vp[(int64_t)(t + 1) * dv + r];

        // ---- predicted state: mu_h, S_hh (the prior at t = 0) ----
        T Shh[KF_D];
        T muh;
        if (t == 0) {
            muh = f;
#pragma unroll
            for (int j = 0; j < KF_D; ++j)
                Shh[j] = F[j];
        } else {
            T Ar[KF_D], T1[KF_D];
            kf_row(Ar, sA + r * Lds::PS);
            muh = T(0);
            kf_mv(muh, Ar, f, dh);           // A f
            kf_zero(T1);
            kf_nt(T1, F, Ar, dh);            // F A^T
            kf_row(Shh, sSh + r * Lds::PS);
            kf_nn(Shh, Ar, T1, dh);          // S_h + A (F A^T)
        }

        // ---- predicted observation: mu_v, M = S_hh B^T, S_vv = B M + S_v ----
        T M[KF_D], S[KF_D];
        T muv = T(0);
        {
            T Br[KF_D];
            kf_row(Br, sB + r * Lds::PS);
            kf_mv(muv, Br, muh, dh);
            kf_zero(M);
            kf_nt(M, Shh, Br, dv);
            kf_row(S, sSv + r * Lds::PS);
            kf_nn(S, Br, M, dh);
        }

        // ---- S_vv = L L^T in place (lower triangle of S; lane r keeps 1 / L_rr) ----
        T invd = one;
        kf_upto<D>(dv, [&](auto kc) {
            constexpr int k = decltype(kc)::value;
            kf_settle1(S[k]);
            T d = T(0);
            kf_fma<D, k>(d, S[k], one, false);  // pivot, from lane k
            if (!(d > T(0)) && bad == 0)
                bad = t + 1;
            const T rs = one / sqrt(d);
            S[k] *= rs;
            if (r == k)
                invd = rs;
            kf_settle1(S[k]);
            static_for<k + 1, KF_D>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                kf_fma<D, j>(S[j], S[k], S[k], true);  // S[r][j] -= L[r][k] L[j][k]
            });
        });
#pragma unroll
        for (int j = 0; j < KF_D; ++j)
            S[j] = (j > r) ? T(0) : S[j];

        // ---- gain K = M L^-T L^-1, row by row inside each lane ----
        kf_settle(S);
        kf_settle1(invd);
        kf_upto<D>(dv, [&](auto jc) {  // X L^T = M
            constexpr int j = decltype(jc)::value;
            T x = T(0);
            kf_fma<D, j>(x, invd, M[j], false);
            M[j] = x;
            static_for<j + 1, KF_D>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                kf_fma<D, i>(M[i], S[j], x, true);  // M[r][i] -= x L[i][j]
            });
        });
        kf_downfrom<D>(dv, [&](auto jc) {  // K L = X
            constexpr int j = decltype(jc)::value;
            T y = T(0);
            kf_fma<D, j>(y, invd, M[j], false);
            M[j] = y;
            static_for<0, j>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                kf_fma<D, j>(M[i], S[i], y, true);  // M[r][i] -= y L[j][i]
            });
        });
        // M now holds K

        // ---- innovation, its likelihood term, filtered mean ----
        T delta = (r < dv) ? vt - muv : T(0);
        T fn = muh;
        kf_mv(fn, M, delta, dv);  // mu_h + K delta
        {
            T dl = delta, zfin = T(0);
            kf_upto<D>(dv, [&](auto kc) {  // z = L^-1 delta, one element per lane
                constexpr int k = decltype(kc)::value;
                T zs = dl * invd;
                if (r == k)
                    zfin = zs;
                kf_settle1(zs);
                kf_fma<D, k>(dl, zs, S[k], true);  // dl[r] -= L[r][k] z[k]
            });
            if (r < dv)
                nll_acc += 0.5 * (double)zfin * (double)zfin - (double)log(invd);
        }
        f = fn;

        // ---- filtered covariance F = (I - K B) S_hh (I - K B)^T + K S_v K^T ----
        T G[KF_D];
        {
            T Br[KF_D];
            kf_row(Br, sB + r * Lds::PS);
#pragma unroll
            for (int j = 0; j < KF_D; ++j)
                G[j] = (j == r) ? one : T(0);
            kf_nn(G, M, Br, dv, true);  // I - K B
        }
        {
            T T2[KF_D];
            kf_zero(T2);
            kf_nt(T2, Shh, G, dh);      // S_hh (I - K B)^T
            kf_zero(F);
            kf_nn(F, G, T2, dh);
        }
        {
            T Svr[KF_D], T3[KF_D];
            kf_row(Svr, sSv + r * Lds::PS);
            kf_zero(T3);
            kf_nt(T3, Svr, M, dh);      // S_v K^T
            kf_nn(F, M, T3, dv);        // + K (S_v K^T)
        }

        if (live && r < dh) {
            if (a.f)
                a.f[(b * steps + t) * dh + r] = f;
            if (a.F) {
                T *Fo = a.F + ((b * steps + t) * dh + r) * dh;
#pragma unroll
                for (int j = 0; j < KF_D; ++j)
                    if (j < dh)
                        Fo[j] = F[j];
            }
        }
    }

    // sum of the per-lane likelihood terms over the group, plus the constant
#pragma unroll
    for (int off = D / 2; off >= 1; off >>= 1)
        nll_acc += __shfl_xor(nll_acc, off, D);
    if (live && r == 0) {
        a.nll[b] = (T)(nll_acc + 0.5 * steps * dv * 1.8378770664093454835606594728112);  // log(2 pi)
        if (a.info)
            a.info[b] = bad;
    }
}

template <typename T, int D>
static la_status launch_kalman_d(const KfArgs<T> &a, hipStream_t st)
{
    using Lds = KfLds<T, D>;
    const int64_t blocks = (a.batch + Lds::GROUPS - 1) / Lds::GROUPS;
    if (blocks > 0x7fffffffll)
        return LA_ERR_UNSUPPORTED;
    const size_t lds = a.shared ? Lds::BYTES / Lds::GROUPS : Lds::BYTES;
    LA_LAUNCH((k_kalman<T, D>), dim3((unsigned)blocks), dim3(64), lds, st, a);
    return launch_check("kalman");
}

// ---------------------------------------------------------------------------------------
// One model for all sequences.  Wavefront 0 of a workgroup walks the covariance recursion; every
// other wavefront carries up to 64 sequences, one step behind it, with the matrices of the step
// from LDS (two buffers, one barrier per step), and writes the common F_t to their places, whole
// items per store instruction.
//
// Everything but the factorisation of S_vv is 16 x 16 x 16 products on the matrix cores, zero
// padded.  RL(X): lane l holds X[l % 16][k(l, s)], s = 0..3; CL(X): X[k(l, s)][l % 16], with k(l, s)
// the accumulator's row map, the contraction index being dealt to the lanes in the same way.  A
// product takes RL(X), CL(Y) and gives CL(X Y), and RL(X) = CL(X^T), so nearly every result
// feeds the next product as it is:
//   CL(F^T A^T) = CL(F) . RL(A)                       RL(S_hh) = RL(A) . CL(F^T A^T) + CL(S_h^T)
//   CL(M) = RL(S_hh) . RL(B),  M = S_hh B^T           CL(M^T) = RL(B) . RL(S_hh)
//   CL(S_vv) = RL(B) . CL(M) + CL(S_v)                S_vv = L L^T, L^-1: registers, by way of LDS
//   CL(X) = RL(L^-1) . CL(M^T)                        RL(K) = CL(L^-1) . CL(X),  K = X^T L^-1   (d_v <= d_h)
//   RL(G) = CL(B) . RL(-K) + 1,  G = 1 - K B          CL(W) = RL(S_hh) . RL(G),  W = S_hh G^T
//   CL(F) = RL(G) . CL(W) + RL(K) . (RL(S_v) . RL(K))
// For d_v > d_h S_vv is factored column by column and the gain substituted row by row instead: B S_hh B^T is a thin product there,
// and with little noise the explicit L^-1 (and pivots that are not scaled by their square roots) made K, hence F, up to 16
// times less accurate (fp32, d_h = 2, d_v = 16, S_v = 1e-4); for d_v <= d_h both are equally accurate.  It costs 0.9 us a
// step: 4096 sequences x 24 steps, d_h = 4, d_v = 16, fp32 45 -> 66 us, fp64 71 -> 95 (one recursion per sequence: 158, 165).
// And per 16 sequences (means and innovations as the columns of a tile)
//   mu = A f,  d = v - B mu,  f = mu + K d,  z = L^-1 d.
//
// Bound by writing F for large batches, by the serial covariance step for small ones.
// 65536 sequences x 32 steps, dh = dv = 16, fp32: 3250 us with every sequence's own recursion, now
// 476 (5 TB/s); 8192 sequences 509 -> 77; 1024 322 -> 63.  fp64: 4088 -> 981, 631 -> 121, 313 -> 98.
// ---------------------------------------------------------------------------------------
template <typename T>
struct KsLds {
    static constexpr int PS = 16 + 16 / (int)sizeof(T);
    T A[16 * PS], B[16 * PS], S[16 * PS];
    struct Step {
        T K[16 * PS], Li[16 * PS], F[16 * PS];
    } step[2];
    double logdet;  // sum over the steps of log det L
    int32_t bad;
};
constexpr int KS_MAX_WORKERS = 2;

template <typename T>
__device__ __forceinline__ typename Mfma<T>::acc_t ks_mul(typename Mfma<T>::acc_t a, typename Mfma<T>::acc_t b,
                                                          typename Mfma<T>::acc_t c)
{
#pragma unroll
    for (int s = 0; s < 4; ++s)
        c = Mfma<T>::run(a[s], b[s], c);
    return c;
}
template <typename T>
__device__ __forceinline__ typename Mfma<T>::acc_t ks_rl(const T *X, int lane)
{
    typename Mfma<T>::acc_t v;
#pragma unroll
    for (int s = 0; s < 4; ++s)
        v[s] = X[(lane & 15) * KsLds<T>::PS + Mfma<T>::row(lane, s)];
    return v;
}
template <typename T>
__device__ __forceinline__ typename Mfma<T>::acc_t ks_cl(const T *X, int lane)
{
    typename Mfma<T>::acc_t v;
#pragma unroll
    for (int s = 0; s < 4; ++s)
        v[s] = X[Mfma<T>::row(lane, s) * KsLds<T>::PS + (lane & 15)];
    return v;
}
// The elements k(lane, s) < n of a vector in memory.  In fp32 they are four consecutive ones.
template <typename T>
__device__ __forceinline__ typename Mfma<T>::acc_t ks_load(const T *p, int n, int lane)
{
    typename Mfma<T>::acc_t v = {0, 0, 0, 0};
    if constexpr (sizeof(T) == 4) {
        const int k = Mfma<T>::row(lane, 0);
        if (k + 4 <= n) {
            const typename LooseVec<T>::type w = *reinterpret_cast<const typename LooseVec<T>::type *>(p + k);
#pragma unroll
            for (int s = 0; s < 4; ++s)
                v[s] = w[s];
            return v;
        }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
        if (Mfma<T>::row(lane, s) < n)
            v[s] = p[Mfma<T>::row(lane, s)];
    return v;
}
template <typename T>
__device__ __forceinline__ void ks_store(T *p, int n, int lane, typename Mfma<T>::acc_t v)
{
    if constexpr (sizeof(T) == 4) {
        const int k = Mfma<T>::row(lane, 0);
        if (k + 4 <= n) {
            typename LooseVec<T>::type w;
#pragma unroll
            for (int s = 0; s < 4; ++s)
                w[s] = v[s];
            *reinterpret_cast<typename LooseVec<T>::type *>(p + k) = w;
            return;
        }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
        if (Mfma<T>::row(lane, s) < n)
            p[Mfma<T>::row(lane, s)] = v[s];
}

// Row r of K = M S^-1 in place of row r of M by way of S = L L^T, S and L one row per lane (the four lane rows hold copies);
// rows and columns from dv on are those of the identity.  Also gives L, and L_rr in lrr.  False: a pivot that is not > 0.
template <typename T>
__device__ __forceinline__ bool ks_factor_gain(T (&S)[16], T (&M)[16], T &lrr, int r, int dv)
{
    bool good = true;
    const T one = T(1);
    T invd = one;
    lrr = one;
    static_for<0, 4>([&](auto bc) {
        constexpr int b0 = 4 * decltype(bc)::value;
        if (b0 >= dv)
            return;
        kf_settle(S);
        static_for<b0, b0 + 4>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            kf_settle1(S[k]);
            const T d = mul_row<k>(S[k], one);
            good = good && d > T(0);
            const T rs = rsqrt_acc(d);
            S[k] *= rs;
            invd = r == k ? rs : invd;
            lrr = r == k ? S[k] : lrr;
            const T x = M[k] * rs;  // X L^T = M
            M[k] = x;
            kf_settle1(S[k]);
            static_for<k + 1, 16>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                fnmac_row<j>(S[j], S[k], S[k]);  // S[r][j] -= L[r][k] L[j][k]
                fnmac_row<j>(M[j], S[k], x);     // M[r][j] -= x L[j][k]
            });
        });
    });
    static_for<0, 4>([&](auto bc) {
        constexpr int b0 = 12 - 4 * decltype(bc)::value;
        if (b0 >= dv)
            return;
        kf_settle(S);
        kf_settle1(invd);
        static_for<0, 4>([&](auto tc) {  // K L = X
            constexpr int j = b0 + 3 - decltype(tc)::value;
            const T y = mul_row<j>(invd, M[j]);
            M[j] = y;
            static_for<0, j>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                fnmac_row<j>(M[i], S[i], y);  // M[r][i] -= y L[j][i]
            });
        });
    });
    return good;
}

// THIN: d_v > d_h
template <typename T, bool THIN>
__global__ __launch_bounds__(64 * (1 + KS_MAX_WORKERS), sizeof(T) == 4 ? 3 : 2) void k_kalman_shared(KfArgs<T> a, int per_worker)
{
    using MF = Mfma<T>;
    using acc_t = typename MF::acc_t;
    using L = typename LooseVec<T>::type;
    constexpr int VW = MF::VW, PS = KsLds<T>::PS;
    __shared__ __align__(16) KsLds<T> sm;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int dh = a.dh, dv = a.dv, steps = a.T_;

    if (wave == 0) {  // A, B zero padded
        const int r = lane & 15, c0 = (lane >> 4) * 4;
#pragma unroll
        for (int c = c0; c < c0 + 4; ++c) {
            sm.A[r * PS + c] = (r < dh && c < dh) ? a.A[r * dh + c] : T(0);
            sm.B[r * PS + c] = (r < dv && c < dh) ? a.B[r * dh + c] : T(0);
        }
    }
    __syncthreads();
    const acc_t rA = ks_rl<T>(sm.A, lane), rB = ks_rl<T>(sm.B, lane), zero = acc_t{0, 0, 0, 0};

    if (wave == 0) {
        const int r = lane & 15, g = lane >> 4;
        int kk[4];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            kk[s] = MF::row(lane, s);
        const acc_t cB = ks_cl<T>(sm.B, lane);
        acc_t cShT, cSv, rSv, rS, cF = zero, one;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = kk[s];
            cShT[s] = (r < dh && k < dh) ? a.Sh[r * dh + k] : T(0);
            one[s] = r == k ? T(1) : T(0);
            rSv[s] = (r < dv && k < dv) ? a.Sv[r * dv + k] : one[s];  // identity padded: a unit pivot there
            cSv[s] = (r < dv && k < dv) ? a.Sv[k * dv + r] : one[s];
            rS[s] = (r < dh && k < dh) ? a.S0[r * dh + k] : T(0);
        }
        double logdet = 0.0;
        int32_t bad = 0;
        for (int t = 0; t <= steps; ++t) {
            if (t < steps) {
                auto &st = sm.step[t & 1];
                if (t > 0)
                    rS = ks_mul<T>(rA, ks_mul<T>(cF, rA, zero), cShT);
                const acc_t cM = ks_mul<T>(rS, rB, zero);
                const acc_t cS = ks_mul<T>(rB, cM, cSv);
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    sm.S[kk[s] * PS + r] = cS[s];
                const acc_t cMT = ks_mul<T>(rB, rS, zero);
                if constexpr (THIN) {  // (M's rows by way of K's place)
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        st.K[r * PS + kk[s]] = cMT[s];
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                T S[16], M[16], x[4];
                kf_row(S, sm.S + r * PS);
                bool failed;
                if constexpr (THIN) {
                    T lrr;
                    kf_row(M, st.K + r * PS);
                    failed = !ks_factor_gain(S, M, lrr, r, dv);
                    diag_invert<T>(S, lrr, x, r, g);
                } else {
                    failed = diag_factor_invert<T, true>(S, x, r, g, dv) != 0;
                }
                if (failed && bad == 0)
                    bad = t + 1;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    st.Li[r * PS + 4 * j + g] = (4 * j + g <= r) ? x[j] : T(0);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                const acc_t rLi = ks_rl<T>(st.Li, lane), cLi = ks_cl<T>(st.Li, lane);
                if (r < dv)
                    logdet -= (double)log(st.Li[r * PS + r]);
                acc_t rK, nK;
                if constexpr (THIN) {
                    if (g == 0) {
#pragma unroll
                        for (int j = 0; j < 16; ++j)
                            st.K[r * PS + j] = M[j];
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                    rK = ks_rl<T>(st.K, lane);
                } else {
                    rK = ks_mul<T>(cLi, ks_mul<T>(rLi, cMT, zero), zero);
                }
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    nK[s] = -rK[s];
                    st.K[r * PS + kk[s]] = rK[s];
                }
                const acc_t rG = ks_mul<T>(cB, nK, one);
                const acc_t cY = ks_mul<T>(rSv, rK, zero);
                const acc_t cW = ks_mul<T>(rS, rG, zero);
                cF = ks_mul<T>(rG, cW, ks_mul<T>(rK, cY, zero));
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    st.F[kk[s] * PS + r] = cF[s];
            } else {
#pragma unroll
                for (int off = 8; off >= 1; off >>= 1)
                    logdet += __shfl_xor(logdet, off, 16);
                if (lane == 0) {
                    sm.logdet = logdet;
                    sm.bad = bad;
                }
            }
            __syncthreads();
        }
        return;
    }

    // ---- a worker: sequences b0 .. b0 + items - 1 in tiles of 16, lane l with sequence l % 16 of each ----
    const int workers = (int)(blockDim.x >> 6) - 1;
    const int64_t b0 = ((int64_t)blockIdx.x * workers + wave - 1) * per_worker;
    const int items = (int)(a.batch - b0 < per_worker ? (a.batch - b0 > 0 ? a.batch - b0 : 0) : per_worker);
    acc_t f[4], v[4];
    double nll[4];
    int64_t seq[4];  // spare lanes repeat the last sequence and store nothing
    const acc_t mu0 = ks_load<T>(a.mu0, dh, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t b = b0 + 16 * q + (lane & 15);
        seq[q] = b < a.batch ? b : a.batch - 1;
        f[q] = mu0;
        v[q] = zero;
        if (steps > 0 && 16 * q < items)
            v[q] = ks_load<T>(a.v + seq[q] * steps * dv, dv, lane);
        nll[q] = 0.0;
    }

    // Writing F: an item has nch chunks of VW elements; 64 lanes take one item (in rounds of 64 chunks) or ipi items at once.
    const int ff = dh * dh, nch = (ff + VW - 1) / VW;
    const int ipi = nch >= 64 ? 1 : 64 / nch;
    const int sub = nch >= 64 ? 0 : lane / nch, c0 = nch >= 64 ? lane : lane - sub * nch;
    constexpr int ROUNDS = 256 / VW / 64;  // 1 in fp32, 2 in fp64
    int src[ROUNDS][VW], left[ROUNDS];
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) {
        const int e0 = (c0 + 64 * q) * VW;
        left[q] = (sub < ipi && (q == 0 || nch > 64)) ? ff - e0 : 0;
#pragma unroll
        for (int u = 0; u < VW; ++u) {
            const int e = e0 + u < ff ? e0 + u : 0, row = e / dh;
            src[q][u] = row * PS + (e - row * dh);
        }
    }
    const int64_t item_stride = (int64_t)steps * ff;

    __syncthreads();  // step 0's matrices
    for (int t = 0; t < steps; ++t) {
        const auto &st = sm.step[t & 1];
        const acc_t rK = ks_rl<T>(st.K, lane), rLi = ks_rl<T>(st.Li, lane);
        acc_t d[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (16 * q >= items)
                break;
            if (t > 0)
                f[q] = ks_mul<T>(rA, f[q], zero);
            d[q] = v[q] - ks_mul<T>(rB, f[q], zero);  // (rows from dv on: zero minus zero)
            if (t + 1 < steps)
                v[q] = ks_load<T>(a.v + (seq[q] * steps + t + 1) * dv, dv, lane);
        }
        if (a.F) {
            L chunk[ROUNDS];
#pragma unroll
            for (int q = 0; q < ROUNDS; ++q)
#pragma unroll
                for (int u = 0; u < VW; ++u)
                    chunk[q][u] = st.F[src[q][u]];
            T *Fo = a.F + (b0 + sub) * item_stride + (int64_t)t * ff + (int64_t)c0 * VW;
            for (int i = sub; i < items; i += ipi, Fo += ipi * item_stride) {
#pragma unroll
                for (int q = 0; q < ROUNDS; ++q) {
                    if (left[q] >= VW) {  // (not read again here: 8192 sequences fp64 166 -> 129 us past the caches)
                        __builtin_nontemporal_store(chunk[q], reinterpret_cast<L *>(Fo + 64 * VW * q));
                    } else {
#pragma unroll
                        for (int u = 0; u < VW - 1; ++u)
                            if (u < left[q])
                                Fo[64 * VW * q + u] = chunk[q][u];
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (16 * q >= items)
                break;
            f[q] = ks_mul<T>(rK, d[q], f[q]);
            if (a.f && 16 * q + (lane & 15) < items)
                ks_store<T>(a.f + (seq[q] * steps + t) * dh, dh, lane, f[q]);
            const acc_t z = ks_mul<T>(rLi, d[q], zero);
#pragma unroll
            for (int s = 0; s < 4; ++s)
                nll[q] += 0.5 * (double)z[s] * (double)z[s];
        }
        __syncthreads();
    }
    const double rest = sm.logdet + 0.5 * steps * dv * 1.8378770664093454835606594728112;  // log(2 pi)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        nll[q] += __shfl_xor(nll[q], 16, 64);
        nll[q] += __shfl_xor(nll[q], 32, 64);
        if (lane < 16 && 16 * q + lane < items) {
            a.nll[seq[q]] = (T)(nll[q] + rest);
            if (a.info)
                a.info[seq[q]] = sm.bad;
        }
    }
}

template <typename T>
static la_status launch_kalman_shared(const KfArgs<T> &a, hipStream_t st)
{
    // Few sequences: two workers of 16 each, so that writing F does not hold a step up (8192 sequences, dh = dv = 16, fp32:
    // 97 us, 121 with 32 each, 193 with 64).  32 each where 16 give more workgroups than are resident (fp64 above 16384
    // sequences: 32767 x 24 steps, d = 4, 163 -> 84 us, d = 16 323 -> 314) or than compute units and a step is short
    // (d_h <= 4 above 8192: 16384 x 24, d = 4, fp32 43 -> 38, fp64 71 -> 59; d_h = 12 79 -> 113 and 115 -> 127).  From 32768 on
    // the workgroups should all be resident (12 wavefronts per compute unit in fp32, 8 in fp64): one worker of 64 where F is
    // large, so that more of them write (65536, dh = 16, fp64: 1000 us against 1052 with two of 32), else two workers of 32, in
    // fp64 of 64 (dh = 4, dv = 3: fp32 100 us against 115 with one worker of 64; fp64 207 against 248 with two of 32), and
    // in fp32 above 65536 as well where a step is short (131072 x 24, d = 4, without states 150 -> 99, with them 161 -> 114;
    // larger d_h gains nothing).
    const bool many = a.batch >= 32768;
    const int workers = many && a.dh > 8 ? 1 : 2;
    const bool wide = (a.dh <= 4 && a.batch > 8192) || (sizeof(T) == 8 && a.batch > 16384);
    const int per_worker = !many ? (wide ? 32 : 16) : (workers == 1 || sizeof(T) == 8 || (a.dh <= 4 && a.batch > 65536) ? 64 : 32);
    const int64_t per_wg = (int64_t)workers * per_worker, blocks = (a.batch + per_wg - 1) / per_wg;
    if (blocks > 0x7fffffffll)
        return LA_ERR_UNSUPPORTED;
    if (a.dv > a.dh)
        LA_LAUNCH((k_kalman_shared<T, true>), dim3((unsigned)blocks), dim3(64 * (1 + workers)), 0, st, a, per_worker);
    else
        LA_LAUNCH((k_kalman_shared<T, false>), dim3((unsigned)blocks), dim3(64 * (1 + workers)), 0, st, a, per_worker);
    return launch_check("kalman");
}

// fp32, one model, dimensions up to 4: the recursion per sequence with 4 lanes each (16 sequences a wavefront) is ahead of the
// common one (24 steps, us, own -> common recursion):
//  * for d_v > d_h, where the gain's substitution is the common recursion's chain: 4096 sequences of d = (1, 3) 34 -> 42, 131072
//    134 -> 174;
//  * on two and three of its wavefronts per SIMD where little is written: d = (3, 2) with states, 32704 50 -> 56, 40960 64 -> 66;
//    without states 45 -> 47 and the same;
//  * on more than four where F's items are not whole runs of 16 bytes, or one: (3, 2) 163840 172 -> 208, (1, 1) 166 -> 188.
// On the fourth (49153 to 65536) the common one is ahead everywhere: (1, 3) 74 -> 68, (4, 2) with states 82 -> 72.
static bool small_dims_prefer_own_recursion(int64_t batch, int dh, int dv, bool states)
{
    if (dh > 4 || dv > 4 || (batch > 49152 && batch <= 65536))
        return false;
    if (dv > dh)
        return true;
    if (batch <= 65536)
        return batch > 16384 && (dh <= 3 || !states);
    return states && dh <= 3;
}

template <typename T>
la_status launch_kalman(const T *A, const T *B, const T *Sh, const T *Sv, const T *mu0, const T *S0, const T *v, T *f,
                        T *F, T *nll, int32_t *info, int64_t batch, int steps, int dh, int dv, int shared,
                        hipStream_t st)
{
    if (batch <= 0)
        return LA_OK;
    if (dh < 1 || dv < 1 || dh > 16 || dv > 16)
        return LA_ERR_UNSUPPORTED;
    KfArgs<T> a{A, B, Sh, Sv, mu0, S0, v, f, F, nll, info, batch, steps, dh, dv, shared};
    if (shared && !(sizeof(T) == 4 && small_dims_prefer_own_recursion(batch, dh, dv, F != nullptr)))
        return launch_kalman_shared<T>(a, st);
    if (dh <= 4 && dv <= 4)
        return launch_kalman_d<T, 4>(a, st);
    // 8 lanes per sequence pay in fp32 only (1.76 -> 0.89 ms per 65536 x 32 steps at d = 8): in fp64 the
    // broadcast is four 32-bit lane moves beside the multiply-add and 16 lanes stay 4 % ahead
    if constexpr (sizeof(T) == 4) {
        if (dh <= 8 && dv <= 8)
            return launch_kalman_d<T, 8>(a, st);
    }
    return launch_kalman_d<T, 16>(a, st);
}

template la_status launch_kalman<float>(const float *, const float *, const float *, const float *, const float *,
                                        const float *, const float *, float *, float *, float *, int32_t *, int64_t,
                                        int, int, int, int, hipStream_t);
template la_status launch_kalman<double>(const double *, const double *, const double *, const double *,
                                         const double *, const double *, const double *, double *, double *, double *,
                                         int32_t *, int64_t, int, int, int, int, hipStream_t);

}  // namespace la
