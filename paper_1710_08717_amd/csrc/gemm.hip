// Batched strided GEMM on the gfx950 matrix cores: the dense contraction inside every
// blocked algorithm of the library (trailing syrk/gemm update of the right-looking potrf,
// the off-diagonal updates of blocked trsm / trmm, and the three triangular phases of the
// potrf backward expression of arXiv 1710.08717, section 4.2).
//
//   C(i,j) = beta * C(i,j) + alpha * sum_k A(i,k) B(k,j)
//
// Operands are strided views (either index may be the contiguous one), so transposes and
// upper/lower variants never copy.  Triangular operands are masked while they are staged
// in LDS and their structurally-zero K range is skipped.
//
// k_gemm: 16-byte vector loads, register prefetch of the next K slab while the current one is
// multiplied out of LDS, 128x128 (K slabs of 16, double-buffered LDS, one barrier per slab),
// 64x64 (K slabs of 32) or 32x32 workgroup tiles (K slabs of 64, for the small, latency-bound
// grids of the recursion's lower levels), four
// wavefronts in a 2 x 2 arrangement, 16x16x4 MFMA (v_mfma_f64_16x16x4_f64 /
// v_mfma_f32_16x16x4_f32).  Two forms: with 16-byte aligned operands and K a multiple of 16 every
// chunk is one aligned load; otherwise (odd sizes and leading dimensions) the chunks are loaded
// with the alignment of one element and the ones that cross the end of the operand element by
// element, zeros behind it.  The second form keeps the pipeline of the first and issues the same
// number of loads; a chunk then spans two cache lines more often.  (Staging such operands element by element without prefetch, as an earlier kernel
// did, was bound by its load instructions and address arithmetic: factor + gradient of one
// fp64 matrix of n = 3001 8.83 ms, now 2.77; 24 fp32 matrices of n = 333 0.70 ms, now 0.23.)
#include <algorithm>

#include "common.hpp"

namespace la {

// ---------------------------------------------------------------------------------------
// Workgroup -> work slot mapping.  Consecutive workgroups are dealt round-robin to the 8 XCDs
// (each with its own L2).  Slots are regrouped in chunks of 8 x 16: inside a chunk every XCD
// gets 16 consecutive slots (neighbouring tiles of one tile row share their A panel in that
// XCD's L2), while all XCDs still advance through the slot list at the same pace, which
// matters because triangular operands make the work per tile vary along the list.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ int64_t xcd_slot(int64_t w, int64_t total, int CH = 16)
{
    const int64_t c = w / (8 * CH);
    if ((c + 1) * 8 * CH > total)
        return w;  // incomplete last chunk keeps its order
    const int r = (int)(w % (8 * CH));
    return c * 8 * CH + (r % 8) * CH + r / 8;
}

// Tile enumeration.  Workgroups go to XCDs in a fixed round-robin, so the list of tiles must be
// (a) free of tiles that have nothing to do and (b) ordered so that the work per tile changes
// slowly along it; then every XCD ends up with the same share.
//   order 0: all tiles, row-major.
//   order 1: tiles on or below the diagonal only (tn <= tm), row by row.
//   order 2: tiles on or above the diagonal only (tm <= tn), column by column.
//   order 3: all tiles of a square grid in "shells" max(tm, tn) = s, s ascending: every tile of
//            a shell has the same K range when both operands are triangular.
//   order 4: all tiles, column-major (the K range depends on the column only when just B is
//            triangular).
//   order 5: tiles on or below the diagonal in bands of 8 diagonals tm - tn = d, the band with the
//            largest d first; inside a band row by row from the last row up, a row's tiles by
//            falling d.  For lower x lower = lower products the K range of a tile is d + 1 tile
//            edges, so this list is nearly sorted by work (which the slots need to fill evenly:
//            the heaviest tile is three times the mean) while the (up to) 8 consecutive tiles of a
//            row still share their A panel.
__device__ __forceinline__ void decode_tile(int order, int t, int tiles_m, int tiles_n, int &tm, int &tn)
{
    if (order == 0) {
        tm = t / tiles_n;
        tn = t % tiles_n;
    } else if (order == 4) {
        tn = t / tiles_m;
        tm = t % tiles_m;
    } else if (order == 5) {
        const int T = tiles_m;
        int b = (T - 1) / 8;
        for (;; --b) {  // band: diagonals 8 b .. min(T - 1, 8 b + 7)
            const int dlo = 8 * b, dhi = min(T - 1, dlo + 7);
            const int cnt = (dhi - dlo + 1) * T - (dlo + dhi) * (dhi - dlo + 1) / 2;  // sum of T - d
            if (t < cnt || b == 0)
                break;
            t -= cnt;
        }
        const int dlo = 8 * b, dhi = min(T - 1, dlo + 7);
        int i = T - 1;
        for (;; --i) {  // row i holds the diagonals min(dhi, i) .. dlo of the band
            const int cnt = min(dhi, i) - dlo + 1;
            if (t < cnt || i == dlo)
                break;
            t -= cnt;
        }
        tm = i;
        tn = i - (min(dhi, i) - t);
    } else if (order == 3) {
        int s_ = (int)sqrt((double)t);
        while ((s_ + 1) * (s_ + 1) <= t)
            ++s_;
        while (s_ * s_ > t)
            --s_;
        const int r = t - s_ * s_;
        if (r <= s_) {
            tm = s_;
            tn = r;
        } else {
            tm = r - s_ - 1;
            tn = s_;
        }
    } else {
        int a = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
        while ((a + 1) * (a + 2) / 2 <= t)
            ++a;
        while (a * (a + 1) / 2 > t)
            --a;
        const int b = t - a * (a + 1) / 2;
        tm = order == 1 ? a : b;
        tn = order == 1 ? b : a;
    }
}

__device__ __forceinline__ int64_t tile_count_dev(int order, int tiles_m, int tiles_n)
{
    if (order == 1 || order == 2 || order == 5)
        return (int64_t)tiles_m * (tiles_m + 1) / 2;
    return (int64_t)tiles_m * tiles_n;
}
static inline int64_t tile_count(int order, int tiles_m, int tiles_n)
{
    if (order == 1 || order == 2 || order == 5)
        return (int64_t)tiles_m * (tiles_m + 1) / 2;
    return (int64_t)tiles_m * tiles_n;
}

__device__ __forceinline__ void k_range(const GemmOpts &o, int i0, int j0, int BM, int BN, int K, int &kbeg, int &kend)
{
    kbeg = 0;
    kend = K;
    if (o.triA == 1)
        kend = min(kend, i0 + BM);
    else if (o.triA == 2)
        kbeg = max(kbeg, i0);
    if (o.triB == 1)
        kbeg = max(kbeg, j0);
    else if (o.triB == 2)
        kend = min(kend, j0 + BN);
}

template <typename T>
__device__ __forceinline__ void store_c(T *Cp, int64_t rs, int64_t cs, int i, int j, int M, int N, T acc, T alpha,
                                        T beta, const GemmOpts &o)
{
    if (i < M && j < N && !(o.maskC == 1 && i < j) && !(o.maskC == 2 && i > j)) {
        T upd = alpha * acc;
        if (o.halfDiag && i == j)
            upd *= T(0.5);
        T *c = Cp + (int64_t)i * rs + (int64_t)j * cs;
        *c = (beta == T(0)) ? upd : fma(beta, *c, upd);
    }
}

// ---------------------------------------------------------------------------------------
// Tile kernel.  AKF: A(i,k) has k contiguous (A.cs == 1), else i contiguous (A.rs == 1).
// BKF: B(k,j) has k contiguous (B.rs == 1), else j contiguous (B.cs == 1).
// LDS slab layouts (chosen so that global->LDS stores are 16-byte vectors and the MFMA
// fragment reads are bank-conflict free):
//   k contiguous:     s[o][BK + VW]      (row stride 18 doubles / 20 floats)
//   outer contiguous: s[k][OUT + 16]
// ---------------------------------------------------------------------------------------
template <typename T, int OUT, int BK, bool KF>
struct Slab {
    using MF = Mfma<T>;
    static constexpr int VW = MF::VW;
    static constexpr int LD = KF ? (BK + VW) : (OUT + 16);
    static constexpr int ELEMS = KF ? OUT * LD : BK * LD;
    static constexpr int NCH = OUT * BK / VW / 256;  // 16-byte chunks per thread
    static_assert(NCH >= 1, "tile too small for 256 threads");
    static constexpr int so = KF ? LD : 1;  // LDS stride of the outer index
    static constexpr int sk = KF ? 1 : LD;  // LDS stride of k

    // (outer, k) of chunk c of this thread
    static __device__ __forceinline__ void coords(int c, int &o, int &k)
    {
        const int q = c * 256 + threadIdx.x;
        if constexpr (KF) {
            o = q / (BK / VW);
            k = (q % (BK / VW)) * VW;
        } else {
            k = q / (OUT / VW);
            o = (q % (OUT / VW)) * VW;
        }
    }
};

// One slab of an operand into registers: outer rows o0 .. o0 + OUT - 1 of `no`, k from k0 on, of `nk`.
// RAG = false: whole aligned chunks only (nk a multiple of BK; `no` a multiple of VW when !KF).
template <typename T, int OUT, int BK, bool KF, bool RAG, typename RV>
__device__ __forceinline__ void slab_fetch(RV &r, const T *src, int64_t so, int64_t sk, int o0, int no, int k0, int nk)
{
    using S = Slab<T, OUT, BK, KF>;
    using V = typename Mfma<T>::vec_t;
    using L = typename LooseVec<T>::type;
    if (RAG && o0 + OUT <= no && k0 + BK <= nk) {  // (uniform) nothing crosses an end
#pragma unroll
        for (int c = 0; c < S::NCH; ++c) {
            int o, k;
            S::coords(c, o, k);
            const L v = *reinterpret_cast<const L *>(src + (int64_t)(o0 + o) * so + (int64_t)(k0 + k) * sk);
            r[c] = __builtin_bit_cast(V, v);
        }
        return;
    }
#pragma unroll
    for (int c = 0; c < S::NCH; ++c) {
        int o, k;
        S::coords(c, o, k);
        V v;
        if constexpr (S::VW == 2)
            v = V{0, 0};
        else
            v = V{0, 0, 0, 0};
        const T *e = src + (int64_t)(o0 + o) * so + (int64_t)(k0 + k) * sk;
        if constexpr (RAG) {
            // elements of the chunk that exist
            const int left = KF ? (o0 + o < no ? nk - (k0 + k) : 0) : (k0 + k < nk ? no - (o0 + o) : 0);
            if (left >= S::VW) {
                const L x = *reinterpret_cast<const L *>(e);
                v = __builtin_bit_cast(V, x);
            } else {
                T *q = reinterpret_cast<T *>(&v);
#pragma unroll
                for (int u = 0; u < S::VW - 1; ++u)
                    if (u < left)
                        q[u] = e[u];
            }
        } else {
            if (o0 + o < no)
                v = *reinterpret_cast<const V *>(e);
        }
        r[c] = v;
    }
}

template <typename T, int OUT, int BK, bool KF, typename RV>
__device__ __forceinline__ void slab_commit(T *s, RV &r, int o0, int k0, int tri)
{
    using S = Slab<T, OUT, BK, KF>;
    using V = typename Mfma<T>::vec_t;
    // Does this slab touch the zero side of a triangular operand at all?  Decided once per slab
    // (a scalar branch); most slabs do not and take the plain copy below.
    bool need_mask = false;
    if (tri == 1)
        need_mask = (o0 < k0 + BK - 1);  // keep o >= k: some (o, k) with o < k exists
    else if (tri == 2)
        need_mask = (o0 + OUT - 1 > k0);
    if (!need_mask) {
#pragma unroll
        for (int c = 0; c < S::NCH; ++c) {
            int o, k;
            S::coords(c, o, k);
            *reinterpret_cast<V *>(s + o * S::so + k * S::sk) = r[c];
        }
        return;
    }
    // keep o >= k (tri 1) or o <= k (tri 2): with d = (o - k) for tri 1 and (k - o) for tri 2, keep d >= 0
    const int sgn = tri == 1 ? 1 : -1;
#pragma unroll
    for (int c = 0; c < S::NCH; ++c) {
        int o, k;
        S::coords(c, o, k);
        V v = r[c];
        T *e = reinterpret_cast<T *>(&v);
        const int d0 = sgn * ((o0 + o) - (k0 + k));
#pragma unroll
        for (int u = 0; u < S::VW; ++u) {
            const int d = d0 + (KF ? -sgn * u : sgn * u);  // element u moves along k (KF) or along o
            e[u] = d >= 0 ? e[u] : T(0);
        }
        *reinterpret_cast<V *>(s + o * S::so + k * S::sk) = v;
    }
}

template <typename T, int BM, int BN, int BK, int NBUF, bool AKF, bool BKF, bool RAG, bool SYM>
__global__ __launch_bounds__(256, 2) void k_gemm(View<const T> A, View<const T> B, View<T> C, int64_t batch, int M,
                                                 int N, int K, T alpha, T beta, GemmOpts o, int tiles_m, int tiles_n)
{
    using MF = Mfma<T>;
    using acc_t = typename MF::acc_t;
    using V = typename MF::vec_t;
    using SA = Slab<T, BM, BK, AKF>;
    using SB = Slab<T, BN, BK, BKF>;
    constexpr int WM = BM / 2, WN = BN / 2;
    constexpr int TM = WM / 16, TN = WN / 16;
    __shared__ __align__(16) T sA[NBUF][SA::ELEMS];
    __shared__ __align__(16) T sB[NBUF][SB::ELEMS];

    const int64_t per = tile_count_dev(o.order, tiles_m, tiles_n);
    int64_t b;
    int tile;
    if (o.xcd_batch) {
        // Batched launch: XCD x (workgroups x, x + 8, ...) owns the items b = x, x + 8, ... and
        // goes through the tile list once for all of them, tile by tile.  The tile lists are
        // heaviest-first, so the uneven tiles of triangular problems pack well over the
        // workgroup slots, and the tiles of one item still meet in one L2.
        const int x = (int)(blockIdx.x & 7);
        const int64_t q = blockIdx.x >> 3, mpx = (batch + 7) >> 3;
        tile = (int)(q / mpx);
        b = (q % mpx) * 8 + x;
        if (b >= batch)
            return;
    } else {
        // a few items: tile-major too (tile t of every item, then tile t + 1, ...)
        const int64_t slot = xcd_slot(blockIdx.x, per * batch, o.order == 5 ? 8 : 16);
        tile = (int)(slot / batch);
        b = slot % batch;
    }
    if (o.reverse && o.order != 5)
        tile = (int)per - 1 - tile;  // heaviest tiles first when the work grows along the tile list
    int tm, tn;
    decode_tile(o.order, tile, tiles_m, tiles_n, tm, tn);
    const int i0 = tm * BM, j0 = tn * BN;
    if ((o.maskC == 1 && j0 > i0 + BM - 1) || (o.maskC == 2 && i0 > j0 + BN - 1))
        return;

    int Kl = K;  // slice s of a split K range: K elements from s * K on, fewer for the last slice
    if (o.ksplit > 1)
        Kl = min(K, o.ktotal - (int)(b % o.ksplit) * K);
    int kbeg, kend;
    k_range(o, i0, j0, BM, BN, Kl, kbeg, kend);
    kbeg = (kbeg / BK) * BK;
    // (whole slabs: the triangular masks clear what lies past kend, the fetch what lies past K)

    const T *Ap = A.item(b);
    const T *Bp = B.item(b);
    T *Cp = C.item(b);
    const int triB_o = o.triB == 1 ? 2 : (o.triB == 2 ? 1 : 0);

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = (w >> 1) * WM, wn = (w & 1) * WN;
    const int l16 = lane & 15, lk = lane >> 4;

    acc_t acc[TM][TN];
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int y = 0; y < TN; ++y)
            acc[x][y] = acc_t{0, 0, 0, 0};

    // Software pipeline.  Slabs travel global memory -> registers -> LDS -> matrix cores.
    // Two LDS buffers: while slab s is multiplied out of one buffer, slab s+1 (already in
    // registers) is written into the other and slab s+2 is requested from memory, so the only
    // thing between two blocks of MFMAs is one barrier: it orders the reads of slab s before
    // the overwrite by slab s+2 and the writes of slab s+1 before their reads.
    // One LDS buffer: slab s+1 is fetched into registers while slab s is multiplied, and written
    // once everybody is done reading (two barriers per slab).
    V ra[SA::NCH], rb[SB::NCH];
    auto multiply = [&](const T *a_s, const T *b_s) {
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4) {
            T af[TM], bf[TN];
#pragma unroll
            for (int x = 0; x < TM; ++x)
                af[x] = a_s[(wm + x * 16 + l16) * SA::so + (kk + lk) * SA::sk];
#pragma unroll
            for (int y = 0; y < TN; ++y)
                bf[y] = b_s[(wn + y * 16 + l16) * SB::so + (kk + lk) * SB::sk];
#pragma unroll
            for (int x = 0; x < TM; ++x)
#pragma unroll
                for (int y = 0; y < TN; ++y)
                    acc[x][y] = MF::run(af[x], bf[y], acc[x][y]);
        }
    };
    // SYM (GemmOpts::symsum): with 1 a second pass adds B^T A^T -- same strides, the base pointers change places
    const int passes = SYM && o.symsum == 1 ? 2 : 1;
    for (int pass = 0; pass < passes; ++pass) {
    if (SYM && pass == 1) {
        const T *t = Ap;
        Ap = Bp;
        Bp = t;
    }
    if constexpr (NBUF == 2) {
        if (kbeg < kend) {
            slab_fetch<T, BM, BK, AKF, RAG>(ra, Ap, A.rs, A.cs, i0, M, kbeg, Kl);
            slab_fetch<T, BN, BK, BKF, RAG>(rb, Bp, B.cs, B.rs, j0, N, kbeg, Kl);
            slab_commit<T, BM, BK, AKF>(sA[0], ra, i0, kbeg, o.triA);
            slab_commit<T, BN, BK, BKF>(sB[0], rb, j0, kbeg, triB_o);
            if (kbeg + BK < kend) {
                slab_fetch<T, BM, BK, AKF, RAG>(ra, Ap, A.rs, A.cs, i0, M, kbeg + BK, Kl);
                slab_fetch<T, BN, BK, BKF, RAG>(rb, Bp, B.cs, B.rs, j0, N, kbeg + BK, Kl);
            }
            __syncthreads();
        }
        int buf = 0;
        for (int k0 = kbeg; k0 < kend; k0 += BK) {
            if (k0 + BK < kend) {
                slab_commit<T, BM, BK, AKF>(sA[buf ^ 1], ra, i0, k0 + BK, o.triA);
                slab_commit<T, BN, BK, BKF>(sB[buf ^ 1], rb, j0, k0 + BK, triB_o);
            }
            if (k0 + 2 * BK < kend) {
                slab_fetch<T, BM, BK, AKF, RAG>(ra, Ap, A.rs, A.cs, i0, M, k0 + 2 * BK, Kl);
                slab_fetch<T, BN, BK, BKF, RAG>(rb, Bp, B.cs, B.rs, j0, N, k0 + 2 * BK, Kl);
            }
            multiply(sA[buf], sB[buf]);
            __syncthreads();
            buf ^= 1;
        }
    } else {
        if (kbeg < kend) {
            slab_fetch<T, BM, BK, AKF, RAG>(ra, Ap, A.rs, A.cs, i0, M, kbeg, Kl);
            slab_fetch<T, BN, BK, BKF, RAG>(rb, Bp, B.cs, B.rs, j0, N, kbeg, Kl);
        }
        for (int k0 = kbeg; k0 < kend; k0 += BK) {
            slab_commit<T, BM, BK, AKF>(sA[0], ra, i0, k0, o.triA);
            slab_commit<T, BN, BK, BKF>(sB[0], rb, j0, k0, triB_o);
            __syncthreads();
            if (k0 + BK < kend) {
                slab_fetch<T, BM, BK, AKF, RAG>(ra, Ap, A.rs, A.cs, i0, M, k0 + BK, Kl);
                slab_fetch<T, BN, BK, BKF, RAG>(rb, Bp, B.cs, B.rs, j0, N, k0 + BK, Kl);
            }
            multiply(sA[0], sB[0]);
            __syncthreads();
        }
    }
    }

    if constexpr (SYM) {
        // Every value goes to both triangles.  A 16 x 16 tile's mirror image is turned in the wavefront's own part of the
        // LDS (free now), so that both are stored row by row: 32 matrices of n = 512, fp64, W of the backward pass
        // 108 -> 103 us against storing the mirror image element by element.
        T *turn = sA[0] + w * (16 * 17);
        static_assert(4 * 16 * 17 <= NBUF * SA::ELEMS, "the turning areas fit the A slabs");
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int y = 0; y < TN; ++y) {
                const int it = i0 + wm + x * 16, jt = j0 + wn + y * 16;  // first row, first column of the tile
                if (jt > it || it >= M)
                    continue;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int u = MF::row(lane, v), i = it + u, j = jt + l16;
                    T upd = alpha * acc[x][y][v];
                    if (i < M && j <= i) {
                        T *c = Cp + (int64_t)i * C.rs + (int64_t)j * C.cs;
                        if (beta != T(0))
                            upd = fma(beta, *c, upd);
                        *c = upd;
                    }
                    turn[u * 17 + l16] = upd;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int u = lk + 4 * v, i = it + l16, j = jt + u;  // row j, column i of the mirror image
                    const T m = turn[l16 * 17 + u];
                    if (i < M && j < i)
                        Cp[(int64_t)j * C.rs + (int64_t)i * C.cs] = m;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            }
        return;
    }
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int y = 0; y < TN; ++y)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                store_c<T>(Cp, C.rs, C.cs, i0 + wm + x * 16 + MF::row(lane, v), j0 + wn + y * 16 + l16, M, N, acc[x][y][v],
                           alpha, beta, o);
}

// ---------------------------------------------------------------------------------------
// Thin products: at most GEMV_N columns (matrix times a few vectors).  They are bound by reading A
// once, which the tile kernels above are not built for.  A may be masked (triA); B and C are plain.
//   A with k contiguous: one wavefront per row, lanes stride over k, shuffle reduction.
//   A with i contiguous: a block takes 64 rows, its eight wavefronts an eighth of the k range each
//   (every load is 64 consecutive elements), LDS reduction.
// ---------------------------------------------------------------------------------------
constexpr int GEMV_N = 8;
constexpr int GEMV_THREADS = 512;

// The loads of several k go out together, those of B with them: with one k at a time and a branch per column a wavefront
// waits for memory twice per k (500 x 9568 times one vector, fp64, 27 -> 22 us; its transpose 59 -> 11).  A
// column more than there are costs its loads (300 items 5 x 200 times 7 columns with A transposed, fp64, bound by the
// loads of B: 31 us with eight), so every count has its own instance.
template <typename T, int N>
__global__ __launch_bounds__(GEMV_THREADS) void k_gemv(View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int K,
                                              T alpha, T beta, int triA, int tiles)
{
    constexpr int NW = GEMV_THREADS / 64;  // wavefronts: rows per block (k contiguous) or slices of k
    constexpr int UN = N == 1 ? 8 : (N <= 4 ? 4 : 2);
    __shared__ T red[NW][64][N];
    const int64_t b = blockIdx.x / tiles;
    const int tile = (int)(blockIdx.x % tiles);
    const T *Ap = A.item(b);
    const T *Bp = B.item(b);
    T *Cp = C.item(b);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t jo[N];
    T acc[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        jo[j] = j * B.cs;
        acc[j] = T(0);
    }
    const bool rows = A.cs == 1;
    const int i = rows ? tile * NW + w : tile * 64 + lane;
    if (i < M) {
        const int kb = triA == 2 ? i : 0, ke = triA == 1 ? min(K, i + 1) : K;
        const int first = rows ? kb + lane : w, step = rows ? 64 : NW, last = rows ? ke : K;
        const T *ar = Ap + (int64_t)i * A.rs;
        for (int k0 = first; k0 < last; k0 += UN * step) {
            T a[UN], x[UN][N];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int k = k0 + u * step;
                const bool in = k >= kb && k < ke;
                a[u] = in ? ar[(int64_t)k * A.cs] : T(0);
#pragma unroll
                for (int j = 0; j < N; ++j)
                    x[u][j] = in ? Bp[(int64_t)k * B.rs + jo[j]] : T(0);
            }
#pragma unroll
            for (int u = 0; u < UN; ++u)
#pragma unroll
                for (int j = 0; j < N; ++j)
                    acc[j] = fma(a[u], x[u][j], acc[j]);
        }
    }
    if (rows) {
        if (i >= M)
            return;
#pragma unroll
        for (int j = 0; j < N; ++j) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
                acc[j] += __shfl_xor(acc[j], off, WAVE);
            if (lane == 0) {
                T *c = Cp + (int64_t)i * C.rs + (int64_t)j * C.cs;
                const T upd = alpha * acc[j];
                *c = (beta == T(0)) ? upd : fma(beta, *c, upd);
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
        red[w][lane][j] = acc[j];
    __syncthreads();
    if (w == 0 && i < M) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            T sum = T(0);
#pragma unroll
            for (int q = 0; q < NW; ++q)
                sum += red[q][lane][j];
            T *c = Cp + (int64_t)i * C.rs + (int64_t)j * C.cs;
            const T upd = alpha * sum;
            *c = (beta == T(0)) ? upd : fma(beta, *c, upd);
        }
    }
}

template <typename T>
static la_status launch_gemv(View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int N, int K, T alpha,
                             T beta, int triA, hipStream_t st)
{
    const int tiles = (A.cs == 1) ? (M + GEMV_THREADS / 64 - 1) / (GEMV_THREADS / 64) : (M + 63) / 64;
    const int64_t blocks = (int64_t)tiles * batch;
    if (blocks > 0x7fffffffll)
        return LA_ERR_UNSUPPORTED;
#define LA_GO(N_)                                                                                                      \
    case N_:                                                                                                           \
        LA_LAUNCH((k_gemv<T, N_>), dim3((unsigned)blocks), dim3(GEMV_THREADS), 0, st, A, B, C, batch, M, K, alpha, beta, triA, \
                  tiles);                                                                                              \
        break
    switch (N) {
        LA_GO(1);
        LA_GO(2);
        LA_GO(3);
        LA_GO(4);
        LA_GO(5);
        LA_GO(6);
        LA_GO(7);
        LA_GO(8);
    default:
        return LA_ERR_UNSUPPORTED;
    }
#undef LA_GO
    return launch_check("gemv");
}

// ---------------------------------------------------------------------------------------
// Split along K for products with few output tiles and a long K (A^T A of a tall A, the syrk of a
// wide panel): the K range is cut into slices that run as extra batch items into a buffer of
// partial results, which a second kernel sums in a fixed order (no atomics: results are
// reproducible) while applying alpha, beta and the output mask.  The buffer comes out of the
// calling operator's workspace (at most SPLITK_MAX_BYTES of it).
// ---------------------------------------------------------------------------------------
constexpr size_t SPLITK_MAX_BYTES = (size_t)64 << 20;

template <typename T>
__global__ __launch_bounds__(256) void k_splitk_reduce(const T *partial, View<T> C, int64_t batch, int M, int N,
                                                       int splits, T alpha, T beta, GemmOpts o)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t mn = (int64_t)M * N;
    if (e >= batch * mn)
        return;
    const int64_t b = e / mn;
    const int64_t r = e - b * mn;
    const int i = (int)(r / N), j = (int)(r - (int64_t)i * N);
    if ((o.maskC == 1 && i < j) || (o.maskC == 2 && i > j))
        return;
    const T *p = partial + b * splits * mn + r;
    T s = T(0);
    for (int q = 0; q < splits; ++q)
        s += p[q * mn];
    store_c<T>(C.item(b), C.rs, C.cs, i, j, M, N, s, alpha, beta, o);
}

template <typename T>
static bool aligned16(const View<const T> &V, int64_t lead)
{
    constexpr int VW = Mfma<T>::VW;
    return (reinterpret_cast<uintptr_t>(V.p) & 15) == 0 && (lead % VW) == 0 && (V.bs % VW) == 0 && (V.bs2 % VW) == 0;
}

static inline int pick_order(const GemmOpts &o, int tiles_m, int tiles_n)
{
    if (o.maskC == 0 && o.triA == 0 && o.triB != 0)
        return 4;  // work depends on the column only
    if (o.symsum)
        return 1;
    if (tiles_m != tiles_n)
        return 0;
    if (o.maskC == 1 && o.triA == 1 && o.triB == 1 && tiles_m >= 16)
        return 5;
    if (o.maskC == 1 || o.maskC == 3)
        return 1;
    if (o.maskC == 2)
        return 2;
    return o.shells ? 3 : 0;
}

template <typename T, int BM, int BN, int BK, int NBUF, bool RAG>
static void launch_form(bool akf, bool bkf, View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int N,
                        int K, T alpha, T beta, GemmOpts o, hipStream_t st)
{
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    o.order = pick_order(o, tiles_m, tiles_n);
    const int64_t per = tile_count(o.order, tiles_m, tiles_n);
    o.xcd_batch = (batch >= 8 && per > 1) ? 1 : 0;
    const int64_t wgs = o.xcd_batch ? 8 * ((batch + 7) / 8) * per : per * batch;
    const dim3 grid((unsigned)wgs), block(256);
#define LA_GO(AK, BKF_, SYM_)                                                                                          \
    LA_LAUNCH((k_gemm<T, BM, BN, BK, NBUF, AK, BKF_, RAG, SYM_>), grid, block, 0, st, A, B, C, batch, M, N, K, alpha,  \
              beta, o, tiles_m, tiles_n)
    if constexpr (BM <= 64) {  // the symmetric sum exists for the small tiles only (launch_gemm picks them)
        if (o.symsum) {         // and its operands have mirrored strides, so akf == bkf
            if (akf)
                LA_GO(true, true, true);
            else
                LA_GO(false, false, true);
            return;
        }
    }
    if (akf && bkf)
        LA_GO(true, true, false);
    else if (akf && !bkf)
        LA_GO(true, false, false);
    else if (!akf && bkf)
        LA_GO(false, true, false);
    else
        LA_GO(false, false, false);
#undef LA_GO
}

struct GemmForm {
    bool akf, bkf;  // k is the contiguous index of A, of B
    bool rag;       // some chunk is unaligned or incomplete
};

template <typename T, int BM, int BN, int BK, int NBUF>
static void launch_tiles(GemmForm f, View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int N, int K,
                         T alpha, T beta, GemmOpts o, hipStream_t st)
{
    if (f.rag)
        launch_form<T, BM, BN, BK, NBUF, true>(f.akf, f.bkf, A, B, C, batch, M, N, K, alpha, beta, o, st);
    else
        launch_form<T, BM, BN, BK, NBUF, false>(f.akf, f.bkf, A, B, C, batch, M, N, K, alpha, beta, o, st);
}

static inline int flip_tri(int t) { return t == 1 ? 2 : (t == 2 ? 1 : 0); }

template <typename T>
la_status launch_gemm(View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int N, int K, T alpha, T beta,
                      GemmOpts o, hipStream_t st)
{
    if (batch <= 0 || M <= 0 || N <= 0)
        return LA_OK;
    if (o.symsum) {
        if (M != N || A.rs != B.cs || A.cs != B.rs || A.bs != B.bs || A.nb2 != 1 || B.nb2 != 1 || C.nb2 != 1)
            return LA_ERR_UNSUPPORTED;
        o.maskC = 0;
        o.halfDiag = 0;
        if (C.cs != 1 && beta != T(0))  // (the lower triangle that beta scales would be the upper one of C.t())
            return LA_ERR_UNSUPPORTED;
        if (C.cs != 1 && C.rs == 1)  // the result is symmetric: its transpose is the same matrix
            C = C.t();
    }
    // a few vectors on either side: one pass over the big operand
    if (!o.maskC && !o.halfDiag && !o.min_tile64 && !o.symsum && K > 0) {
        if (N <= GEMV_N && o.triB == 0)
            return launch_gemv<T>(A, B, C, batch, M, N, K, alpha, beta, o.triA, st);
        if (M <= GEMV_N && o.triA == 0)  // C^T = B^T A^T
            return launch_gemv<T>(B.t(), A.t(), C.t(), batch, N, M, K, alpha, beta, flip_tri(o.triB), st);
    }
    // Keep the stores of C along its contiguous direction: if C is stored with i contiguous,
    // compute C^T = B^T A^T instead (a pure re-labelling of the views).
    if (C.cs != 1 && C.rs == 1 && !o.symsum) {
        GemmOpts t;
        t.triA = flip_tri(o.triB);
        t.triB = flip_tri(o.triA);
        t.maskC = flip_tri(o.maskC);
        t.halfDiag = o.halfDiag;
        t.reverse = o.reverse;
        t.shells = o.shells;
        t.min_tile64 = o.min_tile64;
        t.split_if_room = o.split_if_room;
        return launch_gemm<T>(B.t(), A.t(), C.t(), batch, N, M, K, alpha, beta, t, st);
    }
    constexpr int VW = Mfma<T>::VW;
    GemmForm f;
    f.akf = (A.cs == 1);
    f.bkf = (B.rs == 1);
    if ((!f.akf && A.rs != 1) || (!f.bkf && B.cs != 1))
        return LA_ERR_UNSUPPORTED;  // (no operator of the library builds such a view)
    const bool a_ok = f.akf ? aligned16<T>(A, A.rs) : (aligned16<T>(A, A.cs) && M % VW == 0);
    const bool b_ok = f.bkf ? aligned16<T>(B, B.cs) : (aligned16<T>(B, B.rs) && N % VW == 0);
    f.rag = !(K % 16 == 0 && a_ok && b_ok);
    {
        const int64_t t64 = (int64_t)((M + 63) / 64) * ((N + 63) / 64) * batch;
        if (t64 > 0x1fffffffll)  // (quarter tiles and the batched mapping round the grid up)
            return LA_ERR_UNSUPPORTED;
        // Workgroups a launch would have with each tile size (empty tiles of triangular outputs
        // left out).
        auto wgs = [&](int e) {
            const int tm = (M + e - 1) / e, tn = (N + e - 1) / e;
            return tile_count(pick_order(o, tm, tn), tm, tn) * batch;
        };
        const int64_t wg128 = wgs(128), wg64 = wgs(64);
        // K slabs of 64: the whole range in such slabs, or (ragged) little of the last one empty
        const bool k64 = f.rag ? (K >= 128 || (K & 63) == 0 || (K & 63) > 32) : K % 64 == 0;
        // Quarter tiles exist with slabs of 64 only; aligned operands with another K take them in the ragged form, whose last slab ends where K
        // does and whose loads cost address arithmetic, instead of 64 x 64 tiles in slabs of 16.  Two things decide: how many tiles of 64 there
        // are, `work` (a last slab counts whole), against the 512 slots, and `share`, the quarter tiles' area as a part of theirs.  Gain, mean of
        // 2700 products of 128 <= K <= 2000, by work (300 to 420 / 420 to 520 / 520 to 640 / 640 to 720 / 720 to 820 / above):
        //   uniform, fp64, share above 1 (K far from the end of a slab) 1.07 / 0.88 / 0.90 / 0.79 / 0.76 / 0.79, 0.88 to 1 1.16 / 0.96 / 1.04 / 0.91 / 0.96 /
        //   0.88, 0.75 to 0.88 1.28 / 1.09 / 1.10 / 0.95 / 0.96 / 0.96, below 1.68 / 1.48 / 1.44 / 1.46 / 1.31 / 1.34;
        //   uniform, fp32, above 1 1.23 / 1.01 / 0.99 / 0.91 / 0.88 / 0.89, 0.88 to 1 1.29 / 1.08 / 1.11 / 1.03 / 1.00 / 1.01;
        //   triangular operands, fp64, above 1 1.35 / 1.23 / 1.09 / 1.10 / 1.01 / 0.94, 0.88 to 1 1.47 / 1.29 / 1.23 / 1.22 / 1.11 / 1.02; fp32, above 1
        //   1.63 / 1.46 / 1.26 / 1.18 / 1.08 / 1.07;
        //   symmetric results, fp64, above 1 1.13 / 1.05 / 1.07 / 1.03 / 0.94 / 0.92, 0.88 to 1 1.26 / 1.12 / 1.15 / 1.02 / 1.00 / 0.99, 0.75 to 0.88 1.37 /
        //   1.13 / 1.16 / 1.13 / 1.08 / 1.02; fp32, above 1 1.15 / 1.11 / 1.13 / 1.00 / 0.99 / 0.99.
        // Within 513 to 560 tiles the last round of 64 x 64 ones runs nearly empty (uniform, fp64, share 0.88 to 1: 1.09).  Up to K = 192 the last of two
        // or three slabs is too much of the work: share above 0.88, fp64 0.84 to 0.97, uniform, and 0.79 to 1.07, triangular
        // (0.83: 138 x 144^2 with 80 vectors 0.90).  Of the 2700, 47 are
        // 4 % or more slower than with tiles of 64, ten of them 10 to 22 % (7 x (720 x 300 x 1824) and 237 x (122 x 80 x 1200), fp32).
        const bool f32 = sizeof(T) == 4, tri = (o.triA | o.triB) != 0, uniform = !tri && !o.symsum;
        const double slabs = (double)((K + 63) / 64 * 64) / K, work = (double)wg64 * slabs;
        const double share = 0.25 * (double)wgs(32) / (double)wg64 * slabs;
        double most = f32 ? 1.0 : 0.875;  // share up to which the quarter tiles are taken
        if (work < (uniform && f32 ? 448.0 : 416.0))
            most = 2.0;
        else if (uniform)
            most = f32 || (wg64 > 512 && wg64 <= 560) ? 1.0 : (work < 640.0 ? 0.875 : 0.74);
        else if (work < 720.0)
            most = 1.05;
        else if (tri)
            most = f32 ? (work < 1100.0 ? 1.1 : 1.0) : 0.93;
        if (K <= 192 && work >= 400.0)
            most = std::min(most, 0.8);
        const bool quarters = k64 || (K >= 128 && share <= most);
        if (!o.triA && !o.triB && !o.min_tile64 && !o.ksplit && !o.symsum && wg64 <= 128 && K >= 2048 && A.nb2 == 1 && B.nb2 == 1 &&
            C.nb2 == 1) {
            int splits = (int)std::min<int64_t>(512 / wg64, K / 256);
            const int Kc = (((K + 15) / 16 + splits - 1) / splits) * 16;
            splits = (K + Kc - 1) / Kc;
            const size_t bytes = (size_t)batch * splits * M * N * sizeof(T);
            // (an unaligned or odd-sized product goes without the split where the caller gave no memory for it)
            if (splits >= 2 && bytes <= SPLITK_MAX_BYTES && ((!f.rag && !o.split_if_room) || arena_room(bytes))) {
                ArenaFrame frame;
                void *buf = nullptr;
                LA_TRY(arena_take(bytes, &buf));
                const int64_t mn = (int64_t)M * N;
                View<const T> As = A.level2((int64_t)Kc * A.cs, splits), Bs = B.level2((int64_t)Kc * B.rs, splits);
                View<T> Ps{(T *)buf, (int64_t)splits * mn, N, 1, mn, splits};
                GemmOpts ps;
                ps.maskC = o.maskC;  // tiles beyond the kept triangle are not computed (nor read back)
                ps.ksplit = splits;
                ps.ktotal = K;
                launch_tiles<T, 64, 64, 16, 2>(f, As, Bs, Ps, batch * splits, M, N, Kc, T(1), T(0), ps, st);
                LA_TRY(launch_check("gemm_splitk"));
                const int64_t total = batch * mn;
                LA_LAUNCH((k_splitk_reduce<T>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                                   (const T *)buf, C, batch, M, N, splits, alpha, beta, o);
                return launch_check("splitk_reduce");
            }
        }
        // No 128 x 128 tiles where they stick out of C by a quarter more than tiles of 64 do: 130 products of 129 x 129 x 129
        // 79 -> 41 us in fp64, 40 -> 22 in fp32, 64 of 320 x 320 x 320 146 -> 90 and 75 -> 47, 300 times trmm of 131 with 131
        // vectors 135 -> 68 and 73 -> 35; 383 x 383 (144 tiles against 180 quarters) is the same in both.
        const bool padded = (int64_t)((M + 127) / 128) * ((N + 127) / 128) * 16 > (int64_t)((M + 63) / 64) * ((N + 63) / 64) * 5;
        int e;
        if (o.triA | o.triB) {
            // Triangular operands make the K range, hence the time, of a tile vary along the tile
            // list (heaviest first): the 512 workgroup slots only fill evenly if there are several
            // rounds of tiles, so take the largest tile that still gives 1024 workgroups.
            e = wg128 >= 1024 && !padded ? 128 : ((wg64 >= 1024 || !quarters || o.min_tile64) ? 64 : 32);
        } else {
            // Equal tiles: big tiles once they (nearly) fill the 512 workgroup slots (496 tiles, 3952 x 2048 x 2000, fp64 598 -> 555
            // us and fp32 310 -> 296 against 64 x 64 tiles, 480 the same, 448 262 -> 291; a compute unit with one workgroup waits for
            // its loads: a sparse GP with 300 tiles of 128 1497 -> 1429 us in 64 x 64 tiles, factor + gradient of
            // n = 5500 with 432 of them 7737 -> 7511, fp64; 8192 with 192 to 256 of them in several products 16.84 -> 16.79 ms,
            // in fp32 10.07 -> 9.81), quarter tiles while 64 x 64 tiles
            // would fill the 512 workgroup slots less than twice -- with so few rounds the last one runs
            // part empty (32 x 384 x 384 lower triangle, K = 128: 672 tiles of 64, 38 -> 30 us; potrf of
            // 32 x 512 x 512 0.245 -> 0.231 ms, of 4 x 2048 x 2048 1.14 -> 1.10, 8192 x 8192 with 512
            // vectors trsm 1.19 -> 1.12 ms).  In fp64 nearly one big tile for each of the 256 compute units is as good as many
            // rounds, unless k is contiguous in both operands (us, 64 x 64 -> 128 x 128: 2048^3 355 -> 326 and with both k
            // contiguous 309 -> 338, 8192 x 512 x 1024 181 -> 167, 2304 x 1792 x 512, 252 tiles, 101 -> 88; 7168 x 512 x 1024, 224
            // tiles, 163 -> 168, 2048 x 1536 x 1024, 192 tiles, 144 -> 167; a batch of 13 x 512^3, 208 tiles, 98 -> 88).
            const int64_t t128 = o.maskC ? wg128 : (int64_t)((M + 127) / 128) * ((N + 127) / 128) * batch;
            // Up to K = 32 writing C is most of the work, and more, smaller workgroups overlap it with their loads (us, 128 x 128 ->
            // 64 x 64: 83 items of 1033 x 251, K = 2, fp64 48 -> 39, K = 32 72 -> 58, fp32 28 -> 25 and 37 -> 32; 64 x 512 x 512, K = 16,
            // 32 -> 30 and 22 -> 18; from K = 33 on it depends: 64 x 512 x 512 51 -> 64, 83 x 1033 x 251 89 -> 86).
            const bool big = K > 32 && (o.maskC ? (M >= 2048 && N >= 2048) : (M >= 128 && N >= 128));
            const bool one_round = sizeof(T) == 8 && !f.rag && !(f.akf && f.bkf) && !o.maskC && t128 <= 256 &&
                                   t128 > (batch > 1 ? 192 : 224);
            // Two nearly full rounds of 64 x 64 tiles are better than quarter tiles where the chunks are ragged, which costs address arithmetic
            // per load, and the quarters save no padding (b items of 61 x 174, K = 147, us, 32 x 32 -> 64 x 64: b = 331, 993 tiles, fp64
            // 60 -> 44, fp32 29 -> 22; with one round and a half the products of potri's backward rule, 30 x 297 x 297, 220 -> 232; 26 x 2478 x 22, 1014
            // tiles that the quarters halve, fp32 36 -> 54).
            const bool two_rounds = f.rag && !o.maskC && !o.symsum && wg64 >= 960 &&
                                    (int64_t)((M + 63) / 64) * ((N + 63) / 64) * 4 == (int64_t)((M + 31) / 32) * ((N + 31) / 32);
            e = ((t128 >= (o.maskC ? 512 : 480) || one_round) && big && !padded) ? 128 : ((wg64 < 1024 && quarters && !o.min_tile64 && !two_rounds) ? 32 : 64);
        }
        if (o.symsum && e == 128)  // (the form that stores both triangles has tiles up to 64 only)
            e = 64;
        if (e >= 64 && o.maskC == 1 && !o.triA && !o.triB && !o.halfDiag && !o.shells && !o.min_tile64 && M == N &&
            M % e == 0 && A.nb2 == 1 && B.nb2 == 1 && C.nb2 == 1) {
            // Lower triangle in e x e tiles: T (T + 1) / 2 of them.  When that is a few tiles more than
            // whole rounds of the 512 workgroup slots (T = 32: 528), the last round runs nearly empty.
            // The T diagonal tiles only need their lower halves anyway: take the T (T - 1) / 2 tiles
            // below the diagonal in one launch (whole tiles, no masking) and the diagonal blocks as a
            // batch of T small lower-triangle products.
            const int64_t Tt = M / e, per = Tt * (Tt + 1) / 2, spill = per % 512, below = (per - Tt) % 512;
            if (batch == 1 && per > 512 && spill > 0 && spill <= 64 && (below == 0 || below > 256)) {
                GemmOpts lo = o;
                lo.maskC = 3;  // tiles with tn <= tm of the view that starts e rows down, nothing masked inside
                View<const T> A1 = A.sub(e, 0);
                View<T> C1 = C.sub(e, 0);
                if (e == 128)
                    launch_tiles<T, 128, 128, 16, 2>(f, A1, B, C1, batch, M - e, N - e, K, alpha, beta, lo, st);
                else if (k64)
                    launch_tiles<T, 64, 64, 32, 1>(f, A1, B, C1, batch, M - e, N - e, K, alpha, beta, lo, st);
                else
                    launch_tiles<T, 64, 64, 16, 2>(f, A1, B, C1, batch, M - e, N - e, K, alpha, beta, lo, st);
                LA_TRY(launch_check("gemm"));
                return launch_gemm<T>(A.level2((int64_t)e * A.rs, (int)Tt), B.level2((int64_t)e * B.cs, (int)Tt),
                                      C.level2((int64_t)e * (C.rs + C.cs), (int)Tt), batch * Tt, e, e, K, alpha, beta, o, st);
            }
        }
        if (e == 32 && !k64)
            f.rag = true;
        if (e == 128)
            launch_tiles<T, 128, 128, 16, 2>(f, A, B, C, batch, M, N, K, alpha, beta, o, st);
        else if (e == 32)
            launch_tiles<T, 32, 32, 64, 1>(f, A, B, C, batch, M, N, K, alpha, beta, o, st);
        else if (k64)  // (slabs of 64 in one buffer hold two workgroups a compute unit, of 32 four: 32 matrices of
                       // n = 512, fp64, factor + gradient 593 -> 570 us; slabs of 16 in two buffers 590)
            launch_tiles<T, 64, 64, 32, 1>(f, A, B, C, batch, M, N, K, alpha, beta, o, st);
        else
            launch_tiles<T, 64, 64, 16, 2>(f, A, B, C, batch, M, N, K, alpha, beta, o, st);
        return launch_check("gemm");
    }
}

template la_status launch_gemm<float>(View<const float>, View<const float>, View<float>, int64_t, int, int, int, float,
                                      float, GemmOpts, hipStream_t);
template la_status launch_gemm<double>(View<const double>, View<const double>, View<double>, int64_t, int, int, int,
                                       double, double, GemmOpts, hipStream_t);

}  // namespace la
