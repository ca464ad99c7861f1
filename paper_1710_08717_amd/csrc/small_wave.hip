// Matrices of 16 < n <= 64: one wavefront per matrix, the whole operator in registers (trmm, syrk and the rules with them from n = 33 on).
//
// The one-workgroup kernels of leaf.hip give such a matrix four wavefronts and keep its 16 x 16 tiles in LDS; with nine or ten
// tiles they spend their time in barriers and in LDS round trips between products of one tile each.  Here a wavefront holds all tiles
// itself and never waits for another.  A tile is held as the matrix cores leave their accumulators (the COLS fragments of
// leaf_frag.hpp: lane (g, p) has the rows 4 v + g of column nat(p)), and that is the first operand of A^T B and the second of
// A B.  Every operator is therefore phrased in products  X^T Y  of tiles as they stand, some of them kept transposed; LDS
// only turns a tile where its transpose is wanted, too, or where memory runs the other way.
// What bounds them is registers: 56 to 210 with three tile rows, 76 to 250 with four, so 8 to 2 wavefronts per SIMD, and one only for
// k_potri_backward_wave and k_outer_wave with a triangle, fp64, four tile rows (364 to 367 of the 512 a wavefront can have), where nothing hides a load; the launch bounds
// ask for what each has.
#include "leaf_frag.hpp"

namespace la {

namespace {

constexpr int SW_WAVES = 4;  // matrices per workgroup

constexpr __host__ __device__ int tri_at(int i, int j) { return i * (i + 1) / 2 + j; }  // tile (i, j), i >= j

// One matrix in memory, R x C elements, any strides.
template <typename T>
struct Mat {
    T *p;
    unsigned rs, cs;
    int R, C;
    __device__ __forceinline__ Mat t() const { return Mat{p, cs, rs, C, R}; }
};

template <typename T>
struct Wave {
    static constexpr int PS = LT + 16 / (int)sizeof(T);  // row stride of a tile in LDS
    static constexpr int TILE = LT * PS;
    T *lds;  // one tile's room
    int r, g, c;  // natural row of the lane, lane group, nat(p)

    __device__ __forceinline__ Wave(T *l, int lane) : lds(l), r(lane & 15), g(lane >> 4), c(chain_nat<T>(lane & 15)) {}

    __device__ __forceinline__ void turn(const T (&x)[4], T (&y)[4]) const
    {
        wave_sync();
#pragma unroll
        for (int v = 0; v < 4; ++v)
            lds[(4 * v + g) * PS + c] = x[v];
        wave_sync();
#pragma unroll
        for (int v = 0; v < 4; ++v)
            y[v] = lds[c * PS + 4 * v + g];
    }
    // Element (4 v + g, c) of tile (i, j) as it lies in memory; beyond the matrix one of its other elements, until mask() makes it zero.
    // rin, cin: all rows, columns of the tile exist.
    template <typename M>
    __device__ __forceinline__ void raw(const Mat<M> &m, int i, int j, T (&x)[4], bool rin, bool cin) const
    {
        const int col = LT * j + c, cc = cin ? col : min(col, m.C - 1);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = LT * i + 4 * v + g, rr = rin ? row : min(row, m.R - 1);
            x[v] = *reinterpret_cast<const T *>(reinterpret_cast<const char *>(m.p) +
                                                ((unsigned)rr * m.rs + (unsigned)cc * m.cs) * (unsigned)sizeof(T));
        }
    }
    template <typename M>
    __device__ __forceinline__ void mask(const Mat<M> &m, int i, int j, T (&x)[4], bool rin, bool cin) const
    {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            x[v] = (rin || LT * i + 4 * v + g < m.R) && (cin || LT * j + c < m.C) ? x[v] : T(0);
    }
    template <typename M>
    __device__ __forceinline__ void load_direct(const Mat<M> &m, int i, int j, T (&x)[4], bool rin, bool cin) const
    {
        raw(m, i, j, x, rin, cin);
        mask(m, i, j, x, rin, cin);
    }
    __device__ __forceinline__ void store_direct(const Mat<T> &m, int i, int j, const T (&x)[4], bool rin, bool cin) const
    {
        const int col = LT * j + c;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = LT * i + 4 * v + g;
            if ((rin || row < m.R) && (cin || col < m.C))
                *reinterpret_cast<T *>(reinterpret_cast<char *>(m.p) + ((unsigned)row * m.rs + (unsigned)col * m.cs) * (unsigned)sizeof(T)) =
                    x[v];
        }
    }
    // the same along the direction in which the matrix is contiguous, in two steps: the elements on their way, and in place
    template <typename M>
    __device__ __forceinline__ void fetch(const Mat<M> &m, int i, int j, T (&x)[4], bool rin, bool cin) const
    {
        if (m.cs == 1 || m.rs != 1)
            raw(m, i, j, x, rin, cin);
        else
            raw(m.t(), j, i, x, cin, rin);
    }
    template <typename M>
    __device__ __forceinline__ void arrange(const Mat<M> &m, int i, int j, T (&in)[4], T (&x)[4], bool rin, bool cin) const
    {
        if (m.cs == 1 || m.rs != 1) {
            mask(m, i, j, in, rin, cin);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = in[v];
        } else {
            mask(m.t(), j, i, in, cin, rin);
            turn(in, x);
        }
    }
    template <typename M>
    __device__ __forceinline__ void load(const Mat<M> &m, int i, int j, T (&x)[4], bool rin, bool cin) const
    {
        T y[4];
        fetch(m, i, j, y, rin, cin);
        arrange(m, i, j, y, x, rin, cin);
    }
    __device__ __forceinline__ void store(const Mat<T> &m, int i, int j, const T (&x)[4], bool rin, bool cin) const
    {
        if (m.cs == 1 || m.rs != 1) {
            store_direct(m, i, j, x, rin, cin);
        } else {
            T y[4];
            turn(x, y);
            store_direct(m.t(), j, i, y, cin, rin);
        }
    }
    // lower triangle of a diagonal tile, `pad` on the diagonal beyond row n
    __device__ __forceinline__ void keep_lower(T (&x)[4], int i, int n, T pad) const
    {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 4 * v + g;
            x[v] = row < c ? T(0) : x[v];
            if (row == c && LT * i + row >= n)
                x[v] = pad;
        }
    }
    // tile (i, j) of a symmetric result and its mirror image
    __device__ __forceinline__ void store_sym(const Mat<T> &m, int i, int j, T (&x)[4], bool rin, bool cin) const
    {
        T y[4];
        turn(x, y);
        if (i == j) {  // both halves take the lower half's values: exactly symmetric
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = 4 * v + g < c ? y[v] : x[v];
            store_direct(m, i, i, x, rin, rin);
        } else {
            store_direct(m, i, j, x, rin, cin);
            store_direct(m, j, i, y, cin, rin);
        }
    }
    // inverse of a lower-triangular diagonal tile (zeros above the diagonal) and its transpose; in: the tile
    __device__ __forceinline__ void invert(const T (&l)[4], T (&li)[4], T (&lit)[4]) const
    {
        using V = typename Mfma<T>::vec_t;
        constexpr int VW = Mfma<T>::VW;
        wave_sync();
#pragma unroll
        for (int v = 0; v < 4; ++v)
            lds[(4 * v + g) * PS + c] = l[v];
        wave_sync();
        T a[LT], x[4];
        T *row = lds + r * PS;
#pragma unroll
        for (int q = 0; q < LT; q += VW) {
            const V w = *reinterpret_cast<const V *>(row + q);
            a[q] = w.x;
            a[q + 1] = w.y;
            if constexpr (VW == 4) {
                a[q + 2] = w.z;
                a[q + 3] = w.w;
            }
        }
        diag_invert<T>(a, row[r], x, r, g);
        wave_sync();
#pragma unroll
        for (int j = 0; j < 4; ++j)
            row[4 * j + g] = (4 * j + g <= r) ? x[j] : T(0);
        wave_sync();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            li[v] = lds[(4 * v + g) * PS + c];
            lit[v] = lds[c * PS + 4 * v + g];
        }
    }
};

template <typename T>
using Acc = typename Mfma<T>::acc_t;

template <typename T>
__device__ __forceinline__ void set(T (&x)[4], const Acc<T> &a)
{
#pragma unroll
    for (int v = 0; v < 4; ++v)
        x[v] = a[v];
}
template <typename T>
__device__ __forceinline__ void set_neg(T (&x)[4], const Acc<T> &a)
{
#pragma unroll
    for (int v = 0; v < 4; ++v)
        x[v] = -a[v];
}

// the matrix this wavefront works on
__device__ __forceinline__ int64_t my_item()
{
    return (int64_t)blockIdx.x * SW_WAVES + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}
template <typename T>
__device__ __forceinline__ Mat<T> item_of(const View<T> &v, int64_t b, int R, int C)
{
    return Mat<T>{v.p + b * v.bs, (unsigned)v.rs, (unsigned)v.cs, R, C};
}

// Lower-triangular factor: its tiles, the inverses of the diagonal ones and their transposes.
template <typename T, int K>
__device__ __forceinline__ void load_lower(const Wave<T> &w, const Mat<const T> &m, T pad, T (&l)[K * (K + 1) / 2][4])
{
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j)
            w.load(m, i, j, l[tri_at(i, j)], i < K - 1, j < K - 1);
#pragma unroll
    for (int i = 0; i < K; ++i)
        w.keep_lower(l[tri_at(i, i)], i, m.R, pad);
}

// Li = L^-1, tile by tile:  Li_ij = -Li_ii sum_{k = j..i-1} L_ik Li_kj
template <typename T, int K>
__device__ __forceinline__ void invert_lower(const Wave<T> &w, const T (&l)[K * (K + 1) / 2][4], T (&li)[K * (K + 1) / 2][4])
{
#pragma unroll
    for (int i = 0; i < K; ++i) {
        T lit[4];
        w.invert(l[tri_at(i, i)], li[tri_at(i, i)], lit);
        T lt[K][4];
#pragma unroll
        for (int k = 0; k < i; ++k)
            w.turn(l[tri_at(i, k)], lt[k]);
#pragma unroll
        for (int j = 0; j < i; ++j) {
            Acc<T> acc = {0, 0, 0, 0};
#pragma unroll
            for (int k = j; k < i; ++k)
                acc = frag_mma<T>(lt[k], li[tri_at(k, j)], acc);
            T s[4];
            set_neg<T>(s, acc);
            acc = Acc<T>{0, 0, 0, 0};
            acc = frag_mma<T>(lit, s, acc);
            set<T>(li[tri_at(i, j)], acc);
        }
    }
}

// all tiles of G + G^T
template <typename T, int K>
__device__ __forceinline__ void load_sym_sum(const Wave<T> &w, const Mat<const T> &m, T (&s)[K][K][4])
{
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j < K; ++j)
            w.load_direct(m, i, j, s[i][j], i < K - 1, j < K - 1);
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            T y[4];
            w.turn(s[j][i], y);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                s[i][j][v] += y[v];
            if (i != j)
                w.turn(s[i][j], s[j][i]);
        }
}

}  // namespace

// ---------------------------------------------------------------------------------------
// potrf.  The tiles above the diagonal, U_kj = L_jk^T:  U_kj = L_kk^-1 A_kj,  A_ij -= U_ki^T U_kj (k < i <= j).  chain_diag takes the
// diagonal tile as it stands in the accumulator and leaves the transpose of its inverse, which is what the next product takes.
// ---------------------------------------------------------------------------------------
template <typename T, int K>
__global__ __launch_bounds__(SW_WAVES * 64, sizeof(T) * K <= 16 ? 4 : 2) void k_potrf_wave(View<const T> A, View<T> L, int32_t *info,
                                                                                          int64_t batch, int n)
{
    using W = Wave<T>;
    __shared__ __align__(16) T lds[SW_WAVES][W::TILE];
    const int64_t b = my_item();
    if (b >= batch)
        return;
    const W w(lds[threadIdx.x >> 6], threadIdx.x & 63);
    const Mat<const T> Am = item_of<const T>(A, b, n, n);
    const Mat<T> Lm = item_of<T>(L, b, n, n);

    T u[K * (K + 1) / 2][4];  // tile (i, j) holds A_ij^T
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j)
            w.load(Am, i, j, u[tri_at(i, j)], i < K - 1, j < K - 1);
#pragma unroll
    for (int i = 0; i < K; ++i) {
#pragma unroll
        for (int j = 0; j < i; ++j)
            w.turn(u[tri_at(i, j)], u[tri_at(i, j)]);
        T y[4];
        T(&x)[4] = u[tri_at(i, i)];
        w.turn(x, y);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 4 * v + w.g;
            x[v] = row < w.c ? y[v] : x[v];
            if (row == w.c && LT * i + row >= n)
                x[v] = T(1);
        }
    }
    int fail = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        T d, x[4];
        wave_sync();
        const unsigned bad = chain_diag<T>(u[tri_at(k, k)], w.lds + w.c * W::PS, d, x, w.c, w.g);
        if (bad && fail == 0)
            fail = LT * k + first_row<T>(bad) + 1;
        const T rs = rsqrt_acc(d);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            x[v] *= rs;
        T dt[4];
        wave_sync();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const T e = w.lds[(4 * v + w.g) * W::PS + w.c] * rs;
            dt[v] = 4 * v + w.g < w.c ? T(0) : e;
        }
#pragma unroll
        for (int j = k + 1; j < K; ++j) {
            Acc<T> acc = {0, 0, 0, 0};
            acc = frag_mma<T>(x, u[tri_at(j, k)], acc);
            set<T>(u[tri_at(j, k)], acc);
        }
#pragma unroll
        for (int j = k + 1; j < K; ++j) {
            T nu[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                nu[v] = -u[tri_at(j, k)][v];
#pragma unroll
            for (int i = k + 1; i <= j; ++i) {
                T(&t)[4] = u[tri_at(j, i)];
                Acc<T> acc = {t[0], t[1], t[2], t[3]};
                acc = frag_mma<T>(u[tri_at(i, k)], nu, acc);
                set<T>(t, acc);
            }
        }
        w.store(Lm, k, k, dt, k < K - 1, k < K - 1);
    }
    const T zero[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j < i; ++j) {
            w.store(Lm.t(), j, i, u[tri_at(i, j)], true, i < K - 1);
            if (Lm.cs == 1 || Lm.rs != 1)
                w.store_direct(Lm, j, i, zero, true, i < K - 1);
            else
                w.store_direct(Lm.t(), i, j, zero, i < K - 1, true);
        }
    if (info != nullptr && (threadIdx.x & 63) == 0 && fail != 0 && fail <= n)
        if (info[b] == 0)
            info[b] = fail;
}

// ---------------------------------------------------------------------------------------
// potrf backward:  Abar = sym(L^-T Phi(L^T Lbar) L^-1).  P is formed transposed, so that Z = P Li and
// Abar_ij = 1/2 sum_{k >= i} (Li_ki^T Z_kj + Z_ki^T Li_kj) are products of tiles as they stand.
// ---------------------------------------------------------------------------------------
template <typename T, int K>
__global__ __launch_bounds__(SW_WAVES * 64, sizeof(T) * K <= 16 ? 4 : (sizeof(T) * K <= 24 ? 3 : 2)) void k_backward_wave(
    View<const T> Lam, View<const T> G, View<T> Abar, int64_t batch, int n)
{
    using W = Wave<T>;
    constexpr int NT = K * (K + 1) / 2;
    __shared__ __align__(16) T lds[SW_WAVES][W::TILE];
    const int64_t b = my_item();
    if (b >= batch)
        return;
    const W w(lds[threadIdx.x >> 6], threadIdx.x & 63);
    T l[NT][4], pt[NT][4], li[NT][4];
    {
        T gb[NT][4];
        load_lower<T, K>(w, item_of<const T>(Lam, b, n, n), T(1), l);
        load_lower<T, K>(w, item_of<const T>(G, b, n, n), T(0), gb);
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
            for (int k = 0; k <= i; ++k) {  // (P_ik)^T = sum_{q >= i} Lbar_qk^T L_qi
                Acc<T> acc = {0, 0, 0, 0};
#pragma unroll
                for (int q = i; q < K; ++q)
                    acc = frag_mma<T>(gb[tri_at(q, k)], l[tri_at(q, i)], acc);
                if (i == k) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = 4 * v + w.g;
                        acc[v] = row > w.c ? T(0) : (row == w.c ? T(0.5) * acc[v] : acc[v]);
                    }
                }
                set<T>(pt[tri_at(i, k)], acc);
            }
    }
    invert_lower<T, K>(w, l, li);
    T z[NT][4];
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            Acc<T> acc = {0, 0, 0, 0};
#pragma unroll
            for (int k = j; k <= i; ++k)
                acc = frag_mma<T>(pt[tri_at(i, k)], li[tri_at(k, j)], acc);
            set<T>(z[tri_at(i, j)], acc);
        }
    Mat<T> out = item_of<T>(Abar, b, n, n);
    if (out.rs == 1)  // symmetric: the transposed view is the same matrix
        out = out.t();
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            Acc<T> acc = {0, 0, 0, 0}, mirror = {0, 0, 0, 0};  // (two short sums: less rounding than one, and not one after the other)
#pragma unroll
            for (int k = i; k < K; ++k) {
                acc = frag_mma<T>(li[tri_at(k, i)], z[tri_at(k, j)], acc);
                mirror = frag_mma<T>(z[tri_at(k, i)], li[tri_at(k, j)], mirror);
            }
            T x[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = T(0.5) * (acc[v] + mirror[v]);
            w.store_sym(out, i, j, x, i < K - 1, j < K - 1);
        }
}

// ---------------------------------------------------------------------------------------
// potri:  B_ij = sum_{k >= i} Li_ki^T Li_kj
// ---------------------------------------------------------------------------------------
template <typename T, int K>
__global__ __launch_bounds__(SW_WAVES * 64, sizeof(T) * K <= 16 ? 4 : 2) void k_potri_wave(View<const T> Lam, View<T> B, int64_t batch,
                                                                                          int n)
{
    using W = Wave<T>;
    constexpr int NT = K * (K + 1) / 2;
    __shared__ __align__(16) T lds[SW_WAVES][W::TILE];
    const int64_t b = my_item();
    if (b >= batch)
        return;
    const W w(lds[threadIdx.x >> 6], threadIdx.x & 63);
    T l[NT][4], li[NT][4];
    load_lower<T, K>(w, item_of<const T>(Lam, b, n, n), T(1), l);
    invert_lower<T, K>(w, l, li);
    const Mat<T> out = item_of<T>(B, b, n, n);
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            Acc<T> acc = {0, 0, 0, 0};
#pragma unroll
            for (int k = i; k < K; ++k)
                acc = frag_mma<T>(li[tri_at(k, i)], li[tri_at(k, j)], acc);
            T x[4];
            set<T>(x, acc);
            w.store_sym(out, i, j, x, i < K - 1, j < K - 1);
        }
}

// ---------------------------------------------------------------------------------------
// trsm:  X = alpha t(L)^-1 B on any number of vectors, 16 at a time.
//   fwd:  X_k = L_kk^-1 (B_k - sum_{j < k} L_kj X_j);   otherwise  X_k = L_kk^-T (B_k - sum_{i > k} L_ik^T X_i)
// ---------------------------------------------------------------------------------------
template <typename T, int K, bool FWD>
__global__ __launch_bounds__(SW_WAVES * 64, sizeof(T) * K <= 16 ? 4 : 2) void k_trsm_wave(View<const T> Lam, View<const T> Xin, View<T> X,
                                                                                         int64_t batch, int n, int m, T alpha)
{
    using W = Wave<T>;
    constexpr int NT = K * (K + 1) / 2;
    __shared__ __align__(16) T lds[SW_WAVES][W::TILE];
    const int64_t b = my_item();
    if (b >= batch)
        return;
    const W w(lds[threadIdx.x >> 6], threadIdx.x & 63);
    T l[NT][4];  // below the diagonal L_ij^T (fwd) or L_ij, on it L_ii^-T or L_ii^-1
    load_lower<T, K>(w, item_of<const T>(Lam, b, n, n), T(1), l);
#pragma unroll
    for (int i = 0; i < K; ++i) {
        T li[4], lit[4];
        w.invert(l[tri_at(i, i)], li, lit);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            l[tri_at(i, i)][v] = FWD ? lit[v] : li[v];
        if constexpr (FWD)
#pragma unroll
            for (int j = 0; j < i; ++j)
                w.turn(l[tri_at(i, j)], l[tri_at(i, j)]);
    }
    const Mat<const T> in = item_of<const T>(Xin, b, n, m);
    const Mat<T> out = item_of<T>(X, b, n, m);
    T next[K][4];
#pragma unroll
    for (int k = 0; k < K; ++k)
        w.fetch(in, k, 0, next[k], k < K - 1, false);
    for (int ct = 0; ct * LT < m; ++ct) {
        T x[K][4];
#pragma unroll
        for (int k = 0; k < K; ++k)
            w.arrange(in, k, ct, next[k], x[k], k < K - 1, false);
        if ((ct + 1) * LT < m) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                w.fetch(in, k, ct + 1, next[k], k < K - 1, false);
        }
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int k = FWD ? q : K - 1 - q;
            Acc<T> acc = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < K; ++j)
                if (FWD ? j < k : j > k)
                    acc = frag_mma<T>(l[FWD ? tri_at(k, j) : tri_at(j, k)], x[j], acc);
            T s[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                s[v] = fma(alpha, x[k][v], -acc[v]);
            acc = Acc<T>{0, 0, 0, 0};
            acc = frag_mma<T>(l[tri_at(k, k)], s, acc);
            set<T>(x[k], acc);
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
            w.store(out, k, ct, x[k], k < K - 1, false);
    }
}

// ---------------------------------------------------------------------------------------
// potri backward:  with S = Bbar + Bbar^T and Q = L^-1 S B^T (lower; B for an upper factor) the result is minus the
// part of Q on and above its diagonal, transposed for a lower factor, and zeros.
// ---------------------------------------------------------------------------------------
template <typename T, int K>
__global__ __launch_bounds__(SW_WAVES * 64, sizeof(T) * K <= 12 ? 4 : (sizeof(T) * K <= 24 ? 2 : 1)) void k_potri_backward_wave(
    View<const T> Lam, View<const T> B, View<const T> Bbar, View<T> Lbar, int64_t batch, int n)
{
    using W = Wave<T>;
    constexpr int NT = K * (K + 1) / 2;
    __shared__ __align__(16) T lds[SW_WAVES][W::TILE];
    const int64_t b = my_item();
    if (b >= batch)
        return;
    const W w(lds[threadIdx.x >> 6], threadIdx.x & 63);
    T s[K][K][4];
    load_sym_sum<T, K>(w, item_of<const T>(Bbar, b, n, n), s);
    T l[NT][4];  // L_ij^T below the diagonal, L_ii^-T on it
    load_lower<T, K>(w, item_of<const T>(Lam, b, n, n), T(1), l);
#pragma unroll
    for (int i = 0; i < K; ++i) {
        T li[4], lit[4];
        w.invert(l[tri_at(i, i)], li, lit);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            l[tri_at(i, i)][v] = lit[v];
#pragma unroll
        for (int j = 0; j < i; ++j)
            w.turn(l[tri_at(i, j)], l[tri_at(i, j)]);
    }
    const Mat<const T> Bm = item_of<const T>(B, b, n, n);
    const Mat<T> out = item_of<T>(Lbar, b, n, n);
    const T zero[4] = {0, 0, 0, 0};
    T q[NT][4];  // tile (j, i), i <= j, holds Q_ij
#pragma unroll
    for (int j = 0; j < K; ++j) {
        T bt[K][4];
#pragma unroll
        for (int k = 0; k < K; ++k)
            w.load(Bm, k, j, bt[k], k < K - 1, j < K - 1);
#pragma unroll
        for (int i = 0; i <= j; ++i) {
            Acc<T> y = {0, 0, 0, 0}, acc = {0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < K; ++k)
                y = frag_mma<T>(s[k][i], bt[k], y);
#pragma unroll
            for (int k = 0; k < i; ++k)
                acc = frag_mma<T>(l[tri_at(i, k)], q[tri_at(j, k)], acc);
            T e[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                e[v] = y[v] - acc[v];
            acc = Acc<T>{0, 0, 0, 0};
            acc = frag_mma<T>(l[tri_at(i, i)], e, acc);
            set<T>(q[tri_at(j, i)], acc);
        }
    }
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
        for (int i = 0; i <= j; ++i) {
            T e[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                e[v] = i == j && 4 * v + w.g > w.c ? T(0) : -q[tri_at(j, i)][v];
            w.store(out, i, j, e, i < K - 1, j < K - 1);
            if (i != j) {
                if (out.cs == 1)
                    w.store_direct(out, j, i, zero, j < K - 1, true);
                else
                    w.store_direct(out.t(), i, j, zero, true, j < K - 1);
            }
        }
}

// ---------------------------------------------------------------------------------------
// Products of small matrices:  trmm  X = alpha t(L) B,  16 vectors at a time;  the rule of syrk  Out = alpha (G + G^T) A,  16 columns
// at a time;  U V^T with its triangles treated as in k_outer_leaf16.
// ---------------------------------------------------------------------------------------
template <typename T, int K, bool FWD>
__global__ __launch_bounds__(SW_WAVES * 64, sizeof(T) * K <= 16 ? 4 : 2) void k_trmm_wave(View<const T> Lam, View<const T> Xin, View<T> X,
                                                                                         int64_t batch, int n, int m, T alpha)
{
    using W = Wave<T>;
    constexpr int NT = K * (K + 1) / 2;
    __shared__ __align__(16) T lds[SW_WAVES][W::TILE];
    const int64_t b = my_item();
    if (b >= batch)
        return;
    const W w(lds[threadIdx.x >> 6], threadIdx.x & 63);
    const Mat<const T> in = item_of<const T>(Xin, b, n, m);
    const Mat<T> out = item_of<T>(X, b, n, m);
    T l[NT][4], next[K][4];  // L_ij^T (fwd) or L_ij
    load_lower<T, K>(w, item_of<const T>(Lam, b, n, n), T(0), l);
#pragma unroll
    for (int k = 0; k < K; ++k)
        w.fetch(in, k, 0, next[k], k < K - 1, false);
    if constexpr (FWD)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            w.turn(l[t], l[t]);
    for (int ct = 0; ct * LT < m; ++ct) {
        T x[K][4];
#pragma unroll
        for (int k = 0; k < K; ++k)
            w.arrange(in, k, ct, next[k], x[k], k < K - 1, false);
        if ((ct + 1) * LT < m) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                w.fetch(in, k, ct + 1, next[k], k < K - 1, false);
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            Acc<T> acc = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < K; ++j)
                if (FWD ? j <= i : j >= i)
                    acc = frag_mma<T>(l[FWD ? tri_at(i, j) : tri_at(j, i)], x[j], acc);
            T y[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                y[v] = alpha * acc[v];
            w.store(out, i, ct, y, i < K - 1, false);
        }
    }
}

template <typename T, int K>
__global__ __launch_bounds__(SW_WAVES * 64, sizeof(T) * K <= 12 ? 4 : 2) void k_symm_wave(View<const T> G, View<const T> A, View<T> Out,
                                                                                         int64_t batch, int n, int k, T alpha)
{
    using W = Wave<T>;
    __shared__ __align__(16) T lds[SW_WAVES][W::TILE];
    const int64_t b = my_item();
    if (b >= batch)
        return;
    const W w(lds[threadIdx.x >> 6], threadIdx.x & 63);
    const Mat<const T> in = item_of<const T>(A, b, n, k);
    const Mat<T> out = item_of<T>(Out, b, n, k);
    T s[K][K][4], next[K][4];
    load_sym_sum<T, K>(w, item_of<const T>(G, b, n, n), s);
#pragma unroll
    for (int q = 0; q < K; ++q)
        w.fetch(in, q, 0, next[q], q < K - 1, false);
    for (int ct = 0; ct * LT < k; ++ct) {
        T x[K][4];
#pragma unroll
        for (int q = 0; q < K; ++q)
            w.arrange(in, q, ct, next[q], x[q], q < K - 1, false);
        if ((ct + 1) * LT < k) {
#pragma unroll
            for (int q = 0; q < K; ++q)
                w.fetch(in, q, ct + 1, next[q], q < K - 1, false);
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            Acc<T> acc = {0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < K; ++q)
                acc = frag_mma<T>(s[q][i], x[q], acc);
            T y[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                y[v] = alpha * acc[v];
            w.store(out, i, ct, y, i < K - 1, false);
        }
    }
}

template <typename T, int K, int TRI>
__global__ __launch_bounds__(SW_WAVES * 64, TRI != 0 ? (sizeof(T) * K <= 12 ? 3 : (sizeof(T) * K <= 24 ? 2 : 1)) : (sizeof(T) * K <= 16 ? 4 : 2)) void k_outer_wave(View<const T> U, View<const T> V, View<T> Cv,
                                                                                          int64_t batch, int n, int k, T alpha)
{
    using W = Wave<T>;
    constexpr int NT = K * (K + 1) / 2;
    __shared__ __align__(16) T lds[SW_WAVES][W::TILE];
    const int64_t b = my_item();
    if (b >= batch)
        return;
    const W w(lds[threadIdx.x >> 6], threadIdx.x & 63);
    const Mat<const T> um = item_of<const T>(U, b, n, k).t(), vm = item_of<const T>(V, b, n, k).t();
    T nu[K][4], nv[TRI ? K : 1][4];
    Acc<T> acc[NT];  // tile (i, j) of C on or below the diagonal; with TRI 2 the transpose of tile (j, i)
#pragma unroll
    for (int t = 0; t < NT; ++t)
        acc[t] = Acc<T>{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < K; ++i) {
        w.fetch(um, 0, i, nu[i], false, i < K - 1);
        if constexpr (TRI != 0)
            w.fetch(vm, 0, i, nv[i], false, i < K - 1);
    }
    for (int kk = 0; kk * LT < k; ++kk) {
        T u[K][4], v[TRI ? K : 1][4];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            w.arrange(um, kk, i, nu[i], u[i], false, i < K - 1);
            if constexpr (TRI != 0)
                w.arrange(vm, kk, i, nv[i], v[i], false, i < K - 1);
        }
        if ((kk + 1) * LT < k) {
#pragma unroll
            for (int i = 0; i < K; ++i) {
                w.fetch(um, kk + 1, i, nu[i], false, i < K - 1);
                if constexpr (TRI != 0)
                    w.fetch(vm, kk + 1, i, nv[i], false, i < K - 1);
            }
        }
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j) {
                if constexpr (TRI == 0)
                    acc[tri_at(i, j)] = frag_mma<T>(u[i], u[j], acc[tri_at(i, j)]);
                else if constexpr (TRI == 1)
                    acc[tri_at(i, j)] = frag_mma<T>(u[i], v[j], acc[tri_at(i, j)]);
                else  // tile (j, i)
                    acc[tri_at(i, j)] = frag_mma<T>(u[j], v[i], acc[tri_at(i, j)]);
            }
    }
    const Mat<T> out = item_of<T>(Cv, b, n, n);
    const T zero[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            T x[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = alpha * acc[tri_at(i, j)][v];
            if constexpr (TRI == 0) {
                w.store_sym(out, i, j, x, i < K - 1, j < K - 1);
            } else {
                if (i == j) {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        x[v] = (TRI == 1 ? 4 * v + w.g < w.c : 4 * v + w.g > w.c) ? T(0) : x[v];
                }
                w.store_direct(out, TRI == 1 ? i : j, TRI == 1 ? j : i, x, (TRI == 1 ? i : j) < K - 1, (TRI == 1 ? j : i) < K - 1);
                if (i != j)
                    w.store_direct(out, TRI == 1 ? j : i, TRI == 1 ? i : j, zero, (TRI == 1 ? j : i) < K - 1, (TRI == 1 ? i : j) < K - 1);
            }
        }
}

// ---------------------------------------------------------------------------------------
// launches: two, three or four tile rows
// ---------------------------------------------------------------------------------------
// Products (trmm, syrk and the rules with them): one wavefront alone takes longer than the four or sixteen of the other kernels, which two rounds of
// workgroups a compute unit make up for, one round for less than three whole tile rows and few columns.  300 / 640 / 1024 matrices from memory, time of the
// other kernels over this one's: syrk of n = 33 with k = 24 1.19 / 1.56 / 1.91 in fp32 and 1.16 / 1.50 / 1.72 in fp64, of n = 64 with k = 64 0.99 / 1.29 /
// 1.54 and 0.87 / 1.22 / 1.34, its rule 1.03 / 1.42 / 1.77, 1.12 / 1.46 / 1.65 and 0.93 / 1.29 / 1.43, 1.08 / 1.41 / 1.67; with 128 matrices 0.6 to 1.1.
static bool wave_range(int64_t batch, int n, int cols)
{
    return n > 2 * LT && n <= 4 * LT && batch <= 0x7fffffffll &&
           (batch > 1024 || (cols <= 4 * LT && batch > (n < 3 * LT && cols <= 3 * LT ? 256 : 512)));
}
// the kernels address an item by 32-bit byte offsets
template <typename T>
static bool offsets_fit(int64_t rows, int64_t cols, int64_t rs, int64_t cs, int nb2)
{
    return nb2 == 1 && rs >= 0 && cs >= 0 && ((rows - 1) * rs + (cols - 1) * cs + 1) * (int64_t)sizeof(T) <= 0xffffffffll;
}

// Up to 1024 matrices (us from memory, other kernel -> this one, fp32 and fp64):
//   potrf, 64 matrices of n = 20 12.8 -> 4.4 and 13.6 -> 5.3, of 32 5.8 -> 4.5 and 7.3 -> 5.3, 256 of 33 32 -> 6.7 and 40 -> 8.3, of 49 24.7 -> 9.5 and
//     31.8 -> 12.2, 1024 of 64 20.8 -> 12.3 and 33.5 -> 17.8;
//   backward, 64 of 20 10 -> 5.0 and 10.8 -> 6.4, 1024 of 32 16.0 -> 6.6 and 19.6 -> 9.4, 300 of 41 17.6 -> 8.3 and 20.6 -> 13.2, of 64 16.1 -> 14.3 and
//     22.1 -> 21.9, but 128 of 64 11.0 -> 13.1 and 13.5 -> 19.5, of 48 8.6 -> 8.3 and 10.2 -> 12.0;
//   potri alike (128 of 33 7.4 -> 5.5 and 8.2 -> 7.1, of 64 7.4 -> 8.3 and 8.7 -> 11.1), its rule always (64 of 20 11.7 -> 5.1 and 12.2 -> 6.5,
//     256 of 49 39 -> 16 and 53 -> 21).
// More of them, up to n = 32: the lane-group kernels are ahead where they keep just n columns and take 16-byte pieces (n = 24 and 32): 8192 potrf of
// n = 32 in fp32 11.8 -> 16.9, of 24 8.7 -> 14.2 and 15.3 -> 22.4 (but 31.0 -> 25.5 of n = 32 in fp64), backward of 24 17.4 -> 21.0 and 31.7 -> 38.0, of 32
// 28 -> 26 and 75 -> 43, of 28 41 -> 23 and 94 -> 42; potri of 24 10.8 -> 13.1 and 18.1 -> 20.2, of 32 16.0 -> 15.0 and 33 -> 24; its rule, of 28, 82 -> 27
// and 98 -> 45.
// Above n = 32, against the four-wavefront kernels:
//   12255 of n = 37: potrf 88 -> 41 / 140 -> 69, backward 142 -> 77 / 214 -> 162, potri 73 -> 39 / 96 -> 65, its backward rule
//   207 -> 99 / 370 -> 288; 5001 of n = 51: 55 -> 32 / 83 -> 56, 109 -> 68 / 205 -> 154, 52 -> 32 / 118 -> 66, 311 -> 135 / 575 -> 347;
//   1100 of n = 64: 17 -> 15 / 29 -> 22, 35 -> 25 / 48 -> 39, 18 -> 15 / 29 -> 22.
// Where nothing is ragged the four-wavefront kernels move
// 16-byte pieces, and from memory (not the last-level cache) they are then the faster ones: 16384 of n = 64, fp32, potrf 141 -> 180,
// 4096 37 -> 30; 20000 of n = 48 109 -> 120, 7281 42 -> 33; backward 7281 of n = 48, fp64, 121 -> 138, 2048 39 -> 34.
// potrf in fp64 with four tile rows is equal there: 8000 of n = 60 133 -> 142, 5001 of n = 51 83 -> 56; so is potri with nearly three whole
// ones: 24618 of n = 47 202 -> 231, 12169 102 -> 110, 9000 to 11000 (160 MiB) 1.04 to 1.2 times as fast.
template <typename T>
bool small_wave_takes(SmallWaveOp op, int64_t batch, int n)
{
    if (n <= LT || n > 4 * LT || batch > 0x7fffffffll)
        return false;
    if (op == SmallWaveOp::potri_backward)
        return true;
    if (n <= 2 * LT) {
        if (op == SmallWaveOp::potrf)
            return n % 8 != 0 || batch <= 1024 || (sizeof(T) == 8 && n == 32 && batch >= 4096);
        return n != 24 || batch <= 2048;
    }
    if (batch <= 1024)
        return op == SmallWaveOp::potrf || batch > 256 || n < (sizeof(T) == 4 ? 4 : 3) * LT;
    const double mib = (double)batch * n * n * sizeof(T) / 1048576.0;
    if (n % LT == 0)
        return mib <= 64.0;
    if (sizeof(T) == 4)
        return true;
    return !(op == SmallWaveOp::potrf && n > 3 * LT && mib > 128.0) && !(op == SmallWaveOp::potri && n > 44 && n < 3 * LT && mib > 192.0);
}
template bool small_wave_takes<float>(SmallWaveOp, int64_t, int);
template bool small_wave_takes<double>(SmallWaveOp, int64_t, int);

// any batch: what is not ahead of the paths with scratch stands in for them where there is none
template <typename T>
bool tri_wave_can(int64_t batch, int n, int m, const View<const T> &in, const View<T> &out)
{
    return n > LT && n <= 4 * LT && m >= 1 && batch <= 0x7fffffffll && offsets_fit<T>(n, m, in.rs, in.cs, in.nb2) &&
           offsets_fit<T>(n, m, out.rs, out.cs, out.nb2);
}
template bool tri_wave_can<float>(int64_t, int, int, const View<const float> &, const View<float> &);
template bool tri_wave_can<double>(int64_t, int, int, const View<const double> &, const View<double> &);

// Up to n = 32 against one workgroup an item (up to 48 vectors, and 16 lanes an item for up to 16 vectors of many), the inverse and a product above
// (time of the other over this one's, fp32 and fp64): 64 of n = 20 with 16 vectors 1.6 and 1.5, with 48 1.2 and 1.06, with 64 2.1 and 1.9, with 128 1.5 and
// 1.3, 8192 1.8 and 2.3, 1.9 and 2.0, 5.7 and 6.3, 4.1 and 4.3; behind are 64 of n = 32 with 48 (0.97 and 0.87) and 8192 of n = 24 with one vector in fp32 (0.90).
// Above n = 32 and up to 256 items the sixteen wavefronts of one workgroup are ahead where there is a wavefront's work for each and little padding: 128 items
// of n = 33, 48, 56, 64 with 16 vectors 1.39, 1.14, 1.25, 1.07 and 1.25, 1.03, 1.08, 0.92, with 24 1.18, 1.02, 1.09, 0.94 and 1.03, 0.90, 0.92, 0.84, with 48
// 1.04, 0.90, 1.01, 0.88 and 0.92, 0.82, 0.88, 0.81; so is the inverse for many vectors: with 64 1.95, 1.51, 1.44, 1.27 and 1.83, 1.43, 1.32, 1.22, with 128
// 1.36, 1.10, 0.99, 0.88 and 1.18, 0.92, 0.89, 0.85.  300 items: 1.11 (n = 64 with 48, fp32) to 2.6; 3000 of n = 41 to 64 with up to 48 1.3 to 3.3.
// 5001 of n = 51 with 51 vectors 167 -> 81 / 317 -> 167.  Above 3072, up to 48 vectors, the workgroup gives every tile of vectors a wavefront
// of its own: 9000 of n = 45 with 45 vectors, fp32, 70 -> 79 (with 16
// 46 -> 36; of n = 40 with 40 75 -> 66), 8000 of n = 60 with 16, fp64, 93 -> 133.  Many vectors of few items are left to the product, too (fp32: 1500 of
// n = 60 with 1000 468 -> 663, 1100 of n = 64 with 200 83 -> 96; 4096 of n = 64 with 300 437 -> 336).
template <typename T>
bool trsm_wave_takes(int64_t batch, int n, int m, const View<const T> &in, const View<T> &out)
{
    constexpr bool f32 = sizeof(T) == 4;
    if (!tri_wave_can<T>(batch, n, m, in, out))
        return false;
    if (m > 8 * LT)
        return batch > 3072;
    if (n <= 2 * LT)
        return !(batch <= 256 && n == 2 * LT && m > 2 * LT && m <= 3 * LT) && !(f32 && batch > 4096 && n == 24 && m < 8);
    if (batch > 3072)
        return m > 3 * LT || !(n >= 3 * LT || (n > 40 && m > LT));
    if (batch > 256)
        return true;
    if (m <= LT)
        return f32 || n <= 60;
    if (m <= 3 * LT)
        return f32 ? n < (m <= 2 * LT ? 64 : 45) : (m <= 2 * LT && n < 45);
    return m <= 5 * LT || n < 45;
}
template bool trsm_wave_takes<float>(int64_t, int, int, const View<const float> &, const View<float> &);
template bool trsm_wave_takes<double>(int64_t, int, int, const View<const double> &, const View<double> &);

// Against one workgroup per matrix or the general product, us, fp32 / fp64, 12255 of n = 37: trmm of 16 vectors 52 -> 23 / 61 -> 38, of 40
// 81 -> 46 / 123 -> 94; 16384 of n = 64 75 -> 66 / 111 -> 110.  The general product wins where it fills its tiles: 5000 of n = 48 with
// 300 vectors, fp32, 202 -> 258, 1100 of n = 64 in fp64 105 -> 128 (5000 of n = 61 630 -> 514).
template <typename T>
bool trmm_wave_takes(int64_t batch, int n, int m, const View<const T> &in, const View<T> &out)
{
    if (!tri_wave_can<T>(batch, n, m, in, out) || n <= 2 * LT)
        return false;
    // (below 64 items there is no one-workgroup kernel: 4 of n = 33 with 8 vectors, fp32, 12.1 -> 4.0, of n = 64 with 16, fp64, 15.7 -> 6.3)
    if (batch < 64)
        return m <= LT;
    if (!wave_range(batch, n, m))
        return false;
    // (640 of n = 56 with 24, 48, 64 vectors 0.97, 0.95, 0.83 times as fast in fp64, of n = 41 1.49, 1.35, 1.74)
    if (sizeof(T) == 8 && batch <= 1024 && n >= 3 * LT && m > LT)
        return false;
    // 33 to 47 vectors side by side, in rows of no whole 64 bytes, from memory, fp64: the one-workgroup kernel is the faster one (10463 of n = 44
    // with 47 120 -> 150, 23423 of n = 46 with 41 241 -> 317, 24411 of n = 39 with 47 246 -> 294; 3956 of n = 46 with 45, 64 MiB, 46 -> 42, 11077 of
    // n = 46 with 40 120 -> 113, 44560 of n = 34 with 37 412 -> 366, as rows of n 20618 of n = 42 with 45 215 -> 178)
    if (sizeof(T) == 8 && in.cs == 1 && n > (m > 40 ? 36 : 41) && n <= 3 * LT && m > 2 * LT && m < 3 * LT && m % 8 != 0 &&
        (double)batch * n * n * sizeof(T) > 128.0 * 1048576.0)
        return false;
    return m <= 4 * LT || (sizeof(T) == 8 && (n <= 3 * LT || batch > 3072));
}
template bool trmm_wave_takes<float>(int64_t, int, int, const View<const float> &, const View<float> &);
template bool trmm_wave_takes<double>(int64_t, int, int, const View<const double> &, const View<double> &);

// syrk and its rule, any k: 12255 of n = 37 with k = 32 syrk 51 -> 28 / 67 -> 44, its rule 66 -> 37 / 115 -> 71, with k = 64 66 -> 38 /
// 129 -> 79 and 130 -> 81 / 188 -> 117; 5000 of n = 61 with k = 300 184 -> 128 / 377 -> 243 and 683 -> 340 / 1425 -> 524.
bool syrk_wave_takes(int64_t batch, int n, int k) { return wave_range(batch, n, k) && k >= 1; }

// The gradients of triangular operands, U V^T with one triangle kept: the rule of trmm on 12255 of n = 37 with 16 vectors 97 -> 46 /
// 128 -> 96, with 40 205 -> 100 / 345 -> 181.  With four tile rows the ten sums leave few wavefronts on a compute unit: 8000 of n = 60
// with 16 vectors, fp64, 79 -> 102 for this product alone (40 vectors: 181 -> 132), 1100 of n = 64 with 300 44 -> 56 / 74 -> 120.
template <typename T>
bool outer_wave_takes(int64_t batch, int n, int m)
{
    if (!wave_range(batch, n, m) || m < 1)
        return false;
    if (n <= 3 * LT)
        return true;
    return (sizeof(T) == 4 || m > LT) && (m <= 4 * LT || (m <= 32 * LT && batch > 3072));
}
template bool outer_wave_takes<float>(int64_t, int, int);
template bool outer_wave_takes<double>(int64_t, int, int);

#define LA_GO_WAVE_FROM(K0, KERNEL, ...)                                                                                          \
    do {                                                                                                                         \
        const dim3 grid((unsigned)((batch + SW_WAVES - 1) / SW_WAVES)), block(SW_WAVES * 64);                                    \
        if (n <= 2 * LT)                                                                                                         \
            LA_LAUNCH((KERNEL(K0)), grid, block, 0, st, __VA_ARGS__);                                                            \
        else if (n <= 3 * LT)                                                                                                    \
            LA_LAUNCH((KERNEL(3)), grid, block, 0, st, __VA_ARGS__);                                                             \
        else                                                                                                                     \
            LA_LAUNCH((KERNEL(4)), grid, block, 0, st, __VA_ARGS__);                                                             \
    } while (0)
#define LA_GO_WAVE(KERNEL, ...) LA_GO_WAVE_FROM(2, KERNEL, __VA_ARGS__)
#define LA_GO_WAVE_33(KERNEL, ...) LA_GO_WAVE_FROM(3, KERNEL, __VA_ARGS__)  // (n > 32)

template <typename T>
la_status launch_potrf_wave(View<const T> A, View<T> L, int32_t *info, int64_t batch, int n, hipStream_t st)
{
#define LA_K(K_) k_potrf_wave<T, K_>
    LA_GO_WAVE(LA_K, A, L, info, batch, n);
#undef LA_K
    return launch_check("potrf_wave");
}
template <typename T>
la_status launch_backward_wave(View<const T> Lam, View<const T> G, View<T> Abar, int64_t batch, int n, hipStream_t st)
{
#define LA_K(K_) k_backward_wave<T, K_>
    LA_GO_WAVE(LA_K, Lam, G, Abar, batch, n);
#undef LA_K
    return launch_check("backward_wave");
}
template <typename T>
la_status launch_potri_wave(View<const T> Lam, View<T> B, int64_t batch, int n, hipStream_t st)
{
#define LA_K(K_) k_potri_wave<T, K_>
    LA_GO_WAVE(LA_K, Lam, B, batch, n);
#undef LA_K
    return launch_check("potri_wave");
}
template <typename T>
la_status launch_trsm_wave(View<const T> Lam, View<const T> Xin, View<T> X, int64_t batch, int n, int m, T alpha, bool fwd, hipStream_t st)
{
#define LA_K(K_) k_trsm_wave<T, K_, true>
#define LA_K2(K_) k_trsm_wave<T, K_, false>
    if (fwd)
        LA_GO_WAVE(LA_K, Lam, Xin, X, batch, n, m, alpha);
    else
        LA_GO_WAVE(LA_K2, Lam, Xin, X, batch, n, m, alpha);
#undef LA_K
#undef LA_K2
    return launch_check("trsm_wave");
}
// lower: B as it is stored is B^T of what the kernel multiplies by, and the result is written transposed
template <typename T>
la_status launch_potri_backward_wave(View<const T> Lam, View<const T> B, View<const T> Bbar, View<T> Lbar, int64_t batch, int n,
                                     hipStream_t st)
{
#define LA_K(K_) k_potri_backward_wave<T, K_>
    LA_GO_WAVE(LA_K, Lam, B, Bbar, Lbar, batch, n);
#undef LA_K
    return launch_check("potri_backward_wave");
}
template <typename T>
la_status launch_trmm_wave(View<const T> Lam, View<const T> Xin, View<T> X, int64_t batch, int n, int m, T alpha, bool fwd, hipStream_t st)
{
#define LA_K(K_) k_trmm_wave<T, K_, true>
#define LA_K2(K_) k_trmm_wave<T, K_, false>
    if (fwd)
        LA_GO_WAVE_33(LA_K, Lam, Xin, X, batch, n, m, alpha);
    else
        LA_GO_WAVE_33(LA_K2, Lam, Xin, X, batch, n, m, alpha);
#undef LA_K
#undef LA_K2
    return launch_check("trmm_wave");
}
template <typename T>
la_status launch_symm_wave(T alpha, int64_t batch, int n, int k, View<const T> G, View<const T> A, View<T> Out, hipStream_t st)
{
#define LA_K(K_) k_symm_wave<T, K_>
    LA_GO_WAVE_33(LA_K, G, A, Out, batch, n, k, alpha);
#undef LA_K
    return launch_check("symm_wave");
}
template <typename T>
la_status launch_outer_wave(int tri, T alpha, int64_t batch, int n, int k, View<const T> U, View<const T> V, View<T> C, hipStream_t st)
{
#define LA_K0(K_) k_outer_wave<T, K_, 0>
#define LA_K1(K_) k_outer_wave<T, K_, 1>
#define LA_K2(K_) k_outer_wave<T, K_, 2>
    if (tri == 0)
        LA_GO_WAVE_33(LA_K0, U, V, C, batch, n, k, alpha);
    else if (tri == 1)
        LA_GO_WAVE_33(LA_K1, U, V, C, batch, n, k, alpha);
    else
        LA_GO_WAVE_33(LA_K2, U, V, C, batch, n, k, alpha);
#undef LA_K0
#undef LA_K1
#undef LA_K2
    return launch_check("outer_wave");
}
#define LA_INST(T)                                                                                                               \
    template la_status launch_potrf_wave<T>(View<const T>, View<T>, int32_t *, int64_t, int, hipStream_t);                       \
    template la_status launch_backward_wave<T>(View<const T>, View<const T>, View<T>, int64_t, int, hipStream_t);                \
    template la_status launch_potri_wave<T>(View<const T>, View<T>, int64_t, int, hipStream_t);                                  \
    template la_status launch_trsm_wave<T>(View<const T>, View<const T>, View<T>, int64_t, int, int, T, bool, hipStream_t);      \
    template la_status launch_potri_backward_wave<T>(View<const T>, View<const T>, View<const T>, View<T>, int64_t, int,         \
                                                     hipStream_t);                                                               \
    template la_status launch_trmm_wave<T>(View<const T>, View<const T>, View<T>, int64_t, int, int, T, bool, hipStream_t);      \
    template la_status launch_symm_wave<T>(T, int64_t, int, int, View<const T>, View<const T>, View<T>, hipStream_t);            \
    template la_status launch_outer_wave<T>(int, T, int64_t, int, int, View<const T>, View<const T>, View<T>, hipStream_t);
LA_INST(float)
LA_INST(double)
#undef LA_INST

}  // namespace la
