// The factorisation loop of the one-workgroup kernels (leaf.hip): one block of up to 128 rows, factored and inverted as
// 16 x 16 tiles whose LDS image is the matrix cores' operand order.
#pragma once
#include "leaf_dpp.hpp"

#ifndef LEAF16_STAMP
#define LEAF16_STAMP(i)
#endif

namespace la {

// ---------------------------------------------------------------------------------------
// Tiles as fragments.  Lane (g, p) (g = lane / 16, p = lane % 16) holds four elements v = 0 .. 3 of a tile: of row nat(p) the columns
// 4 v + g (ROWS), or of column nat(p) the rows 4 v + g (COLS), nat = chain_nat.  Contracting index 4 s + g in instruction s,
//   ROWS is either operand of  A B^T  (lane = row of its tile),
//   COLS is the second operand of  A B,  and the first of  A^T B,
// and the accumulator of a product is the COLS fragment of the result: so the ROWS fragment of its transpose.
// In LDS a fragment is one 16-byte piece per lane (fp32) or two, in planes (fp64): operands are read without conflicts
// and without address arithmetic beyond the tile's base, where a row-major tile costs more instructions than the product.
// (fp64: pieces of lane groups 2 and 3 swap fours, and the second plane starts half the banks further on, so that a tile is read
// row by row without conflicts, too, on its way back to memory.)
// ---------------------------------------------------------------------------------------
template <typename T>
struct Frag {
    static constexpr int PLANE = sizeof(T) == 8 ? 144 : 0;
    static constexpr int ELEMS = sizeof(T) == 8 ? 272 : 256;
    // first element of the lane's piece(s)
    static __device__ __forceinline__ int lane_at(int lane)
    {
        const int g = lane >> 4, p = lane & 15;
        if constexpr (sizeof(T) == 8)
            return (g * 16 + (p ^ ((g >> 1) * 4))) * 2;
        else
            return lane * 4;
    }
    // element (u, w) of a ROWS fragment; element (w, u) of a COLS fragment
    static __device__ __forceinline__ int at(int u, int w)
    {
        const int g = w & 3, v = w >> 2, p = chain_nat<T>(u);
        if constexpr (sizeof(T) == 8)
            return (v >> 1) * PLANE + (g * 16 + (p ^ ((g >> 1) * 4))) * 2 + (v & 1);
        else
            return (g * 16 + p) * 4 + v;
    }
    static __device__ __forceinline__ void load(const T *tile, int fo, T (&x)[4])
    {
        using V = typename Mfma<T>::vec_t;
        const V a = *reinterpret_cast<const V *>(tile + fo);
        x[0] = a.x;
        x[1] = a.y;
        if constexpr (sizeof(T) == 8) {
            const V b = *reinterpret_cast<const V *>(tile + fo + PLANE);
            x[2] = b.x;
            x[3] = b.y;
        } else {
            x[2] = a.z;
            x[3] = a.w;
        }
    }
    template <typename R>
    static __device__ __forceinline__ void store(T *tile, int fo, const R &x)
    {
        using V = typename Mfma<T>::vec_t;
        V a;
        a.x = x[0];
        a.y = x[1];
        if constexpr (sizeof(T) == 8) {
            V b;
            b.x = x[2];
            b.y = x[3];
            *reinterpret_cast<V *>(tile + fo + PLANE) = b;
        } else {
            a.z = x[2];
            a.w = x[3];
        }
        *reinterpret_cast<V *>(tile + fo) = a;
    }
};

// c + sum over the four instructions of a b
template <typename T, typename A, typename B>
__device__ __forceinline__ typename Mfma<T>::acc_t frag_mma(const A &a, const B &b, typename Mfma<T>::acc_t c)
{
#pragma unroll
    for (int s = 0; s < 4; ++s)
        c = Mfma<T>::run(a[s], b[s], c);
    return c;
}

__device__ __forceinline__ int frag_off(int i, int j) { return i * (i - 1) / 2 + j; }  // tile (i, j), i > j

template <typename T>
struct FactorLds {
    static constexpr int FT = Frag<T>::ELEMS;
    static constexpr int PS = LT + 16 / (int)sizeof(T);  // row stride of the diagonal tiles of L
    static constexpr int DT = LT * PS;
    T *sL, *sX, *sXD, *sD, *sH, *sLi;
    static __host__ __device__ constexpr int elems(int K) { return K * (K - 1) * FT + K * (FT + DT) + 2 * FT; }
    __device__ __forceinline__ FactorLds(T *lds, int K)
    {
        sL = lds;                             // tiles of L below the diagonal, ROWS
        sX = sL + K * (K - 1) / 2 * FT;       // tiles of the inverse below the diagonal, COLS
        sXD = sX + K * (K - 1) / 2 * FT;      // its diagonal tiles, COLS
        sH = sXD + K * FT;                    // the next diagonal tile of A on its way to the chain, ROWS
        sLi = sH + FT;                        // L_kk^-1 on its way to the workers, ROWS
        sD = sLi + FT;                        // diagonal tiles of L, row by row
    }
    __device__ __forceinline__ T *l(int i, int j) const { return sL + frag_off(i, j) * FT; }
    __device__ __forceinline__ T *x(int i, int j) const { return i == j ? sXD + i * FT : sX + frag_off(i, j) * FT; }
};

// Tiles between an nb x nb block in memory and LDS.  A wavefront moves a tile in four accesses per lane, 16 lanes along the contiguous
// direction of the block (fragments accessed as they lie in the registers would be 64 separate requests each where that is the
// other direction).  A block spans less than 2^31 bytes (128 rows, leading dimensions up to 2^20), so its accesses are 32-bit offsets from one
// uniform base: with 64-bit addresses the instructions in front of the loads alone took 4 to 9 thousand cycles.
template <typename T>
struct TileIO {
    using F = Frag<T>;
    char *p;
    unsigned si, sj, step;  // bytes from one tile row, tile column to the next; from one access to the next, four along the slow direction
    unsigned lane0;         // byte offset of the lane's first access
    int nb, f, s0;          // fast coordinate in the tile, slow one of the first access
    bool colfast;
    int lds0, lds1;         // places of the first two elements in a ROWS fragment; those of the others lie lds2 behind them
    static constexpr int LDS2 = sizeof(T) == 8 ? 16 : 8;

    // frag: the lane's column is the one it holds of a COLS fragment
    __device__ __forceinline__ TileIO(T *p_, int64_t rs, int64_t cs, int nb_, int lane, bool frag = false)
        : p(reinterpret_cast<char *>(p_)), nb(nb_)
    {
        constexpr unsigned size = sizeof(T);
        colfast = cs == 1 || rs != 1;
        f = frag ? chain_nat<T>(lane & 15) : lane & 15;
        s0 = lane >> 4;
        const unsigned r = (unsigned)rs * size, c = (unsigned)cs * size, fast = colfast ? c : r, slow = colfast ? r : c;
        si = LT * r;
        sj = LT * c;
        step = 4 * slow;
        lane0 = (unsigned)f * fast + (unsigned)s0 * slow;
        lds0 = F::at(row(0), col(0));
        lds1 = F::at(row(1), col(1));
    }
    __device__ __forceinline__ int row(int v) const { return colfast ? s0 + 4 * v : f; }
    __device__ __forceinline__ int col(int v) const { return colfast ? f : s0 + 4 * v; }
    __device__ __forceinline__ int lds(int v) const
    {
        // along the columns the places go by lane groups, two planes of two (fp64) or four in a row (fp32): F::at(p, 4 v + g)
        const int by_col = lds0 + (sizeof(T) == 8 ? (v >> 1) * F::PLANE + (v & 1) : v);
        const int by_row = ((v & 1) ? lds1 : lds0) + (v >> 1) * LDS2;
        return colfast ? by_row : by_col;
    }
    __device__ __forceinline__ T *elem(int i, int j, int v) const
    {
        return reinterpret_cast<T *>(p + (lane0 + ((unsigned)i * si + (unsigned)j * sj + (unsigned)v * step)));
    }
    __device__ __forceinline__ bool whole(int i) const { return (i + 1) * LT <= nb; }
    __device__ __forceinline__ bool inside(int i, int j, int v) const { return i * LT + row(v) < nb && j * LT + col(v) < nb; }

    // the elements of tile (i, j), i >= j, on their way; outside the block those of the identity, above the diagonal anything
    __device__ __forceinline__ void fetch(int i, int j, T (&x)[4]) const
    {
        if (whole(i)) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = *elem(i, j, v);
            return;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            x[v] = i == j && row(v) == col(v) ? T(1) : T(0);
            if (inside(i, j, v))
                x[v] = *elem(i, j, v);
        }
    }
    __device__ __forceinline__ void put(int i, int j, const T (&x)[4]) const
    {
        if (whole(i) && whole(j)) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                *elem(i, j, v) = x[v];
            return;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (inside(i, j, v))
                *elem(i, j, v) = x[v];
    }
    // tile (i, j) of L below the diagonal
    __device__ __forceinline__ void store(const T *tile, int i, int j) const
    {
        T x[4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            x[v] = tile[lds(v)];
        put(i, j, x);
    }
};

// tile number t of the lower tiles of eight tile rows counted column by column
__device__ __forceinline__ void col_decode(int t, int &i, int &j)
{
    j = (t >= 8) + (t >= 15) + (t >= 21) + (t >= 26) + (t >= 30) + (t >= 33) + (t >= 35);
    i = t - (15 - j) * j / 2;  // column j starts at its number (17 - j) j / 2, with row j
}

// X_kj up to the product with -L_kk^-1:  sum_{q = j..k-1} L_kq X_qj, the operands of the next product on their way while one runs
template <typename T>
__device__ __forceinline__ typename Mfma<T>::acc_t inverse_sum(const FactorLds<T> &m, int k, int j, int fo)
{
    T a[2][4], b[2][4];
    typename Mfma<T>::acc_t acc = {0, 0, 0, 0};
    const T *lp = m.l(k, j);
    Frag<T>::load(lp, fo, a[0]);
    Frag<T>::load(m.x(j, j), fo, b[0]);
    for (int q = j; q < k; q += 2) {
        if (q + 1 < k) {
            Frag<T>::load(lp + Frag<T>::ELEMS, fo, a[1]);
            Frag<T>::load(m.x(q + 1, j), fo, b[1]);
        }
        acc = frag_mma<T>(a[0], b[0], acc);
        if (q + 1 < k) {
            if (q + 2 < k) {
                Frag<T>::load(lp + 2 * Frag<T>::ELEMS, fo, a[0]);
                Frag<T>::load(m.x(q + 2, j), fo, b[0]);
            }
            acc = frag_mma<T>(a[1], b[1], acc);
        }
        lp += 2 * Frag<T>::ELEMS;
    }
    return acc;
}

// 1-based number of the first pivot of diagonal tile t that is not > 0 (0: none), where the tile is as chain_diag leaves it
template <typename T>
__device__ __forceinline__ int bad_pivot(const FactorLds<T> &m, int t, int lane)
{
    const int c = lane & 15;
    const unsigned b = (unsigned)(__ballot(!(m.sD[t * m.DT + c * m.PS + c] > T(0))) & 0xffffu);
    return b ? t * LT + __builtin_ctz(b) + 1 : 0;
}

// Factor an nb x nb block (K = ceil(nb / 16) tile rows) whose lower triangle is `in`, and with `inverse` invert the factor.  On
// return, after a workgroup barrier, the tiles of both are in the LDS of m; the diagonal tiles of L still lack the square roots of the
// pivots (column c times the diagonal entry of the inverse) and hold leftovers above the diagonal.  STORE: the factor is also written to
// `L` and, with `inverse`, the inverse to `Inv`, with zero_upper zeros above the diagonal tiles of L.  Returns, in
// wavefront 0, the 1-based index of the first pivot that is not > 0 (0: none).
//
// Wavefront 0 walks the chain  diagonal tile k -> panel tile (k + 1, k) -> update of the diagonal tile k + 1  and keeps it in
// registers: chain_diag leaves L_kk^-1 as the operand of the panel product, whose result is in turn both operands of the
// update, whose result is what chain_diag takes.  The workers hold the tiles of the trailing matrix in their accumulators,
// three each, from the load to the tile's own column.  Beside diagonal tile k they apply column k - 1 to them, hand the two tiles
// that the chain takes next over in LDS, and form row k of the inverse up to its product with L_kk^-1 (left-looking, so that a step has
// 25 to 34 tile products whatever k is); beside the chain's panel tile they do the other panel tiles and that product.  Two barriers per
// tile column.
//
// The workers are the wavefronts of the other three SIMDs.  A multiply-add waits for every matrix-core instruction of fp64 or fp32
// that is under way on its SIMD (measured: one dependent fp64 multiply-add per 10 cycles alone, per 72 beside one wavefront with a stream of
// matrix-core instructions, per 136 beside three), so a single tile product next to the chain costs it more than the product itself.
// The chain's neighbours on its SIMD only store: zeros, the diagonal tiles and the chain's panel tiles.
template <typename T, int W, bool STORE>
__device__ __forceinline__ int leaf_factor(const FactorLds<T> &m, const TileIO<T> &in, View<T> L, View<T> Inv, int nb, bool inverse,
                                           bool zero_upper, int wave, int lane)
{
    using MF = Mfma<T>;
    using acc_t = typename MF::acc_t;
    using F = Frag<T>;
    static_assert(W == 16 || (W == 4 && !STORE), "wavefront w runs on SIMD w % 4; three tiles a worker cover 8 (4) tile rows");
    constexpr int PER = W / 4, WORKERS = 3 * PER, SLOTS = 3, MAXK = W == 16 ? 8 : 4;
    const int K = (nb + LT - 1) / LT;
    const int r = chain_nat<T>(lane & 15), g = lane >> 4, fo = F::lane_at(lane);
    // diagonal tile k of L: column c times the diagonal entry of the inverse, zeros above the diagonal
    auto store_diag = [&](const TileIO<T> &l, int k) {
        const T *d = m.sD + k * m.DT, *xd = m.x(k, k);
        T y[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int u = l.row(v), w = l.col(v);
            y[v] = d[u * m.PS + w] * xd[F::at(w, w)];
            y[v] = w <= u ? y[v] : T(0);
        }
        l.put(k, k, y);
    };
    // elements of a diagonal tile as fetched -> its fragment with both triangles, through a place in LDS
    auto symmetric = [&](T *tile, const T (&a)[4], T (&b)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            tile[in.lds(v)] = a[v];
        wave_sync();
        F::load(tile, fo, b);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const T t = tile[F::at(4 * v + g, r)];  // the transpose
            b[v] = 4 * v + g <= r ? b[v] : t;
        }
    };
    auto store_inverse = [&](const TileIO<T> &x, int i, int j) {
        T y[4];
        F::load(m.x(i, j), fo, y);
        x.put(i, j, y);
    };
    if (wave == 0) {
        T S[4];
        {
            T a[4];
            in.fetch(0, 0, a);
            symmetric(m.x(0, 0), a, S);
        }
        LEAF16_STAMP(62);
        for (int k = 0; k < K; ++k) {
            T X[4], d;
            chain_diag<T>(S, m.sD + k * m.DT + r * m.PS, d, X, r, g);
            const T rs_ = rsqrt_acc(d);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                X[v] = (4 * v + g <= r) ? X[v] * rs_ : T(0);
            F::store(m.sLi, fo, X);
            LEAF16_STAMP(1 + 3 * k);
            __syncthreads();
            LEAF16_STAMP(2 + 3 * k);
            if (k + 1 < K) {
                T av[4], sv[4];
                F::load(m.l(k + 1, k), fo, av);
                F::load(m.sH, fo, sv);
                const acc_t P = frag_mma<T>(X, av, acc_t{0, 0, 0, 0});  // L_k+1,k: P[v] = element (r, 4 v + g)
                const T np[4] = {-P[0], -P[1], -P[2], -P[3]};
                const acc_t s = frag_mma<T>(np, P, acc_t{sv[0], sv[1], sv[2], sv[3]});
                F::store(m.l(k + 1, k), fo, P);
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    S[v] = s[v];
            }
            T *xd = m.x(k, k);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                xd[F::at(4 * v + g, r)] = X[v];  // element (r, 4 v + g) of a COLS fragment
            LEAF16_STAMP(3 + 3 * k);
            __syncthreads();
        }
    } else if ((wave & 3) == 0) {
        const int h = wave / 4 - 1;  // of PER - 1
        const TileIO<T> l(L.p, L.rs, L.cs, nb, lane);
        const T zero[4] = {};
        if (STORE && zero_upper)
            for (int i = 1, t = h; i < K; ++i) {
                for (; t < i; t += PER - 1)
                    l.put(t, i, zero);
                t -= i;
            }
        for (int k = 0; k < K; ++k) {
            if (STORE && k > 0) {  // column k - 1 of L is final
                for (int i = k - 1 + h; i < K; i += PER - 1) {
                    if (i == k - 1)
                        store_diag(l, i);
                    else
                        l.store(m.l(i, k - 1), i, k - 1);
                }
            }
            LEAF16_STAMP(1 + 3 * k);
            __syncthreads();
            __syncthreads();
        }
    } else {
        // worker wv runs on SIMD 1 + wv % 3; tiles go to the workers in turn, column by column
        const int wpos = (wave & 3) - 1, wrow = wave >> 2, wv = 3 * wrow + wpos;
        // its column of the row of the inverse: in turn over the SIMDs and back again, the longest sum first
        const int xj = 3 * wrow + ((wrow & 1) ? 2 - wpos : wpos);
        int ti[SLOTS], tj[SLOTS];
        acc_t N[SLOTS], xs = {0, 0, 0, 0};  // minus the tiles
        T a[SLOTS][4] = {};
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int t = 1 + wv + s * WORKERS;  // (not tile (0, 0))
            if constexpr (W == 16) {
                col_decode(t, ti[s], tj[s]);
            } else {  // four tile rows
                tj[s] = (t >= 4) + (t >= 7) + (t >= 9);
                ti[s] = t - (7 - tj[s]) * tj[s] / 2;
            }
            if (ti[s] < K)
                in.fetch(ti[s], tj[s], a[s]);
            else
                ti[s] = tj[s] = -1;
        }
        LEAF16_STAMP(62);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int i = ti[s], j = tj[s];
            N[s] = acc_t{0, 0, 0, 0};
            if (i < 0)
                continue;
            T *tile = m.x(i, j);  // nobody needs that place yet
            T b[4];
            if (i == j) {
                symmetric(tile, a[s], b);
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    tile[in.lds(v)] = a[s][v];
                wave_sync();
                F::load(tile, fo, b);
            }
            N[s] = acc_t{-b[0], -b[1], -b[2], -b[3]};
            if (j <= 1 && i == 1)  // (1, 0) and (1, 1): the chain's
                F::store(j == 0 ? m.l(1, 0) : m.sH, fo, b);
        }
        for (int k = 0; k < K; ++k) {
            if (k > 0) {
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) {
                    const int i = ti[s], j = tj[s];
                    if (j < k || (j == k && i == k))  // done, or the chain has it
                        continue;
                    T b[4], c[4];
                    F::load(m.l(j, k - 1), fo, b);
                    F::load(m.l(i, k - 1), fo, c);
                    N[s] = frag_mma<T>(b, c, N[s]);
                    if (i == k + 1) {  // (k + 1, k) and (k + 1, k + 1): the chain's
                        const T n[4] = {-N[s][0], -N[s][1], -N[s][2], -N[s][3]};
                        F::store(j == k ? m.l(i, k) : m.sH, fo, n);
                    }
                }
            }
            const bool mine = inverse && xj < k;
            if (mine)
                xs = inverse_sum<T>(m, k, xj, fo);
            LEAF16_STAMP(1 + 3 * k);
            __syncthreads();
            T li[4];
            F::load(m.sLi, fo, li);
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                if (tj[s] == k && ti[s] > k + 1) {
                    const acc_t P = frag_mma<T>(li, N[s], acc_t{0, 0, 0, 0});
                    F::store(m.l(ti[s], k), fo, -P);
                }
            if (mine) {
                const acc_t P = frag_mma<T>(li, xs, acc_t{0, 0, 0, 0});
                F::store(m.x(k, xj), fo, -P);
            }
            LEAF16_STAMP(3 + 3 * k);
            __syncthreads();
        }
    }
    if (STORE) {  // the last diagonal tile of L, the inverse
        if (wave == 0)
            store_diag(TileIO<T>(L.p, L.rs, L.cs, nb, lane), K - 1);
        if (inverse) {
            const TileIO<T> x(Inv.p, Inv.rs, Inv.cs, nb, lane, true);
            for (int t = W - 1 - wave; t < MAXK * (MAXK + 1) / 2; t += W) {
                int i, j;
                col_decode(t, i, j);
                if (i < K)
                    store_inverse(x, i, j);
            }
        }
    }
    LEAF16_STAMP(60);
    int fail = 0;
    if (wave == 0)
        for (int t = K - 1; t >= 0; --t) {
            const int f = bad_pivot<T>(m, t, lane);
            fail = f ? f : fail;
        }
    return fail;
}

}  // namespace la
