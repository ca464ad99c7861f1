// Batched strided GEMM on the gfx950 matrix cores: the dense contraction inside every
// blocked algorithm of the library (trailing syrk/gemm update of the right-looking potrf,
// the off-diagonal updates of blocked trsm / trmm, and the three triangular phases of the
// potrf backward expression of arXiv 1710.08717, section 4.2).
//
//   C(i,j) = beta * C(i,j) + alpha * sum_k A(i,k) B(k,j)
//
// Operands are strided views (either index may be the contiguous one), so transposes and
// upper/lower variants never copy.  Triangular operands are masked between LDS and the matrix cores
// and their structurally-zero K range is skipped.
//
// k_gemm: operands whose rows are 16-byte aligned.  Slabs of K go straight from memory to LDS (global_load_lds_dwordx4), slab s + 1 while slab
// s is multiplied; 128 x 128, 64 x 64 and 32 x 32 workgroup tiles, four wavefronts in a 2 x 2 arrangement, 16x16x4 MFMA
// (v_mfma_f64_16x16x4_f64 / v_mfma_f32_16x16x4_f32).  Bound by the matrix cores, and by what else is issued beside them: a vector instruction
// waits for the matrix instruction under way on its SIMD, so the loop has next to none (4 to 9 per 64 to 128 matrix instructions on 128 x 128 tiles, for
// 100 to 150 when slabs passed through registers with their addresses added up and their triangles masked on the way).
// us, slabs through registers -> to LDS: 4096^3 fp64 2240 -> 1965 (70 TFLOP/s), fp32 1170 -> 995 (138); 6144^2 x 1024 1355 -> 1158 and 655 -> 580; 32 x 512^3
// 153 -> 132 and 84 -> 70; 32 x 256^3 29.5 -> 23.5 and 17.4 -> 13.6; 64 x 200^3 49 -> 34 and 25 -> 24; 4096 x 512 x 512 51 -> 41 and 29 -> 22.5.
// k_gemm_staged: ragged operands (odd sizes and leading dimensions), whose chunks are loaded with the alignment of one element.
#include <algorithm>

#include "common.hpp"

namespace la {

// One 16-byte chunk per lane from memory to LDS: lane l's goes to `lds` (uniform) + 16 l.  Written as assembly because the compiler waits for all
// of these before it reads LDS, whichever part, and adds up the addresses in vector registers; wait_loads is where a reader waits.
// (The warning is about any clobber of m0; without it the compiler takes m0 for unchanged.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_lds16(const char *base, uint32_t off, void *lds)
{
    const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(at), "v"(off), "s"(base) : "m0", "memory");
}
#pragma clang diagnostic pop
// until this wavefront's loads have landed
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

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
//
// A slab is BK values of k of one operand, BKB = BK * sizeof(T) bytes, kept in LDS as 16-byte chunks in the order of memory:
//   k contiguous:     row o holds BKB / 16 chunks, chunk c of it at position c ^ (o & 7)
//   outer contiguous: row k holds OUT / VW chunks in their order
// (the exchange of chunks spreads the 16 rows that a fragment read touches over all banks; with 16 chunks a row, BKB = 256, over half of them: 4 conflict
// cycles per LDS instruction with k contiguous in both operands, none with 8).  A lane reads whole chunks: VW consecutive k
// of its row, or (outer contiguous) one k of G neighbouring rows, which are then the rows of G different 16 x 16 tiles.  So the
// contraction index k = (4 s + lane / 16) VW + u belongs to step (s, u), and tile x's row r is row map(x, r) of the wavefront's part.
// ---------------------------------------------------------------------------------------
template <typename T, int OUT, int BKB, bool KF>
struct Slab {
    static constexpr int VW = Mfma<T>::VW;
    static constexpr int BK = BKB / (int)sizeof(T);
    static constexpr int ELEMS = OUT * BK;
    static constexpr int NCH = OUT * BKB / 16 / 256;          // chunks per thread
    static constexpr int RC = KF ? BKB / 16 : OUT / VW;       // chunks per row of the slab
    static constexpr int TILES = OUT / 32;                    // 16-wide tiles of a wavefront (two of them share OUT)
    static constexpr int G = KF ? 1 : (VW < TILES ? VW : TILES);
    static_assert(NCH >= 1 && BKB >= 128, "slab too small for 256 threads");

    // outer index and k of the chunk that thread (w, lane) copies in its i-th turn to position (i * 4 + w) * 64 + lane
    static __device__ __forceinline__ void coords(int i, int w, int lane, int &o, int &k)
    {
        const int p = (i * 4 + w) * 64 + lane, row = p / RC, c = p % RC;
        o = KF ? row : c * VW;
        k = KF ? (c ^ (row & 7)) * VW : row;
    }
    static __device__ __forceinline__ int map(int x, int r) { return KF ? 16 * x + r : 16 * G * (x / G) + G * r + x % G; }
};

// Copies slabs of one operand straight from memory to LDS, in 16-byte chunks: no registers and no vector arithmetic on the way (on this chip a
// vector instruction waits for the matrix instruction under way on its SIMD).  No address lies outside the operand: rows past its end repeat the
// last one (nothing that is kept comes from them), and so does a k past its end (the reader masks it).
template <typename T, int OUT, int BKB, bool KF>
struct Copier {
    using S = Slab<T, OUT, BKB, KF>;
    static constexpr int VW = S::VW;
    uint32_t off[S::NCH];  // bytes from the slab's first element
    const char *next;      // the next slab's first element
    int64_t step;

    // src: the operand's item
    __device__ __forceinline__ void start(const T *src, int64_t so, int64_t sk, int o0, int k0)
    {
        next = reinterpret_cast<const char *>(src + o0 * so + k0 * sk);
        step = S::BK * sk * (int64_t)sizeof(T);
    }
    // no: rows of the operand; where those are contiguous, up to a multiple of VW exist, or may be read (GemmOpts::padA)
    __device__ __forceinline__ void init(int64_t so, int64_t sk, int o0, int no, int w, int lane)
    {
#pragma unroll
        for (int i = 0; i < S::NCH; ++i) {
            int o, k;
            S::coords(i, w, lane, o, k);
            off[i] = (uint32_t)(min(o, (KF ? no - 1 : (no - 1) / VW * VW) - o0) * so + k * sk) * (uint32_t)sizeof(T);
        }
    }
    // k0, nk: the slab's first k, a multiple of VW, and the operand's end, the same for k as above
    __device__ __forceinline__ void fetch(T *lds, int64_t sk, int k0, int nk, int w, int lane)
    {
        const char *base = next;
        next += step;
        if (k0 + S::BK <= nk) {
#pragma unroll
            for (int i = 0; i < S::NCH; ++i)
                load_lds16(base, off[i], lds + (i * 4 + w) * 64 * VW);
        } else {
#pragma unroll
            for (int i = 0; i < S::NCH; ++i) {
                int o, k;
                S::coords(i, w, lane, o, k);
                const int back = max(k - ((KF ? (nk - 1) / VW * VW : nk - 1) - k0), 0);
                load_lds16(base, off[i] - (uint32_t)(back * sk) * (uint32_t)sizeof(T), lds + (i * 4 + w) * 64 * VW);
            }
        }
    }
};

// A wavefront's operand values of NS groups of steps of a slab: value(x, s, u), x the 16-wide tile, step (s, u).
template <typename T, int OUT, int BKB, bool KF, int NS>
struct Fragments {
    using S = Slab<T, OUT, BKB, KF>;
    static constexpr int VW = S::VW, TILES = S::TILES, G = S::G, W = KF ? VW : G, PER = KF ? NS : NS * VW;
    typedef T vec __attribute__((ext_vector_type(W)));
    vec f[PER][TILES / G];  // KF: [s][x], elements u; else [(s, u)][x / G], elements x % G

    __device__ __forceinline__ T value(int x, int s, int u) const
    {
        if constexpr (KF)
            return f[s][x][u];
        else if constexpr (G == 1)
            return f[s * VW + u][x][0];
        else
            return f[s * VW + u][x / G][x % G];
    }
    __device__ __forceinline__ void read(const T *lds, int first, int wo, int lane)
    {
        const int l16 = lane & 15, lk = lane >> 4;
        if constexpr (KF) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const T *p = lds + (wo + l16) * S::BK + ((4 * (first + s) + lk) ^ (l16 & 7)) * VW;
#pragma unroll
                for (int x = 0; x < TILES; ++x)
                    f[s][x] = *reinterpret_cast<const vec *>(p + 16 * x * S::BK);
            }
        } else {
            const T *p = lds + (4 * first + lk) * VW * OUT + wo + G * l16;
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int u = 0; u < VW; ++u)
#pragma unroll
                    for (int g = 0; g < TILES / G; ++g)
                        f[s * VW + u][g] = *reinterpret_cast<const vec *>(p + (4 * s * VW + u) * OUT + 16 * G * g);
        }
    }
    // zeros from k = nk on; k0: first k of these steps
    __device__ __forceinline__ void mask_end(int k0, int nk, int lane)
    {
        asm volatile("" : "+s"(k0));  // (or the compiler keeps one running index per value through the whole loop)
        const int lk = lane >> 4;
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int u = 0; u < VW; ++u) {
                const bool drop = k0 + (4 * s + lk) * VW + u >= nk;
#pragma unroll
                for (int x = 0; x < TILES; ++x)
                    element(x, s, u, drop);
            }
    }
    // zeros on the far side of a triangle: tri 1 keeps outer >= k, 2 outer <= k; o0, k0: first row and k of these steps
    __device__ __forceinline__ void mask_tri(int o0, int k0, int tri, int lane)
    {
        asm volatile("" : "+s"(k0));
        const int l16 = lane & 15, lk = lane >> 4, sgn = tri == 2 ? -1 : 1;
        const int d0 = sgn * (o0 + (KF ? 1 : G) * l16 - k0 - lk * VW);  // sign of (row - k) at x, s, u = 0
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int u = 0; u < VW; ++u)
#pragma unroll
                for (int x = 0; x < TILES; ++x)
                    element(x, s, u, d0 < -sgn * (S::map(x, 0) - 4 * s * VW - u));
    }
    __device__ __forceinline__ void element(int x, int s, int u, bool drop)
    {
        if constexpr (KF)
            f[s][x][u] = drop ? T(0) : f[s][x][u];
        else
            f[s * VW + u][x / G][x % G] = drop ? T(0) : f[s * VW + u][x / G][x % G];
    }
};

template <typename T, int BM, int BN, int BKB, int NB, bool AKF, bool BKF, bool SYM>
__global__ __launch_bounds__(256, BM * BN >= 128 * 128 ? 2 : (sizeof(T) == 4 ? 6 : 4)) void k_gemm(View<const T> A, View<const T> B, View<T> C, int64_t batch, int M,
                                                 int N, int K, T alpha, T beta, GemmOpts o, int tiles_m, int tiles_n)
{
    using MF = Mfma<T>;
    using acc_t = typename MF::acc_t;
    using SA = Slab<T, BM, BKB, AKF>;
    using SB = Slab<T, BN, BKB, BKF>;
    constexpr int BK = SA::BK, VW = SA::VW;
    constexpr int WM = BM / 2, WN = BN / 2;
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int PARTS = BM * BN >= 128 * 128 ? 2 : 1;  // of a slab whose operand values are in registers at a time
    constexpr int PART = WM * (WN + 1);  // a wavefront's part of a symmetric result
    extern __shared__ __align__(16) char lds_bytes[];  // gemm_lds
    T *lds = reinterpret_cast<T *>(lds_bytes);

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
    int kbeg, kend;  // (kbeg is a tile's first row or column: whole chunks start there)
    k_range(o, i0, j0, BM, BN, Kl, kbeg, kend);

    T *Cp = C.item(b);
    const int triB_o = o.triB == 1 ? 2 : (o.triB == 2 ? 1 : 0);

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = (w >> 1) * WM, wn = (w & 1) * WN;

    acc_t acc[TM][TN];
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int y = 0; y < TN; ++y)
            acc[x][y] = acc_t{0, 0, 0, 0};

    // Software pipeline over slabs in two LDS buffers: slab s + 1 is requested as soon as every wavefront has read slab s - 1 (the barrier) and its
    // own part of slab s, and is waited for most of a slab of matrix instructions later.  One buffer (NB = 1): requested once everybody has slab
    // s in registers, a second barrier, but more workgroups a compute unit.  (Three and four buffers: 5 to 15 % slower, fewer workgroups.)
    // SYM (GemmOpts::symsum): with 1 a second pass over the same range adds B^T A^T -- same strides, the base pointers change places.
    if (kbeg < kend) {
        const T *pa = A.item(b), *pb = B.item(b);
        const int ns = (kend - kbeg + BK - 1) / BK, total = SYM && o.symsum == 1 ? 2 * ns : ns;
        Copier<T, BM, BKB, AKF> ca;
        Copier<T, BN, BKB, BKF> cb;
        ca.init(A.rs, A.cs, i0, M, w, lane);
        cb.init(B.cs, B.rs, j0, N, w, lane);
        ca.start(pa, A.rs, A.cs, i0, kbeg);
        cb.start(pb, B.cs, B.rs, j0, kbeg);
        int kr = kbeg;  // first k of the next request
        auto request = [&](int t, T *at) {
            if (SYM && t == ns) {
                ca.start(pb, A.rs, A.cs, i0, kbeg);
                cb.start(pa, B.cs, B.rs, j0, kbeg);
                kr = kbeg;
            }
            ca.fetch(at, A.cs, kr, Kl, w, lane);
            cb.fetch(at + SA::ELEMS, B.rs, kr, Kl, w, lane);
            kr += BK;
        };
        // slabs within [klo, khi) touch neither the zero side of a triangle nor the end of the range: nothing to mask
        const int klo = __builtin_amdgcn_readfirstlane(max(o.triA == 2 ? i0 + BM - 1 : 0, triB_o == 2 ? j0 + BN - 1 : 0));
        const int khi = __builtin_amdgcn_readfirstlane(min(kend, min(o.triA == 1 ? i0 + 1 : kend, triB_o == 1 ? j0 + 1 : kend)));
        constexpr int BUF = SA::ELEMS + SB::ELEMS;
        auto slab = [&](int t, T *at, T *other) {  // other: the buffer of slab t + 1
            wait_loads();
            __syncthreads();
            const int k0 = kbeg + (SYM && t >= ns ? t - ns : t) * BK;
            const bool edge = k0 < klo || k0 + BK > khi;
#pragma unroll
            for (int part = 0; part < PARTS; ++part) {
                constexpr int NS = BK / (4 * VW) / PARTS;
                const int kp = k0 + part * NS * 4 * VW;
                Fragments<T, BM, BKB, AKF, NS> fa;
                Fragments<T, BN, BKB, BKF, NS> fb;
                fa.read(at, part * NS, wm, lane);
                fb.read(at + SA::ELEMS, part * NS, wn, lane);
                if (part == PARTS - 1) {
                    if constexpr (NB == 1)
                        __syncthreads();  // everybody has read the slab
                    if (t + 1 < total)
                        request(t + 1, other);
                }
                if (edge) {
                    if (o.triA)
                        fa.mask_tri(i0 + wm, kp, o.triA, lane);
                    if (triB_o)
                        fb.mask_tri(j0 + wn, kp, triB_o, lane);
                    if (k0 + BK > Kl) {
                        fa.mask_end(kp, Kl, lane);
                        fb.mask_end(kp, Kl, lane);
                    }
                }
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (BM * BN < 128 * 128 && kp + 4 * VW * s >= kend)
                        break;
#pragma unroll
                    for (int u = 0; u < VW; ++u)
#pragma unroll
                        for (int x = 0; x < TM; ++x)
#pragma unroll
                            for (int y = 0; y < TN; ++y)
                                acc[x][y] = MF::run(fa.value(x, s, u), fb.value(y, s, u), acc[x][y]);
                }
            }
        };
        request(0, lds);
        // two slabs a turn: the buffers' places are then part of the instructions
        for (int t = 0; t < total; t += NB) {
            slab(t, lds, lds + (NB - 1) * BUF);
            if (NB == 2 && t + 1 < total)
                slab(t + 1, lds + BUF, lds);
        }
    }

    const int l16 = lane & 15;
    if constexpr (SYM) {
        // Every value goes to both triangles.  The wavefront lays its part out in LDS, stores the entries on and below the diagonal row by
        // row and their mirror images column by column, so that both run along the rows of C.
        constexpr int LD = WN + 1;
        __syncthreads();
        T *part = lds + w * PART;
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int y = 0; y < TN; ++y)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    part[SA::map(x, MF::row(lane, v)) * LD + SB::map(y, l16)] = alpha * acc[x][y][v];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        const int it = i0 + wm, jt = j0 + wn;
        if (jt > it + WM - 1 || it >= M)
            return;
        constexpr int RP = 64 / WN;  // rows per turn
        {
            const int u0 = lane / WN, c = lane % WN, rows = min(M - it, WM) - u0, first = jt + c - it - u0;  // rows q from `first` to `rows` are kept
            T *at = Cp + (int64_t)(it + u0) * C.rs + (int64_t)(jt + c) * C.cs;
            T *p = part + u0 * LD + c;
#pragma unroll
            for (int q = 0; q < WM; q += RP, at += RP * C.rs)
                if (q < rows && q >= first) {
                    T upd = p[q * LD];
                    if (beta != T(0)) {
                        upd = fma(beta, *at, upd);
                        p[q * LD] = upd;
                    }
                    *at = upd;
                }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        constexpr int CP = 64 / WM;  // columns per turn
        const int c0 = lane / WM, u = lane % WM, cols = it + u < M ? it + u - jt - c0 : 0;  // columns q below `cols` have a mirror image
        T *at = Cp + (int64_t)(jt + c0) * C.rs + (int64_t)(it + u) * C.cs;
        const T *p = part + u * LD + c0;
#pragma unroll
        for (int q = 0; q < WN; q += CP, at += CP * C.rs)
            if (q < cols)
                *at = p[q];
        return;
    }
    if (C.cs == 1 && (i0 >= j0 + BN || j0 >= i0 + BM || !(o.halfDiag || o.maskC == 1 || o.maskC == 2))) {
        // Nothing is masked: addresses are a uniform part and one offset per lane, G neighbouring columns are stored at once.
        constexpr int G = SB::G;
        typedef T vec __attribute__((ext_vector_type(G), aligned(sizeof(T))));
        const bool whole = i0 + BM <= M && j0 + BN <= N;
        const int row = SA::map(0, MF::row(lane, 0)), col = SB::map(0, l16), rows = M - i0 - wm - row, cols = N - j0 - wn - col;  // what is left from here
        const uint32_t off = (uint32_t)(row * C.rs + col) * (uint32_t)sizeof(T);
        constexpr int VR = MF::row(0, 1) * SA::G;  // rows from one register of an accumulator to the next
        T *Ct = Cp + (int64_t)(i0 + wm) * C.rs + (j0 + wn);
#pragma unroll
        for (int x = 0; x < TM; ++x) {
            T *Cx = Ct + (int64_t)SA::map(x, 0) * C.rs;
            auto at = [&](int v, int y) { return reinterpret_cast<T *>(reinterpret_cast<char *>(Cx + v * VR * C.rs + SB::map(y, 0)) + off); };
            auto left = [&](int v, int y) { return whole ? G : (SA::map(x, 0) + v * VR < rows ? cols - SB::map(y, 0) : 0); };
            vec old[4][TN / G];
            if (beta != T(0)) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int y = 0; y < TN; y += G) {
                        const int n = left(v, y);
                        if (n >= G) {
                            old[v][y / G] = *reinterpret_cast<const vec *>(at(v, y));
                        } else {
#pragma unroll
                            for (int g = 0; g < G - 1; ++g)
                                if (g < n)
                                    old[v][y / G][g] = at(v, y)[g];
                        }
                    }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int y = 0; y < TN; y += G) {
                    vec r;
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        r[g] = alpha * acc[x][y + g][v];
                        if (beta != T(0))
                            r[g] = fma(beta, old[v][y / G][g], r[g]);
                    }
                    const int n = left(v, y);
                    if (n >= G) {
                        *reinterpret_cast<vec *>(at(v, y)) = r;
                    } else {
#pragma unroll
                        for (int g = 0; g < G - 1; ++g)
                            if (g < n)
                                at(v, y)[g] = r[g];
                    }
                }
        }
        return;
    }
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int y = 0; y < TN; ++y)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                store_c<T>(Cp, C.rs, C.cs, i0 + wm + SA::map(x, MF::row(lane, v)), j0 + wn + SB::map(y, l16), M, N, acc[x][y][v],
                           alpha, beta, o);
}

// ---------------------------------------------------------------------------------------
// Ragged operands (odd sizes and leading dimensions): slabs travel global memory -> registers -> LDS, chunks loaded with the alignment of one
// element, the ones that cross the end of the operand element by element, zeros behind it.  The kernel above with such a copier was
// 10 % behind in the long triangular products of one matrix (n = 3001, fp64, factor + gradient 2270 -> 2550 us): it keeps more in registers.
// LDS slab layouts (chosen so that global->LDS stores are 16-byte vectors and the fragment reads are bank-conflict free):
//   k contiguous:     s[o][BK + VW]      (row stride 18 doubles / 20 floats)
//   outer contiguous: s[k][OUT + 16]
// ---------------------------------------------------------------------------------------
template <typename T, int OUT, int BK, bool KF>
struct StagedSlab {
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
template <typename T, int OUT, int BK, bool KF, typename RV>
__device__ __forceinline__ void slab_fetch(RV &r, const T *src, int64_t so, int64_t sk, int o0, int no, int k0, int nk)
{
    using S = StagedSlab<T, OUT, BK, KF>;
    using V = typename Mfma<T>::vec_t;
    using L = typename LooseVec<T>::type;
    if (o0 + OUT <= no && k0 + BK <= nk) {  // (uniform) nothing crosses an end
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
        r[c] = v;
    }
}

template <typename T, int OUT, int BK, bool KF, typename RV>
__device__ __forceinline__ void slab_commit(T *s, RV &r, int o0, int k0, int tri)
{
    using S = StagedSlab<T, OUT, BK, KF>;
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

template <typename T, int BM, int BN, int BK, int NBUF, bool AKF, bool BKF, bool SYM>
__global__ __launch_bounds__(256, 2) void k_gemm_staged(View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int N, int K,
                                                        T alpha, T beta, GemmOpts o, int tiles_m, int tiles_n)
{
    using MF = Mfma<T>;
    using acc_t = typename MF::acc_t;
    using V = typename MF::vec_t;
    using SA = StagedSlab<T, BM, BK, AKF>;
    using SB = StagedSlab<T, BN, BK, BKF>;
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
            slab_fetch<T, BM, BK, AKF>(ra, Ap, A.rs, A.cs, i0, M, kbeg, Kl);
            slab_fetch<T, BN, BK, BKF>(rb, Bp, B.cs, B.rs, j0, N, kbeg, Kl);
            slab_commit<T, BM, BK, AKF>(sA[0], ra, i0, kbeg, o.triA);
            slab_commit<T, BN, BK, BKF>(sB[0], rb, j0, kbeg, triB_o);
            if (kbeg + BK < kend) {
                slab_fetch<T, BM, BK, AKF>(ra, Ap, A.rs, A.cs, i0, M, kbeg + BK, Kl);
                slab_fetch<T, BN, BK, BKF>(rb, Bp, B.cs, B.rs, j0, N, kbeg + BK, Kl);
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
                slab_fetch<T, BM, BK, AKF>(ra, Ap, A.rs, A.cs, i0, M, k0 + 2 * BK, Kl);
                slab_fetch<T, BN, BK, BKF>(rb, Bp, B.cs, B.rs, j0, N, k0 + 2 * BK, Kl);
            }
            multiply(sA[buf], sB[buf]);
            __syncthreads();
            buf ^= 1;
        }
    } else {
        if (kbeg < kend) {
            slab_fetch<T, BM, BK, AKF>(ra, Ap, A.rs, A.cs, i0, M, kbeg, Kl);
            slab_fetch<T, BN, BK, BKF>(rb, Bp, B.cs, B.rs, j0, N, kbeg, Kl);
        }
        for (int k0 = kbeg; k0 < kend; k0 += BK) {
            slab_commit<T, BM, BK, AKF>(sA[0], ra, i0, k0, o.triA);
            slab_commit<T, BN, BK, BKF>(sB[0], rb, j0, k0, triB_o);
            __syncthreads();
            if (k0 + BK < kend) {
                slab_fetch<T, BM, BK, AKF>(ra, Ap, A.rs, A.cs, i0, M, k0 + BK, Kl);
                slab_fetch<T, BN, BK, BKF>(rb, Bp, B.cs, B.rs, j0, N, k0 + BK, Kl);
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
//   A with k contiguous: one wavefront per row, lanes stride over k, shuffle reduction; or the whole block on one row (SPLIT).
//   A with i contiguous: a block takes 64 rows, its eight wavefronts an eighth of the k range each
//   (every load is 64 consecutive elements), LDS reduction; or 16 rows and a 32nd of the range a quarter wavefront (SPLIT).
// ---------------------------------------------------------------------------------------
constexpr int GEMV_N = 8;
constexpr int GEMV_THREADS = 512;
constexpr int GEMV_FEW = 16;

// The loads of several k go out together, those of B with them: with one k at a time and a branch per column a wavefront
// waits for memory twice per k (500 x 9568 times one vector, fp64, 27 -> 22 us; its transpose 59 -> 11).  A
// column more than there are costs its loads (300 items 5 x 200 times 7 columns with A transposed, fp64, bound by the
// loads of B: 31 us with eight), so every count has its own instance.
// ADD: beta multiplies `add` (one item, C's strides), else C itself.  (An instance of its own, because many items of a row or two are bound by each workgroup's
// first instructions: potri's rule for 52367 matrices of n = 1, fp32, 145 us, 166 with a third operand like the other two, 155 with a pointer that may be null.)
template <typename T, int N, bool SPLIT, bool ADD>
__global__ __launch_bounds__(GEMV_THREADS) void k_gemv(View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int K,
                                              T alpha, T beta, int triA, int tiles, const T *add)
{
    constexpr int NW = GEMV_THREADS / 64;  // wavefronts: rows per block (k contiguous) or slices of k
    constexpr int UN = N == 1 ? 8 : (N <= 4 ? 4 : 2);
    __shared__ T red[NW][64][N];
    const int64_t b = blockIdx.x / tiles;
    const int tile = (int)(blockIdx.x % tiles);
    const T *Ap = A.item(b);
    const T *Bp = B.item(b);
    T *Cp = C.item(b);
    const T *Ci = ADD ? add : Cp;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t jo[N];
    T acc[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        jo[j] = j * B.cs;
        acc[j] = T(0);
    }
    const bool rows = A.cs == 1;
    const int i = rows ? (SPLIT ? tile : tile * NW + w) : (SPLIT ? tile * GEMV_FEW + lane % GEMV_FEW : tile * 64 + lane);
    if (i < M) {
        const int kb = triA == 2 ? i : 0, ke = triA == 1 ? min(K, i + 1) : K;
        const int first = rows ? kb + (SPLIT ? (int)threadIdx.x : lane) : (SPLIT ? (int)threadIdx.x / GEMV_FEW : w);
        const int step = rows ? (SPLIT ? GEMV_THREADS : 64) : (SPLIT ? GEMV_THREADS / GEMV_FEW : NW);
        const int last = rows ? ke : K;
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
        if (i >= M)  // (never where the block has one row)
            return;
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
                acc[j] += __shfl_xor(acc[j], off, WAVE);
        if constexpr (SPLIT) {
            if (lane == 0)
#pragma unroll
                for (int j = 0; j < N; ++j)
                    red[w][0][j] = acc[j];
            __syncthreads();
            if (w != 0)
                return;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                acc[j] = T(0);
#pragma unroll
                for (int q = 0; q < NW; ++q)
                    acc[j] += red[q][0][j];
            }
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if (lane == 0) {
                const int64_t e = (int64_t)i * C.rs + (int64_t)j * C.cs;
                const T upd = alpha * acc[j];
                Cp[e] = (beta == T(0)) ? upd : fma(beta, Ci[e], upd);
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
        red[w][lane][j] = acc[j];
    __syncthreads();
    if (w == 0 && i < M && (!SPLIT || lane < GEMV_FEW)) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            T sum = T(0);
#pragma unroll
            for (int q = 0; q < NW; ++q)
                sum += red[q][lane][j];
            if constexpr (SPLIT)
#pragma unroll
                for (int f = GEMV_FEW; f < 64; f += GEMV_FEW)
#pragma unroll
                    for (int q = 0; q < NW; ++q)
                        sum += red[q][lane + f][j];
            const int64_t e = (int64_t)i * C.rs + (int64_t)j * C.cs;
            const T upd = alpha * sum;
            Cp[e] = (beta == T(0)) ? upd : fma(beta, Ci[e], upd);
        }
    }
}

template <typename T>
static la_status launch_gemv(View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int N, int K, T alpha, T beta, int triA,
                             hipStream_t st, const T *add = nullptr)
{
    const bool rows = A.cs == 1;
    const int per = rows ? GEMV_THREADS / 64 : 64, few = rows ? 1 : GEMV_FEW;
    // Few blocks and long sums: the finer split.  With k contiguous from 12 elements of k a block of rows on (one vector, fp32 and fp64:
    // 500 x 9568 16 -> 6 and 22 -> 9 us, 8 x 30000 43 -> 8 and 54 -> 10; but 2000 x 2048, 250 blocks, 5.9 -> 8.0 and 7.0 -> 8.6), transposed from
    // half an element a block on (500 x 500 7.7 -> 3.9 and 9.3 -> 4.4, 9568 x 500 8.8 -> 7.8 and 11.2 -> 8.9, 4000 x 4000 57 -> 23 and 67 -> 24;
    // but 16000 x 100, 250 blocks, 3.7 -> 5.0 and 4.0 -> 5.1).  Whole blocks are not always full, and what is there to fill the chip are the rows: not above
    // 10240 of them transposed (11 to 13 thousand rows, one to eight columns: 4 to 49 % slower in one case out of four), with k contiguous not above 1500
    // in fp64, 1000 where several items read columns of their own (227 items of 7 x 3460 with eight 32 -> 63).  Of 22000 products with one to eight columns
    // and 16 to 256 whole blocks 2.2 % were 7 % or more slower split without this line, 0.6 % with it.
    const int64_t whole = (int64_t)((M + per - 1) / per) * batch;
    const int64_t all = (int64_t)M * batch, most = !rows ? 10240 : (sizeof(T) == 4 ? 2048 : (batch == 1 || N == 1 ? 1500 : 1000));
    const bool split = whole < 256 && all <= most && (rows ? K >= 2048 && K >= 12 * whole : K >= 64 && 2 * K >= whole);
    const int tiles = split ? (M + few - 1) / few : (M + per - 1) / per;
    const int64_t blocks = (int64_t)tiles * batch;
    if (blocks > 0x7fffffffll)
        return LA_ERR_UNSUPPORTED;
#define LA_GEMV(N_, SPLIT_, ADD_)                                                                                        \
    LA_LAUNCH((k_gemv<T, N_, SPLIT_, ADD_>), dim3((unsigned)blocks), dim3(GEMV_THREADS), 0, st, A, B, C, batch, M, K, alpha, beta, \
              triA, tiles, add)
#define LA_GO(N_)                   \
    case N_:                        \
        if (split)                  \
            LA_GEMV(N_, true, false);  \
        else                        \
            LA_GEMV(N_, false, false); \
        break
    if (add) {  // (launch_gemv_add: one column)
        if (split)
            LA_GEMV(1, true, true);
        else
            LA_GEMV(1, false, true);
        return launch_check("gemv");
    }
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
#undef LA_GEMV
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

// y = beta c + alpha A x for one item (A M x K, triA as in GemmOpts; beta = 0: c is not read), y not one of the others
template <typename T>
la_status launch_gemv_add(View<const T> A, const T *x, const T *c, T *y, int M, int K, T alpha, T beta, int triA, hipStream_t st)
{
    if (M <= 0)
        return LA_OK;
    if (dry_run())
        return LA_OK;
    return launch_gemv<T>(A, View<const T>{x, K, 1, 1}, View<T>{y, M, 1, 1}, 1, M, 1, K, alpha, beta, triA, st, c);
}
template la_status launch_gemv_add<float>(View<const float>, const float *, const float *, float *, int, int, float, float, int, hipStream_t);
template la_status launch_gemv_add<double>(View<const double>, const double *, const double *, double *, int, int, double, double, int, hipStream_t);

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

// Bytes of LDS: no more buffers than slabs.
template <typename T, int BM, int BN, int BKB, int NB>
static size_t gemm_lds(int K, bool sym)
{
    const size_t slab = (size_t)(BM + BN) * BKB;
    const size_t slabs = ((size_t)K * sizeof(T) + BKB - 1) / BKB * (sym ? 2 : 1);
    return std::max(std::min(slabs, (size_t)NB) * slab, sym ? 4 * (BM / 2) * (BN / 2 + 1) * sizeof(T) : 0);
}

struct GemmForm {
    bool akf, bkf;  // k is the contiguous index of A, of B
    bool rag;       // some chunk is unaligned or incomplete
};

// Workgroups of a launch with tiles of BM x BN; chooses the tiles' order.
template <int BM, int BN>
static dim3 gemm_grid(int64_t batch, int M, int N, GemmOpts &o, int &tiles_m, int &tiles_n)
{
    tiles_m = (M + BM - 1) / BM;
    tiles_n = (N + BN - 1) / BN;
    o.order = pick_order(o, tiles_m, tiles_n);
    const int64_t per = tile_count(o.order, tiles_m, tiles_n);
    // (an XCD takes whole items: not the slices of a split K range where that leaves some with a slice more than others, 14 of 500 x 500 x 9568 in
    // the sparse GP 90 -> 78 us)
    o.xcd_batch = (batch >= 8 && per > 1 && (o.ksplit <= 1 || (8 - (batch & 7)) % 8 * 8 <= batch)) ? 1 : 0;
    return dim3((unsigned)(o.xcd_batch ? 8 * ((batch + 7) / 8) * per : per * batch));
}

// (the symmetric sum exists for tiles up to 64, launch_gemm picks them, and its operands have mirrored strides, so akf == bkf)
#define LA_FORMS(GO)                       \
    if constexpr (BM <= 64) {              \
        if (o.symsum) {                    \
            if (f.akf)                     \
                GO(true, true, true);      \
            else                           \
                GO(false, false, true);    \
            return;                        \
        }                                  \
    }                                      \
    if (f.akf && f.bkf)                    \
        GO(true, true, false);             \
    else if (f.akf)                        \
        GO(true, false, false);            \
    else if (f.bkf)                        \
        GO(false, true, false);            \
    else                                   \
        GO(false, false, false)

template <typename T, int BM, int BN, int BKB, int NB = 2>
static void launch_tiles(GemmForm f, View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int N, int K,
                         T alpha, T beta, GemmOpts o, hipStream_t st)
{
    int tiles_m, tiles_n;
    const dim3 grid = gemm_grid<BM, BN>(batch, M, N, o, tiles_m, tiles_n);
#define LA_GO(AK, BKF_, SYM_)                                                                                                       \
    LA_LAUNCH((k_gemm<T, BM, BN, BKB, NB, AK, BKF_, SYM_>), grid, dim3(256), (gemm_lds<T, BM, BN, BKB, NB>(K, SYM_)), st, A, B, C, batch, M, \
              N, K, alpha, beta, o, tiles_m, tiles_n)
    LA_FORMS(LA_GO);
#undef LA_GO
}

template <typename T, int BM, int BN, int BK, int NBUF>
static void launch_staged(GemmForm f, View<const T> A, View<const T> B, View<T> C, int64_t batch, int M, int N, int K,
                          T alpha, T beta, GemmOpts o, hipStream_t st)
{
    int tiles_m, tiles_n;
    const dim3 grid = gemm_grid<BM, BN>(batch, M, N, o, tiles_m, tiles_n);
#define LA_GO(AK, BKF_, SYM_)                                                                                                               \
    LA_LAUNCH((k_gemm_staged<T, BM, BN, BK, NBUF, AK, BKF_, SYM_>), grid, dim3(256), 0, st, A, B, C, batch, M, N, K, alpha, beta, o, tiles_m, \
              tiles_n)
    LA_FORMS(LA_GO);
#undef LA_GO
}
#undef LA_FORMS

// Time of a product in e x e tiles, in us beyond what every launch costs.  A tile takes its matrix instructions (at 2.1 GHz, the clock the chip
// holds under them; small tiles also wait for L2) and a part that nothing overlaps with; a compute unit holds 5, 4 or 2 workgroups at a time, and
// however few there are, a workgroup's slabs follow each other at the latency of memory.  Fitted to 2300 products of 16 to 8192 rows, columns
// and K, uniform and triangular: the tile taken is 0.6 % slower than the best of the three on average.  us, 32 x 32 /
// 64 x 64 / 128 x 128 tiles, fp64: 32 x 128^3 7.2 / 9.0 / 21, 32 x 256^3 26 / 23.5 / 38, 2048^2 x 128 30 / 22.8 / 25, 500 x 9568 x 500 107 / 92 / 132,
// 32 x 512^3 171 / 138 / 132, 3001 x 1024 x 2000 238 / 205 / 256, 4096^3 2540 / 2070 / 1965.
template <typename T>
static double tile_cost(int e, int64_t wgs, int K, const GemmOpts &o)
{
    const bool f32 = sizeof(T) == 4;
    const double g = e == 128 ? 1.0 : (e == 64 ? (f32 ? 1.13 : 1.05) : (f32 ? 1.36 : 1.44));
    const double fixed = e == 128 ? (f32 ? 3.0 : 1.2) : (e == 64 ? (f32 ? 0.25 : 0.3) : 0.32);
    const int held = e == 128 ? 2 : (e == 64 ? 4 : 5), bk = (e == 32 ? 256 : 128) / (int)sizeof(T), passes = o.symsum == 1 ? 2 : 1;
    const double matrix = 2e-6 * e * e * ((K + 15) / 16 * 16) * passes / (f32 ? 0.536 : 0.268);  // a tile over the whole K range
    const double latency = (double)((K + bk - 1) / bk) * passes * (f32 ? 0.46 : 0.63);
    const int tri = (o.triA != 0) + (o.triB != 0);
    if (tri == 0) {
        const double tile = matrix * g + fixed, chain = latency + matrix + fixed;
        const int64_t n = (wgs + 255) / 256;
        return (double)(n / held) * std::max(held * tile, chain) + (n % held ? std::max((double)(n % held) * tile, chain) : 0.0);
    }
    // triangular operands: part of the K range on average, the heaviest tiles first, and part of a tile at the end that does not even out
    const double n = (double)wgs / 256.0, share = tri == 1 ? 0.455 : 0.3, whole = f32 ? 0.74 : 0.87;
    return std::max(n * (matrix * g * share + fixed), whole * (latency + matrix) + fixed) + (n > 1.0 ? (f32 ? 0.26 : 0.35) * (matrix * g + fixed) : 0.0);
}

// Tiles of ragged products: the largest that still fill the chip.
template <typename F>
static int staged_edge(F &&wgs, int64_t batch, int M, int N, int K, bool k64, const GemmOpts &o)
{
    const int64_t wg128 = wgs(128), wg64 = wgs(64);
    // No 128 x 128 tiles where they stick out of C by a quarter more than tiles of 64 do: 130 products of 129 x 129 x 129 79 -> 41 us in fp64,
    // 40 -> 22 in fp32, 300 times trmm of 131 with 131 vectors 135 -> 68 and 73 -> 35; 383 x 383 (144 tiles against 180 quarters) is the same in both.
    const bool padded = (int64_t)((M + 127) / 128) * ((N + 127) / 128) * 16 > (int64_t)((M + 63) / 64) * ((N + 63) / 64) * 5;
    int e;
    if (o.triA | o.triB) {
        // Triangular operands make the K range, hence the time, of a tile vary along the tile list (heaviest first): the 512 workgroup slots only
        // fill evenly if there are several rounds of tiles, so take the largest tile that still gives 1024 workgroups.
        e = wg128 >= 1024 && !padded ? 128 : ((wg64 >= 1024 || !k64 || o.min_tile64) ? 64 : 32);
    } else {
        // Equal tiles: big tiles once they (nearly) fill the 512 workgroup slots, quarter tiles while 64 x 64 tiles would fill them less than twice --
        // with so few rounds the last one runs part empty.  Up to K = 32 writing C is most of the work, and more, smaller workgroups overlap it with
        // their loads (83 items of 1033 x 251, K = 2, fp64 48 -> 39 us, K = 32 72 -> 58, fp32 28 -> 25 and 37 -> 32).
        const int64_t t128 = o.maskC ? wg128 : (int64_t)((M + 127) / 128) * ((N + 127) / 128) * batch;
        const bool big = K > 32 && (o.maskC ? (M >= 2048 && N >= 2048) : (M >= 128 && N >= 128));
        // Two nearly full rounds of 64 x 64 tiles are better than quarter tiles that save no padding: the chunks' address arithmetic counts (b items
        // of 61 x 174, K = 147, us, 32 x 32 -> 64 x 64: b = 331, 993 tiles, fp64 60 -> 44, fp32 29 -> 22; with one round and a half the products of
        // potri's backward rule, 30 x 297 x 297, 220 -> 232; 26 x 2478 x 22, 1014 tiles that the quarters halve, fp32 36 -> 54).
        const bool two_rounds = !o.maskC && !o.symsum && wg64 >= 960 &&
                                (int64_t)((M + 63) / 64) * ((N + 63) / 64) * 4 == (int64_t)((M + 31) / 32) * ((N + 31) / 32);
        e = (t128 >= (o.maskC ? 512 : 480) && big && !padded) ? 128 : ((wg64 < 1024 && k64 && !o.min_tile64 && !two_rounds) ? 32 : 64);
    }
    return o.symsum && e == 128 ? 64 : e;  // (the form that stores both triangles has tiles up to 64 only)
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
        t.padA = o.padB;
        t.padB = o.padA;
        return launch_gemm<T>(B.t(), A.t(), C.t(), batch, N, M, K, alpha, beta, t, st);
    }
    constexpr int VW = Mfma<T>::VW;
    GemmForm f;
    f.akf = (A.cs == 1);
    f.bkf = (B.rs == 1);
    if ((!f.akf && A.rs != 1) || (!f.bkf && B.cs != 1))
        return LA_ERR_UNSUPPORTED;  // (no operator of the library builds such a view)
    const bool a_ok = aligned16<T>(A, f.akf ? A.rs : A.cs) && (o.padA || (f.akf ? K : M) % VW == 0);
    const bool b_ok = aligned16<T>(B, f.bkf ? B.cs : B.rs) && (o.padB || (f.bkf ? K : N) % VW == 0);
    f.rag = !(a_ok && b_ok);
    const int64_t longest = std::max(std::max(std::max(A.rs, A.cs), std::max(B.rs, B.cs)), std::max(C.rs, C.cs));
    if (longest >= (int64_t)1 << 22)  // (k_gemm's offsets inside a tile have 32 bits)
        f.rag = true;
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
        const int64_t wg64 = wgs(64);
        if (!o.triA && !o.triB && !o.min_tile64 && !o.ksplit && !o.symsum && wg64 <= 128 && K >= 2048 && A.nb2 == 1 && B.nb2 == 1 &&
            C.nb2 == 1) {
            int splits = (int)std::min<int64_t>(512 / wg64, K / 256);
            const int Kc = (((K + 15) / 16 + splits - 1) / splits) * 16;
            splits = (K + Kc - 1) / Kc;
            const size_t bytes = (size_t)batch * splits * M * N * sizeof(T);
            // (an unaligned or odd-sized product goes without the split where the caller gave no memory for it)
            if (splits >= 2 && bytes <= SPLITK_MAX_BYTES && ((K % 16 == 0 && a_ok && b_ok && !o.split_if_room) || arena_room(bytes))) {
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
                if (f.rag)
                    launch_staged<T, 64, 64, 16, 2>(f, As, Bs, Ps, batch * splits, M, N, Kc, T(1), T(0), ps, st);
                else
                    launch_tiles<T, 64, 64, 128>(f, As, Bs, Ps, batch * splits, M, N, Kc, T(1), T(0), ps, st);
                LA_TRY(launch_check("gemm_splitk"));
                const int64_t total = batch * mn;
                LA_LAUNCH((k_splitk_reduce<T>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                                   (const T *)buf, C, batch, M, N, splits, alpha, beta, o);
                return launch_check("splitk_reduce");
            }
        }
        // ragged: K slabs of 64, or 32, unless much of the last one would be empty
        const bool k64 = K >= 128 || (K & 63) == 0 || (K & 63) > 32;
        int e = o.min_tile64 ? 64 : 32;
        if (f.rag) {
            e = staged_edge(wgs, batch, M, N, K, k64, o);
        } else {
            double least = 0;
            for (int c = e, first = c; c <= (o.symsum ? 64 : 128); c *= 2) {
                const double cost = tile_cost<T>(c, wgs(c), K, o);
                if (c == first || cost < least) {
                    e = c;
                    least = cost;
                }
            }
        }
        auto launch = [&](View<const T> A_, View<T> C_, int m, int n, GemmOpts op) {
            if (f.rag) {
                if (e == 128)
                    launch_staged<T, 128, 128, 16, 2>(f, A_, B, C_, batch, m, n, K, alpha, beta, op, st);
                else if (e == 32)
                    launch_staged<T, 32, 32, 64, 1>(f, A_, B, C_, batch, m, n, K, alpha, beta, op, st);
                else if (k64)  // (slabs of 64 in one buffer hold two workgroups a compute unit, of 32 four)
                    launch_staged<T, 64, 64, 32, 1>(f, A_, B, C_, batch, m, n, K, alpha, beta, op, st);
                else
                    launch_staged<T, 64, 64, 16, 2>(f, A_, B, C_, batch, m, n, K, alpha, beta, op, st);
            } else if (e == 128) {
                launch_tiles<T, 128, 128, 128>(f, A_, B, C_, batch, m, n, K, alpha, beta, op, st);
            } else if (sizeof(T) == 4 && e == 32 && wgs(32) > 1024) {
                // one LDS buffer: eight workgroups a compute unit instead of five (1000 to 4500 tiles, 64 < K <= 512, 4 to 9 % faster, fewer tiles 1 to
                // 5 % slower)
                launch_tiles<T, 32, 32, 256, sizeof(T) == 4 ? 1 : 2>(f, A_, B, C_, batch, m, n, K, alpha, beta, op, st);
            } else if (e == 32) {
                launch_tiles<T, 32, 32, 256>(f, A_, B, C_, batch, m, n, K, alpha, beta, op, st);
            } else if (sizeof(T) == 4 && K <= 128 && wg64 > 1024) {
                // one LDS buffer: short products of many tiles are bound by C, more workgroups a compute unit (fp32, K <= 64, above 2048 tiles:
                // 4 to 6 % faster on average; above K = 128 up to 5 % slower)
                launch_tiles<T, 64, 64, 128, sizeof(T) == 4 ? 1 : 2>(f, A_, B, C_, batch, m, n, K, alpha, beta, op, st);
            } else {
                launch_tiles<T, 64, 64, 128>(f, A_, B, C_, batch, m, n, K, alpha, beta, op, st);
            }
            return launch_check("gemm");
        };
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
                LA_TRY(launch(A.sub(e, 0), C.sub(e, 0), M - e, N - e, lo));
                return launch_gemm<T>(A.level2((int64_t)e * A.rs, (int)Tt), B.level2((int64_t)e * B.cs, (int)Tt),
                                      C.level2((int64_t)e * (C.rs + C.cs), (int)Tt), batch * Tt, e, e, K, alpha, beta, o, st);
            }
        }
        return launch(A, C, M, N, o);
    }
}

template la_status launch_gemm<float>(View<const float>, View<const float>, View<float>, int64_t, int, int, int, float,
                                      float, GemmOpts, hipStream_t);
template la_status launch_gemm<double>(View<const double>, View<const double>, View<double>, int64_t, int, int, int,
                                       double, double, GemmOpts, hipStream_t);

}  // namespace la
