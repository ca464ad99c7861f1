// C ABI of the library (see include/la.h) and the host-side blocked algorithms.
//
// Everything is phrased on a LOGICAL lower-triangular factor Lam: a lower factor is the
// row-major view of the caller's buffer, an upper factor R = Lam^T (appendix of arXiv
// 1710.08717, "potrf", last paragraph, and the R variants of trsm / trmm) is the transposed
// view of the same memory, so no data is ever transposed or copied for it.
//
// potrf / backward of small matrices are single register-resident kernels, blocks of up to 128
// rows one-workgroup kernels that keep the block in LDS.  Everything larger is host code over
// those and GEMMs on the matrix cores: off-diagonal updates, products with (masked) triangular
// blocks, and solves as products with explicit inverses of diagonal blocks (128 x 128 blocks by
// one launch for the whole batch, merged level by level where larger ones are wanted).
// The library owns no device memory: scratch comes out of the workspace the caller passes to the
// _ws form of an entry point (la_workspace_bytes says how much a call takes).
#include <cstdio>
#include <cstring>
#include <mutex>

#include "common.hpp"

namespace la {

static thread_local char g_err[256] = "no error";

void set_error(hipError_t e, const char *where)
{
    snprintf(g_err, sizeof(g_err), "%s: %s", where, hipGetErrorString(e));
}

// ---------------------------------------------------------------------------------
// Scratch memory (see common.hpp): the arena of the call that is running on this thread.
// ---------------------------------------------------------------------------------
Arena *&current_arena()
{
    static thread_local Arena *a = nullptr;
    return a;
}

la_status arena_take(size_t bytes, void **out)
{
    Arena *a = current_arena();
    const size_t need = (bytes + 255) & ~(size_t)255;
    if (!a || (!a->dry && a->used + need > a->cap)) {
        snprintf(g_err, sizeof(g_err), "workspace too small: %zu more bytes wanted at offset %zu of %zu", need,
                 a ? a->used : (size_t)0, a ? a->cap : (size_t)0);
        return LA_ERR_WORKSPACE;
    }
    *out = a->base + a->used;
    a->used += need;
    if (a->used > a->peak)
        a->peak = a->used;
    return LA_OK;
}

bool arena_room(size_t bytes)
{
    const Arena *a = current_arena();
    if (!a)
        return false;
    if (a->dry)
        return !a->needed_only;
    return a->used + ((bytes + 255) & ~(size_t)255) <= a->cap;
}

// The most scratch that `op` takes at a time, found by a run that launches nothing; needed_only: without what arena_room offers.
template <class F>
static la_status sizing_pass(F &&op, size_t *peak, bool needed_only = false)
{
    Arena a;
    a.dry = true;
    a.needed_only = needed_only;
    a.base = reinterpret_cast<char *>((uintptr_t)1 << 46);  // never dereferenced
    Arena *prev = current_arena();
    current_arena() = &a;
    const la_status s = op();
    current_arena() = prev;
    *peak = a.peak;
    return s;
}

template <typename T>
static la_status scratch_views(int64_t batch, int n, int count, View<T> *out, int ld = 0)
{
    // `count` row-major n x n matrices per batch item, each batch-contiguous, rows ld apart (0: n)
    ld = ld ? ld : n;
    const int64_t nn = (int64_t)n * ld;
    void *p = nullptr;
    LA_TRY(arena_take((size_t)count * batch * nn * sizeof(T), &p));
    for (int c = 0; c < count; ++c)
        out[c] = View<T>{(T *)p + (int64_t)c * batch * nn, nn, ld, 1};
    return LA_OK;
}

// Rows of n elements, padded to whole 16-byte chunks.
template <typename T>
static inline int padded(int n)
{
    constexpr int VW = 16 / (int)sizeof(T);
    return (n + VW - 1) / VW * VW;
}

// Is there room for `squares` working matrices per item with padded rows, and `more` bytes?  Not above 8 GiB a matrix (one of n = 32768 in fp64): the call
// would run in less, and la_workspace_bytes counts what is taken here, which must not keep a problem off the card that fits on it otherwise (n = 80001:
// operands and workspace of potrf 256 GB without the copies, 307 with them; of its gradient 154 and 257).  At the limit, n = 32001, the copies gain
// what they do below: fp64 / fp32, ms, potrf 209 -> 187 / 107 -> 102, its gradient 398 -> 366 / 215 -> 189.
constexpr size_t PADDED_MAX_BYTES = (size_t)8 << 30;
template <typename T>
static bool padded_room(int64_t batch, int n, int squares, size_t more = 0)
{
    const int ld = padded<T>(n);
    const size_t square = (size_t)batch * n * ld * sizeof(T);
    return ld != n && square <= PADDED_MAX_BYTES && arena_room(squares * square + more);
}

// Rough time, per unit of K, of the lower-triangle update C -= P P^T on n2 rows: the product
// kernel runs two workgroups per compute unit (512 slots), with 128 x 128 tiles from 2048 rows on
// and 64 x 64 tiles below, and a launch costs whole rounds of tiles: 528 tiles take twice as long
// as 496.  (Relative figures measured on this kernel: a full round, a round that leaves half of
// the compute units with a single workgroup.)
static double lower_update_cost(int n2)
{
    const bool big = n2 >= 2048;
    const int e = big ? 128 : 64;
    const int64_t t = (n2 + e - 1) / e, c = t * (t + 1) / 2;
    const double full = big ? 0.30 : 0.11, half = big ? 0.18 : 0.06;
    const int64_t rounds = c / 512, rem = c % 512;
    return rounds * full + (rem > 256 ? full : (rem > 0 ? half : 0.0));
}

static inline int split_point(int n)
{
    // first part: a multiple of the tile edge (of 128 for larger n), about half of n, always < n
    // for n > NB; moved up by at most n / 8 if that lets the trailing update run in full rounds
    const int step = n >= 512 ? 2 * NB : NB;
    const int h = (n / 2 + step - 1) / step * step;
    if (n < 2048)
        return h;
    int best = h;
    double best_score = lower_update_cost(n - h) / ((double)(n - h) * (n - h));
    for (int n1 = h + step; n1 <= h + n / 8 && n1 < n; n1 += step) {
        const double score = lower_update_cost(n - n1) / ((double)(n - n1) * (n - n1));
        if (score < 0.95 * best_score) {
            best = n1;
            best_score = score;
        }
    }
    return best;
}

template <typename T>
static inline View<const T> cv(View<T> v)
{
    return {v.p, v.bs, v.rs, v.cs, v.bs2, v.nb2};
}

// ---------------------------------------------------------------------------------
// Explicit inverse of a lower-triangular Lam (n x n) into Inv (n x n, lower triangle; what lies
// above the diagonal is never written and never read).  First the 128 x 128 diagonal blocks (one
// launch for the whole batch), then level by level
//     inv [A 0; C D] = [A^-1 0; -D^-1 C A^-1, D^-1]
// with all pairs of one level in one batched GEMM pair.  Stops when blocks of `upto` are
// inverted (upto >= n: the whole matrix).  Tmp: scratch of at least n*n/2 per item.
// pad: Inv's rows are padded (GemmOpts::padA), with 2 Lam's too.
// ---------------------------------------------------------------------------------
template <typename T>
static la_status inverse_merge(View<const T> Lam, View<T> Inv, View<T> Tmp, int64_t batch, int n, int upto,
                               hipStream_t st, int pad = 0);

template <typename T>
static la_status inverse_build(View<const T> Lam, View<T> Inv, View<T> Tmp, int64_t batch, int n, int upto,
                               hipStream_t st, int pad = 0)
{
    LA_TRY(launch_tri_inverse128<T>(Lam, Inv, batch, n, st));
    return inverse_merge<T>(Lam, Inv, Tmp, batch, n, upto, st, pad);
}

// The merge levels of inverse_build alone: Inv already holds the inverses of the 128 x 128 diagonal blocks.
template <typename T>
static la_status inverse_merge(View<const T> Lam, View<T> Inv, View<T> Tmp, int64_t batch, int n, int upto,
                               hipStream_t st, int pad)
{
    for (int64_t h = 2 * NB; h < upto && h < n; h *= 2) {
        const int nfull = (int)(n / (2 * h));                       // pairs whose right block is a full h
        const int r = (int)(n - (int64_t)nfull * 2 * h - h);        // rows of a ragged right block (if > 0)
        for (int pass = 0; pass < 2; ++pass) {
            const int cnt = pass == 0 ? nfull : (r > 0 ? 1 : 0);
            if (cnt == 0)
                continue;
            const int64_t o0 = pass == 0 ? 0 : (int64_t)nfull * 2 * h;  // first row of the first pair
            const int mr = pass == 0 ? (int)h : r;
            View<const T> A = cv(Inv).sub(o0, o0).level2(2 * h * (Inv.rs + Inv.cs), cnt);
            View<const T> D = cv(Inv).sub(o0 + h, o0 + h).level2(2 * h * (Inv.rs + Inv.cs), cnt);
            View<const T> C = Lam.sub(o0 + h, o0).level2(2 * h * (Lam.rs + Lam.cs), cnt);
            View<T> O = Inv.sub(o0 + h, o0).level2(2 * h * (Inv.rs + Inv.cs), cnt);
            View<T> Tv{Tmp.p + (pass == 0 ? 0 : (int64_t)nfull * h * h), Tmp.bs, h, 1, h * h, cnt};
            GemmOpts o1, o2;
            o1.triA = 1;     // D^-1 is lower triangular: the K range grows with the tile row,
            o1.reverse = 1;  //   so the last rows go first
            o2.triB = 1;     // A^-1 is lower triangular: the K range shrinks with the tile column
                             //   (the launcher enumerates such tiles column by column)
            o1.padA = pad != 0;
            o1.padB = pad == 2;
            LA_TRY(launch_gemm<T>(D, C, Tv, batch * cnt, mr, (int)h, mr, T(1), T(0), o1, st));
            LA_TRY(launch_gemm<T>(cv(Tv), A, O, batch * cnt, mr, (int)h, (int)h, T(-1), T(0), o2, st));
        }
    }
    return LA_OK;
}

// ---------------------------------------------------------------------------------
// Right-looking blocked potrf with panels of 128 columns: per panel one leaf launch (factor and
// inverse of the diagonal block), one product for the rows below (L21 = A21 Li11^T) and one for
// the trailing lower triangle.  No merged inverses, so fewer launches than the recursion for a
// stand-alone problem of a few panels; every update has K = 128 only, which is why large
// matrices take the recursion.
// ---------------------------------------------------------------------------------
template <typename T>
static la_status potrf_right_looking(View<T> Wk, View<T> L, int32_t *info, int off, int64_t batch, int n, View<T> Inv,
                                     bool need_inv, bool pad, hipStream_t st)
{
    constexpr int P = 2 * NB;
    for (int o = 0; o < n; o += P) {
        const int nb = n - o < P ? n - o : P, r = n - o - nb;
        // (nothing below the last block is solved with it: no inverse unless the caller merges them)
        const View<T> inv = r > 0 || need_inv ? Inv.sub(o, o) : View<T>{nullptr, 0, 0, 0};
        LA_TRY(launch_potrf_leaf16<T>(cv(Wk).sub(o, o), L.sub(o, o), inv, info, off + o, batch, nb, false, st));
        if (r == 0)
            break;
        View<T> L21 = L.sub(o + nb, o);
        GemmOpts op, ou;
        op.padA = op.padB = ou.padA = ou.padB = pad;
        op.triB = 2;  // Li11^T is upper triangular
        LA_TRY(launch_gemm<T>(cv(Wk).sub(o + nb, o), cv(Inv).sub(o, o).t(), L21, batch, r, nb, nb, T(1), T(0), op, st));
        ou.maskC = 1;
        LA_TRY(launch_gemm<T>(cv(L21), cv(L21).t(), Wk.sub(o + nb, o + nb), batch, r, r, nb, T(-1), T(1), ou, st));
    }
    return LA_OK;
}

// ---------------------------------------------------------------------------------
// Blocked potrf by recursive halving (section 4.2: A = L L^T).  Wk holds the lower triangle of
// the block still to be factored (a working copy, updated in place), L receives the factor, Inv
// the inverses of the factors of the diagonal sub-blocks; off is the index of the block's first
// row in the whole matrix.
//   [A11 . ; A21 A22]:  L11, Li11 = rec(A11);  L21 = A21 Li11^T;  A22 -= L21 L21^T;  L22 = rec(A22)
// Every panel solve is ONE product with the explicit inverse of the left factor, so a left
// child always returns its complete inverse, merged from its own children's by
//   Li21 = -Li22 (L21 Li11)
// (need_inv; a right child needs it only if its parent does).  The extra products add one sixth
// to the n^3 / 3 of the factorisation and remove every recursive solve.  The temporary
// L21 Li11 lives in the unused upper-right block of the node's part of Inv.
// The halving stops at blocks of about 2000 rows, which are factored panel by panel
// (potrf_right_looking) and, where the parent needs it, inverted level by level with all pairs
// of a level in one launch (inverse_merge, temporary in Tmp): the long dependent chain of small
// launches at the bottom of the recursion is what a large factorisation waits for.
// ---------------------------------------------------------------------------------
template <typename T>
static la_status potrf_rec(View<T> Wk, View<T> L, int32_t *info, int off, int64_t batch, int n, View<T> Inv,
                           View<T> Tmp, bool need_inv, bool pad, hipStream_t st)
{
    if (n <= 2 * NB)  // factor and inverse in one launch
        return launch_potrf_leaf16<T>(cv(Wk), L, need_inv ? Inv : View<T>{nullptr, 0, 0, 0}, info, off, batch, n, false, st);
    // Blocks of up to 2304 rows: panel by panel.  Measured against halving all the way down: one matrix
    // of n = 2048 0.95 -> 0.77 ms, 3000 1.78 -> 1.38, 4096 2.58 -> 2.19, 8192 8.62 -> 7.89 (fp64); with many
    // matrices in the batch the short products of the panels stop paying (32 x 1024: 0.91 -> 0.93).
    if (n <= 2304 && (double)batch * n * n < 24e6) {
        LA_TRY(potrf_right_looking<T>(Wk, L, info, off, batch, n, Inv, need_inv, pad, st));
        return need_inv ? inverse_merge<T>(cv(L), Inv, Tmp, batch, n, n, st, pad ? 2 : 0) : LA_OK;
    }
    const int n1 = split_point(n), n2 = n - n1;
    View<T> L21 = L.sub(n1, 0), Wk22 = Wk.sub(n1, n1);
    LA_TRY(potrf_rec<T>(Wk, L, info, off, batch, n1, Inv, Tmp, true, pad, st));
    GemmOpts op, ou, o1, o2;
    op.padA = op.padB = ou.padA = ou.padB = o1.padA = o1.padB = o2.padA = o2.padB = pad;
    op.triB = 2;  // Li11^T is upper triangular
    LA_TRY(launch_gemm<T>(cv(Wk).sub(n1, 0), cv(Inv).t(), L21, batch, n2, n1, n1, T(1), T(0), op, st));
    ou.maskC = 1;  // trailing update of the lower triangle: A22 -= L21 L21^T
    LA_TRY(launch_gemm<T>(cv(L21), cv(L21).t(), Wk22, batch, n2, n2, n1, T(-1), T(1), ou, st));
    LA_TRY(potrf_rec<T>(Wk22, L.sub(n1, n1), info, off + n1, batch, n2, Inv.sub(n1, n1), Tmp, need_inv, pad, st));
    if (!need_inv)
        return LA_OK;
    View<T> T1 = Inv.sub(0, n1).t();  // n2 x n1 temporary in the upper-right block
    o1.triB = 1;  // Li11 is lower triangular: the K range shrinks with the tile column
    LA_TRY(launch_gemm<T>(cv(L21), cv(Inv), T1, batch, n2, n1, n1, T(1), T(0), o1, st));
    o2.triA = 1;  // Li22 is lower triangular: the K range grows with the tile row
    o2.reverse = 1;
    return launch_gemm<T>(cv(Inv).sub(n1, n1), cv(T1), Inv.sub(n1, 0), batch, n2, n1, n2, T(-1), T(0), o2, st);
}

// ---------------------------------------------------------------------------------
// Pieces of the potrf backward expression (section 4.2; appendix "potrf"):
//   Abar = sym( Lam^-T Phi(Lam^T Lbar) Lam^-1 ),  Phi = lower triangle, halved diagonal.
// ---------------------------------------------------------------------------------

// With the explicit inverse Li of the factor the whole expression is three masked GEMMs whose
// K ranges skip every structural zero (5 n^3 / 3 flops in all, inverse included):
//   P = Phi(tril(Lam^T Lbar))      lower x lower, lower part kept, diagonal halved
//   Z = P Li                       lower x lower = lower
//   Abar = 1/2 (W + W^T), W = Li^T Z (upper x lower = full): the lower tiles of Li^T Z + Z^T Li, mirrored
template <typename T>
static la_status backward_sweep(View<const T> Lam, View<const T> G, View<T> W, int64_t batch, int n, int n0, bool aliased,
                                hipStream_t st);

// Block columns of the reverse sweep, 0 where the inverse-based expression takes the whole matrix.  The expression's 5 n^3 / 3 flops run
// in a few large products, the sweep's 2 n^3 / 3 and n0^3 per block in many smaller, dependent ones: with columns of 256 and more it pays
// from about 4 Mi matrix elements over the whole batch (fp32: 8 Mi), with columns of 128 from 12 Mi (24 Mi).  Expression -> sweep, us:
// 256, fp64 18 x 512^2 226 -> 195, 32 x 512^2 294 -> 240, 13 x 512^2 170 -> 166, 100 x 400^2 494 -> 482, 60 x 333^2 252 -> 252, fp32 32 x 512^2
// 178 -> 153, 18 131 -> 131, 100 x 400^2 276 -> 270; 512, fp64 4 x 1024^2 279 -> 259 (3: 224 -> 229), fp32 8 x 1024^2 278 -> 218, 4 161 -> 175;
// 128, fp64 300 x 222^2 420 -> 398, 200 x 250^2 345 -> 342, 80 x 333^2 292 -> 306, fp32 400 x 256^2 358 -> 292, 300 x 222^2 225 -> 238,
// 150 x 333^2 292 -> 280.  n0 = 256 / 512 / 1024: fp64 8 x 1024^2 401 / 343 / -, 4 x 2048^2 1146 / 941 / 966, 1 x 3001^2 1509 / 1082 / 898
// (2048: 909), 30 x 640^2 391 / 450 / -; 128 / 256: 70 x 480^2 496 / 475 and fp32 309 / 267.  Blocks of 2048 would be 4 to 6 % faster above
// n = 5000 (1 x 8192^2 fp64 8339 -> 7982, fp32 4481 -> 4210), but the errors grow with the blocks' inverses: fp32 7.5e-7 -> 1.05e-6 there
// (halving with substitutions: 9.0e-7).
constexpr int SWEEP_MIN_N = 214;
static int sweep_block(int64_t batch, int n, size_t elem)
{
    const double mi = 1048576.0, b = (double)batch, elements = b * n * n, scale = elem == 4 ? 2.0 : 1.0;
    // (n = 700 to 860 is three blocks of 256 and a bit; with up to 8 matrices, fp32 16, the items of the expression's products fill the 8 XCDs
    // evenly: 8 x 770^2 fp64 291 -> 325, 7 x 785^2 303 -> 354, 15 x 850^2 fp32 322 -> 346, from 5.5 Mi on ahead again; 9 x 737^2 427 -> 335,
    // 20 x 720^2 fp32 308 -> 269)
    const double least = n >= 700 && n < 860 && b <= 8.0 * scale ? 5.5 : 4.0;
    if (n >= 400 && b <= 128.0 && elements >= least * scale * mi) {
        int n0 = 256;
        while (n0 < 1024 && 2.0 * n0 <= 0.6 * n && 4.0 * n0 * n0 * b <= 4.0 * mi)
            n0 *= 2;
        return n0;
    }
    return n >= SWEEP_MIN_N && elements >= 12.0 * scale * mi ? 128 : 0;
}

// Elements of scratch per matrix of a sweep that keeps the inverses of `cols` columns at a time: those as a band of n0 columns, and two
// n0 x n0 blocks, in which the merges' temporary lives before.
static int64_t sweep_scratch(int n0, int64_t cols)
{
    return cols * n0 + (cols + 15) / 16 * 16 + (std::max(2 * (int64_t)n0 * n0, cols * n0 / 4) + 15) / 16 * 16;  // (every part starts a 16-byte chunk)
}

// W = 1/2 (Li^T (P + P^T) Li) for lower triangular Li and P (what lies above their diagonals is not read), both triangles
// of W, exactly symmetric.  X: scratch; W may be P.
template <typename T>
static la_status congruence(View<const T> Li, View<const T> P, View<T> X, View<T> W, int64_t batch, int n, hipStream_t st, bool pad = false)
{
    GemmOpts oz, ow;
    oz.padA = oz.padB = ow.padA = ow.padB = pad;  // the rows of Li, P and X are padded
    oz.triA = 1;
    oz.triB = 1;
    oz.maskC = 1;
    oz.reverse = 1;  // K range of tile (i, j) grows with i - j: bottom rows first
    LA_TRY(launch_gemm<T>(P, Li, X, batch, n, n, n, T(1), T(0), oz, st));
    // 1/2 (Li^T Z + Z^T Li) in one launch: the tiles on and below the diagonal accumulate both products (K range from the
    // tile's first row on) and write every entry with its mirror image
    ow.triA = 2;
    ow.triB = 1;
    ow.symsum = 1;
    return launch_gemm<T>(Li.t(), cv(X), W, batch, n, n, n, T(0.5), T(0), ow, st);
}

template <typename T>
static la_status backward_impl(View<const T> Lam, View<const T> G, View<T> W, int64_t batch, int n, bool aliased,
                               hipStream_t st)
{
    // n <= 16: 16 lanes per matrix, HBM bound; so are many matrices of n = 24.
    if (small_wave_takes<T>(SmallWaveOp::backward, batch, n))  // one wavefront per matrix
        return launch_backward_wave<T>(Lam, G, W, batch, n, st);
    if (n <= 32)
        return launch_backward_tiny<T>(Lam, G, W, batch, n, st);
    if (n <= backward_leaf16_max_n<T>())  // one workgroup per matrix, everything in LDS, no scratch
        return launch_backward_leaf16<T>(Lam, G, W, batch, n, st);
    // (the expression takes two squares; where the workspace has no room for them the sweep does with less)
    const int n0 = sweep_block(batch, n, sizeof(T));
    if (n0 > 0 || (n >= SWEEP_MIN_N && !arena_room((size_t)(2 * batch * n * n) * sizeof(T))))
        return backward_sweep<T>(Lam, G, W, batch, n, n0 > 0 ? n0 : 256, aliased, st);
    ArenaFrame frame;
    // (with room for a third square: all three with rows of whole 16-byte chunks, so that two of the three products run on aligned operands)
    View<T> sc[3];
    const int ld = padded<T>(n);
    const bool pad = padded_room<T>(batch, n, 3);
    LA_TRY(scratch_views<T>(batch, n, pad ? 3 : 2, sc, pad ? ld : n));
    View<T> Li = sc[0], X = sc[1], P = pad ? sc[2] : W;
    LA_TRY(inverse_build<T>(Lam, Li, X, batch, n, n, st, pad));
    View<const T> Gs = G;
    if (aliased) {  // Abar overwrites Lbar: keep a copy of its lower triangle
        LA_TRY(launch_copy<T>(G, X, batch, n, n, T(1), 1, st));
        Gs = cv(X);
    }
    GemmOpts o;
    o.triA = 2;  // Lam^T
    o.triB = 1;
    o.maskC = 1;
    o.halfDiag = 1;
    LA_TRY(launch_gemm<T>(Lam.t(), Gs, P, batch, n, n, n, T(1), T(0), o, st));
    return congruence<T>(cv(Li), cv(P), X, W, batch, n, st, pad);
}

template <typename T>
static la_status tri_apply_v(bool solve, bool fwd, T alpha, int64_t batch, int n, int m, View<const T> Lam,
                             View<const T> Xin, View<T> X, bool inplace, hipStream_t st);

// ---------------------------------------------------------------------------------
// Reverse sweep over the blocked factorisation (section 4.2 names differentiating the blocked algorithm itself as the cheaper
// route), block column by block column of n0 columns.  For the split
//   L11 = chol(A11),  L21 = A21 L11^-T,  S = A22 - L21 L21^T,  L22 = chol(S)
// the adjoints follow in reverse order (W holds Lbar's lower triangle on entry and the symmetric Abar on return, block by
// block, in place; W22 is finished when its turn to the left comes):
//   W21 <- W21 - 2 W22 L21                          adjoint of the update S
//   W21 <- 1/2 W21 L11^-1                           adjoint of the panel solve, halved because A21
//                                                   enters the symmetric A twice
//   W11 <- W11 - 2 tril(W21^T L21)                  the panel solve's effect on L11
//   W11 <- backward(L11, W11)                       the inverse-based expression
//   W12 <- W21^T
// 2 n^3 / 3 flops in the large products instead of 5 n^3 / 3 with the full inverse.  The inverses of all diagonal blocks are formed
// beforehand in one go; they serve the solves with L11 and the blocks' own expressions.  W21 on its way to the product with the inverse is
// kept where W12 comes in the end.
// Where the workspace is short the inverses are formed for fewer columns at a time, down to one block's, and with smaller blocks: what a call
// cannot do without grows with the batch alone, so a workspace that was sized for a larger batch serves every smaller one (full size, three
// quarters, half, least; us, fp64: 128 x 512^2 769, 791, 735, 768, 32 x 512^2 243, 258, 279, 324, 1 x 4096^2 1606, 1669, 1808, 4656).
// Against halving with an inverse (and block substitutions) of their own per block, ms, fp64 / fp32: one matrix of n = 8192 8.87 -> 8.34 /
// 4.90 -> 4.48, 4096 1.83 -> 1.60 / 1.02 -> 0.92, 3001 1.05 -> 0.90 / 0.71 -> 0.57, 1000 of n = 300 2.80 -> 2.06 / 1.51 -> 1.20.
// ---------------------------------------------------------------------------------
// Columns [o, q) of the rows [o, end); `inv` holds the inverses of the diagonal blocks of n0 from row c0 on.  A column wider than n0 has its panel
// solved block by block, from the right, and its diagonal block swept in turn.  pad: the rows of Lam and W are padded (GemmOpts::padA).
template <typename T>
static la_status sweep_column(View<const T> Lam, View<const T> inv, int c0, View<const T> G, View<T> W, View<T> X, View<T> Y, int64_t batch,
                              int o, int q, int end, int n0, bool aliased, bool pad, hipStream_t st)
{
    const int w = q - o, r = end - q;
    View<const T> L11 = Lam.sub(o, o), G11 = G.sub(o, o);
    View<T> W11 = W.sub(o, o), W21 = W.sub(q, o), W12 = W.sub(o, q);
    if (r > 0) {
        View<const T> L21 = Lam.sub(q, o);
        LA_TRY(launch_copy<T>(G.sub(q, o), W12.t(), batch, r, w, T(1), 0, st));
        if (!aliased)
            LA_TRY(launch_copy<T>(G11, W11, batch, w, w, T(1), 2, st));
        GemmOpts plain, ol, om;
        plain.split_if_room = om.split_if_room = 1;  // (the inverses had the first pick of the workspace)
        plain.padA = plain.padB = ol.padA = ol.padB = om.padA = om.padB = pad;
        LA_TRY(launch_gemm<T>(cv(W).sub(q, q), L21, W12.t(), batch, r, w, r, T(-2), T(1), plain, st));
        ol.triB = 1;
        for (int b = (w - 1) / n0 * n0; b >= 0; b -= n0) {
            const int nb = w - b < n0 ? w - b : n0, e = b + nb;
            if (e < w)  // what the blocks to the right take off (W21 holds half of their x)
                LA_TRY(launch_gemm<T>(cv(W21).sub(0, e), L11.sub(e, b), W12.t().sub(0, b), batch, r, nb, w - e, T(-2), T(1), plain, st));
            LA_TRY(launch_gemm<T>(cv(W12).t().sub(0, b), inv.sub(o + b - c0, o + b - c0), W21.sub(0, b), batch, r, nb, nb, T(0.5), T(0), ol,
                                  st));
        }
        om.maskC = 1;
        LA_TRY(launch_gemm<T>(cv(W21).t(), L21, W11, batch, w, w, r, T(-2), T(1), om, st));
        G = cv(W);
        G11 = cv(W11);
        aliased = true;
    }
    if (w > n0) {
        for (int b = (w - 1) / n0 * n0; b >= 0; b -= n0)
            LA_TRY(sweep_column<T>(Lam, inv, c0, G, W, X, Y, batch, o + b, w - b < n0 ? q : o + b + n0, q, n0, aliased, pad, st));
    } else {
        GemmOpts op;
        op.padA = op.padB = pad;
        op.triA = 2;
        op.triB = 1;
        op.maskC = 1;
        op.halfDiag = 1;
        LA_TRY(launch_gemm<T>(L11.t(), G11, X, batch, w, w, w, T(1), T(0), op, st));
        LA_TRY(congruence<T>(inv.sub(o - c0, o - c0), cv(X), Y, W11, batch, w, st, true));  // (n0 columns each)
    }
    return r > 0 ? launch_copy<T>(cv(W21).t(), W12, batch, w, r, T(1), 0, st) : LA_OK;
}

// From n = 10000 on a column of two blocks: the products with W22 and the panel's with itself get twice the columns, where those of 1024 make too few
// tiles for the chip, and the blocks' inverses, which the errors grow with, stay as they are.  One matrix, ms, fp64 / fp32, halving with
// blocks of 2048 -> columns of one block -> of two: 8192 8.87 -> 8.22 -> 8.11 / 4.90 -> 4.47 -> 4.36, 9000 12.3 -> 11.0 -> 11.7 / 6.83 -> 6.12 -> 6.41, 10000
// 16.4 -> 15.3 -> 14.1 / 9.26 -> 8.41 -> 7.67, 12288 25.3 -> 26.1 -> 24.0 / 13.5 -> 13.8 -> 12.7, 16384 55.3 -> 58.2 -> 53.3 / 28.9 -> 30.9 -> 27.9, 24000 170 ->
// 177 -> 164 / 86.6 -> 93.1 -> 84.8 (four blocks: 16384 52.4 / 27.9, 10000 14.1 / 7.7); three 12288 70.2 -> 69.8 -> 66.3, four 94.1 -> 88.4 -> 90.4.  Errors, fp32:
// 12288 8.7e-7 -> 7.6e-7 -> 7.4e-7, 24000 9.0e-7 -> 8.6e-7 -> 8.5e-7.
constexpr int SWEEP_WIDE_N = 10000, SWEEP_WIDE_BATCH = 3;
template <typename T>
static la_status backward_sweep(View<const T> Lam, View<const T> G, View<T> W, int64_t batch, int n, int n0, bool aliased,
                                hipStream_t st)
{
    ArenaFrame frame;
    // Rows that are no whole number of 16-byte chunks: with room for two more squares the sweep of one large matrix runs on copies with padded
    // rows, and its products on aligned operands.  us, fp64 / fp32, n = 2501 648 / 426 -> 621 / 426, 3001 864 / 546 -> 820 / 532, 5003
    // 2714 / 1536 -> 2328 / 1424, 7423 6844 / 3825 -> 6351 / 3613; several smaller matrices lose: 16 x 1001^2 584 / 355 -> 658 / 446, 100 x 401^2
    // 473 / 284 -> 532 / 370, 4 x 2050^2 fp32 632 -> 684.
    View<T> out = W;
    const int ld = padded<T>(n);
    const bool pad = batch == 1 && n >= 2500 && padded_room<T>(1, n, 2, (size_t)sweep_scratch(n0, n) * sizeof(T));
    if (pad) {
        View<T> sc[2];
        LA_TRY(scratch_views<T>(batch, n, 2, sc, ld));
        LA_TRY(launch_copy<T>(Lam, sc[0], batch, n, n, T(1), 2, st));
        LA_TRY(launch_copy<T>(G, sc[1], batch, n, n, T(1), 2, st));
        Lam = cv(sc[0]);
        W = sc[1];
        G = cv(W);
        aliased = true;
    }
    int cols = n;  // whole blocks, or all of them
    while (!arena_room((size_t)(batch * sweep_scratch(n0, cols)) * sizeof(T)) && (cols > n0 || n0 > 2 * NB)) {
        if (cols > n0) {
            cols = (cols / 2 + n0 - 1) / n0 * n0;
        } else {
            n0 /= 2;
            cols = n;
        }
    }
    // (one stride for all of them: the symmetric sum of two products exchanges its operands' base pointers)
    const int64_t item = sweep_scratch(n0, cols);
    void *p = nullptr;
    LA_TRY(arena_take((size_t)(batch * item) * sizeof(T), &p));
    if (!arena_room(0))  // (a sizing pass for the least: the products below take none they need)
        return LA_OK;
    View<T> Li{(T *)p, item, n0, 1}, X{Li.p + (int64_t)cols * n0 + (cols + 15) / 16 * 16, item, n0, 1}, Y{X.p + (int64_t)n0 * n0, item, n0, 1};
    const int wide = n >= SWEEP_WIDE_N && batch <= SWEEP_WIDE_BATCH && cols == n ? 2 * n0 : n0;
    for (int o = (n - 1) / wide * wide; o >= 0; o -= wide) {
        const int q = n - o < wide ? n : o + wide;
        const int c0 = o / cols * cols, cc = n - c0 < cols ? n - c0 : cols;  // the columns whose inverses are there
        if (q == c0 + cc) {
            LA_TRY(launch_tri_inverse128<T>(Lam.sub(c0, c0), Li, batch, cc, st));
            LA_TRY(inverse_merge<T>(Lam.sub(c0, c0), Li, X, batch, cc, n0, st, pad ? 2 : 1));
        }
        LA_TRY(sweep_column<T>(Lam, cv(Li), c0, G, W, X, Y, batch, o, q, n, n0, aliased, pad, st));
    }
    return pad ? launch_copy<T>(cv(W), out.cs == 1 ? out : out.t(), batch, n, n, T(1), 0, st) : LA_OK;  // (symmetric)
}

// ---------------------------------------------------------------------------------
// argument checking helpers
// ---------------------------------------------------------------------------------
static inline bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    const char *pa = (const char *)a, *pb = (const char *)b;
    return pa < pb + nb && pb < pa + na;
}
static inline size_t esize(la_dtype dt) { return dt == LA_F32 ? 4 : 8; }
static inline bool bad_dtype(la_dtype dt) { return dt != LA_F32 && dt != LA_F64; }
constexpr int MAX_N = 1 << 20;

template <typename T>
static inline View<T> tri_view(T *p, int n, int lower)
{
    const int64_t nn = (int64_t)n * n;
    return lower ? View<T>{p, nn, n, 1} : View<T>{p, nn, 1, n};
}

template <typename T>
static la_status potrf_t(int lower, int64_t batch, int n, const void *A, void *L, int32_t *info, hipStream_t st)
{
    View<const T> Av = tri_view<const T>((const T *)A, n, lower);
    View<T> Lv = tri_view<T>((T *)L, n, lower);
    if (info)
        LA_TRY(launch_fill_i32(info, batch, 0, st));
    // Many matrices of three or four tile rows: one wavefront each, or four with the tiles in LDS (against the lane-group kernels at
    // equal data volume, us: n = 41 fp32 146 -> 71, 48 57 -> 42 and fp64 161 -> 73, 56 90 -> 59, 64 56 -> 38 and 123 -> 64).
    if (small_wave_takes<T>(SmallWaveOp::potrf, batch, n))
        return launch_potrf_wave<T>(Av, Lv, info, batch, n, st);
    if (n > 32 && n <= NB)
        return launch_potrf_small16<T>(Av, Lv, info, batch, n, st);
    if (n <= 32)
        return launch_potrf_tiny<T>(Av, Lv, info, 0, batch, n, st);
    if (n <= 2 * NB)  // one leaf: it reads A and writes L directly; nobody wants the inverse
        return launch_potrf_leaf16<T>(Av, Lv, View<T>{nullptr, 0, 0, 0}, info, 0, batch, n, true, st);
    ArenaFrame frame;
    // inverses of the diagonal blocks; working copy of the lower triangle of A; temporary of the inverse merges
    // (not needed where the whole matrix is factored panel by panel without merged inverses)
    const bool outer_panels = (batch == 1 && n >= 4096) || n >= 8192;
    const bool merges = outer_panels || !(n <= 2304 && (double)batch * n * n < 24e6);
    View<T> sc[4], out = Lv;
    // Rows that are no whole number of 16-byte chunks: where the workspace has room for one more square, the factor is built in one with
    // padded rows as well, so that every product runs on aligned operands, and copied into place at the end.  One more pass over the matrix, which
    // the products of smaller ones do not make up for (step with one matrix, us: n = 3001, fp64 2270 -> 2190, n = 7423 12500 -> 11860, n = 986, fp32 440 -> 432;
    // 24 x 333^2, fp32 208 -> 214; several matrices, fp64 4 x 1001^2 608 -> 586, fp32 419 -> 424, 3 x 2049^2 1213 -> 1249).
    const int ld = padded<T>(n), squares = merges ? 3 : 2;
    const bool pad = n >= 800 && (sizeof(T) == 8 || batch == 1) && padded_room<T>(batch, n, squares + 1);
    LA_TRY(scratch_views<T>(batch, n, pad ? squares + 1 : squares, sc, pad ? ld : n));  // (at once: what arena_room was asked for)
    if (pad) {
        Lv = sc[squares];
        LA_TRY(launch_copy<T>(Av, sc[1], batch, n, n, T(1), 2, st));
    } else {
        LA_TRY(launch_tril_split<T>(Av, sc[1], Lv, batch, n, st));  // zeros above the diagonal of L
    }
    if (!merges)
        sc[2] = sc[1];  // never used
    auto finish = [&]() { return pad ? launch_copy<T>(cv(Lv), out, batch, n, n, T(1), 1, st) : LA_OK; };
    // Large matrices: right-looking over panels of 2048 columns -- the panel's diagonal block by the
    // recursion below (which factors it 128 columns at a time and merges its inverse), one product
    // for the rows under it, one for the trailing triangle (K = 2048).  Against halving all the way
    // from the top this drops the merges of the large inverses: n = 8192 7.6 -> 7.2 ms, 12288
    // 19.7 -> 17.3, 6144 4.5 -> 4.1 (fp64; other panel widths from 1024 to 4096 are slower).  Below
    // n = 4096, and for several matrices of that size, the halving is faster (3000: 1.36 against 1.39 ms).
    constexpr int outer = 2048;
    if (outer_panels) {
        View<T> Wk = sc[1], Inv = sc[0];
        for (int o = 0; o < n; o += outer) {
            const int w = n - o < outer ? n - o : outer, r = n - o - w;
            LA_TRY(potrf_rec<T>(Wk.sub(o, o), Lv.sub(o, o), info, o, batch, w, Inv.sub(o, o), sc[2], r > 0, pad, st));
            if (r == 0)
                break;
            View<T> L21 = Lv.sub(o + w, o);
            GemmOpts op, ou;
            op.padA = op.padB = ou.padA = ou.padB = pad;
            ou.split_if_room = pad;  // (the copies had the first pick of the workspace)
            op.triB = 2;  // Li^T is upper triangular
            LA_TRY(launch_gemm<T>(cv(Wk).sub(o + w, o), cv(Inv).sub(o, o).t(), L21, batch, r, w, w, T(1), T(0), op, st));
            ou.maskC = 1;
            LA_TRY(launch_gemm<T>(cv(L21), cv(L21).t(), Wk.sub(o + w, o + w), batch, r, r, w, T(-1), T(1), ou, st));
        }
        return finish();
    }
    LA_TRY(potrf_rec<T>(sc[1], Lv, info, 0, batch, n, sc[0], sc[2], false, pad, st));
    return finish();
}

// Edge of the diagonal blocks of a solve with m vectors that get an explicit inverse; block
// substitution above it.  A merge level of the inverse costs n b^2 multiply-adds per matrix whatever the
// number of vectors, a substitution step three short launches: with few vectors the merges stop paying
// early.  Measured (fp64, us; edge 256 / 512 / 1024): 32 x 512, 64 vectors 93 / 118 / 118; 8 x 1024, 64:
// 112 / 118 / 166; 4 x 2048, 128: 223 / 196 / 234; 1 x 4096, 512: 548 / 431 / 396.
static inline int solve_block(int m)
{
    int b = 256;
    while (b < 1024 && b < 4 * m)
        b *= 2;
    return b;
}

// X <- Lam^-1 X (fwd) or Lam^-T X by blocks of `edge` rows, whose explicit inverses Inv holds.  S: a panel
// that takes one block's solution (a product cannot overwrite its own operand across several tiles).
template <typename T>
static la_status block_substitution(bool fwd, int64_t batch, int n, int m, int edge, View<const T> Lam, View<const T> Inv,
                                    View<T> X, View<T> S, hipStream_t st)
{
    GemmOpts o;
    o.triA = fwd ? 1 : 2;
    o.reverse = fwd ? 1 : 0;
    const int nblk = (n + edge - 1) / edge;
    GemmOpts plain;
    for (int step = 0; step < nblk; ++step) {
        const int j = fwd ? step : nblk - 1 - step;
        const int64_t o0 = (int64_t)j * edge;
        const int nbj = (int)((n - o0) < edge ? (n - o0) : edge);
        View<const T> Ij = Inv.sub(o0, o0);
        View<T> Xj = X.sub(o0, 0);
        LA_TRY(launch_gemm<T>(fwd ? Ij : Ij.t(), cv(Xj), S, batch, nbj, m, nbj, T(1), T(0), o, st));
        if (fwd && o0 + nbj < n) {  // rows below: X -= Lam[below, j] S
            const int rest = (int)(n - o0 - nbj);
            LA_TRY(launch_gemm<T>(Lam.sub(o0 + nbj, o0), cv(S), X.sub(o0 + nbj, 0), batch, rest, m, nbj, T(-1), T(1),
                                  plain, st));
        } else if (!fwd && o0 > 0) {  // rows above: X -= Lam[j, above]^T S
            LA_TRY(launch_gemm<T>(Lam.sub(o0, 0).t(), cv(S), X, batch, (int)o0, m, nbj, T(-1), T(1), plain, st));
        }
        LA_TRY(launch_copy<T>(cv(S), Xj, batch, nbj, m, T(1), 0, st));
    }
    return LA_OK;
}

// trsm / trmm (section 4.2).  vectors: columns of A/B (left) or rows (right); X(e, v) = element e
// of vector v, so that every case is "apply Lam, Lam^T or one of their inverses to vectors".
//   trsm, 16 < n <= 64, and trmm, 32 < n <= 64: one wavefront per item, where trsm_wave_takes and trmm_wave_takes say so.
//   trsm / trmm, n <= 32 and at most 16 vectors: lane groups (two rows per lane above n = 16; a solve there only for many items).
//   trmm, n <= 128 and at most 128 vectors, from 64 items on: one workgroup per item (trmm_leaf_takes).
//   trmm, otherwise: one GEMM with the triangular operand masked.
//   trsm, n <= 128 and at most 48 vectors: one block-substitution kernel.
//   trsm, 128 < n <= 512: one launch per call, one workgroup per item and slab of 16 vectors, the
//     factor streamed from memory (launch_trsm_stream), unless many vectors meet few items.
//   trsm, n <= 128 otherwise: product (in place) with the inverse of the single diagonal block.
//   trsm, otherwise: explicit inverses of the diagonal blocks of 256 to 1024 rows (the more vectors,
//     the larger; see inverse_build); n within one block: one masked GEMM with the whole inverse,
//     else block substitution with two GEMMs per block (the block's solution goes through a scratch
//     panel because a product cannot overwrite its own operand across several tiles).
template <typename T>
static la_status tri_apply_v(bool solve, bool fwd, T alpha, int64_t batch, int n, int m, View<const T> Lam,
                             View<const T> Xin, View<T> X, bool inplace, hipStream_t st)
{
    const int64_t nm = (int64_t)n * m, nn = (int64_t)n * n;
    GemmOpts o;
    o.triA = fwd ? 1 : 2;  // Lam keeps e >= k, Lam^T keeps e <= k; the same holds for their inverses
    o.reverse = fwd ? 1 : 0;  // heavy tile rows first: the last ones for a lower operand

    if (!solve && Lam.nb2 == 1 && trmm_wave_takes<T>(batch, n, m, Xin, X))  // one wavefront per item, in place too
        return launch_trmm_wave<T>(Lam, Xin, X, batch, n, m, alpha, fwd, st);

    if (solve && Lam.nb2 == 1 && trsm_wave_takes<T>(batch, n, m, Xin, X))  // one wavefront per item, no scratch
        return launch_trsm_wave<T>(Lam, Xin, X, batch, n, m, alpha, fwd, st);

    // A multiply on many small items: one workgroup per item, Lam's lower tiles and the vectors in LDS, no scratch.
    // Up to n = 32 with at most 16 vectors the lane-group kernels below are faster; above that this one is.
    const bool leaf_mul = !solve && trmm_leaf_takes<T>(batch, n, m) && Lam.nb2 == 1 && Xin.nb2 == 1 && X.nb2 == 1;
    if (leaf_mul && (n > 32 || m > 16))
        return launch_trmm_leaf<T>(Lam, Xin, X, batch, n, m, alpha, fwd, st);

    // n <= 32 with at most 16 vectors stored as whole items back to back: G lanes per matrix.  (A solve with 16 < n comes here only
    // for many items of 24 rows: trsm_wave_takes.)
    if (n <= 32 && m <= 16 && (!solve || n <= 16 || batch > 1024) && X.bs == nm && Xin.bs == nm && Xin.rs == X.rs && Xin.cs == X.cs && X.nb2 == 1 &&
        Xin.nb2 == 1 && Lam.nb2 == 1) {
        const bool rowmajor = (X.rs == m && X.cs == 1), colmajor = (X.rs == 1 && X.cs == n);
        if ((rowmajor || colmajor) && n > 16)  // 16 lanes per matrix, two rows per lane
            return launch_tri_rows<T>(solve, fwd, alpha, batch, n, m, Lam, Xin.p, X.p, !rowmajor, st);
        if (rowmajor || colmajor)
            return launch_tri_tiny<T>(solve, fwd, alpha, batch, n, m, Lam, Xin.p, X.p, !rowmajor, st);
    }

    if (leaf_mul)  // (operands the lane-group kernels do not take: other strides)
        return launch_trmm_leaf<T>(Lam, Xin, X, batch, n, m, alpha, fwd, st);

    if (solve && n <= 128 && m <= 48)  // small: one workgroup per item does the whole substitution, no scratch
        return launch_trsm_leaf16<T>(Lam, Xin, X, batch, n, m, alpha, fwd, st);

    if (solve && trsm_stream_takes<T>(batch, n, m)) {  // one launch, no scratch
        const la_status s = launch_trsm_stream<T>(Lam, Xin, X, batch, n, m, alpha, fwd, st);
        if (s != LA_ERR_UNSUPPORTED)  // (strides beyond its 32-bit offsets, two-level batches: the blocked path below)
            return s;
    }

    // Many items of 32 < n <= 64, solves of 16 < n <= 64, went to the kernels of one wavefront per item, which take no scratch.  Fewer go through the
    // inverse or a panel, which do; those kernels take them, too, where the workspace has no room, so that one sized for many items serves a few (with
    // scratch -> without, us, fp64 / fp32: trmm, 500 of n = 64 with 300 vectors 50 -> 51 / 25 -> 40, 1000 of n = 48 with 100 31 -> 20 /
    // 18 -> 18; trsm of the same 92 -> 55 / 54 -> 42 and 72 -> 22 / 46 -> 16, 1000 of n = 24 with 200 68 -> 22 / 51 -> 18, 100 of n = 17 with 4096
    // 82 -> 297 / 58 -> 219).
    if (Lam.nb2 == 1 && (solve || n > 32) && tri_wave_can<T>(batch, n, m, Xin, X) && !arena_room((size_t)batch * (solve ? nn : nm) * sizeof(T)))
        return solve ? launch_trsm_wave<T>(Lam, Xin, X, batch, n, m, alpha, fwd, st)
                     : launch_trmm_wave<T>(Lam, Xin, X, batch, n, m, alpha, fwd, st);

    ArenaFrame frame;
    if (solve && n <= NB) {  // inverse of the single block, then one product in place
        if (!inplace || alpha != T(1))
            LA_TRY(launch_copy<T>(Xin, X, batch, n, m, alpha, 0, st));
        View<T> Inv;
        LA_TRY(scratch_views<T>(batch, n, 1, &Inv));
        LA_TRY(launch_tri_inverse128<T>(Lam, Inv, batch, n, st));
        GemmOpts oi;
        oi.triA = fwd ? 1 : 2;
        oi.min_tile64 = 1;  // in place is safe because one 64 x 64 workgroup tile covers all n rows of its vectors
        return launch_gemm<T>(fwd ? cv(Inv) : cv(Inv).t(), cv(X), X, batch, n, m, n, T(1), T(0), oi, st);
    }

    // scratch: [inverse n*n] [merge temporary n*n] (solve only), then a panel shaped like X
    void *sp = nullptr;
    const size_t per_item = (solve ? 2 * (size_t)nn : 0) + (size_t)nm;
    LA_TRY(arena_take(per_item * batch * sizeof(T), &sp));
    T *base = (T *)sp;
    View<T> Inv{base, nn, n, 1}, Tmp{base + (solve ? batch * nn : 0), nn, n, 1};
    // a compact panel whose fast index is the one X has
    View<T> S = X.rs <= X.cs ? View<T>{base + (solve ? 2 * batch * nn : 0), nm, 1, n}
                             : View<T>{base + (solve ? 2 * batch * nn : 0), nm, m, 1};

    const int NBI = solve_block(m);
    if (!solve || n <= NBI) {
        View<const T> M = Lam;
        if (solve) {
            LA_TRY(inverse_build<T>(Lam, Inv, Tmp, batch, n, n, st));
            M = cv(Inv);
        }
        View<const T> src = Xin;
        if (inplace) {
            LA_TRY(launch_copy<T>(Xin, S, batch, n, m, T(1), 0, st));
            src = cv(S);
        }
        return launch_gemm<T>(fwd ? M : M.t(), src, X, batch, n, m, n, alpha, T(0), o, st);
    }

    LA_TRY(inverse_build<T>(Lam, Inv, Tmp, batch, n, NBI, st));
    if (!inplace || alpha != T(1))
        LA_TRY(launch_copy<T>(Xin, X, batch, n, m, alpha, 0, st));
    return block_substitution<T>(fwd, batch, n, m, NBI, Lam, cv(Inv), X, S, st);
}

template <typename T>
static la_status tri_apply_t(bool solve, int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                             const void *L, const void *A, void *B, hipStream_t st)
{
    View<const T> Lam = tri_view<const T>((const T *)L, n, lower);
    const int64_t nm = (int64_t)n * m;
    View<const T> Xin = rightside ? View<const T>{(const T *)A, nm, 1, n} : View<const T>{(const T *)A, nm, m, 1};
    View<T> X = rightside ? View<T>{(T *)B, nm, 1, n} : View<T>{(T *)B, nm, m, 1};
    const bool use_lt = (trans != 0) != (lower == 0);  // t(L) equals Lam^T
    const bool fwd = (use_lt == (rightside != 0));
    return tri_apply_v<T>(solve, fwd, (T)alpha, batch, n, m, Lam, Xin, X, A == B, st);
}

template <typename T>
static la_status syrk_t(int trans, double alpha, int64_t batch, int n, int k, const void *A, void *B, hipStream_t st)
{
    const int64_t nk = (int64_t)n * k, nn = (int64_t)n * n;
    View<const T> Ank = trans ? View<const T>{(const T *)A, nk, 1, n} : View<const T>{(const T *)A, nk, k, 1};  // n x k
    View<T> C{(T *)B, nn, n, 1};
    if (n <= 16 && k >= 1 && k <= 32)  // G lanes per matrix, HBM bound
        return launch_syrk_tiny<T>(trans != 0, (T)alpha, batch, n, k, (const T *)A, C, st);
    if (outer_rows_takes<T>(n, k, false))  // 16 < n <= 32: 16 lanes per matrix, two rows per lane
        return launch_outer_rows<T>(trans != 0, 0, (T)alpha, batch, n, k, (const T *)A, (const T *)A, C, st);
    if (syrk_wave_takes(batch, n, k))  // one wavefront per matrix
        return launch_outer_wave<T>(0, (T)alpha, batch, n, k, Ank, Ank, C, st);
    if (outer_leaf_takes<T>(batch, n, k, false))  // one workgroup per matrix, operands in LDS
        return launch_outer_leaf<T>(0, (T)alpha, batch, n, k, Ank, Ank, C, st);
    GemmOpts o;
    // 64 x 64 tiles and below store both triangles at once; where the product runs on 128 x 128 tiles (or split along a
    // long k) the mirror image is a pass of its own.
    if (n < 2048 && k < 2048) {
        o.symsum = 2;
        return launch_gemm<T>(Ank, Ank.t(), C, batch, n, n, k, (T)alpha, T(0), o, st);
    }
    o.maskC = 1;
    LA_TRY(launch_gemm<T>(Ank, Ank.t(), C, batch, n, n, k, (T)alpha, T(0), o, st));
    return launch_mirror_lower<T>(C, batch, n, st);
}

// The one-workgroup kernel reads an operand as one run, whatever its row length, and pads to 16; the general product
// loads 64 x 64 tiles row by row.  Measured general -> one-workgroup (8192 items m x n x k, us, fp32 and fp64):
// 37 x 32 x 37 59 -> 35 and 122 -> 55, 20 x 20 x 80 62 -> 34 and 112 -> 55, 16 x 16 x 48 44 -> 16 and 75 -> 21,
// 48 x 48 x 32 40 -> 36 and 83 -> 67, 48 x 48 x 48 (18 operand tiles) 51 -> 49 and 105 -> 98, 8 x 37 x 32 (thin
// products, the second operand plain and transposed) 44 -> 19 and 194 -> 19.  The general one is ahead or equal where it fills
// its tile (64 x 64 x 16 33 -> 34, 64 x 64 x 64 80 -> 101) and where little LDS is left for other workgroups
// (33 x 64 x 100, 49 operand tiles, 99 -> 130).  Below 256 items both wait for the launch.
static bool gemm2_prefers_leaf(int64_t batch, int m, int n, int k)
{
    const int tm = (m + 15) / 16, tn = (n + 15) / 16, tk = (k + 15) / 16;
    return batch >= 256 && batch <= 0x7fffffffll && m >= 4 && n >= 4 && m <= 64 && n <= 64 && tm * tn < 16 && k >= 1 &&
           k <= 128 && (tm + tn) * tk <= 20;
}

template <typename T>
static la_status gemm2_t(int ta, int tb, double alpha, int64_t batch, int m, int n, int k, const void *A, const void *B,
                         void *C, hipStream_t st)
{
    const int64_t sa = (int64_t)m * k, sb = (int64_t)k * n, sc = (int64_t)m * n;
    View<const T> Av = ta ? View<const T>{(const T *)A, sa, 1, m} : View<const T>{(const T *)A, sa, k, 1};  // m x k
    View<const T> Bv = tb ? View<const T>{(const T *)B, sb, 1, k} : View<const T>{(const T *)B, sb, n, 1};  // k x n
    View<T> Cv{(T *)C, sc, n, 1};
    if (m <= 16 && n <= 16 && k >= 1 && k <= 16)  // lane groups of 4, 8 or 16 per item, HBM bound
        return launch_gemm2_tiny<T>(ta, tb, (T)alpha, batch, m, n, k, (const T *)A, (const T *)B, (T *)C, st);
    if (gemm2_rows_takes<T>(m, n, k))  // up to 32 each: 16 lanes per item, two rows per lane
        return launch_gemm2_rows<T>(ta, tb, (T)alpha, batch, m, n, k, (const T *)A, (const T *)B, (T *)C, st);
    if (gemm2_prefers_leaf(batch, m, n, k))  // one workgroup per item, operands in LDS
        return launch_gemm2_leaf<T>(ta, tb, (T)alpha, batch, m, n, k, (const T *)A, (const T *)B, (T *)C, st);
    GemmOpts o;
    return launch_gemm<T>(Av, Bv, Cv, batch, m, n, k, (T)alpha, T(0), o, st);
}

}  // namespace la

using namespace la;

// ---------------------------------------------------------------------------------
// Backward rules of trmm and trsm (section 4.2; appendix "trmm", "trsm", both for a lower and an
// upper factor).  The gradient of the triangular operand is the factor's triangle of an outer
// product of two matrices P, Q of the shape of A: with (X1, X2) = (P, Q), or (Q, P) when the
// operator transposes L,
//   left:  G = X1 X2^T,     right:  G = X2^T X1.
// ---------------------------------------------------------------------------------
template <typename T>
static la_status tri_outer_t(int lower, int trans, int rightside, T scale, int64_t batch, int n, int m, const T *P,
                             const T *Q, T *out, hipStream_t st)
{
    const int64_t nn = (int64_t)n * n, nm = (int64_t)n * m;
    View<T> G{out, nn, n, 1};
    if ((n <= 16 && m >= 1 && m <= 32) || outer_rows_takes<T>(n, m, true)) {  // lane groups: product, mask and zeros in one launch
        const T *U = rightside ? (trans ? P : Q) : (trans ? Q : P), *V = rightside ? (trans ? Q : P) : (trans ? P : Q);
        if (n <= 16)
            return launch_outer_tiny<T>(rightside != 0, lower ? 1 : 2, scale, batch, n, m, U, V, G, st);
        return launch_outer_rows<T>(rightside != 0, lower ? 1 : 2, scale, batch, n, m, U, V, G, st);
    }
    if (outer_wave_takes<T>(batch, n, m)) {  // one wavefront per matrix: product, mask and zeros in one launch
        const T *X1 = trans ? Q : P, *X2 = trans ? P : Q;
        if (!rightside)
            return launch_outer_wave<T>(lower ? 1 : 2, scale, batch, n, m, View<const T>{X1, nm, m, 1},
                                        View<const T>{X2, nm, m, 1}, G, st);
        return launch_outer_wave<T>(lower ? 1 : 2, scale, batch, n, m, View<const T>{X2, nm, 1, n},
                                    View<const T>{X1, nm, 1, n}, G, st);
    }
    if (outer_leaf_takes<T>(batch, n, m, true)) {  // one workgroup per matrix: product, mask and zeros in one launch
        const T *X1 = trans ? Q : P, *X2 = trans ? P : Q;
        if (!rightside)
            return launch_outer_leaf<T>(lower ? 1 : 2, scale, batch, n, m, View<const T>{X1, nm, m, 1},
                                        View<const T>{X2, nm, m, 1}, G, st);
        return launch_outer_leaf<T>(lower ? 1 : 2, scale, batch, n, m, View<const T>{X2, nm, 1, n},
                                    View<const T>{X1, nm, 1, n}, G, st);
    }
    LA_TRY(launch_zero_strict_upper<T>(lower ? G : G.t(), batch, n, st));  // the other triangle of the result
    GemmOpts o;
    o.maskC = lower ? 1 : 2;
    o.split_if_room = n <= NB;  // (as the solve or product of the same call: tri_apply_v)
    if (m == 0)  // empty product: the kept triangle is zero too (written without reading what the buffer held)
        return launch_fill_i32((int32_t *)out, batch * nn * (int64_t)(sizeof(T) / 4), 0, st);
    const T *X1 = trans ? Q : P, *X2 = trans ? P : Q;
    if (!rightside)
        return launch_gemm<T>(View<const T>{X1, nm, m, 1}, View<const T>{X2, nm, 1, m}, G, batch, n, n, m, scale, T(0), o,
                              st);
    return launch_gemm<T>(View<const T>{X2, nm, 1, n}, View<const T>{X1, nm, n, 1}, G, batch, n, n, m, scale, T(0), o,
                          st);
}

template <typename T>
static la_status trmm_backward_t(int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                                 const void *L, const void *A, const void *Bbar, void *Abar, void *Lbar, hipStream_t st)
{
    // Lbar = alpha tri(outer(Bbar, A)) first, then Abar = alpha t(L)^T Bbar (which may overwrite Bbar)
    LA_TRY(tri_outer_t<T>(lower, trans, rightside, (T)alpha, batch, n, m, (const T *)Bbar, (const T *)A, (T *)Lbar, st));
    if (m == 0)
        return LA_OK;
    return tri_apply_t<T>(false, lower, !trans, rightside, alpha, batch, n, m, L, Bbar, Abar, st);
}

template <typename T>
static la_status trsm_backward_t(int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                                 const void *L, const void *B, const void *Bbar, void *Abar, void *Lbar, hipStream_t st)
{
    // Y = t(L)^-T Bbar into Abar (which may overwrite Bbar), Lbar = -tri(outer(Y, B)) (which may
    // overwrite L: L is not needed any more), Abar = alpha Y
    if (m > 0)
        LA_TRY(tri_apply_t<T>(true, lower, !trans, rightside, 1.0, batch, n, m, L, Bbar, Abar, st));
    LA_TRY(tri_outer_t<T>(lower, trans, rightside, T(-1), batch, n, m, (const T *)Abar, (const T *)B, (T *)Lbar, st));
    if (m > 0 && alpha != 1.0) {
        View<T> Y{(T *)Abar, (int64_t)n * m, rightside ? n : m, 1};
        LA_TRY(launch_copy<T>(cv(Y), Y, batch, rightside ? m : n, rightside ? n : m, (T)alpha, 0, st));
    }
    return LA_OK;
}

// C = alpha (G + G^T) A, resp. (right) alpha A (G + G^T), as one product with S = G + G^T in scratch (`cols` rows or columns beside S).
// Only where the workspace has room for S and for what that product takes itself, a split inner dimension, and where the product it saves
// pays for the pass over G; *done stays false otherwise.  us, fp64 / fp32: potri's rule on 64 x 200^2 153 -> 110 / 87 -> 71, 64 x 128^2
// 62 -> 58 / 43 -> 41, 2000^2 1051 -> 703 / 613 -> 427, syrk's rule on 64 x 200^2 with 128 columns 62 -> 41 / 34 -> 25, with 32 22 -> 22 / 16 -> 19; on
// 32 x 512^2 with 128 106 -> 80 / 61 -> 53, with 96 83 -> 68 / 45 -> 45, with 32 37 -> 46 / 24 -> 35; on 300 x 128^2 with 128 87 -> 60 / 42 -> 36, with 32
// 34 -> 37 / 18 -> 26.  Single matrices would gain from fewer columns (2000^2 with 32 96 -> 58 / 62 -> 43) and fewer elements (700^2 with 128 37 -> 25 /
// 25 -> 18).
template <typename T>
static la_status symm_product(const T *G, View<const T> A, View<T> C, int64_t batch, int n, int cols, bool right, T alpha, bool *done,
                              hipStream_t st)
{
    const int64_t nn = (int64_t)n * n;
    *done = false;
    if (n < 128 || cols < 128 || (double)batch * nn < 1048576.0)
        return LA_OK;
    ArenaFrame frame;
    View<T> S;
    auto product = [&]() {
        LA_TRY(scratch_views<T>(batch, n, 1, &S));
        LA_TRY(launch_sym_sum<T>(G, S, batch, n, st));
        GemmOpts o;
        return right ? launch_gemm<T>(A, cv(S), C, batch, cols, n, n, alpha, T(0), o, st)
                     : launch_gemm<T>(cv(S), A, C, batch, n, cols, n, alpha, T(0), o, st);
    };
    size_t bytes = 0;
    LA_TRY(sizing_pass(product, &bytes));
    if (!arena_room(bytes))
        return LA_OK;
    *done = true;
    return product();
}

// syrk backward (section 4.2 "syrk"): Abar = alpha (Bbar + Bbar^T) A  resp.  alpha A (Bbar + Bbar^T),
// two products accumulated in Abar.
template <typename T>
static la_status syrk_backward_t(int trans, double alpha, int64_t batch, int n, int k, const void *A, const void *Bbar,
                                 void *Abar, hipStream_t st)
{
    const int64_t nk = (int64_t)n * k, nn = (int64_t)n * n;
    View<const T> G{(const T *)Bbar, nn, n, 1};
    if (n <= 16 && k >= 1 && k <= 32)  // lane groups of 4, 8 or 16 per matrix, one launch
        return launch_symm_tiny<T>(trans != 0, (T)alpha, batch, n, k, G, (const T *)A, (T *)Abar, st);
    if (symm_rows_takes<T>(n, k))  // 16 < n <= 32: 16 lanes per matrix, two rows per lane
        return launch_symm_rows<T>(trans != 0, (T)alpha, batch, n, k, G, (const T *)A, (T *)Abar, st);
    if (syrk_wave_takes(batch, n, k)) {  // one wavefront per matrix; A and Abar as n x k views
        if (!trans)
            return launch_symm_wave<T>((T)alpha, batch, n, k, G, View<const T>{(const T *)A, nk, k, 1}, View<T>{(T *)Abar, nk, k, 1}, st);
        return launch_symm_wave<T>((T)alpha, batch, n, k, G, View<const T>{(const T *)A, nk, 1, n}, View<T>{(T *)Abar, nk, 1, n}, st);
    }
    if (symm_leaf_takes<T>(batch, n, k)) {  // one workgroup per matrix, operands in LDS; A and Abar as n x k views
        if (!trans)
            return launch_symm_leaf<T>((T)alpha, batch, n, k, G, View<const T>{(const T *)A, nk, k, 1},
                                       View<T>{(T *)Abar, nk, k, 1}, st);
        return launch_symm_leaf<T>((T)alpha, batch, n, k, G, View<const T>{(const T *)A, nk, 1, n},
                                   View<T>{(T *)Abar, nk, 1, n}, st);
    }
    GemmOpts o;
    View<const T> Av{(const T *)A, nk, trans ? n : k, 1};
    View<T> Ov{(T *)Abar, nk, trans ? n : k, 1};
    bool done;
    LA_TRY(symm_product<T>(G.p, Av, Ov, batch, n, k, trans != 0, (T)alpha, &done, st));
    if (done)
        return LA_OK;
    if (!trans) {
        LA_TRY(launch_gemm<T>(G, Av, Ov, batch, n, k, n, (T)alpha, T(0), o, st));
        return launch_gemm<T>(G.t(), Av, Ov, batch, n, k, n, (T)alpha, T(1), o, st);
    }
    LA_TRY(launch_gemm<T>(Av, G, Ov, batch, k, n, n, (T)alpha, T(0), o, st));
    return launch_gemm<T>(Av, G.t(), Ov, batch, k, n, n, (T)alpha, T(1), o, st);
}

// C = alpha Li^T Li + beta C for a lower triangular Li (Li = L^-1: alpha A^-1), both triangles of C written from the lower one
// in one pass.  That form has tiles up to 64 x 64; it is ahead of 128 x 128 tiles and a mirror pass also where those fill the chip
// (potri, us, fp64 and fp32: 32 x 1024^2 808 -> 624 and 462 -> 313, 6144^2 3274 -> 2983 and 1836 -> 1519, 8192^2 7089 -> 6914
// and 3607 -> 3361).
template <typename T>
static la_status gram_add(View<const T> Li, T alpha, View<T> C, T beta, int64_t batch, int n, hipStream_t st)
{
    GemmOpts o;
    o.triA = 2;
    o.triB = 1;
    o.symsum = 2;
    return launch_gemm<T>(Li.t(), Li, C, batch, n, n, n, alpha, beta, o, st);
}

// dst = L^-1 src or L^-T src (m vectors, dst not src) where the whole inverse Li of L is at hand: the form that trsm has for
// these sizes.  Where that takes explicit inverses, of the whole or of blocks on the diagonal, they are those of Li (the inverse of a
// diagonal block is the diagonal block of the inverse); where it is a finer substitution it is called.
template <typename T>
static la_status solve_beside_inverse(bool fwd, int64_t batch, int n, int m, const T *L, View<const T> Li, const T *src, T *dst,
                                      hipStream_t st)
{
    const int64_t nm = (int64_t)n * m;
    if (n <= 2 * NB ? m <= 48 : trsm_stream_takes<T>(batch, n, m))
        return tri_apply_t<T>(true, 1, !fwd, 0, 1.0, batch, n, m, L, src, dst, st);
    const View<const T> in{src, nm, m, 1};
    const View<T> out{dst, nm, m, 1};
    const int edge = solve_block(m);
    if (n <= edge) {
        GemmOpts o;
        o.triA = fwd ? 1 : 2;
        o.reverse = fwd ? 1 : 0;
        return launch_gemm<T>(fwd ? Li : Li.t(), in, out, batch, n, m, n, T(1), T(0), o, st);
    }
    ArenaFrame frame;
    void *p = nullptr;
    LA_TRY(arena_take((size_t)batch * edge * m * sizeof(T), &p));
    LA_TRY(launch_copy<T>(in, out, batch, n, m, T(1), 0, st));
    return block_substitution<T>(fwd, batch, n, m, edge, tri_view<const T>(L, n, 1), Li, out,
                                 View<T>{(T *)p, (int64_t)edge * m, m, 1}, st);
}

// One vector solve with an n x n lower factor L whose inverse Li is there: dst = L^-1 src or L^-T src, src kept; tmp: 2 n elements.
// The streaming solve's chain of blocks takes 47 and 56 us at n = 500 in fp64; a product with the inverse and one step of refinement,
// dst += Li (src - L dst), are three products of about 5 each.  The refined result is as accurate as the chain's, since L is no worse
// conditioned than the square root of a matrix that the precision can factor: over 288 problems of U = 129 to 700 in fp32, noise 1e-3 to 10,
// the criterion's errors and its gradients' are 0.98 to 1.01 times those with the chain (geometric means).
template <typename T>
static la_status solve_vector(bool fwd, int n, const T *L, View<const T> Li, const T *src, T *dst, T *tmp, hipStream_t st)
{
    if (n <= 2 * NB)
        return tri_apply_t<T>(true, 1, !fwd, 0, 1.0, 1, n, 1, L, src, dst, st);
    const View<const T> Lv{L, (int64_t)n * n, n, 1}, A = fwd ? Lv : Lv.t(), Ai = fwd ? Li : Li.t();
    const int tri = fwd ? 1 : 2;
    T *first = tmp + n;
    LA_TRY(launch_gemv_add<T>(Ai, src, nullptr, first, n, n, T(1), T(0), tri, st));
    LA_TRY(launch_gemv_add<T>(A, first, src, tmp, n, n, T(-1), T(1), tri, st));
    return launch_gemv_add<T>(Ai, tmp, first, dst, n, n, T(1), T(1), tri, st);
}

// potri (section 4.2 "potri"): A^-1 = Lam^-T Lam^-1 for A = Lam Lam^T (Lam = L, or R^T for an upper
// factor: the same symmetric matrix either way).
template <typename T>
static la_status potri_t(int lower, int64_t batch, int n, const void *L, void *B, hipStream_t st)
{
    View<const T> Lam = tri_view<const T>((const T *)L, n, lower);
    if (small_wave_takes<T>(SmallWaveOp::potri, batch, n))  // one wavefront per matrix
        return launch_potri_wave<T>(Lam, View<T>{(T *)B, (int64_t)n * n, n, 1}, batch, n, st);
    if (n <= 32)  // both solves on the identity in registers, G lanes per matrix (two rows per lane above 16)
        return launch_potri_tiny<T>(Lam, View<T>{(T *)B, (int64_t)n * n, n, 1}, batch, n, st);
    if (n <= 2 * NB)  // one workgroup per matrix, everything in LDS, no scratch
        return launch_potri_leaf16<T>(Lam, View<T>{(T *)B, (int64_t)n * n, n, 1}, batch, n, st);
    ArenaFrame frame;
    View<T> sc[2];
    LA_TRY(scratch_views<T>(batch, n, 2, sc));
    LA_TRY(inverse_build<T>(Lam, sc[0], sc[1], batch, n, n, st));
    return gram_add<T>(cv(sc[0]), T(1), View<T>{(T *)B, (int64_t)n * n, n, 1}, T(0), batch, n, st);
}

// potri backward (section 4.2 "potri"; appendix "potri"):
//   Lbar = -2 tril(B sym(Bbar) L^-T) = -tril((B Bbar + B Bbar^T) L^-T)      (lower factor)
//   Rbar = -2 triu(R^-T sym(Bbar) B) = -triu(R^-T (Bbar B + Bbar^T B))      (upper factor)
// The two products accumulate in Lbar, the solve runs in place there, the other triangle is cleared.
template <typename T>
static la_status potri_backward_t(int lower, int64_t batch, int n, const void *L, const void *B, const void *Bbar,
                                  void *Lbar, hipStream_t st)
{
    const int64_t nn = (int64_t)n * n;
    View<const T> Bv{(const T *)B, nn, n, 1}, G{(const T *)Bbar, nn, n, 1};
    View<T> X{(T *)Lbar, nn, n, 1};
    if (small_wave_takes<T>(SmallWaveOp::potri_backward, batch, n)) {  // all of it in one launch, a wavefront per matrix
        const View<const T> Lam = tri_view<const T>((const T *)L, n, lower);
        return lower ? launch_potri_backward_wave<T>(Lam, Bv.t(), G, X.t(), batch, n, st)
                     : launch_potri_backward_wave<T>(Lam, Bv, G, X, batch, n, st);
    }
    GemmOpts o;
    bool summed;
    LA_TRY(symm_product<T>(G.p, Bv, X, batch, n, n, lower != 0, T(1), &summed, st));
    if (lower) {
        if (!summed) {
            LA_TRY(launch_gemm<T>(Bv, G, X, batch, n, n, n, T(1), T(0), o, st));
            LA_TRY(launch_gemm<T>(Bv, G.t(), X, batch, n, n, n, T(1), T(1), o, st));
        }
        LA_TRY(tri_apply_t<T>(true, 1, 1, 1, -1.0, batch, n, n, L, Lbar, Lbar, st));
        return launch_zero_strict_upper<T>(X, batch, n, st);
    }
    if (!summed) {
        LA_TRY(launch_gemm<T>(G, Bv, X, batch, n, n, n, T(1), T(0), o, st));
        LA_TRY(launch_gemm<T>(G.t(), Bv, X, batch, n, n, n, T(1), T(1), o, st));
    }
    LA_TRY(tri_apply_t<T>(true, 0, 1, 0, -1.0, batch, n, n, L, Lbar, Lbar, st));
    return launch_zero_strict_upper<T>(X.t(), batch, n, st);
}

// gemm2 backward (section 4.2 "gemm2"): each gradient is a gemm2 of Cbar with the other operand.
template <typename T>
static la_status gemm2_backward_t(int ta, int tb, double alpha, int64_t batch, int m, int n, int k, const void *A,
                                  const void *B, const void *Cbar, void *Abar, void *Bbar, hipStream_t st)
{
    if (!ta)  // Abar (m x k) = alpha Cbar t_b(B)^T
        LA_TRY(gemm2_t<T>(0, !tb, alpha, batch, m, k, n, Cbar, B, Abar, st));
    else  // Abar (k x m) = alpha t_b(B) Cbar^T
        LA_TRY(gemm2_t<T>(tb, 1, alpha, batch, k, m, n, B, Cbar, Abar, st));
    if (!tb)  // Bbar (k x n) = alpha t_a(A)^T Cbar
        return gemm2_t<T>(!ta, 0, alpha, batch, k, n, m, A, Cbar, Bbar, st);
    return gemm2_t<T>(1, ta, alpha, batch, n, k, m, Cbar, A, Bbar, st);  // Bbar (n x k) = alpha Cbar^T t_a(A)
}

// ---------------------------------------------------------------------------------
// Variational sparse Gaussian-process criterion (section 3.2) and its gradient through two Cholesky
// factors of U x U matrices -- the evaluation that makes the criterion cost O(n U^2).  One problem per
// call.  With E = B B^T / lam, A = I + E = La La^T and a = A^-1 B y the reverse sweep over the operators'
// backward rules (section 4.2) comes to
//   A_bar   = 1/2 (A^-1 + a a^T / lam^2),     v_bar = -a / lam^2,
//   B_bar   = (2 / lam) (A_bar - I / 2) B + v_bar y^T,
//   Kuf_bar = Lu^-T B_bar,     Kuu_bar = 1/2 Lu^-T Q Lu^-1,     Q = -B_bar B^T.
// Q needs no product over the n columns: with B B^T = lam E and v = B y it is E + A^-1 - I + a a^T / lam^2,
// and E + A^-1 - I = E A^-1 E = S^T S with S = La^-1 E.  Only the last form is accurate for every noise: the sum
// before it is a difference of terms of order one where E is small, and its relative error grows with 1 / E^2
// (fp32, U = n = 100, noise 1000 against a signal of 1: 8e-2 in Kuu_bar, from S 2e-6).
//
// The caller's workspace holds Lu (U^2), B (U n), E (U^2), A -> La -> Q (U^2), A_bar (U^2), v -> a, w, v_bar (U each),
// one scalar, then SGP_SUMS x SGP_PARTIALS fp64 partial sums; what follows (the inverse of Lu, scratch of the
// steps, B_bar) comes from the arena behind it.
// ---------------------------------------------------------------------------------
template <typename T>
static size_t sgp_workspace_elems(int U, int n)
{
    return 4 * (size_t)U * U + (size_t)U * n + 3 * (size_t)U + 16;
}

template <typename T>
static la_status sgp_t(int U, int n, const void *Kuu_, const void *Kuf_, const void *Kff_, const void *y_, double lam,
                       void *phi_, void *Kuu_bar_, void *Kuf_bar_, void *Kff_bar_, void *y_bar_, void *lam_bar_,
                       void *ws, hipStream_t st)
{
    const int64_t uu = (int64_t)U * U, un = (int64_t)U * n;
    T *Lu = (T *)ws, *B = Lu + uu, *E = B + un, *La = E + uu, *Ab = La + uu, *v = Ab + uu, *w = v + U, *vb = w + U,
      *dummy = vb + U;
    double *sums = reinterpret_cast<double *>(((uintptr_t)(dummy + 16) + 7) & ~(uintptr_t)7);
    const T *Kuf = (const T *)Kuf_, *y = (const T *)y_, *Kff = (const T *)Kff_;
    T *Kuf_bar = (T *)Kuf_bar_, *Kuu_bar = (T *)Kuu_bar_, *y_bar = (T *)y_bar_;
    const T r1 = (T)(1.0 / (lam * lam));
    auto square = [&](T *p) { return View<T>{p, uu, U, 1}; };
    auto wide = [&](T *p) { return View<T>{p, un, n, 1}; };
    GemmOpts plain, low, below;
    low.triA = 1;
    low.reverse = 1;
    below.maskC = 1;
    ArenaFrame outer;
    View<T> Liu;
    // Both solves with Lu and n vectors: the whole inverse everywhere is faster but less accurate (U = 333, n = 7777, fp64
    // 796 -> 639 us; U = 500, n = 1000, fp32, 1e-3 on Kuu's diagonal 2.3e-5 -> 2.1e-4 in Kuf_bar at noise 10).
    auto solve_u = [&](bool fwd, const T *src, T *dst) {  // dst = Lu^-1 src or Lu^-T src
        return solve_beside_inverse<T>(fwd, 1, U, n, Lu, cv(Liu), src, dst, st);
    };

    // ---- forward ----------------------------------------------------------------------------
    LA_TRY(potrf_t<T>(1, 1, U, Kuu_, Lu, nullptr, st));                                        // Lu
    LA_TRY(scratch_views<T>(1, U, 1, &Liu));
    {
        ArenaFrame frame;
        View<T> Tmp;
        LA_TRY(scratch_views<T>(1, U, 1, &Tmp));
        LA_TRY(inverse_build<T>(cv(square(Lu)), Liu, Tmp, 1, U, U, st));                       // Lu^-1
    }
    LA_TRY(solve_u(true, Kuf, B));                                                             // B = Lu^-1 Kuf
    LA_TRY(syrk_t<T>(0, 1.0 / lam, 1, U, n, B, E, st));                                        // E = B B^T / lam
    LA_TRY(launch_plus_identity<T>(E, La, U, st));
    LA_TRY(potrf_t<T>(1, 1, U, La, La, nullptr, st));                                          // La
    LA_TRY(gemm2_t<T>(0, 0, 1.0, 1, U, 1, n, B, y, v, st));                                    // v = B y
    {
        ArenaFrame frame;
        View<T> sc[2];
        LA_TRY(scratch_views<T>(1, U, 2, sc));
        LA_TRY(inverse_build<T>(cv(square(La)), sc[0], sc[1], 1, U, U, st));
        const View<const T> Lia = cv(sc[0]);
        LA_TRY(solve_vector<T>(true, U, La, Lia, v, w, sc[1].p, st));                          // w = La^-1 v
        // ---- backward -----------------------------------------------------------------------
        LA_TRY(solve_vector<T>(false, U, La, Lia, w, v, sc[1].p, st));                         // a = La^-T w (in v's buffer)
        const T *a = v;
        LA_TRY(launch_gp_glue<T>(La, w, nullptr, a, dummy, Ab, 1, U, st, T(0.5) * r1));
        LA_TRY(gram_add<T>(Lia, T(0.5), square(Ab), T(1), 1, U, st));                          // A_bar (symmetric)
        const SumList<T> all{{{0, y, nullptr, n, 0}, {0, w, nullptr, U, 0}, {0, B, nullptr, un, 0}, {1, Kff, nullptr, n, 0},
                              {3, La, nullptr, U, U}, {2, Ab, E, uu, 0}}};
        LA_TRY(launch_partial_sums<T>(all, SGP_SUMS, sums, st));
        LA_TRY(launch_sgp_scalars<T>(sums, lam, n, (T *)phi_, (T *)lam_bar_, (T *)Kff_bar_, n, st));
        LA_TRY(launch_gemm<T>(Lia, View<const T>{E, uu, U, 1}, sc[1], 1, U, U, U, T(1), T(0), low, st));  // S = La^-1 E
        LA_TRY(launch_gemm<T>(cv(sc[1]).t(), cv(sc[1]), square(La), 1, U, U, U, T(1), T(0), below, st));  // S^T S
    }
    LA_TRY(launch_sgp_inner<T>(La, Ab, v, r1, vb, U, st));  // La <- Phi(Q),  Ab <- A_bar - I / 2,  v_bar
    {
        ArenaFrame frame;
        void *p = nullptr;
        LA_TRY(arena_take((size_t)un * sizeof(T), &p));
        const View<T> Bb = wide((T *)p);
        LA_TRY(launch_gemm<T>(cv(square(Ab)), cv(wide(B)), Bb, 1, U, n, U, (T)(2.0 / lam), T(0), plain, st));
        LA_TRY(launch_rank1_add<T>(Bb.p, vb, y, U, n, st));                                    // B_bar
        LA_TRY(solve_u(false, Bb.p, Kuf_bar));                                                 // Kuf_bar = Lu^-T B_bar
    }
    // y_bar = B^T v_bar + y / lam
    LA_TRY(launch_gemv_add<T>(View<const T>{B, un, 1, n}, vb, y, y_bar, n, U, T(1), (T)(1.0 / lam), 0, st));
    return congruence<T>(cv(Liu), cv(square(La)), square(E), square(Kuu_bar), 1, U, st);
}

constexpr int GP_FUSED_N = 128;  // the sizes that launch_gp_leaf16 takes: one launch, no workspace

template <typename T>
static la_status gp_t(int64_t batch, int n, const void *A, const void *y, void *loss, void *Abar, int32_t *info,
                      void *workspace, hipStream_t st)
{
    if (n <= GP_FUSED_N) {
        if (info)
            LA_TRY(launch_fill_i32(info, batch, 0, st));
        return launch_gp_leaf16<T>(tri_view<const T>((const T *)A, n, 1), (const T *)y, (T *)loss,
                                   tri_view<T>((T *)Abar, n, 1), info, batch, n, st);
    }
    const int64_t nn = (int64_t)n * n;
    T *Lw = (T *)workspace, *Iw = Lw + batch * nn, *z = Iw + batch * nn, *al = z + batch * n;
    View<T> Li = tri_view<T>(Iw, n, 1);
    LA_TRY(potrf_t<T>(1, batch, n, A, Lw, info, st));
    {
        ArenaFrame frame;
        View<T> Tmp;
        LA_TRY(scratch_views<T>(batch, n, 1, &Tmp));
        LA_TRY(inverse_build<T>(tri_view<const T>(Lw, n, 1), Li, Tmp, batch, n, n, st));
    }
    LA_TRY(solve_beside_inverse<T>(true, batch, n, 1, Lw, cv(Li), (const T *)y, z, st));
    LA_TRY(solve_beside_inverse<T>(false, batch, n, 1, Lw, cv(Li), z, al, st));
    LA_TRY(launch_gp_glue<T>(Lw, (const T *)y, nullptr, al, (T *)loss, (T *)Abar, batch, n, st));
    return gram_add<T>(cv(Li), T(0.5), tri_view<T>((T *)Abar, n, 1), T(1), batch, n, st);
}

// ---------------------------------------------------------------------------------
// Workspace handling of the entry points.  An operator body `op` (host code that enqueues the
// kernels) runs twice: a sizing pass that launches nothing and records how much scratch the body
// cannot do without, then, if the caller's workspace holds that much, for real on that workspace.
// What the body can also use (arena_room) is in the answer of la_workspace_bytes, but nothing is
// refused for the lack of it.
// ---------------------------------------------------------------------------------
template <class F>
static la_status with_workspace(void *ws, size_t ws_bytes, F &&op)
{
    size_t need = 0;
    LA_TRY(sizing_pass(op, &need, true));
    if (need > 0) {
        if (!ws || need > ws_bytes) {
            snprintf(g_err, sizeof(g_err), "this call needs a workspace of at least %zu bytes, %zu given", need,
                     ws ? ws_bytes : (size_t)0);
            return LA_ERR_WORKSPACE;
        }
        if ((uintptr_t)ws & 255) {
            snprintf(g_err, sizeof(g_err), "the workspace must be 256-byte aligned");
            return LA_ERR_INVALID_ARG;
        }
    }
    Arena a;
    a.base = (char *)ws;
    a.cap = ws && ((uintptr_t)ws & 255) == 0 ? ws_bytes : 0;
    Arena *prev = current_arena();
    current_arena() = &a;
    const la_status s = op();
    current_arena() = prev;
    return s;
}

// does the part of the workspace a call may use overlap an operand?
static inline bool ws_hits(const void *ws, size_t ws_bytes, const void *p, size_t bytes)
{
    return ws && ws_bytes && p && bytes && overlap(ws, ws_bytes, p, bytes);
}

// ---- operator bodies: validated arguments in, kernels enqueued, scratch from the current arena ----
static la_status potrf_body(la_dtype dt, int lower, int64_t batch, int n, const void *A, void *L, int32_t *info,
                            hipStream_t st)
{
    return dt == LA_F32 ? potrf_t<float>(lower, batch, n, A, L, info, st)
                        : potrf_t<double>(lower, batch, n, A, L, info, st);
}

static la_status backward_body(la_dtype dt, int lower, int64_t batch, int n, const void *L, const void *Lbar, void *Abar,
                               hipStream_t st)
{
    if (dt == LA_F32)
        return backward_impl<float>(tri_view<const float>((const float *)L, n, lower),
                                    tri_view<const float>((const float *)Lbar, n, lower),
                                    tri_view<float>((float *)Abar, n, lower), batch, n, Lbar == Abar, st);
    return backward_impl<double>(tri_view<const double>((const double *)L, n, lower),
                                 tri_view<const double>((const double *)Lbar, n, lower),
                                 tri_view<double>((double *)Abar, n, lower), batch, n, Lbar == Abar, st);
}

static la_status tri_body(bool solve, la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n,
                          int m, const void *L, const void *A, void *B, hipStream_t st)
{
    return dt == LA_F32 ? tri_apply_t<float>(solve, lower, trans, rightside, alpha, batch, n, m, L, A, B, st)
                        : tri_apply_t<double>(solve, lower, trans, rightside, alpha, batch, n, m, L, A, B, st);
}

static la_status tri_backward_body(bool solve, la_dtype dt, int lower, int trans, int rightside, double alpha,
                                   int64_t batch, int n, int m, const void *L, const void *X, const void *Bbar, void *Abar,
                                   void *Lbar, hipStream_t st)
{
    if (solve)
        return dt == LA_F32 ? trsm_backward_t<float>(lower, trans, rightside, alpha, batch, n, m, L, X, Bbar, Abar, Lbar, st)
                            : trsm_backward_t<double>(lower, trans, rightside, alpha, batch, n, m, L, X, Bbar, Abar, Lbar, st);
    return dt == LA_F32 ? trmm_backward_t<float>(lower, trans, rightside, alpha, batch, n, m, L, X, Bbar, Abar, Lbar, st)
                        : trmm_backward_t<double>(lower, trans, rightside, alpha, batch, n, m, L, X, Bbar, Abar, Lbar, st);
}

static la_status syrk_body(la_dtype dt, int trans, double alpha, int64_t batch, int n, int k, const void *A, void *B,
                           hipStream_t st)
{
    return dt == LA_F32 ? syrk_t<float>(trans, alpha, batch, n, k, A, B, st)
                        : syrk_t<double>(trans, alpha, batch, n, k, A, B, st);
}

static la_status syrk_backward_body(la_dtype dt, int trans, double alpha, int64_t batch, int n, int k, const void *A,
                                    const void *Bbar, void *Abar, hipStream_t st)
{
    return dt == LA_F32 ? syrk_backward_t<float>(trans, alpha, batch, n, k, A, Bbar, Abar, st)
                        : syrk_backward_t<double>(trans, alpha, batch, n, k, A, Bbar, Abar, st);
}

static la_status gemm2_body(la_dtype dt, int ta, int tb, double alpha, int64_t batch, int m, int n, int k, const void *A,
                            const void *B, void *C, hipStream_t st)
{
    return dt == LA_F32 ? gemm2_t<float>(ta, tb, alpha, batch, m, n, k, A, B, C, st)
                        : gemm2_t<double>(ta, tb, alpha, batch, m, n, k, A, B, C, st);
}

static la_status gemm2_backward_body(la_dtype dt, int ta, int tb, double alpha, int64_t batch, int m, int n, int k,
                                     const void *A, const void *B, const void *Cbar, void *Abar, void *Bbar, hipStream_t st)
{
    return dt == LA_F32 ? gemm2_backward_t<float>(ta, tb, alpha, batch, m, n, k, A, B, Cbar, Abar, Bbar, st)
                        : gemm2_backward_t<double>(ta, tb, alpha, batch, m, n, k, A, B, Cbar, Abar, Bbar, st);
}

static la_status potri_body(la_dtype dt, int lower, int64_t batch, int n, const void *L, void *B, hipStream_t st)
{
    return dt == LA_F32 ? potri_t<float>(lower, batch, n, L, B, st) : potri_t<double>(lower, batch, n, L, B, st);
}

static la_status potri_backward_body(la_dtype dt, int lower, int64_t batch, int n, const void *L, const void *B,
                                     const void *Bbar, void *Lbar, hipStream_t st)
{
    return dt == LA_F32 ? potri_backward_t<float>(lower, batch, n, L, B, Bbar, Lbar, st)
                        : potri_backward_t<double>(lower, batch, n, L, B, Bbar, Lbar, st);
}

// ---- argument checks + workspace + body, shared by the plain and the _ws entry points ------------
static la_status potrf_call(la_dtype dt, int lower, int64_t batch, int n, const void *A, void *L, int32_t *info, void *ws,
                            size_t ws_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || n > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || n == 0)
        return LA_OK;
    if (!A || !L)
        return LA_ERR_INVALID_ARG;
    const size_t bytes = (size_t)batch * n * n * esize(dt);
    if (A != L && overlap(A, bytes, L, bytes))
        return LA_ERR_INVALID_ARG;
    if (info && (overlap(info, (size_t)batch * 4, L, bytes) || overlap(info, (size_t)batch * 4, A, bytes)))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, A, bytes) || ws_hits(ws, ws_bytes, L, bytes) || ws_hits(ws, ws_bytes, info, (size_t)batch * 4))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace(ws, ws_bytes, [&] { return potrf_body(dt, lower, batch, n, A, L, info, st); });
}

static la_status backward_call(la_dtype dt, int lower, int64_t batch, int n, const void *L, const void *Lbar, void *Abar,
                               void *ws, size_t ws_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || n > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || n == 0)
        return LA_OK;
    if (!L || !Lbar || !Abar)
        return LA_ERR_INVALID_ARG;
    const size_t bytes = (size_t)batch * n * n * esize(dt);
    if (overlap(L, bytes, Abar, bytes) || (Lbar != Abar && overlap(Lbar, bytes, Abar, bytes)))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, L, bytes) || ws_hits(ws, ws_bytes, Lbar, bytes) || ws_hits(ws, ws_bytes, Abar, bytes))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace(ws, ws_bytes, [&] { return backward_body(dt, lower, batch, n, L, Lbar, Abar, st); });
}

static la_status tri_call(bool solve, la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n,
                          int m, const void *L, const void *A, void *B, void *ws, size_t ws_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || m < 0 || n > MAX_N || m > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || n == 0 || m == 0)
        return LA_OK;
    if (!L || !A || !B)
        return LA_ERR_INVALID_ARG;
    const size_t lb = (size_t)batch * n * n * esize(dt), ab = (size_t)batch * n * m * esize(dt);
    if (overlap(L, lb, B, ab) || (A != B && overlap(A, ab, B, ab)))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, L, lb) || ws_hits(ws, ws_bytes, A, ab) || ws_hits(ws, ws_bytes, B, ab))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace(ws, ws_bytes,
                          [&] { return tri_body(solve, dt, lower, trans, rightside, alpha, batch, n, m, L, A, B, st); });
}

static la_status tri_backward_call(bool solve, la_dtype dt, int lower, int trans, int rightside, double alpha,
                                   int64_t batch, int n, int m, const void *L, const void *X, const void *Bbar, void *Abar,
                                   void *Lbar, void *ws, size_t ws_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || m < 0 || n > MAX_N || m > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || n == 0)
        return LA_OK;
    if (!L || !Lbar || (m > 0 && (!X || !Bbar || !Abar)))
        return LA_ERR_INVALID_ARG;
    const size_t lb = (size_t)batch * n * n * esize(dt), ab = (size_t)batch * n * m * esize(dt);
    // Abar may be Bbar itself; Lbar may be L itself for trsm (L is consumed first).  Everything else
    // must be disjoint.
    if (m > 0) {
        if (overlap(Abar, ab, L, lb) || overlap(Abar, ab, X, ab) || (Abar != Bbar && overlap(Abar, ab, Bbar, ab)) ||
            overlap(Lbar, lb, X, ab) || overlap(Lbar, lb, Bbar, ab) || overlap(Lbar, lb, Abar, ab))
            return LA_ERR_INVALID_ARG;
    }
    if (overlap(Lbar, lb, L, lb) && !(solve && Lbar == L))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, L, lb) || ws_hits(ws, ws_bytes, Lbar, lb) || ws_hits(ws, ws_bytes, X, ab) ||
        ws_hits(ws, ws_bytes, Bbar, ab) || ws_hits(ws, ws_bytes, Abar, ab))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace(ws, ws_bytes, [&] {
        return tri_backward_body(solve, dt, lower, trans, rightside, alpha, batch, n, m, L, X, Bbar, Abar, Lbar, st);
    });
}

static la_status syrk_call(la_dtype dt, int trans, double alpha, int64_t batch, int n, int k, const void *A, void *B,
                           void *ws, size_t ws_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || k < 0 || n > MAX_N || k > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || n == 0)
        return LA_OK;
    if (!B || (k > 0 && !A))
        return LA_ERR_INVALID_ARG;
    const size_t ab = (size_t)batch * n * k * esize(dt), bb = (size_t)batch * n * n * esize(dt);
    if (k > 0 && overlap(A, ab, B, bb))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, A, ab) || ws_hits(ws, ws_bytes, B, bb))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace(ws, ws_bytes, [&] { return syrk_body(dt, trans, alpha, batch, n, k, A, B, st); });
}

static la_status syrk_backward_call(la_dtype dt, int trans, double alpha, int64_t batch, int n, int k, const void *A,
                                    const void *Bbar, void *Abar, void *ws, size_t ws_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || k < 0 || n > MAX_N || k > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || n == 0 || k == 0)
        return LA_OK;
    if (!A || !Bbar || !Abar)
        return LA_ERR_INVALID_ARG;
    const size_t ab = (size_t)batch * n * k * esize(dt), bb = (size_t)batch * n * n * esize(dt);
    if (overlap(Abar, ab, A, ab) || overlap(Abar, ab, Bbar, bb))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, A, ab) || ws_hits(ws, ws_bytes, Bbar, bb) || ws_hits(ws, ws_bytes, Abar, ab))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace(ws, ws_bytes, [&] { return syrk_backward_body(dt, trans, alpha, batch, n, k, A, Bbar, Abar, st); });
}

static la_status gemm2_call(la_dtype dt, int ta, int tb, double alpha, int64_t batch, int m, int n, int k, const void *A,
                            const void *B, void *C, void *ws, size_t ws_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || m < 0 || n < 0 || k < 0 || m > MAX_N || n > MAX_N || k > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || m == 0 || n == 0)
        return LA_OK;
    if (!C || (k > 0 && (!A || !B)))
        return LA_ERR_INVALID_ARG;
    const size_t ab = (size_t)batch * m * k * esize(dt), bb = (size_t)batch * k * n * esize(dt),
                 cb = (size_t)batch * m * n * esize(dt);
    if (k > 0 && (overlap(A, ab, C, cb) || overlap(B, bb, C, cb)))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, A, ab) || ws_hits(ws, ws_bytes, B, bb) || ws_hits(ws, ws_bytes, C, cb))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace(ws, ws_bytes, [&] { return gemm2_body(dt, ta, tb, alpha, batch, m, n, k, A, B, C, st); });
}

static la_status gemm2_backward_call(la_dtype dt, int ta, int tb, double alpha, int64_t batch, int m, int n, int k,
                                     const void *A, const void *B, const void *Cbar, void *Abar, void *Bbar, void *ws,
                                     size_t ws_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || m < 0 || n < 0 || k < 0 || m > MAX_N || n > MAX_N || k > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0)
        return LA_OK;
    const size_t sa = (size_t)batch * m * k * esize(dt), sb = (size_t)batch * k * n * esize(dt),
                 sc = (size_t)batch * m * n * esize(dt);
    if ((sa && (!A || !Abar)) || (sb && (!B || !Bbar)) || (sc && !Cbar))
        return LA_ERR_INVALID_ARG;
    if (overlap(Abar, sa, A, sa) || overlap(Abar, sa, B, sb) || overlap(Abar, sa, Cbar, sc) || overlap(Bbar, sb, A, sa) ||
        overlap(Bbar, sb, B, sb) || overlap(Bbar, sb, Cbar, sc) || overlap(Abar, sa, Bbar, sb))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, A, sa) || ws_hits(ws, ws_bytes, B, sb) || ws_hits(ws, ws_bytes, Cbar, sc) ||
        ws_hits(ws, ws_bytes, Abar, sa) || ws_hits(ws, ws_bytes, Bbar, sb))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    if (m == 0 || n == 0 || k == 0) {  // empty products: the gradients that exist are zero
        if (sa)
            LA_TRY(launch_fill_i32((int32_t *)Abar, (int64_t)(sa / 4), 0, st));
        if (sb)
            LA_TRY(launch_fill_i32((int32_t *)Bbar, (int64_t)(sb / 4), 0, st));
        return LA_OK;
    }
    return with_workspace(ws, ws_bytes,
                          [&] { return gemm2_backward_body(dt, ta, tb, alpha, batch, m, n, k, A, B, Cbar, Abar, Bbar, st); });
}

static la_status potri_call(la_dtype dt, int lower, int64_t batch, int n, const void *L, void *B, void *ws, size_t ws_bytes,
                            void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || n > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || n == 0)
        return LA_OK;
    if (!L || !B)
        return LA_ERR_INVALID_ARG;
    const size_t nb = (size_t)batch * n * n * esize(dt);
    if (L != B && overlap(L, nb, B, nb))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, L, nb) || ws_hits(ws, ws_bytes, B, nb))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace(ws, ws_bytes, [&] { return potri_body(dt, lower, batch, n, L, B, st); });
}

static la_status potri_backward_call(la_dtype dt, int lower, int64_t batch, int n, const void *L, const void *B,
                                     const void *Bbar, void *Lbar, void *ws, size_t ws_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || n > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || n == 0)
        return LA_OK;
    if (!L || !B || !Bbar || !Lbar)
        return LA_ERR_INVALID_ARG;
    const size_t nb = (size_t)batch * n * n * esize(dt);
    if (overlap(Lbar, nb, L, nb) || overlap(Lbar, nb, B, nb) || overlap(Lbar, nb, Bbar, nb))
        return LA_ERR_INVALID_ARG;
    if (ws_hits(ws, ws_bytes, L, nb) || ws_hits(ws, ws_bytes, B, nb) || ws_hits(ws, ws_bytes, Bbar, nb) ||
        ws_hits(ws, ws_bytes, Lbar, nb))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace(ws, ws_bytes, [&] { return potri_backward_body(dt, lower, batch, n, L, B, Bbar, Lbar, st); });
}

// Operand addresses for the sizing passes of la_workspace_bytes: far apart, 256-byte aligned, never dereferenced.
static inline void *fake_operand(int i) { return reinterpret_cast<void *>(((uintptr_t)1 << 45) + ((uintptr_t)i << 41)); }

static inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

extern "C" {

size_t la_workspace_bytes(la_op op, la_dtype dt, int64_t batch, int n, int m, int k)
{
    if (bad_dtype(dt) || batch <= 0 || n < 0 || m < 0 || k < 0 || n > MAX_N || m > MAX_N || k > MAX_N)
        return 0;
    void *p0 = fake_operand(0), *p1 = fake_operand(1), *p2 = fake_operand(2), *p3 = fake_operand(3), *p4 = fake_operand(4);
    size_t most = 0;
    auto take = [&](auto &&body) {
        size_t peak = 0;
        if (sizing_pass(body, &peak) == LA_OK && peak > most)
            most = peak;
    };
    // every flag combination and every permitted aliasing: the answer holds for all of them
    for (int f = 0; f < 8; ++f) {
        const int lower = f & 1, trans = (f >> 1) & 1, right = (f >> 2) & 1;
        switch (op) {
        case LA_OP_POTRF:
            if (n > 0 && f < 2) {
                take([&] { return potrf_body(dt, lower, batch, n, p0, p1, nullptr, nullptr); });
                take([&] { return potrf_body(dt, lower, batch, n, p0, p0, nullptr, nullptr); });
            }
            break;
        case LA_OP_POTRF_BACKWARD:
            if (n > 0 && f < 2) {
                take([&] { return backward_body(dt, lower, batch, n, p0, p1, p2, nullptr); });
                take([&] { return backward_body(dt, lower, batch, n, p0, p1, p1, nullptr); });
            }
            break;
        case LA_OP_TRSM:
        case LA_OP_TRMM:
            if (n > 0 && m > 0) {
                take([&] { return tri_body(op == LA_OP_TRSM, dt, lower, trans, right, 1.0, batch, n, m, p0, p1, p2, nullptr); });
                take([&] { return tri_body(op == LA_OP_TRSM, dt, lower, trans, right, 0.5, batch, n, m, p0, p1, p1, nullptr); });
            }
            break;
        case LA_OP_TRSM_BACKWARD:
        case LA_OP_TRMM_BACKWARD:
            if (n > 0) {
                const bool solve = op == LA_OP_TRSM_BACKWARD;
                take([&] { return tri_backward_body(solve, dt, lower, trans, right, 0.5, batch, n, m, p0, p1, p2, p3, p4, nullptr); });
                take([&] { return tri_backward_body(solve, dt, lower, trans, right, 1.0, batch, n, m, p0, p1, p2, p2, p4, nullptr); });
            }
            break;
        case LA_OP_SYRK:
            if (n > 0 && f < 2)
                take([&] { return syrk_body(dt, f, 1.0, batch, n, k, p0, p1, nullptr); });
            break;
        case LA_OP_SYRK_BACKWARD:
            if (n > 0 && k > 0 && f < 2)
                take([&] { return syrk_backward_body(dt, f, 1.0, batch, n, k, p0, p1, p2, nullptr); });
            break;
        case LA_OP_GEMM2:
            if (m > 0 && n > 0 && f < 4)
                take([&] { return gemm2_body(dt, f & 1, f >> 1, 1.0, batch, m, n, k, p0, p1, p2, nullptr); });
            break;
        case LA_OP_GEMM2_BACKWARD:
            if (m > 0 && n > 0 && k > 0 && f < 4)
                take([&] { return gemm2_backward_body(dt, f & 1, f >> 1, 1.0, batch, m, n, k, p0, p1, p2, p3, p4, nullptr); });
            break;
        case LA_OP_POTRI:
            if (n > 0 && f < 2) {
                take([&] { return potri_body(dt, lower, batch, n, p0, p1, nullptr); });
                take([&] { return potri_body(dt, lower, batch, n, p0, p0, nullptr); });
            }
            break;
        case LA_OP_POTRI_BACKWARD:
            if (n > 0 && f < 2)
                take([&] { return potri_backward_body(dt, lower, batch, n, p0, p1, p2, p3, nullptr); });
            break;
        default:
            return 0;
        }
    }
    return most;
}

la_status la_potrf_batched(la_dtype dt, int lower, int64_t batch, int n, const void *A, void *L, int32_t *info,
                           void *stream)
{
    return potrf_call(dt, lower, batch, n, A, L, info, nullptr, 0, stream);
}
la_status la_potrf_batched_ws(la_dtype dt, int lower, int64_t batch, int n, const void *A, void *L, int32_t *info,
                              void *workspace, size_t workspace_bytes, void *stream)
{
    return potrf_call(dt, lower, batch, n, A, L, info, workspace, workspace_bytes, stream);
}

// ---------------------------------------------------------------------------------
// potrf for callers that cannot allocate: the scratch of the blocked path is a static array in
// device memory, one copy per GPU, held from the moment the library is loaded on that GPU.
// Its device address is looked up once per device (first call on that device) and passed to the
// kernels like any workspace; the host-side name of the array is not an address and is never
// handed to a kernel or a copy.
// ---------------------------------------------------------------------------------
static __device__ __attribute__((used)) __align__(256) unsigned char scratch[LA_NOALLOC_SCRATCH_BYTES];
static std::mutex g_scratch_mutex;
static void *g_scratch_ptr[64] = {};

la_status la_potrf_batched_noalloc(la_dtype dt, int lower, int64_t batch, int n, const void *A, void *L, int32_t *info,
                                   void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || n > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0 || n == 0)
        return LA_OK;
    int dev = 0;
    LA_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64)
        return LA_ERR_UNSUPPORTED;
    void *ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            void *p = nullptr;
            LA_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
            if (!p) {
                snprintf(g_err, sizeof(g_err), "hipGetSymbolAddress returned no address for the static scratch array");
                return LA_ERR_RUNTIME;
            }
            g_scratch_ptr[dev] = p;
        }
        ptr = g_scratch_ptr[dev];
    }
    const la_status s = potrf_call(dt, lower, batch, n, A, L, info, ptr, (size_t)LA_NOALLOC_SCRATCH_BYTES, stream);
    if (s == LA_ERR_WORKSPACE) {
        size_t need = 0;  // (la_workspace_bytes counts room that is optional, too)
        LA_TRY(sizing_pass([&] { return potrf_body(dt, lower, batch, n, A, L, info, (hipStream_t)stream); }, &need, true));
        snprintf(g_err, sizeof(g_err),
                 "la_potrf_batched_noalloc: batch %lld of n = %d needs %zu bytes of scratch, the static buffer holds %zu",
                 (long long)batch, n, need, (size_t)LA_NOALLOC_SCRATCH_BYTES);
    }
    return s;
}

la_status la_potrf_backward(la_dtype dt, int lower, int64_t batch, int n, const void *L, const void *Lbar, void *Abar,
                            void *stream)
{
    return backward_call(dt, lower, batch, n, L, Lbar, Abar, nullptr, 0, stream);
}
la_status la_potrf_backward_ws(la_dtype dt, int lower, int64_t batch, int n, const void *L, const void *Lbar, void *Abar,
                               void *workspace, size_t workspace_bytes, void *stream)
{
    return backward_call(dt, lower, batch, n, L, Lbar, Abar, workspace, workspace_bytes, stream);
}

la_status la_trsm_batched(la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                          const void *L, const void *A, void *B, void *stream)
{
    return tri_call(true, dt, lower, trans, rightside, alpha, batch, n, m, L, A, B, nullptr, 0, stream);
}
la_status la_trsm_batched_ws(la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                             const void *L, const void *A, void *B, void *workspace, size_t workspace_bytes, void *stream)
{
    return tri_call(true, dt, lower, trans, rightside, alpha, batch, n, m, L, A, B, workspace, workspace_bytes, stream);
}

la_status la_trmm_batched(la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                          const void *L, const void *A, void *B, void *stream)
{
    return tri_call(false, dt, lower, trans, rightside, alpha, batch, n, m, L, A, B, nullptr, 0, stream);
}
la_status la_trmm_batched_ws(la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                             const void *L, const void *A, void *B, void *workspace, size_t workspace_bytes, void *stream)
{
    return tri_call(false, dt, lower, trans, rightside, alpha, batch, n, m, L, A, B, workspace, workspace_bytes, stream);
}

la_status la_trsm_backward(la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                           const void *L, const void *B, const void *Bbar, void *Abar, void *Lbar, void *stream)
{
    return tri_backward_call(true, dt, lower, trans, rightside, alpha, batch, n, m, L, B, Bbar, Abar, Lbar, nullptr, 0, stream);
}
la_status la_trsm_backward_ws(la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                              const void *L, const void *B, const void *Bbar, void *Abar, void *Lbar, void *workspace,
                              size_t workspace_bytes, void *stream)
{
    return tri_backward_call(true, dt, lower, trans, rightside, alpha, batch, n, m, L, B, Bbar, Abar, Lbar, workspace,
                             workspace_bytes, stream);
}

la_status la_trmm_backward(la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                           const void *L, const void *A, const void *Bbar, void *Abar, void *Lbar, void *stream)
{
    return tri_backward_call(false, dt, lower, trans, rightside, alpha, batch, n, m, L, A, Bbar, Abar, Lbar, nullptr, 0, stream);
}
la_status la_trmm_backward_ws(la_dtype dt, int lower, int trans, int rightside, double alpha, int64_t batch, int n, int m,
                              const void *L, const void *A, const void *Bbar, void *Abar, void *Lbar, void *workspace,
                              size_t workspace_bytes, void *stream)
{
    return tri_backward_call(false, dt, lower, trans, rightside, alpha, batch, n, m, L, A, Bbar, Abar, Lbar, workspace,
                             workspace_bytes, stream);
}

la_status la_gemm2_backward(la_dtype dt, int ta, int tb, double alpha, int64_t batch, int m, int n, int k,
                            const void *A, const void *B, const void *Cbar, void *Abar, void *Bbar, void *stream)
{
    return gemm2_backward_call(dt, ta, tb, alpha, batch, m, n, k, A, B, Cbar, Abar, Bbar, nullptr, 0, stream);
}
la_status la_gemm2_backward_ws(la_dtype dt, int ta, int tb, double alpha, int64_t batch, int m, int n, int k,
                               const void *A, const void *B, const void *Cbar, void *Abar, void *Bbar, void *workspace,
                               size_t workspace_bytes, void *stream)
{
    return gemm2_backward_call(dt, ta, tb, alpha, batch, m, n, k, A, B, Cbar, Abar, Bbar, workspace, workspace_bytes, stream);
}

la_status la_potri(la_dtype dt, int lower, int64_t batch, int n, const void *L, void *B, void *stream)
{
    return potri_call(dt, lower, batch, n, L, B, nullptr, 0, stream);
}
la_status la_potri_ws(la_dtype dt, int lower, int64_t batch, int n, const void *L, void *B, void *workspace,
                      size_t workspace_bytes, void *stream)
{
    return potri_call(dt, lower, batch, n, L, B, workspace, workspace_bytes, stream);
}

la_status la_potri_backward(la_dtype dt, int lower, int64_t batch, int n, const void *L, const void *B,
                            const void *Bbar, void *Lbar, void *stream)
{
    return potri_backward_call(dt, lower, batch, n, L, B, Bbar, Lbar, nullptr, 0, stream);
}
la_status la_potri_backward_ws(la_dtype dt, int lower, int64_t batch, int n, const void *L, const void *B,
                               const void *Bbar, void *Lbar, void *workspace, size_t workspace_bytes, void *stream)
{
    return potri_backward_call(dt, lower, batch, n, L, B, Bbar, Lbar, workspace, workspace_bytes, stream);
}

la_status la_syrk_backward(la_dtype dt, int trans, double alpha, int64_t batch, int n, int k, const void *A,
                           const void *Bbar, void *Abar, void *stream)
{
    return syrk_backward_call(dt, trans, alpha, batch, n, k, A, Bbar, Abar, nullptr, 0, stream);
}
la_status la_syrk_backward_ws(la_dtype dt, int trans, double alpha, int64_t batch, int n, int k, const void *A,
                              const void *Bbar, void *Abar, void *workspace, size_t workspace_bytes, void *stream)
{
    return syrk_backward_call(dt, trans, alpha, batch, n, k, A, Bbar, Abar, workspace, workspace_bytes, stream);
}

la_status la_syrk_batched(la_dtype dt, int trans, double alpha, int64_t batch, int n, int k, const void *A, void *B,
                          void *stream)
{
    return syrk_call(dt, trans, alpha, batch, n, k, A, B, nullptr, 0, stream);
}
la_status la_syrk_batched_ws(la_dtype dt, int trans, double alpha, int64_t batch, int n, int k, const void *A, void *B,
                             void *workspace, size_t workspace_bytes, void *stream)
{
    return syrk_call(dt, trans, alpha, batch, n, k, A, B, workspace, workspace_bytes, stream);
}

la_status la_gemm2_batched(la_dtype dt, int ta, int tb, double alpha, int64_t batch, int m, int n, int k, const void *A,
                           const void *B, void *C, void *stream)
{
    return gemm2_call(dt, ta, tb, alpha, batch, m, n, k, A, B, C, nullptr, 0, stream);
}
la_status la_gemm2_batched_ws(la_dtype dt, int ta, int tb, double alpha, int64_t batch, int m, int n, int k, const void *A,
                              const void *B, void *C, void *workspace, size_t workspace_bytes, void *stream)
{
    return gemm2_call(dt, ta, tb, alpha, batch, m, n, k, A, B, C, workspace, workspace_bytes, stream);
}

size_t la_sgp_workspace_bytes(la_dtype dt, int U, int n)
{
    if (bad_dtype(dt) || U <= 0 || n <= 0 || U > MAX_N || n > MAX_N)
        return 0;
    const size_t e = dt == LA_F32 ? sgp_workspace_elems<float>(U, n) : sgp_workspace_elems<double>(U, n);
    const size_t fixed = align256(e * esize(dt) + 8 + SGP_SUMS * SGP_PARTIALS * sizeof(double));
    void *p[10];
    for (int i = 0; i < 10; ++i)
        p[i] = fake_operand(i);
    size_t peak = 0;
    const la_status s = sizing_pass(
        [&] {
            return dt == LA_F32 ? sgp_t<float>(U, n, p[0], p[1], p[2], p[3], 1.0, p[4], p[5], p[6], p[7], p[8], p[9],
                                               fake_operand(10), nullptr)
                                : sgp_t<double>(U, n, p[0], p[1], p[2], p[3], 1.0, p[4], p[5], p[6], p[7], p[8], p[9],
                                                fake_operand(10), nullptr);
        },
        &peak);
    return s == LA_OK ? fixed + peak : 0;
}

la_status la_sgp_criterion(la_dtype dt, int U, int n, const void *Kuu, const void *Kuf, const void *Kff_diag,
                           const void *y, double noise_var, void *phi, void *Kuu_bar, void *Kuf_bar, void *Kff_diag_bar,
                           void *y_bar, void *noise_bar, void *workspace, size_t workspace_bytes, void *stream)
{
    if (bad_dtype(dt) || U <= 0 || n <= 0 || U > MAX_N || n > MAX_N || !(noise_var > 0.0))
        return LA_ERR_INVALID_ARG;
    if (!Kuu || !Kuf || !Kff_diag || !y || !phi || !Kuu_bar || !Kuf_bar || !Kff_diag_bar || !y_bar || !noise_bar ||
        !workspace || ((uintptr_t)workspace & 255))
        return LA_ERR_INVALID_ARG;
    const size_t e = dt == LA_F32 ? sgp_workspace_elems<float>(U, n) : sgp_workspace_elems<double>(U, n);
    const size_t fixed = align256(e * esize(dt) + 8 + SGP_SUMS * SGP_PARTIALS * sizeof(double));
    if (workspace_bytes < fixed) {
        snprintf(g_err, sizeof(g_err), "this call needs a workspace of la_sgp_workspace_bytes bytes, %zu given",
                 workspace_bytes);
        return LA_ERR_WORKSPACE;
    }
    const size_t uu = (size_t)U * U * esize(dt), un = (size_t)U * n * esize(dt);
    if (overlap(Kuu_bar, uu, Kuu, uu) || overlap(Kuf_bar, un, Kuf, un) || overlap(Kuu_bar, uu, Kuf_bar, un) ||
        overlap(workspace, workspace_bytes, Kuu_bar, uu) || overlap(workspace, workspace_bytes, Kuf_bar, un) ||
        overlap(workspace, workspace_bytes, Kuu, uu) || overlap(workspace, workspace_bytes, Kuf, un))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return with_workspace((char *)workspace + fixed, workspace_bytes - fixed, [&] {
        return dt == LA_F32 ? sgp_t<float>(U, n, Kuu, Kuf, Kff_diag, y, noise_var, phi, Kuu_bar, Kuf_bar, Kff_diag_bar, y_bar,
                                           noise_bar, workspace, st)
                            : sgp_t<double>(U, n, Kuu, Kuf, Kff_diag, y, noise_var, phi, Kuu_bar, Kuf_bar, Kff_diag_bar, y_bar,
                                            noise_bar, workspace, st);
    });
}

la_status la_kalman_filter(la_dtype dt, int64_t batch, int T, int dh, int dv, int shared_params, const void *A,
                           const void *B, const void *Sh, const void *Sv, const void *mu0, const void *S0,
                           const void *v, void *f, void *F, void *nll, int32_t *info, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || T < 0 || dh < 1 || dv < 1)
        return LA_ERR_INVALID_ARG;
    if (dh > 16 || dv > 16)
        return LA_ERR_UNSUPPORTED;
    if (batch == 0)
        return LA_OK;
    if (!A || !B || !Sh || !Sv || !mu0 || !S0 || !nll || (T > 0 && !v))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    if (dt == LA_F32)
        return launch_kalman<float>((const float *)A, (const float *)B, (const float *)Sh, (const float *)Sv,
                                    (const float *)mu0, (const float *)S0, (const float *)v, (float *)f, (float *)F,
                                    (float *)nll, info, batch, T, dh, dv, shared_params != 0, st);
    return launch_kalman<double>((const double *)A, (const double *)B, (const double *)Sh, (const double *)Sv,
                                 (const double *)mu0, (const double *)S0, (const double *)v, (double *)f, (double *)F,
                                 (double *)nll, info, batch, T, dh, dv, shared_params != 0, st);
}

la_status la_sumlogdiag(la_dtype dt, int64_t batch, int n, const void *L, void *out, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || n > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0)
        return LA_OK;
    if (!out || (n > 0 && !L))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return dt == LA_F32 ? launch_sumlogdiag<float>((const float *)L, (float *)out, batch, n, st)
                        : launch_sumlogdiag<double>((const double *)L, (double *)out, batch, n, st);
}

la_status la_gp_glue(la_dtype dt, int64_t batch, int n, const void *L, const void *y, const void *z, const void *alpha,
                     void *loss, void *Lbar, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || n > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0)
        return LA_OK;
    if (!loss || (n > 0 && (!L || !y || !z || !alpha || !Lbar)))
        return LA_ERR_INVALID_ARG;
    const size_t bytes = (size_t)batch * n * n * esize(dt);
    if (n > 0 && overlap(L, bytes, Lbar, bytes))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    return dt == LA_F32 ? launch_gp_glue<float>((const float *)L, (const float *)y, (const float *)z,
                                                (const float *)alpha, (float *)loss, (float *)Lbar, batch, n, st)
                        : launch_gp_glue<double>((const double *)L, (const double *)y, (const double *)z,
                                                 (const double *)alpha, (double *)loss, (double *)Lbar, batch, n, st);
}

// fixed part of the GP criterion's workspace above the one-launch sizes: L, L^-1, z, alpha
static size_t gp_fixed_bytes(la_dtype dt, int64_t batch, int n)
{
    return align256(((size_t)batch * n * n * 2 + (size_t)batch * n * 2) * esize(dt));
}

size_t la_gp_workspace_bytes(la_dtype dt, int64_t batch, int n)
{
    if (bad_dtype(dt) || batch <= 0 || n <= 0 || n > MAX_N)
        return 0;
    if (n <= GP_FUSED_N)
        return 0;
    size_t peak = 0;
    const la_status s = sizing_pass(
        [&] {
            return dt == LA_F32 ? gp_t<float>(batch, n, fake_operand(0), fake_operand(1), fake_operand(2), fake_operand(3),
                                              nullptr, fake_operand(4), nullptr)
                                : gp_t<double>(batch, n, fake_operand(0), fake_operand(1), fake_operand(2), fake_operand(3),
                                               nullptr, fake_operand(4), nullptr);
        },
        &peak);
    return s == LA_OK ? gp_fixed_bytes(dt, batch, n) + peak : 0;
}

la_status la_gp_criterion(la_dtype dt, int64_t batch, int n, const void *A, const void *y, void *loss, void *Abar,
                          int32_t *info, void *workspace, size_t workspace_bytes, void *stream)
{
    if (bad_dtype(dt) || batch < 0 || n < 0 || n > MAX_N)
        return LA_ERR_INVALID_ARG;
    if (batch == 0)
        return LA_OK;
    if (!loss || (n > 0 && (!A || !y || !Abar)))
        return LA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    if (n == 0)  // empty sums
        return dt == LA_F32 ? launch_gp_glue<float>(nullptr, nullptr, nullptr, nullptr, (float *)loss, nullptr, batch, 0, st)
                            : launch_gp_glue<double>(nullptr, nullptr, nullptr, nullptr, (double *)loss, nullptr, batch, 0,
                                                     st);
    const size_t fixed = n <= GP_FUSED_N ? 0 : gp_fixed_bytes(dt, batch, n);
    const size_t bytes = (size_t)batch * n * n * esize(dt);
    if (fixed > 0) {
        if (!workspace || workspace_bytes < fixed) {
            snprintf(g_err, sizeof(g_err), "this call needs a workspace of la_gp_workspace_bytes bytes, %zu given",
                     workspace ? workspace_bytes : (size_t)0);
            return LA_ERR_WORKSPACE;
        }
        if (((uintptr_t)workspace & 255) || overlap(workspace, workspace_bytes, A, bytes) ||
            overlap(workspace, workspace_bytes, Abar, bytes))
            return LA_ERR_INVALID_ARG;
    }
    if (A != Abar && overlap(A, bytes, Abar, bytes))
        return LA_ERR_INVALID_ARG;
    return with_workspace(fixed ? (char *)workspace + fixed : nullptr, fixed ? workspace_bytes - fixed : 0, [&] {
        return dt == LA_F32 ? gp_t<float>(batch, n, A, y, loss, Abar, info, workspace, st)
                            : gp_t<double>(batch, n, A, y, loss, Abar, info, workspace, st);
    });
}

const char *la_last_error(void) { return g_err; }

int la_version(void) { return 200; }

}  // extern "C"
