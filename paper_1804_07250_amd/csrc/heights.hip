// Lozenge tilings of the a x b x c hexagon and the six-vertex model with
// domain-wall boundary: the two height-function models (Section 1.2).
//
// Both store one bit per height site (a 1-bit residual of the height):
//   lozenge    H(X, Y) mod 2 per triangular vertex; along (1,0), (0,1), (1,1) H
//              changes by 0 or -1, so the parity of two neighbours fixes their
//              difference.  Plane s = X mod 3 holds the vertices X = 3k + s of a
//              row, so one plane of a row is exactly one colour class (colour
//              (X + Y) mod 3).
//   six-vertex floor(h/2) mod 2 per face; neighbouring faces differ by +-1 and
//              h = (I + J) mod 2 + 2 floor(h/2), so the bit fixes the sign.
//              Plane p = I mod 2; colour (I mod 2) + 2 (J mod 2).
// A colour step updates one plane of every other row (six-vertex) or one plane
// of every row (lozenge); each site writes only its own bit, reading the other
// planes of its row and of the rows above and below.
//
// Lozenge move (Section 1.2, lozenge rotations): a vertex is rotateable iff its
// forward neighbours (X+1,Y), (X,Y+1), (X+1,Y+1) share a height f and its
// backward neighbours share f+1; up (add a cube) sets H = f+1, which has the
// parity of the backward neighbours, down sets H = f.
// Six-vertex move (c-flip): a face is flippable iff its four edge neighbours
// share a height m; up sets m+1.  A diagonal face is "high" iff it is at m+1.
// Context of the weights: sA = #high among NE, SW (corners carrying a) and
// sB = #high among NW, SE (corners carrying b); W_up/W_down depends on (sA, sB)
// only.
#include <type_traits>

#include "../../include/tilings.h"
#include "height_common.hpp"
#include "internal.hpp"

namespace tl {

size_t height_words(HeightDev &d)
{
    if (d.model == TL_LOZENGE) {
        d.P = 3;
        d.rows = (uint32_t)(d.b + d.c + 1);
        d.K = (uint32_t)((d.a + d.c + 3) / 3);
    } else {
        d.P = 2;
        d.rows = (uint32_t)(d.N + 1);
        d.K = (uint32_t)((d.N + 2) / 2);
    }
    const uint32_t nw = (d.K + 31u) / 32u;
    d.ng = (nw + 3u) / 4u;
    d.RS = 4u * (d.ng + 2u);
    d.PS = (size_t)d.rows * d.RS;
    return d.P * d.PS;
}

namespace {

enum { kHeatBath = 0, kMetropolis = 1, kUniform = 2 };
static_assert(kHeatBath == kModeHeatBath && kMetropolis == kModeMetropolis && kUniform == kModeUniform,
              "kernel modes and TileJob modes agree");
// (row, group) tasks of a tile (six-vertex: row pairs) and lanes of a work-group.
constexpr uint32_t kTileTasks = 512;
constexpr uint32_t kTileThreads = 1024;
// Layout of a six-vertex threshold table (each layout is its own kernel
// instantiation, so its registers are allocated for it alone): 9 classes
// (sA, sB) [x2 for Metropolis], or 5 classes by sA + sB (heat-bath).  Lozenge
// tables always use kKindClass.
enum { kKindClass = 0, kKindSum = 1 };
static_assert(kKindClass == kTableClass && kKindSum == kTableSum, "table layouts agree");

// Instantiation KERNEL<mode, layout, flag> for a rule (mode), a table layout
// (kind) and a compile-time flag.
#define TL_HEIGHT_PICK_R(KERNEL, mode, kind, R)                                                 \
    ((mode) == kUniform ? KERNEL<kUniform, kKindClass, R>                                       \
     : (mode) == kMetropolis                                                                    \
         ? ((kind) == kKindSum ? KERNEL<kMetropolis, kKindSum, R> : KERNEL<kMetropolis, kKindClass, R>) \
     : (kind) == kKindSum ? KERNEL<kHeatBath, kKindSum, R> : KERNEL<kHeatBath, kKindClass, R>)
// And with two: the colour order (random) and site planes (masked domain).
#define TL_HEIGHT_PICK_RM(KERNEL, mode, kind, R, M)                                             \
    ((mode) == kUniform ? KERNEL<kUniform, kKindClass, R, M>                                    \
     : (mode) == kMetropolis                                                                    \
         ? ((kind) == kKindSum ? KERNEL<kMetropolis, kKindSum, R, M> : KERNEL<kMetropolis, kKindClass, R, M>) \
     : (kind) == kKindSum ? KERNEL<kHeatBath, kKindSum, R, M> : KERNEL<kHeatBath, kKindClass, R, M>)
#define TL_HEIGHT_PICK_ORDER_MASK(KERNEL, mode, kind, order, masked)                            \
    ((order) ? ((masked) ? TL_HEIGHT_PICK_RM(KERNEL, mode, kind, true, true)                    \
                         : TL_HEIGHT_PICK_RM(KERNEL, mode, kind, true, false))                  \
             : ((masked) ? TL_HEIGHT_PICK_RM(KERNEL, mode, kind, false, true)                   \
                         : TL_HEIGHT_PICK_RM(KERNEL, mode, kind, false, false)))

struct Geo {
    int model, a, b, c, N;
    const uint32_t *site;   // site planes of a masked domain (layout sPS, sRS), or nullptr
    size_t sPS;
    uint32_t sRS;
    const uint32_t *freep;  // six-vertex: planes of the free points (same layout), or nullptr
    int free_side;          // their side: 1 north, 2 south, 3 east, 4 west
};

__device__ __forceinline__ int imax(int p, int q) { return p > q ? p : q; }
__device__ __forceinline__ int imin(int p, int q) { return p < q ? p : q; }

// Lozenge: H_min / H_max at (X, Y) = (x + c, y + c).
__device__ __forceinline__ int loz_hmin(const Geo &g, int X, int Y) { return imax(0, imax(g.c - X, g.c - Y)); }
__device__ __forceinline__ int loz_hmax(const Geo &g, int X, int Y)
{
    return imin(g.c, imin(g.a + g.c - X, g.b + g.c - Y));
}
// Vertices of row Y inside the hexagon: X in [loz_xs, loz_xe].
__device__ __forceinline__ int loz_xs(const Geo &g, int Y) { return imax(0, Y - g.b); }
__device__ __forceinline__ int loz_xe(const Geo &g, int Y) { return imin(g.a + g.c, Y + g.a); }

__global__ void height_init_kernel(uint32_t *pa, uint32_t *pb, size_t PS, uint32_t RS, uint32_t rows, uint32_t P,
                                   Geo geo, int init_max)
{
    const uint32_t w = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t y = blockIdx.y, p = blockIdx.z;
    if (w >= RS || y >= rows || p >= P) return;
    uint32_t bits = 0u;
    if (w >= 4u) {
        const int dw = (int)w - 4;
        for (int bb = 0; bb < 32; ++bb) {
            const int k = dw * 32 + bb;
            if (geo.model == TL_LOZENGE) {
                const int X = 3 * k + (int)p, Y = (int)y;
                if (X > geo.a + geo.c || X < loz_xs(geo, Y) || X > loz_xe(geo, Y)) continue;
                const int H = init_max ? loz_hmax(geo, X, Y) : loz_hmin(geo, X, Y);
                bits |= (uint32_t)(H & 1) << bb;
            } else {
                const int I = 2 * k + (int)p, J = (int)y;
                if (I > geo.N) continue;
                const int h = init_max ? geo.N - abs(I + J - geo.N) : abs(I - J);
                bits |= (uint32_t)((h >> 1) & 1) << bb;
            }
        }
    }
    pa[p * PS + (size_t)y * RS + w] = bits;
    if (pb) pb[p * PS + (size_t)y * RS + w] = bits;
}

// Decisions of the 128 sites of a group held by one lane (the streaming
// kernels): the one-bit draw, or the bit-serial comparison.
struct GroupDraws {
    static constexpr bool kPairs = false;   // compare() takes every class
    uint32_t k0, k1, g, r, t, c;
    uint32_t R0[4];   // plane 0 (one-bit decisions)
    __device__ __forceinline__ void one_bit(uint32_t (&D)[4]) const
    {
#pragma unroll
        for (int w = 0; w < 4; ++w) D[w] = ~R0[w];
    }
    template <int NC, uint32_t kPlanes>
    __device__ __forceinline__ void compare(const uint32_t (&T)[NC], const uint32_t (&cm)[NC][4],
                                            const uint32_t (&live)[4], uint32_t (&D)[4]) const
    {
        decide128<NC, kPlanes>(k0, k1, g, r, t, c, T, cm, live, D);
    }
};

// Decisions of one word (32 sites) by lane (row, word) = (lane & 15, lane >> 4)
// of a wavefront that holds 16 rows of a group.  `A` holds the lane's word of
// the planes drawn ahead (kAheadPlanes of them; one-bit decisions: plane 0) if
// `ready`; other planes are drawn four at a time by the four lanes of a row,
// and handed to their words by a transpose over lanes 16 apart.
struct WordDraws {
    static constexpr bool kPairs = true;   // compare() takes the classes but 2^31 (metro_classes)
    uint32_t k0, k1, g, r, t, c, q;
    bool ready;   // the same in every lane
    const uint32_t *A;
    __device__ __forceinline__ void one_bit(uint32_t (&D)[1]) const
    {
        if (ready) {
            D[0] = ~A[0];
            return;
        }
        uint32_t R[4];
        philox4x32_10(g, r, t, c, k0, k1, R);
        D[0] = ~(q < 2u ? (q == 0u ? R[0] : R[1]) : (q == 2u ? R[2] : R[3]));
    }
    // rest: the sites in none of the classes, whose threshold is 2^31
    template <int NC, uint32_t kPlanes>
    __device__ __forceinline__ void compare(const uint32_t (&T)[NC], const uint32_t (&cm)[NC][1],
                                            const uint32_t (&live)[1], uint32_t (&D)[1], uint32_t rest = 0u) const
    {
        // with several classes, T is kept from being hoisted out of the step
        // loop: the selectors of every plane and class are more scalars than
        // there are registers
        uint32_t Ts[NC];
        uint32_t half = rest;   // sites whose threshold is 2^31: plane 0 decides them
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            Ts[i] = T[i];
            if (NC > 1) {
                asm volatile("" : "+s"(Ts[i]));
                half |= cm[i][0] & (Ts[i] == 0x80000000u ? ~0u : 0u);
            }
        }
        // Planes j0 .. j0 + 3, compared from the last to the first: x becomes
        // "u below T within these planes", e "equal there" (two operations a
        // plane).  A site that stays equal to the end has u >= T: 0; bits of T
        // below its lowest 1 change nothing.
        uint32_t eq = live[0], lt = 0u;
        auto four = [&](uint32_t j0, uint32_t R0, uint32_t R1, uint32_t R2, uint32_t R3) {
            const uint32_t R[4] = {R0, R1, R2, R3};
            uint32_t x = 0u, e = ~0u;
#pragma unroll
            for (int y = 3; y >= 0; --y) {
                uint32_t tb = j0 == 0u && y == 0 ? rest : 0u;
                if constexpr (NC == 1) {
                    tb = (uint32_t)((int32_t)(Ts[0] << (j0 + (uint32_t)y)) >> 31);
                } else {
#pragma unroll
                    for (int i = 0; i < NC; ++i)
                        tb |= cm[i][0] & (uint32_t)((int32_t)(Ts[i] << (j0 + (uint32_t)y)) >> 31);
                }
                x = __builtin_amdgcn_bitop3_b32(tb, R[y], x, 0xB2);   // tb ? ~R | x : ~R & x
                e = __builtin_amdgcn_bitop3_b32(tb, R[y], e, 0x82);   // e & ~(tb ^ R)
            }
            lt |= eq & x;
            eq &= e;
            if (NC > 1 && j0 == 0u) eq &= ~half;
        };
        uint32_t j0 = 0u;
        if (ready) {
            static_assert(kAheadPlanes == 8u, "two rounds of planes drawn ahead");
            four(0u, A[0], A[1], A[2], A[3]);
            four(4u, A[4], A[5], A[6], A[7]);
            j0 = kAheadPlanes;
        }
        for (; j0 < 32u; j0 += 4u) {
            if (!__any(eq != 0u)) break;
            uint32_t R[4];
            philox4x32_10(g, r, t, ((j0 + q) << 2) | c, k0, k1, R);
            rows_transpose(R);
            four(j0, R[0], R[1], R[2], R[3]);
        }
        D[0] = lt;
    }
};

// Classes of a lazy Metropolis decision from those of the local weights, s: the
// table has two thresholds a class, current state down and up, and one of the
// two is 2^31 (floor(2^31 min(1, r)) and 2^32 - floor(2^31 min(1, 1 / r)) for a
// weight ratio r).  Plane 0 decides its sites, so the comparison takes the other
// one alone, and half the classes.
template <int NS, uint32_t kPlanes, int W, class Draws>
__device__ __forceinline__ void metro_compare(const Draws &dr, const uint32_t *Tall, const uint32_t (&s)[NS][W],
                                              const uint32_t (&cur)[W], const uint32_t (&live)[W], uint32_t (&D)[W])
{
    if constexpr (Draws::kPairs) {
        uint32_t T[NS], cm[NS][W], rest = ~0u;
#pragma unroll
        for (int x = 0; x < NS; ++x) {
            const bool up = Tall[2 * x] == 0x80000000u;
            T[x] = up ? Tall[2 * x + 1] : Tall[2 * x];
            cm[x][0] = s[x][0] & (cur[0] ^ (up ? 0u : ~0u));
            rest &= ~cm[x][0];
        }
        dr.template compare<NS, kPlanes>(T, cm, live, D, rest);
    } else {
        uint32_t T[2 * NS], cm[2 * NS][W];
#pragma unroll
        for (int x = 0; x < NS; ++x) {
            T[2 * x] = Tall[2 * x];
            T[2 * x + 1] = Tall[2 * x + 1];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                cm[2 * x][w] = s[x][w] & ~cur[w];
                cm[2 * x + 1][w] = s[x][w] & cur[w];
            }
        }
        dr.template compare<2 * NS, kPlanes>(T, cm, live, D);
    }
}
// The same for heat bath: a threshold per class.
template <int NS, uint32_t kPlanes, int W, class Draws>
__device__ __forceinline__ void heat_compare(const Draws &dr, const uint32_t *Tall, const uint32_t (&s)[NS][W],
                                             const uint32_t (&live)[W], uint32_t (&D)[W])
{
    uint32_t T[NS];
#pragma unroll
    for (int x = 0; x < NS; ++x) T[x] = Tall[x];
    dr.template compare<NS, kPlanes>(T, s, live, D);
}

// Contexts: lozenge heat-bath 1, Metropolis 2 (current up); six-vertex
// heat-bath 9 classes 3*sA + sB, Metropolis 18 (2*class + current up), or, when
// the table has 5 or 10 entries, classes by sA + sB alone.
template <int MODE, int W, class Draws>
__device__ __forceinline__ void loz_decide(const Draws &dr, const Thr &Tall, const uint32_t (&cur)[W],
                                           const uint32_t (&live)[W], uint32_t (&D)[W])
{
    if constexpr (MODE == kUniform) {
        dr.one_bit(D);
    } else if constexpr (MODE == kHeatBath) {
        uint32_t T[1] = {Tall.v[0]}, cm[1][W];
#pragma unroll
        for (int w = 0; w < W; ++w) cm[0][w] = ~0u;
        dr.template compare<1, 2>(T, cm, live, D);
    } else {
        uint32_t T[2] = {Tall.v[0], Tall.v[1]}, cm[2][W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            cm[0][w] = ~cur[w];
            cm[1][w] = cur[w];
        }
        dr.template compare<2, 2>(T, cm, live, D);
    }
}

// Points of the free side (no neighbour across it): table Tall.v[kFreeBase ..]
// over the context (first diagonal at m+1) + 2 (second diagonal at m+1)
// [x2: current state up]; the diagonals (hSW, hSE here) are north SW, SE;
// south NW, NE; east SW, NW; west SE, NE.
template <int MODE, int W, class Draws>
__device__ __forceinline__ void sixv_free_decide(const Draws &dr, const Thr &Tall, const uint32_t (&hSW)[W],
                                                 const uint32_t (&hSE)[W], const uint32_t (&cur)[W],
                                                 const uint32_t (&live)[W], uint32_t (&D)[W])
{
    if constexpr (MODE == kUniform) {
        dr.one_bit(D);
    } else {
        uint32_t s[4][W];
#pragma unroll
        for (int w = 0; w < W; ++w)
#pragma unroll
            for (int x = 0; x < 4; ++x) s[x][w] = ((x & 1) ? hSW[w] : ~hSW[w]) & ((x & 2) ? hSE[w] : ~hSE[w]);
        if constexpr (MODE == kMetropolis)
            metro_compare<4, 1>(dr, Tall.v + Thr::kFreeBase, s, cur, live, D);
        else
            heat_compare<4, 1>(dr, Tall.v + Thr::kFreeBase, s, live, D);
    }
}

template <int MODE, int KIND, int W, class Draws>
__device__ __forceinline__ void sixv_decide(const Draws &dr, const Thr &Tall, const uint32_t (&hNE)[W],
                                            const uint32_t (&hNW)[W], const uint32_t (&hSW)[W],
                                            const uint32_t (&hSE)[W], const uint32_t (&cur)[W],
                                            const uint32_t (&live)[W], uint32_t (&D)[W])
{
    if constexpr (MODE == kUniform) {
        dr.one_bit(D);
    } else if constexpr (KIND == kKindSum) {
        // thresholds that depend on sA + sB only (a = b): 5 classes s = 0..4
        uint32_t s[5][W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t A0 = ~hNE[w] & ~hSW[w], A1 = hNE[w] ^ hSW[w], A2 = hNE[w] & hSW[w];
            const uint32_t B0 = ~hNW[w] & ~hSE[w], B1 = hNW[w] ^ hSE[w], B2 = hNW[w] & hSE[w];
            s[0][w] = A0 & B0;
            s[1][w] = (A0 & B1) | (A1 & B0);
            s[2][w] = (A0 & B2) | (A1 & B1) | (A2 & B0);
            s[3][w] = (A1 & B2) | (A2 & B1);
            s[4][w] = A2 & B2;
        }
        if constexpr (MODE == kMetropolis)
            metro_compare<5, 1>(dr, Tall.v, s, cur, live, D);
        else
            heat_compare<5, 1>(dr, Tall.v, s, live, D);
    } else {
        uint32_t s[9][W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t A[3] = {~hNE[w] & ~hSW[w], hNE[w] ^ hSW[w], hNE[w] & hSW[w]};
            const uint32_t B[3] = {~hNW[w] & ~hSE[w], hNW[w] ^ hSE[w], hNW[w] & hSE[w]};
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) s[3 * i + j][w] = A[i] & B[j];
        }
        if constexpr (MODE == kMetropolis)
            metro_compare<9, 1>(dr, Tall.v, s, cur, live, D);
        else
            heat_compare<9, 1>(dr, Tall.v, s, live, D);
    }
}

// What a colour step needs of W words of lozenge sites: the forward (f) and
// backward (b) neighbours, the sites that can move and their current state.
template <int W>
struct LozWords {
    uint32_t O[W], f[W], b[W], live[W], cur[W];
    // m: the words' sites
    __device__ __forceinline__ bool set(const uint32_t (&f1)[W], const uint32_t (&f2)[W], const uint32_t (&f3)[W],
                                        const uint32_t (&b1)[W], const uint32_t (&b2)[W], const uint32_t (&b3)[W],
                                        const uint32_t (&m)[W])
    {
        uint32_t any = 0u;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            f[w] = f1[w];
            b[w] = b1[w];
            live[w] = ~(f1[w] ^ f2[w]) & ~(f1[w] ^ f3[w]) & ~(b1[w] ^ b2[w]) & ~(b1[w] ^ b3[w]) & (f1[w] ^ b1[w]) &
                      m[w];
            cur[w] = ~(O[w] ^ b1[w]);
            any |= live[w];
        }
        return any != 0u;
    }
    template <int MODE, class Draws>
    __device__ __forceinline__ void move(const Draws &dr, const Thr &Tall)
    {
        uint32_t D[W];
        loz_decide<MODE, W>(dr, Tall, cur, live, D);
#pragma unroll
        for (int w = 0; w < W; ++w) O[w] = (O[w] & ~live[w]) | (((D[w] & b[w]) | (~D[w] & f[w])) & live[w]);
    }
};

// The same for six-vertex faces: edge neighbours E, Wn, Nn, Sn, diagonal ones,
// the value `up` of a face at m + 1.  fm: the words' points on the free side.
template <int W>
struct SixvWords {
    uint32_t O[W], E[W], Wn[W], Nn[W], Sn[W], NE[W], NW[W], SE[W], SW[W], fm[W], live[W], up[W], cur[W];
    __device__ __forceinline__ bool set(bool podd, int side, const uint32_t (&m)[W])
    {
        uint32_t any = 0u;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t eEW = ~(E[w] ^ Wn[w]), eEN = ~(E[w] ^ Nn[w]), eES = ~(E[w] ^ Sn[w]);
            // free points: the three neighbours off the free side share m
            const uint32_t lf = side == 1   ? eEW & eES
                                : side == 2 ? eEW & eEN
                                : side == 3 ? ~(Wn[w] ^ Nn[w]) & ~(Wn[w] ^ Sn[w])
                                : side == 4 ? eEN & eES
                                            : 0u;
            live[w] = ((eEW & eEN & eES & ~fm[w]) | (lf & fm[w])) & m[w];
            // residual bit of m + 1 (m read off E, or W across a free east side)
            const uint32_t ref = side == 3 ? (E[w] & ~fm[w]) | (Wn[w] & fm[w]) : E[w];
            up[w] = podd ? ref : ~ref;
            cur[w] = ~(O[w] ^ up[w]);
            any |= live[w];
        }
        return any != 0u;
    }
    template <int MODE, int KIND, bool FREE, class Draws>
    __device__ __forceinline__ void move(const Draws &dr, const Thr &Tall, int side)
    {
        uint32_t D[W], hNE[W], hNW[W], hSW[W], hSE[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            hNE[w] = ~(NE[w] ^ up[w]);
            hNW[w] = ~(NW[w] ^ up[w]);
            hSW[w] = ~(SW[w] ^ up[w]);
            hSE[w] = ~(SE[w] ^ up[w]);
        }
        if constexpr (FREE) {
            uint32_t li[W], lf[W], anyf = 0u;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                li[w] = live[w] & ~fm[w];
                lf[w] = live[w] & fm[w];
                anyf |= lf[w];
            }
            sixv_decide<MODE, KIND, W>(dr, Tall, hNE, hNW, hSW, hSE, cur, li, D);
            if (__any(anyf != 0u)) {
                uint32_t Df[W];
                // context diagonals beside the two cells the flip changes
                const uint32_t (&c0)[W] = side == 2 ? hNW : side == 4 ? hSE : hSW;
                const uint32_t (&c1)[W] = side == 1 ? hSE : side == 3 ? hNW : hNE;
                sixv_free_decide<MODE, W>(dr, Tall, c0, c1, cur, lf, Df);
#pragma unroll
                for (int w = 0; w < W; ++w) D[w] = (D[w] & ~fm[w]) | (Df[w] & fm[w]);
            }
        } else {
            sixv_decide<MODE, KIND, W>(dr, Tall, hNE, hNW, hSW, hSE, cur, live, D);
        }
#pragma unroll
        for (int w = 0; w < W; ++w) O[w] = (O[w] & ~live[w]) | (~(D[w] ^ up[w]) & live[w]);
    }
};

// Sites of word wi of row y in plane p: lozenge X = 3k + p inside the row's
// interior, six-vertex faces 1 <= I = 2k + p <= N - 1.
__device__ __forceinline__ uint32_t loz_row_mask(const Geo &geo, int y, int p, int wi)
{
    const int xlo = imax(0, y - geo.b), xhi = imin(geo.a + geo.c, y + geo.a);
    return range_mask(wi, floordiv(xlo - p, 3) + 1, floordiv(xhi - p - 1, 3));
}
__device__ __forceinline__ uint32_t sixv_row_mask(const Geo &geo, int p, int wi)
{
    return range_mask(wi, p == 0 ? 1 : 0, (geo.N - 1 - p) >> 1);
}

// ---------------------------------------------------------- streaming kernel
// One lozenge group by one lane: sites k = 128 g + (0..127) of plane s0 in
// row Y.
template <int MODE, bool MASKED>
__device__ __forceinline__ void loz_group(uint32_t *base, size_t ps, uint32_t rs, const Geo &geo, int Y, uint32_t g,
                                          uint32_t s0, uint32_t colour, uint32_t t, const Thr &Tall, uint32_t k0,
                                          uint32_t k1)
{
    auto P = [&](uint32_t p, int r) { return base + p * ps + (size_t)r * rs + 4u + 4u * g; };
    LozWords<4> L;
    uint32_t f1[4], f2[4], f3[4], b1[4], b2[4], b3[4], m[4];
    hld4(P(s0, Y), L.O);
    hld4(P(s0, Y + 1), f2);
    hld4(P(s0, Y - 1), b2);
    if (s0 < 2) {
        hld4(P(s0 + 1, Y), f1);
        hld4(P(s0 + 1, Y + 1), f3);
    } else {
        hld4_plus1(P(0, Y), f1);
        hld4_plus1(P(0, Y + 1), f3);
    }
    if (s0 > 0) {
        hld4(P(s0 - 1, Y), b1);
        hld4(P(s0 - 1, Y - 1), b3);
    } else {
        hld4_minus1(P(2, Y), b1);
        hld4_minus1(P(2, Y - 1), b3);
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) m[w] = ~0u;
    if constexpr (MASKED) hld4(geo.site + s0 * geo.sPS + (size_t)Y * geo.sRS + 4u + 4u * g, m);
#pragma unroll
    for (int w = 0; w < 4; ++w) m[w] &= loz_row_mask(geo, Y, (int)s0, (int)(4u * g) + w);
    if (!L.set(f1, f2, f3, b1, b2, b3, m)) return;
    GroupDraws dr{k0, k1, g, (uint32_t)Y, t, colour, {0u, 0u, 0u, 0u}};
    if (MODE == kUniform) philox4x32_10(g, (uint32_t)Y, t, colour, k0, k1, dr.R0);
    L.template move<MODE>(dr, Tall);
    hst4(P(s0, Y), L.O);
}

// One six-vertex group by one lane: faces I = 2k + p, k = 128 g + (0..127), of
// row J.
template <int MODE, int KIND, bool MASKED>
__device__ __forceinline__ void sixv_group(uint32_t *base, size_t ps, uint32_t rs, const Geo &geo, int J, uint32_t g,
                                           uint32_t p, uint32_t colour, uint32_t t, const Thr &Tall, uint32_t k0,
                                           uint32_t k1)
{
    auto P = [&](uint32_t pl, int r) { return base + pl * ps + (size_t)r * rs + 4u + 4u * g; };
    SixvWords<4> S;
    hld4(P(p, J), S.O);
    hld4(P(p, J + 1), S.Nn);
    hld4(P(p, J - 1), S.Sn);
    if (p == 0) {
        hld4(P(1, J), S.E);
        hld4_minus1(P(1, J), S.Wn);
        hld4(P(1, J + 1), S.NE);
        hld4_minus1(P(1, J + 1), S.NW);
        hld4(P(1, J - 1), S.SE);
        hld4_minus1(P(1, J - 1), S.SW);
    } else {
        hld4_plus1(P(0, J), S.E);
        hld4(P(0, J), S.Wn);
        hld4_plus1(P(0, J + 1), S.NE);
        hld4(P(0, J + 1), S.NW);
        hld4_plus1(P(0, J - 1), S.SE);
        hld4(P(0, J - 1), S.SW);
    }
    uint32_t m[4];
    int side = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        m[w] = ~0u;
        S.fm[w] = 0u;
    }
    if constexpr (MASKED) {
        hld4(geo.site + p * geo.sPS + (size_t)J * geo.sRS + 4u + 4u * g, m);
        // points of the free side ignore their (absent) neighbour across it
        if (geo.freep) {
            hld4(geo.freep + p * geo.sPS + (size_t)J * geo.sRS + 4u + 4u * g, S.fm);
            side = geo.free_side;
        }
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) m[w] &= sixv_row_mask(geo, (int)p, (int)(4u * g) + w);
    if (!S.set(((p + (uint32_t)J) & 1u) != 0u, side, m)) return;
    GroupDraws dr{k0, k1, g, (uint32_t)J, t, colour, {0u, 0u, 0u, 0u}};
    if (MODE == kUniform) philox4x32_10(g, (uint32_t)J, t, colour, k0, k1, dr.R0);
    S.template move<MODE, KIND, MASKED>(dr, Tall, side);
    hst4(P(p, J), S.O);
}

// Which plane of row y holds the sites of colour c (-1: none in this row).
__device__ __forceinline__ int colour_plane(const Geo &geo, int y, uint32_t c)
{
    if (geo.model == TL_LOZENGE) return (int)((c + 3u * 1024u - (uint32_t)y % 3u) % 3u);
    return ((c >> 1) == ((uint32_t)y & 1u)) ? (int)(c & 1u) : -1;
}

// Site rows: lozenge 1 .. b+c-1, six-vertex 1 .. N-1.
__device__ __forceinline__ bool site_row(const Geo &geo, int y, uint32_t rows)
{
    return y >= 1 && y <= (int)rows - 2;
}

template <int MODE, int KIND, bool MASKED>
__global__ void __launch_bounds__(256) height_step_kernel(uint32_t *planes, size_t PS, uint32_t RS, uint32_t ng,
                                                          uint32_t rows, Geo geo, uint32_t colour, uint32_t t, Thr T,
                                                          uint32_t k0, uint32_t k1)
{
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t g = gid % ng, y = gid / ng;
    if (!site_row(geo, (int)y, rows)) return;
    const int pl = colour_plane(geo, (int)y, colour);
    if (pl < 0) return;
    if (geo.model == TL_LOZENGE)
        loz_group<MODE, MASKED>(planes, PS, RS, geo, (int)y, g, (uint32_t)pl, colour, t, T, k0, k1);
    else
        sixv_group<MODE, KIND, MASKED>(planes, PS, RS, geo, (int)y, g, (uint32_t)pl, colour, t, T, k0, k1);
}

// ------------------------------------------------------------ tiled kernels
// One tile, many sweeps.  A tile's state is small, and few of its sites can
// move at a time (what moves is a band between the frozen parts of an extremal
// start, or between the arctic regions).  What bounds a launch is the chain of
// colour steps, each as long as its slowest wavefront's chain of dependent
// instructions (4 to 5 clocks each, some 35 for a taken branch, 70 to 130 for
// an LDS read; a Philox call alone is 260).  So:
//   * a wavefront holds a granule, 16 task rows of one group of 128 sites, a
//     lane per (row, word of 32 sites), and runs straight-line code per colour;
//   * a step looks only at granules that can hold a movable site: those that
//     had one, or have a neighbour that had one, since their sites of the
//     step's colour were last looked at (`stamp`, the last step with one);
//   * a granule that had a movable site lately draws ahead while its LDS reads
//     are under way, a draw being a function of counters known in advance: the
//     planes 0..7 of the next step (bit-serial decisions; they settle all but
//     one site in 256) or plane 0 of the next four steps (one-bit decisions).
//     Each of a row's four lanes makes one draw in four, and a transpose hands
//     every lane its word of them.  Other draws are made on the spot.
// A tile with no movable site at all is written back at once.
//
// LDS, in words: a guard row, P planes of the state, P planes of the sites
// that may move (zero outside the tile's inner rows and groups), the stamps of
// the granules.  Local row lr is global row R0 + lr, local group lg is global
// group G0 + lg, in slot lg + 1 of its row (the slots around hold the
// neighbouring groups, or zero).  Rows have an odd number of slots where LDS
// allows, so that the 16 rows of a granule fall in distinct banks; six-vertex
// rows are kept even rows first, then odd ones, since a colour step takes rows of
// one parity.
//
// With a row halo, the rows still valid before sweep s are [rps*s, LR - rps*s)
// (rps rows go stale per sweep on each side), and only those move.  Under the
// random colour order (RANDOM) step n of the launch (K per sweep) draws its
// colour and moves rows [n, LR - n).
constexpr uint32_t kWindow = 8;       // steps after its last movable site that a granule draws ahead

// Word at byte offset `at` of a tile's LDS.
__device__ __forceinline__ uint32_t ldw(const uint32_t *lds, uint32_t at)
{
    return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(lds) + at);
}
__device__ __forceinline__ void stw(uint32_t *lds, uint32_t at, uint32_t v)
{
    *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(lds) + at) = v;
}
// Sites 32 wi + b, b = 0..31, with klo <= site <= khi, as a mask.
__device__ __forceinline__ uint32_t clamp_mask(int klo, int khi, int wi)
{
    const int a = imin(imax(klo - 32 * wi, 0), 32), b = imin(imax(khi + 1 - 32 * wi, 0), 32);
    return (uint32_t)(0xFFFFFFFFull << a) & ~(uint32_t)(0xFFFFFFFFull << b);
}

// Words the threads of a tile share besides the planned LDS: whether it has a
// movable site, and the ring of colours.  Declared once in each kernel: as
// statics of height_tile a multi-job kernel had them once for each of its bodies.
template <bool RANDOM>
constexpr uint32_t kCommonWords = RANDOM ? 1u + kColourRing : 1u;
// GEOM: the model.
enum { kGeomLozenge = 1, kGeomSixv = 2 };
template <int MODE, int KIND, bool RANDOM, bool MASKED, int GEOM>
__device__ __forceinline__ void height_tile(uint32_t *lds, uint32_t *common, const uint32_t *__restrict__ in,
                                            uint32_t *__restrict__ out, size_t PS, uint32_t RS, uint32_t ng,
                                            uint32_t rows, const Geo &geo, uint32_t t0, uint32_t nsweeps,
                                            uint32_t TR, uint32_t TG, uint32_t HR, uint32_t HG, uint32_t tile_r,
                                            uint32_t tile_g, const Thr &T, uint32_t k0, uint32_t k1)
{
    constexpr bool ONEBIT = MODE == kUniform, sixv = GEOM == kGeomSixv;
    constexpr uint32_t P = sixv ? 2u : 3u, K = sixv ? 4u : 3u, rps = sixv ? 2u : 3u;
    const uint32_t LR = TR + 2 * HR, LG = TG + 2 * HG;
    const HeightLds lay = height_lds(sixv, LR, LG);
    // byte strides
    const uint32_t LRS = 4u * lay.row_words, LPS = lay.plane_rows * LRS, trows = lay.task_rows;
    const uint32_t H = lay.plane_rows / 2u * LRS;   // six-vertex: odd rows after even ones
    const uint32_t NG = lay.granules, RB = lay.row_blocks;
    const uint32_t state = LRS, site = state + P * LPS;
    uint32_t *stamp = lds + ((site + P * LPS) >> 2);
    uint32_t *const live = common, *const ring = common + 1;   // the tile has a movable site; its colours
    const int R0 = (int)(tile_r * TR) - (int)HR, G0 = (int)(tile_g * TG) - (int)HG;
    const uint32_t tid = threadIdx.x, nt = blockDim.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = nt >> 6;
    const uint32_t row = lane & 15u, q = lane >> 4;
    auto phys = [&](uint32_t lr) { return sixv ? (lr >> 1) * LRS + (lr & 1u) * H : lr * LRS; };

    // (slot, row, plane) of item i = tid, tid + nt, ... of nslots x nrows x P
    auto each = [&](uint32_t nslots, uint32_t nrows, auto &&f) {
        uint32_t sl = tid % nslots, lr = tid / nslots, p = 0u;
        const uint32_t dsl = nt % nslots, dlr = nt / nslots;
        while (true) {
            while (lr >= nrows) {
                lr -= nrows;
                ++p;
            }
            if (p >= P) break;
            f(sl, lr, p);
            sl += dsl;
            lr += dlr;
            if (sl >= nslots) {
                sl -= nslots;
                ++lr;
            }
        }
    };
    // state, and the sites of the inner rows and groups
    each(LG + 2u, LR, [&](uint32_t sl, uint32_t lr, uint32_t p) {
        const int gr = R0 + (int)lr, gg = G0 - 1 + (int)sl;   // global group, -1 .. ng = pads
        uint32_t v[4] = {0u, 0u, 0u, 0u}, m[4] = {0u, 0u, 0u, 0u};
        if (gr >= 0 && gr < (int)rows && gg >= -1 && gg <= (int)ng)
            hld4(in + p * PS + (size_t)gr * RS + 4 + 4 * gg, v);
        if (sl >= 1u && sl <= LG && gg >= 0 && gg < (int)ng && lr >= 1u && lr + 1u < LR && site_row(geo, gr, rows)) {
            int klo, khi;
            if (sixv) {   // faces 1 <= I = 2k + p <= N - 1
                klo = p == 0u ? 1 : 0;
                khi = (geo.N - 1 - (int)p) >> 1;
            } else {      // vertices X = 3k + p inside the row's interior
                const int xlo = imax(0, gr - geo.b), xhi = imin(geo.a + geo.c, gr + geo.a);
                klo = (int)((uint32_t)(xlo + 3 - (int)p) / 3u);
                khi = (int)((uint32_t)(xhi + 2 - (int)p) / 3u) - 1;
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) m[w] = clamp_mask(klo, khi, 4 * gg + w);
            if constexpr (MASKED) {
                uint32_t sm[4];
                hld4(geo.site + p * geo.sPS + (size_t)gr * geo.sRS + 4 + 4 * gg, sm);
#pragma unroll
                for (int w = 0; w < 4; ++w) m[w] &= sm[w];
            }
        }
        const uint32_t at = (p * LPS + phys(lr) + 16u * sl) >> 2;
        hst4(lds + (state >> 2) + at, v);
        hst4(lds + (site >> 2) + at, m);
    });
    if constexpr (RANDOM)
        for (uint32_t i = tid; i < kColourRing; i += nt) ring[i] = step_colour(K * t0 + i, K, k0, k1);
    for (uint32_t i = tid; i < NG; i += nt) stamp[i] = 0u;
    if (tid == 0u) *live = 0u;
    __syncthreads();

    auto colour_of = [&](uint32_t n) { return RANDOM ? ring[n & (kColourRing - 1u)] : n % K; };
    // six-vertex: local rows of a step of colour c are 2i + odd_rows(c)
    auto odd_rows = [&](uint32_t c) { return ((uint32_t)R0 & 1u) ^ (c >> 1); };

    // gi / RB (gi * RB < 2^16)
    const uint32_t invRB = (0xFFFFu + RB) / RB;
    auto group_of = [&](uint32_t gi) { return (gi * invRB) >> 16; };

    // A granule's lanes: byte offset of this lane's word (plane 0; six-vertex:
    // of the even row), its local row (six-vertex: the even one), its group.
    // Lanes past the last task row read that row and move nothing (their local
    // row is past every valid one).  Lozenges: the word's offsets in the planes
    // of the row's sites of colours 0, 1 and 2, and which of them is plane 2;
    // the forward neighbours in the row lie in the next colour's plane (one
    // word position on from plane 2 to plane 0), the backward ones in the plane
    // before (one position back from plane 0 to plane 2).
    struct Lane {
        uint32_t at, lr, g, gr, off[3], near;
        bool last[3];
    };
    auto lane_of = [&](uint32_t gi) {
        const uint32_t lg = group_of(gi), rb = gi - lg * RB, i = 16u * rb + row;
        Lane l;
        l.at = state + imin(i, trows - 1u) * LRS + 16u * lg + 16u + 4u * q;
        l.lr = i < trows ? (sixv ? 2u * i : i) : 1u << 30;
        l.gr = (uint32_t)(R0 + (int)(sixv ? 2u * i : i));
        l.g = (uint32_t)(G0 + (int)lg);
        if constexpr (!sixv) {
            const uint32_t y3 = (l.gr + 3u * 1024u) % 3u;
#pragma unroll
            for (uint32_t c = 0; c < 3u; ++c) {
                const uint32_t d = c + 3u - y3, s = d >= 3u ? d - 3u : d;
                l.off[c] = l.at + s * LPS;
                l.last[c] = s == 2u;
            }
        }
        // granule whose stamp this lane reads: lane d < 9 looks at the
        // neighbourhood (d / 3 - 1, d % 3 - 1)
        const int d = (int)(lane < 9u ? lane : 4u), l2 = (int)lg + d / 3 - 1, r2 = (int)rb + d % 3 - 1;
        l.near = l2 >= 0 && l2 < (int)LG && r2 >= 0 && r2 < (int)RB ? (uint32_t)l2 * RB + (uint32_t)r2 : gi;
        return l;
    };

    // A colour step's view of a granule: what its words need, and whether any
    // of its sites in rows [lo, hi) can move.
    using Words = std::conditional_t<sixv, SixvWords<1>, LozWords<1>>;
    struct View {
        Words w;
        uint32_t o, any;
        int side;
    };
    auto look = [&](auto ctag, const Lane &l, uint32_t lo, uint32_t hi, auto &&meanwhile) {
        constexpr uint32_t C = decltype(ctag)::value;
        View v;
        v.side = 0;
        if constexpr (!sixv) {
            constexpr uint32_t F = (C + 1u) % 3u, B = (C + 2u) % 3u;
            const uint32_t o = l.off[C], f = l.off[F], b = l.off[B];
            const uint32_t O = ldw(lds, o), f2 = ldw(lds, o + LRS), b2 = ldw(lds, o - LRS);
            const uint32_t fa = ldw(lds, f), fa1 = ldw(lds, f + 4u), fc = ldw(lds, f + LRS), fc1 = ldw(lds, f + LRS + 4u);
            const uint32_t ba1 = ldw(lds, b - 4u), ba = ldw(lds, b), bc1 = ldw(lds, b - LRS - 4u), bc = ldw(lds, b - LRS);
            const uint32_t sm = ldw(lds, o + P * LPS);
            meanwhile();
            const uint32_t m[1] = {l.lr - lo < hi - lo ? sm : 0u};
            const bool wf = l.last[C], wb = l.last[B];   // the own plane is plane 2, plane 0
            const uint32_t f1[1] = {wf ? __builtin_amdgcn_alignbit(fa1, fa, 1) : fa};
            const uint32_t f3[1] = {wf ? __builtin_amdgcn_alignbit(fc1, fc, 1) : fc};
            const uint32_t b1[1] = {wb ? __builtin_amdgcn_alignbit(ba, ba1, 31) : ba};
            const uint32_t b3[1] = {wb ? __builtin_amdgcn_alignbit(bc, bc1, 31) : bc};
            const uint32_t f2a[1] = {f2}, b2a[1] = {b2};
            v.w.O[0] = O;
            v.o = o;
            v.w.set(f1, f2a, f3, b1, b2a, b3, m);
        } else {
            constexpr uint32_t p = C & 1u;
            const uint32_t odd = odd_rows(C);
            // rows J, J + 1, J - 1 in the split order
            const uint32_t pl = l.at + p * LPS, xl = l.at + (1u - p) * LPS;
            const uint32_t a0 = odd ? H : 0u, aN = odd ? LRS : H, aS = odd ? 0u : H - LRS;
            const uint32_t x = xl + a0, xN = xl + aN, xS = xl + aS;
            SixvWords<1> &S = v.w;
            v.o = pl + a0;
            const uint32_t O = ldw(lds, v.o), Nn = ldw(lds, pl + aN), Sn = ldw(lds, pl + aS);
            const uint32_t sm = ldw(lds, v.o + P * LPS);
            // the other plane's words beside: to the left of even, to the right of odd columns
            const uint32_t x0 = ldw(lds, x), n0 = ldw(lds, xN), s0 = ldw(lds, xS);
            const uint32_t x1 = ldw(lds, p ? x + 4u : x - 4u), n1 = ldw(lds, p ? xN + 4u : xN - 4u),
                           s1 = ldw(lds, p ? xS + 4u : xS - 4u);
            meanwhile();
            const uint32_t m[1] = {l.lr + odd - lo < hi - lo ? sm : 0u};
            S.fm[0] = 0u;
            if constexpr (MASKED) {
                if (geo.freep) {
                    v.side = geo.free_side;
                    // a site lies inside the state, its lane may be a halo row outside
                    if (m[0]) S.fm[0] = geo.freep[p * geo.sPS + (size_t)(l.gr + odd) * geo.sRS + 4u + 4u * l.g + q];
                }
            }
            S.O[0] = O;
            S.Nn[0] = Nn;
            S.Sn[0] = Sn;
            auto west = [](uint32_t w, uint32_t beside) { return p ? w : __builtin_amdgcn_alignbit(w, beside, 31); };
            auto east = [](uint32_t w, uint32_t beside) { return p ? __builtin_amdgcn_alignbit(beside, w, 1) : w; };
            S.E[0] = east(x0, x1);
            S.Wn[0] = west(x0, x1);
            S.NE[0] = east(n0, n1);
            S.NW[0] = west(n0, n1);
            S.SE[0] = east(s0, s1);
            S.SW[0] = west(s0, s1);
            S.set(((p + l.gr + odd) & 1u) != 0u, v.side, m);
        }
        v.any = __any(v.w.live[0] != 0u);
        return v;
    };
    auto row_of = [&](const Lane &l, uint32_t c) { return sixv ? l.gr + odd_rows(c) : l.gr; };
    // The draws of a granule ahead: bit-serial, planes 0..7 for colour c, counter
    // t; one-bit, plane 0 for the steps n .. n + 3.
    auto draw = [&](const Lane &l, uint32_t n, uint32_t c, uint32_t t, uint32_t (&A)[ONEBIT ? 4 : kAheadPlanes]) {
        if constexpr (ONEBIT) {
            const uint32_t cq = colour_of(n + q), tq = RANDOM ? K * t0 + n + q : t0 + (n + q) / K;
            philox4x32_10(l.g, row_of(l, cq), tq, cq, k0, k1, A);
            rows_transpose(A);
        } else {
#pragma unroll
            for (uint32_t h = 0; h < kAheadPlanes / 4u; ++h) {
                uint32_t R[4];
                philox4x32_10(l.g, row_of(l, c), t, ((4u * h + q) << 2) | c, k0, k1, R);
                rows_transpose(R);
#pragma unroll
                for (uint32_t x = 0; x < 4u; ++x) A[4u * h + x] = R[x];
            }
        }
    };
    auto move = [&](auto ctag, const Lane &l, View &v, uint32_t t, bool ready, const uint32_t *A) {
        constexpr uint32_t C = decltype(ctag)::value;
        const WordDraws dr{k0, k1, l.g, row_of(l, C), t, C, q, ready, A};
        if constexpr (sixv)
            v.w.template move<MODE, KIND, MASKED>(dr, T, v.side);
        else
            v.w.template move<MODE>(dr, T);
        // lanes with nothing to move write to the guard row
        stw(lds, v.w.live[0] ? v.o : 4u * q, v.w.O[0]);
    };
    // f(colour as a compile-time constant)
    auto with_colour = [&](uint32_t c, auto &&f) {
        if (c == 0u) f(std::integral_constant<uint32_t, 0u>{});
        else if (c == 1u) f(std::integral_constant<uint32_t, 1u>{});
        else if (K == 3u || c == 2u) f(std::integral_constant<uint32_t, 2u>{});
        else f(std::integral_constant<uint32_t, K - 1u>{});
    };
    auto every_colour = [&](auto &&f) {
        f(std::integral_constant<uint32_t, 0u>{});
        f(std::integral_constant<uint32_t, 1u>{});
        f(std::integral_constant<uint32_t, 2u>{});
        if constexpr (K == 4u) f(std::integral_constant<uint32_t, 3u>{});
    };

    if (LR >= 3u) {
        const Lane first = lane_of(wave < NG ? wave : 0u);
        // granules with a site that can move, in any colour; none: the tile
        // stays as it is
        bool live0 = false;   // of this wavefront's first granule
        for (uint32_t gi = wave; gi < NG; gi += waves) {
            const Lane l = gi == wave ? first : lane_of(gi);
            uint32_t any = 0u;
            every_colour([&](auto ctag) { any |= look(ctag, l, 0u, LR, [] {}).any; });
            if (any) {
                stamp[gi] = 1u;
                *live = 1u;
            }
            if (gi == wave) live0 = any != 0u;
        }
        __syncthreads();
        const uint32_t steps = K * nsweeps;
        auto can_move = [&](uint32_t near, uint32_t n) {   // since the step's colour was last looked at
            const uint32_t st = stamp[near];
            return __any(st != 0u && (RANDOM || st + K >= n)) != 0;
        };
        if (*live != 0u && NG <= waves) {
            // a granule per wavefront, its draws ahead in registers
            uint32_t A[ONEBIT ? 4 : kAheadPlanes], N[ONEBIT ? 4 : kAheadPlanes];
            // One-bit: the plane of step n is A[n % 4] where that is the step's
            // colour, else A[0], the planes moving down one a step: an index by n
            // would put A in private memory.
            constexpr bool kIndexed = ONEBIT && !RANDOM && K == 4u;
#pragma unroll
            for (uint32_t x = 0; x < sizeof(A) / 4u; ++x) A[x] = N[x] = 0u;
            uint32_t seen = live0 && wave < NG ? kWindow : 0u;   // steps left to draw ahead in
            uint32_t ready = seen;   // A holds the draws (one-bit: of the current four steps)
            const uint32_t c0 = RANDOM ? (uint32_t)__builtin_amdgcn_readfirstlane(colour_of(0u)) : 0u;
            if (ready) draw(first, 0u, c0, RANDOM ? K * t0 : t0, A);
            auto step = [&](auto ctag, uint32_t n, uint32_t t, uint32_t lo, uint32_t cn, uint32_t tn) {
                if (wave >= NG) return;
                if (seen == 0u && !can_move(first.near, n)) {
                    ready = 0u;
                    return;
                }
                const bool ahead = ONEBIT ? seen != 0u && (n & 3u) == 3u : seen != 0u;
                View v = look(ctag, first, lo, LR - lo, [&] {
                    if (ahead) draw(first, n + 1u, cn, tn, N);
                });
                if (v.any) {
                    move(ctag, first, v, t, ready != 0u, kIndexed ? A + decltype(ctag)::value : A);
                    stamp[wave] = n + 1u;
                    seen = kWindow;
                } else if (seen) {
                    --seen;
                }
                if (!ONEBIT || (n & 3u) == 3u) {
                    ready = ahead;
#pragma unroll
                    for (uint32_t x = 0; x < sizeof(A) / 4u; ++x) A[x] = N[x];
                } else if constexpr (!kIndexed) {
#pragma unroll
                    for (uint32_t x = 0; x + 1u < sizeof(A) / 4u; ++x) A[x] = A[x + 1u];
                }
            };
            if constexpr (RANDOM) {
                uint32_t c = c0;
                for (uint32_t n = 0; n < steps; ++n) {
                    const uint32_t cn = (uint32_t)__builtin_amdgcn_readfirstlane(colour_of(n + 1u));
                    with_colour(c, [&](auto ctag) { step(ctag, n, K * t0 + n, HR ? n : 0u, cn, K * t0 + n + 1u); });
                    c = cn;
                    if (wave == waves - 1u && (n & 63u) == 0u && n)
                        ring[(n + 64u + lane) & (kColourRing - 1u)] = step_colour(K * t0 + n + 64u + lane, K, k0, k1);
                    __syncthreads();
                }
            } else {
                for (uint32_t s = 0; s < nsweeps; ++s)
                    every_colour([&](auto ctag) {
                        constexpr uint32_t C = decltype(ctag)::value;
                        step(ctag, K * s + C, t0 + s, HR ? rps * s : 0u, C + 1u == K ? 0u : C + 1u,
                             C + 1u == K ? t0 + s + 1u : t0 + s);
                        __syncthreads();
                    });
            }
        } else if (*live != 0u) {
            // more granules than wavefronts: taken in turns, every draw on the spot
            for (uint32_t n = 0; n < steps; ++n) {
                const uint32_t c = RANDOM ? (uint32_t)__builtin_amdgcn_readfirstlane(colour_of(n)) : n % K;
                const uint32_t t = RANDOM ? K * t0 + n : t0 + n / K, lo = HR ? (RANDOM ? n : rps * (n / K)) : 0u;
                for (uint32_t gi = wave; gi < NG; gi += waves) {
                    const Lane l = lane_of(gi);
                    if (!can_move(l.near, n)) continue;
                    with_colour(c, [&](auto ctag) {
                        View v = look(ctag, l, lo, LR - lo, [] {});
                        if (!v.any) return;
                        move(ctag, l, v, t, false, nullptr);
                        stamp[gi] = n + 1u;
                    });
                }
                if constexpr (RANDOM)
                    if (wave == waves - 1u && (n & 63u) == 0u && n)
                        ring[(n + 64u + lane) & (kColourRing - 1u)] = step_colour(K * t0 + n + 64u + lane, K, k0, k1);
                __syncthreads();
            }
        }
    }

    each(TG, TR, [&](uint32_t ig, uint32_t ir, uint32_t p) {
        const uint32_t orow = tile_r * TR + ir, og = tile_g * TG + ig;
        if (orow >= rows || og >= ng) return;
        uint32_t v[4];
        hld4(lds + ((state + p * LPS + phys(ir + HR) + 16u * (ig + HG + 1u)) >> 2), v);
        hst4(out + p * PS + (size_t)orow * RS + 4 + 4 * og, v);
    });
}

// Tiled multi-sweep kernels of one state: one work-group per tile.
template <int MODE, int KIND, bool RANDOM, bool MASKED>
__global__ void __launch_bounds__(kTileThreads) height_tiled_kernel(const uint32_t *__restrict__ in,
                                                            uint32_t *__restrict__ out, size_t PS, uint32_t RS,
                                                            uint32_t ng, uint32_t rows, Geo geo, uint32_t t0,
                                                            uint32_t nsweeps, uint32_t TR, uint32_t TG,
                                                            uint32_t HR, uint32_t HG, uint32_t tiles_x, Thr T,
                                                            uint32_t k0, uint32_t k1)
{
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t common[kCommonWords<RANDOM>];
    // plain work-group order: tiles of a hexagon differ in work, and the
    // round-robin dispatch over the XCDs balances them
    height_tile<MODE, KIND, RANDOM, MASKED, kGeomSixv>(lds, common, in, out, PS, RS, ng, rows, geo, t0, nsweeps, TR,
                                                       TG, HR, HG, blockIdx.x / tiles_x, blockIdx.x % tiles_x, T, k0,
                                                       k1);
}
template <int MODE, int KIND, bool RANDOM, bool MASKED>
__global__ void __launch_bounds__(kTileThreads) loz_tiled_kernel(const uint32_t *__restrict__ in,
                                                        uint32_t *__restrict__ out, size_t PS, uint32_t RS,
                                                        uint32_t ng, uint32_t rows, Geo geo, uint32_t t0,
                                                        uint32_t nsweeps, uint32_t TR, uint32_t TG, uint32_t HR,
                                                        uint32_t HG, uint32_t tiles_x, Thr T, uint32_t k0, uint32_t k1)
{
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t common[kCommonWords<RANDOM>];
    height_tile<MODE, kKindClass, RANDOM, MASKED, kGeomLozenge>(lds, common, in, out, PS, RS, ng, rows, geo, t0,
                                                                nsweeps, TR, TG, HR, HG, blockIdx.x / tiles_x,
                                                                blockIdx.x % tiles_x, T, k0, k1);
}

// Multi-job kernel: work-group b runs tile items[b].tile of job items[b].job,
// with that job's geometry, plan, thresholds and key.
template <int MODE, int KIND, bool RANDOM, bool MASKED>
__device__ __forceinline__ void height_item(uint32_t *lds, uint32_t *common, const TileJob &j, uint32_t tile)
{
    const Geo geo{j.model, j.a, j.b, j.c, j.N, j.site, j.PS, j.RS, j.freep, j.free_side};
    const uint32_t tile_r = tile / j.tiles_x, tile_g = tile % j.tiles_x;
    if (j.model == TL_LOZENGE)   // lozenge tables are always classes
        height_tile<MODE, kKindClass, RANDOM, MASKED, kGeomLozenge>(lds, common, j.in, j.out, j.PS, j.RS, j.ng,
                                                                    j.rows, geo, j.t0, j.S, j.TR, j.TG, j.HR, j.HG,
                                                                    tile_r, tile_g, j.T, j.key0, j.key1);
    else
        height_tile<MODE, KIND, RANDOM, MASKED, kGeomSixv>(lds, common, j.in, j.out, j.PS, j.RS, j.ng, j.rows, geo,
                                                           j.t0, j.S, j.TR, j.TG, j.HR, j.HG, tile_r, tile_g, j.T,
                                                           j.key0, j.key1);
}

// Every job of a launch has the colour order RANDOM, and site planes iff MASKED.
template <int MODE, int KIND, bool RANDOM, bool MASKED>
__global__ void __launch_bounds__(kTileThreads) height_items_kernel(const TileJob *__restrict__ jobs,
                                                                      const TileItem *__restrict__ items)
{
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t common[kCommonWords<RANDOM>];
    const TileItem it = items[blockIdx.x];
    const TileJob &j = jobs[it.job];
    if constexpr (MODE == kHeatBath) {
        // one-bit jobs share the heat-bath launches (the lighter kernel body)
        if (j.mode == kUniform) {
            height_item<kUniform, kKindClass, RANDOM, MASKED>(lds, common, j, it.tile);
            return;
        }
    }
    height_item<MODE, KIND, RANDOM, MASKED>(lds, common, j, it.tile);
}

// The same with every rule and table layout in one launch: work-group b takes
// the kernel body of its job's rule and layout (the served ticks, where jobs of
// several rules share one launch instead of a launch per rule on streams
// joined by events).
template <bool RANDOM, bool MASKED>
__global__ void __launch_bounds__(kTileThreads) height_items_mixed_kernel(const TileJob *__restrict__ jobs,
                                                                            const TileItem *__restrict__ items)
{
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t common[kCommonWords<RANDOM>];
    const TileItem it = items[blockIdx.x];
    const TileJob &j = jobs[it.job];
    if (j.mode == kUniform)
        height_item<kUniform, kKindClass, RANDOM, MASKED>(lds, common, j, it.tile);
    else if (j.mode == kMetropolis)
        j.kind == kKindSum ? height_item<kMetropolis, kKindSum, RANDOM, MASKED>(lds, common, j, it.tile)
                           : height_item<kMetropolis, kKindClass, RANDOM, MASKED>(lds, common, j, it.tile);
    else
        j.kind == kKindSum ? height_item<kHeatBath, kKindSum, RANDOM, MASKED>(lds, common, j, it.tile)
                           : height_item<kHeatBath, kKindClass, RANDOM, MASKED>(lds, common, j, it.tile);
}

__device__ __forceinline__ uint32_t hbit(const uint32_t *pl, size_t PS, uint32_t RS, uint32_t p, uint32_t y,
                                         uint32_t k)
{
    return (pl[p * PS + (size_t)y * RS + 4 + (k >> 5)] >> (k & 31u)) & 1u;
}

// Bits k of a row word whose bit k is the point X0 + s k + p (the s planes
// of a row interleave their points) with u <= X0 + s k + p <= v.
__device__ __forceinline__ uint32_t word_mask(int X0, int p, int u, int v, int s)
{
    const int a = u - X0 - p, b = v - X0 - p;
    const int klo = a <= 0 ? 0 : (a + s - 1) / s, khi = b < 0 ? -1 : imin(31, b / s);
    if (klo > khi) return 0u;
    const uint32_t upto = khi >= 31 ? ~0u : (2u << khi) - 1u;
    return upto & ~((1u << klo) - 1u);
}

// Sum of the indices k of the set bits of x.
__device__ __forceinline__ uint32_t bit_index_sum(uint32_t x)
{
    return (uint32_t)__popc(x & 0xAAAAAAAAu) + 2u * (uint32_t)__popc(x & 0xCCCCCCCCu) +
           4u * (uint32_t)__popc(x & 0xF0F0F0F0u) + 8u * (uint32_t)__popc(x & 0xFF00FF00u) +
           16u * (uint32_t)__popc(x & 0xFFFF0000u);
}

// Heights of every point of a row, one wavefront per row.  A chunk is word m
// of each plane: lozenge vertices X in [96m, 96m + 96) (bit k of plane p is
// X = 96m + 3k + p), six-vertex faces I in [64m, 64m + 64) (I = 64m + 2k + p).
// Along a lozenge row H falls by one exactly where the residual bit differs
// from the previous vertex's.  Along a six-vertex row h moves by one at every
// face, and, the bit being bit 1 of h and h having the parity of I + J, it
// goes up exactly where the bit, the previous face's bit and that parity XOR
// to 1.  So each chunk's step words are XORs of its planes: phase one keeps
// them in LDS with the count of steps before the chunk (a wavefront prefix
// sum); phase two writes the row, consecutive lanes on consecutive points,
// each height the row's first one moved by popcounts of the steps up to it.
// LDS: nch words of counts, then 3 nch (lozenge) or 2 nch step words.
__global__ void __launch_bounds__(64) height_export_kernel(const uint32_t *pl, size_t PS, uint32_t RS, Geo geo,
                                                           uint32_t nch, int32_t *out)
{
    extern __shared__ uint32_t xl[];
    const int y = (int)blockIdx.x, lane = (int)threadIdx.x;
    const uint32_t *row = pl + (size_t)y * RS + 4;
    uint32_t *pre = xl, *steps = xl + nch;
    const bool loz = geo.model == TL_LOZENGE;
    const int P = loz ? 3 : 2, span = loz ? 96 : 64;
    // the row's points with a step, and (lozenge) its vertices
    const int xs = loz ? loz_xs(geo, y) : 0, xe = loz ? loz_xe(geo, y) : geo.N;
    int carry = 0;
    for (int m0 = 0; m0 < (int)nch; m0 += 64) {
        const int m = m0 + lane, X0 = span * m;
        const int lo = imax(xs, X0), hi = imin(xe, X0 + span - 1), L = imax(lo, xs + 1);
        uint32_t S[3] = {0u, 0u, 0u};
        int cnt = 0;
        if (m < (int)nch && lo <= hi) {
            if (loz) {
                const uint32_t W0 = row[m], W1 = row[PS + m], W2 = row[2 * PS + m];
                const uint32_t cin = X0 > xs ? row[2 * PS + m - 1] >> 31 : 0u;   // the vertex before X0
                S[0] = W0 ^ ((W2 << 1) | cin);
                S[1] = W1 ^ W0;
                S[2] = W2 ^ W1;
            } else {
                const uint32_t P0 = row[m], P1 = row[PS + m];
                const uint32_t cin = m > 0 ? row[PS + m - 1] >> 31 : 0u;   // the face before I = 64m
                const uint32_t par0 = (y & 1) ? ~0u : 0u;                  // parity of I + J, I even
                S[0] = P0 ^ ((P1 << 1) | cin) ^ par0;
                S[1] = P1 ^ P0 ^ ~par0;
            }
            for (int p = 0; p < P; ++p) cnt += __popc(S[p] & word_mask(X0, p, L, hi, P));
        }
        int incl = cnt;   // inclusive scan over the lanes
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off, 64);
            if (lane >= off) incl += v;
        }
        if (m < (int)nch) {
            pre[m] = (uint32_t)(carry + incl - cnt);
            for (int p = 0; p < P; ++p) steps[P * m + p] = S[p];
        }
        carry += __shfl(incl, 63, 64);
    }
    __syncthreads();
    const int W = loz ? geo.a + geo.c + 1 : geo.N + 1;
    const int h0 = loz ? loz_hmin(geo, xs, y) : y;   // lozenge H at xs, six-vertex h(0, J) = J
    int32_t *o = out + (size_t)y * W;
    for (int X = lane; X < W; X += 64) {
        int32_t v = INT32_MIN;
        if (X >= xs && X <= xe) {
            const int m = X / span, X0 = span * m, L = imax(imax(xs, X0), xs + 1);
            int c = (int)pre[m];
            for (int p = 0; p < P; ++p) c += __popc(steps[P * m + p] & word_mask(X0, p, L, X, P));
            v = loz ? h0 - c : h0 + 2 * c - X;
        }
        o[X] = v;
    }
}

// Six-vertex observable: the type-c vertices (both diagonal pairs of faces
// around the vertex equal) counted into bins of B x B cells (cell (i-1, j-1) =
// vertex (i, j), 1 <= i, j <= N).  One thread per vertex row j and word w: the
// word holds vertices i = 2k+1 (faces I = 2k, 2k+1 from planes 0 and 1) and
// i = 2k+2 (faces 2k+1, 2k+2: plane 1 and plane 0 shifted by one site) for
// k = 32w .. 32w+31, so the test runs on whole words; the counts go to the
// bins by popcounts of the runs of cells that share a bin.
__global__ void sixv_observe_kernel(const uint32_t *pl, size_t PS, uint32_t RS, int N, uint32_t nw, uint32_t B,
                                    uint32_t bins_x, unsigned long long *bins)
{
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t w = gid % nw, j = gid / nw + 1u;
    if (j > (uint32_t)N) return;
    const uint32_t *r0 = pl + (size_t)(j - 1) * RS + 4, *r1 = pl + (size_t)j * RS + 4;   // plane 0 rows
    const uint32_t *q0 = r0 + PS, *q1 = r1 + PS;                                          // plane 1 rows
    const uint32_t p0lo = r0[w], p0hi = r1[w], p1lo = q0[w], p1hi = q1[w];
    const uint32_t p0lo_s = (r0[w] >> 1) | (r0[w + 1] << 31), p0hi_s = (r1[w] >> 1) | (r1[w + 1] << 31);
    // i = 2k+1: a00 = p0[j-1][k], a11 = p1[j][k], a10 = p1[j-1][k], a01 = p0[j][k]
    uint32_t c_odd = ~(p0lo ^ p1hi) & ~(p1lo ^ p0hi);
    // i = 2k+2: a00 = p1[j-1][k], a11 = p0[j][k+1], a10 = p0[j-1][k+1], a01 = p1[j][k]
    uint32_t c_even = ~(p1lo ^ p0hi_s) & ~(p0lo_s ^ p1hi);
    c_odd &= range_mask((int)w, 0, (N - 1) / 2);
    c_even &= N >= 2 ? range_mask((int)w, 0, (N - 2) / 2) : 0u;
    // cells x = i - 1: x = 2k (odd i), x = 2k + 1 (even i), k = 32w + b
    const uint32_t by = (j - 1) / B, x_lo = 64u * w, x_hi = x_lo + 64u;
    for (uint32_t x = x_lo; x < x_hi;) {
        const uint32_t nxt = (x / B + 1u) * B < x_hi ? (x / B + 1u) * B : x_hi;
        // bits b with 2(32w + b) in [x, nxt) and 2(32w + b) + 1 in [x, nxt)
        const uint32_t e0 = (x - x_lo + 1u) / 2u, e1 = (nxt - x_lo + 1u) / 2u;   // even cells 2b in [x, nxt)
        const uint32_t o0 = (x - x_lo) / 2u, o1 = (nxt - x_lo) / 2u;             // odd cells 2b+1 in [x, nxt)
        auto bits = [](uint32_t lo, uint32_t hi) -> uint32_t {
            if (lo >= hi) return 0u;
            const uint32_t up = hi >= 32u ? ~0u : ((1u << hi) - 1u);
            return up & ~((1u << lo) - 1u);
        };
        const uint32_t cnt = (uint32_t)__popc(c_odd & bits(e0, e1)) + (uint32_t)__popc(c_even & bits(o0, o1));
        if (cnt) atomicAdd(&bins[(size_t)by * bins_x + x / B], (unsigned long long)cnt);
        x = nxt;
    }
}

// Six-vertex domain given by a mask: heights of the (h+1) x (w+1) points.  Off
// the domain INT32_MIN; boundary points take their fixed height; a site takes
// the value one away from a neighbour already known whose residual bit
// floor(h/2) mod 2 matches its own.  One thread per row J, walking east from
// each row segment's first point (fixed: it has a west side of a cell on the
// boundary), or, when the west side is free, one thread per column I walking
// north from each column segment's lowest point (fixed by its south side).
__global__ void sixv_region_export_kernel(const uint32_t *pl, size_t PS, uint32_t RS, const int32_t *anchor, int w,
                                          int h, int ox, int oy, int by_columns, int32_t *out)
{
    const int line = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (line > (by_columns ? w : h)) return;
    int32_t prev = 0;
    for (int step = 0; step <= (by_columns ? h : w); ++step) {
        const int I = by_columns ? line : step, J = by_columns ? step : line;
        const size_t v = (size_t)J * (w + 1) + I;
        const int32_t a = anchor[v];
        int32_t x = a;
        if (a == INT32_MAX) {
            // the state holds point (I, J) at (I + ox, J + oy) (even offsets)
            const uint32_t X = (uint32_t)(I + ox), Y = (uint32_t)(J + oy);
            const uint32_t bx = hbit(pl, PS, RS, X & 1u, Y, X >> 1);
            x = ((uint32_t)(((prev + 1) >> 1) & 1) == bx) ? prev + 1 : prev - 1;
        }
        out[v] = x;
        prev = x;
    }
}

// Lozenge domain given by a mask: heights of the (h+1) x (w+1) vertices, one
// thread per row Y.  Off the domain INT32_MIN; boundary vertices take their
// fixed height; a site is its west neighbour's height minus one where the
// parity bits differ (steps along (1,0) are 0 or -1).
__global__ void loz_region_export_kernel(const uint32_t *pl, size_t PS, uint32_t RS, const int32_t *anchor, int w,
                                         int h, int32_t *out)
{
    const int Y = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (Y > h) return;
    int32_t prev = 0;
    uint32_t pbit = 0u;
    for (int X = 0; X <= w; ++X) {
        const size_t v = (size_t)Y * (w + 1) + X;
        const int32_t a = anchor[v];
        const uint32_t bx = hbit(pl, PS, RS, (uint32_t)X % 3u, (uint32_t)Y, (uint32_t)X / 3u);
        const int32_t x = a == INT32_MAX ? prev - (int32_t)(bx ^ pbit) : a;
        out[v] = x;
        prev = x;
        pbit = bx;
    }
}

// Lozenge domain: H - H_min of every vertex of the domain into bins of B x B
// vertices, one thread per vertex.
__global__ void loz_region_volume_kernel(const int32_t *H, const int32_t *hmin, int w, int h, uint32_t B,
                                         uint32_t bins_x, unsigned long long *bins)
{
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t n = (uint32_t)(w + 1) * (uint32_t)(h + 1);
    if (gid >= n) return;
    if (hmin[gid] == INT32_MIN) return;
    const int32_t q = H[gid] - hmin[gid];
    const uint32_t X = gid % (uint32_t)(w + 1), Y = gid / (uint32_t)(w + 1);
    if (q) atomicAdd(&bins[(size_t)(Y / B) * bins_x + X / B], (unsigned long long)q);
}

// Type-c cells of a masked six-vertex domain (both diagonal pairs of corner
// heights equal) into bins of B x B cells, one thread per cell.
__global__ void sixv_region_count_kernel(const int32_t *H, const uint8_t *cells, int w, int h, uint32_t B,
                                         uint32_t bins_x, unsigned long long *bins)
{
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (uint32_t)w * (uint32_t)h) return;
    const int x = (int)(gid % (uint32_t)w), y = (int)(gid / (uint32_t)w);
    if (!cells[gid]) return;
    const size_t sw = (size_t)y * (w + 1) + x, nw = sw + (size_t)(w + 1);
    if (H[sw] == H[nw + 1] && H[sw + 1] == H[nw])
        atomicAdd(&bins[(size_t)((uint32_t)y / B) * bins_x + (uint32_t)x / B], 1ull);
}

// Lozenge observable: H - H_min per vertex, summed into bins of B x B cells.
// One wavefront per row Y, a lane per chunk X in [96m, 96m + 96): word m of
// the three planes holds the residual bits of those vertices (bit k of plane
// p is X = 96m + 3k + p).  H falls by one at every X > xs whose bit differs
// from the bit of X - 1, so XORs of the planes (plane 0 against plane 2
// shifted by one site) give the chunk's drops; a wavefront prefix sum of
// their counts gives every chunk its starting height.  Within a bin the sum
// of H over X in [u, v] is n H(u - 1) minus, for every drop d, the v - d + 1
// vertices from d on, and the sum of H_min = max(c - X, max(0, c - Y)) is an
// arithmetic series: popcounts and closed forms, no loop over vertices.
__global__ void __launch_bounds__(64) loz_observe_kernel(const uint32_t *pl, size_t PS, uint32_t RS, Geo geo,
                                                         uint32_t B, uint32_t bins_x, unsigned long long *bins)
{
    extern __shared__ unsigned long long rowbin[];
    const int Y = (int)blockIdx.x, lane = (int)threadIdx.x;
    for (uint32_t i = (uint32_t)lane; i < bins_x; i += 64u) rowbin[i] = 0ull;
    __syncthreads();
    const int xs = loz_xs(geo, Y), xe = loz_xe(geo, Y);
    const int h0 = imax(0, geo.c - Y), tc = geo.c - h0;   // H_min(X) = c - X for X < tc, else h0
    const uint32_t *row = pl + (size_t)Y * RS + 4;
    int carry = 0;   // drops in the chunks of earlier passes
    for (int m0 = xs / 96; m0 <= xe / 96; m0 += 64) {
        const int m = m0 + lane, X0 = 96 * m;
        const int lo = imax(xs, X0), hi = imin(xe, X0 + 95), L = imax(lo, xs + 1);
        uint32_t D[3] = {0u, 0u, 0u};
        int cnt = 0;
        if (lo <= hi) {
            const uint32_t W0 = row[m], W1 = row[PS + m], W2 = row[2 * PS + m];
            // the bit of X0 - 1 (plane 2, last bit of word m - 1), needed when X0 > xs
            const uint32_t cin = X0 > xs ? row[2 * PS + m - 1] >> 31 : 0u;
            D[0] = W0 ^ ((W2 << 1) | cin);
            D[1] = W1 ^ W0;
            D[2] = W2 ^ W1;
#pragma unroll
            for (int p = 0; p < 3; ++p) cnt += __popc(D[p] & word_mask(X0, p, L, hi, 3));
        }
        int incl = cnt;   // inclusive scan over the lanes
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off, 64);
            if (lane >= off) incl += v;
        }
        const int total = __shfl(incl, 63, 64);
        if (lo <= hi) {
            int H = loz_hmin(geo, xs, Y) - carry - (incl - cnt);   // H before this chunk's drops
            for (int u = lo; u <= hi;) {
                const int j = u / (int)B, v = imin(hi, (j + 1) * (int)B - 1);
                const int du = imax(u, L);
                int c = 0;
                long long sd = 0;   // drops in [du, v] and the sum of their X
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const uint32_t x = D[p] & word_mask(X0, p, du, v, 3);
                    const int cp = __popc(x);
                    c += cp;
                    sd += (long long)cp * (X0 + p) + 3ll * (long long)bit_index_sum(x);
                }
                const long long n = v - u + 1;
                const long long sumH = n * H - ((long long)c * (v + 1) - sd);
                long long sumMin = 0;
                const int aE = imin(v, tc - 1), bS = imax(u, tc);
                if (aE >= u) {
                    const long long na = aE - u + 1;
                    sumMin += na * geo.c - (long long)(u + aE) * na / 2;
                }
                if (bS <= v) sumMin += (long long)(v - bS + 1) * h0;
                if (sumH != sumMin) atomicAdd(&rowbin[j], (unsigned long long)(sumH - sumMin));
                H -= c;
                u = v + 1;
            }
        }
        carry += total;
    }
    __syncthreads();
    const size_t row_bins = (size_t)(Y / (int)B) * bins_x;
    for (uint32_t i = (uint32_t)lane; i < bins_x; i += 64u)
        if (rowbin[i]) atomicAdd(&bins[row_bins + i], rowbin[i]);
}

Geo geo_of(const HeightDev &d)
{
    return Geo{d.model, d.a, d.b, d.c, d.N, d.site, d.PS, d.RS, d.freep, d.free_side};
}

}  // namespace

hipError_t height_init(const HeightDev &d, int init_max, hipStream_t s)
{
    dim3 block(64), grid((d.RS + 63) / 64, d.rows, d.P);
    hipLaunchKernelGGL(height_init_kernel, grid, block, 0, s, d.planes, d.spare, d.PS, d.RS, d.rows, d.P, geo_of(d),
                       init_max);
    return hipGetLastError();
}

hipError_t height_colour_step(const HeightDev &d, int colour, uint32_t t, const Thr &T, int metropolis, uint64_t seed,
                              hipStream_t s, Timing *tm)
{
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const uint32_t threads = d.ng * d.rows;
    dim3 block(256), grid((threads + 255) / 256);
    const int mode = T.uniform() ? kUniform : (metropolis ? kMetropolis : kHeatBath);
    auto k = d.site ? TL_HEIGHT_PICK_R(height_step_kernel, mode, (int)table_kind(T), true)
                    : TL_HEIGHT_PICK_R(height_step_kernel, mode, (int)table_kind(T), false);
    return launch(tm, 1, k, grid, block, 0, s, d.planes, d.PS, d.RS, d.ng, d.rows, geo_of(d), (uint32_t)colour, t, T,
                  k0, k1);
}

HeightTile height_auto_tile(const HeightDev &d, bool uniform, bool random_order)
{
    HeightTile t;
    // Up to 16 granules, a wavefront each: the whole domain in one tile, no halo
    // and no launch after the first (six-vertex N = 200, one-bit: 1.06 us per
    // sweep where tiles of 16 rows take 1.26).  The bit-serial six-vertex steps are
    // long enough that wavefronts sharing a SIMD hold each other up: up to 5
    // granules there (us per sweep, whole / 16 rows x 12 sweeps: N = 128, 5
    // granules, 4.10 / 4.19 heat bath and 4.19 / 4.25 Metropolis; N = 160, 6, 4.77 /
    // 4.28 and 4.76 / 4.33; N = 255, 8, 5.95 / 4.42 and 5.84 / 4.43).
    const HeightLds whole = height_lds(d.model != TL_LOZENGE, d.rows, d.ng);
    if (whole.granules <= (uniform || d.model == TL_LOZENGE ? 16u : 5u) && whole.words) {
        t.TR = d.rows;
        t.TG = d.ng;
        t.S = 1u << 28;
        return t;
    }
    // Rows up to 8 groups wide are one tile wide (no column halo).  The rows of
    // a tile with its halo are a whole number of granules (lozenge 16 rows,
    // six-vertex 32): fewer sweeps per launch pay its fixed time (5 us: reading
    // the tile, the first look, writing it back) more often, more sweeps grow
    // the halo.  Measured on MI355X, us per sweep: hexagon 1024, q = 1999/2000,
    // 8 rows x 4 sweeps 3.6, 14 x 3 4.0, 18 x 5 (2 groups) 4.1; six-vertex N =
    // 1024 weighted 16 x 12 4.56, 8 x 6 4.66, 32 x 8 4.85; one-bit 16 x 12 1.49,
    // 8 x 6 1.68, 32 x 16 1.63; random order 16 x 6 2.94, 8 x 3 3.52, 32 x 8 3.04.
    t.TG = d.ng <= 8 ? d.ng : 4;
    if (d.model == TL_LOZENGE) {
        // (one-bit, 64 rows with the halo: wider tiles would have 16 granules or
        // more than wavefronts, taken in turns with every draw on the spot.  us per
        // sweep, 2 groups / all of them up to 8 or 4 with a halo: (1500, 500, 500), 5
        // groups, 2.53 / 3.60; 1024, 6 groups, 2.56 / 4.21; (2000, 1000, 1000), 8 groups,
        // 2.84 / 4.63; (100, 100, 1500), 4 groups, 2.99 / 3.77; 3 groups 2.39 / 2.42)
        if (uniform && d.ng > 3) t.TG = 2;
        t.TR = uniform ? 16 : 8;
        t.S = uniform ? 8 : 4;
    } else {
        t.TR = 16;
        t.S = random_order ? 6 : 12;
    }
    return t;
}

bool height_plan(const HeightDev &d, const HeightTile &tile, uint32_t S_max, TilePlan *p)
{
    if (d.rows == 0 || S_max == 0) return false;
    // halo rows invalidated per sweep, halo sites (per plane) per sweep; under
    // the random colour order each of the K steps may cost one of each
    const uint32_t K = d.model == TL_LOZENGE ? 3u : 4u;
    const uint32_t rows_per_sweep = tile.order ? K : (d.model == TL_LOZENGE ? 3u : 2u);
    const uint32_t cols_per_sweep = tile.order ? K : (d.model == TL_LOZENGE ? 1u : 2u);
    const uint32_t TG = tile.TG == 0 ? 1u : (tile.TG < d.ng ? tile.TG : d.ng);
    const uint32_t tiles_x = (d.ng + TG - 1) / TG;
    const uint32_t LG0 = TG + (tiles_x > 1 ? 2u : 0u);
    // six-vertex tasks are row pairs (one row of each pair is idle in every
    // colour step), lozenge tasks rows
    uint32_t max_rows = (d.model == TL_LOZENGE ? 1u : 2u) * (kTileTasks / LG0);
    // and as many rows as LDS holds: six-vertex rows of one group have 848 of
    // their 1024.  The shape and the sweeps per launch are upper bounds, clamped
    // to these rows below.
    while (max_rows && !height_lds(d.model != TL_LOZENGE, max_rows, LG0).words) --max_rows;
    if (max_rows < 2u * rows_per_sweep + 3u) return false;
    uint32_t TR = tile.TR == 0 ? 1u : (tile.TR < d.rows ? tile.TR : d.rows);
    if (TR < d.rows && TR > max_rows - 2u * rows_per_sweep) TR = max_rows - 2u * rows_per_sweep;
    if (TR >= d.rows && d.rows > max_rows) TR = max_rows - 2u * rows_per_sweep;
    const uint32_t tiles_y = (d.rows + TR - 1) / TR;
    uint32_t S = S_max < tile.S ? S_max : tile.S;
    if (tiles_x > 1 && S > 128u / cols_per_sweep) S = 128u / cols_per_sweep;
    if (tiles_y > 1 && S > (max_rows - TR) / (2u * rows_per_sweep)) S = (max_rows - TR) / (2u * rows_per_sweep);
    if (S == 0u) S = 1u;
    if (S > 1u << 28) S = 1u << 28;   // the kernel counts colour steps in 32 bits
    const uint32_t HR = tiles_y > 1 ? rows_per_sweep * S : 0u;
    const uint32_t HG = tiles_x > 1 ? 1u : 0u;
    const uint32_t LR = TR + 2 * HR, LG = TG + 2 * HG;
    const HeightLds lay = height_lds(d.model != TL_LOZENGE, LR, LG);
    if (lay.task_rows * LG > kTileTasks || lay.words == 0u) return false;
    p->S = S;
    p->TR = TR;
    p->TG = TG;
    p->HR = HR;
    p->HG = HG;
    p->tiles_x = tiles_x;
    p->tiles_y = tiles_y;
    // a wavefront per granule, up to 16
    p->threads = lay.granules < kTileThreads / 64u ? lay.granules * 64u : kTileThreads;
    p->lds = lay.words * 4u;
    p->order = tile.order;
    return true;
}

hipError_t height_tiled_sweeps(HeightDev &d, const HeightTile &tile, uint32_t t0, uint32_t nsw, const Thr &T,
                               int metropolis, uint64_t seed, hipStream_t s, Timing *tm)
{
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const uint32_t colours = d.model == TL_LOZENGE ? 3u : 4u;
    uint32_t done = 0;
    while (done < nsw) {
        TilePlan p;
        if (!height_plan(d, tile, nsw - done, &p)) return hipErrorInvalidConfiguration;
        const int mode = T.uniform() ? kUniform : (metropolis ? kMetropolis : kHeatBath);
#define TL_LOZ_PICK(R, M)                                                                              \
    (mode == kUniform ? loz_tiled_kernel<kUniform, kKindClass, R, M>                                   \
     : mode == kMetropolis ? loz_tiled_kernel<kMetropolis, kKindClass, R, M>                           \
                           : loz_tiled_kernel<kHeatBath, kKindClass, R, M>)
        const bool masked = d.site != nullptr;
        auto k = d.model == TL_LOZENGE
                     ? (p.order ? (masked ? TL_LOZ_PICK(true, true) : TL_LOZ_PICK(true, false))
                                : (masked ? TL_LOZ_PICK(false, true) : TL_LOZ_PICK(false, false)))
                     : TL_HEIGHT_PICK_ORDER_MASK(height_tiled_kernel, mode, (int)table_kind(T), p.order, masked);
#undef TL_LOZ_PICK
        hipError_t e = launch(tm, colours * p.S, k, dim3(p.tiles()), dim3(p.threads), p.lds, s,
                              (const uint32_t *)d.planes, d.spare, d.PS, d.RS, d.ng, d.rows, geo_of(d),
                              t0 + done, p.S, p.TR, p.TG, p.HR, p.HG, p.tiles_x, T, k0, k1);
        if (e != hipSuccess) return e;
        uint32_t *tmp = d.planes;
        d.planes = d.spare;
        d.spare = tmp;
        done += p.S;
    }
    return hipSuccess;
}

TileJob height_tile_job(const HeightDev &d, const TilePlan &p, uint32_t t0, const Thr &T, int metropolis,
                        uint64_t seed)
{
    TileJob j{};
    j.in = d.planes;
    j.out = d.spare;
    j.PS = d.PS;
    j.RS = d.RS;
    j.ng = d.ng;
    j.rows = d.rows;
    j.P = d.P;
    j.K = d.K;
    j.model = d.model;
    j.a = d.a;
    j.b = d.b;
    j.c = d.c;
    j.N = d.N;
    j.t0 = t0;
    j.S = p.S;
    j.TR = p.TR;
    j.TG = p.TG;
    j.HR = p.HR;
    j.HG = p.HG;
    j.tiles_x = p.tiles_x;
    j.order = p.order;
    j.mode = T.uniform() ? kModeUniform : (metropolis ? kModeMetropolis : kModeHeatBath);
    j.kind = T.uniform() ? (uint32_t)kTableClass : table_kind(T);
    j.site = d.site;
    j.freep = d.freep;
    j.free_side = d.free_side;
    j.key0 = (uint32_t)seed;
    j.key1 = (uint32_t)(seed >> 32);
    j.T = T;
    return j;
}

hipError_t height_items(const TileJob *jobs, const TileItem *items, uint32_t n_items, uint32_t threads, uint32_t lds,
                        uint32_t mode, uint32_t kind, uint32_t order, uint32_t masked, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    if (threads == 0 || threads > kTileThreads || (threads & 63u) || lds > 4u * kLdsWords || mode > 2u || kind > 1u)
        return hipErrorInvalidConfiguration;
    auto k = TL_HEIGHT_PICK_ORDER_MASK(height_items_kernel, (int)mode, (int)kind, order, masked);
    hipLaunchKernelGGL(k, dim3(n_items), dim3(threads), lds, s, jobs, items);
    return hipGetLastError();
}

hipError_t height_items_mixed(const TileJob *jobs, const TileItem *items, uint32_t n_items, uint32_t threads,
                              uint32_t lds, uint32_t order, uint32_t masked, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    if (threads == 0 || threads > kTileThreads || (threads & 63u) || lds > 4u * kLdsWords)
        return hipErrorInvalidConfiguration;
    auto k = order ? (masked ? height_items_mixed_kernel<true, true> : height_items_mixed_kernel<true, false>)
                   : (masked ? height_items_mixed_kernel<false, true> : height_items_mixed_kernel<false, false>);
    hipLaunchKernelGGL(k, dim3(n_items), dim3(threads), lds, s, jobs, items);
    return hipGetLastError();
}

hipError_t height_export(const HeightDev &d, int32_t *dev, hipStream_t s)
{
    // chunks of a row: 96 lozenge vertices or 64 six-vertex faces each
    const uint32_t nch = d.model == TL_LOZENGE ? (uint32_t)(d.a + d.c) / 96u + 1u : (uint32_t)d.N / 64u + 1u;
    const uint32_t shmem = 4u * nch * (d.model == TL_LOZENGE ? 4u : 3u);
    if (shmem > 64u * 1024u) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(height_export_kernel, dim3(d.rows), dim3(64), shmem, s, d.planes, d.PS, d.RS, geo_of(d), nch,
                       dev);
    return hipGetLastError();
}

hipError_t sixv_region_export(const HeightDev &d, const int32_t *anchor, int w, int h, int32_t *out, hipStream_t s)
{
    const int by_columns = d.free_side == 4 ? 1 : 0;
    const int lines = (by_columns ? w : h) + 1;
    hipLaunchKernelGGL(sixv_region_export_kernel, dim3((lines + 63) / 64), dim3(64), 0, s, d.planes, d.PS, d.RS,
                       anchor, w, h, d.ox, d.oy, by_columns, out);
    return hipGetLastError();
}

hipError_t loz_region_export(const HeightDev &d, const int32_t *anchor, int w, int h, int32_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(loz_region_export_kernel, dim3((h + 64) / 64), dim3(64), 0, s, d.planes, d.PS, d.RS, anchor, w,
                       h, out);
    return hipGetLastError();
}

hipError_t loz_region_observe(const HeightDev &d, const int32_t *anchor, const int32_t *hmin, int w, int h,
                              int32_t *heights, uint32_t B, uint32_t bins_x, unsigned long long *bins, hipStream_t s)
{
    hipError_t e = loz_region_export(d, anchor, w, h, heights, s);
    if (e != hipSuccess) return e;
    const uint32_t n = (uint32_t)(w + 1) * (uint32_t)(h + 1);
    hipLaunchKernelGGL(loz_region_volume_kernel, dim3((n + 255) / 256), dim3(256), 0, s, heights, hmin, w, h, B,
                       bins_x, bins);
    return hipGetLastError();
}

hipError_t sixv_region_observe(const HeightDev &d, const int32_t *anchor, const uint8_t *cells, int w, int h,
                               int32_t *heights, uint32_t B, uint32_t bins_x, unsigned long long *bins,
                               hipStream_t s)
{
    hipError_t e = sixv_region_export(d, anchor, w, h, heights, s);
    if (e != hipSuccess) return e;
    const uint32_t n = (uint32_t)w * (uint32_t)h;
    hipLaunchKernelGGL(sixv_region_count_kernel, dim3((n + 255) / 256), dim3(256), 0, s, heights, cells, w, h, B,
                       bins_x, bins);
    return hipGetLastError();
}

hipError_t height_observe(const HeightDev &d, uint32_t B, uint32_t bins_x, unsigned long long *bins, hipStream_t s)
{
    if (d.model == TL_LOZENGE) {
        if ((size_t)bins_x * 8u > 64u * 1024u) return hipErrorInvalidConfiguration;
        hipLaunchKernelGGL(loz_observe_kernel, dim3(d.rows), dim3(64), bins_x * 8u, s, d.planes, d.PS, d.RS,
                           geo_of(d), B, bins_x, bins);
    } else {
        const uint32_t nw = 4u * d.ng, threads = nw * (uint32_t)d.N;
        hipLaunchKernelGGL(sixv_observe_kernel, dim3((threads + 255) / 256), dim3(256), 0, s, d.planes, d.PS, d.RS,
                           d.N, nw, B, bins_x, bins);
    }
    return hipGetLastError();
}

}  // namespace tl
