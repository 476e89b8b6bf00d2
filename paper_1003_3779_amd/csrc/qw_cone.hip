// qw_cone.hip -- torus walks from one site, stored on the sites they can reach.
//
// The walk of Sec. 2.1 (U = S (I (x) C), Eqs. (2), (3), (8)) started at one site
// x0 is, after t steps, non-zero on few of the sites of its light-cone box
// (Eqs. (13)-(18)): with the diagonal table every step moves by one in x and in
// y, so dx + t and dy + t are even; with the axis-aligned tables (pair order,
// Eq. (8)) the same holds for u = dx + dy and v = dx - dy.  Either way the live
// sites are a dense square of (t + 1) x (t + 1) points
//     diagonal table:      I = (dy + t) / 2,  J = (dx + t) / 2
//     axis-aligned tables: I = (u + t) / 2,   J = (v + t) / 2       (0 <= I, J <= t)
// a quarter of the box, and component c moves from (I, J) at time t to
// (I + di_c, J + dj_c) at time t + 1 with di, dj in {0, 1}, each pair once:
//     psi_{t+1}(I + di_c, J + dj_c, c) = sum_c' C[c][c'] psi_t(I, J, c').
// The state is held as that square (eight planes of real numbers, Re and Im of
// each component, row stride ld), at most min(Lx, Ly) / 2 + 1 a side: while
// 2 t <= Lx and 2 t <= Ly no two of its points are the same site (t = L / 2 apart,
// where the outermost points meet in pairs that no component shares).  Every live
// amplitude is the same expression as in the kernels of the whole lattice
// (bitwise equal, but for complex128 numbers that pass below 2^-1022: ConeArgs::marks
// are kept for complex64 alone, 2 % of a 4096^2 walk); the others are exact zeros there
// and absent here.
#include "qw_internal.h"

#include <hip/hip_ext.h>
#include "qw_device.h"

#include <algorithm>
#include <type_traits>

namespace qw {
namespace {

constexpr int kConeMinSide = 32;  // smaller tori stay on the whole lattice: their cone closes within a launch or two
constexpr int kConeWaves = 1;     // waves per SIMD a one-stage launch aims at (2: 7.3 / 30.9 ms, the halo rows of shorter segments)
// launches of more than kK steps: levels a stage, stages, rows a group.  Four stages of
// 8 levels, 4096^2 Grover complex128 / 16384^2 H (x) H complex64: 5.71 / 27.9 ms a
// walk; two of 16 5.74 / 29.3, four with twice the columns a lane and one row a group 6.8 /
// 35.4, one-stage launches of 16 throughout 6.98 / 29.9.  Segments are cut for two waves per SIMD
// (for one: 6.6 / 33.5; for three, of which 182 to 196 registers leave two resident: 6.0 / 29.2).
// Counted: complex128 issues on 58 % of the cycles and its waves wait 36 % of theirs (a barrier
// every two rows, two waves to hide it), complex64 80 % and 26 %.
constexpr int kDeepKL = 8, kDeepNS = 4, kDeepNR = 2;
template <typename R> constexpr int kDeepM = sizeof(R) == 8 ? 2 : 4;  // and columns a lane
constexpr int kDeepSide = 700;  // squares from this side on take them (400 and 1200: the same within 1 %)
constexpr int kConeMinRows = 8;   // shortest segment
constexpr int kConeTilesPerCu = 1;  // a square of at most so many tiles per compute unit takes the tile kernel
template <bool CPLX> constexpr int kTileDepth = CPLX ? 8 : 16;  // steps of a launch there
constexpr int kK = 16;  // most levels of a one-stage launch

__host__ __device__ constexpr int cone_di(int table, int c) {
    return table == TABLE_DIAG ? ((c & 1) == 0) : (table == TABLE_PAIR ? (c == 0 || c == 2) : c < 2);
}
__host__ __device__ constexpr int cone_dj(int table, int c) {
    return table == TABLE_DIAG ? c < 2 : (table == TABLE_PAIR ? (c == 0 || c == 3) : (c == 1 || c == 3));
}

// the rows of component c that a state of time t holds: what the last step moved
// there (t = 0: the start site)
__device__ __forceinline__ int row_lo(int t, int di) { return t == 0 ? 0 : di; }
__device__ __forceinline__ int row_hi(int t, int di) { return t == 0 ? 0 : t - 1 + di; }

struct ConeArgs {
    int64_t ps;  // plane stride, elements
    int ld;      // row stride
    int t;       // time of the input
    int kk;      // steps of this launch
    int rows;    // rows of the launch's output that its segments share out
    int cols;    // columns of the output
    int nstrips, nseg, seg_rows;
    double unscale;  // 2^-(levels since the last mark) (coins that keep their factor 1/2 out)
    double *partial; // non-null: each tile's (tile kernel: block's) sum of the squares it stores, in fp64
    uint32_t marks;  // bit s: multiply the factors back after level s too
};

// 32-bit words one lane over; the lane with no source takes zero (halo)
template <bool RIGHT> __device__ __forceinline__ int dpp_shift(int v) {
    return __builtin_amdgcn_update_dpp(0, v, RIGHT ? 0x130 : 0x138, 0xf, 0xf, true);
}
template <bool RIGHT> __device__ __forceinline__ float lane_shift(float v) {
    return __builtin_bit_cast(float, dpp_shift<RIGHT>(__builtin_bit_cast(int, v)));
}
template <bool RIGHT> __device__ __forceinline__ double lane_shift(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)dpp_shift<RIGHT>((int)(unsigned)u), hi = (unsigned)dpp_shift<RIGHT>((int)(unsigned)(u >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// a copy the compiler does not merge with its source (DPP: the value may be read by
// a cross-lane move next, which the hardware wants two wait states later)
template <bool DPP> __device__ __forceinline__ float copy_out(float v) {
    float o;
    if constexpr (DPP) asm volatile("v_mov_b32 %0, %1\n\ts_nop 1" : "=v"(o) : "v"(v));
    else asm volatile("v_mov_b32 %0, %1" : "=v"(o) : "v"(v));
    return o;
}
template <bool DPP> __device__ __forceinline__ double copy_out(double v) {
    double o;
    if constexpr (DPP) asm volatile("v_mov_b64 %0, %1\n\ts_nop 1" : "=v"(o) : "v"(v));
    else asm volatile("v_mov_b64 %0, %1" : "=v"(o) : "v"(v));
    return o;
}

// coins of one real part of a site (REAL lanes): the same expressions as
// Coin<...> on that part.  COIN_DENSE here is a real matrix: the complex form
// adds exact zeros to these sums.
template <typename R, int COIN> __device__ __forceinline__ void real_coin(const R (&g)[4], R (&o)[4], const CoinR<R> &C) {
    if constexpr (COIN == COIN_GROVER4) {
        const R s = (g[0] + g[1]) + (g[2] + g[3]);
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = fmaR((R)-2, g[c], s);
    } else if constexpr (COIN == COIN_HH4) {
        const R u0 = g[0] + g[1], u1 = g[0] - g[1], u2 = g[2] + g[3], u3 = g[2] - g[3];
        o[0] = u0 + u2;
        o[1] = u1 + u3;
        o[2] = u0 - u2;
        o[3] = u1 - u3;
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            R a = C.re[c * 4] * g[0];
#pragma unroll
            for (int k = 1; k < 4; ++k) a = fmaR(C.re[c * 4 + k], g[k], a);
            o[c] = a;
        }
    }
}

// The 4-point Fourier coin, F[a][b] = i^(ab) / 2, twice the result: two butterfly
// levels (complex128: its entries cos and sin of k pi / 2 are off by rounding in
// the dense matrix, so the two differ by less than that matrix's own error;
// complex64 keeps the dense sums, whose roundings its results show).
constexpr int kCoinFourier4 = 3;
template <typename R> __device__ __forceinline__ void fourier_x2(const cv<R> (&g)[4], cv<R> (&o)[4]) {
    const cv<R> s02 = cadd<R>(g[0], g[2]), d02 = csub<R>(g[0], g[2]), s13 = cadd<R>(g[1], g[3]), d13 = csub<R>(g[1], g[3]);
    o[0] = cadd<R>(s02, s13);
    o[2] = csub<R>(s02, s13);
    o[1].x = d02.x - d13.y;
    o[1].y = d02.y + d13.x;
    o[3].x = d02.x + d13.y;
    o[3].y = d02.y - d13.x;
}

// the coin of one site, complex lanes (g[c][0], g[c][1]: Re, Im) or one real part
// (g[c][0]), in place; scaled: without the factor 1/2 of Grover, H (x) H, Fourier
template <typename R, int COIN, int NP> __device__ __forceinline__ void site_coin(R (&x)[4][NP], const CoinR<R> &C) {
    if constexpr (NP == 2) {
        cv<R> g[4], o[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) { g[c].x = x[c][0]; g[c].y = x[c][1]; }
        if constexpr (COIN == kCoinFourier4) fourier_x2<R>(g, o);
        else Coin<R, 4, COIN_DENSE>::apply(g, o, C);
#pragma unroll
        for (int c = 0; c < 4; ++c) { x[c][0] = o[c].x; x[c][1] = o[c].y; }
    } else {
        R g[4], o[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) g[c] = x[c][0];
        real_coin<R, COIN>(g, o, C);
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c][0] = o[c];
    }
}

// The factor by which level s multiplies its outputs back: 2^-(levels since the
// last mark) at a mark, else 1.
__device__ __forceinline__ bool mark_at(uint32_t marks, int s) { return (marks >> s) & 1u; }
// the marks that are not at the end of a stage of KL levels
template <int KL> __device__ __forceinline__ uint32_t inner_marks(uint32_t marks) {
    constexpr uint32_t ends = KL == 16 ? 0x80008000u : 0x80808080u;
    return marks & ~ends;
}
template <typename R> __device__ __forceinline__ R mark_scale(uint32_t marks, int s) {
    const uint32_t below = marks & ((1u << s) - 1u);
    const int n = below ? s - (31 - __builtin_clz(below)) : s + 1;
    return (R)1 / (R)(1u << n);
}

__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <typename R, int M> struct alignas(sizeof(R) * M) VecR {
    R v[M];
};

// kk steps of the square.  A wave holds 64 * M columns (M per lane) and streams along
// I; level s of row I needs rows I and I - 1 of the level before only, so every
// level works on the rows that have just arrived (NR of them) and keeps, per lane, the
// previous row of the two components that move along I -- no lag between levels
// and half the window of a kernel whose moves go both ways.  The two that move
// along J take one lane exchange per M columns.  INV: the inverse step, psi_{t-1} =
// C^dagger S^-1 psi_t, the same moves mirrored (rows descending, values from the
// right).  CPLX: complex lanes (any coin); else one real part per wave (real coins:
// Re and Im evolve alone), half the registers.
//
// NS waves share a tile: each runs KL levels and hands its rows to the next through
// LDS a group later (two buffers, one barrier per group), so a launch of NS KL
// levels holds the window of KL per wave and the state crosses HBM once.  A strip
// gives 64 M - NS KL columns; a segment of S rows reads S + kk - 1, of which level s
// works from row s on (in stream order: the rows before feed nothing).
template <typename R, int KL, int NS, int M, int NR, int TABLE, int COIN, bool CPLX, bool INV>
__global__ __launch_bounds__(256, 2) void k_cone(const R *__restrict__ in, R *__restrict__ out, ConeArgs A, CoinR<R> C) {
    constexpr int NP = CPLX ? 2 : 1;  // real parts per lane
    constexpr int K = KL * NS, TW = 64 * M - K;
    constexpr bool kScaled = !INV && COIN != COIN_DENSE;
    static_assert(K % M == 0, "strips start at multiples of M");
    static_assert(NS == 1 || NS == 2 || NS == 4, "a block's four waves are whole tiles");
    using V = VecR<R, M>;
    __shared__ V hand[NS > 1 ? 4 / NS * (NS - 1) * 2 * NR * 4 * NP * 64 : 1];  // [tile][stage][buffer][row][plane][lane]
    const int lane = threadIdx.x & 63;
    // the hardware deals blocks to the 8 XCDs in turn: each XCD takes a contiguous
    // range of (segment, strip) pairs, whose halos then meet in its L2
    int lb = blockIdx.x;
    {
        const int nb = gridDim.x, xcd = lb & 7, i = lb >> 3, per = nb >> 3, rem = nb & 7;
        lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + i;
    }
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int stage = w % NS, tile = __builtin_amdgcn_readfirstlane(lb * (4 / NS) + w / NS);
    const int strip = tile % A.nstrips, rest = tile / A.nstrips;
    const int seg = rest % A.nseg, part = rest / A.nseg;
    const int r0 = seg * A.seg_rows;
    const bool active = part < (CPLX ? 1 : 2) && r0 < A.rows;
    if (NS == 1 && !active) return;               // wave-uniform; one stage has no barriers
    const int r1 = min(A.rows, r0 + A.seg_rows);  // own rows [r0, r1)
    const int t = A.t, kk = A.kk;
    const int c0 = strip * TW;
    const int col = c0 + lane * M - (INV ? 0 : K);  // this lane's first column
    const bool lane_in = col >= 0 && col <= t;
    const int lcol = lane_in ? col : 0;
    bool ok[M];
#pragma unroll
    for (int m = 0; m < M; ++m) ok[m] = lane_in && col + m <= t;
    const bool own = INV ? (lane * M < TW && col < A.cols) : (lane * M >= K && col < A.cols);
    const R *src = in + part * A.ps;
    R *dst = out + part * A.ps;
    R prev[KL][2][NP][M];
#pragma unroll
    for (int s = 0; s < KL; ++s)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int m = 0; m < M; ++m) prev[s][k][p][m] = (R)0;
    // NR rows arrive together (in stream order): within the group a row takes the
    // one before it straight from its registers
    V nx[NR][4][NP];
    auto request = [&](int r) {  // NR rows of the input, clamped into the square (masked when used)
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int rc = min(max(INV ? r - q : r + q, 0), t);
            const int64_t o = (int64_t)rc * A.ld + lcol;
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int p = 0; p < NP; ++p) nx[q][c][p] = *(const V *)(src + (2 * c + p) * A.ps + o);
        }
    };
    // rows the stream takes: ascending from r0 - kk + 1 (forward), descending from r1 - 1 + kk (inverse)
    int r = INV ? r1 - 1 + kk : r0 - kk + 1;
    // (several stages: the same count in every wave of the block, and one group more per stage)
    const int iters = ((NS > 1 ? A.seg_rows : r1 - r0) + (INV ? kk : kk - 1) + NR - 1) / NR;
    if (NS == 1 || (active && stage == 0)) request(r);
    r += (INV ? NR : -NR) * stage;
    V *const mine = &hand[NS > 1 ? ((w / NS) * (NS - 1) + stage) * 2 * NR * 4 * NP * 64 : 0];  // what this stage hands on
    const V *const from = stage > 0 ? mine - 2 * NR * 4 * NP * 64 : mine;                       // what the one before did
    // every level with no test (a branch a level costs a fifth to a quarter of the time:
    // 16384^2 H (x) H walk 37.1 against 29.5 ms) -- but in launches of fewer levels, with
    // marks inside a stage, and for the rows the early levels alone work on
    double nacc = 0.0;
    const bool whole = kk == K && (!kScaled || sizeof(R) == 8 || inner_marks<KL>(A.marks) == 0);
    auto group = [&](int g, auto some) {  // g: this stage's group
        constexpr bool SOME = decltype(some)::value;
        const int rn = INV ? r - NR : r + NR;
        {
            R x[NR][4][NP][M];
            if (NS == 1 || stage == 0) {
#pragma unroll
                for (int q = 0; q < NR; ++q)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int di = cone_di(TABLE, c), rq = INV ? r - q : r + q;
                        const bool rok = rq >= row_lo(t, di) && rq <= row_hi(t, di);
#pragma unroll
                        for (int p = 0; p < NP; ++p)
#pragma unroll
                            for (int m = 0; m < M; ++m) x[q][c][p][m] = rok && ok[m] ? nx[q][c][p].v[m] : (R)0;
                    }
                request(rn);
            } else {
#pragma unroll
                for (int q = 0; q < NR; ++q)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
#pragma unroll
                        for (int p = 0; p < NP; ++p) {
                            const V v = from[(((g & 1) * NR + q) * 4 * NP + c * NP + p) * 64 + lane];
#pragma unroll
                            for (int m = 0; m < M; ++m) x[q][c][p][m] = v.v[m];
                        }
            }
            // levels of this stage that the group's last row works on
            const int lim = min(kk, (g + 1) * NR) - stage * KL;
#pragma unroll
            for (int s = 0; s < KL; ++s) {
                if (!SOME || s < lim) {
                    // forward: coin, then the moves (the launch's last move along I is the
                    // row it is stored to); inverse: the moves back, then the coin
                    auto coin = [&]() {
#pragma unroll
                        for (int q = 0; q < NR; ++q)
#pragma unroll
                            for (int m = 0; m < M; ++m) {
                                R v[4][NP];
#pragma unroll
                                for (int c = 0; c < 4; ++c)
#pragma unroll
                                    for (int p = 0; p < NP; ++p) v[c][p] = x[q][c][p][m];
                                site_coin<R, COIN, NP>(v, C);
#pragma unroll
                                for (int c = 0; c < 4; ++c)
#pragma unroll
                                    for (int p = 0; p < NP; ++p) x[q][c][p][m] = v[c][p];
                            }
                    };
                    auto move_j = [&]() {
#pragma unroll
                        for (int q = 0; q < NR; ++q)
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                if (cone_dj(TABLE, c)) {
#pragma unroll
                                    for (int p = 0; p < NP; ++p) {
                                        R(&v)[M] = x[q][c][p];
                                        if constexpr (INV) {
                                            const R e = lane_shift<true>(v[0]);
#pragma unroll
                                            for (int m = 0; m + 1 < M; ++m) v[m] = v[m + 1];
                                            v[M - 1] = e;
                                        } else {
                                            const R e = lane_shift<false>(v[M - 1]);
#pragma unroll
                                            for (int m = M - 1; m > 0; --m) v[m] = v[m - 1];
                                            v[0] = e;
                                        }
                                    }
                                }
                    };
                    // the old rows, copied out before the level's outputs are made: the
                    // outputs can then be written where they were
                    R old[2][NP][M];
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int p = 0; p < NP; ++p)
#pragma unroll
                            for (int m = 0; m < M; ++m) old[k][p][m] = copy_out<INV>(prev[s][k][p][m]);
                    auto move_i = [&]() {
                        int k = 0;
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (cone_di(TABLE, c)) {
#pragma unroll
                                for (int p = 0; p < NP; ++p)
#pragma unroll
                                    for (int m = 0; m < M; ++m) {
                                        prev[s][k][p][m] = x[NR - 1][c][p][m];
                                        asm volatile("" : "+v"(prev[s][k][p][m]));  // made here, not at the loop's end
#pragma unroll
                                        for (int q = NR - 1; q > 0; --q) x[q][c][p][m] = x[q - 1][c][p][m];
                                        x[0][c][p][m] = old[k][p][m];
                                    }
                                ++k;
                            }
                    };
                    if constexpr (INV) {
                        move_i();
                        move_j();
                        coin();
                    } else {
                        const int gs = stage * KL + s;  // level of the launch
                        coin();
                        if constexpr (SOME && kScaled && sizeof(R) == 4) {
                            if (s < KL - 1 && mark_at(A.marks, gs)) {
                                const R f = mark_scale<R>(A.marks, gs);
#pragma unroll
                                for (int q = 0; q < NR; ++q)
#pragma unroll
                                    for (int c = 0; c < 4; ++c)
#pragma unroll
                                        for (int p = 0; p < NP; ++p)
#pragma unroll
                                            for (int m = 0; m < M; ++m) x[q][c][p][m] *= f;
                            }
                        }
                        move_j();
                        if (SOME ? gs < kk - 1 : s < KL - 1 || stage < NS - 1) move_i();
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (NS > 1 && stage < NS - 1) {
                const int last = stage * KL + KL - 1;  // a mark there is applied here
                const R f = kScaled && sizeof(R) == 4 && mark_at(A.marks, last) ? mark_scale<R>(A.marks, last) : (R)1;
#pragma unroll
                for (int q = 0; q < NR; ++q)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
#pragma unroll
                        for (int p = 0; p < NP; ++p) {
                            V v;
#pragma unroll
                            for (int m = 0; m < M; ++m) v.v[m] = kScaled && sizeof(R) == 4 ? x[q][c][p][m] * f : x[q][c][p][m];
                            mine[(((g & 1) * NR + q) * 4 * NP + c * NP + p) * 64 + lane] = v;
                        }
            } else {
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    const int rq = INV ? r - q : r + q;
                    if (rq >= r0 && rq < r1 && own) {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
#pragma unroll
                            for (int p = 0; p < NP; ++p) {
                                V o;
#pragma unroll
                                for (int m = 0; m < M; ++m) o.v[m] = kScaled ? x[q][c][p][m] * (R)A.unscale : x[q][c][p][m];
                                if (A.partial) {
#pragma unroll
                                    for (int m = 0; m < M; ++m)
                                        if (col + m < A.cols) nacc = fmaR((double)o.v[m], (double)o.v[m], nacc);
                                }
                                *(V *)(dst + (2 * c + p) * A.ps + (int64_t)(INV ? rq : rq + cone_di(TABLE, c)) * A.ld + col) = o;
                            }
                    }
                }
            }
        }
    };
    // (two loops in sequence: both kinds of group in one would hold the registers of both)
    const int total = iters + NS - 1, some = whole ? min(total, K / NR + NS - 2) : total;
    int it = 0;
#pragma unroll 1
    for (; it < some; ++it) {
        const int g = it - stage;
        if (NS == 1 || (active && g >= 0 && g < iters)) group(g, std::true_type{});
        if (NS > 1) __syncthreads();
        r += INV ? -NR : NR;
    }
#pragma unroll 1
    for (; it < total; ++it) {
        const int g = it - stage;
        if (NS == 1 || (active && g < iters)) group(g, std::false_type{});
        if (NS > 1) __syncthreads();
        r += INV ? -NR : NR;
    }
    if (A.partial && active && stage == NS - 1) {
        nacc = wave_sum64(nacc);
        if (lane == 0) A.partial[tile] = nacc;
    }
}

// The same steps on a small square, where a launch of k_cone lasts one wave's
// stream (rows x levels in series) and most of the chip idles.  A workgroup of 16
// waves takes a tile of 16 RW rows x 64 columns, RW rows per wave in registers, and
// brings all of it to the next level at once: within a wave rows pass in registers
// and columns by lane exchange, between waves the last row's two moving components
// go through LDS (two buffers, one barrier per level).  After kk levels the rows
// from kk - 1 and the columns from kk on are final.  Waves whose rows no later
// level needs only keep the barriers.
constexpr int kTW = 16;  // waves of a tile
template <typename R, int RW, int TABLE, int COIN, bool CPLX, bool INV>
__global__ __launch_bounds__(64 * kTW) void k_cone_tile(const R *__restrict__ in, R *__restrict__ out, ConeArgs A,
                                                        CoinR<R> C) {
    constexpr int NP = CPLX ? 2 : 1;
    constexpr bool kScaled = !INV && COIN != COIN_DENSE;
    __shared__ R edge[2][kTW + 1][2 * NP][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int strip = blockIdx.x % A.nstrips, rest = blockIdx.x / A.nstrips;
    const int seg = rest % A.nseg, part = rest / A.nseg;
    const int t = A.t, kk = A.kk, spill = INV ? kk : kk - 1;  // rows of the tile that only feed others
    const int r0 = seg * A.seg_rows, r1 = min(A.rows, r0 + A.seg_rows);
    const int c0 = strip * (64 - kk), col = c0 + lane - (INV ? 0 : kk);
    const bool lane_in = col >= 0 && col <= t;
    const int lcol = lane_in ? col : 0;
    const R *src = in + part * A.ps;
    R *dst = out + part * A.ps;
    // row q of this wave in stream order: a row takes from the one before it
    const int first = INV ? r0 + A.seg_rows - 1 + spill - wave * RW : r0 - spill + wave * RW;
    R x[RW][4][NP];
#pragma unroll
    for (int q = 0; q < RW; ++q) {
        const int r = INV ? first - q : first + q;
        const int64_t o = (int64_t)min(max(r, 0), t) * A.ld + lcol;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int di = cone_di(TABLE, c);
            const bool ok = lane_in && r >= row_lo(t, di) && r <= row_hi(t, di);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const R v = src[(2 * c + p) * A.ps + o];
                x[q][c][p] = ok ? v : (R)0;
            }
        }
    }
    if (wave == 0) {
#pragma unroll
        for (int k = 0; k < 2 * NP; ++k) edge[0][0][k][lane] = edge[1][0][k][lane] = (R)0;
    }
#pragma unroll 1
    for (int s = 0; s < kk; ++s) {
        const bool live = (wave + 1) * RW > s;  // some row of this wave still counts
        auto coin = [&]() {
#pragma unroll
            for (int q = 0; q < RW; ++q) site_coin<R, COIN, NP>(x[q], C);
        };
        auto move_j = [&]() {
#pragma unroll
            for (int q = 0; q < RW; ++q)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (cone_dj(TABLE, c))
#pragma unroll
                        for (int p = 0; p < NP; ++p) x[q][c][p] = lane_shift<INV>(x[q][c][p]);
        };
        if (live) {
            if constexpr (!INV) {
                coin();
                if (kScaled && mark_at(A.marks, s)) {
                    const R f = mark_scale<R>(A.marks, s);
#pragma unroll
                    for (int q = 0; q < RW; ++q)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
#pragma unroll
                            for (int p = 0; p < NP; ++p) x[q][c][p] *= f;
                }
                move_j();
            }
            if (INV || s + 1 < kk) {
                int k = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (cone_di(TABLE, c)) {
#pragma unroll
                        for (int p = 0; p < NP; ++p) edge[s & 1][wave + 1][k * NP + p][lane] = x[RW - 1][c][p];
                        ++k;
                    }
            }
        }
        if (INV || s + 1 < kk) {  // (the last move along I is the row it is stored to)
            __syncthreads();
            if (live) {
                int k = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (cone_di(TABLE, c)) {
#pragma unroll
                        for (int p = 0; p < NP; ++p) {
#pragma unroll
                            for (int q = RW - 1; q > 0; --q) x[q][c][p] = x[q - 1][c][p];
                            x[0][c][p] = edge[s & 1][wave][k * NP + p][lane];
                        }
                        ++k;
                    }
            }
        }
        if constexpr (INV) {
            if (live) {
                move_j();
                coin();
            }
        }
    }
    const bool own = INV ? (lane < 64 - kk && col < A.cols) : (lane >= kk && col < A.cols);
    double nacc = 0.0;
#pragma unroll
    for (int q = 0; q < RW; ++q) {
        const int r = INV ? first - q : first + q;
        if (own && r >= r0 && r < r1) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const R v = kScaled ? x[q][c][p] * (R)A.unscale : x[q][c][p];
                    dst[(2 * c + p) * A.ps + (int64_t)(INV ? r : r + cone_di(TABLE, c)) * A.ld + col] = v;
                    nacc = fmaR((double)v, (double)v, nacc);
                }
        }
    }
    if (A.partial) {  // uniform over the launch
        __shared__ double ws[kTW];
        nacc = wave_sum64(nacc);
        if (lane == 0) ws[wave] = nacc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double n = 0.0;
            for (int i = 0; i < kTW; ++i) n += ws[i];
            A.partial[blockIdx.x] = n;
        }
    }
}

// psi_0 at the square's only point
template <typename R> __global__ void k_cone_place(R *a, int64_t ps, ConePsi0 p) {
    const int i = threadIdx.x;
    if (i < 8) a[i * ps] = (R)((i & 1) ? p.im[i >> 1] : p.re[i >> 1]);
}

struct ConeView {  // a state of time t around x0 on its torus
    Geom g;
    int64_t ps;
    int ld, t, x0, y0;
};

// offset of coordinate v from o on a ring of L sites, in (-L/2, L/2]
__device__ __forceinline__ int ring_off(int v, int o, int L) {
    int d = v - o;
    d = d < 0 ? d + L : d;
    return 2 * d > L ? d - L : d;
}

// the square's point of the site at offset (dx, dy); false: not a live site
template <int TABLE> __device__ __forceinline__ bool cone_point(int t, int dx, int dy, int &I, int &J) {
    const int a = TABLE == TABLE_DIAG ? dy : dx + dy, b = TABLE == TABLE_DIAG ? dx : dx - dy;
    if (a < -t || a > t || b < -t || b > t || ((a + t) & 1) || ((b + t) & 1)) return false;
    I = (a + t) >> 1;
    J = (b + t) >> 1;
    return true;
}

// psi(x, y, c): the one or (t = L / 2, across the seam) more points that are the
// site, of which component c is non-zero at one
template <typename R, int TABLE>
__device__ __forceinline__ cv<R> cone_value(const R *__restrict__ a, const ConeView &V, int x, int y, int c) {
    const int dx = ring_off(x, V.x0, V.g.Lx), dy = ring_off(y, V.y0, V.g.Ly);
    const int di = cone_di(TABLE, c);
    cv<R> v = czero<R>();
    for (int k = 0; k < 4; ++k) {
        const int ex = (k & 1) ? dx - V.g.Lx : dx, ey = (k & 2) ? dy - V.g.Ly : dy;
        int I, J;
        if (ex < -V.t || ey < -V.t || !cone_point<TABLE>(V.t, ex, ey, I, J)) continue;
        if (I < row_lo(V.t, di) || I > row_hi(V.t, di)) continue;
        const R *p = a + 2 * c * V.ps + (int64_t)I * V.ld + J;
        v.x += p[0];
        v.y += p[V.ps];
    }
    return v;
}

// psi as complex128 planes over the whole lattice (FULL = false), or the
// whole-lattice pre-shift state a(y, c) = psi(y + e_c, c) (FULL = true)
template <typename R, int TABLE, bool FULL>
__global__ __launch_bounds__(256) void k_cone_expand(const R *__restrict__ a, ConeView V, void *__restrict__ out) {
    // sites in one run (a block a row leaves most lanes idle on narrow tori: 64 x 16384 sites 40 us)
    const unsigned n = (unsigned)V.g.ps, Lx = (unsigned)V.g.Lx;
    for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const int y = (int)(i / Lx), x = (int)(i - (unsigned)y * Lx);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int64_t o = (int64_t)c * V.g.ps + i;
            if constexpr (FULL) {
                ((cv<R> *)out)[o] = cone_value<R, TABLE>(a, V, wrapi(x + V.g.ex[c], V.g.Lx), wrapi(y + V.g.ey[c], V.g.Ly), c);
            } else {
                const cv<R> v = cone_value<R, TABLE>(a, V, x, y, c);
                ((double2 *)out)[o] = make_double2((double)v.x, (double)v.y);
            }
        }
    }
}

// |psi|^2 of point (I, J), components ascending
template <typename R, int TABLE>
__device__ __forceinline__ double point_prob(const R *__restrict__ a, const ConeView &V, int I, int J) {
    const R *q = a + (int64_t)I * V.ld + J;
    double p = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int di = cone_di(TABLE, c);
        if (I >= row_lo(V.t, di) && I <= row_hi(V.t, di)) {
            const double re = (double)q[2 * c * V.ps], im = (double)q[(2 * c + 1) * V.ps];
            p += re * re + im * im;
        }
    }
    return p;
}

// t = L / 2: the points at offset -t along an axis are the sites at +t; p plus theirs, for the
// site at offset (dx, dy)
template <typename R, int TABLE>
__device__ __forceinline__ double seam_prob(const R *__restrict__ a, const ConeView &V, int dx, int dy, double p) {
    const int t = V.t;
    const bool ax = 2 * t == V.g.Lx && t > 0 && dx == t, ay = 2 * t == V.g.Ly && t > 0 && dy == t;
    int I, J;
    if (ax && cone_point<TABLE>(t, -t, dy, I, J)) p += point_prob<R, TABLE>(a, V, I, J);
    if (ay && cone_point<TABLE>(t, dx, -t, I, J)) p += point_prob<R, TABLE>(a, V, I, J);
    if (ax && ay && cone_point<TABLE>(t, -t, -t, I, J)) p += point_prob<R, TABLE>(a, V, I, J);
    return p;
}

// k_cone_prob_sites on lattices of at most so many sites.  Tiles / sites, us, complex128, t = L / 4 and L / 2: 512^2
// pair table 16.2 / 4.6 and 16.4 / 4.9, 2048^2 29.0 / 13.6 and 32.7 / 26.3, diagonal 14.6 / 13.8 and
// 35.5 / 27.1; 4096^2 pair 41 / 46 and 152 / 126, diagonal 35 / 51 and 128 / 137.
constexpr int64_t kProbSites = 1 << 22;

// P over the whole lattice, a site per lane: small lattices, where the tiles below are too
// few to hide their serial loads.  A wave takes 8 x 8 sites (a block 16 x 16): with the
// axis-aligned tables their points are a patch of the square, not one long diagonal.
template <typename R, int TABLE>
__global__ __launch_bounds__(256) void k_cone_prob_sites(const R *__restrict__ a, ConeView V, double *__restrict__ P, int ntx) {
    const int ty = (int)(blockIdx.x / (unsigned)ntx), tx = (int)blockIdx.x - ty * ntx, tid = threadIdx.x;
    const int x = tx * 16 + ((tid >> 6) & 1) * 8 + (tid & 7), y = ty * 16 + (tid >> 7) * 8 + ((tid >> 3) & 7);
    if (x >= V.g.Lx || y >= V.g.Ly) return;
    const int dx = ring_off(x, V.x0, V.g.Lx), dy = ring_off(y, V.y0, V.g.Ly);
    int I, J;
    double p = 0.0;
    if (cone_point<TABLE>(V.t, dx, dy, I, J)) p = point_prob<R, TABLE>(a, V, I, J);
    P[(int64_t)y * V.g.Lx + x] = seam_prob<R, TABLE>(a, V, dx, dy, p);
}

// P over the whole lattice.  A block writes 64 x 64 sites.  With the axis-aligned
// tables a lattice row runs along a diagonal of the square, so the block takes
// its points in the square's order (coalesced loads) into an LDS tile and writes
// the tile's rows; with the diagonal table rows are rows.  A tile off the cone
// (most of them, on a large torus) writes its zeros at once.  Bound by the writes.
constexpr int kPT = 64, kPPitch = kPT + 2;  // pitch: a diagonal's points fall on different banks
struct alignas(8) Pair64 {
    double a, b;
};
template <typename R, int TABLE>
__global__ __launch_bounds__(256) void k_cone_prob(const R *__restrict__ a, ConeView V, double *__restrict__ P, int skew, int ntx) {
    __shared__ double s[kPT * kPPitch];
    // the tile's first offset: offsets run over (-L/2, L/2]; the first column of tiles
    // starts skew sites early, on a 128-byte line of P
    const int Lx = V.g.Lx, Ly = V.g.Ly, t = V.t, tid = threadIdx.x;
    // (one grid dimension: a narrow torus may have more than 65535 rows of tiles)
    const int ty = (int)(blockIdx.x / (unsigned)ntx), tx = (int)blockIdx.x - ty * ntx;
    const int bx = tx * kPT - (Lx - 1) / 2 - skew, by = ty * kPT - (Ly - 1) / 2;
    const int lx0 = tx == 0 ? skew : 0;                                  // tile inside the lattice
    const int nx = min(kPT, Lx / 2 - bx + 1), ny = min(kPT, Ly / 2 - by + 1);
    // distance of the tile from the start site along each axis
    const int gx = max(0, max(bx, -(bx + kPT - 1))), gy = max(0, max(by, -(by + kPT - 1)));
    const bool empty = TABLE == TABLE_DIAG ? gx > t || gy > t : gx + gy > t;  // uniform over the block
    if (!empty) {
        for (int i = tid; i < kPT * kPPitch; i += 256) s[i] = 0.0;
        __syncthreads();
        // points whose sites may lie in the tile (floor halves)
        const int Ia = (TABLE == TABLE_DIAG ? by + t : bx + by + t) >> 1;
        const int Ja = (TABLE == TABLE_DIAG ? bx + t : bx - by - (kPT - 1) + t) >> 1;
        constexpr int kN = TABLE == TABLE_DIAG ? kPT / 2 + 1 : kPT + 1;
        for (int k = tid; k < kN * kN; k += 256) {
            const int I = Ia + k / kN, J = Ja + k % kN;
            if (I < 0 || I > t || J < 0 || J > t) continue;
            const int dx = TABLE == TABLE_DIAG ? 2 * J - t : I + J - t, dy = TABLE == TABLE_DIAG ? 2 * I - t : I - J;
            const int lx = dx - bx, ly = dy - by;
            if (lx < 0 || lx >= nx || ly < 0 || ly >= ny) continue;
            s[ly * kPPitch + lx] = point_prob<R, TABLE>(a, V, I, J);
        }
        __syncthreads();
    }
    auto at = [&](int lx, int ly) -> double {
        if (empty) return 0.0;
        return seam_prob<R, TABLE>(a, V, bx + lx, by + ly, s[ly * kPPitch + lx]);
    };
    for (int k = tid; k < kPT * kPT / 2; k += 256) {
        const int lx = 2 * (k % (kPT / 2)), ly = k / (kPT / 2);
        if (ly >= ny || lx >= nx || lx + 1 < lx0) continue;
        int x = V.x0 + bx + lx, y = V.y0 + by + ly;
        x = x < 0 ? x + Lx : (x >= Lx ? x - Lx : x);
        y = y < 0 ? y + Ly : (y >= Ly ? y - Ly : y);
        double *row = P + (int64_t)y * Lx;
        if (lx >= lx0 && lx + 1 < nx && x + 1 < Lx) {
            *(Pair64 *)(row + x) = Pair64{at(lx, ly), at(lx + 1, ly)};
        } else {
            if (lx >= lx0) row[x] = at(lx, ly);
            if (lx + 1 < nx) row[x + 1 < Lx ? x + 1 : 0] = at(lx + 1, ly);
        }
    }
}

// fp64 norm: block partial sums (rows blockIdx.x, + gridDim.x, ...)
template <typename R, int TABLE>
__global__ __launch_bounds__(256) void k_cone_norm(const R *__restrict__ a, ConeView V, double *__restrict__ partial) {
    __shared__ double ws[4];
    double acc = 0.0;
    for (int I = blockIdx.x; I <= V.t; I += gridDim.x)
        for (int J = threadIdx.x; J <= V.t; J += 256) acc += point_prob<R, TABLE>(a, V, I, J);
    acc = wave_sum64(acc);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

// rescale by 1 / sqrt(n) (fp64) when |n - 1| > tol, as k_renorm
template <typename R>
__global__ __launch_bounds__(256) void k_cone_renorm(R *__restrict__ a, ConeView V, double tol, Scratch *__restrict__ scr) {
    const double n = scr->norm;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        scr->last_check = n;
        if (fabs(n - 1.0) > tol) scr->renorms += 1ull;
    }
    if (!(fabs(n - 1.0) > tol)) return;
    const double sc = 1.0 / sqrt(n);
    for (int k = blockIdx.x; k < 8 * (V.t + 1); k += gridDim.x) {
        R *row = a + (int64_t)(k & 7) * V.ps + (int64_t)(k >> 3) * V.ld;
        for (int J = threadIdx.x; J <= V.t; J += 256) row[J] = (R)((double)row[J] * sc);
    }
}

ConeView cone_view(const Cone &c, const Geom &g) { return ConeView{g, c.ps, c.ld, c.t, c.x0, c.y0}; }

int cone_cus() {
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1) {
            (void)hipGetLastError();
            v = 256;
        }
        return v;
    }();
    return n;
}

// tiles (of TR x TC outputs, RW rows per wave) a launch on the small-square kernel takes
int cone_tiles(int rows, int cols, int kk, bool inv, int RW, int parts) {
    const int TR = kTW * RW - (inv ? kk : kk - 1), TC = 64 - kk;
    return ((rows + TR - 1) / TR) * ((cols + TC - 1) / TC) * parts;
}

template <typename K, typename R>
void cone_go(K kernel, unsigned blocks, unsigned threads, hipStream_t s, hipEvent_t e0, hipEvent_t e1, const void *in,
             void *out, const ConeArgs &A, const CoinF64 &C) {
    if (e0) hipExtLaunchKernelGGL(kernel, dim3(blocks), dim3(threads), 0, s, e0, e1, 0u, (const R *)in, (R *)out, A, to_coin<R>(C));
    else hipLaunchKernelGGL(kernel, dim3(blocks), dim3(threads), 0, s, (const R *)in, (R *)out, A, to_coin<R>(C));
}

// strips, segments and blocks of a launch of k_cone<R, KL, NS, M, ...>
template <typename R, int KL, int NS, int M, bool CPLX> unsigned cone_shape(ConeArgs &A, int waves_per_simd, LaunchInfo *info) {
    constexpr int TW = 64 * M - KL * NS;
    A.nstrips = (A.cols + TW - 1) / TW;
    // segments that give every SIMD its waves, but not so short that the kk - 1 rows
    // each reads before its first cost more than they save
    const long per = (long)A.nstrips * (CPLX ? 1 : 2);
    const long segs = std::max(1L, 4L * cone_cus() * waves_per_simd / NS / per);
    A.seg_rows = std::max((int)((A.rows + segs - 1) / segs), kConeMinRows);
    A.nseg = (A.rows + A.seg_rows - 1) / A.seg_rows;
    const long tiles = per * A.nseg;
    if (info) {
        info->bytes_read = (double)tiles * 64 * M * (CPLX ? 8 : 4) * sizeof(R) * (A.seg_rows + A.kk);
        info->bytes_written = 8.0 * sizeof(R) * A.rows * A.cols;
    }
    return (unsigned)((tiles * NS + 3) / 4);
}

// M, NR: columns per lane and rows per group of the one-stage kernel; the tile
// kernel takes 2 rows per wave (real lanes) or 1
template <typename R, int M, int NR, int TABLE, int COIN, bool CPLX, bool INV>
void cone_launch(const void *in, void *out, const Cone &cn, int kk, uint32_t marks, const CoinF64 &C, hipStream_t s,
                 LaunchInfo *info, Scratch *norm, hipEvent_t ev0, hipEvent_t ev1) {
    constexpr int parts = CPLX ? 1 : 2;
    constexpr int RW = CPLX ? 1 : 2;
    ConeArgs A;
    A.ps = cn.ps;
    A.ld = cn.ld;
    A.t = cn.t;
    A.kk = kk;
    const int t1 = INV ? cn.t - kk : cn.t + kk;
    A.rows = INV ? t1 + 1 : t1;
    A.cols = t1 + 1;
    A.partial = nullptr;
    auto sums = [&](long n) {  // the launch's tiles or blocks, one partial sum each
        if (norm && n <= kRedBlocks) {
            A.partial = norm->partial;
            info->norm_parts = (int)n;
        }
    };
    A.marks = marks & (uint32_t)((1ull << (kk - 1)) - 1u);
    A.unscale = 1.0 / (double)(1ull << (A.marks ? kk - (32 - __builtin_clz(A.marks)) : kk));
    // (a tile deeper than kTileDepth would have no rows left)
    if (kk <= kTileDepth<CPLX> && cone_tiles(A.rows, A.cols, kk, INV, RW, parts) <= kConeTilesPerCu * cone_cus()) {
        A.nstrips = (A.cols + 63 - kk) / (64 - kk);
        A.seg_rows = kTW * RW - (INV ? kk : kk - 1);
        A.nseg = (A.rows + A.seg_rows - 1) / A.seg_rows;
        const unsigned blocks = (unsigned)(A.nstrips * A.nseg * parts);
        if (info) {
            info->bytes_read = (double)blocks * kTW * RW * 64 * (CPLX ? 8 : 4) * sizeof(R);
            info->bytes_written = 8.0 * sizeof(R) * A.rows * A.cols;
        }
        sums(blocks);
        auto *k = k_cone_tile<R, RW, TABLE, COIN, CPLX, INV>;
        cone_go<decltype(k), R>(k, blocks, 64 * kTW, s, ev0, ev1, in, out, A, C);
        return;
    }
    if constexpr (!CPLX && !INV) {
        if (kk > kK) {
            const unsigned blocks = cone_shape<R, kDeepKL, kDeepNS, kDeepM<R>, CPLX>(A, 2, info);
            sums((long)A.nstrips * A.nseg * parts);
            auto *k = k_cone<R, kDeepKL, kDeepNS, kDeepM<R>, kDeepNR, TABLE, COIN, CPLX, INV>;
            cone_go<decltype(k), R>(k, blocks, 256, s, ev0, ev1, in, out, A, C);
            return;
        }
    }
    const unsigned blocks = cone_shape<R, kK, 1, M, CPLX>(A, kConeWaves, info);
    sums((long)A.nstrips * A.nseg * parts);
    auto *k = k_cone<R, kK, 1, M, NR, TABLE, COIN, CPLX, INV>;
    cone_go<decltype(k), R>(k, blocks, 256, s, ev0, ev1, in, out, A, C);
}

template <typename R, int TABLE>
hipError_t cone_table(int coin_impl, bool inverse, const void *in, void *out, const Cone &cn, int kk, uint32_t marks,
                      const CoinF64 &C, hipStream_t s, LaunchInfo *info, Scratch *norm, hipEvent_t e0, hipEvent_t e1) {
    constexpr int M = sizeof(R) == 8 ? 2 : 4;   // real lanes
    constexpr int MC = sizeof(R) == 8 ? 1 : 2;  // complex lanes
    bool real = true;
    for (int i = 0; i < 16; ++i) real = real && C.im[i] == 0.0;
#define QW_CONE_ARGS in, out, cn, kk, marks, C, s, info, norm, e0, e1
    if (inverse) {
        if (real) cone_launch<R, M, 2, TABLE, COIN_DENSE, false, true>(QW_CONE_ARGS);
        else cone_launch<R, MC, 1, TABLE, COIN_DENSE, true, true>(QW_CONE_ARGS);
    } else if (coin_impl == COIN_GROVER4) {
        cone_launch<R, M, 2, TABLE, COIN_GROVER4, false, false>(QW_CONE_ARGS);
    } else if (coin_impl == COIN_HH4) {
        cone_launch<R, M, 2, TABLE, COIN_HH4, false, false>(QW_CONE_ARGS);
    } else if (sizeof(R) == 8 && cn.fourier) {
        if constexpr (sizeof(R) == 8) cone_launch<R, MC, 1, TABLE, kCoinFourier4, true, false>(QW_CONE_ARGS);
    } else {
        cone_launch<R, MC, 1, TABLE, COIN_DENSE, true, false>(QW_CONE_ARGS);
    }
#undef QW_CONE_ARGS
    return hipGetLastError();
}

#define QW_CONE_DISPATCH(prec, table, CALL)                       \
    do {                                                          \
        if ((prec) == C128) {                                     \
            if ((table) == TABLE_PAIR) CALL(double, TABLE_PAIR);  \
            else if ((table) == TABLE_EQ8) CALL(double, TABLE_EQ8); \
            else CALL(double, TABLE_DIAG);                        \
        } else {                                                  \
            if ((table) == TABLE_PAIR) CALL(float, TABLE_PAIR);   \
            else if ((table) == TABLE_EQ8) CALL(float, TABLE_EQ8); \
            else CALL(float, TABLE_DIAG);                         \
        }                                                         \
    } while (0)

}  // namespace

int cone_max_depth() { return 2 * kK; }

int cone_depth(int coin_impl, bool inverse, const Cone &c, const CoinF64 &C, int64_t left, int max_depth) {
    int kk = (int)std::min<int64_t>(left, std::min(max_depth, 2 * kK));
    bool real = coin_impl != COIN_DENSE || inverse;
    for (int i = 0; i < 16; ++i) real = real && C.im[i] == 0.0;
    const int kt = real ? kTileDepth<false> : kTileDepth<true>;
    if (kk <= kt) return kk;
    const int t1 = inverse ? c.t - kt : c.t + kt;
    const int tiles = cone_tiles(inverse ? t1 + 1 : t1, t1 + 1, kt, inverse, real ? 2 : 1, real ? 2 : 1);
    if (tiles <= kConeTilesPerCu * cone_cus()) return kt;
    if (kk > kK && (inverse || !real || c.t < kDeepSide)) kk = kK;
    return kk;
}

bool cone_fits(const Geom &g, int table, size_t state_bytes, int prec, Cone *c) {
    if (g.d != 4 || (table != TABLE_PAIR && table != TABLE_EQ8 && table != TABLE_DIAG)) return false;
    const int L = std::min(g.Lx, g.Ly);
    if (L < kConeMinSide) return false;
    c->tmax = L / 2;
    c->ld = (c->tmax + 1 + 15) / 16 * 16;
    c->ps = (int64_t)c->ld * (c->tmax + 1);
    return (size_t)c->ps * 8 * (prec == C128 ? 8 : 4) <= state_bytes;
}

hipError_t launch_cone_place(int prec, void *state, const Cone &c, const double *psi0, hipStream_t s) {
    ConePsi0 p;
    for (int k = 0; k < 4; ++k) {
        p.re[k] = psi0[2 * k];
        p.im[k] = psi0[2 * k + 1];
    }
    if (prec == C128) hipLaunchKernelGGL(k_cone_place<double>, dim3(1), dim3(64), 0, s, (double *)state, c.ps, p);
    else hipLaunchKernelGGL(k_cone_place<float>, dim3(1), dim3(64), 0, s, (float *)state, c.ps, p);
    return hipGetLastError();
}

hipError_t launch_cone_steps(int prec, int coin_impl, int table, bool inverse, const void *in, void *out, const Cone &c,
                             int kk, uint32_t marks, const CoinF64 &C, hipStream_t s, LaunchInfo *info,
                             Scratch *norm, hipEvent_t ev_start, hipEvent_t ev_stop) {
    if (kk < 1 || kk > 2 * kK || (kk > kK && inverse) || (inverse ? kk > c.t : c.t + kk > c.tmax)) return hipErrorInvalidValue;
#define QW_CALL(R, TAB) return cone_table<R, TAB>(coin_impl, inverse, in, out, c, kk, marks, C, s, info, norm, ev_start, ev_stop)
    QW_CONE_DISPATCH(prec, table, QW_CALL);
#undef QW_CALL
    return hipErrorInvalidValue;
}

hipError_t launch_cone_prob(int prec, int table, const void *state, const Cone &c, const Geom &g, double *P, hipStream_t s) {
    const ConeView V = cone_view(c, g);
    if (g.ps <= kProbSites) {
        const int ntx = (g.Lx + 15) / 16;
        const dim3 grid((unsigned)ntx * (unsigned)((g.Ly + 15) / 16));
#define QW_CALL(R, TAB) hipLaunchKernelGGL((k_cone_prob_sites<R, TAB>), grid, dim3(256), 0, s, (const R *)state, V, P, ntx)
        QW_CONE_DISPATCH(prec, table, QW_CALL);
#undef QW_CALL
        return hipGetLastError();
    }
    // the lattice column of the first offset, down to a line of 16
    int first = (int)(((int64_t)c.x0 - (g.Lx - 1) / 2 + g.Lx) % g.Lx);
    const int skew = first % 16, ntx = (g.Lx + skew + kPT - 1) / kPT;
    const dim3 grid((unsigned)ntx * (unsigned)((g.Ly + kPT - 1) / kPT));
#define QW_CALL(R, TAB) hipLaunchKernelGGL((k_cone_prob<R, TAB>), grid, dim3(256), 0, s, (const R *)state, V, P, skew, ntx)
    QW_CONE_DISPATCH(prec, table, QW_CALL);
#undef QW_CALL
    return hipGetLastError();
}

hipError_t launch_cone_norm(int prec, int table, const void *state, const Cone &c, const Geom &g, Scratch *scr, hipStream_t s) {
    const ConeView V = cone_view(c, g);
    const int blocks = std::min(c.t + 1, kRedBlocks);
#define QW_CALL(R, TAB) hipLaunchKernelGGL((k_cone_norm<R, TAB>), dim3(blocks), dim3(256), 0, s, (const R *)state, V, scr->partial)
    QW_CONE_DISPATCH(prec, table, QW_CALL);
#undef QW_CALL
    return launch_reduce_final(scr, blocks, s);
}

hipError_t launch_cone_renorm(int prec, void *state, const Cone &c, const Geom &g, double tol, Scratch *scr, hipStream_t s) {
    const ConeView V = cone_view(c, g);
    const int blocks = std::min(8 * (c.t + 1), 4096);
    if (prec == C128) hipLaunchKernelGGL(k_cone_renorm<double>, dim3(blocks), dim3(256), 0, s, (double *)state, V, tol, scr);
    else hipLaunchKernelGGL(k_cone_renorm<float>, dim3(blocks), dim3(256), 0, s, (float *)state, V, tol, scr);
    return hipGetLastError();
}

hipError_t launch_cone_expand(int prec, int table, const void *state, const Cone &c, const Geom &g, void *out, bool full,
                              hipStream_t s) {
    const ConeView V = cone_view(c, g);
    const dim3 grid((unsigned)std::min<int64_t>((g.ps + 255) / 256, 1 << 16));
#define QW_CALL(R, TAB)                                                                                                \
    do {                                                                                                               \
        if (full) hipLaunchKernelGGL((k_cone_expand<R, TAB, true>), grid, dim3(256), 0, s, (const R *)state, V, out);  \
        else hipLaunchKernelGGL((k_cone_expand<R, TAB, false>), grid, dim3(256), 0, s, (const R *)state, V, out);      \
    } while (0)
    QW_CONE_DISPATCH(prec, table, QW_CALL);
#undef QW_CALL
    return hipGetLastError();
}

}  // namespace qw
