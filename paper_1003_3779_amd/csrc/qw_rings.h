// qw_rings.h -- ring walks whose cone never wraps, held as the points they can
// reach (device code of qw_batch.hip).
//
// Such a walk runs in the rotation frame (real coin) from one site; after t steps
// its amplitudes live at the offsets d = 2 i - t, i = 0 .. t.  With psi_t at these
// points a step is, point by point,
//     (o0, o1) = coin(psi_t[i]);   psi_{t+1}[i + 1].c0 = o0;   psi_{t+1}[i].c1 = o1:
// one component stays and the other moves up by one.  Same expressions as the tiled
// path (CoinRotS, f^16 every 16 steps, the fp64 norm after every block of K steps
// and its rescale applied to the block's output): the same values bit for bit.
#pragma once

namespace qw {
namespace {

// ---------------------------------------------------------------- short walks
// One walk per workgroup, all its points in registers: a lane holds M consecutive
// points (one lane exchange per step), M growing with the cone.  No memory traffic,
// no halo, no barrier in the steps: bound by the FMAs (4 per point and step of
// complex64, 132 of the 139 instructions of a full lane's step; 16384 rings of 4097
// sites, T in [256, 2048]: 1.64 ms, 63 TFLOP/s of the 78.6 unpacked fp32 ones, against
// 3.76 ms in 128-slot tiles through the slot buffers).  Complex lanes in one wave, or
// a wave for the real and one for the imaginary parts (the coin is real: they meet
// only in norms and in P): always in complex128, whose registers hold no more, and in
// complex64 where the walks are so few that the longest one's steps are the time
// (16 rings 286 us against 450, 4000 rings 500 against 566; 16384 rings 1.84 ms against 1.63).
constexpr int64_t kFewWaves = 6144;
constexpr int kWaveM = 33;                   // most points a lane: T <= 64 * 33 - 1 (rings to 4097 sites whole)
constexpr int kWaveMaxT = 64 * kWaveM - 1;
// the lanes' point counts in turn; a walk moves to the next when its cone fills it
constexpr int kWaveMs[] = {2, 4, 6, 8, 11, 14, 17, 21, 25, 29, 33};
constexpr int kWavePhases = sizeof(kWaveMs) / sizeof(kWaveMs[0]);

template <typename R> __device__ __forceinline__ R lane_up(R v);  // lane l takes lane l - 1's value, lane 0 zero
template <> __device__ __forceinline__ float lane_up<float>(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}
template <> __device__ __forceinline__ double lane_up<double>(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, 0x138, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), 0x138, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// one real part of CoinRotS
template <typename R, bool SWAP> __device__ __forceinline__ R rot0(R t, R g0, R g1) { return SWAP ? fmaR(t, g0, g1) : fmaR(t, g1, g0); }
template <typename R, bool SWAP> __device__ __forceinline__ R rot1(R t, R g0, R g1) { return SWAP ? fmaR(t, g1, -g0) : fmaR(-t, g0, g1); }

// rot0 with a destination of its own: the compiler ties a fused multiply-add whose
// addend dies to the addend's register and then moves the result one register on
// (a third of the instructions of a step)
template <bool SWAP> __device__ __forceinline__ float rot0_to(float t, float g0, float g1) {
    float o;
    if constexpr (SWAP) asm("v_fma_f32 %0, %1, %2, %3" : "=v"(o) : "v"(t), "v"(g0), "v"(g1));
    else asm("v_fma_f32 %0, %1, %2, %3" : "=v"(o) : "v"(t), "v"(g1), "v"(g0));
    return o;
}
template <bool SWAP> __device__ __forceinline__ double rot0_to(double t, double g0, double g1) {
    double o;
    if constexpr (SWAP) asm("v_fma_f64 %0, %1, %2, %3" : "=v"(o) : "v"(t), "v"(g0), "v"(g1));
    else asm("v_fma_f64 %0, %1, %2, %3" : "=v"(o) : "v"(t), "v"(g1), "v"(g0));
    return o;
}

// one step on M points per lane: descending, so that a point's c0 is consumed before
// the point below writes it
template <typename R, int M, int NP, bool SWAP, int MC> __device__ __forceinline__ void point_step(R (&c0)[MC][NP], R (&c1)[MC][NP], R t) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        R up = (R)0;
#pragma unroll
        for (int m = M - 1; m >= 0; --m) {
            const R g0 = c0[m][p], g1 = c1[m][p];
            if (m == M - 1) up = rot0<R, SWAP>(t, g0, g1);
            else c0[m + 1][p] = rot0_to<SWAP>(t, g0, g1);
            c1[m][p] = rot1<R, SWAP>(t, g0, g1);
        }
        c0[0][p] = lane_up<R>(up);
    }
}

// Registers and constants of a short walk
template <typename R, int NP, bool SWAP> struct WaveWalk {  // NP: parts per lane
    static constexpr int NW = 3 - NP;                           // waves
    R c0[kWaveM][NP], c1[kWaveM][NP];
    R t, f16, sc;
    R *buf;           // this wave's LDS buffer: 64 kWaveM values
    double *s_norm;   // 2 x NW
    int T, K, step, lane, wave, npar, renorm, m_end;
    double tol;

    // fp64 norm over the first M points of each lane (the others are zero)
    template <int M> __device__ __forceinline__ double norm() {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                a = fmaR((double)c0[m][p], (double)c0[m][p], a);
                b = fmaR((double)c1[m][p], (double)c1[m][p], b);
            }
        double n = wave_sum64(a + b);
        if constexpr (NW > 1) {
            if (lane == 0) s_norm[npar * NW + wave] = n;
            __syncthreads();
            n = s_norm[npar * NW] + s_norm[npar * NW + 1];
            npar ^= 1;
        }
        return n;
    }
    template <int M> __device__ __forceinline__ void scale(R f) {
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                c0[m][p] *= f;
                c1[m][p] *= f;
            }
    }
    // a plane from M to M2 points per lane
    template <int M, int M2> __device__ __forceinline__ void relayout(R (&c)[kWaveM][NP], int p) {
#pragma unroll
        for (int m = 0; m < M; ++m) buf[lane * M + m] = c[m][p];
        __syncthreads();
#pragma unroll
        for (int m = 0; m < M2; ++m) {
            const int i = lane * M2 + m;
            c[m][p] = i < 64 * M ? buf[i < 64 * M ? i : 0] : (R)0;
        }
        __syncthreads();
    }
    // steps with kWaveMs[I] points per lane until the walk ends or the cone fills the
    // lanes, with what a block does at its end; then on with more points
    template <int I> __device__ __forceinline__ void phases() {
        constexpr int M = kWaveMs[I];
        const int end = min(T, 64 * M - 1);  // after step t the points 0 .. t are live
        while (step < end) {
            const int n = min(kFactorEvery - step % kFactorEvery, end - step);
            for (int k = 0; k < n; ++k) point_step<R, M, NP, SWAP, kWaveM>(c0, c1, t);
            step += n;
            if (step % kFactorEvery == 0) {
                scale<M>(f16);
                if (renorm > 0 && step % K == 0 && step < T) {
                    const double nrm = norm<M>();
                    if (fabs(nrm - 1.0) > tol) scale<M>((R)(1.0 / sqrt(nrm)));
                }
            }
        }
        m_end = M;
        if constexpr (I + 1 < kWavePhases) {
            if (step < T) {  // the same for every wave of the walk
                constexpr int M2 = kWaveMs[I + 1 < kWavePhases ? I + 1 : I];
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    relayout<M, M2>(c0, p);
                    relayout<M, M2>(c1, p);
                }
                phases<I + 1>();
            }
        }
    }
};

constexpr int kWaveChunk = 11;  // points per lane whose P passes through LDS at once
static_assert(kWaveM % kWaveChunk == 0, "whole chunks");

template <typename R, int NP, bool SWAP>
__device__ __forceinline__ void wave_walk(const WalkDesc &w, const BatchArgs &A, int wi, R *buf, double *s_norm, BinAcc *bins) {
    using W = WaveWalk<R, NP, SWAP>;
    constexpr int NW = W::NW;
    W s;
    s.lane = threadIdx.x & 63;
    s.wave = NW > 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    CoinRotS<R, SWAP> cn;
    load_coin<R>(w, cn);
    s.t = cn.t;
    s.f16 = (R)block_factor(cn, kFactorEvery);
    s.buf = buf + s.wave * 64 * kWaveM;
    s.s_norm = s_norm;
    s.T = w.T;
    s.K = kCfgK[w.cfg];
    s.step = s.npar = 0;
    s.renorm = A.renorm_every;
    s.tol = A.renorm_tol;
#pragma unroll
    for (int m = 0; m < kWaveM; ++m)
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const bool im = NP == 2 ? p == 1 : s.wave == 1, first = m == 0 && s.lane == 0;
            s.c0[m][p] = first ? (R)(im ? w.pim[0] : w.pre[0]) : (R)0;
            s.c1[m][p] = first ? (R)(im ? w.pim[1] : w.pre[1]) : (R)0;
        }
    s.template phases<0>();
    // the last block's output: its pending factor and norm, as block_scale
    const double fk = block_factor(cn, w.T % kFactorEvery);
    double f = fk;
    if (A.renorm_every > 0) {
        const double nrm = s.template norm<kWaveM>() * fk * fk;
        if (fabs(nrm - 1.0) > A.renorm_tol) f = fk / sqrt(nrm);
    }
    const R sc = (R)f;
    // P of the live points, a chunk per lane at a time through LDS, into the moments and bins
    double *pw = (double *)s.buf;
    const int M = s.m_end, T = w.T, N = w.N;
    SiteAcc acc;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kWaveM; c += kWaveChunk) {
        if (c < M) {
#pragma unroll
            for (int q = 0; q < kWaveChunk; ++q) {
                const int m = c + q;
                cv<R> a, b;
                a.x = s.c0[m][0] * sc;
                a.y = NP == 2 ? s.c0[m][NP - 1] * sc : (R)0;
                b.x = s.c1[m][0] * sc;
                b.y = NP == 2 ? s.c1[m][NP - 1] * sc : (R)0;
                pw[s.lane * kWaveChunk + q] = abs2d<R>(a) + abs2d<R>(b);
            }
            __syncthreads();
            for (int k = threadIdx.x; k < 64 * kWaveChunk; k += 64 * NW) {
                const int l = k / kWaveChunk, m = c + k - l * kWaveChunk, i = l * M + m;
                if (m < M && i <= T) {
                    double pr = ((const double *)buf)[k];
                    if constexpr (NW > 1) pr += ((const double *)(buf + 64 * kWaveM))[k];
                    acc.add(pr, 2 * i - T, N, A.nbins, bins);
                }
            }
            __syncthreads();
        }
    }
    const double a = wave_sum64(acc.s0), b = wave_sum64(acc.s1), c = wave_sum64(acc.s2);
    double *red = (double *)buf;
    if (s.lane == 0) {
        red[3 * s.wave + 0] = a;
        red[3 * s.wave + 1] = b;
        red[3 * s.wave + 2] = c;
    }
    __syncthreads();  // orders the bin atomics too
    if (threadIdx.x < 3) {
        double v = red[threadIdx.x];
        if constexpr (NW > 1) v += red[3 + threadIdx.x];
        A.moments[3 * (int64_t)wi + threadIdx.x] = v;
    }
    if (A.bins)
        for (int i = threadIdx.x; i < A.nbins; i += 64 * NW)
            A.bins[(int64_t)wi * A.nbins + i] = (float)((double)bins[i] * (1.0 / kBinScale));
}

// block b: the walk at queue position b (longest first).  LDS: a buffer per wave
// (the plane being relaid, then the chunks of P), the norms, the bins.
constexpr int wave_buf(int NP, size_t real) { return 64 * (3 - NP) * kWaveM * (int)real; }
constexpr size_t wave_lds(int NP, size_t real, int nbins) { return (size_t)wave_buf(NP, real) + 32 + sizeof(BinAcc) * nbins; }
template <typename R, int NP> __global__ __launch_bounds__(64 * (3 - NP), sizeof(R) == 8 ? 2 : (NP == 2 ? 3 : 4)) void k_ring_wave(BatchArgs A) {
    constexpr int kBuf = wave_buf(NP, sizeof(R));
    extern __shared__ __attribute__((aligned(16))) unsigned char mem[];
    R *buf = (R *)mem;
    double *s_norm = (double *)(mem + kBuf);
    BinAcc *bins = (BinAcc *)(mem + kBuf + 32);
    for (int i = threadIdx.x; i < A.nbins; i += 64 * (3 - NP)) bins[i] = 0;  // (barriers follow before the first add)
    const int wi = A.order[blockIdx.x];
    const WalkDesc &w = A.walks[wi];
    if (w.rswap) wave_walk<R, NP, true>(w, A, wi, buf, s_norm, bins);
    else wave_walk<R, NP, false>(w, A, wi, buf, s_norm, bins);
}

// ---------------------------------------------------------------- long walks
// The long walks of a batch advance together, a block of K steps per launch (where that ends
// sooner than the queue: long_pays in qw_batch.hip): their
// cones have the same size at the same time, so a launch is (tiles of that cone) x
// (walks still running, longest first) waves, and the largest walks, which alone
// decided when a batch of one workgroup per walk ended, spread over the whole chip.  A
// tile of 64 M points loses K of them (c0 comes from below only).  256 ragged rings
// up to 99999 sites: 12.6 ms against 63.5 with a workgroup per walk, bound by the
// 781 launches in series (10 us where the cones are small) and the tiles' steps.
// M = 4 loses a quarter of its points at K = 64 and is still the fastest: a launch of
// small cones lasts one tile, and larger tiles are read 64 or 128 bytes a lane
// (M = 8, 16: 14.6 ms; turned through LDS 13.5; 2048 rings of 20001 to 99999
// sites 64 ms at M = 4, 102 at 8, 16).
constexpr int kLongM = 4;
struct LongArgs {
    const WalkDesc *walks;
    const int32_t *order;      // of the long walks, descending in T
    const int64_t *off;        // by order position: first point of the walk's planes
    void *psi[2];              // per walk two planes of T + 1 complex points
    double *norms[2];          // partial norms of each block's output: position * max_tiles + tile
    const int32_t *last_tiles; // by position: tiles of the walk's last block
    int32_t max_tiles;
    int32_t t0, K;             // time at the launch's start, steps per block
    int32_t prev_tiles;        // tiles of the block before (0 at t0 = 0)
    int32_t ntiles;
    int32_t renorm;
    double tol;
};

// scale of the state before a block: from its partial norms (in order), fk as in block_scale
__device__ __forceinline__ double long_scale(const double *part, int n, double fk, double tol) {
    double a = 0.0;
    for (int i = threadIdx.x & 63; i < n; i += 64) a += part[i];
    const double nrm = wave_sum64(a) * fk * fk;
    return fabs(nrm - 1.0) > tol ? fk / sqrt(nrm) : fk;
}

template <typename R, bool SWAP>
__device__ __forceinline__ void long_block(const LongArgs &A, const WalkDesc &w, int pos, int tile) {
    constexpr int M = kLongM;
    const int lane = threadIdx.x & 63, t0 = A.t0, k = min(A.K, w.T - t0);
    CoinRotS<R, SWAP> cn;
    load_coin<R>(w, cn);
    const R f16 = (R)block_factor(cn, kFactorEvery);
    R sc = (R)1;
    if (A.renorm > 0 && A.prev_tiles > 0)
        sc = (R)long_scale(A.norms[0] + (int64_t)pos * A.max_tiles, A.prev_tiles, 1.0, A.tol);
    const int64_t np = (int64_t)w.T + 1;
    const cv<R> *i0 = (const cv<R> *)A.psi[0] + A.off[pos], *i1 = i0 + np;
    cv<R> *o0 = (cv<R> *)A.psi[1] + A.off[pos], *o1 = o0 + np;
    const int TW = 64 * M - A.K, first = tile * TW - A.K + lane * M;  // this lane's first point
    R c0[M][2], c1[M][2];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int i = first + m;
        const bool in = i >= 0 && i <= t0;
        cv<R> a = czero<R>(), b = czero<R>();
        if (t0 == 0) {
            a.x = (R)w.pre[0]; a.y = (R)w.pim[0];
            b.x = (R)w.pre[1]; b.y = (R)w.pim[1];
        } else {
            const int j = in ? i : 0;
            a = i0[j];
            b = i1[j];
        }
        c0[m][0] = in ? a.x * sc : (R)0; c0[m][1] = in ? a.y * sc : (R)0;
        c1[m][0] = in ? b.x * sc : (R)0; c1[m][1] = in ? b.y * sc : (R)0;
    }
    for (int left = k; left > 0; left -= kFactorEvery) {
        const int n = min(left, kFactorEvery);
        for (int s = 0; s < n; ++s) point_step<R, M, 2, SWAP, M>(c0, c1, cn.t);
        if (n == kFactorEvery) {
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    c0[m][p] *= f16;
                    c1[m][p] *= f16;
                }
        }
    }
    double nacc = 0.0;
    const int own = tile * TW, top = t0 + k;  // this tile's points: [own, own + TW), of 0 .. top
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int i = first + m;
        if (i >= own && i <= top) {
            cv<R> a, b;
            a.x = c0[m][0]; a.y = c0[m][1];
            b.x = c1[m][0]; b.y = c1[m][1];
            o0[i] = a;
            o1[i] = b;
            if (A.renorm > 0) nacc += abs2d<R>(a) + abs2d<R>(b);
        }
    }
    if (A.renorm > 0) {
        nacc = wave_sum64(nacc);
        if (lane == 0) A.norms[1][(int64_t)pos * A.max_tiles + tile] = nacc;
    }
}

// four tiles of one walk per workgroup
template <typename R> __global__ __launch_bounds__(256) void k_ring_long(LongArgs A) {
    const int per = (A.ntiles + 3) / 4, pos = blockIdx.x / per;
    const int tile = __builtin_amdgcn_readfirstlane((int)((blockIdx.x - pos * per) * 4 + (threadIdx.x >> 6)));
    if (tile >= A.ntiles) return;  // wave-uniform; no barriers
    const WalkDesc &w = A.walks[A.order[pos]];
    if (w.rswap) long_block<R, true>(A, w, pos, tile);
    else long_block<R, false>(A, w, pos, tile);
}

// the ends of all long walks: moments, bins and P, one workgroup each
template <typename R> __global__ __launch_bounds__(kBT) void k_ring_long_end(LongArgs L, BatchArgs A) {
    __shared__ BinAcc s_bins[kMaxBins];
    __shared__ double s_red[3][kWaves];
    for (int i = threadIdx.x; i < A.nbins; i += kBT) s_bins[i] = 0;
    __syncthreads();
    const int pos = blockIdx.x, wi = L.order[pos];
    const WalkDesc &w = A.walks[wi];
    const int T = w.T, N = w.N, blocks = (T + L.K - 1) / L.K;
    double f = 1.0;  // the factor the last block left pending
    for (int i = 0; i < T % kFactorEvery; ++i) f *= w.rf;
    if (L.renorm > 0 && blocks > 0) {
        f = long_scale(L.norms[blocks & 1] + (int64_t)pos * L.max_tiles, L.last_tiles[pos], f, L.tol);
    }
    const R sc = (R)f;
    const cv<R> *p0 = (const cv<R> *)L.psi[blocks & 1] + L.off[pos], *p1 = p0 + (int64_t)T + 1;
    SiteAcc acc;
    // each thread takes its sites in the tiled path's order (the same sums): the box of
    // the cone, one site in two live
    const int64_t ph = (int64_t)T + 2;
    const int pw = (int)min((int64_t)N, 2 * ph + 1), ps = pw == N ? 0 : wrapN((int64_t)w.x0 - ph, N);
    for (int k = threadIdx.x; k < pw; k += kBT) {
        int x = ps + k;
        x = x >= N ? x - N : x;
        const int d = ring_offset(x, w.x0, N);
        if (d < -T || d > T || ((d + T) & 1)) continue;
        const int i = (d + T) >> 1;
        acc.add(abs2d<R>(cscale<R>(p0[i], sc)) + abs2d<R>(cscale<R>(p1[i], sc)), d, N, A.nbins, s_bins);
    }
    if (A.P) {
        for (int x = threadIdx.x; x < N; x += kBT) {
            const int d = ring_offset(x, w.x0, N);
            double pr = 0.0;
            if (d >= -T && d <= T && ((d + T) & 1) == 0) {
                const int i = (d + T) >> 1;
                pr = abs2d<R>(cscale<R>(p0[i], sc)) + abs2d<R>(cscale<R>(p1[i], sc));
            }
            A.P[w.p_off + x] = pr;
        }
    }
    finish_walk<R>(A, wi, acc, s_bins, s_red);
}

}  // namespace
}  // namespace qw
