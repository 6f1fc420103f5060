// Scattered far field (Sec. 2.4) and its adjoint.
//
// The operator of direction d has taps F[tap][d][x][k] (complex, x a
// Cartesian component) and is applied along time:
//   U[l][b][d][x] = sum_tap sum_k F[tap][d][x][k] I[l - m][b][k],  m = m_lo + tap,
//   S[j][b][k]    = sum_tap sum_{d,x} conj(F[tap][d][x][k]) U[j + m][b][d][x].
// With the rows (l, b) of I taken as one index r, tap m shifts a row by m B:
// both are sums over taps of one complex matrix product, FP64, on the
// matrix cores (k_far_gemm).
//
// The field is transverse, so a unit direction carries two components along
// e1, e2 orthogonal to d; the tap table stores c = 0..nc-1 of them,
// F_c = P_dc . sum_q ..., and U_x = sum_c Q_dcx U_c.  Where some direction is
// not a unit vector to FP64 rounding, the projection I - d d is not one onto a
// plane: nc = 3, P = I - d d, Q = I then.
#pragma once
#include "aim.inc.hip"

namespace etaim {

typedef double dx4 __attribute__((ext_vector_type(4)));

// The CPPIF and its derivative at tau; false outside the support.  Its four
// pieces (as cppif_piece) from their coefficients, without its divisions and
// loops.
__device__ __forceinline__ bool far_cppif(double tau, double& T0, double& T1) {
    if (!(tau > -1.0 && tau <= (double)kQ)) return false;
    const double p = ceil(tau), s = tau - p;
    const int i = (int)p;
    const double e1 = 6.0 - p, e2 = i == 0 ? 11.0 : i == 1 ? 6.0 : i == 2 ? 3.0 : 2.0, e3 = i == 0 ? 6.0 : 0.0;
    const double r = i == 0 ? 1.0 / 6.0 : i == 1 ? -0.5 : i == 2 ? 0.5 : -1.0 / 6.0;
    T0 = (((s + e1) * s + e2) * s + e3) * r;
    T1 = ((3.0 * s + 2.0 * e1) * s + e2) * r;
    return true;
}

// (-1)^j / (2j+1)!
struct FarSinc {
    double c[16];
};
__host__ __device__ constexpr FarSinc far_sinc() {
    FarSinc f{};
    double v = 1.0;
    for (int j = 0; j < 16; ++j) {
        if (j > 0) v /= -(2.0 * j) * (2.0 * j + 1.0);
        f.c[j] = v;
    }
    return f;
}

// The BLIF and its derivative at tau (TBasis::blif_at without its second and
// third derivatives and, near tau = 0, its powers: 16 terms of the sinc's
// series by Horner's rule in (pi tau)^2)
__device__ __forceinline__ bool far_blif(const TBasis& tb, double tau, double& T0, double& T1) {
    if (!(tau > tb.lo() && tau <= tb.hi())) return false;
    const double MM = (double)tb.M * (double)tb.M, u = 1.0 - tau * tau / MM, u1 = -2.0 * tau / MM;
    double w0 = 0, w1 = 0;
    for (int k = kBlifTerms - 1; k >= 0; --k) {
        w0 = w0 * u + tb.c[k];
        if (k >= 1) w1 = w1 * u + tb.c[k] * (double)k;
    }
    const double x = kPi * tau, x2 = x * x;
    double S0, S1;
    if (fabs(tau) < 0.25) {
        // sin x / x = sum_j (-x2)^j / (2j+1)!, its x-derivative x sum_j 2 (j+1) (-1)^(j+1) x2^j / (2j+3)!
        constexpr FarSinc f = far_sinc();
        S0 = S1 = 0;
#pragma unroll
        for (int j = 15; j >= 0; --j) {
            S0 = S0 * x2 + f.c[j];
            if (j >= 1) S1 = S1 * x2 + f.c[j] * (2.0 * (double)j);
        }
        S1 = kPi * x * S1;
    } else {
        double sx, cx;
        sincos(x, &sx, &cx);
        S0 = sx / x;
        S1 = kPi * (x * cx - sx) / x2;
    }
    T0 = S0 * w0;
    T1 = S1 * w0 + S0 * (w1 * u1);
    return true;
}

// where a tap's sums start: 0, but NaN for a direction that is not finite (its
// points fall outside the support, so no term would carry it)
__device__ __forceinline__ double far_zero(const double* u) {
    return 0.0 * fabs(u[0]) + 0.0 * fabs(u[1]) + 0.0 * fabs(u[2]);
}

// acc[c] += g[c][q] (a + j b) (cs + j sn), a = T'/dt, b = w T
template <int NC, size_t NQ>
__device__ __forceinline__ void far_term(zd (&acc)[NC], const double (&g)[NC][NQ], int q, double a, double b,
                                         double cs, double sn) {
    const double fr = a * cs - b * sn;
    const double fi = a * sn + b * cs;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        acc[c].x += g[c][q] * fr;
        acc[c].y += g[c][q] * fi;
    }
}

// Tap table F[tap][d nc + c][k] =
//   -(mu/4pi) sum_q (P_dc . Sq[k][q]) [T'(tau)/dt + j w T(tau)] exp(j kc d.r_q),
//   tau = (m_lo + tap) + d.r_q/(c dt);
// geo[d] = {d, P_d0, P_d1, P_d2}.  A thread owns one (d, k) and every nz-th
// tap: the 14 phases and projections do not depend on the tap and stay in
// registers, and the taps outside the basis's support (all but 5 or 6, of
// 27 at N_g = 24) only store zeros.  Bound by the store of the table.  With
// a thread per (tap, d, k), each evaluating the phases again, and the range
// of the cube around the object (43 taps on the unit sphere): 2490 us for 64
// directions x 7680 bases; this kernel 2 x 173 us (27 taps).  Few directions
// leave most of the card idle, with a chain of every tap on each thread: the
// blocks' third index then shares the taps out (one direction of 480 bases, 7
// taps: 16 -> 9 us; of 7680 bases, 27 taps: 63 -> 22 us).  The BLIF's table took
// 520 us for 480 bases and 9 taps with every tap on a thread and the sinc's
// series by powers, 286 with a thread per tap, 17 this way.
template <int NC, bool BLIF>
__global__ void __launch_bounds__(128) k_far_taps(zd* __restrict__ F, const double* __restrict__ Sq,
                                                  const double* __restrict__ rq, const double* __restrict__ geo,
                                                  int nd, int ns, int ntap, int m_lo, double dt, double w,
                                                  double mu4pi, TBasis tb) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x, d = blockIdx.y;
    if (k >= ns) return;
    const double kc = w / kC0, cdt = kC0 * dt, idt = 1.0 / dt;
    const double* u = geo + 12 * (size_t)d;
    double s[14], cs[14], sn[14], g[NC][14];
    double smin = INFINITY, smax = -INFINITY;
#pragma unroll
    for (int q = 0; q < 14; ++q) {
        const double* S = Sq + ((size_t)k * 14 + q) * 3;
        const double* r = rq + ((size_t)k * 14 + q) * 3;
        const double dr = r[0] * u[0] + r[1] * u[1] + r[2] * u[2];
        sincos(kc * dr, &sn[q], &cs[q]);
        s[q] = dr / cdt;
        smin = fmin(smin, s[q]);
        smax = fmax(smax, s[q]);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double* P = u + 3 + 3 * c;
            g[c][q] = -mu4pi * (S[0] * P[0] + S[1] * P[1] + S[2] * P[2]);
        }
    }
    const size_t row = (size_t)d * NC;
    const double z = far_zero(u);
    for (int tap = blockIdx.z; tap < ntap; tap += gridDim.z) {
        const double m = (double)(m_lo + tap);
        zd acc[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = zd{z, z};
        if (!(m + smax <= tb.lo() || m + smin > tb.hi())) {
#pragma unroll
            for (int q = 0; q < 14; ++q) {
                double T0, T1;
                if (!(BLIF ? far_blif(tb, m + s[q], T0, T1) : far_cppif(m + s[q], T0, T1))) continue;
                far_term<NC>(acc, g, q, T1 * idt, w * T0, cs[q], sn[q]);
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) F[((size_t)tap * nd * NC + row + c) * ns + k] = acc[c];
    }
}

// out[r][n] = sum_tap sum_kk A[r + sh (m_lo + tap)][kk] op(F)[tap][kk][n],
// r < M, kk < K, n < N; rows of A outside [0, M) are zero.
//   ADJ = false: A = I [M][K = ns], sh = -B, op(F)[tap][kk][n] = F[tap][n][kk]
//   ADJ = true:  A = W [M][K = ncol], sh = +B, op(F)[tap][kk][n] = conj(F[tap][kk][n])
// A block of four waves owns TR rows x TC columns: 64 x 64, a wave 32 x 32 as
// 2 x 2 complex tiles of v_mfma_f64_16x16x4 (four real products each); for up
// to 16 columns (8 directions, forward) 128 x 16, a wave 32 x 16, whose tiles of
// rows past M are left out.  The K loop runs over groups of 8 kk (outer) and
// taps (inner), so that the taps of a group read the same columns of A, shifted
// by B rows, from cache; a step's pieces of A and F go through LDS, the next
// step's loads in flight during its products (32 per wave, 16 of a narrow
// tile).  Bound by the matrix cores (66.6 TFLOP/s in a large FP64 product on
// this card).  The steps are split over nsplit blocks where the tiles alone
// would leave compute units idle (part[split] then, summed in order by the
// callers' kernels).  The running sums are added to a second set every kFlush
// steps, so that a chain of additions stays at 8 kFlush products.
// One block per output element with every thread on the same (r, n), each
// element reading all of F and I again: 100.9 ms for 640 rows, 64 directions
// and 43 taps of 7680 bases; this kernel 2 x 1.15 ms (27 taps), 49 TFLOP/s.
// One direction, 19200 rows of 480 bases: 255 us that way, 641 with 64 x 64,
// 233 with 128 x 16.
constexpr int kFarTile = 64, kFarNarrow = 16, kFarK = 8, kFlush = 64;
__host__ __device__ constexpr int far_rows(int tc) { return tc == kFarNarrow ? 128 : kFarTile; }

template <bool ADJ, int TC>
__global__ void __launch_bounds__(256, 2) k_far_gemm(const zd* __restrict__ A, const zd* __restrict__ F,
                                                     zd* __restrict__ out, int M, int N, int K, int ntap, int m_lo,
                                                     int B, int mt, int nt, int nsplit, int add) {
    constexpr int LD = kFarK + 1;  // odd row length in 16-byte units: lanes on consecutive rows spread over the banks
    constexpr int TR = far_rows(TC), NJ = TC == kFarNarrow ? 1 : 2, LA = TR / 32;
    static_assert(TC == kFarTile || (TC == kFarNarrow && !ADJ), "tile");
    __shared__ zd sA[2][TR * LD], sB[2][TC * LD];
    // row tiles fastest within one run of blocks per XCD (round-robin
    // dispatch): the blocks that read one piece of F share an L2
    const int per = gridDim.x / kXcds;
    const int lb = (int)(blockIdx.x % kXcds) * per + (int)(blockIdx.x / kXcds);
    if (lb >= mt * nt * nsplit) return;
    const int rt = lb % mt, ct = (lb / mt) % nt, sp = lb / (mt * nt);
    const int r0 = rt * TR, n0 = ct * TC;
    // taps that reach a row of the tile: r + shift in [0, M) for some r
    const int dir = ADJ ? 1 : -1;
    int t0 = 0, t1 = ntap;
    while (t0 < t1) {
        const long long s = (long long)dir * (m_lo + t0) * B;
        if (r0 + s < M && r0 + TR + s > 0) break;
        ++t0;
    }
    while (t1 > t0) {
        const long long s = (long long)dir * (m_lo + t1 - 1) * B;
        if (r0 + s < M && r0 + TR + s > 0) break;
        --t1;
    }
    const int nta = t1 - t0, nk = (K + kFarK - 1) / kFarK;
    const long long steps = (long long)nk * nta;
    const long long s0 = steps * sp / nsplit, s1 = steps * (sp + 1) / nsplit;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = (NJ == 1 ? wave : wave & 1) * 32, wc = NJ == 1 ? 0 : (wave >> 1) * 32;
    dx4 re[2][NJ], im[2][NJ], re2[2][NJ], im2[2][NJ];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) re[i][j] = im[i][j] = re2[i][j] = im2[i][j] = dx4{0, 0, 0, 0};
    zd ga[LA], gb[2];
    // the step being loaded: 8 kk from kk0, one tap
    int kk0 = nta > 0 ? (int)(s0 / nta) * kFarK : 0, tap = nta > 0 ? t0 + (int)(s0 % nta) : 0;
    auto load = [&]() {
        const long long sh = (long long)dir * (m_lo + tap) * B;
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int row = (tid >> 3) + 32 * i, kk = kk0 + (tid & 7);
            const long long r = r0 + row + sh;
            ga[i] = (r >= 0 && r < M && kk < K) ? A[(size_t)r * K + kk] : zd{0, 0};
        }
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            if constexpr (ADJ) {
                const int kf = kk0 + (tid >> 6) + 4 * i, n = n0 + lane;
                gb[i] = (kf < K && n < N) ? conjz(F[((size_t)tap * K + kf) * N + n]) : zd{0, 0};
            } else {
                const int row = (tid >> 3) + 32 * i, kk = kk0 + (tid & 7), n = n0 + row;
                gb[i] = (row < TC && n < N && kk < K) ? F[((size_t)tap * N + n) * K + kk] : zd{0, 0};
            }
        }
        if (++tap == t1) {
            tap = t0;
            kk0 += kFarK;
        }
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int i = 0; i < LA; ++i) sA[buf][((tid >> 3) + 32 * i) * LD + (tid & 7)] = ga[i];
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            if constexpr (ADJ)
                sB[buf][lane * LD + (tid >> 6) + 4 * i] = gb[i];
            else if (NJ == 2 || tid < 8 * TC)
                sB[buf][((tid >> 3) + 32 * i) * LD + (tid & 7)] = gb[i];
        }
    };
    if (s0 < s1) {
        load();
        put(0);
    }
    __syncthreads();
    int buf = 0, since = 0;
    for (long long s = s0; s < s1; ++s, buf ^= 1) {
        const bool more = s + 1 < s1;
        if (more) load();
#pragma unroll
        for (int h = 0; h < kFarK / 4; ++h) {
            // lane l holds row (column) l % 16 and kk = l / 16 of each 16 x 4 piece
            const int kk = 4 * h + (lane >> 4);
            zd a[2], b[NJ];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = sA[buf][(wr + 16 * i + (lane & 15)) * LD + kk];
#pragma unroll
            for (int i = 0; i < NJ; ++i) b[i] = sB[buf][(wc + 16 * i + (lane & 15)) * LD + kk];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (NJ == 1 && r0 + wr + 16 * i >= M) continue;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].x, re[i][j], 0, 0, 0);
                    im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].y, im[i][j], 0, 0, 0);
                    re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[i].y, b[j].y, re[i][j], 0, 0, 0);
                    im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].y, b[j].x, im[i][j], 0, 0, 0);
                }
            }
        }
        if (++since == kFlush) {
            since = 0;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    re2[i][j] += re[i][j];
                    im2[i][j] += im[i][j];
                    re[i][j] = im[i][j] = dx4{0, 0, 0, 0};
                }
        }
        // the other buffer was last read before the previous barrier
        if (more) put(buf ^ 1);
        __syncthreads();
    }
    zd* o = out + (size_t)sp * M * N;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                // element v of a lane: row 4 v + l / 16, column l % 16
                const int r = r0 + wr + 16 * i + 4 * v + (lane >> 4), n = n0 + wc + 16 * j + (lane & 15);
                if (r < M && n < N) {
                    zd& dst = o[(size_t)r * N + n];
                    const zd x{re2[i][j][v] + re[i][j][v], im2[i][j][v] + im[i][j][v]};
                    dst = add ? dst + x : x;
                }
            }
}

// sum over the splits of part[split][e], e < n: a block's 256 threads are 32
// elements x 8 groups of splits, each group summed in order, then the groups;
// the total in group 0's threads
__device__ __forceinline__ zd far_split_sum(const zd* __restrict__ part, size_t e, size_t n, int nsplit) {
    __shared__ zd sh[8][32];
    const int g = threadIdx.x >> 5, c = threadIdx.x & 31;
    zd a{0, 0};
    if (e < n)
        for (int s = g; s < nsplit; s += 8) a += part[(size_t)s * n + e];
    sh[g][c] = a;
    __syncthreads();
    if (g == 0)
        for (int i = 1; i < 8; ++i) a += sh[i][c];
    return a;
}

// part[0][e] = sum_split part[split][e]
__global__ void __launch_bounds__(256) k_far_reduce(zd* __restrict__ part, size_t n, int nsplit) {
    const size_t e = blockIdx.x * (size_t)32 + (threadIdx.x & 31);
    const zd a = far_split_sum(part, e, n, nsplit);
    if (threadIdx.x < 32 && e < n) part[e] = a;
}

// U[r][d0 + d][x] = sum_c Q[d][c][x] part[r][d nc + c]
__global__ void __launch_bounds__(256) k_far_expand(zd* __restrict__ U, const zd* __restrict__ part,
                                                    const double* __restrict__ q, int M, int nd, int nc, int ndt,
                                                    int d0) {
    const size_t tot = (size_t)M * nd;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < tot; e += (size_t)gridDim.x * blockDim.x) {
        const size_t r = e / nd;
        const int d = (int)(e - r * nd);
        zd o[3] = {{0, 0}, {0, 0}, {0, 0}};
        for (int c = 0; c < nc; ++c)
            for (int x = 0; x < 3; ++x) o[x] += q[9 * (size_t)d + 3 * c + x] * part[(r * nd + d) * nc + c];
        for (int x = 0; x < 3; ++x) U[(r * ndt + d0 + d) * 3 + x] = o[x];
    }
}

// W[r][d nc + c] = sum_x Q[d][c][x] U[r][d0 + d][x]
__global__ void __launch_bounds__(256) k_far_project(zd* __restrict__ W, const zd* __restrict__ U,
                                                     const double* __restrict__ q, int M, int nd, int nc, int ndt,
                                                     int d0) {
    const size_t tot = (size_t)M * nd * nc;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < tot; e += (size_t)gridDim.x * blockDim.x) {
        const size_t r = e / ((size_t)nd * nc);
        const int n = (int)(e - r * nd * nc), d = n / nc;
        zd a{0, 0};
        for (int x = 0; x < 3; ++x) a += q[9 * (size_t)d + 3 * (n - d * nc) + x] * U[(r * ndt + d0 + d) * 3 + x];
        W[e] = a;
    }
}

// S[e] = (or +=) sum_split part[split][e]
__global__ void __launch_bounds__(256) k_far_sum(zd* __restrict__ S, const zd* __restrict__ part, size_t n,
                                                 int nsplit, int add) {
    const size_t e = blockIdx.x * (size_t)32 + (threadIdx.x & 31);
    const zd a = far_split_sum(part, e, n, nsplit);
    if (threadIdx.x < 32 && e < n) S[e] = add ? S[e] + a : a;
}

}  // namespace etaim
