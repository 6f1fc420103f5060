// Matvec y/z stage for planes without a register engine of their own: one
// block per plane, lines of N = P Q points held by P lanes with Q registers
// each.
//
// A line's N-point DFT splits as n = p + P j, k = k1 + Q k2: lane p forms the
// Q-point DFT over j of its points in registers, the P lanes exchange through
// LDS, and each then forms Q / P DFTs of P points over p (P divides Q).  The
// inverse mirrors it.  The parity pre-twiddle of the zero-padded line
// w_{2N}^{parity n} = w_{2Q}^{parity j} w_{2N}^{parity p}: its first factor is
// a compile-time constant, the second joins the twiddle between the steps,
// w_{2N}^{p (2 k1 + parity)}.  The lanes of a line share a wave, so an
// exchange needs no block barrier.
//
// Per parity pz of kz: the z lines of the plane's columns (read from memory,
// consecutive columns on consecutive lanes) go into an LDS tile [kz'][y]; the
// rows take, per parity py, the forward DFT, the Green product and the inverse
// DFT, summed over py into the tile; the inverse z lines add to the result,
// which is stored in place at the end.  The plane is read and written once;
// the tiles of both pz (and the twiddles) are all the LDS a block needs: N = 96
// in FP32 takes 157 KB, one block per CU.  Bound by FP32 (FP64) issue and, for
// small planes, by latency.
#pragma once
#include "aim.inc.hip"

namespace etaim {

// LDS row length of a line of N points held by P lanes: an offset of P (or
// an odd length) spreads the rows of a wave over the banks
__host__ __device__ constexpr int plane_ld(int N, int P) { return N + (P == 3 ? 1 : P); }

template <typename R, int NY, int PY, int NZ>
__host__ __device__ constexpr size_t plane_tile() {
    return (size_t)NZ * plane_ld(NY, PY) * sizeof(cplx<R>);
}
// both parities' tiles are in the LDS at once; the threads double and each half
// takes one pz (half), so that a block holds twice the waves and no partial
// result waits in registers.  On flat planes, whose rows occupy a wave either
// way, each thread takes its column for one pz after the other (48x8 in FP64:
// 50 us for 8 columns, 59 with halves; the cubes 10 to 30 % faster with halves
// at one column, equal at eight)
template <typename R, int NY, int PY, int NZ>
__host__ __device__ constexpr bool plane_half() {
    return NZ > 8 || 2 * plane_tile<R, NY, PY, NZ>() > 72 * 1024;
}
// threads: a lane for every (column, p) of the z lines, whole waves
template <typename R, int NY, int PY, int NZ, int PZ>
__host__ __device__ constexpr int plane_threads() {
    return (NY + 64 / PZ - 1) / (64 / PZ) * 64 * (plane_half<R, NY, PY, NZ>() ? 2 : 1);
}
template <typename R, int NY, int PY, int NZ>
__host__ __device__ constexpr size_t plane_lds_bytes() {
    return 2 * plane_tile<R, NY, PY, NZ>() + (size_t)(2 * NY + 2 * NZ) * sizeof(cplx<R>);
}

// the twiddles between the steps, [par][p][k1], from w_{2N}^n: a lane reads
// its Q values as one run
template <typename R, int P, int Q>
__device__ __forceinline__ void mline_table(cplx<R>* tab, const cplx<R>* __restrict__ w) {
    for (int i = threadIdx.x; i < 2 * P * Q; i += blockDim.x) {
        const int k1 = i % Q, r = i / Q;
        tab[i] = w[(r % P) * (2 * k1 + r / P)];
    }
}

// forward: u[j] = x[p + P j] -> u[i P + k2] = X[(p + P i) + Q k2], i < Q / P;
// the exchange through row[e st], e < N; tw[k1] = w_{2N}^{p (2 k1 + par)}, this
// lane's and parity's run of the block's table (mline_table)
template <typename R, int P, int Q>
__device__ __forceinline__ void mline_fwd(cplx<R> (&u)[Q], int p, int par, cplx<R>* row, int st,
                                          const cplx<R>* tw, bool live) {
    if (par) {
#pragma unroll
        for (int j = 1; j < Q; ++j) u[j] = twn_mul<R, 2 * Q>(u[j], j, false);
    }
    dft_small<R, Q>(u, false);
    if (live) {
#pragma unroll
        for (int k1 = 0; k1 < Q; ++k1) row[(k1 * P + p) * st] = cmul_fma(u[k1], tw[k1]);
    }
    wave_sync();
    if (live) {
#pragma unroll
        for (int i = 0; i < Q / P; ++i)
#pragma unroll
            for (int q = 0; q < P; ++q) u[i * P + q] = row[((p + P * i) * P + q) * st];
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < Q / P; ++i) {
        cplx<R> v[P];
#pragma unroll
        for (int q = 0; q < P; ++q) v[q] = u[i * P + q];
        dft_small<R, P>(v, false);
#pragma unroll
        for (int q = 0; q < P; ++q) u[i * P + q] = v[q];
    }
}

// inverse of mline_fwd (unnormalised), the parity's conjugate post-twiddle included
template <typename R, int P, int Q>
__device__ __forceinline__ void mline_inv(cplx<R> (&u)[Q], int p, int par, cplx<R>* row, int st,
                                          const cplx<R>* tw, bool live) {
#pragma unroll
    for (int i = 0; i < Q / P; ++i) {
        cplx<R> v[P];
#pragma unroll
        for (int q = 0; q < P; ++q) v[q] = u[i * P + q];
        dft_small<R, P>(v, true);
#pragma unroll
        for (int q = 0; q < P; ++q) u[i * P + q] = v[q];
    }
    if (live) {
#pragma unroll
        for (int i = 0; i < Q / P; ++i)
#pragma unroll
            for (int q = 0; q < P; ++q) row[((p + P * i) * P + q) * st] = u[i * P + q];
    }
    wave_sync();
    if (live) {
#pragma unroll
        for (int k1 = 0; k1 < Q; ++k1) u[k1] = cmul_fma(row[(k1 * P + p) * st], conjz(tw[k1]));
    }
    wave_sync();
    dft_small<R, Q>(u, true);
    if (par) {
#pragma unroll
        for (int j = 1; j < Q; ++j) u[j] = twn_mul<R, 2 * Q>(u[j], j, true);
    }
}

// In place on A[bc][kx][z < NZ][y < NY]; GT: the folded Green spectra of one m
// with ky and kz exchanged, [t][kx][ky fold][kz fold].  Grid (4B, L_x), bc
// fastest (the blocks of one XCD share the Green plane of their kx).
// waves per SIMD the registers are capped for: what the LDS of the blocks on
// a CU allows, up to four (FP32) or two (FP64)
template <typename R, int NY, int PY, int NZ, int PZ>
__host__ __device__ constexpr int plane_waves() {
    const int blocks = (int)(160 * 1024 / plane_lds_bytes<R, NY, PY, NZ>());
    const int w = blocks * plane_threads<R, NY, PY, NZ, PZ>() / 256, cap = sizeof(R) == 4 ? (NY >= 54 ? 3 : 4) : 2;
    return w < 1 ? 1 : w < cap ? w : cap;
}
template <typename R, int NY, int PY, int NZ, int PZ>
__global__ void __launch_bounds__((plane_threads<R, NY, PY, NZ, PZ>()))
__attribute__((amdgpu_waves_per_eu(plane_waves<R, NY, PY, NZ, PZ>()))) k_plane_green(cplx<R>* __restrict__ A,
                                                                          const cplx<R>* __restrict__ GT,
                                                                          const cplx<R>* __restrict__ twy_g,
                                                                          const cplx<R>* __restrict__ twz_g,
                                                                          GridDims g, int conj_g,
                                                                          const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    constexpr int QY = NY / PY, QZ = NZ / PZ, LD = plane_ld(NY, PY);
    constexpr int T = plane_threads<R, NY, PY, NZ, PZ>(), CW = 64 / PZ, RW = 64 / PY;
    static_assert(QY * PY == NY && QZ * PZ == NZ && QY % PY == 0 && QZ % PZ == 0, "line split");
    static_assert(plane_lds_bytes<R, NY, PY, NZ>() <= 160 * 1024, "the tiles of both parities fit the LDS");
    extern __shared__ unsigned char smem_raw[];
    cplx<R>* tile = reinterpret_cast<cplx<R>*>(smem_raw);
    cplx<R>* twy = tile + (size_t)2 * NZ * LD;
    cplx<R>* twz = twy + 2 * NY;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    mline_table<R, PY, QY>(twy, twy_g);
    mline_table<R, PZ, QZ>(twz, twz_g);
    const int bc = blockIdx.x, kx = blockIdx.y, Lx = g.L[0];
    cplx<R>* pl = A + ((size_t)bc * Lx + kx) * (size_t)(NZ * NY);
    const cplx<R>* Gk = GT + ((size_t)((bc & 3) == 3 ? 1 : 0) * (g.N[0] + 1) + fold(kx, Lx)) * (size_t)((NY + 1) * (NZ + 1));
    // z lines: column y, consecutive columns on consecutive lanes
    constexpr bool HALF = plane_half<R, NY, PY, NZ>();
    constexpr int ZW = HALF ? T / 128 : T / 64;  // waves of the columns
    const int hz = HALF ? wave / ZW : 0;
    const int zp = lane / CW, y = (wave - hz * ZW) * CW + lane % CW;
    const bool zlive = zp < PZ && y < NY;
    cplx<R> acc[QZ];
#pragma unroll
    for (int j = 0; j < QZ; ++j) acc[j] = cplx<R>{0, 0};
    // short lines: read once and kept for the other parity
    constexpr bool KEEP = QZ <= 12 && !HALF;
    cplx<R> in[KEEP ? QZ : 1];
    if constexpr (KEEP) {
#pragma unroll
        for (int j = 0; j < QZ; ++j) in[j] = zlive ? pl[(zp + PZ * j) * NY + y] : cplx<R>{0, 0};
    }
    __syncthreads();
#pragma unroll 1
    for (int pz = hz; pz < (HALF ? hz + 1 : 2); ++pz) {
        cplx<R> u[QZ];
#pragma unroll
        for (int j = 0; j < QZ; ++j) u[j] = KEEP ? in[KEEP ? j : 0] : zlive ? pl[(zp + PZ * j) * NY + y] : cplx<R>{0, 0};
        cplx<R>* col = tile + (size_t)pz * NZ * LD + y;
        mline_fwd<R, PZ, QZ>(u, zp, pz, col, LD, twz + (pz * PZ + (zlive ? zp : 0)) * QZ, zlive);
        if (zlive) {
#pragma unroll
            for (int i = 0; i < QZ / PZ; ++i)
#pragma unroll
                for (int q = 0; q < PZ; ++q) col[(zp + PZ * i + QZ * q) * LD] = u[i * PZ + q];
        }
    }
    __syncthreads();
    // rows kz' of the tiles: RW rows per wave, their PY lanes adjacent
    constexpr int ROUNDS = (2 * NZ + RW - 1) / RW;
    for (int rd = wave; rd < ROUNDS; rd += T / 64) {
        const int p = lane % PY, row = rd * RW + lane / PY;
        const bool live = lane < RW * PY && row < 2 * NZ;
        const int pz = row >= NZ ? 1 : 0, kz = row - pz * NZ;
        const int zf = live ? fold(2 * kz + pz, 2 * NZ) : 0;
        cplx<R>* rp = tile + (size_t)(live ? row : 0) * LD;
        const unsigned up = (unsigned)(2 * p * (NZ + 1) + zf), down = (unsigned)(2 * (PY - 1 - p) * (NZ + 1) + zf);
        // row x times w_{2N}^{py y}: DFT, Green product, inverse DFT, post-twiddle
        auto pass = [&](cplx<R>(&x)[QY], int py) {
            // ky = 2 c + py of c = c0 + p: a group of PY lanes lies on one side of
            // the fold at c = N_y / 2 (PY divides it), so that its address is a
            // uniform row plus the lane's offset up or down
            auto green = [&](int c0) -> cplx<R> {
                if constexpr (NY % (2 * PY) != 0)
                    return Gk[fold(2 * (c0 + p) + py, 2 * NY) * (NZ + 1) + zf];
                else if (2 * c0 < NY)
                    return (Gk + (2 * c0 + py) * (NZ + 1))[up];
                else
                    return (Gk + (2 * NY - 2 * (c0 + PY - 1) - py) * (NZ + 1))[down];
            };
            // short lines: the Green values wait in registers
            constexpr bool AHEAD = QY <= 12;
            cplx<R> gr[AHEAD ? QY : 1];
            if constexpr (AHEAD) {
#pragma unroll
                for (int i = 0; i < QY; ++i) gr[i] = green(PY * (i / PY) + QY * (i % PY));
            }
            mline_fwd<R, PY, QY>(x, p, py, rp, 1, twy + (py * PY + p) * QY, live);
#pragma unroll
            for (int i = 0; i < QY; ++i) {
                cplx<R> gv = AHEAD ? gr[AHEAD ? i : 0] : green(PY * (i / PY) + QY * (i % PY));
                if (conj_g) gv.y = -gv.y;
                x[i] = cmul_fma(x[i], gv);
            }
            mline_inv<R, PY, QY>(x, p, py, rp, 1, twy + (py * PY + p) * QY, live);
        };
        // py = 1 on a copy of the row (its LDS is the exchange's space),
        // then py = 0, one after the other in the registers
        cplx<R> u[QY], v[QY];
#pragma unroll
        for (int j = 0; j < QY; ++j) v[j] = u[j] = live ? rp[p + PY * j] : cplx<R>{0, 0};
        wave_sync();
        pass(v, 1);
        __builtin_amdgcn_sched_barrier(0);
        pass(u, 0);
#pragma unroll
        for (int j = 0; j < QY; ++j) v[j] += u[j];
        if (live) {
#pragma unroll
            for (int j = 0; j < QY; ++j) rp[p + PY * j] = v[j];
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int pz = hz; pz < (HALF ? hz + 1 : 2); ++pz) {
        cplx<R> u[QZ];
        cplx<R>* col = tile + (size_t)pz * NZ * LD + y;
#pragma unroll
        for (int i = 0; i < QZ / PZ; ++i)
#pragma unroll
            for (int q = 0; q < PZ; ++q) u[i * PZ + q] = zlive ? col[(zp + PZ * i + QZ * q) * LD] : cplx<R>{0, 0};
        wave_sync();
        mline_inv<R, PZ, QZ>(u, zp, pz, col, LD, twz + (pz * PZ + (zlive ? zp : 0)) * QZ, zlive);
#pragma unroll
        for (int j = 0; j < QZ; ++j) acc[j] = HALF ? u[j] : acc[j] + u[j];
    }
    if constexpr (HALF) {
        // pz = 1's half hands its columns over in its own tile
        cplx<R>* col = tile + (size_t)NZ * LD + y;
        if (hz == 1 && zlive) {
#pragma unroll
            for (int j = 0; j < QZ; ++j) col[(zp + PZ * j) * LD] = acc[j];
        }
        __syncthreads();
        if (hz == 1) return;
        if (zlive) {
#pragma unroll
            for (int j = 0; j < QZ; ++j) acc[j] += col[(zp + PZ * j) * LD];
        }
    }
    if (zlive) {
#pragma unroll
        for (int j = 0; j < QZ; ++j) pl[(zp + PZ * j) * NY + y] = acc[j];
    }
}

// The planes with an instance, (N_y, lanes per row, N_z, lanes per column),
// for both precisions and for FP32 alone, where the kernel measured faster
// than the passes it replaces.  y/z stage in us, this kernel / the LDS plane
// or line passes (FP32; FP64), for the columns in brackets:
//   18 (8)  13 / 61; 19 / 70      27 (8)  29 / 130; 51 / 151    32 (8)  40 / 120; 78 / 144
//   36 (8)  50 / 146; 93 / 182    54 (8) 192 / 443; 375 / 1587  64 (8) 287 / 469; 642 / 2352
//   96 (3) 377 / 702; 1393 / 1230 (FP32 only: in FP64 the tile leaves 6 waves on a CU and the lines spill)
//   16x8 (8) 8 / 46; 14 / 51      24x8 (8) 12 / 62; 22 / 69     48x8 (8) 26 / 125; 48 / 137
//   96x8 (4) 74 / 142; 213 / 161 (FP32 only)
//   72 (4), with 3 or 6 lanes per line: 236 / 241; 444 / 449: no instance, line passes
// 64 with 8 lanes per line: 396; 947.  36 with 3: 54; 106.
#define ETAIM_PLANES(X)                                                                                       \
    X(18, 3, 18, 3) X(27, 3, 27, 3) X(32, 4, 32, 4) X(36, 6, 36, 6) X(54, 3, 54, 3) X(64, 4, 64, 4) X(16, 4, 8, 2) \
    X(24, 2, 8, 2) X(48, 4, 8, 2)
#define ETAIM_PLANES32(X) X(96, 4, 96, 4) X(96, 4, 8, 2)

}  // namespace etaim
