// FP64 kernels of right-preconditioned restarted GMRES (Sec. 5.1: diagonally
// preconditioned GMRES), one Krylov space per excitation column b.
// Vectors are [B][ns] complex128; the basis is [restart+1][B][ns].
#pragma once
#include "common.hpp"

namespace etaim {

__device__ __forceinline__ double block_sum256(double v, double* sh) {
    // deterministic tree over a 256-thread block
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// Block of the column reductions: 1024 threads, so that the few blocks of
// a reduction (one per column) keep enough loads in flight
constexpr int kRedThreads = 1024;

template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// sum over a wave by the butterfly over lane distances 32, 16, 8, 4, 2, 1,
// with register moves between lanes (half and quarter swaps, rotations of
// rows of 16, quad permutations) instead of LDS permutes
__device__ __forceinline__ double wave_total(double v) {
    {
        const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
        v = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    }
    {
        const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
        v = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    }
    v += dpp_mov<0x128>(v);  // row rotated by 8
    v += dpp_mov<0x124>(v);  // by 4
    v += dpp_mov<0x4e>(v);   // quad lanes 2 3 0 1
    v += dpp_mov<0xb1>(v);   // 1 0 3 2
    return v;
}

// The sums over a wave of NV values (a power of two up to 16), each by the
// same butterfly as wave_total: at the first log2(NV) distances a lane pair
// exchanges one value for another and each keeps half of them, so that all
// NV take little more than twice one value's work.  Lane l then holds the
// sum of value l / (64 / NV).
// the value of lane l ^ 4: rows rotated left by 4 in the quads that need the
// next one, right by 4 in the others
__device__ __forceinline__ double lane_xor4(double v) {
    int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x12c, 0xf, 0x5, false);
    int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x12c, 0xf, 0x5, false);
    lo = __builtin_amdgcn_update_dpp(lo, __double2loint(v), 0x124, 0xf, 0xa, false);
    hi = __builtin_amdgcn_update_dpp(hi, __double2hiint(v), 0x124, 0xf, 0xa, false);
    return __hiloint2double(hi, lo);
}
template <int NV>
__device__ __forceinline__ double wave_totals(double (&t)[NV], int lane) {
    auto swap32 = [](double a, double b) {
        const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
        return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    };
    auto swap16 = [](double a, double b) {
        const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
        return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    };
    constexpr int H1 = NV / 2, H2 = NV / 4, H3 = NV / 8, H4 = NV / 16;
    // (a value swapped with itself: the plain butterfly step)
#pragma unroll
    for (int i = 0; i < (H1 ? H1 : 1); ++i) t[i] = swap32(t[i], t[H1 ? i + H1 : i]);
#pragma unroll
    for (int i = 0; i < (H2 ? H2 : 1); ++i) t[i] = swap16(t[i], t[H2 ? i + H2 : i]);
#pragma unroll
    for (int i = 0; i < (H3 ? H3 : 1); ++i) {
        const bool up = H3 && (lane & 8) != 0;
        const double o = t[H3 ? i + H3 : i];
        t[i] = (up ? o : t[i]) + dpp_mov<0x128>(up ? t[i] : o);
    }
    {
        const bool up = H4 && (lane & 4) != 0;
        const double o = t[H4 ? 1 : 0];
        t[0] = (up ? o : t[0]) + lane_xor4(up ? t[0] : o);
    }
    t[0] += dpp_mov<0x4e>(t[0]);
    t[0] += dpp_mov<0xb1>(t[0]);
    return t[0];
}

// deterministic sum over a kRedThreads block, valid in thread 0: a fixed
// butterfly within each wave, then the wave sums in order
__device__ __forceinline__ double block_sum_t0(double v, double* sh) {
    v = wave_total(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = 0;
    if (threadIdx.x == 0)
        for (int q = 0; q < kRedThreads / 64; ++q) r += sh[q];
    return r;
}

// h[i][b] = <V_i[b], w[b]> = sum_k conj(V_i[b][k]) w[b][k], i < nv.  grid (nv, B)
__global__ void __launch_bounds__(kRedThreads) k_dots(const zd* __restrict__ V, const zd* __restrict__ w,
                                                      zd* __restrict__ h, int ns, int B,
                                                      const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    __shared__ double sh[2][kRedThreads / 64];
    const int i = blockIdx.x, b = blockIdx.y;
    const zd* v = V + ((size_t)i * B + b) * ns;
    const zd* x = w + (size_t)b * ns;
    double re = 0, im = 0;
    for (int k = threadIdx.x; k < ns; k += kRedThreads) {
        const zd a = v[k], c = x[k];
        re += a.x * c.x + a.y * c.y;
        im += a.x * c.y - a.y * c.x;
    }
    re = block_sum_t0(re, sh[0]);
    im = block_sum_t0(im, sh[1]);
    if (threadIdx.x == 0) h[(size_t)i * B + b] = zd{re, im};
}

// The same dot products over long columns, split over nchunk blocks per
// (i, b): each block sums one contiguous chunk (part[(i B + b) nchunk + c]),
// then k_dots_fin adds the chunks in order (deterministic, no atomics).
__global__ void __launch_bounds__(kRedThreads) k_dots_part(const zd* __restrict__ V, const zd* __restrict__ w,
                                                           zd* __restrict__ part, int ns, int B, int nchunk,
                                                           const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    __shared__ double sh[2][kRedThreads / 64];
    const int i = blockIdx.x, b = blockIdx.y, ch = blockIdx.z;
    const int len = (ns + nchunk - 1) / nchunk, k0 = ch * len, k1 = min(ns, k0 + len);
    const zd* v = V + ((size_t)i * B + b) * ns;
    const zd* x = w + (size_t)b * ns;
    double re = 0, im = 0;
    for (int k = k0 + threadIdx.x; k < k1; k += kRedThreads) {
        const zd a = v[k], c = x[k];
        re += a.x * c.x + a.y * c.y;
        im += a.x * c.y - a.y * c.x;
    }
    re = block_sum_t0(re, sh[0]);
    im = block_sum_t0(im, sh[1]);
    if (threadIdx.x == 0) part[((size_t)i * B + b) * nchunk + ch] = zd{re, im};
}
// h[e] = sum_c part[e nchunk + c], e < n
__global__ void k_dots_fin(const zd* __restrict__ part, zd* __restrict__ h, int n, int nchunk,
                           const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    zd acc{0, 0};
    for (int ch = 0; ch < nchunk; ++ch) acc += part[(size_t)e * nchunk + ch];
    h[e] = acc;
}
// nrm[b] = ||w[b]|| over nchunk chunks per column (sum of squares in part,
// finished by k_norm_fin)
__global__ void __launch_bounds__(kRedThreads) k_norm_part(const zd* __restrict__ w, double* __restrict__ part,
                                                           int ns, int nchunk, const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    __shared__ double sh[kRedThreads / 64];
    const int b = blockIdx.x, ch = blockIdx.y;
    const int len = (ns + nchunk - 1) / nchunk, k0 = ch * len, k1 = min(ns, k0 + len);
    const zd* x = w + (size_t)b * ns;
    double s = 0;
    for (int k = k0 + threadIdx.x; k < k1; k += kRedThreads) s += x[k].x * x[k].x + x[k].y * x[k].y;
    s = block_sum_t0(s, sh);
    if (threadIdx.x == 0) part[(size_t)b * nchunk + ch] = s;
}
__global__ void k_norm_fin(const double* __restrict__ part, double* __restrict__ nrm, int B, int nchunk,
                           const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    double s = 0;
    for (int ch = 0; ch < nchunk; ++ch) s += part[(size_t)b * nchunk + ch];
    nrm[b] = sqrt(s);
}

// w[b] -= sum_{i<nv} h[i][b] V_i[b]  (one classical Gram-Schmidt pass)
__global__ void __launch_bounds__(256) k_orth(const zd* __restrict__ V, zd* __restrict__ w, const zd* __restrict__ h,
                                              int nv, int ns, int B, const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    const int b = blockIdx.y;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= ns) return;
    zd acc = w[(size_t)b * ns + k];
    for (int i = 0; i < nv; ++i) acc -= h[(size_t)i * B + b] * V[((size_t)i * B + b) * ns + k];
    w[(size_t)b * ns + k] = acc;
}

// nrm[b] = ||w[b]||  (kRedThreads per block)
__global__ void __launch_bounds__(kRedThreads) k_norm(const zd* __restrict__ w, double* __restrict__ nrm, int ns,
                                                      const int* __restrict__ gate = nullptr, StepRef sr = {}) {
    if (gated_off(gate) || step_off(sr)) return;
    // replayed step: its row of the call's per-step norms [steps][B]
    if (const StepDesc* d = step_of(sr)) nrm = d->nrm + (size_t)d->i * gridDim.x;
    __shared__ double sh[kRedThreads / 64];
    const int b = blockIdx.x;
    const zd* x = w + (size_t)b * ns;
    double s = 0;
    for (int k = threadIdx.x; k < ns; k += kRedThreads) s += x[k].x * x[k].x + x[k].y * x[k].y;
    s = block_sum_t0(s, sh);
    if (threadIdx.x == 0) nrm[b] = sqrt(s);
}

// out[b] = w[b] / nrm[b] (0 if nrm == 0)
__global__ void k_scale(const zd* __restrict__ w, const double* __restrict__ nrm, zd* __restrict__ out, int ns,
                        int B, const int* __restrict__ gate = nullptr) {
    if (gated_off(gate)) return;
    const size_t tot = (size_t)ns * B;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < tot; e += (size_t)gridDim.x * blockDim.x) {
        const int b = (int)(e / ns);
        const double n = nrm[b];
        const double s = n > 0 ? 1.0 / n : 0.0;
        out[e] = zd{w[e].x * s, w[e].y * s};
    }
}

// r = rhs - r  (r holds A x on entry)
__global__ void k_residual(const zd* __restrict__ rhs, zd* __restrict__ r, size_t n,
                           const int* __restrict__ gate = nullptr) {
    if (gated_off(gate)) return;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x)
        r[e] = rhs[e] - r[e];
}

// The iteration's flags: {active columns, non-finite, the next Arnoldi step
// is live, steps taken this cycle, step budget, -, column count (64 bits)}.
// A step is live while a column is active, nothing went non-finite and the
// budget lasts (and, in a whole-step graph, the step is).
constexpr int kFlags = 8;

// Counts a column done, with its state, in the flags' column count: the
// columns in the low 24 bits, the active ones from bit 24, the non-finite
// ones from bit 48, all in one atomic word, so that no fence is needed (a
// device-wide fence writes back the L2).  True in the last of the B columns,
// whose cnt and bad then hold the sums; the count is zero on entry and left
// zero.
__device__ __forceinline__ bool last_column(int* __restrict__ flag, int on, int bad_in, int B, int& cnt, int& bad) {
    cnt = on;
    bad = bad_in;
    if (B == 1) return true;
    unsigned long long* word = reinterpret_cast<unsigned long long*>(flag + 6);
    const unsigned long long mine = 1ull | (unsigned long long)on << 24 | (unsigned long long)bad_in << 48;
    const unsigned long long old = atomicAdd(word, mine), tot = old + mine;
    if ((int)(tot & 0xffffff) != B) return false;
    *word = 0;
    cnt = (int)((tot >> 24) & 0xffffff);
    bad = tot >> 48 ? 1 : 0;
    return true;
}

// Start of a column's cycle: beta = ||r||; active iff beta > tol * bnorm.
// g[b] = (beta, 0, ...), jcnt = 0.  Returns {active, finite}.
__device__ __forceinline__ int2 start_column(double be, double bn, int* __restrict__ active, int* __restrict__ jcnt,
                                             zd* __restrict__ g, double* __restrict__ resid, int b, int ldg,
                                             double tol) {
    const bool fin = isfinite(be);
    const int a = (fin && be > tol * bn) ? 1 : 0;
    active[b] = a;
    jcnt[b] = 0;
    resid[b] = bn > 0 ? be / bn : 0.0;
    for (int i = 0; i < ldg; ++i) g[(size_t)b * ldg + i] = zd{0, 0};
    g[(size_t)b * ldg] = zd{be, 0};
    return int2{a, fin ? 1 : 0};
}

// Start of a cycle for every column, and its flags.  One block, one thread
// per column (strided).
__global__ void __launch_bounds__(256) k_cycle_start(const double* __restrict__ beta, const double* __restrict__ bnorm,
                                                     int* __restrict__ active, int* __restrict__ jcnt,
                                                     zd* __restrict__ g, double* __restrict__ resid,
                                                     int* __restrict__ flag, int B, int ldg, double tol, int budget,
                                                     const int* __restrict__ gate = nullptr) {
    if (gated_off(gate)) {
        if (threadIdx.x == 0) flag[2] = 0;
        return;
    }
    __shared__ int cnt, bad;
    if (threadIdx.x == 0) cnt = bad = 0;
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += blockDim.x) {
        const int2 r = start_column(beta[b], bnorm[b], active, jcnt, g, resid, b, ldg, tol);
        if (r.x) atomicAdd(&cnt, 1);
        if (!r.y) atomicOr(&bad, 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        flag[0] = cnt;
        flag[1] = bad;
        flag[2] = cnt > 0 && !bad && budget > 0 ? 1 : 0;
        flag[3] = 0;
        flag[4] = budget;
    }
}

// The same from the step's right-hand side and w = A x, for columns that one
// block holds: r = rhs - w (stored in w), ||rhs||, ||r||, the cycle start and
// the first basis vector r / ||r||, in one launch instead of seven of a few
// microseconds each.  bnorm is formed where first != 0.  The column that
// ends last sets the flags.
__global__ void __launch_bounds__(kRedThreads) k_cycle_begin(const zd* __restrict__ rhs, zd* __restrict__ w,
                                                             zd* __restrict__ V, double* __restrict__ beta,
                                                             double* __restrict__ bnorm, int* __restrict__ active,
                                                             int* __restrict__ jcnt, zd* __restrict__ g,
                                                             double* __restrict__ resid, int* __restrict__ flag, int ns,
                                                             int B, int ldg, double tol, int budget, int first,
                                                             const int* __restrict__ gate = nullptr) {
    if (gated_off(gate)) {
        if (threadIdx.x == 0 && blockIdx.x == 0) flag[2] = 0;
        return;
    }
    __shared__ double sh[2][kRedThreads / 64], be_s;
    const int b = blockIdx.x;
    const zd* rb = rhs + (size_t)b * ns;
    zd* wb = w + (size_t)b * ns;
    double sb = 0, sr = 0;
    for (int k = threadIdx.x; k < ns; k += kRedThreads) {
        const zd v = rb[k], r = v - wb[k];
        wb[k] = r;
        sb += v.x * v.x + v.y * v.y;
        sr += r.x * r.x + r.y * r.y;
    }
    if (first) sb = block_sum_t0(sb, sh[0]);
    sr = block_sum_t0(sr, sh[1]);
    if (threadIdx.x == 0) be_s = sqrt(sr);
    __syncthreads();
    const double be = be_s, sc = be > 0 ? 1.0 / be : 0.0;
    zd* vb = V + (size_t)b * ns;
    for (int k = threadIdx.x; k < ns; k += kRedThreads) vb[k] = zd{wb[k].x * sc, wb[k].y * sc};
    if (threadIdx.x != 0) return;
    if (first) bnorm[b] = sqrt(sb);
    beta[b] = be;
    const int2 r = start_column(be, first ? sqrt(sb) : bnorm[b], active, jcnt, g, resid, b, ldg, tol);
    int cnt, bad;
    if (!last_column(flag, r.x, !r.y, B, cnt, bad)) return;
    flag[0] = cnt;
    flag[1] = bad;
    flag[2] = cnt > 0 && !bad && budget > 0 ? 1 : 0;
    flag[3] = 0;
    flag[4] = budget;
}

// Arnoldi column j of column b, from its Hessenberg entries col[0..j] (the
// two classical Gram-Schmidt passes added) and h_{j+1,j} = nrm: previous
// Givens rotations c, s, a new rotation, residual estimate |g_{j+1}|.  One
// thread; col[0..j+1], c and s are copies the block holds in LDS.  Returns
// {active, finite}.
__device__ __forceinline__ int2 givens_column(zd* col, double* c, zd* s, double nrm, zd* __restrict__ g,
                                              int* __restrict__ active, int* __restrict__ jcnt,
                                              double* __restrict__ resid, double bn, int j, int b, int restart,
                                              double tol) {
    zd a = col[0];
    for (int i = 0; i < j; ++i) {
        const zd bb = col[i + 1];
        col[i] = c[i] * a + s[i] * bb;
        a = c[i] * bb - conjz(s[i]) * a;
    }
    const double aa = sqrt(a.x * a.x + a.y * a.y);
    const double r = sqrt(aa * aa + nrm * nrm);
    double cj;
    zd sj;
    if (aa == 0.0) {
        cj = 0.0;
        sj = zd{1.0, 0.0};
    } else {
        cj = aa / r;
        sj = zd{a.x / aa * nrm / r, a.y / aa * nrm / r};
    }
    c[j] = cj;
    s[j] = sj;
    col[j] = cj * a + sj * zd{nrm, 0};
    col[j + 1] = zd{0, 0};
    zd* gb = g + (size_t)b * (restart + 1);
    const zd gj = gb[j];
    gb[j] = cj * gj;
    const zd gn = zd{0, 0} - conjz(sj) * gj;
    gb[j + 1] = gn;
    const double est = sqrt(gn.x * gn.x + gn.y * gn.y);
    resid[b] = bn > 0 ? est / bn : 0.0;
    jcnt[b] = j + 1;
    const bool fin = isfinite(est);
    const int on = fin && !(est <= tol * bn || nrm == 0.0 || j + 1 == restart) ? 1 : 0;
    active[b] = on;
    return int2{on, fin ? 1 : 0};
}

// A column's end of an Arnoldi step (one thread): the column that ends last
// sets the flags and the next step's gate.  A non-finite column is sticky
// until the next cycle start.
__device__ __forceinline__ void step_done(int* __restrict__ flag, int on, int bad_in, int B, bool gated,
                                          const int* __restrict__ step_live) {
    int cnt, bad;
    if (!last_column(flag, on, bad_in, B, cnt, bad)) return;
    const int nf = flag[1] | bad;
    flag[0] = cnt;
    flag[1] = nf;
    if (!gated) return;
    const int left = flag[4] - 1;
    flag[3] += 1;
    flag[4] = left;
    flag[2] = (cnt > 0 && nf == 0 && left > 0 && (step_live == nullptr || *step_live != 0)) ? 1 : 0;
}

// Last part of Arnoldi step j, one block per column: norm of w, the next
// basis vector w / norm, Hessenberg column and Givens update, flags.  With
// nrm given, the norm is formed and the vector scaled beforehand (columns
// longer than a block should run over).
__global__ void __launch_bounds__(kRedThreads) k_arnoldi_tail(const zd* __restrict__ w, zd* __restrict__ vn,
                                                              const zd* __restrict__ h1, const zd* __restrict__ h2,
                                                              const double* __restrict__ nrm, zd* __restrict__ H,
                                                              double* __restrict__ cs, zd* __restrict__ sn,
                                                              zd* __restrict__ g, int* __restrict__ active,
                                                              int* __restrict__ jcnt, double* __restrict__ resid,
                                                              const double* __restrict__ bnorm, int* __restrict__ flag,
                                                              int ns, int j, int B, int restart, double tol,
                                                              const int* __restrict__ gate,
                                                              const int* __restrict__ step_live) {
    if (gated_off(gate)) return;
    extern __shared__ unsigned char smem_raw[];
    zd* col = reinterpret_cast<zd*>(smem_raw);  // [j + 2]
    zd* s = col + j + 2;                        // [j + 1]
    double* c = reinterpret_cast<double*>(s + j + 1);  // [j + 1]
    __shared__ double sh[kRedThreads / 64], n_s;
    const int b = blockIdx.x, tid = threadIdx.x;
    const int was = active[b];
    int2 r{0, 1};
    if (was) {
        for (int i = tid; i <= j; i += kRedThreads) col[i] = h1[(size_t)i * B + b] + h2[(size_t)i * B + b];
        for (int i = tid; i < j; i += kRedThreads) {
            c[i] = cs[(size_t)b * restart + i];
            s[i] = sn[(size_t)b * restart + i];
        }
        if (nrm) {
            if (tid == 0) n_s = nrm[b];
            __syncthreads();
        } else {
            const zd* x = w + (size_t)b * ns;
            double t = 0;
            for (int k = tid; k < ns; k += kRedThreads) t += x[k].x * x[k].x + x[k].y * x[k].y;
            t = block_sum_t0(t, sh);
            if (tid == 0) n_s = sqrt(t);
            __syncthreads();
            const double n = n_s, f = n > 0 ? 1.0 / n : 0.0;
            zd* o = vn + (size_t)b * ns;
            for (int k = tid; k < ns; k += kRedThreads) o[k] = zd{x[k].x * f, x[k].y * f};
        }
        if (tid == 0) {
            r = givens_column(col, c, s, n_s, g, active, jcnt, resid, bnorm[b], j, b, restart, tol);
            cs[(size_t)b * restart + j] = c[j];
            sn[(size_t)b * restart + j] = s[j];
        }
        __syncthreads();
        zd* hc = H + ((size_t)b * restart + j) * (restart + 1);
        for (int i = tid; i <= j + 1; i += kRedThreads) hc[i] = col[i];
    }
    if (tid == 0) step_done(flag, r.x, !r.y, B, gate != nullptr, step_live);
}

// The whole orthogonalisation of Arnoldi step j in one launch, one block per
// column: two classical Gram-Schmidt passes (h = V^H w, w -= V h), norm, next
// basis vector, Hessenberg column and Givens update, flags.  A thread holds
// S entries of w (k = thread + kRedThreads s); the sums run in the order of
// k_dots, k_orth and k_norm, so the results are theirs bit for bit.  Bound by
// one compute unit reading the basis four times; for short columns that is
// less than the eight launches it replaces: 11 us against 24 for one column
// of 480 entries (steps 0 to 24), 17 against 26 of 1920 (steps 0 to 16); with
// the first vectors read again for each use 12 and 20.
template <int S>
__global__ void __launch_bounds__(kRedThreads) k_arnoldi_orth(zd* __restrict__ V, const zd* __restrict__ w,
                                                              zd* __restrict__ H, double* __restrict__ cs,
                                                              zd* __restrict__ sn, zd* __restrict__ g,
                                                              int* __restrict__ active, int* __restrict__ jcnt,
                                                              double* __restrict__ resid,
                                                              const double* __restrict__ bnorm, int* __restrict__ flag,
                                                              int ns, int j, int B, int restart, double tol,
                                                              const int* __restrict__ gate,
                                                              const int* __restrict__ step_live) {
    if (gated_off(gate)) return;
    constexpr int NW = kRedThreads / 64;
    extern __shared__ unsigned char smem_raw[];
    zd* red = reinterpret_cast<zd*>(smem_raw);  // [j + 1][NW]
    zd* h = red + (j + 1) * NW;                 // [j + 1]
    zd* col = h + j + 1;                        // [j + 2]
    zd* s = col + j + 2;                        // [j + 1]
    double* c = reinterpret_cast<double*>(s + j + 1);  // [j + 1]
    __shared__ double sh[NW], n_s;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nv = j + 1;
    int2 r{0, 1};
    if (active[b]) {
        const size_t step = (size_t)B * ns;
        const zd* vb = V + (size_t)b * ns;
        zd x[S];
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int k = tid + kRedThreads * q;
            x[q] = k < ns ? w[(size_t)b * ns + k] : zd{0, 0};
        }
        for (int i = tid; i < j; i += kRedThreads) {
            c[i] = cs[(size_t)b * restart + i];
            s[i] = sn[(size_t)b * restart + i];
        }
        // U basis vectors' entries at a time, their loads in flight together
        // (entries past the column or the basis: zeros)
        constexpr int U = S == 1 ? 8 : S <= 4 ? 4 : 2;
        // (columns of up to two entries per thread: the first U vectors stay in
        // registers for all four uses)
        constexpr bool KEEP = S <= 2;
        auto load = [&](int i0, zd(&a)[U][S]) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    const int k = tid + kRedThreads * q;
                    a[u][q] = i0 + u < nv && k < ns ? vb[(i0 + u) * step + k] : zd{0, 0};
                }
        };
        zd first[KEEP ? U : 1][S];
        if constexpr (KEEP) load(0, first);
        for (int pass = 0; pass < 2; ++pass) {
            auto dots = [&](int i0, const zd(&a)[U][S]) {
                double t[2 * U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    double re = 0, im = 0;
#pragma unroll
                    for (int q = 0; q < S; ++q) {
                        if (tid + kRedThreads * q < ns) {
                            re += a[u][q].x * x[q].x + a[u][q].y * x[q].y;
                            im += a[u][q].x * x[q].y - a[u][q].y * x[q].x;
                        }
                    }
                    t[2 * u] = re;
                    t[2 * u + 1] = im;
                }
                const double sum = wave_totals<2 * U>(t, lane);
                constexpr int GL = 64 / (2 * U);
                const int v = lane / GL;
                if (lane % GL == 0 && i0 + v / 2 < nv)
                    reinterpret_cast<double*>(red + (i0 + v / 2) * NW + wave)[v & 1] = sum;
            };
            // (waves past the column's end hold zeros)
            if (wave * 64 < ns) {
                if constexpr (KEEP) dots(0, first);
                for (int i0 = KEEP ? U : 0; i0 < nv; i0 += U) {
                    zd a[U][S];
                    load(i0, a);
                    dots(i0, a);
                }
            } else if (lane == 0) {
                for (int i = 0; i < nv; ++i) red[i * NW + wave] = zd{0, 0};
            }
            __syncthreads();
            for (int i = tid; i < nv; i += kRedThreads) {
                zd t{0, 0};
                for (int q = 0; q < NW; ++q) t += red[i * NW + q];
                h[i] = t;
                col[i] = pass == 0 ? t : col[i] + t;
            }
            __syncthreads();
            auto update = [&](int i0, const zd(&a)[U][S]) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (i0 + u >= nv) break;
                    const zd hi = h[i0 + u];
#pragma unroll
                    for (int q = 0; q < S; ++q) x[q] -= hi * a[u][q];
                }
            };
            if constexpr (KEEP) update(0, first);
            for (int i0 = KEEP ? U : 0; i0 < nv; i0 += U) {
                zd a[U][S];
                load(i0, a);
                update(i0, a);
            }
        }
        double t = 0;
#pragma unroll
        for (int q = 0; q < S; ++q)
            if (tid + kRedThreads * q < ns) t += x[q].x * x[q].x + x[q].y * x[q].y;
        t = block_sum_t0(t, sh);
        if (tid == 0) n_s = sqrt(t);
        __syncthreads();
        const double n = n_s, f = n > 0 ? 1.0 / n : 0.0;
        zd* o = V + (size_t)nv * step + (size_t)b * ns;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int k = tid + kRedThreads * q;
            if (k < ns) o[k] = zd{x[q].x * f, x[q].y * f};
        }
        if (tid == 0) {
            r = givens_column(col, c, s, n, g, active, jcnt, resid, bnorm[b], j, b, restart, tol);
            cs[(size_t)b * restart + j] = c[j];
            sn[(size_t)b * restart + j] = s[j];
        }
        __syncthreads();
        zd* hc = H + ((size_t)b * restart + j) * (restart + 1);
        for (int i = tid; i <= j + 1; i += kRedThreads) hc[i] = col[i];
    }
    if (tid == 0) step_done(flag, r.x, !r.y, B, gate != nullptr, step_live);
}

// Back-substitution R y = g per column (size jcnt[b]); y[b][i].  One wave per
// column: R (up to kBackLds columns) and g come to LDS first, so that the
// serial chain of the sums waits on LDS and not on memory (one thread per
// column on global memory: 21 us at 19 columns of R, this kernel 17).
constexpr int kBackLds = 64;
__global__ void __launch_bounds__(64) k_backsolve(const zd* __restrict__ H, const zd* __restrict__ g,
                                                  const int* __restrict__ jcnt, zd* __restrict__ y, int restart,
                                                  const int* __restrict__ gate = nullptr) {
    if (gated_off(gate)) return;
    __shared__ zd R[kBackLds * (kBackLds + 1) / 2], gs[kBackLds], ys[kBackLds];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int ldh = restart + 1;
    const int n = jcnt[b];
    zd* yb = y + (size_t)b * restart;
    const zd* Hb = H + (size_t)b * restart * ldh;
    const bool lds = n <= kBackLds;
    if (lds) {
        for (int q = 0; q < n; ++q)
            if (tid <= q) R[q * (q + 1) / 2 + tid] = Hb[(size_t)q * ldh + tid];
        if (tid < n) gs[tid] = g[(size_t)b * ldh + tid];
    }
    __syncthreads();
    if (tid != 0) return;
    for (int i = n - 1; i >= 0; --i) {
        zd acc = lds ? gs[i] : g[(size_t)b * ldh + i];
        if (lds)
            for (int q = i + 1; q < n; ++q) acc -= R[q * (q + 1) / 2 + i] * ys[q];
        else
            for (int q = i + 1; q < n; ++q) acc -= Hb[(size_t)q * ldh + i] * yb[q];
        const zd d = lds ? R[i * (i + 1) / 2 + i] : Hb[(size_t)i * ldh + i];
        const double dd = d.x * d.x + d.y * d.y;
        const zd v = dd > 0 ? zd{(acc.x * d.x + acc.y * d.y) / dd, (acc.y * d.x - acc.x * d.y) / dd} : zd{0, 0};
        yb[i] = v;
        if (lds) ys[i] = v;
    }
}

// x[b] += dinv . sum_{i<jcnt[b]} y[b][i] V_i[b]
__global__ void __launch_bounds__(256) k_update_x(zd* __restrict__ x, const zd* __restrict__ V,
                                                  const zd* __restrict__ y, const int* __restrict__ jcnt,
                                                  const zd* __restrict__ dinv, int ns, int B, int restart,
                                                  const int* __restrict__ gate = nullptr) {
    if (gated_off(gate)) return;
    const int b = blockIdx.y;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= ns) return;
    const int n = jcnt[b];
    if (n == 0) return;
    zd acc{0, 0};
    for (int i = 0; i < n; ++i) acc += y[(size_t)b * restart + i] * V[((size_t)i * B + b) * ns + k];
    const zd d = dinv[k];
    x[(size_t)b * ns + k] += acc * d;
}

// y[b] = op(M) x[b] (or y[b] += op(M) x[b]) for every column b, M a complex
// CSR matrix on the near-zone pattern; op(M) = M, or with conj = 1 the
// conjugated values (the host passes the transposed copy for M^H).
__global__ void k_spmv_cols(const int* __restrict__ rowptr, const int* __restrict__ col, const zd* __restrict__ M,
                            const zd* __restrict__ x, zd* __restrict__ y, int ns, int B, int conj, int accumulate,
                            const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    const size_t tot = (size_t)ns * B;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < tot; e += (size_t)gridDim.x * blockDim.x) {
        const int b = (int)(e / ns), i = (int)(e - (size_t)b * ns);
        const zd* xb = x + (size_t)b * ns;
        zd acc{0, 0};
        for (int q = rowptr[i]; q < rowptr[i + 1]; ++q) {
            zd v = M[q];
            if (conj) v.y = -v.y;
            acc += v * xb[col[q]];
        }
        y[e] = accumulate ? y[e] + acc : acc;
    }
}

// (op(M) x)[b][i] from the columns of x transposed to xt[k][b] (FP64), for
// lanes on consecutive columns b of row i: each matrix entry is one broadcast
// load and each x row one coalesced run; entries go in groups of four with
// their loads issued together.
__device__ __forceinline__ zd spmv_row_col(const int* __restrict__ rowptr, const int* __restrict__ col,
                                           const zd* __restrict__ M, const zd* __restrict__ xt, int i, int b, int B,
                                           int conj) {
    const double sg = conj ? -1.0 : 1.0;
    zd acc{0, 0};
    const int q1 = rowptr[i + 1];
    for (int q = rowptr[i]; q < q1; q += 4) {
        zd v[4], xv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool live = q + u < q1;
            const int cu = live ? col[q + u] : 0;
            v[u] = live ? M[q + u] : zd{0, 0};
            xv[u] = xt[(size_t)cu * B + b];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += zd{v[u].x, sg * v[u].y} * xv[u];
    }
    return acc;
}

// (op(M) x)[b][i] for few columns: a group of kSpmvLanes lanes per (row i,
// column b) runs over the row's entries (coalesced entry loads), then sums
// across the group.  x[b][k] is read at x + k xs_k + b xs_b.  rows_out:
// out[i B + b] in the working precision (the operator's scaled-column
// layout); otherwise y[b][i] (FP64), added to y when accumulate.
constexpr int kSpmvLanes = 16;
template <typename R>
__global__ void __launch_bounds__(256) k_spmv_grp(const int* __restrict__ rowptr, const int* __restrict__ col,
                                                  const zd* __restrict__ M, const zd* __restrict__ x, long long xs_k,
                                                  long long xs_b, cplx<R>* __restrict__ out, zd* __restrict__ y,
                                                  int ns, int B, int conj, int accumulate,
                                                  const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const size_t pr = t / kSpmvLanes;
    const int g = (int)(t % kSpmvLanes);
    const bool live = pr < (size_t)ns * B;
    const int i = live ? (int)(pr / B) : 0, b = live ? (int)(pr % B) : 0;
    const double sg = conj ? -1.0 : 1.0;
    zd acc{0, 0};
    if (live) {
        const int q1 = rowptr[i + 1];
        for (int q = rowptr[i] + g; q < q1; q += kSpmvLanes) {
            const zd v = M[q];
            acc += zd{v.x, sg * v.y} * x[(size_t)col[q] * xs_k + (size_t)b * xs_b];
        }
    }
#pragma unroll
    for (int o = kSpmvLanes / 2; o > 0; o >>= 1) {
        acc.x += __shfl_xor(acc.x, o, 64);
        acc.y += __shfl_xor(acc.y, o, 64);
    }
    if (!live || g != 0) return;
    if (out)
        out[(size_t)i * B + b] = to_r<R>(acc);
    else {
        zd& d = y[(size_t)b * ns + i];
        d = accumulate ? d + acc : acc;
    }
}

// out[i][b] = (op(M) x)[b][i] in the working precision, the layout the
// operator's anterpolation and near zone read
template <typename R>
__global__ void __launch_bounds__(256) k_spmv_rows(const int* __restrict__ rowptr, const int* __restrict__ col,
                                                   const zd* __restrict__ M, const zd* __restrict__ xt,
                                                   cplx<R>* __restrict__ out, int ns, int B, int conj,
                                                   const int* __restrict__ gate) {
    if (gated_off(gate)) return;
    const size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (e >= (size_t)ns * B) return;
    const int i = (int)(e / B), b = (int)(e - (size_t)i * B);
    out[e] = to_r<R>(spmv_row_col(rowptr, col, M, xt, i, b, B, conj));
}

// y[b][i] += (op(M) x)[b][i] (FP64, columns of y contiguous)
__global__ void __launch_bounds__(256) k_spmv_rows_add(const int* __restrict__ rowptr, const int* __restrict__ col,
                                                       const zd* __restrict__ M, const zd* __restrict__ xt,
                                                       zd* __restrict__ y, int ns, int B, int conj,
                                                       const int* __restrict__ gate = nullptr) {
    if (gated_off(gate)) return;
    const size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (e >= (size_t)ns * B) return;
    const int i = (int)(e / B), b = (int)(e - (size_t)i * B);
    y[(size_t)b * ns + i] += spmv_row_col(rowptr, col, M, xt, i, b, B, conj);
}

// u[b] = sum_{i < jcnt[b]} y[b][i] V_i[b]  (the Krylov combination before a
// right preconditioner that is not diagonal)
__global__ void __launch_bounds__(256) k_krylov_combine(zd* __restrict__ u, const zd* __restrict__ V,
                                                        const zd* __restrict__ y, const int* __restrict__ jcnt, int ns,
                                                        int B, int restart, const int* __restrict__ gate = nullptr) {
    if (gated_off(gate)) return;
    const int b = blockIdx.y;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= ns) return;
    const int n = jcnt[b];
    zd acc{0, 0};
    for (int i = 0; i < n; ++i) acc += y[(size_t)b * restart + i] * V[((size_t)i * B + b) * ns + k];
    u[(size_t)b * ns + k] = acc;
}

__global__ void k_copy_conj(const zd* __restrict__ in, zd* __restrict__ out, size_t n, int conj) {
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        zd v = in[e];
        if (conj) v.y = -v.y;
        out[e] = v;
    }
}

// Extrapolation orders: the polynomial through the last p solutions at the
// next step, x = sum_i (-1)^(i+1) C(p, i) x_{-i}, p = 1 .. kMaxGuess
constexpr int kMaxGuess = 6;
__constant__ double kExtrap[kMaxGuess][kMaxGuess] = {{1, 0, 0, 0, 0, 0},       {2, -1, 0, 0, 0, 0},
                                                      {3, -3, 1, 0, 0, 0},      {4, -6, 4, -1, 0, 0},
                                                      {5, -10, 10, -5, 1, 0},   {6, -15, 20, -15, 6, -1}};

// Initial guess of a time step: x = sum_{i=1}^{p} a_i I_{l - dir i}, the
// polynomial through the last p solutions evaluated one step ahead
// (a_i = (-1)^(i+1) C(p, i)); p = 0 gives zero.  The march picks p as the
// order whose prediction of the step just solved was closest.
__global__ void k_extrap(const zd* __restrict__ I, zd* __restrict__ x, size_t nB, long long l, int dir, int p,
                         const int* __restrict__ pdev, StepRef sr = {}) {
    if (step_off(sr)) return;
    if (const StepDesc* d = step_of(sr)) {
        I = d->I;
        l = d->cur;
        p = d->p;
        if (!d->pdev) pdev = nullptr;
    }
    // p caps the order (history available); pdev, when given, holds the order chosen on the device
    if (pdev) p = min(p, *pdev);
    const auto& a = kExtrap;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < nB; e += (size_t)gridDim.x * blockDim.x) {
        zd acc{0, 0};
        for (int i = 1; i <= p; ++i) {
            const zd v = I[(size_t)(l - (long long)dir * i) * nB + e];
            acc.x += a[p - 1][i - 1] * v.x;
            acc.y += a[p - 1][i - 1] * v.y;
        }
        x[e] = acc;
    }
}

// Squared error of each extrapolation order p = 1..pmax at the step just
// solved, ||I_l - sum_i a_i I_{l - dir i}||^2: per-block partial sums
// part[blk][p-1] (grid-stride), then k_pred_err_sum adds the blocks in
// order (deterministic).
constexpr int kPredBlocks = 256;
__global__ void __launch_bounds__(kRedThreads) k_pred_err(const zd* __restrict__ I, size_t nB, long long l, int dir,
                                                          int pmax, double* __restrict__ part, StepRef sr = {}) {
    if (step_off(sr)) return;
    if (const StepDesc* d = step_of(sr)) {
        I = d->I;
        l = d->cur;
        pmax = d->pmax;
    }
    __shared__ double sh[kMaxGuess][kRedThreads / 64];
    const auto& a = kExtrap;
    double s[kMaxGuess] = {0, 0, 0, 0, 0, 0};
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < nB; e += (size_t)gridDim.x * blockDim.x) {
        const zd x = I[(size_t)l * nB + e];
        zd v[kMaxGuess];
        // (fixed trip counts: the solutions stay in registers)
#pragma unroll
        for (int i = 1; i <= kMaxGuess; ++i)
            v[i - 1] = i <= pmax ? I[(size_t)(l - (long long)dir * i) * nB + e] : zd{0, 0};
#pragma unroll
        for (int p = 1; p <= kMaxGuess; ++p) {
            if (p > pmax) continue;
            double rx = x.x, ry = x.y;
#pragma unroll
            for (int i = 1; i <= p; ++i) {
                rx -= a[p - 1][i - 1] * v[i - 1].x;
                ry -= a[p - 1][i - 1] * v[i - 1].y;
            }
            s[p - 1] += rx * rx + ry * ry;
        }
    }
    for (int p = 0; p < kMaxGuess; ++p) {
        const double t = block_sum_t0(s[p], sh[p]);
        if (threadIdx.x == 0) part[(size_t)blockIdx.x * kMaxGuess + p] = t;
    }
}

__global__ void __launch_bounds__(256) k_pred_err_sum(const double* __restrict__ part, int nblk,
                                                      double* __restrict__ err, int pmax, int* __restrict__ pbest,
                                                      StepRef sr = {}) {
    if (step_off(sr)) return;
    if (const StepDesc* d = step_of(sr)) pmax = d->pmax;
    __shared__ double sh[256];
    double e[kMaxGuess];
    for (int p = 0; p < kMaxGuess; ++p) {
        double s = 0;
        for (int b = threadIdx.x; b < nblk; b += 256) s += part[(size_t)b * kMaxGuess + p];
        e[p] = block_sum256(s, sh);
        if (threadIdx.x == 0) err[p] = e[p];
    }
    // the order that predicted best (the lowest on ties)
    if (threadIdx.x == 0) {
        int best = 1;
        for (int p = 2; p <= pmax; ++p)
            if (e[p - 1] < e[best - 1]) best = p;
        *pbest = best;
    }
}

// out[e][m] = in[perm[e]][m] (rows of mv values)
__global__ void k_permute_rows(const zd* __restrict__ in, zd* __restrict__ out, const int* __restrict__ perm, int n,
                               int mv) {
    const size_t tot = (size_t)n * mv;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < tot; i += (size_t)gridDim.x * blockDim.x) {
        const size_t e = i / mv, m = i - e * mv;
        out[i] = in[(size_t)perm[e] * mv + m];
    }
}

// out[e] = in[e][0] (rows of mv values)
template <typename R>
__global__ void k_take_column(const cplx<R>* __restrict__ in, cplx<R>* __restrict__ out, size_t n, int mv) {
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x)
        out[e] = in[e * mv];
}

template <typename R>
__global__ void k_to_r(const zd* __restrict__ in, cplx<R>* __restrict__ out, size_t n) {
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x)
        out[e] = cplx<R>{(R)in[e].x, (R)in[e].y};
}

// A step's solution x into I_out (out, or the call's I_out[cur] of a replayed
// step), and, in the working precision with the columns of a basis
// contiguous, into its slot of the current history (slot, or the ring of mn
// slots) and the scaled columns xs of the commit's anterpolation.  out, hist
// and xs may be null.
template <typename R>
__global__ void k_store_step(const zd* __restrict__ x, zd* __restrict__ out, cplx<R>* __restrict__ hist,
                             cplx<R>* __restrict__ xs, int ns, int B, int mn, StepRef sr) {
    if (step_off(sr)) return;
    const size_t tot = (size_t)ns * B;
    if (const StepDesc* d = step_of(sr)) {
        out = d->I + (size_t)d->cur * tot;
        if (hist) hist += (size_t)(d->cur % mn) * tot;
    }
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < tot; e += (size_t)gridDim.x * blockDim.x) {
        const int k = (int)(e / B), b = (int)(e - (size_t)k * B);
        const size_t o = (size_t)b * ns + k;
        const zd v = x[o];
        const cplx<R> r{(R)v.x, (R)v.y};
        if (out) out[o] = v;
        if (hist) hist[e] = r;
        if (xs) xs[e] = r;
    }
}

// Start of a run of replayed steps (one thread): ctl = {descriptor index, live}.
__global__ void k_step_ctl(int* __restrict__ ctl, int idx) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    ctl[0] = idx;
    ctl[1] = 1;
}

// After a replayed step's GMRES cycle (one thread): a column still active
// (not converged within the captured Arnoldi steps) or a non-finite residual
// stops the replays (live = 0) before the step commits anything.
// flag = the Arnoldi flags {active columns, non-finite, ...}.
__global__ void k_step_check(const int* __restrict__ flag, int* __restrict__ live) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    if (*live != 0 && (flag[0] > 0 || flag[1] != 0)) *live = 0;
}

// End of a replayed step (one thread): its Arnoldi step count and largest
// residual estimate into the per-step records, and the descriptor counter
// moves on.
__global__ void k_step_end(const int* __restrict__ flag, const double* __restrict__ resid, int B,
                           int* __restrict__ iters, double* __restrict__ res, int* __restrict__ ctr,
                           const int* __restrict__ live) {
    if (threadIdx.x != 0 || blockIdx.x != 0 || *live == 0) return;
    double w = 0;
    for (int b = 0; b < B; ++b) w = fmax(w, resid[b]);
    iters[*ctr] = flag[3];
    res[*ctr] = w;
    *ctr += 1;
}

template <typename R>
__global__ void k_real_to_r(const double* __restrict__ in, R* __restrict__ out, size_t n) {
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x)
        out[e] = (R)in[e];
}

}  // namespace etaim
