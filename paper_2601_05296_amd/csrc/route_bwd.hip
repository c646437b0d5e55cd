// route_bwd.hip -- router backward. The MoEBlaze paper states the gating
// forward (Section 2.1) but not its gradient; this is the closed form of the
// softmax Jacobian restricted to the top-k gates:
//   no renorm: g_j = p[id_j]            dl = p * (dp - sum_j g_j dg_j)
//   renorm:    g_j = p[id_j]/sum p[id]  dl[id_j] = g_j (dg_j - sum_j' g_j' dg_j')
// followed by dW_g = dl^T x and dx += dl W_g.
//
// bf16 path: one wave per token computes dl and stores it as two bf16 terms
// dl = hi + lo (hi = bf16(dl), lo = bf16(dl - hi); relative error about
// 2^-16), laid out [T][2Ep] with Ep = E rounded up to 32 (zero padding). Both
// products then run on the matrix cores with the grouped GEMM core:
//   dx  += [hi|lo] [W_g; W_g]       (K = 2Ep)
//   dW_g = hi^T x + lo^T x          (K = tokens, split into chunks; the
//                                    chunk partials and the two halves are
//                                    summed in a fixed order)
// f32 path: dl in float32, dx from LDS-staged dl rows (FMA), dW_g from
// token-chunk partials (float32 matrix instructions).
#include "common.hpp"
#include "gemm.hpp"
#include "gemm_rs.hpp"
#include "launch.hpp"
#include "probe.hpp"

namespace moe {
namespace {

constexpr int RB_TOK = 16;        // tokens per workgroup in the f32 dx kernel
constexpr int RB_CHUNK = 1024;    // least tokens per split in the dW_g kernels
constexpr int RB_MAXSPLIT = 128;  // most splits: the partials stay O(E d), not O(T)
constexpr int RB_EB = 32;         // experts per workgroup in the dW_g kernel

__global__ void __launch_bounds__(256)
rb_dlogits(const float* __restrict__ dg, const float* __restrict__ logits,
           const int32_t* __restrict__ ids, const float* __restrict__ gates, int64_t T, int E,
           int k, int renorm, float* __restrict__ dl) {
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    float gdg = 0.f;
    for (int j = 0; j < k; ++j) gdg += gates[t * k + j] * dg[t * k + j];
    float* out = dl + t * E;
    if (renorm) {
        for (int e = lane; e < E; e += 64) {
            float v = 0.f;
            for (int j = 0; j < k; ++j)
                if (ids[t * k + j] == e) v = gates[t * k + j] * (dg[t * k + j] - gdg);
            out[e] = v;
        }
        return;
    }
    const float* lt = logits + t * E;
    float mx = -INFINITY;
    for (int e = lane; e < E; e += 64) mx = fmaxf(mx, lt[e]);
    mx = wave_max(mx);
    float z = 0.f;
    for (int e = lane; e < E; e += 64) z += __expf(lt[e] - mx);
    z = wave_sum(z);
    for (int e = lane; e < E; e += 64) {
        float dp = 0.f;
        for (int j = 0; j < k; ++j)
            if (ids[t * k + j] == e) dp = dg[t * k + j];
        out[e] = (__expf(lt[e] - mx) / z) * (dp - gdg);
    }
}

// dx[t] (+)= sum_e dl[t][e] * W_g[e], one column per thread and RB_TOK tokens
__global__ void __launch_bounds__(256)
rb_dx(const float* __restrict__ dl, const float* __restrict__ wg, int64_t T, int d, int E,
      int accumulate, float* __restrict__ dx) {
    __shared__ float s_dl[RB_TOK][256];
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * RB_TOK;
    const int nt = (int)min((int64_t)RB_TOK, T - t0);
    for (int i = tid; i < RB_TOK * E; i += 256) {
        const int tt = i / E, e = i % E;
        s_dl[tt][e] = tt < nt ? dl[(t0 + tt) * E + e] : 0.f;
    }
    __syncthreads();
    const int c = blockIdx.y * 256 + tid;
    if (c >= d) return;
    // the old values are all loaded before the first store: loads between the
    // stores would wait for one another
    float old[RB_TOK], acc[RB_TOK];
#pragma unroll
    for (int tt = 0; tt < RB_TOK; ++tt) {
        old[tt] = accumulate && tt < nt ? dx[(t0 + tt) * d + c] : 0.f;
        acc[tt] = 0.f;
    }
    for (int e = 0; e < E; ++e) {
        const float w = wg[(int64_t)e * d + c];
#pragma unroll
        for (int tt = 0; tt < RB_TOK; ++tt) acc[tt] = fmaf(s_dl[tt][e], w, acc[tt]);
    }
#pragma unroll
    for (int tt = 0; tt < RB_TOK; ++tt)
        if (tt < nt) dx[(t0 + tt) * d + c] = accumulate ? old[tt] + acc[tt] : acc[tt];
}

// part[split][e][c] = sum over the split's tokens of dl[t][e] * x[t][c], by
// v_mfma_f32_32x32x2_f32 straight from global memory (both operands are rows of
// a token: a lane half takes every other token). A workgroup owns 32 experts x
// 32 columns of a split; its 16 waves take every 16th pair of tokens and meet in
// LDS. Latency-bound: one thread per column with a serial token loop took 416 us
// for T = 1024, E = 8, d = 256.
constexpr int RBP_WAVES = 16;

__global__ void __launch_bounds__(RBP_WAVES * WAVE)
rb_dwg_partial(const float* __restrict__ dl, const float* __restrict__ x, int64_t T, int d, int E,
               int64_t chunk, float* __restrict__ part) {
    __shared__ float red[RBP_WAVES / 2][16][WAVE];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = blockIdx.x * 32 + (lane & 31), e = blockIdx.y * RB_EB + (lane & 31);
    const int64_t tlo = (int64_t)blockIdx.z * chunk, thi = min(T, tlo + chunk);
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const bool ok = e < E;
    constexpr int U = 4;   // steps in flight (16: 12.9 us against 11.2)
    for (int64_t t = tlo + 2 * wv + (lane >> 5); t - (lane >> 5) < thi; t += 2 * RBP_WAVES * U) {
        float a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t tu = t + 2 * RBP_WAVES * u;
            const bool in = tu < thi;
            a[u] = in && ok ? dl[tu * E + e] : 0.f;
            b[u] = in ? x[tu * d + c] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[u], a[u], acc, 0, 0, 0);
    }
    // halves of the waves add up pairwise; lane holds expert lane % 32, columns
    // 8 * (r / 4) + 4 * (lane / 32) + r % 4
    for (int n = RBP_WAVES / 2; n > 0; n >>= 1) {
        if (wv >= n && wv < 2 * n)
#pragma unroll
            for (int r = 0; r < 16; ++r) red[wv - n][r][lane] = acc[r];
        __syncthreads();
        if (wv < n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] += red[wv][r][lane];
        __syncthreads();
    }
    if (wv == 0 && ok) {
        float* o = part + ((int64_t)blockIdx.z * E + e) * d + blockIdx.x * 32 + 4 * (lane >> 5);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4*>(o + 8 * q) =
                f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    }
}

__global__ void rb_dwg_reduce(const float* __restrict__ part, int nsplit, int E, int d,
                              float* __restrict__ dwg) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)E * d;
    if (i >= n) return;
    float acc = 0.f;
    for (int s = 0; s < nsplit; ++s) acc += part[s * n + i];
    dwg[i] = acc;
}

using CR = rs::Cfg<256, 256, 2, 4, 1>;
using CRN = rs::Cfg<128, 128, 2, 2, 1>;
constexpr int RB_MCH = 512;  // least tokens per split of the MFMA dW_g kernel

inline int epad(int E) { return (E + 31) / 32 * 32; }

// dl of token t as bf16 hi/lo pairs: hl[t][e] = hi, hl[t][Ep + e] = lo.
// One wave per token. The token's k (id, gate, gate gradient) triples are read
// once by lanes 0..k-1 and spread through LDS: every expert column then finds
// its own entry there instead of scanning the k ids in global memory. The
// gate sum runs in order j = 0..k-1.
__global__ void __launch_bounds__(256)
rb_dlogits_hilo(const float* __restrict__ dg, const float* __restrict__ logits,
                const int32_t* __restrict__ ids, const float* __restrict__ gates, int64_t T,
                int E, int Ep, int k, int renorm, bf16_t* __restrict__ hl) {
    __shared__ float s_dp[4][256], s_gs[4][256];   // per wave, by expert (Ep <= 256)
    __shared__ float s_g[4][16], s_dg[4][16];       // per wave, by slot j (k <= 16)
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t t = (int64_t)blockIdx.x * 4 + w;
    const bool valid = t < T;
    for (int e = lane; e < Ep; e += 64) { s_dp[w][e] = 0.f; s_gs[w][e] = 0.f; }
    __syncthreads();
    if (valid && lane < k) {
        const int e = ids[t * k + lane];
        const float gj = gates[t * k + lane], dj = dg[t * k + lane];
        s_g[w][lane] = gj;
        s_dg[w][lane] = dj;
        if ((unsigned)e < (unsigned)E) {   // ids outside [0, E) address no logit
            s_dp[w][e] = dj;
            s_gs[w][e] = gj;
        }
    }
    __syncthreads();
    if (!valid) return;
    float gdg = 0.f;
    for (int j = 0; j < k; ++j) gdg += s_g[w][j] * s_dg[w][j];
    const float* lt = logits + t * E;
    float mx = -INFINITY, z = 0.f;
    if (!renorm) {
        for (int e = lane; e < E; e += 64) mx = fmaxf(mx, lt[e]);
        mx = wave_max(mx);
        for (int e = lane; e < E; e += 64) z += __expf(lt[e] - mx);
        z = wave_sum(z);
    }
    bf16_t* out = hl + t * 2 * Ep;
    for (int e = lane; e < Ep; e += 64) {
        float v = 0.f;
        if (e < E) {
            // unselected experts: dp = 0 and (renorm) gate 0
            const float dp = s_dp[w][e];
            if (renorm) v = s_gs[w][e] * (dp - gdg);
            else v = (__expf(lt[e] - mx) / z) * (dp - gdg);
        }
        const uint32_t hi = f2bf(v);
        const uint32_t lo = f2bf(v - bf2f(hi));
        out[e] = (bf16_t)hi;
        out[Ep + e] = (bf16_t)lo;
    }
}

// dx[t] (+)= sum_k hl[t][k] * W_g[k mod Ep]   (tile: BM tokens x BN columns)
template <class C>
__device__ __forceinline__ void rb_dx_tile(int mt, int nt, const bf16_t* __restrict__ hl,
                                           const bf16_t* __restrict__ wg, int64_t T, int d, int E,
                                           int Ep, int accumulate, bf16_t* __restrict__ dx,
                                           char* lds) {
    const int64_t m0 = (int64_t)mt * C::BM;
    const int n0 = nt * C::BN;
    const int rows = (int)min((int64_t)C::BM, T - m0);
    rs::DenseKC2<C, C::BM> la;
    la.init(hl, hl, 2 * Ep, m0, rows, 2 * Ep);
    rs::SplitRowsMC<C, C::BN> lb;
    lb.init(wg, d, n0, d, Ep, E);
    rs::NoLoader nl;
    rs::Acc<C> acc;
    rs::mainloop<C>(la, lb, nl, 2 * Ep / rs::KS, lds, acc);
    WaveCoord<C> wc;
    // The lane's dx values are all loaded before the first store: loads placed
    // after a store to the same rows would each wait for the previous one.
    // (rows >= 1 and d >= 8 hold for every launched tile.)
    uint4 old[C::FM][C::FN][2];
    if (accumulate) {
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int j = 0; j < C::FN; ++j)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    // clamped into the tile's valid rows and columns, so that
                    // the loads need no branch (values off the tile are unused)
                    const int m = min(wc.row(i), rows - 1), n = min(n0 + wc.col8(j, p), d - 8);
                    old[i][j][p] = ld16(dx + (m0 + m) * d + n);
                }
    }
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
        const int m = wc.row(i);
        if (m >= rows) continue;
        bf16_t* row = dx + (m0 + m) * d;
#pragma unroll
        for (int j = 0; j < C::FN; ++j) {
            float v[2][8];
            frag_cols8(acc[0][i][j], v);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int n = n0 + wc.col8(j, p);
                if (n >= d) continue;
                if (accumulate) {
                    float o[8];
                    unpack8(old[i][j][p], o);
#pragma unroll
                    for (int r = 0; r < 8; ++r) v[p][r] += o[r];
                }
                st16(row + n, pack8(v[p]));
            }
        }
    }
}

// part[split][m][n] = sum over the split's tokens of hl[t][m] * x[t][n], m < 2Ep
template <class C>
__device__ __forceinline__ void rb_dwg_tile(int nt, int mt, int split, const bf16_t* __restrict__ hl,
                                            const bf16_t* __restrict__ x, int64_t T, int d, int Ep,
                                            int64_t chunk, float* __restrict__ part, char* lds) {
    const int n0 = nt * C::BN;
    const int m0 = mt * C::BM;
    const int64_t t0 = (int64_t)split * chunk;
    const int cnt = (int)min(chunk, T - t0);
    const int M = 2 * Ep;
    rs::SlotMC<C, C::BM> la;
    la.init(hl, M, t0, m0, M, cnt);
    rs::SlotMC<C, C::BN> lb;
    lb.init(x, d, t0, n0, d, cnt);
    rs::NoLoader nl;
    rs::Acc<C> acc;
    rs::mainloop<C>(la, lb, nl, rs::slices(cnt), lds, acc);
    WaveCoord<C> wc;
    float* out = part + (int64_t)split * M * d;
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
        const int m = m0 + wc.row(i);
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + wc.col(j, q);
                if (n >= d) continue;
                const f32x16& v = acc[0][i][j];
                *reinterpret_cast<f32x4*>(out + (int64_t)m * d + n) =
                    f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
            }
    }
}

// Both products of the router backward in one launch: the first n_dx workgroups
// take dx tiles (bound by reading and writing dx), the others dW_g tiles (by
// reading x), so that neither waits for the other's last wave.
template <class C>
__global__ void __launch_bounds__(C::THREADS, 2)
rb_products(const bf16_t* __restrict__ hl, const bf16_t* __restrict__ wg,
            const bf16_t* __restrict__ x, int64_t T, int d, int E, int Ep, int accumulate,
            int n_dx, int64_t chunk, bf16_t* __restrict__ dx, float* __restrict__ part) {
    extern __shared__ __align__(16) char lds[];
    const int NT = (d + C::BN - 1) / C::BN;
    int b = blockIdx.x;
    if (b < n_dx) {
        rb_dx_tile<C>(b / NT, b % NT, hl, wg, T, d, E, Ep, accumulate, dx, lds);
        return;
    }
    b -= n_dx;
    const int MT = (2 * Ep + C::BM - 1) / C::BM;
    rb_dwg_tile<C>(b % NT, b / NT % MT, b / (NT * MT), hl, x, T, d, Ep, chunk, part, lds);
}

// dw_gate[e][i] = sum_split (part[split][e][i] + part[split][Ep + e][i])
__global__ void rb_dwg_reduce_hilo(const float* __restrict__ part, int nsplit, int E, int Ep,
                                   int d, float* __restrict__ dwg) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)E * d) return;
    const int64_t per = (int64_t)2 * Ep * d;
    const int64_t lo_off = (int64_t)Ep * d;
    float acc = 0.f;
    // unrolled so that the loads of several splits are in flight at once; the
    // sum still runs in split order
#pragma unroll 8
    for (int s = 0; s < nsplit; ++s) acc += part[s * per + i] + part[s * per + lo_off + i];
    dwg[i] = acc;
}

// tokens per split: at least `least`, and at most RB_MAXSPLIT splits
inline int64_t split_tokens(int64_t T, int64_t least) {
    int64_t c = (T + RB_MAXSPLIT - 1) / RB_MAXSPLIT;
    c = (c + 63) / 64 * 64;
    return c > least ? c : least;
}
inline int nsplits(int64_t T) { const int64_t c = split_tokens(T, RB_CHUNK); return (int)((T + c - 1) / c); }
inline int msplits(int64_t T) { const int64_t c = split_tokens(T, RB_MCH); return (int)((T + c - 1) / c); }
inline size_t al256(size_t b) { return (b + 255) / 256 * 256; }

template <class C>
inline int64_t rb_dx_tiles(int64_t T, int d) { return (T + C::BM - 1) / C::BM * ((d + C::BN - 1) / C::BN); }
template <class C>
inline int64_t rb_dwg_tiles(int d, int Ep, int splits) {
    return (int64_t)((d + C::BN - 1) / C::BN) * ((2 * Ep + C::BM - 1) / C::BM) * splits;
}

template <class C>
hipError_t launch_products(const bf16_t* hl, const void* wg, const void* x, int64_t T, int d, int E,
                           int Ep, bool accumulate, void* dx, float* part, hipStream_t st) {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(rb_products<C>), hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (attr != hipSuccess) return attr;
    const int64_t n_dx = rb_dx_tiles<C>(T, d), n_dwg = rb_dwg_tiles<C>(d, Ep, msplits(T));
    hipLaunchKernelGGL(rb_products<C>, dim3((unsigned)(n_dx + n_dwg)), dim3(C::THREADS), C::LDS, st, hl,
                       (const bf16_t*)wg, (const bf16_t*)x, T, d, E, Ep, (int)accumulate, (int)n_dx,
                       split_tokens(T, RB_MCH), (bf16_t*)dx, part);
    probe::mark("rb_products", st);
    return hipGetLastError();
}

}  // namespace

size_t route_bwd_workspace(int64_t T, int d, int E, int k, bool f32) {
    (void)k;
    if (f32) {
        const size_t dl = (size_t)T * E * sizeof(float);
        const size_t part = (size_t)nsplits(T) * E * d * sizeof(float);
        return al256(dl) + part;
    }
    const int Ep = epad(E);
    return al256((size_t)T * 2 * Ep * sizeof(bf16_t)) + (size_t)msplits(T) * 2 * Ep * d * sizeof(float);
}

hipError_t route_bwd(const float* dgates, const float* logits, const int32_t* ids,
                     const float* gates, const void* x, const void* wg, int64_t T, int d,
                     int E, int k, bool f32, bool renorm, bool accumulate, float* dwg,
                     void* dx, void* ws, hipStream_t st) {
    if (f32) {
        float* dl = static_cast<float*>(ws);
        float* part = reinterpret_cast<float*>(static_cast<char*>(ws) + al256((size_t)T * E * sizeof(float)));
        hipLaunchKernelGGL(rb_dlogits, dim3((unsigned)((T + 3) / 4)), dim3(256), 0, st, dgates,
                           logits, ids, gates, T, E, k, (int)renorm, dl);
        probe::mark("rb_dlogits", st);
        hipLaunchKernelGGL(rb_dx, dim3((unsigned)((T + RB_TOK - 1) / RB_TOK), (unsigned)((d + 255) / 256)),
                           dim3(256), 0, st, dl, static_cast<const float*>(wg), T, d, E,
                           (int)accumulate, static_cast<float*>(dx));
        probe::mark("rb_dx", st);
        const int ns = nsplits(T);
        hipLaunchKernelGGL(rb_dwg_partial,
                           dim3((unsigned)(d / 32), (unsigned)((E + RB_EB - 1) / RB_EB), (unsigned)ns),
                           dim3(RBP_WAVES * WAVE), 0, st, dl, static_cast<const float*>(x), T, d, E,
                           split_tokens(T, RB_CHUNK), part);
        probe::mark("rb_dwg_partial", st);
        hipLaunchKernelGGL(rb_dwg_reduce, dim3((unsigned)(((int64_t)E * d + 255) / 256)), dim3(256), 0,
                           st, part, ns, E, d, dwg);
        probe::mark("rb_dwg_reduce", st);
        return hipGetLastError();
    }
    const int Ep = epad(E);
    bf16_t* hl = static_cast<bf16_t*>(ws);
    float* part = reinterpret_cast<float*>(static_cast<char*>(ws) +
                                           al256((size_t)T * 2 * Ep * sizeof(bf16_t)));
    hipLaunchKernelGGL(rb_dlogits_hilo, dim3((unsigned)((T + 3) / 4)), dim3(256), 0, st, dgates,
                       logits, ids, gates, T, E, Ep, k, (int)renorm, hl);
    probe::mark("rb_dlogits", st);
    // Quarter tiles, two workgroups per CU, where the 256 x 256 ones would leave CUs
    // idle (T = 1021, d = 2048, E = 64: 48 tiles).
    const int ms = msplits(T);
    const bool few = rb_dx_tiles<CR>(T, d) + rb_dwg_tiles<CR>(d, Ep, ms) <= 256;
    if (hipError_t e = few ? launch_products<CRN>(hl, wg, x, T, d, E, Ep, accumulate, dx, part, st)
                           : launch_products<CR>(hl, wg, x, T, d, E, Ep, accumulate, dx, part, st);
        e != hipSuccess)
        return e;
    hipLaunchKernelGGL(rb_dwg_reduce_hilo, dim3((unsigned)(((int64_t)E * d + 255) / 256)), dim3(256), 0,
                       st, part, ms, E, Ep, d, dwg);
    probe::mark("rb_dwg_reduce", st);
    return hipGetLastError();
}

}  // namespace moe
