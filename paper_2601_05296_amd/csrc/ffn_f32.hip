// ffn_f32.hip -- the expert FFN in float32 (MOE_F32): the grouped GEMMs G1..G6
// of ffn.hip on the float32 matrix instruction v_mfma_f32_32x32x2_f32 (float32
// products and sums throughout).
//
// Small layers at full precision: a launch has a few hundred tiles and a few
// thousand multiply-adds of K, so the bound is the latency of one tile's K loop
// (a slice of 32 k takes 16 MFMAs of 64 cycles per wave) rather than any rate.
// 64 x 64 tiles of four waves give T = 1024, E = 8, k = 2, d = 256, f = 512
// between 144 and 290 workgroups a launch, 19 to 28 us each (G1..G6: 149 us). One
// output per thread before, with strided reads of the weights: 15.3 ms, of which
// the dh kernel (one thread per slot) took 12.3.
//
// Operand tiles are 64 rows x 32 k, K contiguous in LDS whatever their layout in
// memory: operands whose K is the outer dimension are transposed on the way, in
// 4 x 4 blocks of one thread. A lane reads 4 k at a time (16 bytes) and feeds
// them to 4 MFMAs, so the k of MFMA j, lane half h are 8q + 4h + j: the same
// permutation on both operands. 16-byte chunks are XOR-swizzled by row / 4.
#include "common.hpp"
#include "ffn_epi.hpp"
#include "gemm.hpp"
#include "launch.hpp"
#include "probe.hpp"

namespace moe {
namespace {

constexpr int FT = 64;                 // tile rows and columns
constexpr int FK = 32;                 // K slice
constexpr int F_THREADS = 256;         // 2 x 2 waves of 32 x 32
constexpr int TILE_F = FT * FK;        // floats of one operand tile

__device__ __forceinline__ int f_off(int r, int c) { return r * FK + ((c ^ ((r >> 2) & 7)) << 2); }

// Operand with K contiguous: two 16-byte chunks per thread; off(r) is the
// element offset of tile row r, at(o) the four elements at offset o.
template <class OFF, class AT>
struct LoadKC {
    AT at;
    int64_t o[2];
    f32x4 v[2][2];   // [slice parity][chunk]
    __device__ LoadKC(OFF&& off, AT at_) : at(at_) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = threadIdx.x + i * F_THREADS;
            o[i] = off(q >> 3) + (q & 7) * 4;
        }
    }
    template <int S> __device__ void load(int kt) {
#pragma unroll
        for (int i = 0; i < 2; ++i) v[S][i] = at(o[i] + kt * FK);
    }
    template <int S> __device__ void store(float* t) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = threadIdx.x + i * F_THREADS;
            *reinterpret_cast<f32x4*>(t + f_off(q >> 3, q & 7)) = v[S][i];
        }
    }
};
template <class OFF, class AT>
__device__ LoadKC<OFF, AT> load_kc(OFF off, AT at) { return LoadKC<OFF, AT>(std::move(off), at); }

// Operand with K outermost: one 4 x 4 block per thread of a half workgroup
// (HALF 0 or 1), at(k, c, i) the four elements of K row k from tile column c on.
// i = idx(k) is read one slice ahead of the row (the row of a gathered operand;
// a load that waits for an index read just before it stalls its wave).
struct NoIndex { __device__ int operator()(int) const { return 0; } };
template <int HALF, class AT, class IDX>
struct LoadMC {
    AT at;
    IDX idx;
    f32x4 v[2][4];   // [slice parity][k row]
    int nx[4];       // indices of the next slice's rows
    __device__ LoadMC(AT at_, IDX idx_) : at(at_), idx(idx_) {
        if (!mine()) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) nx[i] = idx(kb() * 4 + i);
    }
    __device__ static bool mine() { return (int)(threadIdx.x >> 7) == HALF; }
    __device__ static int kb() { return (threadIdx.x & 127) >> 4; }
    __device__ static int cb() { return threadIdx.x & 15; }
    template <int S> __device__ void load(int kt) {
        if (!mine()) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[S][i] = at(kt * FK + kb() * 4 + i, cb() * 4, nx[i]);
#pragma unroll
        for (int i = 0; i < 4; ++i) nx[i] = idx((kt + 1) * FK + kb() * 4 + i);
    }
    template <int S> __device__ void store(float* t) {
        if (!mine()) return;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<f32x4*>(t + f_off(cb() * 4 + i, kb())) =
                f32x4{v[S][0][i], v[S][1][i], v[S][2][i], v[S][3][i]};
    }
};
template <int HALF, class AT, class IDX = NoIndex>
__device__ LoadMC<HALF, AT, IDX> load_mc(AT at, IDX idx = IDX{}) { return LoadMC<HALF, AT, IDX>(at, idx); }

struct NoLoad {
    template <int S> __device__ void load(int) {}
    template <int S> __device__ void store(float*) {}
};

__device__ __forceinline__ f32x4 ldf4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// acc[b] += left * right_b over nk slices of K; lds: 2 * (1 + NB) operand tiles.
// The loads of a slice are issued two slices before its LDS write (registers by
// slice parity): G2 33 -> 28 us, G6 27 -> 24 (16 and 32 slices) at the shape
// above. What is left there is mostly fixed: 24 slices more cost G6 only 6 us
// over G4's 8.
template <int NB, class L, class R0, class R1>
__device__ __forceinline__ void f_mainloop(L& l, R0& r0, R1& r1, int nk, float* lds,
                                           f32x16 (&acc)[NB]) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wm = wv >> 1, wn = wv & 1, h = lane >> 5, row = lane & 31;
    if (nk <= 0) return;
    constexpr int STAGE = (1 + NB) * TILE_F;
    auto load = [&](auto s_c, int kt) __attribute__((always_inline)) {
        constexpr int S = decltype(s_c)::value;
        l.template load<S>(kt);
        r0.template load<S>(kt);
        r1.template load<S>(kt);
    };
    auto store = [&](auto s_c) __attribute__((always_inline)) {
        constexpr int S = decltype(s_c)::value;
        float* t = lds + S * STAGE;
        l.template store<S>(t);
        r0.template store<S>(t + TILE_F);
        if constexpr (NB == 2) r1.template store<S>(t + 2 * TILE_F);
    };
    std::integral_constant<int, 0> even;
    std::integral_constant<int, 1> odd;
    // odd slices add up apart from the even ones: two shorter chains of float32
    // additions per output round less than one
    f32x16 half[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) half[b][r] = 0.f;
    auto slice = [&](int kt, auto s_c, auto next_c) __attribute__((always_inline)) {
        constexpr int S = decltype(s_c)::value;
        const float* t = lds + S * STAGE;
        if (kt + 2 < nk) load(s_c, kt + 2);
#pragma unroll
        for (int q = 0; q < FK / 8; ++q) {
            const f32x4 a = ldf4(t + f_off(wm * 32 + row, 2 * q + h));
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const f32x4 w = ldf4(t + (1 + b) * TILE_F + f_off(wn * 32 + row, 2 * q + h));
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f32x16& c = S ? half[b] : acc[b];
                    c = __builtin_amdgcn_mfma_f32_32x32x2f32(w[j], a[j], c, 0, 0, 0);
                }
            }
        }
        if (kt + 1 < nk) store(next_c);
        __syncthreads();
    };
    load(even, 0);
    if (nk > 1) load(odd, 1);
    store(even);
    __syncthreads();
    for (int kt = 0; kt < nk; kt += 2) {
        slice(kt, even, odd);
        if (kt + 1 < nk) slice(kt + 1, odd, even);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] += half[b][r];
}

// output coordinates: row of the tile, first column of run q (four columns)
__device__ __forceinline__ int f_row() { return (threadIdx.x >> 7) * 32 + (threadIdx.x & 31); }
__device__ __forceinline__ int f_col(int q) {
    return ((threadIdx.x >> 6) & 1) * 32 + q * 8 + ((threadIdx.x >> 5) & 1) * 4;
}
__device__ __forceinline__ f32x4 f_run(const f32x16& a, int q) {
    return f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
}
template <int NB>
__device__ __forceinline__ void f_zero(f32x16 (&acc)[NB]) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
}

__device__ __forceinline__ float silu32(float a) { return a / (1.0f + __expf(-a)); }

// h and its derivatives from the first-layer outputs (b unused when non-gated)
template <int ACT>
__device__ __forceinline__ float f32_h(float a, float b) {
    if constexpr (ACT == ACT_SWIGLU) return silu32(a) * b;
    else if constexpr (ACT == ACT_RELU) return a > 0.f ? a : 0.f;
    else return silu32(a);
}
template <int ACT>
__device__ __forceinline__ f32x4 f32_h4(const float* A, const float* B, int64_t o) {
    const f32x4 a = ldf4(A + o), b = ACT == ACT_SWIGLU ? ldf4(B + o) : a;
    return f32x4{f32_h<ACT>(a[0], b[0]), f32_h<ACT>(a[1], b[1]), f32_h<ACT>(a[2], b[2]),
                 f32_h<ACT>(a[3], b[3])};
}

__device__ __forceinline__ bool f_tile(float* lds, const int32_t* offsets, int E, int NT,
                                       SlotTile& t) {
    return find_slot_tile<F_THREADS>(reinterpret_cast<int*>(lds), offsets, E, FT, NT, blockIdx.x,
                                     FT, t, 4);
}

// G1: A = x[eti] W1[e], B = x[eti] W3[e]
template <int ACT>
__global__ void __launch_bounds__(F_THREADS)
f32_g1(const float* __restrict__ x, const float* __restrict__ w1, const float* __restrict__ w3,
       const int32_t* __restrict__ offsets, const int32_t* __restrict__ eti, int d, int f, int E,
       float* __restrict__ A, float* __restrict__ B) {
    constexpr int NB = ACT == ACT_SWIGLU ? 2 : 1;
    __shared__ __align__(16) float lds[2 * (1 + NB) * TILE_F];
    SlotTile t;
    if (!f_tile(lds, offsets, E, f / FT, t)) return;
    const int32_t* idx = eti + t.off + t.m0;
    auto l = load_kc([&](int r) { return (int64_t)idx[r < t.mrows ? r : 0] * d; },
                     [=](int64_t o) { return ldf4(x + o); });
    const float* w1e = w1 + (int64_t)t.e * d * f + t.n0;
    const float* w3e = ACT == ACT_SWIGLU ? w3 + (int64_t)t.e * d * f + t.n0 : nullptr;
    auto r0 = load_mc<0>([=](int k, int c, int) { return ldf4(w1e + (int64_t)k * f + c); });
    f32x16 acc[NB];
    f_zero(acc);
    if constexpr (NB == 2) {
        auto r1 = load_mc<1>([=](int k, int c, int) { return ldf4(w3e + (int64_t)k * f + c); });
        f_mainloop<NB>(l, r0, r1, d / FK, lds, acc);
    } else {
        NoLoad r1;
        f_mainloop<NB>(l, r0, r1, d / FK, lds, acc);
    }
    if (f_row() >= t.mrows) return;
    const int64_t o = ((int64_t)t.off + t.m0 + f_row()) * f + t.n0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        *reinterpret_cast<f32x4*>(A + o + f_col(q)) = f_run(acc[0], q);
        if constexpr (NB == 2) *reinterpret_cast<f32x4*>(B + o + f_col(q)) = f_run(acc[NB - 1], q);
    }
}

// G2: O = h W2[e], h formed on load
template <int ACT>
__global__ void __launch_bounds__(F_THREADS)
f32_g2(const float* __restrict__ A, const float* __restrict__ B, const float* __restrict__ w2,
       const int32_t* __restrict__ offsets, int d, int f, int E, float* __restrict__ O) {
    __shared__ __align__(16) float lds[4 * TILE_F];
    SlotTile t;
    if (!f_tile(lds, offsets, E, d / FT, t)) return;
    const int64_t row0 = (int64_t)t.off + t.m0;
    auto l = load_kc([&](int r) { return (row0 + (r < t.mrows ? r : 0)) * f; },
                     [=](int64_t o) { return f32_h4<ACT>(A, B, o); });
    const float* w2e = w2 + (int64_t)t.e * f * d + t.n0;
    auto r0 = load_mc<0>([=](int k, int c, int) { return ldf4(w2e + (int64_t)k * d + c); });
    NoLoad r1;
    f32x16 acc[1];
    f_zero(acc);
    f_mainloop<1>(l, r0, r1, f / FK, lds, acc);
    if (f_row() >= t.mrows) return;
    float* o = O + (row0 + f_row()) * d + t.n0;
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<f32x4*>(o + f_col(q)) = f_run(acc[0], q);
}

// G4: u = dY[eti] W2[e]^T, dA and dB in place, and part[s][p] = the gate
// gradient's sum of u * h over the columns of part p: column tiles p, p + P, ...
// (P parts per slot; the tile lookup runs over the parts). P = 1: the whole sum,
// straight into the gate gradients.
template <int ACT>
__global__ void __launch_bounds__(F_THREADS)
f32_g4(const float* __restrict__ dy, const float* __restrict__ w2, const float* __restrict__ gates,
       const int32_t* __restrict__ offsets, const int32_t* __restrict__ eti,
       const int32_t* __restrict__ slot_src, int d, int f, int E, int P, float* __restrict__ A,
       float* __restrict__ B, float* __restrict__ part, float* __restrict__ dgates) {
    __shared__ __align__(16) float lds[4 * TILE_F];
    __shared__ float red[2][FT];
    SlotTile t;
    if (!f_tile(lds, offsets, E, P, t)) return;
    const int p0 = t.n0 / FT;
    const int64_t row0 = (int64_t)t.off + t.m0;
    const int32_t* idx = eti + row0;
    const bool valid = f_row() < t.mrows;
    const int64_t s = row0 + (valid ? f_row() : 0);
    const float g = gates[slot_src[s]];
    auto l = load_kc([&](int r) { return (int64_t)idx[r < t.mrows ? r : 0] * d; },
                     [=](int64_t o) { return ldf4(dy + o); });
    const float* w2e = w2 + (int64_t)t.e * f * d;
    float dg = 0.f;
    for (int n0 = p0 * FT; n0 < f; n0 += P * FT) {
        auto r0 = load_kc([&](int r) { return (int64_t)(n0 + r) * d; },
                          [=](int64_t o) { return ldf4(w2e + o); });
        NoLoad r1;
        f32x16 acc[1];
        f_zero(acc);
        f_mainloop<1>(l, r0, r1, d / FK, lds, acc);
        f32x4 av[4], bv[4];   // all loaded before the first store to A or B
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t o = s * f + n0 + f_col(q);
            av[q] = ldf4(A + o);
            bv[q] = ACT == ACT_SWIGLU ? ldf4(B + o) : av[q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t o = s * f + n0 + f_col(q);
            const f32x4 a = av[q], b = bv[q];
            f32x4 da, db;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float u = acc[0][4 * q + r], dh = g * u;
                if constexpr (ACT == ACT_RELU) {
                    dg = fmaf(u, a[r] > 0.f ? a[r] : 0.f, dg);
                    da[r] = a[r] > 0.f ? dh : 0.f;
                } else {
                    const float sg = 1.0f / (1.0f + __expf(-a[r]));
                    const float bb = ACT == ACT_SWIGLU ? b[r] : 1.0f;
                    dg = fmaf(u, a[r] * sg * bb, dg);
                    da[r] = dh * bb * sg * (1.0f + a[r] * (1.0f - sg));
                    db[r] = dh * a[r] * sg;
                }
            }
            if (valid) {
                *reinterpret_cast<f32x4*>(A + o) = da;
                if constexpr (ACT == ACT_SWIGLU) *reinterpret_cast<f32x4*>(B + o) = db;
            }
        }
    }
    dg += __shfl_xor(dg, 32, 64);
    if ((threadIdx.x & 32) == 0) red[(threadIdx.x >> 6) & 1][f_row()] = dg;
    __syncthreads();
    if ((int)threadIdx.x < t.mrows) {
        const float sum = red[0][threadIdx.x] + red[1][threadIdx.x];
        if (P == 1) dgates[slot_src[row0 + threadIdx.x]] = sum;
        else part[(row0 + threadIdx.x) * P + p0] = sum;
    }
}

// G6: dX_slot = dA W1[e]^T + dB W3[e]^T
template <int ACT>
__global__ void __launch_bounds__(F_THREADS)
f32_g6(const float* __restrict__ dA, const float* __restrict__ dB, const float* __restrict__ w1,
       const float* __restrict__ w3, const int32_t* __restrict__ offsets, int d, int f, int E,
       float* __restrict__ dX) {
    __shared__ __align__(16) float lds[4 * TILE_F];
    SlotTile t;
    if (!f_tile(lds, offsets, E, d / FT, t)) return;
    const int64_t row0 = (int64_t)t.off + t.m0;
    f32x16 acc[1];
    f_zero(acc);
    auto run = [&](const float* src, const float* w) {
        const float* we = w + ((int64_t)t.e * d + t.n0) * f;
        auto l = load_kc([&](int r) { return (row0 + (r < t.mrows ? r : 0)) * f; },
                         [=](int64_t o) { return ldf4(src + o); });
        auto r0 = load_kc([&](int r) { return (int64_t)r * f; },
                          [=](int64_t o) { return ldf4(we + o); });
        NoLoad r1;
        f_mainloop<1>(l, r0, r1, f / FK, lds, acc);
    };
    run(dA, w1);
    if constexpr (ACT == ACT_SWIGLU) run(dB, w3);
    if (f_row() >= t.mrows) return;
    float* o = dX + (row0 + f_row()) * d + t.n0;
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<f32x4*>(o + f_col(q)) = f_run(acc[0], q);
}

// weight-gradient tile: expert, first row and column (M rows of N columns)
__device__ __forceinline__ void f_wtile(int M, int N, int& e, int& m0, int& n0) {
    const int NT = N / FT, P = (M / FT) * NT;
    e = blockIdx.x / P;
    const int lt = blockIdx.x % P;
    m0 = lt / NT * FT;
    n0 = lt % NT * FT;
}
// K rows of a weight gradient are the expert's slots; rows at or past cnt are
// zero in both operands
template <class F>
__device__ __forceinline__ f32x4 f_slot(int k, int cnt, F&& f) {
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    return k < cnt ? f() : z;
}
__device__ __forceinline__ void f_out(float* p, const f32x4& v, int add) {
    *reinterpret_cast<f32x4*>(p) = add ? v + ldf4(p) : v;
}

// G3: dW2[e] = sum_s (g h)[s]^T dY[eti[s]]
template <int ACT>
__global__ void __launch_bounds__(F_THREADS)
f32_g3(const float* __restrict__ A, const float* __restrict__ B, const float* __restrict__ dy,
       const float* __restrict__ gates, const int32_t* __restrict__ offsets,
       const int32_t* __restrict__ eti, const int32_t* __restrict__ slot_src, int d, int f, int add,
       float* __restrict__ dw2) {
    __shared__ __align__(16) float lds[4 * TILE_F];
    int e, m0, n0;
    f_wtile(f, d, e, m0, n0);
    const int64_t off = offsets[e];
    const int cnt = offsets[e + 1] - (int)off;
    const int32_t *ss = slot_src + off, *tok = eti + off;
    auto l = load_mc<0>(
        [=](int k, int c, int i) {
            return f_slot(k, cnt, [&] { return gates[i] * f32_h4<ACT>(A, B, (off + k) * f + m0 + c); });
        },
        [=](int k) { return cnt > 0 ? ss[min(k, cnt - 1)] : 0; });
    auto r0 = load_mc<1>(
        [=](int k, int c, int i) {
            return f_slot(k, cnt, [&] { return ldf4(dy + (int64_t)i * d + n0 + c); });
        },
        [=](int k) { return cnt > 0 ? tok[min(k, cnt - 1)] : 0; });
    NoLoad r1;
    f32x16 acc[1];
    f_zero(acc);
    f_mainloop<1>(l, r0, r1, (cnt + FK - 1) / FK, lds, acc);
    float* o = dw2 + ((int64_t)e * f + m0 + f_row()) * d + n0;
#pragma unroll
    for (int q = 0; q < 4; ++q) f_out(o + f_col(q), f_run(acc[0], q), add);
}

// G5: dW1[e] = x[eti]^T dA, dW3[e] = x[eti]^T dB; one right operand per
// workgroup (blockIdx.y: dA or dB)
__global__ void __launch_bounds__(F_THREADS)
f32_g5(const float* __restrict__ x, const float* __restrict__ dA, const float* __restrict__ dB,
       const int32_t* __restrict__ offsets, const int32_t* __restrict__ eti, int d, int f, int add,
       float* __restrict__ dw1, float* __restrict__ dw3) {
    __shared__ __align__(16) float lds[4 * TILE_F];
    int e, m0, n0;
    f_wtile(d, f, e, m0, n0);
    const int64_t off = offsets[e];
    const int cnt = offsets[e + 1] - (int)off;
    const float* src = blockIdx.y ? dB : dA;
    const int32_t* tok = eti + off;
    auto l = load_mc<0>(
        [=](int k, int c, int i) {
            return f_slot(k, cnt, [&] { return ldf4(x + (int64_t)i * d + m0 + c); });
        },
        [=](int k) { return cnt > 0 ? tok[min(k, cnt - 1)] : 0; });
    auto r0 = load_mc<1>([=](int k, int c, int) {
        return f_slot(k, cnt, [&] { return ldf4(src + (off + k) * f + n0 + c); });
    });
    NoLoad r1;
    f32x16 acc[1];
    f_zero(acc);
    f_mainloop<1>(l, r0, r1, (cnt + FK - 1) / FK, lds, acc);
    float* o = (blockIdx.y ? dw3 : dw1) + ((int64_t)e * d + m0 + f_row()) * f + n0;
#pragma unroll
    for (int q = 0; q < 4; ++q) f_out(o + f_col(q), f_run(acc[0], q), add);
}

// worst-case tile count of a row-wise GEMM with NT column tiles
inline unsigned f_grid(int64_t S, int E, int NT) { return (unsigned)(((S + FT - 1) / FT + E) * NT); }

template <int ACT>
hipError_t f32_first_act(const FfnArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(f32_g1<ACT>, dim3(f_grid(a.T * a.k, a.E, a.f / FT)), dim3(F_THREADS), 0, st,
                       (const float*)a.x, (const float*)a.w1, (const float*)a.w3, a.offsets, a.eti,
                       a.d, a.f, a.E, (float*)a.A, (float*)a.B);
    probe::mark("f32_g1", st);
    return hipGetLastError();
}

template <int ACT>
hipError_t f32_fwd_act(const FfnArgs& a, hipStream_t st) {
    if (hipError_t e = f32_first_act<ACT>(a, st); e != hipSuccess) return e;
    float* O = a.y ? static_cast<float*>(a.ws) : (float*)a.O;
    hipLaunchKernelGGL(f32_g2<ACT>, dim3(f_grid(a.T * a.k, a.E, a.d / FT)), dim3(F_THREADS), 0, st,
                       (const float*)a.A, (const float*)a.B, (const float*)a.w2, a.offsets, a.d,
                       a.f, a.E, O);
    probe::mark("f32_g2", st);
    if (a.y) return combine(O, a.gates, a.tim, a.T, a.d, a.k, true, false, a.y, st);
    return hipGetLastError();
}

template <int ACT>
hipError_t f32_bwd_act(const FfnArgs& a, hipStream_t st) {
    const int64_t S = a.T * a.k;
    hipLaunchKernelGGL(f32_g3<ACT>, dim3(a.E * (a.f / FT) * (a.d / FT)), dim3(F_THREADS), 0, st,
                       (const float*)a.A, (const float*)a.B, (const float*)a.dy, a.gates,
                       a.offsets, a.eti, a.slot_src, a.d, a.f, (int)a.accumulate_dw, a.dw2);
    probe::mark("f32_g3", st);
    // dX_slot's space (the output, or the workspace of the combined call) holds
    // the gate-gradient parts until G6 writes it: at most d parts per slot. An
    // output over dy or x, which G4 and G5 still read, holds nothing before G6: one
    // part per slot then.
    float* dX = a.y ? static_cast<float*>(a.ws) : (float*)a.dX;
    auto over = [&](const void* p) {
        const uintptr_t b = reinterpret_cast<uintptr_t>(p), o = reinterpret_cast<uintptr_t>(dX);
        return b < o + (size_t)S * a.d * 4 && o < b + (size_t)a.T * a.d * 4;
    };
    const int P = over(a.dy) || over(a.x) ? 1 : a.f / FT < a.d ? a.f / FT : a.d;
    hipLaunchKernelGGL(f32_g4<ACT>, dim3(f_grid(S, a.E, P)), dim3(F_THREADS), 0, st,
                       (const float*)a.dy, (const float*)a.w2, a.gates, a.offsets, a.eti,
                       a.slot_src, a.d, a.f, a.E, P, (float*)a.A, (float*)a.B, dX, a.dgates);
    probe::mark("f32_g4", st);
    if (P > 1) {
        if (hipError_t e = dgate_sum(dX, P, a.slot_src, a.offsets, a.E, S, a.dgates, st); e != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL(f32_g5, dim3(a.E * (a.d / FT) * (a.f / FT), ACT == ACT_SWIGLU ? 2 : 1),
                       dim3(F_THREADS), 0, st, (const float*)a.x, (const float*)a.A,
                       (const float*)a.B, a.offsets, a.eti, a.d, a.f, (int)a.accumulate_dw, a.dw1,
                       a.dw3);
    probe::mark("f32_g5", st);
    hipLaunchKernelGGL(f32_g6<ACT>, dim3(f_grid(S, a.E, a.d / FT)), dim3(F_THREADS), 0, st,
                       (const float*)a.A, (const float*)a.B, (const float*)a.w1,
                       (const float*)a.w3, a.offsets, a.d, a.f, a.E, dX);
    probe::mark("f32_g6", st);
    if (a.y) return combine(dX, nullptr, a.tim, a.T, a.d, a.k, true, a.accumulate, a.y, st);
    return hipGetLastError();
}

}  // namespace

hipError_t f32_first(const FfnArgs& a, hipStream_t st) {
    return a.act == ACT_SILU   ? f32_first_act<ACT_SILU>(a, st)
           : a.act == ACT_RELU ? f32_first_act<ACT_RELU>(a, st)
                               : f32_first_act<ACT_SWIGLU>(a, st);
}
hipError_t f32_fwd(const FfnArgs& a, hipStream_t st) {
    return a.act == ACT_SILU   ? f32_fwd_act<ACT_SILU>(a, st)
           : a.act == ACT_RELU ? f32_fwd_act<ACT_RELU>(a, st)
                               : f32_fwd_act<ACT_SWIGLU>(a, st);
}
hipError_t f32_bwd(const FfnArgs& a, hipStream_t st) {
    return a.act == ACT_SILU   ? f32_bwd_act<ACT_SILU>(a, st)
           : a.act == ACT_RELU ? f32_bwd_act<ACT_RELU>(a, st)
                               : f32_bwd_act<ACT_SWIGLU>(a, st);
}

}  // namespace moe
