// ffn_epi.hpp -- arithmetic and output stages shared by the grouped GEMMs of the
// expert FFN, whatever core (gemm_rs.hpp, gemm_sk.hpp) ran their main loop:
// activations, h formed from A and B, the first-layer outputs, slot rows out
// (plain, or added into the token rows), and one element of the dh epilogue.
// Both cores' kernels call these, so that they return the same bits.
#pragma once

#include "common.hpp"
#include "gemm.hpp"
#include "gemm_rs.hpp"

namespace moe {

__device__ __forceinline__ float silu_bf(float a) { return a * sigmoidf_(a); }

// Expert activation: SwiGLU (gated, Section 5.1) or the non-gated SiLU / ReLU
// experts of Section 2.2, E(x) = W2 act(W1 x), whose only saved activation is
// A = x W1. ReLU'(0) is taken as 0.
enum : int { ACT_SWIGLU = 0, ACT_SILU = 1, ACT_RELU = 2 };
template <int ACT>
__device__ __forceinline__ float act_f(float a) {
    if constexpr (ACT == ACT_RELU) return a > 0.f ? a : 0.f;
    else return a * sigmoidf_(a);
}
template <int ACT>
__device__ __forceinline__ float act_d(float a) {
    if constexpr (ACT == ACT_RELU) return a > 0.f ? 1.f : 0.f;
    else {
        const float sg = sigmoidf_(a);
        return sg * (1.0f + a * (1.0f - sg));
    }
}
__device__ __forceinline__ void store8_bf16(bf16_t* p, const float (&v)[8]) { st16(p, pack8(v)); }

// A (and B, H) rows of a first-layer tile from its accumulators
template <int ACT, class C>
__device__ __forceinline__ void first_rows_out(const rs::Acc<C>& acc, const SlotTile& t, int f,
                                               bf16_t* __restrict__ A, bf16_t* __restrict__ B,
                                               bf16_t* __restrict__ H) {
    WaveCoord<C> wc;
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
        const int m = wc.row(i);
        if (m >= t.mrows) continue;
        const int64_t s = (int64_t)t.off + t.m0 + m;
#pragma unroll
        for (int j = 0; j < C::FN; ++j) {
            float va[2][8], vb[2][8];
            frag_cols8(acc[0][i][j], va);
            if constexpr (ACT == ACT_SWIGLU) frag_cols8(acc[1][i][j], vb);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int n = t.n0 + wc.col8(j, p);
                if (n >= f) continue;
                float a[8], b[8], h[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    a[r] = bf2f(f2bf(va[p][r]));
                    if constexpr (ACT == ACT_SWIGLU) {
                        b[r] = bf2f(f2bf(vb[p][r]));
                        h[r] = silu_bf(a[r]) * b[r];
                    } else {
                        h[r] = act_f<ACT>(a[r]);
                    }
                }
                store8_bf16(A + s * f + n, a);
                if constexpr (ACT == ACT_SWIGLU) store8_bf16(B + s * f + n, b);
                if (H) store8_bf16(H + s * f + n, h);
            }
        }
    }
}

// Output rows of a slot tile (G2, G6), columns n < ncols of the tile's strip:
// slot row s goes to row s of O, rows ldo apart.
template <class C>
__device__ __forceinline__ void slot_rows_out(const rs::Acc<C>& acc, const SlotTile& t,
                                              int ncols, int64_t ldo, bf16_t* __restrict__ O) {
    WaveCoord<C> wc;
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
        const int m = wc.row(i);
        if (m >= t.mrows) continue;
        const int64_t s = (int64_t)t.off + t.m0 + m;
#pragma unroll
        for (int j = 0; j < C::FN; ++j) {
            float v[2][8];
            frag_cols8(acc[0][i][j], v);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int n = t.n0 + wc.col8(j, p);
                if (n < ncols) store8_bf16(O + s * ldo + n, v[p]);
            }
        }
    }
}

// The combine folded into the epilogue (Section 3.1): slot row s of the tile,
// times gs[s] (1 when gs is null), rounded to bf16, is added into row tok[s]
// of O (rows ldo apart) by packed-bf16 atomics, so that O receives the sum
// over a token's slots in whatever order the tiles finish. The tile goes
// through LDS first (free once the main loop is done), so that each atomic
// instruction of a wave covers 256 contiguous bytes of one row (two rows of 128
// in 64-column tiles): 64 lanes, two columns each (straight from the fragments, a wave's atomics would touch 32
// rows 16 bytes apiece). 16-byte chunks are XOR-swizzled by row, so that both
// the fragment-ordered writes and the row-ordered reads are free of bank
// conflicts.
template <class C>
__device__ __forceinline__ void slot_rows_scatter(const rs::Acc<C>& acc, const SlotTile& t,
                                                  int ncols, int64_t ldo,
                                                  bf16_t* __restrict__ O,
                                                  const int32_t* __restrict__ tok,
                                                  const float* __restrict__ gs, char* lds) {
    constexpr int RB = C::BN * 2;      // bytes per tile row in LDS
    constexpr int CPR = C::BN / 8;     // 16-byte chunks per row
    constexpr int SWZ = (CPR < 32 ? CPR : 32) - 1;
    constexpr int LPR = CPR < 16 ? CPR * 4 : WAVE;   // lanes per row
    constexpr int RPI = WAVE / LPR;                  // rows per atomic instruction
    static_assert(C::BM * RB <= C::LDS && (C::BN % 128 == 0 || C::BN == 64), "scatter staging");
    const WaveCoord<C> wc;
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
        const int m = wc.row(i);
        const float g = (gs && m < t.mrows) ? gs[(int64_t)t.off + t.m0 + m] : 1.0f;
#pragma unroll
        for (int j = 0; j < C::FN; ++j) {
            float v[2][8];
            frag_cols8(acc[0][i][j], v);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
#pragma unroll
                for (int r = 0; r < 8; ++r) v[p][r] *= g;
                const int chunk = (wc.col8(j, p) >> 3) ^ (m & SWZ);
                *reinterpret_cast<uint4*>(lds + m * RB + chunk * 16) = pack8(v[p]);
            }
        }
    }
    __syncthreads();
    const int wv = wave_id();
    const int rows = min(C::BM, t.mrows);
    for (int r0 = wv * RPI; r0 < rows; r0 += C::NW * RPI) {
        const int r = RPI == 1 ? r0 : r0 + wc.lane / LPR;
        if (RPI > 1 && r >= rows) continue;
        bf16_t* dst = O + (int64_t)tok[(int64_t)t.off + t.m0 + r] * ldo + t.n0;
#pragma unroll
        for (int c = 0; c < (C::BN + 127) / 128; ++c) {
            const int col = c * 128 + 2 * (wc.lane % LPR);
            if (t.n0 + col >= ncols) continue;
            const int chunk = (col >> 3) ^ (r & SWZ);
            const uint32_t v =
                *reinterpret_cast<const uint32_t*>(lds + r * RB + chunk * 16 + (col & 7) * 2);
            __builtin_amdgcn_global_atomic_fadd_v2bf16(reinterpret_cast<bf16x2_t*>(dst + col),
                                                       __builtin_bit_cast(bf16x2_t, v));
        }
    }
}

// slot rows out, plain or (SCATTER) added into the token rows
template <bool SCATTER, class C>
__device__ __forceinline__ void slot_rows(const rs::Acc<C>& acc, const SlotTile& t, int ncols,
                                          int64_t ldo, bf16_t* __restrict__ O,
                                          const int32_t* __restrict__ tok,
                                          const float* __restrict__ gs, char* lds) {
    if constexpr (SCATTER) slot_rows_scatter<C>(acc, t, ncols, ldo, O, tok, gs, lds);
    else slot_rows_out<C>(acc, t, ncols, ldo, O);
}

// h of one element from its (bf16-valued) A and B: the arithmetic of G1's
// epilogue, on the same values, so the result is bit-identical to the
// buffered h. Non-gated: act(A), B unused. With a gate g: g * h, the
// arithmetic of G4's epilogue for the dW2 GEMM's operand.
template <int ACT, bool GATE>
__device__ __forceinline__ float h_one(float a, float b, float g) {
    float h;
    if constexpr (ACT == ACT_SWIGLU) h = silu_bf(a) * b;
    else h = act_f<ACT>(a);
    if constexpr (GATE) h = g * h;
    return h;
}
// One element of G4's epilogue from u = (dY W2^T), its A and B and the gate:
// dA, dB, g * h, and u * h added to the gate gradient (in: the column exists).
template <int ACT>
__device__ __forceinline__ void dact_one(float u, float a, float b, float g, bool in, float& da,
                                         float& db, float& hg, float& dg) {
    const float dh = g * u;
    float h;
    if constexpr (ACT == ACT_SWIGLU) {
        const float sg = sigmoidf_(a);
        const float sl = a * sg;
        h = sl * b;
        da = dh * b * sg * (1.0f + a * (1.0f - sg));
        db = dh * sl;
    } else {
        h = act_f<ACT>(a);
        da = dh * act_d<ACT>(a);
    }
    dg += in ? u * h : 0.f;
    hg = g * h;
}

}  // namespace moe
