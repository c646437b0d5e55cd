// ffn_small.hip -- the row-wise grouped GEMMs of the expert FFN (G1, G2, G4, G6
// of ffn.hip) for few rows per expert: decoding, small batches and
// micro-batches, where reading the expert weights once is the bound. The core
// is gemm_sk.hpp; loaders, epilogues and MFMA order give the same bits as the
// 256-row kernels of ffn.hip, so a token's results do not depend on which of
// them a batch size selects.
//
// One layer forward with E = 64, d = 2048, f = 1408, k = 6: first GEMM with one
// token 44 -> 18 us, with 48 tokens (all 64 experts, 739 MB of weights) 149 ->
// 124 us, that is 6.0 TB/s (kernel trace: 126, 121 at best). E = 128, d = f = 2880, 300
// tokens (4.2 GB): 808 -> 696 us. The rule that chooses between the cores, with
// both sides measured, is at small_wide_n and its neighbours in ffn.hip.
#include "common.hpp"
#include "ffn_epi.hpp"
#include "gemm.hpp"
#include "gemm_rs.hpp"
#include "gemm_sk.hpp"
#include "launch.hpp"
#include "probe.hpp"

namespace moe {
namespace {

// Tile configurations <BM, BN, WM, WN, NB, NST, NLA> by rows per tile and by
// column level. D: two right operands (W1 and W3), BN columns of each. S: one
// right operand. H: one right operand, A and B on the left, h formed in LDS.
// (32-row tiles gained nothing over 64-row ones but where h is formed, whose
// vector work grows with the rows.)
// Levels: WIDE reads the longest weight rows and is the best where its tiles
// fill the chip; NARROW and SLIM halve the columns where they do not, and spend
// the LDS on a deeper ring instead (one workgroup per CU).
enum : int { WIDE = SMALL_WIDE, NARROW = SMALL_NARROW, SLIM = SMALL_SLIM };
template <int BM, int LV> struct Sk;
template <> struct Sk<32, WIDE> { using H = sk::Cfg<32, 256, 1, 4, 1, 4, 2>; };
template <> struct Sk<32, NARROW> { using H = sk::Cfg<32, 128, 1, 4, 1, 6, 2>; };
template <> struct Sk<32, SLIM> { using H = sk::Cfg<32, 64, 1, 2, 1, 8, 2>; };
template <> struct Sk<64, WIDE> {
    using D = sk::Cfg<64, 128, 2, 4, 2, 4>;
    using S = sk::Cfg<64, 256, 2, 4, 1, 4>;
    using H = sk::Cfg<64, 256, 2, 4, 1, 3, 2>;
};
template <> struct Sk<64, NARROW> {
    using D = sk::Cfg<64, 64, 2, 2, 2, 6>;
    using S = sk::Cfg<64, 128, 2, 2, 1, 6>;
    using H = sk::Cfg<64, 128, 2, 2, 1, 5, 2>;
};
template <> struct Sk<64, SLIM> {
    using S = sk::Cfg<64, 64, 2, 2, 1, 8>;
    using H = sk::Cfg<64, 64, 2, 2, 1, 6, 2>;
};
template <> struct Sk<128, WIDE> {
    using D = sk::Cfg<128, 128, 2, 4, 2, 3>;
    using S = sk::Cfg<128, 256, 2, 4, 1, 3>;
};
template <> struct Sk<128, NARROW> {
    using D = sk::Cfg<128, 64, 2, 2, 2, 5>;
    using S = sk::Cfg<128, 128, 2, 2, 1, 5>;
};
template <int ACT, class K>
using SkFirst = std::conditional_t<ACT == ACT_SWIGLU, typename K::D, typename K::S>;

constexpr int SK_GM = 4;   // row tiles per raster group: they share a weight panel in L2

template <class C>
__device__ __forceinline__ bool tile_of(char* lds, const int32_t* offsets, int E, int ncols,
                                        SlotTile& t) {
    return find_slot_tile<C::THREADS>(reinterpret_cast<int*>(lds), offsets, E, C::BM,
                                      (ncols + C::BN - 1) / C::BN, blockIdx.x, C::BN, t, SK_GM);
}

// G1: A = x[eti] W1[e], B = x[eti] W3[e] (non-gated: A alone), h into H if given
template <int ACT, class K>
__global__ void __launch_bounds__((SkFirst<ACT, K>::THREADS))
sk_g1(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w1, const bf16_t* __restrict__ w3,
      const int32_t* __restrict__ offsets, const int32_t* __restrict__ eti, int d, int f, int E,
      bf16_t* __restrict__ A, bf16_t* __restrict__ B, bf16_t* __restrict__ H) {
    extern __shared__ __align__(16) char lds[];
    using C = SkFirst<ACT, K>;
    SlotTile t;
    if (!tile_of<C>(lds, offsets, E, f, t)) return;
    sk::KCSrc<C, C::BM, C::NCA> la;
    const int32_t* idx = eti + t.off + t.m0;
    la.init([&](int r) { return x + (int64_t)idx[r < t.mrows ? r : 0] * d; });
    sk::MCSrc<C, C::BN, C::NCB> lb[C::NB];
    lb[0].init(w1 + (int64_t)t.e * d * f, f, t.n0, f);
    if constexpr (C::NB == 2) lb[C::NB - 1].init(w3 + (int64_t)t.e * d * f, f, t.n0, f);
    rs::Acc<C> acc;
    auto issue = [&](int, uint32_t dst) __attribute__((always_inline)) {
        la.issue(dst);
#pragma unroll
        for (int b = 0; b < C::NB; ++b) lb[b].issue(dst + C::A_BYTES + b * C::B_BYTES);
    };
    sk::mainloop<C, true>(issue, sk::NoXform{}, d / sk::KS, lds, acc);
    first_rows_out<ACT, C>(acc, t, f, A, B, H);
}

// h = act(A) * B of the chunks this lane copied, in place of A's (rows past the
// tile's are left as they are: their outputs are not stored)
template <int ACT, class C>
struct HXform {
    static constexpr bool ON = true;
    int mrows;
    __device__ void operator()(char* stage, int) const {
#pragma unroll
        for (int c = 0; c < C::NCA; ++c) {
            if (sk::KCSrc<C, C::BM, C::NCA>::row(c) >= mrows) continue;
            char* p = stage + (wave_id() + c * C::NW) * 1024 + (threadIdx.x & 63) * 16;
            float a[8], b[8], h[8];
            unpack8(*reinterpret_cast<const uint4*>(p), a);
            if constexpr (ACT == ACT_SWIGLU) unpack8(*reinterpret_cast<const uint4*>(p + C::A_BYTES), b);
#pragma unroll
            for (int r = 0; r < 8; ++r) h[r] = h_one<ACT, false>(a[r], b[r], 0.f);
            *reinterpret_cast<uint4*>(p) = pack8(h);
        }
    }
};

// G2: O = h W2[e], output columns [n_base, n_base + ncols) of W2. FORM_H: h is
// formed from A (and B) in LDS; otherwise A is the h buffer. SCATTER: added
// into the token rows (slot_rows_scatter).
template <class H>   // the same tile without a second left array (non-gated)
using OneLeft = sk::Cfg<H::BM, H::BN, H::WM, H::WN, 1, H::NST, 1>;
template <int ACT, bool FORM_H, class K>
struct SecondCfg { using T = typename K::S; };
template <int ACT, class K>
struct SecondCfg<ACT, true, K> {
    using T = std::conditional_t<ACT == ACT_SWIGLU, typename K::H, OneLeft<typename K::H>>;
};
template <int ACT, bool FORM_H, class K>
using SkSecond = typename SecondCfg<ACT, FORM_H, K>::T;
template <int ACT, bool FORM_H, bool SCATTER, class K>
__global__ void __launch_bounds__((SkSecond<ACT, FORM_H, K>::THREADS))
sk_g2(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, const bf16_t* __restrict__ w2,
      const int32_t* __restrict__ offsets, int d, int f, int E, int n_base, int ncols,
      int64_t ldo, bf16_t* __restrict__ O, const int32_t* __restrict__ tok,
      const float* __restrict__ gs) {
    extern __shared__ __align__(16) char lds[];
    using C = SkSecond<ACT, FORM_H, K>;
    SlotTile t;
    if (!tile_of<C>(lds, offsets, E, ncols, t)) return;
    const int64_t row0 = (int64_t)t.off + t.m0;
    sk::KCSrc<C, C::BM, C::NCA> la[C::NLA];
    la[0].init([&](int r) { return A + (row0 + (r < t.mrows ? r : 0)) * f; });
    if constexpr (C::NLA == 2)
        la[C::NLA - 1].init([&](int r) { return B + (row0 + (r < t.mrows ? r : 0)) * f; });
    sk::MCSrc<C, C::BN, C::NCB> lb;
    lb.init(w2 + (int64_t)t.e * f * d, d, n_base + t.n0, n_base + ncols);
    rs::Acc<C> acc;
    auto issue = [&](int, uint32_t dst) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < C::NLA; ++u) la[u].issue(dst + u * C::A_BYTES);
        lb.issue(dst + C::NLA * C::A_BYTES);
    };
    if constexpr (FORM_H)
        sk::mainloop<C, true>(issue, HXform<ACT, C>{t.mrows}, f / sk::KS, lds, acc);
    else
        sk::mainloop<C, true>(issue, sk::NoXform{}, f / sk::KS, lds, acc);
    slot_rows<SCATTER, C>(acc, t, ncols, ldo, O, tok, gs, lds);
}

// G4: u = dY[eti] W2[e]^T; epilogue as g4_kernel's. gs: gates in slot order
// (HG_OUT false), else gathered through slot_src, and g*h written to HG.
template <int ACT, bool HG_OUT, class K>
__global__ void __launch_bounds__((K::S::THREADS))
sk_g4(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ w2, const float* __restrict__ gates,
      const int32_t* __restrict__ offsets, const int32_t* __restrict__ eti,
      const int32_t* __restrict__ slot_src, const float* __restrict__ gs, int d, int f, int E,
      int nparts, bf16_t* __restrict__ A, bf16_t* __restrict__ B, bf16_t* __restrict__ HG,
      float* __restrict__ part) {
    extern __shared__ __align__(16) char lds[];
    using C = typename K::S;
    static_assert(C::WTN == 64, "a gate-gradient partial covers 64 columns");
    SlotTile t;
    if (!tile_of<C>(lds, offsets, E, f, t)) return;
    const WaveCoord<C> wc;
    const int64_t row0 = (int64_t)t.off + t.m0;
    float gr[C::FM];
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
        const int64_t s = row0 + (wc.row(i) < t.mrows ? wc.row(i) : 0);
        gr[i] = HG_OUT ? gates[slot_src[s]] : gs[s];
    }
    sk::KCSrc<C, C::BM, C::NCA> la;
    const int32_t* idx = eti + row0;
    la.init([&](int r) { return dy + (int64_t)idx[r < t.mrows ? r : 0] * d; });
    sk::KCSrc<C, C::BN, C::NCB> lb;   // rows n of W2[e] ([f][d]), K = d
    const bf16_t* W2e = w2 + (int64_t)t.e * f * d;
    lb.init([&](int r) { return W2e + (int64_t)min(t.n0 + r, f - 1) * d; });
    rs::Acc<C> acc;
    auto issue = [&](int, uint32_t dst) __attribute__((always_inline)) {
        la.issue(dst);
        lb.issue(dst + C::A_BYTES);
    };
    sk::mainloop<C, false>(issue, sk::NoXform{}, d / sk::KS, lds, acc);
    const int pidx = t.n0 / 64 + wc.wn;
    const bool last = t.n0 + C::BN >= f;   // this tile also clears the partials past f
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
        const int m = wc.row(i);
        const bool valid = m < t.mrows;
        const int64_t s = row0 + (valid ? m : 0);
        float dg = 0.f;
#pragma unroll
        for (int j = 0; j < C::FN; ++j) {
            float u8[2][8];
            frag_cols8(acc[0][i][j], u8);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int n = t.n0 + wc.col8(j, p);
                const int nc = min(n, f - 8);
                float a[8], b[8], da[8], db[8], hg[8];
                unpack8(ld16(A + s * f + nc), a);
                if constexpr (ACT == ACT_SWIGLU) unpack8(ld16(B + s * f + nc), b);
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    dact_one<ACT>(u8[p][r], a[r], b[r], gr[i], n < f, da[r], db[r], hg[r], dg);
                if (valid && n < f) {
                    store8_bf16(A + s * f + n, da);
                    if constexpr (ACT == ACT_SWIGLU) store8_bf16(B + s * f + n, db);
                    if constexpr (HG_OUT) store8_bf16(HG + s * f + n, hg);
                }
            }
        }
        dg += __shfl_xor(dg, 32, 64);
        if (valid && wc.lane < 32) {
            part[s * nparts + pidx] = dg;
            if (last && wc.wn == 0)
                for (int p = t.n0 / 64 + C::WN; p < nparts; ++p) part[s * nparts + p] = 0.f;
        }
    }
}

// G6: dX_slot = dA W1[e]^T + dB W3[e]^T, output columns [n_base, n_base +
// ncols); kst slices of K from dA and W1, then those of dB and W3
template <bool SCATTER, class K>
__global__ void __launch_bounds__(K::S::THREADS)
sk_g6(const bf16_t* __restrict__ dA, const bf16_t* __restrict__ dB, const bf16_t* __restrict__ w1,
      const bf16_t* __restrict__ w3, const int32_t* __restrict__ offsets, int d, int f, int E,
      int kslices, int n_base, int ncols, int64_t ldo, bf16_t* __restrict__ dX,
      const int32_t* __restrict__ tok) {
    extern __shared__ __align__(16) char lds[];
    using C = typename K::S;
    SlotTile t;
    if (!tile_of<C>(lds, offsets, E, ncols, t)) return;
    const int64_t row0 = (int64_t)t.off + t.m0;
    sk::KCSrc<C, C::BM, C::NCA> la;
    la.init([&](int r) { return dA + (row0 + (r < t.mrows ? r : 0)) * f; });
    sk::KCSrc<C, C::BN, C::NCB> lb;   // rows n of W1[e] / W3[e] ([d][f])
    const bf16_t* W1e = w1 + (int64_t)t.e * d * f;
    lb.init([&](int r) { return W1e + (int64_t)(n_base + min(t.n0 + r, ncols - 1)) * f; });
    const int kst = f / sk::KS;
    rs::Acc<C> acc;
    auto issue = [&](int s, uint32_t dst) __attribute__((always_inline)) {
        if (s == kst) {
            la.jump((dB - dA) - f);
            lb.jump((w3 - w1) - f);
        }
        la.issue(dst);
        lb.issue(dst + C::A_BYTES);
    };
    sk::mainloop<C, false>(issue, sk::NoXform{}, kslices, lds, acc);
    slot_rows<SCATTER, C>(acc, t, ncols, ldo, dX, tok, nullptr, lds);
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// launch with C's LDS (limit raised once per kernel) over the worst-case tiles
template <class C, auto KERNEL, class... Args>
hipError_t launch(const char* name, int64_t S, int E, int ncols, hipStream_t st, Args... args) {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (attr != hipSuccess) return attr;
    const unsigned grid = (unsigned)(((S + C::BM - 1) / C::BM + (S < E ? S : E)) * cdiv(ncols, C::BN));
    hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(C::THREADS), C::LDS, st, args...);
    probe::mark(name, st);
    return hipGetLastError();
}

template <int ACT, class K>
hipError_t first(const FfnArgs& a, void* H, hipStream_t st) {
    return launch<SkFirst<ACT, K>, sk_g1<ACT, K>>(
        "sk_g1", a.T * a.k, a.E, a.f, st, (const bf16_t*)a.x, (const bf16_t*)a.w1,
        (const bf16_t*)a.w3, a.offsets, a.eti, a.d, a.f, a.E, (bf16_t*)a.A, (bf16_t*)a.B,
        (bf16_t*)H);
}

template <int ACT, bool FORM_H, bool SCATTER, class K>
hipError_t second(const FfnArgs& a, const void* left, int c0, int nc, int64_t ldo, void* out,
                  const float* gs, hipStream_t st) {
    return launch<SkSecond<ACT, FORM_H, K>, sk_g2<ACT, FORM_H, SCATTER, K>>(
        FORM_H ? "sk_g2h" : "sk_g2", a.T * a.k, a.E, nc, st, (const bf16_t*)left,
        (const bf16_t*)a.B, (const bf16_t*)a.w2, a.offsets, a.d, a.f, a.E, c0, nc, ldo,
        (bf16_t*)out, a.eti, gs);
}

template <int ACT, bool HG_OUT, class K>
hipError_t dact(const FfnArgs& a, const float* gs, void* HG, float* part, int nparts,
                hipStream_t st) {
    return launch<typename K::S, sk_g4<ACT, HG_OUT, K>>(
        "sk_g4", a.T * a.k, a.E, a.f, st, (const bf16_t*)a.dy, (const bf16_t*)a.w2, a.gates,
        a.offsets, a.eti, a.slot_src, gs, a.d, a.f, a.E, nparts, (bf16_t*)a.A, (bf16_t*)a.B,
        (bf16_t*)HG, part);
}

template <bool SCATTER, class K>
hipError_t dx(const FfnArgs& a, int c0, int nc, int64_t ldo, void* out, hipStream_t st) {
    const bool gated = a.act == ACT_SWIGLU;
    const void* B = gated ? a.B : a.A;
    const void* w3 = gated ? a.w3 : a.w1;
    return launch<typename K::S, sk_g6<SCATTER, K>>(
        "sk_g6", a.T * a.k, a.E, nc, st, (const bf16_t*)a.A, (const bf16_t*)B,
        (const bf16_t*)a.w1, (const bf16_t*)w3, a.offsets, a.d, a.f, a.E,
        (gated ? 2 : 1) * a.f / sk::KS, c0, nc, ldo, (bf16_t*)out, a.eti);
}

// f(integral_constant<int, v>) for the value v of a runtime choice
template <int... V, class F>
hipError_t pick(int v, F&& f) {
    hipError_t r = hipErrorInvalidValue;
    (void)((v == V ? (r = f(std::integral_constant<int, V>{}), true) : false) || ...);
    return r;
}

// f(Sk<BM, LV>{}) for the tile configuration of v (SLIM: a narrow tile where
// there is no slim one)
template <bool HAS_SLIM, int... BM, class F>
hipError_t pick_tile(const SmallTile& v, F&& f) {
    return pick<BM...>(v.rows, [&](auto b) {
        constexpr int R = decltype(b)::value;
        if (v.level == WIDE) return f(Sk<R, WIDE>{});
        if constexpr (HAS_SLIM && R < 128) {
            if (v.level == SLIM) return f(Sk<R, SLIM>{});
        }
        return f(Sk<R, NARROW>{});
    });
}

}  // namespace

hipError_t small_first(const FfnArgs& a, SmallTile v, void* H, hipStream_t st) {
    return pick<ACT_SWIGLU, ACT_SILU, ACT_RELU>(a.act, [&](auto act) {
        return pick_tile<false, 64, 128>(v, [&](auto k) {
            return first<decltype(act)::value, decltype(k)>(a, H, st);
        });
    });
}

hipError_t small_second(const FfnArgs& a, SmallTile v, const void* H, int c0, int nc, int64_t ldo,
                        void* out, const float* gs, hipStream_t st) {
    if (H)   // (the activation plays no part)
        return pick_tile<true, 64, 128>(v, [&](auto k) {
            using K = decltype(k);
            return gs ? second<ACT_RELU, false, true, K>(a, H, c0, nc, ldo, out, gs, st)
                      : second<ACT_RELU, false, false, K>(a, H, c0, nc, ldo, out, gs, st);
        });
    return pick<ACT_SWIGLU, ACT_SILU, ACT_RELU>(a.act, [&](auto act) {
        return pick_tile<true, 32, 64>(v, [&](auto k) {
            constexpr int ACT = decltype(act)::value;
            using K = decltype(k);
            return gs ? second<ACT, true, true, K>(a, a.A, c0, nc, ldo, out, gs, st)
                      : second<ACT, true, false, K>(a, a.A, c0, nc, ldo, out, gs, st);
        });
    });
}

hipError_t small_dact(const FfnArgs& a, SmallTile v, const float* gs, void* HG, float* part,
                      int nparts, hipStream_t st) {
    return pick<ACT_SWIGLU, ACT_SILU, ACT_RELU>(a.act, [&](auto act) {
        return pick_tile<false, 64, 128>(v, [&](auto k) {
            constexpr int ACT = decltype(act)::value;
            using K = decltype(k);
            return HG ? dact<ACT, true, K>(a, gs, HG, part, nparts, st)
                      : dact<ACT, false, K>(a, gs, HG, part, nparts, st);
        });
    });
}

hipError_t small_dx(const FfnArgs& a, SmallTile v, int c0, int nc, int64_t ldo, void* out,
                    bool scatter, hipStream_t st) {
    return pick_tile<true, 64, 128>(v, [&](auto k) {
        using K = decltype(k);
        return scatter ? dx<true, K>(a, c0, nc, ldo, out, st) : dx<false, K>(a, c0, nc, ldo, out, st);
    });
}

}  // namespace moe
