// gemm_sk.hpp -- grouped bf16 MFMA GEMM core for few rows per expert (gfx950).
//
// With a few dozen rows per expert a grouped GEMM is bound by reading the
// expert weights once from HBM: a tile of BM rows does BM multiply-adds per
// weight element, and the matrix cores keep up with about 6 TB/s of weights up
// to 128 rows. The 256-row core (gemm_rs.hpp) computes its padding rows and
// holds 2 slices of one workgroup per CU in flight, which leaves HBM idle
// there. This core is built around the weight stream instead:
//  * row tiles of 32, 64 or 128 rows and column tiles of 64 to 256, so that
//    even a single token's handful of experts gives enough workgroups;
//  * operands come by direct-to-LDS copies into a ring of NST slices of 64 k
//    (no registers hold data in flight), one workgroup per CU with 80 to 140 KB
//    on their way at any time. Where only one round of tiles runs, a slice
//    takes its latency over the ring's depth: tiles of half the columns and
//    twice the depth took 0.73 us a slice against 0.89 (64 rows, 256 and 128
//    workgroups);
//  * one barrier per slice.
// The LDS layouts, the fragment reads and the order of the MFMAs over K are
// those of gemm_rs.hpp, so that every output has the same bits in both cores.
#pragma once

#include "gemm.hpp"
#include "gemm_rs.hpp"

namespace moe {
namespace sk {

using rs::KS;
using rs::KSTEPS;

// BM x BN tile of NB right operands, WM x WN waves, NST ring slices. NLA: left
// arrays per slice (2: A and B, from which h is formed in LDS).
template <int BM_, int BN_, int WM_, int WN_, int NB_, int NST_, int NLA_ = 1>
struct Cfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NB = NB_, NST = NST_, NLA = NLA_;
    static constexpr int NW = WM * WN;
    static constexpr int THREADS = NW * WAVE;
    static constexpr int WTM = BM / WM, WTN = BN / WN;
    static constexpr int FM = WTM / 32, FN = WTN / 32;
    static constexpr int A_BYTES = BM * KS * 2;
    static constexpr int B_BYTES = BN * KS * 2;
    static constexpr int STAGE = NLA * A_BYTES + NB * B_BYTES;
    static constexpr int LDS = NST * STAGE;
    static constexpr int NCA = A_BYTES / 1024 / NW;   // 1 KB copies per wave and left array
    static constexpr int NCB = B_BYTES / 1024 / NW;   // ... and right operand
    static constexpr int PER = NLA * NCA + NB * NCB;  // copies per wave and slice
    static_assert(FM >= 1 && FN >= 1 && NCA >= 1 && NCB >= 1, "wave tile, copies");
    static_assert(A_BYTES % (1024 * NW) == 0 && B_BYTES % (1024 * NW) == 0, "even split");
    static_assert(NST >= 2 && LDS <= 160 * 1024, "ring");
    static_assert(PER * (NST - 2) < 64, "wait count");
};

// ---- operand sources -------------------------------------------------------------------
// A source holds one global pointer per copy of this lane (the 16 bytes that
// land at the lane's place of the copy) and advances it slice by slice. Copy c
// of wave w is copy w + c * NW of the operand tile. Slices are issued in order.

// K-contiguous rows: copy q covers tile rows 8q .. 8q+7, lane l the chunk that
// the layout keeps at physical chunk l % 8 of row 8q + l / 8.
template <class C, int R, int NC>
struct KCSrc {
    static constexpr bool MC = false;
    const bf16_t* p[NC];
    __device__ static int row(int c) { return (wave_id() + c * C::NW) * 8 + ((threadIdx.x & 63) >> 3); }
    __device__ static int chunk(int r) { return (threadIdx.x & 7) ^ ((r >> 1) & 7); }
    // rowptr(r): start of tile row r in K (any valid row for rows past the tile's)
    template <class F>
    __device__ void init(F&& rowptr) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int r = row(c);
            p[c] = rowptr(r) + chunk(r) * 8;
        }
    }
    __device__ void issue(uint32_t dst) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            dma16(p[c], dst + (wave_id() + c * C::NW) * 1024);
            p[c] += KS;
        }
    }
    // continue in another matrix (K split over two sources)
    __device__ void jump(int64_t delta) {
#pragma unroll
        for (int c = 0; c < NC; ++c) p[c] += delta;
    }
};

// Dense row-major [K][ld] matrix, columns n0 .. n0 + R (clamped below ncols):
// copy q covers 1024 / (2R) k rows.
template <class C, int R, int NC>
struct MCSrc {
    static constexpr bool MC = true;
    const bf16_t* p[NC];
    int64_t step;   // elements per slice
    __device__ void init(const bf16_t* W, int ld, int n0, int ncols) {
        constexpr int LPR = R / 8;               // lanes per k row
        const int lane = threadIdx.x & 63;
        step = (int64_t)KS * ld;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int k = (wave_id() + c * C::NW) * (64 / LPR) + lane / LPR;
            const int pc = lane % LPR;
            int n = n0 + 8 * ((((pc >> 1) ^ rs::mc_swz<R>(k)) << 1) | (pc & 1));
            n = n < ncols ? n : ncols - 8;
            p[c] = W + (int64_t)k * ld + n;
        }
    }
    __device__ void issue(uint32_t dst) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            dma16(p[c], dst + (wave_id() + c * C::NW) * 1024);
            p[c] += step;
        }
    }
};

struct NoXform {
    static constexpr bool ON = false;
    __device__ void operator()(char*, int) const {}
};

// ---- main loop ---------------------------------------------------------------------------
// issue(s, dst) starts this wave's C::PER copies of slice s into the stage at
// LDS offset dst (left arrays first, then the right operands). xf(stage, s)
// transforms, in place, the left chunks that this very lane copied (XF::ON).
// The fragments of operand b are acc[b]; RMC: layout of the right operands.
// LDS must be free on entry and is free on return.
template <class C, bool RMC, class ISSUE, class XF>
__device__ __forceinline__ void mainloop(ISSUE&& issue, const XF& xf, int nk, char* lds,
                                         rs::Acc<C>& acc) {
#pragma unroll
    for (int b = 0; b < C::NB; ++b)
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int j = 0; j < C::FN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[b][i][j][r] = 0.f;
    constexpr int NST = C::NST;
    const int lane = threadIdx.x & 63;
    const int wv = wave_id();
    const int wm = wv / C::WN, wn = wv % C::WN;
    const uint32_t base = lds_offset(lds);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): only copies are outstanding from here on
    for (int s = 0; s < NST - 1 && s < nk; ++s) issue(s, base + s * C::STAGE);
    int cur = 0, nxt = NST - 1;           // ring positions of slice s and slice s + NST - 1
    for (int s = 0; s < nk; ++s) {
        // this wave's copies of slice s have landed once only later slices' remain
        if (s + NST - 2 < nk) wait_vmcnt<C::PER * (NST - 2)>();
        else wait_vmcnt<0>();
        char* stage = lds + cur * C::STAGE;
        if constexpr (XF::ON) xf(stage, s);
        // every wave's copies (and transforms) are in LDS, and every wave has
        // read slice s - 1, whose place the next copies take
        lds_barrier();
        if (s + NST - 1 < nk) issue(s + NST - 1, base + nxt * C::STAGE);
        const char* right = stage + C::NLA * C::A_BYTES;
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            bf16x8 l[C::FM], r[C::NB][C::FN];
#pragma unroll
            for (int b = 0; b < C::NB; ++b)
#pragma unroll
                for (int j = 0; j < C::FN; ++j)
                    r[b][j] = rs::frag<RMC, C::BN>(right + b * C::B_BYTES, wn * C::WTN + j * 32, kk, lane);
#pragma unroll
            for (int i = 0; i < C::FM; ++i) l[i] = rs::frag_kc(stage, wm * C::WTM + i * 32, kk, lane);
#pragma unroll
            for (int b = 0; b < C::NB; ++b)
#pragma unroll
                for (int i = 0; i < C::FM; ++i)
#pragma unroll
                    for (int j = 0; j < C::FN; ++j)
                        acc[b][i][j] = rs::mfma32x32x16(r[b][j], l[i], acc[b][i][j]);
        }
        cur = cur + 1 == NST ? 0 : cur + 1;
        nxt = nxt + 1 == NST ? 0 : nxt + 1;
    }
    __syncthreads();
}

}  // namespace sk
}  // namespace moe
