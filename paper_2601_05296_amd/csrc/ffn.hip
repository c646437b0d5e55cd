// ffn.hip -- expert FFN of the MoE layer (SwiGLU, or the non-gated SiLU / ReLU
// expert) as grouped GEMMs that read token rows through the dispatch index
// maps (MoEBlaze paper, Section 3 and Section 5, Algorithm 1), bf16 MFMA with
// float32 accumulation on gfx950.
//
// Forward (moe_ffn_fwd):
//   G1  A|B = x[eti] [W1|W3]      x rows gathered on load, both first-layer
//                                 projections from one x tile (Section 5.2);
//                                 A and B are the only saved activations. The
//                                 epilogue also writes h = SiLU(A)*B into a
//                                 transient buffer for G2.
//   G2  O = h W2                  (MOE_H_ON_LOAD: g2h_kernel forms h from A
//                                 and B as it loads them; no h buffer.)
// Backward (moe_ffn_bwd):
//   G4  u = dY[eti] W2^T, then in the epilogue: d_gate partials sum(u*h),
//       dA = g u B SiLU'(A), dB = g u SiLU(A) written over A and B, and g*h
//       into a transient buffer (h recomputed from A and B).
//   G3  dW2 = (g h)^T dY[eti]     dY rows gathered (the expert-summation
//                                 backward of Section 3.2). MOE_H_ON_LOAD:
//                                 g3h_kernel runs before G4 and forms g*h from
//                                 A, B and the gates on load; no g*h buffer.
//   G5  dW1 = x[eti]^T dA, dW3 = x[eti]^T dB   (one x tile, two products)
//   G6  dX_slot = [dA|dB] [W1|W3]^T             (both branches in one K loop)
// The token gradient is then a unit-weight combine (combine.hip). Forming h
// on load costs the second GEMMs a second operand stream and an in-LDS pass
// per K slice; it returns the same bits.
// The combined calls (moe_ffn_fwd_combine / moe_ffn_bwd_combine) run G2 and
// G6 over column strips, each followed by the ordered combine; with
// MOE_ATOMIC_COMBINE they run once, and the epilogue adds each slot row
// (times its gate in the forward) into the token's row of y or dx by
// packed-bf16 atomics (Section 3.1's reduction as the outputs are produced).
//
// Row-wise GEMMs (G1, G2, G4, G6) tile each expert's slot segment; their grid
// is sized for the worst case (S/BM + E tiles per column block) and each
// workgroup finds its (expert, tile) from `offsets` on the device, so nothing
// waits for the host. The weight-gradient GEMMs (G3, G5) have a fixed tile grid
// per expert and loop over the expert's slots as K.
//
// The float32 mode is in ffn_f32.hip.
#include "common.hpp"
#include "ffn_epi.hpp"
#include "gemm.hpp"
#include "gemm_rs.hpp"
#include "launch.hpp"
#include "probe.hpp"

namespace moe {
namespace {

// Tile configurations (gemm_rs.hpp): <BM, BN, WM, WN, NB>. 256-row tiles,
// 2x4 waves. Single right operand: each wave owns 128 x 64 outputs. Two right
// operands (G1: W1 and W3; G5: dA and dB): 128 x 32 of each.
using RD = rs::Cfg<256, 128, 2, 4, 2>;  // G1, G5
using RS = rs::Cfg<256, 256, 2, 4, 1>;  // G2, G3, G6
constexpr int RASTER_GM = 4;            // M tiles per raster group (find_slot_tile)

// tile configuration of the first-layer and dW1 GEMMs: two right operands
// when gated (W1|W3, dA|dB), one otherwise
template <int ACT> using CFirst = std::conditional_t<ACT == ACT_SWIGLU, RD, RS>;
// GEMMs with h (or g*h) formed on load: 128 x 512 tiles, so that each h
// element is formed once per 512 output columns rather than per 256 (forming
// it costs two transcendentals and some ten other vector operations, about
// as much vector-ALU time per slice as the slice's MFMAs take).
using RHW = rs::Cfg<128, 512, 2, 4, 1>;
// Smaller tiles for launches that would leave CUs idle (the choice between them
// and the large ones is at few_tiles): h formed on load in half the rows, and a
// quarter of the weight-gradient tile on four waves, two workgroups per CU.
using RHN = rs::Cfg<64, 512, 1, 8, 1>;
using RDN = rs::Cfg<128, 64, 2, 2, 2>;
using RSN = rs::Cfg<128, 128, 2, 2, 1>;
template <int ACT> using CNarrow = std::conditional_t<ACT == ACT_SWIGLU, RDN, RSN>;
static_assert(RD::THREADS == RS::THREADS && RD::LDS == RS::LDS, "RD and RS launch alike");

// ============================ kernels ==============================================

// G1: A = x[eti] W1[e], B = x[eti] W3[e]; also H = SiLU(A) * B (from the
// bf16-rounded A and B, exactly as the backward recomputes it). Non-gated:
// A = x[eti] W1[e] and H = act(A). H == NULL: A and B only (the backward's
// recompute under the full-recompute policy).
template <int ACT>
__global__ void __launch_bounds__(RD::THREADS)
g1_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w1,
          const bf16_t* __restrict__ w3, const int32_t* __restrict__ offsets,
          const int32_t* __restrict__ eti, int d, int f, int E, bf16_t* __restrict__ A,
          bf16_t* __restrict__ B, bf16_t* __restrict__ H) {
    extern __shared__ __align__(16) char lds[];
    using C = CFirst<ACT>;
    SlotTile t;
    const int NT = (f + C::BN - 1) / C::BN;
    if (!find_slot_tile<C::THREADS>(reinterpret_cast<int*>(lds), offsets, E, C::BM, NT,
                                    blockIdx.x, C::BN, t, RASTER_GM))
        return;
    rs::GatherKC<C, C::BM> la;
    la.init(x, d, eti + t.off + t.m0, t.mrows);
    rs::DenseMC<C, C::BN> lb0;
    lb0.init(w1 + (int64_t)t.e * d * f, f, t.n0, f);
    rs::Acc<C> acc;
    if constexpr (ACT == ACT_SWIGLU) {
        rs::DenseMC<C, C::BN> lb1;
        lb1.init(w3 + (int64_t)t.e * d * f, f, t.n0, f);
        rs::mainloop<C>(la, lb0, lb1, d / rs::KS, lds, acc);
    } else {
        rs::NoLoader nl;
        rs::mainloop<C>(la, lb0, nl, d / rs::KS, lds, acc);
    }
    first_rows_out<ACT, C>(acc, t, f, A, B, H);
}

// G2: O = H W2[e], output columns [n_base, n_base + ncols) of W2 into columns
// [0, ncols) of O, rows ldo apart (SCATTER: added into the token rows, see
// slot_rows_scatter)
template <bool SCATTER>
__global__ void __launch_bounds__(RS::THREADS)
g2_kernel(const bf16_t* __restrict__ H, const bf16_t* __restrict__ w2,
          const int32_t* __restrict__ offsets, int d, int f, int E, int n_base, int ncols,
          int64_t ldo, bf16_t* __restrict__ O, const int32_t* __restrict__ tok,
          const float* __restrict__ gs) {
    extern __shared__ __align__(16) char lds[];
    using C = RS;
    SlotTile t;
    const int NT = (ncols + C::BN - 1) / C::BN;
    if (!find_slot_tile<C::THREADS>(reinterpret_cast<int*>(lds), offsets, E, C::BM, NT,
                                    blockIdx.x, C::BN, t, RASTER_GM))
        return;
    rs::DenseKC2<C, C::BM> la;
    la.init(H, H, f, (int64_t)t.off + t.m0, t.mrows, f);
    rs::DenseMC<C, C::BN> lb;
    lb.init(w2 + (int64_t)t.e * f * d, d, n_base + t.n0, n_base + ncols);
    rs::NoLoader nl;
    rs::Acc<C> acc;
    rs::mainloop<C>(la, lb, nl, f / rs::KS, lds, acc);
    slot_rows<SCATTER, C>(acc, t, ncols, ldo, O, tok, gs, lds);
}

// h of element pair dword p of (va, vb) as two transform pieces of one element
// each: piece 2p forms the low element into hl, piece 2p+1 the high one and
// packs the pair in place of va's dword (pieces of one element keep the
// vector work between two MFMAs short)
template <int ACT, bool GATE, int P>
__device__ __forceinline__ void h_piece(rs::u32x4& va, const rs::u32x4& vb, float g, float& hl) {
    constexpr int q = P >> 1;
    if constexpr ((P & 1) == 0) hl = h_one<ACT, GATE>(bf_lo(va[q]), bf_lo(vb[q]), g);
    else va[q] = pack_bf2(hl, h_one<ACT, GATE>(bf_hi(va[q]), bf_hi(vb[q]), g));
}

// Left operand of the second GEMM with h formed on load: KC tile of h rows
// row0 + r (r < rows, else row0) from the slot-ordered A (and B), h formed in
// registers between the loads and the LDS write (Section 3.1 keeps only the
// first MLP's output; Section 5.2 recomputes the activation).
template <int ACT, class C, int R>
struct HKC {
    static constexpr bool MC = false;
    using G = rs::KCGeom<C, R>;
    static constexpr int NCH = G::NCH;
    static constexpr bool GATED = ACT == ACT_SWIGLU;
    const bf16_t* pa;      // A + row0 * ld + this thread's chunk column
    int64_t dba;           // B - A, in elements
    int ld, rows;
    rs::u32x4 va[NCH], vb[NCH];
    __device__ void init(const bf16_t* A, const bf16_t* B, int ld_, int64_t row0, int rows_) {
        ld = ld_;
        rows = rows_;
        dba = GATED ? B - A : 0;
        pa = A + rs::roff(row0, ld) + G::chunk(0) * 8;
    }
    template <int i> __device__ void load(int kt) {
        int r = G::row(i);
        r = r < rows ? r : 0;
        const bf16_t* q = pa + rs::roff(r, ld) + kt * rs::KS;
        va[i] = rs::ldg16(q);
        if constexpr (GATED) vb[i] = rs::ldg16(q + dba);
    }
    // h of chunk i in place of A's, one element per piece
    static constexpr int NSUB = 8;
    float hl;
    template <int i, int p> __device__ void sub() { h_piece<ACT, false, p>(va[i], vb[i], 0.f, hl); }
    template <int i, bool TAIL> __device__ void store(char* tile) { rs::sts16(tile + G::lds(i), va[i]); }
};

// G2 with h formed on load: O = h W2[e] from the saved A (and B), no h buffer.
template <int ACT, bool SCATTER, class C>
__global__ void __launch_bounds__(C::THREADS)
g2h_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
           const bf16_t* __restrict__ w2, const int32_t* __restrict__ offsets, int d, int f,
           int E, int n_base, int ncols, int64_t ldo, bf16_t* __restrict__ O,
           const int32_t* __restrict__ tok, const float* __restrict__ gs) {
    extern __shared__ __align__(16) char lds[];
    SlotTile t;
    const int NT = (ncols + C::BN - 1) / C::BN;
    if (!find_slot_tile<C::THREADS>(reinterpret_cast<int*>(lds), offsets, E, C::BM, NT,
                                    blockIdx.x, C::BN, t, RASTER_GM))
        return;
    HKC<ACT, C, C::BM> la;
    la.init(A, B, f, (int64_t)t.off + t.m0, t.mrows);
    rs::DenseMC<C, C::BN> lb;
    lb.init(w2 + (int64_t)t.e * f * d, d, n_base + t.n0, n_base + ncols);
    rs::NoLoader nl;
    rs::Acc<C> acc;
    rs::mainloop<C>(la, lb, nl, f / rs::KS, lds, acc);
    slot_rows<SCATTER, C>(acc, t, ncols, ldo, O, tok, gs, lds);
}

// G4: u = dY[eti] W2[e]^T; epilogue: d_gate partials sum(u*h), dA/dB over
// A/B, and HG = g * h (h recomputed from A, B) for G3. Non-gated: dA = g u
// act'(A) over A, h = act(A). gs: the gates in slot order (read when HG_OUT is
// false, i.e. with h on load, where G3 has built them already).
template <int ACT, bool HG_OUT>
__global__ void __launch_bounds__(RS::THREADS)
g4_kernel(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ w2,
          const float* __restrict__ gates, const int32_t* __restrict__ offsets,
          const int32_t* __restrict__ eti, const int32_t* __restrict__ slot_src,
          const float* __restrict__ gs, int d, int f,
          int E, bf16_t* __restrict__ A, bf16_t* __restrict__ B, bf16_t* __restrict__ HG,
          float* __restrict__ part) {
    extern __shared__ __align__(16) char lds[];
    using C = RS;
    SlotTile t;
    const int NT = (f + C::BN - 1) / C::BN;
    if (!find_slot_tile<C::THREADS>(reinterpret_cast<int*>(lds), offsets, E, C::BM, NT,
                                    blockIdx.x, C::BN, t, RASTER_GM))
        return;
    rs::GatherKC<C, C::BM> la;
    la.init(dy, d, eti + t.off + t.m0, t.mrows);
    rs::DenseKC2<C, C::BN> lb;  // rows c of W2[e] ([f][d]), K = d
    const bf16_t* W2e = w2 + (int64_t)t.e * f * d;
    lb.init(W2e, W2e, d, t.n0, min(C::BN, f - t.n0), d);
    rs::NoLoader nl;
    const WaveCoord<C> wc;
    // The gate of this lane's row in every epilogue round. With h on load
    // (no HG output) they stand in slot order already (gs, for G3) and are
    // loaded before the main loop, whose waits cover them. Otherwise they
    // are gathered through slot_src after it. Either way they are waited for
    // (by a wait the compiler sees) before the epilogue's first copy: the
    // compiler does not see the copies, and a load of its own issued after
    // them would end in a wait for everything outstanding, copies included.
    float gr[C::FM];
    auto gate_row = [&](int i) {
        const int m = wc.row(i);
        return (int64_t)t.off + t.m0 + (m < t.mrows ? m : 0);
    };
    if constexpr (!HG_OUT) {
#pragma unroll
        for (int i = 0; i < C::FM; ++i) gr[i] = gs[gate_row(i)];
    }
    rs::Acc<C> acc;
    rs::mainloop<C>(la, lb, nl, d / rs::KS, lds, acc);
    if constexpr (HG_OUT) {
#pragma unroll
        for (int i = 0; i < C::FM; ++i) gr[i] = gates[slot_src[gate_row(i)]];
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    // ---- epilogue, one round per fragment row-block (64 rows of the tile) ----
    // The A and B rows of a round come into LDS by DMA (1 KB copies, many in
    // flight), two LDS buffers deep: the copies of round i+1 are issued as
    // round i starts and land while round i is computed and stored. Every
    // lane reads its values in LDS, writes dA and dB back in place, and the
    // rows then leave LDS as whole 512-byte runs. g*h goes out straight from
    // registers, 16 bytes per lane (staging it through LDS as well took two
    // more barriers per round and spilled registers: 4% slower). 16-byte
    // chunks are XOR-swizzled by row, so the fragment-ordered LDS accesses
    // (32 rows, one column) are conflict-free.
    constexpr int RR = C::WM * 32;       // rows per round
    constexpr int RB = C::BN * 2;        // bytes per row
    constexpr int CPR = RB / 16;         // 16-byte chunks per row (32)
    constexpr int ARR = RR * RB;         // bytes of one array in LDS
    constexpr int NARR = ACT == ACT_SWIGLU ? 2 : 1;   // A, B or A alone
    constexpr int BUF = 2 * ARR;         // one round's buffer (A and B)
    static_assert(CPR == 32 && 2 * BUF <= C::LDS, "G4 staging layout");
    const int nparts = NT * C::WN;
    const int pidx = (t.n0 / C::BN) * C::WN + wc.wn;
    const uint32_t lds_base = lds_offset(lds);
    const int wv = wave_id();
    auto tile_row = [&](int rr, int i) { return (rr / 32) * C::WTM + i * 32 + (rr & 31); };
    // DMA round i's A and B rows into buffer i & 1: copy q covers rows 2q',
    // 2q'+1 of array q / (ARR/1024)
    auto issue_round = [&](int i) {
#pragma unroll
        for (int c = 0; c < NARR * ARR / 1024 / C::NW; ++c) {
            const int q = wv + c * C::NW;
            const int arr = q / (ARR / 1024), qq = q % (ARR / 1024);
            const int rr = 2 * qq + (wc.lane >> 5);
            const int lc = (wc.lane & 31) ^ (rr & 31);
            int m = tile_row(rr, i);
            m = m < t.mrows ? m : 0;
            int n = t.n0 + lc * 8;
            n = n < f ? n : f - 8;
            const bf16_t* src = (arr ? B : A) + ((int64_t)t.off + t.m0 + m) * f + n;
            dma16(src, lds_base + (i & 1) * BUF + arr * ARR + qq * 1024);
        }
    };
    // Stores a round issues after the copies of the next round: the d_gate
    // partial, the dA (dB) row chunks, the g*h chunks.
    constexpr int NSTORE = 1 + NARR * RR * CPR / C::THREADS + (HG_OUT ? 2 * C::FN : 0);
    // In a full tile every one of them is issued by every wave (no lane
    // condition empties a wave's execution mask).
    const bool full = t.mrows >= C::BM && t.n0 + C::BN <= f;
    issue_round(0);
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
        // Round i's rows have landed. The wait counter counts vector-memory
        // operations down in issue order, so in a full tile, once at most
        // NSTORE remain, round i's copies (issued before round i-1's stores)
        // are done and the stores may still be in flight. Otherwise wait for
        // everything. Buffer (i+1) & 1 was last read by round i-1's stores,
        // before its closing barrier.
        if (i > 0 && full) wait_vmcnt<NSTORE>();
        else wait_vmcnt<0>();
        barrier_only();
        if (i + 1 < C::FM) issue_round(i + 1);
        char* const buf = lds + (i & 1) * BUF;
        // this lane's row of the round and its gate
        const int rr = wc.wm * 32 + (wc.lane & 31);
        const int m = wc.row(i);
        const bool valid = m < t.mrows;
        const int64_t s = (int64_t)t.off + t.m0 + (valid ? m : 0);
        const float g = gr[i];
        char* rowA = buf + rr * RB;
        char* rowB = buf + ARR + rr * RB;
        float dg = 0.f;
        uint4 hgv[C::FN][2];
#pragma unroll
        for (int j = 0; j < C::FN; ++j) {
            float u8[2][8];
            frag_cols8(acc[0][i][j], u8);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int cl = wc.col8(j, p);                       // tile column
                const int off = (((cl >> 3) ^ (rr & 31)) << 4);     // swizzled chunk
                const int n = t.n0 + cl;
                float a[8], b[8], da[8], db[8], hg[8];
                unpack8(*reinterpret_cast<const uint4*>(rowA + off), a);
                if constexpr (ACT == ACT_SWIGLU)
                    unpack8(*reinterpret_cast<const uint4*>(rowB + off), b);
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    dact_one<ACT>(u8[p][r], a[r], b[r], g, n < f, da[r], db[r], hg[r], dg);
                }
                *reinterpret_cast<uint4*>(rowA + off) = pack8(da);
                if constexpr (ACT == ACT_SWIGLU) *reinterpret_cast<uint4*>(rowB + off) = pack8(db);
                hgv[j][p] = pack8(hg);
            }
        }
        dg += __shfl_xor(dg, 32, 64);
        if (valid && wc.lane < 32) part[s * nparts + pidx] = dg;
        // rows out of LDS: chunk id -> (array, row, physical chunk)
        auto store_rows = [&](int narr, bf16_t* const* dst) {
#pragma unroll
            for (int ps = 0; ps < narr * RR * CPR / C::THREADS; ++ps) {
                const int cid = ps * C::THREADS + threadIdx.x;
                const int arr = cid / (RR * CPR);
                const int r2 = (cid / CPR) % RR, pc = cid % CPR;
                const int mm = tile_row(r2, i);
                const int n = t.n0 + ((pc ^ (r2 & 31)) << 3);
                const uint4 v = *reinterpret_cast<const uint4*>(buf + arr * ARR + r2 * RB + pc * 16);
                if (mm < t.mrows && n < f) st16_nt(dst[arr] + ((int64_t)t.off + t.m0 + mm) * f + n, v);
            }
        };
        lds_barrier();
        {
            bf16_t* const dst[2] = {A, B};
            store_rows(NARR, dst);
        }
        lds_barrier();
        if constexpr (HG_OUT) {   // false when G3 forms g*h itself (h on load)
            if (valid) {
#pragma unroll
                for (int j = 0; j < C::FN; ++j)
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const int n = t.n0 + wc.col8(j, p);
                        if (n < f) st16(HG + s * f + n, hgv[j][p]);
                    }
            }
        }
    }
}

// Weight gradients are written once and not read again by this layer:
// nontemporal stores keep them from displacing the operands in L2. ADD: the tile
// is added to what the array holds (gradients of several token chunks).
__device__ __forceinline__ void st_nt(float* p, const f32x4& v) {
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p));
}
// the tile at (m0, n0) of M x N outputs; at(b, m, n): their addresses
template <class C, int IPR, bool ADD, class F>
__device__ __forceinline__ void dw_out(const rs::Acc<C>& acc, char* lds, int m0, int n0, int M, int N,
                                       F&& at) {
    if (ADD && m0 + C::BM <= M && n0 + C::BN <= N) {
        RowStage<C, IPR>::add(acc, lds, [&](int b, int r, int c) { return at(b, m0 + r, n0 + c); }, st_nt);
        return;
    }
    RowStage<C, IPR>::run(acc, lds, [&](int b, int r, int c, const f32x4& v) {
        const int m = m0 + r, n = n0 + c;
        if (m >= M || n >= N) return;
        float* p = at(b, m, n);
        st_nt(p, ADD ? v + *reinterpret_cast<const f32x4*>(p) : v);
    });
}

// G3: dW2[e] = sum_s HG[s]^T dY[eti[s]]   (M = f, N = d, K = slots of e)
template <class C, bool ADD>
__global__ void __launch_bounds__(C::THREADS, 2)
g3_kernel(const bf16_t* __restrict__ HG, const bf16_t* __restrict__ dy,
          const ExpertRank* __restrict__ rank, const int32_t* __restrict__ eti, int d, int f,
          float* __restrict__ dw2) {
    extern __shared__ __align__(16) char lds[];
    const int MT = (f + C::BM - 1) / C::BM, NT = (d + C::BN - 1) / C::BN;
    ExpertRank er;
    int mt, nt;
    if (!wgrad_tile(rank, blockIdx.x, MT, NT, er, mt, nt)) return;
    const int e = er.e, off = er.off, cnt = er.cnt;
    const int m0 = mt * C::BM;
    const int n0 = nt * C::BN;
    rs::SlotMC<C, C::BM> la;
    rs::GatherMC<C, C::BN> lb;
    rs::NoLoader nl;
    if (cnt > 0) {
        la.init(HG, f, off, m0, f, cnt);
        lb.init(dy, d, n0, d, eti + off, cnt);
    }
    rs::Acc<C> acc;
    rs::mainloop<C>(la, lb, nl, rs::slices(cnt), lds, acc);
    float* out = dw2 + (int64_t)e * f * d;
    dw_out<C, 1, ADD>(acc, lds, m0, n0, f, d, [&](int, int m, int n) { return out + (int64_t)m * d + n; });
}


// Left operand of the dW2 GEMM with g*h formed on load: MC tile of g*h slot
// rows off + kr (K = the expert's slots) from the saved A (and B) and the
// slot-ordered gates gs. Rows at or past cnt are read from row cnt - 1 and
// stored as zeros.
template <int ACT, class C, int R>
struct GHMC {
    static constexpr bool MC = true;
    using G = rs::MCGeom<C, R>;
    static constexpr int NCH = G::NCH;
    static constexpr bool GATED = ACT == ACT_SWIGLU;
    const bf16_t* pa;      // A + off * ld + this thread's column
    int64_t dba;           // B - A, in elements
    const float* gsp;      // gates of slots off, off + 1, ...
    int ld, cnt;
    uint32_t zmask;
    rs::u32x4 va[NCH], vb[NCH];
    float g[NCH];
    __device__ void init(const bf16_t* A, const bf16_t* B, int ld_, int64_t off, int col0,
                         int ncols, int cnt_, const float* gs) {
        ld = ld_;
        cnt = cnt_;
        zmask = 0;
        dba = GATED ? B - A : 0;
        int c = col0 + G::col(0);
        c = c < ncols ? c : ncols - 8;
        pa = A + rs::roff(off, ld) + c;
        gsp = gs + off;
    }
    template <int i> __device__ void load(int kt) {
        int k = kt * rs::KS + G::krow(i);
        const bool past = k >= cnt;
        zmask = past ? (zmask | (1u << i)) : (zmask & ~(1u << i));
        k = past ? cnt - 1 : k;
        const bf16_t* q = pa + rs::roff(k, ld);
        va[i] = rs::ldg16(q);
        if constexpr (GATED) vb[i] = rs::ldg16(q + dba);
        g[i] = gsp[k];
    }
    // g * h of chunk i in place of A's, one element per piece
    static constexpr int NSUB = 8;
    float hl;
    template <int i, int p> __device__ void sub() { h_piece<ACT, true, p>(va[i], vb[i], g[i], hl); }
    template <int i, bool TAIL> __device__ void store(char* tile) {
        const rs::u32x4 z = {0u, 0u, 0u, 0u};
        if constexpr (TAIL) rs::sts16(tile + G::lds(i), (zmask >> i) & 1 ? z : va[i]);
        else rs::sts16(tile + G::lds(i), va[i]);
    }
};

// The small preparations of the forward's and the backward's GEMMs, each in one
// launch (a launch of their own took 3 to 5 us each, whatever its work).

// p[0..n) = 0 for n bf16 values, n a multiple of 8, p 16-byte aligned (a
// kernel rather than a memset, so that it can be captured in a graph). One store
// per thread over the whole range: a loop over a grid of 2048 workgroups wrote
// 268 MB in 45 us, this in 37.
__device__ __forceinline__ void clear_bf16(bf16_t* __restrict__ p, int64_t n, int64_t i) {
    if (i * 8 < n) st16(p + i * 8, uint4{0u, 0u, 0u, 0u});
}
__global__ void __launch_bounds__(256) zero_bf16(bf16_t* __restrict__ p, int64_t n) {
    clear_bf16(p, n, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// gs[token_index_map[i]] = gates[i] for the accepted choices i < S: the gate of
// each filled slot in slot order, from the token-side map (the forward has no
// slot_src); y[0..n) = 0
__global__ void __launch_bounds__(256)
fwd_prep(const float* __restrict__ gates, const int32_t* __restrict__ tim, int64_t S,
         float* __restrict__ gs, bf16_t* __restrict__ y, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < S) {
        const int32_t s = tim[i];
        if (s >= 0) gs[s] = gates[i];
    }
    clear_bf16(y, n, i);
}

// rank[r] = (expert, first slot, slot count) of the expert of rank r by slot
// count, descending, ties to the lower index: the order in which the
// weight-gradient GEMMs take the experts (wgrad_tile). One thread per expert of
// one workgroup.
__device__ __forceinline__ void expert_ranks(const int32_t* __restrict__ offsets, int E,
                                             ExpertRank* __restrict__ rank) {
    __shared__ int cnt[256];
    const int t = threadIdx.x;
    if (t < E) cnt[t] = offsets[t + 1] - offsets[t];
    __syncthreads();
    if (t >= E) return;
    const int c = cnt[t];
    int r = 0;
    for (int u = 0; u < E; ++u) {
        const int cu = cnt[u];
        r += (cu > c) | ((cu == c) & (u < t));
    }
    rank[r] = ExpertRank{t, offsets[t], c, 0};
}

// Block 0: the experts' order. The others (with gs): gs[s] = gates[slot_src[s]] for
// the filled slots s < offsets[E] and 0 for the rest up to S (the gate of each slot
// in slot order, for the dW2 GEMM's left operand; fewer than S slots are filled
// only when the index build rejected choices)
__global__ void __launch_bounds__(256)
bwd_prep(const float* __restrict__ gates, const int32_t* __restrict__ slot_src,
         const int32_t* __restrict__ offsets, int E, int64_t S, ExpertRank* __restrict__ rank,
         float* __restrict__ gs) {
    if (blockIdx.x == 0) {
        expert_ranks(offsets, E, rank);
        return;
    }
    const int64_t s = (int64_t)(blockIdx.x - 1) * 256 + threadIdx.x;
    if (s < S) gs[s] = s < offsets[E] ? gates[slot_src[s]] : 0.0f;
}

// G3 with g*h formed on load from the saved A (and B) and the slot-ordered
// gates gs: dW2[e] = sum_s (g h)[s]^T dY[eti[s]]. Runs before G4, which then
// writes dA, dB over A, B and no g*h.
template <int ACT, class C, bool ADD>
__global__ void __launch_bounds__(C::THREADS)
g3h_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
           const float* __restrict__ gs, const bf16_t* __restrict__ dy,
           const ExpertRank* __restrict__ rank, const int32_t* __restrict__ eti, int d, int f,
           float* __restrict__ dw2) {
    extern __shared__ __align__(16) char lds[];
    const int MT = (f + C::BM - 1) / C::BM, NT = (d + C::BN - 1) / C::BN;
    ExpertRank er;
    int mt, nt;
    if (!wgrad_tile(rank, blockIdx.x, MT, NT, er, mt, nt)) return;
    const int e = er.e, off = er.off, cnt = er.cnt;
    const int m0 = mt * C::BM;
    const int n0 = nt * C::BN;
    GHMC<ACT, C, C::BM> la;
    rs::GatherMC<C, C::BN> lb;
    rs::NoLoader nl;
    if (cnt > 0) {
        la.init(A, B, f, off, m0, f, cnt, gs);
        lb.init(dy, d, n0, d, eti + off, cnt);
    }
    rs::Acc<C> acc;
    rs::mainloop<C>(la, lb, nl, rs::slices(cnt), lds, acc);
    float* out = dw2 + (int64_t)e * f * d;
    dw_out<C, 1, ADD>(acc, lds, m0, n0, f, d, [&](int, int m, int n) { return out + (int64_t)m * d + n; });
}

// G5: dW1[e] = x[eti]^T dA, dW3[e] = x[eti]^T dB   (M = d, N = f, K = slots of e)
// (non-gated: dW1 alone)
template <int ACT, class C, bool ADD>
__global__ void __launch_bounds__(C::THREADS, 2)
g5_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ dA,
          const bf16_t* __restrict__ dB, const ExpertRank* __restrict__ rank,
          const int32_t* __restrict__ eti, int d, int f, float* __restrict__ dw1,
          float* __restrict__ dw3) {
    extern __shared__ __align__(16) char lds[];
    const int MT = (d + C::BM - 1) / C::BM, NT = (f + C::BN - 1) / C::BN;
    ExpertRank er;
    int mt, nt;
    if (!wgrad_tile(rank, blockIdx.x, MT, NT, er, mt, nt)) return;
    const int e = er.e, off = er.off, cnt = er.cnt;
    const int m0 = mt * C::BM;
    const int n0 = nt * C::BN;
    rs::GatherMC<C, C::BM> la;
    rs::SlotMC<C, C::BN> lb0;
    std::conditional_t<ACT == ACT_SWIGLU, rs::SlotMC<C, C::BN>, rs::NoLoader> lb1;
    if (cnt > 0) {
        la.init(x, d, m0, d, eti + off, cnt);
        lb0.init(dA, f, off, n0, f, cnt);
        if constexpr (ACT == ACT_SWIGLU) lb1.init(dB, f, off, n0, f, cnt);
    }
    rs::Acc<C> acc;
    rs::mainloop<C>(la, lb0, lb1, rs::slices(cnt), lds, acc);
    float* o1 = dw1 + (int64_t)e * d * f;
    float* o3 = ACT == ACT_SWIGLU ? dw3 + (int64_t)e * d * f : o1;  // dw3 is NULL when non-gated
    dw_out<C, ACT == ACT_SWIGLU ? 2 : 1, ADD>(acc, lds, m0, n0, d, f, [&](int b, int m, int n) {
        return (b ? o3 : o1) + (int64_t)m * f + n;
    });
}

// G6: dX_slot = dA W1[e]^T + dB W3[e]^T, output columns [n_base, n_base + ncols)
// into rows ldo apart   (K = 2f; non-gated: dA W1[e]^T, K = f,
// called with dB = dA and W3 = W1, whose second halves are then never reached)
template <bool SCATTER>
__global__ void __launch_bounds__(RS::THREADS)
g6_kernel(const bf16_t* __restrict__ dA, const bf16_t* __restrict__ dB,
          const bf16_t* __restrict__ w1, const bf16_t* __restrict__ w3,
          const int32_t* __restrict__ offsets, int d, int f, int E, int kslices, int n_base,
          int ncols, int64_t ldo, bf16_t* __restrict__ dX, const int32_t* __restrict__ tok) {
    extern __shared__ __align__(16) char lds[];
    using C = RS;
    SlotTile t;
    const int NT = (ncols + C::BN - 1) / C::BN;
    if (!find_slot_tile<C::THREADS>(reinterpret_cast<int*>(lds), offsets, E, C::BM, NT,
                                    blockIdx.x, C::BN, t, RASTER_GM))
        return;
    rs::DenseKC2<C, C::BM> la;
    la.init(dA, dB, f, (int64_t)t.off + t.m0, t.mrows, f);
    rs::DenseKC2<C, C::BN> lb;  // rows i of W1[e] / W3[e] ([d][f]), K = f then f
    lb.init(w1 + (int64_t)t.e * d * f, w3 + (int64_t)t.e * d * f, f, n_base + t.n0,
            min(C::BN, ncols - t.n0), f);
    rs::NoLoader nl;
    rs::Acc<C> acc;
    rs::mainloop<C>(la, lb, nl, kslices, lds, acc);
    slot_rows<SCATTER, C>(acc, t, ncols, ldo, dX, tok, nullptr, lds);
}

// d_gates[slot_src[s]] = sum of the G4 partials of slot s (fixed order)
// (16-byte loads when a slot's nparts partials fill whole 16-byte vectors;
// the sum runs in order p = 0..nparts-1 either way)
__global__ void dgate_reduce(const float* __restrict__ part, int nparts,
                             const int32_t* __restrict__ slot_src,
                             const int32_t* __restrict__ offsets, int E, int64_t S,
                             float* __restrict__ dgates) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= S || s >= offsets[E]) return;
    const float* row = part + s * nparts;
    float acc = 0.f;
    if ((nparts & 3) == 0) {
        for (int p = 0; p < nparts; p += 4) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(row + p);
            acc += v[0]; acc += v[1]; acc += v[2]; acc += v[3];
        }
    } else {
        for (int p = 0; p < nparts; ++p) acc += row[p];
    }
    dgates[slot_src[s]] = acc;
}

inline dim3 grid1d(int64_t n, int bs) { return dim3((unsigned)((n + bs - 1) / bs)); }

// workgroups of a preparation launch over S slots and n bf16 values to clear
inline unsigned prep_grid(int64_t S, int64_t n) { return grid1d(S > n / 8 ? S : n / 8, 256).x; }

// number of workgroups for a row-wise grouped GEMM (upper bound on tiles)
inline unsigned slot_grid(int64_t S, int E, int BM, int NT) {
    return (unsigned)(((S + BM - 1) / BM + E) * NT);
}
inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// ---- which core runs a row-wise GEMM (ffn_small.hip) ----
// The choice rests on the sizes alone (the host does not see the routing): r =
// S / E rows per expert, and the number of tiles a launch would have, estimated
// as one per expert that can have a slot, or a third of a tile of padding per
// expert once they fill. Measured on one MI355X, kernel times in us as (256-row
// core, small core):
//  - r <= 112: 64-row tiles up to r = 40, then 128-row tiles. First layer, E = 64,
//    d = 2048, f = 1408: r = 4 (149, 124), 48 (152, 136), 96 (159, 148); r = 141
//    (201, 216). E = 128, d = f = 2880: r = 9 (808, 696), 64 (856, 792). dh
//    GEMM there: r = 96 (127, 103), 9 (526, 374); E = 8, d = 4096, f = 14336:
//    r = 112 (219, 202), 150 (230, 315).
//  - the second GEMM and the dX GEMM (N = d, K = f or 2f) leave the chip half
//    idle in 256 x 256 tiles when the experts are few: 128-row tiles then (dX, E = 8, d = 4096, f = 14336: r = 32 (487, 332), 150 (538, 447);
//    E = 16, d = 1024, f = 4096: r = 200 (153, 89)).
//  - columns: the widest tiles if they give 128 workgroups; the dX and second
//    GEMMs, with longer K and fewer columns, take 128 columns while those tiles
//    run in one round (E = 8: 330 against 400 of the wide ones) and 64 while
//    those do (E = 16: 55 against 65 and 95).
//  - h formed on load: the 128 x 512 core (RHW) forms each h once per 512
//    columns and reads at the memory rate from about 100 workgroups on (E = 64,
//    r = 4: 68, the small tiles 68 to 113); below, small tiles while they run in
//    one round (E = 8, d = 4096, f = 14336: r = 4 (345, 130), 75 (381, 280), 112
//    (394, 491); one token of E = 64, d = 2048: (42, 18)).
inline int64_t est_rows(int64_t S, int E, int BM) {   // tile rows of BM
    const int64_t act = S < E ? S : E, full = (S + act * BM / 3) / BM;
    return act > full ? act : full;
}
//  - half-idle launches at any r: with 4 experts, d = 512, f = 2048 a 256-row
//    tile's grid has 16 (T = 2000) to 66 (T = 8192) tiles in the second and dX
//    GEMMs. dX, T = 2000 and 8192: (84, 34), (86, 70), 16384 (99, 143); second in
//    RHW and RHN: (63, 42), (65, 49), 16384 (75, 98); E = 8, d = 4096, f = 14336,
//    T = 600 (418, 307), 1000 (424, 625). Weight gradients, T = 8192: dW2 (71, 50),
//    dW1 and dW3 (61, 47), non-gated (55, 29); E = 16, d = 1024, f = 4096 (1024
//    tiles): dW2 (102, 110). Smaller dW1 / dW3 tiles also where the experts have
//    up to 96 slots, a slice or two of K: E = 64, d = 2048, f = 1408, r = 19 (281,
//    258), 96 (312, 293), 159 (363, 386).
inline bool few_tiles(int64_t tiles) { return tiles <= 128; }
// first GEMM and dh GEMM: N = f, K = d; wide_cols and big_cols columns per tile
// in the wide small tiles and in the 256-row ones. Beyond 112 rows per expert the
// 128-row tiles while a 256-row grid would have up to 80 tiles, whose 128-row ones
// run in one round with room for uneven experts. 256-row core and small core at 80,
// 120 and about 140 tiles, us: first GEMM, E = 4, d = 4096, f = 2048 (86, 65), (89, 69),
// (97, 125); dh GEMM, E = 2, d = 2048, f = 1408 (57, 45), (55, 43), (64, 86).
inline SmallTile small_wide_n(int64_t S, int E, int ncols, int wide_cols, int big_cols) {
    const int64_t r = S / E;
    const bool few = est_rows(S, E, 256) * cdiv(ncols, big_cols) <= 80;
    const int rows = r <= 40 || (few && est_rows(S, E, 64) * cdiv(ncols, 128) <= 256) ? 64
                     : r <= 112 || few                                               ? 128
                                                                                     : 0;
    if (!rows) return {0, 0};
    return {rows, est_rows(S, E, rows) * cdiv(ncols, wide_cols) >= 128 ? SMALL_WIDE : SMALL_NARROW};
}
inline int small_level(int64_t mt, int ncols) {
    return mt * cdiv(ncols, 64) <= 256 ? SMALL_SLIM : mt * cdiv(ncols, 128) <= 256 ? SMALL_NARROW : SMALL_WIDE;
}
// second GEMM from the h buffer, and dX GEMM: N = d
inline SmallTile small_long_k(int64_t S, int E, int ncols) {
    const int64_t r = S / E;
    const bool few = few_tiles(est_rows(S, E, RS::BM) * cdiv(ncols, RS::BN));
    const int rows = r <= 40 || (few && est_rows(S, E, 64) * cdiv(ncols, 128) <= 256) ? 64
                     : r <= 112 || few                                               ? 128
                                                                                     : 0;
    if (!rows) return {0, 0};
    return {rows, small_level(est_rows(S, E, rows), ncols)};
}
// second GEMM with h formed on load
inline SmallTile small_form_h(int64_t S, int E, int ncols) {
    if (est_rows(S, E, RHW::BM) * cdiv(ncols, RHW::BN) > 96) return {0, 0};
    const int rows = S / E <= 24 ? 32 : 64;
    const int64_t mt = est_rows(S, E, rows);
    if (mt * cdiv(ncols, 256) > 256) return {0, 0};
    return {rows, small_level(mt, ncols)};
}

// Raise the dynamic LDS limit of the GEMM kernels once per process.
hipError_t set_lds_limits() {
    static hipError_t status = [] {
        hipError_t e = hipSuccess;
        auto set = [&](const void* fn, int bytes) {
            if (e == hipSuccess)
                e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        };
        auto per_act = [&](auto act) {
            constexpr int ACT = decltype(act)::value;
            set(reinterpret_cast<const void*>(g1_kernel<ACT>), CFirst<ACT>::LDS);
            set(reinterpret_cast<const void*>(g4_kernel<ACT, true>), RS::LDS);
            set(reinterpret_cast<const void*>(g4_kernel<ACT, false>), RS::LDS);
            set(reinterpret_cast<const void*>(g5_kernel<ACT, CFirst<ACT>, false>), CFirst<ACT>::LDS);
            set(reinterpret_cast<const void*>(g5_kernel<ACT, CFirst<ACT>, true>), CFirst<ACT>::LDS);
            set(reinterpret_cast<const void*>(g5_kernel<ACT, CNarrow<ACT>, false>), CNarrow<ACT>::LDS);
            set(reinterpret_cast<const void*>(g5_kernel<ACT, CNarrow<ACT>, true>), CNarrow<ACT>::LDS);
            set(reinterpret_cast<const void*>(g2h_kernel<ACT, false, RHW>), RHW::LDS);
            set(reinterpret_cast<const void*>(g2h_kernel<ACT, true, RHW>), RHW::LDS);
            set(reinterpret_cast<const void*>(g2h_kernel<ACT, false, RHN>), RHN::LDS);
            set(reinterpret_cast<const void*>(g2h_kernel<ACT, true, RHN>), RHN::LDS);
            set(reinterpret_cast<const void*>(g3h_kernel<ACT, RHW, false>), RHW::LDS);
            set(reinterpret_cast<const void*>(g3h_kernel<ACT, RHW, true>), RHW::LDS);
            set(reinterpret_cast<const void*>(g3h_kernel<ACT, RHN, false>), RHN::LDS);
            set(reinterpret_cast<const void*>(g3h_kernel<ACT, RHN, true>), RHN::LDS);
        };
        per_act(std::integral_constant<int, ACT_SWIGLU>{});
        per_act(std::integral_constant<int, ACT_SILU>{});
        per_act(std::integral_constant<int, ACT_RELU>{});
        set(reinterpret_cast<const void*>(g2_kernel<false>), RS::LDS);
        set(reinterpret_cast<const void*>(g2_kernel<true>), RS::LDS);
        set(reinterpret_cast<const void*>(g3_kernel<RS, false>), RS::LDS);
        set(reinterpret_cast<const void*>(g3_kernel<RS, true>), RS::LDS);
        set(reinterpret_cast<const void*>(g3_kernel<RSN, false>), RSN::LDS);
        set(reinterpret_cast<const void*>(g3_kernel<RSN, true>), RSN::LDS);
        set(reinterpret_cast<const void*>(g6_kernel<false>), RS::LDS);
        set(reinterpret_cast<const void*>(g6_kernel<true>), RS::LDS);
        return e;
    }();
    return status;
}

inline size_t align256(size_t b) { return (b + 255) / 256 * 256; }
inline int g4_nparts(int f) { return cdiv(f, RS::BN) * RS::WN; }
// Column strip of the expert output (or of dX_slot) when the combine follows
// strip by strip. Narrow strips save memory, but a launch needs enough tiles
// (here about six waves of 256) or its last partial wave leaves CUs idle, so
// the strips are about as narrow as that allows, in whole tiles of the GEMM
// that produces them (BM x BN): with 256 x 256 tiles about 1024 columns for
// 98k slots and 64 experts, 2048 for 65k slots and 8 experts, 256 for 524k
// slots. `narrow`: round the number of strips up rather than down (the last
// strip may then be narrower), for the memory-lean h-on-load policy.
inline int strip_width(int64_t S, int E, int d, int BM, int BN, bool narrow) {
    const int64_t mtiles = (S + BM - 1) / BM + E / 2;   // tiles per column of tiles
    const int64_t want = 6 * 256;
    int64_t w = (int64_t)BN * ((want + mtiles - 1) / mtiles);
    w = w < d ? w : d;
    const int n = (int)(narrow ? (d + w - 1) / w : d / w);   // strips
    const int width = ((d + n - 1) / n + BN - 1) / BN * BN;
    return width < d ? width : d;
}
// strips of the forward's second GEMM (h on load: its 128 x 512 tiles) and of
// the backward's dX GEMM
inline int fwd_strip(int64_t S, int E, int d, bool h_on_load) {
    return h_on_load ? strip_width(S, E, d, RHW::BM, RHW::BN, true)
                     : strip_width(S, E, d, RS::BM, RS::BN, false);
}
inline int bwd_strip(int64_t S, int E, int d) { return strip_width(S, E, d, RS::BM, RS::BN, false); }

}  // namespace

hipError_t dgate_sum(const float* part, int nparts, const int32_t* slot_src,
                     const int32_t* offsets, int E, int64_t S, float* dgates, hipStream_t st) {
    hipLaunchKernelGGL(dgate_reduce, grid1d(S, 256), dim3(256), 0, st, part, nparts, slot_src,
                       offsets, E, S, dgates);
    probe::mark("dgate_reduce", st);
    return hipGetLastError();
}

size_t ffn_fwd_workspace(int64_t T, int d, int f, int E, int k, bool f32, bool combined,
                         bool h_on_load, bool scatter) {
    const size_t S = (size_t)T * k;
    if (f32) return combined ? align256(S * d * sizeof(float)) : 0;  // O
    const size_t h = h_on_load ? 0 : align256(S * f * sizeof(bf16_t));   // H
    if (!combined) return h;
    if (scatter) return h + align256(S * sizeof(float));                  // slot gates
    return h + align256(S * fwd_strip(S, E, d, h_on_load) * sizeof(bf16_t));
}

namespace {

template <int ACT>
hipError_t ffn_fwd_act(const FfnArgs& a, hipStream_t st) {
    const int64_t S = a.T * a.k;
    if (hipError_t e = set_lds_limits(); e != hipSuccess) return e;
    using C1 = CFirst<ACT>;
    // h buffered between the GEMMs, or (h_on_load) formed again from A, B
    bf16_t* H = a.h_on_load ? nullptr : static_cast<bf16_t*>(a.ws);
    const SmallTile t1 = small_wide_n(S, a.E, a.f, ACT == ACT_SWIGLU ? 128 : 256, CFirst<ACT>::BN);
    if (t1.rows) {
        if (hipError_t e = small_first(a, t1, H, st); e != hipSuccess) return e;
    } else {
        hipLaunchKernelGGL(g1_kernel<ACT>, dim3(slot_grid(S, a.E, C1::BM, cdiv(a.f, C1::BN))),
                           dim3(C1::THREADS), C1::LDS, st, (const bf16_t*)a.x,
                           (const bf16_t*)a.w1, (const bf16_t*)a.w3, a.offsets, a.eti, a.d, a.f,
                           a.E, (bf16_t*)a.A, (bf16_t*)a.B, H);
        probe::mark("g1_kernel", st);
    }
    // the second GEMM over columns [c0, c0 + nc): slot rows into out (ldo
    // apart), or with gs (scatter) added into the token rows of out
    auto second = [&](int c0, int nc, int64_t ldo, bf16_t* out, const float* gs) {
        const SmallTile t2 = H ? small_long_k(S, a.E, nc) : small_form_h(S, a.E, nc);
        if (t2.rows) return small_second(a, t2, H, c0, nc, ldo, out, gs, st);
        if (a.h_on_load) {
            auto run = [&](auto cfg) {
                using C = decltype(cfg);
                auto g2h = gs ? g2h_kernel<ACT, true, C> : g2h_kernel<ACT, false, C>;
                hipLaunchKernelGGL(g2h, dim3(slot_grid(S, a.E, C::BM, cdiv(nc, C::BN))),
                                   dim3(C::THREADS), C::LDS, st, (const bf16_t*)a.A,
                                   (const bf16_t*)a.B, (const bf16_t*)a.w2, a.offsets, a.d, a.f,
                                   a.E, c0, nc, ldo, out, a.eti, gs);
            };
            const bool few = few_tiles(est_rows(S, a.E, RHW::BM) * cdiv(nc, RHW::BN));
            if (few) run(RHN{});
            else run(RHW{});
            probe::mark(few ? "g2h_narrow" : "g2h_kernel", st);
        } else {
            auto g2 = gs ? g2_kernel<true> : g2_kernel<false>;
            hipLaunchKernelGGL(g2, dim3(slot_grid(S, a.E, RS::BM, cdiv(nc, RS::BN))),
                               dim3(RS::THREADS), RS::LDS, st, (const bf16_t*)H,
                               (const bf16_t*)a.w2, a.offsets, a.d, a.f, a.E, c0, nc, ldo, out,
                               a.eti, gs);
            probe::mark("g2_kernel", st);
        }
        return hipGetLastError();
    };
    if (!a.y) {   // O [S, d] for the caller's combine
        return second(0, a.d, (int64_t)a.d, (bf16_t*)a.O, nullptr);
    }
    if (a.scatter) {   // y = 0, then every slot row times its gate added into y
        float* gs = reinterpret_cast<float*>(
            static_cast<char*>(a.ws) + (a.h_on_load ? 0 : align256((size_t)S * a.f * sizeof(bf16_t))));
        hipLaunchKernelGGL(fwd_prep, dim3(prep_grid(S, a.T * a.d)), dim3(256), 0, st, a.gates, a.tim,
                           S, gs, static_cast<bf16_t*>(a.y), a.T * a.d);
        probe::mark("fwd_prep", st);
        return second(0, a.d, (int64_t)a.d, static_cast<bf16_t*>(a.y), gs);
    }
    // combined: one column strip of O at a time, straight into y
    const int sw = fwd_strip(S, a.E, a.d, a.h_on_load);
    bf16_t* strip = reinterpret_cast<bf16_t*>(
        static_cast<char*>(a.ws) + (a.h_on_load ? 0 : align256((size_t)S * a.f * sizeof(bf16_t))));
    for (int c0 = 0; c0 < a.d; c0 += sw) {
        const int nc = min(sw, a.d - c0);
        if (hipError_t e = second(c0, nc, (int64_t)nc, strip, nullptr); e != hipSuccess) return e;
        if (hipError_t e = combine_cols(strip, nc, a.gates, a.tim, a.T, nc, a.k, false, false,
                                        static_cast<bf16_t*>(a.y) + c0, a.d, st);
            e != hipSuccess)
            return e;
    }
    return hipGetLastError();
}

template <int ACT>
hipError_t ffn_first_act(const FfnArgs& a, hipStream_t st) {
    const int64_t S = a.T * a.k;
    if (hipError_t e = set_lds_limits(); e != hipSuccess) return e;
    if (const SmallTile t1 = small_wide_n(S, a.E, a.f, ACT == ACT_SWIGLU ? 128 : 256, CFirst<ACT>::BN); t1.rows)
        return small_first(a, t1, nullptr, st);
    using C1 = CFirst<ACT>;
    hipLaunchKernelGGL(g1_kernel<ACT>, dim3(slot_grid(S, a.E, C1::BM, cdiv(a.f, C1::BN))),
                       dim3(C1::THREADS), C1::LDS, st, (const bf16_t*)a.x, (const bf16_t*)a.w1,
                       (const bf16_t*)a.w3, a.offsets, a.eti, a.d, a.f, a.E, (bf16_t*)a.A,
                       (bf16_t*)a.B, (bf16_t*)nullptr);
    probe::mark("g1_kernel", st);
    return hipGetLastError();
}

}  // namespace

hipError_t ffn_first(const FfnArgs& a, bool f32, hipStream_t st) {
    if (f32) return f32_first(a, st);
    switch (a.act) {
    case ACT_SILU: return ffn_first_act<ACT_SILU>(a, st);
    case ACT_RELU: return ffn_first_act<ACT_RELU>(a, st);
    default: return ffn_first_act<ACT_SWIGLU>(a, st);
    }
}

hipError_t ffn_fwd(const FfnArgs& a, bool f32, hipStream_t st) {
    if (f32) return f32_fwd(a, st);
    switch (a.act) {
    case ACT_SILU: return ffn_fwd_act<ACT_SILU>(a, st);
    case ACT_RELU: return ffn_fwd_act<ACT_RELU>(a, st);
    default: return ffn_fwd_act<ACT_SWIGLU>(a, st);
    }
}

// bytes of the backward workspace before the expert rank table
inline size_t bwd_main_bytes(size_t S, int d, int f, int E, bool combined, bool h_on_load) {
    // combined: the dX strips (none when they are scattered into dx)
    const size_t part = align256(S * g4_nparts(f) * sizeof(float));  // d_gate partials
    const size_t strip = combined ? S * bwd_strip(S, E, d) * sizeof(bf16_t) : 0;
    if (h_on_load) {   // slot-ordered gates for G3, then (same space) the dX strip
        const size_t gs = S * sizeof(float);
        return part + align256(gs > strip ? gs : strip);
    }
    const size_t hg = S * f * sizeof(bf16_t);                         // g*h, then dX strips
    return part + align256(hg > strip ? hg : strip);
}

size_t ffn_bwd_workspace(int64_t T, int d, int f, int E, int k, bool f32, bool combined,
                         bool h_on_load, bool scatter) {
    const size_t S = (size_t)T * k;
    if (f32) return combined ? align256(S * d * sizeof(float)) : 0;  // dX_slot
    return bwd_main_bytes(S, d, f, E, combined && !scatter, h_on_load) +
           align256(E * sizeof(ExpertRank));
}

namespace {

template <int ACT>
hipError_t ffn_bwd_act(const FfnArgs& a, hipStream_t st) {
    const int64_t S = a.T * a.k;
    constexpr bool GATED = ACT == ACT_SWIGLU;
    if (hipError_t e = set_lds_limits(); e != hipSuccess) return e;
    const int nparts = g4_nparts(a.f);
    float* part = static_cast<float*>(a.ws);
    char* const ws2 = static_cast<char*>(a.ws) + align256((size_t)S * nparts * sizeof(float));
    // default: g*h [S, f] from G4's epilogue for G3; h on load: slot-ordered
    // gates, and G3 (run first, before G4 overwrites A and B) forms g*h itself.
    // Either is finished with before the dX strips reuse the space.
    float* gs = a.h_on_load ? reinterpret_cast<float*>(ws2) : nullptr;
    bf16_t* HG = a.h_on_load ? nullptr : reinterpret_cast<bf16_t*>(ws2);
    bf16_t* strip = reinterpret_cast<bf16_t*>(ws2);
    ExpertRank* rank = reinterpret_cast<ExpertRank*>(
        static_cast<char*>(a.ws) +
        bwd_main_bytes(S, a.d, a.f, a.E, a.y != nullptr && !a.scatter, a.h_on_load));
    hipLaunchKernelGGL(bwd_prep, dim3(1 + (gs ? prep_grid(S, 0) : 0)), dim3(256), 0, st, a.gates,
                       a.slot_src, a.offsets, a.E, S, rank, gs);
    probe::mark("bwd_prep", st);
    // non-gated: the second operand of the two-branch kernels is the first again
    const void* Bx = GATED ? a.B : a.A;
    const void* w3x = GATED ? a.w3 : a.w1;
    if (a.h_on_load) {
        auto run = [&](auto cfg) {
            using C = decltype(cfg);
            auto g3h = a.accumulate_dw ? g3h_kernel<ACT, C, true> : g3h_kernel<ACT, C, false>;
            hipLaunchKernelGGL(g3h, dim3(wgrad_grid(a.E, cdiv(a.f, C::BM), cdiv(a.d, C::BN))),
                               dim3(C::THREADS), C::LDS, st, (const bf16_t*)a.A, (const bf16_t*)Bx,
                               (const float*)gs, (const bf16_t*)a.dy, rank, a.eti, a.d, a.f, a.dw2);
        };
        const bool few = few_tiles((int64_t)a.E * cdiv(a.f, RHW::BM) * cdiv(a.d, RHW::BN));
        if (few) run(RHN{});
        else run(RHW{});
        probe::mark(few ? "g3h_narrow" : "g3h_kernel", st);
    }
    const SmallTile t4 = small_wide_n(S, a.E, a.f, 256, RS::BN);
    if (t4.rows) {
        if (hipError_t e = small_dact(a, t4, gs, HG, part, nparts, st); e != hipSuccess) return e;
    } else {
        auto g4 = a.h_on_load ? g4_kernel<ACT, false> : g4_kernel<ACT, true>;
        hipLaunchKernelGGL(g4, dim3(slot_grid(S, a.E, RS::BM, cdiv(a.f, RS::BN))),
                           dim3(RS::THREADS), RS::LDS, st, (const bf16_t*)a.dy,
                           (const bf16_t*)a.w2, a.gates, a.offsets, a.eti, a.slot_src,
                           (const float*)gs, a.d, a.f, a.E, (bf16_t*)a.A, (bf16_t*)a.B, HG, part);
        probe::mark("g4_kernel", st);
    }
    if (hipError_t e = dgate_sum(part, nparts, a.slot_src, a.offsets, a.E, S, a.dgates, st);
        e != hipSuccess)
        return e;
    if (!a.h_on_load) {
        auto run = [&](auto cfg) {
            using C = decltype(cfg);
            auto g3 = a.accumulate_dw ? g3_kernel<C, true> : g3_kernel<C, false>;
            hipLaunchKernelGGL(g3, dim3(wgrad_grid(a.E, cdiv(a.f, C::BM), cdiv(a.d, C::BN))),
                               dim3(C::THREADS), C::LDS, st, (const bf16_t*)HG,
                               (const bf16_t*)a.dy, rank, a.eti, a.d, a.f, a.dw2);
        };
        const bool few = few_tiles((int64_t)a.E * cdiv(a.f, RS::BM) * cdiv(a.d, RS::BN));
        if (few) run(RSN{});
        else run(RS{});
        probe::mark(few ? "g3_narrow" : "g3_kernel", st);
    }
    auto dw13 = [&](auto cfg) {
        using C = decltype(cfg);
        auto g5 = a.accumulate_dw ? g5_kernel<ACT, C, true> : g5_kernel<ACT, C, false>;
        hipLaunchKernelGGL(g5, dim3(wgrad_grid(a.E, cdiv(a.d, C::BM), cdiv(a.f, C::BN))),
                           dim3(C::THREADS), C::LDS, st, (const bf16_t*)a.x, (const bf16_t*)a.A,
                           (const bf16_t*)a.B, rank, a.eti, a.d, a.f, a.dw1, a.dw3);
    };
    const bool few5 = S / a.E <= 96 ||
        few_tiles((int64_t)a.E * cdiv(a.d, CFirst<ACT>::BM) * cdiv(a.f, CFirst<ACT>::BN));
    if (few5) dw13(CNarrow<ACT>{});
    else dw13(CFirst<ACT>{});
    probe::mark(few5 ? "g5_narrow" : "g5_kernel", st);
    const int kslices = (GATED ? 2 : 1) * a.f / rs::KS;
    auto t6 = [&](int nc) { return small_long_k(S, a.E, nc); };
    if (!a.y && t6(a.d).rows) return small_dx(a, t6(a.d), 0, a.d, (int64_t)a.d, a.dX, false, st);
    if (!a.y) {   // dX_slot [S, d] for the caller's combine
        hipLaunchKernelGGL(g6_kernel<false>, dim3(slot_grid(S, a.E, RS::BM, cdiv(a.d, RS::BN))),
                           dim3(RS::THREADS), RS::LDS, st, (const bf16_t*)a.A, (const bf16_t*)Bx,
                           (const bf16_t*)a.w1, (const bf16_t*)w3x, a.offsets, a.d, a.f, a.E,
                           kslices, 0, a.d, (int64_t)a.d, (bf16_t*)a.dX, a.eti);
        probe::mark("g6_kernel", st);
        return hipGetLastError();
    }
    if (a.scatter) {   // every dX_slot row added into dx (cleared first unless accumulating)
        if (!a.accumulate) {   // (only now: every read of dy and x is done)
            hipLaunchKernelGGL(zero_bf16, dim3(prep_grid(0, a.T * a.d)), dim3(256), 0, st,
                               static_cast<bf16_t*>(a.y), a.T * a.d);
            probe::mark("zero_bf16", st);
        }
        if (t6(a.d).rows) return small_dx(a, t6(a.d), 0, a.d, (int64_t)a.d, a.y, true, st);
        hipLaunchKernelGGL(g6_kernel<true>, dim3(slot_grid(S, a.E, RS::BM, cdiv(a.d, RS::BN))),
                           dim3(RS::THREADS), RS::LDS, st, (const bf16_t*)a.A, (const bf16_t*)Bx,
                           (const bf16_t*)a.w1, (const bf16_t*)w3x, a.offsets, a.d, a.f, a.E,
                           kslices, 0, a.d, (int64_t)a.d, static_cast<bf16_t*>(a.y), a.eti);
        probe::mark("g6_kernel", st);
        return hipGetLastError();
    }
    // combined: one column strip of dX_slot at a time, summed straight into dx;
    // by default the strip reuses g*h's workspace, which G3 has finished with
    const int sw = bwd_strip(S, a.E, a.d);
    for (int c0 = 0; c0 < a.d; c0 += sw) {
        const int nc = min(sw, a.d - c0);
        if (t6(nc).rows) {
            if (hipError_t e = small_dx(a, t6(nc), c0, nc, (int64_t)nc, strip, false, st); e != hipSuccess)
                return e;
        } else {
            hipLaunchKernelGGL(g6_kernel<false>, dim3(slot_grid(S, a.E, RS::BM, cdiv(nc, RS::BN))),
                               dim3(RS::THREADS), RS::LDS, st, (const bf16_t*)a.A,
                               (const bf16_t*)Bx, (const bf16_t*)a.w1, (const bf16_t*)w3x,
                               a.offsets, a.d, a.f, a.E, kslices, c0, nc, (int64_t)nc, strip, a.eti);
            probe::mark("g6_kernel", st);
        }
        if (hipError_t e = combine_cols(strip, nc, nullptr, a.tim, a.T, nc, a.k, false,
                                        a.accumulate, static_cast<bf16_t*>(a.y) + c0, a.d, st);
            e != hipSuccess)
            return e;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t ffn_bwd(const FfnArgs& a, bool f32, hipStream_t st) {
    if (f32) return f32_bwd(a, st);
    switch (a.act) {
    case ACT_SILU: return ffn_bwd_act<ACT_SILU>(a, st);
    case ACT_RELU: return ffn_bwd_act<ACT_RELU>(a, st);
    default: return ffn_bwd_act<ACT_SWIGLU>(a, st);
    }
}

}  // namespace moe
