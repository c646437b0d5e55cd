// gemm.hpp -- pieces shared by the grouped GEMM kernels, the router and the
// router backward (gfx950): MFMA and LDS helpers, direct-to-LDS copies (the rings
// of the router and of gemm_sk.hpp, the dh GEMM's epilogue), the 16-byte epilogue
// layout of a 32x32 accumulator fragment, a wave's output coordinates, float32 tile
// output through LDS, and the tile orders of the weight-gradient and the row-wise
// grouped GEMMs. The main loops and their operand loaders are in gemm_rs.hpp and
// gemm_sk.hpp.
//
// MFMA 32x32x16 operand layout (wave64), verified on gfx950: for D = P * Q,
// lane L supplies P[L%32][8*(L/32) + 0..7] and Q[8*(L/32) + 0..7][L%32] and
// receives D[8*(j/4) + 4*(L/32) + j%4][L%32] in accumulator register j. The
// kernels pass P = right-operand tile (rows = output columns n) and
// Q = left-operand tile (rows = output rows m), so lane L ends up holding
// output row m = L%32 at columns n = 8*(j/4) + 4*(L/32) + (j%4): four runs of
// four consecutive columns.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace moe {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void_t;


__device__ __forceinline__ f32x16 mfma32x32x16(const bf16x8& p, const bf16x8& q, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(p, q, c, 0, 0, 0);
}

// Wait until at most N vector-memory operations of this wave are outstanding.
// Inline assembly with a memory clobber, so that the compiler moves no memory
// access across it.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Workgroup barrier without the implicit drain of outstanding loads that
// __syncthreads() adds; also a compiler memory barrier.
__device__ __forceinline__ void barrier_only() { asm volatile("s_barrier" ::: "memory"); }

// Barrier after this wave's LDS accesses have completed.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// 16-byte global -> LDS copy by one lane: lane l writes LDS bytes
// lds_off + 16*l .. +15 (lds_off must be wave-uniform; it goes to M0). Issued
// from inline assembly so that the compiler does not track these copies: it
// would otherwise drain all of them (vmcnt(0)) before every transposing LDS
// read, which it cannot prove independent of the copies in flight. The main
// loop waits for them explicitly (wait_vmcnt), so no compiler-visible vector
// memory access may be issued inside it.
__device__ __forceinline__ void dma16(const void* g, uint32_t lds_off) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 ::"v"(g), "s"(lds_off) : "memory", "m0");
}

// LDS byte offset of a pointer into the workgroup's shared memory.
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

// Wave index as a value the compiler knows to be uniform (kept in an SGPR).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// accumulators of a tile configuration C: [right operand][fragment row][fragment column]
template <class C>
using Acc = f32x16[C::NB][C::FM][C::FN];

// ---- 16-byte epilogue layout ----------------------------------------------------------
// In a 32x32 accumulator fragment lane L holds row L%32 at four runs of four
// columns, 8q + 4*(L/32) + 0..3 (q = 0..3). gfx950's v_permlane32_swap trades
// values between lanes L and L+32 so that, for p = 0, 1, lane L holds the
// eight consecutive columns 16p + 8*(L/32) + 0..7 instead: epilogues then load
// and store 16 bytes of bf16 per lane, whole 32-byte sectors per row.
__device__ __forceinline__ void frag_cols8(const f32x16& a, float (&v)[2][8]) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const auto s = __builtin_amdgcn_permlane32_swap(
                __float_as_uint(a[8 * p + r]), __float_as_uint(a[8 * p + 4 + r]), false, false);
            v[p][r] = __uint_as_float(s[0]);
            v[p][4 + r] = __uint_as_float(s[1]);
        }
}

// ---- output coordinates of a lane ------------------------------------------------
template <class C>
struct WaveCoord {
    int lane, wm, wn;
    __device__ WaveCoord() {
        lane = threadIdx.x & 63;
        const int wv = threadIdx.x >> 6;
        wm = wv / C::WN;
        wn = wv % C::WN;
    }
    // tile-local output row of fragment row-block i
    __device__ int row(int i) const { return wm * C::WTM + i * 32 + (lane & 31); }
    // tile-local first column of run q (0..3) of fragment column-block j
    __device__ int col(int j, int q) const { return wn * C::WTN + j * 32 + q * 8 + (lane >> 5) * 4; }
    // tile-local first column of eight-column group p (0, 1) after frag_cols8
    __device__ int col8(int j, int p) const { return wn * C::WTN + j * 32 + p * 16 + (lane >> 5) * 8; }
};

// ---- f32 tile output through LDS -------------------------------------------------------
// The accumulators go through LDS, IPR fragment row-blocks of every wave per
// round, and leave as whole rows of the tile: a wave's store instruction covers
// 1 KB of consecutive output bytes (or two rows of 512 B), so every 128-byte
// line is written by a single instruction. LDS rows are padded by 16 bytes,
// which keeps both the fragment writes and the row reads free of bank conflicts.
// Call after rs::mainloop (whose final barrier frees the LDS). Between
// rounds only the LDS accesses are ordered: the global stores of a round stay
// in flight while the next round is staged.

template <class C, int IPR>
struct RowStage {
    static constexpr int ROWS = C::WM * 32 * IPR;
    static constexpr int PITCH = C::BN * 4 + 16;
    static constexpr int V4_PER_ROW = C::BN / 4;
    static constexpr int PASSES = ROWS * V4_PER_ROW / C::THREADS;
    static constexpr int ROUNDS = C::NB * C::FM / IPR;
    static_assert(ROWS * PITCH <= C::LDS, "staging fits the LDS ring");
    static_assert(C::FM % IPR == 0 && (ROWS * V4_PER_ROW) % C::THREADS == 0, "even split");
    // f(b, tile_row, tile_col, p) for the passes [p0, p0 + N) of round rd: this
    // thread's 4 consecutive outputs each
    template <int N, class F>
    __device__ static __forceinline__ void passes(int rd, int p0, F&& f) {
        const int b = rd / (C::FM / IPR), i0 = (rd % (C::FM / IPR)) * IPR;
#pragma unroll
        for (int p = 0; p < N; ++p) {
            const int t = threadIdx.x + (p0 + p) * C::THREADS;
            const int cr = t / V4_PER_ROW, c4 = t % V4_PER_ROW;
            const int row = (cr / (32 * IPR)) * C::WTM + (i0 + (cr / 32) % IPR) * 32 + (cr & 31);
            f(b, row, c4 * 4, p);
        }
    }
    // round rd of the accumulators into LDS
    __device__ static __forceinline__ void stage(const Acc<C>& acc, char* lds, int rd) {
        const WaveCoord<C> wc;
        const int b = rd / (C::FM / IPR), i0 = (rd % (C::FM / IPR)) * IPR;
        if (rd > 0) lds_barrier();
#pragma unroll
        for (int ii = 0; ii < IPR; ++ii)
#pragma unroll
            for (int j = 0; j < C::FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int cr = wc.wm * 32 * IPR + ii * 32 + (wc.lane & 31);
                    const f32x16& a = acc[b][i0 + ii][j];
                    *reinterpret_cast<f32x4*>(lds + cr * PITCH + wc.col(j, q) * 4) =
                        f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
                }
        lds_barrier();
    }
    // the staged outputs of passes [p0, p0 + N)
    template <int N>
    __device__ static __forceinline__ void staged(const char* lds, int p0, f32x4 (&v)[N]) {
#pragma unroll
        for (int p = 0; p < N; ++p) {
            const int t = threadIdx.x + (p0 + p) * C::THREADS;
            v[p] = *reinterpret_cast<const f32x4*>(lds + (t / V4_PER_ROW) * PITCH +
                                                   (t % V4_PER_ROW) * 16);
        }
    }
    // store(b, tile_row, tile_col, f32x4) is called for every 4 consecutive outputs
    template <class F>
    __device__ static void run(const Acc<C>& acc, char* lds, F&& store) {
#pragma unroll
        for (int rd = 0; rd < ROUNDS; ++rd) {
            f32x4 v[PASSES];
            stage(acc, lds, rd);
            staged<PASSES>(lds, 0, v);
            passes<PASSES>(rd, 0, [&](int b, int r, int c, int p) { store(b, r, c, v[p]); });
        }
    }
    // The tile added to what memory holds, for a tile that lies inside the matrix as
    // a whole: at(b, tile_row, tile_col) is the address, st(address, value) the
    // store. Eight old values per thread are loaded before the eight stores that
    // precede their use, so that their wait leaves those stores in flight (a load
    // behind each store waits for every one of them: E = 64, d = 4096, f = 2048, three
    // chunks of 800 / 3 tokens, dW1 and dW3 4823 -> 3756 us, dW2 2585 -> 1951).
    template <class F, class ST>
    __device__ static void add(const Acc<C>& acc, char* lds, F&& at, ST&& st) {
        constexpr int N = PASSES < 8 ? PASSES : 8, U = PASSES / N;
        static_assert(PASSES % N == 0, "whole batches");
        f32x4 old[N];
        auto fetch = [&](int rd, int u) __attribute__((always_inline)) {
            passes<N>(rd, u * N, [&](int b, int r, int c, int p) {
                old[p] = *reinterpret_cast<const f32x4*>(at(b, r, c));
            });
        };
        fetch(0, 0);
#pragma unroll
        for (int rd = 0; rd < ROUNDS; ++rd) {
            stage(acc, lds, rd);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                f32x4 v[N];
                staged<N>(lds, u * N, v);
#pragma unroll
                for (int p = 0; p < N; ++p) v[p] = v[p] + old[p];
                if (u + 1 < U) fetch(rd, u + 1);
                else if (rd + 1 < ROUNDS) fetch(rd + 1, 0);
                passes<N>(rd, u * N, [&](int b, int r, int c, int p) { st(at(b, r, c), v[p]); });
            }
        }
    }
};

// ---- weight-gradient tile order ---------------------------------------------------------
// The weight-gradient GEMMs have P = MT*NT output tiles per expert, each looping
// over the expert's tokens, so a tile's length is its expert's token count.
// Workgroup ids are dealt round-robin to the 8 XCDs (each with its own L2).
// Every XCD takes, for every expert, one band of ceil(P/8) consecutive tiles,
// so that every XCD gets the same share of every expert whatever the experts'
// token counts. The experts are taken longest first: rank[r] holds the expert
// of rank r by token count (descending, ties to the lower index), its first
// slot and its count (expert_ranks). Under a skewed routing the longest tiles
// then start first and the many short ones fill in around them, instead of a
// late start of the longest tiles setting the kernel's end. Inside an expert
// the tiles are grouped WG_GM row tiles at a time with the column tile slower:
// the ~32 workgroups an XCD runs at once then cover a WG_GM x 8 block of
// tiles, which read WG_GM + 8 operand panels per K slice from L2 instead of
// the 1 + 32 of a row-major band (an expert's last, narrower group holds its
// remaining rows). Returns false for the padding tiles of the last band.
constexpr int WG_GM = 4;
struct ExpertRank {
    int32_t e, off, cnt, pad;
};
__device__ __forceinline__ bool wgrad_tile(const ExpertRank* __restrict__ rank, int bid, int MT,
                                           int NT, ExpertRank& er, int& mt, int& nt) {
    const int P = MT * NT;
    const int G = (P + 7) >> 3;
    const int x = bid & 7, j = bid >> 3;
    const int lt = x * G + j % G;
    if (lt >= P) return false;
    er = rank[j / G];
    const int grp = lt / (WG_GM * NT);
    const int m_base = grp * WG_GM;
    const int gm = min(WG_GM, MT - m_base);
    const int in = lt - grp * WG_GM * NT;
    mt = m_base + in % gm;
    nt = in / gm;
    return true;
}
inline int wgrad_grid(int E, int MT, int NT) { return E * 8 * ((MT * NT + 7) / 8); }

// ---- grouped tile lookup ------------------------------------------------------------
// Tiles of expert e: ceil(M_e / BM) * NT, laid out expert after expert. With
// GM = 0 the M tile index runs fastest (neighbouring tiles share a weight
// panel). With GM > 0 the tiles come in groups of GM M tiles, N slower
// inside a group: the workgroups that run at the same time on one XCD then
// cover a GM x (32 / GM) block of tiles, which share both their row panels
// and their weight panels in that XCD's L2 (an expert's last, narrower group
// holds its remaining M tiles). The block ids [0, total) of the tiles that
// exist are renumbered over the XCDs (xcd_remap), `total` being the scan's own
// sum: the grid is the worst case of one partial tile per expert, and dealing
// out contiguous ranges of that grid left the last XCDs with padding while the
// first had more than their share (one token, E = 64, k = 6: 66 tiles, all on
// one XCD: layer forward 194 us, now 117; T = 1021 fwd + bwd 1281 -> 1156 us). It
// holds with little padding too: E = 8, d = 4096, f = 14336, k = 2, all four
// row-wise GEMMs over the grid and over the tiles that exist, us: T = 20000
// 27089, 25351; 30000 (1.2% padding) 39754, 38400; 32768 equal within 0.5% (either
// way, by card). Every thread of the block must call this; `sh` is 8 ints of LDS,
// free on entry and again on return. Returns false past the last tile.
struct SlotTile {
    int e;       // expert
    int m0;      // first row inside the expert's slot segment
    int mrows;   // valid rows in this tile (<= BM)
    int n0;      // first output column
    int off;     // offsets[e]
};

template <int THREADS>
__device__ bool find_slot_tile(int* sh, const int32_t* __restrict__ offsets, int E, int BM, int NT,
                               int bid, int BN, SlotTile& t, int GM = 0) {
    constexpr int EPT = THREADS >= 256 ? 1 : 256 / THREADS;   // consecutive experts per thread
    constexpr int NWS = 256 / EPT / WAVE;                     // waves that hold experts
    static_assert(THREADS % WAVE == 0 && NWS <= 4, "at most 256 experts");
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wv = tid / WAVE;
    int tiles[EPT], cnt[EPT], off[EPT], sum = 0;
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        const int x = tid * EPT + u;
        off[u] = cnt[u] = 0;
        if (x < E) {
            off[u] = offsets[x];
            cnt[u] = offsets[x + 1] - off[u];
        }
        tiles[u] = ((cnt[u] + BM - 1) / BM) * NT;
        sum += tiles[u];
    }
    // expert e's tiles are [start, end): a wave-level scan, plus the totals of
    // the waves before
    const int inc = wave_incl_scan(sum);
    if (wv < NWS && lane == WAVE - 1) sh[wv] = inc;
    __syncthreads();
    int total = 0, start = inc - sum;
#pragma unroll
    for (int w = 0; w < NWS; ++w) {
        total += sh[w];
        start += w < wv ? sh[w] : 0;
    }
    if (bid >= total) return false;
    bid = xcd_remap(bid, total);
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        if (bid >= start && bid < start + tiles[u]) {
            sh[4] = tid * EPT + u;
            sh[5] = bid - start;
            sh[6] = off[u];
            sh[7] = cnt[u];
        }
        start += tiles[u];
    }
    __syncthreads();
    const int e = sh[4], local = sh[5];
    const int eoff = sh[6], ecnt = sh[7];
    __syncthreads();
    const int nmt = (ecnt + BM - 1) / BM;
    const int gm = GM > 0 ? GM : nmt;         // M tiles per group
    const int full = nmt / gm * gm;           // M tiles in whole groups
    int mt, nt;
    if (local < full * NT) {
        const int g = local / (gm * NT), w = local % (gm * NT);
        mt = g * gm + w % gm;
        nt = w / gm;
    } else {
        const int rem = nmt - full, l2 = local - full * NT;
        mt = full + l2 % rem;
        nt = l2 / rem;
    }
    t.e = e;
    t.off = eoff;
    t.m0 = mt * BM;
    t.mrows = min(BM, ecnt - t.m0);
    t.n0 = nt * BN;
    return true;
}

}  // namespace moe
