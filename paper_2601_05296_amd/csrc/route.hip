// route.hip -- top-k softmax gating, forward (MoEBlaze paper, Section 2.1:
// topk_experts = TopK(softmax(W_g x)), gate weights of Section 2.3).
//
// bf16 path: the router product logits[T,E] = x W_g^T is a skinny GEMM
// (E <= 256 columns) whose cost is reading x once from HBM, so it runs on the
// matrix cores: each wave owns 16 tokens and all E experts (or, for small
// grids, one of two K halves of them). The x rows of a workgroup (every x
// element is read exactly once) and W_g come through an LDS ring of 64-wide K
// slices filled by direct-to-LDS copies, two or three slices ahead of the one
// being multiplied. Softmax and the top-k selection run on the accumulators
// in registers: the 4 lanes holding one token's logits find the k largest by
// k rounds of (local best, two cross-lane exchanges), ties going to the lower
// expert id.
//
// f32 path: float32 matrix instructions (route_f32).
#include "common.hpp"
#include "gemm.hpp"
#include "launch.hpp"
#include "probe.hpp"

namespace moe {
namespace {

constexpr int RT_BK = 64;    // K slice staged in LDS

// Workgroup shapes. A workgroup routes TB tokens (16 per wave) over all
// experts; its waves form TB/16 token groups times KG K groups, group g taking
// the g-th contiguous share of the K slices. Every workgroup streams all of
// W_g, so larger TB reads fewer W_g bytes per x byte; KG = 2 doubles the waves
// (and with them the copies in flight, which follow the number of waves, not
// the ring depth) for a grid too small to give each CU two workgroups.
//   (64, 1): 4 waves, the default;
//   (64, 2): 8 waves, T < 32768 (fewer than 512 workgroups of 64 tokens);
//   (128, 1): 8 waves, E > 64 and T >= 65536 (W_g is then as large as 128 x rows).
template <int NE, int TB, int KG>
struct RtShape {
    static constexpr int EP = NE * 16;                 // expert rows staged (E padded)
    static constexpr int TG = TB / 16;                 // token groups
    static constexpr int NWAVE = TG * KG;
    static constexpr int THREADS = NWAVE * WAVE;
    static constexpr int RG = (TB + EP) * 128;         // one K group's share of a stage
    static constexpr int STAGE = KG * RG;
    static constexpr int NCOPY = STAGE / 1024;         // 1 KB copies per stage
    static constexpr int PER = NCOPY / NWAVE;          // ... per wave
    // ring depth: four stages, three when four would not fit
    static constexpr int NST = 4 * STAGE <= 160 * 1024 ? 4 : 3;
    static constexpr int LDS = NST * STAGE;
    static_assert(NCOPY % NWAVE == 0, "copies split evenly over the waves");
    static_assert(LDS <= 160 * 1024, "LDS budget");
    static_assert(TG * NE * 4 * WAVE * 4 <= LDS, "K-group reduction fits the ring");
};

// LDS offset (bytes) of 16-byte chunk `c` (0..7) of row `r` in a row-major
// [rows][64] bf16 tile; the chunk index is XOR-swizzled with the row so that
// the 16 rows read by one fragment load hit distinct banks.
__device__ __forceinline__ int kc64_off(int r, int c) { return r * 128 + ((c ^ (r & 7)) << 4); }

// NE: number of 16-expert fragments, E <= 16*NE. nk / KG slices per K group
// (the launch takes KG = 2 only for an even slice count).
template <int NE, int TB, int KG>
__global__ void __launch_bounds__((RtShape<NE, TB, KG>::THREADS))
route_bf16(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wg,
           const float* __restrict__ bias, int64_t T, int d, int E, int k, int renorm,
           int32_t* __restrict__ ids, float* __restrict__ gates, float* __restrict__ logits) {
    using SH = RtShape<NE, TB, KG>;
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wv = tid >> 6;
    const int tg = wv % SH::TG;   // token group: tokens 16*tg .. of the workgroup
    const int kg = wv / SH::TG;   // K group
    const int grp = lane >> 4;    // which 4-column group of each 16-expert fragment
    const int col = lane & 15;    // token within the wave's 16
    const int64_t t0 = (int64_t)blockIdx.x * TB + tg * 16;

    f32x4 acc[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // LDS ring of NST stages; a stage holds, for every K group, the 64-wide K
    // slice of the workgroup's TB x rows and of all EP W_g rows, 128-byte rows
    // swizzled by kc64_off. Both arrive by direct-to-LDS copies of 1 KB (8
    // rows, lane l fetching the 16-byte chunk that lands at byte 16l), so
    // every request is a whole 128-byte line and the copies of the next
    // NST-1 slices are in flight while a slice is multiplied. Rows past T or E
    // repeat the last valid row: their products are never read.
    constexpr int NST = SH::NST, PER = SH::PER, STAGE = SH::STAGE;
    constexpr int QPG = SH::RG / 1024;                // copies per K group
    const int nks = d / RT_BK / KG;                   // slices per K group
    const uint32_t lds_base = lds_offset(lds);
    const int wvu = wave_id();                        // wave index, uniform (SGPR)
    const int64_t xrow0 = (int64_t)blockIdx.x * TB;
    auto issue = [&](int s) {
        const uint32_t dst = lds_base + (s % NST) * STAGE;
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            const int q = wvu + SH::NWAVE * c;        // copy index within the stage
            const int g = q / QPG;                    // its K group
            const int r = (q % QPG) * 8 + (lane >> 3);   // row (x rows first, then W_g)
            const int ch = (lane & 7) ^ (r & 7);      // logical chunk at this lane's slot
            const int k0 = (g * nks + s) * RT_BK;
            const bf16_t* src;
            if (r < TB) {
                int64_t t = xrow0 + r;
                t = t < T ? t : T - 1;
                src = x + t * d + k0 + ch * 8;
            } else {
                int e = r - TB;
                e = e < E ? e : E - 1;
                src = wg + (int64_t)e * d + k0 + ch * 8;
            }
            dma16(src, dst + q * 1024);
        }
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
        if (s < nks) issue(s);
    if (nks >= NST - 1) wait_vmcnt<PER * (NST - 2)>();
    else wait_vmcnt<0>();
    barrier_only();
    for (int s = 0; s < nks; ++s) {
        if (s + NST - 1 < nks) issue(s + NST - 1);
        const char* xt = lds + (s % NST) * STAGE + kg * SH::RG;
        const char* wt = xt + TB * 128;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const bf16x8 q = *reinterpret_cast<const bf16x8*>(
                xt + kc64_off(tg * 16 + col, kk * 4 + grp));
#pragma unroll
            for (int fe = 0; fe < NE; ++fe) {
                const bf16x8 p = *reinterpret_cast<const bf16x8*>(
                    wt + kc64_off(fe * 16 + col, kk * 4 + grp));
                acc[fe] = mfma16x16x32(p, q, acc[fe]);
            }
        }
        if (s + 1 < nks) {
            // slice s+1 has landed once only the copies of later slices remain
            if (s + NST - 1 < nks) wait_vmcnt<PER * (NST - 2)>();
            else wait_vmcnt<0>();
            lds_barrier();
        }
    }
    if constexpr (KG == 2) {
        // the second K group's partial logits join the first group's through LDS
        __syncthreads();
        float* red = reinterpret_cast<float*>(lds) + tg * NE * 4 * WAVE + lane;
        if (kg == 1)
#pragma unroll
            for (int fe = 0; fe < NE; ++fe)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[(fe * 4 + r) * WAVE] = acc[fe][r];
        __syncthreads();
        if (kg == 1) return;
#pragma unroll
        for (int fe = 0; fe < NE; ++fe)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[fe][r] += red[(fe * 4 + r) * WAVE];
    }
    // lane holds logits of token t0+col, experts fe*16 + 4*grp + r
    const int64_t t = t0 + col;
    const bool tvalid = t < T;
    float v[NE * 4];
#pragma unroll
    for (int fe = 0; fe < NE; ++fe)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = fe * 16 + grp * 4 + r;
            float l = acc[fe][r];
            if (e < E) {
                if (bias) l += bias[e];
                if (logits && tvalid) logits[t * E + e] = l;
            }
            v[fe * 4 + r] = l;
        }
    // softmax statistics over all E experts
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NE * 4; ++i) {
        const int e = (i >> 2) * 16 + grp * 4 + (i & 3);
        if (e < E) mx = fmaxf(mx, v[i]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float z = 0.f;
#pragma unroll
    for (int i = 0; i < NE * 4; ++i) {
        const int e = (i >> 2) * 16 + grp * 4 + (i & 3);
        if (e < E) z += __expf(v[i] - mx);
    }
    z += __shfl_xor(z, 16, 64);
    z += __shfl_xor(z, 32, 64);
    // top-k: k rounds of argmax over the untaken experts
    unsigned long long taken = 0ull;
    float selv[16];
    int sele[16];
    float ssum = 0.f;
    for (int j = 0; j < k; ++j) {
        float bv = -INFINITY;
        int be = 0x7fffffff;
#pragma unroll
        for (int i = 0; i < NE * 4; ++i) {
            const int e = (i >> 2) * 16 + grp * 4 + (i & 3);
            const bool ok = e < E && !((taken >> i) & 1ull);
            if (ok && (v[i] > bv || (v[i] == bv && e < be))) { bv = v[i]; be = e; }
        }
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
            const float ov = __shfl_xor(bv, o, 64);
            const int oe = __shfl_xor(be, o, 64);
            if (ov > bv || (ov == bv && oe < be)) { bv = ov; be = oe; }
        }
        // the owner lane of expert be marks it taken
        if (((be & 15) >> 2) == grp) taken |= 1ull << ((be >> 4) * 4 + (be & 3));
        selv[j] = bv;
        sele[j] = be;
        ssum += __expf(bv - mx);
    }
    if (grp == 0 && tvalid) {
        for (int j = 0; j < k; ++j) {
            const float pe = __expf(selv[j] - mx);
            ids[t * k + j] = sele[j];
            gates[t * k + j] = renorm ? pe / ssum : pe / z;
        }
    }
}

// Few tokens, in two launches. One workgroup that reads all of W_g gets some 25 GB/s
// of it (64 experts x 2048: 256 KB, 13 us for a single token), and a short grid has
// no others to share the reading with; so the product is split over blocks of 16
// experts as well, through the logits output, and softmax and top-k follow. Both
// launches add up in route_bf16's order, so that a token's routing has the same bits
// however many tokens it comes with, and whether or not the logits are asked for.

// logits[t][e] = x[t] . W_g[e] + bias[e]: 16 tokens x 16 experts per workgroup. KG
// groups of waves take a contiguous share of K each, as route_bf16's do. A wave holds
// the operands of U steps of 32 k in registers, straight from global memory, and the
// steps of its next round in flight; the accumulator of the group goes from wave to
// wave in K order through LDS (a chain of 32 MFMAs per group at d = 2048; 0.6 us more
// than eight shares of K that are summed at the end, at T = 1, E = 64, d = 2048).
constexpr int RL_WAVES = 8;
template <int KG>
__global__ void __launch_bounds__(RL_WAVES * WAVE)
route_logits(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wg,
             const float* __restrict__ bias, int64_t T, int d, int E, float* __restrict__ logits) {
    constexpr int NW = RL_WAVES / KG;   // waves per K group
    constexpr int U = 8;
    __shared__ f32x4 sum[KG][WAVE];
    const int lane = threadIdx.x & 63, wv = wave_id();
    const int kg = wv / NW, w = wv % NW;
    const int col = lane & 15, grp = lane >> 4;
    const int64_t t0 = (int64_t)blockIdx.x * 16;
    const int e0 = blockIdx.y * 16;
    const int n = d / 32 / KG;          // steps per K group
    const int k0 = kg * n * 32 + grp * 8;
    const bf16_t* xr = x + (t0 + col < T ? t0 + col : T - 1) * d + k0;
    const bf16_t* wr = wg + (int64_t)min(e0 + col, E - 1) * d + k0;
    bf16x8 q[2][U], p[2][U];            // by round parity
    auto load = [&](auto par, int s) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value;
        if (s >= n) return;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int o = min(s + u, n - 1) * 32;
            q[P][u] = *reinterpret_cast<const bf16x8*>(xr + o);
            p[P][u] = *reinterpret_cast<const bf16x8*>(wr + o);
        }
    };
    // steps [s0, s0 + NW * U), U per wave and turn
    auto round = [&](auto par, int s0) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value;
        const int s = s0 + w * U;
        load(std::integral_constant<int, P ^ 1>{}, s + NW * U);
        for (int turn = 0; turn < NW; ++turn) {
            if (turn == w && s < n) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                if (s > 0) acc = sum[kg][lane];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (s + u < n) acc = mfma16x16x32(p[P][u], q[P][u], acc);
                sum[kg][lane] = acc;
            }
            lds_barrier();
        }
    };
    load(std::integral_constant<int, 0>{}, w * U);
    for (int s0 = 0; s0 < n; s0 += 2 * NW * U) {
        round(std::integral_constant<int, 0>{}, s0);
        if (s0 + NW * U < n) round(std::integral_constant<int, 1>{}, s0 + NW * U);
    }
    if (threadIdx.x >= 256) return;
    const int tok = threadIdx.x >> 4, ee = threadIdx.x & 15, e = e0 + ee;
    // lane 16 * (ee / 4) + tok holds expert ee in element ee % 4
    float v = sum[0][(ee >> 2) * 16 + tok][ee & 3];
    if constexpr (KG == 2) v += sum[KG - 1][(ee >> 2) * 16 + tok][ee & 3];
    if (e >= E || t0 + tok >= T) return;
    if (bias) v += bias[e];
    logits[(t0 + tok) * E + e] = v;
}

// Softmax and top-k of given logits, one wave per token. An expert's place is the
// number of experts that come before it: larger logits, and equal ones of lower ids.
// Counting them against the row in LDS (broadcast reads) takes no chain of
// cross-lane exchanges, of which k rounds of argmax take 12 each. A NaN comes before
// nothing and has no place; places without an expert keep id 0x7fffffff.
constexpr int RP_TOK = 4;
__global__ void __launch_bounds__(RP_TOK * WAVE)
route_pick(const float* __restrict__ logits, int64_t T, int E, int k, int renorm,
           int32_t* __restrict__ ids, float* __restrict__ gates) {
    __shared__ __align__(16) float row[RP_TOK][256];
    __shared__ __align__(16) float ex[RP_TOK][256];
    __shared__ float selv[RP_TOK][16];
    __shared__ int sele[RP_TOK][16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t t = (int64_t)blockIdx.x * RP_TOK + w;
    const bool valid = t < T;
    float* l = row[w];
    float mx = -INFINITY, z = 0.f;
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = lane + i * WAVE;
        v[i] = valid && e < E ? logits[t * E + e] : -INFINITY;
        l[e] = v[i];
        if (e < E) mx = fmaxf(mx, v[i]);
    }
    if (lane < 16) { selv[w][lane] = -INFINITY; sele[w][lane] = 0x7fffffff; }
    mx = wave_max(mx);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = lane + i * WAVE;
        ex[w][e] = e < E ? __expf(v[i] - mx) : 0.f;
    }
    __syncthreads();
    // the exponentials add up as in route_bf16: four groups, each over its runs of
    // four experts, then the groups
    for (int o = 4 * (lane & 3); o < E; o += 16) {
        const f32x4 u = *reinterpret_cast<const f32x4*>(ex[w] + o);
#pragma unroll
        for (int r = 0; r < 4; ++r) z += u[r];
    }
    z += __shfl_xor(z, 1, 64);
    z += __shfl_xor(z, 2, 64);
    // (entries E .. 255 of the row are -infinity and come before nothing)
    int place[4] = {0, 0, 0, 0};
    for (int o = 0; o < E; o += 4) {
        const f32x4 u = *reinterpret_cast<const f32x4*>(l + o);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i * WAVE >= E) break;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                place[i] += (u[r] > v[i]) | ((u[r] == v[i]) & (o + r < lane + i * WAVE));
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = lane + i * WAVE;
        if (e < E && v[i] == v[i] && place[i] < k) { selv[w][place[i]] = v[i]; sele[w][place[i]] = e; }
    }
    __syncthreads();
    if (lane < k && valid) {
        const float pe = __expf(selv[w][lane] - mx);
        float sum = z;
        if (renorm) {
            sum = 0.f;
            for (int j = 0; j < k; ++j) sum += __expf(selv[w][j] - mx);
        }
        ids[t * k + lane] = sele[w][lane];
        gates[t * k + lane] = pe / sum;
    }
}

// f32: 16 tokens per workgroup. The product runs on v_mfma_f32_16x16x4_f32
// straight from global memory, each of the four waves taking a quarter of K for
// all experts; the partial logits meet in LDS, and 16 lanes per token then take
// softmax and top-k. A lane loads 4 consecutive k (16 bytes) and feeds them to
// four MFMAs, so the k of MFMA j, lane group g are 16q + 4g + j on both operands.
// Few tokens and a short K: latency is the bound (T = 1024, d = 256, E = 8: 172
// us with one thread per token and serial dot products).
constexpr int RF_TOK = 16;
constexpr int RF_THREADS = 256;

template <int NE>   // 16-expert fragments, E <= 16 * NE
__global__ void __launch_bounds__(RF_THREADS)
route_f32(const float* __restrict__ x, const float* __restrict__ wg,
          const float* __restrict__ bias, int64_t T, int d, int E, int k, int renorm,
          int32_t* __restrict__ ids, float* __restrict__ gates, float* __restrict__ logits) {
    constexpr int EP = NE * 16;
    __shared__ float part[4][RF_TOK][EP];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int64_t t0 = (int64_t)blockIdx.x * RF_TOK;
    {
        f32x4 acc[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int kq = d / 4;   // this wave's share of K (a multiple of 16)
        const int64_t k0 = (int64_t)wv * kq + grp * 4;
        const int64_t tr = t0 + col < T ? t0 + col : T - 1;
        const float* xr = x + tr * d + k0;
        for (int q = 0; q < kq; q += 16) {
            const f32x4 a = *reinterpret_cast<const f32x4*>(xr + q);
#pragma unroll
            for (int fe = 0; fe < NE; ++fe) {
                const int e = min(fe * 16 + col, E - 1);
                const f32x4 w = *reinterpret_cast<const f32x4*>(wg + (int64_t)e * d + k0 + q);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[fe] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j], a[j], acc[fe], 0, 0, 0);
            }
        }
        // lane holds token col, experts fe * 16 + 4 * grp + r
#pragma unroll
        for (int fe = 0; fe < NE; ++fe)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[wv][col][fe * 16 + grp * 4 + r] = acc[fe][r];
    }
    __syncthreads();
    // 16 lanes per token: lane j takes experts j, j + 16, ...
    const int tok = threadIdx.x >> 4, j16 = threadIdx.x & 15;
    const int64_t t = t0 + tok;
    float* l = part[0][tok];
    float mx = -INFINITY;
    for (int e = j16; e < E; e += 16) {
        float v = (l[e] + part[1][tok][e]) + (part[2][tok][e] + part[3][tok][e]);
        if (bias) v += bias[e];
        l[e] = v;
        if (logits && t < T) logits[t * E + e] = v;
        mx = fmaxf(mx, v);
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    float z = 0.f;
    for (int e = j16; e < E; e += 16) z += __expf(l[e] - mx);
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) z += __shfl_xor(z, o, 64);
    // k rounds over the experts not taken yet: the largest logit, ties to the
    // lower id. A NaN is never larger than a number; where the lowest free
    // expert's logit is NaN, no number is larger than it either, and it is taken.
    unsigned taken = 0;   // bit i: expert j16 + 16 * i
    float pe[16];
    int be_[16];
    float ssum = 0.f;
    for (int j = 0; j < k; ++j) {
        float bv = -INFINITY;
        int be = E, first = E, nan = 0;
        for (int i = 0, e = j16; e < E; ++i, e += 16) {
            if ((taken >> i) & 1u) continue;
            const float v = l[e];
            if (first == E) { first = e; nan = v != v; }
            if (v > bv || (v == bv && e < be)) { bv = v; be = e; }
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const float ov = __shfl_xor(bv, o, 64);
            const int oe = __shfl_xor(be, o, 64), of = __shfl_xor(first, o, 64);
            const int on = __shfl_xor(nan, o, 64);
            if (ov > bv || (ov == bv && oe < be)) { bv = ov; be = oe; }
            if (of < first) { first = of; nan = on; }
        }
        if (nan) { be = first; bv = __builtin_nanf(""); }
        if ((be & 15) == j16) taken |= 1u << (be >> 4);
        be_[j] = be;
        pe[j] = __expf(bv - mx);
        ssum += pe[j];
    }
    if (j16 == 0 && t < T)
        for (int j = 0; j < k; ++j) {
            ids[t * k + j] = be_[j];
            gates[t * k + j] = renorm ? pe[j] / ssum : pe[j] / z;
        }
}

template <int NE, int TB, int KG>
hipError_t launch_route_shape(const void* x, const void* wg, const float* bias, int64_t T,
                              int d, int E, int k, bool renorm, int32_t* ids, float* gates,
                              float* logits, hipStream_t st) {
    using SH = RtShape<NE, TB, KG>;
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(route_bf16<NE, TB, KG>),
        hipFuncAttributeMaxDynamicSharedMemorySize, SH::LDS);
    if (attr != hipSuccess) return attr;
    const dim3 grid((unsigned)((T + TB - 1) / TB));
    hipLaunchKernelGGL((route_bf16<NE, TB, KG>), grid, dim3(SH::THREADS), SH::LDS, st,
                       static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(wg), bias, T,
                       d, E, k, (int)renorm, ids, gates, logits);
    probe::mark("route_bf16", st);
    return hipGetLastError();
}

// K groups of the bf16 router (RtShape)
inline int k_groups(int64_t T, int d, int E) {
    return E <= 128 && T < 32768 && (d / RT_BK) % 2 == 0 ? 2 : 1;
}

template <int NE>
hipError_t launch_route_bf16(const void* x, const void* wg, const float* bias, int64_t T,
                             int d, int E, int k, bool renorm, int32_t* ids, float* gates,
                             float* logits, hipStream_t st) {
    if constexpr (NE >= 8) {
        if (T >= 65536)
            return launch_route_shape<NE, 128, 1>(x, wg, bias, T, d, E, k, renorm, ids, gates,
                                                  logits, st);
    }
    if constexpr (NE <= 8) {
        if (k_groups(T, d, E) == 2)
            return launch_route_shape<NE, 64, 2>(x, wg, bias, T, d, E, k, renorm, ids, gates,
                                                 logits, st);
    }
    return launch_route_shape<NE, 64, 1>(x, wg, bias, T, d, E, k, renorm, ids, gates, logits, st);
}

// Two launches where W_g is large (from 128 KB on) and the tokens are few. Times in us
// of one launch and of two (T in brackets):
//  - E = 64, d = 2048: [1] 17.0, 13.8; [1024] 17.4, 16.5; [1536] 17.6, 21.0. E = 48:
//    [1024] 16.7, 15.8; [1536] 16.8, 20.3. Up to 64 experts, as long as the product's
//    16 x 16 tiles run in one round of the 256 CUs.
//  - E = 96, d = 2048: [768] 28.7, 23.5; [1024] 28.8, 23.7; [1536] 28.9, 29.1. E = 128, d =
//    2880: [300] 35.6, 23; [768] 35.7, 30.2. E = 256, d = 2048: [384] 53, 42.1.
//  - the second launch's counting grows with E, the product with d: E = 256, d = 256:
//    [17] 30.2, 34.3; d = 512: [17] 33.0, 33.9, [128] 36.4, 35.0; d = 768: [128] 39.1, 34.9.
//  - up to 32 experts one launch stages few rows of W_g: E = 16, d = 4096: [1] 16.3,
//    15.7, [17] 16.5, 18.6; E = 8, d = 8192: [1] 25.0, 19.0, [4096] 26.7, 31.8; E = 32, d =
//    2048: [1] 12.3, 13.0. A long K and one tile of tokens only.
inline bool two_launches(int64_t T, int d, int E) {
    const int64_t tiles = (T + 15) / 16 * ((E + 15) / 16);
    if (E <= 32) return T <= 16 && d >= 4096 && (int64_t)E * d >= 65536;
    if ((int64_t)E * d < 65536 || d < 2 * E) return false;
    return E <= 64 ? tiles <= 256 : T * E <= 98304;
}

}  // namespace

hipError_t route(const void* x, const void* wg, const float* bias, int64_t T, int d, int E,
                 int k, bool f32, bool renorm, int32_t* ids, float* gates, float* logits,
                 hipStream_t st) {
    if (f32) {
        const dim3 grid((unsigned)((T + RF_TOK - 1) / RF_TOK));
        auto kernel = E <= 16 ? route_f32<1> : E <= 64 ? route_f32<4> : route_f32<16>;
        hipLaunchKernelGGL(kernel, grid, dim3(RF_THREADS), 0, st, static_cast<const float*>(x),
                           static_cast<const float*>(wg), bias, T, d, E, k, (int)renorm, ids,
                           gates, logits);
        probe::mark("route_f32", st);
        return hipGetLastError();
    }
    if (logits && two_launches(T, d, E)) {
        auto product = k_groups(T, d, E) == 2 ? route_logits<2> : route_logits<1>;
        hipLaunchKernelGGL(product, dim3((unsigned)((T + 15) / 16), (unsigned)((E + 15) / 16)),
                           dim3(RL_WAVES * WAVE), 0, st, static_cast<const bf16_t*>(x),
                           static_cast<const bf16_t*>(wg), bias, T, d, E, logits);
        probe::mark("route_logits", st);
        hipLaunchKernelGGL(route_pick, dim3((unsigned)((T + RP_TOK - 1) / RP_TOK)), dim3(RP_TOK * WAVE), 0,
                           st, logits, T, E, k, (int)renorm, ids, gates);
        probe::mark("route_pick", st);
        return hipGetLastError();
    }
    if (E <= 32) return launch_route_bf16<2>(x, wg, bias, T, d, E, k, renorm, ids, gates, logits, st);
    if (E <= 64) return launch_route_bf16<4>(x, wg, bias, T, d, E, k, renorm, ids, gates, logits, st);
    if (E <= 128) return launch_route_bf16<8>(x, wg, bias, T, d, E, k, renorm, ids, gates, logits, st);
    return launch_route_bf16<16>(x, wg, bias, T, d, E, k, renorm, ids, gates, logits, st);
}

}  // namespace moe
