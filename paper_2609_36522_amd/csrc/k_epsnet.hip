// Batched evaluation of the cache misses by the patch-MLP noise network, one fused
// persistent kernel for gfx950 (the single batched forward pass over the misses, Sec. 2.2).
//
// Work item = (miss j, block of 128 tokens, half of the hidden-out units of GEMM2). The
// misses of all samples of a handle form one list (sample-major, each sample's misses in
// its ascending order); a prefix over the samples' miss counts maps a list entry back to
// (sample, miss). For one item the block
//   0. gathers the 128 tokens (2x2 patches, 16 features) of latent x_t, rounds to bf16;
//   1. h1^T = GELU(W1^T x^T + e_t) in K-chunks of 256 units: MFMA 32x32x16 bf16, K = 16, e_t as
//      the accumulator's initial value; bf16 result (as 2 h1, with W2 stored halved) in LDS
//      ([token][unit], padded rows), two chunk buffers of 66 KB;
//   2. h2^T += W2^T h1^T chunk by chunk: each of the 8 waves owns 64 output units x 128
//      tokens (128 accumulator registers); W2^T fragments stream from L2 in MFMA-fragment
//      order (1 KB contiguous per wave load), two register stages in flight; the GEMM1 and
//      GELU of the next chunk are computed between the MFMA groups of the current one;
//   3. eps^T = W3^T GELU(h2^T), MFMA fed straight from the GEMM2 accumulators (reduction
//      index permuted to the accumulator layout; W3 stored pre-permuted);
//   4. per-wave partials summed in a fixed order through LDS and unpatchified.
// Launches of few misses, whose 128-token items would leave most CUs idle, take smaller items
// (fine_items). Two ways to finish the others (chosen per launch from the miss count, identically
// in every block, by the time each takes):
//   split outputs: each item is a work item of its own and writes its half's partial output;
//      the Picard kernel adds the halves in a fixed order and writes the cache;
//   whole outputs (at most two halves): one block runs both halves of a token block in turn,
//      adds their outputs in the same fixed order and writes the fresh output straight into
//      the cache (Eq. (6)-(7), output side). The second half takes its K-chunks in the order
//      2, 3, 1, 0 (generally H/256 - 2, H/256 - 1, H/256 - 3, ..., 0), so the first of them is
//      the h1 chunk the first half left in LDS: no gather, no h1 prologue, one chunk of GELU
//      work less. Odd halves take that order in both ways, so both give the same bits.
// 128 tokens per item make every W2 byte feed 128 FLOP, which keeps the W2 stream under the
// per-CU vector-memory bandwidth; the price is computing h1 (largely) once per half.
// All products are bf16 x bf16 with fp32 accumulation.
//
// Accumulator layout of v_mfma_f32_32x32x16_bf16 (C/D, 16 floats per lane):
//   reg r of lane l holds row (r/4)*8 + (l/32)*4 + r%4, column l%32.
// Operands: lane l supplies row l%32 of A (column l%32 of B) and 8 reduction slots; A and B
// use the same lane->slot convention, so any consistent slot->k assignment is valid.
#include <math.h>

#include <type_traits>

#include <hip/hip_ext.h>

#include "pa_device.h"
#include "pa_parareal.h"
#include "pa_slide.h"

namespace pa {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kTokMax = 128;            // tokens per work item (fewer in launches of few misses)
constexpr int kNH = 512;                // GEMM2 output units per work item
constexpr int kKC = 256;                // h1 units per LDS buffer (K-chunk); two buffers
constexpr int kWaves = 8;               // wave w owns output units [64w, 64w + 64) of the item
constexpr int kFeat = 16;               // 2x2 patch x 4 channels
constexpr int kXRow = kFeat + 8;        // padded LDS row of the token tile (bf16)

// Twice the erf-GELU: 2 x Phi(x) = (x + a) - a 2Q(a) with a = |x| and Q the normal upper tail,
// branch-free (x + a = 2 max(x, 0) exactly). 2Q(a) = 2^(-(P(a) - 1)) with P a degree-7
// polynomial fitted to -log2 Q on [0, 7] toward the minimax absolute error of the result
// (derivation: gelu_fit.py: what a deviation costs once the output is rounded to bf16 is its
// absolute size), its constant term lowered by 1. P increases monotonically for all a >= 0 and
// keeps tracking -log2 Q beyond 7 (a Q(a) < 1e-11 there); for very large a it overflows to
// +inf and Q to 0, so no clamp is needed. One v_add_f32, eight FMAs and one v_exp_f32 per
// element; in fp32 the result is within 4e-7 max(1, |x|) of twice the exact erf GELU. The
// factor 2 is exact and is undone exactly in the next product: W2 and W3 are stored halved
// (bf16 halving is exact for normal values), and bf16(2g) = 2 bf16(g), so every bf16 x bf16
// product equals the one with GELU(x) and the unhalved weight. Every GELU output is rounded to
// bf16 next; the residual error is kept within a few fp32 rounding errors of the result so
// that it adds few rounding flips to those of the fp32 accumulation of the products.
__device__ __forceinline__ float gelu2_erf(float x) {
    const float a = fabsf(x);
    float p = fmaf(a, 1.1180667343069217e-06f, -4.9184127419721335e-05f);
    p = fmaf(p, a, 0.0008520559640601277f);
    p = fmaf(p, a, -0.008282574824988842f);
    p = fmaf(p, a, 0.05366271361708641f);
    p = fmaf(p, a, 0.45861566066741943f);
    p = fmaf(p, a, 1.1512444019317627f);
    p = fmaf(p, a, -1.0669231414794922e-05f);   // P(a) - 1
    const float q2 = __builtin_amdgcn_exp2f(-p);  // 2 Q(a)
    return fmaf(-a, q2, x + a);
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Element index of the token tile <-> latent position. Consecutive e walk along w so that
// global accesses of a block are row-contiguous.
struct TokPos {
    int tl, f, idx;
};
template <int kTok>
__device__ __forceinline__ TokPos tok_pos(int e, int tb, int Himg, int Wimg) {
    constexpr int kLog = kTok == 128 ? 7 : (kTok == 64 ? 6 : 5);
    static_assert(kTok == (1 << kLog), "32, 64 or 128 tokens per item");
    const int dw = e & 1, tl = (e >> 1) & (kTok - 1), dh = (e >> (kLog + 1)) & 1, c = e >> (kLog + 2);
    const int half_w = Wimg >> 1;
    const int tok = tb * kTok + tl;
    const int hp = tok / half_w, wp = tok - hp * half_w;
    TokPos p;
    p.tl = tl;
    p.f = c * 4 + dh * 2 + dw;
    p.idx = (c * Himg + 2 * hp + dh) * Wimg + 2 * wp + dw;
    return p;
}

}  // namespace

// Position i of a half's K-chunk order: natural order for even halves; odd halves start with the
// chunk a whole-output block still holds in buffer 0 (KCH - 2), then KCH - 1, KCH - 3, ..., 0.
template <int KCH>
__device__ __forceinline__ int korder(int odd, int i) {
    return !odd ? i : (i == 0 ? KCH - 2 : (i == 1 ? KCH - 1 : KCH - 1 - i));
}

// Fine items, for launches whose 128-token items would leave most CUs without work: item =
// (list entry, 32 TS tokens, UF output units). The block computes h1 of all H units of its tokens
// into LDS once (KP = 2: half of K at a time), then GEMM2 from there; each wave owns 32 (UF < 512)
// or 64 output units, and its W2^T fragments are in flight from before the gather. Every
// accumulation runs in the order of the 128-token items (K-chunks, the 64 units of a GEMM3 chain,
// the waves of a half), so the outputs are the same bits. UF = 512 covers a half and writes its
// split partial output; a smaller UF writes one partial output per 64 units (a wave's share of a
// half) to Ep[group][list entry], and the consumer adds them in the order the half's reduction takes.
// Bound by one CU's stream of W2^T from L2 (UF x H x 2 bytes at ~46 B/clk: 2.2 us at UF = 128,
// H = 1024) after its h1 GELUs (2.4 us per 32 tokens at H = 1024), hence few units and few tokens
// per item while CUs are free. Launch time with 128-token items -> with these (1024 tokens,
// H = 1024): 1 miss 34 -> 12 us, 2 misses 35 -> 15, 4 36 -> 20, 8 38 -> 28; 256 tokens, H = 512:
// 16 misses 26 -> 11 us; 768 tokens, H = 2048: 1 miss 59 -> 27 us, 5 misses 67 -> 52.
// WHOLE: the item is all units of its tokens, half after half from one h1, and its output goes
// straight into the cache like that of a whole 128-token item.
// map(item): list entry, token block of 32 TS tokens and unit group of an item.
struct FineItem {
    int gm, tb, ug;
};
template <int H, int TS, int UF, int KP, bool WHOLE, class Map>
__device__ __forceinline__ void fine_items(const Dev& d, __bf16* h1, __bf16* xs, float* es, const int* mpre,
                                           const int* fmiss, int fnewest, int items, Map map) {
    constexpr int NT = kWaves * 64, kTok = 32 * TS, HP = H / KP, HR = HP + 8, KS = H / 16, KCH = H / kKC;
    constexpr int NH = WHOLE ? H / kNH : 1;          // halves the item takes in turn
    static_assert(!WHOLE || (UF == kNH && KP == 1), "h1 of all units serves every half");
    constexpr int UBW = UF == 512 ? 2 : 1;           // 32-unit blocks per wave
    constexpr int UB = UF / 32;                      // 32-unit blocks per item
    // k-steps of W2^T fragments in flight: half of K at UBW = 1 (one wave's 32 KB at H = 1024; 16
    // steps leave the stream waiting for round trips, 50 serial steps 882 against 866 us).
    constexpr int DEPTH = UBW == 2 ? 8 : (H == 512 ? 16 : 32);
    constexpr int KCP = KCH / KP;                    // K-chunks (and h1 unit blocks per wave) per pass
    static_assert(UF == 512 || (TS == 1 && (UF == 128 || UF == 256)), "whole GEMM3 chains (64 units)");
    static_assert(KS / KP % DEPTH == 0, "whole fragment groups");
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, l32 = lane & 31;
    const __amdgpu_buffer_rsrc_t w2r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(d.w2f), (short)0, H * H * 2, 0x00020000);
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                           0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const bool active = UB >= 8 || w < UB;
    for (int item = blockIdx.x; item < items; item += gridDim.x) {
        const FineItem it = map(item);
        const int gm = it.gm, tb = it.tb;
        int n = 0;
        while (mpre[n + 1] <= gm) ++n;               // sample of list entry gm (uniform)
        const int jm = gm - mpre[n];
        const Ctrl* ctrl = d.ctrl + n;
        const int t = d.fused_slide ? fmiss[jm] : (d.pr_dev ? fmiss[n] : ctrl->miss_idx[jm]);
        const int newest = d.fused_slide ? fnewest : (d.pr_dev ? t : ctrl->newest);
        const int ns0 = WHOLE ? 0 : it.ug * UF / kNH;
        const int ub00 = it.ug * UB + (UB == 4 ? (w & 3) : w * UBW);   // this wave's first unit block

        // ---- W2^T fragments of the first k-steps, then the gather: one round trip to memory
        bf16x8 A[DEPTH][UBW];
        auto load_a = [&](int hf, int i, int j) {    // k-step i of the half's order, into stage j
            const int ks = korder<KCH>((ns0 + hf) & 1, i / 16) * 16 + i % 16;
            const int ub0 = ub00 + hf * (kNH / 32);
#pragma unroll
            for (int u = 0; u < UBW; ++u)
                A[j][u] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                    w2r, lane * 16, ((ub0 + u) * KS + ks) * 64 * 16, 0));
        };
        // K-chunk in place q of pass ps of h1 (KP = 1: in natural order, for either order of a half)
        auto h1_chunk = [&](int ps, int q) { return KP == 1 ? q : korder<KCH>(ns0 & 1, ps * KCP + q); };
        const float* xt = d.X + ((size_t)n * (d.T + 1) + min(t, newest)) * d.D;
        const float* et = d.temb + (size_t)t * H;
        constexpr int kPer = kTok * kFeat / NT, kEs = (H / 4 + NT - 1) / NT;
        float xv[kPer];
        float4 ev[kEs];
        bf16x8 w1a[KCP];
        auto load_w1 = [&](int ps) {                 // the wave's 32 units of each K-chunk of a pass
#pragma unroll
            for (int q = 0; q < KCP; ++q)
                w1a[q] = *reinterpret_cast<const bf16x8*>(
                    d.w1t + (size_t)(h1_chunk(ps, q) * kKC + w * 32 + l32) * kFeat + g * 8);
        };
#pragma unroll
        for (int k = 0; k < kPer; ++k) xv[k] = xt[tok_pos<kTok>(tid + k * NT, tb, d.Himg, d.Wimg).idx];
#pragma unroll
        for (int k = 0; k < kEs; ++k)
            if (tid + k * NT < H / 4) ev[k] = reinterpret_cast<const float4*>(et)[tid + k * NT];
        load_w1(0);
        if (active) {
#pragma unroll
            for (int j = 0; j < DEPTH; ++j) load_a(0, j, j);
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const TokPos p = tok_pos<kTok>(tid + k * NT, tb, d.Himg, d.Wimg);
            xs[p.tl * kXRow + p.f] = (__bf16)xv[k];
        }
#pragma unroll
        for (int k = 0; k < kEs; ++k)
            if (tid + k * NT < H / 4) reinterpret_cast<float4*>(es)[tid + k * NT] = ev[k];
        __syncthreads();

        f32x16 acc[UBW][TS];
        const __bf16* hb = h1 + l32 * HR + g * 8;
        // DEPTH k-steps from k-step i0 of the half's order; reloads the stages if more follow.
        constexpr int KSP = KS / KP;                 // k-steps per pass
        auto steps = [&](int hf, int i0, auto more_c) {
            int p0 = 0;                              // h1 place of k-step i0 + j, less 16 j % 16
#pragma unroll
            for (int j = 0; j < DEPTH; ++j) {
                if (j % 16 == 0)
                    p0 = KP == 1 ? korder<KCH>((ns0 + hf) & 1, (i0 + j) / 16) * kKC + i0 % 16 * 16 : (i0 + j) % KSP * 16;
                bf16x8 B[TS];
#pragma unroll
                for (int sl = 0; sl < TS; ++sl)
                    B[sl] = *reinterpret_cast<const bf16x8*>(hb + sl * 32 * HR + p0 + j % 16 * 16);
#pragma unroll
                for (int sl = 0; sl < TS; ++sl)
#pragma unroll
                    for (int u = 0; u < UBW; ++u) acc[u][sl] = mfma32(A[j][u], B[sl], acc[u][sl]);
                if constexpr (decltype(more_c)::value) load_a(hf, i0 + DEPTH + j, j);
            }
        };
        auto zero_acc = [&] {
#pragma unroll
            for (int u = 0; u < UBW; ++u)
#pragma unroll
                for (int sl = 0; sl < TS; ++sl) acc[u][sl] = zero16;
        };
        zero_acc();
#pragma unroll
        for (int ps = 0; ps < KP; ++ps) {
            // ---- h1 of the pass's units: rows [token][units, chunk by chunk]
#pragma unroll
            for (int q = 0; q < KCP; ++q) {
                const int u0 = h1_chunk(ps, q) * kKC + w * 32, p0 = q * kKC + w * 32;
#pragma unroll
                for (int sl = 0; sl < TS; ++sl) {
                    const bf16x8 b = *reinterpret_cast<const bf16x8*>(xs + (sl * 32 + l32) * kXRow + g * 8);
                    f32x16 c0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float4 e4 = *reinterpret_cast<const float4*>(es + u0 + g * 4 + r * 8);
                        c0[r * 4 + 0] = e4.x;
                        c0[r * 4 + 1] = e4.y;
                        c0[r * 4 + 2] = e4.z;
                        c0[r * 4 + 3] = e4.w;
                    }
                    c0 = mfma32(w1a[q], b, c0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        bf16x4 v;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = (__bf16)gelu2_erf(c0[r * 4 + i]);
                        *reinterpret_cast<bf16x4*>(h1 + (sl * 32 + l32) * HR + p0 + r * 8 + g * 4) = v;
                    }
                }
            }
            if (ps + 1 < KP) load_w1(ps + 1);
            __syncthreads();
            // ---- GEMM2 over them
            if (active) {
                #pragma unroll 1
                for (int i = 0; i + DEPTH < KSP; i += DEPTH) steps(0, ps * KSP + i, std::true_type{});
                if (ps + 1 < KP) steps(0, (ps + 1) * KSP - DEPTH, std::true_type{});
                else steps(0, KS - DEPTH, std::false_type{});
            }
            if (ps + 1 < KP) __syncthreads();        // the pass's h1 is read before the next one's
        }

        // ---- GEMM3: chains of 64 units (two unit blocks) per token slice
        f32x16 acc3[TS];
        auto gemm3 = [&](int ub0, int u) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const bf16x8 a3 = *reinterpret_cast<const bf16x8*>(
                    d.w3p + (((size_t)(ub0 + u) * 2 + jj) * 64 + lane) * 8);
#pragma unroll
                for (int sl = 0; sl < TS; ++sl) {
                    bf16x8 b3;
#pragma unroll
                    for (int i = 0; i < 8; ++i) b3[i] = (__bf16)gelu2_erf(acc[u][sl][jj * 8 + i]);
                    acc3[sl] = mfma32(a3, b3, acc3[sl]);
                }
            }
        };
#pragma unroll
        for (int sl = 0; sl < TS; ++sl) acc3[sl] = zero16;
        const int half_w = d.Wimg >> 1;
        float* red = reinterpret_cast<float*>(h1);
        if constexpr (UBW == 2) {
            // WHOLE: the first half's sums wait in registers (8 per slice) while the second takes
            // h1, which the reduction overwrites.
            float keep[TS][8];
            if constexpr (NH == 2) {
#pragma unroll
                for (int j = 0; j < DEPTH; ++j) load_a(1, j, j);
            }
            gemm3(ub00, 0);
            gemm3(ub00, 1);
            if constexpr (NH == 2) {
#pragma unroll
                for (int sl = 0; sl < TS; ++sl) {
#pragma unroll
                    for (int r = 0; r < 8; ++r) keep[sl][r] = acc3[sl][r];
                    acc3[sl] = zero16;
                }
                zero_acc();
                #pragma unroll 1
                for (int i = 0; i + DEPTH < KS; i += DEPTH) steps(1, i, std::true_type{});
                steps(1, KS - DEPTH, std::false_type{});
                gemm3(ub00 + kNH / 32, 0);
                gemm3(ub00 + kNH / 32, 1);
            }
            float4 run = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int hf = 0; hf < NH; ++hf) {
                __syncthreads();                         // h1 operands, or the last half's sums, are read
#pragma unroll
                for (int sl = 0; sl < TS; ++sl) {
                    float* dst = red + ((size_t)w * kTok + sl * 32 + l32) * kFeat + g * 4;
                    const bool kept = NH == 2 && hf == 0;
                    float v[8];
#pragma unroll
                    for (int r = 0; r < 8; ++r) v[r] = kept ? keep[sl][r] : acc3[sl][r];
                    *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                    *reinterpret_cast<float4*>(dst + 8) = make_float4(v[4], v[5], v[6], v[7]);
                }
                __syncthreads();
                if (tid < kTok * (kFeat / 4)) {          // as in the 128-token items
                    const int tl = tid & (kTok - 1), c = tid / kTok;
                    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                    for (int ww = 0; ww < kWaves; ++ww) {
                        const float4 v = *reinterpret_cast<const float4*>(red + ((size_t)ww * kTok + tl) * kFeat + c * 4);
                        sum = make_float4(sum.x + v.x, sum.y + v.y, sum.z + v.z, sum.w + v.w);
                    }
                    run = hf == 0 ? sum : make_float4(run.x + sum.x, run.y + sum.y, run.z + sum.z, run.w + sum.w);
                    if (hf == NH - 1) {
                        const int tok = tb * kTok + tl, hp = tok / half_w, wp = tok - hp * half_w;
                        float* out = WHOLE ? d.Eh + ((size_t)n * d.T + t) * d.D
                                           : d.Ep + (((size_t)ns0 * d.N + n) * d.P + jm) * d.D;
                        float* o = out + ((size_t)c * d.Himg + 2 * hp) * d.Wimg + 2 * wp;
                        *reinterpret_cast<float2*>(o) = make_float2(run.x, run.y);
                        *reinterpret_cast<float2*>(o + d.Wimg) = make_float2(run.z, run.w);
                    }
                }
            }
            __syncthreads();                         // red is read before the next item's h1
        } else {
            // The wave of the chain's first unit block hands its sums to the wave of the second
            // (rows 0..15 of the tile: accumulator registers 0..7).
            const bool first = (ub00 & 1) == 0;
            float* pass = red + ((size_t)(w & ~1) * TS * 64 + lane) * 8;
            if (active && first) gemm3(ub00, 0);
            __syncthreads();                         // every wave has read its h1 operands
            if (active && first) {
#pragma unroll
                for (int sl = 0; sl < TS; ++sl) {
                    float4* p = reinterpret_cast<float4*>(pass + (size_t)sl * 64 * 8);
                    p[0] = make_float4(acc3[sl][0], acc3[sl][1], acc3[sl][2], acc3[sl][3]);
                    p[1] = make_float4(acc3[sl][4], acc3[sl][5], acc3[sl][6], acc3[sl][7]);
                }
            }
            __syncthreads();
            if (active && !first) {
#pragma unroll
                for (int sl = 0; sl < TS; ++sl) {
                    const float4* p = reinterpret_cast<const float4*>(pass + (size_t)sl * 64 * 8);
                    const float4 a = p[0], b = p[1];
                    acc3[sl][0] = a.x;
                    acc3[sl][1] = a.y;
                    acc3[sl][2] = a.z;
                    acc3[sl][3] = a.w;
                    acc3[sl][4] = b.x;
                    acc3[sl][5] = b.y;
                    acc3[sl][6] = b.z;
                    acc3[sl][7] = b.w;
                }
                gemm3(ub00, 0);
                // Lane (g, token): features 4g..4g+3 (channel g) and 8+4g.. (channel 2+g).
                float* ep = d.Ep + ((size_t)(ub00 >> 1) * d.fine_rows + gm) * d.D;
#pragma unroll
                for (int sl = 0; sl < TS; ++sl) {
                    const int tok = tb * kTok + sl * 32 + l32, hp = tok / half_w, wp = tok - hp * half_w;
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        float* o = ep + ((size_t)(2 * q + g) * d.Himg + 2 * hp) * d.Wimg + 2 * wp;
                        *reinterpret_cast<float2*>(o) = make_float2(acc3[sl][4 * q], acc3[sl][4 * q + 1]);
                        *reinterpret_cast<float2*>(o + d.Wimg) = make_float2(acc3[sl][4 * q + 2], acc3[sl][4 * q + 3]);
                    }
                }
            }
            // The next item's gather touches xs and es only, and its barrier comes before its h1.
        }
    }
}

// Which fine items a launch of M list entries takes, if any: the finest that still fit the blocks
// in one round. A second round of a finer size costs more than one round of the next (1024
// tokens, H = 1024: 4 misses in 2 rounds of 32 x 256 26 us, in one of 32 x 512 20 us; 2 misses in
// 2 rounds of 32 x 128 21 us, in one of 32 x 256 15 us), and two rounds of 64 x 512 more than one
// of 128-token halves (12 misses: 50 against 41 us).
enum FineChoice { FINE_NONE, FINE_32x128, FINE_32x256, FINE_32x512, FINE_64x512 };
template <int H>
__device__ __forceinline__ int fine_choice(int M, int ntok, int fine_rows, int G) {
    const int sl = M * (ntok / 32);                  // 32-token slices
    if (sl / 2 * (H / 512) > G) return FINE_NONE;
    if (sl * (H / 512) > G) return FINE_64x512;
    if (sl * (H / 256) > G || M > fine_rows) return FINE_32x512;
    return sl * (H / 128) > G ? FINE_32x256 : FINE_32x128;
}

// TOK: tokens per work item, 128; or 64 for some launches of a single latent (launch_eps_mlp): its h1
// GELUs meet the W2 stream, where a fine item of 64 tokens takes them in turn.
template <int H, int TOK>
__global__ __launch_bounds__(kWaves * 64) void k_eps_mlp(Dev d) {
    constexpr int NT = kWaves * 64;
    constexpr int kTok = TOK;
    constexpr int TB4 = kTok / 32;       // 32-token slices per item
    constexpr int NS = H / kNH;          // halves of the output units (work items per tokens)
    constexpr int KCH = H / kKC;         // K-chunks of h1
    constexpr int HRow = kKC + 8;        // padded LDS row of h1 (bf16)
    constexpr int KS = H / 16;           // GEMM2 k-steps (fragment columns of W2^T)
    constexpr int KBC = kKC / 32;        // k-blocks (two k-steps) per chunk
    constexpr int ITER = KBC / 2;        // pipelined iterations per chunk
    static_assert(H % kNH == 0 && H % kKC == 0 && ITER == 4, "unsupported hidden width");
    static_assert(kKC == kWaves * 32, "each wave computes 32 h1 units of a chunk");
    // h1 chunks, double-buffered: chunk c + 1 is computed while GEMM2 consumes chunk c.
    __shared__ __attribute__((aligned(16))) __bf16 h1s[2][kTok * HRow];
    __shared__ __attribute__((aligned(16))) __bf16 xs[kTok * kXRow];
    // e_t of the item's timestep. Read from LDS in the GELU slices: a global load there
    // would share the in-order vector-memory counter with the W2 prefetch, and waiting for
    // it would wait for the prefetched fragments too.
    __shared__ __attribute__((aligned(16))) float es[H];
    // [kWaves][kTok][16] after GEMM2, in the h1 buffer of the last chunk (the other buffer keeps
    // the chunk a whole-output block reuses for the item's second half).
    float* red = reinterpret_cast<float*>(&h1s[1][0]);
    static_assert(kWaves * kTok * kFeat * 4 <= kTok * HRow * 2, "reduction buffer must fit");
    static_assert(KCH % 2 == 0, "the last chunk of either order is consumed from buffer 1");
    static_assert(TOK < kTokMax || (32 * (H + 8) <= 2 * kTok * HRow &&
                                    64 * ((H < 1024 ? H : 1024) + 8) <= 2 * kTok * HRow),
                  "h1 of a fine item must fit");

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index, in a scalar register
    // Misses per sample (0 once a sample is done), inclusive prefix over the samples.
    __shared__ int mpre[PA_MAX_BATCH + 1];
    static_assert(PA_MAX_BATCH <= 64, "one wave scans the samples");
    // Fused sweep (one sample): every block computes the outstanding window slide itself from
    // the Picard kernel's snapshot and partial sums (block 0 publishes it), and keeps the miss
    // list and the newest computed state in LDS; nothing this kernel writes is read back by it.
    __shared__ int fmiss[PA_MAX_WINDOW];
    __shared__ int fnewest;
    if (d.fused_slide) {
        // A launch queued after the one that finished the sample (that launch computed the last
        // slide and published done) has nothing to do: every block leaves at once.
        if (ended_before(d, *d.ctrl)) return;
        static_assert(sizeof(SlideScratch) + 16 + kSlideSubDoubles * sizeof(double) <= sizeof(h1s),
                      "slide scratch must fit");
        SlideScratch& sc = *reinterpret_cast<SlideScratch*>(&h1s[0][0]);
        double* sub = reinterpret_cast<double*>(&h1s[0][0] + (sizeof(SlideScratch) + 15) / 16 * 8);
        const SlidePre pre = d.pre[0];
        slide_partials<NT>(d, 0, sub);       // its loads do not wait for the snapshot
        __syncthreads();
        if (pre.pending) {
            slide_core<NT>(d, 0, pre, blockIdx.x == 0, sc, sub);
            const int m = sc.done ? 0 : sc.m;
            for (int j = tid; j < m; j += NT) fmiss[j] = sc.miss_idx[j];
            if (tid == 0) {
                mpre[0] = 0;
                mpre[1] = m;
                fnewest = sc.newest;
            }
        } else {                             // first sweep after reset: the reset's window
            const Ctrl* c = d.ctrl;
            const int m = c->m;
            for (int j = tid; j < m; j += NT) fmiss[j] = c->miss_idx[j];
            if (tid == 0) {
                mpre[0] = 0;
                mpre[1] = m;
                fnewest = c->newest;
            }
        }
    } else {
        // Parareal: every block computes the hit test of the launch's requests from the partial
        // sums of their deviations, wave by wave (block 0 publishes it); a block of the sampler
        // has at most one miss, at timestep fmiss[block].
        static_assert(PA_PR_MAX_BLOCKS <= PA_MAX_WINDOW, "one timestep per Parareal block");
        if (d.pr_dev) {
            for (int n = w; n < d.N; n += kWaves) {
                int t = 0;
                const bool act = pr_request(d.pr, n, &t) && !d.pr.pc->done;
                double dev = __builtin_nan("");
                if (act && d.valid[t]) {
                    double acc = 0.0;
                    for (int q = lane; q < d.pr.nchunk; q += 64) acc += d.pr_dev[(size_t)n * d.pr.nchunk + q];
                    dev = wave_sum(acc) / (double)d.D;
                }
                const bool hit = dev < d.delta;      // strict: delta == 0 never hits
                if (lane == 0) {
                    fmiss[n] = act && !hit ? t : -1;
                    if (blockIdx.x == 0) {
                        if (act) pr_publish(d, d.pr, n, t, hit, dev);
                        else d.ctrl[n].m = 0;
                    }
                }
            }
            __syncthreads();
        }
    }
    if (!d.fused_slide && w == 0) {
        int v = 0;
        if (lane < d.N) v = d.pr_dev ? fmiss[lane] >= 0 : (d.ctrl[lane].done ? 0 : d.ctrl[lane].m);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int u = __shfl_up(v, off, 64);
            if (lane >= off) v += u;
        }
        if (lane < d.N) mpre[lane + 1] = v;
        if (lane == 0) mpre[0] = 0;
    }
    __syncthreads();
    const int nblk = d.ntok / kTok;
    const int tblocks = mpre[d.N] * nblk;            // (miss, token block) pairs
    const int G = gridDim.x;
    // Whole outputs (if the handle takes fresh outputs in the cache directly) unless they
    // lengthen the launch: a block's whole item costs about 15/16 of NS half items (one
    // gather and one h1 chunk fewer per extra half, measured ~4-6%), so they are taken when
    // 15/16 x NS x the rounds of whole items do not exceed the rounds of half items spread
    // over all blocks: with one item per block when more than half of the blocks get one,
    // and always from about 7 rounds on. (The rule weighs full rounds: it does not know that the
    // items past the last one may be cut, below.)
    const int fine = TOK == kTokMax && d.eps_mode != nullptr ? fine_choice<H>(mpre[d.N], d.ntok, d.fine_rows, G)
                                                             : FINE_NONE;
    const bool whole = fine == FINE_NONE && d.whole_ok && NS <= 2 &&
                       15 * NS * ((tblocks + G - 1) / G) <= 16 * ((tblocks * NS + G - 1) / G);
    if (d.eps_mode != nullptr && blockIdx.x == 0 && tid <= d.N)
        d.eps_mode[tid] = tid > 0 ? mpre[tid - 1]
                                  : (fine == FINE_32x128 || fine == FINE_32x256
                                         ? EPS_FINE
                                         : (whole ? EPS_WHOLE : EPS_SPLIT));
    if constexpr (TOK == kTokMax) if (fine != FINE_NONE) {
        __bf16* hf = &h1s[0][0];
        // Unit groups fastest: with the blocks dealt to the XCDs in turn, an XCD's L2 fills with
        // the W2 columns of few groups.
        auto take = [&](auto ts_c, auto uf_c, auto kp_c) {
            constexpr int TS = decltype(ts_c)::value, NUG = H / decltype(uf_c)::value;
            const int nb = d.ntok / (32 * TS);
            fine_items<H, TS, decltype(uf_c)::value, decltype(kp_c)::value, false>(
                d, hf, xs, es, mpre, fmiss, fnewest, mpre[d.N] * nb * NUG,
                [=](int i) { return FineItem{i / NUG / nb, i / NUG % nb, i % NUG}; });
        };
        typedef std::integral_constant<int, 1> c1;
        typedef std::integral_constant<int, 2> c2;
        switch (fine) {
            case FINE_32x128: take(c1{}, std::integral_constant<int, 128>{}, c1{}); break;
            case FINE_32x256: take(c1{}, std::integral_constant<int, 256>{}, c1{}); break;
            case FINE_32x512: take(c1{}, std::integral_constant<int, 512>{}, c1{}); break;
            default: take(c2{}, std::integral_constant<int, 512>{}, std::integral_constant<int, (H > 1024 ? 2 : 1)>{}); break;
        }
        return;
    }
    const int g = lane >> 5, l32 = lane & 31;
    // W2^T as a buffer resource (out-of-range loads would return zero)
    const __amdgpu_buffer_rsrc_t w2r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(d.w2f), (short)0, H * H * 2, 0x00020000);
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                           0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // Whole outputs: each thread's sum of the halves so far. In LDS where there are two: four
    // registers less across GEMM2, without which some were spilled, and a kernel with scratch
    // memory takes longer to start as well (8 x 1024 tokens, H = 1024: 6755 -> 6707 us a sample).
    float4* runs = nullptr;
    if constexpr (NS == 2) {
        __shared__ float4 runs_lds[NT];
        runs = runs_lds;
    }
    float4 run = make_float4(0.f, 0.f, 0.f, 0.f);
    // One half (output units [512 ns, 512 ns + 512)) of the item (list entry gm, token block tb).
    // WHOLE: part of a whole-output block's item (ns > 0: the gather and the first h1 chunk of
    // the previous half are still in LDS).
    auto half = [&](int gm, int tb, int ns, bool whole_item) {
        int n = 0;
        while (mpre[n + 1] <= gm) ++n;               // sample of list entry gm (uniform)
        const int jm = gm - mpre[n];
        const Ctrl* ctrl = d.ctrl + n;
        const int t = d.fused_slide ? fmiss[jm] : (d.pr_dev ? fmiss[n] : ctrl->miss_idx[jm]);
        const int newest = d.fused_slide ? fnewest : (d.pr_dev ? t : ctrl->newest);
        const int hb0 = ns * (kNH / 32) + w * 2;   // this wave's first 32-unit block of W2^T

        const int odd = ns & 1;
        const bool reuse = whole_item && ns > 0;      // tokens, e_t and chunk KCH - 2 in LDS
        // ---- 0. gather + patchify + bf16; e_t into LDS
        if (reuse) {
            __syncthreads();                 // the previous half's reduction reads are done
        } else {
            const float* xt = d.X + ((size_t)n * (d.T + 1) + min(t, newest)) * d.D;   // beyond newest: its copy
            const float* et = d.temb + (size_t)t * H;
            // Every load of the thread is issued before the first LDS store, so the block waits
            // for one round trip to memory instead of one per element.
            constexpr int kPer = kTok * kFeat / NT;
            static_assert(kPer * NT == kTok * kFeat, "one element per thread and round");
            constexpr int kEs = (H / 4 + NT - 1) / NT;
            float xv[kPer];
            float4 ev[kEs];
#pragma unroll
            for (int k = 0; k < kPer; ++k) xv[k] = xt[tok_pos<kTok>(tid + k * NT, tb, d.Himg, d.Wimg).idx];
#pragma unroll
            for (int k = 0; k < kEs; ++k)
                if (tid + k * NT < H / 4) ev[k] = reinterpret_cast<const float4*>(et)[tid + k * NT];
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const TokPos p = tok_pos<kTok>(tid + k * NT, tb, d.Himg, d.Wimg);
                xs[p.tl * kXRow + p.f] = (__bf16)xv[k];
            }
#pragma unroll
            for (int k = 0; k < kEs; ++k)
                if (tid + k * NT < H / 4) reinterpret_cast<float4*>(es)[tid + k * NT] = ev[k];
            __syncthreads();
        }

        // ---- 1. h1 = GELU(x W1 + e_t): wave w computes units [32w, 32w + 32) of a chunk,
        // one 32-token slice per call, into LDS rows [token][unit].
        bf16x8 w1a;
        const float* ek = es;                // e_t of the chunk's units (LDS)
        auto h1_setup = [&](int kc) {
            const int n0 = kc * kKC + w * 32;
            w1a = *reinterpret_cast<const bf16x8*>(d.w1t + (size_t)(n0 + l32) * kFeat + g * 8);
            ek = es + n0 + g * 4;
        };
        // The W1 fragment of a chunk is loaded while the chunk before the last computes its h1, so
        // that the first GEMM1 of a chunk does not wait for a load younger than the W2 fragments
        // in flight (and so for those too). At H = 2048 it is slower (21 misses of 768 tokens:
        // 150 -> 153 us).
        constexpr bool kW1Ahead = H <= 1024;
        f32x16 h1acc;
        // The accumulator starts at e_t (row = unit), so the MFMA returns x W1 + e_t; the
        // GELU slices store 2 h1 (W2 is stored halved, see gelu2_erf).
        auto h1_mfma = [&](int tb4) {
            const bf16x8 b = *reinterpret_cast<const bf16x8*>(xs + (tb4 * 32 + l32) * kXRow + g * 8);
            f32x16 c0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 ev = *reinterpret_cast<const float4*>(ek + q * 8);
                c0[q * 4 + 0] = ev.x;
                c0[q * 4 + 1] = ev.y;
                c0[q * 4 + 2] = ev.z;
                c0[q * 4 + 3] = ev.w;
            }
            h1acc = mfma32(w1a, b, c0);
        };
        auto h1_gelu = [&](__bf16* buf, int kc, int tb4, int q0) {   // units q0*8.. of the slice
            const int tok = tb4 * 32 + l32;
#pragma unroll
            for (int q = q0; q < q0 + 2; ++q) {
                bf16x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = (__bf16)gelu2_erf(h1acc[q * 4 + i]);
                *reinterpret_cast<bf16x4*>(buf + tok * HRow + w * 32 + q * 8 + g * 4) = v;
            }
        };
        auto h1_slice = [&](__bf16* buf, int kc, int tb4) {
            h1_mfma(tb4);
            h1_gelu(buf, kc, tb4, 0);
            h1_gelu(buf, kc, tb4, 2);
        };
        if (!reuse) {
            const int k0 = korder<KCH>(odd, 0);
            h1_setup(k0);
#pragma unroll
            for (int tb4 = 0; tb4 < TB4; ++tb4) h1_slice(h1s[0], k0, tb4);
            __syncthreads();
        }

        f32x16 acc2[2][TB4];
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
            for (int tb4 = 0; tb4 < TB4; ++tb4) acc2[hb][tb4] = zero16;

        // W2^T fragments of k-block kb of chunk kc, for this wave's two 32-unit blocks.
        // Buffer loads: the fragment's byte offset is wave-uniform (a scalar register), the
        // lane's 16-byte slot is the only per-lane address part.
        auto load_a = [&](bf16x8 (&A)[2][2], int kc, int kb) {
            const int sb = (hb0 * KS + kc * (kKC / 16) + 2 * kb) * 64 * 16;
#pragma unroll
            for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    A[hb][j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                        w2r, lane * 16, sb + (hb * KS + j) * 64 * 16, 0));
        };
        bf16x8 A0[2][2], A1[2][2];
        // GEMM2 step st = (k-block kb, 32-token slice): four MFMAs. The B operands (h1^T from LDS)
        // of the next step, also across k-blocks, are read before them; the scheduling barriers
        // keep the reads there (the compiler otherwise moves each right before its use, and every
        // four MFMAs wait for a round trip to LDS). A wave's cycles per chunk with GELU work fell
        // by 7%; the launch gains less, since with all CUs busy power sets the clock: 29
        // misses of 1024 tokens, H = 1024, 85 -> 83 us. Two steps ahead spills (15 registers).
        // H = 1024: the MFMAs of a step start on 8 bytes, their size (one s_nop at most). Where they
        // fall otherwise follows from the code before the loop, and half of all places cost 1%:
        // with the loop's start moved by 4 bytes at a time, 8 x 1024 tokens take 6738 to 6759 us a
        // sample at the odd words and 6794 to 6811 at the even ones; aligned 6976 where those take
        // 6987 and 7051. At H = 2048 the natural place is the faster one (Parareal 6184 against
        // 6300 us at the other, 6346 against 6369 aligned), at H = 512 either is within 0.4%.
        constexpr int STEPS = KBC * TB4;
        bf16x8 B[2][2];
        auto load_b = [&](const __bf16* h1b, int st) {
            const int kb = st / TB4, tb4 = st % TB4;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                B[st % 2][j] = *reinterpret_cast<const bf16x8*>(h1b + tb4 * 32 * HRow + kb * 32 + j * 16);
        };
        auto mma = [&](const bf16x8 (&A)[2][2], const __bf16* h1b, int kb) {
#pragma unroll
            for (int tb4 = 0; tb4 < TB4; ++tb4) {
                const int st = kb * TB4 + tb4;
                if (st + 1 < STEPS) load_b(h1b, st + 1);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (H == 1024) asm volatile(".p2align 3");
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int hb = 0; hb < 2; ++hb)
                        acc2[hb][tb4] = mfma32(A[hb][j], B[st % 2][j], acc2[hb][tb4]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // One chunk of GEMM2 at position i of the half's chunk order (two register stages of
        // W2^T fragments, the stream running on across chunk boundaries); position i is in
        // buffer i & 1. MORE: a chunk follows; its h1 slices are computed between the MFMA
        // groups. A wave raises its issue priority while it feeds MFMA groups, so that the two
        // waves of a SIMD drift out of step (one in its MFMA group while the other is in its
        // GELU slice).
        auto chunk = [&](int i, auto more_c) {
            constexpr bool more = decltype(more_c)::value;
            const int kc = korder<KCH>(odd, i);
            const int kn = more ? korder<KCH>(odd, i + 1) : 0;
            if constexpr (more) {
                if constexpr (kW1Ahead) ek = es + kn * kKC + w * 32 + g * 4;
                else h1_setup(kn);
            }
            __bf16* nbuf = h1s[(i + 1) & 1];
            const __bf16* h1b = h1s[i & 1] + l32 * HRow + g * 8;
            load_b(h1b, 0);
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int kb = 2 * it;
                load_a(A1, kc, kb + 1);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_setprio(1);
                mma(A0, h1b, kb);
                if constexpr (more) {
                    if (it < TB4) h1_slice(nbuf, kn, it);   // one 32-token slice per iteration
                    if (kW1Ahead && it == TB4 - 1) {
                        const int k2 = i + 2 < KCH ? korder<KCH>(odd, i + 2) : 0;
                        w1a = *reinterpret_cast<const bf16x8*>(d.w1t + (size_t)(k2 * kKC + w * 32 + l32) * kFeat + g * 8);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_setprio(0);
                // Next fragments: this chunk's, or the first of the next chunk (after the
                // last chunk an unused reload of chunk 0, kept unconditional so the wait for
                // A1 below counts exactly these four loads as younger).
                if (kb + 2 < KBC) load_a(A0, kc, kb + 2);
                else load_a(A0, kn, 0);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_setprio(1);
                mma(A1, h1b, kb + 1);
                __builtin_amdgcn_s_setprio(0);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();                 // chunk kc + 1 complete; chunk kc's buffer free
        };
        if constexpr (kW1Ahead) h1_setup(korder<KCH>(odd, 1));
        load_a(A0, korder<KCH>(odd, 0), 0);
        for (int i = 0; i + 1 < KCH; ++i) chunk(i, std::true_type{});
        chunk(KCH - 1, std::false_type{});

        // ---- 3. eps^T partial = W3p GELU(h2^T) straight from the accumulators (2 GELU with W3
        // stored halved)
        f32x16 acc3[TB4];
#pragma unroll
        for (int tb4 = 0; tb4 < TB4; ++tb4) acc3[tb4] = zero16;
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const bf16x8 a3 = *reinterpret_cast<const bf16x8*>(
                    d.w3p + (((size_t)(hb0 + hb) * 2 + jj) * 64 + lane) * 8);
#pragma unroll
                for (int tb4 = 0; tb4 < TB4; ++tb4) {
                    bf16x8 b3;
#pragma unroll
                    for (int i = 0; i < 8; ++i) b3[i] = (__bf16)gelu2_erf(acc2[hb][tb4][jj * 8 + i]);
                    acc3[tb4] = mfma32(a3, b3, acc3[tb4]);
                }
            }
        }
        // valid rows of acc3: regs 0..7 -> feature (r/4)*8 + g*4 + r%4, token tb4*32 + l32
#pragma unroll
        for (int tb4 = 0; tb4 < TB4; ++tb4) {
            float* dst = red + ((size_t)w * kTok + tb4 * 32 + l32) * kFeat;
            *reinterpret_cast<float4*>(dst + g * 4) =
                make_float4(acc3[tb4][0], acc3[tb4][1], acc3[tb4][2], acc3[tb4][3]);
            *reinterpret_cast<float4*>(dst + 8 + g * 4) =
                make_float4(acc3[tb4][4], acc3[tb4][5], acc3[tb4][6], acc3[tb4][7]);
        }
        __syncthreads();

        // ---- 4. fixed-order sum over waves, unpatchify, store this half's partial output.
        // Thread = (channel c, token tl): its four features c*4 + dh*2 + dw are contiguous in
        // the reduction buffer and form two float2 pairs (dw = 0, 1) in rows 2hp and 2hp + 1.
        // Split outputs: this half's partial output; whole outputs: the running sum of the
        // halves (half 0 + half 1, the order the Picard kernel adds split partials in), stored
        // by the last half into the cache output of the miss.
        float* out = whole_item ? d.Eh + ((size_t)n * d.T + t) * d.D
                                : d.Ep + (((size_t)ns * d.N + n) * d.P + jm) * d.D;
        static_assert(kTok * (kFeat / 4) <= NT, "one token and channel per thread");
        if (tid < kTok * (kFeat / 4)) {
            const int tl = tid & (kTok - 1), c = tid / kTok;
            float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int ww = 0; ww < kWaves; ++ww) {
                const float4 v = *reinterpret_cast<const float4*>(red + ((size_t)ww * kTok + tl) * kFeat + c * 4);
                sum.x += v.x;
                sum.y += v.y;
                sum.z += v.z;
                sum.w += v.w;
            }
            if (whole_item) {
                if constexpr (NS == 2) {
                    if (ns == 0) {
                        runs[tid] = sum;
                    } else {
                        const float4 r = runs[tid];
                        sum = make_float4(r.x + sum.x, r.y + sum.y, r.z + sum.z, r.w + sum.w);
                    }
                } else {
                    run = ns == 0 ? sum : make_float4(run.x + sum.x, run.y + sum.y, run.z + sum.z, run.w + sum.w);
                    sum = run;
                }
            }
            if (!whole_item || ns == NS - 1) {
                const int half_w = d.Wimg >> 1;
                const int tok = tb * kTok + tl;
                const int hp = tok / half_w, wp = tok - hp * half_w;
                float* o = out + ((size_t)c * d.Himg + 2 * hp) * d.Wimg + 2 * wp;
                *reinterpret_cast<float2*>(o) = make_float2(sum.x, sum.y);
                *reinterpret_cast<float2*>(o + d.Wimg) = make_float2(sum.z, sum.w);
            }
        }
        // No barrier: the next item's gather writes xs and es only, and its barrier comes
        // before anything overwrites the reduction buffer (h1 buffer 1); a whole-output
        // block's next half starts with one.
    };

    // One block item: both halves of a token block (whole) or one half (split).
    const int per = whole ? NS : 1;
    const int units = tblocks * (NS / per);
    // The items beyond the last full round, if they are few, are cut into items of 32 or 64 tokens
    // (fine_items), so that the launch ends with one short item per block instead of a long one
    // on few. Up to a quarter of the blocks' number: 32 tokens (3/16 for whole outputs of two
    // halves, whose 32 tokens stream all of W2); up to half: 64; beyond that a full-length item
    // is no longer (1024 tokens, H = 1024: 48 misses, half a round over, 138 us either way).
    // Measured without and with: 33 misses 125 -> 110 us, 40 (64 items over) 129 -> 121,
    // 232 (64 over) 595 -> 560; 256 tokens, H = 512: 160 misses 56 -> 47; 768 tokens, H = 2048:
    // 12 misses 137 -> 118, 16 146 -> 136. A handle held to split outputs keeps whole rounds.
    int full = units, cut = 0;
    if (TOK == kTokMax && d.eps_mode != nullptr && units > G) {
        const int rest = units % G;
        if (rest > 0) cut = (NS == 2 && whole ? 16 * rest <= 3 * G : 4 * rest <= G) ? 4 : (2 * rest <= G ? 2 : 0);
        if (cut) full = units - rest;
    }
    for (int item = blockIdx.x; item < full; item += G) {
        const int tbk = whole ? item : item / NS;
        for (int q = 0; q < per; ++q) half(tbk / nblk, tbk % nblk, whole ? q : item % NS, whole);
    }
    if constexpr (TOK == kTokMax) if (cut) {
        __syncthreads();                     // the reduction buffer is read
        auto take = [&](auto ts_c, auto whole_c) {
            constexpr int TS = decltype(ts_c)::value, C = 4 / TS;   // items per 128 tokens
            constexpr bool WH = decltype(whole_c)::value;
            fine_items<H, TS, kNH, (!WH && TS == 2 && H > 1024 ? 2 : 1), WH>(
                d, &h1s[0][0], xs, es, mpre, fmiss, fnewest, (units - full) * C, [=](int i) {
                    const int u = full + i / C, tbk = WH ? u : u / NS;
                    return FineItem{tbk / nblk, tbk % nblk * C + i % C, WH ? 0 : u % NS};
                });
        };
        typedef std::integral_constant<int, 1> c1;
        typedef std::integral_constant<int, 2> c2;
        if constexpr (NS <= 2) {
            if (whole) {
                if (cut == 4) take(c1{}, std::true_type{});
                else take(c2{}, std::true_type{});
                return;
            }
        }
        if (cut == 4) take(c1{}, std::false_type{});
        else take(c2{}, std::false_type{});
    }
}

namespace {

// Half of a bf16 value on its bit pattern, rounded to nearest even. An exponent field of 2 or
// more drops by one (exact). Below that (subnormals and the smallest binade) the magnitude
// bits read as an integer are the value in units of 2^-133, which is halved with ties to even;
// the result is again such a magnitude. NaN is returned quiet, infinity unchanged.
__device__ __forceinline__ uint16_t bf16_half_bits(uint16_t b) {
    const uint16_t sgn = b & 0x8000u, mag = b & 0x7fffu;
    if (mag > 0x7f80u) return b | 0x0040u;
    if (mag == 0x7f80u) return b;
    if (mag >= 0x0100u) return sgn | (uint16_t)(mag - 0x0080u);
    const uint16_t q = mag >> 1;
    return sgn | (uint16_t)(q + ((mag & 1u) & (q & 1u)));
}

// Device layouts of the weights (grid-stride over the three outputs):
//   w1t[n][f] = W1[f][n];
//   w2f: W2^T as MFMA A fragments, fragment (b, ks) = lanes l = 0..63 x 8 values
//        W2[16 ks + 8 (l/32) + i][32 b + l%32] / 2;
//   w3p: fragment (hb, jj) = lanes l x 8 values W3[32 hb + (2 jj + i/4) 8 + 4 (l/32) + i%4][l%32] / 2
//        for l%32 < 16, else 0 (the reduction index permuted to the GEMM2 accumulator layout).
// W2 and W3 are stored halved because the kernel feeds them twice the GELU outputs.
__global__ void k_pack_weights(const uint16_t* __restrict__ w1, const uint16_t* __restrict__ w2,
                               const uint16_t* __restrict__ w3, int H, uint16_t* __restrict__ w1t,
                               uint16_t* __restrict__ w2f, uint16_t* __restrict__ w3p) {
    const size_t n1 = (size_t)H * 16, n2 = (size_t)H * H, n3 = (size_t)H * 32;
    const int KS = H / 16;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n1 + n2 + n3;
         e += (size_t)gridDim.x * blockDim.x) {
        if (e < n1) {
            const int n = (int)(e / 16), f = (int)(e % 16);
            w1t[e] = w1[(size_t)f * H + n];
        } else if (e < n1 + n2) {
            const size_t q = e - n1;
            const int i = (int)(q & 7), lane = (int)((q >> 3) & 63);
            const size_t frag = q >> 9;
            const int ks = (int)(frag % KS), b = (int)(frag / KS);
            const int n = b * 32 + (lane & 31), k = ks * 16 + (lane >> 5) * 8 + i;
            w2f[q] = bf16_half_bits(w2[(size_t)k * H + n]);
        } else {
            const size_t q = e - n1 - n2;
            const int i = (int)(q & 7), lane = (int)((q >> 3) & 63);
            const size_t rest = q >> 9;
            const int jj = (int)(rest & 1), hb = (int)(rest >> 1);
            const int g = lane >> 5, f = lane & 31;
            const int n = hb * 32 + (jj * 2 + i / 4) * 8 + g * 4 + (i % 4);
            w3p[q] = f < 16 ? bf16_half_bits(w3[(size_t)n * 16 + f]) : (uint16_t)0;
        }
    }
}

}  // namespace

hipError_t launch_pack_weights(const uint16_t* w1, const uint16_t* w2, const uint16_t* w3, int H,
                               __bf16* w1t, __bf16* w2f, __bf16* w3p, hipStream_t st) {
    hipLaunchKernelGGL(k_pack_weights, dim3(1024), dim3(256), 0, st, w1, w2, w3, H,
                       reinterpret_cast<uint16_t*>(w1t), reinterpret_cast<uint16_t*>(w2f),
                       reinterpret_cast<uint16_t*>(w3p));
    return hipGetLastError();
}

int mlp_supported(int hidden) { return hidden == 512 || hidden == 1024 || hidden == 2048; }

int mlp_tokens_per_item() { return kTokMax; }

int mlp_splits(int hidden) { return hidden / kNH; }

int mlp_grid_size(int device_cus) { return device_cus > 0 ? device_cus : 256; }

// The most list entries whose items of 32 tokens x 256 units fit the blocks in one round, as
// fine_choice has it (0: one entry does not).
int mlp_fine_rows(int hidden, int ntok, int grid) { return grid / ((ntok / 32) * (hidden / 256)); }

hipError_t launch_eps_mlp(const Dev& d, hipStream_t st, hipEvent_t start, hipEvent_t stop, int single) {
    const dim3 grid(d.mlp_grid), block(kWaves * 64);
    // A single latent in 64-token items where those fit the blocks in one round and the fine items of
    // 32 tokens x 512 units do not. Without -> with them, Parareal samples of 15 such launches and one
    // of 8 latents: H = 1024, 4608 tokens 600 -> 566 us, 6400 664 -> 632, 8192 719 -> 692; one launch
    // at H = 2048, 2304 tokens 43 -> 39 us. Beyond one round the 128-token kernel with its cut last
    // round is faster (H = 1024, 9216 tokens 870 against 1001 us; H = 2048, 5120 1319 against 1513,
    // 6400 1505 against 1630), and at H = 512 it is nowhere slower (9216 tokens 448 us either way,
    // 12544 485 against 491).
    const int it32 = d.ntok / 32 * (d.hidden / 512);
    const bool tok64 = single && d.hidden >= 1024 && it32 > d.mlp_grid && it32 <= 2 * d.mlp_grid;
    switch (d.hidden + (tok64 ? 1 : 0)) {
        case 512: hipExtLaunchKernelGGL((k_eps_mlp<512, 128>), grid, block, 0, st, start, stop, 0, d); break;
        case 1024: hipExtLaunchKernelGGL((k_eps_mlp<1024, 128>), grid, block, 0, st, start, stop, 0, d); break;
        case 1024 + 1: hipExtLaunchKernelGGL((k_eps_mlp<1024, 64>), grid, block, 0, st, start, stop, 0, d); break;
        case 2048: hipExtLaunchKernelGGL((k_eps_mlp<2048, 128>), grid, block, 0, st, start, stop, 0, d); break;
        case 2048 + 1: hipExtLaunchKernelGGL((k_eps_mlp<2048, 64>), grid, block, 0, st, start, stop, 0, d); break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace pa
