// prefill_gemm.hip -- KV-only prefill of many tokens (Sec. 3.4 of the WhiFlash
// paper: the backlog of a drafter switch in one batch) as an LDS-tiled matrix
// product with the RoPE and cache-append epilogue of the small-batch kernel:
//
//   K[g][p+t] = RoPE(W_k[g] x_t, p+t),   V[g][p+t] = W_v[g] x_t
//
// A workgroup owns PW = WF*FB/2 RoPE pairs of 16-feature blocks (block f of a
// head and block f + head_dim/2) times WT*NB*16 tokens and the whole input
// dimension (wf_gemm.h); wave (wf, wt) owns FB/2 pairs, so both halves of
// every rotation sit in one lane.
//
// What bounds it (counters and timing variants, 1013 tokens, 8B shapes): the
// step's copies alone take 21-23 us of the call's 24, compute alone 17; the
// operands of the next half step are read from LDS while the current half's
// MFMAs run (30 -> 26 us), two k groups share a step where one wave per SIMD
// would leave its latencies bare (28 -> 26), and neither the ring's depth
// nor row-major against tiled sources matters.
#include <cmath>

#include "wf_api_internal.h"
#include "wf_device.h"
#include "wf_gemm.h"

namespace wf {

namespace {

constexpr int kMaxHalfDim = 64;

struct GemmParams {
    const char *x, *w_k, *w_v;
    uint16_t *k_cache, *v_cache;
    int n_tok, start_pos, cap, d_in, head_dim;
    int kind_pairs;                      // RoPE pairs of K (and as many of V)
    int token_blocks;                    // workgroups along the tokens
    int pair_blocks;                     // workgroups along the pairs
    int units, units_per_xcd;            // layers * pair_blocks * token_blocks
    int w_tiled, x_tiled;
    long long x_ls, w_ls, c_ls;          // element strides between layers
    double turns[kMaxHalfDim];           // RoPE frequencies in turns per position
};

// cos and sin of 2*pi*t.  The turn is reduced in fp64 (exact) and rounded to
// fp32, then reduced to the nearest quarter (exact), and the rest, at most pi/4
// in size, goes through the Taylor series (truncation below 3e-9).  Against 64
// bits over 2 million positions up to 70000: error at most 1.5e-7, 4.4e-8 in
// the mean square; sincosf of the reduced angle, as the small-batch kernel
// has it, 1.6e-7 and 4.7e-8.
__device__ __forceinline__ void sincos_turns(double t, float &s, float &c) {
    const float f = (float)(t - rint(t));
    const float q = rintf(4.f * f);
    const float a = fmaf(q, -0.25f, f) * 6.283185307179586f;
    const float z = a * a;
    const float sp = fmaf(z, fmaf(z, fmaf(z, fmaf(z, 1.f / 362880.f, -1.f / 5040.f), 1.f / 120.f),
                                  -1.f / 6.f), 0.f);
    const float sa = fmaf(a, sp, a);
    const float ca = fmaf(z, fmaf(z, fmaf(z, fmaf(z, fmaf(z, -1.f / 3628800.f, 1.f / 40320.f),
                                                  -1.f / 720.f), 1.f / 24.f), -0.5f), 1.f);
    const int k = (int)q & 3;            // quarters, mod 4
    const float ss = (k & 1) ? ca : sa, cc = (k & 1) ? sa : ca;
    s = (k & 2) ? -ss : ss;
    c = (k == 1 || k == 2) ? -cc : cc;
}

template <int FB, int NB, int WF, int WT, int WK, int NBUF, bool NT>
__global__ __launch_bounds__(64 * WF * WT * WK) void prefill_gemm(GemmParams a) {
    using G = TileGemm<FB, NB, WF, WT, WK, NBUF, NT>;
    constexpr int PW = G::FBLK / 2;
    __shared__ __attribute__((aligned(1024))) char ring[NBUF * G::STAGE];

    const int unit = (int)(blockIdx.x & 7) * a.units_per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= a.units_per_xcd || unit >= a.units)
        return;
    const int tb = unit % a.token_blocks;
    const int pb = (unit / a.token_blocks) % a.pair_blocks;
    const int layer = unit / (a.token_blocks * a.pair_blocks);
    const int t0 = tb * G::TBLK * 16;
    const int n_pairs = 2 * a.kind_pairs;

    const int lane = threadIdx.x % kWave;
    const int m16 = lane & 15;
    const int c4 = lane >> 4;
    const int wave = wave_id();
    const int wf = wave % WF, wt = (wave / WF) % WT, wk = wave / (WF * WT);

    // pair p of the layer (K's pairs, then V's) -> matrix row of its low block
    const int half_blk = a.head_dim / 32;                // pairs per head
    auto pair_row = [&](int p) {
        const int pk = p >= a.kind_pairs ? p - a.kind_pairs : p;
        return (pk / half_blk) * a.head_dim + (pk % half_blk) * 16;
    };
    const size_t block_bytes = (size_t)a.d_in * 32;      // 16 rows, row-major or tiled
    f32x4 acc[FB][NB];
    G::run(
        ring,
        [&](int b) {
            // (wave row w_f's blocks: the low halves of its pairs, then the high)
            const int w_f = b / FB, fb = b % FB;
            const int p = min(pb * PW + w_f * (FB / 2) + fb % (FB / 2), n_pairs - 1);
            const int row = pair_row(p) + (fb < FB / 2 ? 0 : a.head_dim / 2);
            return GemmBlock{(p >= a.kind_pairs ? a.w_v : a.w_k) + layer * a.w_ls * 2 +
                                 (row / 16) * block_bytes, 16};
        },
        [&](int b) {
            const int blk = min(t0 / 16 + b, (a.n_tok + 15) / 16 - 1);
            return GemmBlock{a.x + layer * a.x_ls * 2 + blk * block_bytes,
                             min(16, a.n_tok - 16 * blk)};
        },
        a.d_in, a.w_tiled, a.x_tiled, acc);

    // ---- RoPE (K) and the cache rows: lane (m16, c4) holds features
    // 4*c4 + i of token m16 of every (feature block, token block)
#pragma unroll
    for (int j = 0; j < FB / 2; ++j) {
        const int p = pb * PW + wf * (FB / 2) + j;
        if (p >= n_pairs)
            continue;
        const bool is_k = p < a.kind_pairs;
        const int pk = is_k ? p : p - a.kind_pairs;
        const int g = pk / half_blk;
        const int i0 = (pk % half_blk) * 16 + 4 * c4;    // first feature of the low half
        uint16_t *cache = (is_k ? a.k_cache : a.v_cache) + layer * a.c_ls +
                          (size_t)g * a.cap * a.head_dim;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int t = t0 + (wt * NB + nb) * 16 + m16;
            if (t >= a.n_tok || !G::owns(wk, j, nb))
                continue;
            const int pos = a.start_pos + t;
            f32x4 lo = acc[j][nb], hi = acc[j + FB / 2][nb];
            if (is_k) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float s, c;
                    sincos_turns((double)pos * a.turns[i0 + i], s, c);
                    const float l = lo[i], h = hi[i];
                    lo[i] = l * c - h * s;
                    hi[i] = h * c + l * s;
                }
            }
            uint16_t *row = cache + (size_t)pos * a.head_dim + i0;
            *reinterpret_cast<u32x2 *>(row) =
                u32x2{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3])};
            *reinterpret_cast<u32x2 *>(row + a.head_dim / 2) =
                u32x2{pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3])};
        }
    }
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Tile of a call: fb x nb blocks per wave, wf x wt x wk waves, nbuf stages.
struct GemmTile {
    int fb, nb, wf, wt, wk, nbuf;
    int features() const { return 16 * fb * wf; }
    int tokens() const { return 16 * nb * wt; }
};

constexpr int kComputeUnits = 256;

// Whether prefill.hip's kernel, which splits the input dimension over
// workgroups, is faster than one workgroup walking all of it.  That walk is a
// serial chain: about 3.6 us and 3.0 (tiled W) or 2.8 us per 1024 dims as long
// as the tiles fit the chip in one round.  The split kernel's chain is ks times
// shorter, but costs an exchange per halving and more per dim; both lines, per
// plan, are fits to calls of 65 to 320 tokens over 1024 to 8192 dims and 1 to
// 16 KV heads.  Split -> whole, us, tiled W unless stated: 8 heads of 128, 81
// tokens, 4096 dims 13.7 -> 15.6, 5120: 15.4 -> 19.9, 2560: 11.9 -> 10.8; 128
// tokens, 4096: 16.0 -> 15.9, row-major 20.4 -> 15.0; 2 heads, 4096 dims, 128
// tokens 11.8 -> 15.9, 256: 15.7 -> 14.9; 2 layers of 1 head, 80 tokens 8.7 ->
// 15.9.  Without a split the whole walk is always the faster.
bool split_is_faster(int n_tok, int d_in, int n_kv_heads, int head_dim, int n_layers,
                     bool w_tiled) {
    const PrefillPlan p = plan_prefill(n_tok, d_in, n_kv_heads, head_dim, n_layers);
    if (p.ksplit == 1)
        return false;
    // us: constant, per halving, per 1024 dims of a slice (tiled, row-major W)
    struct Line {
        double base, level, tiled, row_major;
    };
    const Line l = p.ppu == 2 ? (p.nbt <= 3 ? Line{5.8, 1.4, 4.5, 6.3} : Line{8.7, 1.3, 5.0, 7.2})
                              : (p.nbt <= 3 ? Line{5.0, 0.6, 3.5, 4.6} : Line{6.0, 0.5, 4.8, 5.9});
    const double kdims = d_in / 1024.0;
    const double split = l.base + l.level * std::log2(p.ksplit) +
                         (w_tiled ? l.tiled : l.row_major) * kdims / p.ksplit;
    return split < 3.6 + (w_tiled ? 3.0 : 2.8) * kdims;
}

// The tile for a call, or false where the split-K kernel of prefill.hip is
// the better one (us per call, head_dim 128, 8 KV heads, 4096 dims unless
// stated; that kernel's time -> this one's).
bool pick_tile(int n_tok, int d_in, int n_kv_heads, int head_dim, int n_layers, bool w_tiled,
               GemmTile &t) {
    const int feats = 2 * n_kv_heads * head_dim;
    const int blocks16 = cdiv(n_tok, 16);
    const long long units = (long long)n_layers * cdiv(feats, 32);
    // All tokens in one block, many layers: the call streams W once, with
    // the non-temporal hint, so it is bound by the HBM reads in flight.  The
    // features per workgroup follow the tokens (x is re-read by each feature
    // block), as long as a few workgroups per CU remain; fewer stages where
    // many workgroups share a CU.  36 layers: 16 tokens 124 -> 92 (64
    // features 98, 128: 103), 32: 150 -> 100 (32: 110, 128: 106), 48: 177 ->
    // 113, 80: 258 -> 125, 128: 355 -> 155; 12 layers: 10 tokens 40 -> 34, 32:
    // 54 -> 41; 8 layers: 16 tokens 30 -> 24,
    // 80: 61 -> 31.  Fewer layers leave it latency-bound (4 layers: 16 tokens
    // 17 -> 20, 32: 16 -> 21): there the input dimension has to be split over
    // workgroups.
    if (blocks16 <= 8) {
        const int nb = blocks16 == 7 ? 8 : blocks16;
        // one token block over a short tiled W: the split kernel has all of a
        // wave's loads in flight in one or two round trips (8 tokens, 64
        // layers of 512 features: 1024 dims 14.5 -> 17.0; 512 units of 2048
        // dims 14.2 -> 15.5, 640: 18.6 -> 17.6)
        const int min1 = !w_tiled || d_in > 2048 ? 512 : d_in > 1024 ? 640 : INT32_MAX;
        if (blocks16 == 1 && units >= min1) {
            // (a CU's LDS holds six workgroups of four stages; 1024 units, 1
            // token: two stages 54.7 us, four 45; 2048: 87 and 91)
            t = {2, 1, 1, 1, 2, units > 6 * kComputeUnits ? 2 : 4};
            return true;
        }
        if (blocks16 >= 4 && units >= 8 * kComputeUnits) {
            t = {2, nb, 4, 1, 1, 2};
            return true;
        }
        if (blocks16 >= 2 && units >= (blocks16 <= 3 ? 384 : 512)) {
            t = {2, nb, 2, 1, 2, units >= 4 * kComputeUnits ? 2 : 4};
            return true;
        }
    }
    // Otherwise the smallest tile that still runs in one round of one
    // workgroup per CU: each step costs its LDS traffic and a barrier, so a
    // larger tile only pays once the smaller one needs a second round (one
    // layer: 128 tokens 15.3 -> 13.5, 256: 19.9 -> 13.5, 512: 25.7 -> 16.2,
    // 1013: 43.8 -> 25.1 (row-major W 62 -> 26), 2048: 78.7 -> 40.2, 4096:
    // 154 -> 69.7, where the matrix cores run at 990 TFLOP/s; the next
    // smaller tile 20.6, 30.6, 47.8 and 86.2 from 512 tokens on).  Up to 80
    // tokens of one layer the split over the input dimension is as fast or
    // faster (13.3 against 13.3 at 80, 6.5 at 16).
    if (n_tok <= (n_layers == 1 ? 80 : 64) ||
        split_is_faster(n_tok, d_in, n_kv_heads, head_dim, n_layers, w_tiled))
        return false;
    for (const GemmTile c : {GemmTile{2, 1, 2, 2, 1, 4}, GemmTile{2, 2, 2, 2, 2, 4},
                             GemmTile{4, 2, 2, 2, 2, 3}, GemmTile{2, 4, 4, 2, 1, 3},
                             GemmTile{4, 4, 4, 2, 1, 3}}) {
        t = c;
        if ((long long)n_layers * cdiv(feats, c.features()) * cdiv(n_tok, c.tokens()) <=
            kComputeUnits)
            break;
    }
    return true;
}

}  // namespace

bool prefill_gemm_takes(int n_tok, int d_in, int n_kv_heads, int head_dim, int n_layers,
                        bool w_tiled) {
    GemmTile t;
    // (byte offsets along the input dimension are 32-bit, tiled: 32 bytes a dim)
    return 32LL * d_in < (1LL << 31) &&
           pick_tile(n_tok, d_in, n_kv_heads, head_dim, n_layers, w_tiled, t);
}

wf_status_t launch_prefill_gemm(bool w_tiled, bool x_tiled, const void *x, const void *w_k,
                                const void *w_v, void *k_cache, void *v_cache, int n_tok,
                                int start_pos, int cap, int d_in, int n_kv_heads, int head_dim,
                                double rope_base, hipStream_t stream, int n_layers,
                                long long x_ls, long long w_ls, long long c_ls) {
    GemmTile t;
    if (!pick_tile(n_tok, d_in, n_kv_heads, head_dim, n_layers, w_tiled, t))
        return WF_ERR_UNSUPPORTED;
    GemmParams a{};
    a.x = static_cast<const char *>(x);
    a.w_k = static_cast<const char *>(w_k);
    a.w_v = static_cast<const char *>(w_v);
    a.k_cache = static_cast<uint16_t *>(k_cache);
    a.v_cache = static_cast<uint16_t *>(v_cache);
    a.n_tok = n_tok;
    a.start_pos = start_pos;
    a.cap = cap;
    a.d_in = d_in;
    a.head_dim = head_dim;
    a.kind_pairs = n_kv_heads * (head_dim / 32);
    a.w_tiled = w_tiled;
    a.x_tiled = x_tiled;
    a.x_ls = x_ls;
    a.w_ls = w_ls;
    a.c_ls = c_ls;
    for (int i = 0; i < head_dim / 2; ++i)
        a.turns[i] = std::pow(rope_base, -2.0 * (double)i / (double)head_dim) / 6.283185307179586;
    a.pair_blocks = cdiv(2 * a.kind_pairs, t.features() / 32);
    a.token_blocks = cdiv(n_tok, t.tokens());
    const long long units = (long long)a.pair_blocks * a.token_blocks * n_layers;
    if (units > INT32_MAX / 8)
        return WF_ERR_UNSUPPORTED;
    a.units = (int)units;
    a.units_per_xcd = cdiv(a.units, 8);
    const dim3 grid(a.units_per_xcd * 8), block(64 * t.wf * t.wt * t.wk);
#define WF_GEMM(FBV, NBV, WFV, WTV, WKV, NBUFV, NTV)                                          \
    if (t.fb == FBV && t.nb == NBV && t.wf == WFV && t.wt == WTV && t.wk == WKV &&            \
        t.nbuf == NBUFV) {                                                                    \
        prefill_gemm<FBV, NBV, WFV, WTV, WKV, NBUFV, NTV><<<grid, block, 0, stream>>>(a);     \
    } else
#define WF_GEMM_STREAM(NBV)                                                                   \
    WF_GEMM(2, NBV, 4, 1, 1, 2, true) WF_GEMM(2, NBV, 2, 1, 2, 2, true)                       \
    WF_GEMM(2, NBV, 2, 1, 2, 4, true)
    WF_GEMM(2, 1, 1, 1, 2, 2, true) WF_GEMM(2, 1, 1, 1, 2, 4, true)
    WF_GEMM(2, 2, 2, 1, 2, 2, true) WF_GEMM(2, 2, 2, 1, 2, 4, true)
    WF_GEMM(2, 3, 2, 1, 2, 2, true) WF_GEMM(2, 3, 2, 1, 2, 4, true)
    WF_GEMM_STREAM(4) WF_GEMM_STREAM(5) WF_GEMM_STREAM(6) WF_GEMM_STREAM(8)
    WF_GEMM(2, 1, 2, 2, 1, 4, false) WF_GEMM(2, 2, 2, 2, 2, 4, false)
    WF_GEMM(4, 2, 2, 2, 2, 3, false) WF_GEMM(2, 4, 4, 2, 1, 3, false)
    WF_GEMM(4, 4, 4, 2, 1, 3, false)
    { return WF_ERR_UNSUPPORTED; }
#undef WF_GEMM_STREAM
#undef WF_GEMM
    return hipGetLastError() == hipSuccess ? WF_OK : WF_ERR_HIP;
}

}  // namespace wf
