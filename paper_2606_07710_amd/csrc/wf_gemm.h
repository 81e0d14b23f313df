// wf_gemm.h -- the LDS-tiled matrix product shared by the KV-only prefill of
// many tokens and the LM head over row-major weights of any hidden size (gfx950).  Internal
// header; not part of the C ABI.
//
// A workgroup forms D[feature][token] for WF*FB 16-row blocks of W and WT*NB
// 16-row blocks of x; wave (wf, wt) owns FB x NB of them.  The input
// dimension is walked in steps of 64: the step's rows of both operands travel
// to an NBUF-deep LDS ring with global_load_lds, in whole 128-byte lines, one
// barrier a step.  The operands of the next half step are read from LDS
// while the current half's MFMAs run; with WK == 2 two wave groups take one
// half each, and their sums meet in LDS at the end.
//
// LDS holds a 16-row block of either operand as 2 KB.  Row-major sources:
// row r's eight 16-byte granules at r*128, granule g at g ^ (r/2 mod 8), so
// the 16 rows of an MFMA operand read fall in distinct banks (measured: no
// bank conflicts).  Tiled sources (16x32 tiles of 1 KB in operand order): the
// step's two tiles one after the other.  Either way block b, half kk of the
// step is read at 2048*b + a per-lane offset that depends on kk only.
#pragma once

#include "wf_device.h"
#include "wf_lds_dma.h"

namespace wf {

constexpr int kGemmStep = 64;                // input dims per pipeline step
constexpr int kGemmBlockBytes = 16 * kGemmStep * 2;

// A 16-row block of an operand in memory: its first row (row-major) or tile
// (tiled), and how many of its rows exist (>= 1; a row-major block repeats
// the last one in place of the others, whose sums are never used).
struct GemmBlock {
    const char *p;
    int rows;
};

// NT: W with the non-temporal hint (each workgroup the only reader of its
// W rows; the whole-line copies ask for each line once).
// FAR: offsets of 64 bits per lane, for any input dimension.  Else a lane's
// offset within eight rows is 32-bit, and so is the byte offset along the input
// dimension: for dimensions below 2^28, tiled sources below 2^26.
template <int FB, int NB, int WF, int WT, int WK, int NBUF, bool NT, bool FAR = false>
struct TileGemm {
    using Off = std::conditional_t<FAR, long long, int>;
    static constexpr int WAVES = WF * WT * WK;
    static constexpr int HPW = 2 / WK;                   // 32-dim halves per wave and step
    static constexpr int FBLK = FB * WF, TBLK = NB * WT; // 16-row blocks per workgroup
    static constexpr int STAGE = (FBLK + TBLK) * kGemmBlockBytes;
    static constexpr int NLOAD = STAGE / 1024;
    static constexpr int LPW = (NLOAD + WAVES - 1) / WAVES;   // wave loads per wave and step
    static_assert(WK == 1 || WK == 2, "a step has two halves");
    static_assert(FB % 2 == 0, "exchange items are pairs of feature blocks");

    // Whether this wave ends with the sums of item (feature blocks j and
    // j + FB/2, token block nb).
    static __device__ __forceinline__ bool owns(int wk, int j, int nb) {
        return WK == 1 || (j * NB + nb) % WK == wk;
    }

    // acc[fb][nb]: lane (m16, c4) gets features 4*c4 + i of block wf*FB + fb
    // for token m16 of block wt*NB + nb, i < 4, of the items it owns.
    // w_block(b), b < FBLK, and x_block(b), b < TBLK, name the sources; d_in a
    // multiple of 32.  ring: NBUF * STAGE bytes of LDS, free again on return
    // only after a barrier.
    template <class WB, class XB>
    static __device__ __forceinline__ void run(char *ring, const WB &w_block, const XB &x_block,
                                               int d_in, bool w_tiled, bool x_tiled,
                                               f32x4 (&acc)[FB][NB]) {
        const int wave = wave_id();
        const int lane = threadIdx.x % kWave;
        const int m16 = lane & 15;
        const int c4 = lane >> 4;
        const int wf = wave % WF, wt = (wave / WF) % WT, wk = wave / (WF * WT);

        // this wave's copies: load j fills LDS bytes [1024 j, 1024 j + 1024) of a
        // stage; blocks [0, FBLK) are W, the rest x (the last waves may repeat
        // the last load, so that every wave counts the same number)
        const char *base[LPW];
        std::conditional_t<FAR, size_t, unsigned> voff[LPW];
        Off step_bytes[LPW], last_off[LPW];      // bytes per step, offset of the last step
        const size_t ld = (size_t)d_in * 2;
        // (an input dimension of 32 has no second half to read: it repeats the
        // first, and only the copy in the second half's place counts)
        const bool one_half = d_in < kGemmStep;
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int j = min(wave + WAVES * i, NLOAD - 1);
            const int blk = j / 2, hf = j % 2;
            const bool is_w = blk < FBLK;
            const GemmBlock b = is_w ? w_block(blk) : x_block(blk - FBLK);
            if (is_w ? w_tiled : x_tiled) {
                base[i] = b.p + (one_half ? 0 : hf * 1024);
                voff[i] = lane * 16;
                step_bytes[i] = 2048;
                last_off[i] = (Off)max(d_in / 32 - 2, 0) * 1024;
            } else {
                const int r = 8 * hf + lane / 8;             // row of the block
                const int g = (lane & 7) ^ ((r >> 1) & 7);   // granule of the row's line
                const int r0 = min(8 * hf, b.rows - 1);
                base[i] = b.p + r0 * ld;
                voff[i] = (min(r, b.rows - 1) - r0) * ld + (one_half ? g & 3 : g) * 16;
                step_bytes[i] = kGemmStep * 2;
                last_off[i] = (Off)max(d_in - kGemmStep, 0) * 2;
            }
        }
        // an input dimension of 64k + 32 ends with a step over its last 64 dims,
        // of which only the second half counts
        const bool half_tail = d_in % kGemmStep != 0;
        const int n_steps = d_in / kGemmStep + half_tail;
        auto issue = [&](int st, int buf) __attribute__((always_inline)) {
            const unsigned slot = lds_addr(ring) + buf * STAGE;
#pragma unroll
            for (int i = 0; i < LPW; ++i) {
                const int j = min(wave + WAVES * i, NLOAD - 1);
                const char *src = base[i] + min(st * step_bytes[i], last_off[i]);
                const bool nt = NT && j / 2 < FBLK;
                if constexpr (FAR) {
                    if (nt)
                        lds_dma16<true>(src + voff[i], slot + j * 1024);
                    else
                        lds_dma16<false>(src + voff[i], slot + j * 1024);
                } else if (nt)
                    lds_dma16_so<true>(src, voff[i], slot + j * 1024);
                else
                    lds_dma16_so<false>(src, voff[i], slot + j * 1024);
            }
        };

        unsigned wo[HPW], xo[HPW];           // operand offsets of this wave's halves
#pragma unroll
        for (int k = 0; k < HPW; ++k) {
            const int kk = wk * HPW + k;
            const unsigned rm = m16 * 128 + (((4 * kk + c4) ^ (m16 >> 1)) & 7) * 16;
            const unsigned tl = kk * 1024 + lane * 16;
            wo[k] = (w_tiled ? tl : rm) + wf * FB * kGemmBlockBytes;
            xo[k] = (x_tiled ? tl : rm) + (FBLK + wt * NB) * kGemmBlockBytes;
        }

#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[fb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

        bf16x8 wr[2][FB], xr[2][NB];         // operands in use and those arriving
        auto load = [&](auto set, int bufi, int k) __attribute__((always_inline)) {
            constexpr int P = decltype(set)::value;
            const WF_LDS(char) *sp = (const WF_LDS(char) *)ring + bufi * STAGE;
#pragma unroll
            for (int fb = 0; fb < FB; ++fb)
                wr[P][fb] = __builtin_bit_cast(
                    bf16x8, *(const WF_LDS(u32x4) *)(sp + wo[k] + fb * kGemmBlockBytes));
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                xr[P][nb] = __builtin_bit_cast(
                    bf16x8, *(const WF_LDS(u32x4) *)(sp + xo[k] + nb * kGemmBlockBytes));
        };
        auto mma = [&](auto set) __attribute__((always_inline)) {
            constexpr int P = decltype(set)::value;
#pragma unroll
            for (int fb = 0; fb < FB; ++fb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[fb][nb] = mfma16x16x32(wr[P][fb], xr[P][nb], acc[fb][nb]);
        };
        auto wait_later = [&](int later) __attribute__((always_inline)) {
            static_assert(NBUF <= 4, "wait counts");
            if (NBUF > 3 && later >= 3)
                wait_vmcnt<(NBUF > 3 ? 3 : 0) * LPW>();
            else if (NBUF > 2 && later >= 2)
                wait_vmcnt<(NBUF > 2 ? 2 : 0) * LPW>();
            else if (later >= 1)
                wait_vmcnt<LPW>();
            else
                wait_vmcnt<0>();
        };
        // Step st's operands are in registers (or arriving); make step st + 1's
        // data visible and refill st's ring buffer.
        auto advance = [&](int st, int bufi) __attribute__((always_inline)) {
            wait_later(min(NBUF - 2, n_steps - 2 - st));
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (st + NBUF < n_steps)
                issue(st + NBUF, bufi);
        };

#pragma unroll
        for (int s = 0; s < NBUF; ++s)
            if (s < n_steps)
                issue(s, s);
        wait_later(min(NBUF - 1, n_steps - 1));
        asm volatile("s_barrier" ::: "memory");
        load(ic<0>{}, 0, 0);
        int buf = 0;
        auto next = [&](int b) { return b + 1 == NBUF ? 0 : b + 1; };
        if constexpr (HPW == 2) {
            for (int st = 0; st + 1 < n_steps; ++st) {
                load(ic<1>{}, buf, 1);
                mma(ic<0>{});
                advance(st, buf);
                buf = next(buf);
                load(ic<0>{}, buf, 0);
                mma(ic<1>{});
            }
            load(ic<1>{}, buf, 1);
            if (!half_tail)
                mma(ic<0>{});
            mma(ic<1>{});
        } else {
            const bool skip_last = half_tail && wk == 0;
            int st = 0;
            for (; st + 2 < n_steps; st += 2) {
                advance(st, buf);
                buf = next(buf);
                load(ic<1>{}, buf, 0);
                mma(ic<0>{});
                advance(st + 1, buf);
                buf = next(buf);
                load(ic<0>{}, buf, 0);
                mma(ic<1>{});
            }
            if (st + 1 < n_steps) {
                advance(st, buf);
                load(ic<1>{}, next(buf), 0);
                mma(ic<0>{});
                if (!skip_last)
                    mma(ic<1>{});
            } else if (!skip_last) {
                mma(ic<0>{});
            }
        }

        // ---- the k groups' sums meet in LDS: item (pair j, token block nb) is
        // finished by group (j*NB + nb) mod WK, which adds the others in order
        if constexpr (WK > 1) {
            constexpr int ITEMS = FB / 2 * NB;
            WF_LDS(char) *ex = (WF_LDS(char) *)ring;
            constexpr int GIVEN = ITEMS - ITEMS / WK;        // items a wave hands over, at most
            static_assert(WAVES * GIVEN * 2048 <= NBUF * STAGE, "exchange fits the ring");
            auto slot = [&](int w, int k, int it) {          // wave w of group k, its item it
                return ex + (w * GIVEN + it - (it + WK - 1 - k) / WK) * 2048 + lane * 16;
            };
            __syncthreads();
            const int wq = wave % (WF * WT);
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
                if (it % WK != wk) {
                    WF_LDS(f32x4) *d = (WF_LDS(f32x4) *)slot(wave, wk, it);
                    d[0] = acc[it / NB][it % NB];
                    d[64] = acc[it / NB + FB / 2][it % NB];
                }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
                if (it % WK == wk) {
#pragma unroll
                    for (int o = 0; o < WK; ++o) {
                        if (o == it % WK)
                            continue;
                        const WF_LDS(f32x4) *d = (const WF_LDS(f32x4) *)slot(o * WF * WT + wq, o, it);
                        acc[it / NB][it % NB] += d[0];
                        acc[it / NB + FB / 2][it % NB] += d[64];
                    }
                }
        }
    }
};

}  // namespace wf
