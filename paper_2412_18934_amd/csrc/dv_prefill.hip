// HIP kernels (gfx950 / CDNA4) of the large-M prefill: embedding and first
// norm, the MFMA GEMM with the projections' epilogues, causal attention.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "dv_device.h"
#include "dv_internal.h"

// ---------------------------------------------------------------------------
// Large-M prefill: a prompt chunk of M tokens (padded to Mp, a multiple of 16
// and at least 48) in one causal pass.  The projections are a dense contraction here, so
// they run on an MFMA GEMM over the packed weights of the verify path (block
// (k-step s, 16-row block gb) at (s NB + gb) 512) and split-layout
// activations of the whole chunk (MT = Mp / 16 token tiles), with the verify
// path's epilogues fused: rotary + K/V write, SwiGLU, residual + the next
// norm's input.  Every norm's 1/rms, a per-token scalar, is applied by its
// consumer's epilogue from sums of squares over 64-row slices (Mp x d / 64
// partials), so no fp32 GEMM output goes through HBM.

constexpr int PF_THREADS = 256;

// Embedding rows of the chunk: x = E[token], the first norm's numerator
// x * gain in split layout and the sums of squares of 64-column slices;
// tokens >= M get zeros.  One workgroup per token, 4 columns per thread.
__global__ __launch_bounds__(PF_THREADS) void k_pf_embed(const int32_t *tokens, const uint16_t *embed, int M, int d,
                                                         int MT, const uint16_t *gain, float *x, uint16_t *us,
                                                         float *ssq)
{
    const int m = blockIdx.x, nsq = d / 64;
    for (int k = 4 * threadIdx.x; k < d; k += 4 * PF_THREADS) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (m < M) {
            const uint2 e = *reinterpret_cast<const uint2 *>(embed + (size_t)tokens[m] * d + k);
            v = make_float4(__uint_as_float(e.x << 16), __uint_as_float(e.x & 0xffff0000u), __uint_as_float(e.y << 16),
                            __uint_as_float(e.y & 0xffff0000u));
        }
        *reinterpret_cast<float4 *>(x + (size_t)m * d + k) = v;
        store_split4(us, m, k, MT,
                     make_float4(v.x * bf2f(gain[k]), v.y * bf2f(gain[k + 1]), v.z * bf2f(gain[k + 2]),
                                 v.w * bf2f(gain[k + 3])));
        // 16 neighbouring threads hold one 64-column slice
        float ss = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, v.w * v.w)));
        ss += __shfl_xor(ss, 1);
        ss += __shfl_xor(ss, 2);
        ss += __shfl_xor(ss, 4);
        ss += __shfl_xor(ss, 8);
        if ((threadIdx.x & 15) == 0) ssq[(size_t)m * nsq + k / 64] = ss;
    }
}

// The prefill GEMM.  A unit is 64 NWR rows x a token group of TT (or TT - 1)
// token tiles x one of KS ranges of K, one workgroup of 8 waves each: NWR row
// waves (4 blocks each) in NKG K groups.  A step is a k-step of 32 columns
// (int8 weights: a pair of them); K group kg takes steps kg, kg + NKG, ... of
// the unit.  Per step each wave loads its 4 weight blocks into registers, its
// K group stages the activation slab of the token group (hi + lo) in LDS, and
// each wave runs 8 TT MFMAs per k-step (16x16x32 bf16, hi then lo into the
// same accumulators; all hi parts of a token tile first, so that no MFMA
// waits for the one before it), the next tile's B operands being read from LDS
// meanwhile (read just before use: 27648 x 5120 at 1024 tokens 479 us, read a
// tile ahead 413).  A wave's loads return in order, so weights and activations
// share one lead of LEAD steps (activations first in each step's loads); the
// slab is stashed one step ahead into two LDS buffers.
//
// The K groups' sums are added through LDS, each group taking a share of the
// token tiles, the KS ranges' through memory: every unit publishes its partial sums (device-coherent stores, completed
// before it counts itself), and the unit of a tile that counts last adds them
// in range order and runs the epilogue, so every sum has a fixed order and no
// workgroup waits for another.
//
// int8 QKV (STEP_SUM) adds up each 64-column step by itself, lo parts first,
// and adds that to the running sums: an MFMA rounds at the size of what it
// accumulates into, and in one chain those are 4 roundings per step at the size of
// the whole sum instead of 1.  The keys and values are rounded to bf16 next,
// so every error here moves some of them to the other side of a midpoint, and
// all later layers attend to those.  Relative error of all K/V against 64 bits, two
// 13B layers, 500 tokens: 2.9e-4, 3.7e-4 in one chain (3.4e-4 through the
// verify kernels, whose sums are 4 shorter chains); of layer 0's 2.2e-5,
// 3.7e-5 (3.1e-5).  The same for O, gate/up and down changes neither figure.
// It costs 1% of that prefill (1206 -> 1217 us), at every projection 7%.
template <int EPI, int NWR, int NKG, int TT, int LEAD, bool Q8>
__global__ __launch_bounds__(64 * NWR * NKG) void k_pf_gemm(PfArgs a)
{
    constexpr int NT = 64 * NWR * NKG, GT = 64 * NWR, BW = 4, SK = Q8 ? 2 : 1;
    // the activation slab of a step: XE u32x4 (hi + lo of TT token tiles, SK
    // k-steps), XL of them staged per thread of the K group
    constexpr int XE = SK * TT * 128, XL = (XE + GT - 1) / GT;
    static_assert(NT == 512 && LEAD >= 2, "8 waves; the stash needs its loads a step earlier");
    constexpr int TI = (TT + NKG - 1) / NKG;  // token tiles per K group after the sums
    // blocks of the K groups' sums exchanged at a time, as LDS allows
    constexpr int HB = TT * (NKG - 1) * NWR * BW <= 150 ? BW : 2;
    constexpr bool STEP_SUM = Q8 && EPI == EPI_QKV;
    constexpr int XN = NKG * 2 * XE, RN = TT * (NKG - 1) * NWR * HB * 64;
    __shared__ u32x4 xsm[XN > RN ? XN : RN];
    __shared__ float rinv_s[16 * TT];
    __shared__ int last_s;
    // the wave number is the same in all lanes, which the compiler cannot see:
    // without saying so every buffer load's scalar offset becomes a loop over
    // the lanes' values
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / NWR, wr = wave % NWR, gt = tid - kg * GT;
    // 1-D grid, XCD-aware: workgroups are dispatched to the 8 XCDs round
    // robin (workgroup b to XCD b % 8, 32 CUs each), so XCD x takes units
    // [x per, (x + 1) per) of the row-tile-major order: every XCD gets the
    // same count, and the token groups of a row tile and K range share one
    // XCD's L2 for the weights (at most two XCDs at a chunk boundary).
    const int n_tt = a.n_tt, KS = a.ks, n_rt = (a.NB + NWR * BW - 1) / (NWR * BW);
    const int n_units = n_rt * KS * n_tt, per = (n_units + 7) / 8;
    const int unit = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (unit >= n_units) return;  // padding of the grid to 8 x per
    const int rtile = unit / (KS * n_tt), rest = unit - rtile * KS * n_tt, ks = rest / n_tt, tg = rest - ks * n_tt;
    const int tt0 = tg * a.MT / n_tt;                          // first token tile of the group
    const bool full = (tg + 1) * a.MT / n_tt - tt0 == TT;      // or one tile less
    const int gb0 = (rtile * NWR + wr) * BW;                   // first block of this wave
    const int S = a.K / (32 * SK), sb = ks * S / KS, se = (ks + 1) * S / KS;
    const int rounds = (se - sb + NKG - 1) / NKG;
    // buffer loads: the per-lane byte offsets stay fixed, a scalar offset moves
    // by one step (so no address register is rewritten while a load into a
    // neighbouring register is in flight); blocks past NB re-read the last
    // block (their sums are dropped)
    const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.packed), rx = rsrc_of(a.xs);
    uint32_t wofs[BW], xofs[XL];
#pragma unroll
    for (int b = 0; b < BW; ++b) wofs[b] = (uint32_t)(min(gb0 + b, a.NB - 1) * 1024 + lane * 16);
#pragma unroll
    for (int i = 0; i < XL; ++i) {
        const int e = min(gt + GT * i, XE - 1), hf = e / (TT * 128), r = e - hf * TT * 128;
        const int tile = hf * a.MT + min(tt0 + r / 128, a.MT - 1);
        xofs[i] = (uint32_t)((tile * 128 + r % 128) * 16);
    }
    const uint32_t wstep = (uint32_t)a.NB * 1024u, xstep = (uint32_t)a.MT * 2048u * SK;
    u32x4 wb[LEAD][BW], stg[LEAD][XL];
    auto fetch = [&](int j, int r) {
        const int st = min(sb + r * NKG + kg, S - 1);
#pragma unroll
        for (int i = 0; i < XL; ++i)
            stg[j][i] = __builtin_amdgcn_raw_buffer_load_b128(rx, xofs[i], (uint32_t)st * xstep, 0);
#pragma unroll
        for (int b = 0; b < BW; ++b)
            wb[j][b] = __builtin_amdgcn_raw_buffer_load_b128(rw, wofs[b], (uint32_t)st * wstep, DV_NT);
    };
    u32x4 *slab = xsm + kg * 2 * XE;
    auto stash = [&](int j, int buf) {
#pragma unroll
        for (int i = 0; i < XL; ++i)
            if (XE % GT == 0 || gt + GT * i < XE) slab[buf * XE + gt + GT * i] = stg[j][i];
    };
    f32x4 acc[TT][BW];
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int b = 0; b < BW; ++b) acc[t][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // a step held in register slot j: the B operands of tile and k-step q + 1
    // are read while the MFMAs of q run (the scheduling barriers keep the
    // compiler from moving the reads down to their use, where every tile's
    // MFMAs waited for the LDS)
    auto step = [&](int j, int buf) {
        const u32x4 *x = slab + buf * XE + lane;
        u32x4 hv[2], lv[2];
        auto bread = [&](int q) {
            const int t = q / SK, hf = q % SK;
            hv[q & 1] = x[(hf * TT + t) * 128];
            lv[q & 1] = x[(hf * TT + t) * 128 + 64];
        };
        bread(0);
        f32x4 sum[BW];  // STEP_SUM: of this step and tile
#pragma unroll
        for (int q = 0; q < SK * TT; ++q) {
            const int t = q / SK, hf = q % SK;
            if (t == TT - 1 && !full) break;
            if (q + 1 < SK * TT) bread(q + 1);
            __builtin_amdgcn_sched_barrier(0);
            const bf16x8 hi = __builtin_bit_cast(bf16x8, hv[q & 1]), lo = __builtin_bit_cast(bf16x8, lv[q & 1]);
            bf16x8 w[BW];
#pragma unroll
            for (int b = 0; b < BW; ++b) {
                if constexpr (Q8) {
                    const uint2 c0 = i8x4_to_bf16(wb[j][b][2 * hf]), c1 = i8x4_to_bf16(wb[j][b][2 * hf + 1]);
                    w[b] = __builtin_bit_cast(bf16x8, (u32x4){c0.x, c0.y, c1.x, c1.y});
                } else {
                    w[b] = __builtin_bit_cast(bf16x8, wb[j][b]);
                }
            }
            if constexpr (STEP_SUM) {
#pragma unroll
                for (int b = 0; b < BW; ++b) {
                    if (hf == 0) sum[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
                    sum[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[b], lo, sum[b], 0, 0, 0);
                }
#pragma unroll
                for (int b = 0; b < BW; ++b) sum[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[b], hi, sum[b], 0, 0, 0);
                if (hf == SK - 1) {
                    // (the empty asm keeps each addition in its place: left to
                    // the end of the step they hold every tile's sums at once)
#pragma unroll
                    for (int b = 0; b < BW; ++b) {
                        acc[t][b] += sum[b];
                        asm volatile("" : "+v"(acc[t][b]));
                    }
                }
            } else {
#pragma unroll
                for (int b = 0; b < BW; ++b)
                    acc[t][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[b], hi, acc[t][b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < BW; ++b)
                    acc[t][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[b], lo, acc[t][b], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // Loads and stashes are issued unconditionally (steps past the end re-read
    // the last one and are never used), so the number of loads in flight
    // behind each one is the same on every path and every wait is the one the
    // pipeline needs.  Round r: weights in register slot r % LEAD, activations
    // in LDS buffer r % 2, stashed one round ahead; the barrier after round r
    // makes round r + 1's stash visible, and every read of buffer r % 2 is
    // done before round r + 1 overwrites it.
#pragma unroll
    for (int j = 0; j < LEAD; ++j) fetch(j, j);
    if (EPI != EPI_RESID) {
        // 1/rms of the group's tokens, 4 threads each
        const int m = min(tid >> 2, 16 * TT - 1), c = tid & 3, tok = min(tt0 * 16 + m, 16 * a.MT - 1);
        const float *p = a.ssq_in + (size_t)tok * a.nsq_in;
        float sum = 0.f;
        for (int i0 = c; i0 < a.nsq_in; i0 += 32) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = p[min(i0 + 4 * i, a.nsq_in - 1)];
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += i0 + 4 * i < a.nsq_in ? v[i] : 0.f;
        }
        sum += __shfl_xor(sum, 1);
        sum += __shfl_xor(sum, 2);
        if (c == 0) rinv_s[m] = 1.0f / sqrtf(sum / (float)a.d + a.eps);
    }
    stash(0, 0);
    __syncthreads();
    for (int r0 = 0; r0 < rounds; r0 += LEAD) {
#pragma unroll
        for (int j = 0; j < LEAD; ++j) {
            const int r = r0 + j;
            if (sb + r * NKG + kg < se) step(j, r & 1);
            stash((j + 1) % LEAD, (r + 1) & 1);
            fetch(j, r + LEAD);
            __syncthreads();
        }
    }
    // The K groups share what follows by token tiles: group kg ends up with the
    // tiles kg, kg + NKG, ... (own[i] = tile kg + NKG i), so that all waves
    // sum, fold and run the epilogue.
    const int cnt_t = full ? TT : TT - 1;
    f32x4 own[TI][BW];
    if constexpr (NKG == 1) {
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int b = 0; b < BW; ++b) own[t][b] = acc[t][b];
    } else {
        // through LDS, HB blocks at a time: a wave leaves the tiles of the
        // other groups there and adds theirs to its own, in group order
#pragma unroll
        for (int b0 = 0; b0 < BW; b0 += HB) {
            if (b0) __syncthreads();
#pragma unroll
            for (int t = 0; t < TT; ++t) {
                if (t % NKG == kg) {
#pragma unroll
                    for (int b = 0; b < HB; ++b) own[t / NKG][b0 + b] = acc[t][b0 + b];
                } else {
                    const int r = kg < t % NKG ? kg : kg - 1;
#pragma unroll
                    for (int b = 0; b < HB; ++b)
                        xsm[(((t * (NKG - 1) + r) * NWR + wr) * HB + b) * 64 + lane] =
                            __builtin_bit_cast(u32x4, acc[t][b0 + b]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int t = min(kg + NKG * i, TT - 1);
                f32x4 sum[HB];
#pragma unroll
                for (int b = 0; b < HB; ++b) sum[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < NKG; ++q) {
                    const int r = q < kg ? q : q - 1;
#pragma unroll
                    for (int b = 0; b < HB; ++b)
                        sum[b] += q == kg ? own[i][b0 + b]
                                          : __builtin_bit_cast(f32x4, xsm[(((t * (NKG - 1) + r) * NWR + wr) * HB + b) * 64 + lane]);
                }
#pragma unroll
                for (int b = 0; b < HB; ++b) own[i][b0 + b] = sum[b];
            }
        }
    }
    if (KS > 1) {
        constexpr int PW = NWR * BW * TT * 64;  // 16-byte partials of a unit
        const __amdgpu_buffer_rsrc_t pr = rsrc_of(a.part);
        auto pofs = [&](int u, int t, int b) -> uint32_t {
            return (uint32_t)(u * PW + ((t * BW + b) * NWR + wr) * 64 + lane) * 16u;
        };
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            if (kg + NKG * i >= cnt_t) break;
#pragma unroll
            for (int b = 0; b < BW; ++b)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, own[i][b]), pr,
                                                       pofs(unit, kg + NKG * i, b), 0, 16);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            uint32_t *cnt = a.cnt + rtile * n_tt + tg;
            const uint32_t old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last_s = old == (uint32_t)(KS - 1);
            if (old == (uint32_t)(KS - 1)) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!last_s) return;
        // ranges in order, KB ranges of a tile in flight together
        constexpr int KB = 4;
        const int u0 = rtile * KS * n_tt + tg;
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            const int t = min(kg + NKG * i, cnt_t - 1);
            f32x4 sum[BW];
#pragma unroll
            for (int b = 0; b < BW; ++b) sum[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
            for (int k0 = 0; k0 < KS; k0 += KB) {
                u32x4 raw[KB][BW];
#pragma unroll
                for (int q = 0; q < KB; ++q)
#pragma unroll
                    for (int b = 0; b < BW; ++b)
                        raw[q][b] = __builtin_amdgcn_raw_buffer_load_b128(pr, pofs(u0 + min(k0 + q, KS - 1) * n_tt, t, b), 0, 16);
#pragma unroll
                for (int q = 0; q < KB; ++q) {
                    if (k0 + q < KS) {
#pragma unroll
                        for (int b = 0; b < BW; ++b) sum[b] += __builtin_bit_cast(f32x4, raw[q][b]);
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < BW; ++b) own[i][b] = sum[b];
        }
    }
    if constexpr (Q8) {
        // W = scale[row] q
#pragma unroll
        for (int b = 0; b < BW; ++b) {
            const f32x4 rs = *reinterpret_cast<const f32x4 *>(a.scale + min(gb0 + b, a.NB - 1) * 16 + 4 * (lane >> 4));
#pragma unroll
            for (int i = 0; i < TI; ++i) own[i][b] *= rs;
        }
    }

    // ---- epilogues: lane l holds rows 4 (l / 16) + jj of block gb0 + b for
    // token (tt0 + t) 16 + l % 16
    const int n16 = lane & 15, r4 = 4 * (lane >> 4);
    if (EPI == EPI_QKV) {
        const int per_seg = a.d / DV_GEMM_TILE, per_head = a.hd / DV_GEMM_TILE, half = a.hd / 2;
#pragma unroll
        for (int p = 0; p < BW / 2; ++p) {
            const int gb = gb0 + 2 * p;
            if (gb >= a.NB) break;
            const int tile = gb >> 1, seg = tile / per_seg, tt = tile - seg * per_seg;
            const int h = tt / per_head, j0 = (tt - h * per_head) * 16 + r4;
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int t = kg + NKG * i;
                if (t >= cnt_t) break;
                const int ml = t * 16 + n16, m = tt0 * 16 + ml;
                if (m >= a.M) continue;
                const float ri = rinv_s[ml];
                float y1[4], y2[4];
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    y1[jj] = own[i][2 * p][jj] * ri;
                    y2[jj] = own[i][2 * p + 1][jj] * ri;
                }
                const int pos = a.P0 + m;
                if (seg < 2) {
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) {
                        const float c = a.rope_cos[(size_t)pos * half + j0 + jj];
                        const float sn = a.rope_sin[(size_t)pos * half + j0 + jj];
                        const float o1 = y1[jj] * c - y2[jj] * sn, o2 = y2[jj] * c + y1[jj] * sn;
                        y1[jj] = o1;
                        y2[jj] = o2;
                    }
                }
                if (seg == 0) {
                    float *qr = a.q + (size_t)m * a.d + h * a.hd + j0;
                    *reinterpret_cast<float4 *>(qr) = make_float4(y1[0], y1[1], y1[2], y1[3]);
                    *reinterpret_cast<float4 *>(qr + half) = make_float4(y2[0], y2[1], y2[2], y2[3]);
                } else if (seg == 1) {  // K: [H][cap][hd]
                    uint16_t *kr = reinterpret_cast<uint16_t *>(a.kc) + ((size_t)h * a.cap + pos) * a.hd + j0;
                    *reinterpret_cast<uint2 *>(kr) = make_uint2(f2bf(y1[0]) | (uint32_t)f2bf(y1[1]) << 16,
                                                                f2bf(y1[2]) | (uint32_t)f2bf(y1[3]) << 16);
                    *reinterpret_cast<uint2 *>(kr + half) = make_uint2(f2bf(y2[0]) | (uint32_t)f2bf(y2[1]) << 16,
                                                                       f2bf(y2[2]) | (uint32_t)f2bf(y2[3]) << 16);
                } else {                // V: [H][cap/32][hd][32]
                    uint16_t *vh = reinterpret_cast<uint16_t *>(a.vc) + (size_t)h * a.hd * a.cap;
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) {
                        vh[v_index(j0 + jj, pos, a.hd)] = f2bf(y1[jj]);
                        vh[v_index(j0 + jj + half, pos, a.hd)] = f2bf(y2[jj]);
                    }
                }
            }
        }
    } else if (EPI == EPI_SWIGLU) {
        // gate block 2p and up block 2p + 1 hold h columns 16 (gb / 2) + ...
#pragma unroll
        for (int p = 0; p < BW / 2; ++p) {
            const int gb = gb0 + 2 * p;
            if (gb >= a.NB) break;
            const int f0 = 16 * (gb >> 1) + r4;
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int t = kg + NKG * i;
                if (t >= cnt_t) break;
                const int ml = t * 16 + n16, m = tt0 * 16 + ml;
                float hv[4] = {0.f, 0.f, 0.f, 0.f};
                if (m < a.M) {
                    const float ri = rinv_s[ml];
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) hv[jj] = silu(own[i][2 * p][jj] * ri) * (own[i][2 * p + 1][jj] * ri);
                }
                store_split4(a.hs, m, f0, a.MT, make_float4(hv[0], hv[1], hv[2], hv[3]));
            }
        }
    } else if (EPI == EPI_LOGITS) {
        if (gb0 < a.NB) {
            const size_t V = (size_t)a.NB * 16;
            const int n_parts = (a.NB + 3) / 4;
            const bool vec = (reinterpret_cast<uintptr_t>(a.logits) & 15) == 0;
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int t = kg + NKG * i;
                if (t >= cnt_t) break;
                const int ml = t * 16 + n16, m = tt0 * 16 + ml;
                const float ri = rinv_s[ml];
                float best = -INFINITY;
                int bi = 16 * (gb0 + BW);  // as the streaming kernel's where no value compares larger
#pragma unroll
                for (int b = 0; b < BW; ++b) {
                    if (gb0 + b >= a.NB) break;
                    const int r = 16 * (gb0 + b) + r4;
                    float v[4];
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) {
                        v[jj] = own[i][b][jj] * ri;
                        if (v[jj] > best) {
                            best = v[jj];
                            bi = r + jj;
                        }
                    }
                    if (a.logits && m < a.M) {
                        float *lp = a.logits + m * V + r;
                        if (vec) {
                            *reinterpret_cast<float4 *>(lp) = make_float4(v[0], v[1], v[2], v[3]);
                        } else {
#pragma unroll
                            for (int jj = 0; jj < 4; ++jj) lp[jj] = v[jj];
                        }
                    }
                }
                // larger value, then lower row
#pragma unroll
                for (int off = 16; off < 64; off <<= 1) {
                    const float v2 = __shfl_xor(best, off);
                    const int i2 = __shfl_xor(bi, off);
                    if (v2 > best || (v2 == best && i2 < bi)) {
                        best = v2;
                        bi = i2;
                    }
                }
                if (lane < 16 && m < a.M) {
                    a.arg_val[(size_t)m * n_parts + gb0 / 4] = best;
                    a.arg_idx[(size_t)m * n_parts + gb0 / 4] = bi;
                }
            }
        }
    } else {  // EPI_RESID
        if (gb0 < a.NB) {
            const int nsq = a.d / 64;
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int t = kg + NKG * i;
                if (t >= cnt_t) break;
                const int ml = t * 16 + n16, m = tt0 * 16 + ml;
                float ss = 0.f;
#pragma unroll
                for (int b = 0; b < BW; ++b) {
                    const int r = 16 * (gb0 + b) + r4;
                    float4 xv = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (m < a.M) {
                        float *xp = a.x + (size_t)m * a.d + r;
                        xv = *reinterpret_cast<const float4 *>(xp);
                        xv.x += own[i][b][0];
                        xv.y += own[i][b][1];
                        xv.z += own[i][b][2];
                        xv.w += own[i][b][3];
                        *reinterpret_cast<float4 *>(xp) = xv;
                    }
                    ss = fmaf(xv.x, xv.x, fmaf(xv.y, xv.y, fmaf(xv.z, xv.z, fmaf(xv.w, xv.w, ss))));
                    store_split4(a.us, m, r, a.MT,
                                 make_float4(xv.x * bf2f(a.gain[r]), xv.y * bf2f(a.gain[r + 1]),
                                             xv.z * bf2f(a.gain[r + 2]), xv.w * bf2f(a.gain[r + 3])));
                }
                ss += __shfl_xor(ss, 16);
                ss += __shfl_xor(ss, 32);
                if (lane < 16) a.ssq_out[(size_t)m * nsq + gb0 / 4] = ss;
            }
        }
    }
}

// Causal attention of the chunk's queries (positions P0 + i) over cache slots
// [0, P0 + i].  Workgroup = 64 queries of one head, each wave 16 of them; the
// workgroup stages every 32-key tile up to its last query in LDS once (K rows
// and the tile's V block, rows padded against bank conflicts; the next tile's
// global loads are in flight while the current one is used), and each wave
// uses the tiles up to its own last query.  The scores and the running
// softmax follow the tree-attention kernel (MFMA with q split in hi + lo,
// exp2 in log2 units); the output goes to the O projection's operand (split
// layout of MT token tiles).  Grid (heads, query blocks) with the last query
// block first: workgroups are dispatched in order, so the longest ones (the
// most keys) start first and the short ones fill in behind them.
//
// A wave's tiles are a serial chain of about 1.3 us each, so with few query
// blocks (short prompts) the workgroup takes NKG key groups of 4 waves: group
// kg has the tiles kg, kg + NKG, ..., each group stages its own, and the
// groups' outputs are combined through LDS in group order.  One group and two,
// us (and before the wave number and the tile loads' bounds were made uniform):
// 7B heads, 150 queries behind 333 keys 24.7, 19.6 (26.5); 13B heads, 136
// behind 1839 80, 61 (88); 500 alone 32.5, 26.9 (34.6); 1024 alone 56.7, 60
// (60.9).
template <int HD, int NKG>
__global__ __launch_bounds__(256 * NKG) void k_attn_causal(const float *q, const uint16_t *kc_l, const uint16_t *vc_l,
                                                     int M, int P0, int H, int cap, int MT, uint16_t *out)
{
    constexpr int NC = HD / 32, ND = HD / 16;
    constexpr int KROW = HD * 2 + 16;          // bytes per staged key row (padded)
    constexpr int VROW = 80;                   // bytes per staged dim row of 32 values (padded)
    constexpr int KBYTES = 32 * KROW, VBYTES = HD * VROW;
    constexpr int KCH = 32 * HD / 8, VCH = HD * 4;  // 16-byte chunks of a tile's K and V
    constexpr int CPT = (KCH + VCH + 255) / 256;     // chunks per thread
    constexpr int STG = 2 * (KBYTES + VBYTES);       // a key group's two buffers
    constexpr int OROW = HD + 4, OBYTES = NKG > 1 ? (NKG - 1) * 64 * OROW * 4 : 0;  // combined outputs
    __shared__ __align__(16) unsigned char smem_all[NKG * STG > OBYTES ? NKG * STG : OBYTES];
    __shared__ float sm_m[NKG][64], sm_l[NKG][64];
    // (uniform in a wave, said so for scalar addresses and branches)
    const int kg = NKG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    unsigned char *const smem_g = smem_all + kg * STG;
    const int h = blockIdx.x, tid = threadIdx.x & 255, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int q0 = (gridDim.y - 1 - blockIdx.y) * 64;
    const int qb = q0 + wave * 16;               // first query of this wave
    const int D = H * HD;
    const int kend_wg = P0 + min(q0 + 64, M);    // keys the workgroup may see
    const int ntile = (kend_wg + 31) / 32;
    const bool active = qb < M;
    const int kend = P0 + min(qb + 16, M);       // keys this wave may see
    const int wtiles = active ? (kend + 31) / 32 : 0;
    const float scale2 = 1.4426950408889634f / sqrtf((float)HD);
    const uint16_t *kc = kc_l + (size_t)h * cap * HD;
    const uint16_t *vc = vc_l + (size_t)h * HD * cap;
    const int qi = min(qb + n, M - 1);          // this lane's query (B operand column)
    const int lim = P0 + qb + n;                // last key it sees

    bf16x8 qh[NC], ql[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const float *qp = q + (size_t)qi * D + h * HD + 32 * c + 8 * g;
        split_hi_lo(*reinterpret_cast<const float4 *>(qp), *reinterpret_cast<const float4 *>(qp + 4), qh[c], ql[c]);
    }
    // global -> registers -> LDS staging of tile t: chunk e < KCH is 16 bytes
    // of key row e / (HD / 8) (rows past the workgroup's last key repeat it),
    // the rest 16 bytes of the tile's V block (dim row, 8 slots)
    u32x4 stg[CPT];
    auto fetch = [&](int t) {
        const int k0 = 32 * t;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            const int e = tid + 256 * i;
            if (e < KCH) {
                const int r = e / (HD / 8), c8 = e % (HD / 8);
                const int key = min(k0 + r, kend_wg - 1);
                stg[i] = *reinterpret_cast<const u32x4 *>(kc + (size_t)key * HD + 8 * c8);
            } else if (e < KCH + VCH) {
                const int ev = e - KCH;
                stg[i] = *reinterpret_cast<const u32x4 *>(vc + (size_t)(k0 >> 5) * HD * 32 + 8 * ev);
            }
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            unsigned char *const sm = smem_g + buf * (KBYTES + VBYTES);
            const int e = tid + 256 * i;
            if (e < KCH) {
                const int r = e / (HD / 8), c8 = e % (HD / 8);
                *reinterpret_cast<u32x4 *>(sm + r * KROW + 16 * c8) = stg[i];
            } else if (e < KCH + VCH) {
                const int ev = e - KCH, dr = ev >> 2, c8 = ev & 3;
                *reinterpret_cast<u32x4 *>(sm + KBYTES + dr * VROW + 16 * c8) = stg[i];
            }
        }
    };

    float m_run = -INFINITY, l_run = 0.f;
    f32x4 o[ND];
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) o[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto process = [&](int t, int buf) {
        const int k0 = 32 * t;
        const unsigned char *ks = smem_g + buf * (KBYTES + VBYTES), *vs = ks + KBYTES;
        const int ra = 8 * (n >> 2) + (n & 3), rb = ra + 4;
        f32x4 sa = (f32x4){0.f, 0.f, 0.f, 0.f}, sb = sa;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const bf16x8 ka8 = *reinterpret_cast<const bf16x8 *>(ks + ra * KROW + 64 * c + 16 * g);
            const bf16x8 kb8 = *reinterpret_cast<const bf16x8 *>(ks + rb * KROW + 64 * c + 16 * g);
            sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka8, qh[c], sa, 0, 0, 0);
            sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb8, qh[c], sb, 0, 0, 0);
            sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka8, ql[c], sa, 0, 0, 0);
            sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb8, ql[c], sb, 0, 0, 0);
        }
        // scores of query (lane n) for keys k0 + 8g + i
        float sv[8], mt = -INFINITY;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int key = k0 + 8 * g + i;
            const float sc = (i < 4 ? sa[i] : sb[i - 4]) * scale2;
            sv[i] = key <= lim ? sc : -INFINITY;
            mt = fmaxf(mt, sv[i]);
        }
        mt = fmaxf(mt, __shfl_xor(mt, 16));
        mt = fmaxf(mt, __shfl_xor(mt, 32));
        const float mnew = fmaxf(m_run, mt);
        const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - mnew);
        float ps = 0.f, pv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            pv[i] = sv[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sv[i] - mnew);
            ps += pv[i];
        }
        ps += __shfl_xor(ps, 16);
        ps += __shfl_xor(ps, 32);
        l_run = l_run * alpha + ps;
        m_run = mnew;
        float al[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) al[j] = __shfl(alpha, 4 * g + j);
        u32x4 vt[ND];
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
            vt[dt] = *reinterpret_cast<const u32x4 *>(vs + (dt * 16 + n) * VROW + 16 * g);
        if (k0 + 32 > kend) {
            // slots past the wave's last key hold nothing of this chunk yet
#pragma unroll
            for (int dt = 0; dt < ND; ++dt)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const int key = k0 + 8 * g + 2 * w;
                    uint32_t x = vt[dt][w];
                    if (key >= kend) x &= 0xffff0000u;
                    if (key + 1 >= kend) x &= 0x0000ffffu;
                    vt[dt][w] = x;
                }
        }
        bf16x8 ph, pl;
        split_hi_lo(make_float4(pv[0], pv[1], pv[2], pv[3]), make_float4(pv[4], pv[5], pv[6], pv[7]), ph, pl);
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) {
#pragma unroll
            for (int j = 0; j < 4; ++j) o[dt][j] *= al[j];
            const bf16x8 v8 = __builtin_bit_cast(bf16x8, vt[dt]);
            o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph, v8, o[dt], 0, 0, 0);
            o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl, v8, o[dt], 0, 0, 0);
        }
    };
    fetch(min(kg, ntile - 1));  // (a group past the last tile repeats it, unused)
    stash(0);
    __syncthreads();
    for (int t0 = 0; t0 < ntile; t0 += NKG) {
        const int t = t0 + kg, buf = (t0 / NKG) & 1;
        const bool more = t0 + NKG < ntile;
        if (more) fetch(min(t + NKG, ntile - 1));  // in flight while tile t is used
        if (t < wtiles) process(t, buf);
        if (more) stash(buf ^ 1);
        __syncthreads();
    }
    if constexpr (NKG > 1) {
        // groups 1.. leave their outputs in LDS, group 0 combines them
        float *const so = reinterpret_cast<float *>(smem_all);
        if (g == 0) {
            sm_m[kg][16 * wave + n] = m_run;
            sm_l[kg][16 * wave + n] = l_run;
        }
        if (kg > 0) {
#pragma unroll
            for (int dt = 0; dt < ND; ++dt)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    so[((kg - 1) * 64 + 16 * wave + 4 * g + j) * OROW + dt * 16 + n] = o[dt][j];
        }
        __syncthreads();
        if (kg > 0) return;
        float mx = -INFINITY, l = 0.f;
#pragma unroll
        for (int q = 0; q < NKG; ++q) mx = fmaxf(mx, sm_m[q][16 * wave + n]);
        float wq[NKG];
#pragma unroll
        for (int q = 0; q < NKG; ++q) {
            const float mq = sm_m[q][16 * wave + n];
            wq[q] = mq == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mq - mx);
            l = fmaf(wq[q], sm_l[q][16 * wave + n], l);
        }
        l_run = l;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float wj[NKG];
#pragma unroll
            for (int q = 0; q < NKG; ++q) wj[q] = __shfl(wq[q], 4 * g + j);
#pragma unroll
            for (int dt = 0; dt < ND; ++dt) {
                float v = o[dt][j] * wj[0];
#pragma unroll
                for (int q = 1; q < NKG; ++q)
                    v = fmaf(wj[q], so[((q - 1) * 64 + 16 * wave + 4 * g + j) * OROW + dt * 16 + n], v);
                o[dt][j] = v;
            }
        }
    }
    if (!active) return;
    // rows of o are queries qb + 4g + j; their sums l sit in lanes 4g + j
    float lr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) lr[j] = __shfl(l_run, 4 * g + j);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int i = qb + 4 * g + j;
        if (i >= M) continue;
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) store_split(out, i, h * HD + dt * 16 + n, MT, o[dt][j] / lr[j]);
    }
}

// ---------------------------------------------------------------------------
// launchers

hipError_t launch_pf_embed(const int32_t *tokens, const void *embed, int M, int Mp, int d, const void *gain, float *x,
                           uint16_t *us, float *ssq, hipStream_t s)
{
    if (d % 64 || Mp % 16 || M < 1 || M > Mp) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_pf_embed, dim3(Mp), dim3(PF_THREADS), 0, s, tokens, static_cast<const uint16_t *>(embed), M, d,
                       Mp / 16, static_cast<const uint16_t *>(gain), x, us, ssq);
    return hipGetLastError();
}

namespace {

// Workgroup shapes: rows per unit and K groups; a shape's steps in flight are
// what its registers hold (8 waves of 256 VGPRs; only int8 QKV at 256 rows and 8
// tiles spills, two address registers reloaded per step).
constexpr int SHAPE_NWR[3] = {8, 4, 2};
constexpr int PF_TT_MIN = 4, PF_TT_MAX = 8, PF_KS_MAX = 8;

template <int SHAPE, int TT, bool Q8> constexpr int pf_lead()
{
    if (Q8) return 2;
    return SHAPE == 0 ? 4 : (SHAPE == 1 ? (TT <= 6 ? 4 : 3) : (TT <= 5 ? 3 : 2));
}

template <int EPI, int SHAPE, int TT, bool Q8>
hipError_t pf_launch(const PfArgs &a, hipStream_t s)
{
    constexpr int NWR = SHAPE_NWR[SHAPE];
    const int n_units = (a.NB + 4 * NWR - 1) / (4 * NWR) * a.ks * a.n_tt;
    // 1-D grid: 8 chunks of ceil(units / 8)
    hipLaunchKernelGGL((k_pf_gemm<EPI, NWR, 8 / NWR, TT, pf_lead<SHAPE, TT, Q8>(), Q8>), dim3(8 * ((n_units + 7) / 8)),
                       dim3(512), 0, s, a);
    return hipGetLastError();
}

template <int EPI, int SHAPE, bool Q8>
hipError_t pf_launch_tt(const PfArgs &a, int tt, hipStream_t s)
{
    switch (tt) {
    case 4: return pf_launch<EPI, SHAPE, 4, Q8>(a, s);
    case 5: return pf_launch<EPI, SHAPE, 5, Q8>(a, s);
    case 6: return pf_launch<EPI, SHAPE, 6, Q8>(a, s);
    case 7: return pf_launch<EPI, SHAPE, 7, Q8>(a, s);
    case 8: return pf_launch<EPI, SHAPE, 8, Q8>(a, s);
    default: return hipErrorInvalidValue;
    }
}

template <int EPI>
hipError_t pf_launch_epi(const PfArgs &a, int shape, int tt, hipStream_t s)
{
    if (a.scale) {
        if (shape == 0) return pf_launch_tt<EPI, 0, true>(a, tt, s);
        if (shape == 1) return pf_launch_tt<EPI, 1, true>(a, tt, s);
        return hipErrorInvalidValue;
    }
    if (shape == 0) return pf_launch_tt<EPI, 0, false>(a, tt, s);
    if (shape == 1) return pf_launch_tt<EPI, 1, false>(a, tt, s);
    if (shape == 2) return pf_launch_tt<EPI, 2, false>(a, tt, s);
    return hipErrorInvalidValue;
}

}  // namespace

// The cut with the least estimated time.  A unit takes c + (steps per K group)
// (a + b tiles) us, with one unit per CU at a time; split K adds e us, f us
// per KB of partials the folding unit reads and g us per MB that all units
// write.  Small row counts and short prompts need K ranges or K groups to reach
// every CU; large ones lose to them by the partials' traffic.  The constants
// are a fit to 2900 launches on random data at (d_model, d_ffn) = (4096,
// 11008) and (5120, 13824), 5 to 64 token tiles, every cut: the chosen one is
// 1% slower than the fastest on average, 6% at most.  At widths it was not fitted to
// (1024, 2048, 3072, 8192; 3 to 64 tiles; event-timed launches, every cut) it is 2-4%
// behind on average in bf16 and 0.4-7% in int8: small matrices get too few K
// ranges (worst: int8 gate/up at 2048 x 5504, 48 tokens, 30 us, with 4 ranges 21).
// Before, 512 x
// 128 (QKV, gate/up) and 512 x 48 tiles (O, down) ran over all of K, with the
// B operands read just before use.  160 tokens, 7B width, us: QKV 168 -> 50,
// O 84 -> 30, gate/up 170 -> 75, down 206 -> 49 (38 and 57 for O and down while
// one K group's waves did all sums, folds and epilogues); 1024 tokens, 13B width,
// inside the model: 248 -> 245, 125 -> 116, 473 -> 454, 302 -> 255.
PfPlan pf_plan(int NB, int MT, int K, bool q8, int n_cu)
{
    struct Fit {
        double a, b, c;
    };
    static const Fit fit[2][3] = {{{0.236, 0.126, 5.5}, {0.265, 0.147, 6.1}, {0.389, 0.170, 6.8}},
                                  {{0.492, 0.271, 3.2}, {0.365, 0.334, 3.2}, {0, 0, 0}}};
    const double e = q8 ? 10.3 : 7.7, f = q8 ? 0.017 : 0.018, g = q8 ? 0.26 : 0.33;
    // Where every CU is kept busy the chip's power sets the rate, not the cut:
    // 27648 x 5120 at 1024 tokens takes 424 us as 432 units (84% of two rounds)
    // and 434-466 us as 486 (95%).  Cuts below that time count as equal and the
    // first, with the fewest units, is taken.
    const double power_us = 2.35e-5 * NB * MT * (K / 32);
    const int n_min = (MT + PF_TT_MAX - 1) / PF_TT_MAX;
    // (a shape every size can take; the loops below replace it)
    PfPlan best{1, std::max((MT + n_min - 1) / n_min, PF_TT_MIN), n_min, 1};
    double best_us = 1e30;
    const int S = K / (q8 ? 64 : 32);
    for (int shape = 0; shape < (q8 ? 2 : 3); ++shape) {
        const int nwr = SHAPE_NWR[shape], nkg = 8 / nwr, n_rt = (NB + 4 * nwr - 1) / (4 * nwr);
        for (int n_tt = n_min; n_tt <= std::max(MT / PF_TT_MIN, n_min); ++n_tt) {
            const int tt = std::max((MT + n_tt - 1) / n_tt, PF_TT_MIN);
            for (int ks = 1; ks <= PF_KS_MAX && ks * nkg <= S; ++ks) {
                const long units = (long)n_rt * n_tt * ks;
                if (ks > 1 && units * nwr * 4 * tt > DV_PF_PART_TILES) break;
                const long rounds = (units + n_cu - 1) / n_cu;
                const int steps = ((S + ks - 1) / ks + nkg - 1) / nkg;
                const Fit &t = fit[q8 ? 1 : 0][shape];
                double us = (double)rounds * (steps * (t.a + t.b * MT / n_tt) + t.c);
                const double part_kb = 4.0 * nwr * tt;
                if (ks > 1) us += e + f * ks * part_kb + g * units * part_kb * 1e-3;
                us = std::max(us, power_us);
                if (us < best_us) {
                    best_us = us;
                    best = PfPlan{shape, tt, n_tt, ks};
                }
            }
        }
    }
    return best;
}

int pf_part_tiles(int NB, const PfPlan &p)
{
    const int rows = 4 * SHAPE_NWR[p.shape];  // blocks of a unit
    return p.ks > 1 ? (NB + rows - 1) / rows * p.n_tt * p.ks * rows * p.tt : 0;
}

hipError_t launch_pf_gemm(const PfArgs &a, const PfPlan &p, int epi, hipStream_t s)
{
    if (a.K % (a.scale ? 64 : 32) || a.NB < 1 || a.MT < 1 || a.d % 64 || a.M < 1 || a.M > 16 * a.MT || a.n_tt != p.n_tt ||
        a.ks != p.ks || p.tt != std::max((a.MT + a.n_tt - 1) / a.n_tt, PF_TT_MIN) || (a.ks > 1 && (!a.part || !a.cnt)))
        return hipErrorInvalidValue;
    if (epi == EPI_RESID) return pf_launch_epi<EPI_RESID>(a, p.shape, p.tt, s);
    if (epi == EPI_QKV) {
        if (a.hd != 64 && a.hd != 128) return hipErrorInvalidValue;
        return pf_launch_epi<EPI_QKV>(a, p.shape, p.tt, s);
    }
    if (epi == EPI_SWIGLU) return pf_launch_epi<EPI_SWIGLU>(a, p.shape, p.tt, s);
    if (epi == EPI_LOGITS) {
        if (p.shape != PF_STEP_PLAN.shape || p.tt != PF_STEP_PLAN.tt || a.scale || !a.arg_val || !a.arg_idx)
            return hipErrorInvalidValue;
        return pf_launch<EPI_LOGITS, PF_STEP_PLAN.shape, PF_STEP_PLAN.tt, false>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int HD>
static hipError_t causal_launch(int nkg, const float *q, const void *kc, const void *vc, int M, int P0, int H, int cap,
                                int MT, uint16_t *out, hipStream_t s)
{
    const dim3 grid(H, (M + 63) / 64);
    const uint16_t *k16 = static_cast<const uint16_t *>(kc), *v16 = static_cast<const uint16_t *>(vc);
    if (nkg == 2) hipLaunchKernelGGL((k_attn_causal<HD, 2>), grid, dim3(512), 0, s, q, k16, v16, M, P0, H, cap, MT, out);
    else hipLaunchKernelGGL((k_attn_causal<HD, 1>), grid, dim3(256), 0, s, q, k16, v16, M, P0, H, cap, MT, out);
    return hipGetLastError();
}

hipError_t launch_attn_causal(const float *q, const void *kc, const void *vc, int M, int P0, int H, int hd, int cap,
                              int MT, int n_cu, uint16_t *out, hipStream_t s)
{
    const int nkg = causal_key_groups(M, P0, H, n_cu);
    if (hd == 128) return causal_launch<128>(nkg, q, kc, vc, M, P0, H, cap, MT, out, s);
    if (hd == 64) return causal_launch<64>(nkg, q, kc, vc, M, P0, H, cap, MT, out, s);
    return hipErrorInvalidValue;
}
