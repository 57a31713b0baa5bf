// Dense projections of the target forward (Alg. 1 Step 3): C = A[M,K] W[N,K]^T.
//
// bf16 path: LDS-staged tiles feeding v_mfma_f32_32x32x16_bf16 (64-lane
// wavefronts; both operands are K-contiguous so every lane fetches its 8-element
// fragment with one 16-byte LDS read), float32 accumulation.  The MFMA operands
// are exchanged (weight rows feed the MFMA rows, tokens run over the lanes) and
// the weight rows are fetched with bits 2-3 of the row index swapped, so a lane
// ends up owning one token and runs of 8 consecutive output columns: every
// epilogue reads and writes 16-byte pieces.  Fused epilogues:
//   Q|K|V  -> rotary on the adjacent pairs of a run (float4 table reads) + q buffer / K cache rows; V: the 32 lanes of
//             a half are 32 consecutive tokens = 64 contiguous bytes of a row of the transposed V cache
//   out, down -> residual add into the float32 stream
//   gate|up   -> silu(gate) * up, gate and up columns interleaved inside a tile so
//                that one lane owns both accumulators of a feed-forward column
//   lm-head   -> float32 logits
#include <hip/hip_bf16.h>

#include <utility>

#include "mulo_internal.h"
#include "row_parts.h"

namespace mulo {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __hip_bfloat16 bf16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_LOGITS = 3 };

struct GemmArgs {
    const bf16* A;        // [M, K]
    const bf16* W0;       // QK: wq | SWIGLU: w_gate | else: W [N, K]
    const bf16* W1;       // QK: wk | SWIGLU: w_up
    const bf16* W2;       // QKV: wv
    int M, N, K;          // N: output columns of the fused problem (QK: 2d, SWIGLU: 2f)
    float* Cf;            // RESID: x [M, N] (+=) | LOGITS: logits [M, N]
    bf16* Cb;             // SWIGLU: h [M, N/2] | QK: q buffer
    bf16* kc;             // QK: K cache
    bf16* vc;             // V: V^T cache
    int d;                // QK: model width (segment size)
    int tiles_n;          // column tiles of the launch (set by the launcher)
    int tile_n0;          // first column tile of the launch (set by the launcher)
    float2* parts;        // LOGITS: softmax statistics per 128-column part of every row [M, n_parts], or nullptr
    int n_parts;
    bool stream;          // A is in fragment order: the launch runs in the weight-streaming kernels
    bool w_frag;          // weight-streaming launches: W0 .. W2 point at copies in fragment order
    float* ksums;         // k_gemv_shared: sums of the K slices [ksplit, M, columns]
    int64_t ksum_floats;  // what ksums holds
    int ksplit;           // set by the launcher
    RopeArgs ra;
};


// compile-time loop: the body sees its index as a constant, so accumulator arrays
// indexed by it stay in registers whatever the unroller decides
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

// g * sigmoid(g) with the hardware reciprocal (1 ulp; the product is rounded to bf16 right after)
__device__ __forceinline__ float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// Rotary on an adjacent pair, in one order of fused operations: left to the compiler, which product of the second it rounds first
// differed between instantiations (and with it the last bit of some keys, between 32 and 64 streamed tokens)
__device__ __forceinline__ float rotate0(float x0, float x1, float cs, float sn) { return fmaf(x0, cs, -__fmul_rn(x1, sn)); }
__device__ __forceinline__ float rotate1(float x0, float x1, float cs, float sn) { return fmaf(x1, cs, __fmul_rn(x0, sn)); }

// Source of weight-tile row nl (fixed over the K loop) for each fused problem: row index, and which of the
// two weight matrices (0: W0, 1: W1) it belongs to.
template <int EPI, int BN, int TN>
__device__ __forceinline__ int b_row_src(const GemmArgs& g, int n0, int tile_n, int nl, int& which) {
    int r;
    if constexpr (EPI == EPI_QKV) {
        const int seg = n0 / g.d;
        which = seg;
        r = n0 - seg * g.d + nl;
    } else if constexpr (EPI == EPI_SWIGLU) {
        // tile covers feed-forward columns [f0, f0 + BN/2); the wavefront owning tile columns
        // [w TN, (w+1) TN) gets TN/2 of them: gate rows in its first half, up rows in the second
        const int f = g.N / 2, f0 = tile_n * (BN / 2);
        const int w_ = nl / TN, within = nl % TN;
        r = f0 + w_ * (TN / 2) + (within % (TN / 2));
        r = r < f ? r : f - 1;
        which = within >= TN / 2 ? 1 : 0;
    } else {
        which = 0;
        r = n0 + nl;
        r = r < g.N ? r : g.N - 1;
    }
    return r;
}

// The tiled kernels address their operands through buffer descriptors: the descriptor (base and size) and a byte offset
// live in scalar registers, a lane adds a 32-bit offset of its own.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)(bytes < 0x7fffffff ? bytes : 0x7fffffff), 0x00020000);
}
__device__ __forceinline__ u32x4 bload(rsrc_t r, uint32_t lane_off, uint32_t base_off) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)base_off, 0);
}
// Which tile row feeds MFMA row rho: bits 2 and 3 exchanged.  With it, accumulator r of a lane
// covers, along the MFMA row axis, index 16*(r/8) + 8*lh + r%8: two runs of 8 consecutive indices
// per 32x32 block, so every lane stores 16-byte (bf16) or 2 x 16-byte (float) pieces.
__device__ __forceinline__ int kperm(int l32) { return (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1); }

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8s;

// Fused epilogues.  acc[i][j] is the 32x32 block (i, j) of the wavefront's TM x TN tile whose corner
// is (m0 + wm TM, n0 + wn TN).  The MFMA operands are exchanged, so a lane owns ONE token row
// (m = ... + l32) and, per block, the column runs [16 g + 8 lh, +8), g = 0, 1 (accumulators 8 g .. 8 g + 7).
// Where token row m of a projection lives: b, jj index the q buffer [B, nh, L, dh]; bc is its cache sequence and pos
// its cache row (< 0: an unused slot of a scattered launch, nothing of it is written).
struct TokPlace { int b, jj, bc, pos; };
__device__ __forceinline__ TokPlace place(const RopeArgs& ra, int m) {
    const int b = m / ra.L, jj = m % ra.L;
    if (ra.pos_tab) return {b, jj, b, ra.pos_tab[m]};   // scattered queries: slot jj of sequence b (L slots each)
    return {b, jj, b, ra.P + jj};
}

// Softmax statistics of the wavefront tile's 128 columns, per token, for the accept test (Sec. 3.1, Eq. 1): this lane holds
// half lh of part (tile_n, wn) of token row m, run rr = 2 j + g2 in accumulators 8 g2 .. 8 g2 + 7 of block j; the other half
// sits in lane + 32.  Whole tiles only (every column exists).
template <int BN, int TM, int MB, int NB>
__device__ __forceinline__ void logit_parts(const GemmArgs& g, const f32x16 (&acc)[MB][NB], int m0, int tile_n, int wm, int wn,
                                            int l32, int lh) {
    static_for<MB>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const int m = m0 + wm * TM + i * 32 + l32;
        float mx = rowparts::NEG_INF;
        static_for<NB>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc[i][j][r]);
        });
        float t[8];
        static_for<NB>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
#pragma unroll
            for (int g2 = 0; g2 < 2; ++g2) {
                float zz[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) zz[e] = acc[i][j][g2 * 8 + e];
                t[j * 2 + g2] = rowparts::run_sum(zz, mx, 8);
            }
        });
        const float sm = rowparts::tree8(t);
        const float2 ps = rowparts::merge_halves(mx, sm, __shfl_xor(mx, 32), __shfl_xor(sm, 32));
        if (lh == 0 && m < g.M) g.parts[(int64_t)m * g.n_parts + tile_n * (BN / rowparts::PART) + wn] = ps;
    });
}

template <int EPI, int BN, int TM, int TN, int MB, int NB>
__device__ __forceinline__ void epilogue(const GemmArgs& g, f32x16 (&acc)[MB][NB], int m0, int n0, int tile_n,
                                         int wm, int wn, int l32, int lh) {
    constexpr int NBE = EPI == EPI_SWIGLU ? NB / 2 : NB;   // gate blocks only: up blocks are consumed with them
    if constexpr (EPI == EPI_RESID) {
        // x += acc.  The compiler cannot tell the stream's loads from its stores, so a plain read-add-write per
        // run is a chain of MB * NB * 2 memory round trips per lane (about a microsecond each: the whole
        // epilogue of a launch with one tile per CU).  All runs of one block row are requested first, then
        // added and written: two round trips per lane.
        static_for<MB>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const int m = m0 + wm * TM + i * 32 + l32;
            if (m < g.M) {
                float* const row = g.Cf + (int64_t)m * g.N + n0 + wn * TN + lh * 8;
                const int nrow = n0 + wn * TN + lh * 8;
                f32x4 r[NB][2][2];
                static_for<NB>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
#pragma unroll
                    for (int g2 = 0; g2 < 2; ++g2) {
                        const int cl = j * 32 + g2 * 16;
                        if (nrow + cl + 8 <= g.N) {
                            r[j][g2][0] = *reinterpret_cast<const f32x4*>(row + cl);
                            r[j][g2][1] = *reinterpret_cast<const f32x4*>(row + cl + 4);
                        }
                    }
                });
                static_for<NB>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
#pragma unroll
                    for (int g2 = 0; g2 < 2; ++g2) {
                        const int cl = j * 32 + g2 * 16;
                        if (nrow + cl + 8 <= g.N) {
                            f32x4 lo, hi;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                lo[e] = r[j][g2][0][e] + acc[i][j][g2 * 8 + e];
                                hi[e] = r[j][g2][1][e] + acc[i][j][g2 * 8 + 4 + e];
                            }
                            *reinterpret_cast<f32x4*>(row + cl) = lo;
                            *reinterpret_cast<f32x4*>(row + cl + 4) = hi;
                        } else {
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                if (nrow + cl + e < g.N) row[cl + e] += acc[i][j][g2 * 8 + e];
                        }
                    }
                });
            }
        });
        return;
    }
    if constexpr (EPI == EPI_LOGITS && TN == rowparts::PART) {
        if (g.parts) logit_parts<BN, TM, MB, NB>(g, acc, m0, tile_n, wm, wn, l32, lh);
    }
    static_for<MB>([&](auto ic) {
        static_for<NBE>([&](auto jc) {
            constexpr int i = decltype(ic)::value, j = decltype(jc)::value;
#pragma unroll
            for (int g2 = 0; g2 < 2; ++g2) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = acc[i][j][g2 * 8 + e];
                const int m = m0 + wm * TM + i * 32 + l32;                       // token row of this lane
                const int cl = j * 32 + g2 * 16 + lh * 8;                        // column run inside the wave tile
                if (m < g.M) {
                    if constexpr (EPI == EPI_RESID || EPI == EPI_LOGITS) {
                        const int n = n0 + wn * TN + cl;
                        float* dst = g.Cf + (int64_t)m * g.N + n;
                        if (n + 8 <= g.N) {
                            f32x4 lo = {v[0], v[1], v[2], v[3]}, hi = {v[4], v[5], v[6], v[7]};
                            if constexpr (EPI == EPI_RESID) {
                                lo += *reinterpret_cast<const f32x4*>(dst);
                                hi += *reinterpret_cast<const f32x4*>(dst + 4);
                            }
                            *reinterpret_cast<f32x4*>(dst) = lo;
                            *reinterpret_cast<f32x4*>(dst + 4) = hi;
                        } else {
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                if (n + e < g.N) dst[e] = EPI == EPI_RESID ? dst[e] + v[e] : v[e];
                        }
                    } else if constexpr (EPI == EPI_SWIGLU) {
                        const int f = g.N / 2;
                        const int n = tile_n * (BN / 2) + wn * (TN / 2) + cl;
                        bf16* dst = g.Cb + (int64_t)m * f + n;
                        float h[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) h[e] = silu(v[e]) * acc[i][j + NB / 2][g2 * 8 + e];
                        if (n + 8 <= f) {
                            bf16x8s o;
#pragma unroll
                            for (int e = 0; e < 8; ++e) o[e] = (__bf16)h[e];
                            *reinterpret_cast<bf16x8s*>(dst) = o;
                        } else {
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                if (n + e < f) dst[e] = __float2bfloat16(h[e]);
                        }
                    } else {  // EPI_QKV: rotary on the 4 adjacent pairs of the run, q -> [B, nh, L, dh], k -> cache row
                        const int n = n0 + wn * TN + cl, seg = n / g.d, c = n - seg * g.d;
                        const int dh = g.ra.head_dim, hd = c / dh, cc = c % dh;
                        const TokPlace pl = place(g.ra, m);
                        if (seg == 2) {
                            // a lane holds 8 consecutive channels of ONE token, the 32 lanes of a half are 32
                            // consecutive tokens = 64 contiguous bytes of a row of the transposed cache per store
                            if (pl.pos >= 0) {
                                const int64_t hb = ((int64_t)g.ra.layer * g.ra.max_batch + pl.bc) * g.ra.n_heads + hd;
#pragma unroll
                                for (int e = 0; e < 8; ++e)
                                    g.vc[(hb * dh + cc + e) * g.ra.max_seq + pl.pos] = __float2bfloat16(v[e]);
                            }
                        } else if (pl.pos >= 0) {
                            const int pos = pl.pos;
                            const f32x4 cs = *reinterpret_cast<const f32x4*>(g.ra.cos + (int64_t)pos * (dh / 2) + (cc >> 1));
                            const f32x4 sn = *reinterpret_cast<const f32x4*>(g.ra.sin + (int64_t)pos * (dh / 2) + (cc >> 1));
                            bf16x8s o;
#pragma unroll
                            for (int pr = 0; pr < 4; ++pr) {
                                o[2 * pr] = (__bf16)rotate0(v[2 * pr], v[2 * pr + 1], cs[pr], sn[pr]);
                                o[2 * pr + 1] = (__bf16)rotate1(v[2 * pr], v[2 * pr + 1], cs[pr], sn[pr]);
                            }
                            bf16* dst;
                            if (seg == 0) {
                                dst = g.Cb + (((int64_t)pl.b * g.ra.n_heads + hd) * g.ra.L + pl.jj) * dh + cc;
                            } else {
                                const int64_t hb = ((int64_t)g.ra.layer * g.ra.max_batch + pl.bc) * g.ra.n_heads + hd;
                                dst = g.kc + (hb * g.ra.max_seq + pos) * dh + cc;
                            }
                            *reinterpret_cast<bf16x8s*>(dst) = o;
                        }
                    }
                }
            }
        });
    });
}

// D[n][m]: MFMA rows = weight rows (output columns), lanes = tokens
__device__ __forceinline__ f32x16 mma(const bf16x8& a, const bf16x8& b, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, c, 0, 0, 0);
}

// ---- 256 x 256 tiles: 4 wavefronts of 128 x 128 (one per SIMD) over an LDS ring of five 32 KB items ---------------
// For launches whose tiles fill the chip.  What bounds them is energy: the matrix pipes are busy in 71 to 80 % of the cycles, but
// the shader clock sinks to 1.66 - 1.75 GHz under this load (counters at 4096 tokens; on weights that are all alike the same
// launches of 16384 tokens take 77 to 81 % of the time), so what helps is fewer bytes moved per product and no phases in which
// the matrix pipes rest.
//   - A wavefront owns 128 x 128 outputs (all 256 accumulators of a SIMD lane's second register half), 16 MFMAs per 8 KB of
//     fragments: a 64-deep step reads 128 KB of LDS where 8 wavefronts of 64 x 128 read 192.
//   - Operands go from memory to LDS directly (no staging registers, no ds_write).  An item is 256 rows x 128 bytes of one
//     operand; items alternate W(0) A(0) W(1) A(1) ..., step kt reads two of the five slots, and loads A(kt + 1) and then
//     W(kt + 2) into the two that step kt - 1 has read: a wavefront waits for its loads one step (tokens, out of the L2) or
//     one and a half (weights) after their request, and meets the others once a step.  Chunk c of row r sits at chunk
//     position c ^ ((r / 2) % 8): no bank conflicts.
//   - With one wavefront per SIMD nothing else issues while an instruction waits, so every fragment read, load and scalar
//     update has its place between two MFMAs of the slice before (sched_barrier; left to itself the scheduler collects the
//     loads behind all MFMAs: +12 % time).  The k deal, hence every sum, is k_gemm_ring's.
//   - Persistent: one workgroup per CU walks its tiles; the last two steps of a tile load the next one's first (past the last
//     tile the descriptors are empty, which costs no traffic).
//   - Epilogues go through LDS (the two slots that are free then) so that every access is whole rows, and the residual
//     stream's first half is requested before the K loop.  q|k|v tiles of V exchange the operands' roles in the K loop.
// us per launch, 8 wavefronts staged through registers -> here, cold weights, 4096 tokens: 4096 x 4096 147 -> 115,
// 4096 x 11008 297 -> 267, q|k|v 334 -> 307, gate|up 572 -> 507, lm-head 439 -> 421.
constexpr int LDS_256 = 5 * 256 * 128;
constexpr int ER = 272;   // bytes of a row of the epilogues' LDS block: 256 and 16 more (conflicts in at most 0.8 % of a launch's cycles)

// The float32 output rows of a tile: a descriptor (rows past M lie outside: reads give zeros, writes nothing), this lane's
// offset, and what access t (4 rows of 64 columns) of block h (32 rows x 64 columns) adds to it.
__device__ __forceinline__ rsrc_t c_rsrc(const GemmArgs& g, int m0) {
    const int left = g.M - m0;
    return make_rsrc(g.Cf + (int64_t)m0 * g.N, (int64_t)(left < 256 ? left : 256) * g.N * 4);
}
__device__ __forceinline__ uint32_t c_off(const GemmArgs& g, int n0, int wm, int wn, int lane) {
    return (uint32_t)((wm * 128 + (lane >> 4)) * g.N + n0 + wn * 128 + (lane & 15) * 4) * 4u;
}
__device__ __forceinline__ uint32_t c_step(const GemmArgs& g, int h, int t) {
    return (uint32_t)((h >> 1) * 32 + t * 4) * (uint32_t)g.N * 4u + (h & 1) * 256u;
}

// block h of a wavefront's 128 x 128 accumulators to LDS, a row of 64 columns per token
template <int H>
__device__ __forceinline__ void put_block(const f32x16 (&acc)[4][4], unsigned char* lds, int l32, int lh) {
    static_for<2>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const f32x16& a = acc[H >> 1][(H & 1) * 2 + j];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4*>(lds + l32 * ER + lh * 32 + j * 128 + (q >> 1) * 64 + (q & 1) * 16) =
                f32x4{a[q * 4], a[q * 4 + 1], a[q * 4 + 2], a[q * 4 + 3]};
    });
}

// residual add, logits.  xv: the first XAHEAD blocks of the stream
constexpr int XAHEAD = 4;
template <int EPI, int XN>
__device__ __forceinline__ void epilogue_c(const GemmArgs& g, const f32x16 (&acc)[4][4], f32x4 (&xv)[XN][8], int m0, int n0, int wm,
                                           int wn, int lane, unsigned char* lds) {
    const rsrc_t rc = c_rsrc(g, m0);
    const uint32_t vo = c_off(g, n0, wm, wn, lane);
    unsigned char* const rd = lds + (lane >> 4) * ER + (lane & 15) * 16;
    static_for<8>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        put_block<h>(acc, lds, lane & 31, lane >> 5);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            f32x4 v = *reinterpret_cast<const f32x4*>(rd + t * 4 * ER);
            if constexpr (EPI == EPI_RESID) v = xv[h % XN][t] + v;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rc, (int)(vo + c_step(g, h, t)), 0, 0);
        }
        if constexpr (EPI == EPI_RESID && h + XN < 8) {
#pragma unroll
            for (int t = 0; t < 8; ++t) xv[h % XN][t] = __builtin_bit_cast(f32x4, bload(rc, vo + c_step(g, h + XN, t), 0));
        }
    });
}

// silu(gate) * up: blocks j of a row are gate columns, j + 2 the up columns of the same 32 feed-forward columns
__device__ __forceinline__ void epilogue_h(const GemmArgs& g, const f32x16 (&acc)[4][4], int m0, int tile_n, int wm, int wn, int lane,
                                           unsigned char* lds) {
    constexpr int HR = 144;   // 64 columns of bf16 and 16 bytes more
    const int f = g.N / 2, left = g.M - m0;
    const rsrc_t rc = make_rsrc(g.Cb + (int64_t)m0 * f, (int64_t)(left < 256 ? left : 256) * f * 2);
    const uint32_t vo = (uint32_t)((wm * 128 + (lane >> 3)) * f + tile_n * 128 + wn * 64 + (lane & 7) * 8) * 2u;
    unsigned char* const wr = lds + (lane & 31) * HR + (lane >> 5) * 16;
    unsigned char* const rd = lds + (lane >> 3) * HR + (lane & 7) * 16;
    static_for<4>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        static_for<2>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
#pragma unroll
            for (int g2 = 0; g2 < 2; ++g2) {
                bf16x8s o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (__bf16)(silu(acc[i][j][g2 * 8 + e]) * acc[i][j + 2][g2 * 8 + e]);
                *reinterpret_cast<bf16x8s*>(wr + j * 64 + g2 * 32) = o;
            }
        });
#pragma unroll
        for (int t = 0; t < 4; ++t)
            __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(rd + t * 8 * HR), rc,
                                                   (int)(vo + (uint32_t)(i * 32 + t * 8) * (uint32_t)f * 2u), 0, 0);
    });
}

// q | k | v.  Every block of 32 rows x 64 columns goes through LDS as it is, whatever the tile is of, and only what a lane does with
// the 8 values it reads back differs; where the 128 tokens live is worked out once, two tokens a lane, and kept behind the block.
// (With an epilogue of its own per kind of tile, hence the accumulators in two branches, the kernel kept 65 registers in scratch
// memory, which the runtime allocates at the first dispatch: 4096 tokens of width 4096 325 us, so 315.)
//   q, k   a row is a token: rotary, then 8 channels of its row of the q buffer or the K cache.  The table rows of a block are
//          requested a block ahead.
//   V      operands exchanged: a row is a channel (wm: 128 channels), the columns are tokens (wn: 128 tokens): 8 tokens go to
//          the channel's row of the transposed cache, 128 contiguous bytes per 8 lanes.  A run that does not lie in 8 consecutive
//          cache columns (the end of a sequence, scattered slots, past M) goes token by token.  The address of a run is a
//          multiple of 2 bytes only: its cache row is the caller's P + j.
__device__ __forceinline__ void epilogue_qkv(const GemmArgs& g, const f32x16 (&acc)[4][4], bool v_tile, int m0, int n0, int wm, int wn,
                                             int lane, unsigned char* lds) {
    const int dh = g.ra.head_dim, hsh = dh == 128 ? 7 : 6, mw = m0 + (v_tile ? wn : wm) * 128, nw = n0 + (v_tile ? wm : wn) * 128;
    const int seg = nw / g.d;
    // cache row (< 0: nothing is written); rows in front of the token's own in its buffer, head 0 (a cache that fits has fewer than
    // 2^32): of d_h channels for q and k, of max_seq columns for V
    struct Row { int pos; uint32_t row; };
    Row* const tab = reinterpret_cast<Row*>(lds + 32 * ER);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = mw + i * 64 + lane;
        const TokPlace pl = place(g.ra, m < g.M ? m : g.M - 1);
        tab[i * 64 + lane] = {m < g.M ? pl.pos : -1, seg == 0   ? (uint32_t)pl.b * g.ra.n_heads * g.ra.L + pl.jj
                                                     : seg == 1 ? (uint32_t)pl.bc * g.ra.n_heads * g.ra.max_seq + pl.pos
                                                                : (uint32_t)pl.bc * g.d};
    }
    const int rows = seg == 0 ? g.ra.L : g.ra.max_seq, cl = nw - seg * g.d + (lane & 7) * 8;
    const int64_t layer_elems = (int64_t)g.ra.max_batch * g.d * g.ra.max_seq;
    bf16* const base = seg == 0 ? g.Cb : (seg == 1 ? g.kc : g.vc) + g.ra.layer * layer_elems;
    unsigned char* const rd = lds + (lane >> 3) * ER + (lane & 7) * 32;
    f32x4 cs[2][4], sn[2][4];
    Row rw[2][4];
    auto fetch = [&](auto hc) {   // table rows of block h
        constexpr int h = decltype(hc)::value;
        const int cc = (cl + (h & 1) * 64) & (dh - 1);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            rw[h & 1][t] = tab[(h >> 1) * 32 + t * 8 + (lane >> 3)];
            const int pos = rw[h & 1][t].pos < 0 ? 0 : rw[h & 1][t].pos;
            cs[h & 1][t] = *reinterpret_cast<const f32x4*>(g.ra.cos + (int64_t)pos * (dh / 2) + (cc >> 1));
            sn[h & 1][t] = *reinterpret_cast<const f32x4*>(g.ra.sin + (int64_t)pos * (dh / 2) + (cc >> 1));
        }
    };
    if (!v_tile) fetch(std::integral_constant<int, 0>{});
    static_for<8>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        if constexpr (h < 7) {
            if (!v_tile) fetch(std::integral_constant<int, h + 1>{});
        }
        put_block<h>(acc, lds, lane & 31, lane >> 5);
        f32x4 lo[4], hi[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            lo[t] = *reinterpret_cast<const f32x4*>(rd + t * 8 * ER);
            hi[t] = *reinterpret_cast<const f32x4*>(rd + t * 8 * ER + 16);
        }
        if (!v_tile) {
            const int c = cl + (h & 1) * 64;
            bf16* const dst = base + (int64_t)(c >> hsh) * rows * dh + (c & (dh - 1));
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float v[8] = {lo[t][0], lo[t][1], lo[t][2], lo[t][3], hi[t][0], hi[t][1], hi[t][2], hi[t][3]};
                const f32x4 &cs_ = cs[h & 1][t], &sn_ = sn[h & 1][t];
                bf16x8s o;
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) {
                    o[2 * pr] = (__bf16)rotate0(v[2 * pr], v[2 * pr + 1], cs_[pr], sn_[pr]);
                    o[2 * pr + 1] = (__bf16)rotate1(v[2 * pr], v[2 * pr + 1], cs_[pr], sn_[pr]);
                }
                if (rw[h & 1][t].pos >= 0) *reinterpret_cast<bf16x8s*>(dst + (int64_t)rw[h & 1][t].row * dh) = o;
            }
        } else {
            const Row* const run = tab + (h & 1) * 64 + (lane & 7) * 8;   // this lane's 8 tokens
            const Row first = run[0], last = run[7];
            bf16* const chan = base + (int64_t)(nw - 2 * g.d + (h >> 1) * 32 + (lane >> 3)) * rows;   // its first channel, sequence 0
            if (!g.ra.pos_tab && last.pos >= 0 && last.row == first.row) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    bf16x8s o;
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = (__bf16)(e < 4 ? lo[t][e & 3] : hi[t][e & 3]);
                    __builtin_memcpy(chan + ((int64_t)first.row + t * 8) * rows + first.pos, &o, 16);
                }
            } else {
#pragma unroll 1
                for (int e = 0; e < 8; ++e) {
                    const Row one = run[e];
                    if (one.pos < 0) continue;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const __bf16 x = (__bf16)*reinterpret_cast<const float*>(rd + t * 8 * ER + e * 4);
                        __builtin_memcpy(chan + ((int64_t)one.row + t * 8) * rows + one.pos, &x, 2);
                    }
                }
            }
        }
    });
}

template <int EPI, bool PARTS>
__global__ __launch_bounds__(256, 1) void k_gemm_256(const GemmArgs g) {
    constexpr int BM = 256, BN = 256, TM = 128, TN = 128, MB = 4, NB = 4;
    constexpr int RB = 128, ITEM = 256 * RB;   // bytes of an operand row and of an item
    constexpr int LP = 8;                      // loads of a wavefront per item: 8 rows each, 32 rows apart
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, lh = lane >> 5;
    // Workgroup b runs on XCD b % 8 (round-robin dispatch), and each XCD has its own L2, so the tile sequence is cut into one
    // contiguous chunk per XCD and walks groups of GW column tiles row by row: the workgroups of an XCD work, at any moment,
    // on a near-square patch of output tiles and share its operand rows through that L2.
    constexpr int GW = 8;
    const int tiles_m = (g.M + BM - 1) / BM, total_tiles = tiles_m * g.tiles_n;
    const int nxcd = (gridDim.x & 7) == 0 ? 8 : 1;
    const int tile_stride = gridDim.x / nxcd, chunk = (total_tiles + nxcd - 1) / nxcd;
    const int chunk_base = (blockIdx.x % nxcd) * chunk;
    const int chunk_len = total_tiles - chunk_base < chunk ? total_tiles - chunk_base : chunk;   // may be <= 0
    int tile = blockIdx.x / nxcd;
    if (tile >= chunk_len) return;   // uniform over the workgroup, before any barrier
    // a tile, and its operands: first rows and sizes of the descriptors (token rows past M lie outside and read as zeros; every
    // weight row exists).  Past the chunk everything lies outside.
    struct Tile { int m0, n0, tile_n; const bf16 *a, *w0, *w1; int a_bytes, w_bytes; };
    auto tile_at = [&](int local) -> Tile {
        Tile t{};
        t.a = g.A; t.w0 = g.W0; t.w1 = g.W0;
        if (local >= chunk_len) return t;
        const int i = chunk_base + local, grp = i / (tiles_m * GW), rem = i - grp * tiles_m * GW;
        const int gw = g.tiles_n - grp * GW < GW ? g.tiles_n - grp * GW : GW;
        t.tile_n = g.tile_n0 + grp * GW + rem % gw;
        t.m0 = (rem / gw) * BM;
        t.n0 = t.tile_n * BN;
        const int left = g.M - t.m0;
        t.a += (int64_t)t.m0 * g.K;
        t.a_bytes = (left < BM ? left : BM) * g.K * 2;
        int which;
        const int base = b_row_src<EPI, BN, TN>(g, t.n0, t.tile_n, 0, which);
        t.w0 = (which == 0 ? g.W0 : which == 1 ? g.W1 : g.W2) + (int64_t)base * g.K;
        t.w1 = EPI == EPI_SWIGLU ? g.W1 + (int64_t)base * g.K : t.w0;
        t.w_bytes = 0x7fffffff;
        return t;
    };
    // Load i of an item covers its rows 32 i + 8 wave .. + 7.  Token rows go into the lane offset, which the bounds check
    // sees; weight rows into the scalar offset.  Gate|up: rows 0 .. 63 and 128 .. 191 of an item are gate rows, the rest up rows.
    auto row_key = [](int r) { return (r >> 1) & 7; };   // the same for rows 16 apart
    const int row0 = wave * 8 + (lane >> 3);
    const uint32_t voff = (uint32_t)(row0 * g.K + ((lane & 7) ^ row_key(row0)) * 8) * 2u, rows32 = (uint32_t)g.K * 64u;
    uint32_t va[LP];
#pragma unroll
    for (int i = 0; i < LP; ++i) va[i] = voff + (uint32_t)i * rows32;
    typedef __attribute__((address_space(3))) void lds_void;
    auto load_a = [&](rsrc_t r, int i, int koff, int slot) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(smem + slot + (i * 4 + wave) * 1024), 16, (int)va[i], koff, 0, 0);
    };
    auto load_w = [&](rsrc_t r0, rsrc_t r1, int i, int koff, int slot) {
        const rsrc_t r = EPI == EPI_SWIGLU && (i & 2) ? r1 : r0;
        const uint32_t row = EPI == EPI_SWIGLU ? (i & 1) + (i >> 2) * 2 : i;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(smem + slot + (i * 4 + wave) * 1024), 16, (int)voff, (int)(row * rows32 + koff), 0, 0);
    };
    const int nk = g.K / 64;
    f32x16 acc[MB][NB];
    int ka[4], kb[4];   // this lane's fragment of slice kk in row block 0: chunk 4 lh + kk
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int c = lh * 4 + kk;
        ka[kk] = (wm * TM + l32) * RB + (c ^ row_key(l32)) * 16;
        kb[kk] = (wn * TN + kperm(l32)) * RB + (c ^ row_key(kperm(l32))) * 16;
    }
    bf16x8 af[2][MB], bfr[2][NB];
    // this wavefront's loads but the youngest item's have landed and its fragment reads are done; then meet the others
    auto sync = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LP) : "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    Tile cur = tile_at(tile);
    {
        const rsrc_t ra = make_rsrc(cur.a, cur.a_bytes), r0 = make_rsrc(cur.w0, cur.w_bytes), r1 = make_rsrc(cur.w1, cur.w_bytes);
#pragma unroll
        for (int i = 0; i < LP; ++i) load_w(r0, r1, i, 0, 0);
#pragma unroll
        for (int i = 0; i < LP; ++i) load_a(ra, i, 0, ITEM);
#pragma unroll
        for (int i = 0; i < LP; ++i) load_w(r0, r1, i, RB, 2 * ITEM);   // K >= 128: step 1 exists
    }
    // slots: W and A of the step, W of the next, and where A of the next and W of the one after it go
    int s_w = 0, s_a = ITEM, s_w1 = 2 * ITEM, s_a1 = 3 * ITEM, s_w2 = 4 * ITEM;
    const bf16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
    sync();
    while (true) {
        tile += tile_stride;
        const Tile nxt = tile_at(tile);
        const bool v_tile = EPI == EPI_QKV && cur.n0 >= 2 * g.d;   // tokens feed the MFMA rows
        constexpr int XN = EPI == EPI_RESID ? XAHEAD : 1;
        f32x4 xv[XN][8];
        if constexpr (EPI == EPI_RESID) {   // the tile's own rows of the stream: nobody else writes them
            const rsrc_t rc = c_rsrc(g, cur.m0);
            const uint32_t vo = c_off(g, cur.n0, wm, wn, lane);
#pragma unroll
            for (int h = 0; h < XN; ++h)
#pragma unroll
                for (int t = 0; t < 8; ++t) xv[h][t] = __builtin_bit_cast(f32x4, bload(rc, vo + c_step(g, h, t), 0));
        }
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        // the loop is rotated by one slice, as k_gemm_ring's; nothing is pending at the start of a tile: zeros, which add nothing
#pragma unroll
        for (int i = 0; i < MB; ++i) af[1][i] = zero8;
#pragma unroll
        for (int j = 0; j < NB; ++j) bfr[1][j] = zero8;
        // what the step loads: A of the next step, W of the one after it; past the tile's last step the next tile's first
        const bf16 *pa = cur.a, *pw0 = cur.w0, *pw1 = cur.w1;
        int a_bytes = cur.a_bytes, w_bytes = cur.w_bytes, ko_a = RB, ko_w = 2 * RB;
        if (nk == 2) { pw0 = nxt.w0; pw1 = nxt.w1; w_bytes = nxt.w_bytes; ko_w = 0; }
        int left = nk;
        do {
            const unsigned char* const sb = smem + (v_tile ? s_a : s_w);   // the operand of the MFMA rows
            const unsigned char* const sa = smem + (v_tile ? s_w : s_a);
            static_for<4>([&](auto kc) {
                constexpr int kk = decltype(kc)::value, rd = kk & 1, ms = (kk + 1) & 1;
                static_for<16>([&](auto mc) {   // one MFMA of the slice before and what is issued in front of it
                    constexpr int m = decltype(mc)::value, i = m >> 2, j = (i & 1) ? 3 - (m & 3) : (m & 3), e = kk * 16 + m;
                    if constexpr (m < 4) bfr[rd][m] = *reinterpret_cast<const bf16x8*>(sb + kb[kk] + m * 32 * RB);
                    else if constexpr (m < 8) af[rd][m - 4] = *reinterpret_cast<const bf16x8*>(sa + ka[kk] + (m - 4) * 32 * RB);
                    if constexpr (e % 4 == 3 && e / 4 < LP) load_a(make_rsrc(pa, a_bytes), e / 4, ko_a, s_a1);
                    if constexpr (e % 4 == 3 && e / 4 >= LP) load_w(make_rsrc(pw0, w_bytes), make_rsrc(pw1, w_bytes), e / 4 - LP, ko_w, s_w2);
                    if constexpr (e == 33) ko_a = left == 2 ? 0 : ko_a + RB;
                    if constexpr (e == 34) pa = left == 2 ? nxt.a : pa;
                    if constexpr (e == 36) a_bytes = left == 2 ? nxt.a_bytes : a_bytes;
                    acc[i][j] = mma(af[ms][i], bfr[ms][j], acc[i][j]);
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            ko_w = left == 3 ? 0 : ko_w + RB;
            pw0 = left == 3 ? nxt.w0 : pw0;
            if constexpr (EPI == EPI_SWIGLU) pw1 = left == 3 ? nxt.w1 : pw1;
            w_bytes = left == 3 ? nxt.w_bytes : w_bytes;
            {
                const int w = s_w, a = s_a;
                s_w = s_w1; s_a = s_a1; s_w1 = s_w2; s_a1 = w; s_w2 = a;
            }
            sync();
        } while (--left > 0);
#pragma unroll
        for (int i = 0; i < MB; ++i)   // the tile's last slice
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = mma(af[1][i], bfr[1][j], acc[i][j]);
        // the slots of the last step have been read by everybody and are loaded again after the barrier below
        unsigned char* const lds = smem + (wave >> 1 ? s_w2 : s_a1) + (wave & 1) * (ITEM / 2);
        if constexpr (PARTS) logit_parts<BN, TM, MB, NB>(g, acc, cur.m0, cur.tile_n, wm, wn, l32, lh);
        if constexpr (EPI == EPI_QKV) {
            epilogue_qkv(g, acc, v_tile, cur.m0, cur.n0, wm, wn, lane, lds);
        } else if constexpr (EPI == EPI_SWIGLU) {
            epilogue_h(g, acc, cur.m0, cur.tile_n, wm, wn, lane, lds);
        } else {
            epilogue_c<EPI, XN>(g, acc, xv, cur.m0, cur.n0, wm, wn, lane, lds);
        }
        if (tile >= chunk_len) break;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        cur = nxt;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load into this LDS may outlive the workgroup
}

// ---- BM x BN x 64 tiles over an LDS ring of NS stages, filled by direct loads (global memory -> LDS) ------------
// For launches whose 256 x 256 tiles do not fill the chip.  What bounds them is the operand traffic into a CU: with the
// matrix instructions taken out the loads alone take the kernel's time (576 x 4096 x 4096 on 128 x 128 tiles: 36.5 of
// 37.4 us, the tokens alone 14, the weights alone 26; with the loads taken out 30).  So: no staging registers and no
// ds_write (a wavefront's load puts 1 KB, 8 rows of 64, straight into the ring), NS - 1 stages in flight while one is
// multiplied, and the tile is chosen per launch so that all CUs fetch (choose_tile).  One barrier per stage: it is
// passed when the stage has landed for every wavefront (each waits for its own loads, younger stages stay in flight)
// and every wavefront has read the stage before, whose slot the next loads fill.
// The direct load writes lane l's 16 bytes at 16 l, so a row cannot be padded against bank conflicts; instead chunk c
// of row r sits at chunk position c ^ ((r / 2) % 8): 16 consecutive lanes of a fragment read, 16 rows 128 bytes apart,
// then touch every bank once (no conflicts counted; with c ^ (r % 8) half of the LDS cycles were conflicts).
// The k deal, hence every sum, is that of k_gemm_256 above, whatever the tile.
// us per launch, before (128 x 128 tiles, staged through registers) -> here, cold weights: 186 tokens: 4096 x 4096
// 36 -> 21, 4096 x 11008 83 -> 54, q|k|v 84 -> 40, gate|up 67 -> 58; 1024 tokens of width 1024: out 15 -> 6.6, down
// 27 -> 12, q|k|v 27 -> 14; 1980 tokens of width 4096: out 73 -> 65, down 174 -> 152.
// PAIRED (5 stages): loads go out for two K-steps at a time, every other step, both halves of a 256-byte row segment one
// behind the other, where a row's next 128 bytes otherwise follow a whole step later: 128 x 128 tiles over K = 11008, 576
// tokens 94 -> 87 us, 1024 tokens 111 -> 99; the smaller tiles, which keep fewer bytes in flight, lose by it.
template <int BM, int BN, int WGM, int WGN, int NS, int EPI, bool PAIRED>
__global__ __launch_bounds__(WGM* WGN * 64, 1) void k_gemm_ring(const GemmArgs g) {
    constexpr int NW = WGM * WGN, TM = BM / WGM, TN = BN / WGN, MB = TM / 32, NB = TN / 32;
    constexpr int RB = 128;                                             // bytes of a tile row
    constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW, LPS = LA + LB;    // loads of a wavefront per stage
    constexpr int STAGE = (BM + BN) * RB;
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "whole loads per wavefront");
    static_assert(EPI != EPI_SWIGLU || (NB % 2 == 0 && (TN / 2) % (8 * NW) == 0), "a load never straddles gate and up");
    static_assert((NS - 2) * LPS < 64 && NS >= 3, "the wait counts loads in 6 bits");
    static_assert(!PAIRED || NS == 5, "two pairs and the step between them");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // NS stages of [BM + BN][RB]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN, l32 = lane & 31, lh = lane >> 5;
    // one tile per workgroup; tiles to XCDs as in k_gemm_256 (the grid is a multiple of 8)
    constexpr int GW = 8;
    const int tiles_m = (g.M + BM - 1) / BM, total = tiles_m * g.tiles_n, chunk = (total + 7) / 8;
    const int loc = blockIdx.x >> 3, t = (blockIdx.x & 7) * chunk + loc;
    if (loc >= chunk || t >= total) return;                             // uniform over the workgroup, before any barrier
    const int grp = t / (tiles_m * GW), rem = t - grp * tiles_m * GW;
    const int gw = g.tiles_n - grp * GW < GW ? g.tiles_n - grp * GW : GW;
    const int tile_n = g.tile_n0 + grp * GW + rem % gw, m0 = (rem / gw) * BM, n0 = tile_n * BN;

    // Operand addresses: a descriptor at the tile's first row, a lane offset per load (its row, clamped to the matrix, and
    // the chunk that belongs at its position), the K-step as scalar offset.
    const int lrow = lane >> 3, lch = lane & 7;
    auto row_key = [](int r) { return (r >> 1) & 7; };
    uint32_t va[LA], vb[LB];
    const rsrc_t rA = make_rsrc(g.A + (int64_t)m0 * g.K, 0x7fffffff);
    rsrc_t rW[2];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int r = (i * NW + wave) * 8 + lrow, rc = m0 + r < g.M ? r : g.M - 1 - m0;
        va[i] = (uint32_t)(rc * g.K + (lch ^ row_key(r)) * 8) * 2u;
    }
    {
        int which;
        const int base = b_row_src<EPI, BN, TN>(g, n0, tile_n, 0, which);
        const bf16* w0 = which == 0 ? g.W0 : which == 1 ? g.W1 : g.W2;
        rW[0] = make_rsrc(w0 + (int64_t)base * g.K, 0x7fffffff);
        rW[1] = make_rsrc((EPI == EPI_SWIGLU ? g.W1 : w0) + (int64_t)base * g.K, 0x7fffffff);
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            const int r = (i * NW + wave) * 8 + lrow;
            const int rs = b_row_src<EPI, BN, TN>(g, n0, tile_n, r, which) - base;
            vb[i] = (uint32_t)(rs * g.K + (lch ^ row_key(r)) * 8) * 2u;
        }
    }
    typedef __attribute__((address_space(3))) void lds_void;
    auto load = [&](auto ic, int kt, int slot) {   // load i of this wavefront for K-step kt
        constexpr int i = decltype(ic)::value;
        unsigned char* st = smem + slot * STAGE;
        if constexpr (i < LA) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rA, (lds_void*)(st + (i * NW + wave) * 1024), 16, (int)va[i], kt * RB, 0, 0);
        } else {
            constexpr int j = i - LA;
            constexpr int w = EPI == EPI_SWIGLU ? ((j * NW * 8) % TN >= TN / 2 ? 1 : 0) : 0;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rW[w], (lds_void*)(st + BM * RB + (j * NW + wave) * 1024), 16, (int)vb[j], kt * RB, 0, 0);
        }
    };
    const int nk = g.K / 64;
    f32x16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    int ka[4], kb[4];   // this lane's fragment of slice kk in row block 0: chunk 4 lh + kk
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int c = lh * 4 + kk;
        ka[kk] = (wm * TM + l32) * RB + (c ^ row_key(l32)) * 16;
        kb[kk] = BM * RB + (wn * TN + kperm(l32)) * RB + (c ^ row_key(kperm(l32))) * 16;
    }
    bf16x8 af[2][MB], bfr[2][NB];
    auto lfrag = [&](const unsigned char* st, int kk, int slot) {
#pragma unroll
        for (int i = 0; i < MB; ++i) af[slot][i] = *reinterpret_cast<const bf16x8*>(st + ka[kk] + i * 32 * RB);
#pragma unroll
        for (int j = 0; j < NB; ++j) bfr[slot][j] = *reinterpret_cast<const bf16x8*>(st + kb[kk] + j * 32 * RB);
    };
    auto mm = [&](int slot) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = mma(af[slot][i], bfr[slot][j], acc[i][j]);
    };
    // One K-step, rotated by one slice as in k_gemm_256: the MFMAs of the step before's last slice run while the first
    // fragments are on their way.  more: load step kt + NS - 1 into the slot of step kt - 1 (PAIRED: steps kt + 3 and
    // kt + 4 into the slots of kt - 2 and kt - 1; a step past the end is the last one again, into a slot nobody reads);
    // first: nothing is pending.
    auto step = [&](int slot, int kt, auto more, auto first) {
        const unsigned char* st = smem + slot * STAGE;
        static_for<4>([&](auto kc) {
            constexpr int kk = decltype(kc)::value;
            lfrag(st, kk, kk & 1);
            if constexpr (decltype(more)::value) {
                constexpr int lo = kk * LPS / 4, hi = (kk + 1) * LPS / 4;
                static_for<hi - lo>([&](auto ic) {
                    constexpr std::integral_constant<int, lo + decltype(ic)::value> i;
                    if constexpr (PAIRED) load(i, kt + 3, slot >= 2 ? slot - 2 : slot + 3);
                    load(i, PAIRED && kt + 4 >= nk ? nk - 1 : kt + NS - 1, slot == 0 ? NS - 1 : slot - 1);
                });
            }
            if constexpr (!(kk == 0 && decltype(first)::value)) mm((kk + 1) & 1);
        });
        // per slice: its fragment reads first (left alone, the scheduler puts the pending MFMAs in front of them), then
        // the MFMAs of the slice before with the loads in between
        if constexpr (!decltype(first)::value) static_for<4>([&](auto kc) {
            constexpr int kk = decltype(kc)::value, per = PAIRED ? 2 : 1;
            constexpr int nl = decltype(more)::value ? ((kk + 1) * LPS / 4 - kk * LPS / 4) * per : 0, nm = MB * NB;
            __builtin_amdgcn_sched_group_barrier(0x100, MB + NB, 0);
            static_for<nm>([&](auto mc) {
                constexpr int m = decltype(mc)::value, n = (m + 1) * nl / nm - m * nl / nm;
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if constexpr (n > 0) __builtin_amdgcn_sched_group_barrier(0x010, n, 0);
            });
        });
    };
    // wait until this wavefront's share of the next stage has landed (at most `younger` loads in flight; < 0: it has
    // already) and its fragment reads are done, then meet the others
    auto sync = [&](auto younger) {
        constexpr int n = decltype(younger)::value;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (n >= 0) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(n) : "memory");
        else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::true_type yes;
    constexpr std::false_type no;
    constexpr std::integral_constant<int, 0> none_in_flight;
    int kt = 0, slot = 0;
    auto next = [&]() { ++kt; slot = slot + 1 == NS ? 0 : slot + 1; };
    if constexpr (PAIRED) {
        static_for<LPS>([&](auto ic) { load(ic, 0, 0); load(ic, 1, 1); });   // K >= 128: both steps exist
        if (nk > 2) static_for<LPS>([&](auto ic) { load(ic, 2, 2); load(ic, nk > 3 ? 3 : 2, 3); });
        constexpr std::integral_constant<int, 2 * LPS> next_pair;
        constexpr std::integral_constant<int, -1> landed;                    // an odd step landed with the one before
        if (nk > 2) sync(next_pair);
        else sync(none_in_flight);
        step(slot, kt, no, yes);
        next();
        while (kt + 3 < nk) {                                                // no branch inside: the accumulators would be copied
            sync(landed);
            step(slot, kt, yes, no);
            next();
            sync(next_pair);
            step(slot, kt, no, no);
            next();
        }
        sync(landed);                                                        // the last one to three steps
        step(slot, kt, no, no);
        next();
        if (kt < nk) {
            sync(none_in_flight);
            step(slot, kt, no, no);
            next();
            if (kt < nk) {
                sync(landed);
                step(slot, kt, no, no);
            }
        }
    } else {
        static_for<NS - 1>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            if (s < nk) static_for<LPS>([&](auto ic) { load(ic, s, s); });
        });
        if (nk >= NS) {
            sync(std::integral_constant<int, (NS - 2) * LPS>{});
            step(slot, kt, yes, yes);
            for (next(); kt + NS - 1 < nk; next()) {
                sync(std::integral_constant<int, (NS - 2) * LPS>{});
                step(slot, kt, yes, no);
            }
            static_for<NS - 1>([&](auto ic) {   // the last NS - 1 stages: nothing more to load
                sync(std::integral_constant<int, (NS - 2 - decltype(ic)::value) * LPS>{});
                step(slot, kt, no, no);
                next();
            });
        } else {                                // a short K: everything is in flight already
            sync(none_in_flight);
            step(slot, kt, no, yes);
            for (next(); kt < nk; next()) step(slot, kt, no, no);
        }
    }
    mm(1);
    epilogue<EPI, BN, TM, TN, MB, NB>(g, acc, m0, n0, tile_n, wm, wn, l32, lh);
}

// column tiles [tile_n0, tile_n0 + tiles_n)
template <int EPI, bool PARTS>
void run_256(GemmArgs g, int tile_n0, int tiles_n, hipStream_t st) {
    auto kern = k_gemm_256<EPI, PARTS>;
    constexpr int lds = LDS_256;
    static int attr_state = 0;  // each instantiation is configured once per process
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, &attr_state)) return;
    const int total = (g.M + 255) / 256 * tiles_n, resident = cu_count();
    g.tiles_n = tiles_n;
    g.tile_n0 = tile_n0;
    hipLaunchKernelGGL(kern, dim3(total < resident ? total : resident), dim3(256), lds, st, g);
}

// Epilogue of the weight-streaming kernels on two adjacent output columns n, n + 1 of token m (v1: the up sums of
// gate|up).  The same five fused epilogues as the tiled kernels; a bf16 operand of a following projection is written
// in fragment order.
template <int EPI>
__device__ __forceinline__ void stream_epilogue(const GemmArgs& g, int m, int n, const float (&v0)[2], const float (&v1)[2]) {
    if constexpr (EPI == EPI_RESID || EPI == EPI_LOGITS) {
        float* dst = g.Cf + (int64_t)m * g.N + n;
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (n + e < g.N) dst[e] = EPI == EPI_RESID ? dst[e] + v0[e] : v0[e];
    } else if constexpr (EPI == EPI_SWIGLU) {
        const int f = g.N / 2;
        bf16* dst = g.Cb + frag_index(m, n, f);   // the down projection streams too: its token operand, fragment order
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (n + e < f) dst[e] = __float2bfloat16(silu(v0[e]) * v1[e]);
    } else {
        const TokPlace pl = place(g.ra, m);
        if (pl.pos < 0) return;   // an unused slot of a scattered launch
        const int dh = g.ra.head_dim, pos = pl.pos;
        if (n < 2 * g.d) {
            const int seg = n / g.d, c = n - seg * g.d;
            const int hd = c / dh, cc = c % dh;
            const float cs = g.ra.cos[(int64_t)pos * (dh / 2) + (cc >> 1)], sn = g.ra.sin[(int64_t)pos * (dh / 2) + (cc >> 1)];
            bf16* dst;
            if (seg == 0) {
                dst = g.Cb + (((int64_t)pl.b * g.ra.n_heads + hd) * g.ra.L + pl.jj) * dh + cc;
            } else {
                const int64_t hb = ((int64_t)g.ra.layer * g.ra.max_batch + pl.bc) * g.ra.n_heads + hd;
                dst = g.kc + (hb * g.ra.max_seq + pos) * dh + cc;
            }
            dst[0] = __float2bfloat16(rotate0(v0[0], v0[1], cs, sn));
            dst[1] = __float2bfloat16(rotate1(v0[0], v0[1], cs, sn));
        } else {   // V: transposed cache
            const int nv = n - 2 * g.d;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int hd = (nv + e) / dh, cc = (nv + e) % dh;
                const int64_t hb = ((int64_t)g.ra.layer * g.ra.max_batch + pl.bc) * g.ra.n_heads + hd;
                if (nv + e < g.d) g.vc[(hb * dh + cc) * g.ra.max_seq + pos] = __float2bfloat16(v0[e]);
            }
        }
    }
}

// ---- up to 64 tokens (single-token decoding of a few sequences, island passes): weight-streaming kernel ----
// The work is reading every weight once, so nothing is staged: a workgroup owns 16 output columns (for
// gate|up: 16 feed-forward columns = 16 gate rows + 16 up rows), or up to four such blocks where several token groups
// share them, or 8 feed-forward columns (run_gemv's rules; a sum is the same in each), its 8 wavefronts split K, and every lane
// feeds v_mfma_f32_16x16x32_bf16 from registers loaded straight from global memory.  In that instruction's operand
// layout the four lanes l16, l16 + 16, l16 + 32, l16 + 48 hold 4 x 8 consecutive k of weight row l16, so one load
// instruction of a wavefront reads 64 contiguous bytes of each of 16 rows: whole 64-byte sectors (with the 32-row
// instruction only two lanes share a row, 32 of every 64 bytes fetched per request), and a matrix of N columns
// gives N / 16 workgroups (256 for the 4096-column projections: one per CU).  The tokens are the instruction's
// column dimension (columns m >= M are fed zeros), up to four groups of 16, and arrive in fragment order (the
// producing kernels write them so: one contiguous KB per group and step, no lane exchange); the accumulators come out as
// D[weight row 4 q + i][token l16], q = lane / 16: a lane owns 4 consecutive output columns of one token.  The
// 8 partial sums are added in a fixed order through LDS and the epilogue runs on pairs of adjacent columns.
typedef __attribute__((ext_vector_type(4))) float f32x4v;
enum { UNIT_HALF = 0 };   // gate|up in workgroups of 8 feed-forward columns: 8 gate rows and 8 up rows are one MFMA's 16
template <int EPI, int MT, int NB, bool WFRAG>
__global__ __launch_bounds__(512) void k_gemv_bf16(const GemmArgs g) {
    constexpr bool HALF = NB == UNIT_HALF;
    constexpr int NBLK = HALF ? 1 : NB;                            // column blocks of the workgroup
    constexpr int NA = EPI == EPI_SWIGLU && !HALF ? 2 : 1;         // weight matrices (accumulator sets) per column
    constexpr int NR = NA * NBLK;                                  // 16-row weight blocks a step multiplies
    constexpr int COLS = HALF ? 8 : 16;                            // columns of a block
    static_assert(!HALF || (EPI == EPI_SWIGLU && MT == 1), "half blocks are gate|up's, one token group");
    // 32-deep k-steps in flight per wavefront: what 16 requests of 16 bytes per lane allow, at least 4 (measured at
    // the 7B shape: 16 -> 181 ms, 24 -> 185, 32 -> 186 for a re-sampling run of 21 island passes); with several column blocks
    // one workgroup has a CU to itself, and 24 requests are what its registers hold
    constexpr int U = NBLK > 1 ? (24 / (NR + MT) < 2 ? 2 : 24 / (NR + MT)) : 16 / (NR + MT) < 4 ? 4 : 16 / (NR + MT);
    constexpr int NBUF = NBLK > 1 ? 2 : 1;
    __shared__ float part[NBUF][8][NA * MT][4][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4;
    // Weight loads use another lane order than the MFMA: lane 4 r + c fetches chunk c (16 bytes) of row r, so that
    // four ADJACENT lanes read 64 contiguous bytes (one access of the vector L1; in the MFMA's own order, lane
    // 16 c + r, adjacent lanes sit in different rows and every lane is an access of its own: the L1 then limits the
    // kernel).  Each fetched register is moved to the MFMA's order by a lane permutation (ds_bpermute: lane 16 c + r
    // takes the value of lane 4 r + c); which k a slot holds is unchanged, hence so is every sum.  The permutations
    // occupy the LDS pipe (measured: about half of the kernel's time with one token group when the token operand was
    // fetched and permuted the same way, 16 of 20 permutations per step with four groups), which is why the token
    // operand arrives in fragment order and needs none.
    const int lrow = lane >> 2, lchunk = lane & 3;
    const int from_lane = (4 * l16 + q) << 2;   // byte address of the source lane for ds_bpermute
    const int cols = EPI == EPI_SWIGLU ? g.N / 2 : g.N, nblocks = (cols + COLS - 1) / COLS;
    const int steps = g.K / 32;
    const int blk0 = blockIdx.x * NBLK;    // first block of columns (gate|up: of feed-forward columns)
    const int per = (steps + 7) / 8;
    const int s0 = wave * per, s1 = s0 + per < steps ? s0 + per : steps;

    // weight row(s) this lane fetches; with a copy in fragment order (WFRAG) the KB of (16-row block, step) is
    // contiguous in the MFMA's own lane order: lane l owns its bytes [16 l, 16 l + 16), no exchange afterwards
    const bf16* w[NR];
#pragma unroll
    for (int nb = 0; nb < NBLK; ++nb) {
        int blk = NBLK == 1 || blk0 + nb < nblocks ? blk0 + nb : nblocks - 1;   // a block past the last column re-reads the last one
        const bf16 *base0 = g.W0, *base1 = g.W1;
        if constexpr (EPI == EPI_QKV) {
            const int seg = blk * 16 / g.d;                        // a block never straddles q | k | v (d % 16 == 0)
            base0 = seg == 0 ? g.W0 : seg == 1 ? g.W1 : g.W2;
            blk -= seg * (g.d / 16);
        }
        if constexpr (HALF) {
            if constexpr (WFRAG) {   // rows 0 .. 7 of the MFMA: half of the gate matrix's 16-row block, rows 8 .. 15: of the up matrix's
                w[0] = (l16 < 8 ? base0 : base1) + (int64_t)(blk >> 1) * steps * 512 + (q * 16 + (blk & 1) * 8 + (l16 & 7)) * 8;
            } else {
                const int r = blk * 8 + (lrow & 7);
                w[0] = (lrow < 8 ? base0 : base1) + (int64_t)(r < cols ? r : cols - 1) * g.K;
            }
        } else if constexpr (WFRAG) {
            w[nb * NA] = base0 + (int64_t)blk * steps * 512 + lane * 8;
            if constexpr (NA == 2) w[nb * NA + 1] = base1 + (int64_t)blk * steps * 512 + lane * 8;
        } else {
            int r = blk * 16 + lrow;
            if constexpr (EPI != EPI_QKV) r = r < cols ? r : cols - 1;
            w[nb * NA] = base0 + (int64_t)r * g.K;
            if constexpr (NA == 2) w[nb * NA + 1] = base1 + (int64_t)r * g.K;
        }
    }
    // The token operand is stored in fragment order: the KB of (token group t, step s) is contiguous and lane l owns
    // its bytes [16 l, 16 l + 16) in the MFMA's own order.  Tokens past M are not written by anybody: fed as zeros.
    const bf16* const xg = g.A + lane * 8;
    bool has_x[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) has_x[t] = t * 16 + l16 < g.M;
    if constexpr (!WFRAG) {
#pragma unroll
        for (int i = 0; i < NR; ++i) w[i] += lchunk * 8;
    }
    auto to_mfma_order = [&](u32x4 v) {
        u32x4 r;
        r.x = (uint32_t)__builtin_amdgcn_ds_bpermute(from_lane, (int)v.x);
        r.y = (uint32_t)__builtin_amdgcn_ds_bpermute(from_lane, (int)v.y);
        r.z = (uint32_t)__builtin_amdgcn_ds_bpermute(from_lane, (int)v.z);
        r.w = (uint32_t)__builtin_amdgcn_ds_bpermute(from_lane, (int)v.w);
        return r;
    };

    f32x4v acc[NR][MT];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[i][t] = f32x4v{0.f, 0.f, 0.f, 0.f};
    const u32x4 zero = {0u, 0u, 0u, 0u};
    // U steps in flight per wavefront, all the time: the registers of a step are requested again, for the step U
    // further on, as soon as the step has been multiplied, so the memory pipeline never drains between batches
    // (a batch that is requested, waited for and multiplied as a whole leaves it empty for a memory round trip
    // per batch).  No branch on the step index: steps past the end of the slice re-read the matrix's last step and
    // are multiplied by zeros (a branch there makes the compiler wait for every load in flight).  The last batch
    // requests nothing.
    u32x4 wv[NR][U], xv[MT][U];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int u = 0; u < U; ++u) xv[t][u] = zero;
    auto request = [&](int u, int s) {
        const int sc = s < steps ? s : steps - 1;
#pragma unroll
        for (int i = 0; i < NR; ++i) wv[i][u] = *reinterpret_cast<const u32x4*>(w[i] + sc * (WFRAG ? 512 : 32));
#pragma unroll
        for (int t = 0; t < MT; ++t)   // lanes whose token does not exist request nothing (a 4-token launch reads 4 x 64 bytes of the KB)
            if (has_x[t]) xv[t][u] = *reinterpret_cast<const u32x4*>(xg + ((int64_t)t * steps + sc) * 512);
    };
    auto permute = [&](int u, int s, bf16x8 (&wf)[NR], bf16x8 (&xf)[MT]) {
        const bool in_slice = s < s1;
#pragma unroll
        for (int i = 0; i < NR; ++i) wf[i] = __builtin_bit_cast(bf16x8, WFRAG ? wv[i][u] : to_mfma_order(wv[i][u]));
#pragma unroll
        for (int t = 0; t < MT; ++t) xf[t] = __builtin_bit_cast(bf16x8, (in_slice && has_x[t]) ? xv[t][u] : zero);
    };
    auto multiply = [&](const bf16x8 (&wf)[NR], const bf16x8 (&xf)[MT]) {
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int t = 0; t < MT; ++t)
                acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i], xf[t], acc[i][t], 0, 0, 0);
    };
    if (s0 < s1) {   // uniform over the wavefront
#pragma unroll
        for (int u = 0; u < U; ++u) request(u, s0 + u);
        int sb = s0;
        for (; sb + U < s1; sb += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                bf16x8 wf[NR], xf[MT];
                permute(u, sb + u, wf, xf);
                request(u, sb + U + u);
                multiply(wf, xf);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            bf16x8 wf[NR], xf[MT];
            permute(u, sb + u, wf, xf);
            multiply(wf, xf);
        }
    }
    // reduce the K-slices in a fixed order through LDS, a column block at a time (its successor goes to the other buffer, so one
    // barrier a block); thread (pr, t, lane) of the first 2 * MT wavefronts then owns accumulators 2 pr, 2 pr + 1 of token
    // group t = two adjacent columns of token t * 16 + l16
    const int pr = wave & 1, tg = wave >> 1;
    const int m = tg * 16 + l16;
    static_for<NBLK>([&](auto nbc) {
        constexpr int nb = decltype(nbc)::value, buf = nb % NBUF;
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) part[buf][wave][a * MT + t][r][lane] = acc[nb * NA + a][t][r];
        __syncthreads();
        if (wave < 2 * MT && m < g.M && (NBLK == 1 || blk0 + nb < nblocks) && (!HALF || q < 2)) {
            float v0[2], v1[2] = {0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
                for (int ww = 0; ww < 8; ++ww) {
                    sum0 += part[buf][ww][tg][2 * pr + e][lane];
                    if constexpr (HALF) sum1 += part[buf][ww][tg][2 * pr + e][lane ^ 32];
                    else if constexpr (NA == 2) sum1 += part[buf][ww][MT + tg][2 * pr + e][lane];
                }
                v0[e] = sum0;
                v1[e] = sum1;
            }
            const int n = (blk0 + nb) * COLS + 4 * q + 2 * pr;
            stream_epilogue<EPI>(g, m, n, v0, v1);
        }
    });
}

// ---- 65 to 256 tokens with the weight copy in fragment order, out and down of 17 to 64 tokens: the token operand goes through LDS ----
// With several token groups the kernel above spends its time on the token operand: every workgroup (16 columns) reads
// all of it through its vector L1, a KB per token group and KB of weights.  Here a workgroup owns 128 columns (a
// wavefront 16 of them; 64 columns and four wavefronts: run_gemv's rule) and a slice of K: the slice's token operand, which arrives
// in fragment order, is copied to LDS once per workgroup, 8 k-steps at a time, and every wavefront feeds its MFMAs from there (one
// 16-byte LDS read per lane and token group); only the weights, contiguous KB blocks of the fragment-order copy (or, up to 64 tokens,
// rows as they come, exchanged between lanes as above), come through the memory
// pipeline, 8 steps in flight per wavefront.  K is dealt to `ksplit` workgroups per column group; each leaves its sums
// [M, its columns] in `ksums`, and k_stream_finish (out, down: the norm behind them) adds the slices in index order and runs the
// epilogue (no float atomics: the result does not depend on which workgroup finishes first).  Gate|up and q|k|v are concatenations of
// their weight matrices (`seg_rows` rows each) along the column axis.
// Workgroups of 12 wavefronts and 192 columns were faster at 65 to 160 tokens of width 4096 (gate|up 65 -> 48 us), but by more K slices
// than 161 tokens have, so that a row's sums followed the rows beside it.
template <int MTB, bool WFRAG, int NW>
__global__ __launch_bounds__(NW * 64) void k_gemv_shared(const GemmArgs g, int ncols, int seg_rows, int ncg) {
    constexpr int CH = 8;                         // k-steps per LDS chunk = weight steps in flight per wavefront
    constexpr int PIECES = CH * MTB / NW;         // 16-byte pieces of a chunk per thread
    static_assert(CH % NW == 0, "whole pieces");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // fragment (group t, step j) at (t CH + j) KB
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = blockIdx.x % ncg, kw = blockIdx.x / ncg;   // neighbouring workgroups share a K slice of the token operand
    const int n_w = cg * (NW * 16) + wave * 16;                     // this wavefront's first column
    const int steps = g.K / 32, per = (steps + g.ksplit - 1) / g.ksplit;
    const int s0 = kw * per, s1 = s0 + per < steps ? s0 + per : steps;
    const int n_groups = (g.M + 15) >> 4;

    const bf16* w;
    {
        const int last = (ncols - 1) / 16 * 16;               // a wavefront past the last column re-reads the last block
        const int n_c = n_w < last ? n_w : last;
        const int seg = n_c / seg_rows;                        // 16 columns never straddle two matrices (seg_rows % 16 == 0)
        const bf16* const base = seg == 0 ? g.W0 : seg == 1 ? g.W1 : g.W2;
        if constexpr (WFRAG) {
            w = base + (int64_t)((n_c - seg * seg_rows) / 16) * steps * 512 + lane * 8;
        } else {                                               // chunk lane % 4 of row lane / 4, as in k_gemv_bf16
            const int r = n_c - seg * seg_rows + (lane >> 2);
            w = base + (int64_t)(r < seg_rows ? r : seg_rows - 1) * g.K + (lane & 3) * 8;
        }
    }
    const int from_lane = (4 * (lane & 15) + (lane >> 4)) << 2;
    f32x4v acc[MTB];
#pragma unroll
    for (int t = 0; t < MTB; ++t) acc[t] = f32x4v{0.f, 0.f, 0.f, 0.f};
    const u32x4 zero = {0u, 0u, 0u, 0u};
    u32x4 wv[CH], xr[PIECES];
    auto request = [&](int u, int s) {
        const int sc = s < s1 ? s : s1 - 1;
        wv[u] = *reinterpret_cast<const u32x4*>(w + (int64_t)sc * (WFRAG ? 512 : 32));
    };
    auto to_mfma_order = [&](u32x4 v) {
        if constexpr (!WFRAG)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(from_lane, (int)v[i]);
        return v;
    };
    // chunk of steps [sc0, sc0 + CH): piece p = ((t CH + j) 64 + lane position); steps past the slice and token groups
    // that do not exist are zeros (tokens past M inside the last group are whatever the buffer holds: they only reach
    // accumulator columns that are never stored)
    auto xload = [&](int sc0) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int p = tid + i * (NW * 64), t = p / (CH * 64), j = (p / 64) % CH;
            xr[i] = zero;
            if (t < n_groups && sc0 + j < s1)
                xr[i] = *reinterpret_cast<const u32x4*>(g.A + ((int64_t)t * steps + sc0 + j) * 512 + (p & 63) * 8);
        }
    };
    auto xstore = [&]() {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) *reinterpret_cast<u32x4*>(smem + (size_t)(tid + i * (NW * 64)) * 16) = xr[i];
    };
    auto chunk = [&](int sc0, auto req) {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const bf16x8 wf = __builtin_bit_cast(bf16x8, to_mfma_order(wv[u]));
            if constexpr (decltype(req)::value) request(u, sc0 + CH + u);
#pragma unroll
            for (int t = 0; t < MTB; ++t) {
                const bf16x8 xf = *reinterpret_cast<const bf16x8*>(smem + (size_t)((t * CH + u) * 64 + lane) * 16);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf, acc[t], 0, 0, 0);
            }
        }
    };
    if (s0 < s1) {   // uniform over the workgroup
#pragma unroll
        for (int u = 0; u < CH; ++u) request(u, s0 + u);
        xload(s0);
        xstore();
        __syncthreads();
        int sc0 = s0;
        for (; sc0 + CH < s1; sc0 += CH) {
            xload(sc0 + CH);
            chunk(sc0, std::true_type{});
            __syncthreads();   // every wavefront has read the chunk
            xstore();
            __syncthreads();
        }
        chunk(sc0, std::false_type{});   // the last chunk requests nothing
    }
    // this slice's sums: D[weight row 4 q + i][token l16] -> ksums[kw][m][n_w + 4 q + i].  The lane is counted anew: kept over the
    // loop it was one register too many with 12, 15 and 16 token groups and went to scratch memory.
    const int lane_ = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), l16 = lane_ & 15, q = lane_ >> 4;
#pragma unroll
    for (int t = 0; t < MTB; ++t) {
        const int m = t * 16 + l16, n = n_w + 4 * q;
        if (m < g.M && n < ncols) {
            float* dst = g.ksums + ((int64_t)kw * g.M + m) * ncols + n;
            if (n + 4 <= ncols) {
                *reinterpret_cast<f32x4v*>(dst) = acc[t];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (n + i < ncols) dst[i] = acc[t][i];
            }
        }
    }
}

// adds the K slices of two adjacent columns of a token in index order and runs the projection's epilogue
template <int EPI>
__global__ __launch_bounds__(256) void k_stream_finish(const GemmArgs g, int ncols) {
    const int cols = EPI == EPI_SWIGLU ? ncols / 2 : ncols;   // gate|up: the up sums of column n sit at column f + n
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int pairs = cols / 2;
    const int m = (int)(idx / pairs), n = 2 * (int)(idx % pairs);
    if (m >= g.M) return;
    float v0[2] = {0.f, 0.f}, v1[2] = {0.f, 0.f};
    for (int kw = 0; kw < g.ksplit; ++kw) {
        const float* src = g.ksums + ((int64_t)kw * g.M + m) * ncols + n;
        const float2 a = *reinterpret_cast<const float2*>(src);
        v0[0] += a.x;
        v0[1] += a.y;
        if constexpr (EPI == EPI_SWIGLU) {
            const float2 b = *reinterpret_cast<const float2*>(src + cols);
            v1[0] += b.x;
            v1[1] += b.y;
        }
    }
    stream_epilogue<EPI>(g, m, n, v0, v1);
}

// the sums of g.ksplit slices of K over `ncols` columns into g.ksums; WFRAG: the weights are in fragment order, NW: wavefronts a
// workgroup.  False, with the error noted, where it could not be launched: the sums are not to be read.
template <int MTB, bool WFRAG, int NW>
bool launch_gemv_shared(const GemmArgs& g, int ncols, int seg_rows, hipStream_t st) {
    auto kern = k_gemv_shared<MTB, WFRAG, NW>;
    static int attr_state = 0;
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), MTB * 8 * 1024, &attr_state)) return false;
    if ((int64_t)g.ksplit * g.M * ncols > g.ksum_floats) {   // no room for the slices
        note_hip_error(hipErrorInvalidValue);
        return false;
    }
    const int ncg = (ncols + NW * 16 - 1) / (NW * 16);
    hipLaunchKernelGGL(kern, dim3(ncg * g.ksplit), dim3(NW * 64), (size_t)MTB * 8 * 1024, st, g, ncols, seg_rows, ncg);
    return true;
}

template <int EPI>
int run_gemv_shared(GemmArgs g, hipStream_t st) {
    const int ncols = g.N, seg_rows = EPI == EPI_QKV ? g.d : EPI == EPI_SWIGLU ? g.N / 2 : g.N;
    g.ksplit = stream_slices(g.M, ncols, g.K, true, EPI == EPI_RESID);
    bool ok;
    switch ((g.M + 15) / 16) {   // one instantiation per number of token groups: LDS reads and MFMAs follow it
        case 1: case 2: case 3: case 4: ok = launch_gemv_shared<4, true, 8>(g, ncols, seg_rows, st); break;
        case 5: ok = launch_gemv_shared<5, true, 8>(g, ncols, seg_rows, st); break;
        case 6: ok = launch_gemv_shared<6, true, 8>(g, ncols, seg_rows, st); break;
        case 7: ok = launch_gemv_shared<7, true, 8>(g, ncols, seg_rows, st); break;
        case 8: ok = launch_gemv_shared<8, true, 8>(g, ncols, seg_rows, st); break;
        case 9: ok = launch_gemv_shared<9, true, 8>(g, ncols, seg_rows, st); break;
        case 10: ok = launch_gemv_shared<10, true, 8>(g, ncols, seg_rows, st); break;
        case 11: ok = launch_gemv_shared<11, true, 8>(g, ncols, seg_rows, st); break;
        case 12: ok = launch_gemv_shared<12, true, 8>(g, ncols, seg_rows, st); break;
        case 13: ok = launch_gemv_shared<13, true, 8>(g, ncols, seg_rows, st); break;
        case 14: ok = launch_gemv_shared<14, true, 8>(g, ncols, seg_rows, st); break;
        case 15: ok = launch_gemv_shared<15, true, 8>(g, ncols, seg_rows, st); break;
        default: ok = launch_gemv_shared<16, true, 8>(g, ncols, seg_rows, st); break;
    }
    if (!ok) return 0;
    if constexpr (EPI != EPI_RESID) {
        const int cols = EPI == EPI_SWIGLU ? ncols / 2 : ncols;
        const int64_t threads = (int64_t)g.M * (cols / 2);
        hipLaunchKernelGGL((k_stream_finish<EPI>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, g, ncols);
        return 0;
    }
    return g.ksplit;
}

// Column blocks a workgroup of k_gemv_bf16 takes, with mt > 1 token groups: every workgroup fetches the whole token operand, a KB per
// group and k-step, next to a KB per column block, and a CU takes in about 50 GB/s of the two, so the fewest KB per CU are taken
// (several blocks where that still leaves one round of workgroups).  Per launch, one block -> the rule's choice, 52 tokens of width
// 4096 from the weight copy, us: q|k|v 43.4 -> 29.4 (3 blocks), gate|up 48.1 -> 34.9 (3), lm-head 48.7 -> 34 (4).
inline int gemv_blocks(int blocks, int mt, int na) {
    int best = 1, best_cost = 0x7fffffff;
    for (int nb = 1; nb <= (na == 2 ? 3 : 4); ++nb) {
        const int wgs = (blocks + nb - 1) / nb, rounds = (wgs + cu_count() - 1) / cu_count(), cost = rounds * (nb * na + mt);
        if (cost < best_cost) { best = nb; best_cost = cost; }
    }
    return best;
}

// returns how many slices of K the projection left in g.ksums (RESID: for the norm behind it; 0: the sums are where they belong)
template <int EPI>
int run_gemv(GemmArgs g, hipStream_t st) {
    if (shares_tokens(g.M, g.w_frag))   // several token groups: the token operand goes through LDS
        return run_gemv_shared<EPI>(g, st);
    if (g.M > STREAM_MAX_TOKENS) {   // the kernel below holds four token groups
        note_hip_error(hipErrorInvalidValue);
        return 0;
    }
    const int cols = EPI == EPI_SWIGLU ? g.N / 2 : g.N, mt = (g.M + 15) / 16;
    if constexpr (EPI == EPI_SWIGLU) {
        // One token group: 8 feed-forward columns a workgroup where 16 would be more than a round of CUs.  It is the same bytes in
        // twice the workgroups, so the last ones leave less of the chip waiting (width 4096, 11008 columns, one token: 40.2 -> 35.0 us,
        // from the copy, four tokens, 35.2 -> 32.6); with fewer the tokens are fetched twice as often for nothing (8 layers of
        // width 1024, 2816 columns, 16 tokens: 340 us with 16 columns, 354 with 8).
        if (mt == 1 && (cols + 15) / 16 > cu_count()) {
            const dim3 grid((cols + 7) / 8);
            if (g.w_frag) hipLaunchKernelGGL((k_gemv_bf16<EPI, 1, UNIT_HALF, true>), grid, dim3(512), 0, st, g);
            else hipLaunchKernelGGL((k_gemv_bf16<EPI, 1, UNIT_HALF, false>), grid, dim3(512), 0, st, g);
            return 0;
        }
    }
    if constexpr (EPI == EPI_RESID) {
        g.ksplit = stream_slices(g.M, g.N, g.K, g.w_frag, true);
        if (g.ksplit) {
            // 64 columns a workgroup where 128 leave CUs idle, and for weights as they come, whose lane exchanges want the wavefronts
            // in more workgroups (52 tokens, 8 layers of width 2048 614 -> 580 us, from the copy 544 -> 527; width 4096 1133 -> 1120);
            // 128 of the copy's where those fill the chip (977 -> 968)
            const bool wide = g.w_frag && (g.N + 127) / 128 * g.ksplit >= cu_count();
            auto launch = [&](auto mtc) {
                constexpr int MT = decltype(mtc)::value;
                if (wide) return launch_gemv_shared<MT, true, 8>(g, g.N, g.N, st);
                else if (g.w_frag) return launch_gemv_shared<MT, true, 4>(g, g.N, g.N, st);
                else return launch_gemv_shared<MT, false, 4>(g, g.N, g.N, st);
            };
            const bool ok = mt == 2 ? launch(std::integral_constant<int, 2>{}) : mt == 3 ? launch(std::integral_constant<int, 3>{})
                                                                                        : launch(std::integral_constant<int, 4>{});
            return ok ? g.ksplit : 0;
        }
    }
    const int blocks = (cols + 15) / 16;
    const int nb = mt == 1 ? 1 : gemv_blocks(blocks, mt, EPI == EPI_SWIGLU ? 2 : 1);
    auto launch = [&](auto mtc, auto nbc) {
        constexpr int MT = decltype(mtc)::value, NB = decltype(nbc)::value;
        const dim3 grid((blocks + NB - 1) / NB);
        if (g.w_frag) hipLaunchKernelGGL((k_gemv_bf16<EPI, MT, NB, true>), grid, dim3(512), 0, st, g);
        else hipLaunchKernelGGL((k_gemv_bf16<EPI, MT, NB, false>), grid, dim3(512), 0, st, g);
    };
    auto with_groups = [&](auto nbc) {
        if (mt == 2) launch(std::integral_constant<int, 2>{}, nbc);
        else if (mt == 3) launch(std::integral_constant<int, 3>{}, nbc);
        else launch(std::integral_constant<int, 4>{}, nbc);
    };
    if (mt == 1) {
        launch(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
        return 0;
    }
    if (nb == 1) with_groups(std::integral_constant<int, 1>{});
    else if (nb == 2) with_groups(std::integral_constant<int, 2>{});
    else if (nb == 3) with_groups(std::integral_constant<int, 3>{});
    else if constexpr (EPI != EPI_SWIGLU) with_groups(std::integral_constant<int, 4>{});
    return 0;
}

// one thread per 16-byte piece of the copy: piece p of block (nb, s) is lane p % 64
__global__ __launch_bounds__(256) void k_pack_weights(const bf16* __restrict__ src, bf16* __restrict__ dst, int layers,
                                                      int rows, int K) {
    const int steps = K / 32, nb_per = (rows + 15) / 16;
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x, total = (int64_t)layers * nb_per * steps * 64;
    if (p >= total) return;
    const int lane = (int)(p & 63);
    const int64_t blk = p >> 6;
    const int s = (int)(blk % steps);
    const int64_t nbl = blk / steps;                     // (layer, 16-row block)
    const int layer = (int)(nbl / nb_per), nb = (int)(nbl % nb_per);
    const int row = nb * 16 + (lane & 15), k = s * 32 + (lane >> 4) * 8;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (row < rows) v = *reinterpret_cast<const u32x4*>(src + ((int64_t)layer * rows + row) * K + k);
    *reinterpret_cast<u32x4*>(dst + p * 8) = v;
}

// ---- which tile a launch runs on ----
// Every tile adds the same products in the same order, so the choice is about time alone.  Time of a launch of T tiles on
// S = per_cu x CUs places: c0 + e per round + (K / 64) x (tf per full round; a last round of r tiles between
// t0, where few CUs fetch, and tf: t0 + (tf - t0) r / S).  per_cu is what the LDS holds, but 1 for 32 x 64, of which two fit:
// with 257 tiles the CU that has two of them takes twice the bytes, and the fit knows (4096 x 4096: 128 tokens, 256 tiles, 18 us
// against 22 on 64 x 64; 256 tokens, 512 tiles, 28 against 23).  The constants (us) are fitted over 40 token
// counts from 72 to 4096 and the ten projection shapes of the two bf16 configurations (widths 1024 and 4096), cold weights, for the picks
// first and the times second (so a cost of a round may be below 0), with no pick slower than the one of the rule before: the picks
// take 0.6 % longer than the best tile on average, 20 of 400 more than 5 %; with the least squares fit to the times alone that was
// here before 1.5 % and 43.  Widths that were not fitted, 1536, 2048, 3072 and 5120: 1.0 % and 26 of 320, with the fit before
// 1.3 % and 33; slower than its picks by up to 8 % at width 2048 (q|k|v and lm-head of 288 to 384 tokens), faster by up to 12 % at
// 1536.  The worst are the lm-head of 72 to 128 tokens of width 4096 (51 us on 64 x 64 against 40 on 128 x 64);
// 260 to 320 tokens of that width went from 66 to 52 us (q|k|v, 256 x 128 for 64 x 64) and from 97 to 77 (gate|up, 256 x 256 for 64 x 128).
struct TileCost {
    int bm, bn, stages, per_cu;   // ring stages of bm + bn rows of 128 bytes; 256 x 256: 0, it has a ring of its own
    float c0, tf, t0, e;
    constexpr int fit() const { return 160 * 1024 / (stages ? stages * (bm + bn) * 128 : LDS_256); }
};
enum { TILE_32x64, TILE_64x64, TILE_128x64, TILE_64x128, TILE_128x128, TILE_256x128, TILE_128x256, TILE_256x256, N_TILES };
constexpr TileCost TILE_COST[N_TILES] = {
    {32, 64, 6, 1, 6.12f, 0.184f, 0.116f, -0.38f}, {64, 64, 5, 2, 3.07f, 0.406f, 0.154f, 2.79f},
    {128, 64, 3, 2, 1.6f, 0.761f, 0.368f, 3.95f},  {64, 128, 3, 2, 4.34f, 0.64f, 0.24f, 4.76f},
    {128, 128, 5, 1, 5.17f, 0.487f, 0.45f, 3.35f}, {256, 128, 3, 1, 5.59f, 0.766f, 0.488f, 4.37f},
    {128, 256, 3, 1, 12.65f, 0.796f, 0.686f, -0.34f}, {256, 256, 0, 1, 11.33f, 1.263f, 0.822f, 0.37f}};
constexpr bool tiles_fit() {
    for (int i = 0; i < N_TILES; ++i)
        if (TILE_COST[i].fit() != (i == TILE_32x64 ? 2 : TILE_COST[i].per_cu)) return false;
    return true;
}
static_assert(tiles_fit(), "workgroups per CU");

// Column tiles of a 256 x 256 launch that run as such: a last round that would leave more than half of the CUs idle is
// cut off and runs as 128 x 256 tiles (twice as many workgroups, half the work each).
inline int whole_columns(const GemmArgs& g) {
    const int tiles_m = (g.M + 255) / 256, tiles_n = g.N / 256, cus = cu_count(), total = tiles_m * tiles_n, rem = total % cus;
    int n = tiles_n;
    if (total > cus && rem > 0 && 2 * rem <= cus) n = (total - rem) / tiles_m;
    return (tiles_n - n) * tiles_m * 2 > cus ? tiles_n : n;   // the cut-off part must fit one round
}

// which tiles a projection has
template <int EPI>
bool has_tile(const GemmArgs& g, int i) {
    const int seg = EPI == EPI_QKV ? g.d : g.N;                           // a tile must not straddle two of q | k | v
    if (i == TILE_256x256 && !(g.N % 256 == 0 && seg % 256 == 0 &&
                               (int64_t)256 * (g.N > g.K ? g.N : g.K) * 4 < (1ll << 31)))   // 32-bit offsets inside a tile's rows
        return false;
    if (EPI == EPI_QKV && seg % TILE_COST[i].bn) return false;
    return EPI == EPI_SWIGLU ? i != TILE_32x64 && i != TILE_64x64 && i != TILE_128x64 : i != TILE_64x128;
}

template <int EPI>
int choose_tile(const GemmArgs& g) {
    int best = -1;
    float best_us = 0.f;
    for (int i = 0; i < N_TILES; ++i) {
        const TileCost& t = TILE_COST[i];
        if (!has_tile<EPI>(g, i)) continue;
        const int64_t places = (int64_t)t.per_cu * cu_count();
        int64_t tiles = (int64_t)((g.M + t.bm - 1) / t.bm) * ((g.N + t.bn - 1) / t.bn);
        float us = t.c0;
        if (i == TILE_256x256) {                                        // the cut-off columns are half a tile's time
            const int64_t whole = (int64_t)((g.M + 255) / 256) * whole_columns(g);
            if (whole < tiles) us += 0.5f * (t.e + t.tf * (g.K / 64));
            tiles = whole;
        }
        const int64_t full = tiles / places, r = tiles % places;
        const float part = r ? t.t0 + (t.tf - t.t0) * ((float)r / (float)places) : 0.f;
        us += t.e * (float)(full + (r > 0)) + (float)(g.K / 64) * (t.tf * (float)full + part);
        // softmax parts come from wavefront tiles of 128 columns only; without them the accept test reads the logits
        if (EPI == EPI_LOGITS && g.parts && !(t.bn == 256 && g.N % 256 == 0)) us += (float)g.M * (float)g.N * 4.f / 5e6f;
        if (best < 0 || us < best_us) { best = i; best_us = us; }
    }
    return best;
}

// all columns, or column tiles [tile_n0, tile_n0 + tiles_n)
template <int TILE, int WGM, int WGN, int EPI, bool PAIRED = false>
void run_ring(GemmArgs g, hipStream_t st, int tile_n0 = 0, int tiles_n = 0) {
    constexpr int BM = TILE_COST[TILE].bm, BN = TILE_COST[TILE].bn, NS = TILE_COST[TILE].stages;
    auto kern = k_gemm_ring<BM, BN, WGM, WGN, NS, EPI, PAIRED>;
    const size_t lds = (size_t)NS * (BM + BN) * 128;
    static int attr_state = 0;
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)lds, &attr_state)) return;
    g.tiles_n = tiles_n ? tiles_n : (g.N + BN - 1) / BN;
    g.tile_n0 = tile_n0;
    const int64_t total = (int64_t)((g.M + BM - 1) / BM) * g.tiles_n;
    hipLaunchKernelGGL(kern, dim3((unsigned)((total + 7) / 8 * 8)), dim3(WGM * WGN * 64), lds, st, g);
}

// returns whether the softmax parts were written (LOGITS, wavefront tiles of 128 whole columns), or how many K slices a streamed
// launch left for the norm behind it to add (RESID)
template <int EPI>
int dispatch(GemmArgs g, const StreamMode& sm, hipStream_t st) {
    g.stream = sm.stream; g.w_frag = sm.w_frag; g.ksums = sm.ksums; g.ksum_floats = sm.ksum_floats;
    *sm.ran = -1;
    if (g.stream) {   // a handful of tokens: stream the weights (A is in fragment order)
        return run_gemv<EPI>(g, st);
    }
    const int tile = sm.tile >= 0 && sm.tile < N_TILES && has_tile<EPI>(g, sm.tile) ? sm.tile : choose_tile<EPI>(g);
    *sm.ran = tile;
    const bool parts = EPI == EPI_LOGITS && g.parts && TILE_COST[tile].bn == 256 && g.N % 256 == 0;
    if (!parts) g.parts = nullptr;
    auto run_128x256 = [&](int n0, int n) {
        if constexpr (EPI == EPI_SWIGLU || EPI == EPI_LOGITS) run_ring<TILE_128x256, 2, 2, EPI>(g, st, n0, n);
        else run_ring<TILE_128x256, 2, 4, EPI>(g, st, n0, n);
    };
    switch (tile) {
        case TILE_32x64: if constexpr (EPI != EPI_SWIGLU) run_ring<TILE_32x64, 1, 2, EPI>(g, st); break;
        case TILE_64x64: if constexpr (EPI != EPI_SWIGLU) run_ring<TILE_64x64, 2, 2, EPI>(g, st); break;
        case TILE_128x64: if constexpr (EPI != EPI_SWIGLU) run_ring<TILE_128x64, 2, 2, EPI>(g, st); break;
        case TILE_64x128: if constexpr (EPI == EPI_SWIGLU) run_ring<TILE_64x128, 2, 2, EPI>(g, st); break;
        case TILE_128x128: run_ring<TILE_128x128, 2, 2, EPI, true>(g, st); break;
        case TILE_256x128:   // 4 wavefronts of 128 x 64 (1980 x 4096 x 11008: 152 us against 157 with 8 of 64 x 64), q|k|v and lm-head 8
            if constexpr (EPI == EPI_SWIGLU || EPI == EPI_RESID) run_ring<TILE_256x128, 2, 2, EPI>(g, st);
            else run_ring<TILE_256x128, 4, 2, EPI>(g, st);
            break;
        case TILE_128x256: run_128x256(0, 0); break;
        default: {
            const int tiles_n = g.N / 256, n_main = whole_columns(g);
            if constexpr (EPI == EPI_LOGITS) {
                if (parts) run_256<EPI, true>(g, 0, n_main, st);
                else run_256<EPI, false>(g, 0, n_main, st);
            } else {
                run_256<EPI, false>(g, 0, n_main, st);
            }
            if (n_main < tiles_n) run_128x256(n_main, tiles_n - n_main);
        }
    }
    return parts ? 1 : 0;
}

}  // namespace

int cu_count() {
    static int n = 0;
    if (n == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) n = prop.multiProcessorCount;
        if (n <= 0) n = 256;
    }
    return n;
}

void launch_gemm_qkv_bf16(const void* xh, const void* wq, const void* wk, const void* wv, void* q_out,
                          void* k_cache, void* v_cache, int M, int d, const RopeArgs& ra, const StreamMode& sm, hipStream_t st) {
    GemmArgs g{};
    g.A = (const bf16*)xh; g.W0 = (const bf16*)wq; g.W1 = (const bf16*)wk;
    g.M = M; g.N = 3 * d; g.K = d; g.Cb = (bf16*)q_out; g.kc = (bf16*)k_cache; g.d = d; g.ra = ra;
    g.W2 = (const bf16*)wv; g.vc = (bf16*)v_cache;
    dispatch<EPI_QKV>(g, sm, st);
}

Slices launch_gemm_resid_bf16(const void* a, const void* w, float* x, int M, int N, int K, const StreamMode& sm, hipStream_t st) {
    GemmArgs g{};
    g.A = (const bf16*)a; g.W0 = (const bf16*)w; g.M = M; g.N = N; g.K = K; g.Cf = x;
    return {sm.ksums, dispatch<EPI_RESID>(g, sm, st)};
}

void launch_gemm_swiglu_bf16(const void* xh, const void* wg, const void* wu, void* h, int M, int f, int d,
                             const StreamMode& sm, hipStream_t st) {
    GemmArgs g{};
    g.A = (const bf16*)xh; g.W0 = (const bf16*)wg; g.W1 = (const bf16*)wu; g.M = M; g.N = 2 * f; g.K = d;
    g.Cb = (bf16*)h;
    dispatch<EPI_SWIGLU>(g, sm, st);
}

bool launch_gemm_logits_bf16(const void* xh, const void* w, float* logits, float* parts, int M, int V, int d,
                             const StreamMode& sm, hipStream_t st) {
    GemmArgs g{};
    g.A = (const bf16*)xh; g.W0 = (const bf16*)w; g.M = M; g.N = V; g.K = d; g.Cf = logits;
    g.parts = reinterpret_cast<float2*>(parts);
    g.n_parts = (V + rowparts::PART - 1) / rowparts::PART;
    return dispatch<EPI_LOGITS>(g, sm, st) != 0 && parts != nullptr;
}

void launch_pack_weights(const void* src, void* dst, int layers, int rows, int K, hipStream_t st) {
    const int64_t pieces = (int64_t)layers * ((rows + 15) / 16) * (K / 32) * 64;
    hipLaunchKernelGGL(k_pack_weights, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st, (const bf16*)src, (bf16*)dst,
                       layers, rows, K);
}

}  // namespace mulo
