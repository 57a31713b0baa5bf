// Causal attention of the drafted block over prefix + block (Alg. 1 Step 3: the
// j-th conditional sees cache rows 0 .. P+j).
//
// bf16 path: flash-style, one workgroup per (128 or 256 queries, head, sequence),
// 8 wavefronts (two per SIMD) for 256; K and V^T tiles of 64 or 128 keys (run_attn's
// rule) go from memory to LDS directly (double buffered, 128 KB for 128 keys of a head
// of 128) and are shared by the wavefronts, so a tile is fetched once per workgroup and
// the per-tile work (barrier, running maximum, rescale test) is spread over up to 32
// MFMAs per product; each wavefront owns 32 queries and computes
// S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x16_bf16, so that a lane
// owns ONE query: the softmax row reductions stay inside the lane (plus one
// cross-half shuffle), and the exponentiated scores are already laid out as the
// B operand of the second product.  The K rows are fetched in a permuted order
// (bits 2 and 3 of the row index swapped) so that a lane's accumulators cover 8
// consecutive keys, which is what lets V^T be read with 16-byte LDS loads.
#include <hip/hip_bf16.h>

#include <utility>

#include "mulo_internal.h"

namespace mulo {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __hip_bfloat16 bf16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void glb_void;

constexpr float LOG2E = 1.4426950408889634f;

// compile-time loop: register arrays indexed by it stay in registers
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}
// a descriptor of `bytes` bytes at p (<= 0: nothing; reads outside give zeros)
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)(bytes < 0 ? 0 : bytes < 0x7fffffff ? bytes : 0x7fffffff), 0x00020000);
}

struct AttnArgs {
    const bf16* q;    // [B, nh, L, dh]
    const bf16* kc;   // [nl, maxB, nh, S, dh]
    const bf16* vc;   // [nl, maxB, nh, dh, S]
    bf16* out;        // [B*L, nh*dh]
    int frag;         // out is the token operand of a weight-streaming projection: fragment order (frag_index)
    int B, L, P, nh, max_seq, max_batch, layer;
    float scale_log2;  // log2(e) / sqrt(dh)
    int nsplit;        // > 1: the keys are dealt to nsplit workgroups per (sequence, head); one query tile only
    float* part;       // [nsplit, B, nh, L][dh + 2]: unnormalised output of a query, running maximum, running sum (L <= 32)
    // scattered queries (island passes): query j of sequence b (L slots per sequence) sits at cache row
    // pos_tab[b * L + j] in [P0, P0 + Lblk) (< 0: unused slot) and does not see rows P0 + t of its sequence with
    // hide[b, t] set, its own excepted
    const int32_t* pos_tab;
    const uint8_t* hide;   // [B, Lblk]
    int P0, Lblk;
};
constexpr float LAZY_EXP = 8.0f;     // 4 x 1024 queries against 4096 keys: 0 -> 278 and 281, 8 -> 278 and 273 us, within the noise of a card
constexpr int MAX_SPLIT = 16;
constexpr int NS_TARGET = 512;      // workgroups a key split aims at (a token of 4 sequences of 4000 rows, 32 heads of 128, us in front of the
                                    // combine: 256 -> 58, 512 -> 49, 1024 -> 51, 2048 -> 54)
constexpr int SPLIT_QUERIES = 32;   // a key split serves at most this many queries per (sequence, head)

// two workgroups per CU where their LDS fits twice (2 x 64 KB: 64-key tiles of heads of 128, 128-key tiles of heads of 64)
template <int DH, int BQ, int BKV, int NTH>
__global__ __launch_bounds__(NTH, DH * BKV <= 8192 ? 2 : 1) void k_attn_bf16(const AttnArgs a) {
    constexpr int NKK = DH / 16;   // k-steps of the first product
    constexpr int NDB = DH / 32;   // 32-row blocks of O^T
    constexpr int NKB = BKV / 32;  // 32-key blocks of S^T
    constexpr int NW = NTH / 64;
    constexpr int KRB = DH * 2, VRB = BKV * 2;                            // bytes of a row of the K tile, of the V^T tile
    constexpr int KT = BKV * KRB, BUF = KT + DH * VRB;                    // the K tile, then the V^T tile
    constexpr int LK = KT / 1024 / NW, LV = DH * VRB / 1024 / NW;         // loads of a wavefront per tile, a KB of whole rows each
    constexpr int RK = 1024 / KRB, RV = 1024 / VRB;                       // rows of a load
    static_assert(LK * NW * 1024 == KT && LV * NW * 1024 == DH * VRB, "whole loads per wavefront");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // [2][BUF]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, lh = lane >> 5;
    // Workgroup id -> (query tile, head).  Consecutive ids go to consecutive XCDs, each with its own L2:
    // all query tiles of one (batch, head) are given to ONE XCD, next to each other in its dispatch
    // order, so that they stream that head's K and V through the same L2 side by side (the cache rows
    // are fetched from memory once per head instead of once per query tile).  Long tiles go first.
    const int qtiles = (a.L + BQ - 1) / BQ, nbh = a.B * a.nh;
    const int split = blockIdx.x / (qtiles * nbh), bid = blockIdx.x % (qtiles * nbh);
    int qt, bh;
    if ((nbh & 7) == 0) {
        const int xcd = bid & 7, s = bid >> 3;
        qt = qtiles - 1 - s % qtiles;
        bh = (s / qtiles) * 8 + xcd;
    } else {
        qt = qtiles - 1 - bid % qtiles;
        bh = bid / qtiles;
    }
    const int j0 = qt * BQ, hd = bh % a.nh, b = bh / a.nh;
    // scattered queries run in the short-block configuration only; the long-block one keeps its registers
    const bool scattered = BKV == 64 && a.pos_tab != nullptr;
    const int P = a.P;
    const int64_t hb = ((int64_t)a.layer * a.max_batch + b) * a.nh + hd;
    const bf16* kbase = a.kc + hb * a.max_seq * DH;
    const bf16* vbase = a.vc + hb * DH * a.max_seq;

    // this lane's query (clamped for the ragged last tile; such lanes do not store)
    const int jq_raw = j0 + wave * 32 + l32;
    const int jq = jq_raw < a.L ? jq_raw : a.L - 1;
    int qpos = P + jq;
    bool active = true;
    if (scattered) {   // the slot's own cache row; an unused slot computes on row P0 and stores zeros
        const int row = a.pos_tab[(int64_t)b * a.L + jq];
        active = row >= 0;
        qpos = active ? row : a.P0;
    }
    const int wave_jmin = j0 + wave * 32;
    int wave_jmax = wave_jmin + 31;
    wave_jmax = wave_jmax < a.L ? wave_jmax : a.L - 1;
    const bool wave_live = wave_jmin < a.L;

    bf16x8 qf[NKK];
    {
        const bf16* qp = a.q + (((int64_t)b * a.nh + hd) * a.L + jq) * DH + lh * 8;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16);
    }

    int blk_jmax = j0 + BQ - 1;
    blk_jmax = blk_jmax < a.L ? blk_jmax : a.L - 1;
    const int kmax_blk = scattered ? a.P0 + a.Lblk - 1 : P + blk_jmax;   // last key any query of this workgroup may see
    const int n_tiles = kmax_blk / BKV + 1;
    // key split (single-token decoding, island passes: at most 32 queries, one wavefront): this workgroup covers
    // tiles [t_begin, t_end) and leaves its unnormalised partial results (output, running maximum, running sum)
    // for k_attn_combine
    const int tiles_per = (n_tiles + a.nsplit - 1) / a.nsplit;
    const int t_begin = split * tiles_per, t_end = t_begin + tiles_per < n_tiles ? t_begin + tiles_per : n_tiles;
    float* part = a.nsplit > 1 ? a.part + (((int64_t)split * a.B + b) * a.nh + hd) * a.L * (DH + 2) : nullptr;
    if (t_begin >= t_end) {    // uniform over the workgroup, before any barrier: an empty share
        if (part) {
            for (int c = tid; c < a.L * (DH + 2); c += NTH) {
                const int e = c % (DH + 2);
                part[c] = e == DH ? -__builtin_huge_valf() : 0.f;
            }
        }
        return;
    }

    // Tiles go from memory to LDS directly.  16-byte chunk c of row r sits at chunk position c ^ key(r): 16 lanes that read
    // the same chunk of 16 rows touch every bank once.  (Rows of 128 bytes lie two to a 256-byte line of banks.)
    auto key_of = [](int r, int row_bytes) { return row_bytes == 256 ? r & 15 : (r >> 1) & 7; };
    const int krow = wave * RK + lane / (64 / RK), vrow = wave * RV + lane / (64 / RV);   // this lane's row in load 0 (the key repeats: NW RK, NW RV are multiples of 16)
    const int kchunk = lane % (64 / RK) ^ key_of(krow, KRB), vchunk = lane % (64 / RV) ^ key_of(vrow, VRB);
    static_assert(NW * RK % 16 == 0 && NW * RV % 16 == 0, "the key of a lane's rows");
    // A tile that runs past the end of the cache takes the last row and columns again: nothing sees those keys (max_seq is a multiple
    // of 8, a tile begins in front of it).  One scalar address per operand and tile and a lane offset, not a descriptor per load:
    // building those took about 180 scalar instructions and lane reads a tile, which a CU with one workgroup has nothing to hide
    // behind (32 heads of 128, us: 98 queries, 2949 keys 86 -> 68, 4 x 128, 3128 keys 90 -> 73, 1 x 576, 1856 keys 45 -> 43,
    // 4 x 1024, 4224 keys 272 -> 264).
    const int max_seq = a.max_seq;
    const uint32_t voff = (uint32_t)(lane / (64 / RV)) * (uint32_t)max_seq * 2u;
    const unsigned char* const kbytes = reinterpret_cast<const unsigned char*>(kbase);
    const unsigned char* const vbytes = reinterpret_cast<const unsigned char*>(vbase + (int64_t)wave * RV * max_seq);
    const int64_t vstep = (int64_t)NW * RV * max_seq * 2;   // bytes from a load to the next
    auto to_lds = [](const unsigned char* base, uint32_t off, unsigned char* lds) {
        __builtin_amdgcn_global_load_lds((glb_void*)(base + off), (lds_void*)lds, 16, 0, 0);
    };
    auto load_kv = [&](int t) {
        unsigned char* const lds = smem + (t & 1) * BUF + wave * 1024;
        const unsigned char* const kt = kbytes + (int64_t)t * (BKV * KRB);
        const unsigned char* const vt = vbytes + (int64_t)t * VRB;
        const int left = max_seq - t * BKV;   // rows of the cache from the tile's first on
#pragma unroll
        for (int i = 0; i < LK; ++i) {
            const int row = krow + i * NW * RK;
            to_lds(kt, (uint32_t)(row < left ? row : left - 1) * KRB + kchunk * 16, lds + i * NW * 1024);
        }
        const uint32_t vo = voff + (uint32_t)(vchunk * 8 < left - 8 ? vchunk * 8 : left - 8) * 2u;
#pragma unroll
        for (int i = 0; i < LV; ++i) to_lds(vt + i * vstep, vo, lds + KT + i * NW * 1024);
    };
    // this wavefront's loads have landed and its fragment reads are done; meet the others
    auto meet = [&]() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // Cache columns past the last visible key may be uninitialised memory: their probabilities are 0, and 0 * NaN must not
    // reach the accumulators.  Between the landing of tile t's V^T and the barrier that shows it to the others, every lane
    // clears those of the bytes it has loaded itself.
    auto clear_unseen = [&](int t) {
        if (t * BKV + BKV - 1 > kmax_blk) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const int key = t * BKV + vchunk * 8;
            auto keep = [&](int e) -> uint32_t { return (key + e <= kmax_blk ? 0xFFFFu : 0u) | (key + e + 1 <= kmax_blk ? 0xFFFF0000u : 0u); };
#pragma unroll
            for (int i = 0; i < LV; ++i) {
                u32x4* const at = reinterpret_cast<u32x4*>(smem + (t & 1) * BUF + KT + (i * NW + wave) * 1024 + lane * 16);
                u32x4 v = *at;
                v.x &= keep(0); v.y &= keep(2); v.z &= keep(4); v.w &= keep(6);
                *at = v;
            }
        }
    };

    f32x16 o[NDB];
#pragma unroll
    for (int i = 0; i < NDB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
    float m_run = -__builtin_huge_valf(), l_run = 0.f;

    // MFMA row rho of a K block is fed key kperm(rho): bits 2 and 3 swapped
    const int kperm = (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);

    // Hidden rows (scattered queries): one flag per lane and 64-key tile (lane i: key 64 t + i), requested in front of the
    // tile's K and V loads and turned into a 64-bit mask by a ballot where those have to have landed anyway.  (Loads return
    // in order: requested behind them and used in the middle of the tile before, the flag held that tile's softmax and output
    // product back until the next tile had landed: 4 x 13 slots of 32 heads of 128, 4224 rows 69 -> 59 us, 16 x 10 slots
    // 230 -> 216; single tokens of 4 sequences, which hide nothing, 51.)
    // A row outside the block lies outside the descriptor: 0.
    const rsrc_t hide_rows = make_rsrc(a.hide ? a.hide + (int64_t)b * a.Lblk : nullptr, a.hide ? a.Lblk : 0);
    auto hide_flag = [&](int tile) -> uint32_t {
        const int tpos = tile * BKV + lane - a.P0;
        return __builtin_amdgcn_raw_buffer_load_b8(hide_rows, tpos >= 0 && tpos < a.Lblk ? tpos : -1, 0, 0);
    };
    unsigned long long hide_cur = 0;
    if constexpr (BKV == 64) {
        if (a.hide && wave_live) hide_cur = __ballot(hide_flag(t_begin) != 0);
    }
    // fragment addresses inside a tile: chunk 2 k + lh of this lane's row, k in bits 5 and up
    const int kfrag = kperm * KRB + (lh ^ key_of(kperm, KRB)) * 16, vfrag = l32 * VRB + (lh ^ key_of(l32, VRB)) * 16;
    f32x16 s[NKB];               // the scores of a tile, then
    float m_safe = 0.f, alpha = 1.f;   // the reference of its exponentials and the factor of what has been added up before it
    auto score = [&](int t) {
        const int kv0 = t * BKV;
        const unsigned char* const kt = smem + (t & 1) * BUF;
        // S^T = K Q^T: NKB independent chains, the fragments of a k-step requested during the step before it (left to
        // itself the compiler keeps two fragments in flight and waits for each: the product took 3 times its MFMAs)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
        bf16x8 kf[2][NKB];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) kf[0][kb] = *reinterpret_cast<const bf16x8*>(kt + kfrag + kb * 32 * KRB);
        static_for<NKK>([&](auto kc) {
            constexpr int kk = decltype(kc)::value;
            static_for<NKB>([&](auto bc) {
                constexpr int kb = decltype(bc)::value;
                if constexpr (kk + 1 < NKK) kf[(kk + 1) & 1][kb] = *reinterpret_cast<const bf16x8*>(kt + (kfrag ^ ((kk + 1) << 5)) + kb * 32 * KRB);
                s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk & 1][kb], qf[kk], s[kb], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        // accumulator r of block kb holds key kv0 + kb*32 + 16*(r/8) + 8*lh + r%8 for query l32
        const bool need_mask = scattered ? kv0 + BKV > a.P0 : kv0 + BKV - 1 > P + wave_jmin;
        float mx = -__builtin_huge_valf();
        if (need_mask) {
#pragma unroll
            for (int kb = 0; kb < BKV / 32; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kv0 + kb * 32 + 16 * (r >> 3) + 8 * lh + (r & 7);
                    s[kb][r] = key <= qpos ? s[kb][r] : -__builtin_huge_valf();
                }
        }
        if constexpr (BKV == 64) {
            if (hide_cur != 0) {   // scattered queries: rows of positions that are not settled yet (the query's own excepted);
                                   // uniform over the wavefront; bits are set for rows of the block only
#pragma unroll
                for (int kb = 0; kb < BKV / 32; ++kb) {
                    const uint32_t mine = (uint32_t)(hide_cur >> (kb * 32)) >> (8 * lh);   // this lane's keys: bits 16 (r / 8) + r % 8
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int key = kv0 + kb * 32 + 16 * (r >> 3) + 8 * lh + (r & 7);
                        if (((mine >> (16 * (r >> 3) + (r & 7))) & 1u) && key < qpos) s[kb][r] = -__builtin_huge_valf();
                        if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // all 64 comparisons at once need more scalars than there are
                    }
                }
            }
        }
#pragma unroll
        for (int kb = 0; kb < BKV / 32; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        // The exponentials are taken against a reference m_run (exponent units: scores times log2(e) / sqrt(dh);
        // the scale is positive) that follows the running maximum lazily: it moves only when the maximum has
        // outgrown it by more than 2^LAZY_EXP.  Probabilities then stay below that factor, which float32 and
        // bf16 hold with the same relative precision, the normalisation divides it out, and the accumulators
        // are rescaled a few times per query instead of in most tiles.  From -inf the first finite maximum
        // moves it.
        const float mxs = mx * a.scale_log2;
        const float m_new = mxs > m_run + LAZY_EXP ? mxs : m_run;
        // a query that has seen no key yet (every row of its first tiles hidden) keeps -inf as its maximum:
        // exponents are then taken against 0, which makes every term exp2(-inf) = 0 instead of NaN
        m_safe = m_new == -__builtin_huge_valf() ? 0.f : m_new;
        alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
        m_run = m_new;
    };
    auto output = [&](int t) {
        const unsigned char* const vt = smem + (t & 1) * BUF + KT;
        // O^T += V^T P^T, keys kv0 + 16 ks .. + 15 per step ks; the exponentials of step ks + 1 and its V^T fragments go
        // between the MFMAs of step ks
        float ps = 0.f;
        bf16x8 pf[2], vf[2][NDB];
        // probabilities 2 g, 2 g + 1 of the tile in three stages a slot apart, so that no instruction waits for the one before
        float x[2][2], p[2][2];
        auto arg = [&](auto gc) {
            constexpr int g = decltype(gc)::value, ks = g / 4, e = 2 * (g % 4);
            if constexpr (g < BKV / 4) {
#pragma unroll
                for (int q = 0; q < 2; ++q) x[g & 1][q] = __builtin_fmaf(s[ks >> 1][(ks & 1) * 8 + e + q], a.scale_log2, -m_safe);
            }
        };
        auto expo = [&](auto gc) {
            constexpr int g = decltype(gc)::value;
            if constexpr (g < BKV / 4) {
#pragma unroll
                for (int q = 0; q < 2; ++q) p[g & 1][q] = __builtin_amdgcn_exp2f(x[g & 1][q]);
            }
        };
        auto take = [&](auto gc) {
            constexpr int g = decltype(gc)::value, ks = g / 4, e = 2 * (g % 4);
            if constexpr (g < BKV / 4) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    ps += p[g & 1][q];
                    pf[ks & 1][e + q] = (__bf16)p[g & 1][q];
                }
            }
        };
#pragma unroll
        for (int i = 0; i < NDB; ++i) vf[0][i] = *reinterpret_cast<const bf16x8*>(vt + vfrag + i * 32 * VRB);
        static_for<4>([&](auto gc) { arg(gc); expo(gc); take(gc); });
        arg(std::integral_constant<int, 4>{});
        expo(std::integral_constant<int, 4>{});
        arg(std::integral_constant<int, 5>{});
        // the accumulators are rescaled only when some query of the wavefront raised its maximum
        if (!__all(alpha == 1.0f)) {
#pragma unroll
            for (int i = 0; i < NDB; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[i][r] *= alpha;
        }
        static_for<BKV / 16>([&](auto kc) {
            constexpr int ks = decltype(kc)::value, nxt = ks + 1 < BKV / 16 ? ks + 1 : ks;
            static_for<NDB>([&](auto ic) {
                constexpr int i = decltype(ic)::value, n = 4 / NDB;   // pairs per slot
                if constexpr (nxt > ks) vf[nxt & 1][i] = *reinterpret_cast<const bf16x8*>(vt + (vfrag ^ (nxt << 5)) + i * 32 * VRB);
                static_for<n>([&](auto qc) {
                    constexpr int g = 4 * ks + i * n + decltype(qc)::value + 4;
                    take(std::integral_constant<int, g>{});
                    expo(std::integral_constant<int, g + 1>{});
                    arg(std::integral_constant<int, g + 2>{});
                });
                o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[ks & 1][i], pf[ks & 1], o[i], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        l_run = l_run * alpha + ps;
    };
    load_kv(t_begin);
    clear_unseen(t_begin);
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) asm volatile("" : "+v"(qf[kk]));   // wait for the queries here: among the tiles' loads that wait is for those as well
    meet();
    for (int t = t_begin; t < t_end; ++t) {
        uint32_t hide_next = 0;
        if (t + 1 < t_end) {   // everybody has read the buffer: the barrier at the end of the tile before
            if constexpr (BKV == 64) {
                if (a.hide && wave_live) hide_next = hide_flag(t + 1);
            }
            load_kv(t + 1);
        }
        if (wave_live && (scattered || t * BKV <= P + wave_jmax)) {
            score(t);
            output(t);
        }
        if (t + 1 < t_end) {
            if constexpr (BKV == 64) {
                asm volatile("" : "+v"(hide_next));   // left alone, the compiler tests the flag, and waits for it, before the tile's loads go out
                hide_cur = __ballot(hide_next != 0);
            }
            clear_unseen(t + 1);
            meet();
        }
    }

    l_run += __shfl_xor(l_run, 32);
    if (part) {
        if (wave == 0 && jq_raw < a.L) {     // the tile's queries all belong to the first wavefront
            float* pq = part + (int64_t)jq * (DH + 2);
#pragma unroll
            for (int i = 0; i < NDB; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) pq[i * 32 + (r >> 2) * 8 + lh * 4 + (r & 3)] = o[i][r];
            if (lh == 0) { pq[DH] = m_run; pq[DH + 1] = l_run; }
        }
        return;
    }
    if (jq_raw < a.L) {
        const float inv = 1.0f / l_run;
        const int row = b * a.L + jq;
        bf16* op = a.out + (int64_t)row * (a.nh * DH) + hd * DH;
#pragma unroll
        for (int i = 0; i < NDB; ++i)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                bf16x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = (__bf16)(active ? o[i][g4 * 4 + e] * inv : 0.f);
                const int c = i * 32 + g4 * 8 + lh * 4;   // 4 | c: the four channels share a run of 8
                *reinterpret_cast<bf16x4*>(a.frag ? a.out + frag_index(row, hd * DH + c, a.nh * DH) : op + c) = w;
            }
    }
}

// out[b, hd, :] = sum_s o_s 2^(m_s - M) / sum_s l_s 2^(m_s - M), M = max_s m_s (maxima are in exponent units)
// One memory round trip: all NS >= nsplit shares are requested together (a loop that ends at nsplit pays one per share:
// 11 us for the 16 shares of a single sequence, now 4.7).  Shares past nsplit re-read share 0 and weigh 2^-inf = 0.
template <int DH, int NS>
__global__ __launch_bounds__(DH) void k_attn_combine(const AttnArgs a) {
    const int j = blockIdx.x % a.L, hd = (blockIdx.x / a.L) % a.nh, b = blockIdx.x / (a.L * a.nh), c = threadIdx.x;
    float o[NS], m[NS], l[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const float* p = a.part + ((((int64_t)(s < a.nsplit ? s : 0) * a.B + b) * a.nh + hd) * a.L + j) * (DH + 2);
        o[s] = p[c];
        m[s] = p[DH];
        l[s] = p[DH + 1];
    }
    float M = -__builtin_huge_valf();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        m[s] = s < a.nsplit ? m[s] : -__builtin_huge_valf();
        M = fmaxf(M, m[s]);
    }
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const float wgt = s < a.nsplit ? __builtin_amdgcn_exp2f(m[s] - M) : 0.f;
        num += o[s] * wgt;
        den += l[s] * wgt;
    }
    const int row = b * a.L + j;
    a.out[a.frag ? frag_index(row, hd * DH + c, a.nh * DH) : (int64_t)row * (a.nh * DH) + hd * DH + c] =
        __float2bfloat16(den > 0.f ? num / den : 0.f);
}
static_assert(MAX_SPLIT == 16, "the combine kernels");

template <int DH, int BQ, int BKV, int NTH>
void run_attn_cfg(const AttnArgs& a, hipStream_t st) {
    auto kern = k_attn_bf16<DH, BQ, BKV, NTH>;
    const size_t lds = (size_t)2 * 2 * BKV * DH * sizeof(bf16);
    static int attr_state = 0;
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)lds, &attr_state)) return;
    hipLaunchKernelGGL(kern, dim3(((a.L + BQ - 1) / BQ) * a.nh * a.B * a.nsplit), dim3(NTH), lds, st, a);
    if (a.nsplit > 1) {
        const dim3 grid(a.B * a.nh * a.L);
        if (a.nsplit <= 4) hipLaunchKernelGGL((k_attn_combine<DH, 4>), grid, dim3(DH), 0, st, a);
        else if (a.nsplit <= 8) hipLaunchKernelGGL((k_attn_combine<DH, 8>), grid, dim3(DH), 0, st, a);
        else hipLaunchKernelGGL((k_attn_combine<DH, 16>), grid, dim3(DH), 0, st, a);
    }
}

// Blocks of more than SHORT_BLOCK queries run over 128-key tiles, shorter ones (single-token decoding above all) in 128-query
// workgroups of 4 wavefronts over 64-key tiles, two per CU.  The two add in another order, so which one runs depends on the
// block alone, never on the batch: given the same operands a sequence launched alone gets the bits it gets in a batch, and a
// row the same bits in every block of more than SHORT_BLOCK queries (the key split of a single token per sequence, L == 1, is
// the exception: its number of shares follows the batch).
// Over 128-key tiles a wavefront's 32 queries are added up by themselves, so the queries per workgroup do not show in the
// bits: heads of 128 take 128 (4 wavefronts) where all of those have a CU, else 256 (8 wavefronts: one workgroup per CU
// either way, 128 KB of LDS); heads of 64 take 128, two workgroups per CU.  Measured, 256 / 128 queries, us: 32 heads of 128:
// 1 x 256 queries, 3256 keys 79 / 68, 4 x 256, 3256 keys 100 / 94, 3 x 242, 2656 keys 72 / 69, 1 x 576, 1856 keys 47 / 43,
// 1 x 1024, 4024 keys 106 / 96, 1 x 384, 2795 keys 65 / 59, and past one workgroup per CU 8 x 200, 3146 keys 114 / 164,
// 4 x 1024, 4224 keys 261 / 403; 16 heads of 64: 4 x 256, 832 keys 18.3 / 14.6, 4 x 256, 3256 keys 57 / 43, 1 x 1024, 1524 keys
// 28.6 / 22.0, 16 x 1024, 2024 keys 188 / 179, but 8 x 300, 1300 keys 28.0 / 30.0 and 6 x 512, 1112 keys 25.8 / 27.3: between one
// and two workgroups per CU the line is not where these figures put it.
constexpr int BKV_SMALL = 64, SHORT_BLOCK = 128;
template <int DH>
void run_attn(const AttnArgs& a, hipStream_t st) {
    if (a.L <= SHORT_BLOCK) run_attn_cfg<DH, 128, BKV_SMALL, 256>(a, st);
    else if (DH == 64 || (int64_t)a.B * a.nh * ((a.L + 127) / 128) <= cu_count()) run_attn_cfg<DH, 128, 128, 256>(a, st);
    else if constexpr (DH == 128) run_attn_cfg<DH, 256, 128, 512>(a, st);
}

}  // namespace

size_t attention_scratch_bytes(int max_batch, int n_heads, int head_dim) {
    return (size_t)MAX_SPLIT * max_batch * n_heads * SPLIT_QUERIES * (head_dim + 2) * sizeof(float);
}

void launch_attention_bf16(const void* q, const void* k_cache, const void* v_cache, void* out, float* scratch,
                           int B, int L, int P, int n_heads, int head_dim, int max_seq, int max_batch, int layer,
                           bool frag_out, hipStream_t st) {
    AttnArgs a{};
    a.q = (const bf16*)q; a.kc = (const bf16*)k_cache; a.vc = (const bf16*)v_cache; a.out = (bf16*)out;
    a.B = B; a.L = L; a.P = P; a.nh = n_heads; a.max_seq = max_seq; a.max_batch = max_batch; a.layer = layer;
    a.frag = frag_out ? 1 : 0;   // the out projection of such a launch streams its weights
    a.scale_log2 = LOG2E / sqrtf((float)head_dim);
    // one query per sequence: too few (sequence, head) pairs to fill the chip, so the keys are split as well
    a.nsplit = 1;
    a.part = scratch;
    if (L == 1 && scratch) {
        const int tiles = (P + L - 1) / BKV_SMALL + 1;
        int ns = NS_TARGET / (B * n_heads);
        ns = ns > MAX_SPLIT ? MAX_SPLIT : ns;
        ns = ns > tiles ? tiles : ns;
        a.nsplit = ns < 1 ? 1 : ns;
    }
    if (head_dim == 128) run_attn<128>(a, st);
    else run_attn<64>(a, st);
}

void launch_attention_scattered_bf16(const void* q, const void* k_cache, const void* v_cache, void* out,
                                     float* scratch, int B, const int32_t* pos_tab, int cap, const uint8_t* hide,
                                     int P0, int Lblk, int n_heads, int head_dim, int max_seq, int max_batch,
                                     int layer, bool frag_out, hipStream_t st) {
    AttnArgs a{};
    a.q = (const bf16*)q; a.kc = (const bf16*)k_cache; a.vc = (const bf16*)v_cache; a.out = (bf16*)out;
    a.B = B; a.L = cap; a.P = P0; a.nh = n_heads; a.max_seq = max_seq; a.max_batch = max_batch; a.layer = layer;
    a.frag = frag_out ? 1 : 0;
    a.scale_log2 = LOG2E / sqrtf((float)head_dim);
    a.pos_tab = pos_tab; a.hide = hide; a.P0 = P0; a.Lblk = Lblk;
    // the slots of a sequence are the queries of one workgroup (128 per tile), which streams the sequence's rows
    // once; with few (sequence, head) pairs and at most 32 slots the rows are dealt to several workgroups as well
    a.nsplit = 1;
    a.part = scratch;
    if (scratch && cap <= SPLIT_QUERIES) {
        const int tiles = (P0 + Lblk - 1) / BKV_SMALL + 1;
        int ns = NS_TARGET / (B * n_heads);
        ns = ns > MAX_SPLIT ? MAX_SPLIT : ns;
        ns = ns > tiles ? tiles : ns;
        a.nsplit = ns < 1 ? 1 : ns;
    }
    if (head_dim == 128) run_attn_cfg<128, 128, BKV_SMALL, 256>(a, st);
    else run_attn_cfg<64, 128, BKV_SMALL, 256>(a, st);
}

}  // namespace mulo
