// Decision stage of the verification step: draft up-sampling (Sec. 3.2, Step 2),
// the speculative accept test (Sec. 3.1, Eq. 1 / Eq. 3), local expansion
// (Sec. 3.3, Eq. 6-7) and residual resampling (Sec. 3.1, Eq. 2).
//
// All of it is bound by HBM reads of [rows, V] float32 matrices: one workgroup of
// 256 lanes owns one row, keeps it in registers (V <= 16384) and reduces over the
// codebook with wavefront shuffles, so every logit is read from memory once in
// the accept pass and once more (with the draft row) only for marked positions.
#include <type_traits>

#include "mulo_internal.h"
#include "row_parts.h"

namespace mulo {

namespace {

constexpr int TPB = 256;
constexpr int WAVES = TPB / 64;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float NEAR_TIE = 1e-4f;
constexpr int MAX_CHUNKS = 1024;  // 256 codebook entries per chunk -> V <= 262144

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
// inclusive prefix sum over the 64 lanes of a wavefront
__device__ __forceinline__ unsigned long long wave_scan_u64(unsigned long long v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        unsigned long long n = __shfl_up(v, o);
        if (lane >= o) v += n;
    }
    return v;
}

// Fixed-order block reductions (run-to-run deterministic).
__device__ __forceinline__ float block_max(float v, float* red) {
    v = wave_max(v);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wv] = v;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int i = 1; i < WAVES; ++i) r = fmaxf(r, red[i]);
    return r;
}
__device__ __forceinline__ float block_sum(float v, float* red) {
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wv] = v;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int i = 1; i < WAVES; ++i) r += red[i];
    return r;
}

// exp(z - m) with one hardware exp2; no contraction so every kernel that
// evaluates it gets the same bits.
__device__ __forceinline__ float expm(float z, float m) { return rowparts::expm(z, m); }
__device__ __forceinline__ float prob(float z, float m, float inv) {
    return __fmul_rn(expm(z, m), inv);
}

// Classifier-free guidance of a target logit: z_u + s (z_c - z_u), every operation rounded on its own so
// that all kernels reproduce the same bits; zu == nullptr (no guidance) returns the logit unchanged.
__device__ __forceinline__ float guide(float zc, float zu, float s) {
    return __fadd_rn(zu, __fmul_rn(s, __fsub_rn(zc, zu)));
}
struct Guided {
    const float* zc;   // row of conditional logits
    const float* zu;   // row of unconditional logits or nullptr
    float s;
    __device__ __forceinline__ float at(int i) const { return zu ? guide(zc[i], zu[i], s) : zc[i]; }
    __device__ __forceinline__ float4 at4(int i4) const {
        const float4 c = reinterpret_cast<const float4*>(zc)[i4];
        if (!zu) return c;
        const float4 u = reinterpret_cast<const float4*>(zu)[i4];
        return make_float4(guide(c.x, u.x, s), guide(c.y, u.y, s), guide(c.z, u.z, s), guide(c.w, u.w, s));
    }
};

// Philox4x32-10 (Salmon et al., SC'11), word 0 of the output block.
__device__ __forceinline__ uint32_t philox_word0(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1) {
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(M0, c0), lo0 = M0 * c0;
        const uint32_t hi1 = __umulhi(M1, c2), lo1 = M1 * c2;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += W0; k1 += W1;
    }
    return c0;
}

// ---- a row of V floats held by one workgroup -------------------------------
// NV4 > 0: registers (V <= 1024 * NV4); NV4 == 0: re-read from memory (L2) per pass.
template <int NV4>
struct RowRegs {
    float4 v[NV4 > 0 ? NV4 : 1];
};

template <int NV4>
__device__ __forceinline__ void row_stats(const Guided src, int V, RowRegs<NV4>& rr,
                                          float* red, float& m, float& inv) {
    const int nv4 = V >> 2, tid = threadIdx.x;
    const float NEG = -__builtin_huge_valf();
    float mx = NEG;
    if constexpr (NV4 > 0) {
#pragma unroll
        for (int i = 0; i < NV4; ++i) {
            const int idx = i * TPB + tid;
            rr.v[i] = idx < nv4 ? src.at4(idx) : make_float4(NEG, NEG, NEG, NEG);
            mx = fmaxf(fmaxf(mx, fmaxf(rr.v[i].x, rr.v[i].y)), fmaxf(rr.v[i].z, rr.v[i].w));
        }
    } else {
        for (int idx = tid; idx < nv4; idx += TPB) {
            const float4 t = src.at4(idx);
            mx = fmaxf(fmaxf(mx, fmaxf(t.x, t.y)), fmaxf(t.z, t.w));
        }
    }
    m = block_max(mx, red);
    float s = 0.f;
    if constexpr (NV4 > 0) {
#pragma unroll
        for (int i = 0; i < NV4; ++i) {
            rr.v[i].x = expm(rr.v[i].x, m); rr.v[i].y = expm(rr.v[i].y, m);
            rr.v[i].z = expm(rr.v[i].z, m); rr.v[i].w = expm(rr.v[i].w, m);
            s += (rr.v[i].x + rr.v[i].y) + (rr.v[i].z + rr.v[i].w);
        }
    } else {
        for (int idx = tid; idx < nv4; idx += TPB) {
            const float4 t = src.at4(idx);
            s += (expm(t.x, m) + expm(t.y, m)) + (expm(t.z, m) + expm(t.w, m));
        }
    }
    s = block_sum(s, red);
    inv = 1.0f / s;
}

template <int NV4>
__device__ __forceinline__ void row_write_probs(const Guided src, float* __restrict__ dst,
                                                int V, const RowRegs<NV4>& rr, float m, float inv) {
    const int nv4 = V >> 2, tid = threadIdx.x;
    float4* d4 = reinterpret_cast<float4*>(dst);
    if constexpr (NV4 > 0) {
#pragma unroll
        for (int i = 0; i < NV4; ++i) {
            const int idx = i * TPB + tid;
            if (idx < nv4)
                d4[idx] = make_float4(__fmul_rn(rr.v[i].x, inv), __fmul_rn(rr.v[i].y, inv),
                                      __fmul_rn(rr.v[i].z, inv), __fmul_rn(rr.v[i].w, inv));
        }
    } else {
        for (int idx = tid; idx < nv4; idx += TPB) {
            const float4 t = src.at4(idx);
            d4[idx] = make_float4(prob(t.x, m, inv), prob(t.y, m, inv), prob(t.z, m, inv),
                                  prob(t.w, m, inv));
        }
    }
}

// ---- Step 2: softmax of the draft logits, one workgroup per low-res cell ----
// up.hi: the workgroup also writes its cell's token to the r x r children, x~[b, (rI+a) W + rJ+c] = y~[b, I w + J], and (first sequence)
// their q_row: a launch of 4.7 us less in front of the step.
template <int NV4>
__global__ __launch_bounds__(TPB) void k_softmax_rows(const float* __restrict__ in,
                                                      float* __restrict__ out, int V, const UpTokens up) {
    __shared__ float red[WAVES];
    const int64_t row = blockIdx.x;
    if (up.hi) {
        const int n_lo = up.h * up.w, W = up.w * up.r, b = (int)(row / n_lo), par = (int)(row % n_lo), I = par / up.w, J = par % up.w;
        const int tok = up.lo[row];
        for (int c = threadIdx.x; c < up.r * up.r; c += TPB) {
            const int u = (I * up.r + c / up.r) * W + J * up.r + c % up.r;
            up.hi[(int64_t)b * n_lo * up.r * up.r + u] = tok;
            if (b == 0) up.q_row[u] = par;
        }
    }
    RowRegs<NV4> rr;
    float m, inv;
    const Guided src{in + row * V, nullptr, 1.f};
    row_stats<NV4>(src, V, rr, red, m, inv);
    row_write_probs<NV4>(src, out + row * V, V, rr, m, inv);
}

__global__ __launch_bounds__(TPB) void k_copy(const float4* __restrict__ in, float4* __restrict__ out,
                                              int64_t n4) {
    for (int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x; i < n4; i += (int64_t)gridDim.x * TPB)
        out[i] = in[i];
}

// dst[b, :] = src[b, :] for rows of V floats, destination rows dst_stride floats apart
__global__ __launch_bounds__(TPB) void k_copy_rows_strided(const float4* __restrict__ src, float* __restrict__ dst,
                                                           int nv4, int64_t dst_stride) {
    const int b = blockIdx.y;
    float4* d = reinterpret_cast<float4*>(dst + b * dst_stride);
    for (int i = blockIdx.x * TPB + threadIdx.x; i < nv4; i += gridDim.x * TPB) d[i] = src[(int64_t)b * nv4 + i];
}

// x~[b, (rI+a) W + rJ+c] = y~[b, I w + J];  q_row[u] = (i_u / r) w + j_u / r
__global__ __launch_bounds__(TPB) void k_upsample_tokens(const int32_t* __restrict__ lo,
                                                         int32_t* __restrict__ hi,
                                                         int32_t* __restrict__ q_row, int B, int h,
                                                         int w, int r) {
    const int W = w * r, T = h * r * W;
    const int64_t gid = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (gid >= (int64_t)B * T) return;
    const int b = gid / T, u = gid % T;
    const int par = ((u / W) / r) * w + (u % W) / r;
    hi[gid] = lo[(int64_t)b * h * w + par];
    if (b == 0) q_row[u] = par;
}

// q_hi[b, u, :] = q_lo[b, q_row[u], :]
__global__ __launch_bounds__(TPB) void k_gather_rows(const float* __restrict__ q_lo,
                                                     const int32_t* __restrict__ q_row,
                                                     float* __restrict__ q_hi, int n_lo, int n_hi,
                                                     int V) {
    const int u = blockIdx.x, b = blockIdx.y;
    const float4* s = reinterpret_cast<const float4*>(q_lo + ((int64_t)b * n_lo + q_row[u]) * V);
    float4* d = reinterpret_cast<float4*>(q_hi + ((int64_t)b * n_hi + u) * V);
    for (int i = threadIdx.x; i < (V >> 2); i += TPB) d[i] = s[i];
}

// One integer weight of the draw, floor(w 2^40), as a double: sums of up to 256 of them (2^49) are exact there, at half
// the instructions of the conversion to and the addition of 64-bit integers.
template <bool USE_Q>
__device__ __forceinline__ double weight(float z, float q, float m, float inv) {
    float p = prob(z, m, inv);
    if constexpr (USE_Q) p = fmaxf(0.f, __fsub_rn(p, q));
    return (double)truncf(__fmul_rn(p, 1099511627776.0f));
}
template <bool USE_Q>
__device__ __forceinline__ double weight_sum4(const float4 z, const float4 q, float m, float inv) {
    return (weight<USE_Q>(z.x, q.x, m, inv) + weight<USE_Q>(z.y, q.y, m, inv)) +
           (weight<USE_Q>(z.z, q.z, m, inv) + weight<USE_Q>(z.w, q.w, m, inv));
}
// the same as integers, for the walk inside a chunk: floor(w 2^40) of w = max(0, p - q), or of p (use_p)
__device__ __forceinline__ void weights4(const float4 z, const float4 qv, float m, float inv, bool use_p,
                                         unsigned long long w[4]) {
    const float S = 1099511627776.0f;  // 2^40: w * S is exact in float32
    float p0 = prob(z.x, m, inv), p1 = prob(z.y, m, inv), p2 = prob(z.z, m, inv), p3 = prob(z.w, m, inv);
    if (!use_p) {
        p0 = fmaxf(0.f, __fsub_rn(p0, qv.x)); p1 = fmaxf(0.f, __fsub_rn(p1, qv.y));
        p2 = fmaxf(0.f, __fsub_rn(p2, qv.z)); p3 = fmaxf(0.f, __fsub_rn(p3, qv.w));
    }
    w[0] = (unsigned long long)__fmul_rn(p0, S); w[1] = (unsigned long long)__fmul_rn(p1, S);
    w[2] = (unsigned long long)__fmul_rn(p2, S); w[3] = (unsigned long long)__fmul_rn(p3, S);
}

// ---- Step 4: softmax statistics + accept test, one workgroup per position ---
__device__ __forceinline__ int clamp_tok(int t, int V) { return t < 0 ? 0 : (t >= V ? V - 1 : t); }

// The accept test of one position, by one lane: Eq. 1 without the division (u q < pbar), or the threshold rule of
// Eq. 5 (pbar >= tau); leaves the row statistics for the re-draw kernel, the near-tie flag as the sign of the inverse sum,
// for finish_sequence to count (per-row atomics on the few counters of a sequence cost a quarter of the accept
// kernel's time).
__device__ __forceinline__ bool accept_row(const DecideArgs& a, int64_t row, int b, int t, float qt, float pbar,
                                           float m, float inv) {
    const uint32_t w0 = philox_word0((uint32_t)t, (uint32_t)b, a.ctr_lo, a.ctr_hi24, a.key0, a.key1);
    const float u = (float)(w0 >> 8) * 5.9604644775390625e-08f;  // 2^-24, exact
    // the threshold rule is written as "tau' < pbar or equal" through the same comparison with uq := tau
    const bool tau_rule = a.accept_mode == 1;
    const float uq = tau_rule ? a.tau : __fmul_rn(u, qt);
    const bool ok = tau_rule ? pbar >= uq : uq < pbar;
    a.accept[row] = ok ? 1 : 0;
    a.rowmax[row] = m;
    const bool near = fabsf(__fsub_rn(pbar, uq)) < __fmul_rn(NEAR_TIE, tau_rule ? a.tau : qt);
    a.rowinv[row] = __builtin_copysignf(inv, near ? -1.f : 1.f);
    return ok;
}

constexpr int MAX_PARTS = 2048;   // 128 codebook entries per part -> V <= 262144

// One workgroup per position.  The row is read once: lane `tid` of pass k owns run 256 k + tid (8 consecutive logits),
// so the 16 lanes of a part sit next to each other, the two halves of the part on the even and the odd lanes; the
// part statistics are formed with lane exchanges in the order row_parts.h fixes, left in LDS, and merged by the
// first wavefront.
// A pass's logits are requested while the one before is added up, and without branches (entries that do not exist re-read the row's
// first): with them the two rows of guidance were a round trip each (2 x 1024 rows of 16384 with their twins 47.6 -> 41.9 us; 4 x 1024
// rows of one, test and draw of radius 0, 136 -> 126).
template <bool GUIDED>
__global__ __launch_bounds__(TPB) void k_accept(const DecideArgs a) {
    __shared__ float2 parts[MAX_PARTS];
    __shared__ float red[WAVES];
    __shared__ float2 s_stat;
    const int64_t row = blockIdx.x;
    const int b = row / a.L, t = row % a.L, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const Guided z{a.logits + row * a.V, GUIDED ? a.logits_u + row * a.V : nullptr, a.cfg_scale};
    // the scalar gathers (draft token -> its logit and its draft probability) are issued first, so that
    // their chained latency is hidden behind the streaming of the row
    const int tok = clamp_tok(a.draft_tokens[row], a.V);
    float ztok = 0.f, qt = 0.f;
    if (tid == 0) {
        if (a.accept_mode == 0) {
            const int qr = a.q_row ? a.q_row[t] : t;
            qt = a.q[b * a.q_batch_stride + (int64_t)qr * a.V + tok];
        }
        ztok = z.at(tok);
    }
    const int V = a.V, n_parts = (V + rowparts::PART - 1) / rowparts::PART;
    const float NEG = rowparts::NEG_INF;
    const float4 *c4 = reinterpret_cast<const float4*>(z.zc), *u4 = reinterpret_cast<const float4*>(z.zu);
    const int nv4 = V >> 2;
    float4 nc[2], nu[2];
    auto request = [&](int R) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = 2 * R + h < nv4 ? 2 * R + h : 0;
            nc[h] = c4[i];
            if constexpr (GUIDED) nu[h] = u4[i];
        }
    };
    request(tid);
    for (int base = 0; base < n_parts * 16; base += TPB) {
        const int R = base + tid;                       // run of 8 logits; V is a multiple of 4
        const int n_valid = V - R * 8 >= 8 ? 8 : (V - R * 8 >= 4 ? 4 : 0);
        float4 lo = nc[0], hi = nc[1];
        if constexpr (GUIDED) {
            auto with = [&](const float4 c, const float4 u) { return make_float4(guide(c.x, u.x, z.s), guide(c.y, u.y, z.s), guide(c.z, u.z, z.s), guide(c.w, u.w, z.s)); };
            lo = with(lo, nu[0]);
            hi = with(hi, nu[1]);
        }
        request(R + TPB);
        if (n_valid < 4) lo = make_float4(NEG, NEG, NEG, NEG);
        if (n_valid < 8) hi = make_float4(NEG, NEG, NEG, NEG);
        float zz[8];
        zz[0] = lo.x; zz[1] = lo.y; zz[2] = lo.z; zz[3] = lo.w; zz[4] = hi.x; zz[5] = hi.y; zz[6] = hi.z; zz[7] = hi.w;
        float m = fmaxf(fmaxf(fmaxf(zz[0], zz[1]), fmaxf(zz[2], zz[3])), fmaxf(fmaxf(zz[4], zz[5]), fmaxf(zz[6], zz[7])));
        m = fmaxf(m, __shfl_xor(m, 2));                 // the 8 runs of a half: lanes 2 apart
        m = fmaxf(m, __shfl_xor(m, 4));
        m = fmaxf(m, __shfl_xor(m, 8));
        float s = rowparts::run_sum(zz, m, n_valid);
        s = __fadd_rn(s, __shfl_xor(s, 2));             // ((t0+t1)+(t2+t3))+((t4+t5)+(t6+t7))
        s = __fadd_rn(s, __shfl_xor(s, 4));
        s = __fadd_rn(s, __shfl_xor(s, 8));
        const float2 ps = rowparts::merge_halves(m, s, __shfl_xor(m, 1), __shfl_xor(s, 1));
        if ((tid & 15) == 0 && (R >> 4) < n_parts) parts[R >> 4] = ps;
    }
    __syncthreads();
    if (wv == 0) {
        const float2 st = rowparts::combine_parts(parts, n_parts, lane);
        if (lane == 0) s_stat = st;
    }
    __syncthreads();
    const float m = s_stat.x, inv = 1.0f / s_stat.y;
    if (a.p_probs) {
        RowRegs<0> none;
        row_write_probs<0>(z, a.p_probs + row * a.V, a.V, none, m, inv);
    }
    float pbar;
    if (a.pool_k <= 1) {
        pbar = prob(ztok, m, inv);
    } else {  // Eq. 3: pooled mass over the codebook neighbours of the draft token
        float acc = 0.f;
        for (int i = tid; i < a.pool_k; i += TPB)
            acc += prob(z.at(clamp_tok(a.nbr[(int64_t)tok * a.pool_k + i], a.V)), m, inv);
        pbar = block_sum(acc, red);
    }
    if (tid == 0) accept_row(a, row, b, t, qt, pbar, m, inv);
}

// Eq. 1 without pooling, which also leaves the chunk sums that the re-draw starts from (chunk c: entries [256 c, 256 c + 256)):
// the row stays in registers (V <= 2048 NIT), so a marked position reads its logits once, not twice.  The sums are
// of integers, so they are cdf_draw's whoever adds them; a run of 8 lies in one chunk, 32 lanes share it.  The weights of the
// draw depend on this row's own decision only (use_p), which is known here; whether the position is marked is not, so
// an unmarked one has read its draft row for nothing (launch_accept's rule).
// XCD x takes the x-th eighth of the rows: neighbours, children of one draft row, find it in one L2.
// Latency bounds it, four workgroups a CU with a row each (the arithmetic of the weights taken out: no difference; the draft row taken
// out: 66 of 82 us), so requests go out without a branch, several passes of the draft row together: a branch around an access
// (the end of the row, guidance) had the compiler wait for it before the next.  4 x 1024 rows of 16384, us: 82 -> 74.
// Two positions a workgroup with the draft row they share in LDS: 93 (half as many workgroups to hide behind each other).
template <int NIT, bool GUIDED>
__global__ __launch_bounds__(TPB, GUIDED ? 3 : 4) void k_accept_sums(const DecideArgs a, unsigned long long* __restrict__ sums, int rows_per_xcd) {
    __shared__ float2 parts[NIT * 16];
    __shared__ float2 s_stat;
    __shared__ int s_use_p;
    const int64_t row = (int64_t)(blockIdx.x & 7) * rows_per_xcd + (blockIdx.x >> 3);
    if (row >= (int64_t)a.B * a.L) return;                     // uniform over the workgroup, before any barrier
    const int b = row / a.L, t = row % a.L, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const Guided z{a.logits + row * a.V, GUIDED ? a.logits_u + row * a.V : nullptr, a.cfg_scale};
    const int tok = clamp_tok(a.draft_tokens[row], a.V);
    const int qr = a.q_row ? a.q_row[t] : t;
    const float* q = a.q + b * a.q_batch_stride + (int64_t)qr * a.V;
    float ztok = 0.f, qt = 0.f;
    if (tid == 0) {
        qt = q[tok];
        ztok = z.at(tok);
    }
    const int V = a.V, n_parts = (V + rowparts::PART - 1) / rowparts::PART;
    const float NEG = rowparts::NEG_INF;
    float4 lo[NIT], hi[NIT];
    const int nv4 = V >> 2;
    auto entry = [&](int i4) { return i4 < nv4 ? i4 : 0; };    // entries that do not exist re-read the row's first
    const float4 *c4 = reinterpret_cast<const float4*>(z.zc), *u4 = reinterpret_cast<const float4*>(z.zu);
    auto with = [&](const float4 c, const float4 u) { return make_float4(guide(c.x, u.x, z.s), guide(c.y, u.y, z.s), guide(c.z, u.z, z.s), guide(c.w, u.w, z.s)); };
    // a wavefront that lies past the end of a short row has only barriers to keep (16 x 4096 rows of 1024, test and draw 201 -> 186 us)
    const bool idle = NIT == 1 && __builtin_amdgcn_readfirstlane(wv) * 128 >= nv4;
    if (!idle) {
#pragma unroll
        for (int k = 0; k < NIT; ++k) {
            const int R = k * TPB + tid;
            lo[k] = c4[entry(2 * R)];
            hi[k] = c4[entry(2 * R + 1)];
            if constexpr (GUIDED) {
                lo[k] = with(lo[k], u4[entry(2 * R)]);
                hi[k] = with(hi[k], u4[entry(2 * R + 1)]);
                if (k & 1) asm volatile("" ::: "memory");          // two passes in flight: all of both rows do not fit the registers
            }
        }
#pragma unroll
        for (int k = 0; k < NIT; ++k) {                            // the part statistics, as in k_accept
            const int R = k * TPB + tid;
            if (2 * R >= nv4) lo[k] = make_float4(NEG, NEG, NEG, NEG);
            if (2 * R + 1 >= nv4) hi[k] = make_float4(NEG, NEG, NEG, NEG);
            const int n_valid = V - R * 8 >= 8 ? 8 : (V - R * 8 >= 4 ? 4 : 0);
            const float zz[8] = {lo[k].x, lo[k].y, lo[k].z, lo[k].w, hi[k].x, hi[k].y, hi[k].z, hi[k].w};
            float m = fmaxf(fmaxf(fmaxf(zz[0], zz[1]), fmaxf(zz[2], zz[3])), fmaxf(fmaxf(zz[4], zz[5]), fmaxf(zz[6], zz[7])));
            m = fmaxf(m, __shfl_xor(m, 2));
            m = fmaxf(m, __shfl_xor(m, 4));
            m = fmaxf(m, __shfl_xor(m, 8));
            float s = rowparts::run_sum(zz, m, n_valid);
            s = __fadd_rn(s, __shfl_xor(s, 2));
            s = __fadd_rn(s, __shfl_xor(s, 4));
            s = __fadd_rn(s, __shfl_xor(s, 8));
            const float2 ps = rowparts::merge_halves(m, s, __shfl_xor(m, 1), __shfl_xor(s, 1));
            if ((tid & 15) == 0 && (R >> 4) < n_parts) parts[R >> 4] = ps;
        }
    }
    __syncthreads();
    if (wv == 0) {
        const float2 st = rowparts::combine_parts(parts, n_parts, lane);
        if (lane == 0) s_stat = st;
    }
    __syncthreads();
    const float m = s_stat.x, inv = 1.0f / s_stat.y;
    if (tid == 0) {
        const bool ok = accept_row(a, row, b, t, qt, prob(ztok, m, inv), m, inv);
        s_use_p = a.resample_mode == 1 && ok;
    }
    __syncthreads();
    if (idle) return;                                          // no barrier follows
    const bool use_p = s_use_p != 0;                           // uniform
    const int nchunks = ((V >> 2) + 63) >> 6;
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    auto chunk_pass = [&](auto with_q) {
        constexpr bool WITH_Q = decltype(with_q)::value;
        const float4* q4 = reinterpret_cast<const float4*>(q);
        constexpr int G = NIT <= 2 ? NIT : GUIDED ? 2 : NIT % 4 == 0 ? 4 : 3;   // passes whose draft entries are requested together
#pragma unroll
        for (int k0 = 0; k0 < NIT; k0 += G) {
            float4 q_lo[G], q_hi[G];
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const int R = (k0 + j) * TPB + tid;
                q_lo[j] = WITH_Q ? q4[entry(2 * R)] : zero4;
                q_hi[j] = WITH_Q ? q4[entry(2 * R + 1)] : zero4;
            }
            if (WITH_Q && nv4 < NIT * 2 * TPB) {               // a row that ends inside the passes: entries that do not exist weigh 0
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    const int R = (k0 + j) * TPB + tid;
                    if (2 * R >= nv4) q_lo[j] = zero4;
                    if (2 * R + 1 >= nv4) q_hi[j] = zero4;
                }
            }
            double sum[G];
#pragma unroll
            for (int j = 0; j < G; ++j)
                sum[j] = weight_sum4<WITH_Q>(lo[k0 + j], q_lo[j], m, inv) + weight_sum4<WITH_Q>(hi[k0 + j], q_hi[j], m, inv);
#pragma unroll
            for (int o = 16; o > 0; o >>= 1)
#pragma unroll
                for (int j = 0; j < G; ++j) sum[j] += __shfl_xor(sum[j], o);
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const int R = (k0 + j) * TPB + tid;
                if ((tid & 31) == 0 && (R >> 5) < nchunks) sums[row * nchunks + (R >> 5)] = (unsigned long long)sum[j];
            }
        }
    };
    if (use_p) chunk_pass(std::false_type{});
    else chunk_pass(std::true_type{});
}

// The same test when the lm-head GEMM has already left the parts of every row (a verification step): one
// wavefront per position merges them and gathers the draft token's logit; the row of logits is not read again.
__global__ __launch_bounds__(TPB) void k_accept_parts(const DecideArgs a, const float2* __restrict__ parts, int n_parts) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t row = (int64_t)blockIdx.x * WAVES + wv;
    if (row >= (int64_t)a.B * a.L) return;            // uniform over the wavefront
    const int b = row / a.L, t = row % a.L;
    const int tok = clamp_tok(a.draft_tokens[row], a.V);
    float ztok = 0.f, qt = 0.f;
    if (lane == 0) {
        if (a.accept_mode == 0) {
            const int qr = a.q_row ? a.q_row[t] : t;
            qt = a.q[b * a.q_batch_stride + (int64_t)qr * a.V + tok];
        }
        ztok = a.logits[row * a.V + tok];
    }
    const float2 st = rowparts::combine_parts(parts + row * n_parts, n_parts, lane);
    if (lane == 0) {
        const float m = st.x, inv = 1.0f / st.y;
        accept_row(a, row, b, t, qt, prob(ztok, m, inv), m, inv);
    }
}

// ---- Step 5 (Eq. 6-7) + the step's counters, one workgroup per sequence ----
// From the accept flags of the block (staged in LDS): t0 = first rejected position, the counts of accepted /
// rejected positions and near ties, then R_X: position t is marked when it is at or after t0 and within Chebyshev
// distance rho of some rejected position of the block (rho < 0: the raster rule, everything from t0 on).  Writes
// mask, t0 and stats = (accepted, rejected, marked, near ties); no atomics on global memory anywhere.
// A chain of latencies, so in a launch of its own a position per thread up to blocks of 1024 where there is a window to search (4 x 1024,
// radius 2: 256 threads 7.5 us, 1024 6.8); without one (2 x 1024, radius 0: 4.7 / 5.3) the larger workgroup only costs.
// near_s: [L] of LDS too, or nullptr.  With it a window is searched along its row first, for all positions, and then down the rows:
// 2 (2 rho + 1) flags a position instead of (2 rho + 1)^2.
__device__ __forceinline__ void finish_sequence(const DecideArgs& a, int b, uint8_t* acc_s, uint8_t* near_s, int (*red)[4]) {   // acc_s: [L] of LDS
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wv = tid >> 6;
    const uint8_t* acc_g = a.accept + (int64_t)b * a.L;
    const float* inv_g = a.rowinv + (int64_t)b * a.L;
    uint8_t* mask_g = a.mask + (int64_t)b * a.L;
    int n_acc = 0, n_near = 0, tmin = a.L;
    for (int t = tid; t < a.L; t += nt) {
        const uint8_t ok = acc_g[t];
        acc_s[t] = ok;
        n_acc += ok;
        n_near += __builtin_signbit(inv_g[t]) != 0;
        if (!ok && t < tmin) tmin = t;
    }
    auto reduce_counts = [&](int& x, int& y, int& z_min, int& w) {   // sums of x, y, w and the minimum of z_min over the workgroup
        for (int o = 32; o > 0; o >>= 1) {
            x += __shfl_xor(x, o);
            y += __shfl_xor(y, o);
            w += __shfl_xor(w, o);
            const int other = __shfl_xor(z_min, o);
            z_min = other < z_min ? other : z_min;
        }
        __syncthreads();
        if (lane == 0) { red[wv][0] = x; red[wv][1] = y; red[wv][2] = z_min; red[wv][3] = w; }
        __syncthreads();
        x = y = w = 0;
        z_min = a.L;
        for (int i = 0; i < (nt >> 6); ++i) {
            x += red[i][0]; y += red[i][1]; w += red[i][3];
            z_min = red[i][2] < z_min ? red[i][2] : z_min;
        }
    };
    int zero = 0;
    reduce_counts(n_acc, n_near, tmin, zero);   // the barriers inside also publish acc_s
    const int t0 = tmin;
    if (near_s && a.rho > 0 && t0 < a.L) {             // uniform over the workgroup
        // A block is whole rows of the grid; those before t0's hold no rejection.  Eight flags at a time: a chain of single reads costs
        // the latency of each.  A wavefront leaves a search as one: of lanes that leave on their own the compiler lost the flag
        // that made them (it kept it as the lane mask of the loop's last round).
        const int first = t0 - t0 % a.W, across = 2 * a.rho < a.W - 1 ? 2 * a.rho : a.W - 1;
        for (int t = tid; t < a.L; t += nt) {
            const int gj = t % a.W, u0 = gj < a.rho ? t - gj : t - a.rho, u1 = a.W - 1 - gj < a.rho ? t + a.W - 1 - gj : t + a.rho;
            uint32_t ok = 1;
            for (int o = 0; o <= across && __any(ok && t >= first); o += 8)
#pragma unroll
                for (int k = 0; k < 8; ++k) ok &= acc_s[u0 + o + k < u1 ? u0 + o + k : u1];
            near_s[t] = ok == 0;
        }
        __syncthreads();
    }
    int n_marked = 0;
    for (int t = tid; t < a.L; t += nt) {
        int marked = 0;
        if (t >= t0) {
            if (a.rho < 0) {
                marked = 1;
            } else {
                // the window, cut to the rows of the block (whole rows of the grid) and to the grid's columns
                const int g = a.n0 + t, gi = g / a.W, gj = g % a.W, r0 = a.n0 / a.W, r1 = (a.n0 + a.L - 1) / a.W;
                const int i_lo = gi - a.rho > r0 ? gi - a.rho : r0, i_hi = gi + a.rho < r1 ? gi + a.rho : r1;
                const int j_lo = gj - a.rho > 0 ? gj - a.rho : 0, j_hi = gj + a.rho < a.W - 1 ? gj + a.rho : a.W - 1;
                if (near_s && a.rho > 0) {
                    const int down = 2 * a.rho < r1 - r0 ? 2 * a.rho : r1 - r0;
                    for (int o = 0; o <= down && __any(!marked); o += 8)
#pragma unroll
                        for (int k = 0; k < 8; ++k) marked |= near_s[(i_lo + o + k < i_hi ? i_lo + o + k : i_hi) * a.W + gj - a.n0];
                } else for (int ii = i_lo; ii <= i_hi && !marked; ++ii)
                    for (int jj = j_lo; jj <= j_hi; ++jj)
                        if (acc_s[ii * a.W + jj - a.n0] == 0) { marked = 1; break; }
            }
        }
        mask_g[t] = (uint8_t)marked;
        n_marked += marked;
    }
    int d0 = 0, d1 = a.L;
    reduce_counts(n_marked, d0, d1, zero);
    if (tid == 0) {
        a.t0[b] = t0;
        a.stats[b * 4 + 0] = n_acc;
        a.stats[b * 4 + 1] = a.L - n_acc;
        a.stats[b * 4 + 2] = n_marked;
        a.stats[b * 4 + 3] = n_near;
    }
}

__global__ __launch_bounds__(1024) void k_decide_finish(const DecideArgs a) {
    extern __shared__ uint8_t acc_s[];   // [L]
    __shared__ int red[16][4];
    finish_sequence(a, blockIdx.x, acc_s, nullptr, red);
}

// Small decisions have no launch for it (decide_finish's rule; blocks of up to FUSED_L positions, whose flags the kernels hold): the first workgroups of the re-draw run
// finish_sequence, a sequence each (n_fin of them, whole rounds of XCDs), while those of the positions find out for themselves whether
// theirs is marked, a wavefront each: over the window (a rejection there at or before t says it all, none says no) and, where that leaves
// it open, over the flags in front of t up to the first rejection; windows of more than one batch of flags after those.
constexpr int FUSED_L = 4096;
__device__ __forceinline__ bool position_marked(const DecideArgs& a, int b, int t, int lane) {
    b = __builtin_amdgcn_readfirstlane(b);
    t = __builtin_amdgcn_readfirstlane(t);
    const uint8_t* const acc = a.accept + (int64_t)b * a.L;
    auto rejected_up_to_t = [&]() {
        for (int u0 = 0; u0 <= t; u0 += 256) {
            bool hit = false;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int u = u0 + k * 64 + lane;
                hit |= acc[u < t ? u : t] == 0;
            }
            if (__any(hit)) return true;
        }
        return false;
    };
    if (a.rho < 0) return rejected_up_to_t();
    const int g = a.n0 + t, gi = g / a.W, gj = g % a.W, r0 = a.n0 / a.W, r1 = (a.n0 + a.L - 1) / a.W;
    const int i_lo = gi - a.rho > r0 ? gi - a.rho : r0, i_hi = gi + a.rho < r1 ? gi + a.rho : r1;
    const int j_lo = gj - a.rho > 0 ? gj - a.rho : 0, j_hi = gj + a.rho < a.W - 1 ? gj + a.rho : a.W - 1, nj = j_hi - j_lo + 1;
    const int n = (i_hi - i_lo + 1) * nj;
    const bool wide = n > 256;
    if (wide && !rejected_up_to_t()) return false;
    bool near = false;
    for (int c0 = 0; c0 < n; c0 += 256) {
        bool enough = false;   // a rejection in the window, at or before t unless one is known to be
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (c0 + k * 64 >= n) break;   // uniform
            const int c = c0 + k * 64 + lane < n ? c0 + k * 64 + lane : n - 1, u = (i_lo + c / nj) * a.W + j_lo + c % nj - a.n0;
            const bool hit = acc[u] == 0;
            near |= hit;
            enough |= hit && (wide || u <= t);
        }
        if (__any(enough)) return true;
    }
    return !wide && __any(near) && rejected_up_to_t();
}

// ---- Step 5 + Eq. 2: neighbourhood mask, then the residual draw -------------
// Chunk sums of the integer weights of a row (pass 1 of the draw): chunk c covers the 256 codebook entries
// [256 c, 256 c + 256) = 64 lanes x 4 entries.  G float4 per lane are requested together (both rows), and their G
// wavefront sums run side by side, so that neither the memory latency nor the latency of a lane exchange is paid
// once per chunk.  GUIDED: the logits are z_u + s (z_c - z_u); USE_Q: residual weights max(0, p - q), else p.
template <int G, bool GUIDED, bool USE_Q>
__device__ __forceinline__ void chunk_sums(const Guided z, const float4* __restrict__ q4, float m, float inv, int nv4,
                                           int nchunks, unsigned long long* chunk) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const float4* zc4 = reinterpret_cast<const float4*>(z.zc);
    const float4* zu4 = reinterpret_cast<const float4*>(z.zu);
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int base = 0; base < nv4; base += TPB * G) {
        float4 zc[G], zu[G], qv[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {       // rows past the end re-read entry 0 and are not counted
            const int idx = base + g * TPB + tid, ci = idx < nv4 ? idx : 0;
            zc[g] = zc4[ci];
            if constexpr (GUIDED) zu[g] = zu4[ci];
            if constexpr (USE_Q) qv[g] = q4[ci];
        }
        double sm[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int idx = base + g * TPB + tid;
            float4 zz = zc[g];
            if constexpr (GUIDED)
                zz = make_float4(guide(zz.x, zu[g].x, z.s), guide(zz.y, zu[g].y, z.s), guide(zz.z, zu[g].z, z.s),
                                 guide(zz.w, zu[g].w, z.s));
            const double s4 = weight_sum4<USE_Q>(zz, USE_Q ? qv[g] : zero4, m, inv);
            sm[g] = idx < nv4 ? s4 : 0.0;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int g = 0; g < G; ++g) sm[g] += __shfl_xor(sm[g], o);
        if (lane == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int c = (base >> 6) + g * WAVES + wv;
                if (c < nchunks) chunk[c] = (unsigned long long)sm[g];
            }
        }
    }
}

// Integer-CDF draw of one row by one workgroup: W(x) = floor(w(x) 2^40) with w = max(0, p - q) (or p when
// use_p), T = (word * tot) >> 32, token = first x whose inclusive prefix exceeds T; an empty residual falls
// back to p.  The token is stored to *out by the lane that finds it.
__device__ __forceinline__ void cdf_draw(const Guided z, const float4* __restrict__ q4, float m,
                                         float inv, bool use_p, uint32_t word, int V, int fallback_tok,
                                         int32_t* out, unsigned long long* chunk, int* s_retry) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int nv4 = V >> 2, nchunks = (nv4 + 63) >> 6;
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int attempt = 0; attempt < 2; ++attempt) {
        if (z.zu) {
            if (use_p) chunk_sums<2, true, false>(z, q4, m, inv, nv4, nchunks, chunk);
            else chunk_sums<2, true, true>(z, q4, m, inv, nv4, nchunks, chunk);
        } else {
            if (use_p) chunk_sums<4, false, false>(z, q4, m, inv, nv4, nchunks, chunk);
            else chunk_sums<4, false, true>(z, q4, m, inv, nv4, nchunks, chunk);
        }
        if (tid == 0) *s_retry = 0;
        __syncthreads();
        if (wv == 0) {
            unsigned long long tot = 0;
            for (int c0 = 0; c0 < nchunks; c0 += 64) tot += (c0 + lane < nchunks) ? chunk[c0 + lane] : 0ull;
            tot = wave_sum_u64(tot);
            if (tot == 0) {
                if (lane == 0) *s_retry = 1;  // empty residual: draw from p instead
            } else {
                const unsigned long long T = __umul64hi((unsigned long long)word << 32, tot);
                unsigned long long run = 0, before = 0;
                int cidx = nchunks - 1;
                for (int c0 = 0; c0 < nchunks; c0 += 64) {
                    const unsigned long long v = (c0 + lane < nchunks) ? chunk[c0 + lane] : 0ull;
                    const unsigned long long incl = wave_scan_u64(v, lane) + run;
                    const unsigned long long hit = __ballot(incl > T);
                    if (hit) {
                        const int f = __ffsll((long long)hit) - 1;
                        cidx = c0 + f;
                        before = __shfl(incl - v, f);
                        break;
                    }
                    run = __shfl(incl, 63);
                }
                // inside the chunk: 64 lanes x 4 entries, same weights as above
                const int idx = cidx * 64 + lane;
                unsigned long long w[4] = {0, 0, 0, 0};
                if (idx < nv4) weights4(z.at4(idx), use_p ? zero4 : q4[idx], m, inv, use_p, w);
                const unsigned long long s = (w[0] + w[1]) + (w[2] + w[3]);
                const unsigned long long incl = wave_scan_u64(s, lane) + before;
                const unsigned long long hit = __ballot(incl > T);
                const int f = hit ? __ffsll((long long)hit) - 1 : 63;
                if (lane == f) {
                    unsigned long long cum = incl - s;
                    int tok = fallback_tok;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        cum += w[e];
                        if (cum > T) { tok = idx * 4 + e; break; }
                    }
                    *out = clamp_tok(tok, V);
                }
            }
        }
        __syncthreads();
        if (!*s_retry || use_p) break;
        use_p = true;
        __syncthreads();
    }
}

template <bool FUSED>
__global__ __launch_bounds__(TPB) void k_mask_sample(const DecideArgs a, int n_fin) {
    __shared__ unsigned long long chunk[MAX_CHUNKS];
    __shared__ int s_retry;
    if constexpr (FUSED) {
        if ((int)blockIdx.x < n_fin) {                 // uniform over the workgroup
            __shared__ int red[16][4];
            static_assert(2 * FUSED_L <= MAX_CHUNKS * 8, "two flags a position");
            uint8_t* const acc_s = reinterpret_cast<uint8_t*>(chunk);
            if ((int)blockIdx.x < a.B) finish_sequence(a, blockIdx.x, acc_s, acc_s + FUSED_L, red);
            return;
        }
    }
    const int wg = FUSED ? blockIdx.x - n_fin : blockIdx.x;
    // Which position this workgroup handles.  Workgroup ids go round-robin over the 8 XCDs (each with its own L2).
    // When the draft rows are shared by r x r children (replication up-sampling), the children of a draft row are
    // given to consecutive workgroups of ONE XCD, so that the row comes from memory once instead of once per child.
    int64_t row = wg;
    if (a.up_r > 1) {
        const int r2 = a.up_r * a.up_r, n_par = a.L / r2;
        const int x = wg & 7, k = wg >> 3;
        const int64_t pseq = (int64_t)(k / r2) * 8 + x;
        if (pseq >= (int64_t)a.B * n_par) return;      // uniform over the workgroup (the grid is rounded up)
        const int child = k % r2, bb = pseq / n_par, par = pseq % n_par;
        const int I = par / a.up_w, J = par % a.up_w, W = a.up_r * a.up_w;
        row = (int64_t)bb * a.L + (a.up_r * I + child / a.up_r) * W + a.up_r * J + child % a.up_r;
    }
    const int b = row / a.L, t = row % a.L, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;

    // R_X membership of this position (Eq. 6-7)
    const bool marked = FUSED ? position_marked(a, b, t, lane) : a.mask[row] != 0;
    const int draft = clamp_tok(a.draft_tokens[row], a.V);
    if (!marked) {   // uniform over the workgroup
        if (tid == 0) a.tokens_out[row] = draft;
        return;
    }
    // Residual draw through the integer CDF
    const int V = a.V;
    const Guided z{a.logits + row * V, a.logits_u ? a.logits_u + row * V : nullptr, a.cfg_scale};
    const int qr = a.q_row ? a.q_row[t] : t;
    const bool use_p = a.resample_mode == 2 || ((a.resample_mode == 1) && a.accept[row] != 0);
    // the draft row is read only for residual weights (it may be absent when every draw is from p)
    const float4* q4 = reinterpret_cast<const float4*>(a.q ? a.q + b * a.q_batch_stride + (int64_t)qr * V : z.zc);
    const uint32_t word = philox_word0((uint32_t)t, (uint32_t)b, a.ctr_lo, a.ctr_hi24 | (1u << 24),
                                       a.key0, a.key1);
    cdf_draw(z, q4, a.rowmax[row], fabsf(a.rowinv[row]), use_p, word, V, draft, &a.tokens_out[row], chunk, &s_retry);
}

// The re-draw from the chunk sums that k_accept_sums left (at most 64 chunks, a lane each): one wavefront per position finds
// the chunk and reads its 256 entries.  The same draw as cdf_draw's, empty residual included.
template <bool FUSED>
__global__ __launch_bounds__(TPB) void k_sample_sums(const DecideArgs a, const unsigned long long* __restrict__ sums, int n_fin) {
    if constexpr (FUSED) {
        if ((int)blockIdx.x < n_fin) {                         // uniform over the workgroup
            __shared__ uint8_t acc_s[2 * FUSED_L];
            __shared__ int red[16][4];
            if ((int)blockIdx.x < a.B) finish_sequence(a, blockIdx.x, acc_s, acc_s + FUSED_L, red);
            return;
        }
    }
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)(FUSED ? blockIdx.x - n_fin : blockIdx.x) * WAVES + (threadIdx.x >> 6);
    if (row >= (int64_t)a.B * a.L) return;                     // uniform over the wavefront; no barrier follows
    const int b = row / a.L, t = row % a.L, V = a.V, nv4 = V >> 2, nchunks = (nv4 + 63) >> 6;
    const int draft = clamp_tok(a.draft_tokens[row], V);
    if (!(FUSED ? position_marked(a, b, t, lane) : a.mask[row] != 0)) {
        if (lane == 0) a.tokens_out[row] = draft;
        return;
    }
    const Guided z{a.logits + row * V, a.logits_u ? a.logits_u + row * V : nullptr, a.cfg_scale};
    bool use_p = a.resample_mode == 2 || (a.resample_mode == 1 && a.accept[row] != 0);
    const int qr = a.q_row ? a.q_row[t] : t;
    const float4* q4 = a.q ? reinterpret_cast<const float4*>(a.q + b * a.q_batch_stride + (int64_t)qr * V) : nullptr;
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    const float m = a.rowmax[row], inv = fabsf(a.rowinv[row]);
    unsigned long long v = lane < nchunks ? sums[row * nchunks + lane] : 0ull, tot = wave_sum_u64(v);
    if (tot == 0 && !use_p) {                                  // empty residual: draw from p instead
        use_p = true;
        v = 0;
        for (int c = 0; c < nchunks; ++c) {
            const int idx = c * 64 + lane;
            unsigned long long w[4] = {0, 0, 0, 0};
            if (idx < nv4) weights4(z.at4(idx), zero4, m, inv, true, w);
            const unsigned long long s = wave_sum_u64((w[0] + w[1]) + (w[2] + w[3]));
            if (lane == c) v = s;
        }
        tot = wave_sum_u64(v);
    }
    if (tot == 0) return;                                      // as cdf_draw: nothing to draw from, nothing written
    const uint32_t word = philox_word0((uint32_t)t, (uint32_t)b, a.ctr_lo, a.ctr_hi24 | (1u << 24), a.key0, a.key1);
    const unsigned long long T = __umul64hi((unsigned long long)word << 32, tot);
    const unsigned long long incl_c = wave_scan_u64(v, lane);
    const unsigned long long hit_c = __ballot(incl_c > T);
    const int cidx = hit_c ? __ffsll((long long)hit_c) - 1 : nchunks - 1;
    const unsigned long long before = __shfl(incl_c - v, cidx);
    const int idx = cidx * 64 + lane;
    unsigned long long w[4] = {0, 0, 0, 0};
    if (idx < nv4) weights4(z.at4(idx), use_p ? zero4 : q4[idx], m, inv, use_p, w);
    const unsigned long long s = (w[0] + w[1]) + (w[2] + w[3]);
    const unsigned long long incl = wave_scan_u64(s, lane) + before;
    const unsigned long long hit = __ballot(incl > T);
    const int f = hit ? __ffsll((long long)hit) - 1 : 63;
    if (lane == f) {
        unsigned long long cum = incl - s;
        int tok = draft;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            cum += w[e];
            if (cum > T) { tok = idx * 4 + e; break; }
        }
        a.tokens_out[row] = clamp_tok(tok, V);
    }
}

// ---- Alg. 1 Step 6, one position: inputs of the single-token forward, then the draw from p ----
__global__ void k_seq_input(const int32_t* __restrict__ prev, const int32_t* __restrict__ tokens,
                            int32_t* __restrict__ inp, int B, int L, int u) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) inp[b] = u == 0 ? prev[b] : tokens[(int64_t)b * L + u - 1];
}

// one workgroup per sequence: if position u is marked, tokens[b, u] ~ softmax(logits[b, :])
__global__ __launch_bounds__(TPB) void k_seq_draw(const float* __restrict__ logits, const uint8_t* __restrict__ mask,
                                                  int32_t* __restrict__ tokens, int L, int V, int u, uint32_t key0,
                                                  uint32_t key1, uint32_t ctr_lo, uint32_t ctr_hi24) {
    __shared__ unsigned long long chunk[MAX_CHUNKS];
    __shared__ int s_retry;
    __shared__ float red[WAVES];
    const int b = blockIdx.x;
    if (!mask[(int64_t)b * L + u]) return;   // uniform over the workgroup
    const Guided z{logits + (int64_t)b * V, nullptr, 1.f};
    RowRegs<0> none;
    float m, inv;
    row_stats<0>(z, V, none, red, m, inv);
    const uint32_t word = philox_word0((uint32_t)u, (uint32_t)b, ctr_lo, ctr_hi24 | (2u << 24), key0, key1);
    int32_t* out = tokens + (int64_t)b * L + u;
    cdf_draw(z, reinterpret_cast<const float4*>(z.zc), m, inv, true, word, V, *out, out, chunk, &s_retry);
}

// ---- island-parallel re-sampling (Sec. 3.4): one pass handles the rank-`pass` position of every island ----
// One workgroup per sequence.  All threads write the pass's hidden set (marked positions whose rank is >= pass:
// not re-drawn yet); the first wavefront then deals the positions of rank == pass to the sequence's `cap` slots in
// raster order (ballot + prefix count, so the slot of a position does not depend on timing): its cache row, and
// its input token = the current token of the position before it.  Unused slots get row -1.
__global__ __launch_bounds__(TPB) void k_island_select(const int32_t* __restrict__ prev, const int32_t* __restrict__ tokens,
                                                       const uint8_t* __restrict__ mask, const int32_t* __restrict__ rank,
                                                       int32_t* __restrict__ pos_tab, int32_t* __restrict__ inp,
                                                       uint8_t* __restrict__ hide, int32_t* __restrict__ overflow, int L,
                                                       int P, int cap, int pass) {
    const int b = blockIdx.x, tid = threadIdx.x;
    const uint8_t* mk = mask + (int64_t)b * L;
    const int32_t* rk = rank + (int64_t)b * L;
    for (int t = tid; t < L; t += TPB) hide[(int64_t)b * L + t] = mk[t] && rk[t] >= pass;
    if (tid >= 64) return;
    int cnt = 0;
    for (int base = 0; base < L; base += 64) {
        const int t = base + tid;
        const bool sel = t < L && mk[t] && rk[t] == pass;
        const unsigned long long bal = __ballot(sel);
        const int slot = cnt + __popcll(bal & ((1ull << tid) - 1ull));
        if (sel && slot < cap) {
            pos_tab[b * cap + slot] = P + t;
            inp[b * cap + slot] = t == 0 ? prev[b] : tokens[(int64_t)b * L + t - 1];
        }
        cnt += __popcll(bal);
    }
    for (int slot = cnt + tid; slot < cap; slot += 64) {
        pos_tab[b * cap + slot] = -1;
        inp[b * cap + slot] = 0;
    }
    if (tid == 0 && cnt > cap && overflow) atomicAdd(overflow, cnt - cap);   // the caller's bound was too small
}

// one workgroup per slot: tokens[sequence, u] ~ softmax(logits[slot, :]) for the position u the slot holds.  The row is copied
// with 16-byte accesses and the statistics keep it in registers between their two passes (V <= 1024 NV4; 0: re-read); the copy,
// the statistics and the draw each read it, the second and third time from the L2: 30 -> 13 us for 52 slots of 16384.
template <int NV4>
__global__ __launch_bounds__(TPB) void k_island_draw(const float* __restrict__ logits, const int32_t* __restrict__ pos_tab,
                                                     int32_t* __restrict__ tokens, float* __restrict__ logits_out, int L,
                                                     int V, int P, int cap, uint32_t key0, uint32_t key1, uint32_t ctr_lo,
                                                     uint32_t ctr_hi24) {
    __shared__ unsigned long long chunk[MAX_CHUNKS];
    __shared__ int s_retry;
    __shared__ float red[WAVES];
    const int v = blockIdx.x, b = v / cap, row = pos_tab[v];
    if (row < 0) return;   // uniform over the workgroup
    const int u = row - P;
    const Guided z{logits + (int64_t)v * V, nullptr, 1.f};
    if (logits_out) {
        float* const dst = logits_out + ((int64_t)b * L + u) * V;
        const int nv4 = V >> 2;
        if ((reinterpret_cast<uintptr_t>(dst) & 15) == 0) {   // uniform; the caller's buffer
#pragma unroll 4
            for (int c = threadIdx.x; c < nv4; c += TPB) reinterpret_cast<float4*>(dst)[c] = reinterpret_cast<const float4*>(z.zc)[c];
        } else {
            for (int c = threadIdx.x; c < V; c += TPB) dst[c] = z.zc[c];
        }
    }
    RowRegs<NV4> rr;
    float m, inv;
    row_stats<NV4>(z, V, rr, red, m, inv);
    const uint32_t word = philox_word0((uint32_t)u, (uint32_t)b, ctr_lo, ctr_hi24 | (2u << 24), key0, key1);
    int32_t* out = tokens + (int64_t)b * L + u;
    cdf_draw(z, reinterpret_cast<const float4*>(z.zc), m, inv, true, word, V, *out, out, chunk, &s_retry);
}

// ---- rejection islands (Eq. 8): 8-connected components of the marked set, one workgroup per sequence ----
// Latency is all there is here (a block of labels, no memory traffic), so the phases are few, with one position per thread
// (of 1024; longer blocks take strided passes):
//   union-find in LDS: lab[t] names a marked position of t's island that is not after t (unmarked: -1); a position is
//     linked to its earlier neighbours (left and the three above) by atomicMin on the larger root, so an island's root
//     is its smallest position; every find descends strictly, so every loop ends;
//   members per (segment of the block, island) by atomics, their prefix over the segments, islands and largest island;
//   ranks: a wavefront per segment walks its 64-position chunks in order; a ballot per island present in the chunk
//     ranks its members, a counter per (segment, island) carries on to the next chunk.
// What is not constant: a find follows the links it meets; a chunk takes a step per island in it; the counters of a segment are
// L integers of LDS, so 16 wavefronts share the walk of 1024 positions, 8 that of 4096 and one that of 16384.
// Us, min-label rounds and a scan of the island per position / this: 1024 positions, nothing marked 5.3 / 5.4 (a launch), 0.3 % 62 / 5.4,
// half 201 / 9.9, all 167 / 8.4; 16384 positions, nothing marked 19.5 / 6.1, 2 % 22000 / 88, half 38000 / 153.
constexpr int ISL_TPB = 1024;
constexpr int ISL_LDS = 160 * 1024 - 256;
__global__ __launch_bounds__(ISL_TPB) void k_islands(const uint8_t* __restrict__ mask, int32_t* __restrict__ island,
                                                     int32_t* __restrict__ rank, int32_t* __restrict__ counts, int W,
                                                     int n0, int L, int segs) {
    extern __shared__ int lab[];   // [L]
    int* const cnt = lab + L;      // [segs][L], by root
    __shared__ int n_isl, largest, some[ISL_TPB / 64];
    const int b = blockIdx.x, tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wv = tid >> 6;
    const uint8_t* mk = mask + (int64_t)b * L;
    const int seg_len = ((L + segs - 1) / segs + 63) / 64 * 64;
    if (tid == 0) n_isl = largest = 0;
    int marked = 0;
    for (int t = tid; t < L; t += nt) {
        const int m = mk[t];
        marked |= m;
        lab[t] = m ? t : -1;
    }
    for (int i = tid; i < segs * L; i += nt) cnt[i] = 0;
    const unsigned long long in_wave = __ballot(marked != 0);
    if (lane == 0) some[wv] = in_wave != 0;
    __syncthreads();
    int any = 0;
    for (int i = 0; i < (nt >> 6); ++i) any |= some[i];
    if (!any) {   // nothing is marked: the walk below would still visit every position (39 us for 16384)
        for (int t = tid; t < L; t += nt) {
            island[(int64_t)b * L + t] = 0;
            rank[(int64_t)b * L + t] = -1;
        }
        if (tid < 2) counts[b * 2 + tid] = 0;
        return;
    }
    volatile int* const vl = lab;
    auto find = [&](int x) {   // halves the path on its way: a position that is no root keeps being none, any ancestor will do for it
        for (int p = vl[x]; p != x; p = vl[x]) {
            const int q = vl[p];
            if (q != p) vl[x] = q;
            x = q;
        }
        return x;
    };
    auto unite = [&](int x, int y) {
        while (true) {
            x = find(x);
            y = find(y);
            if (x == y) return;
            if (x < y) { const int z = x; x = y; y = z; }
            const int old = atomicMin(&lab[x], y);
            if (old == x) return;   // x was still a root
            x = old;
        }
    };
    for (int t = tid; t < L; t += nt) {
        if (vl[t] < 0) continue;
        const int j = (n0 + t) % W;   // the block is whole rows of the grid
        if (j > 0 && vl[t - 1] >= 0) unite(t, t - 1);
        if (t >= W) {
            if (vl[t - W] >= 0) {
                unite(t, t - W);      // the other two above are its neighbours
            } else {
                if (j > 0 && vl[t - W - 1] >= 0) unite(t, t - W - 1);
                if (j < W - 1 && vl[t - W + 1] >= 0) unite(t, t - W + 1);
            }
        }
    }
    __syncthreads();
    for (int t = tid; t < L; t += nt)
        if (vl[t] >= 0) {
            int r = t;
            for (int p = vl[r]; p != r; p = vl[r]) r = p;   // reads only: a path halved here could undo another thread's vl[t] = r
            vl[t] = r;
            atomicAdd(&cnt[(t / seg_len) * L + r], 1);
        }
    __syncthreads();
    for (int t = tid; t < L; t += nt)
        if (lab[t] == t) {   // an island's root: where each segment's members start, and the island's size
            int run = 0;
            for (int s = 0; s < segs; ++s) {
                const int c = cnt[s * L + t];
                cnt[s * L + t] = run;
                run += c;
            }
            atomicAdd(&n_isl, 1);
            atomicMax(&largest, run);
        }
    __syncthreads();
    if (tid == 0) { counts[b * 2] = n_isl; counts[b * 2 + 1] = largest; }
    if (wv >= segs) return;
    const int t_end = (wv + 1) * seg_len < L ? (wv + 1) * seg_len : L;
    for (int t0 = wv * seg_len; t0 < t_end; t0 += 64) {
        const int t = t0 + lane, l = t < t_end ? lab[t] : -1;
        int r = -1;
        for (unsigned long long left = __ballot(l >= 0); left;) {
            const int lead = __ffsll((long long)left) - 1, ll = __builtin_amdgcn_readlane(l, lead);
            const unsigned long long m = __ballot(l == ll);
            volatile int* const c = cnt + wv * L + ll;   // another lane may have written it
            const int base = *c;
            if (l == ll) r = base + __popcll(m & ((1ull << lane) - 1ull));
            if (lane == lead) *c = base + __popcll(m);
            left &= ~m;
        }
        if (t < t_end) {
            island[(int64_t)b * L + t] = l + 1;
            rank[(int64_t)b * L + t] = r;
        }
    }
}

template <int NV4>
void softmax_rows_inst(const float* in, float* out, int64_t rows, int V, const UpTokens& up, hipStream_t st) {
    hipLaunchKernelGGL(k_softmax_rows<NV4>, dim3((unsigned)rows), dim3(TPB), 0, st, in, out, V, up);
}
}  // namespace

void launch_softmax_rows(const float* in, float* out, int64_t rows, int V, const UpTokens& up, hipStream_t st) {
    if (rows <= 0) return;
    if (V <= 1024) softmax_rows_inst<1>(in, out, rows, V, up, st);
    else if (V <= 2048) softmax_rows_inst<2>(in, out, rows, V, up, st);
    else if (V <= 4096) softmax_rows_inst<4>(in, out, rows, V, up, st);
    else if (V <= 8192) softmax_rows_inst<8>(in, out, rows, V, up, st);
    else if (V <= 16384) softmax_rows_inst<16>(in, out, rows, V, up, st);
    else softmax_rows_inst<0>(in, out, rows, V, up, st);
}

void launch_copy_rows(const float* in, float* out, int64_t n_floats, hipStream_t st) {
    if (n_floats <= 0 || in == out) return;
    const int64_t n4 = n_floats >> 2;
    const unsigned blocks = (unsigned)((n4 + TPB - 1) / TPB < 65536 ? (n4 + TPB - 1) / TPB : 65536);
    hipLaunchKernelGGL(k_copy, dim3(blocks), dim3(TPB), 0, st, reinterpret_cast<const float4*>(in),
                       reinterpret_cast<float4*>(out), n4);
}

void launch_copy_rows_strided(const float* src, float* dst, int B, int V, int64_t dst_stride, hipStream_t st) {
    if (B <= 0 || V <= 0) return;
    const int nv4 = V >> 2;
    hipLaunchKernelGGL(k_copy_rows_strided, dim3((nv4 + TPB - 1) / TPB < 64 ? (nv4 + TPB - 1) / TPB : 64, B), dim3(TPB), 0, st,
                       reinterpret_cast<const float4*>(src), dst, nv4, dst_stride);
}

void launch_upsample_tokens(const int32_t* draft_tokens, int32_t* tokens_hi, int32_t* q_row, int B,
                            int h, int w, int r, hipStream_t st) {
    const int64_t n = (int64_t)B * h * r * w * r;
    hipLaunchKernelGGL(k_upsample_tokens, dim3((unsigned)((n + TPB - 1) / TPB)), dim3(TPB), 0, st,
                       draft_tokens, tokens_hi, q_row, B, h, w, r);
}

void launch_gather_rows(const float* q_lo, const int32_t* q_row, float* q_hi, int B, int n_lo,
                        int n_hi, int V, hipStream_t st) {
    hipLaunchKernelGGL(k_gather_rows, dim3(n_hi, B), dim3(TPB), 0, st, q_lo, q_row, q_hi, n_lo, n_hi, V);
}

// one thread per position of a block, whole wavefronts, between `least` and 1024
static int block_threads(int L, int least) {
    const int t = L >= 1024 ? 1024 : (L + 63) / 64 * 64;
    return t < least ? least : t;
}

void launch_islands(const uint8_t* mask, int32_t* island, int32_t* rank, int32_t* counts, int B, int W, int n0, int L,
                    hipStream_t st) {   // L <= 16384 (the caller checks): labels and at least one set of counters in LDS
    static int attr_state = 0;
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(k_islands), ISL_LDS, &attr_state)) return;
    const int threads = block_threads(L, 64);
    const int fit = ISL_LDS / ((int)sizeof(int) * L) - 1, segs = fit < threads / 64 ? fit : threads / 64;   // counters [segs][L] next to the labels [L]
    hipLaunchKernelGGL(k_islands, dim3(B), dim3(threads), (size_t)(1 + segs) * L * sizeof(int), st, mask, island, rank, counts, W, n0,
                       L, segs);
}

void launch_seq_input(const int32_t* prev, const int32_t* tokens, int32_t* inp, int B, int L, int u, hipStream_t st) {
    hipLaunchKernelGGL(k_seq_input, dim3((B + 63) / 64), dim3(64), 0, st, prev, tokens, inp, B, L, u);
}

void launch_seq_draw(const float* logits, const uint8_t* mask, int32_t* tokens, int B, int L, int V, int u,
                     uint64_t seed, uint64_t rng_counter, hipStream_t st) {
    hipLaunchKernelGGL(k_seq_draw, dim3(B), dim3(TPB), 0, st, logits, mask, tokens, L, V, u,
                       (uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32), (uint32_t)(rng_counter & 0xFFFFFFFFu),
                       (uint32_t)((rng_counter >> 32) & 0xFFFFFFu));
}

void launch_island_select(const int32_t* prev, const int32_t* tokens, const uint8_t* mask, const int32_t* rank,
                          int32_t* pos_tab, int32_t* inp, uint8_t* hide, int32_t* overflow, int B, int L, int P,
                          int cap, int pass, hipStream_t st) {
    hipLaunchKernelGGL(k_island_select, dim3(B), dim3(TPB), 0, st, prev, tokens, mask, rank, pos_tab, inp, hide,
                       overflow, L, P, cap, pass);
}

void launch_island_draw(const float* logits, const int32_t* pos_tab, int32_t* tokens, float* logits_out, int B,
                        int L, int V, int P, int cap, uint64_t seed, uint64_t rng_counter, hipStream_t st) {
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(B * cap), dim3(TPB), 0, st, logits, pos_tab, tokens, logits_out, L, V, P, cap,
                           (uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32), (uint32_t)(rng_counter & 0xFFFFFFFFu),
                           (uint32_t)((rng_counter >> 32) & 0xFFFFFFu));
    };
    if (V <= 4096) go(k_island_draw<4>);
    else if (V <= 8192) go(k_island_draw<8>);
    else if (V <= 16384) go(k_island_draw<16>);
    else go(k_island_draw<0>);
}

// the counters and the mask, in front of a re-draw that does not make them itself; returns how many workgroups of it do (0: none)
// The re-draw makes them where the launch it saves, 3 to 6 us of a decision, is more than the look that every position takes at
// its window.  us of a decision, launch / none, 1024 entries a row, 60 % accepted and radius 1 where nothing else is said:
//   k_mask_sample: 1 x 256 13.0 / 10.8, 4 x 1024 of radius 2 30.1 / 25.8, 1 x 4096 35.8 / 25.9, of 16384 entries 4 x 1024 143 / 138; but
//     8 x 1024 48.2 / 45.8 and with next to all accepted and radius 0 26.5 / 28.8, 64 x 256 there 38.4 / 49.1, 16 x 1024 81.6 / 83.8
//     and 39.8 / 49.3: up to 4096 positions of all sequences
//   k_sample_sums, four positions a workgroup: 4 x 1024 of radius 2 23.8 / 18.2, 2 x 2048 with 3 % rejected and radius 3 35.8 / 20.3, 16 x 1024
//     52.7 / 48.6, 4 x 4096 56 / 51, 64 x 256 50.1 / 48.7 (30 % accepted): up to 16384
// 1 x 4096 positions can lose by it (radius 8, 20 % accepted, 25.8 / 27.0) and win by it (1 rejected of a thousand, 159 / 33).
static int decide_finish(const DecideArgs& a, int most, hipStream_t st) {   // a.L <= 131072 (the caller checks): flags in LDS
    if (a.L <= FUSED_L && (int64_t)a.B * a.L <= most) return (a.B + 7) / 8 * 8;
    static int attr_state = 0;
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(k_decide_finish), 131072, &attr_state)) return 0;
    hipLaunchKernelGGL(k_decide_finish, dim3(a.B), dim3(a.rho > 0 ? block_threads(a.L, 256) : 256), (size_t)a.L, st, a);
    return 0;
}

bool launch_accept(const DecideArgs& a, unsigned long long* sums, hipStream_t st) {
    // Chunk sums with the test where residual weights are drawn from and a neighbourhood marks most positions around the
    // rejections: Eq. 1 without pooling, whose acceptance is 1 - TV(p, q), 0.8 to 0.3 in the workloads.  Unmarked positions
    // pay for it, so the gain depends on the acceptance a.  4 x 1024 x 16384, test + mask + draw in us, this / the test alone
    // and a draw that reads the marked rows again:
    //   draft rows shared by 4 positions: radius 1: a = 0.38 90 / 111, 0.88 88 / 87, 0.96 88 / 73, 0.99 88 / 64;
    //     radius 2: 0.38 89 / 111, 0.88 85 / 102, 0.96 85 / 85, 0.99 86 / 70;
    //   a row each: radius 1: 0.62 104 / 136, 0.88 103 / 104, 0.96 103 / 77; radius 2: 0.62 104 / 139, 0.88 109 / 135, 0.96 109 / 95.
    // They cross at a = 0.88 (radius 1) and 0.95 (radius 2).  Not here: pooled and threshold tests, made to accept nearly
    // everything (and the threshold reads no draft row); radius 0, which marks the rejected positions alone; draws from p,
    // which have little to re-read (guided, 2 x 1024, threshold rule: 65 / 62).
    if (sums && !a.p_probs && a.V <= 16384 && a.accept_mode == 0 && a.pool_k <= 1 && a.resample_mode != 2 && a.rho != 0) {
        const int rows_per = (int)(((int64_t)a.B * a.L + 7) / 8);
        auto go = [&](auto nit) {
            constexpr int NIT = decltype(nit)::value;
            if (a.logits_u) hipLaunchKernelGGL((k_accept_sums<NIT, true>), dim3((unsigned)rows_per * 8), dim3(TPB), 0, st, a, sums, rows_per);
            else hipLaunchKernelGGL((k_accept_sums<NIT, false>), dim3((unsigned)rows_per * 8), dim3(TPB), 0, st, a, sums, rows_per);
        };
        if (a.V <= 2048) go(std::integral_constant<int, 1>{});
        else if (a.V <= 4096) go(std::integral_constant<int, 2>{});
        else if (a.V <= 8192) go(std::integral_constant<int, 4>{});
        else if (a.V <= 12288) go(std::integral_constant<int, 6>{});   // 10004 entries, 1152 rows: 50 -> 45 us with 6 of 8 passes
        else go(std::integral_constant<int, 8>{});
        return true;
    }
    if (a.logits_u) hipLaunchKernelGGL(k_accept<true>, dim3((unsigned)(a.B * a.L)), dim3(TPB), 0, st, a);
    else hipLaunchKernelGGL(k_accept<false>, dim3((unsigned)(a.B * a.L)), dim3(TPB), 0, st, a);
    return false;
}

void launch_sample_sums(const DecideArgs& a, const unsigned long long* sums, hipStream_t st) {
    const int64_t rows = (int64_t)a.B * a.L;
    const int n_fin = decide_finish(a, 16384, st);
    const dim3 grid((unsigned)((rows + WAVES - 1) / WAVES + n_fin));
    if (n_fin) hipLaunchKernelGGL(k_sample_sums<true>, grid, dim3(TPB), 0, st, a, sums, n_fin);
    else hipLaunchKernelGGL(k_sample_sums<false>, grid, dim3(TPB), 0, st, a, sums, 0);
}

void launch_accept_from_parts(const DecideArgs& a, const float* parts, int n_parts, hipStream_t st) {
    const int64_t rows = (int64_t)a.B * a.L;
    hipLaunchKernelGGL(k_accept_parts, dim3((unsigned)((rows + WAVES - 1) / WAVES)), dim3(TPB), 0, st, a,
                       reinterpret_cast<const float2*>(parts), n_parts);
}

void launch_mask_sample(const DecideArgs& a, hipStream_t st) {
    unsigned blocks = (unsigned)(a.B * a.L);
    if (a.up_r > 1) {   // whole groups of 8 draft rows (one per XCD), r * r workgroups each
        const int r2 = a.up_r * a.up_r;
        const int64_t parents = (int64_t)a.B * (a.L / r2);
        blocks = (unsigned)(((parents + 7) / 8) * 8 * r2);
    }
    const int n_fin = decide_finish(a, 4096, st);
    if (n_fin) hipLaunchKernelGGL(k_mask_sample<true>, dim3(blocks + n_fin), dim3(TPB), 0, st, a, n_fin);
    else hipLaunchKernelGGL(k_mask_sample<false>, dim3(blocks), dim3(TPB), 0, st, a, 0);
}

}  // namespace mulo
