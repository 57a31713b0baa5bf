// The float32 decoder (small configurations): projections, attention and their fused epilogues on the float32
// matrix instruction v_mfma_f32_16x16x4_f32 (exact float32 products and sums).
//
// What bounds it: nothing of the chip.  The tiny configuration has 256 tokens of width 256; a projection is 34 to 180
// MFLOP over operands that sit in the L2, so a launch costs its launch (about 4.5 us back to back) plus one chain of
// memory latencies.  Two things follow: few launches (RMSNorm is part of the projection behind it, rotary and the
// cache append or the SwiGLU product part of the projection before it: 5 launches per layer instead of 13), and a
// short chain: no LDS staging, every lane loads its operand fragments straight from memory, all the loads of a tile in
// flight together, and the four wavefronts of a workgroup split K.
//
// Operand order: a lane's float4 of row lane % 16 holds k = 16 s + 4 q .. + 3 (q = lane / 16); MFMA j of step s takes
// component j of both operands, so its four k are 16 s + 4 q + j: a permutation of k inside a step, the same for both.
// Weight rows feed the instruction's rows and tokens its columns: accumulator i of a lane is column 4 q + i of token
// lane % 16, so a rotary pair sits in one lane.
// Step of 256 tokens at the tiny configuration: 1003 -> 99 us (plain 64 x 64 tile kernel: 61 us a projection, with 16
// to 64 workgroups; row-per-workgroup attention 21 us).
#include "mulo_internal.h"

namespace mulo {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

enum { F32_QKV = 0, F32_RESID = 1, F32_SWIGLU = 2, F32_LOGITS = 3 };

struct F32Args {
    const float* A;          // [M, K] token operand
    const float* gain;       // QKV, SWIGLU: A is the residual stream, its RMSNorm with this gain is multiplied
    float eps;
    const float *W0, *W1, *W2;   // QKV: wq, wk, wv | SWIGLU: gate, up | else W0
    int M, N, K;             // N: output columns (QKV: 3 d, SWIGLU: f)
    int d;                   // QKV: columns per matrix
    float* C;                // RESID: x [M, N] (+=) | SWIGLU: h [M, N] | LOGITS: [M, N] | QKV: q buffer
    float *kc, *vc;
    RopeArgs ra;
};

// four consecutive floats of a row from k on; elements at or past K are zeros.  V4: rows are 16-byte aligned and K is a
// multiple of 4; otherwise the address is a multiple of 4 bytes only (one load all the same where four floats exist)
template <bool V4>
__device__ __forceinline__ f32x4 load4(const float* row, int k, int K) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if constexpr (V4) {
        if (k < K) v = *reinterpret_cast<const f32x4*>(row + k);
    } else if (k + 4 <= K) {
        __builtin_memcpy(&v, row + k, sizeof(v));
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (k + e < K) v[e] = row[k + e];
    }
    return v;
}

// output columns n, n + 1 of token m (n even; v1: the up sums of a SwiGLU column)
template <int EPI>
__device__ __forceinline__ void emit2(const F32Args& g, int m, int n, const float (&v0)[2], const float (&v1)[2]) {
    if constexpr (EPI == F32_QKV) {
        if (n >= g.N) return;                            // d is even: a pair lies inside one matrix and one head
        const int seg = n / g.d, c = n - seg * g.d, dh = g.ra.head_dim, hd = c / dh, cc = c % dh;
        const int b = m / g.ra.L, j = m % g.ra.L, pos = g.ra.P + j;
        const int64_t hb = ((int64_t)g.ra.layer * g.ra.max_batch + b) * g.ra.n_heads + hd;
        if (seg == 2) {
            float* v = g.vc + (hb * dh + cc) * g.ra.max_seq + pos;
            v[0] = v0[0];
            v[g.ra.max_seq] = v0[1];
            return;
        }
        const float cs = g.ra.cos[(int64_t)pos * (dh / 2) + cc / 2], sn = g.ra.sin[(int64_t)pos * (dh / 2) + cc / 2];
        float* o = seg == 0 ? g.C + (((int64_t)b * g.ra.n_heads + hd) * g.ra.L + j) * dh + cc
                            : g.kc + (hb * g.ra.max_seq + pos) * dh + cc;
        o[0] = v0[0] * cs - v0[1] * sn;
        o[1] = v0[0] * sn + v0[1] * cs;
    } else {
        float* o = g.C + (int64_t)m * g.N + n;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (n + e >= g.N) continue;
            if constexpr (EPI == F32_RESID) o[e] += v0[e];
            else if constexpr (EPI == F32_SWIGLU) o[e] = v0[e] / (1.0f + expf(-v0[e])) * v1[e];
            else o[e] = v0[e];
        }
    }
}

// A 16 R x 16 R tile per workgroup; its 4 wavefronts each compute all of it over a quarter of K (every fourth step) and add up
// through LDS in wavefront order.  The order of a sum is that of its K alone, whatever R: a sequence gets the same bits
// alone, in a batch, and a token at a time.
template <int EPI, int R, bool V4>
__global__ __launch_bounds__(256) void k_proj_f32(const F32Args g) {
    constexpr int NA = EPI == F32_SWIGLU ? 2 : 1;
    constexpr bool NORM = EPI == F32_QKV || EPI == F32_SWIGLU;
    constexpr int U = R == 1 ? 4 : 2;                               // steps in flight
    __shared__ float part[4][NA][R * R][4][64];
    __shared__ float ssq[4][R][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, q = lane >> 4;
    const int tiles_n = (g.N + 16 * R - 1) / (16 * R);
    const int m0 = blockIdx.x / tiles_n * 16 * R, n0 = blockIdx.x % tiles_n * 16 * R;
    const float *pa[R], *pw[NA][R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int m = m0 + i * 16 + l16;
        pa[i] = g.A + (int64_t)(m < g.M ? m : g.M - 1) * g.K;
        int n = n0 + i * 16 + l16;
        n = n < g.N ? n : g.N - 1;
        if constexpr (EPI == F32_QKV) {
            const int seg = n / g.d;
            pw[0][i] = (seg == 0 ? g.W0 : seg == 1 ? g.W1 : g.W2) + (int64_t)(n - seg * g.d) * g.K;
        } else {
            pw[0][i] = g.W0 + (int64_t)n * g.K;
            if constexpr (EPI == F32_SWIGLU) pw[1][i] = g.W1 + (int64_t)n * g.K;
        }
    }
    f32x4 acc[NA][R][R];
    float ss[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        ss[i] = 0.f;
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int j = 0; j < R; ++j) acc[a][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int steps = (g.K + 15) / 16;
    f32x4 xa[U][R], xw[U][NA][R], xg[U];
    auto request = [&](int s0) {                          // steps past the last load zeros
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (s0 + u * 4) * 16 + q * 4;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                xa[u][i] = load4<V4>(pa[i], k, g.K);
#pragma unroll
                for (int a = 0; a < NA; ++a) xw[u][a][i] = load4<V4>(pw[a][i], k, g.K);
            }
            if constexpr (NORM) xg[u] = load4<V4>(g.gain, k, g.K);
        }
    };
    request(wave);
    for (int s = wave; s < steps; s += U * 4) {
        f32x4 ca[U][R], cw[U][NA][R];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < R; ++i) {
                ca[u][i] = xa[u][i];
                if constexpr (NORM) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) ss[i] += xa[u][i][e] * xa[u][i][e];
                    ca[u][i] *= xg[u];
                }
#pragma unroll
                for (int a = 0; a < NA; ++a) cw[u][a][i] = xw[u][a][i];
            }
        if (s + U * 4 < steps) request(s + U * 4);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int a = 0; a < NA; ++a)
#pragma unroll
                    for (int i = 0; i < R; ++i)
#pragma unroll
                        for (int j = 0; j < R; ++j)
                            acc[a][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(cw[u][a][j][e], ca[u][i][e], acc[a][i][j], 0, 0, 0);
    }
    // the squares of a row are spread over the four q and over the wavefronts
#pragma unroll
    for (int i = 0; i < R; ++i) {
        ss[i] += __shfl_xor(ss[i], 16);
        ss[i] += __shfl_xor(ss[i], 32);
        if (NORM && q == 0) ssq[wave][i][l16] = ss[i];
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int r = 0; r < 4; ++r) part[wave][a][i * R + j][r][lane] = acc[a][i][j][r];
    }
    __syncthreads();
    // block blk = (i, j) of the tile, columns 4 q + 2 pr, + 1: two pairs of columns per block, dealt to the wavefronts
    for (int x = wave; x < 2 * R * R; x += 4) {
        const int blk = x >> 1, pr = x & 1, i = blk / R, m = m0 + i * 16 + l16;
        float sc = 1.0f;                                  // 1 / rms of the lane's token
        if constexpr (NORM)
            sc = 1.0f / sqrtf(((ssq[0][i][l16] + ssq[1][i][l16]) + (ssq[2][i][l16] + ssq[3][i][l16])) / (float)g.K + g.eps);
        float v[2][2] = {};
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int r = 2 * pr + e;
                v[a][e] = (part[0][a][blk][r][lane] + part[1][a][blk][r][lane]) + (part[2][a][blk][r][lane] + part[3][a][blk][r][lane]);
                if constexpr (NORM) v[a][e] *= sc;
            }
        if (m < g.M) emit2<EPI>(g, m, n0 + blk % R * 16 + 4 * q + 2 * pr, v[0], v[1]);
    }
}

// 32 x 32 tiles halve the operand bytes per product and launch a quarter of the workgroups.  Measured, 16 / 32, us: outputs
// 256 x 768 7.2 / 7.6, 384 x 768 10.5 / 11.0, 384 x 1024 9.2 / 7.8, 512 x 768 12.9 / 10.9, 1024 x 768 19 / 12.7; K = 688:
// 1024 x 256 11.5 / 10.4, 1536 x 256 15.4 / 13.7, 2304 x 256 21.5 / 19.1; gate | up 256 x 688 8.8 / 9.3, 512 x 688 14.2 / 13.0,
// 2304 x 688 46 / 36 (64 x 64 tiles, which add in another order: 32).
constexpr int64_t WIDE_FROM = 300 * 1024;

template <int EPI>
void run_proj(const F32Args& g, hipStream_t st) {
    const bool wide = (int64_t)g.M * g.N >= WIDE_FROM, v4 = (g.K & 3) == 0;
    const int t = wide ? 32 : 16;
    const dim3 grid((unsigned)((int64_t)((g.M + t - 1) / t) * ((g.N + t - 1) / t)));
    if (wide) {
        if (v4) hipLaunchKernelGGL((k_proj_f32<EPI, 2, true>), grid, dim3(256), 0, st, g);
        else hipLaunchKernelGGL((k_proj_f32<EPI, 2, false>), grid, dim3(256), 0, st, g);
    } else {
        if (v4) hipLaunchKernelGGL((k_proj_f32<EPI, 1, true>), grid, dim3(256), 0, st, g);
        else hipLaunchKernelGGL((k_proj_f32<EPI, 1, false>), grid, dim3(256), 0, st, g);
    }
}

// Attention of 16 queries of one (head, sequence) per workgroup; its NW wavefronts take every NW-th tile of 16 keys with a
// running maximum and sum of their own, merged through LDS at the end (a wavefront's tiles are one chain of latencies:
// 8 wavefronts where their outputs fit the LDS, and a tile's operands are requested while the one before is multiplied).  S^T = K Q^T and O^T = V^T P^T, both operands
// straight from memory in the order of the projections above: a lane holds keys 4 q .. 4 q + 3 of query lane % 16, which
// is what the second product takes, so the probabilities never leave their registers.  NB = ceil(head_dim / 16).
// 256 queries, 288 keys, 4 heads: 21 -> 12 us (one workgroup per query before: scores in LDS, strided key reads).
// FULL: head_dim is 16 NB and max_seq a multiple of 4, so every access is one of 16 bytes inside its row, without the branches that
// the ends of rows ask for (four a load, 36 loads a tile).
template <int NB, int NW, bool FULL>
__global__ __launch_bounds__(NW * 64) void k_attn_mfma_f32(const float* __restrict__ qb, const float* __restrict__ kc,
                                                       const float* __restrict__ vc, float* __restrict__ out, int L, int P,
                                                       int nh, int dh, int max_seq, int max_batch, int layer) {
    __shared__ float so[NW][NB * 16][17];
    __shared__ float sm[NW][16], sl[NW][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, q = lane >> 4;
    const int j0 = blockIdx.x * 16, hd = blockIdx.y, b = blockIdx.z;
    const int jq = j0 + l16 < L ? j0 + l16 : L - 1, jlast = j0 + 15 < L ? j0 + 15 : L - 1;
    const int qpos = P + jq, kmax = P + jlast;            // last key of this lane's query, of the workgroup
    const int64_t hb = ((int64_t)layer * max_batch + b) * nh + hd;
    const float* kb = kc + hb * max_seq * dh;
    const float* vb = vc + hb * dh * max_seq;
    const float* qp = qb + (((int64_t)b * nh + hd) * L + jq) * dh;
    const float scale = 1.0f / sqrtf((float)dh), NEG = -__builtin_huge_valf();
    auto at = [](const float* p) { f32x4 v; __builtin_memcpy(&v, p, sizeof(v)); return v; };
    f32x4 qf[NB], o[NB];
#pragma unroll
    for (int s = 0; s < NB; ++s) {
        qf[s] = FULL ? at(qp + s * 16 + q * 4) : load4<false>(qp, s * 16 + q * 4, dh);
        o[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float m_run = NEG, l_run = 0.f;
    f32x4 nk[NB], nv[NB];
    auto request = [&](int k0) {
        const int key = k0 + l16 < kmax ? k0 + l16 : kmax;
        const float* kr = kb + (int64_t)key * dh;
#pragma unroll
        for (int s = 0; s < NB; ++s) nk[s] = FULL ? at(kr + s * 16 + q * 4) : load4<false>(kr, s * 16 + q * 4, dh);
        const int kv = k0 + q * 4 < max_seq ? k0 + q * 4 : max_seq - 4;   // FULL: columns past the cache are the last four again
#pragma unroll
        for (int s = 0; s < NB; ++s) {                    // columns past the last key may be uninitialised: zeros (FULL: below)
            const int c = s * 16 + l16;
            nv[s] = FULL ? at(vb + (int64_t)c * max_seq + kv) : load4<false>(vb + (int64_t)(c < dh ? c : dh - 1) * max_seq, k0 + q * 4, kmax + 1);
        }
    };
    if (wave * 16 <= kmax) request(wave * 16);
    for (int k0 = wave * 16; k0 <= kmax; k0 += 16 * NW) {
        f32x4 kf[NB], vf[NB];
#pragma unroll
        for (int s = 0; s < NB; ++s) { kf[s] = nk[s]; vf[s] = nv[s]; }
        if (FULL && k0 + 15 > kmax) {                     // uniform over the wavefront
#pragma unroll
            for (int s = 0; s < NB; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) vf[s][e] = k0 + q * 4 + e <= kmax ? vf[s][e] : 0.f;
        }
        if (k0 + 16 * NW <= kmax) request(k0 + 16 * NW);
        f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NB; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) p = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[s][e], qf[s][e], p, 0, 0, 0);
        float mx = NEG;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = k0 + q * 4 + e <= qpos ? p[e] * scale : NEG;
            mx = fmaxf(mx, p[e]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx), m_safe = m_new == NEG ? 0.f : m_new, alpha = expf(m_run - m_safe);
        m_run = m_new;
        float ps = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = expf(p[e] - m_safe);
            ps += p[e];
        }
        l_run = l_run * alpha + ps;
#pragma unroll
        for (int s = 0; s < NB; ++s) o[s] *= alpha;
        // A tile that some query sees a part of only: a hidden key's p is 0, and 0 times an infinity or NaN of its V must not
        // reach that query.  Such values are added to the queries that do see them and taken out of the product.
        if (k0 + 15 > P + j0) {
            bool odd = false;
#pragma unroll
            for (int s = 0; s < NB; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) odd |= !__builtin_isfinite(vf[s][e]);
            if (__ballot(odd)) {                              // uniform over the wavefront
                for (int g = 0; g < 4; ++g)                   // key 4 g + e of the tile: V and p sit in the lanes with q = g
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float pk = __shfl(p[e], g * 16 + l16);
                        const bool seen = k0 + g * 4 + e <= qpos;
#pragma unroll
                        for (int s = 0; s < NB; ++s)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const float v = __shfl(vf[s][e], g * 16 + q * 4 + r);
                                if (seen && !__builtin_isfinite(v)) o[s][r] += pk * v;
                            }
                    }
#pragma unroll
                for (int s = 0; s < NB; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) vf[s][e] = __builtin_isfinite(vf[s][e]) ? vf[s][e] : 0.f;
            }
        }
#pragma unroll
        for (int s = 0; s < NB; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[s][e], p[e], o[s], 0, 0, 0);
    }
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    if (q == 0) { sm[wave][l16] = m_run; sl[wave][l16] = l_run; }
#pragma unroll
    for (int s = 0; s < NB; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) so[wave][s * 16 + q * 4 + e][l16] = o[s][e];
    __syncthreads();
    for (int x = tid; x < 16 * dh; x += NW * 64) {
        const int j = x / dh, c = x % dh;
        if (j0 + j >= L) break;
        float m = sm[0][j], num = 0.f, den = 0.f;        // key 0 is visible to every query: m is finite
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmaxf(m, sm[w][j]);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = expf(sm[w][j] - m);
            num += so[w][c][j] * f;
            den += sl[w][j] * f;
        }
        out[((int64_t)b * L + j0 + j) * (nh * dh) + hd * dh + c] = num / den;
    }
}

// Heads wider than 128: one workgroup per (query, head, sequence), scores in LDS.
__global__ __launch_bounds__(256) void k_attn_wide_f32(const float* __restrict__ q, const float* __restrict__ kc,
                                                       const float* __restrict__ vc, float* __restrict__ out, int L,
                                                       int P, int nh, int dh, int max_seq, int max_batch, int layer) {
    extern __shared__ float sc[];   // [dh] query, then [P + j + 1] scores
    __shared__ float red[4];
    const int j = blockIdx.x, hd = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const int n = P + j + 1;
    float* qs = sc;
    float* s = sc + dh;
    const int64_t hb = ((int64_t)layer * max_batch + b) * nh + hd;
    const float* kb = kc + hb * max_seq * dh;
    const float* vb = vc + hb * dh * max_seq;
    for (int c = tid; c < dh; c += 256) qs[c] = q[(((int64_t)b * nh + hd) * L + j) * dh + c];
    __syncthreads();
    const float scale = 1.0f / sqrtf((float)dh);
    float mx = -__builtin_huge_valf();
    for (int t = tid; t < n; t += 256) {
        float acc = 0.f;
        for (int c = 0; c < dh; ++c) acc += qs[c] * kb[(int64_t)t * dh + c];
        acc *= scale;
        s[t] = acc;
        mx = fmaxf(mx, acc);
    }
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    float sum = 0.f;
    for (int t = tid; t < n; t += 256) {
        const float e = expf(s[t] - mx);
        s[t] = e;
        sum += e;
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if ((tid & 63) == 0) red[tid >> 6] = sum;
    __syncthreads();
    sum = (red[0] + red[1]) + (red[2] + red[3]);
    for (int c = tid; c < dh; c += 256) {
        float acc = 0.f;
        for (int t = 0; t < n; ++t) acc += s[t] * vb[(int64_t)c * max_seq + t];
        out[((int64_t)b * L + j) * (nh * dh) + hd * dh + c] = acc / sum;
    }
}

}  // namespace

void launch_qkv_f32(const float* x, const float* gain, float eps, const float* wq, const float* wk, const float* wv, float* q_out,
                    float* k_cache, float* v_cache, int M, int d, const RopeArgs& ra, hipStream_t st) {
    F32Args g{};
    g.A = x; g.gain = gain; g.eps = eps; g.W0 = wq; g.W1 = wk; g.W2 = wv; g.M = M; g.N = 3 * d; g.K = d; g.d = d;
    g.C = q_out; g.kc = k_cache; g.vc = v_cache; g.ra = ra;
    run_proj<F32_QKV>(g, st);
}

void launch_swiglu_f32(const float* x, const float* gain, float eps, const float* wg, const float* wu, float* h, int M, int f,
                       int d, hipStream_t st) {
    F32Args g{};
    g.A = x; g.gain = gain; g.eps = eps; g.W0 = wg; g.W1 = wu; g.M = M; g.N = f; g.K = d; g.C = h;
    run_proj<F32_SWIGLU>(g, st);
}

void launch_resid_f32(const float* a, const float* w, float* x, int M, int N, int K, hipStream_t st) {
    F32Args g{};
    g.A = a; g.W0 = w; g.M = M; g.N = N; g.K = K; g.C = x;
    run_proj<F32_RESID>(g, st);
}

void launch_logits_f32(const float* xh, const float* w, float* logits, int M, int V, int d, hipStream_t st) {
    F32Args g{};
    g.A = xh; g.W0 = w; g.M = M; g.N = V; g.K = d; g.C = logits;
    run_proj<F32_LOGITS>(g, st);
}

void launch_attention_f32(const float* q, const float* k_cache, const float* v_cache, float* out, int B, int L, int P,
                          int n_heads, int head_dim, int max_seq, int max_batch, int layer, hipStream_t st) {
    auto go = [&](auto kern, int waves) {
        hipLaunchKernelGGL(kern, dim3((L + 15) / 16, n_heads, B), dim3(waves * 64), 0, st, q, k_cache, v_cache, out, L, P, n_heads,
                           head_dim, max_seq, max_batch, layer);
    };
    const bool full = (max_seq & 3) == 0;
    if (head_dim == 16 && full) go(k_attn_mfma_f32<1, 8, true>, 8);
    else if (head_dim <= 16) go(k_attn_mfma_f32<1, 8, false>, 8);
    else if (head_dim == 32 && full) go(k_attn_mfma_f32<2, 8, true>, 8);
    else if (head_dim <= 32) go(k_attn_mfma_f32<2, 8, false>, 8);
    else if (head_dim == 64 && full) go(k_attn_mfma_f32<4, 8, true>, 8);
    else if (head_dim <= 64) go(k_attn_mfma_f32<4, 8, false>, 8);
    else if (head_dim == 128 && full) go(k_attn_mfma_f32<8, 4, true>, 4);
    else if (head_dim <= 128) go(k_attn_mfma_f32<8, 4, false>, 4);
    else
        hipLaunchKernelGGL(k_attn_wide_f32, dim3(L, n_heads, B), dim3(256), (size_t)(head_dim + P + L) * sizeof(float), st, q,
                           k_cache, v_cache, out, L, P, n_heads, head_dim, max_seq, max_batch, layer);
}

}  // namespace mulo
