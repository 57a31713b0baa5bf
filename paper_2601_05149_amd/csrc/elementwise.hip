// Row-wise pieces of the target forward (Alg. 1 Step 3): embedding lookup and
// RMSNorm, HBM-bound streams over [M, d] activations.
#include <hip/hip_bf16.h>

#include <type_traits>

#include "mulo_internal.h"

namespace mulo {
namespace {

constexpr int TPB = 256;

__device__ __forceinline__ float ld(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float ld(const __hip_bfloat16* p, int64_t i) { return __bfloat162float(p[i]); }
__device__ __forceinline__ void st(float* p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void st(__hip_bfloat16* p, int64_t i, float v) { p[i] = __float2bfloat16(v); }

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

// Row of the embedding (or of the caller's embeddings) into the float32 stream, one workgroup per row.  VEC: 16-byte loads and
// stores, for rows that allow them; a step's workgroup finds its row's input token itself and writes the position's
// up-sampled token: two launches of 1.5 to 2.3 us less in front of the first layer; element by element a row of 4096 is 16 dependent rounds per lane (one row 7.3 us, in
// 16-byte pieces 4.7; 576 rows 12 and 6.4; 1024 rows of 1024 5.1 and 3.8).
template <typename T, bool VEC>
__global__ __launch_bounds__(TPB) void k_embed(const T* __restrict__ embed, const int32_t* __restrict__ tok,
                                               const T* __restrict__ in_embeds, const StepTokens in, float* __restrict__ x,
                                               int d, int V) {
    const int64_t m = blockIdx.x;
    const T* src;
    if (in_embeds) {
        src = in_embeds + m * d;
    } else {
        int t;
        if (in.up.lo) {
            const int W = in.up.w * in.up.r, L = in.up.h * in.up.r * W, b2 = (int)(m / L), j = (int)(m % L), b = b2 % in.seqs;
            auto cell = [&](int u) { return (u / W / in.up.r) * in.up.w + (u % W) / in.up.r; };   // the draft cell of a position
            const int32_t* const lo = in.up.lo + (int64_t)b * in.up.h * in.up.w;
            t = j == 0 ? in.prev[b] : lo[cell(j - 1)];
            if (threadIdx.x == 0 && b2 == b) {
                const int par = cell(j);
                in.up.hi[m] = lo[par];
                if (b == 0) in.up.q_row[j] = par;
            }
        } else {
            t = tok[m];
        }
        t = t < 0 ? 0 : (t >= V ? V - 1 : t);
        src = embed + (int64_t)t * d;
    }
    if constexpr (VEC) {
        constexpr int W = 16 / sizeof(T);   // elements of a load
        float4* const xr = reinterpret_cast<float4*>(x + m * d);
#pragma unroll 4
        for (int c = threadIdx.x; c < d / W; c += TPB) {
            if constexpr (W == 8) {
                const bf16x8 v = reinterpret_cast<const bf16x8*>(src)[c];
                xr[2 * c] = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
                xr[2 * c + 1] = make_float4((float)v[4], (float)v[5], (float)v[6], (float)v[7]);
            } else {
                xr[c] = reinterpret_cast<const float4*>(src)[c];
            }
        }
    } else {
        for (int c = threadIdx.x; c < d; c += TPB) x[m * d + c] = ld(src, c);
    }
}

// The butterfly sum over a wavefront (lane distances 32, 16, 8, 4, 2, 1).  Inside a row of 16 lanes the sums already repeat with
// period 2 o, so the lane o further round holds what the lane at distance o holds, and no exchange through LDS is needed.
__device__ __forceinline__ float wave_sum(float v) {
    v += __shfl_xor(v, 32);
    v += __shfl_xor(v, 16);
    const auto ror = [](float x, auto n) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x120 + decltype(n)::value, 0xf, 0xf, false));
    };
    v += ror(v, std::integral_constant<int, 8>{});
    v += ror(v, std::integral_constant<int, 4>{});
    v += ror(v, std::integral_constant<int, 2>{});
    v += ror(v, std::integral_constant<int, 1>{});
    return v;
}

// four adjacent gains and four adjacent results as one access each
template <typename T> struct Four;
template <> struct Four<float> { typedef __attribute__((ext_vector_type(4))) float type; };
template <> struct Four<__hip_bfloat16> { typedef __attribute__((ext_vector_type(4))) __bf16 type; };

// out = x / sqrt(mean(x^2) + eps) * gain, one workgroup per row, float32 inside.  The row is read
// once with 16-byte loads and kept in registers (d <= 256 * 4 * NV4); NV4 == 0 re-reads it instead.
// A chain of latencies between two launches that move all the bytes, so the gains are requested with the row, in one access per
// four, results leave the same way, and the sum crosses lanes without LDS where it can: with the embedding's 16-byte pieces a
// token of one sequence over 8 layers (17 norms) 964 - 966 -> 939 - 942 us, of four 1181 - 1184 -> 1158 - 1159 (three pairs of runs).
// NS > 0: x first takes the sums of up to NS slices of a projection's K (slices past the last weigh nothing), requested
// with the row.  It saves the launch that would add them, and its round trip over x.
// The sum of squares is written out in fused operations: left to the compiler, which of two squares it rounds first differed
// between these instantiations, and the row's scale in its last bit with them.
template <typename T, int NV4, int NS>
__global__ __launch_bounds__(TPB) void k_rmsnorm(float* __restrict__ x, const T* __restrict__ gain, T* __restrict__ out, int d,
                                                 float eps, int frag, const float* __restrict__ sums, int n_slices) {
    __shared__ float red[TPB / 64];
    const int64_t m = blockIdx.x;
    float* const xr = x + m * d;
    const int nv4 = d >> 2, tid = threadIdx.x;
    typedef typename Four<T>::type T4;
    typedef T4 T4g __attribute__((aligned(sizeof(T))));   // a layer's gains start anywhere an element may
    float4 v[NV4 > 0 ? NV4 : 1];
    T4 gn[NV4 > 0 ? NV4 : 1];
    float ss = 0.f;
    if constexpr (NV4 > 0) {
#pragma unroll
        for (int i = 0; i < NV4; ++i) {
            const int idx = i * TPB + tid;
            if (idx < nv4) gn[i] = reinterpret_cast<const T4g*>(gain)[idx];
            v[i] = idx < nv4 ? reinterpret_cast<const float4*>(xr)[idx] : make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (NS > 0) {
                if (idx < nv4) {
                    float4 p[NS], s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                    for (int k = 0; k < NS; ++k) p[k] = reinterpret_cast<const float4*>(sums + ((int64_t)(k < n_slices ? k : 0) * gridDim.x + m) * d)[idx];
#pragma unroll
                    for (int k = 0; k < NS; ++k)
                        if (k < n_slices) { s.x += p[k].x; s.y += p[k].y; s.z += p[k].z; s.w += p[k].w; }
                    v[i].x += s.x; v[i].y += s.y; v[i].z += s.z; v[i].w += s.w;
                    reinterpret_cast<float4*>(xr)[idx] = v[i];
                }
            }
            ss += fmaf(v[i].y, v[i].y, __fmul_rn(v[i].x, v[i].x)) + fmaf(v[i].z, v[i].z, __fmul_rn(v[i].w, v[i].w));
        }
    } else {
        for (int c = tid; c < d; c += TPB) {
            float t = xr[c];
            if constexpr (NS > 0) {
                float s = 0.f;
                for (int k = 0; k < n_slices; ++k) s += sums[((int64_t)k * gridDim.x + m) * d + c];
                t += s;
                xr[c] = t;   // read again below by the thread that wrote it
            }
            ss = fmaf(t, t, ss);
        }
    }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    ss = (red[0] + red[1]) + (red[2] + red[3]);
    const float sc = 1.0f / sqrtf(ss / (float)d + eps);
    if constexpr (NV4 > 0) {
#pragma unroll
        for (int i = 0; i < NV4; ++i) {
            const int idx = i * TPB + tid;
            if (idx < nv4) {
                const int c = idx * 4;
                const int64_t o = frag ? frag_index((int)m, c, d) : m * d + c;   // 4 | c: one run of 8 either way
                T4 r;
                r[0] = v[i].x * sc * (float)gn[i][0];
                r[1] = v[i].y * sc * (float)gn[i][1];
                r[2] = v[i].z * sc * (float)gn[i][2];
                r[3] = v[i].w * sc * (float)gn[i][3];
                *reinterpret_cast<T4*>(out + o) = r;
            }
        }
    } else {
        for (int c = tid; c < d; c += TPB) st(out, frag ? frag_index((int)m, c, d) : m * d + c, xr[c] * sc * ld(gain, c));
    }
}

}  // namespace

template <typename T>
static void embed_dispatch(const T* embed, const int32_t* tok, const T* in_embeds, const StepTokens& in, float* x, int M, int d, int V, hipStream_t s) {
    // the caller's rows may start anywhere its elements may
    const bool vec = ((reinterpret_cast<uintptr_t>(in_embeds ? in_embeds : embed) | reinterpret_cast<uintptr_t>(x)) & 15) == 0 && d % (16 / (int)sizeof(T)) == 0;
    if (vec) hipLaunchKernelGGL((k_embed<T, true>), dim3(M), dim3(TPB), 0, s, embed, tok, in_embeds, in, x, d, V);
    else hipLaunchKernelGGL((k_embed<T, false>), dim3(M), dim3(TPB), 0, s, embed, tok, in_embeds, in, x, d, V);
}

void launch_embed(const void* embed, int dtype, const int32_t* tok, const void* in_embeds, const StepTokens& in, float* x,
                  int M, int d, int V, hipStream_t s) {
    if (dtype == 1) embed_dispatch((const __hip_bfloat16*)embed, tok, (const __hip_bfloat16*)in_embeds, in, x, M, d, V, s);
    else embed_dispatch((const float*)embed, tok, (const float*)in_embeds, in, x, M, d, V, s);
}

template <typename T, int NS>
static void rmsnorm_dispatch(float* x, const T* gain, T* out, int M, int d, float eps, int frag, Slices add, hipStream_t s) {
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(M), dim3(TPB), 0, s, x, gain, out, d, eps, frag, add.sums, add.n); };
    if ((d & 3) == 0 && d <= 1024) go(k_rmsnorm<T, 1, NS>);
    else if ((d & 3) == 0 && d <= 4096) go(k_rmsnorm<T, 4, NS>);
    else if ((d & 3) == 0 && d <= 8192) go(k_rmsnorm<T, 8, NS>);
    else go(k_rmsnorm<T, 0, NS>);
}

void launch_rmsnorm(float* x, const void* gain, int dtype, void* out, int M, int d, float eps, bool frag, Slices add,
                    hipStream_t s) {
    typedef __hip_bfloat16 bf16;
    if (dtype != 1) rmsnorm_dispatch<float, 0>(x, (const float*)gain, (float*)out, M, d, eps, 0, add, s);
    else if (add.n == 0) rmsnorm_dispatch<bf16, 0>(x, (const bf16*)gain, (bf16*)out, M, d, eps, frag ? 1 : 0, add, s);
    else if (add.n <= 2) rmsnorm_dispatch<bf16, 2>(x, (const bf16*)gain, (bf16*)out, M, d, eps, frag ? 1 : 0, add, s);
    else if (add.n <= 4) rmsnorm_dispatch<bf16, 4>(x, (const bf16*)gain, (bf16*)out, M, d, eps, frag ? 1 : 0, add, s);
    else rmsnorm_dispatch<bf16, 8>(x, (const bf16*)gain, (bf16*)out, M, d, eps, frag ? 1 : 0, add, s);
}

}  // namespace mulo
