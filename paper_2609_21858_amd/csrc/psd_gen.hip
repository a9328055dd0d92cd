// psd_gen.hip -- the multi-block generation loop on the device (gfx950).
//
// Speculative generation repeats one block per step (Alg. "Batched-target
// direct-top-k MPFR speculative sampling"; App. F's formal multi-draft algorithm):
// the models give the block's target and draft rows, the race and the walk emit
// tau tokens per sequence, and the emitted tokens extend every sequence's text, its
// next start position and its context window.  This file holds the device parts
// that the race does not: the commit of emitted tokens (advance_kernel) and a
// position-indexed toy language model standing in for the models (toy_rows_kernel),
// whose target row depends only on (sequence, absolute position) and whose drafter
// k adds its own noise -- so the emitted text must equal plain keyed decoding with
// the target rows, whatever the drafts (drafter invariance, App. C).
//
// Toy rows are exact functions of integer hashes (SplitMix64 per row, Wellons'
// lowbias32 per element) and of fp32 additions and products, each rounded once
// (no fused multiply-add), so any implementation of the same definition
// reproduces them bit for bit:
//   row words   R_T = sm(seed ^ sm(b << 32 | t)),  R_P = sm(R_T ^ 0xD1B54A32D192ED03),
//               R_D = sm(draft_seed ^ sm((k + 1) << 56 ^ b << 32 ^ t))   (sm = SplitMix64)
//   rank        r(v) = (a v + c) mod V,  c = R_P mod V,  a = (R_P >> 32) mod V moved up
//               to the next value coprime to V (a bijection of [0, V))
//   noise       x = lo32(R) + v * 0x9E3779B9 (mod 2^32), h = lowbias32(x);
//               target: 4 uniforms u = (q + 1/2) / 2^16 from the 16-bit halves of
//               h and of lowbias32(x ^ hi32(R_T)), n = (u1 + u2 + u3 + u4 - 2) * sqrt(3);
//               draft: n' = (u1 + u2 - 1) * sqrt(6) from the halves of h
//   rank term   q(r) = fp32(bits(fp32(1 + r)) - 0x3F800000), i.e. 2^23 times the
//               piecewise-linear log2 of 1 + r read off its fp32 bits, and the weight
//               w = fp32(-alpha ln 2 / 2^23) (computed in double), so w q(r) is close
//               to -alpha ln(1 + r): a Zipf-like head
//   logits      z_v = sigma * n + w * q(r(v)),  draft_v = z_v + tau_b * n'
//               (tau_b = tau[0] for b < tau_split, else tau[1]); bf16 rows are the
//               round-to-nearest-even of those fp32 values.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

#include "psd_launch.hpp"

// The toy rows' definition rounds every product and sum once: no contraction into
// fused multiply-adds anywhere in this file (the build passes -ffp-contract=off too).
#pragma clang fp contract(off)

namespace psd {

namespace {

__device__ __forceinline__ uint64_t sm64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

__device__ __forceinline__ uint32_t lowbias32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7FEB352Du;
    x ^= x >> 15;
    x *= 0x846CA68Bu;
    x ^= x >> 16;
    return x;
}

// Sum of the two (q + 1/2) / 2^16 uniforms held in the halves of h (exact in fp32).
__device__ __forceinline__ float two_uniforms(uint32_t h) {
    return ((float)(h & 0xFFFFu) + (float)(h >> 16) + 1.0f) * 0x1p-16f;
}

__device__ __forceinline__ uint16_t bf16_rne(float f) {
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// 8 consecutive logits of a row from element `at` (any alignment: one or two 16-byte
// stores), the row's last ones singly.
typedef uint32_t u32x4_f32 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_b16 __attribute__((ext_vector_type(4), aligned(2)));
template <bool BF16>
__device__ __forceinline__ void store8(void* rows, size_t at, int n, const float (&z)[8]) {
    if constexpr (BF16) {
        uint16_t* p = (uint16_t*)rows + at;
        uint16_t h[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) h[i] = bf16_rne(z[i]);
        if (n >= 8) {
            u32x4_b16 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = (uint32_t)h[2 * i] | ((uint32_t)h[2 * i + 1] << 16);
            *(u32x4_b16*)p = w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i < n) p[i] = h[i];
        }
    } else {
        float* p = (float*)rows + at;
        if (n >= 8) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4_f32 w;
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = __float_as_uint(z[4 * h + i]);
                *(u32x4_f32*)(p + 4 * h) = w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i < n) p[i] = z[i];
        }
    }
}

// gridDim.y workgroups per (sequence b, depth s): the target row at t = start[b] + s and,
// for s < gamma, the K draft rows of that depth, 8 consecutive tokens per thread.
// Bound by integer arithmetic (about 24 issue slots per logit, two 32-bit products
// among them), so the rows are split over enough workgroups to fill the device
// (13.3 M logits at V = 32000, K = 4, gamma = 5, B = 16: 19 us; one workgroup per
// (b, s), a thread per token and a gcd per thread took 54 us).
template <bool BF16>
__global__ __launch_bounds__(256) void toy_rows_kernel(ToyArgs a) {
    const int G1 = a.gamma + 1;
    const int b = blockIdx.x / G1, s = blockIdx.x % G1;
    const uint64_t t = (uint64_t)(a.start_pos[b] + s);
    const uint32_t V = (uint32_t)a.V;
    const uint64_t RT = sm64(a.seed ^ sm64(((uint64_t)b << 32) | (t & 0xFFFFFFFFull)));
    const uint64_t RP = sm64(RT ^ 0xD1B54A32D192ED03ull);
    const uint32_t c = (uint32_t)(RP % V);
    uint32_t am = (uint32_t)((RP >> 32) % V);
    if (am == 0u) am = 1u;
    // up to the first multiplier coprime to V: divisible by none of V's prime factors
    for (;;) {
        bool coprime = true;
        for (int i = 0; i < a.n_primes; ++i) coprime = coprime && am % a.primes[i] != 0u;
        if (coprime) break;
        am = am + 1u == V ? 1u : am + 1u;
    }
    const float tau = b < a.tau_split ? a.tau0 : a.tau1;
    const bool drafts = s < a.gamma && a.draft_logits;
    __shared__ uint32_t rd[32];  // lo32(R_D) of each drafter at this (b, t)
    if ((int)threadIdx.x < a.K)
        rd[threadIdx.x] = (uint32_t)sm64(a.draft_seed ^ sm64(((uint64_t)(threadIdx.x + 1) << 56) ^
                                                             ((uint64_t)b << 32) ^ (t & 0xFFFFFFFFull)));
    __syncthreads();
    const size_t trow = ((size_t)b * G1 + s) * V;
    const uint32_t stride = 8u * blockDim.x * gridDim.y;
    uint32_t v0 = 8u * (blockIdx.y * blockDim.x + threadIdx.x);
    // r(v) stepped along this thread's tokens: r(v + d) = r(v) + a d (mod V)
    uint32_t r0 = (uint32_t)(((uint64_t)am * v0 + c) % V);
    const uint32_t step = (uint32_t)(((uint64_t)am * stride) % V);
    for (; v0 < V; v0 += stride) {
        float z[8];
        uint32_t r = r0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t x = (uint32_t)RT + (v0 + (uint32_t)i) * 0x9E3779B9u;
            const float u4 = two_uniforms(lowbias32(x)) + two_uniforms(lowbias32(x ^ (uint32_t)(RT >> 32)));
            const float n = __fmul_rn(u4 - 2.0f, 1.7320508075688772f);
            const float q = (float)(int32_t)(__float_as_uint((float)(r + 1u)) - 0x3F800000u);
            z[i] = __fadd_rn(__fmul_rn(a.sigma, n), __fmul_rn(a.w, q));
            r += am;
            if (r >= V) r -= V;
        }
        r0 += step;
        if (r0 >= V) r0 -= V;
        const int n = (int)min(V - v0, 8u);
        store8<BF16>(a.target_logits, trow + v0, n, z);
        if (!drafts) continue;
        for (int k = 0; k < a.K; ++k) {
            float d[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float n2 = __fmul_rn(two_uniforms(lowbias32(rd[k] + (v0 + (uint32_t)i) * 0x9E3779B9u)) - 1.0f, 2.449489742783178f);
                d[i] = __fadd_rn(z[i], __fmul_rn(tau, n2));
            }
            store8<BF16>(a.draft_logits, (((size_t)b * a.K + k) * a.gamma + s) * V + v0, n, d);
        }
    }
}

constexpr int kAdvBlock = 1024;

// Commit the emitted tokens of one block (or, with out_len NULL, set up the first
// block from the prompt), then the next block's start positions and windows and the
// number of sequences still short of max_len.  One workgroup, sequences strided.
__global__ __launch_bounds__(kAdvBlock) void advance_kernel(AdvanceArgs a) {
    __shared__ int red[kAdvBlock / 64];
    const int tid = threadIdx.x;
    int active = 0;
    for (int b = tid; b < a.B; b += kAdvBlock) {
        int32_t* text = a.text + (size_t)b * a.text_stride;
        int64_t L = a.out_len ? a.length[b] : (int64_t)a.m;
        L = L < a.m ? a.m : (L > a.max_len ? a.max_len : L);  // keeps every index below in range
        if (a.out_len && L < a.max_len) {
            const int n = min(max(a.out_len[b], 0), a.gamma + 1);
            for (int i = 0; i < n && L < a.max_len; ++i) {
                const int32_t y = a.out_tokens[(size_t)b * (a.gamma + 1) + i];
                if (y < 0) {  // an empty row: the sequence cannot continue
                    for (; L < a.max_len; ++L) text[L] = -1;
                    break;
                }
                text[L++] = y;
            }
        }
        a.length[b] = L;
        const int64_t st = L < a.max_len ? L : a.max_len - 1;
        a.start_pos[b] = st;
        for (int i = 0; i < a.m; ++i) a.prefix[(size_t)b * a.m + i] = text[st - a.m + i];
        active += L < a.max_len;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) active += __shfl_xor(active, o);
    if ((tid & 63) == 0) red[tid >> 6] = active;
    __syncthreads();
    if (tid == 0) {
        int total = 0;
        for (int w = 0; w < kAdvBlock / 64; ++w) total += red[w];
        *a.n_active = total;
    }
}

}  // namespace

hipError_t launch_toy_rows(const ToyArgs& args, bool bf16, hipStream_t stream) {
    const long rows = (long)args.B * (args.gamma + 1);
    if (rows <= 0) return hipSuccess;
    ToyArgs a = args;
    a.n_primes = 0;
    int rest = a.V;
    for (int p = 2; p * p <= rest; ++p) {
        if (rest % p) continue;
        a.primes[a.n_primes++] = (uint32_t)p;
        while (rest % p == 0) rest /= p;
    }
    if (rest > 1) a.primes[a.n_primes++] = (uint32_t)rest;
    // 2048 tokens per workgroup step; enough workgroups for 8 per CU, at most one step each
    const long steps = (a.V + 2047) / 2048, want = (2048 + rows - 1) / rows;
    const dim3 grid((unsigned)rows, (unsigned)std::min(steps, std::max(1L, want)));
    if (bf16)
        hipLaunchKernelGGL(toy_rows_kernel<true>, grid, dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL(toy_rows_kernel<false>, grid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_advance(const AdvanceArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(kAdvBlock), 0, stream, a);
    return hipGetLastError();
}

}  // namespace psd
