// psd_topk.hip -- logit processing before the race: top-k, then top-p (gfx950).
//
// The paper's experiments race the processed distributions (temperature, top-k,
// top-p; Alg. "Batched-target direct-top-k MPFR speculative sampling"): every
// token outside a row's kept set has probability 0.  With at most 256 kept tokens
// per row the race needs no pruning, so this path has two kernels:
//  * topk_select_kernel, one workgroup per row, one pass over the row in HBM that
//    keeps only the maximum of every 128-token group; the top_k-th largest group
//    maximum bounds the row's top_k-th largest logit from below, so only the groups
//    whose maximum reaches it are read again and their logits that reach it are the
//    candidates (wave buffers in LDS: wave prefix sums, no atomics).  Up to 256 of them
//    are ranked by counting, which leaves the k largest sorted (order-preserving keys,
//    ties to the lowest index); more are cut by block-wide bisections over their keys and
//    then their indices, and sorted.  Rows whose ties at the cut overflow the buffers are
//    selected by exact radix passes instead.  The top-p prefix and the log-sum-exp of the
//    kept set at the row's temperature are formed in fp64;
//  * the races over the lists: float32 clocks of every (token, slot), and fp64 ones where
//    the float32 scores do not decide -- distinct
//    drafters race slot k / all K slots, identical drafters draw each context's nu
//    samples from the cumulative clocks and race the targets on slot 0 -- then the
//    walk.  Distinct drafters (drafting, or with the shared target chain):
//    topk_chain_kernel, one workgroup per (sequence, chain) -- a draft path, or the
//    target chain, whose races four waves share while a fifth folds the next key --
//    then topk_walk_kernel (the walk, one wave per sequence, and the status word).
//    Identical drafters or per-path target rows: topk_race_kernel, one workgroup per
//    sequence with one wave per chain, depth by depth (identical drafters group the
//    paths into contexts at every depth).
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include "psd_device.hpp"
#include "psd_launch.hpp"
#include "psd_layout.hpp"

namespace psd {

namespace {

constexpr int kTBlock = 256;
constexpr int kUnroll = 4;        // candidate groups in flight per thread
constexpr int kStreamUnroll = 8;  // 16-byte loads in flight per thread of the streaming pass (4: 130 vs 123 us per
                                  // top-k 50 call at V = 128256, K = 4, B = 64)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes at any element boundary in one load (rows of an odd vocabulary start off
// the 16-byte grid).
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));

// ---------------------------------------------------------------- keys

// Order-preserving keys (larger value, larger key); -0 takes the key of +0, as the two
// compare equal.
__device__ __forceinline__ uint32_t key_f32(uint32_t u) {
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float val_f32(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}
__device__ __forceinline__ float tload(const unsigned char* row, bool bf16, int v) {
    return bf16 ? __uint_as_float((uint32_t)((const uint16_t*)row)[v] << 16) : ((const float*)row)[v];
}

constexpr int kWaves = kTBlock / 64;
constexpr int kWaveCap = 512;  // candidates a wave holds

// ---------------------------------------------------------------- block helpers

constexpr int kMaxGroups = (1 << 19) / kGroupTokens;  // 128-token groups of the largest row
constexpr int kCandGroups = 2 * kMaxTopK;             // groups re-read for candidates

struct SelShared {
    union {
        struct {
            uint32_t key[kWaves][kWaveCap];  // each wave's candidates: order-preserving key,
            int32_t idx[kWaves][kWaveCap];   // token index
        } wb;
        int hist[2048];         // radix passes (the candidates are given up first)
        float gm[kMaxGroups];   // group maxima of the streaming pass
    } u;
    union {
        struct {
            int tok[kMaxTopK];
            float val[kMaxTopK];
        };
        __align__(16) uint64_t comp[kTBlock];  // candidates being ranked
    };
    union {
        struct {
            int stok[kMaxTopK];
            float sval[kMaxTopK];
        };
        int cgl[kCandGroups];  // groups holding candidates (before the kept list is sorted)
    };
    int red[2][kWaves];
    double dred[kWaves];
    double dsel;
    int s4[kWaves];
    int wcount[kWaves], wover[kWaves];
    int n_keep, n_fin;
    uint32_t tsel;  // a key threshold found by one wave
    uint32_t prefix;
    int above;
};

__device__ __forceinline__ int wave_incl(int x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    return x;
}

// Lanes below this one whose bit is set in m.
__device__ __forceinline__ int lanes_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Entries of the wave (Q per lane) passing a test, counted with ballots (scalar
// popcounts: no lane shuffles).
template <int Q, typename F>
__device__ __forceinline__ int wave_count(F&& pass) {
    int c = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) c += __popcll(__ballot(pass(q)));
    return c;
}

// Sum over the workgroup of a wave-uniform count; the two LDS buffers alternate
// (parity `it`), so one barrier per call suffices.
__device__ __forceinline__ int block_sum_waves(SelShared& sm, int wave_total, int& it) {
    int* r = sm.red[it & 1];
    ++it;
    if ((threadIdx.x & 63) == 0) r[threadIdx.x >> 6] = wave_total;
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += r[w];
    return t;
}

// Inclusive prefix sum of one int per thread (thread order); *total gets the sum.
__device__ __forceinline__ int block_incl_sum(SelShared& sm, int x, int& total) {
    const int wave = threadIdx.x >> 6;
    x = wave_incl(x);
    if ((threadIdx.x & 63) == 63) sm.s4[wave] = x;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        if (w < wave) base += sm.s4[w];
        tot += sm.s4[w];
    }
    __syncthreads();
    total = tot;
    return x + base;
}

// Inclusive prefix sum of one double per thread (thread order); *total gets the sum.
__device__ __forceinline__ double block_incl_sum_f64(SelShared& sm, double x, double& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) sm.dred[wave] = x;
    __syncthreads();
    double base = 0.0, tot = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        if (w < wave) base += sm.dred[w];
        tot += sm.dred[w];
    }
    __syncthreads();
    total = tot;
    return x + base;
}

// ---------------------------------------------------------------- one-wave selection

// The need-th largest key class t of Q keys per lane (0: no entry) with the wave's
// ballots alone (no barrier): largest t (bits below kLow clear) with #{key >= t} >= need
// (0 if there are fewer keys).  t lies between the smallest and the largest key, so it
// has their common leading bits and the search starts below them.
template <int Q, int kLow>
__device__ __forceinline__ uint32_t wave_kth_class(const uint32_t (&kk)[Q], int need) {
    uint32_t mx = 0u, mn = 0xFFFFFFFFu;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        mx = max(mx, kk[q]);
        mn = min(mn, kk[q] ? kk[q] : 0xFFFFFFFFu);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
        mn = min(mn, (uint32_t)__shfl_xor((int)mn, o));
    }
    mx = (uint32_t)__builtin_amdgcn_readfirstlane((int)mx);
    mn = (uint32_t)__builtin_amdgcn_readfirstlane((int)mn);
    if (wave_count<Q>([&](int q) { return kk[q] != 0u; }) < need) return 0u;
    if (mx == mn) return mx >> kLow << kLow;
    const int top = 31 - __builtin_clz(mx ^ mn);  // the highest bit they differ in
    uint32_t t = (uint32_t)((uint64_t)mx >> (top + 1) << (top + 1)) >> kLow << kLow;
    for (int bit = top; bit >= kLow; --bit) {
        const uint32_t cand = t | (1u << bit);
        if (wave_count<Q>([&](int q) { return kk[q] >= cand; }) >= need) t = cand;
    }
    return t;
}

// ---------------------------------------------------------------- one-pass selection

// Keys of bf16 logits differ only in their top 16 bits (the low half is 0x0000 or
// 0xFFFF by sign), so searches over them stop at bit 16; one key class is one value.
template <bool BF16>
struct KeyBits {
    static constexpr int kLow = BF16 ? 16 : 0;
};

template <bool BF16>
__device__ __forceinline__ uint32_t elem_bits(const uint32_t (&w)[4], int i) {
    return BF16 ? ((i & 1) ? (w[i >> 1] & 0xFFFF0000u) : (w[i >> 1] << 16)) : w[i];
}

// Group maxima of the row (128-token groups) into sm.u.gm: one wave per 64 x EPT-token
// chunk in turn (wave w takes chunks w, w + 4, ...; eight 16-byte loads per lane in
// flight), the maximum of each lane's tokens, then of the lanes of a group.  Only a
// maximum per token: the pass costs little more than reading the row.
template <bool BF16>
__device__ __forceinline__ void stream_group_max(SelShared& sm, const unsigned char* row, int V) {
    constexpr int EPT = BF16 ? 8 : 4, WCH = 64 * EPT, STEP = kWaves * kStreamUnroll, LPG = kGroupTokens / EPT;
    constexpr size_t ES = BF16 ? 2 : 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int nch = (V + WCH - 1) / WCH, ng = (V + kGroupTokens - 1) / kGroupTokens;
    for (int c0 = w; c0 < nch; c0 += STEP) {
        uint32_t wv[kStreamUnroll][4];
#pragma unroll
        for (int u = 0; u < kStreamUnroll; ++u) {
            const int base = (c0 + u * kWaves) * WCH + lane * EPT;
            if (base + EPT <= V) {
                const u32x4 q = __builtin_nontemporal_load((const u32x4_any*)(row + (size_t)base * ES));
                wv[u][0] = q.x;
                wv[u][1] = q.y;
                wv[u][2] = q.z;
                wv[u][3] = q.w;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) wv[u][i] = BF16 ? 0xFF80FF80u : 0xFF800000u;  // -inf
#pragma unroll
                for (int i = 0; i < EPT; ++i) {
                    const int v = base + i;
                    if (v < V) {
                        if (BF16) {
                            const uint32_t h = ((const uint16_t*)row)[v];
                            wv[u][i >> 1] = (wv[u][i >> 1] & ~(0xFFFFu << (16 * (i & 1)))) | (h << (16 * (i & 1)));
                        } else {
                            wv[u][i] = ((const uint32_t*)row)[v];
                        }
                    }
                }
            }
        }
        float mx[kStreamUnroll];
#pragma unroll
        for (int u = 0; u < kStreamUnroll; ++u) {
            mx[u] = __uint_as_float(elem_bits<BF16>(wv[u], 0));
#pragma unroll
            for (int i = 1; i < EPT; ++i) mx[u] = fmaxf(mx[u], __uint_as_float(elem_bits<BF16>(wv[u], i)));
        }
        row16_max_n<kStreamUnroll>(mx);
#pragma unroll
        for (int u = 0; u < kStreamUnroll; ++u) {
            if (LPG == 32) mx[u] = fmaxf(mx[u], __shfl_xor(mx[u], 16));
            const int g = (c0 + u * kWaves) * (WCH / kGroupTokens) + lane / LPG;
            if (lane % LPG == 0 && g < ng) sm.u.gm[g] = mx[u];
        }
    }
}

// The top_k-th largest 16-bit key class of ng <= 64 Q group maxima, by one wave.  For
// top_k <= 64 the top_k-th largest of the lanes' own maxima is a first bound (as many
// groups reach it); the group maxima that reach it, usually fewer than 128, are
// compacted through LDS (tmp) and searched two per lane.  With Q = 16 the search over all of
// them took 6.4 us beside other workgroups' streaming.
template <int Q>
__device__ __forceinline__ uint32_t group_threshold(const float* gm, int ng, int top_k, uint32_t* tmp) {
    const int lane = threadIdx.x & 63;
    uint32_t kw[Q], mine[1] = {0u};
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int g = lane + 64 * q;
        const float m = g < ng ? gm[g] : -INFINITY;
        kw[q] = m >= -3.40282347e38f ? key_f32(__float_as_uint(m)) : 0u;
        mine[0] = max(mine[0], kw[q]);
    }
    if (top_k <= 64) {
        const uint32_t t0 = wave_kth_class<1, 16>(mine, top_k);
        if (t0 != 0u) {
            int cnt = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const uint64_t m = __ballot(kw[q] >= t0);
                const int pos = cnt + lanes_below(m);
                if (kw[q] >= t0 && pos < 128) tmp[pos] = kw[q];
                cnt += (int)__popcll(m);
            }
            if (cnt <= 128) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                const uint32_t k2[2] = {lane < cnt ? tmp[lane] : 0u, lane + 64 < cnt ? tmp[lane + 64] : 0u};
                return wave_kth_class<2, 16>(k2, top_k);
            }
        }
    }
    return wave_kth_class<Q, 16>(kw, top_k);
}

// The candidates of the row's top-k set, without a per-logit pass over the row: t =
// the top_k-th largest key class among the group maxima (a bisection with ballot
// counts, in one wave when it holds every group maximum, else block-wide), so
// at least top_k logits reach t and every logit of the top-k set (ties at the cut
// included) reaches it too; only groups whose maximum reaches t can hold such a
// logit, and they are read again.  With fewer groups than top_k, every group with a
// finite logit is read again.  Their finite logits that reach t go to the wave
// buffers (ballot and lane prefix), as the per-logit selection would leave them.
// Returns false when the groups or the candidates do not fit (heavy ties at the
// cut); the caller then selects by radix passes.
template <bool BF16>
__device__ __forceinline__ bool select_candidates(SelShared& sm, const unsigned char* row, int V, int top_k) {
    constexpr int EPT = BF16 ? 8 : 4, LPG = kGroupTokens / EPT, GPW = 64 / LPG;  // groups per wave step
    constexpr int QG = kMaxGroups / kTBlock;
    constexpr size_t ES = BF16 ? 2 : 4;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int ng = (V + kGroupTokens - 1) / kGroupTokens;
    stream_group_max<BF16>(sm, row, V);
    __syncthreads();
    uint32_t kg[QG];
    bool fin[QG];
#pragma unroll
    for (int q = 0; q < QG; ++q) {
        const int g = tid + kTBlock * q;
        const float m = g < ng ? sm.u.gm[g] : -INFINITY;
        fin[q] = m >= -3.40282347e38f;  // a finite (or +inf) logit in the group
        kg[q] = fin[q] ? key_f32(__float_as_uint(m)) : 0u;
    }
    int it = 0;
    uint32_t t = 0u;
    // (any t not above the top_k-th largest group maximum will do, so the search stops at
    // 16-bit classes for fp32 rows too)
    if (ng >= top_k && ng <= 1024) {
        // one wave finds t over all the group maxima; the others wait at one barrier
        if (w == 0) {
            uint32_t* tmp = (uint32_t*)sm.tok;  // (free until the candidates are found)
            const uint32_t tw = ng <= 256 ? group_threshold<4>(sm.u.gm, ng, top_k, tmp) : group_threshold<16>(sm.u.gm, ng, top_k, tmp);
            if (lane == 0) sm.tsel = tw;
        }
        __syncthreads();
        t = sm.tsel;
    } else if (ng >= top_k) {
        for (int bit = 31; bit >= 16; --bit) {
            const uint32_t cand = t | (1u << bit);
            if (block_sum_waves(sm, wave_count<QG>([&](int q) { return fin[q] && kg[q] >= cand; }), it) >= top_k)
                t = cand;
        }
    }
    // the groups to read again, compacted (thread order)
    int nc = 0;
#pragma unroll
    for (int q = 0; q < QG; ++q) nc += fin[q] && kg[q] >= t;
    int n_cg;
    int off = block_incl_sum(sm, nc, n_cg) - nc;
    if (n_cg > kCandGroups) {
        if (tid == 0) sm.wover[0] = 1;
        __syncthreads();
        return false;
    }
#pragma unroll
    for (int q = 0; q < QG; ++q)
        if (fin[q] && kg[q] >= t) sm.cgl[off++] = tid + kTBlock * q;
    __syncthreads();  // (the group maxima are dead: the wave buffers reuse their space)
    // wave w reads groups w*GPW .. of every step of kWaves*GPW list entries
    uint32_t* bk = sm.u.wb.key[w];
    int32_t* bi = sm.u.wb.idx[w];
    // a logit reaches t (finite ones, when t is 0) exactly if it is at least t's value
    const float tv = t ? val_f32(t) : -3.40282347e38f;
    int cnt = 0;
    bool over = false;
    for (int e0 = w * GPW; e0 < n_cg; e0 += kWaves * GPW * kUnroll) {
        uint32_t wv[kUnroll][4];
        int base[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int e = e0 + u * kWaves * GPW + lane / LPG;
            base[u] = -1;
#pragma unroll
            for (int i = 0; i < 4; ++i) wv[u][i] = BF16 ? 0xFF80FF80u : 0xFF800000u;  // -inf
            if (e < n_cg && e < e0 + u * kWaves * GPW + GPW) {
                base[u] = sm.cgl[e] * kGroupTokens + (lane % LPG) * EPT;
                if (base[u] + EPT <= V) {
                    const u32x4 q = *(const u32x4_any*)(row + (size_t)base[u] * ES);
                    wv[u][0] = q.x;
                    wv[u][1] = q.y;
                    wv[u][2] = q.z;
                    wv[u][3] = q.w;
                } else {
#pragma unroll
                    for (int i = 0; i < EPT; ++i) {
                        const int v = base[u] + i;
                        if (v < V) {
                            if (BF16) {
                                const uint32_t h = ((const uint16_t*)row)[v];
                                wv[u][i >> 1] = (wv[u][i >> 1] & ~(0xFFFFu << (16 * (i & 1)))) | (h << (16 * (i & 1)));
                            } else {
                                wv[u][i] = ((const uint32_t*)row)[v];
                            }
                        }
                    }
                }
            }
        }
        // this lane's logits that reach t, as bits (few lanes have any), then their places
        uint32_t mask = 0u;
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
#pragma unroll
            for (int i = 0; i < EPT; ++i)
                mask |= (uint32_t)(__uint_as_float(elem_bits<BF16>(wv[u], i)) >= tv) << (EPT * u + i);
        static_assert(EPT * kUnroll <= 32, "one mask bit per loaded logit");
        const uint32_t c = (uint32_t)__popc(mask), incl = wave_incl_sum(c);
        const int tot = (int)__builtin_amdgcn_readlane((int)incl, 63);
        if (cnt + tot > kWaveCap) {  // ties at the cut: give up (radix passes)
            over = true;
            break;
        }
        int pos = cnt + (int)(incl - c);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t mu = (mask >> (EPT * u)) & ((1u << EPT) - 1u);
            if (mu == 0u) continue;
#pragma unroll
            for (int i = 0; i < EPT; ++i)
                if ((mu >> i) & 1u) {
                    bk[pos] = key_f32(elem_bits<BF16>(wv[u], i));
                    bi[pos] = base[u] + i;
                    ++pos;
                }
        }
        cnt += tot;
    }
    if (lane == 0) {
        sm.wcount[w] = cnt;
        sm.wover[w] = over ? 1 : 0;
    }
    __syncthreads();
    bool ok = true;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) ok = ok && !sm.wover[q];
    return ok;
}

// Exact radix selection of the need = min(top_k, finite logits) largest (ties to the
// lowest index) into sm.tok / sm.val, unsorted: three digit passes (11, 11, 10 bits)
// find the need-th largest key, a fourth collects.  Reads the row four times.
// Returns need.
template <bool BF16>
__device__ int radix_select(SelShared& sm, const unsigned char* row, int V, int top_k) {
    const int tid = threadIdx.x;
    const int shifts[3] = {21, 10, 0};
    const int widths[3] = {11, 11, 10};
    if (tid == 0) {
        sm.prefix = 0u;
        sm.above = 0;
        sm.n_fin = 0;
    }
    int need = 0;
    for (int pass = 0; pass < 3; ++pass) {
        const int nb = 1 << widths[pass];
        for (int i = tid; i < nb; i += kTBlock) sm.u.hist[i] = 0;
        __syncthreads();
        const uint32_t pre = sm.prefix;
        const int hi_shift = shifts[pass] + widths[pass];  // bits above this digit must equal the prefix
        int nf = 0;
        for (int v = tid; v < V; v += kTBlock) {
            const float x = tload(row, BF16, v);
            if (x == -INFINITY) continue;
            ++nf;
            const uint32_t k = key_f32(__float_as_uint(x));
            if (hi_shift < 32 && (k >> hi_shift) != (pre >> hi_shift)) continue;
            atomicAdd(&sm.u.hist[(k >> shifts[pass]) & (uint32_t)(nb - 1)], 1);
        }
        if (pass == 0) atomicAdd(&sm.n_fin, nf);
        __syncthreads();
        if (pass == 0) need = min(top_k, sm.n_fin);
        if (need == 0) return 0;
        if (tid == 0) {
            int acc = sm.above, b = nb - 1;
            for (; b > 0; --b) {
                if (acc + sm.u.hist[b] >= need) break;
                acc += sm.u.hist[b];
            }
            sm.above = acc;
            sm.prefix = pre | ((uint32_t)b << shifts[pass]);
        }
        __syncthreads();
    }
    const uint32_t thr = sm.prefix;
    const int n_eq_take = need - sm.above;
    if (tid == 0) sm.n_keep = 0;
    __syncthreads();
    int ties_before = 0;
    for (int c0 = 0; c0 < V; c0 += kTBlock * 8) {
        float x[8];
        int nt = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int v = c0 + tid * 8 + i;
            x[i] = v < V ? tload(row, BF16, v) : -INFINITY;
            nt += x[i] != -INFINITY && key_f32(__float_as_uint(x[i])) == thr;
        }
        int total;
        const int incl = block_incl_sum(sm, nt, total);
        int rank = ties_before + incl - nt;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (x[i] == -INFINITY) continue;
            const uint32_t k = key_f32(__float_as_uint(x[i]));
            bool keep = k > thr;
            if (k == thr) keep = rank++ < n_eq_take;
            if (keep) {
                const int j = atomicAdd(&sm.n_keep, 1);
                if (j < kMaxTopK) {
                    sm.tok[j] = c0 + tid * 8 + i;
                    sm.val[j] = x[i] == 0.0f ? 0.0f : x[i];
                }
            }
        }
        ties_before += total;
    }
    __syncthreads();
    return need;
}

// One row: kept list, its length and the LSE of the kept set.
template <bool BF16>
__global__ __launch_bounds__(kTBlock) void topk_select_kernel(TopkSelectArgs a) {
    __shared__ SelShared sm;
    const int tid = threadIdx.x;
    const bool s1 = (int)blockIdx.x >= a.seg[0].n_rows;
    const TopkSegment& G = s1 ? a.seg[1] : a.seg[0];
    const int r = (int)blockIdx.x - (s1 ? a.seg[0].n_rows : 0);
    const unsigned char* row = (const unsigned char*)G.logits + (size_t)r * a.V * (BF16 ? 2 : 4);
    const int rid = G.row_id_base + (G.group > 0 ? (r / G.group) * G.group_stride + r % G.group : r);
    const int lse_at = G.lse_index_base + (G.group > 0 ? (r / G.group) * G.lse_group_stride + r % G.group : r);

    int it = 0;
    int need;
    bool sorted = false;
    if (!select_candidates<BF16>(sm, row, a.V, a.top_k)) {
        __syncthreads();  // the candidate buffers are reused by the radix passes
        if (tid == 0 && a.radix_rows) atomicAdd(a.radix_rows, 1u);
        need = radix_select<BF16>(sm, row, a.V, a.top_k);
    } else {
        // the union of the wave buffers holds every logit at least the row's top_k-th
        // largest (ties included), or every finite logit when there are fewer
        constexpr int Q = kWaves * kWaveCap / kTBlock;
        constexpr int PW = kWaveCap / kTBlock;  // entries of one wave's buffer per thread
        uint32_t kk[Q];
        int32_t ii[Q];
        int tot = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) tot += sm.wcount[w];
        need = min(a.top_k, tot);
        if (need > 0 && tot <= kTBlock) {
            // one candidate per thread, whose rank among them (key descending, index
            // ascending: one 64-bit comparison each) is its place in the sorted list
            uint64_t* comp = (uint64_t*)sm.comp;
            uint64_t mine = 0u;
            if (tid < tot) {
                const int c0 = sm.wcount[0], c1 = c0 + sm.wcount[1], c2 = c1 + sm.wcount[2];
                const int bw = tid < c0 ? 0 : tid < c1 ? 1 : tid < c2 ? 2 : 3;
                const int p = tid - (bw == 0 ? 0 : bw == 1 ? c0 : bw == 2 ? c1 : c2);
                mine = ((uint64_t)sm.u.wb.key[bw][p] << 32) | (uint32_t)~sm.u.wb.idx[bw][p];
            }
            comp[tid] = mine;  // (0 past the last: below every candidate)
            __syncthreads();
            if (tid < tot) {
                int rk = 0;
                const ulonglong2* c2 = (const ulonglong2*)comp;
#pragma unroll 4
                for (int i = 0; i < (tot + 1) / 2; ++i) {
                    const ulonglong2 o = c2[i];
                    rk += (int)(o.x > mine) + (int)(o.y > mine);
                }
                if (rk < need) {
                    sm.stok[rk] = (int)~(uint32_t)mine;
                    sm.sval[rk] = val_f32((uint32_t)(mine >> 32));
                }
            }
            sorted = true;
            __syncthreads();
        } else {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int w = q / PW, p = tid + kTBlock * (q % PW);
                const bool ok = p < sm.wcount[w];
                kk[q] = ok ? sm.u.wb.key[w][p] : 0u;
                ii[q] = ok ? sm.u.wb.idx[w][p] : 0;
            }
            if (need > 0) {
                // the need-th largest key class: largest t with #{key >= t} >= need
                uint32_t t = 0u;
                for (int bit = 31; bit >= KeyBits<BF16>::kLow; --bit) {
                    const uint32_t cand = t | (1u << bit);
                    if (block_sum_waves(sm, wave_count<Q>([&](int q) { return kk[q] >= cand; }), it) >= need) t = cand;
                }
                // keys of the next class up (key >= t_up) are strictly larger logits
                const uint32_t t_up = t + (1u << KeyBits<BF16>::kLow);
                const int n_gt = block_sum_waves(sm, wave_count<Q>([&](int q) { return kk[q] >= t_up; }), it);
                const int n_ge = block_sum_waves(sm, wave_count<Q>([&](int q) { return kk[q] >= t; }), it);
                const int take = need - n_gt;  // ties at t to keep, lowest indices first
                int xmax = 0x7FFFFFFF;         // keep the ties with index <= xmax
                if (n_ge - n_gt > take) {
                    // the take-th smallest index among the tied entries: largest x with #{index < x} < take
                    int x = 0;
                    for (int bit = 18; bit >= 0; --bit) {
                        const int cand = x | (1 << bit);
                        if (block_sum_waves(sm, wave_count<Q>([&](int q) {
                                                return kk[q] >= t && kk[q] < t_up && ii[q] < cand;
                                            }),
                                            it) < take)
                            x = cand;
                    }
                    xmax = x;
                }
                int kc = 0;
#pragma unroll
                for (int q = 0; q < Q; ++q) kc += kk[q] >= t_up || (kk[q] >= t && ii[q] <= xmax);
                int total;
                int off = block_incl_sum(sm, kc, total) - kc;
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if ((kk[q] >= t_up || (kk[q] >= t && ii[q] <= xmax)) && off < kMaxTopK) {
                        sm.tok[off] = ii[q];
                        sm.val[off] = val_f32(kk[q]);
                        ++off;
                    }
                __syncthreads();
            }
        }
    }
    if (need == 0) {
        if (tid == 0) {
            a.list_len[rid] = ~0u;
            if (G.lse_out) G.lse_out[lse_at] = -INFINITY;
        }
        return;
    }
    const int n = need;  // both branches leave exactly need entries
    // sort by (logit descending, index ascending): each entry's rank by counting
    if (!sorted && tid < n) {
        const float xv = sm.val[tid];
        const int tv = sm.tok[tid];
        int rk = 0;
        for (int j = 0; j < n; ++j) rk += sm.val[j] > xv || (sm.val[j] == xv && sm.tok[j] < tv);
        sm.stok[rk] = tv;
        sm.sval[rk] = xv;
    }
    __syncthreads();
    // top-p on the sorted list: the shortest prefix whose normalised mass at T reaches
    // top_p; then the LSE of the kept set (fp64)
    const double T = (double)G.T;
    // (a logit equal to the largest has term 1, +inf included)
    const double z0 = (double)sm.sval[0] / T;
    const double e = tid >= n ? 0.0 : sm.sval[tid] == sm.sval[0] ? 1.0 : exp((double)sm.sval[tid] / T - z0);
    double tot;
    const double inc = block_incl_sum_f64(sm, e, tot);
    int keep = n;
    if (a.top_p < 1.0f)
        keep = min(n, block_sum_waves(sm, __popcll(__ballot(tid < n && inc / tot < (double)a.top_p)), it) + 1);
    if (tid == keep - 1) sm.dsel = inc;
    __syncthreads();
    if (tid == 0) {
        const float lse = (float)(z0 + log(sm.dsel));
        a.list_len[rid] = ~(uint32_t)keep;
        if (G.lse_out) G.lse_out[lse_at] = lse;
    }
    if (tid < keep)
        a.list[(size_t)rid * a.cap + tid] = ((uint64_t)~(uint32_t)sm.stok[tid] << 32) | __float_as_uint(sm.sval[tid]);
}

// ---------------------------------------------------------------- races over the lists

template <int LAYOUT>
__device__ __forceinline__ double tclock(uint32_t V, uint32_t slot, uint32_t v, uint32_t k0, uint32_t k1) {
    return LAYOUT == 0 ? tree_clock_f64(V, slot, v, k0, k1) : flat_clock_f64(slot, v, k0, k1);
}

__device__ __forceinline__ bool tlex(double s, int v, int j, double s2, int v2, int j2) {
    return s < s2 || (s == s2 && (v < v2 || (v == v2 && j < j2)));
}

// Lexicographic minimum of (s, v, j) over the wave, with its entry c; every lane
// returns the same result (a strict total order on distinct (v, j)).
__device__ __forceinline__ void wave_lexmin(double& s, int& v, int& j, int& c) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double os = __shfl_xor(s, o);
        const int ov = __shfl_xor(v, o), oj = __shfl_xor(j, o), oc = __shfl_xor(c, o);
        if (tlex(os, ov, oj, s, v, j)) {
            s = os;
            v = ov;
            j = oj;
            c = oc;
        }
    }
}

struct RaceShared {
    int path[32 * 33];    // drafts of each path ([path][depth])
    int chain[33];        // shared target chain
    int pchain[32 * 33];  // per-path target chains
    double ts[8];         // partial minima of a shared-chain target race, one per target wave
    int tv[8], tj[8];
    int pre[16];          // the sequence's context window before the block (m <= 16)
    uint32_t tp[2][2];    // the shared chain's next key without its newest token (by depth parity)
    float fin_s[8][64];   // per wave: arrivals that can be among a context's samples
    int fin_c[8][64];
    float ts1[8], ts2[8];  // float32 minima of a shared-chain target race, one per target wave
    int tvj[8];
    int tclear;            // whether they decide it
};

// Context key of the token at absolute position t whose previous tokens are the last
// m of prefix (m tokens, copied to LDS in pre) || path[0 .. d), folded up to window
// position n (n = m: the whole key; n = m - 1: all but the newest token); every lane
// of the wave computes it.
__device__ __forceinline__ void list_key(const TopkRaceArgs& a, const int* pre, int64_t t, const int* path, int d,
                                         uint32_t& k0, uint32_t& k1, int n) {
    k0 = (uint32_t)a.key;
    k1 = (uint32_t)(a.key >> 32);
    fold(k0, k1, (uint32_t)(uint64_t)t, (uint32_t)((uint64_t)t >> 32), 0u);
    for (int i = 0; i < n; ++i) {
        const int g = d + i;  // index in prefix || path
        const int w = g < a.m ? pre[g] : path[g - a.m];
        fold(k0, k1, (uint32_t)w, (uint32_t)i, 1u);
    }
}

template <int LAYOUT>
__device__ __forceinline__ float tclock32(uint32_t V, uint32_t slot, uint32_t v, uint32_t k0, uint32_t k1) {
    return LAYOUT == 0 ? tree_clock_f32(V, slot, v, k0, k1) : flat_clock_f32(slot, v, k0, k1);
}

// Races are decided by float32 scores where those are certain: the fp32 clocks are within
// 1e-6 relative of the exact ones (-ln U within 1.7e-7, over all its inputs) and scores
// use (l - l_max) / T, so a score errs by about 1e-5 and entries further apart than
// kTMargin are in their exact order.  Closer ones are decided by the exact fp64 race
// (about one race in a thousand).  An fp64 tree clock costs five logarithms and four
// divisions in fp64: a depth of the shared target chain took 4.2 us with it.
constexpr float kTMargin = 1e-3f;

// The smallest score of a set of (token, slot) entries, its entry (token * 32 + slot) and
// the second-smallest score.
struct Best2 {
    float s1, s2;
    int vj;
};
__device__ __forceinline__ void best2_add(Best2& b, float s, int vj) {
    if (s < b.s1) {
        b.s2 = b.s1;
        b.s1 = s;
        b.vj = vj;
    } else {
        b.s2 = fminf(b.s2, s);
    }
}
__device__ __forceinline__ void best2_merge(Best2& b, float s1, float s2, int vj) {
    b.s2 = fminf(fminf(b.s2, s2), fmaxf(b.s1, s1));
    if (s1 < b.s1) {
        b.s1 = s1;
        b.vj = vj;
    }
}
__device__ __forceinline__ void best2_wave(Best2& b) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1)
        best2_merge(b, __shfl_xor(b.s1, o), __shfl_xor(b.s2, o), __shfl_xor(b.vj, o));
}
// Whether the smallest score is certain (that of an empty set is).  (No inf - inf: this file
// is compiled with no NaNs.)
__device__ __forceinline__ bool best2_clear(const Best2& b) { return b.s1 == INFINITY || b.s2 > b.s1 + kTMargin; }

// A kept list's length, and the token and logit of an entry (psd_launch.hpp, TopkLayout).
__device__ __forceinline__ int list_length(const TopkRaceArgs& a, int rid) { return (int)~a.list_len[rid]; }
__device__ __forceinline__ int entry_token(uint64_t e) { return (int)~(uint32_t)(e >> 32); }
__device__ __forceinline__ float entry_logit(uint64_t e) { return __uint_as_float((uint32_t)e); }

// The race of one row's list over slots [slot0, slot0 + nslots) -- argmin of
// ln E_j[v] - l_v / T (exact, fp64) -- over the (token, slot) entries of 64-entry units
// part, part + nparts, ... by one wave.  Returns the wave's winning token (-1 when it
// has none) and, when asked, its score and slot.
template <int LAYOUT>
__device__ int wave_race(const TopkRaceArgs& a, int rid, int slot0, int nslots, float T, uint32_t k0, uint32_t k1,
                         int part = 0, int nparts = 1, double* out_s = nullptr, int* out_j = nullptr) {
    const int lane = threadIdx.x & 63;
    const int n = list_length(a, rid);
    const uint64_t* list = a.list + (size_t)rid * a.cap;
    double bs = INFINITY;
    int bv = 0x7FFFFFFF, bj = 0x7FFFFFFF, bc = -1;
    for (int e = part * 64 + lane; e < n * nslots; e += 64 * nparts) {
        const int c = e / nslots, j = slot0 + e % nslots;
        const uint64_t le = list[c];
        const int v = entry_token(le);
        const double s = log(tclock<LAYOUT>((uint32_t)a.V, (uint32_t)j, (uint32_t)v, k0, k1)) - (double)entry_logit(le) / (double)T;
        if (tlex(s, v, j, bs, bv, bj)) {
            bs = s;
            bv = v;
            bj = j;
            bc = c;
        }
    }
    wave_lexmin(bs, bv, bj, bc);
    if (out_s) {
        *out_s = bs;
        *out_j = bj;
    }
    return bs < INFINITY ? bv : -1;
}

// A lane's first (token, slot) entry of a list race, loaded ahead: the list's length
// and the token and logit of the lane's entry (its index clamped into the row's list,
// so the loads never wait for the length and never leave the list), and the list's
// largest logit.  Length and entry stay as stored until they are used: undoing the
// complement where they are loaded would wait for the loads there.
struct ListHead {
    uint32_t len;
    uint64_t e;
    float xmax;
};

__device__ __forceinline__ ListHead list_head(const TopkRaceArgs& a, int rid, int nslots, int part) {
    const int c = min((part * 64 + (int)(threadIdx.x & 63)) / nslots, a.cap - 1);
    const uint64_t* list = a.list + (size_t)rid * a.cap;
    return ListHead{a.list_len[rid], list[c], entry_logit(list[0])};
}

// The float32 scores of the row's (token, slot) entries of 64-entry units part, part +
// nparts, ..., by one wave; the lane's first entry is taken from h (loaded while the
// previous race of the chain ran), xmax is the list's largest logit.
template <int LAYOUT>
__device__ Best2 wave_race32(const TopkRaceArgs& a, const ListHead& h, int rid, int slot0, int nslots, float T,
                             uint32_t k0, uint32_t k1, int part, int nparts) {
    const int lane = threadIdx.x & 63;
    const int n = (int)~h.len;
    const uint64_t* list = a.list + (size_t)rid * a.cap;
    const float invT = 1.0f / T;
    // (token, slot) packed as token * 32 + slot (tokens < 2^19, slots < 32)
    // (a +inf logit, or a temperature whose reciprocal is not finite, has no float32 score
    // here: never certain, so the exact race decides)
    if (n > 0 && !(h.xmax < INFINITY && invT < INFINITY)) return Best2{0.f, 0.f, -1};
    Best2 b{INFINITY, INFINITY, -1};
    auto add = [&](int e, uint64_t le) {
        const int v = entry_token(le), j = slot0 + e % nslots;
        best2_add(b, ln_f32(tclock32<LAYOUT>((uint32_t)a.V, (uint32_t)j, (uint32_t)v, k0, k1)) -
                         (entry_logit(le) - h.xmax) * invT,
                  (v << 5) | j);
    };
    // (the first entry apart: a wait for a loaded one would also wait for the next race's
    // list, which is in flight)
    int e = part * 64 + lane;
    if (e < n * nslots) add(e, h.e);
    for (e += 64 * nparts; e < n * nslots; e += 64 * nparts) add(e, list[e / nslots]);
    best2_wave(b);
    return b;
}

// A whole race by one wave: the winning token, -1 when the list is empty.
template <int LAYOUT>
__device__ int wave_race_one(const TopkRaceArgs& a, const ListHead& h, int rid, int slot0, int nslots, float T,
                             uint32_t k0, uint32_t k1) {
    const Best2 b = wave_race32<LAYOUT>(a, h, rid, slot0, nslots, T, k0, k1, 0, 1);
    if (best2_clear(b)) return b.vj >= 0 ? b.vj >> 5 : -1;
    return wave_race<LAYOUT>(a, rid, slot0, nslots, T, k0, k1);
}

// The nu MPFR samples of one context from its row's list, by one wave, when float32
// scores decide them: theta = the nu-th smallest first-arrival score bounds the nu-th
// smallest of all, so an entry draws arrivals only while they reach theta; the nu + 1
// smallest are taken out one by one and have to be kTMargin apart.  fin: the wave's LDS
// scratch of 64 scores and entries.  Returns false when they are not (or more than 64
// arrivals reach theta).
constexpr int kTFin = 64;
// h: the list, loaded ahead.
struct ListAll {
    uint32_t len;
    uint64_t e[kMaxTopK / 64];
    float xmax;
};
__device__ __forceinline__ ListAll list_all(const TopkRaceArgs& a, int rid) {
    ListAll h;
    h.len = a.list_len[rid];
    const uint64_t* list = a.list + (size_t)rid * a.cap;
    const int lane = (int)(threadIdx.x & 63);
#pragma unroll
    for (int q = 0; q < kMaxTopK / 64; ++q)
        h.e[q] = 64 * q < a.cap ? list[min(lane + 64 * q, a.cap - 1)] : 0u;  // (inside the row's list)
    h.xmax = entry_logit(list[0]);
    return h;
}

__device__ __forceinline__ float wave_min_f32(float x) {
    x = fminf(x, dpp_row<0xB1>(x));
    x = fminf(x, dpp_row<0x4E>(x));
    x = fminf(x, dpp_row<0x141>(x));
    x = fminf(x, dpp_row<0x140>(x));
    x = fminf(x, __shfl_xor(x, 16));
    return fminf(x, __shfl_xor(x, 32));
}

template <int LAYOUT>
__device__ bool wave_mpfr32(const TopkRaceArgs& a, RaceShared& sm, int w, const ListAll& h, uint32_t members, int s,
                            float T, uint32_t k0, uint32_t k1) {
    constexpr int Q = kMaxTopK / 64;
    const int lane = threadIdx.x & 63;
    const int n = (int)~h.len;
    const int nu = __popc(members);
    if (n == 0) {
        if (lane < nu) {
            uint32_t mm = members;
            for (int r = 0; r < lane; ++r) mm &= mm - 1u;
            sm.path[(__ffs((int)mm) - 1) * 33 + s] = -1;
        }
        return true;
    }
    const float invT = 1.0f / T, xmax = h.xmax;
    if (!(xmax < INFINITY && invT < INFINITY)) return false;
    float G[Q], xs[Q], sc[Q];
    int tok[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int c = lane + 64 * q;
        tok[q] = -1;
        xs[q] = G[q] = 0.f;
        sc[q] = INFINITY;
        if (c < n) {
            tok[q] = entry_token(h.e[q]);
            xs[q] = (entry_logit(h.e[q]) - xmax) * invT;
            G[q] = tclock32<LAYOUT>((uint32_t)a.V, 0u, (uint32_t)tok[q], k0, k1);
            sc[q] = ln_f32(G[q]) - xs[q];
        }
    }
    // theta: nu smallest first arrivals, taken out one by one (the register copies)
    float theta = INFINITY;
    if (n >= nu) {
        float t[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) t[q] = sc[q];
        for (int r = 0; r < nu; ++r) {
            static_assert(Q == 4, "four entries per lane");
            const float m = wave_min_f32(fminf(fminf(t[0], t[1]), fminf(t[2], t[3])));
            theta = m;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (t[q] == m) t[q] = INFINITY;  // (equal scores go together: a looser theta)
        }
        theta += 2.f * kTMargin;
    }
    // every arrival up to theta
    int cnt = 0;
    float* fs = sm.fin_s[w];
    int* fc = sm.fin_c[w];
    for (int j = 0; j < nu; ++j) {
        bool more = false;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (64 * q >= n) break;  // (uniform)
            const bool in = sc[q] <= theta && sc[q] < INFINITY;
            const uint64_t m = __ballot(in);
            const int pos = cnt + lanes_below(m);
            if (in && pos < kTFin) {
                fs[pos] = sc[q];
                fc[pos] = tok[q];
            }
            cnt += (int)__popcll(m);
            if (m != 0u && j + 1 < nu) {
                if (in) {
                    G[q] += tclock32<LAYOUT>((uint32_t)a.V, (uint32_t)(j + 1), (uint32_t)tok[q], k0, k1);
                    sc[q] = ln_f32(G[q]) - xs[q];
                } else {
                    sc[q] = INFINITY;
                }
                more = true;
            } else {
                sc[q] = INFINITY;
            }
        }
        if (!more) break;
    }
    if (cnt > kTFin || cnt < nu) return false;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    // rank by counting (one arrival per lane)
    const float mine = lane < cnt ? fs[lane] : INFINITY;
    const int mt = lane < cnt ? fc[lane] : -1;
    int rk = 0;
    bool near = false;
    for (int i = 0; i < cnt; ++i) {
        const float o = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), i));
        rk += o < mine || (o == mine && i < lane);
        near = near || (i != lane && fabsf(o - mine) <= kTMargin);
    }
    if (__ballot(lane < cnt && rk < nu && near) != 0u) return false;
    if (lane < cnt && rk < nu) {
        uint32_t mm = members;
        for (int r = 0; r < rk; ++r) mm &= mm - 1u;
        sm.path[(__ffs((int)mm) - 1) * 33 + s] = mt;
    }
    return true;
}

// The nu MPFR samples of one context from its row's list, by one wave: the nu
// smallest of ln G_{v,j} - l_v / T over (v, j < nu), G_{v,j} = E_0[v] + ... + E_j[v];
// the r-th goes to the r-th path of `members` (ascending) at depth s.
template <int LAYOUT>
__device__ void wave_mpfr(const TopkRaceArgs& a, RaceShared& sm, int rid, uint32_t members, int s, float T,
                          uint32_t k0, uint32_t k1) {
    constexpr int Q = kMaxTopK / 64;
    const int lane = threadIdx.x & 63;
    const int n = list_length(a, rid);
    const int nu = __popc(members);
    const uint64_t* list = a.list + (size_t)rid * a.cap;
    double Gs[Q], sc[Q], lT[Q];
    int tok[Q], jj[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int c = lane + 64 * q;
        jj[q] = 0;
        if (c < n) {
            const uint64_t e = list[c];
            tok[q] = entry_token(e);
            lT[q] = (double)entry_logit(e) / (double)T;
            Gs[q] = tclock<LAYOUT>((uint32_t)a.V, 0u, (uint32_t)tok[q], k0, k1);
            sc[q] = log(Gs[q]) - lT[q];
        } else {
            tok[q] = 0x7FFFFFFF;
            lT[q] = 0.0;
            Gs[q] = 0.0;
            sc[q] = INFINITY;
        }
    }
    uint32_t mm = members;
    for (int r = 0; r < nu; ++r) {
        double bs = INFINITY;
        int bv = 0x7FFFFFFF, bj = 0x7FFFFFFF, bc = -1;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (tlex(sc[q], tok[q], jj[q], bs, bv, bj)) {
                bs = sc[q];
                bv = tok[q];
                bj = jj[q];
                bc = lane + 64 * q;
            }
        wave_lexmin(bs, bv, bj, bc);
        const int member = __ffs((int)mm) - 1;
        mm &= mm - 1u;
        if (lane == 0) sm.path[member * 33 + s] = bs < INFINITY ? bv : -1;
        if (bs < INFINITY && lane == (bc & 63)) {
            // the winner's next arrival (one clock, then back into its register slot)
            const int qb = bc >> 6;
            int j = 0;
            double g = 0.0, l = 0.0;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (q == qb) {
                    j = jj[q] + 1;
                    g = Gs[q];
                    l = lT[q];
                }
            double ns = INFINITY;
            if (j < nu) {
                g += tclock<LAYOUT>((uint32_t)a.V, (uint32_t)j, (uint32_t)bv, k0, k1);
                ns = log(g) - l;
            }
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (q == qb) {
                    Gs[q] = g;
                    sc[q] = ns;
                    jj[q] = j;
                }
        }
    }
}

// The call's error bits to the sticky word and the caller's status word, and its epoch
// where its words are tagged (one thread).
// The list kernels set none themselves, so the first workgroup of the call's last
// launch does this at its start (a launch of its own took 4.4 us and a gap).
__device__ __forceinline__ void hand_over_status(const TopkRaceArgs& a) {
    const uint32_t bits = __hip_atomic_exchange(a.ctrl + kCtrlCallErrors, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (bits) __hip_atomic_fetch_or(a.ctrl + kCtrlErrors, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (a.status) *a.status = bits | (a.status_in ? *a.status_in : 0u);
    if (a.advance_epoch) a.ctrl[kCtrlEpoch] = epoch_after(a.ctrl[kCtrlEpoch]);
}

template <int LAYOUT>
__global__ __launch_bounds__(512) void topk_race_kernel(TopkRaceArgs a) {
    __shared__ RaceShared sm;
    if (blockIdx.x == 0 && threadIdx.x == 0) hand_over_status(a);
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, nw = (int)(blockDim.x >> 6);
    const int K = a.K, G = a.gamma;
    const int D = a.B * K * G;
    const int64_t t0 = a.start_pos[b];
    // drafts known before the call (depths < s_begin, or all of them as input)
    for (int e = tid; e < K * G; e += blockDim.x)
        sm.path[(e / G) * 33 + e % G] = a.draft_tokens[((size_t)b * K + e / G) * G + e % G];
    for (int e = tid; e < a.m; e += blockDim.x) sm.pre[e] = a.prefix[(size_t)b * a.m + e];
    __syncthreads();
    const bool per = a.target_rows > 1;
    const int tslots = a.mpfr ? 1 : K;
    // waves [dw, nw) share each shared-chain target race; the others race the drafts
    const int twv = a.target_rows == 1 ? a.target_waves : 0, dw = nw - twv;
    const int d_end = a.s_begin + a.s_count;
    const int s_lo = a.target_rows > 0 ? 0 : a.s_begin;
    const int s_hi = a.target_rows > 0 ? G : d_end - 1;
    uint32_t k0, k1;
    ListHead thead = {};  // a target wave's part of the next list, loaded while a depth runs
    if (a.target_rows == 1 && w >= dw) thead = list_head(a, D + b * (G + 1) + s_lo, tslots, w - dw);
    for (int s = s_lo; s <= s_hi; ++s) {
        if (s >= a.s_begin && s < d_end && w < dw) {
            for (int k = w; k < K; k += dw) {
                if (!a.mpfr) {
                    list_key(a, sm.pre, t0 + s, &sm.path[k * 33], s, k0, k1, a.m);
                    const int rid = (b * K + k) * G + s;
                    const int y = wave_race_one<LAYOUT>(a, list_head(a, rid, 1, 0), rid, k, 1, a.T_draft, k0, k1);
                    if (lane == 0) sm.path[k * 33 + s] = y;
                } else {
                    // the context of path k: the paths with its drafts at depths < s; its
                    // lowest path draws the context's samples (wave-uniform)
                    uint32_t members = 0u;
                    bool rep = true;
                    for (int q = 0; q < K; ++q) {
                        bool same = true;
                        for (int d = 0; d < s && same; ++d) same = sm.path[q * 33 + d] == sm.path[k * 33 + d];
                        if (same) {
                            members |= 1u << q;
                            if (q < k) rep = false;
                        }
                    }
                    if (!rep) continue;
                    const ListAll h = list_all(a, (b * K + k) * G + s);  // (in flight while the key is folded)
                    list_key(a, sm.pre, t0 + s, &sm.path[k * 33], s, k0, k1, a.m);
                    if (!wave_mpfr32<LAYOUT>(a, sm, w, h, members, s, a.T_draft, k0, k1))
                        wave_mpfr<LAYOUT>(a, sm, (b * K + k) * G + s, members, s, a.T_draft, k0, k1);
                }
            }
        }
        if (a.target_rows == 1 && w >= dw) {
            const int ti = w - dw;
            if (s > 0 && a.m > 0) {
                // the rest of the key was folded during the previous depth; its newest
                // token is the previous depth's target
                k0 = sm.tp[s & 1][0];
                k1 = sm.tp[s & 1][1];
                fold(k0, k1, (uint32_t)sm.chain[s - 1], (uint32_t)(a.m - 1), 1u);
            } else {
                list_key(a, sm.pre, t0 + s, sm.chain, s, k0, k1, a.m);
            }
            const int rid = D + b * (G + 1) + s;
            const ListHead hs = thead;
            if (s < G) thead = list_head(a, rid + 1, tslots, ti);
            const Best2 p = wave_race32<LAYOUT>(a, hs, rid, 0, tslots, a.T_target, k0, k1, ti, twv);
            if (lane == 0) {
                sm.ts1[ti] = p.s1;
                sm.ts2[ti] = p.s2;
                sm.tvj[ti] = p.vj;
            }
        }
        if (a.target_rows == 1 && w == 0 && a.m > 0 && s < G) {
            // the next depth's shared-chain key up to its newest token (this depth's
            // target, not known yet): folded here by a draft wave, which finishes its
            // races before the target waves do
            uint32_t p0, p1;
            list_key(a, sm.pre, t0 + s + 1, sm.chain, s + 1, p0, p1, a.m - 1);
            if (lane == 0) {  // (the other parity: this depth's key was read from it)
                sm.tp[(s + 1) & 1][0] = p0;
                sm.tp[(s + 1) & 1][1] = p1;
            }
        }
        if (per)
            for (int k = w; k < K; k += nw) {
                list_key(a, sm.pre, t0 + s, &sm.path[k * 33], s, k0, k1, a.m);
                const int rid = D + (b * K + k) * (G + 1) + s;
                const int y = wave_race_one<LAYOUT>(a, list_head(a, rid, tslots, 0), rid, 0, tslots, a.T_target, k0, k1);
                if (lane == 0) sm.pchain[k * 33 + s] = y;
            }
        __syncthreads();
        if (twv > 0) {
            // the shared-chain target of depth s: the minimum of the waves' parts
            if (tid == 0) {
                Best2 p{sm.ts1[0], sm.ts2[0], sm.tvj[0]};
                for (int i = 1; i < twv; ++i) best2_merge(p, sm.ts1[i], sm.ts2[i], sm.tvj[i]);
                sm.chain[s] = p.vj >= 0 ? p.vj >> 5 : -1;
                sm.tclear = best2_clear(p);
            }
            __syncthreads();
            if (!sm.tclear) {  // (uniform)
                if (w >= dw) {
                    double ps;
                    int pj;
                    const int pv = wave_race<LAYOUT>(a, D + b * (G + 1) + s, 0, tslots, a.T_target, k0, k1, w - dw, twv, &ps, &pj);
                    if (lane == 0) {
                        sm.ts[w - dw] = ps;
                        sm.tv[w - dw] = pv;
                        sm.tj[w - dw] = pj;
                    }
                }
                __syncthreads();
                if (tid == 0) {
                    double bs = sm.ts[0];
                    int bv = sm.tv[0], bj = sm.tj[0];
                    for (int i = 1; i < twv; ++i)
                        if (tlex(sm.ts[i], sm.tv[i], sm.tj[i], bs, bv, bj)) {
                            bs = sm.ts[i];
                            bv = sm.tv[i];
                            bj = sm.tj[i];
                        }
                    sm.chain[s] = bs < INFINITY ? bv : -1;
                }
                __syncthreads();
            }
        }
    }
    if (a.s_count > 0)
        for (int e = tid; e < K * a.s_count; e += blockDim.x) {
            const int k = e / a.s_count, s = a.s_begin + e % a.s_count;
            a.draft_tokens[((size_t)b * K + k) * G + s] = sm.path[k * 33 + s];
        }
    if (a.target_rows == 0 || tid != 0) return;
    auto target = [&](int k, int s) { return per ? sm.pchain[k * 33 + s] : sm.chain[s]; };
    if (a.target_tokens)
        for (int k = 0; k < (per ? K : 1); ++k)
            for (int s = 0; s <= G; ++s) a.target_tokens[((size_t)b * (per ? K : 1) + k) * (G + 1) + s] = target(k, s);
    // ---- the walk (as in the fused kernel)
    uint32_t act = K >= 32 ? 0xFFFFFFFFu : ((1u << K) - 1u);
    int tau = 0;
    bool done = false;
    for (int s = 0; s < G && !done; ++s) {
        const int y = target(__ffs((int)act) - 1, s);
        a.out_tokens[(size_t)b * (G + 1) + s] = y;
        tau = s + 1;
        if (y < 0) {
            done = true;
            break;
        }
        uint32_t na = 0u;
        for (int k = 0; k < K; ++k)
            if (((act >> k) & 1u) && sm.path[k * 33 + s] == y) na |= 1u << k;
        if (!na) {
            done = true;
            break;
        }
        act = na;
    }
    if (!done) {
        a.out_tokens[(size_t)b * (G + 1) + G] = target(__ffs((int)act) - 1, G);
        tau = G + 1;
    }
    for (int s = tau; s <= G; ++s) a.out_tokens[(size_t)b * (G + 1) + s] = -1;
    a.out_len[b] = tau;
}

// Distinct drafters, drafting only or with the shared target chain: one workgroup per
// (sequence, chain) -- a draft path (one wave) or the target chain (four waves sharing
// each race, a fifth folding the next key) -- so a sequence's chains run on different
// CUs rather than sharing one CU's SIMDs.  The chains of a sequence are independent
// (the target chain is keyed by its own prefix), so no workgroup waits for another;
// the walk runs in the next launch.
struct ChainShared {
    int path[33];          // this workgroup's chain: drafts of one path, or the targets
    int pre[16];           // the sequence's context window before the block (m <= 16)
    float ts1[4], ts2[4];  // float32 minima of a target race, one per wave
    int tvj[4];
    int tclear;            // whether they decide it
    double ts[4];          // exact partial minima of a target race, one per wave
    int tv[4], tj[4];
    uint32_t tp[2][2];     // the chain's next key without its newest token (by depth parity)
};

constexpr int kChainWaves = 4;  // waves sharing each target race; one more folds the next key

template <int LAYOUT>
__global__ __launch_bounds__(64 * (kChainWaves + 1)) void topk_chain_kernel(TopkRaceArgs a) {
    __shared__ ChainShared sm;
    if (a.target_rows == 0 && blockIdx.x == 0 && threadIdx.x == 0) hand_over_status(a);  // (no walk follows)
    const int K = a.K, G = a.gamma;
    const int nd = a.s_count > 0 ? K : 0, R = nd + (a.target_rows == 1 ? 1 : 0);
    // chain-major, the target chains (the longest) first: each kind of chain spreads over
    // the XCDs, which consecutive workgroups go to in turn
    const int b = (int)blockIdx.x % a.B, r = R - 1 - (int)blockIdx.x / a.B;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t t0 = a.start_pos[b];
    const int d_end = a.s_begin + a.s_count;
    for (int e = tid; e < a.m; e += blockDim.x) sm.pre[e] = a.prefix[(size_t)b * a.m + e];
    if (r < nd)
        for (int e = tid; e < a.s_begin; e += blockDim.x) sm.path[e] = a.draft_tokens[((size_t)b * K + r) * G + e];
    __syncthreads();
    uint32_t k0, k1;
    if (r < nd) {
        // draft path k: its races in depth order, by one wave (every lane keeps the
        // same copy of the path, so no lane reads another lane's LDS write)
        if (w != 0) return;
        const int k = r;
        ListHead h = list_head(a, (b * K + k) * G + a.s_begin, 1, 0);
        for (int s = a.s_begin; s < d_end; ++s) {
            list_key(a, sm.pre, t0 + s, sm.path, s, k0, k1, a.m);
            const ListHead hs = h;
            if (s + 1 < d_end) h = list_head(a, (b * K + k) * G + s + 1, 1, 0);  // the next depth's, in flight
            sm.path[s] = wave_race_one<LAYOUT>(a, hs, (b * K + k) * G + s, k, 1, a.T_draft, k0, k1);
        }
        for (int s = a.s_begin + lane; s < d_end; s += 64) a.draft_tokens[((size_t)b * K + k) * G + s] = sm.path[s];
        return;
    }
    // the shared target chain: each race's (token, slot) entries shared by the waves
    const int tslots = K;
    const int trow = a.B * K * G + b * (G + 1);
    ListHead h = list_head(a, trow, tslots, w);
    for (int s = 0; s <= G; ++s) {
        if (w == kChainWaves) {
            // the next depth's key up to its newest token (this race's winner), folded
            // while the other waves race
            if (a.m > 0 && s < G) {
                uint32_t p0, p1;
                list_key(a, sm.pre, t0 + s + 1, sm.path, s + 1, p0, p1, a.m - 1);
                if (lane == 0) {  // (the other parity: this depth's key was read from it)
                    sm.tp[(s + 1) & 1][0] = p0;
                    sm.tp[(s + 1) & 1][1] = p1;
                }
            }
            __syncthreads();
            __syncthreads();
            if (!sm.tclear) {
                __syncthreads();
                __syncthreads();
            }
            continue;
        }
        if (s > 0 && a.m > 0) {
            k0 = sm.tp[s & 1][0];
            k1 = sm.tp[s & 1][1];
            fold(k0, k1, (uint32_t)sm.path[s - 1], (uint32_t)(a.m - 1), 1u);
        } else {
            list_key(a, sm.pre, t0 + s, sm.path, s, k0, k1, a.m);
        }
        const ListHead hs = h;
        if (s < G) h = list_head(a, trow + s + 1, tslots, w);  // the next depth's, in flight
        const Best2 p = wave_race32<LAYOUT>(a, hs, trow + s, 0, tslots, a.T_target, k0, k1, w, kChainWaves);
        if (lane == 0) {
            sm.ts1[w] = p.s1;
            sm.ts2[w] = p.s2;
            sm.tvj[w] = p.vj;
        }
        __syncthreads();
        if (tid == 0) {
            Best2 q{sm.ts1[0], sm.ts2[0], sm.tvj[0]};
            for (int i = 1; i < kChainWaves; ++i) best2_merge(q, sm.ts1[i], sm.ts2[i], sm.tvj[i]);
            sm.path[s] = q.vj >= 0 ? q.vj >> 5 : -1;
            sm.tclear = best2_clear(q);
        }
        __syncthreads();
        if (!sm.tclear) {  // (uniform)
            double ps;
            int pj;
            const int pv = wave_race<LAYOUT>(a, trow + s, 0, tslots, a.T_target, k0, k1, w, kChainWaves, &ps, &pj);
            if (lane == 0) {
                sm.ts[w] = ps;
                sm.tv[w] = pv;
                sm.tj[w] = pj;
            }
            __syncthreads();
            if (tid == 0) {
                double bs = sm.ts[0];
                int bv = sm.tv[0], bj = sm.tj[0];
                for (int i = 1; i < kChainWaves; ++i)
                    if (tlex(sm.ts[i], sm.tv[i], sm.tj[i], bs, bv, bj)) {
                        bs = sm.ts[i];
                        bv = sm.tv[i];
                        bj = sm.tj[i];
                    }
                sm.path[s] = bs < INFINITY ? bv : -1;
            }
            __syncthreads();
        }
    }
    for (int s = tid; s <= G; s += blockDim.x) {
        a.chain[(size_t)b * (G + 1) + s] = (uint32_t)sm.path[s];  // (tag 0: the walk is a later launch)
        if (a.target_tokens) a.target_tokens[(size_t)b * (G + 1) + s] = sm.path[s];
    }
}

// The walk of every sequence over its drafts and shared-chain targets, then the call's
// error bits to the sticky word and the caller's status word.  One wave per sequence:
// its lanes load the sequence's targets and drafts into LDS together (one memory
// latency instead of one per depth), and lane 0 walks, as the fused kernel does.
constexpr int kWalkWaves = 4;
constexpr int kWalkVals = kMaxDepth + 32 * (kMaxDepth - 1);  // gamma + 1 targets, K <= 32 paths of gamma drafts

__global__ __launch_bounds__(64 * kWalkWaves) void topk_walk_kernel(TopkRaceArgs a) {
    __shared__ int32_t vals[kWalkWaves][kWalkVals];
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int b = (int)blockIdx.x * kWalkWaves + wave;
    const int K = a.K, G = a.gamma;
    if (blockIdx.x == 0 && threadIdx.x == 0) hand_over_status(a);
    const bool valid = b < a.B;
    int32_t* v = vals[wave];
    const int nt = G + 1, n = nt + K * G;  // n <= kWalkVals (K and gamma are checked by the caller)
    if (valid) {
        const uint64_t* y = a.chain + (size_t)b * nt;
        const int32_t* d = a.draft_tokens + (size_t)b * K * G;
        for (int e = lane; e < n; e += 64) v[e] = e < nt ? (int32_t)(uint32_t)y[e] : d[e - nt];
    }
    __syncthreads();
    if (!valid || lane != 0) return;
    const int32_t* d = v + nt;
    uint32_t act = K >= 32 ? 0xFFFFFFFFu : ((1u << K) - 1u);
    int tau = 0;
    bool done = false;
    for (int s = 0; s < G && !done; ++s) {
        const int ys = v[s];
        a.out_tokens[(size_t)b * (G + 1) + s] = ys;
        tau = s + 1;
        if (ys < 0) {
            done = true;
            break;
        }
        uint32_t na = 0u;
        for (int k = 0; k < K; ++k)
            if (((act >> k) & 1u) && d[k * G + s] == ys) na |= 1u << k;
        if (!na) {
            done = true;
            break;
        }
        act = na;
    }
    if (!done) {
        a.out_tokens[(size_t)b * (G + 1) + G] = v[G];
        tau = G + 1;
    }
    for (int s = tau; s <= G; ++s) a.out_tokens[(size_t)b * (G + 1) + s] = -1;
    a.out_len[b] = tau;
}

}  // namespace

hipError_t launch_walk(const TopkRaceArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL(topk_walk_kernel, dim3((unsigned)((a.B + kWalkWaves - 1) / kWalkWaves)), dim3(64 * kWalkWaves), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_topk_select(const TopkSelectArgs& a, bool bf16, hipStream_t stream) {
    const int n = a.seg[0].n_rows + a.seg[1].n_rows;
    if (n <= 0) return hipSuccess;
    if (bf16)
        hipLaunchKernelGGL(topk_select_kernel<true>, dim3(n), dim3(kTBlock), 0, stream, a);
    else
        hipLaunchKernelGGL(topk_select_kernel<false>, dim3(n), dim3(kTBlock), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_topk_race(const TopkRaceArgs& a, int layout, hipStream_t stream) {
    hipError_t e;
    if (!a.mpfr && a.target_rows <= 1) {
        // one workgroup per (sequence, chain), then the walk and the status
        const int R = (a.s_count > 0 ? a.K : 0) + (a.target_rows == 1 ? 1 : 0);
        if (R > 0) {
            const dim3 grid((unsigned)(a.B * R)), block(64 * (kChainWaves + 1));
            if (layout == 0)
                hipLaunchKernelGGL(topk_chain_kernel<0>, grid, block, 0, stream, a);
            else
                hipLaunchKernelGGL(topk_chain_kernel<1>, grid, block, 0, stream, a);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (a.target_rows == 1) {
            hipLaunchKernelGGL(topk_walk_kernel, dim3((unsigned)((a.B + kWalkWaves - 1) / kWalkWaves)), dim3(64 * kWalkWaves), 0, stream, a);
            return hipGetLastError();
        }
        return R > 0 ? hipSuccess : launch_finish_status(a.ctrl, a.status, stream);
    }
    // identical drafters (contexts group paths at every depth) or per-path target rows:
    // one workgroup per sequence, at most 8 waves (the TREE clocks need more than 128
    // registers per lane): one per draft path, and for a shared target chain up to four
    // sharing each of its races (its K-slot races are the longest of a depth)
    TopkRaceArgs b = a;
    int waves;
    if (a.target_rows == 1) {
        b.target_waves = a.K >= 7 ? 1 : (8 - a.K < 4 ? 8 - a.K : 4);
        waves = (a.K < 8 - b.target_waves ? a.K : 8 - b.target_waves) + b.target_waves;
    } else {
        b.target_waves = 0;
        waves = a.K < 8 ? a.K : 8;
    }
    if (layout == 0)
        hipLaunchKernelGGL(topk_race_kernel<0>, dim3(a.B), dim3(64 * waves), 0, stream, b);
    else
        hipLaunchKernelGGL(topk_race_kernel<1>, dim3(a.B), dim3(64 * waves), 0, stream, b);
    return hipGetLastError();
}

}  // namespace psd
