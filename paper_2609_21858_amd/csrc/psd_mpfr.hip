// psd_mpfr.hip -- drafting with identical drafters: multi-sample PFR (gfx950).
//
// Sec. 5 (eq. MPFR) with the direct finite-support sampler of the appendix "A
// better finite-support MPFR implementation": token v's unit-rate clock has
// arrivals G_{v,j} = E_0[v] + ... + E_j[v] (slot i of the keyed source is v's
// (i+1)-th exponential), and the nu samples of a context are the labels of the nu
// smallest ln G_{v,j} - l_v / T over (v, j < nu).  In Alg. "Multi-Draft ...
// (Formal)" the K drafts of a block form a context tree with multiplicities; here
// the tree is held as K paths: at depth s the paths with equal drafts so far share
// one context, whose proposal row is its lowest path's row, and the context's i-th
// sample goes to its i-th path.
//
// Streaming launches write every draft row's group maxima (and, when the caller wants
// it, its log-sum-exp).  Sampling launches have one workgroup per (sequence, path):
// one launch per depth, or one for every depth, each workgroup going on to the next
// depth as soon as the drafts its context depends on have landed.  The workgroup of a
// context's lowest path samples the context:
//  1. seeds: the largest token of the top group of each sixteenth of the row; the
//     nu-th smallest fp32 score of their first arrivals gives theta, an upper bound on
//     the context's nu-th smallest score;
//  2. since G_{v,j} >= E_0[v], every token of a sample has a slot-0 score at most
//     theta: a descent of slot 0's tree (2048- and 128-token nodes, 8-token chunks)
//     lists every token whose slot-0 score, in fp32 with a margin, is at most theta
//     (flat clocks: every group whose clock-floor bound passes);
//  3. the listed tokens' arrivals up to theta are drawn in fp32 and sorted; the first
//     nu are the samples unless two neighbours are closer than fp32 can tell apart, in
//     which case the arrivals are rebuilt exactly in fp64 and nu rounds of a
//     workgroup-wide lexicographic minimum over (score, token, arrival) emit the
//     samples in order (exact ties: lowest token, then lowest arrival).
// Measured at V = 128256, K = 4, gamma = 4, B = 64 beside the streaming launch: 15 us
// from a context's key to its samples at depth 0 (nu = 4), 9-11 us at depths 1 and 2
// (seed arrivals and level-3 draws 1.7, theta 1.2, descent 5, arrivals 2); 43 and
// 17-21 us with a barrier per tree level, theta by nu rounds and fp64 arrivals.
// The fp32 scores use (l - row maximum) / T, like the race kernel.
#include <hip/hip_runtime.h>

#include <math.h>

#include "psd_device.hpp"
#include "psd_launch.hpp"
#include "psd_layout.hpp"

namespace psd {

namespace {

constexpr int kMBlock = 256;
constexpr int kMaxGroups = 4096;  // 128-token groups of V <= 2^19
constexpr int kMCand = 1024;      // listed candidate tokens of a context
constexpr int kSeeds = 16;        // seed tokens of a row, two per workspace word
constexpr float kMMargin = 1e-3f;   // fp32 pruning margin (score units)
constexpr float kMCutSlack = 1e-3f; // slack of the per-token logit cut (score units)
constexpr uint32_t kMErrCand = 2u;
constexpr int kMWork = 2048;        // compacted (level-3 node, group) items
constexpr int kMGroupCap = 512;     // listed groups
constexpr int kMHalfCap = 256;      // listed 4-token halves
constexpr int kMFinal = 256;        // listed arrivals
// Polls of a sampler for a streamed word before it reads the row itself (a poll is about a
// microsecond), and once one row has not come.
constexpr uint32_t kRowPolls = 1u << 14, kRowPollsLate = 1u << 6;

struct MNode {
    uint32_t i;  // node index at its level
    float m;     // slot-0 minimum clock of the node
    uint32_t p;  // token holding it
};

// A 4-token half of a chunk with a token that can reach theta: entry, whether the chunk
// holds its group's minimum, chunk, half and token mask packed; its logits.
struct MHalf {
    uint32_t desc;  // entry << 10 | hold << 9 | chunk << 5 | half << 4 | token mask (4 bits)
    float x[4];
};

struct MShared {
    int seed_g[kSeeds];
    int seed_tok[kSeeds];
    float esum[kMBlock / 64][kSeeds];  // per-wave sums of the seeds' arrivals
    float sc[kMBlock];      // scores of the seeds' arrivals
    union {
        struct {  // the descent
            MNode l3[256];
            uint16_t l3_mask[256];
            uint16_t work[kMWork];
            MNode lg[kMGroupCap];
            MHalf half[kMHalfCap];
        };
        struct {  // the listed arrivals, by number and in order
            float fin_sc[kMFinal], fin_err[kMFinal];
            int fin_c[kMFinal];
            float srt_sc[kMFinal], srt_err[kMFinal];
            int srt_c[kMFinal];
        };
        struct {  // exact (fp64) scores of the listed tokens
            double cand_g[kMCand];
            double cand_s[kMCand];
            int cand_j[kMCand];
        };
        double pair[kMBlock];  // exact scores, every arrival of every listed token
    };
    int cand_v[kMCand];
    float cand_x[kMCand];
    double red_d[kMBlock / 64];
    int red_v[kMBlock / 64], red_j[kMBlock / 64], red_i[kMBlock / 64];
    uint32_t n_l3;             // listed level-3 nodes | their set group bits << 16
    int n_lg, n_half[2], n_cand, n_fin;
    float rowmax, theta;
    uint32_t kappa0, kappa1;
    int samples[32];
    int own[32];               // this path's drafts so far
    uint32_t epoch;            // the call's tag of the handed-over drafts (multi-depth launch)
    int row_late;              // the depth's row has not come (set by any thread)
};

__device__ __forceinline__ float mload(const unsigned char* row, bool bf16, int v) {
    return bf16 ? __uint_as_float((uint32_t)((const uint16_t*)row)[v] << 16) : ((const float*)row)[v];
}

// 16 bytes at any element boundary in one load (rows of an odd vocabulary start off
// the 16-byte grid).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_f32 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_b16 __attribute__((ext_vector_type(4), aligned(2)));
template <bool BF16, bool NT = false>
__device__ __forceinline__ uint4 mld16(const void* p) {
    u32x4 v;
    if constexpr (BF16)
        v = NT ? (u32x4)__builtin_nontemporal_load((const u32x4_b16*)p) : (u32x4)*(const u32x4_b16*)p;
    else
        v = NT ? (u32x4)__builtin_nontemporal_load((const u32x4_f32*)p) : (u32x4)*(const u32x4_f32*)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Raw words of 8 logits for a load issued ahead of its use (one or two 16-byte loads,
// the address clamped into the row).
template <bool BF16>
struct MRaw {
    uint4 w[BF16 ? 1 : 2];
};
template <bool BF16>
__device__ __forceinline__ void mraw_values(const MRaw<BF16>& r, float (&x)[8]) {
    if constexpr (BF16) {
        const uint4 u = r.w[0];
        x[0] = bf16_lo(u.x); x[1] = bf16_hi(u.x); x[2] = bf16_lo(u.y); x[3] = bf16_hi(u.y);
        x[4] = bf16_lo(u.z); x[5] = bf16_hi(u.z); x[6] = bf16_lo(u.w); x[7] = bf16_hi(u.w);
    } else {
        x[0] = __uint_as_float(r.w[0].x); x[1] = __uint_as_float(r.w[0].y);
        x[2] = __uint_as_float(r.w[0].z); x[3] = __uint_as_float(r.w[0].w);
        x[4] = __uint_as_float(r.w[1].x); x[5] = __uint_as_float(r.w[1].y);
        x[6] = __uint_as_float(r.w[1].z); x[7] = __uint_as_float(r.w[1].w);
    }
}

// The words of 8 logits from `base` (-inf past V).
template <bool BF16>
__device__ __forceinline__ void mraw_any(const unsigned char* row, int V, int base, MRaw<BF16>& r) {
    if (base + 8 <= V) {
        r.w[0] = mld16<BF16>(row + (size_t)base * (BF16 ? 2 : 4));
        if constexpr (!BF16) r.w[1] = mld16<BF16>(row + ((size_t)base + 4) * 4);
        return;
    }
    uint32_t b[8];  // float bits
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = __float_as_uint(base + i < V ? mload(row, BF16, base + i) : -INFINITY);
    if constexpr (BF16) {
        r.w[0] = make_uint4((b[0] >> 16) | b[1], (b[2] >> 16) | b[3], (b[4] >> 16) | b[5], (b[6] >> 16) | b[7]);
    } else {
        r.w[0] = make_uint4(b[0], b[1], b[2], b[3]);
        r.w[1] = make_uint4(b[4], b[5], b[6], b[7]);
    }
}

// 8 logits from `base` (-inf past V).
template <bool BF16>
__device__ __forceinline__ void mload8(const unsigned char* row, int V, int base, float (&x)[8]) {
    MRaw<BF16> r;
    mraw_any<BF16>(row, V, base, r);
    mraw_values<BF16>(r, x);
}

// The streaming pass reads a row once and the sampling comes back for a few hundred tokens
// of it, so its loads are non-temporal: 2.19 -> 2.03 ms per block at V = 256000, B = 256,
// K = 16 (rows far larger than the caches), 136.0 -> 135.6 us at V = 128256, B = 64,
// K = 4.
template <bool BF16>
__device__ __forceinline__ void mraw_load(const unsigned char* row, int V, int base, MRaw<BF16>& r) {
    if constexpr (BF16) {
        r.w[0] = mld16<true, true>((const uint16_t*)row + min(base, V - 8));
    } else {
        r.w[0] = mld16<false, true>((const float*)row + min(base, V - 4));
        r.w[1] = mld16<false, true>((const float*)row + min(base + 4, V - 4));
    }
}
// The 8 logits from `base` (-inf past V) out of the raw words; the row's last tokens
// are loaded here when the unit reaches past the row.
template <bool BF16>
__device__ __forceinline__ void mraw_unpack(const unsigned char* row, int V, int base, const MRaw<BF16>& r,
                                            float (&x)[8]) {
    mraw_values<BF16>(r, x);
    if (base + 8 > V) mload8<BF16>(row, V, base, x);
}

template <int LAYOUT>
__device__ __forceinline__ double clock_f64(uint32_t V, uint32_t slot, uint32_t v, uint32_t k0, uint32_t k1) {
    return LAYOUT == 0 ? tree_clock_f64(V, slot, v, k0, k1) : flat_clock_f64(slot, v, k0, k1);
}
template <int LAYOUT>
__device__ __forceinline__ float clock_f32(uint32_t V, uint32_t slot, uint32_t v, uint32_t k0, uint32_t k1) {
    return LAYOUT == 0 ? tree_clock_f32(V, slot, v, k0, k1) : flat_clock_f32(slot, v, k0, k1);
}

__device__ __forceinline__ bool lexless(double s, int v, int j, double s2, int v2, int j2) {
    return s < s2 || (s == s2 && (v < v2 || (v == v2 && j < j2)));
}

// (a list longer than kMCand is counted, not stored: the caller tightens theta and
// lists again)
__device__ __forceinline__ void push_cand(MShared& sm, int v, float x) {
    const int i = atomicAdd(&sm.n_cand, 1);
    if (i < kMCand) {
        sm.cand_v[i] = v;
        sm.cand_x[i] = x;
    }
}

// Flat clocks: the candidates of one 8-token chunk of a group whose clock-floor bound
// passes: slot-0 token clocks, scores against theta.
__device__ __forceinline__ void eval_chunk_flat(MShared& sm, const MpfrArgs& a, const float (&x)[8], uint32_t chunk,
                                                float shift, uint32_t k0, uint32_t k1) {
    const uint32_t V = (uint32_t)a.V;
    const uint32_t cs = chunk * 8u, ce = node_end(kShift1, chunk, V);
    if (cs >= V) return;
    float cmax = -INFINITY;
    for (uint32_t t = 0; t < ce - cs; ++t) cmax = fmaxf(cmax, x[t]);
    if (cmax == -INFINITY) return;
    const float theta = sm.theta;
    if (kLnClockFloor - (cmax - shift) * a.invT > theta) return;
#pragma unroll
    for (uint32_t h = 0; h < 2; ++h) {
        const Words w = philox((cs >> 2) + h, 0u, 0u, kDomainFlat, k0, k1);
        const uint32_t ws[4] = {w.w0, w.w1, w.w2, w.w3};
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
            const uint32_t v = cs + 4u * h + t;
            const float xv = x[4 * h + t];
            if (v >= ce || xv == -INFINITY) continue;
            if (ln_f32(exp1_f32(ws[t])) - (xv - shift) * a.invT <= theta) push_cand(sm, (int)v, xv);
        }
    }
}

// ---- tree clocks: the descent of slot 0's tree to the tokens that can reach theta, in
// the phases of the race kernel's: level-3 nodes with the mask of their surviving
// groups, group draws over the set bits, 16 lanes per listed group, one thread per
// listed half.

// Position of this lane's n list entries behind *count (an LDS counter), one atomic per
// wave; n may pack two counts.
__device__ __forceinline__ uint32_t wave_reserve(uint32_t* count, uint32_t n) {
    const uint32_t incl = wave_incl_sum(n);
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    uint32_t at = 0u;
    if ((threadIdx.x & 63) == 0 && tot != 0u) at = atomicAdd(count, tot);
    return (uint32_t)__builtin_amdgcn_readlane((int)at, 0) + incl - n;
}

// Listed halves of the groups [first, first + cnt) of the list, four entries per 16-lane
// row at a time.
template <bool BF16>
__device__ __forceinline__ void mlist_halves(const MpfrArgs& a, MShared& sm, const unsigned char* row, float shift,
                                             int first, int cnt, int par) {
    constexpr int U = 4;
    const int tid = threadIdx.x, c = tid & 15, r16 = tid >> 4;
    const float theta = sm.theta;
    for (int s0 = 0; s0 < cnt; s0 += 16 * U) {
        MRaw<BF16> ux[U];
        uint32_t m8[U], base[U], hold = 0u;
        float xc[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int le = s0 + q * 16 + r16;
            m8[q] = 0u;
            xc[q] = INFINITY;
            base[q] = 0u;
            if (le < cnt) {
                const MNode nd = sm.lg[first + le];
                base[q] = nd.i * 128u + (uint32_t)c * 8u;
                if ((int)base[q] < a.V) {
                    // ln m - (x - shift) / T <= theta is x - shift >= (ln m - theta) T; the cut is
                    // lowered by far more than the rounding of either form
                    // (above -inf, so that no -inf logit passes)
                    xc[q] = fmaxf((ln_f32(nd.m) - theta - kMCutSlack) * a.T, -3e38f);
                    if (nd.p >= base[q] && nd.p < base[q] + 8u) hold |= 1u << q;
                    mraw_any<BF16>(row, a.V, (int)base[q], ux[q]);
                }
            }
        }
        uint32_t nh = 0u;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (xc[q] < INFINITY) {
                float x[8];
                mraw_values<BF16>(ux[q], x);
#pragma unroll
                for (int i = 0; i < 8; ++i) m8[q] |= (uint32_t)(x[i] - shift >= xc[q]) << i;
                const int nv = a.V - (int)base[q];
                if (nv < 8) m8[q] &= (1u << nv) - 1u;
                nh += (uint32_t)((m8[q] & 15u) != 0u) + (uint32_t)((m8[q] >> 4) != 0u);
            }
        }
        uint32_t jh = wave_reserve((uint32_t*)&sm.n_half[par], nh);
        if (nh == 0u) continue;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (m8[q] == 0u) continue;
            float x[8];
            mraw_values<BF16>(ux[q], x);
            const uint32_t desc = ((uint32_t)(s0 + q * 16 + r16) << 10) | (((hold >> q) & 1u) << 9) | ((uint32_t)c << 5);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t hm = h ? m8[q] >> 4 : m8[q] & 15u;
                if (hm == 0u) continue;
                if (jh < (uint32_t)kMHalfCap) {
                    MHalf& hf = sm.half[jh];
                    hf.desc = desc | ((uint32_t)h << 4) | hm;
#pragma unroll
                    for (int t = 0; t < 4; ++t) hf.x[t] = x[4 * h + t];
                }
                ++jh;
            }
        }
    }
}

// The tokens of the first nh listed halves whose slot-0 score reaches theta.
__device__ __forceinline__ void mscore_halves(const MpfrArgs& a, MShared& sm, float shift, int first, int nh,
                                              uint32_t k0, uint32_t k1) {
    if ((int)threadIdx.x >= nh) return;
    const MHalf hf = sm.half[threadIdx.x];
    const MNode gn = sm.lg[first + (int)(hf.desc >> 10)];
    const uint32_t chunk = gn.i * 16u + ((hf.desc >> 5) & 15u), h = (hf.desc >> 4) & 1u;
    const uint32_t base4 = chunk * 8u + 4u * h;
    float mc = gn.m;
    uint32_t pc = gn.p;
    if (!((hf.desc >> 9) & 1u)) {
        const uint32_t n = node_end(kShift1, chunk, (uint32_t)a.V) - chunk * 8u;
        const Words wc = philox(chunk, 0u, 1u, kDomainTree, k0, k1);
        mc = gn.m + div_n(exp1_f32(wc.w0), n);
        pc = chunk * 8u + uniform_position(wc.w1, wc.w2, n);
    }
    const Words w = philox(chunk, 0u, 8u + h, kDomainTree, k0, k1);
    const uint32_t ws[4] = {w.w0, w.w1, w.w2, w.w3};
    const float theta = sm.theta;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (!((hf.desc >> t) & 1u)) continue;
        const uint32_t v = base4 + (uint32_t)t;
        const float E = v == pc ? mc : mc + exp1_f32(ws[t]);
        if (ln_f32(E) - (hf.x[t] - shift) * a.invT <= theta) push_cand(sm, (int)v, hf.x[t]);
    }
}

// Evaluate and empty the group list (after a barrier; ends with one).  par: parity of
// the half count in use, the other one being 0.
template <bool BF16>
__device__ __forceinline__ void mflush_groups(const MpfrArgs& a, MShared& sm, const unsigned char* row, float shift,
                                              uint32_t k0, uint32_t k1, int& par) {
    const int n = sm.n_lg;
    if (n == 0) {
        __syncthreads();
        return;
    }
    int step = 64;
    for (int first = 0; first < n;) {
        const int cnt = min(n - first, step);
        mlist_halves<BF16>(a, sm, row, shift, first, cnt, par);
        __syncthreads();
        const int nh = sm.n_half[par];
        if (threadIdx.x == 0) {
            sm.n_half[par ^ 1] = 0;  // (last read before the previous barrier)
            sm.n_lg = 0;             // (read by every thread at entry)
        }
        par ^= 1;
        if (nh > kMHalfCap) {  // (eight entries' halves always fit)
            step = max(8, cnt >> 1);
        } else {
            mscore_halves(a, sm, shift, first, nh, k0, k1);
            first += cnt;
            step = 64;
        }
        __syncthreads();
    }
}

// Every token whose slot-0 score can reach theta, counted in n_cand (the first kMCand
// are stored).  nd3: the minimum of this thread's level-3 node i3 (-1: none).  Called
// after a barrier that published theta and zero counts; ends with a barrier.
template <bool BF16>
__device__ __forceinline__ void mlist_tree(const MpfrArgs& a, MShared& sm, const unsigned char* row, const float* gm,
                                           float shift, uint32_t k0, uint32_t k1, int i3, const MNode& nd3, int& par) {
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t V = (uint32_t)a.V;
    {
        uint32_t mask = 0u;
        if (i3 >= 0) {
            const float xc = fmaxf((ln_f32(nd3.m) - sm.theta - kMCutSlack) * a.T, -3e38f);
            const float4* g4 = (const float4*)(gm + i3 * 16);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 x = g4[q];
                mask |= ((uint32_t)(x.x - shift >= xc) | ((uint32_t)(x.y - shift >= xc) << 1) |
                         ((uint32_t)(x.z - shift >= xc) << 2) | ((uint32_t)(x.w - shift >= xc) << 3))
                        << (4 * q);
            }
        }
        const uint32_t at = wave_reserve(&sm.n_l3, mask ? ((uint32_t)__popc(mask) << 16) | 1u : 0u);
        if (mask) {
            const uint32_t i = at & 0xFFFFu;
            uint32_t w = at >> 16;
            sm.l3[i] = nd3;
            sm.l3_mask[i] = (uint16_t)mask;
            for (; mask; mask &= mask - 1u, ++w)
                if (w < (uint32_t)kMWork) sm.work[w] = (uint16_t)(i * 16u + (uint32_t)__builtin_ctz(mask));
        }
    }
    __syncthreads();
    const int nl3 = (int)(sm.n_l3 & 0xFFFFu), nw = (int)(sm.n_l3 >> 16);
    const bool compact = nw <= kMWork;
    const int tot = compact ? nw : nl3 * 16;
    for (int wb = 0; wb < tot;) {
        const int i = wb + tid;
        bool pass = false;
        MNode gn = MNode{0u, 0.f, 0u};
        if (i < tot) {
            const int e = compact ? (int)sm.work[i] : i;
            if (compact || ((sm.l3_mask[e >> 4] >> (e & 15)) & 1u)) {
                const MNode pa = sm.l3[e >> 4];
                gn.i = pa.i * 16u + (uint32_t)(e & 15);
                child_min_f32(pa.m, pa.p, 2, gn.i, gn.i << kShift2, node_end(kShift2, gn.i, V), 0u, k0, k1, gn.m, gn.p);
                pass = ln_f32(gn.m) - (gm[gn.i] - shift) * a.invT <= sm.theta;
            }
        }
        const uint64_t bal = __ballot(pass);
        int at = 0;
        if (lane == 0 && bal != 0u) at = atomicAdd(&sm.n_lg, (int)__builtin_popcountll(bal));
        at = __builtin_amdgcn_readlane(at, 0) +
             (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        if (pass) sm.lg[at] = gn;  // (at most kMBlock are listed between two checks of the count)
        __syncthreads();
        wb += kMBlock;
        if (wb >= tot || sm.n_lg > kMGroupCap - kMBlock)
            mflush_groups<BF16>(a, sm, row, shift, k0, k1, par);
        else
            __syncthreads();
    }
    if (tot == 0) __syncthreads();
}

// The LSE of a far row (far_row), which is read again for the sum of
// exp((l - row maximum) / T).  red is LDS scratch of kMBlock / 64 entries.  Every thread
// calls it, after a barrier; it ends with one.
template <bool BF16>
__device__ __forceinline__ void far_row_lse(const unsigned char* row, int V, float invT, float rowmax, float* lse_out,
                                            float* red) {
    const int tid = threadIdx.x;
    const float c2 = invT * 1.4426950408889634f;
    float s = 0.f;
#pragma unroll 1
    for (int base = 8 * tid; base < V; base += 8 * kMBlock) {
        float x[8];
        mload8<BF16>(row, V, base, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) s += __builtin_amdgcn_exp2f((x[i] - rowmax) * c2);
    }
    s = row16_sum(s);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if ((tid & 63) == 0) red[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) *lse_out = rowmax * invT + ln_f32(((red[0] + red[1]) + red[2]) + red[3]);
    __syncthreads();
}

// Stream one row: the maximum of every 128-token group (to gm in LDS) and the row maximum
// (returned to every thread), and with LSE the log-sum-exp at T (to *lse_out).  red_* are
// LDS scratch of kMBlock / 64 entries.  The pass is bound by vector instructions as much
// as by memory (an exponential takes four issue slots); without LSE there are none.
template <bool BF16, bool LSE>
__device__ __forceinline__ float mstream_row(const unsigned char* row, int V, float invT, float* gm, float* lse_out,
                                             float* red_m, float* red_s, float* red_x, float* rowmax) {
    constexpr int NB = 4;  // units of a set
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ng = (V + 127) / 128;
    const float c2 = invT * 1.4426950408889634f;
    ExpSum es{kNegBig, 0.f};
    float xmax = -INFINITY;
    const int nstep = (V + 2047) / 2048;
    // software-pipelined: two sets of four units; while one is reduced the other's loads
    // are in flight (words past the row are never used; a row of fewer than 8 tokens
    // loads nothing ahead)
    MRaw<BF16> wn[2][NB];
#pragma unroll
    for (int q = 0; q < 2 * NB; ++q)
        if (V >= 8) mraw_load<BF16>(row, V, q * 2048 + 8 * tid, wn[q / NB][q % NB]);
    for (int st = 0; st < nstep; st += 2 * NB) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int st0 = st + h * NB;
            if (st0 >= nstep) break;
            float x[NB][8];
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                mraw_values<BF16>(wn[h][q], x[q]);
                const int base = (st0 + q) * 2048 + 8 * tid;
                if ((st0 + q) * 2048 + 2048 > V && base + 8 > V) mload8<BF16>(row, V, base, x[q]);
            }
            if (st0 + 2 * NB < nstep) {
#pragma unroll
                for (int q = 0; q < NB; ++q) mraw_load<BF16>(row, V, (st0 + 2 * NB + q) * 2048 + 8 * tid, wn[h][q]);
            }
            float um[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q)
                um[q] = fmaxf(fmaxf(fmaxf(x[q][0], x[q][1]), fmaxf(x[q][2], x[q][3])),
                              fmaxf(fmaxf(x[q][4], x[q][5]), fmaxf(x[q][6], x[q][7])));
            const float bm = fmaxf(fmaxf(um[0], um[1]), fmaxf(um[2], um[3]));
            row16_max_n<NB>(um);
            if ((lane & 15) == 0) {
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    const int gi = (st0 + q) * 16 + (tid >> 4);
                    if (gi < ng) gm[gi] = um[q];
                }
            }
            xmax = fmaxf(xmax, bm);
            if constexpr (LSE) {
                expsum_raise(es, bm * c2);
#pragma unroll
                for (int q = 0; q < NB; ++q) expsum_add8(es, x[q], c2);
            }
        }
    }
    float M = 0.f, sum = 0.f;
    if constexpr (LSE) sum = expsum_wave(es, xmax * c2, M);
    xmax = row16_max(xmax);
    xmax = fmaxf(xmax, __shfl_xor(xmax, 16));
    xmax = fmaxf(xmax, __shfl_xor(xmax, 32));
    if (lane == 0) {
        red_m[wave] = M;
        red_s[wave] = sum;
        red_x[wave] = xmax;
    }
    __syncthreads();
    if (tid == 0) {
        float m = red_m[0], sacc = red_s[0], xm = red_x[0];
        for (int w = 1; w < kMBlock / 64; ++w) {
            xm = fmaxf(xm, red_x[w]);
            if constexpr (LSE) {
                const float om = red_m[w], mn = fmaxf(m, om);
                sacc = sacc * __builtin_amdgcn_exp2f(m - mn) + red_s[w] * __builtin_amdgcn_exp2f(om - mn);
                m = mn;
            }
        }
        *rowmax = xm;
        if constexpr (LSE) *lse_out = xm == -INFINITY ? -INFINITY : (m + __builtin_amdgcn_logf(sacc)) * 0.69314718055994531f;
    }
    __syncthreads();
    const float xm = *rowmax;
    if constexpr (LSE) {
        static_assert(kMBlock / 64 == 4, "four waves' sums");
        if (far_row(xm, c2)) far_row_lse<BF16>(row, V, invT, xm, lse_out, red_s);  // (uniform)
    }
    return xm;
}

// Seed groups of a row: the largest group of each sixteenth of the row (lowest index on
// ties; -1 when the part has no finite logit), 16 lanes per part.  Every thread of the
// workgroup calls it; no barrier.
__device__ __forceinline__ void seed_groups(const float* gm, int ng, int* seed_g) {
    static_assert(kSeeds * 16 == kMBlock, "16 lanes per seed");
    const int r = (int)threadIdx.x >> 4, l16 = (int)threadIdx.x & 15;
    const int g0 = r * ng / kSeeds, g1 = (r + 1) * ng / kSeeds;
    float bv = -INFINITY;
    int bg = 0x7FFFFFFF;
    for (int g = g0 + l16; g < g1; g += 16)
        if (gm[g] > bv) {
            bv = gm[g];
            bg = g;
        }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
        const float ov = __shfl_xor(bv, off);
        const int og = __shfl_xor(bg, off);
        if (ov > bv || (ov == bv && og < bg)) {
            bv = ov;
            bg = og;
        }
    }
    if (l16 == 0) seed_g[r] = bv == -INFINITY ? -1 : bg;
}

// Each seed group's largest token (its lowest index holding the maximum), 16 lanes per
// group (after a barrier that published seed_g).  Every thread calls it.
template <bool BF16>
__device__ __forceinline__ void seed_tokens(const unsigned char* row, int V, const float* gm, const int* seed_g,
                                            int* seed_tok) {
    const int i = (int)threadIdx.x >> 4, sub = (int)threadIdx.x & 15, g = seed_g[i];
    int tk = 0x7FFFFFFF;
    if (g >= 0) {
        float x[8];
        const int base = g * 128 + sub * 8;
        mload8<BF16>(row, V, base, x);
#pragma unroll
        for (int t = 7; t >= 0; --t)
            if (base + t < V && x[t] == gm[g]) tk = base + t;
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) tk = min(tk, __shfl_xor(tk, off));
    if (sub == 0) seed_tok[i] = g >= 0 && tk != 0x7FFFFFFF ? tk : -1;
}

// Seed tokens in the workspace: the offset of each from its sixteenth's first group, in
// half a word (a sixteenth of a row has at most 2^15 tokens; 0xFFFF: none).
__device__ __forceinline__ int seed_base(int i, int ng) { return i * ng / kSeeds * 128; }
static_assert(kMaxGroups / kSeeds * 128 <= 0xFFFF, "a seed's offset fits half a word");

// Values that may be read while their launch still runs (the streamed rows' maxima and
// seeds, the drafts of a launch that runs every depth) are tagged words: relaxed
// device-scope atomics are coherent across the XCDs without cache write-back, and
// the tag (the call's epoch) tells a reader that this call's value has landed.
__device__ __forceinline__ void mst_dev(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t mld_dev(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t mld_dev_u32(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The call's epoch for its tagged words.
__device__ __forceinline__ uint32_t call_epoch(const MpfrArgs& a) { return epoch_after(mld_dev_u32(a.ctrl + kCtrlEpoch)); }

// The streaming launch over the draft rows of depths [stream_s, stream_s + stream_n),
// depth-major (the first depth's rows are handed out first), one row per workgroup or
// (stream_grid) several, writing each row's group maxima and, in a launch whose words
// are waited for, its maximum and seed tokens, and its LSE when the caller wants it.
// It never waits.
template <bool BF16, bool LSE>
__global__ __launch_bounds__(kMBlock, kJointPerCu) void mpfr_stream_kernel(MpfrArgs a) {
    __shared__ float red_m[kMBlock / 64], red_s[kMBlock / 64], red_x[kMBlock / 64], rowmax;
    extern __shared__ __align__(16) float gm[];  // one float per group
    __shared__ int seed_g[kSeeds], seed_tok[kSeeds];
    __shared__ uint32_t ep_s;
    const int n = a.B * a.K;
    const int ng = (a.V + 127) / 128;
    const size_t esize = BF16 ? 2 : 4;
    if (threadIdx.x == 0) ep_s = a.tok_slot ? call_epoch(a) : 0u;  // (tag 0: ordered by the streams, no reader waits)
    // rows blockIdx.x, blockIdx.x + gridDim.x, ...: with fewer workgroups than rows, the
    // first depths' rows land first
    for (int r = (int)blockIdx.x; r < n * a.stream_n; r += (int)gridDim.x) {
        const int s = a.stream_s + r / n, b = (r % n) % a.B, k = (r % n) / a.B;  // (path-major, see mpfr_draft_kernel)
        // at depth 0 every path shares one context, whose row is path 0's
        if (!LSE && s == 0 && k != 0) continue;
        const unsigned char* row = (const unsigned char*)a.logits +
                                   (((size_t)b * a.K + k) * a.s_count + (size_t)(s - a.s_begin)) * (size_t)a.V * esize;
        const size_t rid = ((size_t)b * a.K + k) * a.gamma + s;
        const float xm = mstream_row<BF16, LSE>(row, a.V, a.invT, gm, LSE ? a.draft_lse + rid : nullptr, red_m, red_s, red_x, &rowmax);
        // (mstream_row ends with a barrier: the group maxima and the epoch are in LDS)
        const uint64_t tag = (uint64_t)ep_s << 32;
        for (int g = threadIdx.x; g < ng; g += kMBlock) mst_dev(a.row_gm + rid * ng + g, tag | __float_as_uint(gm[g]));
        if (a.row_max) {
            if (threadIdx.x == 0) mst_dev(a.row_max + rid, tag | __float_as_uint(xm));
            // the row's seed tokens, for every context this row may serve
            seed_groups(gm, ng, seed_g);
            __syncthreads();
            seed_tokens<BF16>(row, a.V, gm, seed_g, seed_tok);
            __syncthreads();
            if (threadIdx.x < kSeeds / 2) {
                uint32_t w = 0u;
                for (int h = 0; h < 2; ++h) {
                    const int i = 2 * (int)threadIdx.x + h, tk = seed_tok[i];
                    w |= (tk >= 0 ? (uint32_t)(tk - seed_base(i, ng)) : 0xFFFFu) << (16 * h);
                }
                mst_dev(a.row_seed + rid * (kSeeds / 2) + threadIdx.x, tag | w);
            }
        }
        __syncthreads();  // gm and the seeds are reused by the next row
    }
}

// Bounded wait for the draft of row rid; on timeout the call's error bit 0 is set and
// the token reads as -1.
__device__ __forceinline__ int wait_draft(const MpfrArgs& a, size_t rid, uint32_t ep) {
    uint64_t v = mld_dev(a.tok_slot + rid);
    for (uint32_t i = 0; (uint32_t)(v >> 32) != ep; ++i) {
        if (i >= a.spin_limit) {
            __hip_atomic_fetch_or(a.ctrl + kCtrlCallErrors, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return -1;
        }
        __builtin_amdgcn_s_sleep(2);
        v = mld_dev(a.tok_slot + rid);
    }
    return (int)(uint32_t)v;
}

// Payload of a word the streaming launch wrote.  A launch that runs every depth may
// run beside the streaming launch: it waits (at most `polls`) for this call's tag, and
// notes in *late that the word has not come.  Launches of one depth follow the streaming
// launch in stream order and read the payload.
__device__ __forceinline__ uint32_t row_word(const MpfrArgs& a, const uint64_t* p, uint32_t ep, uint32_t polls, int* late) {
    if (!a.tok_slot) return (uint32_t)*p;
    uint64_t v = mld_dev(p);
    for (uint32_t i = 0; (uint32_t)(v >> 32) != ep; ++i) {
        if (i >= polls) {
            *late = 1;
            break;
        }
        __builtin_amdgcn_s_sleep(2);
        v = mld_dev(p);
    }
    return (uint32_t)v;
}

// The row's group maxima (to gm in LDS) by this workgroup itself, 16 lanes per group.
template <bool BF16>
__device__ __forceinline__ void read_groups(const unsigned char* row, int V, float* gm) {
    const int ng = (V + 127) / 128;
#pragma unroll 1
    for (int g = (int)threadIdx.x >> 4; g < ng; g += kMBlock / 16) {
        float x[8];
        mload8<BF16>(row, V, g * 128 + ((int)threadIdx.x & 15) * 8, x);
        float mx = x[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) mx = fmaxf(mx, x[i]);
        mx = row16_max(mx);
        if ((threadIdx.x & 15) == 0) gm[g] = mx;
    }
}

// The context's samples from the exact (fp64) scores of its nc listed tokens: nu rounds
// of the lexicographic minimum over (score, token, arrival).  Every thread calls it.
template <int LAYOUT>
__device__ __forceinline__ void exact_samples(const MpfrArgs& a, MShared& sm, int nc, int nu, float shift, uint32_t k0,
                                              uint32_t k1) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t V = (uint32_t)a.V;
    if (nc * nu <= kMBlock) {
        // every arrival j < nu of every listed token at once (one fp64 clock per
        // thread, in the seed array, free by now), the cumulative sums in arrival
        // order (the same sums as one arrival at a time), then the nu smallest
        // (score, token, arrival) by one wave: the same samples in the same order
        const int t = tid, c = t / nu, j = t % nu;
        if (t < nc * nu) sm.pair[t] = clock_f64<LAYOUT>(V, (uint32_t)j, (uint32_t)sm.cand_v[c], k0, k1);
        __syncthreads();
        if (t < nc) {
            double G = 0.0;
            for (int i = 0; i < nu; ++i) {
                G += sm.pair[t * nu + i];
                sm.pair[t * nu + i] = G;
            }
        }
        __syncthreads();
        if (t < nc * nu)
            sm.pair[t] = log(sm.pair[t]) - ((double)sm.cand_x[c] - (double)shift) / (double)a.T;
        __syncthreads();
        if (wave == 0) {
            double ps[4];
            int pv[4], pj[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = lane + 64 * q;
                const bool ok = e < nc * nu;
                ps[q] = ok ? sm.pair[e] : INFINITY;
                pv[q] = ok ? sm.cand_v[e / nu] : 0x7FFFFFFF;
                pj[q] = ok ? e % nu : 0x7FFFFFFF;
            }
            for (int r = 0; r < nu; ++r) {
                double bs = INFINITY;
                int bv = 0x7FFFFFFF, bj = 0x7FFFFFFF, bi = -1;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (lexless(ps[q], pv[q], pj[q], bs, bv, bj)) {
                        bs = ps[q];
                        bv = pv[q];
                        bj = pj[q];
                        bi = lane + 64 * q;
                    }
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    const double os = __shfl_xor(bs, off);
                    const int ov = __shfl_xor(bv, off), oj = __shfl_xor(bj, off), oi = __shfl_xor(bi, off);
                    if (lexless(os, ov, oj, bs, bv, bj)) {
                        bs = os;
                        bv = ov;
                        bj = oj;
                        bi = oi;
                    }
                }
                if (lane == 0) sm.samples[r] = bs < INFINITY ? bv : -1;
                if (bi >= 0 && (bi & 63) == lane) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (q == (bi >> 6)) ps[q] = INFINITY;
                }
            }
        }
    } else {
    for (int c = tid; c < nc; c += kMBlock) {
        const int v = sm.cand_v[c];
        const double G = clock_f64<LAYOUT>(V, 0u, (uint32_t)v, k0, k1);
        sm.cand_g[c] = G;
        sm.cand_j[c] = 0;
        sm.cand_s[c] = log(G) - ((double)sm.cand_x[c] - (double)shift) / (double)a.T;
    }
    __syncthreads();
    for (int r = 0; r < nu; ++r) {
        double bs = INFINITY;
        int bv = 0x7FFFFFFF, bj = 0x7FFFFFFF, bi = -1;
        for (int c = tid; c < nc; c += kMBlock)
            if (lexless(sm.cand_s[c], sm.cand_v[c], sm.cand_j[c], bs, bv, bj)) {
                bs = sm.cand_s[c];
                bv = sm.cand_v[c];
                bj = sm.cand_j[c];
                bi = c;
            }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double os = __shfl_xor(bs, off);
            const int ov = __shfl_xor(bv, off), oj = __shfl_xor(bj, off), oi = __shfl_xor(bi, off);
            if (lexless(os, ov, oj, bs, bv, bj)) {
                bs = os;
                bv = ov;
                bj = oj;
                bi = oi;
            }
        }
        if (lane == 0) {
            sm.red_d[wave] = bs;
            sm.red_v[wave] = bv;
            sm.red_j[wave] = bj;
            sm.red_i[wave] = bi;
        }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < kMBlock / 64; ++w)
                if (lexless(sm.red_d[w], sm.red_v[w], sm.red_j[w], bs, bv, bj)) {
                    bs = sm.red_d[w];
                    bv = sm.red_v[w];
                    bj = sm.red_j[w];
                    bi = sm.red_i[w];
                }
            sm.samples[r] = bs < INFINITY ? bv : -1;
            if (bi >= 0 && bs < INFINITY) {
                // the winner's next arrival (or none past nu)
                const int j = sm.cand_j[bi] + 1;
                if (j < nu) {
                    const double G = sm.cand_g[bi] + clock_f64<LAYOUT>(V, (uint32_t)j, (uint32_t)bv, k0, k1);
                    sm.cand_g[bi] = G;
                    sm.cand_j[bi] = j;
                    sm.cand_s[bi] = log(G) - ((double)sm.cand_x[bi] - (double)shift) / (double)a.T;
                } else {
                    sm.cand_s[bi] = INFINITY;
                }
            }
        }
        __syncthreads();
    }
    }
}

// The context's samples from fp32 scores, when those decide the order: every arrival
// whose score reaches theta is listed (8 lanes per listed token draw its next 8
// arrivals), the list is sorted by counting, and the first nu are the samples if each
// is further from its successor than both scores can err.  -ln U in fp32 is within 1.7e-7
// relative of the exact one for every one of the 2^23 uniforms (measured over all of
// them), so sums of clocks are within 1e-6 relative; the logarithm adds at most 4e-6 (3.7e-6
// measured over [2^-44, 2^8)) and the scaled logit 2.4e-7 of its size:
// 2e-5 + 1e-6 |scaled logit| is assumed, four times their sum.  Returns false when the order is not decided (exact_samples then does it).
// Every thread calls it.
template <int LAYOUT>
__device__ __forceinline__ bool sorted_samples(const MpfrArgs& a, MShared& sm, int nc, int nu, float shift, uint32_t k0,
                                               uint32_t k1) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int q = tid & 7;
    const float theta = sm.theta;
    for (int c0 = 0; c0 < nc; c0 += kMBlock / 8) {
        const int c = c0 + (tid >> 3);
        const int v = c < nc ? sm.cand_v[c] : -1;
        const float xs = c < nc ? (sm.cand_x[c] - shift) * a.invT : 0.f;
        float G0 = 0.f;
        for (int j0 = 0; j0 < nu; j0 += 8) {
            const int j = j0 + q;
            const bool on = v >= 0 && j < nu;
            float G = on ? clock_f32<LAYOUT>((uint32_t)a.V, (uint32_t)j, (uint32_t)v, k0, k1) : 0.f;
#pragma unroll
            for (int off = 1; off < 8; off <<= 1) {
                const float o = __shfl_up(G, off, 8);
                if (q >= off) G += o;
            }
            G += G0;
            const float sc = ln_f32(G) - xs;
            if (on && sc <= theta) {
                const int i = atomicAdd(&sm.n_fin, 1);
                if (i < kMFinal) {
                    sm.fin_sc[i] = sc;
                    sm.fin_err[i] = 2e-5f + 1e-6f * fabsf(xs);
                    sm.fin_c[i] = c;
                }
            }
            G0 = __shfl(G, 7, 8);
            // later arrivals score higher: on only while a token's last one reached theta
            if (__ballot(q == 7 && on && sc <= theta) == 0u) break;
        }
    }
    __syncthreads();
    const int n = sm.n_fin;
    if (n < nu || n > kMFinal) return false;  // (uniform)
    if (tid < n) {
        const float s0 = sm.fin_sc[tid];
        int r = 0;
        for (int i = 0; i < n; ++i) {
            const float o = sm.fin_sc[i];
            r += o < s0 || (o == s0 && i < tid);
        }
        sm.srt_sc[r] = s0;
        sm.srt_err[r] = sm.fin_err[tid];
        sm.srt_c[r] = sm.fin_c[tid];
    }
    __syncthreads();
    const bool in = lane < nu;  // (nu <= 32; every wave decides by itself)
    const bool clear = !in || lane + 1 >= n ||
                       sm.srt_sc[lane + 1] - sm.srt_sc[lane] > sm.srt_err[lane + 1] + sm.srt_err[lane];
    if (__ballot(!clear) != 0u) {
        __syncthreads();  // (exact_samples reuses the lists)
        return false;
    }
    if (tid < nu) sm.samples[tid] = sm.cand_v[sm.srt_c[tid]];
    return true;
}

// Depth s of path k of sequence b (every thread of the workgroup calls it; its early
// returns are uniform).  mask: the paths that shared this path's context at depth s - 1
// (in), at depth s (out).  first: no earlier depth was run by this workgroup (the
// context is formed from the caller's drafts at every depth < s).  mine: this workgroup
// sampled that context (in: at depth s - 1, out: at depth s), so it knows the drafts
// without waiting for them.  ep: the call's epoch when the launch runs every depth.  polls: of a
// wait for a streamed word.
template <bool BF16, int LAYOUT>
__device__ __forceinline__ void mpfr_depth(const MpfrArgs& a, MShared& sm, float* gm, int b, int k, int s, uint32_t ep,
                                           uint32_t& polls, bool first, uint32_t& mask, bool& mine) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t V = (uint32_t)a.V;
    const int ng = (a.V + 127) / 128, n3 = (ng + 15) / 16;
    const size_t esize = BF16 ? 2 : 4;
    const unsigned char* row = (const unsigned char*)a.logits +
                               (((size_t)b * a.K + k) * a.s_count + (size_t)(s - a.s_begin)) * (size_t)a.V * esize;
    const size_t rid = ((size_t)b * a.K + k) * a.gamma + s;

    // the row's group maxima, in flight while the context forms (used only by the
    // context's lowest path, whose row is always streamed)
    uint64_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int g = tid + i * kMBlock;
        w[i] = g < ng ? mld_dev(a.row_gm + rid * ng + g) : 0;
    }
    // ---- the context key (wave 3) and the context of path k: the paths whose drafts at
    // depths < s equal its own.  Window position i is index s + i of prefix || path; all
    // tokens but the newest are folded before the newest draft is waited for.
    uint32_t c0 = (uint32_t)a.key, c1 = (uint32_t)(a.key >> 32);
    int pre = 0;
    if (first) {
        for (int d = 0; d < s; ++d) {
            const int tk = lane < a.K ? a.draft_tokens[((size_t)b * a.K + lane) * a.gamma + d] : 0;
            const int my = __builtin_amdgcn_readlane(tk, k);
            mask &= (uint32_t)__ballot(lane < a.K && tk == my);
            if (tid == kMBlock - 64) sm.own[d] = my;
        }
    }
    if (wave == 3) {
        if (lane < a.m) pre = a.prefix[(size_t)b * a.m + lane];
        const uint64_t t = (uint64_t)(a.start_pos[b] + s);
        fold(c0, c1, (uint32_t)t, (uint32_t)(t >> 32), 0u);
        for (int i = 0; i + 1 < a.m; ++i) {
            const int g = s + i;
            const int wt = g < a.m ? __builtin_amdgcn_readlane(pre, g) : sm.own[g - a.m];
            fold(c0, c1, (uint32_t)wt, (uint32_t)i, 1u);
        }
    }
    if (!first) {
        const bool in = (mask >> (lane & 31)) & 1u && lane < 32;
        int tk = 0;
        if (in)
            tk = mine ? sm.samples[__popc(mask & ((1u << lane) - 1u))]
                      : wait_draft(a, ((size_t)b * a.K + lane) * a.gamma + (s - 1), ep);
        const int my = __builtin_amdgcn_readlane(tk, k);
        mask = (uint32_t)__ballot(in && tk == my);
        if (tid == kMBlock - 64) sm.own[s - 1] = my;
    }
    mine = k == __ffs((int)mask) - 1;
    if (!mine) return;  // the context's lowest path samples it (uniform)
    if (wave == 3) {
        if (a.m > 0) {
            const int g = s + a.m - 1;
            const int wt = g < a.m ? __builtin_amdgcn_readlane(pre, g) : sm.own[g - a.m];
            fold(c0, c1, (uint32_t)wt, (uint32_t)(a.m - 1), 1u);
        }
        if (lane == 0) {
            sm.kappa0 = c0;
            sm.kappa1 = c1;
        }
    }
    // ---- the row's maxima (and seeds): streamed by an earlier launch, or, in a launch that
    // runs every depth, by one that may still run (each word is then waited for)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int g = tid + i * kMBlock;
        if (g < ng)
            gm[g] = __uint_as_float(a.tok_slot && (uint32_t)(w[i] >> 32) != ep
                                        ? row_word(a, a.row_gm + rid * ng + g, ep, polls, &sm.row_late)
                                        : (uint32_t)w[i]);
    }
    for (int g = tid + 4 * kMBlock; g < ng; g += kMBlock)
        gm[g] = __uint_as_float(row_word(a, a.row_gm + rid * ng + g, ep, polls, &sm.row_late));
    if (tid < ((ng + 15) & ~15) - ng) gm[ng + tid] = -INFINITY;
    if (a.row_max) {
        if (tid == 0) sm.rowmax = __uint_as_float(row_word(a, a.row_max + rid, ep, polls, &sm.row_late));
        if (tid < kSeeds) {
            const uint32_t h =
                (row_word(a, a.row_seed + rid * (kSeeds / 2) + (tid >> 1), ep, polls, &sm.row_late) >> (16 * (tid & 1))) & 0xFFFFu;
            const int tk = h == 0xFFFFu ? -1 : min(seed_base(tid, ng) + (int)h, a.V - 1);
            sm.seed_tok[tid] = tk;
            sm.seed_g[tid] = tk >= 0 ? tk / 128 : -1;
        }
    }
    if (tid == 0) {
        sm.n_l3 = 0u;
        sm.n_lg = sm.n_half[0] = sm.n_half[1] = sm.n_cand = sm.n_fin = 0;
    }
    __syncthreads();
    // A row that has not come is read here: the streaming workgroup that has it may not have
    // been dispatched (the samplers and other launches may hold the places it needs), so a
    // sampler never depends on one.
    const bool late = sm.row_late != 0;
    if (!a.row_max || late) {  // (uniform)
        if (late) {
            read_groups<BF16>(row, a.V, gm);
            polls = min(polls, kRowPollsLate);
            __syncthreads();
            if (tid == 0) sm.row_late = 0;  // (read by every thread before the barrier)
        }
        seed_groups(gm, ng, sm.seed_g);
        float mx = -INFINITY;
        if (wave == 0) {
            for (int g = lane; g < ng; g += 64) mx = fmaxf(mx, gm[g]);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
            if (lane == 0) sm.rowmax = mx;
        }
        __syncthreads();
        seed_tokens<BF16>(row, a.V, gm, sm.seed_g, sm.seed_tok);
        __syncthreads();
    }
    const int nu = __popc(mask);
    const float shift = sm.rowmax;
    if (shift == -INFINITY) {  // no finite logit: every draft of the context is -1
        if (tid < nu) sm.samples[tid] = -1;
    } else {
        const uint32_t k0 = sm.kappa0, k1 = sm.kappa1;
        // ---- seed arrivals in float32 and, tree clocks, the
        // minimum of this thread's level-3 node (its root and level-4 draws with it: three
        // independent Philox calls instead of a phase per level)
        int i3 = -1;
        MNode nd3 = MNode{0u, 0.f, 0u};
        if constexpr (LAYOUT == 0) {
            const int t3 = kMBlock - 1 - tid;
            if (t3 < n3) {
                i3 = t3;
                float m, m4;
                uint32_t p, p4;
                const uint32_t i4 = (uint32_t)i3 >> 4;
                root_min_f32(V, 0u, k0, k1, m, p);
                child_min_f32(m, p, 4, i4, i4 << kShift4, node_end(kShift4, i4, V), 0u, k0, k1, m4, p4);
                child_min_f32(m4, p4, 3, (uint32_t)i3, (uint32_t)i3 << kShift3, node_end(kShift3, (uint32_t)i3, V), 0u, k0,
                              k1, nd3.m, nd3.p);
                nd3.i = (uint32_t)i3;
            }
        }
        // (one arrival per thread: the first min(nu, 16) arrivals of each seed or, for more
        // samples than that, the first nu arrivals of the better seed of every two.  Any
        // one seed then has nu arrivals, so theta is as good as the best group of the row
        // allows even where every other seed is a masked token: with 16 arrivals of each, a
        // context of 32 samples over a row that leaves one stretch of the vocabulary took
        // its theta from masked seeds and listed the whole row.)
        const int lg = nu > kMBlock / kSeeds ? 3 : 4;  // log2 of the seeds in use
        const int nsd = 1 << lg;
        const int si = tid & (nsd - 1), sj = tid >> lg;  // seed, arrival
        static_assert(kSeeds == 16 && kMBlock == 256, "16 arrivals of 16 seeds or 32 of 8");
        const int na = min(nu, kMBlock >> lg);
        int sid = si;
        if (lg == 3) {
            const int g0 = sm.seed_g[2 * si], g1 = sm.seed_g[2 * si + 1];
            sid = 2 * si + (int)(g1 >= 0 && (g0 < 0 || gm[g1] > gm[g0]));
        }
        const int sv = sm.seed_tok[sid];
        const bool on = sj < na && sv >= 0;
        float G = on ? clock_f32<LAYOUT>(V, (uint32_t)sj, (uint32_t)sv, k0, k1) : 0.f;
        for (int off = nsd; off < 64; off <<= 1) {  // the wave's arrivals of each seed
            const float o = __shfl_up(G, off);
            if (lane >= off) G += o;
        }
        if (lane >= 64 - nsd) sm.esum[wave][si] = G;
        __syncthreads();
        // ---- theta = the nu-th smallest seed score (by counting): it only has to bound the
        // context's nu-th smallest score from above.  Float32 scores are within the
        // pruning margin of the exact ones (the same assumption as every float32 bound of
        // the race), and theta carries one margin for that on top of its own.  A seed
        // token holds its group's maximum, so its logit is that maximum.
        const int ns = nsd * na;
        float s0 = INFINITY;
        if (on) {
            for (int w = 0; w < wave; ++w) G += sm.esum[w][si];
            s0 = ln_f32(G) - (gm[sm.seed_g[sid]] - shift) * a.invT;
        }
        sm.sc[tid] = s0;
        if (tid == 0) sm.theta = INFINITY;  // (fewer than nu finite arrivals)
        __syncthreads();
        if (tid < ns && s0 < INFINITY) {
            int r = 0;
            const float4* s4 = (const float4*)sm.sc;
#pragma unroll 4
            for (int i = 0; i < ns / 4; ++i) {
                const float4 o = s4[i];
                r += (int)(o.x < s0 || (o.x == s0 && 4 * i < tid)) + (int)(o.y < s0 || (o.y == s0 && 4 * i + 1 < tid)) +
                     (int)(o.z < s0 || (o.z == s0 && 4 * i + 2 < tid)) + (int)(o.w < s0 || (o.w == s0 && 4 * i + 3 < tid));
            }
            if (r == nu - 1) sm.theta = s0 + 2.f * kMMargin;
        }
        __syncthreads();

        // ---- list every token whose slot-0 score can reach theta.  A list longer than
        // kMCand tightens theta to the nu-th smallest exact slot-0 score among its first
        // kMCand tokens (nu real arrivals, so still an upper bound) and lists again.
        int par = 0;
        for (int attempt = 0;; ++attempt) {
            if constexpr (LAYOUT == 0) {
                mlist_tree<BF16>(a, sm, row, gm, shift, k0, k1, i3, nd3, par);
            } else {
                for (int g0 = 0; g0 < ng; g0 += 16) {
                    const int g = g0 + (tid >> 4);
                    if (g < ng && kLnClockFloor - (gm[g] - shift) * a.invT <= sm.theta) {
                        const uint32_t chunk = (uint32_t)g * 16u + (uint32_t)(tid & 15);
                        float x[8];
                        mload8<BF16>(row, a.V, (int)(chunk * 8u), x);
                        eval_chunk_flat(sm, a, x, chunk, shift, k0, k1);
                    }
                }
                __syncthreads();
            }
            if (sm.n_cand <= kMCand) break;
            if (attempt == 3) {  // still too many: the samples may be wrong, and the call says so
                if (tid == 0)
                    __hip_atomic_fetch_or(a.ctrl + kCtrlCallErrors, kMErrCand, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            // tighter theta: exact slot-0 scores of the stored tokens, nu-th smallest
            for (int c = tid; c < kMCand; c += kMBlock)
                sm.cand_s[c] = log(clock_f64<LAYOUT>(V, 0u, (uint32_t)sm.cand_v[c], k0, k1)) -
                               ((double)sm.cand_x[c] - (double)shift) / (double)a.T;
            __syncthreads();
            double th = INFINITY;
            for (int r = 0; r < nu; ++r) {
                double bs = INFINITY;
                int bi = 0x7FFFFFFF;
                for (int c = tid; c < kMCand; c += kMBlock)
                    if (sm.cand_s[c] < bs) {
                        bs = sm.cand_s[c];
                        bi = c;
                    }
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    const double os = __shfl_xor(bs, off);
                    const int oi = __shfl_xor(bi, off);
                    if (os < bs || (os == bs && oi < bi)) {
                        bs = os;
                        bi = oi;
                    }
                }
                if (lane == 0) {
                    sm.red_d[wave] = bs;
                    sm.red_i[wave] = bi;
                }
                __syncthreads();
                if (tid == 0) {
                    for (int w = 1; w < kMBlock / 64; ++w)
                        if (sm.red_d[w] < bs || (sm.red_d[w] == bs && sm.red_i[w] < bi)) {
                            bs = sm.red_d[w];
                            bi = sm.red_i[w];
                        }
                    if (bi >= 0 && bi < kMCand) sm.cand_s[bi] = INFINITY;
                    sm.red_d[0] = bs;
                }
                __syncthreads();
                th = sm.red_d[0];
                __syncthreads();
            }
            if (tid == 0) {
                sm.theta = fminf(sm.theta, (float)th + kMMargin);
                sm.n_l3 = 0u;
                sm.n_cand = 0;
            }
            __syncthreads();
        }

        // ---- the samples: in the order of fp32 scores where that is certain, else exact
        const int nc = min(sm.n_cand, kMCand);
        if (!sorted_samples<LAYOUT>(a, sm, nc, nu, shift, k0, k1)) exact_samples<LAYOUT>(a, sm, nc, nu, shift, k0, k1);
    }
    __syncthreads();
    // the context's r-th sample goes to its r-th path
    if (tid < 32 && ((mask >> tid) & 1u)) {
        const int y = sm.samples[__popc(mask & ((1u << tid) - 1u))];
        const size_t at = ((size_t)b * a.K + tid) * a.gamma + s;
        if (a.tok_slot) mst_dev(a.tok_slot + at, ((uint64_t)ep << 32) | (uint32_t)y);
        a.draft_tokens[at] = y;
    }
}

// One workgroup per (sequence, path).  Without tok_slot: depth a.s only.  With it:
// every depth of the call in turn, each depth's contexts formed from the drafts of the
// earlier depths as they land.  A workgroup waits for the drafts of its context's lowest
// path alone, whose workgroup has a lower index (path-major), and for streamed rows only
// for a while (row_word): the running workgroup of lowest index depends on none that
// might not be dispatched.
template <bool BF16, int LAYOUT>
__global__ __launch_bounds__(kMBlock, kJointPerCu) void mpfr_draft_kernel(MpfrArgs a) {
    __shared__ MShared sm;
    extern __shared__ __align__(16) float gm[];  // the row's group maxima (dynamic: one per group)
    // Path-major: consecutive workgroups go to the 8 XCDs in turn, and contexts are sampled
    // by their lowest paths (at depth 0 by path 0 alone), so with the K paths of a
    // sequence side by side the working ones would share 8 / gcd(8, K) of the XCDs.
    const int b = (int)blockIdx.x % a.B, k = (int)blockIdx.x / a.B;
    uint32_t mask = a.K >= 32 ? 0xFFFFFFFFu : (1u << a.K) - 1u;
    bool mine = false;
    uint32_t polls = min(a.spin_limit, kRowPolls);
    if (threadIdx.x == 0) sm.row_late = 0;
    if (!a.tok_slot) {
        mpfr_depth<BF16, LAYOUT>(a, sm, gm, b, k, a.s, 0u, polls, true, mask, mine);
        return;
    }
    if (threadIdx.x == 0) sm.epoch = call_epoch(a);
    __syncthreads();
    const uint32_t ep = sm.epoch;
    for (int s = a.s_begin; s < a.s_begin + a.s_count; ++s) {
        mpfr_depth<BF16, LAYOUT>(a, sm, gm, b, k, s, ep, polls, s == a.s_begin, mask, mine);
        __syncthreads();
    }
}

// The call's error bits to the sticky word and the caller's status word, and its epoch
// (for calls that end without a fused race kernel, whose last workgroup does this).
__global__ void finish_status_kernel(uint32_t* ctrl, uint32_t* status) {
    const uint32_t bits = __hip_atomic_exchange(ctrl + kCtrlCallErrors, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (bits) __hip_atomic_fetch_or(ctrl + kCtrlErrors, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (status) *status = bits;
    ctrl[kCtrlEpoch] = epoch_after(ctrl[kCtrlEpoch]);
}

}  // namespace

namespace {

// Dynamic LDS: the row's group maxima, padded to whole level-3 nodes.
size_t mpfr_smem(const MpfrArgs& a) { return (size_t)(((a.V + 127) / 128 + 15) & ~15) * sizeof(float); }

template <bool BF16, int LAYOUT>
hipError_t mpfr_fit(const MpfrArgs& a, bool* fits, bool* beside) {
    *fits = *beside = false;
    if (a.s_count < 2) return hipSuccess;
    int per_cu = 0, dev = 0, cus = 0;
    hipError_t e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, mpfr_draft_kernel<BF16, LAYOUT>, kMBlock,
                                                          mpfr_smem(a))) != hipSuccess)
        return e;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    *fits = (long)per_cu * cus >= (long)a.B * a.K;
    // (a streaming workgroup's LDS is below a sampler's)
    *beside = *fits && (long)a.B * a.K <= samplers_beside_streaming(cus, sizeof(MShared) + mpfr_smem(a));
    return hipSuccess;
}
// tok_slot set (the caller checked mpfr_all_depths_fit): every depth; otherwise depth a.s.
template <bool BF16, int LAYOUT>
hipError_t mpfr_sample(const MpfrArgs& a, hipStream_t stream) {
    auto fn = mpfr_draft_kernel<BF16, LAYOUT>;
    hipLaunchKernelGGL(fn, dim3((unsigned)(a.B * a.K)), dim3(kMBlock), mpfr_smem(a), stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t mpfr_all_depths_fit(const MpfrArgs& a, bool bf16, int layout, bool* fits, bool* beside) {
    if (bf16) return layout == 0 ? mpfr_fit<true, 0>(a, fits, beside) : mpfr_fit<true, 1>(a, fits, beside);
    return layout == 0 ? mpfr_fit<false, 0>(a, fits, beside) : mpfr_fit<false, 1>(a, fits, beside);
}

hipError_t launch_mpfr_sample(const MpfrArgs& a, bool bf16, int layout, hipStream_t stream) {
    if (bf16) return layout == 0 ? mpfr_sample<true, 0>(a, stream) : mpfr_sample<true, 1>(a, stream);
    return layout == 0 ? mpfr_sample<false, 0>(a, stream) : mpfr_sample<false, 1>(a, stream);
}

hipError_t launch_mpfr_stream(const MpfrArgs& a, bool bf16, hipStream_t stream) {
    const int rows = a.B * a.K * a.stream_n;
    const dim3 grid((unsigned)(a.stream_grid > 0 && a.stream_grid < rows ? a.stream_grid : rows)), block(kMBlock);
    const size_t smem = mpfr_smem(a);
    const bool lse = a.draft_lse != nullptr;
    if (bf16) {
        if (lse) hipLaunchKernelGGL((mpfr_stream_kernel<true, true>), grid, block, smem, stream, a);
        else hipLaunchKernelGGL((mpfr_stream_kernel<true, false>), grid, block, smem, stream, a);
    } else {
        if (lse) hipLaunchKernelGGL((mpfr_stream_kernel<false, true>), grid, block, smem, stream, a);
        else hipLaunchKernelGGL((mpfr_stream_kernel<false, false>), grid, block, smem, stream, a);
    }
    return hipGetLastError();
}

hipError_t launch_finish_status(uint32_t* ctrl, uint32_t* status, hipStream_t stream) {
    hipLaunchKernelGGL(finish_status_kernel, dim3(1), dim3(1), 0, stream, ctrl, status);
    return hipGetLastError();
}

}  // namespace psd
