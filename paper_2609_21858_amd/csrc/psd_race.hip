// psd_race.hip -- fused draft + verify kernel of the keyed Poisson race (gfx950).
//
// One persistent kernel per call.  Rows are numbered depth-major (all rows of
// depth 0, then depth 1, ...) and dealt round-robin to up to eight work queues,
// one per XCD (workgroup w serves queue w mod 8), so the ticket counters are not
// one contended atomic; a queue hands out its rows' 32 KiB segments in order, so
// every row a race depends on is handed out before the rows that depend on it.
//
// Per segment (key-independent, HBM-streaming): coalesced 16-byte non-temporal
// loads, the online log-sum-exp partial (sum of exp2 relative to the segment
// maximum) and the maximum logit of every 128-token group.  Each value is published
// as one 64-bit slot tagged with the call's epoch, so nothing waits for stores to
// drain and nothing is cleared between calls.  Of every nine consecutive workgroups the
// last three finish rows, the others only stream: a finishing workgroup
// gathers a row's slots and does all key-independent work (maxima, seed tokens, LSE, what
// the race draws first), takes the context key from the race one depth up the path,
// runs the keyed race, publishes the winner and the next depth's key and -- for the
// last row of a sequence -- walks the block.
//
// The race (TREE clocks): the largest tokens of the row's eighths give achievable
// scores; a level-by-level descent then expands only nodes whose lower bound
// ln(min clock of the node) - max logit / T can still beat the best score; a
// child's minimum is never below its parent's, so the parent's minimum bounds a
// child before its own draw.  Only the 128-token groups that survive are re-read.
// FLAT clocks: every group whose floor bound ln(clock floor) - max logit / T can
// win is re-read and its surviving tokens draw their Philox word.
//
// Pruning and candidate scores run in float32 with a safety margin; every
// candidate within the margin of the best is re-scored in float64 (clock rebuilt
// exactly, logit / T in double) and the winner is the lexicographic minimum of
// (score, token, slot) -- exact ties go to the lowest token, then slot.
//
// Paper passages: race = eq. EFR (Thm. "PFR reduces to EFR"); draft k races
// slot k and the target races all K slots (Prop. "heterogeneous PML bound",
// augmented space V x [K]); target chain keyed by its own prefix (stopping-time
// drafter invariance); walk = Alg. "Multi-Draft ... (Formal)".
#include <hip/hip_runtime.h>

#include <math.h>

#include <mutex>

#include "psd_device.hpp"
#include "psd_launch.hpp"
#include "psd_layout.hpp"

namespace psd {

namespace {

constexpr int kInit = 8;                   // seed tokens of a race (largest token of each eighth of the row)
constexpr int kL3Cap = 512;
constexpr int kL2Cap = 512;
constexpr int kRowEntries = 2;             // group entries per 16-lane row and evaluation pass
constexpr int kCandCap = 256;
constexpr int kWorkCap = 2048;             // compacted (level-3 node, group) items
constexpr int kRolePeriod = 9;             // workgroup roles: of every kRolePeriod blocks,
constexpr int kRoleFinish = 3;             // kRoleFinish finish rows and the others stream
constexpr int kHalfCap = 256;              // 4-token halves listed by one evaluation pass
constexpr int kPassGroups = 16 * kRowEntries;  // group entries of one evaluation pass
constexpr int kEvalGroups = 128;           // group entries of one evaluation pass (tree clocks; with 64 the V = 32000,
                                           // K = 4 block, a chain of races, takes 4 % longer, 100 vs 96 us, and the
                                           // V = 151936, K = 8 one, bound by streaming, 0.9 % less, 1383 vs 1395)
constexpr int kBuckets = 32;               // bound buckets of the group list's evaluation order
constexpr float kMargin = 1e-3f;           // float32 pruning / candidate margin (score units)
constexpr float kCutSlack = 1e-3f;         // slack of the per-token logit cut (score units)
constexpr uint32_t kErrSpin = 1u, kErrCand = 2u;

struct Node {
    uint32_t id;  // (slot << 20) | node index
    float m;      // float32 minimum clock of the node
    uint32_t p;   // token holding that minimum
};

// A 4-token half of a chunk that can still win: entry (local index), chunk, half
// and token mask packed in desc; cref 0 when the chunk needs its own minimum drawn
// (-1: the chunk holds the group minimum); its logits.
struct Half {
    uint32_t desc;  // entry << 9 | chunk << 5 | half << 4 | token mask (4 bits)
    int cref;
    float x[4];
};

struct Shared {
    float m3[256];
    int init_v[kInit];     // seed groups of the race (-1: none)
    int seed_tok[kInit];   // seed tokens of the race (-1: none)
    float part[64];        // LSE partial sum of every segment
    Node l3[kL3Cap];
    Node l2[kL2Cap];
    int cand_v[kCandCap];
    int cand_j[kCandCap];
    float cand_s[kCandCap];
    float cand_x[kCandCap];
    double red_s[kBlock / 64];
    int red_v[kBlock / 64];
    int red_j[kBlock / 64];
    float red_a[2][kBlock / 64];  // per-wave LSE partials of the streamed segment (by parity)
    float red_b[2][kBlock / 64];
    int n_l2, n_cand;
    uint32_t n_l3;         // listed level-3 nodes | their set group bits << 16
    int best_key;
    int tick[4];
    int ph_first[kMaxPhases], ph_depth[kMaxPhases], ph_nd[kMaxPhases];  // work-order phases
    uint32_t epoch;
    // A finisher streams only before its first row, so the two share their place: the LDS
    // of four workgroups fits a CU up to V = 256000 with K = 16 (2.17 ms per block with three).
    union {
        float gst[2][128];         // group maxima of the streamed segment (by parity)
        uint16_t l3_mask[kL3Cap];  // groups of a listed level-3 node that can still win (bit i: its i-th)
    };
    int win_token, win_slot;
    float rowmax;
    uint32_t kappa0, kappa1;
    int have_key;             // the key was there when the row was folded
    uint32_t next0, next1;  // partial context key of the path's next depth
    int newest;             // winner of the race one depth up the path (it came with the key)
    // where the race's winner goes, ready before the race: the next depth's key words
    // (null: no race of the call reads them), the row's token slot, the caller's outputs
    uint64_t* pub_key;
    uint64_t* pub_tok;
    int32_t* pub_out;
    int key_min, key_max;   // (token, slot) range of the candidates near the best
    uint32_t err_local;       // error bits this workgroup recorded (it then publishes them with a release)
    uint16_t work[kWorkCap];  // compacted work items (level-3 list index * 16 + group)
    uint32_t n_ev[2];                 // listed halves, per pass parity
    Half half[kHalfCap];
    // evaluation order of the group list (order_groups)
    float ord_wmin[kBlock / 64];          // per-wave smallest bound
    int ord_hist[kBuckets];               // entries per bound bucket
    int ord_bmin[kBuckets];               // smallest bound per bucket (ordered key)
    int ord_pass[(kL2Cap + kPassGroups - 1) / kPassGroups];  // bucket of each pass's first entry
};
static_assert(sizeof(Half) * kHalfCap >= sizeof(Node) * kL2Cap, "the reordering stages the group list in half[]");

// Dynamic LDS after Shared: the group maxima gm (ng floats, padded with -inf to whole
// level-3 nodes), then the level-4 node list of a race (K slots x level-4 nodes; sized
// at launch).
__host__ __device__ constexpr int padded_groups(int ng) { return (ng + 15) & ~15; }
__device__ __forceinline__ Node* level4_list(const float* gm, int ng) { return (Node*)(gm + padded_groups(ng)); }

struct Row {
    int kind;  // 0 draft, 1 target
    int b, k, s;
    int row_id;
    const unsigned char* ptr;
    int slot0, nslots;
    float invT;
    float T;
    float shift;  // the row's maximum logit: fp32 scores and bounds use (l - shift) / T
};

// Scaled logit (l - shift) / T of the race's fp32 scores and bounds.  Near the
// top of the row the subtraction is exact (Sterbenz), so the scaled value of every
// token that can still win is O(tens) and rounds to a few 1e-6 score units
// whatever the magnitude of l / T; tokens far below the maximum have scores far
// above the threshold, where rounding cannot change a decision.
__device__ __forceinline__ float scaled(const Row& r, float x) { return (x - r.shift) * r.invT; }

__device__ __forceinline__ uint32_t* ctrl_of(const RaceArgs& a) { return (uint32_t*)(a.ws + a.L.ctrl); }

// Errors of the running call; its last workgroup hands them to the sticky word and
// to the caller's status word.  The workgroup also notes them in LDS, so that its
// exit publishes them with a release (see the end of race_kernel).
__device__ __forceinline__ void set_error(const RaceArgs& a, uint32_t bit) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __hip_atomic_fetch_or(ctrl_of(a) + kCtrlCallErrors, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    atomicOr(&reinterpret_cast<Shared*>(smem_raw)->err_local, bit);
}

// Cross-workgroup slots are touched only with relaxed device-scope atomics, which
// are coherent across the XCDs without L2-wide write-back / invalidate; each slot
// carries its epoch, so a reader knows when the producer's value has landed.
template <typename T>
__device__ __forceinline__ void st_dev(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T ld_dev(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Bounded wait for a slot whose tag (high 32 bits) equals the epoch.  On timeout an
// error bit is recorded and the stale value is returned, so every wave terminates.
__device__ __forceinline__ uint64_t wait_slot(const RaceArgs& a, const uint64_t* p, uint32_t epoch) {
    uint64_t v = ld_dev(p);
    for (uint32_t i = 0; (uint32_t)(v >> 32) != epoch; ++i) {
        if (i >= a.spin_limit) {
            set_error(a, kErrSpin);
            break;
        }
        __builtin_amdgcn_s_sleep(2);
        v = ld_dev(p);
    }
    return v;
}

// Bounded wait of a wave for what the race of row `prod` publishes, one word per lane in
// one load: the two words of the next depth's key (lanes 0 and 1) and, when asked, its
// winner (lane 2).  (Polls served by the XCD's own L2, with a path's rows handed out to
// one XCD, measured the same.)  Returns the lane's word.
__device__ __forceinline__ bool wait_key(const RaceArgs& a, int prod, uint32_t epoch, bool winner, bool once,
                                         uint32_t& word) {
    const int lane = threadIdx.x & 63;
    const int n = winner ? 3 : 2;
    const uint64_t* p = lane < 2 ? (const uint64_t*)(a.ws + a.L.keys) + 2 * (size_t)prod + lane
                                 : (const uint64_t*)(a.ws + a.L.tok) + prod;
    uint64_t w = 0;
    for (uint32_t i = 0;; ++i) {
        if (lane < n) w = ld_dev(p);
        word = (uint32_t)w;
        if (__ballot(lane < n && (uint32_t)(w >> 32) != epoch) == 0u) return true;
        if (once) return false;
        if (i >= a.spin_limit) {
            if (lane == 0) set_error(a, kErrSpin);
            return true;
        }
        __builtin_amdgcn_s_sleep(2);
    }
}

__device__ __forceinline__ int target_row_id(const RaceArgs& a, int b, int k, int s) {
    const int D = a.B * a.K * a.gamma;
    return a.target_rows == 1 ? D + b * (a.gamma + 1) + s : D + (b * a.K + k) * (a.gamma + 1) + s;
}

__device__ __forceinline__ int draft_row_id(const RaceArgs& a, int b, int k, int s) {
    return (b * a.K + k) * a.gamma + s;
}

__device__ __forceinline__ int wait_token(const RaceArgs& a, int rid, uint32_t epoch) {
    return (int)(uint32_t)wait_slot(a, (const uint64_t*)(a.ws + a.L.tok) + rid, epoch);
}

// Next work item of queue q (of nq): the queue's rows are R = q, q + nq, ... in
// depth-major order, each handed out segment by segment.  Returns n_items when the
// queue is exhausted.
__device__ __forceinline__ int take_item(const RaceArgs& a, int q, int nq) {
    const uint32_t t = atomicAdd(ctrl_of(a) + ctrl_queue(q), 1u);
    const uint32_t R = (uint32_t)q + (uint32_t)nq * (t / (uint32_t)a.L.nseg);
    return R >= (uint32_t)a.n_rows ? a.n_items : (int)(R * (uint32_t)a.L.nseg + t % (uint32_t)a.L.nseg);
}

// Next row of row queue q (of nq) for a finishing workgroup: rows R = q, q + nq, ...
// in work order.  Returns n_rows when the queue is exhausted.
__device__ __forceinline__ int take_row(const RaceArgs& a, int q, int nq) {
    const uint32_t t = atomicAdd(ctrl_of(a) + ctrl_queue(kMaxQueues + q), 1u);
    const uint32_t R = (uint32_t)q + (uint32_t)nq * t;
    return R >= (uint32_t)a.n_rows ? a.n_rows : (int)R;
}

// ---------------------------------------------------------------- logits access

template <bool BF16>
__device__ __forceinline__ float load_logit(const unsigned char* row, int v) {
    if constexpr (BF16)
        return __uint_as_float((uint32_t)((const uint16_t*)row)[v] << 16);
    else
        return ((const float*)row)[v];
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes at any element boundary: rows of an odd vocabulary start off the 16-byte
// grid.  gfx950 serves such a load with one instruction (global_load_dwordx4), at the
// price of one more cache line per wave: a whole call at V = 50257, K = 3, gamma = 4,
// B = 24, bf16 takes 105 us against 148 us with element-by-element loads of such rows.
typedef uint32_t u32x4_f32 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_b16 __attribute__((ext_vector_type(4), aligned(2)));

template <bool BF16, bool NT>
__device__ __forceinline__ uint4 ld16(const void* p) {
    u32x4 v;
    if constexpr (BF16)
        v = NT ? (u32x4)__builtin_nontemporal_load((const u32x4_b16*)p) : (u32x4)*(const u32x4_b16*)p;
    else
        v = NT ? (u32x4)__builtin_nontemporal_load((const u32x4_f32*)p) : (u32x4)*(const u32x4_f32*)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Raw 16-byte words of one 8-token unit (bf16: one word, float32: two).
template <bool BF16>
struct Unit {
    uint4 w[BF16 ? 1 : 2];
};

template <bool BF16>
__device__ __forceinline__ void unpack_unit(const Unit<BF16>& u, float (&x)[8]) {
    if constexpr (BF16) {
        x[0] = bf16_lo(u.w[0].x); x[1] = bf16_hi(u.w[0].x); x[2] = bf16_lo(u.w[0].y); x[3] = bf16_hi(u.w[0].y);
        x[4] = bf16_lo(u.w[0].z); x[5] = bf16_hi(u.w[0].z); x[6] = bf16_lo(u.w[0].w); x[7] = bf16_hi(u.w[0].w);
    } else {
        x[0] = __uint_as_float(u.w[0].x); x[1] = __uint_as_float(u.w[0].y);
        x[2] = __uint_as_float(u.w[0].z); x[3] = __uint_as_float(u.w[0].w);
        x[4] = __uint_as_float(u.w[1].x); x[5] = __uint_as_float(u.w[1].y);
        x[6] = __uint_as_float(u.w[1].z); x[7] = __uint_as_float(u.w[1].w);
    }
}

// The words of 8 consecutive logits starting at `base` (-inf past V): vector loads
// where all eight lie inside the row, else element by element.
template <bool BF16>
__device__ __forceinline__ void load_words(const unsigned char* row, int V, int base, Unit<BF16>& u) {
    if (base + 8 <= V) {
        u.w[0] = ld16<BF16, false>(row + (size_t)base * (BF16 ? 2 : 4));
        if constexpr (!BF16) u.w[1] = ld16<BF16, false>(row + ((size_t)base + 4) * 4);
        return;
    }
    uint32_t b[8];  // float bits
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = __float_as_uint(base + i < V ? load_logit<BF16>(row, base + i) : -INFINITY);
    if constexpr (BF16) {
        u.w[0] = make_uint4((b[0] >> 16) | b[1], (b[2] >> 16) | b[3], (b[4] >> 16) | b[5], (b[6] >> 16) | b[7]);
    } else {
        u.w[0] = make_uint4(b[0], b[1], b[2], b[3]);
        u.w[1] = make_uint4(b[4], b[5], b[6], b[7]);
    }
}

template <bool BF16>
__device__ __forceinline__ void load8(const unsigned char* row, int V, int base, float (&x)[8]) {
    Unit<BF16> u;
    load_words<BF16>(row, V, base, u);
    unpack_unit<BF16>(u, x);
}

// The streaming pass's loads: the address is clamped into the row, so every load is
// unconditional (non-temporal: the pass reads the logits once) and the compiler can
// wait for them one by one.  A unit that reaches past the row holds other tokens'
// words; its reader replaces them.  V >= 8.
template <bool BF16>
__device__ __forceinline__ void load_unit(const unsigned char* row, int V, int base, Unit<BF16>& u) {
    if constexpr (BF16) {
        u.w[0] = ld16<true, true>((const uint16_t*)row + min(base, V - 8));
    } else {
        u.w[0] = ld16<false, true>((const float*)row + min(base, V - 4));
        u.w[1] = ld16<false, true>((const float*)row + min(base + 4, V - 4));
    }
}

// ---------------------------------------------------------------- streaming pass

__device__ __forceinline__ void lse_combine(float& m, float& s, float om, float os) {
    const float mn = fmaxf(m, om);
    if (mn == -INFINITY) return;
    s = (m == -INFINITY ? 0.f : s * __builtin_amdgcn_exp2f(m - mn)) +
        (om == -INFINITY ? 0.f : os * __builtin_amdgcn_exp2f(om - mn));
    m = mn;
}

__device__ __forceinline__ void lse_merge_finite(float& m, float& s, float om, float os) {
    const float mn = fmaxf(m, om);
    s = s * __builtin_amdgcn_exp2f(m - mn) + os * __builtin_amdgcn_exp2f(om - mn);
    m = mn;
}

// The LSE of a far row (far_row) by one wave, which reads the row again for the sum of
// exp((l - row maximum) / T).
template <bool BF16>
__device__ __forceinline__ float far_row_lse(const unsigned char* row, int V, float invT, float rowmax) {
    const float c2 = invT * 1.4426950408889634f;
    float s = 0.f;
#pragma unroll 1
    for (int base = 8 * (threadIdx.x & 63); base < V; base += 8 * 64) {
        float x[8];
        load8<BF16>(row, V, base, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) s += __builtin_amdgcn_exp2f((x[i] - rowmax) * c2);
    }
    s = row16_sum(s);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    return rowmax * invT + ln_f32(s);
}

// One 32 KiB segment: the maximum logit of every 128-token group (16 lanes hold a
// group) and the segment's sum of exp2(l * log2e / T - M), M = log2e / T * (segment
// maximum).  Unless the workgroup is about to finish a row (which can wait on other
// workgroups), thread 0 takes its next ticket while the loads are in flight: a
// ticket held through such a wait would stall the rows that need that segment.
template <bool BF16>
constexpr int units_per_segment() {
    return BF16 ? 8 : 4;  // 2048-token units
}

// Issue the loads of one segment (one 8-token unit per thread and unit).
template <bool BF16>
__device__ __forceinline__ void issue_segment(const RaceArgs& a, const Row& r, int seg,
                                              Unit<BF16> (&u)[units_per_segment<BF16>()]) {
    constexpr int NU = units_per_segment<BF16>();
    const int seg0 = seg * (BF16 ? kSegTokensBf16 : kSegTokensF32);
    // a row of fewer than 8 tokens: read (and ignored) from the workspace's control words
    const unsigned char* row = a.V < 8 ? a.ws : r.ptr;
    const int n = max(a.V, 8);
#pragma unroll
    for (int q = 0; q < NU; ++q) load_unit<BF16>(row, n, seg0 + q * kBlock * 8 + 8 * threadIdx.x, u[q]);
}

// Consume a loaded segment: per-wave LSE partials and the maximum of every
// 128-token group, staged in LDS (parity p) for publish_segment.
template <bool BF16>
__device__ __forceinline__ void consume_segment(const RaceArgs& a, const Row& r, int seg, Shared& sm, int p,
                                                const Unit<BF16> (&u)[units_per_segment<BF16>()]) {
    constexpr int NU = units_per_segment<BF16>();
    constexpr int UT = kBlock * 8;
    const int tid = threadIdx.x, lane = tid & 63;
    const int V = a.V;
    const int seg0 = seg * (BF16 ? kSegTokensBf16 : kSegTokensF32);
    const float c2 = r.invT * 1.4426950408889634f;
    float mrun = kNegBig, srun = 0.f;
#pragma unroll
    for (int q = 0; q < NU; ++q) {
        float x[8];
        unpack_unit<BF16>(u[q], x);
        const int ub = seg0 + q * UT;
        if (ub + UT > V) {  // uniform: this unit reaches past the row
            const int base = ub + 8 * tid;
            if (base < V && base + 8 > V) {
                load8<BF16>(r.ptr, V, base, x);  // the row's last tokens (V not a multiple of 8)
            } else if (base >= V) {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = -INFINITY;
            }
        }
        const float um = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
        const float g = row16_max(um);
        if ((lane & 15) == 0) sm.gst[p][q * 16 + (tid >> 4)] = g;
        // (the reference is raised to every new maximum: a branch around that, as in the
        // identical-drafter streaming pass, splits the loop in which the loads are waited for
        // one by one: 118 vs 95 us per call at V = 128256, K = 4, B = 64)
        const float mn = fmaxf(mrun, um * c2);
        float acc = srun * __builtin_amdgcn_exp2f(mrun - mn);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += __builtin_amdgcn_exp2f(fmaf(x[i], c2, -mn));
        srun = acc;
        mrun = mn;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lse_merge_finite(mrun, srun, __shfl_xor(mrun, off), __shfl_xor(srun, off));
    if (lane == 0) {
        sm.red_a[p][tid >> 6] = mrun;
        sm.red_b[p][tid >> 6] = srun;
    }
}

// Publish a consumed segment (after a barrier): one 64-bit slot per group and per
// 2048-token block, written by consecutive lanes, and the segment's LSE partial.
template <bool BF16>
__device__ __forceinline__ void publish_segment(const RaceArgs& a, int row_id, int seg, Shared& sm, int p) {
    constexpr int NU = units_per_segment<BF16>();
    const int tid = threadIdx.x;
    const int seg0 = seg * (BF16 ? kSegTokensBf16 : kSegTokensF32);
    const uint64_t ep = (uint64_t)sm.epoch << 32;
    const int g0 = seg0 >> 7;
    if (tid < NU * 16 && g0 + tid < a.L.ng) {
        uint64_t* gslot = (uint64_t*)(a.ws + a.L.gmax) + (size_t)row_id * a.L.ng;
        st_dev(gslot + g0 + tid, ep | __float_as_uint(sm.gst[p][tid]));
    } else if (tid >= 128 && tid < 128 + NU && (seg0 >> 11) + (tid - 128) < a.L.n3) {
        const int q = tid - 128;
        float mx = sm.gst[p][16 * q];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sm.gst[p][16 * q + i]);
        uint64_t* m3slot = (uint64_t*)(a.ws + a.L.m3) + (size_t)row_id * a.L.n3;
        st_dev(m3slot + (seg0 >> 11) + q, ep | __float_as_uint(mx));
    }
    if (tid == 0) {
        float m = sm.red_a[p][0], s = sm.red_b[p][0];
        for (int w = 1; w < kBlock / 64; ++w) lse_merge_finite(m, s, sm.red_a[p][w], sm.red_b[p][w]);
        uint64_t* part = (uint64_t*)(a.ws + a.L.part) + (size_t)row_id * a.L.nseg;
        st_dev(part + seg, ep | __float_as_uint(s));
    }
}

// ---------------------------------------------------------------- race search

__device__ __forceinline__ float current_threshold(Shared& sm) {
    return ordered_value(__hip_atomic_load(&sm.best_key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) +
           kMargin;
}

__device__ __forceinline__ void push_node(Node* list, int* count, int cap, uint32_t id, float m, uint32_t p) {
    const int i = atomicAdd(count, 1);
    if (i < cap) list[i] = Node{id, m, p};
}

__device__ __forceinline__ void push_candidate(Shared& sm, const RaceArgs& a, int v, int j, float s, float x) {
    const int i = atomicAdd(&sm.n_cand, 1);
    if (i < kCandCap) {
        sm.cand_v[i] = v;
        sm.cand_j[i] = j;
        sm.cand_s[i] = s;
        sm.cand_x[i] = x;
    } else {
        set_error(a, kErrCand);
    }
}

// Keep only candidates within the margin of the current best (thread 0, between barriers).
__device__ __forceinline__ void compact_candidates(Shared& sm) {
    if (sm.n_cand <= kCandCap / 2) return;
    const float lim = ordered_value(sm.best_key) + kMargin;
    const int nc = min(sm.n_cand, kCandCap);
    int o = 0;
    for (int i = 0; i < nc; ++i)
        if (sm.cand_s[i] <= lim) {
            sm.cand_v[o] = sm.cand_v[i];
            sm.cand_j[o] = sm.cand_j[i];
            sm.cand_s[o] = sm.cand_s[i];
            sm.cand_x[o] = sm.cand_x[i];
            ++o;
        }
    sm.n_cand = o;
}

// Scores of the tokens of mask (bit t: token base4 + t) of one 4-token half, given
// the chunk's minimum (mc, pc) and the half's Philox words; INFINITY elsewhere and
// where the token cannot beat thr.
template <int LAYOUT>
__device__ __forceinline__ void half_scores(const Row& r, uint32_t base4, uint32_t mask, const float (&x)[4], float mc,
                                            uint32_t pc, const Words& w, float thr, float (&sc)[4]) {
    const uint32_t ws[4] = {w.w0, w.w1, w.w2, w.w3};
    const float lnmc = LAYOUT == 0 ? ln_f32(mc) : 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        sc[t] = INFINITY;
        if (!((mask >> t) & 1u)) continue;
        const uint32_t v = base4 + (uint32_t)t;
        if constexpr (LAYOUT == 0) {
            if (v == pc)
                sc[t] = lnmc - scaled(r, x[t]);
            else if (lnmc - scaled(r, x[t]) <= thr)
                sc[t] = ln_f32(mc + exp1_f32(ws[t])) - scaled(r, x[t]);
        } else {
            sc[t] = ln_f32(exp1_f32(ws[t])) - scaled(r, x[t]);
        }
    }
}

// Lower the best score to the half's smallest score.
__device__ __forceinline__ void offer_best(Shared& sm, const float (&sc)[4]) {
    const float mn = fminf(fminf(sc[0], sc[1]), fminf(sc[2], sc[3]));
    if (mn < INFINITY) atomicMin(&sm.best_key, ordered_key(mn));
}

// List the half's scores within the margin of the best as candidates.  Callers
// offer every half of the round first and separate the two steps by a barrier, so
// that only near-ties of the best are listed.
__device__ __forceinline__ void list_near(Shared& sm, const RaceArgs& a, uint32_t base4, uint32_t slot,
                                          const float (&sc)[4], const float (&x)[4]) {
    const float thr = current_threshold(sm);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (sc[t] <= thr) push_candidate(sm, a, (int)(base4 + (uint32_t)t), (int)slot, sc[t], x[t]);
}

// ---- flat clocks: evaluation of the listed groups.
//
// Evaluate listed group entries [first, first + n): 16 lanes hold the 16 chunks of
// one entry (8 tokens each); each row takes kRowEntries entries, whose loads are
// issued together.  The 4-token halves with a token that can still win against the
// clock floor go to an LDS list and are scored one per thread (a wave runs every
// branch any of its lanes takes, so the work is listed rather than done by each
// chunk's lane).  Halves beyond the list's capacity are done by their chunk's lane.
// Raw logits of this lane's chunk of the entries of the pass starting at `first`
// (list end `end`; nothing is loaded past it).  Words past V are never used.
template <bool BF16>
__device__ __forceinline__ void load_pass(const RaceArgs& a, const Row& r, const Shared& sm, int first, int end,
                                          Unit<BF16> (&ux)[kRowEntries]) {
    const int c = threadIdx.x & 15, row = threadIdx.x >> 4;
#pragma unroll
    for (int q = 0; q < kRowEntries; ++q) {
        const int e = first + row * kRowEntries + q;
        if (e < end) {
            const uint32_t g = sm.l2[e].id & 0xFFFFFu;
            load_words<BF16>(r.ptr, a.V, (int)(g * kGroupTokens + (uint32_t)c * 8u), ux[q]);
        }
    }
}

// The scored half a thread holds at the end of an evaluation pass (its logits stay
// in the half's list entry).
struct HalfOut {
    float sc[4];
    uint32_t base4, slot;
    bool valid;
};

template <bool BF16>
__device__ __forceinline__ void eval_groups(const RaceArgs& a, const Row& r, Shared& sm, const float* gm, int first,
                                            int n, int end, int par, uint32_t k0, uint32_t k1, HalfOut& ho,
                                            uint32_t& ovf, Unit<BF16> (&ux)[kRowEntries]) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int c = tid & 15;
    const int row = tid >> 4;  // 16 rows of 16 lanes
    const uint32_t V = (uint32_t)a.V;
    // this pass's logits were loaded into ux by the caller or the previous pass
    float x[kRowEntries][8];
    Node nd[kRowEntries];
    bool act[kRowEntries];
#pragma unroll
    for (int q = 0; q < kRowEntries; ++q) {
        const int e = first + row * kRowEntries + q;
        act[q] = e < first + n;
        nd[q] = act[q] ? sm.l2[e] : Node{0u, 0.f, 0u};
        unpack_unit<BF16>(ux[q], x[q]);
    }
    // What each chunk needs: the words of each half with a token that can still win.
    const float thr0 = current_threshold(sm);
    uint32_t hm[kRowEntries][2];
    int nh = 0;
#pragma unroll
    for (int q = 0; q < kRowEntries; ++q) {
        const uint32_t g = nd[q].id & 0xFFFFFu;
        const uint32_t base = g * kGroupTokens + (uint32_t)c * 8u;
        const float lnm = kLnClockFloor;
        hm[q][0] = hm[q][1] = 0u;
        if (act[q] && lnm - scaled(r, gm[g]) <= thr0) {
            // a token can reach thr0 only if lnm - (x - shift) / T <= thr0, i.e.
            // x - shift >= (lnm - thr0) T; the cut is lowered by kCutSlack, far more
            // than the rounding of either form, so the listed tokens include every
            // such token (compared in the shifted frame: no rounding of shift + cut)
            const float xc = (lnm - thr0 - kCutSlack) * r.T;
            uint32_t m8 = 0u;
#pragma unroll
            for (int i = 0; i < 8; ++i) m8 |= (uint32_t)(x[q][i] - r.shift >= xc) << i;
            const int nv = (int)V - (int)base;  // tokens of this chunk inside the row
            if (nv < 8) m8 &= nv > 0 ? (1u << nv) - 1u : 0u;
            hm[q][0] = m8 & 15u;
            hm[q][1] = m8 >> 4;
        }
        nh += (int)(hm[q][0] != 0u) + (int)(hm[q][1] != 0u);
    }
    // list positions: wave prefix sum of the halves, one atomic per wave
    const uint32_t mine = (uint32_t)nh;
    const uint32_t incl = wave_incl_sum(mine);
    const uint32_t wtot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    uint32_t wbase = 0u;
    if (lane == 0 && wtot != 0u) wbase = atomicAdd(&sm.n_ev[par], wtot);
    const uint32_t mb = (uint32_t)__builtin_amdgcn_readlane((int)wbase, 0) + incl - mine;
    int jh = (int)mb;
    ovf = 0u;  // halves beyond the list (bit 8q + 4h + t: token t of half h of entry q)
#pragma unroll
    for (int q = 0; q < kRowEntries; ++q) {
        const int le = row * kRowEntries + q;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (hm[q][h]) {
                if (jh < kHalfCap) {
                    Half& hf = sm.half[jh];
                    hf.desc = ((uint32_t)le << 9) | ((uint32_t)c << 5) | ((uint32_t)h << 4) | hm[q][h];
                    hf.x[0] = x[q][4 * h];
                    hf.x[1] = x[q][4 * h + 1];
                    hf.x[2] = x[q][4 * h + 2];
                    hf.x[3] = x[q][4 * h + 3];
                } else {
                    ovf |= hm[q][h] << (8 * q + 4 * h);
                }
                ++jh;
            }
        }
    }
    // the next pass's logits, in flight while this pass draws and scores
    load_pass<BF16>(a, r, sm, first + kPassGroups, end, ux);
    __syncthreads();
    // the other parity's counts were read in the previous pass: clear them for the next
    if (tid == 0) sm.n_ev[par ^ 1] = 0u;
    // halves, one per thread (at most one: kHalfCap == kBlock): scores, and the best
    // lowered to each half's smallest; the caller lists near-ties after a barrier
    static_assert(kHalfCap == kBlock, "one listed half per thread");
    {
        const int nj = min((int)sm.n_ev[par], kHalfCap);
        const float thr = current_threshold(sm);
#pragma unroll
        for (int t = 0; t < 4; ++t) ho.sc[t] = INFINITY;
        ho.base4 = ho.slot = 0u;
        ho.valid = tid < nj;
        if (ho.valid) {
            const Half hf = sm.half[tid];
            const Node pn = sm.l2[first + (int)(hf.desc >> 9)];
            ho.slot = pn.id >> 20;
            const uint32_t g = pn.id & 0xFFFFFu;
            const uint32_t chunk = g * 16u + ((hf.desc >> 5) & 15u), h = (hf.desc >> 4) & 1u;
            ho.base4 = chunk * 8u + 4u * h;
            const Words w = philox(ho.base4 >> 2, ho.slot, 0u, kDomainFlat, k0, k1);
            half_scores<1>(r, ho.base4, hf.desc & 15u, hf.x, 0.f, 0u, w, thr, ho.sc);
            offer_best(sm, ho.sc);
        }
    }
}

// Halves an evaluation pass could not list (more than kHalfCap): each is scored by
// its chunk's lane (logits read again), one (entry, half) combination at a time,
// with the same offer / barrier / list steps.  Called by every thread.
template <bool BF16>
__device__ __forceinline__ void eval_overflow(const RaceArgs& a, const Row& r, Shared& sm, int first, uint32_t ovf,
                                              uint32_t k0, uint32_t k1) {
    const int tid = threadIdx.x, c = tid & 15, row = tid >> 4;
    const uint32_t V = (uint32_t)a.V;
    // (rare: one copy of the code, not unrolled)
#pragma unroll 1
    for (int q = 0; q < kRowEntries; ++q) {
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            const uint32_t mask = (ovf >> (8 * q + 4 * h)) & 15u;
            float sc[4] = {INFINITY, INFINITY, INFINITY, INFINITY}, xs[4] = {0.f, 0.f, 0.f, 0.f};
            uint32_t base4 = 0u, slot = 0u;
            if (mask != 0u) {
                const Node pn = sm.l2[first + row * kRowEntries + q];
                slot = pn.id >> 20;
                const uint32_t g = pn.id & 0xFFFFFu;
                const uint32_t chunk = g * 16u + (uint32_t)c;
                base4 = chunk * 8u + 4u * (uint32_t)h;
                const Words w = philox(base4 >> 2, slot, 0u, kDomainFlat, k0, k1);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    xs[t] = (mask >> t) & 1u ? load_logit<BF16>(r.ptr, (int)(base4 + (uint32_t)t)) : -INFINITY;
                half_scores<1>(r, base4, mask, xs, 0.f, 0u, w, current_threshold(sm), sc);
                offer_best(sm, sc);
            }
            __syncthreads();
            if (mask != 0u) list_near(sm, a, base4, slot, sc, xs);
            __syncthreads();
        }
    }
}

// Reorder the first n entries of the group list by their bounds (ln of the clock
// floor minus the scaled group maximum), counting-sorted into kBuckets buckets
// between the smallest bound and the threshold; entries above the threshold are
// dropped.  Evaluating the most promising groups first lowers the threshold
// early, and a pass whose first entry's bucket lies above the threshold ends the
// evaluation (later buckets hold larger bounds).  Returns the kept count.  The
// sort stages the list in half[], which is free between evaluation passes.
// Called by every thread.
__device__ __forceinline__ int order_groups(const Row& r, Shared& sm, const float* gm, int n) {
    static_assert(kL2Cap <= 2 * kBlock, "two entries per thread");
    const int tid = threadIdx.x, lane = tid & 63;
    const float thr = current_threshold(sm);
    Node nd[2];
    float b[2];
    float wmin = INFINITY;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + i * kBlock;
        nd[i] = e < n ? sm.l2[e] : Node{0u, 0.f, 0u};
        b[i] = e < n ? kLnClockFloor - scaled(r, gm[nd[i].id & 0xFFFFFu]) : INFINITY;
        if (b[i] <= thr) wmin = fminf(wmin, b[i]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wmin = fminf(wmin, __shfl_xor(wmin, off));
    if (lane == 0) sm.ord_wmin[tid >> 6] = wmin;
    if (tid < kBuckets) {
        sm.ord_hist[tid] = 0;
        sm.ord_bmin[tid] = ordered_key(INFINITY);
    }
    __syncthreads();
    float bmin = sm.ord_wmin[0];
#pragma unroll
    for (int w = 1; w < kBlock / 64; ++w) bmin = fminf(bmin, sm.ord_wmin[w]);
    // bucket = floor((b - bmin) * scale), non-decreasing in b
    const float scale = thr > bmin ? (float)kBuckets / (thr - bmin) : 0.f;
    int k[2], rank[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        k[i] = -1;
        rank[i] = 0;
        if (b[i] <= thr) {
            k[i] = min(kBuckets - 1, (int)((b[i] - bmin) * scale));
            rank[i] = atomicAdd(&sm.ord_hist[k[i]], 1);
            atomicMin(&sm.ord_bmin[k[i]], ordered_key(b[i]));
        }
    }
    __syncthreads();
    // bucket starts: a prefix sum over the kBuckets counts in every wave
    const int h = lane < kBuckets ? sm.ord_hist[lane] : 0;
    int incl = h;
#pragma unroll
    for (int off = 1; off < kBuckets; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    const int excl = incl - h;
    const int kept = __shfl(incl, kBuckets - 1);
    Node* tmp = reinterpret_cast<Node*>(sm.half);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int start = __shfl(excl, max(k[i], 0));
        if (k[i] >= 0) {
            const int dst = start + rank[i];
            tmp[dst] = nd[i];
            if (dst % kPassGroups == 0) sm.ord_pass[dst / kPassGroups] = k[i];
        }
    }
    __syncthreads();
    for (int e = tid; e < kept; e += kBlock) sm.l2[e] = tmp[e];
    __syncthreads();
    return kept;
}

// Evaluate and empty the group list.  Callers read the list count after a barrier
// and before any push of the current pass.
template <bool BF16>
__device__ __forceinline__ void flush_groups(const RaceArgs& a, const Row& r, Shared& sm, const float* gm, uint32_t k0,
                                             uint32_t k1) {
    int n = min(sm.n_l2, kL2Cap);
    const bool ordered = n > kPassGroups;
    if (ordered) n = order_groups(r, sm, gm, n);
    int par = 0;
    Unit<BF16> ux[kRowEntries];
    load_pass<BF16>(a, r, sm, 0, n, ux);
    for (int first = 0; first < n; first += kPassGroups, par ^= 1) {
        // every later entry's bound is at least its bucket's smallest (the threshold
        // and the buckets are read after the previous pass's last barrier)
        if (ordered && first > 0 && ordered_value(sm.ord_bmin[sm.ord_pass[first / kPassGroups]]) > current_threshold(sm))
            break;
        HalfOut ho;
        uint32_t ovf;
        eval_groups<BF16>(a, r, sm, gm, first, min(n - first, kPassGroups), n, par, k0, k1, ho, ovf, ux);
        __syncthreads();
        // every half of the pass has lowered the best: list the near-ties
        if (ho.valid) list_near(sm, a, ho.base4, ho.slot, ho.sc, sm.half[threadIdx.x].x);
        if (sm.n_ev[par] > (uint32_t)kHalfCap) eval_overflow<BF16>(a, r, sm, first, ovf, k0, k1);
        __syncthreads();
        // (the next pass touches the candidates only after two more barriers)
        if (threadIdx.x == 0) compact_candidates(sm);
    }
    if (threadIdx.x == 0) {
        sm.n_l2 = 0;
        sm.n_ev[0] = sm.n_ev[1] = 0u;
    }
    __syncthreads();
}

// ---- tree clocks: descent below level 3 and evaluation of the listed groups.
//
// A race is a chain of short phases in one workgroup, bound by their latency (Philox
// calls, barriers, one trip to memory for the listed groups' logits), so the phases
// are few and wide: level-3 nodes carry the mask of their groups that can still win
// (one pass over the group maxima by the node's own lane), the set bits are the work
// list of the group draws, and up to kEvalGroups listed groups are evaluated at once.
// Whole calls, against passes of 32 groups in the order of their bounds: 114 -> 98 us at
// V = 32000, K = 4, gamma = 5, B = 16 (46 and 68 groups listed per draft and target race,
// 1.3 passes), 103 -> 95 us at V = 128256, K = 4, gamma = 4, B = 64.

// Listed halves of the group entries [first, first + cnt): 16 lanes hold the 16 chunks
// of an entry, each row of 16 lanes takes four entries at a time (their loads in flight
// together).  Only the 4-token halves with a token that can still win are listed; most
// entries list one.  Called by every thread.
template <bool BF16>
__device__ __forceinline__ void list_halves(const RaceArgs& a, const Row& r, Shared& sm, const float* gm, int first,
                                            int cnt, int par) {
    constexpr int U = 4;
    const int tid = threadIdx.x, lane = tid & 63, c = tid & 15, row = tid >> 4;
    const float thr = current_threshold(sm);
    for (int s0 = 0; s0 < cnt; s0 += 16 * U) {
        Unit<BF16> ux[U];
        uint32_t m8[U], hold = 0u;  // surviving tokens; bit q: the chunk holds the group's minimum
        float xc[U];
        uint32_t base[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int le = s0 + q * 16 + row;
            m8[q] = 0u;
            xc[q] = INFINITY;
            base[q] = 0u;
            if (le < cnt) {
                const Node nd = sm.l2[first + le];
                const uint32_t g = nd.id & 0xFFFFFu;
                const float lnm = ln_f32(nd.m);
                base[q] = g * kGroupTokens + (uint32_t)c * 8u;
                if (lnm - scaled(r, gm[g]) <= thr && (int)base[q] < a.V) {
                    // a token can reach thr only if lnm - (x - shift) / T <= thr, i.e.
                    // x - shift >= (lnm - thr) T; the cut is lowered by kCutSlack, far more
                    // than the rounding of either form (compared in the shifted frame)
                    xc[q] = (lnm - thr - kCutSlack) * r.T;
                    if (nd.p >= base[q] && nd.p < base[q] + 8u) hold |= 1u << q;
                    load_words<BF16>(r.ptr, a.V, (int)base[q], ux[q]);
                }
            }
        }
        int nh = 0;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (xc[q] < INFINITY) {
                float x[8];
                unpack_unit<BF16>(ux[q], x);
#pragma unroll
                for (int i = 0; i < 8; ++i) m8[q] |= (uint32_t)(x[i] - r.shift >= xc[q]) << i;
                const int nv = a.V - (int)base[q];  // tokens of this chunk inside the row
                if (nv < 8) m8[q] &= (1u << nv) - 1u;
                nh += (int)((m8[q] & 15u) != 0u) + (int)((m8[q] >> 4) != 0u);
            }
        }
        // list positions: wave prefix sum of the halves, one atomic per wave
        const uint32_t mine = (uint32_t)nh;
        const uint32_t incl = wave_incl_sum(mine);
        const uint32_t wtot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        uint32_t wbase = 0u;
        if (lane == 0 && wtot != 0u) wbase = atomicAdd(&sm.n_ev[par], wtot);
        int jh = (int)((uint32_t)__builtin_amdgcn_readlane((int)wbase, 0) + incl - mine);
        if (nh == 0) continue;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (m8[q] == 0u) continue;
            float x[8];
            unpack_unit<BF16>(ux[q], x);
            const uint32_t desc = ((uint32_t)(s0 + q * 16 + row) << 9) | ((uint32_t)c << 5);
            const int cref = (hold >> q) & 1u ? -1 : 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t hm = h ? m8[q] >> 4 : m8[q] & 15u;
                if (hm == 0u) continue;
                if (jh < kHalfCap) {
                    Half& hf = sm.half[jh];
                    hf.desc = desc | ((uint32_t)h << 4) | hm;
                    hf.cref = cref;
                    hf.x[0] = x[4 * h];
                    hf.x[1] = x[4 * h + 1];
                    hf.x[2] = x[4 * h + 2];
                    hf.x[3] = x[4 * h + 3];
                }
                ++jh;
            }
        }
    }
}

// Score the first nh listed halves (one per thread), lower the best score and list the
// near-ties.  A wave lists its halves after it has offered all of them, so a score is
// listed only if it is within the margin of every earlier one: a few candidates per
// pass (the decision drops those that later scores leave behind).
__device__ __forceinline__ void score_halves(const RaceArgs& a, const Row& r, Shared& sm, int first, int nh, uint32_t k0,
                                             uint32_t k1) {
    const int tid = threadIdx.x;
    if (tid >= nh) return;
    const Half hf = sm.half[tid];
    const Node pn = sm.l2[first + (int)(hf.desc >> 9)];
    const uint32_t slot = pn.id >> 20, g = pn.id & 0xFFFFFu;
    const uint32_t chunk = g * 16u + ((hf.desc >> 5) & 15u), h = (hf.desc >> 4) & 1u;
    const uint32_t base4 = chunk * 8u + 4u * h;
    float mc = pn.m;
    uint32_t pc = pn.p;
    if (hf.cref >= 0) {
        // the chunk's own minimum (its draw is independent of the half's words, so the
        // two Philox calls overlap)
        const uint32_t n = node_end(kShift1, chunk, (uint32_t)a.V) - chunk * 8u;
        const Words wc = philox(chunk, slot, 1u, kDomainTree, k0, k1);
        mc = pn.m + div_n(exp1_f32(wc.w0), n);
        pc = chunk * 8u + uniform_position(wc.w1, wc.w2, n);
    }
    const Words w = philox(chunk, slot, 8u + h, kDomainTree, k0, k1);
    float sc[4];
    half_scores<0>(r, base4, hf.desc & 15u, hf.x, mc, pc, w, current_threshold(sm), sc);
    offer_best(sm, sc);
    list_near(sm, a, base4, slot, sc, hf.x);
}

// Evaluate and empty the group list (called after a barrier that published it; every
// thread calls it, and it ends with a barrier).  par: parity of the half count in use
// (the other one is 0), kept by the race.
template <bool BF16>
__device__ __forceinline__ void eval_list(const RaceArgs& a, const Row& r, Shared& sm, const float* gm, uint32_t k0,
                                          uint32_t k1, int& par) {
    const int n = min(sm.n_l2, kL2Cap);
    if (n == 0) {
        __syncthreads();
        return;
    }
    // A pass that lists more halves than fit scores those that do and lists its entries
    // again: the best score they left usually drops most of the others (a (token, slot)
    // may be scored twice).  If it overflows again the pass is halved, down to eight
    // entries, whose 256 halves always fit.
    int step = kEvalGroups;
    bool again = false;
    for (int first = 0; first < n;) {
        const int cnt = min(n - first, step);
        list_halves<BF16>(a, r, sm, gm, first, cnt, par);
        // (between the barriers after the last candidate was listed and before the next is;
        // thread 0 alone reads the count, so no other's path depends on it)
        if (threadIdx.x == 0) compact_candidates(sm);
        __syncthreads();
        const int nh = (int)sm.n_ev[par];
        if (threadIdx.x == 0) {
            sm.n_ev[par ^ 1] = 0u;  // (last read before the previous barrier)
            sm.n_l2 = 0;            // (read by every thread at entry)
        }
        par ^= 1;
        score_halves(a, r, sm, first, min(nh, kHalfCap), k0, k1);
        if (nh <= kHalfCap) {
            first += cnt;
            step = kEvalGroups;
            again = false;
        } else {
            if (again) step = max(8, cnt >> 1);
            again = true;
        }
        __syncthreads();
    }
}

// Draw the groups of the listed level-3 nodes, list those that can still win and
// evaluate them (called after a barrier that published the list; every thread calls
// it, and it ends with a barrier).
template <bool BF16>
__device__ __forceinline__ void expand_l3(const RaceArgs& a, const Row& r, Shared& sm, const float* gm, uint32_t k0,
                                          uint32_t k1, int& par) {
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t V = (uint32_t)a.V;
    const int nl3 = (int)(sm.n_l3 & 0xFFFFu), nw = (int)(sm.n_l3 >> 16);
    const bool compact = nw <= kWorkCap;  // else every group of the listed nodes, by its mask bit
    const int tot = compact ? nw : nl3 * 16;
    if (tot == 0) {
        __syncthreads();
        return;
    }
    for (int wb = 0; wb < tot;) {
        const int i = wb + tid;
        bool pass = false;
        Node gn = Node{0u, 0.f, 0u};
        if (i < tot) {
            const int e = compact ? (int)sm.work[i] : i;
            const Node pa = sm.l3[e >> 4];
            const uint32_t g = (pa.id & 0xFFFFFu) * 16u + (uint32_t)(e & 15);
            if (compact || ((sm.l3_mask[e >> 4] >> (e & 15)) & 1u)) {
                const uint32_t slot = pa.id >> 20;
                child_min_f32(pa.m, pa.p, 2, g, g << kShift2, node_end(kShift2, g, V), slot, k0, k1, gn.m, gn.p);
                gn.id = (slot << 20) | g;
                pass = ln_f32(gn.m) - scaled(r, gm[g]) <= current_threshold(sm);
            }
        }
        const uint64_t bal = __ballot(pass);
        int at = 0;
        if (lane == 0 && bal != 0u) at = atomicAdd(&sm.n_l2, (int)__builtin_popcountll(bal));
        at = __builtin_amdgcn_readlane(at, 0) +
             (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        if (pass) sm.l2[at] = gn;  // (at most kBlock are listed between two checks of the count)
        __syncthreads();
        if (tid == 0) sm.n_l3 = 0u;  // (read by every thread at entry)
        wb += kBlock;
        if (wb >= tot || sm.n_l2 > kL2Cap - kBlock)
            eval_list<BF16>(a, r, sm, gm, k0, k1, par);
        else
            __syncthreads();
    }
}

// Lexicographic minimum of (score, token, slot).
__device__ __forceinline__ bool lex_less(double s, int v, int j, double s2, int v2, int j2) {
    return s < s2 || (s == s2 && (v < v2 || (v == v2 && j < j2)));
}

__device__ __forceinline__ int path_shift(int l) {
    return l == 1 ? kShift4 : l == 2 ? kShift3 : l == 3 ? kShift2 : kShift1;
}

// Counter words (c0, c2) of path node l of token v (tree clocks): 0 = root, 1..4 =
// the token's level-4..1 ancestors, 5 = the token's own word block.  The counter
// is selected per lane, so lanes of one token draw their nodes in a single call.
__device__ __forceinline__ uint32_t path_c0(int l, uint32_t v) { return l == 0 ? 0u : l == 5 ? v >> 3 : v >> path_shift(l); }
__device__ __forceinline__ uint32_t path_c2(int l, uint32_t v) {
    return l == 0 ? 5u : l == 5 ? 8u + ((v >> 2) & 1u) : (uint32_t)(5 - l);
}
__device__ __forceinline__ Words path_draw(int l, uint32_t v, uint32_t slot, uint32_t k0, uint32_t k1) {
    return philox(path_c0(l, v), slot, path_c2(l, v), kDomainTree, k0, k1);
}

__device__ __forceinline__ uint32_t pick_word(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t i) {
    return i == 0 ? a0 : i == 1 ? a1 : i == 2 ? a2 : a3;
}

// What lane e of pass A draws, all of it known before the context key: the counter and
// slot, the node's size (and its reciprocal) and first token, and the seed it belongs to.
// A row whose key is still on its way works it out meanwhile: 43.3 -> 42.3 us per block at
// V = 1024, K = 2, gamma = 4, B = 1, 97.6 -> 95.2 at V = 32000, K = 4, gamma = 5, B = 16 (two
// builds in turn; that block takes 94 to 104 us from one process to another),
// equal (93.6) at V = 128256, K = 4, gamma = 4, B = 64, whose rows mostly find the key there.
// (With a plan for lanes that draw nothing, the streamers lose the issue slots: 94.0.)
struct SeedPlan {
    uint32_t c0, c2, slot, n, cs, av;  // counter words, slot, node tokens, first token, seed token
    float rn, xs;                      // 1 / n, scaled seed logit
    int j, i4;                         // slot index; level-4 node of lanes 6 and 7 (-1: none)
    bool seed;                         // the seed exists
};
__device__ __forceinline__ SeedPlan seed_plan(const RaceArgs& a, const Row& r, const Shared& sm, const float* gm, int e) {
    const uint32_t V = (uint32_t)a.V;
    const int n4 = (int)((V + (1u << kShift4) - 1) >> kShift4);
    const int pair = e >> 3, l = e & 7;
    static_assert(kInit == 8, "seed index = low 3 bits of the 8-lane group index");
    const int w = pair & 7;  // seed w, slot j
    SeedPlan p;
    p.j = pair >> 3;
    const int tv = sm.seed_tok[w];
    p.seed = tv >= 0;
    p.slot = (uint32_t)(r.slot0 + p.j);
    p.av = (uint32_t)max(tv, 0);
    p.xs = tv >= 0 ? scaled(r, gm[tv >> 7]) : -INFINITY;
    const uint32_t i4 = (uint32_t)(2 * w + (l - 6));
    const bool l4 = l >= 6 && (int)i4 < n4;
    p.i4 = l4 ? (int)i4 : -1;
    p.c0 = l4 ? i4 : path_c0(l, p.av);
    p.c2 = l4 ? 4u : path_c2(l, p.av);
    const int sh = l4 ? kShift4 : path_shift(l);
    const uint32_t node = l4 ? i4 : p.av >> sh;
    p.cs = (l == 0 || l == 5) ? 0u : node << sh;
    p.n = l == 0 ? V : l == 5 ? 1u : node_end(sh, node, V) - p.cs;
    p.rn = __builtin_amdgcn_rcpf((float)p.n);
    return p;
}

template <bool BF16, int LAYOUT>
__device__ __forceinline__ void race(const RaceArgs& a, const Row& r, Shared& sm, const float* gm, uint32_t k0, uint32_t k1,
                                     SeedPlan pl) {
    // (lists, candidates and the best score were reset by the caller)
    const int tid = threadIdx.x;
    const uint32_t V = (uint32_t)a.V;
    const int ng = a.L.ng;
    const int ns = r.nslots;
    const int n4 = (int)((V + (1u << kShift4) - 1) >> kShift4);
    // Pass A: the seed tokens (each the largest logit of its group) in every slot --
    // tree clocks: 8 lanes per (token, slot), lane l < 6 drawing path node l -- and,
    // for tree clocks, the minimum of every (slot, level-4 node): lanes 6 and 7 of the
    // seed lanes of slot j take its level-4 nodes (with the root drawn by lane 0).
    static_assert((1 << (kShift5 - kShift4)) <= 2 * kInit, "two lanes per seed hold every level-4 node");
    const int seed_lanes = kInit * ns * 8;
    for (int e0 = 0; e0 < seed_lanes; e0 += kBlock) {
        const int e = e0 + tid;
        if (e < seed_lanes) {  // whole 8-lane groups: the shuffles stay within active lanes
            const int l = e & 7;
            if (e0 > 0) pl = seed_plan(a, r, sm, gm, e);
            const uint32_t slot = pl.slot, av = pl.av;
            const int j = pl.j;
            if constexpr (LAYOUT == 0) {
                // lane l turns node l's draw into (minimum increment, position): root
                // E'/V, level-4..1 node E'/size at a uniform position in it, token E'
                const uint32_t i4 = (uint32_t)pl.i4;
                const bool l4 = pl.i4 >= 0;
                float val = 0.f;
                uint32_t pos = 0u;
                if (l < 6 || l4) {
                    const Words wd = philox(pl.c0, slot, pl.c2, kDomainTree, k0, k1);
                    val = exp1_f32(l == 5 ? pick_word(wd.w0, wd.w1, wd.w2, wd.w3, av & 3u) : wd.w0) * pl.rn;
                    pos = pl.cs + uniform_position(wd.w1, wd.w2, pl.n);
                }
                const int base = tid & ~7;
                float m = __shfl(val, base);
                uint32_t p = (uint32_t)__shfl((int)pos, base);
                if (l4) {
                    // the root (lane 0) or this node holds the level-4 node's minimum
                    const uint32_t cs = i4 << kShift4, ce = node_end(kShift4, i4, V);
                    const bool hold = p >= cs && p < ce;
                    level4_list(gm, ng)[j * n4 + (int)i4] =
                        Node{(slot << 20) | i4, hold ? m : m + val, hold ? p : pos};
                }
#pragma unroll
                for (int q = 1; q <= 4; ++q) {
                    const float vq = __shfl(val, base + q);
                    const uint32_t pq = (uint32_t)__shfl((int)pos, base + q);
                    const int sh = path_shift(q);
                    const uint32_t i = av >> sh, cs = i << sh, ce = node_end(sh, i, V);
                    if (!(p >= cs && p < ce)) {
                        m = m + vq;
                        p = pq;
                    }
                }
                const float v5 = __shfl(val, base + 5);
                const float E = (av == p) ? m : m + v5;
                if (l == 0 && pl.seed) {
                    const float sc = ln_f32(E) - pl.xs;
                    const float xa = gm[av >> 7];
                    if (sc < INFINITY) {
                        // (listed only if within the margin of the best so far)
                        atomicMin(&sm.best_key, ordered_key(sc));
                        if (sc <= current_threshold(sm)) push_candidate(sm, a, (int)av, (int)slot, sc, xa);
                    }
                }
            } else {
                if (l == 0 && pl.seed) {
                    const float xa = gm[av >> 7];
                    const Words wd = philox(av >> 2, slot, 0u, kDomainFlat, k0, k1);
                    const float sc = ln_f32(exp1_f32(word_at(wd, av & 3u))) - scaled(r, xa);
                    if (sc < INFINITY) {
                        atomicMin(&sm.best_key, ordered_key(sc));
                        push_candidate(sm, a, (int)av, (int)slot, sc, xa);
                    }
                }
            }
        }
    }
    __syncthreads();

    if constexpr (LAYOUT == 0) {
        // Pass B: level-3 children of the level-4 nodes that can still win, each with the
        // mask of its groups that can (the node's minimum bounds theirs).
        const int lane = tid & 63;
        int par = 0;
        const int nB = ns * n4 * 16;
        const int n3 = (ng + 15) / 16;
        for (int base = 0; base < nB;) {
            const int e = base + tid;
            uint32_t mask = 0u;
            Node nd = Node{0u, 0.f, 0u};
            if (e < nB) {
                const Node pa = level4_list(gm, ng)[e >> 4];
                const uint32_t i4 = pa.id & 0xFFFFFu;
                const uint32_t i3 = i4 * 16u + (uint32_t)(e & 15);
                const float thr = current_threshold(sm);
                if ((int)i3 < n3 && ln_f32(pa.m) - scaled(r, sm.m3[i3]) <= thr) {
                    const uint32_t slot = pa.id >> 20;
                    child_min_f32(pa.m, pa.p, 3, i3, i3 << kShift3, node_end(kShift3, i3, V), slot, k0, k1, nd.m, nd.p);
                    nd.id = (slot << 20) | i3;
                    const float xc = (ln_f32(nd.m) - thr - kCutSlack) * r.T;
                    const float4* g4 = (const float4*)(gm + i3 * 16u);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 x = g4[q];
                        mask |= ((uint32_t)(x.x - r.shift >= xc) | ((uint32_t)(x.y - r.shift >= xc) << 1) |
                                 ((uint32_t)(x.z - r.shift >= xc) << 2) | ((uint32_t)(x.w - r.shift >= xc) << 3))
                                << (4 * q);
                    }
                }
            }
            // list positions of the node (low half) and of its group bits (high half)
            const uint32_t mine = mask ? ((uint32_t)__popc(mask) << 16) | 1u : 0u;
            const uint32_t incl = wave_incl_sum(mine);
            const uint32_t wtot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            uint32_t at = 0u;
            if (lane == 0 && wtot != 0u) at = atomicAdd(&sm.n_l3, wtot);
            at = (uint32_t)__builtin_amdgcn_readlane((int)at, 0) + incl - mine;
            if (mask) {
                const uint32_t i = at & 0xFFFFu;
                uint32_t w = at >> 16;
                sm.l3[i] = nd;
                sm.l3_mask[i] = (uint16_t)mask;
                for (; mask; mask &= mask - 1u, ++w)
                    if (w < (uint32_t)kWorkCap) sm.work[w] = (uint16_t)(i * 16u + (uint32_t)__builtin_ctz(mask));
            }
            __syncthreads();
            base += kBlock;
            if (base >= nB || (sm.n_l3 & 0xFFFFu) > (uint32_t)(kL3Cap - kBlock))
                expand_l3<BF16>(a, r, sm, gm, k0, k1, par);
            else
                __syncthreads();
        }
    } else {
        // flat clocks: every (group, slot) whose floor bound can win.
        const int tot = ng * ns;
        for (int base = 0;; base += kBlock) {
            const bool done = base >= tot;  // one call site of flush_groups
            const bool flush = done || sm.n_l2 > kL2Cap - kBlock;
            __syncthreads();
            if (flush) flush_groups<BF16>(a, r, sm, gm, k0, k1);
            if (done) break;
            const int e = base + tid;
            if (e < tot) {
                const int g = e / ns;
                const uint32_t slot = (uint32_t)(r.slot0 + e % ns);
                if (kLnClockFloor - scaled(r, gm[g]) <= current_threshold(sm))
                    push_node(sm.l2, &sm.n_l2, kL2Cap, (slot << 20) | (uint32_t)g, 0.f, 0u);
            }
            __syncthreads();
        }
    }

    // decide: float64 scores of the candidates within the margin of the best; for
    // tree clocks 8 lanes per candidate draw its path nodes in parallel.
    const float best = ordered_value(sm.best_key);
    const int nc = min(sm.n_cand, kCandCap);
    if (nc <= 64) {
        // Every wave looks the candidates over by itself (no barrier): one (token, slot)
        // within the margin of the best, possibly listed twice, is the winner, as below.
        const int l = tid & 63;
        const bool in = l < nc && sm.cand_s[l] <= best + kMargin;
        const uint64_t bal = __ballot(in);
        if (bal != 0u) {
            const int key = l < nc ? sm.cand_v[l] * 32 + sm.cand_j[l] : 0;  // token < 2^19, slot < 32
            const int k = __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(bal));
            if (__ballot(in && key != k) == 0u) {
                if (tid == 0) {
                    sm.win_token = k >> 5;
                    sm.win_slot = k & 31;
                }
                return;
            }
        }
    } else {
        // A single candidate within the margin of the best is the winner: float32
        // scores err by far less than the margin, and every token that was not kept
        // scored above it.
        static_assert(kCandCap <= kBlock, "one candidate per thread");
        const bool in = tid < nc && sm.cand_s[tid] <= best + kMargin;
        if (in) {
            const int key = sm.cand_v[tid] * 32 + sm.cand_j[tid];  // token < 2^19, slot < 32
            atomicMin(&sm.key_min, key);
            atomicMax(&sm.key_max, key);
            sm.win_token = sm.cand_v[tid];
            sm.win_slot = sm.cand_j[tid];
        }
        __syncthreads();
        if (sm.key_min == sm.key_max) return;  // one (token, slot), possibly listed twice
        __syncthreads();
    }
    double bs = INFINITY;
    int bv = 0x7FFFFFFF, bj = 0x7FFFFFFF;
    for (int e0 = 0; e0 < nc * 8; e0 += kBlock) {
        const int e = e0 + tid;
        const int ci = e >> 3, l = e & 7;
        const bool valid = ci < nc && sm.cand_s[ci] <= best + kMargin;
        const int v = valid ? sm.cand_v[ci] : 0, j = valid ? sm.cand_j[ci] : 0;
        double E = 0.0;
        if constexpr (LAYOUT == 0) {
            Words wd = Words{0u, 0u, 0u, 0u};
            if (valid && l < 6) wd = path_draw(l, (uint32_t)v, (uint32_t)j, k0, k1);
            double m = 0.0;
            uint32_t p = 0u;
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                const int src = (tid & ~7) + q;
                const uint32_t a0 = (uint32_t)__shfl((int)wd.w0, src);
                const uint32_t a1 = (uint32_t)__shfl((int)wd.w1, src);
                const uint32_t a2 = (uint32_t)__shfl((int)wd.w2, src);
                const uint32_t a3 = (uint32_t)__shfl((int)wd.w3, src);
                if (l != 0 || !valid) continue;
                if (q == 0) {
                    m = exp1_f64(a0) / (double)V;
                    p = uniform_position(a1, a2, V);
                } else if (q <= 4) {
                    const int sh = path_shift(q);
                    const uint32_t i = (uint32_t)v >> sh, cs = i << sh, ce = node_end(sh, i, V);
                    if (!(p >= cs && p < ce)) {
                        m = m + exp1_f64(a0) / (double)(ce - cs);
                        p = cs + uniform_position(a1, a2, ce - cs);
                    }
                } else {
                    E = ((uint32_t)v == p) ? m : m + exp1_f64(pick_word(a0, a1, a2, a3, (uint32_t)v & 3u));
                }
            }
        } else {
            if (l == 0 && valid) E = flat_clock_f64((uint32_t)j, (uint32_t)v, k0, k1);
        }
        if (l == 0 && valid) {
            const double s = log(E) - (double)sm.cand_x[ci] / (double)r.T;
            if (lex_less(s, v, j, bs, bv, bj)) {
                bs = s;
                bv = v;
                bj = j;
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double os = __shfl_xor(bs, off);
        const int ov = __shfl_xor(bv, off), oj = __shfl_xor(bj, off);
        if (lex_less(os, ov, oj, bs, bv, bj)) {
            bs = os;
            bv = ov;
            bj = oj;
        }
    }
    if ((tid & 63) == 0) {
        sm.red_s[tid >> 6] = bs;
        sm.red_v[tid >> 6] = bv;
        sm.red_j[tid >> 6] = bj;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kBlock / 64; ++w)
            if (lex_less(sm.red_s[w], sm.red_v[w], sm.red_j[w], bs, bv, bj)) {
                bs = sm.red_s[w];
                bv = sm.red_v[w];
                bj = sm.red_j[w];
            }
        sm.win_token = (bs < INFINITY) ? bv : -1;
        sm.win_slot = (bs < INFINITY) ? bj : -1;
    }
    __syncthreads();
}

// ---------------------------------------------------------------- walk

__device__ __forceinline__ int walk_draft(const RaceArgs& a, int b, int k, int s, uint32_t ep) {
    if (a.s_count > 0 && s >= a.s_begin) return wait_token(a, draft_row_id(a, b, k, s), ep);
    return a.draft_tokens[((size_t)b * a.K + k) * a.gamma + s];
}

// Realised-path walk of sequence b; every token it reads carries this call's epoch.
// Called by every thread: the tokens the walk may read are fetched in parallel
// first (into the candidate arrays, free once the race is decided); thread 0 walks.
__device__ __forceinline__ void walk(const RaceArgs& a, Shared& sm, int b, uint32_t ep) {
    const int K = a.K, G = a.gamma, tid = threadIdx.x;
    const int ntp = a.target_rows == 1 ? 1 : K;
    const int nt = ntp * (G + 1), n = nt + K * G;
    const bool staged = n <= kCandCap;
    if (staged) {
        for (int e = tid; e < n; e += kBlock)
            sm.cand_v[e] = e < nt ? wait_token(a, target_row_id(a, b, e / (G + 1), e % (G + 1)), ep)
                                  : walk_draft(a, b, (e - nt) / G, (e - nt) % G, ep);
        __syncthreads();
    }
    if (tid != 0) return;
    auto target = [&](int k, int s) {
        return staged ? sm.cand_v[(ntp == 1 ? 0 : k) * (G + 1) + s] : wait_token(a, target_row_id(a, b, k, s), ep);
    };
    auto draft = [&](int k, int s) { return staged ? sm.cand_v[nt + k * G + s] : walk_draft(a, b, k, s, ep); };
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
            if (((act >> k) & 1u) && draft(k, s) == y) na |= 1u << k;
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

// ---------------------------------------------------------------- row finisher

// Token at path depth d of this row's context (prefix excluded).
__device__ __forceinline__ int path_token(const RaceArgs& a, const Row& r, int d, uint32_t ep) {
    if (r.kind == 1 && a.target_rows == 1) return wait_token(a, target_row_id(a, r.b, 0, d), ep);
    if (a.s_count > 0 && d >= a.s_begin) return wait_token(a, draft_row_id(a, r.b, r.k, d), ep);
    return a.draft_tokens[((size_t)r.b * a.K + r.k) * a.gamma + d];
}

// Row whose race publishes this row's context key (-1: the key is folded here, all
// its tokens being known before the call).  The key of depth s of a path is
// finished by the race at depth s - 1, which alone knows the newest token.
__device__ __forceinline__ int key_producer(const RaceArgs& a, const Row& r) {
    if (a.m == 0 || r.s == 0) return -1;
    if (r.kind == 1 && a.target_rows == 1) return target_row_id(a, r.b, 0, r.s - 1);
    if (a.s_count > 0 && r.s - 1 >= a.s_begin && r.s - 1 < a.s_begin + a.s_count)
        return draft_row_id(a, r.b, r.k, r.s - 1);
    return -1;
}

// Whether this row's race publishes the context key of the next depth of its path.
__device__ __forceinline__ bool key_consumer(const RaceArgs& a, const Row& r) {
    if (a.m == 0) return false;
    if (r.kind == 1) return a.target_rows == 1 && r.s + 1 <= a.gamma;
    return r.s + 1 < a.s_begin + a.s_count || (a.target_rows > 1 && r.s + 1 <= a.gamma);
}

template <bool BF16, int LAYOUT>
__device__ __forceinline__ void finish_row(const RaceArgs& a, const Row& r, Shared& sm, float* gm) {
    // The race is a latency chain (the next depth of this path waits for it) while
    // the other waves on the same SIMDs stream: raise this wave's issue priority,
    // the most for target rows, whose chain is one race longer than a draft path's
    // and ends the launch (102.4 vs 101.7 µs at V = 128256, K = 4, B = 64 against
    // one shared priority; drafts at the streamers' priority: 104 µs).
    if (r.kind == 1)
        __builtin_amdgcn_s_setprio(3);
    else
        __builtin_amdgcn_s_setprio(1);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ng = a.L.ng;
    const int n3 = (ng + 15) / 16;
    const uint32_t ep = sm.epoch;
    const float c2 = r.invT * 1.4426950408889634f;

    // Context-key inputs known before the call (prompt tokens, position) are loaded
    // first, so their latency overlaps the gather.  Wave 3 lanes [0, m) take this
    // row's own window (when no race of this call publishes its key), lanes
    // [m, 2m - 1) the next depth's window without its newest token (when this race
    // publishes the next key); positions index prefix (m tokens) || path.
    const int prod = key_producer(a, r);
    const bool cons = key_consumer(a, r);
    int widx = -1, wtok = 0;
    int64_t wpos = 0;
    if (wave == 3) {
        if (lane < a.m && prod < 0)
            widx = r.s + lane;
        else if (lane >= a.m && lane < 2 * a.m - 1 && cons)
            widx = r.s + 1 + (lane - a.m);
        if (widx >= 0 && widx < a.m) wtok = a.prefix[(size_t)r.b * a.m + widx];
        wpos = a.start_pos[r.b];
    }

    // ---- gather the row's slots (group maxima, block maxima, segment sums):
    // a batch of loads in flight per thread, then a wait only for slots not yet
    // published.
    {
        const uint64_t* gslot = (const uint64_t*)(a.ws + a.L.gmax) + (size_t)r.row_id * ng;
        const uint64_t* m3slot = (const uint64_t*)(a.ws + a.L.m3) + (size_t)r.row_id * n3;
        const uint64_t* pslot = (const uint64_t*)(a.ws + a.L.part) + (size_t)r.row_id * a.L.nseg;
        const int ne = ng + n3 + a.L.nseg;
        if (tid < padded_groups(ng) - ng) gm[ng + tid] = -INFINITY;
        for (int e0 = 0; e0 < ne; e0 += 4 * kBlock) {
            const uint64_t* src[4];
            uint64_t v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = e0 + i * kBlock + tid;
                src[i] = e < ng          ? gslot + e
                         : e < ng + n3     ? m3slot + (e - ng)
                                           : pslot + min(e - ng - n3, a.L.nseg - 1);
                v[i] = e < ne ? ld_dev(src[i]) : 0;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = e0 + i * kBlock + tid;
                if (e < ne) {
                    if ((uint32_t)(v[i] >> 32) != ep) v[i] = wait_slot(a, src[i], ep);
                    const uint32_t w = (uint32_t)v[i];
                    if (e < ng)
                        gm[e] = __uint_as_float(w);
                    else if (e < ng + n3)
                        sm.m3[e - ng] = __uint_as_float(w);
                    else
                        sm.part[e - ng - n3] = __uint_as_float(w);
                }
            }
        }
    }
    __syncthreads();

    // ---- key-independent work: the race's seed tokens, LSE, row maximum.  Seed groups: the largest group of each eighth of the row (lowest index
    // on ties; -1 where the eighth has no finite logit), 32 lanes per eighth.  A row of
    // any size gets up to 8 seeds this way: with one seed per 32 KiB segment a
    // 32000-token bf16 row had two, and its 4-slot races listed 111 (slot, group)
    // pairs on average instead of 88 (46 against the final best score).
    {
        static_assert(kInit * 32 == kBlock, "32 lanes per seed group");
        const int i = tid >> 5, l32 = lane & 31;
        const int g0 = i * ng / kInit, g1 = (i + 1) * ng / kInit;
        float bv = -INFINITY;
        int bg = 0x7FFFFFFF;
        for (int g = g0 + l32; g < g1; g += 32)
            if (gm[g] > bv) {
                bv = gm[g];
                bg = g;
            }
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) {
            const float ov = __shfl_xor(bv, off);
            const int og = __shfl_xor(bg, off);
            if (ov > bv || (ov == bv && og < bg)) {
                bv = ov;
                bg = og;
            }
        }
        if (l32 == 0) sm.init_v[i] = bv == -INFINITY ? -1 : bg;
    }
    __syncthreads();
    // Waves 0-1: the seed tokens, 16 lanes per seed group with 8 tokens each (the
    // group's lowest token holding its maximum); wave 2: LSE, row maximum; wave 3: the
    // context keys.  The four run side by side.
    if (wave < 2) {
        static_assert(kInit * 16 == 128, "one 16-lane row per seed group in waves 0-1");
        const int i = tid >> 4, sub = tid & 15;
        const int g = sm.init_v[i];
        int tk = 0x7FFFFFFF;
        if (g >= 0) {
            float x[8];
            const int base = g * kGroupTokens + sub * 8;
            load8<BF16>(r.ptr, a.V, base, x);
            const float gmax = gm[g];
#pragma unroll
            for (int t = 7; t >= 0; --t)
                if (base + t < a.V && x[t] == gmax) tk = base + t;
        }
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) tk = min(tk, __shfl_xor(tk, off));
        if (sub == 0) sm.seed_tok[i] = g >= 0 && tk != 0x7FFFFFFF ? tk : -1;
    } else if (wave == 2) {
        // LSE: segment i's maximum is the maximum of its groups (the same float product
        // the segment used), merged with the segments' sums in float32.
        constexpr int per = (BF16 ? kSegTokensBf16 : kSegTokensF32) / 2048;  // level-3 blocks per segment
        float mi = -INFINITY, si = 0.f;
        if (lane < a.L.nseg) {
            float gmx = -INFINITY;
            for (int t = lane * per; t < min(n3, lane * per + per); ++t) gmx = fmaxf(gmx, sm.m3[t]);
            mi = gmx * c2;
            si = sm.part[lane];
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const float om = __shfl_xor(mi, off);
            const float os = __shfl_xor(si, off);
            lse_combine(mi, si, om, os);
        }
        // row maximum over the level-3 maxima
        float rm = -INFINITY;
        for (int t = lane; t < n3; t += 64) rm = fmaxf(rm, sm.m3[t]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) rm = fmaxf(rm, __shfl_xor(rm, off));
        float lse = mi == -INFINITY ? -INFINITY : (mi + __builtin_amdgcn_logf(si)) * 0.69314718055994531f;
        if (far_row(rm, c2) && (r.kind == 0 ? a.draft_lse : a.target_lse)) lse = far_row_lse<BF16>(r.ptr, a.V, r.invT, rm);
        if (lane == 0) {
            if (r.kind == 0) {
                if (a.draft_lse) a.draft_lse[((size_t)r.b * a.K + r.k) * a.gamma + r.s] = lse;
            } else if (a.target_lse) {
                const size_t o = a.target_rows == 1 ? (size_t)r.b * (a.gamma + 1) + r.s
                                                    : ((size_t)r.b * a.K + r.k) * (a.gamma + 1) + r.s;
                a.target_lse[o] = lse;
            }
            sm.rowmax = rm;
            sm.n_l3 = 0u;
            sm.n_l2 = sm.n_cand = 0;
            sm.n_ev[0] = sm.n_ev[1] = 0;
            sm.best_key = ordered_key(INFINITY);
            sm.key_min = 0x7FFFFFFF;
            sm.key_max = -1;
            // (thread 0 reads these with one LDS trip after the race, instead of fetching
            // the arguments they are made of then)
            sm.pub_key = cons ? (uint64_t*)(a.ws + a.L.keys) + 2 * (size_t)r.row_id : nullptr;
            sm.pub_tok = (uint64_t*)(a.ws + a.L.tok) + r.row_id;
            const size_t o = r.kind == 0 || a.target_rows > 1
                                 ? ((size_t)r.b * a.K + r.k) * (size_t)(a.gamma + (r.kind == 1)) + r.s
                                 : (size_t)r.b * (a.gamma + 1) + r.s;
            int32_t* outs = r.kind == 0 ? a.draft_tokens : a.target_tokens;
            sm.pub_out = outs ? outs + o : nullptr;
        }
    } else {
        // Context keys: the window's path tokens (published by earlier races of this
        // call, or inputs), both chains folded at once -- lane 0 this row's key (when no
        // race publishes it), lane 1 the next depth's key up to its newest known token.
        // A row whose key comes from the race one depth up the path then waits for it;
        // that race's winner comes with it and is folded after this row's race, so that
        // neither a wait nor a fold stands between the key and the race (from a winner
        // to the next race's start: 0.6 us, 1.9 with the winner waited for and folded here).
        const int nk = a.m - (prod >= 0 && a.m > 1 ? 2 : 1);  // lane 1's tokens
        const bool known = widx >= 0 && (lane < a.m || lane - a.m < nk);
        const int tk = known && widx >= a.m ? path_token(a, r, widx - a.m, ep) : wtok;
        const uint64_t t = (uint64_t)(wpos + r.s) + (uint64_t)(lane == 1);
        uint32_t c0 = (uint32_t)a.key, c1 = (uint32_t)(a.key >> 32);
        const bool chain = (lane == 0 && prod < 0) || (lane == 1 && cons);
        if (chain) fold(c0, c1, (uint32_t)t, (uint32_t)(t >> 32), 0u);
        for (int i = 0; i < a.m; ++i) {
            const int w = __shfl(tk, lane == 0 ? i : a.m + i);
            if (chain && (lane == 0 || i < nk)) fold(c0, c1, (uint32_t)w, (uint32_t)i, 1u);
        }
        if (lane == 0 && prod < 0) {
            sm.kappa0 = c0;
            sm.kappa1 = c1;
        }
        if (lane == 1 && cons) {
            sm.next0 = c0;
            sm.next1 = c1;
        }
        bool have = true;
        if (prod >= 0) {
            uint32_t w;
            have = wait_key(a, prod, ep, cons && a.m > 1, true, w);
            if (lane == 0) sm.kappa0 = w;
            if (lane == 1) sm.kappa1 = w;
            if (lane == 2) sm.newest = (int)w;
        }
        if (lane == 0) sm.have_key = have;
    }
    __syncthreads();
    // what pass A draws, worked out while the key is on its way
    Row rs = r;
    rs.shift = sm.rowmax;
    SeedPlan plan;
    if (tid < kInit * 8 * rs.nslots) plan = seed_plan(a, rs, sm, gm, tid);
    if (!sm.have_key) {  // (uniform; written before the barrier above)
        if (wave == 3) {
            uint32_t w;
            wait_key(a, prod, ep, cons && a.m > 1, false, w);
            if (lane == 0) sm.kappa0 = w;
            if (lane == 1) sm.kappa1 = w;
            if (lane == 2) sm.newest = (int)w;
        }
        __syncthreads();
    }
    const uint32_t k0 = sm.kappa0, k1 = sm.kappa1;
    if (sm.rowmax == -INFINITY) {
        if (tid == 0) {
            sm.win_token = -1;
            sm.win_slot = -1;
        }
        __syncthreads();
    } else {
        race<BF16, LAYOUT>(a, rs, sm, gm, k0, k1, plan);
    }
    if (tid == 0) {
        const int y = sm.win_token;
        if (uint64_t* ks = sm.pub_key) {
            uint32_t n0 = sm.next0, n1 = sm.next1;
            if (prod >= 0 && a.m > 1) fold(n0, n1, (uint32_t)sm.newest, (uint32_t)(a.m - 2), 1u);
            fold(n0, n1, (uint32_t)y, (uint32_t)(a.m - 1), 1u);
            st_dev(ks, ((uint64_t)ep << 32) | n0);
            st_dev(ks + 1, ((uint64_t)ep << 32) | n1);
        }
        st_dev(sm.pub_tok, ((uint64_t)ep << 32) | (uint32_t)y);
        if (int32_t* out = sm.pub_out) *out = y;
    }
    // The last row of a sequence in the work order walks its block.
    if (r.kind == a.walk_kind && r.s == a.walk_s && r.k == a.walk_k) {
        __syncthreads();  // (the walk reuses the candidate arrays: every wave is done with them)
        walk(a, sm, r.b, ep);
    }
    __builtin_amdgcn_s_setprio(0);
}

// ---------------------------------------------------------------- kernel

// Row and segment of a work item (phases of rows, each at one depth: its draft
// rows, then its target rows, each row segment by segment).
template <bool BF16>
__device__ __forceinline__ void decode_item(const RaceArgs& a, const Shared& sm, int item, Row& r, int& seg) {
    const size_t esize = BF16 ? 2 : 4;
    const int D = a.B * a.K * a.gamma;
    // the phase holding the item: the number of later phase starts at or below it
    // (phases start in increasing order; phase 0 starts at 0)
    static_assert(kMaxPhases <= 2 * 64, "phase starts fit two lanes per wave");
    const int lane = threadIdx.x & 63;
    const bool s0 = lane + 1 < a.n_phase && sm.ph_first[lane + 1] <= item;
    const bool s1 = lane + 65 < a.n_phase && sm.ph_first[lane + 65] <= item;
    const int ph = (int)__builtin_popcountll(__ballot(s0)) + (int)__builtin_popcountll(__ballot(s1));
    // (the item is uniform: the table entries are made scalar, so the divisions
    // below run on the scalar unit rather than on every lane)
    const int local = __builtin_amdgcn_readfirstlane(item) - __builtin_amdgcn_readfirstlane(sm.ph_first[ph]);
    const int rl = local / a.L.nseg;
    seg = local % a.L.nseg;
    const int d = __builtin_amdgcn_readfirstlane(sm.ph_depth[ph]);
    const int nd = __builtin_amdgcn_readfirstlane(sm.ph_nd[ph]);
    r.s = d;
    r.shift = 0.f;
    if (rl < nd) {
        r.kind = 0;
        r.b = rl / a.K;
        r.k = rl % a.K;
        r.row_id = (r.b * a.K + r.k) * a.gamma + d;
        r.ptr = (const unsigned char*)a.draft_logits +
                (((size_t)r.b * a.K + r.k) * a.s_count + (size_t)(d - a.s_begin)) * (size_t)a.V * esize;
        r.slot0 = r.k;
        r.nslots = 1;
        r.invT = a.inv_T_draft;
        r.T = a.T_draft;
    } else {
        const int rt = rl - nd;
        r.kind = 1;
        size_t off;
        if (a.target_rows == 1) {
            r.b = rt;
            r.k = 0;
            r.row_id = D + r.b * (a.gamma + 1) + d;
            off = (size_t)r.b * (a.gamma + 1) + d;
        } else {
            r.b = rt / a.K;
            r.k = rt % a.K;
            r.row_id = D + (r.b * a.K + r.k) * (a.gamma + 1) + d;
            off = ((size_t)r.b * a.K + r.k) * (a.gamma + 1) + d;
        }
        r.ptr = (const unsigned char*)a.target_logits + off * (size_t)a.V * esize;
        r.slot0 = 0;
        r.nslots = a.target_slots;
        r.invT = a.inv_T_target;
        r.T = a.T_target;
    }
}

// Four workgroups per CU (128 VGPRs).  Of every kRolePeriod blocks, kRoleFinish
// finish rows and the others only stream segments, so the streaming loop
// (software-pipelined) and the races neither share a loop nor wait for each other
// (the share of finishing blocks was measured: 1/3, 94.3 us per call at V = 128256, K = 4,
// gamma = 4, B = 64; 4/11 95.9, 4/13 97.4, 3/7 98.2).  Both
// kinds take work in order from per-XCD queues (row R goes to queue R mod nq for
// both): streaming never waits, and a finishing workgroup waits only for segments
// (streamed without waiting) and for races of rows earlier in the order (taken
// earlier by running finishing workgroups), so every wait ends.
template <bool BF16, int LAYOUT>
__global__ __launch_bounds__(kBlock, 4) void race_kernel(RaceArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    Shared& sm = *reinterpret_cast<Shared*>(smem_raw);
    float* gm = reinterpret_cast<float*>(smem_raw + ((sizeof(Shared) + 15) & ~(size_t)15));
    const int tid = threadIdx.x;
    uint32_t* ctrl = ctrl_of(a);
    // roles: of every kRolePeriod consecutive blocks the last kRoleFinish finish rows
    // (the launch has at least kRolePeriod blocks); kRolePeriod is odd, so with
    // 8 kRolePeriod or more blocks every XCD queue (block mod 8) has both kinds
    const bool finisher = blockIdx.x % (unsigned)kRolePeriod >= (unsigned)(kRolePeriod - kRoleFinish);
    const int nq = gridDim.x >= 8u * kRolePeriod ? kMaxQueues : 1;
    const int q = (int)(blockIdx.x % (unsigned)nq);
    if (tid == 0) {
        sm.err_local = 0u;
        sm.epoch = epoch_after(ld_dev(ctrl + kCtrlEpoch));
        sm.tick[0] = finisher ? take_row(a, q, nq) : take_item(a, q, nq);
    }
    for (int i = tid; i < a.n_phase; i += kBlock) {
        sm.ph_first[i] = a.phase_first[i];
        sm.ph_depth[i] = a.phase_depth[i];
        sm.ph_nd[i] = a.phase_nd[i];
    }
    __syncthreads();
    if (finisher) {
        // Before its first row, a finishing workgroup streams segments from its queue
        // until that row's segments are all taken: at the start the streaming is
        // behind and the first rows' races wait for it.  (It never waits here.)
        int R = sm.tick[0];
        if (R < a.n_rows) {
            const int last = R * a.L.nseg + a.L.nseg - 1;
            for (int p = 0;; p ^= 1) {
                if (tid == 0) sm.tick[2 + p] = take_item(a, q, nq);
                __syncthreads();
                const int item = sm.tick[2 + p];
                if (item >= a.n_items) break;
                Row rs;
                int ss;
                decode_item<BF16>(a, sm, item, rs, ss);
                Unit<BF16> u[units_per_segment<BF16>()];
                issue_segment<BF16>(a, rs, ss, u);
                consume_segment<BF16>(a, rs, ss, sm, p, u);
                __syncthreads();
                publish_segment<BF16>(a, rs.row_id, ss, sm, p);
                if (item >= last) break;
            }
        }
        while (R < a.n_rows) {
            Row r;
            int seg;
            decode_item<BF16>(a, sm, R * a.L.nseg + a.L.nseg - 1, r, seg);
            finish_row<BF16, LAYOUT>(a, r, sm, gm);
            if (tid == 0) sm.tick[0] = take_row(a, q, nq);
            __syncthreads();
            R = sm.tick[0];
        }
    } else {
        // Software-pipelined: the next segment's loads are issued before the current
        // one is published.
        Unit<BF16> u[units_per_segment<BF16>()];
        int item = sm.tick[0], seg = 0;
        Row r;
        if (item < a.n_items) {
            decode_item<BF16>(a, sm, item, r, seg);
            issue_segment<BF16>(a, r, seg, u);
        }
        for (int parity = 0; item < a.n_items; parity ^= 1) {
            if (tid == 0) sm.tick[parity ^ 1] = take_item(a, q, nq);
            consume_segment<BF16>(a, r, seg, sm, parity, u);
            __syncthreads();
            const int pub_row = r.row_id, pub_seg = seg;
            item = sm.tick[parity ^ 1];
            if (item < a.n_items) {
                decode_item<BF16>(a, sm, item, r, seg);
                issue_segment<BF16>(a, r, seg, u);
            }
            publish_segment<BF16>(a, pub_row, pub_seg, sm, parity);
        }
    }
    // The last workgroup to leave resets the queues, hands over the call's error bits
    // and (unless a later kernel of the call does) records the epoch.  A workgroup that recorded errors fences (release)
    // before it counts its exit, and the last one fences (acquire) after it: its
    // read of the call's bits then sees every error of the call.  The exit count
    // itself stays relaxed (a release per workgroup writes back its L2: ~19 us).
    __syncthreads();
    if (tid == 0) {
        if (sm.err_local) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const uint32_t old = __hip_atomic_fetch_add(ctrl + kCtrlExited, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == gridDim.x - 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            const uint32_t bits =
                __hip_atomic_exchange(ctrl + kCtrlCallErrors, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (bits) __hip_atomic_fetch_or(ctrl + kCtrlErrors, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (a.status) *a.status = bits;
            for (int i = 0; i < 2 * kMaxQueues; ++i) st_dev(ctrl + ctrl_queue(i), 0u);
            st_dev(ctrl + kCtrlExited, 0u);
            if (!a.keep_epoch) st_dev(ctrl + kCtrlEpoch, sm.epoch);
        }
    }
}

// Shared, the group maxima and the level-4 list (K slots x level-4 nodes, 256 groups
// each), in the order level4_list assumes.
size_t shared_bytes(int ng, int K) {
    return ((sizeof(Shared) + 15) & ~(size_t)15) + (size_t)padded_groups(ng) * sizeof(float) +
           (size_t)K * (size_t)((ng + 255) / 256) * sizeof(Node);
}

template <bool BF16, int LAYOUT>
hipError_t launch_one(const RaceArgs& a, hipStream_t stream) {
    const size_t smem = shared_bytes(a.L.ng, a.K);
    auto fn = race_kernel<BF16, LAYOUT>;
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBlock, smem);
    if (e != hipSuccess) return e;
    int dev = 0, cus = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
    // both kinds of workgroup: at least kRolePeriod blocks
    long grid = (long)per_cu * cus;
    if (grid > (long)kRolePeriod * a.n_items) grid = (long)kRolePeriod * a.n_items;
    if (a.max_grid > 0 && grid > a.max_grid) grid = a.max_grid;
    if (grid < kRolePeriod) grid = kRolePeriod;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(kBlock), smem, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_race(const RaceArgs& a, bool bf16, int layout, hipStream_t stream) {
    if (bf16) return layout == 0 ? launch_one<true, 0>(a, stream) : launch_one<true, 1>(a, stream);
    return layout == 0 ? launch_one<false, 0>(a, stream) : launch_one<false, 1>(a, stream);
}

// ---------------------------------------------------------------- static scratch

// The allocation-free entry point's workspace: one fixed array per device, held
// until the process ends.  In host code `scratch` is only a handle for the
// runtime; its device address is looked up once per device (with that device
// current) and kept, and only that address is passed to kernels.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch(void** out, hipStream_t stream) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
        if (!p || ((uintptr_t)p & 255u) != 0) return hipErrorInvalidSymbol;
        // zero once (control words, epoch, queues) with a fill kernel ahead of the
        // first call on the caller's stream
        if ((e = launch_fill_zero((uint32_t*)p, kStaticScratchBytes / 4, stream)) != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace psd
