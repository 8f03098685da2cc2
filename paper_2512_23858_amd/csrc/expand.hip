// Equal-growth expansion: one draft step keeps exactly W new nodes, the candidates (frontier
// node p, token v) with the largest cumulative draft log-probability (paper Sec. 4.2, "Draft
// Width Selection").
//
// Two kernels:
//   scan     one workgroup per chunk of a logits row: streams the fp32 logits once and leaves the chunk's list: its sum of
//            exponentials in fp64 and its W largest logits, best first.  Inside one row the candidate order is the order
//            of the raw logits, so the lists are exact whatever the row's normaliser turns out to be.
//   finish   one workgroup per sequence, one list per thread: per-row log-sum-exp, fp64 scores cum[p] + (x - lse_p), and
//            the W best of all lists; ties go to the lower flat index p*V + v.  With free attachment the rows' W best
//            join the carried pool instead (below).
//
// Both are chains of dependent steps on little data: what counts is how many instructions, branches (a taken one costs
// about 50 cycles), barriers and memory trips follow each other.  Hence
//   - few candidates per thread (four at the small sizes), so that a chain is short and all compute units have work;
//   - "the W best" is never sorted out of all candidates: a threshold that at least W and few more candidates reach comes
//     from lane maxima, the candidates above it are pooled in LDS and ranked against each other;
//   - the sum of exponentials needs no maximum first (fp64 holds exp of any logit up to 500; a reference other than 0 is
//     kept only beyond that), and the row sums are plain sums of the chunks';
//   - a list's four best entries decide almost every step: the finish kernel requests them together with the list's sum, so
//     that it makes one trip to memory (the rest of a list is read only if all four reach the threshold).
// Measured per step, back to back (16 logits per thread, four list merges by binary search and a bitonic pool sort in LDS
// -> this): 8 rows of 32000 logits 12.8 -> 6.6 us, 128 rows of 32000 (batch 16) 18.4 -> 11.9, free attachment with 16 rows
// of 128256 24.6 -> 14.8.  Left at the small size: 1.5 us of launch per kernel, memory latency once per kernel, and 1 to
// 1.5 us of dependent steps in each; at the large one the fp64 exponentials (21 instructions per logit) and the selection.
#include "ygg_internal.h"
#include "ygg_device.h"

#include <algorithm>
#include <type_traits>

namespace ygg {
namespace {

constexpr uint32_t kNone = 0xffffffffu;
constexpr int kFront = 4;        // list entries read with the sum
constexpr int kMaxLists = 1024;  // lists of one sequence, padded to a power of two per row: one per thread of the finish kernel
constexpr float kPlainRange = 500.f;  // logits whose exponential is summed as it is

struct Cand {
    float val;
    int32_t idx;
};
struct __align__(16) ListStat {
    double sumexp;          // sum exp(x - ref) over the chunk
    float ref;              // 0, or the chunk's maximum where that lies outside +-kPlainRange
    int32_t count;          // entries of the list: min(W, logits in the chunk)
};
// A list as the finish kernels read it: its record and four entries.  Entries are dense, W to a list, so that a list takes no
// more scratch than its contents; they come in two 16-byte loads (8-byte aligned, which global loads allow).  Where W < 4 these
// reach into the next list or, behind the last one, into the records that follow the entries in the scratch.
struct ListHead {
    ListStat stat;
    Cand front[kFront];
};
__device__ __forceinline__ ListHead read_list(const ListStat* stats, const Cand* cands, int64_t list, int W) {
    ListHead h;
    h.stat = stats[list];
    const Cand* c = cands + list * W;
    __builtin_memcpy(&h.front[0], c, 16);
    __builtin_memcpy(&h.front[2], c + 2, 16);
    return h;
}

// Largest found t with at least `want` (and not many more) of the wavefront's NK*64 keys >= t; key 0 = no candidate.
// Returns 1, which every candidate reaches, if there are fewer than `want`.  Bisection in rounds of four steps: a step is
// a chain of about 60 cycles, a branch as much again.
template <int NK>
__device__ __forceinline__ uint32_t wave_threshold(const uint32_t (&g)[NK], int want) {
    auto count = [&](uint32_t t) {
        int n = 0;
#pragma unroll
        for (int i = 0; i < NK; ++i) n += (int)__popcll(__ballot(g[i] >= t));
        return n;
    };
    uint32_t top = g[0];
#pragma unroll
    for (int i = 1; i < NK; ++i) top = max(top, g[i]);
    uint32_t hi = wave_max_u32(top);
    uint32_t lo = wave_min_u32(top ? top : kNone);   // as many keys as there are lanes with any reach the smallest lane maximum
    int n = count(lo);
    if (n < want) n = count(lo = 1u);
    if (n < want) return 1u;
    const int enough = want + (want >> 3);
    while (lo < hi && n > enough) {              // n = count(lo) >= want; no key exceeds hi
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t mid = lo + ((hi - lo + 1) >> 1);
            const int m = count(mid);
            const bool ok = m >= want;
            lo = ok ? mid : lo;
            n = ok ? m : n;
            hi = ok ? hi : mid - 1;
        }
        hi = max(hi, lo);
    }
    return lo;
}

// Threshold over a workgroup's keys, one per thread, published in keys[64 * wave + lane] (barrier before): every wavefront
// works it out for itself from the 64 lane-wise maxima.  LOOSE and W <= 8: the lanes form eight groups, and W keys reach
// the smallest group maximum -- about 22 candidates are pooled instead of 9, which costs less time than a bisection (but
// more instructions: not where many workgroups share a compute unit).  W > 32: four maxima per lane, or too many candidates
// would lie above the threshold.
template <bool LOOSE>
__device__ __forceinline__ uint32_t group_threshold(const uint32_t* keys, int nwaves, int lane, int want) {
    uint32_t g[4] = {0, 0, 0, 0};
    for (int w = 0; w < nwaves; w += 4)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (w + u < nwaves) g[u] = max(g[u], keys[64 * (w + u) + lane]);
    if (want > 32) return wave_threshold<4>(g, want);
    const uint32_t one[1] = {max(max(g[0], g[1]), max(g[2], g[3]))};
    if (LOOSE && want <= 8) {
        uint32_t v = max(one[0], row_xor<8>(one[0]));
        auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = max(p[0], p[1]);
        p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = max(p[0], p[1]);
        v = min(v, row_xor<1>(v));
        v = min(v, row_xor<2>(v));
        v = min(v, row_xor<7>(v));
        const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
        if (t) return t;
    }
    return wave_threshold<1>(one, want);
}

// ---- scan ---------------------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanPool = 512;   // pooled candidates per chunk

struct ScanArgs {
    const float* logits;
    ListStat* stats;     // [rows][nchunk]
    Cand* cands;         // [rows][nchunk][W], best first
    int32_t V, W, chunk, nchunk;
};

__device__ __forceinline__ uint64_t order_of(uint32_t key, uint32_t idx) {   // larger = better: value, then lower index
    return ((uint64_t)key << 32) | (uint32_t)~idx;
}

// Exact but slow: for chunks of several passes whose logits climb from pass to pass until the pool is full.  Each round finds the
// best candidate after the last.
__device__ __noinline__ void scan_ties(const float* x, int c0, int c1, int want, int lane, Cand* out) {
    uint64_t last = ~0ull;
    for (int r = 0; r < want; ++r) {
        uint64_t best = 0;
        for (int i = c0 + lane; i < c1; i += 64) {
            const uint64_t o = order_of(key_of(x[i]), (uint32_t)i);
            if (o < last && o > best) best = o;
        }
        const uint32_t bh = wave_max_u32((uint32_t)(best >> 32));
        const uint32_t bl = wave_max_u32((uint32_t)(best >> 32) == bh ? (uint32_t)best : 0u);
        last = ((uint64_t)bh << 32) | bl;
        if (lane == 0) {
            const Cand cd = {float_of(bh), (int32_t)~bl};
            out[r] = cd;
        }
    }
}

// Appends the wavefront's selected candidates to a pool: the positions follow from ballots and one count per wavefront.
// Few candidates are selected, so what(i), the candidate's pool entry, is formed only where some lane has it.  Does nothing and
// returns false if there are more than `limit`.
template <int N, typename T, typename What>
__device__ __forceinline__ bool pool_put(const bool (&sel)[N], What what, T* pool, int cap, int* counter, int lane, int limit) {
    uint64_t m[N];
    int total = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        m[i] = __ballot(sel[i]);
        total += (int)__popcll(m[i]);
    }
    if (total == 0) return true;
    if (__builtin_expect(total > limit, 0)) return false;
    int base = 0;
    if (lane == 0) base = atomicAdd(counter, total);
    base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (__builtin_expect(m[i] != 0, 0)) {
            const int pos = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m[i] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[i], 0));
            pool[sel[i] && pos < cap ? pos : cap + lane] = what(i);   // (a slot of the lane's own behind the pool: no branch)
            base += (int)__popcll(m[i]);
        }
    }
    return true;
}

// Narrows a wavefront's selection (more than 64 candidates, keys 0 elsewhere) to the `want` best, or an eighth more where that
// spares bisection steps: the threshold among them alone, and of the candidates that tie with it those of the lowest indices, as
// many as are wanted.  Indices ascend from lane to lane with QUAD places each, then to the next group
// of QUAD places.
template <int E, int QUAD>
__device__ __forceinline__ void narrow(const uint32_t (&key)[E], int want, int lane, bool (&sel)[E]) {
    const uint32_t t = wave_threshold<E>(key, want);
    int room = want;
#pragma unroll
    for (int i = 0; i < E; ++i) room -= (int)__popcll(__ballot(key[i] > t));
    int before = 0;   // ties in the groups in front
#pragma unroll
    for (int i0 = 0; i0 < E; i0 += QUAD) {
        int mine = before, all = 0;
#pragma unroll
        for (int u = 0; u < QUAD; ++u) {
            const uint64_t m = __ballot(key[i0 + u] == t);
            mine += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
            all += (int)__popcll(m);
        }
#pragma unroll
        for (int u = 0; u < QUAD; ++u) {
            const bool tie = key[i0 + u] == t;
            sel[i0 + u] = key[i0 + u] > t || (tie && mine < room);
            mine += tie;
        }
        before += all;
    }
}

// Number of pool entries better than the lane's own, for pools of up to 64 entries followed by zeros.  Up to 32 entries the
// two halves of the wavefront share the comparisons (lane j and lane j + 32 get the rank of entry j).
__device__ __forceinline__ int rank_in_wave(const uint64_t* pool, int n, int lane, uint64_t& mine) {
    const bool halves = n <= 32;
    mine = pool[halves ? lane & 31 : lane];
    uint32_t r = 0;
    const int step = halves ? 8 : 4;
    const uint64_t* q = pool + (halves ? (lane >> 5) * 4 : 0);
    for (int i = 0; i < n; i += step) {
        uint64_t x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = q[i + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) r += x[u] > mine;
    }
    if (halves) {
        const auto p = __builtin_amdgcn_permlane32_swap(r, r, false, false);
        r = p[0] + p[1];
    }
    return (int)r;
}

// E logits per thread and pass; a chunk is one pass (256 E logits) or, with ONE = false, several.  VEC: 16-byte loads (row
// starts and V are multiples of four logits).
// Chunks of 1024 and 2048 logits leave a compute unit one to three workgroups (plan_expand), whose chain of steps is the kernel's time:
// four more wavefronts load the same logits and sum their exponentials while the first four select and rank.  us per step, four
// wavefronts for both -> this: 8 rows of 32000 logits 7.0 -> 6.5, 16 rows of 32000 (512 chunks of 1024) 7.6 -> 7.2, one row of 128256
// 7.3 -> 6.7, 12 rows of 128256 (756 chunks of 2048) 10.3 -> 9.6.
// Longer chunks keep every SIMD busy with several workgroups: what counts is the work, so one wavefront finds the threshold, while the
// others are at the exponentials already, and candidates are pooled behind those (128 rows of 32000 logits 14.1 -> 13.6 us per step,
// 256 rows of 128256 49.8 -> 47.2; with chunks of 2048 one to four rows of 70000 to 128256 lost 1 to 3 % that way).
template <int E>
constexpr int scan_threads() { return E <= 8 ? 2 * kScanThreads : kScanThreads; }
template <int E, bool VEC, bool ONE>
__global__ __launch_bounds__(scan_threads<E>()) void expand_scan_kernel(ScanArgs a) {
    constexpr int PASS = kScanThreads * E;
    constexpr bool SPLIT = E <= 8;   // (always one pass)
    __shared__ __align__(16) uint64_t pool[kScanPool + 64];
    __shared__ uint32_t keys[kScanThreads];
    __shared__ double sums[4];
    __shared__ int pooled;
    __shared__ uint32_t thr;
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave_all & 3;
    const bool selects = !SPLIT || wave_all < 4, adds = !SPLIT || wave_all >= 4;
    const int lane = threadIdx.x & 63, tid = 64 * wave + lane;
    const int c = blockIdx.y;
    const int64_t row = blockIdx.x, list = row * a.nchunk + c;
    const int c0 = c * a.chunk, c1 = min(a.V, c0 + a.chunk);
    const float* __restrict__ x = a.logits + row * a.V;
    const int want = min(a.W, c1 - c0);
    uint32_t best = 0;      // key of the thread's largest logit
    float ref = 0.f;
    double sum = 0.0;       // this thread's share of sum exp(x - ref)
    uint32_t t_seen = 0;    // at least `want` logits of the passes so far reach it
    int base = c0;
    do {
        float v[E];
        const int w0 = base + wave * (64 * E);
        const bool full = base + PASS <= c1;
        auto index = [&](int i) { return VEC ? w0 + 256 * (i >> 2) + 4 * lane + (i & 3) : w0 + 64 * i + lane; };
        auto load = [&](auto whole) {   // places past the end hold NaN: it loses every comparison and adds nothing to the sum
            constexpr float none = __builtin_nanf("");
#pragma unroll
            for (int k = 0; k < E / 4; ++k) {
                if constexpr (VEC) {
                    float4 q = make_float4(none, none, none, none);
                    if (whole || index(4 * k) < c1) q = *reinterpret_cast<const float4*>(x + index(4 * k));
                    v[4 * k] = q.x; v[4 * k + 1] = q.y; v[4 * k + 2] = q.z; v[4 * k + 3] = q.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[4 * k + e] = whole || index(4 * k + e) < c1 ? x[index(4 * k + e)] : none;
                }
            }
        };
        if (full) load(std::true_type{}); else load(std::false_type{});
        if (selects) {
            if (base == c0) {   // while the loads are out
#pragma unroll
                for (int i = tid; i < kScanPool; i += kScanThreads) pool[i] = 0;
                if (tid == 0) pooled = 0;
            }
            float vmax = v[0];
#pragma unroll
            for (int i = 1; i < E; ++i) vmax = fmaxf(vmax, v[i]);
            best = index(0) < c1 ? max(best, key_of(vmax)) : best;
            keys[tid] = best;
        }
        __syncthreads();
        if (!SPLIT && wave == 0) {
            const uint32_t t = max(group_threshold<false>(keys, 4, lane, want), t_seen);
            if (lane == 0) thr = t;
        }
        if (adds) {   // sum of exponentials
            const uint32_t top = max(max(keys[lane], keys[64 + lane]), max(keys[128 + lane], keys[192 + lane]));
            const float cmax = float_of(wave_max_u32(top));   // of the chunk so far
            const float r = fabsf(cmax) <= kPlainRange || cmax == -INFINITY ? 0.f : cmax;
            if (r != ref) {   // a first pass has nothing to rescale; later the reference only moves so that the sum shrinks
                sum = sum == 0.0 ? 0.0 : sum * exp_nonpos((double)ref - (double)r);
                ref = r;
            }
            constexpr int NE = E < 8 ? E : 8;   // independent series in step: a dependent fp64 operation takes 20 cycles
#pragma unroll
            for (int i0 = 0; i0 < E; i0 += NE) {
                double t[NE], e[NE];
#pragma unroll
                for (int i = 0; i < NE; ++i) t[i] = (double)fmaxf(v[i0 + i], -746.f);   // (places past the end, -inf: next to nothing)
                if (__builtin_expect(ref != 0.f, 0)) {   // subtracted in fp64: where fp32 has no 746 any more (2^34), a bound formed there is ref itself
#pragma unroll
                    for (int i = 0; i < NE; ++i) t[i] = fmax((double)v[i0 + i] - (double)ref, -746.0);
                }
                exp_clamped_n(t, e);
#pragma unroll
                for (int i = 0; i < NE; i += 4) sum += (e[i] + e[i + 1]) + (e[i + 2] + e[i + 3]);
            }
        }
        if (!SPLIT) __syncthreads();   // the threshold is there
        if (selects) {
            const uint32_t t = SPLIT ? group_threshold<E == 4>(keys, 4, lane, want) : thr;
            // (equal ones of a later pass come too late, for their higher indices: from the next key on, where +inf is followed by a NaN,
            // which nothing reaches, and -0 by 0, which -0 reaches as well: one candidate more)
            const uint32_t least = !ONE && t == t_seen ? t + 1 : t;
            const float tf = least <= 1u ? -INFINITY : float_of(least);
            bool sel[E];
#pragma unroll
            for (int i = 0; i < E; ++i) sel[i] = v[i] >= tf;
            if (!ONE && t > 1u) t_seen = t;
            auto entry = [&](int i) { return order_of(key_of(v[i]), (uint32_t)index(i)); };
            // Of many equal logits (a masked vocabulary's -inf or -1e9) a wavefront keeps the W best by index: a step of 32 x 128256
            // logits with 1000 of the vocabulary unmasked 283 -> 31 us (every such chunk went through the rounds of scan_ties).
            constexpr int kMost = ONE ? kScanPool / 4 : kMaxWidth + kMaxWidth / 8;
            if (!pool_put(sel, entry, pool, kScanPool, &pooled, lane, kMost)) {
                uint32_t key[E];
#pragma unroll
                for (int i = 0; i < E; ++i) key[i] = sel[i] ? key_of(v[i]) : 0u;
                narrow<E, VEC ? 4 : 1>(key, want, lane, sel);
                pool_put(sel, entry, pool, kScanPool, &pooled, lane, kMost);
            }
        }
        base += PASS;
        if (ONE || base >= c1) break;
        __syncthreads();   // the next pass writes keys and the threshold again
    } while (true);
    if (adds) {
        sum = group_sum(sum, 64);
        if (lane == 0) sums[wave] = sum;
    }
    __syncthreads();
    Cand* out = a.cands + list * a.W;
    if (adds && tid == 0) {
        ListStat st;
        st.sumexp = (sums[0] + sums[1]) + (sums[2] + sums[3]);
        st.ref = ref;
        st.count = min(want, pooled);   // (fewer than wanted only if there are NaNs, which no list takes: it says what it holds)
        a.stats[list] = st;
    }
    if (!selects) return;
    auto store = [&](int rank, uint64_t o) {
        const Cand cd = {float_of((uint32_t)(o >> 32)), (int32_t)~(uint32_t)o};
        if (rank < want) out[rank] = cd;
    };
    const int n = __builtin_amdgcn_readfirstlane(pooled);
    if (n <= 64) {
        if (wave > 0) return;
        uint64_t mine;
        const int rank = rank_in_wave(pool, n, lane, mine);
        if (lane < n) store(rank, mine);
    } else if (n <= kScanPool) {
        for (int j = tid; j < n; j += kScanThreads) {
            const uint64_t mine = pool[j];
            int rank = 0;
            for (int i = 0; i < n; i += 8) {   // (zeros follow the pooled entries)
                uint64_t x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = pool[i + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) rank += x[u] > mine;
            }
            store(rank, mine);
        }
    } else if (!ONE && wave == 0) {   // (one pass leaves no more than the pool holds)
        scan_ties(x, c0, c1, want, lane, out);
    }
}

// Log-sum-exp of a row from its lists, which sit in an aligned group of `width` lanes (fixed order of summation).
__device__ __forceinline__ double row_lse(const ListStat& h, int width) {
    if (!__any(h.ref != 0.f)) return log(group_sum(h.sumexp, width));
    const float ref = h.sumexp > 0.0 ? h.ref : -INFINITY;
    const float mx = group_reduce(ref, width, [](float x, float y) { return fmaxf(x, y); });
    const double s = ref > -INFINITY ? h.sumexp * exp_nonpos((double)ref - (double)mx) : 0.0;
    return (double)mx + log(group_sum(s, width));
}

// ---- finish, frontier rule ------------------------------------------------------------------------
// A candidate: larger key first, then lower tie; key == 0 means "no candidate" (real keys are > 0).
struct __align__(16) Entry {
    uint64_t key;
    uint32_t tie;
    uint32_t tag;
};
__device__ __forceinline__ bool beats(const Entry& a, const Entry& b) {
    return a.key > b.key || (a.key == b.key && a.tie < b.tie);
}

struct FinishArgs {
    const ListStat* stats;
    const Cand* cands;
    int32_t* parent_idx;
    int32_t* token_ids;
    float* cum_logprob;
    unsigned char* pool;   // free attachment only: per sequence {int32 count, pad to 16 B, pool_cap offers}
    int32_t pool_cap;
    int32_t D, W, V, N, d, F, nchunk, shift;   // 1 << shift: lists of a row padded to a power of two
};

constexpr int kMergePool = 1024;   // pooled candidates of one sequence

// Where a row has few lists for many new nodes, W of the lists' first four entries are all or most of these: nearly everything would
// reach the threshold.  The first 32 or 64 entries of every list then decide, sixteen to a lane: lanes c << share .. share a list.
// That is a trip to memory more.  us per first step, the first four -> this: 12 nodes from 5 lists 8.5 -> 9.5, 8 from one 7.1 -> 7.7,
// 16 from 5 8.8 -> 9.2, 24 from 10 9.3 -> 9.8; 16 from one 8.8 -> 8.3, 20 from 5 14.8 -> 9.7, 40 from 10 86 -> 11.
__device__ __forceinline__ bool few_lists(int nchunk, int W) { return W > 12 && nchunk * kFront < W + W / 4; }   // (fewer than 20 lists)
struct Shared16 {
    Cand cd[16];
    const Cand* list;   // the lane's list, its length, what the lanes hold of it, and how many entries this lane holds
    int count, covered, mine;
    bool last;          // holds the last of these
};
__device__ __forceinline__ Shared16 read_shared(const Cand* row, int nchunk, int W, int count, int lane) {
    const int share = nchunk <= 16 ? 2 : 1, step = 1 << share, c = lane >> share, q = lane & (step - 1);
    Shared16 x;
    x.count = __shfl(count, c);
    x.list = row + (x.count > 0 ? c * W : 0);
    x.covered = 16 * step;
    x.mine = min(max((x.count - q + step - 1) >> share, 0), 16);
    x.last = q == step - 1;
#pragma unroll
    for (int i = 0; i < 16; ++i) x.cd[i] = x.list[max(min(q + step * i, x.count - 1), 0)];
    return x;
}
// Goes on through a list, four entries at a time, while put says that they reach the threshold.
template <typename Put>
__device__ __forceinline__ void read_on(const Cand* list, int from, int count, Put put) {
    for (int i = from; i < count; i += 4) {
        Cand cd[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) cd[u] = list[min(i + u, count - 1)];
        bool more = true;
#pragma unroll
        for (int u = 0; u < 4; ++u) more = more && i + u < count && put(cd[u]);
        if (!more) break;
    }
}

// The W best of up to 64 lists, one per lane, in order: a round per entry, every lane offering the next entry of its list, which it
// holds four at a time, the next four already requested.  Used where a threshold over the first four entries leaves too many
// candidates to rank them against each other: many equal ones (masked vocabularies).  About 0.6 us a round; returns the number of
// entries.
template <typename EntryOf, typename Emit>
__device__ __forceinline__ int merge_rounds(const Cand* list, int count, int W, EntryOf entry_of, Emit emit) {
    Cand now[4], next[4];
    auto request = [&](int i0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) next[u] = list[max(min(i0 + u, count - 1), 0)];
    };
    int cur = -1;
    Entry mine;
    auto advance = [&]() {
        ++cur;
        if ((cur & 3) == 0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) now[u] = next[u];
            request(cur + 4);
        }
        Cand cd = now[0];
#pragma unroll
        for (int u = 1; u < 4; ++u) cd = (cur & 3) == u ? now[u] : cd;
        mine = cur < count ? entry_of(cd) : Entry{0, kNone, 0};
    };
    request(0);
    advance();
    int r = 0;
    for (; r < W; ++r) {
        const uint32_t kh = wave_max_u32((uint32_t)(mine.key >> 32));
        const uint32_t kl = wave_max_u32((uint32_t)(mine.key >> 32) == kh ? (uint32_t)mine.key : 0u);
        const uint64_t k = ((uint64_t)kh << 32) | kl;
        const uint32_t t = wave_min_u32(mine.key == k ? mine.tie : kNone);
        if (k == 0) break;
        emit(r, Entry{k, t, 0});
        if (mine.key == k && mine.tie == t) advance();
    }
    return r;
}

// Bounded by latency: one trip to memory, two row reductions, a bisection, two barriers.
__global__ __launch_bounds__(kMaxLists) void expand_merge_kernel(FinishArgs a, int nwaves) {
    __shared__ uint32_t coarse[kMaxLists];   // upper halves of the keys of the list heads
    __shared__ Entry pool[kMergePool + 64];
    __shared__ int pooled;
    __shared__ uint32_t thr;
    const int tid = threadIdx.x, lane = tid & 63;
    const int b = blockIdx.x;
    const int base_prev = a.d == 1 ? 0 : 1 + (a.d - 2) * a.W;
    const int p = tid >> a.shift, c = tid & ((1 << a.shift) - 1);
    const bool active = p < a.F && c < a.nchunk;
    const int64_t list = ((int64_t)b * a.F + (active ? p : 0)) * a.nchunk + (active ? c : 0);
    ListHead h = read_list(a.stats, a.cands, list, a.W);
    const double cum = (double)a.cum_logprob[(int64_t)b * a.N + base_prev + (active ? p : 0)];
    if (!active) h.stat = ListStat{0.0, 0.f, 0};
    const Cand* cands = a.cands + list * a.W;
    for (int i = tid; i < kMergePool; i += 64 * nwaves) pool[i] = Entry{0, kNone, 0};   // while the loads are out
    if (tid == 0) pooled = 0;

    const double lse = row_lse(h.stat, 1 << a.shift);
    auto entry_of = [&](Cand cd) {
        return Entry{key_of(cum + ((double)cd.val - lse)), (uint32_t)(p * a.V + cd.idx), (uint32_t)p};   // tie: flat index p*V + v
    };
    Entry e[kFront];
#pragma unroll
    for (int i = 0; i < kFront; ++i) e[i] = i < h.stat.count ? entry_of(h.front[i]) : Entry{0, kNone, 0};

    // threshold: W list heads reach it (with fewer lists than four times W, W of the first entries of every list: the lowest of these
    // heads would let too many through), so nothing below it can be among the W best
    const bool few = nwaves == 1 && a.F * a.nchunk < 4 * a.W;   // (below 2W it is one wavefront: F == 1 or one list a row)
    const bool deep = few && a.F == 1 && few_lists(a.nchunk, a.W);
    auto put = [&](const Entry& x) {
        const int pos = atomicAdd(&pooled, 1);
        if (pos < kMergePool) pool[pos] = x;
    };
    uint32_t t;
    if (deep) {   // (one row: the first lane's sum is everyone's)
        const double lse0 = __longlong_as_double(((long long)__builtin_amdgcn_readfirstlane((int)(__double_as_longlong(lse) >> 32)) << 32) |
                                                 (uint32_t)__builtin_amdgcn_readfirstlane((int)__double_as_longlong(lse)));
        const Shared16 x = read_shared(a.cands + (int64_t)b * a.nchunk * a.W, a.nchunk, a.W, h.stat.count, lane);
        auto entry = [&](Cand cd) { return Entry{key_of(cum + ((double)cd.val - lse0)), (uint32_t)cd.idx, 0}; };
        uint32_t g[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) g[i] = i < x.mine ? (uint32_t)(entry(x.cd[i]).key >> 32) : 0u;
        __syncthreads();   // (pooled is zero)
        t = wave_threshold<16>(g, a.W);
        bool sel[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) sel[i] = g[i] >= t;
        pool_put(sel, [&](int i) { return entry(x.cd[i]); }, pool, kMergePool, &pooled, lane, kMergePool);
        if (x.last && g[15] >= t)
            read_on(x.list, x.covered, x.count, [&](Cand cd) {
                const Entry y = entry(cd);
                const bool reaches = (uint32_t)(y.key >> 32) >= t;
                if (reaches) put(y);
                return reaches;
            });
    } else if (few) {
        uint32_t g[kFront];
#pragma unroll
        for (int i = 0; i < kFront; ++i) g[i] = (uint32_t)(e[i].key >> 32);
        __syncthreads();   // (pooled is zero)
        t = wave_threshold<kFront>(g, a.W);
    } else {
        coarse[tid] = (uint32_t)(e[0].key >> 32);
        __syncthreads();
        if (nwaves <= 4) {
            t = group_threshold<true>(coarse, nwaves, lane, a.W);
        } else {   // several wavefronts on a SIMD would slow each other down: one bisects for all
            if (tid < 64) {
                t = group_threshold<true>(coarse, nwaves, lane, a.W);
                if (tid == 0) thr = t;
            }
            __syncthreads();
            t = thr;
        }
    }

    if (!deep) {
        bool sel[kFront];
#pragma unroll
        for (int i = 0; i < kFront; ++i) sel[i] = (uint32_t)(e[i].key >> 32) >= t;
        pool_put(sel, [&](int i) { return e[i]; }, pool, kMergePool, &pooled, lane, kMergePool);
        if ((uint32_t)(e[kFront - 1].key >> 32) >= t)
            read_on(cands, kFront, h.stat.count, [&](Cand cd) {
                const Entry y = entry_of(cd);
                const bool reaches = (uint32_t)(y.key >> 32) >= t;
                if (reaches) put(y);
                return reaches;
            });
    }
    __syncthreads();
    const int n = __builtin_amdgcn_readfirstlane(pooled);
    auto emit_of_row = [&](int rank, const Entry& x, uint32_t row) {
        if (rank >= a.W) return;
        const int64_t node = (int64_t)b * a.N + 1 + (a.d - 1) * a.W + rank;
        a.parent_idx[node] = base_prev + (int)row;
        a.token_ids[node] = (int)(x.tie - row * (uint32_t)a.V);
        a.cum_logprob[node] = (float)double_of(x.key);
    };
    auto emit = [&](int rank, const Entry& x) { emit_of_row(rank, x, x.tie / (uint32_t)a.V); };   // (no tag)
    const int nthr = 64 * nwaves;
    if (n > 64 && (n + nthr - 1) / nthr * n > 24 * a.W) {   // four comparisons of all entries cost 0.1 us
        Entry* mine = pool + (tid >> 6) * a.W;   // the wavefronts' lists
        const int m = merge_rounds(cands, h.stat.count, a.W, entry_of, [&](int r, const Entry& x) {
            if (lane == 0) {
                if (nwaves == 1) emit(r, x); else mine[r] = x;
            }
        });
        if (nwaves == 1) return;
        for (int r = m + lane; r < a.W; r += 64) mine[r] = Entry{0, kNone, 0};
        __syncthreads();
        for (int j = tid; j < nwaves * a.W; j += nthr) {   // places: those of every list are found by halving
            const Entry x = pool[j];
            int rank = 0;
            for (int w = 0; w < nwaves; ++w) {
                int lo = 0, hi = a.W;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (beats(pool[w * a.W + mid], x)) lo = mid + 1; else hi = mid;
                }
                rank += lo;
            }
            if (x.key != 0) emit(rank, x);
        }
        return;
    }
    if (n <= 64) {
        if (tid >= 64) return;
        const bool halves = n <= 32;   // the halves of the wavefront share the comparisons
        const Entry mine = pool[halves ? lane & 31 : lane];
        const Entry* q = pool + (halves ? lane >> 5 : 0) * 4;
        const int step = halves ? 8 : 4;
        uint32_t rank = 0;
        for (int i = 0; i < n; i += step) {   // (empty entries follow the pooled ones)
            Entry x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = q[i + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) rank += beats(x[u], mine);
        }
        if (halves) {
            const auto r = __builtin_amdgcn_permlane32_swap(rank, rank, false, false);
            rank = r[0] + r[1];
        }
        if (lane < n) emit_of_row((int)rank, mine, mine.tag);
        return;
    }
    for (int j = tid; j < n; j += nthr) {
        const Entry mine = pool[j];
        int rank = 0;
        for (int i = 0; i < n; i += 4) {
            Entry x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = pool[i + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) rank += beats(x[u], mine);
        }
        emit_of_row(rank, mine, mine.tag);
    }
}

// ---- finish, free attachment ------------------------------------------------------------------------
// Every node, once the drafter has run on it, offers its W most probable tokens; the pool holds the
// offers not yet taken; a step takes the W best of the pool (paper Sec. 4.2: the W new leaves of a
// step may hang anywhere in the partial tree).  One workgroup per sequence: its wavefronts take a new row each (one list
// per lane), work out the row's W offers, and the workgroup sorts pool + offers, emits the W new nodes and keeps the best
// W*(D-t) of the rest: an entry of rank r needs r / W more steps before it can be taken and later offers only push
// it down, so nothing beyond the slots still to be filled can ever be chosen.
struct __align__(16) Offer {
    double score;
    int32_t node;
    int32_t token;
};
constexpr int kPoolHeader = 16;  // bytes: int32 count, padding
constexpr int kRowPool = 512;    // pooled candidates of one row
// At most this many comparisons to a thread: places are counted instead of sorted.  The sort is a chain of 28 to 45 exchanges; counting
// takes a pass over the entries for every 64 of them (1024 threads).  us per step with all sorted -> 48 / 128 / 400: 16 nodes of 128256
// logits 14.6 -> 13.3 / 13.5 / 13.5, 12 x 4 sequences of 32000 13.1 -> 12.0 / 12.2 / 12.2, 20 nodes 15.7 -> 14.6 / 14.7 / 16.5, 24 of 50257
// 17.0 -> 16.2 / 16.2 / 19.8.
constexpr int kCountPerThread = 48;

// Bitonic sort of one entry per thread, best first; n2 (a power of two) threads take part, the others only meet the
// barriers.  Exchanges inside a wavefront stay in registers (39 of the 45 stages for 512 entries).
__device__ __forceinline__ Entry sort_in_registers(Entry mine, Entry* e, int tid, int n2) {
    auto keep = [&](const Entry& other, int j, int k) {
        const bool better = ((tid & j) == 0) == ((tid & k) == 0);   // this side of the pair keeps the better entry
        if (beats(other, mine) == better) mine = other;
    };
    for (int k = 2; k <= n2; k <<= 1) {
        for (int j = k >> 1; j >= 64; j >>= 1) {
            if (tid < n2) e[tid] = mine;
            __syncthreads();
            if (tid < n2) keep(e[tid ^ j], j, k);
            __syncthreads();
        }
        auto step = [&](auto jc) {
            constexpr int J = decltype(jc)::value;
            if (k > J) {
                Entry o;
                o.key = ((uint64_t)lane_xor<J>((uint32_t)(mine.key >> 32)) << 32) | lane_xor<J>((uint32_t)mine.key);
                o.tie = lane_xor<J>(mine.tie);
                o.tag = 0;
                keep(o, J, k);
            }
        };
        step(std::integral_constant<int, 32>{}); step(std::integral_constant<int, 16>{}); step(std::integral_constant<int, 8>{});
        step(std::integral_constant<int, 4>{}); step(std::integral_constant<int, 2>{}); step(std::integral_constant<int, 1>{});
    }
    return mine;
}

// The entries of a list from `from` on that reach t.
__device__ __forceinline__ void pool_rest(const Cand* list, int from, int count, uint32_t t, uint64_t* pool, int* counter) {
    read_on(list, from, count, [&](Cand cd) {
        const uint32_t key = key_of(cd.val);
        if (key < t) return false;
        const int pos = atomicAdd(counter, 1);
        if (pos < kRowPool) pool[pos] = order_of(key, (uint32_t)cd.idx);
        return true;
    });
}
// The candidates of a row of few lists (a function of its own: its registers would make the kernel spill).
__device__ __noinline__ void pool_of_few_lists(const Cand* row, int nchunk, int W, int count, int lane, uint64_t* pool, int* counter) {
    const Shared16 x = read_shared(row, nchunk, W, count, lane);
    uint32_t g[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) g[i] = i < x.mine ? key_of(x.cd[i].val) : 0u;
    const uint32_t t = wave_threshold<16>(g, W);
    bool sel[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) sel[i] = g[i] >= t;
    pool_put(sel, [&](int i) { return order_of(g[i], (uint32_t)x.cd[i].idx); }, pool, kRowPool, counter, lane, 1024);
    if (x.last && g[15] >= t) pool_rest(x.list, x.covered, x.count, t, pool, counter);
}

// Keeps the `need` best of n entries (and not many more, but for ties), in any order; n up to four times the threads, *counter 0.
// Returns their number.  More entries than threads are sorted through LDS with a barrier per stage, which costs several times as much:
// 32 rows of 50257 logits with 160 to keep 57 -> 33 us per step, 60 rows of 14000 132 -> 56.
__device__ __forceinline__ int drop_unneeded(Entry* e, int n, int need, int tid, int nthr, int* counter, uint32_t (*part)[16]) {
    const int lane = tid & 63, wave = tid >> 6, nwaves = nthr >> 6;
    Entry x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = tid + u * nthr < n ? e[tid + u * nthr] : Entry{0, kNone, 0};
    auto upper = [&](int u) { return (uint32_t)(x[u].key >> 32); };
    const uint32_t top = wave_max_u32(max(max(upper(0), upper(1)), max(upper(2), upper(3))));
    if (lane == 0) part[0][wave] = top;
    __syncthreads();
    uint32_t lo = 1, hi = 0;
    for (int w = 0; w < nwaves; ++w) hi = max(hi, part[0][w]);
    int have = n, turn = 1;
    while (lo < hi && have > need + (need >> 3)) {   // have: entries that reach lo
        const uint32_t mid = lo + ((hi - lo + 1) >> 1);
        int m = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) m += (int)__popcll(__ballot(upper(u) >= mid));
        if (lane == 0) part[turn][wave] = (uint32_t)m;
        __syncthreads();
        m = 0;
        for (int w = 0; w < nwaves; ++w) m += (int)part[turn][w];
        turn ^= 1;
        if (m >= need) { lo = mid; have = m; } else hi = mid - 1;
    }
    bool sel[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) sel[u] = upper(u) >= lo;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint64_t m = __ballot(sel[u]);
        int at = 0;
        if (lane == 0 && m) at = atomicAdd(counter, (int)__popcll(m));
        at = __builtin_amdgcn_readfirstlane(at);
        if (sel[u]) e[at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))] = x[u];
    }
    __syncthreads();
    return *counter;
}

__global__ __launch_bounds__(1024) void attach_finish_kernel(FinishArgs a, int nwaves, int n2_max) {
    extern __shared__ __align__(16) unsigned char raw_s[];
    Entry* e = reinterpret_cast<Entry*>(raw_s);                                        // [n2_max]
    uint64_t* pools = reinterpret_cast<uint64_t*>(raw_s + (size_t)n2_max * sizeof(Entry));   // [nwaves][kRowPool + 64]
    __shared__ int n_live, n_kept, row_n[16];
    __shared__ uint64_t floor_s;
    __shared__ uint32_t bisect_s[2][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nthr = 64 * nwaves;
    const int b = blockIdx.x;
    unsigned char* pool_b = a.pool + (size_t)b * (kPoolHeader + (size_t)a.pool_cap * sizeof(Offer));
    int32_t* pool_count = reinterpret_cast<int32_t*>(pool_b);
    Offer* pool = reinterpret_cast<Offer*>(pool_b + kPoolHeader);
    const int first = a.d == 1 ? 0 : 1 + (a.d - 2) * a.W;   // first of the nodes whose rows came in

    // Only W*(D-t+1) entries are ever needed: the W new nodes and the pool kept for later.  When the carried pool
    // alone already holds that many, an offer scoring below the pool's last entry cannot be among them, so it is
    // dropped before the sort (exact: equal scores are kept).
    const int need = a.W * (a.D - a.d + 1);
    int n_old = 0;
    if (a.d > 1) {
        const int most = min(a.pool_cap, need);   // what the previous step may have left
        const int count = *pool_count;
        n_old = min(max(count, 0), most);
        for (int i = tid; i < most; i += nthr) {  // (requested together with the count)
            const Offer o = pool[i];
            if (i < n_old) e[i] = Entry{key_of(o.score), (uint32_t)o.node * (uint32_t)a.V + (uint32_t)o.token, 0};
        }
    }
    if (tid == 0) {
        n_live = n_old;
        n_kept = 0;
    }
    __syncthreads();
    if (tid == 0) floor_s = n_old >= need && n_old > 0 ? e[n_old - 1].key : 0ull;
    uint64_t* mypool = pools + wave * (kRowPool + 64);

    for (int p = wave; p < a.F; p += nwaves) {
        const int64_t list = ((int64_t)b * a.F + p) * a.nchunk + min(lane, a.nchunk - 1);
        ListHead h = read_list(a.stats, a.cands, list, a.W);
        const double cum = (double)a.cum_logprob[(int64_t)b * a.N + first + p];
        if (lane >= a.nchunk) h.stat = ListStat{0.0, 0.f, 0};
        const Cand* cands = a.cands + list * a.W;
        const double lse = row_lse(h.stat, 64);
        // the row's W best, by raw logit: threshold over the first four entries of every list (over all entries of few lists), then
        // pool and rank
        if (lane == 0) row_n[wave] = 0;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (few_lists(a.nchunk, a.W)) {
            pool_of_few_lists(a.cands + ((int64_t)b * a.F + p) * a.nchunk * a.W, a.nchunk, a.W, h.stat.count, lane, mypool, &row_n[wave]);
        } else {
            uint32_t g[kFront];
#pragma unroll
            for (int i = 0; i < kFront; ++i) g[i] = i < h.stat.count ? key_of(h.front[i].val) : 0u;
            const uint32_t head_key[1] = {g[0]};
            // (W of fewer than 2W heads: the lowest of them let too many through, 24 rows of 25 lists 34.9 -> 47.0 us for two steps)
            const uint32_t t = a.nchunk >= 2 * a.W ? wave_threshold<1>(head_key, a.W) : wave_threshold<kFront>(g, a.W);
            bool sel[kFront];
#pragma unroll
            for (int i = 0; i < kFront; ++i) sel[i] = g[i] >= t;
            pool_put(sel, [&](int i) { return order_of(g[i], (uint32_t)h.front[i].idx); }, mypool, kRowPool, &row_n[wave], lane, kRowPool);
            if (g[kFront - 1] >= t) pool_rest(cands, kFront, h.stat.count, t, mypool, &row_n[wave]);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        int n = __builtin_amdgcn_readfirstlane(row_n[wave]);
        if (n > 64 && (n + 63) / 64 * n > 24 * a.W) {   // (as in the merge kernel, one wavefront)
            n = merge_rounds(cands, h.stat.count, a.W, [&](Cand cd) { return Entry{order_of(key_of(cd.val), (uint32_t)cd.idx), 0, 0}; },
                             [&](int r, const Entry& x) { if (lane == 0) mypool[r] = x.key; });
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        if (p == wave) __syncthreads();   // floor_s is there (every wavefront passes here once: nwaves <= F)
        if (a.d == 1 && lane == 0) n_live = min(n, a.W);
        if (lane < 8) mypool[n + lane] = 0;   // zeros follow the entries (there is room: 64 slots behind the pool)
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        auto offer = [&](int rank, uint64_t o) {
            if (rank >= a.W) return;
            const Entry x = {key_of(cum + ((double)float_of((uint32_t)(o >> 32)) - lse)),
                             (uint32_t)(first + p) * (uint32_t)a.V + (uint32_t)~(uint32_t)o, 0};
            if (a.d == 1) e[rank] = x;   // the root's offers alone: already in order
            else if (x.key >= floor_s) e[atomicAdd(&n_live, 1)] = x;
        };
        if (n <= 64) {
            uint64_t mine;
            const int rank = rank_in_wave(mypool, n, lane, mine);
            if (lane < n) offer(rank, mine);
        } else {
            for (int j = lane; j < n; j += 64) {
                const uint64_t mine = mypool[j];
                int rank = 0;
                for (int i = 0; i < n; i += 4) {
                    uint64_t x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) x[u] = mypool[i + u];
#pragma unroll
                    for (int u = 0; u < 4; ++u) rank += x[u] > mine;
                }
                offer(rank, mine);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // the next row reuses the pool
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    int n_sort = n_live;
    if (n_sort > nthr && n_sort <= 4 * nthr && n_sort > need) n_sort = drop_unneeded(e, n_sort, need, tid, nthr, &n_kept, bisect_s);
    const int base_new = 1 + (a.d - 1) * a.W;
    const int keep = min(a.W * (a.D - a.d), max(n_sort - a.W, 0));
    auto emit = [&](int i, const Entry& x) {
        if (i >= min(n_sort, a.W + keep)) return;
        const uint32_t node = x.tie / (uint32_t)a.V;
        const int token = (int)(x.tie - node * (uint32_t)a.V);
        const double score = double_of(x.key);
        if (i < a.W) {
            const int64_t dst = (int64_t)b * a.N + base_new + i;
            a.parent_idx[dst] = (int)node;
            a.token_ids[dst] = token;
            a.cum_logprob[dst] = (float)score;
        } else {
            Offer o;
            o.score = score; o.node = (int)node; o.token = token;
            pool[i - a.W] = o;
        }
    };
    if (tid == 0) *pool_count = keep;
    // Few entries for the threads there are: a row of 16 lanes counts the entries better than its own, which is that one's place (no two
    // are equal: they differ in node or token).
    if (a.d > 1 && n_sort * n_sort <= kCountPerThread * nthr) {
        for (int i = tid >> 4; i < n_sort; i += nthr >> 4) {
            const Entry mine = e[i];
            uint32_t r = 0;
            for (int j0 = tid & 15; j0 < n_sort; j0 += 64) {
                Entry x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = e[min(j0 + 16 * u, n_sort - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) r += j0 + 16 * u < n_sort && beats(x[u], mine);
            }
            r += row_xor<1>(r);
            r += row_xor<2>(r);
            r += row_xor<7>(r);
            r += row_xor<15>(r);
            if ((tid & 15) == 0) emit((int)r, mine);
        }
        return;
    }
    int n2 = 2;
    while (n2 < n_sort) n2 <<= 1;   // <= n2_max: the launch sized the buffer for every offer surviving
    if (n2 <= nthr) {
        Entry mine = tid < n_sort ? e[tid] : Entry{0, kNone, 0};
        if (a.d > 1) {
            __syncthreads();
            mine = sort_in_registers(mine, e, tid, n2);
        }
        emit(tid, mine);
        return;
    }
    for (int i = n_sort + tid; i < n2; i += nthr) e[i] = Entry{0, kNone, 0};
    __syncthreads();
    // bitonic sort in LDS, best first (larger key, then lower node*V + token); empty slots sink to the end
    for (int k = 2; k <= n2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < (n2 >> 1); i += nthr) {
                const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1));
                const int hi = lo | j;
                const Entry x = e[lo], y = e[hi];
                const bool down = (lo & k) == 0;
                if (down ? beats(y, x) : beats(x, y)) { e[lo] = y; e[hi] = x; }
            }
            // Pairs at distance <= 64 stay inside one 128-element block, and a block belongs to the same wavefront
            // in every stage: two such stages in a row need no workgroup barrier (LDS accesses of one wavefront
            // complete in order; the fence keeps the compiler from moving them).
            const int j_next = j > 1 ? j >> 1 : k;   // first distance of the next k is k
            if (j <= 64 && j_next <= 64) {
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
            } else {
                __syncthreads();
            }
        }
    __syncthreads();  // the sorted order is read by every wavefront
    for (int i = tid; i < min(n_sort, a.W + keep); i += nthr) emit(i, e[i]);
}

int pow2_at_least(int64_t x) {
    int n = 1;
    while (n < x) n <<= 1;
    return n;
}

hipError_t launch_scan(const ExpandArgs& a, hipStream_t st) {
    ScanArgs s;
    s.logits = a.logits;
    s.stats = static_cast<ListStat*>(a.stats);
    s.cands = static_cast<Cand*>(a.cands);
    s.V = a.V; s.W = a.W; s.chunk = a.chunk; s.nchunk = a.nchunk;
    const dim3 grid((unsigned)(a.B * a.F), (unsigned)a.nchunk);
    const bool vec = (a.V & 3) == 0 && (reinterpret_cast<uintptr_t>(a.logits) & 15u) == 0;
    auto go = [&](auto e, auto one) {
        constexpr int E = decltype(e)::value;
        constexpr bool ONE = decltype(one)::value;
        const dim3 block(scan_threads<E>());
        if (vec) hipLaunchKernelGGL((expand_scan_kernel<E, true, ONE>), grid, block, 0, st, s);
        else hipLaunchKernelGGL((expand_scan_kernel<E, false, ONE>), grid, block, 0, st, s);
    };
    if (a.chunk == 4 * kScanThreads) go(std::integral_constant<int, 4>{}, std::true_type{});
    else if (a.chunk == 8 * kScanThreads) go(std::integral_constant<int, 8>{}, std::true_type{});
    else if (a.chunk == 16 * kScanThreads) go(std::integral_constant<int, 16>{}, std::true_type{});
    else go(std::integral_constant<int, 16>{}, std::false_type{});
    return hipGetLastError();
}

FinishArgs finish_args(const ExpandArgs& a) {
    FinishArgs f;
    f.stats = static_cast<const ListStat*>(a.stats);
    f.cands = static_cast<const Cand*>(a.cands);
    f.parent_idx = a.parent_idx; f.token_ids = a.token_ids; f.cum_logprob = a.cum_logprob;
    f.pool = static_cast<unsigned char*>(a.pool); f.pool_cap = a.pool_cap;
    f.D = a.D; f.W = a.W; f.V = a.V; f.N = a.N; f.d = a.d; f.F = a.F; f.nchunk = a.nchunk;
    f.shift = 0;
    while ((1 << f.shift) < a.nchunk) ++f.shift;
    return f;
}

}  // namespace

// The most lists a step takes of 1024 and of 2048 logits (plan_expand).
constexpr int64_t kListsOf1024 = 512, kListsOf2048 = 768;
static size_t stat_bytes_of(int64_t lists) { return ((size_t)lists * sizeof(ListStat) + 255) / 256 * 256; }
static size_t cand_bytes_of(int64_t lists, int32_t width) { return ((size_t)lists * (size_t)width * sizeof(Cand) + 255) / 256 * 256; }

// Chunk length: the finish kernel takes one list per thread and a row's lists from one wavefront, which bounds the lists
// per row; within that, short chunks (1024 logits, four per thread) keep every compute unit busy and each thread's chain
// short, long ones (4096) leave a quarter of the fixed work of a workgroup, of the lists to write and of those to read back.
// us per step with chunks of 1024 / 2048 / 4096, by the number of chunks of 2048: 272 (17 rows of 32000) 8.5 / 7.7 / 8.2; 384 (3 x 8 rows
// of 32000) 7.6 / 7.2 / 8.2; 512 (32 rows) 12.0 / 10.3 / 10.9; 512 (32 x 16 rows of 1500) 11.5 / 10.7 / 12.5; 768 (6 x 8 rows of 32000)
// 9.9 / 9.0 / 10.4; 756 (12 rows of 128256) - / 9.6 / 9.8; 1008 (16 rows of 128256) - / 11.7 / 10.7; 2048 (128 rows of 32000) 16.5 / 14.3 /
// 13.6; 8192 (512 rows of 32000) 47.0 / 37.8 / 29.3.  The lines were drawn for a scan with four wavefronts to every chunk; with eight, 256
// chunks of 2048 (16 rows of 32000) would be a little faster than 512 of 1024 (7.1 / 6.7 / 8.2) and 1024 of 64 rows of 32000 than 512 of
// 4096 (10.9 / 10.1 / 10.6), which 16 rows of 128256 are not.
ExpandPlan plan_expand(const ygg_shape& s, int32_t d) {
    ExpandPlan p;
    p.F = d == 1 ? 1 : s.width;
    const int64_t most = std::min(64, kMaxLists / pow2_at_least(p.F));   // lists per row
    const int64_t rows = (int64_t)s.batch * p.F;
    auto lists = [&](int64_t chunk) { return (s.vocab + chunk - 1) / chunk; };
    int64_t chunk = 1024;
    if (lists(chunk) > most || rows * lists(chunk) > kListsOf1024) chunk = 2048;
    if (chunk == 2048 && (lists(chunk) > most || rows * lists(chunk) > kListsOf2048)) chunk = 4096;
    if (lists(chunk) > most) chunk = ((int64_t)s.vocab + 4096 * most - 1) / (4096 * most) * 4096;
    p.chunk = (int32_t)chunk;
    p.nchunk = (int32_t)lists(chunk);
    const int64_t total = rows * p.nchunk;
    p.stat_bytes = stat_bytes_of(total);
    p.cand_bytes = cand_bytes_of(total, s.width);
    return p;
}

// Fewer rows or logits can mean more lists, shorter ones: the bound is that of chunks of 4096, or of every list there may be while
// chunks are shorter, so that scratch sized for the largest batch and vocabulary serves the smaller ones.
size_t expand_scratch_bytes(const ygg_shape& s) {
    const int64_t lists = std::max((int64_t)s.batch * s.width * (((int64_t)s.vocab + 4095) / 4096), kListsOf2048);
    return cand_bytes_of(lists, s.width) + stat_bytes_of(lists);
}

// The largest dynamic LDS the attachment kernel may ask for: 4096 entries and the row pools of sixteen wavefronts.
hipError_t raise_limits_expand() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(attach_finish_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(4096 * sizeof(Entry) + 16 * (kRowPool + 64) * sizeof(uint64_t)));
}

hipError_t launch_expand(const ExpandArgs& a, hipStream_t st) {
    if (hipError_t e = launch_scan(a, st)) return e;
    const FinishArgs f = finish_args(a);
    const int nwaves = ((a.F << f.shift) + 63) / 64;
    hipLaunchKernelGGL(expand_merge_kernel, dim3((unsigned)a.B), dim3(64 * nwaves), 0, st, f, nwaves);
    return hipGetLastError();
}

int64_t attach_pool_capacity(const ygg_shape& s) { return (int64_t)s.width * (s.depth > 1 ? s.depth - 1 : 1); }
size_t attach_pool_bytes(const ygg_shape& s) {
    return ((size_t)s.batch * (kPoolHeader + (size_t)attach_pool_capacity(s) * sizeof(Offer)) + 255) / 256 * 256;
}

hipError_t launch_attach(const ExpandArgs& a, hipStream_t st) {
    if (hipError_t e = launch_scan(a, st)) return e;
    const FinishArgs f = finish_args(a);
    const int n = a.F * a.W + (a.d == 1 ? 0 : a.W * (a.D - a.d + 1));
    const int n2 = pow2_at_least(std::max(n, 2));
    // a wavefront per new row; the sort wants a thread per entry, which all wavefronts below sixteen cannot give: rows
    // are then shared out anyway
    const int nwaves = std::min(16, a.F);
    const size_t lds = (size_t)n2 * sizeof(Entry) + (size_t)nwaves * (kRowPool + 64) * sizeof(uint64_t);
    hipLaunchKernelGGL(attach_finish_kernel, dim3((unsigned)a.B), dim3(64 * nwaves), lds, st, f, nwaves, n2);
    return hipGetLastError();
}

}  // namespace ygg
