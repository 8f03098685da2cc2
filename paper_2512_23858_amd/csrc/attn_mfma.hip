// Tree-masked verify attention on the gfx950 matrix cores (bf16 storage, head_dim 128 or 64).
//
// Operation (paper Sec. 2 "Source of Improvements", Sec. 4.2 last paragraph): every tree node
// attends to the confirmed prefix, to its ancestors and to itself, all nodes in one pass.
//
// Decomposition.  For one sequence b and kv head g the N tree nodes and the Hq/Hkv query heads
// of the group form R = N*(Hq/Hkv) query rows that all read the same K/V stream.  A workgroup
// owns (b, g, one tile of query rows, one split of the key range); its NW wavefronts own RB
// blocks of 32 rows each and share every K/V tile through LDS, so a K/V byte is fetched from
// L2/HBM once per 32*RB*NW rows.  Workgroup ids are laid out so that all row tiles of one
// (b, g, split) land on the same XCD and hit in its L2.
//
// Per 32-key block and 32-row block (all MFMA are v_mfma_f32_32x32x16_bf16):
//   S^T = K . Q^T      A = K rows from LDS (16-byte reads), B = Q held in registers
//   online softmax     a lane owns one query row: 16 scores in registers; base-2 exponentials
//                      against a per-row reference that moves rarely (no row maximum on the
//                      common path)
//   O^T += V^T . P^T   A = V^T through the LDS transpose read (ds_read_b64_tr_b16), B = P^T,
//                      which is exactly the accumulator layout of S^T packed to bf16
// The tree's own keys are the tail of the key range; their ancestor mask comes from per-node
// bitmasks built in LDS from parent_idx.
//
// The same kernel also serves K/V stored as 8-bit E4M3 codes (template flag KV8): extra loading
// wavefronts widen the codes to bf16 while filling the LDS tiles, everything else is shared.
#include "attn_common.h"

#include <cstdlib>
#include <type_traits>

namespace ygg {
namespace {

using namespace attn;

// 16-byte load from global memory proper (a pointer chosen between two arrays would otherwise be
// loaded through the generic path, whose completion also counts as an LDS event).
// Streaming hint: the codes are used once (a plain streaming read of the same size measures 6.9 TB/s with it, 6.1 without).
__device__ __forceinline__ u32x4 global_load16(uint64_t gaddr) {
    return __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) u32x4*>(gaddr));
}

// Sixteen E4M3 codes (memory order) -> sixteen bf16; exact, the format has 3 mantissa bits.  One
// conversion instruction per pair of codes (scale operand 1.0).
__device__ __forceinline__ void e4m3x16_to_bf16(const u32x4& raw, uint4& first8, uint4& last8) {
    const uint32_t w[4] = {raw[0], raw[1], raw[2], raw[3]};
    uint32_t o[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o[2 * i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[i], 1.0f, false));     // bytes 0, 1
        o[2 * i + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[i], 1.0f, true));  // bytes 2, 3
    }
    first8 = make_uint4(o[0], o[1], o[2], o[3]);
    last8 = make_uint4(o[4], o[5], o[6], o[7]);
}

// NW wavefronts, RB 32-row blocks per wavefront, KT keys per tile, KS key shares: with KS = 2 the
// wavefronts pair up on the same rows and each takes one of the two 32-key blocks of every tile (a
// tree of few nodes has too few rows to occupy a workgroup otherwise); the pair's (m, l, O~) are
// merged through LDS before the result is written.
//
// KV8: K and V are stored as 8-bit E4M3 codes with one scale per kv head.  The codes are widened
// to bf16 on their way into LDS (exactly), so tiles, operand reads and matrix work are those of
// the bf16 kernel; the scales fold into the softmax scale and into the final normalisation.  The
// direct-to-LDS path cannot convert, so the workgroup gets four extra wavefronts that do nothing but
// load codes into registers (four tiles ahead; eight measured no faster), widen them and store the
// rows into the tile buffers; the NW computing wavefronts never touch global K/V.  Both kinds meet
// at the same one barrier per tile.
//
// NT: the direct-to-LDS tile fills carry the streaming hint (the host sets it when a K/V stream has one
// row tile, i.e. is read by a single workgroup; with several row tiles the re-reads are meant to hit in L2).
//
// BAL: balanced batches (see the segment loop below); a separate instantiation, so that the single-segment variants
// carry none of its loop state.
//
// DHT: head_dim, 128 or 64 (bf16 K/V only for 64).  Everything below counts in k-steps of 16 and output blocks of 32
// head_dim positions, and a direct-to-LDS instruction brings 1024 / ROWB rows.
template <int NW, int RB, int KT, int KS, bool KV8, bool NT, bool BAL = false, int DHT = 128, bool PING = false>
__global__ __launch_bounds__((NW + (KV8 ? 4 : 0)) * 64, (RB == 1 && !KV8 ? 2 : 1)) void attn_mfma_kernel(AttnArgs a) {
    static_assert(!BAL || KS == 1, "balanced batches: plain 32-row wavefronts only");
    static_assert(DHT == 128 || (DHT == 64 && !KV8), "head_dim 64: bf16 K/V only");
    constexpr int DH = DHT;
    constexpr int ROWB = 2 * DH;                                 // bytes of one K or V row in LDS
    constexpr int NS = DH / 16;                                  // k-steps of S^T = K.Q^T
    constexpr int NDB = DH / 32;                                 // 32-wide blocks of head_dim in O^T
    constexpr int SLOTS = ROWB / 16;                             // 16-byte slots per row = lanes that fill one row
    constexpr int RPI = 1024 / ROWB;                             // rows one direct-to-LDS wave-instruction brings
    static_assert(KS == 1 || (KS == 2 && NW % 2 == 0 && KT == 64), "key shares: one block of the tile each");
    constexpr int NLD = KV8 ? 4 : 0;                             // loading wavefronts (KV8 only)
    constexpr int NSET = 4;                                      // register sets (tiles in flight) per loader
    constexpr int THREADS = (NW + NLD) * 64;
    static_assert(!KV8 || NW <= 4, "loading wavefronts share the SIMDs with at most one computing wavefront each");
    constexpr int NRW = NW / KS;                                 // wavefronts along the rows
    constexpr int RW = NRW * RB * 32;                            // query rows per workgroup
    constexpr int TILEB = KT * ROWB;                             // bytes of one K (or V) tile
    // Tiles are prefetched two ahead.  PING (plan_attention says when): the two wavefronts of a SIMD run half a block apart, which takes
    // a fourth tile buffer.
    static_assert(!PING || (KS == 1 && (NW == 8 || (NW == 6 && !BAL && DH == 128)) && !KV8), "SIMDs with two wavefronts");
    constexpr int NBUF = PING ? 4 : 3;
    // wavefronts that issue tile fills (a power of two, so that each issues the same number per tile)
    constexpr int FILLERS = NW >= 8 ? 8 : NW >= 4 ? 4 : NW >= 2 ? 2 : 1;
    constexpr int PT = 2 * (KT / RPI) / FILLERS;  // direct-to-LDS loads per filling wavefront and tile
    static_assert((KT / RPI) % FILLERS == 0, "every filling wavefront issues the same number of loads");
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* k_s = smem;                                   // [NBUF][KT][ROWB]
    unsigned char* v_s = smem + NBUF * TILEB;                    // [NBUF][KT][ROWB]
    // Q passes through the tile buffers from the third on (tile 2 is requested once it is read) and, where these
    // do not hold it, through space behind them.  In space of its own, shared by the wavefronts of a pair and with a third tile
    // requested at once, it leaves room for two workgroups of four wavefronts of head_dim 64 to a compute unit instead of three: 48
    // sequences of 300 tokens, 49 rows on 12 kv heads 16.9 -> 18.8 us per call; and where one is enough it gains nothing: 22 of 192 with
    // 5 rows 8.3 -> 8.7, one of 2048 with 65 rows 10.2 either way, of 1024 with 49 rows on 32 kv heads of 128 12.7 -> 12.8.
    // QSHARED: the two wavefronts of the 32-row shape fetch the rows that there are once between them, instead of 32 each: on 32 kv heads 2
    // rows x 62 tokens 8.80 -> 8.52 us per call, 5 x 267 9.10 -> 8.85, 16 x 46 9.20 -> 9.00, 25 x 488 10.33 -> 10.27; on 8, 12 rows x 113 8.61
    // -> 8.35.  At head_dim 64, where 32 rows are half as many bytes, 8.20 either way (32 x 214 on 8).  Skipped rows alone, without sharing:
    // half of the gain, and wider pairs lose 1 %.
    constexpr int QW = 32 * RB * ROWB;           // a wavefront's rows
    constexpr int QB = 2 * (NBUF - 2);           // wavefronts whose rows fit the spare K (or V) buffers
    constexpr int QX = NW > 2 * QB ? (NW - 2 * QB) * QW : 0;
    constexpr bool QSHARED = !KV8 && KS == 2 && NW == 2 && DH == 128;
    static_assert(RB == 1 && QW * 2 == TILEB, "two wavefronts' rows to a tile buffer");
    uint32_t* anc_s = reinterpret_cast<uint32_t*>(smem + 2 * NBUF * TILEB + QX);  // [local node][aw], then parent[N]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction
    const int n = lane & 31, g2 = lane >> 5;
    const bool is_loader = KV8 && wave >= NW;      // wave-uniform
    const int wrow = KS == 1 ? wave : wave % NRW;  // position along the rows (computing wavefronts)
    const int kh = KS == 1 ? 0 : wave / NRW;       // which block of every tile (KS = 2)
    const int wq = QSHARED ? wrow : wave;
    unsigned char* q_s = (wq < QB ? k_s + 2 * TILEB + wq * QW
                                  : wq < 2 * QB ? v_s + 2 * TILEB + (wq - QB) * QW : smem + 2 * NBUF * TILEB + (wq - 2 * QB) * QW);

    // All arguments at once: left to itself the compiler fetches each where it is first needed, one scalar-cache miss after
    // the other in front of the first tile fill (32 layers of a 516-row verify pass: 923 -> 887 us).  The paired shapes'
    // short launches measured 3 % slower that way and fetch as they go.
    if constexpr (KS == 1)
        asm volatile("" ::"s"(a.q), "s"(a.k_cache), "s"(a.v_cache), "s"(a.k_tree), "s"(a.v_tree), "s"(a.seq_lens), "s"(a.parent_idx),
                     "s"(a.N), "s"(a.Hq), "s"(a.Hkv), "s"(a.G), "s"(a.nsplit), "s"(a.max_seq_len), "s"(a.S), "s"(a.row_tiles),
                     "s"(a.mul_nsplit), "s"(a.mul_last), "s"(a.tree_cost), "s"(a.mul_hkv), "s"(a.mul_g), "s"(a.mul_rt), "s"(a.cap));
    // workgroup id -> (stream sigma = (b, kv head, split) or (kv head, slot), row tile); sigma % 8 picks the XCD
    const int wg8 = (int)divide(blockIdx.x >> 3, a.row_tiles, a.mul_rt);
    const int rt = (int)(blockIdx.x >> 3) - wg8 * a.row_tiles;
    const int sigma = wg8 * 8 + (blockIdx.x & 7);
    if (sigma >= a.S) return;
    const int R = a.N * a.G;
    const int row_base = rt * RW;

    // Which (sequence, key range) segments does this workgroup serve?
    //   classic   one segment: sigma = (sequence, kv head, split); the split is one of nsplit shares of that
    //             sequence's own key tiles (below).
    //   balanced  (a.slots > 0, batches) sigma = (kv head, slot).  The sequences' 64-key tiles are laid end to end and
    //             cut into a.slots runs of equal length; the workgroup serves its run, i.e. the tail of one sequence,
    //             whole short sequences, the head of another, one segment after the other.  Every workgroup then has the
    //             same work whatever the mix of lengths (a ragged batch otherwise takes as long as its longest sequence).
    //             A segment costs more than its tiles (Q, masks, an empty pipeline, the partial rows), so every sequence
    //             is laid out with `lead` empty tiles in front of it: the runs that hold many short sequences get
    //             fewer tiles.  Sequences of equal lengths with a whole number of runs to each get as many as let the runs
    //             end where the sequences do (none or a few): every workgroup then has one segment.  A run may fall wholly
    //             inside these and then has nothing to do; a sequence's own tiles are contiguous, so the runs it falls into
    //             are consecutive.  Segment number (slot - first slot of the sequence) is the split index of its partials;
    //             nsplit = a.slots bounds it.  A sequence that lies inside one slot is written out directly.
    //             Equal lengths, the same lead for all -> this, us per call on 8 kv heads: 4 x 1024 tokens with 776 rows
    //             38.0 -> 35.1, 2 x 2048 with 1544 53.8 -> 50.2, 4 x 2048 with 392 32.6 -> 31.1.
    // The head of the kernel is a chain of dependent scalar work in front of the first tile fill (the length is a load from
    // device memory), so divisions are multiplications by host-made reciprocals and the lengths of a batch are read by one
    // vector load.
    constexpr bool balanced = BAL;
    int hk, b_first, b_last, slot = 0, run_lo = 0, run_hi = 0, tiles_before = 0;
    int lead = 0;
    int run_q = 1, run_r = 0;   // the first run_r runs have run_q + 1 tiles, the others run_q
    if constexpr (!balanced) {
        const int hb = (int)divide(sigma, a.nsplit, a.mul_nsplit);
        b_first = b_last = (int)divide(hb, a.Hkv, a.mul_hkv);
        hk = hb - b_first * a.Hkv;
    } else {
        hk = (int)divide(sigma, a.slots, a.mul_nsplit);   // (nsplit == slots)
        slot = sigma - hk * a.slots;
        constexpr int CH = 4;   // 64 sequences at a time: batches of up to 256
        int tl[CH] = {};        // (all of them: the sum below takes those beyond the batch too)
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (64 * c >= a.B) break;
            const int bb = 64 * c + lane;
            int Lb = bb < a.B ? a.seq_lens[bb] : 0;
            Lb = Lb < 0 ? 0 : (Lb > a.max_seq_len ? a.max_seq_len : Lb);
            tl[c] = bb < a.B ? (Lb + a.N + kKeyTile - 1) / kKeyTile : 0;
        }
        lead = a.lead;
        if (a.seq_runs > 0) {
            const int first = __builtin_amdgcn_readfirstlane(tl[0]);
            bool other = false;
#pragma unroll
            for (int c = 0; c < CH; ++c) other = other || (64 * c + lane < a.B && tl[c] != first);
            if (!__any(other)) lead = a.seq_runs - 1 - (first + a.seq_runs - 1) % a.seq_runs;
        }
        int mine = 0;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (64 * c + lane < a.B) tl[c] += lead;
            mine += tl[c];
        }
        const int tiles_all = wave_sum_i32(mine);
        // (never more runs than units: the host sized the grid for the longest lengths the shape allows)
        const int nruns = min(a.slots, tiles_all);
        if (slot >= nruns) return;   // a workgroup beyond the last run: nothing to do
        run_q = nruns == a.slots ? (int)divide(tiles_all, a.slots, a.mul_nsplit) : 1;
        run_r = tiles_all - run_q * nruns;
        run_lo = slot * run_q + min(slot, run_r);
        run_hi = run_lo + run_q + (slot < run_r);
        // first and last sequence with tiles inside [run_lo, run_hi), from the prefix sums over the batch
        b_first = 0;
        b_last = -1;
        int base = 0;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (64 * c >= a.B) break;
            const int incl = base + wave_prefix_i32(tl[c], lane);
            const uint64_t upto = __ballot(incl <= run_lo), before = __ballot(incl - tl[c] + lead < run_hi && tl[c] > 0);
            const int nf = (int)__popcll(upto), nl = (int)__popcll(before);
            if (b_first == 64 * c && nf < 64) tiles_before = __builtin_amdgcn_readlane(incl - tl[c], nf);
            if (b_first == 64 * c) b_first += nf;
            if (nl > 0) b_last = 64 * c + nl - 1;
            base = __builtin_amdgcn_readlane(incl, 63);
        }
    }
    // the run that holds tile x of the concatenation
    auto slot_of_tile = [&](int x) {
        const int head = run_r * (run_q + 1);
        return x < head ? x / (run_q + 1) : run_r + (x - head) / run_q;
    };
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    if constexpr (balanced) {
        b_first = uni(b_first); b_last = uni(b_last); run_lo = uni(run_lo); run_hi = uni(run_hi);
        lead = uni(lead); tiles_before = uni(tiles_before) + lead; run_q = uni(run_q); run_r = uni(run_r);
    }

    for (int b = b_first; b <= b_last; ++b) {
    if (balanced && b != b_first) __syncthreads();   // the previous segment's tile buffers and masks are free again
    // What depends on the lane is formed anew for every segment: kept from one to the next it takes the registers of the tile
    // loop (33 to 43 spilled per lane; two sequences of 2048 tokens x 776 rows on 8 kv heads 42.2 -> 32.9 us per call).
    int tid = threadIdx.x;
    if constexpr (balanced) asm volatile("" : "+v"(tid));
    const int lane = tid & 63, n = lane & 31, g2 = lane >> 5;
    int L = a.seq_lens[b];   // (requested first)
    // rows of this lane: block rb of this wave -> row_base + (wrow*RB + rb)*32 + n
    int rg_of[RB];       // global row index (b, node, q head) or -1; fits 31 bits (checked on the host)
    int node_of[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = row_base + (wrow * RB + rb) * 32 + n;
        const int rc = min(row, R - 1);
        const int i = (int)divide(rc, a.G, a.mul_g);
        node_of[rb] = i;
        rg_of[rb] = row < R && !is_loader ? (b * a.N + i) * a.Hq + hk * a.G + (rc - i * a.G) : -1;
    }
    // The wavefront's rows of Q pass through LDS, requested before the length is needed: direct-to-LDS loads into a part of
    // its own (no barrier before it reads them back), with the slot permutation of K.  Rows beyond the last one repeat it and
    // are never stored.  As plain register loads they would hold up the first block until every tile in flight has landed:
    // the compiler's wait for them does not know of the tile fills behind them and awaits those as well.
    bf16x8 qreg[RB][NS];
    const int q_last = QSHARED ? min(R - 1 - row_base, 31) : 31;   // the last row of the block that is fetched; those behind repeat it
    if constexpr (KV8) {   // (the computing wavefronts have nothing else in flight: plain loads)
        if (!is_loader) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int rg = (b * a.N + node_of[rb]) * a.Hq + hk * a.G + (min(row_base + (wrow * RB + rb) * 32 + n, R - 1) - node_of[rb] * a.G);
                const bf16x8* qp = reinterpret_cast<const bf16x8*>(static_cast<const uint16_t*>(a.q) + (int64_t)rg * DH + 8 * g2);
#pragma unroll
                for (int s = 0; s < NS; ++s) qreg[rb][s] = qp[2 * s];
            }
        }
    } else {
        const uint32_t q_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)q_s;
#pragma unroll
        for (int i0 = 0; i0 < 32 * RB / RPI; i0 += QSHARED ? KS : 1) {
            const int it = i0 + (QSHARED ? kh : 0);   // (the two take turns)
            if (RPI * it > q_last) break;             // wave-uniform
            const int lrow = RPI * it + lane / SLOTS;
            const int rc = min(row_base + wrow * RB * 32 + lrow, R - 1);
            const int i = (int)divide(rc, a.G, a.mul_g);
            const int rg = (b * a.N + i) * a.Hq + hk * a.G + (rc - i * a.G);
            dma_load16_flat<false>(static_cast<const unsigned char*>(a.q) + (int64_t)rg * ROWB + 16 * ((lane % SLOTS) ^ (lrow & (SLOTS - 1))),
                                   __builtin_amdgcn_readfirstlane(q_lds + it * 1024));
        }
    }

    auto fetch_parents = [&](int32_t* to) {   // straight into LDS
        const int32_t* parent = a.parent_idx + (int64_t)b * a.N;
        const uint32_t lds = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)to;
        for (int t = 64 * wave; t < a.N; t += 64 * NW)   // (the last lanes repeat the last entry; LDS is sized for that)
            dma_load4(parent + min(t + lane, a.N - 1), __builtin_amdgcn_readfirstlane(lds + 4 * t));
    };
    // where the masks end and the parents begin: behind those of the nodes this workgroup's rows belong to
    auto parents_at = [&]() { return reinterpret_cast<int32_t*>(anc_s + (min(R - 1, row_base + RW - 1) / a.G - row_base / a.G + 1) * ((a.N + 31) >> 5)); };
    // Shapes without pairs: requested before the length says who needs them.
    constexpr bool kParentsFirst = !KV8 && !BAL && KS == 1;
    if constexpr (kParentsFirst) fetch_parents(parents_at());

    L = L < 0 ? 0 : (L > a.max_seq_len ? a.max_seq_len : L);
    const int Tk = L + a.N;
    int k0, k1, split = 0;
    bool direct = a.nsplit == 1;   // this segment is the whole sequence: final rows are written here
    const int nt = (Tk + kKeyTile - 1) / kKeyTile;
    if constexpr (!balanced) {
        // The sequence's own 64-key tiles, dealt out as evenly as whole tiles allow.  The last split has the tree's keys and their
        // masks to do as well, which takes about tree_cost tiles more (plan_attention): as many fewer are its share, as far as that
        // shortens the longest split and leaves it the tree's keys.  The others get equal shares, the first of them one tile more.
        // Pairs: few tiles to a workgroup and no time for the arithmetic in front of the first (49 rows x 1024 tokens on 32 kv heads
        // 12.8 -> 13.1 us per call).  The last split takes the smaller share; at head_dim 64 it gives a tile away if that leaves the
        // longest split no longer and the tree's keys in the last one (12 heads, 65 rows x 2048 tokens 10.7 -> 10.3 us per call; with the
        // tree cut in two, 524 rows x 277 tokens on 8 kv heads 10.3 -> 10.8).  At head_dim 128 three sequences of up to 1531 tokens, 144 rows
        // on 8 lost: 16.5 -> 16.9.
        const int hb = (int)divide(sigma, a.nsplit, a.mul_nsplit), last = a.nsplit - 1;
        split = sigma - hb * a.nsplit;
        const int even = (int)divide(nt, a.nsplit, a.mul_nsplit);
        int t0, share;
        if constexpr (KS == 2) {
            int r = nt - even * a.nsplit;
            if constexpr (DH == 64) r += r > 0 && r < last && even > 1 && (last * even + r + 1) * kKeyTile <= L;
            t0 = split * even + min(split, r);
            share = DH == 64 && split == last ? nt - t0 : even + (split < r);
        } else if (last == 0) {
            t0 = 0;
            share = nt;
        } else {
            const int longest = (int)divide(nt + a.tree_cost + last, a.nsplit, a.mul_nsplit);
            const int tree = max(min(longest - a.tree_cost, even), min(even, (a.N + 2 * kKeyTile - 2) / kKeyTile));
            const int end = nt - max(max(tree, nt - last * longest), 1);   // the last split's first tile
            const int q = (int)divide(end, last, a.mul_last), r = end - q * last;
            t0 = split == last ? end : split * q + min(split, r);
            share = split == last ? nt - end : q + (split < r);
        }
        k0 = t0 * kKeyTile;
        k1 = min(Tk, (t0 + share) * kKeyTile);
    } else {
        const int t0 = max(run_lo, tiles_before) - tiles_before, t1 = min(run_hi, tiles_before + nt) - tiles_before;
        const int s_first = slot_of_tile(tiles_before), s_last = slot_of_tile(tiles_before + nt - 1);
        tiles_before += nt + lead;
        k0 = t0 * kKeyTile;
        k1 = min(Tk, t1 * kKeyTile);
        if (t0 >= t1) {   // (cannot happen for b_first .. b_last; keeps a wrong split index out of the workspace)
            dma_wait_keep<0>();
            continue;
        }
        split = slot - s_first;
        direct = s_first == s_last;
        // the workgroup of kv head 0 and row tile 0 that holds the sequence's first tile tells the merge how many runs the
        // sequence fell into (the run boundaries are the same for every kv head and row tile)
        if (slot == s_first && hk == 0 && rt == 0 && tid == 0) a.seq_splits[b] = direct ? 0 : s_last - s_first + 1;
        k0 = uni(k0); k1 = uni(k1); split = uni(split); L = uni(L);
        direct = uni(direct) != 0;
    }
    [&]() {   // one segment; wavefronts that have nothing more to do leave through `return`

    if (k0 >= k1) {  // empty split (uniform over the workgroup): mark the partials as absent
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            if (rg_of[rb] >= 0 && g2 == 0 && kh == 0) {
                a.part_rec[(int64_t)split * a.rows_total + rg_of[rb]] = make_float3(-INFINITY, 0.f, 1.f);
            }
        dma_wait_keep<0>();   // (the rows of Q still on their way belong to nobody)
        return;
    }

    // ancestor bitmasks of the nodes this workgroup's rows belong to
    const int aw = (a.N + 31) >> 5;
    const int i_first = row_base / a.G;
    const int i_last = min(R - 1, row_base + RW - 1) / a.G;
    const bool has_tree_keys = k1 > L;  // uniform over the workgroup
    int32_t* parent_s = parents_at();

    // slab bases of this (sequence, kv head): wave-uniform, pinned to scalar registers
    constexpr int EB = KV8 ? 1 : 2;  // bytes of a stored K/V element
    auto uniform_ptr = [](const unsigned char* p) {
        const uint64_t v = (uint64_t)p;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return reinterpret_cast<const unsigned char*>(((uint64_t)hi << 32) | lo);
    };
    const unsigned char* kc = uniform_ptr(static_cast<const unsigned char*>(a.k_cache) + ((int64_t)b * a.cap * a.Hkv + hk) * (DH * EB));
    const unsigned char* vc = uniform_ptr(static_cast<const unsigned char*>(a.v_cache) + ((int64_t)b * a.cap * a.Hkv + hk) * (DH * EB));
    const unsigned char* kt = uniform_ptr(static_cast<const unsigned char*>(a.k_tree) + ((int64_t)b * a.N * a.Hkv + hk) * (DH * EB));
    const unsigned char* vt = uniform_ptr(static_cast<const unsigned char*>(a.v_tree) + ((int64_t)b * a.N * a.Hkv + hk) * (DH * EB));

    const int clean_end = min(L, k1);   // tiles that end here or earlier hold cache rows only
    // Direct-to-LDS tile fill: wave-instruction `inst` brings rows RPI*inst .. RPI*inst+RPI-1 of the tile;
    // lane l lands at byte 1024*inst + 16*l, i.e. row RPI*inst + l/SLOTS, slot' = l%SLOTS, and therefore
    // fetches the slot that the row's permutation maps there.  Rows past the end of the split fetch
    // the split's last key again: their scores are masked, and their V rows are finite, so that a
    // zero weight times them stays zero.  Every filling wavefront issues exactly PT loads per tile.
    const uint32_t k_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)k_s;  // LDS byte addresses
    const uint32_t v_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)v_s;
    // Addresses are a wave-uniform 64-bit base (one sequence's K or V slab) plus a 32-bit byte offset;
    // the host checks that a slab stays below 4 GiB.
    const uint32_t tok_bytes = (uint32_t)a.Hkv * DH * EB;
    // Per-lane byte offsets of this wavefront's loads inside a tile of cache rows.  Its wave-instructions are STEP rows apart,
    // a multiple of the permutations' period or (two filling wavefronts) of half of it.
    constexpr int FPW = (KT / RPI) / FILLERS;  // wave-instructions per filling wavefront, tile and tensor
    constexpr int STEP = RPI * FILLERS, NPAT = STEP % SLOTS == 0 ? 1 : 2;
    static_assert(STEP * NPAT % SLOTS == 0 && FPW % NPAT == 0, "the offsets repeat");
    uint32_t fill_k[NPAT], fill_v[NPAT];
#pragma unroll
    for (int it = 0; it < NPAT; ++it) {
        const int row = RPI * wave + it * STEP + lane / SLOTS;
        const int slotp = lane % SLOTS;
        fill_k[it] = (uint32_t)row * tok_bytes + 16 * (slotp ^ (row & (SLOTS - 1)));
        fill_v[it] = (uint32_t)row * tok_bytes + 16 * (slotp ^ ((row & (NDB - 1)) << 2));
    }
    // loads FROM .. TO-1 of the tile's PT: load i brings rows of wave-instruction i/2, of K (even) or V (odd)
    auto fill_loads = [&](auto from, auto to, int buf, int tile_base, auto known_clean) __attribute__((always_inline)) {
        constexpr int FROM = decltype(from)::value, TO = decltype(to)::value;
        if (FILLERS < NW && wave >= FILLERS) return;
        const uint32_t dst0 = buf * TILEB + wave * 1024;
        if (known_clean || tile_base + KT <= clean_end) {  // a whole tile of cache rows: the tile's base joins the scalar
            // pointer, the per-lane offsets are constants of the kernel (no vector arithmetic per load)
            const uint32_t dst = __builtin_amdgcn_readfirstlane(k_lds + dst0);
            static_for<FROM, TO>([&](auto i) {
                constexpr int it = decltype(i)::value / 2;
                constexpr bool is_v = decltype(i)::value % 2 != 0;
                const size_t off = (size_t)((uint32_t)(tile_base + it / NPAT * NPAT * STEP) * tok_bytes);
                dma_load16<NT, (is_v ? NBUF * TILEB : 0) + it * FILLERS * 1024>(uniform_ptr((is_v ? vc : kc) + off),
                                                                                is_v ? fill_v[it % NPAT] : fill_k[it % NPAT], dst);
            });
        } else if (tile_base < k1) {
            static_for<FROM, TO>([&](auto i) {
                constexpr int it = decltype(i)::value / 2;
                constexpr bool is_v = decltype(i)::value % 2 != 0;
                const int row = RPI * (wave + it * FILLERS) + lane / SLOTS;
                const int slotp = lane % SLOTS;
                const int j = min(tile_base + row, k1 - 1);
                const bool in_cache = j < L;             // rows of cache and tree by lane: no branches
                const uint32_t off = (uint32_t)(in_cache ? j : j - L) * tok_bytes;
                const unsigned char* base = is_v ? (in_cache ? vc : vt) : (in_cache ? kc : kt);
                dma_load16_flat<NT>(base + off + 16 * (is_v ? slotp ^ ((row & (NDB - 1)) << 2) : slotp ^ (row & (SLOTS - 1))),
                                    __builtin_amdgcn_readfirstlane((is_v ? v_lds : k_lds) + dst0 + it * FILLERS * 1024));
            });
        }
    };
    auto fill_tile = [&](int buf, int tile_base) { fill_loads(IntC<0>{}, IntC<PT>{}, buf, tile_base, std::false_type{}); };

    // KV8 loaders.  A tile is 16 wave-instructions of 16-byte loads: instruction g < 8 covers rows
    // 8g .. 8g+7 of K, instruction 8 + g the same rows of V, eight lanes per row and sixteen codes per
    // lane.  Loader lw takes instructions lw, lw + NLD, ... (NLD divides 8, so whether a load is K's or
    // V's is known at compile time).  Rows past the end of the split repeat
    // its last key, as above; every address is a cache row below L or a tree row below N whatever
    // tile_base is, so a load may be issued for a tile that does not exist.
    constexpr int LPT = 16 / (NLD > 0 ? NLD : 16);  // loads per loader and tile
    struct Stage {
        u32x4 d[LPT];
    };
    const int lw = wave - NW;
    // per-lane constants of this loader's LPT loads: byte offset inside a tile of cache rows, and the
    // two LDS byte offsets (relative to buffer 0) its sixteen widened values go to
    uint32_t ld_off[LPT], st_off0[LPT], st_off1[LPT];
#pragma unroll
    for (int it = 0; it < LPT; ++it) {
        const bool is_v = it * NLD >= 8;  // known once the loop is unrolled
        const int row = 8 * ((lw + it * NLD) & 7) + (lane >> 3);
        const int c2 = 2 * (lane & 7);    // this lane's two 16-byte slots: c2, c2 + 1
        const int x = is_v ? ((row & 3) << 2) : (row & 15);
        ld_off[it] = (uint32_t)row * tok_bytes + 16 * (lane & 7);
        st_off0[it] = (is_v ? NBUF * TILEB : 0) + row * ROWB + 16 * (c2 ^ x);
        st_off1[it] = (is_v ? NBUF * TILEB : 0) + row * ROWB + 16 * ((c2 + 1) ^ x);
    }
    const int cache_end = min(L, k1);
    auto stage_issue = [&](Stage& sg, int tile_base) {
        if (tile_base + KT <= cache_end) {  // a whole tile of cache rows: uniform base + constant per-lane offsets
            const uint64_t kb = (uint64_t)kc + (uint64_t)((uint32_t)tile_base * tok_bytes);
            const uint64_t vb = (uint64_t)vc + (uint64_t)((uint32_t)tile_base * tok_bytes);
#pragma unroll
            for (int it = 0; it < LPT; ++it) sg.d[it] = global_load16((it * NLD >= 8 ? vb : kb) + ld_off[it]);
            return;
        }
#pragma unroll
        for (int it = 0; it < LPT; ++it) {
            const bool is_v = it * NLD >= 8;
            const int row = 8 * ((lw + it * NLD) & 7) + (lane >> 3);
            const int j = min(tile_base + row, k1 - 1);
            const bool in_cache = j < L;
            const uint32_t off = (uint32_t)(in_cache ? j : j - L) * tok_bytes + 16 * (lane & 7);
            const uint64_t base = is_v ? (in_cache ? (uint64_t)vc : (uint64_t)vt) : (in_cache ? (uint64_t)kc : (uint64_t)kt);
            sg.d[it] = global_load16(base + off);
        }
    };
    // widens the staged codes and stores them where the direct-to-LDS path would have put the bf16 row
    auto stage_write = [&](const Stage& sg, int buf) {
        unsigned char* base = smem + buf * TILEB;
#pragma unroll
        for (int it = 0; it < LPT; ++it) {
            uint4 w0, w1;
            e4m3x16_to_bf16(sg.d[it], w0, w1);
            *reinterpret_cast<uint4*>(base + st_off0[it]) = w0;
            *reinterpret_cast<uint4*>(base + st_off1[it]) = w1;
        }
    };

    f32x16 o[RB][NDB];
    float m_ref[RB], l_run[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        m_ref[rb] = -INFINITY;
        l_run[rb] = 0.f;
#pragma unroll
        for (int db = 0; db < NDB; ++db) o[rb][db] = f32x16{};
    }
    // KV8: K = k_scale * code value, so the scale (positive) joins the softmax scale
    const float c_scale = a.scale * kLog2e * (KV8 ? a.k_scale[hk] : 1.f);

    // ---- the pipeline over 32-key blocks ---------------------------------------------------------
    // Each wavefront alternates between a vector phase (LDS operand reads issued, then the softmax
    // of block j) and a matrix phase (O^T += V^T.P^T of block j, then S^T of block j+1), so that the
    // two wavefronts resident on a SIMD keep its matrix pipe and its vector pipe busy in turn.
    //
    // Softmax uses a per-row reference m_ref, set at the first block in which the row sees a key and
    // raised only when a block's weights p = 2^(x - m_ref) sum to more than kWeightSumLimit: floating
    // point keeps the relative precision of the weights (bf16) and of the sums (fp32) whatever their
    // magnitude, so the common path takes no row maximum at all, and O and l -- which carry the same
    // reference -- are rescaled only in that rare, wave-uniform branch.  Scores far below the
    // reference underflow to weight 0, which is what they are worth next to the key that set it.  The
    // result O / l and lse = m_ref ln 2 + ln l do not depend on the reference.
    const int j16 = lane & 15;
    // K operand of step s: row n, slot 2s+g2 -> slot' = (2s+g2) ^ (n % SLOTS) = 2*(s ^ (n % SLOTS)>>1) + (g2 ^ (n&1))
    const int k_lane_off = n * ROWB + 16 * (g2 ^ (n & 1));
    const int k_pair_xor = ((n & (SLOTS - 1)) >> 1) << 5;
    // V operand: row z = 4*g2 + j16/4 (+ multiples of 8), 32-byte pair 2*db + (lane/16)%2 -> pair' = pair ^ 2*(z % NDB)
    const int v_z = 4 * g2 + (j16 >> 2);
    const int v_lane_off = v_z * ROWB + 8 * (j16 & 3);
    const int v_pair = (lane >> 4) & 1;
    const int v_px = (v_z & (NDB - 1)) << 1;

    auto read_k = [&](int buf, int kb, bf16x8 (&ka)[NS]) {
        const unsigned char* kbuf = k_s + buf * TILEB + kb * 32 * ROWB + k_lane_off;
#pragma unroll
        for (int s = 0; s < NS; ++s) ka[s] = *reinterpret_cast<const bf16x8*>(kbuf + ((32 * s) ^ k_pair_xor));
    };
    // lane j of a 16-lane group addresses key row (j/4), dh 4*(j%4); the transpose read hands each
    // lane four keys of one dh, i.e. the A operand of O^T += V^T.P^T
    auto read_v = [&](int buf, int kb, i16x8 (&va)[NDB][2]) {
        const unsigned char* vbuf = v_s + buf * TILEB + kb * 32 * ROWB + v_lane_off;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int m2 = 0; m2 < 2; ++m2) {
                const unsigned char* p = vbuf + (16 * m2) * ROWB + 32 * ((2 * db + v_pair) ^ v_px);
                const i16x4 lo = lds_read_tr16(p);
                const i16x4 hi = lds_read_tr16(p + 8 * ROWB);
                va[db][m2] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
    };
    auto qk = [&](const bf16x8 (&ka)[NS], f32x16 (&st)[RB]) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) st[rb] = f32x16{};
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                st[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s], qreg[rb][s], st[rb], 0, 0, 0);
    };
    auto pv = [&](const i16x8 (&va)[NDB][2], const i16x8 (&pb)[RB][2]) {
#pragma unroll
        for (int m2 = 0; m2 < 2; ++m2)
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    o[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8, va[db][m2]), __builtin_bit_cast(bf16x8, pb[rb][m2]), o[rb][db], 0, 0, 0);
    };
    auto block_max = [](const f32x16& x) {
        float m = x[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) m = fmaxf(m, x[v]);
        return m;
    };
    // blk0 = first key of the 32-key block; clean = the block's tile lies wholly inside the prefix.  (The mask's words read in front of
    // the operands, so that the wait for them does not await these, with the mask formed there: us per call in the shapes without
    // pairs, 24 sequences of 63 tokens, 208 rows on 40 kv heads 90.6 -> 92.4, 8 of 500 to 4096, 804 rows on 8 of head_dim 64 67.8 -> 68.3,
    // two of 3000, 1284 rows on 8 55.2 -> 56.1, three of up to 1531, 144 rows on 8 16.1 -> 16.2.)
    auto softmax = [&](f32x16 (&st)[RB], i16x8 (&pb)[RB][2], int blk0, bool clean) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (__builtin_expect(!clean, 0)) {
                uint32_t okmask = 0xffffffffu;  // bit u: key u of this block is visible to this lane's row
                const int bt = blk0 - L;        // tree-node index of the block's first key (negative inside the prefix)
                const uint32_t* w = anc_s + (node_of[rb] - i_first) * aw;
                if (bt >= 0) {
                    const int wi = bt >> 5;
                    const uint64_t w0 = wi < aw ? w[wi] : 0u;
                    const uint64_t w1 = wi + 1 < aw ? w[wi + 1] : 0u;
                    okmask = (uint32_t)(((w1 << 32) | w0) >> (bt & 31));
                } else if (bt > -32) {          // block straddles the end of the prefix
                    okmask = (0xffffffffu >> (32 + bt)) | (w[0] << (-bt));
                }
                const int left = k1 - blk0;     // keys of this block inside the split
                if (left < 32) okmask &= left <= 0 ? 0u : (0xffffffffu >> (32 - left));
                okmask >>= 4 * g2;  // this half-lane's keys are now bits 8*(v/4) + v%4
#pragma unroll
                for (int v = 0; v < 16; ++v) {   // (two instructions a key)
                    const uint32_t see = (uint32_t)__builtin_amdgcn_sbfe((int)okmask, 8 * (v >> 2) + (v & 3), 1);
                    st[rb][v] = __uint_as_float((see & __float_as_uint(st[rb][v])) | (~see & 0xff800000u));
                }
            }
            // weights of this lane's 16 keys relative to the reference ms, packed for the P.V product; returns their sum
            auto weights = [&](float ms) __attribute__((always_inline)) {
                float ps = 0.f;
#pragma unroll
                for (int m2 = 0; m2 < 2; ++m2) {
                    union { bf16x2 h[4]; i16x8 v; } pk;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float p0 = __builtin_amdgcn_exp2f(fmaf(st[rb][8 * m2 + 2 * e], c_scale, -ms));
                        const float p1 = __builtin_amdgcn_exp2f(fmaf(st[rb][8 * m2 + 2 * e + 1], c_scale, -ms));
                        ps += p0;
                        ps += p1;
                        const f32x2 pr = {p0, p1};
                        pk.h[e] = __builtin_convertvector(pr, bf16x2);  // v_cvt_pk_bf16_f32, round to nearest even
                    }
                    pb[rb][m2] = pk.v;
                }
                return ps;
            };
            // Common case: the row has a reference and no weight comes out large -- no maximum is taken at all.  A row
            // without a reference yet makes its sum infinite or NaN and so takes the other branch as well.
            float ps = weights(m_ref[rb]);
            if (__builtin_expect(__any(!(ps <= kWeightSumLimit)), 0)) {
                // Rare, wave-uniform: set or raise the reference from the block's row maxima, rescale what has been summed.
                const float mt = block_max(st[rb]) * c_scale;  // c_scale > 0: the maximum commutes with the scaling
                const float row_max = fmaxf(mt, __shfl_xor(mt, 32));
                const bool raise = row_max > m_ref[rb] + kRescaleGap;  // same answer in both half-lanes of a row
                const float alpha = raise ? __builtin_amdgcn_exp2f(m_ref[rb] - row_max) : 1.f;
                if (raise) m_ref[rb] = row_max;
                l_run[rb] *= alpha;
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[rb][db][v] *= alpha;
                ps = weights(m_ref[rb] == -INFINITY ? 0.f : m_ref[rb]);  // the scores are still in st
            }
            l_run[rb] += ps;
        }
    };

    static_assert(KT == 64, "the block pipeline below is written for two 32-key blocks per tile");
    const int ntiles = (k1 - k0 + KT - 1) / KT;
    // Every wavefront of the workgroup takes part, behind the barrier that publishes the parents.  The time is a chain of one LDS
    // read per ancestor: the bits go out as atomics that nothing waits for, and there is a branch to every three steps (depth 8:
    // 1.35 -> 0.85 us).
    auto build_masks = [&]() {
        for (int t = tid; t <= i_last - i_first; t += THREADS) {
            uint32_t* w = anc_s + t * aw;
            for (int x = 0; x < aw; ++x) w[x] = 0;
            // (three steps to a check; behind the root, as behind a parent that is no node, a lane goes on and sets no bit)
            int c = i_first + t;
            for (int guard = 0; guard < a.N && __any(c >= 0); guard += 3)
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    const int at = min(max(c, 0), a.N - 1);
                    const uint32_t bit = (uint32_t)c < (uint32_t)a.N ? 1u << (at & 31) : 0u;
                    c = bit ? parent_s[at] : -1;
                    __hip_atomic_fetch_or(w + (at >> 5), bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
        }
    };

    // KV8, loading wavefronts.  Tile tau travels in register set tau % NSET; iteration t (after the
    // barrier that retires tile t) stores tile t+3 into tile t's buffer and reuses the set for the
    // loads of tile t+3+NSET.  Every staged load is issued whether or not its tile exists: the
    // number of loads in flight at each point is then the same on every path, and the compiler's
    // wait for one register set leaves the NSET-1 younger sets in flight.  The barriers match those
    // of the computing wavefronts one for one.
    if constexpr (KV8) {
        if (is_loader) {
            Stage stage[NSET];
            static_for<0, NSET>([&](auto i) { stage_issue(stage[i.value], k0 + i.value * KT); });
            if (has_tree_keys) {
                lds_barrier();   // the computing wavefronts have the parents in LDS
                build_masks();
            }
            static_for<0, 3>([&](auto i) {
                stage_write(stage[i.value], i.value);
                stage_issue(stage[i.value], k0 + (NSET + i.value) * KT);
            });
            lds_barrier();  // tiles 0..2 are in LDS for everybody; anc_s published
            int lbuf = 0;
            auto lstep = [&](int t, Stage& sg) {
                lds_barrier();
                if (t + 3 < ntiles) stage_write(sg, lbuf);
                stage_issue(sg, k0 + (t + 3 + NSET) * KT);
                lbuf = lbuf + 1 == NBUF ? 0 : lbuf + 1;
            };
            int t = 0;
            for (; t + NSET - 1 < ntiles; t += NSET)
                static_for<0, NSET>([&](auto i) { lstep(t + i.value, stage[(i.value + 3) % NSET]); });
            static_for<0, NSET - 1>([&](auto i) {
                if (t + i.value < ntiles) lstep(t + i.value, stage[(i.value + 3) % NSET]);
            });
            if constexpr (KS == 2) {  // the merge of the key shares has two more workgroup barriers, and one for partial rows
                __syncthreads();
                __syncthreads();
                if (!direct) __syncthreads();
            }
            return;
        }
    }

    // prologue of the computing wavefronts: behind Q the parents and two tiles go into flight at once (direct-to-LDS path);
    // meanwhile Q is read back and the ancestor masks are built; the barrier that publishes tile 0 also says that all of Q
    // has left the buffer that tile 2 is then requested into
    if constexpr (!kParentsFirst) {
        if (has_tree_keys) fetch_parents(parent_s);
    }
    if constexpr (!KV8) {
        fill_tile(0, k0);
        if (ntiles > 1) fill_tile(1, k0 + KT);
    }
    auto wait_tiles_out = [&](bool both) {   // until at most the last one or both of the two tiles are out
        if (KV8 || (FILLERS < NW && wave >= FILLERS)) dma_wait_keep<0>();
        else if (both) dma_wait_keep<2 * PT>();
        else dma_wait_keep<PT>();
    };
    if constexpr (!KV8) {
        wait_tiles_out(ntiles > 1);
        if constexpr (QSHARED) lds_barrier();   // the other wavefront's rows of Q, and the parents
        const int nq = min(n, q_last);
        const unsigned char* qp = q_s + nq * ROWB + 16 * (g2 ^ (nq & 1));
        const int pair_xor = ((nq & (SLOTS - 1)) >> 1) << 5;
#pragma unroll
        for (int s = 0; s < NS; ++s) qreg[0][s] = *reinterpret_cast<const bf16x8*>(qp + ((32 * s) ^ pair_xor));
    }
    // (Built in the iteration before they are needed, in the shapes of four wavefronts: no gain over 27 calls, and 12 heads of 64, 64 rows x
    // 10258 tokens 14.3 -> 14.9 us per call.)
    if (has_tree_keys) {
        if constexpr (KV8) dma_wait_keep<0>();
        if constexpr (!QSHARED) lds_barrier();
        build_masks();
    }
    if constexpr (!KV8) {
        if (ntiles > 1) wait_tiles_out(false); else dma_wait_keep<0>();
    }
    lds_barrier();  // tile 0 has landed for everybody, anc_s is published, Q is read
    if constexpr (!KV8) {
        if (ntiles > 2) fill_tile(2, k0 + 2 * KT);
    }

    // The barrier of iteration t publishes tile t+1 and frees a buffer for tile t+3: that of tile t (three buffers: every
    // wavefront has read it) or of tile t-1 (four buffers, PING: a wavefront may meet the barrier anywhere in iteration t).
    // The new tile comes by direct-to-LDS loads that the barrier of iteration t+2 awaits, or (KV8) from the loaders.
    auto turn = [&](int t, int buf, int tile_base) {
        if constexpr (KV8) {
            lds_barrier();
        } else {
            if (t + 2 < ntiles) dma_wait_keep<PT>(); else dma_wait_keep<0>();  // tile t+1 landed, t+2 may be in flight
            lds_barrier();
            if (t + 3 < ntiles) fill_tile(buf, tile_base + 3 * KT);
        }
    };
    // PING: the barrier alone.  The loads of a tile are dealt out over the two matrix phases of an iteration instead (half 0
    // in that of block 1 of iteration t, half 1 in that of block 0 of iteration t+1): all at once they queue up in front of
    // the address unit, and the wavefronts stand behind them.
    auto await_tile = [&](int t, bool late_, bool steady_) {   // tile t+1; a late wavefront is here before its second half of tile t+2
        if (steady_ || t + 2 < ntiles) {
            if (late_) dma_wait_keep<PT / 2>(); else dma_wait_keep<PT>();
        } else {
            dma_wait_keep<0>();
        }
    };
    // No fence: what a wavefront has read from the freed buffer it consumed long ago, and LDS reads of its own that are still
    // out need not be awaited here.
    auto step = [] { asm volatile("s_barrier" ::: "memory"); };

    bf16x8 ka[NS];
    i16x8 va[NDB][2];
    f32x16 st[RB];
    i16x8 pb[RB][2];
    // Tile t lives in buffer t % NBUF.  The loop is unrolled NBUF-fold with the buffer index a compile-time constant (PING:
    // but for the first tile and the last ones), so that every LDS operand address is a loop-invariant per-lane register
    // plus an immediate (no address arithmetic per block).
    // A wavefront whose 32 rows all lie beyond the last query row (the padding of the last row tile) only keeps the
    // barriers and its share of the tile fills company: its matrix and vector work would be spent on repeats of the last
    // row, and what it does not burn the others get back as clock (392 rows per kv head, a ragged batch of 16: 3 of 16
    // wavefronts per K/V stream, call 172.4 -> 165.9 us).
    // Wavefronts 0 to 4 always work, so that one SIMD keeps its pair and the workgroup keeps the pace of the other row
    // tiles of its K/V stream: a workgroup that runs ahead of them fetches every tile from HBM a second time (1284 rows x
    // 32768 keys with all seven idle wavefronts of the last row tile skipping: 221 MB fetched per launch instead of 149).
    // The six-wavefront shape measured 1.5 % slower with the branch.
    // (With opposite phases it takes the branch as well: without a condition in the loop the compiler moves every buffer's addresses in
    // front of it and spills 464 registers.)
    constexpr bool kSkipIdle = (NW == 8 && KS == 1) || PING;
    const bool has_rows = !kSkipIdle || wave <= 4 || __builtin_amdgcn_readfirstlane((int)(row_base + wrow * RB * 32 < R)) != 0;
    // PING: matrix and vector instructions of different wavefronts run side by side, but two wavefronts that want the same
    // pipe get it one after the other, the older one first even if the younger is half through its phase: a pair that meets
    // at one barrier per tile stays in step and takes turns at everything (3479 cycles per tile of 64 keys x 256 rows, of
    // which the matrix pipe is busy 2262).  So the pair of a SIMD (wavefronts w and w + 4) is held in opposite phases: a
    // barrier between any two phases, the later wavefront one phase behind.  2755 cycles per tile that way, 2660 with the
    // conditions of the first and last tiles out of the loop (1284 rows x 32768 keys on 8 kv heads: 197 -> 182 us).  The
    // shape of four wavefronts keeps one barrier per tile, as each is alone on its SIMD; that of six, where two SIMDs have a pair and
    // set the pace, takes the phases too (516 rows x 8192 keys on 8 kv heads 33.0 -> 31.3 us per call, 129 x 4096 on 40 31.7 -> 29.9).
    const bool late = PING && wave >= 4;
    auto interleave_reads = [&]() {   // two LDS reads behind each of the NS matrix instructions
        static_for<0, NS>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2 * NDB * 2 / NS, 0);
        });
    };
    auto body = [&](int t, auto bufc, auto steady) __attribute__((always_inline)) {
        constexpr bool STEADY = decltype(steady)::value;   // PING: tiles t .. t+3 are whole tiles of cache rows, t > 0
        const int buf = bufc;   // (a compile-time constant after inlining, but for PING's general body)
        const int buf_next = buf + 1 == NBUF ? 0 : buf + 1;
        const int tile_base = k0 + t * KT;
        const bool clean = STEADY || tile_base + KT <= clean_end;
        if (!has_rows) {
            if constexpr (PING) {   // (an early or late wavefront alike: its loads keep to the second barrier of four)
                if (!late) step();
                await_tile(t, false, STEADY);
                step();
                if (t + 3 < ntiles) fill_tile((buf + 3) % NBUF, tile_base + 3 * KT);
                step();
                step();
                if (late) step();
            } else {
                turn(t, buf, tile_base);
            }
            return;
        }
        if constexpr (PING) {
            const int buf_p2 = (buf + 2) % NBUF, buf_p3 = (buf + 3) % NBUF;   // buffers of tiles t+2 and t+3
            // Vector phase of block 0: the K operand of block 1 is requested, then the softmax.
            read_k(buf, 1, ka);
            __builtin_amdgcn_sched_barrier(0);
            softmax(st, pb, tile_base, clean);
            __builtin_amdgcn_sched_barrier(0);
            if (late) await_tile(t, true, STEADY);
            step();
            // Matrix phase: O += V.P of this block; once its V operand is consumed the next one's is requested, between the
            // matrix instructions of the next block's scores.
            pv(va, pb);
            __builtin_amdgcn_sched_barrier(0);
            if (STEADY || t > 0) fill_loads(IntC<PT / 2>{}, IntC<PT>{}, buf_p2, tile_base + 2 * KT, steady);   // (the first three tiles came before the loop)
            read_v(buf, 1, va);
            qk(ka, st);
            interleave_reads();
            __builtin_amdgcn_sched_barrier(0);
            // block 1 of the tile; the next tile is visible before its first operand is read
            if (!late) await_tile(t, false, STEADY);
            step();
            if (STEADY || t + 1 < ntiles) read_k(buf_next, 0, ka);
            __builtin_amdgcn_sched_barrier(0);
            softmax(st, pb, tile_base + 32, clean);
            __builtin_amdgcn_sched_barrier(0);
            step();
            pv(va, pb);
            __builtin_amdgcn_sched_barrier(0);
            fill_loads(IntC<0>{}, IntC<PT / 2>{}, buf_p3, tile_base + 3 * KT, steady);
            if (STEADY || t + 1 < ntiles) {
                read_v(buf_next, 0, va);
                qk(ka, st);
                interleave_reads();
            }
            __builtin_amdgcn_sched_barrier(0);
            step();
            return;
        } else if constexpr (KS == 1) {
            // block 0 of the tile
            read_v(buf, 0, va);
            __builtin_amdgcn_sched_barrier(0);
            softmax(st, pb, tile_base, clean);
            read_k(buf, 1, ka);
            __builtin_amdgcn_sched_barrier(0);
            pv(va, pb);
            qk(ka, st);
            __builtin_amdgcn_sched_barrier(0);
            // block 1 of the tile; the next tile becomes visible before its first K operand is read
            read_v(buf, 1, va);
            __builtin_amdgcn_sched_barrier(0);
            softmax(st, pb, tile_base + 32, clean);
        } else {
            read_v(buf, kh, va);
            __builtin_amdgcn_sched_barrier(0);
            softmax(st, pb, tile_base + 32 * kh, clean);
        }
        turn(t, buf, tile_base);
        if (t + 1 < ntiles) read_k(buf_next, kh, ka);
        __builtin_amdgcn_sched_barrier(0);
        pv(va, pb);
        if (t + 1 < ntiles) qk(ka, st);
        __builtin_amdgcn_sched_barrier(0);
    };
    if (has_rows) {
        read_k(0, kh, ka);
        if constexpr (PING) read_v(0, 0, va);
        qk(ka, st);
        // A first block of cache keys, which every row sees, sets the reference here: its row maxima, as the rare branch of the
        // softmax would take them, but without the weights that only find out that there is none yet and without rescaling an O of
        // zeros (49 rows x 1024 tokens on 32 kv heads 13.03 -> 12.87 us per call, 516 rows x 4096 on 8 23.8 -> 23.6).
        if (k0 + KT <= clean_end) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const float mt = block_max(st[rb]) * c_scale;
                m_ref[rb] = fmaxf(mt, __shfl_xor(mt, 32));
            }
        }
    }
    int t = 0;
    if (late) step();
    if constexpr (PING) {
        // The long middle part, where every tile touched is a whole tile of cache rows, carries no conditions and is unrolled
        // with the buffer index a compile-time constant; the first tile and the last ones share one general body.
        const int steady_end = (clean_end - k0) / KT - 3;   // (clean_end may lie below k0: then there is none)
        while (t < ntiles) {
            body(t, t % NBUF, std::false_type{});
            ++t;
            if (t != 1) continue;
            while (t < steady_end) {
                body(t, IntC<1>{}, std::true_type{});
                if (++t >= steady_end) break;
                body(t, IntC<2>{}, std::true_type{});
                if (++t >= steady_end) break;
                body(t, IntC<3>{}, std::true_type{});
                if (++t >= steady_end) break;
                body(t, IntC<0>{}, std::true_type{});
                ++t;
            }
        }
    } else {
        for (; t + NBUF <= ntiles; t += NBUF) static_for<0, NBUF>([&](auto i) { body(t + i.value, i, std::false_type{}); });
        static_for<0, NBUF - 1>([&](auto i) {
            if (t + i.value < ntiles) body(t + i.value, i, std::false_type{});
        });
    }
    if (PING && !late) step();
    // epilogue: lane (n, g2) holds, for its row, dh = 32 db + 8 (v/4) + 4 g2 + (v%4); finish writes the blocks db = FROM .. TO-1
    // (l_tot: the row's sum of weights; c: its largest magnitude)
    auto finish = [&](auto from, auto to, int rb, float l_tot, float c) __attribute__((always_inline)) {
        constexpr int FROM = decltype(from)::value, TO = decltype(to)::value;
        const float v_unit = KV8 ? a.v_scale[hk] : 1.f;  // KV8: V = v_scale * code value
        if (rg_of[rb] < 0) return;
        if (direct) {
            const float inv = v_unit / l_tot;
            uint16_t* op = static_cast<uint16_t*>(a.out) + (int64_t)rg_of[rb] * DH + 4 * g2;
#pragma unroll
            for (int db = FROM; db < TO; ++db)
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    uint2 w;
                    w.x = pack_bf16x2(o[rb][db][4 * vq] * inv, o[rb][db][4 * vq + 1] * inv);
                    w.y = pack_bf16x2(o[rb][db][4 * vq + 2] * inv, o[rb][db][4 * vq + 3] * inv);
                    *reinterpret_cast<uint2*>(op + 32 * db + 8 * vq) = w;
                }
            if (a.lse && g2 == 0 && FROM == 0) a.lse[rg_of[rb]] = m_ref[rb] * kLn2 + logf(l_tot);
        } else {
            // Partial outputs travel as fp16 relative to the row's largest magnitude c (kept in fp32 beside m and l):
            // half the traffic of fp32 here and in the merge, an error of at most 2^-12 c per element whatever the
            // range of V (bf16 partials would cost up to a whole bf16 ulp of the merged row, which outputs of
            // magnitude 4 cannot afford inside 2e-2).  Streaming stores: the partials are read once, by the merge,
            // and leaving them dirty in L2 only lengthens the write-back at the end of this kernel.
            c = fmaxf(c, 1e-30f);
            const float inv_c = 1.f / c;   // (v_rcp_f32 alone would give 0 for c above 2^126, whose reciprocal is subnormal)
            // The two lanes of a row hold alternating groups of four head_dim positions; swapping halves between them
            // (v_permlane32_swap) leaves each with eight consecutive ones, so a store covers 32 contiguous bytes of a row.
            _Float16* po = reinterpret_cast<_Float16*>(a.part_o) + ((int64_t)split * a.rows_total + rg_of[rb]) * DH + 8 * g2;
            u32x4 w[NDB][2];
#pragma unroll
            for (int db = FROM; db < TO; ++db)
#pragma unroll
                for (int vp = 0; vp < 2; ++vp) {
                    const f32x4 ve = {o[rb][db][8 * vp] * inv_c, o[rb][db][8 * vp + 1] * inv_c,
                                      o[rb][db][8 * vp + 2] * inv_c, o[rb][db][8 * vp + 3] * inv_c};
                    const f32x4 vo = {o[rb][db][8 * vp + 4] * inv_c, o[rb][db][8 * vp + 5] * inv_c,
                                      o[rb][db][8 * vp + 6] * inv_c, o[rb][db][8 * vp + 7] * inv_c};
                    const u32x2 he = __builtin_bit_cast(u32x2, __builtin_convertvector(ve, f16x4));
                    const u32x2 ho = __builtin_bit_cast(u32x2, __builtin_convertvector(vo, f16x4));
                    const auto s0 = __builtin_amdgcn_permlane32_swap(he[0], ho[0], false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(he[1], ho[1], false, false);
                    w[db][vp] = u32x4{s0[0], s1[0], s0[1], s1[1]};
                }
            // the stores of a row leave back to back: neighbouring 32-byte pieces then combine into whole lines
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int db = FROM; db < TO; ++db)
#pragma unroll
                for (int vp = 0; vp < 2; ++vp)
                    __builtin_nontemporal_store(w[db][vp], reinterpret_cast<u32x4*>(po + 32 * db + 16 * vp));
            __builtin_amdgcn_sched_barrier(0);
            if (g2 == 0 && FROM == 0)   // reference in base-2 units of the scaled scores; KV8: V = v_scale * code value
                a.part_rec[(int64_t)split * a.rows_total + rg_of[rb]] = make_float3(m_ref[rb], l_tot, c * v_unit);
        }
    };
    if constexpr (KS == 2) {
        // Merge of the two key shares of a row block.  Both carry O~ and l relative to their own reference m_ref.  Each
        // keeps one half of head_dim and hands the other over through the (now idle) tile buffers, lane for lane, with m and l;
        // both then rescale what they have of both shares to the larger reference and finish their
        // halves side by side (49 rows x 1024 tokens on 32 kv heads 12.9 -> 12.7 us per call).  Partial rows take a third barrier
        // (0.07 us of that call): their scale c comes from the merged values of both halves, because where the shares cancel each
        // other their own maxima say nothing about these.
        static_assert(RB == 1, "one row block to a pair");
        constexpr int HV = 8 * NDB;        // values of a lane's half
        constexpr int XR = HV + 3;
        float* const xch = reinterpret_cast<float*>(smem) + (wrow * 2 * XR) * 64 + lane;   // [wrow][share it is for][XR][64 lanes]
        __syncthreads();  // every wavefront is done with the tiles
        auto half = [&](auto h) __attribute__((always_inline)) {   // this wavefront keeps half h
            constexpr int H = decltype(h)::value;
            float* out = xch + (1 - H) * XR * 64;
            const float* in = xch + H * XR * 64;
#pragma unroll
            for (int x = 0; x < HV; ++x) out[x * 64] = o[0][(1 - H) * NDB / 2 + x / 16][x % 16];
            out[HV * 64] = m_ref[0];
            out[(HV + 1) * 64] = l_run[0];
            __syncthreads();
            const float m_other = in[HV * 64], l_other = in[(HV + 1) * 64];
            const float mm = fmaxf(m_ref[0], m_other);
            // a share that saw no visible key has m = -inf, l = 0, O~ = 0: weight 0 keeps it out
            const float w_own = m_ref[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_ref[0] - mm);
            const float w_other = m_other == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_other - mm);
            m_ref[0] = mm;
            auto both = [&](float own, float other) {   // rounded alike on both sides: share 1's product, then share 0's
                return H == 0 ? fmaf(own, w_own, other * w_other) : fmaf(other, w_other, own * w_own);
            };
            const float l_lane = both(l_run[0], l_other);
            const float l_tot = l_lane + __shfl_xor(l_lane, 32);
            float c = 0.f;
#pragma unroll
            for (int x = 0; x < HV; ++x) {
                const float y = both(o[0][H * NDB / 2 + x / 16][x % 16], in[x * 64]);
                o[0][H * NDB / 2 + x / 16][x % 16] = y;
                c = fmaxf(c, fabsf(y));
            }
            if (!direct) {
                c = fmaxf(c, __shfl_xor(c, 32));
                out[(HV + 2) * 64] = c;
                __syncthreads();
                c = fmaxf(c, in[(HV + 2) * 64]);
            }
            finish(IntC<H * NDB / 2>{}, IntC<(H + 1) * NDB / 2>{}, 0, l_tot, c);
        };
        if (kh == 0) half(IntC<0>{}); else half(IntC<1>{});
    } else {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const float l_tot = l_run[rb] + __shfl_xor(l_run[rb], 32);
            if (rg_of[rb] < 0) continue;
            float c = 0.f;
            if (!direct) {
                float rmax = 0.f;
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int v = 0; v < 16; ++v) rmax = fmaxf(rmax, fabsf(o[rb][db][v]));
                c = fmaxf(rmax, __shfl_xor(rmax, 32));
            }
            finish(IntC<0>{}, IntC<NDB>{}, rb, l_tot, c);
        }
    }
    }();   // one segment
    }      // segments of this workgroup
}

// Every variant's limit is raised to all the shared memory of a compute unit once per device.
constexpr size_t kMaxSmem = kAttnMfmaMaxSmem;

template <int NW, int RB, int KT, int KS, bool KV8, bool NT, bool BAL = false, int DHT = 128, bool PING = false>
hipError_t raise_variant() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(attn_mfma_kernel<NW, RB, KT, KS, KV8, NT, BAL, DHT, PING>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxSmem);
}

template <int NW, int RB, int KT, int KS, bool KV8, bool NT, bool BAL = false, int DHT = 128, bool PING = false>
hipError_t launch_variant(const AttnArgs& a, const AttnPlan& p, hipStream_t st) {
    // K/V streams, each read by p.row_tiles workgroups, which share an XCD (workgroups are dealt out to the XCDs in turn)
    const dim3 grid((unsigned)((a.S + 7) / 8 * 8 * p.row_tiles));
    const size_t smem = attn_mfma_smem(NW, KS, DHT, a.G, a.N);
    auto kern = attn_mfma_kernel<NW, RB, KT, KS, KV8, NT, BAL, DHT, PING>;
    const unsigned threads = (NW + (KV8 ? 4 : 0)) * 64;  // KV8: plus the four loading wavefronts
    if (a.Dh != DHT) return hipErrorInvalidValue;
    if (smem > kMaxSmem) return hipErrorInvalidValue;  // cannot happen for N <= 1024: checked again for the sake of the launch
    hipLaunchKernelGGL(kern, grid, dim3(threads), smem, st, a);
    return hipGetLastError();
}

template <int NW, int RB, int KT, int KS, bool KV8 = false, int DHT = 128>
hipError_t launch_cfg(const AttnArgs& a, const AttnPlan& p, hipStream_t st) {
    if constexpr (KV8) {
        if constexpr (KS == 1) {
            if (a.slots > 0) return launch_variant<NW, RB, KT, KS, true, false, true>(a, p, st);
        }
        if (a.slots > 0) return hipErrorInvalidValue;
        return launch_variant<NW, RB, KT, KS, true, false>(a, p, st);  // the loaders' register loads always stream
    } else {
        auto go = [&](auto bal, auto ping) {
            constexpr bool BAL = decltype(bal)::value, PING = decltype(ping)::value;
            return p.row_tiles == 1 ? launch_variant<NW, RB, KT, KS, false, true, BAL, DHT, PING>(a, p, st)
                                    : launch_variant<NW, RB, KT, KS, false, false, BAL, DHT, PING>(a, p, st);
        };
        if constexpr (KS == 1 && NW == 6 && DHT == 128) {
            if (p.phases && a.slots == 0) return go(std::false_type{}, std::true_type{});
        }
        if constexpr (KS == 1 && NW == 8) {
            if (p.phases) return a.slots > 0 ? go(std::true_type{}, std::true_type{}) : go(std::false_type{}, std::true_type{});
        }
        if constexpr (KS == 1) {
            if (a.slots > 0) return go(std::true_type{}, std::false_type{});
        }
        if (a.slots > 0 || p.phases) return hipErrorInvalidValue;
        return go(std::false_type{}, std::false_type{});
    }
}

// the six workgroup shapes of the bf16 kernel for one head_dim
template <int DHT>
hipError_t launch_shape(const AttnArgs& a, const AttnPlan& p, hipStream_t st) {
    switch (p.waves * 10 + p.kshares) {
        case 41: return launch_cfg<4, 1, 64, 1, false, DHT>(a, p, st);
        case 61: return launch_cfg<6, 1, 64, 1, false, DHT>(a, p, st);
        case 81: return launch_cfg<8, 1, 64, 1, false, DHT>(a, p, st);
        case 22: return launch_cfg<2, 1, 64, 2, false, DHT>(a, p, st);
        case 42: return launch_cfg<4, 1, 64, 2, false, DHT>(a, p, st);
        case 82: return launch_cfg<8, 1, 64, 2, false, DHT>(a, p, st);
        default: return hipErrorInvalidValue;
    }
}

template <int DHT>
hipError_t raise_shapes() {
    hipError_t e = hipSuccess;
    auto both = [&](auto nw, auto ks, auto ping) {
        constexpr int NW = decltype(nw)::value, KS = decltype(ks)::value;
        constexpr bool PING = decltype(ping)::value;
        if (e == hipSuccess) e = raise_variant<NW, 1, 64, KS, false, false, false, DHT, PING>();
        if (e == hipSuccess) e = raise_variant<NW, 1, 64, KS, false, true, false, DHT, PING>();
        if constexpr (KS == 1) {
            if (e == hipSuccess) e = raise_variant<NW, 1, 64, 1, false, false, true, DHT, PING>();
            if (e == hipSuccess) e = raise_variant<NW, 1, 64, 1, false, true, true, DHT, PING>();
        }
    };
    constexpr std::false_type no;
    both(IntC<4>{}, IntC<1>{}, no); both(IntC<6>{}, IntC<1>{}, no); both(IntC<8>{}, IntC<1>{}, no);
    both(IntC<8>{}, IntC<1>{}, std::true_type{});
    if constexpr (DHT == 128) {
        if (e == hipSuccess) e = raise_variant<6, 1, 64, 1, false, false, false, DHT, true>();
        if (e == hipSuccess) e = raise_variant<6, 1, 64, 1, false, true, false, DHT, true>();
    }
    both(IntC<2>{}, IntC<2>{}, no); both(IntC<4>{}, IntC<2>{}, no); both(IntC<8>{}, IntC<2>{}, no);
    return e;
}

}  // namespace

// Dynamic shared memory of a workgroup: three K and V tile buffers of 64 keys, space for the rows of Q that the spare buffers do not
// hold (as much as the fourth buffer of opposite phases, which then holds Q, in the shapes that may take them), the ancestor
// bitmasks of the nodes the rows belong to, and the parent table.
size_t attn_mfma_smem(int waves, int kshares, int head_dim, int group, int nodes) {
    const size_t tile = (size_t)64 * 2 * head_dim;
    const int rw = waves / kshares * 32;
    const int nodes_local = rw % group == 0 ? rw / group : (rw + group - 1) / group + 1;
    const int nbuf = 3, q_outside = waves == 6 && head_dim == 128 ? 4 : waves - 4 * (nbuf - 2);
    return 2 * nbuf * tile + (q_outside > 0 ? q_outside * tile / 2 : 0) +
           (size_t)nodes_local * ((nodes + 31) / 32) * 4 + (size_t)((nodes + 63) / 64) * 256;
}

hipError_t raise_limits_attn_mfma() {
    hipError_t e = raise_shapes<128>();
    if (e == hipSuccess) e = raise_shapes<64>();
    if (e == hipSuccess) e = raise_variant<2, 1, 64, 2, true, false>();
    if (e == hipSuccess) e = raise_variant<4, 1, 64, 2, true, false>();
    if (e == hipSuccess) e = raise_variant<4, 1, 64, 1, true, false>();
    if (e == hipSuccess) e = raise_variant<4, 1, 64, 1, true, false, true>();
    return e;
}

hipError_t launch_attn_mfma(const AttnArgs& a, const AttnPlan& p, hipStream_t st) {
    if (p.rblocks != 1) return hipErrorInvalidValue;
    if (a.k_scale || a.v_scale) {  // K/V held as E4M3 codes (head_dim 128)
        if (!a.k_scale || !a.v_scale || a.Dh != 128) return hipErrorInvalidValue;
        switch (p.waves * 10 + p.kshares) {  // computing wavefronts; four loaders on top
            case 22: return launch_cfg<2, 1, 64, 2, true>(a, p, st);
            case 42: return launch_cfg<4, 1, 64, 2, true>(a, p, st);
            case 41: return launch_cfg<4, 1, 64, 1, true>(a, p, st);
            default: return hipErrorInvalidValue;
        }
    }
    if (a.Dh == 128) return launch_shape<128>(a, p, st);
    if (a.Dh == 64) return launch_shape<64>(a, p, st);
    return hipErrorInvalidValue;
}

}  // namespace ygg
