// Tree-masked verify attention, fp32 vector-ALU path (paper Sec. 2 "Source of Improvements",
// Sec. 4.2 last paragraph: one parallel pass, mask = the tree's causal dependency), and the
// split-KV combine shared with the matrix-core path.
//
// One wavefront owns one query row (sequence b, node i, query head h) and one split of the key
// range.  Lanes split the keys of a 64-key tile for q.k (one key per lane), the tile's softmax
// statistics are wave reductions, and lanes split head_dim for the value product.  This path is
// exact fp32 throughout and serves the fp32 configuration and any shape the matrix-core kernel
// does not take; it is not the bandwidth path.
#include "attn_common.h"

#include <hip/hip_bf16.h>

#include <type_traits>

namespace ygg {
namespace {

using namespace attn;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;

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
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ void load4(const float* p, float (&o)[4]) {
        const float4 v = *reinterpret_cast<const float4*>(p);
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    }
    static __device__ __forceinline__ float load1(const float* p) { return *p; }
};
template <> struct Elem<uint16_t> {
    static __device__ __forceinline__ void load4(const uint16_t* p, float (&o)[4]) {
        const uint2 v = *reinterpret_cast<const uint2*>(p);
        o[0] = bf16_bits_to_f32(v.x & 0xffffu); o[1] = bf16_bits_to_f32(v.x >> 16);
        o[2] = bf16_bits_to_f32(v.y & 0xffffu); o[3] = bf16_bits_to_f32(v.y >> 16);
    }
    static __device__ __forceinline__ float load1(const uint16_t* p) { return bf16_bits_to_f32(*p); }
};

template <typename T, int DH>
__global__ __launch_bounds__(256) void attn_vector_kernel(AttnArgs a) {
    constexpr int EPL = DH / 64;  // head_dim elements per lane in the value product
    __shared__ float q_s[4][DH];
    __shared__ uint32_t anc_s[4][kMaxNodes / 32];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t rows = (int64_t)a.B * a.N * a.Hq;
    const int64_t r = (int64_t)blockIdx.x * 4 + wave;
    if (r >= rows) return;  // no barrier below: waves are independent
    const int split = blockIdx.y;
    const int h = (int)(r % a.Hq), i = (int)((r / a.Hq) % a.N), b = (int)(r / ((int64_t)a.Hq * a.N));
    const int hk = h / a.G;
    int L = a.seq_lens[b];
    L = L < 0 ? 0 : (L > a.max_seq_len ? a.max_seq_len : L);
    const int Tk = L + a.N;  // keys of this sequence
    int chunk = (Tk + a.nsplit - 1) / a.nsplit;
    chunk = (chunk + kKeyTile - 1) / kKeyTile * kKeyTile;
    const int k0 = split * chunk;
    const int k1 = min(Tk, k0 + chunk);

    const T* qp = static_cast<const T*>(a.q) + r * DH;
    for (int d = lane; d < DH; d += 64) q_s[wave][d] = Elem<T>::load1(qp + d);
    const int32_t* parent = a.parent_idx + (int64_t)b * a.N;
    if (k1 > L) {  // this split touches tree keys: bitmask of {i, parent[i], ..., root}
        for (int w = lane; w < (a.N + 31) / 32; w += 64) anc_s[wave][w] = 0;
        __builtin_amdgcn_wave_barrier();
        int guard = 0;
        for (int t = i; t >= 0 && t < a.N && guard < a.N; t = parent[t], ++guard)
            if (lane == 0) anc_s[wave][t >> 5] |= 1u << (t & 31);
    }
    __builtin_amdgcn_wave_barrier();

    const T* kc = static_cast<const T*>(a.k_cache) + ((int64_t)b * a.cap * a.Hkv + hk) * DH;
    const T* vc = static_cast<const T*>(a.v_cache) + ((int64_t)b * a.cap * a.Hkv + hk) * DH;
    const T* kt = static_cast<const T*>(a.k_tree) + ((int64_t)b * a.N * a.Hkv + hk) * DH;
    const T* vt = static_cast<const T*>(a.v_tree) + ((int64_t)b * a.N * a.Hkv + hk) * DH;
    const int64_t tok_stride = (int64_t)a.Hkv * DH;

    float m = -INFINITY, l = 0.f, acc[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;

    for (int t0 = k0; t0 < k1; t0 += 64) {
        const int j = t0 + lane;
        bool ok = j < k1;
        if (ok && j >= L) ok = (anc_s[wave][(j - L) >> 5] >> ((j - L) & 31)) & 1u;
        float s = -INFINITY;
        if (ok) {
            const T* kp = j < L ? kc + (int64_t)j * tok_stride : kt + (int64_t)(j - L) * tok_stride;
            float dot = 0.f;
#pragma unroll 8
            for (int d = 0; d < DH; d += 4) {
                float kv[4];
                Elem<T>::load4(kp + d, kv);
                const float4 qv = *reinterpret_cast<const float4*>(&q_s[wave][d]);
                dot = fmaf(qv.x, kv[0], dot);
                dot = fmaf(qv.y, kv[1], dot);
                dot = fmaf(qv.z, kv[2], dot);
                dot = fmaf(qv.w, kv[3], dot);
            }
            s = dot * a.scale;
        }
        const float tmax = wave_max(s);
        if (tmax == -INFINITY) continue;  // nothing visible in this tile (wave-uniform)
        const float m_new = fmaxf(m, tmax);
        const float alpha = expf(m - m_new);  // m = -inf on the first live tile -> 0
        const float p = ok ? expf(s - m_new) : 0.f;
        l = l * alpha + wave_sum(p);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] *= alpha;
        m = m_new;

        if (t0 + 64 <= min(k1, L)) {  // whole tile inside the prefix: fixed trip count
#pragma unroll 16
            for (int jj = 0; jj < 64; ++jj) {
                const float pj = __shfl(p, jj);
                const T* vp = vc + (int64_t)(t0 + jj) * tok_stride + lane * EPL;
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[e] = fmaf(pj, Elem<T>::load1(vp + e), acc[e]);
            }
        } else {
            uint64_t live = __ballot(ok);
            while (live) {
                const int jj = __ffsll((unsigned long long)live) - 1;
                live &= live - 1;
                const float pj = __shfl(p, jj);
                const int key = t0 + jj;
                const T* vp = (key < L ? vc + (int64_t)key * tok_stride : vt + (int64_t)(key - L) * tok_stride) + lane * EPL;
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[e] = fmaf(pj, Elem<T>::load1(vp + e), acc[e]);
            }
        }
    }

    float* po = static_cast<float*>(a.part_o) + ((int64_t)split * rows + r) * DH + lane * EPL;
#pragma unroll
    for (int e = 0; e < EPL; ++e) po[e] = acc[e];
    if (lane == 0) a.part_rec[(int64_t)split * rows + r] = make_float3(m, l, 1.f);
}

// Merge of the per-split partials: m* = max_s m_s, l* = sum_s l_s e^{m_s - m*}, O = sum_s O~_s e^{m_s - m*} / l*,
// lse = m* + ln l*.  References come in the units that their kernel works in, so that their differences are exact: base-2
// ones from the matrix-core kernels (2^{m_s - m*}, m* ln 2), natural ones from the vector kernel.
// A group of TPR lanes covers a row with 16 bytes per lane (eight fp16 or four fp32 values); G such groups share one row,
// taking every G-th split each (G = 64 / TPR where there are few rows: a lane then has few loads to wait for; G = 2 for some more
// rows of more splits than a lane requests at once; else G = 1).
// The records {m, l, c} are read once per row -- lane t of the row's lanes takes splits t, t + LPR, .. -- and m*, the
// weights and l* are formed between them.  The kernel is one trip to memory: the first GS partial outputs are requested
// together with the records, whatever their weights turn out to be; an empty split (m = -inf) has weight 0 and its row,
// which was never written, is replaced by zeros.  Balanced batches: a sequence's splits are the runs its keys fell into,
// seq_splits[b] of them (a table the main kernel fills); 0 means one run held the whole sequence and its rows are final
// already.
//
// HALF: the partial outputs are the matrix-core kernels' (fp16, each row divided by its scale c): split s then enters with
// weight w_s c_s instead of w_s; the normaliser is the same.
template <typename T, int DH, bool HALF, int G>
__global__ __launch_bounds__(256) void attn_combine_kernel(AttnArgs a) {
    constexpr int EPL = HALF ? 8 : 4;     // values per lane
    constexpr int TPR = DH / EPL;         // lanes across a row: 8, 16 or 32
    constexpr int LPR = TPR * G;          // lanes of a row
    constexpr int GS = G == 1 || (G == 2 && HALF) ? 8 : 4;   // partial outputs in flight per lane
    constexpr int NH = 64 / LPR;          // records per lane: the host never plans more than 64 splits
    const int b = blockIdx.y;
    const int rows_seq = a.N * a.Hq;
    int nsp = a.nsplit;
    if (a.seq_splits) {  // balanced batches: the sequence's own number of runs; 0 = its rows are final already
        nsp = a.seq_splits[b];
        if (nsp == 0) return;
    }
    const int r_raw = blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
    const bool in_range = r_raw < rows_seq;   // lanes beyond the last row keep their group's exchanges company
    const int64_t r = (int64_t)b * rows_seq + (in_range ? r_raw : rows_seq - 1);
    const int64_t rows = a.rows_total;
    const int t = threadIdx.x % LPR, col = t % TPR, grp = t / TPR;
    const uint4* po = static_cast<const uint4*>(a.part_o) + r * TPR + col;   // split s: + s * rows * TPR

    float3 rec[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        rec[h] = make_float3(-INFINITY, 0.f, 1.f);
        if (h * LPR >= nsp) continue;
        const int sp = t + h * LPR;
        if (sp < nsp) rec[h] = a.part_rec[(int64_t)sp * rows + r];
    }
    uint4 raw[GS];
    auto request = [&](int s0) {   // splits s0 + grp, s0 + grp + G, ..
#pragma unroll
        for (int u = 0; u < GS; ++u) raw[u] = po[(int64_t)min(s0 + grp + u * G, nsp - 1) * rows * TPR];
    };
    request(0);

    float mstar = rec[0].x;
#pragma unroll
    for (int h = 1; h < NH; ++h) mstar = fmaxf(mstar, rec[h].x);
    mstar = group_reduce(mstar, LPR, [](float x, float y) { return fmaxf(x, y); });
    // a row always has a visible key (itself), so some split is live and mstar is finite
    float w[NH], lstar = 0.f;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        w[h] = rec[h].x == -INFINITY ? 0.f : HALF ? exp2f(rec[h].x - mstar) : expf(rec[h].x - mstar);
        lstar = fmaf(rec[h].y, w[h], lstar);
        w[h] = w[h] == 0.f ? 0.f : w[h] * rec[h].z;   // from here on w weighs the stored partial output
    }
    lstar = group_reduce(lstar, LPR, [](float x, float y) { return x + y; });

    float acc[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
    for (int s0 = 0; s0 < nsp; s0 += GS * G) {
        float ws[GS];
#pragma unroll
        for (int u = 0; u < GS; ++u) {   // weight of split s: lane s % LPR of the row's lanes, slot s / LPR
            const int s = s0 + grp + u * G;
            float wh = w[0];
#pragma unroll
            for (int h = 1; h < NH; ++h) wh = s / LPR == h ? w[h] : wh;
            ws[u] = __shfl(wh, s % LPR, LPR);
            if (s >= nsp) ws[u] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < GS; ++u) {
            const uint4 x = ws[u] != 0.f ? raw[u] : make_uint4(0, 0, 0, 0);
            const uint32_t d[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (HALF) {
                    const f16x2 h2 = __builtin_bit_cast(f16x2, d[e]);
                    acc[2 * e] = fmaf((float)h2[0], ws[u], acc[2 * e]);
                    acc[2 * e + 1] = fmaf((float)h2[1], ws[u], acc[2 * e + 1]);
                } else {
                    acc[e] = fmaf(__uint_as_float(d[e]), ws[u], acc[e]);
                }
            }
        }
        if (s0 + GS * G < nsp) request(s0 + GS * G);
    }
    if constexpr (G > 1) {   // the groups' shares of the sum
#pragma unroll
        for (int o = TPR; o < LPR; o <<= 1)
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
                const uint32_t u = __float_as_uint(acc[e]);
                float other[2];
                if (o == 8) {   // (within a row of 16 lanes)
                    other[0] = acc[e];
                    other[1] = __uint_as_float(row_xor<8>(u));
                } else {
                    const auto p = o == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false) : __builtin_amdgcn_permlane32_swap(u, u, false, false);
                    other[0] = __uint_as_float(p[0]);
                    other[1] = __uint_as_float(p[1]);
                }
                acc[e] = other[0] + other[1];
            }
    }
    if (!in_range || grp > 0) return;
    const float inv = 1.f / lstar;
    if constexpr (sizeof(T) == 4) {
        static_assert(!HALF, "fp32 outputs come from the vector kernel");
        *reinterpret_cast<float4*>(static_cast<float*>(a.out) + r * DH + EPL * col) =
            make_float4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
    } else {
        __hip_bfloat16 h[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) h[e] = __float2bfloat16(acc[e] * inv);  // round to nearest even
        uint16_t* dst = static_cast<uint16_t*>(a.out) + r * DH + EPL * col;
        if constexpr (HALF) *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<uint4*>(h);
        else *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<uint2*>(h);
    }
    if (a.lse && t == 0) a.lse[r] = (HALF ? mstar * kLn2 : mstar) + logf(lstar);
}

template <typename T>
hipError_t launch_vector_t(const AttnArgs& a, const AttnPlan& p, hipStream_t st) {
    const int64_t rows = (int64_t)a.B * a.N * a.Hq;
    dim3 grid((unsigned)((rows + 3) / 4), (unsigned)p.nsplit);
    if (a.Dh == 128) hipLaunchKernelGGL((attn_vector_kernel<T, 128>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((attn_vector_kernel<T, 64>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

template <typename T, bool HALF>
hipError_t launch_combine_t(const AttnArgs& a, hipStream_t st) {
    // up to four wavefronts' worth of rows per SIMD: a whole wavefront per row
    const bool few = a.rows_total <= 4096;
    auto go = [&](auto dh) {
        constexpr int DH = decltype(dh)::value, TPR = DH / (HALF ? 8 : 4);
        auto grid = [&](int lanes) { return dim3((unsigned)((a.N * a.Hq + 256 / lanes - 1) / (256 / lanes)), (unsigned)a.B); };
        // One trip to memory instead of two for nine to sixteen splits (the plan has no more for so many rows): 4128 rows of ten splits, us
        // per attention call with G = 1 -> 2, head_dim 128 23.1 -> 22.7, 64 37.0 -> 36.3.  Up to eight splits two groups only add an
        // exchange: 10272 rows of five 40.6 -> 42.5.
        if constexpr (HALF) {
            if (!few && a.nsplit > 8 && !a.seq_splits && a.rows_total <= 16384) {
                hipLaunchKernelGGL((attn_combine_kernel<T, DH, HALF, 2>), grid(2 * TPR), dim3(256), 0, st, a);
                return;
            }
        }
        if (few) hipLaunchKernelGGL((attn_combine_kernel<T, DH, HALF, 64 / TPR>), grid(64), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((attn_combine_kernel<T, DH, HALF, 1>), grid(TPR), dim3(256), 0, st, a);
    };
    if (a.Dh == 128) go(std::integral_constant<int, 128>{});
    else go(std::integral_constant<int, 64>{});
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_vector(const AttnArgs& a, const AttnPlan& p, int dtype, hipStream_t st) {
    return dtype == YGG_F32 ? launch_vector_t<float>(a, p, st) : launch_vector_t<uint16_t>(a, p, st);
}

hipError_t launch_attn_combine(const AttnArgs& a, const AttnPlan& p, int dtype, hipStream_t st) {
    if (p.use_mfma) return launch_combine_t<uint16_t, true>(a, st);
    return dtype == YGG_F32 ? launch_combine_t<float, false>(a, st) : launch_combine_t<uint16_t, false>(a, st);
}

}  // namespace ygg
