// spec.hip -- speculative sampling: the verification rule that keeps the
// target model's output distribution (Sec. 1 and Sec. 2.1 rely on it).
//
// At temperature tau, p_j = softmax(target row j / tau) and q_j =
// softmax(drafter row j / tau).  Drafted token x_j passes when
// u_j q_j(x_j) < p_j(x_j); after the first failure (position m) the next
// token is drawn by inversion from max(0, p_m - q_m), after k passes from p_k.
// Three launches, the kernel boundaries their only synchronisation:
//   stats:  per (row, chunk of 8192 logits) the max of x / tau and the sum of
//           e^(x / tau - max), for the target rows 0..k and drafter rows 0..k-1;
//   mass:   per (sequence, chunk) every row's chunks merged in a fixed tree,
//           lane j tests drafted token j, m = the first failure, and the mass of
//           the distribution drawn from (residual and plain target) in the
//           chunk, summed in a fixed order;
//   sample: per sequence, the chunk where the cumulative mass passes
//           u * total, then a scan of that chunk in index order.
// A call moves a few MB, so it is bound by its chain of dependent loads: the
// row merges and the decision are a few KB and are redone by every chunk's
// workgroup rather than given launches of their own, and the loads of a stage
// go out together (4 sequences of 6 drafted tokens, 128256-token vocabulary,
// bf16: 34.6 us of kernel time in five launches, 25.5 us in three).
// Everything is fp32.  The chunk masses and the in-chunk scan add in
// different orders; when rounding leaves the scan short of the target, the
// chunk's last element with mass is drawn.
#include "device_common.h"
#include "launch.h"
#include "logit_common.h"

namespace ssl {
namespace {

using lc::kLog2e;
using lc::kThreads;
constexpr int kWaves = kThreads / kWave;

// Row r of sequence b in the row tables: target rows 0..max_k, then drafter
// rows 0..max_k-1.
__device__ __forceinline__ const char* row_base(const SpecArgs& a, int b, int r, bool f32) {
    const size_t esz = f32 ? 4 : 2;
    if (r <= a.max_k)
        return static_cast<const char*>(a.tlogits) + ((size_t)b * (a.max_k + 1) + r) * a.row_stride * esz;
    return static_cast<const char*>(a.dlogits) + ((size_t)b * a.max_k + (r - a.max_k - 1)) * a.row_stride * esz;
}

__device__ __forceinline__ bool row_needed(const SpecArgs& a, int b, int r) {
    const int k = a.k_len[b];
    return r <= a.max_k ? r <= k : (r - a.max_k - 1) < k;
}

__device__ __forceinline__ float2 ms_merge(float2 p, float2 q) {
    const float m = fmaxf(p.x, q.x);
    if (m == -INFINITY) return make_float2(-INFINITY, 0.f);
    return make_float2(m, p.y * fast_exp2((p.x - m) * kLog2e) + q.y * fast_exp2((q.x - m) * kLog2e));
}

__device__ __forceinline__ float2 wave_ms(float2 v) {
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1)
        v = ms_merge(v, make_float2(__shfl_xor(v.x, o, kWave), __shfl_xor(v.y, o, kWave)));
    return v;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// v of the lane the DPP control selects (0 where there is none).
template <int kCtrl, int kRows>
__device__ __forceinline__ float dpp_f(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl,
                                                                 kRows, 0xf, false));
}

// Inclusive scan of one float per lane over the wave (fixed order).
__device__ __forceinline__ float wave_incl_scan_f(float x) {
    x += dpp_f<0x111, 0xf>(x);   // row_shr:1
    x += dpp_f<0x112, 0xf>(x);   // row_shr:2
    x += dpp_f<0x114, 0xf>(x);   // row_shr:4
    x += dpp_f<0x118, 0xf>(x);   // row_shr:8
    x += dpp_f<0x142, 0xa>(x);   // row_bcast:15 -> rows 1, 3
    x += dpp_f<0x143, 0xc>(x);   // row_bcast:31 -> rows 2, 3
    return x;
}

// ---- stats: grid (n_chunks, batch * (2 max_k + 1)) ----------------------------
template <bool kF32>
__global__ __launch_bounds__(kThreads) void spec_stats_kernel(SpecArgs a) {
    const int chunk = blockIdx.x, rows = 2 * a.max_k + 1;
    const int b = blockIdx.y / rows, r = blockIdx.y - b * rows;
    if (!row_needed(a, b, r)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float x[32];
    lc::load_chunk<kF32>(row_base(a, b, r, kF32), a.vocab, chunk, tid, x);
    float m = -INFINITY;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
        x[q] *= a.inv_tau;
        m = fmaxf(m, x[q]);
    }
    float s = 0.f;
    if (m != -INFINITY) {
#pragma unroll
        for (int q = 0; q < 32; ++q) s += fast_exp2((x[q] - m) * kLog2e);
    }
    __shared__ float2 wv[kWaves];
    const float2 v = wave_ms(make_float2(m, s));
    if (lane == 0) wv[wave] = v;
    __syncthreads();
    if (tid == 0) {
        float2 t = wv[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) t = ms_merge(t, wv[w]);
        a.chunk_ms[((size_t)b * rows + r) * a.n_chunks + chunk] = t;
    }
}

// p(x) for a row with merged (max, sum) ms at scaled logit y = x / tau.
__device__ __forceinline__ float prob(float y, float2 ms) {
    return fast_exp2((y - ms.x) * kLog2e) / ms.y;
}

template <bool kF32>
__device__ __forceinline__ float logit_at(const char* row, int i) {
    if (kF32) return reinterpret_cast<const float*>(row)[i];
    return bf16_lo((uint32_t)reinterpret_cast<const uint16_t*>(row)[i]);
}

// The merged (max, sum) of every row of sequence b into rms[] (LDS); rows that
// are not needed are left alone.  A wave takes 64 / np2 rows at once, np2 the
// power of two that holds a row's chunks, and four such sets in flight (a wave
// per row and six levels whatever the chunks made every workgroup of 8
// sequences of 63 drafted tokens and 32000 tokens merge for 17 us).
__device__ __forceinline__ void merge_rows(const SpecArgs& a, int b, float2* rms) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, rows = 2 * a.max_k + 1;
    const int lg = a.n_chunks > 1 ? 32 - __builtin_clz(a.n_chunks - 1) : 0, np2 = 1 << lg;
    const int sub = lane >> lg, c = lane & (np2 - 1), step = kWaves * (kWave >> lg);
    for (int r0 = wave * (kWave >> lg); r0 < rows; r0 += 4 * step) {
        float2 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = min(r0 + u * step + sub, rows - 1);
            v[u] = a.chunk_ms[((size_t)b * rows + r) * a.n_chunks + min(c, a.n_chunks - 1)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = c < a.n_chunks ? v[u] : make_float2(-INFINITY, 0.f);
        for (int o = 1; o < np2; o <<= 1) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (r0 + u * step < rows)   // wave-uniform
                    v[u] = ms_merge(v[u], make_float2(__shfl_xor(v[u].x, o, kWave), __shfl_xor(v[u].y, o, kWave)));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r0 + u * step + sub;
            if (c == 0 && r < rows && row_needed(a, b, r)) rms[r] = v[u];
        }
    }
}

// The blocks that thread tid weighs in chunk `chunk`: target row m and, with a
// residual (m < k), drafter row m.
template <bool kF32>
struct Weights {
    static constexpr int kPer = lc::per_load<kF32>(), kLoads = lc::loads<kF32>();
    uint4 raw[2][kLoads];
    float2 mt, md;
    bool resid;

    __device__ __forceinline__ void load(const SpecArgs& a, int b, int m, int chunk, int tid) {
        resid = m < a.k_len[b];
        lc::load_blocks<kF32>(row_base(a, b, m, kF32), a.vocab, chunk, tid, raw[0]);
        if (resid) lc::load_blocks<kF32>(row_base(a, b, a.max_k + 1 + m, kF32), a.vocab, chunk, tid, raw[1]);
    }
    // The weights of the block at the head of the queue, the thread's load j:
    // max(0, p_m - q_m) in w and p_m in pw, or p_k in both without a residual.
    __device__ __forceinline__ void block(const SpecArgs& a, int chunk, int j, int tid, float (&w)[kPer],
                                          float (&pw)[kPer]) const {
        float x[kPer];
        lc::unpack_block<kF32>(raw[0][0], a.vocab, chunk, j, tid, x);
#pragma unroll
        for (int e = 0; e < kPer; ++e) w[e] = pw[e] = x[e] == -INFINITY ? 0.f : prob(x[e] * a.inv_tau, mt);
        if (!resid) return;   // (uniform)
        lc::unpack_block<kF32>(raw[1][0], a.vocab, chunk, j, tid, x);
#pragma unroll
        for (int e = 0; e < kPer; ++e) w[e] = fmaxf(pw[e] - (x[e] == -INFINITY ? 0.f : prob(x[e] * a.inv_tau, md)), 0.f);
    }
};

// ---- mass: grid (n_chunks, batch) -----------------------------------------------------
template <bool kF32>
__global__ __launch_bounds__(kThreads) void spec_mass_kernel(SpecArgs a) {
    const int chunk = blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int k = a.k_len[b];
    __shared__ float2 rms[2 * kAcceptMaxK + 1];
    __shared__ int sh_m;
    // drafted token j's logits in both rows, its uniform (lane j of wave 0)
    float xt = 0.f, xd = 0.f, u = 0.f;
    if (wave == 0 && lane < k) {
        const int x = min(max(a.draft[(size_t)b * a.max_k + lane], 0), a.vocab - 1);
        u = a.u_acc[(size_t)b * a.max_k + lane];
        xt = logit_at<kF32>(row_base(a, b, lane, kF32), x);
        xd = logit_at<kF32>(row_base(a, b, a.max_k + 1 + lane, kF32), x);
    }
    merge_rows(a, b, rms);
    __syncthreads();
    if (wave == 0) {
        const float p = prob(xt * a.inv_tau, rms[lane]);
        const float q = prob(xd * a.inv_tau, rms[a.max_k + 1 + min(lane, a.max_k - 1)]);
        const bool pass = lane >= k || u * q < p;
        const uint64_t fail = __ballot(!pass);
        if (lane == 0) sh_m = fail ? __builtin_ctzll(fail) : k;
    }
    __syncthreads();
    const int m = sh_m;
    const float2 mt = rms[m];
    const float2 md = m < k ? rms[a.max_k + 1 + m] : make_float2(0.f, 1.f);   // (a row past k is not there)
    if (chunk == 0 && tid == 0) {
        a.n_accepted[b] = m;
        a.pick[b] = m;
        a.row_ms[2 * b] = mt;
        a.row_ms[2 * b + 1] = md;
    }
    Weights<kF32> wt;
    wt.mt = mt;
    wt.md = md;
    wt.load(a, b, m, chunk, tid);
    float s = 0.f, sp = 0.f;
    lc::for_blocks(wt.raw, [&](int j) {
        float w[wt.kPer], pw[wt.kPer];
        wt.block(a, chunk, j, tid, w, pw);
#pragma unroll
        for (int e = 0; e < wt.kPer; ++e) {
            s += w[e];
            sp += pw[e];
        }
    });
    s = wave_sum(s);
    sp = wave_sum(sp);
    __shared__ float2 wv[kWaves];
    if (lane == 0) wv[wave] = make_float2(s, sp);
    __syncthreads();
    if (tid == 0) {
        float2 t = wv[0];
#pragma unroll
        for (int v = 1; v < kWaves; ++v) {
            t.x += wv[v].x;
            t.y += wv[v].y;
        }
        a.mass[(size_t)b * a.n_chunks + chunk] = t;
    }
}

// ---- sample: one workgroup per sequence -------------------------------------------------
template <bool kF32>
__global__ __launch_bounds__(kThreads) void spec_sample_kernel(SpecArgs a) {
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ int sh_chunk, sh_use_p, sh_found, sh_last;
    __shared__ float sh_target;
    __shared__ float wtot[kWaves];
    const int m = a.pick[b];
    const float2 mt = a.row_ms[2 * b], md = a.row_ms[2 * b + 1];
    if (wave == 0) {
        // the residual when it has mass, else the plain target row; the chunk
        // where the cumulative mass (chunk order) passes u * total.  Lane c
        // holds chunk c's masses; the sums run in chunk order, wave-uniform.
        const float2 v = a.mass[(size_t)b * a.n_chunks + min(lane, a.n_chunks - 1)];
        const float usmp = a.u_smp[b];
        auto at = [&](float x, int c) {
            return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), c));
        };
        float tot = 0.f, totp = 0.f;
        for (int c = 0; c < a.n_chunks; ++c) {
            tot += at(v.x, c);
            totp += at(v.y, c);
        }
        const bool use_p = !(tot > 0.f);
        const float mine = use_p ? v.y : v.x;
        const float total = use_p ? totp : tot;
        const float target = usmp * total;
        float run = 0.f;
        int cstar = -1, last = 0;
        for (int c = 0; c < a.n_chunks; ++c) {
            const float mc = at(mine, c);
            if (mc > 0.f) last = c;
            if (cstar < 0 && run + mc > target) cstar = c;
            if (cstar < 0) run += mc;
        }
        if (cstar < 0) {   // rounding left the cumulative mass short: the last chunk with mass
            cstar = last;
            run = 0.f;
            for (int c = 0; c < last; ++c) run += at(mine, c);
        }
        if (lane == 0) {
            sh_chunk = cstar;
            sh_use_p = use_p ? 1 : 0;
            sh_target = target - run;
            sh_found = 0x7fffffff;
            sh_last = -1;
        }
    }
    __syncthreads();
    const int chunk = sh_chunk;
    const float target = sh_target;
    Weights<kF32> wt;
    wt.mt = mt;
    wt.md = md;
    wt.load(a, b, m, chunk, tid);
    const bool use_p = sh_use_p != 0;
    // scan in index order: load j of every thread, thread by thread, then its
    // elements in order
    float carry = 0.f;
    int last = -1;
    bool found = false;   // uniform
    lc::for_blocks(wt.raw, [&](int j) {
        if (found) return;
        float w[wt.kPer], pw[wt.kPer];
        wt.block(a, chunk, j, tid, w, pw);
        const int i0 = lc::elem<kF32>(chunk, j * wt.kPer, tid);
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < wt.kPer; ++e) {
            w[e] = use_p ? pw[e] : w[e];
            s += w[e];
            if (w[e] > 0.f) last = i0 + e;
        }
        const float incl = wave_incl_scan_f(s);
        if (lane == kWave - 1) wtot[wave] = incl;
        __syncthreads();
        float before = carry, all = carry;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) {
            before += v < wave ? wtot[v] : 0.f;
            all += wtot[v];
        }
        float run = before + incl - s;
        int cand = 0x7fffffff;
#pragma unroll
        for (int e = 0; e < wt.kPer; ++e) {
            run += w[e];
            if (cand == 0x7fffffff && run > target) cand = i0 + e;
        }
        if (cand != 0x7fffffff) atomicMin(&sh_found, cand);
        __syncthreads();
        carry = all;
        found = sh_found != 0x7fffffff;   // read after the barrier
    });
    if (last >= 0) atomicMax(&sh_last, last);
    __syncthreads();
    if (tid == 0) a.next_token[b] = sh_found != 0x7fffffff ? sh_found : max(sh_last, 0);
}

}  // namespace

hipError_t launch_spec_accept(const SpecArgs& a, int batch, bool f32, hipStream_t stream) {
    const dim3 block(kThreads), per_chunk(a.n_chunks, batch);
    const dim3 per_row(a.n_chunks, batch * (2 * a.max_k + 1));
    if (f32) {
        hipLaunchKernelGGL(spec_stats_kernel<true>, per_row, block, 0, stream, a);
        hipLaunchKernelGGL(spec_mass_kernel<true>, per_chunk, block, 0, stream, a);
        hipLaunchKernelGGL(spec_sample_kernel<true>, dim3(batch), block, 0, stream, a);
    } else {
        hipLaunchKernelGGL(spec_stats_kernel<false>, per_row, block, 0, stream, a);
        hipLaunchKernelGGL(spec_mass_kernel<false>, per_chunk, block, 0, stream, a);
        hipLaunchKernelGGL(spec_sample_kernel<false>, dim3(batch), block, 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace ssl
