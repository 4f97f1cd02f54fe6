// verify_stream.hip -- single-sweep verify attention with fused Eq. 3 scores
// (Sec. 3.1 verification, Sec. 3.2 Eq. 3) for calls whose chunks take more
// than one round of one workgroup per CU.
//
// What bounds such a call is the K and V stream, as long as nothing idles
// while a chunk's row statistics travel: a score needs the normalizer of every
// verify row over the whole context, and a workgroup that has streamed its
// chunk can only wait for it.  So two workgroups share a CU (at most half of
// its LDS and 256 registers per lane each): while one waits, merges and writes
// scores, the other streams.  Measured per verify call, before (a persistent
// grid, or two sweeps where that did not fit) and after: 16 chat sequences of
// 1K-8K keys 106 -> 82 us, 12 paged sequences of 3K-30K keys 201 -> 183 us,
// 8 sequences of 16K-64K keys and up to 40 rows 383 -> 292 us.
//
// A workgroup:
//   1. streams its chunk of K and V once, a wave per 32-key tile, online
//      softmax, P.V on the MFMA.  It keeps in LDS the probabilities of its
//      keys, per verify row of the sequence (no padding rows), relative to the
//      wave's reference maximum of the row: as 16-bit codes (kU16), or in fp32,
//      where each wave's last tile stays in its registers, which adds 128 keys
//      to what the LDS holds.  The fp32
//      reference is the row's maximum over the wave's first tile: probabilities
//      are scale-free in fp32 and in bf16, so it moves only when a key exceeds
//      it by 2^32 (the accumulators and the wave's stash are rescaled then).
//      One tile's K and V are in registers at a time: K of the next tile is
//      requested when the logits are formed, V when P.V is, and eight waves per
//      CU keep the memory system busy.  The Q operand is read from LDS (it
//      would not fit the register budget at three row tiles);
//   2. publishes its (max, sum) per row, tagged, and then its partial P.V;
//   3. for its share of the unit's rows (row s, s + nchunk, ... for chunk s)
//      waits for every chunk's (max, sum) and publishes the row's log-sum-exp.
//      Every chunk reading every chunk's statistics would load
//      nchunk^2 * rows words per unit (at 131072 keys and 36 rows over half
//      as much as K and V themselves);
//   4. waits for the unit's log-sum-exps (one word per row) and writes the
//      scores of its keys from the stash;
//   5. for its share of the rows, adds the chunks' partial P.V (each chunk's
//      landed once its own tag is there) and writes the output.
// A KV head with more than 40 verify rows runs as several row blocks of at
// most 32 rows, each an exchange group (a unit, in the list above) of its own;
// the blocks of a chunk run on one die, at about the same time where the device
// holds all of a head's, and the blocks' scores are added by a second, small
// kernel.
// (128 rows over 8 heads of 20011 keys: 98.6 us as two blocks of 64 rows of two
// sweeps each, whose 160 items leave CUs idle; 71.2 us as four of 32 rows, which
// fetch 164 MB for the 82 MB of K and V, so half of the four reads hit the L2.)
// Publication, tags, epochs and bounded waits are those of verify_fused.hip.
// The waits end: workgroups are dispatched in index order, the chunks of a
// group (of both blocks, where two are interleaved) are consecutive and at most
// 128, a quarter of what the device holds, so that the calls of four streams
// cannot fill it with groups that wait; publications wait for nothing, and a
// row's reduction waits for publications only.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "verify_common.h"

namespace ssl {
namespace {

using namespace vc;

constexpr int kQStride = kHeadDim * 2 + 16;               // bytes per Q row in LDS
constexpr int kParkStride = 36;                           // floats per parked quarter row
constexpr int kParkBytes = kWaves * 16 * kParkStride * 4;
constexpr float kSlack = 32.f;                            // reference-maximum slack, log2 units
constexpr float kEmpty = -3.402823466e38f;                // reference maximum of a row without keys so far

constexpr size_t stream_lds_bytes(int rows, int tiles) {
    const int alloc = std::max(4, tiles - 4);
    return (size_t)rows * (alloc * kTile + 4) * 4 + (size_t)std::max(kParkBytes, rows * kQStride);
}

// The same for 16-bit codes, with a reference maximum per tile and row.
constexpr size_t code_lds_bytes(int rows, int chunk) {
    return (size_t)rows * ((chunk + 8) * 2 + chunk / kTile * 4) + (size_t)std::max(kParkBytes, rows * kQStride);
}

// A chunk of one row block of one (sequence, KV head): the verify positions of
// a sequence are cut into `blocks` row blocks, each an exchange group of its
// own (grp) over the same chunks.
struct SChunk {
    int unit, grp, b, c, s, blk, slot0, nchunk, T, nq, qoff, qfull, R, key_begin, key_end, stride;
    size_t row0;   // the group's first row in part_o; chunk s's rows start R * s further on
};

__device__ __forceinline__ SChunk schunk_of(const StreamArgs& fa, int slot) {
    const VerifyArgs& a = fa.v;
    // The last sequence whose items start at or before this one, sixteen scalar
    // loads together (starts past the table's end are larger than any slot).
    int b = 0;
    for (int b0 = 0; b0 + 1 < a.seq.n_seq; b0 += 16) {
#pragma unroll
        for (int i = 1; i <= 16; ++i) b += slot >= a.seq.item_start[b0 + i] ? 1 : 0;
    }
    SChunk k;
    const int chunk = fa.chunk[b];
    const int nb = fa.blocks[b], pos = fa.block_pos[b];
    k.b = b;
    k.T = a.seq.ctx[b];
    k.qfull = a.seq.qlen[b];
    k.nchunk = (k.T + chunk - 1) / chunk;
    const int local = slot - a.seq.item_start[b], per_head = k.nchunk * nb;
    k.c = __builtin_amdgcn_readfirstlane(local / per_head);
    int r = local - k.c * per_head;
    k.blk = 0;
    k.s = r;
    if (nb == 2 && per_head <= fa.together) {
        // Eight chunks of block 0, the same eight of block 1: workgroups eight
        // apart run on one die at about the same time, so the blocks of a chunk
        // find its K and V in that die's L2 (64 rows over 2 x 20000 keys, 8
        // heads: 76.9 us against 80.5 block after block).
        const int o = __builtin_amdgcn_readfirstlane(r / (8 * nb));
        const int w = min(8, k.nchunk - 8 * o);
        r -= 8 * nb * o;
        k.blk = __builtin_amdgcn_readfirstlane(r / w);
        k.s = 8 * o + r - k.blk * w;
    } else if (nb > 1) {
        // Block after block, so that only a block's own chunks have to be on the
        // device together; each block is rotated so that (but for its last ones)
        // a chunk runs on the die it has in block 0.  With three and more blocks
        // a group also ends sooner (128 rows over 2 x 9000 keys, 8 heads: 69.5 us
        // against 74.8 interleaved).
        k.blk = __builtin_amdgcn_readfirstlane(r / k.nchunk);
        k.s = (r - k.blk * k.nchunk + (k.blk * k.nchunk & 7)) % k.nchunk;
    }
    k.qoff = k.blk * pos;
    k.nq = min(pos, k.qfull - k.qoff);
    k.R = k.nq * a.group;
    k.key_begin = k.s * chunk;
    k.key_end = min(k.key_begin + chunk, k.T);
    k.unit = b * a.n_kv_heads + k.c;
    k.grp = k.unit * fa.max_blocks + k.blk;
    k.slot0 = a.seq.item_start[b] + k.c * per_head + k.blk * k.nchunk;
    k.row0 = (size_t)a.seq.row_start[b] + (size_t)k.nchunk * a.group * (k.c * k.qfull + k.qoff);
    k.stride = fa.u16 ? chunk + 8 : max(4, chunk / kTile - 4) * kTile + 4;
    return k;
}

// (a decode step whose draft reads most of the cache again keeps it in the L2
// instead: kKeep, see ssl_decode_step)
template <bool kKeep>
__device__ __forceinline__ u32x4 ld_rsrc(__amdgpu_buffer_rsrc_t r, int off) {
    constexpr int kNonTemporal = 2;   // the buffer instructions' nt bit
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kKeep ? 0 : kNonTemporal));
}

// The 32-key tile at key0 of a cache as a buffer of its valid rows: rows past
// the sequence read as zero (their probabilities are masked to zero), so the
// loads need no clamps.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const uint16_t* base, int rows) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, min(rows, kTile) * kHeadDim * 2, 0x00027000);
}

// Probabilities of one tile (before normalization) for row tile rt: p, the
// row's running sum, and the reference maximum with its rare moves.  Logits a
// row may not see are -inf.
template <int NRT>
__device__ __forceinline__ void tile_probs(int rt, const f32x4 (&acc)[2], float scale, float* srow, int t,
                                           int wave, bool own_row, float (&M)[NRT], float (&L)[NRT],
                                           f32x4 (&oacc)[8][NRT], f32x4 (&p)[2]) {
    float z[8];
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        z[e] = __builtin_fmaf(acc[e >> 2][e & 3], scale, -M[rt]);
        mx = fmaxf(mx, z[e]);
    }
    if (__any(mx > kSlack)) {   // the wave's first tile, or a key far above the reference
        float mt = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) mt = fmaxf(mt, acc[e >> 2][e & 3] * scale);
        mt = fmaxf(mt, shfl_xor_f(mt, 16));
        mt = fmaxf(mt, shfl_xor_f(mt, 32));
        const bool grow = mt > M[rt] + kSlack;
        const bool had = grow && M[rt] != kEmpty;
        if (__any(had)) {
            const float alpha = grow ? fast_exp2(M[rt] - mt) : 1.f;
            L[rt] *= alpha;
#pragma unroll
            for (int jd = 0; jd < 8; ++jd) oacc[jd][rt] *= alpha;
            if (had && own_row) {   // this lane's stashed probabilities of the row
                for (int tt = wave; tt < t; tt += kWaves) {
                    f32x4* q = reinterpret_cast<f32x4*>(srow + tt * kTile);
                    q[0] *= alpha;
                    q[4] *= alpha;
                }
            }
        }
        M[rt] = grow ? mt : M[rt];
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = __builtin_fmaf(acc[e >> 2][e & 3], scale, -M[rt]);
    }
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p[e >> 2][e & 3] = fast_exp2(z[e]);
        sum += p[e >> 2][e & 3];
    }
    L[rt] += sum;
}

// The same for 16-bit codes: the reference follows the row's maximum over the
// wave's tiles within 2^8 (kLazy), since a code spans 2^-54 .. 2^9 of it.
constexpr float kLazy = 8.f;
template <int NRT>
__device__ __forceinline__ void tile_probs_lazy(int rt, const f32x4 (&acc)[2], float scale, float (&M)[NRT],
                                                float (&L)[NRT], f32x4 (&oacc)[8][NRT], f32x4 (&p)[2]) {
    float y[8];
    float mt = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        y[e] = acc[e >> 2][e & 3] * scale;
        mt = fmaxf(mt, y[e]);
    }
    mt = fmaxf(mt, shfl_xor_f(mt, 16));
    mt = fmaxf(mt, shfl_xor_f(mt, 32));
    const bool grow = mt > M[rt] + kLazy;
    if (__any(grow)) {
        const float alpha = grow ? fast_exp2(M[rt] - mt) : 1.f;
        M[rt] = grow ? mt : M[rt];
        L[rt] *= alpha;
#pragma unroll
        for (int jd = 0; jd < 8; ++jd) oacc[jd][rt] *= alpha;
    }
    const float Mr = M[rt] == kEmpty ? 0.f : M[rt];
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p[e >> 2][e & 3] = fast_exp2(y[e] - Mr);
        sum += p[e >> 2][e & 3];
    }
    L[rt] += sum;
}

// 16-bit codes of probabilities relative to a reference maximum (at most
// 2^kLazy): 6 exponent bits (2^-54 .. 2^9) above the top 10 mantissa bits,
// rounded to nearest (relative error at most 2^-11, so a score, a sum of such
// terms times exact factors, keeps that bound); values below 2^-54 of the
// reference are coded 0.
constexpr uint32_t kCodeBias = 72u << 10;   // exponent field 72 at code 0
__device__ __forceinline__ uint32_t code_of(float v) {
    const uint32_t r = (__float_as_uint(v) + 0x1000u) >> 13;   // 10 mantissa bits, rounded
    return r >= kCodeBias + 1024u ? min(r - kCodeBias, 0xFFFFu) : 0u;
}
__device__ __forceinline__ float of_code(uint32_t c) { return c ? __uint_as_float((c + kCodeBias) << 13) : 0.f; }

template <int NRT, bool kPaged, bool kU16, bool kKeep>
__device__ __forceinline__ void stream_chunk(const StreamArgs& fa, const SChunk& k, char* lds,
                                             float2* wml, float* row_lse, int* wait_failed) {
    const VerifyArgs& a = fa.v;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar, so buffer descriptors are
    const int m16 = lane & 15, G = lane >> 4;
    const int R = k.R, stride = k.stride, g = a.group;
    using Elem = std::conditional_t<kU16, uint16_t, float>;
    Elem* stash = reinterpret_cast<Elem*>(lds);                 // [R][stride]
    const int mts = kU16 ? fa.chunk[k.b] / kTile : 0;
    float* mtile = reinterpret_cast<float*>(lds + (size_t)R * stride * sizeof(Elem));   // [R][mts] references of the tiles
    char* park_c = reinterpret_cast<char*>(mtile + R * mts);    // Q during the sweep, then scratch
    float* park = reinterpret_cast<float*>(park_c);

    // The unit's exchange epoch, loaded first: the waits below cover it.
    const uint64_t ep = fa.epoch ? ld_dev64(fa.epoch + k.grp) : 0ull;

    // ---- 1. the sweep ---------------------------------------------------------
    u32x4 qreg[NRT];
#pragma unroll
    for (int it = 0; it < NRT; ++it) {
        const int row = min(it * 16 + (tid >> 4), R - 1);
        const int j = row / g, hh = row - j * g;
        qreg[it] = ld_u32x4(a.q + (((size_t)k.b * a.max_q + k.qoff + j) * a.n_q_heads + k.c * g + hh) * kHeadDim +
                            8 * (tid & 15));
    }
    const int ntile = (k.key_end - k.key_begin + kTile - 1) / kTile;
    const size_t cache_off = (size_t)k.unit * a.max_ctx * kHeadDim;
    const int pages = kPaged ? wave_pages(a, k.b, k.key_begin, ntile, wave, lane) : 0;
    const int k_off = a_row_key(m16) * (kHeadDim * 2) + 16 * G;
    const int v_off = G * (kHeadDim * 2) + 16 * m16;
    u32x4 kr[2][4], vr[8];
    // tile t of the chunk, in elements from the cache's start
    auto tile_at = [&](int t) -> size_t {
        const int key0 = k.key_begin + t * kTile;
        if constexpr (kPaged) return paged_row(a, tile_page(pages, t, wave), k.c, key0) * kHeadDim;
        return cache_off + (size_t)key0 * kHeadDim;
    };
    auto load_k_tile = [&](int t) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t r = tile_rsrc(a.k + tile_at(t), k.T - (k.key_begin + t * kTile));
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) kr[h][kb] = ld_rsrc<kKeep>(r, k_off + 16 * h * (kHeadDim * 2) + 64 * kb);
    };
    auto load_v_tile = [&](int t) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t r = tile_rsrc(a.v + tile_at(t), k.T - (k.key_begin + t * kTile));
#pragma unroll
        for (int e = 0; e < 8; ++e)
            vr[e] = ld_rsrc<kKeep>(r, v_off + (16 * (e >> 2) + 4 * (e & 3)) * (kHeadDim * 2));
    };
    // (in this order also after scheduling: the loop's waits count on K being
    // the older of the two)
    if (wave < ntile) {
        load_k_tile(wave);
        __builtin_amdgcn_sched_barrier(0);
        load_v_tile(wave);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int it = 0; it < NRT; ++it) {
        const int row = it * 16 + (tid >> 4);
        if (row < R) *reinterpret_cast<u32x4*>(park_c + row * kQStride + 16 * (tid & 15)) = qreg[it];
    }
    if (tid == 0) *wait_failed = 0;

    float M[NRT], L[NRT];
    f32x4 oacc[8][NRT];
    f32x4 plast[NRT][2];   // probabilities of the wave's last tile
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) {
        M[rt] = kEmpty;
        L[rt] = 0.f;
#pragma unroll
        for (int jd = 0; jd < 8; ++jd) oacc[jd][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (!kU16) plast[rt][0] = plast[rt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();   // Q is in LDS

    const int all_see = k.T - k.qfull + k.qoff;   // keys up to here are visible to every row
    auto tile_step = [&](int t, bool last) __attribute__((always_inline)) {
        const int key0 = k.key_begin + t * kTile;
        u32x4 pb[NRT];
        auto logits = [&](int rt, f32x4 (&acc)[2]) __attribute__((always_inline)) {
            // (rows past R re-read the last row: nothing of theirs is kept)
            const char* qrow = park_c + min(rt * 16 + m16, R - 1) * kQStride + 16 * G;
            u32x4 qv[4];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) qv[kb] = *reinterpret_cast<const u32x4*>(qrow + 64 * kb);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) s = mfma_bf16(kr[h][kb], qv[kb], s);
                acc[h] = s;
            }
            if (key0 + kTile - 1 > all_see) {   // wave-uniform: some row does not see some key
                const int plim = all_see + (rt * 16 + m16) / g;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    acc[e >> 2][e & 3] = key0 + 16 * (e >> 2) + G + 4 * (e & 3) <= plim ? acc[e >> 2][e & 3] : -INFINITY;
            }
        };
        auto probs = [&](int rt, const f32x4 (&acc)[2]) __attribute__((always_inline)) {
            const bool own = rt * 16 + m16 < R;
            Elem* srow = stash + (rt * 16 + m16) * stride + 4 * G;
            f32x4 (&p)[2] = plast[rt];
            if constexpr (kU16) {
                tile_probs_lazy<NRT>(rt, acc, a.scale_log2, M, L, oacc, p);
                if (own) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        *reinterpret_cast<uint2*>(srow + t * kTile + 16 * h) =
                            make_uint2(code_of(p[h][0]) | code_of(p[h][1]) << 16, code_of(p[h][2]) | code_of(p[h][3]) << 16);
                    // (kEmpty for a row that has seen no key: its factor is 0)
                    if (G == 0) mtile[(rt * 16 + m16) * mts + t] = M[rt];
                }
            } else {
                tile_probs<NRT>(rt, acc, a.scale_log2, srow, t, wave, own, M, L, oacc, p);
                if (!last && own) {
                    f32x4* q = reinterpret_cast<f32x4*>(srow + t * kTile);
                    q[0] = p[0];
                    q[4] = p[1];
                }
            }
            pb[rt] = u32x4{pack_bf16(p[0][0], p[0][1]), pack_bf16(p[0][2], p[0][3]),
                           pack_bf16(p[1][0], p[1][1]), pack_bf16(p[1][2], p[1][3])};
        };
        f32x4 acc[NRT][2];
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) logits(rt, acc[rt]);
        if (!last) load_k_tile(t + kWaves);
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) probs(rt, acc[rt]);
#pragma unroll
        for (int jd = 0; jd < 8; ++jd) {
            u32x4 av;
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2) {
                const uint32_t x = vr[2 * s2][jd >> 1], y = vr[2 * s2 + 1][jd >> 1];
                av[s2] = (jd & 1) ? perm_hi(x, y) : perm_lo(x, y);
            }
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt) oacc[jd][rt] = mfma_bf16(av, pb[rt], oacc[jd][rt]);
        }
        if (!last) load_v_tile(t + kWaves);
    };
    // (the wave's last tile is peeled off: a load that may be skipped at the
    // loop's end would make every wait for K also wait for V)
    int t = wave;
    for (; t + kWaves < ntile; t += kWaves) tile_step(t, false);
    if (t < ntile) tile_step(t, true);

    // ---- 2. publish the row statistics, then the partial output --------------------
    const uint64_t epv = scalar_here(ep);
    const uint64_t want = exchange_tag(fa.call_tag, epv);
    const uint64_t tag_hi = (want & 0xFFFFFFFFull) << 32;
    const uint64_t pub = ((want ^ fa.xc.tag_flip) & 0xFFFFFFFFull) << 32;
    const bool clean = !epoch_is_dirty(epv);   // else an earlier captured call on this workspace gave up
    uint64_t* ml64 = reinterpret_cast<uint64_t*>(a.part_ml) + (size_t)k.slot0 * kRowCap * 2;   // [row][chunk][2]
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) {
        L[rt] += shfl_xor_f(L[rt], 16);
        L[rt] += shfl_xor_f(L[rt], 32);
        if (G == 0) wml[wave * kRowCap + rt * 16 + m16] = make_float2(M[rt], L[rt]);
    }
    __syncthreads();   // (and no wave reads Q any more)
    if (clean && tid < R) {
        float own_m = kEmpty, own_l = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) own_m = fmaxf(own_m, wml[w * kRowCap + tid].x);
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            own_l += wml[w * kRowCap + tid].y * fast_exp2(wml[w * kRowCap + tid].x - own_m);
        uint64_t* e = ml64 + ((size_t)tid * k.nchunk + k.s) * 2;
        st_dev64(e, pub | __float_as_uint(own_m));
        st_dev64(e + 1, pub | __float_as_uint(own_l));
    }
    // The waves' partial P.V, relative to the workgroup's row maxima, added in
    // LDS a quarter row (accumulator elements i) of a row tile at a time.  A
    // published row holds its head-dim elements in the order [i][G][jd].
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) {
        float mw = kEmpty;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) mw = fmaxf(mw, wml[w * kRowCap + rt * 16 + m16].x);
        const float f = fast_exp2(M[rt] - mw);
        const int pr = tid >> 4, c2 = tid & 15;
        uint64_t* po = reinterpret_cast<uint64_t*>(a.part_o + (k.row0 + (size_t)k.s * R + rt * 16 + pr) * kHeadDim);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f32x4* dst = reinterpret_cast<f32x4*>(park + (wave * 16 + m16) * kParkStride + 8 * G);
            dst[0] = f32x4{oacc[0][rt][i], oacc[1][rt][i], oacc[2][rt][i], oacc[3][rt][i]} * f;
            dst[1] = f32x4{oacc[4][rt][i], oacc[5][rt][i], oacc[6][rt][i], oacc[7][rt][i]} * f;
            __syncthreads();
            float2 o = *reinterpret_cast<const float2*>(park + pr * kParkStride + 2 * c2);
#pragma unroll
            for (int w = 1; w < kWaves; ++w) {
                const float2 v = *reinterpret_cast<const float2*>(park + (w * 16 + pr) * kParkStride + 2 * c2);
                o.x += v.x;
                o.y += v.y;
            }
            if (rt * 16 + pr < R) st_dev64(po + 16 * i + c2, __builtin_bit_cast(uint64_t, o));
            __syncthreads();
        }
    }
    uint64_t* lse64 = fa.lse + (size_t)k.grp * kRowCap;
    auto give_up = [&]() {
        if (tid == 0) exchange_gave_up(fa.xc, kStatusVerify, fa.epoch ? fa.epoch + k.grp : nullptr);
    };

    // ---- 3. the log-sum-exp of this chunk's share of the rows: s, s + nchunk, ... -----
    // thread rk * np2 + cc holds chunk cc of the rk-th row (nr * np2 <= 256:
    // several rows only when the unit has fewer chunks than rows, <= 64)
    const int nr = k.s < R ? (R - k.s + k.nchunk - 1) / k.nchunk : 0;
    const int lg = k.nchunk > 1 ? 32 - __builtin_clz(k.nchunk - 1) : 0, np2 = 1 << lg;
    float my_wt = 0.f;   // chunk cc's weight 2^(m - lse) in the rk-th row
    if (nr > 0) {
        const int rk = tid >> lg, cc = tid & (np2 - 1);
        const bool active = rk < nr && cc < k.nchunk;
        const int row = active ? k.s + rk * k.nchunk : k.s;
        const uint64_t* e = ml64 + ((size_t)row * k.nchunk + (active ? cc : 0)) * 2;
        uint64_t w0 = 0, w1 = 0;
        bool all_in = clean;
        if (clean) {
            int spins = 0;
            do {
                w0 = ld_dev64(e);
                w1 = ld_dev64(e + 1);
                all_in = __all((w0 & ~0xFFFFFFFFull) == tag_hi && (w1 & ~0xFFFFFFFFull) == tag_hi);
                if (!all_in) __builtin_amdgcn_s_sleep(1);
            } while (!all_in && ++spins < fa.xc.spin_limit);
        }
        if (!all_in && lane == 0) *wait_failed = 1;
        const float m = active && all_in ? __uint_as_float((uint32_t)w0) : kEmpty;
        float Mx = m, Lx = active && all_in ? __uint_as_float((uint32_t)w1) : 0.f;
        for (int o = 1; o < min(np2, kWave); o <<= 1) ml_merge(Mx, Lx, shfl_xor_f(Mx, o), shfl_xor_f(Lx, o));
        if (np2 > kWave) {   // one row over up to four waves
            float2* wpart = reinterpret_cast<float2*>(park);
            if (lane == 0) wpart[wave] = make_float2(Mx, Lx);
            __syncthreads();
            all_in = *wait_failed == 0;   // (a sum may be NaN: it says nothing about the wait)
            Mx = kEmpty;
            Lx = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) ml_merge(Mx, Lx, wpart[w].x, wpart[w].y);
        }
        const float lse = Lx > 0.f ? Mx + fast_log2(Lx) : INFINITY;
        if (all_in && active && cc == 0) st_dev64(lse64 + row, pub | __float_as_uint(lse));
        my_wt = active ? fast_exp2(m - lse) : 0.f;
    }

    // ---- 4. the scores of this chunk's keys --------------------------------------------
    wait_stores_done();   // this wave's partial output has landed
    if (wave == 0) {
        const uint64_t* e = lse64 + min(lane, R - 1);
        uint64_t w0 = 0;
        bool all_in = clean;
        if (clean) {
            int spins = 0;
            do {
                w0 = ld_dev64(e);
                all_in = __all((w0 & ~0xFFFFFFFFull) == tag_hi);
                if (!all_in) __builtin_amdgcn_s_sleep(1);
            } while (!all_in && ++spins < fa.xc.spin_limit);
        }
        if (lane < R) row_lse[lane] = __uint_as_float((uint32_t)w0);
        if (!all_in && lane == 0) *wait_failed = 1;
    }
    __syncthreads();
    if (*wait_failed) {
        give_up();
        return;
    }
    if (tid == 0) st_dev64(fa.otag + k.slot0 + k.s, want ^ fa.xc.tag_flip);   // every wave's has landed
    // a stashed probability times its factor, f[row][w] for wave w's tiles (or
    // 2^(reference of the tile - lse)), is exact
    float* f = park;   // [R][4]
    if constexpr (!kU16) {
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) {
            const int row = rt * 16 + m16;
            if (G == 0 && row < R) f[row * kWaves + wave] = fast_exp2(M[rt] - row_lse[row]);
        }
        __syncthreads();
    }
    const int wn = min(a.window, k.qfull);
    const int r0 = max(0, k.qfull - wn - k.qoff) * g;   // first window row of this block
    const int nk = k.key_end - k.key_begin;
    // Quad q4 of the stash is four positions of a row: tile q4 / 8, wave
    // (tile % 4), keys 16 ((q4 / 4) & 1) + (q4 & 3) + 4 i of the tile.
    auto get = [&](int q4, int row) __attribute__((always_inline)) {
        const Elem* pq = stash + 4 * q4 + row * stride;
        if constexpr (kU16) {
            const uint2 c = *reinterpret_cast<const uint2*>(pq);
            return f32x4{of_code(c.x & 0xFFFFu), of_code(c.x >> 16), of_code(c.y & 0xFFFFu), of_code(c.y >> 16)};
        } else {
            return *reinterpret_cast<const f32x4*>(pq);
        }
    };
    auto factor = [&](int row, int tile, int w) __attribute__((always_inline)) {
        if constexpr (kU16) return fast_exp2(mtile[row * mts + tile] - row_lse[row]);
        else return f[row * kWaves + w];
    };
    auto key_of = [](int q4, int tile) { return tile * kTile + 16 * ((q4 >> 2) & 1) + (q4 & 3); };
    // (a later row block's scores go to its own copy and are added afterwards)
    float* scores = k.blk == 0 ? a.scores : fa.score_part + (size_t)(k.blk - 1) * fa.score_elems;
    // A wave takes 16 quads, its lane groups a quarter of the rows each (a row's
    // quads are consecutive, so the reads are free of bank conflicts), and lane
    // group i writes element i: two tiles' 64 scores in one store.
    auto scores_of = [&](int q4, bool valid, int tile, int w) __attribute__((always_inline)) {
        f32x4 sc = {0.f, 0.f, 0.f, 0.f};
        int row = r0 + G;
        for (; row + 12 < R; row += 16) {   // four rows' reads in flight
            f32x4 v[4];
            float fr[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = get(q4, row + 4 * j);
                fr[j] = factor(row + 4 * j, tile, w);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) sc += v[j] * fr[j];
        }
        for (; row < R; row += 4) sc += get(q4, row) * factor(row, tile, w);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sc[i] += shfl_xor_f(sc[i], 16);
            sc[i] += shfl_xor_f(sc[i], 32);
        }
        const float v = G == 0 ? sc[0] : G == 1 ? sc[1] : G == 2 ? sc[2] : sc[3];
        const int x = key_of(q4, tile) + 4 * G;
        if (valid && x < nk) scores[(size_t)k.unit * a.max_ctx + k.key_begin + x] = v;
    };
    // One score row per query head of the group: a head has few rows, so a
    // thread takes a quad and a head, row after row (64 heads over 8, 29920 and
    // 27334 keys, 2 positions: 70.6 us with the lane groups above, 53.7 so).
    auto head_scores_of = [&](int q4, int tile, int w, int hh) __attribute__((always_inline)) {
        f32x4 sc = {0.f, 0.f, 0.f, 0.f};
        int row = r0 + hh;
        for (; row + g < R; row += 2 * g) {
            const f32x4 v0 = get(q4, row), v1 = get(q4, row + g);
            const float f0 = factor(row, tile, w), f1 = factor(row + g, tile, w);
            sc += v0 * f0;
            sc += v1 * f1;
        }
        if (row < R) sc += get(q4, row) * factor(row, tile, w);
        float* hrow = scores + ((size_t)k.b * a.n_q_heads + k.c * g + hh) * a.max_ctx + k.key_begin;
        const int x = key_of(q4, tile);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (x + 4 * i < nk) hrow[x + 4 * i] = sc[i];
    };
    const int nq4 = max(kU16 ? ntile : ntile - kWaves, 0) * (kTile / 4);   // the tiles kept in LDS
    if (a.per_head) {
        for (int it = tid; it < nq4 * g; it += kThreads) {
            const int hh = it / nq4, q4 = it - hh * nq4;
            head_scores_of(q4, q4 >> 3, (q4 >> 3) & (kWaves - 1), hh);
        }
    } else {
        for (int q0 = 16 * wave; q0 < nq4; q0 += 16 * kWaves) {
            const int q4 = min(q0 + m16, nq4 - 1);
            scores_of(q4, q0 + m16 < nq4, q4 >> 3, (q4 >> 3) & (kWaves - 1));
        }
    }
    if constexpr (!kU16) {   // the waves' last tiles, through the stash's first four tiles
        __syncthreads();
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) {
            const int row = rt * 16 + m16;
            if (row < R) {
                f32x4* q = reinterpret_cast<f32x4*>(stash + row * stride + wave * kTile + 4 * G);
                q[0] = plast[rt][0];
                q[4] = plast[rt][1];
            }
        }
        __syncthreads();
        // (the tile of wave w's last 32 keys in the chunk)
        auto last_of = [&](int w) { return w + (ntile - 1 - min(w, ntile - 1)) / kWaves * kWaves; };
        if (a.per_head) {
            const int q4 = tid & 31, w = q4 >> 3;
            for (int hh = tid >> 5; w < ntile && hh < g; hh += kThreads / 32) head_scores_of(q4, last_of(w), w, hh);
        } else if (wave < 2) {
            const int q4 = 16 * wave + m16, w = q4 >> 3;
            scores_of(q4, w < ntile, last_of(w), w);
        }
    }

    // ---- 5. the output rows of this chunk's share ------------------------------------------
    if (nr > 0) {
        __syncthreads();   // the stash and the factors are free
        float* wts = reinterpret_cast<float*>(lds);                  // [256]
        f32x4* red = reinterpret_cast<f32x4*>(wts + 256);            // [256]
        wts[tid] = my_wt;
        // every chunk's partial output has landed once its tag is there
        {
            const uint64_t* e = fa.otag + k.slot0 + min(tid, k.nchunk - 1);
            int spins = 0;
            bool all_in;
            do {
                all_in = __all(ld_dev64(e) == want);
                if (!all_in) __builtin_amdgcn_s_sleep(1);
            } while (!all_in && ++spins < fa.xc.spin_limit);
            if (!all_in && lane == 0) *wait_failed = 1;
        }
        __syncthreads();
        if (*wait_failed) {
            give_up();
            return;
        }
        // eight groups of 32 lanes: gp of them per row, chunks sub, sub + gp, ...
        const int nrp = nr > 4 ? 8 : nr > 2 ? 4 : nr;
        const int gp = 8 / nrp, sg = tid >> 5, d4 = tid & 31, sub = sg % gp;
        auto write_row = [&](int r2, const f32x4& o) {
            const int jl = r2 / g, h = k.c * g + (r2 - jl * g);
            const int dim = 32 * ((d4 >> 1) & 3) + 8 * (d4 >> 3) + 4 * (d4 & 1);
            const size_t base = (((size_t)k.b * a.max_q + k.qoff + jl) * a.n_q_heads + h) * kHeadDim + dim;
            if (a.out_fp32) {
                *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + base) = o;
            } else {
                const uint2 pk = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
                *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.out) + base) = pk;
            }
        };
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int r2 = sg / gp; r2 < nr; r2 += nrp) {   // (one turn when gp > 1)
            const int rr = k.s + r2 * k.nchunk;
            acc = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int c0 = sub; c0 < k.nchunk; c0 += 8 * gp) {
                f32x4 v[8];
                float wt[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int c2 = min(c0 + u * gp, k.nchunk - 1);
                    const uint64_t* s64 =
                        reinterpret_cast<const uint64_t*>(a.part_o + (k.row0 + (size_t)c2 * R + rr) * kHeadDim + 4 * d4);
                    const float2 lo = __builtin_bit_cast(float2, ld_dev64(s64));
                    const float2 hi = __builtin_bit_cast(float2, ld_dev64(s64 + 1));
                    v[u] = f32x4{lo.x, lo.y, hi.x, hi.y};
                    wt[u] = c0 + u * gp < k.nchunk ? wts[r2 * np2 + c2] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += v[u] * wt[u];
            }
            if (gp == 1) write_row(rr, acc);
        }
        if (gp > 1) {
            red[tid] = acc;
            __syncthreads();
            if (sub == 0 && sg / gp < nr) {
                f32x4 o = red[tid];
                for (int q = 1; q < gp; ++q) o += red[tid + 32 * q];
                write_row(k.s + (sg / gp) * k.nchunk, o);
            }
        }
    }
    // every chunk has published, so has read the epoch
    if (tid == 0 && k.s == 0) {
        if (fa.epoch) epoch_advance(fa.epoch + k.grp);
        if (fa.heal) st_dev64(fa.heal + k.grp, fa.heal_value + k.grp);
    }
}

// Sequences of one call have their own row counts: each workgroup runs the
// body for its own number of row tiles (four would spill registers).
template <bool kPaged, bool kU16, bool kKeep = false>
__global__ __launch_bounds__(kThreads, 2) void verify_stream_kernel(StreamArgs fa) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ float2 wml[kWaves * kRowCap];
    __shared__ float row_lse[kRowCap];
    __shared__ int wait_failed;
    const SChunk k = schunk_of(fa, blockIdx.x);
    if (k.R <= 16)
        stream_chunk<1, kPaged, kU16, kKeep>(fa, k, lds, wml, row_lse, &wait_failed);
    else if (k.R <= 32)
        stream_chunk<2, kPaged, kU16, kKeep>(fa, k, lds, wml, row_lse, &wait_failed);
    else
        stream_chunk<3, kPaged, kU16, kKeep>(fa, k, lds, wml, row_lse, &wait_failed);
}

constexpr int kStreamMaxRows = 48;

// scores += the row blocks' copies, in block order (grid: key blocks, score
// rows of `heads` per sequence).  A pass over a few MB, bound by its chain of
// loads, so a thread has one key and the loads of two blocks go out together.  A chunk whose
// row blocks did not all get to their scores (a wait gave up) is left alone:
// its copies in the workspace are not this call's.  A block got there once its
// tag for the chunk is this call's; under capture the tag is that of the epoch
// before the group's finisher advanced it.
__global__ __launch_bounds__(kThreads) void verify_add_scores_kernel(StreamArgs fa, int heads) {
    const int row = blockIdx.y, b = row / heads;
    const int T = fa.v.seq.ctx[b], nb = fa.blocks[b], chunk = fa.chunk[b];
    const int key = blockIdx.x * kThreads + threadIdx.x;
    if (nb < 2 || (int)blockIdx.x * kThreads >= T) return;
    const int x = min(key, T - 1), s = x / chunk, nchunk = (T + chunk - 1) / chunk;
    const int c = (row - b * heads) / (heads / fa.v.n_kv_heads);
    const uint64_t* tag0 = fa.otag + fa.v.seq.item_start[b] + (size_t)c * nb * nchunk + s;
    const uint64_t* ep0 = fa.epoch ? fa.epoch + (size_t)(b * fa.v.n_kv_heads + c) * fa.max_blocks : nullptr;
    const size_t at = (size_t)row * fa.v.max_ctx + x;
    float v = fa.v.scores[at];
    bool done = key < T;
    for (int j0 = 0; j0 < nb; j0 += 2) {
        uint64_t tag[2], ep[2];
        float part[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int j = min(j0 + u, nb - 1);
            tag[u] = tag0[(size_t)j * nchunk];
            ep[u] = ep0 ? ep0[j] : 1ull;
            part[u] = fa.score_part[(size_t)max(j - 1, 0) * fa.score_elems + at];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            done = done && !epoch_is_dirty(ep[u]) && tag[u] == exchange_tag(fa.call_tag, ep[u] - 1);
            v += j0 + u > 0 && j0 + u < nb ? part[u] : 0.f;
        }
    }
    if (done) fa.v.scores[at] = v;
}
constexpr size_t kStreamStatic = kWaves * kRowCap * sizeof(float2) + kRowCap * 4 + 16;
constexpr size_t kStreamDynMax = 160 * 1024 / 2 - kStreamStatic;   // two workgroups per CU

// Once per device: raises the dynamic LDS limit and reads the workgroups a CU
// holds at the largest use (0 when the device cannot be asked).
int stream_setup() {
    constexpr int kMaxDevices = 64;
    static std::atomic<int> state[kMaxDevices];   // workgroups per CU + 1; 0: not read yet
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    const bool cached = dev >= 0 && dev < kMaxDevices;
    int st = cached ? state[dev].load(std::memory_order_relaxed) : 0;
    if (st == 0) {
        int blocks = 1 << 10;
        const void* fns[5] = {reinterpret_cast<const void*>(verify_stream_kernel<false, false>),
                              reinterpret_cast<const void*>(verify_stream_kernel<true, false>),
                              reinterpret_cast<const void*>(verify_stream_kernel<false, true>),
                              reinterpret_cast<const void*>(verify_stream_kernel<true, true>),
                              reinterpret_cast<const void*>(verify_stream_kernel<false, true, true>)};
        for (const void* f : fns) {
            int b = 0;
            if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStreamDynMax) != hipSuccess ||
                hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, f, kThreads, kStreamDynMax) != hipSuccess) {
                (void)hipGetLastError();
                return 0;
            }
            blocks = std::min(blocks, b);
        }
        st = blocks + 1;
        if (cached) state[dev].store(st, std::memory_order_relaxed);
    }
    return st - 1;
}

}  // namespace

int stream_blocks_per_cu() { return stream_setup(); }

// (a chunk of a paged cache has its pages in one set of wave_pages() registers;
// the LDS alone would hold more tiles for one or two rows)
int stream_max_tiles(int rows) {
    int tiles = 0;
    if (rows <= kStreamMaxRows)
        while (tiles < kPageRunTiles && stream_lds_bytes(rows, tiles + 1) <= kStreamDynMax) ++tiles;
    return tiles;
}

int stream_max_code_chunk(int row_tiles) {
    int chunk = 0;
    if (row_tiles * 16 <= kStreamMaxRows)
        while (code_lds_bytes(row_tiles * 16, chunk + 128) <= kStreamDynMax) chunk += 128;
    return chunk;
}

hipError_t launch_verify_stream(const StreamArgs& a, int n_slots, hipStream_t stream) {
    size_t dyn = 0;
    int rows = 0, max_ctx = 0;
    for (int b = 0; b < a.v.seq.n_seq; ++b) {
        const int r = a.block_pos[b] * a.v.group;
        rows = std::max(rows, r);
        max_ctx = std::max(max_ctx, a.v.seq.ctx[b]);
        dyn = std::max(dyn, a.u16 ? code_lds_bytes(r, a.chunk[b]) : stream_lds_bytes(r, a.chunk[b] / kTile));
    }
    if (dyn > kStreamDynMax || rows > kStreamMaxRows) return hipErrorInvalidValue;   // (the host plans less)
    for (int b = 0; b < a.v.seq.n_seq; ++b)
        if (a.chunk[b] > kPageRunTiles * kTile) return hipErrorInvalidValue;
    // (raises the dynamic LDS limit on the device's first launch)
    if (stream_setup() < 1) return hipErrorInvalidValue;
    const dim3 grid(n_slots), block(kThreads);
    if (a.v.block_table) {
        if (a.u16)
            hipLaunchKernelGGL((verify_stream_kernel<true, true>), grid, block, dyn, stream, a);
        else
            hipLaunchKernelGGL((verify_stream_kernel<true, false>), grid, block, dyn, stream, a);
    } else {
        if (a.u16 && a.keep)
            hipLaunchKernelGGL((verify_stream_kernel<false, true, true>), grid, block, dyn, stream, a);
        else if (a.u16)
            hipLaunchKernelGGL((verify_stream_kernel<false, true>), grid, block, dyn, stream, a);
        else
            hipLaunchKernelGGL((verify_stream_kernel<false, false>), grid, block, dyn, stream, a);
    }
    if (a.max_blocks > 1) {
        const int heads = a.v.per_head ? a.v.n_q_heads : a.v.n_kv_heads;
        hipLaunchKernelGGL(verify_add_scores_kernel, dim3((max_ctx + kThreads - 1) / kThreads, a.v.seq.n_seq * heads),
                           block, 0, stream, a, heads);
    }
    return hipGetLastError();
}

}  // namespace ssl
