// Fused Predict+Verify attention for bfloat16 caches with head_dim 128, the steps that do not fill the
// chip on the streaming kernel's terms: a few short sequences, and wide steps (prompt chunks,
// memory-token passes) over caches that fit the on-chip caches.
//
// What is computed: see attention.hip (MemoSight paper, Sections 2.1.1 and 2.3).  Such a call is bound
// by the chain of dependent latencies inside a workgroup, not by bytes.  So:
//   * No work plan: a (sequence, chunk of query rows, KV head) is cut into n_splits equal shares of
//     32-token tiles, cached tiles first, the step's own (in-flight) tiles last.  Everything a
//     workgroup needs first follows from its index and the kernel arguments.
//   * Steps of more than 64 rows per KV head are cut into chunks of 64 / group queries, a workgroup
//     each: the cache is read once per chunk, from L2 after the first.
//   * A workgroup has four waves: wave w owns row block w % 2 (32 query rows, the rotated Q operand in
//     registers) and every second tile of the share.  Only two waves hold states of the same rows, so
//     the merge at the end moves 32 KB through LDS (eight waves with both row blocks each: 512 KB).
//   * The shares' partial results go to a second launch, where more workgroups read them: the share that
//     finishes last folding them in the same launch was slower from 2 shares on (us inside / in a second
//     launch: 1 x 64 tokens, 7 queries, 2 shares 12.0 / 10.2; 8 x 200 tokens, 9 queries 14.8 / 12.9; 2 x 2000
//     tokens, 41 queries, 6 shares 22.3 / 20.6; 16 x 1000 tokens 20.6 / 20.1; never ahead).
// Tile layout, rotation, rounding and softmax are the streaming kernel's (attention_mfma.hip).  Tiles
// are assigned by index: results do not depend on timing.
#include <algorithm>

#include "attention.h"
#include "attention_tile.h"
#include "ms_internal.h"

namespace ms {

constexpr int kSplitWaves = 4;
constexpr int kSplitThreads = 64 * kSplitWaves;

struct SplitArgs {
    const uint16_t* pool_layer;
    const int* d_pt;
    const int* d_len;
    const float* inv_freq;
    const uint16_t* q;
    const uint16_t* k_new;
    const uint16_t* v_new;
    const int* pos;
    const int* ctx_new;
    uint16_t* out;
    float* ws;              // partials [sequence][chunk][share][KV head] of kPartFloats
    int n_q, n_verify, n_q_heads, n_kv_heads, group, max_pages;
    int n_chunks, per_chunk, n_splits, share_tiles;
    long page_elems;
    float scale_log2;
    int seq[MS_MAX_BATCH];
};

// LDS: cos/sin of the position ids the workgroup needs, one V tile per wave; at the end each wave's
// half of an O block (8 KB) and its softmax scalars lie over its V tile.
constexpr int kSplitMergeBytes = 32 * 64 * 4 + 2 * 64 * 4;
static_assert(kSplitMergeBytes <= kVTileBytes, "the merge region lies over the wave's V tile");
static int split_lds_bytes(int n_q) { return kSplitWaves * kVTileBytes + n_q * 64 * (int)sizeof(float2); }

__global__ __launch_bounds__(kSplitThreads, 2) void pv_attn_mfma_split(SplitArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int split = blockIdx.x, g = blockIdx.y, b = blockIdx.z / a.n_chunks, chunk = blockIdx.z % a.n_chunks;
    const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31, l16 = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), rb = w & 1, ts = w >> 1;
    float2* cs = reinterpret_cast<float2*>(smem + kSplitWaves * kVTileBytes);
    const int q0 = chunk * a.per_chunk, cn = min(a.per_chunk, a.n_q - q0), n_rows = cn * a.group;

    // ---- raw query rows of this wave's block: lane = row, d = 16 kk + 8 hf .. + 8 ----
    const int row = 32 * rb + l32;
    const bool live = row < n_rows;
    const int qi = q0 + (live ? row / a.group : 0);
    uint4 x[8];
    {
        const uint16_t* qp = a.q + (((size_t)b * a.n_q + qi) * a.n_q_heads + g * a.group + (live ? row % a.group : 0)) * kD + 8 * hf;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) x[kk] = *reinterpret_cast<const uint4*>(qp + 16 * kk);
    }
    const float inv_f = a.inv_freq[lane];

    // ---- this wave's tiles: every second one of the share.  Where a share begins does not depend on the
    // device's length, so that the length and the first page ids are asked for together; the last share
    // runs to the end, whatever has been committed since the host last looked ----
    const int seq = a.seq[b], L = uniform_load(a.d_len + seq);
    const int* pt = a.d_pt + (size_t)seq * a.max_pages;
    const int t_lo = split * a.share_tiles;
    const char* pool = reinterpret_cast<const char*>(a.pool_layer);
    const size_t page_bytes = (size_t)a.page_elems * 2;
    const uint32_t lane_off_k = ((uint32_t)g * 2 * MS_PAGE_SIZE * kD + l16 * kD + 8 * hf) * 2;
    const uint32_t lane_off_v = (((uint32_t)g * 2 + 1) * MS_PAGE_SIZE * kD + (lane >> 4) * kD + 8 * l16) * 2;
    // a cached tile's pages; entries past the sequence's last page are stale page ids: read, not used
    auto pages = [&](int t, int& pa, int& pb) {
        pa = uniform_load(pt + min(2 * t, a.max_pages - 1));
        pb = uniform_load(pt + min(2 * t + 1, a.max_pages - 1));
    };
    int t = t_lo + ts, pa, pb, pa_n, pb_n;
    pages(t, pa, pb);
    pages(t + 2, pa_n, pb_n);
    const int n_cache = (L + kTile - 1) / kTile, n_tiles = n_cache + (a.n_q + kTile - 1) / kTile;   // in-flight tiles behind the cached ones
    const int t_hi = split == a.n_splits - 1 ? n_tiles : min(n_tiles, t_lo + a.share_tiles);
    uint4 k[8], v[8];
    // tile T's rows (past the end: the last in-flight tile's again, so that loads are unconditional):
    // k: token l32, d = 16 kk + 8 hf .. + 8; v[rr]: token 4 rr + lane / 16, d = 8 l16 .. + 8
    auto load_k_tile = [&](int T, int pa, int pb) {
        const char* base;
        if (T < n_cache) {
            const bool one_page = 2 * T + 1 >= (L + MS_PAGE_SIZE - 1) / MS_PAGE_SIZE;   // the tile's second page does not exist
            base = pool + (size_t)(uint32_t)((lane & 16) && !one_page ? pb : pa) * page_bytes + lane_off_k;
        } else {
            const int tok = min(kTile * (T - n_cache) + l32, a.n_q - 1);
            base = reinterpret_cast<const char*>(a.k_new + (((size_t)b * a.n_q + tok) * a.n_kv_heads + g) * kD + 8 * hf);
        }
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) k[kk] = *reinterpret_cast<const uint4*>(base + 32 * kk);
    };
    auto load_v_tile = [&](int T, int pa, int pb) {
        const char* p[8];
        if (T < n_cache) {
            const bool one_page = 2 * T + 1 >= (L + MS_PAGE_SIZE - 1) / MS_PAGE_SIZE;
            const char* base_a = pool + (size_t)(uint32_t)pa * page_bytes + lane_off_v;
            const char* base_b = pool + (size_t)(uint32_t)(one_page ? pa : pb) * page_bytes + lane_off_v;
#pragma unroll
            for (int rr = 0; rr < 8; ++rr) p[rr] = (rr < 4 ? base_a : base_b) + 4 * (rr & 3) * kD * 2;
        } else {
            const uint16_t* v0 = a.v_new + ((size_t)b * a.n_q * a.n_kv_heads + g) * kD + 8 * l16;
#pragma unroll
            for (int rr = 0; rr < 8; ++rr)
                p[rr] = reinterpret_cast<const char*>(v0 + (size_t)(min(kTile * (T - n_cache) + 4 * rr + (lane >> 4), a.n_q - 1) * a.n_kv_heads) * kD);
        }
#pragma unroll
        for (int rr = 0; rr < 8; ++rr) v[rr] = *reinterpret_cast<const uint4*>(p[rr]);
    };
    load_k_tile(min(t, n_tiles - 1), pa, pb);
    load_v_tile(min(t, n_tiles - 1), pa, pb);

    // ---- cos/sin of the chunk's position ids (of every in-flight key's in a share that reaches them) ----
    const bool has_new = t_hi > n_cache && t_lo < t_hi;
    const int c_lo = has_new ? 0 : q0, c_hi = has_new ? a.n_q : q0 + cn;
    for (int i = c_lo + w; i < c_hi; i += kSplitWaves) {
        float sn, c;
        sincos_reduced((float)uniform_load(a.pos + b * a.n_q + i) * inv_f, &sn, &c);
        cs[i * 64 + lane] = make_float2(c, sn);
    }
    lds_barrier();
    // element i pairs with i + 64: register kk with kk + 4
    auto rotate = [&](uint4 (&r)[8], const float2* f, float scale) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const uint32_t w0[4] = {r[kk].x, r[kk].y, r[kk].z, r[kk].w};
            const uint32_t w1[4] = {r[kk + 4].x, r[kk + 4].y, r[kk + 4].z, r[kk + 4].w};
            uint32_t y0[4], y1[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float r0[2], r1[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float a0 = h ? __uint_as_float(w0[e] & 0xffff0000u) : __uint_as_float(w0[e] << 16);
                    const float a1 = h ? __uint_as_float(w1[e] & 0xffff0000u) : __uint_as_float(w1[e] << 16);
                    const float2 c = f[16 * kk + 8 * hf + 2 * e + h];
                    r0[h] = (a0 * c.x - a1 * c.y) * scale;
                    r1[h] = (a1 * c.x + a0 * c.y) * scale;
                }
                y0[e] = pack_bf16x2(r0[0], r0[1]);
                y1[e] = pack_bf16x2(r1[0], r1[1]);
            }
            r[kk] = make_uint4(y0[0], y0[1], y0[2], y0[3]);
            r[kk + 4] = make_uint4(y1[0], y1[1], y1[2], y1[3]);
        }
    };
    rotate(x, cs + qi * 64, a.scale_log2);   // (rows past the chunk's: computed like row 0 of it, not stored)

    float m = -INFINITY, l = 0.f;   // row maximum in use (log2 units); this lane's share of the row sum
    f32x16_t o[4];                  // O^T accumulators per d block; lane column = query row
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
    char* vl = smem + w * kVTileBytes;
    char* vwrite = vl + (lane >> 4) * kVRowBytes + l16 * 16;
    const char* vbase = vl + (4 * hf + (l16 >> 2)) * kVRowBytes + (16 * ((lane >> 4) & 1) + 4 * (l16 & 3)) * 2;   // see the streaming kernel

    auto qk = [&](f32x16_t& s) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, k[kk]), __builtin_bit_cast(bf16x8_t, x[kk]), s, 0, 0, 0);
    };
    auto weigh = [&](f32x16_t& s) {   // scores to softmax weights, and what a new maximum does to the state
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const bool grow = mx > m + kRescaleThreshold;
        if (__any(grow)) {
            const float f = grow ? __builtin_amdgcn_exp2f(m - mx) : 1.f;   // 2^-inf = 0 on the first tile
            m = grow ? mx : m;
            l *= f;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][i] *= f;
        }
        const float mu = m == -INFINITY ? 0.f : m;   // nothing visible to the row so far: its weights are 2^-inf
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            s[i] = __builtin_amdgcn_exp2f(s[i] - mu);
            sum += s[i];
        }
        l += sum;
    };
    auto pv = [&](const f32x16_t& s) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            uint4 pw;
            pw.x = pack_bf16x2(s[8 * ks + 0], s[8 * ks + 1]);
            pw.y = pack_bf16x2(s[8 * ks + 2], s[8 * ks + 3]);
            pw.z = pack_bf16x2(s[8 * ks + 4], s[8 * ks + 5]);
            pw.w = pack_bf16x2(s[8 * ks + 6], s[8 * ks + 7]);
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                const char* p0 = vbase + (16 * ks) * kVRowBytes + 64 * db;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p0));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p0 + 8 * kVRowBytes));
                const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, both), __builtin_bit_cast(bf16x8_t, pw), o[db], 0, 0, 0);
            }
        }
    };

    for (; t < t_hi; t += 2) {
        const bool cached = t < n_cache;
        const int tok0 = kTile * (t - n_cache);              // in-flight tile: its first token
        const int valid = cached ? L - t * kTile : a.n_q - tok0;
        if (!cached) rotate(k, cs + min(tok0 + l32, a.n_q - 1) * 64, 1.f);   // the step's own keys come as they are
        f32x16_t s;
        qk(s);
        const int tn = min(t + 2, n_tiles - 1);
        load_k_tile(tn, pa_n, pb_n);
        if (cached) {
            if (valid < kTile) mask_tail(s, valid, hf);
        } else {
            int ctx = a.ctx_new ? a.ctx_new[b * a.n_q + qi] : (qi < a.n_verify ? qi : a.n_verify);
            ctx = live ? min(ctx, a.n_q) : 0;
            mask_inflight(s, ctx - tok0, qi - tok0, hf);
        }
        weigh(s);
#pragma unroll
        for (int rr = 0; rr < 8; ++rr)   // rows past the end become zeros (stale pool bytes may be NaN)
            *reinterpret_cast<uint4*>(vwrite + 4 * rr * kVRowBytes) = 4 * rr + (lane >> 4) < valid ? v[rr] : make_uint4(0, 0, 0, 0);
        load_v_tile(tn, pa_n, pb_n);
        pages(t + 4, pa_n, pb_n);
        pv(s);
    }

    // ---- the two waves of a row block: each keeps two of the four d blocks and hands the other two over ----
    l += __shfl_xor(l, 32, 64);   // the half-waves hold the two halves of a row's sum
    float* mine = reinterpret_cast<float*>(smem + w * kVTileBytes);
    const float* other = reinterpret_cast<const float*>(smem + (w ^ 2) * kVTileBytes);
#pragma unroll
    for (int d2 = 0; d2 < 2; ++d2) {
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            const int i = 4 * i4;
            const float4 give = ts == 0 ? make_float4(o[2 + d2][i], o[2 + d2][i + 1], o[2 + d2][i + 2], o[2 + d2][i + 3])
                                        : make_float4(o[d2][i], o[d2][i + 1], o[d2][i + 2], o[d2][i + 3]);
            *reinterpret_cast<float4*>(mine + ((d2 * 4 + i4) * 64 + lane) * 4) = give;
        }
    }
    mine[32 * 64 + lane] = m;
    mine[33 * 64 + lane] = l;
    lds_barrier();
    const float m2 = other[32 * 64 + lane], l2 = other[33 * 64 + lane];
    const float m_all = fmaxf(m, m2), mu = m_all == -INFINITY ? 0.f : m_all;
    const float f1 = __builtin_amdgcn_exp2f(m - mu), f2 = __builtin_amdgcn_exp2f(m2 - mu);   // a wave without tiles: 2^-inf = 0
    const float l_all = l * f1 + l2 * f2;
    const float norm = a.n_splits == 1 ? 1.f / l_all : 1.f;
    float* part = a.ws + ((size_t)((size_t)blockIdx.z * a.n_splits + split) * a.n_kv_heads + g) * kPartFloats;
    uint16_t* op = a.out + (((size_t)b * a.n_q + qi) * a.n_q_heads + g * a.group + (live ? row % a.group : 0)) * kD;
#pragma unroll
    for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            const int db = 2 * ts + d2, i = 4 * i4;
            const float4 own = ts == 0 ? make_float4(o[d2][i], o[d2][i + 1], o[d2][i + 2], o[d2][i + 3])
                                       : make_float4(o[2 + d2][i], o[2 + d2][i + 1], o[2 + d2][i + 2], o[2 + d2][i + 3]);
            const float4 got = *reinterpret_cast<const float4*>(other + ((d2 * 4 + i4) * 64 + lane) * 4);
            const float4 r = make_float4((own.x * f1 + got.x * f2) * norm, (own.y * f1 + got.y * f2) * norm, (own.z * f1 + got.z * f2) * norm,
                                         (own.w * f1 + got.w * f2) * norm);
            if (a.n_splits > 1) {
                *reinterpret_cast<float4*>(part + 2 * kRows + (((rb * 4 + db) * 4 + i4) * 64 + lane) * 4) = r;
            } else if (live) {
                uint2 pk;
                pk.x = pack_bf16x2(r.x, r.y);
                pk.y = pack_bf16x2(r.z, r.w);
                *reinterpret_cast<uint2*>(op + 32 * db + 8 * i4 + 4 * hf) = pk;
            }
        }
    if (a.n_splits > 1 && ts == 0 && hf == 0) {
        part[row] = m_all;
        part[kRows + row] = l_all;
    }
}

// Folds the shares' partials in their order, normalises and writes the bf16 rows.  A workgroup takes one
// 32-row x 32-column block of a (sequence, chunk, KV head); a thread four columns of a row, with kBatch
// partials requested in one memory round trip.  Bound by those round trips: 26 shares (one sequence of
// 4096 tokens, 7 queries) in four trips of 8 or one of 32: 17.4 / 16.7 us per call of both launches (by blocks).
// As long as there is a compute unit for each, a workgroup of one wave takes a quarter of a block's columns, so that
// the partials come in through more compute units: one sequence of 4096 tokens 4.9 / 4.1 us for this launch; us per
// call of both launches, blocks / quarters, 28 / 4 heads: 1 x 1000 tokens 12.7 / 11.9, 1 x 4096 15.6 / 14.8, 1 x 16000
// 22.6 / 21.3, 2 x 4096 17.3 / 17.0; 32 / 8 heads 1 x 4096 17.1 / 15.7; behind from there on: 3 x 4096 18.0 / 18.4, 7 x
// 2000 17.1 / 18.2, 64 queries over 2 x 1000 18.6 / 19.3.
template <int kBatch>
__global__ __launch_bounds__(256) void pv_attn_mfma_fold(SplitArgs a) {
    const int quarter = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), rb = quarter >> 4, db = quarter >> 2 & 3;
    const int g = blockIdx.y, b = blockIdx.z / a.n_chunks, chunk = blockIdx.z % a.n_chunks;
    const int lane = threadIdx.x & 63, i4 = quarter & 3, hf = lane >> 5, row = 32 * rb + (lane & 31);
    const int q0 = chunk * a.per_chunk, n_rows = min(a.per_chunk, a.n_q - q0) * a.group;
    if (row >= n_rows) return;
    const size_t stride = (size_t)a.n_kv_heads * kPartFloats;
    const float* p0 = a.ws + ((size_t)blockIdx.z * a.n_splits * a.n_kv_heads + g) * kPartFloats;
    const int at = 2 * kRows + (((rb * 4 + db) * 4 + i4) * 64 + lane) * 4;
    float m = -INFINITY, l = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < a.n_splits; s0 += kBatch) {
        float pm[kBatch], pl[kBatch];
        float4 px[kBatch];
#pragma unroll
        for (int s = 0; s < kBatch; ++s) {   // past the end: the last one again, without weight
            const float* p = p0 + min(s0 + s, a.n_splits - 1) * stride;
            pm[s] = p[row];
            pl[s] = p[kRows + row];
            px[s] = *reinterpret_cast<const float4*>(p + at);
        }
        float mn = m;
#pragma unroll
        for (int s = 0; s < kBatch; ++s) mn = fmaxf(mn, pm[s]);
        const float mu = mn == -INFINITY ? 0.f : mn, fo = __builtin_amdgcn_exp2f(m - mu);
        m = mn;
        l *= fo;
        acc.x *= fo; acc.y *= fo; acc.z *= fo; acc.w *= fo;
#pragma unroll
        for (int s = 0; s < kBatch; ++s) {
            if (s0 + s >= a.n_splits) continue;
            const float f = __builtin_amdgcn_exp2f(pm[s] - mu);
            l += pl[s] * f;
            acc.x += px[s].x * f;
            acc.y += px[s].y * f;
            acc.z += px[s].z * f;
            acc.w += px[s].w * f;
        }
    }
    const float inv = 1.f / l;
    uint2 pk;
    pk.x = pack_bf16x2(acc.x * inv, acc.y * inv);
    pk.y = pack_bf16x2(acc.z * inv, acc.w * inv);
    *reinterpret_cast<uint2*>(a.out + (((size_t)b * a.n_q + q0 + row / a.group) * a.n_q_heads + g * a.group + row % a.group) * kD + 32 * db + 8 * i4 + 4 * hf) = pk;
}

constexpr int kSplitDecodeQueries = 16;   // a decode step: the streaming kernel could take it
static int split_chunks(int group, int n_q) { return (n_q + kRows / group - 1) / (kRows / group); }

// Tiles per share; 0: the call belongs on the streaming or the wide kernel.  Measured on 256 compute
// units, us per call with the second launch against the kernel that would take the call otherwise
// (7 queries, 28 / 4 heads unless said):
//   decode  1 x 1000 tokens 15 / 18, 1 x 4096 17 / 21, 1 x 16000 23 / 32, 4 x 4096 19 / 24, 8 x 4096
//           26 / 29, 16 x 2048 26 / 26; 32 x 2048 39 / 35, 16 x 8000 62 / 54.  The streaming kernel's last
//           workgroup folds 256 / pairs shares by itself, this kernel's waves read the cache once per row
//           block: the fewer the (sequence, KV head) pairs, the more (tile, KV head) pairs it takes until
//           the bytes count.  9 queries: 4 pairs 1 x 96000 57 / 64, 1 x 128000 71 / 74; 8 pairs 2 x 40000 47 /
//           51, 2 x 64000 68 / 65; 16 pairs 4 x 16000 38 / 40, 4 x 20000 46 / 46, 4 x 24000 52 / 50; 24 pairs
//           3 x 10000 38 / 37; 32 pairs 8 x 6000 31 / 33, 8 x 8000 38 / 38; 64 pairs 16 x 3000 32 / 31: the
//           break-even falls with the root of the pairs.  Below four shares per pair the streaming
//           kernel's eight waves per share hide more (32 x 500 tokens: 20 / 19)
//   wide    64 queries: 1 x 100 16 / 35, 1 x 2000 19 / 140, 4 x 2000 35 / 109, 8 x 4000 87 / 114, 32 / 8
//           heads 8 x 4000 91 / 97; 41 queries: 8 x 4000 68 / 100.  2.7 ns per (tile, KV head, chunk)
//           there; the wide kernel reads the cache once and is ahead from about 32768 of them on
// Shares are sized by the longest sequence, those of shorter ones end early, and nothing levels that: a
// decode batch counts with the tiles it would have if all sequences were that long, a wide step (whose
// throughput goes by the tiles there are) may have shares of up to 160 tiles.  us, this kernel / the other:
//   decode  9 queries, 28 / 4 heads: 12000 + 15 x 100 tokens 75 / 30, 8 x 500 .. 8000 35 / 32, 16 x 500 ..
//           4000 29 / 29, 4 x 1000 .. 16000 35 / 38, 8 x 200 .. 5000 26 / 29, 16 x 100 .. 1600 22 / 29; 32 / 8
//           heads: 8000 + 7 x 64 55 / 28, 2000 + 7 x 64 24 / 39
//   wide    one long sequence and 7 of 64 tokens, 64 queries: 5000 tokens (159 tiles) 105 / 134, 7000 (221)
//           142 / 130, 9000 179 / 127; 32 / 8 heads, 41 queries: 5000 107 / 112, 6000 (190) 125 / 109
constexpr long kSplitMaxTiles = 32768, kSplitMaxPairs = 64, kSplitMaxWideTiles = 32768;   // decode: over the root of the pairs
constexpr long kSplitMaxWideShare = 160;
int split_share_tiles(const ms_cache* c, const int* lens, int B, int n_q, size_t ws_partials, int* n_splits) {
    const long chunks = split_chunks(c->group, n_q), n_new = (n_q + kTile - 1) / kTile;
    long tiles = 0, longest = 0;
    for (int b = 0; b < B; ++b) {
        const long t = (lens[b] + kTile - 1) / kTile;
        tiles += t;
        longest = std::max(longest, t);
    }
    const long base = B * chunks * c->d.n_kv_heads;   // workgroups per share
    const bool wide = chunks > 1 || n_q > kSplitDecodeQueries;
    const long work = (wide ? tiles : B * longest) * c->d.n_kv_heads * chunks;
    if (!wide && (base > kSplitMaxPairs || work > kSplitMaxTiles || work * work * base > kSplitMaxTiles * kSplitMaxTiles)) return 0;
    if (wide && work > kSplitMaxWideTiles) return 0;
    // one workgroup per compute unit; two where one would leave a quarter of the chip idle
    const long per = longest + n_new;
    long s = std::max(1L, c->n_cus / base);
    if (4 * s * base < 3 * c->n_cus) s = std::max(1L, 2 * c->n_cus / base);
    s = std::min(s, (per + 1) / 2);                  // a tile for every wave
    s = std::min(s, std::max(32L, per / 8));         // more partials than that cost the second launch what the first gains
    s = std::min(s, std::max(1L, (long)ws_partials / (B * chunks)));
    const long share = (per + s - 1) / s;
    if (wide && share > kSplitMaxWideShare) return 0;
    *n_splits = (int)((per + share - 1) / share);
    return (int)share;
}

int launch_split(ms_cache* c, const AttnArgs& ga, const BatchMeta& bm, int B, int share_tiles, int n_splits, hipStream_t stream) {
    SplitArgs a;
    a.pool_layer = (const uint16_t*)ga.pool_layer;
    a.d_pt = ga.d_pt;
    a.d_len = ga.d_len;
    a.inv_freq = ga.inv_freq;
    a.q = (const uint16_t*)ga.q;
    a.k_new = (const uint16_t*)ga.k_new;
    a.v_new = (const uint16_t*)ga.v_new;
    a.pos = ga.pos;
    a.ctx_new = ga.ctx_new;
    a.out = (uint16_t*)ga.out;
    a.ws = ga.ws;
    a.n_q = ga.n_q;
    a.n_verify = ga.n_verify;
    a.n_q_heads = ga.n_q_heads;
    a.n_kv_heads = ga.n_kv_heads;
    a.group = ga.group;
    a.max_pages = ga.max_pages;
    a.per_chunk = kRows / ga.group;
    a.n_chunks = split_chunks(ga.group, ga.n_q);
    a.n_splits = n_splits;
    a.share_tiles = share_tiles;
    a.page_elems = ga.page_elems;
    a.scale_log2 = ga.scale * 1.44269504088896340736f;
    for (int b = 0; b < B; ++b) a.seq[b] = bm.seq[b];
    for (int b = B; b < MS_MAX_BATCH; ++b) a.seq[b] = 0;
    c->launches++;
    c->last_attention = n_splits > 1 ? "pv_attn_mfma_split+pv_attn_mfma_fold" : "pv_attn_mfma_split";
    hipLaunchKernelGGL(pv_attn_mfma_split, dim3(n_splits, a.n_kv_heads, B * a.n_chunks), dim3(kSplitThreads), split_lds_bytes(a.n_q), stream, a);
    if (n_splits > 1) {
        c->launches++;
        const int waves = 32l * a.n_kv_heads * B * a.n_chunks <= c->n_cus ? 1 : 4;
        const dim3 grid(32 / waves, a.n_kv_heads, B * a.n_chunks), block(64 * waves);
        if (n_splits <= 8) hipLaunchKernelGGL(pv_attn_mfma_fold<8>, grid, block, 0, stream, a);
        else if (n_splits <= 16) hipLaunchKernelGGL(pv_attn_mfma_fold<16>, grid, block, 0, stream, a);
        else hipLaunchKernelGGL(pv_attn_mfma_fold<32>, grid, block, 0, stream, a);
    }
    MS_HIP_TRY(hipGetLastError());
    return MS_OK;
}

int split_allow_lds() {
    MS_HIP_TRY(hipFuncSetAttribute((const void*)pv_attn_mfma_split, hipFuncAttributeMaxDynamicSharedMemorySize, split_lds_bytes(MS_MAX_QUERIES)));
    return MS_OK;
}

}  // namespace ms
