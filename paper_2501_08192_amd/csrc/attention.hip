// gfx950 (MI355X, CDNA4) kernels of the PRESERVE decode step: rotary table, decode attention over the block-structured cache, merge of its partials.
//
// Weights and the KV-cache are bf16 (or int8 codes with fp32 scales) in HBM; every accumulation is fp32.  The step
// is bound by HBM bandwidth (Section 2, "LLM decoding is memory BW-limited"), so the kernels are built around
// 16-byte-per-lane coalesced loads with many loads in flight per 64-lane wave; the matrix cores are used where a
// vector-ALU formulation would bind on arithmetic (batch > 2 projections, grouped-query attention).
#include <type_traits>

#include "device.h"

namespace psv {

// ------------------------------------------------------------------------------------ RoPE table

// Attention span of a sequence; a length outside the descriptor's range is treated as an empty sequence.
__device__ __forceinline__ int attn_span(int T, int max_tokens) { return T < 0 || T > max_tokens ? 0 : T; }

constexpr unsigned kAttnLast = 1u << 31;        // in AttnPlan::map: the sequence's last chunk

// Attention's work list of a step (AttnPlan), made by one wave with a lane per sequence (batch <= 64).  The chunk size is the
// smallest number of units with which the chunks of all sequences fit the slots.
__device__ __forceinline__ void make_attn_plan(const int32_t *seq_lens, int max_tokens, int batch, const AttnPlan &p, int lane)
{
    const int T = lane < batch ? attn_span(seq_lens[lane], max_tokens) : 0;
    const int units = (T + p.unit - 1) / p.unit;
    int n = 0;
    auto total = [&](int c) {
        n = (units + c - 1) / c;
        return (int)wave_sum((float)n);                 // exact: far below 2^24
    };
    const int all = (int)wave_sum((float)units);
    int lo = max((p.max_units + kAttnMaxChunks - 1) / kAttnMaxChunks, (all + p.slots - 1) / p.slots);
    if (lo < 1) lo = 1;
    if (total(lo) > p.slots) {                          // binary search: fewer chunks with larger sizes, and max_units always fits
        int hi = p.max_units;
        ++lo;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (total(mid) <= p.slots) hi = mid;
            else lo = mid + 1;
        }
        (void)total(lo);
    }
    if (lane < batch) p.chunks[lane] = n;
    int v = n;                                          // inclusive scan: within rows of 16, then the rows before
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    const int r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31), r2 = __builtin_amdgcn_readlane(v, 47);
    const int row = lane >> 4, start = v - n + (row > 0 ? r0 : 0) + (row > 1 ? r1 : 0) + (row > 2 ? r2 : 0);
    const int at = __builtin_amdgcn_readlane(start + n, 63);
    const int chunk = lo * p.unit;
    auto put = [&](int k, int b, int c, int nb, int Tb) {
        p.map[k] = make_uint2((unsigned)b << 24 | (unsigned)c << 12 | (unsigned)lo, (unsigned)min(Tb, (c + 1) * chunk) | (c == nb - 1 ? kAttnLast : 0u));
    };
    if (wave_max((float)n) < 2.f * batch) {             // a lane writes its sequence's chunks; long sequences: the wave, one by one
        for (int c = 0; c < n; ++c) put(start + c, lane, c, n, T);
    } else {
        for (int b = 0; b < batch; ++b) {
            const int nb = __builtin_amdgcn_readlane(n, b), sb = __builtin_amdgcn_readlane(start, b), Tb = __builtin_amdgcn_readlane(T, b);
            for (int c = lane; c < nb; c += 64) put(sb + c, b, c, nb, Tb);
        }
    }
    for (int k = at + lane; k < p.slots; k += 64) p.map[k] = make_uint2(0u, 0u);       // nothing to do
}

// cos/sin of the rotary angles at position seq_len-1, one row of 64 pairs per sequence.  The angle
// is formed and reduced in double (position * theta^(-2i/128)), so long contexts lose nothing to
// fp32 range reduction.  The position is the same for every layer, so this runs once per step -- as does the plan of the
// attention's work, by one more workgroup (blockIdx.x == batch).
__global__ __launch_bounds__(64) void k_rope_table(const int32_t *__restrict__ seq_lens, const double *__restrict__ inv_freq,
                                                   int max_tokens, int batch, float2 *__restrict__ table, AttnPlan plan)
{
    const int b = blockIdx.x, i = threadIdx.x;
    if (b == batch) {
        make_attn_plan(seq_lens, max_tokens, batch, plan, i);
        return;
    }
    int T = seq_lens[b];
    if (T < 1 || T > max_tokens) T = 1;
    float2 cs = make_float2(1.f, 0.f);
    if (inv_freq) {
        double sd, cd;
        sincos((double)(T - 1) * inv_freq[i], &sd, &cd);
        cs = make_float2((float)cd, (float)sd);
    }
    table[b * 64 + i] = cs;
}

hipError_t launch_rope_table(const int32_t *seq_lens, const double *inv_freq, int max_tokens, int batch, float2 *table,
                             const AttnPlan *plan, hipStream_t s)
{
    if (plan && (batch > 64 || plan->slots < batch)) return hipErrorInvalidValue;
    PSV_LAUNCH(k_rope_table, dim3(batch + (plan ? 1 : 0)), dim3(64), 0, s, seq_lens, inv_freq, max_tokens, batch, table, plan ? *plan : AttnPlan{});
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------ decode attention

constexpr float kAttnScale = 0.08838834764831845f * 1.4426950408889634f;   // 1/sqrt(128) * log2(e)

AttnSplit attn_split(uint32_t batch, uint32_t n_kv_heads, uint32_t max_seq, bool kv_int8)
{
    // Two workgroups of the attention kernel fit on a CU (register bound), 512 on the chip.  Measured on the
    // large shapes, one round of somewhat fewer workgroups (400-450) is fastest: a second, partial round costs a
    // whole chunk time, and a completely full chip is slower than a nearly full one.  So: at most kAttnResident
    // workgroups, chunks of whole steps (4 waves x one tile) and at most kAttnMaxChunks chunks per
    // (sequence, kv head).  psv_tune_attention replaces this guess by a measurement.
    const int unit = (kv_int8 ? kAttnTileTokensInt8 : kAttnTileTokens) * kAttnWaves;
    const uint64_t seqs = (uint64_t)batch * n_kv_heads;
    uint64_t max_chunks = kAttnResident / (seqs ? seqs : 1);
    if (max_chunks < 1) max_chunks = 1;
    if (max_chunks > (uint64_t)kAttnMaxChunks) max_chunks = kAttnMaxChunks;
    uint64_t chunk = ((uint64_t)max_seq + max_chunks - 1) / max_chunks;
    chunk = (chunk + unit - 1) / unit * unit;
    if (chunk < (uint64_t)unit) chunk = unit;
    AttnSplit sp;
    sp.chunk_tokens = (int)chunk;
    sp.n_chunks = (int)((max_seq + chunk - 1) / chunk);
    if (sp.n_chunks < 1) sp.n_chunks = 1;
    return sp;
}

// The split above divides the longest possible sequence: in a batch of mixed lengths most of its workgroups are empty and the
// longest sequence's chunks decide, and so it is for lengths far below max_seq.  A plan divides the lengths of the step, for
// the same one resident round of workgroups: as many slots per kv head, filled by the smallest chunk size that fits
// (make_attn_plan, once a step); a workgroup reads its chunk from its slot, a sequence's partials lie where its longest
// possible number of chunks would put them.  Measured: 39 sequences of 375-6000 tokens, int8 cache, 31.0 -> 15.9 us a layer.
bool attn_plan(uint32_t batch, uint32_t n_kv_heads, uint32_t max_seq, bool kv_int8, uint2 *map, size_t map_bytes, int *chunks, AttnPlan *p)
{
    p->unit = (kv_int8 ? kAttnTileTokensInt8 : kAttnTileTokens) * kAttnWaves;
    p->max_units = (int)(((uint64_t)max_seq + p->unit - 1) / p->unit);
    p->max_chunks = p->max_units < kAttnMaxChunks ? p->max_units : kAttnMaxChunks;
    uint64_t slots = kAttnResident / n_kv_heads;
    if (slots < batch) slots = batch;                               // every sequence needs one
    const uint64_t finest = (uint64_t)batch * p->max_chunks;
    p->slots = (int)(slots < finest ? slots : finest);
    p->map = map;
    p->chunks = chunks;
    // an entry holds a sequence in 8 bits, chunk and chunk size in 12 each
    return batch <= 64 && p->max_units < 4096 && p->slots * sizeof(uint2) <= map_bytes;
}

struct AttnArgs {
    const float *qkv;          // [batch][(nq+2nkv)*128] projection output, not yet rotated
    const uint8_t *q;          // prepared queries (k_attn_prep)
    int appended;              // ... which has also appended the new rows
    int batch;
    AttnPlan plan;             // plan.map null: chunks of chunk_tokens, n_chunks a sequence
    const float2 *rope;        // [batch][64] (cos, sin)
    KvView kv;
    int nq, nkv, chunk_tokens, n_chunks;
    float *part_ml;            // [batch][nkv][n_chunks][16][2]
    float *part_o;             // [batch][nkv][n_chunks][G][128]
    float *out_f32;            // [batch][nq*128]
    uint16_t *out_bf16;        // same as hi/lo bf16 planes (operand of the MFMA O projection)
    size_t out_plane;          // distance between the planes, elements
    int out_digits;            // out_bf16 receives int8 digit planes (operand of an int8 projection) instead
};

// Prepares the attention of a layer from the split-K partials of its QKV projection: sums them (split order), rotates queries
// and new key, leaves the queries as the attention's matrix operands (two bf16 planes [batch][nq * 128], or for an int8 cache
// two digit planes and a scale per head) and appends key and value to the cache.  A lane holds V channels and their rotary
// partners, 64 / V lanes a row of 128; all splits are requested at once.  Bound by its launch and one round
// trip.  What it takes out of the attention kernel stood there in every wave of every chunk, and in the workgroup of the last
// chunk as a second load of the tile with the new rows.
struct AttnPrepArgs {
    const float *part;          // [splits][batch][(nq + 2 nkv) * 128]
    int splits;
    const float2 *rope;
    KvView kv;
    int batch, nq, nkv;
    float *qkv;                 // the sums, [batch][(nq + 2 nkv) * 128]
    uint8_t *q;
};
template <bool Q8, int V, bool APPEND>
__global__ __launch_bounds__(64) void k_attn_prep(AttnPrepArgs a)
{
    constexpr int LANES = 64 / V;
    using Vec = typename std::conditional<V == 2, float2, float4>::type;
    const int lane = threadIdx.x % LANES, f = lane * V, nr = a.nq + 2 * a.nkv, nq = a.nq;
    const int row = blockIdx.x * V + threadIdx.x / LANES;
    const bool live = row < a.batch * nr;
    const int b = live ? row / nr : 0, j = live ? row % nr : 0;
    const size_t at = ((size_t)b * nr + j) * 128 + f, stride = (size_t)a.batch * nr * 128;
    union Piece { Vec v; float e[V]; };
    Piece lo[kSkMaxSplits], hi[kSkMaxSplits];
#pragma unroll
    for (int ks = 0; ks < kSkMaxSplits; ++ks) {
#pragma unroll
        for (int e = 0; e < V; ++e) lo[ks].e[e] = hi[ks].e[e] = 0.f;
        if (ks < a.splits) {
            lo[ks].v = ld_once(reinterpret_cast<const Vec *>(a.part + ks * stride + at));
            hi[ks].v = ld_once(reinterpret_cast<const Vec *>(a.part + ks * stride + at + 64));
        }
    }
    float2 cs[V];
#pragma unroll
    for (int e = 0; e < V; e += 2) *reinterpret_cast<float4 *>(cs + e) = *reinterpret_cast<const float4 *>(a.rope + b * 64 + f + e);
    // the new token's place, for the rows that go to the cache
    const KvView &kv = a.kv;
    const int T = APPEND ? attn_span(kv.seq_lens[b], kv.max_tokens) : 0, r = (T - 1) & 15;
    const bool key = j < nq + a.nkv;
    const int blk = live && j >= nq && T >= 1 ? kv_phys_block(kv.page_table, kv.max_blocks, kv.num_pool_blocks, b, (T - 1) >> 4) : -1;
    const int kvh = key ? j - nq : j - nq - a.nkv;
    Piece l = lo[0], h = hi[0];
#pragma unroll
    for (int ks = 1; ks < kSkMaxSplits; ++ks)
#pragma unroll
        for (int e = 0; e < V; ++e) { l.e[e] += lo[ks].e[e]; h.e[e] += hi[ks].e[e]; }
    if (live) {
        *reinterpret_cast<Vec *>(a.qkv + at) = l.v;
        *reinterpret_cast<Vec *>(a.qkv + at + 64) = h.v;
    }
    if (key) {          // queries and the key are rotated
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float l0 = l.e[e], h0 = h.e[e];
            l.e[e] = l0 * cs[e].x - h0 * cs[e].y;
            h.e[e] = h0 * cs[e].x + l0 * cs[e].y;
        }
    }
    const size_t plane = (size_t)a.batch * nq * 128, qat = ((size_t)b * nq + j) * 128 + f;
    if constexpr (Q8) {
        static_assert(V == 2, "a head is half a wave");
        const float amax = max32(fmaxf(fmaxf(fabsf(l.e[0]), fabsf(l.e[1])), fmaxf(fabsf(h.e[0]), fabsf(h.e[1]))));
        if (j >= nq) {
            if (blk < 0) return;
            const float sc = amax > 0.f ? amax / 127.0f : 1.0f;
            uint8_t *d = reinterpret_cast<uint8_t *>(key ? kv.k_pool : kv.v_pool) + ((size_t)blk * a.nkv + kvh) * PSV_KV_UNIT_BYTES_INT8;
            const int at8 = key ? r * 128 + f : f * 16 + r, step = key ? 1 : 16, far = key ? 64 : 64 * 16;
            d[at8] = quant_i8(l.e[0], sc);
            d[at8 + step] = quant_i8(l.e[1], sc);
            d[at8 + far] = quant_i8(h.e[0], sc);
            d[at8 + far + step] = quant_i8(h.e[1], sc);
            if (lane == 0) reinterpret_cast<float *>(d + 2048)[r] = sc;
            return;
        }
        if (!live) return;
        const float inv = amax > 0.f ? 127.0f / amax : 0.f;
        float d1[4], d2[4];
        two_digits(l.e[0] * inv, d1[0], d2[0]);
        two_digits(l.e[1] * inv, d1[1], d2[1]);
        two_digits(h.e[0] * inv, d1[2], d2[2]);
        two_digits(h.e[1] * inv, d1[3], d2[3]);
        const uint32_t w1 = pack_magic_bytes(d1[0], d1[1], d1[2], d1[3]), w2 = pack_magic_bytes(d2[0], d2[1], d2[2], d2[3]);
        *reinterpret_cast<uint16_t *>(a.q + qat) = (uint16_t)w1;
        *reinterpret_cast<uint16_t *>(a.q + qat + 64) = (uint16_t)(w1 >> 16);
        *reinterpret_cast<uint16_t *>(a.q + plane + qat) = (uint16_t)w2;
        *reinterpret_cast<uint16_t *>(a.q + plane + qat + 64) = (uint16_t)(w2 >> 16);
        if (lane == 0) reinterpret_cast<float *>(a.q + 2 * plane)[b * nq + j] = amax / 127.0f / 254.0f * kAttnScale;
    } else {
        if (j >= nq) {
            if (blk < 0) return;
            const bool tm = kv.token_major;
            uint16_t *d = key ? kv.k_pool : kv.v_pool;
            if (tm || key) d += (tm ? (((size_t)blk * 16 + r) * a.nkv + kvh) * 128 : (((size_t)blk * a.nkv + kvh) * 16 + r) * 128) + f;
            else d += (((size_t)blk * a.nkv + kvh) * 128 + f) * 16 + r;
            const int step = tm || key ? 1 : 16;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                d[e * step] = (uint16_t)f32_to_bf16(l.e[e]);
                d[(64 + e) * step] = (uint16_t)f32_to_bf16(h.e[e]);
            }
            return;
        }
        if (!live) return;
        uint16_t *q = reinterpret_cast<uint16_t *>(a.q) + qat;
        uint32_t wl[V / 2], wll[V / 2], wh[V / 2], whl[V / 2];
#pragma unroll
        for (int e = 0; e < V / 2; ++e) {
            pack_split(l.e[2 * e], l.e[2 * e + 1], wl[e], wll[e]);
            pack_split(h.e[2 * e], h.e[2 * e + 1], wh[e], whl[e]);
        }
#pragma unroll
        for (int e = 0; e < V / 2; ++e) {
            reinterpret_cast<uint32_t *>(q)[e] = wl[e];
            reinterpret_cast<uint32_t *>(q + 64)[e] = wh[e];
            reinterpret_cast<uint32_t *>(q + plane)[e] = wll[e];
            reinterpret_cast<uint32_t *>(q + plane + 64)[e] = whl[e];
        }
    }
}

// Who appends: this kernel, which has the rows at hand; but its end waits for the value rows' 2-byte stores, one into every
// channel, so that a larger bf16 batch's rows are left to the attention, which has the time for them, and the sums are taken in
// pieces of four channels: half the waves.  Measured here / there, us a layer, no windows: one kv head, 1k tokens, batch 5 70.2 /
// 71.5, 8 71.0 / 72.1, 12 72.8 / 73.9, 16 73.4 / 74.3, 17 77.6 / 78.6, 24 80.0 / 81.1, 32 83.0 / 83.3, 64 103.3 / 103.3; 8k tokens,
// 16 85.7 / 85.9, 24 97.4 / 97.2, 32 105.7 / 105.3; two kv heads, 12 108.3 / 109.8, 16 111.4 / 111.5, 24 122.5 / 122.4, 32 127.9 /
// 127.4, 64 160.6 / 160.0.  The two meet between batch 16 and 32, later with fewer kv heads and shorter sequences; the line is at
// the end of a batch tile.
static bool prep_appends(const KvView &kv, int batch) { return kv.int8 || batch <= 16; }

hipError_t launch_attn_prep(const float *part, int splits, const float2 *rope, KvView kv, int batch, int nq, int nkv, float *qkv,
                            void *q, hipStream_t s)
{
    if (splits < 1 || splits > kSkMaxSplits) return hipErrorInvalidValue;
    const AttnPrepArgs a{part, splits, rope, kv, batch, nq, nkv, qkv, static_cast<uint8_t *>(q)};
    const unsigned n_rows = (unsigned)(batch * (nq + 2 * nkv));
    if (kv.int8) PSV_LAUNCH((k_attn_prep<true, 2, true>), dim3((n_rows + 1) / 2), dim3(64), 0, s, a);
    else if (prep_appends(kv, batch)) PSV_LAUNCH((k_attn_prep<false, 2, true>), dim3((n_rows + 1) / 2), dim3(64), 0, s, a);
    else PSV_LAUNCH((k_attn_prep<false, 4, false>), dim3((n_rows + 3) / 4), dim3(64), 0, s, a);
    return hipGetLastError();
}

// What a workgroup works on: chunk c of sequence b, tokens [t_begin, t_end); its partial's place.
struct AttnChunk { int b, t_begin, t_end; bool last; size_t slot; };     // last: it holds the new token, t_end - 1
template <bool PREP>
__device__ __forceinline__ AttnChunk attn_chunk(const AttnArgs &a, int kvh)
{
    AttnChunk k;
    if (PREP && a.plan.map) {
        const uint2 m = a.plan.map[blockIdx.x];     // the same for the whole grid column: a scalar load
        const int c = (int)(m.x >> 12 & 0xfffu);
        k.b = (int)(m.x >> 24);
        k.t_begin = c * (int)(m.x & 0xfffu) * a.plan.unit;
        k.t_end = (int)(m.y & ~kAttnLast);
        k.last = m.y & kAttnLast;
        k.slot = ((size_t)k.b * a.nkv + kvh) * a.plan.max_chunks + c;
    } else {
        k.b = blockIdx.z;
        const int T = attn_span(a.kv.seq_lens[k.b], a.kv.max_tokens);
        k.t_begin = blockIdx.x * a.chunk_tokens;
        k.t_end = min(T, k.t_begin + a.chunk_tokens);
        k.last = T >= 1 && (int)blockIdx.x == (T - 1) / a.chunk_tokens;
        k.slot = ((size_t)k.b * a.nkv + kvh) * a.n_chunks + blockIdx.x;
    }
    return k;
}

// Split-K decode attention with everything around it fused in.  grid (chunks, kv heads, batch),
// 4 waves; wave w of chunk c takes the 32-token tiles c*chunk + (w + 4*it)*32.
//
//  * prologue: the G <= 16 query heads sharing the kv head are rotated (RoPE) straight into MFMA
//    B-fragments; the workgroup whose chunk holds token T-1 also rotates the new key, rounds key and
//    value to bf16, appends them to the cache and puts them into the tile it has already requested.
//    PREP: k_attn_prep has left the queries as fragments and, for small batches, appended the rows.
//  * main loop: all G heads ride in the N side of the MFMAs, so K and V are read from HBM once.
//        S^T[token][g]  = K[token][:] . Q[g][:]          A = K rows (token-major in the pool)
//        O^T[chan][g]  += V^T[chan][token] P[g][token]   A = V^T rows (channel-major in the pool)
//    A load instruction of K takes whole 128-byte lines, 8 tokens x 64 channels: row i of the A operand is half a line, the two
//    halves of a token in neighbouring rows.  Each half needs its own channels of Q, so every operand is multiplied with both
//    and a lane adds the two useful rows: twice the score products, on matrix cores that idle.  What that buys is the
//    non-temporal load (ONCE), which reads scattered 4 KB blocks at 6.5 TB/s instead of 5.75 (and at 5.1 when an instruction
//    takes half lines): 537 MB 103.8 -> 87.9 us, 268 MB 56.7 -> 49.3, 134 MB 29.4 -> 25.8.  So it is after a window that has prefetched
//    part of them: eight layers of the 70B-shaped TP=8 shard, cache-only, ordinary / non-temporal, batch 8 861 / 855 us, batch 32 1322 / 1313;
//    12 of the 8B-shaped one, batch 16 of 8k tokens 1629 / 1613, batch 64 of 2k 1790 / 1777.  The four groups of 8 tokens are chosen so
//    that lane (g, q) ends up with the scores of the 8 consecutive tokens 8q..8q+7 of its head: exactly the B-fragment the O^T MFMA
//    needs.  Probabilities never leave registers.
//  * epilogue: the 4 waves merge through LDS and the workgroup stores one partial (max, sum, O);
//    k_attn_merge then combines the partials of a (sequence, kv head) in chunk order.
//
// TM: token-major cache (both pools [block][16 tokens][kv head][128 channels]).  One head's key rows are then 256-byte
// pieces at a stride of n_kv_heads * 256 bytes -- the strided read of a shard with several local kv heads -- and are
// loaded exactly like the head-major rows.  The value tile arrives token-major as well, but the second contraction
// needs, per lane, eight consecutive tokens of one channel: each wave passes its 32 x 128 tile through LDS (whole
// 256-byte token rows in, 16-byte pieces XOR-swizzled by the token's group of eight so that the transposed 2-byte
// reads of all 64 lanes fall into different banks) and picks its fragments up transposed.
template <bool TM, bool PREP, bool ONCE>
__global__ __launch_bounds__(256, PREP ? 2 : 1) void k_attn(AttnArgs a)
{
    __shared__ __align__(16) uint16_t fresh[2][128];      // the new key and value row
    __shared__ float ms[kAttnWaves][16], ls[kAttnWaves][16];
    __shared__ f32x4 accs[kAttnWaves][8][64];      // TM: also the waves' value tiles (4 x 8 KiB) while the loop runs

    const int kvh = blockIdx.y;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, i = lane & 15, q4 = lane >> 4;
    const int nq = a.nq, nkv = a.nkv, G = nq / nkv;
    const KvView &kv = a.kv;
    const int qkv_rows = (nq + 2 * nkv) * 128;
    const AttnChunk ch = attn_chunk<PREP>(a, kvh);
    const bool planned = PREP && a.plan.map;
    if (planned && ch.t_end == 0) return;      // no chunk left for this workgroup
    const int b = ch.b, t_begin = ch.t_begin, t_end = ch.t_end;
    const float *qkv_b = a.qkv + (size_t)b * qkv_rows;
    const float2 *rope_b = a.rope + b * 64;

    // ---- K/V tile loader.  The addresses depend on the page table only, not on the sequence length (tokens
    //      past the span are masked later, and every logical block below max_blocks maps into the pool), so
    //      each wave issues the loads of its first tile right away, ahead of everything else in the kernel.
    // K row i of load (j, line): token 8 * (i / 4) + 2j + (i / 2) % 2 of the 32, half i % 2 of a 128-byte line
    const int tau = 8 * (i >> 2) + ((i >> 1) & 1), half = (i & 1) * 32 + q4 * 8;
    auto ld = [](const uint16_t *p) { if constexpr (ONCE) return ld16_once(p); else return ld16(p); };
    uint4 kf[4][2], vf[8];
    auto lookup = [&](int t0, int &blkA, int &blkB) {
        const int lb = t0 >> 4;
        blkA = kv_phys_block(kv.page_table, kv.max_blocks, kv.num_pool_blocks, b, lb);
        blkB = (lb + 1 < kv.max_blocks) ? kv_phys_block(kv.page_table, kv.max_blocks, kv.num_pool_blocks, b, lb + 1) : -1;
    };
    auto load_blocks = [&](int blkA, int blkB) {
        {
            const int blk = (i < 8) ? blkA : blkB;
            if (blk >= 0) {
                const uint16_t *base = TM ? kv.k_pool + (((size_t)blk * 16 + (tau & 15)) * nkv + kvh) * 128 + half
                                          : kv.k_pool + (((size_t)blk * nkv + kvh) * 16 + (tau & 15)) * 128 + half;
                const size_t row2 = TM ? (size_t)2 * nkv * 128 : (size_t)2 * 128;      // two tokens further
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    kf[j][0] = ld(base + j * row2);
                    kf[j][1] = ld(base + j * row2 + 64);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) { kf[j][0] = zero16(); kf[j][1] = zero16(); }
            }
        }
        if constexpr (TM) {
            // value tile, token-major: load j brings the whole rows of tokens 4j .. 4j+3 (lane = token q4, 16-byte piece i)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int blk = j < 4 ? blkA : blkB;
                vf[j] = blk >= 0 ? ld(kv.v_pool + (((size_t)blk * 16 + ((4 * j + q4) & 15)) * nkv + kvh) * 128 + i * 8) : zero16();
            }
            return;
        }
        // V^T fragments: row = channel dg*16 + i, k-slots of lane group q4 = tokens 8*q4 .. 8*q4+7
        {
            const int blk = (q4 < 2) ? blkA : blkB;
            if (blk >= 0) {
                const uint16_t *base = kv.v_pool + (((size_t)blk * nkv + kvh) * 128 + i) * 16 + (q4 & 1) * 8;
#pragma unroll
                for (int dg = 0; dg < 8; ++dg) vf[dg] = ld(base + dg * 16 * 16);
            } else {
#pragma unroll
                for (int dg = 0; dg < 8; ++dg) vf[dg] = zero16();
            }
        }
    };
    auto load_tile = [&](int t0) {
        int blkA, blkB;
        lookup(t0, blkA, blkB);
        load_blocks(blkA, blkB);
    };
    // Order of the first requests: page-table entries of the first tile, then the query rows and the rotary
    // table, then the tile itself.  Loads return in order, so the query can be rotated while the tile -- the one
    // request that goes all the way to HBM -- is still on its way.
    const int t_first = t_begin + w * kAttnTileTokens;
    const bool early = t_first < (planned ? t_end : kv.max_blocks * 16);      // planned: the span is known by now
    int blkA0 = -1, blkB0 = -1;
    if (early) lookup(t_first, blkA0, blkB0);
    float qlo[2][8], qhi[2][8];
    float2 qcs[2][8];
    bf16x8 qf[4], qfl[4];
    if constexpr (PREP) {
        const uint16_t *q = reinterpret_cast<const uint16_t *>(a.q) + ((size_t)b * nq + kvh * G + (i < G ? i : 0)) * 128 + q4 * 8;
        const size_t plane = (size_t)a.batch * nq * 128;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {        // a column past the heads repeats the first one; nothing of it is stored
            qf[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(q + ks * 32));
            qfl[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(q + plane + ks * 32));
        }
    } else if (i < G) {
        const float *qrow = qkv_b + (size_t)(kvh * G + i) * 128;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int f0 = ks * 32 + q4 * 8;
            *reinterpret_cast<float4 *>(qlo[ks]) = *reinterpret_cast<const float4 *>(qrow + f0);
            *reinterpret_cast<float4 *>(qlo[ks] + 4) = *reinterpret_cast<const float4 *>(qrow + f0 + 4);
            *reinterpret_cast<float4 *>(qhi[ks]) = *reinterpret_cast<const float4 *>(qrow + f0 + 64);
            *reinterpret_cast<float4 *>(qhi[ks] + 4) = *reinterpret_cast<const float4 *>(qrow + f0 + 68);
#pragma unroll
            for (int e = 0; e < 8; ++e) qcs[ks][e] = rope_b[f0 + e];
        }
    }
    if (early) load_blocks(blkA0, blkB0);

    // ---- Q fragments, rotated: lane (g = i, q4) holds channels ks*32 + q4*8 + e; channel f < 64
    //      pairs with f + 64, i.e. fragment ks with fragment ks + 2 of the same lane.  The rotated query is carried
    //      as two bf16 fragments, q = hi + lo: a single bf16 query (2^-9 relative) puts a 2e-3 relative error on the
    //      attention output, which wide models amplify past the tolerance in the MLP block that follows.
    if constexpr (!PREP) {
        uint4 z = zero16();
        qf[0] = qf[1] = qf[2] = qf[3] = __builtin_bit_cast(bf16x8, z);
        qfl[0] = qfl[1] = qfl[2] = qfl[3] = __builtin_bit_cast(bf16x8, z);
        if (i < G) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const float *lo = qlo[ks], *hi = qhi[ks];
                uint32_t lh[4], ll[4], hh[4], hl[4];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const float2 c0 = qcs[ks][e], c1 = qcs[ks][e + 1];
                    pack_split(lo[e] * c0.x - hi[e] * c0.y, lo[e + 1] * c1.x - hi[e + 1] * c1.y, lh[e >> 1], ll[e >> 1]);
                    pack_split(hi[e] * c0.x + lo[e] * c0.y, hi[e + 1] * c1.x + lo[e + 1] * c1.y, hh[e >> 1], hl[e >> 1]);
                }
                qf[ks] = __builtin_bit_cast(bf16x8, make_uint4(lh[0], lh[1], lh[2], lh[3]));
                qfl[ks] = __builtin_bit_cast(bf16x8, make_uint4(ll[0], ll[1], ll[2], ll[3]));
                qf[ks + 2] = __builtin_bit_cast(bf16x8, make_uint4(hh[0], hh[1], hh[2], hh[3]));
                qfl[ks + 2] = __builtin_bit_cast(bf16x8, make_uint4(hl[0], hl[1], hl[2], hl[3]));
            }
        }
    }

    // ---- append the new token's K and V (one workgroup per kv head does it)
    if (!PREP && ch.last) {
        const int T = t_end;
        if (tid < 64) {
            const int pos = T - 1;
            const int blk = kv_phys_block(kv.page_table, kv.max_blocks, kv.num_pool_blocks, b, pos >> 4);
            if (blk >= 0) {
                const float2 cs = rope_b[tid];
                const float *krow = qkv_b + (size_t)(nq + kvh) * 128;
                const float *vrow = qkv_b + (size_t)(nq + nkv + kvh) * 128;
                const float lo = krow[tid], hi = krow[tid + 64];
                const int r = pos & 15;
                const size_t tm_row = (((size_t)blk * 16 + r) * nkv + kvh) * 128;
                uint16_t *kdst = TM ? kv.k_pool + tm_row : kv.k_pool + (((size_t)blk * nkv + kvh) * 16 + r) * 128;
                kdst[tid] = (uint16_t)f32_to_bf16(lo * cs.x - hi * cs.y);
                kdst[tid + 64] = (uint16_t)f32_to_bf16(hi * cs.x + lo * cs.y);
                if constexpr (TM) {
                    kv.v_pool[tm_row + tid] = (uint16_t)f32_to_bf16(vrow[tid]);
                    kv.v_pool[tm_row + tid + 64] = (uint16_t)f32_to_bf16(vrow[tid + 64]);
                } else {
                    uint16_t *vdst = kv.v_pool + ((size_t)blk * nkv + kvh) * 128 * 16 + r;
                    vdst[(size_t)tid * 16] = (uint16_t)f32_to_bf16(vrow[tid]);
                    vdst[(size_t)(tid + 64) * 16] = (uint16_t)f32_to_bf16(vrow[tid + 64]);
                }
            }
        }
        // the new rows are read back within this workgroup only, through the CU's cache: the barrier's workgroup-scope
        // ordering suffices (later kernels see them after this one has ended)
        __syncthreads();   // uniform: the condition depends on the workgroup only
        if (early && T - 1 >= t_first && T - 1 < t_first + kAttnTileTokens) load_tile(t_first);   // now with the new entry
    }
    // ... and, where the preparing kernel has left it to this one, put it into the tile that holds it, which is on its way already: a
    // second load of it would cost the memory latency again.  (On the vector path, one sequence with 16k tokens, the second load is
    // the better one: 754 us for eight layers against 767.)
    if (PREP && ch.last && !a.appended) {
        const int pos = t_end - 1;
        const int blk = kv_phys_block(kv.page_table, kv.max_blocks, kv.num_pool_blocks, b, pos >> 4);
        if (tid < 64) {
            const float2 cs = rope_b[tid];
            const float *krow = qkv_b + (size_t)(nq + kvh) * 128;
            const float *vrow = qkv_b + (size_t)(nq + nkv + kvh) * 128;
            const float lo = krow[tid], hi = krow[tid + 64];
            const uint16_t k0 = (uint16_t)f32_to_bf16(lo * cs.x - hi * cs.y), k1 = (uint16_t)f32_to_bf16(hi * cs.x + lo * cs.y);
            const uint16_t v0 = (uint16_t)f32_to_bf16(vrow[tid]), v1 = (uint16_t)f32_to_bf16(vrow[tid + 64]);
            fresh[0][tid] = k0; fresh[0][tid + 64] = k1;
            fresh[1][tid] = v0; fresh[1][tid + 64] = v1;
            if (blk >= 0) {
                const int r = pos & 15;
                const size_t tm_row = (((size_t)blk * 16 + r) * nkv + kvh) * 128;
                uint16_t *kdst = TM ? kv.k_pool + tm_row : kv.k_pool + (((size_t)blk * nkv + kvh) * 16 + r) * 128;
                kdst[tid] = k0;
                kdst[tid + 64] = k1;
                if constexpr (TM) {
                    kv.v_pool[tm_row + tid] = v0;
                    kv.v_pool[tm_row + tid + 64] = v1;
                } else {
                    uint16_t *vdst = kv.v_pool + ((size_t)blk * nkv + kvh) * 128 * 16 + r;
                    vdst[(size_t)tid * 16] = v0;
                    vdst[(size_t)(tid + 64) * 16] = v1;
                }
            }
        }
        // the new rows are read back within this workgroup only, through LDS or the CU's cache: the barrier's workgroup-scope
        // ordering suffices (later kernels see them after this one has ended)
        __syncthreads();   // uniform: the condition depends on the workgroup only
        if (blk >= 0 && early && pos >= t_first && pos < t_first + kAttnTileTokens) {
            const int dt = pos - t_first;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint4 k8 = *reinterpret_cast<const uint4 *>(&fresh[0][c * 64 + half]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (tau + 2 * j == dt) kf[j][c] = k8;
            }
            if constexpr (TM) {
                const uint4 v8 = *reinterpret_cast<const uint4 *>(&fresh[1][i * 8]);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (4 * j + q4 == dt) vf[j] = v8;
            } else {
                const int e = dt - 8 * q4;          // token within this lane's eight, if it is one of them
                const uint32_t keep = e & 1 ? 0x0000ffffu : 0xffff0000u;
#pragma unroll
                for (int dg = 0; dg < 8; ++dg) {
                    const uint32_t v = fresh[1][dg * 16 + i], x = e & 1 ? v << 16 : v;
                    if (e >> 1 == 0) vf[dg].x = (vf[dg].x & keep) | x;
                    if (e >> 1 == 1) vf[dg].y = (vf[dg].y & keep) | x;
                    if (e >> 1 == 2) vf[dg].z = (vf[dg].z & keep) | x;
                    if (e >> 1 == 3) vf[dg].w = (vf[dg].w & keep) | x;
                }
            }
        }
    }

    const float kScale = kAttnScale;
    float m_run = -1.0e30f, l_part = 0.f;
    f32x4 acc[8];
#pragma unroll
    for (int dg = 0; dg < 8; ++dg) acc[dg] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int t0 = t_first; t0 < t_end; t0 += kAttnWaves * kAttnTileTokens) {
        if (t0 != t_first || !early) load_tile(t0);

        // d[j][h]: rows of half h hold the products of their line halves with the query's channels 64c + 32h; the other rows nothing of use
        f32x4 d[4][2];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < 2; ++c) x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[j][c]), qfl[2 * c + h], x, 0, 0, 0);
#pragma unroll
                for (int c = 0; c < 2; ++c) x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[j][c]), qf[2 * c + h], x, 0, 0, 0);
                d[j][h] = x;
            }
        // lane (g = i, q4) now holds tokens t0 + 8*q4 + e, e = 0..7
        float sv[8];
        const int tl = t0 + 8 * q4;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = e >> 1, r = 2 * (e & 1);
            sv[e] = (tl + e < t_end) ? (d[j][0][r] + d[j][1][r + 1]) * kScale : -INFINITY;
        }
        float tmax = sv[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) tmax = fmaxf(tmax, sv[e]);
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
        const float m_new = fmaxf(m_run, tmax);
        const float alpha = exp2f(m_run - m_new);
        float p[8], psum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            p[e] = exp2f(sv[e] - m_new);
            psum += p[e];
        }
        l_part = l_part * alpha + psum;
        m_run = m_new;
#pragma unroll
        for (int dg = 0; dg < 8; ++dg) acc[dg] *= alpha;

        if constexpr (TM) {
            // the wave's own 8 KiB of LDS: token rows in (piece index XOR 2 * (token / 8)), fragments out transposed
            unsigned char *vt = reinterpret_cast<unsigned char *>(&accs[w][0][0]);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int tok = 4 * j + q4;
                *reinterpret_cast<uint4 *>(vt + tok * 256 + ((i ^ (2 * (tok >> 3))) << 4)) = vf[j];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int dg = 0; dg < 8; ++dg) {
                const int piece = (2 * dg + (i >> 3)) ^ (2 * q4);        // tokens 8 q4 .. 8 q4 + 7 all have token / 8 = q4
                const unsigned char *src = vt + (8 * q4) * 256 + (piece << 4) + (i & 7) * 2;
                uint32_t h[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) h[e] = *reinterpret_cast<const uint16_t *>(src + e * 256);
                vf[dg] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();      // the next tile's rows overwrite the buffer only after these reads
        }
        // probabilities as two bf16 fragments as well (p = hi + lo)
        uint4 pk, pkl;
        pack_split(p[0], p[1], pk.x, pkl.x);
        pack_split(p[2], p[3], pk.y, pkl.y);
        pack_split(p[4], p[5], pk.z, pkl.z);
        pack_split(p[6], p[7], pk.w, pkl.w);
        if (t0 + kAttnTileTokens > t_end) {
            // ragged tail: cache slots past the span may hold anything (even NaN); blank them so
            // that 0 * garbage cannot reach the accumulators.
            uint32_t mlo[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                uint32_t m0 = (tl + 2 * h < t_end) ? 0x0000ffffu : 0u;
                uint32_t m1 = (tl + 2 * h + 1 < t_end) ? 0xffff0000u : 0u;
                mlo[h] = m0 | m1;
            }
#pragma unroll
            for (int dg = 0; dg < 8; ++dg) {
                vf[dg].x &= mlo[0]; vf[dg].y &= mlo[1]; vf[dg].z &= mlo[2]; vf[dg].w &= mlo[3];
            }
        }
        const bf16x8 pfrag = __builtin_bit_cast(bf16x8, pk), pfrag_lo = __builtin_bit_cast(bf16x8, pkl);
#pragma unroll
        for (int dg = 0; dg < 8; ++dg) {
            acc[dg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[dg]), pfrag_lo, acc[dg], 0, 0, 0);
            acc[dg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[dg]), pfrag, acc[dg], 0, 0, 0);
        }
    }

    // ---- merge the 4 waves (wave order)
    l_part += __shfl_xor(l_part, 16, 64);
    l_part += __shfl_xor(l_part, 32, 64);
    if (q4 == 0) ms[w][i] = m_run;
    __syncthreads();      // (TM: every wave is also done with its value tile in accs)
    const float M = fmaxf(fmaxf(ms[0][i], ms[1][i]), fmaxf(ms[2][i], ms[3][i]));
    const float sc = exp2f(m_run - M);
    if (q4 == 0) ls[w][i] = l_part * sc;
#pragma unroll
    for (int dg = 0; dg < 8; ++dg) accs[w][dg][lane] = acc[dg] * sc;
    __syncthreads();
    if (i < G) {
        const size_t slot = ch.slot;
        if (w == 0 && q4 == 0) {
            a.part_ml[(slot * 16 + i) * 2 + 0] = M;
            a.part_ml[(slot * 16 + i) * 2 + 1] = ls[0][i] + ls[1][i] + ls[2][i] + ls[3][i];
        }
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int dg = 2 * w + d;
            f32x4 v = accs[0][dg][lane];
            v += accs[1][dg][lane];
            v += accs[2][dg][lane];
            v += accs[3][dg][lane];
            *reinterpret_cast<float4 *>(a.part_o + (slot * G + i) * 128 + dg * 16 + 4 * q4) = make_float4(v[0], v[1], v[2], v[3]);
        }
    }

}

// ---- int8 cache: decode attention on the int8 matrix cores -------------------------------------------------
//
// Same split-K scheme and the same partials as k_attn, but the cache codes go into v_mfma_i32_16x16x64_i8 as
// they are (no widening): the floating-point operand of each contraction is cut into two int8 "digits" with
// a per-column scale, x ~ s * (d1 + d2 / 254), |d| <= 127, which keeps 15-16 bits of the column's largest
// element, and the two exact i32 results are recombined as 254 * D1 + D2 before one conversion to fp32.
//   S^T[token][g] = K[token][:] . Q[g][:]      A = K codes, 16 bytes = 16 channels per lane and k step
//                                              B = digits of the rotated query (scale per head)
//   O^T[chan][g] += V^T[chan][token] P'[g][token]   A = V codes, 16 bytes = the 16 tokens of one block
//                                              B = digits of P' = softmax numerator x value scale (scale per
//                                                  head and tile)
// A wave tile is 64 tokens = 4 cache blocks.  Row i of score tile m (m = 0..3) is token 16*(i/4) + 4m + i%4,
// so that lane (g, q4) ends up with the scores of tokens 16*q4 .. 16*q4+15 -- block q4, in byte order -- which
// is exactly the B operand of the second contraction.  Key scales multiply the scores, value scales the
// probabilities.  The appended rows are quantised per row in single precision (scale = max|v| / 127,
// code = rint(v / scale)), stored, and re-read by the wave whose tile holds them.
// Bound by the latency of a wave's few tiles (two at 39 sequences of 375-6000 tokens) and their vector work, 500 instructions
// for 17 KB: digit sums fold with 24-bit multiply-adds (the compiler's own choice is a 64-bit one, 48 a tile), what only the tile
// at a span's end or a missing block needs stands behind one branch a tile, and the next tile is requested into the registers that
// the scores (keys) and the second contraction (values) have just read.  Event times: that case 15.8 -> 14.5 us, batch 64 of 8k tokens
// 34.1 -> 32.1, batch 8 of 4k 6.9 -> 6.2, one sequence of 16k 8.8 -> 8.2.
// Two workgroups a CU in both forms, as attn_split counts on: left a register budget of 512 the form that prepares its own queries
// took 264, one workgroup a CU and two rounds for 257-448 of them (now 215).  Eight layers: eight kv heads, one sequence of 12k
// tokens 292 -> 262 us, two of 20k with two kv heads 413 -> 388.

template <bool PREP>
__global__ __launch_bounds__(256, 2) void k_attn_q8(AttnArgs a)
{
    constexpr int TT = kAttnTileTokensInt8;
    __shared__ float ms[kAttnWaves][16], ls[kAttnWaves][16];
    __shared__ f32x4 accs[kAttnWaves][8][64];

    const int kvh = blockIdx.y;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, i = lane & 15, q4 = lane >> 4;
    const int nq = a.nq, nkv = a.nkv, G = nq / nkv;
    const KvView &kv = a.kv;
    const int qkv_rows = (nq + 2 * nkv) * 128;
    const AttnChunk ch = attn_chunk<PREP>(a, kvh);
    const bool planned = PREP && a.plan.map;
    if (planned && ch.t_end == 0) return;      // no chunk left for this workgroup
    const int b = ch.b, t_begin = ch.t_begin, t_end = ch.t_end;
    const float *qkv_b = a.qkv + (size_t)b * qkv_rows;
    const float2 *rope_b = a.rope + b * 64;
    uint8_t *k8 = reinterpret_cast<uint8_t *>(kv.k_pool), *v8 = reinterpret_cast<uint8_t *>(kv.v_pool);

    // ---- tile loader (addresses depend on the page table only, so the first tile is requested right away)
    uint4 kc[4][2], vc[8];
    float4 ksc[4], vsc[4];
    auto lookup = [&](int t0, int &blkK, int &blkV) {
        const int lb = t0 >> 4;
        const int lbk = lb + (i >> 2), lbv = lb + q4;        // block of this lane's K rows / of its V tokens
        blkK = lbk < kv.max_blocks ? kv_phys_block(kv.page_table, kv.max_blocks, kv.num_pool_blocks, b, lbk) : -1;
        blkV = lbv < kv.max_blocks ? kv_phys_block(kv.page_table, kv.max_blocks, kv.num_pool_blocks, b, lbv) : -1;
    };
    // A block outside the table (or a corrupt entry) reads block 0 and is blanked before its use.
    bool bad_k = false, bad_ks = false, bad_v = false;
    auto load_k = [&](int blkK, int blkV) {
        const uint8_t *base = k8 + ((size_t)max(blkK, 0) * nkv + kvh) * PSV_KV_UNIT_BYTES_INT8 + (i & 3) * 128 + q4 * 16;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int j = 0; j < 2; ++j) kc[m][j] = *reinterpret_cast<const uint4 *>(base + m * 4 * 128 + j * 64);
        const float4 *ks4 = reinterpret_cast<const float4 *>(k8 + ((size_t)max(blkV, 0) * nkv + kvh) * PSV_KV_UNIT_BYTES_INT8 + 2048);
#pragma unroll
        for (int m = 0; m < 4; ++m) ksc[m] = ks4[m];
        bad_k = blkK < 0;
        bad_ks = blkV < 0;
    };
    auto load_v = [&](int blkV) {
        const uint8_t *unit = v8 + ((size_t)max(blkV, 0) * nkv + kvh) * PSV_KV_UNIT_BYTES_INT8;
        const float4 *vs4 = reinterpret_cast<const float4 *>(unit + 2048);
#pragma unroll
        for (int m = 0; m < 4; ++m) vsc[m] = vs4[m];
#pragma unroll
        for (int dg = 0; dg < 8; ++dg) vc[dg] = *reinterpret_cast<const uint4 *>(unit + (dg * 16 + i) * 16);
        bad_v = blkV < 0;
    };
    auto blank4 = [](bool z, auto &v) { v.x = z ? 0 : v.x; v.y = z ? 0 : v.y; v.z = z ? 0 : v.z; v.w = z ? 0 : v.w; };
    auto load_blocks = [&](int blkK, int blkV) {
        load_k(blkK, blkV);
        load_v(blkV);
    };
    auto load_tile = [&](int t0) {
        int blkK, blkV;
        lookup(t0, blkK, blkV);
        load_blocks(blkK, blkV);
    };
    // Order of the first requests: page-table entries of the first tile, then the query row and the rotary table,
    // then the tile itself; loads return in order, so the query digits are formed while the tile is on its way.
    const int t_first = t_begin + w * TT;
    const bool early = t_first < (planned ? t_end : kv.max_blocks * 16);      // planned: the span is known by now
    int blkK0 = -1, blkV0 = -1;
    if (early) lookup(t_first, blkK0, blkV0);
    const bool have_q = i < G;
    float4 q_lo[4], q_hi[4];
    float2 q_cs[16];
    uint4 qd1[2], qd2[2];
    float q_back = 0.f;                       // head scale / 254 * softmax scale, applied to 254*S1 + S2
    if constexpr (PREP) {
        const size_t row = (size_t)b * nq + kvh * G + (have_q ? i : 0), plane = (size_t)a.batch * nq * 128;
        const uint8_t *q = a.q + row * 128 + q4 * 16;
#pragma unroll
        for (int j = 0; j < 2; ++j) {           // a column past the heads repeats the first one; nothing of it is stored
            qd1[j] = *reinterpret_cast<const uint4 *>(q + j * 64);
            qd2[j] = *reinterpret_cast<const uint4 *>(q + plane + j * 64);
        }
        q_back = reinterpret_cast<const float *>(a.q + 2 * plane)[row];
    } else {
        const float *qrow = qkv_b + (size_t)(kvh * G + (have_q ? i : 0)) * 128 + q4 * 16;
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            q_lo[e4] = *reinterpret_cast<const float4 *>(qrow + e4 * 4);
            q_hi[e4] = *reinterpret_cast<const float4 *>(qrow + 64 + e4 * 4);
#pragma unroll
            for (int u = 0; u < 4; ++u) q_cs[e4 * 4 + u] = rope_b[q4 * 16 + e4 * 4 + u];
        }
    }
    if (early) load_blocks(blkK0, blkV0);

    // ---- query digits: lane (g = i, q4) holds channels j*64 + q4*16 + e (j = 0, 1; e = 0..15), the byte order of
    //      its K codes; channel f < 64 pairs with f + 64 for the rotation, i.e. j = 0 with j = 1 of the same lane
    if constexpr (!PREP) {
        float ql[16], qh[16];
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            const float4 lo = q_lo[e4], hi = q_hi[e4];
            const float2 c0 = q_cs[e4 * 4 + 0], c1 = q_cs[e4 * 4 + 1], c2 = q_cs[e4 * 4 + 2], c3 = q_cs[e4 * 4 + 3];
            ql[e4 * 4 + 0] = have_q ? lo.x * c0.x - hi.x * c0.y : 0.f;
            qh[e4 * 4 + 0] = have_q ? hi.x * c0.x + lo.x * c0.y : 0.f;
            ql[e4 * 4 + 1] = have_q ? lo.y * c1.x - hi.y * c1.y : 0.f;
            qh[e4 * 4 + 1] = have_q ? hi.y * c1.x + lo.y * c1.y : 0.f;
            ql[e4 * 4 + 2] = have_q ? lo.z * c2.x - hi.z * c2.y : 0.f;
            qh[e4 * 4 + 2] = have_q ? hi.z * c2.x + lo.z * c2.y : 0.f;
            ql[e4 * 4 + 3] = have_q ? lo.w * c3.x - hi.w * c3.y : 0.f;
            qh[e4 * 4 + 3] = have_q ? hi.w * c3.x + lo.w * c3.y : 0.f;
        }
        float amax = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) amax = fmaxf(amax, fmaxf(fabsf(ql[e]), fabsf(qh[e])));
        amax = fmaxf(amax, __shfl_xor(amax, 16, 64));
        amax = fmaxf(amax, __shfl_xor(amax, 32, 64));
        const float inv = amax > 0.f ? 127.0f / amax : 0.f;
        q_back = amax / 127.0f / 254.0f * kAttnScale;
        uint32_t w1[2][4], w2[2][4];
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            float a1[4], a2[4], b1[4], b2[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                two_digits(ql[e4 * 4 + u] * inv, a1[u], a2[u]);
                two_digits(qh[e4 * 4 + u] * inv, b1[u], b2[u]);
            }
            w1[0][e4] = pack_magic_bytes(a1[0], a1[1], a1[2], a1[3]);
            w2[0][e4] = pack_magic_bytes(a2[0], a2[1], a2[2], a2[3]);
            w1[1][e4] = pack_magic_bytes(b1[0], b1[1], b1[2], b1[3]);
            w2[1][e4] = pack_magic_bytes(b2[0], b2[1], b2[2], b2[3]);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            qd1[j] = make_uint4(w1[j][0], w1[j][1], w1[j][2], w1[j][3]);
            qd2[j] = make_uint4(w2[j][0], w2[j][1], w2[j][2], w2[j][3]);
        }
    }

    // ---- append the new token's K and V (one workgroup per kv head does it)
    if (!PREP && ch.last) {
        const int T = t_end;
        if (tid < 64) {
            const int pos = T - 1;
            const int blk = kv_phys_block(kv.page_table, kv.max_blocks, kv.num_pool_blocks, b, pos >> 4);
            if (blk >= 0) {    // uniform over the wave
                const float2 cs = rope_b[tid];
                const float *krow = qkv_b + (size_t)(nq + kvh) * 128;
                const float *vrow = qkv_b + (size_t)(nq + nkv + kvh) * 128;
                const float lo = krow[tid], hi = krow[tid + 64];
                const int r = pos & 15;
                const float k0 = lo * cs.x - hi * cs.y, k1 = hi * cs.x + lo * cs.y;
                const float v0 = vrow[tid], v1 = vrow[tid + 64];
                const float ka_max = wave_max(fmaxf(fabsf(k0), fabsf(k1)));
                const float va_max = wave_max(fmaxf(fabsf(v0), fabsf(v1)));
                const float ksc1 = ka_max > 0.f ? ka_max / 127.0f : 1.0f;
                const float vsc1 = va_max > 0.f ? va_max / 127.0f : 1.0f;
                const size_t unit = ((size_t)blk * nkv + kvh) * PSV_KV_UNIT_BYTES_INT8;
                uint8_t *kdst = k8 + unit, *vdst = v8 + unit;
                kdst[r * 128 + tid] = quant_i8(k0, ksc1);
                kdst[r * 128 + tid + 64] = quant_i8(k1, ksc1);
                vdst[tid * 16 + r] = quant_i8(v0, vsc1);
                vdst[(tid + 64) * 16 + r] = quant_i8(v1, vsc1);
                if (tid == 0) {
                    reinterpret_cast<float *>(kdst + 2048)[r] = ksc1;
                    reinterpret_cast<float *>(vdst + 2048)[r] = vsc1;
                }
            }
        }
        // the new rows are read back within this workgroup only, through the CU's cache: the barrier's workgroup-scope
        // ordering suffices (later kernels see them after this one has ended)
        __syncthreads();   // uniform: the condition depends on the workgroup only
        if (early && T - 1 >= t_first && T - 1 < t_first + TT) load_tile(t_first);   // now with the new entry
    }

    float m_run = -1.0e30f, l_part = 0.f;
    f32x4 acc[8];
#pragma unroll
    for (int dg = 0; dg < 8; ++dg) acc[dg] = f32x4{0.f, 0.f, 0.f, 0.f};

    // One tile.  MORE: another one follows; its blocks are looked up first, its keys are requested as soon as the scores have
    // taken this one's, its values when the second contraction has, into the same registers.
    constexpr int STEP = kAttnWaves * TT;
    auto tile = [&](int t0, auto more) {
        constexpr bool MORE = decltype(more)::value;
        int blkK, blkV;
        if (MORE) lookup(t0 + STEP, blkK, blkV);
        if (__any(bad_k || bad_ks)) {               // one branch a tile instead of a select for every register of it
#pragma unroll
            for (int m = 0; m < 4; ++m) { blank4(bad_k, kc[m][0]); blank4(bad_k, kc[m][1]); blank4(bad_ks, ksc[m]); }
        }

        // scores of tokens t0 + 16*q4 + e, e = 4m + j
        float sv[16];
        const int tl = t0 + 16 * q4;
        const bool ragged = t0 + TT > t_end;        // only the tile with the end of the span has slots to mask
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            i32x4 s1 = {0, 0, 0, 0}, s2 = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const i32x4 ak = __builtin_bit_cast(i32x4, kc[m][j]);
                s1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(ak, __builtin_bit_cast(i32x4, qd1[j]), s1, 0, 0, 0);
                s2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(ak, __builtin_bit_cast(i32x4, qd2[j]), s2, 0, 0, 0);
            }
            const float kk4[4] = {ksc[m].x, ksc[m].y, ksc[m].z, ksc[m].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sv[4 * m + j] = (float)mad_digits(s1[j], s2[j]) * q_back * kk4[j];
            }
        }
        if (ragged) {
#pragma unroll
            for (int e = 0; e < 16; ++e) sv[e] = tl + e < t_end ? sv[e] : -INFINITY;
        }
        if (MORE) load_k(blkK, blkV);
        if (__any(bad_v)) {
#pragma unroll
            for (int m = 0; m < 4; ++m) { blank4(bad_v, vsc[m]); blank4(bad_v, vc[m]); blank4(bad_v, vc[m + 4]); }
        }
        float tmax = sv[0], tmin = sv[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) {
            tmax = fmaxf(tmax, sv[e]);
            tmin = fminf(tmin, sv[e]);
        }
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
        const float m_new = fmaxf(m_run, tmax);
        const float alpha = exp2f(m_run - m_new);
        float pv[16], psum = 0.f, pmax = 0.f;
        // a probability below 2^-126 counts where its value scale is that much larger (out of line: 0.3 us a layer less, 0.2 for the check)
        if (__builtin_expect(__any(tmin < m_new - 126.f), 0)) {
#pragma unroll
            for (int e = 0; e < 16; ++e) pv[e] = exp2f(sv[e] - m_new);
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) pv[e] = exp2_raw(sv[e] - m_new);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const float vv4[4] = {vsc[m].x, vsc[m].y, vsc[m].z, vsc[m].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int e = 4 * m + j;
                psum += pv[e];
                pv[e] *= vv4[j];
            }
        }
        if (ragged) {
            // slots past the span may hold any scale: their probability is an exact zero only while it is not multiplied by
            // a NaN or an infinity
#pragma unroll
            for (int e = 0; e < 16; ++e) pv[e] = tl + e < t_end ? pv[e] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) pmax = fmaxf(pmax, fabsf(pv[e]));
        l_part = l_part * alpha + psum;
        m_run = m_new;
        pmax = fmaxf(pmax, __shfl_xor(pmax, 16, 64));
        pmax = fmaxf(pmax, __shfl_xor(pmax, 32, 64));
        const float p_inv = pmax > 0.f ? 127.0f / pmax : 0.f;
        const float p_back = pmax / 127.0f / 254.0f;
        uint32_t pw1[4], pw2[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            float a1[4], a2[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) two_digits(pv[4 * m + j] * p_inv, a1[j], a2[j]);
            pw1[m] = pack_magic_bytes(a1[0], a1[1], a1[2], a1[3]);
            pw2[m] = pack_magic_bytes(a2[0], a2[1], a2[2], a2[3]);
        }
        const i32x4 pd1 = {(int)pw1[0], (int)pw1[1], (int)pw1[2], (int)pw1[3]};
        const i32x4 pd2 = {(int)pw2[0], (int)pw2[1], (int)pw2[2], (int)pw2[3]};
#pragma unroll
        for (int dg = 0; dg < 8; ++dg) {
            const i32x4 av = __builtin_bit_cast(i32x4, vc[dg]);
            const i32x4 z = {0, 0, 0, 0};
            const i32x4 o1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, pd1, z, 0, 0, 0);
            const i32x4 o2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, pd2, z, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[dg][j] = fmaf(acc[dg][j], alpha, p_back * (float)mad_digits(o1[j], o2[j]));
        }
        if (MORE) load_v(blkV);
    };
    int t0 = t_first;
    if (!early && t0 < t_end) load_tile(t0);
    for (; t0 + STEP < t_end; t0 += STEP) tile(t0, std::true_type{});
    if (t0 < t_end) tile(t0, std::false_type{});

    // ---- merge the 4 waves (wave order); same partials as k_attn
    l_part += __shfl_xor(l_part, 16, 64);
    l_part += __shfl_xor(l_part, 32, 64);
    if (q4 == 0) ms[w][i] = m_run;
    __syncthreads();
    const float M = fmaxf(fmaxf(ms[0][i], ms[1][i]), fmaxf(ms[2][i], ms[3][i]));
    const float sc = exp2f(m_run - M);
    if (q4 == 0) ls[w][i] = l_part * sc;
#pragma unroll
    for (int dg = 0; dg < 8; ++dg) accs[w][dg][lane] = acc[dg] * sc;
    __syncthreads();
    if (i < G) {
        const size_t slot = ch.slot;
        if (w == 0 && q4 == 0) {
            a.part_ml[(slot * 16 + i) * 2 + 0] = M;
            a.part_ml[(slot * 16 + i) * 2 + 1] = ls[0][i] + ls[1][i] + ls[2][i] + ls[3][i];
        }
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int dg = 2 * w + d;
            f32x4 v = accs[0][dg][lane];
            v += accs[1][dg][lane];
            v += accs[2][dg][lane];
            v += accs[3][dg][lane];
            *reinterpret_cast<float4 *>(a.part_o + (slot * G + i) * 128 + dg * 16 + 4 * q4) = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
}

// Merge of the chunk partials of one (sequence, query head): grid (heads of a group, kv heads, batch), W waves of 64 lanes x 2
// channels.  Wave w takes chunks w, w + W, ...: its first two, and the (max, sum) pairs of the first sixteen, do not wait for the number of chunks, so
// that a sequence of up to 2 W of them costs one round trip.  Every wave forms the softmax weights for itself (no barrier before
// the one that adds the waves' sums, in wave order).  All orders are fixed, so the result is reproducible.  Bound by launch and
// that round trip.  Against 1024 threads a head, one channel a lane, weights by the first wave (two rounds of workgroups at batch
// 64 with 16 heads): that case 7.6 -> 4.8 us, batch 5-16 4.3 -> 3.8.
// PLAN: by the step's plan, whose number of chunks has to be read first (on the vector path that read cost 0.6 us a layer).
template <bool PLAN, int W>
__global__ __launch_bounds__(W * 64) void k_attn_merge(AttnArgs a)
{
    __shared__ float wl[W][kAttnMaxChunks + 8 * W];    // weights of the chunks, a row per wave (zeros behind them for the last batch of loads)
    __shared__ __align__(16) float psum[W][128];
    const int g = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);        // uniform: a wave's places, and which of them are past the chunks, are scalar
    const int nq = a.nq, nkv = a.nkv, G = gridDim.x, j = kvh * G + g;
    const int most = PLAN ? a.plan.max_chunks : a.n_chunks;       // partials a sequence has room for, and has
    const size_t slot0 = ((size_t)b * nkv + kvh) * most, stride = (size_t)G * 128;       // chunk to chunk
    const float *po = a.part_o + (slot0 * G + g) * 128 + 2 * lane;
    auto pair_of = [&](int sp) { return *reinterpret_cast<const float2 *>(a.part_ml + ((slot0 + sp) * 16 + g) * 2); };
    auto piece = [&](int sp, int n) { return ld_once(reinterpret_cast<const float2 *>(po + (size_t)min(sp, n - 1) * stride)); };     // n >= 1
    const int nc = PLAN ? a.plan.chunks[b] : a.n_chunks;
    constexpr int MU = kAttnMaxChunks / 64;
    float2 ml[MU];
    ml[0] = pair_of(min(lane, min(most, PLAN ? 16 : 64) - 1));
    const float2 v0 = piece(w, most), v1 = piece(w + W, most);
    if (PLAN && lane >= 16 && lane < nc) ml[0] = pair_of(lane);
    if (lane >= nc) ml[0] = make_float2(-1.0e30f, 0.f);
    float Mx = ml[0].x;
#pragma unroll
    for (int u = 1; u < MU; ++u) {
        const int sp = lane + 64 * u;
        ml[u] = make_float2(-1.0e30f, 0.f);
        if (64 * u < nc && sp < nc) ml[u] = pair_of(sp);
        Mx = fmaxf(Mx, ml[u].x);
    }
    Mx = wave_max(Mx);
    float den = 0.f;
#pragma unroll
    for (int u = 0; u < MU; ++u) {
        const int sp = lane + 64 * u;
        const float wgt = ml[u].y > 0.f ? exp2f(ml[u].x - Mx) : 0.f;       // 0 past the chunks
        wl[w][sp] = wgt;
        den += wgt * ml[u].y;
    }
    if (lane < 8 * W) wl[w][kAttnMaxChunks + lane] = 0.f;
    den = wave_sum(den);
    const float inv_den = den > 0.f ? 1.0f / den : 0.f;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // a place past the chunks holds anything: it is left out, not multiplied by zero
    float2 num = make_float2(0.f, 0.f);
    if (w < nc) num = make_float2(wl[w][w] * v0.x, wl[w][w] * v0.y);
    if (w + W < nc) num = make_float2(fmaf(wl[w][w + W], v1.x, num.x), fmaf(wl[w][w + W], v1.y, num.y));
    for (int sp = w + 2 * W; sp < nc; sp += 8 * W) {
        float2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = piece(sp + u * W, nc);
#pragma unroll
        for (int u = 1; u < 8; ++u)                        // past the chunks: the last one again, which may be an infinity
            if (sp + u * W >= nc) v[u] = make_float2(0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            num.x = fmaf(wl[w][sp + u * W], v[u].x, num.x);
            num.y = fmaf(wl[w][sp + u * W], v[u].y, num.y);
        }
    }
    *reinterpret_cast<float2 *>(&psum[w][2 * lane]) = num;
    __syncthreads();
    if (w) return;
    num = *reinterpret_cast<const float2 *>(&psum[0][2 * lane]);
#pragma unroll
    for (int k = 1; k < W; ++k) {                          // wave order
        const float2 p = *reinterpret_cast<const float2 *>(&psum[k][2 * lane]);
        num.x += p.x;
        num.y += p.y;
    }
    num.x *= inv_den;
    num.y *= inv_den;
    const size_t idx = ((size_t)b * nq + j) * 128 + 2 * lane;
    *reinterpret_cast<float2 *>(a.out_f32 + idx) = num;
    if (!a.out_digits) {
        uint32_t hi, lo;
        pack_split(num.x, num.y, hi, lo);
        *reinterpret_cast<uint32_t *>(a.out_bf16 + idx) = hi;
        *reinterpret_cast<uint32_t *>(a.out_bf16 + a.out_plane + idx) = lo;
        return;
    }
    // one head = one 128-element block of the digit planes: 32 lanes x 4 channels, the other half of the wave repeats them
    *reinterpret_cast<float2 *>(&psum[0][2 * lane]) = num;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int f = 4 * (lane & 31);
    const float4 v = *reinterpret_cast<const float4 *>(&psum[0][f]);
    store_digits4(reinterpret_cast<uint8_t *>(a.out_bf16), a.out_plane, nq * 128, (size_t)b, j * 128 + f, v);
}

static AttnArgs attn_args(const float *qkv, const float2 *rope, KvView kv, int batch, int nq, int nkv, AttnSplit sp,
                          float *part_ml, float *part_o, float *out_f32, uint16_t *out_bf16)
{
    const size_t out_plane = (size_t)((batch + 15) / 16 * 16) * nq * 128;
    return AttnArgs{qkv, nullptr, 0, batch, AttnPlan{}, rope, kv, nq, nkv, sp.chunk_tokens, sp.n_chunks, part_ml, part_o, out_f32, out_bf16, out_plane, 0};
}

template <bool PREP>
static void launch_attn_kernel(const AttnArgs &a, dim3 grid, hipStream_t s)
{
    if (a.kv.int8) PSV_LAUNCH((k_attn_q8<PREP>), grid, dim3(256), 0, s, a);
    else if (a.kv.token_major && a.kv.once) PSV_LAUNCH((k_attn<true, PREP, true>), grid, dim3(256), 0, s, a);
    else if (a.kv.token_major) PSV_LAUNCH((k_attn<true, PREP, false>), grid, dim3(256), 0, s, a);
    else if (a.kv.once) PSV_LAUNCH((k_attn<false, PREP, true>), grid, dim3(256), 0, s, a);
    else PSV_LAUNCH((k_attn<false, PREP, false>), grid, dim3(256), 0, s, a);
}

hipError_t launch_attn(const float *qkv, const float2 *rope, KvView kv, int batch, int nq, int nkv, AttnSplit sp,
                       float *part_ml, float *part_o, hipStream_t s)
{
    launch_attn_kernel<false>(attn_args(qkv, rope, kv, batch, nq, nkv, sp, part_ml, part_o, nullptr, nullptr),
                              dim3(sp.n_chunks, nkv, batch), s);
    return hipGetLastError();
}

hipError_t launch_attn_prepared(const void *q, const float *qkv, const float2 *rope, KvView kv, int batch, int nq, int nkv, AttnSplit sp, const AttnPlan *plan,
                                float *part_ml, float *part_o, hipStream_t s)
{
    AttnArgs a = attn_args(qkv, rope, kv, batch, nq, nkv, sp, part_ml, part_o, nullptr, nullptr);
    a.q = static_cast<const uint8_t *>(q);
    a.appended = prep_appends(kv, batch) ? 1 : 0;
    if (plan) a.plan = *plan;
    launch_attn_kernel<true>(a, plan ? dim3(plan->slots, nkv) : dim3(sp.n_chunks, nkv, batch), s);
    return hipGetLastError();
}

hipError_t launch_attn_merge(const float *part_ml, const float *part_o, int batch, int nq, int nkv, AttnSplit sp, const AttnPlan *plan,
                             float *out_f32, uint16_t *out_bf16, bool digits, hipStream_t s)
{
    AttnArgs a = attn_args(nullptr, nullptr, KvView{}, batch, nq, nkv, sp, const_cast<float *>(part_ml),
                           const_cast<float *>(part_o), out_f32, out_bf16);
    a.out_digits = digits ? 1 : 0;
    if (plan) a.plan = *plan;
    // eight waves where a sequence can have more than 64 chunks, else four: four rounds of the loop at most, or two
    const bool many = (plan ? plan->max_chunks : sp.n_chunks) > 64;
    const dim3 grid(nq / nkv, nkv, batch);
    if (plan && many) PSV_LAUNCH((k_attn_merge<true, 8>), grid, dim3(512), 0, s, a);
    else if (plan) PSV_LAUNCH((k_attn_merge<true, 4>), grid, dim3(256), 0, s, a);
    else if (many) PSV_LAUNCH((k_attn_merge<false, 8>), grid, dim3(512), 0, s, a);
    else PSV_LAUNCH((k_attn_merge<false, 4>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace psv
