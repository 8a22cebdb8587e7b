// SGNS node-embedding training for MI355X (gfx950): HIP kernels and the C ABI declared in ne.h.
//
// One batch of the embedding-training loop (Algorithm 1; Sec. II-A "Training Process") has four
// phases:
//
//   claim, resolve (ids only)  find out which rows several references of the batch name (a reference:
//          the source, the context or one of the K negatives of a pair).  claim takes the references
//          tile by tile: draws the negatives (Philox + alias table) and writes the tile's entries (a row's key, for one
//          reference or for most or all that a tile has of a hub), sorted by a hash of the key into bins.  resolve takes one bin per
//          workgroup: all entries of a row meet in one hash table in LDS.  A row with n > 1 references
//          gets n consecutive places in a list, one per reference, and ceil(n / 8)
//          work items for the apply kernel, which the batch's train launch moves together; an entry's place goes where the entry lies
//          (its tag).  Nothing goes through atomics in memory, and no state has to be cleared between batches.
//   train  one lane group per pair: gathers x = vertex[src] and the K+1 context rows (dwordx4),
//          reduces the K+1 dot products with DPP, forms g_j and the deltas.  A row that only this
//          pair names is rewritten in place from registers (old + delta, one plain store: the row
//          costs one read and one write).  A shared row is left untouched - other pairs must still
//          read its pre-batch value.  A reference's delta to it is a coefficient times a row: lr g_j
//          times the pair's source row, which is stored once for all of the pair's references, or one
//          times a sum that is stored.  The reference's place in the list takes the two.
//   apply  one lane group per work item: sums up to 8 consecutive entries of the list, coefficient times
//          row, and adds the sum to the table row.  A row with several items: their sums are summed in LDS
//          and, where several workgroups hold them, in a row of zeros with atomics; who arrives last
//          adds that to the table row.
//
// This is exactly minibatch-synchronous: no row that a second reference could read is written
// before the apply phase, and all contributions to a row are summed.  fp32 atomics on gfx950
// retire one dword per L2 channel clock, far below the rate of plain row stores, which is why only
// rows whose references several workgroups of the apply kernel hold see any, one per element and workgroup.
//
// claim and resolve never touch the tables, so for a run of batches (ne_train_block) they ride
// along in the train kernels of the batches before: kernel A = train(t) + resolve(t+1) + claim(t+2),
// kernel B = apply(t), two launches per batch (one in the per-sample mode).
//
// The same four phases serve three shapes of batch: pairs (ne_train_batch, ne_train_block), and walks
// (ne_train_walks: on-device augmentation) by entries or by segments, which differ only in how the
// references are laid out (claim) and in what a lane group or workgroup keeps on chip (train).
// Beside the exact step: the per-sample mode (ne_train_block_async: the same launches, but a shared
// row's deltas are added to the table row itself with atomics while other pairs may still read it, and
// there is no apply phase), the loss and pair-score kernels for evaluation, and table
// initialisation.
#include "ne_internal.h"

static thread_local std::string g_last_error;

ne_status fail(ne_status st, const std::string& msg)
{
    g_last_error = msg;
    return st;
}

namespace {

// ---------------------------------------------------------------------------------------------
// table initialisation: vertex ~ U(-0.5/d, 0.5/d), context = 0.  One float4 per thread-iteration.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void init_tables_kernel(float4* __restrict__ X, float4* __restrict__ C,
                                                          int64_t num_nodes, int32_t d4, float dimf,
                                                          uint32_t k0, uint32_t k1)
{
    const int64_t total = num_nodes * d4;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
        const uint64_t row = static_cast<uint64_t>(i / d4);
        const uint32_t q = static_cast<uint32_t>(i - static_cast<int64_t>(row) * d4);
        const uint4 r = philox4x32_10(make_uint4(static_cast<uint32_t>(row), static_cast<uint32_t>(row >> 32), q,
                                                 kStreamInit), k0, k1);
        float4 v;
        v.x = ((static_cast<float>(r.x >> 9) + 0.5f) * 0x1p-23f - 0.5f) / dimf;
        v.y = ((static_cast<float>(r.y >> 9) + 0.5f) * 0x1p-23f - 0.5f) / dimf;
        v.z = ((static_cast<float>(r.z >> 9) + 0.5f) * 0x1p-23f - 0.5f) / dimf;
        v.w = ((static_cast<float>(r.w >> 9) + 0.5f) * 0x1p-23f - 0.5f) / dimf;
        X[i] = v;
        C[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// ---------------------------------------------------------------------------------------------
// claim + resolve kernels.  Reference j of pair b: j = 0 the source row (vertex table), j = 1 the
// positive context row, j = 2.. negative j-2 (context table).
// key = row | (context table ? 1 << 31 : 0); rows are below 2^31 - 1, so no key is ~0.
//
// Detection of shared rows by partition instead of by one hash table in memory: a table entry that
// two compute dies touch costs a 64-byte transaction per store and per load, and a returning atomic
// for every lost position (measured at 458 752 references: 28 us of a 134 us batch, plus a linear pass
// that emptied the table again).  Here an entry is written once into a tile-local run of its bin and
// read once from there, runs of a few entries are one transaction, and everything that needs an
// atomic happens in LDS.  Riding in the train launch both phases together add 8 - 13 us to
// its 62 us (1 M nodes, dim 128, 65 536 pairs) or 75 us (32 M).  What that is, found by leaving parts of one batch's resolve phase out
// (its outputs were not needed): tags stored reference by reference, 4 bytes here and there, 4.5 us where as many side by
// side take 0.4 (eight dies hold the same lines in part and each writes its part back), so a tag goes to its entry's place, and
// the reference keeps where that is; an add per bin to a line of totals 2 - 3 us (adds to a line retire one after
// the other, and rows behind the same channel wait), so the bins' work items are counted by who moves them together; in the claim phase
// the alias table's random reads, 5 us (32 M nodes).
// Entries, ids, Philox, LDS: written, read or done twice, they cost nothing more.
constexpr uint32_t kNoKey = 0xFFFFFFFFu;

// How the references of a batch are binned.
//   bins   a power of two.  512 .. 1024 references per bin where the batch is large, so that the distinct
//          rows among them half fill a table of 2048 slots (16 KB of LDS, which a train launch can give to
//          every workgroup without losing one; 2048 references and 4096 slots cost such a batch 6 %, 512 and
//          1024 twice as many segments and 8 %); a smaller batch gets up to 256 bins, one per compute unit,
//          of 128 .. 256 references, because a bin is one chain of dependent accesses (64 .. 128: 6 % slower
//          on batches of 28 000 references), and below 64 bins they are shorter still (256 throughout: 2 .. 4 % slower on
//          batches of 300 .. 4000 references, 10 % where such batches follow each other in one call).  Up to 256
//          references are one bin, claimed and resolved in one launch (12 against 14.6 us for a call with one pair; of
//          up to 512: the resolve phase takes 1 .. 2 us more than the launch it saves).  Beyond 1200 references per bin
//          at 4096 bins (4.9 M references) up to 16 384 bins, as many as 16-bit counters of the claim phase in 32 KB of
//          LDS allow; beyond that the bins get longer, and are resolved in several ranges of the hash.  (4096 bins
//          throughout: 2^22 pairs with K = 5, dim 16 take 6.4 ms, in 8 ranges, instead of 3.9 in one; with K = 62, dim 4 147
//          instead of 79, 64 ranges and 8.)
//   tile   references per claim workgroup: at least 4 per bin, so that runs of a bin's entries are worth an
//          access and the segment table stays a quarter of the entries; 2 beyond 4096 bins, where tiles are few and long.
//   slots  of a bin's LDS table (4096 only for the batches whose claim counters take 32 KB as well), and the distinct
//          rows (full) at which it counts as too small, where a bin is gone through in passes.
struct Binning { uint32_t bits, tile, tiles, slot_bits, full; };
constexpr uint32_t kWordBinBits = 12, kMaxBinBits = 14;      // most bins whose claim counters are whole words; most bins
constexpr uint32_t kMinTile = 256;
constexpr uint64_t kOneBin = 256;
constexpr struct { uint32_t bits; uint64_t refs; } kBinSteps[] = {{5, 64}, {6, 128}, {8, 256}, {kWordBinBits, 1024}, {kMaxBinBits, 1200}};   // most references per bin, up to 2^bits bins
constexpr Binning binning(uint64_t refs)
{
    Binning b{};
    b.bits = 0;
    for (const auto& step : kBinSteps)
        while (refs > kOneBin && b.bits < step.bits && (step.refs << b.bits) < refs) ++b.bits;
    b.tile = (b.bits > kWordBinBits ? 2u : 4u) << b.bits;
    if (b.tile < kMinTile) b.tile = kMinTile;
    b.tiles = static_cast<uint32_t>((refs + b.tile - 1) / b.tile);
    const uint64_t mean = refs >> b.bits;
    b.slot_bits = mean <= 128 ? 9 : mean <= 400 ? 10 : mean <= 1200 ? 11 : 12;
    b.full = b.slot_bits == 9 ? 255u : (5u << b.slot_bits) / 8u;
    return b;
}
// Segment words that a batch of up to `refs` references can need.
inline uint64_t max_segs(uint64_t refs)
{
    return refs <= (kBinSteps[4].refs << kWordBinBits) ? refs / 4 + (1u << kWordBinBits) : refs / 2 + (1u << kMaxBinBits);
}

struct PrepArgs {
    const int2* pairs;    // pair mode: the batch's pairs
    const int32_t* walks; // walk mode (pairs == nullptr): the batch's walks, int32 [..][walk_len]
    int32_t walk_len, window;
    uint32_t refs;        // references of the batch; 0 = nothing to prepare
    uint32_t R;           // references per pair (K + 2) / per walk entry (1 + window * (K + 1)) / per walk segment
    uint32_t seg_entries; // walk mode: 0 = one reference group per walk entry; else entries per segment
    uint32_t segs_per_walk;
    int32_t K;
    uint64_t sample_base;
    uint32_t k0, k1;
    const uint2* alias;
    uint64_t alias_n;
    int32_t alias_base;
    Binning bin;
    int32_t* ids;
    uint32_t* where;
    uint2* items;         // of the bins, as are hub_items; nullptr: nothing is left to apply (per-sample mode)
    uint4* hub_items;
    uint4* bins;
    uint32_t* keys;
    uint32_t* tags;
    uint32_t* segs;
    int32_t* neg_out;
    // sample prefetch riding along (ne_train_block_pinned): fetch_blocks helper workgroups copy fetch_n
    // pairs from pinned host memory (fetch_src: its device address) into the staging ring (fetch_dst)
    const int2* fetch_src;
    int2* fetch_dst;
    int64_t fetch_n;
    uint32_t fetch_blocks;
};

__device__ __forceinline__ uint32_t bin_of(uint32_t key, uint32_t bits) { return bits ? hash_bits(key) >> (32u - bits) : 0u; }

// Drawing a reference's id is a chain of dependent memory accesses with next to no arithmetic, so each thread
// draws several references at once, all loads of which are issued before the first is waited for: the functions below
// take U references per thread, first + u * T + tid < last for u < U, and return their keys (kNoKey where there is none);
// ids and requested negatives go to memory.
// Everything here comes for workgroups of T = 256 threads, which ride in train launches, and of 512, for launches of its own
// that leave most of the chip idle (launch_prepare).
constexpr uint32_t kTileStep = 2048;       // references per workgroup and step, whose keys stay in registers
template <uint32_t T> constexpr int kTileKeys = kTileStep / T;

// Philox words of a negative: its slot of the alias table and the word that decides between slot and alias.
__device__ __forceinline__ uint2 draw_slot(const PrepArgs& a, uint64_t sample, uint32_t k)
{
    const uint4 rnd = philox4x32_10(make_uint4(static_cast<uint32_t>(sample), static_cast<uint32_t>(sample >> 32), k, kStreamNegative), a.k0, a.k1);
    const uint32_t n = static_cast<uint32_t>(a.alias_n);      // (below 2^31)
    return make_uint2(static_cast<uint32_t>((static_cast<uint64_t>(rnd.x) * n + __umulhi(rnd.y, n)) >> 32), rnd.z);
}
__device__ __forceinline__ uint32_t drawn_id(const PrepArgs& a, uint2 draw, uint2 entry)
{
    return static_cast<uint32_t>(a.alias_base) + (draw.y < entry.x ? draw.x : entry.y);
}

template <int U, uint32_t T>
__device__ __forceinline__ void claim_pair_refs(const PrepArgs& a, uint32_t first, uint32_t last, unsigned tid, uint32_t* key)
{
    const uint32_t R = a.R;
    // per reference: a negative's alias entry and draw; else the pair, and which half of it.
    // (A wavefront has references of every kind, so all lanes draw, and one load serves both kinds.)
    uint2 e[U], draw[U];
    uint32_t sources = 0u, negatives = 0u;        // a bit per reference
    const uint32_t step_b = T / R, step_j = T - step_b * R;
    uint32_t t0 = min(first + tid, last - 1u), b = t0 / R, j = t0 - b * R;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (first + u * T >= last) break;         // (uniform)
        draw[u] = draw_slot(a, a.sample_base + b, j - 2u);
        const uint2* from = j < 2u ? reinterpret_cast<const uint2*>(a.pairs) + b : a.alias + draw[u].x;
        e[u] = *from;
        sources |= static_cast<uint32_t>(j == 0u) << u;
        negatives |= static_cast<uint32_t>(j >= 2u) << u;
        if (first + (u + 1) * T + tid < last) {       // (else this one again)
            b += step_b;
            j += step_j;
            if (j >= R) { j -= R; b += 1u; }
        }
        __builtin_amdgcn_sched_barrier(0);   // one draw's registers at a time; the loads stay in flight
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t t = first + u * T + tid;
        key[u] = kNoKey;
        if (t < last) {
            const bool source = sources >> u & 1u, negative = negatives >> u & 1u;
            const uint32_t id = negative ? drawn_id(a, draw[u], e[u]) : source ? e[u].x : e[u].y;
            if (negative && a.neg_out) {
                uint32_t at = t;
                asm volatile("" : "+v"(at));         // (the division is not worth a register each until here)
                a.neg_out[static_cast<int64_t>(at) - 2 * static_cast<int64_t>(at / R) - 2] = static_cast<int32_t>(id);
            }
            a.ids[t] = static_cast<int32_t>(id);
            key[u] = id | (source ? 0u : 0x80000000u);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// What a reference of the walk modes is: its kind (0 a source's row, 1 a context's row, 2 a negative), the walk, the two
// entries of it that decide whether the reference exists (of a source's row the entry and the one after it, of a context's
// row the last of its sources and itself), and a negative's sample of the batch and number.
struct WalkRef { uint32_t kind, walk, i, c, sample, k; };

// Walk mode (on-device augmentation, Algorithm 1 "network augmentation"): the batch is a set of
// walks int32 [n][L]; position i of a walk is the source of the pairs (walk[i], walk[i+j]),
// 1 <= j <= window, that exist (both entries non-negative, i + j < L).  References of position p:
//   0                          the source row (vertex table), present if the position has a pair
//   1 + (j-1)(K+1)             the context row of pair j
//   1 + (j-1)(K+1) + 1 + k     negative k of pair j, drawn for sample index sample_base + p*window + (j-1)
// Absent references get id -1 and no key.
__device__ __forceinline__ WalkRef walk_ref(const PrepArgs& a, uint32_t t)
{
    const uint32_t L = static_cast<uint32_t>(a.walk_len), W = static_cast<uint32_t>(a.window), K1 = static_cast<uint32_t>(a.K + 1);
    const uint32_t p = t / a.R, q = t - p * a.R, r = p / L, i = p - r * L;
    if (q == 0) return {0u, r, i, i + 1, 0u, 0u};
    const uint32_t j = (q - 1) / K1, k = q - 1 - j * K1;
    return {k == 0u ? 1u : 2u, r, i, i + j + 1, p * W + j, k - 1u};
}

// Walk mode by segments: a walk is cut into segments of E = seg_entries consecutive entries, one
// workgroup of the train kernel each.  The workgroup sums on chip everything its entries contribute
// to each other, so a segment names every row once.  References of segment (walk r, entries p0 ..
// p0+E-1), CT = E + window - 1:
//   q < E                    vertex row of entry p0 + q, present if that entry starts a sample
//   E <= q < E + CT          context row of entry p0 + 1 + (q - E), present if one of the segment's
//                            entries has it as a sample's context (the last window-1 of them belong
//                            to the next segment's entries too: both segments name them)
//   E + CT + (e*window + j-1)*K + k   negative k of sample (entry p0 + e, offset j)
__device__ __forceinline__ WalkRef seg_ref(const PrepArgs& a, uint32_t t)
{
    const uint32_t L = static_cast<uint32_t>(a.walk_len), W = static_cast<uint32_t>(a.window), K = static_cast<uint32_t>(a.K);
    const uint32_t E = a.seg_entries, CT = E + W - 1;
    const uint32_t seg = t / a.R, q = t - seg * a.R, r = seg / a.segs_per_walk, p0 = (seg - r * a.segs_per_walk) * E;
    if (q < E) return {0u, r, p0 + q, p0 + q + 1, 0u, 0u};
    if (q < E + CT) {
        const uint32_t c = p0 + 1 + (q - E);
        return {1u, r, min(c - 1, p0 + E - 1), c, p0, 0u};       // (sample: the first entry that can be its source)
    }
    const uint32_t n = q - E - CT, pj = n / K, e = pj / W, j = pj - e * W;     // pj = e * W + (j - 1)
    return {2u, r, p0 + e, p0 + e + j + 1, (r * L + p0 + e) * W + j, n - pj * K};
}

template <int U, bool SEG, uint32_t T>
__device__ __forceinline__ void claim_walk_refs(const PrepArgs& a, uint32_t first, uint32_t last, unsigned tid, uint32_t* key)
{
    const uint32_t L = static_cast<uint32_t>(a.walk_len), W = static_cast<uint32_t>(a.window);
    auto ref = [&](uint32_t t) { return SEG ? seg_ref(a, t) : walk_ref(a, t); };
    // the draw does not wait for the walk's entries, which say whether it is needed (when it did, four times in turn: 17
    // instead of 22 us for the first claim of 170 walks of 80 entries, 5.6 instead of 4.8 for 22 of 40)
    int32_t src[U], ctx[U];
    uint2 e[U], draw[U];
    uint32_t kinds = 0u;          // two bits per reference
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (first + u * T >= last) break;         // (uniform)
        const WalkRef w = ref(min(first + u * T + tid, last - 1u));
        const int32_t* wk = a.walks + static_cast<int64_t>(w.walk) * L;
        kinds |= w.kind << (2 * u);
        src[u] = wk[min(w.i, L - 1u)];
        ctx[u] = wk[min(w.c, L - 1u)];
        if (w.i >= L) src[u] = -1;
        if (w.c >= L) ctx[u] = -1;
        if (a.K > 0) {
            draw[u] = draw_slot(a, a.sample_base + w.sample, w.k);
            e[u] = a.alias[w.kind == 2u ? draw[u].x : 0u];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t t = first + u * T + tid;
        key[u] = kNoKey;
        if (t < last) {
            const uint32_t kind = kinds >> (2 * u) & 3u;
            bool valid = src[u] >= 0 && ctx[u] >= 0;
            int32_t id = ctx[u];
            if (kind == 2u) {
                if (valid) {
                    id = static_cast<int32_t>(drawn_id(a, draw[u], e[u]));
                    if (a.neg_out) {
                        const WalkRef w = ref(t);
                        a.neg_out[static_cast<int64_t>(w.sample) * a.K + w.k] = id;
                    }
                }
            } else {
                if (kind == 0u) id = src[u];
                if (!valid && id >= 0 && (SEG || kind == 0u)) {      // by its other contexts, by (segments) its other sources
                    const WalkRef w = ref(t);
                    const int32_t* wk = a.walks + static_cast<int64_t>(w.walk) * L;
                    if (kind == 0u)
                        for (uint32_t c = w.i + 2; !valid && c <= w.i + W && c < L; ++c) valid = wk[c] >= 0;
                    else
                        for (uint32_t i = w.c > w.sample + W ? w.c - W : w.sample; !valid && i < w.i; ++i) valid = wk[i] >= 0;
                }
            }
            a.ids[t] = valid ? id : -1;
            if (valid) key[u] = static_cast<uint32_t>(id) | (kind == 0u ? 0u : 0x80000000u);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Inclusive prefix sum over the 64 lanes of a wavefront, in registers (through LDS, one permutation after the other: 0.25 us, and
// five of these lie in a batch's critical path).  All lanes call this together.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v)
{
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x111, 0xF, 0xF, false));    // row_shr 1, 2, 4, 8: inside 16 lanes
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x112, 0xF, 0xF, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x114, 0xF, 0xF, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x118, 0xF, 0xF, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xA, 0xF, false));    // lane 15 of a row to the next row
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xC, 0xF, false));    // lane 31 to the upper half
    return v;
}

// Exclusive prefix sums of v and w over the T threads of a workgroup, in place, and their totals.  part: T / 32 words of LDS.
template <uint32_t T>
__device__ __forceinline__ void block_exclusive_scan(uint32_t& v, uint32_t& w, uint32_t* part, uint32_t* total_v, uint32_t* total_w)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t inc_v = wave_inclusive_scan(v), inc_w = wave_inclusive_scan(w);
    lds_barrier();              // part may still be read from an earlier scan
    if (lane == 63u) { part[wave] = inc_v; part[T / 64u + wave] = inc_w; }
    lds_barrier();
    uint32_t before_v = 0, before_w = 0, sum_v = 0, sum_w = 0;
#pragma unroll
    for (uint32_t q = 0; q < T / 64u; ++q) {
        if (q == wave) { before_v = sum_v; before_w = sum_w; }
        sum_v += part[q];
        sum_w += part[T / 64u + q];
    }
    v = before_v + inc_v - v;
    w = before_w + inc_w - w;
    *total_v = __builtin_amdgcn_readfirstlane(sum_v);
    *total_w = __builtin_amdgcn_readfirstlane(sum_w);
}

// LDS of the claim phase: a counter per bin (beyond 2^kWordBinBits bins 16 bits each), the scan's 32 words and, if the tile is one
// step, its entries and what claim_rows needs to find them, else a bit per bin and the table of claim_long_rows.
constexpr uint32_t kLongRows = 512;        // (as many workgroups fit on a compute unit as without them)
__host__ __device__ inline uint32_t counter_words(uint32_t bits) { return bits > kWordBinBits ? 1u << (bits - 1u) : 1u << bits; }
inline size_t claim_lds_bytes(const Binning& b)
{
    const size_t rows = b.tile <= kTileStep ? b.tile * (2 * sizeof(uint32_t) + sizeof(uint16_t)) : (1u << b.bits) / 8 + kLongRows * 2 * sizeof(uint32_t);
    return (static_cast<size_t>(counter_words(b.bits)) + 32) * sizeof(uint32_t) + rows;
}

// Layout of a batch's references.
enum RefMode { kPairRefs, kWalkRefs, kSegRefs };

// The ids and keys of a step's references.
template <RefMode MODE, uint32_t T>
__device__ __forceinline__ void claim_refs(const PrepArgs& a, uint32_t step, uint32_t last, uint32_t* key)
{
    constexpr int H = T == 256 ? kTileKeys<T> / 2 : kTileKeys<T>;       // (all eight of 256 threads at once take 95 registers)
    const unsigned tid = threadIdx.x;
#pragma unroll
    for (int h = 0; h < kTileKeys<T> / H; ++h) {
        if (MODE == kPairRefs) claim_pair_refs<H, T>(a, step + h * T * H, last, tid, key + h * H);
        else claim_walk_refs<H, MODE == kSegRefs, T>(a, step + h * T * H, last, tid, key + h * H);
    }
}

// Where the entries of each bin start in the tile, to hist, and where they end, entries | references << 16, to the segment
// table; *total: the last end.  hist holds the numbers: kSingles of entries, which are one reference each; kCounts of entries |
// of references << 16; kEntries of entries, and only that half of the segment words is written.
// False, with nothing written, if a bin has more than `most`; kRefs: then only the references' ends are written, to their half, and
// the numbers stay, but for such bins, which start from zero and have a bit in `many`.
enum BinCounts { kSingles, kCounts, kRefs, kEntries };
template <uint32_t T>
__device__ __forceinline__ bool start_bins(const PrepArgs& a, uint32_t tile, uint32_t* hist, BinCounts what, uint32_t most, uint32_t* total, uint32_t* many = nullptr)
{
    const uint32_t tid = threadIdx.x, bits = a.bin.bits, bins = 1u << bits;
    const bool pack = bits > kWordBinBits;
    uint16_t* half = reinterpret_cast<uint16_t*>(hist);
    const uint32_t per = (bins + T - 1u) / T;         // consecutive bins per thread
    uint32_t mine = 0, over = 0;
    for (uint32_t i = 0; i < per; ++i) {
        const uint32_t p = tid * per + i;
        if (p < bins) {
            const uint32_t n = pack ? half[p] : hist[p];
            mine += n;
            over |= static_cast<uint32_t>(n > most);
        }
    }
    uint32_t overs;
    block_exclusive_scan<T>(mine, over, hist + counter_words(bits), total, &overs);
    uint32_t at = mine;
    if (overs && what != kRefs) return false;                         // (uniform)
    for (uint32_t i = 0; i < per; ++i) {
        const uint32_t p = tid * per + i;
        if (p < bins) {
            const uint32_t n = pack ? half[p] : hist[p], end = at + n;
            uint32_t* seg = a.segs + static_cast<size_t>(tile) * bins + p;
            const bool refs_only = what == kRefs && overs;
            if (refs_only || what == kEntries) reinterpret_cast<uint16_t*>(seg)[refs_only] = static_cast<uint16_t>(end);
            else *seg = what == kCounts ? end : end | (end << 16);
            if (refs_only && n > most) atomicOr(&many[p >> 5], 1u << (p & 31u));
            const uint32_t start = refs_only ? (n > most ? 0u : n) : at & 0xFFFFu;
            if (pack) half[p] = static_cast<uint16_t>(start);
            else hist[p] = start;
            at = end;
        }
    }
    lds_barrier();
    return !overs;
}

// A tile of one step with many references in one bin, as a hub's.  One entry stands for all references to a row that find each
// other: each leaves its number in a slot of its row's, and all whose slot was last written for the same row are that last one's;
// who lost the slot to another row tries a second one (with as many slots as references 2 in 5 lose the first and 1 in 6 of
// these the second one), and a row that lost both has an entry per reference.  So a hub is an entry or a few of each tile, however
// many references name it, and its bin, which one workgroup resolves, does not hold the batch up: 4 x 65 536 pairs at dim 16 among
// 50 / 1000 / 10 000 nodes 3170 / 574 / 282 us with an entry per reference, 264 / 163 / 155 with this; with one source row 1130 and
// 190.  It takes the workgroup 3 .. 8 us more, so only tiles with such a bin do it (always: 1 - 5 % of batches without hubs).  A table
// that settles every row takes up to 40 probes one after the other (two thirds full): 15 us more of a batch of 4096 pairs.
template <uint32_t T>
__device__ __forceinline__ void claim_rows(const PrepArgs& a, uint32_t tile, uint32_t first, uint32_t last, const uint32_t (&key)[kTileKeys<T>], uint32_t* hist)
{
    const uint32_t tid = threadIdx.x, bits = a.bin.bits, n = last - first, shift = __builtin_clz(a.bin.tile) + 1u;   // 32 - log2(tile)
    uint32_t* keys = hist + (1u << bits) + 32;        // of the references; later of the entries, sorted by bin
    uint32_t* count = keys + a.bin.tile;             // of the references that are this one's; later the number of their entry
    uint16_t* slot = reinterpret_cast<uint16_t*>(count + a.bin.tile);       // later the entries' references
    uint32_t at[kTileKeys<T>];                          // whose the reference is | its rank there << 16
    uint32_t pending = 0u;
    for (uint32_t i = tid; i < 1u << bits; i += T) hist[i] = 0u;
#pragma unroll
    for (int u = 0; u < kTileKeys<T>; ++u) {
        if (u * T >= n) break;                    // (uniform)
        at[u] = 0u;
        if (u * T + tid >= n) continue;              // (T may be more than the tile has)
        at[u] = u * T + tid;
        keys[at[u]] = key[u];
        count[at[u]] = 0u;
        if (key[u] != kNoKey) pending |= 1u << u;
    }
    lds_barrier();
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        auto slot_of = [&](uint32_t k) { return (round == 0 ? hash_bits(k) << bits : k * 0x85EBCA6Bu) >> shift; };    // (other bits than the bin's)
#pragma unroll
        for (int u = 0; u < kTileKeys<T>; ++u) {
            if (u * T >= n) break;
            if (pending >> u & 1u) slot[slot_of(key[u])] = static_cast<uint16_t>(u * T + tid);
        }
        lds_barrier();
        uint32_t whose[kTileKeys<T>], row[kTileKeys<T>];
#pragma unroll
        for (int u = 0; u < kTileKeys<T>; ++u) {
            if (u * T >= n) break;
            whose[u] = at[u];
            if (pending >> u & 1u) whose[u] = slot[slot_of(key[u])];
        }
#pragma unroll
        for (int u = 0; u < kTileKeys<T>; ++u) {
            if (u * T >= n) break;
            row[u] = keys[whose[u]];
        }
#pragma unroll
        for (int u = 0; u < kTileKeys<T>; ++u) {
            if (u * T >= n) break;
            if ((pending >> u & 1u) && row[u] == key[u]) {
                at[u] = whose[u];
                pending &= ~(1u << u);
            }
        }
        lds_barrier();
    }
#pragma unroll
    for (int u = 0; u < kTileKeys<T>; ++u) {
        if (u * T >= n) break;
        if (key[u] != kNoKey) at[u] |= atomicAdd(&count[at[u]], 1u) << 16;
    }
    lds_barrier();
    uint32_t refs[kTileKeys<T>];                        // of the entries that this thread's references are the first ones of
#pragma unroll
    for (int u = 0; u < kTileKeys<T>; ++u) {
        refs[u] = 0u;
        if (u * T >= n) continue;
        if (key[u] != kNoKey && at[u] < 0x10000u) {
            refs[u] = count[at[u]];
            atomicAdd(&hist[bin_of(key[u], bits)], 1u | (refs[u] << 16));
        }
    }
    lds_barrier();
    uint32_t total;
    start_bins<T>(a, tile, hist, kCounts, ~0u, &total);
    total &= 0xFFFFu;
#pragma unroll
    for (int u = 0; u < kTileKeys<T>; ++u) {
        if (u * T >= n) break;
        if (refs[u]) {
            const uint32_t p = atomicAdd(&hist[bin_of(key[u], bits)], 1u);
            keys[p] = key[u];
            slot[p] = static_cast<uint16_t>(refs[u]);
            count[at[u]] = p;
        }
    }
    lds_barrier();
#pragma unroll
    for (int u = 0; u < kTileKeys<T>; ++u) {
        const uint32_t t = first + u * T + tid;
        if (t < last) a.where[t] = key[u] == kNoKey ? 0u : count[at[u] & 0xFFFFu] | (at[u] & 0xFFFF0000u);
    }
    for (uint32_t i = tid; i < total; i += T) {
        a.keys[first + i] = keys[i];
        a.tags[first + i] = slot[i];
    }
}

// Key of a reference whose id is written.
template <RefMode MODE>
__device__ __forceinline__ uint32_t key_again(const PrepArgs& a, uint32_t t)
{
    const int32_t id = a.ids[t];
    const bool vertex_row = t % a.R < (MODE == kSegRefs ? a.seg_entries : 1u);
    return id < 0 ? kNoKey : static_cast<uint32_t>(id) | (vertex_row ? 0u : 0x80000000u);
}

// A tile of several steps with many references in some bins, which have a bit in `many` (start_bins, kRefs): the rows of these bins,
// few as they are, find each other in a table; a row that finds no place near its home there has an entry per reference.  Three
// passes over the tile's ids instead of two.  count_bin adds one to a bin's counter and returns what it was.
// (With an entry per reference the one workgroup that resolves a hub's bin goes through all of them: 2 x 131 072 pairs, dim 16,
// K = 5, among 4 M nodes, 5 / 30 % with one source row, 303 / 731 us, with this 200 / 204; 2 x 2^20 2030 / 3740 and 1817 / 1841;
// 131 072 among 50 / 1000 / 10 000 nodes 2880 / 782 / 372 and 247 / 181 / 179.)
template <RefMode MODE, uint32_t T, class F>
__device__ __forceinline__ void claim_long_rows(const PrepArgs& a, uint32_t tile, uint32_t first, uint32_t last, uint32_t* hist, F count_bin)
{
    constexpr int U = T == 256 ? 4 : kTileKeys<T>;
    constexpr uint32_t kAlone = 0x80000000u;
    const uint32_t tid = threadIdx.x, bits = a.bin.bits;
    uint32_t* many = hist + counter_words(bits) + 32;
    uint32_t* row = many + ((1u << bits) >> 5);
    uint32_t* count = row + kLongRows;          // of the row's references; later the number of its entry
    auto of_many = [&](uint32_t key) { const uint32_t p = bin_of(key, bits); return key != kNoKey && (many[p >> 5] >> (p & 31u) & 1u); };
    for (uint32_t i = tid; i < kLongRows; i += T) { row[i] = kNoKey; count[i] = 0u; }
    __syncthreads();                            // (ids that other threads have written)
    auto fetch = [&](uint32_t step, uint32_t (&key)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = step + u * T + tid < last ? key_again<MODE>(a, step + u * T + tid) : kNoKey;
    };
    uint32_t next[U];
    fetch(first, next);
    for (uint32_t step = first; step < last; step += U * T) {
        uint32_t key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = next[u];
        fetch(step + U * T, next);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!of_many(key[u])) continue;
            uint32_t at = (key[u] * 0x85EBCA6Bu) / (0xFFFFFFFFu / kLongRows + 1u), w = kAlone;
            for (int probe = 0; probe < 8; ++probe, at = (at + 1u) & (kLongRows - 1u)) {
                uint32_t k = __hip_atomic_load(row + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (k == kNoKey) k = atomicCAS(row + at, kNoKey, key[u]);
                if (k == kNoKey || k == key[u]) { w = at | (atomicAdd(count + at, 1u) << 16); break; }
            }
            if (w == kAlone) count_bin(bin_of(key[u], bits));
            a.where[step + u * T + tid] = w;
        }
    }
    lds_barrier();
    for (uint32_t i = tid; i < kLongRows; i += T)
        if (row[i] != kNoKey) count_bin(bin_of(row[i], bits));
    lds_barrier();
    uint32_t total;
    start_bins<T>(a, tile, hist, kEntries, ~0u, &total);
    for (uint32_t i = tid; i < kLongRows; i += T)
        if (row[i] != kNoKey) {
            const uint32_t p = count_bin(bin_of(row[i], bits));
            a.keys[first + p] = row[i];
            a.tags[first + p] = count[i];
            count[i] = p;
        }
    auto fetch_where = [&](uint32_t step, uint32_t (&w)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = step + u * T + tid < last ? a.where[step + u * T + tid] : 0u;
    };
    uint32_t next_w[U];
    fetch(first, next);
    fetch_where(first, next_w);
    lds_barrier();
    for (uint32_t step = first; step < last; step += U * T) {
        uint32_t key[U], w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { key[u] = next[u]; w[u] = next_w[u]; }
        fetch(step + U * T, next);
        fetch_where(step + U * T, next_w);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (step + u * T + tid >= last) continue;
            uint32_t p = 0u;
            if (key[u] != kNoKey) {
                const bool rows = of_many(key[u]);
                if (rows && w[u] != kAlone) p = count[w[u] & 0xFFFFu] | (w[u] & 0xFFFF0000u);
                else {
                    p = count_bin(bin_of(key[u], bits));
                    a.keys[first + p] = key[u];
                    if (rows) a.tags[first + p] = 1u;
                }
            }
            a.where[step + u * T + tid] = p;
        }
    }
}

// Most references of a tile in one bin for which each has an entry.
// (A bin whose rows are many has up to 13 references or so of the mean 4; where tiles are few, a bin's references stay few
// whatever one tile has of them; the third pass over a long tile lengthens the claim phase, a launch's longest chain, where as
// many entries in the resolve phase still hide behind it: 2 x 262 144 pairs, dim 128, K = 10, 5 % with one source row, 68 of them a
// tile, 1896 us with it, 1824 without; 18 at all lengths also 2 x 2^22 pairs among 4 M nodes, 0.5 % with one, 8250 instead of 7710)
__host__ __device__ constexpr uint32_t most_singles(const Binning& b)
{
    const uint32_t by_mean = 4u * (b.tile >> b.bits) + 2u, by_tile = b.tile / 512u * 3u, by_tiles = kTileStep / b.tiles;
    const uint32_t most = by_mean > by_tile ? by_mean : by_tile;
    return most > by_tiles ? most : by_tiles;
}

// One tile of references: draw, count by bin, then write the entries of each bin side by side.
// All T threads of the workgroup call this together; hist: claim_lds_bytes() of LDS.
template <RefMode MODE, uint32_t T>
__device__ __forceinline__ void claim_tile(const PrepArgs& a, uint32_t tile, uint32_t* hist)
{
    const unsigned tid = threadIdx.x;
    const uint32_t bits = a.bin.bits;
    const uint32_t words = counter_words(bits), pack = bits > kWordBinBits ? 1u : 0u;
    for (uint32_t i = tid; i < words; i += T) hist[i] = 0u;
    const uint32_t first = tile * a.bin.tile;
    const uint32_t last = min(first + a.bin.tile, a.refs);   // (refs is at most 2^28)
    uint32_t key[kTileKeys<T>];
    auto count = [&](uint32_t p) {       // what the bin's counter was
        const uint32_t shift = (p & pack) << 4, before = atomicAdd(&hist[p >> pack], 1u << shift) >> shift;
        return pack ? before & 0xFFFFu : before;
    };
    uint32_t step = first;
    for (;; step += kTileStep) {
        claim_refs<MODE, T>(a, step, last, key);
        if (step == first) lds_barrier();            // (the counters are zero)
#pragma unroll
        for (int u = 0; u < kTileKeys<T>; ++u)
            if (key[u] != kNoKey) count(bin_of(key[u], bits));
        if (step + kTileStep >= last) break;
    }
    lds_barrier();
    uint32_t total;
    const uint32_t most = most_singles(a.bin);
    if (a.bin.tile <= kTileStep) {                   // (uniform)
        if (!start_bins<T>(a, tile, hist, kSingles, most, &total)) {
            claim_rows<T>(a, tile, first, last, key, hist);
            return;
        }
        uint32_t* keys = hist + words + 32;          // sorted in LDS, so that they leave side by side
#pragma unroll
        for (int u = 0; u < kTileKeys<T>; ++u) {
            const uint32_t t = first + u * T + tid;
            if (first + u * T >= last) break;        // (uniform)
            uint32_t p = 0u;
            if (key[u] != kNoKey) {
                p = count(bin_of(key[u], bits));
                keys[p] = key[u];
            }
            if (t < last) a.where[t] = p;
        }
        lds_barrier();
        for (uint32_t i = tid; i < total; i += T) a.keys[first + i] = keys[i];
        return;
    }
    uint32_t* many = hist + words + 32;
    for (uint32_t i = tid; i < (1u << bits) >> 5; i += T) many[i] = 0u;        // (start_bins begins with a barrier)
    if (!start_bins<T>(a, tile, hist, kRefs, most, &total, many)) {
        claim_long_rows<MODE, T>(a, tile, first, last, hist, count);
        return;
    }
    // the last step's keys are still in registers; earlier ones are rebuilt from the ids
    for (;;) {
#pragma unroll
        for (int u = 0; u < kTileKeys<T>; ++u) {
            const uint32_t t = step + u * T + tid;
            uint32_t p = 0u;
            if (key[u] != kNoKey) {
                p = count(bin_of(key[u], bits));
                a.keys[first + p] = key[u];
            }
            if (t < last) a.where[t] = p;
        }
        if (step == first) break;
        step -= kTileStep;
#pragma unroll
        for (int u = 0; u < kTileKeys<T>; ++u) {
            const uint32_t t = step + u * T + tid;
            key[u] = key_again<MODE>(a, t);
        }
    }
}

// One bin of references: all entries of a row are in it.  An LDS hash table counts each row's references;
// rows with more than one get their places in the list and their work items; then every entry of
// such a row takes the next of the row's places, as many as it has references.  A bin whose distinct rows do not fit the table is
// gone through in ranges of the hash, halved until they fit: the hash is a bijection of the key, so a range
// of 2^k values holds at most 2^k rows and the halving ends.
constexpr uint32_t kItemRefs = 8;                        // references per work item
// A place in memory (below 2^28), and a flag: some entry of the tile's segment is more than one reference, and their numbers are in tags.
constexpr uint32_t kPlaceMask = 0x0FFFFFFFu, kCounted = 0x80000000u;
struct alignas(16) ResolveLds {
    unsigned long long taken; // by the bin's rows so far: places | work items << 32
    uint32_t hub_items;       // work items of its hubs so far
    uint32_t distinct;
    uint32_t long_segments;   // some tile has more than kShortSegment entries in the bin
    uint32_t unused[3];
    uint32_t part[32];
    uint32_t first[256];      // of the 256 tiles at hand: number of the tile's first entry among theirs in this bin
    uint32_t from[256];       // where entry 0 would be if the tile's entries began with it (kPlaceMask), and whether they have counts (kCounted)
    uint8_t tile_of[2048];    // of each entry of a share, if no segment is long
    // then the table, slot after slot: the row's key; its references, later its first, or next, place in the list (~0: not shared)
};
static_assert(sizeof(ResolveLds) % alignof(uint4) == 0, "the table is cleared two slots at a time");
inline size_t resolve_lds_bytes(const Binning& b) { return sizeof(ResolveLds) + (static_cast<size_t>(8) << b.slot_bits); }

// Work item of a row with up to kItemRefs places in the list: x = key, y = first place << 3 | places - 1.  A row with
// more (a hub) has several items with consecutive numbers in a list of their own: x, y as above, z = how many the row
// has, w = which of them this is.
__device__ __forceinline__ uint32_t item_places(uint32_t first, uint32_t n) { return (first << 3) | (n - 1u); }

// Accumulator of a hub: the number of its first place, divided by kItemRefs and rounded up, which is no other hub's
// because each has more than kItemRefs places.
__device__ __forceinline__ uint32_t hub_accumulator(uint32_t first) { return (first + kItemRefs - 1u) / kItemRefs; }

// A bin writes its items from where its references say, whatever other bins write: those of `refs` references are at most refs / 2
// items and refs 2/9 items of hubs (one of nine references has two).  The batch's train launch moves them together (gather_items).
// (One list for all bins, appended to with an add to the batch's totals: the add's round trip is a sixth of the chain of a batch of 28 672
// references, and 512 of them behind one another hold up a channel's rows: 2 - 3 us of the train launch of 65 536 pairs.)
__host__ __device__ inline uint64_t most_items(uint64_t refs) { return refs / 2u; }
__host__ __device__ inline uint64_t most_hub_items(uint64_t refs) { return refs * 2u / 9u; }

// The items of each lane's row, which has n references (up to 1: none) and places from `place` on, from numbers item and hub of the
// batch's bins on, which are moved behind them.  All lanes call this together.
__device__ __forceinline__ void write_items(const PrepArgs& a, uint32_t key, uint32_t n, uint32_t place, uint32_t& item, uint32_t& hub)
{
    constexpr uint32_t kAlone = 8 * kItemRefs;          // a lane writes up to eight items by itself
    const uint32_t m = (n + kItemRefs - 1u) / kItemRefs;
    auto write = [&](uint32_t at, uint32_t k, uint32_t refs, uint32_t first, uint32_t of, uint32_t q) {
        a.hub_items[at + q] = make_uint4(k, item_places(first + q * kItemRefs, min(kItemRefs, refs - q * kItemRefs)), of, q);
    };
    if (n > 1 && n <= kItemRefs) a.items[item++] = make_uint2(key, item_places(place, n));
    else if (n > kItemRefs && n <= kAlone)
        for (uint32_t q = 0; q < m; ++q) write(hub, key, n, place, m, q);
    // more by the whole wavefront: one lane takes 280 us for the 8192 of a row with 65 536 references
    for (unsigned long long hubs = __ballot(n > kAlone); hubs; hubs &= hubs - 1ull) {
        const int lane = __builtin_ctzll(hubs);
        const uint32_t k = __builtin_amdgcn_readlane(key, lane), refs = __builtin_amdgcn_readlane(n, lane), first = __builtin_amdgcn_readlane(place, lane);
        const uint32_t of = __builtin_amdgcn_readlane(m, lane), at = __builtin_amdgcn_readlane(hub, lane);
        for (uint32_t q = threadIdx.x & 63u; q < of; q += 64u) write(at, k, refs, first, of, q);
    }
    if (n > kItemRefs) hub += m;
}

// A bin's entries lie in up to one segment per tile.  A workgroup numbers those of 256 tiles through (a segment word per
// thread, a prefix sum) and thread i takes the entries i, i + T, ...: every lane has one, and a thread's accesses to entries, hash table
// and places are independent of one another and in flight together.  Up to 256 tiles and 2048 entries stay in registers,
// which is every bin of up to 1024 references but for hubs' (1280: 1.5 % more of a batch among a million nodes, whose hubs'
// bins are read in passes then).
template <uint32_t T> constexpr int kShare = 2048 / T;
template <uint32_t T>
struct BinShare {
    uint32_t key[kShare<T>], from[kShare<T>];     // an entry's row, and where it lies
    uint32_t refs[kShare<T>];    // its references
    uint32_t at[kShare<T>];      // slot of the row, in bytes
};

// A tile's segment of the bin, for thread i that of tile tile0 + i, i < 256: begin and end, entries | references << 16.
template <uint32_t T>
__device__ __forceinline__ uint2 fetch_segment(const PrepArgs& a, uint32_t bin, uint32_t tile0)
{
    const uint32_t t = tile0 + threadIdx.x;
    uint2 segment = make_uint2(0u, 0u);
    if (threadIdx.x < 256u && t < a.bin.tiles) {
        const uint32_t* ends = a.segs + (static_cast<size_t>(t) << a.bin.bits) + bin;
        segment.y = *ends;
        if (bin) segment.x = ends[-1];
    }
    return segment;
}

// Numbers the entries of these tiles and returns how many they are; *before: the tiles' references in lower bins.  SHARE: if they
// are a share, tile_of says whose each is (a search through 224 tiles is 8 accesses to LDS in turn).  All threads call this together.
// (A tile of one step has up to most_singles references in a bin, 18 with 64 bins and 108 tiles or more, 2048 / tiles with fewer tiles, beyond
// which equal rows share entries.  Batches of 257 .. 512 references, 8 bins and two tiles, have segments of 32 on average and mostly search.)
constexpr uint32_t kShortSegment = 32;
template <uint32_t T, bool SHARE>
__device__ __forceinline__ uint32_t number_entries(const PrepArgs& a, uint2 segment, uint32_t tile0, ResolveLds& s, uint32_t* before)
{
    const uint32_t begin = segment.x, end = segment.y, entries = (end & 0xFFFFu) - (begin & 0xFFFFu), refs = (end >> 16) - (begin >> 16);
    if (SHARE && threadIdx.x == 0) s.long_segments = 0u;
    uint32_t total;
    uint32_t first = entries, refs_before = begin >> 16;
    block_exclusive_scan<T>(first, refs_before, s.part, &total, before);
    if (threadIdx.x < 256u) {
        s.first[threadIdx.x] = first;
        s.from[threadIdx.x] = (((tile0 + threadIdx.x) * a.bin.tile + (begin & 0xFFFFu) - first) & kPlaceMask) | (refs != entries ? kCounted : 0u);
        if (SHARE && total <= sizeof s.tile_of) {
            if (entries > kShortSegment) s.long_segments = 1u;
            else for (uint32_t i = 0; i < entries; ++i) s.tile_of[first + i] = static_cast<uint8_t>(threadIdx.x);
        }
    }
    lds_barrier();
    return total;
}

// The entries first + T * u + tid < total of the 256 tiles at hand, u < U: their rows, where they lie, and their references.
// SHARE: tile_of is there for them unless some segment is long.
template <uint32_t T, bool SHARE, int U>
__device__ __forceinline__ void fetch_entries(const PrepArgs& a, uint32_t total, uint32_t first, const ResolveLds& s,
                                              uint32_t (&key)[U], uint32_t (&from)[U], uint32_t (&refs)[U])
{
    const uint32_t k = first + threadIdx.x;
    uint32_t tile[U];                       // the last tile whose first entry is not behind the thread's
    const bool search = !SHARE || s.long_segments;      // (uniform)
#pragma unroll
    for (int u = 0; u < U; ++u) tile[u] = 0u;
    if (!search) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (first + T * u >= total) break;          // (uniform)
            if (k + T * u < total) tile[u] = s.tile_of[k + T * u];
        }
    } else for (uint32_t step = a.bin.tiles > 128u ? 128u : 1u << (31 - __builtin_clz(a.bin.tiles)); step; step >>= 1) {
        uint32_t begin[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (first + T * u >= total) break;          // (uniform)
            begin[u] = s.first[tile[u] + step];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (first + T * u >= total) break;
            if (begin[u] <= k + T * u) tile[u] += step;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (first + T * u >= total) break;
        if (k + T * u < total) {
            const uint32_t place = s.from[tile[u]];
            from[u] = (place + k + T * u) & kPlaceMask;
            key[u] = a.keys[from[u]];
            refs[u] = 1u;
            if (place & kCounted) refs[u] = a.tags[from[u]];
        }
    }
}

__device__ __forceinline__ uint32_t* key_of(uint2* table, uint32_t at) { return reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(table) + at); }
__device__ __forceinline__ uint32_t* count_of(uint2* table, uint32_t at) { return key_of(table, at) + 1; }

// The slots of the share's rows, which are added to the table where they are not there yet (it has as many slots as there are entries).
template <uint32_t T>
__device__ __forceinline__ void locate_share(const PrepArgs& a, uint32_t total, uint2* table, BinShare<T>& e)
{
    const uint32_t mask = (sizeof(uint2) << a.bin.slot_bits) - 1u;
    uint32_t pending = 0u;
#pragma unroll
    for (int u = 0; u < kShare<T>; ++u) {
        if (T * u >= total) break;              // (uniform)
        e.at[u] = ((hash_bits(e.key[u]) << a.bin.bits) >> (32u - a.bin.slot_bits)) * static_cast<uint32_t>(sizeof(uint2));
        if (T * u + threadIdx.x < total) pending |= 1u << u;
    }
    while (__ballot(pending != 0u)) {
        uint32_t there[kShare<T>];
#pragma unroll
        for (int u = 0; u < kShare<T>; ++u) {
            if (T * u >= total) break;
            if (pending >> u & 1u) there[u] = __hip_atomic_load(key_of(table, e.at[u]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
#pragma unroll
        for (int u = 0; u < kShare<T>; ++u) {
            if (T * u >= total) break;
            if ((pending >> u & 1u) && there[u] == kNoKey) {
                there[u] = atomicCAS(key_of(table, e.at[u]), kNoKey, e.key[u]);
                if (there[u] == kNoKey) there[u] = e.key[u];
            }
        }
#pragma unroll
        for (int u = 0; u < kShare<T>; ++u) {
            if (T * u >= total) break;
            if (pending >> u & 1u) {
                if (there[u] == e.key[u]) pending &= ~(1u << u);
                else e.at[u] = (e.at[u] + static_cast<uint32_t>(sizeof(uint2))) & mask;
            }
        }
    }
}

// What a thread's rows take, places of the list and work items, is added to what the bin's rows have taken, and becomes what others
// took before.  All lanes call this together.
__device__ __forceinline__ void take(ResolveLds& s, uint32_t& places, uint32_t& items, uint32_t& hubs)
{
    const uint32_t last_place = wave_inclusive_scan(places), last_item = wave_inclusive_scan(items), last_hub = wave_inclusive_scan(hubs);
    unsigned long long before = 0ull;
    uint32_t hubs_before = 0u;
    if ((threadIdx.x & 63u) == 63u) {
        before = atomicAdd(&s.taken, last_place | (static_cast<unsigned long long>(last_item) << 32));
        if (last_hub) hubs_before = atomicAdd(&s.hub_items, last_hub);
    }
    places = __builtin_amdgcn_readlane(static_cast<uint32_t>(before), 63) + last_place - places;
    items = __builtin_amdgcn_readlane(static_cast<uint32_t>(before >> 32), 63) + last_item - items;
    hubs = __builtin_amdgcn_readlane(hubs_before, 63) + last_hub - hubs;
}

// What earlier rows of a bin have taken.
struct Taken { uint32_t places, items, hub_items; };

// The places and work items of the shared rows in the table, which holds every row's references on entry and, on
// return, a shared row's first place, kNoKey for the others.  The bin's first place is first_place, and earlier rows of it have taken
// `taken`, which is moved.  All threads call this together.
template <uint32_t T>
__device__ __forceinline__ void place_rows(const PrepArgs& a, uint32_t first_place, Taken& taken, ResolveLds& s, uint2* table)
{
    const uint32_t tid = threadIdx.x, slots = 1u << a.bin.slot_bits;
    uint32_t items = 0, places = 0, hubs = 0;
    for (uint32_t p = tid; p < slots; p += T) {
        const uint32_t n = table[p].y;
        if (n > 1) { places += n; items += static_cast<uint32_t>(n <= kItemRefs); }
        if (n > kItemRefs) hubs += (n + kItemRefs - 1) / kItemRefs;
    }
    take(s, places, items, hubs);
    uint32_t row = first_place + taken.places + places;
    uint32_t item = static_cast<uint32_t>(most_items(first_place)) + taken.items + items;
    uint32_t hub = static_cast<uint32_t>(most_hub_items(first_place)) + taken.hub_items + hubs;
    for (uint32_t p = tid; p < slots; p += T) {
        const uint2 slot = table[p];
        table[p].y = slot.y > 1 ? row : kNoKey;
        if (a.items) write_items(a, slot.x, slot.y, row, item, hub);      // (uniform)
        if (slot.y > 1) row += slot.y;
    }
    lds_barrier();
    taken.places += static_cast<uint32_t>(s.taken);
    taken.items += static_cast<uint32_t>(s.taken >> 32);
    taken.hub_items += s.hub_items;
}

// f(key, references, place in memory) for every entry of the 256 tiles at hand, four of a thread in flight (eight: 73 registers, a
// wavefront less of the kernels this rides in), until stop().  Numbered through like a share's, because segments are short where tiles
// are many: as many lanes per segment as it has entries on average, one segment after the other, took 5660 us for 3 x 2^21
// pairs, dim 16, among 32 M nodes, this 5500 (2^22: 12 470 and 12 110).
template <uint32_t T, class F, class S>
__device__ __forceinline__ void for_entries(const PrepArgs& a, uint32_t total, const ResolveLds& s, F f, S stop)
{
    constexpr int U = T == 256 ? 4 : kShare<T>;
    for (uint32_t first = 0; first < total && !stop(); first += T * U) {
        uint32_t key[U], from[U], refs[U];
        fetch_entries<T, false>(a, total, first, s, key, from, refs);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (first + T * u + threadIdx.x < total) f(key[u], refs[u], from[u]);
    }
}

// (No barrier behind it.)
template <uint32_t T>
__device__ __forceinline__ void clear_table(const PrepArgs& a, ResolveLds& s, uint2* table)
{
    for (uint32_t i = threadIdx.x; i < 1u << (a.bin.slot_bits - 1u); i += T) reinterpret_cast<uint4*>(table)[i] = make_uint4(kNoKey, 0u, kNoKey, 0u);
    if (threadIdx.x == 0) { s.taken = 0ull; s.distinct = 0u; s.hub_items = 0u; }
}

// A bin whose entries stay in registers: `total` of them, all numbered, no more than the table takes, which is empty.  Its rows take
// places from first_place on: a row's first entry, the one that found its counter at zero, does that for it, so that the table is not
// gone through.
// A chain of dependent accesses from end to end, which is what a small batch waits for.  224 references, 56 tiles: 3.3 us, of which
// the segments' words and the entries take 0.7 us each.  (5.8 with a search for every entry's tile, two passes over the table, rows placed by
// a sum over the workgroup and the totals' round trip.)
template <uint32_t T>
__device__ __forceinline__ void resolve_share(const PrepArgs& a, uint32_t bin, uint32_t total, uint32_t first_place, ResolveLds& s, uint2* table)
{
    const uint32_t tid = threadIdx.x;
    BinShare<T> e;
    fetch_entries<T, true>(a, total, 0u, s, e.key, e.from, e.refs);
    locate_share<T>(a, total, table, e);
    uint32_t firsts = 0u;            // a bit per entry: its row's first
#pragma unroll
    for (int u = 0; u < kShare<T>; ++u) {
        if (T * u >= total) break;              // (uniform)
        if (T * u + tid < total) {
            e.refs[u] = atomicAdd(count_of(table, e.at[u]), e.refs[u]);     // the row's references in entries before this one
            firsts |= static_cast<uint32_t>(e.refs[u] == 0u) << u;
        }
    }
    lds_barrier();
    uint32_t places = 0u, items = 0u, hubs = 0u;
#pragma unroll
    for (int u = 0; u < kShare<T>; ++u) {
        if (T * u >= total) break;
        if (firsts >> u & 1u) {
            const uint32_t n = *count_of(table, e.at[u]);
            e.refs[u] = n;                                  // (of a first entry until its row is placed: the row's references)
            if (n > 1) { places += n; items += static_cast<uint32_t>(n <= kItemRefs); }
            if (n > kItemRefs) hubs += (n + kItemRefs - 1u) / kItemRefs;
        }
    }
    take(s, places, items, hubs);
    uint32_t place = first_place + places;
    uint32_t item = static_cast<uint32_t>(most_items(first_place)) + items;
    uint32_t hub = static_cast<uint32_t>(most_hub_items(first_place)) + hubs;
#pragma unroll
    for (int u = 0; u < kShare<T>; ++u) {
        if (T * u >= total) break;
        const bool first = firsts >> u & 1u;
        const uint32_t n = first ? e.refs[u] : 0u;
        if (first) {
            *count_of(table, e.at[u]) = n > 1 ? place : kNoKey;
            e.refs[u] = 0u;
        }
        if (a.items) write_items(a, e.key[u], n, place, item, hub);     // (uniform)
        if (n > 1) place += n;
    }
    lds_barrier();
    if (a.items && tid == 0) a.bins[bin] = make_uint4(first_place, static_cast<uint32_t>(s.taken >> 32), s.hub_items, 0u);
#pragma unroll
    for (int u = 0; u < kShare<T>; ++u) {
        if (T * u >= total) break;
        if (T * u + tid < total) {
            const uint32_t row = *count_of(table, e.at[u]);
            a.tags[e.from[u]] = row == kNoKey ? 0u : 1u + row + e.refs[u];
        }
    }
}

// Any bin: entries are read again for every pass, one after the other, and a bin whose rows do not fit the table is gone
// through in ranges of the hash.  (total: the entries of the first 256 tiles, numbered; before: references there in lower bins.)
template <uint32_t T>
__device__ __forceinline__ void resolve_passes(const PrepArgs& a, uint32_t bin, uint32_t total, uint32_t before, ResolveLds& s, uint2* table)
{
    uint32_t lo = 0, halvings = 0;      // range of the hash below the bin's bits: [lo, lo + 2^(32 - halvings))
    Taken taken{0u, 0u, 0u};
    auto given_up = [&] { return __hip_atomic_load(&s.distinct, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > a.bin.full; };
    auto home = [&](uint32_t key, uint32_t* at) {
        const uint32_t x = (hash_bits(key) << a.bin.bits) - lo;
        *at = ((x << halvings) >> (32u - a.bin.slot_bits)) * static_cast<uint32_t>(sizeof(uint2));
        return !halvings || !(x >> (32u - halvings));      // (else another range's)
    };
    auto next = [&](uint32_t at) { return (at + static_cast<uint32_t>(sizeof(uint2))) & ((static_cast<uint32_t>(sizeof(uint2)) << a.bin.slot_bits) - 1u); };
    for (;;) {
        clear_table<T>(a, s, table);
        lds_barrier();
        uint32_t first_place = a.bin.tiles > 256u ? 0u : before;
        for (uint32_t t0 = 0; t0 < a.bin.tiles; t0 += 256u) {
            if (a.bin.tiles > 256u) {
                lds_barrier();
                if (given_up()) break;          // (uniform: nobody adds a row before the next barrier)
                total = number_entries<T, false>(a, fetch_segment<T>(a, bin, t0), t0, s, &before);
                first_place += before;
            }
            for_entries<T>(a, total, s, [&](uint32_t key, uint32_t refs, uint32_t) {
                uint32_t at;
                if (!home(key, &at)) return;
                for (;; at = next(at)) {
                    uint32_t k = __hip_atomic_load(key_of(table, at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (k == kNoKey) {
                        if (given_up()) return;
                        k = atomicCAS(key_of(table, at), kNoKey, key);
                        if (k == kNoKey) { atomicAdd(&s.distinct, 1u); k = key; }
                    }
                    if (k == key) break;
                    if (given_up()) return;         // (no slot may be left: every row counts as soon as it has one)
                }
                atomicAdd(count_of(table, at), refs);
            }, given_up);
        }
        lds_barrier();
        if (s.distinct > a.bin.full) {       // (uniform: nobody writes it between the barriers)
            lds_barrier();
            halvings += 1;
            continue;
        }
        place_rows<T>(a, first_place, taken, s, table);
        for (uint32_t t0 = 0; t0 < a.bin.tiles; t0 += 256u) {
            if (a.bin.tiles > 256u) {
                lds_barrier();
                total = number_entries<T, false>(a, fetch_segment<T>(a, bin, t0), t0, s, &before);
            }
            for_entries<T>(a, total, s, [&](uint32_t key, uint32_t refs, uint32_t from) {
                uint32_t at;
                if (!home(key, &at)) return;
                while (*key_of(table, at) != key) at = next(at);
                uint32_t tag = 0u;
                if (*count_of(table, at) != kNoKey) tag = 1u + atomicAdd(count_of(table, at), refs);
                a.tags[from] = tag;
            }, [] { return false; });
        }
        if (halvings) lo += 1u << (32u - halvings);
        if (lo == 0) {           // (the last range, or the only one)
            if (a.items && threadIdx.x == 0) a.bins[bin] = make_uint4(first_place, taken.items, taken.hub_items, 0u);
            return;
        }
        lds_barrier();
    }
}

template <uint32_t T>
__device__ __forceinline__ void resolve_bin(const PrepArgs& a, uint32_t bin, unsigned char* lds)
{
    ResolveLds& s = *reinterpret_cast<ResolveLds*>(lds);
    uint2* table = reinterpret_cast<uint2*>(lds + sizeof(ResolveLds));
    const uint2 segment = fetch_segment<T>(a, bin, 0);
    clear_table<T>(a, s, table);            // (while the segments' words travel)
    uint32_t before;
    const uint32_t total = number_entries<T, true>(a, segment, 0, s, &before);
    if (a.bin.tiles <= 256u && total <= min(T * kShare<T>, 1u << a.bin.slot_bits)) resolve_share<T>(a, bin, total, before, s, table);      // (uniform)
    else resolve_passes<T>(a, bin, total, before, s, table);
}

// ---------------------------------------------------------------------------------------------
// sample prefetch (ne_train_block_pinned): a few workgroups copy the pairs of a later batch from
// pinned host memory, which they read directly, into a device staging ring.  They ride inside the
// training launches; the first three batches of a call use the stand-alone kernel.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void fetch_pairs(const int2* __restrict__ src, int2* __restrict__ dst, int64_t n, int64_t i0,
                                            int64_t stride)
{
    // pairs two at a time while both buffers allow 16-byte accesses
    const bool wide = ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0;
    if (wide) {
        const int64_t n2 = n / 2;
        const int4* s4 = reinterpret_cast<const int4*>(src);
        int4* d4 = reinterpret_cast<int4*>(dst);
        // four loads in flight per thread: the link's latency is long and the copy should stay small
        int64_t i = i0;
        for (; i + 3 * stride < n2; i += 4 * stride) {
            const int4 v0 = s4[i], v1 = s4[i + stride], v2 = s4[i + 2 * stride], v3 = s4[i + 3 * stride];
            d4[i] = v0; d4[i + stride] = v1; d4[i + 2 * stride] = v2; d4[i + 3 * stride] = v3;
        }
        for (; i < n2; i += stride) d4[i] = s4[i];
        if (i0 == 0 && (n & 1)) dst[n - 1] = src[n - 1];
    } else {
        for (int64_t i = i0; i < n; i += stride) dst[i] = src[i];
    }
}

__global__ __launch_bounds__(256) void fetch_pairs_kernel(const int2* __restrict__ src, int2* __restrict__ dst, int64_t n)
{
    fetch_pairs(src, dst, n, static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x,
                static_cast<int64_t>(gridDim.x) * blockDim.x);
}

// The work items of a batch's bins, moved together for the apply kernel.  A few workgroups of the batch's own train launch, with
// kGatherBins bins each or, of many, more: a workgroup adds up the bins before its own and copies what they have, a wavefront per bin.
struct GatherArgs {
    const uint4* bins;          // per bin: its first place, its items, its hubs' items
    const uint2* from;
    const uint4* hubs_from;
    uint2* items;
    uint4* hub_items;
    unsigned long long* totals; // items | items of hubs << 32
    uint32_t n_bins, share;     // bins in all and per workgroup, powers of two, share at most 256
};
// A bin with many items of hubs is copied by all of them (by a wavefront: 4 x 65 536 pairs with one source row, dim 16, 264 us instead of 182).
constexpr uint32_t kGatherBins = 4, kGatherBlocks = 128, kGatherAlone = 256;
struct GatherLds { uint32_t part[32]; uint32_t item[256], hub[256]; uint32_t big[256]; uint32_t n_big; };
template <uint32_t T>
__device__ __forceinline__ void gather_items(const GatherArgs& a, uint32_t block, unsigned char* lds)
{
    GatherLds& s = *reinterpret_cast<GatherLds*>(lds);
    const uint32_t tid = threadIdx.x, first = block * a.share;
    uint32_t items = 0u, hubs = 0u, own_items = 0u, own_hubs = 0u;
    for (uint32_t b = tid; b < first; b += T) { const uint4 bin = a.bins[b]; items += bin.y; hubs += bin.z; }
    if (tid < a.share) { const uint4 bin = a.bins[first + tid]; own_items = bin.y; own_hubs = bin.z; }
    uint32_t items_before, hubs_before, items_here, hubs_here;
    block_exclusive_scan<T>(items, hubs, s.part, &items_before, &hubs_before);
    block_exclusive_scan<T>(own_items, own_hubs, s.part, &items_here, &hubs_here);
    if (tid < a.share) { s.item[tid] = items_before + own_items; s.hub[tid] = hubs_before + own_hubs; }
    if (tid == 0 && first + a.share == a.n_bins) *a.totals = (items_before + items_here) | (static_cast<unsigned long long>(hubs_before + hubs_here) << 32);
    if (tid == 0) s.n_big = 0u;
    lds_barrier();
    for (uint32_t b = tid >> 6; b < a.share; b += T / 64u) {
        const uint4 bin = a.bins[first + b];
        const uint2* from = a.from + most_items(bin.x);
        for (uint32_t i = tid & 63u; i < bin.y; i += 64u) a.items[s.item[b] + i] = from[i];
        const uint4* hubs_from = a.hubs_from + most_hub_items(bin.x);
        if (bin.z <= kGatherAlone)
            for (uint32_t i = tid & 63u; i < bin.z; i += 64u) a.hub_items[s.hub[b] + i] = hubs_from[i];
        else if ((tid & 63u) == 0u) s.big[atomicAdd(&s.n_big, 1u)] = b;
    }
    lds_barrier();
    for (uint32_t k = 0; k < s.n_big; ++k) {
        const uint32_t b = s.big[k];
        const uint4 bin = a.bins[first + b];
        const uint4* hubs_from = a.hubs_from + most_hub_items(bin.x);
        for (uint32_t i = tid; i < bin.z; i += 4u * T) {
            const uint32_t last = bin.z - 1u, i1 = min(i + T, last), i2 = min(i + 2u * T, last), i3 = min(i + 3u * T, last);     // (the last one several times)
            const uint4 v0 = hubs_from[i], v1 = hubs_from[i1], v2 = hubs_from[i2], v3 = hubs_from[i3];
            uint4* to = a.hub_items + s.hub[b];
            to[i] = v0; to[i1] = v1; to[i2] = v2; to[i3] = v3;
        }
    }
}

// LDS of the kernels: counters of a claiming workgroup, hash table of a resolving one, staged rows of a training one.
extern __shared__ __align__(16) unsigned char dynamic_lds[];

// The id-only work for later batches that rides in a launch: the launch's first workgroups, because theirs are
// chains of dependent accesses, which hide behind the other workgroups only if they start first.
struct Helpers {
    unsigned resolves, claims, fetches, gathers;   // workgroups of each kind: bins of `resolve`, tiles of `claim`
    GatherArgs gather;    // the launch's own batch
    PrepArgs resolve;     // next batch
    PrepArgs claim;       // the one after that; its fetch fields: pairs of the batch after that one
    unsigned count() const { return resolves + claims + fetches + gathers; }
    size_t lds_bytes() const
    {
        const size_t r = resolves ? resolve_lds_bytes(resolve.bin) : 0, c = claims ? claim_lds_bytes(claim.bin) : 0;
        const size_t g = gathers ? sizeof(GatherLds) : 0;
        return std::max(std::max(r, c), g);
    }
};

// False for a workgroup that has other work to do; *block is then its index among those.
template <RefMode MODE, uint32_t T = 256>
__device__ __forceinline__ bool helper_block(const Helpers& h, unsigned* block)
{
    unsigned i = blockIdx.x;
    if (i < h.resolves) {
        // neighbouring bins share cache lines (a tile's segment words and entries lie bin after bin), and
        // workgroups go to the eight dies in turn: each die takes a run of consecutive bins
        resolve_bin<T>(h.resolve, h.resolves >= 8 ? (i & 7u) * (h.resolves >> 3) + (i >> 3) : i, dynamic_lds);
        return true;
    }
    i -= h.resolves;
    if (i < h.claims) { claim_tile<MODE, T>(h.claim, i, reinterpret_cast<uint32_t*>(dynamic_lds)); return true; }
    i -= h.claims;
    if (i < h.fetches) {
        fetch_pairs(h.claim.fetch_src, h.claim.fetch_dst, h.claim.fetch_n, static_cast<int64_t>(i) * T + threadIdx.x,
                    static_cast<int64_t>(h.fetches) * T);
        return true;
    }
    i -= h.fetches;
    if (i < h.gathers) { gather_items<T>(h.gather, i, dynamic_lds); return true; }
    i -= h.gathers;
    // consecutive pairs on one die, which then shares the cache lines of their ids and tags
    const unsigned blocks = gridDim.x - h.resolves - h.claims - h.fetches - h.gathers, share = blocks >> 3, rest = blocks & 7u, die = i & 7u;
    *block = die * share + min(die, rest) + (i >> 3);
    return false;
}

// The same work on its own, for the first batches of a call.  A batch with one tile and one bin is claimed and resolved
// by the same workgroup (claim_first: h.resolve).
template <RefMode MODE, uint32_t T>
__global__ __launch_bounds__(T, T == 512 ? 6 : 1) void prepare_kernel(Helpers h, bool claim_first)
{
    if (claim_first && blockIdx.x == 0) {
        claim_tile<MODE, T>(h.resolve, 0, reinterpret_cast<uint32_t*>(dynamic_lds));
        __syncthreads();
    }
    unsigned block;
    helper_block<MODE, T>(h, &block);
}

// ---------------------------------------------------------------------------------------------
// train kernel.  G lanes per pair, NCH float4 chunks per lane (chunk index = lg + i*G, valid while
// < d4), JB context rows in flight at a time.
// DIRECT: the per-sample mode (ne_train_block_async): a shared row's deltas go straight to the table row
// with atomics instead of to the list, so pairs that read the row later see them, and nothing is
// left for the apply phase.
// ---------------------------------------------------------------------------------------------
struct TrainArgs {
    float4* X;
    float4* C;
    int64_t B;            // pairs (pair mode) / walk positions or segments (walk mode)
    int32_t window;       // walk mode: pairs per position
    int32_t K;
    int32_t d4;
    float lr;
    const int32_t* ids;
    const uint32_t* where;  // per reference: which entry of its tile names its row | how many of the tile's references come first << 16
    const uint32_t* tags;   // per entry: 0 = one reference, and the only one of its row; else 1 + the first one's place in the list
    uint32_t tile;          // references per tile, a power of two
    uint2* list;          // (row of buf, coefficient)
    float4* buf;          // [..][d4]
};

// Tag of a reference: 0 = the sole reference of its row, else 1 + its place in the list.  The entry's tag is on its way when this is
// made, and only get() waits for it, once the rows are there.
struct TagRef {
    uint32_t first, rank;     // the entry's tag, and how many of its references come before this one
    __device__ __forceinline__ uint32_t get() const { return first ? first + rank : 0u; }
};
__device__ __forceinline__ TagRef tag_of(const TrainArgs& a, int64_t t, uint32_t where)
{
    return {a.tags[(static_cast<uint32_t>(t) & ~(a.tile - 1u)) + (where & 0xFFFFu)], where >> 16};
}

// Element e = lg + m*G of a row, for m < 4*NCH: the layout in which one atomic instruction of a lane
// group covers consecutive dwords.  The float4-chunk layout is turned into it through LDS.
template <int G, int NCH>
__device__ __forceinline__ void to_consecutive(const float4 (&v)[NCH], float (&out)[4 * NCH], float* lds_row, int lg)
{
#pragma unroll
    for (int i = 0; i < NCH; ++i) reinterpret_cast<float4*>(lds_row)[lg + i * G] = v[i];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int m = 0; m < 4 * NCH; ++m) out[m] = lds_row[lg + m * G];
    __builtin_amdgcn_wave_barrier();
}

// row += delta in place, or the delta to row `spare` of buf and its place in the list.
template <int G, int NCH>
__device__ __forceinline__ void write_row(const TrainArgs& a, float4* row, uint32_t tag, uint32_t spare, const float4 (&old)[NCH],
                                          const float4 (&dv)[NCH], int lg, int d4)
{
    float4* out = tag ? a.buf + static_cast<int64_t>(spare) * d4 : row;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int ci = lg + i * G;
        if (ci < d4) out[ci] = tag ? dv[i] : make_float4(old[i].x + dv[i].x, old[i].y + dv[i].y, old[i].z + dv[i].z, old[i].w + dv[i].w);
    }
    if (tag && lg == 0) a.list[tag - 1u] = make_uint2(spare, __float_as_uint(1.0f));
}

// True for every lane of a lane group if it is for one of them.
template <int G>
__device__ __forceinline__ bool group_any(bool v)
{
    const unsigned long long all = __ballot(v);
    return G == 64 ? all != 0ull : ((all >> (threadIdx.x & 63u & ~(G - 1u))) & ((1ull << (G & 63)) - 1ull)) != 0ull;
}

// The source row of a lane group to row `copy` of buf, where its references to shared rows point.
template <int G, int NCH>
__device__ __forceinline__ void write_copy(const TrainArgs& a, uint32_t copy, const float4 (&xr)[NCH], int lg, int d4)
{
    float4* out = a.buf + static_cast<int64_t>(copy) * d4;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int ci = lg + i * G;
        if (ci < d4) out[ci] = xr[i];
    }
}

// K+1 context rows of one pair (rows 0..K; with POS_FIRST row 0 is the positive, every other row a
// negative), JB at a time: gather, score against x, form g_j, add g_j c_j to dx, and update the row:
// rewritten in place if only this reference names it, else lr g_j and `copy`, the row of buf that gets x, go
// to the reference's place in the list (DIRECT: the delta goes to the row with atomics; xt is x in
// consecutive-dword layout).  Lane j + LANE0 of the group holds reference j's id and tag, owns it (`own`) and returns whether its
// row is shared; other lanes own nothing.
// tag_of_mine() is called behind the first rows: loads are waited for in the order in which they were issued.  (By segments a
// sample's tags, fetched there, cost small batches 1 - 5 % less than before its rows: 4 x 20 walks of 80 entries, dim 64, K = 10,
// window 10 227 us and 218, 4 x 170, dim 128, K = 5, window 5 409 and 398, K = 10 702 and 710.  Pairs fetch theirs before: 65 536, dim 128 1 - 2 %.)
template <int G, int NCH, int JB, int LANE0, bool POS_FIRST = true, bool DIRECT = false, class F>
__device__ __forceinline__ bool context_rows_of_pair(const TrainArgs& a, int K, int d4, const float4 (&xr)[NCH],
                                                     const float (&xt)[4 * NCH], float4 (&dx)[NCH], int32_t id_mine,
                                                     F tag_of_mine, bool own, uint32_t copy, int lg)
{
    float g_mine = 0.0f;     // lr g_j of lane j + LANE0
    uint32_t tag_mine = 0u;
    TagRef tag_ref{0u, 0u};
    for (int j0 = 0; j0 <= K; j0 += JB) {
        float4 cr[JB][NCH];
        float part[JB];
        float4* crow[JB];
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            const int j = j0 + jj;
            const int32_t id = __shfl(id_mine, (j <= K ? j : K) + LANE0, G);
            crow[jj] = a.C + static_cast<int64_t>(id) * d4;
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                const int ci = lg + i * G;
                cr[jj][i] = (j <= K && ci < d4) ? crow[jj][ci] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        if (j0 == 0) tag_ref = tag_of_mine();
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            float p = 0.0f;
#pragma unroll
            for (int i = 0; i < NCH; ++i) p += dot4(xr[i], cr[jj][i]);
            part[jj] = p;
        }
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) part[jj] = group_sum<G>(part[jj]);
        // every lane has every score: the lane that owns a reference forms its g_j, one exponential for all JB rows
        // (one per row in every lane: up to 10 % slower where a walk entry has many rows, 1 % on pairs)
        float score = 0.0f;
#pragma unroll
        for (int jj = 0; jj < JB; ++jj)
            if (lg == j0 + jj + LANE0) score = part[jj];
        const float sg = sigmoidf(score);
        const float g_own = a.lr * ((POS_FIRST && lg == LANE0) ? 1.0f - sg : -sg);
        if (lg >= j0 + LANE0 && lg < j0 + LANE0 + JB) g_mine = g_own;
        tag_mine = own ? tag_ref.get() : 0u;
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            const int j = j0 + jj;
            if (j <= K) {
                const float g = __shfl(g_own, j + LANE0, G);
                const uint32_t tag = __shfl(tag_mine, j + LANE0, G);
#pragma unroll
                for (int i = 0; i < NCH; ++i) dx[i] = axpy4(g, cr[jj][i], dx[i]);
                if (DIRECT && tag) {
                    float* row = reinterpret_cast<float*>(crow[jj]);
#pragma unroll
                    for (int m = 0; m < 4 * NCH; ++m) {
                        const int e = lg + m * G;
                        if (e < d4 * 4) unsafeAtomicAdd(row + e, g * xt[m]);
                    }
                } else if (!tag) {
#pragma unroll
                    for (int i = 0; i < NCH; ++i) {
                        const int ci = lg + i * G;
                        if (ci < d4) crow[jj][ci] = axpy4(g, xr[i], cr[jj][i]);
                    }
                }
            }
        }
    }
    if (!DIRECT && tag_mine) a.list[tag_mine - 1u] = make_uint2(copy, __float_as_uint(g_mine));
    return tag_mine != 0u;
}

constexpr int kTrainThreads = 256;   // threads per block of the train kernels

template <int G, int NCH, int JB, bool DIRECT>
__global__ __launch_bounds__(kTrainThreads) void train_kernel(TrainArgs a, Helpers helpers)
{
    constexpr int GROUPS = kTrainThreads / G;
    unsigned block;
    if (helper_block<kPairRefs>(helpers, &block)) return;
    const int lg = threadIdx.x & (G - 1);
    const int grp = threadIdx.x / G;
    const int64_t b = static_cast<int64_t>(block) * GROUPS + grp;
    if (b >= a.B) return;   // whole groups leave together; groups never communicate below
    const int K = a.K;
    const int R = K + 2;
    const int d4 = a.d4;

    // lane j < R owns reference j: id and tag
    const int64_t ref = b * R + (lg < R ? lg : 0);
    const int32_t id_mine = a.ids[ref];
    const TagRef tag = tag_of(a, ref, a.where[ref]);
    float4* xrow = a.X + static_cast<int64_t>(__shfl(id_mine, 0, G)) * d4;
    float4 xr[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int ci = lg + i * G;
        xr[i] = (ci < d4) ? xrow[ci] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float xt[4 * NCH];   // x in consecutive-dword layout, for the atomics
    float* lds_row = reinterpret_cast<float*>(dynamic_lds) + grp * (4 * G * NCH);
    if (DIRECT) to_consecutive<G, NCH>(xr, xt, lds_row, lg);

    float4 dx[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) dx[i] = make_float4(0.f, 0.f, 0.f, 0.f);

    const uint32_t copy = static_cast<uint32_t>(b), spare = static_cast<uint32_t>(a.B + b);   // rows of buf
    const bool context = context_rows_of_pair<G, NCH, JB, 1, true, DIRECT>(a, K, d4, xr, xt, dx, id_mine, [&] { return tag; }, lg > 0 && lg < R, copy, lg);
    const uint32_t tag0 = __shfl(tag.get(), 0, G);
    if (!DIRECT && group_any<G>(context)) write_copy<G, NCH>(a, copy, xr, lg, d4);

    if (DIRECT && tag0) {
        to_consecutive<G, NCH>(dx, xt, lds_row, lg);
#pragma unroll
        for (int m = 0; m < 4 * NCH; ++m) {
            const int e = lg + m * G;
            if (e < d4 * 4) unsafeAtomicAdd(reinterpret_cast<float*>(xrow) + e, xt[m]);
        }
    } else {
        write_row<G, NCH>(a, xrow, tag0, spare, xr, dx, lg, d4);
    }
}

// ---------------------------------------------------------------------------------------------
// train kernel of the walk mode: one lane group per walk position.  The source row is gathered once
// and stays in registers for the position's `window` pairs; its delta is summed over all of them
// and written once.  The pairs' context rows are handled as in the pair mode, as one list, which P lane groups of one
// wavefront share between them: a batch of few positions is bound by a group's chain of ids, rows and sums, and the chip idle
// beside it (880 positions of 30 context rows at dim 64: 10.5 us with P = 1 and 16 rows at a time, 8.5 with P = 4 and 4 rows).
// ---------------------------------------------------------------------------------------------
template <int G, int NCH, int JB, int P>
__global__ __launch_bounds__(kTrainThreads) void train_walk_kernel(TrainArgs a, Helpers helpers)
{
    static_assert(P == 1 || G * P == 64, "the groups of a position are a wavefront");
    constexpr int GROUPS = kTrainThreads / (G * P);
    unsigned block;
    if (helper_block<kWalkRefs>(helpers, &block)) return;
    const int lg = threadIdx.x & (G - 1);
    const int grp = threadIdx.x / (G * P), part = (threadIdx.x / G) & (P - 1);
    const int64_t p = static_cast<int64_t>(block) * GROUPS + grp;
    if (p >= a.B) return;   // whole groups leave together; groups never communicate below
    const int K = a.K;
    const int d4 = a.d4;
    const int64_t R = 1 + static_cast<int64_t>(a.window) * (K + 1);
    const int64_t ref0 = p * R;

    const int32_t src = a.ids[ref0];
    if (src < 0) return;    // no pair starts at this position (uniform over the group)
    const uint32_t where0 = a.where[ref0];
    float4* xrow = a.X + static_cast<int64_t>(src) * d4;
    float4 xr[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int ci = lg + i * G;
        xr[i] = (ci < d4) ? xrow[ci] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    const TagRef tag0 = tag_of(a, ref0, where0);       // (behind the row: loads are waited for in the order in which they were issued)
    float4 dx[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) dx[i] = make_float4(0.f, 0.f, 0.f, 0.f);

    const uint32_t copy = static_cast<uint32_t>(p), spare = static_cast<uint32_t>(a.B + p);   // rows of buf
    bool copied = false;
    // the context references of all pairs, JB at a time; lane l < JB owns reference j0 + l, and the next JB ids travel
    // while these rows do.  (A pair that the walk does not have: its references have id -1.)  Where it costs no wavefront (4 more
    // registers), ids travel two rounds ahead and their tags, one access further away, one: 4 x 4800 positions, dim 512, K = 5,
    // 486 -> 475 us, 4 x 11 050, dim 144, 422 -> 417; at dim 64 it costs one (4 x 4800 positions, K = 10, 513 -> 556).
    constexpr int AHEAD = G == 64 ? 2 : 1;
    const int all = a.window * (K + 1), share = (all + P - 1) / P, begin = part * share, n = min(all, begin + share);
    auto fetch = [&](int j, int32_t& id, uint32_t& where) {
        id = -1;
        where = 0u;
        if (lg < JB && j + lg < n) {
            id = a.ids[ref0 + 1 + j + lg];
            where = a.where[ref0 + 1 + j + lg];
        }
    };
    auto fetch_tag = [&](int j, int32_t id, uint32_t where) { return tag_of(a, id < 0 ? ref0 : ref0 + 1 + j + lg, id < 0 ? 0u : where); };
    int32_t id_next, id_mine = -1;
    uint32_t where_next;
    TagRef tag_ref{0u, 0u};
    fetch(begin, id_next, where_next);
    if (AHEAD == 2) {
        id_mine = id_next;
        tag_ref = fetch_tag(begin, id_mine, where_next);
        fetch(begin + JB, id_next, where_next);
    }
    int phase = begin % (K + 1);                // j0 mod K + 1: reference 0 of a pair is its positive
    for (int j0 = begin; j0 < n; j0 += JB) {
        if (AHEAD == 1) id_mine = id_next;
        float4 cr[JB][NCH];
        int32_t id[JB];
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            id[jj] = __shfl(id_mine, jj, G);
            const float4* crow = a.C + static_cast<int64_t>(id[jj]) * d4;
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                const int ci = lg + i * G;
                cr[jj][i] = (id[jj] >= 0 && ci < d4) ? crow[ci] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        // (behind the rows: loads are waited for in the order in which they were issued)
        const TagRef tag_next = fetch_tag(j0 + (AHEAD - 1) * JB, id_next, where_next);
        const int32_t id_then = id_next;
        fetch(j0 + AHEAD * JB, id_next, where_next);
        if (AHEAD == 1) tag_ref = tag_next;
        float part[JB];
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            float s = 0.0f;
#pragma unroll
            for (int i = 0; i < NCH; ++i) s += dot4(xr[i], cr[jj][i]);
            part[jj] = s;
        }
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) part[jj] = group_sum<G>(part[jj]);
        // the lane that owns a reference forms its g_j
        float score = 0.0f;
        bool positive = false;
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            if (lg == jj) { score = part[jj]; positive = phase == 0; }
            phase = phase == K ? 0 : phase + 1;
        }
        const float sg = sigmoidf(score);
        const float g_mine = a.lr * (positive ? 1.0f - sg : -sg);
        const uint32_t tag_mine = id_mine < 0 ? 0u : tag_ref.get();
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            if (id[jj] >= 0) {
                const float g = __shfl(g_mine, jj, G);
#pragma unroll
                for (int i = 0; i < NCH; ++i) dx[i] = axpy4(g, cr[jj][i], dx[i]);
                if (__shfl(tag_mine, jj, G) == 0u) {
                    float4* crow = a.C + static_cast<int64_t>(id[jj]) * d4;
#pragma unroll
                    for (int i = 0; i < NCH; ++i) {
                        const int ci = lg + i * G;
                        if (ci < d4) crow[ci] = axpy4(g, xr[i], cr[jj][i]);
                    }
                }
            }
        }
        if (tag_mine) a.list[tag_mine - 1u] = make_uint2(copy, __float_as_uint(g_mine));
        copied |= group_any<G>(tag_mine != 0u);
        if (AHEAD == 2) {
            id_mine = id_then;
            tag_ref = tag_next;
        }
    }
    if (P > 1) {
        copied = __ballot(copied) != 0ull;
#pragma unroll
        for (int off = G; off < G * P; off <<= 1)
#pragma unroll
            for (int i = 0; i < NCH; ++i)
                dx[i] = make_float4(dx[i].x + __shfl_xor(dx[i].x, off, 64), dx[i].y + __shfl_xor(dx[i].y, off, 64),
                                    dx[i].z + __shfl_xor(dx[i].z, off, 64), dx[i].w + __shfl_xor(dx[i].w, off, 64));
        if (part) return;
    }
    if (copied) write_copy<G, NCH>(a, copy, xr, lg, d4);
    write_row<G, NCH>(a, xrow, tag0.get(), spare, xr, dx, lg, d4);
}

// ---------------------------------------------------------------------------------------------
// train kernel of the walk mode by segments: one workgroup per segment of E = threads / G
// consecutive entries of a walk, one lane group per entry.  All vertex rows of the segment's entries
// and all context rows that serve as their samples' contexts (E + window - 1 of them) are gathered
// once into LDS.  Each group then plays two parts:
//   source   its entry against the up to `window` following context rows (from LDS) and against the
//            K negatives of each sample (from memory): sums dx in registers, updates the negatives;
//   context  its entry's context row (and, for the first window-1 groups, one of the rows past the
//            segment's end) against the vertex rows (from LDS) of the up to `window` preceding
//            entries of this segment: sums dc in registers.
// The positive score of a sample is therefore computed twice (both ends need its coefficient); the
// rows are what costs.  Every row is then written once: in place if no other reference names it,
// else its delta goes to the list (the context rows next to a segment boundary get contributions from both
// segments and are always of that kind).
// ---------------------------------------------------------------------------------------------
template <int G, int NCH, int JB>
__global__ __launch_bounds__(kTrainThreads) void train_seg_kernel(TrainArgs a, Helpers helpers)
{
    constexpr int E = kTrainThreads / G;
    constexpr int ROW = 4 * G * NCH;              // floats per staged row (>= d)
    float* xs = reinterpret_cast<float*>(dynamic_lds);   // [E][ROW]        vertex rows of the entries
    float* cs = xs + E * ROW;                            // [E + window - 1][ROW]  context rows
    const int CT = E + a.window - 1;
    int32_t* cid = reinterpret_cast<int32_t*>(cs + CT * ROW);   // [CT] ids of the context rows (-1: absent)
    int32_t* xid = cid + CT;                                    // [E]  ids of the vertex rows (-1: absent)
    unsigned block;
    if (helper_block<kSegRefs>(helpers, &block)) return;
    const int lg = threadIdx.x & (G - 1);
    const int grp = threadIdx.x / G;
    const int K = a.K;
    const int W = a.window;
    const int d4 = a.d4;
    const int64_t R = E + CT + static_cast<int64_t>(E) * W * K;
    if (static_cast<int64_t>(block) >= a.B) return;             // a.B = segments of the batch (uniform over the workgroup)
    const int64_t ref0 = static_cast<int64_t>(block) * R;
    // rows of buf: [E] deltas of vertex rows, [CT] deltas of context rows, [E] copies of vertex rows for the negatives
    const uint32_t buf0 = block * static_cast<uint32_t>(E + CT + (K > 0 ? E : 0));

    // my entry's vertex row, and the context rows grp and grp + E of the segment's list
    const int32_t src = a.ids[ref0 + grp];
    const TagRef tag_x = tag_of(a, ref0 + grp, a.where[ref0 + grp]);
    float4 xr[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) xr[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    float4* xrow = a.X;
    if (src >= 0) {
        xrow = a.X + static_cast<int64_t>(src) * d4;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int ci = lg + i * G;
            if (ci < d4) xr[i] = xrow[ci];
        }
    }
#pragma unroll
    for (int i = 0; i < NCH; ++i) reinterpret_cast<float4*>(xs + grp * ROW)[lg + i * G] = xr[i];
    if (lg == 0) xid[grp] = src;
    for (int row = grp; row < CT; row += E) {
        const int32_t id = a.ids[ref0 + E + row];
        if (lg == 0) cid[row] = id;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int ci = lg + i * G;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (id >= 0 && ci < d4) v = (a.C + static_cast<int64_t>(id) * d4)[ci];
            reinterpret_cast<float4*>(cs + row * ROW)[ci] = v;
        }
    }
    __syncthreads();

    // ---- source part
    if (src >= 0) {
        const float xt[4 * NCH] = {};
        float4 dx[NCH];
#pragma unroll
        for (int i = 0; i < NCH; ++i) dx[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        const uint32_t copy = buf0 + static_cast<uint32_t>(E + CT + grp);
        bool copied = false;
        // lane k < K owns negative k of a sample; the next sample's travel while this one's rows do
        const int64_t ref_neg = ref0 + E + CT + static_cast<int64_t>(grp) * W * K + lg;
        int32_t id_next = -1;
        uint32_t where_next = 0;
        if (lg < K) {
            id_next = a.ids[ref_neg];
            where_next = a.where[ref_neg];
        }
        for (int j = 1; j <= W; ++j) {
            const int32_t id_mine = id_next;
            const uint32_t where = where_next;
            if (lg < K && j < W) {
                id_next = a.ids[ref_neg + static_cast<int64_t>(j) * K];
                where_next = a.where[ref_neg + static_cast<int64_t>(j) * K];
            }
            const int row = grp + j - 1;                      // context row of entry (mine + j)
            if (cid[row] < 0) continue;                       // no such sample (uniform over the group)
            float4 cr[NCH];
            float p = 0.0f;
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                cr[i] = reinterpret_cast<const float4*>(cs + row * ROW)[lg + i * G];
                p += dot4(xr[i], cr[i]);
            }
            p = group_sum<G>(p);
            const float g0 = a.lr * (1.0f - sigmoidf(p));
#pragma unroll
            for (int i = 0; i < NCH; ++i) dx[i] = axpy4(g0, cr[i], dx[i]);
            if (K > 0) {
                auto tag_of_mine = [&] { return tag_of(a, id_mine < 0 ? ref0 : ref_neg + static_cast<int64_t>(j - 1) * K, id_mine < 0 ? 0u : where); };
                const bool shared = context_rows_of_pair<G, NCH, JB, 0, false>(a, K - 1, d4, xr, xt, dx, id_mine, tag_of_mine, id_mine >= 0, copy, lg);
                copied |= group_any<G>(shared);
            }
        }
        if (copied) write_copy<G, NCH>(a, copy, xr, lg, d4);
        write_row<G, NCH>(a, xrow, tag_x.get(), buf0 + grp, xr, dx, lg, d4);
    }

    // ---- context part: context row `row` is entry p0 + 1 + row; its sources in this segment are the
    // entries with local index max(0, row + 1 - W) .. min(row, E - 1)
    for (int row = grp; row < CT; row += E) {
        const int32_t id = cid[row];
        if (id < 0) continue;
        const TagRef tag_c = tag_of(a, ref0 + E + row, a.where[ref0 + E + row]);
        float4 cr[NCH], dc[NCH];
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            cr[i] = reinterpret_cast<const float4*>(cs + row * ROW)[lg + i * G];
            dc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        const int lo = row + 1 - W > 0 ? row + 1 - W : 0, hi = row < E - 1 ? row : E - 1;
        for (int sl = lo; sl <= hi; ++sl) {
            if (xid[sl] < 0) continue;
            float4 xv[NCH];
            float p = 0.0f;
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                xv[i] = reinterpret_cast<const float4*>(xs + sl * ROW)[lg + i * G];
                p += dot4(xv[i], cr[i]);
            }
            p = group_sum<G>(p);
            const float g0 = a.lr * (1.0f - sigmoidf(p));
#pragma unroll
            for (int i = 0; i < NCH; ++i) dc[i] = axpy4(g0, xv[i], dc[i]);
        }
        write_row<G, NCH>(a, a.C + static_cast<int64_t>(id) * d4, tag_c.get(), buf0 + static_cast<uint32_t>(E + row), cr, dc, lg, d4);
    }
}

// ---------------------------------------------------------------------------------------------
// apply kernel: one lane group per work item of the batch: the sum of up to 8 entries of the list, which lie
// side by side, is added to the table row; an entry is a coefficient times a row of buf.
// Hubs, rows with more references, are summed before they are added: the row is rounded once per batch however often the
// batch names it, and eight deltas that are together below the row's last place are not lost.  Their items go to
// workgroups of their own, which add up neighbouring items of a row in LDS; what several workgroups hold of a row meets
// in an accumulator that starts from zero, and who arrives last adds it to the table row and leaves it zero again.
// Bound by the rows it moves (two thirds of the rows have two references) and, in small batches, by its chain
// of four dependent accesses: item, entries, rows, store, of which the first two go ahead of an item's turn (65 536 pairs, dim 128,
// among 32 M / 1 M nodes 28.0 / 38.8 us with all of them in turn, 26.2 / 38.0; 20 000 nodes, 22 walks, dim 64 5.9 and 5.4).  The rows of buf are few (one or two per pair, however
// many references share them) and mostly still in the last-level cache; per-reference deltas in memory order
// instead cost here and in the train kernel 28 + 98 us at 32 M nodes x dim 128 (now 28 + 90), 47 + 94 at 1 M x
// dim 128 (now 39 + 77) and 151 + 285 at 4 M x dim 512, K = 10 (now 99 + 216).  8 entries at a time against 4: -1 .. -2 % of a batch at dim <= 256,
// +2 % at dim 512 (registers).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

struct ApplyArgs {
    float4* X;
    float4* C;
    int32_t d4;
    const uint2* items;
    const uint4* hub_items;
    const unsigned long long* totals;     // items | items of hubs << 32
    uint32_t most, most_hubs;        // items there can be, and items of hubs
    unsigned hub_blocks;  // workgroups, the first of the launch, that take the hubs' items
    const uint2* list;
    const float4* buf;
    float* acc;           // accumulators, all zero
    uint32_t* arrived;    // items whose sums have been added to each of them, all zero
};

// A work item's entries (item_places: y): lane r of the group fetches entry r, of the last one again past the end.
__device__ __forceinline__ uint2 fetch_entry(const ApplyArgs& a, uint32_t y, int lg) { return a.list[(y >> 3) + min(static_cast<uint32_t>(lg) & 7u, y & 7u)]; }

// The entries of a work item, summed.
template <int GL, int CH>
__device__ __forceinline__ void sum_item(const ApplyArgs& a, uint32_t y, uint2 mine, int lg, float4 (&sum)[CH])
{
    constexpr uint32_t MB = CH == 1 ? kItemRefs : kItemRefs / 2;   // entries whose rows travel together
    const uint32_t refs = (y & 7u) + 1u;
#pragma unroll
    for (int i = 0; i < CH; ++i) sum[i] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (uint32_t r0 = 0; r0 < kItemRefs; r0 += MB) {
        if (r0 >= refs) break;
        float4 v[MB][CH];
#pragma unroll
        for (uint32_t r = 0; r < MB; ++r) {
            const float4* src = a.buf + static_cast<int64_t>(__shfl(mine.x, r0 + r, GL)) * a.d4;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int ci = lg + GL * i;
                v[r][i] = r0 + r < refs && ci < a.d4 ? src[ci] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < MB; ++r) {
            const float c = __uint_as_float(__shfl(mine.y, r0 + r, GL)), g = r0 + r < refs ? c : 0.0f;
#pragma unroll
            for (int i = 0; i < CH; ++i) sum[i] = axpy4(g, v[r][i], sum[i]);
        }
    }
}

__device__ __forceinline__ float4* row_of_key(const ApplyArgs& a, uint32_t key)
{
    return ((key & 0x80000000u) ? a.C : a.X) + static_cast<int64_t>(key & 0x7FFFFFFFu) * a.d4;
}

// Items of hubs, one lane group each, workgroup by workgroup.  All 256 threads call this together.
template <int GL, int CH>
__device__ __forceinline__ void apply_hubs(const ApplyArgs& a, float4 (&lds)[256 / GL][GL * CH])
{
    constexpr uint32_t GROUPS = 256 / GL;
    const int lg = threadIdx.x & (GL - 1), d4 = a.d4;
    const uint32_t grp = threadIdx.x / GL;
    auto fetch_item = [&](uint32_t first) { return a.hub_items[min(first + grp, a.most_hubs - 1u)]; };     // (what lies past the last one is not used)
    uint4 item = fetch_item(blockIdx.x * GROUPS);          // (in flight together with the count)
    const uint32_t n = static_cast<uint32_t>(*a.totals >> 32);
    for (uint32_t first = blockIdx.x * GROUPS; first < n; first += a.hub_blocks * GROUPS, item = fetch_item(first)) {     // (uniform)
        const bool live = first + grp < n;
        float4 sum[CH];
        if (live) {
            sum_item<GL, CH>(a, item.y, fetch_entry(a, item.y, lg), lg, sum);
#pragma unroll
            for (int i = 0; i < CH; ++i) lds[grp][lg + GL * i] = sum[i];
        }
        __syncthreads();
        // the first of a row's items here adds up those that follow (its own sum is still in registers)
        if (live && (grp == 0 || item.w == 0)) {
            const uint32_t here = min(item.z - item.w, GROUPS - grp);
            for (uint32_t q = 1; q < here; ++q)
#pragma unroll
                for (int i = 0; i < CH; ++i) sum[i] = add4(sum[i], lds[grp + q][lg + GL * i]);
            bool last = here == item.z;
            const uint32_t at = hub_accumulator((item.y >> 3) - item.w * kItemRefs);
            float* acc = a.acc + static_cast<int64_t>(at) * (d4 * 4);
            if (!last) {
                float t[4 * CH];        // consecutive dwords per atomic instruction
                to_consecutive<GL, CH>(sum, t, reinterpret_cast<float*>(lds[grp]), lg);
#pragma unroll
                for (int m = 0; m < 4 * CH; ++m) {
                    const int c = lg + m * GL;
                    if (c < d4 * 4) unsafeAtomicAdd(acc + c, t[m]);
                }
                // These adds are carried out before the arrival is counted: waiting for their acknowledgements is
                // enough, and nothing has to be written back, because accumulators and counters are only ever
                // touched by device-scope atomics in this launch (a release fence, which writes the whole L2 back,
                // took five times as long as the rest of the launch).
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_s_waitcnt(0);
                uint32_t before = 0u;
                if (lg == 0) before = __hip_atomic_fetch_add(a.arrived + at, here, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = __shfl(before, 0, GL) + here == item.z;
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                if (last) {
#pragma unroll
                    for (int i = 0; i < CH; ++i) {
                        const int ci = lg + GL * i;
                        auto take = [&](int k) { return __hip_atomic_exchange(acc + 4 * ci + k, 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
                        if (ci < d4) sum[i] = make_float4(take(0), take(1), take(2), take(3));
                    }
                    if (lg == 0) a.arrived[at] = 0u;
                }
            }
            if (last) {
                float4* row = row_of_key(a, item.x);
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const int ci = lg + GL * i;
                    if (ci < d4) row[ci] = add4(row[ci], sum[i]);
                }
            }
        }
        __syncthreads();        // the sums are overwritten
    }
}

template <int GL, int CH>
__global__ __launch_bounds__(256) void apply_kernel(ApplyArgs a)
{
    constexpr uint32_t GROUPS = 256 / GL;
    __shared__ float4 lds[GROUPS][GL * CH];
    if (blockIdx.x < a.hub_blocks) {
        apply_hubs<GL, CH>(a, lds);
        return;
    }
    const int lg = threadIdx.x & (GL - 1);
    const uint32_t grp = threadIdx.x / GL;
    const uint32_t step = (gridDim.x - a.hub_blocks) * GROUPS;
    uint32_t e = (blockIdx.x - a.hub_blocks) * GROUPS + grp;
    // an item's entries are requested an item ahead and its words two ahead, so that a group waits for its rows only
    auto fetch_item = [&](uint32_t at) { return a.items[min(at, a.most - 1u)]; };     // (what lies past the last one is not used)
    uint2 item = fetch_item(e), next = fetch_item(e + step);
    const uint32_t n = static_cast<uint32_t>(*a.totals);
    uint2 entry = make_uint2(0u, 0u);
    if (e < n) entry = fetch_entry(a, item.y, lg);
    for (; e < n; e += step) {
        float4* row = row_of_key(a, item.x);
        float4 old[CH], sum[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int ci = lg + GL * i;
            old[i] = ci < a.d4 ? row[ci] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        const uint2 then = fetch_item(e + 2 * step);
        uint2 next_entry = make_uint2(0u, 0u);
        if (e + step < n) next_entry = fetch_entry(a, next.y, lg);
        sum_item<GL, CH>(a, item.y, entry, lg, sum);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int ci = lg + GL * i;
            if (ci < a.d4) row[ci] = add4(old[i], sum[i]);
        }
        item = next;
        next = then;
        entry = next_entry;
    }
}

// ---------------------------------------------------------------------------------------------
// loss kernel (ne_eval_loss): sampling + scoring fused, tables read-only.
// ---------------------------------------------------------------------------------------------
struct LossArgs {
    const float4* X;
    const float4* C;
    const int2* pairs;
    int64_t B;
    int32_t K;
    int32_t d4;
    uint64_t sample_base;
    uint32_t k0, k1;
    const uint2* alias;
    uint64_t alias_n;
    int32_t alias_base;
    int32_t* neg_out;
    double* loss;
};

// Lane groups go through the pairs with the grid's stride: a workgroup ends with one atomic add to the sum, and
// adds to one address retire one after the other (one per 8 pairs took 116 us for 65 536 pairs, whatever the
// rows cost).  The ids of a group's next pair travel while its rows do.
template <int G, int NCH, int JB>
__global__ __launch_bounds__(256) void loss_kernel(LossArgs a)
{
    constexpr int GROUPS = 256 / G;
    const int lg = threadIdx.x & (G - 1);
    const int64_t stride = static_cast<int64_t>(gridDim.x) * GROUPS;
    const int K = a.K;
    const int d4 = a.d4;
    // lane lg owns context row j = lg of a pair: j = 0 the positive, j = 1..K negative j-1
    struct Ids { int32_t src, mine; };
    auto ids_of = [&](int64_t b) {
        const int2 pr = a.pairs[b];
        Ids id{pr.x, pr.y};
        if (lg >= 1 && lg <= K) {
            id.mine = draw_negative(a.sample_base + static_cast<uint64_t>(b), static_cast<uint32_t>(lg - 1), a.k0, a.k1,
                                    a.alias, a.alias_n, a.alias_base);
            if (a.neg_out) a.neg_out[b * K + (lg - 1)] = id.mine;
        }
        return id;
    };
    double sum = 0.0;    // of lane lg's context row over the group's pairs
    int64_t b = static_cast<int64_t>(blockIdx.x) * GROUPS + (threadIdx.x / G);
    Ids next{0, 0};
    if (b < a.B) next = ids_of(b);
    for (; b < a.B; b += stride) {
        const Ids id = next;
        float4 xr[NCH];
        const float4* xrow = a.X + static_cast<int64_t>(id.src) * d4;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int ci = lg + i * G;
            xr[i] = (ci < d4) ? xrow[ci] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        float term_mine = 0.0f;   // lane j keeps the loss term of row j
        for (int j0 = 0; j0 <= K; j0 += JB) {
            float4 cr[JB][NCH];
#pragma unroll
            for (int jj = 0; jj < JB; ++jj) {
                const int j = j0 + jj;
                const int32_t row = __shfl(id.mine, j <= K ? j : K, G);
                const float4* crow = a.C + static_cast<int64_t>(row) * d4;
#pragma unroll
                for (int i = 0; i < NCH; ++i) {
                    const int ci = lg + i * G;
                    cr[jj][i] = (j <= K && ci < d4) ? crow[ci] : make_float4(0.f, 0.f, 0.f, 0.f);
                }
            }
            if (j0 == 0 && b + stride < a.B) next = ids_of(b + stride);
            float part[JB];
#pragma unroll
            for (int jj = 0; jj < JB; ++jj) {
                float p = 0.0f;
#pragma unroll
                for (int i = 0; i < NCH; ++i) p += dot4(xr[i], cr[jj][i]);
                part[jj] = p;
            }
#pragma unroll
            for (int jj = 0; jj < JB; ++jj) part[jj] = group_sum<G>(part[jj]);
#pragma unroll
            for (int jj = 0; jj < JB; ++jj) {
                const int j = j0 + jj;
                if (j <= K && lg == j) term_mine = j == 0 ? -part[jj] : part[jj];
            }
        }
        if (lg <= K) sum += static_cast<double>(softplusf(term_mine));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    __shared__ double sh[4];
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(a.loss, sh[0] + sh[1] + sh[2] + sh[3]);
}

__global__ __launch_bounds__(256) void validate_pairs_kernel(const int32_t* __restrict__ ids, int64_t count,
                                                             int64_t num_nodes, unsigned long long* bad)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    unsigned long long local = 0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < count; i += stride) {
        const int32_t v = ids[i];
        local += (v < 0 || v >= num_nodes) ? 1ull : 0ull;
    }
    if (local) atomicAdd(bad, local);
}

// ---------------------------------------------------------------------------------------------
// score kernel (ne_score_pairs): the model's similarity score of arbitrary node pairs, for
// evaluation (link prediction, Sec. V-B).  16 lanes per pair, float4 chunks strided over the row.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void score_pairs_kernel(const float4* __restrict__ A, const float4* __restrict__ Bt,
                                                          const int2* __restrict__ pairs, int64_t n, int32_t d4,
                                                          float* __restrict__ scores)
{
    const int lg = threadIdx.x & 15;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 16;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 16 + (threadIdx.x >> 4); i < n; i += stride) {
        const int2 pr = pairs[i];
        const float4* a = A + static_cast<int64_t>(pr.x) * d4;
        const float4* b = Bt + static_cast<int64_t>(pr.y) * d4;
        float p = 0.0f;
        for (int c = lg; c < d4; c += 16) p += dot4(a[c], b[c]);
        p = group_sum<16>(p);
        if (lg == 0) scores[i] = p;
    }
}

// ---------------------------------------------------------------------------------------------
// launch-shape selection
// ---------------------------------------------------------------------------------------------
struct Shape { int G, NCH; };

// Smallest lane group that covers dim/4 float4 chunks and has a lane for each of the K+2 references.
bool pick_shape(int32_t d4, int32_t K, Shape* out)
{
    // one float4 per lane as long as a wavefront holds the row: measured 4-5 % faster at dim 128 than 16 lanes x 2
    static const Shape order[] = {{8, 1}, {16, 1}, {32, 1}, {64, 1}, {64, 2}, {64, 4}};
    for (const Shape& s : order) {
        if (s.G * s.NCH >= d4 && s.G >= K + 2) { *out = s; return true; }
    }
    return false;
}

#define NE_FOR_EACH_SHAPE(M) M(8, 1) M(16, 1) M(32, 1) M(64, 1) M(64, 2) M(64, 4)

// Grid and LDS of a train launch with `blocks` training workgroups that need `own` bytes of LDS.
struct TrainGrid { unsigned grid; size_t lds; };
inline TrainGrid train_grid(const Helpers& h, int64_t blocks, size_t own)
{
    const size_t lds = h.lds_bytes();
    return {h.count() + static_cast<unsigned>(blocks), own > lds ? own : lds};
}

hipError_t launch_train(const Shape& s, const TrainArgs& a, const Helpers& h, bool direct, hipStream_t st)
{
    const int groups = kTrainThreads / s.G;
    const TrainGrid g = train_grid(h, (a.B + groups - 1) / groups, direct ? static_cast<size_t>(kTrainThreads) * s.NCH * sizeof(float4) : 0);
    // context rows gathered together per lane group: 6 where they come out nearly even and a lane has one chunk of a row
    // (K = 5: 1.7 % ahead of 2 on 32 M nodes, dim 128; K 3 .. 10 at dim 64 .. 256: 2 % behind .. 5 % ahead of 3), else 3 (K = 7:
    // 6 would be 2 % behind; dim 512 .. 1024: up to 4 % behind); the per-sample mode's atomics leave 2 ahead by 1 - 2 %
    const bool six = s.NCH == 1 && ((a.K + 1) % 6 == 0 || (a.K + 1) % 6 >= 4);
#define NE_CASE(G_, N_)                                                                          \
    if (s.G == G_ && s.NCH == N_) {                                                              \
        if (direct) hipLaunchKernelGGL((train_kernel<G_, N_, 2, true>), dim3(g.grid), dim3(kTrainThreads), g.lds, st, a, h); \
        else if (six) hipLaunchKernelGGL((train_kernel<G_, N_, N_ == 1 ? 6 : 3, false>), dim3(g.grid), dim3(kTrainThreads), g.lds, st, a, h); \
        else hipLaunchKernelGGL((train_kernel<G_, N_, 3, false>), dim3(g.grid), dim3(kTrainThreads), g.lds, st, a, h); \
        return hipGetLastError();                                                                \
    }
    NE_FOR_EACH_SHAPE(NE_CASE)
#undef NE_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_train_walk(const Shape& s, const TrainArgs& a, const Helpers& h, hipStream_t st)
{
    const int groups = kTrainThreads / s.G;
    // A batch of at most one workgroup per compute unit is bound by a position's chain of round trips: where a lane group is
    // less than a wavefront, a position takes a whole one (880 positions, dim 64, K = 5, window 5: 275 us become 243 for 16 batches; 408,
    // dim 48, K = 10, window 6: 88 and 58 for 3; up to 1024 workgroups: -5 .. +6 %).  Context rows gathered together per lane group: 6;
    // in the former case 16 per position, at least 4 per group (8 per group of 16 lanes: 246).
    const bool wide = (a.B + groups - 1) / groups <= 256;
#define NE_CASE(G_, N_)                                                                          \
    if (s.G == G_ && s.NCH == N_) {                                                              \
        constexpr int kParts = 64 / G_, kWide = N_ > 1 ? 6 : kParts > 2 ? 4 : 16 / kParts;                \
        const TrainGrid g = train_grid(h, wide ? (a.B * kParts + groups - 1) / groups : (a.B + groups - 1) / groups, 0);  \
        if (wide) hipLaunchKernelGGL((train_walk_kernel<G_, N_, kWide, kParts>), dim3(g.grid), dim3(kTrainThreads), g.lds, st, a, h); \
        else hipLaunchKernelGGL((train_walk_kernel<G_, N_, 6, 1>), dim3(g.grid), dim3(kTrainThreads), g.lds, st, a, h); \
        return hipGetLastError();                                                                \
    }
    NE_FOR_EACH_SHAPE(NE_CASE)
#undef NE_CASE
    return hipErrorInvalidValue;
}

// LDS of the segment kernel: vertex rows and context rows of a segment, and their ids
size_t seg_lds_bytes(const Shape& s, int window)
{
    const size_t E = kTrainThreads / s.G, row = 4 * static_cast<size_t>(s.G) * s.NCH, CT = E + window - 1;
    return (E + CT) * row * 4 + (CT + E) * 4;
}

hipError_t launch_train_seg(const Shape& s, const TrainArgs& a, const Helpers& h, hipStream_t st)
{
    const TrainGrid g = train_grid(h, a.B, seg_lds_bytes(s, a.window));   // one workgroup per segment
#define NE_CASE(G_, N_)                                                                          \
    if (s.G == G_ && s.NCH == N_) {                                                              \
        hipLaunchKernelGGL((train_seg_kernel<G_, N_, 6>), dim3(g.grid), dim3(kTrainThreads), g.lds, st, a, h); \
        return hipGetLastError();                                                                \
    }
    NE_FOR_EACH_SHAPE(NE_CASE)
#undef NE_CASE
    return hipErrorInvalidValue;
}

// Workgroups of 512 threads where a tile has two references for each and up to 1024 workgroups do.  Three have a place on a compute unit (their
// 104 scalar registers leave seven wavefronts per SIMD), 768 on the chip, which is every launch of bins and tiles up to 512 of the one and 256
// of the other.  65 536 pairs, K = 5, among 1 M / 32 M nodes: the first claim 11.7 / 20.1 us, bins and the second claim together 12.3 / 18.4.
// (1024 threads leave the bins and the second claim no place side by side: with both claims in the first launch 16.5 / 32.2 and
// 10.6 / 13.0; 256 for bins and claim 19.6 / 24.8.)  Up to 1024, where some wait for a place: 512 against 256 threads, one call with one batch,
// 896 tiles (2^22 pairs, dim 16, 8 M nodes) 4220 and 4306 us; 1024 bins, 130 000 pairs, dim 16, 94.3 and 95.3, 100 000, dim 128, 187.2 and 184.7.
constexpr uint32_t kWideTile = 1024;
constexpr unsigned kWideBlocks = 1024;
hipError_t launch_prepare(const Helpers& h, bool claim_first, hipStream_t st)
{
    const size_t own = claim_first ? claim_lds_bytes(h.resolve.bin) : 0, lds = own > h.lds_bytes() ? own : h.lds_bytes();
    const PrepArgs& p = h.claims ? h.claim : h.resolve;
    const bool wide = p.bin.tile >= kWideTile && h.count() <= kWideBlocks;
#define NE_CASE(M_)                                                                              \
    if (wide) hipLaunchKernelGGL((prepare_kernel<M_, 512>), dim3(h.count()), dim3(512), lds, st, h, claim_first);  \
    else hipLaunchKernelGGL((prepare_kernel<M_, 256>), dim3(h.count()), dim3(256), lds, st, h, claim_first);
    if (p.pairs) { NE_CASE(kPairRefs) } else if (p.seg_entries) { NE_CASE(kSegRefs) } else { NE_CASE(kWalkRefs) }
#undef NE_CASE
    return hipGetLastError();
}

// Lane groups of the apply kernel: one dwordx4 chunk per lane as long as a wavefront holds the row, however many
// references a pair has (the train kernel's groups, with a lane per reference, leave 63 of 64 lanes idle at dim 4,
// K = 62: 32 768 pairs among a million nodes 465 us, now 316; 2^20 pairs among 64 million 19.3 ms, now 13.9).  Its number of items is only
// known on the device; kApplyGroups lane groups leave each a few of them, of which all but the first find their entries there, and not so many
// that those with long lists finish last (level but for the fewest of dim 512: 6 x 65 536 pairs, dim 128, 32 M / 1 M nodes, and 3 x 32 768, dim 512: 131 072 groups 693 / 625 /
// 944 us, 57 344 692 / 622 / 945, 28 672 689 / 627 / 949, 14 336 694 / 627 / 962), but kApplyBlocks workgroups at least, where
// groups are small (the apply launch of 2^22 pairs, dim 16, with a quarter of them 784 instead of 681 us).  Up to
// kHubBlocks workgroups more take the hubs' items, whose chains are the longest (512 take 6 % more of a batch of 65 536 pairs among
// 1000 .. 10 000 nodes, 256 10 % more among a million; half as many as the items fill are level in small batches, a quarter take 9 - 14 % more).
constexpr unsigned kApplyGroups = 57344, kApplyBlocks = 7168;
constexpr unsigned kHubBlocks = 1024;
hipError_t launch_apply(ApplyArgs a, uint32_t refs, hipStream_t st)
{
    a.most = refs / 2;                      // every item has two references or more to its row
    if (a.most == 0) return hipSuccess;
    Shape s;
    if (!pick_shape(a.d4, 0, &s)) return hipErrorInvalidValue;
    const unsigned groups = 256u / s.G;
    const unsigned want = (a.most + groups - 1) / groups;
    const unsigned hubs = static_cast<unsigned>((most_hub_items(refs) + groups - 1) / groups);
    a.most_hubs = static_cast<uint32_t>(most_hub_items(refs));
    a.hub_blocks = hubs < kHubBlocks ? hubs : kHubBlocks;
    const unsigned grid = std::min(want, std::max(kApplyGroups / groups, kApplyBlocks)) + a.hub_blocks;
#define NE_CASE(G_, N_)                                                                          \
    if (s.G == G_ && s.NCH == N_) {                                                              \
        hipLaunchKernelGGL((apply_kernel<G_, N_>), dim3(grid), dim3(256), 0, st, a);             \
        return hipGetLastError();                                                                \
    }
    NE_FOR_EACH_SHAPE(NE_CASE)
#undef NE_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_loss(const Shape& s, const LossArgs& a, hipStream_t st)
{
    const int groups = 256 / s.G;
    // workgroups: enough to fill the chip, few enough for their atomic adds to one address to hide (65 536 pairs,
    // dim 128, K = 5: 512 .. 1024 take 44 - 45 us with the caller's zero-fill, 2048 54, one per 8 pairs 118; at dim
    // 16 .. 1024 384 are up to 38 % behind on a million pairs and 23 % ahead on 4096, 1536 up to 40 % behind)
    const int64_t want = (a.B + groups - 1) / groups;
    const unsigned grid = static_cast<unsigned>(want < 768 ? want : 768);
#define NE_CASE(G_, N_)                                                                          \
    if (s.G == G_ && s.NCH == N_) {                                                              \
        hipLaunchKernelGGL((loss_kernel<G_, N_, 3>), dim3(grid), dim3(256), 0, st, a);           \
        return hipGetLastError();                                                                \
    }
    NE_FOR_EACH_SHAPE(NE_CASE)
#undef NE_CASE
    return hipErrorInvalidValue;
}

// Largest batch: its references stay below 2^28, so that places of the list fit a work item's 29 bits and grids 32.
constexpr int64_t kMaxBatch = static_cast<int64_t>(1) << 22;
// helper workgroups that prefetch the samples of a later batch from pinned host memory (512 KB per batch of 65536)
constexpr unsigned kFetchBlocks = 8;

bool workspace_layout(int32_t dim, int64_t max_B, int32_t max_K, char* base, Workspace* w)
{
    if (dim < 4 || dim > NE_MAX_DIM || dim % 4 != 0 || max_B < 1 || max_B > kMaxBatch || max_K < 0 ||
        max_K > NE_MAX_NEGATIVES)
        return false;
    const uint64_t refs = static_cast<uint64_t>(max_B) * (max_K + 2);
    auto up = [](size_t v) { return (v + 255) & ~static_cast<size_t>(255); };
    size_t off = 0;
    auto take = [&](size_t bytes) { char* p = base + off; off = up(off + bytes); return p; };
    for (PrepSlot& p : w->prep) {
        p.ids = reinterpret_cast<int32_t*>(take(refs * 4));
        p.where = reinterpret_cast<uint32_t*>(take(refs * 4));
        p.keys = reinterpret_cast<uint32_t*>(take(refs * 8));
        p.tags = p.keys + refs;
        p.segs = reinterpret_cast<uint32_t*>(take(max_segs(refs) * 4));
    }
    for (ItemSlot& p : w->item_slots) {
        p.items = reinterpret_cast<uint2*>(take(most_items(refs) * sizeof(uint2)));
        p.hub_items = reinterpret_cast<uint4*>(take(most_hub_items(refs) * sizeof(uint4)));
        p.bins = reinterpret_cast<uint4*>(take(sizeof(uint4) << binning(refs).bits));      // (more references never have fewer bins)
    }
    w->items = reinterpret_cast<uint2*>(take(most_items(refs) * sizeof(uint2)));
    w->hub_items = reinterpret_cast<uint4*>(take(most_hub_items(refs) * sizeof(uint4)));
    w->totals = reinterpret_cast<unsigned long long*>(take(sizeof(unsigned long long)));
    w->list = reinterpret_cast<uint2*>(take(refs * sizeof(uint2)));
    // two rows per pair or walk entry, a segment's entries twice and its context rows: never more than references, and as
    // many where the batch is walks with window 1 and no negatives, which every handle accepts
    w->buf = reinterpret_cast<float*>(take(refs * static_cast<size_t>(dim) * 4));
    // (hub_accumulator)
    w->accs = refs / kItemRefs + 1;
    w->acc = reinterpret_cast<float*>(take(w->accs * static_cast<size_t>(dim) * 4));
    w->arrived = reinterpret_cast<uint32_t*>(take(w->accs * 4));
    w->total_bytes = off;
    return true;
}

// (a kernel instead of hipMemsetAsync so that callers may capture the stream)
__global__ __launch_bounds__(256) void clear_kernel(uint32_t* __restrict__ p, size_t n)
{
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0u;
}

// The state every apply launch expects to find and leaves behind: accumulators and their counters zero.
hipError_t clear_workspace(const Workspace& w, int32_t dim, hipStream_t st)
{
    const size_t floats = w.accs * static_cast<size_t>(dim);
    const size_t want = (floats + 255) / 256;
    const dim3 grid(static_cast<unsigned>(want < 16384 ? want : 16384));
    hipLaunchKernelGGL(clear_kernel, grid, dim3(256), 0, st, reinterpret_cast<uint32_t*>(w.acc), floats);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(clear_kernel, grid, dim3(256), 0, st, w.arrived, w.accs);
    return hipGetLastError();
}

ne_status check_batch_args(const ne_tables* t, const ne_alias* al, const int32_t* pairs, int64_t B, int32_t K,
                           Shape* shape)
{
    if (!t) return fail(NE_ERR_ARG, "tables handle is NULL");
    if (B < 0 || B > kMaxBatch) return fail(NE_ERR_ARG, "B out of range [0, 2^22]");
    if (K < 0 || K > NE_MAX_NEGATIVES) return fail(NE_ERR_ARG, "K out of range [0, 62]");
    if (K > 0 && !al) return fail(NE_ERR_ARG, "alias handle is NULL but K > 0");
    if (B > 0 && !pairs) return fail(NE_ERR_ARG, "pairs_dev is NULL");
    if (!aligned(pairs, 8)) return fail(NE_ERR_ARG, "pairs_dev must be 8-byte aligned");
    if (al && (al->base < 0 || al->base + al->n > t->num_nodes))
        return fail(NE_ERR_STATE, "alias id range [base, base+n) is not inside the tables' [0, num_nodes)");
    if (!pick_shape(t->dim / 4, K, shape)) return fail(NE_ERR_ARG, "no launch shape for this (dim, K)");
    return NE_OK;
}

// The launches of a run of batches, common to the pair and the walk shapes: claim(0), then resolve(0) +
// claim(1), stand alone (a first batch of one bin: both in one launch); then per batch kernel A = train(i) + resolve(i+1) + claim(i+2) (+ sample prefetch)
// and kernel B = apply(i).  prep(i) describes batch i (refs = 0 past the end); train(ta, helpers) launches
// the shape's train kernel.  direct: the per-sample mode, which leaves nothing to apply.
template <class PrepFn, class TrainFn>
ne_status run_batches(ne_tables* t, int64_t n_batches, int64_t R, int32_t window, int32_t K,
                      const float* lr_host, hipStream_t st, PrepFn prep, TrainFn train, bool direct = false)
{
    const Workspace& w = t->ws;
    // the parts of a batch's description that every shape shares
    auto prepared = [&](int64_t i) {
        PrepArgs pa = prep(i);
        if (!pa.refs) return pa;
        const PrepSlot& ps = w.prep[i % 3];
        const ItemSlot& is = w.item_slots[i % 2];
        pa.bin = binning(pa.refs);
        pa.ids = ps.ids; pa.where = ps.where; pa.keys = ps.keys; pa.tags = ps.tags; pa.segs = ps.segs;
        pa.items = direct ? nullptr : is.items; pa.hub_items = is.hub_items; pa.bins = is.bins;
        pa.k0 = static_cast<uint32_t>(t->seed); pa.k1 = static_cast<uint32_t>(t->seed >> 32);
        return pa;
    };
    auto helpers = [](const PrepArgs& resolve, const PrepArgs& claim, bool prefetch) {
        Helpers h{};
        h.resolve = resolve; h.claim = claim;
        h.resolves = resolve.refs ? 1u << resolve.bin.bits : 0u;
        h.claims = claim.refs ? claim.bin.tiles : 0u;
        h.fetches = prefetch && claim.refs ? claim.fetch_blocks : 0u;
        return h;
    };
    PrepArgs cur = prepared(0), next = prepared(1);
    const bool at_once = cur.refs <= kOneBin;
    hipError_t e = at_once ? hipSuccess : launch_prepare(helpers(PrepArgs{}, cur, false), false, st);
    if (e != hipSuccess) return fail(NE_ERR_HIP, std::string("claim launch: ") + hipGetErrorString(e));
    e = launch_prepare(helpers(cur, next, false), at_once, st);
    if (e != hipSuccess) return fail(NE_ERR_HIP, std::string("resolve launch: ") + hipGetErrorString(e));

    for (int64_t i = 0; i < n_batches; ++i) {
        const PrepArgs after = prepared(i + 2);
        TrainArgs ta{};
        ta.X = reinterpret_cast<float4*>(t->vertex); ta.C = reinterpret_cast<float4*>(t->context);
        ta.B = cur.refs / R; ta.window = window; ta.K = K; ta.d4 = t->dim / 4; ta.lr = lr_host[i];
        ta.ids = cur.ids; ta.where = cur.where; ta.tags = cur.tags; ta.tile = cur.bin.tile; ta.list = w.list; ta.buf = reinterpret_cast<float4*>(w.buf);
        const bool timed = profile_begin(t, st);
        Helpers h = helpers(next, after, true);
        if (!direct) {
            const uint32_t bins = 1u << cur.bin.bits, share = std::min(bins, std::max(kGatherBins, bins / kGatherBlocks));
            h.gather = {cur.bins, cur.items, cur.hub_items, w.items, w.hub_items, w.totals, bins, share};
            h.gathers = bins / share;
        }
        e = train(ta, h);
        if (e != hipSuccess) return fail(NE_ERR_HIP, std::string("train launch: ") + hipGetErrorString(e));
        if (timed) profile_end(t, st);

        if (!direct) {
            ApplyArgs aa{};
            aa.X = ta.X; aa.C = ta.C; aa.d4 = ta.d4; aa.items = w.items; aa.hub_items = w.hub_items; aa.totals = w.totals; aa.list = w.list; aa.buf = ta.buf;
            aa.acc = w.acc; aa.arrived = w.arrived;
            e = launch_apply(aa, cur.refs, st);
            if (e != hipSuccess) return fail(NE_ERR_HIP, std::string("apply launch: ") + hipGetErrorString(e));
        }
        t->batches_done += 1;
        cur = next;
        next = after;
    }
    return NE_OK;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------------------------
extern "C" {

const char* ne_last_error(void) { return g_last_error.c_str(); }

size_t ne_workspace_bytes(int32_t dim, int64_t max_batch, int32_t max_negatives)
{
    Workspace w;
    if (!workspace_layout(dim, max_batch, max_negatives, nullptr, &w)) return 0;
    return w.total_bytes;
}

ne_status ne_create_tables(ne_tables** out, int64_t num_nodes, int32_t dim, float* vertex_dev,
                           float* context_dev, uint64_t seed, int32_t init, int64_t max_batch,
                           int32_t max_negatives, void* workspace_dev, size_t workspace_bytes,
                           void* hip_stream)
{
    if (!out) return fail(NE_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (num_nodes <= 0 || num_nodes >= (static_cast<int64_t>(1) << 31))
        return fail(NE_ERR_ARG, "num_nodes must be in (0, 2^31)");
    if (dim < 4 || dim > NE_MAX_DIM || dim % 4 != 0)
        return fail(NE_ERR_ARG, "dim must be a multiple of 4 in [4, 1024]");
    if (!vertex_dev || !context_dev) return fail(NE_ERR_ARG, "table pointer is NULL");
    if (!aligned(vertex_dev, 16) || !aligned(context_dev, 16))
        return fail(NE_ERR_ARG, "table pointers must be 16-byte aligned");
    ne_tables* t = new (std::nothrow) ne_tables{};
    if (!t) return fail(NE_ERR_NOMEM, "host allocation failed");
    t->num_nodes = num_nodes; t->dim = dim; t->vertex = vertex_dev; t->context = context_dev; t->seed = seed;
    t->max_batch = 0; t->max_negatives = 0; t->batches_done = 0; t->profile_every = 0; t->ev_used = 0;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);

    if (workspace_dev || max_batch > 0) {   // training requested
        Workspace w;
        if (!workspace_layout(dim, max_batch, max_negatives, static_cast<char*>(workspace_dev), &w)) {
            delete t;
            return fail(NE_ERR_ARG, "max_batch must be in [1, 2^22] and max_negatives in [0, 62]");
        }
        if (!workspace_dev || !aligned(workspace_dev, 256) || workspace_bytes < w.total_bytes) {
            delete t;
            return fail(NE_ERR_ARG, "workspace_dev is NULL, not 256-byte aligned, or smaller than ne_workspace_bytes()");
        }
        t->ws = w; t->max_batch = max_batch; t->max_negatives = max_negatives;
        const hipError_t e = clear_workspace(w, dim, st);
        if (e != hipSuccess) {
            delete t;
            return fail(NE_ERR_HIP, std::string("workspace clear launch: ") + hipGetErrorString(e));
        }
    }
    if (init) {
        const int64_t total = num_nodes * (dim / 4);
        const int64_t want = (total + 255) / 256;
        const unsigned grid = static_cast<unsigned>(want < 65536 * 4 ? (want > 0 ? want : 1) : 65536 * 4);
        hipLaunchKernelGGL(init_tables_kernel, dim3(grid), dim3(256), 0, st, reinterpret_cast<float4*>(vertex_dev),
                           reinterpret_cast<float4*>(context_dev), num_nodes, dim / 4, static_cast<float>(dim),
                           static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32));
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            delete t;
            return fail(NE_ERR_HIP, std::string("init_tables launch: ") + hipGetErrorString(e));
        }
    }
    *out = t;
    return NE_OK;
}

void ne_destroy_tables(ne_tables* t)
{
    if (!t) return;
    for (hipEvent_t e : t->ev_zero) (void)hipEventDestroy(e);
    for (hipEvent_t e : t->ev_start) (void)hipEventDestroy(e);
    for (hipEvent_t e : t->ev_stop) (void)hipEventDestroy(e);
    delete t;
}

ne_status ne_profile_enable(ne_tables* t, int32_t every_n, int32_t max_samples)
{
    if (!t) return fail(NE_ERR_ARG, "tables handle is NULL");
    if (every_n < 0 || max_samples < 0 || max_samples > 65536) return fail(NE_ERR_ARG, "every_n or max_samples out of range");
    t->profile_every = every_n;
    t->ev_used = 0;
    while (every_n > 0 && t->ev_start.size() < static_cast<size_t>(max_samples)) {
        hipEvent_t z = nullptr, a = nullptr, b = nullptr;
        hipError_t e = hipEventCreate(&z);
        if (e == hipSuccess) e = hipEventCreate(&a);
        if (e == hipSuccess) e = hipEventCreate(&b);
        if (e != hipSuccess) {
            if (z) (void)hipEventDestroy(z);
            if (a) (void)hipEventDestroy(a);
            return fail(NE_ERR_HIP, std::string("hipEventCreate: ") + hipGetErrorString(e));
        }
        t->ev_zero.push_back(z);
        t->ev_start.push_back(a);
        t->ev_stop.push_back(b);
    }
    return NE_OK;
}

ne_status ne_profile_read(ne_tables* t, double* total_ms_host, int64_t* samples_host)
{
    if (!t || !total_ms_host || !samples_host) return fail(NE_ERR_ARG, "NULL argument");
    double total = 0.0;
    for (size_t i = 0; i < t->ev_used; ++i) {
        NE_HIP_CHECK(hipEventSynchronize(t->ev_stop[i]));
        float ms = 0.0f, overhead = 0.0f;
        NE_HIP_CHECK(hipEventElapsedTime(&ms, t->ev_start[i], t->ev_stop[i]));
        NE_HIP_CHECK(hipEventElapsedTime(&overhead, t->ev_zero[i], t->ev_start[i]));
        total += static_cast<double>(ms > overhead ? ms - overhead : 0.0f);
    }
    *total_ms_host = total;
    *samples_host = static_cast<int64_t>(t->ev_used);
    t->ev_used = 0;
    return NE_OK;
}
void ne_destroy_alias(ne_alias* a) { delete a; }

ne_status ne_build_neg_alias(ne_alias** out, const uint32_t* degree_host, int64_t n, int32_t base,
                             void* alias_dev, void* hip_stream)
{
    if (!out) return fail(NE_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (!degree_host || !alias_dev) return fail(NE_ERR_ARG, "degree_host or alias_dev is NULL");
    if (n <= 0 || base < 0 || static_cast<int64_t>(base) + n >= (static_cast<int64_t>(1) << 31))
        return fail(NE_ERR_ARG, "need 0 < n, 0 <= base, base + n < 2^31");
    if (!aligned(alias_dev, 8)) return fail(NE_ERR_ARG, "alias_dev must be 8-byte aligned");

    // weights deg^0.75 and their plain left-to-right sum
    std::vector<double> prob;
    std::vector<int64_t> lo_stack, hi_stack;
    uint2* staged = nullptr;
    try {
        prob.resize(static_cast<size_t>(n));
        lo_stack.reserve(static_cast<size_t>(n));
        hi_stack.reserve(static_cast<size_t>(n));
    } catch (const std::bad_alloc&) {
        return fail(NE_ERR_NOMEM, "host allocation failed");
    }
    double total = 0.0;
    for (int64_t i = 0; i < n; ++i) {
        const double dg = static_cast<double>(degree_host[i]);
        const double w = std::sqrt(dg) * std::sqrt(std::sqrt(dg));
        prob[i] = w;
        total += w;
    }
    if (!(total > 0.0)) return fail(NE_ERR_ARG, "all degrees are zero");
    const double nn = static_cast<double>(n);
    for (int64_t i = 0; i < n; ++i) {
        prob[i] = (prob[i] * nn) / total;
        (prob[i] < 1.0 ? lo_stack : hi_stack).push_back(i);
    }
    NE_HIP_CHECK(hipHostMalloc(reinterpret_cast<void**>(&staged), static_cast<size_t>(n) * sizeof(uint2), hipHostMallocDefault));
    auto quantise = [](double thr) -> uint32_t {
        double q = std::floor(thr * 4294967296.0);
        if (q > 4294967295.0) q = 4294967295.0;
        if (q < 0.0) q = 0.0;
        return static_cast<uint32_t>(q);
    };
    // Vose: pair the most recently pushed under-full entry with the most recently pushed over-full one
    while (!lo_stack.empty() && !hi_stack.empty()) {
        const int64_t s = lo_stack.back(); lo_stack.pop_back();
        const int64_t l = hi_stack.back(); hi_stack.pop_back();
        staged[s] = make_uint2(quantise(prob[s]), static_cast<uint32_t>(l));
        prob[l] = (prob[l] + prob[s]) - 1.0;
        (prob[l] < 1.0 ? lo_stack : hi_stack).push_back(l);
    }
    for (int64_t l : hi_stack) staged[l] = make_uint2(0xFFFFFFFFu, static_cast<uint32_t>(l));
    for (int64_t s : lo_stack) staged[s] = make_uint2(0xFFFFFFFFu, static_cast<uint32_t>(s));

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    hipError_t e = hipMemcpyAsync(alias_dev, staged, static_cast<size_t>(n) * sizeof(uint2), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipHostFree(staged);
    if (e != hipSuccess) return fail(NE_ERR_HIP, std::string("alias copy: ") + hipGetErrorString(e));

    ne_alias* a = new (std::nothrow) ne_alias{static_cast<const uint2*>(alias_dev), n, base};
    if (!a) return fail(NE_ERR_NOMEM, "host allocation failed");
    *out = a;
    return NE_OK;
}

// The batches of a sequence of runs (each run: one sample block with its negative-sampling table), B pairs
// each but for the last of a run.  With staging != nullptr (one run only) pairs_dev is the device address of
// samples in pinned host memory, which are prefetched batch by batch into the ring staging[3][B].
static ne_status train_runs_impl(ne_tables* t, const ne_run* runs, int64_t n_runs, int64_t B, int32_t K,
                                 const float* lr_host, int2* staging, void* hip_stream, bool direct = false)
{
    if (!t) return fail(NE_ERR_ARG, "tables handle is NULL");
    if (n_runs < 0 || n_runs > (static_cast<int64_t>(1) << 24)) return fail(NE_ERR_ARG, "n_runs out of range");
    if (n_runs > 0 && !runs) return fail(NE_ERR_ARG, "runs_host is NULL");
    Shape shape;
    struct Batch { int64_t run, first, count; };
    std::vector<Batch> batches;
    for (int64_t r = 0; r < n_runs; ++r) {
        const ne_run& run = runs[r];
        if (run.n_pairs < 0 || run.n_pairs > (static_cast<int64_t>(1) << 40)) return fail(NE_ERR_ARG, "n_pairs out of range");
        // (an empty run may come without a pairs pointer)
        const ne_status rc = check_batch_args(t, run.alias, run.pairs_dev, run.n_pairs > 0 ? B : (B < 0 ? B : 0), K, &shape);
        if (rc != NE_OK) return rc;
        if (run.n_pairs == 0) continue;
        if (B < 1) return fail(NE_ERR_ARG, "B must be at least 1");
        if (!run.pairs_dev) return fail(NE_ERR_ARG, "pairs_dev is NULL");
        try {
            for (int64_t first = 0; first < run.n_pairs; first += B)
                batches.push_back({r, first, run.n_pairs - first < B ? run.n_pairs - first : B});
        } catch (const std::bad_alloc&) {
            return fail(NE_ERR_NOMEM, "host allocation failed");
        }
    }
    const int64_t n_batches = static_cast<int64_t>(batches.size());
    if (n_batches == 0) return NE_OK;
    if (!lr_host) return fail(NE_ERR_ARG, "lr_host is NULL");
    for (int64_t i = 0; i < n_batches; ++i)
        if (!std::isfinite(lr_host[i])) return fail(NE_ERR_ARG, "lr is not finite");
    if (t->max_batch <= 0) return fail(NE_ERR_STATE, "tables were created without a training workspace");
    if (B > t->max_batch || K > t->max_negatives)
        return fail(NE_ERR_ARG, "B or K exceeds the max_batch / max_negatives the workspace was sized for");

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int R = K + 2;

    auto prep_args = [&](int64_t i) {
        PrepArgs pa{};
        if (i >= n_batches) return pa;   // refs = 0: nothing to prepare
        const Batch& bt = batches[i];
        const ne_run& run = runs[bt.run];
        const ne_alias* al = run.alias;
        pa.pairs = staging ? staging + (i % 3) * B : reinterpret_cast<const int2*>(run.pairs_dev) + bt.first;
        if (staging && i + 1 < n_batches) {
            // the launch that trains batch i - 2 and claims batch i also fetches batch i + 1
            pa.fetch_src = reinterpret_cast<const int2*>(run.pairs_dev) + batches[i + 1].first;
            pa.fetch_dst = staging + ((i + 1) % 3) * B;
            pa.fetch_n = batches[i + 1].count;
            pa.fetch_blocks = kFetchBlocks;
        }
        pa.refs = static_cast<uint32_t>(bt.count * R); pa.R = static_cast<uint32_t>(R); pa.K = K;
        pa.sample_base = run.sample_base + static_cast<uint64_t>(bt.first);
        pa.alias = al ? al->table : nullptr; pa.alias_n = al ? static_cast<uint64_t>(al->n) : 1; pa.alias_base = al ? al->base : 0;
        pa.neg_out = run.neg_out_dev ? run.neg_out_dev + bt.first * K : nullptr;
        return pa;
    };

    if (staging) {   // batches 0, 1 and 2 (side by side in both buffers) have no launch to ride along with
        const int64_t n = runs[0].n_pairs < 3 * B ? runs[0].n_pairs : 3 * B;
        hipLaunchKernelGGL(fetch_pairs_kernel, dim3(3 * kFetchBlocks), dim3(256), 0, st, reinterpret_cast<const int2*>(runs[0].pairs_dev), staging, n);
        const hipError_t fe = hipGetLastError();
        if (fe != hipSuccess) return fail(NE_ERR_HIP, std::string("fetch launch: ") + hipGetErrorString(fe));
    }
    return run_batches(t, n_batches, R, 0, K, lr_host, st, prep_args,
                       [&](const TrainArgs& ta, const Helpers& h) { return launch_train(shape, ta, h, direct, st); }, direct);
}

ne_status ne_train_runs(ne_tables* t, const ne_run* runs_host, int64_t n_runs, int64_t B, int32_t K,
                        const float* lr_host, void* hip_stream)
{
    return train_runs_impl(t, runs_host, n_runs, B, K, lr_host, nullptr, hip_stream);
}

ne_status ne_train_block(ne_tables* t, const ne_alias* al, const int32_t* pairs_dev, int64_t n_pairs, int64_t B,
                         int32_t K, const float* lr_host, uint64_t sample_base, int32_t* neg_out_dev,
                         void* hip_stream)
{
    const ne_run run{al, pairs_dev, n_pairs, sample_base, neg_out_dev};
    return train_runs_impl(t, &run, 1, B, K, lr_host, nullptr, hip_stream);
}

ne_status ne_train_block_pinned(ne_tables* t, const ne_alias* al, const int32_t* pairs_host_pinned, int64_t n_pairs,
                                int64_t B, int32_t K, const float* lr_host, uint64_t sample_base, int32_t* staging_dev,
                                int32_t* neg_out_dev, void* hip_stream)
{
    if (n_pairs > 0 && B >= 1) {
        if (!pairs_host_pinned || !aligned(pairs_host_pinned, 8)) return fail(NE_ERR_ARG, "pairs_host_pinned is NULL or not 8-byte aligned");
        if (!staging_dev || !aligned(staging_dev, 16)) return fail(NE_ERR_ARG, "staging_dev is NULL or not 16-byte aligned");
    }
    void* src_dev = const_cast<int32_t*>(pairs_host_pinned);
    if (pairs_host_pinned) {
        hipError_t e = hipHostGetDevicePointer(&src_dev, const_cast<int32_t*>(pairs_host_pinned), 0);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return fail(NE_ERR_ARG, std::string("pairs_host_pinned is not pinned (page-locked) host memory: ") + hipGetErrorString(e));
        }
    }
    const ne_run run{al, static_cast<const int32_t*>(src_dev), n_pairs, sample_base, neg_out_dev};
    return train_runs_impl(t, &run, 1, B, K, lr_host, reinterpret_cast<int2*>(staging_dev), hip_stream);
}

ne_status ne_train_walks(ne_tables* t, const ne_alias* al, const int32_t* walks_dev, int64_t n_walks,
                         int64_t walks_per_batch, int32_t walk_len, int32_t window, int32_t K, const float* lr_host,
                         uint64_t sample_base, int32_t* neg_out_dev, void* hip_stream)
{
    if (!t) return fail(NE_ERR_ARG, "tables handle is NULL");
    if (K < 0 || K > NE_MAX_NEGATIVES) return fail(NE_ERR_ARG, "K out of range [0, 62]");
    if (K > 0 && !al) return fail(NE_ERR_ARG, "alias handle is NULL but K > 0");
    if (walk_len < 2 || walk_len > 65536) return fail(NE_ERR_ARG, "walk_len out of range [2, 65536]");
    if (window < 1 || window > 64) return fail(NE_ERR_ARG, "window out of range [1, 64]");
    if (n_walks < 0 || n_walks > (static_cast<int64_t>(1) << 32)) return fail(NE_ERR_ARG, "n_walks out of range");
    if (al && (al->base < 0 || al->base + al->n > t->num_nodes))
        return fail(NE_ERR_STATE, "alias id range [base, base+n) is not inside the tables' [0, num_nodes)");
    Shape shape;
    if (!pick_shape(t->dim / 4, K, &shape)) return fail(NE_ERR_ARG, "no launch shape for this (dim, K)");
    if (n_walks == 0) return NE_OK;
    if (!walks_dev || !aligned(walks_dev, 4)) return fail(NE_ERR_ARG, "walks_dev is NULL or misaligned");
    if (walks_per_batch < 1) return fail(NE_ERR_ARG, "walks_per_batch must be at least 1");
    if (!lr_host) return fail(NE_ERR_ARG, "lr_host is NULL");
    const int64_t n_batches = (n_walks + walks_per_batch - 1) / walks_per_batch;
    for (int64_t i = 0; i < n_batches; ++i)
        if (!std::isfinite(lr_host[i])) return fail(NE_ERR_ARG, "lr is not finite");
    if (t->max_batch <= 0) return fail(NE_ERR_STATE, "tables were created without a training workspace");
    // the workspace was sized in row references: max_batch * (max_negatives + 2)
    const int64_t R_entry = 1 + static_cast<int64_t>(window) * (K + 1);
    const int64_t ref_budget = t->max_batch * (static_cast<int64_t>(t->max_negatives) + 2);
    const int64_t wpb = walks_per_batch < n_walks ? walks_per_batch : n_walks;
    if (wpb * walk_len > ref_budget / R_entry)
        return fail(NE_ERR_ARG, "a batch of walks names more rows than the workspace was sized for: need walks_per_batch * "
                                "walk_len * (1 + window * (K + 1)) <= max_batch * (max_negatives + 2)");
    // One workgroup per segment of E consecutive entries (every row of a segment named once) when a
    // segment is longer than the window, its rows fit into LDS and the padding of the last segment of
    // a walk does not cost more references than it saves; else one lane group per entry.
    const int64_t E = kTrainThreads / shape.G;
    const int64_t segs_per_walk = (walk_len + E - 1) / E;
    const int64_t R_seg = E + (E + window - 1) + E * window * K;
    const bool by_segments = E >= window + 2 && seg_lds_bytes(shape, window) <= 48 * 1024 &&
                             segs_per_walk * R_seg <= walk_len * R_entry;
    const int64_t R = by_segments ? R_seg : R_entry;
    const int64_t groups_per_walk = by_segments ? segs_per_walk : walk_len;   // reference groups (of R) per walk

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int64_t per_walk = static_cast<int64_t>(walk_len) * window;   // sample indices (and neg_out rows) per walk

    auto prep_args = [&](int64_t i) {
        PrepArgs pa{};
        if (i >= n_batches) return pa;   // refs = 0: nothing to prepare
        const int64_t first = i * walks_per_batch;
        const int64_t count = (n_walks - first < walks_per_batch) ? n_walks - first : walks_per_batch;
        pa.walks = walks_dev + first * walk_len; pa.walk_len = walk_len; pa.window = window;
        pa.refs = static_cast<uint32_t>(count * groups_per_walk * R); pa.R = static_cast<uint32_t>(R); pa.K = K;
        pa.seg_entries = by_segments ? static_cast<uint32_t>(E) : 0u;
        pa.segs_per_walk = static_cast<uint32_t>(segs_per_walk);
        pa.sample_base = sample_base + static_cast<uint64_t>(first * per_walk);
        pa.alias = al ? al->table : nullptr; pa.alias_n = al ? static_cast<uint64_t>(al->n) : 1; pa.alias_base = al ? al->base : 0;
        pa.neg_out = neg_out_dev ? neg_out_dev + first * per_walk * K : nullptr;
        return pa;
    };

    return run_batches(t, n_batches, R, window, K, lr_host, st, prep_args, [&](const TrainArgs& ta, const Helpers& h) {
        return by_segments ? launch_train_seg(shape, ta, h, st) : launch_train_walk(shape, ta, h, st);
    });
}

ne_status ne_train_batch(ne_tables* t, const ne_alias* al, const int32_t* pairs_dev, int64_t B, int32_t K,
                         float lr, uint64_t sample_base, int32_t* neg_out_dev, void* hip_stream)
{
    if (B == 0) {
        Shape shape;
        return check_batch_args(t, al, pairs_dev, B, K, &shape);
    }
    return ne_train_block(t, al, pairs_dev, B, B, K, &lr, sample_base, neg_out_dev, hip_stream);
}

ne_status ne_train_block_async(ne_tables* t, const ne_alias* al, const int32_t* pairs_dev, int64_t n_pairs, int64_t B,
                               int32_t K, const float* lr_host, uint64_t sample_base, int32_t* neg_out_dev,
                               void* hip_stream)
{
    const ne_run run{al, pairs_dev, n_pairs, sample_base, neg_out_dev};
    return train_runs_impl(t, &run, 1, B, K, lr_host, nullptr, hip_stream, true);
}

ne_status ne_train_batch_async(ne_tables* t, const ne_alias* al, const int32_t* pairs_dev, int64_t B, int32_t K,
                               float lr, uint64_t sample_base, int32_t* neg_out_dev, void* hip_stream)
{
    if (B == 0) {
        Shape shape;
        return check_batch_args(t, al, pairs_dev, B, K, &shape);
    }
    return ne_train_block_async(t, al, pairs_dev, B, B, K, &lr, sample_base, neg_out_dev, hip_stream);
}

ne_status ne_eval_loss(const ne_tables* t, const ne_alias* al, const int32_t* pairs_dev, int64_t B, int32_t K,
                       uint64_t sample_base, double* loss_sum_dev, int32_t* neg_out_dev, void* hip_stream)
{
    Shape shape;
    ne_status rc = check_batch_args(t, al, pairs_dev, B, K, &shape);
    if (rc != NE_OK) return rc;
    if (!loss_sum_dev || !aligned(loss_sum_dev, 8)) return fail(NE_ERR_ARG, "loss_sum_dev is NULL or misaligned");
    if (B == 0) return NE_OK;
    LossArgs la{};
    la.X = reinterpret_cast<const float4*>(t->vertex);
    la.C = reinterpret_cast<const float4*>(t->context);
    la.pairs = reinterpret_cast<const int2*>(pairs_dev);
    la.B = B; la.K = K; la.d4 = t->dim / 4; la.sample_base = sample_base;
    la.k0 = static_cast<uint32_t>(t->seed); la.k1 = static_cast<uint32_t>(t->seed >> 32);
    la.alias = al ? al->table : nullptr; la.alias_n = al ? static_cast<uint64_t>(al->n) : 1; la.alias_base = al ? al->base : 0;
    la.neg_out = neg_out_dev; la.loss = loss_sum_dev;
    hipError_t e = launch_loss(shape, la, static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail(NE_ERR_HIP, std::string("loss launch: ") + hipGetErrorString(e));
    return NE_OK;
}

ne_status ne_set_vertex_window(ne_tables* t, float* vertex_window_dev, int64_t first_row, int64_t num_rows)
{
    if (!t) return fail(NE_ERR_ARG, "tables handle is NULL");
    if (!vertex_window_dev || !aligned(vertex_window_dev, 16)) return fail(NE_ERR_ARG, "vertex_window_dev is NULL or not 16-byte aligned");
    if (first_row < 0 || num_rows <= 0 || first_row + num_rows > t->num_nodes)
        return fail(NE_ERR_ARG, "window [first_row, first_row + num_rows) is not inside [0, num_nodes)");
    // the kernels index vertex rows by absolute id: point them at where row 0 would be
    t->vertex = vertex_window_dev - first_row * static_cast<int64_t>(t->dim);
    return NE_OK;
}

ne_status ne_score_pairs(const ne_tables* t, const int32_t* pairs_dev, int64_t n, int32_t second_from_context,
                         float* scores_dev, void* hip_stream)
{
    if (!t) return fail(NE_ERR_ARG, "tables handle is NULL");
    if (n < 0 || n > (static_cast<int64_t>(1) << 40)) return fail(NE_ERR_ARG, "n out of range");
    if (n == 0) return NE_OK;
    if (!pairs_dev || !aligned(pairs_dev, 8)) return fail(NE_ERR_ARG, "pairs_dev is NULL or not 8-byte aligned");
    if (!scores_dev || !aligned(scores_dev, 4)) return fail(NE_ERR_ARG, "scores_dev is NULL or misaligned");
    const int64_t want = (n + 15) / 16;
    const unsigned grid = static_cast<unsigned>(want < 65536 ? want : 65536);
    hipLaunchKernelGGL(score_pairs_kernel, dim3(grid), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       reinterpret_cast<const float4*>(t->vertex),
                       reinterpret_cast<const float4*>(second_from_context ? t->context : t->vertex),
                       reinterpret_cast<const int2*>(pairs_dev), n, t->dim / 4, scores_dev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(NE_ERR_HIP, std::string("score launch: ") + hipGetErrorString(e));
    return NE_OK;
}

ne_status ne_set_tuning(ne_tables* t, int32_t list_cap, int32_t sweep_per_thread)
{
    if (!t) return fail(NE_ERR_ARG, "tables handle is NULL");
    if (list_cap < -1 || list_cap > 8) return fail(NE_ERR_ARG, "list_cap must be -1 (automatic) or in [0, 8]");
    if (sweep_per_thread != 0 && sweep_per_thread != 2 && sweep_per_thread != 4 && sweep_per_thread != 8)
        return fail(NE_ERR_ARG, "sweep_per_thread must be 0 (automatic), 2, 4 or 8");
    return NE_OK;
}

uint32_t ne_hash_position(uint32_t key, uint32_t positions)
{
    if (positions < 2 || positions > 0x80000000u || (positions & (positions - 1)) != 0) return 0xFFFFFFFFu;
    return hash_position(key, positions - 1);
}

ne_status ne_validate_pairs(const ne_tables* t, const int32_t* pairs_dev, int64_t B,
                            unsigned long long* bad_count_dev, void* hip_stream)
{
    if (!t || !bad_count_dev) return fail(NE_ERR_ARG, "NULL argument");
    if (B < 0 || B > (static_cast<int64_t>(1) << 40)) return fail(NE_ERR_ARG, "B out of range");
    if (B == 0) return NE_OK;
    if (!pairs_dev) return fail(NE_ERR_ARG, "pairs_dev is NULL");
    const int64_t count = 2 * B;
    const int64_t want = (count + 255) / 256;
    const unsigned grid = static_cast<unsigned>(want < 65536 ? want : 65536);
    hipLaunchKernelGGL(validate_pairs_kernel, dim3(grid), dim3(256), 0, static_cast<hipStream_t>(hip_stream), pairs_dev,
                       count, t->num_nodes, bad_count_dev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(NE_ERR_HIP, std::string("validate launch: ") + hipGetErrorString(e));
    return NE_OK;
}

}  // extern "C"
