// Attention of many query items over one context (a prefill chunk of hundreds of rows, or the verify rows
// of several sequences): a workgroup of four wavefronts takes 64 items (row, head of a key head's group)
// of one key head over one part of the keys, a wavefront 16 of them.  The kernel for fewer items
// (attn_rows_kernel, fast.hip) gives a workgroup 16 items and shares the keys out over its wavefronts: every
// block of 16 then pulls all keys through the vector cache, on every die, and ends in a merge of eight states.
// Here a page of keys (64) goes to LDS once for the four wavefronts, one page ahead by direct loads, and the
// workgroups that share it are neighbours on one die.
// What bounds it: a page takes a wavefront 1.05 us (2500 cycles: 768 of matrix instructions, about as many of
// softmax arithmetic, the rest latencies of one dependent chain), and two workgroups on a compute unit read
// their fragments at the LDS's rate (160 KB a page).  Measured and not taken: rings of three and four pages
// (nothing, and one workgroup a compute unit: 10 to 30 % slower), eight wavefronts and 128 items (0 to 20 %
// slower), pages of 32 keys (two softmax chains for one: 53 -> 45 us on the mix of 16 sequences), 32 items a
// wavefront on those (slower: half the wavefronts, each 1.1 us a tile).
#include <algorithm>

#include "fast_common.h"
#include "lds_stream.h"

namespace {

constexpr int ITEMS_WAVES = 4, ITEMS_GROUP = ITEMS_WAVES * 16, ITEMS_STAGES = 2;

__host__ __device__ inline int items_parts(const SeqDesc &s, int part_pages) {
    const int keys = s.len_ub + s.nrows < s.capacity ? s.len_ub + s.nrows : s.capacity;
    return ((keys + VF_TILE - 1) / VF_TILE + part_pages - 1) / part_pages;
}

// Sum over the four lanes that share an item (lane & 15).
__device__ __forceinline__ float item_sum(float x) {
    x += __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
}

template <int HD>
__global__ __launch_bounds__(ITEMS_WAVES * 64) VF_MFMA_KERNEL void attn_items_kernel(
    Batch b, ItemsGrid grid, int layer, const bf16_t *__restrict__ q, bf16_t *__restrict__ o, int hq, int hkv, int ncb,
    float scale_log2e, float *__restrict__ part) {
    constexpr int KD = HD / 32, DB = HD / 16, FR = HD / 4, LPW = FR / ITEMS_WAVES, S = ITEMS_STAGES;
    extern __shared__ __align__(1024) unsigned char smem[];   // ring of S pages: K fragments, then V^T
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g4 = lane >> 4, l15 = lane & 15;
    const int group = hq / hkv;
    // The item groups that read the same keys are neighbours, so that they share a die's L2; the one that
    // sees the most keys comes first.
    int l = die_order(blockIdx.x, gridDim.x), seq = 0;
#pragma unroll
    for (int i = 1; i < VF_MAX_BATCH; ++i) seq += l >= grid.first[i];
    seq = __builtin_amdgcn_readfirstlane(seq);
    const SeqDesc &s = b.s[seq];
    l -= grid.first[seq];
    const int n_items = s.nrows * group, groups = (n_items + ITEMS_GROUP - 1) / ITEMS_GROUP;
    const int parts = items_parts(s, grid.part_pages);
    const int kpart = __builtin_amdgcn_readfirstlane(l / groups % parts), kvh = __builtin_amdgcn_readfirstlane(l / (groups * parts));
    const int group0 = __builtin_amdgcn_readfirstlane(groups - 1 - l % groups) * ITEMS_GROUP, wave0 = group0 + wave * 16;
    const int len = __builtin_amdgcn_readfirstlane(s.state[0]), kmax = min(len + s.nrows, s.capacity);
    const int group_last = __builtin_amdgcn_readfirstlane(min(kmax - 1, len + min(n_items - 1, group0 + ITEMS_GROUP - 1) / group));   // last key any item sees
    const int pages = group_last / VF_TILE + 1, p_begin = kpart * grid.part_pages;
    // the last part also takes what a length beyond the host's bound adds (a call replayed from a graph)
    const int p_end = kpart == parts - 1 ? pages : min(pages, p_begin + grid.part_pages);
    if (p_begin >= p_end) return;
    const bool has_items = wave0 < n_items;   // a wavefront without items still loads its share of the pages
    const int wave_last = min(group_last, len + min(n_items - 1, wave0 + 15) / group);   // last key one of its items sees
    const int wave_first = min(kmax - 1, len + min(n_items - 1, wave0) / group);         // last key they all see
    const int item = min(n_items - 1, wave0 + l15);   // past the last item: the last one again, not stored
    const int row = s.row0 + item / group, head = kvh * group + item % group, last_key = len + item / group;
    bf16x8 qf[KD];
#pragma unroll
    for (int kd = 0; kd < KD; ++kd) qf[kd] = *reinterpret_cast<const bf16x8 *>(q + ((size_t)row * hq + head) * HD + kd * 32 + g4 * 8);
    // this wavefront's share of a page: half of its K or of its V^T fragments
    const size_t page_bytes = (size_t)2 * hkv * VF_TILE * HD * 2;
    const char *src = s.kv + (size_t)layer * s.n_pages * page_bytes + (size_t)(wave < ITEMS_WAVES / 2 ? kvh : hkv + kvh) * (VF_TILE * HD * 2) +
                      wave % (ITEMS_WAVES / 2) * (LPW * 1024);
    const unsigned lds0 = lds_address(smem) + wave * (LPW * 1024), lane_off = lane * 16;
    const int32_t *table = s.block_table;
    int page_v = 0;   // ids of this part's pages, one per lane, read once
    if (table) page_v = table[min(p_begin + lane, pages - 1)];
    auto issue = [&](int i) {
        const int t = min(p_begin + i, p_end - 1), pi = t - p_begin;   // past the end: the last page again, not used
        const int page = !table ? t
                         : pi < 64      ? __builtin_amdgcn_readlane(page_v, pi)
                                        : __builtin_amdgcn_readfirstlane(table[t]);
        const char *p = src + (size_t)page * page_bytes;
        const unsigned dst = lds0 + (unsigned)i % S * (FR * 1024);
        static_for<0, LPW>([&](auto f) { fragment_to_lds<(int)f * 1024>(p + (int)f * 1024, lane_off, dst); });
    };
    floatx4 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = floatx4{0.f, 0.f, 0.f, 0.f};
    float m_run = -1e30f, l_run = 0.f;   // l_run: this lane's own keys; the four lanes of an item are added at the end
    auto update = [&](const unsigned char *st, int t0, auto masked) {
        constexpr bool MASKED = decltype(masked)::value;
        floatx4 sc[4];   // [32-key half of the page][16-key half]: lane holds keys t0 + 32 * t + 8 * g4 + 4 * h + j of item l15
#pragma unroll
        for (int f = 0; f < 4; ++f) sc[f] = floatx4{0.f, 0.f, 0.f, 0.f};
        // All of a page's fragments leave LDS together, K first and V^T under the softmax: left to the
        // compiler, each pair of them is read right in front of its products, which wait out the latency.
        bf16x8 kf[4 * KD], vf[2 * DB];
#pragma unroll
        for (int kd = 0; kd < KD; ++kd)
#pragma unroll
            for (int f = 0; f < 4; ++f) kf[f * KD + kd] = *reinterpret_cast<const bf16x8 *>(st + (f * KD + kd) * 1024);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int f = 0; f < 2 * DB; ++f) vf[f] = *reinterpret_cast<const bf16x8 *>(st + (FR / 2 + f) * 1024);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int kd = 0; kd < KD; ++kd)
#pragma unroll
            for (int f = 0; f < 4; ++f) sc[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[f * KD + kd], qf[kd], sc[f], 0, 0, 0);
        if constexpr (MASKED)
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (t0 + (j >> 3) * 32 + g4 * 8 + (j & 7) > last_key) sc[j >> 2][j & 3] = -INFINITY;
        float mx = fmaxf(sc[0][0], sc[0][1]);
#pragma unroll
        for (int j = 2; j < 16; ++j) mx = fmaxf(mx, sc[j >> 2][j & 3]);
        mx = over_item(mx, [](float x, float y) { return fmaxf(x, y); });
        const float m_new = fmaxf(m_run, mx * scale_log2e);
        if (__builtin_amdgcn_ballot_w64(m_new != m_run)) {
            const float corr = __builtin_amdgcn_exp2f(m_run - m_new);
            l_run *= corr;
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] *= corr;
            m_run = m_new;
        }
        // probabilities as a sum of two bfloat16 values (16 significant bits): the P V product then
        // carries no more rounding than its bfloat16 V operand
        bf16x8 hi[2], lo[2];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float p = __builtin_amdgcn_exp2f(fmaf(sc[j >> 2][j & 3], scale_log2e, -m_new));
            l_run += p;
            hi[j >> 3][j & 7] = (bf16_t)p;
            lo[j >> 3][j & 7] = (bf16_t)(p - (float)hi[j >> 3][j & 7]);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (MASKED && t0 + t * 32 > wave_last) continue;   // no item sees a key of this half: nor does 0 times its values
            if constexpr (MASKED)   // rows of the cache at or past kmax may hold anything
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (t0 + t * 32 + g4 * 8 + j >= kmax)
#pragma unroll
                        for (int db = 0; db < DB; ++db) vf[t * DB + db][j] = (bf16_t)0.f;
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[t * DB + db], hi[t], acc[db], 0, 0, 0);
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[t * DB + db], lo[t], acc[db], 0, 0, 0);
        }
    };
#pragma unroll
    for (int i = 0; i < S - 1; ++i) issue(i);
    // the query fragments have landed here, or the compiler would wait for every load in flight at each page
#pragma unroll
    for (int kd = 0; kd < KD; ++kd) asm volatile("" : "+v"(qf[kd]));
    const int n = p_end - p_begin;
    for (int i = 0; i < n; ++i) {
        vm_wait<(S - 2) * LPW>();   // page i has landed; behind the barrier everyone's share of it has,
        lds_sync();                 // and page i - 1 has been read, so its slot takes page i + S - 1
        issue(i + S - 1);
        const int t0 = (p_begin + i) * VF_TILE;
        const unsigned char *st = smem + (unsigned)i % S * (FR * 1024) + lane_off;
        if (!has_items || t0 > wave_last) continue;
        if (t0 + VF_TILE - 1 <= wave_first) update(st, t0, std::false_type{});
        else update(st, t0, std::true_type{});
    }
    vm_wait<0>();   // nothing is on its way to LDS when the workgroup ends
    const float sum = item_sum(l_run);
    if (wave0 + l15 >= n_items) return;
    if (grid.merge) {   // a record [max, sum, -, -, O[hd]] for the merge kernel
        float *rec = part + ((size_t)(grid.record[seq] + (row - s.row0) * parts + kpart) * hq + head) * (HD + ATTF_STRIDE_PAD);
        if (g4 == 0) *reinterpret_cast<float2 *>(rec) = float2{m_run, sum};
#pragma unroll
        for (int db = 0; db < DB; ++db) *reinterpret_cast<floatx4 *>(rec + ATTF_STRIDE_PAD + db * 16 + g4 * 4) = acc[db];
    } else {
        const float inv = 1.0f / sum;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const floatx4 v = acc[db] * inv;
            *reinterpret_cast<u32x2 *>(o + xfrag_index(row, head * HD + db * 16 + g4 * 4, ncb)) = pack4_bf16(v[0], v[1], v[2], v[3]);
        }
    }
}

// Merge of the key parts by log-sum-exp: HD / 4 threads per (row, head), four output values each.  What bounds it is the
// chain of memory round trips: where a row's records lie comes from the kernel arguments (a descriptor looked up per lane
// and its sequence's length behind it were two trips more), eight records are requested together without knowing how many
// there are, and the row's last key, which says that, with them.
struct ItemsMerge { int row0[VF_MAX_BATCH], parts[VF_MAX_BATCH], record[VF_MAX_BATCH], rows, part_keys; };   // row0: a huge number past the last sequence

template <int HD>
__global__ __launch_bounds__(256) void attn_items_merge_kernel(ItemsMerge g, const RowPlace *__restrict__ place, const float *__restrict__ part,
                                                               bf16_t *__restrict__ o, int hq, int ncb) {
    constexpr int REC = HD + ATTF_STRIDE_PAD, TH = HD / 4, NR = 8;
    const int idx = blockIdx.x * (256 / TH) + threadIdx.x / TH, d0 = threadIdx.x % TH * 4;
    if (idx >= g.rows * hq) return;
    const int row = idx / hq, head = idx % hq;
    int row0 = 0, parts = g.parts[0], record = g.record[0];
#pragma unroll
    for (int i = 1; i < VF_MAX_BATCH; ++i)
        if (row >= g.row0[i]) { row0 = g.row0[i]; parts = g.parts[i]; record = g.record[i]; }
    const int last_key = place[row].last_key;
    const float *p = part + ((size_t)(record + (row - row0) * parts) * hq + head) * REC;
    float M = -1e30f, L = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    int used = parts;
    for (int i0 = 0; i0 < used; i0 += NR) {
        float2 ml[NR];
        floatx4 v[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const float *r = p + (size_t)min(i0 + i, parts - 1) * hq * REC;
            ml[i] = *reinterpret_cast<const float2 *>(r);
            v[i] = *reinterpret_cast<const floatx4 *>(r + ATTF_STRIDE_PAD + d0);
        }
        used = min(parts, last_key / g.part_keys + 1);   // parts with keys of this row: the records of others hold anything
        float m = M;
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (i0 + i < used) m = fmaxf(m, ml[i].x);
        const float keep = exp2f(M - m);
        L *= keep;
        acc *= keep;
        M = m;
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (i0 + i < used) {
                const float add = exp2f(ml[i].x - m);
                L += ml[i].y * add;
                acc += v[i] * add;
            }
    }
    const float inv = 1.0f / L;
    *reinterpret_cast<u32x2 *>(o + xfrag_index(row, head * HD + d0, ncb)) =
        pack4_bf16(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
}

template <int HD>
int launch_items(const vf_model *m, const Batch &b, const ItemsGrid &grid, int layer, int workgroups, hipStream_t st) {
    const vf_config &c = m->cfg;
    const int ncb = (b.total_rows + 15) >> 4, lds = ITEMS_STAGES * (HD / 4) * 1024;
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)HD);
    hipLaunchKernelGGL(attn_items_kernel<HD>, dim3(workgroups), dim3(ITEMS_WAVES * 64), lds, st, b, grid, layer, (const bf16_t *)m->q,
                       (bf16_t *)m->o, c.n_q_heads, c.n_kv_heads, ncb, scale_log2e, m->attn_part);
    VF_LAUNCH_CHECK("attn_items");
    if (grid.merge) {
        constexpr int PER = 256 / (HD / 4);
        ItemsMerge g;
        g.rows = b.total_rows;
        g.part_keys = grid.part_pages * VF_TILE;
        for (int i = 0; i < VF_MAX_BATCH; ++i) {
            const bool is = i < b.n_seqs;
            g.row0[i] = is ? b.s[i].row0 : 0x7fffffff;
            g.parts[i] = is ? items_parts(b.s[i], grid.part_pages) : 1;
            g.record[i] = is ? grid.record[i] : 0;
        }
        hipLaunchKernelGGL(attn_items_merge_kernel<HD>, dim3((b.total_rows * c.n_q_heads + PER - 1) / PER), dim3(256), 0, st, g,
                           m->row_place, m->attn_part, (bf16_t *)m->o, c.n_q_heads, ncb);
        VF_LAUNCH_CHECK("attn_items_merge");
    }
    return VF_OK;
}

}  // namespace

// Which kernel, and how many pages make a part: once a call, the same for every layer.  Both kernels are modelled (us a
// layer; what is the same for both left out):
//   here:      what a page of a part costs while a compute unit has one workgroup, or two; with more workgroups than the chip
//              holds (512) their mean for each full round of the chip, and for the rest (of up to 256 workgroups, or more) a
//              round of theirs; a merge is a launch, and reads eight parts at a time and the records
//   attn_rows: its wavefronts' chain of tiles, or where that is longer the chip's share of all tiles (16 items x 32 keys) and
//              workgroups; a merge, records, and keys and values (its blocks of 16 items read them on every die)
// The constants are fits to whole layers of 3610 calls of eleven models (chunks of 49 to 1056 rows over up to 7600 keys, batches of
// 2 to 32 sequences) with attn_rows and every size of a part (profiles/attention_plan_timings.txt): the choice costs a
// layer 0.4 % on average against the best of them.  Without the launch of a merge, and with constants fitted to few
// calls, it was 1.3 %: few rows over long contexts came here for a merge more (64 rows over 2048 keys at 0.5B 42.3 us a
// layer, attn_rows 39.6), many over longer ones ran in parts of uneven rounds (1024 over 7600 at 1.5B 289 where parts of 28
// pages take 257).
struct AttnCost {
    float page1, page2, mean2, round, last, rest1, rest2, rest_mean2, merge, merge8, record_mb;                    // here
    float rows, chain, tile, workgroup, rows_merge, rows_record_mb, rows_kv_mb;                                    // attn_rows
};
constexpr AttnCost COST_64 = {0.68f, 0.50f, 0.49f, 1.07f, 0.07f, 0.26f, 0.40f, 0.64f, 5.13f, 1.03f, 0.21f,
                              -1.38f, 0.65f, 0.24e-3f, 4.2e-3f, 3.64f, 1.36f, 0.38f};
constexpr AttnCost COST_128 = {1.08f, 0.94f, 0.66f, 1.90f, 0.22f, 0.89f, 1.07f, 0.06f, 4.55f, 1.02f, 0.34f,
                               -2.44f, 1.09f, 0.58e-3f, 11.7e-3f, 4.02f, 0.92f, 0.37f};

static void plan_items(const vf_model *m, const Batch &b, AttnPlan &best) {
    best.workgroups = 0;
    const vf_config &c = m->cfg;
    const int group = c.n_q_heads / c.n_kv_heads;
    const AttnCost &t = c.head_dim == 128 ? COST_128 : COST_64;
    float seen_keys = 0.f, group_pages = 0.f, block_tiles = 0.f;
    int max_keys = 0, blocks = 0;
    for (int i = 0; i < b.n_seqs; ++i) {
        if ((uintptr_t)b.s[i].kv & 15) return;   // the direct loads move 16 bytes a lane
        const int items = b.s[i].nrows * group, item_blocks = (items + 15) / 16 * c.n_kv_heads;
        const float seen = b.s[i].len_ub + 0.5f * b.s[i].nrows;   // keys an item sees on average
        group_pages += (float)((items + ITEMS_GROUP - 1) / ITEMS_GROUP) * c.n_kv_heads * (seen / VF_TILE + 1.f);
        block_tiles += item_blocks * (seen / ATT_TILE + 0.5f);
        blocks += item_blocks;
        seen_keys += b.s[i].len_ub + b.s[i].nrows;
        max_keys = max(max_keys, b.s[i].len_ub + b.s[i].nrows);
    }
    const size_t record_floats = (size_t)c.n_q_heads * (c.head_dim + ATTF_STRIDE_PAD), room = m->attn_part_floats / record_floats;
    const float record_mb = 4e-6f * record_floats;
    const int rows_parts = vf_attention_rows_parts(m, b), tiles = (max_keys + ATT_TILE - 1) / ATT_TILE;
    float best_cost = t.rows + std::max(t.chain * tiles / (8 * rows_parts), t.tile * block_tiles + t.workgroup * blocks * rows_parts) +
                      t.rows_kv_mb * 4e-6f * c.n_kv_heads * c.head_dim * seen_keys;
    if (rows_parts > 1) best_cost += t.rows_merge + t.rows_record_mb * record_mb * b.total_rows * rows_parts;
    const int max_pages = (max_keys + VF_TILE - 1) / VF_TILE;
    ItemsGrid grid;
    // sizes of a part: every one up to 14, then an eighth to a quarter apart, and no parts
    for (grid.part_pages = 3;; grid.part_pages += grid.part_pages < 14 ? 1 : grid.part_pages < 32 ? 2 + grid.part_pages / 20 * 2 : grid.part_pages / 4) {
        int records = 0, workgroups = 0, parts_max = 1;
        grid.part_pages = min(grid.part_pages, max_pages);
        for (int i = 0; i < VF_MAX_BATCH; ++i) {
            grid.first[i] = i < b.n_seqs ? workgroups : 0x7fffffff;
            grid.record[i] = records;
            if (i >= b.n_seqs) continue;
            const int parts = items_parts(b.s[i], grid.part_pages);
            workgroups += (b.s[i].nrows * group + ITEMS_GROUP - 1) / ITEMS_GROUP * c.n_kv_heads * parts;
            records += b.s[i].nrows * parts;
            parts_max = max(parts_max, parts);
        }
        grid.merge = parts_max > 1;
        const float pages = grid.part_pages, mean = std::min(pages, group_pages / workgroups);   // (the unqualified one is int here)
        const int rest = workgroups % 512;
        float cost = workgroups <= 256   ? t.page1 * pages
                     : workgroups <= 512 ? t.page2 * pages + t.mean2 * mean
                                         : t.round * mean * (workgroups / 512) + t.last * pages +
                                               (rest == 0 ? 0.f : rest <= 256 ? t.rest1 * pages : t.rest2 * pages + t.rest_mean2 * mean);
        if (grid.merge) cost += t.merge + t.merge8 * ((parts_max - 1) / 8) + t.record_mb * record_mb * records;
        if (cost < best_cost && (!grid.merge || (size_t)records <= room)) {
            best_cost = cost;
            best.grid = grid;
            best.workgroups = workgroups;
        }
        if (grid.part_pages == max_pages) break;
    }
}

int vf_attention_items_plan(const vf_model *m, const Batch &b, int *merge) {
    AttnPlan plan;
    plan_items(m, b, plan);
    if (!plan.workgroups) return 0;
    *merge = plan.grid.merge;
    return plan.grid.part_pages;
}

void vf_attention_plan(const vf_model *m, const Batch &b, AttnPlan *plan) { plan_items(m, b, *plan); }

int vf_launch_attention_items(const vf_model *m, const Batch &b, const AttnPlan &plan, int layer, hipStream_t st) {
    return m->cfg.head_dim == 128 ? launch_items<128>(m, b, plan.grid, layer, plan.workgroups, st)
                                  : launch_items<64>(m, b, plan.grid, layer, plan.workgroups, st);
}
