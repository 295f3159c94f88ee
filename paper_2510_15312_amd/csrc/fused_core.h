// Device code shared by the persistent kernels (fused.hip, fused_direct.hip): grid barrier, row table, epilogues, sums,
// the exchange of partial tiles, the attention phase, and the memory protocol between workgroups (fused.hip).
#pragma once

#include "fast_common.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int FW = 8;            // wavefronts per workgroup
constexpr int FT = FW * 64;      // threads per workgroup
constexpr int FROWS = 48;        // most rows of a call
constexpr int MAX_DOWN_SPLITS = 9;   // K splits of the down projection
#ifndef BAR_COUNTERS
#define BAR_COUNTERS 64           // counters a barrier's arrivals are spread over
#endif
// words of the barrier block behind the counters, in memory lines of their own (from word 8192 on: phase timelines)
constexpr int BAR_START = 7936, BAR_FAIL = 8000, BAR_WORDS = 16384;
static_assert(BAR_COUNTERS * 64 <= BAR_START, "counters end below");
constexpr int LDS_BYTES = 152 * 1024;  // dynamic LDS of the one workgroup a CU holds (160 KB less the static part)
constexpr long long SPIN_LIMIT = 4000000;  // polls before a barrier gives up (seconds, not microseconds)

#ifndef FUSED_MAXP
#define FUSED_MAXP 6              // most key parts per attention block (verify step of 1.5B, 17 rows, 2048 keys: 9 parts 1135 us, 6 1126, 5 1143,
                                  // 4 1157; the 0.5B shape at 1024 keys takes five: 4 577 for 582; with parts merged by the last of them every setting gave
                                  // the same mean logit error at the full 1.5B size, 1.3e-2, but with 4 and 5 parts one row of 136 landed at
                                  // 2.12e-2 and 2.005e-2, past the stated 2e-2)
#endif
// One workgroup of 8 wavefronts per CU: two wavefronts per SIMD, so each may use up to 256 vector
// registers (weight ring + staging loads in flight) without spilling.
#ifndef FUSED_G
#define FUSED_G 256
#endif

// Pointers that reach the kernel through memory lose their address space; loads through them would
// be generic (flat) loads, which the compiler orders against every other load in flight.
typedef const floatx4 __attribute__((address_space(1))) *global_f4_ptr;
__device__ inline floatx4 load_global_f4(const float *p) { return *(global_f4_ptr)(p); }
typedef const u32x4 __attribute__((address_space(1))) *global_w_ptr;

// Loads from the single-assignment buffers (one version per phase and layer, written once per launch
// before they are read): no cache can hold an older copy of such a line, so an ordinary load will do.
__device__ __forceinline__ floatx4 ssa_load_f4(const float *p) { return *reinterpret_cast<const floatx4 *>(p); }
__device__ __forceinline__ u32x4 ssa_load_16(const void *p) { return *reinterpret_cast<const u32x4 *>(p); }
__device__ __forceinline__ float ssa_load_f1(const float *p) { return *p; }

struct FusedLayer {
    const u32x4 *wqkv, *wo, *wgu, *wd;
    const float *attn_norm, *ffn_norm, *bqkv;
};

struct FusedArgs {
    FusedLayer layer0;              // the first layer's parameters; the others follow at equal distances
    unsigned long long layer_bytes;
    const bf16_t *embed;
    const u32x4 *lm_head;
    const float *final_norm, *cosv, *sinv;
    const int32_t *tree_depth;      // tree-structured drafts (else NULL): depth and ancestor mask of every row
    const tree_mask_t *tree_anc;
    const int32_t *tokens;
    int frows;        // rows of the buffers below: the model's max_rows in blocks of 16, at most FROWS
    float *hv;        // residual stream, [2L+1][frows][d]
    float *ssv;       // sums of squares of its rows per 16 columns, [2L+1][d/16][64]
    bf16_t *qv, *ov, *av;  // per layer: q [frows][Hq*hd], attention output, SwiGLU product [frows][F]
    bf16_t *xv;       // fused_direct.hip: normalised rows, [2L][frows][d]
    float *h_last;    // fused_direct.hip: the residual stream behind the last layer
    float *xch;       // partial tiles of the down projection's K splits, then of the attention's key parts; marks between uses
    unsigned *bar, *fail, *bar_start;   // barrier counters, whether one gave up, the counters' value at launch start
    float *logits;
    int n_layers, d, F, hq, hkv, hd, vocab, m, has_bias;
    int att_blocks, att_parts;  // (query block, kv head, sequence) blocks of the call; key parts per block
    // First attention work item of every workgroup (-1: none).  Workgroup w runs on compute die w % 8;
    // the map puts the query blocks that read the same keys (same sequence, kv head and key part) on one
    // die, so that its L2 serves all but the first of those reads.
    short att_first[FUSED_G];
    float inv_d, eps, scale_log2e;
    int ks_down;              // K splits of the down projection
    int down_ub;              // weight blocks of a down projection item
    int gu_light;            // gate/up: the first gu_light workgroups (busy in the O projection) take one unit each (0: even shares)
    int lds_total;    // dynamic LDS bytes of this launch
};

// Counting barrier, split into arrive and wait.  The workgroups are spread over BAR_COUNTERS counters
// (each in a memory channel of its own, so that the increments of a barrier are not all serialised
// at one address); an arrival is one increment that returns nothing, and a barrier is complete when
// every counter has grown by the number of workgroups mapped to it.  Counters only ever grow:
// barrier number e of a launch waits for the counters' value at launch start + e * (G / BAR_COUNTERS).
// That start value is in device memory, not an argument: every workgroup reads it before its first arrival, and the
// launch leaves it advanced (barrier_advance), so that a launch replayed from a graph finds its own.
// Lanes 0..BAR_COUNTERS-1 of the first wavefront poll one counter each.
struct GridBar {
    unsigned *mem, *fail;
    unsigned target, per;  // target: at first the counters' value at launch start; per: workgroups per counter
    bool dead;
#ifdef FUSED_ARRIVALS
    unsigned long long *stamps;  // [barrier][2][workgroup]: clock at the arrival and at the end of the wait
    int n_arr, n_wait;
#endif
    __device__ __forceinline__ void arrive() {
        stores_done();  // this wavefront's write-through stores have reached memory
        __syncthreads();
#ifdef FUSED_ARRIVALS
        if (threadIdx.x == 0) stamps[((size_t)n_arr * 2) * gridDim.x + blockIdx.x] = wall_clock64();
        ++n_arr;
#endif
        target += per;
        if (threadIdx.x == 0)
            __hip_atomic_fetch_add(mem + (blockIdx.x % BAR_COUNTERS) * 64, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void wait() {
        if (threadIdx.x < 64 && !dead) {
            const int lane = threadIdx.x;
            const unsigned *mine = mem + min(lane, BAR_COUNTERS - 1) * 64;
            long long spins = 0;
            for (;;) {
                const bool done = (int)(__hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) >= 0;
                if (__all(done)) break;
                __builtin_amdgcn_s_sleep(1);
                ++spins;
                if (spins > SPIN_LIMIT ||
                    ((spins & 1023) == 0 && __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                    __hip_atomic_store(fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    dead = true;  // give up for good: the launch drains without waiting again
                    break;
                }
            }
        }
        lds_sync();
#ifdef FUSED_ARRIVALS
        if (threadIdx.x == 0) stamps[((size_t)n_wait * 2 + 1) * gridDim.x + blockIdx.x] = wall_clock64();
        ++n_wait;
#endif
    }
};

// The counters' value at launch start: requested first thing in a kernel, used when its first phase is done.
__device__ __forceinline__ unsigned barrier_start(const unsigned *start) { return __hip_atomic_load(start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Debug build FUSED_ARRIVALS: the stamps' place is behind the barrier block, room for every barrier of either kernel and
// the end of the output head.
__device__ __forceinline__ GridBar grid_bar(unsigned *mem, unsigned *fail, unsigned start) {
    return GridBar{mem, fail, start, gridDim.x / BAR_COUNTERS, false,
#ifdef FUSED_ARRIVALS
                   reinterpret_cast<unsigned long long *>(mem + BAR_WORDS), 0, 0
#endif
    };
}
// For the next launch: what the counters have grown to when all arrivals of this one are in.  Anywhere behind this
// workgroup's first wait, when every workgroup has read the old value, and its last arrival.
__device__ __forceinline__ void barrier_advance(unsigned *start, const GridBar &bar) {
    if (blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(start, bar.target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Optional phase timeline of one workgroup (build with -DFUSED_TRACE=<workgroup>): thread 0 stamps the
// constant-rate clock at the marked points into the second half of the barrier block.
#ifdef FUSED_TRACE
struct Trace {
    unsigned long long *buf;
    int n;
    __device__ __forceinline__ void mark(int id) {
        if (blockIdx.x == FUSED_TRACE && threadIdx.x == 0 && n < 2040) {
            buf[2 * n] = wall_clock64();
            buf[2 * n + 1] = ((unsigned long long)clock64() << 8) | (unsigned long long)id;  // shader-clock count
            ++n;
        }
    }
};
#define TRACE(id) trace.mark(id)
#define TRACE_ARG , Trace &trace
#define TRACE_PASS , trace
#else
#define TRACE(id)
#define TRACE_ARG
#define TRACE_PASS
#endif

// Where a row of the call goes in the KV cache and which rotary angle it takes; the same in every
// layer of a launch (sequence lengths do not change while it runs), so it is worked out once.
struct RowMeta {
    bf16_t *kv;      // the sequence's KV pool
    int n_pages;     // pages in that pool
    int page, tin;   // page and row inside the page of the row's cache slot
    int pos;         // position whose rotary angle the row takes
    int live;        // 0: the slot lies outside the sequence's capacity, nothing is written
};
struct FusedShared {
    float rs_tmp[FW][64];
    RowMeta rows[FROWS];
};

// (sequence, kv head, query block, key part) of attention work item i
struct AttItem { int seq, kvh, qb, part, blk; };
__device__ __forceinline__ AttItem att_item(const FusedArgs &a, const Batch &b, int i) {
    const int group = a.hq / a.hkv;
    AttItem it;
    it.part = i / a.att_blocks;
    it.blk = i % a.att_blocks;
    int blk = it.blk, seq = 0;
    while (seq + 1 < b.n_seqs) {
        const int nb_seq = a.hkv * ((b.s[seq].nrows * group + 15) >> 4);
        if (blk < nb_seq) break;
        blk -= nb_seq;
        ++seq;
    }
    const int nqb = (b.s[seq].nrows * group + 15) >> 4;
    it.seq = seq;
    it.kvh = blk / nqb;
    it.qb = blk % nqb;
    return it;
}

// Everything that is the same for a whole launch: the row table, and the length of the sequence of this workgroup's first
// attention item (lengths are constant during a launch).
__device__ __forceinline__ int launch_tables(const FusedArgs &a, const Batch &b, FusedShared &sh) {
    int len0 = 0;
    if (a.att_first[blockIdx.x] >= 0) len0 = b.s[att_item(a, b, a.att_first[blockIdx.x]).seq].state[0];
    if ((int)threadIdx.x < FROWS) {
        const int row = min((int)threadIdx.x, a.m - 1);
        const SeqDesc &s = b.s[find_seq(b, row)];
        const int len = s.state[0], slot = len + (row - s.row0);
        RowMeta rm;
        rm.kv = reinterpret_cast<bf16_t *>(s.kv);
        rm.n_pages = s.n_pages;
        rm.live = slot >= 0 && slot < s.capacity;
        rm.page = rm.live ? kv_page(s, slot) : 0;
        rm.tin = rm.live ? slot % VF_TILE : 0;
        rm.pos = rm.live ? (a.tree_depth ? len + a.tree_depth[row] : slot) : 0;
        sh.rows[threadIdx.x] = rm;
    }
    return len0;
}
// Kernel arguments and a multiple of the layer's number: addresses that the scalar unit forms, no load.
__device__ __forceinline__ FusedLayer layer_params(const FusedArgs &a, int l) {
    FusedLayer lp = a.layer0;
    const size_t lo = (size_t)l * a.layer_bytes;
    auto at_layer = [&](auto &p) { p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(reinterpret_cast<uintptr_t>(p) + lo); };
    at_layer(lp.wqkv); at_layer(lp.wo); at_layer(lp.wgu); at_layer(lp.wd);
    at_layer(lp.attn_norm); at_layer(lp.ffn_norm); at_layer(lp.bqkv);
    return lp;
}

// ---- embedding: row r by workgroup r ---------------------------------------------------------------
__device__ __forceinline__ void embed_phase(const FusedArgs &a, const Batch &b) {
    const int d = a.d;
    for (int row = blockIdx.x; row < a.m; row += gridDim.x) {
        int tok = a.tokens[row];
        if (tok == VF_PENDING) tok = b.s[find_seq(b, row)].state[1];
        if (tok < 0 || tok >= a.vocab) tok = 0;
        for (int k0 = 0; k0 < d; k0 += FT) {
            const int k = k0 + threadIdx.x;
            float v = 0.f;
            if (k < d) {
                v = (float)a.embed[wfrag_index(tok, k, d)];
                st_f32<true>(a.hv + (size_t)row * d + k, v);
            }
            float sq = v * v;
            sq += __shfl_xor(sq, 8, 64);
            sq += __shfl_xor(sq, 4, 64);
            sq += __shfl_xor(sq, 2, 64);
            sq += __shfl_xor(sq, 1, 64);
            if (k < d && (threadIdx.x & 15) == 0) st_f32<true>(a.ssv + (k >> 4) * 64 + row, sq);
        }
    }
}

// Epilogues of the persistent kernel.  What they read from memory is requested ahead of the products, for a phase's
// first item before the grid barrier, so that no round trip is left between the last product and the stores.
//   QKV: bias, rotary embedding, q to its buffer, K and V rows into the cache (row table in LDS)
//   residual: h = h_in + y, and the tile's sums of squares for the next RMSNorm
struct EpiPre { floatx4 v, bias; };
// nb: the same for all lanes
template <int HD>
__device__ __forceinline__ EpiPre epi_qkv_ask(const FastGemm &g, const FusedShared &sh, int row, int nb, int lane) {
    EpiPre p;
    p.bias = floatx4{0.f, 0.f, 0.f, 0.f};
    if (g.bias) p.bias = load_global_f4(g.bias + nb * 16 + (lane >> 4) * 4);
    const unsigned at = sh.rows[row].pos * (HD / 2) + (((nb * 16) % HD + (lane >> 4) * 4) >> 1);   // past the K heads: loaded, not used
    const float2 c = *reinterpret_cast<const float2 *>(g.cosv + at), sn = *reinterpret_cast<const float2 *>(g.sinv + at);
    p.v = floatx4{c.x, sn.x, c.y, sn.y};
    return p;
}
__device__ __forceinline__ void epi_resid_pre(const FastGemm &g, int row, bool live, int nb, int lane, floatx4 v, const EpiPre &pre) {
    const int n0 = nb * 16 + (lane >> 4) * 4;
    floatx4 hv = {0.f, 0.f, 0.f, 0.f};
    if (live) {
        hv = pre.v + v;
        st_f32x4<true>(g.h + (size_t)row * g.N + n0, hv);
    }
    float ssq = hv[0] * hv[0] + hv[1] * hv[1] + hv[2] * hv[2] + hv[3] * hv[3];
    ssq += __shfl_xor(ssq, 16, 64);
    ssq += __shfl_xor(ssq, 32, 64);
    if (live && (lane >> 4) == 0) st_f32<true>(g.ss_out + nb * 64 + row, ssq);
}
template <int HD>
__device__ __forceinline__ void epi_qkv_store(const FastGemm &g, const FusedShared &sh, int row, int nb, int lane, floatx4 v, const EpiPre &pre) {
    const int head = nb * 16 / HD, p0 = nb * 16 % HD + (lane >> 4) * 4;   // the head is the same for all lanes
    v += pre.bias;
    const RowMeta rm = sh.rows[row];
    if (!rm.live) return;
    if (head < g.hq + g.hkv) {
        const int i0 = p0 >> 1;  // packed columns 2i, 2i+1 are elements i and i + HD/2
        const float c0 = pre.v[0], s0 = pre.v[1], c1 = pre.v[2], s1 = pre.v[3];
        const float a0 = v[0] * c0 - v[1] * s0, b0 = v[1] * c0 + v[0] * s0;
        const float a1 = v[2] * c1 - v[3] * s1, b1 = v[3] * c1 + v[2] * s1;
        // i0 is even: elements i0, i0 + 1 are neighbours in either layout, 4-byte aligned
        bf16_t *d0, *d1;
        if (head < g.hq) {
            d0 = g.q + ((size_t)row * g.hq + head) * HD + i0;
            d1 = d0 + HD / 2;
        } else {
            d0 = rm.kv + kv_k_index(g.layer, rm.n_pages, rm.page, g.hkv, head - g.hq, rm.tin, i0, HD);
            d1 = rm.kv + kv_k_index(g.layer, rm.n_pages, rm.page, g.hkv, head - g.hq, rm.tin, i0 + HD / 2, HD);
        }
        st_u32<true>(d0, pack2_bf16(a0, a1));
        st_u32<true>(d1, pack2_bf16(b0, b1));
    } else {
        bf16_t *d = rm.kv + kv_v_index(g.layer, rm.n_pages, rm.page, g.hkv, head - g.hq - g.hkv, rm.tin, p0, HD);
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // four dimensions of a key: 16 bytes apart
            const bf16_t x = (bf16_t)v[i];
            st_u16<true>(d + i * 8, __builtin_bit_cast(unsigned short, x));
        }
    }
}

// SwiGLU product in MFMA operand order (fragment (K block, row block), see xfrag_index).  v0, v1: tiles of the weight
// blocks nb (even) and nb + 1: a lane holds ffn columns f, f + 1 and f + 8, f + 9 of its row.
__device__ __forceinline__ void epi_swiglu_frag(const FastGemm &g, int row, int nb, int lane, floatx4 v0, floatx4 v1, int ncb) {
    bf16_t *out = g.a_out + xfrag_index(row, nb * 8, ncb) + (lane >> 4) * 2;
    auto act = [](float gt, float up) { return gt / (1.0f + expf(-gt)) * up; };
    st_u32<true>(out, pack2_bf16(act(v0[0], v0[1]), act(v0[2], v0[3])));
    st_u32<true>(out + 128, pack2_bf16(act(v1[0], v1[1]), act(v1[2], v1[3])));
}

// ---- sums over wavefronts and K splits -------------------------------------------------------------------
// red: partial tiles [tile][wavefront][lane].  Pairs (w, w + 4), then the four pairs in order.
__device__ __forceinline__ floatx4 sum_waves(const floatx4 *red, int tile, int lane) {
    floatx4 p[FW], v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < FW; ++i) p[i] = red[(tile * FW + i) * 64 + lane];
    asm volatile("" ::: "memory");   // all reads are issued before the first sum
#pragma unroll
    for (int i = 0; i < FW / 2; ++i) v += p[i] + p[i + FW / 2];
    return v;
}
// ---- exchange of partial tiles ------------------------------------------------------------------------------
// K splits of a down projection tile, and key parts of an attention block, meet through memory that holds a mark
// (all bits set, which no sent value has) wherever nothing has been sent.  Each tile has an owner among the
// workgroups that share it; the others send theirs and go on, the owner reads until no mark is left, puts the marks
// back and goes on with the sum.  Against a counter that the last to arrive reads (store, wait for the store,
// increment with its round trip, read): the wait and the increment are gone from the chain, and the owners of
// different tiles work at the same time.
// Everyone who sends is resident and sends without waiting for anybody, so the wait ends; it is bounded like the
// grid barrier's all the same.  Attention and down projection together: 1.5B, 17 rows 1252 -> 1154 us a pass, 0.5B, 9
// rows 714 -> 674.
constexpr unsigned XCH_MARK = 0xffffffffu;
__device__ __forceinline__ void xch_send(float *slot, floatx4 v) {
    u32x4 r = __builtin_bit_cast(u32x4, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = r[i] == XCH_MARK ? 0x7fc00000u : r[i];   // a NaN like any other
    st_f32x4<true>(slot, __builtin_bit_cast(floatx4, r));
}
// What parts 0 .. n - 1 (n >= 2) but `self` have sent: NV values a lane and part, value k of part i `at` + i * stride +
// k * 1024 bytes into the exchange.  t[i] of part `self` and of parts past the last is undefined.  A round of the wait
// is one round trip to memory and what its code costs: 16-byte loads past the caches (two of 8 bytes each before),
// and a maximum over the words instead of a comparison of each.
template <int MAXN, int NV>
__device__ __forceinline__ void xch_receive(floatx4 (&t)[MAXN][NV], float *xch, unsigned at, unsigned stride, int n, int self, int lane,
                                            unsigned *fail) {
    constexpr int AGENT = 16;   // cache policy of an agent-scope load
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(xch, 0, 0x7fffffff, 0x00027000);
    const int other = self == 0 ? 1 : 0;
    for (int spins = 0;;) {
        asm volatile("" ::: "memory");   // read again in every round
#pragma unroll
        for (int i = 0; i < MAXN; ++i)
#pragma unroll
            for (int k = 0; k < NV; ++k)
                t[i][k] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          rsrc, lane * 16, at + (i < n && i != self ? i : other) * stride + k * 1024, AGENT));
        unsigned most = 0;
#pragma unroll
        for (int i = 0; i < MAXN; ++i)
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const u32x4 r = __builtin_bit_cast(u32x4, t[i][k]);
                most = max(max(most, r[0]), max(r[1], max(r[2], r[3])));
            }
        if (!__any(most == XCH_MARK)) break;
        ++spins;
        if (spins > SPIN_LIMIT || ((spins & 1023) == 0 && __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
            __hip_atomic_store(fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
    }
}
// Puts the marks back where this workgroup has received: tiles self, self + n, ... of `tiles`, NV values a lane.  Called
// behind the arrival at the grid barrier, when all wavefronts are done with the values; the next arrival waits for
// these stores, the next use is a phase or more behind that.  Not by the wavefront that polls the barrier: its polls
// would wait for the stores (1.5B, 17 rows: 1178 us a pass; marks put back at the end of the phase 1162; so 1154).
struct XchUsed { unsigned at, stride; int n, self, tiles; };   // at: of tile 0; n = 0: nothing received
template <int NV>
__device__ __forceinline__ void xch_clear(float *xch, const XchUsed &u) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (u.n < 2 || wave < 2) return;
    const floatx4 mark = __builtin_bit_cast(floatx4, u32x4{XCH_MARK, XCH_MARK, XCH_MARK, XCH_MARK});
    for (int t = u.self + (FW - 1 - wave) * u.n; t < u.tiles; t += (FW - 2) * u.n) {
        float *p = xch + (u.at + t * NV * 1024) / 4 + (threadIdx.x & 63) * 4;
        for (int i = 0; i < u.n; ++i)
            if (i != u.self)
#pragma unroll
                for (int k = 0; k < NV; ++k) st_f32x4<true>(p + (i * u.stride + k * 1024) / 4, mark);
    }
}
// Sum of a tile over its K splits, in split order.
template <int MAXN>
__device__ __forceinline__ floatx4 xch_sum(floatx4 v, float *xch, unsigned at, unsigned stride, int n, int self, int lane, unsigned *fail) {
    floatx4 t[MAXN][1], sum = {0.f, 0.f, 0.f, 0.f};
    xch_receive<MAXN, 1>(t, xch, at, stride, n, self, lane, fail);
#pragma unroll
    for (int i = 0; i < MAXN; ++i)
        if (i < n) sum += i == self ? v : t[i][0];
    return sum;
}

// ---- attention phase -----------------------------------------------------------------------------------
// Work item = (block of 16 query items, kv head, sequence, part of the keys); a query item is a
// (row, head of the group) pair.  The eight wavefronts of a workgroup take the 32-key tiles of the
// part in turn; K and V^T fragments go from the cache straight into registers in MFMA operand
// order (no LDS staging: every fragment is used by exactly one wavefront).  Scores
// S^T[key, item] = K Q^T leave the MFMA with eight keys per lane once the K rows are fed in the
// order 8*(rho >> 2) + (rho & 3) (+ 4 for the second 16-key block): that is the B-operand layout
// of O^T[d, item] += V^T[d, key] P[key, item], and the matching V^T fragment is one 16-byte load.
// Wavefront results (running max, sum, O^T) are merged through LDS; with several parts the
// parts exchange their d-blocks (above), one owner each.  No second grid-wide phase is needed
// for the merge.
constexpr int FKT = ATT_TILE;  // keys per tile

// len0: length of the sequence of this workgroup's first item, read once per launch (lengths do
// not change during a launch).
template <int HD>
__device__ __forceinline__ XchUsed attn_phase(const FusedArgs &a, const Batch &b, int layer, const bf16_t *q, bf16_t *o, int ncb,
                                  int len0, GridBar &bar, unsigned char *smem, FusedShared &sh TRACE_ARG) {
    XchUsed used{0, 0, 0, 0, 0};
    constexpr int KD = HD / 32, DB = HD / 16, MAXP = FUSED_MAXP;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    // the wavefront's number as a scalar: which tile it takes, and whether that tile holds keys of
    // this launch, are then decided by scalar branches
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g4 = lane >> 4, l15 = lane & 15;
    const int G = gridDim.x, hq = a.hq, hkv = a.hkv, group = hq / hkv, P = a.att_parts;
    floatx4 *o_s = reinterpret_cast<floatx4 *>(smem);                      // [wave][db][lane]
    float *ml_s = reinterpret_cast<float *>(smem + FW * DB * 64 * 16);    // [wave][2][16]
    const int n_work = a.att_blocks * P;
    AttTile<HD> tile;
    auto tile_range = [&](const SeqDesc &s, const AttItem &it, int len, int &t_begin, int &t_end, int &kmax) {
        kmax = min(len + s.nrows, s.capacity);  // keys 0..kmax-1 exist
        const int blk_last = min(kmax - 1, len + min(s.nrows - 1, (it.qb * 16 + 15) / group));
        const int tiles = blk_last / FKT + 1, tpp = (tiles + P - 1) / P;
        t_begin = it.part * tpp;
        t_end = min(tiles, t_begin + tpp);
    };
    // keys below the sequence length were written by earlier calls: a first tile made of them is
    // loaded before the barrier wait
    bool preloaded = false;
    const int i_first = a.att_first[blockIdx.x];
    if (i_first >= 0) {
        const AttItem it = att_item(a, b, i_first);
        int t_begin, t_end, kmax;
        tile_range(b.s[it.seq], it, len0, t_begin, t_end, kmax);
        const int t = t_begin + wave;
        if (t < t_end && (t + 1) * FKT <= len0) {
            tile.load(b.s[it.seq], layer, hkv, it.kvh, t, false, lane);
            preloaded = true;
        }
    }
    TRACE(1);
    bar.wait();
    TRACE(2);
    // further items (more work than workgroups; then there is one part per block) follow in steps of G
    for (int i = i_first; i >= 0 && i < n_work; i += G) {
        const AttItem it = att_item(a, b, i);
        const SeqDesc &s = b.s[it.seq];
        const int kvh = it.kvh, part = it.part;
        const int n_items = s.nrows * group;
        const int len = i == i_first ? len0 : s.state[0];
        int t_begin, t_end, kmax;
        tile_range(s, it, len, t_begin, t_end, kmax);
        const int item = it.qb * 16 + l15;
        const bool valid = item < n_items;
        const int r = valid ? item / group : 0, head = kvh * group + (valid ? item % group : 0);
        const int row = s.row0 + r;
        const int last_key = valid ? len + r : -1;
        // a value every lane shares (kernel argument and the item's sequence length)
        const int own_base = a.tree_anc ? __builtin_amdgcn_readfirstlane(len) : ATT_NO_TREE;
        const tree_mask_t own_mask = a.tree_anc && valid ? a.tree_anc[row] : 0;

        bf16x8 qf[KD];
#pragma unroll
        for (int kd = 0; kd < KD; ++kd)
            qf[kd] = __builtin_bit_cast(bf16x8, ssa_load_16(q + ((size_t)row * hq + head) * HD + kd * 32 + g4 * 8));
        AttState<HD> st;
#pragma unroll
        for (int db = 0; db < DB; ++db) st.o[db] = floatx4{0.f, 0.f, 0.f, 0.f};
        st.m_run = -1e30f;
        st.l_run = 0.f;
        // The next tile's keys are requested when this one's have been multiplied, its values when these have: no
        // registers for a second tile (with whole tiles in two register sets 400 of them were spilled), and a round trip
        // a tile less than one tile after the other.
        int t = t_begin + wave;
        if (t < t_end && !preloaded) tile.load(s, layer, hkv, kvh, t, (t + 1) * FKT > len, lane);
        preloaded = false;
#pragma unroll 1
        for (; t + FW < t_end; t += FW) {
            const int n = t + FW, page = kv_page(s, n * FKT);
            const bool coh = (n + 1) * FKT > len;   // (a tile with keys past the last is the part's last: none here)
            att_tile_update<HD>(st, qf, tile, t * FKT, last_key, own_base, own_mask, (t + 1) * FKT <= len, a.scale_log2e, lane, [&] {
                if (coh) tile.template load_keys<true>(s, layer, hkv, kvh, n, page, lane);
                else tile.template load_keys<false>(s, layer, hkv, kvh, n, page, lane);
            });
            if (coh) tile.template load_values<true>(s, layer, hkv, kvh, n, page, lane);
            else tile.template load_values<false>(s, layer, hkv, kvh, n, page, lane);
        }
        if (t < t_end) {
            tile.mask_values(t * FKT, kmax, lane);
            att_tile_update<HD>(st, qf, tile, t * FKT, last_key, own_base, own_mask, (t + 1) * FKT <= len, a.scale_log2e, lane);
        }
        TRACE(20);
        // ---- merge of the eight wavefronts through LDS ----
        if (i != i_first) lds_sync();  // the previous item's merge has been read
#pragma unroll
        for (int db = 0; db < DB; ++db) o_s[(wave * DB + db) * 64 + lane] = st.o[db];
        if (g4 == 0) {
            ml_s[(wave * 2 + 0) * 16 + l15] = st.m_run;
            ml_s[(wave * 2 + 1) * 16 + l15] = st.l_run;
        }
        lds_sync();
        // thread (db = wave, lane) owns O^T[d = 16*db + 4*g4 + j][item l15]; HD = 64 leaves waves 4..7 idle
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        float M = -1e30f, L = 0.f;
        if (wave < DB) {
            // all LDS reads of the merge are issued together, ahead of the arithmetic
            float mw[FW], lw[FW];
            floatx4 ow[FW];
#pragma unroll
            for (int w = 0; w < FW; ++w) {
                mw[w] = ml_s[(w * 2) * 16 + l15];
                lw[w] = ml_s[(w * 2 + 1) * 16 + l15];
                ow[w] = o_s[(w * DB + wave) * 64 + lane];
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int w = 0; w < FW; ++w) M = fmaxf(M, mw[w]);
#pragma unroll
            for (int w = 0; w < FW; ++w) {
                const float wt = exp2f(mw[w] - M);
                L += lw[w] * wt;
                acc += ow[w] * wt;
            }
        }
        TRACE(21);
        if (P > 1) {
            // The parts of a block exchange their results: d-block db is put together by part db % P, whose wavefront
            // db has the other parts' O tiles and (max, sum) pairs sent to it.
            const unsigned at = (unsigned)(it.blk * P * DB + wave) * 2048, stride = DB * 2048;
            used = XchUsed{at - wave * 2048, stride, P, part, DB};
            if (wave < DB && wave % P != part) {
                float *slot = a.xch + (at + part * stride) / 4 + lane * 4;
                xch_send(slot, acc);
                xch_send(slot + 256, floatx4{M, L, 0.f, 0.f});
            } else if (wave < DB) {
                floatx4 t[MAXP][2];
                xch_receive<MAXP, 2>(t, a.xch, at, stride, P, part, lane, a.fail);
                TRACE(22);
                float Mg = M;
#pragma unroll
                for (int pp = 0; pp < MAXP; ++pp) Mg = pp < P && pp != part ? fmaxf(Mg, t[pp][1][0]) : Mg;
                float Lg = 0.f;
                floatx4 og = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int pp = 0; pp < MAXP; ++pp) {
                    if (pp < P) {
                        const float wt = exp2f((pp == part ? M : t[pp][1][0]) - Mg);
                        Lg += (pp == part ? L : t[pp][1][1]) * wt;
                        og += (pp == part ? acc : t[pp][0]) * wt;
                    }
                }
                if (valid) {
                    const float inv = 1.0f / Lg;
                    st_u32x2<true>(o + xfrag_index(row, head * HD + wave * 16 + g4 * 4, ncb),
                                   pack4_bf16(og[0] * inv, og[1] * inv, og[2] * inv, og[3] * inv));
                }
            }
        } else if (wave < DB && valid) {
            const float inv = 1.0f / L;
            st_u32x2<true>(o + xfrag_index(row, head * HD + wave * 16 + g4 * 4, ncb),
                           pack4_bf16(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv));
        }
    }
    return used;
}


// ---- host side, both kernels ---------------------------------------------------------------------------

// Rows the buffers of a launch are laid out for.
inline int fused_rows(const vf_config &c) { return std::min(FROWS, (c.max_rows + 15) / 16 * 16); }
inline bool fused_shape_ok(const vf_config &c) { return c.dtype == VF_BF16 && c.d_model % 64 == 0 && FUSED_G % BAR_COUNTERS == 0; }

// Everything but the splits, the output and the barrier's start.
inline void fused_args(const vf_model *m, const Batch &b, const int32_t *tokens, bool tree, FusedArgs &a) {
    const vf_config &c = m->cfg;
    const int G = FUSED_G;
    a.lds_total = LDS_BYTES;
    a.frows = fused_rows(c);
    a.xv = (bf16_t *)m->fz_x;
    int max_keys = 0;
    for (int i = 0; i < b.n_seqs; ++i) max_keys = std::max(max_keys, b.s[i].len_ub + b.s[i].nrows);
    // attention: blocks of 16 query items per (sequence, kv head); as many key parts per block as
    // fill the grid, but no more than give every wavefront of a part a tile of its own
    const int group = c.n_q_heads / c.n_kv_heads;
    int blocks = 0;
    for (int i = 0; i < b.n_seqs; ++i) blocks += c.n_kv_heads * ((b.s[i].nrows * group + 15) / 16);
    int parts = std::max(1, std::min(G / std::max(1, blocks), ((max_keys + FKT - 1) / FKT + FW - 1) / FW));
    parts = std::min(parts, FUSED_MAXP);
    if (blocks * parts > FUSED_G) parts = 1;  // the exchange has room for one item per workgroup
    const LayerPacked &l0 = m->layers[0];
    a.layer0 = FusedLayer{(const u32x4 *)l0.wqkv, (const u32x4 *)l0.wo, (const u32x4 *)l0.wgu, (const u32x4 *)l0.wd, l0.attn_norm, l0.ffn_norm, l0.bqkv};
    a.layer_bytes = c.n_layers > 1 ? (unsigned long long)((char *)m->layers[1].wqkv - (char *)l0.wqkv) : 0;
    a.embed = (const bf16_t *)m->embed;
    a.lm_head = (const u32x4 *)m->lm_head;
    a.final_norm = m->final_norm;
    a.cosv = m->rope_cos;
    a.sinv = m->rope_sin;
    a.tree_depth = tree ? m->tree_depth : nullptr;
    a.tree_anc = tree ? m->tree_anc : nullptr;
    a.tokens = tokens;
    a.hv = m->fz_h;
    a.ssv = m->fz_ss;
    a.qv = (bf16_t *)m->fz_q;
    a.ov = (bf16_t *)m->fz_o;
    a.av = (bf16_t *)m->fz_a;
    a.xch = m->fz_xch;
    a.bar = m->fz_bar;
    a.fail = m->fz_bar + BAR_FAIL;
    a.bar_start = m->fz_bar + BAR_START;
    a.n_layers = c.n_layers;
    a.d = c.d_model;
    a.F = c.d_ffn;
    a.hq = c.n_q_heads;
    a.hkv = c.n_kv_heads;
    a.hd = c.head_dim;
    a.vocab = c.vocab;
    a.m = b.total_rows;
    a.att_blocks = blocks;
    a.att_parts = parts;
    {
        // item = part * blocks + block, block = (sequence, kv head, query block) in that order
        const int n_work = blocks * parts;
        for (int w = 0; w < FUSED_G; ++w) a.att_first[w] = (short)(w < n_work && n_work > G ? w : -1);
        if (n_work <= G) {
            // from the top of the grid downwards: the QKV phase before it keeps the lowest workgroups busy
            // (one item each), and a workgroup that is idle there has worked out its attention item and
            // requested its first key tile by the time the others arrive
            int next[8], die = 0;
            for (int x = 0; x < 8; ++x) next[x] = G - 8 + x;
            int blk0 = 0;
            for (int sq = 0; sq < b.n_seqs; ++sq) {
                const int nqb = (b.s[sq].nrows * group + 15) / 16;
                for (int kvh = 0; kvh < c.n_kv_heads; ++kvh)
                    for (int p = 0; p < parts; ++p) {
                        for (int qb = 0; qb < nqb; ++qb) {
                            int x = die;
                            for (int tries = 0; tries < 8 && (next[x] >= G || next[x] < 0); ++tries) x = (x + 1) % 8;  // that die is full
                            a.att_first[next[x]] = (short)(p * blocks + blk0 + kvh * nqb + qb);
                            next[x] += -8;
                        }
                        die = (die + 1) % 8;
                    }
                blk0 += c.n_kv_heads * nqb;
            }
        }
    }
    a.has_bias = c.qkv_bias;
    a.inv_d = 1.0f / (float)c.d_model;
    a.eps = c.rms_eps;
    a.scale_log2e = 1.4426950408889634f / sqrtf((float)c.head_dim);
}

template <auto KERN> int fused_launch(const FusedArgs &a, const Batch &b, hipStream_t st) {
    static int max_wgs = -1;  // workgroups that can be resident at once
    const void *kern = reinterpret_cast<const void *>(KERN);
    if (max_wgs < 0) {
        VF_HIP(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES));
        int per_cu = 0, dev = 0;
        hipDeviceProp_t prop;
        VF_HIP(hipGetDevice(&dev));
        VF_HIP(hipGetDeviceProperties(&prop, dev));
        VF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, FT, LDS_BYTES));
        max_wgs = per_cu * prop.multiProcessorCount;
    }
    if (FUSED_G > max_wgs)
        return vf_fail(VF_ERR_UNSUPPORTED, "persistent kernel: %d workgroups wanted, %d can be resident", FUSED_G, max_wgs);
    hipLaunchKernelGGL(KERN, dim3(FUSED_G), dim3(FT), a.lds_total, st, a, b);
    VF_LAUNCH_CHECK("persistent kernel");
    return VF_OK;
}

}  // namespace
