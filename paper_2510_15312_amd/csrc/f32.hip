// The float32 decoder stack, any row count (prefill chunk, verify, tree verify; paper Sec. 3, 4.1,
// 4.3).  Per layer five kernels, on the float32 matrix instructions (16x16x4, exact float32 products,
// float32 sums):
//   QKV     : (h * gain) * Wqkv^T, row scale 1/rms, bias, rotary embedding -> q and the KV cache
//   attn    : split-KV causal (or tree) attention, one online softmax per wavefront, merge in LDS
//   O       : o * Wo^T + h -> h, and the sums of squares of its rows per 16 columns
//   gate/up : (h * gain) * [Wg|Wu]^T, row scale, SwiGLU -> a
//   down    : a * Wd^T + h -> h, sums of squares
// then (h * gain) * E^T, row scale -> logits.
//
// What bounds it: the float32 shape is small (15 MB of weights), everything sits in the caches, and a
// kernel's time is its launch plus a few dependent memory round trips.  So norm, rotary embedding,
// SwiGLU and the residual are prologues and epilogues (five launches a layer instead of nine), a
// workgroup's eight wavefronts split K so that most of a tile's operands are requested at once, and
// operands go from memory straight to registers.  Measured on a 512-token prompt in chunks of 128 plus
// a verify of 5 rows: 8607 us with one wavefront per output column on the vector units and scalar
// attention (180 and 80 us per launch), 391 us like this.
#include "vf_internal.h"

namespace {

constexpr int NW = 8;  // wavefronts per workgroup; they split K (GEMM) or the key tiles (attention)

enum { F_QKV = 0, F_RESID = 1, F_SWIGLU = 2, F_LOGITS = 3 };

struct GemmF32 {
    const float *W, *X;          // [N, K] and [rows, K], row-major
    int N, K, rows, row_lo;      // rows row_lo .. rows - 1 are computed
    const float *gain, *ss_in;   // normalising epilogues: RMSNorm gain, sums of squares [n_ss][ss_ld]
    int n_ss, ss_ld;
    float inv_d, eps;
    float *out;                  // F_RESID: h (in place); F_SWIGLU: a [rows, N / 2]; F_LOGITS: row row_lo first
    float *ss_out;
    const float *bias, *cosv, *sinv;   // F_QKV
    float *q;
    int layer, hq, hkv, hd;
    const int32_t *depth;
};

// sum of N partial sums, in pairs
template <int N> __device__ __forceinline__ floatx4 pairwise(const floatx4 *p) {
    if constexpr (N == 1) return p[0];
    else return pairwise<N / 2>(p) + pairwise<N - N / 2>(p + N / 2);
}

// One workgroup: 16 * RB rows x 16 * UB columns.  A 16-wide K chunk is one 16-byte load per lane and
// operand block: lane (g, i) holds columns 4 g .. 4 g + 3 of row i, and matrix instruction j of the
// chunk takes column 4 g + j from every lane, of both operands.
template <int RB, int UB, int EPI>
__global__ __launch_bounds__(NW * 64) VF_MFMA_KERNEL void gemm_f32_kernel(GemmF32 p, Batch b) {
    constexpr bool NORMED = EPI != F_RESID;
    constexpr int U = RB * UB > 2 ? 2 : 4;                // chunks requested together
    // Eight partial sums of a wavefront: matrix instruction j of a chunk adds to sum j, and the four are put aside half
    // way through the wavefront's chunks.  A sum is a chain of K / 64 products, as with one product a lane, and sums are
    // added in pairs: with one sum a wavefront the logits' error was a third to two thirds larger (1.41e-7 for 1.07e-7 at
    // d 256, 2.37e-7 for 1.43e-7 at d 512), and its instructions waited for one another (512 tokens and 5 rows: 400 us
    // for 391; eight sums kept to the end: 412).
    constexpr int A = 4;
    constexpr int TILES = RB * UB;                        // epilogue tiles, one per wavefront
    static_assert(TILES <= NW, "one epilogue tile per wavefront");
    __shared__ floatx4 red[NW * UB * RB * 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g4 = lane >> 4, l15 = lane & 15;
    const int nb0 = blockIdx.x * UB, NBt = p.N >> 4;
    const int r0 = p.row_lo + blockIdx.y * (16 * RB);
    const int K = p.K, KC = K >> 4;
    const float *wp[UB], *xp[RB];
#pragma unroll
    for (int u = 0; u < UB; ++u) wp[u] = p.W + (size_t)(min(nb0 + u, NBt - 1) * 16 + l15) * K + g4 * 4;
#pragma unroll
    for (int r = 0; r < RB; ++r) xp[r] = p.X + (size_t)min(r0 + r * 16 + l15, p.rows - 1) * K + g4 * 4;
    // epilogue tile of this wavefront: row block er, weight block eu
    const int er = wave % RB, eu = (wave / RB) % UB;
    const int row = r0 + er * 16 + l15;
    const bool live = wave < TILES && row < p.rows && nb0 + eu < NBt;
    float ssq = 0.f;
    if (NORMED && wave < TILES)
        _Pragma("unroll 4") for (int j = g4; j < p.n_ss; j += 4) ssq += p.ss_in[(size_t)j * p.ss_ld + min(row, p.rows - 1)];

    floatx4 acc[A][UB][RB], first[UB][RB];
    auto clear = [&] {
#pragma unroll
        for (int a = 0; a < A; ++a)
#pragma unroll
            for (int u = 0; u < UB; ++u)
#pragma unroll
                for (int r = 0; r < RB; ++r) acc[a][u][r] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    auto total = [&](int u, int r) {
        floatx4 part[A];
#pragma unroll
        for (int a = 0; a < A; ++a) part[a] = acc[a][u][r];
        return pairwise<A>(part);
    };
    clear();
    // first chunk of the second half of this wavefront's chunks; at or past KC where it has one or none
    const int half = wave + ((KC - wave + NW - 1) / NW + 1) / 2 * NW;
    for (int c0 = wave; c0 < KC; c0 += NW * U) {
        floatx4 w[U][UB], x[U][RB], gn[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int k = min(c0 + i * NW, KC - 1) * 16;  // past the end: the last chunk again, not multiplied
#pragma unroll
            for (int u = 0; u < UB; ++u) w[i][u] = *reinterpret_cast<const floatx4 *>(wp[u] + k);
#pragma unroll
            for (int r = 0; r < RB; ++r) x[i][r] = *reinterpret_cast<const floatx4 *>(xp[r] + k);
            if (NORMED) gn[i] = *reinterpret_cast<const floatx4 *>(p.gain + k + g4 * 4);
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (c0 + i * NW == half && half < KC) {
#pragma unroll
                for (int u = 0; u < UB; ++u)
#pragma unroll
                    for (int r = 0; r < RB; ++r) first[u][r] = total(u, r);
                clear();
            }
            if (c0 + i * NW < KC) {  // the same for the whole wavefront
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const floatx4 xv = NORMED ? x[i][r] * gn[i] : x[i][r];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int u = 0; u < UB; ++u)
                            acc[(i * 4 + j) % A][u][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i][u][j], xv[j], acc[(i * 4 + j) % A][u][r], 0, 0, 0);
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int r = 0; r < RB; ++r) red[((wave * UB + u) * RB + r) * 64 + lane] = half < KC ? first[u][r] + total(u, r) : total(u, r);
    __syncthreads();
    if (wave >= TILES) return;
    // lane holds Y[row][16 nb + 4 g4 + 0..3]
    floatx4 part[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) part[w] = red[((w * UB + eu) * RB + er) * 64 + lane];
    floatx4 v = pairwise<NW>(part);
    if (NORMED) {
        ssq += __shfl_xor(ssq, 16, 64);
        ssq += __shfl_xor(ssq, 32, 64);
        v *= 1.0f / sqrtf(ssq * p.inv_d + p.eps);
    }
    const int n0 = (nb0 + eu) * 16 + g4 * 4;
    if (EPI == F_RESID) {
        floatx4 hv = {0.f, 0.f, 0.f, 0.f};
        float *hp = p.out + (size_t)row * p.N + n0;
        if (live) {
            hv = *reinterpret_cast<const floatx4 *>(hp) + v;
            *reinterpret_cast<floatx4 *>(hp) = hv;
        }
        float s = hv[0] * hv[0] + hv[1] * hv[1] + hv[2] * hv[2] + hv[3] * hv[3];
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (live && g4 == 0) p.ss_out[(size_t)(nb0 + eu) * p.ss_ld + row] = s;
    } else if (EPI == F_LOGITS) {
        if (live) *reinterpret_cast<floatx4 *>(p.out + (size_t)(row - p.row_lo) * p.N + n0) = v;
    } else if (EPI == F_SWIGLU) {
        if (live) {
            // gate row f is packed column 2 f, up row f column 2 f + 1
            const float2 o = {v[0] / (1.0f + expf(-v[0])) * v[1], v[2] / (1.0f + expf(-v[2])) * v[3]};
            *reinterpret_cast<float2 *>(p.out + (size_t)row * (p.N >> 1) + (n0 >> 1)) = o;
        }
    } else if (live) {
        const int hd = p.hd, half = hd >> 1;
        if (p.bias) v += *reinterpret_cast<const floatx4 *>(p.bias + n0);
        const SeqDesc &s = b.s[find_seq(b, row)];
        // slot: the cache row the call's row is written to; pos: the position whose rotary angle it takes
        const int len = s.state[0], slot = len + (row - s.row0), pos = p.depth ? len + p.depth[row] : slot;
        if (slot < 0 || slot >= s.capacity) return;
        const int head = n0 / hd, p0 = n0 % hd;
        float *kv = reinterpret_cast<float *>(s.kv);
        if (head < p.hq + p.hkv) {
            const int i0 = p0 >> 1;  // packed columns 2i, 2i+1 are elements i and i + hd/2
            const float2 c = *reinterpret_cast<const float2 *>(p.cosv + (size_t)pos * half + i0);
            const float2 sn = *reinterpret_cast<const float2 *>(p.sinv + (size_t)pos * half + i0);
            float *d0, *d1;
            if (head < p.hq) {
                d0 = p.q + ((size_t)row * p.hq + head) * hd + i0;
                d1 = d0 + half;
            } else {
                const int page = kv_page(s, slot), tin = slot % VF_TILE;
                d0 = kv + kv_k_index(p.layer, s.n_pages, page, p.hkv, head - p.hq, tin, i0, hd);
                d1 = kv + kv_k_index(p.layer, s.n_pages, page, p.hkv, head - p.hq, tin, i0 + half, hd);
            }
            *reinterpret_cast<float2 *>(d0) = float2{v[0] * c.x - v[1] * sn.x, v[2] * c.y - v[3] * sn.y};
            *reinterpret_cast<float2 *>(d1) = float2{v[1] * c.x + v[0] * sn.x, v[3] * c.y + v[2] * sn.y};
        } else {
            const int page = kv_page(s, slot), tin = slot % VF_TILE;
            for (int j = 0; j < 4; ++j)
                kv[kv_v_index(p.layer, s.n_pages, page, p.hkv, head - p.hq - p.hkv, tin, p0 + j, hd)] = v[j];
        }
    }
}

// h = embedding row, and its sums of squares per 16 columns
__global__ __launch_bounds__(256) void embed_f32_kernel(const float *__restrict__ E, const int32_t *__restrict__ tokens, Batch b,
                                                        float *__restrict__ h, float *__restrict__ ss, int d, int vocab, int ss_ld) {
    const int row = blockIdx.x;
    int tok = tokens[row];
    if (tok == VF_PENDING) tok = b.s[find_seq(b, row)].state[1];
    if (tok < 0 || tok >= vocab) tok = 0;
    for (int k0 = 0; k0 < d; k0 += 256) {
        const int k = k0 + threadIdx.x;
        const float v = k < d ? E[(size_t)tok * d + k] : 0.f;
        if (k < d) h[(size_t)row * d + k] = v;
        float s = v * v;
        s += __shfl_xor(s, 8, 64);
        s += __shfl_xor(s, 4, 64);
        s += __shfl_xor(s, 2, 64);
        s += __shfl_xor(s, 1, 64);
        if (k < d && (k & 15) == 0) ss[(size_t)(k >> 4) * ss_ld + row] = s;
    }
}

// What exponents are taken against where the largest score is m: m, or 0 where no key has been seen yet.
__device__ __forceinline__ float f32_reference(float m) { return m == -INFINITY ? 0.f : m; }

// Attention: one workgroup per (16 query items, kv head, sequence, part of the keys); a query item is a
// (row, head of the group) pair.  The wavefronts take the 32-key tiles in turn, operands straight from
// the cache: its fragment order gives lane (g, i) eight consecutive features of key 8 (i >> 2) + (i & 3)
// + 4 half, so the scores S^T[key, item] leave the matrix unit with keys 8 g .. 8 g + 7 in one lane,
// which is how the P V product takes them.  An item takes nothing from a key it does not see, whatever that
// key's value is (0 * infinity is not 0): tiles with such keys look at their values first.
template <int HD>
__global__ __launch_bounds__(NW * 64) VF_MFMA_KERNEL void attn_f32_kernel(
    Batch b, int layer, const float *__restrict__ q, float *__restrict__ o, int hq, int hkv, float scale,
    int n_parts, float *__restrict__ part, const tree_mask_t *__restrict__ anc) {
    constexpr int KD = HD / 32, DB = HD / 16, REC = HD + 4;
    extern __shared__ __align__(16) unsigned char smem[];
    floatx4 *o_s = reinterpret_cast<floatx4 *>(smem);                 // [wave][db][lane]
    float *ml_s = reinterpret_cast<float *>(smem + NW * DB * 1024);   // [wave][2][16]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g4 = lane >> 4, l15 = lane & 15;
    const int kvh = blockIdx.y, kpart = blockIdx.z % n_parts;
    const SeqDesc &s = b.s[blockIdx.z / n_parts];
    const int group = hq / hkv, n_items = s.nrows * group, item0 = blockIdx.x * 16;
    if (item0 >= n_items) return;
    const int len = s.state[0], kmax = min(len + s.nrows, s.capacity);
    const int item = item0 + l15;
    const bool valid = item < n_items;
    const int r = valid ? item / group : 0, head = kvh * group + (valid ? item % group : 0), row = s.row0 + r;
    const int last_key = valid ? len + r : -1;
    const int blk_last = min(kmax - 1, len + min(s.nrows - 1, (item0 + 15) / group));
    const tree_mask_t mask = anc && valid ? anc[row] : ~(tree_mask_t)0;
    auto visible = [&](int key) { return key <= last_key && (!anc || key < len || ((mask >> ((unsigned)(key - len) & 63u)) & 1)); };
    floatx4 qf[KD][2], oacc[DB];
#pragma unroll
    for (int kd = 0; kd < KD; ++kd)
#pragma unroll
        for (int i = 0; i < 2; ++i)
            qf[kd][i] = *reinterpret_cast<const floatx4 *>(q + ((size_t)row * hq + head) * HD + kd * 32 + g4 * 8 + i * 4) * scale;
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] = floatx4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    const int tiles = blk_last / 32 + 1, tpp = (tiles + n_parts - 1) / n_parts;
    const int t_begin = kpart * tpp, t_end = min(tiles, t_begin + tpp);
    const float *kv = reinterpret_cast<const float *>(s.kv);
    for (int t = t_begin + wave; t < t_end; t += NW) {
        const int t0 = t * 32, page = kv_page(s, t0), tin = t0 % VF_TILE;
        const float *kb = kv + kv_k_index(layer, s.n_pages, page, hkv, kvh, tin, 0, HD) + lane * 8;
        const float *vb = kv + kv_v_index(layer, s.n_pages, page, hkv, kvh, tin, 0, HD) + lane * 8;
        floatx4 kf[2][KD][2], vf[DB][2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int kd = 0; kd < KD; ++kd)
#pragma unroll
                for (int i = 0; i < 2; ++i) kf[h][kd][i] = *reinterpret_cast<const floatx4 *>(kb + (h * KD + kd) * 512 + i * 4);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 2; ++i) vf[db][i] = *reinterpret_cast<const floatx4 *>(vb + db * 512 + i * 4);
        floatx4 sc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int kd = 0; kd < KD; ++kd)
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    sc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[h][kd][j >> 2][j & 3], qf[kd][j >> 2][j & 3], sc[h], 0, 0, 0);
        // lane holds keys t0 + 8 g4 + j of item l15
        float pr[8], tmax = -INFINITY;
        bool vis[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            vis[j] = visible(t0 + g4 * 8 + j);
            pr[j] = vis[j] ? sc[j >> 2][j & 3] : -INFINITY;
            tmax = fmaxf(tmax, pr[j]);
        }
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
        const float m_old = m_run;
        m_run = fmaxf(m_run, tmax);
        const float m_new = f32_reference(m_run), corr = expf(m_old - m_new);
        float psum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            pr[j] = vis[j] ? expf(pr[j] - m_new) : 0.f;
            psum += pr[j];
        }
        psum += __shfl_xor(psum, 16, 64);
        psum += __shfl_xor(psum, 32, 64);
        l_run = l_run * corr + psum;
#pragma unroll
        for (int db = 0; db < DB; ++db) oacc[db] *= corr;
        float odd = 0.f;   // 0, or NaN where a value that some item may not see is not finite
        if (t0 + 31 > len) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    // rows of the cache at or past kmax may hold anything
                    if (t0 + g4 * 8 + j >= kmax) vf[db][j >> 2][j & 3] = 0.f;
                    odd = fmaf(vf[db][j >> 2][j & 3], 0.f, odd);
                }
        }
        if (__builtin_amdgcn_ballot_w64(odd != 0.f)) {   // key by key, what the item sees
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll 1
                    for (int g = 0; g < 4; ++g) {
                        const float p = __shfl(pr[j], g * 16 + l15, 64);
                        const bool seen = visible(t0 + g * 8 + j);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float v = __shfl(vf[db][j >> 2][j & 3], g * 16 + g4 * 4 + e, 64);
                            if (seen) oacc[db][e] = fmaf(p, v, oacc[db][e]);
                        }
                    }
        } else {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    oacc[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[db][j >> 2][j & 3], pr[j], oacc[db], 0, 0, 0);
        }
    }
#pragma unroll
    for (int db = 0; db < DB; ++db) o_s[(wave * DB + db) * 64 + lane] = oacc[db];
    if (g4 == 0) {
        ml_s[(wave * 2 + 0) * 16 + l15] = m_run;
        ml_s[(wave * 2 + 1) * 16 + l15] = l_run;
    }
    __syncthreads();
    if (wave >= DB) return;
    // wavefront = 16-wide block of the head dimension
    float M = -INFINITY, L = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, ml_s[(w * 2) * 16 + l15]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float wt = expf(ml_s[(w * 2) * 16 + l15] - f32_reference(M));
        L += ml_s[(w * 2 + 1) * 16 + l15] * wt;
        acc += o_s[(w * DB + wave) * 64 + lane] * wt;
    }
    if (!valid) return;
    if (n_parts > 1) {
        float *rec = part + (((size_t)row * hq + head) * n_parts + kpart) * REC;
        if (wave == 0 && g4 == 0) *reinterpret_cast<float2 *>(rec) = float2{M, L};
        *reinterpret_cast<floatx4 *>(rec + 4 + wave * 16 + g4 * 4) = acc;
    } else {
        *reinterpret_cast<floatx4 *>(o + ((size_t)row * hq + head) * HD + wave * 16 + g4 * 4) = acc * (1.0f / L);
    }
}

// merge of the key parts; one workgroup per (row, head), one thread per feature
template <int HD>
__global__ __launch_bounds__(HD) void attn_f32_combine_kernel(const float *__restrict__ part, float *__restrict__ o, int n_parts) {
    constexpr int REC = HD + 4;
    const int d = threadIdx.x;
    const float *p = part + (size_t)blockIdx.x * n_parts * REC;
    float M = -INFINITY, L = 0.f, acc = 0.f;
    for (int i = 0; i < n_parts; ++i) M = fmaxf(M, p[i * REC]);
    for (int i = 0; i < n_parts; ++i) {
        const float w = expf(p[i * REC] - f32_reference(M));
        L += p[i * REC + 1] * w;
        acc += p[i * REC + 4 + d] * w;
    }
    o[(size_t)blockIdx.x * HD + d] = acc / L;
}

// Rows per workgroup: 32 (16 for calls of at most 16 rows) until the grid has eight workgroups per
// compute unit anyway, then 64 rows by 32 columns, which reads half the operand bytes per product.
template <int EPI>
int launch_gemm(const GemmF32 &p, const Batch &b, hipStream_t st) {
    const int NBt = p.N >> 4, n = p.rows - p.row_lo;
    if (n <= 0) return VF_OK;
    auto go = [&](auto kern, int rb, int ub) {
        hipLaunchKernelGGL(kern, dim3((NBt + ub - 1) / ub, (n + 16 * rb - 1) / (16 * rb)), dim3(NW * 64), 0, st, p, b);
    };
    if ((size_t)NBt * ((n + 31) / 32) > 2048) go(gemm_f32_kernel<4, 2, EPI>, 4, 2);
    else if (n > 16) go(gemm_f32_kernel<2, 1, EPI>, 2, 1);
    else go(gemm_f32_kernel<1, 1, EPI>, 1, 1);
    VF_LAUNCH_CHECK("gemm_f32");
    return VF_OK;
}

template <int HD>
int launch_attn(const vf_model *m, const Batch &b, int layer, const tree_mask_t *anc, hipStream_t st) {
    const vf_config &c = m->cfg;
    const int group = c.n_q_heads / c.n_kv_heads;
    int max_items = 0, max_keys = 0;
    for (int i = 0; i < b.n_seqs; ++i) {
        max_items = max(max_items, b.s[i].nrows * group);
        max_keys = max(max_keys, b.s[i].len_ub + b.s[i].nrows);
    }
    // 64 key tiles per workgroup, eight per wavefront, before the keys are shared out over several
    int n_parts = min(16, max(1, ((max_keys + 31) / 32 + 63) / 64));
    while (n_parts > 1 && (size_t)b.total_rows * c.n_q_heads * n_parts * (HD + 4) > m->attn_part_floats) --n_parts;
    const int lds = NW * (HD / 16) * 1024 + NW * 2 * 16 * 4;
    hipLaunchKernelGGL(attn_f32_kernel<HD>, dim3((max_items + 15) / 16, c.n_kv_heads, b.n_seqs * n_parts), dim3(NW * 64), lds, st,
                       b, layer, (const float *)m->q, (float *)m->o, c.n_q_heads, c.n_kv_heads,
                       1.0f / sqrtf((float)HD), n_parts, m->attn_part, anc);
    VF_LAUNCH_CHECK("attn_f32");
    if (n_parts > 1) {
        hipLaunchKernelGGL(attn_f32_combine_kernel<HD>, dim3(b.total_rows * c.n_q_heads), dim3(HD), 0, st, m->attn_part,
                           (float *)m->o, n_parts);
        VF_LAUNCH_CHECK("attn_f32_combine");
    }
    return VF_OK;
}

GemmF32 base_args(const vf_model *m, int rows) {
    const vf_config &c = m->cfg;
    GemmF32 p;
    memset(&p, 0, sizeof p);
    p.rows = rows;
    p.ss_in = m->ss;
    p.ss_out = m->ss;
    p.n_ss = c.d_model / 16;
    p.ss_ld = m->ss_ld;
    p.inv_d = 1.0f / (float)c.d_model;
    p.eps = c.rms_eps;
    return p;
}

}  // namespace

int vf_f32_init(const vf_model *m) {
    if (m->cfg.head_dim != 128) return VF_OK;
    VF_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(attn_f32_kernel<128>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               NW * 8 * 1024 + NW * 2 * 16 * 4));
    return VF_OK;
}

// Decoder layers over the rows of `b`; leaves the residual stream in m->h and its sums of squares in m->ss.
int vf_run_layers_f32(vf_model *m, const Batch &b, const int32_t *tokens, bool tree, hipStream_t st) {
    const vf_config &c = m->cfg;
    const int rows = b.total_rows, d = c.d_model, F = c.d_ffn, nq = c.n_q_heads * c.head_dim, nkv = c.n_kv_heads * c.head_dim;
    hipLaunchKernelGGL(embed_f32_kernel, dim3(rows), dim3(256), 0, st, (const float *)m->embed, tokens, b, m->h, m->ss, d, c.vocab,
                       m->ss_ld);
    VF_LAUNCH_CHECK("embed_f32");
    for (int l = 0; l < c.n_layers; ++l) {
        const LayerPacked &lp = m->layers[l];
        int rc;
        GemmF32 p = base_args(m, rows);
        p.W = (const float *)lp.wqkv; p.X = m->h; p.N = nq + 2 * nkv; p.K = d; p.gain = lp.attn_norm;
        p.bias = c.qkv_bias ? lp.bqkv : nullptr; p.cosv = m->rope_cos; p.sinv = m->rope_sin; p.q = (float *)m->q;
        p.layer = l; p.hq = c.n_q_heads; p.hkv = c.n_kv_heads; p.hd = c.head_dim; p.depth = tree ? m->tree_depth : nullptr;
        { ProfScope ps(m, VF_SITE_QKV, st);
          if ((rc = launch_gemm<F_QKV>(p, b, st))) return rc; }
        { ProfScope ps(m, VF_SITE_ATTN, st);
          const tree_mask_t *anc = tree ? m->tree_anc : nullptr;
          if ((rc = c.head_dim == 64 ? launch_attn<64>(m, b, l, anc, st) : launch_attn<128>(m, b, l, anc, st))) return rc; }
        p = base_args(m, rows);
        p.W = (const float *)lp.wo; p.X = (const float *)m->o; p.N = d; p.K = nq; p.out = m->h;
        { ProfScope ps(m, VF_SITE_O, st);
          if ((rc = launch_gemm<F_RESID>(p, b, st))) return rc; }
        p = base_args(m, rows);
        p.W = (const float *)lp.wgu; p.X = m->h; p.N = 2 * F; p.K = d; p.gain = lp.ffn_norm; p.out = (float *)m->a;
        { ProfScope ps(m, VF_SITE_GATEUP, st);
          if ((rc = launch_gemm<F_SWIGLU>(p, b, st))) return rc; }
        p = base_args(m, rows);
        p.W = (const float *)lp.wd; p.X = (const float *)m->a; p.N = d; p.K = F; p.out = m->h;
        { ProfScope ps(m, VF_SITE_DOWN, st);
          if ((rc = launch_gemm<F_RESID>(p, b, st))) return rc; }
    }
    return VF_OK;
}

// Final norm + output head for rows [row_lo, row_hi) -> out[row - row_lo][vocab].
int vf_run_head_f32(vf_model *m, int row_lo, int row_hi, float *out, hipStream_t st) {
    const vf_config &c = m->cfg;
    Batch none;
    none.n_seqs = 0;
    none.total_rows = 0;
    GemmF32 p = base_args(m, row_hi);
    p.row_lo = row_lo; p.W = (const float *)m->lm_head; p.X = m->h; p.N = c.vocab; p.K = c.d_model; p.gain = m->final_norm;
    p.out = out;
    ProfScope ps(m, VF_SITE_HEAD, st);
    return launch_gemm<F_LOGITS>(p, none, st);
}
