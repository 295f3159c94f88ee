// Small kernels around the GEMMs: weight re-packing, rotary tables, embedding gather,
// residual + RMSNorm, the QKV epilogue (bias, rotary embedding, KV append), SwiGLU, and the
// device-side sequence state.  Each adds the split-K partial sums of the GEMM before it in a
// fixed order.
#include <type_traits>

#include "vf_internal.h"

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
namespace {

// ---- model creation -----------------------------------------------------------------------------

// Row-major bf16 [n_rows, K] -> 16x32 fragments of the packed rows 16 * dst_nb0 + n.  With a second
// source the two alternate: packed row 2 f is row f of the first, 2 f + 1 row f of the second (gate and
// up: a lane of the GEMM then holds both factors of a SwiGLU product).
// perm_hd > 0: within every head of perm_hd rows, packed row 2i is source row i and packed row 2i+1
// is source row i + perm_hd/2, so that the two elements of a rotary pair are neighbours.
__device__ inline int pack_src_row(int n, int perm_hd) {
    if (perm_hd <= 0) return n;
    const int head = n / perm_hd, p = n % perm_hd;
    return head * perm_hd + (p >> 1) + (p & 1) * (perm_hd >> 1);
}

__global__ void pack_bf16_kernel(const uint16_t *__restrict__ src, const uint16_t *__restrict__ src2, uint4 *__restrict__ dst,
                                 int n_rows, int K, int dst_nb0, int perm_hd) {
    const int KB = K >> 5;
    size_t total = (size_t)(n_rows >> 4) * KB * 64;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        int lane = (int)(i & 63);
        size_t f = i >> 6;
        int kb = (int)(f % KB), nb = (int)(f / KB);
        int n = nb * 16 + (lane & 15), k = kb * 32 + (lane >> 4) * 8;
        const uint16_t *from = src2 ? ((n & 1) ? src2 : src) + (size_t)(n >> 1) * K : src + (size_t)pack_src_row(n, perm_hd) * K;
        dst[((size_t)(dst_nb0 + nb) * KB + kb) * 64 + lane] = *reinterpret_cast<const uint4 *>(from + k);
    }
}

// float32 model: the same order of rows, plain row-major.
__global__ void pack_f32_kernel(const float *__restrict__ src, const float *__restrict__ src2, float *__restrict__ dst, int n_rows,
                                int K, int dst_nb0, int perm_hd) {
    size_t total = (size_t)n_rows * K;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        int n = (int)(i / K), k = (int)(i % K);
        const float *from = src2 ? ((n & 1) ? src2 : src) + (size_t)(n >> 1) * K : src + (size_t)pack_src_row(n, perm_hd) * K;
        dst[(size_t)(dst_nb0 * 16 + n) * K + k] = from[k];
    }
}

// cos/sin of pos * theta^(-2i/hd), evaluated in float64 and stored as float32.
__global__ void rope_table_kernel(float *__restrict__ cosv, float *__restrict__ sinv, int max_pos, int half,
                                  double theta) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= max_pos * half) return;
    int pos = i / half, j = i % half;
    double inv = pow(theta, -2.0 * (double)j / (double)(2 * half));
    double ang = (double)pos * inv;
    cosv[i] = (float)cos(ang);
    sinv[i] = (float)sin(ang);
}

// ---- forward pass helpers -----------------------------------------------------------------------

// One workgroup per row.  The first wavefronts gather, pieces of eight elements that lie together in the packed matrix; the
// last finds the row's place.
__global__ __launch_bounds__(256) void embed_kernel(const bf16_t *__restrict__ E, const int32_t *__restrict__ tokens, Batch b,
                                                    float *__restrict__ h, int d, int vocab, const int32_t *__restrict__ depth, int hkv, int hd,
                                                    const float *__restrict__ cosv, const float *__restrict__ sinv, RowPlace *__restrict__ place,
                                                    float *__restrict__ row_cos, float *__restrict__ row_sin) {
    const int row = blockIdx.x, half = hd / 2, i = threadIdx.x - 192;
    if (i >= 0 && i < half) {
        const RowPlace p = row_place(b, depth, hkv, hd, row);
        if (i == 0) place[row] = p;
        row_cos[(size_t)row * half + i] = cosv[(size_t)p.pos * half + i];
        row_sin[(size_t)row * half + i] = sinv[(size_t)p.pos * half + i];
    }
    int tok = tokens[row];
    if (tok == VF_PENDING) tok = b.s[find_seq(b, row)].state[1];
    if (tok < 0 || tok >= vocab) tok = 0;
    for (int k = threadIdx.x * 8; k < d; k += 2048) {
        const bf16x8 e = *reinterpret_cast<const bf16x8 *>(E + wfrag_index(tok, k, d));
        float *p = h + (size_t)row * d + k;
        *reinterpret_cast<floatx4 *>(p) = floatx4{(float)e[0], (float)e[1], (float)e[2], (float)e[3]};
        *reinterpret_cast<floatx4 *>(p + 4) = floatx4{(float)e[4], (float)e[5], (float)e[6], (float)e[7]};
    }
}

__device__ inline float block_sum(float v, float *red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    float s = 0.f;
    for (int i = 0; i < nw; ++i) s += red[i];
    __syncthreads();
    return s;
}

// The same for 256 threads, in one exchange: lanes by register exchanges, wavefronts by one barrier; `red` is written once.
// (Six shuffles through LDS and two barriers were 0.7 us of the norm's 2.3 to 3 at 128 rows of 0.5B: a prompt of 777 tokens
// in chunks of 128 6586 -> 6472 us.)
__device__ __forceinline__ float block_sum_256(float v, float *red) {
    auto add = [&](auto ctrl) {
        v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    add(std::integral_constant<int, 0xb1>{});    // the other lane of a pair
    add(std::integral_constant<int, 0x4e>{});    // the other pair of four
    add(std::integral_constant<int, 0x141>{});   // the other four of eight
    add(std::integral_constant<int, 0x140>{});   // the other eight of sixteen
    auto row = [&](int lane) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane)); };
    const float s = (row(0) + row(16)) + (row(32) + row(48));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    lds_sync();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// h[row] += sum of partials (if any); x[row] = bf16(rmsnorm(h[row]) * gain) in activation layout.
__global__ __launch_bounds__(256) void norm_kernel(float *__restrict__ h, const float *__restrict__ part,
                                                   int nparts, int ld_rows, const float *__restrict__ gain,
                                                   bf16_t *__restrict__ x, int d, int ncb, float eps) {
    __shared__ float red[4];
    const int row = blockIdx.x;
    float ss = 0.f;
    for (int k = threadIdx.x; k < d; k += 256) {
        float v = h[(size_t)row * d + k];
        for (int p = 0; p < nparts; ++p) v += part[((size_t)p * ld_rows + row) * d + k];
        if (nparts) h[(size_t)row * d + k] = v;
        ss += v * v;
    }
    ss = block_sum(ss, red);
    const float inv = 1.0f / sqrtf(ss / (float)d + eps);
    for (int k = threadIdx.x; k < d; k += 256)
        x[xfrag_index(row, k, ncb)] = (bf16_t)(h[(size_t)row * d + k] * inv * gain[k]);
}

// The same for d up to 4096: a thread owns runs of eight consecutive
// elements (one 16-byte piece of an activation fragment), keeps them in registers between the
// sum of squares and the scaling, and stores the piece whole.  NP: partial sums requested together (one after
// the other, each waited for the one before: 5.5 us per launch at 256 rows, 8 partials); the smallest of 1, 2,
// 4, 8 that holds them, as the loads past the last one repeat it: with 8 for one
// partial 1024 rows of 3072 took 12.9 us instead of 11.6, 876 rows 12.1 instead of 10.2.
template <int VPT, int NP>
__global__ __launch_bounds__(256) void norm_bf16_vec_kernel(float *__restrict__ h, const float *__restrict__ part,
                                                            int nparts, int ld_rows, const float *__restrict__ gain,
                                                            u32x4_t *__restrict__ x, int d, int ncb, float eps) {
    __shared__ float red[4];
    const int row = blockIdx.x;
    float v[VPT][8];
    floatx4 g[VPT][2];   // the gain is requested with the row, not behind its sum
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int k0 = (threadIdx.x + i * 256) * 8;
        if (k0 < d) {
            g[i][0] = *reinterpret_cast<const floatx4 *>(gain + k0);
            g[i][1] = *reinterpret_cast<const floatx4 *>(gain + k0 + 4);
            float *hp = h + (size_t)row * d + k0;
            const float4 a = *reinterpret_cast<const float4 *>(hp), b = *reinterpret_cast<const float4 *>(hp + 4);
            v[i][0] = a.x; v[i][1] = a.y; v[i][2] = a.z; v[i][3] = a.w;
            v[i][4] = b.x; v[i][5] = b.y; v[i][6] = b.z; v[i][7] = b.w;
            for (int p0 = 0; p0 < nparts; p0 += NP) {
                float4 c[NP], e[NP];
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const float *pp = part + ((size_t)min(p0 + p, nparts - 1) * ld_rows + row) * d + k0;
                    c[p] = *reinterpret_cast<const float4 *>(pp);
                    e[p] = *reinterpret_cast<const float4 *>(pp + 4);
                }
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    if (p0 + p < nparts) {
                        v[i][0] += c[p].x; v[i][1] += c[p].y; v[i][2] += c[p].z; v[i][3] += c[p].w;
                        v[i][4] += e[p].x; v[i][5] += e[p].y; v[i][6] += e[p].z; v[i][7] += e[p].w;
                    }
                }
            }
            if (nparts) {
                *reinterpret_cast<float4 *>(hp) = float4{v[i][0], v[i][1], v[i][2], v[i][3]};
                *reinterpret_cast<float4 *>(hp + 4) = float4{v[i][4], v[i][5], v[i][6], v[i][7]};
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[i][j] = 0.f;
        }
    }
    // the sum runs over k in the order of the scalar kernel's threads only up to rounding; both
    // are sums of d squares in float32
#pragma unroll
    for (int i = 0; i < VPT; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) ss += v[i][j] * v[i][j];
    ss = block_sum_256(ss, red);
    const float inv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int k0 = (threadIdx.x + i * 256) * 8;
        if (k0 >= d) continue;
        const float gv[8] = {g[i][0][0], g[i][0][1], g[i][0][2], g[i][0][3], g[i][1][0], g[i][1][1], g[i][1][2], g[i][1][3]};
        u32x4_t out;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bf16_t lo = (bf16_t)(v[i][2 * j] * inv * gv[2 * j]), hi = (bf16_t)(v[i][2 * j + 1] * inv * gv[2 * j + 1]);
            out[j] = (unsigned)__builtin_bit_cast(unsigned short, lo) | ((unsigned)__builtin_bit_cast(unsigned short, hi) << 16);
        }
        const int kb = k0 >> 5, lane = (((k0 >> 3) & 3) << 4) | (row & 15);
        x[((size_t)kb * ncb + (row >> 4)) * 64 + lane] = out;
    }
}

// QKV epilogue of a GEMM whose K was split: one thread per (row, four packed columns).
__global__ __launch_bounds__(256) void qkv_finish_kernel(const float *__restrict__ part, int nparts, int ld_rows, QkvEpilogue e) {
    const int N = (e.hq + 2 * e.hkv) * e.hd, per_row = N >> 2;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= e.b.total_rows * per_row) return;
    const int row = idx / per_row, n0 = (idx % per_row) * 4;
    const int nb = n0 >> 4, g4 = n0 >> 2 & 3;
    const RowPlace place = row_place(e.b, e.depth, e.hkv, e.hd, row);
    const QkvPlace at = qkv_place(e, place, g4);
    const QkvAngles angles = qkv_angles(e, place.pos, nb, g4);
    floatx4 v = {0.f, 0.f, 0.f, 0.f};
    for (int q0 = 0; q0 < nparts; q0 += 4) {   // requested together, added in order
        floatx4 t[4];
#pragma unroll
        for (int p = 0; p < 4; ++p)
            t[p] = *reinterpret_cast<const floatx4 *>(part + ((size_t)min(q0 + p, nparts - 1) * ld_rows + row) * N + n0);
#pragma unroll
        for (int p = 0; p < 4; ++p)
            if (q0 + p < nparts) v += t[p];
    }
    qkv_store(e, at, angles, row, nb, g4, v);
}

// a[row, f] = bf16(silu(gate) * up); gate and up alternate in the columns of the gate/up GEMM's output.
__global__ void swiglu_kernel(const float *__restrict__ part, int nparts, int ld_rows, bf16_t *__restrict__ a,
                              int rows, int F, int ncb) {
    size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= (size_t)rows * F) return;
    const int row = (int)(idx / F), f = (int)(idx % F);
    float g = 0.f, u = 0.f;
    for (int p = 0; p < nparts; ++p) {
        const float2 gu = *reinterpret_cast<const float2 *>(part + ((size_t)p * ld_rows + row) * (2 * (size_t)F) + 2 * f);
        g += gu.x;
        u += gu.y;
    }
    const float sg = g / (1.0f + expf(-g));
    a[xfrag_index(row, f, ncb)] = (bf16_t)(sg * u);
}

__global__ void state_set_kernel(int32_t *state, int idx, int32_t value) { state[idx] = value; }
__global__ void state_add_kernel(int32_t *state, int idx, int32_t delta) { state[idx] += delta; }

template <typename T>
__global__ void kv_read_kernel(SeqDesc s, int layer, int t0, int n, int hkv, int hd, float *__restrict__ k_out,
                               float *__restrict__ v_out) {
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * hkv * hd) return;
    const int r = idx / (hkv * hd), head = (idx / hd) % hkv, d = idx % hd;
    const int t = t0 + r;
    const T *kv = reinterpret_cast<const T *>(s.kv);
    const int page = kv_page(s, t), tin = t % VF_TILE;
    k_out[idx] = to_f32(kv[kv_k_index(layer, s.n_pages, page, hkv, head, tin, d, hd)]);
    v_out[idx] = to_f32(kv[kv_v_index(layer, s.n_pages, page, hkv, head, tin, d, hd)]);
}

template <typename T>
__global__ void kv_write_kernel(SeqDesc s, int layer, int t0, int n, int hkv, int hd, const float *__restrict__ k_in,
                                const float *__restrict__ v_in) {
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * hkv * hd) return;
    const int r = idx / (hkv * hd), head = (idx / hd) % hkv, d = idx % hd;
    const int t = t0 + r;
    T *kv = reinterpret_cast<T *>(s.kv);
    const int page = kv_page(s, t), tin = t % VF_TILE;
    kv[kv_k_index(layer, s.n_pages, page, hkv, head, tin, d, hd)] = from_f32<T>(k_in[idx]);
    kv[kv_v_index(layer, s.n_pages, page, hkv, head, tin, d, hd)] = from_f32<T>(v_in[idx]);
}

inline int nblocks(size_t n, int bs) { return (int)((n + bs - 1) / bs); }

__global__ void pack_vec_kernel(const float *__restrict__ src, float *__restrict__ dst, int n, int perm_hd) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[pack_src_row(i, perm_hd)];
}

// Tree-structured drafts: lane r of the sequence's wavefront walks from row r to the root and
// collects the ancestor mask (bit j = row j lies on the path, r itself included) and the depth.
// The host has checked 0 <= parent < r, so the walk ends after at most r steps.
__global__ __launch_bounds__(64) void tree_prep_kernel(Batch b, TreeDesc tree, tree_mask_t *__restrict__ anc,
                                                       int32_t *__restrict__ depth) {
    const SeqDesc &s = b.s[blockIdx.x];
    const int r = threadIdx.x;
    if (r >= s.nrows) return;
    tree_mask_t mask = 0;
    int d = 0;
    for (int a = r, steps = 0; a >= 0 && steps <= VF_MAX_DRAFTS; ++steps) {
        mask |= (tree_mask_t)1 << a;
        const int p = a > 0 ? tree.parent[blockIdx.x][a] : -1;
        if (p >= 0) ++d;
        a = p;
    }
    anc[s.row0 + r] = mask;
    depth[s.row0 + r] = d;
}

// After a tree verify: cache rows of the accepted path go to len_old + 1 .. len_old + a in path
// order (row len_old, the root, stays).  Path rows increase and path[j] >= j, so a destination row
// j can be the source only of an earlier step (path[j'] = j with j' < j).  One thread per (layer,
// kv head, element) copies its element for j = 1, 2, ... in turn: it has read row path[j'] before
// it overwrites that row at step j.
template <typename T>
__global__ void kv_compact_kernel(Batch b, const int32_t *__restrict__ n_accept, const int32_t *__restrict__ path,
                                  int n_layers, int hkv, int hd) {
    const SeqDesc &s = b.s[blockIdx.y];
    const int a = n_accept[blockIdx.y];
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n_layers * hkv * hd || a <= 0 || a >= s.nrows) return;
    const int layer = idx / (hkv * hd), head = (idx / hd) % hkv, d = idx % hd;
    const int len_old = s.state[0] - 1 - a;  // the acceptance kernels have already advanced the length
    T *kv = reinterpret_cast<T *>(s.kv);
    for (int j = 1; j <= a; ++j) {
        const int r = path[s.row0 + j];
        if (r == j || r < j || r >= s.nrows) continue;
        const int src = len_old + r, dst = len_old + j;
        if (src >= s.capacity) continue;
        const int ps = kv_page(s, src), pd = kv_page(s, dst);
        kv[kv_k_index(layer, s.n_pages, pd, hkv, head, dst % VF_TILE, d, hd)] =
            kv[kv_k_index(layer, s.n_pages, ps, hkv, head, src % VF_TILE, d, hd)];
        kv[kv_v_index(layer, s.n_pages, pd, hkv, head, dst % VF_TILE, d, hd)] =
            kv[kv_v_index(layer, s.n_pages, ps, hkv, head, src % VF_TILE, d, hd)];
    }
}

}  // namespace

int vf_launch_pack_vec(const float *src, float *dst, int n, int perm_hd, hipStream_t st) {
    hipLaunchKernelGGL(pack_vec_kernel, dim3((n + 255) / 256), dim3(256), 0, st, src, dst, n, perm_hd);
    VF_LAUNCH_CHECK("pack_vec");
    return VF_OK;
}

int vf_launch_pack(const vf_model *m, const void *src, const void *src2, void *dst, int n_rows, int K, int dst_nb0,
                   int perm_hd, hipStream_t st) {
    const bool bf16 = m->cfg.dtype == VF_BF16;
    const size_t total = bf16 ? (size_t)(n_rows >> 4) * (K >> 5) * 64 : (size_t)n_rows * K;
    const int grid = (int)((total + 255) / 256 < 65535 ? (total + 255) / 256 : 65535);
    if (bf16)
        hipLaunchKernelGGL(pack_bf16_kernel, dim3(grid), dim3(256), 0, st, (const uint16_t *)src, (const uint16_t *)src2, (uint4 *)dst,
                           n_rows, K, dst_nb0, perm_hd);
    else
        hipLaunchKernelGGL(pack_f32_kernel, dim3(grid), dim3(256), 0, st, (const float *)src, (const float *)src2, (float *)dst, n_rows,
                           K, dst_nb0, perm_hd);
    VF_LAUNCH_CHECK("pack");
    return VF_OK;
}

int vf_launch_rope_table(const vf_model *m, hipStream_t st) {
    const int half = m->cfg.head_dim / 2, n = m->cfg.max_positions * half;
    hipLaunchKernelGGL(rope_table_kernel, dim3(nblocks(n, 256)), dim3(256), 0, st, m->rope_cos, m->rope_sin,
                       m->cfg.max_positions, half, (double)m->cfg.rope_theta);
    VF_LAUNCH_CHECK("rope_table");
    return VF_OK;
}

int vf_launch_embed(const vf_model *m, const Batch &b, const int32_t *tokens, const int32_t *depth, hipStream_t st) {
    const vf_config &c = m->cfg;
    hipLaunchKernelGGL(embed_kernel, dim3(b.total_rows), dim3(256), 0, st, (const bf16_t *)m->embed, tokens, b, m->h, c.d_model, c.vocab,
                       depth, c.n_kv_heads, c.head_dim, m->rope_cos, m->rope_sin, m->row_place, m->row_cos, m->row_sin);
    VF_LAUNCH_CHECK("embed");
    return VF_OK;
}

int vf_launch_norm(const vf_model *m, const float *gain, void *x_out, const float *part, int nparts, int rows,
                   int ld_rows, hipStream_t st) {
    const int ncb = (rows + 15) >> 4;
    const int d = m->cfg.d_model;
    auto vec = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(rows), dim3(256), 0, st, m->h, part, nparts, ld_rows, gain, (u32x4_t *)x_out, d, ncb,
                           m->cfg.rms_eps);
    };
    if (d <= 2048) {
        if (nparts <= 1) vec(norm_bf16_vec_kernel<1, 1>);
        else if (nparts <= 2) vec(norm_bf16_vec_kernel<1, 2>);
        else if (nparts <= 4) vec(norm_bf16_vec_kernel<1, 4>);
        else vec(norm_bf16_vec_kernel<1, 8>);
    } else if (d <= 4096) {
        if (nparts <= 1) vec(norm_bf16_vec_kernel<2, 1>);
        else if (nparts <= 2) vec(norm_bf16_vec_kernel<2, 2>);
        else if (nparts <= 4) vec(norm_bf16_vec_kernel<2, 4>);
        else vec(norm_bf16_vec_kernel<2, 8>);
    } else {
        hipLaunchKernelGGL(norm_kernel, dim3(rows), dim3(256), 0, st, m->h, part, nparts, ld_rows, gain, (bf16_t *)x_out, d, ncb,
                           m->cfg.rms_eps);
    }
    VF_LAUNCH_CHECK("norm");
    return VF_OK;
}

QkvColumns vf_qkv_columns(const vf_model *m, int layer) {
    const vf_config &c = m->cfg;
    return {layer, c.n_q_heads, c.n_kv_heads, c.head_dim, c.qkv_bias ? m->layers[layer].bqkv : nullptr, m->rope_cos, m->rope_sin,
            (bf16_t *)m->q};
}
QkvEpilogue vf_qkv_epilogue(const vf_model *m, const Batch &b, int layer, const int32_t *depth) {
    return {vf_qkv_columns(m, layer), b, depth};
}

int vf_launch_qkv_finish(const vf_model *m, const QkvEpilogue &e, const float *part, int nparts, int ld_rows, hipStream_t st) {
    const int total = e.b.total_rows * (e.hq + 2 * e.hkv) * (e.hd / 4);
    hipLaunchKernelGGL(qkv_finish_kernel, dim3(nblocks(total, 256)), dim3(256), 0, st, part, nparts, ld_rows, e);
    VF_LAUNCH_CHECK("qkv_finish");
    return VF_OK;
}

int vf_launch_swiglu(const vf_model *m, const float *part, int nparts, int rows, int ld_rows, hipStream_t st) {
    const int F = m->cfg.d_ffn, ncb = (rows + 15) >> 4;
    hipLaunchKernelGGL(swiglu_kernel, dim3(nblocks((size_t)rows * F, 256)), dim3(256), 0, st, part, nparts, ld_rows,
                       (bf16_t *)m->a, rows, F, ncb);
    VF_LAUNCH_CHECK("swiglu");
    return VF_OK;
}

int vf_launch_state_set(int32_t *state, int idx, int32_t value, hipStream_t st) {
    hipLaunchKernelGGL(state_set_kernel, dim3(1), dim3(1), 0, st, state, idx, value);
    VF_LAUNCH_CHECK("state_set");
    return VF_OK;
}
int vf_launch_state_add(int32_t *state, int idx, int32_t delta, hipStream_t st) {
    hipLaunchKernelGGL(state_add_kernel, dim3(1), dim3(1), 0, st, state, idx, delta);
    VF_LAUNCH_CHECK("state_add");
    return VF_OK;
}

namespace {
// Every thread streams 16-byte pieces at a stride of the whole grid; the xor of what it read goes to a
// word nobody reads unless it is a magic value (so the loads cannot be dropped).
__global__ __launch_bounds__(512) void stream_read_kernel(const u32x4_t *__restrict__ p, size_t n, int32_t *sink) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    u32x4_t acc = {0u, 0u, 0u, 0u};
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 7 * stride < n; i += 8 * stride) {
        u32x4_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = __builtin_nontemporal_load(p + i + j * stride);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc ^= v[j];
    }
    for (; i < n; i += stride) acc ^= __builtin_nontemporal_load(p + i);
    if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x9e3779b9u) *sink = 1;
}
}  // namespace

int vf_launch_stream_read(const vf_model *m, size_t *bytes, hipStream_t st) {
    // the packed weights sit at the start of the model's buffer, up to the rotary tables
    const size_t n = ((const char *)m->rope_cos - (const char *)m->base) / 16;
    hipLaunchKernelGGL(stream_read_kernel, dim3(1024), dim3(512), 0, st, (const u32x4_t *)m->base, n, m->scratch_i32 + 63);
    VF_LAUNCH_CHECK("stream_read");
    *bytes = n * 16;
    return VF_OK;
}

int vf_launch_kv_write(const vf_model *m, const SeqDesc &s, int layer, int t0, int n, const float *k_in,
                       const float *v_in, hipStream_t st) {
    const vf_config &c = m->cfg;
    const int total = n * c.n_kv_heads * c.head_dim;
    if (total <= 0) return VF_OK;
    if (c.dtype == VF_BF16)
        hipLaunchKernelGGL(kv_write_kernel<bf16_t>, dim3(nblocks(total, 256)), dim3(256), 0, st, s, layer, t0, n,
                           c.n_kv_heads, c.head_dim, k_in, v_in);
    else
        hipLaunchKernelGGL(kv_write_kernel<float>, dim3(nblocks(total, 256)), dim3(256), 0, st, s, layer, t0, n,
                           c.n_kv_heads, c.head_dim, k_in, v_in);
    VF_LAUNCH_CHECK("kv_write");
    return VF_OK;
}

int vf_launch_kv_read(const vf_model *m, const SeqDesc &s, int layer, int t0, int n, float *k_out, float *v_out,
                      hipStream_t st) {
    const vf_config &c = m->cfg;
    const int total = n * c.n_kv_heads * c.head_dim;
    if (total <= 0) return VF_OK;
    if (c.dtype == VF_BF16)
        hipLaunchKernelGGL(kv_read_kernel<bf16_t>, dim3(nblocks(total, 256)), dim3(256), 0, st, s, layer, t0, n,
                           c.n_kv_heads, c.head_dim, k_out, v_out);
    else
        hipLaunchKernelGGL(kv_read_kernel<float>, dim3(nblocks(total, 256)), dim3(256), 0, st, s, layer, t0, n,
                           c.n_kv_heads, c.head_dim, k_out, v_out);
    VF_LAUNCH_CHECK("kv_read");
    return VF_OK;
}

int vf_launch_tree_prep(const vf_model *m, const Batch &b, const TreeDesc &tree, hipStream_t st) {
    hipLaunchKernelGGL(tree_prep_kernel, dim3(b.n_seqs), dim3(64), 0, st, b, tree, m->tree_anc, m->tree_depth);
    VF_LAUNCH_CHECK("tree_prep");
    return VF_OK;
}

int vf_launch_kv_compact(const vf_model *m, const Batch &b, const int32_t *n_accept, const int32_t *path,
                         hipStream_t st) {
    const vf_config &c = m->cfg;
    const int total = c.n_layers * c.n_kv_heads * c.head_dim;
    if (c.dtype == VF_BF16)
        hipLaunchKernelGGL(kv_compact_kernel<bf16_t>, dim3(nblocks(total, 256), b.n_seqs), dim3(256), 0, st, b,
                           n_accept, path, c.n_layers, c.n_kv_heads, c.head_dim);
    else
        hipLaunchKernelGGL(kv_compact_kernel<float>, dim3(nblocks(total, 256), b.n_seqs), dim3(256), 0, st, b,
                           n_accept, path, c.n_layers, c.n_kv_heads, c.head_dim);
    VF_LAUNCH_CHECK("kv_compact");
    return VF_OK;
}
