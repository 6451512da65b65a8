// Precomputing the f-gram embedding layer: F(w) = A_fgram(T(w_0..w_{n-1})),
// the f-gram model's output at the last token, for every f-gram w (Section
// 3.2; Algorithm 1's training branch is the same map).  The model is a
// pre-LayerNorm causal decoder with absolute position embeddings of one row
// per position up to the longest f-gram (implementation appendix), biases on
// every linear map, exact GELU, LayerNorm epsilon 1e-5, and a final LayerNorm.
//
// Under causal attention the state of token i depends on tokens 0..i only, so
// f-grams that begin alike share the states of their common prefix: the states
// form a prefix tree, and each node of it is computed once (fgram_tree.h).  The
// paper pads the f-grams of a batch to the longest one; here nothing is padded,
// since with padding on the right the last token never sees a pad.  1M f-grams of
// length 2 or 3 with Zipf tokens (2.65M tokens) have 1.30M distinct states and a
// tree of 1.34M nodes (a prefix that is itself an f-gram is a second node where
// that f-gram sorts after a longer one).  The call took 423 ms with one row per
// token, 227 with the tree (the same bits) and takes 222 now.
//
// A chunk is a run of f-grams in sorted order with up to kChunkRows nodes: one
// row per node, first each f-gram's last token (row f for the chunk's f-th
// f-gram), then the inner nodes:
//
//   k_embed_ln   h = T[w] + P[i] (f32),  a = LN1_0(h) (bf16)
//   per layer:   [k_ln a = LN1(h)]  qkv = a Wqkv^T + b       (MFMA)
//                o = attention of each row over its path      (k_attn)
//                h += o Wo^T + b                              (MFMA, fused residual)
//                a = LN2(h);  f = GELU(a W1^T + b1)           (MFMA, fused GELU)
//                h += f W2^T + b2                             (MFMA, fused residual)
//   k_final      rows[row_id] = bf16(LNf(h of row f))
//
// After the last layer's attention only the f-grams' own rows matter, so its
// products run on those.
//
// Matrix products run on the matrix cores (gemm_bf16.h); the rest is
// bandwidth-bound and one wavefront handles one row or one f-gram.
#include "fgram_tree.h"
#include "gemm_bf16.h"

#include <algorithm>
#include <new>
#include <vector>

namespace scone {
namespace {

using gemm::bf16_to_f32;
using gemm::f32_to_bf16;

using tree::Chunk;
using tree::Node;

constexpr int kThreads = 256;
constexpr float kLnEps = 1e-5f;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// -------------------------------------------------------------- row kernels --
// One wavefront per row of d = 256 * R elements; lane holds elements
// c * 256 + lane * 4 + (0..3), c < R.

template <int R>
__device__ __forceinline__ void layer_norm_store(float (&x)[R][4], const uint16_t* __restrict__ g,
                                                 const uint16_t* __restrict__ b, int lane,
                                                 uint16_t* __restrict__ dst) {
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < R; ++c) s += (x[c][0] + x[c][1]) + (x[c][2] + x[c][3]);
    const float mean = wave_sum(s) * (1.0f / (256 * R));
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < R; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float t = x[c][e] - mean;
            q += t * t;
        }
    const float rstd = rsqrtf(wave_sum(q) * (1.0f / (256 * R)) + kLnEps);
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const int e0 = c * 256 + lane * 4;
        const u32x2 gg = *reinterpret_cast<const u32x2*>(g + e0);
        const u32x2 bb = *reinterpret_cast<const u32x2*>(b + e0);
        const float gv[4] = {bf16_to_f32(gg.x & 0xFFFFu), bf16_to_f32(gg.x >> 16),
                             bf16_to_f32(gg.y & 0xFFFFu), bf16_to_f32(gg.y >> 16)};
        const float bv[4] = {bf16_to_f32(bb.x & 0xFFFFu), bf16_to_f32(bb.x >> 16),
                             bf16_to_f32(bb.y & 0xFFFFu), bf16_to_f32(bb.y >> 16)};
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16((x[c][e] - mean) * rstd * gv[e] + bv[e]);
        *reinterpret_cast<u32x2*>(dst + e0) = u32x2{o[0] | (o[1] << 16), o[2] | (o[3] << 16)};
    }
}

// h[r] = T[token] + P[pos]; a[r] = LN(h[r]) for the nodes r < rows.
template <int R>
__global__ __launch_bounds__(kThreads) void k_embed_ln(
    const Node* __restrict__ nodes, int64_t rows, const uint16_t* __restrict__ tok_rows,
    const uint16_t* __restrict__ pos, const uint16_t* __restrict__ g,
    const uint16_t* __restrict__ b, float* __restrict__ h, uint16_t* __restrict__ a) {
    constexpr int d = 256 * R;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / 64) +
                      __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    const int32_t tok = nodes[r].tok;
    const int i = nodes[r].pos;
    const uint16_t* trow = tok_rows + (int64_t)tok * d;
    const uint16_t* prow = pos + (int64_t)i * d;
    float x[R][4];
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const int e0 = c * 256 + lane * 4;
        const u32x2 tv = *reinterpret_cast<const u32x2*>(trow + e0);
        const u32x2 pv = *reinterpret_cast<const u32x2*>(prow + e0);
        x[c][0] = bf16_to_f32(tv.x & 0xFFFFu) + bf16_to_f32(pv.x & 0xFFFFu);
        x[c][1] = bf16_to_f32(tv.x >> 16) + bf16_to_f32(pv.x >> 16);
        x[c][2] = bf16_to_f32(tv.y & 0xFFFFu) + bf16_to_f32(pv.y & 0xFFFFu);
        x[c][3] = bf16_to_f32(tv.y >> 16) + bf16_to_f32(pv.y >> 16);
        *reinterpret_cast<float4*>(h + r * d + e0) =
            make_float4(x[c][0], x[c][1], x[c][2], x[c][3]);
    }
    layer_norm_store<R>(x, g, b, lane, a + r * d);
}

// a[r] = LN(h[r]) for r < rows.
template <int R>
__global__ __launch_bounds__(kThreads) void k_ln(const float* __restrict__ h, int64_t rows,
                                                 const uint16_t* __restrict__ g,
                                                 const uint16_t* __restrict__ b,
                                                 uint16_t* __restrict__ a) {
    constexpr int d = 256 * R;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    float x[R][4];
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const float4 v = *reinterpret_cast<const float4*>(h + r * d + c * 256 + lane * 4);
        x[c][0] = v.x; x[c][1] = v.y; x[c][2] = v.z; x[c][3] = v.w;
    }
    layer_norm_store<R>(x, g, b, lane, a + r * d);
}

// rows[row_id] = bf16(LNf(h of the f-gram's last token, row f)).  Row ids
// outside [0, n_rows) raise EROW and write nothing.
template <int R>
__global__ __launch_bounds__(kThreads) void k_final(const float* __restrict__ h,
                                                    const int32_t* __restrict__ order,
                                                    int64_t n_f,
                                                    const int32_t* __restrict__ row_ids,
                                                    const uint16_t* __restrict__ g,
                                                    const uint16_t* __restrict__ b,
                                                    uint16_t* __restrict__ rows, int64_t n_rows,
                                                    unsigned* __restrict__ status) {
    constexpr int d = 256 * R;
    const int64_t f = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (f >= n_f) return;
    const int lane = threadIdx.x & 63;
    const int32_t id = row_ids[order[f]];
    if (id < 0 || id >= n_rows) {
        if (lane == 0) atomicOr(status, err_bit(SCONE_EROW));
        return;
    }
    const float* src = h + f * d;
    float x[R][4];
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const float4 v = *reinterpret_cast<const float4*>(src + c * 256 + lane * 4);
        x[c][0] = v.x; x[c][1] = v.y; x[c][2] = v.z; x[c][3] = v.w;
    }
    layer_norm_store<R>(x, g, b, lane, rows + (int64_t)id * d);
}

// ---------------------------------------------------------------- attention --
// One wavefront per node.  A pass covers 512 columns of the model: lane holds
// 8 consecutive columns, so a head of dh columns spans dh / 8 lanes and its dot
// products are reduced over that many lanes.  qkv row r = [q | k | v], each d
// wide; o row r = concatenated heads.  The node's query attends to the keys of
// its path (its ancestors, then itself), whose length N is the same for the
// whole wavefront.
template <int LPH, int N>  // lanes per head (dh / 8), path length
__device__ __forceinline__ void attend(const uint16_t* __restrict__ qkv,
                                       uint16_t* __restrict__ o, int64_t r,
                                       const int64_t (&path)[SCONE_MAX_FGRAM_LEN], int d,
                                       float scale, int lane) {
    const int64_t ld = 3 * (int64_t)d;
    for (int c0 = 0; c0 < d; c0 += 512) {
        const int col = c0 + lane * 8;
        const u32x4 qq = *reinterpret_cast<const u32x4*>(qkv + r * ld + col);
        u32x4 kk[N], vv[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint16_t* row = qkv + path[j] * ld + col;
            kk[j] = *reinterpret_cast<const u32x4*>(row + d);
            vv[j] = *reinterpret_cast<const u32x4*>(row + 2 * d);
        }
        float s[N];
        float mx = -3.0e38f;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            float t = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                t += bf16_to_f32(qq[e] & 0xFFFFu) * bf16_to_f32(kk[j][e] & 0xFFFFu);
                t += bf16_to_f32(qq[e] >> 16) * bf16_to_f32(kk[j][e] >> 16);
            }
#pragma unroll
            for (int w = LPH / 2; w >= 1; w >>= 1) t += __shfl_xor(t, w);
            s[j] = t * scale;
            mx = fmaxf(mx, s[j]);
        }
        float den = 0.f;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            s[j] = __expf(s[j] - mx);
            den += s[j];
        }
        const float inv = 1.0f / den;
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const float p = s[j] * inv;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[2 * e] += p * bf16_to_f32(vv[j][e] & 0xFFFFu);
                acc[2 * e + 1] += p * bf16_to_f32(vv[j][e] >> 16);
            }
        }
        u32x4 ov;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            ov[e] = f32_to_bf16(acc[2 * e]) | (f32_to_bf16(acc[2 * e + 1]) << 16);
        *reinterpret_cast<u32x4*>(o + r * (int64_t)d + col) = ov;
    }
}

// Attention of the nodes r < rows.  Workgroups are renumbered so that each XCD
// takes a contiguous run of rows: sorted neighbours share ancestors, whose keys
// and values then come from that XCD's L2.
template <int LPH>
__global__ __launch_bounds__(kThreads) void k_attn(const uint16_t* __restrict__ qkv,
                                                   uint16_t* __restrict__ o, int64_t rows, int d,
                                                   float scale, const Node* __restrict__ nodes) {
    const int64_t per = gridDim.x / 8, b = blockIdx.x;
    const int64_t blk = b < per * 8 ? (b % 8) * per + b / 8 : b;
    const int64_t r = blk * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    const Node nd = nodes[r];
    int64_t path[SCONE_MAX_FGRAM_LEN];
#pragma unroll
    for (int j = 0; j < SCONE_MAX_FGRAM_LEN; ++j)
        path[j] = j < nd.pos ? nd.up[j < SCONE_MAX_FGRAM_LEN - 1 ? j : 0] : r;
    switch (nd.pos) {  // wave-uniform, 0..6
        case 0: attend<LPH, 1>(qkv, o, r, path, d, scale, lane); break;
        case 1: attend<LPH, 2>(qkv, o, r, path, d, scale, lane); break;
        case 2: attend<LPH, 3>(qkv, o, r, path, d, scale, lane); break;
        case 3: attend<LPH, 4>(qkv, o, r, path, d, scale, lane); break;
        case 4: attend<LPH, 5>(qkv, o, r, path, d, scale, lane); break;
        case 5: attend<LPH, 6>(qkv, o, r, path, d, scale, lane); break;
        default: attend<LPH, 7>(qkv, o, r, path, d, scale, lane); break;
    }
}

hipError_t attention(const uint16_t* qkv, uint16_t* o, int64_t rows, int d, int dh, float scale,
                     const Node* nodes, hipStream_t st) {
    const dim3 grid((unsigned)((rows + 3) / 4)), block(kThreads);
    if (dh == 64)
        hipLaunchKernelGGL(k_attn<8>, grid, block, 0, st, qkv, o, rows, d, scale, nodes);
    else
        hipLaunchKernelGGL(k_attn<16>, grid, block, 0, st, qkv, o, rows, d, scale, nodes);
    return hipGetLastError();
}

// ------------------------------------------------------------------ layout --

constexpr int kPerLayer = 12;

int64_t align_up(int64_t x) { return (x + 127) & ~(int64_t)127; }

// Element counts of the parameters in packing order.
std::vector<int64_t> param_sizes(int64_t d, int64_t d_ff, int n_layers, int max_len) {
    std::vector<int64_t> s;
    s.push_back((int64_t)max_len * d);  // pos
    for (int l = 0; l < n_layers; ++l) {
        const int64_t per[kPerLayer] = {d,        d,    3 * d * d, 3 * d, d * d,    d,
                                        d,        d,    d_ff * d,  d_ff,  d * d_ff, d};
        for (int64_t v : per) s.push_back(v);
    }
    s.push_back(d);  // lnf_g
    s.push_back(d);  // lnf_b
    return s;
}

bool dims_ok(int32_t d, int32_t n_heads, int32_t d_ff, int32_t n_layers, int32_t max_len) {
    if (d <= 0 || d % 512 != 0 || d > 4096) return false;
    if (n_heads <= 0 || d % n_heads != 0) return false;
    const int dh = d / n_heads;
    if (dh != 64 && dh != 128) return false;
    if (d_ff <= 0 || d_ff % 128 != 0 || d_ff > 65536) return false;
    if (n_layers < 0 || n_layers > 1024) return false;
    if (max_len < 2 || max_len > SCONE_MAX_FGRAM_LEN) return false;
    return true;
}

struct Weights {
    const uint16_t* pos;
    struct Layer {
        const uint16_t *ln1_g, *ln1_b, *w_qkv, *b_qkv, *w_o, *b_o, *ln2_g, *ln2_b, *w_fc1,
            *b_fc1, *w_fc2, *b_fc2;
    };
    std::vector<Layer> layers;
    const uint16_t *lnf_g, *lnf_b;
};

Weights bind_weights(const uint16_t* blob, int64_t d, int64_t d_ff, int n_layers, int max_len) {
    const std::vector<int64_t> sz = param_sizes(d, d_ff, n_layers, max_len);
    std::vector<const uint16_t*> p;
    int64_t off = 0;
    for (int64_t s : sz) {
        p.push_back(blob + off);
        off += align_up(s);
    }
    Weights w;
    size_t k = 0;
    w.pos = p[k++];
    for (int l = 0; l < n_layers; ++l) {
        Weights::Layer L;
        L.ln1_g = p[k++]; L.ln1_b = p[k++]; L.w_qkv = p[k++]; L.b_qkv = p[k++];
        L.w_o = p[k++];   L.b_o = p[k++];   L.ln2_g = p[k++]; L.ln2_b = p[k++];
        L.w_fc1 = p[k++]; L.b_fc1 = p[k++]; L.w_fc2 = p[k++]; L.b_fc2 = p[k++];
        w.layers.push_back(L);
    }
    w.lnf_g = p[k++];
    w.lnf_b = p[k++];
    return w;
}

// ------------------------------------------------------------------ driver --

struct Buffers {
    Node* nodes;
    float* h;
    uint16_t *a, *qkv, *f;
};

// One chunk whose nodes are in B.nodes; `order` holds its f-grams.
template <int R>
hipError_t run_chunk(const Weights& w, const int32_t* order, const Chunk& c,
                     const uint16_t* tok_rows, int d_ff, int n_heads, const int32_t* row_ids,
                     uint16_t* rows, int64_t n_rows, const Buffers& B, unsigned* status,
                     hipStream_t st) {
    constexpr int d = 256 * R;
    const int64_t M = c.rows, n_f = c.n_f;
    const unsigned g_rows = (unsigned)((M + 3) / 4);
    const unsigned g_f = (unsigned)((n_f + 3) / 4);
    const int n_layers = (int)w.layers.size();
    const uint16_t* ln_g = n_layers ? w.layers[0].ln1_g : w.lnf_g;
    const uint16_t* ln_b = n_layers ? w.layers[0].ln1_b : w.lnf_b;
    hipLaunchKernelGGL(k_embed_ln<R>, dim3(g_rows), dim3(kThreads), 0, st, B.nodes, M, tok_rows,
                       w.pos, ln_g, ln_b, B.h, B.a);
    const int dh = d / n_heads;
    const float scale = 1.0f / sqrtf((float)dh);
    hipError_t e = hipGetLastError();
    for (int l = 0; l < n_layers && e == hipSuccess; ++l) {
        const Weights::Layer& L = w.layers[l];
        if (l > 0)
            hipLaunchKernelGGL(k_ln<R>, dim3(g_rows), dim3(kThreads), 0, st, B.h, M, L.ln1_g,
                               L.ln1_b, B.a);
        e = gemm::launch<gemm::kBias>(B.a, L.w_qkv, L.b_qkv, B.qkv, 3 * d, (int)M, 3 * d, d, st);
        if (e != hipSuccess) break;
        // Only the f-grams' last tokens reach F, so from the last layer's
        // attention on, the first n_f rows are all that is computed.
        const int64_t Mr = l == n_layers - 1 ? n_f : M;
        const unsigned g_r = (unsigned)((Mr + 3) / 4);
        // attention output overwrites a (its input to the qkv product is consumed)
        e = attention(B.qkv, B.a, Mr, d, dh, scale, B.nodes, st);
        if (e != hipSuccess) break;
        e = gemm::launch<gemm::kResid>(B.a, L.w_o, L.b_o, B.h, d, (int)Mr, d, d, st);
        if (e != hipSuccess) break;
        hipLaunchKernelGGL(k_ln<R>, dim3(g_r), dim3(kThreads), 0, st, B.h, Mr, L.ln2_g, L.ln2_b,
                           B.a);
        e = gemm::launch<gemm::kGelu>(B.a, L.w_fc1, L.b_fc1, B.f, d_ff, (int)Mr, d_ff, d, st);
        if (e != hipSuccess) break;
        e = gemm::launch<gemm::kResid>(B.f, L.w_fc2, L.b_fc2, B.h, d, (int)Mr, d, d_ff, st);
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_final<R>, dim3(g_f), dim3(kThreads), 0, st, B.h, order, n_f, row_ids,
                       w.lnf_g, w.lnf_b, rows, n_rows, status);
    return hipGetLastError();
}

// The call's scratch, carved from one workspace: the tree (fgram_tree.h) and the
// activations of one chunk.
struct ModelLayout {
    tree::Layout tree;
    size_t h, a, qkv, f, total;
};

ModelLayout model_layout(int64_t n, int max_len, int64_t d, int64_t d_ff) {
    ModelLayout l{};
    l.tree = tree::layout(n, max_len);
    size_t off = l.tree.total;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = (off + bytes + 255) & ~(size_t)255;
        return at;
    };
    const int64_t rows = l.tree.max_rows;
    // matrix-product inputs (a, f) are readable up to a whole 256-row tile
    const int64_t padded = (rows + 255) / 256 * 256;
    l.h = take((size_t)(rows * d) * 4);
    l.a = take((size_t)(padded * d) * 2);
    l.qkv = take((size_t)(rows * 3 * d) * 2);
    l.f = take((size_t)(padded * d_ff) * 2);
    l.total = off;
    return l;
}

typedef hipError_t (*ChunkFn)(const Weights&, const int32_t*, const Chunk&, const uint16_t*, int,
                              int, const int32_t*, uint16_t*, int64_t, const Buffers&, unsigned*,
                              hipStream_t);

ChunkFn chunk_fn(int d) {
    switch (d / 256) {
        case 2: return run_chunk<2>;
        case 4: return run_chunk<4>;
        case 6: return run_chunk<6>;
        case 8: return run_chunk<8>;
        case 10: return run_chunk<10>;
        case 12: return run_chunk<12>;
        case 14: return run_chunk<14>;
        case 16: return run_chunk<16>;
        default: return nullptr;
    }
}

}  // namespace
}  // namespace scone

extern "C" int scone_fgram_model_layout(int32_t d, int32_t n_heads, int32_t d_ff,
                                        int32_t n_layers, int32_t max_len, int64_t* offsets,
                                        int64_t* n_params, int64_t* total_elems) {
    using namespace scone;
    if (!dims_ok(d, n_heads, d_ff, n_layers, max_len)) return SCONE_EINVAL;
    const std::vector<int64_t> sz = param_sizes(d, d_ff, n_layers, max_len);
    int64_t off = 0;
    for (size_t k = 0; k < sz.size(); ++k) {
        if (offsets) offsets[k] = off;
        off += align_up(sz[k]);
    }
    if (n_params) *n_params = (int64_t)sz.size();
    if (total_elems) *total_elems = off;
    return SCONE_OK;
}

extern "C" int64_t scone_fgram_model_workspace(int64_t n, int32_t max_len, int32_t d,
                                               int32_t n_heads, int32_t d_ff) {
    using namespace scone;
    if (!dims_ok(d, n_heads, d_ff, 0, max_len) || n < 0 || n > 0x7fffffffLL) return -1;
    return (int64_t)model_layout(n, max_len, d, d_ff).total;
}

namespace scone {
namespace {

// Everything after the argument checks, in a workspace of model_layout's size.
int run_model(const int32_t* fgrams, const int32_t* lengths, const int32_t* row_ids, int64_t n,
              int32_t max_len, const uint16_t* tok_rows, int64_t vocab, const uint16_t* params,
              int32_t d, int32_t n_heads, int32_t d_ff, int32_t n_layers, uint16_t* rows,
              int64_t n_rows, uint8_t* ws, hipStream_t st) {
    const ChunkFn fn = chunk_fn(d);
    if (!fn) return SCONE_EINVAL;
    const ModelLayout lay = model_layout(n, max_len, d, d_ff);
    const tree::Builder tb{fgrams, lengths, n, max_len, vocab, ws, lay.tree, n_layers == 0, st};
    std::vector<Chunk> chunks;
    unsigned bits = 0;
    const int rc = tb.build(chunks, bits);
    if (rc != SCONE_OK) return rc;
    if (bits & err_bit(SCONE_ELEN)) return SCONE_ELEN;
    const Weights w = bind_weights(params, d, d_ff, n_layers, max_len);
    Buffers B;
    B.nodes = tb.nodes();
    B.h = reinterpret_cast<float*>(ws + lay.h);
    B.a = reinterpret_cast<uint16_t*>(ws + lay.a);
    B.qkv = reinterpret_cast<uint16_t*>(ws + lay.qkv);
    B.f = reinterpret_cast<uint16_t*>(ws + lay.f);
    for (const Chunk& c : chunks) {
        if (tb.fill_nodes(c) != hipSuccess ||
            fn(w, tb.order() + c.first, c, tok_rows, d_ff, n_heads, row_ids, rows, n_rows, B,
               tb.status(), st) != hipSuccess)
            return SCONE_EHIP;
    }
    unsigned hs = 0;
    if (hipMemcpyAsync(&hs, tb.status(), sizeof(unsigned), hipMemcpyDeviceToHost, st) !=
            hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return SCONE_EHIP;
    return hs ? code_from_bits(hs) : SCONE_OK;
}

}  // namespace
}  // namespace scone

extern "C" int scone_fgram_model_forward_in(const int32_t* fgrams, const int32_t* lengths,
                                            const int32_t* row_ids, int64_t n, int32_t max_len,
                                            const void* tok_rows, int64_t vocab,
                                            const void* params, int32_t d, int32_t n_heads,
                                            int32_t d_ff, int32_t n_layers, void* rows,
                                            int64_t n_rows, void* workspace,
                                            int64_t workspace_bytes, void* stream) {
    using namespace scone;
    if (!dims_ok(d, n_heads, d_ff, n_layers, max_len)) return SCONE_EINVAL;
    if (n < 0 || vocab <= 0 || n_rows < 0 || n > 0x7fffffffLL) return SCONE_EINVAL;
    if (n == 0) return SCONE_OK;
    if (!fgrams || !lengths || !row_ids || !tok_rows || !params || !rows) return SCONE_EINVAL;
    if (((uintptr_t)tok_rows | (uintptr_t)params | (uintptr_t)rows) % 16 != 0)
        return SCONE_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    void* own = nullptr;
    int rc;
    try {
        // Rows are written chunk by chunk while later chunks still read the
        // f-grams, lengths, row ids and parameters: `rows` may share memory
        // with none of them (tok_rows may lie inside it, as documented), and
        // the workspace with nothing at all.
        const size_t need = model_layout(n, max_len, d, d_ff).total;
        int64_t p_elems = 0;
        for (int64_t e : param_sizes(d, d_ff, n_layers, max_len)) p_elems += align_up(e);
        const void* buf[6] = {fgrams, lengths, row_ids, params, rows, tok_rows};
        const int64_t len[6] = {span_bytes(n, 4 * (int64_t)max_len), span_bytes(n, 4),
                                span_bytes(n, 4), span_bytes(p_elems, 2),
                                span_bytes(n_rows, 2 * (int64_t)d),
                                span_bytes(vocab, 2 * (int64_t)d)};
        for (int i = 0; i < 4; ++i)
            if (overlaps(rows, len[4], buf[i], len[i])) return SCONE_EINVAL;
        if (workspace) {
            if (workspace_bytes < 0 || (uint64_t)workspace_bytes < need ||
                (uintptr_t)workspace % 256 != 0)
                return SCONE_EINVAL;
            for (int i = 0; i < 6; ++i)
                if (overlaps(workspace, (int64_t)need, buf[i], len[i])) return SCONE_EINVAL;
        } else {
            if (hipMalloc(&own, need) != hipSuccess) {
                (void)hipGetLastError();
                return SCONE_ENOMEM;
            }
            workspace = own;
        }
        rc = run_model(fgrams, lengths, row_ids, n, max_len,
                       static_cast<const uint16_t*>(tok_rows), vocab,
                       static_cast<const uint16_t*>(params), d, n_heads, d_ff, n_layers,
                       static_cast<uint16_t*>(rows), n_rows, static_cast<uint8_t*>(workspace),
                       st);
    } catch (const std::bad_alloc&) {
        rc = SCONE_ENOMEM;
    }
    // On an error kernels may still be running; the scratch stays until they end.
    if (rc != SCONE_OK) (void)hipStreamSynchronize(st);
    if (own) (void)hipFree(own);
    return rc;
}

extern "C" int scone_fgram_model_forward(const int32_t* fgrams, const int32_t* lengths,
                                         const int32_t* row_ids, int64_t n, int32_t max_len,
                                         const void* tok_rows, int64_t vocab, const void* params,
                                         int32_t d, int32_t n_heads, int32_t d_ff,
                                         int32_t n_layers, void* rows, int64_t n_rows,
                                         void* stream) {
    return scone_fgram_model_forward_in(fgrams, lengths, row_ids, n, max_len, tok_rows, vocab,
                                        params, d, n_heads, d_ff, n_layers, rows, n_rows, nullptr,
                                        0, stream);
}
