// HBM-bound streaming kernels of the hot path: column statistics (LayerNorm gain/offset and dense-bias
// gradients), embedding-table gradients (per-example segment reduction for the norms, stable radix sort
// plus ordered segment sums for the clip-weighted scatter), and the ordered reduction of partial buffers.
//
// Roofline: HBM.  Each kernel reads its bf16 (or fp32) inputs exactly once; algorithmic bytes per
// example are T*d*elem for every tensor read.  Threads own 4 consecutive columns (8-byte bf16 / 16-byte
// fp32 loads), a wave covers 256 consecutive columns of one row, so every row read is fully coalesced.
#include "dp_common.h"

namespace {

// ------------------------------------------------------------------------------------------------
// element access: VW consecutive elements starting at element index `idx`
// ------------------------------------------------------------------------------------------------
// (non-temporal: every input byte of these kernels is read once and by one workgroup)
typedef uint32_t rw_u32x2 __attribute__((ext_vector_type(2)));
// The same in two steps, for loads that stay in flight: raw bits (RawVec), then values.
template <bool BF16, int VW>
struct RawVec {
    uint32_t w[BF16 ? VW / 2 : VW];
};
typedef const __attribute__((address_space(1))) char* rw_global;
template <bool BF16, int VW>
__device__ __forceinline__ RawVec<BF16, VW> load_raw(rw_global row, uint32_t byte) {  // row: the same for the wave
    RawVec<BF16, VW> r;
    if constexpr (BF16) {
        static_assert(VW == 4, "bf16 rows are read four elements at a time");
        const rw_u32x2 t = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) rw_u32x2*>(row + byte));
        r.w[0] = t[0]; r.w[1] = t[1];
    } else if constexpr (VW == 4) {
        const f32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) f32x4_t*>(row + byte));
#pragma unroll
        for (int k = 0; k < 4; ++k) r.w[k] = __float_as_uint(t[k]);
    } else {
        r.w[0] = __float_as_uint(__builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) float*>(row + byte)));
    }
    return r;
}
template <bool BF16, int VW>
__device__ __forceinline__ float raw_value(const RawVec<BF16, VW>& r, int k) {
    if constexpr (BF16) return k & 1 ? dp_bf16_hi(r.w[k >> 1]) : dp_bf16_lo(r.w[k >> 1]);
    else return __uint_as_float(r.w[k]);
}
template <bool BF16, int VW>
__device__ __forceinline__ void load_vec(const void* __restrict__ base, size_t idx, float out[VW]) {
    if constexpr (BF16) {
        static_assert(VW == 4, "bf16 rows are read four elements at a time");
        const rw_u32x2 w =
            __builtin_nontemporal_load(reinterpret_cast<const rw_u32x2*>(reinterpret_cast<const uint16_t*>(base) + idx));
        out[0] = dp_bf16_lo(w[0]);
        out[1] = dp_bf16_hi(w[0]);
        out[2] = dp_bf16_lo(w[1]);
        out[3] = dp_bf16_hi(w[1]);
    } else if constexpr (VW == 4) {
        const f32x4_t w = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(reinterpret_cast<const float*>(base) + idx));
        out[0] = w[0]; out[1] = w[1]; out[2] = w[2]; out[3] = w[3];
    } else {
        out[0] = __builtin_nontemporal_load(reinterpret_cast<const float*>(base) + idx);
    }
}

// ------------------------------------------------------------------------------------------------
// column statistics, per example (pass 1)
//   grid (B, ceil(d / (64*VW))), 256 threads = 4 row groups x 64 column lanes
// ------------------------------------------------------------------------------------------------
// Up to COL_MAX_BATCH same-shaped layers per launch (blockIdx.z = layer): the 48 LayerNorms of the model are 2 launches
// per pass instead of 48, and their per-example partials meet in one ordered reduction.
constexpr int COL_MAX_BATCH = 32;
struct ColBatch {
    const void* X[COL_MAX_BATCH];
    const void* G[COL_MAX_BATCH];
};
struct ColOut {
    float* out_x[COL_MAX_BATCH];
    float* out_1[COL_MAX_BATCH];
};
struct ColKeep {
    float* keep[COL_MAX_BATCH];  // per layer: [B][2][d] fp32, the per-example column statistics themselves
};

// out: direct (one layer, one column block): sqnorms, "+="; otherwise partials [B][layers * J], stored.
// KEEP: the statistics of example i (sum_t g x and sum_t g per column: its LayerNorm gain / offset gradient) are also
// written to ck.keep[layer][i], so that pass 2 can weight and add 8 KB per example instead of reading X and G again.
template <bool BF16, int VW, bool USE_X, bool USE_1, bool KEEP>
__global__ __launch_bounds__(256) void colstat_sqnorms_kernel(ColBatch cb, ColKeep ck, int T, int d, float* __restrict__ out,
                                                              int J, int direct) {
    __shared__ float red[4][64][2 * VW];
    __shared__ float wred[4];
    const void* __restrict__ X = cb.X[blockIdx.z];
    const void* __restrict__ G = cb.G[blockIdx.z];
    const int i = blockIdx.x;
    const int lane = threadIdx.x & 63, tg = threadIdx.x >> 6;
    const int col = (blockIdx.y * 64 + lane) * VW;
    float sx[VW], s1[VW];
#pragma unroll
    for (int k = 0; k < VW; ++k) sx[k] = s1[k] = 0.f;
    if (col < d) {
        const size_t base = (size_t)i * T * d + col;
#pragma unroll 4
        for (int t = tg; t < T; t += 4) {
            float g[VW];
            load_vec<BF16, VW>(G, base + (size_t)t * d, g);
            if constexpr (USE_X) {
                float x[VW];
                load_vec<BF16, VW>(X, base + (size_t)t * d, x);
#pragma unroll
                for (int k = 0; k < VW; ++k) sx[k] += g[k] * x[k];
            }
#pragma unroll
            for (int k = 0; k < VW; ++k) s1[k] += g[k];
        }
    }
#pragma unroll
    for (int k = 0; k < VW; ++k) {
        red[tg][lane][k] = sx[k];
        red[tg][lane][VW + k] = s1[k];
    }
    __syncthreads();
    float val = 0.f;
    float sv[2 * VW];
    if (tg == 0) {
#pragma unroll
        for (int k = 0; k < 2 * VW; ++k) {
            sv[k] = (red[0][lane][k] + red[1][lane][k]) + (red[2][lane][k] + red[3][lane][k]);
            const bool on = k < VW ? USE_X : USE_1;
            if (on) val += sv[k] * sv[k];
        }
    }
    const float tot = dp_block_sum<256>(val, wred);
    if (threadIdx.x == 0) {
        if (direct) out[i] += tot;
        else out[((size_t)i * gridDim.z + blockIdx.z) * J + blockIdx.y] = tot;
    }
    // The kept statistics go out last: a store ahead of the reduction's barrier would make every workgroup wait for it.
    if constexpr (KEEP) {
        if (tg == 0 && col < d) {
            float* __restrict__ kp = ck.keep[blockIdx.z] + (size_t)i * 2 * d + col;
            if constexpr (VW == 4) {  // d % 4 == 0 and a 16-byte aligned buffer are checked at the API
                __builtin_nontemporal_store(f32x4_t{sv[0], sv[1], sv[2], sv[3]}, reinterpret_cast<f32x4_t*>(kp));
                __builtin_nontemporal_store(f32x4_t{sv[4], sv[5], sv[6], sv[7]}, reinterpret_cast<f32x4_t*>(kp + d));
            } else {
#pragma unroll
                for (int k = 0; k < VW; ++k) {
                    kp[k] = sv[k];
                    kp[d + k] = sv[VW + k];
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// clip-weighted column sums (pass 2)
//   grid (R, ceil(d / (64*VW))): WG r reduces rows [r*rows_per, (r+1)*rows_per) of the B*T rows
//   partial layout: part[layer][r][0][d] = sum c g x,  part[layer][r][1][d] = sum c g   (blockIdx.z = layer)
// ------------------------------------------------------------------------------------------------
template <bool BF16, int VW, bool USE_X>
// (the clip factors come precomputed: forming them here, a square root and a division per row and thread, cost 2 %)
__global__ __launch_bounds__(256) void colstat_sums_kernel(ColBatch cb, const float* __restrict__ c, int T, int d,
                                                           long nrows, int rows_per, float* __restrict__ part) {
    __shared__ float red[4][64][2 * VW];
    const void* __restrict__ X = cb.X[blockIdx.z];
    const void* __restrict__ G = cb.G[blockIdx.z];
    const int lane = threadIdx.x & 63, tg = threadIdx.x >> 6;
    const int col = (blockIdx.y * 64 + lane) * VW;
    const long r0 = (long)blockIdx.x * rows_per;
    const long r1 = r0 + rows_per < nrows ? r0 + rows_per : nrows;
    float sx[VW], s1[VW];
#pragma unroll
    for (int k = 0; k < VW; ++k) sx[k] = s1[k] = 0.f;
    if (col < d) {
#pragma unroll 4
        for (long r = r0 + tg; r < r1; r += 4) {
            const float w = c[r / T];
            float g[VW];
            load_vec<BF16, VW>(G, (size_t)r * d + col, g);
            if constexpr (USE_X) {
                float x[VW];
                load_vec<BF16, VW>(X, (size_t)r * d + col, x);
#pragma unroll
                for (int k = 0; k < VW; ++k) sx[k] += w * (g[k] * x[k]);
            }
#pragma unroll
            for (int k = 0; k < VW; ++k) s1[k] += w * g[k];
        }
    }
#pragma unroll
    for (int k = 0; k < VW; ++k) {
        red[tg][lane][k] = sx[k];
        red[tg][lane][VW + k] = s1[k];
    }
    __syncthreads();
    if (tg == 0 && col < d) {
        float* p = part + ((size_t)blockIdx.z * gridDim.x + blockIdx.x) * 2 * d;
#pragma unroll
        for (int k = 0; k < VW; ++k) {
            p[col + k] = (red[0][lane][k] + red[1][lane][k]) + (red[2][lane][k] + red[3][lane][k]);
            p[d + col + k] = (red[0][lane][VW + k] + red[1][lane][VW + k]) + (red[2][lane][VW + k] + red[3][lane][VW + k]);
        }
    }
}

// Pass 2 from kept per-example statistics: out_x[j] += sum_i c_i keep[i][0][j], out_1[j] += sum_i c_i keep[i][1][j].
// grid (ceil(2d / 256), layers); 256 threads = 64 float4 columns x 4 example groups; group g adds the examples
// i = g, g+4, ... in ascending order, the four group sums are added as (0+1)+(2+3): fixed order.
__global__ __launch_bounds__(256) void kept_sums_kernel(ColKeep ck, ColOut co, const float* __restrict__ c, int B, int d) {
    __shared__ float4 red[4][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int n4 = 2 * d / 4, d4 = d / 4;
    const int j = blockIdx.x * 64 + lane;
    const float4* __restrict__ src = reinterpret_cast<const float4*>(ck.keep[blockIdx.y]);
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    if (j < n4) {
        int i = g;
        for (; i + 28 < B; i += 32) {
            float4 p[8];
            float w[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                p[u] = src[(size_t)(i + 4 * u) * n4 + j];
                w[u] = c[i + 4 * u];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                t.x += w[u] * p[u].x; t.y += w[u] * p[u].y; t.z += w[u] * p[u].z; t.w += w[u] * p[u].w;
            }
        }
        for (; i < B; i += 4) {
            const float4 p = src[(size_t)i * n4 + j];
            const float w = c[i];
            t.x += w * p.x; t.y += w * p.y; t.z += w * p.z; t.w += w * p.w;
        }
    }
    red[g][lane] = t;
    __syncthreads();
    if (g == 0 && j < n4) {
        const float4 a = red[0][lane], b = red[1][lane], e = red[2][lane], f = red[3][lane];
        float4* dst = j < d4 ? reinterpret_cast<float4*>(co.out_x[blockIdx.y]) + j
                             : reinterpret_cast<float4*>(co.out_1[blockIdx.y]) + (j - d4);
        float4 o = *dst;
        o.x += (a.x + b.x) + (e.x + f.x);
        o.y += (a.y + b.y) + (e.y + f.y);
        o.z += (a.z + b.z) + (e.z + f.z);
        o.w += (a.w + b.w) + (e.w + f.w);
        *dst = o;
    }
}

// out[j] += sum_{r<R} part[r*stride + j], r ascending (fixed order)
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* __restrict__ part, int R, size_t stride,
                                                              size_t n, float* __restrict__ out) {
    const size_t j = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    float t = 0.f;
    for (int r = 0; r < R; ++r) t += part[(size_t)r * stride + j];
    out[j] += t;
}

__global__ __launch_bounds__(256) void reduce_partials_vec4_kernel(const float4* __restrict__ part, int R,
                                                                   size_t stride4, size_t n4,
                                                                   float4* __restrict__ out) {
    const size_t j = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= n4) return;
    float4 o = out[j];
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    int r = 0;
    // eight independent 16-byte loads in flight per thread; the additions keep the order r = 0, 1, 2, ...
    for (; r + 8 <= R; r += 8) {
        float4 p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = part[(size_t)(r + u) * stride4 + j];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            t.x += p[u].x; t.y += p[u].y; t.z += p[u].z; t.w += p[u].w;
        }
    }
    for (; r < R; ++r) {
        const float4 p = part[(size_t)r * stride4 + j];
        t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
    }
    o.x += t.x; o.y += t.y; o.z += t.z; o.w += t.w;
    out[j] = o;
}

// Few outputs, many partials (column sums): 256 threads = 64 float4 columns x 4 partial groups.  Group g adds
// the partials r = g, g+4, g+8, ... in ascending order; the four group sums are added as (0+1)+(2+3): fixed order.
__global__ __launch_bounds__(256) void reduce_partials_tall_kernel(const float4* __restrict__ part, int R,
                                                                   size_t stride4, size_t n4,
                                                                   float4* __restrict__ out) {
    __shared__ float4 red[4][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const size_t j = (size_t)blockIdx.x * 64 + lane;
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    if (j < n4) {
        int r = g;
        for (; r + 28 < R; r += 32) {
            float4 p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = part[(size_t)(r + 4 * u) * stride4 + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                t.x += p[u].x; t.y += p[u].y; t.z += p[u].z; t.w += p[u].w;
            }
        }
        for (; r < R; r += 4) {
            const float4 p = part[(size_t)r * stride4 + j];
            t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
        }
    }
    red[g][lane] = t;
    __syncthreads();
    if (g == 0 && j < n4) {
        const float4 a = red[0][lane], b = red[1][lane], c = red[2][lane], d = red[3][lane];
        float4 o = out[j];
        o.x += (a.x + b.x) + (c.x + d.x);
        o.y += (a.y + b.y) + (c.y + d.y);
        o.z += (a.z + b.z) + (c.z + d.z);
        o.w += (a.w + b.w) + (c.w + d.w);
        out[j] = o;
    }
}

// The two column-sum vectors of every layer's partial buffer [R][2][d] in one launch: columns j < d4 go to out_x, the
// others to out_1 (same order of additions as reduce_partials_tall_kernel).
__global__ __launch_bounds__(256) void reduce_partials_pair_kernel(const float4* __restrict__ part, int R, size_t d4,
                                                                   ColOut co) {
    __shared__ float4 red[4][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const size_t j = (size_t)blockIdx.x * 64 + lane, n4 = 2 * d4;
    part += (size_t)blockIdx.y * R * n4;  // blockIdx.y = layer
    float4* __restrict__ out_x = reinterpret_cast<float4*>(co.out_x[blockIdx.y]);
    float4* __restrict__ out_1 = reinterpret_cast<float4*>(co.out_1[blockIdx.y]);
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    if (j < n4) {
        int r = g;
        for (; r + 28 < R; r += 32) {
            float4 p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = part[(size_t)(r + 4 * u) * n4 + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                t.x += p[u].x; t.y += p[u].y; t.z += p[u].z; t.w += p[u].w;
            }
        }
        for (; r < R; r += 4) {
            const float4 p = part[(size_t)r * n4 + j];
            t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
        }
    }
    red[g][lane] = t;
    __syncthreads();
    if (g == 0 && j < n4) {
        const float4 a = red[0][lane], b = red[1][lane], c = red[2][lane], e = red[3][lane];
        float4* dst = j < d4 ? out_x + j : out_1 + (j - d4);
        float4 o = *dst;
        o.x += (a.x + b.x) + (c.x + e.x);
        o.y += (a.y + b.y) + (c.y + e.y);
        o.z += (a.z + b.z) + (c.z + e.z);
        o.w += (a.w + b.w) + (c.w + e.w);
        *dst = o;
    }
}

// ------------------------------------------------------------------------------------------------
// embedding, per-example norms (pass 1): one workgroup per example and ncb blocks of 64*VW columns; `parts` waves (as many as there
// are pieces of EMB_PIECE positions, up to 8 or 16 waves in all) share the example's positions in a column block.
// The workgroup ranks the T ids (stable counting rank in LDS: every key, the id above the position, against all others), then
// every wave walks its run of sorted positions, emb_ahead rows in flight, adding up rows of equal id.  What the walk decides by
// is the same for the wave: row addresses and run ends are formed 64 positions at a time, one a lane, and read back as scalars
// (two LDS reads and 34 vector instructions a row, the ends as selects, kept short examples from the memory's rate: T = 128,
// d = 2,048, B = 514 62 -> 56 us; T = 64, B = 400 26 -> 22).  Runs that are complete inside a wave are squared there; the sums of
// a wave's first and last run go to LDS, where they are joined across the waves, column by column.
// One wave walking all positions of its columns was a chain of T / 8 round trips: B = 23, T = 375, d = 832: 61 -> 23 us;
// B = 512, T = 128, d = 1024 (134 MB): 31 + 5 -> 28.  Waves without positions would only make the joining of the parts longer: T = 16,
// d = 256, B = 4 12 us with 16 waves, 6 with 1; B = 514 16 | 7.
// ------------------------------------------------------------------------------------------------
// Rows in flight of a wave; without runs to form, position rows of B = 256, T = 128, d = 1,024 take 12.6 us with 8 and 11.4 with 16.
constexpr int emb_ahead(bool distinct) { return distinct ? 16 : 8; }
constexpr int EMB_PIECE = 16;  // positions that are worth a wave

// EMB_WAVES: the most waves that a launch may have; it has ncb * parts.
template <bool BF16, int VW, bool DISTINCT, int EMB_WAVES>
__global__ __launch_bounds__(64 * EMB_WAVES) void embedding_sqnorms_kernel(const int32_t* __restrict__ ids,
                                                                           const void* __restrict__ G, int T, int d, int V, int ncb, int parts,
                                                                           float* __restrict__ out, int J, int direct,
                                                                           int* __restrict__ err) {
    extern __shared__ uint32_t lds[];
    __shared__ float head[EMB_WAVES][64 * VW], tail[EMB_WAVES][64 * VW];  // first and last run of a wave
    __shared__ uint32_t whole[EMB_WAVES];                                 // the wave saw one run only: it is in head
    __shared__ float wred[EMB_WAVES];
    uint32_t* sid = lds;        // [T rounded up to 4] ids of this example
    uint16_t* order = reinterpret_cast<uint16_t*>(lds + (T + 3) / 4 * 4);  // [T] row index at each sorted position (T <= 4096)
    constexpr int AHEAD = emb_ahead(DISTINCT);
    const int i = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nt = 64 * ncb * parts;
    bool bad = false;
    for (int t = threadIdx.x; t < (T + 3) / 4 * 4; t += nt) {
        const int32_t v = t < T ? ids[(size_t)i * T + t] : 0;
        if (t < T && (v < 0 || v >= V)) bad = true;
        sid[t] = t >= T ? 0xFFFFFFFFu : v == -1 ? 0xFFFFFFFEu : (uint32_t)v;  // (the padding ranks behind everything, also behind -1)
    }
    if (bad) atomicOr(err, 1);
    __syncthreads();
    if constexpr (!DISTINCT) {
        const uint4* s4 = reinterpret_cast<const uint4*>(sid);
        const int n4 = (T + 3) / 4;
        for (int t0 = wave * 64; t0 < T; t0 += nt) {  // (the same bounds for all lanes: the reads stay in flight)
            const int t = t0 + lane, mid = t0 / 4 + 16 < n4 ? t0 / 4 + 16 : n4;
            const uint32_t v = sid[t < T ? t : T - 1];
            // keys are unique as (id, position): before position t an equal id ranks lower, after it higher
            int rank = 0;
#pragma unroll 4
            for (int s = 0; s < t0 / 4; ++s) {
                const uint4 u = s4[s];
                rank += (u.x <= v) + (u.y <= v) + (u.z <= v) + (u.w <= v);
            }
#pragma unroll 4
            for (int s = t0 / 4; s < mid; ++s) {
                const uint4 u = s4[s];
                const int e = t - 4 * s;
                rank += (u.x < v + (e > 0)) + (u.y < v + (e > 1)) + (u.z < v + (e > 2)) + (u.w < v + (e > 3));
            }
#pragma unroll 4
            for (int s = mid; s < n4; ++s) {
                const uint4 u = s4[s];
                rank += (u.x < v) + (u.y < v) + (u.z < v) + (u.w < v);
            }
            if (t < T) order[rank] = (uint16_t)t;
        }
        __syncthreads();
    }
    const int cb = wave % ncb, part = wave / ncb;
    const int col0 = (blockIdx.y * ncb + cb) * 64 * VW, col = col0 + lane * VW;
    const int per = (T + parts - 1) / parts, lo = part * per, hi = lo + per < T ? lo + per : T;  // this wave's positions
    float sq[VW], run[VW];  // squares of the finished runs, the run at hand
#pragma unroll
    for (int k = 0; k < VW; ++k) sq[k] = run[k] = 0.f;
    bool one = true;  // no run has ended yet
    if (col0 < d && lo < hi) {  // (whole waves: lanes past the width read its last columns again and drop them below)
        constexpr int E = BF16 ? 2 : 4;
        const uint32_t at = ((col < d ? col : d - VW) - col0) * E;
        const char* base = reinterpret_cast<const char*>(G) + ((size_t)i * T * d + col0) * E;
        for (int q0 = lo; q0 < hi; q0 += 64) {
            // 64 positions, one a lane: the address of the row, and whether the run before it is complete
            const int p = q0 + lane < hi ? q0 + lane : hi - 1, row = DISTINCT ? p : (int)order[p], n = hi - q0;
            const uint64_t addr = (uint64_t)base + (uint64_t)row * ((uint64_t)d * E);
            const int a_lo = (int)(uint32_t)addr, a_hi = (int)(addr >> 32);
            const uint64_t ends = DISTINCT ? 0 : __ballot(q0 + lane < hi && p > lo && sid[row] != sid[order[p > lo ? p - 1 : lo]]);
            for (int u0 = 0; u0 < 64 && u0 < n; u0 += AHEAD) {
                RawVec<BF16, VW> g[AHEAD];
                const int left = n - u0;
                const uint32_t e = (uint32_t)(ends >> u0);
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    const uint64_t r = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(a_hi, u0 + u) << 32 | (uint32_t)__builtin_amdgcn_readlane(a_lo, u0 + u);
                    g[u] = load_raw<BF16, VW>((rw_global)r, at);
                }
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    if (u >= left) continue;
                    if constexpr (DISTINCT) {
#pragma unroll
                        for (int k = 0; k < VW; ++k) sq[k] += raw_value<BF16, VW>(g[u], k) * raw_value<BF16, VW>(g[u], k);
                    } else if (!(e & (1u << u))) {
#pragma unroll
                        for (int k = 0; k < VW; ++k) run[k] += raw_value<BF16, VW>(g[u], k);
                    } else {
                        if (one && parts > 1) {
#pragma unroll
                            for (int k = 0; k < VW; ++k) head[wave][lane * VW + k] = run[k];
                        } else {
#pragma unroll
                            for (int k = 0; k < VW; ++k) sq[k] += run[k] * run[k];
                        }
                        one = false;
#pragma unroll
                        for (int k = 0; k < VW; ++k) run[k] = raw_value<BF16, VW>(g[u], k);
                    }
                }
            }
        }
    }
    float tot = 0.f;
#pragma unroll
    for (int k = 0; k < VW; ++k) tot += sq[k];
    if (col >= d) {
        tot = 0.f;
#pragma unroll
        for (int k = 0; k < VW; ++k) run[k] = 0.f;
    }
    if (!DISTINCT && parts == 1) {  // nothing to join
#pragma unroll
        for (int k = 0; k < VW; ++k) tot += run[k] * run[k];
    } else if constexpr (!DISTINCT) {
#pragma unroll
        for (int k = 0; k < VW; ++k) {
            if (one) head[wave][lane * VW + k] = run[k];  // (its only run; otherwise the first is there already)
            tail[wave][lane * VW + k] = run[k];
        }
        if (lane == 0) whole[wave] = one ? 1u : 0u;
        __syncthreads();
        if (part == 0 && col < d) {
            // the parts of this column block in order of position: a part's first run continues the one before it when the ids agree
            float carry[VW];
#pragma unroll
            for (int k = 0; k < VW; ++k) carry[k] = 0.f;
            uint32_t carry_id = 0;
            for (int q = 0; q < parts && q * per < T; ++q) {
                const int w = q * ncb + cb, end = (q + 1) * per < T ? (q + 1) * per : T;
                const bool joins = q > 0 && sid[order[q * per]] == carry_id, single = whole[w] != 0u;
#pragma unroll
                for (int k = 0; k < VW; ++k) {
                    const float h = head[w][lane * VW + k];
                    tot += joins ? 0.f : carry[k] * carry[k];
                    carry[k] = joins ? carry[k] + h : h;
                    if (!single) {
                        tot += carry[k] * carry[k];
                        carry[k] = tail[w][lane * VW + k];
                    }
                }
                carry_id = sid[order[end - 1]];
            }
#pragma unroll
            for (int k = 0; k < VW; ++k) tot += carry[k] * carry[k];
        }
    }
    tot = dp_wave_sum(tot);
    if (lane == 0) wred[wave] = tot;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < ncb * parts; ++w) tot += wred[w];  // in wave order
        // (an out-of-range id only changes the grouping; the error itself is reported by dp_sync)
        if (direct) out[i] += tot;
        else out[(size_t)i * J + blockIdx.y] = tot;
    }
}

// ------------------------------------------------------------------------------------------------
// embedding, clip-weighted scatter (pass 2): stable LSD radix sort of (id, row) + ordered segment sums
// ------------------------------------------------------------------------------------------------
// Launches: a histogram and a scatter per 8-bit digit (the first pair reads the ids themselves), segment sums, fix-up; up to
// SORT_INLINE chunks a scatter forms its own bases from the histogram, beyond that a scan does.  Every launch of a few
// microseconds of work costs about five: B * T = 65,536, V = 30,522: 46 -> 24 us for the sort (7 launches, now 4).
// ------------------------------------------------------------------------------------------------
constexpr int SORT_CHUNK = 1024;
constexpr int SORT_INLINE = 256;  // chunks up to which every workgroup can afford to read the whole histogram (1 KiB a chunk)

// A row of the histogram (one digit) is padded to a multiple of 4 chunks where the workspace allows, the padding zero.
inline int sort_pitch(int nchunks) { return (nchunks + 3) / 4 * 4; }

// Key of position r: the id, or the sentinel V (sorts last and is skipped) for an id out of range.
template <bool FIRST>
__device__ __forceinline__ uint32_t sort_key(const uint32_t* __restrict__ keys, int r, int V) {
    const uint32_t k = keys[r];
    return FIRST ? ((int32_t)k < 0 || k >= (uint32_t)V ? (uint32_t)V : k) : k;
}

// hist[b * pitch + c] = number of keys of chunk c whose digit is b (integer counters in LDS: the order of the
// additions does not matter).  FIRST: `keys` are the ids, range-checked here.
template <bool FIRST>
__global__ __launch_bounds__(256) void sort_hist(const uint32_t* __restrict__ keys, int N, int V, int shift,
                                                 uint32_t* __restrict__ hist, int nchunks, int pitch, int* __restrict__ err) {
    __shared__ uint32_t cnt[256];
    const int c = blockIdx.x;
    const int n0 = c * SORT_CHUNK;
    const int valid = N - n0 < SORT_CHUNK ? N - n0 : SORT_CHUNK;
    cnt[threadIdx.x] = 0;
    __syncthreads();
    bool bad = false;
#pragma unroll
    for (int u = 0; u < SORT_CHUNK / 256; ++u) {
        const int k = threadIdx.x + 256 * u;
        if (k < valid) {
            const uint32_t key = sort_key<FIRST>(keys, n0 + k, V);
            bad = bad || (FIRST && key == (uint32_t)V);
            atomicAdd(&cnt[(key >> shift) & 255u], 1u);
        }
    }
    if (bad) atomicOr(err, 1);
    __syncthreads();
    hist[(size_t)threadIdx.x * pitch + c] = cnt[threadIdx.x];
    if (c == 0)
        for (int k = nchunks; k < pitch; ++k) hist[(size_t)threadIdx.x * pitch + k] = 0;
}

// In-place exclusive prefix sum of hist[0..n): one workgroup, thread t owns a contiguous slice, read and written as
// 16-byte vectors, eight in flight, where it is a multiple of 4 (n is 256 digits x the row pitch).
__global__ __launch_bounds__(256) void sort_scan(uint32_t* __restrict__ hist, int n) {
    __shared__ uint32_t tsum[256];
    const int per = (n + 255) / 256;  // n % 256 == 0: every slice is full
    const int lo = threadIdx.x * per;
    const int hi = lo + per < n ? lo + per : n;
    const bool vec = per % 4 == 0;
    uint32_t s = 0;
    if (vec) {
        const uint4* p4 = reinterpret_cast<const uint4*>(hist + lo);
        const int n4 = (hi - lo) / 4;
        for (int k = 0; k < n4; k += 8) {
            uint4 t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = k + u < n4 ? p4[k + u] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int u = 0; u < 8; ++u) s += (t[u].x + t[u].y) + (t[u].z + t[u].w);
        }
    } else {
        for (int k = lo; k < hi; ++k) s += hist[k];
    }
    tsum[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int k = 0; k < 256; ++k) {
            const uint32_t t = tsum[k];
            tsum[k] = run;
            run += t;
        }
    }
    __syncthreads();
    uint32_t run = tsum[threadIdx.x];
    if (vec) {
        uint4* p4 = reinterpret_cast<uint4*>(hist + lo);
        const int n4 = (hi - lo) / 4;
        for (int k = 0; k < n4; k += 8) {
            uint4 t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = k + u < n4 ? p4[k + u] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                uint4 o;
                o.x = run; run += t[u].x;
                o.y = run; run += t[u].y;
                o.z = run; run += t[u].z;
                o.w = run; run += t[u].w;
                if (k + u < n4) p4[k + u] = o;
            }
        }
    } else {
        for (int k = lo; k < hi; ++k) {
            const uint32_t t = hist[k];
            hist[k] = run;
            run += t;
        }
    }
}

// Stable scatter of one chunk by the current digit.  The chunk is cut into groups of 64 consecutive keys (one wave
// handles a group at a time): digit counts per group (LDS integer counters), an exclusive scan over the groups per
// digit on top of the chunk's global base, and inside a group the rank of a key among the keys of equal digit at lower
// positions, from eight ballots.  INLINE: `base` is the histogram itself, its pitch a multiple of 4; thread b adds up digit b's counts of all chunks and of
// the chunks before this one, and a scan over the digits makes them bases.  Otherwise it has been scanned.
template <bool FIRST, bool INLINE>
__global__ __launch_bounds__(256) void sort_scatter(const uint32_t* __restrict__ keys,
                                                    const uint32_t* __restrict__ vals, int N, int V, int shift,
                                                    const uint32_t* __restrict__ base, int pitch,
                                                    uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out) {
    constexpr int NG = SORT_CHUNK / 64;  // groups per chunk
    __shared__ uint32_t gcnt[NG][256];
    __shared__ uint32_t wtot[4];
    const int c = blockIdx.x;
    const int n0 = c * SORT_CHUNK;
    const int valid = N - n0 < SORT_CHUNK ? N - n0 : SORT_CHUNK;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int e = threadIdx.x; e < NG * 256; e += 256) (&gcnt[0][0])[e] = 0;
    uint32_t key[NG / 4], val[NG / 4];
#pragma unroll
    for (int q = 0; q < NG / 4; ++q) {
        const int k = (wave + 4 * q) * 64 + lane;
        key[q] = val[q] = 0;
        if (k < valid) {
            key[q] = sort_key<FIRST>(keys, n0 + k, V);
            val[q] = FIRST ? (uint32_t)(n0 + k) : vals[n0 + k];
        }
    }
    uint32_t start;  // output position of the chunk's first key with digit threadIdx.x
    if constexpr (INLINE) {
        const uint4* __restrict__ row = reinterpret_cast<const uint4*>(base + (size_t)threadIdx.x * pitch);
        uint32_t total = 0, before = 0;
        for (int k4 = 0; k4 < pitch / 4; k4 += 8) {
            uint4 t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = k4 + u < pitch / 4 ? row[k4 + u] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = 4 * (k4 + u);
                total += (t[u].x + t[u].y) + (t[u].z + t[u].w);
                before += (k < c ? t[u].x : 0u) + (k + 1 < c ? t[u].y : 0u) + (k + 2 < c ? t[u].z : 0u) + (k + 3 < c ? t[u].w : 0u);
            }
        }
        uint32_t incl = total;  // inclusive scan over the lanes, then over the waves
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        if (lane == 63) wtot[wave] = incl;
        __syncthreads();
        uint32_t pre = 0;
#pragma unroll
        for (int w = 0; w < 3; ++w) pre += w < wave ? wtot[w] : 0u;
        start = pre + incl - total + before;
    } else {
        __syncthreads();
        start = base[(size_t)threadIdx.x * pitch + c];
    }
#pragma unroll
    for (int q = 0; q < NG / 4; ++q) {
        const int g = wave + 4 * q, k = g * 64 + lane;
        if (k < valid) atomicAdd(&gcnt[g][(key[q] >> shift) & 255u], 1u);
    }
    __syncthreads();
    {
        const uint32_t b = threadIdx.x;
        uint32_t run = start;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const uint32_t t = gcnt[g][b];
            gcnt[g][b] = run;
            run += t;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NG / 4; ++q) {
        const int g = wave + 4 * q, k = g * 64 + lane;
        const bool ok = k < valid;
        const uint32_t dgt = (key[q] >> shift) & 255u;
        unsigned long long same = __ballot(ok);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const bool one = (dgt >> bit) & 1u;
            const unsigned long long bal = __ballot(ok && one);
            same &= one ? bal : ~bal;
        }
        if (ok) {
            const uint32_t rank = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
            const uint32_t o = gcnt[g][dgt] + rank;
            keys_out[o] = key[q];
            vals_out[o] = val[q];
        }
    }
}

// Ordered segment sums over the sorted (id, row) list.  A workgroup owns the SEG_CHUNK sorted positions [pc*SEG_CHUNK, ...)
// and 256*VW columns, 64*VW a wave.  A run of equal ids that lies wholly inside the chunk is added to sum_E directly (this
// workgroup is its only writer).  A run that continues from the previous chunk goes to first[pc], a run that starts here
// and continues into the next chunk goes to last[pc]; segment_fixup_kernel adds those pieces in chunk order.
// The table row of a finished run is asked for when the run ends and written when the next one does, so that its round trip
// hides behind the rows that follow.  Clip factors are formed here.  B * T = 65,536, d = 1024: 57 -> 41 us
// (134 MB of rows, 80 MB of the table and 30 MB of pieces: near what memory gives).
constexpr int SEG_CHUNK = 32;

template <bool BF16, int VW>
__global__ __launch_bounds__(256) void segment_sums_kernel(const uint32_t* __restrict__ keys,
                                                           const uint32_t* __restrict__ vals,
                                                           const void* __restrict__ G, const float* __restrict__ sqnorms, float C,
                                                           int N, int T, int d, int V, float* __restrict__ sum_E,
                                                           float* __restrict__ first, float* __restrict__ last, int* __restrict__ err) {
    __shared__ uint32_t skey[SEG_CHUNK + 2];  // [0] = key before the chunk, [1..n] = chunk, [n+1] = key after
    __shared__ uint32_t srow[SEG_CHUNK];
    __shared__ float sc[SEG_CHUNK];
    const int pc = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p0 = pc * SEG_CHUNK;
    const int n = N - p0 < SEG_CHUNK ? N - p0 : SEG_CHUNK;
    const uint32_t NONE = 0xFFFFFFFFu;
    if ((int)threadIdx.x < n) {
        const int k = threadIdx.x;
        skey[1 + k] = keys[p0 + k];
        const uint32_t row = vals[p0 + k];
        srow[k] = row;
        const float c = dp_clip_factor(sqnorms[row / (uint32_t)T], C);
        sc[k] = c;
        if (c != c) atomicOr(err, DP_ERRBIT_NORM);
    }
    if (threadIdx.x == 64) skey[0] = p0 > 0 ? keys[p0 - 1] : NONE;
    if (threadIdx.x == 65) skey[n + 1] = p0 + n < N ? keys[p0 + n] : NONE;
    __syncthreads();
    const int col = ((blockIdx.y * 4 + wave) * 64 + lane) * VW;
    if (col >= d) return;
    float acc[VW], pend[VW], old[VW];  // the run under way; a finished run and the table row it adds to
    float* pdst = nullptr;
#pragma unroll
    for (int k = 0; k < VW; ++k) acc[k] = pend[k] = old[k] = 0.f;
    auto flush = [&]() {
        if (pdst) {
#pragma unroll
            for (int e = 0; e < VW; ++e) pdst[e] = old[e] + pend[e];
        }
    };
    int seg_start = 0;
    constexpr int AHEAD = 16;
    for (int k0 = 0; k0 < n; k0 += AHEAD) {
        float g[AHEAD][VW];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int k = k0 + u < n ? k0 + u : n - 1;
            load_vec<BF16, VW>(G, (size_t)srow[k] * d + col, g[u]);
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int k = k0 + u;
            if (k < n) {
                const uint32_t key = skey[1 + k];
                const float w = sc[k];
#pragma unroll
                for (int e = 0; e < VW; ++e) acc[e] += w * g[u][e];
                if (skey[2 + k] != key) {  // the run ends at position k (the same for all lanes)
                    if (key < (uint32_t)V) {
                        if (seg_start == 0 && skey[0] == key) {
                            float* dst = first + (size_t)pc * d + col;
#pragma unroll
                            for (int e = 0; e < VW; ++e) dst[e] = acc[e];
                        } else {
                            flush();
                            pdst = sum_E + (size_t)key * d + col;
#pragma unroll
                            for (int e = 0; e < VW; ++e) {
                                old[e] = pdst[e];
                                pend[e] = acc[e];
                            }
                        }
                    }
#pragma unroll
                    for (int e = 0; e < VW; ++e) acc[e] = 0.f;
                    seg_start = k + 1;
                }
            }
        }
    }
    if (seg_start < n) {
        // the last run continues into the next chunk (skey[n+1] equals its key)
        const uint32_t key = skey[n];
        if (key < (uint32_t)V) {
            const bool from_prev = seg_start == 0 && skey[0] == key;
            float* dst = from_prev ? first + (size_t)pc * d + col : last + (size_t)pc * d + col;
#pragma unroll
            for (int e = 0; e < VW; ++e) dst[e] = acc[e];
        }
    }
    flush();
}

// Workgroups (pc, column block) for every chunk pc whose last run starts in pc and continues into pc+1: add last[pc],
// then first[q] for the chunks q = pc+1 .. that the run reaches, and add the total to sum_E[key].  The end of the run is found by
// bisection of the sorted keys (the most frequent token spans hundreds of chunks); four groups of threads take the pieces
// q = pc+1+g, pc+5+g, ... in ascending order, eight loads in flight, and their sums are added as (0+1)+(2+3): fixed order.
// 64 * VW columns a workgroup.  22 -> 12 us (one group, one column a thread, before).
template <int VW>
__global__ __launch_bounds__(256) void segment_fixup_kernel(const uint32_t* __restrict__ keys, int N, int d, int V,
                                                            int nchunks, const float* __restrict__ first,
                                                            const float* __restrict__ last,
                                                            float* __restrict__ sum_E) {
    __shared__ float red[4][64][VW];
    const int pc = blockIdx.x;
    const int pend = (pc + 1) * SEG_CHUNK;  // first position of the next chunk
    if (pend >= N) return;
    const uint32_t key = keys[pend - 1];
    if (key >= (uint32_t)V || keys[pend] != key) return;             // no run crosses this boundary
    const int p0 = pc * SEG_CHUNK;
    if (p0 > 0 && keys[p0 - 1] == key && keys[p0] == key) return;    // the run started earlier: not its head
    int lo = pend, hi = N;  // keys[lo] == key; the run ends at the first position in (lo, hi] whose key differs
    // most runs end in the next chunk: look there before bisecting
    if (pend + SEG_CHUNK >= N || keys[pend + SEG_CHUNK] != key) hi = pend + 1;
    while (hi - lo > 1) {
        const int mid = lo + (hi - lo) / 2;
        if (keys[mid] == key) lo = mid;
        else hi = mid;
    }
    const int qlast = lo / SEG_CHUNK;  // every chunk pc+1 .. qlast starts inside the run, so its first[] holds a piece
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int col = (blockIdx.y * 64 + lane) * VW;
    float acc[VW];
#pragma unroll
    for (int e = 0; e < VW; ++e) acc[e] = 0.f;
    if (col < d) {
        auto piece = [&](const float* __restrict__ src, int q, float out[VW]) {
            if constexpr (VW == 4) {
                const float4 t = *reinterpret_cast<const float4*>(src + (size_t)q * d + col);
                out[0] = t.x; out[1] = t.y; out[2] = t.z; out[3] = t.w;
            } else {
                out[0] = src[(size_t)q * d + col];
            }
        };
        if (g == 0) piece(last, pc, acc);
        int q = pc + 1 + g;
        for (; q + 28 <= qlast; q += 32) {
            float f[8][VW];
#pragma unroll
            for (int u = 0; u < 8; ++u) piece(first, q + 4 * u, f[u]);
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int e = 0; e < VW; ++e) acc[e] += f[u][e];
        }
        for (; q <= qlast; q += 4) {
            float f[VW];
            piece(first, q, f);
#pragma unroll
            for (int e = 0; e < VW; ++e) acc[e] += f[e];
        }
    }
#pragma unroll
    for (int e = 0; e < VW; ++e) red[g][lane][e] = acc[e];
    __syncthreads();
    if (g == 0 && col < d) {
        float* dst = sum_E + (size_t)key * d + col;
#pragma unroll
        for (int e = 0; e < VW; ++e)
            dst[e] += (red[0][lane][e] + red[1][lane][e]) + (red[2][lane][e] + red[3][lane][e]);
    }
}

inline int bit_length(uint32_t v) {
    int b = 0;
    while (v) {
        ++b;
        v >>= 1;
    }
    return b;
}

inline bool vec4_ok(dp_dtype dt, int d, const void* p, const void* q) {
    if (dt == DP_BF16) return true;  // d % 8 == 0 and 16-byte alignment are checked at the API
    return d % 4 == 0 && (((uintptr_t)p | (uintptr_t)q) & 15) == 0;
}

}  // namespace

// ================================================================================================
// host launchers
// ================================================================================================
dp_status dpk_reduce_partials(dp_ctx* ctx, const float* part, int R, size_t stride, size_t n, float* out) {
    if (n == 0) return DP_OK;
    if (n % 4 == 0 && stride % 4 == 0 && (((uintptr_t)part | (uintptr_t)out) & 15) == 0) {
        const size_t n4 = n / 4;
        if (R >= 32 && n4 <= 16384)
            hipLaunchKernelGGL(reduce_partials_tall_kernel, dim3((unsigned)((n4 + 63) / 64)), dim3(256), 0, ctx->stream,
                               reinterpret_cast<const float4*>(part), R, stride / 4, n4, reinterpret_cast<float4*>(out));
        else
            hipLaunchKernelGGL(reduce_partials_vec4_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0,
                               ctx->stream, reinterpret_cast<const float4*>(part), R, stride / 4, n4,
                               reinterpret_cast<float4*>(out));
    } else {
        hipLaunchKernelGGL(reduce_partials_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream, part,
                           R, stride, n, out);
    }
    DP_LAUNCH_CHECK(ctx, "reduce_partials");
    return DP_OK;
}

template <bool BF16, int VW>
static dp_status colstat_sqnorms_launch(dp_ctx* ctx, int L, const void* const* X, const void* const* G, int B, int T, int d,
                                        int use_x, int use_1, float* sqnorms, float* const* keep) {
    const int J = (d + 64 * VW - 1) / (64 * VW);
    ColBatch cb;
    ColKeep ck;
    for (int l = 0; l < COL_MAX_BATCH; ++l) {
        cb.X[l] = use_x ? X[l < L ? l : 0] : nullptr;
        cb.G[l] = G[l < L ? l : 0];
        ck.keep[l] = keep ? keep[l < L ? l : 0] : nullptr;
    }
    float* out = sqnorms;
    int direct = 1;
    if (J > 1 || L > 1) {
        dp_ws_alloc ws(ctx);
        out = ws.get<float>((size_t)B * L * J);
        if (!out) {
            DP_SET_ERR(ctx, "workspace too small for %d x %d norm partials", B, L * J);
            return DP_ERR_WORKSPACE;
        }
        direct = 0;
    }
    dim3 grid(B, J, L);
    if (keep)  // (LayerNorm only: both statistics)
        hipLaunchKernelGGL((colstat_sqnorms_kernel<BF16, VW, true, true, true>), grid, dim3(256), 0, ctx->stream, cb, ck, T, d, out, J, direct);
    else if (use_x && use_1)
        hipLaunchKernelGGL((colstat_sqnorms_kernel<BF16, VW, true, true, false>), grid, dim3(256), 0, ctx->stream, cb, ck, T, d, out, J, direct);
    else if (use_x)
        hipLaunchKernelGGL((colstat_sqnorms_kernel<BF16, VW, true, false, false>), grid, dim3(256), 0, ctx->stream, cb, ck, T, d, out, J, direct);
    else
        hipLaunchKernelGGL((colstat_sqnorms_kernel<BF16, VW, false, true, false>), grid, dim3(256), 0, ctx->stream, cb, ck, T, d, out, J, direct);
    DP_LAUNCH_CHECK(ctx, "colstat_sqnorms");
    if (!direct) return dpk_finish_partials(ctx, out, B, L * J, sqnorms);  // (in an order fixed by L * J)
    return DP_OK;
}

// keep: NULL, or n pointers to [B][2][d] fp32 buffers that receive every example's two statistics (then use_x = use_1 = 1)
dp_status dpk_colstat_sqnorms_batched(dp_ctx* ctx, int n, const void* const* X, const void* const* G, dp_dtype dt, int B, int T,
                                      int d, int use_x, int use_1, float* sqnorms, float* const* keep) {
    if (B == 0 || T == 0 || d == 0 || n == 0 || (!use_x && !use_1)) return DP_OK;
    bool v4 = true;
    for (int l = 0; l < n; ++l) v4 = v4 && vec4_ok(dt, d, use_x ? X[l] : G[l], G[l]);
    // layers per launch: as many as one may hold and as have room for their partial norms (at least one)
    const int vw = dt == DP_BF16 || v4 ? 4 : 1;
    size_t per = ctx->ws_bytes / ((size_t)B * ((d + 64 * vw - 1) / (64 * vw)) * sizeof(float));
    per = per < 1 ? 1 : per > COL_MAX_BATCH ? COL_MAX_BATCH : per;
    for (int l0 = 0; l0 < n; l0 += (int)per) {
        const int L = n - l0 < (int)per ? n - l0 : (int)per;
        const void* const* Xl = use_x ? X + l0 : nullptr;
        dp_status st;
        float* const* kl = keep ? keep + l0 : nullptr;
        if (dt == DP_BF16) st = colstat_sqnorms_launch<true, 4>(ctx, L, Xl, G + l0, B, T, d, use_x, use_1, sqnorms, kl);
        else if (v4) st = colstat_sqnorms_launch<false, 4>(ctx, L, Xl, G + l0, B, T, d, use_x, use_1, sqnorms, kl);
        else st = colstat_sqnorms_launch<false, 1>(ctx, L, Xl, G + l0, B, T, d, use_x, use_1, sqnorms, kl);
        if (st != DP_OK) return st;
    }
    return DP_OK;
}

dp_status dpk_colstat_sqnorms(dp_ctx* ctx, const void* X, const void* G, dp_dtype dt, int B, int T, int d, int use_x,
                              int use_1, float* sqnorms) {
    return dpk_colstat_sqnorms_batched(ctx, 1, &X, &G, dt, B, T, d, use_x, use_1, sqnorms, nullptr);
}

// sum_x[l][j] += sum_i c_i keep[l][i][0][j], sum_1[l][j] += sum_i c_i keep[l][i][1][j]; d % 4 == 0, 16-byte aligned buffers
dp_status dpk_kept_sums_batched(dp_ctx* ctx, int n, float* const* keep, int B, int d, const float* c, float* const* sum_x,
                                float* const* sum_1) {
    if (B == 0 || d == 0 || n == 0) return DP_OK;
    int L;
    for (int l0 = 0; l0 < n; l0 += L) {
        L = dp_disjoint_layers(n - l0 < COL_MAX_BATCH ? n - l0 : COL_MAX_BATCH, sum_x + l0, d, sum_1 + l0, d);
        ColKeep ck;
        ColOut co;
        for (int l = 0; l < COL_MAX_BATCH; ++l) {
            ck.keep[l] = keep[l0 + (l < L ? l : 0)];
            co.out_x[l] = sum_x[l0 + (l < L ? l : 0)];
            co.out_1[l] = sum_1[l0 + (l < L ? l : 0)];
        }
        hipLaunchKernelGGL(kept_sums_kernel, dim3((unsigned)((2 * d / 4 + 63) / 64), L), dim3(256), 0, ctx->stream, ck, co, c, B, d);
        DP_LAUNCH_CHECK(ctx, "kept_sums");
    }
    return DP_OK;
}

// Runs of rows that the column sums of a layer are cut into (`vw` columns a lane), and the rows of a run.
static long colstat_runs(long nrows, int d, int vw, int* rows_per) {
    const int J = (d + 64 * vw - 1) / (64 * vw);
    long R = 1024 / J;  // about 1024 workgroups per layer
    if (R < 1) R = 1;
    const long maxR = (nrows + 63) / 64;
    if (R > maxR) R = maxR;
    *rows_per = (int)((nrows + R - 1) / R);
    return (nrows + *rows_per - 1) / *rows_per;
}

// out_x / out_1: tables of L pointers, or NULL when that statistic is not wanted (the same for every layer of the call)
template <bool BF16, int VW>
static dp_status colstat_sums_launch(dp_ctx* ctx, int L, const void* const* X, const void* const* G, int B, int T, int d,
                                     const float* c, float* const* out_x, float* const* out_1) {
    const long nrows = (long)B * T;
    const int J = (d + 64 * VW - 1) / (64 * VW);
    int rows_per;
    const long R = colstat_runs(nrows, d, VW, &rows_per);
    dp_ws_alloc ws(ctx);
    float* part = ws.get<float>((size_t)L * R * 2 * d);
    if (!part) {
        DP_SET_ERR(ctx, "workspace too small for column-sum partials (%d x %ld x 2 x %d floats)", L, R, d);
        return DP_ERR_WORKSPACE;
    }
    ColBatch cb;
    for (int l = 0; l < COL_MAX_BATCH; ++l) {
        cb.X[l] = out_x ? X[l < L ? l : 0] : nullptr;
        cb.G[l] = G[l < L ? l : 0];
    }
    dim3 grid((unsigned)R, J, L);
    if (out_x)
        hipLaunchKernelGGL((colstat_sums_kernel<BF16, VW, true>), grid, dim3(256), 0, ctx->stream, cb, c, T, d, nrows, rows_per, part);
    else
        hipLaunchKernelGGL((colstat_sums_kernel<BF16, VW, false>), grid, dim3(256), 0, ctx->stream, cb, c, T, d, nrows, rows_per, part);
    DP_LAUNCH_CHECK(ctx, "colstat_sums");
    bool pair = out_x && out_1 && d % 4 == 0 && R >= 32 && d <= 32768 && ((uintptr_t)part & 15) == 0;
    for (int l = 0; pair && l < L; ++l) pair = (((uintptr_t)out_x[l] | (uintptr_t)out_1[l]) & 15) == 0;
    if (pair) {
        ColOut co;
        for (int l = 0; l < COL_MAX_BATCH; ++l) {
            co.out_x[l] = out_x[l < L ? l : 0];
            co.out_1[l] = out_1[l < L ? l : 0];
        }
        const size_t d4 = (size_t)d / 4;
        hipLaunchKernelGGL(reduce_partials_pair_kernel, dim3((unsigned)((2 * d4 + 63) / 64), L), dim3(256), 0, ctx->stream,
                           reinterpret_cast<const float4*>(part), (int)R, d4, co);
        DP_LAUNCH_CHECK(ctx, "reduce_partials_pair");
        return DP_OK;
    }
    for (int l = 0; l < L; ++l) {
        const float* pl = part + (size_t)l * R * 2 * d;
        dp_status st = DP_OK;
        if (out_x) st = dpk_reduce_partials(ctx, pl, (int)R, (size_t)2 * d, d, out_x[l]);
        if (st == DP_OK && out_1) st = dpk_reduce_partials(ctx, pl + d, (int)R, (size_t)2 * d, d, out_1[l]);
        if (st != DP_OK) return st;
    }
    return DP_OK;
}

dp_status dpk_colstat_sums_batched(dp_ctx* ctx, int n, const void* const* X, const void* const* G, dp_dtype dt, int B, int T,
                                   int d, const float* c, float* const* out_x, float* const* out_1) {
    if (B == 0 || T == 0 || d == 0 || n == 0 || (!out_x && !out_1)) return DP_OK;
    bool v4 = true;
    for (int l = 0; l < n; ++l) v4 = v4 && vec4_ok(dt, d, out_x ? X[l] : G[l], G[l]);
    // layers per launch: as many as one may hold and as have room for their partial sums (at least one)
    int rows_per;
    size_t per = ctx->ws_bytes / (colstat_runs((long)B * T, d, dt == DP_BF16 || v4 ? 4 : 1, &rows_per) * 2 * (size_t)d * sizeof(float));
    per = per < 1 ? 1 : per > COL_MAX_BATCH ? COL_MAX_BATCH : per;
    int L;
    for (int l0 = 0; l0 < n; l0 += L) {
        const void* const* Xl = out_x ? X + l0 : nullptr;
        float* const* ox = out_x ? out_x + l0 : nullptr;
        float* const* o1 = out_1 ? out_1 + l0 : nullptr;
        L = dp_disjoint_layers(n - l0 < (int)per ? n - l0 : (int)per, ox, d, o1, d);
        dp_status st;
        if (dt == DP_BF16) st = colstat_sums_launch<true, 4>(ctx, L, Xl, G + l0, B, T, d, c, ox, o1);
        else if (v4) st = colstat_sums_launch<false, 4>(ctx, L, Xl, G + l0, B, T, d, c, ox, o1);
        else st = colstat_sums_launch<false, 1>(ctx, L, Xl, G + l0, B, T, d, c, ox, o1);
        if (st != DP_OK) return st;
    }
    return DP_OK;
}

dp_status dpk_colstat_sums(dp_ctx* ctx, const void* X, const void* G, dp_dtype dt, int B, int T, int d, const float* c,
                           float* out_x, float* out_1) {
    return dpk_colstat_sums_batched(ctx, 1, &X, &G, dt, B, T, d, c, out_x ? &out_x : nullptr, out_1 ? &out_1 : nullptr);
}

template <bool BF16, int VW>
static dp_status embedding_sqnorms_launch(dp_ctx* ctx, const int32_t* ids, const void* G, int B, int T, int d, int V,
                                          int distinct, float* sqnorms) {
    // Column blocks per workgroup: as many as there are (up to 4), so that the ids are ranked once and the example needs no
    // reduction launch; one, and all waves on its positions, when the examples alone are too few for the chip and long enough
    // for 16 waves.  16 waves of this kernel are what the registers of a CU hold: they are shared by the workgroups that a CU gets
    // (B = 512: 36 us with 16 waves, 28 with 8; B = 514, T = 128, d = 256: 21 with 8, 14 with 4; B = 256: 21 with 16).
    const int blocks = (d + 64 * VW - 1) / (64 * VW), pieces = (T + EMB_PIECE - 1) / EMB_PIECE;
    int ncb = blocks >= 3 ? 4 : blocks;
    if ((long)B * ((blocks + ncb - 1) / ncb) < 128 && ncb * pieces > 16) ncb = 1;
    int J = (blocks + ncb - 1) / ncb;
    float* out = sqnorms;
    int direct = 1;
    if (J > 1) {
        dp_ws_alloc ws(ctx);
        out = ws.get<float>((size_t)B * J);
        if (!out) {
            DP_SET_ERR(ctx, "workspace too small for %d x %d norm partials", B, J);
            return DP_ERR_WORKSPACE;
        }
        direct = 0;
    }
    dim3 grid(B, J);
    const size_t lds = ((size_t)T + 3) / 4 * 4 * sizeof(uint32_t) + (size_t)T * sizeof(uint16_t);
    const long per_cu = ((long)B * J + 255) / 256;
    const int room = 16 / ncb / per_cu < 1 ? 1 : (int)(16 / ncb / per_cu), parts = pieces < room ? pieces : room, waves = ncb * parts;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), lds, ctx->stream, ids, G, T, d, V, ncb, parts, out, J, direct, ctx->err_word);
    };
    if (distinct && waves <= 8) launch(embedding_sqnorms_kernel<BF16, VW, true, 8>);
    else if (distinct) launch(embedding_sqnorms_kernel<BF16, VW, true, 16>);
    else if (waves <= 8) launch(embedding_sqnorms_kernel<BF16, VW, false, 8>);
    else launch(embedding_sqnorms_kernel<BF16, VW, false, 16>);
    DP_LAUNCH_CHECK(ctx, "embedding_sqnorms");
    if (!direct) return dpk_finish_partials(ctx, out, B, J, sqnorms);
    return DP_OK;
}

dp_status dpk_embedding_sqnorms(dp_ctx* ctx, const int32_t* ids, const void* G, dp_dtype dt, int B, int T, int d, int V,
                                int distinct, float* sqnorms) {
    if (B == 0 || T == 0 || d == 0) return DP_OK;
    if (T > 4096) {
        DP_SET_ERR(ctx, "dp_sqnorms_embedding: T = %d exceeds the supported maximum of 4096", T);
        return DP_ERR_SHAPE;
    }
    if (dt == DP_BF16) return embedding_sqnorms_launch<true, 4>(ctx, ids, G, B, T, d, V, distinct, sqnorms);
    if (vec4_ok(dt, d, G, G)) return embedding_sqnorms_launch<false, 4>(ctx, ids, G, B, T, d, V, distinct, sqnorms);
    return embedding_sqnorms_launch<false, 1>(ctx, ids, G, B, T, d, V, distinct, sqnorms);
}

template <bool BF16, int VW>
static dp_status embedding_sums_launch(dp_ctx* ctx, const int32_t* ids, const void* G, int B, int T, int d, int V,
                                       const float* sqnorms, float C, float* sum_E) {
    const long Nl = (long)B * T;
    if (Nl > 0x7FFFFFFFl - SORT_CHUNK) {
        DP_SET_ERR(ctx, "dp_clip_accumulate_embedding: B*T too large");
        return DP_ERR_SHAPE;
    }
    const int N = (int)Nl;
    const int nsort = (N + SORT_CHUNK - 1) / SORT_CHUNK;
    const int nseg = (N + SEG_CHUNK - 1) / SEG_CHUNK;
    dp_ws_alloc ws(ctx);
    uint32_t* k0 = ws.get<uint32_t>(N);
    uint32_t* k1 = ws.get<uint32_t>(N);
    uint32_t* v0 = ws.get<uint32_t>(N);
    uint32_t* v1 = ws.get<uint32_t>(N);
    uint32_t* hist;
    float *first, *last;
    const size_t mark = ws.off;
    int pitch = sort_pitch(nsort);
    for (;; pitch = nsort) {  // without padding when there is no room for it: the scan takes any pitch
        ws.off = mark;
        hist = ws.get<uint32_t>((size_t)256 * pitch);
        first = ws.get<float>((size_t)nseg * d);
        last = ws.get<float>((size_t)nseg * d);
        if ((hist && first && last) || pitch == nsort) break;
    }
    if (!k0 || !k1 || !v0 || !v1 || !hist || !first || !last) {
        DP_SET_ERR(ctx, "workspace too small for the embedding sort of %d tokens", N);
        return DP_ERR_WORKSPACE;
    }
    const int bits = bit_length((uint32_t)V);  // the sentinel V itself must be representable
    const bool scan = nsort > SORT_INLINE || pitch % 4 != 0;
    const dim3 grid(nsort), block(256);
    for (int shift = 0; shift < bits; shift += 8) {
        const uint32_t* kin = shift ? k0 : reinterpret_cast<const uint32_t*>(ids);
        if (shift) hipLaunchKernelGGL((sort_hist<false>), grid, block, 0, ctx->stream, kin, N, V, shift, hist, nsort, pitch, ctx->err_word);
        else hipLaunchKernelGGL((sort_hist<true>), grid, block, 0, ctx->stream, kin, N, V, shift, hist, nsort, pitch, ctx->err_word);
        if (scan) hipLaunchKernelGGL(sort_scan, dim3(1), block, 0, ctx->stream, hist, 256 * pitch);
        auto scatter = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, ctx->stream, kin, v0, N, V, shift, hist, pitch, k1, v1); };
        if (shift && scan) scatter(sort_scatter<false, false>);
        else if (shift) scatter(sort_scatter<false, true>);
        else if (scan) scatter(sort_scatter<true, false>);
        else scatter(sort_scatter<true, true>);
        DP_LAUNCH_CHECK(ctx, "radix sort pass");
        uint32_t* t = k0; k0 = k1; k1 = t;
        t = v0; v0 = v1; v1 = t;
    }
    const int J = (d + 256 * VW - 1) / (256 * VW);
    hipLaunchKernelGGL((segment_sums_kernel<BF16, VW>), dim3(nseg, J), dim3(256), 0, ctx->stream, k0, v0, G, sqnorms, C, N, T, d, V, sum_E, first, last, ctx->err_word);
    DP_LAUNCH_CHECK(ctx, "segment_sums");
    if (nseg > 1) {
        const bool v4 = d % 4 == 0;  // the pieces lie in the workspace, aligned
        if (v4) hipLaunchKernelGGL((segment_fixup_kernel<4>), dim3(nseg - 1, (d + 255) / 256), dim3(256), 0, ctx->stream, k0, N, d, V, nseg, first, last, sum_E);
        else hipLaunchKernelGGL((segment_fixup_kernel<1>), dim3(nseg - 1, (d + 63) / 64), dim3(256), 0, ctx->stream, k0, N, d, V, nseg, first, last, sum_E);
        DP_LAUNCH_CHECK(ctx, "segment_fixup");
    }
    return DP_OK;
}

dp_status dpk_embedding_sums(dp_ctx* ctx, const int32_t* ids, const void* G, dp_dtype dt, int B, int T, int d, int V,
                             const float* sqnorms, float C, float* sum_E) {
    if (B == 0 || T == 0 || d == 0) return DP_OK;
    if (dt == DP_BF16) return embedding_sums_launch<true, 4>(ctx, ids, G, B, T, d, V, sqnorms, C, sum_E);
    if (vec4_ok(dt, d, G, G)) return embedding_sums_launch<false, 4>(ctx, ids, G, B, T, d, V, sqnorms, C, sum_E);
    return embedding_sums_launch<false, 1>(ctx, ids, G, B, T, d, V, sqnorms, C, sum_E);
}
