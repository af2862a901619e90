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
typedef uint32_t rw_u32x4 __attribute__((ext_vector_type(4)));
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
constexpr int COL_FACTORS = 2048;  // clip factors that a workgroup forms itself
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
// The factors of up to COL_FACTORS examples are formed here, once per workgroup (OWN: `c` holds the squared norms); per row and thread, a square root and a division,
// they cost 2 %.  One run of rows (DIRECT) is added to the sums themselves.  T x d = 45 x 384 entries of 171 examples: three launches of 4.1, 6.9 and 3.8 us, now two.
template <bool BF16, int VW, bool USE_X, bool OWN>
__global__ __launch_bounds__(256) void colstat_sums_kernel(ColBatch cb, ColOut co, const float* __restrict__ c, float C, int T, int d,
                                                           long nrows, int rows_per, float* __restrict__ part, int direct, int* __restrict__ err) {
    __shared__ float red[4][64][2 * VW];
    __shared__ float own[OWN ? COL_FACTORS : 1];
    const void* __restrict__ X = cb.X[blockIdx.z];
    const void* __restrict__ G = cb.G[blockIdx.z];
    const int lane = threadIdx.x & 63, tg = threadIdx.x >> 6;
    const int col = (blockIdx.y * 64 + lane) * VW;
    const long r0 = (long)blockIdx.x * rows_per;
    const long r1 = r0 + rows_per < nrows ? r0 + rows_per : nrows;
    long e0 = 0;  // the example that `c` begins with
    if constexpr (OWN) {
        e0 = r0 / T;
        for (long e = e0 + threadIdx.x; e * T < r1; e += 256) {
            const float ce = dp_clip_factor(c[e], C);
            own[e - e0] = ce;
            if (ce != ce) atomicOr(err, DP_ERRBIT_NORM);
        }
        __syncthreads();
        c = own;
    }
    float sx[VW], s1[VW];
#pragma unroll
    for (int k = 0; k < VW; ++k) sx[k] = s1[k] = 0.f;
    if (col < d) {
#pragma unroll 4
        for (long r = r0 + tg; r < r1; r += 4) {
            const float w = c[r / T - e0];
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
    if (tg == 0 && col < d && direct) {
        float *x = USE_X ? co.out_x[blockIdx.z] : nullptr, *o = co.out_1[blockIdx.z];
        float ox[VW], oo[VW];
#pragma unroll
        for (int k = 0; k < VW; ++k) {
            ox[k] = x ? x[col + k] : 0.f;
            oo[k] = o ? o[col + k] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < VW; ++k) {
            if (x) x[col + k] = ox[k] + ((red[0][lane][k] + red[1][lane][k]) + (red[2][lane][k] + red[3][lane][k]));
            if (o) o[col + k] = oo[k] + ((red[0][lane][VW + k] + red[1][lane][VW + k]) + (red[2][lane][VW + k] + red[3][lane][VW + k]));
        }
    } else if (tg == 0 && col < d) {
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
// i = g, g+4, ... in ascending order, the four group sums are added as (0+1)+(2+3): fixed order.  A workgroup forms the factors itself
// (OWN: `c` holds the squared norms, up to COL_FACTORS of them): they are a launch that it would wait for otherwise.
template <bool OWN>
__global__ __launch_bounds__(256) void kept_sums_kernel(ColKeep ck, ColOut co, const float* __restrict__ c, float C, int B, int d, int* __restrict__ err) {
    __shared__ float4 red[4][64];
    __shared__ float own[OWN ? COL_FACTORS : 1];
    if constexpr (OWN) {
        for (int i = threadIdx.x; i < B; i += 256) {
            const float ci = dp_clip_factor(c[i], C);
            own[i] = ci;
            if (ci != ci) atomicOr(err, DP_ERRBIT_NORM);
        }
        __syncthreads();
        c = own;
    }
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
// B = 512, T = 128, d = 1024 (134 MB): 31 + 5 -> 28.  Where there are two waves and more to 64 positions they share the comparisons of the ranking, and the
// joining finds out which parts continue one another for all parts at once (B = 74, T = 295, d = 128, norms and sums 37.7 -> 35.6 us; B = 23, T = 375, d = 832 40.9 -> 38.6).
// Waves without positions would only make the joining of the parts longer: T = 16, d = 256, B = 4 12 us with 16 waves, 6 with 1; B = 514 16 | 7.
// ------------------------------------------------------------------------------------------------
// Rows in flight of a wave; without runs to form, position rows of B = 256, T = 128, d = 1,024 take 12.6 us with 8 and 11.4 with 16.
constexpr int emb_ahead(bool distinct) { return distinct ? 16 : 8; }
constexpr int EMB_PIECE = 16;  // positions that are worth a wave
constexpr int EMB_SHARED = 512;  // positions up to which 16 waves are two and more to 64 of them
__host__ __device__ constexpr int emb_shared_ranks(int T) { return T <= EMB_SHARED ? (T + 3) / 4 * 4 : 0; }

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
    uint32_t* part_rank = lds + (T + 3) / 4 * 4;  // [T up to EMB_SHARED, otherwise none] ranks that several waves add up
    uint16_t* order = reinterpret_cast<uint16_t*>(part_rank + emb_shared_ranks(T));  // [T] row index at each sorted position (T <= 4096)
    constexpr int AHEAD = emb_ahead(DISTINCT);
    const int i = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nt = 64 * ncb * parts;
    bool bad = false;
    for (int t = threadIdx.x; t < (T + 3) / 4 * 4; t += nt) {
        const int32_t v = t < T ? ids[(size_t)i * T + t] : 0;
        if (t < T && (v < 0 || v >= V)) bad = true;
        sid[t] = t >= T ? 0xFFFFFFFFu : v == -1 ? 0xFFFFFFFEu : (uint32_t)v;  // (the padding ranks behind everything, also behind -1)
        if (T <= EMB_SHARED) part_rank[t] = 0;
    }
    if (bad) atomicOr(err, 1);
    __syncthreads();
    if constexpr (!DISTINCT) {
        const uint4* s4 = reinterpret_cast<const uint4*>(sid);
        const int n4 = (T + 3) / 4, waves = ncb * parts, chunks = (T + 63) / 64;
        // keys are unique as (id, position): before position t an equal id ranks lower, after it higher; against the positions 4 from .. 4 to
        auto rank_of = [&](int t0, int from, int to) {
            const int t = t0 + lane, mid = t0 / 4 + 16;
            const uint32_t v = sid[t < T ? t : T - 1];
            int rank = 0;
#pragma unroll 4
            for (int s = from; s < (t0 / 4 < to ? t0 / 4 : to); ++s) {
                const uint4 u = s4[s];
                rank += (u.x <= v) + (u.y <= v) + (u.z <= v) + (u.w <= v);
            }
#pragma unroll 4
            for (int s = from > t0 / 4 ? from : t0 / 4; s < (mid < to ? mid : to); ++s) {
                const uint4 u = s4[s];
                const int e = t - 4 * s;
                rank += (u.x < v + (e > 0)) + (u.y < v + (e > 1)) + (u.z < v + (e > 2)) + (u.w < v + (e > 3));
            }
#pragma unroll 4
            for (int s = from > mid ? from : mid; s < to; ++s) {
                const uint4 u = s4[s];
                rank += (u.x < v) + (u.y < v) + (u.z < v) + (u.w < v);
            }
            return rank;
        };
        if (waves >= 2 * chunks) {  // (then T <= EMB_SHARED) several waves to 64 positions, each against its share of all
            const int split = waves / chunks, chunk = wave % chunks, share = wave / chunks, t = chunk * 64 + lane;
            if (share < split) {
                const int rank = rank_of(chunk * 64, n4 * share / split, n4 * (share + 1) / split);
                if (t < T) atomicAdd(&part_rank[t], (uint32_t)rank);
            }
            __syncthreads();
            for (int t = threadIdx.x; t < T; t += nt) order[part_rank[t]] = (uint16_t)t;
        } else {
            for (int t0 = wave * 64; t0 < T; t0 += nt) {  // (the same bounds for all lanes: the reads stay in flight)
                const int rank = rank_of(t0, 0, n4);
                if (t0 + lane < T) order[rank] = (uint16_t)(t0 + lane);
            }
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
        if (part == 0) {
            // the parts of this column block in order of position: a part's first run continues the one before it when the ids agree
            // (a part a lane: read one after the other, ids through the order, they are a chain of LDS reads)
            const int q0 = lane < parts ? lane : 0, p0 = q0 * per;
            const uint64_t joins = __ballot(q0 > 0 && p0 < T && sid[order[p0 < T ? p0 : 0]] == sid[order[p0 < T && p0 > 0 ? p0 - 1 : 0]]);
            const uint64_t single = __ballot(lane < parts && whole[q0 * ncb + cb] != 0u);
            float carry[VW];
#pragma unroll
            for (int k = 0; k < VW; ++k) carry[k] = 0.f;
            for (int q = 0; q < parts && q * per < T && col < d; ++q) {
                const int w = q * ncb + cb;
                const bool join = joins >> q & 1;
#pragma unroll
                for (int k = 0; k < VW; ++k) {
                    const float h = head[w][lane * VW + k], l = tail[w][lane * VW + k];
                    tot += join ? 0.f : carry[k] * carry[k];
                    carry[k] = join ? carry[k] + h : h;
                    if (!(single >> q & 1)) {
                        tot += carry[k] * carry[k];
                        carry[k] = l;
                    }
                }
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
// embedding, clip-weighted scatter (pass 2): the positions grouped by id (group_ids_kernel, or a stable LSD radix sort of (id, row)) + ordered segment sums
// ------------------------------------------------------------------------------------------------
// Launches of the sort: a histogram and a scatter per 8-bit digit (the first pair reads the ids themselves); up to
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
// additions does not matter).  FIRST: `keys` are the ids, range-checked here, and `tickets` is cleared for the sums.
template <bool FIRST>
__global__ __launch_bounds__(256) void sort_hist(const uint32_t* __restrict__ keys, int N, int V, int shift,
                                                 uint32_t* __restrict__ hist, int nchunks, int pitch, uint32_t* __restrict__ tickets, int n_tickets,
                                                 int* __restrict__ err) {
    __shared__ uint32_t cnt[256];
    const int c = blockIdx.x;
    const int n0 = c * SORT_CHUNK;
    const int valid = N - n0 < SORT_CHUNK ? N - n0 : SORT_CHUNK;
    if (FIRST)
        for (int e = c * 256 + threadIdx.x; e < n_tickets; e += gridDim.x * 256) tickets[e] = 0;
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

// One launch that brings the positions of equal ids together, for up to GROUP_MAX_N positions.  The ids are dealt to 2^lg buckets by
// their low lg bits; a workgroup writes the positions of one of the PARTS of a bucket to their places.  Its waves share all positions; each
// counts, over all of its own, those of lower buckets (the bucket's place in the output) and by digit (the bits above lg, an id of its own
// each) those of the bucket, then writes those of the part: the bucket's digits in order, in a digit the waves, in a wave the parts, in a part
// the groups of 64 positions, in these by ballots.  So equal ids keep the order of their positions; the order of the ids does not matter to the sums.
// `tickets` is cleared for the sums.  Bound: the instructions of the count, which takes the low bytes of four groups at a time.
// Us, with the four launches of a histogram and a scatter per digit of 8 bits that took its place before: 464 positions 4.2 | 18, 16,384 7.6 | 18,
// 65,536 20.7 | 24 (of 30,522 ids); beyond, and with more than 65,408 ids, they still are the sort.
constexpr int GROUP_DIGITS = 512, GROUP_WAVES = 16, GROUP_MAX_N = 64 * 64 * GROUP_WAVES, GROUP_MAX_V = (GROUP_DIGITS - 1) << 7;
// Low bits: 64 buckets where there are as many ids, 128 where the digits do not suffice for the rest and for the one of ids out of range.
inline int group_bits(int V) {
    int lg = 0;
    while (lg < 6 && (1 << lg) < V) ++lg;
    while (((V - 1) >> lg) + 1 >= GROUP_DIGITS) ++lg;
    return lg;
}

// A wave has Q * PARTS groups of 64 positions, Q of them in each part.
template <int Q, int PARTS>
__global__ __launch_bounds__(64 * GROUP_WAVES) void group_ids_kernel(const int32_t* __restrict__ ids, int N, int V, int lg,
                                                                     uint32_t* __restrict__ keys, uint32_t* __restrict__ rows,
                                                                     uint32_t* __restrict__ tickets, int n_tickets, int* __restrict__ err) {
    constexpr int W = GROUP_WAVES, QUAD = Q < 4 ? Q : 4;
    __shared__ uint32_t cnt[2][W][GROUP_DIGITS];  // of a wave's own positions: in the parts before this one, in the others
    __shared__ uint32_t below[W], wtot[GROUP_DIGITS / 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = blockIdx.x >> lg;
    const uint32_t mask = (1u << lg) - 1u, b = blockIdx.x & mask, none = ((uint32_t)(V - 1) >> lg) + 1u;  // none: the digit of ids out of range
    const int w0 = wave * (Q * PARTS * 64);
    // Places past the last position hold an id out of range of the last bucket: they come behind everything and are not written.  A wave's
    // resource is its own positions (none: no bytes), all of its offsets lie in the range-checked part: the scalar offset is not checked.
    const int first = w0 < N ? w0 : N;
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc((void*)(ids + first), 0, (N - first) * 4, 0x00020000);
    auto load = [&](uint32_t (&id)[Q], int q) {
#pragma unroll
        for (int u = 0; u < Q; ++u) id[u] = __builtin_amdgcn_raw_buffer_load_b32(src, lane * 4 + (q * Q + u) * 256, 0, 0);
    };
    auto close = [&](uint32_t (&id)[Q], int q) {
        if (w0 + (q * Q + Q) * 64 <= N) return;
#pragma unroll
        for (int u = 0; u < Q; ++u) id[u] = w0 + (q * Q + u) * 64 + lane < N ? id[u] : 0xFFFFFFFFu;
    };
    auto digit = [&](uint32_t k) { return k < (uint32_t)V ? k >> lg : none; };
    uint32_t mine[Q], id[2][Q];
    load(id[0], 0);
    load(mine, part);
    if (threadIdx.x <= none) {
#pragma unroll
        for (int w = 0; w < W; ++w) cnt[0][w][threadIdx.x] = cnt[1][w][threadIdx.x] = 0;
    }
    for (int e = blockIdx.x * 64 * W + threadIdx.x; e < n_tickets; e += gridDim.x * 64 * W) tickets[e] = 0;
    __syncthreads();
    const uint32_t mask4 = mask * 0x01010101u, b4 = b * 0x01010101u;  // (lg <= 7: the high bit of each byte is free)
    uint32_t lower = 0;
#pragma unroll
    for (int q = 0; q < PARTS; ++q) {
        if (q + 1 < PARTS) load(id[(q + 1) & 1], q + 1);
        close(id[q & 1], q);
        uint32_t* __restrict__ to = cnt[q < part ? 0 : 1][wave];
        uint32_t seen = 0, times = 0;  // a lane counts an id that follows itself by itself: most of a frequent one's
#pragma unroll
        for (int u = 0; u < Q; u += QUAD) {
            uint32_t k[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) k[e] = id[q & 1][u + (e < QUAD ? e : 0)];
            uint32_t low = (k[0] & 0xFFu) | (k[1] & 0xFFu) << 8 | (k[2] & 0xFFu) << 16 | k[3] << 24;
            low &= mask4;
            constexpr uint32_t USED = QUAD == 4 ? 0x80808080u : QUAD == 2 ? 0x8080u : 0x80u;
            lower += (uint32_t)__popc(~((low | 0x80808080u) - b4) & USED);  // a byte's high bit stays where it is not below b
            uint32_t eq = ~((low ^ b4) + 0x7F7F7F7Fu) & USED;               // ... where it differs from b
            while (__builtin_amdgcn_ballot_w64(eq != 0)) {  // each lane's next one
                if (eq) {
                    const uint32_t e = __builtin_ctz(eq);
                    const uint32_t x = e < 16 ? (e < 8 ? k[0] : k[1]) : (e < 24 ? k[2] : k[3]);
                    if (x != seen && times) {
                        atomicAdd(&to[digit(seen)], times);
                        times = 0;
                    }
                    seen = x;
                    ++times;
                    eq &= eq - 1;
                }
            }
        }
        if (times) atomicAdd(&to[digit(seen)], times);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lower += (uint32_t)__shfl_xor((int)lower, o, 64);
    if (lane == 0) below[wave] = lower;
    __syncthreads();
    uint32_t total = 0, incl = 0;
    if (threadIdx.x < GROUP_DIGITS) {
        uint32_t x[W], y[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            x[w] = threadIdx.x <= none ? cnt[0][w][threadIdx.x] : 0u;
            y[w] = threadIdx.x <= none ? cnt[1][w][threadIdx.x] : 0u;
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t t = x[w] + y[w];
            x[w] += total;  // where the part's positions of this wave begin
            total += t;
        }
        incl = total;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        if (lane == 63) wtot[wave] = incl;
#pragma unroll
        for (int w = 0; w < W; ++w) cnt[1][w][threadIdx.x] = x[w] + incl - total;
    }
    __syncthreads();
    uint32_t base = 0;  // of the bucket; and, in a digit's thread, of the waves of digits before its own
#pragma unroll
    for (int w = 0; w < W; ++w) base += below[w];
    uint32_t* __restrict__ from = cnt[1][wave];
    uint32_t* __restrict__ keys_b = keys + __builtin_amdgcn_readfirstlane((int)base);
    uint32_t* __restrict__ rows_b = rows + __builtin_amdgcn_readfirstlane((int)base);
    // (places inside 64 digits so far: the digits of the waves before are added here)
    uint32_t pre = 0;
#pragma unroll
    for (int w = 0; w < GROUP_DIGITS / 64; ++w) {
        const uint32_t t = wtot[w];
        if (lane == w) base = pre;
        pre += t;
    }
    bool bad = false;
    close(mine, part);
#pragma unroll
    for (int u = 0; u < Q; ++u) {
        const uint32_t k = mine[u], dgt = digit(k);
        const int p = w0 + (part * Q + u) * 64 + lane;
        const bool own = (k & mask) == b && p < N;
        uint64_t rest = __builtin_amdgcn_ballot_w64(own);
        if (rest == 0) continue;
        const uint32_t at = own ? from[dgt] : 0u, block = (uint32_t)__shfl((int)base, (int)(dgt >> 6), 64);
        uint32_t rank = 0, all = 1;
        if (rest & (rest - 1)) {
            while (rest) {  // one distinct digit after the other
                const uint64_t same = __builtin_amdgcn_ballot_w64(own && dgt == (uint32_t)__builtin_amdgcn_readlane((int)dgt, __builtin_ctzll(rest)));
                if (same >> lane & 1) {
                    rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
                    all = (uint32_t)__popcll(same);
                }
                rest &= ~same;
            }
        }
        if (own) {
            keys_b[at + block + rank] = dgt == none ? (uint32_t)V : k;
            rows_b[at + block + rank] = (uint32_t)p;
            if (rank == 0) from[dgt] = at + all;
            bad |= dgt == none;
        }
    }
    if (bad) atomicOr(err, DP_ERRBIT_INDEX);
}

// Ordered segment sums over the grouped (id, row) list.  A workgroup owns 4 PW positions and 64 VW columns, a wave PW of the positions in
// turn: the factors, row addresses and run ends of its positions sit one a lane and are read back as scalars; 8 rows, and the table rows of the
// runs that end in them, are in flight.  A run that lies inside a wave is added to sum_E there (this wave is its only writer).  What crosses waves is joined in LDS in their order, what crosses workgroups goes to `first`
// (continues from the workgroup before) or `last` (starts here); the workgroup of such a run that takes its last ticket adds those pieces in order:
// wave g the pieces h + 1 + g, h + 5 + g, ... of the run from workgroup h on, then the waves in order.  The order is fixed, only who does it is not.
// Pieces are written and read past the caches of an XCD, and a workgroup's pieces have arrived before it takes its ticket.
// Bound: HBM where there are many positions, otherwise the chain id - row - piece - ticket - piece.  Us, with the sums of the sort's 32-position chunks and the second
// launch that joined them before: B * T = 65,536, d = 1,024 48.8 | 41 + 12 (134 MB of rows, 80 MB of the table), 16,384, d = 768 14.8 | 10 + 7, 464, d = 128 7.3 | 12.
constexpr int SEG_WAVES = 4;

template <int PW, bool BF16, int VW>
__global__ __launch_bounds__(64 * SEG_WAVES) void segment_sums_kernel(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ rows,
                                                           const void* __restrict__ G, const float* __restrict__ sqnorms, float C, int N, int T, int d,
                                                           int V, int ncb, uint32_t* __restrict__ tickets,
                                                           float* __restrict__ sum_E, float* __restrict__ first, float* __restrict__ last,
                                                           int* __restrict__ err) {
    constexpr int WAVES = SEG_WAVES, SEG = WAVES * PW, AHEAD = 8, COLS = 64 * VW;
    static_assert(PW % AHEAD == 0 && PW < 63, "a wave's positions, the one after them and the one before them sit one a lane");
    constexpr uint32_t HEAD = 1, WHOLE = 2, TAIL = 4;  // of a wave: its first run continues one, is its only one and goes on; its last run (another) goes on
    __shared__ float head[WAVES][COLS], tail[WAVES][COLS];
    __shared__ uint32_t flags[WAVES], wkey[WAVES][2], mine[2];
    __shared__ int span[3];  // the run that covers the first position: its first and last workgroup; the last one of the run that covers the position behind
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pc = blockIdx.x / ncb, cb = blockIdx.x - pc * ncb, p0 = pc * SEG, col0 = cb * COLS;
    const int lo = p0 + wave * PW, n = N - lo < 0 ? 0 : N - lo < PW ? N - lo : PW;  // this wave's positions
    // The run that covers position k SEG reaches as many workgroups on (STEP 1) or back (-1) as there is its id at their first positions:
    // the next 64 first, where nearly all end, then 64 at equal distances over all that are left, and so on between two of these (six rounds for
    // any N; a run of n workgroups is looked for by all n of them, 64 after 64 that was 3.6 ms of 2 ids at 4,194,304 positions, d = 64, now 1.2, and
    // 12.3 at twice as many, d = 8, now 2.4).  Ids out of range are added nowhere; theirs are no single run.
    const int nseg = (N + SEG - 1) / SEG;
    auto reach = [&](int k, int step) {
        const uint32_t key = keys[k * SEG];
        if (key >= (uint32_t)V) return k;
        for (int left = step > 0 ? nseg - 1 - k : k, stride = 1;;) {  // the last one with the id is one of the `left` beyond k, or k
            const int m = stride * (lane + 1);
            const uint64_t off = __builtin_amdgcn_ballot_w64(m > left || keys[(m > left ? k : k + step * m) * SEG] != key);
            const int n = off ? __builtin_ctzll(off) : 64;
            k += step * (n * stride);
            left -= n * stride;
            if (n < 64 && left > stride - 1) left = stride - 1;
            if (left == 0) return k;
            stride = (left + 63) / 64;
        }
    };
    if (wave == 0) {
        const int j = reach(pc, -1);
        if (lane == 0) span[0] = j > 0 && keys[j * SEG - 1] == keys[j * SEG] ? j - 1 : j;
    } else if (wave == 1) {
        const int j = reach(pc, 1);
        if (lane == 0) span[1] = j;
    } else if (wave == 2 && pc + 1 < nseg) {
        const int j = reach(pc + 1, 1);
        if (lane == 0) span[2] = j;
    }
    uint32_t flag = 0, k_first = 0, k_last = 0;
    if (n > 0) {
        constexpr int E = BF16 ? 2 : 4;
        const int col = col0 + lane * VW;
        const int p = lane == 63 ? (lo > 0 ? lo - 1 : 0) : lane <= n ? lo + lane : lo;
        const uint32_t key = keys[p < N ? p : N - 1];
        const uint32_t row = rows[lane < n ? lo + lane : lo];
        const float c = dp_clip_factor(sqnorms[row / (uint32_t)T], C);
        if (c != c) atomicOr(err, DP_ERRBIT_NORM);
        const uint64_t addr = (uint64_t)G + ((uint64_t)row * (uint64_t)d + col0) * E;
        const int a_lo = (int)(uint32_t)addr, a_hi = (int)(addr >> 32);
        const uint32_t at = ((col < d ? col : d - VW) - col0) * E;  // (lanes past the width read its last columns again)
        const uint32_t next = (uint32_t)__shfl_down((int)key, 1, 64);
        const uint64_t ends = __builtin_amdgcn_ballot_w64(lane < n && (lo + lane + 1 >= N || next != key));
        k_first = (uint32_t)__builtin_amdgcn_readlane((int)key, 0);
        k_last = (uint32_t)__builtin_amdgcn_readlane((int)key, n - 1);
        const bool from_prev = lo > 0 && (uint32_t)__builtin_amdgcn_readlane((int)key, 63) == k_first;
        // The table row that the run ending at this lane's position is added to: no bytes where none ends, or where it began before this
        // wave, or for ids out of range: such an access touches no memory.
        const bool adds = (ends >> lane & 1) && key < (uint32_t)V && !(from_prev && lane == __builtin_ctzll(ends | 1ull << 63));
        const uint64_t taddr = (uint64_t)sum_E + ((uint64_t)(adds ? key : 0u) * (uint64_t)d + col0) * 4u;
        const int t_lo = (int)(uint32_t)taddr, t_hi = (int)(taddr >> 32), t_len = adds ? (d - col0) * 4 : 0;
        auto table = [&](int k) {
            const uint64_t r = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(t_hi, k) << 32 | (uint32_t)__builtin_amdgcn_readlane(t_lo, k);
            return __builtin_amdgcn_make_buffer_rsrc((void*)r, 0, __builtin_amdgcn_readlane(t_len, k), 0x00020000);
        };
        float acc[VW];  // the run under way
#pragma unroll
        for (int e = 0; e < VW; ++e) acc[e] = 0.f;
        bool begun = from_prev;  // it began before this wave
#pragma unroll
        for (int k0 = 0; k0 < PW; k0 += AHEAD) {
            if (k0 >= n) break;
            RawVec<BF16, VW> g[AHEAD];
            float old[AHEAD][VW];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {  // (lanes past the last position hold the address of the first)
                const uint64_t r = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(a_hi, k0 + u) << 32 | (uint32_t)__builtin_amdgcn_readlane(a_lo, k0 + u);
                g[u] = load_raw<BF16, VW>((rw_global)r, at);
            }
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                if constexpr (VW == 4) {
                    const f32x4_t t = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(table(k0 + u), lane * 16, 0, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) old[u][e] = t[e];
                } else {
                    old[u][0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(table(k0 + u), lane * 4, 0, 0));
                }
            }
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                if (k0 + u >= n) continue;
                const float w = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(c), k0 + u));
#pragma unroll
                for (int e = 0; e < VW; ++e) acc[e] += w * raw_value<BF16, VW>(g[u], e);
                if (!(ends >> (k0 + u) & 1)) continue;
                if (begun) {
                    flag |= HEAD;
#pragma unroll
                    for (int e = 0; e < VW; ++e) head[wave][lane * VW + e] = acc[e];
                } else if constexpr (VW == 4) {
                    const f32x4_t t = {old[u][0] + acc[0], old[u][1] + acc[1], old[u][2] + acc[2], old[u][3] + acc[3]};
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(rw_u32x4, t), table(k0 + u), lane * 16, 0, 0);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(old[u][0] + acc[0]), table(k0 + u), lane * 4, 0, 0);
                }
                begun = false;
#pragma unroll
                for (int e = 0; e < VW; ++e) acc[e] = 0.f;
            }
        }
        if (!(ends >> (n - 1) & 1)) {
            flag |= begun ? HEAD | WHOLE : TAIL;
#pragma unroll
            for (int e = 0; e < VW; ++e) (begun ? head : tail)[wave][lane * VW + e] = acc[e];
        }
    }
    if (lane == 0) {
        flags[wave] = flag;
        wkey[wave][0] = k_first;
        wkey[wave][1] = k_last;
    }
    __syncthreads();
    // Join: a thread per column walks the waves.  First, for all alike, what becomes of each wave's first run: `open`: a run is under way,
    // `in`: it came from the workgroup before; the table rows of the runs that end are asked for here.
    const int c = threadIdx.x < COLS ? threadIdx.x : 0, col = col0 + c;
    const bool on = threadIdx.x < COLS && col < d;
    uint32_t f[WAVES], ends_in[WAVES];  // ends_in[w]: the id of the run that ends in wave w
    bool open = false, in = false, in_piece = false;
    uint32_t open_key = 0;
    float old[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        f[w] = (uint32_t)__builtin_amdgcn_readfirstlane((int)flags[w]);
        ends_in[w] = (uint32_t)V;
        old[w] = 0.f;
        if (f[w] & HEAD) {
            if (!open) {
                open = in = true;
                open_key = (uint32_t)__builtin_amdgcn_readfirstlane((int)wkey[w][0]);
            }
            if (!(f[w] & WHOLE)) {
                if (in) in_piece = open_key < (uint32_t)V;
                else ends_in[w] = open_key;
                open = in = false;
                if (ends_in[w] < (uint32_t)V && on) old[w] = sum_E[(size_t)ends_in[w] * d + col];
            }
        }
        if (f[w] & TAIL) {
            open = true;
            open_key = (uint32_t)__builtin_amdgcn_readfirstlane((int)wkey[w][1]);
        }
    }
    const uint32_t in_key = (uint32_t)__builtin_amdgcn_readfirstlane((int)wkey[0][0]);
    const bool out = open && !in && open_key < (uint32_t)V;  // a run that starts here goes on
    in_piece = in_piece || (open && in && open_key < (uint32_t)V);
    {
        float carry = 0.f;
        bool from_before = f[0] & HEAD;
        auto put = [&](float* dst) {
            if (on) __hip_atomic_store(dst + (size_t)pc * d + col, carry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            if (f[w] & HEAD) {
                carry += head[w][c];
                if (!(f[w] & WHOLE)) {
                    if (from_before && in_piece) put(first);
                    else if (ends_in[w] < (uint32_t)V && on) sum_E[(size_t)ends_in[w] * d + col] = old[w] + carry;
                    from_before = false;
                }
            }
            if (f[w] & TAIL) {
                carry = tail[w][c];
                from_before = false;
            }
        }
        if (out) put(last);
        else if (open && in_piece && in) put(first);
    }
    if (!in_piece && !out) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0 || threadIdx.x == 64) {
        const bool take = threadIdx.x == 0 ? in_piece : out;
        const int h = threadIdx.x == 0 ? span[0] : pc, q = threadIdx.x == 0 ? span[1] : span[2];
        mine[threadIdx.x >> 6] =
            take && __hip_atomic_fetch_add(&tickets[h * ncb + cb], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(q - h) ? 1u : 0u;
    }
    __syncthreads();
    for (int s = 0; s < 2; ++s) {
        if (!__builtin_amdgcn_readfirstlane((int)mine[s])) continue;
        const int h = s == 0 ? span[0] : pc, qlast = s == 0 ? span[1] : span[2];
        const uint32_t key = s == 0 ? in_key : open_key;
        const float was = on ? sum_E[(size_t)key * d + col] : 0.f;
        const int lcol = col0 + lane * VW;
        float acc[VW];
#pragma unroll
        for (int e = 0; e < VW; ++e) acc[e] = 0.f;
        if (lcol < d) {
            constexpr int SC1 = 16;  // past this XCD's caches
            auto piece = [&](const float* src, int q, float (&x)[VW]) {
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(src + (size_t)q * d), 0, d * 4, 0x00020000);
                if constexpr (VW == 4) {
                    const f32x4_t t = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, lcol * 4, 0, SC1));
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = t[e];
                } else {
                    x[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, lcol * 4, 0, SC1));
                }
            };
            float f0[VW];
#pragma unroll
            for (int e = 0; e < VW; ++e) f0[e] = 0.f;
            if (wave == 0) piece(last, h, f0);
            constexpr int AT_ONCE = 8;
            for (int q = h + 1 + wave; q <= qlast; q += AT_ONCE * WAVES) {
                float x[AT_ONCE][VW];
#pragma unroll
                for (int u = 0; u < AT_ONCE; ++u) {
                    if (q + WAVES * u <= qlast) piece(first, q + WAVES * u, x[u]);
                    else
#pragma unroll
                        for (int e = 0; e < VW; ++e) x[u][e] = 0.f;
                }
#pragma unroll
                for (int u = 0; u < AT_ONCE; ++u)
#pragma unroll
                    for (int e = 0; e < VW; ++e) acc[e] += x[u][e];
            }
#pragma unroll
            for (int e = 0; e < VW; ++e) acc[e] += f0[e];
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < VW; ++e) head[wave][lane * VW + e] = acc[e];
        __syncthreads();
        if (on) {
            float t = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) t += head[w][c];
            sum_E[(size_t)key * d + col] = was + t;
        }
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
dp_status dpk_kept_sums_batched(dp_ctx* ctx, int n, float* const* keep, int B, int d, const float* sqnorms, float C, float* const* sum_x,
                                float* const* sum_1) {
    if (B == 0 || d == 0 || n == 0) return DP_OK;
    const bool own = B <= COL_FACTORS;
    if (!own) {
        const dp_status st = dpk_clip_factors(ctx, sqnorms, B, C, ctx->cbuf);
        if (st != DP_OK) return st;
    }
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
        const dim3 grid((unsigned)((2 * d / 4 + 63) / 64), L);
        if (own) hipLaunchKernelGGL(kept_sums_kernel<true>, grid, dim3(256), 0, ctx->stream, ck, co, sqnorms, C, B, d, ctx->err_word);
        else hipLaunchKernelGGL(kept_sums_kernel<false>, grid, dim3(256), 0, ctx->stream, ck, co, ctx->cbuf, C, B, d, ctx->err_word);
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
                                     const float* sqnorms, float C, float* const* out_x, float* const* out_1) {
    const long nrows = (long)B * T;
    const int J = (d + 64 * VW - 1) / (64 * VW);
    int rows_per;
    const long R = colstat_runs(nrows, d, VW, &rows_per);
    const bool direct = R == 1, own = rows_per / T + 2 <= COL_FACTORS;
    if (!own) {
        const dp_status st = dpk_clip_factors(ctx, sqnorms, B, C, ctx->cbuf);
        if (st != DP_OK) return st;
    }
    dp_ws_alloc ws(ctx);
    float* part = direct ? nullptr : ws.get<float>((size_t)L * R * 2 * d);
    if (!direct && !part) {
        DP_SET_ERR(ctx, "workspace too small for column-sum partials (%d x %ld x 2 x %d floats)", L, R, d);
        return DP_ERR_WORKSPACE;
    }
    ColBatch cb;
    ColOut co;
    for (int l = 0; l < COL_MAX_BATCH; ++l) {
        const int src = l < L ? l : 0;
        cb.X[l] = out_x ? X[src] : nullptr;
        cb.G[l] = G[src];
        co.out_x[l] = out_x ? out_x[src] : nullptr;
        co.out_1[l] = out_1 ? out_1[src] : nullptr;
    }
    dim3 grid((unsigned)R, J, L);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, ctx->stream, cb, co, own ? sqnorms : ctx->cbuf, C, T, d, nrows, rows_per, part, direct ? 1 : 0, ctx->err_word);
    };
    if (out_x && own) launch(colstat_sums_kernel<BF16, VW, true, true>);
    else if (out_x) launch(colstat_sums_kernel<BF16, VW, true, false>);
    else if (own) launch(colstat_sums_kernel<BF16, VW, false, true>);
    else launch(colstat_sums_kernel<BF16, VW, false, false>);
    DP_LAUNCH_CHECK(ctx, "colstat_sums");
    if (direct) return DP_OK;
    bool pair = out_x && out_1 && d % 4 == 0 && R >= 32 && d <= 32768 && ((uintptr_t)part & 15) == 0;
    for (int l = 0; pair && l < L; ++l) pair = (((uintptr_t)out_x[l] | (uintptr_t)out_1[l]) & 15) == 0;
    if (pair) {
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
                                   int d, const float* sqnorms, float C, float* const* out_x, float* const* out_1) {
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
        if (dt == DP_BF16) st = colstat_sums_launch<true, 4>(ctx, L, Xl, G + l0, B, T, d, sqnorms, C, ox, o1);
        else if (v4) st = colstat_sums_launch<false, 4>(ctx, L, Xl, G + l0, B, T, d, sqnorms, C, ox, o1);
        else st = colstat_sums_launch<false, 1>(ctx, L, Xl, G + l0, B, T, d, sqnorms, C, ox, o1);
        if (st != DP_OK) return st;
    }
    return DP_OK;
}

dp_status dpk_colstat_sums(dp_ctx* ctx, const void* X, const void* G, dp_dtype dt, int B, int T, int d, const float* sqnorms, float C,
                           float* out_x, float* out_1) {
    return dpk_colstat_sums_batched(ctx, 1, &X, &G, dt, B, T, d, sqnorms, C, out_x ? &out_x : nullptr, out_1 ? &out_1 : nullptr);
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
    const size_t lds = (((size_t)T + 3) / 4 * 4 + emb_shared_ranks(T)) * sizeof(uint32_t) + (size_t)T * sizeof(uint16_t);
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
    const int ncb = (d + 64 * VW - 1) / (64 * VW);
    // Positions a wave: 8 while that does not fill the chip (B * T = 8,192, d = 768: 29.5 us the call with 8, 31.6 with 16, 34.6 with 32),
    // 16, and 32 once it does twice over (65,536, d = 1,024: 113 | 102 | 99); 32 also where few ids make long runs, whose pieces
    // are what the last of their workgroups adds (32,768 of 2 ids: 102 | 68 | 55).
    const long tiles = Nl * ncb;
    // (What a choice needs of the workspace is no more than two pairs of lists, a radix sort's counters and two rows per 32 positions.)
    const bool group = N <= GROUP_MAX_N && V <= GROUP_MAX_V;
    const int pw = !group || ncb > 64 || tiles > 131072 || Nl >= 256l * V ? 32 : tiles > 32768 ? 16 : 8;
    const int seg = SEG_WAVES * pw, nseg = (N + seg - 1) / seg;
    dp_ws_alloc ws(ctx);
    uint32_t* k0 = ws.get<uint32_t>(N);
    uint32_t* v0 = ws.get<uint32_t>(N);
    uint32_t* tickets = ws.get<uint32_t>((size_t)nseg * ncb);
    float* first = ws.get<float>((size_t)nseg * d);
    float* last = ws.get<float>((size_t)nseg * d);
    uint32_t *k1 = nullptr, *v1 = nullptr, *hist = nullptr;
    const int nsort = (N + SORT_CHUNK - 1) / SORT_CHUNK;
    int pitch = sort_pitch(nsort);
    if (!group) {
        k1 = ws.get<uint32_t>(N);
        v1 = ws.get<uint32_t>(N);
        hist = ws.get<uint32_t>((size_t)256 * pitch);
        if (!hist) hist = ws.get<uint32_t>((size_t)256 * (pitch = nsort));  // without padding when there is no room for it: the scan takes any pitch
    }
    if (!k0 || !v0 || !tickets || !first || !last || (!group && (!k1 || !v1 || !hist))) {
        DP_SET_ERR(ctx, "workspace too small for the embedding sort of %d tokens", N);
        return DP_ERR_WORKSPACE;
    }
    const dim3 block(256);
    if (group) {
        const int lg = group_bits(V);
        auto launch = [&](auto kernel, int parts) {
            hipLaunchKernelGGL(kernel, dim3(parts << lg), dim3(64 * GROUP_WAVES), 0, ctx->stream, ids, N, V, lg, k0, v0, tickets, nseg * ncb, ctx->err_word);
        };
        if (N <= 64 * GROUP_WAVES) launch(group_ids_kernel<1, 1>, 1);
        else if (N <= 4 * 64 * GROUP_WAVES) launch(group_ids_kernel<1, 4>, 4);
        else if (N <= 8 * 64 * GROUP_WAVES) launch(group_ids_kernel<2, 4>, 4);
        else if (N <= 16 * 64 * GROUP_WAVES) launch(group_ids_kernel<4, 4>, 4);
        else if (N <= 32 * 64 * GROUP_WAVES) launch(group_ids_kernel<8, 4>, 4);
        else launch(group_ids_kernel<16, 4>, 4);
        DP_LAUNCH_CHECK(ctx, "group_ids");
    } else {
        const int bits = bit_length((uint32_t)V);  // the sentinel V itself must be representable
        const bool scan = nsort > SORT_INLINE || pitch % 4 != 0;
        const dim3 grid(nsort);
        for (int shift = 0; shift < bits; shift += 8) {
            const uint32_t* kin = shift ? k0 : reinterpret_cast<const uint32_t*>(ids);
            if (shift) hipLaunchKernelGGL((sort_hist<false>), grid, block, 0, ctx->stream, kin, N, V, shift, hist, nsort, pitch, tickets, nseg * ncb, ctx->err_word);
            else hipLaunchKernelGGL((sort_hist<true>), grid, block, 0, ctx->stream, kin, N, V, shift, hist, nsort, pitch, tickets, nseg * ncb, ctx->err_word);
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
    }
    auto sums = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(nseg * ncb)), block, 0, ctx->stream, k0, v0, G, sqnorms, C, N, T, d, V, ncb, tickets, sum_E, first, last, ctx->err_word);
    };
    if (pw == 8) sums(segment_sums_kernel<8, BF16, VW>);
    else if (pw == 16) sums(segment_sums_kernel<16, BF16, VW>);
    else sums(segment_sums_kernel<32, BF16, VW>);
    DP_LAUNCH_CHECK(ctx, "segment_sums");
    return DP_OK;
}

dp_status dpk_embedding_sums(dp_ctx* ctx, const int32_t* ids, const void* G, dp_dtype dt, int B, int T, int d, int V,
                             const float* sqnorms, float C, float* sum_E) {
    if (B == 0 || T == 0 || d == 0) return DP_OK;
    if (dt == DP_BF16) return embedding_sums_launch<true, 4>(ctx, ids, G, B, T, d, V, sqnorms, C, sum_E);
    if (vec4_ok(dt, d, G, G)) return embedding_sums_launch<false, 4>(ctx, ids, G, B, T, d, V, sqnorms, C, sum_E);
    return embedding_sums_launch<false, 1>(ctx, ids, G, B, T, d, V, sqnorms, C, sum_E);
}
