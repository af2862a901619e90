// Per-example squared norm of a dense layer's weight (and bias) gradient from Gram matrices:
//     ||A_i^T G_i||_F^2 = sum_{t,s} (a_t . a_s)(g_t . g_s),      ||sum_t g_t||^2 = sum_{t,s} g_t . g_s
// (the identity follows from the outer-product form of a dense layer's gradient, Section 4.3).
//
// bf16 kernel: one workgroup (4 waves) owns a 128 x 128 block (tb, sb), tb <= sb, of one example's T x T
// plane.  It forms that block of A A^T (contraction over d_in) and of G G^T (over d_out) with
// v_mfma_f32_32x32x16_bf16, both operands being rows of the same tensor with the contraction index
// contiguous in memory (the layout MFMA wants: no transpose anywhere), then multiplies the two
// accumulator sets element by element in registers.  Symmetry halves the work: blocks below the diagonal
// are never launched, and inside a diagonal block the lower-left wave quadrant is skipped while the
// upper-right one counts twice.
//
// Roofline: HBM at T = 128 (2*T*(d_in+d_out) bytes per example against 2*T^2*(d_in+d_out) flops, i.e.
// T flop/B, below the machine balance of ~310 flop/B); each row panel is read once per block it is in.
#include <type_traits>

#include "dp_common.h"

namespace {

constexpr int GB = 128;       // block edge in the (t, s) plane
constexpr int GK = 64;        // contraction chunk staged per step
constexpr int GLD = GK + 8;   // LDS row pitch in bf16 elements (144 B: 16-byte reads of consecutive rows
                              // fall into distinct banks)

struct GramStage {
    uint4 r[4];  // row panel: 4 x 16 B per thread
    uint4 c[4];  // column panel (off-diagonal blocks only)
};

// Load one GK-wide chunk of a 128-row panel of X (rows row0.., all of example `ex`) into registers.
__device__ __forceinline__ void gram_load_panel(const uint16_t* __restrict__ X, size_t ex_base, int row0, int T, int d,
                                                int k0, uint4 v[4]) {
    const int tid = threadIdx.x;
    const int kc = k0 + (tid & 7) * 8;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = row0 + (tid >> 3) + 32 * j;
        if (row < T && kc < d)
            v[j] = *reinterpret_cast<const uint4*>(X + ex_base + (size_t)row * d + kc);
        else
            v[j] = make_uint4(0u, 0u, 0u, 0u);
    }
}

__device__ __forceinline__ void gram_store_panel(uint16_t* __restrict__ panel, const uint4 v[4]) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = (tid >> 3) + 32 * j;
        *reinterpret_cast<uint4*>(panel + row * GLD + (tid & 7) * 8) = v[j];
    }
}

__device__ __forceinline__ bf16x8_t gram_frag(const uint16_t* __restrict__ panel, int row, int koff) {
    const uint4 w = *reinterpret_cast<const uint4*>(panel + row * GLD + koff);
    return __builtin_bit_cast(bf16x8_t, w);
}

// Accumulate the (tb, sb) block of X X^T into acc[2][2] (this wave's 64 x 64 quadrant).
template <bool OFFDIAG>
__device__ __forceinline__ void gram_accumulate(const uint16_t* __restrict__ X, size_t ex_base, int T, int d, int tb,
                                                int sb, uint16_t* __restrict__ lds, bool active, int wr, int wc,
                                                f32x16_t acc[2][2]) {
    // LDS layout: [stage][panel(0=row,1=col)][128][GLD]
    constexpr int PANEL = GB * GLD;
    constexpr int STAGE = (OFFDIAG ? 2 : 1) * PANEL;
    const int lane = threadIdx.x & 63;
    const int nch = (d + GK - 1) / GK;
    GramStage st;
    gram_load_panel(X, ex_base, tb * GB, T, d, 0, st.r);
    if (OFFDIAG) gram_load_panel(X, ex_base, sb * GB, T, d, 0, st.c);
    __syncthreads();  // the previous contraction's readers are done with stage 0
    gram_store_panel(lds, st.r);
    if (OFFDIAG) gram_store_panel(lds + PANEL, st.c);
    __syncthreads();
    for (int ch = 0; ch < nch; ++ch) {
        const uint16_t* cur = lds + (ch & 1) * STAGE;
        uint16_t* nxt = lds + ((ch + 1) & 1) * STAGE;
        const bool more = ch + 1 < nch;
        if (more) {
            gram_load_panel(X, ex_base, tb * GB, T, d, (ch + 1) * GK, st.r);
            if (OFFDIAG) gram_load_panel(X, ex_base, sb * GB, T, d, (ch + 1) * GK, st.c);
        }
        if (active) {
            const uint16_t* rp = cur;
            const uint16_t* cp = OFFDIAG ? cur + PANEL : cur;
#pragma unroll
            for (int kk = 0; kk < GK / 16; ++kk) {
                const int koff = kk * 16 + (lane >> 5) * 8;
                bf16x8_t fr[2], fc[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    fr[u] = gram_frag(rp, wr * 64 + u * 32 + (lane & 31), koff);
                    fc[u] = gram_frag(cp, wc * 64 + u * 32 + (lane & 31), koff);
                }
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[mt], fc[nt], acc[mt][nt], 0, 0, 0);
            }
        }
        if (more) {
            gram_store_panel(nxt, st.r);
            if (OFFDIAG) gram_store_panel(nxt + PANEL, st.c);
        }
        __syncthreads();
    }
}

template <bool OFFDIAG>
__device__ __forceinline__ float gram_block(const uint16_t* __restrict__ A, const uint16_t* __restrict__ G, int i, int T,
                                            int d_in, int d_out, int tb, int sb, float bias_term, uint16_t* lds) {
    const int wave = threadIdx.x >> 6;
    const int wr = wave >> 1, wc = wave & 1;
    const bool diag = tb == sb;
    const bool active = !(diag && wr > wc);
    const float weight = diag ? (wr == wc ? 1.f : (wr < wc ? 2.f : 0.f)) : 2.f;
    f32x16_t accA[2][2], accG[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) accA[a][b][r] = accG[a][b][r] = 0.f;
    gram_accumulate<OFFDIAG>(A, (size_t)i * T * d_in, T, d_in, tb, sb, lds, active, wr, wc, accA);
    gram_accumulate<OFFDIAG>(G, (size_t)i * T * d_out, T, d_out, tb, sb, lds, active, wr, wc, accG);
    float s = 0.f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) s += (accA[a][b][r] + bias_term) * accG[a][b][r];
    return s * weight;
}

// grid: npairs == 1: one workgroup per example.  npairs > 1: workgroup id g -> XCD g % 8 (hardware
// round-robin); all block pairs of an example are given ids of one XCD so that the example's row panels,
// each needed by several pairs, are served by that XCD's L2:  example = (g / 8 / npairs) * 8 + g % 8.
__global__ __launch_bounds__(256, 2) void gram_bf16_kernel(const uint16_t* __restrict__ A,
                                                           const uint16_t* __restrict__ G, int B, int T, int d_in,
                                                           int d_out, int has_bias, int nblk, int npairs,
                                                           float* __restrict__ out, int direct) {
    extern __shared__ __attribute__((aligned(16))) uint16_t gram_lds[];
    __shared__ float wred[4];
    int i, pair;
    if (npairs == 1) {
        i = blockIdx.x;
        pair = 0;
    } else {
        const int g = blockIdx.x;
        const int slot = g >> 3;
        i = (slot / npairs) * 8 + (g & 7);
        pair = slot % npairs;
        if (i >= B) return;
    }
    int tb = 0, sb = 0;
    {
        int p = pair;
        while (p >= nblk - tb) {  // row tb of the upper triangle holds nblk - tb pairs
            p -= nblk - tb;
            ++tb;
        }
        sb = tb + p;
    }
    const float bias_term = has_bias ? 1.f : 0.f;
    float s;
    if (tb == sb) s = gram_block<false>(A, G, i, T, d_in, d_out, tb, sb, bias_term, gram_lds);
    else s = gram_block<true>(A, G, i, T, d_in, d_out, tb, sb, bias_term, gram_lds);
    const float tot = dp_block_sum<256>(s, wred);
    if (threadIdx.x == 0) {
        if (direct) out[i] += tot;
        else out[(size_t)i * npairs + pair] = tot;
    }
}

// ------------------------------------------------------------------------------------------------
// T <= 128 (one block per example): the same computation with the row panels streamed straight into an LDS ring (2 to 9
// stages of 8 to 32 KiB, by the form) by LDS-filling buffer loads, all but one stage in flight per workgroup (the
// register-staged kernel above keeps one chunk: at two workgroups per CU that is too few bytes in flight to cover the
// HBM latency at full bandwidth).  The loads go through inline assembly so that the wave
// waits (vmcnt) for the chunk it is about to publish only, not for every load in flight.
// LDS layout: [64 or 128 rows][8 or 16 chunks of 16 B], chunk position c of row r holds global chunk c ^ ((r >> 1) & 7), or
// c ^ (r & 15) with 16 chunks: the 16-byte reads of 16 consecutive rows then fall into 64 distinct banks.
// ------------------------------------------------------------------------------------------------
typedef int gram_i32x4 __attribute__((ext_vector_type(4)));

// STREAM: non-temporal hint, for data that no other workgroup reads again (every byte of a T <= 128 example is read
// once; +4 % there).  The units of a longer example share their panels through L2 and must not use it, nor do rows that do not begin
// and end on the 128-byte lines: a line that two chunks or rows share is read twice then (T = 128, 200 x 1000, B = 500: 46 us with
// the hint, 37 without; 12 layers, B = 200: 185 | 146).
template <bool STREAM>
__device__ __forceinline__ void gram_dma16(gram_i32x4 rsrc, uint32_t lds_byte_addr, int voff, int soff) {
    if (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                     :
                     : "s"(lds_byte_addr), "v"(voff), "s"(rsrc), "s"(soff)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :
                     : "s"(lds_byte_addr), "v"(voff), "s"(rsrc), "s"(soff)
                     : "memory", "m0");
}

__device__ __forceinline__ gram_i32x4 gram_rsrc(const void* base, uint32_t bytes) {
    const uint64_t p = (uint64_t)base;
    gram_i32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
    r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    r[3] = 0x00020000;
    return r;
}

// Waits until at most the newest min(m, K) stages of LPS loads are in flight (they land in the order they were issued).  Nothing is
// issued past the last stage, so towards the end fewer than K are: stages of zeros that kept one count for all iterations cost a
// layer of two chunks as much as its work (12 layers of 64 x 64, B = 500, T = 33: 78 -> 70 us; 8 x 100 x 72 x 136: 11.4 -> 10.9).
template <int LPS, int K>
__device__ __forceinline__ void gram_wait(int m) {
    if constexpr (K > 0) {
        if (m < K) return gram_wait<LPS, K - 1>(m);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(K * LPS) : "memory");
}

// An offset outside every example's byte range (below 2^31): such a lane's 16 bytes of LDS receive zeros.
constexpr int GRAM_OUTSIDE = (int)0x80000000u;

// GDK: contraction chunk per stage (a row segment of 2*GDK bytes per load); NS: ring stages.
// Up to GRAM_MAX_BATCH same-shaped layers per launch: workgroup g works on example g % B of layer g / B.  More
// workgroups than the chip holds at once keep the memory pipeline full across examples (one round of 512
// workgroups spends a fifth of its time filling and draining it), and with few examples many layers are what fills the chip
// at all (48 layers of 768 x 768, B = 8: three launches of 16 layers 53 us, one 27).
constexpr int GRAM_MAX_BATCH = 64;
struct GramBatch {
    const uint16_t* A[GRAM_MAX_BATCH];
    const uint16_t* G[GRAM_MAX_BATCH];
    // layers that share their input (Q, K, V of one block): entry l stands for n_out layers with input A[l] and
    // output gradients G[l], G2[l], G3[l].  Their norms add up to <A A^T (+1), sum_j G_j G_j^T>, so A A^T is formed
    // once and the G_j chunks all go into one accumulator (T <= 128 kernel only).
    const uint16_t* G2[GRAM_MAX_BATCH];
    const uint16_t* G3[GRAM_MAX_BATCH];
    int n_out;
    int n_layers;
    int B;
};

// out: n_layers == 1: sqnorms, "+="; otherwise partials [B][n_layers], stored.
// ROWS: rows of a panel, 128 (four quadrants of 64 x 64, one of them the mirror of another) or 64 (one).  The WAVES waves are
// dealt to the quadrants and, where that leaves several to a quadrant, to the k steps of a chunk (their accumulators meet in LDS
// at the end): a wave alone on its SIMD waits for its fragments k step by k step, 1.4 us a chunk, so with 128 rows and a
// workgroup or less per CU 8 waves take half the k steps each (12 layers of 768 x 3072, B = 8: 41 -> 36 us; a deeper ring
// alone changed nothing), and with 64 rows, where one wave of four had work, all four take a quarter each (4 layers of
// 192 x 2264, B = 106, T = 47: 42 -> 30 us).
// The next k step's fragments are read while one multiplies, those of a diagonal quadrant once for rows and columns, and a
// stage's loads are issued behind the first fragments (12 layers of 768 x 3072, B = 8: 36.6 -> 34.6 us; one layer of 768 x 768,
// B = 8: 16.7 -> 15.7; 8 layers of 1024 x 1024, B = 512: the same within the runs of one side, 320 us, 6.7 TB/s).
// RAGGED: a width that is no multiple of GDK; what lies past a row's end in its last chunk is left out lane by lane.
template <int ROWS, int GDK, int NS, int WAVES, int WGS_PER_CU, bool RAGGED>
__global__ __launch_bounds__(64 * WAVES, WGS_PER_CU * WAVES / 4) void gram_dma_kernel(GramBatch gb, int T, int d_in, int d_out,
                                                                   int has_bias, float* __restrict__ out) {
    constexpr int STAGE = ROWS * GDK;      // bf16 elements per stage
    constexpr int CPR = GDK / 8;           // 16-byte chunks per row (8 or 16)
    constexpr int RPI = 64 / CPR;          // rows filled by one wave-wide load
    constexpr int LPS = ROWS / RPI / WAVES;  // loads per wave per stage
    constexpr int NQ = ROWS == 128 ? 4 : 1, KS = WAVES / NQ;  // quadrants, waves that share a quadrant's k steps
    constexpr bool EXACT = WAVES < 8;  // nothing issued past the last stage (eight waves: many stages, where the test costs 2 % and gives nothing)
    static_assert(LPS >= 1 && GDK / 16 >= KS, "more waves than there is work");
    constexpr int XCH = 2 * (NQ == 1 ? 3 : 4) * 16 * 64;  // floats that a wave hands over
    static_assert(NS * STAGE * 2 >= NQ * (KS / 2) * XCH * 4, "the ring doubles as the exchange buffer");
    __shared__ __attribute__((aligned(16))) uint16_t ring[NS][STAGE];
    __shared__ float wred[WAVES];
    const int layer = blockIdx.x / gb.B, i = blockIdx.x - layer * gb.B;
    const uint16_t* __restrict__ A = gb.A[layer];
    const uint16_t* __restrict__ G = gb.G[layer];
    const int tid = threadIdx.x, lane = tid & 63, wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int quad = NQ == 1 ? 0 : KS == 1 ? wave : wave % NQ, kg = KS == 1 ? 0 : wave / NQ, wr = quad >> 1, wc = quad & 1;
    const bool active = wr <= wc;  // the lower-left quadrant mirrors the upper-right one
    const bool diagw = wr == wc;   // ... and inside a diagonal quadrant the lower-left 32 x 32 tile the upper-right one
    const int nchA = (d_in + GDK - 1) / GDK, nchG1 = (d_out + GDK - 1) / GDK, nch = nchA + gb.n_out * nchG1;
    // chunk position c of row r holds global chunk c ^ swz(r): 16 consecutive rows -> 64 distinct banks
    auto swz = [](int r) { return CPR == 8 ? (r >> 1) & 7 : r & 15; };

    // rows >= T of the panel lie outside the example's byte range and read as zero
    const gram_i32x4 rA = gram_rsrc(A + (size_t)i * T * d_in, (uint32_t)((size_t)T * d_in * 2));
    const gram_i32x4 rG = gram_rsrc(G + (size_t)i * T * d_out, (uint32_t)((size_t)T * d_out * 2));
    const gram_i32x4 rG2 = gram_rsrc((gb.n_out > 1 ? gb.G2[layer] : G) + (size_t)i * T * d_out, (uint32_t)((size_t)T * d_out * 2));
    const gram_i32x4 rG3 = gram_rsrc((gb.n_out > 2 ? gb.G3[layer] : G) + (size_t)i * T * d_out, (uint32_t)((size_t)T * d_out * 2));
    // load j of this wave fills rows (LPS*wave + j)*RPI .. : lane l -> row + l/CPR, chunk position l%CPR
    int voffA[LPS], voffG[LPS];
    uint32_t ldsoff[LPS];
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        const int row0 = (LPS * wave + j) * RPI, row = row0 + lane / CPR;
        const int cg = (lane % CPR) ^ swz(row);
        voffA[j] = (row * d_in + cg * 8) * 2;
        voffG[j] = (row * d_out + cg * 8) * 2;
        ldsoff[j] = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)&ring[0][row0 * GDK];
    }
    int ibuf = 0;  // buffer of the next stage to issue
    const int rotA = i % nchA, rotG = i % nchG1;
    auto issue = [&](int st) {
        if (EXACT && st >= nch) return;
        const bool isA = st < nchA;
        const int cgi = st - nchA;                                             // chunk index over all output gradients
        const int which = cgi >= 2 * nchG1 ? 2 : (cgi >= nchG1 ? 1 : 0);       // which of the (up to three) tensors
        // The chunks of a tensor are taken in an order rotated by the example index: the contraction does not care, and
        // workgroups that start together (and advance in step) then read different column ranges at any moment.  With one
        // order for all, every workgroup reads the same 256 bytes of rows that lie 2-8 KiB apart, i.e. the same few memory
        // channels (+12 % bandwidth on 1024 x 4096 layers, +2 % on 1024 x 1024).
        const int c0 = isA ? st : cgi - which * nchG1, nc = isA ? nchA : nchG1, r0 = isA ? rotA : rotG;
        const int cr = c0 + r0 >= nc ? c0 + r0 - nc : c0 + r0;
        const int soff = __builtin_amdgcn_readfirstlane(cr * GDK * 2);
        // one choice of the source per stage, then a straight run of loads (every descriptor is a variable of its own
        // and stays in scalar registers; with the choice inside the loop each load of an output-gradient stage went
        // through a chain of branches)
        const int left = st >= nch ? 0 : (isA ? d_in : d_out) - cr * GDK;  // columns of the row from this chunk on; past the end: none
        auto run = [&](const gram_i32x4& rs, const int (&voff)[LPS], int so) {
#pragma unroll
            for (int j = 0; j < LPS; ++j) {
                int v = voff[j];
                if (RAGGED && ((lane % CPR) ^ swz((LPS * wave + j) * RPI + lane / CPR)) * 8 >= left) v = GRAM_OUTSIDE;  // past the row's end: zeros
                gram_dma16<!RAGGED>(rs, __builtin_amdgcn_readfirstlane(ldsoff[j] + ibuf * (STAGE * 2)), v, so);
            }
        };
        const bool past = !EXACT && st >= nch;
        if (isA) run(rA, voffA, soff);
        else if (past || which == 0) {
            if constexpr (EXACT) {
                run(rG, voffG, soff);
            } else {  // past the end: a resource of no bytes reads zeros and keeps the load count uniform (a scalar offset is not range-checked)
                gram_i32x4 rg = rG;
                rg[2] = past ? 0 : rG[2];
                run(rg, voffG, soff);
            }
        } else if (which == 1) run(rG2, voffG, soff);
        else run(rG3, voffG, soff);
        ibuf = ibuf + 1 == NS ? 0 : ibuf + 1;
    };
    // fragment addresses (elements) inside a stage for k step 0
    int fr[2], fc[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int r = wr * 64 + u * 32 + (lane & 31), c = wc * 64 + u * 32 + (lane & 31);
        fr[u] = r * GDK + (((lane >> 5) ^ swz(r)) << 3);
        fc[u] = c * GDK + (((lane >> 5) ^ swz(c)) << 3);
    }
    f32x16_t accA[2][2], accG[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) accA[a][b][r] = accG[a][b][r] = 0.f;

#pragma unroll
    for (int st = 0; st < NS - 1; ++st) issue(st);
    int cbuf = 0, s = 0;
    // The multiply of one stage is straight-line code: which Gram matrix it feeds and whether the wave owns a diagonal
    // quadrant are decided outside it (a branch per MFMA pair otherwise).
    auto compute = [&](f32x16_t (&acc)[2][2], auto diag_tag) {
        constexpr bool DG = decltype(diag_tag)::value;
        const uint16_t* st = ring[cbuf];
        constexpr int STEPS = GDK / 16 / KS;
        bf16x8_t a[2][2], b[2][2];  // [step % 2]: the next step's fragments are on their way while one multiplies
        auto fragments = [&](int step) {
            const int kk = step * KS + kg;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                // k chunk 2*kk + lane/32: its swizzled position differs from the kk = 0 one by XOR 2*kk
                const int xr = fr[u] ^ ((2 * kk) << 3), xc = fc[u] ^ ((2 * kk) << 3);
                a[step & 1][u] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(st + xr));
                if (DG) b[step & 1][u] = a[step & 1][u];  // rows and columns of a diagonal quadrant are the same
                else b[step & 1][u] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(st + xc));
            }
        };
        fragments(0);
        issue(s + NS - 1);
#pragma unroll
        for (int step = 0; step < STEPS; ++step) {
            if (step + 1 < STEPS) fragments(step + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    if (!(DG && mt == 1 && nt == 0))
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[step & 1][mt], b[step & 1][nt], acc[mt][nt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto phase = [&](int end, f32x16_t (&acc)[2][2]) {
        for (; s < end; ++s) {
            // my loads of chunk s have landed (later chunks may be in flight); after the barrier everyone's have,
            // and everyone is done reading chunk s-1, whose buffer the newest chunk overwrites
            if constexpr (EXACT) gram_wait<LPS, NS - 2>(nch - 1 - s);
            else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * LPS) : "memory");
            __syncthreads();
            if (!active) issue(s + NS - 1);
            else if (diagw) compute(acc, std::true_type{});
            else compute(acc, std::false_type{});
            cbuf = cbuf + 1 == NS ? 0 : cbuf + 1;
        }
    };
    phase(nchA, accA);
    phase(nch, accG);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may still be writing LDS when the workgroup ends, or when it is reused
    // The k groups' sums meet pairwise: groups KS/2 .. hand theirs to groups 0 .., then the same with half as many.  (A wave whose
    // quadrant is the whole plane leaves out the tile below the diagonal, which holds zeros.)
    auto each = [&](auto f) {
        int e = 0;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                if (NQ == 1 && a == 1 && b == 0) continue;
                f(accA[a][b], e++);
                f(accG[a][b], e++);
            }
    };
#pragma unroll
    for (int half = KS / 2; half > 0; half /= 2) {
        float* part = reinterpret_cast<float*>(&ring[0][0]) + (quad * half + kg % half) * XCH + lane;
        __syncthreads();
        if (kg >= half && kg < 2 * half)
            each([&](f32x16_t& x, int e) {
#pragma unroll
                for (int r = 0; r < 16; ++r) part[(e * 16 + r) * 64] = x[r];
            });
        __syncthreads();
        if (kg < half)
            each([&](f32x16_t& x, int e) {
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] += part[(e * 16 + r) * 64];
            });
    }
    const float bias_term = has_bias ? 1.f : 0.f;
    float sum = 0.f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                sum += (a == 0 && b == 1 && diagw ? 2.f : 1.f) * ((accA[a][b][r] + bias_term) * accG[a][b][r]);  // skipped tiles hold zeros
    sum *= kg > 0 ? 0.f : wr == wc ? 1.f : (wr < wc ? 2.f : 0.f);
    const float tot = dp_block_sum<64 * WAVES>(sum, wred);
    if (threadIdx.x == 0) {
        if (gb.n_layers == 1) out[i] += tot;
        else out[(size_t)i * gb.n_layers + layer] = tot;
    }
}

// ------------------------------------------------------------------------------------------------
// 128 < T <= 2048: the panels of a 64-wide contraction chunk go straight into an LDS ring (no staging
// registers, no LDS store instructions), as in the kernel above.  At this size the contraction, not HBM, is the bound on
// paper (T flop per byte against ~310 at the machine balance); in practice it is the path that fills the LDS (a CU takes
// about 120 GB/s from L2 this way, and a panel costs 16 KiB per stage) together with the matrix pipe.  A
// workgroup of 8 waves (two per SIMD, one workgroup per CU) works on a UNIT of cells of the example's T x T plane, cut into
// 128 x 128 cells of which only the upper triangle is formed (by symmetry a cell (R, C) with C < R stands for (C, R)):
//  * a DIAGONAL BLOCK: the three cells (a, a), (a, b), (b, b) of two neighbouring panels a, b = a + 1 - two panel fills
//    for three cells.  The two diagonal cells need only the tiles on and above their diagonals, so the block has 136
//    tiles of 16 x 16 where two full cells have 128, and they fit the same registers: cut into 64-wide strips the block
//    is a 4 x 4 triangle of quadrants; waves 0-5 take the six quadrants off the diagonal (16 tiles each), waves 6 and 7
//    two diagonal quadrants each (2 x 10 tiles; both operands of such a quadrant are the same fragments).
//  * a ROW PAIR: two cells (R, C1), (R, C2) that share their row panel R, which is filled once for both: three panel fills
//    where two workgroups with a cell each fill four (two when the leading cell is the diagonal one, C1 == R).  Waves 0-3
//    own the 64 x 64 quadrants of the first cell, waves 4-7 those of the second; a leading diagonal cell skips its
//    lower-left quadrant and the mirrored tiles of its diagonal quadrants.
// Over the upper triangle of a 4 x 4 plane that is 2 blocks and 2 row pairs: 10 panel fills and 4 workgroups where a
// workgroup per cell needs 16 and 10.  A ring that uses all of the LDS for stages in flight (three stages of 48 KiB
// for three panels, five of 32 KiB for two) covers the latency of the fills: every panel comes from HBM once, the units
// of an example share it through L2.
// ------------------------------------------------------------------------------------------------
constexpr int GU_K = 64;         // contraction chunk per stage
constexpr int GU_LDS = 5 * 2 * GB * GU_K;  // bf16 elements of the ring: 160 KiB, all of a CU's LDS
// Ring stages by the number of panels a stage holds (48, 32 or 16 KiB a stage): a fill that misses L2 takes a few
// microseconds, so a unit with fewer panels per stage runs further ahead.
__host__ __device__ constexpr int gu_stages(int npl) { return npl == 3 ? 3 : (npl == 2 ? 5 : 10); }
constexpr int GU_MAX_BLK = 16;   // T <= 2048
constexpr int GU_MAX_UNITS = GU_MAX_BLK * (GU_MAX_BLK + 1) / 4 + 1;
struct GramUnits {
    int n_units;
    // row pair: R | C1 << 8 | C2 << 16 (C2 == 255: the unit has one cell only); diagonal block of panels a, b: a | a << 8 | b << 16 | 1 << 24
    uint32_t rc[GU_MAX_UNITS];
};

// NPL: panels filled per stage (1: a diagonal cell alone; 2: a diagonal block, a diagonal cell + one more of its row, or
// one off-diagonal cell; 3: two off-diagonal cells).  BLK: the unit is a diagonal block (cells (R, R), (R, C2), (C2, C2)).
template <int NPL, bool BLK, bool RAGGED>
__device__ __forceinline__ float gram_unit_ring(const uint16_t* __restrict__ A, const uint16_t* __restrict__ G, int T, int d_in,
                                                int d_out, int R, int C1, int C2, float bias_term, uint16_t* ring) {
    static_assert(!BLK || NPL == 2, "a diagonal block has two panels");
    constexpr int PANEL = GB * GU_K;   // bf16 elements of one panel of a stage
    constexpr int STAGE = NPL * PANEL; // ... of one stage: its NPL panels side by side
    constexpr int GU_NS = gu_stages(NPL);
    static_assert(GU_NS * STAGE <= GU_LDS, "ring exceeds the LDS array");
    constexpr int LPP = 2;             // loads per wave per panel: 8 rows of 8 chunks each, 16 loads a panel
    constexpr int LPS = NPL * LPP;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cell = wave >> 2, wr = (wave >> 1) & 1, wc = wave & 1;
    const bool diag0 = C1 == R, two = C2 != 255;
    // panels of a stage, in this order: rows R; rows C1 when the first cell is off the diagonal; rows C2 when there is a second cell
    const bool active = BLK || (cell == 0 ? (!diag0 || wr <= wc) : two);
    const bool diagw = !BLK && cell == 0 && diag0 && wr == wc;  // a diagonal quadrant of a diagonal cell: tiles below its diagonal mirror those above
    const bool twodiag = BLK && wave >= 6;                      // two diagonal quadrants of a diagonal block
    const int nchA = (d_in + GU_K - 1) / GU_K, nch = nchA + (d_out + GU_K - 1) / GU_K;
    auto swz = [](int r) { return (r >> 1) & 7; };
    // rows >= T lie outside the example's byte range and read as zero
    const gram_i32x4 rA = gram_rsrc(A, (uint32_t)((size_t)T * d_in * 2));
    const gram_i32x4 rG = gram_rsrc(G, (uint32_t)((size_t)T * d_out * 2));
    // load j of this wave fills rows (LPP*wave + j)*8 .. +7 of a panel: lane l -> row + l/8, chunk position l%8
    const int prow[3] = {R, diag0 ? C2 : C1, C2};  // the rows (in units of 128) of the p-th panel of a stage
    int voffA[NPL][LPP], voffG[NPL][LPP];
    uint32_t ldsoff[NPL][LPP];
#pragma unroll
    for (int p = 0; p < NPL; ++p)
#pragma unroll
        for (int j = 0; j < LPP; ++j) {
            const int row0 = (LPP * wave + j) * 8, row = row0 + (lane >> 3);
            const int cg = (lane & 7) ^ swz(row);
            voffA[p][j] = ((prow[p] * GB + row) * d_in + cg * 8) * 2;
            voffG[p][j] = ((prow[p] * GB + row) * d_out + cg * 8) * 2;
            ldsoff[p][j] = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)&ring[p * PANEL + row0 * GU_K];
        }
    int ibuf = 0;
    auto issue = [&](int st) {
        // past the last chunk the loads still go out (the wait counts stay uniform): they read the last chunk again, into
        // a slot that nobody multiplies any more
        const int stc = st < nch ? st : nch - 1;
        const bool isA = stc < nchA;
        // (rotating the chunk order by the example index, which pays in gram_dma_kernel, costs 1-2 % here: the units of an
        // example need their panels at the same time, and any order serves that)
        const int soff = __builtin_amdgcn_readfirstlane((isA ? stc : stc - nchA) * GU_K * 2);
        const int left = isA ? d_in - stc * GU_K : d_out - (stc - nchA) * GU_K;  // columns of the row from this chunk on
        auto run = [&](const gram_i32x4& rs, const int (&voff)[NPL][LPP]) {  // (the choice of the source stays outside the run of loads)
#pragma unroll
            for (int p = 0; p < NPL; ++p)
#pragma unroll
                for (int j = 0; j < LPP; ++j) {
                    int v = voff[p][j];
                    if (RAGGED && ((lane & 7) ^ swz((LPP * wave + j) * 8 + (lane >> 3))) * 8 >= left) v = GRAM_OUTSIDE;  // past the row's end: zeros
                    gram_dma16<false>(rs, __builtin_amdgcn_readfirstlane(ldsoff[p][j] + ibuf * (STAGE * 2)), v, soff);
                }
        };
        if (isA) run(rA, voffA);
        else run(rG, voffG);
        ibuf = ibuf + 1 == GU_NS ? 0 : ibuf + 1;
    };
    // operand of the 16x16x32 MFMA: lane l holds k = 8*(l/16) .. +7 of row l%16 of its 16-row tile, i.e. 16-byte chunk
    // 4*kk + l/16 of that row; a wave's 64 x 64 quadrant is 4 x 4 such tiles.  The 64-row strip its row fragments come
    // from is (panel rslot, half rhalf), that of its column fragments (cslot, chalf).  In a diagonal block the four strips
    // of the two panels are numbered 0..3; wave w < 6 has the quadrant (strip SR[w], strip SC[w]) above the diagonal,
    // waves 6 and 7 the diagonal quadrants of the strips (0, 1) and (2, 3): their "row" fragments are strip SR and their
    // "column" fragments strip SC, each multiplied with itself.
    int rslot = 0, rhalf = wr, cslot = cell == 0 ? (diag0 ? 0 : 1) : NPL - 1, chalf = wc;
    if (BLK) {
        const int sr = (0x20211000u >> (4 * wave)) & 15, sc = (0x31332321u >> (4 * wave)) & 15;
        rslot = sr >> 1, rhalf = sr & 1, cslot = sc >> 1, chalf = sc & 1;
    }
    int fr[4], fc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int r = rhalf * 64 + u * 16 + (lane & 15), c = chalf * 64 + u * 16 + (lane & 15);
        fr[u] = r * GU_K + (((lane >> 4) ^ swz(r)) << 3) + rslot * PANEL;
        fc[u] = c * GU_K + (((lane >> 4) ^ swz(c)) << 3) + cslot * PANEL;
    }

#pragma unroll
    for (int st = 0; st < GU_NS - 1; ++st) issue(st);
    int cbuf = 0, s_next = GU_NS - 1;
    // A stage is two k steps of 32.  Fragment reads run half a stage ahead of the multiplies and across the barrier:
    // behind the barrier that publishes stage s the wave first asks for the fragments of (s, k step 0), then multiplies
    // those of (s-1, k step 1), which it already holds, asks for (s, k step 1) into the registers just freed, and
    // multiplies (s, k step 0).  All eight waves come out of the barrier together; without the step held over, the
    // matrix pipes would idle behind every barrier until the LDS has served the first reads of all of them.
    struct Frags {
        bf16x8_t a[4], b[4];
    };
    struct Acc {
        f32x4_t t[4][4], t2[4][4];  // t2: the second diagonal quadrant of MODE 3 (never touched otherwise)
    };
    auto read_frags = [&](Frags& f, int kk) {
        const uint16_t* st = ring + cbuf * STAGE;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int xr = fr[u] ^ ((4 * kk) << 3), xc = fc[u] ^ ((4 * kk) << 3);
            f.a[u] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(st + xr));
            f.b[u] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(st + xc));
        }
    };
    // MODE 0: a wave with nothing to multiply (it still fills its share of every stage), 1: a full quadrant, 2: a diagonal
    // quadrant (tiles below its diagonal mirror those above and are skipped), 3: two diagonal quadrants.  The mode is fixed
    // per wave, so the loops exist once per mode, each with accumulators of its own and the final sum inside: a choice
    // inside the loop body would merge the accumulators of its arms after every stage, which costs the register allocator
    // more than it has.
    auto all_stages = [&](auto mode_tag) -> float {
        constexpr int MODE = decltype(mode_tag)::value;
        Acc accA, accG;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) accA.t[a][b][r] = accG.t[a][b][r] = accA.t2[a][b][r] = accG.t2[a][b][r] = 0.f;
        auto multiply = [&](Acc& acc, const Frags& f) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) {
                    if (MODE == 3) {
                        if (mt <= nt) {
                            acc.t[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[mt], f.a[nt], acc.t[mt][nt], 0, 0, 0);
                            acc.t2[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.b[mt], f.b[nt], acc.t2[mt][nt], 0, 0, 0);
                        }
                    } else if (!(MODE == 2 && mt > nt)) {
                        acc.t[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[mt], f.b[nt], acc.t[mt][nt], 0, 0, 0);
                    }
                }
        };
        Frags X, Y;
        auto stage = [&](Acc& acc_prev, Acc& acc_cur, auto first_tag) {
            // my loads of this chunk have landed (later chunks may be in flight); after the barrier everyone's have,
            // and everyone is done reading the chunk before this one, whose slot the newest chunk overwrites
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((GU_NS - 2) * LPS) : "memory");
            __syncthreads();
            issue(s_next++);
            if (MODE != 0) {
                read_frags(X, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (!decltype(first_tag)::value) multiply(acc_prev, Y);
                __builtin_amdgcn_sched_barrier(0);
                read_frags(Y, 1);
                __builtin_amdgcn_sched_barrier(0);
                multiply(acc_cur, X);
                __builtin_amdgcn_sched_barrier(0);
            }
            cbuf = cbuf + 1 == GU_NS ? 0 : cbuf + 1;
        };
        stage(accA, accA, std::true_type{});
        for (int s = 1; s < nchA; ++s) stage(accA, accA, std::false_type{});
        stage(accA, accG, std::false_type{});  // the first chunk of G: the step held over still belongs to A
        for (int s = nchA + 1; s < nch; ++s) stage(accG, accG, std::false_type{});
        if (MODE != 0) multiply(accG, Y);
        float sum = 0.f;
        if (MODE != 0) {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // in a diagonal quadrant the tiles above the diagonal stand for their mirror images too; skipped tiles hold zeros
                        const float w = (MODE >= 2 && a < b) ? 2.f : 1.f;
                        sum += w * ((accA.t[a][b][r] + bias_term) * accG.t[a][b][r]);
                        if (MODE == 3) sum += w * ((accA.t2[a][b][r] + bias_term) * accG.t2[a][b][r]);
                    }
        }
        return sum;
    };
    float sum;
    if (!active) sum = all_stages(std::integral_constant<int, 0>{});
    else if (twodiag) sum = all_stages(std::integral_constant<int, 3>{});
    else if (diagw) sum = all_stages(std::integral_constant<int, 2>{});
    else sum = all_stages(std::integral_constant<int, 1>{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may still be writing LDS past this point
    // a quadrant off the diagonal of the plane counts twice (its mirror image is never formed): every quadrant of a cell off
    // the diagonal, the upper-right quadrant of a diagonal cell, and the six quadrants above the diagonal of a diagonal block
    float weight;
    if (BLK) weight = twodiag ? 1.f : 2.f;
    else weight = !active ? 0.f : ((cell == 0 && diag0) ? (wr == wc ? 1.f : 2.f) : 2.f);
    return sum * weight;
}

// out: partials [B][n_layers * n_units], stored; one unit of one layer: sqnorms, "+=".  Workgroup id g -> XCD g % 8; (layer, example) u = (g / 8 / n_units) * 8 + g % 8,
// unit = (g / 8) % n_units: the units of one example share an XCD, so that each panel comes from HBM once.
template <bool RAGGED>
__global__ __launch_bounds__(512, 1) void gram_units_kernel(GramBatch gb, GramUnits gu, int T, int d_in, int d_out, int has_bias,
                                                            float* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) uint16_t ring[GU_LDS];
    const int slot = blockIdx.x >> 3;
    const int u = (slot / gu.n_units) * 8 + (blockIdx.x & 7);
    const int unit = slot % gu.n_units;
    if (u >= gb.n_layers * gb.B) return;
    const int layer = u / gb.B, i = u - layer * gb.B;
    const uint32_t rc = gu.rc[unit];
    const int R = rc & 255, C1 = (rc >> 8) & 255, C2 = (rc >> 16) & 255;
    const bool blk = (rc >> 24) & 1;
    const uint16_t* A = gb.A[layer] + (size_t)i * T * d_in;
    const uint16_t* G = gb.G[layer] + (size_t)i * T * d_out;
    const float bias_term = has_bias ? 1.f : 0.f;
    const int npl = 1 + (C1 != R ? 1 : 0) + (C2 != 255 ? 1 : 0);
    float s;
    if (blk) s = gram_unit_ring<2, true, RAGGED>(A, G, T, d_in, d_out, R, C1, C2, bias_term, ring);
    else if (npl == 3) s = gram_unit_ring<3, false, RAGGED>(A, G, T, d_in, d_out, R, C1, C2, bias_term, ring);
    else if (npl == 2) s = gram_unit_ring<2, false, RAGGED>(A, G, T, d_in, d_out, R, C1, C2, bias_term, ring);
    else s = gram_unit_ring<1, false, RAGGED>(A, G, T, d_in, d_out, R, C1, C2, bias_term, ring);
    __syncthreads();  // the ring is free: its first floats serve the reduction
    const float tot = dp_block_sum<512>(s, reinterpret_cast<float*>(&ring[0]));
    if (threadIdx.x == 0) {
        if (gb.n_layers * gu.n_units == 1) out[i] += tot;
        else out[((size_t)i * gb.n_layers + layer) * gu.n_units + unit] = tot;
    }
}

// ------------------------------------------------------------------------------------------------
// T <= 32 (prediction slots: 20 rows per example; the output projection of a tied table has a 30K-wide input): one 32 x 32
// Gram tile per operand, where the 128-row kernel above would spend its time on empty rows.  Every wave works by itself: it fills
// stages of its own (64 columns of the 32 rows, 4 KiB, four 16-byte-per-lane loads straight into LDS, coalesced over 8 rows each)
// and multiplies them, wave w the chunks w, w + WAVES, ...; no barrier until the waves' accumulators meet in LDS.  (Stages that all
// waves filled and shared cost a barrier each, 127 ns a chunk of 64 columns whatever the batch: 63 us for 31,552 columns.)  NS - 1
// stages in flight per wave.  Workgroup g works on example g % B of layer g / B, as above.
// Bound: HBM, B*T*(d_in+d_out)*2 bytes read once.  T = 20, 1024 + 30,528 columns: B = 256 (323 MB) 69 -> 52 us, B = 8 63 -> 29;
// 1024 + 1024, B = 512: 28 us on the 128-row kernel, 11.5 with shared stages, 10.7.
// ------------------------------------------------------------------------------------------------
template <int WAVES, int NS, bool RAGGED>
__global__ __launch_bounds__(64 * WAVES, WAVES == 8 ? 1 : 2) void gram_small_dma_kernel(GramBatch gb, int T, int d_in, int d_out, int has_bias,
                                                                                        float* __restrict__ out) {
    constexpr int GDK = 64, ROWS = 32, STAGE = ROWS * GDK, RPI = 8, LOADS = ROWS / RPI;
    static_assert(NS * STAGE * 2 >= 2 * 16 * 64 * 4, "a wave's ring doubles as its part of the reduction buffer");
    __shared__ __attribute__((aligned(16))) uint16_t ring[WAVES][NS][STAGE];
    __shared__ float wred[WAVES];
    const int layer = __builtin_amdgcn_readfirstlane(blockIdx.x / gb.B), i = blockIdx.x - layer * gb.B;
    const uint16_t* __restrict__ A = gb.A[layer];
    const uint16_t* __restrict__ G = gb.G[layer];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nchA = (d_in + GDK - 1) / GDK, nch = nchA + (d_out + GDK - 1) / GDK;
    auto swz = [](int r) { return (r >> 1) & 7; };  // chunk position c of row r holds global chunk c ^ swz(r)
    // rows >= T lie outside the example's byte range and read as zero
    const gram_i32x4 rA = gram_rsrc(A + (size_t)i * T * d_in, (uint32_t)((size_t)T * d_in * 2));
    const gram_i32x4 rG = gram_rsrc(G + (size_t)i * T * d_out, (uint32_t)((size_t)T * d_out * 2));
    int cg[LOADS], voffA[LOADS], voffG[LOADS];
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
        const int lrow = q * RPI + lane / 8;
        cg[q] = (lane % 8) ^ swz(lrow);
        voffA[q] = (lrow * d_in + cg[q] * 8) * 2;
        voffG[q] = (lrow * d_out + cg[q] * 8) * 2;
    }
    const uint32_t ldsoff = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)&ring[wave][0][0];
    int ibuf = 0;  // buffer of the next stage to issue
    auto issue = [&](int st) {
        if (st >= nch) return;
        const bool isA = st < nchA;
        const int soff = __builtin_amdgcn_readfirstlane((isA ? st : st - nchA) * GDK * 2);
        const uint32_t dst = __builtin_amdgcn_readfirstlane(ldsoff + ibuf * (STAGE * 2));
        const int left = isA ? d_in - st * GDK : d_out - (st - nchA) * GDK;  // columns of the row from this chunk on
        if (isA) {
#pragma unroll
            for (int q = 0; q < LOADS; ++q)  // past the row's end: zeros
                gram_dma16<!RAGGED>(rA, dst + q * RPI * GDK * 2, RAGGED && cg[q] * 8 >= left ? GRAM_OUTSIDE : voffA[q], soff);
        } else {
#pragma unroll
            for (int q = 0; q < LOADS; ++q)
                gram_dma16<!RAGGED>(rG, dst + q * RPI * GDK * 2, RAGGED && cg[q] * 8 >= left ? GRAM_OUTSIDE : voffG[q], soff);
        }
        ibuf = ibuf + 1 == NS ? 0 : ibuf + 1;
    };
    const int r = lane & 31;
    int fpos[GDK / 16];
#pragma unroll
    for (int k = 0; k < GDK / 16; ++k) fpos[k] = r * GDK + (((2 * k + (lane >> 5)) ^ swz(r)) << 3);
    f32x16_t accA, accG;
#pragma unroll
    for (int q = 0; q < 16; ++q) accA[q] = accG[q] = 0.f;
#pragma unroll
    for (int st = 0; st < NS - 1; ++st) issue(wave + st * WAVES);
    int cbuf = 0, s = wave;
    auto phase = [&](int end, f32x16_t& acc) {
        for (; s < end; s += WAVES) {
            // stage s has landed (later ones may be in flight), and the fragments of the one before it are in registers: the newest
            // stage may overwrite its buffer
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            gram_wait<LOADS, NS - 2>((nch - 1 - s) / WAVES);
            issue(s + (NS - 1) * WAVES);
            const uint16_t* buf = ring[wave][cbuf];
            bf16x8_t x[GDK / 16];
#pragma unroll
            for (int k = 0; k < GDK / 16; ++k) x[k] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(buf + fpos[k]));
#pragma unroll
            for (int k = 0; k < GDK / 16; ++k) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[k], x[k], acc, 0, 0, 0);
            cbuf = cbuf + 1 == NS ? 0 : cbuf + 1;
        }
    };
    phase(nchA, accA);
    phase(nch, accG);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // nothing may still be writing LDS when the ring is reused
    // [wave][A|G][register][lane], each wave's part in its own ring
    float* part = reinterpret_cast<float*>(&ring[0][0][0]);
    constexpr int PITCH = NS * STAGE / 2;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        part[wave * PITCH + q * 64 + lane] = accA[q];
        part[wave * PITCH + (16 + q) * 64 + lane] = accG[q];
    }
    __syncthreads();
    const float bias_term = has_bias ? 1.f : 0.f;
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 16 / WAVES; ++q) {  // wave w finishes its share of the accumulator registers, the waves' partial tiles added in wave order
        const int reg = wave * (16 / WAVES) + q;
        float a = 0.f, g = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            a += part[w * PITCH + reg * 64 + lane];
            g += part[w * PITCH + (16 + reg) * 64 + lane];
        }
        sum += (a + bias_term) * g;
    }
    const float tot = dp_block_sum<64 * WAVES>(sum, wred);
    if (threadIdx.x == 0) {
        if (gb.n_layers == 1) out[i] += tot;
        else out[(size_t)i * gb.n_layers + layer] = tot;
    }
}

// ------------------------------------------------------------------------------------------------
// fp32 inputs, on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: products and sums in fp32).  The T x T plane of an
// example is cut into 32 x 32 cells of which the upper triangle is formed; a workgroup takes the cells cell0, cell0 + gridDim.y,
// ... of an example, its W waves (8, or as many as there are blocks) split the contraction in blocks of 32 columns (128 bytes of a row: lane = (row, half), a half
// is 64 contiguous bytes; the MFMA's k slots take the same columns of both operands, which is all a dot product needs) and the
// waves' accumulators meet in LDS.  Operands come straight from global memory, the next block in flight while one multiplies:
// every panel is read once per cell it is in, out of L2 (8 flop per byte, 20 TB/s at the full matrix rate).
// B = 16, T = 128, 768 x 768: 6,170 -> 16 us (one thread per pair of rows, scalar loads, before).  Waves without a
// block only add to the exchange: T = 17, B = 600, 64 x 64 12.7 us with 8 waves, 7.1 with 2; 30 x 30 16.1 | 6.4 with 1.
// ------------------------------------------------------------------------------------------------
template <bool VEC>
__device__ __forceinline__ void gram_f32_load(const float* __restrict__ row, bool valid, int d, int kb, float f[16]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = kb + 4 * j;
        if constexpr (VEC) {  // d % 4 == 0, 16-byte aligned rows: a group of four is inside the row or not at all
            const float4 w = valid && k < d ? *reinterpret_cast<const float4*>(row + k) : make_float4(0.f, 0.f, 0.f, 0.f);
            f[4 * j] = w.x; f[4 * j + 1] = w.y; f[4 * j + 2] = w.z; f[4 * j + 3] = w.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) f[4 * j + e] = valid && k + e < d ? row[k + e] : 0.f;
        }
    }
}

// This wave's share of the cell of X X^T with rows r (va: inside the example) and columns c.
template <bool VEC, int W>
__device__ __forceinline__ void gram_f32_cell(const float* __restrict__ r, bool va, const float* __restrict__ c, bool vb, bool diag, int d,
                                              int wave, int half, f32x16_t& acc) {
    constexpr int STEP = W * 32;
    float a0[16], b0[16], a1[16], b1[16];
    auto load = [&](int kb, float (&a)[16], float (&b)[16]) {
        gram_f32_load<VEC>(r, va, d, kb + 16 * half, a);
        if (!diag) gram_f32_load<VEC>(c, vb, d, kb + 16 * half, b);
    };
    auto mma = [&](const float (&a)[16], const float (&b)[16]) {
#pragma unroll
        for (int e = 0; e < 16; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], diag ? a[e] : b[e], acc, 0, 0, 0);
    };
    int kb = wave * 32;
    if (kb >= d) return;
    load(kb, a0, b0);
    while (true) {
        if (kb + STEP < d) load(kb + STEP, a1, b1);
        mma(a0, b0);
        if ((kb += STEP) >= d) break;
        if (kb + STEP < d) load(kb + STEP, a0, b0);
        mma(a1, b1);
        if ((kb += STEP) >= d) break;
    }
}

// out: gridDim.y == 1: sqnorms, "+="; otherwise partials [B][gridDim.y], stored.
template <bool VEC, int W>
__global__ __launch_bounds__(64 * W) void gram_f32_kernel(const float* __restrict__ A, const float* __restrict__ G, int T, int d_in, int d_out,
                                                          int has_bias, int nblk, float* __restrict__ out) {
    constexpr int H = W / 2;
    __shared__ float part[H ? H : 1][2][16][64];
    __shared__ float wred[W];
    const int i = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r32 = lane & 31, half = lane >> 5;
    const int ncells = nblk * (nblk + 1) / 2;
    const float bias_term = has_bias ? 1.f : 0.f;
    float s = 0.f;
    for (int cell = blockIdx.y; cell < ncells; cell += gridDim.y) {
        int tb = 0, sb = cell;
        while (sb >= nblk - tb) {  // row tb of the upper triangle holds nblk - tb cells
            sb -= nblk - tb;
            ++tb;
        }
        sb += tb;
        const int t = tb * 32 + r32, u = sb * 32 + r32;
        const bool va = t < T, vb = u < T, diag = tb == sb;
        const size_t rt = (size_t)i * T + (va ? t : 0), ru = (size_t)i * T + (vb ? u : 0);
        f32x16_t accA, accG;
#pragma unroll
        for (int r = 0; r < 16; ++r) accA[r] = accG[r] = 0.f;
        gram_f32_cell<VEC, W>(A + rt * d_in, va, A + ru * d_in, vb, diag, d_in, wave, half, accA);
        gram_f32_cell<VEC, W>(G + rt * d_out, va, G + ru * d_out, vb, diag, d_out, wave, half, accG);
        float p = 0.f;
        if constexpr (W == 1) {
#pragma unroll
            for (int r = 0; r < 16; ++r) p += (accA[r] + bias_term) * accG[r];
        } else {
            __syncthreads();  // the previous cell's readers are done
            // waves w + W / 2 hand their tiles to waves w, then the sums of these meet
            if (wave >= H) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    part[wave - H][0][r][lane] = accA[r];
                    part[wave - H][1][r][lane] = accG[r];
                }
            }
            __syncthreads();
            if (wave < H) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    part[wave][0][r][lane] += accA[r];
                    part[wave][1][r][lane] += accG[r];
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 16 / W; ++q) {  // wave w finishes its share of the accumulator registers, the parts added in a fixed order
                const int r = 16 / W * wave + q;
                float a = 0.f, g = 0.f;
#pragma unroll
                for (int h = 0; h < H; h += 2) {
                    a += part[h][0][r][lane] + (h + 1 < H ? part[h + 1 < H ? h + 1 : h][0][r][lane] : 0.f);
                    g += part[h][1][r][lane] + (h + 1 < H ? part[h + 1 < H ? h + 1 : h][1][r][lane] : 0.f);
                }
                p += (a + bias_term) * g;
            }
        }
        s += diag ? p : 2.f * p;  // rows past T are zeros in G G^T
    }
    const float tot = dp_block_sum<64 * W>(s, wred);
    if (threadIdx.x == 0) {
        if (gridDim.y == 1) out[i] += tot;
        else out[(size_t)i * gridDim.y + blockIdx.y] = tot;
    }
}

// fp32 materialise: A_i^T G_i in 64 x 64 blocks, a 32 x 32 tile per wave (operands as they lie in memory: lane = (column,
// k parity) reads 128 contiguous bytes of a row per half-wave), entries squared and summed.  A workgroup takes the blocks
// blockIdx.y, blockIdx.y + gridDim.y, ...; out as above.
__global__ __launch_bounds__(256) void materialise_f32_kernel(const float* __restrict__ A, const float* __restrict__ G,
                                                              int T, int d_in, int d_out, int tiles_m, int tiles_n, float* __restrict__ out) {
    __shared__ float wred[4];
    const int i = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5;
    const float* __restrict__ Ai = A + (size_t)i * T * d_in;
    const float* __restrict__ Gi = G + (size_t)i * T * d_out;
    float s = 0.f;
    for (int blk = blockIdx.y; blk < tiles_m * tiles_n; blk += gridDim.y) {
        const int p0 = blk / tiles_n * 64 + (wave >> 1) * 32, q0 = blk % tiles_n * 64 + (wave & 1) * 32;
        // columns past the widths repeat the last one and are left out of the sum
        const int p = p0 + (lane & 31), q = q0 + (lane & 31);
        const int pc = p < d_in ? p : d_in - 1, qc = q < d_out ? q : d_out - 1;
        f32x16_t acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        for (int t0 = 0; t0 < T && p0 < d_in && q0 < d_out; t0 += 16) {  // (a wave whose tile lies outside has nothing to do)
            float a[8], g[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int t = t0 + 2 * u + half, tc = t < T ? t : T - 1;
                a[u] = Ai[(size_t)tc * d_in + pc];
                g[u] = Gi[(size_t)tc * d_out + qc];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool ok = t0 + 2 * u + half < T;
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ok ? a[u] : 0.f, ok ? g[u] : 0.f, acc, 0, 0, 0);
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float v = p0 + 8 * (r >> 2) + 4 * half + (r & 3) < d_in && q < d_out ? acc[r] : 0.f;
            s += v * v;
        }
    }
    const float tot = dp_block_sum<256>(s, wred);
    if (threadIdx.x == 0) {
        if (gridDim.y == 1) out[i] += tot;
        else out[(size_t)i * gridDim.y + blockIdx.y] = tot;
    }
}

}  // namespace

// The LDS-ring kernels serve one block of up to 128 rows per example.
static bool gram_dma_ok(int T, int d_in, int d_out) {
    return T <= GB && d_in > 0 && d_out > 0 && (size_t)GB * (d_in > d_out ? d_in : d_out) * 2 < (1u << 31);
}

static dp_status gram_dma_launch(dp_ctx* ctx, const GramBatch& gb, int T, int d_in, int d_out, int has_bias, float* out,
                                 double bytes) {
    dp_prof_scope prof(ctx, DP_PROF_GRAM, bytes);
    const long wgs = (long)gb.n_layers * gb.B;
    const dim3 grid((unsigned)wgs);
    // 256-byte row segments (stages of 32 KiB) when the widths allow, else 128-byte segments (16 KiB)
    const bool wide = d_in % 128 == 0 && d_out % 128 == 0, ragged = d_in % 64 != 0 || d_out % 64 != 0;
    const bool few = wgs <= 256;  // a workgroup or less per CU: it may have all of the CU
    const long nch = (d_in + 63) / 64 + (long)gb.n_out * ((d_out + 63) / 64);  // chunks of 64 columns
    // Up to 64 rows one wave takes 0.8 us a chunk and four that share the k steps 0.2, but these spend 1 us on their exchange and hold
    // four wave slots and 64 KiB of LDS, 512 workgroups on the chip: one wave for three chunks and less, and up to twelve where
    // there are more workgroups than that (one | four, us: B = 200, T = 64, 64 x 64 8.1 | 9.2, 72 x 136 10.6 | 10.0; four layers of
    // 320 x 320 20.5 | 25.7; twelve layers, B = 500, T = 33: 64 x 64 30 | 70, 544 x 152 85 | 108, 200 x 1000 133 | 147).
    const bool one = T <= 64 && (nch <= 3 || (wgs > 512 && nch <= 12));
    // Up to 128 rows, a workgroup or less per CU: eight waves and all of the LDS pay from so many chunks on (four | eight: 72 x 136 9.2 |
    // 10.9, 128 x 256 9.9 | 10.4, 384 x 384 13.6 | 12.9, 448 x 704 17.6 | 18.3, 832 x 3136 46.2 | 41.5).
    const bool eight = few && nch > (wide ? 8 : 32);
    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, ctx->stream, gb, T, d_in, d_out, has_bias, out);
    };
    if (T <= 32 && gb.n_out == 1 && ragged && few) launch(gram_small_dma_kernel<8, 4, true>, 512);
    else if (T <= 32 && gb.n_out == 1 && ragged) launch(gram_small_dma_kernel<4, 4, true>, 256);
    else if (T <= 32 && gb.n_out == 1 && few) launch(gram_small_dma_kernel<8, 4, false>, 512);
    else if (T <= 32 && gb.n_out == 1) launch(gram_small_dma_kernel<4, 4, false>, 256);
    else if (one && ragged) launch(gram_dma_kernel<64, 64, 4, 1, 4, true>, 64);
    else if (one) launch(gram_dma_kernel<64, 64, 4, 1, 4, false>, 64);
    else if (T <= 64 && wide) launch(gram_dma_kernel<64, 128, 4, 4, 2, false>, 256);
    else if (T <= 64 && ragged) launch(gram_dma_kernel<64, 64, 8, 4, 2, true>, 256);
    else if (T <= 64) launch(gram_dma_kernel<64, 64, 8, 4, 2, false>, 256);
    else if (wide && eight) launch(gram_dma_kernel<128, 128, 4, 8, 1, false>, 512);
    else if (wide) launch(gram_dma_kernel<128, 128, 2, 4, 2, false>, 256);
    else if (ragged && eight) launch(gram_dma_kernel<128, 64, 9, 8, 1, true>, 512);
    else if (ragged) launch(gram_dma_kernel<128, 64, 4, 4, 2, true>, 256);
    else if (eight) launch(gram_dma_kernel<128, 64, 9, 8, 1, false>, 512);
    else launch(gram_dma_kernel<128, 64, 4, 4, 2, false>, 256);
    DP_LAUNCH_CHECK(ctx, "gram_dma");
    return DP_OK;
}

// The upper triangle of an nblk x nblk plane of 128 x 128 cells, cut into units.  Panels go two by two: the pair (2I, 2I+1)
// gives the diagonal block (2I, 2I), (2I, 2I+1), (2I+1, 2I+1); two pairs I < J give the four cells of rows 2I, 2I+1 and
// columns 2J, 2J+1, i.e. two row pairs.  With an odd nblk the last panel has no partner: its diagonal cell leads the row
// pair (last, last), (last, 0) - by symmetry (last, r) stands for the cell (r, last) - the cells (r, last) of the other
// rows pair up through the shared panel, (last, r1), (last, r2), and one of them stays alone.
static GramUnits gram_make_units(int nblk) {
    GramUnits gu;
    int n = 0;
    const int npair = nblk / 2, last = nblk - 1;
    for (int I = 0; I < npair; ++I) gu.rc[n++] = (uint32_t)(2 * I) | (uint32_t)(2 * I) << 8 | (uint32_t)(2 * I + 1) << 16 | 1u << 24;
    for (int I = 0; I < npair; ++I)
        for (int J = I + 1; J < npair; ++J)
            for (int r = 2 * I; r < 2 * I + 2; ++r) gu.rc[n++] = (uint32_t)r | (uint32_t)(2 * J) << 8 | (uint32_t)(2 * J + 1) << 16;
    if (nblk & 1) {
        gu.rc[n++] = (uint32_t)last | (uint32_t)last << 8 | (last > 0 ? 0u : 255u) << 16;
        int r = 1;
        for (; r + 1 < last; r += 2) gu.rc[n++] = (uint32_t)last | (uint32_t)r << 8 | (uint32_t)(r + 1) << 16;
        if (r < last) gu.rc[n++] = (uint32_t)r | (uint32_t)last << 8 | 255u << 16;
    }
    gu.n_units = n;
    return gu;
}

// The unit kernel: T up to GU_MAX_BLK cells of 128 rows.
static bool gram_units_ok(int T, int d_in, int d_out) {
    return T > GB && T <= GB * GU_MAX_BLK && d_in > 0 && d_out > 0 &&
           (size_t)((T + GB - 1) / GB * GB) * (d_in > d_out ? d_in : d_out) * 2 < (1u << 31);
}

dp_status dpk_gram_unit_plan(int T, uint32_t* units, int capacity, int* n_units) {
    if (T <= GB || T > GB * GU_MAX_BLK) return DP_ERR_SHAPE;
    const GramUnits gu = gram_make_units((T + GB - 1) / GB);
    if (gu.n_units > capacity) return DP_ERR_WORKSPACE;
    for (int k = 0; k < gu.n_units; ++k) units[k] = gu.rc[k];
    *n_units = gu.n_units;
    return DP_OK;
}

// nl <= GRAM_MAX_BATCH same-shaped layers: partials [B][nl * n_units] through the workspace, added in a fixed order.
static dp_status gram_units_launch(dp_ctx* ctx, const GramBatch& gb, int T, int d_in, int d_out, int has_bias,
                                   float* sqnorms) {
    const GramUnits gu = gram_make_units((T + GB - 1) / GB);
    const long units = (long)gb.n_layers * gb.B;
    const long nwg = (units + 7) / 8 * 8 * gu.n_units;
    if (nwg > 0x7FFFFFFFl) {
        DP_SET_ERR(ctx, "dp_sqnorms_dense: B * T^2 too large for one launch");
        return DP_ERR_SHAPE;
    }
    const bool direct = gb.n_layers * gu.n_units == 1;  // up to 256 rows: nothing to add behind
    dp_ws_alloc ws(ctx);
    float* part = direct ? sqnorms : ws.get<float>((size_t)units * gu.n_units);
    if (!part) {
        DP_SET_ERR(ctx, "workspace too small for %ld x %d Gram partials", units, gu.n_units);
        return DP_ERR_WORKSPACE;
    }
    {
        dp_prof_scope prof(ctx, DP_PROF_GRAM, 2.0 * (double)gb.B * T * ((double)d_in + d_out) * gb.n_layers);
        if (d_in % GU_K == 0 && d_out % GU_K == 0)
            hipLaunchKernelGGL((gram_units_kernel<false>), dim3((unsigned)nwg), dim3(512), 0, ctx->stream, gb, gu, T, d_in, d_out, has_bias, part);
        else
            hipLaunchKernelGGL((gram_units_kernel<true>), dim3((unsigned)nwg), dim3(512), 0, ctx->stream, gb, gu, T, d_in, d_out, has_bias, part);
    }
    DP_LAUNCH_CHECK(ctx, "gram_units");
    return direct ? DP_OK : dpk_finish_partials(ctx, part, gb.B, gu.n_units * gb.n_layers, sqnorms);
}

// One layer on the register-staged kernel: a workgroup per 128 x 128 block of the upper triangle.
static dp_status gram_block_sqnorms(dp_ctx* ctx, const void* A, const void* G, int B, int T, int d_in, int d_out, int has_bias, float* sqnorms) {
    const int nblk = (T + GB - 1) / GB;
    const long npairs = (long)nblk * (nblk + 1) / 2;
    const size_t lds = (size_t)2 * (nblk > 1 ? 2 : 1) * GB * GLD * sizeof(uint16_t);
    static bool lds_attr_set = false;  // off-diagonal blocks stage two panels per step: 72 KiB of dynamic LDS
    if (!lds_attr_set) {
        DP_HIP_CHECK(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(gram_bf16_kernel),
                                              hipFuncAttributeMaxDynamicSharedMemorySize,
                                              2 * 2 * GB * GLD * (int)sizeof(uint16_t)));
        lds_attr_set = true;
    }
    const double bytes = 2.0 * (double)B * T * ((double)d_in + d_out);
    if (npairs == 1) {
        dp_prof_scope prof(ctx, DP_PROF_GRAM, bytes);
        hipLaunchKernelGGL(gram_bf16_kernel, dim3(B), dim3(256), lds, ctx->stream, (const uint16_t*)A,
                           (const uint16_t*)G, B, T, d_in, d_out, has_bias, nblk, 1, sqnorms, 1);
        DP_LAUNCH_CHECK(ctx, "gram_bf16");
        return DP_OK;
    }
    const long groups = (B + 7) / 8;
    const long nwg = groups * 8 * npairs;
    if (nwg > 0x7FFFFFFFl) {
        DP_SET_ERR(ctx, "dp_sqnorms_dense: B * T^2 too large for one launch");
        return DP_ERR_SHAPE;
    }
    dp_ws_alloc ws(ctx);
    float* part = ws.get<float>((size_t)B * npairs);
    if (!part) {
        DP_SET_ERR(ctx, "workspace too small for %d x %ld Gram partials", B, npairs);
        return DP_ERR_WORKSPACE;
    }
    {
        dp_prof_scope prof(ctx, DP_PROF_GRAM, bytes);
        hipLaunchKernelGGL(gram_bf16_kernel, dim3((unsigned)nwg), dim3(256), lds, ctx->stream, (const uint16_t*)A,
                           (const uint16_t*)G, B, T, d_in, d_out, has_bias, nblk, (int)npairs, part, 0);
    }
    DP_LAUNCH_CHECK(ctx, "gram_bf16");
    return dpk_finish_partials(ctx, part, B, (int)npairs, sqnorms);
}

// Whether that is the better one for a single layer of more than 128 rows: widths that end inside a chunk, and so few units that the
// chip is three quarters idle (B = 24, T = 195, 544 x 152: 18.0 | 19.2 us; B = 4, T = 300, 72 x 136: 12.0 | 13.5).
static bool gram_block_better(const dp_ctx* ctx, int B, int T, int d_in, int d_out) {
    const long nblk = (T + GB - 1) / GB, npairs = nblk * (nblk + 1) / 2;
    return (d_in % GU_K || d_out % GU_K) && (long)B * gram_make_units((int)nblk).n_units <= 96 && (size_t)B * npairs * sizeof(float) <= ctx->ws_bytes;
}

// Layers of one launch: as many as it may hold and as have room for their partial norms; a single one adds to sqnorms itself.
static int gram_layers_per_launch(const dp_ctx* ctx, int n, int B) {
    int nl = n < GRAM_MAX_BATCH ? n : GRAM_MAX_BATCH;
    while (nl > 1 && ((size_t)nl * B * sizeof(float) > ctx->ws_bytes || (long)nl * B > 0x7FFFFFFFl)) nl = (nl + 1) / 2;
    return nl;
}

dp_status dpk_gram_sqnorms_batched(dp_ctx* ctx, int n_layers, const void* const* A, const void* const* G, dp_dtype dt,
                                   int B, int T, int d_in, int d_out, int has_bias, float* sqnorms) {
    if (dt == DP_BF16 && n_layers == 1 && gram_units_ok(T, d_in, d_out) && gram_block_better(ctx, B, T, d_in, d_out))
        return gram_block_sqnorms(ctx, A[0], G[0], B, T, d_in, d_out, has_bias, sqnorms);
    if (dt == DP_BF16 && gram_units_ok(T, d_in, d_out)) {
        // enough layers per launch for a few rounds of workgroups, and partials that fit the workspace
        const int nblk = (T + GB - 1) / GB;
        const long npairs = (long)nblk * (nblk + 1) / 2;  // (an upper bound of the units per example)
        int per = GRAM_MAX_BATCH;
        while (per > 1 && ((size_t)per * B * npairs * sizeof(float) > ctx->ws_bytes / 2 ||
                           (long)per * B * npairs > (1l << 22)))
            per /= 2;
        for (int l0 = 0; l0 < n_layers; l0 += per) {
            const int nl = n_layers - l0 < per ? n_layers - l0 : per;
            GramBatch gb;
            for (int l = 0; l < GRAM_MAX_BATCH; ++l) {
                gb.A[l] = (const uint16_t*)A[l0 + (l < nl ? l : 0)];
                gb.G[l] = (const uint16_t*)G[l0 + (l < nl ? l : 0)];
                gb.G2[l] = gb.G3[l] = gb.G[l];
            }
            gb.n_layers = nl;
            gb.n_out = 1;
            gb.B = B;
            dp_status st = gram_units_launch(ctx, gb, T, d_in, d_out, has_bias, sqnorms);
            if (st != DP_OK) return st;
        }
        return DP_OK;
    }
    if (dt != DP_BF16 || !gram_dma_ok(T, d_in, d_out)) {
        for (int l = 0; l < n_layers; ++l) {
            dp_status st = dpk_gram_sqnorms(ctx, A[l], G[l], dt, B, T, d_in, d_out, has_bias, sqnorms);
            if (st != DP_OK) return st;
        }
        return DP_OK;
    }
    for (int l0 = 0; l0 < n_layers;) {
        const int nl = gram_layers_per_launch(ctx, n_layers - l0, B);
        dp_ws_alloc ws(ctx);
        float* part = nl > 1 ? ws.get<float>((size_t)B * nl) : nullptr;
        GramBatch gb;
        for (int l = 0; l < GRAM_MAX_BATCH; ++l) {
            gb.A[l] = (const uint16_t*)A[l0 + (l < nl ? l : 0)];
            gb.G[l] = (const uint16_t*)G[l0 + (l < nl ? l : 0)];
            gb.G2[l] = gb.G3[l] = gb.G[l];
        }
        gb.n_layers = nl;
        gb.n_out = 1;
        gb.B = B;
        dp_status st = gram_dma_launch(ctx, gb, T, d_in, d_out, has_bias, part ? part : sqnorms, 2.0 * (double)B * T * ((double)d_in + d_out) * nl);
        if (st == DP_OK && part) st = dpk_finish_partials(ctx, part, B, nl, sqnorms);   // (in an order fixed by nl)
        if (st != DP_OK) return st;
        l0 += nl;
    }
    return DP_OK;
}

// n_groups groups of n_out (2 or 3) same-shaped layers, the layers of a group sharing their input A[g]; G is
// group-major: G[g * n_out + j].
dp_status dpk_gram_sqnorms_shared(dp_ctx* ctx, int n_groups, const void* const* A, int n_out, const void* const* G,
                                  dp_dtype dt, int B, int T, int d_in, int d_out, int has_bias, float* sqnorms) {
    if (dt == DP_BF16 && gram_units_ok(T, d_in, d_out)) {  // (the units form every layer's input again, many layers a launch)
        const void *a[GRAM_MAX_BATCH], *go[GRAM_MAX_BATCH];
        int n = 0;
        for (int g = 0; g < n_groups; ++g)
            for (int j = 0; j < n_out; ++j) {
                a[n] = A[g];
                go[n++] = G[(size_t)g * n_out + j];
                if (n < GRAM_MAX_BATCH && !(g + 1 == n_groups && j + 1 == n_out)) continue;
                const dp_status st = dpk_gram_sqnorms_batched(ctx, n, a, go, dt, B, T, d_in, d_out, has_bias, sqnorms);
                if (st != DP_OK) return st;
                n = 0;
            }
        return DP_OK;
    }
    if (dt != DP_BF16 || n_out < 2 || n_out > 3 || !gram_dma_ok(T, d_in, d_out)) {
        for (int g = 0; g < n_groups; ++g)
            for (int j = 0; j < n_out; ++j) {
                dp_status st = dpk_gram_sqnorms(ctx, A[g], G[(size_t)g * n_out + j], dt, B, T, d_in, d_out, has_bias, sqnorms);
                if (st != DP_OK) return st;
            }
        return DP_OK;
    }
    for (int g0 = 0; g0 < n_groups;) {
        const int ng = gram_layers_per_launch(ctx, n_groups - g0, B);
        dp_ws_alloc ws(ctx);
        float* part = ng > 1 ? ws.get<float>((size_t)B * ng) : nullptr;
        GramBatch gb;
        for (int l = 0; l < GRAM_MAX_BATCH; ++l) {
            const size_t g = (size_t)g0 + (l < ng ? l : 0);
            gb.A[l] = (const uint16_t*)A[g];
            gb.G[l] = (const uint16_t*)G[g * n_out];
            gb.G2[l] = (const uint16_t*)G[g * n_out + 1];
            gb.G3[l] = (const uint16_t*)G[g * n_out + (n_out > 2 ? 2 : 1)];
        }
        gb.n_layers = ng;
        gb.n_out = n_out;
        gb.B = B;
        const double bytes = 2.0 * (double)B * T * ((double)d_in + (double)n_out * d_out) * ng;
        dp_status st = gram_dma_launch(ctx, gb, T, d_in, d_out, has_bias, part ? part : sqnorms, bytes);
        if (st == DP_OK && part) st = dpk_finish_partials(ctx, part, B, ng, sqnorms);
        if (st != DP_OK) return st;
        g0 += ng;
    }
    return DP_OK;
}

// Workgroups per example of the fp32 norm kernels: one per piece (cell or block) up to about 4,096 in all, as far as their
// partial norms fit the workspace; one workgroup per example walks all its pieces and needs none of it.  So it does where
// the examples, many of them above all, have a few short pieces each (`steps`: blocks of the contraction of all of them), which take less than the launch that
// adds the partial norms.
static float* f32_partials(dp_ctx* ctx, int B, long pieces, long steps, float* sqnorms, int* per) {
    long g = pieces < 4096 ? pieces : 4096;
    if (steps <= (B >= 128 ? 8 : 3)) g = 1;
    if (g > 1 && (long)B * g > 4096) g = 4096 / B < 1 ? 1 : 4096 / B;
    float* part = nullptr;
    if (g > 1) {
        dp_ws_alloc ws(ctx);
        part = ws.get<float>((size_t)B * g);
    }
    *per = part ? (int)g : 1;
    return part ? part : sqnorms;
}

dp_status dpk_gram_sqnorms(dp_ctx* ctx, const void* A, const void* G, dp_dtype dt, int B, int T, int d_in, int d_out,
                           int has_bias, float* sqnorms) {
    if (dt == DP_F32) {
        const int nblk = (T + 31) / 32;
        int per;
        const int blocks = ((d_in > d_out ? d_in : d_out) + 31) / 32;  // of the contraction: no more waves than these
        const long cells = (long)nblk * (nblk + 1) / 2;
        float* part = f32_partials(ctx, B, cells, cells * ((blocks + 7) / 8) * 2, sqnorms, &per);
        const bool vec = d_in % 4 == 0 && d_out % 4 == 0 && (((uintptr_t)A | (uintptr_t)G) & 15) == 0;
        auto launch = [&](auto kernel, int waves) {
            hipLaunchKernelGGL(kernel, dim3(B, per), dim3(64 * waves), 0, ctx->stream, (const float*)A, (const float*)G, T, d_in, d_out, has_bias,
                               nblk, part);
        };
        const long share = 2048 / ((long)B * per), most = blocks < share ? blocks : share;  // ... nor than the chip runs at once
        auto pick = [&](auto vec_tag) {
            constexpr bool VEC = decltype(vec_tag)::value;
            if (most <= 1) launch(gram_f32_kernel<VEC, 1>, 1);
            else if (most <= 2) launch(gram_f32_kernel<VEC, 2>, 2);
            else if (most <= 4) launch(gram_f32_kernel<VEC, 4>, 4);
            else launch(gram_f32_kernel<VEC, 8>, 8);
        };
        if (vec) pick(std::true_type{});
        else pick(std::false_type{});
        DP_LAUNCH_CHECK(ctx, "gram_f32");
        return per > 1 ? dpk_finish_partials(ctx, part, B, per, sqnorms) : DP_OK;
    }
    if (gram_dma_ok(T, d_in, d_out) || gram_units_ok(T, d_in, d_out))
        return dpk_gram_sqnorms_batched(ctx, 1, &A, &G, dt, B, T, d_in, d_out, has_bias, sqnorms);
    return gram_block_sqnorms(ctx, A, G, B, T, d_in, d_out, has_bias, sqnorms);
}

dp_status dpk_materialise_f32(dp_ctx* ctx, const float* A, const float* G, int B, int T, int d_in, int d_out,
                              float* sqnorms) {
    const int tiles_m = (d_in + 63) / 64, tiles_n = (d_out + 63) / 64;
    int per;
    float* part = f32_partials(ctx, B, (long)tiles_m * tiles_n, (long)tiles_m * tiles_n * ((T + 15) / 16), sqnorms, &per);
    hipLaunchKernelGGL(materialise_f32_kernel, dim3(B, per), dim3(256), 0, ctx->stream, A, G, T, d_in, d_out, tiles_m, tiles_n, part);
    DP_LAUNCH_CHECK(ctx, "materialise_f32");
    return per > 1 ? dpk_finish_partials(ctx, part, B, per, sqnorms) : DP_OK;
}
