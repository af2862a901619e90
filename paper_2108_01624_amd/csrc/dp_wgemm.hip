// Clip-weighted dense gradient sum  S_W += sum_i c_i A_i^T G_i = A_flat^T diag(c (x) 1_T) G_flat
// (the sum over the batch of clip(grad, C) in the g_t line of Algorithm 1, for a dense layer whose
// per-example gradient is the outer-product form of Section 4.3), and the tile-by-tile materialisation
// of one example's A_i^T G_i for the squared-norm path that sums squares of the entries.
//
// Both are "TN" contractions: the contraction index (token row k) is the SLOW index of both operands in
// memory, while the bf16 MFMA wants each lane to hold 8 consecutive k for one output row/column.
// Tiles are staged in LDS as they lie in memory ([k][column], 16-byte chunks) and fragments are fetched
// with the gfx950 transposing LDS read (ds_read_b64_tr_b16): inside a group of 16 lanes, lane i supplies
// the address of 4 adjacent columns of row k0 + i/4 and receives column i of rows k0..k0+3, so two reads
// give a lane its 8 consecutive k.  No permute instructions, natural output layout.
//
// LDS bank conflicts: the four rows a 16-lane group touches are one row pitch (512 B or 256 B) apart, i.e.
// in the same banks.  The 16-byte chunk index is therefore XOR-ed with bits of the row when a chunk is stored,
// which spreads the four rows of a group, and the two groups of a half-wave, over 256 distinct bytes.
//
// Roofline: MFMA.  2*B*T*d_in*d_out flops per layer against (d_in + d_out)*B*T*2 bytes read once.

#include <type_traits>

#include "dp_common.h"

namespace {

constexpr int BK = 32;  // token rows per staged tile

enum { EPI_STORE = 0, EPI_ADD = 1, EPI_SQNORM = 2 };

struct WgemmArgs {
    const float* sqnorms;  // [B] squared norms; c_i = min(1, C / sqrt(sqnorms[i])) (unused without scaling)
    float C;
    float* bias_part;    // column sums of the scaled G rows, one row of d_out per (unit, tile row, wave row), or nullptr
    int T, d_in, d_out;
    long K;              // total rows
    long rows_per_split; // whole examples; without factors (flat) a multiple of BK, or T for the materialisation
    int tiles_m, tiles_n, nsplit;
    float* out;          // EPI_SQNORM: [nsplit][layers][ntiles] partial norms (the sums' outputs are per layer, below)
    int xcd_map;         // 1: whole units dealt to the 8 XCDs; 2: each XCD owns one rect_m x rect_n-th sub-rectangle of a unit's
                         // tile grid; 3: the (unit, tile) sequence cut into 8 equal runs
    int rect_m, rect_n;  // mode 2: the tile grid is cut into rect_m x rect_n rectangles, 8 / units per unit;
                         // modes 1 and 3: a unit's tiles are walked in rectangles of this size
    int* err;            // device error word: DP_ERRBIT_NORM is set when a clip factor is NaN (non-finite squared norm)
    int bias_direct;     // sums: no bias partials, the kernel adds to sum_b (one row split); norms: count the bias gradient
    int flat;            // no clip factors (G holds c * g already, or the norms are wanted), a unit is one run of rows
};

// Several layers of one shape in one launch: the unit of work distribution is the pair (layer, row split); `base`
// describes the common shape.
constexpr int MAX_BATCH = 64;
struct LayerPtrs {
    const uint16_t* A;
    const uint16_t* G;
    float* out;      // EPI_ADD: the layer's sum_W; EPI_STORE: the layer's first partial [nsplit][d_in][d_out]
    float* sum_b;    // the layer's bias sum buffer or nullptr
};
struct WgemmBatchArgs {
    WgemmArgs base;
    int n_layers;
    LayerPtrs L[MAX_BATCH];
};

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// 8 consecutive k (rows) of one column, as an MFMA operand: two transposing reads of 4 rows each.
__device__ __forceinline__ bf16x8_t read_frag(const uint16_t* lds_lane_ptr, int row_pitch_elems) {
    typedef s16x4_t __attribute__((address_space(3))) * lptr;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(lds_lane_ptr));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(lds_lane_ptr + 4 * row_pitch_elems));
    const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
}

// ------------------------------------------------------------------------------------------------
// The clip-weighted sum in bf16: block tiles of 256 or 128 by 256 or 128, 8 waves (2 x 4; at 256 x 256 a wave tile of
// 128 x 64, accumulators in VGPRs, two waves per SIMD).
//
//  * Both operand tiles go from global memory straight into LDS (buffer_load ... lds, 16 bytes per lane, a wave
//    fills two tile rows per instruction): no staging registers, no LDS store instructions, nothing for the
//    VALU to do per element.  The loads are issued through inline assembly because the compiler would otherwise
//    wait for ALL outstanding LDS-filling loads before every LDS read; here the wave waits (vmcnt) only for the
//    stage it is about to publish and keeps the later stages in flight.  Ring of five 32 KiB stages at 256 x 256: all of the CU's LDS.
//  * The clip factor is not applied to the operands at all.  All rows of a stage belong to one example, so the
//    accumulators carry sum_{j<=i} (c_j / c_i) A_j^T G_j: when the stage's example changes they are multiplied
//    by c_prev / c_next (128 + 32 VALU multiplies per wave per example, spread over the two half-iterations
//    around the boundary), and by the last c at the end.  The bf16 products are exact in fp32, so this path is
//    more accurate than rounding c*g to bf16.  Row splits are whole examples.  The last stage of an example whose T is no
//    multiple of 32 is filled up with zero rows by the range check of its buffer resource: up to 31 rows of work for nothing,
//    still 2.2 times the rate of scaling G while it is staged (4 layers of 768 x 3072, B = 96, T = 100: 615 -> 255 us).
//    Where that waste is large (T = 20: 12 rows of 32) scale_rows_kernel writes bf16(c*g) once and the rows are contracted as
//    one run (1024 x 1024, B = 512, T = 20: 62 -> 50 us; a 30,528 x 1,024 table: 659 -> 308); the host prices both forms.
//  * Bias gradient: column sums of G are one more MFMA with an all-ones A fragment.  Every wave takes that duty
//    for one stage in 2*tiles_m (tile row pm, wave row wr: stages s with s % (2*tiles_m) == 2*pm + wr), so the
//    extra work is spread evenly; the partial sums of (split, pm, wr) are added in a fixed order afterwards.
// ------------------------------------------------------------------------------------------------
typedef int i32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void dma_load16(i32x4_t rsrc, uint32_t lds_byte_addr, int voff, int soff) {
    // LDS destination of lane l: M0 + 16*l.  voff: per-lane byte offset; soff: wave-uniform byte offset.
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_byte_addr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
}

__device__ __forceinline__ i32x4_t make_rsrc(const void* base, uint32_t bytes) {
    const uint64_t p = (uint64_t)base;
    i32x4_t r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));  // stride 0
    r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    r[3] = 0x00020000;
    return r;
}

// A resource for the buffer builtins whose address and size are the same in every lane but were computed in vector registers
// (after an integer division, say): made scalar by hand, or every access becomes a loop over its distinct values.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const void* base, uint32_t bytes) {
    const uint64_t p = (uint64_t)base;
    const uint64_t s = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32)) << 32 |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    return __builtin_amdgcn_make_buffer_rsrc((void*)s, 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}

// The kernel uses the 16x16x32 MFMA.  Per flop it moves as many fragment bytes through LDS as 32x32x16 would, but the
// matrix pipe draws less power: a loop of nothing but MFMAs on random operands sustains 2.1 PFLOP/s with this shape
// against 1.4 with 32x32x16 (the chip holds 2.07 against 1.7 GHz; on zeros 2.47 against 1.63 PFLOP/s), and this kernel
// lives under the power limit.  Wave tile 128 x 64 = 8 x 4 tiles of 16 x 16; a stage (32 rows) is one MFMA step per tile,
// worked on in two halves of 16 MFMAs (tile rows 0..3, then 4..7) so that the fragments of the next half arrive while
// this one multiplies: 12 fragments in flight in 48 registers.  Rows r and r + 8 of a stage are read by lanes of the
// same pass, so the chunk swizzle also takes bit 3 of the row.
__device__ __forceinline__ int swz16(int row) { return ((row & 3) << 2) | (((row >> 3) & 1) << 1); }

// Stages of (BM + BN) columns x 32 rows in the ring: 256 x 256 takes 5 of 32 KiB, the whole 160 KiB of LDS, the mixed tiles 6 of
// 24 KiB, and 128 x 128 5 of 16 KiB, which leaves room for a second workgroup on the CU.
constexpr int dma_stages(int bm, int bn) { return bm + bn >= 512 ? 5 : (bm + bn >= 384 ? 6 : 5); }

// MI x NI tiles of 16 x 16 per wave, 2 x 4 waves: block tile 32 MI x 64 NI (256 or 128 wide either way).
// ONE_STAGE: examples of one stage (T <= 32) with factors; every stage then rescales.
template <int MI, int NI, int EPI, bool ONE_STAGE>
__global__ __launch_bounds__(512, MI * NI <= 8 ? 4 : 2) void wgemm_dma16_kernel(WgemmBatchArgs b) {
    constexpr int MH = MI / 2, WVN = 4;  // a stage is worked on in two halves of MH tile rows
    constexpr int WM = 16 * MI, WN = 16 * NI, BM = 2 * WM, BN = 4 * WN;
    constexpr int NS = dma_stages(BM, BN);
    constexpr int LA = BM / 128, LG = BN / 128, LPS = LA + LG;  // LDS-filling loads per wave per stage
    constexpr int CA = BM / 8, CG = BN / 8;                     // 16-byte chunks per tile row
    __shared__ __attribute__((aligned(16))) uint16_t As[NS][BK * BM];
    __shared__ __attribute__((aligned(16))) uint16_t Gs[NS][BK * BN];
    const WgemmArgs& a = b.base;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: everything derived from it stays in SGPRs
    const int wr = wave / WVN, wc = wave % WVN;
    const int ntiles = a.tiles_m * a.tiles_n;
    const int nunits = b.n_layers * a.nsplit;  // unit = layer * nsplit + split
    // Workgroup ids are dealt to the 8 XCDs round-robin: an XCD gets whole units (mode 1) or one rectangle of
    // one unit's tile grid (mode 2), so that its L2 sees each operand row and column about once.
    int tile, unit;
    if (a.xcd_map == 1) {
        // nunits is a multiple of 8: XCD x works through the CONSECUTIVE units x * nunits/8 ... (x+1) * nunits/8 - 1.  With
        // 16-tile units two of them run on an XCD at a time, so neighbouring layers that read the same input (the query
        // and key projections of a block, when the caller hands them one tensor) fetch its panels from HBM once.
        const int g = blockIdx.x, slot = g >> 3;
        unit = (g & 7) * (nunits >> 3) + slot / ntiles;
        if (unit >= nunits) return;
        // An XCD runs about 32 workgroups at a time: walk the unit's tile grid in rect_m x rect_n rectangles so
        // that those 32 share as many operand columns as possible (rect 1 x 1 = plain row-major order).
        const int t = slot % ntiles, per = a.rect_m * a.rect_n, rect = t / per, w = t % per;
        const int rpr = a.tiles_n / a.rect_n;
        tile = ((rect / rpr) * a.rect_m + w / a.rect_n) * a.tiles_n + (rect % rpr) * a.rect_n + w % a.rect_n;
    } else if (a.xcd_map == 2) {
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        const int nrect = a.rect_m * a.rect_n;
        const int rect = xcd % nrect;
        const int tm = a.tiles_m / a.rect_m, tn = a.tiles_n / a.rect_n;
        unit = xcd / nrect;
        tile = ((rect / a.rect_n) * tm + slot / tn) * a.tiles_n + (rect % a.rect_n) * tn + slot % tn;
    } else {
        // mode 3: the (unit, tile) pairs in unit-major order, cut into 8 equal runs, one per XCD: balanced for any
        // unit and tile count; at most 7 units have their tiles on two XCDs
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        const int total = nunits * ntiles, per_xcd = (total + 7) >> 3;
        const int w = xcd * per_xcd + slot;
        if (slot >= per_xcd || w >= total) return;
        unit = w / ntiles;
        const int t = w - unit * ntiles, per = a.rect_m * a.rect_n, rect = t / per, r = t % per;
        const int rpr = a.tiles_n / a.rect_n;
        tile = ((rect / rpr) * a.rect_m + r / a.rect_n) * a.tiles_n + (rect % rpr) * a.rect_n + r % a.rect_n;
    }
    const int layer = unit / a.nsplit, split = unit % a.nsplit;
    const int pm = tile / a.tiles_n, qn = tile % a.tiles_n;
    const int p0 = pm * BM, q0 = qn * BN;
    const long k_lo = (long)split * a.rows_per_split;
    const long k_hi = k_lo + a.rows_per_split < a.K ? k_lo + a.rows_per_split : a.K;
    const int nrows = __builtin_amdgcn_readfirstlane(k_hi > k_lo ? (int)(k_hi - k_lo) : 0);
    // The unit's rows are n_ex examples of T rows, each cut into spe stages of 32 rows, the last one of T_last (the rows
    // that follow belong to the next example: the stage's buffer resource ends at the example's last row, so they arrive
    // as zeros and multiply nothing).  Without factors (a.flat) the unit is one run of nrows rows.
    const int T = a.flat ? nrows : a.T;
    const int spe = (T + BK - 1) / BK, T_last = T - (spe - 1) * BK;
    const int n_ex = a.flat ? (nrows > 0 ? 1 : 0) : __builtin_amdgcn_readfirstlane(nrows / a.T);

    // Resources over the rows of the stage that is issued next; advanced from stage to stage.  (The stage's start is part of
    // the base: a scalar offset would have to be trusted to the resource's range check.)
    i32x4_t rA = make_rsrc(b.L[layer].A + (size_t)k_lo * a.d_in, 0);
    i32x4_t rG = make_rsrc(b.L[layer].G + (size_t)k_lo * a.d_out, 0);
    int q_issue = 0, left = n_ex * spe;  // stage of its example, and stages still to issue
    int rows_issue = 0;
    auto stage_open = [&]() {   // past the last stage: no rows, the loads bring zeros and touch no memory
        rows_issue = left > 0 ? (q_issue == spe - 1 ? T_last : BK) : 0;
        rA[2] = __builtin_amdgcn_readfirstlane(rows_issue * a.d_in * 2);
        rG[2] = __builtin_amdgcn_readfirstlane(rows_issue * a.d_out * 2);
    };
    auto advance = [](i32x4_t& r) {
        const uint64_t p = ((uint64_t)(uint32_t)r[1] << 32 | (uint32_t)r[0]) + (uint32_t)r[2];
        r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
        r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
    };
    auto stage_close = [&]() {
        advance(rA);
        advance(rG);
        q_issue = q_issue + 1 == spe ? 0 : q_issue + 1;
        --left;
    };

    // Load j of this wave fills tile rows (LA * wave + j) * 64 / CA .. of A (G likewise): lane l -> row + l / CA, LDS chunk
    // l % CA, which holds global chunk (l % CA) ^ swz16(row).  Columns past the layer width read neighbouring (valid or
    // zero) data and only feed output columns that are never stored.
    int voffA[LA], voffG[LG];
    uint32_t ldsA[LA], ldsG[LG];
#pragma unroll
    for (int j = 0; j < LA; ++j) {
        const int row0 = (LA * wave + j) * (64 / CA), row = row0 + lane / CA;
        voffA[j] = (row * a.d_in + p0 + ((lane % CA) ^ swz16(row)) * 8) * 2;
        ldsA[j] = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)&As[0][row0 * BM];
    }
#pragma unroll
    for (int j = 0; j < LG; ++j) {
        const int row0 = (LG * wave + j) * (64 / CG), row = row0 + lane / CG;
        voffG[j] = (row * a.d_out + q0 + ((lane % CG) ^ swz16(row)) * 8) * 2;
        ldsG[j] = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)&Gs[0][row0 * BN];
    }
    // The LPS loads of a stage in the order A0, G0, A1, G1 (what exists of it).
    auto fill = [&](int k, int slot) {
        constexpr int MIN = LA < LG ? LA : LG;
        const bool isA = k < 2 * MIN ? k % 2 == 0 : LA > LG;
        const int j = k < 2 * MIN ? k / 2 : k - MIN;
        if (isA) dma_load16(rA, __builtin_amdgcn_readfirstlane(ldsA[j < LA ? j : 0] + slot * (BK * BM * 2)), voffA[j < LA ? j : 0], 0);
        else dma_load16(rG, __builtin_amdgcn_readfirstlane(ldsG[j < LG ? j : 0] + slot * (BK * BN * 2)), voffG[j < LG ? j : 0], 0);
    };
    // Operand of the 16x16x32 MFMA: lane l holds the 8 consecutive k = 8*(l/16) .. +7 of column l%16 of its tile.  The
    // transposing read hands lane i of a 16-lane group column i of the 4 rows x 16 columns that the group addresses
    // (lane i: row i/4, columns 4*(i%4) .. +3): two reads, rows frow and frow + 4 (same swizzle: bits 0, 1, 3 agree).
    const int frow = 8 * (lane >> 4) + ((lane & 15) >> 2);
    const int fsw = swz16(frow);
    int foffA[MI], foffG[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int col = wr * WM + 16 * i + 4 * (lane & 3);
        foffA[i] = frow * BM + (((col >> 3) ^ fsw) << 3) + (col & 7);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int col = wc * WN + 16 * i + 4 * (lane & 3);
        foffG[i] = frow * BN + (((col >> 3) ^ fsw) << 3) + (col & 7);
    }
    auto load_fa = [&](int buf, int half, bf16x8_t* fa) {
#pragma unroll
        for (int i = 0; i < MH; ++i) fa[i] = read_frag(&As[buf][foffA[half * MH + i]], BM);
    };

    f32x4_t acc[MI][NI], bacc[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
#pragma unroll
        for (int r = 0; r < 4; ++r) bacc[j][r] = 0.f;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
    }
    const bool want_bias = EPI == EPI_SQNORM ? a.bias_direct != 0 : b.L[layer].sum_b != nullptr;
    // bias_direct (norms; sums with one row split and few stages): the first wave row of tile row 0 takes every stage
    const int duty_mod = a.bias_direct ? 1 : 2 * a.tiles_m, duty = 2 * pm + wr;
    const uint32_t one2 = 0x3F803F80u;  // two bf16 ones
    const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, u32x4_t{one2, one2, one2, one2});
    auto mma_bias = [&](const bf16x8_t* fg) {
#pragma unroll
        for (int j = 0; j < NI; ++j) bacc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, fg[j], bacc[j], 0, 0, 0);
    };
    // fragments of one stage: the first (lo) and second (hi) half of the tile rows of A and the tile columns of G
    bf16x8_t fa_lo[MH], fa_hi[MH], fg[NI];
    float c_cur = 1.f;  // clip factor of the example being accumulated (set by the example's first stage)

    // prologue: NS - 1 stages in flight; publish stage 0
    constexpr int AHEAD = NS - 1;  // the newest stage in flight is AHEAD stages past the one being multiplied
#pragma unroll
    for (int st = 0; st < AHEAD; ++st) {
        stage_open();
#pragma unroll
        for (int k = 0; k < LPS; ++k) fill(k, st);
        stage_close();
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 1) * LPS) : "memory");  // stage 0 has landed
    __syncthreads();
    int buf = 0;      // ring slot of the stage being multiplied
    int ibuf = AHEAD; // ring slot the next load fills
    load_fa(buf, 0, fa_lo);
#pragma unroll
    for (int j = 0; j < NI; ++j) fg[j] = read_frag(&Gs[buf][foffG[j]], BN);

    // One loop iteration = one stage = one barrier.
    int duty_ctr = 0;  // (index of the stage being multiplied) % duty_mod
    int ex_run = __builtin_amdgcn_readfirstlane(a.flat ? 0 : (int)((uint32_t)k_lo / (uint32_t)a.T));  // the next example to start (row splits begin on examples)
    const int nex = a.flat ? 0 : (int)(a.K / a.T);
    // lane l: clip factor c_e of example e = (ex & ~63) + l and the rescaling ratio c_{e-1} / c_e that applies when
    // example e starts.  Two plain loads per 64 examples; the compiler's wait for them also waits for the
    // LDS-filling loads in flight, a bubble once per 64 examples.
    float cvec = 1.f, rvec = 1.f;
    auto load_factors = [&](int ex) {
        const int e = (ex & ~63) + lane;
        const float n_e = e < nex ? a.sqnorms[e] : 1.f;
        const float n_p = (e >= 1 && e - 1 < nex) ? a.sqnorms[e - 1] : n_e;
        cvec = dp_clip_factor(n_e, a.C);
        rvec = dp_clip_factor(n_p, a.C) / cvec;
        if (cvec != cvec) atomicOr(a.err, DP_ERRBIT_NORM);  // NaN factor: this unit's sums become NaN as well
    };
    if (n_ex > 0 && !a.flat) load_factors(ex_run);
    // Rescaling at an example boundary (every accumulator register times c_prev / c_next) is spread over the two halves
    // around it: in the second half of the example's last stage (PRE) a tile of the first half is multiplied in every
    // MFMA slot and a tile of the second half two MFMAs after its own MFMA; the last two tiles directly before their
    // MFMAs in the second half of the next example's first stage (POST).  Every stage kind is a straight-line body.
    // An example of one stage is both at once (ONE): the two ratios meet in different tiles.
    constexpr int PLAIN = 0, POST = 1, PRE = 2, ONE = 3;
    float ratio = 1.f;  // c_prev / c_next of the boundary being worked on (set in PRE, used up in POST)
    auto scale_tile = [&](int i, int j, float by) {
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] *= by;
    };
    auto body = [&](auto kind_tag) {
        constexpr int KIND = decltype(kind_tag)::value;
        const float ratio_post = ratio;
        const int buf1 = buf + 1 == NS ? 0 : buf + 1;
        const bool bias_now = want_bias && duty_ctr == duty;
        duty_ctr = duty_ctr + 1 == duty_mod ? 0 : duty_ctr + 1;
        load_fa(buf, 1, fa_hi);  // needed by the second half
        if (KIND & POST) {
            // first stage of example ex_run: take over the example's factor
            const int el = __builtin_amdgcn_readfirstlane(ex_run & 63);
            c_cur = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, cvec), el));
            ++ex_run;
        }
        // first half, tile column by tile column
#pragma unroll
        for (int t = 0; t < MH * NI; ++t) {
            const int i = t % MH, j = t / MH;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa_lo[i], fg[j], acc[i][j], 0, 0, 0);
        }
        if (KIND & POST) {
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) bacc[j][r] *= ratio_post;
        }
        if (bias_now) mma_bias(fg);
        __builtin_amdgcn_s_setprio(0);
        // my loads of the next stage have landed (later stages may still be in flight); after the barrier every
        // wave's have, and every wave has finished reading the stage whose ring slot the newest stage now overwrites
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 2) * LPS) : "memory");
        __syncthreads();
        load_fa(buf1, 0, fa_lo);  // the next stage's first half
        if (KIND & PRE) {
            // last stage of example ex_run - 1; the factors of 64 examples sit in registers (lane = example mod 64)
            if ((ex_run & 63) == 0) load_factors(ex_run);
            const int el = __builtin_amdgcn_readfirstlane(ex_run & 63);
            ratio = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, rvec), el));
        }
        // second half.  When a tile column is done its G fragment makes room for the next stage's, and the LDS-filling
        // loads of the newest stage go out one by one (spread, not back to back: issued together by all eight waves they
        // queue up in the address unit).
        {
            // of the two waves that share a SIMD, the one in the half that also issues the fills goes first (+3 %
            // measured; raising the priority in the first half as well costs 1 %)
            __builtin_amdgcn_s_setprio(1);
            stage_open();
#pragma unroll
            for (int t = 0; t < MH * NI; ++t) {
                const int i = MH + t % MH, j = t / MH;
                if ((KIND & POST) && t >= MH * NI - 2) {
                    __builtin_amdgcn_sched_barrier(0);
                    scale_tile(i, j, ratio_post);
                    __builtin_amdgcn_sched_barrier(0);
                }
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa_hi[t % MH], fg[j], acc[i][j], 0, 0, 0);
                if (t % MH == MH - 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    fg[j] = read_frag(&Gs[buf1][foffG[j]], BN);
#pragma unroll
                    for (int k = 0; k < LPS; ++k)
                        if (k * NI / LPS == j) fill(k, ibuf);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (KIND & PRE) {
                    __builtin_amdgcn_sched_barrier(0);
                    scale_tile(t % MH, t / MH, ratio);
                    if (t >= 2) scale_tile(MH + (t - 2) % MH, (t - 2) / MH, ratio);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            stage_close();
        }
        __builtin_amdgcn_s_setprio(0);
        ibuf = ibuf + 1 == NS ? 0 : ibuf + 1;
        buf = buf1;
    };
    // The unit's rows are whole examples (the host aligns row splits to examples), or, flat, one run.
    if (EPI != EPI_SQNORM) {
        if constexpr (ONE_STAGE) {
            for (int e = 0; e + 1 < n_ex; ++e) body(std::integral_constant<int, ONE>{});
        } else {
            for (int e = 0; e + 1 < n_ex; ++e) {
                body(std::integral_constant<int, POST>{});
                for (int q = 0; q < spe - 2; ++q) body(std::integral_constant<int, PLAIN>{});
                body(std::integral_constant<int, PRE>{});
            }
        }
    }
    if (n_ex > 0) {
        body(std::integral_constant<int, POST>{});
        for (int q = 0; q < spe - 1; ++q) body(std::integral_constant<int, PLAIN>{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may still be writing LDS when the workgroup ends

    if constexpr (EPI == EPI_SQNORM) {
        // rows / columns past the layer's widths hold products of neighbouring data: leave them out
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int p = p0 + wr * WM + 16 * i + 4 * (lane >> 4) + r;
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const float v = (p < a.d_in && q0 + wc * WN + 16 * j + (lane & 15) < a.d_out) ? acc[i][j][r] : 0.f;
                    s += v * v;
                }
            }
        // the bias gradient's entries (the columns of G summed: every row of the ones-product) count like a row of the weights
        if (want_bias && duty == 0 && lane < 16) {
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const float v = q0 + wc * WN + 16 * j + lane < a.d_out ? bacc[j][0] : 0.f;
                s += v * v;
            }
        }
        const float tot = dp_block_sum<512>(s, reinterpret_cast<float*>(&As[0][0]));
        if (tid == 0) a.out[((size_t)split * b.n_layers + layer) * ntiles + tile] = tot;
        return;
    }

    // MFMA tile (i, j): accumulator register r of lane l holds row 4*(l/16) + r, column l%16.  Buffer accesses over 16 rows of
    // the output at a time: rows past d_in lie outside the resource, lanes of columns past d_out get an offset outside it, so
    // there is no branch around an access.  The loads of two tile rows (32 a lane) are in flight while the two before them are
    // stored: written as one "*dst += x" after the other, each of the 128 accesses of a lane waited for its own round trip,
    // 40 us a workgroup (28 layers of 768 x 768, K = 1,024 rows: 95 -> 59 us a launch; 30,528 x 1,024, K = 5,120: 435 -> 368 us;
    // 4 layers of 1024 x 4096, K = 65,536: 1,902 -> 1,871 us).
    float* base = b.L[layer].out + (EPI == EPI_STORE ? (size_t)split * a.d_in * a.d_out : (size_t)0);
    uint32_t voff[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int q = q0 + wc * WN + 16 * j + (lane & 15);
        voff[j] = q < a.d_out ? (uint32_t)(4 * (lane >> 4) * a.d_out + q) * 4u : 0x80000000u;  // + at most 3 rows: still outside
    }
    const uint32_t pitch = (uint32_t)a.d_out * 4u;
    auto row_rsrc = [&](int i) {
        const int p = p0 + wr * WM + 16 * i;
        const int rows = a.d_in - p < 16 ? (a.d_in - p < 0 ? 0 : a.d_in - p) : 16;
        return uniform_rsrc(base + (size_t)p * a.d_out, rows * pitch);
    };
    float old[2][2][4][NI];
    auto fetch = [&](int g) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const __amdgpu_buffer_rsrc_t rs = row_rsrc(2 * g + u);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    old[g & 1][u][r][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(voff[j] + r * pitch), 0, 0));
        }
    };
    if (EPI == EPI_ADD) fetch(0);
#pragma unroll
    for (int g = 0; g < MI / 2; ++g) {
        if (EPI == EPI_ADD && g + 1 < MI / 2) fetch(g + 1);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const __amdgpu_buffer_rsrc_t rs = row_rsrc(2 * g + u);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const float x = acc[2 * g + u][j][r] * c_cur;
                    const float y = EPI == EPI_ADD ? old[g & 1][u][r][j] + x : x;
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, y), rs, (int)(voff[j] + r * pitch), 0, 0);
                }
        }
    }
    // every row of the ones-product equals the column sums; row 0 sits in register 0 of lanes 0..15
    if (want_bias && lane < 16 && (!a.bias_direct || duty == 0)) {
        float* bp = a.bias_direct ? b.L[layer].sum_b : a.bias_part + ((size_t)(unit * a.tiles_m + pm) * 2 + wr) * a.d_out;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int q = q0 + wc * WN + 16 * j + lane;
            if (q < a.d_out) bp[q] = (a.bias_direct ? bp[q] : 0.f) + bacc[j][0] * c_cur;
        }
    }
}

// Calibration: the clip-weighted GEMM's matrix work with nothing around it - 32 accumulator tiles of 16 x 16 per wave
// (128 registers), 8 + 4 operand fragments that stay in registers, 32 MFMAs per iteration, 8 waves per workgroup (two
// per SIMD), one workgroup per CU.  Operands are pseudo-random bf16 values in +-[1, 2) (the rate the chip sustains
// depends on the data: on zeros it holds a higher clock).  What this loop sustains is the ceiling of any kernel that
// executes these MFMAs on this card under its power limit.
__global__ __launch_bounds__(512) void mfma_ceiling_kernel(int iters, float* __restrict__ sink) {
    constexpr int MI = 8, NI = 4;
    const uint32_t t = blockIdx.x * 512u + threadIdx.x;
    auto rnd = [&](uint32_t k) {  // two bf16 values with random sign and mantissa, exponent 0
        uint32_t h = (t * 0x9E3779B1u) ^ (k * 0x85EBCA77u);
        h ^= h >> 15; h *= 0x2C1B3C6Du; h ^= h >> 12; h *= 0x297A2D39u; h ^= h >> 15;
        return (h & 0x807F807Fu) | 0x3F803F80u;
    };
    bf16x8_t fa[MI], fg[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[i] = __builtin_bit_cast(bf16x8_t, u32x4_t{rnd(8 * i), rnd(8 * i + 1), rnd(8 * i + 2), rnd(8 * i + 3)});
#pragma unroll
    for (int j = 0; j < NI; ++j) fg[j] = __builtin_bit_cast(bf16x8_t, u32x4_t{rnd(100 + 8 * j), rnd(101 + 8 * j), rnd(102 + 8 * j), rnd(103 + 8 * j)});
    f32x4_t acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fg[j], acc[i][j], 0, 0, 0);
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) s += (acc[i][j][0] + acc[i][j][1]) + (acc[i][j][2] + acc[i][j][3]);
    sink[t] = s;
}

// Operands for the GEMM without factors: Gs = bf16(c_i * G) (products formed in fp32, rounded to nearest even), rows of one example after the other, and the column sums of the fp32 products
// of a run of rows for the bias (part[layer][run][d], if wanted).  8 columns a thread, 256 columns x 8 rows a workgroup.
// Bound: HBM, 4 bytes per element.  grid (runs, d / 256, layers).
struct ScaleBatch {
    const uint16_t* G[MAX_BATCH];
    uint16_t* Gs[MAX_BATCH];
};
__global__ __launch_bounds__(256) void scale_rows_kernel(ScaleBatch sb, const float* __restrict__ sqnorms, float C, int T, long K, int d,
                                                         int rows_per, float* __restrict__ part, int* __restrict__ err) {
    __shared__ float red[8][32][9];
    const uint16_t* __restrict__ G = sb.G[blockIdx.z];
    uint16_t* __restrict__ Gs = sb.Gs[blockIdx.z];
    const int cl = threadIdx.x & 31, ry = threadIdx.x >> 5;
    const int col = blockIdx.y * 256 + cl * 8;
    const long r0 = (long)blockIdx.x * rows_per, r1 = r0 + rows_per < K ? r0 + rows_per : K;
    float s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = 0.f;
    if (col < d) {
#pragma unroll 4
        for (long r = r0 + ry; r < r1; r += 8) {
            const float c = dp_clip_factor(sqnorms[(uint32_t)r / (uint32_t)T], C);
            if (c != c) atomicOr(err, DP_ERRBIT_NORM);
            u32x4_t v = *reinterpret_cast<const u32x4_t*>(G + (size_t)r * d + col);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const f32x2_t x = {dp_bf16_lo(v[w]) * c, dp_bf16_hi(v[w]) * c};
                s[2 * w] += x[0];
                s[2 * w + 1] += x[1];
                v[w] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));
            }
            *reinterpret_cast<u32x4_t*>(Gs + (size_t)r * d + col) = v;
        }
    }
    if (!part) return;
#pragma unroll
    for (int e = 0; e < 8; ++e) red[ry][cl][e] = s[e];
    __syncthreads();
    const int c2 = threadIdx.x >> 3, e2 = threadIdx.x & 7;
    if (blockIdx.y * 256 + c2 * 8 < d) {
        float t = 0.f;
#pragma unroll
        for (int r = 0; r < 8; ++r) t += red[r][c2][e2];
        part[((size_t)blockIdx.z * gridDim.x + blockIdx.x) * d + blockIdx.y * 256 + c2 * 8 + e2] = t;
    }
}

// ------------------------------------------------------------------------------------------------
// fp32 inputs, on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: products and sums in fp32).  The contraction index is
// the slow index of both operands in memory and the MFMA wants one k per half-wave: a lane's operand is simply the element
// (row k + lane / 32, column lane % 32), 128 contiguous bytes a half-wave, straight from global memory into registers.  A
// workgroup owns a tile of 32 TM x 32 TN; its 8 waves take the row pairs in turn (24 flop per byte of L2 at 3 x 3, 16 at 2 x 2, 12 at 3 x 1: 6, 10 and
// 13 TB/s at the full matrix rate) and their accumulators meet in LDS.  c_i multiplies G on the way in; the workgroups of tile row
// 0 also add up the columns of c * G for the bias.
// A block of rows is addressed by 32-bit offsets into one buffer resource; where a layer is so wide that a block's bytes do not
// fit 32 bits (from 2^23 columns), WIDE forms 64-bit addresses per lane.
// 1024 x 1024, 8,192 rows: 107 TFLOP/s of the 154 that the vendor's fp32 product reaches.
// B * T = 2,048 rows, 768 x 768: 397 + 9 (bias) -> 38 us (16 x 16 threads with 4 x 4 sums each, before); 64 x 64, 512 rows: 70 -> 8 us.
// ------------------------------------------------------------------------------------------------
constexpr int F32_WAVES = 8;
constexpr int F32_FACTORS = 1024;  // clip factors a workgroup forms itself; with more examples in its rows they come precomputed

// Row pairs a wave of a TM x TN tile has in flight beside those it multiplies, and the rows of a workgroup's block of them.
constexpr int f32_pairs(int tm, int tn) { return tm + tn < 3 ? 16 : tm + tn > 4 ? 4 : 8; }
constexpr int f32_block(int tm, int tn) { return 2 * F32_WAVES * f32_pairs(tm, tn); }

template <int TM, int TN, bool OWN, bool WIDE>
__global__ __launch_bounds__(64 * F32_WAVES) void wgemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ G,
                                                                   const float* __restrict__ c_or_sq, float C, int T, long K,
                                                                   int d_in, int d_out, long rows_per_split, int add, float* __restrict__ out,
                                                                   float* __restrict__ out_b, int* __restrict__ err) {
    constexpr int NR = TM * TN * 16;      // accumulator registers of a wave
    constexpr int U = f32_pairs(TM, TN);
    __shared__ float part[F32_WAVES / 2][NR][64];
    __shared__ float bpart[F32_WAVES][TN][64];
    __shared__ float ctab[OWN ? F32_FACTORS : 1];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5;
    const int p0 = blockIdx.y * 32 * TM, q0 = blockIdx.x * 32 * TN;
    const long k_lo = (long)blockIdx.z * rows_per_split;
    const long k_hi = k_lo + rows_per_split < K ? k_lo + rows_per_split : K;
    f32x16_t acc[TM][TN];
    float bs[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        bs[j] = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    }
    const bool do_bias = out_b != nullptr && blockIdx.y == 0;
    if constexpr (OWN) {
        const int e_lo = (int)((uint32_t)k_lo / (uint32_t)T), e_hi = k_hi > k_lo ? (int)((uint32_t)(k_hi - 1) / (uint32_t)T) : e_lo - 1;
        for (int e = e_lo + threadIdx.x; e <= e_hi; e += 64 * F32_WAVES) {
            const float ce = dp_clip_factor(c_or_sq[e], C);
            ctab[e - e_lo] = ce;
            if (ce != ce) atomicOr(err, DP_ERRBIT_NORM);
        }
    }
    // Rows of this lane, relative to k_lo: 2 * wave + half, then every 16th, in blocks of 16 U.  Buffer loads whose resource ends
    // at the split's last row: a row past it arrives as zeros, and there is no branch or select around a load.
    constexpr int BLK = f32_block(TM, TN);
    const int r_first = 2 * wave + half, n_rows = k_hi > k_lo ? (int)(k_hi - k_lo) : 0;
    const uint32_t pitchA = (uint32_t)d_in * 4u, pitchG = (uint32_t)d_out * 4u;
    uint32_t voffA[TM], voffG[TN];  // columns past the widths repeat the last one and feed entries that are never stored
#pragma unroll
    for (int e = 0; e < TM; ++e) {
        const int p = p0 + 32 * e + (lane & 31);
        voffA[e] = r_first * pitchA + (p < d_in ? p : d_in - 1) * 4u;
    }
#pragma unroll
    for (int e = 0; e < TN; ++e) {
        const int q = q0 + 32 * e + (lane & 31);
        voffG[e] = r_first * pitchG + (q < d_out ? q : d_out - 1) * 4u;
    }
    struct Rows {
        float a[U][TM], g[U][TN];
    };
    struct Src {
        __amdgpu_buffer_rsrc_t A, G;
    };
    struct WideSrc {
        long row;
    };
    auto block = [&](int it) {  // resources over the rows of block `it`
        if constexpr (WIDE) {
            return WideSrc{(long)it * BLK + r_first};
        } else {
            const int left = n_rows - it * BLK, rows = left < 0 ? 0 : left < BLK ? left : BLK;
            const size_t at = (size_t)k_lo + (size_t)it * BLK;
            return Src{uniform_rsrc(A + at * d_in, rows * pitchA), uniform_rsrc(G + at * d_out, rows * pitchG)};
        }
    };
    auto load = [&](Rows& x, const auto& s, int u) {
        if constexpr (WIDE) {
            const long r = s.row + u * 2 * F32_WAVES;
            const bool in = r < n_rows;  // past the last row: that row is read, and zeros taken in its place
            const size_t at = (size_t)k_lo + (size_t)(in ? r : n_rows - 1);
#pragma unroll
            for (int e = 0; e < TM; ++e) {
                const int p = p0 + 32 * e + (lane & 31);
                const float v = A[at * d_in + (p < d_in ? p : d_in - 1)];
                x.a[u][e] = in ? v : 0.f;
            }
#pragma unroll
            for (int e = 0; e < TN; ++e) {
                const int q = q0 + 32 * e + (lane & 31);
                const float v = G[at * d_out + (q < d_out ? q : d_out - 1)];
                x.g[u][e] = in ? v : 0.f;
            }
        } else {
#pragma unroll
            for (int e = 0; e < TM; ++e)
                x.a[u][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(s.A, (int)(voffA[e] + u * 2 * F32_WAVES * pitchA), 0, 0));
#pragma unroll
            for (int e = 0; e < TN; ++e)
                x.g[u][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(s.G, (int)(voffG[e] + u * 2 * F32_WAVES * pitchG), 0, 0));
        }
    };
    // The factor of the lane's row.  One step of 16 rows passes one boundary at most when T >= 16: the example follows by
    // comparison; shorter examples are found by division.  (Either way no memory access and no loop under a branch: the
    // compiler's count of loads in flight would be lost at the join.)
    const int e_off = OWN ? (int)((uint32_t)k_lo / (uint32_t)T) : 0;
    int row = r_first;  // the next row to multiply
    int ex = (int)((uint32_t)(k_lo + r_first < K ? k_lo + r_first : K - 1) / (uint32_t)T) - e_off;
    long bound = (long)(ex + e_off + 1) * T - k_lo;  // first row of the next example
    auto factors = [&](float (&w)[U]) {
        int e[U];
        if (T >= 2 * F32_WAVES) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool over = row + u * 2 * F32_WAVES >= bound && row + u * 2 * F32_WAVES < n_rows;
                ex += over ? 1 : 0;
                bound += over ? T : 0;
                e[u] = ex;
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = row + u * 2 * F32_WAVES < n_rows ? row + u * 2 * F32_WAVES : n_rows - 1;
                e[u] = (int)((uint32_t)(k_lo + r) / (uint32_t)T) - e_off;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = OWN ? ctab[e[u]] : c_or_sq[e[u]];
        row += BLK;
    };
    auto mma = [&](const Rows& x, int u, float w) {
        float g[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            // zeros past the range stay zeros: the repeated factor is that of a row inside it, finite or NaN with it
            g[j] = w * x.g[u][j];
            bs[j] += g[j];
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.a[u][i], g[j], acc[i][j], 0, 0, 0);
    };
    const int n_iter = (n_rows + BLK - 1) / BLK;  // (the same for every wave)
    Rows x0, x1;
    {
        const auto s = block(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {  // (in order: the wait counts of the loop are only as tight as the order on entry is certain)
            load(x0, s, u);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (OWN) __syncthreads();  // the factors are in place
    auto step = [&](const Rows& now, Rows& next, int it_next) {  // multiply a block, the next one's loads spread between the MFMAs
        float w[U];
        factors(w);
        const auto s = block(it_next);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            load(next, s, u);
            mma(now, u, w[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int it = 0; it < n_iter; it += 2) {
        step(x0, x1, it + 1);
        step(x1, x0, it + 2);
    }
    // waves w + 4 hand their tiles to waves w, whose four sums every wave then adds for an eighth of the registers
    constexpr int HW = F32_WAVES / 2;
#pragma unroll
    for (int e = 0; e < TN; ++e) bpart[wave][e][lane] = bs[e];
    if (wave >= HW) {
#pragma unroll
        for (int r = 0; r < NR; ++r) part[wave - HW][r][lane] = acc[r / (16 * TN)][r / 16 % TN][r % 16];
    }
    __syncthreads();
    if (wave < HW) {
#pragma unroll
        for (int r = 0; r < NR; ++r) part[wave][r][lane] += acc[r / (16 * TN)][r / 16 % TN][r % 16];
    }
    __syncthreads();
    float* __restrict__ dst = out + (size_t)blockIdx.z * (add ? 0 : (size_t)d_in * d_out);
    constexpr int NK = NR / F32_WAVES;
    float old[NK];
    auto place = [&](int k, int& p, int& q) {  // accumulator register r of lane l: row 8*(r/4) + 4*(l/32) + r%4, column l%32 of its tile
        const int r = wave * NK + k, rr = r % 16;
        p = p0 + 32 * (r / (16 * TN)) + 8 * (rr >> 2) + 4 * half + (rr & 3);
        q = q0 + 32 * (r / 16 % TN) + (lane & 31);
        return p < d_in && q < d_out;
    };
#pragma unroll
    for (int k = 0; k < NK; ++k) {  // all the reads first: one after the other with the writes, each waits for its round trip
        int p, q;
        old[k] = place(k, p, q) && add ? dst[(size_t)p * d_out + q] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int r = wave * NK + k;
        const float v = (part[0][r][lane] + part[1][r][lane]) + (part[2][r][lane] + part[3][r][lane]);
        int p, q;
        if (place(k, p, q)) dst[(size_t)p * d_out + q] = old[k] + v;
    }
    if (do_bias && threadIdx.x < 32 * TN && q0 + (int)threadIdx.x < d_out) {
        const int e = threadIdx.x >> 5, l = threadIdx.x & 31;
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < F32_WAVES; ++w) t += bpart[w][e][l] + bpart[w][e][l + 32];
        float* o = out_b + (size_t)blockIdx.z * (add ? 0 : d_out) + q0 + threadIdx.x;
        *o = add ? *o + t : t;
    }
}

}  // namespace

namespace {
// What is left to add behind a launch of the GEMM, all layers in one launch (blockIdx.y = layer); the first w_blocks workgroups of
// a layer add the row splits' partial sums, the others the bias partials:
//   out_l[j] += sum_{r<R} part_l[r*n4 + j]         (float4 columns j < n4)
//   sum_b_l[q] += sum_{r<nb} bias_part[(l*nb + r)*d_out + q]
// Many partials of few columns (TALL, and the bias): 64 columns and four groups of partials a workgroup, group g adding
// r = g, g + 4, ... with eight loads in flight, then (0 + 1) + (2 + 3).  Otherwise a thread per column, r ascending.  Fixed orders.
// (One thread walking all partials of its column: 10 us for 32 bias rows, this way 5; 64 splits of 64 x 64 12 | 4.  As two launches,
// one behind the other, a call of a small layer waits for the host: B = 147, T = 192, 72 x 136 22.5 us, 17.2 as one.)
struct FinishArgs {
    const float4* part[MAX_BATCH];
    float4* out[MAX_BATCH];
    float* sum_b[MAX_BATCH];
};
template <typename V>
__device__ __forceinline__ V add_partials(const V* __restrict__ src, size_t stride, int first, int step, int n) {
    V t{};
    int r = first;
    for (; r + 7 * step < n; r += 8 * step) {
        V p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = src[(size_t)(r + u * step) * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) t += p[u];
    }
    for (; r < n; r += step) t += src[(size_t)r * stride];
    return t;
}
template <bool TALL>
__global__ __launch_bounds__(256) void finish_layers_kernel(FinishArgs f, int R, size_t n4, int w_blocks, const float* __restrict__ bias_part,
                                                            int nb, int d_out) {
    __shared__ f32x4_t red[4][64];
    __shared__ float bred[4][64];
    const int layer = blockIdx.y, lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    if ((int)blockIdx.x >= w_blocks) {
        float* dst = f.sum_b[layer];
        if (!dst) return;
        const int q = ((int)blockIdx.x - w_blocks) * 64 + lane;
        bred[g][lane] = q < d_out ? add_partials(bias_part + (size_t)layer * nb * d_out + q, (size_t)d_out, g, 4, nb) : 0.f;
        __syncthreads();
        if (g == 0 && q < d_out) dst[q] += (bred[0][lane] + bred[1][lane]) + (bred[2][lane] + bred[3][lane]);
        return;
    }
    const f32x4_t* __restrict__ part = reinterpret_cast<const f32x4_t*>(f.part[layer]);
    f32x4_t* __restrict__ out = reinterpret_cast<f32x4_t*>(f.out[layer]);
    if constexpr (TALL) {
        const size_t j = (size_t)blockIdx.x * 64 + lane;
        red[g][lane] = j < n4 ? add_partials(part + j, n4, g, 4, R) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        __syncthreads();
        if (g == 0 && j < n4) out[j] += (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    } else {
        const size_t j = (size_t)blockIdx.x * 256 + threadIdx.x;
        if (j < n4) {
            const f32x4_t old = out[j];  // asked for with the partials
            out[j] = old + add_partials(part + j, n4, 0, 1, R);
        }
    }
}
}  // namespace

// R = 1: no partial sums of the weights, nb = 0: none of the biases.
static dp_status finish_layers(dp_ctx* ctx, const FinishArgs& f, int nl, int R, size_t n4, const float* bias_part, int nb, int d_out) {
    const bool tall = R >= 16 && n4 * nl <= 16384;  // too few columns to fill the chip one a thread
    const long w_blocks = R > 1 ? (long)((n4 + (tall ? 63 : 255)) / (tall ? 64 : 256)) : 0, b_blocks = nb ? (d_out + 63) / 64 : 0;
    const dim3 grid((unsigned)(w_blocks + b_blocks), nl);
    if (tall) hipLaunchKernelGGL(finish_layers_kernel<true>, grid, dim3(256), 0, ctx->stream, f, R, n4, (int)w_blocks, bias_part, nb, d_out);
    else hipLaunchKernelGGL(finish_layers_kernel<false>, grid, dim3(256), 0, ctx->stream, f, R, n4, (int)w_blocks, bias_part, nb, d_out);
    DP_LAUNCH_CHECK(ctx, "finish_layers");
    return DP_OK;
}

static dp_status weighted_sum_single(dp_ctx* ctx, const void* A, const void* G, dp_dtype dt, int B, int T, int d_in, int d_out,
                                     const float* sqnorms, float C, float* sum_W, float* sum_b);

// What a launch of the direct-to-LDS kernel is made of: block tile, with or without factors, and layers per launch.
constexpr long BIAS_DIRECT_STAGES = 64;

struct DmaPlan {
    int bm, bn;
    bool flat;
    int per_launch;
    long nsplit;  // of a launch of min(n, per_launch) layers
};

// What a workgroup of a tile costs in microseconds, measured over 16 layers of 1024 x 1024 and 28 of 768 x 768 with 1,024 to
// 32,768 rows: a stage of BK rows (256 x 256: 0.94; 128 x 128: 0.61 with two workgroups on a CU and 0.40 alone; mixed tiles
// 0.58: per flop the large tile is the fastest by a fifth, it reads the fewest fragment bytes from LDS), and prologue plus
// epilogue, whose share that is bandwidth grows with the part of the chip that is at it.
struct DmaCost {
    int wgs;  // workgroups a CU holds
    double t_stage, t_stage_alone, t_ends, t_ends_full;
};
static DmaCost dma_cost(int bm, int bn, bool one_stage) {
    if (bm == 256 && bn == 256) return {1, 0.94, 0.94, 7.0, 13.0};
    if (bm == 128 && bn == 128) return one_stage ? DmaCost{2, 0.9, 0.5, 5.0, 7.0} : DmaCost{2, 0.61, 0.40, 5.0, 7.0};
    return {1, 0.58, 0.58, 6.0, 7.0};
}
// The same for launches of several rounds of workgroups, fitted to 170 shapes timed with every tile and row split (2 to 65,536 rows, widths of
// 64 to 4,096, 1 to 64 layers): the workgroups of later rounds do not run in step, so the bandwidth part is paid by the workgroup, whatever the round holds.
static DmaCost dma_cost_rounds(int bm, int bn, bool one_stage) {
    if (bm == 256 && bn == 256) return {1, 0.855, 0.855, 6.9, 16.3};
    if (bm == 128 && bn == 128) return one_stage ? DmaCost{2, 0.75, 0.365, 3.2, 7.2} : DmaCost{2, 0.61, 0.375, 3.2, 7.2};
    if (bm == 256) return {1, 0.575, 0.585, 6.5, 5.2};
    return {1, 0.57, 0.55, 6.5, 5.2};
}

// Row-split count of one launch over `nl` layers of `ntiles` tiles: the count with the smallest modelled time, in
// microseconds to *t_out.  An XCD runs 32 * wgs workgroups at a time and gets an eighth of the launch's workgroups, so
// the launch takes ceil(workgroups / 8 / (32 wgs)) rounds of one workgroup's time; more than one split sends partial sums
// through memory and costs one reduction launch (which finds most of them in the cache: 4 layers of 768 x 3072 in three
// splits, 190 MB in 30 us).  `spe`: stages per example
// (splits start on examples).  ROUNDS: by the costs of several rounds, and only splits that the workspace holds.
template <bool ROUNDS>
static long choose_nsplit_dma(int nl, int ntiles, long ksteps, long spe, int d_in, int d_out, const DmaCost& c, size_t ws_bytes, double* t_out) {
    const long max_split = ksteps / 8 < 1 ? 1 : ksteps / 8;
    long best = 1;
    double best_t = 0.0;
    for (long s = 1; s <= max_split && s <= 64; ++s) {
        const long steps_per = ((ksteps + s - 1) / s + spe - 1) / spe * spe;
        const long se = (ksteps + steps_per - 1) / steps_per;  // the splits that are not empty
        if (se != s && s > 1) continue;                        // the same plan as a smaller s
        if (ROUNDS && s > 1 && (size_t)nl * se * d_in * d_out * 4 > ws_bytes) break;
        const long wg = (long)nl * se * ntiles;
        const long per_xcd = (wg + 7) / 8;
        const long rounds = (per_xcd + 32 * c.wgs - 1) / (32 * c.wgs);
        const double full = (double)wg / (256.0 * c.wgs), stages = (double)steps_per * (wg <= 256 ? c.t_stage_alone : c.t_stage);
        double t = ROUNDS ? (double)rounds * (stages + c.t_ends) + c.t_ends_full * full
                          : (double)rounds * (stages + c.t_ends + c.t_ends_full * (full < 1.0 ? full : 1.0));
        if (se > 1) t += (double)nl * (double)(se + 2) * d_in * d_out * 4.0 / (ROUNDS ? 11.3e6 : 8.0e6) + (ROUNDS ? 3.6 : 5.0);
        if (s == 1 || t < best_t) {
            best = se;
            best_t = t;
        }
    }
    *t_out = best_t;
    return best;
}

// Layers per launch in the scaled form: those whose scaled output gradients fit half the workspace, with room for their bias partials besides (one row for up
// to 32 token rows and no more than 256: a sixteenth of the gradients, but more than they take for a single row).
static long scaled_layers(long K, int d_out, size_t ws_bytes) {
    if (ws_bytes / 2 < 1024) return 0;
    const size_t scaled = (size_t)K * d_out * 2 + 256, bias = (size_t)((K + BK - 1) / BK < 256 ? (K + BK - 1) / BK : 256) * d_out * 4;
    size_t per = (ws_bytes / 2 - 1024) / scaled;
    if (per > (ws_bytes - 1024) / (scaled + bias)) per = (ws_bytes - 1024) / (scaled + bias);
    return per < MAX_BATCH ? (long)per : MAX_BATCH;
}

// Tile and form for n layers: the smallest modelled time of the whole call.
static DmaPlan choose_dma_plan(int n, int B, int T, int d_in, int d_out, size_t ws_bytes) {
    DmaPlan best{0, 0, false, 1, 1};
    double best_t = 0.0;
    const long K = (long)B * T;
    // calls f(tile rows, tile columns, stages of one example only, tiles, stages, stages per example, most layers per launch) for the tiles of a form
    auto tiles = [&](bool flat, auto f) {
        if (flat && T % BK == 0 && T > BK) return;  // whole stages: nothing to gain
        if (flat && d_out > 65535 * 256) return;    // (scale_rows_kernel has a grid row per 256 columns)
        const long most = flat ? scaled_layers(K, d_out, ws_bytes) : MAX_BATCH;
        if (most < 1) return;
        const long spe = flat ? 1 : (T + BK - 1) / BK;
        const long ksteps = flat ? (K + BK - 1) / BK : (long)B * spe;
        const bool one_stage = !flat && T <= BK;
        for (int bm = one_stage ? 128 : 256; bm >= 128; bm -= 128)
            for (int bn = one_stage ? 128 : 256; bn >= 128; bn -= 128)
                f(bm, bn, one_stage, ((d_in + bm - 1) / bm) * ((d_out + bn - 1) / bn), ksteps, spe, most);
    };
    auto scaling = [&](bool flat, long launches, double rate) { return flat ? (double)launches * 4.0 + 4.0 * (double)K * d_out * n / rate : 0.0; };
    for (const bool flat : {false, true})
        tiles(flat, [&](int bm, int bn, bool one_stage, int ntiles, long ksteps, long spe, long most) {
            const DmaCost c = dma_cost(bm, bn, one_stage);
            // layers per launch: enough to give every CU its workgroups, but no more than one round of them when a layer has many tiles
            long per = 256l * c.wgs / ntiles;
            per = per < 1 ? 1 : per > most ? most : per;
            double t = 0.0, tl;
            const long full = n / per, rest = n % per;
            long nsplit = 1;
            if (rest) {
                nsplit = choose_nsplit_dma<false>((int)rest, ntiles, ksteps, spe, d_in, d_out, c, ws_bytes, &tl);
                t += tl + 4.0;
            }
            if (full) {
                nsplit = choose_nsplit_dma<false>((int)per, ntiles, ksteps, spe, d_in, d_out, c, ws_bytes, &tl);
                t += full * (tl + 4.0);
            }
            t += scaling(flat, full + (rest ? 1 : 0), 4.0e6);
            if (!best.bm || t < best_t) {
                best = DmaPlan{bm, bn, flat, (int)per, nsplit};
                best_t = t;
            }
        });
    if (best.per_launch >= n || K > 64 * BK) return best;
    // Several launches so: the layers together, in one launch of as many rounds as it takes, where that is faster by the costs of such launches.  Short sums
    // are, up to 64 stages: 32 stages, 48 layers of 768 x 768 97 us apart, 88 together; 64 of 1024 x 1024 215 | 199; 6 stages, 36 layers of 640 x 640 53 | 44.  Long ones of which a second
    // round would be partly empty are not, and the others gain nothing: B = 23, T = 375, 6 layers of 832 x 3328 350 | 402; B = 128, T = 128, 32 of 1024 x 1024 975 | 972.  (In the form chosen above: the scaled one rounds c * g.)
    const bool scaled = best.flat;
    double apart = 0.0;
    tiles(best.flat, [&](int bm, int bn, bool one_stage, int ntiles, long ksteps, long spe, long) {
        if (bm != best.bm || bn != best.bn) return;
        const DmaCost c = dma_cost_rounds(bm, bn, one_stage);
        const long full = n / best.per_launch, rest = n % best.per_launch;
        double tl = 0.0;
        if (rest) choose_nsplit_dma<true>((int)rest, ntiles, ksteps, spe, d_in, d_out, c, ws_bytes, &tl);
        apart = rest ? tl + 7.0 : 0.0;
        choose_nsplit_dma<true>(best.per_launch, ntiles, ksteps, spe, d_in, d_out, c, ws_bytes, &tl);
        apart += full * (tl + 7.0) + scaling(best.flat, full + (rest ? 1 : 0), 6.0e6);
    });
    best_t = 0.97 * apart;  // (by more than the model is wrong)
    tiles(scaled, [&](int bm, int bn, bool one_stage, int ntiles, long ksteps, long spe, long most) {
        const DmaCost c = dma_cost_rounds(bm, bn, one_stage);
        const long per = n < most ? n : most, full = n / per, rest = n % per;
        double t = 0.0, tl;
        if (rest) {
            choose_nsplit_dma<true>((int)rest, ntiles, ksteps, spe, d_in, d_out, c, ws_bytes, &tl);
            t += tl + 7.0;
        }
        const long nsplit = choose_nsplit_dma<true>((int)per, ntiles, ksteps, spe, d_in, d_out, c, ws_bytes, &tl);
        t += full * (tl + 7.0) + scaling(scaled, full + (rest ? 1 : 0), 6.0e6);
        if (t < best_t) {
            best = DmaPlan{bm, bn, scaled, (int)per, nsplit};
            best_t = t;
        }
    });
    return best;
}

template <int MI, int NI, bool ONE_STAGE>
static void dma_launch(dp_ctx* ctx, const WgemmBatchArgs& b, unsigned grid, bool split) {
    if (split) hipLaunchKernelGGL((wgemm_dma16_kernel<MI, NI, EPI_STORE, ONE_STAGE>), dim3(grid), dim3(512), 0, ctx->stream, b);
    else hipLaunchKernelGGL((wgemm_dma16_kernel<MI, NI, EPI_ADD, ONE_STAGE>), dim3(grid), dim3(512), 0, ctx->stream, b);
}

// Clip-weighted sums of n same-shaped dense layers.  bf16 layers go out in launches of the direct-to-LDS kernel; fp32 layers
// and layers without weights one by one.
dp_status dpk_weighted_gemm_batched(dp_ctx* ctx, int n, const void* const* A, const void* const* G, dp_dtype dt, int B,
                                    int T, int d_in, int d_out, const float* sqnorms, float C, float* const* sum_W,
                                    float* const* sum_b) {
    if (dt != DP_BF16 || d_in == 0) {
        dp_status st = DP_OK;
        for (int l = 0; st == DP_OK && l < n; ++l)
            st = weighted_sum_single(ctx, A[l], G[l], dt, B, T, d_in, d_out, sqnorms, C, sum_W[l], sum_b ? sum_b[l] : nullptr);
        return st;
    }
    const DmaPlan plan = choose_dma_plan(n, B, T, d_in, d_out, ctx->ws_bytes);
    const bool one_stage = !plan.flat && T <= BK;
    const DmaCost cost = dma_cost(plan.bm, plan.bn, one_stage);
    const long K = (long)B * T;
    const long spe = plan.flat ? 1 : (T + BK - 1) / BK;  // row splits begin on examples: the kernel rescales across example boundaries only
    const long ksteps = plan.flat ? (K + BK - 1) / BK : (long)B * spe;
    int nl;
    for (int l0 = 0; l0 < n; l0 += nl) {
        nl = dp_disjoint_layers(n - l0 < plan.per_launch ? n - l0 : plan.per_launch, sum_W + l0, (size_t)d_in * d_out, sum_b ? sum_b + l0 : nullptr,
                                d_out);
        WgemmBatchArgs b;
        WgemmArgs& a = b.base;
        a.out = nullptr;
        a.sqnorms = sqnorms;
        a.C = C;
        a.err = ctx->err_word;
        a.flat = plan.flat ? 1 : 0;
        a.T = T;
        a.d_in = d_in;
        a.d_out = d_out;
        a.K = K;
        a.tiles_m = (d_in + plan.bm - 1) / plan.bm;
        a.tiles_n = (d_out + plan.bn - 1) / plan.bn;
        const int ntiles = a.tiles_m * a.tiles_n;
        double t_model;
        long nsplit = nl == (n < plan.per_launch ? n : plan.per_launch) ? plan.nsplit
                                                                       : choose_nsplit_dma<false>(nl, ntiles, ksteps, spe, d_in, d_out, cost, ctx->ws_bytes, &t_model);
        bool any_bias = false;
        for (int l = 0; l < nl; ++l)
            if (sum_b && sum_b[l0 + l]) any_bias = true;
        // flat: the scaled output gradients and their column sums per run of rows
        ScaleBatch sb;
        const int dblk = (d_out + 255) / 256;
        long runs = 0, rows_per = 0;
        dp_ws_alloc ws(ctx);
        float* bias_part = nullptr;
        if (plan.flat) {
            runs = 2048 / ((long)dblk * nl) < 1 ? 1 : 2048 / ((long)dblk * nl);
            if (runs > (K + 31) / 32) runs = (K + 31) / 32;
            if (runs > 256) runs = 256;
            rows_per = (K + runs - 1) / runs;
            runs = (K + rows_per - 1) / rows_per;
            for (int l = 0; l < MAX_BATCH; ++l) {  // (the plan has seen that they fit)
                sb.G[l] = (const uint16_t*)G[l0 + (l < nl ? l : 0)];
                sb.Gs[l] = l < nl ? ws.get<uint16_t>((size_t)K * d_out) : sb.Gs[0];
            }
            if (any_bias) bias_part = ws.get<float>((size_t)nl * runs * d_out);
            if (!sb.Gs[nl - 1] || (any_bias && !bias_part)) {
                DP_SET_ERR(ctx, "workspace too small for the scaled output gradients");
                return DP_ERR_WORKSPACE;
            }
        }

        const size_t ws_mark = ws.off;
        // partial sums [nl][nsplit][d_in][d_out] and bias partials (one row per unit, tile row and wave row):
        // fewer splits until the workspace holds both.  One split of few stages adds its bias sums itself: a launch less for
        // an extra MFMA column in an eighth of the waves' work (and the form that needs no workspace at all).
        float* part = nullptr;
        a.bias_direct = 0;
        for (;;) {
            ws.off = ws_mark;
            if (!plan.flat && any_bias && nsplit == 1 && ksteps <= BIAS_DIRECT_STAGES) {
                a.bias_direct = 1;
                break;
            }
            part = nsplit > 1 ? ws.get<float>((size_t)nl * nsplit * d_in * d_out) : nullptr;
            if (!plan.flat) bias_part = any_bias ? ws.get<float>((size_t)nl * nsplit * a.tiles_m * 2 * d_out) : nullptr;
            if ((nsplit == 1 || part) && (!any_bias || bias_part)) break;
            if (nsplit == 1) {
                a.bias_direct = 1;
                break;
            }
            nsplit = nsplit > 8 ? nsplit - 8 : nsplit / 2;
        }
        const long steps_per = ((ksteps + nsplit - 1) / nsplit + spe - 1) / spe * spe;
        a.rows_per_split = plan.flat ? steps_per * BK : steps_per / spe * T;
        nsplit = (ksteps + steps_per - 1) / steps_per;
        a.nsplit = (int)nsplit;
        const long nunits = (long)nl * nsplit;
        // whole units dealt to the XCDs when that is balanced; otherwise equal runs of the (unit, tile) sequence
        a.xcd_map = nunits % 8 == 0 ? 1 : 3;
        a.rect_m = a.rect_n = 1;
        if (nunits < 8 && 8 % nunits == 0) {
            // 8 / nunits rectangles per unit: the cut with the smallest half-perimeter (operand bytes per XCD)
            const int nrect = 8 / (int)nunits;
            int best = -1;
            for (int rm = 1; rm <= nrect; ++rm) {
                if (nrect % rm) continue;
                const int rn = nrect / rm;
                if (a.tiles_m % rm || a.tiles_n % rn) continue;
                const int cost = a.tiles_m / rm + a.tiles_n / rn;
                if (best < 0 || cost < best) {
                    best = cost;
                    a.rect_m = rm;
                    a.rect_n = rn;
                }
            }
            if (best >= 0) a.xcd_map = 2;
        }
        if (a.xcd_map != 2 && ntiles > 32) {
            // rectangle of about 32 tiles (one XCD's worth of workgroups) with the smallest half-perimeter
            int best = -1;
            for (int tm = 1; tm <= a.tiles_m && tm <= 32; ++tm) {
                if (a.tiles_m % tm) continue;
                int tn = 32 / tm;
                if (tn > a.tiles_n) tn = a.tiles_n;
                while (tn > 1 && a.tiles_n % tn) --tn;
                const int cost = (tm + tn) * 1024 / (tm * tn);  // operand columns fetched per tile
                if (best < 0 || cost < best) {
                    best = cost;
                    a.rect_m = tm;
                    a.rect_n = tn;
                }
            }
        }
        const long nwg = a.xcd_map == 3 ? (nunits * ntiles + 7) / 8 * 8 : nunits * ntiles;
        if (nwg > 0x7FFFFFFFl) {
            DP_SET_ERR(ctx, "dp_clip_accumulate_dense: too many tiles");
            return DP_ERR_SHAPE;
        }
        if (plan.flat) {
            hipLaunchKernelGGL(scale_rows_kernel, dim3((unsigned)runs, dblk, nl), dim3(256), 0, ctx->stream, sb, sqnorms, C, T, K, d_out,
                               (int)rows_per, bias_part, ctx->err_word);
            DP_LAUNCH_CHECK(ctx, "scale_rows");
        }
        b.n_layers = nl;
        for (int l = 0; l < MAX_BATCH; ++l) {
            const int src = l0 + (l < nl ? l : 0);
            b.L[l].A = (const uint16_t*)A[src];
            b.L[l].G = plan.flat ? sb.Gs[l] : (const uint16_t*)G[src];
            b.L[l].out = nsplit == 1 ? sum_W[src] : part + (size_t)(l < nl ? l : 0) * nsplit * d_in * d_out;
            b.L[l].sum_b = sum_b && !plan.flat ? sum_b[src] : nullptr;
        }
        a.bias_part = bias_part;
        {
            dp_prof_scope prof(ctx, DP_PROF_WGEMM, 2.0 * (double)K * d_in * d_out * nl);
            if (one_stage) dma_launch<4, 2, true>(ctx, b, (unsigned)nwg, nsplit > 1);
            else if (plan.bm == 256 && plan.bn == 256) dma_launch<8, 4, false>(ctx, b, (unsigned)nwg, nsplit > 1);
            else if (plan.bm == 256) dma_launch<8, 2, false>(ctx, b, (unsigned)nwg, nsplit > 1);
            else if (plan.bn == 256) dma_launch<4, 4, false>(ctx, b, (unsigned)nwg, nsplit > 1);
            else dma_launch<4, 2, false>(ctx, b, (unsigned)nwg, nsplit > 1);
        }
        DP_LAUNCH_CHECK(ctx, "wgemm_dma");
        const int nb = !any_bias || a.bias_direct ? 0 : plan.flat ? (int)runs : (int)nsplit * a.tiles_m * 2;  // bias partial rows per layer
        if (nsplit > 1 || nb) {
            FinishArgs f;
            for (int l = 0; l < nl; ++l) {
                f.part[l] = reinterpret_cast<const float4*>(b.L[l].out);
                f.out[l] = reinterpret_cast<float4*>(sum_W[l0 + l]);
                f.sum_b[l] = nb ? sum_b[l0 + l] : nullptr;
            }
            const size_t n4 = (size_t)d_in * d_out / 4;  // d_out is a multiple of 8
            const dp_status st = finish_layers(ctx, f, nl, (int)nsplit, n4, bias_part, nb, d_out);
            if (st != DP_OK) return st;
        }
    }
    return DP_OK;
}

dp_status dpk_mfma_ceiling(dp_ctx* ctx, int iters, int launches, double* tflops) {
    int cus = 0;
    DP_HIP_CHECK(ctx, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device));
    if (cus <= 0) cus = 256;
    dp_ws_alloc ws(ctx);
    float* sink = ws.get<float>((size_t)cus * 512);
    if (!sink) {
        DP_SET_ERR(ctx, "workspace too small for the calibration kernel");
        return DP_ERR_WORKSPACE;
    }
    hipEvent_t e0, e1;
    DP_HIP_CHECK(ctx, hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        DP_SET_ERR(ctx, "hipEventCreate failed");
        return DP_ERR_HIP;
    }
    hipLaunchKernelGGL(mfma_ceiling_kernel, dim3(cus), dim3(512), 0, ctx->stream, iters, sink);  // warm-up
    hipError_t e = hipEventRecord(e0, ctx->stream);
    for (int l = 0; l < launches; ++l) hipLaunchKernelGGL(mfma_ceiling_kernel, dim3(cus), dim3(512), 0, ctx->stream, iters, sink);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = hipEventRecord(e1, ctx->stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e != hipSuccess) {
        DP_SET_ERR(ctx, "mfma calibration failed: %s", hipGetErrorString(e));
        return DP_ERR_HIP;
    }
    const double flops = (double)launches * cus * 8.0 * (double)iters * 32.0 * (2.0 * 16 * 16 * 32);
    *tflops = ms > 0.f ? flops / (ms * 1e-3) / 1e12 : 0.0;
    return DP_OK;
}

dp_status dpk_weighted_gemm(dp_ctx* ctx, const void* A, const void* G, dp_dtype dt, int B, int T, int d_in, int d_out,
                            const float* sqnorms, float C, float* sum_W, float* sum_b) {
    return dpk_weighted_gemm_batched(ctx, 1, &A, &G, dt, B, T, d_in, d_out, sqnorms, C, &sum_W, &sum_b);
}

// Tile of the fp32 kernel (in units of 32) and row splits.
struct F32Plan {
    int m32, n32;
    long nsplit;
    bool wide;
};

// The tile and row splits with the smallest modelled time: rounds of the 256 workgroups that run at once, each a tile's microseconds at its ends and its
// nanoseconds a row (of whole pairs of blocks), measured alone and on a full chip; where one round is not filled the rows are split as often as it takes, or half
// as often, if the workspace holds the partial sums, which cost a launch, of 3.8 us, and their bytes.  3 x 3 has the fewest loads to a product (87 % of the matrix rate, 3 x 1 70 %)
// and the longest ends, 144 registers a lane through LDS.  Us, the best of the other tiles, in splits of 1,024 rows and more as they were | 3 x 3: 768 x 768, 8,192 rows 120 | 88 (2,048: 34.5 | 33.8, not taken);
// 768 x 3072, 2,048 rows 100 | 84, 150 rows 25 | 20.6.  Shorter splits: 256 x 256, 2,048 rows 13.4 | 10.7 (2 x 1, eight of 256).
// A tile whose block of rows (of 128, where it has fewer) does not fit a 32-bit buffer resource is no candidate; without any, 2 x 2 with 64-bit addresses.
static F32Plan choose_f32_plan(long K, int d_in, int d_out, size_t ws_bytes) {
    static constexpr struct {
        int m, n;
        double ns_row, us_ends;
    } kTiles[] = {{2, 2, 17.5, 7.0}, {3, 1, 14.0, 5.6}, {2, 1, 10.2, 5.0}, {1, 1, 6.5, 4.6}, {3, 3, 34.6, 12.5}};
    const uint64_t width = d_in > d_out ? d_in : d_out;
    const size_t n = (size_t)d_in * d_out;
    F32Plan plan{0, 0, 1, false};
    double best = 0.0;
    for (const auto& t : kTiles) {
        const long a = (d_in + 32l * t.m - 1) / (32 * t.m), b = (d_out + 32l * t.n - 1) / (32 * t.n), pair = 2 * f32_block(t.m, t.n);
        const bool wide = (uint64_t)(pair < 256 ? 128 : pair / 2) * 4u * width > 0xFFFFFFFFu;
        long most = 256 / (a * b);
        if (most > K / 128) most = K / 128;
        for (int k = 0; k < 3; ++k) {
            const long ns = k == 0 ? 1 : k == 1 ? most : most / 2;
            if (k > 0 && (ns < 2 || (size_t)ns * (n + d_out) * sizeof(float) + 1024 > ws_bytes)) continue;
            const long rows = ((K + ns - 1) / ns + pair - 1) / pair * pair;
            const double us = (double)((a * b * ns + 255) / 256) * ((double)rows * t.ns_row * 1e-3 + t.us_ends) + (ns > 1 ? 3.8 + (double)(ns + 2) * n * 4.0 / 8e6 : 0.0);
            if (plan.m32 && (us >= best || a > 65535 || wide)) continue;  // (a launch has at most 65,535 tile rows)
            best = us;
            plan = F32Plan{t.m, t.n, ns, wide};
        }
    }
    return plan;
}

// A layer in fp32, or one without weights.
static dp_status weighted_sum_single(dp_ctx* ctx, const void* A, const void* G, dp_dtype dt, int B, int T, int d_in, int d_out,
                                     const float* sqnorms, float C, float* sum_W, float* sum_b) {
    if (dt != DP_F32 && !sum_b) return DP_OK;
    if (d_in == 0) {
        if (!sum_b) return dpk_clip_factors(ctx, sqnorms, B, C, ctx->cbuf);  // (nothing to add; a norm that is no number is still reported)
        return dpk_colstat_sums(ctx, nullptr, G, dt, B, T, d_out, sqnorms, C, nullptr, sum_b);
    }
    const bool own = B <= F32_FACTORS;
    dp_status st = own ? DP_OK : dpk_clip_factors(ctx, sqnorms, B, C, ctx->cbuf);
    if (st != DP_OK) return st;
    // (fp32 from here)
    const long K = (long)B * T;
    const F32Plan plan = choose_f32_plan(K, d_in, d_out, ctx->ws_bytes);
    long nsplit = plan.nsplit;
    float *part = nullptr, *bpart = nullptr;
    if (nsplit > 1) {
        dp_ws_alloc ws(ctx);
        part = ws.get<float>((size_t)nsplit * d_in * d_out);
        bpart = ws.get<float>((size_t)nsplit * d_out);
    }
    if (!part || !bpart) nsplit = 1;
    const long rows = ((K + nsplit - 1) / nsplit + 1) / 2 * 2;
    nsplit = (K + rows - 1) / rows;
    const dim3 grid((unsigned)((d_out + 32 * plan.n32 - 1) / (32 * plan.n32)), (unsigned)((d_in + 32 * plan.m32 - 1) / (32 * plan.m32)),
                    (unsigned)nsplit);
    const dim3 block(64 * F32_WAVES);
    const int add = nsplit == 1 ? 1 : 0;
    float* o = add ? sum_W : part;
    float* ob = !sum_b ? nullptr : add ? sum_b : bpart;
    auto launch = [&](auto m_tag, auto n_tag, auto wide_tag) {
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, 0, ctx->stream, (const float*)A, (const float*)G, own ? sqnorms : ctx->cbuf, C, T, K, d_in,
                               d_out, rows, add, o, ob, ctx->err_word);
        };
        constexpr int M = decltype(m_tag)::value, N = decltype(n_tag)::value;
        constexpr bool W = decltype(wide_tag)::value;
        if (own) go(wgemm_f32_kernel<M, N, true, W>);
        else go(wgemm_f32_kernel<M, N, false, W>);
    };
    using one = std::integral_constant<int, 1>;
    using two = std::integral_constant<int, 2>;
    using three = std::integral_constant<int, 3>;
    if (plan.wide) launch(two{}, two{}, std::true_type{});
    else if (plan.m32 == 2 && plan.n32 == 2) launch(two{}, two{}, std::false_type{});
    else if (plan.m32 == 3 && plan.n32 == 3) launch(three{}, three{}, std::false_type{});
    else if (plan.m32 == 3) launch(three{}, one{}, std::false_type{});
    else if (plan.m32 == 2) launch(two{}, one{}, std::false_type{});
    else launch(one{}, one{}, std::false_type{});
    DP_LAUNCH_CHECK(ctx, "wgemm_f32");
    if (add) return DP_OK;
    const size_t n = (size_t)d_in * d_out;
    if (n % 4 == 0 && (((uintptr_t)part | (uintptr_t)sum_W) & 15) == 0) {
        FinishArgs f;
        f.part[0] = reinterpret_cast<const float4*>(part);
        f.out[0] = reinterpret_cast<float4*>(sum_W);
        f.sum_b[0] = sum_b;
        return finish_layers(ctx, f, 1, (int)nsplit, n / 4, bpart, sum_b ? (int)nsplit : 0, d_out);
    }
    st = dpk_reduce_partials(ctx, part, (int)nsplit, n, n, sum_W);
    if (st == DP_OK && sum_b) st = dpk_reduce_partials(ctx, bpart, (int)nsplit, (size_t)d_out, (size_t)d_out, sum_b);
    return st;
}

// What dpk_weighted_gemm_batched does with these sizes, for its tests: tile rows and columns, flat, layers a launch, row splits of a
// full launch (the workspace may hold fewer), rows that one 32-bit buffer resource covers (0: 64-bit addresses).
dp_status dpk_dense_sum_plan(dp_dtype dt, int n, int B, int T, int d_in, int d_out, size_t ws_bytes, int32_t* out) {
    const long K = (long)B * T;
    if (dt == DP_F32) {
        const F32Plan p = choose_f32_plan(K, d_in, d_out, ws_bytes);
        out[0] = 32 * p.m32;
        out[1] = 32 * p.n32;
        out[2] = 0;
        out[3] = 1;
        out[4] = (int32_t)p.nsplit;
        out[5] = p.wide ? 0 : f32_block(p.m32, p.n32);
        return DP_OK;
    }
    const DmaPlan p = choose_dma_plan(n, B, T, d_in, d_out, ws_bytes);
    out[0] = p.bm;
    out[1] = p.bn;
    out[2] = p.flat ? 1 : 0;
    out[3] = n < p.per_launch ? n : p.per_launch;
    out[4] = (int32_t)p.nsplit;
    out[5] = BK;
    return DP_OK;
}

// The tile of n layers' norms by materialisation, and the modelled time of their launch: the stage costs above (a workgroup without a sum to
// add to takes about 3 us besides its stages).
static double materialise_tile(int n, int B, int T, int d_in, int d_out, int* bm, int* bn) {
    double best_t = 0.0;
    *bm = *bn = 0;
    for (int m = 256; m >= 128; m -= 128)
        for (int k = 256; k >= 128; k -= 128) {
            const long wgs = (long)n * B * ((d_in + m - 1) / m) * ((d_out + k - 1) / k);
            const DmaCost c = dma_cost(m, k, false);
            const double t = (double)((wgs + 256 * c.wgs - 1) / (256 * c.wgs)) * ((T + BK - 1) / BK * (wgs <= 256 ? c.t_stage_alone : c.t_stage) + 3.0);
            if (!*bm || t < best_t) {
                *bm = m;
                *bn = k;
                best_t = t;
            }
        }
    return best_t;
}

// Whether bf16 norms that take fewer operations from Gram matrices are there sooner by materialisation: with few examples the Gram kernels run one workgroup to an
// example (and unit), a chain of chunks of 64 columns on a chip that is mostly idle, while the gradient's tiles fill it.  Microseconds a chunk, measured:
// 0.68 above 128 rows, 0.41 (chunks of 128 columns in pairs) and 0.54 from 65, 0.15 and 0.22 from 33; shorter examples split their chunks over waves.
// Of 205 shapes 23 change by it; us, Gram | materialised: B = 3, T = 98, 1024 x 4096 38 | 11; B = 17, T = 80, 3664 x 296 40 | 16; three layers of 896 x 3584, B = 3,
// T = 164 53 | 21; B = 9, T = 330, 1920 x 640 34 | 16; B = 32, T = 64, 27168 x 256 100 | 78.  The entries of a materialised gradient are squared and added: no cancellation,
// the error is no larger.
bool dpk_materialise_sooner(const dp_ctx* ctx, int n, int B, int T, int d_in, int d_out) {
    uint32_t words[70];
    int units = 1, bm, bn;
    if (T <= 32 || n > MAX_BATCH || !dp_sum_width_ok(DP_BF16, d_in, d_out)) return false;
    if (T > 128 && dpk_gram_unit_plan(T, words, 70, &units) != DP_OK) return false;
    if ((long)n * B * units > 256) return false;
    const bool wide = d_in % 128 == 0 && d_out % 128 == 0;
    const double chunk = T > 128 ? 0.68 : T > 64 ? (wide ? 0.41 : 0.54) : (wide ? 0.15 : 0.22);
    const double gram = 4.0 + chunk * ((d_in + 63) / 64 + (d_out + 63) / 64), sooner = 4.0 + materialise_tile(n, B, T, d_in, d_out, &bm, &bn);
    if ((size_t)B * n * ((d_in + bm - 1) / bm) * ((d_out + bn - 1) / bn) * sizeof(float) > ctx->ws_bytes) return false;
    return sooner < 0.85 * gram;
}

// Norms by materialisation: a unit of the kernel is one example, its tiles of A_i^T G_i are squared and summed as they leave the
// accumulators; partial norms [B][layers * tiles] through the workspace.
dp_status dpk_materialise_sqnorms_batched(dp_ctx* ctx, int n, const void* const* A, const void* const* G, dp_dtype dt, int B, int T,
                                          int d_in, int d_out, int has_bias, float* sqnorms) {
    dp_status st = DP_OK;
    if (dt == DP_F32) {
        for (int l = 0; st == DP_OK && l < n; ++l)
            st = dpk_materialise_f32(ctx, (const float*)A[l], (const float*)G[l], B, T, d_in, d_out, sqnorms);
        if (st == DP_OK && has_bias && n > 0) st = dpk_colstat_sqnorms_batched(ctx, n, nullptr, G, dt, B, T, d_out, 0, 1, sqnorms, nullptr);
    }
    if (!dp_sum_width_ok(dt, d_in, d_out)) {
        DP_SET_ERR(ctx, "dp_sqnorms_dense: a width above %d (bf16, by materialisation)", DP_BF16_MAX_WIDTH);
        return DP_ERR_SHAPE;
    }
    for (int l0 = 0; dt == DP_BF16 && l0 < n;) {
        int nl = n - l0 < MAX_BATCH ? n - l0 : MAX_BATCH, bm = 0, bn = 0;
        float* part = nullptr;
        for (;; nl = (nl + 1) / 2) {  // fewer layers, and at last the largest tile, until the partial norms fit
            materialise_tile(nl, B, T, d_in, d_out, &bm, &bn);
            dp_ws_alloc ws(ctx);
            part = ws.get<float>((size_t)B * nl * ((d_in + bm - 1) / bm) * ((d_out + bn - 1) / bn));
            if (!part && nl == 1) {
                bm = d_in < 256 ? 128 : 256;
                bn = d_out < 256 ? 128 : 256;
                part = ws.get<float>((size_t)B * ((d_in + bm - 1) / bm) * ((d_out + bn - 1) / bn));
            }
            if ((part && (long)nl * B * ((d_in + bm - 1) / bm) * ((d_out + bn - 1) / bn) < 0x7FFFFFF0l) || nl == 1) break;
        }
        WgemmBatchArgs b;
        WgemmArgs& a = b.base;
        a = WgemmArgs{};
        a.err = ctx->err_word;
        a.C = 1.f;
        a.flat = 1;
        a.bias_direct = has_bias ? 1 : 0;
        a.T = T;
        a.d_in = d_in;
        a.d_out = d_out;
        a.K = (long)B * T;
        a.rows_per_split = T;  // one "split" per example
        a.nsplit = B;
        a.tiles_m = (d_in + bm - 1) / bm;
        a.tiles_n = (d_out + bn - 1) / bn;
        a.xcd_map = 3;
        a.rect_m = a.rect_n = 1;
        a.out = part;
        const long ntiles = (long)a.tiles_m * a.tiles_n, nwg = ((long)nl * B * ntiles + 7) / 8 * 8;
        if (!part) {
            DP_SET_ERR(ctx, "workspace too small for %d x %ld materialise partials", B, ntiles);
            return DP_ERR_WORKSPACE;
        }
        if (nwg > 0x7FFFFFFFl) {
            DP_SET_ERR(ctx, "dp_sqnorms_dense: too many tiles");
            return DP_ERR_SHAPE;
        }
        b.n_layers = nl;
        for (int l = 0; l < MAX_BATCH; ++l) {
            const int src = l0 + (l < nl ? l : 0);
            b.L[l] = LayerPtrs{(const uint16_t*)A[src], (const uint16_t*)G[src], nullptr, nullptr};
        }
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)nwg), dim3(512), 0, ctx->stream, b); };
        if (bm == 256 && bn == 256) launch(wgemm_dma16_kernel<8, 4, EPI_SQNORM, false>);
        else if (bm == 256) launch(wgemm_dma16_kernel<8, 2, EPI_SQNORM, false>);
        else if (bn == 256) launch(wgemm_dma16_kernel<4, 4, EPI_SQNORM, false>);
        else launch(wgemm_dma16_kernel<4, 2, EPI_SQNORM, false>);
        DP_LAUNCH_CHECK(ctx, "wgemm_dma (materialise)");
        st = dpk_finish_partials(ctx, part, B, (int)(nl * ntiles), sqnorms);
        if (st != DP_OK) return st;
        l0 += nl;
    }
    return st;
}
