// moe_expert_ffn_sliced: SwiGLU expert FFN over all (slice, expert) row groups of a schedule
// (Section 2.1 "compute"; Section 2.2: per-batch fixed overheads are what fragmenting
// decompositions pay, so all slices are issued by launches whose number does not depend on the
// number of matchings).
//
// Two grouped GEMMs on the bf16 MFMA units:
//   phase 1:  H = silu(X Wg^T) * (X Wu^T)
//   phase 2:  Y = H Wd^T
// A tile holds rows of one expert (of any slices, see FfnArgs).  Both operands are K-contiguous, are copied
// global -> LDS in K slabs (2 to 4 in flight, XOR-swizzled 16-byte chunks) and read back as 16-byte MFMA fragments.
// The weights feed the MFMA "A" port so that each lane ends up with 4 consecutive output columns of one row.
// From the fewest rows per expert to the most (route() chooses): ffn_skinny_kernel streams the weights; ffn_tile_kernel works in tiles of 64, 128 or 256
// rows by 128 columns and splits contractions that would leave the chip idle; ffn_fused_kernel (bf16) runs both phases in one persistent
// launch over tiles of 256 x 256, phase-2 tiles waiting for the rows of H they read (ffn_adaptive_kernel: one launch per phase).
// moe_expert_ffn_backward_sliced (the backward pass: the exchange of Section 2.1 repeated for the gradients) runs the
// adaptive-shape and the tile kernels on other operands, and ffn_bwd_dw_kernel for the weight gradients.
#include "common.hpp"
#include "rows.hpp"
#include "parts.hpp"
#include <type_traits>
#include <algorithm>
#include <cmath>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

constexpr int BN = 256;                // tile columns (phase 1: 128 gate + 128 up)
constexpr int PLAN_THREADS = 1024;
constexpr int MAX_GROUPS = 65536;
constexpr int PLAN_EXPERTS_LDS = 2048; // row bases of the experts kept in LDS by the plan kernel (more: in the workspace)
constexpr int LIST_PAD = 256;          // valid entries behind the last row of the row list (a row block may read past its end)
constexpr int TILE_COUNTERS = 512;     // counters per phase of the parts of split contractions (see ffn_tile_kernel; a split call has fewer tiles)
constexpr int TILE_LAUNCHES = 3;       // launches of such a kernel behind one plan, at most
constexpr int PLAN_HDR = 5;            // plan[0] = (row blocks, 0, 0, 0); plan[1..2] / plan[3..4] = tile queue counters of phase 1 / 2

struct FfnArgs {
    const __bf16* x;                   // [M][d]
    __bf16* h;                         // [M][f]   workspace, in the row order of the plan (see below)
    __bf16* y;                         // [M][d]
    const void *wg, *wu, *wd;          // bf16 or fp8 codes
    const float *sg, *su, *sd;         // block scales (fp8) or null
    int4* plan;                        // plan[0].x = number of row blocks; plan[PLAN_HDR + i] = (row0, row_end, expert, class)
    int M, d, f;
    // Rows are worked on expert by expert, an expert's rows of all slices side by side ("positions" 0 .. M-1): what a
    // row becomes depends on its expert and not on its slice, so a schedule of many small slices costs no more tiles, and
    // reads the weights no more often, than one big slice.  36 833 rows of 4 experts, d = 2048, f = 1408: 228 slices
    // (912 groups of 40 rows on average) 2099 -> 558 us, 10 slices (920 rows) with row map and weights 592 -> 554 us; 61 111
    // rows of 4 experts, d = 7168, f = 2048, 18 slices: 4741 -> 4343 us (before: one tile never spanned two groups).
    const int32_t* list;               // [M + LIST_PAD] or null (identity): position p is row list[p] of x and of y
    const float* gate;                 // [M] or null: the y row of position p is scaled by gate[p]
    int panel1, panel2;                // column groups per panel of the tile walk, phase 1 / phase 2 (see TileGeom)
    int* ready;                        // [row blocks] column units of h complete per row block (fused launch), zeroed by the plan kernel
    // The plain grouped GEMM of the adaptive-shape kernels' "phase 2": out[m][n] = sum_k A[m][k] * B_e[n][k] for the
    // rows m of every row block (expert e), n over NU units of 256 columns.  The forward pass sets A = h, B = w_down,
    // out = y; the backward pass runs it on other operands (see moe_expert_ffn_backward_sliced).
    struct Gemm {
        const __bf16* A; int lda;          // [rows][lda], K contiguous
        const __bf16* B; int ldb;          // B_e = B + e * strideB: [NU * 256][ldb], K contiguous
        long long strideB;
        __bf16* O; int ldo;
        int K, NU;
        unsigned int o_bytes;              // bytes of O when rows are scattered with 32-bit offsets
        int* queues;                       // 8 tile queue counters, zero at launch
    } g2;
    // backward pass, phase 1 with the gradient read-out (EPI == 1): dh in, [dg | du] and h out
    const __bf16* dh; int lddh;            // [M][lddh]
    __bf16* dgu;                           // [M][2 f]: dg in columns 0 .. f-1, du in f .. 2f-1
    int* queues1;                          // 8 tile queue counters of phase 1, zero at launch
};
// row of x that position p reads (phase 1) / row of y it writes (phase 2)
__device__ __forceinline__ int mapped_row(const FfnArgs& a, int p) { return a.list ? a.list[p] : p; }

// ---------------------------------------------------------------------------------- plan kernel
// Orders the rows by expert (see FfnArgs), writes the row list where the order differs from the schedule's, and splits
// every expert's rows into row blocks of bm rows.  Malformed offsets cannot make it write outside its tables: boundaries
// are clamped to [0, M] and to non-decreasing order, positions are saturated sums that never pass M (rows.hpp), and entries
// beyond `cap` are dropped.
// Plan entry = (first position, end of the expert's positions, local expert, shape class of the block: 0 for more than
// 128 rows, else 1).
// The partial last blocks of the experts come first in the table and the full blocks after them: a partial block's
// tiles take longer than a full block's (they read twice the weights per MFMA), and a long tile handed out late is
// what the whole launch then waits for.  (A third class of 64 rows x 1024 columns for blocks of <= 64 rows was
// measured: its tiles take twice as long as any other and made phase 1 of the bench schedule 7 % slower by finishing
// last; it is not in the kernel.)
__device__ __forceinline__ int plan_scan(int v, int tid, int* wave_tot, int& total) {       // exclusive prefix over the workgroup
    const int lane = tid & 63, wave = tid >> 6;
    int incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    __syncthreads();
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int base = 0;
    total = 0;
    for (int w = 0; w < PLAN_THREADS / 64; ++w) {
        if (w < wave) base += wave_tot[w];
        total += wave_tot[w];
    }
    return base + incl - v;
}

// exclusive prefix over the workgroup of row counts 0 .. M each, every sum saturated at M
__device__ __forceinline__ int plan_scan_rows(int rows, int M, int tid, int* wave_tot, int& total) {
    const int lane = tid & 63, wave = tid >> 6;
    int incl = rows;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl = add_rows(incl, o, M);
    }
    int excl = __shfl_up(incl, 1);                       // (a saturated sum less the own count would not be the sum before it)
    if (lane == 0) excl = 0;
    __syncthreads();
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int base = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < PLAN_THREADS / 64; ++w) {
        if (w < wave) base = add_rows(base, wave_tot[w], M);
        total = add_rows(total, wave_tot[w], M);
    }
    return add_rows(base, excl, M);
}

// two prefixes behind one pair of barriers
__device__ __forceinline__ void plan_scan2(int a, int b, int tid, int* wave_a, int* wave_b, int& excl_a, int& excl_b, int& total_a,
                                           int& total_b) {
    const int lane = tid & 63, wave = tid >> 6;
    int ia = a, ib = b;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int oa = __shfl_up(ia, off), ob = __shfl_up(ib, off);
        if (lane >= off) { ia += oa; ib += ob; }
    }
    __syncthreads();
    if (lane == 63) { wave_a[wave] = ia; wave_b[wave] = ib; }
    __syncthreads();
    int base_a = 0, base_b = 0;
    total_a = 0; total_b = 0;
    for (int w = 0; w < PLAN_THREADS / 64; ++w) {
        if (w < wave) { base_a += wave_a[w]; base_b += wave_b[w]; }
        total_a += wave_a[w]; total_b += wave_b[w];
    }
    excl_a = base_a + ia - a;
    excl_b = base_b + ib - b;
}
// The workgroups of the launch share the row list: each scans all groups by itself (a few microseconds, and no hand-over
// between workgroups) and fills its share of the entries; workgroup 0 also writes the table.  Without a list one
// workgroup is launched.
struct PlanArgs {
    const int32_t* offsets;
    int S, e_loc, M, bm, cap;
    int4* plan;
    int* ready;
    const int32_t* row_map;            // [M] or null
    const float* row_gate;             // [M] or null
    int32_t* list;                     // [M + LIST_PAD] or null: not wanted
    float* gate;                       // [M] or null: row_gate in list order
    int* ebase;                        // [e_loc + 1], used when e_loc > PLAN_EXPERTS_LDS
    int* bases;                        // [e_loc + 1] or null: first position of every expert, and the end
};
__global__ __launch_bounds__(PLAN_THREADS)
void ffn_plan_kernel(PlanArgs a) {
    __shared__ int wave_tot[PLAN_THREADS / 64], wave_tot2[PLAN_THREADS / 64];
    __shared__ int g_pos[PLAN_THREADS + 1], g_row[PLAN_THREADS], g_end[PLAN_THREADS];
    __shared__ int eb_lds[PLAN_EXPERTS_LDS + 1];
    const int tid = threadIdx.x;
    const int G = a.S * a.e_loc, M = a.M, bm = a.bm;
    int* const eb = a.e_loc <= PLAN_EXPERTS_LDS ? eb_lds : a.ebase;      // first position of every expert (workgroup 0)
    const bool table = blockIdx.x == 0;
    // ---- the groups in expert-major order: entry i = group (slice i % S, expert i / S).  Listed positions count from 0; without a list
    //      a position is a schedule row, and they begin where the first group does
    int base = a.list ? 0 : first_row(a.offsets, M);
    for (int i0 = 0; i0 < G; i0 += PLAN_THREADS) {
        const int i = i0 + tid, e = i / a.S, s = i - e * a.S;
        int lo = 0, rows = 0;
        if (i < G) rows = group_rows(a.offsets, s * a.e_loc + e, M, lo);
        int total;
        const int excl = plan_scan_rows(rows, M, tid, wave_tot, total);
        const int pos = add_rows(base, excl, M);
        if (table && i < G && s == 0) eb[e] = pos;
        if (a.list) {
            g_pos[tid] = pos; g_row[tid] = lo;
            if (tid == 0) g_pos[PLAN_THREADS] = add_rows(base, total, M);
            __syncthreads();
            const int last = g_pos[PLAN_THREADS];
            for (int p = g_pos[0] + (int)blockIdx.x * PLAN_THREADS + tid; p < last; p += (int)gridDim.x * PLAN_THREADS) {
                int t = 0;                                                // the last entry that starts at or before p
#pragma unroll
                for (int step = PLAN_THREADS / 2; step > 0; step >>= 1)
                    if (g_pos[t + step] <= p) t += step;
                const int m = g_row[t] + (p - g_pos[t]);
                int row = m;
                if (a.row_map) { row = a.row_map[m]; row = (unsigned)row < (unsigned)M ? row : 0; }
                a.list[p] = row;
                if (a.gate) a.gate[p] = a.row_gate[m];
            }
            __syncthreads();                                              // the next pass overwrites the entries
        }
        base = add_rows(base, total, M);
    }
    if (!table) return;
    const int used = base;
    if (tid == 0) eb[a.e_loc] = used;
    if (a.list && tid < LIST_PAD) a.list[used + tid] = 0;                 // (used <= M: inside the list)
    __threadfence_block();
    __syncthreads();
    if (a.bases)
        for (int e = tid; e <= a.e_loc; e += PLAN_THREADS) a.bases[e] = eb[e];
    // ---- number of partial blocks (experts whose row count is not a multiple of bm); with at most one expert per thread
    //      the scan of the table pass below yields it
    int n_partial = 0;
    if (a.e_loc > PLAN_THREADS) {
        int partial = 0;
        for (int e = tid; e < a.e_loc; e += PLAN_THREADS) partial += (eb[e + 1] - eb[e]) % bm != 0;
        plan_scan(partial, tid, wave_tot, n_partial);
    }
    // ---- table: partial blocks in expert order, then the full blocks in expert order
    int run_partial = 0, run_full = n_partial;                        // (uniform: every thread adds the same totals)
    for (int e0 = 0; e0 < a.e_loc; e0 += PLAN_THREADS) {
        const int e = e0 + tid;
        const int lo = e < a.e_loc ? eb[e] : 0, hi = e < a.e_loc ? eb[e + 1] : 0;
        const int rows = hi - lo, nfull = rows / bm, has_partial = rows % bm != 0;
        int ex_partial, ex_full, tot_partial, tot_full;
        plan_scan2(has_partial, nfull, tid, wave_tot, wave_tot2, ex_partial, ex_full, tot_partial, tot_full);
        if (a.e_loc <= PLAN_THREADS) run_full = tot_partial;          // the only pass: all partial blocks are known now
        const int at_partial = run_partial + ex_partial;
        run_partial += tot_partial;
        const int at_full0 = run_full, at_full = run_full + ex_full;
        run_full += tot_full;
        g_pos[tid] = at_full; g_row[tid] = lo; g_end[tid] = hi;
        __syncthreads();
        for (int at = at_full0 + tid; at < run_full; at += PLAN_THREADS) {
            int t = 0;                                                    // the last expert whose full blocks start at or before `at`
#pragma unroll
            for (int step = PLAN_THREADS / 2; step > 0; step >>= 1)
                if (g_pos[t + step] <= at) t += step;
            if (at < a.cap) a.plan[PLAN_HDR + at] = make_int4(g_row[t] + (at - g_pos[t]) * bm, g_end[t], e0 + t, bm > 128 ? 0 : 1);
        }
        __syncthreads();
        if (has_partial && at_partial < a.cap) {
            const int row = lo + nfull * bm;
            a.plan[PLAN_HDR + at_partial] = make_int4(row, hi, e, hi - row > 128 ? 0 : 1);
        }
    }
    // per row block: column units of h complete (fused kernel); per tile of a split contraction: parts that are done (tile kernel)
    for (int i = tid; i < min(max(run_full, TILE_LAUNCHES * TILE_COUNTERS), a.cap); i += PLAN_THREADS) a.ready[i] = 0;
    if (tid == 0) a.plan[0] = make_int4(min(run_full, a.cap), 0, 0, 0);
    if (tid >= 1 && tid < PLAN_HDR) a.plan[tid] = make_int4(0, 0, 0, 0);    // tile queue counters
}

// The same plan for a call with few groups and rows: a group per thread, one scan and two barriers instead of loops around ten.  4 experts, 1024
// rows in 6 slices: 6.6 -> 4.6 us (with the events around the launch); a call of that size takes 42.  (At most 33 experts and blocks of 64
// rows, i.e. 2111 rows: the list is filled in three passes at most, and one wavefront's first threads write the table.)
constexpr int SMALL_PLAN_BLOCKS = 33;
bool small_plan(int M, int S, int e_loc) { return (long long)S * e_loc <= PLAN_THREADS && M / 64 + e_loc <= SMALL_PLAN_BLOCKS; }
__global__ __launch_bounds__(PLAN_THREADS)
void ffn_small_plan_kernel(PlanArgs a) {
    __shared__ int wave_tot[PLAN_THREADS / 64];
    __shared__ int g_pos[PLAN_THREADS + 1], g_row[PLAN_THREADS], eb[SMALL_PLAN_BLOCKS + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, M = a.M, bm = a.bm;
    const int e = tid / a.S, s = tid - e * a.S;
    int lo = 0, rows = 0;
    if (e < a.e_loc) rows = group_rows(a.offsets, s * a.e_loc + e, M, lo);
    const int start = a.list ? 0 : first_row(a.offsets, M);
    for (int i = tid; i < TILE_LAUNCHES * TILE_COUNTERS && i < a.cap; i += PLAN_THREADS) a.ready[i] = 0;
    int incl = rows;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl = add_rows(incl, o, M);
    }
    int pos = __shfl_up(incl, 1);
    if (lane == 0) pos = 0;
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int base = start, used = start;
#pragma unroll
    for (int w = 0; w < PLAN_THREADS / 64; ++w) {
        if (w < wave) base = add_rows(base, wave_tot[w], M);
        used = add_rows(used, wave_tot[w], M);
    }
    pos = add_rows(base, pos, M);
    g_pos[tid] = pos; g_row[tid] = lo;
    if (e < a.e_loc && s == 0) eb[e] = pos;
    if (tid == 0) { eb[a.e_loc] = used; g_pos[PLAN_THREADS] = used; }
    __syncthreads();
    if (a.list) {
        for (int p = tid; p < used; p += PLAN_THREADS) {
            int t = 0;                                                    // the last group that starts at or before p
#pragma unroll
            for (int step = PLAN_THREADS / 2; step > 0; step >>= 1)
                if (g_pos[t + step] <= p) t += step;
            const int m = g_row[t] + (p - g_pos[t]);
            int row = m;
            if (a.row_map) { row = a.row_map[m]; row = (unsigned)row < (unsigned)M ? row : 0; }
            a.list[p] = row;
            if (a.gate) a.gate[p] = a.row_gate[m];
        }
        if (tid < LIST_PAD) a.list[used + tid] = 0;
    }
    // partial blocks in expert order, then the full blocks in expert order
    if (tid <= a.e_loc) {
        int partials = 0, partial_at = 0, full_at = 0, fulls = 0;
        for (int j = 0; j < a.e_loc; ++j) {
            const int n = eb[j + 1] - eb[j];
            partial_at += j < tid && n % bm != 0;
            partials += n % bm != 0;
            full_at += j < tid ? n / bm : 0;
            fulls += n / bm;
        }
        if (tid < a.e_loc) {
            const int first = eb[tid], end = eb[tid + 1], nfull = (end - first) / bm;
            for (int i = 0; i < nfull; ++i)
                if (partials + full_at + i < a.cap) a.plan[PLAN_HDR + partials + full_at + i] = make_int4(first + i * bm, end, tid, bm > 128 ? 0 : 1);
            if (first + nfull * bm < end && partial_at < a.cap)
                a.plan[PLAN_HDR + partial_at] = make_int4(first + nfull * bm, end, tid, end - first - nfull * bm > 128 ? 0 : 1);
        } else {
            a.plan[0] = make_int4(min(partials + fulls, a.cap), 0, 0, 0);
        }
    }
    if (tid >= 1 && tid < PLAN_HDR) a.plan[tid] = make_int4(0, 0, 0, 0);
}

// ---------------------------------------------------------------------------------- helpers
// g * sigmoid(g) with the hardware reciprocal (1 ulp) instead of an IEEE division: the result is rounded to bf16 anyway,
// and the division's dozen instructions per value were a visible part of a tile's read-out
__device__ __forceinline__ float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

__device__ __forceinline__ u32x2 pack4(float a, float b, float c, float d) {
    bf16x4 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
    return __builtin_bit_cast(u32x2, v);
}

// 8 consecutive OCP FP8 E4M3 codes (8 bytes; bias 7, subnormals at exponent field 0, no infinities, S.1111.111 = NaN)
// times one scale -> 8 bf16.  gfx950 decodes two codes per v_cvt_pk_f32_fp8.
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x4 dequant8(u32x2 codes, float scale) {
    const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8((int)codes.x, false), b = __builtin_amdgcn_cvt_pk_f32_fp8((int)codes.x, true);
    const f32x2 c = __builtin_amdgcn_cvt_pk_f32_fp8((int)codes.y, false), d = __builtin_amdgcn_cvt_pk_f32_fp8((int)codes.y, true);
    bf16x8 o = {(__bf16)(a.x * scale), (__bf16)(a.y * scale), (__bf16)(b.x * scale), (__bf16)(b.y * scale),
                (__bf16)(c.x * scale), (__bf16)(c.y * scale), (__bf16)(d.x * scale), (__bf16)(d.y * scale)};
    return __builtin_bit_cast(u32x4, o);
}

// half of 16 consecutive codes -> 8 bf16, without their block's scale but times CODE_UNIT: every E4M3 value is a bf16 value, and 128 products of the
// largest ones with any finite x stay finite in fp32 (with the codes as they are sums overflowed from |x| = 6e33 on, whatever the scale).  The scale that multiplies
// a sum is divided by it, a power of two: no bit of a result changes.
constexpr float CODE_UNIT = 0x1p-16f;
__device__ __forceinline__ bf16x8 widen8(u32x4 codes, int half) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    const unsigned int lo = half ? codes.z : codes.x, hi = half ? codes.w : codes.y;
    const bf16x2 v0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, CODE_UNIT, false), v1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, CODE_UNIT, true);
    const bf16x2 v2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, CODE_UNIT, false), v3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, CODE_UNIT, true);
    return bf16x8{v0.x, v0.y, v1.x, v1.y, v2.x, v2.y, v3.x, v3.y};
}

// ---------------------------------------------------------------------------------- persistent tiles
// Tiles are handed out by eight atomic queues, one per XCD (workgroup id modulo 8), each
// walking its own chunks of neighbouring tiles so that the workgroups sharing an L2 also share
// operand slabs; a workgroup whose queue runs dry takes from the others.

struct TileGeom {                      // how tiles are grouped into chunks, and the order in which the chunks are walked
    int nblocks, NT, NCG, CN, RB, NRG, W, nchunks;
    __device__ __forceinline__ void init(int nblocks_, int NT_, int panel) {
        nblocks = nblocks_; NT = NT_;
        NCG = (NT + 7) / 8;                        // column groups of at most 8 (11 -> 2 x 6)
        CN = (NT + NCG - 1) / NCG;
        RB = 32 / CN < 1 ? 1 : 32 / CN;            // about 32 tiles per chunk
        NRG = (nblocks + RB - 1) / RB;             // row groups
        W = panel < 1 ? 1 : (panel > NCG ? NCG : panel);      // column groups per panel
        nchunks = NRG * NCG;
    }
    // ticket k of queue x -> tile; returns 1 = valid, 0 = hole in the padded grid, -1 = queue exhausted.
    // Chunks are walked panel by panel: inside a panel of W column groups the row groups are the outer loop, so the
    // panel's weights are touched again after one row group's worth of other traffic and stay in the memory-side cache
    // while the activations stream past; W = NCG (one panel) when an expert's weights are small.
    __device__ __forceinline__ int decode(int x, int k, int& blk, int& nt) const {
        const int chs = RB * CN;
        const int c = (k / chs) * 8 + x, j = k % chs;
        if (c >= nchunks) return -1;
        const int full = (NCG / W) * W;            // column groups inside whole panels
        const int c0 = NRG * full;
        int rg, cg;
        if (c < c0) {
            const int per = NRG * W, p = c / per, rem = c - p * per;
            rg = rem / W; cg = p * W + rem - rg * W;
        } else {
            const int wl = NCG - full, rem = c - c0;
            rg = rem / wl; cg = full + rem - rg * wl;
        }
        blk = rg * RB + j / CN;
        nt = cg * CN + j % CN;
        return (blk < nblocks && nt < NT) ? 1 : 0;
    }
};

template <int N> __device__ __forceinline__ void wait_vmcnt();
#define MOE_WAIT_VMCNT(n) template <> __device__ __forceinline__ void wait_vmcnt<n>() { asm volatile("s_waitcnt vmcnt(" #n ")" ::: "memory"); }
MOE_WAIT_VMCNT(0) MOE_WAIT_VMCNT(1) MOE_WAIT_VMCNT(2) MOE_WAIT_VMCNT(3) MOE_WAIT_VMCNT(4) MOE_WAIT_VMCNT(5) MOE_WAIT_VMCNT(6) MOE_WAIT_VMCNT(7) 
MOE_WAIT_VMCNT(8) MOE_WAIT_VMCNT(9) MOE_WAIT_VMCNT(10) MOE_WAIT_VMCNT(11) MOE_WAIT_VMCNT(12) MOE_WAIT_VMCNT(13) MOE_WAIT_VMCNT(14) MOE_WAIT_VMCNT(15) 
MOE_WAIT_VMCNT(16) MOE_WAIT_VMCNT(17) MOE_WAIT_VMCNT(18) MOE_WAIT_VMCNT(19) MOE_WAIT_VMCNT(20) MOE_WAIT_VMCNT(21) MOE_WAIT_VMCNT(22) MOE_WAIT_VMCNT(23) 
MOE_WAIT_VMCNT(24) MOE_WAIT_VMCNT(25) MOE_WAIT_VMCNT(26) MOE_WAIT_VMCNT(27) MOE_WAIT_VMCNT(28) MOE_WAIT_VMCNT(29) MOE_WAIT_VMCNT(30) MOE_WAIT_VMCNT(31) 
MOE_WAIT_VMCNT(32) MOE_WAIT_VMCNT(33) MOE_WAIT_VMCNT(34) MOE_WAIT_VMCNT(35) MOE_WAIT_VMCNT(36) MOE_WAIT_VMCNT(37) MOE_WAIT_VMCNT(38) MOE_WAIT_VMCNT(39) 
MOE_WAIT_VMCNT(40) MOE_WAIT_VMCNT(41) MOE_WAIT_VMCNT(42) MOE_WAIT_VMCNT(43) MOE_WAIT_VMCNT(44) MOE_WAIT_VMCNT(45) MOE_WAIT_VMCNT(46) MOE_WAIT_VMCNT(47) 
MOE_WAIT_VMCNT(48) MOE_WAIT_VMCNT(49) MOE_WAIT_VMCNT(50) MOE_WAIT_VMCNT(51) MOE_WAIT_VMCNT(52) MOE_WAIT_VMCNT(53) MOE_WAIT_VMCNT(54) MOE_WAIT_VMCNT(55) 
MOE_WAIT_VMCNT(56) MOE_WAIT_VMCNT(57) MOE_WAIT_VMCNT(58) MOE_WAIT_VMCNT(59) MOE_WAIT_VMCNT(60) MOE_WAIT_VMCNT(61) MOE_WAIT_VMCNT(62) MOE_WAIT_VMCNT(63) 
#undef MOE_WAIT_VMCNT

// Workgroup barrier that orders LDS traffic only.  (__syncthreads() also drains every outstanding global
// access, which would serialise the slab copies that are meant to stay in flight across K steps.)
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---------------------------------------------------------------------------------- adaptive-shape GEMM kernel (bf16)
// Eight wavefronts of 64 x 128 each, K slabs copied global -> LDS as they lie.  The arrangement of the wavefronts is chosen
// per row block so that ragged slices do not pay for 256 rows they do not have:
//   class 0: 4 x 2 wavefronts = 256 rows x 256 columns;  64-wide K slabs (128-byte rows) of 64 KiB, two in LDS
//   class 1: 2 x 4            = 128 rows x 512 columns;  32-wide K slabs (64-byte rows) of 40 KiB, three in LDS
// Both classes run the same number of MFMAs per tile.  (A 1 x 8 arrangement of 64 rows x 1024 columns was measured
// too: its tiles read four times the weights per row and take twice as long as the others -- see the plan kernel.)
// Columns come in units (phase 1: 128 hidden units = 128 gate + 128 up rows; phase 2: 256 rows of w_down); a tile of
// class c covers 1 / 2 consecutive units.  A unit past the end is fetched as the last valid one and not stored.
// The 256-row class, which does most of the work, has 128-byte slab rows so that every copy fetches whole cache
// lines: a 64-byte row is half a line whose other half is requested again by the next slab, which doubles the
// requests to the L2 and the fill traffic into the L1 and keeps the address FIFO of the memory pipeline full (and
// the MFMAs queued behind a copy waiting) for a fifth of the time.
// The barrier at the end of slab s publishes slab s + 1 and frees the buffer of slab s; the copies of slab s + NSS
// go out from there on, spaced between the MFMAs (slot 0 = rest of slab s, slot i = K step i - 1 of slab s + 1).
constexpr int NW = 8;                                         // wavefronts per workgroup
template <int CLS> struct Cls {
    static_assert(CLS == 0 || CLS == 1, "two shape classes");
    static constexpr int WMW = (CLS == 0 ? 4 : 2) * NW / 8, WNW = NW / WMW;
    static constexpr int MB = 16 / NW, NQ = 4;                                    // 32-row / 32-column blocks per wavefront
    static constexpr int BMc = 32 * MB * WMW, BNc = 32 * NQ * WNW;
    static constexpr int U = BNc / 256;                                     // column units per tile
    static constexpr int ROWB = CLS == 0 ? 128 : 64;                        // bytes per slab row
    static constexpr int SUB = ROWB / 32;                                   // MFMA K steps (of 16) per slab
    static constexpr int RPC = NW * 1024 / ROWB;                                 // slab rows one copy of the workgroup deposits
    static constexpr int A_BYTES = BMc * ROWB, B_BYTES = BNc * ROWB, SLAB = A_BYTES + B_BYTES;
    static constexpr int NSS = CLS == 1 ? 3 : 2;                            // slabs resident in LDS
    static constexpr int CA = BMc / RPC, CB = BNc / RPC, NCOPY = CA + CB;   // copies per wavefront and slab
    // copies per slot (slot 0, 1, 2; none later)
    static constexpr int S0 = (CLS == 0 ? 4 : 3) * 8 / NW, S1 = NCOPY - S0, S2 = 0;
    static_assert(S0 + S1 + S2 == NCOPY && (S2 == 0 || SUB > 2) && (S1 == 0 || SUB > 1), "the slots hold every copy and end before the next slab's last K step");
};
constexpr int STAGE_OFF = 131072;                             // slab buffers below (2 x 64 KiB >= 3 x 40 KiB), output staging above
constexpr int STAGE_WAVE = 4096;                              // staging per wavefront: 32 rows x 128 bytes
constexpr int ADAPTIVE_LDS = STAGE_OFF + NW * STAGE_WAVE;      // 160 KiB: all of a compute unit's LDS

// AROWS / OROWS say how the rows of the A operand / of the output behind a tile's positions are addressed (the forward
// pass lists x in phase 1 and y in phase 2; h lies in position order).
//   ROWS_PLAIN   they are consecutive: one buffer descriptor per tile (64-bit base at the tile's first row) plus 32-bit
//                offsets inside the tile, whatever the size of the operand
//   ROWS_LIST32  they are listed and the matrix is smaller than 4 GiB: one descriptor for the whole operand and 32-bit offsets.
//                A wavefront's copy or store instruction covers 8 (16) consecutive list entries, which it fetches with
//                scalar loads: nothing is added to the vector memory operations in flight, whose number the waits count
//   ROWS_LIST64  they are listed and lie anywhere: every thread carries the 64-bit addresses of its rows
// FUSED (both phases in one launch, see ffn_fused_kernel): a phase-1 tile, once its rows of h are stored, adds the
// column units it covered to the ready counter of its row block; a phase-2 ticket is handed to the workgroup only when
// the counter of its row block has reached the number of column units of h.  The hidden activations cross from one
// workgroup to another inside the launch, possibly from one die's L2 to another's: their stores (phase 1) and their
// loads (phase 2) are issued at device scope (the sc1 bit of the instruction: the store is written through to where
// every die sees it before it counts as complete, the load does not take a copy that is private to its die), and the
// counters are device-scope atomics; a writer signals after all its stores have completed (vmcnt(0) in every wavefront,
// then a barrier), a reader issues its loads after it has seen the count.
constexpr int DEVICE_SCOPE = 16;       // cache-policy bit sc1 of a buffer instruction
// EPI (phase 1): 0 = h = silu(g) * u is stored; 1 = the backward pass: with dh read from memory, dg = dh * u * silu'(g) and
// du = dh * silu(g) are stored side by side and h beside them.
enum { ROWS_PLAIN = 0, ROWS_LIST32 = 1, ROWS_LIST64 = 2 };
template <int PHASE, int AROWS, int OROWS, bool FUSED, int EPI = 0>
__device__ __forceinline__ void ffn_adaptive_body(const FfnArgs& a, unsigned char* smem) {
    constexpr bool GATHER = AROWS == ROWS_LIST64;
    static_assert(PHASE == 2 || OROWS == ROWS_PLAIN, "phase 1 stores in position order");
    static_assert(EPI == 0 || (PHASE == 1 && !FUSED), "the gradient read-out belongs to phase 1 of a launch of its own");
    // next tile: (block, tile index, class, first row, end row, expert); block -1 = none.  It shares its bytes with
    // wavefront 0's output staging: written by that wavefront after its read-out, read by the others before the
    // next read-out begins (inside the slab loop, or ahead of a barrier).
    int* const s_ticket = reinterpret_cast<int*>(smem + STAGE_OFF);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, lhi = lane >> 5;
    const int K = PHASE == 1 ? a.d : a.g2.K;
    const int NU = PHASE == 1 ? a.f / 128 : a.g2.NU;            // column units
    const int lda = PHASE == 1 ? a.d : a.g2.lda, ldb = PHASE == 1 ? a.d : a.g2.ldb;      // row pitch of the operands, elements
    TileGeom geom;
    geom.init(a.plan[0].x, NU, PHASE == 1 ? a.panel1 : a.panel2);
    int* queues = PHASE == 1 ? a.queues1 : a.g2.queues;
    const int my_xcd = blockIdx.x & 7;

    // Slab layout: row-major, 16-byte chunk c of row r sits at position c ^ swz(r); swz(r) = (r >> 2) & 3 for 64-byte
    // rows and (r >> 1) & 7 for 128-byte rows (16 consecutive rows of a fragment read then cover all 64 banks).
    // One copy instruction of the workgroup deposits 8 KiB = RPC whole rows: thread t writes position t % (ROWB / 16)
    // of row t / (ROWB / 16), so it fetches the chunk that belongs there.
    const int row0_64 = tid >> 2, row0_128 = tid >> 3;
    const int kcg_64 = (tid & 3) ^ ((row0_64 >> 2) & 3), kcg_128 = (tid & 7) ^ ((row0_128 >> 1) & 7);
    const int wave_bytes = wave * 1024;
    int frag_off64[2], frag_off128[4];
#pragma unroll
    for (int u = 0; u < 2; ++u) frag_off64[u] = l31 * 64 + ((((u << 1) | lhi) ^ ((l31 >> 2) & 3)) << 4);
#pragma unroll
    for (int u = 0; u < 4; ++u) frag_off128[u] = l31 * 128 + ((((u << 1) | lhi) ^ ((l31 >> 1) & 7)) << 4);

    // thread 0 pulls tickets (own queue first, then the others).  A ticket names (block, unit); it is a tile only if
    // the unit is the first of the tile its block's class makes of it.
    auto fetch = [&](int first_k) __attribute__((always_inline)) {
        int q = my_xcd, blk = -1, unit = -1, cls = 0;
        int4 info = make_int4(0, 0, 0, 0);
        // 1 = a tile, 0 = no tile behind this ticket, -1 = queue exhausted
        auto look = [&](int k) __attribute__((always_inline)) -> int {
            const int st = geom.decode(q, k, blk, unit);
            if (st != 1) { blk = -1; return st; }
            // (a scalar load: the plan is read-only here, and a vector load's return would be counted behind the
            //  slab copies in flight)
            const __attribute__((address_space(4))) int* entry =
                (const __attribute__((address_space(4))) int*)a.plan + 4 * (PLAN_HDR + __builtin_amdgcn_readfirstlane(blk));
            info = make_int4(entry[0], entry[1], entry[2], entry[3]);
            cls = info.w;
            if ((unit & ((1 << cls) - 1)) == 0) return 1;
            blk = -1;
            return 0;
        };
        // the first look stands outside the loop: the wait for first_k then counts the copies issued since
        int st = look(first_k);
        for (int tries = 0; st != 1;) {
            if (st < 0) { if (++tries == 8) break; q = (q + 1) & 7; }
            st = look(atomicAdd(&queues[q], 1));
        }
        if (FUSED && PHASE == 2 && blk >= 0) {
            // The rows of h this tile reads are complete when every phase-1 tile of the row block has signalled.  Phase-1
            // tickets are all taken before the first phase-2 ticket, and a workgroup that holds a phase-1 ticket never
            // waits, so the wait ends; the bound on it only turns a defect into a flagged wrong result instead of a hang.
            const int need = a.f / 128;
            for (int spins = 0; __hip_atomic_load(&a.ready[blk], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need; ++spins) {
                __builtin_amdgcn_s_sleep(32);                                           // about 2048 cycles
                if (spins > (1 << 20)) { atomicOr((int*)&a.plan[0].y, 1); break; }      // seconds: a defect, flagged in the plan header
            }
        }
        s_ticket[0] = blk; s_ticket[1] = blk >= 0 ? (unit >> cls) : 0; s_ticket[2] = cls;
        s_ticket[3] = info.x; s_ticket[4] = info.y; s_ticket[5] = info.z;      // the plan entry travels with the ticket
    };
    if (tid == 0) fetch(atomicAdd(&queues[my_xcd], 1));
    __syncthreads();
    if (s_ticket[0] < 0) return;

    // FUSED phase 1: the last two tiles of this workgroup whose completion has not been signalled yet (row block and
    // column units; block -1 = none).  A tile's output stores are the youngest memory operations when the next tile
    // begins, so waiting for them there would also wait for that tile's second slab; one tile later they are older
    // than everything the opening wait of a tile leaves outstanding (its second slab and the stores of the tile before
    // it) and are known to be complete at no extra cost.  So tile t is signalled when tile t + 2 opens, and what is left
    // when the workgroup runs out of tiles is signalled after a full wait.
    int sig_blk[2] = {-1, -1}, sig_units[2] = {0, 0};                // [0] = the tile before the previous one
    auto signal_ready = [&](int n) __attribute__((always_inline)) {
        // (every wavefront has passed the wait that covers these stores, and a barrier since)
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (i < n && tid == 0 && sig_blk[i] >= 0)
                __hip_atomic_fetch_add(&a.ready[sig_blk[i]], sig_units[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (n == 1) { sig_blk[0] = sig_blk[1]; sig_units[0] = sig_units[1]; sig_blk[1] = -1; }
        else        { sig_blk[0] = sig_blk[1] = -1; }
    };
    int cur_blk = 0;

    // ---- per-tile copy state: buffer resources and scalar offsets carry what is uniform, the per-thread byte offsets
    //      are fixed for a tile, so a copy costs no vector ALU work.  Rows past the end of the block re-read its last row.
    const __bf16* Abase = (PHASE == 1 ? a.x : a.g2.A);
    unsigned long long aB = 0;                         // address of the tile's first row of the A operand (plain rows)
    const unsigned char* a_ptr[GATHER ? 32 / NW : 1];        // address of this thread's chunk of each of its rows (gathered rows)
    // B rows come from w_gate / w_up (phase 1) or w_down (phase 2) of the tile's expert: base address of the first and
    // distance to the second.  (One variable per quantity, set once per tile: a choice between variables inside the
    // unrolled copy code would keep them in memory.)
    unsigned long long wB = 0, wB_up = 0;
    unsigned int b_voff = 0;
    bool counted_stores = false;                       // the previous tile's output went out as a known number of stores
    int m0 = 0, m_end = 0, nt = 0;
    unsigned int a_voff[32 / NW];
    unsigned int b_soff[8];

    // the rows behind WR consecutive positions: lane l gets the one of position at + l / (64 / WR)
    auto list_row = [&](auto wr_tag, int at) __attribute__((always_inline)) -> int {
        constexpr int WR = decltype(wr_tag)::value;
        const __attribute__((address_space(4))) int* l = (const __attribute__((address_space(4))) int*)a.list + __builtin_amdgcn_readfirstlane(at);
        int v = l[0];
#pragma unroll
        for (int k = 1; k < WR; ++k) v = lane / (64 / WR) == k ? l[k] : v;
        return v;
    };
    auto setup = [&](auto tag, int nt_) __attribute__((always_inline)) {
        typedef Cls<decltype(tag)::value> C;
        nt = __builtin_amdgcn_readfirstlane(nt_);
        if (FUSED && PHASE == 1) cur_blk = __builtin_amdgcn_readfirstlane(s_ticket[0]);
        m0 = __builtin_amdgcn_readfirstlane(s_ticket[3]); m_end = __builtin_amdgcn_readfirstlane(s_ticket[4]);
        const int e = __builtin_amdgcn_readfirstlane(s_ticket[5]);
        const int rows = min(C::BMc, m_end - m0);
        const int row0 = C::ROWB == 128 ? row0_128 : row0_64, kcg = C::ROWB == 128 ? kcg_128 : kcg_64;
        if constexpr (GATHER) {
#pragma unroll
            for (int i = 0; i < C::CA; ++i) {
                const int m = m0 + min(row0 + C::RPC * i, rows - 1);
                a_ptr[i] = (const unsigned char*)Abase + ((unsigned long long)(unsigned int)a.list[m] * (unsigned int)lda + kcg * 8) * 2ull;
            }
        } else if constexpr (AROWS == ROWS_LIST32) {
            aB = (unsigned long long)Abase;
            constexpr int WR = C::RPC / NW;                               // rows of a wavefront's copy instruction
#pragma unroll
            for (int i = 0; i < C::CA; ++i)                               // (entries past the block's end are rows too: LIST_PAD)
                a_voff[i] = (unsigned int)list_row(std::integral_constant<int, WR>{}, m0 + C::RPC * i + WR * wave) * (unsigned int)(lda * 2) + (unsigned int)(kcg * 16);
        } else {
            aB = (unsigned long long)Abase + (unsigned long long)(unsigned int)m0 * (unsigned int)lda * 2ull;
#pragma unroll
            for (int i = 0; i < C::CA; ++i) a_voff[i] = (unsigned int)(min(row0 + C::RPC * i, rows - 1) * lda + kcg * 8) * 2u;
        }
        // the B rows of the tile: 64-bit base at the tile's first column unit, 32-bit offsets from there
        const int u0 = min(nt * C::U, NU - 1);
        if (PHASE == 1) {
            wB = (unsigned long long)((const __bf16*)a.wg + ((size_t)e * a.f + (size_t)u0 * 128) * ldb);
            wB_up = (unsigned long long)((const __bf16*)a.wu + ((size_t)e * a.f + (size_t)u0 * 128) * ldb) - wB;
        } else {
            wB = (unsigned long long)(a.g2.B + (size_t)e * a.g2.strideB + (size_t)u0 * 256 * ldb);
            wB_up = 0;
        }
        b_voff = (unsigned int)(row0 * ldb + kcg * 8) * 2u;
        constexpr int CPSTRIP = 128 / C::RPC;                             // copies per 128-row strip of the B slab
#pragma unroll
        for (int j = 0; j < C::CB; ++j) {
            const int strip = j / CPSTRIP;
            const int ug = min(nt * C::U + (strip >> 1), NU - 1) - u0;
            const int strip_row = PHASE == 1 ? ug * 128 : ug * 256 + (strip & 1) * 128;   // row from the tile's first B row
            b_soff[j] = (unsigned int)(strip_row + (j % CPSTRIP) * C::RPC) * (unsigned int)ldb * 2u;
        }
    };
    // copy n of slab s into slab buffer sbuf
    auto issue_copy = [&](auto tag, int s, int sbuf, int n) __attribute__((always_inline)) {
        typedef Cls<decltype(tag)::value> C;
        constexpr int CPSTRIP = 128 / C::RPC;
        unsigned char* base = smem + sbuf * C::SLAB + wave_bytes;
        const int koff = s * C::ROWB;                           // (plain locals: the builtin's operands must not be dependent expressions)
        if (n < C::CA) {
            if constexpr (GATHER) {
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(a_ptr[n] + koff),
                                                 (__attribute__((address_space(3))) void*)(base + n * (NW * 1024)), 16, 0, 0);
            } else {
                const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc((void*)aB, 0, 0xFFFFFFFF, 0x00020000);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (__attribute__((address_space(3))) void*)(base + n * (NW * 1024)), 16,
                                                         a_voff[n], koff, 0, FUSED && PHASE == 2 ? DEVICE_SCOPE : 0);
            }
        } else {
            const int j = n - C::CA;
            const unsigned long long up = (j / CPSTRIP) & 1;
            const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc((void*)(wB + up * wB_up), 0, 0xFFFFFFFF, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB,
                                                     (__attribute__((address_space(3))) void*)(base + C::A_BYTES + j * (NW * 1024)), 16,
                                                     b_voff, b_soff[j] + koff, 0, 0);
        }
    };
    // slabs [first, last) of the tile go out at once (the tile's opening; later slabs are spaced between the MFMAs)
    auto prologue = [&](auto tag, int first, int last) __attribute__((always_inline)) {
        typedef Cls<decltype(tag)::value> C;
        const int NS = K / (C::ROWB / 2);
#pragma unroll
        for (int s = 0; s < C::NSS; ++s)
            if (s >= first && s < last && s < NS) {
#pragma unroll
                for (int n = 0; n < C::NCOPY; ++n) issue_copy(tag, s, s, n);
            }
    };
    // Addresses of the tile and its first slabs, one per buffer (every K here has more slabs than there are buffers).
    auto start_tile = [&](int nt_, int cls) __attribute__((always_inline)) {
        if (cls == 0)      { setup(std::integral_constant<int, 0>{}, nt_); prologue(std::integral_constant<int, 0>{}, 0, 2); }
        else               { setup(std::integral_constant<int, 1>{}, nt_); prologue(std::integral_constant<int, 1>{}, 0, 3); }
    };

    // One tile of the class given by `tag`; its first slabs (one per buffer) are in flight.  Returns the class of the
    // next tile (whose first slabs it has issued: slab 0 in its last slabs or before its own read-out, the others
    // before the read-out) or -1.
    auto run_tile = [&](auto tag) __attribute__((always_inline)) -> int {
        typedef Cls<decltype(tag)::value> C;
        constexpr int MB = C::MB, NQ = C::NQ, NSS = C::NSS, SUB = C::SUB;
        constexpr int ROWB = C::ROWB, NMF = MB * NQ, NR = MB + NQ;
        constexpr int LPS = C::NCOPY;                                   // copies every wavefront issues per slab
        constexpr int NSTORE = MB * (PHASE == 1 ? 4 : 8) * (EPI == 1 ? 3 : 1);      // 1 KiB stores per wavefront and tile
        constexpr bool COUNTABLE = (NSS - 1) * C::NCOPY + NSTORE < 64;     // (the counter of memory operations in flight has 6 bits)
        static_assert((NSS - 1) * C::NCOPY < 64 && NSS * C::SLAB <= STAGE_OFF, "pipeline shape");
        static_assert(Cls<0>::MB == Cls<1>::MB, "a tile of either class issues NSTORE output stores");
        const int NS = K / (ROWB / 2);
        const int wm = wave / C::WNW, wn = wave % C::WNW;
        const int b_wave_row = PHASE == 1 ? (wn >> 1) * 256 + (wn & 1) * 64 : wn * 128;
        auto bq = [](int q) { return PHASE == 1 ? (q >> 1) * 128 + (q & 1) * 32 : q * 32; };
        const unsigned char* fragA = smem + (wm * 32 * MB) * ROWB;
        const unsigned char* fragB = smem + C::A_BYTES + b_wave_row * ROWB;

        auto load_frag_one = [&](bf16x8 (&wf)[NQ], bf16x8 (&xf)[MB], int sbuf, int u, int i) __attribute__((always_inline)) {
            const int off = sbuf * C::SLAB + (ROWB == 128 ? frag_off128[u] : frag_off64[u & 1]);
            if (i < NQ) wf[i] = *reinterpret_cast<const bf16x8*>(fragB + off + bq(i) * ROWB);
            else        xf[i - NQ] = *reinterpret_cast<const bf16x8*>(fragA + off + (i - NQ) * 32 * ROWB);
        };
        auto wait_slabs = [&](int y) __attribute__((always_inline)) {
            if (y >= 2) wait_vmcnt<2 * LPS>(); else if (y == 1) wait_vmcnt<LPS>(); else wait_vmcnt<0>();
        };

        f32x16 acc[MB][NQ];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mb][q][v] = 0.f;
        const int em0 = m0, em_end = m_end, ent = nt;                   // this tile's rows and column unit, for the read-out
        const int eblk = cur_blk;
        int nblk = -1, nnt = 0, ncls = 0;                                // ticket of the next tile
        bool chained = false;                                            // the next tile's slab 0 was issued inside this tile

        // Issued so far, oldest first: slab 0, the slabs of the other buffers, the previous tile's output stores.  The
        // stores need not be awaited when their number is known (memory operations of a wavefront are counted in order).
        if (COUNTABLE && counted_stores) wait_vmcnt<COUNTABLE ? (NSS - 1) * LPS + NSTORE : 0>(); else wait_vmcnt<(NSS - 1) * LPS>();
        lds_barrier();                   // slab 0 is in LDS
        if (FUSED && PHASE == 1) signal_ready(1);
        // Ticket of the next tile: the counter's old value returns while slab 0 is multiplied and is turned into a
        // ticket after that slab (waiting for it here would hold wavefront 0, and with it every barrier, until the
        // copies just issued have landed: memory operations of a wavefront return in order).
        int next_k = 0;
        if (tid == 0) next_k = atomicAdd(&queues[my_xcd], 1);
        // router weights of this wavefront's rows: fetched here, where they are older than every copy still to be issued
        float gate[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) gate[mb] = 1.0f;
        if (PHASE == 2 && OROWS != ROWS_PLAIN && a.gate) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) gate[mb] = a.gate[min(em0 + (wm * MB + mb) * 32 + l31, em_end - 1)];
        }
        bf16x8 wf[2][NQ], xf[2][MB];
#pragma unroll
        for (int i = 0; i < NR; ++i) load_frag_one(wf[0], xf[0], 0, 0, i);

        auto hold_gate = [&]() __attribute__((always_inline)) {             // (waited for here, not at the read-out behind the next tile's copies)
            if (PHASE == 2 && OROWS != ROWS_PLAIN) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+v"(gate[mb]));
            }
        };

        // Slab s in buffer buf.  NEW: slab s + NSS exists (its slot 0 follows this slab's barrier); OLD: slab s - 1 + NSS
        // exists (its later slots go out during this slab's K steps); FINAL: the tile's last slab.
        // CHAIN (256-row class followed by another tile of it): the next tile's slab 0 takes the place of "slab NS" --
        // 1: this is slab NS - 2; after its first K step no copy of this tile is left, the next tile's addresses are
        //    set up, and slot 0 of that slab 0 follows this slab's barrier;  2: this is slab NS - 1, slot 1 goes out.
        auto slab = [&](int s, int buf, auto new_tag, auto old_tag, auto final_tag, auto chain_tag) __attribute__((always_inline)) {
            constexpr bool NEW = decltype(new_tag)::value, OLD = decltype(old_tag)::value, FINAL = decltype(final_tag)::value;
            constexpr int CHAIN = decltype(chain_tag)::value;
            static_assert(CHAIN == 0 || (C::S2 == 0 && NSS == 2 && !NEW && (CHAIN == 1 ? OLD && !FINAL : !OLD && FINAL)), "chained slabs");
            const int nbuf = buf + 1 == NSS ? 0 : buf + 1;              // buffer of slab s + 1
            const int pbuf = buf == 0 ? NSS - 1 : buf - 1;              // buffer slab s - 1 has left
#pragma unroll
            for (int u = 0; u < SUB; ++u) {
                const int cur = u & 1, nxt = cur ^ 1;
                const bool last = u + 1 == SUB;
                // fragment reads of the next K step (from the next slab after the barrier) and this K step's share
                // of the copies alternate in program order, so that the scheduler may interleave them with the MFMAs
                int rbuf = buf, ru = u + 1;
                const bool reads = !(last && FINAL);
                if (last && !FINAL) {
                    if (NEW) wait_vmcnt<(NSS - 2) * LPS>(); else wait_slabs(min(NSS - 2, NS - 2 - s));
                    lds_barrier();
                    rbuf = nbuf; ru = 0;
                }
                const int n = last ? (NEW || CHAIN == 1 ? C::S0 : 0)
                                   : (CHAIN == 2 ? (u == 0 ? C::S1 : 0) : (!OLD ? 0 : (u == 0 ? C::S1 : (u == 1 ? C::S2 : 0))));
                const int c0 = last ? 0 : (u == 0 ? C::S0 : C::S0 + C::S1);
                const int cslab = (CHAIN == 1 && last) || CHAIN == 2 ? 0 : (last ? s + NSS : s - 1 + NSS);
                const int cbuf = last ? buf : pbuf;
#pragma unroll
                for (int i = 0; i < NMF; ++i) {
                    if (i < NR && reads) load_frag_one(wf[nxt], xf[nxt], rbuf, ru, i);
#pragma unroll
                    for (int j = (i * n + NMF - 1) / NMF; j < ((i + 1) * n + NMF - 1) / NMF; ++j) issue_copy(tag, cslab, cbuf, c0 + j);
                }
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
                        acc[mb][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[cur][q], xf[cur][mb], acc[mb][q], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < NMF; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                  // MFMA
                    if (i < NR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                      // LDS read
#pragma unroll
                    for (int j = (i * n + NMF - 1) / NMF; j < ((i + 1) * n + NMF - 1) / NMF; ++j)
                        __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);                              // slab copy
                }
                __builtin_amdgcn_sched_barrier(0);
                if (CHAIN == 1 && u == 0) {                              // this tile's last copies are out
                    if (chained) setup(tag, nnt);                        // addresses of the next tile
                }
            }
        };
        {
            const std::true_type T{};
            const std::false_type F{};
            const std::integral_constant<int, 0> C0{};
            if constexpr (decltype(tag)::value == 0) {
                // 256-row class: K is a multiple of 128 and at least 256, so NS is even and >= 4; slab s sits in buffer s & 1
                slab(0, 0, T, F, F, C0);
                hold_gate();
                if (tid == 0) fetch(next_k);
                int s = 1;
                for (; s + 2 < NS; ++s) slab(s, s & 1, T, T, F, C0);
                // a barrier has passed since the next tile's ticket was written
                nblk = __builtin_amdgcn_readfirstlane(s_ticket[0]); nnt = __builtin_amdgcn_readfirstlane(s_ticket[1]);
                ncls = __builtin_amdgcn_readfirstlane(s_ticket[2]);
                chained = nblk >= 0 && ncls == 0 && !GATHER;
                // not chained: the two slots re-fetch this tile's slab 0 into the free buffer 0, which nobody reads
                slab(NS - 2, 0, F, T, F, std::integral_constant<int, 1>{});
                slab(NS - 1, 1, F, F, T, std::integral_constant<int, 2>{});
                if (!chained) wait_vmcnt<0>();                           // ... and is complete before buffer 0 is reused
            } else {
                int buf = 0;
                auto next = [&]() __attribute__((always_inline)) { buf = buf + 1 == NSS ? 0 : buf + 1; };
                if (NSS < NS) slab(0, 0, T, F, F, C0); else slab(0, 0, F, F, F, C0);        // (every K here has at least 2 slabs)
                next();
                hold_gate();
                if (tid == 0) fetch(next_k);
                int s = 1;
                for (; s + NSS < NS; ++s) { slab(s, buf, T, T, F, C0); next(); }
                if (s + 1 < NS && s - 1 + NSS < NS) { slab(s, buf, F, T, F, C0); next(); ++s; }
                for (; s + 1 < NS; ++s) { slab(s, buf, F, F, F, C0); next(); }
                slab(NS - 1, buf, F, F, T, C0);
            }
        }
        lds_barrier();                   // every fragment is in registers: all buffers are free; next ticket visible
        if (chained) {
            prologue(tag, 1, NSS);                                      // slab 0 is under way; the other buffers follow
        } else {
            nblk = __builtin_amdgcn_readfirstlane(s_ticket[0]); nnt = __builtin_amdgcn_readfirstlane(s_ticket[1]);
            ncls = __builtin_amdgcn_readfirstlane(s_ticket[2]);         // uniform: keeps the copy descriptors in scalar registers
            if (nblk >= 0) start_tile(nnt, ncls);                       // the next tile's first slabs fly during the epilogue
            lds_barrier();                                              // the ticket has been read: its bytes may stage output
        }

        // ---- epilogue.  acc[mb][q][v]: row l31 of row block mb; column 8*(v>>2) + 4*lhi + (v&3) of column block q.
        // A lane holds 4 consecutive columns of one row: stored from there, one instruction would touch 32 rows with
        // 16 bytes each, and the L2 takes one request per piece.  Each wavefront instead passes 32 rows x 64 columns at
        // a time through a private staging area in LDS (above the slab buffers, where the next tile is arriving) and
        // stores whole 128-byte lines: 16-byte chunk c of row r sits at position c ^ swz(r), conflict-free both ways.
        const int ug = ent * C::U + (wn >> 1);
        constexpr int SROW = 128;                                           // staged bytes per row: 64 columns
        constexpr int CPR = SROW / 16;                                      // chunks per row
        constexpr int RPI = 64 / CPR;                                       // rows one store instruction covers
        constexpr int NH = PHASE == 1 ? 1 : 2;                              // 64-column halves of the wavefront's output
        int lane_e = lane;
        asm volatile("" : "+v"(lane_e));                                    // address arithmetic stays here, not in registers held across the tile loop
        const int el31 = lane_e & 31, elhi = lane_e >> 5;
        const int sr = lane_e / CPR, sc = lane_e % CPR;
        auto swz = [](int r) { return (r >> 1) & 7; };
        unsigned char* stage = smem + STAGE_OFF + wave * STAGE_WAVE;
        unsigned char* wr = stage + el31 * SROW + elhi * 8;
        const int wrow = em0 + wm * 32 * MB;                                // first row of this wavefront
        constexpr bool scatter = PHASE == 2 && OROWS == ROWS_LIST64;
        // plain case: rows and columns past the end fall outside the buffer descriptor and are dropped, so every
        // wavefront issues exactly NSTORE stores per tile
        constexpr int NPASS = EPI == 1 ? 3 : 1;                             // outputs per tile: h, or dg, du and h
        const int live = ug < NU ? min(max(em_end - wrow, 0), 32 * MB) : 0;
        __amdgpu_buffer_rsrc_t rsO[NPASS];
        int rowb[NPASS];
#pragma unroll
        for (int pass = 0; pass < NPASS; ++pass) {
            __bf16* obase;
            if (PHASE == 2 && OROWS == ROWS_LIST32) { obase = a.g2.O + ug * 256 + (wn & 1) * 128; rowb[pass] = a.g2.ldo * 2; }
            else if (PHASE == 2)             { obase = a.g2.O + (long long)wrow * a.g2.ldo + ug * 256 + (wn & 1) * 128; rowb[pass] = a.g2.ldo * 2; }
            else if (EPI == 0 || pass == 2)  { obase = a.h + (long long)wrow * a.f + ug * 128 + (wn & 1) * 64; rowb[pass] = a.f * 2; }
            else                             { obase = a.dgu + (long long)wrow * (2 * a.f) + pass * a.f + ug * 128 + (wn & 1) * 64; rowb[pass] = a.f * 4; }
            const unsigned long long ob = (unsigned long long)obase;      // (made uniform explicitly: the descriptor must sit in scalar registers)
            const unsigned int ob_lo = (unsigned int)__builtin_amdgcn_readfirstlane((unsigned int)ob);       // (the builtin returns int:
            const unsigned int ob_hi = (unsigned int)__builtin_amdgcn_readfirstlane((unsigned int)(ob >> 32)); //  widen as unsigned)
            const unsigned long long ob_u = ((unsigned long long)ob_hi << 32) | ob_lo;
            unsigned int bytes = live * rowb[pass];
            if (PHASE == 2 && OROWS == ROWS_LIST32) bytes = ug < NU ? a.g2.o_bytes - (unsigned int)(ug * 512 + (wn & 1) * 256) : 0u;
            rsO[pass] = __builtin_amdgcn_make_buffer_rsrc((void*)ob_u, 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
        }
        counted_stores = !scatter;
        if (!scatter || ug < NU) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                if (PHASE == 2 && OROWS != ROWS_PLAIN && a.gate) {         // router weight of the row
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[mb][q][v] *= gate[mb];
                }
                // byte offsets of the listed rows this lane stores; a row past the end gets one past the end of y
                unsigned int srow[PHASE == 2 && OROWS == ROWS_LIST32 ? 32 / RPI : 1];
                if constexpr (PHASE == 2 && OROWS == ROWS_LIST32) {
#pragma unroll
                    for (int i = 0; i < 32 / RPI; ++i) {
                        const int at = wrow + mb * 32 + i * RPI;
                        // (positions that no row of the tile has are not looked up: the list ends LIST_PAD after its last row)
                        const int row = list_row(std::integral_constant<int, RPI>{}, min(at, em_end - 1));
                        srow[i] = at + sr < em_end ? (unsigned int)row * (unsigned int)rowb[0] : 0xFFFFFF00u;
                    }
                }
                // backward pass: the gradient of the hidden activations at this lane's 2 x 4 groups of 4 columns (rows
                // and units past the end read the last valid ones; what is computed from them is not stored)
                u32x2 dhv[EPI == 1 ? 8 : 1];
                if constexpr (EPI == 1) {
                    const int row_c = min(wrow + mb * 32 + el31, em_end - 1);
                    const __bf16* src = a.dh + (long long)row_c * a.lddh + min(ug, NU - 1) * 128 + (wn & 1) * 64 + elhi * 4;
#pragma unroll
                    for (int c = 0; c < 8; ++c) dhv[c] = *reinterpret_cast<const u32x2*>(src + c * 8);
                }
#pragma unroll
                for (int step = 0; step < NPASS; ++step) {
                // backward pass: h goes out first; the same sweep leaves dg and du in the accumulators of g and u, from
                // where the two later sweeps store them (one exponential per element)
                const int pass = EPI == 1 ? (step + 2) % 3 : 0;
#pragma unroll
                for (int hq = 0; hq < NH; ++hq) {
#pragma unroll
                    for (int q = 0; q < 2; ++q)
#pragma unroll
                        for (int vg = 0; vg < 4; ++vg) {
                            float hv[4];
                            if constexpr (EPI == 1) {
                                if (step == 0) {
                                    const bf16x4 d4 = __builtin_bit_cast(bf16x4, dhv[q * 4 + vg]);
#pragma unroll
                                    for (int j = 0; j < 4; ++j) {
                                        const float g = acc[mb][q][vg * 4 + j], u = acc[mb][q + 2][vg * 4 + j], dh = (float)d4[j];
                                        const float sig = __builtin_amdgcn_rcpf(1.0f + __expf(-g));
                                        hv[j] = (g * sig) * u;                                                  // h
                                        acc[mb][q][vg * 4 + j] = dh * u * (sig * (1.0f + g * (1.0f - sig)));    // dg = dh * u * silu'(g)
                                        acc[mb][q + 2][vg * 4 + j] = dh * (g * sig);                            // du = dh * silu(g)
                                    }
                                } else {
#pragma unroll
                                    for (int j = 0; j < 4; ++j) hv[j] = acc[mb][step == 1 ? q : q + 2][vg * 4 + j];
                                }
                            } else {
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    hv[j] = PHASE == 1 ? silu(acc[mb][q][vg * 4 + j]) * acc[mb][q + 2][vg * 4 + j]
                                                       : acc[mb][hq * 2 + q][vg * 4 + j];
                            }
                            *reinterpret_cast<u32x2*>(wr + (((q * 4 + vg) ^ swz(el31)) << 4)) = pack4(hv[0], hv[1], hv[2], hv[3]);
                        }
                    u32x4 v[32 / RPI];
#pragma unroll
                    for (int i = 0; i < 32 / RPI; ++i) {
                        const int r = i * RPI + sr;
                        v[i] = *reinterpret_cast<const u32x4*>(stage + r * SROW + ((sc ^ swz(r)) << 4));
                    }
                    if constexpr (PHASE == 2 && OROWS == ROWS_LIST32) {
#pragma unroll
                        for (int i = 0; i < 32 / RPI; ++i)
                            __builtin_amdgcn_raw_buffer_store_b128(v[i], rsO[pass], srow[i] + hq * SROW + sc * 16, 0, 0);
                    } else if (!scatter) {
#pragma unroll
                        for (int i = 0; i < 32 / RPI; ++i)
                            __builtin_amdgcn_raw_buffer_store_b128(v[i], rsO[pass], (mb * 32 + i * RPI + sr) * rowb[pass] + hq * SROW + sc * 16, 0,
                                                                   FUSED && PHASE == 1 ? DEVICE_SCOPE : 0);
                    } else {
#pragma unroll
                        for (int i = 0; i < 32 / RPI; ++i) {
                            const int m = wrow + mb * 32 + i * RPI + sr;
                            if (m < em_end)
                                *reinterpret_cast<u32x4*>(a.g2.O + (long long)mapped_row(a, m) * a.g2.ldo + ug * 256 + (wn & 1) * 128 + hq * 64 + sc * 8) = v[i];
                        }
                    }
                }
                }
                __builtin_amdgcn_sched_barrier(0);     // one row block at a time: keeps the accumulator read-out short-lived
            }
        }
        if (FUSED && PHASE == 1) { sig_blk[1] = eblk; sig_units[1] = min(C::U, NU - ent * C::U); }
        return nblk >= 0 ? ncls : -1;
    };

    int cls = __builtin_amdgcn_readfirstlane(s_ticket[2]);
    start_tile(__builtin_amdgcn_readfirstlane(s_ticket[1]), cls);
    while (cls >= 0) {
        if (cls == 0)      cls = run_tile(std::integral_constant<int, 0>{});
        else               cls = run_tile(std::integral_constant<int, 1>{});
    }
    if (FUSED && PHASE == 1) {           // the last two tiles of this workgroup
        wait_vmcnt<0>();
        lds_barrier();
        signal_ready(2);
    }
}

template <int PHASE, int AROWS, int OROWS, int EPI>
__global__ __launch_bounds__(NW * 64, 1)
void ffn_adaptive_kernel(FfnArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    ffn_adaptive_body<PHASE, AROWS, OROWS, false, EPI>(a, smem);
}

// Both phases in one launch: a workgroup works through the phase-1 tiles until none is left to hand out, then
// through the phase-2 tiles, each of which starts when the rows of h it reads are complete (release by the writers,
// acquire by the reader, at device scope).  The tail of phase 1 is filled with phase-2 tiles, and a call costs one
// launch of the matrix kernels whatever the number of slices.
template <int ROWS>
__global__ __launch_bounds__(NW * 64, 1)
void ffn_fused_kernel(FfnArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    ffn_adaptive_body<1, ROWS, ROWS_PLAIN, true>(a, smem);
    __syncthreads();                     // the ticket area and the staging buffers change hands
    ffn_adaptive_body<2, ROWS_PLAIN, ROWS, true>(a, smem);
}

// ---------------------------------------------------------------------------------- few rows per expert (decoding)
// Bound by the weights' way from HBM: with few rows per expert a tile kernel has too few tiles for the chip
// (f / 128 and d / 256 column tiles per expert) and too few bytes in flight per tile.  Here a workgroup takes a strip of
// 16 * NC weight rows of one expert (phase 1: half of them gate, half up) and up to 16 * MT of the expert's rows, and its W wavefronts
// share the contraction: 64 values of K each in turn, weights and activations straight from memory into MFMA fragments, the
// next two (D - 1) steps in flight while one is multiplied.  The W partial sums meet in LDS and are added in fp32 in a fixed order.
// No plan: every workgroup finds its rows in the offsets by itself (a scan over the S groups of its expert), h lies in schedule
// order, K-major (8 values of K of all rows side by side): a fragment load of phase 2 then covers runs of 16 rows x 16 bytes
// instead of 16 rows that lie a power of two apart in the same memory channel (phase 2 of d = 4096, f = 14336 at 64 rows 69 ->
// 48 us; d = 7168, f = 2048, four fp8 experts 42 -> 28 us).  For the same reason the strips start at different steps of K
// (one expert, d 4096, f 14336, 5 rows: 86 -> 70 us).
// One expert, d 4096, f 14336 (352 MB of weights): 5 rows 68 us, 5.2 TB/s; with more rows the activations' way from L2 counts too (37 rows 96 us, in
// tiles of 64 rows 85).
struct SkinnyArgs {
    const __bf16* x; __bf16* h; __bf16* y;
    const __bf16* xk;                  // the rows of x in schedule order, K-major as h, or null: phase 1 reads x
    const void *wg, *wu, *wd;
    const float *sg, *su, *sd;
    const int32_t* offsets;
    const int32_t* row_map; const float* row_gate;
    int M, S, E, d, f;
};
typedef __attribute__((ext_vector_type(4))) float f32x4;
constexpr int SKINNY_MAX_SLICES = 1024;

// xk[k / 8][m][8] = row m's x: 8 lanes fetch 128 bytes of a row, the 8 rows of a wavefront lie side by side in the result
__global__ __launch_bounds__(256)
void ffn_kmajor_kernel(const __bf16* __restrict__ x, const int32_t* __restrict__ row_map, const int32_t* __restrict__ last, int M, int d,
                       __bf16* __restrict__ xk) {
    const int m = blockIdx.x * 32 + (threadIdx.x >> 3), k8 = blockIdx.y * 8 + (threadIdx.x & 7);       // (d is a multiple of 64)
    if (m >= M) return;
    int row = m;
    if (row_map) {
        if (m >= *last) return;                                           // the map ends with the last group
        row = row_map[m];
        row = (unsigned)row < (unsigned)M ? row : 0;
    }
    *reinterpret_cast<u32x4*>(xk + ((size_t)k8 * M + m) * 8) = *reinterpret_cast<const u32x4*>(x + (size_t)row * d + k8 * 8);
}

// W wavefronts, NC 16-row column tiles of weights, at most MT 16-row tiles of activations, D register buffers
// (fp8, two row tiles: two workgroups per compute unit.  Its registers would let in three, which leaves other units with one: 448 workgroups of E 16, d 7168, f 2048,
// 24 rows, phase 1 65 us, with two 50; E 32, d 2048, f 768, 17 rows 18, 14.)
template <int PHASE, int W, int NC, int MT, int D, bool FP8>
__global__ __attribute__((amdgpu_waves_per_eu(1, FP8 && MT == 2 ? 2 : 8))) __launch_bounds__(W * 64)
void ffn_skinny_kernel(SkinnyArgs a) {
    static_assert(PHASE == 2 || NC % 2 == 0, "gate and up tiles in pairs");
    constexpr int ESZ = FP8 ? 1 : 2, WL = FP8 ? 1 : 2;                     // 16-byte weight loads per lane, column tile and 64 values of K
    constexpr int PASS = 32 / (W * NC) < 1 ? 1 : (32 / (W * NC) > MT ? MT : 32 / (W * NC));     // row tiles per reduction pass
    constexpr int NH = PHASE == 1 ? NC / 2 : NC;                           // column tiles of the output
    constexpr int ROWS = 16 * MT;                                          // rows per workgroup
    __shared__ int s_row[ROWS];
    __shared__ int s_scan[W];
    __shared__ f32x4 s_red[W * NC * PASS * 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g4 = lane >> 4;
    const int strip = blockIdx.x, e = blockIdx.y;
    const int K = PHASE == 1 ? a.d : a.f, NO = PHASE == 1 ? a.f : a.d;     // contraction, output columns
    const int col0 = strip * 16 * NH;
    const int KT = K / 64, n = (KT - wave + W - 1) / W;                    // steps in all, and of this wavefront (K >= 128)
    const int rot = (int)(((unsigned)strip * 3u + (unsigned)e * 3u) % (unsigned)KT);

    for (int first = (int)blockIdx.z * ROWS;; first += (int)gridDim.z * ROWS) {
        // ---- positions first .. first + ROWS - 1 of the expert's rows
        int total = 0;
        for (int s0 = 0; s0 < a.S; s0 += W * 64) {
            const int s = s0 + tid;
            int lo = 0, rows = 0;
            if (s < a.S) {
                const int gi = s * a.E + e;
                lo = min(max(a.offsets[gi], 0), a.M);
                rows = min(max(a.offsets[gi + 1], lo), a.M) - lo;
            }
            int incl = rows;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(incl, off);
                if (lane >= off) incl += o;
            }
            if (lane == 63) s_scan[wave] = incl;
            __syncthreads();
            int base = total;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int t = s_scan[w];
                if (w < wave) base += t;
                total += t;
            }
            const int p0 = base + incl - rows;
            for (int p = max(p0, first); p < min(p0 + rows, first + ROWS); ++p) s_row[p - first] = lo + (p - p0);
            __syncthreads();
        }
        const int rows = min(total - first, ROWS);
        if (rows <= 0) return;

        auto mapped = [&](int m) __attribute__((always_inline)) -> int {
            if (!a.row_map) return m;
            const int r = a.row_map[m];
            return (unsigned)r < (unsigned)a.M ? r : 0;
        };
        auto work = [&](auto tag) __attribute__((always_inline)) {
            constexpr int T = decltype(tag)::value;                        // 16-row tiles of this workgroup's rows
            constexpr int TS = FP8 ? T : 1;
            f32x4 acc[NC][T];
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int t = 0; t < T; ++t) acc[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
            // Lane (r16, g4) holds row r16 of a 16-row tile and 8 consecutive values of K per MFMA step.  The order of K inside a
            // step is free as long as both operands agree: fp8 lanes fetch 16 consecutive codes, the two steps' worth.
            const bool kmajor = PHASE == 2 || a.xk;
            unsigned int xoff[T];                                          // (M * K * 2 < 2^32 is a condition of this route)
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int m = s_row[min(t * 16 + r16, rows - 1)];          // rows past the end repeat the last one and are not stored
                xoff[t] = !kmajor ? ((unsigned int)mapped(m) * (unsigned int)K + (unsigned int)g4 * (FP8 ? 16 : 8)) * 2u
                                  : ((unsigned int)g4 * (FP8 ? 2 : 1) * (unsigned int)a.M + (unsigned int)m) * 16u;
            }
            const void* const xbase = PHASE == 2 ? (const void*)a.h : (const void*)(a.xk ? a.xk : a.x);
            const unsigned int xbytes = (unsigned int)a.M * (unsigned int)K * 2u;
            // bytes per value of K, and from the first MFMA step of 64 values to the second
            const unsigned int xstep = kmajor ? 2u * (unsigned int)a.M : 2u;
            const unsigned int xhalf = (FP8 ? 16u : 64u) * (kmajor ? (unsigned int)a.M : 1u);
            const unsigned int woff = ((unsigned int)r16 * (unsigned int)K) * ESZ + (unsigned int)g4 * 16u;
            const unsigned int wbytes = 16u * (unsigned int)K * ESZ;
            const unsigned char* wbase[NC];
            const float* sbase[2] = {nullptr, nullptr};                    // scale row of the strip's 128 x 128 blocks (gate / up or down)
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const void* w = PHASE == 2 ? a.wd : (c < NH ? a.wg : a.wu);
                wbase[c] = (const unsigned char*)w + ((size_t)e * NO + col0 + (c % NH) * 16) * (size_t)K * ESZ;
            }
            if (FP8) {
                const size_t srow = ((size_t)e * (NO / 128) + col0 / 128) * (size_t)(K / 128);
                sbase[0] = (PHASE == 2 ? a.sd : a.sg) + srow;
                sbase[1] = (PHASE == 2 ? a.sd : a.su) + srow;
            }
            struct Buf { u32x4 w[NC][WL], x[T][2]; float sc[2]; };
            Buf buf[D];
            // steps past the last one read through an empty descriptor: zeros, and no memory traffic
            auto load = [&](Buf& b, int i) __attribute__((always_inline)) {
                const bool live = i < n;
                int kc = wave + W * i + rot;                               // (a step past the last one may lie up to W * D further: not read)
                kc = kc >= KT ? kc - KT : kc;
                const unsigned int k0 = (unsigned int)kc * 64u;
                const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)xbase, 0, live ? xbytes : 0u, 0x00020000);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)wbase[c], 0, live ? wbytes : 0u, 0x00020000);
#pragma unroll
                    for (int j = 0; j < WL; ++j) b.w[c][j] = __builtin_amdgcn_raw_buffer_load_b128(rw, woff + k0 * ESZ + j * 64, 0, 0);
                }
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int j = 0; j < 2; ++j) b.x[t][j] = __builtin_amdgcn_raw_buffer_load_b128(rx, xoff[t] + k0 * xstep + j * xhalf, 0, 0);
                if (FP8) {
                    const int kb = (int)(min(k0, (unsigned int)K - 64u) >> 7);
                    b.sc[0] = sbase[0][kb];
                    if (PHASE == 1) b.sc[1] = sbase[1][kb];
                }
            };
            // fp8: codes are widened to bf16 (exactly), and the scale multiplies the fp32 sum over the step's 64 values of K
            auto multiply = [&](const Buf& b) __attribute__((always_inline)) {
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    f32x4 sum[TS];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const bf16x8 wv = FP8 ? widen8(b.w[c][0], j) : __builtin_bit_cast(bf16x8, b.w[c][FP8 ? 0 : j]);
#pragma unroll
                        for (int t = 0; t < T; ++t) {
                            if (FP8) sum[FP8 ? t : 0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, __builtin_bit_cast(bf16x8, b.x[t][j]), j == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[FP8 ? t : 0], 0, 0, 0);
                            else     acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, __builtin_bit_cast(bf16x8, b.x[t][j]), acc[c][t], 0, 0, 0);
                        }
                    }
                    if (FP8) {
                        const float sc = b.sc[PHASE == 1 && c >= NH ? 1 : 0] * (1.0f / CODE_UNIT);
#pragma unroll
                        for (int t = 0; t < T; ++t)
#pragma unroll
                            for (int v = 0; v < 4; ++v) acc[c][t][v] = __builtin_fmaf(sum[FP8 ? t : 0][v], sc, acc[c][t][v]);
                    }
                }
            };
#pragma unroll
            for (int i = 0; i < D - 1; ++i) load(buf[i], i);
            for (int i = 0; i < n; i += D) {
#pragma unroll
                for (int u = 0; u < D; ++u) {
                    load(buf[(u + D - 1) % D], i + u + D - 1);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(buf[u]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // ---- partial sums of the wavefronts; acc[c][t][v]: weight row 4 * g4 + v of column tile c, row r16 of row tile t
#pragma unroll
            for (int t0 = 0; t0 < T; t0 += PASS) {
                if (t0 > 0) __syncthreads();
#pragma unroll
                for (int t = t0; t < t0 + PASS && t < T; ++t)
#pragma unroll
                    for (int c = 0; c < NC; ++c) s_red[((t - t0) * NC + c) * (W * 64) + wave * 64 + lane] = acc[c][t];
                __syncthreads();
                const int here = min(PASS, T - t0);
                for (int it = tid; it < here * NH * 64; it += W * 64) {
                    const int l = it & 63, c = (it >> 6) % NH, t = (it >> 6) / NH;
                    const int pos = (t0 + t) * 16 + (l & 15);
                    f32x4 s0 = s_red[(t * NC + c) * (W * 64) + l], s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int w = 1; w < W; ++w) s0 += s_red[(t * NC + c) * (W * 64) + w * 64 + l];
                    if (PHASE == 1) {
#pragma unroll
                        for (int w = 0; w < W; ++w) s1 += s_red[(t * NC + c + NH) * (W * 64) + w * 64 + l];
                    }
                    if (pos < rows) {
                        const int m = s_row[pos];
                        const int col = col0 + c * 16 + 4 * (l >> 4);
                        if (PHASE == 1) {
                            *reinterpret_cast<u32x2*>(a.h + ((size_t)(col >> 3) * a.M + m) * 8 + (col & 7)) =
                                pack4(silu(s0[0]) * s1[0], silu(s0[1]) * s1[1], silu(s0[2]) * s1[2], silu(s0[3]) * s1[3]);
                        } else {
                            const float gate = a.row_gate ? a.row_gate[m] : 1.0f;
                            *reinterpret_cast<u32x2*>(a.y + (size_t)mapped(m) * a.d + col) =
                                pack4(gate * s0[0], gate * s0[1], gate * s0[2], gate * s0[3]);
                        }
                    }
                }
            }
        };
        const int tiles = (rows + 15) / 16;
        if (MT == 1 || tiles == 1)      work(std::integral_constant<int, 1>{});
        else if (MT == 2 || tiles == 2) work(std::integral_constant<int, (MT < 2 ? MT : 2)>{});
        else if (MT == 3 || tiles == 3) work(std::integral_constant<int, (MT < 3 ? MT : 3)>{});
        else if (MT == 4 || tiles == 4) work(std::integral_constant<int, (MT < 4 ? MT : 4)>{});
        else if (MT == 6 || tiles <= 6) work(std::integral_constant<int, (MT < 6 ? MT : 6)>{});
        else                            work(std::integral_constant<int, MT>{});
        __syncthreads();                                                   // s_row and s_red are used again
    }
}

// ---------------------------------------------------------------------------------- a few hundred rows per expert
// Between streaming and the 256 x 256 tiles a call has too few of those tiles for the chip (d = 4096 makes 16 column tiles of w_down, each a contraction over
// all of f), so that it lasts as long as one tile's chain of K slabs.  Here a tile is 128 rows x 128 columns (phase 1: 64 gate + 64 up), four wavefronts of
// 64 x 64, two workgroups per compute unit, and where the tiles do not fill the slots (both workgroups of every compute unit) the contraction of
// a tile is split over up to TILE_MAX_PARTS workgroups, which add their sums in fp32 in part order (the last one to finish does).
// The plan says how many row blocks there are, so every workgroup works out the tiles, the split and its unit by itself; workgroups beyond the last unit
// leave at once.  With few rows bound by the weights' way from memory (37 rows of E 1, d 4096, f 14336: 5.0 and 4.2 TB/s in the two phases; 203 fp8 rows of E 4, d 7168, f 2048: 3.2 and
// 3.0, where 160 tiles of phase 1 are too many to be split over 256 compute units and leave 96 of them idle), above that by the operands' way through LDS, 32 KiB per slab of 64 values
// of K for 4.2 Mflop: 4000 rows of the latter 281 and 133 us, matrix cores busy 51 % of the cycles in which a compute unit has work, wavefronts waiting 27 %.
// Both operands are copied global -> LDS as they lie; fp8 codes are widened to bf16 (exactly) on the way from LDS to the matrix cores, two values per
// v_cvt_scalef32_pk_bf16_fp8, and the scale of a 128 x 128 block multiplies the fp32 sum over that block's 128 values of K.
constexpr int TILE = 128;                                    // columns
constexpr int TILE_MAX_PARTS = 16, TILE_MIN_SLABS = 12;       // parts of a contraction, slabs of 64 values of K per part at least
constexpr int TILE_SQUARE = 8;                               // column tiles that many row blocks are walked for at a time
// ROWS = rows per tile:
//    64: 4 wavefronts (2 x 2) of 32 x 64, three slabs of 24 KiB (fp8: four of activations, three of codes), 2 workgroups per compute unit
//   128: 4 wavefronts (2 x 2) of 64 x 64, two slabs of 32 KiB, 2 workgroups per compute unit
//   256: 8 wavefronts (4 x 2) of 64 x 64, three slabs of 48 KiB, 1 workgroup per compute unit
template <int ROWS, bool FP8> struct TileShape {
    static constexpr int WM = ROWS == 256 ? 4 : 2, MB = ROWS / (32 * WM), THREADS = 128 * WM;
    // Workgroups per compute unit up to which contractions are split.  (64 rows, one / two: E 1, d 4096, f 14336, 37 rows 85 / 100 us; fp8 E 4, d 7168, f 2048, 64
    // rows 48 / 58, 203 rows 69 / 65.  128 rows, 203 rows of the former 139 / 134; E 2, d 3584, f 4864, 512 rows 130 / 103.)
    static constexpr int SPLIT_PER_CU = ROWS == 128 ? 2 : 1;
    // Row blocks up to which they are innermost in the order of the units.  Innermost against walked for 8 column tiles at a time, mean of 36 shapes, bf16 / fp8:
    // 64 rows, 17 .. 20 / 25 .. 32 / 33 .. 48 blocks 0.97 / 1.01 / 1.04, 0.99 / 1.03 / 1.06; 128 rows, 13 .. 16 / 17 .. 20 / 33 .. 48 0.99 / 1.01 / 1.09, 1.03 / 1.04 /
    // 1.15; 256 rows, 9 .. 12 / 13 .. 16 / 33 .. 48 1.01 / 1.03 / 1.21, 1.01 / 1.03 / 1.14.  E 8, d 7168, f 2048, 1250 rows per expert, 128 / 256 rows: bf16 1199 -> 1022 us,
    // 1209 -> 975; fp8 1080 -> 911, 1103 -> 937.
    static constexpr int FEW_BLOCKS = ROWS == 64 ? 24 : (ROWS == 128 ? 16 : 12);
    static constexpr int NST = ROWS == 64 ? (FP8 ? 4 : 3) : (ROWS == 128 ? 2 : 3);      // places for slabs of 64 values of K of the activations
    static constexpr int NB = !FP8 ? NST : (ROWS == 64 ? 3 : 2);                        // places for slabs of 128 bytes per weight row
    static constexpr int A_BYTES = ROWS * 128, B_BYTES = TILE * 128;                    // of a place
    static constexpr size_t LDS = NST * A_BYTES + NB * B_BYTES;
    static constexpr size_t UNIT_BYTES = (size_t)ROWS * TILE * sizeof(float);
};
// parts per contraction with `tiles` tiles, at most `cap` units having room for their sums
__host__ __device__ inline int tile_parts(long long tiles, int slots, int K, int cap) {
    if (tiles < 1 || tiles >= TILE_COUNTERS) return 1;
    long long P = slots / tiles;
    const long long most = K / 64 / TILE_MIN_SLABS, room = cap / tiles;
    P = P < most ? P : most;
    P = P < room ? P : room;
    P = P < TILE_MAX_PARTS ? P : TILE_MAX_PARTS;
    return P < 1 ? 1 : (int)P;
}

struct TileArgs {
    FfnArgs a;
    f32x4* part;                       // [cap] units
    int* arrived;                      // [TILE_COUNTERS] parts of the tile that are done
    int slots, cap;
};
// What a launch computes.  FORWARD: phase 1 or 2 of the forward pass.  The backward pass's row products: BWD_DH = phase 2's arithmetic with listed rows in and
// plain rows out (dh = dy Wd), BWD_ACT = phase 1 with the gradient read-out (EPI 1 of the adaptive kernel), BWD_DX = phase 2's without router weights.
enum { FORWARD = 0, BWD_DH = 1, BWD_ACT = 2, BWD_DX = 3 };
template <int PHASE, bool FP8, int ROWS, bool WIDE, int KIND>
__global__ __launch_bounds__((TileShape<ROWS, FP8>::THREADS), 2)
void ffn_tile_kernel(TileArgs t) {
    typedef TileShape<ROWS, FP8> S;
    const FfnArgs& a = t.a;
    constexpr int ROWB = 128, NST = S::NST, NB = S::NB, MB = S::MB, A_BYTES = S::A_BYTES, B_BYTES = S::B_BYTES, B_AT = NST * A_BYTES;
    constexpr int RPC = S::THREADS / 8, CA = ROWS / RPC, CB = TILE / RPC; // rows one copy of the workgroup deposits, copies of a slab
    static_assert(CA <= 4 && (CB == 2 || CB == 4), "copies");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, l31 = lane & 31, lhi = lane >> 5;
    constexpr bool LISTED_IN = PHASE == 1 || KIND == BWD_DH, LISTED_OUT = PHASE == 2 && KIND != BWD_DH;
    const int K = PHASE == 1 ? a.d : a.g2.K, NT = PHASE == 1 ? a.f / 64 : a.g2.NU * 2;
    const int nblocks = a.plan[0].x;
    const int P = tile_parts((long long)nblocks * NT, t.slots, K, t.cap);
    // workgroup -> unit: every die (workgroup number modulo 8) takes a stretch of the units.  With few row blocks these are innermost, so that those which share
    // weights share an L2; more of them are walked for TILE_SQUARE column tiles at a time, so that the tiles which run together on a die are about as many
    // columns wide as rows high, and a row is read once per TILE_SQUARE column tiles instead of for each
    const int units = nblocks * NT * P, xcd = blockIdx.x & 7;              // (< 2^28: a condition of this route)
    const int last = units * (xcd + 1) / 8, unit = units * xcd / 8 + (int)(blockIdx.x >> 3);
    if (unit >= last) return;
    int blk, p = 0, nt;
    if (P > 1 || nblocks <= S::FEW_BLOCKS) {
        const int rest = unit / nblocks;
        blk = unit - rest * nblocks; nt = rest / P; p = rest - nt * P;
    } else {
        const int first = unit / (nblocks * TILE_SQUARE) * TILE_SQUARE, rest = unit - first * nblocks, width = min(TILE_SQUARE, NT - first);
        blk = rest / width; nt = first + rest - blk * width;
    }
    const int4 info = a.plan[PLAN_HDR + blk];
    const int m0 = __builtin_amdgcn_readfirstlane(info.x), m_end = __builtin_amdgcn_readfirstlane(info.y), e = __builtin_amdgcn_readfirstlane(info.z);
    const int rows = min(ROWS, m_end - m0);
    // this part's K: whole blocks of 128
    const int KB = K / 128, kb0 = KB * p / P, NP = KB * (p + 1) / P - kb0, NS = 2 * NP;

    // ---- copies.  A slab row is 128 bytes; 16-byte chunk c of row r sits at position c ^ ((r >> 1) & 7).
    const int row0 = tid >> 3, kcg = (tid & 7) ^ ((row0 >> 1) & 7);
    // Rows past the end lie behind the buffer descriptor: zeros are deposited, from no memory.  WIDE: x or h does not fit 32-bit offsets.
    const unsigned char* a_ptr[WIDE ? 4 : 1];
    unsigned int a_voff[4];
    const __bf16* const A = PHASE == 1 ? a.x : a.g2.A;                      // (row pitch K)
#pragma unroll
    for (int i = 0; i < CA; ++i) {
        const int r = row0 + RPC * i, m = m0 + min(r, rows - 1);
        const unsigned int row = (unsigned int)(LISTED_IN ? mapped_row(a, m) : m);
        if (WIDE) a_ptr[WIDE ? i : 0] = (const unsigned char*)(A + (size_t)row * K) + (size_t)kb0 * 256 + kcg * 16;     // (repeats the last row)
        else      a_voff[i] = r < rows ? row * (unsigned int)K * 2u + (unsigned int)kb0 * 256u + (unsigned int)kcg * 16u : 0xFFFFFF00u;
    }
    const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, (int)((unsigned int)a.M * (unsigned int)K * 2u), 0x00020000);
    constexpr int ESZ = FP8 ? 1 : 2;
    const size_t pitch = (size_t)K * ESZ;
    const unsigned char *b_lo, *b_hi;                                     // weight rows 0 .. 63 and 64 .. 127 of the tile
    if (PHASE == 1) {
        const size_t at = ((size_t)e * a.f + (size_t)nt * 64) * pitch;
        b_lo = (const unsigned char*)a.wg + at; b_hi = (const unsigned char*)a.wu + at;
    } else {
        b_lo = (const unsigned char*)a.g2.B + ((size_t)e * a.g2.strideB + (size_t)nt * TILE * K) * ESZ; b_hi = b_lo + 64 * pitch;
    }
    b_lo += (size_t)kb0 * 128 * ESZ; b_hi += (size_t)kb0 * 128 * ESZ;
    const unsigned int b_voff = (unsigned int)row0 * (unsigned int)pitch + (unsigned int)kcg * 16u;
    const __amdgpu_buffer_rsrc_t rs_lo = __builtin_amdgcn_make_buffer_rsrc((void*)b_lo, 0, 0xFFFFFFFF, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_hi = __builtin_amdgcn_make_buffer_rsrc((void*)b_hi, 0, 0xFFFFFFFF, 0x00020000);
    auto copy_a = [&](int s, int st, int i) __attribute__((always_inline)) {        // slab s into place st
        void* const to = smem + st * A_BYTES + i * RPC * ROWB + wave * 1024;
        if constexpr (WIDE) {
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(a_ptr[i] + (size_t)s * ROWB), (__attribute__((address_space(3))) void*)to, 16, 0, 0);
        } else {
            const int koff = s * ROWB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_a, (__attribute__((address_space(3))) void*)to, 16, a_voff[i], koff, 0, 0);
        }
    };
    auto copy_b = [&](int s, int st, int i) __attribute__((always_inline)) {        // 128 bytes per weight row: 64 bf16 values, or 128 codes
        const int koff = s * ROWB;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(2 * i < CB ? rs_lo : rs_hi, (__attribute__((address_space(3))) void*)(smem + B_AT + st * B_BYTES + i * RPC * ROWB + wave * 1024),
                                                 16, b_voff, (i % (CB / 2)) * RPC * (int)pitch + koff, 0, 0);
    };

    // ---- fragments.  Column blocks of the wavefront: phase 1 gate columns 32 wn .. and up columns 32 wn .., phase 2 columns 64 wn .. and 64 wn + 32 ..
    // The order of K inside 32 values is free as long as both operands agree: fp8 lanes read 16 consecutive codes, the two MFMA steps' worth.
    const int swz = (l31 >> 1) & 7;
    const unsigned char* const fa = smem + (wm * 32 * MB + l31) * ROWB;
    const int brow[2] = {(PHASE == 1 ? wn * 32 : wn * 64) + l31, (PHASE == 1 ? 64 + wn * 32 : wn * 64 + 32) + l31};
    bf16x8 xf[2][MB];
    u32x4 wf[2][2];                                                       // of K step u in wf[u & 1]; fp8: of steps 2 g and 2 g + 1 in wf[g]
    auto load_frags = [&](int s, int st, int bst, int u) __attribute__((always_inline)) {     // K step u of slab s, whose operands lie at st and bst
        const int ca = FP8 ? 4 * (u >> 1) + 2 * lhi + (u & 1) : 2 * u + lhi;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) xf[u & 1][mb] = *reinterpret_cast<const bf16x8*>(fa + st * A_BYTES + mb * 32 * ROWB + ((ca ^ swz) << 4));
        if (!FP8 || (u & 1) == 0) {
            const int cb = FP8 ? 2 * (2 * (s & 1) + (u >> 1)) + lhi : ca;
#pragma unroll
            for (int q = 0; q < 2; ++q) wf[FP8 ? u >> 1 : u & 1][q] = *reinterpret_cast<const u32x4*>(smem + B_AT + bst * B_BYTES + brow[q] * ROWB + ((cb ^ swz) << 4));
        }
    };
    typedef const __attribute__((address_space(4))) float* scalar_floats;
    scalar_floats scale[2] = {nullptr, nullptr};                          // scale row of the tile's 128 x 128 blocks: gate and up, or down
    if (FP8) {
        const size_t row = PHASE == 1 ? (size_t)e * (a.f / 128) + nt / 2 : (size_t)e * (a.d / 128) + nt;
        scale[0] = (scalar_floats)((PHASE == 1 ? a.sg : a.sd) + row * (K / 128) + kb0);
        scale[1] = (scalar_floats)((PHASE == 1 ? a.su : a.sd) + row * (K / 128) + kb0);
    }

    f32x16 acc[MB][2], sum[FP8 ? MB : 1][FP8 ? 2 : 1];            // fp8: sums over the current 128 values of K
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][q][v] = 0.f;

    // Slab s.  The barrier ahead of its last K step publishes slab s + 1 and frees its own place, into which slab s + NST is copied (fp8: the codes of
    // 128 values of K with every other slab, NB blocks ahead, behind the activations).  NEW: that slab exists.
    int st = 0, bst = 0;                                                  // places of slab s
    auto next_slab = [&](int s, auto odd_tag, auto new_tag) __attribute__((always_inline)) {         // the barrier
        constexpr bool ODD = decltype(odd_tag)::value, NEW = decltype(new_tag)::value;
        // still in flight behind what slab s + 1 needs: NST - 2 slabs, and the codes of NB - 2 blocks (while slab s + 1 is in this one's block, NB - 1)
        if (!NEW)      wait_vmcnt<0>();
        else if (!FP8) wait_vmcnt<(NST - 2) * (CA + CB)>();
        else           wait_vmcnt<(NST - 2) * CA + (NB - (ODD ? 2 : 1)) * CB>();
        lds_barrier();
    };
    auto copies_of = [&](int s, auto odd_tag) __attribute__((always_inline)) {                       // what goes out behind slab s
        constexpr bool ODD = decltype(odd_tag)::value;
#pragma unroll
        for (int i = 0; i < CA; ++i) copy_a(s + NST, st, i);
        if (!FP8) {
#pragma unroll
            for (int i = 0; i < CB; ++i) copy_b(s + NST, st, i);
        } else if (ODD) {                                                 // (ahead of the last blocks: the last one once more, into a free place)
            const int b = min((s >> 1) + NB, NP - 1);
#pragma unroll
            for (int i = 0; i < CB; ++i) copy_b(b, bst, i);
        }
    };
    auto advance = [&](auto odd_tag) __attribute__((always_inline)) {
        constexpr bool ODD = decltype(odd_tag)::value;
        st = st + 1 == NST ? 0 : st + 1;
        if (!FP8) bst = st; else if (ODD) bst = bst + 1 == NB ? 0 : bst + 1;
    };
    auto slab = [&](int s, auto odd_tag, auto new_tag, auto final_tag) __attribute__((always_inline)) {
        constexpr bool ODD = decltype(odd_tag)::value, NEW = decltype(new_tag)::value, FINAL = decltype(final_tag)::value;
        if (FP8 && !ODD) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 16; ++v) sum[FP8 ? mb : 0][FP8 ? q : 0][v] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int cur = u & 1;
            const bool last = u == 3, reads = !(last && FINAL), copies = last && NEW;
            if (last && !FINAL) {
                next_slab(s, odd_tag, new_tag);
                const int nst = st + 1 == NST ? 0 : st + 1, nbst = !FP8 ? nst : (ODD ? (bst + 1 == NB ? 0 : bst + 1) : bst);
                load_frags(s + 1, nst, nbst, 0);
            } else if (reads) {
                load_frags(s, st, bst, u + 1);
            }
            if (copies) copies_of(s, odd_tag);
            bf16x8 w[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) w[q] = FP8 ? widen8(wf[u >> 1][q], u & 1) : __builtin_bit_cast(bf16x8, wf[cur][q]);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    f32x16& c = FP8 ? sum[FP8 ? mb : 0][FP8 ? q : 0] : acc[mb][q];
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[q], xf[cur][mb], c, 0, 0, 0);
                }
#pragma unroll
            for (int i = 0; i < 2 * MB; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                         // MFMA
                if (reads) __builtin_amdgcn_sched_group_barrier(0x100, MB == 1 ? 2 : 1, 0);                // LDS reads
                if (copies) __builtin_amdgcn_sched_group_barrier(0x010, MB == 1 ? 3 : 2, 0);               // slab copies
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (FP8 && ODD) {
            const float sc[2] = {scale[0][s >> 1] * (1.0f / CODE_UNIT), scale[1][s >> 1] * (1.0f / CODE_UNIT)};
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[mb][q][v] = __builtin_fmaf(sum[FP8 ? mb : 0][FP8 ? q : 0][v], sc[q], acc[mb][q][v]);
        }
        advance(odd_tag);
    };
    // a wavefront without rows has its share of the copies and barriers only
    auto idle_slab = [&](int s, auto odd_tag, auto new_tag, auto final_tag) __attribute__((always_inline)) {
        constexpr bool NEW = decltype(new_tag)::value, FINAL = decltype(final_tag)::value;
        if (!FINAL) next_slab(s, odd_tag, new_tag);
        if (NEW) copies_of(s, odd_tag);
        advance(odd_tag);
    };
    auto all_slabs = [&](auto one) __attribute__((always_inline)) {
        const std::true_type T{};
        const std::false_type F{};
        int s = 0;
        for (; s + 1 + NST < NS; s += 2) { one(s, F, T, F); one(s + 1, T, T, F); }
        // (NS is even: 2 slabs are left, or 4; with three places slab NS - 1 is copied behind slab NS - 4)
        if (NS - s > 2) {
            if (NST == 3) one(s, F, T, F); else one(s, F, F, F);
            one(s + 1, T, F, F);
            s += 2;
        }
        one(s, F, F, F);
        one(s + 1, T, F, T);
    };
    // The first slabs, in the order of the steady state: slab k with, behind every other one, a block of codes.  (Past the end: the last ones once more.)
    if (FP8) {
#pragma unroll
        for (int i = 0; i < CB; ++i) copy_b(0, 0, i);
    }
#pragma unroll
    for (int s = 0; s < NST; ++s) {
#pragma unroll
        for (int i = 0; i < CA; ++i) copy_a(min(s, NS - 1), s, i);
        constexpr int EVEN = NST & 1;                                     // (a block follows the slabs that have as many behind them as places, up to an even number)
        if (!FP8 || ((s & 1) != EVEN && s > 0)) {
            const int b = FP8 ? (s - NST + 1) / 2 + NB - 1 : s;
#pragma unroll
            for (int i = 0; i < CB; ++i) copy_b(FP8 ? min(b, NP - 1) : min(b, NS - 1), b, i);
        }
    }
    wait_vmcnt<(NST - 1) * CA + (NB - 1) * CB>();
    lds_barrier();
    if (wm * 32 * MB < rows) {
        load_frags(0, 0, 0, 0);
        all_slabs(slab);
    } else {
        all_slabs(idle_slab);
    }
    __syncthreads();                     // the slabs' places stage the output

    // ---- a part of the contraction: its sums go to memory where every die sees them; the workgroup that finds the others there adds them up in order
    if (P > 1) {
        const int tile = nt * nblocks + blk;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)t.part, 0, 0xFFFFFFFF, 0x00020000);
        const unsigned int at = (unsigned int)(tile * P) * (unsigned int)S::UNIT_BYTES + (unsigned int)wave * (8192u * MB);
        const int live = min(MB, (rows - wm * 32 * MB + 31) / 32);        // 32-row blocks of this wavefront that hold rows (may be negative)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            if (mb < live) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const f32x4 v = {acc[mb][i >> 2][(i & 3) * 4], acc[mb][i >> 2][(i & 3) * 4 + 1], acc[mb][i >> 2][(i & 3) * 4 + 2], acc[mb][i >> 2][(i & 3) * 4 + 3]};
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, lane * 16,
                                                           at + (unsigned int)p * (unsigned int)S::UNIT_BYTES + (unsigned int)(mb * 8 + i) * 1024u, DEVICE_SCOPE);
                }
            }
        wait_vmcnt<0>();
        __syncthreads();
        int* const s_arrived = reinterpret_cast<int*>(smem);
        if (tid == 0) *s_arrived = __hip_atomic_fetch_add(&t.arrived[tile], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const int others = *s_arrived;
        __syncthreads();
        if (others != P - 1) return;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            acc[mb][0] = acc[mb][1] = f32x16{0.f};
            if (mb >= live) continue;
            for (int k = 0; k < P; ++k) {
                u32x4 v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, at + (unsigned int)k * (unsigned int)S::UNIT_BYTES + (unsigned int)(mb * 8 + i) * 1024u, DEVICE_SCOPE);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const f32x4 w = __builtin_bit_cast(f32x4, v[i]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[mb][i >> 2][(i & 3) * 4 + j] += w[j];
                }
            }
        }
    }

    // ---- output.  acc[mb][q][v]: row l31 of row block mb, column 8 * (v >> 2) + 4 * lhi + (v & 3) of column block q; through a private staging area, 32
    // rows at a time (phase 1: of 32 hidden units, phase 2: of 64 columns), so that a store covers runs of 64 or 128 bytes
    unsigned char* const stage = smem + wave * 4096;
    constexpr int SROW = PHASE == 1 ? 64 : 128, CPR = SROW / 16, RPI = 64 / CPR;
    auto swz_out = [](int r) { return (r >> 1) & (CPR - 1); };
    const int sr = lane / CPR, sc = lane % CPR;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int wrow = m0 + wm * 32 * MB + mb * 32;
        auto stage4 = [&](int q, int g, float v0, float v1, float v2, float v3) __attribute__((always_inline)) {
            *reinterpret_cast<u32x2*>(stage + l31 * SROW + (((q * 4 + g) ^ swz_out(l31)) << 4) + lhi * 8) = pack4(v0, v1, v2, v3);
        };
        auto store = [&](__bf16* base, int ld, int col, bool listed) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 32 / RPI; ++i) {
                const int r = i * RPI + sr, m = wrow + r;
                const u32x4 v = *reinterpret_cast<const u32x4*>(stage + r * SROW + ((sc ^ swz_out(r)) << 4));
                if (m < m_end) *reinterpret_cast<u32x4*>(base + (size_t)(unsigned int)(listed ? mapped_row(a, m) : m) * ld + col + sc * 8) = v;
            }
        };
        if constexpr (PHASE == 1) {
            const int col = nt * 64 + wn * 32;
            if constexpr (KIND == BWD_ACT) {
                // h, then dg = dh * u * silu'(g) and du = dh * silu(g), left in the accumulators of g and u
                const __bf16* const src = a.dh + (size_t)(unsigned int)min(wrow + l31, m_end - 1) * a.lddh + col + lhi * 4;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const bf16x4 d4 = __builtin_bit_cast(bf16x4, *reinterpret_cast<const u32x2*>(src + g * 8));
                    float hv[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float gv = acc[mb][0][g * 4 + j], uv = acc[mb][1][g * 4 + j], dv = (float)d4[j];
                        const float sig = __builtin_amdgcn_rcpf(1.0f + __expf(-gv));
                        hv[j] = (gv * sig) * uv;
                        acc[mb][0][g * 4 + j] = dv * uv * (sig * (1.0f + gv * (1.0f - sig)));
                        acc[mb][1][g * 4 + j] = dv * (gv * sig);
                    }
                    stage4(0, g, hv[0], hv[1], hv[2], hv[3]);
                }
                store(a.h, a.f, col, false);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) stage4(0, g, acc[mb][q][g * 4], acc[mb][q][g * 4 + 1], acc[mb][q][g * 4 + 2], acc[mb][q][g * 4 + 3]);
                    store(a.dgu + (q ? a.f : 0), 2 * a.f, col, false);
                }
            } else {
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    stage4(0, g, silu(acc[mb][0][g * 4]) * acc[mb][1][g * 4], silu(acc[mb][0][g * 4 + 1]) * acc[mb][1][g * 4 + 1],
                           silu(acc[mb][0][g * 4 + 2]) * acc[mb][1][g * 4 + 2], silu(acc[mb][0][g * 4 + 3]) * acc[mb][1][g * 4 + 3]);
                store(a.h, a.f, col, false);
            }
        } else {
            float gate = 1.0f;
            if (KIND == FORWARD && a.gate) gate = a.gate[min(wrow + l31, m_end - 1)];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int g = 0; g < 4; ++g) stage4(q, g, gate * acc[mb][q][g * 4], gate * acc[mb][q][g * 4 + 1], gate * acc[mb][q][g * 4 + 2], gate * acc[mb][q][g * 4 + 3]);
            store(a.g2.O, a.g2.ldo, nt * TILE + wn * 64, LISTED_OUT);
        }
    }
}

// Expands block-scaled E4M3 codes [rows][cols] to bf16, eight values per thread and step (HBM bound: 3 bytes per weight).
__global__ __launch_bounds__(256)
void ffn_expand_fp8_kernel(const unsigned char* __restrict__ codes, const float* __restrict__ scales, __bf16* __restrict__ out,
                           long long n8, int cols) {
    const int sc_cols = cols / 128;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n8; i += (long long)gridDim.x * blockDim.x) {
        const long long e = i * 8;                                     // 8 consecutive codes of one row (cols % 128 == 0)
        const long long row = e / cols;
        const int col = (int)(e - row * cols);
        const float scale = scales[(row / 128) * sc_cols + col / 128];
        const u32x2 c = *reinterpret_cast<const u32x2*>(codes + e);
        *reinterpret_cast<u32x4*>(out + e) = dequant8(c, scale);
    }
}

int plan_capacity(int M) { return M / 64 + MAX_GROUPS + 1; }
size_t h_bytes(int M, int f) { return (((size_t)M * f * 2) + 255) & ~(size_t)255; }
size_t plan_bytes(int M) { return (((size_t)(plan_capacity(M) + PLAN_HDR) * sizeof(int4)) + 255) & ~(size_t)255; }
size_t list_bytes(int M) { return ((((size_t)M + LIST_PAD) * sizeof(int32_t)) + 255) & ~(size_t)255; }
constexpr size_t EBASE_BYTES = (((size_t)MAX_GROUPS + 1) * sizeof(int) + 255) & ~(size_t)255;
size_t ready_bytes(int M) { return (((size_t)plan_capacity(M) * sizeof(int)) + 255) & ~(size_t)255; }

size_t ffn_base_bytes(int M, int f) { return h_bytes(M, f) + plan_bytes(M) + ready_bytes(M) + 2 * list_bytes(M) + EBASE_BYTES; }
constexpr int KMAJOR_ROWS = 4096;          // the K-major copy of x is for calls of at most this many rows
size_t kmajor_bytes(int M, int d) { return (((size_t)M * d * 2) + 255) & ~(size_t)255; }

std::atomic<int> g_force_rows{0};          // moe_ffn_tile_override: 0 = rows per tile chosen per call, else 64 / 128 / 256
std::atomic<int> g_force_kernels{0};       //                        1 = never the adaptive-shape kernels, 2 = adaptive-shape kernels, one launch per phase
std::atomic<int> g_force_panel{0};         //                        0 = panel width of the tile walk chosen per call, else column groups per panel
std::atomic<int> g_num_cus[64];            // compute units of device d (0 = not asked yet)
int num_cus() {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
    n = g_num_cus[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        g_num_cus[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Column groups per panel of the tile walk.  The walk sweeps a panel's weights once per row group; as long as one
// expert's weights of the phase (plus a row group's activations and results) fit the 256 MB memory-side cache with room
// to spare, one panel holds all column groups.  Beyond that every sweep would evict what the next one needs (a cyclic
// pattern just above an LRU cache's size misses every time), so the columns are split into panels of about 64 MB and
// the activations are streamed once per panel instead.
int panel_width(int units, size_t expert_weight_bytes, size_t unit_bytes) {
    const int ncg = (units + 7) / 8, cn = (units + ncg - 1) / ncg;
    if (expert_weight_bytes <= ((size_t)128 << 20)) return ncg;
    const size_t group_bytes = (size_t)cn * unit_bytes;
    const int w = (int)(((size_t)64 << 20) / (group_bytes ? group_bytes : 1));
    return w < 1 ? 1 : (w > ncg ? ncg : w);
}

// `max_tiles`: workgroups wanted, at most one per compute unit is launched
template <int PHASE, int AROWS, int OROWS, int EPI = 0>
moe_status launch_adaptive(const FfnArgs& a, long long max_tiles, hipStream_t s, const char* name = nullptr) {
    static moe::DeviceOnce attr;
    auto kern = ffn_adaptive_kernel<PHASE, AROWS, OROWS, EPI>;
    int dev;
    if (attr.needed(dev)) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, ADAPTIVE_LDS);
        if (e != hipSuccess) { moe::note_hip_error(e, "hipFuncSetAttribute(MaxDynamicSharedMemorySize)"); return MOE_ERR_HIP; }
        attr.mark(dev);
    }
    const long long slots = num_cus();
    const int grid = (int)(max_tiles < slots ? max_tiles : slots);
    moe::LaunchScope k(name ? name : (PHASE == 1 ? "ffn_gemm1_kernel" : "ffn_gemm2_kernel"), s);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NW * 64), ADAPTIVE_LDS, s, a);
    return k.done();
}

template <int ROWS>
moe_status launch_fused(const FfnArgs& a, long long max_tiles, hipStream_t s) {
    static moe::DeviceOnce attr;
    auto kern = ffn_fused_kernel<ROWS>;
    int dev;
    if (attr.needed(dev)) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, ADAPTIVE_LDS);
        if (e != hipSuccess) { moe::note_hip_error(e, "hipFuncSetAttribute(MaxDynamicSharedMemorySize)"); return MOE_ERR_HIP; }
        attr.mark(dev);
    }
    const long long slots = num_cus();
    const int grid = (int)(max_tiles < slots ? max_tiles : slots);
    moe::LaunchScope k("ffn_fused_kernel", s);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NW * 64), ADAPTIVE_LDS, s, a);
    return k.done();
}

// One workgroup per tile of the larger phase, half as many more with one expert: its row blocks make few chunks, so that more of the
// workgroups find their own queue empty and come late to the others.  us, 1 / 1.5 / 2 per tile: E 1, d 2048, f 1408, 384 / 2048
// rows 119 / 84 / 85, 132 / 96 / 103; E 1, d 1024, f 512, 2048 rows 73 / 51 / 53; E 1, d = f = 4096, 512 / 640 rows 260 / 207 / 212, 212 / 246 / 213; E 4, d = f =
// 512, 2048 rows per expert 57 / 66 / 74.  Mean over the best of the three: one expert 1.09 / 1.02 / 1.02, two 1.02 / 1.02 / 1.03, more 1.01 / 1.02 / 1.04.
// Not below d = 1024: where a tile takes a few microseconds and M may be a bound above the rows, the idle ones show (8 ranks, d 256, f 512, M
// 4096: 80 -> 82 us for the layer as a whole).
template <int ROWS>
moe_status launch_both_adaptive(const FfnArgs& a, long long max_blocks, int E_loc, hipStream_t s) {
    if (g_force_kernels.load(std::memory_order_relaxed) != 2) {
        const long long tiles = max_blocks * std::max(a.f / 128, a.d / 256);
        return launch_fused<ROWS>(a, E_loc == 1 && a.d >= 1024 ? tiles + tiles / 2 : tiles, s);
    }
    moe_status st = launch_adaptive<1, ROWS, ROWS_PLAIN>(a, max_blocks * (a.f / 128), s);
    if (st != MOE_OK) return st;
    return launch_adaptive<2, ROWS_PLAIN, ROWS>(a, max_blocks * (a.d / 256), s);
}

template <int PHASE, bool FP8, int ROWS, bool WIDE, int KIND>
moe_status launch_tile(const TileArgs& a, long long max_blocks, hipStream_t s) {
    typedef TileShape<ROWS, FP8> S;
    static moe::DeviceOnce attr;
    auto kern = ffn_tile_kernel<PHASE, FP8, ROWS, WIDE, KIND>;
    int dev;
    if (attr.needed(dev)) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
        if (e != hipSuccess) { moe::note_hip_error(e, "hipFuncSetAttribute(MaxDynamicSharedMemorySize)"); return MOE_ERR_HIP; }
        attr.mark(dev);
    }
    const long long units = std::max<long long>(max_blocks * (PHASE == 1 ? a.a.f / 64 : a.a.g2.NU * 2), a.cap > 0 ? a.slots : 0);
    moe::LaunchScope k(KIND == BWD_DH ? "ffn_bwd_dh_kernel" : KIND == BWD_ACT ? "ffn_bwd_act_kernel" : KIND == BWD_DX ? "ffn_bwd_dx_kernel"
                       : PHASE == 1 ? "ffn_gemm1_kernel" : "ffn_gemm2_kernel", s);
    hipLaunchKernelGGL(kern, dim3((unsigned int)((units + 7) / 8 * 8)), dim3(S::THREADS), S::LDS, s, a);
    return k.done();
}
// One launch; `counters`: which TILE_COUNTERS of the plan's it uses
template <int PHASE, bool FP8, int ROWS, int KIND>
moe_status launch_tiles(const FfnArgs& a, int counters, long long max_blocks, f32x4* part, size_t part_bytes, hipStream_t s) {
    typedef TileShape<ROWS, FP8> S;
    TileArgs t;
    t.a = a;
    t.part = part;
    t.slots = S::SPLIT_PER_CU * num_cus();
    t.cap = (int)std::min<size_t>(part_bytes / S::UNIT_BYTES, (size_t)t.slots);
    t.arrived = a.ready + counters * TILE_COUNTERS;
    const bool wide = (unsigned long long)a.M * (PHASE == 1 ? a.d : a.g2.K) * 2 >= 0xFFFFFF00ull;
    return wide ? launch_tile<PHASE, FP8, ROWS, true, KIND>(t, max_blocks, s) : launch_tile<PHASE, FP8, ROWS, false, KIND>(t, max_blocks, s);
}
template <bool FP8, int ROWS>
moe_status launch_both_tile(const FfnArgs& a, long long max_blocks, f32x4* part, size_t part_bytes, hipStream_t s) {
    const moe_status st = launch_tiles<1, FP8, ROWS, FORWARD>(a, 0, max_blocks, part, part_bytes, s);
    if (st != MOE_OK) return st;
    return launch_tiles<2, FP8, ROWS, FORWARD>(a, 1, max_blocks, part, part_bytes, s);
}

template <int PHASE, int W, int NC, int MT, int D, bool FP8>
moe_status launch_skinny_tiles(const SkinnyArgs& a, hipStream_t s) {
    const int strips = (PHASE == 1 ? a.f / (8 * NC) : a.d / (16 * NC));
    // The chunks of an expert's rows are spread over as many workgroups as the chip holds at once, 8 at least (M bounds the rows, they
    // may be fewer, and an expert may hold most of them); a workgroup walks on from there.
    const int resident = num_cus() * (MT == 8 ? 1 : 2);
    const long long fill = resident / ((long long)strips * a.E);
    const dim3 grid(strips, a.E, (int)std::min<long long>((a.M + 16 * MT - 1) / (16 * MT), std::max(8LL, fill)));
    moe::LaunchScope k(PHASE == 1 ? "ffn_gemm1_kernel" : "ffn_gemm2_kernel", s);
    hipLaunchKernelGGL((ffn_skinny_kernel<PHASE, W, NC, MT, D, FP8>), grid, dim3(W * 64), 0, s, a);
    return k.done();
}
template <int PHASE, int W, int NC, int D, bool FP8>
moe_status launch_skinny(const SkinnyArgs& a, hipStream_t s) {
    // (fewer rows in the whole call than a workgroup takes: the variants with fewer row tiles need fewer registers)
    if (a.M <= 16) return launch_skinny_tiles<PHASE, W, NC, 1, D, FP8>(a, s);
    if (a.M <= 32) return launch_skinny_tiles<PHASE, W, NC, 2, D, FP8>(a, s);
    // bf16: 128 rows per workgroup (one wavefront per SIMD) halve the readings of the weights, as long as enough workgroups are left for the
    // chip: for more than every other compute unit with one expert, for three units in eight with several, whose rows are unequal.
    // From more than 64 rows per expert on average; from 32 with 5 to 16 experts, the popular ones of which have several chunks of 64, and
    // where a second reading of the weights is long (a matrix of 16 MiB).  64 / 128 rows, us: E 1, d 256, f 512, 300 / 1000 rows 17 / 21, 18 / 25; E 4, d 256, f 512,
    // 75 rows per expert 16 / 19; E 8, d 256, f 512, 75 / 100 23.3 / 20.6, 25.4 / 23.8; E 8, d 512, f 1024, 35 / 50 26 / 23, 27 / 25; E 16, d 2048, f 1408, 32 / 75 / 93
    // 114 / 97, 158 / 138, 190 / 156.  In fp8 the scales of 128 rows' sums cost more than a second reading: E 16, d 2048, f 1408, 18 / 32 rows 63 / 64, 76 / 80; E 32,
    // d 2048, f 768, 18 rows 81 / 95; E 8, d 256, f 512, 37 / 100 rows 16.7 / 19.0, 21.4 / 24.3.
    if constexpr (!FP8) {
        const long long groups = (long long)a.E * (a.f / 32) * ((a.M / a.E + 127) / 128);
        const bool fills = a.E == 1 ? 2 * groups > num_cus() : 8 * groups >= 3 * num_cus();
        const bool early = a.E > 4 ? a.E <= 16 && a.M >= 32LL * a.E : a.E > 1 && a.M > 32LL * a.E && (long long)a.d * a.f >= (8LL << 20);
        if (fills && (a.M > 64LL * a.E || early)) return launch_skinny_tiles<PHASE, W, NC, 8, 2, FP8>(a, s);
    }
    return launch_skinny_tiles<PHASE, W, NC, 4, D, FP8>(a, s);
}

// Weight rows per workgroup: 64 (the 64 rows of activations are then fetched as often as the weights), but 16 in phase 2 when
// the strips of 64 would leave half the compute units idle: d = 4096, f = 14336, one expert, phase 2 at 37 rows: 64 rows 75 us,
// 16 rows 39 us; d = 7168, f = 2048, four fp8 experts, 203 rows: 28 us, 59 us.
// Up to 32 rows it is the experts that can hold rows which count, not all of them, and a strip's chain over f costs more than the activations (at most
// two 16-row tiles): 16 rows below three strips per four compute units, as long as the workgroups of the other experts are few (they leave at once, some 5 ns each).
// 64 / 16 rows, us: E 2, d 4096, f 14336, 1 / 8 rows 104 / 68, 156 / 136, in fp8 68 / 46, 96 / 83; E 8, d 1280, f 5248, 1 / 8 rows 34 / 21, 55 / 51; E 2, d 6912,
// f 3968, 1 / 8 rows (108 and 216 strips) 51 / 46, 66 / 67; E 8, d 7168, f 2048, one row (3584 workgroups) 42 / 43, in fp8 27 / 29.
int skinny_strips2(int M, int E_loc, int d) {                              // strips per expert in phase 2
    const int cus = num_cus(), wide = d / 64, narrow = d / 16;
    if ((long long)wide * E_loc < cus / 2) return narrow;
    return M <= 32 && 4LL * wide * std::min(E_loc, M) < 3LL * cus && (long long)narrow * E_loc <= 8LL * cus ? narrow : wide;
}
template <bool FP8>
moe_status launch_both_skinny(const SkinnyArgs& a, hipStream_t s) {
    moe_status st;
    if (a.xk) {
        moe::LaunchScope k("ffn_kmajor_kernel", s);
        hipLaunchKernelGGL(ffn_kmajor_kernel, dim3((a.M + 31) / 32, a.d / 64), dim3(256), 0, s, a.x, a.row_map, a.offsets + (size_t)a.S * a.E,
                           a.M, a.d, (__bf16*)a.xk);
        if ((st = k.done()) != MOE_OK) return st;
    }
    if ((st = launch_skinny<1, 4, 4, 2, FP8>(a, s)) != MOE_OK) return st;
    if (skinny_strips2(a.M, a.E, a.d) == a.d / 64) return launch_skinny<2, 4, 4, 2, FP8>(a, s);
    return launch_skinny<2, 4, 1, 4, FP8>(a, s);
}

// ---- which kernels a call takes.  Only M, an upper bound of the rows, is known here, and not how unequal the experts are.  Up to 8 experts the times
// of the ways are estimated (us) and the least is taken.  The constants were fitted to 2999 calls timed in every way (75 shapes of E 1 .. 8, d 256 .. 7168, f 256 .. 14336;
// 33 rows .. 5000 rows per expert, Zipf popularity, bf16 and fp8): the chosen way takes 1.6 % (bf16) and 0.6 % (fp8) longer than the best one on average.
// (Up to 32 rows: streams_few.)  Where M is twice the rows, bf16 calls take 4.0 % longer than in the best way.
// us, streaming / tiles of 64 / 128 / 256 rows / fused, rows in all:
//   bf16 E 1, d 4096, f 14336: 36 rows 94 87 107 94 -, 69 rows 124 97 116 97 -, 274 rows 349 218 182 160 453, 1063 rows 1089 582 453 425 578, 4497 rows - 2006 1635 1513 1456
//   bf16 E 4, d 2048, f 1408: 42 rows 23 26 35 30 -, 293 rows 51 28 38 40 -, 1449 rows 124 56 53 51 116, 5042 rows - 137 114 112 148, 16073 rows - 374 299 313 273
//   fp8  E 4, d 7168, f 2048: 40 rows 49 45 59, 310 rows 118 72 79, 1028 rows 287 155 159, 3851 rows 919 435 371, 15617 rows - 1597 1376
enum Route { STREAM, TILE_64, TILE_128, TILE_256, FUSED, EXPAND };         // (EXPAND: fp8 weights to bf16, then fused)
struct Estimate {
    // Tiles of 64, 128 and (bf16) 256 rows: us per slab of 64 values of K, per tile besides, share of a full round that an empty one takes, us per phase with split contractions;
    // us per phase with whole ones, share of a round that does not end with the others; us per call and MB/us of the weights' way from memory
    double slab[3], tile[3], least[3], split[3], whole, spread, open, bytes;
    // Streaming: us per phase and MB/us of the weights' way from memory; us per phase at least, per 64 values of K with strips of 64 and of 16 rows, share per 16-row
    // tile; us per row and 10^8 weights of a matrix
    double stream_open, stream_bytes, chain, wide, narrow, row_tile, rows;
};
constexpr Estimate ESTIMATE[2] = {{{0.749, 1.19, 0.809}, {0.332, 1.57, 6.04}, {0.268, 0.325, 0.471}, {6.22, 15, 11}, 7.17, 0.713, 12.7, 3.7, 1.79, 3.84, 6.7, 0.179, 0.0144, 0.212, 3.27},        // bf16
                                  {{0.635, 0.968}, {0.87, 2.37}, {0.306, 0.266}, {12.9, 17.8}, 6.95, 0.843, 11.7, 4.31, 3.73, 3.65, 7.08, 0.101, 0.00953, 0.323, 2.49}};       // fp8
size_t tile_part_bytes(int d, int f) { return std::max(d, f) / 64 < 2 * TILE_MIN_SLABS ? 0 : (size_t)TILE_COUNTERS * TileShape<128, false>::UNIT_BYTES; }
double experts_with_rows(int M, int E_loc) { return (double)E_loc * M / (M + E_loc - 1); }       // (about, with Zipf popularity)
// of two times of which one hides behind the other, less so where both are about as long
double overlapped(double a, double b) {
    const double ratio = std::min(a, b) / std::max(a, b);
    return std::max(a, b) * std::pow(1.0 + std::pow(ratio, 6.0), 1.0 / 6.0);
}
// Tiles: rounds of the units the chip holds at once, times what a unit takes on a full chip.  An expert's last block is half full; the parts of a round that is not full count
// less (the compute units hold one workgroup instead of two, or wait less for memory).
double tile_us(int M, int E_loc, int d, int f, bool fp8, int rows, int cus) {
    const Estimate& c = ESTIMATE[fp8];
    const int k = rows == 64 ? 0 : (rows == 128 ? 1 : 2);
    const double blocks = E_loc == 1 ? (M + rows - 1) / rows : std::max<double>(std::min(E_loc, M), (double)M / rows + 0.5 * E_loc);
    const int slots = (rows == 256 ? 1 : 2) * cus, split_slots = (rows == 128 ? 2 : 1) * cus;
    double us = 0.0;
    for (int phase = 1; phase <= 2; ++phase) {
        const int K = phase == 1 ? d : f;
        const double tiles = blocks * (phase == 1 ? f / 64 : d / TILE);
        const int P = tile_parts((long long)(tiles + 0.5), split_slots, K, split_slots);
        const double full = tiles * P / slots;
        us += (full <= 1.0 ? c.least[k] + (1.0 - c.least[k]) * full : c.spread * full + (1.0 - c.spread) * std::ceil(full)) * (K / 64.0 / P * c.slab[k] + c.tile[k]) +
              (P > 1 ? c.split[k] : c.whole);
    }
    const double weights = 3.0 * experts_with_rows(M, E_loc) * d * f * (fp8 ? 1e-6 : 2e-6);
    return overlapped(us, c.open + weights / c.bytes);
}
// fused: the same with tiles of 256 x 256 and one round at least per phase
double fused_us(int M, int E_loc, int d, int f, int cus) {
    const double blocks = E_loc == 1 ? (M + 255) / 256 : (double)M / 256 + 0.5 * E_loc;
    double us = 44.6;
    for (int phase = 1; phase <= 2; ++phase) {
        const double full = blocks * (phase == 1 ? f / 128 : d / 256) / cus;
        us += (full <= 1.0 ? 1.0 : 0.884 * full + 0.116 * std::ceil(full)) * ((phase == 1 ? d : f) / 64 * 1.65 + 2.3);
    }
    return us;
}
// expansion of fp8 weights: 3 bytes of traffic per weight
double expand_us(int E_loc, int d, int f) { return 6.0 + 1.59e-6 * E_loc * d * f; }
// streaming: per phase the weights' way from memory or the chain over K of a strip, which gets longer with the rows of the most popular expert (Zipf, up to four
// 16-row tiles at once), and every strip reads all activations
double stream_us(int M, int E_loc, int d, int f, bool fp8) {
    const Estimate& c = ESTIMATE[fp8];
    double popular = 0.0;
    for (int e = 1; e <= E_loc; ++e) popular += std::pow(e, -1.2);
    const double chain = 1.0 + c.row_tile * std::min(4.0, std::ceil(M / popular / 16.0));
    const double matrix = experts_with_rows(M, E_loc) * d * f * (fp8 ? 1e-6 : 2e-6);
    const bool narrow = skinny_strips2(M, E_loc, d) != d / 64;
    return std::max(c.stream_open + 2.0 * matrix / c.stream_bytes, c.chain + c.wide * (d / 64) * chain) +
           std::max(c.stream_open + matrix / c.stream_bytes, c.chain + (narrow ? c.narrow : c.wide) * (f / 64) * chain) + 1e-8 * c.rows * M * d * f;
}
// More than 8 experts: a popular expert's rows are chunks behind each other that each read its weights, so at most 3072 rows are streamed (E 16, d = f = 256,
// Zipf, 4096 rows 59 / 40, 8192 rows 98 / 42), in bf16 up to a constant over the column tiles and at least 64 rows per expert, in fp8 up to 32 (E 16, d 2048, f 1408, 553 /
// 1365 / 2227 rows streamed 85 / 134 / 180 us, in tiles 48 / 62 / 82; E 32, d 2048, f 768, 2192 rows 182, 66); and as every expert gets
// workgroups for up to 8 chunks, most of which find no rows (some 5 ns each on the whole chip), a limit to those beyond the first.
bool streams_many(int M, int E_loc, int d, int f, bool fp8) {
    const long long col_tiles = (long long)E_loc * (d / 256 + f / 128);
    const long long most = fp8 ? 32LL : std::min(384LL, std::max(64LL, 36000 / col_tiles));
    if (M > most * E_loc && !(M <= 2048 && (long long)M * d * f <= (1LL << 30))) return false;
    const long long strips = f / 32 + skinny_strips2(M, E_loc, d);
    const long long spare = E_loc * strips * (std::min(8, (M + 63) / 64) - 1);
    return M <= 3072 && spare <= (fp8 ? 64 : 36) * (long long)num_cus();
}
// Up to 32 rows in the whole call (one or two 16-row tiles per strip) rows are so few that the experts which hold any count, about E M / (M + E - 1) of them with
// Zipf popularity.  Streaming: per phase the weights' way from memory or the chain over K of a strip, which is four times as long for strips of 64 rows.  Tiles:
// per phase what a launch takes to open, multiply and add up, or the weights' way from memory.  Fitted to 540 calls (E 1 .. 8, d 256 .. 7168, f 256 ..
// 14336, weights not in any cache): the chosen way takes 0.6 % longer than the better one on average, 1.27 times at most (5 to 8 rows for eight fp8 experts); with
// the estimates above it took 3.4 % longer, 1.43 times at most.  Streaming / tiles, us: E 1, d 7168, f 2048, 3 rows 40 / 33, in fp8 26 / 30; E 2, d 5376, f 640, 8
// rows 31 / 23, in fp8 22 / 24; E 1, d 4096, f 14336, 12 rows 73 / 82, in fp8 51 / 54; E 4, d 7168, f 2048, 24 rows 71 / 77, in fp8 48 / 46.
struct FewRows {
    double open, bytes, wide, narrow, least, rows;         // streaming: us per phase, MB/us, us per 64 values of K with strips of 64 and 16 rows, us at least, share per 32 rows
    double slab, split, whole, tile_open, tile_bytes;      // tiles: us per slab, us per phase with split and whole contractions; us per call, MB/us
};
constexpr FewRows FEW_ROWS[2] = {{4.88, 5.29, 0.218, 0.0343, 5.92, 0.151, 0.25, 10.3, 7.24, 12.9, 4.9},          // bf16
                                 {3.88, 4.26, 0.115, 0.028, 5.85, 0.247, 0.25, 12.1, 9.05, 10.2, 4.06}};        // fp8
bool streams_few(int M, int E_loc, int d, int f, bool fp8) {
    const FewRows& c = FEW_ROWS[fp8];
    const int cus = num_cus();
    const double experts = experts_with_rows(M, E_loc);
    const double matrix = experts * d * f * (fp8 ? 1e-6 : 2e-6);
    const bool narrow = skinny_strips2(M, E_loc, d) != d / 64;
    const double stream = (std::max(c.open + 2.0 * matrix / c.bytes, c.least + c.wide * (d / 64)) +
                           std::max(c.open + matrix / c.bytes, c.least + (narrow ? c.narrow : c.wide) * (f / 64))) * (1.0 + c.rows * M / 32.0);
    double tiles = 0.0;
    for (int phase = 1; phase <= 2; ++phase) {
        const int K = phase == 1 ? d : f;
        const double n = experts * (phase == 1 ? f / 64 : d / TILE);
        const int P = tile_parts((long long)(n + 0.5), cus, K, cus);
        const double full = n * P / (2.0 * cus);
        tiles += (full <= 1.0 ? std::max(full, 0.55) : 0.7 * full + 0.3 * std::ceil(full)) * (K / 64.0 / P) * c.slab + (P > 1 ? c.split : c.whole);
    }
    return stream <= overlapped(tiles, c.tile_open + 3.0 * matrix / c.tile_bytes);
}
// `room`: for the expanded weights, which are not made below 2048 rows per expert
Route route(int M, int S, int E_loc, int d, int f, bool fp8, bool room) {
    // (streaming: 32-bit offsets into x and h; every workgroup scans the slices of its expert)
    const bool can_stream = S <= SKINNY_MAX_SLICES && E_loc <= 4096 && (unsigned long long)M * std::max(d, f) * 2 < 0xFFFFFF00ull;
    if (E_loc > 8 && can_stream && streams_many(M, E_loc, d, f, fp8)) return STREAM;
    if (E_loc <= 8 && can_stream && M <= 32) return streams_few(M, E_loc, d, f, fp8) ? STREAM : TILE_64;
    const int cus = num_cus();
    Route best = TILE_64;
    double least = tile_us(M, E_loc, d, f, fp8, 64, cus);
    auto consider = [&](Route r, double us) { if (us < least) { least = us; best = r; } };
    consider(TILE_128, tile_us(M, E_loc, d, f, fp8, 128, cus));
    if (!fp8) consider(TILE_256, tile_us(M, E_loc, d, f, fp8, 256, cus));
    // (below 256 rows per expert the fused kernel was never the best one; f >= 256: it chains tiles over their last two slabs and needs four)
    if (!fp8 && f >= 256 && M >= 256LL * E_loc) consider(FUSED, fused_us(M, E_loc, d, f, cus));
    if (fp8 && f >= 256 && M >= 2048LL * E_loc && room) consider(EXPAND, expand_us(E_loc, d, f) + fused_us(M, E_loc, d, f, cus));
    if (E_loc <= 8 && can_stream) consider(STREAM, stream_us(M, E_loc, d, f, fp8));
    return best;
}

// the choice that moe_ffn_tile_override has pinned, if any
Route pinned(Route way, int f, bool fp8) {
    const int rows = g_force_rows.load(std::memory_order_relaxed);
    if (rows != 0) way = rows == 64 ? TILE_64 : (rows == 128 || fp8 ? TILE_128 : (f < 256 ? TILE_256 : FUSED));
    return way == FUSED && g_force_kernels.load(std::memory_order_relaxed) == 1 ? TILE_256 : way;
}

moe_status launch_plan(const PlanArgs& p, hipStream_t s) {
    if (!p.bases && small_plan(p.M, p.S, p.e_loc)) {
        moe::LaunchScope k("ffn_small_plan_kernel", s);
        hipLaunchKernelGGL(ffn_small_plan_kernel, dim3(1), dim3(PLAN_THREADS), 0, s, p);
        return k.done();
    }
    // one workgroup per 8192 list entries, at most 64: each scans the groups anew
    const int blocks = p.list ? std::min(64, p.M / (8 * PLAN_THREADS) + 1) : 1;
    moe::LaunchScope k("ffn_plan_kernel", s);
    hipLaunchKernelGGL(ffn_plan_kernel, dim3(blocks), dim3(PLAN_THREADS), 0, s, p);
    return k.done();
}

// ---------------------------------------------------------------------------------- backward pass: weight gradients
// dW_gate = dg^T x, dW_up = du^T x, dW_down = dy^T h: contractions over the rows of an expert, whose operands all lie with a row's features
// side by side, i.e. with the contraction as the slow dimension.  K slabs of 64 rows x 256 features (512-byte rows: whole cache lines) go
// global -> LDS as they lie, and the MFMA fragments are read with ds_read_b64_tr_b16, which hands lane c of 16 the values of four rows
// in column c.  x and dy are gathered through the row list by the copies themselves (a row number is a scalar load, one slab
// ahead); rows past an expert's end lie behind the buffer descriptor, for which the copy deposits zeros.
// Bound by the matrix cores (busy 69 % of the cycles in which a compute unit has work, 57 % of the launch's; 1.03 PFLOP/s) and, beside them, by unequal experts.  E 4, d 2048,
// f 1408, 36833 rows: 620 us, whole backward pass 1654; with transposed copies of x, dy, h, dg and du (295 us), three launches of the row GEMM that each waited for the most popular
// expert (797) and partial sums rounded to bf16 and added in three more (110) 2327.  E 1, d 4096, f 14336, 6000 rows: 1620 us, before 2480.
// All products and experts are one launch, the longest contractions first.  A unit of work is a 256 x 256 tile of one expert's [dW_gate; dW_up] or
// dW_down over one part of its rows; only experts behind which too little work is left to even out the ends are split (parts.hpp).
// Parts are added in fp32 in part order by the workgroup that finishes a tile's last part.
constexpr size_t DW_UNIT_BYTES = 256 * 256 * sizeof(float);
constexpr int DW_QUEUES = 24;                  // first of the 8 queue counters of the weight gradients
constexpr int BWD_COUNTERS = 32;               // tile queue counters of a backward call: dh, act, dx, dW
constexpr int DW_ZEROS = 1024;                 // bytes of zeros that rows past an expert's end read where the operands need 64-bit addresses

constexpr int DW_CHUNK = 5;                    // log2 of the largest chunk of tiles
struct DwGrid {                                // tiles of one product of one expert, walked in chunks of at most 32 for the workgroups of one L2
    int C, CN, RB, R, ncg, chunks;
    __host__ __device__ __forceinline__ void init(int rows, int cols) {
        R = rows; C = cols;
        ncg = (C + 7) / 8;
        CN = (C + ncg - 1) / ncg;
        RB = 32 / CN;
        chunks = (R + RB - 1) / RB * ncg;
    }
    __device__ __forceinline__ bool at(int chunk, int j, int& r, int& c) const {
        const int rg = chunk / ncg, cg = chunk - rg * ncg;
        r = rg * RB + j / CN;
        c = cg * CN + j % CN;
        return j < RB * CN && r < R && c < C;
    }
};
// log2 of the tickets of a chunk, which hold either product's tiles: with 32 for few tiles per expert most tickets are empty, an atomic operation each.  E 64 / 1024 / 4096,
// d = f = 256, 20000 rows: 83 -> 40, 778 -> 111, 3011 -> 371 us; E 1, d 256, f 512, 26206 rows in 32 parts 139 -> 125.
int dw_tickets(int d, int f) {
    DwGrid g[2];
    g[0].init(f / 128, d / 256);
    g[1].init(d / 256, (f + 255) / 256);
    int shift = 0;
    for (const DwGrid& p : g)
        while ((1 << shift) < std::min(p.R, p.RB) * p.CN) ++shift;
    return shift;
}
__host__ __device__ inline int dw_tiles(int d, int f) { return f / 128 * (d / 256) + d / 256 * ((f + 255) / 256); }       // per expert

struct DwArgs {
    const __bf16 *x, *dy;              // [M][d], rows listed (or in order)
    const __bf16 *dgu, *h;             // [M][2 f], [M][f] in position order
    const int32_t* list;
    const int4* entries;               // [0].x = number; then per part of an expert's rows (position, rows, expert, part), (parts, first unit, 0, 0)
    int* queues;
    int* arrived;                      // [units] parts of the tile that are done (at the tile's first unit)
    f32x4* part;                       // [units][256 * 256 / 4]
    const unsigned char* zeros;
    __bf16 *dwg, *dwu, *dwd;
    int M, d, f, tickets;              // (dw_tickets)
};

// One workgroup: the table of the weight gradients' parts (parts.hpp), and what has to be zero behind it
__global__ __launch_bounds__(PLAN_THREADS)
void bwd_prep_kernel(const int* __restrict__ bases, int e_loc, int tiles, int cus, int cap, int4* __restrict__ entries, int* __restrict__ counters,
                     int* __restrict__ arrived, unsigned int* __restrict__ zeros) {
    __shared__ int rows[DW_MAX_EXPERTS], order[DW_MAX_EXPERTS], parts[DW_MAX_EXPERTS], sums[PLAN_THREADS];
    const int tid = threadIdx.x;
    for (int i = tid; i < BWD_COUNTERS; i += PLAN_THREADS) counters[i] = 0;
    for (int i = tid; i < cap; i += PLAN_THREADS) arrived[i] = 0;
    for (int i = tid; i < DW_ZEROS / 4; i += PLAN_THREADS) zeros[i] = 0;
    dw_split(bases, e_loc, tiles, cus, cap, entries, rows, order, parts, sums, tid, PLAN_THREADS, [] { __syncthreads(); });
}

// FEW: chunks of fewer than 32 tickets (a number read at run time moves enough scalar registers in the slab loop to cost the other calls 2 %)
template <bool LISTED, bool WIDE, bool FEW>
__global__ __launch_bounds__(512, 1)
void ffn_bwd_dw_kernel(DwArgs a) {
    constexpr int ROWB = 512, OPERAND = 64 * ROWB, SLAB = 2 * OPERAND;    // bytes of a slab row, of an operand's slab, of both
    constexpr int LPS = 8, NSTORE = 16;                                   // copies per wavefront and slab, stores per wavefront and tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // next unit (entry, product, row tile, column tile; entry -1 = none).  Shares its bytes with wavefront 0's output staging: written by that wavefront
    // after its read-out, read by all between the two barriers ahead of the next one.
    int* const s_ticket = reinterpret_cast<int*>(smem + STAGE_OFF);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;                              // 4 x 2 wavefronts of 64 x 128
    const int l31 = lane & 31, lhi = lane >> 5;
    const int my_xcd = blockIdx.x & 7;

    typedef const __attribute__((address_space(4))) int* scalar_ints;
    auto fetch = [&]() __attribute__((always_inline)) {
        int q = my_xcd, entry = -1, product = 0, r = 0, c = 0;
        DwGrid gu, dn;                                                    // tiles of [dW_gate; dW_up] (2 f rows, d columns) and of dW_down (d rows, f columns)
        gu.init(a.f / 128, a.d / 256);
        dn.init(a.d / 256, (a.f + 255) / 256);
        const int per = gu.chunks + dn.chunks, n_chunks = ((scalar_ints)a.entries)[0] * per;
        for (int tries = 0; tries < 8;) {
            const int shift = FEW ? a.tickets : DW_CHUNK, k = atomicAdd(&a.queues[q], 1), chunk = (k >> shift) * 8 + q, j = k & ((1 << shift) - 1);
            if (chunk >= n_chunks) { ++tries; q = (q + 1) & 7; continue; }
            const int en = chunk / per, rem = chunk - en * per;
            product = rem >= gu.chunks;
            const bool tile = product ? dn.at(rem - gu.chunks, j, r, c) : gu.at(rem, j, r, c);
            if (tile && ((scalar_ints)a.entries)[4 * (1 + 2 * __builtin_amdgcn_readfirstlane(en)) + 2] >= 0) { entry = en; break; }
        }
        s_ticket[0] = entry; s_ticket[1] = product; s_ticket[2] = r; s_ticket[3] = c;
    };
    if (tid == 0) fetch();
    __syncthreads();
    if (s_ticket[0] < 0) return;

    // ---- per-unit state.  "Plain" operand: dgu or h, rows in position order; "listed" operand: x or dy.  What only the read-out needs is
    //      looked up again there (scalar registers are short).
    int entry = 0, row_tile = 0, col_tile = 0, product = 0, pos0 = 0, rows = 0;
    unsigned long long pbase = 0, lbase = 0;           // first row and first column of the plain operand, first column of the listed one
    unsigned int lbytes = 0;                           // of the listed operand from there
    // Byte offsets of the 16-byte pieces this lane copies: row 8 * wave + 2 * i + lhi of a slab, piece l31.  64-byte unit c of row r sits at position
    // c ^ (r & 3), so that the four rows and two units that 32 lanes of a transposed read touch lie in different banks
    unsigned int pvoff[4], lvoff[LISTED ? 2 : 4];
    auto setup = [&]() __attribute__((always_inline)) {
        entry = __builtin_amdgcn_readfirstlane(s_ticket[0]);
        product = __builtin_amdgcn_readfirstlane(s_ticket[1]);
        row_tile = __builtin_amdgcn_readfirstlane(s_ticket[2]); col_tile = __builtin_amdgcn_readfirstlane(s_ticket[3]);
        const scalar_ints t = (scalar_ints)a.entries + 4 * (1 + 2 * entry);
        pos0 = t[0]; rows = t[1];
        const int pc = 256 * (product ? col_tile : row_tile), lc = 256 * (product ? row_tile : col_tile);
        const unsigned int ppitch = (unsigned int)(product ? a.f : 2 * a.f) * 2u, lpitch = (unsigned int)a.d * 2u;
        pbase = (unsigned long long)(product ? a.h : a.dgu) + (unsigned long long)(unsigned int)pos0 * ppitch + (unsigned int)pc * 2u;
        lbase = (unsigned long long)(product ? a.dy : a.x) + (unsigned int)lc * 2u;
        if (!LISTED) lbase += (unsigned long long)(unsigned int)pos0 * lpitch;
        lbytes = (unsigned int)a.M * lpitch - (unsigned int)lc * 2u;      // (read where M * d * 2 < 2^32 only)
        const bool half = product && pc + 128 >= a.f;                     // only the first 128 columns exist: the others repeat them and are not stored
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int u = (l31 >> 2) ^ (2 * (i & 1) + lhi);
            const unsigned int row = (unsigned int)(8 * wave + 2 * i + lhi);
            pvoff[i] = row * ppitch + (unsigned int)((half ? u & 3 : u) * 64 + (l31 & 3) * 16);
            if (!LISTED || i < 2) lvoff[i] = (LISTED ? 0u : row * lpitch) + (unsigned int)(u * 64 + (l31 & 3) * 16);
        }
    };
    int lr[8];                                                            // rows of the listed operand that this wavefront copies next
    auto list_rows = [&](int s) __attribute__((always_inline)) {
        if constexpr (LISTED) {
            const scalar_ints l = (scalar_ints)a.list + __builtin_amdgcn_readfirstlane(pos0 + min(s * 64 + 8 * wave, rows));   // (the list goes on for LIST_PAD entries)
#pragma unroll
            for (int k = 0; k < 8; ++k) lr[k] = l[k];
        }
    };
    // Copies are written out: the compiler would hold every transposed read of LDS until all copies in flight have landed.  (No register
    // but m0 is written; the waits that cover the copies are wait_vmcnt's.  The five wait states between a scalar register that a vector
    // instruction has written, as one that was kept in a vector lane, and a memory instruction that reads it are not counted into assembly by the
    // compiler: they stand in the text.)
    auto copy = [&](unsigned long long base, unsigned int bytes, unsigned int voff, int to) __attribute__((always_inline)) {
        const u32x4 rs = {(unsigned int)base, (unsigned int)(base >> 32), bytes, 0x00020000u};
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(to), "v"(voff), "s"(rs) : "memory", "m0");
    };
    auto slab_bytes = [&](int s, unsigned int pitch) __attribute__((always_inline)) -> unsigned int {       // rows past the end: zeros are deposited
        const int left = min(rows - s * 64, 64);
        return left > 0 ? (unsigned int)(left - 1) * pitch + 512u : 0u;
    };
    const int lds0 = (int)(unsigned int)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem + wave * (8 * ROWB);
    auto copy_plain = [&](int s, int buf, int i) __attribute__((always_inline)) {
        const unsigned int pitch = (unsigned int)(product ? a.f : 2 * a.f) * 2u;
        copy(pbase + (unsigned long long)(unsigned int)(s * 64) * pitch, slab_bytes(s, pitch), pvoff[i], lds0 + buf * SLAB + 2 * i * ROWB);
    };
    auto copy_listed = [&](int s, int buf, int i) __attribute__((always_inline)) {
        const unsigned int pitch = (unsigned int)a.d * 2u;
        const int to = lds0 + buf * SLAB + OPERAND + 2 * i * ROWB;
        if constexpr (!LISTED) {
            copy(lbase + (unsigned long long)(unsigned int)(s * 64) * pitch, slab_bytes(s, pitch), lvoff[i], to);
        } else {
            const unsigned int row = (unsigned int)(lhi ? lr[2 * i + 1] : lr[2 * i]);
            const bool live = s * 64 + 8 * wave + 2 * i + lhi < rows;
            if constexpr (WIDE) {
                const unsigned char* const from = live ? (const unsigned char*)lbase + (unsigned long long)row * pitch + lvoff[i & 1] : a.zeros + l31 * 16;
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(to), "v"(from) : "memory", "m0");
            } else {
                copy(lbase, lbytes, live ? row * pitch + lvoff[i & 1] : 0xFFFFFF00u, to);
            }
        }
    };
    auto prologue = [&]() __attribute__((always_inline)) {                // slabs 0 and 1 (past the end: zeros, from no memory)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            list_rows(s);
#pragma unroll
            for (int i = 0; i < 4; ++i) copy_plain(s, s, i);
#pragma unroll
            for (int i = 0; i < 4; ++i) copy_listed(s, s, i);
        }
        list_rows(2);
    };
    // fragment of 32 columns x 16 rows: two transposed reads of 4 rows each; lane -> rows 8 * lhi + 4 * j + (lane & 15) / 4, columns
    // 16 * (lane / 16 & 1) + 4 * (lane & 3) of the block
    const int frag = (8 * lhi + ((lane & 15) >> 2)) * ROWB + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    const int sw = (lane >> 2) & 3;
    int foff[6];                                                          // 4 column blocks of the n operand, 2 of the m operand
#pragma unroll
    for (int q = 0; q < 4; ++q) foff[q] = frag + (((wn * 4 + q) ^ sw) << 6);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) foff[4 + mb] = frag + (((wm * 2 + mb) ^ sw) << 6);

    bool counted = false;
    setup();
    prologue();
    while (true) {
        f32x16 acc[2][4];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mb][q][v] = 0.f;
        // issued so far, oldest first: slab 0, slab 1, the output of the unit before
        if (counted) wait_vmcnt<LPS + NSTORE>(); else wait_vmcnt<LPS>();
        lds_barrier();
        const int n_area = product ? 0 : OPERAND, m_area = OPERAND - n_area, NS = (rows + 63) >> 6;
        auto load_frag = [&](bf16x8& to, int i, int buf, int u) __attribute__((always_inline)) {
            typedef __attribute__((address_space(3))) bf16x4* lds4;
            unsigned char* const at = smem + foff[i] + buf * SLAB + (i < 4 ? n_area : m_area) + u * 16 * ROWB;
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds4)at), hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds4)(at + 4 * ROWB));
            to = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        };
        bf16x8 frags[2][6];
#pragma unroll
        for (int i = 0; i < 6; ++i) load_frag(frags[0][i], i, 0, 0);
        // Slab s.  The barrier ahead of its last K step publishes slab s + 1 and frees its own buffer, into which the plain operand of slab s + 2
        // (NEW) is copied at once; the listed operand follows in the first K step of the next slab (OLD: slab s + 1's half is due here).
        auto slab = [&](int s, auto new_tag, auto old_tag, auto final_tag) __attribute__((always_inline)) {
            constexpr bool NEW = decltype(new_tag)::value, OLD = decltype(old_tag)::value, FINAL = decltype(final_tag)::value;
            const int buf = s & 1;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int cur = u & 1, nxt = cur ^ 1;
                const bool last = u == 3, reads = !(last && FINAL);
                if (last && !FINAL) { wait_vmcnt<0>(); lds_barrier(); }
                const int rbuf = last ? buf ^ 1 : buf, ru = last ? 0 : u + 1;
                const bool copies = last ? NEW : (OLD && u == 0);
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    if (reads) load_frag(frags[nxt][i], i, rbuf, ru);
                    if (copies && i < 4) { if (last) copy_plain(s + 2, buf, i); else copy_listed(s + 1, buf ^ 1, i); }
                }
                if (OLD && u == 0) list_rows(s + 2);
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[mb][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frags[cur][q], frags[cur][4 + mb], acc[mb][q], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                     // MFMA
                    if (reads && i < 6) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);                 // LDS reads
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        {
            const std::true_type T{};
            const std::false_type F{};
            const int draw = max(NS - 5, 0);                              // (late: the longest contractions come first, and a unit drawn early waits for its holder)
            if (draw == 0 && tid == 0) fetch();
            if (NS > 2)       slab(0, T, F, F);
            else if (NS == 2) slab(0, F, F, F);
            int s = 1;
            for (; s + 2 < NS; ++s) {
                if (s == draw && tid == 0) fetch();
                slab(s, T, T, F);
            }
            if (NS > 2) slab(NS - 2, F, T, F);
            if (NS > 0) slab(NS - 1, F, F, T);
        }
        lds_barrier();                   // every fragment is in registers: both buffers are free; the next ticket is visible
        const int eentry = entry, erow = row_tile, ecol = col_tile, eproduct = product;
        const bool more = __builtin_amdgcn_readfirstlane(s_ticket[0]) >= 0;
        if (more) { setup(); prologue(); }                                // the next unit's first slabs fly during the read-out
        lds_barrier();                   // the ticket has been read: its bytes may stage output

        // ---- a part: its sums go to memory where every die sees them; the workgroup that finds the others there adds them up, in part order
        const scalar_ints t = (scalar_ints)a.entries + 4 * (1 + 2 * eentry);
        const int ee = t[2], epart = t[3], eparts = t[4];
        bool store = true;
        counted = false;
        if (eparts > 1) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.part, 0, 0xFFFFFFFF, 0x00020000);
            const int eunit = t[5] + (eproduct ? a.f / 128 * (a.d / 256) + erow * ((a.f + 255) / 256) + ecol : erow * (a.d / 256) + ecol) * eparts;
            const unsigned int first = (unsigned int)eunit * (unsigned int)DW_UNIT_BYTES + (unsigned int)wave * 32768u;
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 v = {acc[mb][q][g * 4], acc[mb][q][g * 4 + 1], acc[mb][q][g * 4 + 2], acc[mb][q][g * 4 + 3]};
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, lane * 16,
                                                               first + (unsigned int)epart * (unsigned int)DW_UNIT_BYTES + (unsigned int)((mb * 4 + q) * 4 + g) * 1024u, DEVICE_SCOPE);
                    }
            wait_vmcnt<0>();
            lds_barrier();
            if (tid == 0) s_ticket[0] = __hip_atomic_fetch_add(&a.arrived[eunit], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            lds_barrier();
            store = __builtin_amdgcn_readfirstlane(s_ticket[0]) == eparts - 1;
            lds_barrier();
            if (store) {
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        f32x16 sum;
#pragma unroll
                        for (int v = 0; v < 16; ++v) sum[v] = 0.f;
                        for (int p = 0; p < eparts; p += 4) {             // (four parts' loads in flight: each is a round trip to where every die sees them)
                            f32x4 v[4][4];
#pragma unroll
                            for (int i = 0; i < 4; ++i)
#pragma unroll
                                for (int g = 0; g < 4; ++g)
                                    v[i][g] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16,
                                                  first + (unsigned int)min(p + i, eparts - 1) * (unsigned int)DW_UNIT_BYTES + (unsigned int)((mb * 4 + q) * 4 + g) * 1024u, DEVICE_SCOPE));
#pragma unroll
                            for (int i = 0; i < 4; ++i) {                 // (every load is used: one left behind would be waited for among the next unit's copies)
                                const bool live = p + i < eparts;
#pragma unroll
                                for (int g = 0; g < 4; ++g)
#pragma unroll
                                    for (int k = 0; k < 4; ++k) sum[g * 4 + k] += live ? v[i][g][k] : 0.f;
                            }
                        }
                        acc[mb][q] = sum;
                    }
            }
        }
        if (store) {
            // acc[mb][q][v]: row l31 of row block mb, column 8 * (v >> 2) + 4 * lhi + (v & 3) of column block q: 32 rows x 64 columns at a time
            // through a private staging area, so that whole cache lines are stored
            int lane_e = lane;
            asm volatile("" : "+v"(lane_e));                              // (address arithmetic stays here)
            const int el31 = lane_e & 31, elhi = lane_e >> 5, sr = lane_e >> 3, sc = lane_e & 7;
            auto swz = [](int r) { return (r >> 1) & 7; };
            unsigned char* const stage = smem + STAGE_OFF + wave * STAGE_WAVE;
            unsigned char* const wr = stage + el31 * 128 + elhi * 8;
            const int row = erow * 256 + wm * 64, col = ecol * 256 + wn * 128;
            __bf16* out;
            if (eproduct)       out = a.dwd + ((size_t)ee * a.d + row) * a.f + col;
            else if (row < a.f) out = a.dwg + ((size_t)ee * a.f + row) * a.d + col;       // (f is a multiple of 128: a wavefront's rows are all of one matrix)
            else                out = a.dwu + ((size_t)ee * a.f + row - a.f) * a.d + col;
            const int pitch = (eproduct ? a.f : a.d) * 2;
            const unsigned long long ob = (unsigned long long)out;
            const unsigned int ob_lo = (unsigned int)__builtin_amdgcn_readfirstlane((unsigned int)ob);
            const unsigned int ob_hi = (unsigned int)__builtin_amdgcn_readfirstlane((unsigned int)(ob >> 32));
            const bool exists = !eproduct || col < a.f;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(((unsigned long long)ob_hi << 32) | ob_lo), 0,
                                                                                __builtin_amdgcn_readfirstlane(exists ? 64 * pitch : 0), 0x00020000);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
                for (int hq = 0; hq < 2; ++hq) {
#pragma unroll
                    for (int q = 0; q < 2; ++q)
#pragma unroll
                        for (int g = 0; g < 4; ++g)
                            *reinterpret_cast<u32x2*>(wr + (((q * 4 + g) ^ swz(el31)) << 4)) =
                                pack4(acc[mb][hq * 2 + q][g * 4], acc[mb][hq * 2 + q][g * 4 + 1], acc[mb][hq * 2 + q][g * 4 + 2], acc[mb][hq * 2 + q][g * 4 + 3]);
                    u32x4 v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const u32x4*>(stage + (i * 8 + sr) * 128 + ((sc ^ swz(i * 8 + sr)) << 4));
#pragma unroll
                    for (int i = 0; i < 4; ++i) __builtin_amdgcn_raw_buffer_store_b128(v[i], rs, (mb * 32 + i * 8 + sr) * pitch + hq * 128 + sc * 16, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            counted = eparts == 1;
        }
        if (!more) break;
    }
}

__global__ void bwd_zero_kernel(unsigned int* __restrict__ p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

// The weights as the backward pass's row products need them (K contiguous), all three of all experts in one launch:
// w_down [E][d][f] -> wdt [E][f_pad][d] (rows f .. f_pad - 1 zero);  w_gate, w_up [E][f][d] -> wgut [E][d][2 f] = [gate^T | up^T].
// HBM bound: 64 x 64 blocks through LDS, 16 bytes per lane both ways (with 2 bytes per lane, in three
// launches: E 4, d 2048, f 1408, 69 MB each way, 76 us, now 27; E 1, d 4096, f 14336, 352 MB, 294 us, now 129: 5.5 TB/s).
struct TransposeArgs {
    const __bf16 *wg, *wu, *wd;
    __bf16 *wdt, *wgut;
    int d, f, f_pad, gu_blocks, d_blocks;      // blocks per expert of w_gate (and of w_up), of w_down with its padding
};
__global__ __launch_bounds__(256)
void bwd_transpose_kernel(TransposeArgs a) {
    __shared__ unsigned short tile[64][72];                              // [column][row], padded
    typedef unsigned short us8 __attribute__((ext_vector_type(8)));
    const int e = blockIdx.y, b = blockIdx.x;
    const bool down = b >= 2 * a.gu_blocks;
    const int which = down ? 2 : b / a.gu_blocks, i = down ? b - 2 * a.gu_blocks : b % a.gu_blocks;
    const int R = down ? a.d : a.f, C = down ? a.f : a.d;                 // of the source
    const int rows = R / 64, r0 = i % rows * 64, c0 = i / rows * 64;      // (d and f are multiples of 64)
    const unsigned short* const src = (const unsigned short*)(down ? a.wd : (which ? a.wu : a.wg)) + (size_t)e * R * C;
    unsigned short* const dst = (unsigned short*)(down ? a.wdt : a.wgut) + (size_t)e * (down ? (size_t)a.f_pad * a.d : (size_t)a.d * 2 * a.f) + (which == 1 ? a.f : 0);
    const size_t ldd = down ? a.d : 2 * a.f;
    const int part = threadIdx.x & 7, line = threadIdx.x >> 3;           // 8 lanes per 64 values, 32 lines per pass
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int r = line + 32 * p;
        us8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (c0 < C) v = *reinterpret_cast<const us8*>(src + (size_t)(r0 + r) * C + c0 + part * 8);
#pragma unroll
        for (int k = 0; k < 8; ++k) tile[part * 8 + k][r] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int c = line + 32 * p;
        *reinterpret_cast<us8*>(dst + (size_t)(c0 + c) * ldd + r0 + part * 8) = *reinterpret_cast<const us8*>(&tile[c][part * 8]);
    }
}

template <bool LISTED, bool WIDE, bool FEW>
moe_status launch_dw(const DwArgs& a, long long most_units, hipStream_t s) {
    static moe::DeviceOnce attr;
    auto kern = ffn_bwd_dw_kernel<LISTED, WIDE, FEW>;
    int dev;
    if (attr.needed(dev)) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, ADAPTIVE_LDS);
        if (e != hipSuccess) { moe::note_hip_error(e, "hipFuncSetAttribute(MaxDynamicSharedMemorySize)"); return MOE_ERR_HIP; }
        attr.mark(dev);
    }
    moe::LaunchScope k("ffn_bwd_dw_kernel", s);
    hipLaunchKernelGGL(kern, dim3((int)std::min<long long>(most_units, num_cus())), dim3(512), ADAPTIVE_LDS, s, a);
    return k.done();
}

inline size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

struct BwdLayout {                              // byte offsets into the workspace of a backward call
    size_t plan_rows, ready_rows, list, ebase, bases, counters, entries, arrived, zeros, wdt, wgut, dh, dgu, h, part;
    int f_pad;
};
BwdLayout bwd_layout(int M, int E_loc, int d, int f) {
    BwdLayout L;
    L.f_pad = (f + 255) / 256 * 256;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += al256(bytes); return at; };
    L.plan_rows = take((size_t)(plan_capacity(M) + PLAN_HDR) * sizeof(int4));
    L.ready_rows = take((size_t)plan_capacity(M) * sizeof(int));
    L.list = take(list_bytes(M));
    L.ebase = take(EBASE_BYTES);
    L.bases = take((size_t)(E_loc + 1) * sizeof(int));
    L.counters = take((size_t)BWD_COUNTERS * sizeof(int));
    L.entries = take((1 + dw_entries(E_loc)) * sizeof(int4));
    L.arrived = take((size_t)DW_MAX_UNITS * sizeof(int));
    L.zeros = take(DW_ZEROS);
    L.wdt = take((size_t)E_loc * L.f_pad * d * 2);
    L.wgut = take((size_t)E_loc * d * 2 * f * 2);
    L.dh = take((size_t)M * L.f_pad * 2);
    L.dgu = take((size_t)M * 2 * f * 2);
    L.h = take((size_t)M * f * 2);
    L.part = o;                                  // (last: bwd_part_bytes)
    return L;
}
// Places for the sums of the weight gradients' parts: an expert of r rows has at most r / DW_PART_ROWS parts with a place per tile, and fewer than two of
// them serve nobody
int dw_places(int M, int d, int f) {
    const long long tiles = dw_tiles(d, f), places = std::min<long long>(DW_MAX_UNITS, (long long)(M / DW_PART_ROWS) * tiles);
    return places < 2 * tiles ? 0 : (int)places;
}
// The tables, dh, dg, du, h, the transposed weights (all that a call must have), and places for the sums of the weight gradients' parts or of the row products' split
// contractions, without which these are in fewer parts.  More room than that changes nothing.
size_t bwd_part_bytes(int M, int d, int f) { return std::max(dw_places(M, d, f) * DW_UNIT_BYTES, tile_part_bytes(d, 2 * f)); }
size_t bwd_workspace_bytes(int M, int E_loc, int d, int f) { return bwd_layout(M, E_loc, d, f).part + bwd_part_bytes(M, d, f); }

}  // namespace

extern "C" size_t moe_ffn_workspace_bytes(int M, int d, int f) {
    if (M < 0 || d < 1 || f < 1) return 0;
    // hidden activations, plan, ready counters, row list, router weights in list order, row bases of the experts
    // (all that a call must have), and room for the K-major rows of x of a small call or the sums of split contractions; a larger M has room for the smaller
    // calls too, so that the size never falls when M grows
    return ffn_base_bytes(M, f) + std::max(kmajor_bytes(std::min(M, KMAJOR_ROWS), d), tile_part_bytes(d, f));
}

extern "C" moe_status moe_ffn_tile_override(int tile_rows, int kernels, int panel_groups) {
    if (tile_rows != 0 && tile_rows != 64 && tile_rows != 128 && tile_rows != 256) return MOE_ERR_INVALID_ARG;
    if (kernels < 0 || kernels > 2) return MOE_ERR_INVALID_ARG;
    if (panel_groups < 0) return MOE_ERR_INVALID_ARG;
    g_force_rows.store(tile_rows, std::memory_order_relaxed);
    g_force_kernels.store(kernels, std::memory_order_relaxed);
    g_force_panel.store(panel_groups, std::memory_order_relaxed);
    return MOE_OK;
}

extern "C" size_t moe_ffn_expanded_weights_bytes(int E_loc, int d, int f) {
    if (E_loc < 1 || d < 1 || f < 1) return 0;
    return (((size_t)3 * E_loc * d * f * 2) + 255) & ~(size_t)255;
}

extern "C" moe_status moe_expert_ffn_sliced_mapped(const void* x, const int32_t* offsets, int M, int S, int E_loc, int d, int f,
                                                   int weight_format, const void* w_gate, const void* w_up, const void* w_down,
                                                   const float* s_gate, const float* s_up, const float* s_down,
                                                   const int32_t* row_map, const float* row_gate, void* y,
                                                   void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (M < 0 || S < 0 || E_loc < 1 || d < 1 || f < 1 || !offsets) return MOE_ERR_INVALID_ARG;
    if (weight_format != MOE_W_BF16 && weight_format != MOE_W_FP8_E4M3_B128) return MOE_ERR_INVALID_ARG;
    if (!w_gate || !w_up || !w_down) return MOE_ERR_INVALID_ARG;
    const bool fp8 = weight_format == MOE_W_FP8_E4M3_B128;
    if (fp8 && (!s_gate || !s_up || !s_down)) return MOE_ERR_INVALID_ARG;
    if (d % 256 != 0 || f % 128 != 0) return MOE_ERR_UNSUPPORTED_SHAPE;
    const long long G = (long long)S * E_loc;
    if (G > MAX_GROUPS) return MOE_ERR_UNSUPPORTED_SHAPE;
    // (32-bit byte offsets inside one 256-row tile and inside one expert's matrices)
    if (d > (1 << 22) || f > (1 << 22) || (long long)d * f >= (1LL << 31)) return MOE_ERR_UNSUPPORTED_SHAPE;
    if (M == 0 || G == 0) return MOE_OK;
    if (!x || !y) return MOE_ERR_INVALID_ARG;
    // every operand is moved in 16-byte pieces
    if ((((uintptr_t)x | (uintptr_t)y | (uintptr_t)w_gate | (uintptr_t)w_up | (uintptr_t)w_down | (uintptr_t)workspace) & 15) != 0)
        return MOE_ERR_INVALID_ARG;
    const size_t base_bytes = ffn_base_bytes(M, f);
    if (!workspace || workspace_bytes < base_bytes) return MOE_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)hip_stream;

    // fp8 weights and many rows per expert: when the caller has added room for it the weights may be expanded to bf16 once per call, for the fused
    // kernel, which takes bf16 only.  Where that is estimated to be the faster way, us, tiles on the codes / expansion and fused kernel: E 4, d 7168, f 2048, 2100 /
    // 3300 / 5000 rows per expert 746 / 788, 1105 / 1064, 1675 / 1514; E 8, d 1024, f 3456, 3100 / 5000 578 / 551, 901 / 813; E 1, d 4096, f 14336, 2560 / 3600
    // 870 / 929, 1166 / 1132.
    const Route chosen = route(M, S, E_loc, d, f, fp8, workspace_bytes - base_bytes >= moe_ffn_expanded_weights_bytes(E_loc, d, f));
    if (chosen == EXPAND) {
        __bf16* wg = (__bf16*)((char*)workspace + base_bytes);
        __bf16* wu = wg + (size_t)E_loc * f * d;
        __bf16* wd = wu + (size_t)E_loc * f * d;
        const long long n8 = (long long)E_loc * f * d / 8;
        const int blocks = (int)std::min<long long>((n8 + 255) / 256, 16LL * num_cus());
        moe::LaunchScope k("ffn_expand_fp8_kernel", s);
        // gate and up: [E_loc * f][d] with scales [E_loc * f / 128][d / 128]; down: [E_loc * d][f]
        hipLaunchKernelGGL(ffn_expand_fp8_kernel, dim3(blocks), dim3(256), 0, s, (const unsigned char*)w_gate, s_gate, wg, n8, d);
        hipLaunchKernelGGL(ffn_expand_fp8_kernel, dim3(blocks), dim3(256), 0, s, (const unsigned char*)w_up, s_up, wu, n8, d);
        hipLaunchKernelGGL(ffn_expand_fp8_kernel, dim3(blocks), dim3(256), 0, s, (const unsigned char*)w_down, s_down, wd, n8, f);
        moe_status st = k.done();
        if (st != MOE_OK) return st;
        return moe_expert_ffn_sliced_mapped(x, offsets, M, S, E_loc, d, f, MOE_W_BF16, wg, wu, wd, nullptr, nullptr, nullptr,
                                            row_map, row_gate, y, workspace, base_bytes, hip_stream);
    }

    const Route way = pinned(chosen, f, fp8);
    if (way == STREAM) {
        // x K-major: where rows of x lie a multiple of 4 KiB apart (all 16 rows of a fragment in one memory channel) and there are
        // enough of them to pay for the launch (more than 8 experts: fewer work in tiles from there on).  Without / with, us: E 16, d 2048, f 1408, 800 / 1200 / 1500 rows
        // 122 / 140 / 162, 123 / 138 / 156.
        __bf16* xk = nullptr;
        const bool pays = d % 2048 == 0 && M >= ((long long)E_loc * f >= 8192 ? 48LL : 160LL) * E_loc;
        if (pays && M <= KMAJOR_ROWS && workspace_bytes - base_bytes >= kmajor_bytes(M, d)) xk = (__bf16*)((char*)workspace + base_bytes);
        const SkinnyArgs k = {(const __bf16*)x, (__bf16*)workspace, (__bf16*)y, xk, w_gate, w_up, w_down, s_gate, s_up, s_down,
                              offsets, row_map, row_gate, M, S, E_loc, d, f};
        return fp8 ? launch_both_skinny<true>(k, s) : launch_both_skinny<false>(k, s);
    }

    const int bm = way == TILE_64 ? 64 : (way == TILE_128 ? 128 : 256);

    FfnArgs a;
    a.x = (const __bf16*)x;
    a.h = (__bf16*)workspace;
    a.y = (__bf16*)y;
    a.wg = w_gate; a.wu = w_up; a.wd = w_down;
    a.sg = s_gate; a.su = s_up; a.sd = s_down;
    char* at = (char*)workspace + h_bytes(M, f);
    auto take = [&](size_t bytes) { char* p = at; at += bytes; return p; };
    int4* plan = (int4*)take(plan_bytes(M));
    a.plan = plan;
    a.ready = (int*)take(ready_bytes(M));
    int32_t* list = (int32_t*)take(list_bytes(M));
    float* gate = (float*)take(list_bytes(M));
    int* ebase = (int*)take(EBASE_BYTES);
    a.M = M; a.d = d; a.f = f;
    // with one slice or one expert the rows already lie expert by expert.  (Otherwise they are always listed: what the
    // list costs, 1 % where every group is many tiles long, is less than the one ragged tile per group it saves.)
    const bool listed = row_map || row_gate || (S > 1 && E_loc > 1);
    a.list = listed ? list : nullptr;
    a.gate = row_gate ? gate : nullptr;
    a.queues1 = (int*)(plan + 1);
    a.g2.A = a.h; a.g2.lda = f;
    a.g2.B = (const __bf16*)w_down; a.g2.ldb = f; a.g2.strideB = (long long)d * f;
    a.g2.O = a.y; a.g2.ldo = d;
    a.g2.K = f; a.g2.NU = d / 256;
    const bool off32 = (unsigned long long)M * d * 2 < 0xFFFFFF00ull;       // x and y addressed with 32-bit offsets
    a.g2.o_bytes = off32 ? (unsigned int)M * (unsigned int)d * 2u : 0u;
    a.g2.queues = (int*)(plan + 3);
    a.dh = nullptr; a.lddh = 0; a.dgu = nullptr;
    a.panel1 = panel_width(f / 128, (size_t)2 * d * f * 2, (size_t)256 * d * 2);
    a.panel2 = panel_width(d / 256, (size_t)d * f * 2, (size_t)256 * f * 2);
    if (const int forced = g_force_panel.load(std::memory_order_relaxed)) a.panel1 = a.panel2 = forced;
    const PlanArgs plan_args = {offsets, S, E_loc, M, bm, plan_capacity(M), plan, a.ready, row_map, row_gate, listed ? list : nullptr,
                                row_gate ? gate : nullptr, ebase, nullptr};
    moe_status st = launch_plan(plan_args, s);
    if (st != MOE_OK) return st;
    const long long max_blocks = M / bm + E_loc;
    if (way == FUSED)
        return !listed ? launch_both_adaptive<ROWS_PLAIN>(a, max_blocks, E_loc, s)
               : off32 ? launch_both_adaptive<ROWS_LIST32>(a, max_blocks, E_loc, s) : launch_both_adaptive<ROWS_LIST64>(a, max_blocks, E_loc, s);
    f32x4* part = (f32x4*)((char*)workspace + base_bytes);
    const size_t part_bytes = workspace_bytes - base_bytes;
    if (bm == 256) return launch_both_tile<false, 256>(a, max_blocks, part, part_bytes, s);
    if (bm == 128) return fp8 ? launch_both_tile<true, 128>(a, max_blocks, part, part_bytes, s) : launch_both_tile<false, 128>(a, max_blocks, part, part_bytes, s);
    return fp8 ? launch_both_tile<true, 64>(a, max_blocks, part, part_bytes, s) : launch_both_tile<false, 64>(a, max_blocks, part, part_bytes, s);
}

extern "C" moe_status moe_expert_ffn_sliced(const void* x, const int32_t* offsets, int M, int S, int E_loc, int d, int f,
                                            int weight_format, const void* w_gate, const void* w_up, const void* w_down,
                                            const float* s_gate, const float* s_up, const float* s_down, void* y,
                                            void* workspace, size_t workspace_bytes, void* hip_stream) {
    return moe_expert_ffn_sliced_mapped(x, offsets, M, S, E_loc, d, f, weight_format, w_gate, w_up, w_down, s_gate, s_up,
                                        s_down, nullptr, nullptr, y, workspace, workspace_bytes, hip_stream);
}

extern "C" size_t moe_ffn_backward_workspace_bytes(int M, int E_loc, int d, int f) {
    if (M < 0 || E_loc < 1 || d < 1 || f < 1) return 0;
    return bwd_workspace_bytes(M, E_loc, d, f);
}

extern "C" moe_status moe_expert_ffn_backward_sliced(const void* x, const void* dy, const int32_t* offsets, int M, int S, int E_loc,
                                                     int d, int f, const void* w_gate, const void* w_up, const void* w_down,
                                                     void* dx, void* dw_gate, void* dw_up, void* dw_down, void* workspace,
                                                     size_t workspace_bytes, void* hip_stream) {
    if (M < 0 || S < 0 || E_loc < 1 || d < 1 || f < 1 || !offsets) return MOE_ERR_INVALID_ARG;
    if (!w_gate || !w_up || !w_down || !dw_gate || !dw_up || !dw_down) return MOE_ERR_INVALID_ARG;
    if (d % 256 != 0 || f % 128 != 0 || f < 256) return MOE_ERR_UNSUPPORTED_SHAPE;
    const long long G = (long long)S * E_loc;
    if (G > MAX_GROUPS || E_loc > DW_MAX_EXPERTS || (long long)E_loc * 16 * f >= (1LL << 31)) return MOE_ERR_UNSUPPORTED_SHAPE;
    if (d > (1 << 22) || f > (1 << 21) || (long long)d * f >= (1LL << 30)) return MOE_ERR_UNSUPPORTED_SHAPE;
    if (M > 0 && (!x || !dy || !dx)) return MOE_ERR_INVALID_ARG;
    if ((((uintptr_t)x | (uintptr_t)dy | (uintptr_t)dx | (uintptr_t)w_gate | (uintptr_t)w_up | (uintptr_t)w_down | (uintptr_t)dw_gate |
          (uintptr_t)dw_up | (uintptr_t)dw_down | (uintptr_t)workspace) & 15) != 0)
        return MOE_ERR_INVALID_ARG;
    const BwdLayout L = bwd_layout(M, E_loc, d, f);
    if (M + 256LL * E_loc >= (1LL << 22)) return MOE_ERR_UNSUPPORTED_SHAPE;       // (a limit of the interface, which no kernel here needs any more)
    if (!workspace || workspace_bytes < L.part) return MOE_ERR_WORKSPACE;
    const size_t part_bytes = std::min(workspace_bytes - L.part, bwd_part_bytes(M, d, f));
    hipStream_t s = (hipStream_t)hip_stream;
    char* ws = (char*)workspace;
    int4* plan_rows = (int4*)(ws + L.plan_rows);
    int* counters = (int*)(ws + L.counters);
    __bf16 *wdt = (__bf16*)(ws + L.wdt), *wgut = (__bf16*)(ws + L.wgut), *dh = (__bf16*)(ws + L.dh), *dgu = (__bf16*)(ws + L.dgu);
    __bf16* h = (__bf16*)(ws + L.h);
    moe_status st;

    if (M == 0 || G == 0) {
        // no rows: the weight gradients are zero, dx is empty
        moe::LaunchScope k("bwd_zero_kernel", s);
        const size_t words = (size_t)E_loc * f * d / 2;
        for (void* p : {dw_gate, dw_up, dw_down}) hipLaunchKernelGGL(bwd_zero_kernel, dim3(1024), dim3(256), 0, s, (unsigned int*)p, words);
        return k.done();
    }

    // ---- row blocks of the schedule, order and parts of the weight gradients, transposed weights
    const bool listed = S > 1 && E_loc > 1;      // else the rows already lie expert by expert
    int32_t* list = listed ? (int32_t*)(ws + L.list) : nullptr;
    int* bases = (int*)(ws + L.bases);
    // The row products run in tiles of 128 columns where the forward pass would (see route: the shapes are alike), with few rows of 64 where it would stream.
    // us, whole call with 256 x 256 tiles / now: E 4, d 2048, f 1408, 200 / 1000 / 4000 rows 260 / 122, 300 / 159, 540 / 299; E 1, d 4096, f 14336, 200 / 1000 / 4000 rows 1190 / 510, 1630 /
    // 1067, 3450 / 3171; E 8, d 1024, f 640, 1000 / 4000 rows 190 / 95, 270 / 153.
    const Route way = pinned(route(M, S, E_loc, d, f, false, false), f, false);
    const int bm = way == TILE_64 || way == STREAM ? 64 : (way == TILE_128 ? 128 : 256);
    const PlanArgs rows_plan = {offsets, S, E_loc, M, bm, plan_capacity(M), plan_rows, (int*)(ws + L.ready_rows), nullptr, nullptr, list, nullptr,
                                (int*)(ws + L.ebase), bases};
    if ((st = launch_plan(rows_plan, s)) != MOE_OK) return st;
    const int tiles = dw_tiles(d, f), units = (int)std::min<size_t>(dw_places(M, d, f), part_bytes / DW_UNIT_BYTES);
    {
        moe::LaunchScope k("bwd_prep_kernel", s);
        hipLaunchKernelGGL(bwd_prep_kernel, dim3(1), dim3(PLAN_THREADS), 0, s, bases, E_loc, tiles, num_cus(), units, (int4*)(ws + L.entries), counters,
                           (int*)(ws + L.arrived), (unsigned int*)(ws + L.zeros));
        if ((st = k.done()) != MOE_OK) return st;
    }
    {
        moe::LaunchScope k("bwd_transpose_kernel", s);
        const TransposeArgs t = {(const __bf16*)w_gate, (const __bf16*)w_up, (const __bf16*)w_down, wdt, wgut, d, f, L.f_pad, f / 64 * (d / 64), d / 64 * (L.f_pad / 64)};
        hipLaunchKernelGGL(bwd_transpose_kernel, dim3(2 * t.gu_blocks + t.d_blocks, E_loc), dim3(256), 0, s, t);
        if ((st = k.done()) != MOE_OK) return st;
    }

    FfnArgs a;
    a.x = (const __bf16*)x; a.h = h; a.y = nullptr;
    a.wg = w_gate; a.wu = w_up; a.wd = w_down;
    a.sg = a.su = a.sd = nullptr;
    a.plan = plan_rows;
    a.ready = (int*)(ws + L.ready_rows);
    a.M = M; a.d = d; a.f = f;
    a.list = list; a.gate = nullptr;
    a.panel1 = a.panel2 = 1 << 20;
    a.dh = dh; a.lddh = L.f_pad; a.dgu = dgu;
    a.queues1 = counters + 8;
    // Workgroups of the kernels over rows: two per tile (one per tile draws its next ticket before others have found their first), but one on every compute unit where a tile is long
    // (K >= 4096), since what the idle ones cost the queues, some 8 us, does not count there.  Whole call, us, one per tile / two per
    // tile / every unit: E 1, d 4096, f 14336, 3000 rows 3970 / 3365 / 3365, 700 rows 2190 / 2050 / 1695; E 1, d 2048, f 1408, 700 rows 395 /
    // 310 / 390; E 1, d = f = 256, 1500 rows 256 / 222 / 312.
    auto workgroups = [&](int units, int K) -> long long { return K >= 4096 ? num_cus() : 2LL * (M / 256 + E_loc) * units; };
    const bool off32 = (unsigned long long)M * d * 2 < 0xFFFFFF00ull;

    f32x4* const part = (f32x4*)(ws + L.part);
    const long long max_blocks = M / bm + E_loc;
    // ---- dh = dy Wd: rows x f_pad, K = d
    a.g2.A = (const __bf16*)dy; a.g2.lda = d;
    a.g2.B = wdt; a.g2.ldb = d; a.g2.strideB = (long long)L.f_pad * d;
    a.g2.O = dh; a.g2.ldo = L.f_pad;
    a.g2.K = d; a.g2.NU = L.f_pad / 256;
    a.g2.queues = counters + 0;
    a.g2.o_bytes = 0;
    st = way != FUSED ? (bm == 64    ? launch_tiles<2, false, 64, BWD_DH>(a, 0, max_blocks, part, part_bytes, s)
                         : bm == 128 ? launch_tiles<2, false, 128, BWD_DH>(a, 0, max_blocks, part, part_bytes, s)
                                     : launch_tiles<2, false, 256, BWD_DH>(a, 0, max_blocks, part, part_bytes, s))
       : !listed ? launch_adaptive<2, ROWS_PLAIN, ROWS_PLAIN>(a, workgroups(a.g2.NU, a.g2.K), s, "ffn_bwd_dh_kernel")
       : off32   ? launch_adaptive<2, ROWS_LIST32, ROWS_PLAIN>(a, workgroups(a.g2.NU, a.g2.K), s, "ffn_bwd_dh_kernel")
                 : launch_adaptive<2, ROWS_LIST64, ROWS_PLAIN>(a, workgroups(a.g2.NU, a.g2.K), s, "ffn_bwd_dh_kernel");
    if (st != MOE_OK) return st;
    // ---- g, u recomputed; dg, du, h
    st = way != FUSED ? (bm == 64    ? launch_tiles<1, false, 64, BWD_ACT>(a, 1, max_blocks, part, part_bytes, s)
                         : bm == 128 ? launch_tiles<1, false, 128, BWD_ACT>(a, 1, max_blocks, part, part_bytes, s)
                                     : launch_tiles<1, false, 256, BWD_ACT>(a, 1, max_blocks, part, part_bytes, s))
       : !listed ? launch_adaptive<1, ROWS_PLAIN, ROWS_PLAIN, 1>(a, workgroups(f / 128, d), s, "ffn_bwd_act_kernel")
       : off32   ? launch_adaptive<1, ROWS_LIST32, ROWS_PLAIN, 1>(a, workgroups(f / 128, d), s, "ffn_bwd_act_kernel")
                 : launch_adaptive<1, ROWS_LIST64, ROWS_PLAIN, 1>(a, workgroups(f / 128, d), s, "ffn_bwd_act_kernel");
    if (st != MOE_OK) return st;
    // ---- dx = [dg | du] [Wg ; Wu]: rows x d, K = 2f
    a.g2.A = dgu; a.g2.lda = 2 * f;
    a.g2.B = wgut; a.g2.ldb = 2 * f; a.g2.strideB = (long long)d * 2 * f;
    a.g2.O = (__bf16*)dx; a.g2.ldo = d;
    a.g2.K = 2 * f; a.g2.NU = d / 256;
    a.g2.queues = counters + 16;
    a.g2.o_bytes = off32 ? (unsigned int)M * (unsigned int)d * 2u : 0u;
    st = way != FUSED ? (bm == 64    ? launch_tiles<2, false, 64, BWD_DX>(a, 2, max_blocks, part, part_bytes, s)
                         : bm == 128 ? launch_tiles<2, false, 128, BWD_DX>(a, 2, max_blocks, part, part_bytes, s)
                                     : launch_tiles<2, false, 256, BWD_DX>(a, 2, max_blocks, part, part_bytes, s))
       : !listed ? launch_adaptive<2, ROWS_PLAIN, ROWS_PLAIN>(a, workgroups(a.g2.NU, a.g2.K), s, "ffn_bwd_dx_kernel")
       : off32   ? launch_adaptive<2, ROWS_PLAIN, ROWS_LIST32>(a, workgroups(a.g2.NU, a.g2.K), s, "ffn_bwd_dx_kernel")
                 : launch_adaptive<2, ROWS_PLAIN, ROWS_LIST64>(a, workgroups(a.g2.NU, a.g2.K), s, "ffn_bwd_dx_kernel");
    if (st != MOE_OK) return st;

    // ---- weight gradients
    DwArgs w;
    w.x = (const __bf16*)x; w.dy = (const __bf16*)dy; w.dgu = dgu; w.h = h;
    w.list = list;
    w.entries = (const int4*)(ws + L.entries);
    w.queues = counters + DW_QUEUES;
    w.arrived = (int*)(ws + L.arrived);
    w.part = part;
    w.zeros = (const unsigned char*)(ws + L.zeros);
    w.dwg = (__bf16*)dw_gate; w.dwu = (__bf16*)dw_up; w.dwd = (__bf16*)dw_down;
    w.M = M; w.d = d; w.f = f; w.tickets = dw_tickets(d, f);
    const long long most = (long long)E_loc * tiles + units;
    if (w.tickets < DW_CHUNK)
        return !listed ? launch_dw<false, false, true>(w, most, s) : off32 ? launch_dw<true, false, true>(w, most, s) : launch_dw<true, true, true>(w, most, s);
    return !listed ? launch_dw<false, false, false>(w, most, s) : off32 ? launch_dw<true, false, false>(w, most, s) : launch_dw<true, true, false>(w, most, s);
}
