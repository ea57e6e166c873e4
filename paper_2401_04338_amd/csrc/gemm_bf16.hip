// Grouped bf16 GEMM on the CDNA4 matrix cores (v_mfma_f32_32x32x16_bf16), fp32 accumulation.
//
// One kernel serves every dense product of the MAML step (G-Meta Alg. 1: inner forward, local
// back-propagation, outer forward, and the tangent passes of the second-order term):
//     C_g[M, N] = sum_p  A_p,g[M, K] * B_p,g[K, N]          (up to GEMM_MAX_PAIRS products, and those of GemmExt)
// A lane's MFMA fragment is 8 consecutive contraction values.  An operand stored contraction-contiguous
// delivers them as one 16-byte LDS read; an operand stored with the contraction index slowest (template
// flags KA / KB) goes to LDS row by row as it lies in memory and the lane collects its 8 values with two
// transposing LDS reads (ds_read_b64_tr_b16).  Every matrix therefore exists once, in the orientation it
// was produced in:
//   forward      A = activations [rows, d_in]  (contiguous),  B = W [d_in, d_out]          (KB)
//   backward dA  A = deltas      [rows, d_out] (contiguous),  B = W [d_in, d_out] read as [n][k] (contiguous)
//   weight grad  A = activations [rows, d_in]  (KA),          B = deltas [rows, d_out]     (KB), K = rows of the task
// A group is a task: its rows are [row_offsets[g], row_offsets[g+1]) and, once theta has been adapted,
// its weights are its own (group stride != 0).
#include <algorithm>

#include "gm_internal.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

#define GK 64          // k extent of one LDS tile
#define GLD (GK + 8)   // LDS row stride in elements: 144 bytes, an odd number of 16-byte units
#define GPADK 32       // pad of a contraction-slowest tile's rows: four consecutive rows start 16 banks apart

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// What an epilogue does is fixed at compile time for the launches the step makes (EP >= 0: bits 0-2 the fused
// operation, then whether the fp32 output, the bf16 output, the accumulate-into output and the added input exist), so
// that the per-element code is straight-line; EP < 0 reads the same facts from the arguments at run time (any other
// combination).  With everything decided per element at run time the epilogue of a 256 x 256 tile ran to some 14,000
// instructions -- as long as twelve k-tiles of its main loop.
enum { EP_CF = 8, EP_CB = 16, EP_CACC = 32, EP_CIN = 64, EP_RUNTIME = -1 };
static int ep_of(const GemmBArgs& a) {
    const bool cin = a.epi == EPI_AXPBY && a.Cin;
    return a.epi | (a.Cf ? EP_CF : 0) | (a.Cb ? EP_CB : 0) | ((a.Cacc && !cin) ? EP_CACC : 0) | (cin ? EP_CIN : 0);
}
template <int EP>
struct EpiFlags {
    int epi;
    bool cf, cb, cacc, cin;
    __device__ __forceinline__ explicit EpiFlags(const GemmBArgs& a) {
        if constexpr (EP >= 0) {
            epi = EP & 7; cf = (EP & EP_CF) != 0; cb = (EP & EP_CB) != 0; cacc = (EP & EP_CACC) != 0; cin = (EP & EP_CIN) != 0;
        } else {
            epi = a.epi; cf = a.Cf != nullptr; cb = a.Cb != nullptr;
            cin = a.epi == EPI_AXPBY && a.Cin != nullptr; cacc = a.Cacc != nullptr && !cin;
        }
    }
};

// The epilogue.  The first operand of the MFMAs is the B fragment, so a lane holds ROW l32 of each 32x32 block and four
// consecutive columns per group of four registers; stored straight from the registers that is 16 bytes per lane in 32
// different rows per instruction, which the memory pipeline takes several times longer over than whole row segments
// (256 x 256 tiles: 32 -> 26 thousand cycles forward, 56 -> 33 backward).  So every wave passes its accumulators through
// LDS one 32-row strip at a time, applies the fused operation on 4 consecutive columns per lane and writes whole row segments.
// Memory is reached through buffers of the wave's rows (RowBuffer): a 32-bit offset per access, nothing done past the last row or column,
// no branch.  With 64-bit addresses and a test per row these were a third and more of a short product's vector instructions, the
// multiplications at a quarter of the rate (a wave of a 128 x 128 weight-gradient tile: 678 -> 376), and a strip's reads were
// waited for with the stores before them.  700 tasks of a median 32 rows 25.7 -> 25.1 ms, 512 of 256 rows 31.8 -> 31.2, 3 of 512
// rows 1561 -> 1529 us.
template <int BM, int BN, int MI, int NI, int EP>
__device__ __forceinline__ void gemm_epilogue(const GemmBArgs& a, f32x16 (&acc)[MI][NI], bf16_t* smem, int g, int64_t r0, int m0,
                                              int n0, int M, int N, int wm0, int wn0, int lane, int wave) {
    const EpiFlags<EP> fl(a);
    const int l32 = lane & 31, lhi = lane >> 5;
    const bool has_bias = (fl.epi == EPI_BIAS_RELU || fl.epi == EPI_BIAS_MASK) && a.bias;
    const bool has_mask = fl.epi == EPI_BIAS_MASK || fl.epi == EPI_MASK;
    const bool has_cin = fl.cin, has_acc = fl.cacc;
    constexpr int SW = NI * 32, ELD = SW + 4;      // strip width, LDS row stride (floats)
    constexpr int LPR = SW / 4, RPI = 64 / LPR;    // lanes per strip row, rows per pass
    constexpr int IT = 32 / RPI;
    float* E = reinterpret_cast<float*>(smem) + wave * (32 * ELD);
    const int er = lane / LPR, ec = (lane % LPR) * 4;
    const int n = n0 + wn0 + ec, mw = __builtin_amdgcn_readfirstlane(m0 + wm0), rows = __builtin_amdgcn_readfirstlane(max(min(M - mw, MI * 32), 0));   // (uniform, as buffers have to be)
    const bool nok = n < N;
    auto buffer = [&](const void* p, bool on, int64_t g_off, int64_t row, int64_t ld, int elem) {   // element (mw + r, n) is row r
        return RowBuffer(reinterpret_cast<const char*>(p) + (on ? g_off * elem : 0), on ? row + mw : 0, ld, elem, on ? rows : 0, er, n, nok);
    };
    const RowBuffer mask = buffer(a.mask, has_mask, 0, r0, a.ld_mask, 2);
    const RowBuffer cin = buffer(a.Cin, has_cin, (int64_t)g * a.gCin, 0, a.ldcin, 4);
    const RowBuffer cacc = buffer(a.Cacc, has_acc, r0 * a.rCacc, 0, a.ldcacc, 4), csum = buffer(a.Cold ? a.Cold : a.Cacc, has_acc, r0 * a.rCacc, 0, a.ldcacc, 4);
    const float sum_scale = a.Cold ? a.cacc : 1.f;
    const RowBuffer cf = buffer(a.Cf, fl.cf, (int64_t)g * a.gCf + r0 * a.rCf, 0, a.ldcf, 4);
    const RowBuffer cb = buffer(a.Cb, fl.cb, (int64_t)g * a.gCb + r0 * a.rCb + (fl.epi == EPI_SPLIT ? (int64_t)blockIdx.y * a.ext.slot : 0), 0, a.ldcb, 2);
    float4 bn = make_float4(0.f, 0.f, 0.f, 0.f);
    if (has_bias && nok) bn = *reinterpret_cast<const float4*>(a.bias + (int64_t)g * a.gBias + n);
    // What a strip reads from memory is requested before anything of the strip before it is stored: the outputs may alias the
    // inputs (an in-place update, element by element), which would otherwise chain every load behind the previous store.
    const bool read_acc = has_acc && !a.cacc_init;
    uint2 mk_all[2][IT];
    float4 ci_all[2][IT];
    auto request = [&](int i, uint2 (&mk)[IT], float4 (&ci)[IT]) {
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int r = i * 32 + it * RPI;
            if (has_mask) mk[it] = mask.load2(r);
            if (has_cin) ci[it] = cin.load4(r);
            else if (read_acc) ci[it] = csum.load4(r);
            else ci[it] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    request(0, mk_all[0], ci_all[0]);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4*>(E + l32 * ELD + j * 32 + 8 * q + 4 * lhi) =
                    make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        if (i + 1 < MI) request(i + 1, mk_all[(i + 1) & 1], ci_all[(i + 1) & 1]);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the strip is this wave's own: LDS order within the wave suffices
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int r = i * 32 + it * RPI;
            float4 x = *reinterpret_cast<const float4*>(E + (it * RPI + er) * ELD + ec);
            if (fl.epi == EPI_BIAS_RELU) {
                x = make_float4(fmaxf(x.x + bn.x, 0.f), fmaxf(x.y + bn.y, 0.f), fmaxf(x.z + bn.z, 0.f), fmaxf(x.w + bn.w, 0.f));
            } else if (has_mask) {
                const uint2 mk = mk_all[i & 1][it];
                if (fl.epi == EPI_BIAS_MASK) x = make_float4(x.x + bn.x, x.y + bn.y, x.z + bn.z, x.w + bn.w);
                // a bf16 is positive iff it is neither zero nor has its sign bit set
                const u32 h0 = mk.x & 0xffffu, h1 = mk.x >> 16, h2 = mk.y & 0xffffu, h3 = mk.y >> 16;
                x.x = (h0 != 0 && h0 < 0x8000u) ? x.x : 0.f;
                x.y = (h1 != 0 && h1 < 0x8000u) ? x.y : 0.f;
                x.z = (h2 != 0 && h2 < 0x8000u) ? x.z : 0.f;
                x.w = (h3 != 0 && h3 < 0x8000u) ? x.w : 0.f;
            } else if (fl.epi == EPI_AXPBY) {
                if (has_cin) {   // (fmaf: the same rounding in every instance)
                    const float4 ci = ci_all[i & 1][it];
                    x = make_float4(fmaf(a.c1, x.x, a.c0 * ci.x), fmaf(a.c1, x.y, a.c0 * ci.y), fmaf(a.c1, x.z, a.c0 * ci.z), fmaf(a.c1, x.w, a.c0 * ci.w));
                } else {
                    x = make_float4(a.c1 * x.x, a.c1 * x.y, a.c1 * x.z, a.c1 * x.w);
                }
            }
            if (fl.cf) cf.store<STREAM>(r, x);
            if (has_acc) {
                const float4 ci = ci_all[i & 1][it];
                cacc.store(r, make_float4(fmaf(a.cacc, x.x, sum_scale * ci.x), fmaf(a.cacc, x.y, sum_scale * ci.y), fmaf(a.cacc, x.z, sum_scale * ci.z), fmaf(a.cacc, x.w, sum_scale * ci.w)));
            }
            if (fl.epi == EPI_SPLIT) {
                const float c = a.ext.c[blockIdx.y];
                x = make_float4(c * x.x, c * x.y, c * x.z, c * x.w);
            }
            if (fl.cb) {
                uint2 pk;
                pk.x = f2bf2(x.x, x.y);
                pk.y = f2bf2(x.z, x.w);
                cb.store(r, pk);
                if (fl.epi == EPI_SPLIT) {
                    uint2 lo;
                    lo.x = f2bf2(x.x - bf2f((bf16_t)(pk.x & 0xffffu)), x.y - bf2f((bf16_t)(pk.x >> 16)));
                    lo.y = f2bf2(x.z - bf2f((bf16_t)(pk.y & 0xffffu)), x.w - bf2f((bf16_t)(pk.y >> 16)));
                    RowBuffer low = cb;
                    if (nok) low.at += (u32)a.ext.ld * 2u;
                    low.store(r, lo);
                }
            }
        }
        asm volatile("" ::: "memory");   // (no block barrier: it would also wait for the strip's global stores to land)
    }
}

// WM waves along m and WN along n: a wave's share of a BM x BN tile is BM / WM x BN / WN.
//
// Bound: contractions of a few hundred (weights of a task's own, a task's rows) leave a tile four to sixteen steps, so what a
// workgroup waits for -- its first operands, a barrier's last wave, the epilogue's loads -- has to be hidden by the other
// waves of its compute unit.  Eight waves with a quarter of the accumulators of four, operands through buffer loads (no branch
// around a load, addresses once per product) and DEPTH tiles in registers on their way: 256 x 128 tiles of four waves held a
// compute unit alone.  More than one tile ahead costs waves and pays only where compute units have a workgroup each.
// Measured against four waves of plain loads (products of 512 tasks of 256 rows, layers 1677-512-256): backward with the
// gradient stored 398 -> 387 us, hidden layer 125 -> 116, weight gradients over runs of tasks 575 -> 452, per task (four waves
// there: what they write is the bound, and wider stores of a wave help) 532 -> 496; 3 tasks of 512 rows, 4109-1024-512-256,
// 64-row tiles: forward 47 -> 26 us a layer.
//
// 256 x 256 tiles (256 tasks of 512 rows, layers 4109-1024-512-256: the matrix cores are the bound) have a compute unit to
// themselves, two waves a SIMD: the waves' order of instructions has to hide what other workgroups hide elsewhere (PIPE below).
// Against four waves of 128 x 128 each with the same two stages: backward 687 -> 648 us, forward 341 -> 312 and 439 -> 423,
// weight gradients 616 -> 549 a task, 1107 -> 1080 over runs of tasks.  Eight waves that park the next tile before the first step:
// backward 682, weight gradients over runs 1222; parked between steps without reading ahead: 662, 1098.
// One product of a sum: its operands from the tile's first row (or, contraction-slowest, from the group's first row) on, row
// strides in bytes, contraction length.  on false: nothing is read.
struct GemmOp {
    const bf16_t *A, *B;
    u32 la, lb;
    int K;
    bool on;
};
// acc += the products open(0), open(1), .. of the tile at (m0, n0) of an M x N result, n_kt tiles of 64 contraction values in all.
template <int BM, int BN, int WM, int WN, int DEPTH, int NS, bool KA, bool KB, class Open>
__device__ __forceinline__ void gemm_tiles(f32x16 (&acc)[BM / (32 * WM)][BN / (32 * WN)], bf16_t* smem, int M, int N, int m0, int n0, int n_kt, Open&& open) {
    constexpr int NT = WM * WN * 64;                          // threads
    constexpr int MI = BM / (32 * WM), NI = BN / (32 * WN);   // 32x32 blocks per wave in each direction
    constexpr int LDA_K = BM + GPADK, LDB_K = BN + GPADK;  // LDS row strides of contraction-slowest tiles [GK][BM] and [GK][BN]
    constexpr int A_ELEMS = KA ? GK * LDA_K : BM * GLD;    // LDS elements of the A tile; the B tile follows
    constexpr int TILE = A_ELEMS + (KB ? GK * LDB_K : BN * GLD);
    constexpr bool PIPE = NS == 2 && DEPTH == 1;   // one workgroup a compute unit: nobody else's products hide its waits
    static_assert(!PIPE || GK == 64, "four steps a tile");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
    const int l32 = lane & 31, lhi = lane >> 5;

    // global -> register staging: 16-byte chunks, 8 chunks per tile row
    constexpr int CA = BM * 8 / NT, CB = BN * 8 / NT;  // chunks per thread
    constexpr int CR = NT / 8;                          // tile rows covered by one chunk round
    constexpr int RA = NT / (BM / 8), RB = NT / (BN / 8);   // rows of a contraction-slowest tile covered by one round
    u32x4 ra[DEPTH][CA], rb[DEPTH][CB];
    const int crow = tid >> 3, ccol = (tid & 7) * 8;     // chunk c = tid + NT*i: row = crow + CR*i, k = ccol
    const int arow = tid / (BM / 8), acol = (tid % (BM / 8)) * 8, brow = tid / (BN / 8), bcol = (tid % (BN / 8)) * 8;

    // Operand tiles come through buffer loads: what lies outside the operand reads as zero without a branch, also whole tiles
    // past the last one.  (The tile's first row is in the base address: offsets stay far below 32 bits.)
    const u32 OOB = 1u << 31;    // (beyond any tile: 256 rows of at most MAX_WIDTH columns; row steps added to it stay below 2^32)
    // (the product's operands are taken from the arguments once per product: a scalar load in every tile is a wait in every tile)
    int pr = -1, k0 = 0;         // product and contraction offset of the next tile to be requested
    GemmOp op;
    int left_a = 0, left_b = 0;  // rows of the operand from its base on
    auto open_product = [&]() {
        op = open(++pr);
        left_a = op.on ? (KA ? op.K : min(M - m0, BM)) : 0;
        left_b = op.on ? (KB ? op.K : min(N - n0, BN)) : 0;
        k0 = 0;
    };
    open_product();
    auto load_tile = [&](u32x4 (&da)[CA], u32x4 (&db)[CB]) {
        const __amdgpu_buffer_rsrc_t qa = __builtin_amdgcn_make_buffer_rsrc((void*)op.A, 0, (int)((u32)(KA ? min(left_a, GK) : left_a) * op.la), 0x00020000);
        const __amdgpu_buffer_rsrc_t qb = __builtin_amdgcn_make_buffer_rsrc((void*)op.B, 0, (int)((u32)(KB ? min(left_b, GK) : left_b) * op.lb), 0x00020000);
        const bool kok = k0 + ccol < op.K;
        {
            const bool ok = KA ? m0 + acol < M : kok;
            const u32 o = !ok ? OOB : KA ? (u32)arow * op.la + (u32)(m0 + acol) * 2u : (u32)crow * op.la + (u32)(k0 + ccol) * 2u;
#pragma unroll
            for (int i = 0; i < CA; ++i) da[i] = __builtin_amdgcn_raw_buffer_load_b128(qa, (int)(o + (u32)((KA ? RA : CR) * i) * op.la), 0, 0);
        }
        {
            const bool ok = KB ? n0 + bcol < N : kok;
            const u32 o = !ok ? OOB : KB ? (u32)brow * op.lb + (u32)(n0 + bcol) * 2u : (u32)crow * op.lb + (u32)(k0 + ccol) * 2u;
#pragma unroll
            for (int i = 0; i < CB; ++i) db[i] = __builtin_amdgcn_raw_buffer_load_b128(qb, (int)(o + (u32)((KB ? RB : CR) * i) * op.lb), 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);   // (tiles are requested in the order they are waited for)
        k0 += GK;
        if (k0 >= op.K) {
            open_product();
        } else {
            // (never negative: past the last product nothing is left, however many tiles are asked for)
            if constexpr (KA) { op.A += (u64)GK * (op.la / 2u); left_a = max(left_a - GK, 0); }
            if constexpr (KB) { op.B += (u64)GK * (op.lb / 2u); left_b = max(left_b - GK, 0); }
        }
    };
    auto store_tile = [&](bf16_t* stage, const u32x4 (&da)[CA], const u32x4 (&db)[CB]) {
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            if constexpr (KA) *reinterpret_cast<u32x4*>(stage + (arow + RA * i) * LDA_K + acol) = da[i];
            else *reinterpret_cast<u32x4*>(stage + (crow + CR * i) * GLD + ccol) = da[i];
        }
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            if constexpr (KB) *reinterpret_cast<u32x4*>(stage + A_ELEMS + (brow + RB * i) * LDB_K + bcol) = db[i];
            else *reinterpret_cast<u32x4*>(stage + A_ELEMS + (crow + CR * i) * GLD + ccol) = db[i];
        }
    };
    // 8 contraction values of one column of a contraction-slowest tile: two transposing LDS reads
    // (ds_read_b64_tr_b16).  Such a read serves 16 lanes at a time: lane s of the 16 points at 4 consecutive
    // columns (s % 4) * 4.. of row s / 4, and lane i receives column i of those 4 rows.
    const int tr_off_row = lhi * 8 + ((lane & 15) >> 2), tr_off_col = (lane & 16) + (lane & 3) * 4;
    auto frag = [&](const bf16_t* tile, int ld, int c0, int k) {
        const bf16_t* p = tile + (k + tr_off_row) * ld + c0 + tr_off_col;
        typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * ld));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_frags = [&](const bf16_t* stage, int kk, bf16x8 (&af)[MI], bf16x8 (&bfr)[NI]) {   // step kk: 16 contraction values
        const bf16_t* As = stage;
        const bf16_t* Bs = stage + A_ELEMS;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if constexpr (KA) af[i] = frag(As, LDA_K, wm0 + i * 32, kk * 16);
            else af[i] = *reinterpret_cast<const bf16x8*>(As + (wm0 + i * 32 + l32) * GLD + kk * 16 + lhi * 8);
        }
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            if constexpr (KB) bfr[j] = frag(Bs, LDB_K, wn0 + j * 32, kk * 16);
            else bfr[j] = *reinterpret_cast<const bf16x8*>(Bs + (wn0 + j * 32 + l32) * GLD + kk * 16 + lhi * 8);
        }
    };
    auto mfmas = [&](const bf16x8 (&af)[MI], const bf16x8 (&bfr)[NI]) {
        if constexpr (PIPE) __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
        if constexpr (PIPE) __builtin_amdgcn_s_setprio(0);
    };
    // (not __syncthreads: that would also wait for the tiles on their way)
    auto barrier = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    if constexpr (PIPE) {
        // the fragments of a step are read while the step before it is multiplied; the next tile is parked in the other stage, and
        // the one after it requested, between the second and the third step: one barrier a tile
        load_tile(ra[0], rb[0]);
        store_tile(smem, ra[0], rb[0]);
        load_tile(ra[0], rb[0]);
        barrier();
        for (int kt = 0; kt < n_kt; ++kt) {
            const bf16_t* cur = smem + (kt & 1) * TILE;
            bf16_t* nxt = smem + ((kt + 1) & 1) * TILE;
            bf16x8 a0[MI], b0[NI], a1[MI], b1[NI];
            read_frags(cur, 0, a0, b0);
            read_frags(cur, 1, a1, b1);
            mfmas(a0, b0);
            read_frags(cur, 2, a0, b0);
            mfmas(a1, b1);
            store_tile(nxt, ra[0], rb[0]);
            read_frags(cur, 3, a1, b1);
            load_tile(ra[0], rb[0]);
            mfmas(a0, b0);
            mfmas(a1, b1);
            barrier();
        }
        return;
    }
    // DEPTH tiles are on their way from memory at any time, in registers; NS LDS stages.  With one stage two barriers a tile:
    // everyone has read the last one before it is overwritten.  With two, a wave that passed the barrier of tile kt has read
    // tile kt - 1, which tile kt + 1 overwrites.
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load_tile(ra[d], rb[d]);
    for (int kt0 = 0; kt0 < n_kt; kt0 += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (kt0 + d >= n_kt) break;
            bf16_t* stage = smem + (NS == 2 ? (kt0 + d) & 1 : 0) * TILE;
            if (NS == 1 && kt0 + d > 0) barrier();
            store_tile(stage, ra[d], rb[d]);
            load_tile(ra[d], rb[d]);
            barrier();
#pragma unroll
            for (int kk = 0; kk < GK / 16; ++kk) {
                bf16x8 af[MI], bfr[NI];
                read_frags(stage, kk, af, bfr);
                mfmas(af, bfr);
            }
        }
    }
}

// XT: the products of the argument's `ext` list are added to the ordinary ones (see GemmExt).
template <int BM, int BN, int WM, int WN, int DEPTH, int NS, bool KA, bool KB, int EP, bool XT>
__global__ __launch_bounds__(64 * WM * WN) void gemm_bf16_kernel(GemmBArgs a, int n_ntiles, int mt_per_group, int n_tiles) {
    constexpr int MI = BM / (32 * WM), NI = BN / (32 * WN);   // 32x32 blocks per wave in each direction
    extern __shared__ __attribute__((aligned(16))) bf16_t smem[];

    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Re-number them so that
    // consecutive tiles -- the n-tiles of one row block, then the next row block of the same task, which
    // read the same rows and the same weights -- run on the same XCD.
    const int per_xcd = gridDim.x >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= n_tiles) return;
    const int ntile = tile % n_ntiles;
    const int mtile = tile / n_ntiles;
    int g, m0;
    if (a.tile_group) {
        g = a.tile_group[mtile];
        m0 = a.tile_m0[mtile];
    } else {
        g = mtile / mt_per_group;
        m0 = (mtile % mt_per_group) * BM;
    }
    const int64_t r0 = a.row_offsets[g];
    const int rows_g = (int)(a.row_offsets[g + 1] - r0);
    const int M = a.M < 0 ? rows_g : a.M;
    const int K = a.K < 0 ? rows_g : a.K;
    constexpr bool SPLIT = EP == (EPI_SPLIT | EP_CB);   // the columns are rows of B, those of the group in another set
    const int e = SPLIT ? (int)blockIdx.y : 0;
    const int64_t r0b = SPLIT ? a.ext.rows[e][g] : r0;
    const int N = SPLIT ? (int)(a.ext.rows[e][g + 1] - r0b) : a.N;
    const int n0 = ntile * BN;
    if (SPLIT && n0 >= N) return;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    // (not __syncthreads: that would also wait for the tiles on their way)
    auto barrier = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    gemm_tiles<BM, BN, WM, WN, DEPTH, NS, KA, KB>(acc, smem, M, N, m0, n0, (K + GK - 1) / GK * a.n_pairs, [&](int pr) {
        const bool on = pr < a.n_pairs;
        const int p = on ? pr : 0;
        const int64_t lda = a.lda[p], ldb = a.ldb[p];
        return GemmOp{a.A[p] + (int64_t)g * a.gA[p] + r0 * a.rA[p] + (KA ? 0 : (int64_t)m0 * lda),
                      (SPLIT ? a.ext.Q[e] : a.B[p] + (int64_t)g * a.gB[p]) + r0b * a.rB[p] + (KB ? 0 : (int64_t)n0 * ldb), (u32)lda * 2u, (u32)ldb * 2u, K, on};
    });
    barrier();   // every wave is done with the operand tiles
    if constexpr (XT) {
        const GemmExt& x = a.ext;
        int n_kt = 0;
        for (int e = 0; e < x.n; ++e) n_kt += 2 * max((x.rows[e][g + 1] - x.rows[e][g] + GK - 1) / GK, 1);   // (no rows: one tile of zeros)
        gemm_tiles<BM, BN, WM, WN, DEPTH, NS, false, true>(acc, smem, M, N, m0, n0, n_kt, [&](int pr) {
            const bool on = pr < 2 * x.n;
            const int e = on ? pr >> 1 : 0;
            const int64_t f0 = x.rows[e][g];
            return GemmOp{x.S[e] + (r0 + m0) * 2 * x.ld + (pr & 1) * x.ld, x.Q[e] + f0 * x.ldq, (u32)x.ld * 4u, (u32)x.ldq * 2u, (int)(x.rows[e][g + 1] - f0), on};
        });
        barrier();
    }

    gemm_epilogue<BM, BN, MI, NI, EP>(a, acc, smem, g, r0, m0, n0, M, N, wm0, wn0, lane, wave);
}

static void tile_counts(const GemmBArgs& a, int BM, int BN, int& n_ntiles, int& mt_per_group, int64_t& n_tiles) {
    n_ntiles = ((a.N < 0 ? a.most_n : a.N) + BN - 1) / BN;
    int64_t n_mtiles;
    mt_per_group = 1;
    if (a.tile_group) {
        n_mtiles = a.n_mtiles;
    } else {
        mt_per_group = (a.M + BM - 1) / BM;
        n_mtiles = (int64_t)mt_per_group * a.G;
    }
    n_tiles = (n_mtiles <= 0 || n_ntiles <= 0) ? 0 : n_mtiles * n_ntiles;
}

template <int BM, int BN, int WM, int WN, int DEPTH, int NS, bool KA, bool KB, int EP, bool XT = false>
static void launch_variant(hipStream_t st, const GemmBArgs& a) {
    int n_ntiles, mt_per_group;
    int64_t n_tiles;
    tile_counts(a, BM, BN, n_ntiles, mt_per_group, n_tiles);
    if (n_tiles <= 0) return;
    size_t shmem = ((KA ? (size_t)GK * (BM + GPADK) : (size_t)BM * GLD) + (KB || XT ? (size_t)GK * (BN + GPADK) : (size_t)BN * GLD)) * sizeof(bf16_t) * NS;
    const size_t epi = (size_t)WM * WN * 32 * (BN / WN + 4) * sizeof(float);  // the epilogue's strips, one per wave
    if (shmem < epi) shmem = epi;
    auto kern = gemm_bf16_kernel<BM, BN, WM, WN, DEPTH, NS, KA, KB, EP, XT>;
    if (shmem > 48 * 1024) (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    const unsigned grid = (unsigned)((n_tiles + 7) / 8 * 8);
    hipLaunchKernelGGL(kern, dim3(grid, a.epi == EPI_SPLIT ? a.ext.n : 1), dim3(64 * WM * WN), shmem, st, a, n_ntiles, mt_per_group, (int)n_tiles);
}

// Tile shapes of one operand form.  bm: row tile the caller built its (tile_group, tile_m0) lists for (64, 128 or
// 256); bn: 128, or 256 (with bm = 256).  With further products (a.ext: many small tasks) one tile on
// its way and one stage leave room for more workgroups (700 tasks of a median 32 rows: a forward launch 424 -> 410 us, their thin
// products 227 -> 208); other 64-row tiles keep two tiles on their way and two LDS
// stages (3 tasks of 512 rows: a layer's forward 23.1 us, with four tiles and four waves 24.9); for the others one of each
// leaves room for more workgroups (512 tasks of 256 rows: a backward launch 387 us, 518 with two tiles on their way).
template <bool KB, int EP>
static void launch_rows_form(hipStream_t st, const GemmBArgs& a, int bm, int bn) {
    if (a.ext.n > 0) launch_variant<64, 128, 2, 4, 1, 1, false, KB, EP, true>(st, a);   // (bm is 64)
    else if (bm == 256 && bn == 256) launch_variant<256, 256, 2, 4, 1, 2, false, KB, EP>(st, a);
    else if (bm == 256) launch_variant<256, 128, 4, 2, 1, 1, false, KB, EP>(st, a);
    else if (bm == 128) launch_variant<128, 128, 2, 4, 1, 1, false, KB, EP>(st, a);
    else launch_variant<64, 128, 2, 4, 2, 2, false, KB, EP>(st, a);
}

// backward form: both operands contraction-contiguous
void launch_gemm_bf16(hipStream_t st, const GemmBArgs& a, int bm, int bn) {
    switch (ep_of(a)) {
        case EPI_MASK | EP_CB: launch_rows_form<false, EPI_MASK | EP_CB>(st, a, bm, bn); break;
        case EPI_NONE | EP_CF: launch_rows_form<false, EPI_NONE | EP_CF>(st, a, bm, bn); break;
        case EPI_NONE | EP_CF | EP_CACC: launch_rows_form<false, EPI_NONE | EP_CF | EP_CACC>(st, a, bm, bn); break;
        case EPI_NONE | EP_CACC: launch_rows_form<false, EPI_NONE | EP_CACC>(st, a, bm, bn); break;
        case EPI_SPLIT | EP_CB: launch_variant<64, 64, 2, 2, 1, 1, false, false, EPI_SPLIT | EP_CB>(st, a); break;
        default: launch_rows_form<false, EP_RUNTIME>(st, a, bm, bn); break;
    }
}

// Weight-gradient form: both operands stored with the contraction index slowest (A [K, M], B [K, N]).  tile: 128, or 256
// (N a multiple of 256), which the caller takes from some 200 rows of a group on where they fill the device.  In 128 x 128 tiles a
// product per task (K = a task's rows, every task writing its own [M, N]) is bound by what it writes.
template <int EP>
static void launch_kmajor_tile(hipStream_t st, const GemmBArgs& a, int tile) {
    if (tile == 256) launch_variant<256, 256, 2, 4, 1, 2, true, true, EP>(st, a);
    // (eight waves where only sums over runs of tasks are written: a long contraction; else four)
    else launch_variant<128, 128, 2, (EP & ~EP_CIN) == (EPI_AXPBY | EP_CF) ? 4 : 2, 1, 1, true, true, EP>(st, a);
}
void launch_gemm_bf16_kmajor(hipStream_t st, const GemmBArgs& a, int tile) {
    switch (ep_of(a)) {
        case EPI_AXPBY | EP_CF: launch_kmajor_tile<EPI_AXPBY | EP_CF>(st, a, tile); break;
        case EPI_AXPBY | EP_CF | EP_CB: launch_kmajor_tile<EPI_AXPBY | EP_CF | EP_CB>(st, a, tile); break;
        case EPI_AXPBY | EP_CB: launch_kmajor_tile<EPI_AXPBY | EP_CB>(st, a, tile); break;
        case EPI_AXPBY | EP_CF | EP_CIN: launch_kmajor_tile<EPI_AXPBY | EP_CF | EP_CIN>(st, a, tile); break;
        case EPI_AXPBY | EP_CF | EP_CB | EP_CIN: launch_kmajor_tile<EPI_AXPBY | EP_CF | EP_CB | EP_CIN>(st, a, tile); break;
        case EPI_AXPBY | EP_CB | EP_CIN: launch_kmajor_tile<EPI_AXPBY | EP_CB | EP_CIN>(st, a, tile); break;
        default: launch_variant<128, 128, 2, 2, 1, 1, true, true, EP_RUNTIME>(st, a); break;
    }
}

// Forward form with the weights as they are stored (B [K, N] = W [d_in, d_out]): no transposed copy of theta.
void launch_gemm_bf16_bkmajor(hipStream_t st, const GemmBArgs& a, int bm, int bn) {
    switch (ep_of(a)) {
        case EPI_BIAS_RELU | EP_CB: launch_rows_form<true, EPI_BIAS_RELU | EP_CB>(st, a, bm, bn); break;
        case EPI_BIAS_MASK | EP_CB: launch_rows_form<true, EPI_BIAS_MASK | EP_CB>(st, a, bm, bn); break;
        default: launch_rows_form<true, EP_RUNTIME>(st, a, bm, bn); break;
    }
}
