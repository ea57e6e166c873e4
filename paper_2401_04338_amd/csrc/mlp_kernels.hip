// Dense side of the MAML step (G-Meta Alg. 1): inner forward / local back-propagation on theta, outer
// forward with the task's adapted theta', and the tangent passes of the second-order term.  Every
// product is a GROUPED GEMM: one group per task, each group with its own rows and (when theta has been
// adapted) its own weights.
#include <algorithm>

#include "gm_internal.h"

// ------------------------------------------------------------------------------------------------
// fp32 grouped GEMM on the matrix cores (fp32 operands, products and sums), C = A1*B1 (+ A2*B2)
// with a fused epilogue
// ------------------------------------------------------------------------------------------------
// Bound: the fp32 matrix rate (157 TFLOP/s; plain vector FMA reaches half of it and has to fetch 8 LDS values per 16
// FMAs) where the tiles fill the device, the latency of the k-loop's loads where a call has a few tasks only.
// A workgroup of four waves takes the k-range in pieces that are requested a whole piece ahead (registers), so that
// the memory latency runs beside the MFMAs of the piece before.  Two shapes:
//   SMALL false  64 x 64 tile, 2 x 2 blocks of 16 x 16 per wave, pieces of 64
//   SMALL true   32 x 32 tile, one block per wave, pieces of 128: four times the workgroups and a quarter of the MFMA time
// ORDER OF THE SUMS: v_mfma_f32_16x16x4_f32 adds its four products one after the other, each a fused multiply-add rounded
// to fp32 (measured: the same bits as an fmaf chain in ascending k, denormals included), and every MFMA takes the next four
// contraction values.  So an output has the bits of the plain loop over k whatever the tile: a task's results do not depend
// on how many tasks share its launch.
// Operands stay in LDS as they lie in memory; lane group q of the four reads contraction value 4 j + q for MFMA j.
// Contraction-contiguous rows are 4 floats longer than a piece and contraction-slowest rows change places in blocks of 16
// columns from one to the next: in both forms the 64 lanes read 64 different banks.
// Measured on one second-order step, all 18 products together: 64 tasks x (128 + 128) rows through 845-256-128-1
// 2.03 -> 0.69 ms, 37 tasks of about 50 rows through 189-100-52-1 0.45 -> 0.12 ms, 4 tasks x (32 + 32) rows through
// 141-64-32-1 0.29 -> 0.10 ms (before: vector FMA, loads not overlapped).  Small tiles whose waves share the contraction and
// 32 x 32 blocks in the large ones take the same time (0.69 ms), but add in orders of their own.
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

template <bool SMALL>
struct F32Tile {
    static constexpr int R = SMALL ? 1 : 2;         // a wave's blocks of 16 rows, and of 16 columns
    static constexpr int T = 32 * R;                // rows and columns of the tile
    static constexpr int BK = SMALL ? 128 : 64;     // contraction values per piece
    static constexpr int V = T * BK / 4 / 256;      // 16-byte pieces per thread and operand
    static constexpr int LD_CONT = BK + 4, LD_SLOW = T;
    static constexpr int WORDS_CONT = T * LD_CONT, WORDS_SLOW = BK * LD_SLOW;
    static constexpr int NJ = SMALL ? 8 : 4;        // values of a lane that are read ahead, per block
    // column i of contraction-slowest row k: blocks of 16 columns exchanged
    __device__ __forceinline__ static int swap(int k, int i) { return i ^ (SMALL ? (k & 2) << 3 : (k & 3) << 4); }
};

typedef __attribute__((__vector_size__(4 * sizeof(u32)))) u32 u32x4_t;

// One operand's pieces [T x BK] from memory to registers to LDS.  CONT: element (i, k) at p + i*ld + k, else at
// p + k*ld + i (extents along the contiguous direction and strides are multiples of 4: every matrix is padded to 32).
// The piece's base is uniform and moves on; a thread's offsets inside it stay.  What lies outside the operand is asked
// for beyond the buffer's end and reads as zero.
template <bool SMALL, bool CONT>
struct F32Operand {
    using TT = F32Tile<SMALL>;
    static constexpr u32 OOB = 0x80000000u;
    const float* base;
    int64_t step;
    u32 off[TT::V];
    __device__ __forceinline__ static int row(int u) { const int e = threadIdx.x + u * 256; return CONT ? e / (TT::BK / 4) : e % (TT::T / 4) * 4; }
    __device__ __forceinline__ static int col(int u) { const int e = threadIdx.x + u * 256; return CONT ? e % (TT::BK / 4) * 4 : e / (TT::T / 4); }
    __device__ __forceinline__ void init(const float* p, int64_t ld, int n_i) {
        base = p;
        step = CONT ? TT::BK : TT::BK * ld;
#pragma unroll
        for (int u = 0; u < TT::V; ++u) {
            const u32 o = CONT ? (u32)row(u) * (u32)ld + (u32)col(u) : (u32)col(u) * (u32)ld + (u32)row(u);
            off[u] = row(u) < n_i ? o * 4u : OOB;
        }
    }
    __device__ __forceinline__ void fetch(int k_left, u32x4_t (&v)[TT::V]) {   // the next piece; k_left: contraction values from its start on
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00020000);
#pragma unroll
        for (int u = 0; u < TT::V; ++u) v[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(col(u) < k_left ? off[u] : OOB), 0, 0);
        base += step;
    }
    __device__ __forceinline__ static void store(float* s, const u32x4_t (&v)[TT::V]) {
#pragma unroll
        for (int u = 0; u < TT::V; ++u)
            *reinterpret_cast<u32x4_t*>(s + (CONT ? row(u) * TT::LD_CONT + col(u) : col(u) * TT::LD_SLOW + TT::swap(col(u), row(u)))) = v[u];
    }
    // a lane's values of the next NJ MFMAs (contraction values from k on): row or column i of the tile, q the lane group
    __device__ __forceinline__ static void frag(const float* s, int i, int k, int q, float (&f)[TT::R][TT::NJ]) {
#pragma unroll
        for (int r = 0; r < TT::R; ++r) {
            const float* p = CONT ? s + (i + r * 16) * TT::LD_CONT + k + q : s + (k + q) * TT::LD_SLOW + TT::swap(q, i + r * 16);
#pragma unroll
            for (int j = 0; j < TT::NJ; ++j) f[r][j] = p[j * 4 * (CONT ? 1 : TT::LD_SLOW)];
        }
    }
};

// block, n_blocks: the workgroup's number among those of this product
template <bool SMALL, bool KA, bool KB>
__device__ __forceinline__ void gemm_f32_tile(const GemmArgs& a, int n_ntiles, int mt_per_group, int block, int n_blocks) {
    using TT = F32Tile<SMALL>;
    using OpA = F32Operand<SMALL, KA>;
    using OpB = F32Operand<SMALL, KB>;
    constexpr int WA = KA ? TT::WORDS_CONT : TT::WORDS_SLOW, WB = KB ? TT::WORDS_CONT : TT::WORDS_SLOW;
    __shared__ float4 stage[(WA + WB) / 4];
    float* const As = reinterpret_cast<float*>(stage);
    float* const Bs = As + WA;
    // workgroups are dealt round-robin to the 8 XCDs: neighbouring tiles (same rows, same weights) go to the same one
    const int per = n_blocks >> 3, rest = n_blocks & 7, xcd = block & 7;
    const int tile = xcd * per + (xcd < rest ? xcd : rest) + (block >> 3);
    const int ntile = tile % n_ntiles;
    const int mtile = tile / n_ntiles;
    int g, m0;
    if (a.tile_group) {   // the list's tiles have 64 rows
        constexpr int PER = 64 / TT::T;
        g = a.tile_group[mtile / PER];
        m0 = a.tile_m0[mtile / PER] + mtile % PER * TT::T;
    } else {
        g = mtile / mt_per_group;
        m0 = (mtile % mt_per_group) * TT::T;
    }
    const int64_t r0 = a.row_offsets ? a.row_offsets[g] : 0;
    const int rows_g = a.row_offsets ? (int)(a.row_offsets[g + 1] - r0) : 0;
    const int M = a.M < 0 ? rows_g : a.M;
    const int K = a.K < 0 ? rows_g : a.K;
    const int N = a.N;
    if (m0 >= M) return;
    const int n0 = ntile * TT::T;
    constexpr int R = TT::R, NJ = TT::NJ;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, q = lane >> 4;
    const int mb = (wv >> 1) * 16 * R, nb = (wv & 1) * 16 * R;
    f32x4 acc[R][R];
#pragma unroll
    for (int i = 0; i < R * R * 4; ++i) acc[i / 4 / R][i / 4 % R][i % 4] = 0.f;

    for (int pr = 0; pr < a.n_pairs; ++pr) {
        OpA A;
        OpB B;
        A.init(a.A[pr] + (int64_t)g * a.gA[pr] + r0 * a.rA[pr] + m0 * a.sAm[pr], KA ? a.sAm[pr] : a.sAk[pr], M - m0);
        B.init(a.B[pr] + (int64_t)g * a.gB[pr] + r0 * a.rB[pr] + n0 * a.sBn[pr], KB ? a.sBn[pr] : a.sBk[pr], N - n0);
        u32x4_t va[TT::V], vb[TT::V];
        A.fetch(K, va);
        B.fetch(K, vb);
        for (int left = K; left > 0; left -= TT::BK) {
            __syncthreads();   // the piece before has been read
            OpA::store(As, va);
            OpB::store(Bs, vb);
            __syncthreads();
            if (left > TT::BK) {
                A.fetch(left - TT::BK, va);
                B.fetch(left - TT::BK, vb);
            }
            // (what lies beyond the contraction is zero: the loop may run past it)
            float fa[2][R][NJ], fb[2][R][NJ];
            OpA::frag(As, mb + li, 0, q, fa[0]);
            OpB::frag(Bs, nb + li, 0, q, fb[0]);
            constexpr int STEPS = TT::BK / 4 / NJ;
#pragma unroll
            for (int kb = 0; kb < STEPS; ++kb) {   // the next values are on their way while these are multiplied
                if (kb + 1 < STEPS) {
                    OpA::frag(As, mb + li, (kb + 1) * 4 * NJ, q, fa[(kb + 1) & 1]);
                    OpB::frag(Bs, nb + li, (kb + 1) * 4 * NJ, q, fb[(kb + 1) & 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < R; ++c) acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[kb & 1][c][j], fa[kb & 1][r][j], acc[r][c], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // The first operand of the MFMAs is B's, so a lane holds row li of a block and its columns 4 q .. 4 q + 3: 16 bytes an access
    // (widths and strides are multiples of 4) through a buffer.  Element by element, with 64-bit addresses and a test each, this took
    // more vector instructions than the products of a short contraction (756 of a wave, now 404): 64 tasks x (128 + 128) rows through
    // 845-256-128-1 a gradient launch 59 -> 56 us, a forward one 35 -> 32, the step 1277 -> 1230.
    // All that is read is requested before anything is stored (an update may be in place).
    const int rows = __builtin_amdgcn_readfirstlane(max(min(M - m0, (int)TT::T), 0));
    const bool has_bias = a.epi == EPI_BIAS_RELU || a.epi == EPI_BIAS_MASK, has_mask = a.epi == EPI_BIAS_MASK || a.epi == EPI_MASK;
    const bool axpby = a.epi == EPI_AXPBY, has_cin = axpby && a.Cin;
    f32x4 in[R][R], bias[R];
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const int n = n0 + nb + c * 16 + q * 4;
        const bool nok = n < N;
        bias[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (has_bias && nok) bias[c] = *reinterpret_cast<const f32x4*>(a.bias + (int64_t)g * a.gBias + n);
        const RowBuffer src(has_mask ? a.mask + r0 * a.ld_mask : a.Cin + (int64_t)g * a.gCin + r0 * a.rCin, m0, has_mask ? a.ld_mask : a.ldc, 4,
                            has_mask || has_cin ? rows : 0, mb + li, n, nok);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            in[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (has_mask || has_cin) in[r][c] = __builtin_bit_cast(f32x4, src.load4(r * 16));
        }
    }
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const int n = n0 + nb + c * 16 + q * 4;
        const RowBuffer dst(a.C + (int64_t)g * a.gC + r0 * a.rC, m0, a.ldc, 4, rows, mb + li, n, n < N);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {   // (fmaf: the same rounding in every instance)
                v[i] = has_bias ? acc[r][c][i] + bias[c][i] : acc[r][c][i];
                if (a.epi == EPI_BIAS_RELU) v[i] = fmaxf(v[i], 0.f);
                if (has_mask) v[i] = in[r][c][i] > 0.f ? v[i] : 0.f;
                if (axpby) v[i] = fmaf(a.c1, acc[r][c][i], has_cin ? a.c0 * in[r][c][i] : 0.f);
            }
            dst.store(r * 16, make_float4(v[0], v[1], v[2], v[3]));
        }
    }
}

template <bool SMALL, bool KA, bool KB>
__global__ __launch_bounds__(256, 4) void gemm_f32_kernel(GemmArgs a, int n_ntiles, int mt_per_group) {
    gemm_f32_tile<SMALL, KA, KB>(a, n_ntiles, mt_per_group, (int)blockIdx.x, (int)gridDim.x);
}

// Weight gradients of several layers in one launch: they are independent, and with a handful of tasks each of them is one
// launch's latency long (4 tasks x (32 + 32) rows through 141-64-32: the three passes of a step 34.7 us in six launches, 20.8 us in three).
template <bool SMALL>
__global__ __launch_bounds__(256, 4) void gemm_f32_wgrads_kernel(GemmList l) {
    int i = 0;
    while (i + 1 < l.n && (int)blockIdx.x >= l.block0[i + 1]) ++i;
    const GemmArgs& a = l.job[i];
    constexpr int T = F32Tile<SMALL>::T;
    gemm_f32_tile<SMALL, false, false>(a, (a.N + T - 1) / T, (a.M + T - 1) / T, (int)blockIdx.x - l.block0[i],
                                       (i + 1 < l.n ? l.block0[i + 1] : (int)gridDim.x) - l.block0[i]);
}

template <bool SMALL>
static void gemm_f32_shape(hipStream_t st, const GemmArgs& a) {
    constexpr int T = F32Tile<SMALL>::T;
    const int n_ntiles = (a.N + T - 1) / T, mt_per_group = a.tile_group ? 1 : (a.M + T - 1) / T;
    const int64_t n_mtiles = a.tile_group ? (int64_t)a.n_mtiles * (64 / T) : (int64_t)mt_per_group * a.G;
    if (n_mtiles <= 0 || n_ntiles <= 0) return;
    const dim3 grid((unsigned)(n_mtiles * n_ntiles));
    if (a.sBk[0] == 1) hipLaunchKernelGGL((gemm_f32_kernel<SMALL, true, true>), grid, dim3(256), 0, st, a, n_ntiles, mt_per_group);
    else hipLaunchKernelGGL((gemm_f32_kernel<SMALL, true, false>), grid, dim3(256), 0, st, a, n_ntiles, mt_per_group);
}

// The small tiles where 64 x 64 ones would not give every compute unit two workgroups.  The forward and the backward products
// of 269-256-1, 128 rows a task, three passes, small against large: 64 tiles 45 / 34 against 60 / 47 us, 256 tiles 63 / 47
// against 61 / 49, 512 tiles 104 / 74 against 87 / 69.  Either way the results have the same bits.
#define F32_SMALL_TILES 512
void launch_gemm_f32(hipStream_t st, const GemmArgs& a) {
    const int64_t tiles = (int64_t)((a.N + 63) / 64) * (a.tile_group ? a.n_mtiles : (int64_t)((a.M + 63) / 64) * a.G);
    if (tiles < F32_SMALL_TILES) gemm_f32_shape<true>(st, a);
    else gemm_f32_shape<false>(st, a);
}
void launch_gemm_f32_wgrads(hipStream_t st, const GemmArgs* list, int n) {
    for (int i0 = 0; i0 < n; i0 += GEMM_LIST) {
        GemmList l;
        l.n = std::min(n - i0, (int)GEMM_LIST);
        int64_t tiles64 = 0;
        for (int i = 0; i < l.n; ++i) {
            l.job[i] = list[i0 + i];
            tiles64 = std::max(tiles64, (int64_t)((l.job[i].M + 63) / 64) * ((l.job[i].N + 63) / 64) * l.job[i].G);   // (the largest decides)
        }
        const bool small = tiles64 < F32_SMALL_TILES;
        const int T = small ? 32 : 64;
        int64_t blocks = 0;
        for (int i = 0; i < l.n; ++i) {
            l.block0[i] = (int)blocks;
            blocks += (int64_t)((l.job[i].M + T - 1) / T) * ((l.job[i].N + T - 1) / T) * l.job[i].G;
        }
        if (blocks <= 0) continue;
        if (small) hipLaunchKernelGGL(gemm_f32_wgrads_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, st, l);
        else hipLaunchKernelGGL(gemm_f32_wgrads_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, l);
    }
}

// ------------------------------------------------------------------------------------------------
// per-task column sums (bias gradients, last-layer weight gradient, per-task mean loss), all those of a pass in one launch:
// out[g,n] = c0*in[g,n] + c1 * sum_{s in g} ( X1[s,n]*w1[s] + X2[s,n]*w2[s] ), rows summed in a fixed order
// ------------------------------------------------------------------------------------------------
// Bound: HBM with many tasks; with a few the chain of dependent row batches of one workgroup, and the launches
// themselves.  A workgroup (bf16: of up to 16 waves, fp32: of four) takes one task and one block of columns of one job.
// bf16: a lane owns 16 bytes of columns; rows narrower than a wave's 64 lanes are taken several at a time.  The waves take the
// rows round-robin in batches of UB independent loads; lanes that share columns are added first, then the waves in wave
// order.  fp32: four chains per column (rows 8 c .. 8 c + 7 of every 32, one after the other), which are added in order; four
// waves take the chains of 64 columns, a lane one column, sixteen rows requested at once.  (The task's thetas, and with
// them which side of zero a hidden unit falls on, follow from these sums: in fp32 their order stays whatever the launch.)
// Either partition depends on the job's width alone: results do not depend on how the tasks are cut into waves.
// Measured: the 16 launches of a step of 3 tasks x (512 + 512) rows through 1024-512-256 hidden units, bf16, 0.37 -> 0.03 ms
// in 3 launches (4 waves and a launch per sum before); 512 tasks x 256 rows through 512-256, 28 launches, 0.62 -> 0.60 ms in 7.
enum { COLSUM_WAVES = 16, COLSUM_WAVES_F32 = 4 };   // of a workgroup, at most

// the job of a workgroup
__device__ __forceinline__ const ColJob& colsum_job(const ColJobs& jobs) {
    int ji = 0;
    while (ji + 1 < jobs.n && (int)blockIdx.x >= jobs.job[ji + 1].block0) ++ji;
    return jobs.job[ji];
}
__device__ __forceinline__ void colsum_store(const ColJob& j, int n, float sum) {
    const int g = blockIdx.y;
    j.out[(int64_t)g * j.g_out + n] = j.c1 * sum + (j.in ? j.c0 * j.in[(int64_t)g * j.g_in + n] : 0.f);
}

// rows r0 .. r1 of one column block, this wave's share; the lane's columns start at n of rows r0 + sub, r0 + sub + rpi, ...
template <bool TWO>
__device__ __forceinline__ void colsum_rows(const ColJob& j, int64_t r0, int64_t r1, int wv, int rpi, int sub, int n, float (&acc)[8]) {
    constexpr int UB = TWO ? 4 : 8;
    const bf16_t *X1 = reinterpret_cast<const bf16_t*>(j.X1) + n, *X2 = reinterpret_cast<const bf16_t*>(j.X2) + n;
    auto open = [](const uint4& x, float (&v)[8]) {
        const u32 w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[2 * k] = __builtin_bit_cast(float, w[k] << 16);
            v[2 * k + 1] = __builtin_bit_cast(float, w[k] & 0xFFFF0000u);
        }
    };
    for (int64_t s0 = r0 + (int64_t)wv * UB * rpi; s0 < r1; s0 += (int64_t)COLSUM_WAVES * UB * rpi) {
        uint4 x1[UB], x2[TWO ? UB : 1];
        float f1[UB], f2[TWO ? UB : 1];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int64_t s = s0 + u * rpi + sub;
            const bool ok = s < r1;
            const int64_t sc = ok ? s : r0;
            x1[u] = *reinterpret_cast<const uint4*>(X1 + sc * j.ldx);
            f1[u] = ok ? (j.w1 ? j.w1[sc] : 1.f) : 0.f;
            if (TWO) {
                x2[u] = *reinterpret_cast<const uint4*>(X2 + sc * j.ldx);
                f2[u] = ok ? (j.w2 ? j.w2[sc] : 1.f) : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            float a[8], b[8];
            open(x1[u], a);
            if (TWO) open(x2[u], b);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                float v = a[k] * f1[u];
                if (TWO) v += b[k] * f2[u];
                acc[k] += v;
            }
        }
    }
}

// WAVES: of the sixteen that the rows are dealt to, those that have rows in some task
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void task_colsum_bf16_kernel(const int32_t* __restrict__ row_offsets, ColJobs jobs) {
    constexpr int V = 8;
    __shared__ float part[WAVES > 1 ? WAVES - 1 : 1][64 * V];
    const ColJob& j = colsum_job(jobs);
    const int g = blockIdx.y, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t r0 = row_offsets[g], r1 = row_offsets[g + 1];
    float acc[V];
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = 0.f;
    if (j.N == 1) {   // one fp32 value per row: a lane per row
        const float* X = reinterpret_cast<const float*>(j.X1);
        for (int64_t s = r0 + threadIdx.x; s < r1; s += 64 * COLSUM_WAVES) acc[0] += X[s * j.ldx];
        for (int d = 32; d > 0; d >>= 1) acc[0] += __shfl_xor(acc[0], d, 64);
        if (wv > 0 && lane == 0) part[wv - 1][0] = acc[0];
        __syncthreads();
        if (threadIdx.x == 0) {
            float sum = acc[0];
#pragma unroll
            for (int w = 0; w < WAVES - 1; ++w) sum += part[w][0];
            colsum_store(j, 0, sum);
        }
        return;
    }
    int lpr = 64;   // lanes per row: as few as cover it (a power of two)
    while (lpr > 1 && (lpr / 2) * V >= j.N) lpr /= 2;
    const int sub = lane / lpr, n = (((int)blockIdx.x - j.block0) * 64 + lane % lpr) * V;
    if (n < j.N) {
        if (j.X2) colsum_rows<true>(j, r0, r1, wv, 64 / lpr, sub, n, acc);
        else colsum_rows<false>(j, r0, r1, wv, 64 / lpr, sub, n, acc);
    }
    for (int d = 32; d >= lpr; d >>= 1)
#pragma unroll
        for (int k = 0; k < V; ++k) acc[k] += __shfl_xor(acc[k], d, 64);
    if (wv > 0) {
#pragma unroll
        for (int k = 0; k < V; ++k) part[wv - 1][k * 64 + lane] = acc[k];
    }
    __syncthreads();
    if (wv == 0 && sub == 0 && n < j.N) {
#pragma unroll
        for (int k = 0; k < V; ++k) {
            float sum = acc[k];
#pragma unroll
            for (int w = 0; w < WAVES - 1; ++w) sum += part[w][k * 64 + lane];
            colsum_store(j, n + k, sum);
        }
    }
}

// one chain of one column: rows r0 + 8 * chain .. + 7 of every 32
template <bool TWO>
__device__ __forceinline__ float colsum_chain(const ColJob& j, int64_t r0, int64_t r1, int chain, int n) {
    const float *X1 = reinterpret_cast<const float*>(j.X1) + n, *X2 = reinterpret_cast<const float*>(j.X2) + n;
    float acc = 0.f;
    for (int64_t s0 = r0 + chain * 8; s0 < r1; s0 += 64) {
        float x1[16], f1[16], x2[TWO ? 16 : 1], f2[TWO ? 16 : 1];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int64_t s = s0 + (u < 8 ? u : u + 24);
            const bool ok = s < r1;
            const int64_t sc = ok ? s : r0;
            x1[u] = X1[sc * j.ldx];
            f1[u] = ok ? (j.w1 ? j.w1[sc] : 1.f) : 0.f;
            if (TWO) {
                x2[u] = X2[sc * j.ldx];
                f2[u] = ok ? (j.w2 ? j.w2[sc] : 1.f) : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
#pragma clang fp contract(off)   // (a product is rounded before it is added, in both forms)
            float v = x1[u] * f1[u];
            if (TWO) v = fmaf(x2[u], f2[u], v);
            acc += v;
        }
    }
    return acc;
}

// chains: of every column, those that have rows in some task (1, 2 or 4): the waves beyond them take further columns
__global__ __launch_bounds__(64 * COLSUM_WAVES_F32) void task_colsum_f32_kernel(const int32_t* __restrict__ row_offsets, int chains, ColJobs jobs) {
    constexpr int NT = 64 * COLSUM_WAVES_F32;
    __shared__ float part[NT];
    const ColJob& j = colsum_job(jobs);
    const int g = blockIdx.y, tid = threadIdx.x;
    const int64_t r0 = row_offsets[g], r1 = row_offsets[g + 1];
    if (j.N == 1) {   // one value per row: read by all lanes, added by four
        const float* X = reinterpret_cast<const float*>(j.X1);
        float acc = 0.f;
        for (int64_t s0 = r0; s0 < r1; s0 += NT) {
            __syncthreads();   // the values before have been added
            part[tid] = s0 + tid < r1 ? X[(s0 + tid) * j.ldx] : 0.f;
            __syncthreads();
            const int n = (int)min(r1 - s0, (int64_t)NT);
            if (tid < 4)
                for (int b = tid * 8; b < n; b += 32)
#pragma unroll
                    for (int u = 0; u < 8; ++u) acc += part[b + u];
        }
        const float a1 = __shfl(acc, 1, 64), a2 = __shfl(acc, 2, 64), a3 = __shfl(acc, 3, 64);
        if (tid == 0) colsum_store(j, 0, ((acc + a1) + a2) + a3);
        return;
    }
    const int lane = tid & 63, wv = tid >> 6, chain = wv & (chains - 1), group = wv / chains;
    const int n = (((int)blockIdx.x - j.block0) * (COLSUM_WAVES_F32 / chains) + group) * 64 + lane;
    float acc = 0.f;
    if (n < j.N) acc = j.X2 ? colsum_chain<true>(j, r0, r1, chain, n) : colsum_chain<false>(j, r0, r1, chain, n);
    if (chains > 1) {
        part[tid] = acc;
        __syncthreads();
        if (chain == 0)
            for (int w = 1; w < chains; ++w) acc += part[tid + w * 64];
    }
    if (chain == 0 && n < j.N) colsum_store(j, n, acc);
}

// most_rows: of the largest task.  Waves that no task has rows for are not launched (they would only add zeros, so the results
// are the same; 1024 threads for every task before): 20000 tasks x (1 + 1) rows, 32 units, fp32, 0.81 -> 0.15 ms a step; 5000 tasks x (2 + 2)
// rows, 256-128, bf16, 0.48 -> 0.09 ms; 512 tasks x (128 + 128) rows, 1024-512, fp32, 0.36 -> 0.37 ms.
void launch_task_colsum(hipStream_t st, int bf16, int G, int most_rows, const int32_t* row_offsets, const ColJob* list, int n) {
    int chains = 1;
    while (chains < 4 && chains * 8 < most_rows) chains *= 2;
    const int cols = bf16 ? 64 * 8 : 64 * (COLSUM_WAVES_F32 / chains);   // of a workgroup
    for (int i0 = 0; i0 < n; i0 += COL_JOBS) {
        ColJobs jobs;
        jobs.n = std::min(n - i0, (int)COL_JOBS);
        int blocks = 0, waves = 1;
        for (int i = 0; i < jobs.n; ++i) {
            ColJob& j = jobs.job[i];
            j = list[i0 + i];
            j.block0 = blocks;
            blocks += (j.N + cols - 1) / cols;
            int first = 64;   // rows that a wave of the bf16 kernel starts with
            if (j.N > 1) {
                first = j.X2 ? 4 : 8;
                for (int lanes = 64; lanes > 1 && lanes / 2 * 8 >= j.N; lanes /= 2) first *= 2;
            }
            while (waves < COLSUM_WAVES && waves * first < most_rows) waves *= 2;
        }
        if (G <= 0 || blocks <= 0) continue;
        const dim3 grid(blocks, G), block(64 * (bf16 ? waves : (int)COLSUM_WAVES_F32));
        if (!bf16) hipLaunchKernelGGL(task_colsum_f32_kernel, grid, block, 0, st, row_offsets, chains, jobs);
        else if (waves == 1) hipLaunchKernelGGL(task_colsum_bf16_kernel<1>, grid, block, 0, st, row_offsets, jobs);
        else if (waves == 2) hipLaunchKernelGGL(task_colsum_bf16_kernel<2>, grid, block, 0, st, row_offsets, jobs);
        else if (waves == 4) hipLaunchKernelGGL(task_colsum_bf16_kernel<4>, grid, block, 0, st, row_offsets, jobs);
        else if (waves == 8) hipLaunchKernelGGL(task_colsum_bf16_kernel<8>, grid, block, 0, st, row_offsets, jobs);
        else hipLaunchKernelGGL(task_colsum_bf16_kernel<COLSUM_WAVES>, grid, block, 0, st, row_offsets, jobs);
    }
}

// ------------------------------------------------------------------------------------------------
// last layer (d_L = 1) fused with the sigmoid / binary cross-entropy and the delta of the layer below it
// Rows may be padded per task: row r of task g is sample real_offsets[g] + (r - row_offsets[g]) when that
// is below real_offsets[g+1]; pad rows get delta = 0 and loss = 0.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// 16 bytes of columns of a row in either activation type (and as many fp32 weights)
__device__ __forceinline__ void load_cols(const bf16_t* p, float (&v)[8]) {
    const uint4 x = *reinterpret_cast<const uint4*>(p);
    const u32 w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[2 * k] = __builtin_bit_cast(float, w[k] << 16);
        v[2 * k + 1] = __builtin_bit_cast(float, w[k] & 0xFFFF0000u);
    }
}
__device__ __forceinline__ void load_cols(const float* p, float (&v)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load_cols(const float* p, float (&v)[4]) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
}
__device__ __forceinline__ void store_cols(bf16_t* p, const float (&v)[8]) {
    *reinterpret_cast<uint4*>(p) = make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
}
__device__ __forceinline__ void store_cols(float* p, const float (&v)[4]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

// lpr: lanes per row, a power of two; 16 bytes of columns per lane and step (width and strides are multiples of 32, rows
// 16-byte aligned: every activation is padded to 32 columns).  fp32: 16 lanes hold 64 partial sums, one for every column modulo
// 64, and add them in halves (a fixed order, whatever the row's width).  The row's logit and delta are known to all of its
// lanes, which then write the delta of the last hidden layer, d[s, n] = (delta * w_n (+ delta' * w'_n in the tangent pass))
// * (a[s, n] > 0), from the activations they just read (cache hits).  Bound: HBM with many rows -- the activations are read
// once instead of twice -- and the launch with few.
// Measured: the three passes of a step of 4 tasks x (32 + 32) rows, 32 units, fp32, 20.8 us in six launches (logits and
// deltas apart) -> 12.2 us in three; the seven of 512 tasks x (256 + 256) rows, 256 units, bf16, 0.37 ms.
template <typename T>
__global__ __launch_bounds__(256) void last_layer_kernel(LastArgs a, int lpr) {
    constexpr int V = 16 / sizeof(T), SUMS = sizeof(T) == 4 ? 4 : 1;   // columns per lane and step, partial sums per lane
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t s = gt / lpr;
    const int lane = (int)(gt % lpr);
    if (s >= a.n) return;
    const int g = a.row_task[s];
    const int r_in = (int)(s - a.row_offsets[g]);
    const int n_real = a.real_offsets[g + 1] - a.real_offsets[g];
    T* const d = a.d ? reinterpret_cast<T*>(a.d) + s * a.ld : nullptr;
    if (r_in >= n_real) {  // pad row
        if (lane == 0) {
            a.delta_out[s] = 0.f;
            if (a.z_out) a.z_out[s] = 0.f;
            if (a.loss_out) a.loss_out[s] = 0.f;
        }
        const float zero[V] = {};
        if (d)
            for (int n = lane * V; n < a.N; n += lpr * V) store_cols(d + n, zero);
        return;
    }
    const float* w = a.w + (int64_t)g * a.gW;
    const float* tw = a.ta ? a.tw + (int64_t)g * a.gTW : nullptr;
    const T* x = reinterpret_cast<const T*>(a.a) + s * a.ld;
    const T* tx = a.ta ? reinterpret_cast<const T*>(a.ta) + s * a.ld : nullptr;
    float sums[SUMS] = {};
    for (int n = lane * V; n < a.N; n += lpr * V) {
        float xv[V], wv[V];
        load_cols(x + n, xv);
        load_cols(w + n, wv);
        if (!tx) {
#pragma unroll
            for (int k = 0; k < V; ++k) sums[k % SUMS] = fmaf(xv[k], wv[k], sums[k % SUMS]);
        } else {
            float tv[V], twv[V];
            load_cols(tx + n, tv);
            load_cols(tw + n, twv);
#pragma unroll
            for (int k = 0; k < V; ++k) sums[k % SUMS] += tv[k] * wv[k] + xv[k] * twv[k];
        }
    }
    for (int m = lpr >> 1; m > 0; m >>= 1)   // within the row's lanes: all of them hold the sum
#pragma unroll
        for (int k = 0; k < SUMS; ++k) sums[k] += __shfl_xor(sums[k], m, 64);
#pragma unroll
    for (int h = SUMS / 2; h > 0; h /= 2)
#pragma unroll
        for (int k = 0; k < h; ++k) sums[k] += sums[k + h];
    const float acc = sums[0];
    const float inv_n = 1.f / (float)n_real;
    const float z = tx ? a.z_in[s] : acc + a.b[(int64_t)g * a.gW];
    const float e = __expf(-fabsf(z));
    const float sig = z >= 0.f ? 1.f / (1.f + e) : e / (1.f + e);
    float delta, delta2 = 0.f;
    if (!tx) {
        const float y = a.labels[a.real_offsets[g] + r_in];
        delta = (sig - y) * inv_n;
        if (lane == 0) {
            if (a.z_out) a.z_out[s] = z;
            if (a.loss_out) a.loss_out[s] = (fmaxf(z, 0.f) - y * z + log1pf(e)) * inv_n;
        }
    } else {
        delta = sig * (1.f - sig) * (acc + a.tb[(int64_t)g * a.gTW]) * inv_n;
        delta2 = a.delta_in[s];
    }
    if (lane == 0) a.delta_out[s] = delta;
    if (!d) return;
    for (int n = lane * V; n < a.N; n += lpr * V) {
        float xv[V], wv[V], v[V];
        load_cols(x + n, xv);
        load_cols(w + n, wv);
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] = delta * wv[k];
        if (tx) {
            load_cols(tw + n, wv);
#pragma unroll
            for (int k = 0; k < V; ++k) v[k] += delta2 * wv[k];
        }
#pragma unroll
        for (int k = 0; k < V; ++k)
            if (!(xv[k] > 0.f)) v[k] = 0.f;
        store_cols(d + n, v);
    }
}

void launch_last_layer(hipStream_t st, const LastArgs& a) {
    if (a.n <= 0) return;
    int lpr = a.bf16 ? 64 : 16;
    while (a.bf16 && lpr > 4 && (lpr / 2) * 8 >= a.N) lpr /= 2;
    const dim3 grid((unsigned)((a.n * lpr + 255) / 256));
    if (a.bf16) hipLaunchKernelGGL(last_layer_kernel<bf16_t>, grid, dim3(256), 0, st, a, lpr);
    else hipLaunchKernelGGL(last_layer_kernel<float>, grid, dim3(256), 0, st, a, lpr);
}

// A model without hidden layers: the gradient w.r.t. the pooled inputs, d[s, c] = dl[s]*w_g[c] (+ dl2[s]*w2_g[c]), c < N
__global__ void input_delta_kernel(int64_t n, int N, const int32_t* __restrict__ row_task, const float* __restrict__ dl,
                                   const float* __restrict__ w, int64_t gW, const float* __restrict__ dl2,
                                   const float* __restrict__ w2, int64_t gW2, float* d) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * N) return;
    const int64_t s = i / N;
    const int c = (int)(i - s * N);
    const int g = row_task[s];
    float v = dl[s] * w[(int64_t)g * gW + c];
    if (dl2) v += dl2[s] * w2[(int64_t)g * gW2 + c];
    d[i] = v;
}
void launch_input_delta(hipStream_t st, int64_t n, int N, const int32_t* row_task, const float* dl, const float* w, int64_t gW,
                        const float* dl2, const float* w2, int64_t gW2, float* d) {
    if (n <= 0 || N <= 0) return;
    hipLaunchKernelGGL(input_delta_kernel, dim3((unsigned)((n * N + 255) / 256)), dim3(256), 0, st, n, N, row_task, dl, w, gW,
                       dl2, w2, gW2, d);
}

// ------------------------------------------------------------------------------------------------
// cross-task reduction of the dense meta-gradient (Alg. 1, global back-propagation on theta; Sec. 2.1.3), the pieces of
// theta in one launch: out[j] (+)= sum_g v[g, j] + scale * sum_r vsum[r, j], tasks (and runs of tasks) added in order
// ------------------------------------------------------------------------------------------------
// Bound: HBM (the tasks' gradients once).  A thread takes four consecutive values of a piece (offsets and lengths are
// multiples of 32) and requests eight tasks' before it adds the first.
__global__ __launch_bounds__(256) void reduce_tasks_kernel(ReduceArgs a) {
    int pi = 0;
    while (pi + 1 < a.n && (int)blockIdx.x >= a.piece[pi + 1].block0) ++pi;
    const ReducePiece& p = a.piece[pi];
    const int64_t i = ((int64_t)((int)blockIdx.x - p.block0) * 256 + threadIdx.x) * 4;
    if (i >= p.n) return;
    const int64_t j = p.j0 + i;
    float4* out = reinterpret_cast<float4*>(a.out + j);
    float4 acc = a.accumulate ? *out : make_float4(0.f, 0.f, 0.f, 0.f);
    auto add = [&](const float* v, int G, float4 sum) {
        int g = 0;
        for (; g + 8 <= G; g += 8) {
            float4 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = *reinterpret_cast<const float4*>(v + (int64_t)(g + u) * a.ld + j);
#pragma unroll
            for (int u = 0; u < 8; ++u) { sum.x += x[u].x; sum.y += x[u].y; sum.z += x[u].z; sum.w += x[u].w; }
        }
        for (; g < G; ++g) {
            const float4 x = *reinterpret_cast<const float4*>(v + (int64_t)g * a.ld + j);
            sum.x += x.x; sum.y += x.y; sum.z += x.z; sum.w += x.w;
        }
        return sum;
    };
    if (p.G > 0) acc = add(a.v, p.G, acc);
    if (p.Gsum > 0) {
        const float4 s = add(a.vsum, p.Gsum, make_float4(0.f, 0.f, 0.f, 0.f));
        acc.x += a.scale * s.x; acc.y += a.scale * s.y; acc.z += a.scale * s.z; acc.w += a.scale * s.w;
    }
    *out = acc;
}

void launch_reduce_tasks(hipStream_t st, const ReduceArgs& base, const ReducePiece* list, int n) {
    for (int i0 = 0; i0 < n; i0 += REDUCE_PIECES) {
        ReduceArgs a = base;
        a.n = std::min(n - i0, (int)REDUCE_PIECES);
        int blocks = 0;
        for (int i = 0; i < a.n; ++i) {
            a.piece[i] = list[i0 + i];
            a.piece[i].block0 = blocks;
            blocks += (int)((a.piece[i].n + 1023) / 1024);
        }
        if (blocks > 0) hipLaunchKernelGGL(reduce_tasks_kernel, dim3(blocks), dim3(256), 0, st, a);
    }
}

// Per-row tables from per-task offsets, several at once: row off[g] + i of task g gets g, or first[g] + i
__global__ void expand_tasks_kernel(ExpandJobs jobs) {
    const ExpandJob& j = jobs.job[blockIdx.y];
    const int g = blockIdx.x;
    const int64_t lo = j.off64 ? j.off64[g] : j.off32[g], hi = j.off64 ? j.off64[g + 1] : j.off32[g + 1];
    if (g == 0 && blockIdx.y == 0 && (int)threadIdx.x < jobs.clear_words) jobs.clear[threadIdx.x] = 0u;
    for (int64_t s = lo + threadIdx.x; s < hi; s += blockDim.x) j.out[s] = j.first ? j.first[g] + (int32_t)(s - lo) : g;
}
void launch_expand_tasks(hipStream_t st, int G, const ExpandJobs& jobs) {
    if (G <= 0 || jobs.n <= 0) return;
    hipLaunchKernelGGL(expand_tasks_kernel, dim3(G, jobs.n), dim3(256), 0, st, jobs);
}

// Matrices between row-major and padded form, all layers' in one launch (the launch is what bounds it): dst [rows, cols]
// with leading dimension ld_dst takes src [src_rows, src_cols] with ld_src and zeros around it, and a bf16 copy
// (and, by one workgroup more, the sum of sum_n values in a fixed order)
__global__ __launch_bounds__(256) void copy_matrices_kernel(MatrixJobs jobs) {
    if ((int)blockIdx.x == jobs.sum_block) {   // one wavefront: lanes stride the array, then a butterfly
        if (threadIdx.x >= 64) return;
        float acc = 0.f;
        for (int i = threadIdx.x; i < jobs.sum_n; i += 64) acc += jobs.sum_src[i];
        acc = wave_sum(acc);
        if (threadIdx.x == 0) *jobs.sum_dst = acc;
        return;
    }
    int ji = 0;
    while (ji + 1 < jobs.n && (int)blockIdx.x >= jobs.job[ji + 1].block0) ++ji;
    const MatrixJob& m = jobs.job[ji];
    const int64_t e0 = (int64_t)((int)blockIdx.x - m.block0) * 1024, n = (int64_t)m.rows * m.cols;
    const int r0 = (int)(e0 / m.cols);
    const u32 c0 = (u32)(e0 - (int64_t)r0 * m.cols);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const u32 o = c0 + threadIdx.x + u * 256, dr = o / (u32)m.cols;
        if (e0 + threadIdx.x + u * 256 >= n) break;
        const int64_t r = r0 + (int64_t)dr;
        const int c = (int)(o - dr * (u32)m.cols);
        const float v = r < m.src_rows && c < m.src_cols ? m.src[r * m.ld_src + c] : 0.f;
        m.dst[r * m.ld_dst + c] = v;
        if (m.dst_bf) m.dst_bf[r * m.ld_dst + c] = f2bf(v);
    }
}
void launch_copy_matrices(hipStream_t st, const MatrixJob* list, int n, const float* sum_src, int sum_n, float* sum_dst) {
    for (int i0 = 0; i0 < n; i0 += MATRIX_JOBS) {
        MatrixJobs a;
        a.sum_src = sum_src; a.sum_n = sum_n; a.sum_dst = sum_dst; a.sum_block = -1;
        a.n = std::min(n - i0, (int)MATRIX_JOBS);
        int64_t blocks = 0;
        for (int i = 0; i < a.n; ++i) {
            a.job[i] = list[i0 + i];
            a.job[i].block0 = (int)blocks;
            blocks += ((int64_t)a.job[i].rows * a.job[i].cols + 1023) / 1024;
        }
        if (sum_dst && i0 + MATRIX_JOBS >= n) a.sum_block = (int)blocks++;
        if (blocks > 0) hipLaunchKernelGGL(copy_matrices_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a);
    }
}

__global__ void axpy_kernel(int64_t n, float a, const float* __restrict__ x, float* y) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] += a * x[i];
}
__global__ void scale_kernel(int64_t n, float a, const float* __restrict__ x, float* y) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) y[i] = a * x[i];
}
void launch_scale(hipStream_t st, int64_t n, float a, const float* x, float* y) {
    if (n <= 0) return;
    hipLaunchKernelGGL(scale_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 65536)), dim3(256), 0, st, n, a, x, y);
}
// y += a * x and x = 0 in one pass (the table-shaped sparse meta-gradient applied to the tables and cleared for the next
// iteration); 16 bytes per lane
__global__ void axpy_clear_kernel(int64_t n4, float a, float4* x, float4* y) {
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x) {
        const float4 g = x[i];
        if (g.x == 0.f && g.y == 0.f && g.z == 0.f && g.w == 0.f) continue;   // (rows nobody looked up: nothing to read or write)
        float4 v = y[i];
        v.x += a * g.x; v.y += a * g.y; v.z += a * g.z; v.w += a * g.w;
        y[i] = v;
        x[i] = zero;
    }
}
void launch_axpy_clear(hipStream_t st, int64_t n, float a, float* x, float* y) {   // n a multiple of 4, both 16-byte aligned
    if (n <= 0) return;
    const int64_t n4 = n / 4;
    const unsigned grid = (unsigned)std::min<int64_t>((n4 + 255) / 256, 256 * 64);
    hipLaunchKernelGGL(axpy_clear_kernel, dim3(grid), dim3(256), 0, st, n4, a, reinterpret_cast<float4*>(x), reinterpret_cast<float4*>(y));
}
void launch_axpy(hipStream_t st, int64_t n, float a, const float* x, float* y) {
    if (n <= 0) return;
    int64_t nb = (n + 255) / 256;
    if (nb > 65536) nb = 65536;
    hipLaunchKernelGGL(axpy_kernel, dim3((unsigned)nb), dim3(256), 0, st, n, a, x, y);
}
