// Dense side of the MAML step (G-Meta Alg. 1): inner forward / local back-propagation on theta, outer
// forward with the task's adapted theta', and the tangent passes of the second-order term.  Every
// product is a GROUPED GEMM: one group per task, each group with its own rows and (when theta has been
// adapted) its own weights.
#include <algorithm>

#include "gm_internal.h"

// ------------------------------------------------------------------------------------------------
// fp32 grouped GEMM on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, products and sums), C = A1*B1 (+ A2*B2)
// with a fused epilogue
// ------------------------------------------------------------------------------------------------
// Bound: the fp32 matrix rate (157 TFLOP/s; plain vector FMA reaches half of it and has to fetch 8 LDS values per 16
// FMAs) where the tiles fill the device, the latency of the k-loop's loads where a call has a few tasks only.
// A workgroup of four waves takes the k-range in pieces that are requested a whole piece ahead (registers), so that
// the memory latency runs beside the MFMAs of the piece before.  Two shapes:
//   SPLIT false  64 x 64 tile, one 32 x 32 block per wave, pieces of 64
//   SPLIT true   32 x 32 tile, the four waves take a quarter of every piece of 128 each and their blocks are added in
//                wave order through LDS: four times the workgroups and a quarter of the MFMA chain per wave
// Operands stay in LDS as they lie in memory.  Within 16 contraction values MFMA j takes values j and j + 8 (any pairing
// gives the same sum as long as both operands use it): a contraction-contiguous row then delivers a lane's 8 values as
// two 16-byte reads, and in a contraction-slowest tile the two halves of a wave read rows 8 apart, which with a row
// stride of (tile + 4) floats are 32 banks apart: neither form has bank conflicts.
// Measured on one second-order step, all 18 products together: 64 tasks x (128 + 128) rows through 845-256-128-1
// 2.03 -> 0.69 ms (a first-layer forward product 113 -> 43 us, 84 TFLOP/s), 37 tasks of about 50 rows through 189-100-52-1 0.45 ->
// 0.12 ms, 4 tasks x (32 + 32) rows through 141-64-32-1 0.29 -> 0.10 ms (before: vector FMA, loads not overlapped).
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

template <bool SPLIT>
struct F32Tile {
    static constexpr int T = SPLIT ? 32 : 64;       // rows and columns of the tile
    static constexpr int BK = SPLIT ? 128 : 64;     // contraction values per piece
    static constexpr int V = T * BK / 4 / 256;      // 16-byte pieces per thread and operand
    static constexpr int WORDS_CONT = T * (BK + 4), WORDS_SLOW = BK * (T + 4);
};

typedef __attribute__((__vector_size__(4 * sizeof(u32)))) u32 u32x4_t;

// One operand's pieces [T x BK] from memory to registers to LDS.  CONT: element (i, k) at p + i*ld + k, else at
// p + k*ld + i (extents along the contiguous direction and strides are multiples of 4: every matrix is padded to 32).
// The piece's base is uniform and moves on; a thread's offsets inside it stay.  What lies outside the operand is asked
// for beyond the buffer's end and reads as zero.
template <bool SPLIT, bool CONT>
struct F32Operand {
    using TT = F32Tile<SPLIT>;
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
            *reinterpret_cast<u32x4_t*>(s + (CONT ? row(u) * (TT::BK + 4) + col(u) : col(u) * (TT::T + 4) + row(u))) = v[u];
    }
    // a lane's 8 values (row or column i of the tile, contraction values k .. k + 7)
    __device__ __forceinline__ static void frag(const float* s, int i, int k, float (&f)[8]) {
        if (CONT) {
            const float4 a = *reinterpret_cast<const float4*>(s + i * (TT::BK + 4) + k), b = *reinterpret_cast<const float4*>(s + i * (TT::BK + 4) + k + 4);
            f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = s[(k + j) * (TT::T + 4) + i];
        }
    }
};

template <bool SPLIT, bool KA, bool KB>
__global__ __launch_bounds__(256, 4) void gemm_f32_kernel(GemmArgs a, int n_ntiles, int mt_per_group) {
    using TT = F32Tile<SPLIT>;
    using OpA = F32Operand<SPLIT, KA>;
    using OpB = F32Operand<SPLIT, KB>;
    constexpr int WA = KA ? TT::WORDS_CONT : TT::WORDS_SLOW, WB = KB ? TT::WORDS_CONT : TT::WORDS_SLOW;
    static_assert(!SPLIT || WA + WB >= 4 * 32 * 33, "the waves' blocks are added in the operand stage");
    __shared__ float4 stage[(WA + WB) / 4];
    float* const As = reinterpret_cast<float*>(stage);
    float* const Bs = As + WA;
    // workgroups are dealt round-robin to the 8 XCDs: neighbouring tiles (same rows, same weights) go to the same one
    const int per = gridDim.x >> 3, rest = gridDim.x & 7, xcd = blockIdx.x & 7;
    const int tile = xcd * per + (xcd < rest ? xcd : rest) + (blockIdx.x >> 3);
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
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, l32 = lane & 31, half = lane >> 5;
    const int mi = SPLIT ? l32 : (wv >> 1) * 32 + l32, ni = SPLIT ? l32 : (wv & 1) * 32 + l32;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;

    constexpr int KW = SPLIT ? TT::BK / 4 : TT::BK;    // contraction values of a piece that a wave takes
    const int kw0 = (SPLIT ? wv * KW : 0) + half * 8;
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
            float fa[2][8], fb[2][8];
            OpA::frag(As, mi, kw0, fa[0]);
            OpB::frag(Bs, ni, kw0, fb[0]);
#pragma unroll
            for (int kb = 0; kb < KW / 16; ++kb) {   // the next 16 values are on their way while these are multiplied
                if (kb + 1 < KW / 16) {
                    OpA::frag(As, mi, kw0 + (kb + 1) * 16, fa[(kb + 1) & 1]);
                    OpB::frag(Bs, ni, kw0 + (kb + 1) * 16, fb[(kb + 1) & 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[kb & 1][j], fb[kb & 1][j], acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    float* C = a.C + (int64_t)g * a.gC + r0 * a.rC;
    const float* bias = a.bias ? a.bias + (int64_t)g * a.gBias : nullptr;
    const float* mask = a.mask ? a.mask + r0 * a.ld_mask : nullptr;
    const float* Cin = a.Cin ? a.Cin + (int64_t)g * a.gCin : nullptr;
    auto emit = [&](int m, int n, float v) {
        if (m >= M || n >= N) return;
        switch (a.epi) {
            case EPI_BIAS_RELU: v = fmaxf(v + bias[n], 0.f); break;
            case EPI_BIAS_MASK: v = (mask[(int64_t)m * a.ld_mask + n] > 0.f) ? v + bias[n] : 0.f; break;
            case EPI_MASK: v = (mask[(int64_t)m * a.ld_mask + n] > 0.f) ? v : 0.f; break;
            case EPI_AXPBY: v = a.c1 * v + (Cin ? a.c0 * Cin[(int64_t)m * a.ldc + n] : 0.f); break;
            default: break;
        }
        C[(int64_t)m * a.ldc + n] = v;
    };
    // a lane holds column l32 of its block and rows 8*(i/4) + 4*half + i%4
    if (SPLIT) {
        float* red = As;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; ++i) red[(wv * 32 + (i >> 2) * 8 + half * 4 + (i & 3)) * 33 + l32] = acc[i];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = threadIdx.x + u * 256, r = e >> 5, c = e & 31;
            emit(m0 + r, n0 + c, ((red[r * 33 + c] + red[(32 + r) * 33 + c]) + red[(64 + r) * 33 + c]) + red[(96 + r) * 33 + c]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) emit(m0 + (wv >> 1) * 32 + (i >> 2) * 8 + half * 4 + (i & 3), n0 + ni, acc[i]);
    }
}

template <bool SPLIT>
static void gemm_f32_shape(hipStream_t st, const GemmArgs& a) {
    constexpr int T = F32Tile<SPLIT>::T;
    const int n_ntiles = (a.N + T - 1) / T, mt_per_group = a.tile_group ? 1 : (a.M + T - 1) / T;
    const int64_t n_mtiles = a.tile_group ? (int64_t)a.n_mtiles * (64 / T) : (int64_t)mt_per_group * a.G;
    if (n_mtiles <= 0 || n_ntiles <= 0) return;
    const dim3 grid((unsigned)(n_mtiles * n_ntiles));
    const bool ka = a.sAk[0] == 1, kb = a.sBk[0] == 1;
    if (ka && kb) hipLaunchKernelGGL((gemm_f32_kernel<SPLIT, true, true>), grid, dim3(256), 0, st, a, n_ntiles, mt_per_group);
    else if (ka) hipLaunchKernelGGL((gemm_f32_kernel<SPLIT, true, false>), grid, dim3(256), 0, st, a, n_ntiles, mt_per_group);
    else hipLaunchKernelGGL((gemm_f32_kernel<SPLIT, false, false>), grid, dim3(256), 0, st, a, n_ntiles, mt_per_group);
}

// The split tiles where 64 x 64 ones would not give every compute unit two workgroups: at 128 to 256 tiles 13.9 -> 12.0 us
// and 33.9 -> 18.6 us for products of the step above; from 512 tiles on the large ones are ahead (43 against 48 us, 53 against 73).
#define F32_SPLIT_TILES 512
void launch_gemm_f32(hipStream_t st, const GemmArgs& a) {
    const int64_t tiles = (int64_t)((a.N + 63) / 64) * (a.tile_group ? a.n_mtiles : (int64_t)((a.M + 63) / 64) * a.G);
    if (tiles < F32_SPLIT_TILES) gemm_f32_shape<true>(st, a);
    else gemm_f32_shape<false>(st, a);
}

// ------------------------------------------------------------------------------------------------
// element access in either activation type
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ float ldf(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float ldf(const bf16_t* p, int64_t i) { return bf2f(p[i]); }
__device__ __forceinline__ void stf(float* p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void stf(bf16_t* p, int64_t i, float v) { p[i] = f2bf(v); }

// ------------------------------------------------------------------------------------------------
// per-task column sums (bias gradients, last-layer weight gradient, per-task mean loss), all those of a pass in one launch:
// out[g,n] = c0*in[g,n] + c1 * sum_{s in g} ( X1[s,n]*w1[s] + X2[s,n]*w2[s] ), rows summed in a fixed order
// ------------------------------------------------------------------------------------------------
// Bound: HBM with many tasks; with a few the chain of dependent row batches of one workgroup, and the launches
// themselves.  A workgroup of 16 waves takes one task and one block of columns of one job.  A lane owns 16 bytes of
// columns (8 bf16 or 4 fp32); rows narrower than a wave's 64 lanes are taken several at a time.  The waves take the
// rows round-robin in batches of UB independent loads; lanes that share columns are added first, then the waves in wave
// order.  The partition depends on the job's width alone: results do not depend on how the tasks are cut into waves.
// Measured: the 16 launches of a step of 3 tasks x (512 + 512) rows through 1024-512-256 hidden units 0.37 -> 0.03 ms
// in 3 launches (4 waves and a launch per sum before); 512 tasks x 256 rows through 512-256, 28 launches, 0.62 -> 0.60 ms in 7.
template <typename T>
struct ColVec;
template <>
struct ColVec<float> {
    static constexpr int N = 4;
    typedef float4 Raw;
    __device__ static void open(const Raw& x, float (&v)[4]) { v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; }
};
template <>
struct ColVec<bf16_t> {
    static constexpr int N = 8;
    typedef uint4 Raw;
    __device__ static void open(const Raw& x, float (&v)[8]) {
        const u32 w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[2 * k] = __builtin_bit_cast(float, w[k] << 16);
            v[2 * k + 1] = __builtin_bit_cast(float, w[k] & 0xFFFF0000u);
        }
    }
};

enum { COLSUM_WAVES = 16 };

// rows r0 .. r1 of one column block, this wave's share; the lane's columns start at n of rows r0 + sub, r0 + sub + rpi, ...
template <typename T, bool TWO>
__device__ __forceinline__ void colsum_rows(const ColJob& j, int64_t r0, int64_t r1, int wv, int rpi, int sub, int n, float (&acc)[ColVec<T>::N]) {
    typedef typename ColVec<T>::Raw Raw;
    constexpr int V = ColVec<T>::N, UB = TWO ? 4 : 8;
    const T *X1 = reinterpret_cast<const T*>(j.X1) + n, *X2 = reinterpret_cast<const T*>(j.X2) + n;
    for (int64_t s0 = r0 + (int64_t)wv * UB * rpi; s0 < r1; s0 += (int64_t)COLSUM_WAVES * UB * rpi) {
        Raw x1[UB], x2[TWO ? UB : 1];
        float f1[UB], f2[TWO ? UB : 1];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int64_t s = s0 + u * rpi + sub;
            const bool ok = s < r1;
            const int64_t sc = ok ? s : r0;
            x1[u] = *reinterpret_cast<const Raw*>(X1 + sc * j.ldx);
            f1[u] = ok ? (j.w1 ? j.w1[sc] : 1.f) : 0.f;
            if (TWO) {
                x2[u] = *reinterpret_cast<const Raw*>(X2 + sc * j.ldx);
                f2[u] = ok ? (j.w2 ? j.w2[sc] : 1.f) : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            float a[V], b[V];
            ColVec<T>::open(x1[u], a);
            if (TWO) ColVec<T>::open(x2[u], b);
#pragma unroll
            for (int k = 0; k < V; ++k) {
                float v = a[k] * f1[u];
                if (TWO) v += b[k] * f2[u];
                acc[k] += v;
            }
        }
    }
}

template <typename T>
__global__ __launch_bounds__(64 * COLSUM_WAVES) void task_colsum_kernel(const int32_t* __restrict__ row_offsets, ColJobs jobs) {
    constexpr int V = ColVec<T>::N;
    __shared__ float part[COLSUM_WAVES - 1][64 * V];
    int ji = 0;
    while (ji + 1 < jobs.n && (int)blockIdx.x >= jobs.job[ji + 1].block0) ++ji;
    const ColJob& j = jobs.job[ji];
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
            for (int w = 0; w < COLSUM_WAVES - 1; ++w) sum += part[w][0];
            j.out[(int64_t)g * j.g_out] = j.c1 * sum + (j.in ? j.c0 * j.in[(int64_t)g * j.g_in] : 0.f);
        }
        return;
    }
    int lpr = 64;   // lanes per row: as few as cover it (a power of two)
    while (lpr > 1 && (lpr / 2) * V >= j.N) lpr /= 2;
    const int sub = lane / lpr, n = (((int)blockIdx.x - j.block0) * 64 + lane % lpr) * V;
    if (n < j.N) {
        if (j.X2) colsum_rows<T, true>(j, r0, r1, wv, 64 / lpr, sub, n, acc);
        else colsum_rows<T, false>(j, r0, r1, wv, 64 / lpr, sub, n, acc);
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
            for (int w = 0; w < COLSUM_WAVES - 1; ++w) sum += part[w][k * 64 + lane];
            j.out[(int64_t)g * j.g_out + n + k] = j.c1 * sum + (j.in ? j.c0 * j.in[(int64_t)g * j.g_in + n + k] : 0.f);
        }
    }
}

void launch_task_colsum(hipStream_t st, int bf16, int G, const int32_t* row_offsets, const ColJob* list, int n) {
    const int cols = 64 * (bf16 ? ColVec<bf16_t>::N : ColVec<float>::N);
    for (int i0 = 0; i0 < n; i0 += COL_JOBS) {
        ColJobs jobs;
        jobs.n = std::min(n - i0, (int)COL_JOBS);
        int blocks = 0;
        for (int i = 0; i < jobs.n; ++i) {
            jobs.job[i] = list[i0 + i];
            jobs.job[i].block0 = blocks;
            blocks += (jobs.job[i].N + cols - 1) / cols;
        }
        if (G <= 0 || blocks <= 0) continue;
        const dim3 grid(blocks, G), block(64 * COLSUM_WAVES);
        if (bf16) hipLaunchKernelGGL(task_colsum_kernel<bf16_t>, grid, block, 0, st, row_offsets, jobs);
        else hipLaunchKernelGGL(task_colsum_kernel<float>, grid, block, 0, st, row_offsets, jobs);
    }
}

// ------------------------------------------------------------------------------------------------
// last layer (d_L = 1) fused with the sigmoid / binary cross-entropy: one wavefront per row.
// Rows may be padded per task: row r of task g is sample real_offsets[g] + (r - row_offsets[g]) when that
// is below real_offsets[g+1]; pad rows get delta = 0 and loss = 0.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

__device__ __forceinline__ void load8(const bf16_t* p, float (&v)[8]) {
    const uint4 x = *reinterpret_cast<const uint4*>(p);
    const u32 w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[2 * k] = __builtin_bit_cast(float, w[k] << 16);
        v[2 * k + 1] = __builtin_bit_cast(float, w[k] & 0xFFFF0000u);
    }
}
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// lpr: lanes per row, a power of two (64: one row per wave; fewer when 8 columns per lane cover the row with less,
// so that a wave takes 64 / lpr rows at once)
template <typename T>
__global__ void last_fwd_kernel(LastFwdArgs a, int lpr) {
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t s = gt / lpr;
    const int lane = (int)(gt % lpr);
    if (s >= a.n) return;
    const int g = a.row_task[s];
    const int r_in = (int)(s - a.row_offsets[g]);
    const int n_real = a.real_offsets[g + 1] - a.real_offsets[g];
    if (r_in >= n_real) {  // pad row
        if (lane == 0) {
            a.delta_out[s] = 0.f;
            if (a.z_out) a.z_out[s] = 0.f;
            if (a.loss_out) a.loss_out[s] = 0.f;
        }
        return;
    }
    const float* w = a.w + (int64_t)g * a.gW;
    const T* x = reinterpret_cast<const T*>(a.a) + s * a.ld;
    float acc = 0.f;
    // bf16 rows whose width and stride are multiples of 8: 16-byte loads (pad columns hold zeros on both sides)
    const bool vec = sizeof(T) == 2 && (a.N % 8 == 0) && (a.ld % 8 == 0) && (a.gW % 4 == 0) && (!a.ta || a.gTW % 4 == 0) &&
                     reinterpret_cast<uintptr_t>(a.w) % 16 == 0 && (!a.ta || reinterpret_cast<uintptr_t>(a.tw) % 16 == 0);
    if (vec) {
        const bf16_t* xb = reinterpret_cast<const bf16_t*>(x);
        const bf16_t* txb = a.ta ? reinterpret_cast<const bf16_t*>(a.ta) + s * a.ld : nullptr;
        const float* tw = a.ta ? a.tw + (int64_t)g * a.gTW : nullptr;
        for (int n = lane * 8; n < a.N; n += lpr * 8) {
            float xv[8], wv[8];
            load8(xb + n, xv);
            load8(w + n, wv);
            if (!a.ta) {
#pragma unroll
                for (int k = 0; k < 8; ++k) acc = fmaf(xv[k], wv[k], acc);
            } else {
                float tv[8], twv[8];
                load8(txb + n, tv);
                load8(tw + n, twv);
#pragma unroll
                for (int k = 0; k < 8; ++k) acc += tv[k] * wv[k] + xv[k] * twv[k];
            }
        }
    } else if (!a.ta) {
        for (int n = lane; n < a.N; n += 64) acc = fmaf(ldf(x, n), w[n], acc);
    } else {
        const T* tx = reinterpret_cast<const T*>(a.ta) + s * a.ld;
        const float* tw = a.tw + (int64_t)g * a.gTW;
        for (int n = lane; n < a.N; n += 64) acc += ldf(tx, n) * w[n] + ldf(x, n) * tw[n];
    }
    for (int d = lpr >> 1; d > 0; d >>= 1) acc += __shfl_xor(acc, d, 64);   // within the row's lanes
    if (lane != 0) return;
    const float inv_n = 1.f / (float)n_real;
    if (!a.ta) {
        const float z = acc + a.b[(int64_t)g * a.gW];
        const float y = a.labels[a.real_offsets[g] + r_in];
        const float e = __expf(-fabsf(z));
        const float sig = z >= 0.f ? 1.f / (1.f + e) : e / (1.f + e);
        if (a.z_out) a.z_out[s] = z;
        a.delta_out[s] = (sig - y) * inv_n;
        if (a.loss_out) a.loss_out[s] = (fmaxf(z, 0.f) - y * z + log1pf(e)) * inv_n;
    } else {
        const float tz = acc + a.tb[(int64_t)g * a.gTW];
        const float z = a.z_in[s];
        const float e = __expf(-fabsf(z));
        const float sig = z >= 0.f ? 1.f / (1.f + e) : e / (1.f + e);
        a.delta_out[s] = sig * (1.f - sig) * tz * inv_n;
    }
}

void launch_last_fwd(hipStream_t st, const LastFwdArgs& a) {
    if (a.n <= 0) return;
    int lpr = 64;
    // the 16-byte path of the kernel (same conditions) reads 8 columns per lane: narrow rows need fewer lanes
    if (a.bf16 && a.N % 8 == 0 && a.ld % 8 == 0 && a.gW % 4 == 0 && (!a.ta || a.gTW % 4 == 0) &&
        reinterpret_cast<uintptr_t>(a.w) % 16 == 0 && (!a.ta || reinterpret_cast<uintptr_t>(a.tw) % 16 == 0)) {
        while (lpr > 8 && (lpr / 2) * 8 >= a.N) lpr /= 2;
    }
    const dim3 grid((unsigned)((a.n * lpr + 255) / 256));
    if (a.bf16) hipLaunchKernelGGL(last_fwd_kernel<bf16_t>, grid, dim3(256), 0, st, a, lpr);
    else hipLaunchKernelGGL(last_fwd_kernel<float>, grid, dim3(256), 0, st, a, lpr);
}

template <typename T>
__global__ void last_bwd_kernel(int64_t n, int N, int64_t ld_a, int64_t ld_d, const int32_t* __restrict__ row_task,
                                const float* __restrict__ dl, const float* __restrict__ w, int64_t gW,
                                const float* __restrict__ dl2, const float* __restrict__ w2, int64_t gW2,
                                const T* __restrict__ act, T* d, float* d_f32) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * N) return;
    const int64_t s = i / N;
    const int c = (int)(i - s * N);
    const int g = row_task[s];
    float v = dl[s] * w[(int64_t)g * gW + c];
    if (dl2) v += dl2[s] * w2[(int64_t)g * gW2 + c];
    if (act && !(ldf(act, s * ld_a + c) > 0.f)) v = 0.f;
    if (d) stf(d, s * ld_d + c, v);
    if (d_f32) d_f32[s * ld_d + c] = v;
}

// bf16 rows, 8 columns per thread (N, strides and the weight strides allow 16-byte accesses)
__global__ void last_bwd_vec_kernel(int64_t n, int N, int64_t ld_a, int64_t ld_d, const int32_t* __restrict__ row_task,
                                    const float* __restrict__ dl, const float* __restrict__ w, int64_t gW,
                                    const float* __restrict__ dl2, const float* __restrict__ w2, int64_t gW2,
                                    const bf16_t* __restrict__ act, bf16_t* d, float* d_f32) {
    const int per_row = N / 8;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * per_row) return;
    const int64_t s = i / per_row;
    const int c = (int)(i - s * per_row) * 8;
    const int g = row_task[s];
    float wv[8], v[8];
    load8(w + (int64_t)g * gW + c, wv);
    const float a1 = dl[s];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = a1 * wv[k];
    if (dl2) {
        load8(w2 + (int64_t)g * gW2 + c, wv);
        const float a2 = dl2[s];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] += a2 * wv[k];
    }
    if (act) {
        float av[8];
        load8(act + s * ld_a + c, av);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (!(av[k] > 0.f)) v[k] = 0.f;
    }
    if (d) *reinterpret_cast<uint4*>(d + s * ld_d + c) = make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
    if (d_f32) {
        *reinterpret_cast<float4*>(d_f32 + s * ld_d + c) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(d_f32 + s * ld_d + c + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
}

// d[s,n] = (dl[s]*w_g[n] (+ dl2[s]*w2_g[n])) * (act[s,n] > 0); act null: no mask.  Output in the
// activation type (d) and/or fp32 (d_f32).
void launch_last_bwd(hipStream_t st, int bf16, int64_t n, int N, int64_t ld_a, int64_t ld_d, const int32_t* row_task,
                     const float* dl, const float* w, int64_t gW, const float* dl2, const float* w2, int64_t gW2,
                     const void* act, void* d, float* d_f32) {
    if (n <= 0 || N <= 0) return;
    const dim3 grid((unsigned)((n * N + 255) / 256));
    if (bf16 && N % 8 == 0 && ld_a % 8 == 0 && ld_d % 8 == 0 && gW % 4 == 0 && (!dl2 || gW2 % 4 == 0) &&
        reinterpret_cast<uintptr_t>(w) % 16 == 0 && (!w2 || reinterpret_cast<uintptr_t>(w2) % 16 == 0))
        hipLaunchKernelGGL(last_bwd_vec_kernel, dim3((unsigned)((n * (N / 8) + 255) / 256)), dim3(256), 0, st, n, N, ld_a, ld_d,
                           row_task, dl, w, gW, dl2, w2, gW2, (const bf16_t*)act, (bf16_t*)d, d_f32);
    else if (bf16)
        hipLaunchKernelGGL(last_bwd_kernel<bf16_t>, grid, dim3(256), 0, st, n, N, ld_a, ld_d, row_task, dl, w, gW, dl2,
                           w2, gW2, (const bf16_t*)act, (bf16_t*)d, d_f32);
    else
        hipLaunchKernelGGL(last_bwd_kernel<float>, grid, dim3(256), 0, st, n, N, ld_a, ld_d, row_task, dl, w, gW, dl2, w2,
                           gW2, (const float*)act, (float*)d, d_f32);
}

// ------------------------------------------------------------------------------------------------
// cross-task reduction of the dense meta-gradient (Alg. 1, global back-propagation on theta; Sec. 2.1.3):
// out[j] (+)= sum_g v[g, j], tasks added in task order; with a scale other than 1: out[j] (+)= scale * (sum_g v[g, j])
// ------------------------------------------------------------------------------------------------
__global__ void reduce_tasks_kernel(const float* __restrict__ v, int64_t ld, int G, int64_t n, float* out,
                                    int accumulate, float scale) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    // eight tasks' values are requested before the first is added (the order of the sum stays the task order)
    float acc = (accumulate && scale == 1.f) ? out[j] : 0.f;
    int g = 0;
    for (; g + 8 <= G; g += 8) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = v[(int64_t)(g + u) * ld + j];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += x[u];
    }
    for (; g < G; ++g) acc += v[(int64_t)g * ld + j];
    out[j] = scale == 1.f ? acc : (accumulate ? out[j] : 0.f) + scale * acc;
}

void launch_reduce_tasks(hipStream_t st, const float* v, int64_t ld, int G, int64_t n, float* out, int accumulate,
                         float scale) {
    if (n <= 0) return;
    hipLaunchKernelGGL(reduce_tasks_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, v, ld, G, n, out,
                       accumulate, scale);
}

__global__ void fill_sample_task_kernel(const int32_t* row_offsets, int32_t* sample_task) {
    const int g = blockIdx.x;
    for (int s = row_offsets[g] + threadIdx.x; s < row_offsets[g + 1]; s += blockDim.x) sample_task[s] = g;
}
void launch_fill_sample_task(hipStream_t st, const int32_t* row_offsets, int G, int32_t* sample_task) {
    if (G <= 0) return;
    hipLaunchKernelGGL(fill_sample_task_kernel, dim3(G), dim3(256), 0, st, row_offsets, sample_task);
}

// W [din, dout] row-major  <->  padded [ld_in, ld_out] (pad rows / columns zero)
__global__ void pack_weights_kernel(const float* W, int din, int dout, int ld_in, int ld_out, float* dst) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)ld_in * ld_out) return;
    const int r = (int)(i / ld_out), c = (int)(i % ld_out);
    dst[i] = (r < din && c < dout) ? W[(int64_t)r * dout + c] : 0.f;
}
void launch_pack_weights(hipStream_t st, const float* W, int din, int dout, int ld_in, int ld_out, float* dst) {
    const int64_t n = (int64_t)ld_in * ld_out;
    hipLaunchKernelGGL(pack_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, W, din, dout, ld_in,
                       ld_out, dst);
}
__global__ void unpack_weights_kernel(const float* src, int din, int dout, int ld_out, float* W) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)din * dout) return;
    const int r = (int)(i / dout), c = (int)(i % dout);
    W[i] = src[(int64_t)r * ld_out + c];
}
void launch_unpack_weights(hipStream_t st, const float* src, int din, int dout, int ld_out, float* W) {
    const int64_t n = (int64_t)din * dout;
    if (n <= 0) return;
    hipLaunchKernelGGL(unpack_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, din, dout,
                       ld_out, W);
}

__global__ void axpy_kernel(int64_t n, float a, const float* __restrict__ x, float* y) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] += a * x[i];
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

__global__ void sum_to_scalar_kernel(const float* x, int n, float* out, int accumulate) {
    // one wavefront, fixed order: lanes stride the array, then a butterfly
    float acc = 0.f;
    for (int i = threadIdx.x; i < n; i += 64) acc += x[i];
    acc = wave_sum(acc);
    if (threadIdx.x == 0) *out = accumulate ? *out + acc : acc;
}
void launch_sum_to_scalar(hipStream_t st, const float* x, int n, float* out, int accumulate) {
    hipLaunchKernelGGL(sum_to_scalar_kernel, dim3(1), dim3(64), 0, st, x, n, out, accumulate);
}
