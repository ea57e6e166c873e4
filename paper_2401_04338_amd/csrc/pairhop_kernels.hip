// Task-local embedding-row arithmetic as a dense contraction on the matrix cores.
//
// Every row-space operation of the inner loop and of the second-order chain (G-Meta Alg. 1: local
// back-propagation on xi^Sup, the overlap update of Sec. 2.1.2, and their tangents) is, for one
// (task, field),
//     Y[i, :] = Y_in[i, :] + c * sum_j M[i][j] * Z[j, :],      M = P_out * P_in^T,
// where P_set[bag][row] counts how often the bag looks the row up, restricted to the rows of the
// task's support set.  M[i][j] is therefore the number of (lookup of out-bag i, lookup of in-bag j)
// pairs that hit the same row: a small integer that depends on the indices only.  It is the same for
// every inner step and for the whole second-order chain, so it is counted ONCE per call
// (pair_count_kernel, integer atomics in LDS: exact and order-free) and stored as bytes; each of the
// hops is then a [n_out, n_in] x [n_in, D] product on MFMA (pair_hop_kernel).
//
// fp32 accuracy on bf16 matrix cores: an fp32 value splits EXACTLY into three bf16 pieces (its 24
// significand bits cut 8+8+8 by truncation, every remainder exact), counts up to 255 are exact in
// bf16, and every product count*piece is exact in the fp32 accumulator; only the accumulation rounds,
// as it would in an fp32 loop.
//
// Counts above 255 or tasks too large for this path are handled by the sparse two-hop kernel instead.
#include <algorithm>

#include "gm_internal.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 ph_short8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float ph_float16;

__host__ __device__ __forceinline__ int pad64(int n) { return (n + 63) & ~63; }

// ------------------------------------------------------------------------------------------------
// counting: M[i][j] for one (task, field) and one pair of sets, in tiles of out-rows held in LDS
//
// M = sum over the rows u of the task's support set of  c_out(:, u) (x) c_in(:, u),  with c_set(b, u) the
// number of times bag b looks row u up.  Under a skewed row distribution a few hot rows carry nearly all
// of the pairs (a row looked up a times by one set and b times by the other adds a*b of them), and LDS
// atomics retire only about one lane per cycle, so the hot rows do not go through pair-by-pair atomics:
// a batch of HB hot rows at a time, their count vectors are laid out densely ([bags, HB] bytes, one atomic per
// lookup) and multiplied on the matrix cores as 8-bit integers (v_mfma_i32_32x32x32_i8: a count is at
// most the bag's length, which this path limits to 127; sums are exact in 32 bits).
// Only the remaining rows (fewer than PC_HOT lookups from either set, at most 9 pairs each) are counted
// pair by pair with atomics on the byte cells, on top of the stored hot part.  Everything is integer
// arithmetic: the result does not depend on any order.
//
// The kernel is bound by latency, not by arithmetic, so everything it walks more than once is staged in
// LDS when the workgroup starts: the bag of every lookup of both lists (16 bits each) and one record per
// row with pairs (hot: the bounds of its two lookup ranges; cold: packed starts and sizes).  After that
// only LDS is read until the matrix is written out.  Hot rows are numbered in the lists' order and every lookup
// of one carries its number within its batch beside its bag, so that a batch is one range of each list that all
// threads walk side by side; a wave per row waited for the hottest one, three barriers for every 32 rows.  The
// count blocks lie where the tile will: with 64 rows a batch they take no more LDS than it.
// Measured, one launch (before: 32 rows a batch, a wave per row and batch, one workgroup per compute unit): 512 tasks of 256 + 256
// rows x 26 fields, bags of 1..20, two kinds 2.14 -> 1.21 ms; 201 tasks of 75..225 + 122..365 rows 0.63 -> 0.37; 128 tasks of
// 512 + 512 rows x 64 fields, bags of 1..32 3.38 -> 2.30 (1.0 ms of it the time its 4.3 GB take to write); 3 of them 111 -> 78 us.
// Tried: a bag's further lookups of a row found beside the first and only those added, the first ones stored: the second pass
// costs more than the atomics it saves (2.30 -> 2.65).
// ------------------------------------------------------------------------------------------------
#define PC_TPW 4          // MFMA tiles per wave: a workgroup of NT threads covers NT / 16 tiles per row tile
#define PC_SMALL_ROWS 128 // samples per set of a 'small' task: 16 tiles, four waves
#define PC_SMALL_N 1984   // lookups per set of a 'small' (task, field)
#define PC_TWO_LDS (PAIR_LDS_BYTES / 2)   // LDS of a workgroup that shares its compute unit with another
#define PC_HOT 4     // a row is hot when one of the two sets looks it up at least this often
// bytes per bag in a count block of hb rows (16-byte fragment reads; 12 or 20 words spread them over the banks)
__host__ __device__ constexpr int pc_stride(int hb) { return hb + 16; }
// LDS of one row tile of R out-rows: the byte cells, or the count blocks of a batch that come before them
__host__ __device__ __forceinline__ size_t pc_tile_bytes(int R, int colsP, int hb) {
    const size_t cells = (size_t)colsP * (R + 4), counts = (size_t)(R + colsP) * pc_stride(hb);
    return cells > counts ? cells : counts;
}

typedef int pc_int4 __attribute__((ext_vector_type(4)));
typedef int pc_int16 __attribute__((ext_vector_type(16)));

// (LDS only: the matrices' stores go on behind it)
__device__ __forceinline__ void pc_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// HBITS: log2 of the hot rows of a batch; a lookup's 16 bits hold its bag in the lower 15 - HBITS
// (at least four waves a SIMD: with registers to spare the four-wave workgroups of small tasks took 189 each, two workgroups a compute
// unit where the LDS holds four: 700 tasks of a median 32 rows 835 -> 463 us, 64 tasks of 128 + 128 rows 47 -> 32)
template <int NT, int HBITS>
__global__ __launch_bounds__(NT, 4) void pair_count_kernel(PairCountArgs a) {
    constexpr int HB = 1 << HBITS, HBS = pc_stride(HB), BAG_BITS = 15 - HBITS, BAG_MASK = (1 << BAG_BITS) - 1;
    extern __shared__ __attribute__((aligned(16))) u32 pc_lds[];
    __shared__ int sh_ncold, sh_wave_hot[2][NT / 64];
    const int f = blockIdx.x, t = a.order[blockIdx.y];
    const bool qs = blockIdx.z == 0;   // query x support (and its transpose), 1: support x support
    if (!a.task_path[t]) return;   // (another field's counts did not fit)
    const size_t tf = (size_t)t * a.F + f;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, ln = lane & 31, h = lane >> 5;
    const int ns = a.real_off_s[t + 1] - a.real_off_s[t], nq = a.real_off_q[t + 1] - a.real_off_q[t];
    const int n_out = qs ? nq : ns;
    const int colsP = pad64(ns), rowsP = pad64(n_out);
    if (colsP == 0 || rowsP == 0) return;
    const u32 B = a.base_s[tf], Bq = a.base_q[tf];
    const int nu = (int)a.n_slots[tf];
    const int n_in_entries = (int)a.cnt_s[tf];
    const int n_out_entries = qs ? (int)a.cnt_q[tf] : n_in_entries;
    if (a.cls) {   // uneven tasks: the small (task, field)s have a launch of their own, with small workgroups
        const bool small = max(ns, nq) <= PC_SMALL_ROWS && max(n_in_entries, n_out_entries) <= a.small_n;
        if (small != (a.cls == 1)) return;
    }
    // LDS, from the end (6 * n_max bytes): the bag of every out lookup and of every in lookup (16 bits each, in the
    // order of the row-sorted lists; one array when both sets are the support set), then the records: hot rows
    // from the front (two words: in range, out range), cold rows with pairs from the back (one word).
    // From the start: the two dense count blocks of a batch, [R] and [colsP] bags of HBS bytes (one block when both sets
    // are the support set); then in their place the tile of R out-rows, TRANSPOSED, one byte per cell: cell (i, j) at
    // j * ldT + i with ldT = R + 4 (an odd number of words: the MFMA result, the transposed read-out and the atomics all
    // spread over the banks).
    const int nmax = a.n_max;                                  // a multiple of 8
    uint16_t* out_rows = reinterpret_cast<uint16_t*>(pc_lds) + (a.lds_bytes / 2 - nmax);
    uint16_t* in_rows = qs ? out_rows - nmax : out_rows;
    const int RW = qs ? nmax / 2 : nmax;                       // record words
    u32* recs = reinterpret_cast<u32*>(in_rows) - RW;
    if (threadIdx.x == 0) sh_ncold = 0;
    // The first lookups of both lists are on their way while the rows are classified: eight loads per thread and list, as the
    // workgroup has little company on its compute unit to hide the latency of these first reads.
    const int2 *in_list = a.sup_sorted + B, *out_list = a.qry_sorted + Bq;   // {row, slot}, slot-sorted
    int2 in_first[8], out_first[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        in_first[q] = out_first[q] = make_int2(0, -1);
        if ((int)threadIdx.x + q * NT < n_in_entries) in_first[q] = in_list[threadIdx.x + q * NT];
        if (qs && (int)threadIdx.x + q * NT < n_out_entries) out_first[q] = out_list[threadIdx.x + q * NT];
    }
    uint8_t* const mark = reinterpret_cast<uint8_t*>(pc_lds);   // [nu] 0, or HB | the row's number within its batch of hot rows (where the tile will be)
    pc_barrier();
    int nhot = 0;                                              // (the same in all threads)
    for (int ub = 0; ub < nu; ub += 4 * NT) {                  // four rows per thread, their bounds in flight together
        const int u0 = ub + 4 * (int)threadIdx.x;
        int lo_[5], lo2_[4], hi2_[4];
#pragma unroll
        for (int q = 0; q < 5; ++q) lo_[q] = a.slot_start[B + tf + min(u0 + q, nu)] - (int)B;
        if (qs) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                lo2_[q] = a.qseg_lo[B + min(u0 + q, nu - 1)] - (int)Bq;
                hi2_[q] = a.qseg_hi[B + min(u0 + q, nu - 1)] - (int)Bq;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) { lo2_[q] = lo_[q]; hi2_[q] = lo_[q + 1]; }
        }
        // hot rows numbered in list order: those of the waves before this one, of the lanes before this one, the thread's own
        bool hot[4];
        int k = nhot, mine = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int na = lo_[q + 1] - lo_[q], nb = hi2_[q] - lo2_[q];
            hot[q] = u0 + q < nu && na > 0 && nb > 0 && (na >= PC_HOT || nb >= PC_HOT);
            const unsigned long long in_wave = __ballot(hot[q]);
            k += __popcll(in_wave & ((1ull << lane) - 1ull));
            mine += __popcll(in_wave);
        }
        int* const counts = sh_wave_hot[(ub / (4 * NT)) & 1];  // (two sets in turn: one barrier each)
        if (lane == 0) counts[wv] = mine;
        pc_barrier();
        for (int w = 0; w < NT / 64; ++w) {
            const int c = counts[w];
            if (w < wv) k += c;
            nhot += c;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (u0 + q >= nu) continue;
            const int na = lo_[q + 1] - lo_[q], nb = hi2_[q] - lo2_[q];
            mark[u0 + q] = hot[q] ? (uint8_t)(HB | (k & (HB - 1))) : (uint8_t)0;
            if (hot[q]) {
                if (2 * k + 1 < RW) {
                    recs[2 * k] = (u32)lo_[q] | ((u32)lo_[q + 1] << 16);
                    recs[2 * k + 1] = (u32)lo2_[q] | ((u32)hi2_[q] << 16);
                }
                ++k;
            } else if (na > 0 && nb > 0) {
                const int kc = atomicAdd(&sh_ncold, 1);
                if (kc < RW) recs[RW - 1 - kc] = (u32)lo_[q] | ((u32)lo2_[q] << 14) | ((u32)na << 28) | ((u32)nb << 30);
            }
        }
    }
    pc_barrier();
    const int ncold = sh_ncold;
    if (2 * nhot + ncold > RW) {   // the records do not fit (they may have overwritten each other): sparse kernel
        if (threadIdx.x == 0) {
            a.task_path[t] = 0u;
            a.status[ST_PAIR_OVF] = 1u;
        }
        return;
    }
    const size_t budget = (size_t)a.lds_bytes - 6 * (size_t)nmax;
    int R = min(rowsP, a.max_tile_rows);   // at most NT / 16 MFMA tiles per row tile
    while (R > 32 && (pc_tile_bytes(R, colsP, HB) > budget || R * colsP > NT * 64)) R -= 32;
    if (pc_tile_bytes(R, colsP, HB) > budget) {   // not even 32 rows fit: sparse kernel
        if (threadIdx.x == 0) {
            a.task_path[t] = 0u;
            a.status[ST_PAIR_OVF] = 1u;
        }
        return;
    }
    // the lists: every lookup's bag, and where its row is hot the row's number within its batch
    auto stage = [&](const int2* list, const int2 (&first)[8], int n, int row0, uint16_t* dst) {
        auto put = [&](int e, int2 v) { dst[e] = (uint16_t)((v.x - row0) | (v.y >= 0 ? (int)mark[v.y] << BAG_BITS : 0)); };
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if ((int)threadIdx.x + q * NT < n) put(threadIdx.x + q * NT, first[q]);
        for (int e0 = threadIdx.x + 8 * NT; e0 < n; e0 += 8 * NT) {
            int2 v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = list[min(e0 + q * NT, n - 1)];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (e0 + q * NT < n) put(e0 + q * NT, v[q]);
        }
    };
    stage(in_list, in_first, n_in_entries, a.row_off_s[t], in_rows);
    if (qs) stage(out_list, out_first, n_out_entries, a.row_off_q[t], out_rows);
    const int ldT = R + 4;
    uint8_t* tile = reinterpret_cast<uint8_t*>(pc_lds);
    uint8_t* c_in = tile;
    uint8_t* c_block = tile + (size_t)colsP * HBS;   // of the out bags, where they are another set's
    uint8_t* M = a.mat + (size_t)(qs ? a.off_qs[t] : a.off_ss[t]) * PAIR_BLOCK + (size_t)f * rowsP * colsP;
    uint8_t* Mt = (qs && a.want_sq) ? a.mat + (size_t)a.off_sq[t] * PAIR_BLOCK + (size_t)f * colsP * rowsP : nullptr;  // [colsP rows][rowsP cols]
    const int tiles_c = colsP / 32;
    bool ovf = false;
    for (int i0 = 0; i0 < rowsP; i0 += R) {
        const int rows_here = min(R, rowsP - i0);
        // A wave's four tiles are two pairs side by side: two by two where the tile rows are even in number, so that every
        // fragment read feeds two products.
        const int pairs_c = tiles_c / 2, tile_rows = rows_here / 32;
        const bool square = (tile_rows & 1) == 0;
        int my_tr[2], my_tc[2];      // of each pair: its tile row, its first tile column
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int unit = square ? wv : 2 * wv + p, r = unit / pairs_c * (square ? 2 : 1) + (square ? p : 0);
            my_tr[p] = r < tile_rows ? r : -1;
            my_tc[p] = unit % pairs_c * 2;
        }
        pc_int16 acc[PC_TPW];
#pragma unroll
        for (int q = 0; q < PC_TPW; ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[q][v] = 0;
        const uint8_t* c_out = qs ? c_block : c_in + (size_t)i0 * HBS;
        for (int hb = 0; hb < nhot; hb += HB) {
            pc_barrier();   // the previous batch's fragments (or the previous tile) have been read
            for (int i = threadIdx.x; i < (colsP + (qs ? rows_here : 0)) * HBS / 16; i += NT)   // both count blocks, contiguous
                reinterpret_cast<uint4*>(c_in)[i] = make_uint4(0u, 0u, 0u, 0u);
            pc_barrier();
            // one atomic per lookup (a count is at most the bag's length)
            auto count = [&](const uint16_t* list, int lo, int hi, uint8_t* block, int first, int rows) {
                for (int e0 = lo + (int)threadIdx.x; e0 < hi; e0 += 4 * NT) {
                    u32 v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = e0 + q * NT < hi ? list[e0 + q * NT] : 0u;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int i = (int)(v[q] & BAG_MASK) - first, k = (int)(v[q] >> BAG_BITS) & (HB - 1);
                        if ((v[q] & 0x8000u) && (unsigned)i < (unsigned)rows)
                            atomicAdd(reinterpret_cast<u32*>(block) + ((i * HBS + k) >> 2), 1u << (8 * (k & 3)));
                    }
                }
            };
            const int last = min(hb + HB, nhot) - 1;
            count(in_rows, (int)(recs[2 * hb] & 0xFFFFu), (int)(recs[2 * last] >> 16), c_in, 0, colsP);
            if (qs) count(out_rows, (int)(recs[2 * hb + 1] & 0xFFFFu), (int)(recs[2 * last + 1] >> 16), c_block, i0, rows_here);
            pc_barrier();
            if (my_tr[0] >= 0) {
#pragma unroll
                for (int kk = 0; kk < HB; kk += 32) {
                    auto frag = [&](const uint8_t* block, int tile_no) { return *reinterpret_cast<const pc_int4*>(block + (tile_no * 32 + ln) * HBS + kk + h * 16); };
                    pc_int4 qb[2] = {frag(c_in, my_tc[0]), frag(c_in, my_tc[0] + 1)};
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        if (my_tr[p] < 0) continue;
                        if (p == 1 && !square) { qb[0] = frag(c_in, my_tc[1]); qb[1] = frag(c_in, my_tc[1] + 1); }
                        const pc_int4 qa = frag(c_out, my_tr[p]);
#pragma unroll
                        for (int c = 0; c < 2; ++c) acc[2 * p + c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(qa, qb[c], acc[2 * p + c], 0, 0, 0);
                    }
                }
            }
        }
        // ---- the hot part becomes the tile's initial content (every cell of the tile's rows is written); a lane
        //      holds four consecutive rows of one column: one word of the transposed tile.  255 stands for
        //      "255 or more" and is reported when the tile is read out.
        pc_barrier();   // the previous tile has been read out, and the last batch's counts
#pragma unroll
        for (int q = 0; q < PC_TPW; ++q) {
            if (my_tr[q >> 1] >= 0) {
                uint8_t* col = tile + (size_t)((my_tc[q >> 1] + (q & 1)) * 32 + ln) * ldT + my_tr[q >> 1] * 32 + 4 * h;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const u32 b0 = min((u32)acc[q][4 * g + 0], 255u), b1 = min((u32)acc[q][4 * g + 1], 255u);
                    const u32 b2 = min((u32)acc[q][4 * g + 2], 255u), b3 = min((u32)acc[q][4 * g + 3], 255u);
                    *reinterpret_cast<u32*>(col + 8 * g) = b0 | (b1 << 8) | (b2 << 16) | (b3 << 24);
                }
            }
        }
        pc_barrier();
        // ---- the other rows, pair by pair; a cell that was at 254 or more before an increment may have
        //      wrapped: reported
        for (int k = threadIdx.x; k < ncold; k += NT) {
            const u32 r = recs[RW - 1 - k];
            const int lo = (int)(r & 0x3FFFu), lo2 = (int)((r >> 14) & 0x3FFFu), na = (int)((r >> 28) & 3u), nb = (int)(r >> 30);
            int i[3], j[3];        // (at most three lookups from either set: all reads, then all atomics in flight)
#pragma unroll
            for (int y = 0; y < 3; ++y) {
                i[y] = y < nb ? (int)out_rows[lo2 + y] - i0 : -1;
                j[y] = y < na ? (int)in_rows[lo + y] : 0;
            }
            u32 old[3][3];
#pragma unroll
            for (int y = 0; y < 3; ++y)
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    old[y][x] = 0u;
                    if ((unsigned)i[y] < (unsigned)rows_here && x < na) {
                        const int sh = 8 * (i[y] & 3);
                        old[y][x] = atomicAdd(&pc_lds[(j[x] * ldT + i[y]) >> 2], 1u << sh) >> sh;
                    }
                }
#pragma unroll
            for (int y = 0; y < 3; ++y)
#pragma unroll
                for (int x = 0; x < 3; ++x) ovf |= (old[y][x] & 0xFFu) >= 254u;
        }
        pc_barrier();
        // ---- rows [i0, i0 + rows_here) of M.  A thread takes 4 rows x 8 columns: eight words of the transposed tile (four rows
        //      of one column each), turned in registers into four pairs of words of M.  Of a wave, 8 lanes lie along the
        //      columns and 8 along the rows: every lane has a bank of its own, and every row gets 64 contiguous bytes per store.
        {
            const int jl = lane & 7, il = lane >> 3;
            const int pj_n = colsP / 64, n_patches = pj_n * (rows_here / 32);
            for (int wq = wv; wq < n_patches; wq += NT / 64) {
                const int pj = wq % pj_n, pi = wq / pj_n;
                const int j8 = (pj * 8 + jl) * 8, i4 = (pi * 8 + il) * 4;
                u32 w[8];
#pragma unroll
                for (int x = 0; x < 8; ++x) w[x] = *reinterpret_cast<const u32*>(tile + (j8 + x) * ldT + i4);
#pragma unroll
                for (int x = 0; x < 8; ++x) ovf |= ((~w[x] - 0x01010101u) & w[x] & 0x80808080u) != 0u;   // a byte of 255: some byte of the complement is zero
                u32 o[4][2];
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const u32 t0 = __builtin_amdgcn_perm(w[4 * x + 1], w[4 * x], 0x05010400u), t1 = __builtin_amdgcn_perm(w[4 * x + 1], w[4 * x], 0x07030602u);
                    const u32 u0 = __builtin_amdgcn_perm(w[4 * x + 3], w[4 * x + 2], 0x05010400u), u1 = __builtin_amdgcn_perm(w[4 * x + 3], w[4 * x + 2], 0x07030602u);
                    o[0][x] = __builtin_amdgcn_perm(u0, t0, 0x05040100u);
                    o[1][x] = __builtin_amdgcn_perm(u0, t0, 0x07060302u);
                    o[2][x] = __builtin_amdgcn_perm(u1, t1, 0x05040100u);
                    o[3][x] = __builtin_amdgcn_perm(u1, t1, 0x07060302u);
                }
                uint8_t* dst = M + (size_t)(i0 + i4) * colsP + j8;
#pragma unroll
                for (int y = 0; y < 4; ++y) *reinterpret_cast<uint2*>(dst + (size_t)y * colsP) = make_uint2(o[y][0], o[y][1]);
            }
        }
        if (Mt) {  // the transpose is the tile as it lies: row j holds columns [i0, i0 + rows_here)
            const int gpr = rows_here / 16;
            for (int w = threadIdx.x; w < colsP * gpr; w += NT) {
                const int j = w / gpr, i16 = (w - j * gpr) * 16;
                const u32* src = reinterpret_cast<const u32*>(tile + j * ldT + i16);
                *reinterpret_cast<uint4*>(Mt + (size_t)j * rowsP + i0 + i16) = make_uint4(src[0], src[1], src[2], src[3]);
            }
        }
    }
    if (ovf) {   // this task goes to the sparse kernel
        a.task_path[t] = 0u;
        a.status[ST_PAIR_OVF] = 1u;
    }
}

// LDS of a launch: what the largest (task, field) needs for one tile of as many rows as NT threads take
static size_t pc_lds_need(int NT, int HBITS, int n_max, int max_rows, int max_tile_rows) {
    const int P = pad64(max_rows > 0 ? max_rows : 1);
    const int R = std::max(32, std::min({P, max_tile_rows, NT * 64 / P / 32 * 32}));
    return 6 * (size_t)n_max + std::max(pc_tile_bytes(R, P, 1 << HBITS), (size_t)n_max) + 64;   // (a mark per row to begin with)
}
static int pc_n_max(int max_tf) { return (max_tf + 7) / 8 * 8 + 8; }

// n_tasks tasks of a.order, of at most max_rows samples a set and max_tf lookups a (task, field) and set
template <int NT, int HBITS>
static void launch_pair_count_nt(hipStream_t st, PairCountArgs a, int n_tasks, int max_tf, int max_rows) {
    a.n_max = pc_n_max(max_tf);
    const size_t need = std::min<size_t>(pc_lds_need(NT, HBITS, a.n_max, max_rows, a.max_tile_rows), PAIR_LDS_BYTES);
    a.lds_bytes = (int)(need / 16 * 16);
    auto kern = pair_count_kernel<NT, HBITS>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, PAIR_LDS_BYTES);
    hipLaunchKernelGGL(kern, dim3(a.F, n_tasks, a.want_ss ? 2 : 1), dim3(NT), (size_t)a.lds_bytes, st, a);
}

// Uneven tasks in up to three launches, over the tasks that each can hold: a workgroup with nothing to do still costs its compute unit
// (or half of it) the latency of finding out, and a single task of more than 512 rows would send all that share its launch through sixteen
// waves and batches of 32 hot rows (its bags' numbers take ten of a lookup's 16 bits).  700 tasks of a median 32 rows x
// 40 fields: all but the small ones 904 us in one launch over all tasks, 421 + 210 so (421: the one or two of more than 512 rows, fewer
// workgroups than compute units).
void launch_pair_count(hipStream_t st, PairCountArgs a, const int32_t* order, const std::vector<int>& rows, int max_tf, int max_bag, int max_tile_rows) {
    if (rows.empty() || a.F <= 0) return;
    a.max_tile_rows = max_tile_rows > 0 ? (max_tile_rows + 31) / 32 * 32 : 1 << 20;
    a.small_n = PC_SMALL_N;
    const int n = (int)rows.size(), max_rows = rows.front(), min_rows = rows.back();
    auto above = [&](int size) {   // tasks of more rows
        return (int)(std::partition_point(rows.begin(), rows.end(), [&](int r) { return r > size; }) - rows.begin());
    };
    // Eight waves where a compute unit's LDS then holds two workgroups, whose phases hide each other's latency; else sixteen,
    // which take twice the rows a tile.
    auto launch = [&](int t0, int t1) {
        if (t0 >= t1) return;
        a.order = order + t0;
        const int most = rows[t0];
        // (as long a list as any, for its room for records, where that takes nothing else)
        const int tf = pc_lds_need(512, 6, pc_n_max(max_tf), most, a.max_tile_rows) <= PC_TWO_LDS ? max_tf : (int)std::min<int64_t>(max_tf, (int64_t)most * max_bag);
        if (most > 512) launch_pair_count_nt<1024, 5>(st, a, t1 - t0, tf, most);   // (a bag's number takes ten bits)
        else if (pc_lds_need(512, 6, pc_n_max(tf), most, a.max_tile_rows) <= PC_TWO_LDS) launch_pair_count_nt<512, 6>(st, a, t1 - t0, tf, most);
        else launch_pair_count_nt<1024, 6>(st, a, t1 - t0, tf, most);
    };
    a.order = order;
    if (max_rows <= PC_SMALL_ROWS && max_tf <= PC_SMALL_N) {   // every task is small
        a.cls = 0;
        launch_pair_count_nt<256, 6>(st, a, n, max_tf, max_rows);
    } else if (max_rows > 2 * PC_SMALL_ROWS && min_rows <= PC_SMALL_ROWS && (int64_t)n * a.F >= 32) {   // uneven: each workgroup of the first two checks its class
        const int large = above(512), mid = above(PC_SMALL_ROWS);
        a.cls = 1;
        a.order = order + mid;
        launch_pair_count_nt<256, 6>(st, a, n - mid, std::min<int>(max_tf, PC_SMALL_N), PC_SMALL_ROWS);
        a.cls = 2;
        // (tasks of few rows but long bags may have (task, field)s that are not small)
        const int end = above(std::min<int>(PC_SMALL_ROWS, PC_SMALL_N / std::max(max_bag, 1)));
        launch(large, end);
        a.cls = 0;
        launch(0, large);
    } else {
        const int large = (int64_t)n * a.F >= 32 ? above(512) : 0;
        a.cls = 0;
        launch(0, large);
        launch(large, n);
    }
}

// ------------------------------------------------------------------------------------------------
// the hop: Y = Y_in + c * M * Z on MFMA 32x32x16 (bf16 operands, fp32 accumulation)
//
// Z is staged 64 rows at a time: split into its three bf16 pieces and stored contraction-contiguous per column, so that
// a B fragment is one 16-byte LDS read.  M is read straight from memory: within a 64-wide chunk the lane half h contracts
// columns [32h, 32h+32) of the chunk (the contraction index may be enumerated in any order as long as A and B agree),
// which makes a lane's share of a strip 32 contiguous bytes of one row of M.
//
// Bound: HBM (M, Z, Y read, Y written) for tasks of 256 rows; with uneven or small tasks it was workgroups that had
// nothing to do, waves that multiplied rows of no one and one XCD with the large tasks.  So the work is a list made from the
// task sizes (hop_plan):
//   tasks of at most 64 rows in both sets   one workgroup per (task, field, DS columns) takes both outputs from one staged Z
//   the others                              tiles of 256 out-rows; a last tile of at most 128 (64) rows gives every wave one
//                                           strip of 32 rows (and half the columns).  The tasks are dealt to the XCDs by
//                                           size, largest first, a task's tiles to one XCD (all of a field's read the same Z);
//                                           a few tasks are dealt in runs of fields.
// Measured: the four hops of a step of 700 tasks of log-normal size (median 32 + 32 rows) x 40 fields of 64 columns
// 11.6 -> 1.95 ms, the three of 201 tasks of 75..225 + 122..365 rows x 26 fields 2.34 -> 1.43 ms; the six of 512 tasks x
// (256 + 256) rows x 26 fields 6.7 -> 6.5 ms (before: a grid of (task, output, 256 rows) in task order, 64 rows a wave).
// Inside a run of fields the tiles come first, field by field, where an output has several of equal height: they find the field's Z
// in L2 (two hops of 256 tasks x (512 + 512) rows x 64 fields, two tiles each, fetch 15.4 GB instead of 19.6; eleven runs of a side
// 4.86..5.12 against 5.05..5.35 ms).  Otherwise the fields come first.  With one tile per output a tile's pieces of the same rows follow
// each other (six hops of 512 tasks x (256 + 256) rows x 26 fields 6.35..6.57 ms; tiles first they fetch 19.0 GB instead of 20.1 and
// take 1-2 % longer).  With a short last tile, high and low ones in turn would fall on the same compute units again and again: the
// hops of 100 tasks x (300 + 300) rows x 26 fields 1.24 ms, tiles first 1.58 ms, of 100 x (400 + 400) rows 1.86 against 1.82..1.92 ms.
// ------------------------------------------------------------------------------------------------
#define PH_KC 64

__device__ __forceinline__ u32 ph_pack_hi(u32 e0, u32 e1) {  // {e1[31:16], e0[31:16]}
    return __builtin_amdgcn_perm(e1, e0, 0x07060302u);
}

// four counts (bytes of x) -> four bf16 (exact for 0..255)
__device__ __forceinline__ void ph_cvt4(u32 x, u32& lo, u32& hi) {
    const float f0 = (float)(x & 0xFFu), f1 = (float)((x >> 8) & 0xFFu), f2 = (float)((x >> 16) & 0xFFu), f3 = (float)(x >> 24);
    lo = ph_pack_hi(__builtin_bit_cast(u32, f0), __builtin_bit_cast(u32, f1));
    hi = ph_pack_hi(__builtin_bit_cast(u32, f2), __builtin_bit_cast(u32, f3));
}

// LDS layout of the staged chunk: per (piece, column) 64 contraction values = eight 16-byte groups; group g of
// column c sits at position g ^ key(c).  With this key both the 16-byte fragment reads (32 consecutive columns,
// one group) and the staging writes (every fourth column, one group) spread over all banks.
__device__ __forceinline__ int ph_key(int col) { return ((col >> 1) + (col >> 4)) & 7; }

// One workgroup's share of a 64-row chunk of Z, the sum of NZ arrays: DS/16 rows of four columns per thread.
template <int DS, int NZ>
struct HopStage {
    static constexpr int CG = DS / 4;        // float4 column groups of a row of Z
    static constexpr int RPT = CG / 4;       // rows of the 64-row chunk staged per thread (256 threads)
    static constexpr int WORDS = 3 * DS * PH_KC;   // bf16 values of a staged chunk
    int rg, wr_off[4];   // element offsets of this thread's staging writes, per column of its float4
    const float* Zt[NZ];
    int64_t ldz;
    int n_in;
    float4 z[NZ][RPT];
    __device__ __forceinline__ HopStage(const PairHopArgs& a, int64_t off, int n_in_) : ldz(a.ldz), n_in(n_in_) {   // off: of the first row's first column
        const int cg = threadIdx.x % CG;
        rg = threadIdx.x / CG;
#pragma unroll
        for (int j = 0; j < NZ; ++j) Zt[j] = a.Z[j] + off + cg * 4;
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
            const int col = cg * 4 + cc, k0 = rg * RPT;
            wr_off[cc] = col * PH_KC + (((k0 >> 3) ^ ph_key(col)) << 3) + (k0 & 7);
        }
    }
    __device__ __forceinline__ void load(int kc) {
#pragma unroll
        for (int r = 0; r < RPT; ++r) {   // branch-free: a row beyond the task reads the task's last row and is zeroed
            const int64_t at = (int64_t)min(kc + rg * RPT + r, n_in - 1) * ldz;
#pragma unroll
            for (int j = 0; j < NZ; ++j) z[j][r] = *reinterpret_cast<const float4*>(Zt[j] + at);
        }
    }
    // splits the loaded rows into their three bf16 pieces and writes them into an LDS buffer
    __device__ __forceinline__ void store(bf16_t* buf, int kc) const {
        u32 p0[4][RPT], p1[4][RPT], p2[4][RPT];  // [column][row]: the three pieces as fp32 bit patterns
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const float keep = kc + rg * RPT + r < n_in ? 1.f : 0.f;
            float4 x = z[0][r];
#pragma unroll
            for (int j = 1; j < NZ; ++j) x = make_float4(x.x + z[j][r].x, x.y + z[j][r].y, x.z + z[j][r].z, x.w + z[j][r].w);
            const float zz[4] = {x.x * keep, x.y * keep, x.z * keep, x.w * keep};
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                const u32 u0 = __builtin_bit_cast(u32, zz[cc]);
                const float r1 = zz[cc] - __builtin_bit_cast(float, u0 & 0xFFFF0000u);
                const u32 u1 = __builtin_bit_cast(u32, r1);
                const float r2 = r1 - __builtin_bit_cast(float, u1 & 0xFFFF0000u);
                p0[cc][r] = u0; p1[cc][r] = u1; p2[cc][r] = __builtin_bit_cast(u32, r2);
            }
        }
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
            bf16_t* d0 = buf + wr_off[cc];
            bf16_t* d1 = d0 + DS * PH_KC;
            bf16_t* d2 = d1 + DS * PH_KC;
            if constexpr (RPT == 4) {
                *reinterpret_cast<uint2*>(d0) = make_uint2(ph_pack_hi(p0[cc][0], p0[cc][1]), ph_pack_hi(p0[cc][2], p0[cc][3]));
                *reinterpret_cast<uint2*>(d1) = make_uint2(ph_pack_hi(p1[cc][0], p1[cc][1]), ph_pack_hi(p1[cc][2], p1[cc][3]));
                *reinterpret_cast<uint2*>(d2) = make_uint2(ph_pack_hi(p2[cc][0], p2[cc][1]), ph_pack_hi(p2[cc][2], p2[cc][3]));
            } else {
                *reinterpret_cast<u32*>(d0) = ph_pack_hi(p0[cc][0], p0[cc][1]);
                *reinterpret_cast<u32*>(d1) = ph_pack_hi(p1[cc][0], p1[cc][1]);
                *reinterpret_cast<u32*>(d2) = ph_pack_hi(p2[cc][0], p2[cc][1]);
            }
        }
    }
};

// one staged chunk times NS strips of counts, for NC column tiles from column tile ct0 on
template <int DS, int NS, int NC>
__device__ __forceinline__ void hop_multiply(const bf16_t* zb, const uint4 (&araw)[NS][2], int ct0, ph_float16 (&acc)[NS][NC]) {
    const int lane = threadIdx.x & 63, ln = lane & 31, h = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        ph_short8 af[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint4 q = araw[s][ks >> 1];
            const u32 b0 = (ks & 1) ? q.z : q.x, b1 = (ks & 1) ? q.w : q.y;
            u32 w0, w1, w2, w3;
            ph_cvt4(b0, w0, w1);
            ph_cvt4(b1, w2, w3);
            const uint4 packed = make_uint4(w0, w1, w2, w3);
            af[s] = __builtin_bit_cast(ph_short8, packed);
        }
        ph_short8 bfrag[NC][3];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int col = (ct0 + c) * 32 + ln;
            const bf16_t* src = zb + col * PH_KC + (((h * 4 + ks) ^ ph_key(col)) << 3);
#pragma unroll
            for (int sp = 0; sp < 3; ++sp) bfrag[c][sp] = *reinterpret_cast<const ph_short8*>(src + sp * DS * PH_KC);
        }
#pragma unroll
        for (int sp = 2; sp >= 0; --sp)  // smallest pieces first
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    acc[s][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfrag[c][sp], af[s], acc[s][c], 0, 0, 0);
    }
}

// A wave's 32 x (NC * 32) strips of the output.  The first operand of the MFMAs is the Z fragment, so a lane holds row ln of each
// 32 x 32 block and four consecutive columns per group of four registers; stored from there, or with the operands the other way
// round (one row's 32 columns, four bytes a lane), a strip of 64 columns takes 32 reads, 32 stores of fp32 and 32 of two bytes a lane,
// and the memory pipeline is busy with instructions.  Through LDS, 16 bytes a lane, whole row segments: eight of each.
// (y_in may be y_out: a strip's reads are asked for together, ahead of its stores.)
// Y streams past once, read or written: with the non-temporal hint it leaves the caches to the counts, of which a chunk takes half a
// line at a time, and to Z, which an output's other tiles read again.  The six hops of 512 tasks x (256 + 256) rows x 26 fields
// 5.25 -> 4.61 ms (hint on the reads and fp32 stores only 4.72; on the counts too 6.1).
template <int NC>
struct HopStrip {
    static constexpr int SW = NC * 32, ELD = SW + 4, LPR = SW / 4, RPI = 64 / LPR, IT = 32 / RPI;   // width, LDS row stride, lanes a row, rows a pass
    static constexpr int FLOATS = 32 * ELD;   // of LDS, per wave
    RowBuffer yi, yo, yb;
    int er, ec;
    float c;
    // rows [0, rows) from row `row` on, columns [col, col + SW)
    __device__ __forceinline__ HopStrip(const PairHopOut& out, int64_t row, int rows, int64_t col)
        : yi(out.y_in ? out.y_in + col : nullptr, out.y_in ? row : 0, out.ld, 4, out.y_in ? rows : 0, (int)(threadIdx.x & 63) / LPR, (int)(threadIdx.x & 63) % LPR * 4, true),
          yo(out.y_out ? out.y_out + col : nullptr, out.y_out ? row : 0, out.ld, 4, out.y_out ? rows : 0, (int)(threadIdx.x & 63) / LPR, (int)(threadIdx.x & 63) % LPR * 4, true),
          yb(out.y_bf ? out.y_bf + col : nullptr, out.y_bf ? row : 0, out.ld, 2, out.y_bf ? rows : 0, (int)(threadIdx.x & 63) / LPR, (int)(threadIdx.x & 63) % LPR * 4, true),
          er((int)(threadIdx.x & 63) / LPR), ec((int)(threadIdx.x & 63) % LPR * 4), c(out.c) {}
    __device__ __forceinline__ void request(int r0, float4 (&y)[IT]) const {   // (no input: zeros)
#pragma unroll
        for (int it = 0; it < IT; ++it) y[it] = yi.load4<STREAM>(r0 + it * RPI);
    }
    __device__ __forceinline__ void park(float* E, const ph_float16 (&acc)[NC]) const {
        const int ln = threadIdx.x & 31, h = (threadIdx.x & 63) >> 5;
#pragma unroll
        for (int j = 0; j < NC; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4*>(E + ln * ELD + j * 32 + 8 * q + 4 * h) = make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
    }
    __device__ __forceinline__ void finish(const float* E, int r0, const float4 (&y)[IT]) const {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the strip is this wave's own: LDS order within the wave suffices
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const float4 x = *reinterpret_cast<const float4*>(E + (it * RPI + er) * ELD + ec);
            const float4 r = make_float4(fmaf(c, x.x, y[it].x), fmaf(c, x.y, y[it].y), fmaf(c, x.z, y[it].z), fmaf(c, x.w, y[it].w));
            yo.store<STREAM>(r0 + it * RPI, r);
            yb.store<STREAM>(r0 + it * RPI, make_uint2(f2bf2(r.x, r.y), f2bf2(r.z, r.w)));
        }
        asm volatile("" ::: "memory");
    }
};

// A tile of up to 64 * NS * 2 out-rows from row0 on.  NS strips per wave, NC column tiles per wave: with fewer than all of
// them the waves lie side by side along the columns.
template <int DS, int NZ, int NS, int NC>
__device__ __forceinline__ void hop_tile(const PairHopArgs& a, const PairHopOut& out, const uint8_t* M, int64_t z_off, int n_in, int n_out, int row0,
                                         int64_t row_base, int64_t colz, bf16_t* zs) {
    constexpr int WC = DS / 32 / NC;   // waves along the columns
    const int colsP = pad64(n_in);
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, ln = lane & 31, h = lane >> 5;
    const int ct0 = (wv % WC) * NC, row_w = __builtin_amdgcn_readfirstlane(row0 + (wv / WC) * 32 * NS);   // first out-row of this wave
    const bool wave_on = row_w < n_out;               // its strips then lie inside the padded matrix
    const uint8_t* Mw = M + (size_t)(row_w + ln) * colsP + h * 32;
    typedef HopStage<DS, NZ> Stage;
    Stage st(a, z_off, n_in);
    ph_float16 acc[NS][NC];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[s][c][v] = 0.f;
    uint4 araw[NS][2], anext[NS][2];
    auto load_a = [&](int kc, uint4 (&dst)[NS][2]) {
        if (!wave_on) return;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint4* src = reinterpret_cast<const uint4*>(Mw + (size_t)(s * 32) * colsP + kc);
            dst[s][0] = src[0];
            dst[s][1] = src[1];
        }
    };
    const HopStrip<NC> strip(out, row_base + row_w, __builtin_amdgcn_readfirstlane(max(min(n_out - row_w, 32 * NS), 0)), colz + __builtin_amdgcn_readfirstlane(ct0 * 32));
    float4 y[2][HopStrip<NC>::IT];
    // Two LDS buffers: while chunk c is multiplied out of one, chunk c+1 (loaded during the multiplication) is
    // split into the other; one barrier per chunk.
    if (colsP > 0) {
        st.load(0);
        load_a(0, araw);
        st.store(zs, 0);
    }
    __syncthreads();
    int cur = 0;
    for (int kn = PH_KC; kn < colsP; kn += PH_KC) {
        st.load(kn);
        load_a(kn, anext);
        __builtin_amdgcn_sched_barrier(0);   // the loads above are consumed only after the multiplication below
        if (wave_on) hop_multiply<DS, NS, NC>(zs + cur * Stage::WORDS, araw, ct0, acc);
        __builtin_amdgcn_sched_barrier(0);
        cur ^= 1;
        st.store(zs + cur * Stage::WORDS, kn);
#pragma unroll
        for (int s = 0; s < NS; ++s) { araw[s][0] = anext[s][0]; araw[s][1] = anext[s][1]; }
        __syncthreads();
    }
    strip.request(0, y[0]);
    __builtin_amdgcn_sched_barrier(0);
    if (wave_on && colsP > 0) hop_multiply<DS, NS, NC>(zs + cur * Stage::WORDS, araw, ct0, acc);
    __syncthreads();   // every wave is done with the staged chunks
    if (!wave_on) return;
    float* E = reinterpret_cast<float*>(zs) + wv * HopStrip<NC>::FLOATS;
    static_assert(4 * HopStrip<NC>::FLOATS * 4 <= 2 * Stage::WORDS * 2, "the waves' strips fit the staged chunks' LDS");
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        strip.park(E, acc[s]);
        if (s + 1 < NS) strip.request((s + 1) * 32, y[(s + 1) & 1]);
        strip.finish(E, s * 32, y[s & 1]);
    }
}

// (a sum of several arrays: a chunk's rows of all of them are on their way together, in registers)
template <int DS, int NZ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void pair_hop_kernel(PairHopArgs a) {
    constexpr int NCT = DS / 32;      // 32-column tiles
    __shared__ __attribute__((aligned(16))) bf16_t zs[2 * HopStage<DS, NZ>::WORDS];
    // workgroups are dealt round-robin to the 8 XCDs; every XCD walks its own list, all (tile, field)s of one task's run in a row
    const int nsl = a.D / DS, fx = a.F * nsl;
    const int xcd = blockIdx.x & 7, k = (int)(blockIdx.x >> 3), e = a.tiles[xcd] + k / a.run;
    if (e >= a.tiles[xcd + 1]) return;
    const u32 entry = (u32)a.tiles[9 + e];
    const int t = (int)(entry & 0xFFFFu);
    // (both outputs' values are asked for at once: which of them is meant follows from their sizes)
    const u32 on = a.task_path[t];
    const int n_in = a.in_real_off[t + 1] - a.in_real_off[t], in_row = a.in_row_off[t];
    int n[2], row_off[2];
    u32 mat_off[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        n[o] = a.out[o].real_off[t + 1] - a.out[o].real_off[t];
        row_off[o] = a.out[o].row_off[t];
        mat_off[o] = a.out[o].mat_off[t];
    }
    if (!on) return;
    const int nt0 = (n[0] + 255) >> 8, nt1 = a.out[1].enabled ? (n[1] + 255) >> 8 : 0, nt = nt0 + nt1;
    int tile = (int)((entry >> 16) & 7u), i = k % a.run;   // (tile, field) in the run, fields first
    auto even = [](int rows) { const int last = rows & 255; return last == 0 || last > 192; };   // every wave of every tile has rows
    if ((nt0 > 1 || nt1 > 1) && even(n[0]) && (nt1 == 0 || even(n[1]))) {   // tiles first
        const int u = tile * a.run + i;
        i = u / nt;
        tile = u - i * nt;
    }
    const int o = tile >= nt0, row0 = (o ? tile - nt0 : tile) * 256;
    const int fs = (int)(entry >> 19) * a.run + i, f = fs / nsl, sl = fs - f * nsl;
    if (fs >= fx) return;
    const PairHopOut& out = a.out[o];
    const int n_out = o ? n[1] : n[0];
    const uint8_t* M = a.mat + (size_t)(o ? mat_off[1] : mat_off[0]) * PAIR_BLOCK + (size_t)f * pad64(n_out) * pad64(n_in);
    const int64_t colz = (int64_t)f * a.D + (int64_t)sl * DS;
    const int64_t z_off = (int64_t)in_row * a.ldz + colz;
    const int64_t row_base = o ? row_off[1] : row_off[0];
    if (n_out - row0 > 128) hop_tile<DS, NZ, 2, NCT>(a, out, M, z_off, n_in, n_out, row0, row_base, colz, zs);
    else if (n_out - row0 > 64) hop_tile<DS, NZ, 1, NCT>(a, out, M, z_off, n_in, n_out, row0, row_base, colz, zs);
    else hop_tile<DS, NZ, 1, 1>(a, out, M, z_off, n_in, n_out, row0, row_base, colz, zs);
}

// Tasks of at most 64 rows in both sets: one chunk of Z, at most two strips per output.  What is bound here is the chain of
// dependent reads (task -> offsets -> M, Z and Y -> LDS), so everything is requested at once and half the LDS and registers
// of the large tiles let twice as many workgroups run side by side.
template <int DS, int NZ>
__global__ __launch_bounds__(256, 4) void pair_hop_small_kernel(PairHopArgs a) {
    constexpr int NCT = DS / 32;
    __shared__ __attribute__((aligned(16))) bf16_t zs[HopStage<DS, NZ>::WORDS];
    const int nsl = a.D / DS, fx = a.F * nsl;
    const int per_xcd = gridDim.x >> 3, wid = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);   // neighbouring fields on one XCD
    if (wid >= a.n_small * fx) return;
    const int t = a.small[wid / fx], fs = wid % fx, f = fs / nsl, sl = fs - f * nsl;
    if (!a.task_path[t]) return;
    const int n_in = a.in_real_off[t + 1] - a.in_real_off[t];
    const int64_t colz = (int64_t)f * a.D + (int64_t)sl * DS;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, ln = lane & 31, h = lane >> 5;
    const int row_w = (wv >> 1) * 32, ct = wv & 1;
    uint4 araw[2][1][2];
    float4 y[2][HopStrip<1>::IT];
    bool on[2];
    auto strip = [&](int o) {
        const int rows = on[o] ? a.out[o].real_off[t + 1] - a.out[o].real_off[t] - row_w : 0;
        return HopStrip<1>(a.out[o], (int64_t)a.out[o].row_off[t] + __builtin_amdgcn_readfirstlane(row_w), __builtin_amdgcn_readfirstlane(min(rows, 32)), colz + __builtin_amdgcn_readfirstlane(ct * 32));
    };
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        on[o] = false;
        if (!a.out[o].enabled) continue;
        on[o] = row_w < a.out[o].real_off[t + 1] - a.out[o].real_off[t] && ct < NCT;
        if (on[o] && n_in > 0) {
            const uint4* src = reinterpret_cast<const uint4*>(a.mat + (size_t)a.out[o].mat_off[t] * PAIR_BLOCK + ((size_t)f * 64 + row_w + ln) * 64 + h * 32);
            araw[o][0][0] = src[0];
            araw[o][0][1] = src[1];
        }
    }
    if (n_in > 0) {
        HopStage<DS, NZ> st(a, (int64_t)a.in_row_off[t] * a.ldz + colz, n_in);
        st.load(0);
        st.store(zs, 0);
    }
#pragma unroll
    for (int o = 0; o < 2; ++o)
        if (on[o]) strip(o).request(0, y[o]);
    __syncthreads();
    ph_float16 acc[2][1][1];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[o][0][0][v] = 0.f;
        if (on[o] && n_in > 0) hop_multiply<DS, 1, 1>(zs, araw[o], ct, acc[o]);
    }
    __syncthreads();   // every wave is done with the staged chunk
    float* E = reinterpret_cast<float*>(zs) + (NCT == 1 ? wv >> 1 : wv) * HopStrip<1>::FLOATS;
    static_assert(2 * NCT * HopStrip<1>::FLOATS * 4 <= HopStage<DS, NZ>::WORDS * 2, "the strips fit the staged chunk's LDS");
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        if (!on[o]) continue;
        const HopStrip<1> sp = strip(o);
        sp.park(E, acc[o][0]);
        sp.finish(E, 0, y[o]);
    }
}

int hop_slices(int F, int D) { return F * (D / (D % 64 == 0 ? 64 : 32)); }
// With fewer than eight large tasks for every XCD the XCDs take runs of HOP_RUN (field, slice)s of a task instead of whole
// tasks (3 tasks x (512 + 512) rows x 64 fields, two hops: 180 -> 93 us).
enum { HOP_RUN = 8, HOP_WHOLE_TASKS = 64 };
int64_t hop_entries(int64_t tiles, int fx) { return std::max(tiles, std::min<int64_t>(tiles, (HOP_WHOLE_TASKS - 1) * 4) * ((fx + HOP_RUN - 1) / HOP_RUN)); }

HopPlan hop_plan(const std::vector<HopTask>& tasks, int fx) {
    HopPlan p;
    std::vector<HopTask> large;
    for (const HopTask& t : tasks) {
        if (std::max(t.ns, t.nq) <= HOP_SMALL) p.small.push_back(t.t);
        else large.push_back(t);
    }
    const bool whole = large.size() >= HOP_WHOLE_TASKS || fx > HOP_RUN << 13;   // (13 bits hold a run's number)
    p.run = whole ? fx : (int)HOP_RUN;
    const int runs = (fx + p.run - 1) / p.run;
    // largest first, there and back over the XCDs: equal numbers of tasks and nearly equal work on each
    std::stable_sort(large.begin(), large.end(), [](const HopTask& a, const HopTask& b) { return (int64_t)(a.ns + a.nq) > (int64_t)(b.ns + b.nq); });
    for (int kind = 0; kind < 3; ++kind) {
        std::vector<int32_t> of[8];
        size_t unit = 0;
        for (const HopTask& t : large)
            for (int r = 0; r < runs; ++r, ++unit) {
                const int x = (int)(unit & 8 ? 7 - (unit & 7) : unit & 7);
                u32 nt = 0;   // the task's tiles: as many entries, which share its (tile, field)s
                if (kind != HOP_QUERY) nt += (u32)(t.ns + 255) / 256;
                if (kind != HOP_SUPPORT) nt += (u32)(t.nq + 255) / 256;
                for (u32 j = 0; j < nt; ++j) of[x].push_back((int32_t)((u32)t.t | (j << 16) | ((u32)r << 19)));
            }
        std::vector<int32_t>& l = p.tiles[kind];
        l.assign(9, 0);
        for (int x = 0; x < 8; ++x) {
            l[x + 1] = l[x] + (int32_t)of[x].size();
            p.longest[kind] = std::max(p.longest[kind], (int)of[x].size());
        }
        for (int x = 0; x < 8; ++x) l.insert(l.end(), of[x].begin(), of[x].end());
    }
    return p;
}

void launch_pair_hop(hipStream_t st, PairHopArgs a, const int32_t* const tiles[3], const int longest[3]) {
    const int kind = a.out[0].enabled ? (a.out[1].enabled ? HOP_BOTH : HOP_SUPPORT) : HOP_QUERY;
    if (a.F <= 0 || !(a.out[0].enabled || a.out[1].enabled)) return;
    if (kind == HOP_QUERY) a.out[0] = a.out[1];
    if (kind != HOP_BOTH) {   // (its arrays are read all the same)
        a.out[1] = a.out[0];
        a.out[1].enabled = 0;
    }
    a.tiles = tiles[kind];
    const int ds = a.D % 64 == 0 ? 64 : 32;
    const int64_t fx = (int64_t)a.F * (a.D / ds), n_large = 8 * (int64_t)a.run * longest[kind], n_small = (fx * a.n_small + 7) / 8 * 8;
    if (n_large >= ((int64_t)1 << 31) || n_small >= ((int64_t)1 << 31)) return;   // cannot happen within the library's own limits on a call
#define HOP_LAUNCH(DS_, NZ_)                                                                                                             \
    do {                                                                                                                                 \
        if (n_large > 0) hipLaunchKernelGGL((pair_hop_kernel<DS_, NZ_>), dim3((unsigned)n_large), dim3(256), 0, st, a);                  \
        if (n_small > 0) hipLaunchKernelGGL((pair_hop_small_kernel<DS_, NZ_>), dim3((unsigned)n_small), dim3(256), 0, st, a);            \
    } while (0)
#define HOP_WIDTH(NZ_)                                  \
    do {                                                \
        if (ds == 64) HOP_LAUNCH(64, NZ_);              \
        else HOP_LAUNCH(32, NZ_);                       \
    } while (0)
    switch (a.n_z) {
        case 1: HOP_WIDTH(1); break;
        case 2: HOP_WIDTH(2); break;
        default: HOP_WIDTH(3); break;
    }
#undef HOP_WIDTH
#undef HOP_LAUNCH
}
