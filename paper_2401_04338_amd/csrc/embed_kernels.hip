// Embedding side of the MAML step (G-Meta Alg. 1): the one-pass prefetch of support and query rows
// with sum pooling (prefetch step, Sec. 2.1.1), the task-local row updates and the overlap update
// (their dense and pad columns; the row arithmetic itself is in twohop_kernels.hip), and the segment reduction that coalesces the sparse
// meta-gradient (global back-propagation on xi).  All HBM-bound: rows are read as float4 by groups of
// D/4 lanes so that one wavefront keeps several independent row reads in flight.
#include "gm_internal.h"

__device__ __forceinline__ void store_bf4(bf16_t* dst, float4 v) {
    uint2 o;
    o.x = f2bf2(v.x, v.y);
    o.y = f2bf2(v.z, v.w);
    *reinterpret_cast<uint2*>(dst) = o;
}

__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }
__device__ __forceinline__ float4 fma4(float s, float4 a, float4 b) { return make_float4(fmaf(s, a.x, b.x), fmaf(s, a.y, b.y), fmaf(s, a.z, b.z), fmaf(s, a.w, b.w)); }

// ------------------------------------------------------------------------------------------------
// prefetch + sum pooling: x[s, f*D:(f+1)*D] = sum over bag(s,f) of emb[field_base[f] + index]
// ------------------------------------------------------------------------------------------------
// One launch takes both sets: sample u of the launch is sample u of the first set or u - n0 of the second, and the last
// blocks write the dense features and the zero padding behind the pooled fields.
struct PoolArgs {
    int F, D, LG, n_dense, ldx;
    unsigned pool_blocks;
    const int64_t* field_base;
    const float4* emb;
    PoolSet set[2];
};

__device__ __forceinline__ void pool_tail(const PoolArgs& a) {
    const int FD = a.F * a.D, tail = a.ldx - FD;
    const int64_t i = (int64_t)(blockIdx.x - a.pool_blocks) * blockDim.x + threadIdx.x, n0 = a.set[0].n_samples;
    if (i >= (n0 + a.set[1].n_samples) * tail) return;
    int64_t s = i / tail;
    const int c = (int)(i - s * tail);
    const PoolSet& S = a.set[s >= n0];
    if (s >= n0) s -= n0;
    const float v = (S.dense && c < a.n_dense) ? S.dense[(S.sample0 + s) * a.n_dense + c] : 0.f;
    const int64_t o = (int64_t)(S.row_map[s] - S.row_base) * a.ldx + FD + c;
    if (S.x) S.x[o] = v;
    if (S.x_bf) S.x_bf[o] = f2bf(v);
    if (S.zero) S.zero[o] = 0.f;
    if (S.zero_bf) S.zero_bf[o] = 0;
}

__global__ __launch_bounds__(256) void gather_pool_kernel(PoolArgs a) {
    if (blockIdx.x >= a.pool_blocks) { pool_tail(a); return; }
    const int LG = a.LG, F = a.F;
    const int groups_per_block = blockDim.x / LG;
    const int g_in_block = threadIdx.x / LG, l = threadIdx.x % LG;
    const int64_t n_groups = (int64_t)a.pool_blocks * groups_per_block, n0 = a.set[0].n_samples, n_bags = (n0 + a.set[1].n_samples) * F;
    for (int64_t bag = (int64_t)blockIdx.x * groups_per_block + g_in_block; bag < n_bags; bag += n_groups) {
        int64_t s = bag / F;
        const int f = (int)(bag - s * F);
        const PoolSet& S = a.set[s >= n0];
        if (s >= n0) s -= n0;
        const int64_t gb = (S.sample0 + s) * F + f;
        const int64_t p0 = S.bag_offsets[gb], p1 = S.bag_offsets[gb + 1];
        const int64_t fb = a.field_base[f];
        // the order of the sums is gather_pool_xcd_kernel's, bit for bit: eight lookups at a time, the first four into
        // one chain and the next four into the other (one chain when a lane group is narrower than eight lanes)
        float4 acc0 = make_float4(0.f, 0.f, 0.f, 0.f), acc1 = acc0;
        const float4 zero = acc0;
        for (int64_t p = p0; p < p1; p += 8) {
            float4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = p + j < p1 ? a.emb[(fb + S.indices[p + j]) * LG + l] : zero;
            acc0 = add4(add4(add4(add4(acc0, v[0]), v[1]), v[2]), v[3]);
            if (LG >= 8) acc1 = add4(add4(add4(add4(acc1, v[4]), v[5]), v[6]), v[7]);
            else acc0 = add4(add4(add4(add4(acc0, v[4]), v[5]), v[6]), v[7]);
        }
        const float4 acc = add4(acc0, acc1);
        const int64_t o = (int64_t)(S.row_map[s] - S.row_base) * a.ldx + (int64_t)f * a.D + l * 4;
        if (S.x) *reinterpret_cast<float4*>(S.x + o) = acc;
        if (S.x_bf) store_bf4(S.x_bf + o, acc);
    }
}

// The same pooling with the fields dealt to the 8 XCDs: workgroup b runs on XCD b % 8 and pools one eighth of the
// (field, sample) pairs in field-major order, i.e. about F / 8 consecutive fields (a field may be shared by two
// neighbours, so that the shares are equal whatever F is).  Under Zipf skew most lookups of a field hit a few thousand
// hot rows; with an eighth of the fields per XCD the hot rows of "its" fields fit that XCD's L2 (8 fields x 1000 rows
// x 256 B = 2 MB of 4 MB), so they stop travelling over the fabric for every lookup -- the fabric, not HBM, is what
// this kernel is bound by.  (The lookups of a bag are summed in two interleaved chains of four, a fixed order.)  Indices
// and the fp32 outputs stream past once: they are read and written with the non-temporal hint, which leaves L2 to the
// rows (measured: 2-3 %; whether all XCDs sweep one field range together or each its own eighth makes no difference).
// A field's support and query samples follow each other, so that its rows are fetched for both sets at once.
// Measured: 201 tasks of about (150 + 243) samples x 26 fields, bags of 1..20, 0.67 ms in two launches -> 0.63 ms; 128 tasks x (512 + 512)
// samples x 64 fields, bags of 1..32, 3.63 -> 3.62 ms, 9.8 TB/s of rows.
// Where the rows are in L2 the instructions around a read are the bound: the width is a constant of the kernel, the indices of
// eight reads are handed round together, offsets count from the set's first bag in 32 bits, and what does not depend on the rows
// (the table's base, the output row) is read a bag ahead of them: 18 million lookups of 64 columns 475 -> 448 us, 72 million 2.10 -> 2.01 ms.
template <int LG>
__global__ __launch_bounds__(256) void gather_pool_xcd_kernel(PoolArgs a) {
    if (blockIdx.x >= a.pool_blocks) { pool_tail(a); return; }
    constexpr int GPB = 256 / LG;
    const int F = a.F;
    const int g_in_block = threadIdx.x / LG, l = threadIdx.x % LG;
    const int xcd = blockIdx.x & 7, bi = blockIdx.x >> 3, nbx = a.pool_blocks >> 3;
    // work items of this XCD: pairs [lo, hi) of the field-major list (pair = field * samples + sample; fewer than 2^32)
    const u32 n0 = (u32)a.set[0].n_samples, n = n0 + (u32)a.set[1].n_samples;
    const int64_t n_pairs = (int64_t)n * F;
    const int64_t hi = n_pairs * (xcd + 1) / 8, stride = (int64_t)nbx * GPB;
    int64_t it = n_pairs * xcd / 8 + (int64_t)bi * GPB + g_in_block;
    if (it >= hi) return;
    int f = (int)(it / n);
    u32 u = (u32)(it - (int64_t)f * n);
    const int64_t* const bags[2] = {a.set[0].bag_offsets + a.set[0].sample0 * F, a.set[1].bag_offsets + a.set[1].sample0 * F};
    // A bag is a chain of dependent reads (offsets -> indices -> rows).  The chain of the NEXT bag is started before
    // the rows of this one are summed: its offsets and its first LG indices (one per lane of the group, handed round
    // by lane shuffles) are in registers when its turn comes, and up to 8 row reads are in flight per lane.
    int64_t p0, p1, base_row;
    int32_t idx_l, row;
    auto open_bag = [&](int bf, u32 bu) {
        const bool second = bu >= n0;
        const u32 s = second ? bu - n0 : bu;
        const int32_t* ix = second ? a.set[1].indices : a.set[0].indices;
        const int64_t* bo = (second ? bags[1] : bags[0]) + (u32)(s * (u32)F + (u32)bf);
        p0 = bo[0]; p1 = bo[1];
        base_row = a.field_base[bf];
        row = (second ? a.set[1].row_map : a.set[0].row_map)[s];
        idx_l = (p0 + l < p1) ? __builtin_nontemporal_load(ix + p0 + l) : 0;
    };
    open_bag(f, u);
    while (true) {
        const bool second = u >= n0;
        const int32_t* indices = second ? a.set[1].indices : a.set[0].indices;
        const float4* const rows = a.emb + base_row * LG + l;
        const int64_t o = (int64_t)(row - (second ? a.set[1].row_base : a.set[0].row_base)) * a.ldx + (f * (4 * LG) + l * 4);
        const int64_t c0 = p0, c1 = p1;
        int32_t cur_idx = idx_l;
        // the next bag
        it += stride;
        int fn = f;
        int64_t un = (int64_t)u + stride;
        while (un >= (int64_t)n) { un -= n; ++fn; }
        if (it < hi) open_bag(fn, (u32)un);
        float4 acc0 = make_float4(0.f, 0.f, 0.f, 0.f), acc1 = acc0;
        for (int64_t base = c0; base < c1; base += LG) {
            if (base > c0) cur_idx = (base + l < c1) ? __builtin_nontemporal_load(indices + base + l) : 0;
            const int m = (int)min<int64_t>(LG, c1 - base);
            for (int j0 = 0; j0 < m; j0 += 8) {
                u32 r[8];
                float4 v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) r[j] = LG >= 8 || j < LG ? (u32)__shfl(cur_idx, j0 + j, LG) : 0u;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if ((LG >= 8 || j < LG) && j0 + j < m) v[j] = rows[(u64)r[j] * LG];
                }
                acc0 = add4(add4(add4(add4(acc0, v[0]), v[1]), v[2]), v[3]);
                acc1 = add4(add4(add4(add4(acc1, v[4]), v[5]), v[6]), v[7]);
            }
        }
        const float4 acc = add4(acc0, acc1);
        float* x = second ? a.set[1].x : a.set[0].x;
        bf16_t* x_bf = second ? a.set[1].x_bf : a.set[0].x_bf;
        if (x) {
            __builtin_nontemporal_store(acc.x, x + o); __builtin_nontemporal_store(acc.y, x + o + 1);
            __builtin_nontemporal_store(acc.z, x + o + 2); __builtin_nontemporal_store(acc.w, x + o + 3);
        }
        if (x_bf) store_bf4(x_bf + o, acc);
        if (it >= hi) break;
        f = fn;
        u = (u32)un;
    }
}

static inline unsigned pool_grid(int64_t n_bags, int groups_per_block) {
    int64_t nb = (n_bags + groups_per_block - 1) / groups_per_block;
    const int64_t cap = 256 * 32;  // grid-stride beyond 32 blocks per CU
    if (nb > cap) nb = cap;
    if (nb < 1) nb = 1;
    return (unsigned)nb;
}

void launch_gather_pool(hipStream_t st, int F, int D, int n_dense, const int64_t* field_base, const float* emb, int ldx,
                        const PoolSet& s0, const PoolSet& s1) {
    const int64_t n = s0.n_samples + s1.n_samples, n_bags = n * F;
    if (n <= 0) return;
    PoolArgs a{F, D, F > 0 ? D / 4 : 1, n_dense, ldx, 0, field_base, reinterpret_cast<const float4*>(emb), {s0, s1}};
    const bool by_xcd = n_bags > 0 && F >= 8 && n_bags >= (1 << 14);
    if (n_bags > 0) a.pool_blocks = by_xcd ? pool_grid(n_bags, 256 / a.LG) / 8 * 8 : pool_grid(n_bags, 256 / a.LG);
    const unsigned grid = a.pool_blocks + (unsigned)((n * (ldx - F * D) + 255) / 256);
#define POOL_XCD(LG_) case LG_: hipLaunchKernelGGL(gather_pool_xcd_kernel<LG_>, dim3(grid), dim3(256), 0, st, a); break;
    if (by_xcd) {
        switch (a.LG) { POOL_XCD(1) POOL_XCD(2) POOL_XCD(4) POOL_XCD(8) POOL_XCD(16) POOL_XCD(32) POOL_XCD(64) default: break; }
    } else if (grid > 0) {
        hipLaunchKernelGGL(gather_pool_kernel, dim3(grid), dim3(256), 0, st, a);
    }
#undef POOL_XCD
}

// dense and pad columns of every (padded) row, copied from x_base
__global__ void copy_tail_kernel(int FD, const float* x_base, int64_t n_rows, float* x_out, int ldx, bf16_t* x_bf) {
    const int tail = ldx - FD;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_rows * tail) return;
    const int64_t s = i / tail;
    const int c = (int)(i - s * tail);
    const float v = x_base[s * ldx + FD + c];
    if (x_out) x_out[s * ldx + FD + c] = v;
    if (x_bf) x_bf[s * ldx + FD + c] = f2bf(v);
}

void launch_copy_tail(hipStream_t st, int FD, const float* x_base, int64_t n_rows, float* x_out, int ldx, bf16_t* x_bf) {
    const int64_t nt = n_rows * (ldx - FD);
    if (nt > 0)
        hipLaunchKernelGGL(copy_tail_kernel, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, st, FD, x_base, n_rows,
                           x_out, ldx, x_bf);
}

// ------------------------------------------------------------------------------------------------
// global segment reduction: emb_grad[seg] = sum over the segment's lookups (stable (field,row) order) of
// gx[(row of the sample, field)], gx laid out [rows (support then query), F, D].
//
// Under Zipf skew a hot row's segment holds a large share of all lookups, so segments are not the unit
// of work: the sorted lookup list is cut into fixed chunks of SEG_CH positions, one lane group walks one
// chunk, a segment that lies inside one chunk is written directly, and a segment that crosses chunk
// borders leaves one partial sum per chunk that a second pass adds in chunk order.  The cutting depends
// only on positions, so the order of every sum is fixed.
// ------------------------------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 load_once(const float* p) { return __builtin_bit_cast(float4, __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p))); }
__device__ __forceinline__ float4 only(float4 x, u32 keep) {   // x or zeros, by a mask of all bits or none (a condition becomes branches around every read)
    uint4 b = __builtin_bit_cast(uint4, x);
    b.x &= keep; b.y &= keep; b.z &= keep; b.w &= keep;
    return __builtin_bit_cast(float4, b);
}
__device__ __forceinline__ void store_once(float* p, float4 v) { __builtin_nontemporal_store(__builtin_bit_cast(f32x4, v), reinterpret_cast<f32x4*>(p)); }

#define SEG_CH 64         // positions per chunk
#define SEG_SMALL_N 32768 // Short lists of narrow rows take chunks of 16 or 32, as the room for their partial rows allows: 64 leave the
                          // device idle and a lane group of D/4 <= 4 lanes walking its chunk 4 positions at a time (2048 lookups of
                          // 16 columns: 23 -> 8 us).  The chunk follows from n, F and D alone.
static size_t seg_floats(int64_t n, int D, int ch) { return (size_t)((n + ch - 1) / ch) * 2 * D + 16; }
size_t seg_reduce_partial_floats(int64_t n, int D) { return seg_floats(n, D, SEG_CH); }
int seg_chunk(int64_t n, int F, int D) {
    if (n > SEG_SMALL_N || D > 16) return SEG_CH;
    const size_t room = (size_t)n + radix_hist_words(n, F) + seg_floats(n, D, SEG_CH);   // at least this, see launch_seg_reduce
    for (int ch = 16; ch < SEG_CH; ch *= 2)
        if (seg_floats(n, D, ch) <= room) return ch;
    return SEG_CH;
}

#define SEG_BLOCK 256               // positions whose first keys tell a long segment: four chunks
#define SEG_SLICE (1 << 19)         // bytes of one field's gradient rows that a place in the list covers
#define SEG_BUCKETS 4096            // places in the list
#define SEG_HOT_N (4 << 20)         // lookups from which on the list is made
__device__ __forceinline__ bool seg_block_hot(const u32* keys, int64_t b, int64_t n) {   // all of the block, and a position on either side, has one key
    if (b == 0 || (b + 1) * SEG_BLOCK >= n) return false;
    const u32 k0 = keys[(b - 1) * SEG_BLOCK], k2 = keys[(b + 1) * SEG_BLOCK];
    return k0 == k2;
}

// One lane group (LG = D/4 lanes, a float4 of the row each) walks one chunk.  The chunk's metadata is read LG positions
// at a time, one position per lane (coalesced), and handed round the group by lane shuffles; the head flags of
// the LG positions come back as one ballot word.  Whether a run began before the chunk or continues past it
// follows from the head flags at the chunk's two borders, so no segment table is read here.
// What is written goes past the caches (non-temporal), which are the gradient rows': 72 million lookups, 7 million rows listed 1.64 -> 1.52 ms;
// 26 million added to table rows 1.48 -> 1.45.
// CH: the chunk's length, 0 where `short_ch` says it.  ZERO: places of gx below `zero` are zeros: a chunk reads one and the same of the `others` + 1 behind
// them in their stead and does not look at it (a first-order gradient has nothing for the support set's lookups: 201 tasks of 75..225 + 122..365 rows, 22 million lookups, their zeros filled in (27 us)
// and read 492 + 195 us in the two kernels, 403 + 127 so; the hot one leaves chunks of zeros out).
template <int LG, int CH, bool ZERO>
__global__ void __launch_bounds__(256)
seg_reduce_chunks_kernel(int D, int F, int short_ch, ValEnc enc, const u32* __restrict__ keys, const u32* __restrict__ scan,
                         const int64_t* __restrict__ n_rows, int64_t capacity, int64_t n,
                         const u32* __restrict__ sorted_vals, const float* __restrict__ gx, int64_t* emb_rows, float* emb_grad,
                         float* partial, float* table, float scale, int hot, u32 zero, u32 others) {
    constexpr int GPB = 256 / LG;            // lane groups per workgroup
    constexpr int U = LG < 8 ? LG : 8;       // row loads in flight per lane
    const int ch = CH ? CH : short_ch;
    const int g_in_block = threadIdx.x / LG, l = threadIdx.x % LG;
    const int group_lane0 = (threadIdx.x % 64) / LG * LG;   // the group's first lane inside its wave
    const int64_t n_valid = table ? 0 : min(*n_rows, capacity);
    const int64_t n_chunks = (n + ch - 1) / ch;
    const int64_t n_groups = (int64_t)gridDim.x * GPB;
    const float4* gx4 = reinterpret_cast<const float4*>(gx);
    for (int64_t c = (int64_t)blockIdx.x * GPB + g_in_block; c < n_chunks; c += n_groups) {
        const u32 spare = ZERO ? zero + ((u32)c & others) : 0u;
        const int64_t cb = c * ch;
        const int cnt = (int)min((int64_t)ch, n - cb);
        if (hot && seg_block_hot(keys, cb / SEG_BLOCK, n)) continue;   // (the other kernel's)
        // borders: does the chunk's last run go on in the next chunk; which segment does position cb lie in
        const bool goes_on = (cb + cnt < n) && keys[cb + cnt] == keys[cb + cnt - 1];
        int64_t seg = table ? 0 : (int64_t)scan[c] - 1;     // + 1 at every head, the one at cb included
        int64_t listed = seg + 1;                           // segments whose row is in the list
        u32 v_next = 0, k_next = 0;
        bool h_next = false;
        auto load_meta = [&](int p0) {       // positions cb + p0 + l of the chunk
            const int p = p0 + l;
            v_next = 0, k_next = 0, h_next = false;
            if (p < cnt) {
                const int64_t i = cb + p;
                v_next = sorted_vals[i];
                // (bit-field values: the bag's place in the gradient buffer is row * F + field)
                if (enc.rshift) v_next = (v_next >> enc.rshift) * (u32)F + ((v_next >> enc.pshift) & enc.fmask);
                k_next = keys[i];
                h_next = (i == 0) || keys[i - 1] != k_next;
            }
        };
        load_meta(0);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        bool began_before = false;           // the current run began in an earlier chunk
        u32 run_key = 0;
        auto flush = [&](bool continues) {
            float* dst;
            if (began_before) dst = partial + (c * 2 + 0) * D;
            else if (continues) dst = partial + (c * 2 + 1) * D;
            else if (table) {  // table-shaped output: added to the segment's row (rows of one call are distinct)
                float* tp = table + (int64_t)run_key * D + l * 4;
                store_once(tp, fma4(scale, acc, load_once(tp)));
                return;
            } else {
                if (seg >= n_valid) return;
                dst = emb_grad + seg * D;
            }
            store_once(dst + l * 4, acc);
        };
        for (int p0 = 0; p0 < cnt; p0 += LG) {
            const u32 v = v_next, k = k_next;
            const unsigned long long heads = (__ballot(h_next) >> group_lane0) & (~0ull >> (64 - LG));
            if (!table) {   // (the row list: the positions' segments in one store)
                const int64_t at = listed + __popcll(heads & ((1ull << l) - 1ull));
                if (h_next && at < n_valid) __builtin_nontemporal_store((int64_t)k, emb_rows + at);
                listed += __popcll(heads);
            }
            if (p0 + LG < cnt) load_meta(p0 + LG);
            const int m = min(LG, cnt - p0);
            for (int s0 = 0; s0 < m; s0 += U) {
                u32 vv[U], kk[U];
                float4 x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    vv[u] = __shfl(v, s0 + u, LG);          // lanes past cnt hold row 0: a valid, unused read
                    kk[u] = __shfl(k, s0 + u, LG);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const u32 keep = !ZERO || vv[u] >= zero ? ~0u : 0u;
                    x[u] = only(gx4[(int64_t)(ZERO ? (vv[u] & keep) | (spare & ~keep) : vv[u]) * LG + l], keep);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int s = s0 + u;
                    if (s >= m) break;
                    const bool head = (heads >> s) & 1;
                    if (p0 + s == 0) {
                        began_before = !head;
                        seg += head ? 1 : 0;
                        run_key = kk[u];
                        acc = x[u];
                    } else if (head) {
                        flush(false);
                        began_before = false;
                        seg += 1;
                        run_key = kk[u];
                        acc = x[u];
                    } else {
                        acc = add4(acc, x[u]);
                    }
                }
            }
        }
        flush(goes_on);
    }
}

// Chunks in the middle of a long segment -- half the lookups of a skewed batch and more -- all read the gradient rows of one
// field, but chunk by chunk in the rows' order every segment walks through all of the batch's samples anew, far more than an
// L2 holds, and the memory-side cache is the bound (7.1 TB/s of line fills, 12 % of the reads found in L2).  So they are taken
// in another order: field by field, and inside a field by where in the batch their samples lie (SEG_SLICE bytes of gradient rows
// at a time), each XCD its own part of that list.  The chunks, their sums and the places they go to stay the same.
// 72 million lookups of 64 columns, Zipf 1.1: 2.81 ms in one kernel, 1.56 + 0.80 and 0.04 for the list in two; 138 million,
// 64 fields, Zipf 1.05: 6.08, 4.51 + 1.32 + 0.07; 18 million 0.65, 0.43 + 0.17 + 0.01 -- shorter lists have little to gain
// (SEG_HOT_N).
// Two passes over the blocks: FILL false counts a bucket's chunks, FILL true writes their numbers to list[at[bucket] ..].
template <bool FILL>
__global__ __launch_bounds__(256) void seg_reduce_hot_list_kernel(int F, ValEnc enc, const u32* __restrict__ keys, const u32* __restrict__ vals, int64_t n,
                                                                  int shift, int slices, u32* at, u32* list) {
    __shared__ u32 cnt[SEG_BUCKETS];
    const int n_buckets = F * slices;
    for (int i = threadIdx.x; i < n_buckets; i += 256) cnt[i] = 0;
    __syncthreads();
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool on = seg_block_hot(keys, b, n);
    int bucket[4];
    if (on) {
        u32 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = vals[b * SEG_BLOCK + j * SEG_CH];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const u32 row = enc.rshift ? v[j] >> enc.rshift : v[j] / (u32)F, f = enc.rshift ? (v[j] >> enc.pshift) & enc.fmask : v[j] % (u32)F;
            bucket[j] = (int)min(f * (u32)slices + min(row >> shift, (u32)slices - 1u), (u32)n_buckets - 1u);
            atomicAdd(&cnt[bucket[j]], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n_buckets; i += 256) {
        const u32 c = cnt[i];
        if (c) cnt[i] = atomicAdd(&at[i], c);   // (FILL: where this workgroup's chunks of the bucket go)
    }
    if (!FILL) return;
    __syncthreads();
    if (on)
#pragma unroll
        for (int j = 0; j < 4; ++j) list[atomicAdd(&cnt[bucket[j]], 1u)] = (u32)(b * (SEG_BLOCK / SEG_CH) + j);
}
// One lane group per listed chunk: its 64 gradient rows, added in order.
template <int LG, bool ZERO>
__global__ __launch_bounds__(256) void seg_reduce_hot_kernel(int F, ValEnc enc, const u32* __restrict__ vals, const u32* __restrict__ list,
                                                             const u32* __restrict__ n_list, const float* __restrict__ gx, float* partial, u32 zero) {
    constexpr int GPB = 256 / LG, V = SEG_CH / LG > 0 ? SEG_CH / LG : 1, D = 4 * LG;
    constexpr int W = LG < SEG_CH ? LG : SEG_CH;   // lanes of a group that hold values
    const int g = threadIdx.x / LG, l = threadIdx.x % LG;
    const int64_t total = *n_list, x = blockIdx.x & 7, lo = total * x / 8, hi = total * (x + 1) / 8;
    const int64_t step = (int64_t)(gridDim.x >> 3) * GPB;
    const float4* gx4 = reinterpret_cast<const float4*>(gx);
    u32 c = 0, v[V];
    auto request = [&](int64_t i) {
        c = list[min(i, hi - 1)];
#pragma unroll
        for (int q = 0; q < V; ++q) v[q] = vals[(int64_t)c * SEG_CH + q * W + (l & (W - 1))];
    };
    int64_t i = lo + (int64_t)(blockIdx.x >> 3) * GPB + g;
    if (i >= hi) return;
    request(i);
    for (; i < hi; i += step) {
        const u32 cc = c;
        u32 r[V];
#pragma unroll
        for (int q = 0; q < V; ++q) r[q] = enc.rshift ? (v[q] >> enc.rshift) * (u32)F + ((v[q] >> enc.pshift) & enc.fmask) : v[q];
        request(i + step);   // (the next chunk's, beside this one's rows)
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        auto sum = [&](auto masked) {
#pragma unroll
            for (int q = 0; q < V; ++q)
#pragma unroll
                for (int s0 = 0; s0 < W; s0 += 8) {
                    float4 y[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const u32 at = (u32)__shfl((int)r[q], s0 + u, LG), keep = !masked || at >= zero ? ~0u : 0u;
                        y[u] = only(gx4[(int64_t)(masked ? max(at, zero) : at) * LG + l], keep);
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) acc = q == 0 && s0 == 0 && u == 0 ? y[0] : add4(acc, y[u]);
                }
        };
        if constexpr (ZERO) {   // (inside a row the places ascend)
            if ((u32)__shfl((int)r[V - 1], W - 1, LG) >= zero) {
                if ((u32)__shfl((int)r[0], 0, LG) >= zero) sum(std::false_type());
                else sum(std::true_type());
            }
        } else sum(std::false_type());
        *reinterpret_cast<float4*>(partial + (int64_t)cc * 2 * D + l * 4) = acc;
    }
}

// One lane group per CHUNK: if the chunk's last run begins inside the chunk and goes on past it, this group adds
// the pieces the following chunks left (each of them starts with the same key) in chunk order.  Every such
// segment is the last one of exactly one chunk.
//
// Bound: a segment is a serial chain of sums, and a hot row's has thousands of pieces; a lane group keeps eight reads in flight.
// Segments of more than JOIN_LONG pieces are therefore left to the whole workgroup, which stages JOIN_U pieces per lane group
// in LDS (the next ones on their way meanwhile) while a thread per column adds them in the same order: the same bits.
// Measured: 18 M lookups of 26 fields (128 tasks, rows by Zipf 1.1) 154 -> 78 us, 70 M of 26 fields 502 -> 265, 138 M of 64 fields 572 -> 440.
#define JOIN_LONG 32      // pieces of a segment that a lane group adds by itself (four rounds of reads)
#define JOIN_U 4          // pieces per lane group and round of the workgroup: 64 of 64 columns, 16 KB of LDS
#define JOIN_LIST 32      // long segments a workgroup puts off; further ones are added by their lane groups
template <int LG>
__global__ __launch_bounds__(256) void seg_reduce_join_kernel(int ch, const u32* __restrict__ keys, const u32* __restrict__ scan,
                                                              const int64_t* __restrict__ n_rows, int64_t capacity, int64_t n,
                                                              const float* __restrict__ partial, float* emb_grad, float* table, float scale) {
    constexpr int GPB = 256 / LG, D = 4 * LG, ROUND = GPB * JOIN_U;
    __shared__ float4 stage[ROUND * LG];
    __shared__ int64_t list_c[JOIN_LIST], list_row[JOIN_LIST];
    __shared__ int n_list;
    if (threadIdx.x == 0) n_list = 0;
    __syncthreads();
    const int g_in_block = threadIdx.x / LG, l = threadIdx.x % LG;
    const int64_t n_valid = table ? 0 : min(*n_rows, capacity);
    const int64_t n_chunks = (n + ch - 1) / ch;
    const int64_t n_groups = (int64_t)gridDim.x * GPB;
    auto piece = [&](int64_t c, int which) { return *reinterpret_cast<const float4*>(partial + (c * 2 + which) * D + l * 4); };
    auto finish = [&](int64_t row, float4 acc) {
        float4* dst = reinterpret_cast<float4*>((table ? table : emb_grad) + row * D + l * 4);
        *dst = table ? fma4(scale, acc, *dst) : acc;
    };
    for (int64_t c = (int64_t)blockIdx.x * GPB + g_in_block; c + 1 < n_chunks; c += n_groups) {
        const int64_t cb = c * ch, ce = cb + ch;   // not the last chunk, so it is full and ce < n
        const u32 key = keys[ce - 1];
        if (keys[ce] != key) continue;                     // the run ends with the chunk
        if (cb > 0 && keys[cb - 1] == key) continue;       // began in an earlier chunk, which adds it up
        int64_t row = key;
        if (!table) {
            row = (int64_t)scan[c + 1] - 1;   // (the chunk's last segment)
            if (row >= n_valid) continue;
        }
        auto starts_with_key = [&](int64_t cc) { return cc < n_chunks && keys[cc * ch] == key; };
        int64_t c1 = c + 1, hi = n_chunks;     // chunk c1 starts with the key; from chunk hi on none does
        if (starts_with_key(c + JOIN_LONG + 1)) {
            int at = 0;
            if (l == 0) at = atomicAdd(&n_list, 1);
            at = __shfl(at, 0, LG);
            if (at < JOIN_LIST) {
                if (l == 0) { list_c[at] = c; list_row[at] = row; }
                continue;
            }
            c1 = c + JOIN_LONG + 1;
        } else {
            hi = min(n_chunks, c + JOIN_LONG + 1);
        }
        // c1 becomes the last chunk that starts with the key.  Most segments end in chunk c + 1: gallop forward in doubling
        // steps, then bisect (the keys are sorted).
        int64_t step = 1;
        while (c1 + step < hi && starts_with_key(c1 + step)) {
            c1 += step;
            step *= 2;
        }
        hi = min(hi, c1 + step);
        while (hi - c1 > 1) {
            const int64_t mid = c1 + (hi - c1) / 2;
            if (starts_with_key(mid)) c1 = mid;
            else hi = mid;
        }
        float4 acc = piece(c, 1);
        int64_t cc = c + 1;
        for (; cc + 8 <= c1 + 1; cc += 8) {       // 8 independent loads in flight, added in chunk order
            float4 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = piece(cc + u, 0);
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = add4(acc, x[u]);
        }
        for (; cc <= c1; ++cc) acc = add4(acc, piece(cc, 0));
        finish(row, acc);
    }
    __syncthreads();
    const int n_long = min(n_list, JOIN_LIST);
    for (int i = 0; i < n_long; ++i) {
        const int64_t c = list_c[i];
        const u32 key = keys[(c + 1) * ch];
        int64_t c1 = c + JOIN_LONG + 1;            // starts with the key; all threads look for the last chunk that does
        for (int64_t hi = n_chunks; hi - c1 > 1;) {
            const int64_t step = (hi - c1 + 255) / 256, at = c1 + threadIdx.x * step;
            const int k = __syncthreads_count(at < hi && keys[at * ch] == key);   // (the first one does)
            c1 += (k - 1) * step;
            hi = min(hi, c1 + step);
        }
        float4 x[JOIN_U];
        auto request = [&](int64_t first) {        // (past the segment's end: its last piece again, not added)
#pragma unroll
            for (int u = 0; u < JOIN_U; ++u) x[u] = piece(min(first + u * GPB + g_in_block, c1), 0);
        };
        const float* column = reinterpret_cast<const float*>(stage) + threadIdx.x;   // of the thread below that adds it up
        float acc = threadIdx.x < D ? partial[(c * 2 + 1) * D + threadIdx.x] : 0.f;
        request(c + 1);
        for (int64_t first = c + 1; first <= c1; first += ROUND) {
            __syncthreads();                       // the previous pieces have been added
#pragma unroll
            for (int u = 0; u < JOIN_U; ++u) stage[(u * GPB + g_in_block) * LG + l] = x[u];
            __syncthreads();
            if (first + ROUND <= c1) request(first + ROUND);
            if (threadIdx.x < D) {
                const int m = (int)min<int64_t>(ROUND, c1 + 1 - first);
                int q = 0;
                for (; q + 16 <= m; q += 16) {
                    float y[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) y[u] = column[(q + u) * D];
#pragma unroll
                    for (int u = 0; u < 16; ++u) acc += y[u];
                }
                for (; q < m; ++q) acc += column[q * D];
            }
        }
        if (threadIdx.x < D) {
            float* dst = (table ? table : emb_grad) + list_row[i] * D + threadIdx.x;
            *dst = table ? fmaf(scale, acc, *dst) : acc;
        }
    }
}

void launch_seg_reduce(hipStream_t st, int D, int F, ValEnc enc, const u32* keys, const u32* scan, const int64_t* n_rows, int64_t capacity, int64_t n, const u32* sorted_vals, const float* gx,
                       int64_t* emb_rows, float* emb_grad, float* partial, float* table, float scale, int64_t gx_rows, int64_t zero_rows, u32* room) {
    if (n <= 0 || capacity <= 0) return;
    const int LG = D / 4, ch = seg_chunk(n, F, D);
    const int64_t n_chunks = (n + ch - 1) / ch;
    const dim3 grid(pool_grid(n_chunks, 256 / LG));
    const u32 zero = gx_rows > zero_rows ? (u32)(zero_rows * F) : 0u;   // (row * F + field fits 32 bits; without other rows they hold zeros)
    u32 others = 0;   // places read in the zeros' stead, less one
    while (2 * (others + 1) <= 65536u && 2 * (int64_t)(others + 1) <= (gx_rows - zero_rows) * F) others = 2 * others + 1;
    const int hot = D >= 32 && D <= 128 && F <= SEG_BUCKETS / 2 && n >= SEG_HOT_N;
    if (hot) {
        int shift = 0;   // samples of a slice, as a power of two
        while (((int64_t)D * 4 << shift) < SEG_SLICE || (gx_rows >> shift) + 1 > SEG_BUCKETS / F) ++shift;
        const int slices = (int)(gx_rows >> shift) + 1;
        u32 *at = room, *total = room + SEG_BUCKETS, *tmp = total + 64, *list = tmp + 4096;
        const unsigned nb = (unsigned)((n / SEG_BLOCK + 255) / 256);
        launch_fill_u32(st, at, SEG_BUCKETS, 0);
        hipLaunchKernelGGL((seg_reduce_hot_list_kernel<false>), dim3(nb), dim3(256), 0, st, F, enc, keys, sorted_vals, n, shift, slices, at, list);
        launch_scan_u32(st, at, at, SEG_BUCKETS, tmp, total);
        hipLaunchKernelGGL((seg_reduce_hot_list_kernel<true>), dim3(nb), dim3(256), 0, st, F, enc, keys, sorted_vals, n, shift, slices, at, list);
#define SEG_HOT(LG_)                                                                                                 \
    case LG_:                                                                                                        \
        if (zero) hipLaunchKernelGGL((seg_reduce_hot_kernel<LG_, true>), dim3(4096), dim3(256), 0, st, F, enc, sorted_vals, list, total, gx, partial, zero); \
        else hipLaunchKernelGGL((seg_reduce_hot_kernel<LG_, false>), dim3(4096), dim3(256), 0, st, F, enc, sorted_vals, list, total, gx, partial, zero); \
        break;
        switch (LG) { SEG_HOT(8) SEG_HOT(16) SEG_HOT(32) default: break; }
#undef SEG_HOT
    }
    // (the long chunk is a constant of its kernels: 100 tasks x (300 + 300) rows of 32 columns 99 us with a variable length, 90 with 64)
#define SEG_CHUNKS(LG_, CH_)                                                                                         \
    case LG_:                                                                                                        \
        if (zero) hipLaunchKernelGGL((seg_reduce_chunks_kernel<LG_, CH_, true>), grid, dim3(256), 0, st, D, F, ch, enc, keys, scan, n_rows, capacity, n, \
                                     sorted_vals, gx, emb_rows, emb_grad, partial, table, scale, hot, zero, others);             \
        else hipLaunchKernelGGL((seg_reduce_chunks_kernel<LG_, CH_, false>), grid, dim3(256), 0, st, D, F, ch, enc, keys, scan, n_rows, capacity, n, \
                                sorted_vals, gx, emb_rows, emb_grad, partial, table, scale, hot, zero, others);                  \
        break;
    if (ch == SEG_CH) {
        switch (LG) {
            SEG_CHUNKS(1, SEG_CH) SEG_CHUNKS(2, SEG_CH) SEG_CHUNKS(4, SEG_CH) SEG_CHUNKS(8, SEG_CH) SEG_CHUNKS(16, SEG_CH) SEG_CHUNKS(32, SEG_CH) SEG_CHUNKS(64, SEG_CH)
            default: return;   // emb_dim is a power of two in 4..256 (checked when the context is made)
        }
    } else {
        switch (LG) {
            SEG_CHUNKS(1, 0) SEG_CHUNKS(2, 0) SEG_CHUNKS(4, 0)   // (short chunks: at most 16 columns)
            default: return;
        }
    }
#undef SEG_CHUNKS
#define SEG_JOIN(LG_)                                                                                                \
    case LG_:                                                                                                        \
        hipLaunchKernelGGL(seg_reduce_join_kernel<LG_>, grid, dim3(256), 0, st, ch, keys, scan, n_rows, capacity, n, partial, emb_grad, table, scale); \
        break;
    switch (LG) { SEG_JOIN(1) SEG_JOIN(2) SEG_JOIN(4) SEG_JOIN(8) SEG_JOIN(16) SEG_JOIN(32) SEG_JOIN(64) default: break; }
#undef SEG_JOIN
}

__global__ void scatter_add_kernel(int D, int LG, float* table, const int64_t* __restrict__ rows,
                                   const float* __restrict__ grad, int64_t n_rows, float scale) {
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = gt / LG;
    const int l = (int)(gt % LG);
    if (i >= n_rows) return;
    float4* dst = reinterpret_cast<float4*>(table + rows[i] * D + l * 4);
    const float4 g = *reinterpret_cast<const float4*>(grad + i * D + l * 4);
    float4 o = *dst;
    o.x += scale * g.x; o.y += scale * g.y; o.z += scale * g.z; o.w += scale * g.w;
    *dst = o;
}

void launch_scatter_add(hipStream_t st, int D, float* table, const int64_t* rows, const float* grad, int64_t n_rows,
                        float scale) {
    if (n_rows <= 0) return;
    const int LG = D / 4;
    const int64_t nt = n_rows * LG;
    hipLaunchKernelGGL(scatter_add_kernel, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, st, D, LG, table, rows, grad,
                       n_rows, scale);
}
