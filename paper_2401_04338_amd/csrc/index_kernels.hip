// Integer side of the MAML step (G-Meta Alg. 1): the per-(task, field) row dictionaries behind the
// inner-loop row update and the overlap join of Sec. 2.1.2, and the global (field,row) ordering that
// routes the sparse meta-gradient (Alg. 1, global back-propagation on xi).  Everything here has exactly
// one correct answer and is compared bit-exactly with the CPU oracle.
#include <algorithm>

#include "gm_internal.h"

#define WAVE 64

// ------------------------------------------------------------------------------------------------
// small helpers
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ int wave_incl_scan(int v) {
    const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        int o = __shfl_up(v, d, WAVE);
        if (lane >= d) v += o;
    }
    return v;
}

// Exclusive scan of one int per thread over the block; `sh` holds >= blockDim/64 + 1 ints.
__device__ __forceinline__ int block_excl_scan(int v, int* sh, int* total) {
    const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
    int incl = wave_incl_scan(v);
    __syncthreads();
    if (lane == WAVE - 1) sh[wid] = incl;
    __syncthreads();
    if (wid == 0) {
        int x = lane < nw ? sh[lane] : 0;
        int xi = wave_incl_scan(x);
        if (lane < nw) sh[lane] = xi - x;
        if (lane == nw - 1) sh[nw] = xi;
    }
    __syncthreads();
    int r = sh[wid] + incl - v;
    *total = sh[nw];
    return r;
}

// ------------------------------------------------------------------------------------------------
// validation + per-(task, field) lookup counts
// ------------------------------------------------------------------------------------------------
// One (task, set) per workgroup, or gridDim.z of them where the tasks are few: then cnt_sup / cnt_qry must be zero on entry.
// A well-formed input that exceeds a size limit of the index kernels (a bag of more than 65,535 lookups, a task of more
// than 65,536 samples in one set) raises ST_TOO_LARGE, not ST_BAD_INDEX.
// uniform_rows >= 0: every table has that many rows, so an index is checked without knowing its field: the task's
// lookups, one contiguous range, are then read by all lanes in order instead of bag by bag.
// Bound: the two reads and the atomics.  Those that leave the workgroup queue at the memory side (some 30 ns each on one
// address, about one a nanosecond in all), so there are none but a status word's where a workgroup has its (task, set) for itself,
// and that one only where the word holds less: 13 workgroups a task, both sets in each, took 93 us for 128 tasks x (256 + 256)
// samples x 26 fields and 160 us for 128 x (512 + 512) x 64.
#define TC_NT 1024
__global__ __launch_bounds__(TC_NT) void tf_count_kernel(int F, int t0, SetView sup, SetView qry, const int64_t* field_base,
                                int64_t nnz_sup, int64_t nnz_qry, int64_t uniform_rows, u32* cnt_sup, u32* cnt_qry, u32* status) {
    extern __shared__ u32 sh_cnt[];  // [F]
    __shared__ u32 sh_most, sh_longest, sh_flags;
    const int t = blockIdx.x, set = blockIdx.y;
    for (int i = threadIdx.x; i < F; i += TC_NT) sh_cnt[i] = 0;
    if (threadIdx.x == 0) { sh_most = 0; sh_longest = 0; sh_flags = 0; }
    __syncthreads();
    bool bad = false, too_large = false;
    u32 longest = 0;
    const SetView& v = set ? qry : sup;
    const int64_t nnz = set ? nnz_qry : nnz_sup;
    const int64_t s_lo = v.task_offsets[t0 + t], s_hi = v.task_offsets[t0 + t + 1];
    if (s_hi - s_lo > 65536) too_large = true;
    const int64_t n = (s_hi - s_lo) * F, step = (int64_t)gridDim.z * TC_NT, i0 = (int64_t)blockIdx.z * TC_NT + threadIdx.x;
    const int64_t* bags = v.bag_offsets + s_lo * F;
    int f = (int)((u32)i0 % (u32)F);   // field of the bag
    const int f_step = (int)((u32)step % (u32)F);
    for (int64_t i = i0; i < n; i += 4 * step) {
        int64_t p[4][2];   // four bags in flight
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t j = i + k * step < n ? i + k * step : i;
            p[k][0] = bags[j];
            p[k][1] = bags[j + 1];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i + k * step >= n) break;
            const int64_t p0 = p[k][0], p1 = p[k][1];
            const int f0 = f;
            f += f_step;
            if (f >= F) f -= F;
            if (p0 < 0 || p1 < p0 || p1 > nnz) {
                bad = true;
                continue;
            }
            if (p1 - p0 > 65535) {
                too_large = true;
                continue;
            }
            if (uniform_rows < 0) {
                const int64_t R = field_base[f0 + 1] - field_base[f0];
                for (int64_t q = p0; q < p1; ++q) {
                    const int32_t r = v.indices[q];
                    if (r < 0 || r >= R) bad = true;
                }
            }
            atomicAdd(&sh_cnt[f0], (u32)(p1 - p0));
            longest = max(longest, (u32)(p1 - p0));
        }
    }
    if (uniform_rows >= 0 && n > 0) {   // (offsets outside [0, nnz] are flagged above; the range read here is clamped)
        const int64_t q0 = min(max(bags[0], (int64_t)0), nnz), q1 = min(max(bags[n], q0), nnz);
        for (int64_t p = q0 + i0; p < q1; p += 8 * step) {
            int32_t r[8];   // eight reads in flight (past the end: the first one's index again)
#pragma unroll
            for (int k = 0; k < 8; ++k) r[k] = v.indices[p + k * step < q1 ? p + k * step : p];
#pragma unroll
            for (int k = 0; k < 8; ++k) bad |= r[k] < 0 || r[k] >= uniform_rows;
        }
    }
    if (t == 0 && blockIdx.z == 0 && threadIdx.x == 0)  // the ends of the offset array
        if (v.bag_offsets[0] != 0 || v.bag_offsets[v.n_samples * F] != nnz) bad = true;
    __syncthreads();
    u32 most = 0;
    u32* const cnt = (set ? cnt_qry : cnt_sup) + (size_t)t * F;
    for (int i = threadIdx.x; i < F; i += TC_NT) {
        const u32 c = sh_cnt[i];
        if (gridDim.z == 1) {
            cnt[i] = c;
            most = max(most, c);
        } else if (c) most = max(most, atomicAdd(&cnt[i], c) + c);     // the (task, field)'s count so far: the last adder sees the total
    }
    for (int d = WAVE / 2; d > 0; d >>= 1) {
        most = max(most, (u32)__shfl_xor((int)most, d, WAVE));
        longest = max(longest, (u32)__shfl_xor((int)longest, d, WAVE));
    }
    const int flags = (__ballot(bad) ? 1 : 0) | (__ballot(too_large) ? 2 : 0);
    if ((threadIdx.x & (WAVE - 1)) == 0) {
        atomicMax(&sh_most, most);
        atomicMax(&sh_longest, longest);
        if (flags) atomicOr(&sh_flags, (u32)flags);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        auto raise = [&](u32 value, int word) {
            if (value > __hip_atomic_load(&status[word], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&status[word], value);
        };
        raise(sh_most, ST_MAX_TF);
        raise(sh_longest, ST_MAX_BAG);
        if (sh_flags & 1u) atomicOr(&status[ST_BAD_INDEX], 1u);
        if (sh_flags & 2u) atomicOr(&status[ST_TOO_LARGE], 1u);
    }
}

void launch_tf_count(hipStream_t st, int F, int t0, int Tw, int64_t most_bags, int64_t all_bags, SetView sup, SetView qry, const int64_t* field_base,
                     int64_t nnz_sup, int64_t nnz_qry, int64_t uniform_rows, u32* cnt_sup, u32* cnt_qry, u32* status, bool cleared) {
    if (Tw <= 0) return;
    // A (task, set) is split, down to a bag a thread, while the workgroups are fewer than 128: a few large tasks would leave the chip
    // idle (3 tasks x 32,768 + 32,768 bags: 57 us whole, 18 in 21 parts).  From there on a part costs as much as it saves (the counts are cleared and
    // added with atomics: 64 tasks x 3,328 + 3,328 bags 12 us whole, 20 in two; 96 x 6,656 + 6,656 23 and 32) but for parts of 8,192 bags or more:
    // while the workgroups are fewer than 256 (48 tasks x 32,768 + 32,768 bags 113 us whole, 94 in two), and where one task is larger than the
    // others and would alone be the launch's time, fewer than 2,048, most of which then find nothing to do (one task of 81,920 + 81,920 bags and 99
    // of 80 + 80 67 us whole, 31 in ten; 299 70, in three 46; two tasks of 40,960 and 28,000 and 700 of 1,600 56, in two 63).
    const int64_t most_parts = 4 * all_bags < most_bags * Tw ? 1024 / Tw : 128 / Tw;
    const int split = (int)std::max<int64_t>({1, std::min<int64_t>(most_bags / TC_NT, 64 / Tw), std::min(most_bags / (2 * 8192), most_parts)});
    const int64_t counts = split > 1 ? (int64_t)Tw * F : 0;
    if (split > 1 || !cleared) launch_zero(st, ZeroJobs{split > 1 ? 3 : 1, {status, cnt_sup, cnt_qry}, {ST_WORDS, counts, counts}});
    hipLaunchKernelGGL(tf_count_kernel, dim3(Tw, 2, split), dim3(TC_NT), F * sizeof(u32), st, F, t0, sup, qry, field_base,
                       nnz_sup, nnz_qry, uniform_rows, cnt_sup, cnt_qry, status);
}

// ------------------------------------------------------------------------------------------------
// device-wide exclusive scan of u32 (three-phase, recursive on the block sums)
// ------------------------------------------------------------------------------------------------
#define SCAN_NT 256
#define SCAN_ITEMS 8
#define SCAN_TILE (SCAN_NT * SCAN_ITEMS)

// (a thread's 8 items are 32 contiguous bytes: two 16-byte accesses when the pointers allow and the items are all inside)
__global__ void scan_block_kernel(const u32* in, u32* out, int64_t n, u32* block_sums) {
    __shared__ int sh[SCAN_NT / WAVE + 2];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    const bool wide = base + SCAN_ITEMS <= n && ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
    u32 v[SCAN_ITEMS];
    u32 sum = 0;
    if (wide) {
        const uint4 a = *reinterpret_cast<const uint4*>(in + base), b = *reinterpret_cast<const uint4*>(in + base + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
        for (int i = 0; i < SCAN_ITEMS; ++i) v[i] = (base + i < n) ? in[base + i] : 0u;
    }
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) sum += v[i];
    int total;
    u32 run = (u32)block_excl_scan((int)sum, sh, &total);
    u32 o[SCAN_ITEMS];
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        o[i] = run;
        run += v[i];
    }
    if (wide) {
        *reinterpret_cast<uint4*>(out + base) = make_uint4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<uint4*>(out + base + 4) = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
#pragma unroll
        for (int i = 0; i < SCAN_ITEMS; ++i)
            if (base + i < n) out[base + i] = o[i];
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = (u32)total;
}

__global__ void scan_add_kernel(u32* out, int64_t n, const u32* block_offsets) {
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    const u32 o = block_offsets[blockIdx.x];
    if (base + SCAN_ITEMS <= n && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
        uint4* p = reinterpret_cast<uint4*>(out + base);
        uint4 a = p[0], b = p[1];
        a.x += o; a.y += o; a.z += o; a.w += o; b.x += o; b.y += o; b.z += o; b.w += o;
        p[0] = a;
        p[1] = b;
        return;
    }
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i)
        if (base + i < n) out[base + i] += o;
}

// One workgroup scans the whole array, 16384 values at a time: up to SCAN_ONE values that is faster than a launch per
// level.  Measured: 2304 values, 8.8 us in three launches -> 3.9 us in one.
#define SCAN_ONE 32768
struct ScanPair { const u32* in[2]; u32* out[2]; };   // blockIdx.x picks one
struct SegTotal {   // where the number of segments goes (n_rows null: nowhere)
    int64_t* n_rows = nullptr;
    int64_t capacity = 0;
    u32* status = nullptr;
    __device__ __forceinline__ void put(u32 total) const {
        *n_rows = (int64_t)total;
        status[ST_NROWS] = total;
        if ((int64_t)total > capacity) atomicOr(&status[ST_CAPACITY], 1u);
    }
};
__global__ __launch_bounds__(1024) void scan_one_kernel(ScanPair p, int64_t n, u32* total, SegTotal segs) {
    __shared__ int sh[1024 / WAVE + 2];
    const u32* in = p.in[blockIdx.x];
    u32* out = p.out[blockIdx.x];
    const bool wide = ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
    u32 carry = 0;
    for (int64_t base0 = 0; base0 < n; base0 += 16384) {
        const int64_t base = base0 + (int64_t)threadIdx.x * 16;
        u32 v[16];
        u32 sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (wide && base + 4 * q + 4 <= n) {
                const uint4 x = *reinterpret_cast<const uint4*>(in + base + 4 * q);
                v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
            } else {
#pragma unroll
                for (int k = 4 * q; k < 4 * q + 4; ++k) v[k] = base + k < n ? in[base + k] : 0u;
            }
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) sum += v[k];
        int all;
        u32 run = carry + (u32)block_excl_scan((int)sum, sh, &all);
        carry += (u32)all;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32 o[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) { o[k] = run; run += v[4 * q + k]; }
            if (wide && base + 4 * q + 4 <= n) *reinterpret_cast<uint4*>(out + base + 4 * q) = make_uint4(o[0], o[1], o[2], o[3]);
            else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (base + 4 * q + k < n) out[base + 4 * q + k] = o[k];
            }
        }
        __syncthreads();   // the scan's scratch is used again
    }
    if (total && threadIdx.x == 0) *total = carry;
    if (segs.n_rows && threadIdx.x == 0) segs.put(carry);
}
void launch_scan_u32_pair(hipStream_t st, const u32* in0, u32* out0, const u32* in1, u32* out1, int64_t n, u32* tmp) {
    if (n > 0 && n <= SCAN_ONE) {
        hipLaunchKernelGGL(scan_one_kernel, dim3(2), dim3(1024), 0, st, ScanPair{{in0, in1}, {out0, out1}}, n, (u32*)nullptr, SegTotal());
        return;
    }
    launch_scan_u32(st, in0, out0, n, tmp, nullptr);
    launch_scan_u32(st, in1, out1, n, tmp, nullptr);
}

size_t scan_tmp_words(int64_t n) {
    size_t w = 0;
    while (true) {
        int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
        if (nb < 1) nb = 1;
        w += (size_t)((nb + 63) / 64 * 64);
        if (nb <= 1) break;
        n = nb;
    }
    return w + 64;
}

static void launch_scan(hipStream_t st, const u32* in, u32* out, int64_t n, u32* tmp, u32* total, const SegTotal& segs) {
    if (n <= SCAN_ONE) {
        hipLaunchKernelGGL(scan_one_kernel, dim3(1), dim3(1024), 0, st, ScanPair{{in, nullptr}, {out, nullptr}}, n, total, segs);
        return;
    }
    const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    hipLaunchKernelGGL(scan_block_kernel, dim3((unsigned)nb), dim3(SCAN_NT), 0, st, in, out, n, tmp);
    u32* next = tmp + (nb + 63) / 64 * 64;
    launch_scan(st, tmp, tmp, nb, next, total, segs);
    hipLaunchKernelGGL(scan_add_kernel, dim3((unsigned)nb), dim3(SCAN_NT), 0, st, out, n, tmp);
}
void launch_scan_u32(hipStream_t st, const u32* in, u32* out, int64_t n, u32* tmp, u32* total) {
    if (n > 0) launch_scan(st, in, out, n, tmp, total, SegTotal());
    else if (total) launch_fill_u32(st, total, 1, 0);
}

// ------------------------------------------------------------------------------------------------
// per-(task, field) dictionaries: LDS sort of the support lookups, then the query join
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void bitonic_sort_lds(u64* keys, int n2) {
    for (int k = 2; k <= n2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int p = threadIdx.x; p < (n2 >> 1); p += blockDim.x) {
                const int i = ((p & ~(j - 1)) << 1) | (p & (j - 1));
                const int ixj = i + j;
                const bool asc = (i & k) == 0;
                const u64 a = keys[i], b = keys[ixj];
                if ((a > b) == asc) {
                    keys[i] = b;
                    keys[ixj] = a;
                }
            }
            __syncthreads();
        }
    }
}

__device__ __forceinline__ int load_tf_keys(u64* keys, int* sh_fill, const SetView& v, int F, int f, int64_t s_lo,
                                            int64_t s_hi, u32 fb) {
    if (threadIdx.x == 0) *sh_fill = 0;
    __syncthreads();
    const int ns = (int)(s_hi - s_lo);
    for (int s = threadIdx.x; s < ns; s += blockDim.x) {
        const int64_t bag = (s_lo + s) * F + f;
        const int64_t p0 = v.bag_offsets[bag];
        const int len = (int)(v.bag_offsets[bag + 1] - p0);
        if (len > 0) {
            const int base = atomicAdd(sh_fill, len);
            for (int j = 0; j < len; ++j)
                keys[base + j] = ((u64)(fb + (u32)v.indices[p0 + j]) << 32) | ((u64)s << 16) | (u64)j;
        }
    }
    __syncthreads();
    return *sh_fill;
}

// The same keys in (row, sample, position) order by a stable LSD radix sort inside LDS: the keys are written in
// (sample, position) order first (an exclusive scan of the bag lengths places every bag), so only the row bits
// have to be sorted, in passes of at most 8 bits.  Per pass every wave ranks a contiguous share of the keys, 64 at
// a time, with ballot matching (equal digits keep their order), and the per-(digit, wave) counts are turned into
// positions.  Returns the buffer (one of the two) that holds the result.  At most TFR_ROUNDS * 64 keys per wave
// and TFR_MAXS bags per task and set.
#define TFR_ROUNDS 16
#define TF_SMALL_N 1984    // lookups per set of a 'small' (task, field): its key buffer is 2048 + 64 keys
#define TF_SMALL_MS 512    // samples per set of a 'small' task
#define TFR_MAXS 2048
struct TfRadixLds {
    u64* buf;               // [cap]: every pass holds all keys in registers between its read and its write
    u32 *sbase, *sp0;       // [ms + 1], [ms]: first key / first lookup (relative to the wave's) of every bag
    uint16_t* cnt;          // [waves][256]
    u32* digstart;          // [256]
    int* sh_scan;
};
__device__ __forceinline__ u64* tf_radix_sorted(const TfRadixLds& L, const SetView& v, int F, int f, int64_t s_lo,
                                                int64_t s_hi, u32 fb, int bits, int n) {
    const int NT = blockDim.x, W = NT / WAVE, lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    const int ns = (int)(s_hi - s_lo);
    // bag lengths -> first key of every bag
    {
        const int per = (ns + NT - 1) / NT;
        const int b0 = min(ns, (int)threadIdx.x * per), b1 = min(ns, b0 + per);
        int sum = 0;
        for (int sidx = b0; sidx < b1; ++sidx) {
            const int64_t bag = (s_lo + sidx) * F + f;
            sum += (int)(v.bag_offsets[bag + 1] - v.bag_offsets[bag]);
        }
        int total;
        int run = block_excl_scan(sum, L.sh_scan, &total);
        for (int sidx = b0; sidx < b1; ++sidx) {
            const int64_t bag = (s_lo + sidx) * F + f;
            const int64_t p0 = v.bag_offsets[bag];
            L.sbase[sidx] = (u32)run;
            L.sp0[sidx] = (u32)(p0 - v.lookup0);
            run += (int)(v.bag_offsets[bag + 1] - p0);
        }
        if (threadIdx.x == 0) L.sbase[ns] = (u32)n;
    }
    __syncthreads();
    // Every thread builds a run of consecutive keys: one bisection for the bag of its first key, then a walk along the
    // bag table; the index loads of the run are all requested before the first key is assembled.
    {
        const int C = (n + NT - 1) / NT;   // at most TFR_ROUNDS + 1
        const int e0 = min(n, (int)threadIdx.x * C), e1 = min(n, e0 + C);
        int lo = 0;
        if (e0 < e1) {
            int hi = ns;   // last bag whose first key is <= e0 (empty bags share their successor's first key)
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (L.sbase[mid] <= (u32)e0) lo = mid;
                else hi = mid;
            }
        }
        u32 meta[TFR_ROUNDS + 1], idx[TFR_ROUNDS + 1];
#pragma unroll
        for (int q = 0; q < TFR_ROUNDS + 1; ++q) {
            const int e = e0 + q;
            if (e < e1) {
                while (L.sbase[lo + 1] <= (u32)e) ++lo;   // (the table ends with n: the walk stops)
                const u32 j = (u32)e - L.sbase[lo];
                meta[q] = ((u32)lo << 16) | j;
                idx[q] = (u32)v.indices[v.lookup0 + L.sp0[lo] + j];
            }
        }
#pragma unroll
        for (int q = 0; q < TFR_ROUNDS + 1; ++q)
            if (e0 + q < e1) L.buf[e0 + q] = ((u64)(fb + idx[q]) << 32) | (u64)meta[q];
    }
    const int passes = (bits + 7) / 8 > 0 ? (bits + 7) / 8 : 1;
    const int width = (bits + passes - 1) / passes > 0 ? (bits + passes - 1) / passes : 1;
    const int NB = 1 << width;
    const int chunk = ((n + W * WAVE - 1) / (W * WAVE)) * WAVE;   // keys per wave, a multiple of 64
    const int rounds = chunk / WAVE;
    const u64 lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    u64* const in = L.buf;
    u64* const out = L.buf;   // in place: the barriers between ranking and placing separate the last read from the first write
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = pass * width;
        for (int i = threadIdx.x; i < W * NB; i += NT) L.cnt[i] = 0;
        __syncthreads();   // also: the keys of the previous step are in place
        u64 key[TFR_ROUNDS];
        u32 rank[TFR_ROUNDS];
        const int w_end = min(n, (wv + 1) * chunk);
#pragma unroll
        for (int r = 0; r < TFR_ROUNDS; ++r) {
            if (r < rounds) {
                const int i = wv * chunk + r * WAVE + lane;
                const bool valid = i < w_end;
                key[r] = valid ? in[i] : ~0ull;
                const u32 d = (((u32)(key[r] >> 32) - fb) >> shift) & (u32)(NB - 1);
                u64 peers = __ballot(valid);
                for (int b = 0; b < width; ++b) {
                    const bool bit = (d >> b) & 1u;
                    const u64 m = __ballot(bit);
                    peers &= bit ? m : ~m;
                }
                const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : lane;
                u32 old = 0;
                if (valid && lane == leader) {
                    old = L.cnt[wv * NB + d];
                    L.cnt[wv * NB + d] = (uint16_t)(old + (u32)__popcll(peers));
                }
                old = __shfl(old, leader, WAVE);
                rank[r] = old + (u32)__popcll(peers & lt_mask);
            }
        }
        __syncthreads();
        u32 total = 0;
        if ((int)threadIdx.x < NB) {
            for (int ww = 0; ww < W; ++ww) {
                const u32 cc = L.cnt[ww * NB + threadIdx.x];
                L.cnt[ww * NB + threadIdx.x] = (uint16_t)total;
                total += cc;
            }
        }
        int tile_count;
        const int ds = block_excl_scan((int)total, L.sh_scan, &tile_count);
        if ((int)threadIdx.x < NB) L.digstart[threadIdx.x] = (u32)ds;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < TFR_ROUNDS; ++r) {
            if (r < rounds) {
                const int i = wv * chunk + r * WAVE + lane;
                if (i < w_end) {
                    const u32 d = (((u32)(key[r] >> 32) - fb) >> shift) & (u32)(NB - 1);
                    out[L.digstart[d] + L.cnt[wv * NB + d] + rank[r]] = key[r];
                }
            }
        }
        __syncthreads();   // every wave has placed its keys and is done with the counters
    }
    return L.buf;
}

// cap: key capacity of an LDS buffer (bitonic: a power of two); ms: most samples a task has in one set (radix)
// cls: 0 = every (task, field); 1 = only the small ones (at most small_n lookups and small_ms samples per set);
// 2 = only the others.  A launch is sized for its largest (task, field): with very uneven tasks the small ones get a
// launch of their own, with workgroups and LDS that let several share a compute unit.
template <bool LDS_UNIQ, bool RADIX>
__global__ void tf_sort_kernel(TfSortArgs a, int cap, int ms, int cls, int small_n, int small_ms) {
    extern __shared__ u64 sh_dyn[];  // bitonic: keys [cap] (+ u32 uniq[cap]); radix: two key buffers, uniq, bag tables, counters
    __shared__ int sh_scan[20];
    __shared__ int sh_fill;
    __shared__ u32 sh_digstart[256];
    u64* sh_keys = sh_dyn;
    TfRadixLds L;
    if (RADIX) {
        L.buf = sh_dyn;
        u32* w32 = reinterpret_cast<u32*>(sh_dyn + cap) + (LDS_UNIQ ? cap : 0);
        L.sbase = w32;
        L.sp0 = w32 + (ms + 1);
        L.cnt = reinterpret_cast<uint16_t*>(w32 + 2 * ms + 2);
        L.digstart = sh_digstart;
        L.sh_scan = sh_scan;
    }
    const int f = blockIdx.x, t = blockIdx.y;
    const size_t tf = (size_t)t * a.F + f;
    const u32 fb = (u32)a.field_base[f];
    const u32 n = a.cnt_sup[tf], B = a.base_sup[tf];
    const u32 nq = a.cnt_qry[tf], Bq = a.base_qry[tf];
    if (cls) {
        const int64_t ns_ = a.sup.task_offsets[a.t0 + t + 1] - a.sup.task_offsets[a.t0 + t];
        const int64_t nq_ = a.qry.task_offsets[a.t0 + t + 1] - a.qry.task_offsets[a.t0 + t];
        const bool small = (int)max(n, nq) <= small_n && max(ns_, nq_) <= (int64_t)small_ms;
        if (small != (cls == 1)) return;
    }
    u32* uniq = LDS_UNIQ ? (u32*)(sh_dyn + cap) : (a.slot_rows + B);
    int bits = 1;
    while (((int64_t)1 << bits) < a.field_base[f + 1] - a.field_base[f]) ++bits;
    int n_unique = 0;

    // ---- phase A: support lookups sorted by (row, sample, position in bag)
    const int64_t s_lo = a.sup.task_offsets[a.t0 + t], s_hi = a.sup.task_offsets[a.t0 + t + 1];
    if (n > 0) {
        if (RADIX) {
            sh_keys = tf_radix_sorted(L, a.sup, a.F, f, s_lo, s_hi, fb, bits, (int)n);
        } else {
            load_tf_keys(sh_keys, &sh_fill, a.sup, a.F, f, s_lo, s_hi, fb);
            int n2 = 1;
            while (n2 < (int)n) n2 <<= 1;
            for (int i = n + threadIdx.x; i < n2; i += blockDim.x) sh_keys[i] = ~0ull;
            __syncthreads();
            bitonic_sort_lds(sh_keys, n2);
        }
        const int chunk = ((int)n + blockDim.x - 1) / blockDim.x;
        const int i0 = min((int)n, (int)threadIdx.x * chunk), i1 = min((int)n, i0 + chunk);
        int c = 0;
        // row of the key before this thread's range, read before any key is rewritten below
        const u32 row_before = i0 > 0 && i0 < (int)n ? (u32)(sh_keys[i0 - 1] >> 32) : ~0u;
        for (int i = i0; i < i1; ++i) c += (i == 0) || ((sh_keys[i] >> 32) != (sh_keys[i - 1] >> 32));
        int slot = block_excl_scan(c, sh_scan, &n_unique) - 1;
        // radix: the slot of every key replaces its row first, so that the second sweep below has independent
        // iterations and reads only LDS (the bag tables of the sort give every lookup's position)
        u32 prev = row_before;
        for (int i = i0; i < i1; ++i) {
            const u64 key = sh_keys[i];
            const u32 row = (u32)(key >> 32);
            const bool head = RADIX ? (i == 0 || row != prev) : ((i == 0) || (row != (u32)(sh_keys[i - 1] >> 32)));
            prev = row;
            if (head) {
                ++slot;
                a.slot_start[B + tf + slot] = (int32_t)(B + i);
                a.slot_rows[B + slot] = row;
                if (LDS_UNIQ) uniq[slot] = row;
            }
            if (RADIX) {
                sh_keys[i] = ((u64)(u32)slot << 32) | (key & 0xFFFFFFFFull);
            } else {
                const int s = (int)((key >> 16) & 0xFFFF), j = (int)(key & 0xFFFF);
                const int64_t p = a.sup.bag_offsets[(s_lo + s) * a.F + f] + j;
                a.sup_slot[p - a.sup.lookup0] = slot;
                a.sup_sorted[B + i] = make_int2(a.sup_rows[s_lo + s] - a.sup_row_base, slot);
            }
        }
        if (RADIX) {
            __syncthreads();
            const int prow0 = a.sup_rows[s_lo] - a.sup_row_base;   // rows of a task are consecutive
            for (int i = threadIdx.x; i < (int)n; i += blockDim.x) {
                const u64 key = sh_keys[i];
                const int s = (int)((key >> 16) & 0xFFFF), j = (int)(key & 0xFFFF);
                const int sl = (int)(key >> 32);
                a.sup_slot[L.sp0[s] + j] = sl;
                a.sup_sorted[B + i] = make_int2(prow0 + s, sl);
            }
        }
    }
    if (threadIdx.x == 0) {
        a.slot_start[B + tf + n_unique] = (int32_t)(B + n);
        a.n_slots[tf] = (u32)n_unique;
    }
    __threadfence_block();
    __syncthreads();

    // ---- phase B: query lookups sorted the same way, joined against the support rows
    if (nq == 0) {
        for (int u = threadIdx.x; u < n_unique; u += blockDim.x) {
            a.qseg_lo[B + u] = (int32_t)Bq;
            a.qseg_hi[B + u] = (int32_t)Bq;
        }
        return;
    }
    const int64_t q_lo = a.qry.task_offsets[a.t0 + t], q_hi = a.qry.task_offsets[a.t0 + t + 1];
    if (RADIX) {
        sh_keys = tf_radix_sorted(L, a.qry, a.F, f, q_lo, q_hi, fb, bits, (int)nq);
    } else {
        sh_keys = sh_dyn;
        load_tf_keys(sh_keys, &sh_fill, a.qry, a.F, f, q_lo, q_hi, fb);
        int n2 = 1;
        while (n2 < (int)nq) n2 <<= 1;
        for (int i = nq + threadIdx.x; i < n2; i += blockDim.x) sh_keys[i] = ~0ull;
        __syncthreads();
        bitonic_sort_lds(sh_keys, n2);
    }
    const int qprow0 = a.qry_rows[q_lo] - a.qry_row_base;
    for (int i = threadIdx.x; i < (int)nq; i += blockDim.x) {
        const u64 key = sh_keys[i];
        const u32 row = (u32)(key >> 32);
        int lo = 0, hi = n_unique;  // first slot with uniq >= row
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (uniq[mid] < row) lo = mid + 1;
            else hi = mid;
        }
        const int slot = (lo < n_unique && uniq[lo] == row) ? lo : -1;
        const int s = (int)((key >> 16) & 0xFFFF), j = (int)(key & 0xFFFF);
        if (RADIX) {
            a.qry_slot[L.sp0[s] + j] = slot;
            a.qry_sorted[Bq + i] = make_int2(qprow0 + s, slot);
        } else {
            const int64_t p = a.qry.bag_offsets[(q_lo + s) * a.F + f] + j;
            a.qry_slot[p - a.qry.lookup0] = slot;
            a.qry_sorted[Bq + i] = make_int2(a.qry_rows[q_lo + s] - a.qry_row_base, slot);
        }
    }
    for (int u = threadIdx.x; u < n_unique; u += blockDim.x) {
        const u64 klo = (u64)uniq[u] << 32, khi = ((u64)uniq[u] + 1) << 32;
        int lo = 0, hi = (int)nq;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sh_keys[mid] < klo) lo = mid + 1;
            else hi = mid;
        }
        int lo2 = lo, hi2 = (int)nq;
        while (lo2 < hi2) {
            const int mid = (lo2 + hi2) >> 1;
            if (sh_keys[mid] < khi) lo2 = mid + 1;
            else hi2 = mid;
        }
        a.qseg_lo[B + u] = (int32_t)(Bq + lo);
        a.qseg_hi[B + u] = (int32_t)(Bq + lo2);
    }
}

int tf_sort_max_cap() { return 16384; }

// max_tf: the largest number of lookups any (task, field) of the wave has in one set; max_set_rows: the largest
// number of samples any task of the wave has in one set
void launch_tf_sort(hipStream_t st, const TfSortArgs& a, int max_tf, int max_set_rows) {
    if (a.Tw <= 0 || a.F <= 0) return;
    dim3 grid(a.F, a.Tw);
    int cap = 1024;
    while (cap < max_tf) cap <<= 1;
    if (max_set_rows <= TFR_MAXS) {   // radix sort in LDS
        auto launch = [&](int mtf, int mrows, int cls, int small_n, int small_ms) {
            int cp = 1024;
            while (cp < mtf) cp <<= 1;
            const int kcap = (mtf + 63) / 64 * 64 + 64;                   // keys in the buffer
            const int ms = mrows > 0 ? mrows : 1;
            int nt = cp / 8;                                              // at most 8 rounds of 64 keys per wave while the block
            nt = nt < 256 ? 256 : (nt > 1024 ? 1024 : nt);                // allows (TFR_ROUNDS = 16 at the largest capacity)
            const size_t fixed = (size_t)(2 * ms + 2) * 4 + (size_t)(nt / WAVE) * 256 * 2;
            // the row list in LDS while two workgroups still fit a compute unit -- or when only one fits anyway
            const bool lds_uniq = (size_t)kcap * 12 + fixed <= 80 * 1024 ||
                                  ((size_t)kcap * 8 + fixed > 80 * 1024 && (size_t)kcap * 12 + fixed <= 158 * 1024);
            const size_t shmem = (size_t)kcap * 8 + (lds_uniq ? (size_t)kcap * 4 : 0) + fixed;
            if (lds_uniq) {
                hipFuncSetAttribute((const void*)tf_sort_kernel<true, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
                hipLaunchKernelGGL((tf_sort_kernel<true, true>), grid, dim3(nt), shmem, st, a, kcap, ms, cls, small_n, small_ms);
            } else {
                hipFuncSetAttribute((const void*)tf_sort_kernel<false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
                hipLaunchKernelGGL((tf_sort_kernel<false, true>), grid, dim3(nt), shmem, st, a, kcap, ms, cls, small_n, small_ms);
            }
        };
        // uneven tasks: the (task, field)s of at most TF_SMALL_N lookups and TF_SMALL_MS samples per set run in a launch
        // of their own (every workgroup of either launch checks its class first)
        if (max_tf > 2 * TF_SMALL_N && (int64_t)a.Tw * a.F >= 32) {
            launch(TF_SMALL_N, max_set_rows < TF_SMALL_MS ? max_set_rows : TF_SMALL_MS, 1, TF_SMALL_N, TF_SMALL_MS);
            launch(max_tf, max_set_rows, 2, TF_SMALL_N, TF_SMALL_MS);
        } else {
            launch(max_tf, max_set_rows, 0, 0, 0);
        }
        return;
    }
    const bool lds_uniq = cap <= 8192;
    const size_t shmem = (size_t)cap * (lds_uniq ? 12 : 8);
    const int nt = cap <= 1024 ? 256 : (cap <= 4096 ? 512 : 1024);
    if (lds_uniq) {
        hipFuncSetAttribute((const void*)tf_sort_kernel<true, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        hipLaunchKernelGGL((tf_sort_kernel<true, false>), grid, dim3(nt), shmem, st, a, cap, 0, 0, 0, 0);
    } else {
        hipFuncSetAttribute((const void*)tf_sort_kernel<false, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
        hipLaunchKernelGGL((tf_sort_kernel<false, false>), grid, dim3(nt), shmem, st, a, cap, 0, 0, 0, 0);
    }
}

// ------------------------------------------------------------------------------------------------
// global (field,row) ordering of all lookups: keys, stable LSD radix sort, segments
// ------------------------------------------------------------------------------------------------
// One workgroup per 256 consecutive bags: their lookups are one contiguous range, walked by all lanes with
// coalesced reads and writes; the bag of a lookup is found by bisection of the 257 staged offsets.
// The value of a lookup names its bag in the gradient buffer: (row of the sample) * F + field when enc.rshift is 0, else
// the bit fields row << rshift | field << pshift | position of the lookup in its bag (ValEnc).
__global__ __launch_bounds__(256) void build_keys_kernel(int F, const int64_t* field_base, const int64_t* bag_offsets,
                                                         const int32_t* indices, int64_t n_bags, int64_t lookup0,
                                                         const int32_t* __restrict__ row_map, u32 row0, ValEnc enc, u32* keys,
                                                         u32* vals) {
    __shared__ int64_t offs[257];
    const int64_t b0 = (int64_t)blockIdx.x * 256;
    const int nb = (int)min<int64_t>(256, n_bags - b0);
    for (int i = threadIdx.x; i <= nb; i += 256) offs[i] = bag_offsets[b0 + i];
    __syncthreads();
    const int64_t p0 = offs[0], p1 = offs[nb];
    for (int64_t p = p0 + threadIdx.x; p < p1; p += 256) {
        int lo = 0, hi = nb;   // last bag with offs[bag] <= p
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (offs[mid] <= p) lo = mid;
            else hi = mid;
        }
        const int64_t b = b0 + lo;
        const int f = (int)(b % F);
        const u32 row = row0 + (u32)row_map[b / F];   // row of the sample in the gradient buffer
        keys[p - lookup0] = (u32)field_base[f] + (u32)indices[p];
        vals[p - lookup0] = enc.rshift ? (row << enc.rshift) | ((u32)f << enc.pshift) | (u32)(p - offs[lo]) : row * (u32)F + (u32)f;
    }
}

// bag_offsets / row_map point at the first bag / sample of the range (a multiple of F bags); lookup0 is the range's first
// lookup: keys and vals are numbered from it
void launch_build_keys(hipStream_t st, int F, const int64_t* field_base, const int64_t* bag_offsets,
                       const int32_t* indices, int64_t n_bags, int64_t lookup0, const int32_t* row_map, u32 row0, ValEnc enc,
                       u32* keys, u32* vals) {
    if (n_bags <= 0) return;
    hipLaunchKernelGGL(build_keys_kernel, dim3((unsigned)((n_bags + 255) / 256)), dim3(256), 0, st, F, field_base,
                       bag_offsets, indices, n_bags, lookup0, row_map, row0, enc, keys, vals);
}

// ------------------------------------------------------------------------------------------------
// the same keys laid out field after field (support lookups of a field first, then its query lookups, each in input
// order): the field needs no sorting then -- every field's range is sorted by row alone, in fewer radix passes
// ------------------------------------------------------------------------------------------------
// One workgroup per field: fm_off_*[t * F + f] = lookups of field f in the tasks before t (per set), tot[f] / tot[F + f]
// = the field's support / query lookups in the wave.
__global__ __launch_bounds__(256) void field_offsets_kernel(int F, int Tw, const u32* cnt_s, const u32* cnt_q, u32* fm_off_s,
                                                            u32* fm_off_q, u32* tot) {
    __shared__ int sh[8];
    const int f = blockIdx.x;
    for (int set = 0; set < 2; ++set) {
        const u32* cnt = set ? cnt_q : cnt_s;
        u32* off = set ? fm_off_q : fm_off_s;
        u32 run = 0;
        for (int t0 = 0; t0 < Tw; t0 += 256) {
            const int t = t0 + threadIdx.x;
            const u32 c = t < Tw ? cnt[(size_t)t * F + f] : 0u;
            int total;
            const u32 ex = (u32)block_excl_scan((int)c, sh, &total);
            if (t < Tw) off[(size_t)t * F + f] = run + ex;
            run += (u32)total;
            __syncthreads();
        }
        if (threadIdx.x == 0) tot[set * F + f] = run;
    }
}

// first key and first tile of every field's range, and what a key of the field has in front of its row number
__global__ __launch_bounds__(256) void field_table_kernel(int F, const u32* tot, const int64_t* field_base, int tile_keys, u32* key_pos, u32* tile_base,
                                                          u32* key_sub) {
    __shared__ int sh[8];
    u32 k = 0, tl = 0;
    for (int f0 = 0; f0 <= F; f0 += 256) {   // (entry F: the ends)
        const int f = f0 + (int)threadIdx.x;
        const u32 nf = f < F ? tot[f] + tot[F + f] : 0u;
        int n_keys, n_tiles;
        const u32 kx = (u32)block_excl_scan((int)nf, sh, &n_keys);
        __syncthreads();
        const u32 tx = (u32)block_excl_scan((int)((nf + (u32)tile_keys - 1) / (u32)tile_keys), sh, &n_tiles);
        __syncthreads();
        if (f <= F) {
            key_pos[f] = k + kx;
            tile_base[f] = tl + tx;
            key_sub[f] = f < F ? (u32)field_base[f] : 0u;
        }
        k += (u32)n_keys;
        tl += (u32)n_tiles;
    }
}

// Few (task, field)s: the scans of their counts, the fields' offsets and their table by one workgroup instead of three launches that are
// mostly their latency (4.5 + 4.1 + 3.4 us for 32 of them, and what lies between).  Waves take a field each, a lane a task.  Beyond FP_TF
// counts they no longer fit the LDS, and there is work for several workgroups.
#define FP_TF 4096
#define FP_NT 1024
__global__ __launch_bounds__(FP_NT) void field_prepare_kernel(int F, int Tw, const u32* __restrict__ cnt_s, const u32* __restrict__ cnt_q, const int64_t* __restrict__ field_base,
                                                              int tile_keys, u32* base_s, u32* base_q, u32* fm_off_s, u32* fm_off_q, u32* key_pos, u32* tile_base, u32* key_sub, u32* tot) {
    __shared__ u32 cnt[2][FP_TF], sum[2][FP_TF];   // (F <= F * Tw)
    __shared__ int sh[FP_NT / WAVE + 2];
    constexpr int PER = FP_TF / FP_NT;
    const int TF = F * Tw, lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    for (int i = threadIdx.x; i < TF; i += FP_NT) {
        cnt[0][i] = cnt_s[i];
        cnt[1][i] = cnt_q[i];
    }
    __syncthreads();
    for (int set = 0; set < 2; ++set) {
        u32* const base = set ? base_q : base_s;
        u32 c[PER];
        u32 mine = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = (int)threadIdx.x * PER + k;
            c[k] = i < TF ? cnt[set][i] : 0u;
            mine += c[k];
        }
        int all;
        u32 run = (u32)block_excl_scan((int)mine, sh, &all);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = (int)threadIdx.x * PER + k;
            if (i < TF) base[i] = run;
            run += c[k];
        }
    }
    for (int i = wv; i < 2 * F; i += FP_NT / WAVE) {   // (field, set)
        const int set = i & 1, f = i >> 1;
        u32* const off = set ? fm_off_q : fm_off_s;
        u32 run = 0;
        for (int t0 = 0; t0 < Tw; t0 += WAVE) {
            const int t = t0 + lane;
            const u32 c = t < Tw ? cnt[set][t * F + f] : 0u;
            const u32 incl = (u32)wave_incl_scan((int)c);
            if (t < Tw) off[t * F + f] = run + incl - c;
            run += (u32)__shfl((int)incl, WAVE - 1, WAVE);
        }
        if (lane == 0) {
            sum[set][f] = run;
            tot[set * F + f] = run;
        }
    }
    __syncthreads();
    u32 k = 0, tl = 0;
    for (int f0 = 0; f0 <= F; f0 += FP_NT) {   // (entry F: the ends)
        const int f = f0 + (int)threadIdx.x;
        const u32 nf = f < F ? sum[0][f] + sum[1][f] : 0u;
        int n_keys, n_tiles;
        const u32 kx = (u32)block_excl_scan((int)nf, sh, &n_keys);
        __syncthreads();
        const u32 tx = (u32)block_excl_scan((int)((nf + (u32)tile_keys - 1) / (u32)tile_keys), sh, &n_tiles);
        __syncthreads();
        if (f <= F) {
            key_pos[f] = k + kx;
            tile_base[f] = tl + tx;
            key_sub[f] = f < F ? (u32)field_base[f] : 0u;
        }
        k += (u32)n_keys;
        tl += (u32)n_tiles;
    }
}

enum { RS_ITEMS = 8 };   // keys per thread of a radix tile
static int rs_tile_keys(int64_t n);

#define BKF_CH 1024     // bags of a task staged at a time
#define BKF_TILE 4096   // their lookups whose bags are written out at a time
#define BKF_BAG 64      // longest bag for which they are
// One workgroup per (field, task, set): the bags (sample, field) of the task, BKF_CH at a time -- their lengths are
// scanned into LDS, then every lane takes lookups of the piece in order (coalesced writes).
// Bound: memory, once a lookup's bag costs little.  SHORT: every bag writes its number to its lookups' places in LDS; a bag of
// thousands would keep its lane busy, so with longer ones a lookup finds its bag by bisection of the staged table, ten dependent LDS reads
// (72 million lookups 303 us, written out 270; 138 million of 64 fields 504 and 470; 3 million of three tasks 37 and 20).
template <bool SHORT>
__global__ __launch_bounds__(256) void build_keys_fm_kernel(FieldKeysArgs a) {
    __shared__ u32 sbase[BKF_CH + 1];
    __shared__ u32 sp0[BKF_CH], srow[BKF_CH];
    __shared__ uint16_t bag_of[SHORT ? BKF_TILE : 1];
    __shared__ int sh[8];
    // The fields of a task on one XCD: their bags lie side by side, and their offsets and indices share lines (dealt over all of them
    // 72 million lookups took 337 us instead of 303).
    const int per_xcd = (int)(gridDim.x >> 3);
    const int64_t id = (int64_t)blockIdx.z * gridDim.x + (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (id >= (int64_t)a.F * a.Tw) return;
    const int t = (int)(id / a.F), f = (int)(id - (int64_t)t * a.F), set = blockIdx.y;
    const SetView& v = set ? a.qry : a.sup;
    const size_t tf = (size_t)t * a.F + f;
    const u32 n_tf = (set ? a.cnt_q : a.cnt_s)[tf];
    if (n_tf == 0) return;
    const int64_t s_lo = v.task_offsets[a.t0 + t], s_hi = v.task_offsets[a.t0 + t + 1];
    const int32_t* prow = set ? a.prow_q : a.prow_s;
    const u32 row0 = set ? a.row0_q : a.row0_s;
    const u32 fb = (u32)a.field_base[f];
    size_t dest = (size_t)a.key_pos[f] + (set ? a.tot[f] : 0u) + (set ? a.fm_off_q : a.fm_off_s)[tf];
    for (int64_t c0 = s_lo; c0 < s_hi; c0 += BKF_CH) {
        const int nb = (int)min<int64_t>(BKF_CH, s_hi - c0);
        const int per = (nb + 255) >> 8;   // consecutive bags per thread, at most four
        const int b0 = (int)threadIdx.x * per;
        u32 len[4];
        __syncthreads();   // the table of the piece before has been read
        {
            u32 p0r[4];
            u32 sum = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                len[q] = 0; p0r[q] = 0;
                if (q < per && b0 + q < nb) {
                    const int64_t bag = (c0 + b0 + q) * a.F + f;
                    const int64_t p0 = v.bag_offsets[bag];
                    len[q] = (u32)(v.bag_offsets[bag + 1] - p0);
                    p0r[q] = (u32)(p0 - v.lookup0);
                    srow[b0 + q] = row0 + (u32)prow[c0 + b0 + q];
                }
                sum += len[q];
            }
            int total;
            u32 run = (u32)block_excl_scan((int)sum, sh, &total);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < per && b0 + q < nb) {
                    sbase[b0 + q] = run;
                    sp0[b0 + q] = p0r[q];
                    run += len[q];
                }
            if (threadIdx.x == 0) sbase[nb] = (u32)total;
        }
        __syncthreads();
        const u32 total = sbase[nb];
        for (u32 s0 = 0; s0 < total; s0 += SHORT ? (u32)BKF_TILE : total) {
            const u32 s1 = SHORT ? min(total, s0 + (u32)BKF_TILE) : total;
            if constexpr (SHORT) {
                if (s0 > 0) __syncthreads();   // the tile before has been read
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (len[q]) {
                        const u32 first = sbase[b0 + q], lo = max(first, s0), hi = min(first + len[q], s1);
                        for (u32 e = lo; e < hi; ++e) bag_of[e - s0] = (uint16_t)(b0 + q);
                    }
                __syncthreads();
            }
            for (u32 e0 = s0 + threadIdx.x; e0 < s1; e0 += 4 * 256) {
                int bag[4];
                u32 j[4], idx[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u32 e = e0 + q * 256;
                    bag[q] = 0; j[q] = 0; idx[q] = 0;
                    if (e < s1) {
                        int lo = 0;
                        if constexpr (SHORT) lo = bag_of[e - s0];
                        else {
                            int hi = nb;   // last bag whose first lookup is <= e (empty bags share their successor's)
                            while (hi - lo > 1) {
                                const int mid = (lo + hi) >> 1;
                                if (sbase[mid] <= e) lo = mid;
                                else hi = mid;
                            }
                        }
                        bag[q] = lo;
                        j[q] = e - sbase[lo];
                        idx[q] = (u32)v.indices[v.lookup0 + sp0[lo] + j[q]];
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u32 e = e0 + q * 256;
                    if (e < s1) {
                        a.keys[dest + e] = fb + idx[q];
                        a.vals[dest + e] = (srow[bag[q]] << a.enc.rshift) | ((u32)f << a.enc.pshift) | j[q];
                    }
                }
            }
        }
        dest += total;
    }
}

// tables: 3 (F + 1) words (key_pos, tile_base, key_sub), then 2 F words of totals
void launch_build_keys_by_field(hipStream_t st, FieldKeysArgs a, u32* tables, u32* scan_tmp, int64_t n, int max_bag) {
    if (a.F <= 0 || a.Tw <= 0) return;
    u32* key_pos = tables;
    u32* tile_base = key_pos + (a.F + 1);
    u32* key_sub = tile_base + (a.F + 1);
    u32* tot = key_sub + (a.F + 1);
    if ((int64_t)a.F * a.Tw <= FP_TF) {
        hipLaunchKernelGGL(field_prepare_kernel, dim3(1), dim3(FP_NT), 0, st, a.F, a.Tw, a.cnt_s, a.cnt_q, a.field_base, rs_tile_keys(n), a.base_s, a.base_q, a.fm_off_s,
                           a.fm_off_q, key_pos, tile_base, key_sub, tot);
    } else {
        launch_scan_u32_pair(st, a.cnt_s, a.base_s, a.cnt_q, a.base_q, (int64_t)a.F * a.Tw, scan_tmp);
        hipLaunchKernelGGL(field_offsets_kernel, dim3(a.F), dim3(256), 0, st, a.F, a.Tw, a.cnt_s, a.cnt_q, a.fm_off_s, a.fm_off_q, tot);
        hipLaunchKernelGGL(field_table_kernel, dim3(1), dim3(256), 0, st, a.F, tot, a.field_base, rs_tile_keys(n), key_pos, tile_base, key_sub);
    }
    a.key_pos = key_pos;
    a.tot = tot;
    const int64_t tf = ((int64_t)a.F * a.Tw + 7) / 8 * 8, nx = std::min<int64_t>(tf, 1 << 22);   // (a launch's threads along x stay below 2^32)
    const dim3 grid((unsigned)nx, 2, (unsigned)((tf + nx - 1) / nx));
    if (max_bag <= BKF_BAG) hipLaunchKernelGGL(build_keys_fm_kernel<true>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(build_keys_fm_kernel<false>, grid, dim3(256), 0, st, a);
}
SegTab field_seg_tab(int F, u32* tables) { return SegTab{F, tables + (F + 1), tables, tables + 2 * (F + 1)}; }
size_t field_table_words(int F) { return (size_t)5 * (F + 1); }

// Digits are BITS wide (8, or 9 where that saves a pass): 25-bit row keys sort in three 9-bit passes instead of four 8-bit ones.
// Bound: memory, if enough of it is under way.  All of a thread's RS_ITEMS keys (and their places in the output) are asked for
// before the first is used: asked for one by one, inside the conditions that guard the list's end, a scatter of 138 million pairs
// took 740 us and a digit count 267; now 525 and 143 (4.2 and 3.9 TB/s).
// Tiles are dealt to workgroups so that every XCD (workgroups are spread over the 8 XCDs round-robin) walks one
// contiguous range of tiles: the pieces that neighbouring tiles write into a digit's output range then meet in one L2.
__device__ __forceinline__ int rs_tile_of_block(int nblk) {
    const int per = (nblk + 7) >> 3;
    return (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
}

// What a pass sorts by: a digit of the key, or (BYTASK) a digit of the task that the value's sample belongs to --
// the stable pass that turns the (field, row) order of a wave's lookups into (task, field, row) order.
__device__ __forceinline__ u32 rs_task_of(const TaskOf& m, u32 val) {
    const u32 r = min(val >> m.rshift, m.n_rows - 1u);   // (every value names a row of the wave; the bound keeps any other inside the tables)
    // tasks of one size (a power of two of padded rows in both sets): the task is a shift of the row, no table read
    if (m.uniform_shift >= 0) return (r < m.n_sup_rows ? r : r - m.n_sup_rows) >> m.uniform_shift;
    return (u32)(r < m.n_sup_rows ? m.row_task_s[r] : m.row_task_q[r - m.n_sup_rows]);
}

// A pass may sort several independent ranges of the list at once (SegTab: the fields of a wave's lookups, each range
// holding one field's keys).  Tiles then never straddle two ranges: tile numbers run range after range, a range's
// share of the digit-count table is laid out [digit][tile of the range] behind the shares of the ranges before it, so
// that ONE exclusive scan over the whole table still yields every (range, digit, tile)'s place in the output; the
// digit is taken from the key minus the range's key base.  seg.n_seg == 0: one range, the whole list.
// FEW: few tiles.  The table is [tile][digit] and nobody scans it: every workgroup of the scatter adds up its range's counts itself,
// beside its first loads (the scan was a launch of one workgroup, RS_FEW_TILES).  OWN: so few that it counts the range's other tiles
// itself, too, and there is no table (RS_OWN_TILES).
enum { RS_SCAN, RS_FEW, RS_OWN };
struct RsTile {
    int64_t k0, k1;      // keys of the tile
    u32 key_base;        // subtracted from a key before its digit is taken
    size_t h0;           // count-table index of (digit 0, this tile)
    size_t hstride;      // ... and the distance between digits
    int64_t pos0, pos1;  // the range's keys,
    int t0, nt;          // first tile and number of tiles
    bool any;
};
template <int TILE, bool FEW>
__device__ __forceinline__ RsTile rs_tile(const SegTab& seg, int tile, int nblk, int64_t n, int nb) {
    RsTile t;
    if (seg.n_seg == 0) {
        t.k0 = (int64_t)tile * TILE;
        t.k1 = min(n, t.k0 + TILE);
        t.key_base = 0u;
        t.h0 = FEW ? (size_t)tile * nb : (size_t)tile;
        t.hstride = FEW ? 1 : (size_t)nblk;
        t.pos0 = 0;
        t.pos1 = n;
        t.t0 = 0;
        t.nt = nblk;
        t.any = tile < nblk;
        return t;
    }
    int lo = 0, hi = seg.n_seg;   // last range whose first tile is <= tile
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (seg.tile_base[mid] <= (u32)tile) lo = mid;
        else hi = mid;
    }
    const u32 tb = seg.tile_base[lo], te = seg.tile_base[lo + 1];
    t.any = (u32)tile < te;       // (tiles past the last range's: nothing to do)
    t.k0 = (int64_t)seg.key_base_pos[lo] + (int64_t)((u32)tile - tb) * TILE;
    t.k1 = min((int64_t)seg.key_base_pos[lo + 1], t.k0 + TILE);
    t.key_base = seg.key_sub[lo];
    t.hstride = FEW ? 1 : (size_t)(te - tb);
    t.h0 = FEW ? (size_t)tile * nb : (size_t)nb * tb + ((u32)tile - tb);
    t.pos0 = (int64_t)seg.key_base_pos[lo];
    t.pos1 = (int64_t)seg.key_base_pos[lo + 1];
    t.t0 = (int)tb;
    t.nt = (int)(te - tb);
    return t;
}

template <int BITS, bool BYTASK, int NT, bool FEW>
__global__ __launch_bounds__(NT) void radix_hist_kernel(const u32* src, int64_t n, int shift, u32* hist, int nblk, TaskOf tk, SegTab seg) {
    constexpr int NB = 1 << BITS;
    __shared__ u32 h[NB];
    const int tile = rs_tile_of_block(nblk);
    if (tile >= nblk) return;
    const RsTile T = rs_tile<NT * RS_ITEMS, FEW>(seg, tile, nblk, n, NB);
    if (!T.any) return;
    for (int i = threadIdx.x; i < NB; i += NT) h[i] = 0;
    __syncthreads();
    const int64_t base = T.k0;
    const int64_t n_end = T.k1;
    const int lane = threadIdx.x & (WAVE - 1);
    u32 item[RS_ITEMS];   // (all of a thread's items are asked for before the first is looked at; past the tile its last one)
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) item[i] = src[min(base + i * NT + (int64_t)threadIdx.x, n_end - 1)];
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        const int64_t idx = base + i * NT + threadIdx.x;
        // One atomic per run of equal digits in the wave instead of one per lane.  By task: inside a row the lookups
        // are in input order, i.e. by task, so a hot row gives long runs of one digit, which as one atomic per lane
        // would all queue on one counter.  By key: from the second pass on the keys of a hot row lie next to each
        // other (they share every digit sorted so far), and LDS atomics retire about one lane per cycle.
        const bool valid = idx < n_end;
        u32 d = 0xFFFFFFFFu;
        if (valid) d = ((BYTASK ? rs_task_of(tk, item[i]) : item[i] - T.key_base) >> shift) & (NB - 1);
        const u32 dp = __shfl_up(d, 1, WAVE);
        const u64 heads = __ballot(lane == 0 || d != dp);
        if (valid && (lane == 0 || d != dp)) {
            const u64 later = lane == 63 ? 0ull : (heads >> (lane + 1));   // heads after this lane
            const int run = later ? __ffsll((unsigned long long)later) : 64 - lane;
            atomicAdd(&h[d], (u32)run);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < NB; i += NT) hist[T.h0 + (size_t)i * T.hstride] = h[i];
}

// Stable scatter: every wave owns a contiguous 1/4 of the tile and ranks its keys round by round (64
// consecutive keys per round) with ballot matching, so equal digits keep their input order.
template <int BITS, bool BYTASK, int NT, int MODE>
__global__ __launch_bounds__(NT) void radix_scatter_kernel(const u32* kin, const u32* vin, u32* kout, u32* vout, const u32* gofs,
                                     int64_t n_all, int shift, int nblk, TaskOf tk, SegTab seg) {
    constexpr int NB = 1 << BITS, DPT = NB > NT ? NB / NT : 1;   // digits per thread in the per-digit phase
    constexpr int TILE = NT * RS_ITEMS, WAVES = NT / WAVE;
    constexpr bool FEW = MODE != RS_SCAN, OWN = MODE == RS_OWN;
    __shared__ u32 others[OWN ? 2 : 1][OWN ? NB : 1];   // keys of a digit in the range's tiles before this one, after it
    __shared__ __attribute__((aligned(16))) uint16_t cnt[WAVES][NB];   // (cleared four bytes at a time)
    __shared__ u32 digstart[NB];
    __shared__ u32 skeys[TILE];
    __shared__ u32 svals[TILE];
    __shared__ uint16_t sdig[BYTASK ? TILE : 1];   // the digit of every staged pair (a key names its own)
    __shared__ int sh_scan[WAVES + 2];
    __shared__ u32 place[FEW ? NB : 1];            // where the tile's keys of a digit go
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const int tile = rs_tile_of_block(nblk);
    if (tile >= nblk) return;
    const RsTile T = rs_tile<TILE, FEW>(seg, tile, nblk, n_all, NB);
    if (!T.any) return;
    for (int i = threadIdx.x; i < WAVES * NB / 2; i += NT) reinterpret_cast<u32*>(&cnt[0][0])[i] = 0;
    __syncthreads();
    const int64_t tile0 = T.k0, n = T.k1;
    u32 key[RS_ITEMS], val[RS_ITEMS], rank[RS_ITEMS], dig[RS_ITEMS];
    const u64 lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {   // (as above)
        const int64_t idx = min(tile0 + (int64_t)w * (WAVE * RS_ITEMS) + r * WAVE + lane, n - 1);
        key[r] = kin[idx];
        val[r] = vin[idx];
    }
    u32 before[DPT], all[DPT];   // FEW: keys of a thread's digits in the range's tiles before this one, in all of them
    static_assert(!FEW || NB >= NT, "a thread's digits lie next to each other");
    if constexpr (OWN) {
        for (int i = threadIdx.x; i < 2 * NB; i += NT) others[i / NB][i % NB] = 0;
        __syncthreads();
        for (int64_t k0 = T.pos0; k0 < T.pos1; k0 += TILE) {
            if (k0 == tile0) continue;
            u32 item[RS_ITEMS];
#pragma unroll
            for (int i = 0; i < RS_ITEMS; ++i) item[i] = (BYTASK ? vin : kin)[min(k0 + i * NT + (int64_t)threadIdx.x, T.pos1 - 1)];
#pragma unroll
            for (int i = 0; i < RS_ITEMS; ++i)
                if (k0 + i * NT + (int64_t)threadIdx.x < T.pos1)
                    atomicAdd(&others[k0 > tile0][((BYTASK ? rs_task_of(tk, item[i]) : item[i] - T.key_base) >> shift) & (NB - 1)], 1u);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < DPT; ++k) {   // (.. and this one's, below)
            before[k] = others[0][threadIdx.x * DPT + k];
            all[k] = before[k] + others[1][threadIdx.x * DPT + k];
        }
    } else if constexpr (FEW) {
#pragma unroll
        for (int k = 0; k < DPT; ++k) before[k] = all[k] = 0;
        for (int t0 = 0; t0 < T.nt; t0 += 8) {
            u32 c[8][DPT];
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int k = 0; k < DPT; ++k) c[u][k] = gofs[(size_t)(T.t0 + min(t0 + u, T.nt - 1)) * NB + threadIdx.x * DPT + k];
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int k = 0; k < DPT; ++k) {
                    if (t0 + u < T.nt) all[k] += c[u][k];
                    if (T.t0 + t0 + u < tile) before[k] += c[u][k];
                }
        }
    }
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const bool valid = tile0 + (int64_t)w * (WAVE * RS_ITEMS) + r * WAVE + lane < n;
        const u32 d = ((BYTASK ? (valid ? rs_task_of(tk, val[r]) : 0u) : key[r] - T.key_base) >> shift) & (NB - 1);
        dig[r] = d;
        u64 peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < BITS; ++b) {
            const bool bit = (d >> b) & 1u;
            const u64 m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : lane;
        u32 old = 0;
        if (valid && lane == leader) {
            old = cnt[w][d];
            cnt[w][d] = (uint16_t)(old + (u32)__popcll(peers));
        }
        old = __shfl(old, leader, WAVE);
        rank[r] = old + (u32)__popcll(peers & lt_mask);   // (a wave's counters are its own: no barrier between rounds)
    }
    __syncthreads();
    // per digit: exclusive prefix over the waves, block total, start of each digit inside the tile
    u32 total[DPT];
    u32 mine = 0;
#pragma unroll
    for (int k = 0; k < DPT; ++k) {
        const int d = threadIdx.x * DPT + k;
        total[k] = 0;
        if (NB < NT && d >= NB) continue;
        u32 t = 0;
#pragma unroll
        for (int ww = 0; ww < WAVES; ++ww) {
            const u32 c = cnt[ww][d];
            cnt[ww][d] = (uint16_t)t;
            t += c;
        }
        total[k] = t;
        if (OWN) all[k] += t;
        mine += t;
    }
    int tile_count;
    u32 ds = (u32)block_excl_scan((int)mine, sh_scan, &tile_count);
    if constexpr (FEW) {
        u32 sum = 0;
        int ignored;
#pragma unroll
        for (int k = 0; k < DPT; ++k) sum += all[k];
        __syncthreads();   // (the scan's scratch is used again)
        u32 at = (u32)T.pos0 + (u32)block_excl_scan((int)sum, sh_scan, &ignored);
#pragma unroll
        for (int k = 0; k < DPT; ++k) {
            place[threadIdx.x * DPT + k] = at + before[k];
            at += all[k];
        }
    }
#pragma unroll
    for (int k = 0; k < DPT; ++k) {
        const int d = threadIdx.x * DPT + k;
        if (NB >= NT || d < NB) digstart[d] = ds;
        ds += total[k];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int64_t idx = tile0 + (int64_t)w * (WAVE * RS_ITEMS) + r * WAVE + lane;
        if (idx < n) {
            const u32 d = dig[r];
            const u32 pos = digstart[d] + cnt[w][d] + rank[r];
            skeys[pos] = key[r];
            svals[pos] = val[r];
            if (BYTASK) sdig[pos] = (uint16_t)d;
        }
    }
    __syncthreads();
    u32 at[RS_ITEMS];
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        const int pos = min(i * NT + (int)threadIdx.x, tile_count - 1);
        key[i] = skeys[pos];
        val[i] = svals[pos];
        const u32 d = BYTASK ? (u32)sdig[pos] : ((key[i] - T.key_base) >> shift) & (NB - 1);
        at[i] = (FEW ? place[d] : gofs[T.h0 + (size_t)d * T.hstride]) - digstart[d];
    }
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        const int pos = i * NT + threadIdx.x;
        if (pos < tile_count) {
            kout[(size_t)(at[i] + (u32)pos)] = key[i];
            vout[(size_t)(at[i] + (u32)pos)] = val[i];
        }
    }
}

// Lists of a million and more are cut into tiles of 512 threads: a digit's run in a tile is twice as long, the count table half
// as large.  138 million lookups, three passes of 8 bits and one by task, 256 and 512 threads: 3.2 / 2.9 ms.  (Two passes of 10
// bits instead of the three take 2.05 ms against 2.0, and a table of twice the size.)
static bool rs_long(int64_t n) { return n >= (int64_t)1 << 20; }
static int rs_tile_keys(int64_t n) { return (rs_long(n) ? 512 : 256) * RS_ITEMS; }
// extra_tiles: tiles beyond ceil(n / tile) that a pass over several ranges may need (one per range)
size_t radix_hist_words(int64_t n, int extra_tiles) {
    const int64_t nblk = (n + 256 * RS_ITEMS - 1) / (256 * RS_ITEMS) + extra_tiles;   // (never fewer than a pass has)
    return (size_t)(512 * nblk + 64) + scan_tmp_words(512 * nblk);
}

// Up to RS_FEW_TILES tiles (ranges' tiles are counted one by one, so few of them lie in one range) the scatter's workgroups add up
// the digit counts themselves: a pass is two launches instead of three or five.  Whole steps with the scan's launches and without:
// 2,048 lookups 389 / 377 us, 134,000 of 11 fields 486 / 467, 461,000 of 20 fields (245 tiles) 590 / 573, 614,000 of 40 fields (340)
// 804 / 796, 899,000 of 26 fields (465) 853 / 856: from there on what the workgroups read again outweighs a launch.
#define RS_FEW_TILES 384
// Up to RS_OWN_TILES of them the digit counts' launch goes, too: 4,096 lookups 335 / 324 us a step, 12,000 343 / 332, 25,000 (13 tiles) no difference.
#define RS_OWN_TILES 8
template <int BITS, bool BYTASK, int NT, int MODE>
static void radix_pass_nt(hipStream_t st, const u32* ki, const u32* vi, u32* ko, u32* vo, int64_t n, int shift, u32* hist, int nblk,
                          const TaskOf& tk, const SegTab& seg) {
    u32* scan_tmp = hist + ((size_t)512 * nblk + 63) / 64 * 64;
    const dim3 grid((nblk + 7) / 8 * 8);
    if (MODE != RS_OWN)
        hipLaunchKernelGGL((radix_hist_kernel<BITS, BYTASK, NT, MODE == RS_FEW>), grid, dim3(NT), 0, st, BYTASK ? vi : ki, n, shift, hist, nblk, tk, seg);
    if (MODE == RS_SCAN) launch_scan_u32(st, hist, hist, (int64_t)(1 << BITS) * nblk, scan_tmp, nullptr);
    hipLaunchKernelGGL((radix_scatter_kernel<BITS, BYTASK, NT, MODE>), grid, dim3(NT), 0, st, ki, vi, ko, vo, hist, n, shift, nblk, tk, seg);
}
template <bool BYTASK, int NT, int MODE>
static void radix_pass_width(hipStream_t st, int width, const u32* ki, const u32* vi, u32* ko, u32* vo, int64_t n, int shift, u32* hist,
                             int nblk, const TaskOf& tk, const SegTab& seg) {
    if (width <= 8) radix_pass_nt<8, BYTASK, NT, MODE>(st, ki, vi, ko, vo, n, shift, hist, nblk, tk, seg);
    else radix_pass_nt<9, BYTASK, NT, MODE>(st, ki, vi, ko, vo, n, shift, hist, nblk, tk, seg);
}
template <bool BYTASK>
static void radix_pass(hipStream_t st, int width, const u32* ki, const u32* vi, u32* ko, u32* vo, int64_t n, int shift, u32* hist,
                       const TaskOf& tk, const SegTab& seg) {
    // ranges: at most one partly filled tile per range beyond the tiles of the whole list (the tiles past the last range's
    // write nothing into the count table: what the table holds there stands behind every count and moves none's place)
    const int tile = rs_tile_keys(n), nblk = (int)((n + tile - 1) / tile) + seg.n_seg;
    if (rs_long(n)) radix_pass_width<BYTASK, 512, RS_SCAN>(st, width, ki, vi, ko, vo, n, shift, hist, nblk, tk, seg);
    else if (n <= RS_OWN_TILES * tile) radix_pass_width<BYTASK, 256, RS_OWN>(st, width, ki, vi, ko, vo, n, shift, hist, nblk, tk, seg);
    else if (nblk <= RS_FEW_TILES) radix_pass_width<BYTASK, 256, RS_FEW>(st, width, ki, vi, ko, vo, n, shift, hist, nblk, tk, seg);
    else radix_pass_width<BYTASK, 256, RS_SCAN>(st, width, ki, vi, ko, vo, n, shift, hist, nblk, tk, seg);
}

// Returns the number of passes made: after an odd number the result is in (keys_tmp, vals_tmp).
int launch_radix_sort(hipStream_t st, u32* keys, u32* vals, u32* keys_tmp, u32* vals_tmp, int64_t n, int bits,
                      u32* hist, const SegTab* seg_in) {
    if (n <= 0) return 0;
    const SegTab seg = seg_in ? *seg_in : SegTab{0, nullptr, nullptr, nullptr};
    if (bits < 1) bits = 1;
    if (bits > 32) bits = 32;
    const int passes = (bits + 8) / 9, width = (bits + passes - 1) / passes;
    const TaskOf none{nullptr, nullptr, 0u, 0u, 0, -1};
    u32 *ki = keys, *vi = vals, *ko = keys_tmp, *vo = vals_tmp;
    for (int p = 0; p < passes; ++p) {
        radix_pass<false>(st, width, ki, vi, ko, vo, n, width * p, hist, none, seg);
        u32* t = ki; ki = ko; ko = t;
        t = vi; vi = vo; vo = t;
    }
    return passes;
}

// The pairs of (keys, vals), which are in (field, row) order, stably re-ordered by the task of their sample: the result
// is in (task, field, row) order, support lookups before query lookups inside a row, each in input order.  One pass
// for up to 512 tasks into (out_keys, out_vals); two passes of at most 8 bits beyond that, the first into
// (mid_keys, mid_vals).  The input is left as it is.
void launch_task_sort(hipStream_t st, const u32* keys, const u32* vals, u32* mid_keys, u32* mid_vals, u32* out_keys,
                      u32* out_vals, int64_t n, int n_tasks, const TaskOf& tk, u32* hist) {
    if (n <= 0) return;
    int bits = 1;
    while ((1 << bits) < n_tasks) ++bits;
    const SegTab one{0, nullptr, nullptr, nullptr};
    if (bits <= 9) {
        radix_pass<true>(st, bits, keys, vals, out_keys, out_vals, n, 0, hist, tk, one);
    } else {   // (the second pass masks with 8 bits: bits <= 16)
        radix_pass<true>(st, 8, keys, vals, mid_keys, mid_vals, n, 0, hist, tk, one);
        radix_pass<true>(st, 8, mid_keys, mid_vals, out_keys, out_vals, n, 8, hist, tk, one);
    }
}
int task_sort_passes(int n_tasks) { return n_tasks > 512 ? 2 : 1; }

// ------------------------------------------------------------------------------------------------
// per-(task, field) dictionaries and overlap join read off the (task, field, row) order of the wave's lookups
// ------------------------------------------------------------------------------------------------
// One workgroup per (task, field): its lookups are one contiguous run of the ordered list, support lookups before
// query lookups inside every row.  The run is walked NT * E entries at a time, a wave's as E rounds of 64 neighbours:
// what an entry needs from before it -- how many support lookups, how many distinct support rows, and the slot of the row it belongs to
// (none when the support set does not look the row up) -- are bit counts of the round's ballots, sums of the rounds before and one
// exchange of the waves' totals a piece.  Writes exactly what tf_sort_kernel writes, for (task, field)s of any size.
// Bound: memory, if neighbouring entries' stores fall into the same lines and the next piece is asked for ahead.  With four
// consecutive entries a thread, two block-wide scans and four barriers a piece 72 million lookups took 432 us, 138 million 754; now 317 and
// 650.  A few long runs (3 tasks x 64 fields of 17,000 entries) are walked by 1024 threads: 57 -> 35 us; short ones a round at a time (37 tasks x
// 11 fields of 330 entries: four rounds 13 us, one 7.4).
template <int NT, int E, bool SLOTS>
__global__ __launch_bounds__(NT) void tf_join_kernel(TfJoinArgs a) {
    constexpr int NW = NT / WAVE, SPAN = WAVE * E, PIECE = NT * E;
    __shared__ u32 sh_count[2][NW], sh_state[2][NW];   // a wave's support lookups and distinct support rows (16 bits each); state after it
    const int f = blockIdx.x, t = blockIdx.y;
    const size_t tf = (size_t)t * a.F + f;
    const u32 ns = a.cnt_s[tf], nq = a.cnt_q[tf], B = a.base_s[tf], Bq = a.base_q[tf];
    const u32 n = ns + nq;
    const u32* K = a.keys + ((size_t)B + Bq);
    const u32* V = a.vals + ((size_t)B + Bq);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u64 lt = (1ull << lane) - 1ull, le = lt | (1ull << lane);
    const u32 posmask = (1u << a.pshift) - 1u;
    u32 a_carry = 0, u_carry = 0, st_carry = 0;   // the same on every thread
    u32 kn[E + 2], vn[E + 1];   // of the next piece: kn[0] the entry before the wave's first, [1..E] the rounds' own, [E + 1] / vn[E] the entry after its last
    auto request = [&](u32 c0) {
        const u32 w0 = c0 + wv * SPAN;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const u32 i = min(w0 + e * 64 + lane, n - 1u);
            kn[e + 1] = K[i];
            vn[e] = V[i];
        }
        kn[0] = K[min(max(w0, 1u) - 1u, n - 1u)];   // (one address for the wave)
        kn[E + 1] = K[min(w0 + (u32)SPAN, n - 1u)];
        vn[E] = V[min(w0 + (u32)SPAN, n - 1u)];
    };
    if (n > 0) request(0);
    int buf = 0;
    for (u32 c0 = 0; c0 < n; c0 += PIECE, buf ^= 1) {
        const u32 w0 = c0 + wv * SPAN;
        u32 k[E + 2], v[E + 1];
#pragma unroll
        for (int e = 0; e < E + 2; ++e) k[e] = kn[e];
#pragma unroll
        for (int e = 0; e < E + 1; ++e) v[e] = vn[e];
        if (c0 + PIECE < n) request(c0 + PIECE);
        u64 bs[E], bh[E];   // support lookups, first entries of a row
        u32 nk[E];          // the key after each entry
        bool nsup[E];       // and whether it is a support lookup
        u32 n_sup = 0, n_sh = 0, state = 0x80000000u;   // (none yet: the state from before the wave goes on)
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const u32 i = w0 + e * 64 + lane;
            const bool in = i < n;
            u32 pk = __shfl_up(k[e + 1], 1, 64);
            const u32 last = e == 0 ? k[0] : (u32)__builtin_amdgcn_readlane((int)k[e], 63);
            if (lane == 0) pk = last;
            bs[e] = __ballot(in && (v[e] >> a.rshift) < a.n_sup_rows);
            bh[e] = __ballot(in && (i == 0 || pk != k[e + 1]));
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            nk[e] = __shfl_down(k[e + 1], 1, 64);
            const u32 next = e == E - 1 ? k[E + 1] : (u32)__builtin_amdgcn_readlane((int)k[e + 2], 0);
            if (lane == 63) nk[e] = next;
            const bool after = e == E - 1 ? (v[E] >> a.rshift) < a.n_sup_rows : (bs[e + 1 < E ? e + 1 : e] & 1ull) != 0;
            nsup[e] = lane == 63 ? after : ((bs[e] >> 1) >> lane) & 1ull;
            n_sup += (u32)__popcll(bs[e]);
            n_sh += (u32)__popcll(bs[e] & bh[e]);
            if (bh[e]) state = (bs[e] >> (63 - __clzll((long long)bh[e]))) & 1ull ? n_sh : 0x40000000u;
        }
        if (lane == 0) {
            sh_count[buf][wv] = n_sup | (n_sh << 16);
            sh_state[buf][wv] = state;
        }
        __syncthreads();   // (the other buffer is the next piece's)
        u32 ab = a_carry, ub = u_carry, st = st_carry;   // before the wave
#pragma unroll
        for (int w = 0; w < NW; ++w) {   // (all waves: the piece's end is carried)
            if (w == wv) { ab = a_carry; ub = u_carry; st = st_carry; }
            const u32 cw = sh_count[buf][w], sw = sh_state[buf][w];
            if (!(sw & 0x80000000u)) st_carry = sw & 0x40000000u ? 0u : u_carry + sw;   // slot + 1 of the last row begun, 0: not a support row
            a_carry += cw & 0xFFFFu;
            u_carry += cw >> 16;
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const u32 i = w0 + e * 64 + lane;
            const u64 hs = bs[e] & bh[e], seen = bh[e] & le;
            const u32 aex = ab + (u32)__popcll(bs[e] & lt);
            u32 mine = st;
            if (seen) mine = (bs[e] >> (63 - __clzll((long long)seen))) & 1ull ? ub + (u32)__popcll(hs & le) : 0u;
            if (i < n) {
                const u32 key = k[e + 1], val = v[e];
                const u32 row = val >> a.rshift;
                const bool sup = (bs[e] >> lane) & 1ull, head = (bh[e] >> lane) & 1ull;
                const bool next_same = i + 1 < n && nk[e] == key;
                const int32_t slot = (int32_t)mine - 1;
                // (every index below is in range when the list is in the stated order; the checks keep a list that is
                //  not -- a defect elsewhere -- from writing outside the (task, field)'s own ranges)
                if (sup) {
                    if (slot >= 0 && (u32)slot < ns && aex < ns) {
                        a.sup_sorted[B + aex] = make_int2((int)row, slot);
                        if (head) {
                            a.slot_rows[B + slot] = key;
                            a.slot_start[B + tf + slot] = (int32_t)(B + aex);
                        }
                        if (!(next_same && nsup[e])) a.qseg_lo[B + slot] = (int32_t)(Bq + (i - aex));
                        if (SLOTS) {
                            const int rel = (int)row - a.row_off_s[t];
                            if (rel >= 0 && rel < a.real_off_s[t + 1] - a.real_off_s[t]) {
                                const int64_t lk = a.bag_s[(a.sample0_s + a.real_off_s[t] + rel) * a.F + f] - a.lookup0_s + (val & posmask);
                                if (lk >= 0 && lk < a.n_lookups_s) a.sup_slot[lk] = slot;
                            }
                        }
                    }
                } else if (i - aex < nq) {
                    const u32 rq = row - a.n_sup_rows;
                    a.qry_sorted[Bq + (i - aex)] = make_int2((int)rq, slot);
                    if (SLOTS) {
                        const int rel = (int)rq - a.row_off_q[t];
                        if (rel >= 0 && rel < a.real_off_q[t + 1] - a.real_off_q[t]) {
                            const int64_t lk = a.bag_q[(a.sample0_q + a.real_off_q[t] + rel) * a.F + f] - a.lookup0_q + (val & posmask);
                            if (lk >= 0 && lk < a.n_lookups_q) a.qry_slot[lk] = slot;
                        }
                    }
                }
                if (!next_same && slot >= 0 && (u32)slot < ns) a.qseg_hi[B + slot] = (int32_t)(Bq + (i + 1) - (aex + (sup ? 1u : 0u)));
            }
            if (bh[e]) st = (bs[e] >> (63 - __clzll((long long)bh[e]))) & 1ull ? ub + (u32)__popcll(hs) : 0u;
            ab += (u32)__popcll(bs[e]);
            ub += (u32)__popcll(hs);
        }
    }
    if (threadIdx.x == 0) {
        const u32 nu = min(u_carry, ns);
        a.n_slots[tf] = nu;
        a.slot_start[B + tf + nu] = (int32_t)(B + ns);
    }
}

void launch_tf_join(hipStream_t st, const TfJoinArgs& a) {
    if (a.Tw <= 0 || a.F <= 0) return;
    const int64_t runs = (int64_t)a.F * a.Tw, n = a.n_lookups_s + a.n_lookups_q;
    const dim3 grid(a.F, a.Tw);
#define TF_JOIN(NT_, E_)                                                                                             \
    do {                                                                                                             \
        if (a.sup_slot) hipLaunchKernelGGL((tf_join_kernel<NT_, E_, true>), grid, dim3(NT_), 0, st, a);              \
        else hipLaunchKernelGGL((tf_join_kernel<NT_, E_, false>), grid, dim3(NT_), 0, st, a);                        \
    } while (0)
    if (n <= runs * 512) TF_JOIN(256, 1);
    else if (runs <= 1024 && n > runs * 1024) TF_JOIN(1024, 4);   // (fewer workgroups than the chip holds, with several pieces each)
    else TF_JOIN(256, 4);
#undef TF_JOIN
}

// Segments (runs of equal keys) that begin in front of every chunk of `ch` keys (16, 32 or 64): all that the segment reduction
// needs to number them, which also writes the row list.  Bound: the keys read once.  A scan of every key's head flag, then a kernel that
// wrote rows and starts from it, took 520 us for 72 million keys and 125 for 18 million; this 95 and 25.
__device__ __forceinline__ u32 seg_heads(const u32* __restrict__ keys, int64_t base, int64_t n) {   // of the 8 keys from base (a multiple of 8) on; by all lanes of a wave
    const int lane = threadIdx.x & (WAVE - 1);
    u32 k[9];
    if (base + 8 <= n) {   // (the buffers are 16-byte aligned)
        const uint4 a = *reinterpret_cast<const uint4*>(keys + base), b = *reinterpret_cast<const uint4*>(keys + base + 4);
        k[1] = a.x; k[2] = a.y; k[3] = a.z; k[4] = a.w; k[5] = b.x; k[6] = b.y; k[7] = b.z; k[8] = b.w;
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) k[i + 1] = base + i < n ? keys[base + i] : 0u;
    }
    k[0] = __shfl_up(k[8], 1, WAVE);
    if (lane == 0) k[0] = base > 0 && base < n ? keys[base - 1] : 0u;
    u32 c = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) c += base + i < n && (base + i == 0 || k[i + 1] != k[i]) ? 1u : 0u;
    return c;
}
__global__ __launch_bounds__(256) void seg_count_kernel(const u32* __restrict__ keys, int64_t n, int ch, u32* counts) {
    const int64_t base = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
    u32 c = seg_heads(keys, base, n);
    for (int d = 1; d < ch / 8; d *= 2) c += __shfl_xor(c, d, WAVE);
    if (base < n && base % ch == 0) counts[base / ch] = c;
}
// Short lists: one workgroup counts and scans, 8192 keys at a time.
#define SEG_ONE 32768
__global__ __launch_bounds__(1024) void seg_scan_one_kernel(const u32* __restrict__ keys, int64_t n, int ch, u32* out, SegTotal segs) {
    __shared__ int sh[1024 / WAVE + 2];
    u32 carry = 0;
    for (int64_t b0 = 0; b0 < n; b0 += 8192) {
        const int64_t base = b0 + (int64_t)threadIdx.x * 8;
        int all;
        const u32 before = carry + (u32)block_excl_scan((int)seg_heads(keys, base, n), sh, &all);
        if (base < n && base % ch == 0) out[base / ch] = before;
        carry += (u32)all;
        __syncthreads();   // the scan's scratch is used again
    }
    if (threadIdx.x == 0) segs.put(carry);
}

// the segments themselves, a key per thread: row and first position
__global__ __launch_bounds__(256) void seg_emit_kernel(const u32* __restrict__ keys, int64_t n, int ch, const u32* __restrict__ scan, int64_t* emb_rows, u32* seg_start,
                                                       const int64_t* n_rows, int64_t capacity) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool head = i < n && (i == 0 || keys[i] != keys[i - 1]);
    const u64 heads = __ballot(head);
    if (i >= n) return;
    const int lane = threadIdx.x & (WAVE - 1), first = lane / ch * ch;   // the chunk's first lane
    const int64_t seg = (int64_t)scan[i / ch] + __popcll((heads >> first) & ((1ull << (lane - first)) - 1ull));
    if (head && seg < capacity) {
        if (emb_rows) emb_rows[seg] = (int64_t)keys[i];
        seg_start[seg] = (u32)i;
    }
    if (i == n - 1 && *n_rows <= capacity) seg_start[*n_rows] = (u32)n;
}

__global__ void seg_counts_kernel(const u32* seg_start, const int64_t* n_rows, int64_t capacity, int64_t* counts) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = min(*n_rows, capacity);
    if (i < n) counts[i] = (int64_t)seg_start[i + 1] - (int64_t)seg_start[i];
}

__global__ void zero_rows_kernel(int64_t* n_rows_out, u32* status) {
    *n_rows_out = 0;
    status[ST_NROWS] = 0;
}

void launch_segments(hipStream_t st, const u32* sorted_keys, int64_t n, int ch, u32* chunk_scan, u32* scan_tmp,
                     int64_t* emb_rows, u32* seg_start, int64_t* seg_counts, int64_t capacity,
                     int64_t* n_rows_out, u32* status) {
    if (n <= 0) {
        hipLaunchKernelGGL(zero_rows_kernel, dim3(1), dim3(1), 0, st, n_rows_out, status);
        return;
    }
    SegTotal segs;
    segs.n_rows = n_rows_out;
    segs.capacity = capacity;
    segs.status = status;
    if (n <= SEG_ONE) {
        hipLaunchKernelGGL(seg_scan_one_kernel, dim3(1), dim3(1024), 0, st, sorted_keys, n, ch, chunk_scan, segs);
    } else {
        hipLaunchKernelGGL(seg_count_kernel, dim3((unsigned)((n + 2047) / 2048)), dim3(256), 0, st, sorted_keys, n, ch, chunk_scan);
        launch_scan(st, chunk_scan, chunk_scan, (n + ch - 1) / ch, scan_tmp, nullptr, segs);
    }
    if (!emb_rows && !seg_counts) return;
    hipLaunchKernelGGL(seg_emit_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, sorted_keys, n, ch, chunk_scan, emb_rows, seg_start,
                       n_rows_out, capacity);
    const int64_t m = capacity < n ? capacity : n;
    if (seg_counts && m > 0) hipLaunchKernelGGL(seg_counts_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, seg_start, n_rows_out, capacity, seg_counts);
}

// ------------------------------------------------------------------------------------------------
__global__ void zero_kernel(ZeroJobs z) {
    u32* p = z.p[blockIdx.y];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < z.words[blockIdx.y]; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0u;
}
void launch_zero(hipStream_t st, const ZeroJobs& z) {
    int64_t most = 0;
    for (int i = 0; i < z.n; ++i) most = std::max(most, z.words[i]);
    if (most <= 0) return;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)std::min<int64_t>((most + 255) / 256, 4096), z.n), dim3(256), 0, st, z);
}
__global__ void zero_pad_rows_kernel(PadJobs z) {
    const int g = blockIdx.x, set = z.set[blockIdx.y], bytes = z.row_bytes[blockIdx.y];
    const int n_real = z.real[set][g + 1] - z.real[set][g], r0 = z.off[set][g] + n_real, n_pad = z.off[set][g + 1] - r0;
    uint4* p = reinterpret_cast<uint4*>(z.p[blockIdx.y] + (int64_t)r0 * bytes);
    const int n = n_pad * (bytes / 16);
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = make_uint4(0u, 0u, 0u, 0u);
}
void launch_zero_pad_rows(hipStream_t st, int G, const PadJobs& z) {
    if (G <= 0 || z.n <= 0) return;
    hipLaunchKernelGGL(zero_pad_rows_kernel, dim3(G, z.n), dim3(256), 0, st, z);
}
__global__ void fill_u32_kernel(u32* p, int64_t n, u32 v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
void launch_fill_u32(hipStream_t st, u32* p, int64_t n, u32 v) {
    if (n <= 0) return;
    int64_t nb = (n + 255) / 256;
    if (nb > 65536) nb = 65536;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)nb), dim3(256), 0, st, p, n, v);
}
void launch_fill_f32(hipStream_t st, float* p, int64_t n, float v) {
    launch_fill_u32(st, (u32*)p, n, __builtin_bit_cast(u32, v));
}
