// Host side of the library: the C ABI of include/gmeta.h and the orchestration of one MAML step
// (G-Meta Alg. 1 with "worker" read as "task") as a fixed sequence of kernel launches on one stream.
//
// Data layout in HBM (per wave of tasks; a wave is as many tasks as the workspace holds):
//   activations  [rows, ld]   rows = samples of the wave, each task's rows padded to a multiple of
//                             `row_pad` (1 for fp32, 8 for bf16); ld = width rounded up to 32
//   theta        [Tw, n_theta] fp32, per task once adapted; layer l at offW[l] ([ld_{l-1}, ld_l],
//                             zero padded) and offb[l]
//   bf16 mode    every GEMM operand also lives as bf16, once, in the orientation it is produced in
//                (activations and deltas [rows, ld], weights [ld_{l-1}, ld_l]); the GEMMs read an operand
//                whose contraction index is the slow one through LDS
//   row arithmetic: no row table in HBM; per (task, field) either byte matrices of pair counts or sorted
//                {row, slot} lists (see pairhop_kernels.hip / twohop_kernels.hip)
#include <algorithm>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../../include/gmeta.h"
#include "gm_internal.h"

struct Arena {
    char* base = nullptr;
    size_t cap = 0, off = 0;
    bool overflow = false;
    template <typename T>
    T* get(size_t n) {
        const size_t bytes = (n * sizeof(T) + 255) / 256 * 256;
        if (off + bytes > cap) {
            overflow = true;
            off += bytes;
            return nullptr;
        }
        T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
        off += bytes;
        return p;
    }
};

struct ProfEntry {
    int64_t launches = 0;
    double ms = 0, bytes = 0, flops = 0;
};
struct ProfPending {
    std::string name;
    hipEvent_t e0, e1;
    double bytes, flops;
};

struct gm_ctx {
    int F = 0, D = 0, n_dense = 0, L = 0, mlp_dtype = 0;
    std::vector<int64_t> rows, field_base;
    std::vector<int> dims, ld;
    std::vector<int64_t> offW, offb;    // fp32 theta layout
    std::vector<int64_t> offWb;         // bf16 theta layout: W_l as stored ([d_in, d_out]), l = 1..L-1
    int64_t n_theta = 0, n_theta_b = 0;
    int FD = 0, row_pad = 1;
    int device = 0;
    hipStream_t stream = nullptr;
    char* ws = nullptr;
    size_t ws_bytes = 0;
    size_t persistent = 0;
    int64_t* d_field_base = nullptr;
    u32* d_status = nullptr;
    u32* d_status_side = nullptr;   // status words of the work on the side stream
    // The ordering of the lookups by row depends on the indices only: it runs on a stream of its own beside the dense
    // computation (same priority) and is joined before the segment reduction.
    hipStream_t side = nullptr;
    hipEvent_t ev_side = nullptr, ev_main = nullptr, ev_go = nullptr;
    // The pair-count matrices depend on the indices only and are first read by the first row hop: counting them on the
    // side stream lets the prefetch and the first forward / backward pass (bound by memory traffic) run beside a kernel
    // that is bound by latency and instruction issue.
    hipEvent_t ev_pairs_go = nullptr, ev_pairs = nullptr;
    int overlap_pairs = 0;
    int overlap_sort = 0;   // measured: 1-1.5 % (both streams contend for the same memory system), so off unless asked for
    std::string err;
    int pair_tile_rows = 0;
    int adapt_rows = 1;   // 0: the inner loop adapts the dense parameters only (embedding rows are read, not updated)
    int gemm_tile_n = 0;
    int wgrad_wide = 1;      // weight gradients over runs of tasks in 256 x 256 tiles where the shape allows
    int chain_factors = 0;   // the second-order chain's direction on a task's hidden layers: 0 by size, 1 matrices, 2 factors where they can be (see factor_rows)
    int theta_from_meta = 1; // bf16, several inner steps: a step's weights from theta and all steps' gradients, in first order where tasks are small
    int coarse_groups = 0;   // runs of tasks for the products only summed over tasks (0: chosen by shape)
    int n_cus = 256;
    int row_path = 0;   // task-local row arithmetic: 0 = choose per wave, 1 = sparse two-hop kernel, 2 = pair-count matrices
    int sort_fields = 1; // with index_path's row order: 1 = the keys are laid out field after field and every field's range sorted by row alone (fewer radix passes), 0 = one sort on (field, row)
    int index_path = 0; // per-(task, field) dictionaries: 0 = choose per wave, 1 = sorted per (task, field) in LDS, 2 = read off the wave's (task, field, row) order
    int max_wave_tasks = 0;   // 0: as many tasks per wave as the workspace holds
    char* static_scratch = nullptr;   // this device's copy of the static scratch array (gm_meta_step_static)
    // optional kernel timing
    bool prof_on = false;
    std::vector<ProfPending> prof_pending;
    std::vector<hipEvent_t> prof_free;
    std::map<std::string, ProfEntry> prof;
    std::string prof_text;
};

// Scratch of gm_meta_step_static: one array per GPU, part of the loaded code object (held until the process ends).
// Host code never passes the array's name to a kernel: the device address is looked up once per device at gm_create
// (hipGetSymbolAddress) and only that pointer is used.
#define GM_STATIC_SCRATCH_BYTES ((size_t)GM_STATIC_SCRATCH_MIB << 20)
static __device__ __align__(256) unsigned char scratch[GM_STATIC_SCRATCH_BYTES];
enum { GM_MAX_DEVICES = 64 };
static char* g_scratch_ptr[GM_MAX_DEVICES];   // device address of `scratch` on each GPU (null: not looked up yet)

static int fail(gm_ctx* c, int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (c) c->err = buf;
    return code;
}

#define HIPCHK(c, call)                                                                            \
    do {                                                                                           \
        hipError_t e_ = (call);                                                                    \
        if (e_ != hipSuccess) return fail(c, GM_ERR_HIP, "%s: %s", #call, hipGetErrorString(e_)); \
    } while (0)

// Brackets the launches issued during its lifetime with two events on the context's stream.
struct Prof {
    gm_ctx* c;
    ProfPending p;
    bool on;
    hipStream_t st;
    Prof(gm_ctx* c_, const char* name, double bytes, double flops, hipStream_t st_ = nullptr, bool use_st = false)
        : c(c_), on(c_->prof_on), st(use_st ? st_ : c_->stream) {
        if (!on) return;
        p.name = name;
        p.bytes = bytes;
        p.flops = flops;
        for (hipEvent_t* e : {&p.e0, &p.e1}) {
            if (!c->prof_free.empty()) {
                *e = c->prof_free.back();
                c->prof_free.pop_back();
            } else if (hipEventCreate(e) != hipSuccess) {
                on = false;
                return;
            }
        }
        (void)hipEventRecord(p.e0, st);
    }
    ~Prof() {
        if (!on) return;
        (void)hipEventRecord(p.e1, st);
        c->prof_pending.push_back(p);
    }
};

static void prof_drain(gm_ctx* c) {  // after the stream has been synchronised
    for (ProfPending& p : c->prof_pending) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, p.e0, p.e1) == hipSuccess) {
            ProfEntry& e = c->prof[p.name];
            e.launches += 1;
            e.ms += ms;
            e.bytes += p.bytes;
            e.flops += p.flops;
        }
        c->prof_free.push_back(p.e0);
        c->prof_free.push_back(p.e1);
    }
    c->prof_pending.clear();
}

static void zero_bf16(hipStream_t st, bf16_t* p, int64_t n) { launch_fill_u32(st, reinterpret_cast<u32*>(p), (n + 1) / 2, 0u); }

static int round_up(int x, int m) { return (x + m - 1) / m * m; }
static int64_t round_up64(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

static int model_layout(gm_ctx* c, const gm_model_desc* m) {
    if (!m || m->n_fields < 0 || m->n_layers < 1 || !m->layer_dims || (m->n_fields > 0 && !m->rows_per_field))
        return fail(c, GM_ERR_ARG, "bad model description");
    const int D = m->emb_dim;
    if (D < 4 || D > 256 || (D & (D - 1))) return fail(c, GM_ERR_ARG, "emb_dim must be a power of two in 4..256");
    if (m->mlp_dtype != 0 && m->mlp_dtype != 1) return fail(c, GM_ERR_ARG, "mlp_dtype must be 0 or 1");
    c->F = m->n_fields;
    c->D = D;
    c->n_dense = m->n_dense;
    c->L = m->n_layers;
    c->mlp_dtype = m->mlp_dtype;
    c->row_pad = m->mlp_dtype ? 8 : 1;
    c->FD = c->F * D;
    c->rows.assign(m->rows_per_field, m->rows_per_field + c->F);
    c->field_base.assign(c->F + 1, 0);
    for (int f = 0; f < c->F; ++f) {
        if (c->rows[f] <= 0) return fail(c, GM_ERR_ARG, "rows_per_field must be positive");
        c->field_base[f + 1] = c->field_base[f] + c->rows[f];
    }
    if (c->field_base[c->F] >= (int64_t)1 << 32) return fail(c, GM_ERR_ARG, "more than 2^32 rows in total");
    c->dims.assign(m->layer_dims, m->layer_dims + c->L + 1);
    if (c->n_dense < 0 || c->dims[0] != c->FD + c->n_dense || c->dims[c->L] != 1)
        return fail(c, GM_ERR_ARG, "layer_dims must start at F*D+n_dense and end at 1");
    c->ld.resize(c->L + 1);
    for (int l = 0; l <= c->L; ++l) {
        if (c->dims[l] <= 0) return fail(c, GM_ERR_ARG, "layer_dims must be positive");
        if (c->dims[l] > MAX_WIDTH) return fail(c, GM_ERR_ARG, "a layer of %d columns: at most %d", c->dims[l], (int)MAX_WIDTH);
        c->ld[l] = l == c->L ? 1 : round_up(c->dims[l], 32);
    }
    c->offW.assign(c->L + 1, 0);
    c->offb.assign(c->L + 1, 0);
    c->offWb.assign(c->L + 1, 0);
    int64_t o = 0, ob = 0;
    for (int l = 1; l <= c->L; ++l) {
        c->offW[l] = o;
        o += round_up64((int64_t)c->ld[l - 1] * c->ld[l], 32);
        c->offb[l] = o;
        o += round_up(c->ld[l], 32);
        if (l < c->L) {
            c->offWb[l] = ob;
            ob += (int64_t)c->ld[l - 1] * c->ld[l];
        }
    }
    c->n_theta = o;
    c->n_theta_b = std::max<int64_t>(ob, 32);
    return GM_OK;
}

// ------------------------------------------------------------------------------------------------
// handles
// ------------------------------------------------------------------------------------------------
struct Act {  // one activation-shaped buffer [rows, ld] in the type(s) the GEMMs read
    float* f = nullptr;    // fp32 mode
    bf16_t* b = nullptr;   // bf16 mode: [rows, ld]
    int ld = 0;
};
// The second-order chain's direction on the hidden layers' weights, for small tasks, as what it is made of: c * P^T Q of some
// passes over the task's rows, P a pass's inputs of the layer and Q its deltas.  X * V is then the sum of c * (X P^T) Q, two thin
// products contracted over the task's rows (the first kept as two bf16 parts, 16 significant bits; V itself would be rounded
// to 8), and no task's direction is written, rounded, read or summed: with a few dozen rows a task that traffic was half a step.
// (The weights theta' themselves stay matrices: their bf16 rounding decides ReLU gates.)
struct Factor {
    const Act* X;                       // P of layer 1 (null: none)
    const std::vector<Act>*A, *D;       // P of layer l > 1: A[l - 1]; Q: D[l]
    bool query;                         // whose rows
    float c;
};
struct FactorRoom {                     // where the thin products' results go
    bf16_t* S = nullptr;                // slots of [rows, 2 * ld], upper and lower parts
    int64_t slot = 0;
    int ld = 0;
    const int32_t *rows_s = nullptr, *rows_q = nullptr;
    int most_s = 0, most_q = 0;         // rows of the largest task
};
struct Theta {  // parameters as the GEMMs read them; stride 0 = shared by all tasks
    float* f = nullptr;
    int64_t sf = 0;
    bf16_t* b = nullptr;
    int64_t sb = 0;
    const std::vector<Factor>* fac = nullptr;   // the hidden layers' weights as factors (b is null)
};

struct StepState {  // what one inner step leaves behind for the second-order pass
    Act X;
    std::vector<Act> A, Dl;  // [1..L-1]
    float *dL = nullptr, *zL = nullptr;
    Theta th;                // parameters the step was taken at (GEMM operands)
    const float* wL = nullptr;  // last-layer weights of the step, fp32
    int64_t wL_stride = 0;
    float* wL_copy = nullptr;   // bf16 mode: copy of the last-layer weights (the master is updated in place)
};

// buffers of one sort + segment reduction of (row key, gradient-buffer slot) pairs
struct SortBufs {
    u32 *keys = nullptr, *vals = nullptr, *keys_tmp = nullptr, *vals_tmp = nullptr, *hist = nullptr, *scan_tmp = nullptr,
        *seg_start = nullptr;
    float* seg_partial = nullptr;
};

// Most tasks of a wave: they are one grid dimension of several kernels (the column sums put them in y), and the hops' work
// lists and the pass by task keep a task's number in 16 bits.
enum { MAX_WAVE_TASKS = 32768 };
static int most_wave_tasks(const gm_ctx* c) { return c->max_wave_tasks > 0 ? std::min<int>(c->max_wave_tasks, MAX_WAVE_TASKS) : MAX_WAVE_TASKS; }
enum { COARSE_GROUPS = 32 };   // most runs of tasks (gm_configure "coarse_groups" says how many are used)

static int most_runs(const gm_ctx* c, int Tw, int64_t rows);

struct WaveBufs {
    int32_t *row_off_s, *row_off_q, *real_off_s, *real_off_q;
    int32_t *row_task_s, *row_task_q;
    int32_t *tile_g_s, *tile_m_s, *tile_g_q, *tile_m_q;
    u32 *cnt_s, *base_s, *cnt_q, *base_q, *n_slots, *scan_tmp;
    u32* slot_rows;
    int32_t *slot_start, *sup_slot, *qry_slot, *qseg_lo, *qseg_hi;
    int2 *sup_sorted, *qry_sorted;
    u32 *fm_off_s = nullptr, *fm_off_q = nullptr, *field_tab = nullptr;   // keys laid out field after field: places and ranges
    u32 *tmid_keys = nullptr, *tmid_vals = nullptr;   // more than 512 tasks: the first of the two passes that order the lookups by task
    bool slots_written = true;   // sup_slot / qry_slot hold the slot of every lookup (only the sparse row kernel reads them)
    float *Xs0, *Xq0, *TXf, *dX, *loss_q;
    float* dX_kept = nullptr;   // (query_sum 3 without a chain: the second step's, see Spare)
    Theta v;  // direction / query gradient w.r.t. theta'
    // the last weight-gradient products of a call are only ever summed over the tasks: they are taken over COARSE_GROUPS
    // runs of consecutive tasks instead (row offsets of the runs, one sum per run)
    int32_t *coarse_off_s, *coarse_off_q;
    Theta vsum;
    Act Xs_scratch;
    std::vector<StepState> steps;
    std::vector<Theta> thetas;
    Act Xq;
    std::vector<Act> Aq, Dq;
    float *dLq, *zq;
    Act TX;
    std::vector<Act> TA, TD;
    // factors: what every step of the second-order chain leaves (TX, TA, TD of step k are TXk[k], ..)
    std::vector<Act> TXk;
    std::vector<std::vector<Act>> TAk, TDk;
    FactorRoom room;
    float* tdL;
    // pair-count matrices of the wave (null when the sparse kernel does the row arithmetic)
    uint8_t* pair_mat;
    u32 *pair_off_ss, *pair_off_qs, *pair_off_sq;
    int32_t *hop_small = nullptr, *hop_tiles[3] = {nullptr, nullptr, nullptr};   // the hops' work lists (HopPlan)
    int hop_longest[3] = {0, 0, 0}, hop_run = 1, n_hop_small = 0;
    int32_t* count_order = nullptr;   // the tasks whose pairs are counted, by falling size
    std::vector<int> count_rows;      // their sizes: samples of the larger set
    u32* task_path;   // [Tw] 1: pair-count path, 0: sparse kernel (the counting kernel clears it on overflow)
    // table-shaped sparse output only: the wave's own gradient buffer (support rows, then query rows) and sort
    float* GX = nullptr;
    int64_t* n_rows = nullptr;
    SortBufs so;
};

struct WaveDims {
    int Tw;
    int64_t Ss, Sq, Ps, Pq, nnz_s, nnz_q;  // real samples, padded rows, lookups
    int mt_s, mt_q;
    bool pair = false;                     // some task of the wave takes the pair-count path (matrices are allocated)
    bool any_sparse = false;               // some task of the wave takes the sparse kernel
    bool pair_ss = false, pair_sq = false; // which kinds besides query x support
    int64_t pair_bytes = 0;
    bool mat_apart = false;                // the matrices' room belongs to the dense side (gm_meta_train: one batch's at a time)
    int64_t hop_tiles_s = 0, hop_tiles_q = 0;   // tiles of 256 rows of the tasks beyond HOP_SMALL (the hops' work lists)
    bool table = false;                    // the sparse gradient is reduced wave by wave into a table-shaped output
    int query_sum = 0;                     // > 1: so many steps' input gradients are kept, and the query set's row update is taken once, from their sum
    bool from_meta = false;                // an inner step's weights are written from the meta parameters and all steps' gradients so far
    int factor_ld = 0;                     // > 0: the chain's direction stays factors (see Factor); rows of the largest task of the batch
};
struct FirstOrder { bool grads, acts; };   // what a call without a chain keeps of its inner steps: input gradients (query_sum 3), activations (from_meta)
static int query_sum(const gm_ctx* c, int K);
static bool theta_from_meta(const gm_ctx* c, int64_t T, int64_t n_support, int K, int order);
static FirstOrder first_order_keeps(const gm_ctx* c, int64_t T, int64_t n_support, int64_t Ps, int64_t Pq, int K);
static int factor_slots(int K) { return 2 * K - 1; }   // most factors of the direction: the query pass's, two of every later step

// Without a chain the steps' activations and input gradients are dead once the outer pass begins, and until then nothing touches three
// stretches that the call has anyway: the query set's activations and deltas, its rows of the gradient buffer and the per-task query
// gradient.  What the steps of such a call keep beyond one step's activations goes there (first_order_keeps).
struct Spare {
    Arena part[3];
    Arena* beyond;   // for what does not fit there
    template <typename T>
    T* get(size_t n) {
        for (Arena& p : part) {
            Arena a = p;
            T* const got = a.get<T>(n);
            if (!a.overflow) { p = a; return got; }
        }
        return beyond->get<T>(n);
    }
};
template <typename Mem>   // Arena or Spare
static Act alloc_act(const gm_ctx* c, Mem& ar, int64_t rows, int ld) {
    Act a;
    a.ld = ld;
    if (c->mlp_dtype == 0) {
        a.f = ar.template get<float>(rows * ld);
    } else {
        a.b = ar.template get<bf16_t>(rows * ld + 8);
    }
    return a;
}
// hidden layers' activations and deltas of a step, and its last layer's
template <typename Mem>
static void alloc_step(const gm_ctx* c, Mem& ar, StepState& s, int64_t rows) {
    s.A.assign(c->L, Act());
    s.Dl.assign(c->L, Act());
    for (int l = 1; l < c->L; ++l) {
        s.A[l] = alloc_act(c, ar, rows, c->ld[l]);
        s.Dl[l] = alloc_act(c, ar, rows, c->ld[l]);
    }
    s.dL = ar.template get<float>(rows + 1);
    s.zL = ar.template get<float>(rows + 1);
}
// the query set's activations and deltas of the hidden layers, one stretch
static size_t alloc_query(const gm_ctx* c, Arena& ar, std::vector<Act>& A, std::vector<Act>& D, int64_t rows) {
    const size_t from = ar.off;
    A.assign(c->L, Act());
    D.assign(c->L, Act());
    for (int l = 1; l < c->L; ++l) {
        A[l] = alloc_act(c, ar, rows, c->ld[l]);
        D[l] = alloc_act(c, ar, rows, c->ld[l]);
    }
    return ar.off - from;
}
static Spare make_spare(const gm_ctx* c, int64_t Tw, int64_t Pq, void* query, size_t query_bytes, float* query_grad, float* v, Arena* beyond) {
    Spare s;
    s.part[0].base = static_cast<char*>(query); s.part[0].cap = query_bytes;
    s.part[1].base = reinterpret_cast<char*>(query_grad); s.part[1].cap = (size_t)Pq * c->FD * sizeof(float);
    s.part[2].base = reinterpret_cast<char*>(v); s.part[2].cap = (size_t)Tw * c->n_theta * sizeof(float);
    s.beyond = beyond;
    return s;
}
// What a call without a chain keeps in spare memory: the second of three steps' input gradients (grads), and every step's activations (acts)
// but for the first step's and the second one's input, which have the room of two steps' that take turns.
static void alloc_first_order(const gm_ctx* c, Spare& sp, WaveBufs& w, int64_t rows, int K, bool grads, bool acts) {
    w.dX_kept = grads ? sp.get<float>(rows * c->FD) : nullptr;
    for (int k = 1; acts && k < K; ++k) {
        if (k > 1) w.steps[k].X = alloc_act(c, sp, rows, c->ld[0]);
        alloc_step(c, sp, w.steps[k], rows);
    }
}
static Theta alloc_theta(const gm_ctx* c, Arena& ar, int Tw, bool need_f) {
    Theta t;
    if (need_f) {
        t.f = ar.get<float>((int64_t)Tw * c->n_theta);
        t.sf = c->n_theta;
    }
    if (c->mlp_dtype) {
        t.b = ar.get<bf16_t>((int64_t)Tw * c->n_theta_b);
        t.sb = c->n_theta_b;
    }
    return t;
}

static void alloc_sort(const gm_ctx* c, Arena& ar, SortBufs& so, int64_t nnz, int64_t max_segs, size_t extra_hist_words,
                       bool need_gx) {
    so.keys = ar.get<u32>(nnz + 1);
    so.keys_tmp = ar.get<u32>(nnz + 1);
    so.vals = ar.get<u32>(nnz + 1);   // (vals .. vals_tmp: seg_room)
    so.hist = ar.get<u32>(radix_hist_words(nnz, c->F) + extra_hist_words);
    so.scan_tmp = ar.get<u32>(scan_tmp_words(nnz));
    so.seg_start = ar.get<u32>(std::min(nnz, max_segs) + 2);
    so.seg_partial = need_gx ? ar.get<float>(seg_reduce_partial_floats(nnz, c->D)) : nullptr;
    so.vals_tmp = ar.get<u32>(nnz + 1);
}
// Room for the segment reduction's partial rows.  Nothing of the sort but its result and the flags' scan (keys_tmp) is read
// any more by then: the unused values, the digit counts and what lies beside them are one stretch with seg_partial, so narrow
// rows can be cut into short chunks without more workspace.
static float* seg_room(const gm_ctx* c, const SortBufs& so) { return c->D <= 16 ? reinterpret_cast<float*>(std::min(so.hist, so.vals_tmp)) : so.seg_partial; }

// What depends on the indices only (row dictionaries, overlap join, pair-count matrices, and with the table-shaped
// output the wave's own sort buffers): a batch's can be prepared while another batch computes.
static void alloc_wave_index(const gm_ctx* c, Arena& ar, WaveBufs& w, const WaveDims& d) {
    const int F = c->F;
    const int64_t TF = (int64_t)d.Tw * F;
    w.row_off_s = ar.get<int32_t>(d.Tw + 1);
    w.row_off_q = ar.get<int32_t>(d.Tw + 1);
    w.real_off_s = ar.get<int32_t>(d.Tw + 1);
    w.real_off_q = ar.get<int32_t>(d.Tw + 1);
    w.tile_g_s = ar.get<int32_t>(d.mt_s + 1);
    w.tile_m_s = ar.get<int32_t>(d.mt_s + 1);
    w.tile_g_q = ar.get<int32_t>(d.mt_q + 1);
    w.tile_m_q = ar.get<int32_t>(d.mt_q + 1);
    w.coarse_off_s = ar.get<int32_t>(COARSE_GROUPS + 1);
    w.coarse_off_q = ar.get<int32_t>(COARSE_GROUPS + 1);
    w.task_path = ar.get<u32>(d.Tw + 1);
    w.pair_off_ss = w.pair_off_qs = w.pair_off_sq = nullptr;
    w.count_order = nullptr;
    if (d.pair) {   // (one stretch: four of a task's 32-bit words take what three of 64 bits would, and less)
        u32* const p = ar.get<u32>(4 * (d.Tw + 1));
        w.pair_off_ss = p;
        w.pair_off_qs = p + (d.Tw + 1);
        w.pair_off_sq = p + 2 * (d.Tw + 1);
        w.count_order = reinterpret_cast<int32_t*>(p + 3 * (d.Tw + 1));
    }
    const int fx = hop_slices(F, c->D);
    if (d.pair) {
        const int64_t es = hop_entries(d.hop_tiles_s, fx), eq = hop_entries(d.hop_tiles_q, fx);
        const int64_t words[4] = {d.Tw + 1, 9 + es + eq, 9 + es, 9 + eq};
        w.hop_small = ar.get<int32_t>(words[0] + words[1] + words[2] + words[3]);
        for (int k = 0; k < 3; ++k) w.hop_tiles[k] = (k ? w.hop_tiles[k - 1] : w.hop_small) + words[k];
    }
    // (down to here: filled by setup_wave, in one copy)
    w.row_task_s = ar.get<int32_t>(d.Ps + 1);
    w.row_task_q = ar.get<int32_t>(d.Pq + 1);
    w.cnt_s = ar.get<u32>(TF + 1);
    w.base_s = ar.get<u32>(TF + 1);
    w.cnt_q = ar.get<u32>(TF + 1);
    w.base_q = ar.get<u32>(TF + 1);
    w.n_slots = ar.get<u32>(TF + 1);
    w.scan_tmp = ar.get<u32>(scan_tmp_words(TF + 1));
    w.slot_rows = ar.get<u32>(d.nnz_s + 1);
    w.slot_start = ar.get<int32_t>(d.nnz_s + TF + 1);
    w.sup_sorted = ar.get<int2>(d.nnz_s + 1);
    w.sup_slot = ar.get<int32_t>(d.nnz_s + 1);
    w.qry_slot = ar.get<int32_t>(d.nnz_q + 1);
    w.qry_sorted = ar.get<int2>(d.nnz_q + 1);
    w.qseg_lo = ar.get<int32_t>(d.nnz_s + 1);
    w.qseg_hi = ar.get<int32_t>(d.nnz_s + 1);
    w.fm_off_s = ar.get<u32>(TF + 1);
    w.fm_off_q = ar.get<u32>(TF + 1);
    w.field_tab = ar.get<u32>(field_table_words(F));
    w.tmid_keys = w.tmid_vals = nullptr;
    if (F > 0 && c->adapt_rows && c->index_path != 1 && task_sort_passes(d.Tw) > 1) {
        w.tmid_keys = ar.get<u32>(d.nnz_s + d.nnz_q + 1);
        w.tmid_vals = ar.get<u32>(d.nnz_s + d.nnz_q + 1);
    }
    w.pair_mat = d.pair && !d.mat_apart ? ar.get<uint8_t>(d.pair_bytes + 64) : nullptr;
}

// activations, per-task parameters and gradient buffers of a wave; query_grad: the wave's query rows of the batch-wide gradient buffer
// (null where sizes are all that is asked, and with the table-shaped output, which has a buffer per wave)
static void alloc_wave_dense(const gm_ctx* c, Arena& ar, WaveBufs& w, const WaveDims& d, int K, int order, float* query_grad = nullptr) {
    const int L = c->L;
    const bool bf = c->mlp_dtype != 0;
    const int ld0 = c->ld[0];
    if (d.pair && d.mat_apart) w.pair_mat = ar.get<uint8_t>(d.pair_bytes + 64);
    // bf16: the sums over runs of tasks lie where the support set's fp32 input was, which nothing reads after the last inner step
    const int64_t input = d.Ps * ld0, sums = (int64_t)most_runs(c, d.Tw, std::min(d.Ps, d.Pq)) * c->n_theta;
    w.Xs0 = ar.get<float>(bf ? std::max(input, sums) : input);
    w.Xq0 = ar.get<float>(d.Pq * ld0);
    const bool second = order == 2 && K > 0;
    w.TXf = (second && bf) ? ar.get<float>(d.Ps * ld0) : nullptr;
    w.dX = ar.get<float>(std::max(d.Ps, d.Pq) * (int64_t)std::max(c->FD, 1) + 4);
    w.loss_q = ar.get<float>(d.Pq + 1);
    const bool factors = d.factor_ld > 0;
    w.v = Theta{ar.get<float>((int64_t)d.Tw * c->n_theta), c->n_theta, c->mlp_dtype && !factors ? ar.get<bf16_t>((int64_t)d.Tw * c->n_theta_b) : nullptr, c->n_theta_b};
    w.vsum = Theta{bf ? w.Xs0 : ar.get<float>(sums), c->n_theta, nullptr, 0};
    if (!second) w.v.b = nullptr;  // the direction is a GEMM operand only in the second-order pass
    w.Xs_scratch = Act();
    const bool keep = second || d.from_meta;   // every step's activations and deltas
    if (K > 1 && !keep) {
        w.Xs_scratch = alloc_act(c, ar, d.Ps, ld0);
    }
    const int kept = keep ? K : (K > 0 ? 1 : 0);
    w.steps.assign(kept, StepState());
    for (int k = 0; k < kept; ++k) {
        StepState& s = w.steps[k];
        // fp32: step 0 reads Xs0 itself; later steps (second order) keep their own input
        const bool here = second || k == 0;   // (not in spare memory)
        if ((bf || k > 0) && (here || k == 1)) s.X = alloc_act(c, ar, d.Ps, ld0);
        s.X.ld = ld0;
        if (here) alloc_step(c, ar, s, d.Ps);
        s.wL_copy = (bf && second && k > 0) ? ar.get<float>((int64_t)d.Tw * c->ld[L - 1]) : nullptr;
    }
    const size_t query_bytes = alloc_query(c, ar, w.Aq, w.Dq, d.Pq);
    // theta^(k+1), k = 0..K-1.  fp32: one buffer per kept step (the second-order pass needs them all), or one
    // updated in place.  bf16: ONE fp32 master updated in place, and bf16 operand copies per kept step.
    const int n_bufs = second ? K : (K > 0 ? 1 : 0);
    w.thetas.assign(n_bufs, Theta());
    for (int k = 0; k < n_bufs; ++k) {
        if (bf) {
            w.thetas[k] = alloc_theta(c, ar, d.Tw, k == 0);
            if (k > 0) { w.thetas[k].f = w.thetas[0].f; w.thetas[k].sf = w.thetas[0].sf; }
        } else {
            w.thetas[k] = alloc_theta(c, ar, d.Tw, true);
        }
    }
    w.Xq = alloc_act(c, ar, d.Pq, ld0);
    w.dLq = ar.get<float>(d.Pq + 1);
    w.zq = ar.get<float>(d.Pq + 1);
    w.TX = Act();
    w.TA.assign(L, Act());
    w.TD.assign(L, Act());
    w.tdL = nullptr;
    if (second) {
        w.TX = alloc_act(c, ar, d.Ps, ld0);
        for (int l = 1; l < L; ++l) {
            w.TA[l] = alloc_act(c, ar, d.Ps, c->ld[l]);
            w.TD[l] = alloc_act(c, ar, d.Ps, c->ld[l]);
        }
        w.tdL = ar.get<float>(d.Ps + 1);
    }
    w.TXk.clear(); w.TAk.clear(); w.TDk.clear();
    if (factors) {
        for (int k = 0; k < K; ++k) {   // (the last step's are the ones above)
            if (k == K - 1) { w.TXk.push_back(w.TX); w.TAk.push_back(w.TA); w.TDk.push_back(w.TD); break; }
            w.TXk.push_back(alloc_act(c, ar, d.Ps, ld0));
            w.TAk.emplace_back(L);
            w.TDk.emplace_back(L);
            for (int l = 1; l < L; ++l) {
                w.TAk[k][l] = alloc_act(c, ar, d.Ps, c->ld[l]);
                w.TDk[k][l] = alloc_act(c, ar, d.Ps, c->ld[l]);
            }
        }
        w.room.ld = round_up(d.factor_ld, 64);
        w.room.slot = std::max(d.Ps, d.Pq) * 2 * w.room.ld;
        w.room.S = ar.get<bf16_t>(w.room.slot * factor_slots(K) + 8);
    }
    if (d.table) {
        w.GX = ar.get<float>((d.Ps + d.Pq) * (int64_t)std::max(c->FD, 1) + 4);
        query_grad = w.GX ? w.GX + d.Ps * (int64_t)c->FD : nullptr;
        w.n_rows = ar.get<int64_t>(2);
        alloc_sort(c, ar, w.so, d.nnz_s + d.nnz_q, c->field_base[c->F], 0, true);
    }
    w.dX_kept = nullptr;
    if (!second) {
        Spare sp = make_spare(c, d.Tw, d.Pq, L > 1 ? w.Aq[1].b : nullptr, bf ? query_bytes : 0, query_grad, w.v.f, &ar);
        alloc_first_order(c, sp, w, d.Ps, K, d.query_sum > 2, d.from_meta);
    }
}

static void alloc_wave(const gm_ctx* c, Arena& ar, WaveBufs& w, const WaveDims& d, int K, int order) {
    alloc_wave_index(c, ar, w, d);
    alloc_wave_dense(c, ar, w, d, K, order);
}

struct BatchBufs {
    int64_t *toff_s, *toff_q;
    int32_t *prow_s, *prow_q, *prow_off_s, *prow_off_q;
    float *GX, *g_theta, *task_loss;
    Theta theta0;
    SortBufs so;
};

// per batch, from the indices only: device copies of the task offsets, the row of every sample in the activation
// buffers, and the buffers of the batch-wide sort
static void alloc_batch_index(const gm_ctx* c, Arena& ar, BatchBufs& b, int T, int64_t Ss, int64_t Sq, int64_t nnz,
                              int64_t capacity, bool need_gx) {
    b.toff_s = ar.get<int64_t>(T + 1);
    b.toff_q = ar.get<int64_t>(T + 1);
    b.prow_off_s = ar.get<int32_t>(T + 1);
    b.prow_off_q = ar.get<int32_t>(T + 1);
    b.prow_s = ar.get<int32_t>(Ss + 1);
    b.prow_q = ar.get<int32_t>(Sq + 1);
    // the histogram area doubles as the scratch of the per-task lookup offsets (2 (T+1) 64-bit words) before any sort
    alloc_sort(c, ar, b.so, nnz, capacity, 2 * (size_t)(T + 1) * 2, need_gx);
}
static void alloc_batch_dense(const gm_ctx* c, Arena& ar, BatchBufs& b, int T, int64_t Ps, int64_t Pq, bool need_gx) {
    b.GX = need_gx ? ar.get<float>((Ps + Pq) * (int64_t)std::max(c->FD, 1) + 4) : nullptr;
    b.theta0 = Theta();
    b.theta0.f = ar.get<float>(c->n_theta);
    if (c->mlp_dtype) b.theta0.b = ar.get<bf16_t>(c->n_theta_b);
    b.g_theta = ar.get<float>(c->n_theta);
    b.task_loss = ar.get<float>(T + 1);
}
static void alloc_batch(const gm_ctx* c, Arena& ar, BatchBufs& b, int T, int64_t Ss, int64_t Sq, int64_t Ps, int64_t Pq,
                        int64_t nnz, int64_t capacity, bool need_gx) {
    alloc_batch_index(c, ar, b, T, Ss, Sq, nnz, capacity, need_gx);
    alloc_batch_dense(c, ar, b, T, Ps, Pq, need_gx);
}

// ------------------------------------------------------------------------------------------------
// ABI: create / destroy / sizes / timing
// ------------------------------------------------------------------------------------------------
extern "C" int gm_create(gm_ctx** out, const gm_model_desc* model, int device, void* hip_stream,
                         size_t workspace_bytes) {
    if (!out) return GM_ERR_ARG;
    gm_ctx* c = new gm_ctx();
    *out = c;  // kept on failure too, so that the message can be read; gm_destroy frees it
    int rc = model_layout(c, model);
    if (rc != GM_OK) return rc;
    c->device = device;
    c->stream = reinterpret_cast<hipStream_t>(hip_stream);
    HIPCHK(c, hipSetDevice(device));
    {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && n > 0) c->n_cus = n;
    }
    if (device < 0 || device >= GM_MAX_DEVICES) return fail(c, GM_ERR_ARG, "device must be in [0, %d)", (int)GM_MAX_DEVICES);
    if (!g_scratch_ptr[device]) {   // once per device, with that device current: every GPU holds its own copy
        void* p = nullptr;
        HIPCHK(c, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        g_scratch_ptr[device] = static_cast<char*>(p);
    }
    c->static_scratch = g_scratch_ptr[device];
    c->ws_bytes = std::max<size_t>(workspace_bytes, 1 << 20);
    HIPCHK(c, hipMalloc(reinterpret_cast<void**>(&c->ws), c->ws_bytes));
    Arena ar;
    ar.base = c->ws;
    ar.cap = c->ws_bytes;
    c->d_field_base = ar.get<int64_t>(c->F + 1);
    c->d_status = ar.get<u32>(ST_WORDS);
    c->d_status_side = ar.get<u32>(ST_WORDS);
    HIPCHK(c, hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking));
    HIPCHK(c, hipEventCreateWithFlags(&c->ev_side, hipEventDisableTiming));
    HIPCHK(c, hipEventCreateWithFlags(&c->ev_main, hipEventDisableTiming));
    HIPCHK(c, hipEventCreateWithFlags(&c->ev_go, hipEventDisableTiming));
    HIPCHK(c, hipEventCreateWithFlags(&c->ev_pairs_go, hipEventDisableTiming));
    HIPCHK(c, hipEventCreateWithFlags(&c->ev_pairs, hipEventDisableTiming));
    c->persistent = ar.off;
    HIPCHK(c, hipMemcpy(c->d_field_base, c->field_base.data(), (c->F + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
    return GM_OK;
}

extern "C" void gm_destroy(gm_ctx* c) {
    if (!c) return;
    if (c->ws) {
        (void)hipSetDevice(c->device);
        for (ProfPending& p : c->prof_pending) {
            (void)hipEventDestroy(p.e0);
            (void)hipEventDestroy(p.e1);
        }
        for (hipEvent_t e : c->prof_free) (void)hipEventDestroy(e);
        if (c->side) { (void)hipStreamSynchronize(c->side); (void)hipStreamDestroy(c->side); }
        if (c->ev_side) (void)hipEventDestroy(c->ev_side);
        if (c->ev_main) (void)hipEventDestroy(c->ev_main);
        if (c->ev_go) (void)hipEventDestroy(c->ev_go);
        if (c->ev_pairs_go) (void)hipEventDestroy(c->ev_pairs_go);
        if (c->ev_pairs) (void)hipEventDestroy(c->ev_pairs);
        (void)hipFree(c->ws);
    }
    delete c;
}

extern "C" const char* gm_last_error(const gm_ctx* c) { return c ? c->err.c_str() : "null context"; }

extern "C" int gm_configure(gm_ctx* c, const char* key, int64_t value) {
    if (!c) return GM_ERR_ARG;
    if (!key) return fail(c, GM_ERR_ARG, "null key");
    if (!strcmp(key, "pair_tile_rows")) {   // most out-rows of a pair-count matrix counted at a time (0: as many as fit)
        if (value < 0 || value > 1024) return fail(c, GM_ERR_ARG, "pair_tile_rows must be in [0, 1024]");
        c->pair_tile_rows = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "gemm_tile_n")) {   // column tile of the forward / backward products with 256-row tiles (0: chosen by shape)
        if (value != 0 && value != 128 && value != 256) return fail(c, GM_ERR_ARG, "gemm_tile_n must be 0, 128 or 256");
        c->gemm_tile_n = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "wgrad_wide")) {
        if (value != 0 && value != 1) return fail(c, GM_ERR_ARG, "wgrad_wide must be 0 or 1");
        c->wgrad_wide = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "chain_factors")) {
        if (value < 0 || value > 2) return fail(c, GM_ERR_ARG, "chain_factors must be 0, 1 or 2");
        c->chain_factors = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "theta_from_meta")) {
        if (value != 0 && value != 1) return fail(c, GM_ERR_ARG, "theta_from_meta must be 0 or 1");
        c->theta_from_meta = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "coarse_groups")) {
        if (value < 0 || value > COARSE_GROUPS) return fail(c, GM_ERR_ARG, "coarse_groups must be in [0, 32]");
        c->coarse_groups = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "adapt_rows")) {
        if (value != 0 && value != 1) return fail(c, GM_ERR_ARG, "adapt_rows must be 0 or 1");
        c->adapt_rows = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "overlap_pairs")) {   // (ignored while overlap_sort is on: one side stream, one set of status words)
        if (value != 0 && value != 1) return fail(c, GM_ERR_ARG, "overlap_pairs must be 0 or 1");
        c->overlap_pairs = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "overlap_sort")) {
        if (value != 0 && value != 1) return fail(c, GM_ERR_ARG, "overlap_sort must be 0 or 1");
        c->overlap_sort = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "max_wave_tasks")) {
        if (value < 0 || value > MAX_WAVE_TASKS) return fail(c, GM_ERR_ARG, "max_wave_tasks must be in [0, %d]", (int)MAX_WAVE_TASKS);
        c->max_wave_tasks = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "row_path")) {
        if (value < 0 || value > 2) return fail(c, GM_ERR_ARG, "row_path must be 0, 1 or 2");
        c->row_path = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "sort_fields")) {
        if (value != 0 && value != 1) return fail(c, GM_ERR_ARG, "sort_fields must be 0 or 1");
        c->sort_fields = (int)value;
        return GM_OK;
    }
    if (!strcmp(key, "index_path")) {
        if (value < 0 || value > 2) return fail(c, GM_ERR_ARG, "index_path must be 0, 1 or 2");
        c->index_path = (int)value;
        return GM_OK;
    }
    return fail(c, GM_ERR_ARG, "unknown key '%s'", key);
}

extern "C" int gm_profile(gm_ctx* c, int enable) {
    if (!c) return GM_ERR_ARG;
    c->prof_on = enable != 0;
    if (enable) c->prof.clear();
    return GM_OK;
}

extern "C" const char* gm_profile_report(gm_ctx* c) {
    if (!c) return "";
    c->prof_text.clear();
    char line[256];
    for (auto& kv : c->prof) {
        snprintf(line, sizeof line, "%s %lld %.6f %.6e %.6e\n", kv.first.c_str(), (long long)kv.second.launches,
                 kv.second.ms, kv.second.bytes, kv.second.flops);
        c->prof_text += line;
    }
    return c->prof_text.c_str();
}

// Streaming and matrix-core ceilings of this GPU, measured with kernels of the library's own on the context's
// workspace (whose contents are scratch between calls anyway).
extern "C" int gm_ceilings(gm_ctx* c, double* copy_gbs, double* read_gbs, double* mfma_tflops, double* mfma_random_tflops,
                           int64_t* buffer_bytes) {
    if (!c) return GM_ERR_ARG;
    if (!copy_gbs || !read_gbs || !mfma_tflops || !mfma_random_tflops) return fail(c, GM_ERR_ARG, "null outputs");
    HIPCHK(c, hipSetDevice(c->device));
    hipStream_t st = c->stream;
    const size_t avail = (c->ws_bytes - c->persistent) / 2 / 4096 * 4096;
    const int64_t bytes = (int64_t)std::min<size_t>(avail, (size_t)2 << 30);
    if (bytes < (64 << 20)) return fail(c, GM_ERR_WORKSPACE, "gm_ceilings needs a workspace of at least 130 MiB");
    char* a = c->ws + (c->persistent + 4095) / 4096 * 4096;
    char* b = a + bytes;
    if (buffer_bytes) *buffer_bytes = bytes;
    hipEvent_t e0, e1;
    HIPCHK(c, hipEventCreate(&e0));
    HIPCHK(c, hipEventCreate(&e1));
    auto timed = [&](auto&& launch, int reps, float* best) -> int {
        *best = 1e30f;
        for (int r = 0; r < reps + 1; ++r) {   // the first repetition warms up
            HIPCHK(c, hipEventRecord(e0, st));
            launch();
            HIPCHK(c, hipEventRecord(e1, st));
            HIPCHK(c, hipEventSynchronize(e1));
            float ms = 0.f;
            HIPCHK(c, hipEventElapsedTime(&ms, e0, e1));
            if (r > 0) *best = std::min(*best, ms);
        }
        return GM_OK;
    };
    launch_fill_u32(st, reinterpret_cast<u32*>(a), bytes / 4, 0x3f800000u);
    float ms = 0.f;
    int rc = timed([&] { launch_stream_copy(st, a, b, bytes); }, 5, &ms);
    if (rc == GM_OK) {
        *copy_gbs = 2.0 * bytes / (ms * 1e-3) / 1e9;
        rc = timed([&] { launch_stream_read(st, a, bytes, reinterpret_cast<u32*>(b)); }, 5, &ms);
    }
    if (rc == GM_OK) {
        *read_gbs = (double)bytes / (ms * 1e-3) / 1e9;
        double flops = 0.0;
        rc = timed([&] { flops = launch_mfma_loop(st, 20000, reinterpret_cast<float*>(b)); }, 3, &ms);
        if (rc == GM_OK) {
            *mfma_tflops = flops / (ms * 1e-3) / 1e12;
            rc = timed([&] { flops = launch_mfma_loop_random(st, 40000, reinterpret_cast<float*>(b)); }, 3, &ms);
            if (rc == GM_OK) *mfma_random_tflops = flops / (ms * 1e-3) / 1e12;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != GM_OK) return rc;
    HIPCHK(c, hipStreamSynchronize(st));
    HIPCHK(c, hipGetLastError());
    return GM_OK;
}

static int64_t padded_upper(const gm_ctx* c, int64_t n, int T) { return n + (int64_t)T * (c->row_pad - 1); }

extern "C" size_t gm_workspace_bytes(const gm_model_desc* model, int32_t n_tasks, int64_t n_support, int64_t n_query,
                                     int64_t nnz_support, int64_t nnz_query, int32_t inner_steps, int32_t order) {
    gm_ctx c;
    if (model_layout(&c, model) != GM_OK || n_tasks < 0) return 0;
    Arena ar;
    ar.cap = ~(size_t)0 >> 1;
    ar.get<int64_t>(c.F + 1);
    ar.get<u32>(ST_WORDS);
    BatchBufs b;
    const int64_t total_rows = c.field_base[c.F];
    const int64_t Ps = padded_upper(&c, n_support, n_tasks), Pq = padded_upper(&c, n_query, n_tasks);
    alloc_batch(&c, ar, b, n_tasks, n_support, n_query, Ps, Pq, nnz_support + nnz_query,
                std::min(total_rows, nnz_support + nnz_query), true);
    WaveBufs w;
    WaveDims d;
    d.Tw = n_tasks;
    d.Ss = n_support; d.Sq = n_query; d.Ps = Ps; d.Pq = Pq;
    d.nnz_s = nnz_support; d.nnz_q = nnz_query;
    const FirstOrder first = first_order_keeps(&c, n_tasks, n_support, Ps, Pq, inner_steps);
    d.from_meta = order == 1 ? first.acts : theta_from_meta(&c, n_tasks, n_support, inner_steps, order);
    d.mt_s = (int)(Ps / 64 + n_tasks + 1);  // upper bound on m-tiles
    d.mt_q = (int)(Pq / 64 + n_tasks + 1);
    // pair-count matrices, for tasks of equal size (a batch of uneven tasks may need more and then runs in waves)
    if (n_tasks > 0 && inner_steps > 0 && c.F > 0 && c.D % 32 == 0) {
        const int64_t ns = (n_support + n_tasks - 1) / n_tasks, nq = (n_query + n_tasks - 1) / n_tasks;
        if (std::max(ns, nq) > 0 && std::max(ns, nq) <= 512) {
            const int64_t ps = (ns + 63) & ~(int64_t)63, pq = (nq + 63) & ~(int64_t)63;
            d.pair = true;
            d.query_sum = query_sum(&c, inner_steps);
            if (order == 1 && d.query_sum > 2 && !first.grads) d.query_sum = 0;
            d.pair_ss = inner_steps >= 2;
            d.pair_sq = order == 2;
            if (std::max(ns, nq) > HOP_SMALL) {
                d.hop_tiles_s = n_tasks * ((ns + 255) / 256);
                d.hop_tiles_q = n_tasks * ((nq + 255) / 256);
            }
            d.pair_bytes = (int64_t)n_tasks * c.F * ((d.pair_ss ? ps * ps : 0) + pq * ps * (d.pair_sq ? 2 : 1));
        }
    }
    alloc_wave(&c, ar, w, d, inner_steps, order);
    return ar.off + (1 << 20);
}

// ------------------------------------------------------------------------------------------------
// argument checks shared by the entry points
// ------------------------------------------------------------------------------------------------
static int check_set(gm_ctx* c, const gm_set* s, int T, const char* name, bool any_nnz = false) {
    if (!s || !s->task_offsets) return fail(c, GM_ERR_ARG, "%s: null set or task_offsets", name);
    if (s->n_samples < 0 || s->nnz < 0) return fail(c, GM_ERR_ARG, "%s: negative size", name);
    if (s->task_offsets[0] != 0 || s->task_offsets[T] != s->n_samples)
        return fail(c, GM_ERR_ARG, "%s: task_offsets must start at 0 and end at n_samples", name);
    for (int t = 0; t < T; ++t)
        if (s->task_offsets[t + 1] < s->task_offsets[t]) return fail(c, GM_ERR_ARG, "%s: task_offsets not monotone", name);
    if (s->n_samples > 0 && (!s->bag_offsets || !s->labels || (c->n_dense > 0 && !s->dense)))
        return fail(c, GM_ERR_ARG, "%s: null array", name);
    if (s->nnz > 0 && !s->indices) return fail(c, GM_ERR_ARG, "%s: null indices", name);
    if (s->n_samples == 0 && s->nnz != 0) return fail(c, GM_ERR_ARG, "%s: nnz without samples", name);
    // any_nnz: the call orders lookups wave by wave, so only a wave's lookups must number below 2^31
    if ((s->n_samples + (int64_t)T * 8) * (int64_t)std::max(c->F, 1) >= ((int64_t)1 << 31) ||
        (!any_nnz && s->nnz >= ((int64_t)1 << 31)))
        return fail(c, GM_ERR_ARG, "%s: more than 2^31 bags or lookups in one call", name);
    return GM_OK;
}

static SetView make_view(const gm_set* s, const int64_t* d_toff, int64_t sample0, int64_t lookup0) {
    SetView v;
    v.bag_offsets = s->bag_offsets;
    v.indices = s->indices;
    v.task_offsets = d_toff;
    v.sample0 = sample0;
    v.lookup0 = lookup0;
    v.n_samples = s->n_samples;
    return v;
}

static int read_status(gm_ctx* c, u32* host) {
    HIPCHK(c, hipMemcpyAsync(host, c->d_status, ST_WORDS * sizeof(u32), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return GM_OK;
}

// ------------------------------------------------------------------------------------------------
// dense operators on handles (MFMA GEMMs: fp32 or bf16 operands)
// ------------------------------------------------------------------------------------------------
struct Grp {  // grouping of one set's rows by task inside the wave
    const int32_t *row_off, *real_off, *row_task;
    const int32_t *tile_g, *tile_m;
    int n_mtiles, G, bm;
    int64_t rows;  // padded rows of the set in the wave
    int most_rows; // of one task
    const FactorRoom* room = nullptr;
    bool whole = false;  // all rows as one group (the tasks have the weights in common)
};
// The same rows as one group for products with shared weights: tiles then run over the tasks' borders (bf16; 700 tasks of a
// median 32 rows, a first-layer product of the first step 0.76 -> 0.27 ms; 201 tasks of 75..225 rows 0.15 -> 0.08).
static Grp whole_group(const gm_ctx* c, const Grp& g);


// column tile of a forward / backward product.  256 (256-row tiles, a multiple of 256 columns): it wins where the
// contraction is long enough to pay for its unhidden prologue and epilogue (one workgroup per compute unit).  512 tasks of 256
// rows: contraction 1,677, a forward launch 309 us (256 x 128 tiles 364); contraction 256, backward 126 us (115).  Results are
// identical either way.
static int gemm_bn(const gm_ctx* c, int bm, int N, int K) {
    if (bm != 256 || N < 256 || N % 256 != 0) return 128;
    if (c->gemm_tile_n) return c->gemm_tile_n;
    return K >= 1024 ? 256 : 128;
}

// Row tile of products of N columns and contraction K whose rows are cut into mtiles(bm) tiles: bm, or smaller where compute units
// would be left without a tile (the contraction of a tile is a serial chain whatever its size).  256 x 256 tiles become four each,
// and pay down to half a tile a compute unit: second-order steps of 64 / 72 / 96 / 127 tasks of 256 rows (1677-512-256, 128 / 144 / 192 /
// 254 tiles) in 256 rows 2.52 / 2.80 / 3.39 / 4.28 ms, in 128 rows 2.47 / 2.81 / 3.42 / 4.37; 16 / 18 / 24 tasks of 512 rows
// (4109-1024-512-256, 128 / 144 / 192) 3.28 / 3.78 / 4.32 and 3.22 / 3.83 / 4.45; products of shared weights alike (28 x 512 rows, 224
// tiles, 3.36 / 3.42).  Narrower tiles become two each: 50 / 70 tasks of 256 rows (1677-264-136, 150 / 210 tiles of 256 x 128) 1.96 / 2.43
// and 1.94 / 2.43; in 128 rows / in 64 20 tasks of 128 rows (160 tiles) 2.73 / 2.67, of 256 rows 1.15 / 1.16.
template <class MTiles>
static int row_tile(const gm_ctx* c, int bm, int N, int K, MTiles&& mtiles) {
    for (; bm > 64; bm /= 2) {
        const int bn = gemm_bn(c, bm, N, K);
        if (mtiles(bm) * ((N + bn - 1) / bn) >= (bn == 256 ? c->n_cus / 2 + 1 : c->n_cus)) break;
    }
    return bm;
}

// out[rows, ld_l] = epi( sum_p in_p[rows, ld_{l-1}] * W_p,l + bias )
// The factors of th's layer-l weights, for a product with `in` (forward: in * W, else in * W^T): the thin products with P (Q)
// are made here, in one launch, the ones with Q (P) are added to a's list.
static void add_factors(gm_ctx* c, const Grp& g, int l, const Act* in, const Theta* th, bool forward, GemmBArgs& a) {
    if (!th->fac) return;
    const FactorRoom* room = g.room;
    GemmBArgs s;
    memset(&s, 0, sizeof s);
    for (const Factor& f : *th->fac) {
        const Act *P = l == 1 ? f.X : &(*f.A)[l - 1], *Q = &(*f.D)[l];
        if (!P) continue;
        if (!forward) std::swap(P, Q);
        const int e = a.ext.n++;
        s.ext.n = a.ext.n;
        s.ext.Q[e] = P->b; s.ext.c[e] = f.c;
        s.ext.rows[e] = a.ext.rows[e] = f.query ? room->rows_q : room->rows_s;
        s.most_n = std::max(s.most_n, f.query ? room->most_q : room->most_s);
        s.ext.ldq = P->ld; a.ext.ldq = Q->ld;
        a.ext.S[e] = room->S + e * room->slot; a.ext.Q[e] = Q->b;
    }
    const int W = in->ld;
    s.row_offsets = g.row_off; s.G = g.G; s.n_pairs = 1;
    s.A[0] = in->b; s.lda[0] = W; s.rA[0] = W; s.ldb[0] = W; s.rB[0] = W;
    s.M = -1; s.N = -1; s.K = W;
    s.tile_group = g.tile_g; s.tile_m0 = g.tile_m; s.n_mtiles = g.n_mtiles;
    s.epi = EPI_SPLIT;
    s.Cb = room->S; s.ldcb = 2 * room->ld; s.rCb = 2 * room->ld; s.ext.ld = a.ext.ld = room->ld; s.ext.slot = room->slot;
    launch_gemm_bf16(c->stream, s, 64);
}

static void dense_nn(gm_ctx* c, const Grp& g, int l, int np, const Act* in0, const Theta* th0, const Act* in1,
                     const Theta* th1, const float* bias, int64_t bias_stride, const Act* mask, int epi, Act& out) {
    const int K = c->ld[l - 1], N = c->ld[l];
    // algorithmic bytes: operands once (per-task weights once per task), every output once
    const double esz = c->mlp_dtype ? 2.0 : 4.0;
    double by = (double)g.rows * N * esz + (mask ? (double)g.rows * N * esz : 0.0);
    for (int i = 0; i < np; ++i) {
        const Theta* t = i ? th1 : th0;
        by += (double)g.rows * K * esz + (double)((c->mlp_dtype ? t->sb : t->sf) ? g.G : 1) * K * N * esz;
    }
    Prof p(c, "gemm_fwd", by, 2.0 * g.rows * N * K * np);
    const Act* ins[2] = {in0, in1};
    const Theta* ths[2] = {th0, th1};
    if (c->mlp_dtype == 0) {
        GemmArgs a;
        memset(&a, 0, sizeof a);
        a.row_offsets = g.row_off; a.G = g.G; a.n_pairs = np;
        for (int i = 0; i < np; ++i) {
            a.A[i] = ins[i]->f; a.sAm[i] = K; a.sAk[i] = 1; a.rA[i] = K;
            a.B[i] = ths[i]->f + c->offW[l]; a.sBk[i] = N; a.sBn[i] = 1; a.gB[i] = ths[i]->sf;
        }
        a.C = out.f; a.ldc = N; a.rC = N; a.M = -1; a.N = N; a.K = K;
        a.tile_group = g.tile_g; a.tile_m0 = g.tile_m; a.n_mtiles = g.n_mtiles;
        a.epi = epi; a.bias = bias; a.gBias = bias_stride;
        if (mask) { a.mask = mask->f; a.ld_mask = mask->ld; }
        launch_gemm_f32(c->stream, a);
    } else {
        GemmBArgs a;
        memset(&a, 0, sizeof a);
        a.row_offsets = g.row_off; a.G = g.G; a.n_pairs = 0;
        for (int i = 0; i < np; ++i) {   // W as stored, [d_in, d_out]: the contraction index is its slow one
            if (ths[i]->b) {
                const int p = a.n_pairs++;
                a.A[p] = ins[i]->b; a.lda[p] = K; a.rA[p] = K;
                a.B[p] = ths[i]->b + c->offWb[l]; a.ldb[p] = N; a.gB[p] = ths[i]->sb;
            }
            add_factors(c, g, l, ins[i], ths[i], true, a);
        }
        a.Cb = out.b; a.ldcb = N; a.rCb = N; a.M = g.whole ? (int)g.rows : -1; a.N = N; a.K = K;
        a.tile_group = g.tile_g; a.tile_m0 = g.tile_m; a.n_mtiles = g.n_mtiles;
        a.epi = epi; a.bias = bias; a.gBias = bias_stride;
        if (mask) { a.mask = mask->b; a.ld_mask = mask->ld; }
        launch_gemm_bf16_bkmajor(c->stream, a, g.bm, gemm_bn(c, g.bm, N, K * np));
    }
}

// out[rows, ld_{l-1}] = mask .* sum_p d_p[rows, ld_l] * W_p,l^T ; for l == 1: dX[rows, FD] fp32, no mask
// dX (layer 1 only): the fp32 gradient w.r.t. the pooled input.  With write_dx = false it goes, scaled, into gx_acc instead
// (gx_acc += gx_scale * dX, or = with gx_init); bf16 mode can do both in the same pass, and with gx_old make it gx_scale * (what dX
// held before + dX).
static void dense_nt(gm_ctx* c, const Grp& g, int l, int np, const Act* d0, const Theta* th0, const Act* d1,
                     const Theta* th1, const Act* mask, Act* out, float* dX, float* gx_acc = nullptr, float gx_scale = 0.f,
                     bool write_dx = true, bool gx_init = false, bool gx_old = false) {
    const int K = c->ld[l], N = dX ? c->FD : c->ld[l - 1];
    if (N <= 0) return;
    const double esz = c->mlp_dtype ? 2.0 : 4.0;
    double by = dX ? (double)g.rows * N * 4.0 * ((write_dx ? 1 : 0) + (gx_acc ? (gx_init ? 1 : 2) : 0)) : (double)g.rows * N * esz;
    if (mask) by += (double)g.rows * N * esz;
    for (int i = 0; i < np; ++i) {
        const Theta* t = i ? th1 : th0;
        by += (double)g.rows * K * esz + (double)((c->mlp_dtype ? t->sb : t->sf) ? g.G : 1) * K * N * esz;
    }
    Prof p(c, "gemm_bwd", by, 2.0 * g.rows * N * K * np);
    const Act* ds[2] = {d0, d1};
    const Theta* ths[2] = {th0, th1};
    if (c->mlp_dtype == 0) {
        GemmArgs a;
        memset(&a, 0, sizeof a);
        a.row_offsets = g.row_off; a.G = g.G; a.n_pairs = np;
        for (int i = 0; i < np; ++i) {
            a.A[i] = ds[i]->f; a.sAm[i] = K; a.sAk[i] = 1; a.rA[i] = K;
            a.B[i] = ths[i]->f + c->offW[l]; a.sBk[i] = 1; a.sBn[i] = K; a.gB[i] = ths[i]->sf;
        }
        a.M = -1; a.N = N; a.K = K;
        a.tile_group = g.tile_g; a.tile_m0 = g.tile_m; a.n_mtiles = g.n_mtiles;
        if (dX && !write_dx) {   // straight into the sum
            a.C = gx_acc; a.ldc = N; a.rC = N; a.epi = EPI_AXPBY; a.c1 = gx_scale;
            if (!gx_init) { a.Cin = gx_acc; a.rCin = N; a.c0 = 1.f; }
        } else if (dX) { a.C = dX; a.ldc = N; a.rC = N; a.epi = EPI_NONE; }
        else { a.C = out->f; a.ldc = N; a.rC = N; a.epi = EPI_MASK; a.mask = mask->f; a.ld_mask = mask->ld; }
        launch_gemm_f32(c->stream, a);
    } else {
        GemmBArgs a;
        memset(&a, 0, sizeof a);
        a.row_offsets = g.row_off; a.G = g.G; a.n_pairs = 0;
        for (int i = 0; i < np; ++i) {
            if (ths[i]->b) {
                const int p = a.n_pairs++;
                a.A[p] = ds[i]->b; a.lda[p] = K; a.rA[p] = K;
                a.B[p] = ths[i]->b + c->offWb[l]; a.ldb[p] = K; a.gB[p] = ths[i]->sb;
            }
            add_factors(c, g, l, ds[i], ths[i], false, a);
        }
        a.M = g.whole ? (int)g.rows : -1; a.N = N; a.K = K;
        a.tile_group = g.tile_g; a.tile_m0 = g.tile_m; a.n_mtiles = g.n_mtiles;
        if (dX) {
            if (write_dx) { a.Cf = dX; a.ldcf = N; a.rCf = N; }
            a.epi = EPI_NONE;
            if (gx_acc) { a.Cacc = gx_acc; a.ldcacc = N; a.rCacc = N; a.cacc = gx_scale; a.cacc_init = gx_init ? 1 : 0; a.Cold = gx_old ? dX : nullptr; }
        } else {
            a.Cb = out->b; a.ldcb = N; a.rCb = N; a.epi = EPI_MASK; a.mask = mask->b; a.ld_mask = mask->ld;
        }
        launch_gemm_bf16(c->stream, a, g.bm, gemm_bn(c, g.bm, N, K * np));
    }
}

static Grp whole_group(const gm_ctx* c, const Grp& g) {
    if (c->L < 2) return g;
    Grp w = g;
    w.whole = true;
    w.G = 1;
    w.tile_g = w.tile_m = nullptr;
    w.n_mtiles = 0;
    w.bm = row_tile(c, 256, c->ld[1], c->ld[0], [&](int bm) { return (g.rows + bm - 1) / bm; });
    return w;
}

// Weight gradient [M, N] of G groups over `rows` rows in all: 256 x 256 tiles pay once a group's contraction is some 200
// rows long and the tiles fill the device several times over.  Dense-only steps of 256 tasks, first layer 1677 x 512, with
// them and without: 64 rows a task 2.25 / 2.26 ms, 128 4.09 / 4.14, 192 5.51 / 5.58, 256 6.76 / 6.85; 128 tasks, 4109 x 1024: 64
// rows 3.83 / 3.74, 128 7.04 / 7.01, 192 9.05 / 9.07, 256 10.82 / 10.97.  Narrow layers lose to padded rows of the last tile
// (512 tasks, 269 x 256, 256 rows: 2.54 / 2.53).
// Long contractions (runs of tasks) also take them where the tiles fill the compute units' rounds: 512 tasks of 256 rows, 1677 x 512, two
// products, 16 runs in 128 x 128 tiles (896) 691 us, 18 runs in 256 x 256 ones (252) 445; 128 tasks, one product, 89 and 71.
enum { WIDE_LONG = 1024 };
static constexpr double WIDE_FILL = 0.85;
static bool wgrad_wide_shape(const gm_ctx* c, int M, int N) { return c->mlp_dtype && M >= 1024 && N % 256 == 0; }
static double round_fill(const gm_ctx* c, int64_t tiles) { return (double)tiles / (double)((tiles + c->n_cus - 1) / c->n_cus * c->n_cus); }
static bool wgrad_wide_ok(const gm_ctx* c, int M, int N, int64_t rows, int G) {
    if (!c->wgrad_wide || !wgrad_wide_shape(c, M, N) || G <= 0 || rows / G < 192) return false;
    const int64_t tiles = (int64_t)((M + 255) / 256) * (N / 256) * G;
    return tiles >= 2 * (int64_t)c->n_cus || (rows / G >= WIDE_LONG && round_fill(c, tiles) >= WIDE_FILL);
}

// Runs of consecutive tasks that the products only summed over tasks are taken over.  16, unless the first layer's
// product can run in 256 x 256 tiles, one workgroup per compute unit: the count in [12, 18] whose tiles fill the
// last round over the compute units best, the largest run counted (the larger count on a tie).
// The bound: each run is another set of sums to write and read again, and up to 18 nine in ten numbers of tiles a run (4 to 128) fill 85 % of a
// round.  Products and sums of 256 or 128 tasks x 256 + 256 rows, 16 and 18 runs: 14 tiles a run (1677 x 512) 499 and 494 us, 24 (1933 x 768) 859 and 865, 44
// (2573 x 1024) 847 and 884 (17: 869), 68 (4109 x 1024) 1282 and 1284.  More runs gain where a run has few tiles (1037 x 512, ten of them: 24 runs 373, 16 in
// 128 x 128 tiles 409) and lose beyond (20 to 32 runs of the others: 832..888, 864..904, 1288..1353).
enum { MOST_RUNS = 18 };
// rows: of the wave's smaller set.  (The sums have the support input's room, as long as it is, and that of 16 runs otherwise.)
static bool runs_in_wide_tiles(const gm_ctx* c, int64_t rows) {
    return c->L > 1 && c->wgrad_wide && wgrad_wide_shape(c, c->ld[0], c->ld[1]) && rows / MOST_RUNS >= WIDE_LONG && (MOST_RUNS - 16) * c->n_theta <= rows * c->ld[0];
}
static int most_runs(const gm_ctx* c, int Tw, int64_t rows) {   // of a wave (a run has a task at least)
    return std::min(std::max(Tw, 1), c->coarse_groups ? c->coarse_groups : runs_in_wide_tiles(c, rows) ? (int)MOST_RUNS : 16);
}
static int coarse_group_count(const gm_ctx* c, int Tw, int64_t rows) {
    if (c->coarse_groups) return std::min(Tw, c->coarse_groups);
    int n = std::min(Tw, 16);
    if (n < 16 || !runs_in_wide_tiles(c, rows)) return n;
    const int64_t per = (int64_t)((c->ld[0] + 255) / 256) * (c->ld[1] / 256);
    double best = -1.0;
    for (int k = 12; k <= std::min<int>(MOST_RUNS, Tw); ++k) {
        const double fill = round_fill(c, per * k), score = fill * ((double)Tw / k) / ((Tw + k - 1) / k);
        if (fill >= WIDE_FILL && score >= best) { best = score; n = k; }
    }
    return n;
}

// Whether the query gradient, where the second-order chain's direction starts, is summed over runs of tasks beside being written per
// task as the chain's bf16 operand, instead of being written in fp32 per task and read again for the sum: one inner step (the chain's
// next product is summed over runs anyway), and eight bytes a weight and task cost more than the extra product of a layer -- its operations, its
// operands, which narrow layers read for few of them, and a launch.  The four figures are the least squares over 81 steps (24 to 512 tasks of 64
// to 512 query rows, weighted by the power -0.7 of their times; 10, 26, 40 and 64 fields of 64 columns; 128-64 to 1024-512-256).  With the runs
// and with the fp32 copy: 128 tasks of 128 rows, 1677-512-256 1.46 / 1.58 ms, 4109-1024-512-256 4.35 / 4.81, 653-256-128 0.73 / 0.72; of 256 rows
// 1.87 / 1.91, 5.66 / 5.95, 0.87 / 0.83; 200 of 384 rows, 4109-1024-512-256 10.76 / 11.00; 256 of 512 rows 15.12 / 15.04, 1677-512-256 4.64 / 4.61; 128
// of 512, 1677-128-64 1.89 / 1.83.  Where the rule takes the slower one it is by 1.5 % at most.
static constexpr double RUNS_BYTES = 6.56e12, RUNS_RATE = 1.23e15, RUNS_OPERANDS = 5.81e12, RUNS_LAUNCH = 5.27e-6, RUNS_MARGIN = 1.05;
static bool query_runs(const gm_ctx* c, int Tw, int64_t rows_q, int n_runs, int K, int order) {
    if (!c->mlp_dtype || order != 2 || K != 1) return false;
    double saved = 0, cost = 0;
    for (int l = 1; l < c->L; ++l) {
        const double w = (double)c->ld[l - 1] * c->ld[l];
        saved += 8.0 * (Tw - n_runs) * w / RUNS_BYTES;
        cost += 2.0 * rows_q * w / RUNS_RATE + 2.0 * rows_q * (c->ld[l - 1] + c->ld[l]) / RUNS_OPERANDS + RUNS_LAUNCH;
    }
    return saved > RUNS_MARGIN * cost;
}

// fp32 weight gradients of one pass that depend on nothing of each other, collected and launched together
struct WGrads {
    std::vector<GemmArgs> list;
    std::vector<double> bytes, flops;   // algorithmic, of every product
    void add(const GemmArgs& a, double by, double fl) { list.push_back(a); bytes.push_back(by); flops.push_back(fl); }
    void launch(gm_ctx* c) {
        for (size_t i0 = 0; i0 < list.size(); i0 += GEMM_LIST) {
            const size_t i1 = std::min(list.size(), i0 + (size_t)GEMM_LIST);
            double by = 0, fl = 0;
            for (size_t i = i0; i < i1; ++i) { by += bytes[i]; fl += flops[i]; }
            Prof p(c, "gemm_wgrad", by, fl);
            launch_gemm_f32_wgrads(c->stream, list.data() + i0, (int)(i1 - i0));
        }
    }
};

// out_g[ld_{l-1}, ld_l] = c0*in_g + c1 * sum_p a_p[rows_g, ld_{l-1}]^T d_p[rows_g, ld_l]  (and its bf16 copies)
// later: where an fp32 product goes instead of a launch of its own
static void dense_tn_n(gm_ctx* c, const Grp& g, int l, int np, const Act* const* as, const Act* const* ds, Theta& out,
                       const float* in, int64_t in_stride, float c0, float c1, bool write_f32 = true, WGrads* later = nullptr) {
    const int M = c->ld[l - 1], N = c->ld[l];
    const double esz = c->mlp_dtype ? 2.0 : 4.0;
    const double out_b = c->mlp_dtype ? ((write_f32 || !out.b) ? 4.0 : 0.0) + (out.b ? 2.0 : 0.0) : 4.0;
    const double by = (double)np * g.rows * (M + N) * esz + (double)g.G * M * N * (out_b + ((in && in_stride) ? 4.0 : 0.0));
    const double fl = 2.0 * g.rows * N * M * np;
    if (c->mlp_dtype == 0) {
        GemmArgs a;
        memset(&a, 0, sizeof a);
        a.row_offsets = g.row_off; a.G = g.G; a.n_pairs = np;
        for (int i = 0; i < np; ++i) {
            a.A[i] = as[i]->f; a.sAm[i] = 1; a.sAk[i] = M; a.rA[i] = M;
            a.B[i] = ds[i]->f; a.sBk[i] = N; a.sBn[i] = 1; a.rB[i] = N;
        }
        a.C = out.f + c->offW[l]; a.ldc = N; a.gC = out.sf; a.M = M; a.N = N; a.K = -1;
        a.epi = EPI_AXPBY; a.Cin = in ? in + c->offW[l] : nullptr; a.gCin = in_stride; a.c0 = c0; a.c1 = c1;
        WGrads alone;
        (later ? *later : alone).add(a, by, fl);
        alone.launch(c);
    } else {
        Prof p(c, "gemm_wgrad", by, fl);
        GemmBArgs a;
        memset(&a, 0, sizeof a);
        a.row_offsets = g.row_off; a.G = g.G; a.n_pairs = np;
        for (int i = 0; i < np; ++i) {   // activations and deltas as they are stored: [rows, width]
            a.A[i] = as[i]->b; a.lda[i] = M; a.rA[i] = M;
            a.B[i] = ds[i]->b; a.ldb[i] = N; a.rB[i] = N;
        }
        if (write_f32 || !out.b) { a.Cf = out.f + c->offW[l]; a.ldcf = N; a.gCf = out.sf; }
        a.M = M; a.N = N; a.K = -1;
        if (out.b) {  // the bf16 operand copy of W
            a.Cb = out.b + c->offWb[l]; a.ldcb = N; a.gCb = out.sb;
        }
        a.epi = EPI_AXPBY; a.Cin = in ? in + c->offW[l] : nullptr; a.gCin = in_stride; a.ldcin = N; a.c0 = c0; a.c1 = c1;
        launch_gemm_bf16_kmajor(c->stream, a, wgrad_wide_ok(c, M, N, g.rows, g.G) ? 256 : 128);
    }
}

static void dense_tn(gm_ctx* c, const Grp& g, int l, int np, const Act* a0, const Act* d0, const Act* a1, const Act* d1,
                     Theta& out, const float* in, int64_t in_stride, float c0, float c1, bool write_f32 = true,
                     WGrads* later = nullptr) {
    const Act* as[2] = {a0, a1};
    const Act* ds[2] = {d0, d1};
    dense_tn_n(c, g, l, np, as, ds, out, in, in_stride, c0, c1, write_f32, later);
}

// The per-task column sums of one pass, collected and launched together.
struct ColSums {
    gm_ctx* c;
    const Grp& g;
    std::vector<ColJob> jobs;
    double bytes = 0;   // algorithmic: every operand row once (and its per-row weights), one output row per task (read back when updated)
    void add(int N, const Act* X1, const float* w1, const Act* X2, const float* w2, float* out, int64_t g_out, const float* in,
             int64_t g_in, float c0, float c1) {
        bytes += (double)g.rows * N * (c->mlp_dtype ? 2.0 : 4.0) * (X2 ? 2 : 1) + 4.0 * g.rows * ((w1 ? 1 : 0) + (w2 ? 1 : 0)) +
                 4.0 * g.G * N * (in ? 2 : 1);
        auto data = [&](const Act* x) { return c->mlp_dtype ? (const void*)x->b : (const void*)x->f; };
        jobs.push_back(ColJob{N, 0, data(X1), w1, X2 ? data(X2) : nullptr, w2, X1->ld, out, g_out, in, g_in, c0, c1});
    }
    void add_scalar(const float* x, float* out, int64_t g_out, const float* in, int64_t g_in, float c0, float c1) {   // one value per row
        bytes += 4.0 * g.rows + 4.0 * g.G * (in ? 2 : 1);
        jobs.push_back(ColJob{1, 0, x, nullptr, nullptr, nullptr, 1, out, g_out, in, g_in, c0, c1});
    }
    void launch() {
        Prof p(c, "task_colsum", bytes, 0);
        launch_task_colsum(c->stream, c->mlp_dtype, g.G, g.most_rows, g.row_off, jobs.data(), (int)jobs.size());
    }
};

static const void* act_ptr(const gm_ctx* c, const Act& a) { return c->mlp_dtype ? (const void*)a.b : (const void*)a.f; }
static void* act_ptr(const gm_ctx* c, Act& a) { return c->mlp_dtype ? (void*)a.b : (void*)a.f; }

struct Pass {  // activations of one forward/backward pass over one set
    Act* X;
    std::vector<Act>*A, *Dl;
    float *dL, *zL;
};

// forward with parameters th (GEMM operands) / thf (fp32: biases and the last layer), loss and delta_L; then
// backward to the deltas of every layer and, when dX is given, to the pooled-input gradient [rows, FD].
static void forward_backward(gm_ctx* c, const Grp& g, const float* labels, const Pass& p, const Theta& th,
                             const float* thf, int64_t thf_stride, float* loss_out, float* dX) {
    hipStream_t st = c->stream;
    const int L = c->L;
    const Act* prev = p.X;
    const Grp gd = c->mlp_dtype && th.sb == 0 && thf_stride == 0 ? whole_group(c, g) : g;
    for (int l = 1; l < L; ++l) {
        dense_nn(c, gd, l, 1, prev, &th, nullptr, nullptr, thf + c->offb[l], thf_stride, nullptr, EPI_BIAS_RELU, (*p.A)[l]);
        prev = &(*p.A)[l];
    }
    const float* wL = thf + c->offW[L];
    {
        // algorithmic bytes: the last hidden activations read, the delta of the last hidden layer written, 20 bytes of
        // per-row scalars (label, logit, delta, loss, task)
        const double esz_l = c->mlp_dtype ? 2.0 : 4.0;
        Prof pr(c, "last_layer", (double)g.rows * c->ld[L - 1] * esz_l * (L > 1 ? 2 : 1) + 20.0 * g.rows + (L == 1 && dX ? 4.0 * g.rows * c->FD : 0.0), 0);
        LastArgs f;
        memset(&f, 0, sizeof f);
        f.n = g.rows; f.N = c->ld[L - 1]; f.ld = c->ld[L - 1]; f.bf16 = c->mlp_dtype;
        f.row_task = g.row_task; f.row_offsets = g.row_off; f.real_offsets = g.real_off;
        f.a = act_ptr(c, *prev); f.w = wL; f.gW = thf_stride; f.b = thf + c->offb[L];
        f.labels = labels; f.z_out = p.zL; f.delta_out = p.dL; f.loss_out = loss_out;
        if (L > 1) f.d = act_ptr(c, (*p.Dl)[L - 1]);
        launch_last_layer(st, f);
        if (L == 1) {
            if (dX) launch_input_delta(st, g.rows, c->FD, g.row_task, p.dL, wL, thf_stride, nullptr, nullptr, 0, dX);
            return;
        }
    }
    for (int l = L - 1; l >= 1; --l) {
        if (l == 1) {
            if (dX) dense_nt(c, gd, l, 1, &(*p.Dl)[l], &th, nullptr, nullptr, nullptr, nullptr, dX);
        } else {
            dense_nt(c, gd, l, 1, &(*p.Dl)[l], &th, nullptr, nullptr, &(*p.A)[l - 1], &(*p.Dl)[l - 1], nullptr);
        }
    }
}

// out = c0*in + c1 * (gradient of the pass w.r.t. theta), per task; out.b (if any) gets the bf16 operand copies.
// coarse / coarse_out: the hidden layers' weight matrices are summed over runs of tasks instead (c1 times the gradient,
// nothing added), for a caller that only wants their sum over the tasks -- and, where out has room for bf16 operands, those per
// task; biases and the last layer stay per task.
// hist / in0 (bf16 operands, an inner step of a call that keeps its steps' activations): the passes of all inner steps so far, this
// one last, and the meta parameters.  The step's weight matrices are then written as theta - alpha * (sum of the steps'
// gradients), one product per step accumulated in the matrix cores, from the shared fp32 theta: no per-task fp32
// master of a weight matrix is written or read (it was most of what a step of small tasks moved); biases and the
// last layer keep their per-task fp32 chain (in, in_stride).
// loss / task_loss: the rows' losses, summed per task along with the rest.
static void theta_grad(gm_ctx* c, const Grp& g, const Pass& p, Theta& out, const float* in, int64_t in_stride, float c0,
                       float c1, float* wL_copy, bool write_f32 = true, const Grp* coarse = nullptr,
                       Theta* coarse_out = nullptr, const std::vector<Pass>* hist = nullptr, const float* in0 = nullptr,
                       const float* loss = nullptr, float* task_loss = nullptr) {
    const int L = c->L;
    const int64_t nt = out.sf;
    ColSums sums{c, g};
    WGrads later;
    for (int l = 1; l < L; ++l) {
        const Act* prev = l == 1 ? p.X : &(*p.A)[l - 1];
        if (coarse) {
            dense_tn(c, *coarse, l, 1, prev, &(*p.Dl)[l], nullptr, nullptr, *coarse_out, nullptr, 0, 0.f, c1, true, &later);
            if (out.b) dense_tn(c, g, l, 1, prev, &(*p.Dl)[l], nullptr, nullptr, out, nullptr, 0, 0.f, c1, false);
        }
        else if (hist) {
            const Act* as[GEMM_MAX_PAIRS];
            const Act* ds[GEMM_MAX_PAIRS];
            const int np = (int)hist->size();
            for (int j = 0; j < np; ++j) {
                as[j] = l == 1 ? (*hist)[j].X : &(*(*hist)[j].A)[l - 1];
                ds[j] = &(*(*hist)[j].Dl)[l];
            }
            dense_tn_n(c, g, l, np, as, ds, out, in0, 0, c0, c1, false);
        } else dense_tn(c, g, l, 1, prev, &(*p.Dl)[l], nullptr, nullptr, out, in, in_stride, c0, c1, write_f32, &later);
        sums.add(c->ld[l], &(*p.Dl)[l], nullptr, nullptr, nullptr, out.f + c->offb[l], nt, in ? in + c->offb[l] : nullptr,
                 in_stride, c0, c1);
    }
    later.launch(c);
    const Act* prev = L == 1 ? p.X : &(*p.A)[L - 1];
    sums.add(c->ld[L - 1], prev, p.dL, nullptr, nullptr, out.f + c->offW[L], nt, in ? in + c->offW[L] : nullptr, in_stride, c0, c1);
    sums.add_scalar(p.dL, out.f + c->offb[L], nt, in ? in + c->offb[L] : nullptr, in_stride, c0, c1);
    if (loss) sums.add_scalar(loss, task_loss, 1, nullptr, 0, 0.f, 1.f);
    sums.launch();
    if (wL_copy)
        (void)hipMemcpy2DAsync(wL_copy, c->ld[L - 1] * sizeof(float), out.f + c->offW[L], nt * sizeof(float),
                               c->ld[L - 1] * sizeof(float), g.G, hipMemcpyDeviceToDevice, c->stream);
}

// v <- v - alpha * (H v)_theta ;  w.dX [rows, FD] <- (H v)'s pooled-input part
// (tangent pass through the forward and the backward pass of step s, direction (v, TX))
// gx_acc (bf16 mode): the support rows of the sparse-gradient buffer, which take -alpha * (tangent of dX) in the
// layer-1 product itself; need_dx: the tangent of dX is also wanted in w.dX (for the row arithmetic of the next step); gx_init: the sum's
// first term; gx_old: the first is what w.dX still holds
// coarse (the chain's last step; with factors, every step): the weight matrices' part of H v is not folded into every task's v but summed
// over runs of tasks into w.vsum.  fold: -alpha times it is added to what w.vsum holds, the query gradient's sums (v's own weight
// matrices are then not reduced: factors, query_runs); else it is stored unscaled, and the caller adds -alpha times its sum to the reduced v
static void hvp_step(gm_ctx* c, const Grp& g, const StepState& s, WaveBufs& w, float alpha, bool refresh_v_copies,
                     float* gx_acc, bool need_dx, bool gx_init, bool gx_old, bool tx, const Grp* coarse = nullptr, bool fold = false) {
    hipStream_t st = c->stream;
    const int L = c->L;
    Theta& v = w.v;
    const int64_t nt = v.sf;
    const Act* tprev = &w.TX;
    const Act* prev = &s.X;
    for (int l = 1; l < L; ++l) {
        // (tx false: no direction on the inputs -- rows not adapted -- so layer 1 has one product only)
        if (l == 1 && !tx) dense_nn(c, g, l, 1, prev, &v, nullptr, nullptr, v.f + c->offb[l], nt, &s.A[l], EPI_BIAS_MASK, w.TA[l]);
        else dense_nn(c, g, l, 2, tprev, &s.th, prev, &v, v.f + c->offb[l], nt, &s.A[l], EPI_BIAS_MASK, w.TA[l]);
        tprev = &w.TA[l];
        prev = &s.A[l];
    }
    const float* vwL = v.f + c->offW[L];
    {
        // (tangent pass: activations and their tangents read, the tangent delta written)
        const double esz_l = c->mlp_dtype ? 2.0 : 4.0;
        Prof pr(c, "last_layer", (double)g.rows * c->ld[L - 1] * esz_l * (L > 1 ? 3 : 2) + 24.0 * g.rows + (L == 1 ? 4.0 * g.rows * c->FD : 0.0), 0);
        LastArgs f;
        memset(&f, 0, sizeof f);
        f.n = g.rows; f.N = c->ld[L - 1]; f.ld = c->ld[L - 1]; f.bf16 = c->mlp_dtype;
        f.row_task = g.row_task; f.row_offsets = g.row_off; f.real_offsets = g.real_off;
        f.a = act_ptr(c, *prev); f.ta = act_ptr(c, *tprev); f.w = s.wL; f.gW = s.wL_stride; f.b = nullptr;
        f.tw = vwL; f.gTW = nt; f.tb = v.f + c->offb[L];
        f.z_in = s.zL; f.delta_in = s.dL; f.delta_out = w.tdL;
        // tangent of the backward pass, top layer first; each layer's direction is consumed before it is updated
        if (L > 1) f.d = act_ptr(c, w.TD[L - 1]);
        launch_last_layer(st, f);
        if (L == 1) launch_input_delta(st, g.rows, c->FD, g.row_task, w.tdL, s.wL, s.wL_stride, s.dL, vwL, nt, w.dX);
    }
    ColSums sums{c, g};   // (biases and the last layer's direction: nothing below reads them)
    sums.add(c->ld[L - 1], tprev, s.dL, prev, w.tdL, v.f + c->offW[L], nt, v.f + c->offW[L], nt, 1.f, -alpha);
    sums.add_scalar(w.tdL, v.f + c->offb[L], nt, v.f + c->offb[L], nt, 1.f, -alpha);
    Theta vout = v;
    WGrads later;   // (fp32: the loop's products read every layer's direction before any is updated)
    if (!refresh_v_copies) vout.b = nullptr;
    for (int l = L - 1; l >= 1; --l) {
        if (l == 1) dense_nt(c, g, l, 2, &w.TD[l], &s.th, &s.Dl[l], &v, nullptr, nullptr, w.dX, gx_acc, -alpha, need_dx || !gx_acc, gx_init, gx_old);
        else dense_nt(c, g, l, 2, &w.TD[l], &s.th, &s.Dl[l], &v, &s.A[l - 1], &w.TD[l - 1], nullptr);
        const Act* ta_prev = l == 1 ? &w.TX : &w.TA[l - 1];
        const Act* a_prev = l == 1 ? &s.X : &s.A[l - 1];
        if (coarse) {
            const float* in = fold ? w.vsum.f : nullptr;
            const float c0 = fold ? 1.f : 0.f, c1 = fold ? -alpha : 1.f;
            if (l == 1 && !tx) dense_tn(c, *coarse, l, 1, a_prev, &w.TD[l], nullptr, nullptr, w.vsum, in, w.vsum.sf, c0, c1, true, &later);
            else dense_tn(c, *coarse, l, 2, ta_prev, &s.Dl[l], a_prev, &w.TD[l], w.vsum, in, w.vsum.sf, c0, c1, true, &later);
        } else if (l == 1 && !tx) dense_tn(c, g, l, 1, a_prev, &w.TD[l], nullptr, nullptr, vout, v.f, nt, 1.f, -alpha, true, &later);
        else dense_tn(c, g, l, 2, ta_prev, &s.Dl[l], a_prev, &w.TD[l], vout, v.f, nt, 1.f, -alpha, true, &later);
        sums.add(c->ld[l], &w.TD[l], nullptr, nullptr, nullptr, v.f + c->offb[l], nt, v.f + c->offb[l], nt, 1.f, -alpha);
    }
    later.launch(c);
    sums.launch();
}

// ------------------------------------------------------------------------------------------------
// the step
// ------------------------------------------------------------------------------------------------
struct WavePlan {
    int t0, t1;
    int64_t s0, s1, q0, q1;      // sample ranges
    int64_t ps0, ps1, pq0, pq1;  // padded row ranges
    int64_t ls0, ls1, lq0, lq1;  // lookup ranges
};

__global__ void gather_task_lookup_offsets(const int64_t* toff, const int64_t* bag_offsets, int F, int T, int64_t* out) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t <= T) out[t] = bag_offsets[toff[t] * F];
}

static void build_tiles(const std::vector<int64_t>& poff, int t0, int t1, int bm, std::vector<int32_t>& row_off,
                        std::vector<int32_t>& tg, std::vector<int32_t>& tm) {
    row_off.clear(); tg.clear(); tm.clear();
    const int64_t base = poff[t0];
    for (int t = t0; t < t1; ++t) {
        row_off.push_back((int32_t)(poff[t] - base));
        const int n = (int)(poff[t + 1] - poff[t]);
        for (int m = 0; m < n; m += bm) {
            tg.push_back(t - t0);
            tm.push_back(m);
        }
    }
    row_off.push_back((int32_t)(poff[t1] - base));
}

// What a call sends to the device lives here until the stream has taken it.
struct HostImages {
    hipStream_t st = nullptr;
    std::vector<std::vector<char>> held;
    ~HostImages() { if (!held.empty()) (void)hipStreamSynchronize(st); }
};
// Arrays that lie side by side in the workspace, sent in one copy (a copy of a few hundred bytes costs what a launch does).
struct Upload {
    char* dev;
    std::vector<char> host;
    template <typename T>
    void put(T* dst, const T* src, size_t n) {
        const size_t off = (size_t)(reinterpret_cast<char*>(dst) - dev);
        if (host.size() < off + n * sizeof(T)) host.resize(off + n * sizeof(T));
        if (n > 0) memcpy(host.data() + off, src, n * sizeof(T));
    }
    template <typename T>
    void put(T* dst, const std::vector<T>& v) { put(dst, v.data(), v.size()); }
    int send(gm_ctx* c, HostImages& keep) {
        keep.st = c->stream;
        keep.held.push_back(std::move(host));
        const std::vector<char>& v = keep.held.back();
        if (!v.empty()) HIPCHK(c, hipMemcpyAsync(dev, v.data(), v.size(), hipMemcpyHostToDevice, c->stream));
        return GM_OK;
    }
};

enum { PAIR_ROWS = 512, PAIR_ROWS_FEW = 1024 };
struct Batch {  // host-side description of one call
    int T;
    const gm_set *sup, *qry;
    std::vector<int64_t> poff_s, poff_q;  // padded row offsets per task, whole batch
    std::vector<int64_t> ls, lq;          // lookup offsets per task (filled when several waves are needed)
    bool table = false;                   // table-shaped sparse output: every wave sorts and reduces its own lookups
    int pair_rows = PAIR_ROWS;            // a task of at most so many rows in each set goes through pair-count matrices
    bool tight = false;                   // a call without a chain keeps no steps' activations or gradients (see first_order_keeps)
    BatchBufs b;
    HostImages images;
};

// The lookups of samples [s0, s1) of the support set and [q0, q1) of the query set, ordered by global row and cut into
// one segment per distinct row.  Gradient-buffer rows are row0_* + the batch-wide padded row of the sample (mod 2^32).
struct SortRange {
    int64_t s0, s1, q0, q1;      // samples
    int64_t ls0, ls1, lq0, lq1;  // their lookups
    u32 row0_s, row0_q;
};

static const ValEnc kPlainVals{0, 0, 0u};

enum { ORDER_SORT = 1, ORDER_SEGMENTS = 2, ORDER_ALL = 3 };

// parts: the sort (keys built, ordered by row: left in so.keys / so.vals), the segments (one per distinct row, from
// the sorted keys), or both
static int global_order(gm_ctx* c, Batch& B, SortBufs& so, const SortRange& r, int64_t* emb_rows, int64_t* seg_counts,
                        int64_t capacity, int64_t* n_rows, bool on_side = false, ValEnc enc = kPlainVals, int parts = ORDER_ALL) {
    hipStream_t st = on_side ? c->side : c->stream;
    u32* status = on_side ? c->d_status_side : c->d_status;
    const int F = c->F;
    const gm_set *sup = B.sup, *qry = B.qry;
    BatchBufs& b = B.b;
    const int64_t n_s = r.ls1 - r.ls0, nnz = n_s + (r.lq1 - r.lq0);
    Prof p(c, "global_sort", 0, 0, st, true);
    if (parts & ORDER_SORT) {
        if (F > 0) {
            launch_build_keys(st, F, c->d_field_base, sup->bag_offsets + r.s0 * F, sup->indices, (r.s1 - r.s0) * F, r.ls0,
                              b.prow_s + r.s0, r.row0_s, enc, so.keys, so.vals);
            launch_build_keys(st, F, c->d_field_base, qry->bag_offsets + r.q0 * F, qry->indices, (r.q1 - r.q0) * F, r.lq0,
                              b.prow_q + r.q0, r.row0_q, enc, so.keys + n_s, so.vals + n_s);
        }
        int bits = 1;
        while (((int64_t)1 << bits) < c->field_base[c->F]) ++bits;
        const int passes = launch_radix_sort(st, so.keys, so.vals, so.keys_tmp, so.vals_tmp, nnz, bits, so.hist);
        // algorithmic bytes: keys built from the lookups (4 B index read, 8 B of key and value written, 8 B of offsets per bag),
        // 20 B per key and radix pass (the key read for the digit counts; key and value read and written by the scatter)
        p.p.bytes += (double)nnz * (12.0 + 20.0 * passes) + 8.0 * F * ((r.s1 - r.s0) + (r.q1 - r.q0));
        if (passes & 1) {
            std::swap(so.keys, so.keys_tmp);   // an odd number of passes leaves the result in the second pair of buffers
            std::swap(so.vals, so.vals_tmp);
        }
    }
    // the table-shaped output adds every segment to the row its key names: no segment numbers, no row list
    if ((parts & ORDER_SEGMENTS) && n_rows) {
        p.p.bytes += 4.0 * (double)nnz;   // the sorted keys read once more
        launch_segments(st, so.keys, nnz, seg_chunk(nnz, F, c->D), so.keys_tmp, so.scan_tmp, emb_rows, so.seg_start, seg_counts, capacity,
                        n_rows, status);
    }
    return GM_OK;
}

// Asks run_index_wave to take the wave's per-(task, field) dictionaries from the (field, row) order of its lookups --
// the order the sparse meta-gradient needs anyway -- instead of sorting every (task, field) by itself: the wave's
// lookups are ordered by row first (left in `so` for the segment reduction), one more stable pass orders them by task,
// and the dictionaries, the lookup lists and the overlap join are read off that list.  Applies when the sort's range is
// exactly the wave and a gradient-buffer row, a field number and a position in a bag fit 32 bits together.
struct JoinReq {
    SortBufs* so = nullptr;
    SortRange range{};
    int64_t* emb_rows = nullptr;     // row-list output: the segments are cut right after the sort (n_rows null: table-shaped output)
    int64_t* seg_counts = nullptr;
    int64_t capacity = 0;
    int64_t* n_rows = nullptr;
    int64_t n_sup_rows = 0, n_qry_rows = 0;   // padded rows of the wave's two sets (gradient-buffer rows: support first)
    bool slots = false;              // the slot of every lookup is wanted whatever the row path
    bool pair_only = false;          // every task of the wave is planned for the pair-count matrices (which do not read those slots)
    bool used = false;               // out: the wave's lookups are ordered, `enc` says how their values read
    ValEnc enc = kPlainVals;
};

static int64_t uniform_rows(const gm_ctx* c) {   // rows of every table when they are all of one size, else -1
    for (int f = 1; f < c->F; ++f)
        if (c->rows[f] != c->rows[0]) return -1;
    return c->F > 0 ? c->rows[0] : -1;
}

static int bits_for(int64_t n) {   // bits that hold every value below n
    int b = 0;
    while (((int64_t)1 << b) < n) ++b;
    return b;
}

// The per-(task, field) dictionaries, lookup lists and overlap join of a wave, every (task, field) sorted by itself in LDS
// (w.cnt_* / w.base_* are in place).
static void sort_task_fields(gm_ctx* c, const Batch& B, const WavePlan& wp, WaveBufs& w, int max_tf) {
    const int F = c->F, Tw = wp.t1 - wp.t0;
    TfSortArgs a;
    a.F = F; a.t0 = wp.t0; a.Tw = Tw;
    a.sup = make_view(B.sup, B.b.toff_s, wp.s0, wp.ls0); a.qry = make_view(B.qry, B.b.toff_q, wp.q0, wp.lq0);
    a.field_base = c->d_field_base;
    a.cnt_sup = w.cnt_s; a.base_sup = w.base_s; a.cnt_qry = w.cnt_q; a.base_qry = w.base_q;
    a.n_slots = w.n_slots; a.slot_rows = w.slot_rows; a.slot_start = w.slot_start;
    a.sup_sorted = w.sup_sorted; a.sup_slot = w.sup_slot; a.qry_slot = w.qry_slot;
    a.qry_sorted = w.qry_sorted; a.qseg_lo = w.qseg_lo; a.qseg_hi = w.qseg_hi; a.status = c->d_status;
    a.sup_rows = B.b.prow_s; a.sup_row_base = (int32_t)wp.ps0;
    a.qry_rows = B.b.prow_q; a.qry_row_base = (int32_t)wp.pq0;
    Prof p(c, "tf_sort", 12.0 * ((wp.ls1 - wp.ls0) + (wp.lq1 - wp.lq0)), 0);
    int64_t max_set_rows = 0;
    for (int t = wp.t0; t < wp.t1; ++t)
        max_set_rows = std::max(max_set_rows, std::max(B.sup->task_offsets[t + 1] - B.sup->task_offsets[t],
                                                       B.qry->task_offsets[t + 1] - B.qry->task_offsets[t]));
    launch_tf_sort(c->stream, a, max_tf, (int)std::min<int64_t>(max_set_rows, 1 << 30));
    w.slots_written = true;
}

// bags of the largest of tasks [t0, t1), both sets together
static int64_t most_bags(const gm_set* sup, const gm_set* qry, int t0, int t1, int F) {
    const int64_t *s = sup->task_offsets, *q = qry->task_offsets;
    int64_t most = 0;
    for (int t = t0; t < t1; ++t) most = std::max(most, (s[t + 1] - s[t]) + (q[t + 1] - q[t]));
    return most * F;
}

static int run_index_wave(gm_ctx* c, Batch& B, const WavePlan& wp, WaveBufs& w, int* cap_out = nullptr,
                          int* max_bag_out = nullptr, int* max_tf_out = nullptr, JoinReq* jr = nullptr) {
    hipStream_t st = c->stream;
    const int F = c->F, Tw = wp.t1 - wp.t0;
    if (jr) jr->used = false;
    if (F == 0 || Tw == 0) return GM_OK;
    const int64_t TF = (int64_t)Tw * F;
    SetView vs = make_view(B.sup, B.b.toff_s, wp.s0, wp.ls0), vq = make_view(B.qry, B.b.toff_q, wp.q0, wp.lq0);
    {
        Prof p(c, "tf_count", 8.0 * ((wp.s1 - wp.s0) + (wp.q1 - wp.q0)) * F + 4.0 * ((wp.ls1 - wp.ls0) + (wp.lq1 - wp.lq0)), 0);
        launch_tf_count(st, F, wp.t0, Tw, most_bags(B.sup, B.qry, wp.t0, wp.t1, F), ((wp.s1 - wp.s0) + (wp.q1 - wp.q0)) * F, vs, vq, c->d_field_base, B.sup->nnz, B.qry->nnz, uniform_rows(c), w.cnt_s, w.cnt_q, c->d_status, true);
    }
    u32 hs[ST_WORDS];
    int rc = read_status(c, hs);
    if (rc != GM_OK) return rc;
    if (hs[ST_BAD_INDEX]) return fail(c, GM_ERR_INDEX, "index outside its table, or bag_offsets not monotone / beyond nnz");
    if (hs[ST_TOO_LARGE])
        return fail(c, GM_ERR_CAPACITY, "a bag has more than 65535 lookups, or a task more than 65536 samples in one set");
    int cap = 1024;
    while (cap < (int)hs[ST_MAX_TF]) cap <<= 1;
    if (cap_out) *cap_out = cap;
    if (max_bag_out) *max_bag_out = (int)hs[ST_MAX_BAG];
    if (max_tf_out) *max_tf_out = (int)hs[ST_MAX_TF];
    if (!c->adapt_rows) return GM_OK;   // validated; no row arithmetic, so no per-(task, field) dictionaries
    if (cap > tf_sort_max_cap())
        return fail(c, GM_ERR_CAPACITY, "a (task, field) has %u lookups in one set; the limit is %d", hs[ST_MAX_TF],
                    tf_sort_max_cap());
    const double tf_bytes = 12.0 * ((wp.ls1 - wp.ls0) + (wp.lq1 - wp.lq0));
    // ---- the dictionaries read off the row order of the wave's lookups
    bool join = jr && jr->so && c->index_path != 1;
    ValEnc enc = kPlainVals;
    if (join) {
        const int pbits = bits_for((int64_t)hs[ST_MAX_BAG]), fbits = bits_for(F);
        const int rbits = bits_for(jr->n_sup_rows + jr->n_qry_rows);
        if (rbits + fbits + pbits > 32 || (task_sort_passes(Tw) > 1 && !w.tmid_keys)) join = false;
        else enc = ValEnc{fbits + pbits > 0 ? fbits + pbits : 1, pbits, (1u << fbits) - 1u};
        if (join && enc.rshift + rbits > 32) join = false;   // (no field and no position bits: the shift of 1 marks the form)
    }
    if (jr && c->index_path == 2 && !join)
        return fail(c, GM_ERR_CAPACITY, "index_path 2: the wave's lookups cannot be ordered as one list of 32-bit bit-field values");
    const bool by_field = join && c->sort_fields;
    if (!by_field) launch_scan_u32_pair(st, w.cnt_s, w.base_s, w.cnt_q, w.base_q, TF, w.scan_tmp);
    if (join) {
        SortBufs& so = *jr->so;
        if (by_field) {
            // the keys field after field (the per-(task, field) counts give every lookup its place), then every field's
            // range sorted by its row bits alone
            const int64_t nw = (wp.ls1 - wp.ls0) + (wp.lq1 - wp.lq0);
            Prof p(c, "global_sort", 0, 0, st, true);
            FieldKeysArgs fa;
            memset(&fa, 0, sizeof fa);
            fa.F = F; fa.t0 = wp.t0; fa.Tw = Tw; fa.sup = vs; fa.qry = vq; fa.field_base = c->d_field_base;
            fa.cnt_s = w.cnt_s; fa.cnt_q = w.cnt_q; fa.base_s = w.base_s; fa.base_q = w.base_q; fa.fm_off_s = w.fm_off_s; fa.fm_off_q = w.fm_off_q;
            fa.prow_s = B.b.prow_s; fa.prow_q = B.b.prow_q; fa.row0_s = jr->range.row0_s; fa.row0_q = jr->range.row0_q;
            fa.enc = enc; fa.keys = so.keys; fa.vals = so.vals;
            launch_build_keys_by_field(st, fa, w.field_tab, w.scan_tmp, nw, (int)hs[ST_MAX_BAG]);
            int64_t max_rows = 1;
            for (int f = 0; f < F; ++f) max_rows = std::max(max_rows, c->field_base[f + 1] - c->field_base[f]);
            const SegTab seg = field_seg_tab(F, w.field_tab);
            const int passes = launch_radix_sort(st, so.keys, so.vals, so.keys_tmp, so.vals_tmp, nw, std::max(1, bits_for(max_rows)), so.hist, &seg);
            p.p.bytes += (double)nw * (12.0 + 20.0 * passes) + 8.0 * F * ((wp.s1 - wp.s0) + (wp.q1 - wp.q0));
            if (passes & 1) {
                std::swap(so.keys, so.keys_tmp);
                std::swap(so.vals, so.vals_tmp);
            }
        } else {
            global_order(c, B, so, jr->range, nullptr, nullptr, jr->capacity, nullptr, false, enc, ORDER_SORT);
        }
        {
            Prof p(c, "tf_sort", tf_bytes, 0);
            const int64_t nw = (wp.ls1 - wp.ls0) + (wp.lq1 - wp.lq0);
            int uniform_shift = -1;   // all tasks of the wave of one power-of-two size (padded rows, both sets alike)?
            {
                const int64_t r0 = B.poff_s[wp.t0 + 1] - B.poff_s[wp.t0];
                bool same = r0 > 0 && (r0 & (r0 - 1)) == 0;
                for (int t = wp.t0; t < wp.t1 && same; ++t)
                    same = B.poff_s[t + 1] - B.poff_s[t] == r0 && B.poff_q[t + 1] - B.poff_q[t] == r0;
                if (same) uniform_shift = bits_for(r0);
            }
            TaskOf tk{w.row_task_s, w.row_task_q, (u32)jr->n_sup_rows, (u32)(jr->n_sup_rows + jr->n_qry_rows), enc.rshift, uniform_shift};
            launch_task_sort(st, so.keys, so.vals, w.tmid_keys, w.tmid_vals, so.keys_tmp, so.vals_tmp, nw, Tw, tk, so.hist);
            TfJoinArgs a;
            memset(&a, 0, sizeof a);
            a.F = F; a.Tw = Tw; a.keys = so.keys_tmp; a.vals = so.vals_tmp;
            a.cnt_s = w.cnt_s; a.base_s = w.base_s; a.cnt_q = w.cnt_q; a.base_q = w.base_q;
            a.rshift = enc.rshift; a.pshift = enc.pshift; a.n_sup_rows = (u32)jr->n_sup_rows;
            a.n_slots = w.n_slots; a.slot_rows = w.slot_rows; a.slot_start = w.slot_start;
            a.sup_sorted = w.sup_sorted; a.qry_sorted = w.qry_sorted; a.qseg_lo = w.qseg_lo; a.qseg_hi = w.qseg_hi;
            // the slot of every lookup (scattered 4-byte writes) only where the sparse row kernel may read it
            const bool write_slots = jr->slots || !jr->pair_only || cap > PAIR_MAX_CAP || (int)hs[ST_MAX_BAG] > PAIR_MAX_BAG;
            a.sup_slot = write_slots ? w.sup_slot : nullptr;
            a.qry_slot = write_slots ? w.qry_slot : nullptr;
            w.slots_written = write_slots;
            a.bag_s = B.sup->bag_offsets; a.bag_q = B.qry->bag_offsets;
            a.sample0_s = wp.s0; a.sample0_q = wp.q0; a.lookup0_s = wp.ls0; a.lookup0_q = wp.lq0;
            a.n_lookups_s = wp.ls1 - wp.ls0; a.n_lookups_q = wp.lq1 - wp.lq0;
            a.row_off_s = w.row_off_s; a.row_off_q = w.row_off_q; a.real_off_s = w.real_off_s; a.real_off_q = w.real_off_q;
            launch_tf_join(st, a);
        }
        // (the list in task order is done with: the second pair of buffers is free for the segment scan)
        if (jr->n_rows)
            global_order(c, B, so, jr->range, jr->emb_rows, jr->seg_counts, jr->capacity, jr->n_rows, false, enc, ORDER_SEGMENTS);
        jr->used = true;
        jr->enc = enc;
        return GM_OK;
    }
    w.slots_written = true;
    sort_task_fields(c, B, wp, w, (int)hs[ST_MAX_TF]);
    return GM_OK;
}

static SortRange whole_batch_range(const Batch& B) {
    return SortRange{0, B.sup->n_samples, 0, B.qry->n_samples, 0, B.sup->nnz, 0, B.qry->nnz, 0u, (u32)B.poff_s[B.T]};
}

static inline int64_t pad64(int64_t n) { return (n + 63) & ~(int64_t)63; }

// What decides between matrices and factors of the chain's direction (factor_rows): the thin products' rate over padded sizes,
// the matrices' over bytes, the memory-side cache, and the most rows of a task (a slot of the thin products is that wide).
static constexpr double FACTOR_RATE = 2.5e14, MATRIX_RATE = 4.5e12, FACTOR_CACHE = 2.56e8;
enum { FACTOR_MOST_ROWS = 2048 };

// Whether a task's row arithmetic should go through pair-count matrices: the product costs
// n_out * n_in * D per (task, field) against lookups * D for the sparse kernel, on units that are far
// faster, so it pays while the task is moderately small.
static bool task_pair_ok(const gm_ctx* c, const Batch& B, int t, int K) {
    if (c->row_path == 1 || K <= 0 || c->F == 0 || c->D % 32 != 0 || !c->adapt_rows) return false;
    const int64_t mx = std::max(B.sup->task_offsets[t + 1] - B.sup->task_offsets[t], B.qry->task_offsets[t + 1] - B.qry->task_offsets[t]);
    return mx > 0 && mx <= (c->row_path == 2 ? (int)PAIR_ROWS_FEW : B.pair_rows);
}

// A few tasks of 513 to 1024 rows among smaller ones go the others' way: for them alone the sparse kernel would run at every
// hop, a workgroup a (task, field), as long as the largest takes.  Among 700 tasks of a median 32 rows two of them, 16 launches
// of 100 us: a step of 28.9 ms takes 27.9; four of them (a third of the others' matrices) 28.8 / 27.7; 24 tasks of 700 rows among 30 of
// 500, 26 fields 9.1 / 7.8 ms, 10 of 1000 among 60 of 300 8.3 / 7.5.  Where lookups are few (up to three a bag: 32 tasks x 600 rows x 26
// fields 2.80 / 2.98 ms with matrices; six: 8.67 / 8.39) or the (task, field)s do not fill the device (8 tasks x 700 rows x 26 fields 2.10
// / 2.16 ms; 16 tasks, which do, 3.55 / 2.82) the sparse kernel is the faster one; and they shall take no more memory than the others.
// A rule on the batch alone: the two ways add in different orders, and losses and row gradients shall not depend on the workspace,
// on the waves or on whether training iterations overlap.  (A workspace that cannot hold such a task's matrices at all: plan_waves.)
static int pair_rows(const gm_ctx* c, const Batch& B) {
    const double bags = (double)(B.sup->n_samples + B.qry->n_samples) * c->F;
    if ((double)(B.sup->nnz + B.qry->nnz) < 4.0 * bags || (int64_t)B.T * c->F < c->n_cus) return PAIR_ROWS;
    double few = 0, others = 0;
    for (int t = 0; t < B.T; ++t) {
        const int64_t ns = B.sup->task_offsets[t + 1] - B.sup->task_offsets[t], nq = B.qry->task_offsets[t + 1] - B.qry->task_offsets[t];
        const int64_t mx = std::max(ns, nq);
        if (mx > PAIR_ROWS_FEW) continue;
        (mx > PAIR_ROWS ? few : others) += (double)pad64(ns) * (double)(pad64(ns) + pad64(nq));
    }
    return few > 0 && few <= others ? PAIR_ROWS_FEW : PAIR_ROWS;
}

// Where every task's pair-count matrices begin (kind by kind, fields back to back; nothing for a task
// that takes the sparse kernel), in PAIR_BLOCKs, which every matrix is a whole number of; returns the total in bytes.
static int64_t pair_layout(const gm_ctx* c, const Batch& B, const WavePlan& p, int K, bool ss, bool sq,
                           std::vector<u32>* off_ss, std::vector<u32>* off_qs, std::vector<u32>* off_sq,
                           std::vector<u32>* path) {
    int64_t acc = 0;
    for (int t = p.t0; t < p.t1; ++t) {
        const bool ok = task_pair_ok(c, B, t, K);
        const int64_t ns = ok ? pad64(B.sup->task_offsets[t + 1] - B.sup->task_offsets[t]) : 0;
        const int64_t nq = ok ? pad64(B.qry->task_offsets[t + 1] - B.qry->task_offsets[t]) : 0;
        if (path) path->push_back(ok ? 1u : 0u);
        if (off_ss) off_ss->push_back((u32)(acc / PAIR_BLOCK));
        if (ss) acc += c->F * ns * ns;
        if (off_qs) off_qs->push_back((u32)(acc / PAIR_BLOCK));
        acc += c->F * nq * ns;
        if (off_sq) off_sq->push_back((u32)(acc / PAIR_BLOCK));
        if (sq) acc += c->F * ns * nq;
    }
    return acc;
}

// Whether the chain's direction stays factors (then: rows of the batch's largest task): where the thin products cost less than
// writing, reading and summing the matrices, and these do not stay in the memory-side cache anyway.  A rule on the whole batch,
// so that the waves it is cut into do not change results.
static int factor_rows(const gm_ctx* c, const Batch& B, int bm, int K, int order) {
    if (!c->mlp_dtype || order != 2 || K < 1 || factor_slots(K) > GEMM_EXT || c->L < 2 || bm != 64 || c->chain_factors == 1) return 0;
    double widths = 0, weights = 0;
    for (int l = 1; l < c->L; ++l) {
        widths += c->ld[l - 1] + c->ld[l];
        weights += (double)c->ld[l - 1] * c->ld[l];
    }
    double ss = 0, sq = 0, rows = 0;
    int most = 0;
    for (int t = 0; t < B.T; ++t) {
        const int64_t ns = B.poff_s[t + 1] - B.poff_s[t], nq = B.poff_q[t + 1] - B.poff_q[t];
        most = (int)std::max<int64_t>(most, std::max(ns, nq));
        rows += (double)std::max(ns, nq);
        ss += (double)pad64(ns) * (double)pad64(ns);
        sq += (double)pad64(ns) * (double)pad64(nq);
    }
    if (most <= 0 || most > FACTOR_MOST_ROWS) return 0;
    if (c->chain_factors == 2) return most;
    // (of every step: the query pass's factor and two of each later step; both directions; the second thin product has two parts)
    const double flops = 2.0 * 3.0 * widths * (K * (K - 1) * ss + K * sq);
    const double bytes = weights * B.T * (6.0 + 10.0 * (K - 1) + 4.0 * K + 4.0);   // written, updated, read, summed
    const double room = rows * (4.0 * round_up(most, 64) * factor_slots(K) + 2.0 * (K - 1) * (c->ld[0] + 2.0 * widths));
    return flops / FACTOR_RATE < bytes / MATRIX_RATE && weights * B.T * 6.0 > FACTOR_CACHE && room < 2.0 * weights * B.T ? most : 0;
}

// Steps whose input gradients are kept until the last one: the query set's update X - alpha M (Z_0 + .. + Z_k) is then one hop instead of
// one a step, each of which reads M and X and writes X.  Two steps, or three with bf16 operands: the buffers are ones that nothing
// uses before: the support rows of the gradient buffer, and the chain's fp32 direction or, without a chain, Spare.
static int query_sum(const gm_ctx* c, int K) { return K == 2 || (K == 3 && c->mlp_dtype) ? K : 0; }

// bf16, 2..GEMM_MAX_PAIRS inner steps: every step's weights straight from the meta parameters and the gradients of all steps so far, bf16
// copy only.  Second order keeps the steps' activations and deltas for the chain anyway.  First order does so where the extra products
// (k + 1 of step k instead of one) cost less than the fp32 master, written and read again by the next step: with r rows a task
// r K (K - 1) operations a weight against 8 (K - 1) bytes, so K r decides whatever the layers and the steps.  Whole steps with the master and
// without, 200 tasks, 1677-512-256: K r = 290 2.62 / 2.47, 3.07 / 2.77 and 3.80 / 3.38 ms with two, three and four steps, 600 3.62 / 3.55, 4.13 / 3.97, 4.63
// / 4.42, 800 4.56 / 4.53, 4.88 / 4.80, 5.26 / 5.13, 1024 5.32 / 5.33, 5.79 / 5.80, 5.72 / 5.63; 64 tasks, 4109-1024-512-256: 600 4.31 / 4.23, 4.97 / 4.78,
// 5.75 / 5.46, 800 4.96 / 4.97, 5.95 / 5.93, 6.18 / 6.25, 1024 5.53 / 5.62, 6.37 / 6.46, 6.85 / 6.85, 2000 10.03 / 10.89 (four); 200 tasks,
// 1677-128-64: 290 1.63 / 1.61, 1.66 / 1.61, 1.95 / 1.87, 600 2.47 / 2.47, 2.52 / 2.50, 2.62 / 2.63, 800 and more within 1 % either way.
enum { FROM_META_ROWS = 800 };
static bool theta_from_meta(const gm_ctx* c, int64_t T, int64_t n_support, int K, int order) {
    if (!c->mlp_dtype || K < 2 || K > GEMM_MAX_PAIRS || !c->theta_from_meta || T <= 0) return false;
    return order == 2 || (c->L > 1 && (double)K * n_support < FROM_META_ROWS * (double)T);
}

// What a call without a chain keeps of its inner steps: only what spare memory holds if the batch runs as one wave, so that no call needs
// more workspace for it (201 tasks of 150 + 243 rows, 1677-512-256, three steps: 0.6 of 6 GB); the input gradients first, which save more.
// A rule on the batch.  An uneven wave of several may need some beyond the spare memory (then see plan_waves).
static FirstOrder first_order_keeps(const gm_ctx* c, int64_t T, int64_t n_support, int64_t Ps, int64_t Pq, int K) {
    auto fits = [&](const FirstOrder& k) {
        Arena none, query;
        query.cap = ~(size_t)0 >> 1;
        std::vector<Act> A, D;
        Spare sp = make_spare(c, T, Pq, nullptr, alloc_query(c, query, A, D, Pq), nullptr, nullptr, &none);
        WaveBufs w;
        w.steps.resize(k.acts ? K : 0);
        alloc_first_order(c, sp, w, Ps, K, k.grads, k.acts);
        return !none.overflow;
    };
    FirstOrder k{query_sum(c, K) > 2 && c->F > 0 && c->D % 32 == 0 && c->adapt_rows && c->row_path != 1, false};
    if (k.grads && !fits(k)) k.grads = false;
    k.acts = theta_from_meta(c, T, n_support, K, 1);
    if (k.acts && !fits(k)) k.acts = false;
    return k;
}

static WaveDims wave_dims(const gm_ctx* c, const Batch& B, const WavePlan& p, int bm, int K, int order) {
    WaveDims d;
    d.table = B.table;
    d.factor_ld = factor_rows(c, B, bm, K, order);
    FirstOrder first{false, false};
    if (order == 1 && !B.tight) first = first_order_keeps(c, B.T, B.sup->n_samples, B.poff_s[B.T], B.poff_q[B.T], K);
    d.from_meta = order == 1 ? first.acts : theta_from_meta(c, B.T, B.sup->n_samples, K, order);
    for (int t = p.t0; t < p.t1; ++t) {
        if (task_pair_ok(c, B, t, K)) {
            d.pair = true;
            const int64_t ns = B.sup->task_offsets[t + 1] - B.sup->task_offsets[t], nq = B.qry->task_offsets[t + 1] - B.qry->task_offsets[t];
            if (std::max(ns, nq) > HOP_SMALL) {
                d.hop_tiles_s += (ns + 255) / 256;
                d.hop_tiles_q += (nq + 255) / 256;
            }
        } else d.any_sparse = true;
    }
    if (d.pair) {
        d.pair_ss = K >= 2;
        d.pair_sq = order == 2;
        d.pair_bytes = pair_layout(c, B, p, K, d.pair_ss, d.pair_sq, nullptr, nullptr, nullptr, nullptr);
        d.query_sum = query_sum(c, K);
        if (order == 1 && d.query_sum > 2 && !first.grads) d.query_sum = 0;   // (two steps' have buffers that nobody else needs)
    }
    d.Tw = p.t1 - p.t0;
    d.Ss = p.s1 - p.s0; d.Sq = p.q1 - p.q0; d.Ps = p.ps1 - p.ps0; d.Pq = p.pq1 - p.pq0;
    d.nnz_s = p.ls1 - p.ls0; d.nnz_q = p.lq1 - p.lq0;
    int64_t ms = 0, mq = 0;
    for (int t = p.t0; t < p.t1; ++t) {
        ms += (B.poff_s[t + 1] - B.poff_s[t] + bm - 1) / bm;
        mq += (B.poff_q[t + 1] - B.poff_q[t] + bm - 1) / bm;
    }
    d.mt_s = (int)ms; d.mt_q = (int)mq;
    return d;
}

// Row tile of the forward and backward products: by the tasks' average size and how the first layer's tiles fill the device.
static int pick_bm(const gm_ctx* c, const Batch& B) {
    if (B.T == 0) return 64;
    const int64_t avg = (B.poff_s[B.T] + B.poff_q[B.T]) / (2 * (int64_t)B.T);
    if (!c->mlp_dtype) return 64;
    return row_tile(c, avg >= 192 ? 256 : (avg >= 96 ? 128 : 64), c->ld[1], c->ld[0], [&](int bm) {
        int64_t m = 0;
        for (int t = 0; t < B.T; ++t) m += (B.poff_s[t + 1] - B.poff_s[t] + bm - 1) / bm;
        return m;
    });
}

// splits the tasks into waves that fit `avail` bytes of workspace
static int plan_waves(gm_ctx* c, Batch& B, size_t avail, int K, int order, int bm, std::vector<WavePlan>& plans) {
    const int F = c->F, T = B.T;
    const gm_set *sup = B.sup, *qry = B.qry;
    B.ls.assign(T + 1, 0);
    B.lq.assign(T + 1, 0);
    bool have_offsets = false;
    auto fetch = [&]() -> int {
        if (have_offsets || F == 0) return GM_OK;
        int64_t* d = reinterpret_cast<int64_t*>(B.b.so.hist);  // scratch: the histogram area is free until the global sort
        hipLaunchKernelGGL(gather_task_lookup_offsets, dim3((T + 256) / 256), dim3(256), 0, c->stream, B.b.toff_s,
                           sup->bag_offsets, F, T, d);
        hipLaunchKernelGGL(gather_task_lookup_offsets, dim3((T + 256) / 256), dim3(256), 0, c->stream, B.b.toff_q,
                           qry->bag_offsets, F, T, d + T + 1);
        HIPCHK(c, hipMemcpyAsync(B.ls.data(), d, (T + 1) * sizeof(int64_t), hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipMemcpyAsync(B.lq.data(), d + T + 1, (T + 1) * sizeof(int64_t), hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        for (int t = 0; t <= T; ++t)
            if (B.ls[t] < 0 || B.ls[t] > sup->nnz || B.lq[t] < 0 || B.lq[t] > qry->nnz ||
                (t && (B.ls[t] < B.ls[t - 1] || B.lq[t] < B.lq[t - 1])))
                return fail(c, GM_ERR_INDEX, "bag_offsets not monotone / beyond nnz at a task boundary");
        have_offsets = true;
        return GM_OK;
    };
    B.pair_rows = pair_rows(c, B);
    // Waves of (nearly) equal numbers of tasks: the fewest waves whose every wave fits.
    const int max_per = std::min(std::max(T, 1), most_wave_tasks(c));
    const int fewest = (std::max(T, 1) + max_per - 1) / max_per;
    int n_waves = fewest;
    const FirstOrder keeps = order == 1 ? first_order_keeps(c, T, sup->n_samples, B.poff_s[T], B.poff_q[T], K) : FirstOrder{false, false};
    while (true) {
        const int per = (std::max(T, 1) + n_waves - 1) / n_waves;
        plans.clear();
        bool fits = true;
        if (per < T) {
            int rc = fetch();
            if (rc != GM_OK) return rc;
        } else {
            B.ls[T] = sup->nnz;
            B.lq[T] = qry->nnz;
        }
        for (int t0 = 0; t0 < T || (T == 0 && plans.empty()); t0 += per) {
            WavePlan p;
            p.t0 = t0;
            p.t1 = std::min(T, t0 + per);
            p.s0 = sup->task_offsets[p.t0]; p.s1 = sup->task_offsets[p.t1];
            p.q0 = qry->task_offsets[p.t0]; p.q1 = qry->task_offsets[p.t1];
            p.ps0 = B.poff_s[p.t0]; p.ps1 = B.poff_s[p.t1]; p.pq0 = B.poff_q[p.t0]; p.pq1 = B.poff_q[p.t1];
            p.ls0 = B.ls[p.t0]; p.ls1 = B.ls[p.t1]; p.lq0 = B.lq[p.t0]; p.lq1 = B.lq[p.t1];
            plans.push_back(p);
            // a wave's lookups are numbered in 32 bits
            if ((p.ls1 - p.ls0) + (p.lq1 - p.lq0) >= ((int64_t)1 << 31)) { fits = false; break; }
            Arena ar;
            ar.cap = avail;
            WaveBufs w;
            alloc_wave(c, ar, w, wave_dims(c, B, p, bm, K, order), K, order);
            if (ar.overflow) { fits = false; break; }
            if (T == 0) break;
        }
        if (fits) return GM_OK;
        // (a wave less is worth more than what the steps keep)
        B.tight = !B.tight && (keeps.grads || keeps.acts);
        if (B.tight) continue;
        if (per == 1) {
            if (B.pair_rows == PAIR_ROWS) return fail(c, GM_ERR_WORKSPACE, "workspace of %zu bytes cannot hold one task", c->ws_bytes);
            B.pair_rows = PAIR_ROWS;   // (a large task does not fit with its matrices, not even alone)
            n_waves = fewest;
            continue;
        }
        n_waves = std::min(std::max(T, 1), std::max(n_waves + 1, n_waves + n_waves / 16));
    }
}

// batch-level set-up shared by gm_meta_step and gm_index_prep
// ar: where the index-side buffers go; dense_ar: where the batch's dense buffers go (null: the caller places them)
static int begin_batch(gm_ctx* c, Batch& B, Arena& ar, int64_t capacity, bool need_gx, Arena* dense_ar) {
    const int T = B.T, pad = c->row_pad;
    B.poff_s.assign(T + 1, 0);
    B.poff_q.assign(T + 1, 0);
    for (int t = 0; t < T; ++t) {
        B.poff_s[t + 1] = B.poff_s[t] + round_up64(B.sup->task_offsets[t + 1] - B.sup->task_offsets[t], pad);
        B.poff_q[t + 1] = B.poff_q[t] + round_up64(B.qry->task_offsets[t + 1] - B.qry->task_offsets[t], pad);
    }
    if ((B.poff_s[T] + B.poff_q[T]) * (int64_t)std::max(c->F, 1) >= ((int64_t)1 << 32))
        return fail(c, GM_ERR_ARG, "more than 2^32 (row, field) pairs in one call");
    // (no batch-wide sort when every wave reduces its own lookups into a table)
    alloc_batch_index(c, ar, B.b, T, B.sup->n_samples, B.qry->n_samples, B.table ? 0 : B.sup->nnz + B.qry->nnz, capacity, need_gx);
    if (dense_ar) alloc_batch_dense(c, *dense_ar, B.b, T, B.poff_s[T], B.poff_q[T], need_gx);
    if (ar.overflow || (dense_ar && dense_ar->overflow))
        return fail(c, GM_ERR_WORKSPACE, "workspace too small for the batch-level buffers (%zu needed)", ar.off);
    hipStream_t st = c->stream;
    std::vector<int32_t> ps(B.poff_s.begin(), B.poff_s.end()), pq(B.poff_q.begin(), B.poff_q.end());
    Upload up{reinterpret_cast<char*>(B.b.toff_s), {}};
    up.put(B.b.toff_s, B.sup->task_offsets, T + 1);
    up.put(B.b.toff_q, B.qry->task_offsets, T + 1);
    up.put(B.b.prow_off_s, ps);
    up.put(B.b.prow_off_q, pq);
    int rc = up.send(c, B.images);
    if (rc != GM_OK) return rc;
    launch_expand_tasks(st, T, ExpandJobs{2, {{B.b.toff_s, nullptr, B.b.prow_off_s, B.b.prow_s}, {B.b.toff_q, nullptr, B.b.prow_off_q, B.b.prow_q}}});
    return GM_OK;
}

static int setup_wave(gm_ctx* c, Batch& B, const WavePlan& wp, int bm, int K, WaveBufs& w, const WaveDims& d, Grp& gs,
                      Grp& gq) {
    hipStream_t st = c->stream;
    std::vector<int32_t> ro_s, tg_s, tm_s, ro_q, tg_q, tm_q, re_s, re_q;
    build_tiles(B.poff_s, wp.t0, wp.t1, bm, ro_s, tg_s, tm_s);
    build_tiles(B.poff_q, wp.t0, wp.t1, bm, ro_q, tg_q, tm_q);
    for (int t = wp.t0; t <= wp.t1; ++t) {
        re_s.push_back((int32_t)(B.sup->task_offsets[t] - wp.s0));
        re_q.push_back((int32_t)(B.qry->task_offsets[t] - wp.q0));
    }
    // runs of consecutive tasks for the products that are only summed over the tasks
    std::vector<int32_t> co_s, co_q;
    const int n_coarse = coarse_group_count(c, d.Tw, std::min(d.Ps, d.Pq));
    for (int i = 0; i <= n_coarse; ++i) {
        const int t = (int)((int64_t)i * d.Tw / n_coarse);
        co_s.push_back(ro_s[t]);
        co_q.push_back(ro_q[t]);
    }
    Upload up{reinterpret_cast<char*>(w.row_off_s), {}};
    up.put(w.row_off_s, ro_s); up.put(w.row_off_q, ro_q);
    up.put(w.real_off_s, re_s); up.put(w.real_off_q, re_q);
    up.put(w.tile_g_s, tg_s); up.put(w.tile_m_s, tm_s);
    up.put(w.tile_g_q, tg_q); up.put(w.tile_m_q, tm_q);
    up.put(w.coarse_off_s, co_s); up.put(w.coarse_off_q, co_q);
    std::vector<u32> po_ss, po_qs, po_sq;
    std::vector<u32> path;
    pair_layout(c, B, wp, K, d.pair_ss, d.pair_sq, &po_ss, &po_qs, &po_sq, &path);
    up.put(w.task_path, path);
    if (d.pair) { up.put(w.pair_off_ss, po_ss); up.put(w.pair_off_qs, po_qs); up.put(w.pair_off_sq, po_sq); }
    if (d.pair) {
        std::vector<HopTask> tasks;
        for (int t = 0; t < d.Tw; ++t)
            if (path[t]) tasks.push_back(HopTask{t, re_s[t + 1] - re_s[t], re_q[t + 1] - re_q[t]});
        std::vector<HopTask> by_size = tasks;
        auto size = [](const HopTask& x) { return std::max(x.ns, x.nq); };
        std::stable_sort(by_size.begin(), by_size.end(), [&](const HopTask& a, const HopTask& b) { return size(a) > size(b); });
        std::vector<int32_t> order;
        w.count_rows.clear();
        for (const HopTask& x : by_size) {
            order.push_back(x.t);
            w.count_rows.push_back(size(x));
        }
        up.put(w.count_order, order);
        const HopPlan plan = hop_plan(tasks, hop_slices(c->F, c->D));
        w.n_hop_small = (int)plan.small.size();
        w.hop_run = plan.run;
        up.put(w.hop_small, plan.small);
        for (int k = 0; k < 3; ++k) {
            w.hop_longest[k] = plan.longest[k];
            up.put(w.hop_tiles[k], plan.tiles[k]);
        }
    }
    const int rc = up.send(c, B.images);
    if (rc != GM_OK) return rc;
    launch_expand_tasks(st, d.Tw, ExpandJobs{2, {{nullptr, w.row_off_s, nullptr, w.row_task_s}, {nullptr, w.row_off_q, nullptr, w.row_task_q}}, c->d_status, ST_WORDS});
    auto most = [](const std::vector<int32_t>& off) { int32_t m = 0; for (size_t t = 1; t < off.size(); ++t) m = std::max(m, off[t] - off[t - 1]); return (int)m; };
    gs = Grp{w.row_off_s, w.real_off_s, w.row_task_s, w.tile_g_s, w.tile_m_s, d.mt_s, d.Tw, bm, d.Ps, most(ro_s)};
    gq = Grp{w.row_off_q, w.real_off_q, w.row_task_q, w.tile_g_q, w.tile_m_q, d.mt_q, d.Tw, bm, d.Pq, most(ro_q)};
    return GM_OK;
}

// Pair-count matrices for the tasks that qualify, when the wave's bags and (task, field)s are within the counting
// kernel's limits; a task with a count that does not fit a byte is handed to the sparse kernel (its flag is cleared on
// the device).  allow_side: the counting may run on the second stream (gm_configure "overlap_pairs"); the caller then
// joins it before the first row hop.
static int count_pairs(gm_ctx* c, const Batch& B, const WavePlan& wp, WaveBufs& w, const WaveDims& d, int tf_cap,
                       int max_bag, int max_tf, bool allow_side, bool& pair, bool& any_sparse, bool& pairs_on_side) {
    hipStream_t st = c->stream;
    const int F = c->F, Tw = wp.t1 - wp.t0;
    pair = d.pair && tf_cap <= PAIR_MAX_CAP && max_bag <= PAIR_MAX_BAG;
    any_sparse = d.any_sparse || (d.pair && !pair);
    pairs_on_side = false;
    if (d.pair && !pair) launch_fill_u32(st, w.task_path, Tw, 0u);
    if (!pair) return GM_OK;
    PairCountArgs pa;
    memset(&pa, 0, sizeof pa);
    pa.F = F;
    pa.real_off_s = w.real_off_s; pa.real_off_q = w.real_off_q; pa.row_off_s = w.row_off_s; pa.row_off_q = w.row_off_q;
    pa.base_s = w.base_s; pa.base_q = w.base_q; pa.cnt_s = w.cnt_s; pa.cnt_q = w.cnt_q; pa.n_slots = w.n_slots;
    pa.slot_start = w.slot_start; pa.qseg_lo = w.qseg_lo; pa.qseg_hi = w.qseg_hi;
    pa.sup_sorted = w.sup_sorted; pa.qry_sorted = w.qry_sorted;
    pa.off_ss = w.pair_off_ss; pa.off_qs = w.pair_off_qs; pa.off_sq = w.pair_off_sq;
    pa.mat = w.pair_mat; pa.want_ss = d.pair_ss; pa.want_sq = d.pair_sq; pa.status = c->d_status;
    pa.task_path = w.task_path;
    pairs_on_side = allow_side && c->overlap_pairs && !c->overlap_sort;
    hipStream_t pst = pairs_on_side ? c->side : st;
    if (pairs_on_side) {   // everything the kernel reads is in place once the main stream gets here
        HIPCHK(c, hipEventRecord(c->ev_pairs_go, st));
        HIPCHK(c, hipStreamWaitEvent(c->side, c->ev_pairs_go, 0));
        launch_fill_u32(c->side, c->d_status_side, ST_WORDS, 0);
        pa.status = c->d_status_side;
    }
    {
        Prof p(c, "pair_count", 8.0 * (d.nnz_s + d.nnz_q) + (double)d.pair_bytes, 0, pst, true);
        launch_pair_count(pst, pa, w.count_order, w.count_rows, max_tf, max_bag, c->pair_tile_rows);
    }
    if (pairs_on_side) {
        HIPCHK(c, hipEventRecord(c->ev_pairs, c->side));
    } else {
        u32 hs[ST_WORDS];
        int rc = read_status(c, hs);
        if (rc != GM_OK) return rc;
        if (hs[ST_PAIR_OVF]) any_sparse = true;   // some task's flag was cleared on the device
        // the sparse kernel reads the slot of every lookup: written now if the wave was planned without it
        if (any_sparse && !w.slots_written) sort_task_fields(c, B, wp, w, max_tf);
    }
    return GM_OK;
}

// Everything of a one-wave batch with the row-list output that depends on its indices only, prepared ahead of the step
// (by gm_meta_train, on the second stream, while the previous batch computes): validated offsets and indices, padded
// row numbers, tile lists, per-(task, field) dictionaries and overlap join, pair-count matrices (unless their room is
// apart: WaveDims), the batch-wide order of the lookups by row.  The buffers live in an arena of their own.
struct Prepared {
    Batch B;
    WavePlan wp;
    WaveDims d;
    WaveBufs w;        // index part only
    Grp gs, gq;
    int bm = 64;
    int tf_cap = 0, max_bag = 0, max_tf = 0;
    bool pair = false, any_sparse = false;
    ValEnc enc = kPlainVals;   // how the values of the ordered lookups name their bags
};

// Global back-propagation on xi (Alg. 1) as part of a step: emb[row] += scale * (the row's gradient) straight from the segment
// reduction.  Only a batch of one wave of tasks can (`done`): the next wave's prefetch reads the tables.
struct EmbUpdate {
    float* emb;
    float scale;
    bool done = false;
};

// The step.  pre: null, or the batch's index side prepared beforehand (one wave, row-list output); no_sync: return with
// the work enqueued and the stream not drained (the caller synchronises and reads nothing from the host side but the
// stream's error state; only with pre).  up: see EmbUpdate (where done, no list is written and no table-shaped output touched).
static int meta_step_impl(gm_ctx* c, int32_t T, const gm_set* sup, const gm_set* qry, const gm_params* params, float alpha,
                          int32_t K, int32_t order, float* loss, gm_grads* out, Prepared* pre, bool no_sync,
                          EmbUpdate* up = nullptr) {
    if (!c) return GM_ERR_ARG;
    if (T < 0 || K < 0 || (order != 1 && order != 2)) return fail(c, GM_ERR_ARG, "bad n_tasks / inner_steps / order");
    if (!out) return fail(c, GM_ERR_ARG, "null outputs");
    float* const table = c->F > 0 ? out->emb_grad_table : nullptr;
    int rc = check_set(c, sup, T, "support", table != nullptr);
    if (rc != GM_OK) return rc;
    rc = check_set(c, qry, T, "query", table != nullptr);
    if (rc != GM_OK) return rc;
    if (!params || !params->W || !params->b || (c->F > 0 && !params->emb)) return fail(c, GM_ERR_ARG, "null params");
    if (!loss || !out->dW || !out->db || !out->n_emb_rows) return fail(c, GM_ERR_ARG, "null outputs");
    for (int l = 0; l < c->L; ++l)
        if (!params->W[l] || !params->b[l] || !out->dW[l] || !out->db[l]) return fail(c, GM_ERR_ARG, "null layer pointer");
    if (!table && (out->emb_rows_capacity < 0 || (out->emb_rows_capacity > 0 && (!out->emb_rows || !out->emb_grad))))
        return fail(c, GM_ERR_ARG, "bad sparse output buffers");
    HIPCHK(c, hipSetDevice(c->device));
    hipStream_t st = c->stream;
    const int F = c->F, D = c->D, L = c->L, FD = c->FD, ld0 = c->ld[0];
    const bool bf = c->mlp_dtype != 0;
    const int64_t nt = c->n_theta;
    const int64_t nnz = sup->nnz + qry->nnz;
    const int64_t capacity = table ? 0 : out->emb_rows_capacity;

    if (pre && table) return fail(c, GM_ERR_ARG, "internal: a prepared batch uses the row-list output");
    Arena ar;
    ar.base = c->ws; ar.cap = c->ws_bytes; ar.off = c->persistent;
    Batch local_batch;
    Batch& B = pre ? pre->B : local_batch;
    std::vector<WavePlan> plans;
    int bm;
    if (pre) {   // the index side exists already; the dense buffers of the batch go to this call's arena
        alloc_batch_dense(c, ar, B.b, T, B.poff_s[T], B.poff_q[T], true);
        if (ar.overflow) return fail(c, GM_ERR_WORKSPACE, "workspace too small for the batch-level buffers (%zu needed)", ar.off);
        bm = pre->bm;
        plans.push_back(pre->wp);
    } else {
        B.T = T; B.sup = sup; B.qry = qry;
        B.table = table != nullptr;
        rc = begin_batch(c, B, ar, capacity, !B.table, &ar);
        if (rc != GM_OK) return rc;
        bm = pick_bm(c, B);
        rc = plan_waves(c, B, c->ws_bytes - ar.off, K, order, bm, plans);
        if (rc != GM_OK) return rc;
    }
    BatchBufs& b = B.b;
    const int64_t Ps_tot = B.poff_s[T];
    const size_t wave_mark = ar.off;
    const bool apply = up && F > 0 && plans.size() == 1;
    float* const row_table = apply ? up->emb : table;        // where the segment reduction adds rows (null: it lists them)
    const float row_scale = apply ? up->scale : 1.f;
    int64_t* const n_list = apply ? nullptr : out->n_emb_rows;   // (null: no list)
    struct SideGuard {   // whatever way this call ends, nothing of it is left running on the side stream
        gm_ctx* c;
        bool active = false;
        ~SideGuard() { if (active) (void)hipStreamSynchronize(c->side); }
    } side{c};
    bool side_list = false;
    bool list_ordered = false;   // row-list output: the batch's lookups were ordered and cut into segments inside its (only) wave
    ValEnc enc = kPlainVals;     // how the values that travel with the row keys name their bags

    // meta theta in the padded internal layout (and its bf16 operand copies); accumulators
    std::vector<MatrixJob> mats;
    for (int l = 1; l <= L; ++l) {
        mats.push_back(MatrixJob{params->W[l - 1], c->dims[l - 1], c->dims[l], c->dims[l], b.theta0.f + c->offW[l],
                                 bf && l < L ? b.theta0.b + c->offWb[l] : nullptr, c->ld[l - 1], c->ld[l], c->ld[l], 0});
        mats.push_back(MatrixJob{params->b[l - 1], 1, c->dims[l], c->dims[l], b.theta0.f + c->offb[l], nullptr, 1,
                                 l == L ? 32 : c->ld[l], 32, 0});
    }
    launch_copy_matrices(st, mats.data(), (int)mats.size());
    bool theta_summed = false;   // the first wave's sums are stored, later waves' added
    // Gradient w.r.t. the pooled inputs: the query rows are written whole by the outer backward pass; the support rows
    // are the second-order chain's sum, whose first product stores instead of adding; without a chain they are zeros, and left out.
    const bool no_chain = order == 1 || K == 0;
    float* task_loss = out->task_loss ? out->task_loss : b.task_loss;

    for (const WavePlan& wp : plans) {
        ar.off = wave_mark;
        const int Tw = wp.t1 - wp.t0;
        if (Tw == 0) continue;
        WaveBufs w;
        if (pre) w = pre->w;
        const WaveDims d = pre ? pre->d : wave_dims(c, B, wp, bm, K, order);
        if (!pre) alloc_wave_index(c, ar, w, d);
        alloc_wave_dense(c, ar, w, d, K, order, b.GX ? b.GX + (Ps_tot + wp.pq0) * (int64_t)FD : nullptr);
        if (ar.overflow) return fail(c, GM_ERR_WORKSPACE, "internal: wave does not fit");
        Grp gs, gq;
        const bool adapt = c->adapt_rows != 0;
        int tf_cap = 0, max_bag = 0, max_tf = 0;
        bool pair = false, any_sparse = false, pairs_on_side = false;
        bool ordered = false;   // this wave's lookups are in row order already (its dictionaries were read off that order)
        if (pre) {
            enc = pre->enc;
            gs = pre->gs; gq = pre->gq;
            tf_cap = pre->tf_cap; max_bag = pre->max_bag; max_tf = pre->max_tf;
            pair = pre->pair; any_sparse = pre->any_sparse;
            if (d.mat_apart) {
                launch_fill_u32(st, c->d_status, ST_WORDS, 0);
                if ((rc = count_pairs(c, B, wp, w, d, tf_cap, max_bag, max_tf, false, pair, any_sparse, pairs_on_side))) return rc;
            }
        } else {
            if ((rc = setup_wave(c, B, wp, bm, K, w, d, gs, gq))) return rc;
            // a0: row dictionaries and the overlap join -- read off the row order of the wave's lookups when that order
            // is the one the sparse gradient needs (table-shaped output: every wave's own; row list: a batch of one wave)
            JoinReq jr;
            if (F > 0 && !c->overlap_sort && (table || plans.size() == 1)) {
                jr.so = table ? &w.so : &b.so;
                jr.range = table ? SortRange{wp.s0, wp.s1, wp.q0, wp.q1, wp.ls0, wp.ls1, wp.lq0, wp.lq1,
                                             (u32)(0 - (uint64_t)wp.ps0), (u32)((uint64_t)d.Ps - (uint64_t)wp.pq0)}
                                 : whole_batch_range(B);
                jr.n_sup_rows = d.Ps; jr.n_qry_rows = d.Pq;
                if (!table) { jr.capacity = capacity; jr.n_rows = n_list; }
                jr.pair_only = d.pair && !d.any_sparse;
            }
            rc = run_index_wave(c, B, wp, w, &tf_cap, &max_bag, &max_tf, &jr);
            if (rc != GM_OK) return rc;
            if (jr.used) { ordered = true; enc = jr.enc; }
            if ((rc = count_pairs(c, B, wp, w, d, tf_cap, max_bag, max_tf, true, pair, any_sparse, pairs_on_side))) return rc;
            if (pairs_on_side) side.active = true;
        }
        // joins the counting on the side stream: the host learns whether a task fell back to the sparse kernel, the main
        // stream waits for the matrices (called before the first row hop, which is their first reader)
        auto join_pairs = [&]() -> int {
            if (!pairs_on_side) return GM_OK;
            pairs_on_side = false;
            u32 hs[ST_WORDS];
            HIPCHK(c, hipMemcpyAsync(hs, c->d_status_side, ST_WORDS * sizeof(u32), hipMemcpyDeviceToHost, c->side));
            HIPCHK(c, hipStreamSynchronize(c->side));
            HIPCHK(c, hipStreamWaitEvent(st, c->ev_pairs, 0));
            if (hs[ST_PAIR_OVF]) any_sparse = true;
            if (c->row_path == 2 && any_sparse && adapt)
                return fail(c, GM_ERR_CAPACITY, "pair-count path forced, but a task, count, bag or (task, field) exceeds its limits");
            if (any_sparse && !w.slots_written) sort_task_fields(c, B, wp, w, max_tf);
            return GM_OK;
        };
        if (!pairs_on_side && c->row_path == 2 && any_sparse && adapt)
            return fail(c, GM_ERR_CAPACITY, "pair-count path forced, but a task, count, bag or (task, field) exceeds its limits");
        const int n_tf = Tw * F;
        const int32_t* rows_s = b.prow_s + wp.s0;
        const int32_t* rows_q = b.prow_q + wp.q0;
        const int32_t rb_s = (int32_t)wp.ps0, rb_q = (int32_t)wp.pq0;
        const bool second = order == 2 && K > 0;

        const bool factors = d.factor_ld > 0;
        if (factors) {
            w.room.rows_s = w.row_off_s; w.room.rows_q = w.row_off_q;
            w.room.most_s = gs.most_rows; w.room.most_q = gq.most_rows;
            gs.room = gq.room = &w.room;
        }

        // a1: one prefetch pass for both sets.  Every real row is written whole (pooled fields, dense and pad columns); only
        // the pad rows of what the row arithmetic writes real rows of are cleared.
        const bool padded = d.Ps != d.Ss || d.Pq != d.Sq;
        // bf16: the fp32 input is kept only where a row update still adds to it -- the support set's from the second inner step on
        const bool hops = F > 0 && adapt && K > 0, q_once = bf && !hops;
        float* const xs_f32 = bf && !(hops && K > 1) ? nullptr : w.Xs0;
        float* const xq_f32 = q_once ? nullptr : w.Xq0;
        Act X0s;  // step-0 support input
        X0s.ld = ld0;
        if (bf) X0s = K > 0 ? w.steps[0].X : Act();
        else X0s.f = w.Xs0;
        {
            const double lookups = (double)(d.nnz_s + d.nnz_q), bags = (double)(d.Ss + d.Sq) * F;
            Prof p(c, "gather_pool", lookups * (4.0 * D + 4) + bags * (4.0 * D + 8 + (bf ? 2.0 * D : 0)), 0);
            launch_gather_pool(st, F, D, c->n_dense, c->d_field_base, params->emb, ld0,
                               PoolSet{sup->bag_offsets, sup->indices, sup->dense, wp.s0, d.Ss, rows_s, rb_s, xs_f32, bf ? X0s.b : nullptr,
                                       second ? (bf ? w.TXf : w.TX.f) : nullptr, second ? w.TX.b : nullptr},   // (dense features are not parameters: their direction is zero)
                               PoolSet{qry->bag_offsets, qry->indices, qry->dense, wp.q0, d.Sq, rows_q, rb_q, xq_f32, q_once ? w.Xq.b : nullptr});
        }
        if (padded) {
            PadJobs pj;
            memset(&pj, 0, sizeof pj);
            pj.off[0] = w.row_off_s; pj.off[1] = w.row_off_q; pj.real[0] = w.real_off_s; pj.real[1] = w.real_off_q;
            auto pad = [&](void* p, int elem, int set) {
                if (!p) return;
                pj.p[pj.n] = static_cast<char*>(p); pj.row_bytes[pj.n] = ld0 * elem; pj.set[pj.n] = set;
                if (++pj.n == PAD_JOBS) { launch_zero_pad_rows(st, Tw, pj); pj.n = 0; }
            };
            pad(xs_f32, 4, 0); pad(xq_f32, 4, 1);
            pad(X0s.b, 2, 0); pad(w.Xq.b, 2, 1); pad(w.Xs_scratch.b, 2, 0);
            for (size_t k = 1; k < w.steps.size(); ++k) pad(w.steps[k].X.b, 2, 0);
            if (second) { pad(w.TX.b, 2, 0); pad(w.TX.f, 4, 0); pad(w.TXf, 4, 0); }
            launch_zero_pad_rows(st, Tw, pj);
        }
        // The wave's offsets and indices are validated.  Ordering the lookups by row needs nothing else: it runs on the
        // side stream from here on -- beside the dense phase, which is bound by memory traffic, not beside the index
        // kernels above, which are bound by the same things as the sort -- and is joined before the segment reduction
        // (row-list output: only when the batch is one wave, so that everything it reads has been validated).
        if (!pre && c->overlap_sort && F > 0 && (table || plans.size() == 1)) {
            HIPCHK(c, hipEventRecord(c->ev_go, st));
            HIPCHK(c, hipStreamWaitEvent(c->side, c->ev_go, 0));
        }
        const bool side_table = table && c->overlap_sort && F > 0;
        if (side_table) {
            if (side.active) HIPCHK(c, hipStreamWaitEvent(c->side, c->ev_main, 0));   // the previous wave is done with this memory
            side.active = true;
            launch_fill_u32(c->side, c->d_status_side, ST_WORDS, 0);
            const SortRange r{wp.s0, wp.s1, wp.q0, wp.q1, wp.ls0, wp.ls1, wp.lq0, wp.lq1,
                              (u32)(0 - (uint64_t)wp.ps0), (u32)((uint64_t)d.Ps - (uint64_t)wp.pq0)};
            global_order(c, B, w.so, r, nullptr, nullptr, d.nnz_s + d.nnz_q, nullptr, true);
            HIPCHK(c, hipEventRecord(c->ev_side, c->side));
        } else if (!pre && !table && c->overlap_sort && F > 0 && plans.size() == 1) {
            side.active = true;
            side_list = true;
            launch_fill_u32(c->side, c->d_status_side, ST_WORDS, 0);
            global_order(c, B, b.so, whole_batch_range(B), nullptr, nullptr, capacity, n_list, true);
            HIPCHK(c, hipEventRecord(c->ev_side, c->side));
        }
        // row arithmetic of one (task, field) at a time, through LDS (no row table in HBM)
        int max_bags = 0;
        for (int t = wp.t0; t < wp.t1; ++t)
            max_bags = std::max<int>(max_bags, (int)std::max(sup->task_offsets[t + 1] - sup->task_offsets[t],
                                                               qry->task_offsets[t + 1] - qry->task_offsets[t]));
        int max_prows = 0;
        for (int t = wp.t0; t < wp.t1; ++t)
            max_prows = std::max<int>(max_prows, (int)std::max(B.poff_s[t + 1] - B.poff_s[t], B.poff_q[t + 1] - B.poff_q[t]));
        if (K > 0 && F > 0 && max_prows > 2048)
            return fail(c, GM_ERR_CAPACITY, "a task has %d samples in one set; the limit with inner steps is 2048", max_prows);
        // gradient w.r.t. the pooled inputs: the wave's rows of the batch-wide buffer, or the wave's own buffer
        float* gxs = table ? w.GX : b.GX + wp.ps0 * (int64_t)FD;
        float* gxq = table ? w.GX + d.Ps * (int64_t)FD : b.GX + (Ps_tot + wp.pq0) * (int64_t)FD;
        auto hop_out = [&](bool support, const float* y_in, float* y_out, bf16_t* y_bf, float cc) {
            TwoHopOut o;
            memset(&o, 0, sizeof o);
            o.enabled = 1;
            o.bag_offsets = support ? sup->bag_offsets : qry->bag_offsets;
            o.sample0 = support ? wp.s0 : wp.q0;
            o.lookup0 = support ? wp.ls0 : wp.lq0;
            o.real_offsets = support ? w.real_off_s : w.real_off_q;
            o.slot_of_lookup = support ? w.sup_slot : w.qry_slot;
            o.row_map = support ? rows_s : rows_q;
            o.row_base = support ? rb_s : rb_q;
            o.y_in = y_in; o.y_out = y_out; o.y_bf = y_bf; o.ld = ld0; o.c = cc;
            return o;
        };
        // (query_sum: the pair-count tasks' query output is left out before the last step, which adds the steps' gradients up)
        const int n_kept = pair && adapt ? d.query_sum : 0;
        float* const kept[HOP_SUM] = {w.dX, gxs, second ? w.TXf : w.dX_kept};   // of the last step, the first, the second
        auto two_hop = [&](bool in_support, const float* Z, const TwoHopOut* o0, const TwoHopOut* o1, bool keep = false) {
            const double bags_ = (o0 ? (double)d.Ss : 0.0) + (o1 ? (double)d.Sq : 0.0);
            const double in_l_ = in_support ? (double)d.nnz_s : (double)d.nnz_q;
            const double out_l_ = (o0 ? (double)d.nnz_s : 0.0) + (o1 ? (double)d.nnz_q : 0.0);
            // algorithmic bytes: Z once per (sample, field), Y read + written per (sample, field), 4 B per lookup and hop
            const double alg_bytes = 4.0 * D * F * (in_support ? d.Ss : d.Sq) + bags_ * F * (8.0 * D + (bf ? 2.0 * D : 0)) + 4.0 * (in_l_ + out_l_);
            const TwoHopOut* const o1_pair = keep && n_kept && o0 ? nullptr : o1;
            if (pair && (o0 || o1_pair)) {   // o0 is always the support side, o1 the query side
                PairHopArgs pa;
                memset(&pa, 0, sizeof pa);
                pa.F = F; pa.D = D; pa.mat = w.pair_mat; pa.task_path = w.task_path;
                pa.in_real_off = in_support ? w.real_off_s : w.real_off_q;
                pa.in_row_off = in_support ? w.row_off_s : w.row_off_q;
                pa.Z[0] = Z; pa.n_z = 1; pa.ldz = FD;
                if (keep && n_kept && !o0)
                    for (; pa.n_z < n_kept; ++pa.n_z) pa.Z[pa.n_z] = kept[pa.n_z];
                auto fill = [&](PairHopOut& po, const TwoHopOut& o, bool out_support) {
                    po.enabled = 1;
                    po.mat_off = out_support ? (in_support ? w.pair_off_ss : w.pair_off_sq) : w.pair_off_qs;
                    po.real_off = out_support ? w.real_off_s : w.real_off_q;
                    po.row_off = out_support ? w.row_off_s : w.row_off_q;
                    po.y_in = o.y_in; po.y_out = o.y_out; po.y_bf = o.y_bf; po.ld = o.ld; po.c = o.c;
                };
                if (o0) fill(pa.out[0], *o0, true);
                if (o1_pair) fill(pa.out[1], *o1_pair, false);
                pa.small = w.hop_small; pa.n_small = w.n_hop_small; pa.run = w.hop_run;
                Prof p(c, "pair_hop", alg_bytes, 0);
                launch_pair_hop(st, pa, w.hop_tiles, w.hop_longest);
            }
            if (!any_sparse) return;
            TwoHopArgs a;
            memset(&a, 0, sizeof a);
            a.F = F; a.D = D;
            a.tf_base = w.base_s; a.n_slots = w.n_slots;
            if (in_support) { a.in_seg_lo = w.slot_start; a.in_seg_hi = w.slot_start + 1; a.in_seg_tf_stride = 1; a.in_sorted = w.sup_sorted; }
            else { a.in_seg_lo = w.qseg_lo; a.in_seg_hi = w.qseg_hi; a.in_seg_tf_stride = 0; a.in_sorted = w.qry_sorted; }
            a.Z = Z; a.ldz = FD; a.task_path = w.task_path;
            a.in_row_offsets = in_support ? w.row_off_s : w.row_off_q;
            a.max_in_rows = max_prows;
            if (o0) a.out[0] = *o0;
            if (o1) a.out[1] = *o1;
            Prof p(c, "two_hop", alg_bytes, 0);
            launch_two_hop(st, a, Tw, max_bags);
        };

        // inner loop on the support set
        const float* labels_s = sup->labels + wp.s0;
        const float* labels_q = qry->labels + wp.q0;
        Theta th = b.theta0;        // GEMM operands of the current step
        const float* thf = b.theta0.f;  // fp32 view (biases, last layer)
        int64_t thf_stride = 0;
        const float* xs_cur = w.Xs0;    // fp32 support input of the current step
        Act Xq = w.Xq;                  // query input as the GEMMs read it
        if (!bf) Xq.f = w.Xq0;          // fp32: the prefetched buffer, updated in place by the overlap update
        const bool from_theta0 = d.from_meta, keep = second || from_theta0;
        std::vector<Factor> v_fac;   // of the direction
        const float* thf0 = thf;
        std::vector<Pass> passes;
        for (int k = 0; k < K; ++k) {
            StepState& s = w.steps[keep ? k : 0];
            if (k == 0) s.X = X0s;
            s.th = th;
            s.wL = thf + c->offW[L];
            s.wL_stride = thf_stride;
            Pass p{&s.X, &s.A, &s.Dl, s.dL, s.zL};
            float* const dX = n_kept && k + 1 < K ? kept[1 + k] : w.dX;
            forward_backward(c, gs, labels_s, p, th, thf, thf_stride, nullptr, F > 0 ? dX : nullptr);
            // local back-propagation: theta' = theta - alpha dtheta (per task)
            Theta& next = w.thetas[second ? k : 0];
            float* wl_copy = (bf && second && k + 1 < K) ? w.steps[k + 1].wL_copy : nullptr;
            // bf16: after the last inner step only the operand copies of W' are read again, not its fp32 master
            if (from_theta0) {
                passes.push_back(p);
                theta_grad(c, gs, p, next, thf, thf_stride, 1.f, -alpha, wl_copy, false, nullptr, nullptr, &passes, thf0);
            } else theta_grad(c, gs, p, next, thf, thf_stride, 1.f, -alpha, wl_copy, !(bf && k + 1 == K));
            th = next;
            thf = next.f;
            thf_stride = nt;
            // rows' = rows - alpha drows, seen through the pooled inputs: the support input of the next step and
            // (overlap update) the query input; a query row that the support set does not touch keeps its meta value
            const bool more = k + 1 < K;
            Act Xn;  // support input of step k+1
            if (more) Xn = keep ? w.steps[k + 1].X : w.Xs_scratch;
            if (F > 0 && adapt) {
                if ((rc = join_pairs())) return rc;
                float* xs_next = nullptr;
                if (more) {
                    xs_next = bf ? w.Xs0 : Xn.f;  // bf16: the fp32 master is updated in place
                }
                // (bf16: of the last update of a set only the operand copy is read)
                const bool last = !more;
                TwoHopOut os = hop_out(true, xs_cur, bf && k + 2 == K ? nullptr : xs_next, more && bf ? Xn.b : nullptr, -alpha);
                TwoHopOut oq = hop_out(false, w.Xq0, bf && last ? nullptr : w.Xq0, (bf && last) ? Xq.b : nullptr, -alpha);
                two_hop(true, dX, more ? &os : nullptr, &oq, true);
                if (more) {
                    launch_copy_tail(st, FD, xs_cur, d.Ps, bf ? nullptr : (xs_next != xs_cur ? xs_next : nullptr), ld0, bf ? Xn.b : nullptr);
                    xs_cur = xs_next;
                }
            } else if (more) {  // no sparse fields, or rows not adapted: every step reads the same input
                Xn = s.X;
            }
            if (more) {
                w.steps[keep ? k + 1 : 0].X = Xn;
            }
        }
        // bf16 second order with K > 1: steps k >= 1 read their last-layer weights from the copies taken above
        if (bf && second)
            for (int k = 1; k < K; ++k) {
                w.steps[k].wL = w.steps[k].wL_copy;
                w.steps[k].wL_stride = c->ld[L - 1];
            }

        if ((rc = join_pairs())) return rc;   // (no inner step took a row hop)
        // outer forward/backward on the query set with the adapted parameters
        if (bf && hops) launch_copy_tail(st, FD, w.Xq0, d.Pq, nullptr, ld0, Xq.b);
        Pass pq{&Xq, &w.Aq, &w.Dq, w.dLq, w.zq};
        forward_backward(c, gq, labels_q, pq, th, thf, thf_stride, w.loss_q, F > 0 ? gxq : nullptr);
        // The query gradient w.r.t. theta' per task starts the second-order chain; without a chain it is only summed
        // over the tasks, so it is taken over runs of tasks straight away.
        const int n_coarse = coarse_group_count(c, Tw, std::min(d.Ps, d.Pq));
        Grp gs_coarse = gs, gq_coarse = gq;
        gs_coarse.row_off = w.coarse_off_s; gs_coarse.G = n_coarse;
        gq_coarse.row_off = w.coarse_off_q; gq_coarse.G = n_coarse;
        // (factors: the chain's other terms are added to these sums, no task's direction is formed)
        const bool runs_only = !second || factors || query_runs(c, Tw, d.Pq, n_coarse, K, order);
        theta_grad(c, gq, pq, w.v, nullptr, 0, 0.f, 1.f, nullptr, true, runs_only ? &gq_coarse : nullptr, runs_only ? &w.vsum : nullptr,
                   nullptr, nullptr, w.loss_q, task_loss + wp.t0);
        if (factors) {
            v_fac.push_back(Factor{&Xq, &w.Aq, &w.Dq, true, 1.f});
            w.v.fac = &v_fac;
        }

        // second-order chain back through the inner steps: v_k = v_{k+1} - alpha H_k v_{k+1}
        if (second) {
            float* txf = bf ? w.TXf : w.TX.f;  // fp32 pooled direction (support rows); TX.b is its GEMM operand copy
            if (!adapt) {   // no direction on the inputs: whatever still reads it (a model without hidden layers) sees zeros
                if (bf) zero_bf16(st, w.TX.b, d.Ps * ld0);
                else launch_fill_f32(st, w.TX.f, d.Ps * ld0, 0.f);
            }
            for (int k = 0; factors && k + 1 < K; ++k) zero_bf16(st, w.TXk[k].b, d.Ps * ld0);   // (the columns and rows that no hop writes)
            if (F > 0 && adapt) {
                // direction on the support rows = query gradient routed through the rows both sets share
                TwoHopOut os = hop_out(true, nullptr, bf && K == 1 ? nullptr : txf, w.TX.b, 1.f);
                two_hop(false, gxq, &os, nullptr);
            }
            for (int k = K - 1; k >= 0; --k) {
                const StepState& s = w.steps[k];
                if (factors) { w.TX = w.TXk[k]; w.TA = w.TAk[k]; w.TD = w.TDk[k]; }
                // bf16 with hidden layers: the layer-1 product adds -alpha * dX to the gradient buffer itself
                // (fp32 does so when nothing else reads dX)
                const bool fused_gx = L > 1 && F > 0 && (bf || !(k > 0 && adapt));
                // (the chain's first step starts that sum: the buffer's support rows need no clearing.  Where dX is written anyway the
                // second step starts it, from what dX still holds: the same bits, and one array less to write: the first step's launch of
                // 512 tasks x 256 rows x 1664 columns 770 -> 636 us)
                const bool gx_old = fused_gx && bf && adapt && k == K - 2;
                hvp_step(c, gs, s, w, alpha, k > 0, fused_gx && !(bf && adapt && k > 0 && k == K - 1) ? gxs : nullptr, k > 0 && adapt, k == K - 1, gx_old, adapt,
                         k == 0 || factors ? &gs_coarse : nullptr, runs_only);
                if (factors) {
                    v_fac.push_back(Factor{adapt && F > 0 ? &w.TXk[k] : nullptr, &w.TAk[k], &s.Dl, false, -alpha});
                    v_fac.push_back(Factor{&s.X, &s.A, &w.TDk[k], false, -alpha});
                }
                if (F > 0) {
                    if (!fused_gx) {
                        Prof p(c, "axpy_gx", (k == K - 1 ? 8.0 : 12.0) * d.Ps * FD, 0);
                        if (k == K - 1) launch_scale(st, d.Ps * (int64_t)FD, -alpha, w.dX, gxs);
                        else launch_axpy(st, d.Ps * (int64_t)FD, -alpha, w.dX, gxs);
                    }
                    if (k > 0 && adapt) {
                        TwoHopOut os = hop_out(true, txf, bf && k == 1 ? nullptr : txf, factors ? w.TXk[k - 1].b : w.TX.b, -alpha);
                        two_hop(true, w.dX, &os, nullptr);
                    }
                }
            }
        }
        // cross-task reduction of the dense part (tasks of the wave in order, waves in order).  vsum: the weight matrices'
        // part summed over runs of tasks -- the chain's last step, or (first order) all of it
        {
            Prof p(c, "reduce_tasks", 4.0 * (runs_only ? n_coarse : Tw) * nt, 0);
            ReduceArgs ra{w.v.f, w.vsum.f, nt, runs_only ? 1.f : -alpha, b.g_theta, theta_summed, 0, {}};
            std::vector<ReducePiece> pieces;
            for (int l = 1; l < L; ++l) {
                pieces.push_back(ReducePiece{c->offW[l], c->offb[l] - c->offW[l], runs_only ? 0 : Tw, n_coarse, 0});
                pieces.push_back(ReducePiece{c->offb[l], c->offW[l + 1] - c->offb[l], Tw, 0, 0});
            }
            pieces.push_back(ReducePiece{c->offW[L], nt - c->offW[L], Tw, 0, 0});
            launch_reduce_tasks(st, ra, pieces.data(), (int)pieces.size());
            theta_summed = true;
        }
        // table-shaped sparse output: the wave's lookups are ordered by row and every row's sum is added to its row of
        // the table (rows are distinct within a wave; waves follow each other on the stream)
        if (table) {
            const SortRange r{wp.s0, wp.s1, wp.q0, wp.q1, wp.ls0, wp.ls1, wp.lq0, wp.lq1,
                              (u32)(0 - (uint64_t)wp.ps0), (u32)((uint64_t)d.Ps - (uint64_t)wp.pq0)};
            const int64_t nw = d.nnz_s + d.nnz_q;
            if (side_table) HIPCHK(c, hipStreamWaitEvent(st, c->ev_side, 0));
            else if (!ordered) global_order(c, B, w.so, r, nullptr, nullptr, nw, nullptr);
            if (no_chain && d.Pq == 0 && FD > 0) launch_fill_f32(st, w.GX, d.Ps * (int64_t)FD, 0.f);   // (there is nothing but zeros)
            {
                Prof p(c, "seg_reduce", (double)nw * (4.0 * D + 4), 0);
                launch_seg_reduce(st, D, F, ordered ? enc : kPlainVals, w.so.keys, w.so.keys_tmp, nullptr, nw, nw, w.so.vals, w.GX,
                                  nullptr, nullptr, seg_room(c, w.so), row_table, row_scale, d.Ps + d.Pq, no_chain ? d.Ps : 0, w.so.hist);
            }
            if (side_table) HIPCHK(c, hipEventRecord(c->ev_main, st));
        } else if (ordered) {
            list_ordered = true;
        }
    }

    // outputs: dense meta-gradient, loss, coalesced sparse meta-gradient
    if (!theta_summed) launch_fill_f32(st, b.g_theta, nt, 0.f);   // no tasks
    mats.clear();
    for (int l = 1; l <= L; ++l) {
        mats.push_back(MatrixJob{b.g_theta + c->offW[l], c->dims[l - 1], c->dims[l], c->ld[l], out->dW[l - 1], nullptr, c->dims[l - 1],
                                 c->dims[l], c->dims[l], 0});
        mats.push_back(MatrixJob{b.g_theta + c->offb[l], 1, c->dims[l], c->dims[l], out->db[l - 1], nullptr, 1, c->dims[l], c->dims[l], 0});
    }
    launch_copy_matrices(st, mats.data(), (int)mats.size(), task_loss, T, loss);
    // (a batch whose segments were cut inside its wave keeps the status words of that: the row count, the capacity flag)
    if (!pre && !list_ordered) launch_fill_u32(st, c->d_status, ST_WORDS, 0);
    if (table) {
        launch_fill_u32(st, reinterpret_cast<u32*>(out->n_emb_rows), 2, 0u);
    } else {
        if (side_list) HIPCHK(c, hipStreamWaitEvent(st, c->ev_side, 0));
        else if (!pre && !list_ordered) global_order(c, B, b.so, whole_batch_range(B), nullptr, nullptr, capacity, n_list);
        if (no_chain && B.poff_q[T] == 0 && FD > 0) launch_fill_f32(st, b.GX, Ps_tot * (int64_t)FD, 0.f);   // (there is nothing but zeros)
        if (F > 0) {
            Prof p(c, "seg_reduce", (double)nnz * (4.0 * D + 4), 0);
            launch_seg_reduce(st, D, F, (pre || list_ordered) ? enc : kPlainVals, b.so.keys, b.so.keys_tmp, n_list, apply ? nnz : capacity, nnz,
                              b.so.vals, b.GX, out->emb_rows, out->emb_grad, seg_room(c, b.so), row_table, row_scale, Ps_tot + B.poff_q[T], no_chain ? Ps_tot : 0, b.so.hist);
        }
    }
    if (up) up->done = apply;
    if (pre && no_sync) return GM_OK;   // the caller drains the stream; a prepared batch has passed every check already
    u32 hs[ST_WORDS];
    memset(hs, 0, sizeof hs);
    if (pre) {
        HIPCHK(c, hipStreamSynchronize(st));
        HIPCHK(c, hipGetLastError());
        prof_drain(c);
        return GM_OK;
    }
    if (side_list)   // the ordering's own status words (the main stream has waited for it)
        HIPCHK(c, hipMemcpyAsync(hs, c->d_status_side, ST_WORDS * sizeof(u32), hipMemcpyDeviceToHost, st));
    rc = side_list ? (hipStreamSynchronize(st) == hipSuccess ? GM_OK : fail(c, GM_ERR_HIP, "stream synchronisation failed"))
                   : read_status(c, hs);
    if (rc != GM_OK) return rc;
    B.images.held.clear();   // (the stream has been drained)
    HIPCHK(c, hipGetLastError());
    prof_drain(c);
    if (hs[ST_CAPACITY])
        return fail(c, GM_ERR_CAPACITY, "emb_rows_capacity %lld is smaller than the %u rows touched", (long long)capacity,
                    hs[ST_NROWS]);
    return GM_OK;
}

extern "C" int gm_meta_step(gm_ctx* c, int32_t T, const gm_set* sup, const gm_set* qry, const gm_params* params,
                            float alpha, int32_t K, int32_t order, float* loss, gm_grads* out) {
    return meta_step_impl(c, T, sup, qry, params, alpha, K, order, loss, out, nullptr, false);
}

// The same step with every intermediate buffer in the static scratch array instead of the context's workspace: no
// device memory is allocated or freed anywhere below (the persistent words -- table bases, status -- stay where
// gm_create put them).  Kernel timing is off for the call: its events would have to be created.
extern "C" int gm_meta_step_static(gm_ctx* c, int32_t T, const gm_set* sup, const gm_set* qry, const gm_params* params,
                                   float alpha, int32_t K, int32_t order, float* loss, gm_grads* out) {
    if (!c) return GM_ERR_ARG;
    if (!c->static_scratch) return fail(c, GM_ERR_HIP, "the static scratch array was not located at gm_create");
    char* const ws = c->ws;
    const size_t ws_bytes = c->ws_bytes, persistent = c->persistent;
    const bool prof_on = c->prof_on;
    c->ws = c->static_scratch;
    c->ws_bytes = GM_STATIC_SCRATCH_BYTES;
    c->persistent = 0;
    c->prof_on = false;
    const int rc = gm_meta_step(c, T, sup, qry, params, alpha, K, order, loss, out);
    c->ws = ws;
    c->ws_bytes = ws_bytes;
    c->persistent = persistent;
    c->prof_on = prof_on;
    if (rc == GM_ERR_WORKSPACE) {
        const std::string why = c->err;
        return fail(c, GM_ERR_WORKSPACE, "the call does not fit the %d MiB of static scratch of gm_meta_step_static (%s); "
                    "use gm_meta_step with a workspace", (int)GM_STATIC_SCRATCH_MIB, why.c_str());
    }
    return rc;
}

static void host_layout(const gm_ctx* c, Batch& B, int T, const gm_set* sup, const gm_set* qry) {
    B.T = T; B.sup = sup; B.qry = qry; B.table = false;
    B.poff_s.assign(T + 1, 0);
    B.poff_q.assign(T + 1, 0);
    for (int t = 0; t < T; ++t) {
        B.poff_s[t + 1] = B.poff_s[t] + round_up64(sup->task_offsets[t + 1] - sup->task_offsets[t], c->row_pad);
        B.poff_q[t + 1] = B.poff_q[t] + round_up64(qry->task_offsets[t + 1] - qry->task_offsets[t], c->row_pad);
    }
}
static WavePlan whole_batch_plan(const Batch& B) {
    WavePlan p;
    const int T = B.T;
    p.t0 = 0; p.t1 = T;
    p.s0 = 0; p.s1 = B.sup->n_samples; p.q0 = 0; p.q1 = B.qry->n_samples;
    p.ps0 = 0; p.ps1 = B.poff_s[T]; p.pq0 = 0; p.pq1 = B.poff_q[T];
    p.ls0 = 0; p.ls1 = B.sup->nnz; p.lq0 = 0; p.lq1 = B.qry->nnz;
    return p;
}
// bytes of the index side and of the dense side of a batch run as ONE wave of tasks
static void one_wave_bytes(const gm_ctx* c, int T, const gm_set* sup, const gm_set* qry, int K, int order, bool mat_apart,
                           size_t* index_bytes, size_t* dense_bytes) {
    Batch B;
    host_layout(c, B, T, sup, qry);
    B.pair_rows = pair_rows(c, B);
    const WavePlan p = whole_batch_plan(B);
    WaveDims d = wave_dims(c, B, p, pick_bm(c, B), K, order);
    d.mat_apart = mat_apart;
    Arena ia, da;
    ia.cap = da.cap = ~(size_t)0 >> 1;
    BatchBufs b;
    WaveBufs w;
    alloc_batch_index(c, ia, b, T, sup->n_samples, qry->n_samples, sup->nnz + qry->nnz, 0, true);
    alloc_wave_index(c, ia, w, d);
    alloc_batch_dense(c, da, b, T, B.poff_s[T], B.poff_q[T], true);
    alloc_wave_dense(c, da, w, d, K, order);
    *index_bytes = ia.off;
    *dense_bytes = da.off;
}
// Whether gm_meta_train_step's batch runs as one wave with `top` bytes at the workspace's end taken (no lists then)
static bool runs_as_one_wave(const gm_ctx* c, int T, const gm_set* sup, const gm_set* qry, int K, int order, size_t top) {
    if (T < 0 || T > most_wave_tasks(c) || !sup->task_offsets || !qry->task_offsets || sup->n_samples < 0 || qry->n_samples < 0 ||
        sup->task_offsets[T] != sup->n_samples || qry->task_offsets[T] != qry->n_samples || K < 0 || sup->nnz + qry->nnz >= ((int64_t)1 << 31))
        return false;   // (several waves, or the step reports what is wrong)
    size_t index_bytes, dense_bytes;
    one_wave_bytes(c, T, sup, qry, K, order, false, &index_bytes, &dense_bytes);
    return c->persistent + index_bytes + dense_bytes + top + 256 <= c->ws_bytes;
}

extern "C" int gm_meta_train_step(gm_ctx* c, int32_t T, const gm_set* sup, const gm_set* qry, const gm_params* params,
                                  float alpha, int32_t K, int32_t order, float beta, float* loss, float* task_loss) {
    if (!c) return GM_ERR_ARG;
    if (!sup || !qry || sup->nnz < 0 || qry->nnz < 0) return fail(c, GM_ERR_ARG, "null set / negative size");
    if (!params || !params->W || !params->b) return fail(c, GM_ERR_ARG, "null params");
    HIPCHK(c, hipSetDevice(c->device));
    const int L = c->L, D = c->D;
    // the meta-gradient of this iteration lives at the top of the workspace, the step gets what is below it: its dense part, and
    // where the tasks do not run as one wave (which adds to the tables itself) the row lists
    int64_t n_dense = 0;
    for (int l = 0; l < L; ++l) n_dense += (int64_t)(c->dims[l] + 1) * c->dims[l + 1];
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const bool lists = c->F > 0 && !runs_as_one_wave(c, T, sup, qry, K, order, up((size_t)n_dense * 4) + 256);
    const int64_t capacity = lists ? std::min<int64_t>(sup->nnz + qry->nnz, c->field_base[c->F]) : 0;
    const size_t need = up((size_t)n_dense * 4) + up((size_t)capacity * 8) + up((size_t)capacity * std::max(D, 1) * 4) + 256;
    if (need + c->persistent + (1 << 20) > c->ws_bytes)
        return fail(c, GM_ERR_WORKSPACE, "workspace of %zu bytes cannot hold the meta-gradient (%zu bytes) beside the step", c->ws_bytes, need);
    const size_t full = c->ws_bytes;
    char* top = c->ws + (full - need) / 256 * 256;
    float* dense = reinterpret_cast<float*>(top);
    int64_t* rows = reinterpret_cast<int64_t*>(top + up((size_t)n_dense * 4));
    float* grad = reinterpret_cast<float*>(reinterpret_cast<char*>(rows) + up((size_t)capacity * 8));
    int64_t* n_rows = reinterpret_cast<int64_t*>(reinterpret_cast<char*>(grad) + up((size_t)capacity * std::max(D, 1) * 4));
    std::vector<float*> dW(L), db(L);
    {
        float* p = dense;
        for (int l = 0; l < L; ++l) {
            dW[l] = p; p += (int64_t)c->dims[l] * c->dims[l + 1];
            db[l] = p; p += c->dims[l + 1];
        }
    }
    gm_grads out;
    memset(&out, 0, sizeof out);
    out.dW = dW.data(); out.db = db.data();
    out.emb_rows = rows; out.emb_grad = grad; out.n_emb_rows = n_rows; out.emb_rows_capacity = capacity;
    out.task_loss = task_loss;
    c->ws_bytes = static_cast<size_t>(top - c->ws);
    EmbUpdate xi{const_cast<float*>(params->emb), -beta};
    const int rc = meta_step_impl(c, T, sup, qry, params, alpha, K, order, loss, &out, nullptr, false, &xi);
    c->ws_bytes = full;
    if (rc != GM_OK) return rc;
    hipStream_t st = c->stream;
    int64_t h_rows = 0;
    if (!xi.done) HIPCHK(c, hipMemcpyAsync(&h_rows, n_rows, sizeof h_rows, hipMemcpyDeviceToHost, st));
    for (int l = 0; l < L; ++l) {
        launch_axpy(st, (int64_t)c->dims[l] * c->dims[l + 1], -beta, dW[l], const_cast<float*>(params->W[l]));
        launch_axpy(st, c->dims[l + 1], -beta, db[l], const_cast<float*>(params->b[l]));
    }
    if (!xi.done) HIPCHK(c, hipStreamSynchronize(st));
    if (c->F > 0 && h_rows > 0) {
        Prof p(c, "scatter_add", (double)h_rows * (12.0 * D + 8), 0);
        launch_scatter_add(st, D, const_cast<float*>(params->emb), rows, grad, h_rows, -beta);
    }
    HIPCHK(c, hipStreamSynchronize(st));
    HIPCHK(c, hipGetLastError());
    prof_drain(c);
    return GM_OK;
}

// The same iteration for any number of lookups.  Tasks in several waves: the sparse meta-gradient is accumulated in a
// table-shaped buffer of the caller's and applied to the tables in one streaming pass that clears the buffer again.  One wave:
// the segment reduction adds to the tables itself and the buffer stays as it is, all zero (48 tasks x (512 + 512) rows, 64
// tables of 131,072 rows: that pass over 4 GB was 1.2 ms of 13.7).
extern "C" int gm_meta_train_step_table(gm_ctx* c, int32_t T, const gm_set* sup, const gm_set* qry, const gm_params* params,
                                        float alpha, int32_t K, int32_t order, float beta, float* loss, float* task_loss,
                                        float* emb_grad_table) {
    if (!c) return GM_ERR_ARG;
    if (!sup || !qry || sup->nnz < 0 || qry->nnz < 0) return fail(c, GM_ERR_ARG, "null set / negative size");
    if (!params || !params->W || !params->b) return fail(c, GM_ERR_ARG, "null params");
    if (c->F > 0 && (!emb_grad_table || !params->emb)) return fail(c, GM_ERR_ARG, "null emb_grad_table / emb");
    if ((reinterpret_cast<uintptr_t>(emb_grad_table) | reinterpret_cast<uintptr_t>(params->emb)) & 15)
        return fail(c, GM_ERR_ARG, "emb_grad_table and emb must be 16-byte aligned");
    HIPCHK(c, hipSetDevice(c->device));
    const int L = c->L, D = c->D;
    int64_t n_dense = 0;
    for (int l = 0; l < L; ++l) n_dense += (int64_t)(c->dims[l] + 1) * c->dims[l + 1];
    const size_t dense_bytes = ((size_t)n_dense * 4 + 255) & ~(size_t)255;
    const size_t need = dense_bytes + 512;   // the dense meta-gradient and the row counter, at the top of the workspace
    if (need + c->persistent + (1 << 20) > c->ws_bytes)
        return fail(c, GM_ERR_WORKSPACE, "workspace of %zu bytes cannot hold the dense meta-gradient (%zu bytes) beside the step", c->ws_bytes, need);
    const size_t full = c->ws_bytes;
    char* top = c->ws + (full - need) / 256 * 256;
    std::vector<float*> dW(L), db(L);
    {
        float* p = reinterpret_cast<float*>(top);
        for (int l = 0; l < L; ++l) {
            dW[l] = p; p += (int64_t)c->dims[l] * c->dims[l + 1];
            db[l] = p; p += c->dims[l + 1];
        }
    }
    gm_grads out;
    memset(&out, 0, sizeof out);
    out.dW = dW.data(); out.db = db.data();
    out.emb_grad_table = emb_grad_table;
    out.n_emb_rows = reinterpret_cast<int64_t*>(top + dense_bytes);   // (0 with the table-shaped output)
    out.task_loss = task_loss;
    c->ws_bytes = static_cast<size_t>(top - c->ws);
    EmbUpdate xi{const_cast<float*>(params->emb), -beta};
    const int rc = meta_step_impl(c, T, sup, qry, params, alpha, K, order, loss, &out, nullptr, false, &xi);
    c->ws_bytes = full;
    if (rc != GM_OK) return rc;
    hipStream_t st = c->stream;
    for (int l = 0; l < L; ++l) {
        launch_axpy(st, (int64_t)c->dims[l] * c->dims[l + 1], -beta, dW[l], const_cast<float*>(params->W[l]));
        launch_axpy(st, c->dims[l + 1], -beta, db[l], const_cast<float*>(params->b[l]));
    }
    if (c->F > 0 && !xi.done) {
        const int64_t n = c->field_base[c->F] * (int64_t)D;   // (D is a multiple of 4)
        Prof p(c, "table_update", 16.0 * n, 0);
        launch_axpy_clear(st, n, -beta, emb_grad_table, const_cast<float*>(params->emb));
    }
    HIPCHK(c, hipStreamSynchronize(st));
    HIPCHK(c, hipGetLastError());
    prof_drain(c);
    return GM_OK;
}

// ------------------------------------------------------------------------------------------------
// several iterations of Alg. 1 in one call, the index side of batch i+1 prepared while batch i computes
// ------------------------------------------------------------------------------------------------
// The index side of one batch, on the context's current stream, into the arena `ia`; mat_apart: without the pair-count matrices.
static int prepare_batch(gm_ctx* c, Arena& ia, int32_t T, const gm_set* sup, const gm_set* qry, int K, int order, bool mat_apart, Prepared& P) {
    int rc = check_set(c, sup, T, "support");
    if (rc != GM_OK) return rc;
    rc = check_set(c, qry, T, "query");
    if (rc != GM_OK) return rc;
    P = Prepared();
    JoinReq jr;
    Batch& B = P.B;
    B.T = T; B.sup = sup; B.qry = qry; B.table = false;
    if ((rc = begin_batch(c, B, ia, 0, true, nullptr))) return rc;
    P.bm = pick_bm(c, B);
    B.pair_rows = pair_rows(c, B);
    P.wp = whole_batch_plan(B);
    if (sup->nnz + qry->nnz >= ((int64_t)1 << 31)) return fail(c, GM_ERR_WORKSPACE, "the batch does not run as one wave of tasks");
    P.d = wave_dims(c, B, P.wp, P.bm, K, order);
    P.d.mat_apart = mat_apart;
    alloc_wave_index(c, ia, P.w, P.d);
    if (ia.overflow) return fail(c, GM_ERR_WORKSPACE, "the batch's index structures do not fit their arena");
    if (T > 0) {
        if ((rc = setup_wave(c, B, P.wp, P.bm, K, P.w, P.d, P.gs, P.gq))) return rc;
        if (c->F > 0) {
            jr.so = &B.b.so;
            jr.range = whole_batch_range(B);
            jr.n_sup_rows = P.d.Ps; jr.n_qry_rows = P.d.Pq;
            jr.pair_only = P.d.pair && !P.d.any_sparse;
        }
        if ((rc = run_index_wave(c, B, P.wp, P.w, &P.tf_cap, &P.max_bag, &P.max_tf, &jr))) return rc;
        if (jr.used) P.enc = jr.enc;
        bool on_side = false;
        if (!mat_apart && (rc = count_pairs(c, B, P.wp, P.w, P.d, P.tf_cap, P.max_bag, P.max_tf, false, P.pair, P.any_sparse, on_side))) return rc;
        if (c->row_path == 2 && P.any_sparse && c->adapt_rows)
            return fail(c, GM_ERR_CAPACITY, "pair-count path forced, but a task, count, bag or (task, field) exceeds its limits");
    }
    if (!jr.used) {
        launch_fill_u32(c->stream, c->d_status, ST_WORDS, 0);
        global_order(c, B, B.b.so, whole_batch_range(B), nullptr, nullptr, 0, nullptr);
    }
    HIPCHK(c, hipStreamSynchronize(c->stream));
    B.images.held.clear();
    HIPCHK(c, hipGetLastError());
    return GM_OK;
}

extern "C" int gm_meta_train(gm_ctx* c, int32_t n_iters, const int32_t* n_tasks, const gm_set* support, const gm_set* query,
                             const gm_params* params, float alpha, int32_t K, int32_t order, float beta, float* losses,
                             int32_t* n_done) {
    if (!c) return GM_ERR_ARG;
    if (n_done) *n_done = 0;
    if (n_iters < 0 || (n_iters > 0 && (!n_tasks || !support || !query || !losses)))
        return fail(c, GM_ERR_ARG, "bad iteration count / null arrays");
    if (K < 0 || (order != 1 && order != 2)) return fail(c, GM_ERR_ARG, "bad inner_steps / order");
    if (!params || !params->W || !params->b || (c->F > 0 && !params->emb)) return fail(c, GM_ERR_ARG, "null params");
    for (int l = 0; l < c->L; ++l)
        if (!params->W[l] || !params->b[l]) return fail(c, GM_ERR_ARG, "null layer pointer");
    if (n_iters == 0) return GM_OK;
    HIPCHK(c, hipSetDevice(c->device));
    const int L = c->L, D = c->D;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    // What the overlapped loop needs: two index arenas, the dense meta-gradient and the dense side of the largest batch.  Where two
    // batches' pair-count matrices do not fit, one batch's do: a step then counts its own before it starts (82 uneven tasks, two of
    // them large, 26 fields: 3.05 ms an iteration with both, 3.26 with one, 3.50 without overlap).
    bool overlapped = true, apart = false;
    size_t idx_bytes[2] = {0, 0}, dense_bytes[2] = {0, 0};   // [apart]
    for (int i = 0; i < n_iters; ++i) {
        const gm_set *s = &support[i], *q = &query[i];
        if (n_tasks[i] < 0 || !s->task_offsets || !q->task_offsets || s->nnz < 0 || q->nnz < 0 || s->n_samples < 0 || q->n_samples < 0 ||
            s->task_offsets[n_tasks[i]] != s->n_samples || q->task_offsets[n_tasks[i]] != q->n_samples ||
            s->nnz + q->nnz >= ((int64_t)1 << 31) || n_tasks[i] > most_wave_tasks(c)) {
            overlapped = false;   // (the per-iteration call takes the tasks in waves, or reports what is wrong)
            break;
        }
        for (int a = 0; a < 2; ++a) {
            size_t ib, db;
            one_wave_bytes(c, n_tasks[i], s, q, K, order, a == 1, &ib, &db);
            idx_bytes[a] = std::max(idx_bytes[a], up(ib) + 4096);
            dense_bytes[a] = std::max(dense_bytes[a], db);
        }
    }
    int64_t n_dense = 0;
    for (int l = 0; l < L; ++l) n_dense += (int64_t)(c->dims[l] + 1) * c->dims[l + 1];
    const size_t top = up((size_t)n_dense * 4) + 2 * 256;
    auto fits = [&](bool a) { return c->persistent + dense_bytes[a] + 2 * idx_bytes[a] + top + (1 << 20) <= c->ws_bytes; };
    apart = !fits(false);
    overlapped = overlapped && fits(apart);
    const size_t idx_max = idx_bytes[apart];
    if (!overlapped) {   // one iteration after the other (several waves of tasks, or a workspace for one batch only)
        for (int i = 0; i < n_iters; ++i) {
            const int rc = gm_meta_train_step(c, n_tasks[i], &support[i], &query[i], params, alpha, K, order, beta, losses + i, nullptr);
            if (rc != GM_OK) return rc;
            if (n_done) *n_done = i + 1;
        }
        return GM_OK;
    }
    const size_t full = c->ws_bytes;
    char* const top_p = c->ws + (full - top) / 256 * 256;
    float* dense = reinterpret_cast<float*>(top_p);
    int64_t* const n_rows = reinterpret_cast<int64_t*>(top_p + up((size_t)n_dense * 4));   // (no list: not written)
    char* const idx_p[2] = {top_p - 2 * idx_max, top_p - idx_max};
    const size_t dense_end = static_cast<size_t>(idx_p[0] - c->ws);
    std::vector<float*> dW(L), db(L);
    {
        float* p = dense;
        for (int l = 0; l < L; ++l) {
            dW[l] = p; p += (int64_t)c->dims[l] * c->dims[l + 1];
            db[l] = p; p += c->dims[l + 1];
        }
    }
    // the side-stream settings of single steps do not apply here: the second stream belongs to the preparation
    const int keep_sort = c->overlap_sort, keep_pairs = c->overlap_pairs;
    c->overlap_sort = c->overlap_pairs = 0;
    struct Restore {
        gm_ctx* c; size_t full; int s, p;
        ~Restore() { c->ws_bytes = full; c->overlap_sort = s; c->overlap_pairs = p; (void)hipStreamSynchronize(c->side); }
    } restore{c, full, keep_sort, keep_pairs};
    hipStream_t st = c->stream;
    Prepared P[2];
    auto prepare = [&](int i, bool on_side) -> int {
        Arena ia;
        ia.base = idx_p[i & 1]; ia.cap = idx_max; ia.off = 0;
        if (on_side) { std::swap(c->stream, c->side); std::swap(c->d_status, c->d_status_side); }
        const int rc = prepare_batch(c, ia, n_tasks[i], &support[i], &query[i], K, order, apart, P[i & 1]);
        if (on_side) { std::swap(c->stream, c->side); std::swap(c->d_status, c->d_status_side); }
        return rc;
    };
    int rc = prepare(0, false);
    if (rc != GM_OK) return rc;
    for (int i = 0; i < n_iters; ++i) {
        gm_grads out;
        memset(&out, 0, sizeof out);
        out.dW = dW.data(); out.db = db.data();
        out.n_emb_rows = n_rows;
        EmbUpdate xi{const_cast<float*>(params->emb), -beta};
        c->ws_bytes = dense_end;
        rc = meta_step_impl(c, n_tasks[i], &support[i], &query[i], params, alpha, K, order, losses + i, &out, &P[i & 1], true, &xi);
        c->ws_bytes = full;
        if (rc != GM_OK) { (void)hipStreamSynchronize(st); return rc; }
        // the two global back-propagation steps with the outer step size (Alg. 1), in place: xi's by the step itself
        for (int l = 0; l < L; ++l) {
            launch_axpy(st, (int64_t)c->dims[l] * c->dims[l + 1], -beta, dW[l], const_cast<float*>(params->W[l]));
            launch_axpy(st, c->dims[l + 1], -beta, db[l], const_cast<float*>(params->b[l]));
        }
        // the next batch's index side, on the second stream, while this batch computes, in the arena of batch i-1, which the
        // host has waited for
        int rc_next = GM_OK;
        if (i + 1 < n_iters) rc_next = prepare(i + 1, true);
        HIPCHK(c, hipStreamSynchronize(st));
        HIPCHK(c, hipGetLastError());
        prof_drain(c);
        if (n_done) *n_done = i + 1;
        if (rc_next != GM_OK) return rc_next;
    }
    return GM_OK;
}

// ------------------------------------------------------------------------------------------------
// one-task batches out of a flat record stream
// ------------------------------------------------------------------------------------------------
// lens[d * F + f] = length of bag f of source record perm[d], then one zero; flags offsets that are not monotone inside [0, nnz]
__global__ void group_lens_kernel(const int32_t* __restrict__ perm, int64_t n_dst, int F, const int64_t* __restrict__ bo,
                                  int64_t nnz, u32* lens, u32* status) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_dst * F) {
        if (i == n_dst * F) lens[i] = 0u;
        return;
    }
    const int64_t d = i / F;
    const int f = (int)(i - d * F);
    const int64_t b = (int64_t)perm[d] * F + f;
    const int64_t p0 = bo[b], p1 = bo[b + 1];
    const bool bad = p0 < 0 || p1 < p0 || p1 > nnz;
    if (bad) atomicOr(&status[ST_BAD_INDEX], 1u);
    lens[i] = bad ? 0u : (u32)(p1 - p0);
}
// The destination of up to two sets whose records lie one set after the other in perm (and their bags in offs).
struct GroupOut {
    int64_t n;   // records
    int64_t* bag_offsets;
    int32_t* indices;
    float *dense, *labels;
};
// One workgroup per 256 destination bags of a set: their lookups are one contiguous destination range; the bag of a lookup is
// found by bisection of the staged offsets (as in build_keys_kernel).  Also widens the offsets to 64 bits.
__global__ __launch_bounds__(256) void group_copy_kernel(const int32_t* __restrict__ perm, int F, const int64_t* __restrict__ bo,
                                                         const int32_t* __restrict__ idx_in, const u32* __restrict__ offs, GroupOut o0, GroupOut o1) {
    __shared__ u32 so[257];
    __shared__ int64_t src0[256];
    const int64_t bags0 = o0.n * F, blocks0 = (bags0 + 255) / 256;
    const bool second = (int64_t)blockIdx.x >= blocks0;
    const GroupOut& o = second ? o1 : o0;
    const int64_t first = second ? bags0 : 0, n_bags = o.n * F, b0 = ((int64_t)blockIdx.x - (second ? blocks0 : 0)) * 256;
    const u32 base = offs[first];
    const int nb = (int)min<int64_t>(256, n_bags - b0);
    for (int i = threadIdx.x; i <= nb; i += 256) {
        so[i] = offs[first + b0 + i] - base;
        o.bag_offsets[b0 + i] = (int64_t)so[i];
    }
    for (int i = threadIdx.x; i < nb; i += 256) {
        const int64_t d = (first + b0 + i) / F;
        src0[i] = bo[(int64_t)perm[d] * F + (first + b0 + i - d * F)];
    }
    __syncthreads();
    const u32 p0 = so[0], p1 = so[nb];
    for (u32 p = p0 + threadIdx.x; p < p1; p += 256) {
        int lo = 0, hi = nb;   // last bag with so[bag] <= p
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (so[mid] <= p) lo = mid;
            else hi = mid;
        }
        o.indices[p] = idx_in[src0[lo] + (p - so[lo])];
    }
}
__global__ void group_rows_kernel(const int32_t* __restrict__ perm, int nd, const float* __restrict__ dense, const float* __restrict__ labels,
                                  GroupOut o0, GroupOut o1) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (o0.n + o1.n) * (nd + 1)) return;
    int64_t d = i / (nd + 1);
    const int k = (int)(i - d * (nd + 1));
    const int64_t s = perm[d];
    const bool second = d >= o0.n;
    const GroupOut& o = second ? o1 : o0;
    if (second) d -= o0.n;
    if (k < nd) o.dense[d * nd + k] = dense[s * nd + k];
    else o.labels[d] = labels[s];
}
// A batch's place: its first record in (task, batch) order, how many of its records are support records, and where its
// support and its query records go in perm.
struct GroupBin { int32_t start, n_support, support0, query0; };
__global__ void group_expand_kernel(const uint16_t* __restrict__ key, int64_t n, u32* keys, u32* vals) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys[i] = key[i];
    vals[i] = (u32)i;
}
__global__ void group_place_kernel(const u32* __restrict__ keys, const u32* __restrict__ vals, int64_t n, const GroupBin* __restrict__ bins, int32_t* perm) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const GroupBin b = bins[keys[i]];
    const int32_t r = (int32_t)i - b.start;
    perm[r < b.n_support ? b.support0 + r : b.query0 + (r - b.n_support)] = (int32_t)vals[i];
}

// Dense (task, batch) numbers: the bits in which the numbers differ, where these are few, or the numbers less their smallest
// (`bits` of them; no keys where they would take more than GROUP_KEY_BITS).
// From GROUP_DEVICE_N records on the order is made on the device: 4,354 records 169 us a call on the host, 173 on the device, 16,398
// 193 / 195, 33,073 232 / 223, 66,140 308 / 284, 133,820 494 / 441 (26 bags a record; before, 65,536 records: 577).
// Up to GROUP_BINS_EACH numbers a record they are counted; sorted / counted, numbers below 8,192: 64 records 96 / 110 us, 512 115 / 125,
// 1,024 124 / 130, 2,048 153 / 152; 256 records with numbers below 1,024 109 / 110.
enum { GROUP_KEY_BITS = 13, GROUP_DEVICE_N = 32768, GROUP_BINS_EACH = 4 };
struct GroupKeys { int bits = -1, batch_bits = 0; uint64_t t0 = 0, b0 = 0; };
static GroupKeys group_keys(const int64_t* task, const int64_t* batch_id, int64_t n) {
    GroupKeys g;
    if (n <= 0) return g;
    auto bits_of = [](uint64_t span) { int b = 0; while (b < 64 && (span >> b)) ++b; return b; };
    uint64_t td = 0, bd = 0;
    for (int64_t i = 0; i < n; ++i) {
        td |= (uint64_t)(task[i] ^ task[0]);
        bd |= (uint64_t)(batch_id[i] ^ batch_id[0]);
    }
    int tb = bits_of(td), bb = bits_of(bd);
    if (tb + bb <= GROUP_KEY_BITS) {
        g.t0 = (uint64_t)task[0] >> tb << tb;
        g.b0 = (uint64_t)batch_id[0] >> bb << bb;
    } else {   // (numbers on both sides of a power of two, or of zero)
        const auto mt = std::minmax_element(task, task + n), mb = std::minmax_element(batch_id, batch_id + n);
        g.t0 = (uint64_t)*mt.first;
        g.b0 = (uint64_t)*mb.first;
        tb = bits_of((uint64_t)*mt.second - g.t0);
        bb = bits_of((uint64_t)*mb.second - g.b0);
        if (tb + bb > GROUP_KEY_BITS) return g;
    }
    g.bits = tb + bb;
    g.batch_bits = bb;
    return g;
}

// Record numbers in (task, batch) order, stream order inside a batch, where the numbers take more bits than a table holds: a
// stable counting sort, least significant digits first, over the bits in which the numbers (less their smallest) differ.
static std::vector<int32_t> record_order(const int64_t* task, const int64_t* batch_id, int64_t n) {
    std::vector<int32_t> order((size_t)n), next;
    for (int64_t i = 0; i < n; ++i) order[(size_t)i] = (int32_t)i;
    if (n < 2) return order;
    const auto mt = std::minmax_element(task, task + n), mb = std::minmax_element(batch_id, batch_id + n);
    const uint64_t t0 = (uint64_t)*mt.first, b0 = (uint64_t)*mb.first, t_span = (uint64_t)*mt.second - t0, b_span = (uint64_t)*mb.second - b0;
    auto bits_of = [](uint64_t span) { int b = 0; while (b < 64 && (span >> b)) ++b; return b; };
    const int tb = bits_of(t_span), bb = bits_of(b_span);
    // Few records with numbers far apart are compared: every pass also walks its digits' table.  256 records of one batch each,
    // 63-bit task numbers, 3 us (27 us by digits), 1024 20 (48), 2048 80 (67); 31-bit ones, 512 7.2 (7.4), 1024 22 (15).
    auto table = [](int bits) { const int passes = (bits + 12) / 13; return passes ? (int64_t)passes << ((bits + passes - 1) / passes) : 0; };
    if ((tb + bb <= 64 ? table(tb + bb) : table(tb) + table(bb)) > 24 * n) {
        std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return task[a] != task[b] ? task[a] < task[b] : batch_id[a] < batch_id[b]; });
        return order;
    }
    std::vector<uint64_t> key((size_t)n);
    auto sort_by_key = [&](int bits) {   // key[i]: of record i
        const int passes = (bits + 12) / 13, width = passes ? (bits + passes - 1) / passes : 0;
        next.resize((size_t)n);
        std::vector<int64_t> at((size_t)1 << width);
        for (int p = 0; p < passes; ++p) {
            const uint64_t mask = ((uint64_t)1 << width) - 1;
            std::fill(at.begin(), at.end(), 0);
            for (int64_t i = 0; i < n; ++i) ++at[(size_t)((key[(size_t)i] >> (p * width)) & mask)];
            int64_t run = 0;
            for (int64_t& a : at) { const int64_t cnt = a; a = run; run += cnt; }
            for (int64_t i = 0; i < n; ++i) {
                const int32_t r = order[(size_t)i];
                next[(size_t)at[(size_t)((key[(size_t)r] >> (p * width)) & mask)]++] = r;
            }
            order.swap(next);
        }
    };
    if (tb + bb <= 64) {
        for (int64_t i = 0; i < n; ++i)
            key[(size_t)i] = (bb < 64 ? ((uint64_t)task[i] - t0) << bb : 0) | ((uint64_t)batch_id[i] - b0);
        sort_by_key(tb + bb);
    } else {
        for (int64_t i = 0; i < n; ++i) key[(size_t)i] = (uint64_t)batch_id[i] - b0;
        sort_by_key(bb);
        for (int64_t i = 0; i < n; ++i) key[(size_t)i] = (uint64_t)task[i] - t0;
        sort_by_key(tb);
    }
    return order;
}

extern "C" int gm_group_batch(gm_ctx* c, int64_t n, int64_t nnz, const int64_t* task, const int64_t* batch_id,
                              const int64_t* bag_offsets, const int32_t* indices, const float* dense, const float* labels,
                              int32_t support_num, int32_t support_den, gm_set_buffers* sup, gm_set_buffers* qry,
                              int32_t* n_tasks) {
    if (!c) return GM_ERR_ARG;
    if (n < 0 || nnz < 0 || !sup || !qry || !n_tasks) return fail(c, GM_ERR_ARG, "bad sizes / null outputs");
    if (support_den <= 0 || support_num < 0 || support_num > support_den) return fail(c, GM_ERR_ARG, "support share must be in [0, 1]");
    if (n >= ((int64_t)1 << 31) / std::max(c->F, 1) || nnz >= ((int64_t)1 << 32))
        return fail(c, GM_ERR_ARG, "the stream must hold fewer than 2^31 bags and 2^32 lookups");
    if (n > 0 && (!task || !batch_id || !bag_offsets || !labels || (c->n_dense > 0 && !dense) || (nnz > 0 && !indices)))
        return fail(c, GM_ERR_ARG, "null stream array");
    gm_set_buffers* outs[2] = {sup, qry};
    for (gm_set_buffers* o : outs)
        if (!o->task_offsets || (n > 0 && (!o->bag_offsets || !o->labels || (c->n_dense > 0 && !o->dense) || (nnz > 0 && !o->indices))))
            return fail(c, GM_ERR_ARG, "null output buffer");
    HIPCHK(c, hipSetDevice(c->device));
    hipStream_t st = c->stream;
    const int F = c->F, nd = c->n_dense;
    // Records in (task, batch_id) order, stream order inside a batch: perm holds the support records of all batches, then the
    // query records.  Where (task, batch) takes few bits the batches follow from counts on the host, and the order itself is
    // made on the device from GROUP_DEVICE_N records on, else by the same counting sort on the host; numbers of more bits
    // are sorted on the host.
    std::vector<int32_t> perm;
    u32 total[3];      // offsets at the sets' borders
    HostImages keep;   // (the stream is drained on every way out, before what copies read and write goes)
    keep.st = st;
    keep.held.resize(1);
    Arena both;
    both.base = c->ws; both.cap = c->ws_bytes; both.off = c->persistent;
    int32_t* perm_dev = both.get<int32_t>(n + 2);
    u32* lens_dev = both.get<u32>(n * F + 2);
    u32* scan_dev = both.get<u32>(scan_tmp_words(n * F + 1));
    sup->task_offsets[0] = qry->task_offsets[0] = 0;
    int32_t T = 0;
    int64_t nw[2] = {0, 0};
    auto split = [&](int64_t m) { return (m * support_num + support_den - 1) / support_den; };
    auto add_batch = [&](int64_t m) {
        const int64_t k = split(m);
        nw[0] += k;
        nw[1] += m - k;
        ++T;
        sup->task_offsets[T] = nw[0];
        qry->task_offsets[T] = nw[1];
    };
    bool on_device = false;
    const GroupKeys gk = group_keys(task, batch_id, n);
    if (gk.bits >= 0 && ((int64_t)1 << gk.bits) <= GROUP_BINS_EACH * n) {
        const int64_t n_bins = (int64_t)1 << gk.bits;
        std::vector<char>& image = keep.held[0];   // the bins, then the keys: one upload
        image.resize((size_t)n_bins * sizeof(GroupBin) + (size_t)n * sizeof(uint16_t));
        GroupBin* bins = reinterpret_cast<GroupBin*>(image.data());
        uint16_t* key = reinterpret_cast<uint16_t*>(bins + n_bins);
        for (int64_t i = 0; i < n; ++i)
            key[i] = (uint16_t)((((uint64_t)task[i] - gk.t0) << gk.batch_bits) | ((uint64_t)batch_id[i] - gk.b0));
        std::vector<int32_t> count((size_t)n_bins * 4);   // (four tables: neighbouring records are often of one batch)
        for (int64_t i = 0; i < n; ++i) ++count[(size_t)((i & 3) * n_bins + key[i])];
        int32_t start = 0;
        for (int64_t k = 0; k < n_bins; ++k) {
            const int32_t m = count[(size_t)k] + count[(size_t)(n_bins + k)] + count[(size_t)(2 * n_bins + k)] + count[(size_t)(3 * n_bins + k)];
            bins[k] = GroupBin{start, (int32_t)split(m), (int32_t)nw[0], (int32_t)nw[1]};
            start += m;
            if (m > 0) add_batch(m);
        }
        for (int64_t k = 0; k < n_bins; ++k) bins[k].query0 += (int32_t)nw[0];
        Arena sort = both;
        char* image_dev = sort.get<char>(image.size());
        u32 *keys = sort.get<u32>(n), *vals = sort.get<u32>(n), *keys_tmp = sort.get<u32>(n), *vals_tmp = sort.get<u32>(n);
        u32* hist = sort.get<u32>(radix_hist_words(n, 0));
        on_device = n >= GROUP_DEVICE_N && !sort.overflow;
        if (on_device) {
            const unsigned grid = (unsigned)((n + 255) / 256);
            HIPCHK(c, hipMemcpyAsync(image_dev, image.data(), image.size(), hipMemcpyHostToDevice, st));
            hipLaunchKernelGGL(group_expand_kernel, dim3(grid), dim3(256), 0, st, reinterpret_cast<const uint16_t*>(image_dev + n_bins * sizeof(GroupBin)), n, keys, vals);
            if (launch_radix_sort(st, keys, vals, keys_tmp, vals_tmp, n, std::max(1, gk.bits), hist) & 1) {
                std::swap(keys, keys_tmp);
                std::swap(vals, vals_tmp);
            }
            hipLaunchKernelGGL(group_place_kernel, dim3(grid), dim3(256), 0, st, keys, vals, n, reinterpret_cast<const GroupBin*>(image_dev), perm_dev);
        } else {
            perm.resize((size_t)n);
            for (int64_t i = 0; i < n; ++i) {
                GroupBin& b = bins[key[i]];
                perm[(size_t)(b.n_support > 0 ? (--b.n_support, b.support0++) : b.query0++)] = (int32_t)i;
            }
        }
    } else if (n > 0) {
        const std::vector<int32_t> order = record_order(task, batch_id, n);
        std::vector<int32_t> query;
        perm.reserve((size_t)n);
        query.reserve((size_t)n);
        for (int64_t i = 0; i < n;) {
            const int64_t ti = task[order[(size_t)i]], bi = batch_id[order[(size_t)i]];
            int64_t j = i + 1;
            while (j < n && task[order[(size_t)j]] == ti && batch_id[order[(size_t)j]] == bi) ++j;
            const int64_t k = split(j - i);
            perm.insert(perm.end(), order.begin() + i, order.begin() + i + k);
            query.insert(query.end(), order.begin() + i + k, order.begin() + j);
            add_batch(j - i);
            i = j;
        }
        perm.insert(perm.end(), query.begin(), query.end());
    }
    *n_tasks = T;
    // Both sets together, so that the host waits for the totals once; one after the other where the workspace holds only one.
    launch_fill_u32(st, c->d_status, ST_WORDS, 0);
    for (int w0 = 0; w0 < 2; w0 += both.overflow ? 1 : 2) {
        const int w1 = both.overflow ? w0 + 1 : 2;
        const int64_t nd_all = both.overflow ? nw[w0] : n, nbags = nd_all * F;
        if (both.overflow) {
            Arena ar;
            ar.base = c->ws; ar.cap = c->ws_bytes; ar.off = c->persistent;
            perm_dev = ar.get<int32_t>(nd_all + 1);
            lens_dev = ar.get<u32>(nbags + 2);
            scan_dev = ar.get<u32>(scan_tmp_words(nbags + 1));
            if (ar.overflow) return fail(c, GM_ERR_WORKSPACE, "workspace too small for the grouping (%zu bytes needed)", ar.off);
        }
        u32 hs[ST_WORDS];
        total[0] = total[1] = total[2] = 0;
        if (!on_device && nd_all > 0)
            HIPCHK(c, hipMemcpyAsync(perm_dev, perm.data() + (w0 == 1 ? nw[0] : 0), nd_all * sizeof(int32_t), hipMemcpyHostToDevice, st));
        if (nbags > 0) {
            // (one length past the last, zero, so that the exclusive scan's last entry is the total)
            hipLaunchKernelGGL(group_lens_kernel, dim3((unsigned)((nbags + 256) / 256)), dim3(256), 0, st, perm_dev, nd_all, F, bag_offsets, nnz,
                               lens_dev, c->d_status);
            launch_scan_u32(st, lens_dev, lens_dev, nbags + 1, scan_dev, nullptr);
            if (w1 - w0 == 2 && nw[0] > 0 && nw[1] > 0) HIPCHK(c, hipMemcpyAsync(&total[1], lens_dev + nw[0] * F, sizeof(u32), hipMemcpyDeviceToHost, st));
            HIPCHK(c, hipMemcpyAsync(&total[w1 - w0], lens_dev + nbags, sizeof(u32), hipMemcpyDeviceToHost, st));
        }
        for (int w = w0; w < w1; ++w) {
            outs[w]->n_samples = nw[w];
            outs[w]->nnz = 0;
        }
        int rc = read_status(c, hs);   // (synchronises: the offsets are trusted below)
        if (rc != GM_OK) return rc;
        if (hs[ST_BAD_INDEX]) return fail(c, GM_ERR_INDEX, "bag_offsets not monotone / beyond nnz");
        if (w1 - w0 == 2 && nw[1] == 0) total[1] = total[2];   // (a set without records: nothing of it was read back)
        for (int w = w0; w < w1; ++w)   // (after the copies to the host, each of which waits for the kernels before it)
            if (nw[w] * F == 0 && n > 0) launch_fill_u32(st, reinterpret_cast<u32*>(outs[w]->bag_offsets), 2, 0u);
        GroupOut go[2] = {};
        for (int w = w0; w < w1; ++w) {
            outs[w]->nnz = (int64_t)(total[w - w0 + 1] - total[w - w0]);
            go[w - w0] = GroupOut{nw[w], outs[w]->bag_offsets, outs[w]->indices, outs[w]->dense, outs[w]->labels};
        }
        const int64_t blocks = (go[0].n * F + 255) / 256 + (go[1].n * F + 255) / 256;
        if (blocks > 0)
            hipLaunchKernelGGL(group_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, st, perm_dev, F, bag_offsets, indices, lens_dev, go[0], go[1]);
        if (nd_all > 0)
            hipLaunchKernelGGL(group_rows_kernel, dim3((unsigned)((nd_all * (nd + 1) + 255) / 256)), dim3(256), 0, st, perm_dev, nd, dense, labels, go[0], go[1]);
        HIPCHK(c, hipStreamSynchronize(st));
    }
    keep.held.clear();
    HIPCHK(c, hipGetLastError());
    return GM_OK;
}

extern "C" int gm_scatter_add(gm_ctx* c, float* table, const int64_t* rows, const float* grad, int64_t n_rows,
                              float scale) {
    if (!c) return GM_ERR_ARG;
    if (n_rows < 0 || (n_rows > 0 && (!table || !rows || !grad))) return fail(c, GM_ERR_ARG, "bad scatter arguments");
    HIPCHK(c, hipSetDevice(c->device));
    launch_scatter_add(c->stream, c->D, table, rows, grad, n_rows, scale);
    HIPCHK(c, hipStreamSynchronize(c->stream));
    HIPCHK(c, hipGetLastError());
    return GM_OK;
}

// copies a padded [n, ld] buffer into a dense [n, d] one
__global__ void strip_pad_kernel(const float* src, int64_t n, int ld, int d, float* dst) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * d) return;
    const int64_t s = i / d;
    dst[i] = src[s * ld + (i - s * d)];
}
__global__ void iota_i32_kernel(int32_t* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = (int32_t)i;
}

extern "C" int gm_gather_pool(gm_ctx* c, int32_t T, const gm_set* set, const float* emb, float* x) {
    if (!c) return GM_ERR_ARG;
    if (T < 0) return fail(c, GM_ERR_ARG, "bad n_tasks");
    int rc = check_set(c, set, T, "set");
    if (rc != GM_OK) return rc;
    if (set->n_samples > 0 && (!x || (c->F > 0 && !emb))) return fail(c, GM_ERR_ARG, "null emb / x");
    HIPCHK(c, hipSetDevice(c->device));
    hipStream_t st = c->stream;
    Arena ar;
    ar.base = c->ws; ar.cap = c->ws_bytes; ar.off = c->persistent;
    int64_t* toff = ar.get<int64_t>(T + 1);
    u32* cnt = ar.get<u32>(2 * ((int64_t)T * c->F + 1));
    if (ar.overflow) return fail(c, GM_ERR_WORKSPACE, "workspace too small");
    HIPCHK(c, hipMemcpyAsync(toff, set->task_offsets, (T + 1) * sizeof(int64_t), hipMemcpyHostToDevice, st));
    // validate before the gather trusts offsets and indices
    SetView v = make_view(set, toff, 0, 0);
    if (c->F == 0 || T == 0) launch_fill_u32(st, c->d_status, ST_WORDS, 0);
    else
        launch_tf_count(st, c->F, 0, T, most_bags(set, set, 0, T, c->F), 2 * set->n_samples * c->F, v, v, c->d_field_base, set->nnz, set->nnz, uniform_rows(c), cnt, cnt + (int64_t)T * c->F + 1, c->d_status, false);
    u32 hs[ST_WORDS];
    rc = read_status(c, hs);
    if (rc != GM_OK) return rc;
    if (hs[ST_BAD_INDEX]) return fail(c, GM_ERR_INDEX, "index outside its table, or bag_offsets not monotone / beyond nnz");
    if (hs[ST_TOO_LARGE])
        return fail(c, GM_ERR_CAPACITY, "a bag has more than 65535 lookups, or a task more than 65536 samples in one set");
    // process in chunks of samples that fit the workspace
    const size_t mark = ar.off;
    const int ld0 = c->ld[0], d0 = c->dims[0];
    const size_t avail = c->ws_bytes - mark;
    int64_t chunk = (int64_t)(avail / ((size_t)(ld0 + 1) * sizeof(float))) - 128;
    if (chunk < 1) return fail(c, GM_ERR_WORKSPACE, "workspace too small");
    chunk = std::min<int64_t>(chunk, (int64_t)1 << 30);
    for (int64_t s0 = 0; s0 < set->n_samples; s0 += chunk) {
        const int64_t n = std::min(chunk, set->n_samples - s0);
        ar.off = mark;
        float* xp = ar.get<float>(n * ld0);
        int32_t* ident = ar.get<int32_t>(n);
        hipLaunchKernelGGL(iota_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, ident, n);
        Prof p(c, "gather_pool", 0, 0);
        launch_gather_pool(st, c->F, c->D, c->n_dense, c->d_field_base, emb, ld0,
                           PoolSet{set->bag_offsets, set->indices, set->dense, s0, n, ident, 0, xp, nullptr}, PoolSet{});
        hipLaunchKernelGGL(strip_pad_kernel, dim3((unsigned)((n * d0 + 255) / 256)), dim3(256), 0, st, xp, n, ld0, d0,
                           x + s0 * d0);
    }
    HIPCHK(c, hipStreamSynchronize(st));
    HIPCHK(c, hipGetLastError());
    prof_drain(c);
    return GM_OK;
}

__global__ void widen_u32_kernel(const u32* src, int64_t n, int64_t* dst) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = (int64_t)src[i];
}
// packs the gapped per-(task, field) row lists: dst[packed_base[tf] + u] = slot_rows[base[tf] + u]
__global__ void pack_slot_rows_kernel(const u32* slot_rows, const u32* base, const u32* n_slots, const u32* packed_base,
                                      int64_t out0, int64_t* dst) {
    const int tf = blockIdx.x;
    for (u32 u = threadIdx.x; u < n_slots[tf]; u += blockDim.x)
        dst[out0 + packed_base[tf] + u] = (int64_t)slot_rows[base[tf] + u];
}

extern "C" int gm_index_prep(gm_ctx* c, int32_t T, const gm_set* sup, const gm_set* qry, int64_t* slot_counts,
                             int64_t* slot_rows, int32_t* sup_slot, int32_t* qry_slot, int64_t* emb_rows,
                             int64_t* seg_counts, int64_t* n_emb_rows, int64_t capacity) {
    if (!c) return GM_ERR_ARG;
    if (T < 0) return fail(c, GM_ERR_ARG, "bad n_tasks");
    int rc = check_set(c, sup, T, "support");
    if (rc != GM_OK) return rc;
    rc = check_set(c, qry, T, "query");
    if (rc != GM_OK) return rc;
    if (!n_emb_rows || capacity < 0) return fail(c, GM_ERR_ARG, "bad outputs");
    HIPCHK(c, hipSetDevice(c->device));
    hipStream_t st = c->stream;
    const int F = c->F;
    Arena ar;
    ar.base = c->ws; ar.cap = c->ws_bytes; ar.off = c->persistent;
    Batch B;
    B.T = T; B.sup = sup; B.qry = qry;
    rc = begin_batch(c, B, ar, capacity, false, &ar);
    if (rc != GM_OK) return rc;
    std::vector<WavePlan> plans;
    rc = plan_waves(c, B, c->ws_bytes - ar.off, 1, 2, 64, plans);
    if (rc != GM_OK) return rc;
    const size_t mark = ar.off;
    int64_t packed0 = 0;
    bool ordered = false;
    for (const WavePlan& wp : plans) {
        ar.off = mark;
        const int Tw = wp.t1 - wp.t0;
        if (Tw == 0 || F == 0) continue;
        WaveBufs w;
        const WaveDims d = wave_dims(c, B, wp, 64, 0, 1);
        alloc_wave(c, ar, w, d, 1, 2);
        if (ar.overflow) return fail(c, GM_ERR_WORKSPACE, "internal: wave does not fit");
        Grp gs, gq;
        if ((rc = setup_wave(c, B, wp, 64, 0, w, d, gs, gq))) return rc;
        JoinReq jr;
        if (plans.size() == 1) {   // the batch-wide order is this wave's: both come out of one sort
            jr.so = &B.b.so;
            jr.range = whole_batch_range(B);
            jr.n_sup_rows = d.Ps; jr.n_qry_rows = d.Pq;
            jr.emb_rows = emb_rows; jr.seg_counts = seg_counts; jr.capacity = capacity; jr.n_rows = n_emb_rows;
            jr.slots = true;
        }
        rc = run_index_wave(c, B, wp, w, nullptr, nullptr, nullptr, &jr);
        if (rc != GM_OK) return rc;
        ordered = jr.used;
        const int64_t TF = (int64_t)Tw * F;
        hipLaunchKernelGGL(widen_u32_kernel, dim3((unsigned)((TF + 255) / 256)), dim3(256), 0, st, w.n_slots, TF,
                           slot_counts + (int64_t)wp.t0 * F);
        u32* total = w.cnt_q + TF;  // spare word
        launch_scan_u32(st, w.n_slots, w.cnt_s, TF, w.scan_tmp, total);  // cnt_s reused as the packed base
        hipLaunchKernelGGL(pack_slot_rows_kernel, dim3((unsigned)TF), dim3(64), 0, st, w.slot_rows, w.base_s, w.n_slots,
                           w.cnt_s, packed0, slot_rows);
        u32 h_total = 0;
        HIPCHK(c, hipMemcpyAsync(&h_total, total, sizeof(u32), hipMemcpyDeviceToHost, st));
        HIPCHK(c, hipMemcpyAsync(sup_slot + wp.ls0, w.sup_slot, d.nnz_s * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
        HIPCHK(c, hipMemcpyAsync(qry_slot + wp.lq0, w.qry_slot, d.nnz_q * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
        HIPCHK(c, hipStreamSynchronize(st));
        packed0 += h_total;
    }
    if (!ordered) {
        launch_fill_u32(st, c->d_status, ST_WORDS, 0);
        global_order(c, B, B.b.so, whole_batch_range(B), emb_rows, seg_counts, capacity, n_emb_rows);
    }
    u32 hs[ST_WORDS];
    rc = read_status(c, hs);
    if (rc != GM_OK) return rc;
    B.images.held.clear();   // (the stream has been drained)
    HIPCHK(c, hipGetLastError());
    prof_drain(c);
    if (hs[ST_CAPACITY])
        return fail(c, GM_ERR_CAPACITY, "emb_rows_capacity %lld is smaller than the %u rows touched", (long long)capacity,
                    hs[ST_NROWS]);
    return GM_OK;
}
