// C-ABI layer of libqsv.so: argument validation, workspace carving, plan cache, launch order.
// Every numeric step runs in the HIP kernels; nothing here touches amplitudes on the host.
#include <hip/hip_runtime.h>

#include <array>
#include <cstdio>
#include <cstring>
#include <deque>
#include <iterator>
#include <list>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "qsv.h"
#include "qsv_kernels.h"
#include "qsv_lower.h"
#include "qsv_plan.h"

using namespace qsv;

namespace {

constexpr size_t kAlign = 256;
constexpr size_t kOpsRegion = 4u << 20;  // persistent: uploaded pass programs
// Passes that go through at least this many bytes store their tiles nontemporally: the chip's last-level
// cache is 256 MiB.  Measured with two buffers in turn: 2 x 256 MiB (20 qubits x 32) 1206 -> 1140 us, 2 x 512 MiB
// (26 qubits) 3663 -> 3451 us; 2 x 128 MiB (24 qubits) 761 -> 849 us.
constexpr uint64_t kNtStoreBytes = 384ull << 20;
constexpr uint64_t kSplitBytes = 32ull << 20;    // see run_circuit
// Amplitudes of a layer's gradient rows (B slots n 2^n) from which one circuit per parameter is run instead of two (see
// qsv_param_shift_grad).  Its tables, and reading the unshifted states at the end of the last pass, take some 4 us a layer; up to 13
// qubits, where a row is one or two tiles, little else than rows is saved, and of a single layer least.  Measured in turn, two / one:
//   10 qubits  1 layer x 118 55.4 / 56.4 us (2^21.2); 2 x 63 74.6 / 76.8 (2^20.3), x 78 78.4 / 77.4 (2^20.6); 5 x 126 167 / 176
//              (2^20.3), x 52 206 / 194 (2^20.6)
//   11         1 x 29 49.4 / 50.4 (2^20.9), x 53 47.9 / 48.1 (2^21.2); 2 x 29 75.0 / 77.6 (2^20.3), x 71 82.2 / 81.4 (2^20.6);
//              5 x 23 162 / 178 (2^20.0), x 19 198 / 195 (2^20.3)
//   12         1 x 32 46.4 / 47.2 (2^20.6), x 16 54.5 / 54.3 (2^21.2); 2 x 13 81.1 / 83.2 (2^20.3), x 32 82.1 / 81.4 (2^20.6)
//   13         1 x 6 56.4 / 57.6 (2^20.9); 2 x 8 78.9 / 83.8 (2^19.7), x 5 90.9 / 88.8 (2^20.0); 5 x 4 240 / 256 (2^19.7)
//   14         1 x 1 60.6 / 62.8 (2^19.4), x 2 60.8 / 61.1 (2^19.8); 2 x 2 102.3 / 104.8 (2^18.8), x 1 126.6 / 121.5 (2^19.4)
//   15         1 x 1 65.6 / 64.2 (2^19.9); 16 x 256, 10 layers 98.4 / 52.7 ms (2^29).
constexpr uint64_t turn_amplitudes(int n, int layers) {
    const int single = n <= 14 && layers == 1 ? 1 : 0;
    if (n <= 12) return n == 10 || layers <= 2 ? 3ull << (19 + single) : 5ull << 18;
    return 1ull << ((n == 13 ? 20 : 19) + single);
}
// ... and from which the layer's rotations are applied to the start states first: that is one more pass or two over the
// batch for every layer.  Measured without / with: 15 x 4, 5 layers 502 / 549 us (2^21.9), 16 x 4, 6 layers 680 / 742 (2^23),
// 14 x 64, 4 layers 1141 / 1137 (2^24.8), 16 x 16, 6 layers 1662 / 1579 (2^25), 12 x 1024, 4 layers 3019 / 2587 (2^27), 16 x 256,
// 10 layers 52.7 / 49.7 ms.
constexpr uint64_t kAheadAmplitudes = 1ull << 25;
constexpr int kChunkBits = 12;
constexpr int kMaxBatch = 1 << 24;
constexpr int64_t kMaxAmplitudes = (int64_t)1 << 36;

std::string g_create_error;

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

int ceil_log2_i64(int64_t v) {
    int b = 0;
    while (((int64_t)1 << b) < v) ++b;
    return b;
}

// kSweep: of a fused reverse-mode sweep: groups end with their passes, the inverse is the circuit's mirror image for the
// paired interpreter.  kTurned: gradient rows turn an angle of the first layer (see Rows); kTurnedAhead: and that layer's
// unitaries are in the start states.  kGrouped: the circuit's plan as it is.  All but kPlain have Plan::groups.
enum PlanForm { kPlain = 0, kSweep = 1, kTurned = 2, kTurnedAhead = 3, kGrouped = 4 };

// A plan the context has built.  Entries are never destroyed before qsv_destroy and never move (a
// std::deque only grows at its end), so pointers to them, and the host arrays uploads read from,
// stay valid for the life of the context: also for a HIP graph that recorded such an upload.
struct CachedPlan {
    qsv_circuit c;
    int inverse, tile, grad, low;   // tile: the resolved tile size (the default depends on the rows)
    int defer = 0;                  // planned with deferred CNOTs (index maps)
    int direct = 0;                 // for the direct interpreter: `low_ops` is uploaded in place of plan.ops
    int form = kPlain;
    DirectPlan low_ops;
    std::vector<unsigned> mates;   // of a mirrored plan's passes: PassArgs::mate
    size_t maps_off = 0;            // uint32[plan.maps.size()]: the index maps of its passes
    Plan plan;
    bool resident = false;          // its arrays are in the ops region right now
    size_t dev_off;     // byte offset of the ops inside the ops region
    size_t order_off;   // int32[n_mats]: execution order -> (layer*n + qubit)
    size_t execof_off;  // int32[]: (layer*n + qubit) -> execution order; kSweep: execution order -> table entry;
                        // kTurnedAhead: qubit -> what its OP_TURN is called by
    size_t groups_off = 0;          // int32[plan.groups.size()]
    std::vector<int32_t> exec_of;
};

}  // namespace

struct qsv_ctx {
    int n = 0;
    int64_t batch = 0;
    int device = 0;
    hipStream_t stream = nullptr;
    float2* state = nullptr;
    char* ws = nullptr;
    size_t ws_bytes = 0;
    std::string err;
    int opt_tile = 0;
    int opt_naive = 0;
    int opt_low = 0;
    int opt_planes = 1;
    int opt_grad_layered = 1;
    int opt_nt_store = -1;   // -1: by state size
    int opt_rev = -1;        // every other pass takes its tiles in descending order; -1: yes
    int probe_count = 0;
    int opt_probe_layout = -1;  // probe pass: register run of the load and the store (-1: the highest)
    int64_t opt_grad_chunk = 0;
    int opt_split = -1;      // state rows of a launch sequence in two halves on two streams; -1: by state size
    int opt_prio = 1;        // raised issue priority around a tile's loads and stores (2 % off configs 3 and 4 with k_pass, none with k_pass_direct)
    int opt_small_apply = 1; // at most 10 qubits: qsv_apply_layers (up to small_apply_amplitudes) and reverse mode in one launch
    int opt_small_regs = 0;  // qsv_forward_small: amplitudes per thread = 2^this (2..4); 0: by batch size
    int opt_defer = -1;      // qsv_apply_layers defers CNOTs whose target lies outside a pass's tile; -1: when it can
    hipStream_t side = nullptr;          // second stream for that (default priority, non-blocking)
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    bool forked = false;                 // a caller further up already runs two halves on the two streams
    std::deque<CachedPlan> cache;
    size_t ops_used = 0;
};

namespace {

qsv_status fail(qsv_ctx* ctx, qsv_status st, const std::string& msg) {
    if (ctx) ctx->err = msg;
    return st;
}

qsv_status hip_fail(qsv_ctx* ctx, hipError_t e, const char* where) {
    return fail(ctx, QSV_ERR_HIP, std::string(where) + ": " + hipGetErrorString(e));
}

#define QSV_HIP(ctx, expr, where)                                \
    do {                                                         \
        hipError_t e__ = (expr);                                 \
        if (e__ != hipSuccess) return hip_fail(ctx, e__, where); \
    } while (0)

// Per-call scratch carved from the workspace after the persistent ops region.  Work on one
// stream is ordered, so consecutive calls may reuse the same bytes.
struct Arena {
    char* base;
    size_t off, limit;
    bool fixed;      // the library's fixed scratch array instead of the caller's workspace
    explicit Arena(qsv_ctx* c) : base(c->ws), off(kOpsRegion), limit(c->ws_bytes), fixed(false) {}
    Arena(void* fixed_scratch, size_t bytes) : base((char*)fixed_scratch), off(0), limit(bytes), fixed(true) {}
    void* take(size_t bytes) {
        const size_t a = align_up(bytes ? bytes : 1);
        if (off + a > limit) { need = off + a; return nullptr; }
        void* p = base + off;
        off += a;
        return p;
    }
    size_t remaining() const { return limit > off ? limit - off : 0; }
    size_t need = 0;
};

qsv_status ws_fail(qsv_ctx* ctx, const Arena& ar, const char* what) {
    char buf[200];
    if (ar.fixed)
        snprintf(buf, sizeof buf, "%s needs %zu bytes of scratch, more than the fixed array of %zu bytes: "
                 "use the entry point that works in the caller's workspace", what, ar.need, ar.limit);
    else
        snprintf(buf, sizeof buf, "workspace too small for %s: needs at least %zu bytes, has %zu", what,
                 ar.need, ar.limit);
    return fail(ctx, QSV_ERR_WORKSPACE, buf);
}

CircDev to_dev(const qsv_circuit& c, int n) {
    CircDev d;
    d.n = n;
    d.n_layers = c.n_layers;
    d.reupload = c.reupload;
    d.n_rot = c.n_rot;
    for (int i = 0; i < 3; ++i) d.rot[i] = c.rot[i];
    return d;
}

int chunk_blocks(int bits) { return bits > kChunkBits ? 1 << (bits - kChunkBits) : 1; }

bool same_circuit(const qsv_circuit& a, const qsv_circuit& b) {
    if (a.n_layers != b.n_layers || a.reupload != b.reupload || a.n_rot != b.n_rot ||
        a.entangler != b.entangler)
        return false;
    for (int i = 0; i < a.n_rot; ++i)
        if (a.rot[i] != b.rot[i]) return false;
    return true;
}

// build_plan's results, kept for the contexts of the whole process: planning depends on the circuit's shape and the sizes
// only and takes longer than the call it is for (20 qubits, 20 layers 25 ms, 4.4 ms there and back; 26 qubits, 30 layers
// 129 and 10.8 ms), and programs make several contexts for one circuit.  The latest kKeptPlans plans, and no more than
// kKeptPlanBytes of operations, are held; any thread may ask.
constexpr size_t kKeptPlans = 64, kKeptPlanBytes = (size_t)8 << 20;

std::shared_ptr<const Plan> planned(const qsv_circuit& c, int n, int64_t rows, bool inverse, int tile, bool grad, int low,
                                    bool defer) {
    // of the circuit, what build_plan looks at; of the rows, the number of index bits
    const std::array<int, 11> key = {c.n_layers, c.reupload, c.n_rot > 0, c.entangler, n, ceil_log2_i64(rows),
                                     inverse,    tile,       grad,        low,         defer};
    struct Kept { std::array<int, 11> key; std::shared_ptr<const Plan> plan; };
    static std::mutex mu;
    static std::list<Kept> kept;       // the latest first
    {
        std::lock_guard<std::mutex> lock(mu);
        for (auto it = kept.begin(); it != kept.end(); ++it)
            if (it->key == key) {
                kept.splice(kept.begin(), kept, it);
                return it->plan;
            }
    }
    auto plan = std::make_shared<const Plan>(build_plan(c, n, rows, inverse, tile, grad, low, defer));
    std::lock_guard<std::mutex> lock(mu);
    kept.push_front({key, plan});
    size_t count = 0, bytes = 0;
    for (auto it = kept.begin(); it != kept.end();) {
        bytes += it->plan->ops.size() * sizeof(Op);
        it = ++count > kKeptPlans || bytes > kKeptPlanBytes ? kept.erase(it) : std::next(it);
    }
    return plan;
}

int tile_of(const qsv_ctx* ctx, int64_t rows, int layers, int defer) {
    const int tile = ctx->opt_tile > 0 ? ctx->opt_tile : defer ? defer_tile(ctx->n, rows, layers) : default_tile(ctx->n, rows);
    return std::max(kMinTile, std::min(kMaxTile, tile));
}

// tiles of one row through one LDS plane (tiles of 2^14 have no other way): see kDirectMaxQubits
bool is_direct(const qsv_ctx* ctx, int tile) {
    return ctx->n >= tile && ctx->n <= kDirectMaxQubits && (ctx->opt_planes == 1 || tile == kMaxTile);
}

// The context's plan for a circuit, built if it has none yet: host memory only.
qsv_status find_plan(qsv_ctx* ctx, const qsv_circuit& c, int64_t rows, int inverse, int grad, CachedPlan** out, int defer = 0,
                     PlanForm form = kPlain) {
    const int tile = tile_of(ctx, rows, c.n_layers, defer);
    const bool sweep = form == kSweep;
    const int direct = is_direct(ctx, tile) ? 1 : 0;
    CachedPlan* hit = nullptr;
    for (CachedPlan& cp : ctx->cache)
        if (cp.inverse == inverse && cp.tile == tile && cp.grad == grad && cp.low == ctx->opt_low &&
            cp.defer == defer && cp.direct == direct && cp.form == form && same_circuit(cp.c, c)) {
            hit = &cp;
            break;
        }
    if (!hit) {
        CachedPlan cp;
        cp.c = c;
        cp.inverse = inverse;
        cp.tile = tile;
        cp.grad = grad;
        cp.low = ctx->opt_low;
        cp.defer = defer;
        cp.direct = direct;
        cp.form = form;
        auto build = [&](bool inv) {
            return planned(c, ctx->n, rows, inv, tile, grad != 0, ctx->opt_low, defer != 0);
        };
        if (direct && defer && inverse) {
            cp.plan = mirror_plan(*build(false));      // the mirror image of the circuit's own plan
        } else if (sweep && !defer && !inverse) {
            // Without deferral either direction plans as well as the other.  The way back is planned and the way there
            // is its mirror image: then the gates that an observable of a few qubits depends on come last, and what is
            // rounded before them shows less in it (<Z_0> of a ladder of 10 layers, 16 qubits: 7.8e-7 from 64 bits, the
            // other way round 9.6e-7, layer by layer 7.9e-7).
            cp.plan = mirror_plan(*build(true));
        } else {
            cp.plan = *build(inverse != 0);
        }
        if (cp.plan.gather)
            for (const Pass& ps : cp.plan.passes) cp.mates.push_back(line_mate(cp.plan, ps));
        else
            cp.mates.assign(cp.plan.passes.size(), 0);
        if (!cp.plan.complete) return fail(ctx, QSV_ERR_UNSUPPORTED, "internal: pass planner failed");
        if (form == kTurnedAhead) turn_first_layer(&cp.plan);
        if (form != kPlain) group_by_passes(&cp.plan);
        const SumAxes axes = sum_axes(c);
        const Rows what = form == kTurned ? Rows::turn : form == kTurnedAhead || !grad ? Rows::none : Rows::replace;
        if (direct && !lower_plan(cp.plan, what, &cp.low_ops, sweep && inverse ? &axes : nullptr))
            return fail(ctx, QSV_ERR_UNSUPPORTED, "internal: lowering the pass plan failed");
        const size_t nm = cp.plan.mat_order.size();
        cp.exec_of.assign(nm, 0);
        if (sweep) {
            for (size_t g = 0; g + 1 < cp.plan.groups.size(); ++g)
                for (int32_t k = cp.plan.groups[g]; k < cp.plan.groups[g + 1]; ++k) cp.exec_of[k] = k + (int32_t)g;
        } else if (form == kTurnedAhead) {
            cp.exec_of.resize(ctx->n);
            for (int q = 0; q < ctx->n; ++q) cp.exec_of[q] = q;
        } else {
            for (size_t k = 0; k < nm; ++k) cp.exec_of[cp.plan.mat_order[k]] = (int32_t)k;
        }
        ctx->cache.push_back(std::move(cp));
        hit = &ctx->cache.back();
    }
    *out = hit;
    return QSV_OK;
}

// What a plan's arrays take of the ops region.
struct PlanRoom {
    size_t ops, table, maps, groups;
    explicit PlanRoom(const CachedPlan& cp)
        : ops(align_up(std::max(cp.plan.ops.size(), cp.low_ops.ops.size()) * sizeof(Op) + sizeof(Op))),
          table(align_up(std::max(cp.plan.mat_order.size(), cp.exec_of.size()) * sizeof(int32_t) + 4)),
          maps(align_up(cp.plan.maps.size() * sizeof(uint32_t) + 4)),
          groups(align_up(cp.plan.groups.size() * sizeof(int32_t) + 4)) {}
    size_t bytes() const { return ops + 2 * table + maps + groups; }
};

// Makes sure the plan's arrays are resident in the ops region.  Uploads are
// asynchronous copies on the context's stream from host arrays that live as long as the context.
// When the region is full, every plan in it is dropped from the region (not from the host) and the
// region is filled again from its start: the copies that overwrite it are ordered, on the stream,
// behind every kernel that read the old contents, so nothing waits on the host.
qsv_status upload_plan(qsv_ctx* ctx, CachedPlan& cp) {
    if (cp.resident) return QSV_OK;
    const PlanRoom room(cp);
    const size_t bytes = room.bytes();
    if (bytes > kOpsRegion) return fail(ctx, QSV_ERR_UNSUPPORTED, "circuit too long for the plan buffer");
    if (ctx->ops_used + bytes > kOpsRegion) {
        // While a call has work on the second stream, kernels there may still read the region, and
        // this upload would not be ordered behind them.
        if (ctx->forked)
            return fail(ctx, QSV_ERR_UNSUPPORTED, "the plans of this call do not fit the plan buffer together");
        for (CachedPlan& other : ctx->cache) other.resident = false;
        ctx->ops_used = 0;
    }
    cp.dev_off = ctx->ops_used;
    cp.order_off = cp.dev_off + room.ops;
    cp.execof_off = cp.order_off + room.table;
    cp.maps_off = cp.execof_off + room.table;
    cp.groups_off = cp.maps_off + room.maps;
    if (!cp.plan.groups.empty())
        QSV_HIP(ctx, hipMemcpyAsync(ctx->ws + cp.groups_off, cp.plan.groups.data(), cp.plan.groups.size() * sizeof(int32_t),
                                    hipMemcpyHostToDevice, ctx->stream),
                "upload groups");
    if (!cp.plan.maps.empty())
        QSV_HIP(ctx, hipMemcpyAsync(ctx->ws + cp.maps_off, cp.plan.maps.data(), cp.plan.maps.size() * sizeof(uint32_t),
                                    hipMemcpyHostToDevice, ctx->stream),
                "upload index maps");
    if (!cp.plan.ops.empty())
        QSV_HIP(ctx, hipMemcpyAsync(ctx->ws + cp.dev_off,
                                    cp.direct ? (const void*)cp.low_ops.ops.data() : (const void*)cp.plan.ops.data(),
                                    (cp.direct ? cp.low_ops.ops.size() : cp.plan.ops.size()) * sizeof(Op),
                                    hipMemcpyHostToDevice, ctx->stream),
                "upload plan");
    if (!cp.plan.mat_order.empty())
        QSV_HIP(ctx, hipMemcpyAsync(ctx->ws + cp.order_off, cp.plan.mat_order.data(), cp.plan.mat_order.size() * sizeof(int32_t),
                                    hipMemcpyHostToDevice, ctx->stream),
                "upload matrix order");
    if (!cp.exec_of.empty())
        QSV_HIP(ctx, hipMemcpyAsync(ctx->ws + cp.execof_off, cp.exec_of.data(), cp.exec_of.size() * sizeof(int32_t),
                                    hipMemcpyHostToDevice, ctx->stream),
                "upload matrix order");
    ctx->ops_used += bytes;
    cp.resident = true;
    return QSV_OK;
}

// Both: the plan, in the ops region.
qsv_status get_plan(qsv_ctx* ctx, const qsv_circuit& c, int64_t rows, int inverse, int grad, const CachedPlan** out,
                    int defer = 0, PlanForm form = kPlain) {
    CachedPlan* cp = nullptr;
    qsv_status st = find_plan(ctx, c, rows, inverse, grad, &cp, defer, form);
    if (st == QSV_OK) st = upload_plan(ctx, *cp);
    *out = cp;
    return st;
}

RowMap plain_rows(int n) {
    RowMap rm;
    rm.grad = 0; rm.two_p = 0; rm.per = 1; rm.row0 = 0; rm.slots_n = 1; rm.n = n;
    return rm;
}

// What a circuit needs before it can run: the pass plan (fused path) and the fused matrices, which
// are laid out in the plan's execution order (natural order on the one-gate-per-launch path).
struct Prepared {
    const CachedPlan* cp = nullptr;  // null: one-gate-per-launch path
    float* mats = nullptr;
    int mat_stride = 0;              // entries per sample in a per-sample table; 0: the matrices of the circuit run
    int layer_entries = 0;           // entries per layer of a table of layers
    const int* exec_of = nullptr;    // gradient: for the shifted matrices
    const double* scale = nullptr;   // gradient: the table's scalars (null: a plain table)
    MatForm form = MatForm::plain;   // of the table
};

size_t mats_table_bytes(const qsv_circuit& c, int n, int64_t samples) {
    // one extra entry: the interpreter prefetches the matrix after the one it is using
    return align_up(((size_t)(c.reupload ? samples : 1) * c.n_layers * n + 1) * 32);
}

// the matrix table followed by its scale table
size_t mats_bytes(const qsv_circuit& c, int n, int64_t samples) {
    return mats_table_bytes(c, n, samples) + align_up(mat_scale_bytes(to_dev(c, n), samples));
}

// layered: the layers of c run one by one as one-layer circuits (`run` = c with n_layers = 1): the plan
// is the one-layer circuit's, and the matrices of all layers are built by one launch, every layer's in
// that plan's order; layer l then runs with layer_of(prepared, l).  Otherwise run = c.
qsv_status prepare(qsv_ctx* ctx, const qsv_circuit& c, const qsv_circuit& run, bool layered, int64_t rows, int inverse,
                   int grad, const float* params, const float* feats, int64_t samples, float* mats, Prepared* out,
                   int defer, PlanForm plan_form = kPlain, double* residues = nullptr) {
    const int n = ctx->n;
    const bool has_u = (c.reupload + c.n_rot) > 0 && c.n_layers > 0;
    out->mats = mats;
    out->cp = nullptr;
    out->layer_entries = n;
    out->mat_stride = layered ? c.n_layers * n : 0;
    const int* order = nullptr;
    MatForm& form = out->form;
    form = MatForm::plain;
    if (!(ctx->opt_naive || n < kRegBits)) {
        qsv_status st = get_plan(ctx, run, rows, inverse, grad, &out->cp, defer, plan_form);
        if (st != QSV_OK) return st;
        order = reinterpret_cast<const int*>(ctx->ws + out->cp->order_off);
        out->exec_of = reinterpret_cast<const int*>(ctx->ws + out->cp->execof_off);
        // rows that share a tile and differ in their matrices read them per lane, as matrices
        if (!(n < out->cp->plan.tile && (c.reupload || grad)))
            form = out->cp->direct ? MatForm::direct : MatForm::factored;
    }
    if (!has_u) return QSV_OK;
    // groups with their scalars as entries of their own: so many more entries a table or layer
    const int n_groups = out->cp && !out->cp->plan.groups.empty() ? (int)out->cp->plan.groups.size() - 1 : 0;
    out->layer_entries = n + n_groups;
    out->mat_stride = layered ? c.n_layers * out->layer_entries : n_groups ? c.n_layers * n + n_groups : 0;
    double* scale = n_groups ? residues : grad && form != MatForm::plain
        ? reinterpret_cast<double*>(reinterpret_cast<char*>(mats) + mats_table_bytes(c, n, samples)) : nullptr;
    out->scale = scale;
    QSV_HIP(ctx, launch_build_mats(to_dev(c, n), params, feats, samples, inverse, order, layered && order ? n : 0,
                                   n_groups ? reinterpret_cast<const int*>(ctx->ws + out->cp->groups_off) : nullptr, n_groups,
                                   form, mats, scale, ctx->stream),
            "build matrices");
    return QSV_OK;
}

qsv_status prepare_circuit(qsv_ctx* ctx, const qsv_circuit& c, int64_t rows, int inverse, int grad,
                           const float* params, const float* feats, int64_t samples, float* mats,
                           Prepared* out, int defer = 0) {
    return prepare(ctx, c, c, false, rows, inverse, grad, params, feats, samples, mats, out, defer);
}

qsv_status prepare_layers(qsv_ctx* ctx, const qsv_circuit& c, const qsv_circuit& one, int64_t rows, int inverse,
                          const float* params, const float* feats, int64_t samples, float* mats, Prepared* out,
                          PlanForm form = kPlain, double* residues = nullptr) {
    return prepare(ctx, c, one, true, rows, inverse, 0, params, feats, samples, mats, out, 0, form, residues);
}

// What the wavefronts of a pass fetch ahead (see warm_scalar_cache), where all its tiles run at once and find the caches cold:
// with more of them, later ones find what earlier ones have fetched.  Without / with, 8 layers of a ladder: 16 qubits 67 -> 59
// us, 19 qubits 86 -> 77, 18 x 8 111 -> 105, 16 x 64 (1024 tiles) 127 -> 123.5, 16 x 128 (2048) 174 / 173, 16 x 256 295 /
// 296; 26 qubits, 30 layers 10.94 / 11.02 ms, 22 qubits (1024) 165.5 / 167.2 us.  Rows that have matrices of their own: 13
// x 128 53.3 -> 52.3, 13 x 512 79.3 / 80.2.  Reverse mode: 18 x 8 264 -> 256, 16 x 64 305 -> 299, re-uploading 469 / 477.
template <class Args>
void warm(Args* a, const DirectPass& low, uint64_t tiles) {
    if (a->n > 20 || tiles > (a->rowdep ? 256u : 1024u)) return;
    a->warm_ops = low.n_ops * (int)sizeof(DirectOp);
    a->warm_mats = low.n_mats * 32;
}

inline Prepared layer_of(const Prepared& all, int l) {
    Prepared pr = all;
    pr.mats = all.mats + (size_t)l * all.layer_entries * 8;
    return pr;
}

// Runs the prepared circuit on `rows` state rows starting at `state`.
// src (optional): per-sample start states [samples][2^n]; the rows then start from the state of
// their sample.  The fused path reads them in its first pass when a tile never spans two rows,
// otherwise a copy pass fills the rows first.
// zs (optional): what the gradient wants of the final states, <Z_q> per row scattered into out.
// The fused path computes it in its last pass (which then stores nothing) when a tile never spans
// two rows; otherwise the reduction kernels read the final states.  zpart: room for partials.
// unturned (optional, direct plans): see PassArgs; two results a row then, and what follows is for launch_turned_finish.
struct ZSpec {
    int q; double* out; Scatter sc; double* zpart;
    const float2* unturned; int64_t unturned_at; Residues ra, rb1, rb2;
};

// pong (needed when the plan defers CNOTs): a second buffer of the state's shape.  A pass with an
// index map reads one buffer and writes the other; the result always ends up in `state`.
qsv_status run_circuit(qsv_ctx* ctx, const qsv_circuit& c, const Prepared& pr, float2* state, int64_t rows,
                       int inverse, const float* ovr, const RowMap& rm, const float2* src = nullptr,
                       const ZSpec* zs = nullptr, float2* pong = nullptr) {
    const int n = ctx->n;
    const bool has_u = (c.reupload + c.n_rot) > 0;
    const int n_mats = has_u ? (pr.mat_stride > 0 ? pr.mat_stride : c.n_layers * n) : 0;
    const float* mats = pr.mats;
    const bool src_in_pass = src && pr.cp && n >= pr.cp->plan.tile && !pr.cp->plan.passes.empty();
    if (src && !src_in_pass)
        QSV_HIP(ctx, launch_gather_rows(src, n, rows, rm, state, ctx->stream), "gather rows");
    auto z_after = [&]() -> qsv_status {
        if (!zs) return QSV_OK;
        QSV_HIP(ctx, launch_expz_block(state, rows, n, zs->zpart, ctx->stream), "expz block");
        QSV_HIP(ctx, launch_expz_finish_scatter(zs->zpart, rows, n, zs->q, zs->out, zs->sc, ctx->stream),
                "expz finish");
        return QSV_OK;
    };
    if (!pr.cp) {
        auto layer_u = [&](int l) -> hipError_t {
            if (!has_u) return hipSuccess;
            for (int q = 0; q < n; ++q) {
                hipError_t e = launch_naive_u(state, rows, n, q, mats, ovr, l * n + q, n_mats,
                                              c.reupload, rm, ctx->stream);
                if (e != hipSuccess) return e;
            }
            return hipSuccess;
        };
        for (int li = 0; li < c.n_layers; ++li) {
            const int l = inverse ? c.n_layers - 1 - li : li;
            if (!inverse) QSV_HIP(ctx, layer_u(l), "naive rotation");
            if (c.entangler == QSV_ENT_CNOT_RING && n >= 2) {
                for (int i = 0; i < n; ++i) {
                    const int q = inverse ? n - 1 - i : i;
                    QSV_HIP(ctx, launch_naive_cnot(state, rows, n, q, (q + 1) % n, ctx->stream),
                            "naive cnot");
                }
            }
            if (c.entangler == QSV_ENT_CZ_LADDER && n >= 2)
                QSV_HIP(ctx, launch_naive_cz_ladder(state, rows, n, ctx->stream), "naive cz");
            if (inverse) QSV_HIP(ctx, layer_u(l), "naive rotation");
        }
        return z_after();
    }
    const CachedPlan* cp = pr.cp;
    if (!cp->resident) return fail(ctx, QSV_ERR_UNSUPPORTED, "internal: the plan was dropped from the plan buffer before use");
    const Plan& pl = cp->plan;
    const Op* dev_ops = reinterpret_cast<const Op*>(ctx->ws + cp->dev_off);
    const bool z_in_pass = zs && n >= pl.tile && !pl.passes.empty();
    if (zs && zs->unturned && !(z_in_pass && cp->direct))
        return fail(ctx, QSV_ERR_UNSUPPORTED, "internal: turned rows need the direct kernel");
    // Two rows or more: the rows go through the passes as two halves on two streams.  The halves
    // never meet (a tile lies inside one row when n > tile, and the geometry of the passes does not
    // depend on the number of rows), and each one's launch gaps and tails are covered by the
    // other's kernels.  Measured, 10 layers of a ring: 16 qubits x 64 rows 169 -> 157 us, 20 x 16 726 -> 601 us,
    // 24 x 4 3394 -> 3293 us; below 32 MiB the second launch of every pass costs more than that: 16 x 16
    // 115 -> 124 us, 14 x 16 89 -> 105 us.
    const uint64_t state_bytes = ((uint64_t)rows << n) * 8;
    const bool split = rows >= 2 && n > pl.tile && pl.passes.size() >= 2 && !ctx->forked &&
                       (ctx->opt_split >= 0 ? ctx->opt_split == 1 : state_bytes >= kSplitBytes);
    const int64_t rows_a = split ? rows / 2 : rows, rows_b = rows - rows_a;
    struct Join {      // the second stream always rejoins the caller's, also when a launch fails
        qsv_ctx* c; bool on;
        ~Join() {
            if (!on) return;
            if (hipEventRecord(c->ev_join, c->side) == hipSuccess) (void)hipStreamWaitEvent(c->stream, c->ev_join, 0);
        }
    } join{ctx, false};
    if (split) {
        QSV_HIP(ctx, hipEventRecord(ctx->ev_fork, ctx->stream), "fork");
        QSV_HIP(ctx, hipStreamWaitEvent(ctx->side, ctx->ev_fork, 0), "fork");
        join.on = true;
    }
    auto tiles_of = [&](int64_t r) -> uint64_t {
        if (cp->direct) return (uint64_t)r << (n - pl.tile);
        const int e = n + ceil_log2_i64(r);
        return e > pl.tile ? (1ull << (e - pl.tile)) : 1ull;
    };
    const int planes = cp->direct ? 1 : ctx->opt_planes;
    const int waves_per_group = std::max(1, (1 << (pl.tile - kRegBits)) / 64);
    // Which passes change buffers: those with an index map must; when their number is odd, one pass
    // without a map changes too (any pass may), so that the last one writes into `state`.  A plan in
    // which every pass has a map and their number is odd ends with a copy.
    size_t n_mapped = 0, extra_switch = pl.passes.size();
    for (const Pass& ps : pl.passes) n_mapped += ps.map_begin >= 0;
    if (n_mapped && (!pong || src || zs || n > 28))
        return fail(ctx, QSV_ERR_UNSUPPORTED, "internal: a plan with deferred CNOTs needs a second buffer");
    if (n_mapped & 1)
        for (size_t pi = 0; pi < pl.passes.size(); ++pi)
            if (pl.passes[pi].map_begin < 0) { extra_switch = pi; break; }
    float2* cur = state;
    const uint64_t touched = n_mapped ? 2 * state_bytes : state_bytes;   // what the passes go through in turn
    bool first = true;
    for (size_t pi = 0; pi < pl.passes.size(); ++pi) {
        const Pass& ps = pl.passes[pi];
        PassArgs a{};
        const bool switches = ps.map_begin >= 0 || pi == extra_switch;
        float2* const dst = switches ? (cur == state ? pong : state) : cur;
        a.state = dst;
        a.in = cur;
        a.imap = ps.map_begin >= 0 ? reinterpret_cast<const unsigned*>(ctx->ws + cp->maps_off) + ps.map_begin : nullptr;
        cur = dst;
        a.src = (first && src_in_pass) ? src : nullptr;
        first = false;
        const bool last = pi + 1 == pl.passes.size();
        a.zout = (last && z_in_pass) ? zs->zpart : nullptr;
        a.zq = zs ? zs->q : 0;
        a.nostore = a.zout ? 1 : 0;
        a.turns = zs && zs->unturned ? 1 : 0;
        a.unturned = a.zout ? zs->unturned : nullptr;
        a.ops = dev_ops + (cp->direct ? cp->low_ops.passes[pi].begin : ps.op_begin);
        a.mats = mats;
        a.exec_of = reinterpret_cast<const int*>(ctx->ws + cp->execof_off);
        a.ovr = ovr;
        a.total = (uint64_t)rows_a << n;
        a.nt_store = ctx->opt_nt_store >= 0 ? ctx->opt_nt_store : (touched >= kNtStoreBytes ? 1 : 0);
        // Every other pass walks the tiles downwards, so that it starts with what the pass before
        // wrote last and may still find in a cache (measured, two buffers of 32 to 256 MiB: 16 qubits
        // x 64 175 -> 166 us, 24 qubits 828 -> 761 us).  A pass without a map finds its tiles where they were: it keeps them
        // on their XCDs, whose L2s hold 32 MiB together (ladders of 2 layers: 21 qubits 67 -> 52 us, 52 without any reversing;
        // 22 qubits 63 -> 58).  Passes through a map read or write all over the row (kept on its XCD, 20 qubits x 4, 10
        // layers back 211 -> 216 us).
        a.rev = ctx->opt_rev != 0 && (pi & 1) ? (ps.map_begin < 0 ? 2 : 1) : 0;
        // Beside the other chunk of a reverse-mode sweep the passes share the chip with the transition sums, which a
        // raised priority holds up.  Measured, raised / not: 20 qubits x 32 12350 / 11900 us, 22 x 16 10607 / 10378, 24 x 4
        // 10700 / 10474, 18 x 64 1853 / 1838; 16 x 256, whose rows the caches hold, 2967 / 3010.
        a.prio = ctx->opt_prio && !(ctx->forked && n >= 18);
        a.n = n; a.c = ps.c; a.w = ps.w;
        a.n_mats = n_mats;
        a.rowdep = c.reupload;
        a.rm = rm;
        a.direct = cp->direct;
        a.gather = pl.gather ? 1 : 0;
        a.mate = a.gather && ps.map_begin >= 0 ? cp->mates[pi] : 0;
        a.s_in = a.s_out = a.first_mat = 0;
        a.g_sample0 = (unsigned)(rm.row0 / rm.per);
        a.g_rem0 = (unsigned)(rm.row0 % rm.per);
        if (cp->direct) {
            a.s_in = cp->low_ops.passes[pi].s_in;
            a.s_out = cp->low_ops.passes[pi].s_out;
            a.first_mat = cp->low_ops.passes[pi].first_mat;
            warm(&a, cp->low_ops.passes[pi], tiles_of(rows));
        }
        QSV_HIP(ctx, launch_pass(pl.tile, planes, a, tiles_of(rows_a), ctx->stream), "fused pass");
        if (!split) continue;
        // second half: rows rows_a .. rows - 1.  With a gradient row map the kernel works with global
        // row numbers (row0 moves); otherwise a row's matrices and start state are found relative to
        // the launch, so those pointers move with the state.
        PassArgs b = a;
        b.state = a.state + ((uint64_t)rows_a << n);
        b.in = a.in + ((uint64_t)rows_a << n);
        b.total = (uint64_t)rows_b << n;
        if (rm.grad) {
            b.rm.row0 = rm.row0 + rows_a;
            b.g_sample0 = (unsigned)(b.rm.row0 / rm.per);
            b.g_rem0 = (unsigned)(b.rm.row0 % rm.per);
        } else {
            if (b.src) b.src = b.src + ((uint64_t)rows_a << n);
            if (c.reupload && b.mats) b.mats = b.mats + (uint64_t)rows_a * (uint64_t)n_mats * 8;
        }
        if (b.zout)
            b.zout = b.zout + (b.unturned ? 3 : 1) * (uint64_t)rows_a * ((uint64_t)1 << (n - pl.tile)) * (uint64_t)waves_per_group;
        QSV_HIP(ctx, launch_pass(pl.tile, planes, b, tiles_of(rows_b), ctx->side), "fused pass");
    }
    if (split) {       // what follows on the caller's stream sees both halves
        join.on = false;
        QSV_HIP(ctx, hipEventRecord(ctx->ev_join, ctx->side), "join");
        QSV_HIP(ctx, hipStreamWaitEvent(ctx->stream, ctx->ev_join, 0), "join");
    }
    if (cur != state)
        QSV_HIP(ctx, hipMemcpyAsync(state, cur, state_bytes, hipMemcpyDeviceToDevice, ctx->stream), "copy back");
    if (z_in_pass) {
        // partials per row: tiles of the row x wavefronts of a workgroup
        const int64_t per_row = ((int64_t)1 << (n - pl.tile)) * (((int64_t)1 << (pl.tile - kRegBits)) / 64 > 0
                                                                    ? ((int64_t)1 << (pl.tile - kRegBits)) / 64 : 1);
        if (zs->unturned)
            QSV_HIP(ctx, launch_turned_finish(zs->zpart, rows, per_row, zs->out, zs->sc, zs->unturned_at, zs->ra, zs->rb1,
                                              zs->rb2, c.reupload, ctx->stream),
                    "z finish");
        else
            QSV_HIP(ctx, launch_zsum_finish(zs->zpart, rows, per_row, zs->out, zs->sc, ctx->stream), "z finish");
        return QSV_OK;
    }
    return z_after();
}

qsv_status bind_device(qsv_ctx* ctx) {
    QSV_HIP(ctx, hipSetDevice(ctx->device), "hipSetDevice");
    return QSV_OK;
}

}  // namespace

// ================================================================================================
extern "C" {

int64_t qsv_num_params(const qsv_circuit* c, int n_qubits) {
    if (!check_circuit(c, n_qubits, nullptr)) return -1;
    return (int64_t)c->n_layers * (c->reupload + c->n_rot) * n_qubits;
}

size_t qsv_workspace_bytes(int n_qubits, int batch) {
    if (n_qubits < 1 || n_qubits > 30 || batch < 1) return 0;
    const size_t n = (size_t)n_qubits, B = (size_t)batch;
    const size_t row_bytes = ((size_t)8) << n;
    size_t total = kOpsRegion;
    total += align_up(B * 64 * n * 32 + 32) + align_up(B * 64 * (n * 16 + 64));  // per-sample matrices + builder's side buffer, 64 layers
    total += align_up(B * 2 * (16 * 4 * n) * 32);             // shifted matrices, 16 layers x 4 slots
    total += align_up(B * (2 * 64 * 4 * n + 1) * 8);          // gradient values f[B][2P+1]
    total += align_up(B * (size_t)chunk_blocks(n_qubits) * 13 * 8 * 2);  // reduction partials
    total += align_up(B * 16) * 4;                            // norms, scales
    const size_t grad_states = row_bytes * 4 > ((size_t)256 << 20) ? row_bytes * 4 : ((size_t)256 << 20);
    total += grad_states + (8u << 20);
    // the second state buffer of qsv_apply_layers with deferred CNOTs (it shares the bytes above with the
    // gradient's circuit states; this makes sure a copy of the whole state fits whatever the batch)
    if (n_qubits <= 28 && B * row_bytes > grad_states) total += align_up(B * row_bytes - grad_states);
    return total;
}

size_t qsv_grad_workspace_bytes(int n_qubits, int batch, const qsv_circuit* c) {
    const size_t base = qsv_workspace_bytes(n_qubits, batch);
    if (base == 0 || !check_circuit(c, n_qubits, nullptr)) return 0;
    const size_t state_bytes = (size_t)8 << n_qubits;
    return base + align_up((size_t)batch * (size_t)(c->n_layers + 1) * state_bytes) + 4 * kAlign;
}

qsv_status qsv_create(qsv_ctx** out, int n_qubits, int batch, int device, void* hip_stream,
                      void* state_dev, void* ws_dev, size_t ws_bytes) {
    if (!out) { g_create_error = "out is NULL"; return QSV_ERR_INVALID_ARG; }
    *out = nullptr;
    if (n_qubits < 1 || n_qubits > 30) { g_create_error = "n_qubits must be in 1..30"; return QSV_ERR_INVALID_ARG; }
    if (batch < 1 || batch > kMaxBatch || ((int64_t)batch << n_qubits) > kMaxAmplitudes) {
        g_create_error = "batch must be in 1..2^24 with batch * 2^n_qubits <= 2^36";
        return QSV_ERR_INVALID_ARG;
    }
    if (device < 0) { g_create_error = "device must be >= 0"; return QSV_ERR_INVALID_ARG; }
    if (!state_dev || !ws_dev) { g_create_error = "state_dev and ws_dev must not be NULL"; return QSV_ERR_INVALID_ARG; }
    if (((uintptr_t)state_dev & 15) || ((uintptr_t)ws_dev & 255)) {
        g_create_error = "state_dev must be 16-byte aligned and ws_dev 256-byte aligned";
        return QSV_ERR_INVALID_ARG;
    }
    if (ws_bytes < qsv_workspace_bytes(n_qubits, batch)) {
        g_create_error = "workspace smaller than qsv_workspace_bytes(n_qubits, batch)";
        return QSV_ERR_WORKSPACE;
    }
    hipError_t e = hipSetDevice(device);
    if (e == hipSuccess) e = set_pass_attributes(device);
    if (e != hipSuccess) {
        g_create_error = std::string("HIP initialisation failed: ") + hipGetErrorString(e);
        return QSV_ERR_HIP;
    }
    qsv_ctx* ctx = new qsv_ctx();
    ctx->n = n_qubits;
    ctx->batch = batch;
    ctx->device = device;
    ctx->stream = static_cast<hipStream_t>(hip_stream);
    ctx->state = static_cast<float2*>(state_dev);
    ctx->ws = static_cast<char*>(ws_dev);
    ctx->ws_bytes = ws_bytes;
    e = hipStreamCreateWithFlags(&ctx->side, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_fork, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_join, hipEventDisableTiming);
    if (e != hipSuccess) {
        g_create_error = std::string("creating the second stream failed: ") + hipGetErrorString(e);
        qsv_destroy(ctx);
        return QSV_ERR_HIP;
    }
    *out = ctx;
    return QSV_OK;
}

void qsv_destroy(qsv_ctx* ctx) {
    if (!ctx) return;
    if (hipSetDevice(ctx->device) == hipSuccess) {
        if (ctx->ev_fork) (void)hipEventDestroy(ctx->ev_fork);
        if (ctx->ev_join) (void)hipEventDestroy(ctx->ev_join);
        if (ctx->side) (void)hipStreamDestroy(ctx->side);
    }
    delete ctx;
}

const char* qsv_last_error(const qsv_ctx* ctx) {
    return ctx ? ctx->err.c_str() : g_create_error.c_str();
}

qsv_status qsv_set_option(qsv_ctx* ctx, const char* name, int64_t value) {
    if (!ctx || !name) return QSV_ERR_INVALID_ARG;
    if (!strcmp(name, "tile_log2")) {
        if (value != 0 && (value < kMinTile || value > kMaxTile))
            return fail(ctx, QSV_ERR_INVALID_ARG, "tile_log2 must be 0 or in 10..14");
        ctx->opt_tile = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "low_bits")) {
        if (value != 0 && (value < 3 || value > kMinTile))
            return fail(ctx, QSV_ERR_INVALID_ARG, "low_bits must be 0 or in 3..10");
        ctx->opt_low = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "lds_planes")) {
        if (value != 1 && value != 2)
            return fail(ctx, QSV_ERR_INVALID_ARG, "lds_planes must be 1 or 2");
        ctx->opt_planes = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "grad_chunk_rows")) {
        if (value < 0 || value > 32768) return fail(ctx, QSV_ERR_INVALID_ARG, "grad_chunk_rows must be in 0..32768");
        ctx->opt_grad_chunk = value;
        return QSV_OK;
    }
    if (!strcmp(name, "reverse_passes")) {
        if (value < -1 || value > 1) return fail(ctx, QSV_ERR_INVALID_ARG, "reverse_passes must be -1, 0 or 1");
        ctx->opt_rev = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "split_streams")) {
        if (value < -1 || value > 1) return fail(ctx, QSV_ERR_INVALID_ARG, "split_streams must be -1, 0 or 1");
        ctx->opt_split = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "load_store_priority")) {
        if (value < 0 || value > 1) return fail(ctx, QSV_ERR_INVALID_ARG, "load_store_priority must be 0 or 1");
        ctx->opt_prio = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "small_apply")) {
        if (value < 0 || value > 1) return fail(ctx, QSV_ERR_INVALID_ARG, "small_apply must be 0 or 1");
        ctx->opt_small_apply = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "small_regs")) {
        if (value != 0 && (value < 2 || value > 4)) return fail(ctx, QSV_ERR_INVALID_ARG, "small_regs must be 0, 2, 3 or 4");
        ctx->opt_small_regs = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "defer_cnots")) {
        if (value < -1 || value > 1) return fail(ctx, QSV_ERR_INVALID_ARG, "defer_cnots must be -1, 0 or 1");
        ctx->opt_defer = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "probe_layout")) {
        if (value < -1 || value > kMaxTile - kRegBits)
            return fail(ctx, QSV_ERR_INVALID_ARG, "probe_layout must be -1 or in 0..10");
        ctx->opt_probe_layout = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "nt_store")) {
        if (value < -1 || value > 1) return fail(ctx, QSV_ERR_INVALID_ARG, "nt_store must be -1, 0 or 1");
        ctx->opt_nt_store = (int)value;
        return QSV_OK;
    }
    if (!strcmp(name, "grad_layered")) {
        ctx->opt_grad_layered = value != 0;
        return QSV_OK;
    }
    if (!strcmp(name, "naive")) {
        ctx->opt_naive = value != 0;
        return QSV_OK;
    }
    return fail(ctx, QSV_ERR_INVALID_ARG, std::string("unknown option ") + name);
}

qsv_status qsv_amp_encode(qsv_ctx* ctx, const float* x_dev, int64_t dim, float* norm_out_dev) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    if (!x_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "x_dev is NULL");
    if (dim < 1 || dim > ((int64_t)1 << ctx->n)) return fail(ctx, QSV_ERR_INVALID_ARG, "dim must be in 1..2^n");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    Arena ar(ctx);
    int nblk = (int)((dim + 4095) / 4096);
    if (nblk > 1024) nblk = 1024;
    double* partial = (double*)ar.take((size_t)ctx->batch * nblk * 8);
    double* inv = (double*)ar.take((size_t)ctx->batch * 8);
    if (!partial || !inv) return ws_fail(ctx, ar, "qsv_amp_encode");
    QSV_HIP(ctx, launch_encode(x_dev, ctx->batch, dim, ctx->n, partial, nblk, inv, norm_out_dev, ctx->state, ctx->stream), "encode");
    return QSV_OK;
}

qsv_status qsv_apply_layers(qsv_ctx* ctx, const qsv_circuit* c, const float* params_dev,
                            const float* feats_dev, int inverse) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    std::string why;
    if (!check_circuit(c, ctx->n, &why)) return fail(ctx, QSV_ERR_INVALID_ARG, why);
    if (inverse != 0 && inverse != 1) return fail(ctx, QSV_ERR_INVALID_ARG, "inverse must be 0 or 1");
    const int64_t P = qsv_num_params(c, ctx->n);
    if (P > 0 && !params_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "params_dev is NULL");
    if (c->reupload && !feats_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "reupload = 1 needs feats_dev");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    // States small enough that launches cost more than arithmetic: the whole call in one launch, gates in
    // registers and lane exchanges (the kernel of qsv_forward_small, started from the state).
    if (ctx->opt_small_apply != 0 && ctx->n <= kSmallMaxQubits && ctx->opt_tile == 0 && !ctx->opt_naive &&
        ((int64_t)ctx->batch << ctx->n) <= small_apply_amplitudes(ctx->n)) {
        const CircDev cd = to_dev(*c, ctx->n);
        const int regs = ctx->opt_small_regs ? ctx->opt_small_regs : small_choose_regs(cd, ctx->batch);
        if (regs != 0 && ctx->n - regs <= 8 && small_mats_per_group(cd, regs) <= kSmallMats) {
            QSV_HIP(ctx, launch_forward_small(regs, nullptr, 0, ctx->batch, cd, c->entangler, params_dev, feats_dev, inverse,
                                              inverse, 0, ctx->state, nullptr, nullptr, ctx->stream),
                    "apply_small");
            return QSV_OK;
        }
    }
    Arena ar(ctx);
    float* mats = (float*)ar.take(mats_bytes(*c, ctx->n, ctx->batch));
    if (!mats) return ws_fail(ctx, ar, "qsv_apply_layers");
    // CNOTs whose target lies outside a pass's tile can be carried by the pass's index map (fewer
    // passes over the state); such passes write a second buffer, taken from the workspace.
    const size_t state_bytes = ((size_t)ctx->batch << ctx->n) * 8;
    float2* pong = nullptr;
    int defer = 0;
    if (ctx->opt_defer != 0 && c->entangler == QSV_ENT_CNOT_RING && ctx->n <= 28 && !ctx->opt_naive &&
        ar.remaining() >= align_up(state_bytes)) {
        int tile = ctx->opt_tile > 0 ? ctx->opt_tile : defer_tile(ctx->n, ctx->batch, c->n_layers);
        if (ctx->n > tile) {
            pong = (float2*)ar.take(state_bytes);
            defer = pong ? 1 : 0;
        }
    }
    Prepared pr;
    st = prepare_circuit(ctx, *c, ctx->batch, inverse, 0, params_dev, feats_dev, ctx->batch, mats, &pr, defer);
    if (st != QSV_OK) return st;
    return run_circuit(ctx, *c, pr, ctx->state, ctx->batch, inverse, nullptr, plain_rows(ctx->n), nullptr, nullptr, pong);
}

// Every measurement kind; ar is where the kernels' partial results go (the caller's workspace, or the
// library's fixed scratch array).  The partials are written in full before they are read, so the
// bytes need no clearing between calls.
static qsv_status measure_impl(qsv_ctx* ctx, const qsv_measure_req* req, Arena& ar) {
    if (!req) return fail(ctx, QSV_ERR_INVALID_ARG, "req is NULL");
    if (!req->out_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "out_dev is NULL");
    if (req->reserved != 0) return fail(ctx, QSV_ERR_INVALID_ARG, "reserved must be 0");
    const int n = ctx->n;
    const int64_t B = ctx->batch;
    const uint64_t full = (n >= 64) ? ~0ull : ((1ull << n) - 1);
    qsv_status st;
    switch (req->kind) {
        case QSV_M_PROBS: {
            if ((st = bind_device(ctx)) != QSV_OK) return st;
            QSV_HIP(ctx, launch_probs(ctx->state, (uint64_t)B << n, (float*)req->out_dev, ctx->stream),
                    "probs");
            return QSV_OK;
        }
        case QSV_M_EXPZ_ALL:
        case QSV_M_EXPZ_ONE: {
            const int q = req->kind == QSV_M_EXPZ_ONE ? req->qubit : -1;
            if (req->kind == QSV_M_EXPZ_ONE && (q < 0 || q >= n))
                return fail(ctx, QSV_ERR_INVALID_ARG, "qubit out of range");
            if ((st = bind_device(ctx)) != QSV_OK) return st;
            double* partial = n > 12 ? (double*)ar.take((size_t)B * chunk_blocks(n) * 13 * 8) : nullptr;
            if (n > 12 && !partial) return ws_fail(ctx, ar, "qsv_measure(EXPZ)");
            if (expz_in_one_launch(n, B)) {       // a block has a row: no partial sums to combine
                QSV_HIP(ctx, launch_expz_small(ctx->state, B, n, q, (float*)req->out_dev, ctx->stream), "expz");
                return QSV_OK;
            }
            QSV_HIP(ctx, launch_expz_block(ctx->state, B, n, partial, ctx->stream), "expz block");
            QSV_HIP(ctx, launch_expz_finish(partial, B, n, q, (float*)req->out_dev, nullptr, ctx->stream),
                    "expz finish");
            return QSV_OK;
        }
        case QSV_M_MARGINAL:
        case QSV_M_PROJECT_ZERO: {
            if (req->mask == 0 || (req->mask & ~full)) return fail(ctx, QSV_ERR_INVALID_ARG, "mask must be a non-empty subset of the qubits");
            const int m = __builtin_popcountll(req->mask);
            const bool proj = req->kind == QSV_M_PROJECT_ZERO;
            if (!proj && m > 20) return fail(ctx, QSV_ERR_UNSUPPORTED, "marginal over more than 20 qubits");
            if (proj && req->renormalise != 0 && req->renormalise != 1)
                return fail(ctx, QSV_ERR_INVALID_ARG, "renormalise must be 0 or 1");
            const int64_t n_v = proj ? 1 : ((int64_t)1 << m);
            const int64_t nblk = chunk_blocks(n - m);
            if ((uint64_t)B * (uint64_t)n_v * (uint64_t)nblk > 0x7fffffffull)
                return fail(ctx, QSV_ERR_UNSUPPORTED, "marginal too large for one launch");
            if ((st = bind_device(ctx)) != QSV_OK) return st;
            double* partial = (double*)ar.take((size_t)B * n_v * nblk * 8);
            double* scale = (double*)ar.take((size_t)B * 8);
            if (!partial || !scale) return ws_fail(ctx, ar, "qsv_measure(MARGINAL/PROJECT)");
            QSV_HIP(ctx, launch_marginal_block(ctx->state, B, n, req->mask, n_v, partial, ctx->stream),
                    "marginal block");
            QSV_HIP(ctx, launch_marginal_finish(partial, B * n_v, nblk, (float*)req->out_dev,
                                                proj ? (req->renormalise ? 2 : 1) : 0, scale, ctx->stream),
                    "marginal finish");
            if (proj)
                QSV_HIP(ctx, launch_project(ctx->state, B, n, req->mask, scale, ctx->stream), "project");
            return QSV_OK;
        }
        case QSV_M_FIDELITY: {
            if (!req->x_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "x_dev is NULL");
            if (req->dim < 1 || req->dim > ((int64_t)1 << n)) return fail(ctx, QSV_ERR_INVALID_ARG, "dim must be in 1..2^n");
            if ((st = bind_device(ctx)) != QSV_OK) return st;
            int nblk = (int)((req->dim + 4095) / 4096);
            if (nblk > 1024) nblk = 1024;
            double* partial = (double*)ar.take((size_t)B * nblk * 3 * 8);
            if (!partial) return ws_fail(ctx, ar, "qsv_measure(FIDELITY)");
            QSV_HIP(ctx, launch_fidelity_block(ctx->state, B, n, req->x_dev, req->dim, partial, nblk, plain_rows(n), ctx->stream),
                    "fidelity block");
            QSV_HIP(ctx, launch_fidelity_finish(partial, nblk, B, (float*)req->out_dev, nullptr, ctx->stream),
                    "fidelity finish");
            return QSV_OK;
        }
        case QSV_M_SAMPLE: {
            if (req->shots < 0) return fail(ctx, QSV_ERR_INVALID_ARG, "shots must be >= 0");
            if (req->shots > 0 && !req->uniforms_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "uniforms_dev is NULL");
            if ((st = bind_device(ctx)) != QSV_OK) return st;
            unsigned long long* cum = (unsigned long long*)ar.take((size_t)B * chunk_blocks(n) * 8);
            if (!cum) return ws_fail(ctx, ar, "qsv_measure(SAMPLE)");
            // Finer sums, of 256 amplitudes each, where the scratch has room for them: they save the draws most of their
            // reading.  Up to 7 qubits the scan has only two steps at most, which are less than the search (64 rows x 1024
            // shots, scan / sums: 4 qubits 24 / 33 us, 7 qubits 27 / 33; 8 qubits 34 / 33, 9 qubits 53 / 33).
            unsigned long long* sub = n < 8 ? nullptr : (unsigned long long*)ar.take((size_t)B * chunk_blocks(n) * 16 * 8);
            QSV_HIP(ctx, launch_sample(ctx->state, B, n, req->uniforms_dev, req->shots, cum, sub,
                                       (long long*)req->out_dev, ctx->stream),
                    "sample");
            return QSV_OK;
        }
        default:
            return fail(ctx, QSV_ERR_INVALID_ARG, "unknown measurement kind");
    }
}

qsv_status qsv_forward_small(qsv_ctx* ctx, const float* x_dev, int64_t dim, const qsv_circuit* c,
                             const float* params_dev, const float* feats_dev, int decode, int kind, void* out_dev,
                             float* norm_out_dev) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    if (!x_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "x_dev is NULL");
    if (dim < 1 || dim > ((int64_t)1 << ctx->n)) return fail(ctx, QSV_ERR_INVALID_ARG, "dim must be in 1..2^n");
    std::string why;
    if (!check_circuit(c, ctx->n, &why)) return fail(ctx, QSV_ERR_INVALID_ARG, why);
    if (decode != 0 && decode != 1) return fail(ctx, QSV_ERR_INVALID_ARG, "decode must be 0 or 1");
    if (kind != QSV_M_PROBS && kind != QSV_M_EXPZ_ALL)
        return fail(ctx, QSV_ERR_INVALID_ARG, "kind must be QSV_M_PROBS or QSV_M_EXPZ_ALL");
    if (!out_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "out_dev is NULL");
    const int64_t P = qsv_num_params(c, ctx->n);
    if (P > 0 && !params_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "params_dev is NULL");
    if (c->reupload && !feats_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "reupload = 1 needs feats_dev");
    if (ctx->n > kSmallMaxQubits)
        return fail(ctx, QSV_ERR_UNSUPPORTED, "qsv_forward_small takes at most 10 qubits: use the separate calls");
    const CircDev cd = to_dev(*c, ctx->n);
    int regs = ctx->opt_small_regs;
    if (regs == 0) regs = small_choose_regs(cd, ctx->batch);
    if (regs == 0 || ctx->n - regs > 8 || small_mats_per_group(cd, regs) > kSmallMats)
        return fail(ctx, QSV_ERR_UNSUPPORTED,
                    "qsv_forward_small keeps at most 512 matrices per workgroup (layers * qubits, times the samples "
                    "that share a wavefront when the circuit re-uploads data): use the separate calls");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    QSV_HIP(ctx, launch_forward_small(regs, x_dev, dim, ctx->batch, cd, c->entangler, params_dev, feats_dev, 0, decode, kind,
                                      ctx->state, (float*)out_dev, norm_out_dev, ctx->stream),
            "forward_small");
    return QSV_OK;
}

qsv_status qsv_measure(qsv_ctx* ctx, const qsv_measure_req* req) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    Arena ar(ctx);
    return measure_impl(ctx, req, ar);
}

qsv_status qsv_measure_static(qsv_ctx* ctx, const qsv_measure_req* req) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    void* fixed = nullptr;     // this device's copy of the fixed array (address looked up once per device)
    QSV_HIP(ctx, static_scratch(ctx->device, &fixed), "address of the fixed scratch array");
    Arena ar(fixed, kStaticScratchBytes);
    return measure_impl(ctx, req, ar);
}

qsv_status qsv_pauli_expect(qsv_ctx* ctx, uint64_t xmask, uint64_t ymask, uint64_t zmask, float* out_dev) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    const int n = ctx->n;
    if (!out_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "out_dev is NULL");
    if ((xmask & ymask) || (xmask & zmask) || (ymask & zmask))
        return fail(ctx, QSV_ERR_INVALID_ARG, "xmask, ymask and zmask must not overlap");
    if ((xmask | ymask | zmask) >> n) return fail(ctx, QSV_ERR_INVALID_ARG, "mask names a qubit >= n_qubits");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    Arena ar(ctx);
    double* partial = (double*)ar.take((size_t)ctx->batch * chunk_blocks(n) * 2 * 8);
    if (!partial) return ws_fail(ctx, ar, "qsv_pauli_expect");
    QSV_HIP(ctx, launch_pauli(ctx->state, ctx->batch, n, xmask, ymask, zmask, partial, out_dev, ctx->stream),
            "pauli expectation");
    return QSV_OK;
}

qsv_status qsv_reset_fidelity(qsv_ctx* ctx, const qsv_circuit* c, const float* params_dev,
                              const float* feats_dev, uint64_t mask, const float* x_dev, int64_t dim,
                              float* out_dev) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    std::string why;
    if (!check_circuit(c, ctx->n, &why)) return fail(ctx, QSV_ERR_INVALID_ARG, why);
    const int n = ctx->n;
    const int64_t B = ctx->batch;
    const int64_t P = qsv_num_params(c, n);
    if (P > 0 && !params_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "params_dev is NULL");
    if (c->reupload && !feats_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "reupload = 1 needs feats_dev");
    if (!x_dev || !out_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "x_dev or out_dev is NULL");
    if (dim < 1 || dim > ((int64_t)1 << n)) return fail(ctx, QSV_ERR_INVALID_ARG, "dim must be in 1..2^n");
    if (mask == 0 || (mask >> n) != 0) return fail(ctx, QSV_ERR_INVALID_ARG, "mask must be a non-empty subset of the qubits");
    const int m = __builtin_popcountll(mask);
    if (m > 10) return fail(ctx, QSV_ERR_UNSUPPORTED, "reset of more than 10 qubits");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    const int64_t per = (int64_t)1 << m;
    const int64_t rows_all = B * per;
    Arena ar(ctx);
    const size_t state_bytes = (size_t)8 << n;
    float* mats = (float*)ar.take(mats_bytes(*c, n, B));
    double* Frow = (double*)ar.take((size_t)rows_all * 8);
    if (!mats || !Frow) return ws_fail(ctx, ar, "qsv_reset_fidelity");
    int nblk = (int)((dim + 4095) / 4096);
    if (nblk > 1024) nblk = 1024;
    const size_t row_bytes = state_bytes + (size_t)nblk * 3 * 8 + 2 * kAlign;
    int64_t chunk = (int64_t)(ar.remaining() / row_bytes);
    if (chunk < 1) { ar.need = ar.off + row_bytes; return ws_fail(ctx, ar, "qsv_reset_fidelity"); }
    if (chunk > rows_all) chunk = rows_all;
    if (chunk > 32768) chunk = 32768;
    if (ctx->opt_grad_chunk > 0 && chunk > ctx->opt_grad_chunk) chunk = ctx->opt_grad_chunk;
    if (chunk < rows_all) { int64_t p2 = 1; while (p2 * 2 <= chunk) p2 *= 2; chunk = p2; }
    float2* work = (float2*)ar.take((size_t)chunk * state_bytes);
    double* partial = (double*)ar.take((size_t)chunk * nblk * 3 * 8);
    if (!work || !partial) return ws_fail(ctx, ar, "qsv_reset_fidelity");
    Prepared pr;
    st = prepare_circuit(ctx, *c, chunk, 1, 0, params_dev, feats_dev, B, mats, &pr);
    if (st != QSV_OK) return st;
    for (int64_t row0 = 0; row0 < rows_all; row0 += chunk) {
        const int64_t rows = (rows_all - row0) < chunk ? (rows_all - row0) : chunk;
        RowMap rm;
        rm.grad = 1; rm.two_p = 0; rm.per = (int)per; rm.row0 = row0;
        rm.slots_n = 1; rm.n = n;
        QSV_HIP(ctx, launch_reset_rows(ctx->state, n, mask, rows, rm, work, ctx->stream), "reset rows");
        st = run_circuit(ctx, *c, pr, work, rows, 1, nullptr, rm);
        if (st != QSV_OK) return st;
        QSV_HIP(ctx, launch_fidelity_block(work, rows, n, x_dev, dim, partial, nblk, rm, ctx->stream),
                "fidelity block");
        QSV_HIP(ctx, launch_fidelity_finish(partial, nblk, rows, nullptr, Frow + row0, ctx->stream),
                "fidelity finish");
    }
    QSV_HIP(ctx, launch_reset_sum(Frow, per, B, out_dev, ctx->stream), "reset sum");
    return QSV_OK;
}

qsv_status qsv_shot_expz(qsv_ctx* ctx, const long long* samples_dev, int64_t shots, float* out_dev) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    if (!samples_dev || !out_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "samples_dev or out_dev is NULL");
    if (shots < 0) return fail(ctx, QSV_ERR_INVALID_ARG, "shots must be >= 0");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    QSV_HIP(ctx, launch_shot_expz(samples_dev, shots, ctx->batch, ctx->n, out_dev, ctx->stream), "shot expz");
    return QSV_OK;
}

qsv_status qsv_param_shift_grad(qsv_ctx* ctx, const qsv_circuit* c, const float* x_dev, int64_t dim,
                                const float* params_dev, const float* feats_dev, int32_t obs_qubit,
                                float* loss_dev, float* grad_dev, float* mean_loss_dev,
                                float* mean_grad_dev) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    std::string why;
    if (!check_circuit(c, ctx->n, &why)) return fail(ctx, QSV_ERR_INVALID_ARG, why);
    const int n = ctx->n;
    const int64_t B = ctx->batch;
    if (!x_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "x_dev is NULL");
    if (dim < 1 || dim > ((int64_t)1 << n)) return fail(ctx, QSV_ERR_INVALID_ARG, "dim must be in 1..2^n");
    if (obs_qubit < 0 || obs_qubit >= n) return fail(ctx, QSV_ERR_INVALID_ARG, "obs_qubit out of range");
    const int64_t P = qsv_num_params(c, n);
    if (P > 0 && !params_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "params_dev is NULL");
    if (c->reupload && !feats_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "reupload = 1 needs feats_dev");
    if (!loss_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "loss_dev is NULL");
    if (P > 0 && !grad_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "grad_dev is NULL");
    if (2 * P + 1 > 0x3fffffff) return fail(ctx, QSV_ERR_UNSUPPORTED, "too many parameters");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;

    Arena ar(ctx);
    const CircDev cd = to_dev(*c, n);
    const int64_t per = 2 * P + 1;
    const int64_t circuits = B * per;
    const size_t msamples = (size_t)(c->reupload ? B : 1);
    const size_t state_bytes = (size_t)8 << n;
    int nblk = (int)((dim + 4095) / 4096);
    if (nblk > 1024) nblk = 1024;
    double* npart = (double*)ar.take((size_t)B * nblk * 8);
    double* inv = (double*)ar.take((size_t)B * 8);
    float* mats = (float*)ar.take(mats_bytes(*c, n, B));
    float* ovr = (float*)ar.take(msamples * (size_t)(2 * P) * 32);
    double* f = (double*)ar.take((size_t)circuits * 8);
    if (!npart || !inv || !mats || !ovr || !f) return ws_fail(ctx, ar, "qsv_param_shift_grad");

    // rows of a chunk, at most `want`: their circuit states and the reduction partials of as many rows, or of `least` if those are
    // more, sized to what is left of the workspace
    const size_t zbytes = (size_t)chunk_blocks(n) * 13 * 8, row_bytes = state_bytes + zbytes + 2 * kAlign;
    auto chunk_rows = [&](const Arena& left, int64_t want, int64_t least) -> int64_t {
        const size_t room = left.remaining(), least_bytes = align_up((size_t)least * zbytes);
        int64_t chunk = (int64_t)(room / row_bytes);
        if (chunk < least) chunk = room > least_bytes ? (int64_t)((room - least_bytes) / kAlign * kAlign / state_bytes) : 0;
        if (chunk > want) chunk = want;
        if (chunk > 32768) chunk = 32768;  // rows index a grid dimension
        if (ctx->opt_grad_chunk > 0 && chunk > ctx->opt_grad_chunk) chunk = ctx->opt_grad_chunk;
        // keep the row count a power of two when several rows share a tile (extended-index tiling)
        if (chunk >= 1 && chunk < want) { int64_t p2 = 1; while (p2 * 2 <= chunk) p2 *= 2; chunk = p2; }
        return chunk;
    };

    // ---- layer by layer: the circuits that shift a parameter of layer l share layers 0..l-1 with
    // the unshifted circuit, so its state before layer l is kept per sample and each shifted
    // circuit runs layers l..L-1 only.  Needs room for (L+1) states per sample; otherwise every
    // shifted circuit is run whole (below).  Where the direct kernel takes the rows, one circuit per parameter is run instead of
    // two, with the angle turned by pi: R(t +- pi/2) = (R(t) +- R(t + pi)) / sqrt 2, so both shifted states are
    // combinations of its state and the unshifted circuit's, and the last pass forms them and takes both expectation values.
    // See turn_amplitudes for what it gives and where it pays.
    const int L = c->n_layers;
    const int slots_n = (c->reupload + c->n_rot) * n;
    struct Layered { float2 *ckpt, *states; double *residues, *zpart; int64_t chunk; } lay{};
    // what is taken of the workspace for per_l rows per sample and layer; false: it has no room for that
    auto carve = [&](int64_t per_l, size_t residue_count) -> bool {
        Arena a = ar;
        lay.ckpt = (float2*)a.take((size_t)B * (size_t)(L + 1) * state_bytes);
        lay.residues = residue_count ? (double*)a.take(residue_count * 16) : nullptr;
        if (!lay.ckpt || (residue_count && !lay.residues)) return false;
        lay.chunk = chunk_rows(a, std::max(B * per_l, B), B);
        if (lay.chunk < 1) return false;
        lay.states = (float2*)a.take((size_t)lay.chunk * state_bytes);
        lay.zpart = (double*)a.take((size_t)std::max(lay.chunk, B) * zbytes);
        return lay.states && lay.zpart;
    };
    if (ctx->opt_grad_layered && P > 0 && carve(2 * (int64_t)slots_n, 0)) {
        qsv_circuit one = *c;
        one.n_layers = 1;
        qsv_circuit rot = one;
        rot.entangler = QSV_ENT_NONE;
        // the tile of gradient rows does not depend on their number from 10 qubits on
        bool turns = !ctx->opt_naive && n >= kMinTile && is_direct(ctx, tile_of(ctx, B, 1, 0)) &&
                     ((uint64_t)(B * slots_n) << n) >= turn_amplitudes(n, L);
        // A unitary with a turned angle is a turn times the unturned one, so the circuits of layer l also share that layer's
        // rotations: the states go through them once per sample, and a circuit starts with one matrix on one qubit instead of n
        // unitaries.  See kAheadAmplitudes for where that pays.
        bool ahead = turns && ((uint64_t)(B * slots_n) << n) >= kAheadAmplitudes;
        // The groups of a layer, of its rotations and of every tail: their scalars are entries of the tables, beside which the
        // region for matrices has room for L n / 2 others (tables with groups have no scale table), and what these lack is kept per group.
        // Options that leave a tile few qubits to choose (tile_log2, low_bits) make more passes, and with them groups, than
        // that: two circuits per parameter then, as where a tail's plan is too long for the ops region.
        int g_one = 0, g_rot = 0, g_tail = 0;
        std::vector<CachedPlan*> tails;
        if (turns) {
            auto groups_of = [&](const qsv_circuit& k, int grad, PlanForm form, CachedPlan** cp, int* groups) -> qsv_status {
                const qsv_status s = find_plan(ctx, k, B, 0, grad, cp, 0, form);
                if (s == QSV_OK) *groups = (int)(*cp)->plan.groups.size() - 1;
                return s;
            };
            const size_t entries = mats_bytes(*c, n, B) / 32 - 1;      // one is only prefetched
            auto fits = [&](int64_t per_sample) { return msamples * (size_t)per_sample <= entries; };
            CachedPlan* cp = nullptr;
            st = groups_of(one, 0, kGrouped, &cp, &g_one);
            if (st == QSV_OK && ahead) st = groups_of(rot, 0, kGrouped, &cp, &g_rot);
            turns = fits((int64_t)L * (n + std::max(g_one, g_rot)));
            for (int l = 0; l < L && turns && st == QSV_OK; ++l) {
                qsv_circuit tail = *c;
                tail.n_layers = L - l;
                int g = 0;
                st = groups_of(tail, 1, ahead ? kTurnedAhead : kTurned, &cp, &g);
                if (st != QSV_OK) break;
                turns = fits((int64_t)(L - l) * n + g) && PlanRoom(*cp).bytes() <= kOpsRegion;
                g_tail = std::max(g_tail, g);
                tails.push_back(cp);
            }
            if (st != QSV_OK) return st;
            ahead = ahead && turns;
        }
        const size_t res_one_count = msamples * (size_t)L * g_one, res_rot_count = msamples * (size_t)L * g_rot;
        // (rows half as many make another chunk)
        if (turns && !carve(slots_n, res_one_count + res_rot_count + msamples * (size_t)g_tail)) {
            turns = ahead = false;
            carve(2 * (int64_t)slots_n, 0);
        }
        double *res_one = lay.residues, *res_rot = turns ? res_one + 2 * res_one_count : nullptr,
               *res_tail = turns ? res_rot + 2 * res_rot_count : nullptr;
        const int64_t per_l = (turns ? 1 : 2) * (int64_t)slots_n, chunk = lay.chunk;
        float2 *const ckpt = lay.ckpt, *const states = lay.states;
        double* const zpart = lay.zpart;
        const size_t sample_stride = (size_t)1 << n;          // amplitudes per state
        auto ck = [&](int l) { return ckpt + (size_t)l * (size_t)B * sample_stride; };
        // unshifted circuit, one layer at a time: ck(l) = state of every sample before layer l
        QSV_HIP(ctx, launch_encode(x_dev, B, dim, n, npart, nblk, inv, nullptr, ck(0), ctx->stream), "encode");
        RowMap rm_fwd;    // rows are the samples: the first pass of layer l reads state l and writes state l + 1
        rm_fwd.grad = 1; rm_fwd.two_p = 0; rm_fwd.per = 1; rm_fwd.row0 = 0;
        rm_fwd.slots_n = slots_n < 1 ? 1 : slots_n; rm_fwd.n = n;
        Prepared all;
        // (with turned rows the states are combined with theirs: unitaries rounded alike)
        const PlanForm unshifted = turns ? kGrouped : kPlain;
        st = prepare_layers(ctx, *c, one, B, 0, params_dev, feats_dev, B, mats, &all, unshifted, res_one);
        if (st != QSV_OK) return st;
        for (int l = 0; l < L; ++l) {
            st = run_circuit(ctx, one, layer_of(all, l), ck(l + 1), B, 0, nullptr, rm_fwd, ck(l));
            if (st != QSV_OK) return st;
        }
        QSV_HIP(ctx, launch_expz_block(ck(L), B, n, zpart, ctx->stream), "expz block");
        const Residues through{res_one, 0, L * g_one, L * g_one};
        QSV_HIP(ctx, launch_expz_finish_scatter(zpart, B, n, obs_qubit, f, Scatter{0, 1, per, 2 * P}, ctx->stream,
                                                turns ? &through : nullptr, c->reupload),
                "expz finish");
        if (ahead) {
            st = prepare_layers(ctx, *c, rot, B, 0, params_dev, feats_dev, B, mats, &all, unshifted, res_rot);
            for (int l = 0; l < L && st == QSV_OK; ++l)
                st = run_circuit(ctx, rot, layer_of(all, l), ck(l), B, 0, nullptr, rm_fwd);
            if (st != QSV_OK) return st;
        }
        // shifted circuits of layer l: start from ck(l), run layers l..L-1 with one matrix replaced
        const CircDev cd1 = to_dev(one, n);
        for (int l = 0; l < L; ++l) {
            qsv_circuit tail = *c;
            tail.n_layers = L - l;
            const float* p_l = params_dev + (size_t)l * slots_n;
            Prepared pr;
            int groups = 0;
            if (turns) {
                st = upload_plan(ctx, *tails[l]);
                if (st != QSV_OK) return st;
                pr.cp = tails[l];
                CircDev rest = to_dev(tail, n);
                if (ahead) rest.n_layers -= 1;
                groups = (int)pr.cp->plan.groups.size() - 1;
                pr.mats = mats;
                pr.mat_stride = rest.n_layers * n + groups;
                pr.form = MatForm::direct;
                if (groups > 0)
                    QSV_HIP(ctx, launch_build_mats(rest, ahead ? p_l + slots_n : p_l, feats_dev, B, 0,
                                                   reinterpret_cast<const int*>(ctx->ws + pr.cp->order_off), 0,
                                                   reinterpret_cast<const int*>(ctx->ws + pr.cp->groups_off), groups,
                                                   MatForm::direct, mats, res_tail, ctx->stream),
                            "build matrices");
                QSV_HIP(ctx, launch_build_turns(cd1, p_l, feats_dev, B, ahead ? 1 : 0, ovr, ctx->stream), "build turns");
            } else {
                st = prepare_circuit(ctx, tail, chunk, 0, 1, p_l, feats_dev, B, mats, &pr);
                if (st != QSV_OK) return st;
                QSV_HIP(ctx, launch_build_shifted(cd1, p_l, feats_dev, B, pr.exec_of, pr.scale, tail.n_layers * n, ovr, ctx->stream), "build shifted");
            }
            const int64_t circuits_l = B * per_l;
            for (int64_t row0 = 0; row0 < circuits_l; row0 += chunk) {
                const int64_t rows = (circuits_l - row0) < chunk ? (circuits_l - row0) : chunk;
                RowMap rm;
                rm.grad = 1;
                rm.two_p = (int)per_l;
                rm.per = (int)per_l;
                rm.row0 = row0;
                rm.slots_n = slots_n;
                rm.n = n;
                const ZSpec zs{obs_qubit, f, Scatter{row0, per_l, per, 2 * (int64_t)l * slots_n}, zpart, turns ? ck(L) : nullptr, 2 * P,
                               Residues{res_one, l * g_one, (L - l) * g_one, L * g_one}, Residues{res_tail, 0, groups, groups},
                               ahead ? Residues{res_rot, l * g_rot, g_rot, L * g_rot} : Residues{res_rot, 0, 0, 0}};
                st = run_circuit(ctx, tail, pr, states, rows, 0, ovr, rm, ck(l), &zs);
                if (st != QSV_OK) return st;
            }
        }
        QSV_HIP(ctx, launch_grad_finish(f, B, P, cd, feats_dev, loss_dev, grad_dev, mean_loss_dev,
                                        mean_grad_dev, ctx->stream),
                "grad finish");
        return QSV_OK;
    }

    // ---- every shifted circuit whole
    QSV_HIP(ctx, launch_norms(x_dev, B, dim, npart, nblk, inv, nullptr, ctx->stream), "norms");
    const int64_t chunk = chunk_rows(ar, circuits, 0);
    if (chunk < 1) { ar.need = ar.off + row_bytes; return ws_fail(ctx, ar, "qsv_param_shift_grad"); }
    float2* states = (float2*)ar.take((size_t)chunk * state_bytes);
    double* zpart = (double*)ar.take((size_t)chunk * chunk_blocks(n) * 13 * 8);
    if (!states || !zpart) return ws_fail(ctx, ar, "qsv_param_shift_grad");
    Prepared pr;
    st = prepare_circuit(ctx, *c, chunk, 0, 1, params_dev, feats_dev, B, mats, &pr);
    if (st != QSV_OK) return st;
    if (P > 0)
        QSV_HIP(ctx, launch_build_shifted(cd, params_dev, feats_dev, B, pr.exec_of, pr.scale, L * n, ovr, ctx->stream), "build shifted");
    for (int64_t row0 = 0; row0 < circuits; row0 += chunk) {
        const int64_t rows = (circuits - row0) < chunk ? (circuits - row0) : chunk;
        RowMap rm;
        rm.grad = 1;
        rm.two_p = (int)(2 * P);
        rm.per = (int)per;
        rm.row0 = row0;
        rm.slots_n = slots_n < 1 ? 1 : slots_n;
        rm.n = n;
        QSV_HIP(ctx, launch_encode_write(x_dev, dim, n, rows, inv, rm, states, ctx->stream), "encode rows");
        const ZSpec zs{obs_qubit, f, Scatter{row0, 1, 1, 0}, zpart, nullptr, 0, {}, {}, {}};
        st = run_circuit(ctx, *c, pr, states, rows, 0, ovr, rm, nullptr, &zs);
        if (st != QSV_OK) return st;
    }
    QSV_HIP(ctx, launch_grad_finish(f, B, P, cd, feats_dev, loss_dev, grad_dev, mean_loss_dev,
                                    mean_grad_dev, ctx->stream),
            "grad finish");
    return QSV_OK;
}

// The chunks of a reverse-mode sweep alternate between the caller's stream and the context's second one; this forks the
// second one off, and always joins it again.
struct Fork {
    qsv_ctx* c;
    hipStream_t main;
    bool on;
    explicit Fork(qsv_ctx* ctx) : c(ctx), main(ctx->stream), on(false) {}
    qsv_status begin() {
        QSV_HIP(c, hipEventRecord(c->ev_fork, main), "fork");
        QSV_HIP(c, hipStreamWaitEvent(c->side, c->ev_fork, 0), "fork");
        on = true;
        c->forked = true;
        return QSV_OK;
    }
    // chunk i runs on stream i % 2 with scratch set i % 2 (stream order guards the reuse of a set)
    int take(int64_t i) {
        const int set = on ? (int)(i & 1) : 0;
        c->stream = set ? c->side : main;
        return set;
    }
    qsv_status join() {        // what follows sees both streams' work
        c->stream = main;
        if (!on) return QSV_OK;
        on = false;
        c->forked = false;
        QSV_HIP(c, hipEventRecord(c->ev_join, c->side), "join");
        QSV_HIP(c, hipStreamWaitEvent(main, c->ev_join, 0), "join");
        return QSV_OK;
    }
    ~Fork() {
        c->stream = main;
        if (!on) return;
        c->forked = false;
        if (hipEventRecord(c->ev_join, c->side) == hipSuccess) (void)hipStreamWaitEvent(main, c->ev_join, 0);
    }
};

// What reverse mode differentiates: kind 0 <Z_q>; 1 the loss 1 - P0(mask); 2 the mean squared error of <Z_q> against targets.
struct Objective { int kind, q; uint64_t mask; const float* targets; };

// The losses of rows 0 .. rows - 1 of A (samples sample0 + row) into f[sample][2P]; kind 2 also the coefficients of lambda.
// res, rowdep: see launch_expz_finish; of row 0's sample on.
static qsv_status losses(qsv_ctx* ctx, const Objective& ob, const float2* A, int64_t rows, int64_t sample0, int64_t P,
                         double* zpart, double* zall, double* coef, double* f, const Residues* res = nullptr,
                         int rowdep = 0) {
    const int n = ctx->n;
    if (ob.kind == 1) {
        QSV_HIP(ctx, launch_trash_loss(A, n, ob.mask, rows, sample0, P, zpart, f, ctx->stream, res, rowdep), "trash loss");
        return QSV_OK;
    }
    QSV_HIP(ctx, launch_expz_block(A, rows, n, zpart, ctx->stream), "expz block");
    if (ob.kind == 0) {
        QSV_HIP(ctx, launch_expz_finish_scatter(zpart, rows, n, ob.q, f, Scatter{sample0, 1, 2 * P + 1, 2 * P}, ctx->stream,
                                                res, rowdep),
                "expz finish");
        return QSV_OK;
    }
    QSV_HIP(ctx, launch_expz_finish(zpart, rows, n, -1, nullptr, zall, ctx->stream, res, rowdep), "expz finish");
    QSV_HIP(ctx, launch_mse_coef(zall, ob.targets, n, rows, sample0, P, coef, f, ctx->stream), "mse loss");
    return QSV_OK;
}

// Reverse mode in the passes of the whole circuit's plan.  The forward run keeps the state after every pass; the mirrored
// passes take lambda = O psi back, and with it, tile by tile, the kept psi of their end, and read the transition sums of
// every unitary off the registers where it is undone.  So a sweep moves five states a pass (two there; psi and lambda in,
// lambda out on the way back) of a plan with deferral, where the layers one by one move twelve each: 20 qubits x 32, 20
// layers 18 passes, 24 GB instead of 64; a 16-qubit ladder of 10 layers 3 passes, 2 GB instead of 16.
// *done = false: nothing was launched: the scratch has no room, the plans are too long for the ops region, or the options ask
// for another way.
// f: [batch][2P+1]; inv: room for the norms; what is taken of ar is taken for good.
static qsv_status fused_sweep(qsv_ctx* ctx, const qsv_circuit& c, const Objective& ob, const float* x_dev, int64_t dim,
                              const float* params, const float* feats, double* npart, int nblk, double* inv, double* f,
                              Arena& ar, bool* done) {
    *done = false;
    const int n = ctx->n, L = c.n_layers;
    const int64_t B = ctx->batch, P = qsv_num_params(&c, n), per = (int64_t)L * n;
    if (!ctx->opt_grad_layered || P < 1 || ctx->opt_naive || n < kMinTile || n > kDirectMaxQubits || ctx->opt_planes != 1)
        return QSV_OK;
    const int64_t most = ctx->opt_grad_chunk > 0 ? ctx->opt_grad_chunk : B;
    int defer = ctx->opt_defer != 0 && c.entangler == QSV_ENT_CNOT_RING;
    if (defer && n <= tile_of(ctx, B, L, 1)) defer = 0;
    const int tile = tile_of(ctx, B, L, defer);
    if (tile > kPairMaxTile || n < tile) return QSV_OK;
    const size_t state_bytes = (size_t)8 << n;
    const size_t sums_bytes = pair_sums_bytes(n, per), zbytes = (size_t)chunk_blocks(n) * 13 * 8;
    auto sample_bytes = [&](size_t passes) {
        return (passes + 1) * state_bytes + sums_bytes + zbytes + 2 * (size_t)n * 8;
    };
    // a table: the unitaries and at most as many groups' scalars, and one entry that is only prefetched
    const size_t table_bytes = 2 * mats_table_bytes(c, n, B), corr_bytes = mat_scale_bytes(to_dev(c, n), B);
    // (a group's residue for every unitary at most)
    const size_t fixed = 2 * table_bytes + 2 * corr_bytes + 16 * kAlign;
    // Two halves on two streams pay as in run_circuit: 20 qubits x 32, 20 layers 8.66 -> 8.24 ms, 16 x 256 1.25 -> 1.17, 22 x 2,
    // 6 layers 0.98 -> 0.88; 18 x 4 296 -> 312 us, 16 x 16 357 -> 374, 13 x 37 163 -> 210, 11 x 64 135 -> 168.
    const bool two = B >= 2 && !ctx->forked &&
                     (ctx->opt_split >= 0 ? ctx->opt_split == 1 : (uint64_t)B * state_bytes >= kSplitBytes);
    const int sets = two ? 2 : 1;
    const int64_t half = std::min(most, two ? (B + 1) / 2 : B);
    // without planning for it: a deep circuit's plan takes longer than the call (20 qubits, 1024 layers of a ring 2.9 s)
    if (ar.remaining() < fixed + (size_t)sets * half * sample_bytes((size_t)fewest_passes(c, n, tile))) return QSV_OK;
    CachedPlan *fp = nullptr, *bp = nullptr;
    qsv_status st = find_plan(ctx, c, B, 0, 0, &fp, defer, kSweep);
    if (st == QSV_OK) st = find_plan(ctx, c, B, 1, 0, &bp, defer, kSweep);
    if (st != QSV_OK) return st;
    // (the other way needs no more than one layer's plans in the ops region)
    const size_t passes = fp->plan.passes.size();
    if (PlanRoom(*fp).bytes() + PlanRoom(*bp).bytes() > kOpsRegion || passes == 0 ||
        ar.remaining() < fixed + (size_t)sets * half * sample_bytes(passes))
        return QSV_OK;
    st = upload_plan(ctx, *fp);
    if (st == QSV_OK) st = upload_plan(ctx, *bp);
    if (st == QSV_OK) st = upload_plan(ctx, *fp);      // should the second one have recycled the region
    if (st != QSV_OK) return st;
    int64_t chunk = std::min<int64_t>(half, 32768);
    // the records of a unitary are at most 4 GiB
    while (chunk > 1 && ((uint64_t)chunk << (n - 10)) * 16 > 0xffffffffull) chunk = (chunk + 1) / 2;

    float* fmats = (float*)ar.take(table_bytes);
    float* bmats = (float*)ar.take(table_bytes);
    double* corr = (double*)ar.take(corr_bytes);
    double* residues = (double*)ar.take(corr_bytes);
    struct Scratch { float2* psi; float* sums; double *zpart, *zall, *coef; } scr[2];
    for (int i = 0; i < sets; ++i) {
        scr[i].psi = (float2*)ar.take((passes + 1) * (size_t)chunk * state_bytes);
        scr[i].sums = (float*)ar.take((size_t)chunk * sums_bytes);
        scr[i].zpart = (double*)ar.take((size_t)chunk * zbytes);
        scr[i].zall = (double*)ar.take((size_t)chunk * n * 8);
        scr[i].coef = (double*)ar.take((size_t)chunk * n * 8);
        if (!scr[i].coef) return ws_fail(ctx, ar, "qsv_adjoint_grad");
    }
    *done = true;
    const CircDev cd = to_dev(c, n);
    auto table = [&](const CachedPlan* cp, int inverse, MatForm form, float* out, double* scale) -> qsv_status {
        QSV_HIP(ctx, launch_build_mats(cd, params, feats, B, inverse, reinterpret_cast<const int*>(ctx->ws + cp->order_off), 0,
                                       reinterpret_cast<const int*>(ctx->ws + cp->groups_off), (int)cp->plan.groups.size() - 1,
                                       form, out, scale, ctx->stream),
                "build matrices");
        return QSV_OK;
    };
    st = table(fp, 0, MatForm::direct, fmats, residues);
    if (st == QSV_OK) st = table(bp, 1, MatForm::paired, bmats, corr);
    if (st != QSV_OK) return st;

    const size_t amps = (size_t)1 << n;
    const int groups = (int)fp->plan.groups.size() - 1;      // the mirror image has as many
    auto run_chunk = [&](int64_t b0, int64_t rows, const Scratch& sc) -> qsv_status {
        auto state = [&](size_t k) { return sc.psi + k * (size_t)chunk * amps; };   // 0: encoded; k: after pass k - 1
        RowMap rm;
        rm.grad = 1; rm.two_p = 0; rm.per = 1; rm.row0 = b0; rm.slots_n = 1; rm.n = n;
        QSV_HIP(ctx, launch_encode(x_dev + (size_t)b0 * dim, rows, dim, n, npart + (size_t)b0 * nblk, nblk, inv + b0, nullptr,
                                   state(0), ctx->stream),
                "encode rows");
        const uint64_t touched = ((uint64_t)rows << n) * 16;
        const int nt = ctx->opt_nt_store >= 0 ? ctx->opt_nt_store : (touched >= kNtStoreBytes ? 1 : 0);
        for (size_t k = 0; k < passes; ++k) {
            const Pass& ps = fp->plan.passes[k];
            const DirectPass& low = fp->low_ops.passes[k];
            PassArgs a{};
            a.state = state(k + 1);
            a.in = state(k);
            a.imap = ps.map_begin >= 0 ? reinterpret_cast<const unsigned*>(ctx->ws + fp->maps_off) + ps.map_begin : nullptr;
            a.ops = reinterpret_cast<const Op*>(ctx->ws + fp->dev_off) + low.begin;
            a.mats = fmats;
            a.total = (uint64_t)rows << n;
            a.nt_store = nt;
            a.rev = ctx->opt_rev != 0 && (k & 1) ? (ps.map_begin < 0 ? 2 : 1) : 0;
            a.prio = 0;      // raised / not: 20 qubits x 32, 20 layers 8.24 / 7.88 ms, 22 x 2 877 / 839 us, below 18 no difference
            a.n = n; a.c = ps.c; a.w = ps.w;
            a.n_mats = (int)per + groups;
            a.rowdep = c.reupload;
            a.rm = rm;
            a.direct = 1;
            a.s_in = low.s_in; a.s_out = low.s_out; a.first_mat = low.first_mat;
            a.g_sample0 = (unsigned)b0;
            warm(&a, low, (uint64_t)rows << (n - tile));
            QSV_HIP(ctx, launch_pass(tile, 1, a, (uint64_t)rows << (n - tile), ctx->stream), "fused pass");
        }
        const Residues through{residues + (c.reupload ? (size_t)b0 * groups * 2 : 0), 0, groups, groups};
        qsv_status s = losses(ctx, ob, state(passes), rows, b0, P, sc.zpart, sc.zall, sc.coef, f, &through, c.reupload);
        if (s != QSV_OK) return s;
        // backwards: lambda changes between the encoded states' buffer and the last states', whose pass comes first
        const float2* lam = nullptr;
        for (size_t k = 0; k < passes; ++k) {
            const Pass& ps = bp->plan.passes[k];
            const DirectPass& low = bp->low_ops.passes[k];
            PairArgs a{};
            a.psi = state(passes - k);
            a.lam_in = lam;
            a.lam_out = k + 1 == passes ? nullptr : k & 1 ? state(passes) : state(0);
            lam = a.lam_out;
            a.imap = ps.map_begin >= 0 ? reinterpret_cast<const unsigned*>(ctx->ws + bp->maps_off) + ps.map_begin : nullptr;
            a.ops = reinterpret_cast<const Op*>(ctx->ws + bp->dev_off) + low.begin;
            a.mats = bmats;
            a.sums = sc.sums;
            a.sample0 = b0;
            a.rows = rows;
            a.n = n; a.c = ps.c; a.w = ps.w;
            a.n_mats = (int)per + groups;
            a.rowdep = c.reupload;
            a.s_in = low.s_in; a.s_out = low.s_out; a.first_mat = low.first_mat; a.first_u = low.first_u;
            a.mate = ps.map_begin >= 0 ? bp->mates[k] : 0;
            warm(&a, low, (uint64_t)rows << (n - tile));
            // the forward run's last pass was number passes - 1: go on in turns
            a.rev = ctx->opt_rev != 0 && ((passes + k) & 1) ? (ps.map_begin < 0 ? 2 : 1) : 0;
            a.nt_store = nt;
            a.kind = ob.kind; a.q = ob.q; a.mask = ob.mask; a.coef = sc.coef;
            QSV_HIP(ctx, launch_pair_pass(tile, a, ctx->stream), "reverse pass");
        }
        QSV_HIP(ctx, launch_pair_finish(sc.sums, rows, cd, params, b0, P, reinterpret_cast<const int*>(ctx->ws + bp->order_off),
                                        reinterpret_cast<const int*>(ctx->ws + bp->execof_off), bmats, (int)per + groups,
                                        corr, f, ctx->stream),
                "adjoint layers");
        return QSV_OK;
    };
    Fork fork(ctx);
    if (two && chunk < B && (st = fork.begin()) != QSV_OK) return st;
    int64_t ci = 0;
    for (int64_t b0 = 0; b0 < B; b0 += chunk, ++ci) {
        st = run_chunk(b0, std::min(chunk, B - b0), scr[fork.take(ci)]);
        if (st != QSV_OK) return st;
    }
    return fork.join();
}

// Reverse-mode loss and gradient for a diagonal observable (see Objective).
static qsv_status adjoint_impl(qsv_ctx* ctx, const qsv_circuit* c, const float* x_dev, int64_t dim,
                               const float* params_dev, const float* feats_dev, int kind, int32_t obs_qubit,
                               uint64_t mask, const float* targets_dev, float* loss_dev, float* grad_dev,
                               float* mean_loss_dev, float* mean_grad_dev) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    std::string why;
    if (!check_circuit(c, ctx->n, &why)) return fail(ctx, QSV_ERR_INVALID_ARG, why);
    const int n = ctx->n;
    const int64_t B = ctx->batch;
    if (!x_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "x_dev is NULL");
    if (dim < 1 || dim > ((int64_t)1 << n)) return fail(ctx, QSV_ERR_INVALID_ARG, "dim must be in 1..2^n");
    if (kind == 0 && (obs_qubit < 0 || obs_qubit >= n)) return fail(ctx, QSV_ERR_INVALID_ARG, "obs_qubit out of range");
    if (kind == 1 && (mask == 0 || (mask >> n) != 0))
        return fail(ctx, QSV_ERR_INVALID_ARG, "mask must name at least one qubit and none beyond n_qubits");
    if (kind == 2 && !targets_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "targets_dev is NULL");
    const int64_t P = qsv_num_params(c, n);
    if (P > 0 && !params_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "params_dev is NULL");
    if (c->reupload && !feats_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "reupload = 1 needs feats_dev");
    if (!loss_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "loss_dev is NULL");
    if (P > 0 && !grad_dev) return fail(ctx, QSV_ERR_INVALID_ARG, "grad_dev is NULL");
    if (2 * P + 1 > 0x3fffffff) return fail(ctx, QSV_ERR_UNSUPPORTED, "too many parameters");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;

    Arena ar(ctx);
    const CircDev cd = to_dev(*c, n);
    const int64_t per = 2 * P + 1;
    const size_t state_bytes = (size_t)8 << n;
    int nblk = (int)((dim + 4095) / 4096);
    if (nblk > 1024) nblk = 1024;
    double* npart = (double*)ar.take((size_t)B * nblk * 8);
    double* inv = (double*)ar.take((size_t)B * 8);
    double* f = (double*)ar.take((size_t)B * per * 8);
    if (!npart || !inv || !f) return ws_fail(ctx, ar, "qsv_adjoint_grad");

    // Two ways to have psi at the start of every layer on the way back.  With room for L + 1 states per
    // sample the forward run keeps them (layer l reads state l and writes state l + 1, no copies) and
    // only lambda is taken back: 2 L layers of gates per sample.  Otherwise psi is taken back together
    // with lambda (rows 2r, 2r+1 of one buffer): 3 L layers, 3 states per sample of a chunk.
    const int L = c->n_layers;
    const size_t tpart = (size_t)n * (adj_trans_blocks(n) + 1) * 8 * 8;
    const size_t zbytes = (size_t)chunk_blocks(n) * 13 * 8;
    const size_t small_bytes = tpart + zbytes + 2 * (size_t)n * 8 + 6 * kAlign;
    const size_t ckpt_bytes = (size_t)B * (size_t)(L + 1) * state_bytes;
    const size_t tables = mats_bytes(*c, n, B);
    const bool keep = ctx->opt_grad_layered && P > 0 &&
                      ar.remaining() >= align_up(ckpt_bytes) + state_bytes + small_bytes + 2 * tables + 2 * kAlign;
    const Objective ob{kind, obs_qubit, mask, targets_dev};
    auto fused = [&](bool* done) -> qsv_status {
        Arena fs = ar;       // what is taken here is given back if it does not fit
        qsv_status s = fused_sweep(ctx, *c, ob, x_dev, dim, params_dev, feats_dev, npart, nblk, inv, f, fs, done);
        if (s != QSV_OK || !*done) return s;
        QSV_HIP(ctx, launch_grad_finish(f, B, P, cd, feats_dev, loss_dev, grad_dev, mean_loss_dev, mean_grad_dev, ctx->stream),
                "grad finish");
        return QSV_OK;
    };
    bool done = false;
    // 10 qubits have both: one launch is faster up to 1024 samples (512, 4 layers 45 against 84 us), passes beyond (4096, 6
    // layers 306 / 230), but for re-uploading circuits, whose tables cost them as much (2048, 12 layers 326 / 318)
    if (n >= kMinTile && !c->reupload && (B << n) > small_apply_amplitudes(kSmallMaxQubits)) {
        st = fused(&done);
        if (st != QSV_OK || done) return st;
    }
    // Small states: the whole sweep in one launch, where the scratch has room for its sums.  It keeps psi too where there
    // is room: the gradient is then no further from 64 bits than layer by layer (psi taken back 1.2 to 1.6 times).
    if (ctx->opt_small_apply != 0 && n <= kSmallMaxQubits && P > 0 && ctx->opt_tile == 0 && !ctx->opt_naive &&
        ctx->opt_grad_layered && ctx->opt_grad_chunk == 0 && (int64_t)L * n <= kSmallMats) {
        Arena sm = ar;       // what is taken here is given back if it does not fit
        float* mats = (float*)sm.take(mats_table_bytes(*c, n, B));
        double* sums = (double*)sm.take((size_t)B * L * sweep_record_bytes(n));
        float2* kept = (float2*)sm.take((size_t)B * L * state_bytes);
        if (mats && sums && (kept || !keep)) {
            QSV_HIP(ctx, launch_build_mats(cd, params_dev, feats_dev, B, 1, nullptr, 0, nullptr, 0, MatForm::phaseless, mats, nullptr,
                                           ctx->stream),
                    "build matrices");
            QSV_HIP(ctx, launch_sweep_small(x_dev, dim, B, cd, c->entangler, params_dev, mats, kind, obs_qubit, mask,
                                            targets_dev, kept, sums, f, ctx->stream),
                    "small sweep");
            QSV_HIP(ctx, launch_grad_finish(f, B, P, cd, feats_dev, loss_dev, grad_dev, mean_loss_dev, mean_grad_dev,
                                            ctx->stream),
                    "grad finish");
            return QSV_OK;
        }
    }
    st = fused(&done);
    if (st != QSV_OK || done) return st;
    QSV_HIP(ctx, launch_norms(x_dev, B, dim, npart, nblk, inv, nullptr, ctx->stream), "norms");
    float2* ckpt = keep ? (float2*)ar.take(ckpt_bytes) : nullptr;
    if (keep && !ckpt) return ws_fail(ctx, ar, "qsv_adjoint_grad");
    // The samples go through the sweep in chunks; with two samples or more the chunks alternate
    // between the caller's stream and the context's second one, each with scratch of its own, so that
    // the launch gaps and tails of one chunk's kernels are covered by the other's.
    const size_t sample_bytes = (keep ? 1 : 3) * state_bytes + small_bytes;
    const bool two = B >= 2 && ctx->opt_split != 0 && !ctx->forked &&
                     ar.remaining() >= 2 * (sample_bytes + tables + kAlign);
    const int sets = two ? 2 : 1;
    const size_t fixed = (size_t)sets * (tables + kAlign);
    int64_t chunk = ar.remaining() > fixed ? (int64_t)((ar.remaining() - fixed) / (sets * sample_bytes)) : 0;
    if (chunk < 1) {
        ar.need = ar.off + fixed + sets * sample_bytes;
        return ws_fail(ctx, ar, "qsv_adjoint_grad");
    }
    if (two && chunk > (B + 1) / 2) chunk = (B + 1) / 2;
    if (chunk > B) chunk = B;
    if (chunk > 16384) chunk = 16384;   // rows of a chunk index a grid dimension
    if (ctx->opt_grad_chunk > 0 && chunk > ctx->opt_grad_chunk) chunk = ctx->opt_grad_chunk;
    // keep row counts a power of two when several rows share a tile (extended-index tiling)
    if (chunk < B) { int64_t p2 = 1; while (p2 * 2 <= chunk) p2 *= 2; chunk = p2; }
    struct Scratch { float* mats; float2 *Abuf, *S; double *tp, *zpart, *zall, *coef; } scr[2];
    for (int i = 0; i < sets; ++i) {
        Scratch& sc = scr[i];
        sc.mats = (float*)ar.take(tables);
        sc.Abuf = keep ? nullptr : (float2*)ar.take((size_t)chunk * state_bytes);
        sc.S = (float2*)ar.take((size_t)(keep ? 1 : 2) * chunk * state_bytes);
        sc.tp = (double*)ar.take((size_t)chunk * tpart);
        sc.zpart = (double*)ar.take((size_t)chunk * zbytes);
        sc.zall = (double*)ar.take((size_t)chunk * n * 8);
        sc.coef = (double*)ar.take((size_t)chunk * n * 8);
        if (!sc.mats || (!keep && !sc.Abuf) || !sc.S || !sc.tp || !sc.zpart || !sc.zall || !sc.coef)
            return ws_fail(ctx, ar, "qsv_adjoint_grad");
    }
    // With room for the transition sums of all layers, adding them up and the derivatives are two launches for a whole
    // chunk instead of two short ones (6 to 8 us each, nothing of the same chunk runs beside them) for every layer:
    // 16 qubits x 256, 10 layers 2948 -> 2865 us.  At 20 qubits x 32, 20 layers the two sets would take 210 MB, which a
    // workspace of qsv_grad_workspace_bytes does not have left; with so much more 11.87 -> 11.83 ms (bound by traffic).
    bool late = L > 1 && P > 0;
    {
        Arena all = ar;     // what is taken here is given back if it does not fit
        double* tp[2];
        for (int i = 0; i < sets && late; ++i)
            late = (tp[i] = (double*)all.take((size_t)L * chunk * tpart)) != nullptr;
        for (int i = 0; i < sets && late; ++i) scr[i].tp = tp[i];
    }

    const int slots_n = (c->reupload + c->n_rot) * n;
    const size_t amps = (size_t)1 << n;
    auto ck = [&](int l, int64_t b0) { return ckpt + ((size_t)l * (size_t)B + (size_t)b0) * amps; };
    qsv_circuit one = *c;
    one.n_layers = 1;
    // one chunk of samples b0 .. b0 + bc - 1 on ctx->stream, with the scratch set sc
    auto run_chunk = [&](int64_t b0, int64_t bc, const Scratch& sc) -> qsv_status {
        // forward: rows are samples b0..b0+bc-1
        RowMap rm1;
        rm1.grad = 1; rm1.two_p = 0; rm1.per = 1; rm1.row0 = b0; rm1.slots_n = slots_n < 1 ? 1 : slots_n; rm1.n = n;
        float2* A = keep ? ck(L, b0) : sc.Abuf;                 // the final states of the chunk
        if (keep) {
            QSV_HIP(ctx, launch_encode_write(x_dev, dim, n, bc, inv, rm1, ck(0, b0), ctx->stream), "encode rows");
            Prepared all;
            st = prepare_layers(ctx, *c, one, bc, 0, params_dev, feats_dev, B, sc.mats, &all);
            if (st != QSV_OK) return st;
            for (int l = 0; l < L; ++l) {
                // the start states are addressed by sample (ck(l, 0)), the rows written are the chunk's
                st = run_circuit(ctx, one, layer_of(all, l), ck(l + 1, b0), bc, 0, nullptr, rm1, ck(l, 0));
                if (st != QSV_OK) return st;
            }
        } else {
            QSV_HIP(ctx, launch_encode_write(x_dev, dim, n, bc, inv, rm1, A, ctx->stream), "encode rows");
            Prepared pr;
            st = prepare_circuit(ctx, *c, bc, 0, 0, params_dev, feats_dev, B, sc.mats, &pr);
            if (st != QSV_OK) return st;
            st = run_circuit(ctx, *c, pr, A, bc, 0, nullptr, rm1);
            if (st != QSV_OK) return st;
        }
        st = losses(ctx, ob, A, bc, b0, P, sc.zpart, sc.zall, sc.coef, f);
        if (st != QSV_OK) return st;
        if (P == 0) return QSV_OK;
        // backward: lambda = O psi (and psi beside it unless its states were kept), taken back layer by layer
        QSV_HIP(ctx, launch_adj_init(A, n, kind, obs_qubit, mask, sc.coef, bc, sc.S, keep ? 0 : 1, ctx->stream),
                "adjoint init");
        RowMap rm2 = rm1;
        if (!keep) {
            rm2.per = 2;
            rm2.row0 = 2 * b0;
        }
        const int64_t back_rows = keep ? bc : 2 * bc;
        Prepared back;      // all layers' inverse matrices by one launch
        st = prepare_layers(ctx, *c, one, back_rows, 1, params_dev, feats_dev, B, sc.mats, &back);
        if (st != QSV_OK) return st;
        for (int l = L - 1; l >= 0; --l) {
            st = run_circuit(ctx, one, layer_of(back, l), sc.S, back_rows, 1, nullptr, rm2);
            if (st != QSV_OK) return st;
            const float2* psi0 = keep ? ck(l, b0) : sc.S;
            const float2* lam0 = keep ? sc.S : sc.S + amps;
            double* tp = sc.tp + (late ? (size_t)l * bc * n * adj_trans_count(n, bc) * 8 : 0);
            QSV_HIP(ctx, launch_trans(psi0, lam0, keep ? 1 : 2, n, bc, tp, ctx->stream), "transition sums");
            if (late && l > 0) continue;
            QSV_HIP(ctx, launch_adj_layers(sc.tp, bc, cd, l, late ? L : 1, params_dev, b0, P, back.mats, back.exec_of,
                                           back.form, f, ctx->stream),
                    "adjoint layers");
        }
        return QSV_OK;
    };
    Fork fork(ctx);
    if (two && chunk < B) {
        // Plans are uploaded on the stream that first asks for them: have the ones the chunks will use
        // in place before the second stream branches off (three calls: should the second one recycle
        // the plan buffer, the third brings the first plan back).
        if (!(ctx->opt_naive || n < kRegBits)) {
            const CachedPlan* warm = nullptr;
            for (int k = 0; k < 3; ++k) {
                const bool inv_plan = (k == 1);
                if (inv_plan && P == 0) continue;
                st = get_plan(ctx, (inv_plan || keep) ? one : *c, chunk, inv_plan ? 1 : 0, 0, &warm);
                if (st != QSV_OK) return st;
            }
        }
        if ((st = fork.begin()) != QSV_OK) return st;
    }
    int64_t ci = 0;
    for (int64_t b0 = 0; b0 < B; b0 += chunk, ++ci) {
        const int64_t bc = (B - b0) < chunk ? (B - b0) : chunk;
        st = run_chunk(b0, bc, scr[fork.take(ci)]);
        if (st != QSV_OK) return st;
    }
    if ((st = fork.join()) != QSV_OK) return st;
    QSV_HIP(ctx, launch_grad_finish(f, B, P, cd, feats_dev, loss_dev, grad_dev, mean_loss_dev,
                                    mean_grad_dev, ctx->stream),
            "grad finish");
    return QSV_OK;
}

qsv_status qsv_adjoint_grad(qsv_ctx* ctx, const qsv_circuit* c, const float* x_dev, int64_t dim,
                            const float* params_dev, const float* feats_dev, int32_t obs_qubit,
                            float* loss_dev, float* grad_dev, float* mean_loss_dev, float* mean_grad_dev) {
    return adjoint_impl(ctx, c, x_dev, dim, params_dev, feats_dev, 0, obs_qubit, 0, nullptr, loss_dev,
                        grad_dev, mean_loss_dev, mean_grad_dev);
}

qsv_status qsv_loss_grad(qsv_ctx* ctx, const qsv_circuit* c, const float* x_dev, int64_t dim,
                         const float* params_dev, const float* feats_dev, const qsv_loss* loss,
                         float* loss_dev, float* grad_dev, float* mean_loss_dev, float* mean_grad_dev) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    if (!loss) return fail(ctx, QSV_ERR_INVALID_ARG, "loss is NULL");
    if (loss->kind != QSV_LOSS_TRASH && loss->kind != QSV_LOSS_MSE_Z)
        return fail(ctx, QSV_ERR_INVALID_ARG, "unknown loss kind");
    return adjoint_impl(ctx, c, x_dev, dim, params_dev, feats_dev, loss->kind == QSV_LOSS_TRASH ? 1 : 2, 0,
                        loss->mask, loss->targets_dev, loss_dev, grad_dev, mean_loss_dev, mean_grad_dev);
}

qsv_status qsv_sgd_step(qsv_ctx* ctx, float* params_dev, const float* grad_dev, int64_t count, double lr) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    if (count < 0 || (count > 0 && (!params_dev || !grad_dev)))
        return fail(ctx, QSV_ERR_INVALID_ARG, "qsv_sgd_step: bad arguments");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    QSV_HIP(ctx, launch_sgd(params_dev, grad_dev, count, lr, ctx->stream), "sgd step");
    return QSV_OK;
}

qsv_status qsv_adam_step(qsv_ctx* ctx, float* params_dev, const float* grad_dev, float* m_dev, float* v_dev,
                         int64_t count, int64_t t, double lr, double beta1, double beta2, double eps) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    if (count < 0 || t < 1 || (count > 0 && (!params_dev || !grad_dev || !m_dev || !v_dev)) ||
        !(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0) || !(eps > 0.0))
        return fail(ctx, QSV_ERR_INVALID_ARG, "qsv_adam_step: bad arguments");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    QSV_HIP(ctx, launch_adam(params_dev, grad_dev, m_dev, v_dev, count, t, lr, beta1, beta2, eps, ctx->stream),
            "adam step");
    return QSV_OK;
}

qsv_status qsv_probe_pass(qsv_ctx* ctx, int low_bits, int window_start, int transposes) {
    if (!ctx) return QSV_ERR_INVALID_ARG;
    const int n = ctx->n;
    if (n < kRegBits) return fail(ctx, QSV_ERR_UNSUPPORTED, "probe needs n_qubits >= 4");
    const int tile = ctx->opt_tile ? ctx->opt_tile : default_tile(n, ctx->batch);
    const int ext = n + ceil_log2_i64(ctx->batch);
    if (low_bits < kLowBits || low_bits > tile || window_start < low_bits ||
        (ext > tile && window_start + (tile - low_bits) > ext) || (ext <= tile && window_start != low_bits))
        return fail(ctx, QSV_ERR_INVALID_ARG, "probe geometry does not fit the state");
    if (transposes < 0 || transposes > 16) return fail(ctx, QSV_ERR_INVALID_ARG, "transposes must be in 0..16");
    qsv_status st = bind_device(ctx);
    if (st != QSV_OK) return st;
    Arena ar(ctx);
    Op* dev = (Op*)ar.take(32 * sizeof(Op));
    if (!dev) return ws_fail(ctx, ar, "qsv_probe_pass");
    std::vector<Op> ops;
    const int smax = tile - kRegBits;
    const int sio = ctx->opt_probe_layout >= 0 ? std::min(ctx->opt_probe_layout, smax) : smax;
    ops.push_back({OP_LOAD, (uint8_t)sio, 0, 0, 0});
    for (int i = 0; i < transposes; ++i)
        ops.push_back({OP_XPOSE, (uint8_t)((i & 1) ? sio : (sio ? 0 : smax)), 0, 0, 0});
    ops.push_back({OP_END, 0, 0, 0, 0});
    set_transpose_barriers(ops);
    // a window over qubits alone goes through the kernel that the circuits use
    DirectPlan low;
    const bool direct = n >= tile && n <= kDirectMaxQubits && window_start + tile - low_bits <= n &&
                        (ctx->opt_planes == 1 || tile == kMaxTile) && lower_pass(ops.data(), (int)ops.size(), &low);
    // a small synchronous upload: this is a measurement aid, not part of the hot path
    const void* list = direct ? (const void*)low.ops.data() : (const void*)ops.data();
    QSV_HIP(ctx, hipMemcpyAsync(dev, list, (direct ? low.ops.size() : ops.size()) * sizeof(Op), hipMemcpyHostToDevice,
                                ctx->stream),
            "upload probe");
    QSV_HIP(ctx, hipStreamSynchronize(ctx->stream), "upload probe");
    PassArgs a{};
    a.state = ctx->state;
    a.in = ctx->state;
    a.imap = nullptr;
    a.src = nullptr;
    a.zout = nullptr; a.unturned = nullptr; a.turns = 0; a.zq = 0; a.nostore = 0;
    a.nt_store = ctx->opt_nt_store >= 0 ? ctx->opt_nt_store : ((((uint64_t)ctx->batch << n) * 8) >= kNtStoreBytes ? 1 : 0);
    a.rev = ctx->opt_rev != 0 && (ctx->probe_count++ & 1) ? 2 : 0;      // as run_circuit's passes without a map
    a.ops = dev;
    a.mats = reinterpret_cast<const float*>(dev);   // no unitaries, but the first table entry is fetched unseen
    a.exec_of = nullptr;
    a.ovr = nullptr;
    a.total = (uint64_t)ctx->batch << n;
    a.prio = ctx->opt_prio;
    a.n = n; a.c = low_bits; a.w = window_start;
    a.n_mats = 0;
    a.rowdep = 0;
    a.rm = plain_rows(n);
    a.direct = direct;
    a.gather = 0;
    a.mate = 0;
    a.s_in = direct ? low.passes[0].s_in : 0;
    a.s_out = direct ? low.passes[0].s_out : 0;
    a.first_mat = 0;
    a.g_sample0 = a.g_rem0 = 0;
    const uint64_t n_tiles = direct ? (uint64_t)ctx->batch << (n - tile) : ext > tile ? (1ull << (ext - tile)) : 1ull;
    QSV_HIP(ctx, launch_pass(tile, direct ? 1 : ctx->opt_planes, a, n_tiles, ctx->stream), "probe pass");
    return QSV_OK;
}

}  // extern "C"
