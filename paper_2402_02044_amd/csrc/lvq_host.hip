// lvq_host.hip -- host side of the C ABI declared in include/lvq.h: argument
// checks, the device store, per-stream workspaces, epochs, and kernel
// dispatch.  Every computation of the path runs in the kernels; this file
// only validates, allocates and launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <new>
#include <vector>

#include "lvq_index.h"

namespace lvq {

bool make_format(const lvq_config &c, Format *f)
{
    if (c.dim < 1 || c.dim > 8192) return false;
    if (c.bits1 != 4 && c.bits1 != 8) return false;
    if (c.bits2 != 0 && c.bits2 != 4 && c.bits2 != 8) return false;
    if (c.layout != LVQ_SEQUENTIAL && c.layout != LVQ_TURBO) return false;
    if (c.align != 32 && c.align != 64 && c.align != 128) return false;
    if (c.metric != LVQ_L2 && c.metric != LVQ_IP) return false;
    auto up = [](int v, int m) { return (v + m - 1) / m * m; };
    int blk = c.layout == LVQ_TURBO ? (c.bits1 == 4 ? 128 : 64) : (c.bits1 == 4 ? 8 : 4);
    f->dim = c.dim;
    f->bits1 = c.bits1;
    f->bits2 = c.bits2;
    f->layout = c.layout;
    f->align = c.align;
    f->npos = up(c.dim, blk);
    f->code_bytes = f->npos * c.bits1 / 8;
    f->row_bytes = up(kHeaderBytes + f->code_bytes, c.align);
    f->resid_bytes = c.bits2 ? up(f->npos * c.bits2 / 8, c.align) : 0;
    f->kchunks = up(f->code_bytes, 16) / 16;
    f->kpos = f->kchunks * 16 * 8 / c.bits1;
    return true;
}

// dimension held at code position p (the row format of lvq.h)
static int pos_dim(const Format &f, int p)
{
    if (p >= f.npos) return -1;
    int dim = p;
    if (f.layout == LVQ_TURBO) {
        const int per = 32 / f.bits1, blk = f.bits1 == 4 ? 128 : 64;
        const int b = p / blk, r = p % blk, w = r / per, k = r % per;
        dim = b * blk + 16 * k + w;
    }
    return dim < f.dim ? dim : -1;
}

void kernel_order_dims(const Format &f, int32_t *kdim)
{
    for (int s = 0; s < f.kpos; ++s) {
        int p = s;
        if (f.bits1 == 4) {
            const int w = s / 8, r = s % 8;
            p = 8 * w + (r < 4 ? 2 * r : 2 * (r - 4) + 1);
        }
        kdim[s] = pos_dim(f, p);
    }
}

}  // namespace lvq

using namespace lvq;

namespace {

int map_hip(hipError_t e)
{
    if (e == hipSuccess) return LVQ_OK;
    if (e == hipErrorOutOfMemory) return LVQ_ERR_OOM;
    return LVQ_ERR_DEVICE;
}

#define LVQ_HIP(x)                         \
    do {                                   \
        hipError_t e_ = (x);               \
        if (e_ != hipSuccess) return map_hip(e_); \
    } while (0)

int dev_alloc(lvq_index *ix, DevBuf &b, size_t bytes)
{
    if (b.bytes >= bytes && b.p) return LVQ_OK;
    if (ix->capturing) return LVQ_ERR_INVALID_ARG;   // no allocation inside graph capture
    if (b.pinned) return LVQ_ERR_INVALID_ARG;        // a captured graph still reads it
    if (bytes == 0) bytes = 16;
    const int64_t grow = (int64_t)bytes - (int64_t)b.bytes;
    if (ix->cfg.mem_budget_bytes > 0 && ix->device_bytes + grow > ix->cfg.mem_budget_bytes)
        return LVQ_ERR_OOM;
    void *p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) return LVQ_ERR_OOM;
    if (b.p) {
        (void)hipDeviceSynchronize();
        (void)hipFree(b.p);
    }
    ix->device_bytes += grow;
    b.p = p;
    b.bytes = bytes;
    return LVQ_OK;
}

void dev_free(lvq_index *ix, DevBuf &b)
{
    if (b.p) (void)hipFree(b.p);
    ix->device_bytes -= (int64_t)b.bytes;
    b.p = nullptr;
    b.bytes = 0;
}

template <class T>
T *P(DevBuf &b)
{
    return reinterpret_cast<T *>(b.p);
}

bool finite_host(const float *v, size_t n)
{
    for (size_t i = 0; i < n; ++i)
        if (!std::isfinite(v[i])) return false;
    return true;
}

// Rebuild the device means tables for ids [0, n_means).
int upload_means(lvq_index *ix, const std::vector<float> &all)
{
    const Format &f = ix->f;
    const int M = ix->n_means, d = f.dim;
    std::vector<float> mt((size_t)d * kMaxMeans, 0.0f), mk((size_t)M * f.kpos, 0.0f);
    std::vector<int32_t> kd(f.kpos);
    kernel_order_dims(f, kd.data());
    for (int m = 0; m < M; ++m)
        for (int j = 0; j < d; ++j) mt[(size_t)j * kMaxMeans + m] = all[(size_t)m * d + j];
    for (int m = 0; m < M; ++m)
        for (int s = 0; s < f.kpos; ++s)
            if (kd[s] >= 0) mk[(size_t)m * f.kpos + s] = all[(size_t)m * d + kd[s]];
    int rc;
    if ((rc = dev_alloc(ix, ix->means, sizeof(float) * (size_t)kMaxMeans * d))) return rc;
    if ((rc = dev_alloc(ix, ix->means_t, sizeof(float) * (size_t)kMaxMeans * d))) return rc;
    if ((rc = dev_alloc(ix, ix->muk, sizeof(float) * (size_t)kMaxMeans * f.kpos))) return rc;
    LVQ_HIP(hipMemcpy(ix->means.p, all.data(), sizeof(float) * (size_t)M * d, hipMemcpyHostToDevice));
    LVQ_HIP(hipMemcpy(ix->means_t.p, mt.data(), sizeof(float) * mt.size(), hipMemcpyHostToDevice));
    LVQ_HIP(hipMemcpy(ix->muk.p, mk.data(), sizeof(float) * mk.size(), hipMemcpyHostToDevice));
    return LVQ_OK;
}

Workspace &workspace(lvq_index *ix, hipStream_t s) { return ix->ws[s]; }

// After a captured call on `s`: its workspace buffers (which the graph's
// kernels read and write) are never freed or grown again, and the occupied-
// slot list a captured scan walks is never recycled by consolidation.
void pin_after_capture(lvq_index *ix, hipStream_t s, bool reads_list)
{
    if (!ix->capturing) return;
    Workspace &w = ix->ws[s];
    for (DevBuf *b : {&w.qk, &w.qsum, &w.cm, &w.order, &w.queue, &w.part, &w.q16, &w.gthr, &w.mkeys, &w.members, &w.moffs,
                      &w.mcount, &w.mcursor, &w.probe, &w.qoffs, &w.qids, &w.assign})
        if (b->p) b->pinned = true;
    if (reads_list && ix->list_active >= 0) ix->lists[ix->list_active].captured = true;
}

// Record whether `s` is capturing a HIP graph: captured calls allocate
// nothing, skip cross-stream ordering and in-flight bookkeeping, and replay
// at the epoch of capture.
int begin_call(lvq_index *ix, hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    LVQ_HIP(hipStreamIsCapturing(s, &st));
    ix->capturing = st != hipStreamCaptureStatusNone;
    return LVQ_OK;
}

// The same question for a call that keeps no record of a capture: updates and
// lvq_encode, which leave ix->capturing false.
bool stream_captures(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;   // (another stream's capture forbids the question: nothing is allocated)
}

// Make work on `s` wait for the latest store update issued on another stream.
int order_after_updates(lvq_index *ix, hipStream_t s)
{
    if (ix->capturing) return LVQ_OK;
    if (ix->have_update && ix->update_stream != s) LVQ_HIP(hipStreamWaitEvent(s, ix->update_ev, 0));
    return LVQ_OK;
}

int note_update(lvq_index *ix, hipStream_t s)
{
    ix->version += 1;
    LVQ_HIP(hipEventRecord(ix->update_ev, s));
    ix->update_stream = s;
    ix->have_update = true;
    return LVQ_OK;
}

// may_create = false (the allocation-free entry point): with no spare event,
// wait for the oldest in-flight launch and take its event (lvq_create makes
// a few spare events, so one of the two lists is never empty).
int note_query(lvq_index *ix, hipStream_t s, uint32_t epoch, bool may_create = true)
{
    if (ix->capturing) return LVQ_OK;
    hipEvent_t ev;
    if (ix->spare_events.empty() && !may_create) {
        if (ix->inflight.empty()) return LVQ_ERR_DEVICE;
        LVQ_HIP(hipEventSynchronize(ix->inflight.front().ev));
        ix->spare_events.push_back(ix->inflight.front().ev);
        ix->inflight.pop_front();
    }
    if (!ix->spare_events.empty()) {
        ev = ix->spare_events.back();
        ix->spare_events.pop_back();
    } else {
        LVQ_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    }
    LVQ_HIP(hipEventRecord(ev, s));
    ix->inflight.push_back({epoch, ++ix->query_seq, ev});
    // retire completed entries from the front
    while (!ix->inflight.empty() && hipEventQuery(ix->inflight.front().ev) == hipSuccess) {
        ix->spare_events.push_back(ix->inflight.front().ev);
        ix->inflight.pop_front();
    }
    return LVQ_OK;
}

// Bracket the main kernel with events when timing is enabled.
int timing_begin(lvq_index *ix, hipStream_t s)
{
    if (!ix->timing || ix->capturing) return LVQ_OK;
    hipEvent_t a, b;
    LVQ_HIP(hipEventCreate(&a));
    LVQ_HIP(hipEventCreate(&b));
    LVQ_HIP(hipEventRecord(a, s));
    ix->tev.push_back({a, b});
    return LVQ_OK;
}

int timing_end(lvq_index *ix, hipStream_t s)
{
    if (!ix->timing || ix->capturing || ix->tev.empty()) return LVQ_OK;
    LVQ_HIP(hipEventRecord(ix->tev.back().second, s));
    return LVQ_OK;
}

PrepArgs prep_args(lvq_index *ix, const float *q, int64_t nq, float *qk, float *qsum, float *cm)
{
    const Format &f = ix->f;
    PrepArgs pa;
    pa.q = q;
    pa.nq = nq;
    pa.dim = f.dim;
    pa.kpos = f.kpos;
    pa.n_means = ix->n_means;
    pa.metric = ix->cfg.metric;
    pa.kdim = P<int32_t>(ix->kdim);
    pa.means = P<float>(ix->means);
    pa.qk = qk;
    pa.qsum = qsum;
    pa.cm = cm;
    return pa;
}

// Query prep into the given buffers (nq x kpos, nq, nq x n_means floats).
int prep_into(lvq_index *ix, const float *q, int64_t nq, float *qk, float *qsum, float *cm, hipStream_t s)
{
    LVQ_HIP(launch_prep(prep_args(ix, q, nq, qk, qsum, cm), s));
    return LVQ_OK;
}

// Bytes of the vector scan's query table, in tiles of tq queries, and of the
// queries' shared bounds behind it (both in Workspace::qk).
size_t scan_table_bytes(const lvq_index *ix, int64_t nq, int tq)
{
    return sizeof(float) * (size_t)((nq + tq - 1) / tq * tq * ix->f.kpos + nq);
}

// Room for the prepared queries of a batch in the stream's workspace (without a
// budget, for a scan of as many queries in tiles of 16 too: after a capture it
// cannot grow).
int size_queries(lvq_index *ix, Workspace &w, int64_t nq)
{
    nq = std::max<int64_t>(nq, 1);
    const size_t exact = sizeof(float) * (size_t)nq * ix->f.kpos;
    int rc = LVQ_ERR_OOM;
    if (w.qk.bytes < exact && !ix->capturing && !w.qk.pinned && ix->cfg.mem_budget_bytes <= 0 &&
        (rc = dev_alloc(ix, w.qk, scan_table_bytes(ix, nq, 16))))
        (void)hipGetLastError();
    if (rc && (rc = dev_alloc(ix, w.qk, exact))) return rc;
    if ((rc = dev_alloc(ix, w.qsum, sizeof(float) * (size_t)nq))) return rc;
    return dev_alloc(ix, w.cm, sizeof(float) * (size_t)nq * ix->n_means);
}

int prep_queries(lvq_index *ix, Workspace &w, const float *q, int64_t nq, hipStream_t s)
{
    const int rc = size_queries(ix, w, nq);
    return rc ? rc : prep_into(ix, q, nq, P<float>(w.qk), P<float>(w.qsum), P<float>(w.cm), s);
}

// Order of sums of the default tile shape: that of the shape, among those
// with an order of their own, whose round covers the code bytes with the
// least waste, preferring more lanes per candidate.
int order_shape(const Format &f, void *(*lookup)(int, int, int), int bits2, int variant)
{
    const int bytes = f.kchunks * 16;
    int best = -1;
    double best_cost = 1e30;
    for (int i = 0; i < num_tile_shapes(); ++i) {
        if (!lookup(bits2, variant, i)) continue;
        TileShape t = tile_shape(i);
        if (t.pipe & 48) continue;
        const int round = t.g * t.ch * t.nch;
        const int rounds = (bytes + round - 1) / round;
        if (t.pipe && rounds > 1) continue;
        const double waste = (double)rounds * round / bytes;
        const double cost = waste * 16.0 / t.g + (rounds > 1 ? 0.5 * rounds : 0.0);
        if (cost < best_cost) {
            best_cost = cost;
            best = i;
        }
    }
    return best;
}

// A shape can score the rows of a format at a level: it is instantiated, and a
// pipelined one reads the whole row in its one round.
bool shape_fits(const Format &f, void *(*lookup)(int, int, int), int bits2, int variant, int shape)
{
    if (shape < 0 || shape >= num_tile_shapes() || !lookup(bits2, variant, shape)) return false;
    TileShape t = tile_shape(shape);
    return !t.pipe || t.g * t.ch * t.nch >= f.kchunks * 16;
}

// Short rows: up to this many workgroups per compute unit run as they come,
// without an order and a counter, resident or not (see host_distances).
constexpr int kShortRowsPerUnit = 6;

// Default tile shape: the layout measured fastest among those that give every
// value with the order of sums of order_shape, so that results do not depend
// on the choice.  Microseconds for 3.0e6 pairs of 3,000 ragged lists, top-10
// (the 16-lane shape of that order first, then the layouts compared):
//   rows of <= 64 B    30: 4-bit d = 128 L2 573 / 137; 4x8 d = 96 IP 711 / 302
//   rows of <= 96 B    31: 8-bit d = 96 L2 411 / 118, 16 means 391 / 119, IP
//                      360 / 116 (34: 194, 209, 159); not 4-bit codes at both
//                      levels, whose four sums per lane spill (698 / 550; 35: 353)
//   rows of <= 128 B   32 at the first level: 8-bit d = 128 L2 451 / 168 (34:
//                      200); not 4-bit Euclidean with one mean (580 / 303; 34:
//                      212), nor both levels (645 / 290; 34: 243)
//   up to 384 B        34, or 35 (query in registers) where its registers cost
//                      no occupancy: IP with both levels of 4-bit codes (4x8 d
//                      = 768 1189 / 561, 34: 578) or 8-bit codes alone (d = 256
//                      414 / 189, 34: 199), L2 with 8-bit codes alone (d = 256
//                      465 / 208, 34: 277; but 4x8 d = 768 34: 636, 35: 784)
//   up to 512 B        18 (query in registers), 10 with several means: 8-bit
//                      d = 512 IP 551 / 317, L2 529 / 320
//   padding positions  33 up to 128 B (8-bit d = 100 L2 586 / 137), 10 up to 512
//                      B (8-bit d = 333 L2 636 / 303)
// Many lists per compute unit (per_unit) of few entries each (avg) keep the
// 16-lane shape where it was faster for them, microseconds (16-lane / above):
// below 32 entries the first level in up to 128 B (3,000 lists of 20, IP, 8-bit d
// = 96 65 / 73, d = 128 66 / 75, of 50 76 / 74 and 78 / 78; both levels gain: 4x8
// d = 96 73 / 67); with both levels of 4-bit codes the 8-lane shapes hold two
// waves per SIMD, the 16-lane one four, which hide the lists' set-up (4x8 d = 768 IP, 10,000 lists of 50 269 / 276, of
// 100 366 / 350, 3,000 of 50 108 / 99; d = 192 10,000 of 100 308 / 316; L2 d = 768
// 3,000 of 50 89 / 93, of 400 258 / 267, of 1,000 581 / 560; 16 means, of 5 131 /
// 148, of 20 158 / 159).
// *idle: query slots a lane without a piece multiplied by zero codes in the
// 16-lane shape (see CandArgs::idle_slots).
int default_shape(const Format &f, void *(*lookup)(int, int, int), int bits2, int variant, double per_unit,
                  double avg, int *idle)
{
    const int base = order_shape(f, lookup, bits2, variant);
    *idle = 0;
    if (base < 0) return base;
    const int bytes = f.kchunks * 16;
    const TileShape t = tile_shape(base);
    const bool ip = variant == 0, one = variant < 2;
    int pick = base;
    if (t.g == 16 && t.ch == 8 && t.nch == 3 && !t.pipe) {
        const bool b4 = f.bits1 == 4, both = bits2 != 0;
        if (bytes <= 64) pick = 30;
        else if (bytes <= 96 && !(b4 && both)) pick = 31;
        else if (bytes <= 128 && !both && !(b4 && variant == 1)) pick = 32;
        else pick = one && (ip ? b4 == both : !b4 && !both) ? 35 : 34;
        const bool deep = pick >= 34 && b4 && both;
        const double few = deep ? (ip ? 100.0 : one ? 512.0 : 20.0) : pick > 32 || both ? 0.0 : 32.0;
        const double from = !deep ? kShortRowsPerUnit : !ip && bytes > 192 && avg >= 32.0 ? 10.0 : 16.0;
        if (per_unit > from && avg < few) return base;
    } else if (t.g == 16 && t.ch == 16 && t.nch == 2) {
        if (variant >= 3) pick = bytes <= 128 ? 33 : 10;
        else pick = one ? 18 : 10;
    }
    // (rows of 1040 to 1152 bytes take the order of three rounds of 384)
    if (pick == base || !shape_fits(f, lookup, bits2, variant, pick)) return base;
    if (ip && bytes < t.g * t.ch * t.nch) *idle = t.ch * 8 / f.bits1;
    return pick;
}

}  // namespace

namespace lvq {

int host_begin_call(lvq_index *ix, hipStream_t s) { return begin_call(ix, s); }
int host_note_query(lvq_index *ix, hipStream_t s, uint32_t epoch, bool may_create)
{
    return note_query(ix, s, epoch, may_create);
}
int host_alloc(lvq_index *ix, DevBuf &b, size_t bytes) { return dev_alloc(ix, b, bytes); }
void host_free(lvq_index *ix, DevBuf &b) { dev_free(ix, b); }

}  // namespace lvq

extern "C" {

const char *lvq_strerror(int code)
{
    switch (code) {
    case LVQ_OK: return "ok";
    case LVQ_ERR_INVALID_ARG: return "invalid argument";
    case LVQ_ERR_UNSUPPORTED: return "unsupported configuration";
    case LVQ_ERR_OOM: return "out of device memory or over the memory budget";
    case LVQ_ERR_CAPACITY: return "not enough free slots";
    case LVQ_ERR_DEVICE: return "HIP runtime error";
    case LVQ_ERR_NONFINITE: return "non-finite input vector";
    case LVQ_ERR_BAD_SLOT: return "slot out of range or not live";
    case LVQ_ERR_SCRATCH: return "request exceeds the fixed scratch of the allocation-free entry point";
    default: return "unknown error";
    }
}

int lvq_row_format(const lvq_config *cfg, int32_t *row_bytes, int32_t *resid_bytes, int32_t *code_positions)
{
    Format f;
    if (!cfg || !make_format(*cfg, &f)) return LVQ_ERR_INVALID_ARG;
    if (row_bytes) *row_bytes = f.row_bytes;
    if (resid_bytes) *resid_bytes = f.resid_bytes;
    if (code_positions) *code_positions = f.npos;
    return LVQ_OK;
}

int lvq_create(const lvq_config *cfg, const float *means_host, int32_t n_means, lvq_index **out)
{
    if (!cfg || !out || !means_host) return LVQ_ERR_INVALID_ARG;
    *out = nullptr;
    Format f;
    if (!make_format(*cfg, &f)) return LVQ_ERR_INVALID_ARG;
    if (n_means < 1 || n_means > kMaxMeans || cfg->capacity < 0 || cfg->capacity > INT32_MAX)
        return LVQ_ERR_INVALID_ARG;
    if (!finite_host(means_host, (size_t)n_means * cfg->dim)) return LVQ_ERR_NONFINITE;
    lvq_index *ix = new (std::nothrow) lvq_index();
    if (!ix) return LVQ_ERR_OOM;
    ix->cfg = *cfg;
    ix->f = f;
    ix->n_means = n_means;
    int rc = LVQ_OK;
    do {
        if (hipGetDevice(&ix->device) != hipSuccess) { rc = LVQ_ERR_DEVICE; break; }
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, ix->device) == hipSuccess) {
            ix->n_cu = prop.multiProcessorCount;
            ix->lds_max = prop.sharedMemPerBlock;
        }
        std::vector<float> all(means_host, means_host + (size_t)n_means * cfg->dim);
        if ((rc = upload_means(ix, all))) break;
        std::vector<int32_t> kd(f.kpos);
        kernel_order_dims(f, kd.data());
        std::vector<float> km(f.kpos);
        for (int s = 0; s < f.kpos; ++s) km[s] = kd[s] >= 0 ? 1.0f : 0.0f;
        if ((rc = dev_alloc(ix, ix->kdim, sizeof(int32_t) * f.kpos))) break;
        if ((rc = dev_alloc(ix, ix->kmask, sizeof(float) * f.kpos))) break;
        if ((rc = dev_alloc(ix, ix->err, 16))) break;
        if ((rc = dev_alloc(ix, ix->scratch, 4096))) break;
        if ((rc = dev_alloc(ix, ix->mean_active, kMaxMeans))) break;
        if ((rc = dev_alloc(ix, ix->mean_counts, sizeof(uint64_t) * kMaxMeans))) break;
        ix->retired.assign(kMaxMeans, 0);
        if (hipMemset(ix->mean_active.p, 1, kMaxMeans)) {
            rc = LVQ_ERR_DEVICE;
            break;
        }
        if (hipMemcpy(ix->kdim.p, kd.data(), sizeof(int32_t) * f.kpos, hipMemcpyHostToDevice) ||
            hipMemcpy(ix->kmask.p, km.data(), sizeof(float) * f.kpos, hipMemcpyHostToDevice) ||
            hipMemset(ix->err.p, 0, 16)) {
            rc = LVQ_ERR_DEVICE;
            break;
        }
        const int64_t cap = cfg->capacity;
        if (cap > 0) {
            if ((rc = dev_alloc(ix, ix->rows, (size_t)cap * f.row_bytes))) break;
            if (f.resid_bytes && (rc = dev_alloc(ix, ix->resid, (size_t)cap * f.resid_bytes))) break;
            if ((rc = dev_alloc(ix, ix->stack, sizeof(int32_t) * (size_t)cap))) break;
            if (hipMemset(ix->rows.p, 0, (size_t)cap * f.row_bytes) ||
                (f.resid_bytes && hipMemset(ix->resid.p, 0, (size_t)cap * f.resid_bytes))) {
                rc = LVQ_ERR_DEVICE;
                break;
            }
            std::vector<int32_t> st(cap);
            for (int64_t i = 0; i < cap; ++i) st[i] = (int32_t)(cap - 1 - i);
            if (hipMemcpy(ix->stack.p, st.data(), sizeof(int32_t) * cap, hipMemcpyHostToDevice)) {
                rc = LVQ_ERR_DEVICE;
                break;
            }
        }
        ix->free_top = cap;
        if (cap > 0) {
            ix->lists.resize(1);
            if ((rc = dev_alloc(ix, ix->lists[0].buf, sizeof(int32_t) * (size_t)cap))) break;
            ix->list_active = 0;
            ix->list_len = 0;
        }
        if (hipEventCreateWithFlags(&ix->update_ev, hipEventDisableTiming)) { rc = LVQ_ERR_DEVICE; break; }
        for (int i = 0; i < 8 && rc == LVQ_OK; ++i) {
            hipEvent_t ev;
            if (hipEventCreateWithFlags(&ev, hipEventDisableTiming)) rc = LVQ_ERR_DEVICE;
            else ix->spare_events.push_back(ev);
        }
        if (rc) break;
        if ((rc = noalloc_setup(ix->device))) break;
    } while (0);
    if (rc) {
        lvq_destroy(ix);
        return rc;
    }
    *out = ix;
    return LVQ_OK;
}

int lvq_destroy(lvq_index *ix)
{
    if (!ix) return LVQ_ERR_INVALID_ARG;
    (void)hipDeviceSynchronize();
    for (auto &kv : ix->ws) {
        Workspace &w = kv.second;
        for (DevBuf *b : {&w.qk, &w.qsum, &w.cm, &w.order, &w.queue, &w.part, &w.q16, &w.gthr, &w.mkeys, &w.members, &w.moffs,
                          &w.mcount, &w.mcursor, &w.probe, &w.qoffs, &w.qids, &w.assign})
            dev_free(ix, *b);
    }
    for (DevBuf *b : {&ix->means, &ix->means_t, &ix->muk, &ix->kmask, &ix->kdim, &ix->rows,
                      &ix->resid, &ix->stack, &ix->err, &ix->scratch, &ix->slot_bits, &ix->mean_active, &ix->mean_counts})
        dev_free(ix, *b);
    for (SlotList &l : ix->lists) dev_free(ix, l.buf);
    for (auto &f : ix->inflight) (void)hipEventDestroy(f.ev);
    for (auto e : ix->spare_events) (void)hipEventDestroy(e);
    if (ix->update_ev) (void)hipEventDestroy(ix->update_ev);
    delete ix;
    return LVQ_OK;
}

int lvq_set_means(lvq_index *ix, const float *means_host, int32_t n_means, int32_t *first_id_out, void *stream)
{
    if (!ix || !means_host || n_means < 1 || n_means > kMaxMeans) return LVQ_ERR_INVALID_ARG;
    const Format &f = ix->f;
    const int d = f.dim;
    if (!finite_host(means_host, (size_t)n_means * d)) return LVQ_ERR_NONFINITE;
    hipStream_t s = (hipStream_t)stream;
    // tables for the new ids only: work already queued reads ids below the old count
    std::vector<float> mt((size_t)d * n_means), mk((size_t)n_means * f.kpos, 0.0f);
    std::vector<int32_t> kd(f.kpos);
    kernel_order_dims(f, kd.data());
    for (int m = 0; m < n_means; ++m)
        for (int j = 0; j < d; ++j) mt[(size_t)j * n_means + m] = means_host[(size_t)m * d + j];
    for (int m = 0; m < n_means; ++m)
        for (int t = 0; t < f.kpos; ++t)
            if (kd[t] >= 0) mk[(size_t)m * f.kpos + t] = means_host[(size_t)m * d + kd[t]];
    int first = 0;
    {
        std::lock_guard<std::mutex> lk(ix->mu);
        if (ix->n_means + n_means > kMaxMeans) return LVQ_ERR_CAPACITY;
        int rc = begin_call(ix, s);
        if (rc) return rc;
        if (ix->capturing) {
            ix->capturing = false;
            return LVQ_ERR_INVALID_ARG;
        }
        if ((rc = order_after_updates(ix, s))) return rc;
        first = ix->n_means;
        LVQ_HIP(hipMemcpyAsync(P<float>(ix->means) + (size_t)first * d, means_host, sizeof(float) * mt.size(),
                               hipMemcpyHostToDevice, s));
        LVQ_HIP(hipMemcpy2DAsync(P<float>(ix->means_t) + first, sizeof(float) * kMaxMeans, mt.data(),
                                 sizeof(float) * n_means, sizeof(float) * n_means, d, hipMemcpyHostToDevice, s));
        LVQ_HIP(hipMemcpyAsync(P<float>(ix->muk) + (size_t)first * f.kpos, mk.data(), sizeof(float) * mk.size(),
                               hipMemcpyHostToDevice, s));
        ix->n_means += n_means;
        if ((rc = note_update(ix, s))) return rc;
    }
    // the host sources must outlive the copies
    LVQ_HIP(hipStreamSynchronize(s));
    if (first_id_out) *first_id_out = first;
    return LVQ_OK;
}

constexpr int64_t kAssignRun = 1 << 20;   // vectors per pass of the nearest-mean kernel

static int encode_common(lvq_index *ix, const float *x, int64_t n, uint8_t *rows, uint8_t *resid,
                         const uint64_t *ext, int32_t *slots_out, bool store, hipStream_t s)
{
    EncodeArgs a;
    a.x = x;
    a.n = n;
    a.means = P<float>(ix->means);
    a.means_t = P<float>(ix->means_t);
    a.means_t_stride = kMaxMeans;
    a.n_means = ix->n_means;
    a.means_lds = ix->n_means > 1 && (size_t)ix->n_means * ix->f.dim * sizeof(float) <= 32768 ? 1 : 0;
    a.mean_active = P<uint8_t>(ix->mean_active);
    a.f = ix->f;
    a.rows = rows;
    a.resid = resid;
    a.free_stack = store ? P<int32_t>(ix->stack) : nullptr;
    a.free_top = ix->free_top;
    a.list_out = store ? P<int32_t>(ix->lists[ix->list_active].buf) + ix->list_len : nullptr;
    a.slots_out = slots_out;
    a.ext_ids = ext;
    a.epoch = ix->epoch;
    a.err = P<uint32_t>(ix->err);
    // Several means: found in a kernel of its own where that pays and there is
    // room for the ids (this stream's own buffer; in a captured call or under a
    // memory budget, which it would take from the queries, the encoder searches).
    int32_t *buf = nullptr;
    if (encode_assigns(n, ix->f.dim, ix->n_means) && !stream_captures(s) && ix->cfg.mem_budget_bytes <= 0) {
        Workspace &w = workspace(ix, s);
        // (one size for the index's life: growing would wait for the whole device)
        if (dev_alloc(ix, w.assign, sizeof(int32_t) * (size_t)kAssignRun) == LVQ_OK)
            buf = P<int32_t>(w.assign);
        else
            (void)hipGetLastError();   // the call goes on without it
    }
    if (!buf) {
        LVQ_HIP(launch_encode(a, nullptr, s));
        return LVQ_OK;
    }
    for (int64_t at = 0; at < n; at += kAssignRun) {
        EncodeArgs p = a;
        p.n = std::min<int64_t>(n - at, kAssignRun);
        p.x = x + at * ix->f.dim;
        if (store) {
            p.free_top = a.free_top - at;
            p.list_out = a.list_out + at;
            p.slots_out = slots_out + at;
            if (ext) p.ext_ids = ext + at;
        } else {
            p.rows = rows + at * ix->f.row_bytes;
            if (resid) p.resid = resid + at * ix->f.resid_bytes;
        }
        LVQ_HIP(launch_encode(p, buf, s));
    }
    return LVQ_OK;
}

int lvq_encode(lvq_index *ix, const float *x_dev, int64_t n, uint8_t *rows_dev, uint8_t *resid_dev, void *stream)
{
    if (!ix || n < 0 || (n > 0 && (!x_dev || !rows_dev))) return LVQ_ERR_INVALID_ARG;
    if (ix->f.bits2 && n > 0 && !resid_dev) return LVQ_ERR_INVALID_ARG;
    if (n == 0) return LVQ_OK;
    std::lock_guard<std::mutex> lk(ix->mu);
    return encode_common(ix, x_dev, n, rows_dev, resid_dev, nullptr, nullptr, false, (hipStream_t)stream);
}

int lvq_insert(lvq_index *ix, const float *x_dev, int64_t n, const uint64_t *ext_ids_dev, int32_t *slots_out_dev,
               void *stream)
{
    if (!ix || n < 0 || (n > 0 && (!x_dev || !slots_out_dev))) return LVQ_ERR_INVALID_ARG;
    if (n == 0) return LVQ_OK;
    std::lock_guard<std::mutex> lk(ix->mu);
    if (n > ix->free_top) return LVQ_ERR_CAPACITY;
    hipStream_t s = (hipStream_t)stream;
    int rc = order_after_updates(ix, s);
    if (rc) return rc;
    ix->epoch += 1;
    rc = encode_common(ix, x_dev, n, P<uint8_t>(ix->rows), P<uint8_t>(ix->resid), ext_ids_dev, slots_out_dev,
                       true, s);
    if (rc) return rc;
    ix->free_top -= n;
    ix->list_len += n;
    return note_update(ix, s);
}

static StoreArgs store_args(lvq_index *ix)
{
    StoreArgs a;
    a.rows = P<uint8_t>(ix->rows);
    a.resid = P<uint8_t>(ix->resid);
    a.row_bytes = ix->f.row_bytes;
    a.resid_bytes = ix->f.resid_bytes;
    a.capacity = ix->cfg.capacity;
    a.epoch = ix->epoch;
    a.err = P<uint32_t>(ix->err);
    return a;
}

int lvq_delete(lvq_index *ix, const int32_t *slots_dev, int64_t n, void *stream)
{
    if (!ix || n < 0 || (n > 0 && !slots_dev)) return LVQ_ERR_INVALID_ARG;
    if (n == 0) return LVQ_OK;
    std::lock_guard<std::mutex> lk(ix->mu);
    hipStream_t s = (hipStream_t)stream;
    int rc = order_after_updates(ix, s);
    if (rc) return rc;
    ix->epoch += 1;
    LVQ_HIP(launch_delete(store_args(ix), slots_dev, n, s));
    return note_update(ix, s);
}

int lvq_consolidate(lvq_index *ix, void *stream, int64_t *n_freed_out)
{
    if (!ix) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    if (n_freed_out) *n_freed_out = 0;
    const int64_t cap = ix->cfg.capacity;
    if (cap == 0) return LVQ_OK;
    hipStream_t s = (hipStream_t)stream;
    int rc = order_after_updates(ix, s);
    if (rc) return rc;
    // the oldest epoch an unfinished query may still observe, and the oldest
    // launch still running
    uint32_t safe = ix->epoch;
    uint64_t oldest = UINT64_MAX;
    for (auto it = ix->inflight.begin(); it != ix->inflight.end();) {
        if (hipEventQuery(it->ev) == hipSuccess) {
            ix->spare_events.push_back(it->ev);
            it = ix->inflight.erase(it);
        } else {
            safe = std::min(safe, it->epoch);
            oldest = std::min(oldest, it->seq);
            ++it;
        }
    }
    // a list buffer for the compacted list: a retired one no running query
    // reads, else a new one
    int next = -1;
    for (int i = 0; i < (int)ix->lists.size(); ++i)
        if (i != ix->list_active && ix->lists[i].retire_seq < oldest && !ix->lists[i].captured) {
            next = i;
            break;
        }
    if (next < 0) {
        SlotList fresh_list;
        if ((rc = dev_alloc(ix, fresh_list.buf, sizeof(int32_t) * (size_t)cap))) return rc;
        ix->lists.push_back(fresh_list);
        next = (int)ix->lists.size() - 1;
    }
    // Room for a bit per slot, in a buffer of its own that never grows (growing
    // one waits for the device); not taken from a memory budget, nor where the
    // allocation fails: then the passes keep a count per block alone.
    auto up16 = [](size_t b) { return (b + 15) & ~(size_t)15; };
    size_t tail_at = up16(consolidate_scratch(cap, true));
    DevBuf *mem = ix->scratch.bytes >= tail_at + 16 ? &ix->scratch : &ix->slot_bits;
    if (mem == &ix->slot_bits && !mem->p && ix->cfg.mem_budget_bytes <= 0 && dev_alloc(ix, *mem, tail_at + 16) != LVQ_OK)
        (void)hipGetLastError();
    const bool bits = mem->p != nullptr;
    if (!bits) {
        mem = &ix->scratch;
        tail_at = up16(consolidate_scratch(cap, false));
        if ((rc = dev_alloc(ix, *mem, tail_at + 16))) return rc;
    }
    int64_t *tail = reinterpret_cast<int64_t *>(static_cast<char *>(mem->p) + tail_at);
    LVQ_HIP(launch_consolidate(store_args(ix), safe, P<int32_t>(ix->stack), ix->free_top,
                               P<int32_t>(ix->lists[next].buf), mem->p, bits, tail, s));
    int64_t got[2] = {0, 0};   // new stack top, list length
    LVQ_HIP(hipMemcpyAsync(got, tail, sizeof(got), hipMemcpyDeviceToHost, s));
    LVQ_HIP(hipStreamSynchronize(s));
    if (n_freed_out) *n_freed_out = got[0] - ix->free_top;
    ix->free_top = got[0];
    ix->lists[ix->list_active].retire_seq = ix->query_seq;   // every launch so far may read it
    ix->list_active = next;
    ix->list_len = got[1];
    return note_update(ix, s);
}

}  // extern "C"

int lvq::host_distances(lvq_index *ix, const float *q_dev, int64_t nq, const int64_t *offsets_dev,
                        const int32_t *ids_dev, int64_t total, int32_t level, float *dist_dev, int32_t k,
                        int32_t *topk_ids_dev, float *topk_dist_dev, hipStream_t s, int force_shape,
                        uint32_t epoch, bool neg_empty, const int32_t *list_means, int list_nmeans,
                        const int64_t *seg_offs, const int32_t *seg_members, const DistScratch *fixed)
{
    if (!ix || nq < 0 || total < 0 || nq > INT32_MAX) return LVQ_ERR_INVALID_ARG;
    const bool segmented = seg_members != nullptr;
    if (segmented && (!seg_offs || !list_means)) return LVQ_ERR_INVALID_ARG;
    if (level != LVQ_PRIMARY && level != LVQ_FULL) return LVQ_ERR_INVALID_ARG;
    if (k < 0 || k > kMaxTopK) return LVQ_ERR_INVALID_ARG;
    if (nq == 0) return LVQ_OK;
    if (!q_dev || !offsets_dev || (total > 0 && !ids_dev && !segmented)) return LVQ_ERR_INVALID_ARG;
    if (k == 0 && !dist_dev) return LVQ_ERR_INVALID_ARG;
    if (k > 0 && (!topk_ids_dev || !topk_dist_dev)) return LVQ_ERR_INVALID_ARG;
    if (ix->cfg.capacity == 0) return LVQ_ERR_INVALID_ARG;
    if (level == LVQ_FULL && ix->f.bits2 == 0) return LVQ_ERR_INVALID_ARG;
    const Format &f = ix->f;
    const int bits2 = level == LVQ_FULL ? f.bits2 : 0;
    const bool l2 = ix->cfg.metric == LVQ_L2;
    const bool multi = l2 && ix->n_means > 1;
    const bool masked = l2 && f.kpos != f.dim;
    const int variant = !l2 ? 0 : (masked ? (multi ? 4 : 3) : (multi ? 2 : 1));
    auto lookup = f.bits1 == 4 ? cand_kernel_b4 : cand_kernel_b8;
    int shape = force_shape >= 0 ? force_shape : ix->cand_shape[level == LVQ_FULL][k > 0];
    int idle_slots = 0;
    // entries per list (one whose entries are not counted on the host is taken
    // as its means' share of the store)
    const double avg = total == INT64_MAX ? (double)ix->list_len * list_nmeans / ix->n_means : (double)total / nq;
    if (!shape_fits(f, lookup, bits2, variant, shape)) {
        if (force_shape >= 0) return LVQ_ERR_UNSUPPORTED;
        shape = default_shape(f, lookup, bits2, variant, (double)nq / ix->n_cu, avg, &idle_slots);
    }
    void *kern = shape >= 0 ? lookup(bits2, variant, shape) : nullptr;
    if (!kern) return LVQ_ERR_UNSUPPORTED;
    const bool sub = multi && list_means != nullptr;
    if (list_means && (list_nmeans < 1 || list_nmeans > ix->n_means)) return LVQ_ERR_INVALID_ARG;
    const int nseg = segmented ? list_nmeans : 0;
    const int ntab = multi ? (sub ? list_nmeans : ix->n_means) : 1;
    // top-k key buffer per wave: about 2k + one block of candidates (a block
    // holds at most 32 per wave), at least 64 and at most 2048 entries,
    // halved while the launch does not fit the workgroup's LDS
    int cw = 64;
    while (cw < 2 * k + 32 && cw < 2048) cw *= 2;
    size_t lds = cand_lds_bytes(f.kpos, ntab, masked, l2 ? 0 : ix->n_means, k, cw, sub, nseg);
    while (lds > ix->lds_max && cw / 2 >= k + 32) {
        cw /= 2;
        lds = cand_lds_bytes(f.kpos, ntab, masked, l2 ? 0 : ix->n_means, k, cw, sub, nseg);
    }
    if (lds > ix->lds_max) return LVQ_ERR_UNSUPPORTED;
    // several means: a second set of tables keeps the means in LDS if it fits
    int mu_lds = 0;
    if (multi && !sub) {
        const size_t with = cand_lds_bytes(f.kpos, 2 * ntab, masked, 0, k, cw, false, nseg);
        if (with <= ix->lds_max) {
            mu_lds = 1;
            lds = with;
        }
    }

    int rc = order_after_updates(ix, s);
    if (rc) return rc;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, lds) != hipSuccess || per_cu < 1) per_cu = 1;
    const int64_t slots = (int64_t)ix->n_cu * per_cu;
    // The kernel prepares each list's query itself, which saves a launch; for
    // inner products not where many means make that long (a wave sums four of
    // sixteen), nor where workgroups take several lists and would each wait
    // for those sums between them (10^4 x 1,000 pairs: 2,129 us, prepared before
    // 2,049 us).
    bool prep = !l2 && (list_means ? list_nmeans : ix->n_means) > 16;
    // A batch that leaves workgroups idle has its lists split: parts of at
    // least one block of candidates, and more where a part builds many query
    // tables.  One list of 256 at 4x8 d = 768: 31 us whole, 20 us in
    // eight parts, merge included; 5,000 entries 323 and 26 us.
    const int ppb = 4 * (64 / tile_shape(shape).g);
    const TileShape ts = tile_shape(shape);
    const bool quads = (ts.pipe & 16) && ts.ch == 8;   // the four-lane shapes of short rows
    int parts = (int)std::min<double>((double)(slots / nq), avg / (ppb * (1.0 + ntab * f.kpos / 4096)));
    // The query buffers are sized whatever this call's route is, so that a later
    // captured call of as many queries finds room (one that does not need them
    // goes on without).  The keys of split lists follow the prepared queries, or
    // take their place; the buffer grows for them only where nothing limits it
    // (no budget, no capture, past or present), and the lists are split into as
    // many parts as there is room for.
    const size_t qk_bytes = sizeof(float) * (size_t)nq * f.kpos, keys_at = prep ? (qk_bytes + 255) & ~(size_t)255 : 0;
    const size_t per_part = sizeof(uint64_t) * (size_t)nq * k;
    Workspace *ws = fixed ? nullptr : &workspace(ix, s);
    const size_t want = keys_at + (k > 0 && parts > 1 ? parts * per_part : 0);
    if (ws && want > keys_at && ws->qk.bytes < want && !ix->capturing && !ws->qk.pinned && ix->cfg.mem_budget_bytes <= 0) {
        size_t grow = 65536;   // (doubled, so that it seldom grows: that waits for the device)
        while (grow < std::max(want, scan_table_bytes(ix, nq, 16))) grow *= 2;
        if (dev_alloc(ix, ws->qk, grow) != LVQ_OK) (void)hipGetLastError();
    }
    if (ws && (rc = size_queries(ix, *ws, nq))) {
        if (prep) return rc;
        (void)hipGetLastError();
    }
    if (k > 0 && parts > 1) {
        const size_t room = fixed ? (prep ? 0 : fixed->bytes) : ws->qk.bytes;
        parts = (int)std::min<size_t>(parts, room > keys_at ? (room - keys_at) / per_part : 0);
    }
    parts = std::max(1, parts);
    // Every item resident at once: no order, no counter; nor with the four-lane
    // shapes of short rows up to 1.5 times as many, where the two launches cost
    // more than the order gives (1,500 lists at 4x8 d = 96, both levels, L2, ordered
    // / as they come: of 20 entries 39 / 17 us, of 400 61 / 43, of 30 to 2,000 61 /
    // 66; with longer rows 4x8 d = 768 L2, of 30 to 2,000 163 / 231).
    const bool queued = nq * parts > (quads ? std::max(slots, (int64_t)kShortRowsPerUnit * ix->n_cu) : slots);
    if (queued && !l2 && !prep) {
        prep = true;   // (of whole lists: no keys behind the queries)
        if (ws && (rc = size_queries(ix, *ws, nq))) return rc;
    }
    DistScratch sc;
    uint64_t *part_keys = nullptr;
    if (fixed) {
        sc = *fixed;
        if (parts > 1 && k > 0) part_keys = reinterpret_cast<uint64_t *>(sc.all);
        if (prep && (rc = prep_into(ix, q_dev, nq, sc.qk, sc.qsum, sc.cm, s))) return rc;
    } else {
        Workspace &w = *ws;
        if (prep && (rc = prep_queries(ix, w, q_dev, nq, s))) return rc;
        if ((rc = dev_alloc(ix, w.order, sizeof(int32_t) * (size_t)nq))) return rc;
        if ((rc = dev_alloc(ix, w.queue, 64))) return rc;
        if (parts > 1 && k > 0) part_keys = reinterpret_cast<uint64_t *>(static_cast<char *>(w.qk.p) + keys_at);
        sc = {P<float>(w.qk), P<float>(w.qsum), P<float>(w.cm), P<int32_t>(w.order), P<int32_t>(w.queue), nullptr, 0};
    }

    CandArgs a;
    a.rows = P<uint8_t>(ix->rows);
    a.resid = P<uint8_t>(ix->resid);
    a.row_bytes = f.row_bytes;
    a.resid_bytes = f.resid_bytes;
    a.kchunks = f.kchunks;
    a.kpos = f.kpos;
    a.capacity = ix->cfg.capacity;
    a.q = prep ? nullptr : q_dev;
    a.kdim = P<int32_t>(ix->kdim);
    a.means = P<float>(ix->means);
    a.dim = f.dim;
    a.qk = sc.qk;
    a.qsum = sc.qsum;
    a.cm = sc.cm;
    a.muk = P<float>(ix->muk);
    a.kmask = P<float>(ix->kmask);
    a.n_means = ix->n_means;
    a.offsets = offsets_dev;
    a.ids = ids_dev;
    a.nq = nq;
    a.total = total;
    a.dist = dist_dev;
    a.k = k;
    a.topk_ids = topk_ids_dev;
    a.topk_dist = topk_dist_dev;
    a.epoch = epoch;
    a.err = P<uint32_t>(ix->err);
    a.neg_empty = neg_empty ? 1 : 0;
    a.cw = cw;
    a.mu_lds = mu_lds;
    a.idle_slots = idle_slots;
    a.list_means = (sub || segmented) ? list_means : nullptr;
    a.list_nmeans = (sub || segmented) ? list_nmeans : 0;
    a.seg_offs = segmented ? seg_offs : nullptr;
    a.seg_members = segmented ? seg_members : nullptr;
    a.order = queued ? sc.order : nullptr;
    a.queue = queued ? sc.queue : nullptr;
    a.parts = parts;
    a.part_keys = part_keys;
    if (queued) {
        // persistent launch: lists longest-first from a device work counter
        LVQ_HIP(launch_list_order(offsets_dev, nq, sc.order, sc.queue, s));
    }
    // (less than two lists per workgroup: equal rounds of them, with at least three
    // workgroups per unit to hide each other's waits: 1,500 lists of 20 at 8-bit d =
    // 512 IP, room for 1,024: 49 us, 768 workgroups 46; 1,100 of 30 to 2,000 117
    // and 114; not the probe's, which make their tables between lists: 2,000 queries,
    // two of 256 means over 10^6 rows 1,111 us with 1,000 workgroups, 1,006 with all)
    const int64_t grid = !queued         ? nq * parts
                         : nq < 2 * slots && !segmented ? std::min(slots, std::max((nq + 1) / 2, 3 * (int64_t)ix->n_cu))
                                                        : slots;
    ix->last_wg = grid;
    ix->last_lists = nq;
    ix->last_parts = 0;
    if (!fixed && (rc = timing_begin(ix, s))) return rc;
    hipLaunchKernelGGL(reinterpret_cast<void (*)(CandArgs)>(kern), dim3((unsigned)grid), dim3(256), lds, s, a);
    LVQ_HIP(hipGetLastError());
    if (!fixed && (rc = timing_end(ix, s))) return rc;
    if (parts > 1 && k > 0)
        LVQ_HIP(launch_topk_merge(part_keys, nq, parts, k, ix->cfg.metric, topk_ids_dev, topk_dist_dev, s));
    return LVQ_OK;
}

extern "C" {

int lvq_distances(lvq_index *ix, const float *q_dev, int64_t nq, const int64_t *offsets_dev, const int32_t *ids_dev,
                  int64_t total, int32_t level, float *dist_dev, int32_t k, int32_t *topk_ids_dev,
                  float *topk_dist_dev, void *stream)
{
    if (!ix) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    int rc = begin_call(ix, (hipStream_t)stream);
    if (rc) return rc;
    rc = host_distances(ix, q_dev, nq, offsets_dev, ids_dev, total, level, dist_dev, k, topk_ids_dev,
                        topk_dist_dev, (hipStream_t)stream, -1, ix->epoch, false);
    if (rc == LVQ_OK) rc = note_query(ix, (hipStream_t)stream, ix->epoch);
    if (rc == LVQ_OK) pin_after_capture(ix, (hipStream_t)stream, false);
    ix->capturing = false;
    return rc;
}

int lvq_set_tile(lvq_index *ix, int32_t level, int32_t topk, int32_t shape)
{
    if (!ix || (level != LVQ_PRIMARY && level != LVQ_FULL) || shape < -1 || shape >= num_tile_shapes())
        return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    ix->cand_shape[level == LVQ_FULL][topk != 0] = shape;
    return LVQ_OK;
}

int lvq_num_tile_shapes(void) { return num_tile_shapes(); }

int lvq_tile_shape(int32_t shape, int32_t *lanes, int32_t *piece_bytes, int32_t *pieces, int32_t *pipe)
{
    if (shape < 0 || shape >= num_tile_shapes()) return LVQ_ERR_INVALID_ARG;
    const TileShape t = tile_shape(shape);
    if (lanes) *lanes = t.g;
    if (piece_bytes) *piece_bytes = t.ch;
    if (pieces) *pieces = t.nch;
    if (pipe) *pipe = t.pipe;
    return LVQ_OK;
}

int lvq_autotune(lvq_index *ix, const float *q_dev, int64_t nq, const int64_t *offsets_dev, const int32_t *ids_dev,
                 int64_t total, int32_t level, int32_t k, int32_t *shape_out, float *ms_out, void *stream)
{
    if (!ix || nq < 1 || total < 0 || k < 0 || k > kMaxTopK) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    hipStream_t s = (hipStream_t)stream;
    ix->capturing = false;
    float *dist = nullptr;
    int32_t *ti = nullptr;
    float *td = nullptr;
    LVQ_HIP(hipMalloc((void **)&dist, sizeof(float) * (size_t)std::max<int64_t>(total, 1)));
    if (k > 0) {
        LVQ_HIP(hipMalloc((void **)&ti, sizeof(int32_t) * (size_t)nq * k));
        LVQ_HIP(hipMalloc((void **)&td, sizeof(float) * (size_t)nq * k));
    }
    hipEvent_t a, b;
    LVQ_HIP(hipEventCreate(&a));
    LVQ_HIP(hipEventCreate(&b));
    int best = -1;
    float best_ms = 0.0f;
    int rc = LVQ_OK;
    for (int i = 0; i < num_tile_shapes() && rc == LVQ_OK; ++i) {
        if (host_distances(ix, q_dev, nq, offsets_dev, ids_dev, total, level, dist, k, ti, td, s, i, ix->epoch,
                           false) != LVQ_OK)
            continue;   // shape not available for this format
        float ms = 0.0f;
        if (hipEventRecord(a, s) != hipSuccess) { rc = LVQ_ERR_DEVICE; break; }
        for (int r = 0; r < 3 && rc == LVQ_OK; ++r)
            rc = host_distances(ix, q_dev, nq, offsets_dev, ids_dev, total, level, dist, k, ti, td, s, i, ix->epoch,
                                false);
        if (hipEventRecord(b, s) != hipSuccess || hipEventSynchronize(b) != hipSuccess ||
            hipEventElapsedTime(&ms, a, b) != hipSuccess) {
            rc = LVQ_ERR_DEVICE;
            break;
        }
        if (best < 0 || ms < best_ms) {
            best = i;
            best_ms = ms;
        }
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    (void)hipStreamSynchronize(s);
    (void)hipFree(dist);
    if (ti) (void)hipFree(ti);
    if (td) (void)hipFree(td);
    if (rc) return rc;
    if (best < 0) return LVQ_ERR_UNSUPPORTED;
    ix->cand_shape[level == LVQ_FULL][k > 0] = best;
    if (shape_out) *shape_out = best;
    if (ms_out) *ms_out = best_ms / 3.0f;
    return LVQ_OK;
}

}  // extern "C"

static int topk_mfma(lvq_index *ix, const void *q_dev, int32_t prec, int64_t nq, int32_t k, int32_t level,
                     int32_t *ids_dev, float *dist_dev, hipStream_t s, uint32_t epoch);

constexpr int64_t kPairsMaxQueries = 8;
constexpr int kScanFewQueries = 4;   // of the small tiles

// The FP32 vector scan of a format: the kernel that processes a whole row in
// one round with the least padding, and whether it takes nq queries at this k.
struct ScanPlan {
    void *kern = nullptr;
    int tq = 0;           // queries per tile
    int pair_chunk = 0;   // positions of a matrix-core chunk, in that order of sums
    size_t lds = 0;
    int64_t slots = 0;    // workgroups resident at once
};

static void scan_slots(const lvq_index *ix, ScanPlan *p)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, p->kern, 256, p->lds) != hipSuccess || per_cu < 1)
        per_cu = 1;
    p->slots = (int64_t)ix->n_cu * per_cu;
}

// Few FP32 queries, inner product, of a format the wide matrix-core kernel
// takes: the vector scan in that kernel's order of sums (the same values).
// The matrix cores work on 32 queries at a time, whatever the batch: over 10^6
// 4x8 rows of d = 768, both levels, 687 us for one query, 713 for four, 841 for
// eight; this 311, 382 and 610 us (its vector work grows with every query: past
// eight, a second tile reads the rows again).
static bool scan_plan_pairs(const lvq_index *ix, int64_t nq, int32_t k, int32_t level, ScanPlan *p)
{
    const Format &f = ix->f;
    const int bits2 = level == LVQ_FULL ? f.bits2 : 0;
    if (nq > kPairsMaxQueries || ix->cfg.metric != LVQ_IP) return false;
    const bool few = 2 * nq <= scan_tile_queries(1, 16, f.bits1, false);
    p->kern = (f.bits1 == 4 ? scan_pairs_kernel_b4 : scan_pairs_kernel_b8)(bits2, few);
    p->tq = scan_tile_queries(1, 16, f.bits1, few);
    p->lds = scan_lds_bytes(p->tq, ix->n_means, k, 1, f.bits1, bits2);
    p->pair_chunk = f.bits1 == 4 ? 64 : 32;
    if (!p->kern || p->lds > ix->lds_max) {
        p->kern = nullptr;
        return false;
    }
    scan_slots(ix, p);
    return true;
}

static bool scan_plan(const lvq_index *ix, int64_t nq, int32_t k, int32_t level, ScanPlan *p, bool few_only = false)
{
    const Format &f = ix->f;
    const bool l2 = ix->cfg.metric == LVQ_L2;
    const int variant = !l2 ? 0 : (f.kpos != f.dim ? 2 : 1);
    const int bits2 = level == LVQ_FULL ? f.bits2 : 0;
    const int nm = l2 ? 0 : ix->n_means;
    auto lookup = f.bits1 == 4 ? scan_kernel_b4 : scan_kernel_b8;
    int shape = -1;
    for (int i = 0; i < num_tile_shapes(); ++i) {
        if (!lookup(bits2, variant, i, false)) continue;
        TileShape t = tile_shape(i);
        if (t.g * t.ch * t.nch < f.kchunks * 16) continue;
        if (shape < 0) { shape = i; continue; }
        TileShape b = tile_shape(shape);
        if (t.g * t.ch * t.nch < b.g * b.ch * b.nch) shape = i;
    }
    if (shape < 0) return false;
    // The sizes taken are those of a scan that held 16 queries of kpos values, k +
    // 512 / g keys of each, c_m and 4 k keys of scratch in one workgroup's LDS:
    // larger ones stay refused.  (The kernel itself keeps no queries there and needs
    // less, which is tested below.)
    const size_t need = (size_t)16 * f.kpos * 4 + (((size_t)16 * (((nm + 1) & ~1) + 2) * 4 + 15) & ~(size_t)15) + 256 +
                        ((size_t)16 * (k + 512 / tile_shape(shape).g) + 4 * (size_t)k) * 8;
    if (need > ix->lds_max) return false;
    // few queries take tiles of four (over 300,000 rows of d = 96, 256 workgroups:
    // one query 55 us, eight 102 us, a tile of sixteen 191 us), and so do key
    // lists too long for a full tile's LDS
    const int g = tile_shape(shape).g, ch = tile_shape(shape).ch;
    const int full = scan_tile_queries(g, ch, f.bits1, false);
    const bool few = few_only || 2 * nq <= full || scan_lds_bytes(full, nm, k, g, f.bits1, bits2) > ix->lds_max;
    p->tq = scan_tile_queries(g, ch, f.bits1, few);
    p->lds = scan_lds_bytes(p->tq, nm, k, g, f.bits1, bits2);
    if (p->lds > ix->lds_max) return false;
    p->kern = lookup(bits2, variant, shape, few);
    p->pair_chunk = 0;
    scan_slots(ix, p);
    return true;
}

// Row parts of the FP32 vector scan: the count with the least modelled time, in
// rows of one workgroup.  A compute unit runs its c = workgroups / units at
// once up to the resident ones; they share its vector ALUs, so the time is c
// times one's rounds of 256 rows, more where too few are resident to hide each
// other's loads (600 queries over 300,000 rows of d = 96: one per unit 1,908 us, two
// 1,136, three 970).  A part costs 2.3 rounds of d = 96 to begin with (its
// first ones append nearly every row), every part its k keys, sorted and merged, whose
// time does not grow with the row (two fifths where lists are folded whole, k >
// 64), and parts of more than one round the atomics that share the bounds, one
// address for all parts of a query: 250,000 rows of d = 96, L2, 16 queries, top-1, 156
// us with 128 parts, 170 with 256, 272 with 512, 392 with 768, but 197 with 977 of
// one round; eight queries at d = 128 118, 113, 177, 217 and 101.  Top-10 of three
// queries: 70 us with 256, 105 with 512, 84 with 977; 30,000 rows, 300 queries, 130
// with 40, 174 with 12.  On 798 cases (10^4 to 5x10^5 rows of d = 96 to 768, 1 to
// 700 queries, k = 1 to 100) the counts taken are 1% over the best one measured on
// average and 8% in one of 20.  At most 20,480 keys per query, a bound on the scratch
// (the merge takes any number).
//
// Under a memory budget no more than four workgroups of sixteen queries per
// unit and 1,024 rows per part: the keys are charged to the budget, and the
// counts above can ask for 16 times as many (nq x parts x k keys).
static int64_t scan_parts_fp32(const lvq_index *ix, const ScanPlan &pl, int64_t nq, int32_t k, int64_t n_rows)
{
    const double keys = (k <= 64 ? 0.77 : 0.31) * k;   // to merge, per part
    const double sorts = 0.065 * keys * std::min<int64_t>(nq, pl.tq);
    const double bounds = 7.3 * std::min<int64_t>(nq, 20);
    const int64_t qtiles = (nq + pl.tq - 1) / pl.tq, occ = std::max<int64_t>(1, pl.slots / ix->n_cu);
    int64_t most = std::max<int64_t>(1, std::min<int64_t>({(n_rows + 255) / 256, (int64_t)(ix->lds_max / 8 - k) / k,
                                                           2 * pl.slots / qtiles + 1}));
    if (ix->cfg.mem_budget_bytes > 0) {
        const int64_t tiles16 = (nq + 15) / 16;
        most = std::min(most, std::max<int64_t>(1, std::min<int64_t>((4 * (int64_t)ix->n_cu + tiles16 - 1) / tiles16,
                                                                     n_rows / 1024)));
    }
    const double unit = ix->f.kpos / 96.0 * (1.0 + 0.7 * pl.tq);   // a row
    const double begin = 2.3 * std::min(1.0, 96.0 / ix->f.kpos);
    const double two = pl.tq == kScanFewQueries && ix->f.kchunks <= 6 ? 1.38 : 1.18;
    auto shared = [two](int64_t c) { return (double)c * (c == 1 ? 1.8 : c == 2 ? two : 1.0); };
    int64_t parts = 1;
    double best = 0.0;
    // (the fewest parts of every number of rounds: more cost more)
    for (int64_t p = most, next; p >= 1; p = next) {
        const int64_t n = ((n_rows + p - 1) / p + 255) / 256;
        if (n > 0) p = std::min(p, (n_rows + 256 * n - 1) / (256 * n));
        next = p - 1;
        const int64_t c = (qtiles * p + ix->n_cu - 1) / ix->n_cu;
        const double first = (double)std::min<int64_t>(n, 3) / 3.0;
        const double cost = unit * ((double)(c / occ) * shared(occ) + shared(c % occ)) * 256.0 * ((double)n + begin) +
                            (double)p * (keys + sorts * first + (n > 1 ? bounds : 0.0));
        if (p == most || best == 0.0 || cost <= best) {
            best = cost;
            parts = p;
        }
    }
    return parts;
}

// Row parts of the MFMA scan (one resident workgroup per compute unit).
// Time model: whole rounds of workgroups over the compute units, each
// workgroup streaming n_rows / parts rows, plus a per-part overhead (a part
// starts with a loose top-k bound and adds k keys to the merge) of 2% of a
// part's scan per extra part.  Parts keep at least 64 row rounds,
// and a query's keys at most 20,480 (lds_max / 8): a bound on the scratch, as the
// merge takes any number.
static int64_t scan_parts_mfma(const lvq_index *ix, int64_t qtiles, int32_t k, int64_t n_rows)
{
    const int64_t max_parts = std::max<int64_t>(
        1, std::min<int64_t>(n_rows / (64 * 128), (int64_t)(ix->lds_max / 8 - k) / k));
    int64_t parts = 1;
    double best = 0.0;
    for (int64_t p = 1; p <= max_parts; ++p) {
        const int64_t rounds = (qtiles * p + ix->n_cu - 1) / ix->n_cu;
        const double cost = (double)rounds / (double)p * (1.0 + 0.02 * (double)p);
        if (p == 1 || cost < best) {
            best = cost;
            parts = p;
        }
    }
    return parts;
}

// Sample pass of the wide MFMA scan: `parts` stretches of `rows` rows, spread
// over the list, are scored first and only each wave's largest score per query
// is kept; the k-th largest of these 8 * parts maxima is a bound that k rows
// reach, so the scan proper starts with it instead of with none.
//
// A scan without it keeps every score of a part's first round and about
// k ln(rows) more per part and query, at the price of sorts and of LDS atomics;
// with it N k / S scores pass for a sample of S rows, so S goes with
// sqrt(N k / price of a row).  10^6 x 768 4x8 (16 means) at both levels, k = 10,
// 300 queries: 1658 us without, 1398 / 1331 / 1317 / 1271 / 1322 with S = 4k / 8k / 16k /
// 33k / 66k; 64 queries 1843 and 425; 10^6 x 512 first level: 16 queries 587 and 230,
// 1000 queries 1686 and 1190; 4096 x 2x10^6, k = 100: 10,448 and 9035; 10^6 x 96, 300
// queries 1123 and 245; FP32, 10^6 x 512, 100 queries 1915 and 1170.  The maxima of
// fewer than 4 k groups miss much of the top k (3x10^5 x 768 both levels, k = 500: 512
// groups 3388 us, 2048 1623, none 4104).
struct ScanSample {
    int64_t parts, rows;   // parts = 0: no sample
};

static ScanSample scan_sample(const lvq_index *ix, int64_t qtiles, int32_t k, int64_t n_rows, int bits2, int32_t prec)
{
    const Format &f = ix->f;
    const int64_t round = mfma_wide_round(f.bits1, bits2, f.kpos, prec);
    const bool f32 = prec == LVQ_FP32;
    const double row_cost = f32 ? 8.0 : 1.0;
    // (a part's own bound catches up with larger samples: 10^4 queries x 5x10^6 x
    // 512, k = 100: 51.8 ms with 65k rows, 52.5 with 200k and with none)
    const double want = std::min(65536.0, std::sqrt(80.0 * 512.0 / (f.kpos * row_cost) * (double)n_rows * k));
    const int64_t most = n_rows / (2 * round);   // at most half the rows
    const int64_t slots = std::max<int64_t>(8, ix->n_cu / 8 * 8);
    // (a pass that leaves half the chip idle costs no more with larger samples)
    const int64_t rounds =
        std::min<int64_t>(most, std::max<int64_t>((int64_t)(want / round) + 1, slots / (2 * qtiles)));
    const int64_t least = std::min<int64_t>({most, 256, std::max<int64_t>(2, (k + 1) / 2)});
    // a tile's queries are staged once: up to four rounds each where the tiles
    // fill the chip anyway
    int64_t per = 1;
    while (per < 4 && rounds >= 2 * per * least && qtiles * ((rounds + per - 1) / per) > 2 * slots) per *= 2;
    while (per < 8 && (rounds + per - 1) / per > 256) per *= 2;
    int64_t parts = std::min<int64_t>(256, std::max(least, (rounds + per - 1) / per));
    // whole waves of workgroups, where there is more than one
    if (qtiles * parts > slots && slots / qtiles >= least) {
        const int64_t waves = std::max<int64_t>(1, (qtiles * parts + slots / 2) / slots);
        parts = std::min<int64_t>(256, std::max(least, waves * slots / qtiles));
    }
    if (parts < 1 || 8 * parts < k || parts * per * round > n_rows) return {0, 0};
    return {parts, per * round};
}

// Row parts and persistent grid of the wide MFMA scan (one workgroup per
// compute unit, a multiple of 8 for the XCD-aware tile walk).  Time model:
// each workgroup runs ceil(tiles per XCD / workgroups per XCD) tiles of
// R = n_rows / parts rows, plus a per-tile cost in 16-bit row equivalents: 2200
// for staging the queries and the final merge (10^5 x 512, 1000 queries: 8 x 32
// tiles 199 us, 8 x 64 251; 10^6 x 96, 300 queries: 3 x 64 tiles 271, 3 x 256 278) and
// 16 for each key that passes: R k / S per query while R is less than the S sampled rows,
// k (1 + ln(R / S)) beyond.  Every tile after a workgroup's first adds 2.5%: the
// workgroups of an XCD then no longer read the same rows at the same time (10^4
// queries x 5x10^6 x 512: 79 x 3 tiles 51.8 ms, x 6 52.2, x 16 53.2, x 29 58.6; 4096 x
// 2x10^6: 32 x 8 8.98 ms, x 16 9.06, x 32 9.51; FP32 rows, an eighth of it).  Without a sample a part's bound starts loose: a 32 x 32
// block of scores holds a key beating the running k-th best of t rows with
// probability about min(1, 1024 k / t), so the blocks that append add about
// 512 k (1 + ln(R / 1024 k)) rows' worth, and 10,240 for the rest.
// An FP32 row costs about 8 16-bit ones (a sixteenth of the matrix-core
// rate, half the queries per tile).  Parts keep at least 512 rows (4096 without a
// sample), and a query's keys at most 20,480, as above.
static int64_t scan_parts_wide(const lvq_index *ix, int64_t qtiles, int32_t k, int64_t n_rows, int32_t prec,
                               const ScanSample &sm, int64_t *grid)
{
    const int64_t slots = std::max<int64_t>(8, ix->n_cu / 8 * 8);
    const int64_t max_parts = std::max<int64_t>(
        1, std::min<int64_t>(n_rows / (sm.parts ? 512 : 4096), (int64_t)(ix->lds_max / 8 - k) / k));
    const double sampled = (double)std::max<int64_t>(1, sm.parts * sm.rows);
    const double warm = 1024.0 * k, row_cost = prec == LVQ_FP32 ? 8.0 : 1.0;
    const double least = (sm.parts ? 2200.0 : 10240.0) / row_cost;   // of any tile
    auto later = [&](int64_t iters) { return sm.parts ? 1.0 + 0.025 / row_cost * (double)(iters - 1) : 1.0; };
    int64_t parts = 1;
    double best = 0.0;
    // (the most parts of every number of tiles per workgroup: with more, shorter
    // tiles the time falls as long as that number stays)
    for (int64_t i = (qtiles + slots - 1) / slots;; ++i) {
        const int64_t most = std::min(max_parts, i * slots / qtiles);
        const int64_t n = (n_rows + most - 1) / most;                      // rows per part,
        const int64_t p = n > 0 ? (n_rows + n - 1) / n : 1;                // and the fewest such parts
        const int64_t iters = (qtiles * p + slots - 1) / slots;
        const double rows = (double)n;
        const double extra = sm.parts ? 2200.0 + 16.0 * k * (rows < sampled ? rows / sampled : 1.0 + std::log(rows / sampled))
                                      : 10240.0 + 0.5 * warm * (1.0 + std::log(std::max(1.0, rows / warm)));
        const double cost = (double)iters * (rows + extra / row_cost) * later(iters);
        if (best == 0.0 || cost < best) {
            best = cost;
            parts = p;
        }
        if (most == max_parts || (double)(i + 1) * least * later(i + 1) >= best) break;
    }
    *grid = std::min<int64_t>(slots, (qtiles * parts + 7) / 8 * 8);
    return parts;
}

int lvq::host_topk(lvq_index *ix, const void *q_dev, int32_t prec, int64_t nq, int32_t k, int32_t level,
                   int32_t *ids_dev, float *dist_dev, hipStream_t s, uint32_t epoch)
{
    if (nq < 0 || nq > INT32_MAX || k < 1 || k > kMaxTopK) return LVQ_ERR_INVALID_ARG;
    if (level != LVQ_PRIMARY && level != LVQ_FULL) return LVQ_ERR_INVALID_ARG;
    if (prec != LVQ_FP32 && prec != LVQ_BF16 && prec != LVQ_FP16 && prec != LVQ_FP32_VALU)
        return LVQ_ERR_INVALID_ARG;
    if (nq == 0) return LVQ_OK;
    if (!q_dev || !ids_dev || !dist_dev) return LVQ_ERR_INVALID_ARG;
    if (level == LVQ_FULL && ix->f.bits2 == 0) return LVQ_ERR_INVALID_ARG;
    const Format &f = ix->f;
    if (prec == LVQ_BF16 || prec == LVQ_FP16)
        return topk_mfma(ix, q_dev, prec, nq, k, level, ids_dev, dist_dev, s, epoch);
    const bool l2 = ix->cfg.metric == LVQ_L2;
    ScanPlan pl;
    // the inner product runs on the FP32 matrix cores when the format, k and
    // the means' c_m table allow
    // (LVQ_FP32_VALU: the vector path whatever the format)
    if (prec == LVQ_FP32 && !l2 &&
        mfma_wide_query_block(f.bits1, level == LVQ_FULL ? f.bits2 : 0, f.kpos, LVQ_FP32, k, ix->n_means,
                              ix->lds_max)) {
        if (!scan_plan_pairs(ix, nq, k, level, &pl))
            return topk_mfma(ix, q_dev, LVQ_FP32, nq, k, level, ids_dev, dist_dev, s, epoch);
    }
    if (l2 && ix->n_means > 1) return LVQ_ERR_UNSUPPORTED;
    if (!pl.kern && !scan_plan(ix, nq, k, level, &pl)) return LVQ_ERR_UNSUPPORTED;

    int rc = order_after_updates(ix, s);
    if (rc) return rc;
    Workspace &w = workspace(ix, s);
    // Where the workspace has no room and cannot grow (a capture, a budget): the
    // bounds behind the table, the smallest tiles, or for few inner products the
    // matrix cores; and the row parts whose keys there is room for.
    const bool own_bounds = dev_alloc(ix, w.gthr, sizeof(uint32_t) * (size_t)nq) == LVQ_OK;
    if (!own_bounds) (void)hipGetLastError();
    auto table = [&]() {
        return dev_alloc(ix, w.qk, scan_table_bytes(ix, nq, pl.tq) - (own_bounds ? sizeof(uint32_t) * (size_t)nq : 0));
    };
    if ((rc = table())) {
        (void)hipGetLastError();
        if (pl.pair_chunk) return topk_mfma(ix, q_dev, LVQ_FP32, nq, k, level, ids_dev, dist_dev, s, epoch);
        if (!scan_plan(ix, nq, k, level, &pl, true)) return rc;
        if ((rc = table())) return rc;
    }
    const int tq = pl.tq;
    const int64_t qtiles = (nq + tq - 1) / tq;
    const int64_t n_rows = ix->list_len;
    int64_t parts = scan_parts_fp32(ix, pl, nq, k, n_rows);
    if (!l2) {   // (Euclidean scans use neither)
        if ((rc = dev_alloc(ix, w.qsum, sizeof(float) * (size_t)nq))) return rc;
        if ((rc = dev_alloc(ix, w.cm, sizeof(float) * (size_t)nq * ix->n_means))) return rc;
    }
    const size_t per_part = sizeof(uint64_t) * (size_t)nq * k;
    while ((rc = dev_alloc(ix, w.part, per_part * parts))) {
        if (parts == 1) return rc;
        (void)hipGetLastError();
        // what the buffer has now, or half as many
        parts = std::max<int64_t>(1, std::max<int64_t>(parts / 2, std::min<int64_t>(parts - 1, w.part.bytes / per_part)));
    }
    const int64_t rows_per_part = std::max<int64_t>(1, (n_rows + parts - 1) / parts);
    uint32_t *bounds = own_bounds ? P<uint32_t>(w.gthr)
                                  : reinterpret_cast<uint32_t *>(P<float>(w.qk) + qtiles * tq * f.kpos);
    LVQ_HIP(launch_prep_rows(prep_args(ix, (const float *)q_dev, nq, P<float>(w.qk), P<float>(w.qsum), P<float>(w.cm)),
                             P<float>(ix->muk), tq, pl.pair_chunk, bounds, s));

    ScanArgs a;
    a.rows = P<uint8_t>(ix->rows);
    a.resid = P<uint8_t>(ix->resid);
    a.row_bytes = f.row_bytes;
    a.resid_bytes = f.resid_bytes;
    a.kchunks = f.kchunks;
    a.kpos = f.kpos;
    a.list = P<int32_t>(ix->lists[ix->list_active].buf);
    a.n_rows = n_rows;
    a.qk = P<float>(w.qk);
    a.qsum = P<float>(w.qsum);
    a.cm = P<float>(w.cm);
    a.muk = P<float>(ix->muk);
    a.kmask = P<float>(ix->kmask);
    a.q16 = nullptr;
    a.n_means = ix->n_means;
    a.nq = nq;
    a.k = k;
    a.epoch = epoch;
    a.rows_per_part = rows_per_part;
    a.n_parts = (int)parts;
    a.capq = 0;
    a.gthr = bounds;
    a.part_keys = P<uint64_t>(w.part);
    a.err = P<uint32_t>(ix->err);
    a.mks = scan_sorted_keys(k);
    a.gmax = nullptr;
    a.sample_rows = 0;
    ix->last_wg = qtiles * parts;
    ix->last_lists = 0;
    ix->last_parts = (int32_t)parts;
    if ((rc = timing_begin(ix, s))) return rc;
    hipLaunchKernelGGL(reinterpret_cast<void (*)(ScanArgs)>(pl.kern), dim3((unsigned)qtiles, (unsigned)parts),
                       dim3(256), pl.lds, s, a);
    LVQ_HIP(hipGetLastError());
    if ((rc = timing_end(ix, s))) return rc;
    LVQ_HIP(launch_topk_merge(a.part_keys, nq, (int)parts, k, ix->cfg.metric, ids_dev, dist_dev, s));
    return LVQ_OK;
}

extern "C" {

int lvq_topk(lvq_index *ix, const void *q_dev, int32_t prec, int64_t nq, int32_t k, int32_t level, int32_t *ids_dev,
             float *dist_dev, void *stream)
{
    if (!ix) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    hipStream_t s = (hipStream_t)stream;
    int rc = begin_call(ix, s);
    if (rc) return rc;
    rc = host_topk(ix, q_dev, prec, nq, k, level, ids_dev, dist_dev, s, ix->epoch);
    if (rc == LVQ_OK && nq > 0) rc = note_query(ix, s, ix->epoch);
    if (rc == LVQ_OK) pin_after_capture(ix, s, true);
    ix->capturing = false;
    return rc;
}

}  // extern "C"

// Exhaustive top-k on the matrix cores: inner product; bf16 / fp16 queries
// at either level, FP32 queries on the wide kernel only.
static int topk_mfma(lvq_index *ix, const void *q_dev, int32_t prec, int64_t nq, int32_t k, int32_t level,
                     int32_t *ids_dev, float *dist_dev, hipStream_t s, uint32_t epoch)
{
    const Format &f = ix->f;
    if (ix->cfg.metric != LVQ_IP) return LVQ_ERR_UNSUPPORTED;
    const int bits2 = level == LVQ_FULL ? f.bits2 : 0;
    if (bits2 != 0 && bits2 != 8) return LVQ_ERR_UNSUPPORTED;   // both levels need 8-bit residual codes
    // the wide kernel (queries in LDS) when it takes the case; else the
    // register-resident kernel (16-bit queries only)
    const int qbw = mfma_wide_query_block(f.bits1, bits2, f.kpos, prec, k, ix->n_means, ix->lds_max);
    if (prec == LVQ_FP32 && !qbw) return LVQ_ERR_UNSUPPORTED;
    const int qb = qbw ? qbw : mfma_query_block(f.bits1, bits2, f.kpos);
    if (!qb) return LVQ_ERR_UNSUPPORTED;
    const int capq = qbw ? 0 : mfma_capq(qb, ix->n_means, k, ix->lds_max);
    if (!qbw && !capq) return LVQ_ERR_UNSUPPORTED;
    int rc = order_after_updates(ix, s);
    if (rc) return rc;
    Workspace &w = workspace(ix, s);
    const int tq = 32 * qb;
    const int64_t qtiles = (nq + tq - 1) / tq;
    if ((rc = dev_alloc(ix, w.q16, (size_t)qtiles * tq * f.kpos * (prec == LVQ_FP32 ? 4 : 2)))) return rc;
    if ((rc = dev_alloc(ix, w.qsum, sizeof(float) * (size_t)nq))) return rc;
    if ((rc = dev_alloc(ix, w.cm, sizeof(float) * (size_t)nq * ix->n_means))) return rc;
    if ((rc = dev_alloc(ix, w.gthr, sizeof(uint32_t) * (size_t)nq))) return rc;
    LVQ_HIP(launch_prep_scan(q_dev, nq, f.dim, f.kpos, f.bits1, qb, prec, P<int32_t>(ix->kdim), P<float>(ix->means),
                             ix->n_means, w.q16.p, P<float>(w.qsum), P<float>(w.cm), P<uint32_t>(w.gthr), s));
    const int64_t n_rows = ix->list_len;
    // Under a memory budget the scan is sized as without a sample, and where the
    // buffers have no room (a captured call), in fewer parts and without one.
    ScanSample sm = {0, 0};
    // One query over rows enough to fill the chip with parts of 4,096 goes without:
    // what passes its loose bounds costs less than the pass (sample / none, d = 96
    // top-10: 800,000 rows 97 / 86 us, 4x10^6 256 / 237; d = 768 both levels 2x10^6
    // 682 / 672; but 300,000 76 / 80, two queries over 10^6 103 / 106, top-200 187 / 242).
    const bool alone = nq == 1 && k <= 64 && prec != LVQ_FP32 && n_rows >= (int64_t)ix->n_cu * 3 / 4 * 4096;
    if (qbw && !alone && ix->cfg.mem_budget_bytes <= 0) sm = scan_sample(ix, qtiles, k, n_rows, bits2, prec);
    int64_t grid = 0;
    int64_t parts = qbw ? scan_parts_wide(ix, qtiles, k, n_rows, prec, sm, &grid) : scan_parts_mfma(ix, qtiles, k, n_rows);
    for (;;) {
        const size_t keys = sizeof(uint64_t) * (size_t)nq * parts * k;
        rc = dev_alloc(ix, w.part, std::max(keys, sizeof(float) * 8 * (size_t)nq * sm.parts));
        if (rc == LVQ_OK && qbw) rc = dev_alloc(ix, w.mkeys, sizeof(uint64_t) * (size_t)grid * tq * mfma_wide_cap(k));
        if (rc == LVQ_OK) break;
        if (!sm.parts && parts == 1) return rc;
        (void)hipGetLastError();
        if (sm.parts) {
            sm = {0, 0};
            if (qbw) parts = scan_parts_wide(ix, qtiles, k, n_rows, prec, sm, &grid);
        } else if (qbw) {
            parts /= 2;
            grid = std::min<int64_t>(grid, (qtiles * parts + 7) / 8 * 8);
        } else {
            return rc;
        }
    }
    const int64_t rows_per_part = std::max<int64_t>(1, (n_rows + parts - 1) / parts);
    ScanArgs a;
    a.rows = P<uint8_t>(ix->rows);
    a.resid = P<uint8_t>(ix->resid);
    a.row_bytes = f.row_bytes;
    a.resid_bytes = f.resid_bytes;
    a.kchunks = f.kchunks;
    a.kpos = f.kpos;
    a.list = P<int32_t>(ix->lists[ix->list_active].buf);
    a.n_rows = n_rows;
    a.qk = nullptr;
    a.qsum = P<float>(w.qsum);
    a.cm = P<float>(w.cm);
    a.muk = nullptr;
    a.kmask = nullptr;
    a.q16 = w.q16.p;
    a.n_means = ix->n_means;
    a.nq = nq;
    a.k = k;
    a.epoch = epoch;
    a.rows_per_part = rows_per_part;
    a.n_parts = (int)parts;
    a.capq = capq;
    a.gthr = P<uint32_t>(w.gthr);
    a.part_keys = P<uint64_t>(w.part);
    a.err = P<uint32_t>(ix->err);
    a.mkeys = qbw ? P<uint64_t>(w.mkeys) : nullptr;
    a.mcap = qbw ? mfma_wide_cap(k) : 0;
    a.mks = qbw ? mfma_wide_sorted(k) : 0;
    a.gmax = nullptr;
    a.sample_rows = 0;
    ix->last_wg = qbw ? grid : (qtiles * parts + 7) / 8 * 8;
    ix->last_lists = 0;
    ix->last_parts = (int32_t)parts;
    if ((rc = timing_begin(ix, s))) return rc;
    if (sm.parts) {
        ScanArgs b = a;
        b.gmax = P<float>(w.part);   // (the scan proper overwrites it)
        b.sample_rows = sm.rows;
        b.rows_per_part = n_rows / sm.parts;
        b.n_parts = (int)sm.parts;
        const int64_t g = std::min<int64_t>(std::max<int64_t>(8, ix->n_cu / 8 * 8), (qtiles * sm.parts + 7) / 8 * 8);
        LVQ_HIP(launch_scan_mfma_wide(b, f.bits1, bits2, prec, g, ix->lds_max, s));
        LVQ_HIP(launch_sample_bound(b.gmax, (int)sm.parts * 8, nq, k, a.gthr, s));
    }
    if (qbw)
        LVQ_HIP(launch_scan_mfma_wide(a, f.bits1, bits2, prec, grid, ix->lds_max, s));
    else
        LVQ_HIP(launch_scan_mfma(a, f.bits1, bits2, prec, s));
    if ((rc = timing_end(ix, s))) return rc;
    LVQ_HIP(launch_topk_merge(a.part_keys, nq, (int)parts, k, LVQ_IP, ids_dev, dist_dev, s));
    return LVQ_OK;
}

// Per-mean member lists of stream s's workspace, rebuilt after any update.
static int ensure_members(lvq_index *ix, Workspace &w, hipStream_t s)
{
    if (w.members_version == ix->version) return LVQ_OK;
    const int M = ix->n_means;
    const int64_t n = ix->list_len;
    int rc;
    if ((rc = dev_alloc(ix, w.members, sizeof(int32_t) * (size_t)std::max<int64_t>(n, 1)))) return rc;
    if ((rc = dev_alloc(ix, w.moffs, sizeof(int64_t) * (size_t)(kMaxMeans + 1)))) return rc;
    if ((rc = dev_alloc(ix, w.mcount, sizeof(uint64_t) * (size_t)kMaxMeans))) return rc;
    if ((rc = dev_alloc(ix, w.mcursor, sizeof(uint64_t) * (size_t)kMaxMeans))) return rc;
    if (n > 0) LVQ_HIP(launch_fill_i32(P<int32_t>(w.members), -1, n, s));
    LVQ_HIP(launch_members(n > 0 ? P<int32_t>(ix->lists[ix->list_active].buf) : nullptr, n, P<uint8_t>(ix->rows),
                           ix->f.row_bytes, M, P<unsigned long long>(w.mcount), P<unsigned long long>(w.mcursor),
                           P<int64_t>(w.moffs), P<int32_t>(w.members), s));
    w.members_version = ix->version;
    return LVQ_OK;
}

// Soft inverted index: route, build the probed means' candidate lists, and
// run the candidate kernel's fused top-k over them.
static int probe_topk(lvq_index *ix, const float *q_dev, int64_t nq, int32_t nprobe, int32_t k, int32_t level,
                      int32_t *probe_out_dev, int32_t *ids_dev, float *dist_dev, hipStream_t s)
{
    if (nq < 0 || nq > INT32_MAX || k < 1 || k > kMaxTopK) return LVQ_ERR_INVALID_ARG;
    if (level != LVQ_PRIMARY && level != LVQ_FULL) return LVQ_ERR_INVALID_ARG;
    if (level == LVQ_FULL && ix->f.bits2 == 0) return LVQ_ERR_INVALID_ARG;
    const int M = ix->n_means;
    if (nprobe < 1 || nprobe > M) return LVQ_ERR_INVALID_ARG;
    if (nq == 0) return LVQ_OK;
    if (!q_dev || !ids_dev || !dist_dev || ix->cfg.capacity == 0) return LVQ_ERR_INVALID_ARG;
    int rc = order_after_updates(ix, s);
    if (rc) return rc;
    Workspace &w = workspace(ix, s);
    if ((rc = ensure_members(ix, w, s))) return rc;
    int32_t *probe = probe_out_dev;
    if (!probe) {
        if ((rc = dev_alloc(ix, w.probe, sizeof(int32_t) * (size_t)nq * nprobe))) return rc;
        probe = P<int32_t>(w.probe);
    }
    if ((rc = dev_alloc(ix, w.qoffs, sizeof(int64_t) * (size_t)(nq + 1)))) return rc;
    LVQ_HIP(launch_route(q_dev, nq, ix->f.dim, P<float>(ix->means_t), kMaxMeans, M, nprobe, probe, s));
    LVQ_HIP(launch_probe_offsets(probe, nq, nprobe, P<int64_t>(w.moffs), P<int64_t>(w.qoffs), s));
    // the lists are the probed means' member ranges, walked in place
    return host_distances(ix, q_dev, nq, P<int64_t>(w.qoffs), nullptr, INT64_MAX, level, nullptr, k, ids_dev,
                          dist_dev, s, -1, ix->epoch, true, probe, nprobe, P<int64_t>(w.moffs),
                          P<int32_t>(w.members));
}

extern "C" {

int lvq_probe_topk(lvq_index *ix, const float *q_dev, int64_t nq, int32_t nprobe, int32_t k, int32_t level,
                   int32_t *probe_out_dev, int32_t *ids_dev, float *dist_dev, void *stream)
{
    if (!ix) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    hipStream_t s = (hipStream_t)stream;
    int rc = begin_call(ix, s);
    if (rc) return rc;
    rc = probe_topk(ix, q_dev, nq, nprobe, k, level, probe_out_dev, ids_dev, dist_dev, s);
    if (rc == LVQ_OK && nq > 0) rc = note_query(ix, s, ix->epoch);
    if (rc == LVQ_OK) pin_after_capture(ix, s, true);
    ix->capturing = false;
    return rc;
}

int lvq_graph_search(lvq_index *ix, const float *q_dev, int64_t nq, const int32_t *graph_dev, int32_t degree,
                     const int32_t *entries_dev, int32_t n_entries, int32_t window, int32_t k, int32_t *ids_dev,
                     float *dist_dev, int32_t *explored_dev, void *stream)
{
    if (!ix || nq < 0 || nq > INT32_MAX || degree < 1 || degree > 64 || n_entries < 1 || n_entries > 64 ||
        k < 1 || window < k || window > 256)
        return LVQ_ERR_INVALID_ARG;
    if (nq > 0 && (!q_dev || !graph_dev || !entries_dev || !ids_dev || !dist_dev)) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    if (ix->cfg.capacity == 0) return LVQ_ERR_INVALID_ARG;
    const Format &f = ix->f;
    if (graph_lds_bytes(f.kpos, window, degree) > ix->lds_max) return LVQ_ERR_UNSUPPORTED;
    if (nq == 0) return LVQ_OK;
    hipStream_t s = (hipStream_t)stream;
    int rc = begin_call(ix, s);
    if (rc) return rc;
    if ((rc = order_after_updates(ix, s)) == LVQ_OK) {
        Workspace &w = workspace(ix, s);
        if ((rc = prep_queries(ix, w, q_dev, nq, s)) == LVQ_OK) {
            GraphLaunch l;
            l.rows = P<uint8_t>(ix->rows);
            l.row_bytes = f.row_bytes;
            l.kchunks = f.kchunks;
            l.kpos = f.kpos;
            l.bits1 = f.bits1;
            l.metric = ix->cfg.metric;
            l.capacity = ix->cfg.capacity;
            l.qk = P<float>(w.qk);
            l.qsum = P<float>(w.qsum);
            l.cm = P<float>(w.cm);
            l.muk = P<float>(ix->muk);
            l.kmask = P<float>(ix->kmask);
            l.n_means = ix->n_means;
            l.nq = nq;
            l.graph = graph_dev;
            l.degree = degree;
            l.entries = entries_dev;
            l.n_entries = n_entries;
            l.window = window;
            l.k = k;
            l.epoch = ix->epoch;
            l.ids = ids_dev;
            l.dist = dist_dev;
            l.explored = explored_dev;
            l.err = P<uint32_t>(ix->err);
            if ((rc = timing_begin(ix, s)) == LVQ_OK) {
                hipError_t e = launch_graph_search(l, s);
                rc = e == hipSuccess ? timing_end(ix, s) : map_hip(e);
            }
        }
    }
    if (rc == LVQ_OK) rc = note_query(ix, s, ix->epoch);
    if (rc == LVQ_OK) pin_after_capture(ix, s, false);
    ix->capturing = false;
    return rc;
}

int lvq_retire_means(lvq_index *ix, const int32_t *ids_host, int32_t n, void *stream)
{
    if (!ix || n < 0 || (n > 0 && !ids_host)) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    hipStream_t s = (hipStream_t)stream;
    std::vector<uint8_t> next = ix->retired;
    for (int32_t i = 0; i < n; ++i) {
        if (ids_host[i] < 0 || ids_host[i] >= ix->n_means) return LVQ_ERR_INVALID_ARG;
        next[ids_host[i]] = 1;
    }
    int active = 0;
    for (int m = 0; m < ix->n_means; ++m) active += !next[m];
    if (active == 0) return LVQ_ERR_INVALID_ARG;
    int rc = begin_call(ix, s);
    if (rc) return rc;
    if (ix->capturing) {
        ix->capturing = false;
        return LVQ_ERR_UNSUPPORTED;
    }
    if ((rc = order_after_updates(ix, s))) return rc;
    ix->retired = next;
    std::vector<uint8_t> act(kMaxMeans);
    for (int m = 0; m < kMaxMeans; ++m) act[m] = !ix->retired[m];
    LVQ_HIP(hipMemcpyAsync(ix->mean_active.p, act.data(), kMaxMeans, hipMemcpyHostToDevice, s));
    LVQ_HIP(hipStreamSynchronize(s));   // the host flags must outlive the copy
    return note_update(ix, s);
}

int lvq_add_means(lvq_index *ix, const float *means_host, int32_t n, int32_t *ids_out_host, void *stream)
{
    if (!ix || !means_host || !ids_out_host || n < 1 || n > kMaxMeans) return LVQ_ERR_INVALID_ARG;
    const Format &f = ix->f;
    const int d = f.dim;
    if (!finite_host(means_host, (size_t)n * d)) return LVQ_ERR_NONFINITE;
    std::lock_guard<std::mutex> lk(ix->mu);
    hipStream_t s = (hipStream_t)stream;
    int rc = begin_call(ix, s);
    if (rc) return rc;
    if (ix->capturing) {
        ix->capturing = false;
        return LVQ_ERR_UNSUPPORTED;
    }
    if ((rc = order_after_updates(ix, s))) return rc;
    // rows per id over the occupied slots: a retired id none refers to is free
    std::vector<uint64_t> cnt(kMaxMeans, 0);
    if (ix->list_len > 0) {
        LVQ_HIP(launch_mean_counts(P<int32_t>(ix->lists[ix->list_active].buf), ix->list_len, P<uint8_t>(ix->rows),
                                   f.row_bytes, ix->n_means, P<unsigned long long>(ix->mean_counts), s));
        LVQ_HIP(hipMemcpyAsync(cnt.data(), ix->mean_counts.p, sizeof(uint64_t) * ix->n_means,
                               hipMemcpyDeviceToHost, s));
        LVQ_HIP(hipStreamSynchronize(s));
    }
    std::vector<int32_t> ids;
    for (int m = 0; m < ix->n_means && (int)ids.size() < n; ++m)
        if (ix->retired[m] && cnt[m] == 0) ids.push_back(m);
    int next_new = ix->n_means;
    while ((int)ids.size() < n && next_new < kMaxMeans) ids.push_back(next_new++);
    if ((int)ids.size() < n) return LVQ_ERR_CAPACITY;
    std::vector<int32_t> kd(f.kpos);
    kernel_order_dims(f, kd.data());
    std::vector<float> col((size_t)d * n), mk((size_t)n * f.kpos, 0.0f);
    for (int i = 0; i < n; ++i) {
        for (int j = 0; j < d; ++j) col[(size_t)i * d + j] = means_host[(size_t)i * d + j];
        for (int t = 0; t < f.kpos; ++t)
            if (kd[t] >= 0) mk[(size_t)i * f.kpos + t] = means_host[(size_t)i * d + kd[t]];
    }
    for (int i = 0; i < n; ++i) {
        const int m = ids[i];
        LVQ_HIP(hipMemcpyAsync(P<float>(ix->means) + (size_t)m * d, means_host + (size_t)i * d, sizeof(float) * d,
                               hipMemcpyHostToDevice, s));
        // column m of the transposed table: d values with a stride of kMaxMeans
        LVQ_HIP(hipMemcpy2DAsync(P<float>(ix->means_t) + m, sizeof(float) * kMaxMeans, col.data() + (size_t)i * d,
                                 sizeof(float), sizeof(float), d, hipMemcpyHostToDevice, s));
        LVQ_HIP(hipMemcpyAsync(P<float>(ix->muk) + (size_t)m * f.kpos, mk.data() + (size_t)i * f.kpos,
                               sizeof(float) * f.kpos, hipMemcpyHostToDevice, s));
        ix->retired[m] = 0;
    }
    ix->n_means = std::max(ix->n_means, next_new);
    std::vector<uint8_t> act(kMaxMeans);
    for (int m = 0; m < kMaxMeans; ++m) act[m] = !ix->retired[m];
    LVQ_HIP(hipMemcpyAsync(ix->mean_active.p, act.data(), kMaxMeans, hipMemcpyHostToDevice, s));
    if ((rc = note_update(ix, s))) return rc;
    LVQ_HIP(hipStreamSynchronize(s));   // the host sources must outlive the copies
    for (int i = 0; i < n; ++i) ids_out_host[i] = ids[i];
    return LVQ_OK;
}

int lvq_mean_members(lvq_index *ix, const int32_t *mean_ids_host, int32_t n, int64_t *offsets_host,
                     int32_t *slots_dev, int64_t cap, void *stream)
{
    if (!ix || n < 0 || (n > 0 && (!mean_ids_host || !offsets_host)) || cap < 0 || (cap > 0 && !slots_dev))
        return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    for (int32_t i = 0; i < n; ++i)
        if (mean_ids_host[i] < 0 || mean_ids_host[i] >= ix->n_means) return LVQ_ERR_INVALID_ARG;
    if (offsets_host) offsets_host[0] = 0;
    if (n == 0) return LVQ_OK;
    hipStream_t s = (hipStream_t)stream;
    int rc = begin_call(ix, s);
    if (rc) return rc;
    if (ix->capturing) {
        ix->capturing = false;
        return LVQ_ERR_UNSUPPORTED;
    }
    if ((rc = order_after_updates(ix, s))) return rc;
    Workspace &w = workspace(ix, s);
    if ((rc = ensure_members(ix, w, s))) return rc;
    // requested ids and, later, the output offsets share the probe buffer
    if ((rc = dev_alloc(ix, w.probe, sizeof(int32_t) * (size_t)n))) return rc;
    if ((rc = dev_alloc(ix, w.qoffs, sizeof(int64_t) * (size_t)(n + 1)))) return rc;
    if ((rc = dev_alloc(ix, w.qids, sizeof(uint64_t) * (size_t)n))) return rc;
    LVQ_HIP(hipMemcpyAsync(w.probe.p, mean_ids_host, sizeof(int32_t) * n, hipMemcpyHostToDevice, s));
    const uint32_t epoch = ix->epoch;
    unsigned long long *counts = P<unsigned long long>(w.qids);
    LVQ_HIP(launch_members_live(P<int32_t>(w.probe), n, P<int64_t>(w.moffs), P<int32_t>(w.members), P<uint8_t>(ix->rows),
                                ix->f.row_bytes, epoch, nullptr, nullptr, counts, s));
    std::vector<uint64_t> c(n);
    LVQ_HIP(hipMemcpyAsync(c.data(), counts, sizeof(uint64_t) * n, hipMemcpyDeviceToHost, s));
    LVQ_HIP(hipStreamSynchronize(s));
    for (int32_t i = 0; i < n; ++i) offsets_host[i + 1] = offsets_host[i] + (int64_t)c[i];
    if (offsets_host[n] > cap) return LVQ_ERR_CAPACITY;
    LVQ_HIP(hipMemcpyAsync(w.qoffs.p, offsets_host, sizeof(int64_t) * (n + 1), hipMemcpyHostToDevice, s));
    LVQ_HIP(launch_members_live(P<int32_t>(w.probe), n, P<int64_t>(w.moffs), P<int32_t>(w.members), P<uint8_t>(ix->rows),
                                ix->f.row_bytes, epoch, P<int64_t>(w.qoffs), slots_dev, counts, s));
    LVQ_HIP(hipStreamSynchronize(s));   // offsets_host is read by the copy above
    ix->capturing = false;
    return LVQ_OK;
}

}  // extern "C"

int lvq::host_reserve(lvq_index *ix, hipStream_t s, int64_t max_nq, int32_t k_first, int32_t prec,
                      int32_t scan_level, int32_t k_rerank, int32_t rerank_level)
{
    if (max_nq < 1 || max_nq > INT32_MAX || k_first < 1 || k_first > kMaxTopK || k_rerank < 0 ||
        k_rerank > kMaxTopK)
        return LVQ_ERR_INVALID_ARG;
    if (scan_level != LVQ_PRIMARY && scan_level != LVQ_FULL) return LVQ_ERR_INVALID_ARG;
    if (k_rerank > 0 && rerank_level != LVQ_PRIMARY && rerank_level != LVQ_FULL) return LVQ_ERR_INVALID_ARG;
    const Format &f = ix->f;
    const int64_t n_rows = ix->cfg.capacity;   // the part counts grow with the rows scanned
    size_t qk = 0, part = 0, q16 = 0, gthr = 0, order = 0, mkeys = 0;
    const size_t qsum = sizeof(float) * (size_t)max_nq;
    const size_t cm = sizeof(float) * (size_t)max_nq * kMaxMeans;   // any mean count the index may reach
    if (prec == LVQ_FP32) qk = scan_table_bytes(ix, max_nq, 16);
    else if (k_rerank > 0) qk = sizeof(float) * (size_t)max_nq * f.kpos;
    // the wide matrix-core scan, at the most queries of every tile count; with
    // a sample its part count does not only grow with the rows, so fewer are
    // looked at too
    auto reserve_wide = [&](int64_t tq, int bits2) {
        for (int64_t rows = n_rows;; rows = rows * 7 / 8) {
            for (int64_t qtiles = 1; (qtiles - 1) * tq < max_nq; ++qtiles) {
                const int64_t nq = std::min<int64_t>(max_nq, qtiles * tq);
                int64_t grid = 0;
                ScanSample sm = {0, 0};
                if (ix->cfg.mem_budget_bytes <= 0) sm = scan_sample(ix, qtiles, k_first, rows, bits2, prec);
                const int64_t parts = scan_parts_wide(ix, qtiles, k_first, rows, prec, sm, &grid);
                part = std::max(part, sizeof(uint64_t) * (size_t)(nq * parts * k_first));
                part = std::max(part, sizeof(float) * 8 * (size_t)(nq * sm.parts));
                mkeys = std::max(mkeys, sizeof(uint64_t) * (size_t)grid * tq * mfma_wide_cap(k_first));
            }
            if (rows <= 512 || ix->cfg.mem_budget_bytes > 0) break;
        }
    };
    if (prec == LVQ_FP32) {
        // the vector scans, over fewer rows too: their part counts do not only grow
        // with the rows (under a budget they do, nearly).  The tile size changes
        // once with the batch size, up to 9 queries.
        ScanPlan pl, pp;
        bool have = false;
        for (int64_t nq = 1; nq <= max_nq; ++nq) {
            if (nq <= 9) have = scan_plan(ix, nq, k_first, scan_level, &pl);
            const bool pairs = scan_plan_pairs(ix, nq, k_first, scan_level, &pp);
            for (int64_t rows = n_rows; have || pairs; rows = rows * 7 / 8) {
                int64_t parts = have ? scan_parts_fp32(ix, pl, nq, k_first, rows) : 0;
                if (pairs) parts = std::max(parts, scan_parts_fp32(ix, pp, nq, k_first, rows));
                part = std::max(part, sizeof(uint64_t) * (size_t)(nq * parts * k_first));
                if (rows <= 512 || ix->cfg.mem_budget_bytes > 0) break;
            }
        }
        // the FP32 matrix-core scan (inner product; its query block does not
        // depend on the mean count, which only decides whether the c_m table
        // fits)
        const int qbf = ix->cfg.metric == LVQ_IP
                            ? mfma_wide_query_block(f.bits1, scan_level == LVQ_FULL ? f.bits2 : 0, f.kpos, LVQ_FP32,
                                                    k_first, 1, ix->lds_max)
                            : 0;
        if (qbf) {
            const int64_t tq = 32 * qbf;
            gthr = sizeof(uint32_t) * (size_t)max_nq;
            q16 = (size_t)((max_nq + tq - 1) / tq) * tq * f.kpos * 4;
            reserve_wide(tq, scan_level == LVQ_FULL ? f.bits2 : 0);
        }
    } else {
        const int bits2 = scan_level == LVQ_FULL ? f.bits2 : 0;
        const int qbw = mfma_wide_query_block(f.bits1, bits2, f.kpos, prec, k_first, kMaxMeans, ix->lds_max);
        const int qb = qbw ? qbw : mfma_query_block(f.bits1, bits2, f.kpos);
        if (!qb) return LVQ_ERR_UNSUPPORTED;
        // the wide kernel when it takes any mean count the index may reach;
        // else reserve for both kernels (the register-resident one serves
        // what the wide one cannot)
        const int qbw_any = mfma_wide_query_block(f.bits1, bits2, f.kpos, prec, k_first, 1, ix->lds_max);
        const int qbo = mfma_query_block(f.bits1, bits2, f.kpos);
        for (int kind = 0; kind < 2; ++kind) {
            const bool wide = kind == 0;
            const int q = wide ? qbw_any : (qbw ? 0 : qbo);
            if (!q) continue;
            const int64_t tq = 32 * q;
            q16 = std::max(q16, (size_t)((max_nq + tq - 1) / tq) * tq * f.kpos * 2);
            if (wide) {
                reserve_wide(tq, bits2);
                continue;
            }
            for (int64_t nq = 1; nq <= max_nq; ++nq) {
                const int64_t parts = scan_parts_mfma(ix, (nq + tq - 1) / tq, k_first, n_rows);
                part = std::max(part, sizeof(uint64_t) * (size_t)(nq * parts * k_first));
            }
        }
        gthr = sizeof(uint32_t) * (size_t)max_nq;
    }
    if (k_rerank > 0) {
        order = sizeof(int32_t) * (size_t)max_nq;
        // keys of split lists, behind the queries: at most one item per resident
        // workgroup of 256 lanes (host_distances takes no room for them under a budget)
        if (ix->cfg.mem_budget_bytes <= 0) qk += 256 + sizeof(uint64_t) * (size_t)ix->n_cu * 8 * k_rerank;
    }
    Workspace &w = workspace(ix, s);
    int rc;
    if (qk && (rc = dev_alloc(ix, w.qk, qk))) return rc;
    if ((rc = dev_alloc(ix, w.qsum, qsum))) return rc;
    if ((rc = dev_alloc(ix, w.cm, cm))) return rc;
    if (part && (rc = dev_alloc(ix, w.part, part))) return rc;
    if (q16 && (rc = dev_alloc(ix, w.q16, q16))) return rc;
    if (gthr && (rc = dev_alloc(ix, w.gthr, gthr))) return rc;
    if (mkeys && (rc = dev_alloc(ix, w.mkeys, mkeys))) return rc;
    if (order && (rc = dev_alloc(ix, w.order, order))) return rc;
    if (k_rerank > 0 && (rc = dev_alloc(ix, w.queue, 64))) return rc;
    return LVQ_OK;
}

extern "C" {

int lvq_read_rows(lvq_index *ix, const int32_t *slots_dev, int64_t n, uint8_t *rows_dev, uint8_t *resid_dev,
                  void *stream)
{
    if (!ix || n < 0 || (n > 0 && (!slots_dev || !rows_dev))) return LVQ_ERR_INVALID_ARG;
    if (n == 0) return LVQ_OK;
    std::lock_guard<std::mutex> lk(ix->mu);
    hipStream_t s = (hipStream_t)stream;
    int rc = order_after_updates(ix, s);
    if (rc) return rc;
    LVQ_HIP(launch_gather_rows(store_args(ix), slots_dev, n, rows_dev, resid_dev, s));
    return LVQ_OK;
}

int lvq_bw_stream(const void *src_dev, int64_t bytes, uint32_t *sink_dev, void *stream)
{
    if (!sink_dev || bytes < 0 || (bytes & 15) || (bytes > 0 && (!src_dev || ((uintptr_t)src_dev & 15))))
        return LVQ_ERR_INVALID_ARG;
    LVQ_HIP(launch_bw_stream(src_dev, bytes / 16, sink_dev, (hipStream_t)stream));
    return LVQ_OK;
}

int lvq_bw_gather(lvq_index *ix, const int32_t *ids_dev, int64_t n, int32_t level, uint32_t *sink_dev, void *stream)
{
    if (!ix || !sink_dev || n < 0 || (n > 0 && !ids_dev) || (level != LVQ_PRIMARY && level != LVQ_FULL))
        return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    const Format &f = ix->f;
    if (level == LVQ_FULL && !f.bits2) return LVQ_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    int rc = order_after_updates(ix, s);
    if (rc) return rc;
    const bool full = level == LVQ_FULL;
    LVQ_HIP(launch_bw_gather(P<uint8_t>(ix->rows), f.row_bytes, (kHeaderBytes + 16 * f.kchunks) / 16,
                             full ? P<uint8_t>(ix->resid) : nullptr, f.resid_bytes, f.resid_bytes / 16, ids_dev, n,
                             ix->cfg.capacity, sink_dev, s));
    return LVQ_OK;
}

int lvq_get_stats(lvq_index *ix, lvq_stats *out)
{
    if (!ix || !out) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    out->capacity = ix->cfg.capacity;
    out->free_slots = ix->free_top;
    out->live_estimate = ix->cfg.capacity - ix->free_top;
    out->device_bytes = ix->device_bytes;
    out->n_means = ix->n_means;
    out->row_bytes = ix->f.row_bytes;
    out->resid_bytes = ix->f.resid_bytes;
    out->code_positions = ix->f.npos;
    out->epoch = ix->epoch;
    out->last_workgroups = ix->last_wg;
    out->last_lists = ix->last_lists;
    out->last_parts = ix->last_parts;
    return LVQ_OK;
}

int lvq_set_timing(lvq_index *ix, int enable)
{
    if (!ix) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    ix->timing = enable != 0;
    return LVQ_OK;
}

int lvq_kernel_time(lvq_index *ix, double *ms_out, int64_t *launches_out)
{
    if (!ix || !ms_out) return LVQ_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(ix->mu);
    double total = 0.0;
    for (auto &p : ix->tev) {
        LVQ_HIP(hipEventSynchronize(p.second));
        float ms = 0.0f;
        LVQ_HIP(hipEventElapsedTime(&ms, p.first, p.second));
        total += ms;
        (void)hipEventDestroy(p.first);
        (void)hipEventDestroy(p.second);
    }
    if (launches_out) *launches_out = (int64_t)ix->tev.size();
    ix->tev.clear();
    *ms_out = total;
    return LVQ_OK;
}

int lvq_sync(lvq_index *ix, void *stream)
{
    if (!ix) return LVQ_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    LVQ_HIP(hipStreamSynchronize(s));
    uint32_t e = 0;
    {
        std::lock_guard<std::mutex> lk(ix->mu);
        LVQ_HIP(hipMemcpy(&e, ix->err.p, sizeof(uint32_t), hipMemcpyDeviceToHost));
        if (e) LVQ_HIP(hipMemset(ix->err.p, 0, sizeof(uint32_t)));
    }
    if (e & kErrNonFinite) return LVQ_ERR_NONFINITE;
    if (e & kErrBadSlot) return LVQ_ERR_BAD_SLOT;
    if (e & (kErrBadOffsets | kErrOverflow)) return LVQ_ERR_INVALID_ARG;
    return LVQ_OK;
}

int lvq_mean(const float *x_dev, int64_t n, int32_t dim, float *mean_out_dev, void *stream)
{
    if (!x_dev || !mean_out_dev || n < 1 || dim < 1) return LVQ_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    const int64_t nchunks = (n + 4095) / 4096;
    double *scratch = nullptr;
    LVQ_HIP(hipMallocAsync((void **)&scratch, sizeof(double) * (size_t)nchunks * dim, s));
    hipError_t e = launch_mean(x_dev, n, dim, mean_out_dev, scratch, s);
    hipError_t e2 = hipFreeAsync(scratch, s);
    LVQ_HIP(e);
    LVQ_HIP(e2);
    return LVQ_OK;
}

int lvq_kmeans(const float *x_dev, int64_t n, int32_t dim, int32_t k, const int64_t *init_idx_host, int32_t iters,
               float *means_out_dev, void *stream)
{
    if (!x_dev || !means_out_dev || !init_idx_host || n < 1 || dim < 1 || k < 1 || k > n || iters < 0)
        return LVQ_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    for (int m = 0; m < k; ++m) {
        if (init_idx_host[m] < 0 || init_idx_host[m] >= n) return LVQ_ERR_INVALID_ARG;
        LVQ_HIP(hipMemcpyAsync(means_out_dev + (size_t)m * dim, x_dev + (size_t)init_idx_host[m] * dim,
                               sizeof(float) * dim, hipMemcpyDeviceToDevice, s));
    }
    int32_t *assign = nullptr;
    LVQ_HIP(hipMallocAsync((void **)&assign, sizeof(int32_t) * (size_t)n, s));
    hipError_t e = hipSuccess;
    for (int it = 0; it < iters && e == hipSuccess; ++it) {
        e = launch_kmeans_assign(x_dev, n, dim, means_out_dev, k, assign, s);
        if (e == hipSuccess) e = launch_kmeans_update(x_dev, n, dim, assign, k, means_out_dev, s);
    }
    hipError_t e2 = hipFreeAsync(assign, s);
    LVQ_HIP(e);
    LVQ_HIP(e2);
    return LVQ_OK;
}

}  // extern "C"

// ---- graph construction (App. A) ---------------------------------------------

namespace {

int graph_device_lds(size_t *out)
{
    int dev = 0, bytes = 0;
    LVQ_HIP(hipGetDevice(&dev));
    LVQ_HIP(hipDeviceGetAttribute(&bytes, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    *out = (size_t)bytes;
    return LVQ_OK;
}

int graph_kernel_error(uint32_t e)
{
    if (e & kErrBadSlot) return LVQ_ERR_BAD_SLOT;
    if (e & kErrBadOffsets) return LVQ_ERR_INVALID_ARG;
    return LVQ_OK;   // a search that stopped at the seen-set capacity still yields candidates
}

// Device buffers of one construction call: parts of one allocation (each
// allocation and release costs about as much as a small batch), released on
// every exit path.
struct GraphScratch {
    void *mem = nullptr;
    size_t bytes = 0;
    std::vector<std::pair<void **, size_t>> parts;
    hipStream_t s;
    explicit GraphScratch(hipStream_t st) : s(st) {}
    template <typename T>
    void want(T **p, size_t count)
    {
        *p = nullptr;
        parts.emplace_back(reinterpret_cast<void **>(p), bytes);
        bytes += (std::max<size_t>(count, 1) * sizeof(T) + 255) / 256 * 256;
    }
    int get()
    {
        LVQ_HIP(hipMalloc(&mem, bytes));
        for (auto &p : parts) *p.first = static_cast<char *>(mem) + p.second;
        return LVQ_OK;
    }
    ~GraphScratch()
    {
        if (!mem) return;
        (void)hipStreamSynchronize(s);
        (void)hipFree(mem);
    }
};

// The update routine of graph construction (App. A) for the nodes of
// `order`, `passes` times (alpha = 1 first when there are two passes):
// their rows are cleared, then batch by batch each node's window nearest
// nodes found from `entry` are pruned into its out-neighbours and it joins
// their out-neighbours (pruned on overflow).  A batch is at most max_batch
// nodes and, in the first pass, at most the number already in the graph
// (in_graph before the first node, plus the nodes inserted so far).
int graph_update(const float *x_dev, int64_t n, int dim, int metric, const std::vector<int32_t> &order,
                 int64_t in_graph, int R, int window, float alpha, int passes, int32_t entry, int32_t max_batch,
                 int32_t *graph_dev, hipStream_t s)
{
    if (dim < 1 || dim > kGraphMaxDim || (metric != LVQ_L2 && metric != LVQ_IP) || R < 1 || R > kGraphMaxDegree ||
        window < R || window > 256 || !(alpha > 0.0f) || !std::isfinite(alpha) || max_batch < 1)
        return LVQ_ERR_INVALID_ARG;
    size_t lds_max = 0;
    int rc = graph_device_lds(&lds_max);
    if (rc) return rc;
    if (graph_lds_bytes(dim, window, R) > lds_max) return LVQ_ERR_UNSUPPORTED;
    const int64_t count = (int64_t)order.size();
    if (count == 0) return LVQ_OK;
    const int64_t B = std::min<int64_t>(max_batch, count);
    GraphScratch sc(s);
    int32_t *order_d, *res, *cnt, *rev, *touched, *ntouched, *entry_d;
    int64_t *offs, *scan;
    uint32_t *err;
    const int64_t nb = (n + 2047) / 2048;
    sc.want(&order_d, (size_t)count);
    sc.want(&res, (size_t)(B * window));
    sc.want(&cnt, (size_t)n);
    sc.want(&offs, (size_t)n + 1);
    sc.want(&scan, (size_t)nb + 1);
    sc.want(&rev, (size_t)(B * R));
    sc.want(&touched, (size_t)(B * R));
    sc.want(&ntouched, 1);
    sc.want(&entry_d, 1);
    sc.want(&err, 1);
    if ((rc = sc.get())) return rc;
    LVQ_HIP(hipMemcpyAsync(order_d, order.data(), sizeof(int32_t) * (size_t)count, hipMemcpyHostToDevice, s));
    LVQ_HIP(hipMemcpyAsync(entry_d, &entry, sizeof(int32_t), hipMemcpyHostToDevice, s));
    LVQ_HIP(launch_graph_clear_rows(graph_dev, R, n, nullptr, order_d, count, s));
    LVQ_HIP(launch_fill_i32(cnt, 0, n, s));
    LVQ_HIP(launch_fill_u32(err, 0, 1, s));
    for (int pass = 0; pass < passes; ++pass) {
        const float a = (passes == 2 && pass == 0) ? 1.0f : alpha;
        for (int64_t b = 0; b < count;) {
            const int64_t now = pass == 0 ? in_graph + b : n;
            const int64_t bs = std::min<int64_t>({B, std::max<int64_t>(1, now), count - b});
            const int32_t *nodes = order_d + b;
            GraphLaunch g{};
            g.capacity = n;
            g.kpos = dim;
            g.metric = metric;
            g.n_means = 1;
            g.nq = bs;
            g.graph = graph_dev;
            g.degree = R;
            g.entries = entry_d;
            g.n_entries = 1;
            g.window = window;
            g.k = window;
            g.ids = res;
            g.err = err;
            g.xf = x_dev;
            g.dim = dim;
            g.qnodes = nodes;
            LVQ_HIP(launch_graph_search(g, s));
            PruneLaunch p{};
            p.xf = x_dev;
            p.dim = dim;
            p.metric = metric;
            p.n = n;
            p.nodes = nodes;
            p.m = bs;
            p.cids = res;
            p.cstride = window;
            p.always = 1;
            p.graph = graph_dev;
            p.R = R;
            p.alpha = a;
            p.err = err;
            LVQ_HIP(launch_graph_prune(p, s));
            LVQ_HIP(launch_reverse_edges(graph_dev, R, nodes, bs, n, cnt, offs, scan, rev, touched, ntouched, s));
            // (the host does not wait for the count: a wave per possible node is
            // launched, and those past it end at once)
            PruneLaunch r = p;
            r.nodes = touched;
            r.m = std::min<int64_t>(n, bs * R);
            r.m_dev = ntouched;
            r.coffs = offs;
            r.by_node = 1;
            r.cids = rev;
            r.cstride = 0;
            r.always = 0;
            LVQ_HIP(launch_graph_prune(r, s));
            b += bs;
        }
    }
    uint32_t herr = 0;
    LVQ_HIP(hipMemcpyAsync(&herr, err, sizeof(herr), hipMemcpyDeviceToHost, s));
    LVQ_HIP(hipStreamSynchronize(s));
    return graph_kernel_error(herr);
}

}  // namespace

extern "C" {

int lvq_graph_prune(const float *x_dev, int64_t n, int32_t dim, int32_t metric, const int32_t *nodes_dev, int64_t m,
                    const int64_t *cand_offsets_dev, const int32_t *cand_ids_dev, int32_t degree, float alpha,
                    int32_t *graph_dev, void *stream)
{
    if (n < 1 || n > INT32_MAX || dim < 1 || dim > kGraphMaxDim || (metric != LVQ_L2 && metric != LVQ_IP) || m < 0 ||
        m > INT32_MAX || degree < 1 || degree > kGraphMaxDegree || !(alpha > 0.0f) || !std::isfinite(alpha))
        return LVQ_ERR_INVALID_ARG;
    if (m == 0) return LVQ_OK;
    if (!x_dev || !nodes_dev || !cand_offsets_dev || !cand_ids_dev || !graph_dev) return LVQ_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    GraphScratch sc(s);
    uint32_t *err = nullptr;
    sc.want(&err, 1);
    int rc = sc.get();
    if (rc) return rc;
    LVQ_HIP(launch_fill_u32(err, 0, 1, s));
    PruneLaunch l{};
    l.xf = x_dev;
    l.dim = dim;
    l.metric = metric;
    l.n = n;
    l.nodes = nodes_dev;
    l.m = m;
    l.coffs = cand_offsets_dev;
    l.by_node = 0;
    l.cids = cand_ids_dev;
    l.always = 1;
    l.graph = graph_dev;
    l.R = degree;
    l.alpha = alpha;
    l.err = err;
    LVQ_HIP(launch_graph_prune(l, s));
    uint32_t herr = 0;
    LVQ_HIP(hipMemcpyAsync(&herr, err, sizeof(herr), hipMemcpyDeviceToHost, s));
    LVQ_HIP(hipStreamSynchronize(s));
    return graph_kernel_error(herr);
}

int lvq_graph_build(const float *x_dev, int64_t n, int32_t dim, int32_t metric, int64_t first, int32_t degree,
                    int32_t window, float alpha, int32_t passes, int32_t entry, int32_t max_batch, int32_t *graph_dev,
                    void *stream)
{
    if (!x_dev || !graph_dev || n < 1 || n > INT32_MAX || first < 0 || first > n || passes < 1 || passes > 2 ||
        entry < 0 || entry >= n || (first > 0 && entry >= first))
        return LVQ_ERR_INVALID_ARG;
    std::vector<int32_t> order;
    order.reserve((size_t)(n - first));
    if (first == 0) {
        order.push_back(entry);
        for (int64_t v = 0; v < n; ++v)
            if (v != entry) order.push_back((int32_t)v);
    } else {
        for (int64_t v = first; v < n; ++v) order.push_back((int32_t)v);
    }
    return graph_update(x_dev, n, dim, metric, order, first, degree, window, alpha, passes, entry, max_batch,
                        graph_dev, (hipStream_t)stream);
}

int lvq_graph_insert(const float *x_dev, int64_t n, int32_t dim, int32_t metric, const int32_t *nodes_host,
                     int64_t m, int32_t degree, int32_t window, float alpha, int32_t entry, int32_t max_batch,
                     int32_t *graph_dev, void *stream)
{
    if (!x_dev || !graph_dev || n < 1 || n > INT32_MAX || m < 0 || m > n || (m > 0 && !nodes_host) || entry < 0 ||
        entry >= n)
        return LVQ_ERR_INVALID_ARG;
    std::vector<int32_t> order(nodes_host, nodes_host + m);
    std::vector<int32_t> sorted = order;
    std::sort(sorted.begin(), sorted.end());
    for (size_t i = 0; i < sorted.size(); ++i)
        if (sorted[i] < 0 || sorted[i] >= n || sorted[i] == entry || (i > 0 && sorted[i] == sorted[i - 1]))
            return LVQ_ERR_INVALID_ARG;
    return graph_update(x_dev, n, dim, metric, order, n - m, degree, window, alpha, 1, entry, max_batch, graph_dev,
                        (hipStream_t)stream);
}

int lvq_graph_delete(const float *x_dev, int64_t n, int32_t dim, int32_t metric, const uint8_t *deleted_dev,
                     int32_t degree, float alpha, int32_t *graph_dev, void *stream)
{
    if (!x_dev || !deleted_dev || !graph_dev || n < 1 || n > INT32_MAX || dim < 1 || dim > kGraphMaxDim ||
        (metric != LVQ_L2 && metric != LVQ_IP) || degree < 1 || degree > kGraphMaxDegree || !(alpha > 0.0f) ||
        !std::isfinite(alpha))
        return LVQ_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    GraphScratch sc(s);
    int32_t *affected, *count;
    uint32_t *err;
    int rc;
    sc.want(&affected, (size_t)n);
    sc.want(&count, 1);
    sc.want(&err, 1);
    if ((rc = sc.get())) return rc;
    LVQ_HIP(launch_fill_u32(err, 0, 1, s));
    LVQ_HIP(launch_graph_affected(graph_dev, degree, n, deleted_dev, affected, count, s));
    int32_t na = 0;
    LVQ_HIP(hipMemcpyAsync(&na, count, sizeof(na), hipMemcpyDeviceToHost, s));
    LVQ_HIP(hipStreamSynchronize(s));
    PruneLaunch p{};
    p.xf = x_dev;
    p.dim = dim;
    p.metric = metric;
    p.n = n;
    p.nodes = affected;
    p.m = na;
    p.always = 0;
    p.graph = graph_dev;
    p.R = degree;
    p.alpha = alpha;
    p.err = err;
    p.deleted = deleted_dev;
    LVQ_HIP(launch_graph_prune(p, s));
    LVQ_HIP(launch_graph_clear_rows(graph_dev, degree, n, deleted_dev, nullptr, 0, s));
    uint32_t herr = 0;
    LVQ_HIP(hipMemcpyAsync(&herr, err, sizeof(herr), hipMemcpyDeviceToHost, s));
    LVQ_HIP(hipStreamSynchronize(s));
    return graph_kernel_error(herr);
}

}  // extern "C"
