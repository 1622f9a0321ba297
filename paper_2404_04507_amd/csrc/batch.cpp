// batch.cpp - ragged batches of plans applied by one persistent launch per
// pass (e.g. a sweep of couplings whose windows differ), optionally replayed
// from a captured hipGraph.
//
// The work table (per instance: geometry, tables, schedule, vector and
// workspace pointers, and the first work item of each pass) lives in device
// memory and is refreshed by an asynchronous copy before every apply; the
// launches (and the captured graph) only see its address, so one graph
// serves every apply of the batch.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "apply_kernels.hpp"
#include "apply_launch.hpp"
#include "plan.hpp"

using namespace iwfpm;

struct iwfpm_batch_s {
    int B = 0;
    int prec = 0;
    int device = 0;
    std::vector<iwfpm_plan_s*> plans;
    DeviceBuf d_table;           // BatchHead, B BatchItems, B FewCalls, B + 1 starts per few-mode launch
    DeviceBuf d_few;             // B FewItems
    std::vector<FewItem> items;  // the same on the host
    unsigned char* h_table = nullptr;  // pinned staging
    size_t table_bytes = 0;
    hipEvent_t staged = nullptr;  // the last copy out of the staging buffer
    int maxs = 16;
    size_t lds = 0;
    int grid = 0;
    bool use_graph = false;
    bool all_transforms = false;          // no plan takes the few-mode route
    bool transforms = false;              // some plan takes the transform passes
    std::vector<FewLaunch> few;           // few-mode plans: one launch per kind of kernel
    size_t call_off = 0, start_off = 0;   // table offsets of the FewCalls and the starts
    hipGraphExec_t gexec = nullptr;
    hipStream_t gstream = nullptr;
    bool few_of(const iwfpm_plan_s* p) const { return !all_transforms && p->few_modes[prec]; }
};

static size_t items_offset() { return (sizeof(BatchHead) + 255) / 256 * 256; }

// Few-mode plans without a walk have a kernel for each number of pairs.  In a
// batch of small ones the launches cost more than the work, so they share the
// kernel that takes any number; its registers are those of the largest, which
// large batches would pay for.  us, a launch each : one launch : transforms, with
// 2 to 12 pairs (float64, one vector, then six):
//   8 plans of some 600 points          48 : 19 : 32     48 : 19 : 34
//   16 of 10,000 (160 thousand in all)  42 : 30 : 38     45 : 36 : 43
//   64 of 10,000 (640 thousand)        101 : 86 : 93    101 : 88 : 109
//   64 of 26,000 (1.7 million)         102 : 130 : 114  123 : 166 : 198
constexpr long long kJointPoints = 786432;
// A graph costs more than the few launches that a batch of few-mode plans has
// (one launch, 8 plans 41 : 19 us, 64 plans 117 : 86; five launches 54 : 48)
constexpr size_t kDirectLaunches = 5;
static void join_point_kinds(std::vector<FewItem>& items) {
    for (int d = 1; d <= kStencilMaxD; ++d) {
        long long points = 0;
        int first = 0;
        bool several = false;
        for (const FewItem& it : items) {
            if (it.kind / 100 != d) continue;
            points += it.g.N;
            several = several || (first && it.kind != first);
            first = it.kind;
        }
        if (!several || points > kJointPoints) continue;
        for (FewItem& it : items)
            if (it.kind / 100 == d) it.kind = few_joint_kind(d);
    }
}

static hipError_t launch_few(iwfpm_batch_s* b, hipStream_t st) {
    const unsigned char* table = (const unsigned char*)b->d_table.ptr;
    for (size_t k = 0; k < b->few.size(); ++k) {
        const int* start = reinterpret_cast<const int*>(table + b->start_off) + k * (b->B + 1);
        hipError_t e = launch_few_batch(b->few[k], (const FewItem*)b->d_few.ptr,
                                        reinterpret_cast<const FewCall*>(table + b->call_off), start, b->B, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename R>
static hipError_t launch_passes(iwfpm_batch_s* b, hipStream_t st) {
    if (hipError_t e = launch_few(b, st); e != hipSuccess) return e;
    if (!b->transforms) return hipSuccess;
    const void* head = b->d_table.ptr;
    const void* items = (const unsigned char*)b->d_table.ptr + items_offset();
    for (int pass = 0; pass < 3; ++pass) {
        hipError_t e;
        switch (b->maxs) {
            case 16: e = launch_batch<R, 16>(head, items, b->grid, b->lds, pass, st); break;
            case 32: e = launch_batch<R, 32>(head, items, b->grid, b->lds, pass, st); break;
            default: e = launch_batch<R, 64>(head, items, b->grid, b->lds, pass, st); break;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename R>
static hipError_t occupancy(int maxs, size_t lds, int* n) {
    switch (maxs) {
        case 16: return occupancy_batch<R, 16>(lds, n);
        case 32: return occupancy_batch<R, 32>(lds, n);
        default: return occupancy_batch<R, 64>(lds, n);
    }
}

int iwfpm::batch_create(int B, const iwfpm_plan_t* plans, int precision, int use_graph, bool transforms,
                        iwfpm_batch_t* out) {
    if (!out || B < 1 || !plans) return IWFPM_ERR_ARG;
    *out = nullptr;
    if (precision != IWFPM_PREC_FP64 && precision != IWFPM_PREC_FP32) return IWFPM_ERR_ARG;
    const int prec = precision == IWFPM_PREC_FP32 ? 1 : 0;
    const size_t esz = prec ? 8 : 16;
    int dev = -1, maxe = 1;
    size_t lds = 0;
    for (int i = 0; i < B; ++i) {
        iwfpm_plan_s* p = plans[i];
        if (!p) return IWFPM_ERR_ARG;
        if (p->host_only) return IWFPM_ERR_NODEVICE;
        for (int j = 0; j < i; ++j)
            if (plans[j] == p) return IWFPM_ERR_ARG;  // each plan owns one workspace
        if (dev < 0) dev = p->opts.device;
        if (p->opts.device != dev) return IWFPM_ERR_ARG;  // one device per batch
        const Schedule& sc = p->sched[prec];
        if (!sc.ok) return IWFPM_ERR_UNSUPPORTED;
        if (!sc.fused && sc.pd.split_mid > 0) return IWFPM_ERR_UNSUPPORTED;  // five-pass grids: apply one by one
        if (!transforms && p->few_modes[prec]) continue;
        for (int ax = 0; ax < p->n; ++ax) maxe = std::max(maxe, axis_class(p->geom, ax));
        if (sc.fused) lds = std::max(lds, lds_fused(p->geom, esz));
        else lds = std::max({lds, lds_slabs(p->geom, sc.pd, esz), lds_columns(p->geom, sc.pd, esz)});
    }
    DeviceGuard guard(dev);
    if (!guard.ok) return IWFPM_ERR_DEVICE;
    iwfpm_batch_s* b = new (std::nothrow) iwfpm_batch_s();
    if (!b) return IWFPM_ERR_ALLOC;
    b->B = B;
    b->prec = prec;
    b->all_transforms = transforms;
    b->device = dev;
    b->plans.assign(plans, plans + B);
    b->maxs = extent_class_of(maxe);
    b->lds = lds;
    b->use_graph = use_graph != 0;
    b->items.resize(B);
    for (int i = 0; i < B; ++i) {
        const iwfpm_plan_s* p = plans[i];
        FewItem& it = b->items[i];
        std::memset(&it, 0, sizeof(it));
        it.kind = -1;
        if (!b->few_of(p)) {
            b->transforms = true;
            continue;
        }
        it.g = p->geom;
        it.t = p->tabs;
        it.sd = p->stencil;
        it.w = p->star;
        it.kind = few_kind(it.g, it.sd, it.w);
    }
    join_point_kinds(b->items);
    for (const FewItem& it : b->items) {
        bool known = it.kind < 0;
        for (const FewLaunch& l : b->few) known = known || l.kind == it.kind;
        if (!known) b->few.push_back(FewLaunch{it.kind, 0, 0, 0});
    }
    b->call_off = (items_offset() + (size_t)B * sizeof(BatchItem) + 255) / 256 * 256;
    b->start_off = (b->call_off + (size_t)B * sizeof(FewCall) + 255) / 256 * 256;
    b->table_bytes = b->start_off + b->few.size() * (B + 1) * sizeof(int);
    int rc = dev_alloc(b->d_table, b->table_bytes);
    if (rc == IWFPM_OK && hipHostMalloc((void**)&b->h_table, b->table_bytes) != hipSuccess) rc = IWFPM_ERR_ALLOC;
    if (rc == IWFPM_OK && hipEventCreateWithFlags(&b->staged, hipEventDisableTiming) != hipSuccess)
        rc = IWFPM_ERR_DEVICE;
    if (rc == IWFPM_OK && !b->few.empty()) {
        rc = dev_alloc(b->d_few, (size_t)B * sizeof(FewItem));
        if (rc == IWFPM_OK &&
            hipMemcpy(b->d_few.ptr, b->items.data(), (size_t)B * sizeof(FewItem), hipMemcpyHostToDevice) != hipSuccess)
            rc = IWFPM_ERR_DEVICE;
    }
    int per_cu = 0, cus = 0;
    for (FewLaunch& l : b->few)
        if (rc == IWFPM_OK && few_launch_config(l, b->items.data(), B) != hipSuccess) rc = IWFPM_ERR_DEVICE;
    if (rc == IWFPM_OK && b->transforms) {
        hipError_t e = prec ? occupancy<float>(b->maxs, lds, &per_cu) : occupancy<double>(b->maxs, lds, &per_cu);
        if (e != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            rc = IWFPM_ERR_DEVICE;
    }
    if (rc != IWFPM_OK) {
        iwfpm_batch_destroy(b);
        return rc;
    }
    b->grid = std::max(1, per_cu) * std::max(1, cus);
    *out = b;
    return IWFPM_OK;
}

extern "C" {

int iwfpm_batch_create(int B, const iwfpm_plan_t* plans, int precision, int use_graph, iwfpm_batch_t* out) {
    return batch_create(B, plans, precision, use_graph, false, out);
}

int iwfpm_batch_apply(iwfpm_batch_t b, const void* const* psi, void* const* hpsi, const int* nvec, void* stream) {
    if (!b || !psi || !hpsi || !nvec) return IWFPM_ERR_ARG;
    hipStream_t st = (hipStream_t)stream;
    DeviceGuard guard(b->device);
    if (!guard.ok) return IWFPM_ERR_DEVICE;
    for (int i = 0; i < b->B; ++i) {
        if (nvec[i] < 0 || (nvec[i] > 0 && (!psi[i] || !hpsi[i]))) return IWFPM_ERR_ARG;
        if (nvec[i] > 0) {
            int rc = plan_ensure_ws(b->plans[i], nvec[i], b->prec, st, b->all_transforms);
            if (rc) return rc;
        }
    }
    // the staging buffer may still be read by the previous copy
    if (hipEventSynchronize(b->staged) != hipSuccess) return IWFPM_ERR_DEVICE;
    BatchHead* head = reinterpret_cast<BatchHead*>(b->h_table);
    BatchItem* items = reinterpret_cast<BatchItem*>(b->h_table + items_offset());
    int tot[3] = {0, 0, 0};
    FewCall* calls = reinterpret_cast<FewCall*>(b->h_table + b->call_off);
    int* start = reinterpret_cast<int*>(b->h_table + b->start_off);
    double few_points = 0.0;
    for (int i = 0; i < b->B; ++i) {
        FewCall& c = calls[i];
        std::memset(&c, 0, sizeof(c));
        if (b->items[i].kind < 0 || nvec[i] == 0) continue;
        // results over the vectors themselves: the convolution reads neighbours,
        // while the transforms have read all of a vector before they write it
        const char *x = (const char*)psi[i], *y = (const char*)hpsi[i];
        const size_t bytes = (size_t)nvec[i] * (size_t)b->items[i].g.N * 16;
        if (x < y + bytes && y < x + bytes) {
            const int rc = plan_apply(b->plans[i], psi[i], hpsi[i], nvec[i],
                                      b->prec ? IWFPM_PREC_FP32 : IWFPM_PREC_FP64, st, 1, true);
            if (rc) return rc;
            continue;
        }
        c.psi = reinterpret_cast<const double2*>(psi[i]);
        c.hpsi = reinterpret_cast<double2*>(hpsi[i]);
        c.nvec = nvec[i];
        few_points += (double)b->items[i].g.N * nvec[i];
    }
    for (int i = 0; b->transforms && i < b->B; ++i) {
        iwfpm_plan_s* p = b->plans[i];
        const Schedule& sc = p->sched[b->prec];
        BatchItem& it = items[i];
        std::memset(&it, 0, sizeof(it));
        it.g = p->geom;
        it.t = p->tabs;
        it.pd = sc.pd;
        it.rg = row_geom(p->geom);
        it.psi = reinterpret_cast<const double2*>(psi[i]);
        it.hpsi = reinterpret_cast<double2*>(hpsi[i]);
        it.ws = p->d_ws.ptr;
        it.fused = sc.fused ? 1 : 0;
        for (int k = 0; k < 3; ++k) it.start[k] = tot[k];
        const int nv = nvec[i];
        if (b->items[i].kind >= 0) {
            // no workgroups here: see below
        } else if (sc.fused) {
            tot[0] += nv;
        } else {
            const int bpv = (sc.pd.s_out + sc.pd.slabs_per_wg - 1) / sc.pd.slabs_per_wg;
            const int ntile = (sc.pd.s_in + sc.pd.tile - 1) / sc.pd.tile;
            tot[0] += bpv * nv;
            tot[1] += ntile * nv;
            tot[2] += bpv * nv;
        }
    }
    for (size_t k = 0; k < b->few.size(); ++k) {
        int* s = start + k * (b->B + 1);
        s[0] = 0;
        // A star item deals its groups (the steps of one vector) to the XCDs from
        // the first on, and the next item goes on where it ended: all from the
        // first left the last XCDs idle (the launch on eight windows, ragged, 181
        // -> 146 us of the call's 224 -> 178; 8 plans of 24^2 x 32^2 points, one
        // vector each: 93 -> 54 us)
        int rot = 0;
        for (int i = 0; i < b->B; ++i) {
            s[i + 1] = s[i];
            if (b->items[i].kind != b->few[k].kind) continue;
            FewCall& c = calls[i];
            s[i + 1] += few_blocks(b->items[i], c, few_points);
            c.rot = (8 - rot) & 7;
            rot = (rot + c.w.chunks * c.nvec) & 7;
        }
    }
    head->B = b->B;
    for (int k = 0; k < 3; ++k) head->total[k] = tot[k];
    const size_t from = b->transforms ? 0 : b->call_off;
    if (hipMemcpyAsync((unsigned char*)b->d_table.ptr + from, b->h_table + from, b->table_bytes - from,
                       hipMemcpyHostToDevice, st) != hipSuccess)
        return IWFPM_ERR_DEVICE;
    if (hipEventRecord(b->staged, st) != hipSuccess) return IWFPM_ERR_DEVICE;
    // graphs cannot be captured on the null stream: launch directly there
    if (!b->use_graph || st == nullptr || (!b->transforms && b->few.size() <= kDirectLaunches))
        return (b->prec ? launch_passes<float>(b, st) : launch_passes<double>(b, st)) == hipSuccess ? IWFPM_OK
                                                                                                   : IWFPM_ERR_DEVICE;
    if (!b->gexec || b->gstream != st) {
        if (b->gexec) (void)hipGraphExecDestroy(b->gexec);
        b->gexec = nullptr;
        hipGraph_t graph = nullptr;
        if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess) return IWFPM_ERR_DEVICE;
        hipError_t e = b->prec ? launch_passes<float>(b, st) : launch_passes<double>(b, st);
        hipError_t e2 = hipStreamEndCapture(st, &graph);
        if (e != hipSuccess || e2 != hipSuccess || !graph) return IWFPM_ERR_DEVICE;
        e = hipGraphInstantiate(&b->gexec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) {
            b->gexec = nullptr;
            return IWFPM_ERR_DEVICE;
        }
        b->gstream = st;
    }
    return hipGraphLaunch(b->gexec, st) == hipSuccess ? IWFPM_OK : IWFPM_ERR_DEVICE;
}

int iwfpm_batch_destroy(iwfpm_batch_t b) {
    if (!b) return IWFPM_ERR_ARG;
    {
        DeviceGuard guard(b->device);
        if (b->gexec) (void)hipGraphExecDestroy(b->gexec);
        if (b->staged) (void)hipEventSynchronize(b->staged);
        if (b->staged) (void)hipEventDestroy(b->staged);
        (void)hipDeviceSynchronize();
        dev_free(b->d_table);
        dev_free(b->d_few);
        if (b->h_table) (void)hipHostFree(b->h_table);
    }
    delete b;
    return IWFPM_OK;
}

}  // extern "C"
