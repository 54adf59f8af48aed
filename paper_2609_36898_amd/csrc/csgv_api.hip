// C ABI of the decoder: argument checks, scratch, the plain and persistent
// launch forms, and batched plans.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/csgv.h"
#include "csgv_format.h"
#include "decode_kernel.h"

using namespace csgv;

namespace {

thread_local std::string g_last_error;

csgv_status fail(csgv_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return s;
}

#define HIP_TRY(expr)                                                                         \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess) return fail(CSGV_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

uint32_t rd32(const uint8_t* p) {
    uint32_t v;
    memcpy(&v, p, 4);
    return v;
}
uint64_t rd64(const uint8_t* p) {
    uint64_t v;
    memcpy(&v, p, 8);
    return v;
}

std::once_flag g_attr_once;
hipError_t g_attr_err = hipSuccess;

hipError_t ensure_attrs() {
    std::call_once(g_attr_once, [] { g_attr_err = set_kernel_attrs(); });
    return g_attr_err;
}

int device_cus() {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
    return n;
}

int device_lds_per_cu() {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 160 * 1024;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess || n <= 0)
        return 160 * 1024;
    return n;
}

bool valid_wg(int wg) { return wg == 128 || wg == 256 || wg == 512 || wg == 1024; }

// resident work-groups per CU for a shape (HIP occupancy: registers, LDS, waves)
int resident_per_cu(int wg, uint32_t cap16) {
    const int by_lds = device_lds_per_cu() / (int)shared_bytes(cap16);
    return std::max(1, std::min(by_lds, max_resident_per_cu(wg, std::max<uint32_t>(cap16, kMinCap16))));
}

// The LDS split of a work-group size whose split the caller left to the default.  A
// CU holds one work-group of 1024 threads, whatever its LDS (16 wavefronts of 128
// VGPRs), so it takes the largest split: with that of four work-groups of 256 its
// passes over a level in chunks are as short as theirs, and behind more barriers
// (2000 cubes of 32^3 noise, rANS: 0.87 ms with 10,240 slots, 0.56 with 32,760;
// three labels at random 1.05 and 0.48).
uint32_t default_slots(int wg) { return wg == 1024 ? kMaxCap16 : kDefaultCap16; }

// The shape of a launch whose work-group size and LDS split the caller left to
// the default.  With at most two tasks per CU a task's latency is the launch's,
// and 512 threads shorten it (64 bricks of 32^3: 58 -> 50 us, 512: 63 -> 55; 64
// bricks of 64^3 0.63 -> 0.47 ms; 1024 threads 55 and 89 us and 0.41 ms); such
// work-groups leave LDS for 24,576 slots, which hold level 5 of most 64^3 bricks
// at LOD 1 (512 cubes: 0.18 -> 0.14 ms).  1024 threads are the faster ones for 64^3
// cubes alone; a volume of 64^3 bricks decodes 32^3 cubes too, at LOD 1, and the
// LODs are in device memory, so the number of tasks is what the rule goes by.
// From three tasks per CU on, work-groups of 256 threads keep more bricks in flight.
void auto_shape(uint32_t n, int* wg, uint32_t* cap16) {
    if (n <= 2u * (uint32_t)device_cus()) {
        *wg = 512;
        *cap16 = 24576;
    }
}

RansFreq pack_freq(const csgv_volume_info* vol, bool* ok) {
    RansFreq f;
    uint32_t sum = 0;
    for (int s = 0; s < 16; ++s) sum += vol->rans_freq[s];
    *ok = sum == kRansM;
    for (int k = 0; k < 8; ++k) f.w[k] = (uint32_t)vol->rans_freq[2 * k] | ((uint32_t)vol->rans_freq[2 * k + 1] << 16);
    return f;
}

Params make_params(const csgv_volume_info* vol, const void* d_container, const uint32_t* ids, const uint8_t* lods,
                   const uint64_t* offs, uint32_t n, void* out, uint64_t cap, uint32_t* status) {
    Params P;
    memset(&P, 0, sizeof(P));
    P.vol = (const uint8_t*)d_container;
    P.vol_bytes = vol->total_bytes;
    P.off_pos = vol->offsets_pos;
    P.n_bricks = vol->n_bricks;
    P.label_bytes = vol->label_bytes;
    bool ok;
    (void)pack_freq(vol, &ok);
    P.freq_ok = ok;
    P.max_log2b = vol->max_log2b ? std::min<uint32_t>(vol->max_log2b, kMaxLog2b) : kMaxLog2b;
    P.ids = ids;
    P.lods = lods;
    P.out_offs = offs;
    P.n_tasks = n;
    P.out = (uint8_t*)out;
    P.out_cap = cap;
    P.status = status;
    P.scratch_stride = scratch_per_wg(P.max_log2b);
    P.scratch_sym = scr_sym(P.max_log2b);
    P.cap16 = kDefaultCap16;
    return P;
}

csgv_status check_task_args(const csgv_volume_info* vol, const void* d_container, const uint32_t* ids,
                            const uint8_t* lods, uint32_t n, void* out) {
    if (!vol) return fail(CSGV_EINVAL, "volume info is NULL");
    if (vol->label_bytes != 4 && vol->label_bytes != 8) return fail(CSGV_EINVAL, "label_bytes must be 4 or 8");
    if (vol->offsets_pos < kHeaderBytes || vol->offsets_pos + 8ull * ((uint64_t)vol->n_bricks + 1) > vol->total_bytes)
        return fail(CSGV_EINVAL, "offset table outside the container");
    if (n == 0) return CSGV_OK;
    if (!d_container || !ids || !lods || !out) return fail(CSGV_EINVAL, "NULL device pointer");
    return CSGV_OK;
}

csgv_status check_opts(const csgv_decode_opts* o) {
    if (!o) return CSGV_OK;
    if (o->wg_size != 0 && !valid_wg(o->wg_size)) return fail(CSGV_EINVAL, "wg_size %d (128, 256, 512 or 1024)", o->wg_size);
    if (o->lds_slots < 0 || (uint32_t)o->lds_slots > kMaxCap16)
        return fail(CSGV_EINVAL, "lds_slots %d (0, or %u..%u)", o->lds_slots, kMinCap16, kMaxCap16);
    if (o->lds_slots > 0 && (uint32_t)o->lds_slots < kMinCap16)
        return fail(CSGV_EINVAL, "lds_slots %d below %u (the slot area also holds the rANS table)", o->lds_slots,
                    kMinCap16);
    if (o->bricks_per_wave < 0) return fail(CSGV_EINVAL, "bricks_per_wave %d", o->bricks_per_wave);
    if (o->wgs_per_cu < -1) return fail(CSGV_EINVAL, "wgs_per_cu %d", o->wgs_per_cu);
    if (o->palette_bits < -1 || o->palette_bits > 31) return fail(CSGV_EINVAL, "palette_bits %d (0..31)", o->palette_bits);
    return CSGV_OK;
}

// device memory of one launch sequence (a plan's, or a one-shot call's)
struct Bufs {
    uint8_t* scratch = nullptr;
    Control* ctl = nullptr;
    uint32_t* lists = nullptr;   // kClasses * max_tasks
    uint32_t list_cap = 0;
    uint32_t* rans_tab = nullptr;
    uint64_t* dense = nullptr;   // max_tasks
    uint64_t* base = nullptr;    // one per block of kBinTasks
    uint64_t* totals = nullptr;  // one per block of kBinTasks
    bool prepared = false;       // the table is built and the binning kernel's counts are zero
};

uint64_t bin_blocks(uint64_t max_tasks) { return (max_tasks + kBinTasks - 1) / kBinTasks; }

// (the lists come last: a call in task order does without)
uint64_t aux_bytes(uint32_t max_tasks, bool lists = true) {
    return 256 + 4ull * kRansM + (lists ? 4ull * kClasses * max_tasks : 0) + 8 + 8ull * max_tasks + 16 * bin_blocks(max_tasks) + 256;
}

void carve(uint8_t* base, uint64_t scratch_bytes, uint32_t max_tasks, Bufs* b) {
    b->scratch = base;
    uint8_t* a = base + scratch_bytes;
    b->ctl = (Control*)a;
    b->rans_tab = (uint32_t*)(a + 256);
    b->dense = (uint64_t*)(b->rans_tab + kRansM);
    b->base = b->dense + max_tasks;
    b->totals = b->base + bin_blocks(max_tasks);
    b->lists = (uint32_t*)(b->totals + bin_blocks(max_tasks));
    b->list_cap = max_tasks;
}

// Everything a launch enqueues, in order: for buffers that are not prepared, the
// rANS table and zeroed control words; the task lists when tasks have to wait
// for a work-group and their cost decides the order, and the dense offsets when
// they are asked for; the decode.  With no more tasks than work-groups every
// task starts at once, so there is no queue and no order.  (Direct launches: a
// plan's one or two kernels leave 5.6 us between calls, a captured graph of
// them 8.4.)
hipError_t enqueue(Params P, const Bufs& b, const csgv_volume_info* vol, int wg, uint32_t grid, bool queue, bool sort,
                   hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    P.scratch = b.scratch;
    P.rans_tab = b.rans_tab;
    queue = queue && P.n_tasks > grid;
    sort = sort && queue;
    hipError_t e;
    // a call without a plan builds its rANS table and sets its control words: in
    // the binning kernel if there is one, of one block, else in a kernel before it
    const bool bin = queue || !P.out_offs, solo = bin && (P.n_tasks <= kBinTasks || (!sort && P.out_offs));
    bool table = false;
    RansFreq f{};
    if (!b.prepared) {
        f = pack_freq(vol, &table);
        if (!solo && (e = launch_prepare(b.ctl, table ? b.rans_tab : nullptr, &f, s)) != hipSuccess) return e;
    }
    P.ctl = b.ctl;
    P.list_cap = b.list_cap;
    if (!P.out_offs) {
        P.dense_offs = b.dense;
        P.dense_base = b.base;
    }
    if (bin && (e = launch_bin(P, sort ? b.lists : nullptr, P.out_offs ? nullptr : b.dense, b.base, b.totals,
                               solo && table ? b.rans_tab : nullptr, &f, s)) != hipSuccess)
        return e;
    if (sort) P.lists = b.lists;
    if (!queue) P.ctl = nullptr;
    if (ev0 && (e = hipEventRecord(ev0, s)) != hipSuccess) return e;
    if ((e = launch_decode(P, wg, grid, s)) != hipSuccess) return e;
    if (ev1 && (e = hipEventRecord(ev1, s)) != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace

// ------------------------------------------------------------------ C ABI
extern "C" {

const char* csgv_last_error(void) { return g_last_error.c_str(); }

csgv_status csgv_volume_parse(const void* h_container, uint64_t bytes, csgv_volume_info* out) {
    if (!h_container || !out) return fail(CSGV_EINVAL, "NULL argument");
    if (bytes < kHeaderBytes) return fail(CSGV_EINVAL, "container shorter than its header");
    const uint8_t* h = (const uint8_t*)h_container;
    if (rd32(h) != kMagic) return fail(CSGV_EINVAL, "bad magic");
    if (rd32(h + 4) != kVersion) return fail(CSGV_EINVAL, "unsupported version %u", rd32(h + 4));
    csgv_volume_info v;
    memset(&v, 0, sizeof(v));
    for (int a = 0; a < 3; ++a) {
        v.dims[a] = rd32(h + kHdrDims + 4 * a);
        v.grid[a] = rd32(h + kHdrGrid + 4 * a);
    }
    v.log2b = rd32(h + kHdrLog2b);
    v.label_bytes = rd32(h + kHdrLabelBytes);
    v.op_mask = rd32(h + kHdrOpMask);
    v.n_bricks = rd32(h + kHdrNBricks);
    memcpy(v.rans_freq, h + kHdrFreq, 32);
    v.offsets_pos = rd64(h + kHdrOffsetsPos);
    v.dir_pos = rd64(h + kHdrDirPos);
    v.total_bytes = rd64(h + kHdrTotal);
    v.neighbor_mode = rd32(h + kHdrNeighborMode);
    if (v.label_bytes != 4 && v.label_bytes != 8) return fail(CSGV_EINVAL, "label_bytes %u", v.label_bytes);
    if (v.total_bytes > bytes)
        return fail(CSGV_EINVAL, "header claims %llu bytes, only %llu given", (unsigned long long)v.total_bytes,
                    (unsigned long long)bytes);
    if (v.offsets_pos < kHeaderBytes || v.offsets_pos > v.total_bytes ||
        8ull * ((uint64_t)v.n_bricks + 1) > v.total_bytes - v.offsets_pos)
        return fail(CSGV_EINVAL, "offset table outside the container");
    // largest brick side any record claims (sizes the decoder's scratch)
    // and the largest palette (|P|max of cache paletting)
    uint32_t mx = 0, mp = 0;
    for (uint64_t k = 0; k < v.n_bricks; ++k) {
        const uint64_t a = rd64(h + v.offsets_pos + 8 * k), b = rd64(h + v.offsets_pos + 8 * k + 8);
        if (a > b || b > v.total_bytes || b - a < 8) continue;
        const uint32_t L = h[a + 1];
        if (L >= 1 && L <= kMaxLog2b) mx = std::max(mx, L);
        mp = std::max(mp, rd32(h + a + 4));
    }
    v.max_log2b = mx ? mx : 1;
    v.max_palette = mp;
    *out = v;
    return CSGV_OK;
}

}  // extern "C"

namespace {

// Enqueue one call of csgv_decode_bricks on buffers b (scratch of `grid`
// work-groups).
csgv_status decode_on(hipStream_t stream, const csgv_volume_info* vol, const Params& P, const csgv_decode_opts* opts,
                      int mode, int wg, uint32_t grid, const Bufs& b) {
    const bool queue = mode == CSGV_MODE_PERSISTENT, sort = opts ? opts->sort_tasks != 0 : true;
    const hipError_t e = enqueue(P, b, vol, wg, grid, queue, sort, stream, nullptr, nullptr);
    if (e != hipSuccess) return fail(CSGV_EHIP, "decode launch: %s", hipGetErrorString(e));
    return CSGV_OK;
}

// checks shared by both one-shot entry points; fills P, the mode and the shape
csgv_status prepare_call(const csgv_volume_info* vol, const void* d_container, const uint32_t* d_brick_ids,
                         const uint8_t* d_lods, const uint64_t* d_out_offsets, uint32_t n, void* d_out,
                         uint64_t out_capacity, uint32_t* d_status, const csgv_decode_opts* opts, Params* P, int* mode,
                         int* wg, int* per_cu) {
    csgv_status st = check_task_args(vol, d_container, d_brick_ids, d_lods, n, d_out);
    if (st != CSGV_OK || n == 0) return st;  // n = 0 enqueues nothing
    if ((st = check_opts(opts)) != CSGV_OK) return st;
    HIP_TRY(ensure_attrs());
    *mode = opts ? opts->mode : CSGV_MODE_PLAIN;
    if (*mode != CSGV_MODE_PLAIN && *mode != CSGV_MODE_PERSISTENT) return fail(CSGV_EINVAL, "unknown mode %d", *mode);
    *P = make_params(vol, d_container, d_brick_ids, d_lods, d_out_offsets, n, d_out, out_capacity, d_status);
    if (opts && opts->palette_bits > 0) P->pal_bits = (uint32_t)opts->palette_bits;
    *wg = opts && opts->wg_size ? opts->wg_size : 256;
    P->cap16 = std::max<uint32_t>(opts && opts->lds_slots > 0 ? (uint32_t)opts->lds_slots : default_slots(*wg), kMinCap16) & ~7u;
    if (!(opts && (opts->wg_size || opts->lds_slots || opts->wgs_per_cu > 0))) auto_shape(n, wg, &P->cap16);
    *per_cu = opts && opts->wgs_per_cu > 0 ? opts->wgs_per_cu : resident_per_cu(*wg, P->cap16);
    // (in task order more work-groups than the GPU holds only take scratch)
    if (*mode == CSGV_MODE_PLAIN) *per_cu = std::min(*per_cu, resident_per_cu(*wg, P->cap16));
    return CSGV_OK;
}

}  // namespace

extern "C" {

csgv_status csgv_decode_bricks(hipStream_t stream, const csgv_volume_info* vol, const void* d_container,
                               const uint32_t* d_brick_ids, const uint8_t* d_lods, const uint64_t* d_out_offsets,
                               uint32_t n, void* d_out, uint64_t out_capacity, uint32_t* d_status,
                               const csgv_decode_opts* opts) {
    Params P;
    int mode, wg, per_cu;
    csgv_status st = prepare_call(vol, d_container, d_brick_ids, d_lods, d_out_offsets, n, d_out, out_capacity,
                                  d_status, opts, &P, &mode, &wg, &per_cu);
    if (st != CSGV_OK || n == 0) return st;
    // A plain call decodes with any number of work-groups, so it makes do with the
    // memory there is, down to one work-group's scratch.  (It asks for all at first:
    // with half of them 2304 uneven bricks take 2.1 ms instead of 1.4.)
    const bool plain = mode == CSGV_MODE_PLAIN;
    uint32_t grid = (uint32_t)std::min<uint64_t>((uint64_t)device_cus() * per_cu, n);
    void* mem = nullptr;
    uint64_t sb;
    for (;; grid = (grid + 1) / 2) {
        sb = P.scratch_stride * grid;
        const hipError_t e = hipMallocAsync(&mem, sb + aux_bytes(n, !plain), stream);
        if (e == hipSuccess) break;
        (void)hipGetLastError();  // (the next launch asks for it)
        if (!plain || grid == 1 || e != hipErrorOutOfMemory) return fail(CSGV_EHIP, "hipMallocAsync: %s", hipGetErrorString(e));
    }
    Bufs b;
    carve((uint8_t*)mem, sb, n, &b);
    st = decode_on(stream, vol, P, opts, mode, wg, grid, b);
    hipError_t e2 = hipFreeAsync(mem, stream);
    if (st != CSGV_OK) return st;
    if (e2 != hipSuccess) return fail(CSGV_EHIP, "hipFreeAsync: %s", hipGetErrorString(e2));
    return CSGV_OK;
}

csgv_status csgv_check_status(const uint32_t* d_status, uint32_t n, hipStream_t stream) {
    if (n == 0) return CSGV_OK;
    if (!d_status) return fail(CSGV_EINVAL, "NULL status");
    std::vector<uint32_t> h(n);
    HIP_TRY(hipMemcpyAsync(h.data(), d_status, 4ull * n, hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    for (uint32_t j = 0; j < n; ++j)
        if (h[j]) return fail(CSGV_ECORRUPT, "task %u status %u", j, h[j]);
    return CSGV_OK;
}

}  // extern "C"

// ------------------------------------------------------------------ plans
struct csgv_plan {
    csgv_volume_info vol;
    uint32_t max_tasks = 0;
    csgv_decode_opts opts;
    bool auto_shape = false;  // the caller never chose a shape
    uint32_t grid = 0;
    uint64_t scratch_bytes = 0;
    uint8_t* mem = nullptr;
    Bufs b;
    bool timing = false;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    bool ev_valid = false;
};

namespace {

uint32_t plan_grid(const csgv_plan* p, uint32_t n) {
    return std::min<uint32_t>(p->grid, std::max<uint32_t>(n, 1));
}

uint32_t plan_slots(const csgv_plan* p) {
    return p->opts.lds_slots > 0 ? (uint32_t)p->opts.lds_slots : default_slots(p->opts.wg_size);
}

// the shape that a launch of n tasks runs
void plan_shape(const csgv_plan* p, uint32_t n, int* wg, uint32_t* cap16) {
    *wg = p->opts.wg_size;
    *cap16 = std::max<uint32_t>(plan_slots(p), kMinCap16) & ~7u;
    if (p->auto_shape) auto_shape(n, wg, cap16);
}

csgv_status plan_enqueue(csgv_plan* p, hipStream_t s, const Params& P0, bool with_events) {
    Params P = P0;
    P.pal_bits = p->opts.palette_bits > 0 ? (uint32_t)p->opts.palette_bits : 0u;
    int wg;
    plan_shape(p, P.n_tasks, &wg, &P.cap16);
    hipError_t e = enqueue(P, p->b, &p->vol, wg, plan_grid(p, P.n_tasks), true, p->opts.sort_tasks != 0, s,
                           with_events ? p->ev0 : nullptr, with_events ? p->ev1 : nullptr);
    if (e != hipSuccess) return fail(CSGV_EHIP, "plan launch: %s", hipGetErrorString(e));
    return CSGV_OK;
}

// Device memory of a plan for `grid` work-groups: their scratch, and behind it the
// control words, lists, offsets and the volume's rANS table, which is built here
// once for every launch of the plan.
csgv_status plan_take(csgv_plan* p, uint32_t grid, uint64_t sb) {
    hipError_t e = hipMalloc(&p->mem, sb + aux_bytes(p->max_tasks));
    if (e != hipSuccess) {
        (void)hipGetLastError();  // (the next launch asks for it)
        p->mem = nullptr;
        return fail(CSGV_ENOMEM, "plan scratch (%llu bytes): %s", (unsigned long long)sb, hipGetErrorString(e));
    }
    carve(p->mem, sb, p->max_tasks, &p->b);
    p->grid = grid;
    p->scratch_bytes = sb;
    bool ok;
    const RansFreq f = pack_freq(&p->vol, &ok);
    if ((e = launch_prepare(p->b.ctl, ok ? p->b.rans_tab : nullptr, &f, nullptr)) != hipSuccess ||
        (e = hipDeviceSynchronize()) != hipSuccess) {
        (void)hipFree(p->mem);
        p->mem = nullptr;
        return fail(CSGV_EHIP, "rANS table: %s", hipGetErrorString(e));
    }
    p->b.prepared = true;
    return CSGV_OK;
}

// (re)size the plan's grid and scratch for its current shape; when that fails the
// plan takes back the memory it had
csgv_status plan_alloc(csgv_plan* p) {
    const int per_cu = p->opts.wgs_per_cu > 0 ? p->opts.wgs_per_cu : resident_per_cu(p->opts.wg_size, plan_slots(p));
    const uint32_t grid = (uint32_t)std::min<uint64_t>((uint64_t)device_cus() * per_cu, p->max_tasks);
    const uint32_t lmax = p->vol.max_log2b ? std::min<uint32_t>(p->vol.max_log2b, kMaxLog2b) : kMaxLog2b;
    const uint64_t sb = scratch_per_wg(lmax) * grid;
    if (p->mem && grid <= p->grid && sb <= p->scratch_bytes) {
        p->grid = grid;
        return CSGV_OK;
    }
    const uint32_t had = p->mem ? p->grid : 0;
    const uint64_t had_bytes = p->scratch_bytes;
    if (p->mem) {
        (void)hipDeviceSynchronize();
        (void)hipFree(p->mem);
        p->mem = nullptr;
    }
    const csgv_status st = plan_take(p, grid, sb);
    if (st != CSGV_OK && had) {
        const std::string why = g_last_error;
        (void)plan_take(p, had, had_bytes);
        g_last_error = why;
    }
    return st;
}

// Change a plan's options; a work-group size, LDS split or number of work-groups
// that is given ends the choice of the shape by the number of tasks.
csgv_status plan_set(csgv_plan* p, const csgv_decode_opts& o) {
    csgv_status st = check_opts(&o);
    if (st != CSGV_OK) return st;
    const csgv_decode_opts old = p->opts;
    csgv_decode_opts& n = p->opts;
    if (o.wg_size) n.wg_size = o.wg_size;
    if (o.wgs_per_cu >= 0) n.wgs_per_cu = o.wgs_per_cu;
    if (o.sort_tasks >= 0) n.sort_tasks = o.sort_tasks ? 1 : 0;
    if (o.bricks_per_wave > 0) n.bricks_per_wave = o.bricks_per_wave;
    if (o.lds_slots > 0) n.lds_slots = o.lds_slots;
    if (o.palette_bits >= 0) n.palette_bits = o.palette_bits;
    if ((st = plan_alloc(p)) != CSGV_OK) p->opts = old;
    else if (o.wg_size || o.lds_slots > 0 || o.wgs_per_cu > 0) p->auto_shape = false;
    return st;
}

}  // namespace

extern "C" {

csgv_status csgv_plan_create(const csgv_volume_info* vol, uint32_t max_tasks, const csgv_decode_opts* opts,
                             csgv_plan** out) {
    if (!vol || !out) return fail(CSGV_EINVAL, "NULL argument");
    if (max_tasks == 0) return fail(CSGV_EINVAL, "max_tasks must be positive");
    csgv_status st = check_opts(opts);
    if (st != CSGV_OK) return st;
    HIP_TRY(ensure_attrs());
    csgv_plan* p = new csgv_plan();
    p->auto_shape = !(opts && (opts->wg_size || opts->lds_slots || opts->wgs_per_cu > 0));
    p->vol = *vol;
    p->max_tasks = max_tasks;
    p->opts.mode = CSGV_MODE_PERSISTENT;
    p->opts.wg_size = opts && opts->wg_size ? opts->wg_size : 256;
    p->opts.wgs_per_cu = opts && opts->wgs_per_cu > 0 ? opts->wgs_per_cu : 0;
    p->opts.sort_tasks = opts && opts->sort_tasks >= 0 ? opts->sort_tasks : 1;
    p->opts.bricks_per_wave = opts && opts->bricks_per_wave > 0 ? opts->bricks_per_wave : 1;
    p->opts.lds_slots = opts && opts->lds_slots > 0 ? opts->lds_slots : 0;
    p->opts.palette_bits = opts && opts->palette_bits > 0 ? opts->palette_bits : 0;
    if ((st = plan_alloc(p)) != CSGV_OK) {
        csgv_plan_destroy(p);
        return st;
    }
    if (hipEventCreate(&p->ev0) != hipSuccess || hipEventCreate(&p->ev1) != hipSuccess) {
        csgv_plan_destroy(p);
        return fail(CSGV_EHIP, "plan events");
    }
    *out = p;
    return CSGV_OK;
}

csgv_status csgv_plan_set_graph(csgv_plan* p, int enable) {
    (void)enable;
    return p ? CSGV_OK : fail(CSGV_EINVAL, "NULL plan");
}

csgv_status csgv_plan_set_timing(csgv_plan* p, int enable) {
    if (!p) return fail(CSGV_EINVAL, "NULL plan");
    p->timing = enable != 0;
    return CSGV_OK;
}

csgv_status csgv_plan_set_opts(csgv_plan* p, const csgv_decode_opts* o) {
    if (!p || !o) return fail(CSGV_EINVAL, "NULL argument");
    // the shape that the plan reports, handed back, is no choice of a shape
    csgv_decode_opts now, n = *o;
    (void)csgv_plan_get_opts(p, &now);
    if (o->wg_size == now.wg_size && o->lds_slots == now.lds_slots && o->wgs_per_cu == now.wgs_per_cu) {
        n.wg_size = n.lds_slots = 0;
        n.wgs_per_cu = -1;
    }
    return plan_set(p, n);
}

csgv_status csgv_plan_launch(csgv_plan* p, hipStream_t stream, const void* d_container, const uint32_t* d_brick_ids,
                             const uint8_t* d_lods, const uint64_t* d_out_offsets, uint32_t n, void* d_out,
                             uint64_t out_capacity, uint32_t* d_status) {
    if (!p) return fail(CSGV_EINVAL, "NULL plan");
    csgv_status st = check_task_args(&p->vol, d_container, d_brick_ids, d_lods, n, d_out);
    if (st != CSGV_OK) return st;
    if (n == 0) return CSGV_OK;
    if (n > p->max_tasks) return fail(CSGV_EINVAL, "n = %u exceeds the plan's max_tasks = %u", n, p->max_tasks);
    if (!p->mem) return fail(CSGV_ENOMEM, "the plan lost its scratch to a change of shape that did not fit");
    Params P = make_params(&p->vol, d_container, d_brick_ids, d_lods, d_out_offsets, n, d_out, out_capacity, d_status);
    st = plan_enqueue(p, stream, P, p->timing);
    p->ev_valid = st == CSGV_OK && p->timing;
    return st;
}

csgv_status csgv_plan_get_opts(const csgv_plan* p, csgv_decode_opts* out) {
    if (!p || !out) return fail(CSGV_EINVAL, "NULL argument");
    *out = p->opts;
    uint32_t cap16;
    plan_shape(p, p->max_tasks, &out->wg_size, &cap16);
    if (p->opts.lds_slots == 0) out->lds_slots = (int)cap16;
    if (out->wgs_per_cu == 0) out->wgs_per_cu = (int)(p->grid / std::max(1, device_cus()));
    return CSGV_OK;
}

csgv_status csgv_plan_last_kernel_ms(csgv_plan* p, float* ms) {
    if (!p || !ms) return fail(CSGV_EINVAL, "NULL argument");
    if (!p->ev_valid) return fail(CSGV_EINVAL, "no timed launch recorded (enable timing first)");
    HIP_TRY(hipEventSynchronize(p->ev1));
    HIP_TRY(hipEventElapsedTime(ms, p->ev0, p->ev1));
    return CSGV_OK;
}

void csgv_plan_destroy(csgv_plan* p) {
    if (!p) return;
    if (p->ev0) (void)hipEventDestroy(p->ev0);
    if (p->ev1) (void)hipEventDestroy(p->ev1);
    if (p->mem) (void)hipFree(p->mem);
    delete p;
}

void csgv_free_host(void* p) { free(p); }

}  // extern "C"

// ------------------------------------------------------------------ autotuner
namespace {

std::string tune_key(const csgv_plan* p, const std::vector<uint8_t>& lods, uint32_t n) {
    int dev = 0;
    hipDeviceProp_t prop;
    std::string arch = "unknown";
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) {
        arch = prop.gcnArchName;
        const size_t colon = arch.find(':');
        if (colon != std::string::npos) arch = arch.substr(0, colon);
    }
    uint32_t hist[8] = {0};
    for (uint8_t l : lods) ++hist[l < 7 ? l : 7];
    char buf[512];
    snprintf(buf, sizeof(buf), "%s|cus=%d|lb=%u|L=%u|bricks=%u|bytes=%llu|n=%u|lods=%u,%u,%u,%u,%u,%u,%u,%u|I=%d",
             arch.c_str(), device_cus(), p->vol.label_bytes, p->vol.max_log2b, p->vol.n_bricks,
             (unsigned long long)p->vol.total_bytes, n, hist[0], hist[1], hist[2], hist[3], hist[4], hist[5],
             hist[6], hist[7], p->opts.palette_bits);
    return buf;
}

bool tune_lookup(const char* path, const std::string& key, csgv_decode_opts* o) {
    if (!path) return false;
    FILE* f = fopen(path, "r");
    if (!f) return false;
    char line[1024];
    bool found = false;
    while (fgets(line, sizeof(line), f)) {
        char* tab = strchr(line, '\t');
        if (!tab) continue;
        *tab = 0;
        int wg, lds, wpc;
        if (key == line && sscanf(tab + 1, "%d %d %d", &wg, &lds, &wpc) == 3) {
            o->wg_size = wg;
            o->lds_slots = lds;
            o->wgs_per_cu = wpc;
            found = true;  // the last matching line wins
        }
    }
    fclose(f);
    return found;
}

void tune_store(const char* path, const std::string& key, const csgv_decode_opts& o) {
    if (!path) return;
    FILE* f = fopen(path, "a");
    if (!f) return;
    fprintf(f, "%s\t%d %d %d\n", key.c_str(), o.wg_size, o.lds_slots, o.wgs_per_cu);
    fclose(f);
}

}  // namespace

extern "C" csgv_status csgv_plan_autotune(csgv_plan* p, hipStream_t stream, const void* d_container,
                                          const uint32_t* d_brick_ids, const uint8_t* d_lods,
                                          const uint64_t* d_out_offsets, uint32_t n, void* d_out,
                                          uint64_t out_capacity, uint32_t* d_status, const char* cache_path,
                                          csgv_tune_report* report) {
    if (!p) return fail(CSGV_EINVAL, "NULL plan");
    csgv_status st = check_task_args(&p->vol, d_container, d_brick_ids, d_lods, n, d_out);
    if (st != CSGV_OK) return st;
    if (n == 0 || n > p->max_tasks) return fail(CSGV_EINVAL, "n = %u (plan max_tasks %u)", n, p->max_tasks);
    std::vector<uint8_t> lods(n);
    HIP_TRY(hipMemcpyAsync(lods.data(), d_lods, n, hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    const std::string key = tune_key(p, lods, n);
    csgv_tune_report rep;
    memset(&rep, 0, sizeof(rep));
    csgv_decode_opts cached = p->opts;
    if (tune_lookup(cache_path, key, &cached)) {
        if ((st = plan_set(p, cached)) != CSGV_OK) return st;
        rep.from_cache = 1;
        rep.chosen = p->opts;
        if (report) *report = rep;
        return CSGV_OK;
    }
    const bool had_timing = p->timing;
    p->timing = true;
    const csgv_decode_opts start = p->opts;
    auto time_shape = [&](const csgv_decode_opts& o, float* best) -> csgv_status {
        csgv_status s2 = plan_set(p, o);
        if (s2 != CSGV_OK) return s2;
        *best = 1e30f;
        for (int rep_i = 0; rep_i < 4; ++rep_i) {
            s2 = csgv_plan_launch(p, stream, d_container, d_brick_ids, d_lods, d_out_offsets, n, d_out, out_capacity,
                                  d_status);
            if (s2 != CSGV_OK) return s2;
            float ms = 0;
            if ((s2 = csgv_plan_last_kernel_ms(p, &ms)) != CSGV_OK) return s2;
            if (rep_i > 0) *best = std::min(*best, ms);  // the first launch of a shape warms caches
        }
        return CSGV_OK;
    };
    static const int kWg[] = {128, 256, 512};
    static const int kLds[] = {8192, 10240, 16384, 24576};
    int wg0 = 256;  // the default shape of n tasks, one of those tried
    uint32_t lds0 = kDefaultCap16;
    auto_shape(n, &wg0, &lds0);
    float best_ms = 1e30f;
    csgv_decode_opts best = start;
    int tried = 0;
    for (int wg : kWg)
        for (int lds : kLds) {
            csgv_decode_opts o = start;
            o.wg_size = wg;
            o.lds_slots = lds;
            o.wgs_per_cu = 0;
            float ms;
            st = time_shape(o, &ms);
            if (st != CSGV_OK) {
                p->timing = had_timing;
                return st;
            }
            ++tried;
            if (wg == wg0 && lds == (int)lds0) rep.default_ms = ms;
            if (ms < best_ms) {
                best_ms = ms;
                best = o;
            }
        }
    p->timing = had_timing;
    if ((st = plan_set(p, best)) != CSGV_OK) return st;
    tune_store(cache_path, key, best);
    rep.tried = tried;
    rep.best_ms = best_ms;
    rep.chosen = p->opts;
    if (report) *report = rep;
    return CSGV_OK;
}

// ------------------------------------------------- decode without allocating
// Scratch of csgv_decode_bricks_noalloc: one array per GPU the library runs
// on, held until the process ends.  Host code uses it only through the device
// address hipGetSymbolAddress returns on each device (the array's name is a
// host-side stand-in there).
static __device__ __align__(256) uint8_t scratch[CSGV_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
uint8_t* g_noalloc_base[kMaxDevices] = {};

// device address of this GPU's array, looked up once per device
csgv_status noalloc_base(uint8_t** out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(CSGV_EINVAL, "device %d beyond the supported %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    if (!g_noalloc_base[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        g_noalloc_base[dev] = (uint8_t*)p;
    }
    *out = g_noalloc_base[dev];
    return CSGV_OK;
}

}  // namespace

extern "C" {

csgv_status csgv_decode_bricks_noalloc(hipStream_t stream, const csgv_volume_info* vol, const void* d_container,
                                       const uint32_t* d_brick_ids, const uint8_t* d_lods,
                                       const uint64_t* d_out_offsets, uint32_t n, void* d_out, uint64_t out_capacity,
                                       uint32_t* d_status, const csgv_decode_opts* opts) {
    Params P;
    int mode, wg, per_cu;
    csgv_status st = prepare_call(vol, d_container, d_brick_ids, d_lods, d_out_offsets, n, d_out, out_capacity,
                                  d_status, opts, &P, &mode, &wg, &per_cu);
    if (st != CSGV_OK || n == 0) return st;
    if (n > CSGV_NOALLOC_MAX_TASKS)
        return fail(CSGV_EINVAL, "n = %u exceeds the %u tasks of the fixed scratch", n, (uint32_t)CSGV_NOALLOC_MAX_TASKS);
    // per-task arrays for CSGV_NOALLOC_MAX_TASKS after the work-groups' scratch
    const uint64_t aux = aux_bytes(CSGV_NOALLOC_MAX_TASKS);
    const uint64_t sb = (CSGV_NOALLOC_SCRATCH_BYTES - aux) / 256 * 256;
    const uint64_t fit = sb / P.scratch_stride;
    if (fit == 0)
        return fail(CSGV_EINVAL, "records of brick side 2^%u need %llu scratch bytes per work-group, more than the "
                    "fixed scratch holds", P.max_log2b, (unsigned long long)P.scratch_stride);
    const uint32_t grid = (uint32_t)std::min<uint64_t>(std::min<uint64_t>((uint64_t)device_cus() * per_cu, n), fit);
    uint8_t* base = nullptr;
    if ((st = noalloc_base(&base)) != CSGV_OK) return st;
    Bufs b;
    carve(base, sb, CSGV_NOALLOC_MAX_TASKS, &b);
    return decode_on(stream, vol, P, opts, mode, wg, grid, b);
}

}  // extern "C"
