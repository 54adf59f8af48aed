// CSGV brick decoder for gfx950 (MI355X).
//
// A work-group decodes one task = (brick id, LOD, output offset): it rebuilds
// the brick's multi-resolution levels coarse to fine and writes the level of
// the requested LOD as a cube of labels, linear with x fastest (paper:
// Results > "CSGV" for the encoding -- one operation per explicit node of the
// multi-resolution grid, copying from the parent, a neighbour or the palette,
// with stop bits for all-constant children; Methods > "GPU rendering
// pipeline" for the decode stage; Methods > "Memory management" for LODs).
//
// The kernel is bound by instruction issue and by the serial chain of a task's
// phases, not by memory (a 32^3 brick is about 3 KB read and 128 KB written): 4096
// Voronoi bricks run at 56 % VALU busy, and the output is written at about 2.6 TB/s.
// A 32^3 cube at full resolution takes 100k cycles with four work-groups of 256
// threads on a CU: 9k staging, 25k rANS rounds and levels 0..3, 18k level 4, 34k
// level 5, 10k output.  That is why the levels are decoded by expanding parents,
// with no work for nodes that are implied.
//
// Storage of the levels of a task (node order within a level is Morton; the k-th
// operation of a level is its k-th explicit node):
//   levels 0..4   full grids in LDS (4681 nodes), and bitmaps of the nodes that
//                 expand, with a popcount prefix;
//   level 5       explicit nodes only, by operation rank: 8 slots, a row, for
//                 every expanding parent, found through the rank of the parent
//                 in the level-4 bitmap.  In LDS when the rows fit there (32^3
//                 cubes), else palette indices in the work-group's scratch;
//   level 6       (64^3 bricks at full resolution) nowhere: labels go straight to
//                 the task's output, from which later nodes copy.
// A level is decoded in two steps.  ops_pass ranks the level's symbols: a thread
// takes up to four words of eight 4-bit symbols, summarises them for both entry
// states of the automaton (inside a chain of delta entries or not), and one scan
// and one barrier give it its state, its first operation rank and its palette
// (ADV) rank; it writes each operation's slot, a palette index or a copy's code.
// Then a thread per expanding parent turns the 8 slots of its children into
// values or references to slots of the same level (resolve8), and the references
// are followed (chase_open), which ends because every target precedes its source
// in Morton order.  Levels 1 and 2 take a lane per symbol and per node instead.
//   Levels whose rows do not fit in LDS, and level 6, do the same in chunks of a
// 32-bit buffer in LDS, parent by parent as their operations are complete
// (chunk_level).
//
// rANS-coded records are first decoded into 4-bit symbols: every 64-lane group of
// the interleaved coder is one wavefront, and the lanes that renormalise in a
// round find their word offsets with a ballot and a masked bit count.  Words,
// decoding table and symbols are all in LDS where they fit, as those of nearly
// every 32^3 record do; longer streams go through a ring (rans_stream).
//
// Levels 0..3 (at most 585 nodes) are decoded by one wavefront, while the others
// still decode symbols if there is one to spare; meanwhile lane 0 of the last
// wavefront parses the work-group's next task (claimed when the current one
// started) into a second header.  Cubes of side <= 8 are decoded by single
// wavefronts throughout (wave_tasks).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "csgv_format.h"
#include "decode_kernel.h"

namespace csgv {

// ------------------------------------------------------------------ layout
// full grids of levels 0..4 at these slot offsets (8-aligned for 16-byte fills)
__device__ __forceinline__ uint32_t fbase(uint32_t i) {
    return i == 0 ? 0u : i == 1 ? 8u : i == 2 ? 16u : i == 3 ? 80u : 592u;
}
// expansion bitmaps of levels 0..4 at these word offsets
__device__ __forceinline__ uint32_t ebase(uint32_t i) {
    return i == 0 ? 0u : i == 1 ? 1u : i == 2 ? 2u : i == 3 ? 4u : 20u;
}
__host__ __device__ constexpr uint32_t ewords(uint32_t i) { return i <= 1 ? 1u : i == 2 ? 2u : (1u << (3 * i - 5)); }

// header words of a record: w0, palette count, sym_end[0..L], up to 4 group word counts
constexpr uint32_t kHdrWords = 2 + 7 + 4;

struct TaskHdr {
    uint32_t hw[kHdrWords];  // the record's first words (parse_task)
    uint32_t task, status, write_ok, coder, L, t, log2W, pc, nsym;
    uint32_t sym_end[7];
    uint32_t gw[4], gstart[4];
    uint64_t out_off, pal_off, pay_off, states_off;
};

// Fixed part of a work-group's LDS; the parent list / palette area (u_bytes) and
// the slot area follow it.
struct Shared {
    TaskHdr h;   // the task being decoded
    TaskHdr hn;  // the work-group's next task, parsed ahead
    uint32_t err;
    uint32_t tab_ok;                // the rANS table is in LDS from an earlier task
    uint32_t prog[4];               // per rANS lane group: symbols out so far (release/acquire)
    uint32_t nexp;                  // expanding nodes of the parent level of the next level
    uint32_t adv;                   // PALETTE_ADV operations decoded so far (handed between phases)
    uint32_t n_jobs;                // tasks of the launch for work-groups, and of each of its lists
    uint32_t small[2];              // claims on the lists for single wavefronts, this one and the next
    uint32_t job[kClasses];
    alignas(16) uint16_t refs[64];  // open slots of level 3
    alignas(16) uint4 pub[2][kMaxWaves];  // per pass and wave: run summary (exit states, counts)
    alignas(16) uint2 EP[kEWords];        // expansion bitmaps of levels 0..4: bits, prefix
    alignas(16) uint16_t G[kFullSlots];   // full grids of levels 0..4
};
static_assert(sizeof(Shared) % 16 == 0, "the areas behind Shared are 16-byte aligned");
static_assert(sizeof(TaskHdr) % 4 == 0 && sizeof(TaskHdr) / 4 <= 128, "a header is copied one word per thread");
static_assert(offsetof(Shared, G) + sizeof(Shared::G) == sizeof(Shared),
              "grids, parent list and slot area form one range (rANS staging)");

// ------------------------------------------------------ wave/block helpers
__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }
// The launch's parameters, read again from the kernel arguments: held in scalar
// registers over the whole kernel they push loop masks and counters out of them
// (spills to vector lanes).  Every phase takes its own.
__device__ __forceinline__ const Params& params() {
    auto p = (const __attribute__((address_space(4))) Params*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const Params*)p;
}

// a value that is the same in every lane of the wavefront, in a scalar register
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint64_t uni64(uint64_t v) { return ((uint64_t)uni((uint32_t)(v >> 32)) << 32) | uni((uint32_t)v); }
__device__ __forceinline__ uint32_t wave_id() { return uni(threadIdx.x >> 6); }

__device__ __forceinline__ uint32_t mbcnt(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint32_t spread3(uint32_t v) {
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}
__device__ __forceinline__ uint32_t compact3(uint32_t v) {
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030C30C3u;
    v = (v | (v >> 4)) & 0x0300F00Fu;
    v = (v | (v >> 8)) & 0x030000FFu;
    v = (v | (v >> 16)) & 0x000003FFu;
    return v;
}

// Work-group barrier for data exchanged through LDS: outstanding global stores
// and loads are not waited for.  Data exchanged through global memory takes
// __syncthreads().
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Barrier of the threads that decode a level: the work-group, or (NT = 64) one
// wavefront alone, whose LDS accesses complete in order.
template <int NT>
__device__ __forceinline__ void lsync() {
    if (NT == 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        lds_barrier();
    }
}

// DPP moves (GFX9 controls).  A lane whose source lane does not exist, or
// whose row is masked off, keeps `old`.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xF, false);
}
constexpr int kDppRowShr = 0x110;   // + n: lane l takes lane l - n of its row of 16
constexpr int kDppBcast15 = 0x142;   // rows 1, 3 take lane 15 of the row before
constexpr int kDppBcast31 = 0x143;   // rows 2, 3 take lane 31

// inclusive sum over the wavefront (lane 0 first)
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t x) {
    x += dpp<kDppRowShr + 1>(0u, x);
    x += dpp<kDppRowShr + 2>(0u, x);
    x += dpp<kDppRowShr + 4>(0u, x);
    x += dpp<kDppRowShr + 8>(0u, x);
    x += dpp<kDppBcast15, 0xA>(0u, x);
    x += dpp<kDppBcast31, 0xC>(0u, x);
    return x;
}

// -------------------------------------------------------------- palette
// Palette entry idx: staged in LDS (PAL_LDS) or read from the record.  LT is
// the label type (u32 or u64); a global read is bounded by the palette count.
template <typename LT, bool PAL_LDS>
__device__ __forceinline__ LT pal_get(const LT* pal, uint32_t idx, uint32_t pc) {
    if (PAL_LDS) return pal[idx];
    return idx < pc ? pal[idx] : (LT)0;
}

// -------------------------------------------------------------- task parse
__device__ __forceinline__ uint32_t ld32(const uint8_t* p) { return *(const uint32_t*)p; }

// Validate task j and its record with the same checks, in the same order, as
// the CPU decoder; fills the header (thread 0 only).
__device__ __forceinline__ void parse_task(const Params& P, uint32_t task, TaskHdr& h) {
    h.task = task;
    h.status = kTaskOk;
    h.write_ok = 0;
    const uint32_t id = P.ids[task];
    const uint32_t lod = P.lods[task];
    const uint64_t out_off = P.out_offs ? P.out_offs[task] : P.dense_base[task / kBinTasks] + P.dense_offs[task];
    h.out_off = out_off;
    if (id >= P.n_bricks) { h.status = kTaskInvalid; return; }
    const uint64_t* offs = (const uint64_t*)(P.vol + P.off_pos);
    const uint64_t a = offs[id], b = offs[id + 1];
    if (a > b || b > P.vol_bytes || (a & 7) || b - a < 8) { h.status = kTaskCorrupt; return; }
    const uint8_t* rec = P.vol + a;
    const uint64_t extent = b - a;
    // the record's first kHdrWords words (more than any header holds) are loaded
    // at once, at offsets clamped into the record; the checks below use a word
    // only after placing it inside the header
    {
        const uint64_t last = (extent & ~3ull) - 4u;
#pragma unroll
        for (uint32_t k = 0; k < kHdrWords; ++k) h.hw[k] = ld32(rec + (4u * k < last ? 4u * k : last));
    }
    const uint32_t w0 = h.hw[0];
    const uint32_t coder = w0 & 0xFF, L = (w0 >> 8) & 0xFF, lb = (w0 >> 16) & 0xFF, log2W = w0 >> 24;
    const uint32_t pc = h.hw[1];
    // (a record larger than every brick the container was parsed with cannot
    // occur for the parsed bytes; it is refused because scratch is sized by them)
    if (L < 1 || L > kMaxLog2b || L > P.max_log2b) { h.status = kTaskCorrupt; return; }
    if (lod > L) { h.status = kTaskInvalid; return; }
    const uint32_t t = L - lod;
    const uint64_t S = 1ull << t, n_out = out_units(S * S * S, P.pal_bits);
    if (out_off > P.out_cap || n_out > P.out_cap - out_off) { h.status = kTaskInvalid; return; }
    h.write_ok = 1;
    h.L = L;
    h.t = t;
    if (lb != P.label_bytes || coder > 1 || (coder == kRaw4 && log2W != 0) || (coder == kRans && log2W > 8)) {
        h.status = kTaskCorrupt;
        return;
    }
    const uint64_t hdr = record_header_bytes(L, coder, log2W);
    if (hdr > extent) { h.status = kTaskCorrupt; return; }
    const uint64_t al = lb == 8 ? 8 : 4;
    const uint64_t pal_rel = (hdr + al - 1) / al * al;
    if (pal_rel > extent || (uint64_t)pc * lb > extent - pal_rel) { h.status = kTaskCorrupt; return; }
    const uint64_t pay_rel = pal_rel + (uint64_t)pc * lb;
    const uint64_t pay_bytes = extent - pay_rel;
    uint32_t prev = 0;
    for (uint32_t i = 0; i <= L; ++i) {
        const uint32_t e = h.hw[2 + i];
        h.sym_end[i] = e;
        if (i > 0 && e < prev) { h.status = kTaskCorrupt; return; }
        prev = e;
    }
    if ((uint64_t)prev > 8 * total_nodes(L)) { h.status = kTaskCorrupt; return; }
    if (coder == kRaw4) {
        if ((uint64_t)prev > 2 * pay_bytes) { h.status = kTaskCorrupt; return; }
    } else {
        const uint32_t W = 1u << log2W, G = (W + 63) / 64;
        uint64_t tw = 0;
        for (uint32_t g = 0; g < G; ++g) {
            const uint32_t c = h.hw[3 + L + g];
            h.gw[g] = c;
            h.gstart[g] = (uint32_t)tw;
            tw += c;
        }
        if (2 * tw > pay_bytes) { h.status = kTaskCorrupt; return; }
        if (!P.freq_ok) { h.status = kTaskCorrupt; return; }
        h.states_off = a + 8 + 4 * (L + 1) + 4 * G;
    }
    h.coder = coder;
    h.log2W = log2W;
    h.pc = pc;
    h.pal_off = a + pal_rel;
    h.pay_off = a + pay_rel;
    h.nsym = h.sym_end[t];
    // cache-paletted output: a palette beyond 2^I entries, or a 64^3 cube, has no packed form
    if (P.pal_bits && (t == 6 || (uint64_t)pc > (1ull << P.pal_bits))) {
        h.status = kTaskInvalid;
        h.write_ok = 0;
    }
}


// The work-group's next task: claimed by lane 0 of its last wavefront (jt, in
// that lane's register) when a task starts, and parsed into sh.hn by the same
// lane while that wavefront has nothing else to do (levels 0..3 are decoded by
// one wavefront alone), else at the end of the task.
struct Ahead {
    uint32_t jt;
    bool done;
};

// (The claim's result is waited for here, not where it was claimed.)
__device__ __forceinline__ void parse_ahead(const Params& P, Shared& sh, uint32_t jt) {
    TaskHdr& hn = sh.hn;
    const uint32_t n = sh.n_jobs;
    if (jt >= n) {
        hn.task = 0xFFFFFFFFu;
        // (the work-group's first claim on the other lists, while its last task is decoded)
        if (P.lists) sh.small[0] = n ? atomicAdd(&P.ctl->small, 1u) : blockIdx.x;
        return;
    }
    uint32_t task = jt;
    if (P.lists) {  // the jt-th task over the classes' lists
        uint32_t c = 0;
        for (; c < kClasses - 1u && jt >= sh.job[c]; ++c) jt -= sh.job[c];
        task = P.lists[(uint64_t)c * P.list_cap + jt];
    }
    parse_task(params(), task, hn);
}

// The next claim of a work-group after jt; its first task is its own number.
// (Claims of all work-groups on the one counter take 9 ns each.)
__device__ __forceinline__ uint32_t claim(const Params& P, const Shared& sh, uint32_t jt) {
    if (jt >= sh.n_jobs) return jt;
    return gridDim.x + (P.ctl ? atomicAdd(&P.ctl->queue, 1u) : jt);
}

// ----------------------------------------------------------------- rANS
// Decode the first h.nsym symbols of the record into 4-bit symbols at nib[]
// (low nibble first).  Wavefront w handles lane groups w, w + NW, ...  A
// group's words sit in a 192-word register window; the third 64-word block is
// fetched as soon as the window moves, one window move before it is needed.
template <int NT, typename SH>
__device__ __forceinline__ void rans_decode(const Params& P, SH& sh, const uint32_t* tab, uint8_t* nib) {
    const TaskHdr& h = sh.h;
    const uint32_t lane = lane_id(), wave = NT == 64 ? 0u : wave_id();
    const uint32_t W = 1u << uni(h.log2W), G = (W + 63) / 64, lanes = W < 64 ? W : 64;
    const uint32_t nsym = uni(h.nsym);
    const uint16_t* words = (const uint16_t*)(P.vol + uni64(h.pay_off));
    const uint32_t* states = (const uint32_t*)(P.vol + uni64(h.states_off));
    for (uint32_t g = wave; g < G; g += NT / 64) {
        const bool active = lane < lanes;
        const uint32_t gl = 64 * g + lane;
        const uint32_t gcount = uni(h.gw[g]), gbase = uni(h.gstart[g]);
        uint32_t x = active ? states[gl] : 0u;
        uint32_t wbase = 0;
        uint32_t win0 = lane < gcount ? words[gbase + lane] : 0u;
        uint32_t win1 = 64 + lane < gcount ? words[gbase + 64 + lane] : 0u;
        uint32_t win2 = 128 + lane < gcount ? words[gbase + 128 + lane] : 0u;
        uint32_t gpos = 0, pend = 0;
        bool bad = false;
        // the loop-carried state and window start from loads: let them land here,
        // or every round would wait for all outstanding memory operations
        __builtin_amdgcn_s_waitcnt(0);
        for (uint32_t r0 = 64 * g; r0 < nsym; r0 += W) {
            const uint32_t j = r0 + lane;
            const bool act = active && j < nsym;
            uint32_t s = 0;
            if (act) {
                const uint32_t e = tab[x & (kRansM - 1)];
                s = e & 15u;
                x = ((e >> 4) & 0x1FFFu) * (x >> kRansBits) + (e >> 17);
            }
            const bool need = act && x < kRansL;
            const uint64_t m = __ballot(need);
            const uint32_t widx = gpos + mbcnt(m);
            const uint32_t rel = widx - wbase;  // < 128: at most 64 words per round, gpos - wbase < 64
            const uint32_t v0 = __shfl(win0, rel & 63, 64), v1 = __shfl(win1, rel & 63, 64);
            if (need) {
                if (widx >= gcount) bad = true;
                x = (x << 16) | (rel < 64 ? v0 : v1);
            }
            gpos += (uint32_t)__popcll(m);
            // two consecutive symbols per output byte
            if (W >= 2) {
                const uint32_t hi = __shfl_xor(s, 1, 64);
                if (act && !(lane & 1)) nib[j >> 1] = (uint8_t)(s | (j + 1 < nsym ? hi << 4 : 0u));
            } else if (lane == 0) {
                if (!(j & 1)) {
                    pend = s;
                    if (j + 1 == nsym) nib[j >> 1] = (uint8_t)pend;
                } else {
                    nib[j >> 1] = (uint8_t)(pend | (s << 4));
                }
            }
            if (gpos - wbase >= 64) {
                wbase += 64;
                win0 = win1;
                win1 = win2;
                const uint32_t p = wbase + 128 + lane;
                win2 = p < gcount ? words[gbase + p] : 0u;
            }
        }
        if (__ballot(bad) && lane == 0) atomicOr(&sh.err, 1u);
    }
}

// The same for streams that do not fit in LDS whole and 64 lanes or more: every
// wavefront keeps the next words of its lane group in a ring of 512 in LDS,
// refilled by halves that were loaded one refill ahead, and hands its symbols
// to scratch by eight rounds, so a round is as long as with everything staged
// (330 cycles; 800 with a register window, two bpermutes and a byte store to
// global memory in each).
constexpr uint32_t kRing = 512, kStreamBytes = 2u * kRing + 256u;  // LDS of a wavefront
typedef uint32_t u32x2_a4 __attribute__((vector_size(8), aligned(4)));
template <int NT>
__device__ __forceinline__ void rans_stream(const Params& P, Shared& sh, const uint32_t* tab, uint8_t* lds, uint8_t* nib) {
    const TaskHdr& h = sh.h;
    const uint32_t lane = lane_id(), wave = wave_id();
    const uint32_t W = 1u << uni(h.log2W), G = W / 64u, nsym = uni(h.nsym);
    const uint32_t* states = (const uint32_t*)(P.vol + uni64(h.states_off));
    uint16_t* const ring = (uint16_t*)(lds + wave * kStreamBytes);
    uint8_t* const buf = (uint8_t*)(ring + kRing);
    // reads stay inside the container; what lies past it only feeds what the word
    // count at the end refuses
    const uint64_t pay = uni64(h.pay_off), avail = P.vol_bytes - pay;
    for (uint32_t g = wave; g < G; g += NT / 64) {
        const uint32_t gcount = uni(h.gw[g]), start = uni(h.gstart[g]), odd = start & 1u;
        const uint8_t* const src = P.vol + pay;
        // words 256 k .. 256 k + 255 of the group's stream (from its even start), 4 per lane
        auto fetch = [&](uint32_t k) -> uint2 {
            const uint64_t o = 2ull * (start & ~1u) + 512ull * k + 8u * lane;
            if (o + 8u <= avail) {
                const u32x2_a4 v = *(const u32x2_a4*)(src + o);
                return make_uint2(v[0], v[1]);
            }
            uint32_t q[4];  // the container's last words
#pragma unroll
            for (uint32_t c = 0; c < 4; ++c) q[c] = o + 2u * c + 2u <= avail ? *(const uint16_t*)(src + o + 2u * c) : 0u;
            return make_uint2(q[0] | (q[1] << 16), q[2] | (q[3] << 16));
        };
        uint32_t x = states[64 * g + lane];
        uint2 a = fetch(0), b = fetch(1), ahead = fetch(2);
        ((uint2*)ring)[lane] = a;
        ((uint2*)ring)[64u + lane] = b;
        uint32_t pos = odd, loaded = 2, r0 = 64u * g, n = 0;
        lsync<64>();
        __builtin_amdgcn_s_waitcnt(0);
        auto flush = [&] {  // the symbols of the last n <= 8 rounds
            lsync<64>();
            const uint32_t r = lane >> 3, j = r0 - (n - r) * W + 8u * (lane & 7u);
            if (r < n && j < nsym) *(uint32_t*)(nib + j / 2u) = ((const uint32_t*)buf)[lane];
            lsync<64>();
            n = 0;
        };
        for (; r0 < nsym; r0 += W) {
            if (pos + 64u > 256u * loaded) {
                ((uint2*)ring)[64u * (loaded & 1u) + lane] = ahead;
                ++loaded;
                ahead = fetch(loaded);
                lsync<64>();
            }
            const bool act = r0 + lane < nsym;
            const uint32_t e = tab[x & (kRansM - 1)];
            const uint32_t xd = ((e >> 4) & 0x1FFFu) * (x >> kRansBits) + (e >> 17);
            const bool need = act && xd < kRansL;
            const uint64_t m = __ballot(need);
            uint32_t wv = ring[(pos + mbcnt(m)) & (kRing - 1u)];
            asm volatile("" : "+v"(wv));
            x = need ? ((xd << 16) | wv) : act ? xd : x;
            pos += (uint32_t)__popcll(m);
            const uint32_t s = e & 15u;
            buf[32u * n + (lane >> 1)] = (uint8_t)(dpp<0xA0>(0u, s) | (dpp<0xF5>(0u, s) << 4));
            if (++n == 8u) {
                r0 += W;
                flush();
                r0 -= W;
            }
        }
        if (n) flush();
        if (pos - odd > gcount && lane == 0) atomicOr(&sh.err, 1u);
    }
}

// Copy the record's rANS words into LDS at `wl` and, with `tab`, the decoding
// table (no barrier); returns this thread's state for its wavefront's first
// lane group.  All loads are issued before the first one is waited for: the
// words of a typical 32^3 record are one 16-byte load per thread.
typedef uint32_t u32x4_a4 __attribute__((vector_size(16), aligned(4)));
template <int NT>
__device__ __forceinline__ uint32_t rans_stage(const Params& P, const TaskHdr& h, uint16_t* wl, uint32_t wl_bytes, uint4* tab) {
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    const uint32_t W = 1u << uni(h.log2W), G = (W + 63) / 64, lanes = W < 64 ? W : 64;
    const uint8_t* const src = P.vol + uni64(h.pay_off);
    const uint32_t* states = (const uint32_t*)(P.vol + uni64(h.states_off));
    constexpr uint32_t TN = kRansM / 4 / NT;
    const uint32_t x0 = wave < G && lane < lanes ? states[64 * wave + lane] : 0u;
    const bool wide = uni64(h.pay_off) + wl_bytes <= P.vol_bytes;  // (wl_bytes is rounded up to 16)
    u32x4_a4 first = {0u, 0u, 0u, 0u};
    if (wide && 16u * tid < wl_bytes) first = *(const u32x4_a4*)(src + 16u * tid);
    if (tab) {
        uint4 t[TN];
#pragma unroll
        for (uint32_t k = 0; k < TN; ++k) t[k] = ((const uint4*)P.rans_tab)[k * NT + tid];
#pragma unroll
        for (uint32_t k = 0; k < TN; ++k) tab[k * NT + tid] = t[k];
    }
    if (wide) {
        if (16u * tid < wl_bytes) ((uint4*)wl)[tid] = make_uint4(first[0], first[1], first[2], first[3]);
        for (uint32_t q = tid + NT; 16u * q < wl_bytes; q += NT) {
            const u32x4_a4 v = *(const u32x4_a4*)(src + 16u * q);
            ((uint4*)wl)[q] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    } else {
        const uint32_t tw = uni(h.gstart[G - 1]) + uni(h.gw[G - 1]);
        for (uint32_t q = tid; q < tw; q += NT) wl[q] = ((const uint16_t*)src)[q];
    }
    return x0;
}

// The rounds of the decode from words staged in LDS at `wl` (after a barrier),
// symbols written to LDS at `nl`: a lane that renormalises reads its word from
// LDS, and no round waits on a global store.  Wavefront w decodes lane groups
// w, w + NW, ...  With `mark`, lane 0 publishes in sh.prog[g], with release
// order, that group g's symbols below index `mark` are out as soon as they are
// (its next round would start at or past `mark`), and ~0 when the group is done.
// A round is a serial chain (table, multiply, ballot, word, next state), so what
// counts is its length: a round of all lanes has no lane checks, and a
// group that consumes more words than it has is found out at its end (the word
// index is held inside the staged words plus one round).
template <int NT, typename SH>
__device__ __forceinline__ void rans_rounds(const Params& P, SH& sh, const uint32_t* tab, const uint16_t* wl,
                                            uint8_t* nl, uint32_t x0, uint32_t mark) {
    const TaskHdr& h = sh.h;
    const uint32_t lane = lane_id(), wave = NT == 64 ? 0u : wave_id();
    const uint32_t W = 1u << uni(h.log2W), G = (W + 63) / 64, lanes = W < 64 ? W : 64;
    const uint32_t nsym = uni(h.nsym);
    const uint32_t* states = (const uint32_t*)(P.vol + uni64(h.states_off));
    for (uint32_t g = uni(wave); g < G; g += NT / 64) {
        const uint32_t gcount = uni(h.gw[g]), gbase = uni(h.gstart[g]);
        uint32_t x = g == wave ? x0 : lane < lanes ? states[64 * g + lane] : 0u;
        uint32_t gpos = 0, pend = 0, r0 = 64 * g;
        __builtin_amdgcn_s_waitcnt(0);
        // full rounds, first those below `mark`
        if (W >= 2u && lane < lanes) {
#pragma nounroll
            for (uint32_t part = mark ? 0u : 1u; part < 2u; ++part) {
                const uint32_t last = nsym >= lanes ? nsym - lanes + 1u : 0u, end = uni(part ? last : min(mark, last));
                // (uni: the compiler takes the position for a lane's own otherwise)
                for (r0 = uni(r0); r0 < end; r0 += W) {
                    const uint32_t e = tab[x & (kRansM - 1)];
                    const uint32_t xd = ((e >> 4) & 0x1FFFu) * (x >> kRansBits) + (e >> 17);
                    const bool need = xd < kRansL;
                    const uint64_t m = __ballot(need);
                    uint32_t wv = wl[gbase + min(gpos, gcount) + mbcnt(m)];
                    asm volatile("" : "+v"(wv));  // (read by every lane: a branch around the read costs more)
                    x = need ? ((xd << 16) | wv) : xd;
                    gpos += (uint32_t)__popcll(m);
                    // two consecutive symbols per byte
                    const uint32_t s = e & 15u;  // quad_perm [0,0,2,2], [1,1,3,3]: both lanes write the pair's byte
                    nl[(r0 >> 1) + (lane >> 1)] = (uint8_t)(dpp<0xA0>(0u, s) | (dpp<0xF5>(0u, s) << 4));
                }
                if (part == 0u && r0 >= mark && lane == 0)
                    __hip_atomic_store(&sh.prog[g], mark, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        gpos = uni(gpos);
        for (r0 = uni(r0); r0 < nsym; r0 += W) {  // the last round (all rounds of one lane)
            const uint32_t j = r0 + lane;
            const bool act = lane < lanes && j < nsym;
            const uint32_t e = tab[x & (kRansM - 1)];
            const uint32_t s = e & 15u;
            const uint32_t xd = ((e >> 4) & 0x1FFFu) * (x >> kRansBits) + (e >> 17);
            const bool need = act && xd < kRansL;
            const uint64_t m = __ballot(need);
            const uint32_t wv = wl[gbase + min(gpos, gcount) + mbcnt(m)];
            x = need ? ((xd << 16) | wv) : act ? xd : x;
            gpos += (uint32_t)__popcll(m);
            if (W >= 2) {
                const uint32_t hi = dpp<0xB1>(0u, s);
                if (act && !(lane & 1)) nl[j >> 1] = (uint8_t)(s | (j + 1 < nsym ? hi << 4 : 0u));
            } else if (lane == 0) {
                if (!(j & 1)) {
                    pend = s;
                    if (j + 1 == nsym) nl[j >> 1] = (uint8_t)pend;
                } else {
                    nl[j >> 1] = (uint8_t)(pend | (s << 4));
                }
            }
        }
        if (gpos > gcount && lane == 0) atomicOr(&sh.err, 1u);
        if (mark && lane == 0) __hip_atomic_store(&sh.prog[g], 0xFFFFFFFFu, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// ------------------------------------------------------------------ output
// Decoded labels are written once and not read again by the kernel: vector
// stores carry the non-temporal hint, so they do not displace the records and
// symbols other work-groups still read from L2.
typedef uint32_t u32x4 __attribute__((vector_size(16)));
__device__ __forceinline__ void st16_nt(void* p, uint4 v) {
    const u32x4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, (u32x4*)p);
}

template <typename LT, bool NT_HINT = true>
__device__ __forceinline__ void store4(LT* o, LT a, LT b, LT c, LT d, bool vec) {
    if (!vec) {
        o[0] = a;
        o[1] = b;
        o[2] = c;
        o[3] = d;
        return;
    }
    uint4 w[sizeof(LT) / 4];
    if (sizeof(LT) == 4) {
        w[0] = make_uint4((uint32_t)a, (uint32_t)b, (uint32_t)c, (uint32_t)d);
    } else {
        w[0] = make_uint4((uint32_t)a, (uint32_t)((uint64_t)a >> 32), (uint32_t)b, (uint32_t)((uint64_t)b >> 32));
        w[sizeof(LT) / 4 - 1] = make_uint4((uint32_t)c, (uint32_t)((uint64_t)c >> 32), (uint32_t)d, (uint32_t)((uint64_t)d >> 32));
    }
#pragma unroll
    for (uint32_t k = 0; k < sizeof(LT) / 4; ++k) {
        if (NT_HINT) st16_nt((uint4*)o + k, w[k]);
        else ((uint4*)o)[k] = w[k];
    }
}

template <typename LT>
__device__ __forceinline__ void store2(LT* o, LT a, LT b, bool vec) {
    if (!vec) {
        o[0] = a;
        o[1] = b;
    } else if (sizeof(LT) == 4) {
        *(uint2*)o = make_uint2((uint32_t)a, (uint32_t)b);
    } else {
        *(uint4*)o = make_uint4((uint32_t)a, (uint32_t)((uint64_t)a >> 32), (uint32_t)b, (uint32_t)((uint64_t)b >> 32));
    }
}

template <int NT>
__device__ __forceinline__ void zero_output(const Params& P, const TaskHdr& h) {
    const uint32_t t = uni(h.t);
    const uint64_t unit = P.pal_bits ? 4u : P.label_bytes;
    uint8_t* out = P.out + uni64(h.out_off) * unit;
    const uint64_t bytes = out_units(1ull << (3 * t), P.pal_bits) * unit;
    if (((uintptr_t)out & 15u) == 0 && (bytes & 15u) == 0) {
        for (uint64_t u = threadIdx.x & (NT - 1); u < bytes / 16; u += NT) ((uint4*)out)[u] = make_uint4(0, 0, 0, 0);
    } else {
        for (uint64_t u = threadIdx.x & (NT - 1); u < bytes / 4; u += NT) ((uint32_t*)out)[u] = 0u;
    }
}

// ------------------------------------------------------------ level bitmaps
// Expansion bits of levels 0..4, one entry per 32 nodes: x the bits, y the
// number of expanding nodes before the word (level_prefix).  A 64^3 brick keeps
// level 5 the same way in the slot area.
__device__ __forceinline__ bool ep_bit(uint2 e, uint32_t q) { return (e.x >> (q & 31)) & 1u; }
__device__ __forceinline__ uint32_t ep_rank(uint2 e, uint32_t q) {
    return e.y + (uint32_t)__popc(e.x & ((1u << (q & 31)) - 1u));
}

// Exclusive popcount prefix of the words of one level's bitmap (one wavefront;
// each lane takes a run of words); returns the number of expanding nodes.
__device__ __forceinline__ uint32_t level_prefix(uint2* ep, uint32_t words) {
    const uint32_t lane = lane_id(), per = (words + 63u) / 64u, w0 = lane * per;
    uint32_t sum = 0;
    for (uint32_t q = 0; q < per; ++q)
        if (w0 + q < words) sum += (uint32_t)__popc(ep[w0 + q].x);
    const uint32_t incl = wave_incl_sum(sum);
    uint32_t run = incl - sum;
    for (uint32_t q = 0; q < per; ++q)
        if (w0 + q < words) {
            const uint32_t bits = ep[w0 + q].x;
            ep[w0 + q].y = run;
            run += (uint32_t)__popc(bits);
        }
    return (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
}

// ------------------------------------------------------ symbols to operations
// A symbol is an operation or a 4-bit entry of the delta chain before it: a
// 2-state automaton (state 1 = the symbol is an entry).  A symbol's effect on
// the state depends on its code and bit 3 alone:
//   DELTA code, bit 3 set      -> 1         DELTA code, bit 3 clear -> inverted
//   other code, bit 3 clear    -> 0         other code, bit 3 set   -> kept
// With the inversions taken out by a parity prefix, what is left is a carry
// chain (generate, kill, propagate), so one addition gives the state before
// each of a word's 8 symbols: nibble q of A is 15 where the symbol generates
// or propagates, bit 4q of B is 1 where it generates, and the carry into nibble
// q is the state before symbol q (up to the parity).
constexpr uint32_t kNib = 0x11111111u;  // bit 4q <-> symbol q of a word ("nibble mask")

// nibble masks of a word's symbols by operation code (4 ADV, 5 LAST, 6 DELTA, 7 invalid)
// and bit 3; other bits of the masks are arbitrary
struct Planes {
    uint32_t b0, b1, b2, b3;
    __device__ __forceinline__ explicit Planes(uint32_t w) : b0(w), b1(w >> 1), b2(w >> 2), b3(w >> 3) {}
    __device__ __forceinline__ uint32_t adv() const { return b2 & ~(b1 | b0); }
    __device__ __forceinline__ uint32_t last() const { return b2 & ~b1 & b0; }
    __device__ __forceinline__ uint32_t delta() const { return b2 & b1 & ~b0; }
    __device__ __forceinline__ uint32_t bad() const { return b2 & b1 & b0; }
};

struct WordRun {
    uint32_t A, B, par;  // carry chain; inclusive parity of the inversions
    // nibble mask of the symbols that are delta entries when the word is entered in state e
    __device__ __forceinline__ uint32_t entries(uint32_t e) const { return (((A + B + e) ^ A ^ B) & kNib) ^ (par << 4); }
    __device__ __forceinline__ uint32_t exit(uint32_t e) const { return ((A & ~(A + B + e)) >> 31) ^ (par >> 28); }
};

// V: the symbols of the word that belong to the level; the others keep the state
__device__ __forceinline__ WordRun word_run(const Planes& pl, uint32_t V) {
    const uint32_t D = pl.delta(), C = pl.b3;
    const uint32_t set = D & C & V, rst = ~(D | C) & V;
    uint32_t p = D & ~C & V;
    p ^= p << 4;
    p ^= p << 8;
    p ^= p << 16;
    const uint32_t pg = kNib & ~((set & p) | (rst & ~p));
    return WordRun{(pg << 4) - pg, (set & ~p) | (rst & p), p};
}

// nibble mask of the symbols of word w inside [s0, s1)
__device__ __forceinline__ uint32_t word_valid(uint32_t w, uint32_t s0, uint32_t s1) {
    const uint32_t j = 8u * w;
    const uint32_t hi = s1 > j ? min(s1 - j, 8u) : 0u, lo = s0 > j ? min(s0 - j, 8u) : 0u;
    const uint32_t mh = hi >= 8u ? kNib : ((1u << (4u * hi)) - 1u) & kNib;
    return lo >= 8u ? 0u : mh & ~((1u << (4u * lo)) - 1u);
}

// The same carry chain over the lanes of a wavefront, in scalar registers: b0, b1
// hold each lane's exit state for entry state 0 and 1.
struct LaneRun {
    uint64_t A, B, p;
    __device__ __forceinline__ LaneRun(uint64_t b0, uint64_t b1) {
        p = b0 & ~b1;  // lanes that invert
        if (p) {
            p ^= p << 1;
            p ^= p << 2;
            p ^= p << 4;
            p ^= p << 8;
            p ^= p << 16;
            p ^= p << 32;
        }
        const uint64_t set = b0 & b1, rst = ~(b0 | b1);
        B = (set & ~p) | (rst & p);
        A = (b0 ^ b1) | B;
    }
    // the lanes' entry states, and the state after the last lane, when lane 0 is entered in state e
    __device__ __forceinline__ uint64_t entry(uint32_t e) const { return (A + B + e) ^ A ^ B ^ (p << 1); }
    __device__ __forceinline__ uint32_t exit(uint32_t e) const { return (uint32_t)(((B | (A & ~(A + B + e))) ^ p) >> 63); }
};

__device__ __forceinline__ uint32_t lane_bit(uint64_t m) {
    const uint32_t l = lane_id();
    return ((l & 32u ? (uint32_t)(m >> 32) : (uint32_t)m) >> (l & 31u)) & 1u;
}

// where a level's symbols have been read to
struct RunState {
    uint32_t state;  // automaton state
    uint32_t k;      // operations so far
    uint32_t adv;    // PALETTE_ADV operations so far, all levels
};

// slot values: a final palette index, or an operation that copies (its code, 0..3).
// 16-bit slots hold 15-bit indices (13 with a stop bit: levels up to 4), 32-bit
// slots 21 bits (a 64^3 brick has fewer than 2^19 nodes).
template <bool W32>
struct SlotBits {
    static constexpr uint32_t kFinal = W32 ? 0x800000u : 0x8000u;
    static constexpr uint32_t kStop = W32 ? 0x400000u : 0x4000u;
};

// One pass over words [w_at, w_at + nw) of a level with symbols [s0, s1): every
// thread takes 1 << lr (at most 4) consecutive words, summarises them for both
// entry states (operations | ADVs << 16), a wavefront scan and one barrier give
// it its entry state, its first operation rank k and its ADV count, and it then
// writes the slot of each of its operations, slot[k - kbase]: palette
// operations as final indices (ADV -> a, LAST -> a - 1, DELTA -> a - delta),
// copies as their code; with STOP the stop bit goes along.  False (to every
// thread, nothing written) when the operations exceed `expected`.  Needs at
// least one ADV before the pass (level 0 is decoded apart).
template <int NT, bool W32, bool STOP, typename SH, typename SLOT>
__device__ __forceinline__ bool ops_pass(SH& sh, const uint32_t* sym, uint32_t s0, uint32_t s1, uint32_t w_at,
                                         uint32_t nw, uint32_t lr, uint32_t expected, uint32_t kbase, SLOT* slot,
                                         RunState& rs, uint32_t& pbuf, bool& bad) {
    constexpr uint32_t NW = NT / 64;
    constexpr uint32_t FIN = SlotBits<W32>::kFinal, STP = SlotBits<W32>::kStop;
    const uint32_t tid = threadIdx.x & (NT - 1), wave = NW == 1 ? 0u : wave_id();
    const uint32_t w_last = (s1 - 1u) >> 3, w_end = w_at + nw, w0 = w_at + (tid << lr), R = 1u << lr;
    // the thread's words and the one after them (delta entries), at clamped indices
    uint32_t W[5];
    W[0] = sym[min(w0, w_last)];
    W[1] = sym[min(w0 + 1u, w_last)];
    if (lr >= 1u) W[2] = sym[min(w0 + 2u, w_last)];
    if (lr >= 2u) {
        W[3] = sym[min(w0 + 3u, w_last)];
        W[4] = sym[min(w0 + 4u, w_last)];
    }
    auto valid = [&](uint32_t r) -> uint32_t { return w0 + r < w_end ? word_valid(w0 + r, s0, s1) : 0u; };
    const bool wave_on = w_at + ((64u * wave) << lr) < w_end;
    uint32_t n0 = 0, n1 = 0, i0 = 0, i1 = 0, x0 = 0, x1 = 1;  // counts, their scans, the wave's exit states
    uint32_t O0[4], O1[4];                                     // the words' operations (nibble masks)
    uint64_t m0 = 0, m1 = 0;                                   // the lanes' entry states
    if (wave_on) {
        uint32_t e0 = 0, e1 = 1;
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            if (r < R) {
                const uint32_t V = valid(r);
                const Planes pl(W[r]);
                const WordRun wr = word_run(pl, V);
                const uint32_t advm = pl.adv();
                O0[r] = V & ~wr.entries(e0);
                O1[r] = V & ~wr.entries(e1);
                n0 += (uint32_t)__popc(O0[r]) | ((uint32_t)__popc(O0[r] & advm) << 16);
                n1 += (uint32_t)__popc(O1[r]) | ((uint32_t)__popc(O1[r] & advm) << 16);
                e0 = wr.exit(e0);
                e1 = wr.exit(e1);
            }
        }
        const LaneRun run(__ballot(e0 != 0u), __ballot(e1 != 0u));
        m0 = run.entry(0u);
        m1 = run.entry(1u);
        x0 = run.exit(0u);
        x1 = run.exit(1u);
        i0 = wave_incl_sum(lane_bit(m0) ? n1 : n0);
        i1 = wave_incl_sum(lane_bit(m1) ? n1 : n0);
    }
    uint32_t st = rs.state, k = rs.k, adv = rs.adv, my_st = st, my_k = k, my_adv = adv;
    auto add_run = [&](uint32_t xs, uint32_t t0, uint32_t t1) {
        const uint32_t tot = st ? t1 : t0;
        k += tot & 0xFFFFu;
        adv += tot >> 16;
        st = (xs >> st) & 1u;
    };
    const uint32_t t0 = (uint32_t)__builtin_amdgcn_readlane((int)i0, 63);
    const uint32_t t1 = (uint32_t)__builtin_amdgcn_readlane((int)i1, 63);
    if (NW == 1) {
        add_run(x0 | (x1 << 1), t0, t1);
    } else {
        if (lane_id() == 0) sh.pub[pbuf][wave] = make_uint4(x0 | (x1 << 1), t0, t1, 0u);
        lds_barrier();
#pragma unroll
        for (uint32_t w = 0; w < NW; ++w) {
            const uint4 pw = sh.pub[pbuf][w];
            if (w == wave) {
                my_st = st;
                my_k = k;
                my_adv = adv;
            }
            add_run((uint32_t)__builtin_amdgcn_readfirstlane((int)pw.x), (uint32_t)__builtin_amdgcn_readfirstlane((int)pw.y),
                    (uint32_t)__builtin_amdgcn_readfirstlane((int)pw.z));
        }
        pbuf ^= 1u;
    }
    rs = RunState{st, k, adv};
    if (k > expected) return false;
    if (!wave_on) return true;
    const uint32_t e = lane_bit(my_st ? m1 : m0);
    const uint32_t excl = (my_st ? i1 : i0) - (e ? n1 : n0);
    uint32_t kk = my_k - kbase + (excl & 0xFFFFu), aa = my_adv + (excl >> 16);
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r)
        if (r < R) O0[r] = e ? O1[r] : O0[r];
#pragma nounroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint32_t word = W[0], opm = O0[0];
        const Planes pl(word);
        const uint32_t advm = opm & pl.adv();
        bad = bad || (opm & pl.bad());
        // Slot of symbol q, by nibbles: a copy's code, or for a palette operation
        // its distance from the palette index before the word's first ADV (the
        // ADVs before it, less one for LAST, plus one) with the base aa - 1 added
        const uint32_t pal = pl.b2 & kNib, pal15 = (pal << 4) - pal;
        const uint32_t off = (advm * 0x11111110u) + (kNib & ~pl.last());
        const uint32_t nibs = (off & pal15) | (word & 0x33333333u & ~pal15), base = FIN | (aa - 1u);
        SLOT* at = slot + kk;
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
            if ((opm >> (4 * q)) & 1u) {
                uint32_t v = __umul24((pal >> (4 * q)) & 1u, base) + ((nibs >> (4 * q)) & 15u);
                if (STOP) v += __umul24((word >> (4 * q + 3)) & 1u, STP);
                *at++ = (SLOT)v;
            }
        }
        // back references: the entries that follow, in the word, the next word, or (rarely) beyond
        for (uint32_t m = opm & pl.delta(); m; m &= m - 1u) {
            const uint32_t b = (uint32_t)__builtin_ctz(m), below = (1u << b) - 1u;
            const uint32_t a = aa + (uint32_t)__popc(advm & below);
            uint32_t win = (uint32_t)(((((uint64_t)W[1]) << 32) | word) >> (b + 4u));  // the next entries: 8 at least
            uint32_t en = win & 15u, d = en & 7u, j = 8u * (w0 + r) + (b >> 2) + 1u, left = 7u;
            while (en & 8u) {
                if (++j >= s1) break;  // (the chain leaves the level: its end state says so)
                win >>= 4;
                if (left == 0u) {
                    win = sym[j >> 3] >> (4u * (j & 7u));
                    left = 8u - (j & 7u);
                }
                --left;
                en = win & 15u;
                d = d >= (1u << 29) ? 0xFFFFFFFFu : ((d << 3) | (en & 7u));
            }
            if (d - 1u >= a) {
                bad = true;
                d = a;
            }
            uint32_t v = FIN | (a - d);
            if (STOP) v += __umul24((word >> (b + 3u)) & 1u, STP);
            slot[kk + (uint32_t)__popc(opm & below)] = (SLOT)v;
        }
        kk += (uint32_t)__popc(opm);
        aa += (uint32_t)__popc(advm);
        W[0] = W[1];
        W[1] = W[2];
        W[2] = W[3];
        W[3] = W[4];
        O0[0] = O0[1];
        O0[1] = O0[2];
        O0[2] = O0[3];
    }
    return true;
}

// All passes of a level whose slots are slot[0 .. expected); true when the
// symbols are exactly its operations (and the ADVs stay inside the palette).
template <int NT, bool STOP, typename SH>
__device__ __forceinline__ bool ops_level(SH& sh, const uint32_t* sym, uint32_t s0, uint32_t s1, uint32_t expected,
                                          uint16_t* slot, uint32_t& adv, uint32_t& pbuf, bool& bad) {
    RunState rs{0u, 0u, adv};
    if (s1 > s0) {
        const uint32_t w_first = s0 >> 3, n_words = ((s1 - 1u) >> 3) - w_first + 1u;
        const uint32_t lr = n_words <= NT ? 0u : n_words <= 2u * NT ? 1u : 2u;
        for (uint32_t w = 0; w < n_words; w += NT << lr)
            if (!ops_pass<NT, false, STOP>(sh, sym, s0, s1, w_first + w, min(n_words - w, (uint32_t)NT << lr), lr, expected, 0u,
                                           slot, rs, pbuf, bad))
                return false;
    }
    adv = rs.adv;
    return rs.k == expected && rs.state == 0u && adv <= uni(sh.h.pc);
}

// -------------------------------------------------------- operations to values
// A level's values: in 16-bit slots a palette index, or with the top bit
// (kOpen) set a reference to the slot of a node before it whose value it takes.
// (So a value is used without masking, and a test for its sign finds what is
// open.)  A row of slots as ops_pass leaves it, with the top bits inverted, has
// the palette operations final and the copies open.
constexpr uint32_t kOpen = 0x8000u;

// The 8 children of one expanding parent: op(c) is child c's operation (open:
// its code in the low bits, else the palette index), pv the parent's value,
// ext(axis, c) the value of (or a reference to) the node beside child c across
// the parent's lower face; inv[axis]: there is no such node.  A copy from a
// sibling takes the sibling's value, which may be a reference itself.
template <uint32_t OPEN, typename OP, typename EXT>
__device__ __forceinline__ void resolve8(uint32_t v[8], OP op, uint32_t pv, EXT ext, const bool inv[3], bool& bad) {
#pragma unroll
    for (uint32_t c = 0; c < 8; ++c) {
        const uint32_t o = op(c);
        uint32_t r = pv;
#pragma unroll
        for (uint32_t a = 0; a < 3; ++a) {
            const bool is = o == (OPEN | (a + 1u));
            if (c & (1u << a)) {
                r = is ? v[c ^ (1u << a)] : r;
            } else {
                r = is ? ext(a, c) : r;
                bad = bad || (is && inv[a]);
            }
        }
        v[c] = (o & OPEN) ? r : o;
    }
}

__device__ __forceinline__ uint4 flip8(const uint4& w) {
    constexpr uint32_t m = kOpen * 0x10001u;
    return make_uint4(w.x ^ m, w.y ^ m, w.z ^ m, w.w ^ m);
}
__device__ __forceinline__ uint4 pack8(const uint32_t v[8]) {
    return make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
}
__device__ __forceinline__ uint32_t half_of(const uint4& w, uint32_t c) {
    const uint32_t x = c < 2 ? w.x : c < 4 ? w.y : c < 6 ? w.z : w.w;
    return c & 1u ? x >> 16 : x & 0xFFFFu;
}

// node below q along `axis` (Morton; mask am = the axis's bits): q itself when there is none
__device__ __forceinline__ uint32_t node_below(uint32_t q, uint32_t am) {
    const uint32_t x = q & am;
    return (x ? (x - 1u) & am : 0u) | (q & ~am);
}

// The open slots of a row of 16-bit slots (bit c for child c).
__device__ __forceinline__ uint32_t open_of(const uint4& w) {
    const uint32_t m = ((w.x >> 15) & 0x10001u) | ((w.y >> 13) & 0x40004u) | ((w.z >> 11) & 0x100010u) | ((w.w >> 9) & 0x400040u);
    return (m | (m >> 15)) & 0xFFu;
}

// Replace references by the values at the ends of their chains: the open slots
// (bits of `open`) of the rows whose first slots are base[at], one row per lane.
// A reference points to an explicit node of the same level before its source in
// Morton order, so chains end.  About a fifth of the slots are open and a chain
// has up to 20 links, so the wavefront first lists its open slots in LDS (`refs`,
// room for `cap` >= 8, as many rows at a time as fit) and then follows one chain
// per lane; following the 8 slots of a row side by side in each lane took three
// times the instructions.  Every step is written back, so that the lanes behind
// skip what this one has passed (any value on the way has the same end: waves
// that follow chains through each other's rows may see any of them): 4096 cubes
// of 32^3 0.217 -> 0.213 ms.
template <typename V, V OPEN>
__device__ __forceinline__ void chase_open(V* base, uint32_t at, uint32_t open, uint16_t* refs, uint32_t cap) {
    const uint32_t lane = lane_id();
    while (__ballot(open != 0u)) {
        const uint32_t n = (uint32_t)__popc(open), incl = wave_incl_sum(n);
        const bool now = incl <= cap;
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63 - __builtin_clzll(__ballot(now)));
        if (now)
            for (uint32_t k = incl - n; open; open &= open - 1u) refs[k++] = (uint16_t)(at + (uint32_t)__builtin_ctz(open));
        lsync<64>();
        for (uint32_t i = lane; i < total; i += 64u) {
            const uint32_t me = refs[i];
            uint32_t v = base[me];
            while (v & OPEN) {
                v = base[v ^ OPEN];
                base[me] = (V)v;
            }
        }
        lsync<64>();
    }
}

// The list of the expanding nodes among the 8 * bytes nodes of a level, by rank:
// each of NT threads lists those of some bytes of the bitmap.
template <int NT>
__device__ __forceinline__ void list_parents(const uint2* ep, uint32_t bytes, uint16_t* list) {
    for (uint32_t b = threadIdx.x; b < bytes; b += NT) {
        const uint2 e = ep[b >> 2];
        uint32_t r = ep_rank(e, 8u * b), bits = (e.x >> (8u * (b & 3u))) & 0xFFu;
#pragma unroll
        for (uint32_t c = 0; c < 8; ++c)
            if ((bits >> c) & 1u) list[r++] = (uint16_t)(8u * b + c);
    }
}

// ------------------------------------------------------------- full levels
// Level 3 or 4 into its full grid: the calling wavefront alone (NT = 64, level 3:
// a lane per parent) or the work-group (level 4: a thread per expanding
// parent, from a list in `work`).  The operations are written compactly into the
// grid's own space, read back by the parents they belong to, and then every
// parent writes its 8 children and their expansion bits: an expanding one what
// its operations say, any other its own value.  work: LDS for lists of
// references (and of the parents), work_bytes in all.
template <int NT, typename SH>
__device__ __forceinline__ bool full_level(SH& sh, const uint32_t* sym, uint32_t i, uint32_t nexp, uint32_t& adv,
                                           uint32_t& pbuf, uint8_t* work, uint32_t work_bytes) {
    constexpr uint32_t PP = NT >= 512 ? 1u : NT == 64 ? 1u : 512u / NT;  // parents per thread
    constexpr uint32_t STP = SlotBits<false>::kStop;
    const uint32_t tid = threadIdx.x & (NT - 1);
    uint16_t* const grid = sh.G + fbase(i);
    const uint16_t* const par = sh.G + fbase(i - 1);
    const uint2* const ep = sh.EP + ebase(i - 1);
    const uint32_t np = 1u << (3 * (i - 1));
    uint16_t* const list = (uint16_t*)work;
    uint16_t* refs = (uint16_t*)work;
    uint32_t cap = work_bytes / 2u;
    if (NT > 64) {
        constexpr uint32_t NW = NT / 64;
        list_parents<NT>(ep, 64u, list);
        cap = (work_bytes - 1024u) / (2u * NW);
        refs += 512u + wave_id() * cap;
    }
    bool bad = false;
    if (!ops_level<NT, true>(sh, sym, uni(sh.h.sym_end[i - 1]), uni(sh.h.sym_end[i]), 8u * nexp, grid, adv, pbuf, bad)) return false;
    lsync<NT>();
    uint4 raw[PP];
    uint32_t qs[PP];
    bool ex[PP];
#pragma unroll
    for (uint32_t p = 0; p < PP; ++p) {
        if (NT == 64) {
            qs[p] = tid;
            const uint2 e = ep[tid < np ? tid >> 5 : 0u];
            ex[p] = tid < np && ep_bit(e, tid);
            if (ex[p]) raw[p] = *(const uint4*)(grid + 8u * ep_rank(e, tid));
        } else {
            const uint32_t r = tid + p * NT;
            ex[p] = r < nexp;
            if (ex[p]) {
                qs[p] = list[r];
                raw[p] = *(const uint4*)(grid + 8u * r);
            }
        }
    }
    lsync<NT>();
    const uint32_t mx = 0x09249249u & (np - 1u);
    uint32_t open[PP];
#pragma unroll
    for (uint32_t p = 0; p < PP; ++p) {
        open[p] = 0;
        if (ex[p]) {
            const uint32_t q = qs[p], pv = par[q];
            uint32_t v[8], eb[3], ea[3];
            bool inv[3];
#pragma unroll
            for (uint32_t a = 0; a < 3; ++a) {
                const uint32_t am = mx << a, tq = node_below(q, am);
                inv[a] = !(q & am);
                const bool te = !inv[a] && ep_bit(ep[tq >> 5], tq);
                eb[a] = te ? kOpen | (8u * tq) : par[tq];
                ea[a] = te ? 7u : 0u;
            }
            const uint4 w = raw[p];
            const uint32_t keep = ~(STP * 0x10001u);
            const uint4 ops = flip8(make_uint4(w.x & keep, w.y & keep, w.z & keep, w.w & keep));
            resolve8<kOpen>(v, [&](uint32_t c) { return half_of(ops, c); }, pv,
                          [&](uint32_t a, uint32_t c) { return eb[a] | ((c | (1u << a)) & ea[a]); }, inv, bad);
            // (stop bits: children 0, 2, 4, 6 in the low halves, 1, 3, 5, 7 in the high ones)
            const uint32_t m = ((w.x >> 14) & 0x10001u) | ((w.y >> 12) & 0x40004u) | ((w.z >> 10) & 0x100010u) |
                               ((w.w >> 8) & 0x400040u);
            const uint32_t bits = ~(m | (m >> 15)) & 0xFFu;
            const uint4 row = pack8(v);
            open[p] = open_of(row);
            ((uint4*)grid)[q] = row;
            uint2* const eo = sh.EP + ebase(i) + (q >> 2);
            ((uint8_t*)&eo->x)[q & 3u] = (uint8_t)bits;
        }
    }
    // the other parents
    for (uint32_t q = tid; q < np; q += NT) {
        if (!ep_bit(ep[q >> 5], q)) {
            const uint32_t v2 = par[q] * 0x10001u;
            ((uint4*)grid)[q] = make_uint4(v2, v2, v2, v2);
            uint2* const eo = sh.EP + ebase(i) + (q >> 2);
            ((uint8_t*)&eo->x)[q & 3u] = 0;
        }
    }
    if (bad) sh.err = 1u;
    lsync<NT>();
#pragma unroll
    for (uint32_t p = 0; p < PP; ++p) chase_open<uint16_t, kOpen>(grid, 8u * qs[p], open[p], refs, cap);
    return true;
}

// Level i = 1 or 2 by the calling wavefront alone, a lane per symbol and then a
// lane per node: no words to unpack, no lists, and chains of references followed
// in registers, by doubling.  These levels are a serial chain that the rest of a
// cube waits for: 8.8k and 9.6k cycles as level 3 does it, 3.0k and 4.3k so
// (1400 cubes of side 8: 0.029 -> 0.025 ms, 4096 of 32: 0.227 -> 0.217).
template <typename SH>
__device__ __forceinline__ bool lane_level(SH& sh, const uint32_t* sym, uint32_t i, uint32_t& nexp, uint32_t& adv) {
    constexpr uint32_t STP = SlotBits<false>::kStop;
    const uint32_t lane = lane_id(), n = 1u << (3 * i), expected = 8u * nexp, pm = uni(sh.EP[ebase(i - 1)].x);
    const uint32_t s0 = uni(sh.h.sym_end[i - 1]), s1 = uni(sh.h.sym_end[i]);
    uint16_t* const grid = sh.G + fbase(i);
    uint32_t state = 0, k = 0;
    bool bad = false;
    for (uint32_t at = s0; at < s1; at += 64u) {
        const uint32_t j = at + lane, left = s1 - at;
        const uint32_t sy = j < s1 ? (sym[j >> 3] >> (4u * (j & 7u))) & 15u : 0u, code = sy & 7u;
        const bool delta = code == kDelta, on = (sy & 8u) != 0u;
        const LaneRun run(__ballot(delta), __ballot(on));
        const uint64_t m = run.entry(state);
        const uint64_t ops = ~m & (left < 64u ? (1ull << left) - 1u : ~0ull), advs = ops & __ballot(code == kAdv);
        state = left < 64u ? (uint32_t)(m >> left) & 1u : run.exit(state);
        const uint32_t r = k + mbcnt(ops), a = adv + mbcnt(advs);
        k += (uint32_t)__popcll(ops);
        adv += (uint32_t)__popcll(advs);
        if (lane_bit(ops)) {
            uint32_t v = code < 4u ? kOpen | code : a - (code == kLast ? 1u : 0u);
            bad = bad || code == kBadOp;
            if (delta) {
                uint32_t d = 0, q = j + 1u, en = 8u;
                for (; q < s1 && (en & 8u); ++q) {  // (a chain that leaves the level: its end state says so)
                    en = sym[q >> 3] >> (4u * (q & 7u));
                    d = d >= (1u << 29) ? 0xFFFFFFFFu : ((d << 3) | (en & 7u));
                }
                if (d - 1u >= a) {
                    bad = true;
                    d = a;
                }
                v = a - d;
            }
            if (r < expected) grid[r] = (uint16_t)(v | (on ? STP : 0u));
        }
    }
    if (k != expected || state || adv > uni(sh.h.pc)) return false;
    lsync<64>();
    // the nodes; a reference is the lane of the node whose value is taken
    const uint32_t q = lane >> 3, mx = 0x09249249u & (n - 1u);
    const bool node = lane < n, ex = node && ((pm >> q) & 1u);
    const uint32_t pv = sh.G[fbase(i - 1) + (node ? q : 0u)];
    const uint32_t slot = ex ? grid[8u * (uint32_t)__popc(pm & ((1u << q) - 1u)) + (lane & 7u)] : 0u;
    lsync<64>();
    uint32_t v = pv;
    if (ex) {
        const uint32_t o = slot & ~STP;
        if (!(o & kOpen)) {
            v = o;
        } else if (o != kOpen) {
            const uint32_t am = mx << (o - kOpen - 1u);
            if (lane & am) v = kOpen | node_below(lane, am);
            else bad = true;
        }
    }
    while (__ballot((v & kOpen) != 0u)) {  // (references go to lower lanes: at most 6 rounds)
        const uint32_t to = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * (v & 63u)), (int)v);
        v = v & kOpen ? to : v;
    }
    const uint64_t bits = __ballot(ex && !(slot & STP));
    if (node) grid[lane] = (uint16_t)v;
    if (lane == 0) {
        sh.EP[ebase(i)] = make_uint2((uint32_t)bits, 0u);
        if (i == 2) sh.EP[ebase(i) + 1u] = make_uint2((uint32_t)(bits >> 32), (uint32_t)__popc((uint32_t)bits));
    }
    if (bad) sh.err = 1u;
    nexp = (uint32_t)__popcll(bits);
    return true;
}

// Levels 0..last (at most 3) by the calling wavefront alone; then the parent
// prefix of the next level, the number of its expanding nodes in sh.nexp and
// the ADV count in sh.adv; work: LDS for lists of references.  Level 0 is one node whose only valid operation is
// PALETTE_ADV (entry 0), with or without a stop bit.
template <typename SH>
__device__ __forceinline__ void small_levels(SH& sh, const uint32_t* sym, uint32_t last, uint8_t* work, uint32_t work_bytes) {
    const uint32_t s0 = sym[0] & 15u;
    if (uni(sh.h.sym_end[0]) != 1u || (s0 & 7u) != kAdv || uni(sh.h.pc) == 0u) {
        sh.err = 1u;
        return;
    }
    if (lane_id() == 0) {
        sh.G[fbase(0)] = 0u;
        sh.EP[ebase(0)] = make_uint2(s0 & 8u ? 0u : 1u, 0u);
    }
    lsync<64>();
    uint32_t adv = 1, pbuf = 0, nexp = s0 & 8u ? 0u : 1u;
    for (uint32_t i = 1; i <= last; ++i) {
        if (!(i < 3 ? lane_level(sh, sym, i, nexp, adv) : full_level<64>(sh, sym, i, nexp, adv, pbuf, work, work_bytes))) {
            sh.err = 1u;
            return;
        }
        lsync<64>();
        if (i == 3) nexp = level_prefix(sh.EP + ebase(i), ewords(i));
        lsync<64>();
    }
    if (lane_id() == 0) {
        sh.nexp = nexp;
        sh.adv = adv;
    }
}

// ------------------------------------------------------- level 5 in LDS
// Level 5 of a 32^3 cube at full resolution: its explicit nodes by operation
// rank in the slot area (child c of the r-th expanding parent at 8r + c).
template <int NT>
__device__ __forceinline__ bool level5(Shared& sh, const uint32_t* sym, uint16_t* c5, uint8_t* u_area, uint32_t u_bytes, uint32_t nexp,
                                       uint32_t pal_words, const uint32_t* pal, uint32_t& adv, uint32_t& pbuf) {
    const uint2* const ep = sh.EP + ebase(4);
    const uint16_t* const par = sh.G + fbase(4);
    uint16_t* const list = (uint16_t*)u_area;
    list_parents<NT>(ep, 512u, list);
    bool bad = false;
    if (!ops_level<NT, false>(sh, sym, uni(sh.h.sym_end[4]), uni(sh.h.sym_end[5]), 8u * nexp, c5, adv, pbuf, bad)) return false;
    lds_barrier();
    for (uint32_t r = threadIdx.x; r < nexp; r += NT) {
        const uint32_t q = list[r], pv = par[q];
        const uint4 raw = flip8(((const uint4*)c5)[r]);
        uint32_t eb[3], ea[3], v[8];
        bool inv[3];
#pragma unroll
        for (uint32_t a = 0; a < 3; ++a) {
            const uint32_t am = 0x249u << a, tq = node_below(q, am);
            const uint2 e = ep[tq >> 5];
            inv[a] = !(q & am);
            const bool te = !inv[a] && ep_bit(e, tq);
            eb[a] = te ? kOpen | (8u * ep_rank(e, tq)) : par[tq];
            ea[a] = te ? 7u : 0u;
        }
        resolve8<kOpen>(v, [&](uint32_t c) { return half_of(raw, c); }, pv,
                      [&](uint32_t a, uint32_t c) { return eb[a] | ((c | (1u << a)) & ea[a]); }, inv, bad);
        ((uint4*)c5)[r] = pack8(v);
    }
    if (bad) sh.err = 1u;
    lds_barrier();
    // the parent list has been read: its area takes the palette, for the output
    // pass, and the lists of references
    for (uint32_t w = threadIdx.x; w < pal_words; w += NT) ((uint32_t*)u_area)[w] = pal[w];
    const uint32_t cap = (u_bytes - 4u * pal_words) / (2u * (NT / 64));
    uint16_t* const refs = (uint16_t*)(u_area + 4u * pal_words) + wave_id() * cap;
    for (uint32_t r0 = 64u * wave_id(); r0 < nexp; r0 += NT) {
        const uint32_t r = r0 + lane_id();
        chase_open<uint16_t, kOpen>(c5, 8u * r, r < nexp ? open_of(((const uint4*)c5)[r]) : 0u, refs, cap);
    }
    return true;
}

// ------------------------------------------------ levels 5 and 6 in chunks
// A level whose explicit nodes do not fit in LDS: level 6, level 5 of a 64^3
// cube, and level 5 of a 32^3 cube that outgrows the slot area or whose palette
// indices need more than 15 bits.  The symbols are read in passes; the
// operations of a pass go to a buffer of 32-bit slots in LDS, and the parents
// whose 8 operations are there are finished before the next pass.  References
// point into the buffer; a node finished earlier is read where its result went:
//   LABELS  the task's output, which holds the labels of all nodes before the
//           chunk and of all implied nodes (fill_implied);
//   else    the work-group's scratch (c5: the palette index by operation rank).
constexpr uint32_t kChunkDone = 0x200000u;  // slot: the result is where the low bits say (c5 rank, output voxel)

struct ChunkMem {
    uint2* ep5;      // level-5 bitmap (64^3 cubes), 1024 entries at the start of the slot area
    uint32_t* buf;   // operation buffer behind it
    uint32_t cap;    // its 32-bit slots
    uint16_t* c5;    // scratch: level-5 palette indices by operation rank
    uint32_t* list;  // scratch: expanding parents by rank, node | palette index << 15
    const void* pal;         // palette of the record
    const uint8_t* pal_lds;  // the same in LDS, or null
    uint8_t* work;   // LDS for lists of references
    uint32_t work_bytes;
};

// palette index of a level-5 node (64^3 cubes; levels 4 and 5 final)
__device__ __forceinline__ uint32_t value5(const Shared& sh, const ChunkMem& cm, uint32_t node) {
    const uint32_t q = node >> 3;
    const uint2 e = sh.EP[ebase(4) + (q >> 5)];
    return ep_bit(e, q) ? (uint32_t)cm.c5[8u * ep_rank(e, q) + (node & 7u)] : (uint32_t)sh.G[fbase(4) + q];
}

template <int NT, bool LABELS, typename LT>
__device__ __forceinline__ bool chunk_level(const Params& P, Shared& sh, const ChunkMem& cm, const uint32_t* sym, uint32_t i,
                                            uint32_t nexp, uint32_t& adv, uint32_t& pbuf) {
    constexpr uint32_t OPEN = SlotBits<true>::kFinal, STP = SlotBits<true>::kStop;
    const uint32_t tid = threadIdx.x, S = 1u << i, pc = uni(sh.h.pc);
    const LT* const pal = (const LT*)cm.pal;
    const uint2* const ep = i == 5 ? sh.EP + ebase(4) : cm.ep5;
    const uint16_t* const par4 = sh.G + fbase(4);
    const bool with_bits = i == 5 && uni(sh.h.t) == 6;
    LT* const out = (LT*)(P.out + uni64(sh.h.out_off) * sizeof(LT));
    const bool vec = ((uintptr_t)out & (2 * sizeof(LT) - 1)) == 0;
    const uint32_t cap = cm.work_bytes / (2u * (NT / 64));
    uint16_t* const refs = (uint16_t*)cm.work + wave_id() * cap;
    // expanding parents by rank
    const uint32_t nb = 1u << (3 * (i - 1) - 3);
    for (uint32_t b = tid; b < nb; b += NT) {
        const uint2 e = ep[b >> 2];
        uint32_t r = ep_rank(e, 8u * b), bits = (e.x >> (8u * (b & 3u))) & 0xFFu;
        if (!bits) continue;
        // the values of 8 nodes at once: a row of the grid, or of c5 (level-5 nodes
        // 8b .. 8b + 7 are the children of level-4 node b, which expands)
        const uint4 row = i == 5 ? ((const uint4*)par4)[b]
                                 : ((const uint4*)cm.c5)[ep_rank(sh.EP[ebase(4) + (b >> 5)], b)];
#pragma unroll
        for (uint32_t c = 0; c < 8; ++c)
            if ((bits >> c) & 1u) cm.list[r++] = (8u * b + c) | (half_of(row, c) << 15);
    }
    if (with_bits)
        for (uint32_t w = tid; w < 1024u; w += NT) cm.ep5[w].x = 0;
    __syncthreads();
    const uint32_t s0 = uni(sh.h.sym_end[i - 1]), s1 = uni(sh.h.sym_end[i]), expected = 8u * nexp;
    const uint32_t mx = 0x09249249u & ((1u << (3 * (i - 1))) - 1u);
    RunState rs{0u, 0u, adv};
    uint32_t r_next = 0;
    bool bad = false;
    const uint32_t w_first = s0 >> 3, n_words = s1 > s0 ? ((s1 - 1u) >> 3) - w_first + 1u : 0u;
    // words of a pass: their operations fit the buffer; two words per thread when
    // that still fills the work-group (a pass is bound by latency, not by work)
    const uint32_t room = (cm.cap - 8u) / 8u, lr = room >= NT + NT / 2u ? 1u : 0u, step = min((uint32_t)NT << lr, room);
    for (uint32_t w = 0; w < n_words; w += step) {
        const uint32_t kbase = 8u * r_next;
        if (!ops_pass<NT, true, true>(sh, sym, s0, s1, w_first + w, min(n_words - w, step), lr, expected, kbase, cm.buf, rs,
                                      pbuf, bad))
            return false;
        // (the results of the pass before, which this one may read, have been
        // stored by now; the other barriers of a pass exchange LDS only)
        __syncthreads();
        const uint32_t n_par = (rs.k >> 3) - r_next;
        for (uint32_t x = tid; x < n_par; x += NT) {
            const uint32_t qv = cm.list[r_next + x], q = qv & 0x7FFFu, pv = qv >> 15;
            uint32_t v[8], eb[3];
            bool inv[3], in[3], te[3];
            const uint4 ra = ((const uint4*)cm.buf)[2u * x], rb = ((const uint4*)cm.buf)[2u * x + 1u];
            const uint32_t raw[8] = {ra.x, ra.y, ra.z, ra.w, rb.x, rb.y, rb.z, rb.w};
            const uint32_t vox = (compact3(q >> 2) * 2u * S + compact3(q >> 1) * 2u) * S + compact3(q) * 2u;  // child 0's
#pragma unroll
            for (uint32_t a = 0; a < 3; ++a) {
                const uint32_t am = mx << a, tq = node_below(q, am);
                const uint2 e = ep[tq >> 5];
                inv[a] = !(q & am);
                te[a] = !inv[a] && ep_bit(e, tq);
                const uint32_t kt = 8u * ep_rank(e, tq);
                in[a] = te[a] && kt >= kbase;
                eb[a] = in[a] ? OPEN | (kt - kbase) : kChunkDone | kt;
                if (!te[a] && i == 5) eb[a] = par4[tq];
            }
            auto ext = [&](uint32_t a, uint32_t c) -> uint32_t {
                const uint32_t ct = c | (1u << a);
                if (!te[a] && i == 5) return eb[a];
                if (!LABELS) return eb[a] | ct;
                const uint32_t at = vox + ((c >> 2) * S + ((c >> 1) & 1u)) * S + (c & 1u) - (a == 0 ? 1u : a == 1 ? S : S * S);
                return in[a] ? eb[a] | ct : inv[a] ? 0u : kChunkDone | at;
            };
            resolve8<OPEN>(v, [&](uint32_t c) { return (raw[c] & ~STP) ^ OPEN; }, pv, ext, inv, bad);
            if (with_bits) {
                uint32_t bits = 0;
#pragma unroll
                for (uint32_t c = 0; c < 8; ++c) bits |= (raw[c] & STP) ? 0u : 1u << c;
                ((uint8_t*)&cm.ep5[q >> 2].x)[q & 3u] = (uint8_t)bits;
            }
            ((uint4*)cm.buf)[2u * x] = make_uint4(v[0], v[1], v[2], v[3]);
            ((uint4*)cm.buf)[2u * x + 1u] = make_uint4(v[4], v[5], v[6], v[7]);
        }
        // operations of a parent that the next pass completes move to the front
        const uint32_t rest = rs.k & 7u, keep = tid < rest ? cm.buf[8u * n_par + tid] : 0u;
        lds_barrier();
        for (uint32_t x0 = 64u * wave_id(); x0 < n_par; x0 += NT) {
            const uint32_t x = x0 + lane_id();
            uint32_t open = 0, q = 0;
            if (x < n_par) {
                q = cm.list[r_next + x] & 0x7FFFu;  // (needed after the chains)
                const uint4 ra = ((const uint4*)cm.buf)[2u * x], rb = ((const uint4*)cm.buf)[2u * x + 1u];
                const uint32_t o[8] = {ra.x, ra.y, ra.z, ra.w, rb.x, rb.y, rb.z, rb.w};
#pragma unroll
                for (uint32_t c = 0; c < 8; ++c) open |= (o[c] & OPEN) ? 1u << c : 0u;
            }
            chase_open<uint32_t, OPEN>(cm.buf, 8u * x, open, refs, cap);
            if (x >= n_par) continue;
            const uint4 ra = ((const uint4*)cm.buf)[2u * x], rb = ((const uint4*)cm.buf)[2u * x + 1u];
            uint32_t v[8] = {ra.x, ra.y, ra.z, ra.w, rb.x, rb.y, rb.z, rb.w};
            // (loads at clamped places instead of branches around them, and none of
            // earlier results when no lane needs one)
            const bool any = __ballot(((v[0] | v[1] | v[2] | v[3] | v[4] | v[5] | v[6] | v[7]) & kChunkDone) != 0u);
            if (!LABELS) {
                uint32_t got[8];
                if (any)
#pragma unroll
                    for (uint32_t c = 0; c < 8; ++c) got[c] = cm.c5[(v[c] & kChunkDone) ? v[c] & (kChunkDone - 1u) : 0u];
#pragma unroll
                for (uint32_t c = 0; c < 8; ++c) v[c] = (v[c] & kChunkDone) ? got[c] : v[c] & 0xFFFFu;
                ((uint4*)cm.c5)[r_next + x] = pack8(v);
            } else {
                LT* const o = out + (compact3(q >> 2) * 2u * S + compact3(q >> 1) * 2u) * S + compact3(q) * 2u;
#pragma unroll
                for (uint32_t z = 0; z < 2; ++z) {  // (4 children at a time: registers)
                    LT l[4], got[4];
                    const uint32_t* const vz = v + 4u * z;
                    if (any)
#pragma unroll
                        for (uint32_t c = 0; c < 4; ++c) got[c] = out[(vz[c] & kChunkDone) ? vz[c] & (kChunkDone - 1u) : 0u];
                    if (cm.pal_lds) {
                        const LT* const lp = (const LT*)cm.pal_lds;
#pragma unroll
                        for (uint32_t c = 0; c < 4; ++c) l[c] = lp[(vz[c] & kChunkDone) ? 0u : min(vz[c], pc - 1u)];
                    } else {
#pragma unroll
                        for (uint32_t c = 0; c < 4; ++c) l[c] = pal[(vz[c] & kChunkDone) ? 0u : min(vz[c], pc - 1u)];
                    }
#pragma unroll
                    for (uint32_t c = 0; c < 4; ++c) l[c] = (vz[c] & kChunkDone) ? got[c] : l[c];
                    store2<LT>(o + z * S * S, l[0], l[1], vec);
                    store2<LT>(o + z * S * S + S, l[2], l[3], vec);
                }
            }
        }
        lds_barrier();
        if (tid < rest) cm.buf[tid] = keep;
        r_next += n_par;
    }
    if (bad) sh.err = 1u;
    adv = rs.adv;
    return rs.k == expected && rs.state == 0u && adv <= pc;
}

// Labels of the implied nodes of level t = 5 or 6 (children of the level t - 1
// nodes that do not expand), by pairs of such nodes along x.
template <int NT, typename LT, bool L6>
__device__ __forceinline__ void fill_implied(const Params& P, Shared& sh, const ChunkMem& cm, const LT* pal) {
    const uint32_t t = L6 ? 6u : 5u, S = 1u << t, hb = t - 1, H = 1u << hb, pc = uni(sh.h.pc);
    LT* const out = (LT*)(P.out + uni64(sh.h.out_off) * sizeof(LT));
    const bool vec = ((uintptr_t)out & (4 * sizeof(LT) - 1)) == 0;
    const uint2* const ep = L6 ? cm.ep5 : sh.EP + ebase(4);
    for (uint32_t u = threadIdx.x; u < (H >> 1) * H * H; u += NT) {
        const uint32_t px = u & ((H >> 1) - 1), qy = (u >> (hb - 1)) & (H - 1), qz = u >> (2 * hb - 1);
        const uint32_t q = spread3(2 * px) | (spread3(qy) << 1) | (spread3(qz) << 2);
        const uint32_t ex = (ep[q >> 5].x >> (q & 31)) & 3u;  // the x neighbour differs in bit 0
        if (ex == 3u) continue;
        LT l[2];
        uint32_t idx2;  // the two nodes' palette indices (level 5: they have one parent)
        if (L6) {
            const uint2 e4 = sh.EP[ebase(4) + (q >> 8)];
            const uint32_t p4 = q >> 3;
            idx2 = ep_bit(e4, p4) ? *(const uint32_t*)(cm.c5 + 8u * ep_rank(e4, p4) + (q & 7u))
                                  : (uint32_t)sh.G[fbase(4) + p4] * 0x10001u;
        } else {
            idx2 = *(const uint32_t*)(sh.G + fbase(4) + q);
        }
        const uint32_t i0 = min(idx2 & 0xFFFFu, pc - 1u), i1 = min(idx2 >> 16, pc - 1u);
        if (cm.pal_lds) {
            l[0] = ((const LT*)cm.pal_lds)[i0];
            l[1] = ((const LT*)cm.pal_lds)[i1];
        } else {
            l[0] = pal[i0];
            l[1] = pal[i1];
        }
        LT* const o = out + ((2 * qz) * S + 2 * qy) * S + 4 * px;
#pragma unroll
        for (uint32_t zy = 0; zy < 4; ++zy) {
            LT* const d = o + ((zy >> 1) * S + (zy & 1u)) * S;
            if (ex == 0u) store4<LT, false>(d, l[0], l[0], l[1], l[1], vec);
            else store2<LT>(d + (ex == 1u ? 2 : 0), l[ex & 1u], l[ex & 1u], vec);
        }
    }
}

template <int NT, typename LT>
__device__ __forceinline__ bool chunk_labels(const Params& P, Shared& sh, const ChunkMem& cm, const uint32_t* sym, uint32_t& adv,
                                             uint32_t& pbuf) {
    const uint32_t t = uni(sh.h.t);
    if (t == 6) fill_implied<NT, LT, true>(P, sh, cm, (const LT*)cm.pal);
    else fill_implied<NT, LT, false>(P, sh, cm, (const LT*)cm.pal);
    return chunk_level<NT, true, LT>(P, sh, cm, sym, t, uni(sh.nexp), adv, pbuf);
}

// Levels 4..t (0..3 are decoded); wavefront 0 computes a level's parent prefix
// before the barrier that ends it.  False (to every thread) on an error; labels:
// the output pass is left to do, from c5g (scratch) when it is set; pal_lds: the
// palette is in the list area.  sym_at: place of the symbols in the slot area (0:
// they are elsewhere); rows: level 5's slots in LDS.
template <int NT>
__device__ __forceinline__ bool decode_levels(const Params& P, Shared& sh, uint8_t* u_area, uint16_t* slots, uint8_t* scratch,
                                              const uint32_t* sym, uint32_t sym_at, uint16_t*& rows, uint16_t*& c5g, bool& labels, bool& pal_lds) {
    const uint32_t t = uni(sh.h.t), wave = wave_id();
    uint32_t adv = uni(sh.adv), pbuf = 0;
    bool ok = true;
    labels = true;
    if (t >= 4) {
        ok = full_level<NT>(sh, sym, 4, uni(sh.nexp), adv, pbuf, u_area, list_bytes(P.cap16));
        if (ok && t >= 5) {
            if (wave == 0) {
                const uint32_t n = level_prefix(sh.EP + ebase(4), ewords(4));
                if (threadIdx.x == 0) sh.nexp = n;
            }
            lds_barrier();
            const uint32_t nexp = uni(sh.nexp);
            // level 5 in LDS: the parent list from u_area on, the rows of slots behind
            // it, both before the level's symbols when those are in LDS (else they
            // go to scratch)
            const uint32_t o_rows = max(list_bytes(P.cap16), (2u * nexp + 15u) & ~15u), end5 = o_rows + 16u * nexp;
            const bool in_lds = t == 5 && end5 <= list_bytes(P.cap16) + slot_bytes(P.cap16) && uni(sh.h.pc) <= 32768u;
            if (sym_at && !(in_lds && end5 <= list_bytes(P.cap16) + sym_at + 4u * (uni(sh.h.sym_end[4]) >> 3))) {
                uint32_t* const nib = (uint32_t*)(scratch + P.scratch_sym);
                for (uint32_t q = threadIdx.x; q < (uni(sh.h.nsym) + 7u) / 8u; q += NT) nib[q] = sym[q];
                sym = nib;
                __syncthreads();
            }
            if (in_lds) {
                pal_lds = !P.pal_bits && uni(sh.h.pc) <= list_bytes(P.cap16) / 2u / P.label_bytes;
                rows = (uint16_t*)(u_area + o_rows);
                ok = level5<NT>(sh, sym, rows, u_area, o_rows, nexp, pal_lds ? uni(sh.h.pc) * P.label_bytes / 4u : 0u,
                                (const uint32_t*)(P.vol + uni64(sh.h.pal_off)), adv, pbuf);
            } else {
                ChunkMem cm;
                cm.ep5 = (uint2*)slots;
                cm.buf = (uint32_t*)(cm.ep5 + 1024);
                cm.cap = slot_bytes(P.cap16) / 4u - 2048u;
                cm.c5 = (uint16_t*)(scratch + kScrComp);
                cm.list = (uint32_t*)(scratch + kScrList);
                cm.pal = P.vol + uni64(sh.h.pal_off);
                cm.pal_lds = nullptr;
                const uint32_t pb = uni(sh.h.pc) * P.label_bytes;
                cm.work = u_area;
                cm.work_bytes = list_bytes(P.cap16);
                if (uni(sh.h.pc) <= kUBytesMin / 2u / P.label_bytes && !P.pal_bits) {  // (staged behind the next barrier)
                    for (uint32_t w = threadIdx.x; w < pb / 4u; w += NT) ((uint32_t*)u_area)[w] = ((const uint32_t*)cm.pal)[w];
                    cm.pal_lds = u_area;
                    cm.work += pb;
                    cm.work_bytes -= pb;
                }
                c5g = cm.c5;
                if (t == 6 || P.pal_bits) {
                    ok = chunk_level<NT, false, uint32_t>(params(), sh, cm, sym, 5, nexp, adv, pbuf);
                    if (ok && t == 6) {
                        if (wave == 0) {
                            const uint32_t n = level_prefix(cm.ep5, 1024u);
                            if (threadIdx.x == 0) sh.nexp = n;
                        }
                    }
                }
                __syncthreads();
                if (ok && !P.pal_bits) {
                    labels = false;
                    ok = P.label_bytes == 4 ? chunk_labels<NT, uint32_t>(params(), sh, cm, sym, adv, pbuf)
                                            : chunk_labels<NT, uint64_t>(params(), sh, cm, sym, adv, pbuf);
                }
            }
        }
    }
    lds_barrier();
    return ok && !(t == uni(sh.h.L) && adv != uni(sh.h.pc)) && !uni(sh.err);
}
// Labels of a level 5 in LDS as a 32^3 cube, x fastest, by pairs of 2x2x2 blocks
// along x under two level-4 nodes; a wavefront writes whole lines (the blocks of
// the expanding parents alone, written as they were decoded, left L2 with
// partly written lines: 0.41 ms against 0.28 for 4096 cubes of Voronoi cells).
// With the palette in LDS every block takes its 8 indices from a row of slots,
// a block of an implied node from a row made of its one value: looking 16
// indices up in every lane costs less than branching over the two kinds, which
// occur in nearly every wavefront.
template <int NT, typename LT, bool PAL_LDS>
__device__ __forceinline__ void write_labels5(const Params& P, Shared& sh, const uint8_t* u_area, const uint16_t* c5) {
    const uint32_t pc = uni(sh.h.pc), tid = threadIdx.x;
    LT* const out = (LT*)(P.out + uni64(sh.h.out_off) * sizeof(LT));
    const LT* const pal = PAL_LDS ? (const LT*)u_area : (const LT*)(P.vol + uni64(sh.h.pal_off));
    const bool vec = ((uintptr_t)out & (4 * sizeof(LT) - 1)) == 0;
    // unit u = px + 8 qy + 128 qz: the pair of level-4 nodes (2 px, qy, qz), (2 px + 1, qy, qz)
    const uint32_t px = tid & 7u, qy = (tid >> 3) & 15u;
    const uint32_t q_xy = spread3(2 * px) | (spread3(qy) << 1), at_xy = 64u * qy + 4u * px;
    for (uint32_t u = tid; u < 2048u; u += NT) {
        const uint32_t qz = u >> 7, q = q_xy | (spread3(qz) << 2);
        const uint2 e = sh.EP[ebase(4) + (q >> 5)];
        const uint32_t r = ep_rank(e, q), ex = e.x >> (q & 31);  // the x neighbour differs in bit 0
        const uint32_t f2 = *(const uint32_t*)(sh.G + fbase(4) + q);
        LT l[2][8];
#pragma unroll
        for (uint32_t hx = 0; hx < 2; ++hx) {
            const uint32_t f = hx ? f2 >> 16 : f2 & 0xFFFFu;
            const bool expl = (ex >> hx) & 1u;
            const uint4* const row = (const uint4*)c5 + (r + (hx & ex));
            if (PAL_LDS) {
                const uint32_t ff = f | (f << 16);
                uint4 w = make_uint4(ff, ff, ff, ff);
                if (expl) w = *row;
#pragma unroll
                for (uint32_t c = 0; c < 8; ++c) l[hx][c] = pal[half_of(w, c)];
            } else if (expl) {
                const uint4 w = *row;
#pragma unroll
                for (uint32_t c = 0; c < 8; ++c) l[hx][c] = pal_get<LT, false>(pal, half_of(w, c), pc);
            } else {
                const LT v = pal_get<LT, false>(pal, f, pc);
#pragma unroll
                for (uint32_t c = 0; c < 8; ++c) l[hx][c] = v;
            }
        }
        LT* const o = out + (at_xy + 2048u * qz);
#pragma unroll
        for (uint32_t zy = 0; zy < 4; ++zy)
            store4<LT>(o + ((zy >> 1) * 32u + (zy & 1u)) * 32u, l[0][2 * zy], l[0][2 * zy + 1], l[1][2 * zy], l[1][2 * zy + 1], vec);
    }
}

// Labels of level t <= 4 (all slots final) as an S^3 x-fastest cube, 4 voxels
// per thread.
template <int NT, typename LT, bool PAL_LDS, typename SH>
__device__ __forceinline__ void write_labels(const Params& P, SH& sh, const LT* lds_pal) {
    const TaskHdr& h = sh.h;
    const uint32_t t = uni(h.t), S = 1u << t, pc = uni(h.pc);
    LT* out = (LT*)(P.out + uni64(h.out_off) * sizeof(LT));
    const LT* pal = PAL_LDS ? lds_pal : (const LT*)(P.vol + uni64(h.pal_off));
    const bool vec = ((uintptr_t)out & (4 * sizeof(LT) - 1)) == 0;
    const uint16_t* g = sh.G + fbase(t);
    if (S < 4) {
        const uint32_t n = S * S * S;
        for (uint32_t v = threadIdx.x & (NT - 1); v < n; v += NT) {
            const uint32_t x = v & (S - 1), y = (v >> t) & (S - 1), z = v >> (2 * t);
            const LT l = pal_get<LT, PAL_LDS>(pal, g[spread3(x) | (spread3(y) << 1) | (spread3(z) << 2)], pc);
            __builtin_nontemporal_store(l, out + v);
        }
        return;
    }
    const uint32_t units = (S * S * S) >> 2;
    for (uint32_t u = threadIdx.x & (NT - 1); u < units; u += NT) {
        const uint32_t lin = u << 2;
        const uint32_t x = lin & (S - 1), y = (lin >> t) & (S - 1), z = lin >> (2 * t);
        const uint32_t m = spread3(x) | (spread3(y) << 1) | (spread3(z) << 2);
        store4<LT>(out + lin, pal_get<LT, PAL_LDS>(pal, g[m], pc), pal_get<LT, PAL_LDS>(pal, g[m + 1], pc),
                   pal_get<LT, PAL_LDS>(pal, g[m + 8], pc), pal_get<LT, PAL_LDS>(pal, g[m + 9], pc), vec);
    }
}

// Cache-paletted output: the cube's palette indices, I bits each, floor(32/I)
// to a 32-bit word (voxel k, x fastest, in word k / e at bit (k mod e) * I).
// The index of voxel v; level 5 (c5: explicit nodes by rank) is reached through
// the level-4 parent.
template <typename SH>
__device__ __forceinline__ uint32_t voxel_index(const SH& sh, const uint16_t* c5, uint32_t t, uint32_t v) {
    const uint32_t mask = (1u << t) - 1u;
    const uint32_t m = spread3(v & mask) | (spread3((v >> t) & mask) << 1) | (spread3(v >> (2 * t)) << 2);
    if (t <= 4) return sh.G[fbase(t) + m];
    const uint2 ep = sh.EP[ebase(4) + (m >> 8)];
    return ep_bit(ep, m >> 3) ? c5[8u * ep_rank(ep, m >> 3) + (m & 7u)] : sh.G[fbase(4) + (m >> 3)];
}

// One thread per word, voxel by voxel: cubes of side <= 8, and larger ones
// where the rows below find no room.
template <int NT, typename SH>
__device__ __forceinline__ void write_indices(const Params& P, SH& sh, const uint16_t* c5) {
    const TaskHdr& h = sh.h;
    const uint32_t t = uni(h.t), bits = P.pal_bits, e = 32u / bits, n = 1u << (3 * t), words = (n + e - 1u) / e;
    uint32_t* const out = (uint32_t*)P.out + uni64(h.out_off);
    for (uint32_t w = threadIdx.x & (NT - 1); w < words; w += NT) {
        uint32_t acc = 0;
        for (uint32_t q = 0; q < e && w * e + q < n; ++q) acc |= voxel_index(sh, c5, t, w * e + q) << (q * bits);
        __builtin_nontemporal_store(acc, out + w);
    }
}

// Cubes of side 16 and 32: every wavefront lays 512 voxels at a time (half a
// plane, two planes) out in raster order in LDS, from whole pairs of values, and
// packs words from there; voxels of a word that 512 voxels end in move to the
// front of the next 512.  Per voxel that is a 16-bit LDS read and a shift, where
// finding each voxel's node takes its Morton code and two lookups: 4096 cubes of
// 32^3 neurites at 6 bits, 0.499 -> 0.348 ms; of Voronoi cells at 12 bits, 0.410
// -> 0.279 (their labels: 0.280 and 0.227).  Bound by instruction issue.
constexpr uint32_t kRasterVoxels = 512;
constexpr uint32_t kRasterBytes = 2u * (32u + kRasterVoxels + 32u);  // leftover voxels | 512 | zeros past the cube

template <int NT>
__device__ __forceinline__ void write_indices_raster(const Params& P, Shared& sh, const uint16_t* c5, uint16_t* st) {
    const uint32_t t = uni(sh.h.t), bits = P.pal_bits, e = 32u / bits, n = 1u << (3 * t), lane = lane_id();
    uint32_t* const out = (uint32_t*)P.out + uni64(sh.h.out_off);
    const uint32_t per = max(n / kRasterVoxels / (NT / 64), 1u), s0 = wave_id() * per * kRasterVoxels;
    if (s0 >= n) return;
    uint32_t w = s0 / e;  // the first word that is not whole before voxel s0
    const uint32_t left0 = s0 - w * e;
    if (lane < left0) st[32u - left0 + lane] = (uint16_t)voxel_index(sh, c5, t, w * e + lane);
    if (lane < 16u) ((uint32_t*)(st + 32u + kRasterVoxels))[lane] = 0u;
    // a lane's 8 voxels of the 512 from v0 on: 4 voxels of 2 rows, from half the
    // children of two level-4 nodes, or twice 4 voxels of level 4 along x
    uint2 lo, hi;
    const uint32_t q_lane = t == 5 ? spread3(2u * (lane & 7u)) | (spread3(lane >> 3) << 1) : spread3(4u * (lane & 3u)) | (spread3(lane >> 2) << 1);
    const auto values = [&](uint32_t v0) {
        if (t == 5) {
            const uint32_t z = v0 >> 10, q = q_lane | (spread3((v0 >> 6) & 8u) << 1) | (spread3(z >> 1) << 2);
            const uint2 ep = sh.EP[ebase(4) + (q >> 5)];
            const uint32_t r = ep_rank(ep, q), ex = ep.x >> (q & 31u);
            const uint32_t f2 = *(const uint32_t*)(sh.G + fbase(4) + q);
            const uint2* const row = (const uint2*)c5 + (2u * r + (z & 1u));
            lo.x = hi.x = (f2 & 0xFFFFu) * 0x10001u;
            lo.y = hi.y = (f2 >> 16) * 0x10001u;
            if (ex & 1u) lo.x = row[0].x, hi.x = row[0].y;
            if (ex & 2u) lo.y = row[2u * (ex & 1u)].x, hi.y = row[2u * (ex & 1u)].y;
        } else {
            const uint16_t* const g = sh.G + (fbase(4) + (q_lane | (spread3(v0 >> 8) << 2)));  // (v0 >> 8 is even: the next plane is 4 nodes on)
            lo = make_uint2(*(const uint32_t*)g, *(const uint32_t*)(g + 8));
            hi = make_uint2(*(const uint32_t*)(g + 4), *(const uint32_t*)(g + 12));
        }
    };
    const uint32_t at = t == 5 ? 16u * (lane >> 3) + (lane & 7u) : lane, up = t == 5 ? 8u : 64u;
    values(s0);
    for (uint32_t v0 = s0; v0 < s0 + per * kRasterVoxels; v0 += kRasterVoxels) {
        ((uint2*)(st + 32u))[at] = lo;
        ((uint2*)(st + 32u))[at + up] = hi;
        lsync<64>();
        values(min(v0 + kRasterVoxels, n - kRasterVoxels));  // in flight while the words are packed
        const uint32_t end = v0 + kRasterVoxels, w_end = end < n ? end / e : (n + e - 1u) / e;
        const uint16_t* src = st + (32u + (w + lane) * e - v0);
        for (uint32_t x = w + lane; x < w_end; x += 64u, src += 64u * e) {
            uint32_t acc = src[0];
            uint32_t k = 1;
            for (; k + 3u < e; k += 4u) {
                const uint32_t a0 = src[k], a1 = src[k + 1], a2 = src[k + 2], a3 = src[k + 3], at4 = k * bits;
                acc |= (a0 << at4) | (a1 << (at4 + bits)) | (a2 << (at4 + 2u * bits)) | (a3 << (at4 + 3u * bits));
            }
            for (; k < e; ++k) acc |= (uint32_t)src[k] << (k * bits);
            __builtin_nontemporal_store(acc, out + x);
        }
        w = w_end;
        const uint32_t left = end < n ? end - w * e : 0u;
        uint16_t keep = 0;
        if (lane < left) keep = st[32u + kRasterVoxels - left + lane];
        lsync<64>();
        if (lane < left) st[32u - left + lane] = keep;
    }
}

// Packed output of a work-group's cube.  Free at this point: the list area up to
// level 5's rows and what lies behind them; all of both after a level 5 in
// scratch (c5g); for a level 4 what lies behind the rANS table, which stays.
template <int NT>
__device__ __forceinline__ void write_paletted(const Params& P, Shared& sh, uint8_t* u_area, uint16_t* rows, const uint16_t* c5g) {
    const uint32_t t = uni(sh.h.t), area = list_bytes(P.cap16) + slot_bytes(P.cap16);
    uint32_t a = list_bytes(P.cap16), b = a + 4u * kRansM;  // free: [0, a) and [b, area)
    if (t == 5) {
        a = c5g ? area : (uint32_t)((uint8_t*)rows - u_area);
        b = c5g ? area : a + 16u * uni(sh.nexp);
    }
    const uint32_t n_a = a / kRasterBytes, n = n_a + (area - b) / kRasterBytes, wave = wave_id();
    if (t < 4 || n < min(NT / 64u, (1u << (3u * t)) / kRasterVoxels)) {
        if (c5g) write_indices<NT>(P, sh, c5g);
        else write_indices<NT>(P, sh, rows);
    } else {
        uint16_t* const st = (uint16_t*)(u_area + (wave < n_a ? wave * kRasterBytes : b + (wave - n_a) * kRasterBytes));
        if (c5g) write_indices_raster<NT>(P, sh, c5g, st);
        else write_indices_raster<NT>(P, sh, rows, st);
    }
}

// Output pass; c5g: the level-5 palette indices in scratch (null: slots in LDS);
// pal_lds: the palette is staged already (level 5).
template <int NT, typename LT>
__device__ __forceinline__ void write_output(const Params& P, Shared& sh, uint8_t* u_area, const uint16_t* slots, bool pal_lds) {
    const uint32_t t = uni(sh.h.t), pc = uni(sh.h.pc);
    if (t == 5) {
        if (pal_lds) write_labels5<NT, LT, true>(P, sh, u_area, slots);
        else write_labels5<NT, LT, false>(P, sh, u_area, slots);
    } else if (t == 4 && pc <= list_bytes(P.cap16) / (uint32_t)sizeof(LT)) {
        const uint32_t* src = (const uint32_t*)(P.vol + uni64(sh.h.pal_off));
        for (uint32_t w = threadIdx.x; w < pc * (uint32_t)sizeof(LT) / 4u; w += NT) ((uint32_t*)u_area)[w] = src[w];
        lds_barrier();
        write_labels<NT, LT, true>(P, sh, (const LT*)u_area);
    } else {  // (a cube of side <= 8 reads its few labels straight from the record)
        write_labels<NT, LT, false>(P, sh, (const LT*)nullptr);
    }
}

// ------------------------------------------------------------------ a task
template <int NT>
__device__ __forceinline__ void decode_task(const Params& P, uint8_t* lds, uint8_t* scratch, Ahead& ah) {
    Shared& sh = *reinterpret_cast<Shared*>(lds);
    const TaskHdr& h = sh.h;
    if (uni(h.status) != kTaskOk) {
        if (uni(h.status) == kTaskCorrupt && uni(h.write_ok)) zero_output<NT>(params(), h);
        return;
    }
    const uint32_t u_bytes = list_bytes(P.cap16);
    uint8_t* const u_area = lds + sizeof(Shared);
    uint16_t* const slots = (uint16_t*)(u_area + u_bytes);
    // The symbols, 4 bits each, are read by the level passes as aligned 32-bit
    // words: plain payloads from the record itself, rANS symbols from LDS when they
    // fit there together with the record's words and the decoding table (`fits`, as
    // nearly all of a 32^3 brick do), else from the work-group's scratch.
    const uint32_t wave = wave_id(), t = uni(h.t), nsym = uni(h.nsym), n_words = (nsym + 7u) / 8u;
    const bool rans = uni(h.coder) == kRans;
    // While the symbols are decoded: the words between the level 0..3 grids and
    // the slot area, the decoding table in its first 16 KiB (it stays until a
    // level 5 overwrites it; later tasks find it there until then), the symbols at
    // its end, where the level passes read them.
    constexpr uint32_t kLoGrid = 1280;  // bytes of the level 0..3 grids (1184), rounded up
    const uint32_t o_words = (uint32_t)offsetof(Shared, G) + kLoGrid;
    const uint32_t o_tab = (uint32_t)sizeof(Shared) + u_bytes, o_end = o_tab + slot_bytes(P.cap16);
    const uint32_t G = rans ? ((1u << uni(h.log2W)) + 63u) / 64u : 0u;
    const uint64_t words = rans ? (uint64_t)uni(h.gstart[G - 1]) + uni(h.gw[G - 1]) : 0u;
    const uint32_t sym_bytes = symbol_bytes(nsym);
    // (a round may read up to 63 words past a group's end)
    const bool fits = rans && o_words + 2u * words + 16u + 128u <= o_tab && o_tab + 4u * kRansM + sym_bytes + 16u <= o_end;
    const uint32_t words_bytes = fits ? (2u * (uint32_t)words + 15u) & ~15u : 0u, o_sym = fits ? (o_end - sym_bytes) & ~15u : 0u;
    // Overlap, for a cube with a level 3 whose lane groups leave a wavefront free:
    // wavefronts 0..G-1 decode the lane groups, wavefront G decodes levels 0..3 as
    // soon as every group is past their symbols.  (two or more lanes: a round
    // writes whole bytes of symbol pairs)
    const bool overlap = fits && G < NT / 64 && uni(h.log2W) >= 1u && t >= 3;
    const uint32_t small = min(t, 3u), need = uni(h.sym_end[small]);
    uint8_t* const nib = scratch + P.scratch_sym;
    const uint32_t* sym = fits ? (const uint32_t*)(lds + o_sym) : (const uint32_t*)nib;
    uint32_t x0 = 0;
    if (!rans) {
        if (uni64(h.pay_off) + 4ull * max(n_words, 1u) <= P.vol_bytes) {
            sym = (const uint32_t*)(P.vol + uni64(h.pay_off));
        } else {  // the last record's last word would end past the container
            for (uint32_t b = threadIdx.x; b < (nsym + 1u) / 2u; b += NT) nib[b] = P.vol[uni64(h.pay_off) + b];
            __syncthreads();
        }
    } else {
        if (threadIdx.x < 4) sh.prog[threadIdx.x] = 0;
        x0 = rans_stage<NT>(params(), h, (uint16_t*)(lds + o_words), words_bytes, uni(sh.tab_ok) ? nullptr : (uint4*)(lds + o_tab));
        lds_barrier();
    }
    // step 0 decodes the symbols; step 1 levels 0..3, on one wavefront, while lane
    // 0 of the last wavefront parses the next task; with overlap both in step 1
#pragma nounroll
    for (uint32_t step = rans && !overlap ? 0u : 1u; step < 2u; ++step) {
        const uint32_t* const tab = (const uint32_t*)(lds + o_tab);
        if (fits && (step == 0u || wave < (overlap ? G : 0u))) {
            rans_rounds<NT>(params(), sh, tab, (const uint16_t*)(lds + o_words), lds + o_sym, x0, overlap ? max(need, 1u) : 0u);
        } else if (step == 0u) {
            if (uni(h.log2W) >= 6u && kStreamBytes * (NT / 64) <= o_tab - o_words) rans_stream<NT>(params(), sh, tab, lds + o_words, nib);
            else rans_decode<NT>(params(), sh, tab, nib);
            __syncthreads();
        } else if (wave == (overlap ? G : 0u)) {
            // bounded: every group publishes ~0 when its rounds end
            if (overlap)
                for (uint32_t g = 0; g < G; ++g)
                    while (__hip_atomic_load(&sh.prog[g], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < need)
                        __builtin_amdgcn_s_sleep(1);
            small_levels(sh, sym, small, (uint8_t*)sh.refs, (uint32_t)sizeof(sh.refs));
        } else if (threadIdx.x == NT - 64 && !ah.done) {
            parse_ahead(params(), sh, ah.jt);
            ah.done = true;
        }
        lds_barrier();
    }
    // (sh.err is not written again before the next barrier)
    bool ok = !uni(sh.err);
    if (ok) {
        uint16_t *rows = slots, *c5g = nullptr;
        bool labels, pal_lds = false;
        ok = decode_levels<NT>(params(), sh, u_area, slots, scratch, sym, fits ? o_sym - o_tab : 0u, rows, c5g, labels, pal_lds);
        if (ok && labels) {
            if (P.pal_bits) {
                write_paletted<NT>(params(), sh, u_area, rows, c5g);
            } else if (P.label_bytes == 4) {
                write_output<NT, uint32_t>(params(), sh, u_area, rows, pal_lds);
            } else {
                write_output<NT, uint64_t>(params(), sh, u_area, rows, pal_lds);
            }
        }
    }
    if (!ok) {
        __syncthreads();  // the zeros come after what the work-group has written
        if (threadIdx.x == 0) sh.h.status = kTaskCorrupt;
        zero_output<NT>(params(), h);
    }
    // (read again only after the task loop's next barriers)
    if (threadIdx.x == 0) sh.tab_ok = t >= 5 ? 0u : rans ? 1u : sh.tab_ok;
}

// ------------------------------------------------------- tasks of one wavefront
// Cubes of side <= 8 have at most 585 nodes, which one wavefront decodes alone, as
// it does levels 0..3 of any cube: in a work-group of four wavefronts three would
// wait for most of such a task.  When the lists of larger tasks are used up, up
// to four wavefronts of a work-group each take tasks of their own, with no
// barrier among them; the rANS table in LDS is shared.  Kernel time of 1400
// neurite cubes of side 8: 0.066 -> 0.034 ms (0.025 with lane_level); 4096 of side
// 2..16: 0.107 -> 0.080 (0.063).
struct WaveShared {
    TaskHdr q[4];  // the tasks of a claim, parsed by one lane each
    TaskHdr h;     // the task being decoded
    uint32_t err, nexp, adv, prog[1];
    alignas(16) uint4 pub[1][1];
    alignas(16) uint2 EP[20];      // levels 0..3
    alignas(16) uint16_t G[592];
    alignas(16) uint32_t pal[128];
};
constexpr uint32_t kWaves = 4;
static_assert(sizeof(WaveShared) % 16 == 0 && kWaves * sizeof(WaveShared) <= sizeof(Shared::G) + kUBytesMin,
              "the wavefronts' areas take the place of the grids and the parent list");

__device__ __forceinline__ void wave_task(const Params& P, WaveShared& ws, const uint32_t* tab, uint8_t* area, uint32_t area_bytes,
                                          uint8_t* nib) {
    const TaskHdr& h = ws.h;
    const uint32_t lane = lane_id(), nsym = uni(h.nsym), n_words = (nsym + 7u) / 8u, t = uni(h.t), pc = uni(h.pc);
    const uint32_t* sym = (const uint32_t*)nib;
    if (t > 3u || nsym > kWaveSyms) {  // (the binning kernel does not hand such a task over)
        ws.err = 1u;
        return;
    }
    const uint32_t pal_bytes = pc <= sizeof(ws.pal) / P.label_bytes && !P.pal_bits ? pc * P.label_bytes : 0u;
    uint32_t pw[2];
#pragma unroll
    for (uint32_t k = 0; k < 2; ++k)
        pw[k] = 4u * (64u * k + lane) < pal_bytes ? ((const uint32_t*)(P.vol + uni64(h.pal_off)))[64u * k + lane] : 0u;
    if (uni(h.coder) == kRaw4) {
        if (uni64(h.pay_off) + 4ull * max(n_words, 1u) <= P.vol_bytes) {
            sym = (const uint32_t*)(P.vol + uni64(h.pay_off));
        } else {  // the last record's last word would end past the container
            for (uint32_t b = lane; b < (nsym + 1u) / 2u; b += 64u) nib[b] = P.vol[uni64(h.pay_off) + b];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
    } else {
        // the words that the cube's symbols can need, group by group behind the symbols
        const uint32_t W = 1u << uni(h.log2W), G = (W + 63u) / 64u;
        const uint32_t x0 = lane < W ? ((const uint32_t*)(P.vol + uni64(h.states_off)))[lane] : 0u;
        uint32_t at = (4u * n_words + 15u) & ~15u;
        bool fits = true;
        uint32_t from[4], to[4];
#pragma unroll
        for (uint32_t g = 0; g < 4; ++g) {
            from[g] = to[g] = 0;
            if (g < G && 64u * g < nsym) {
                const uint32_t rounds = (nsym - 64u * g + W - 1u) / W, start = uni(h.gstart[g]);
                const uint32_t n = min(uni(h.gw[g]), 64u * rounds) + (start & 1u);
                fits = fits && uni64(h.pay_off) + 2ull * (start & ~1u) + ((2u * n + 15u) & ~15u) <= P.vol_bytes;
                from[g] = at;
                at += (2u * n + 15u) & ~15u;
                to[g] = at;
            }
        }
        if (fits && at + 128u <= area_bytes) {
#pragma unroll
            for (uint32_t g = 0; g < 4; ++g) {
                if (g < G) {
                    const uint32_t start = uni(h.gstart[g]);
                    const uint8_t* const src = P.vol + uni64(h.pay_off) + 2ull * (start & ~1u);
                    for (uint32_t o = 16u * lane; from[g] + o < to[g]; o += 1024u) {
                        const u32x4_a4 v = *(const u32x4_a4*)(src + o);
                        *(uint4*)(area + from[g] + o) = make_uint4(v[0], v[1], v[2], v[3]);
                    }
                    if (lane == 0) ws.h.gstart[g] = from[g] / 2u + (start & 1u);  // now within `area`
                }
            }
            lsync<64>();
            rans_rounds<64>(params(), ws, tab, (const uint16_t*)area, area, x0, 0u);
            sym = (const uint32_t*)area;
        } else {
            rans_decode<64>(params(), ws, tab, nib);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
    }
#pragma unroll
    for (uint32_t k = 0; k < 2; ++k)
        if (4u * (64u * k + lane) < pal_bytes) ws.pal[64u * k + lane] = pw[k];
    lsync<64>();
    const uint32_t used = sym == (const uint32_t*)area ? (4u * n_words + 15u) & ~15u : 0u;
    small_levels(ws, sym, t, area + used, area_bytes - used);
    lsync<64>();
    if (uni(ws.err) || (t == uni(h.L) && uni(ws.adv) != pc)) {
        ws.err = 1u;
        return;
    }
    if (P.pal_bits) write_indices<64>(params(), ws, (const uint16_t*)nullptr);
    else if (P.label_bytes == 4 && pal_bytes) write_labels<64, uint32_t, true>(params(), ws, (const uint32_t*)ws.pal);
    else if (P.label_bytes == 4) write_labels<64, uint32_t, false>(params(), ws, (const uint32_t*)nullptr);
    else if (pal_bytes) write_labels<64, uint64_t, true>(params(), ws, (const uint64_t*)ws.pal);
    else write_labels<64, uint64_t, false>(params(), ws, (const uint64_t*)nullptr);
}

template <int NT>
__device__ __forceinline__ void wave_tasks(const Params& P, uint8_t* lds, uint8_t* scratch) {
    Shared& sh = *reinterpret_cast<Shared*>(lds);
    static_assert(kClasses == kWgClasses + 2, "two lists");
    const uint32_t n_first = uni(sh.job[kWgClasses]), n = n_first + uni(sh.job[kWgClasses + 1]);
    if (n == 0u) return;
    constexpr uint32_t NW = NT / 64 < kWaves ? NT / 64 : kWaves;
    const uint32_t u_bytes = list_bytes(P.cap16), o_tab = (uint32_t)sizeof(Shared) + u_bytes, wave = wave_id(), lane = lane_id();
    if (!uni(sh.tab_ok))
        for (uint32_t w = threadIdx.x; w < kRansM / 4; w += NT) ((uint4*)(lds + o_tab))[w] = ((const uint4*)P.rans_tab)[w];
    lds_barrier();
    WaveShared& ws = *reinterpret_cast<WaveShared*>(lds + offsetof(Shared, G) + min(wave, NW - 1u) * sizeof(WaveShared));
    const uint32_t area_bytes = ((slot_bytes(P.cap16) - 4u * kRansM) / kWaves) & ~15u;
    uint8_t* const area = lds + o_tab + 4u * kRansM + wave * area_bytes;
    uint8_t* const nib = scratch + P.scratch_sym + wave * (kWaveSyms / 2u);
    // A work-group's claim is up to 4 tasks for each wavefront, which parses them
    // side by side: as many as give every work-group one claim.  (Claims of single
    // wavefronts took 70 us of a launch of 3000 cubes on the counter.)  Without
    // tasks for work-groups the first claim is the work-group's own number.
    const uint32_t per = min((n + gridDim.x * NW - 1u) / (gridDim.x * NW), 4u), claims = (n + NW * per - 1u) / (NW * per);
    const bool fixed = uni(sh.n_jobs) == 0u;
    uint32_t j = uni(sh.small[0]), turn = 0;
    while (j < claims) {
        uint32_t ahead = 0xFFFFFFFFu;
        if (threadIdx.x == 0 && !(fixed && claims <= gridDim.x)) ahead = (fixed ? gridDim.x : 0u) + atomicAdd(&P.ctl->small, 1u);
        const uint32_t k0 = (j * NW + wave) * per, m = wave < NW && k0 < n ? min(per, n - k0) : 0u;
        if (lane < m) {
            const uint32_t k = k0 + lane;
            const uint32_t task = k < n_first ? P.lists[(uint64_t)kWgClasses * P.list_cap + k]
                                              : P.lists[(uint64_t)(kWgClasses + 1) * P.list_cap + (k - n_first)];
            parse_task(params(), task, ws.q[lane]);
        }
        lsync<64>();
        for (uint32_t x = 0; x < m; ++x) {
            if (lane < sizeof(TaskHdr) / 4) ((uint32_t*)&ws.h)[lane] = ((const uint32_t*)&ws.q[x])[lane];
            if (lane == 0) ws.err = 0;
            lsync<64>();
            uint32_t status = uni(ws.h.status);
            if (status == kTaskOk) {
                wave_task(params(), ws, (const uint32_t*)(lds + o_tab), area, area_bytes, nib);
                lsync<64>();
                if (uni(ws.err)) status = kTaskCorrupt;
            }
            if (status == kTaskCorrupt && uni(ws.h.write_ok)) zero_output<64>(params(), ws.h);
            if (lane == 0 && P.status) P.status[uni(ws.h.task)] = status;
            lsync<64>();
        }
        turn ^= 1u;
        if (threadIdx.x == 0) sh.small[turn] = ahead;
        lds_barrier();
        j = uni(sh.small[turn]);
    }
}

// at least 4 waves per SIMD: 128 VGPRs per lane at most
template <int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) decode_kernel(Params P) {
    extern __shared__ uint8_t dyn_smem[];
    Shared& sh = *reinterpret_cast<Shared*>(dyn_smem);
    const uint32_t tid = threadIdx.x;
    uint8_t* scratch = P.scratch + (uint64_t)blockIdx.x * P.scratch_stride;
    // lane 0 of the last wavefront claims and parses the next task while the
    // current one is decoded (the atomic's and the header loads' latency hide
    // behind the decode)
    constexpr uint32_t PT = NT - 64;
    Ahead ah{0u, true};
    if (tid == PT) {
        uint32_t n = P.n_tasks;
        if (P.lists) {
            n = 0;
#pragma unroll
            for (uint32_t c = 0; c < kClasses; ++c) {
                const uint32_t k = sh.job[c] = P.ctl->job[c];
                n += c < kWgClasses ? k : 0u;
            }
        }
        sh.n_jobs = n;
        ah.jt = blockIdx.x;
        parse_ahead(params(), sh, ah.jt);
    }
    if (tid == 0) sh.tab_ok = 0;
    for (;;) {
        lds_barrier();  // sh.hn is parsed, the last task's status written
        if (tid < sizeof(TaskHdr) / 4) ((uint32_t*)&sh.h)[tid] = ((const uint32_t*)&sh.hn)[tid];
        if (tid == 0) sh.err = 0;
        lds_barrier();
        const uint32_t task = uni(sh.h.task);
        if (task == 0xFFFFFFFFu) break;
        if (tid == PT) {
            ah.jt = claim(params(), sh, ah.jt);
            ah.done = false;
        }
        decode_task<NT>(params(), dyn_smem, scratch, ah);
        if (tid == PT && !ah.done) {
            parse_ahead(params(), sh, ah.jt);
            ah.done = true;
        }
        if (tid == 0 && P.status) P.status[task] = uni(sh.h.status);
    }
    if (P.lists) wave_tasks<NT>(params(), dyn_smem, scratch);
}

// ------------------------------------------------------------ small kernels
// The control words of a one-shot call and the volume's rANS decoding table:
// slot -> symbol | freq << 4 | (slot - cum) << 17
__device__ __forceinline__ void table_slot(uint32_t* tab, const RansFreq& f, uint32_t slot) {
    uint32_t cum = 0, s = 0, fs = 0;
    for (uint32_t k = 0; k < 16; ++k) {
        const uint32_t fk = (f.w[k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
        if (slot >= cum && slot < cum + fk) {
            s = k;
            fs = fk;
            break;
        }
        cum += fk;
    }
    tab[slot] = s | (fs << 4) | ((slot - cum) << 17);
}

__global__ void prepare_kernel(Control* ctl, uint32_t* tab, RansFreq f) {
    const uint32_t slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (ctl && slot < sizeof(Control) / 4) ((uint32_t*)ctl)[slot] = 0;
    if (tab && slot < kRansM) table_slot(tab, f, slot);
}

// side exponent of a task's cube (0xFF when the task or record is unusable)
__device__ __forceinline__ uint32_t task_t(const Params& P, uint32_t j, uint64_t* rec_bytes) {
    const uint32_t id = P.ids[j];
    *rec_bytes = 0;
    if (id >= P.n_bricks) return 0xFFu;
    const uint64_t* offs = (const uint64_t*)(P.vol + P.off_pos);
    const uint64_t a = offs[id], b = offs[id + 1];
    if (a > b || b > P.vol_bytes || (a & 7) || b - a < 8) return 0xFFu;
    *rec_bytes = b - a;
    const uint32_t L = P.vol[a + 1];
    const uint32_t lod = P.lods[j];
    if (L < 1 || L > kMaxLog2b || lod > L) return 0xFFu;
    return L - lod;
}

// Lanes of one wavefront grouped by class: for every distinct class c among
// the lanes with c < 64, f(c, mask of the lanes holding it) runs once, with
// the lowest such lane as the leader: a lane's rank among its class and the
// wavefront's count of it, from which the block takes one atomic per class.
template <typename F>
__device__ __forceinline__ void for_each_class(uint32_t c, F f) {
    uint64_t left = __ballot(c < 64u);
    while (left) {
        const uint32_t lead = (uint32_t)__builtin_ctzll(left);
        const uint32_t cc = (uint32_t)__builtin_amdgcn_readlane((int)c, (int)lead);
        const uint64_t m = __ballot(c == cc);
        f(cc, m, lead);
        left &= ~m;
    }
}

// Cost class of a task: the cube's side, then the compressed size; a cube takes
// longer the more of it is explicit, which its record's bytes follow.
__device__ __forceinline__ uint32_t cost_class(const Params& P, uint32_t id, uint32_t t, uint64_t rec_bytes) {
    if (t > kMaxLog2b) return kClasses - 1;  // unusable: refused when it is parsed
    if (t <= 3 && rec_bytes >= 12u + 4u * t) {  // (a shorter record is refused too)
        const uint64_t a = ((const uint64_t*)(P.vol + P.off_pos))[id];
        if (ld32(P.vol + a + 8u + 4u * t) > kWaveSyms) return 3u;
    }
    const bool heavy = rec_bytes > (t == 6 ? 65536u : 8192u);
    return t == 6 ? (heavy ? 0u : 1u) : t == 5 ? (heavy ? 1u : 2u) : t == 4 ? 3u : t == 3 ? 4u : 5u;
}

// One pass over the tasks, kBinTasks per block: each goes to its class's list
// (one atomic per block and class), and with `dense` it gets its output offset
// within the block; the block that finishes last turns the blocks' totals into
// the blocks' own offsets.  A task that names no brick is refused here and goes
// to no list.  (One launch; a histogram, a scan and a scatter took four, 4.7 us
// each.)  The blocks from `bins` on build the rANS table, for a one-shot call whose
// tasks are one block's: that block needs no control words set before it, so the
// call has no other kernel before the decode (64 bricks, packed: 47.6 -> 43.1 us).
__global__ void __launch_bounds__(kBinTasks) bin_kernel(Params P, uint32_t* lists, uint64_t* dense, uint64_t* base,
                                                        uint64_t* totals, uint32_t bins, uint32_t* tab, RansFreq f) {
    __shared__ uint32_t cnt[4][8];
    __shared__ uint32_t first[8];
    __shared__ uint64_t wsum[4];
    __shared__ uint32_t last;
    if (blockIdx.x >= bins) {
        const uint32_t slot = (blockIdx.x - bins) * kBinTasks + threadIdx.x;
        if (slot < kRansM) table_slot(tab, f, slot);
        return;
    }
    if (!lists && !dense) {  // nothing to do but the control words
        if (threadIdx.x < sizeof(Control) / 4) ((uint32_t*)P.ctl)[threadIdx.x] = 0;
        return;
    }
    const uint32_t tid = threadIdx.x, j = blockIdx.x * kBinTasks + tid, lane = lane_id(), wave = tid >> 6;
    uint64_t rec = 0;
    const bool in = j < P.n_tasks;
    const uint32_t t = in ? task_t(P, j, &rec) : 0xFFu;
    if (lists) {
        uint32_t c = 64;
        if (in) {
            if (P.ids[j] < P.n_bricks) c = cost_class(P, P.ids[j], t, rec);
            else if (P.status) P.status[j] = kTaskInvalid;
        }
        if (lane < 8) cnt[wave][lane] = 0;
        uint32_t rank = 0;
        for_each_class(c, [&](uint32_t cc, uint64_t m, uint32_t lead) {
            if (c == cc) rank = mbcnt(m);
            if (lane == lead) cnt[wave][cc] = (uint32_t)__popcll(m);
        });
        __syncthreads();
        if (tid < kClasses) {
            const uint32_t tot = cnt[0][tid] + cnt[1][tid] + cnt[2][tid] + cnt[3][tid];
            first[tid] = bins == 1u ? 0u : tot ? atomicAdd(&P.ctl->count[tid], tot) : 0u;
        }
        __syncthreads();
        if (c < kClasses) {
            uint32_t pos = first[c] + rank;
            for (uint32_t w = 0; w < wave; ++w) pos += cnt[w][c];
            lists[(uint64_t)c * P.list_cap + pos] = j;
        }
    }
    // exclusive prefix of the tasks' cube sizes (labels, or words of packed
    // indices) in task order; an unusable task occupies nothing
    const uint64_t sz = t <= kMaxLog2b ? out_units(1ull << (3 * t), P.pal_bits) : 0;
    auto block_scan = [&](uint64_t v, uint64_t* total) -> uint64_t {
        uint64_t incl = v;
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t o = __shfl_up(incl, d, 64);
            if (lane >= (uint32_t)d) incl += o;
        }
        __syncthreads();
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        uint64_t before = 0, tot = 0;
        for (uint32_t w = 0; w < 4; ++w) {
            before += w < wave ? wsum[w] : 0;
            tot += wsum[w];
        }
        *total = tot;
        return before + incl - v;
    };
    uint64_t total = 0;
    if (dense) {
        const uint64_t off = block_scan(sz, &total);
        if (in) dense[j] = off;
    }
    __syncthreads();  // the block's counts are out
    if (tid == 0) {
        if (dense) __hip_atomic_store(&totals[blockIdx.x], total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (bins > 1u) __threadfence();
        last = bins == 1u || atomicAdd(&P.ctl->ticket, 1u) == bins - 1u;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    if (tid < kClasses) {
        P.ctl->job[tid] = bins > 1u ? __hip_atomic_load(&P.ctl->count[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                          : lists   ? cnt[0][tid] + cnt[1][tid] + cnt[2][tid] + cnt[3][tid]
                                    : 0u;
        P.ctl->count[tid] = 0;
    }
    if (tid == 0) P.ctl->ticket = P.ctl->queue = P.ctl->small = 0;
    uint64_t carry = 0;
    for (uint32_t b = 0; dense && b < bins; b += kBinTasks) {
        const uint64_t v = b + tid < bins
                               ? __hip_atomic_load(&totals[b + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        const uint64_t o = block_scan(v, &total);
        if (b + tid < bins) base[b + tid] = carry + o;
        carry += total;
    }
}

// ------------------------------------------------------------ host launch
size_t shared_bytes(uint32_t cap16) {
    const uint32_t c = cap16 < kMinCap16 ? kMinCap16 : cap16;
    return sizeof(Shared) + list_bytes(c) + slot_bytes(c);
}

template <int NT>
static hipError_t launch_nt(const Params& P, uint32_t grid, hipStream_t s) {
    hipLaunchKernelGGL(decode_kernel<NT>, dim3(grid), dim3(NT), shared_bytes(P.cap16), s, P);
    return hipGetLastError();
}

hipError_t set_kernel_attrs() {
    const int maxb = (int)shared_bytes(kMaxCap16);
    hipError_t e;
    if ((e = hipFuncSetAttribute((const void*)decode_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, maxb)))
        return e;
    if ((e = hipFuncSetAttribute((const void*)decode_kernel<256>, hipFuncAttributeMaxDynamicSharedMemorySize, maxb)))
        return e;
    if ((e = hipFuncSetAttribute((const void*)decode_kernel<512>, hipFuncAttributeMaxDynamicSharedMemorySize, maxb)))
        return e;
    return hipFuncSetAttribute((const void*)decode_kernel<1024>, hipFuncAttributeMaxDynamicSharedMemorySize, maxb);
}

template <int NT>
static int resident_nt(uint32_t cap16) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, decode_kernel<NT>, NT, shared_bytes(cap16)) != hipSuccess)
        return 1;
    return n > 0 ? n : 1;
}

int max_resident_per_cu(int wg_size, uint32_t cap16) {
    switch (wg_size) {
    case 128: return resident_nt<128>(cap16);
    case 256: return resident_nt<256>(cap16);
    case 512: return resident_nt<512>(cap16);
    case 1024: return resident_nt<1024>(cap16);
    default: return 1;
    }
}

hipError_t launch_decode(const Params& P, int wg_size, uint32_t grid, hipStream_t s) {
    switch (wg_size) {
    case 128: return launch_nt<128>(P, grid, s);
    case 256: return launch_nt<256>(P, grid, s);
    case 512: return launch_nt<512>(P, grid, s);
    case 1024: return launch_nt<1024>(P, grid, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_prepare(Control* ctl, uint32_t* tab, const RansFreq* f, hipStream_t s) {
    hipLaunchKernelGGL(prepare_kernel, dim3(tab ? kRansM / 256 : 1), dim3(256), 0, s, ctl, tab, f ? *f : RansFreq{});
    return hipGetLastError();
}

hipError_t launch_bin(const Params& P, uint32_t* lists, uint64_t* dense, uint64_t* base, uint64_t* totals, uint32_t* tab,
                      const RansFreq* f, hipStream_t s) {
    const uint32_t bins = lists || dense ? (P.n_tasks + kBinTasks - 1) / kBinTasks : 1u;
    hipLaunchKernelGGL(bin_kernel, dim3(bins + (tab ? kRansM / kBinTasks : 0u)), dim3(kBinTasks), 0, s, P, lists, dense, base,
                       totals, bins, tab, f ? *f : RansFreq{});
    return hipGetLastError();
}

}  // namespace csgv
