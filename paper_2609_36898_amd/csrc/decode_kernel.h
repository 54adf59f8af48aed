// Launch interface between the C ABI and the decode kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "csgv_format.h"

namespace csgv {

// ---- LDS of a decode work-group: a fixed part plus `cap16` 16-bit slots for
// the explicit nodes of level 5 (the LDS split chosen per launch).  The slot
// area also holds the 16 KiB rANS decoding table while a record's symbols are
// decoded, so it is never smaller than kMinCap16 slots.
constexpr uint32_t kMaxWaves = 16;       // work-groups of up to 1024 threads
constexpr uint32_t kFullSlots = 4688;    // full grids of levels 0..4 at 0, 8, 16, 80, 592
constexpr uint32_t kEWords = 148;        // expansion bitmaps of levels 0..4: 1+1+2+16+128 words
constexpr uint32_t kUBytesMin = 2048;    // parent list / palette area of the smallest slot area
constexpr uint32_t kMinCap16 = 8192;     // 16 KiB: the rANS table
constexpr uint32_t kMaxCap16 = 32760;    // largest LDS slot share accepted
constexpr uint32_t kDefaultCap16 = 10240;
// parent list of level 5 (one 16-bit entry per 8 slots) | staged palette
__host__ __device__ constexpr uint32_t list_bytes(uint32_t cap16) { return (cap16 / 4u + 15u) & ~15u; }
// Slot area: the slots and, up to the LDS that four default work-groups leave of
// a CU's 160 KiB, room for the record's symbols behind the rANS table.
constexpr uint32_t kSlotBytesShared = 26624;
__host__ __device__ constexpr uint32_t slot_bytes(uint32_t cap16) {
    const uint32_t with = 2u * cap16 + 6144u;
    return with <= kSlotBytesShared ? with : 2u * cap16 > kSlotBytesShared ? 2u * cap16 : kSlotBytesShared;
}
static_assert(list_bytes(kMinCap16) >= kUBytesMin, "palette area");

// Room of n 4-bit symbols, in whole words.  The first symbol is looked at whatever
// n is (a damaged record may have none), so there is a word of it always.
__host__ __device__ constexpr uint32_t symbol_bytes(uint32_t n) { return 4u * (n ? (n + 7u) / 8u : 1u); }
static_assert(symbol_bytes(0) == 4u && symbol_bytes(8) == 4u && symbol_bytes(9) == 8u, "the first symbol has a place");

// cubes of side <= 8 with at most this many symbols are decoded by one wavefront
// each, up to four in a work-group
constexpr uint32_t kWaveSyms = 4096;

// ---- per work-group global scratch (byte offsets): palette indices of a level 5
// decoded in chunks (16 bits each), its and level 6's parent lists, then the
// record's 4-bit symbols, whose size depends on the largest brick side of the
// volume (as does the list's: level 6 occurs in 64^3 bricks only).
constexpr uint64_t kScrComp = 0;                                   // 32768 x u16
constexpr uint64_t kScrList = kScrComp + 2ull * 32768;             // 4096 or 32768 x u32
constexpr uint64_t scr_sym(uint32_t max_log2b) { return kScrList + 4ull * (max_log2b > 5 ? 32768 : 4096); }
constexpr uint64_t scratch_per_wg(uint32_t max_log2b) {
    const uint64_t sym = ((4 * total_nodes(max_log2b) + 255) / 256) * 256;
    return scr_sym(max_log2b) + (sym < 4ull * kWaveSyms / 2 ? 4ull * kWaveSyms / 2 : sym);
}

// ---- task lists of a queue launch, by decreasing cost: each class has room for
// every task; a claim walks the classes in order.  The classes from kWgClasses
// on are decoded by single wavefronts.
constexpr uint32_t kClasses = 6, kWgClasses = 4;
// Control words of a launch.  The binning kernel's last block leaves them ready
// for the decode that follows: the classes' sizes in job, everything else zero.
// That decode leaves queue, small and job as it used them, so every decode with
// ctl set comes behind a binning kernel; ticket and count are zero in between.
struct Control {
    uint32_t ticket;            // blocks of the binning kernel done
    uint32_t count[kClasses];   // tasks per class while they are binned
    uint32_t queue;             // claims of the work-groups beyond their first task
    uint32_t small;             // claims of the single wavefronts beyond their first
    uint32_t job[kClasses];     // tasks per class
};
constexpr uint32_t kBinTasks = 256;  // tasks per block of the binning kernel

struct RansFreq {
    uint32_t w[8];  // 16 x u16 frequencies, two per word
};

struct Params {
    const uint8_t* vol;  // container in device memory
    uint64_t vol_bytes;
    uint64_t off_pos;
    uint32_t n_bricks;
    uint32_t label_bytes;
    uint32_t freq_ok;          // the volume's frequency table sums to 4096
    uint32_t max_log2b;        // records with a larger brick side are rejected (scratch bound)
    const uint32_t* rans_tab;  // decoding table built by prepare_kernel (4096 entries)
    const uint32_t* ids;
    const uint8_t* lods;
    const uint64_t* out_offs;    // caller's element offsets, or null
    const uint64_t* dense_offs;  // offsets computed on the device when out_offs is null: within the
    const uint64_t* dense_base;  // task's block of kBinTasks, and the block's own
    uint32_t n_tasks;
    uint8_t* out;
    uint64_t out_cap;   // elements
    uint32_t* status;   // may be null
    Control* ctl;           // queue launch: claims and class counts (null: work-group b takes tasks b, b + grid, ...)
    const uint32_t* lists;  // queue launch: tasks of class c at c * list_cap
    uint32_t list_cap;
    uint8_t* scratch;
    uint64_t scratch_stride;
    uint64_t scratch_sym;   // scr_sym of the volume
    uint32_t cap16;     // LDS slots for the explicit nodes of level 5 (>= kMinCap16)
    uint32_t pal_bits;  // 0: labels; I > 0: packed I-bit palette indices, floor(32/I) per word
};

// output units of an S^3 cube: labels, or 32-bit words of packed palette indices
__host__ __device__ inline uint64_t out_units(uint64_t voxels, uint32_t pal_bits) {
    if (!pal_bits) return voxels;
    const uint64_t e = 32u / pal_bits;
    return (voxels + e - 1) / e;
}

size_t shared_bytes(uint32_t cap16);
int max_resident_per_cu(int wg_size, uint32_t cap16);  // occupancy of the decode kernel
hipError_t set_kernel_attrs();
hipError_t launch_decode(const Params& P, int wg_size, uint32_t grid, hipStream_t s);
hipError_t launch_prepare(Control* ctl, uint32_t* tab, const RansFreq* f, hipStream_t s);
hipError_t launch_bin(const Params& P, uint32_t* lists, uint64_t* dense, uint64_t* base, uint64_t* totals, uint32_t* tab,
                      const RansFreq* f, hipStream_t s);

}  // namespace csgv
