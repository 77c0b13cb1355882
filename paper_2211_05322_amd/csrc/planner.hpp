// planner.hpp -- host-side planning of one cross-mesh resharding task.
//
// Steps (all host, no HIP):
//   parse      spec strings -> mesh axes per tensor dimension (Section 2.2)
//   layout     device -> shard index per dimension, shard bounds per dimension
//   tasks      unit tasks = non-empty intersections of a source shard and a
//              destination shard, with all owners and all receivers
//              (Section 2.2; the same slices as the appendix cut-point
//              decomposition, computed here dimension by dimension as
//              intersections of shard intervals)
//   senders    one owner per task: naive (lowest index) or longest-first
//              greedy balancing of sent bytes (Section 3.2, Eq. 4)
//   lowering   each task -> pieces (collapsed strided boxes) -> chunks
//              (descriptors, one per workgroup)
#pragma once

#include <atomic>
#include <cstdint>
#include <mutex>
#include <string>
#include <vector>

#include "desc.h"

namespace rs {

struct Layout {
    std::vector<int64_t> mesh;               // mesh shape
    std::vector<std::vector<int>> axes;      // per tensor dim: mesh axes, major to minor
    std::vector<int64_t> nshards;            // per tensor dim
    std::vector<std::vector<int64_t>> bounds;  // per dim: nshards+1 cut positions
    int64_t ndev = 0;
    std::vector<int64_t> dev_shard;          // [dev * ndim + dim] -> shard index
    std::vector<int64_t> shard_devs_off;     // CSR over linearised shard tuples
    std::vector<int32_t> shard_devs;         //   -> devices holding that shard (ascending)
};

struct UnitTask {
    std::vector<int64_t> lo, hi;   // slice of D
    int64_t src_shard = 0;         // linearised source shard tuple
    int64_t dst_shard = 0;         // linearised destination shard tuple
    int64_t bytes = 0;
    int32_t sender = -1;           // chosen owner
};

struct Tuning {
    int64_t chunk_bytes = 0;   // 0: automatic
    int32_t block_threads = 256;
    bool block_is_default = true;  // the caller left the block size to the library
    int32_t max_wgs_per_cu = 0;  // the caller's cap (0: none)
    bool cap_is_default = true;  // the caller left the cap to the library (chosen at launch)
    int32_t gather_band = 0;     // row gather: segments per column band (0: whole rows)
};

// A number no other plan of this process has (plans are told apart by it,
// not by address, which a later plan may reuse).
inline uint64_t next_plan_serial() {
    static std::atomic<uint64_t> n{0};
    return ++n;
}

struct Plan {
    const uint64_t serial = next_plan_serial();
    int ndim = 0;
    std::vector<int64_t> shape;
    int64_t es = 0;            // element size in bytes
    unsigned flags = 0;
    Tuning tuning;
    Layout src, dst;
    // Local layouts: dimension k of a device's buffer is tensor dimension
    // perm[k] (identity unless the caller permuted a side).
    std::vector<int> sperm, dperm;
    std::vector<UnitTask> tasks;
    std::vector<Desc> descs;
    std::vector<int32_t> fan;  // receiver lists, referenced by Desc::fan_off/nfan
    int64_t bytes_read = 0, bytes_written = 0, max_fanout = 0;
    int64_t align = 1;         // required buffer alignment in bytes
    bool too_many = false;     // lowering stopped: descriptor table over its cap
    bool tile_span_too_long = false;  // lowering stopped: one transpose tile spans 2^32 bytes or more
    uint32_t lds_bytes = 0;    // LDS the realignment chunks need per workgroup
    size_t n_direct = 0;       // descs[0, n_direct): direct chunks
    size_t n_gather = 0;       // descs[n_direct, n_direct + n_gather): row-gather chunks;
    size_t n_gather_u = 0;     // then n_gather_u unaligned row-gather chunks (the last n_unit
    size_t n_unit = 0;         // of them unit-gather chunks, their own kernel);
    size_t n_transpose = 0;    // then n_transpose tile-transpose chunks;
                               // the rest: realignment chunks
    bool shortest_table = false;  // lowered without the forms that take more chunks
    bool longer_forms = false;    // some group or piece has such a form,
    int64_t extra_chunks = 0;     //     and the chunks that these add
    size_t n_blocked = 0;      // direct chunks in blocks of two dimensions
    size_t n_spread = 0;       // direct chunks whose receiver sets share sender rows (chunk order)
    bool sets_in_turn = false; // ... and these take turns
    uint64_t n_tiles = 0, n_part_tiles = 0;  // transpose tiles; those that write parts of 64-byte groups
    bool transpose_plain = false;  // stored through L2 (enough of these)
    uint32_t transpose_lds = 0;  // LDS bytes of the largest set of tiles moved at once
    std::vector<Seg> segs;     // row-gather segment entries
    int64_t gather_fanout = 0; // largest receiver count among row-gather chunks
    int64_t gather_u_fanout = 0; // ... among unaligned row-gather chunks
    int64_t gather_u_segs = 0;   // most segments per row among unaligned row-gather groups
    bool gather_u_parts = false; // some one-sender slot group reads parts, 1 KiB and more, of its sender's rows
    uint64_t gather_u_bytes = 0; // destination bytes of the slot chunks, and their nominal
    uint64_t gather_u_room = 0;  //     capacity (chunks x chunk size): how full they are
    bool gather_u_short = false; // some slot group has segments under 16 bytes
    int64_t unit_fanout = 0;     // ... and among the unit-gather groups:
    int64_t unit_segs = 0;       //     receivers, segments per row
    int64_t direct_fanout = 0; // largest receiver count among direct chunks
    size_t n_phase1 = 0;       // descs[0, n_phase1) run before descs[n_phase1, n_direct)
                               // (two launches; only the all-gather strategy has a second phase)
    std::vector<int64_t> src_local_numel, dst_local_numel;  // per device

    // Device copy of [descs | fan], uploaded on the first execute on each HIP
    // device (index = device ordinal).
    static constexpr int kMaxHipDevices = 64;
    mutable std::mutex mu;
    mutable void *d_table[kMaxHipDevices] = {};
};

// Bytes of the plan's device tables: descriptors, receiver lists, segment
// entries (from a 16-byte boundary).
inline size_t table_bytes(const Plan &p) {
    const size_t head = p.descs.size() * sizeof(Desc) + p.fan.size() * sizeof(int32_t);
    return ((head + 15) & ~size_t(15)) + p.segs.size() * sizeof(Seg);
}

// Bytes read and written up to which a reshard runs with 32 waves per CU
// instead of its kernel's cap (why: launch).  Direct chunks, by receivers:
// to 16 cold buffers 50 MB 1.04 times as fast, 90 MB 0.97, 130 MB 0.95, to 32
// 82 MB 1.09.
inline int64_t cached_direct_limit(int64_t fanout) {
    return int64_t(fanout == 1 ? 120 : fanout > 8 ? 96 : 144) << 20;
}
// Slots, by receivers, senders per row, and whether rows are parts, 1 KiB and
// more wide, of a sender's (shorter ones gain longer: bf16 [48,501,886] to 4,
// 213 MB, 1.18).  Rows from one sender fill the cap's fewer waves well, and the more
// receivers, the sooner they lose with 32 waves, parts of wider rows first
// (times as fast, buffers cold / warm): to 2, parts 200 MB 1.02 / 0.98, 230 MB
// 0.97 / 0.95, whole rows 1.0; to 3, 262 MB 1.2 to 1.4 / 1.05 to 1.2; to 4,
// parts 165 MB 1.5 / 1.25, 171 MB 1.05 / 0.88, whole rows 262 MB 0.95 to
// 1.14 / 0.92 to 1.12; to 5, whole rows 200 MB 1.11 / 1.06, 230 MB 0.93 / 0.92;
// to 6, whole rows 180 MB 0.94 and 1.19 / 0.93 and 1.17, 262 MB 0.92, parts
// 25 MB 1.06, 90 MB 1.05 / 0.88; to 7, 90 MB 0.93; to 8, 40 MB 1.05, 70 MB 0.92
// to 0.95, 262 MB 0.83 to 0.89; to 16, 110 MB 1.01, 130 MB 0.95, to 32, 82 MB
// 1.09.  From several senders: to 4 and 8, 1.02 to
// 1.1 up to 262 MB (bf16 [10,2157,626] to 4, 135 MB, 42.9 -> 27.0 us; 215 ->
// 247 at 1.1 GB); to 16, 90 MB 1.02 / 0.99, 130 MB 0.96.
inline int64_t cached_slots_limit(int64_t fanout, int64_t senders, bool parts) {
    int64_t mib = 256;
    if (senders > 1 || (fanout > 8 && !parts)) mib = fanout > 8 ? 96 : 256;
    else if (parts) mib = fanout <= 2 ? 200 : fanout == 3 ? 256 : fanout <= 5 ? 160 : 40;
    else if (fanout > 4) mib = fanout <= 6 ? 192 : 40;
    return mib << 20;
}

// LDS per workgroup of the tile transpose's launch: its largest set of tiles,
// and at least what the cap on resident workgroups reserves (user_lds: the
// caller's; by default 6 per CU for 4096 chunks and more).  Measured against
// no cap: bf16 [8,2047,4098] to [batch, hidden, seq] 59.7 -> 57.0 us (4 per CU
// 56.9, 2 72.0), fp16 [5,176,48,5376] at fan-out 2 263 -> 260 (281, 396),
// uint8 [16,17408,344] to 4 receivers 103.4 -> 94.9.  4- and 8-byte elements
// to one or two receivers lose and have none (fp32 [16,4400,864] 117.3 against
// 122.6, int64 [2,8192,1824] 84.9 against 92.8, fp32 [16,4352,576] to two
// 103.3 against 107.1); at more the two are level or the cap is ahead (int64
// [16,2200,192] to 8 143.3 -> 133.8).
constexpr uint32_t kTLeastLds = 27000;
inline uint32_t transpose_launch_lds(const Plan &p, uint32_t user_lds) {
    uint32_t least = user_lds;
    if (p.tuning.cap_is_default) least = p.n_transpose >= 4096 && (p.es <= 2 || p.max_fanout > 2) ? kTLeastLds : 0u;
    return p.transpose_lds > least ? p.transpose_lds : least;
}

// Returns "" on success, else an error message; `code` receives the status.
std::string parse_spec(const char *spec, int ndim, int mesh_ndim, std::vector<std::vector<int>> &axes);
std::string build_layout(const std::vector<int64_t> &shape, const std::vector<int64_t> &mesh,
                         const std::vector<std::vector<int>> &axes, Layout &out);
void build_tasks(Plan &p);
void choose_senders(Plan &p);
void lower(Plan &p);

// Local (per-device) shape on one side.
void local_shape(const Plan &p, int side, int64_t dev, int64_t *out);

}  // namespace rs
