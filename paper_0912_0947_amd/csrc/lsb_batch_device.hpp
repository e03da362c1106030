// lsb_batch_device.hpp -- device side of the batched embed/extract: the job
// table and the batched kernel, shared by the translation unit of
// header-only plans and the one of plans with raw-slice jobs.
#pragma once

#include <stddef.h>

#include <utility>

#include "lsb_host.hpp"

namespace lsb {

struct DevJob {
    uint64_t cover_off, stego_off, msg_off, n;
    uint64_t cap_bits;  // header extract: msg_cap; raw: end bit (embed: stream_bits, extract: e)
    uint64_t t0;        // raw: logical field index of buffer byte 0; header jobs: 0
    uint64_t vectors;   // vectors that a run may have to visit (host: tile counts)
    uint32_t len;
    uint8_t k, op;
    int8_t status;  // host-validated status; header extract: decoded on device
    uint8_t raw;    // 1: raw slice, no header
};
static_assert(sizeof(DevJob) == 64, "DevJob is one 64-byte record");
static_assert(sizeof(lsb_job) == 64 && offsetof(lsb_job, len) == 56, "lsb_job layout of the C ABI");

// The job table: the records, every job's first tile id (then kFirstPad
// entries of ~0), and a map from tile ids to jobs: entry i names the job that
// holds tile i << map_shift, with the smallest shift whose map fits 4 entries
// per job plus 4096.  A map of shift 0 names a tile's job outright; a larger
// one (big covers) leaves the jobs that begin inside the entry's tiles.
constexpr int kMaxJobs = 1 << 24;
constexpr int kFirstPad = 8;

struct TableLayout {
    uint64_t first_off, map_off;  // byte offsets behind the records
    uint64_t map_max;             // entries
    uint64_t bytes;               // with a full map
};

__host__ __device__ constexpr TableLayout table_layout(uint64_t n_jobs) {
    TableLayout t{};
    t.first_off = sizeof(DevJob) * n_jobs;
    t.map_off = t.first_off + 8 * (n_jobs + kFirstPad);
    t.map_max = 4 * n_jobs + 4096;
    t.bytes = t.map_off + 4 * t.map_max;
    return t;
}

// Everything a run needs, by value.
struct BatchArgs {
    const DevJob *jobs;
    const uint64_t *first;
    const uint32_t *map;
    uint64_t n_jobs, total_tiles;
    uint64_t embed_vectors, extract_vectors;  // per tile of either kind
    const uint8_t *cover_arena;
    uint8_t *stego_arena, *msg_arena;
    uint32_t *len_dev;
    int32_t *status_dev;
    int32_t map_shift;
    int32_t empty_jobs;  // some job has no tile
};

// One tile of a job: ranges with k known at compile time, then the walk
// over the tile's vectors.
template <int K, int UNR, bool NT>
__device__ __forceinline__ void embed_tile(const Span &s, uint64_t v_begin, uint64_t tile_vectors, uint32_t wave,
                                           uint32_t n_waves, uint32_t lane) {
    const Ranges r = embed_ranges<K>(s);
    uint64_t v_end = v_begin + tile_vectors;
    if (v_end > r.count) v_end = r.count;
    if (v_begin < v_end) embed_walk<K, UNR, NT>(s, r, v_begin, v_end, wave, n_waves, lane);
}

template <int K, int UNR, bool NT>
__device__ __forceinline__ void extract_tile(const Span &s, uint64_t v_begin, uint64_t tile_vectors, uint32_t wave,
                                             uint32_t n_waves, uint32_t lane) {
    const Ranges r = extract_ranges<K>(s);
    uint64_t v_end = v_begin + tile_vectors;
    if (v_end > r.count) v_end = r.count;
    if (v_begin < v_end) extract_walk<K, UNR, NT>(s, r, v_begin, v_end, wave, n_waves, lane);
}

// Job classes of a plan.  CLS = 1 + 8*op + (k - 1): every job has that
// (op, k), and only its walker is compiled in.  CLS = 17 / 18: every job is
// an extract / an embed, k dispatched by a switch over the eight walkers of
// that kind.  CLS = 0: (op, k) read from each job, a switch over all sixteen.
// Header and raw-slice jobs share the walkers: only the span's stream fields
// differ.  RAW = false compiles the raw-slice case out (the plan has none):
// the header span's constant t0 and header length then fold into the walk.
constexpr int kClsExtractAnyK = 17, kClsEmbedAnyK = 18, kClasses = 19;

template <int UNR, bool NT, int CLS, bool RAW>
__device__ __forceinline__ void run_tile(const DevJob &J, uint64_t v_begin, uint64_t tile_vectors,
                                         const uint8_t *cover_arena, uint8_t *stego_arena, uint8_t *msg_arena,
                                         uint32_t len, uint32_t wave, uint32_t n_waves, uint32_t lane) {
    constexpr bool EMB = CLS == 0 || CLS == kClsEmbedAnyK || (CLS >= 1 && CLS <= 8);
    constexpr bool EXT = CLS == 0 || CLS == kClsExtractAnyK || (CLS >= 9 && CLS <= 16);
    constexpr int KC = CLS >= 1 && CLS <= 16 ? (CLS - 1) % 8 + 1 : 0;  // fixed k, 0: any
    Span s{};
    s.n = J.n;
    s.t0 = 0;
    s.k = J.k;
    s.hdr_len = 4;
    const bool raw = RAW && J.raw;
    if (raw) {
        s.t0 = J.t0;
        s.hdr_len = 0;
    }
    if constexpr (EMB) {
        if (!EXT || J.op == LSB_OP_EMBED) {
            s.src = cover_arena + J.cover_off;
            s.dst = stego_arena + J.stego_off;
            s.body = msg_arena + J.msg_off;
            s.bits = raw ? J.cap_bits : 8 * (4 + (uint64_t)J.len);
            s.hdr = J.len;
            if constexpr (KC > 0) {
                embed_tile<KC, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane);
            } else {
                switch (J.k) {
                    case 1: embed_tile<1, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                    case 2: embed_tile<2, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                    case 3: embed_tile<3, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                    case 4: embed_tile<4, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                    case 5: embed_tile<5, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                    case 6: embed_tile<6, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                    case 7: embed_tile<7, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                    default: embed_tile<8, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                }
            }
            return;
        }
    }
    if constexpr (EXT) {
        s.src = stego_arena + J.stego_off;
        s.out = msg_arena + J.msg_off;
        s.bits = raw ? J.cap_bits : 8 * (4 + (uint64_t)len);
        if constexpr (KC > 0) {
            extract_tile<KC, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane);
        } else {
            switch (J.k) {
                case 1: extract_tile<1, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                case 2: extract_tile<2, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                case 3: extract_tile<3, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                case 4: extract_tile<4, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                case 5: extract_tile<5, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                case 6: extract_tile<6, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                case 7: extract_tile<7, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
                default: extract_tile<8, UNR, NT>(s, v_begin, tile_vectors, wave, n_waves, lane); break;
            }
        }
    }
}

// Waves per SIMD the launch bound asks for: as many as each kernel's walkers
// fit without spilling (the sixteen-way switch holds every walker at once).
template <int UNR, int CLS, bool RAW>
constexpr int batch_min_waves() {
    if constexpr (UNR == 1) return 8;
    else if constexpr (UNR == 2) return CLS == kClsExtractAnyK && !RAW ? 8 : (RAW && CLS <= 1 ? 5 : 6);
    else return 4;
}

__device__ __forceinline__ uint32_t uniform32(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    return ((uint64_t)uniform32((uint32_t)(v >> 32)) << 32) | uniform32((uint32_t)v);
}

// What a job reports in len_dev / status_dev.  The host-validated status
// and length, except for a header extract job that the host let through:
// its length is the stego's 32-bit header (Section VII, the stream's first
// 32 bits), which must fit the cover's room and the job's output buffer.
// J is wave-uniform: the decode spreads the header's bits over the lanes.
struct JobReport {
    uint32_t len;
    int32_t status;
};

__device__ __forceinline__ JobReport job_report(const DevJob &J, const uint8_t *stego_arena, uint32_t lane) {
    JobReport r{J.len, J.status};
    if (J.op == LSB_OP_EXTRACT && !J.raw && J.status == LSB_OK) {
        r.len = 0;
        r.status = LSB_E_HEADER;
        if ((uint64_t)J.k * J.n >= 32) {
            r.len = decode_header(stego_arena + J.stego_off, J.k, lane);
            if (4 + (uint64_t)r.len > room_bytes(J.n, J.k)) r.status = LSB_E_HEADER;
            else if ((uint64_t)r.len > J.cap_bits) r.status = LSB_E_BUFFER;
            else r.status = LSB_OK;
        }
    }
    return r;
}

// Reports of the jobs without tiles (refused on the host, empty slices, and
// header extract jobs whose cover holds fewer than 32 bits), one thread per
// job over the grid.  No tile is ever handed out for these jobs, so nothing
// else writes their entries.  A header extract job the host let through has
// a tile whenever k n >= 32, so one without tiles is refused here.
__device__ __forceinline__ void report_empty_jobs(const BatchArgs &a) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < a.n_jobs; j += stride) {
        const uint64_t end = j + 1 < a.n_jobs ? a.first[j + 1] : a.total_tiles;
        if (a.first[j] != end) continue;  // the block of its first tile reports it
        const DevJob &J = a.jobs[j];
        uint32_t len = J.len;
        int32_t status = J.status;
        if (J.op == LSB_OP_EXTRACT && !J.raw && status == LSB_OK) {
            len = 0;
            status = LSB_E_HEADER;
        }
        if (a.len_dev) a.len_dev[j] = len;
        a.status_dev[j] = status;
    }
}

// Read-only table entries at wave-uniform places, through the scalar cache:
// the table does not change while a kernel runs, and scalar loads have a
// counter of their own, so a lookup never waits for the wave's stores.
template <typename T>
using Uniform = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ Uniform<T> uniform_ptr(const T *p) {
    return (Uniform<T>)(uintptr_t)p;
}

// The job of tile t, and its first tile id: the largest j with first[j] <= t.
// One map entry, then the first tile ids from there on: usually the entry's
// own job or one of the next few; where a group of tiles holds many small
// jobs, 64 per step and ballot.
__device__ __forceinline__ uint64_t find_job(const BatchArgs &a, uint64_t t, uint32_t lane, uint64_t *first_tile) {
    uint64_t j = uniform_ptr(a.map)[t >> a.map_shift];
    const Uniform<uint64_t> f = uniform_ptr(a.first) + j;
    uint64_t ft = f[0];
    uint32_t step = 0;
#pragma unroll
    for (int i = 1; i < kFirstPad; ++i) {
        const uint64_t x = f[i];
        if (x <= t) {
            step = i;
            ft = x;
        }
    }
    j += step;
    if (step == kFirstPad - 1) {
        for (;;) {
            const uint64_t idx = j + 1 + lane;
            const uint64_t tb = idx < a.n_jobs ? a.first[idx] : ~0ull;
            const uint32_t cnt = (uint32_t)__popcll(__ballot(tb <= t));
            j += cnt;
            if (cnt < 64) break;
        }
        j = uniform64(j);
        ft = uniform64(a.first[j]);
    }
    *first_tile = ft;
    return j;
}

// Consecutive tiles that one XCD takes (see the kernel).
constexpr uint32_t kTileRun = 32;

// One block per tile: each wave finds the tile's job through the map and
// streams its share of the tile.  HBM bounds it, as the plain kernels: blocks
// of other tiles stream while one looks its job up, and a wave ends after its
// last store without waiting for it.  Tiles go to the XCDs in runs of kTileRun
// (xcd_run_block): neighbours share lines at their ends, the table entries and an
// L2, and an XCD touches fewer memory pages at a time.  35.7 GB in 4096 covers,
// us: runs of 16, 32, 64, 128 extract 4049, 3899, 3906, 4001, embed 11,690,
// 11,530, 11,650, 11,520; launch order extracts a sixth slower than runs of 16.
// A grid capped below the tile count walks the tiles with a stride.  Embed +
// extract passes, against persistent blocks whose producer wave took tiles from
// one counter and handed them to 15 workers: 4096 covers of 64..256 px 225 -> 123
// us, 256 covers of 64..4096 px 947 -> 890 us (6.2 TB/s), 120 frames of 1080p 345
// -> 320 us.  An embed tile is one step of the block: with two steps the second
// waits for the first one's stores (256 covers' embed 646 us at 512 vectors a tile,
// 678 us at 1024); extracts store little, so theirs may take two (lsb_batch.hip).
template <int UNR, bool NT, int CLS, bool RAW>
__global__ void __launch_bounds__(1024, (batch_min_waves<UNR, CLS, RAW>())) lsb_batch_kernel(BatchArgs a) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = uniform32(threadIdx.x >> 6);
    const uint32_t waves = blockDim.x >> 6;
    if (a.empty_jobs) report_empty_jobs(a);
    for (uint64_t t = xcd_run_block<kTileRun>(blockIdx.x, gridDim.x); t < a.total_tiles; t += gridDim.x) {
        uint64_t first_tile;
        const uint64_t j = find_job(a, t, lane, &first_tile);
        DevJob J;
        {
            const Uniform<uint32_t> src = uniform_ptr(reinterpret_cast<const uint32_t *>(a.jobs + j));
            uint32_t *dst = reinterpret_cast<uint32_t *>(&J);
#pragma unroll
            for (int i = 0; i < (int)(sizeof(DevJob) / 4); ++i) dst[i] = src[i];
        }
        const JobReport r = job_report(J, a.stego_arena, lane);
        if (t == first_tile && threadIdx.x == 0) {  // the job's first tile: report the job
            if (a.len_dev) a.len_dev[j] = r.len;
            a.status_dev[j] = r.status;
        }
        if (r.status != LSB_OK) continue;
        const uint64_t tv = J.op == LSB_OP_EXTRACT ? a.extract_vectors : a.embed_vectors;
        run_tile<UNR, NT, CLS, RAW>(J, (t - first_tile) * tv, tv, a.cover_arena, a.stego_arena, a.msg_arena, r.len,
                                    wave, waves, lane);
    }
}

typedef void (*BatchFn)(BatchArgs);

// Kernel table of one launch shape: entry CLS of the class sequence.
template <int UNR, bool NT, bool RAW, int... C>
BatchFn batch_fn_of(int cls, std::integer_sequence<int, C...>) {
    static const BatchFn table[] = {lsb_batch_kernel<UNR, NT, C, RAW>...};
    return table[cls];
}

// Kernel for a launch shape and plan class (0 = mixed jobs).
template <bool RAW>
BatchFn batch_fn_for(int unroll, int nt, int cls) {
    using Classes = std::make_integer_sequence<int, kClasses>;
    if (unroll == 1)
        return nt ? batch_fn_of<1, true, RAW>(cls, Classes{}) : batch_fn_of<1, false, RAW>(cls, Classes{});
    if (unroll == 2)
        return nt ? batch_fn_of<2, true, RAW>(cls, Classes{}) : batch_fn_of<2, false, RAW>(cls, Classes{});
    return nt ? batch_fn_of<4, true, RAW>(cls, Classes{}) : batch_fn_of<4, false, RAW>(cls, Classes{});
}

// Kernels of plans holding raw-slice jobs (instantiated in their own
// translation unit, which builds in parallel with the header-only one).
BatchFn batch_fn_raw(int unroll, int nt, int cls);

}  // namespace lsb
