// lsb_host.hpp -- host-side helpers shared by the translation units of
// liblsb.so: error reporting, device properties, launch-configuration table.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "../../include/lsb.h"
#include "lsb_device.hpp"

namespace lsb {

// Thread-local message for lsb_last_error().
int fail(int code, const char *fmt, ...);
void clear_error();

// Map a HIP error to LSB_E_HIP with a message naming the call.
int hip_fail(hipError_t e, const char *what);

// Events set by lsb_time_next_launch for the calling thread; returns them
// and clears the request (both null when none is pending).
void take_launch_events(hipEvent_t *start, hipEvent_t *stop);
int set_launch_events(void *start, void *stop);

// Scope of an entry point that honours lsb_time_next_launch: clears the
// error message on entry and, on return, a timing request that no launch
// took (the call failed or had nothing to launch), so that the events never
// reach a later call.
struct TimedCall {
    TimedCall() { clear_error(); }
    ~TimedCall() { set_launch_events(nullptr, nullptr); }
    TimedCall(const TimedCall &) = delete;
    TimedCall &operator=(const TimedCall &) = delete;
};

// Compute units of the current device (cached per device).
int device_cus();

// true if [a, a+na) and [b, b+nb) share a byte.
inline bool overlaps(const void *a, uint64_t na, const void *b, uint64_t nb) {
    if (!na || !nb) return false;
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + nb && y < x + na;
}

// Launch configuration table, indexed by op (0 embed, 1 extract), k and
// size bucket floor(log2(n)).
constexpr int kBuckets = 64;
lsb_launch_cfg tune_lookup(int op, int k, uint64_t n);
bool cfg_valid(const lsb_launch_cfg &c);

// Grid size for `vectors` 16-byte vectors under configuration c.
inline unsigned grid_for(const lsb_launch_cfg &c, uint64_t vectors) {
    const uint64_t per_block = (uint64_t)c.block * (uint64_t)c.unroll;  // vectors per block step
    uint64_t blocks = ceil_div(vectors, per_block);
    if (blocks == 0) blocks = 1;
    if (c.blocks_per_cu > 0) {
        const uint64_t cap = (uint64_t)c.blocks_per_cu * (uint64_t)device_cus();
        if (blocks > cap) blocks = cap;
    }
    if (blocks > 0x7FFFFFFFull) blocks = 0x7FFFFFFFull;
    return (unsigned)blocks;
}

// Cached or streaming (non-temporal) accesses of the layout kernels, by image
// bytes n.  Cached while three images and their stegos come and go through the
// caches of a program that embeds and then reads the stego: up to 40 MB an embed +
// extract pass takes 10-15 % less (36 MB plane: 19.1 against 22.0 us).  Above,
// loads stream and stores stay cached (100 MB plane: 48.0 us; all cached 52.6, all
// streaming 50.8).  Cached loads still gain there where one image is embedded into
// again and again, and lose where images are new, which decides; us a pass, cached
// / loads streaming, planes of 3 channels, the same image, 3 and 40 images in turn:
// 48 MB 25.5 / 29.0, 27.7 / 27.0, 29.2 / 28.1; 66 MB at k=6 36.2 / 39.4, 41.9 /
// 38.0, 42.6 / 39.4; 88 MB 42.7 / 44.9, 48.5 / 44.7, 49.8 / 45.4; the paper's
// layout 60 MB of 1 channel 33.3 / 34.7, 37.2 / 35.1, 37.9 / 37.8.  From 128 MB
// on stores stream too: one stego no longer fits beside its cover in the 256 MB
// last-level cache, and its dirty lines would slow whatever runs next.
inline Access access_kind(uint64_t n) {
    if (n <= 40ull * 1000 * 1000) return CACHED;
    return n < (1ull << 27) ? STREAM_LOADS : STREAM;
}

// Plain-kernel launchers (lsb_plain.hip); they validate nothing.
int launch_embed(const Span &s, const lsb_launch_cfg &c, hipStream_t stream);
int launch_extract(const Span &s, int header, uint64_t out_cap, uint32_t *len_out,
                   int32_t *status_out, uint64_t max_vectors, const lsb_launch_cfg &c,
                   hipStream_t stream);

}  // namespace lsb
