// lsb_paper.hip -- the paper's own layout on gfx950 (arXiv:0912.0947,
// Section VI steps 2-7 and Section VII steps 2-6): 2 bits per byte in one
// colour plane of an h x w x c image, the data split greedily over the rows
// (each row takes L = min(remaining, w/4) bytes, Section VI step 5), and bit
// pair i of data byte j in plane pixel L*i + j of its row.
//
// The paper runs this as 4 blocks of at most 32 threads per row, one MEX call
// per row.  Here one launch covers the whole image: the embed kernels stream
// every cover byte once (16 bytes per lane, copy plus in-plane update) and
// the extract kernels give each run of data bytes one lane that reads its
// four runs of pixels, so each output byte has a single writer (the paper's
// four blocks OR into the same byte).
#include <hip/hip_ext.h>

#include "lsb_host.hpp"
#include "lsb_paper_device.hpp"

using namespace lsb;

static int paper_check(uint32_t h, uint32_t w, uint32_t c, uint32_t plane, uint64_t len, const char *who) {
    if (c == 0 || plane >= c) return fail(LSB_E_ARG, "%s: plane %u outside 0..%u", who, plane, c ? c - 1 : 0);
    if ((uint64_t)h * w > (1ull << 48) / c) return fail(LSB_E_ARG, "%s: h*w*c above 2^48 bytes", who);
    const uint64_t cap = (uint64_t)h * (w / 4);
    if (len > cap)
        return fail(LSB_E_CAPACITY, "%s: %llu data bytes exceed the capacity h*floor(w/4) = %llu", who,
                    (unsigned long long)len, (unsigned long long)cap);
    return LSB_OK;
}

typedef void (*RowFn)(PaperSpan, RowMap, uint64_t);

// Run a unit kernel over n_rows rows of `units` units, `unr` units per
// thread: short rows share blocks of 256 threads, long ones are cut into equal
// shares of at most 512 units (1024 for rows that one block takes whole).
// False, nothing launched, if the grid would pass the limits of a launch
// (images of tens of gigabytes: the grid-stride kernels take them).
static bool launch_rows(const RowFn fn[2], const PaperSpan &p, uint64_t units, uint64_t n_rows, uint32_t unr,
                        hipStream_t stream) {
    if (units > (1u << 28)) return false;
    RowMap m{(uint32_t)units, 1, 1, (uint32_t)units, 0};
    uint64_t per_block = units;
    if (2 * units <= 256 * unr) {
        m.rows = 256 * unr / (uint32_t)units;
        m.magic = (uint32_t)(((1u << 20) + units - 1) / units);
        per_block = m.rows * units;
    } else if (units > 1024) {
        m.blocks = (uint32_t)ceil_div(units, 512);
        m.share = (uint32_t)ceil_div(units, m.blocks);
        per_block = m.share;
    }
    const uint64_t block = ceil_div(ceil_div(per_block, unr), 64) * 64;
    const uint64_t blocks = ceil_div(n_rows, m.rows) * m.blocks;
    if (blocks * block > 0xFFFFFFFFull || blocks > 0x7FFFFFFFull) return false;
    hipEvent_t e0, e1;
    take_launch_events(&e0, &e1);
    hipExtLaunchKernelGGL(fn[m.rows > 1], dim3((unsigned)blocks), dim3((unsigned)block), 0, stream, e0, e1, 0, p, m,
                          n_rows);
    return true;
}

// [access kind][short rows]
template <int C>
struct PaperEmbed {
    static constexpr RowFn fn[3][2] = {
        {lsb_paper_embed_units_kernel<C, false, CACHED>, lsb_paper_embed_units_kernel<C, true, CACHED>},
        {lsb_paper_embed_units_kernel<C, false, STREAM_LOADS>, lsb_paper_embed_units_kernel<C, true, STREAM_LOADS>},
        {lsb_paper_embed_units_kernel<C, false, STREAM>, lsb_paper_embed_units_kernel<C, true, STREAM>}};
};
template <int C>
struct PaperExtract {
    static constexpr RowFn fn[2] = {lsb_paper_extract_units_kernel<C, false>, lsb_paper_extract_units_kernel<C, true>};
};

// Largest data chunk per row staged in LDS by the row kernel.
static constexpr uint64_t kPaperRowChunkMax = 60 * 1024;
static_assert(paper_row_lds_bytes(kPaperRowChunkMax) <= 64 * 1024, "row kernel LDS within 64 KiB");

// Whether the row kernel takes an embed of `rows` rows of another channel count
// than 1, 3, 4: aligned rows whose chunk fits the LDS, of at least 64 vectors (a
// quarter of a block's threads; 1000 rows of 512 x 2 bytes 5.1 us against 5.9 by
// the grid-stride kernel, 10,000 of them 12.1 against 11.6, 10,000 rows of 256 x 2
// bytes 11.9 against 7.8), and at least one data-carrying row per CU (512 x 512 x
// 64 in place: 154 such rows 10.2 against 7.4 us, 512 rows 14.9 against 15.8).
static bool paper_row_kernel(const PaperSpan &p, uint64_t rows) {
    return (((uintptr_t)p.src | (uintptr_t)p.dst | p.rowbytes) & 15u) == 0 && p.q + 4 <= kPaperRowChunkMax &&
           p.rowbytes >= 1024 && p.len >= (uint64_t)device_cus() * p.q && rows <= 0xFFFFFFFFull / 256;
}

static int launched(const char *what) {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? LSB_OK : hip_fail(e, what);
}

extern "C" {

int64_t lsb_paper_capacity(uint32_t h, uint32_t w) { return (int64_t)h * (w / 4); }

int lsb_paper_embed(const uint8_t *cover, uint8_t *stego, uint32_t h, uint32_t w, uint32_t c, uint32_t plane,
                    const uint8_t *data, uint64_t len, void *stream) {
    const TimedCall timed_call;
    int rc = paper_check(h, w, c, plane, len, "lsb_paper_embed");
    if (rc) return rc;
    const uint64_t n = (uint64_t)h * w * c;
    if (n == 0) return LSB_OK;
    if (!cover || !stego) return fail(LSB_E_ARG, "lsb_paper_embed: null cover/stego");
    if (len && !data) return fail(LSB_E_ARG, "lsb_paper_embed: null data");
    if (cover != stego && overlaps(cover, n, stego, n))
        return fail(LSB_E_ARG, "lsb_paper_embed: cover and stego overlap (only stego == cover is allowed)");
    if (overlaps(data, len, stego, n)) return fail(LSB_E_ARG, "lsb_paper_embed: data overlaps stego");
    PaperSpan p{};
    p.src = cover;
    p.dst = stego;
    p.data = data;
    p.n = n;
    p.len = len;
    p.rowbytes = (uint64_t)w * c;
    p.w = w;
    p.c = c;
    p.plane = plane;
    p.q = w / 4;
    p.inplace = cover == stego;
    if (p.rowbytes >= (1ull << 31)) return fail(LSB_E_ARG, "lsb_paper_embed: rows of 2^31 bytes or more");
    // rows past the last data-carrying one: copied out-of-place, untouched in-place
    const uint64_t rows = p.inplace ? (p.q ? ceil_div(len, p.q) : 0) : h;
    if (rows == 0) return LSB_OK;
    const bool vec = p.rowbytes >= 16;
    if (vec && (c == 1 || c == 3 || c == 4)) {
        // vectors from 16-byte addresses on, plus the partial ones at a row's two ends
        const uint64_t units = ceil_div(p.rowbytes + (p.rowbytes % 16 ? 15 : (uintptr_t)stego % 16), 16);
        const Access a = access_kind(n);
        const RowFn *fn = c == 1 ? PaperEmbed<1>::fn[a] : (c == 3 ? PaperEmbed<3>::fn[a] : PaperEmbed<4>::fn[a]);
        if (launch_rows(fn, p, units, rows, 2, (hipStream_t)stream)) return launched("paper embed kernel launch");
    }
    hipEvent_t e0, e1;
    if ((c == 2 || c > 4) && paper_row_kernel(p, rows)) {
        take_launch_events(&e0, &e1);
        hipExtLaunchKernelGGL(lsb_paper_embed_rows_kernel, dim3((unsigned)rows), dim3(256),
                              (size_t)paper_row_lds_bytes(p.q), (hipStream_t)stream, e0, e1, 0, p);
        return launched("paper row embed kernel launch");
    }
    const uint64_t items = vec ? ceil_div(n, 16) : n;
    uint64_t blocks = ceil_div(items, 256);
    const uint64_t cap = (uint64_t)device_cus() * 16;
    if (blocks > cap) blocks = cap;
    take_launch_events(&e0, &e1);
    if (vec)
        hipExtLaunchKernelGGL(lsb_paper_embed_kernel<true>, dim3((unsigned)blocks), dim3(256), 0,
                              (hipStream_t)stream, e0, e1, 0, p);
    else
        hipExtLaunchKernelGGL(lsb_paper_embed_kernel<false>, dim3((unsigned)blocks), dim3(256), 0,
                              (hipStream_t)stream, e0, e1, 0, p);
    return launched("paper embed kernel launch");
}

int lsb_paper_extract(const uint8_t *stego, uint32_t h, uint32_t w, uint32_t c, uint32_t plane, uint8_t *data_out,
                      uint64_t len, void *stream) {
    const TimedCall timed_call;
    int rc = paper_check(h, w, c, plane, len, "lsb_paper_extract");
    if (rc) return rc;
    if (len == 0) return LSB_OK;
    const uint64_t n = (uint64_t)h * w * c;
    if (!stego || !data_out) return fail(LSB_E_ARG, "lsb_paper_extract: null stego/data_out");
    if (overlaps(data_out, len, stego, n)) return fail(LSB_E_ARG, "lsb_paper_extract: data_out overlaps stego");
    PaperSpan p{};
    p.src = stego;
    p.out = data_out;
    p.n = n;
    p.len = len;
    p.rowbytes = (uint64_t)w * c;
    p.w = w;
    p.c = c;
    p.plane = plane;
    p.q = w / 4;
    if (c <= 4) {
        const uint64_t units = ceil_div(p.q < len ? p.q : len, c == 1 ? 16 : 4);
        const RowFn *fn = c == 1   ? PaperExtract<1>::fn
                          : c == 2 ? PaperExtract<2>::fn
                          : c == 3 ? PaperExtract<3>::fn
                                   : PaperExtract<4>::fn;
        if (launch_rows(fn, p, units, ceil_div(len, p.q), 1, (hipStream_t)stream))
            return launched("paper extract kernel launch");
    }
    uint64_t blocks = ceil_div(len, 256);
    const uint64_t cap = (uint64_t)device_cus() * 16;
    if (blocks > cap) blocks = cap;
    hipEvent_t e0, e1;
    take_launch_events(&e0, &e1);
    hipExtLaunchKernelGGL(lsb_paper_extract_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, e0,
                          e1, 0, p);
    return launched("paper extract kernel launch");
}

}  // extern "C"
