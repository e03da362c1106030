// lsb_paper_device.hpp -- device code of the paper's own layout
// (arXiv:0912.0947, Section VI steps 2-7, Section VII steps 2-6): 2 bits per
// byte in one colour plane, greedy per-row data chunks, bit pair i of data
// byte j in plane pixel L*i + j.  Included by lsb_paper.hip.
#pragma once

#include "lsb_device.hpp"

namespace lsb {

struct PaperSpan {
    const uint8_t *src;
    uint8_t *dst;
    const uint8_t *data;
    uint8_t *out;
    uint64_t n;         // h * w * c
    uint64_t len;       // data bytes
    uint64_t rowbytes;  // w * c
    uint32_t w, c, plane, q;  // q = w / 4 data bytes per full row
    int inplace;
};

// New value of the plane byte at row y, pixel x (Section VI step 7: clear
// the low two bits, OR in bits 2i+1..2i of data byte j, with x = L*i + j).
__device__ __forceinline__ uint32_t paper_pixel(const PaperSpan &p, uint64_t y, uint32_t x, uint32_t byte) {
    const uint64_t first = y * p.q;  // first data byte of row y
    if (first >= p.len) return byte;
    const uint64_t left = p.len - first;
    const uint32_t L = left < p.q ? (uint32_t)left : p.q;
    if (x >= 4 * L) return byte;
    const uint32_t i = (x >= L) + (x >= 2 * L) + (x >= 3 * L);
    const uint32_t j = x - i * L;
    const uint32_t d = p.data[first + j];
    return (byte & 0xFCu) | ((d >> (2 * i)) & 3u);
}

// Bytes [t, t_end) of one row-ordered run, with (y, x, ch) the position of t.
// Walks positions by increments; applies paper_pixel to plane bytes.
__device__ __forceinline__ void paper_walk_bytes(const PaperSpan &p, uint64_t t, uint64_t t_end, uint8_t *bytes) {
    uint64_t y = t / p.rowbytes;
    const uint64_t rem = t - y * p.rowbytes;
    uint32_t x = (uint32_t)(rem / p.c);
    uint32_t ch = (uint32_t)(rem - (uint64_t)x * p.c);
    for (uint64_t k = 0; t + k < t_end; ++k) {
        if (ch == p.plane) bytes[k] = (uint8_t)paper_pixel(p, y, x, bytes[k]);
        if (++ch == p.c) {
            ch = 0;
            if (++x == p.w) {
                x = 0;
                ++y;
            }
        }
    }
}

// One 16-byte vector starting at cover byte t, for rows of at least 16
// bytes (so the vector touches at most two rows).  Positions advance by
// selects, all data-byte gathers of the vector are issued together, then the
// plane bytes of carrying rows are updated (Section VI step 7).
__device__ __forceinline__ u32x4 paper_vec16(const PaperSpan &p, uint64_t t, u32x4 v) {
    const uint64_t y = t / p.rowbytes;
    const uint32_t rem = (uint32_t)(t - y * p.rowbytes);
    uint32_t x = rem / p.c;
    uint32_t ch = rem - x * p.c;
    // data chunk of row y and of row y + 1
    uint64_t first[2];
    uint32_t L[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        first[r] = (y + r) * p.q;
        const uint64_t left = first[r] < p.len ? p.len - first[r] : 0;
        L[r] = left < p.q ? (uint32_t)left : p.q;
    }
    uint32_t row = 0;
    bool need[16];
    uint32_t pair[16];
    uint64_t at[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint32_t Lr = row ? L[1] : L[0];
        need[k] = ch == p.plane && x < 4 * Lr;
        const uint32_t i = (x >= Lr) + (x >= 2 * Lr) + (x >= 3 * Lr);
        pair[k] = 2 * i;
        at[k] = (row ? first[1] : first[0]) + (x - i * Lr);
        // advance to the next byte: channel, then pixel, then row
        const bool ch_wrap = ch + 1 == p.c;
        const bool x_wrap = ch_wrap && x + 1 == p.w;
        ch = ch_wrap ? 0 : ch + 1;
        x = x_wrap ? 0 : (ch_wrap ? x + 1 : x);
        row = x_wrap ? 1 : row;
    }
    uint32_t d[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) d[k] = need[k] ? p.data[at[k]] : 0u;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (need[k]) {
            const int sh = 8 * (k & 3);
            const uint32_t val = (d[k] >> pair[k]) & 3u;
            v[k >> 2] = (v[k >> 2] & ~(3u << sh)) | (val << sh);
        }
    }
    return v;
}

// Embed of channel counts without a unit kernel (below) where the row kernel
// does not apply either, and of rows under 16 bytes: every cover byte is read once and written once (16 bytes per lane
// when rows hold at least 16 bytes, else one byte per lane).
template <bool VEC>
__global__ void __launch_bounds__(256) lsb_paper_embed_kernel(PaperSpan p) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t rows_with_data = p.q ? ceil_div(p.len, p.q) : 0;
    const uint64_t data_end = rows_with_data * p.rowbytes;  // bytes past it never change
    if constexpr (VEC) {
        const uint64_t vecs = ceil_div(p.n, 16);
        for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < vecs; u += stride) {
            const uint64_t t = 16 * u;
            if (t + 16 <= p.n) {
                u32x4 v = load16<true>(p.src + t);
                if (t >= data_end) {  // no data in this vector's rows
                    if (!p.inplace) store16<true>(p.dst + t, v);
                    continue;
                }
                store16<true>(p.dst + t, paper_vec16(p, t, v));
            } else {
                uint8_t b[16];
                const uint64_t m = p.n - t;
                for (uint64_t k = 0; k < m; ++k) b[k] = p.src[t + k];
                paper_walk_bytes(p, t, p.n, b);
                for (uint64_t k = 0; k < m; ++k) p.dst[t + k] = b[k];
            }
        }
    } else {
        for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < p.n; t += stride) {
            uint8_t b = p.src[t];
            if (t < data_end) paper_walk_bytes(p, t, t + 1, &b);
            if (!p.inplace || t < data_end) p.dst[t] = b;
        }
    }
}

// -------------------------------------------------------------------------
// Row-per-block embed of channel counts without a unit kernel (2, and more than
// 4).  Block y handles image row y: it stages the row's data chunk (data bytes
// [y*q, y*q + L)) in LDS with dword loads, then each lane streams 16-byte vectors
// of the row and rewrites their plane bytes from LDS (Section VI steps 5-7).  No
// 64-bit division and no scattered global gathers, which the grid-stride kernel
// above pays for: 134 MB of two
// channels 77 us against 106, 101 MB of six 59 against 80, 24 MB of two 17.7
// against 21.6; in place likewise.  Used where rows are long, aligned and many
// enough (lsb_paper.hip).

struct PaperRow {
    const uint8_t *src;
    uint8_t *dst;
    uint64_t first;  // first data byte of the row
    uint32_t L;      // data bytes of the row (0: the row carries none)
    uint32_t h0;     // (data + first) % 4: LDS offset of data byte `first`
};

__device__ __forceinline__ PaperRow paper_row(const PaperSpan &p, uint64_t y) {
    PaperRow r;
    r.src = p.src + y * p.rowbytes;
    r.dst = p.dst + y * p.rowbytes;
    r.first = y * p.q;
    const uint64_t left = r.first < p.len ? p.len - r.first : 0;
    r.L = left < p.q ? (uint32_t)left : p.q;
    r.h0 = (uint32_t)((uintptr_t)(p.data + r.first) & 3u);
    return r;
}

// Copy a row that carries no data (out-of-place only).
__device__ __forceinline__ void paper_row_copy(const PaperSpan &p, const PaperRow &r, uint32_t tid, uint32_t nthreads) {
    const uint32_t rowvecs = (uint32_t)(p.rowbytes / 16);
    for (uint32_t u = tid; u < rowvecs; u += nthreads) store16<true>(r.dst + 16 * (uint64_t)u, load16<true>(r.src + 16 * (uint64_t)u));
}

// Stage data bytes [first, first + L) at chunk[h0 .. h0 + L): whole dwords
// of the data buffer land on aligned LDS dwords; the partial dwords at the
// two ends are copied byte by byte, so no byte outside the chunk is read.
__device__ __forceinline__ void paper_row_stage(const PaperSpan &p, const PaperRow &r, uint8_t *chunk, uint32_t tid,
                                                uint32_t nthreads) {
    const uint8_t *a = p.data + r.first;
    const uint32_t *aw = reinterpret_cast<const uint32_t *>(a - r.h0);
    const uint32_t end = r.h0 + r.L;
    const uint32_t nw = (end + 3) / 4;
    for (uint32_t w = tid; w < nw; w += nthreads) {
        const uint32_t lo = 4 * w;
        if (lo >= r.h0 && lo + 4 <= end) {
            reinterpret_cast<uint32_t *>(chunk)[w] = aw[w];
        } else {
            for (uint32_t b = lo; b < lo + 4; ++b)
                if (b >= r.h0 && b < end) chunk[b] = a[b - r.h0];
        }
    }
}

// New value of the 16 row bytes at row offset o (Section VI step 7): for a
// plane byte of pixel x < 4L, i = x / L (by three compares) and j = x - i*L;
// its low two bits become bits 2i+1..2i of data byte j (data = the staged
// chunk, data[j] = data byte first + j).  All 16 LDS reads are issued before
// any is used; bytes that take no data read data[0] and keep their value.
__device__ __forceinline__ u32x4 paper_row_vec(const PaperSpan &p, const uint8_t *data, uint32_t L, uint32_t o,
                                               u32x4 v) {
    uint32_t x = o / p.c;
    uint32_t ch = o - x * p.c;
    const uint32_t four_l = 4 * L;
    bool need[16];
    uint32_t shift[16], d[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        need[k] = ch == p.plane && x < four_l;
        const uint32_t i = (x >= L) + (x >= 2 * L) + (x >= 3 * L);
        shift[k] = 2 * i;
        d[k] = data[need[k] ? x - i * L : 0];
        const bool wrap = ch + 1 == p.c;
        ch = wrap ? 0 : ch + 1;
        x = wrap ? x + 1 : x;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int sh = 8 * (k & 3);
        const uint32_t nv = (v[k >> 2] & ~(3u << sh)) | (((d[k] >> shift[k]) & 3u) << sh);
        v[k >> 2] = need[k] ? nv : v[k >> 2];
    }
    return v;
}

// This lane's vectors of a data-carrying row: UNR loads in flight, then the
// updates and stores.  `chunk` is the block's staged chunk.
__device__ __forceinline__ void paper_row_update(const PaperSpan &p, const PaperRow &r, const uint8_t *chunk,
                                                 uint32_t tid, uint32_t nthreads) {
    constexpr int UNR = 4;
    const uint32_t rowvecs = (uint32_t)(p.rowbytes / 16);
    for (uint32_t base = tid; base < rowvecs; base += UNR * nthreads) {
        u32x4 v[UNR];
#pragma unroll
        for (int m = 0; m < UNR; ++m) {
            const uint32_t u = base + m * nthreads;
            if (u < rowvecs) v[m] = load16<true>(r.src + 16 * (uint64_t)u);
        }
#pragma unroll
        for (int m = 0; m < UNR; ++m) {
            const uint32_t u = base + m * nthreads;
            if (u < rowvecs) store16<true>(r.dst + 16 * (uint64_t)u, paper_row_vec(p, chunk + r.h0, r.L, 16 * u, v[m]));
        }
    }
}

// LDS bytes of the row kernel for rows of q data bytes (at offset h0 < 4).
__host__ __device__ constexpr uint64_t paper_row_lds_bytes(uint64_t q) { return (q + 3 + 15) / 16 * 16; }

__global__ void __launch_bounds__(256) lsb_paper_embed_rows_kernel(PaperSpan p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t paper_chunk[];
    const PaperRow r = paper_row(p, blockIdx.x);
    if (r.L == 0) {
        if (!p.inplace) paper_row_copy(p, r, threadIdx.x, blockDim.x);
        return;
    }
    paper_row_stage(p, r, paper_chunk, threadIdx.x, blockDim.x);
    __syncthreads();
    paper_row_update(p, r, paper_chunk, threadIdx.x, blockDim.x);
}

// 128-bit value t shifted left by r bytes (r < 4), dword 0 lowest.
__device__ __forceinline__ void shl_bytes(uint32_t *t, uint32_t r) {
    const uint32_t sh = 32 - 8 * r;
#pragma unroll
    for (int d = 3; d >= 0; --d) t[d] = (uint32_t)((((uint64_t)t[d] << 32) | (d ? t[d - 1] : 0u)) >> sh);
}

// Six packed bytes (bytes 0..3 of p0, 0..1 of p1) to bytes 0, 3, 6, 9, 12,
// 15 of a 128-bit value, then shifted left by r bytes.
__device__ __forceinline__ void spread3(uint32_t p0, uint32_t p1, uint32_t r, uint32_t *t) {
    t[0] = (p0 & 0xFFu) | ((p0 & 0xFF00u) << 16);
    t[1] = p0 & 0xFF0000u;
    t[2] = (p0 >> 16) & 0xFF00u;
    t[3] = (p1 & 0xFFu) | ((p1 & 0xFF00u) << 16);
    shl_bytes(t, r);
}

// Extract of more than 4 channels: one lane per data byte d; row y = d / q holds bytes
// [y*q, y*q + L); byte j of the row is ORed together from the low two bits
// of pixels L*i + j, shifted left by 2i (Section VII step 6).
__global__ void __launch_bounds__(256) lsb_paper_extract_kernel(PaperSpan p) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t d = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; d < p.len; d += stride) {
        const uint64_t y = d / p.q;
        const uint64_t first = y * p.q;
        const uint32_t j = (uint32_t)(d - first);
        const uint64_t left = p.len - first;
        const uint32_t L = left < p.q ? (uint32_t)left : p.q;
        const uint8_t *row = p.src + y * p.rowbytes + p.plane;
        uint32_t v = 0;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) v |= ((uint32_t)row[(uint64_t)(L * i + j) * p.c] & 3u) << (2 * i);
        p.out[d] = (uint8_t)v;
    }
}

// -------------------------------------------------------------------------
// Units of rows.  Each row of a plane is cut into units (16-byte vectors of
// the image for embed, runs of 16 or 4 data bytes for extract) that start at
// the row's start and, where the row is no multiple, end with one unit moved
// back to the row's end: it overlaps its neighbour and both write the same
// bytes.  A block takes whole rows if they are short, else an equal share of
// one row, so that no width leaves a block nearly empty.
struct RowMap {
    uint32_t units;   // per row
    uint32_t rows;    // rows per block (> 1: short rows)
    uint32_t blocks;  // blocks per row (> 1: long rows)
    uint32_t share;   // units per block of a long row
    uint32_t magic;   // thread / units = thread * magic >> 20 (thread < 1024)
};

// (row, unit) of item t of this block; false for none.  SHORT: several rows
// per block; otherwise the row is the block's and stays in scalars.
template <bool SHORT>
__device__ __forceinline__ bool row_unit(const RowMap &m, uint64_t n_rows, uint32_t t, uint64_t *y, uint32_t *u) {
    const uint32_t b = xcd_run_block(blockIdx.x, gridDim.x);
    if constexpr (SHORT) {
        const uint32_t r = (t * m.magic) >> 20;
        *y = (uint64_t)b * m.rows + r;
        *u = t - r * m.units;
        return r < m.rows && *y < n_rows;
    } else {
        const uint32_t row = m.blocks > 1 ? __builtin_amdgcn_readfirstlane(b / m.blocks) : b;
        *y = row;
        *u = (b - row * m.blocks) * m.share + t;
        return t < m.share && *u < m.units;
    }
}

// Eight data bytes from index a on, as far as the buffer goes (zero past its
// end), for buffers of at least 8 bytes: the load moves back inside.
__device__ __forceinline__ uint64_t data8(const uint8_t *data, uint64_t len, uint64_t a) {
    if (a >= len) return 0;
    const uint64_t at = a < len - 8 ? a : len - 8;
    const u32_any *q = reinterpret_cast<const u32_any *>(data + at);
    return ((uint64_t)q[1] << 32 | q[0]) >> (8 * (uint32_t)(a - at));
}

// Bit pairs of the W pixels xf .. xf + W - 1 of a row (W <= 8), one per byte,
// and 0x03 in keep for each pixel that takes data.  The pixels' data bytes
// are one run of the row's chunk [first, first + L), or, where the run meets
// the end of a quarter, the end of one run and the start of the chunk (bit
// pair i + 1).  Needs L >= W, so that at most one quarter ends in the run.
template <int W>
__device__ __forceinline__ void row_pairs(const PaperSpan &p, uint64_t first, uint32_t L, uint32_t xf,
                                          uint64_t *pairs, uint64_t *keep) {
    const uint64_t threes = 0x0303030303030303ull;
    const uint32_t i = (xf >= L) + (xf >= 2 * L) + (xf >= 3 * L);
    const uint32_t j = xf - i * L;
    const uint32_t ms = L - j;  // pixels left in quarter i
    uint64_t v = (data8(p.data, p.len, first + j) >> (2 * i)) & threes;
    uint64_t k = threes;
    if (ms < W) {
        const uint64_t low = (1ull << (8 * ms)) - 1;
        uint64_t next = 0;
        if (i < 3) next = ((data8(p.data, p.len, first) << (8 * ms)) >> (2 * (i + 1))) & threes;
        v = (v & low) | (next & ~low);
        k = i < 3 ? threes : threes & low;
    }
    *pairs = v;
    *keep = k;
}

// Same for any L, pixel by pixel (rows that carry fewer than W bytes).
template <int W>
__device__ __forceinline__ void row_pairs_short(const PaperSpan &p, uint64_t first, uint32_t L, uint32_t xf,
                                                uint64_t *pairs, uint64_t *keep) {
    *pairs = *keep = 0;
#pragma unroll
    for (uint32_t m = 0; m < W; ++m) {
        const uint32_t x = xf + m;
        const uint32_t i = (x >= L) + (x >= 2 * L) + (x >= 3 * L);
        if (x >= 4 * L) continue;
        const uint64_t d = p.data[first + x - i * L];
        *pairs |= ((d >> (2 * i)) & 3u) << (8 * m);
        *keep |= 3ull << (8 * m);
    }
}

template <int W>
__device__ __forceinline__ void row_pairs_any(const PaperSpan &p, uint64_t first, uint32_t L, uint32_t xf,
                                              uint64_t *pairs, uint64_t *keep) {
    if (xf >= 4 * L) {
        *pairs = *keep = 0;
    } else if (L >= W && p.len >= 8) {
        row_pairs<W>(p, first, L, xf, pairs, keep);
    } else {
        row_pairs_short<W>(p, first, L, xf, pairs, keep);
    }
}

// Place a vector's bit pairs (one per plane byte, dword 0 first) and their
// keep masks into v; r is the offset of its first plane byte (c = 3).
template <int C>
__device__ __forceinline__ u32x4 place_pairs(const PaperSpan &p, u32x4 v, const uint32_t *pr, const uint32_t *kp,
                                             uint32_t r) {
    if constexpr (C == 1) {
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = (v[d] & ~kp[d]) | pr[d];
    } else if constexpr (C == 3) {
        uint32_t tp[4], tk[4];
        spread3(pr[0], pr[1], r, tp);
        spread3(kp[0], kp[1], r, tk);
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = (v[d] & ~tk[d]) | tp[d];
    } else {
        static_assert(C == 4, "units of c = 1, 3, 4");
        const uint32_t sh = 8 * p.plane;  // whole pixels: byte `plane` of each dword
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t pd = ((pr[0] >> (8 * d)) & 3u) << sh, kd = ((kp[0] >> (8 * d)) & 3u) << sh;
            v[d] = (v[d] & ~kd) | pd;
        }
    }
    return v;
}

// One row vector: its row's data chunk and its first plane byte.
struct RowVec {
    uint64_t first;  // first data byte of the row
    uint32_t L;      // data bytes of the row
    uint32_t o;      // row offset
    uint32_t r, xf;  // first plane byte and its pixel
};

template <int C>
__device__ __forceinline__ RowVec row_vec(const PaperSpan &p, uint64_t y, uint32_t o) {
    RowVec t;
    t.first = y * p.q;
    const uint64_t left = t.first < p.len ? p.len - t.first : 0;
    t.L = left < p.q ? (uint32_t)left : p.q;
    t.o = o;
    t.r = C == 3 ? (p.plane + 3u - o % 3u) % 3u : 0;
    t.xf = C == 1 ? o : (C == 3 ? (o + t.r) / 3u : o / 4u);
    return t;
}

// Dwords of data bytes a vector reads, and the pixels it may hold.
template <int C>
struct RowUnit {
    static constexpr int ND = C == 1 ? 4 : 2, W = C == 1 ? 16 : (C == 3 ? 6 : 4);
};

// Whether the vector's pixels all lie in one quarter and its data dwords in
// the buffer; then their place and shift.
template <int C>
__device__ __forceinline__ bool row_direct(const PaperSpan &p, const RowVec &t, const uint8_t **at, uint32_t *shift) {
    const uint32_t i = (t.xf >= t.L) + (t.xf >= 2 * t.L) + (t.xf >= 3 * t.L);
    const uint32_t j = t.xf - i * t.L;
    *at = p.data + t.first + j;
    *shift = 2 * i;
    return j + RowUnit<C>::W <= t.L && t.first + j + 4 * RowUnit<C>::ND <= p.len;
}

// Any vector, pairs looked up pixel run by pixel run.
template <int C>
__device__ __forceinline__ u32x4 row_general(const PaperSpan &p, const RowVec &t, u32x4 v) {
    uint64_t pr[2] = {}, kp[2] = {};
    row_pairs_any<C == 1 ? 8 : RowUnit<C>::W>(p, t.first, t.L, t.xf, &pr[0], &kp[0]);
    if constexpr (C == 1) row_pairs_any<8>(p, t.first, t.L, t.xf + 8, &pr[1], &kp[1]);
    const uint32_t prw[4] = {(uint32_t)pr[0], (uint32_t)(pr[0] >> 32), (uint32_t)pr[1], (uint32_t)(pr[1] >> 32)};
    const uint32_t kpw[4] = {(uint32_t)kp[0], (uint32_t)(kp[0] >> 32), (uint32_t)kp[1], (uint32_t)(kp[1] >> 32)};
    return place_pairs<C>(p, v, prw, kpw, t.r);
}

// Embed, two 16-byte vectors of a row per thread (t and t + the block), any
// width of at least 16 bytes and any alignment (Section VI steps 5-7).  Where
// all vectors of a wave are direct, the loads of both and of their data
// bytes are issued together.  HBM bounds it; a data byte is read by four
// vectors of its row, from L2 after the first (XCD runs keep a row's blocks on
// one XCD).  8192x8192x3: 65.4 us (6.4 TB/s), 67.2 us by a block per row that
// staged the data in LDS and needed aligned rows of 16-byte multiples; other
// widths, by 16-byte vectors across rows with a gather per byte: 8191x8191x3
// 159 -> 69 us, 14000x14001x1 174 -> 74 us, 768x1366x3 5.3 -> 4.1 us.
template <int C, bool SHORT, int ACC>
__global__ void __launch_bounds__(1024) lsb_paper_embed_units_kernel(PaperSpan p, RowMap map, uint64_t n_rows) {
    constexpr bool NT = ACC != CACHED, NTS = ACC == STREAM;
    constexpr int UNR = 2, ND = RowUnit<C>::ND;
    const uint32_t rowbytes = (uint32_t)p.rowbytes;
    uint64_t pos[UNR];
    RowVec t[UNR];
    const uint8_t *at[UNR];
    uint32_t shift[UNR];
    bool any[UNR], direct = true;
    u32x4 v[UNR];
#pragma unroll
    for (int m = 0; m < UNR; ++m) {
        uint64_t y;
        uint32_t u;
        any[m] = row_unit<SHORT>(map, n_rows, threadIdx.x + m * blockDim.x, &y, &u);
        const uint32_t mis = (uint32_t)(uintptr_t)(p.dst + y * p.rowbytes) & (C == 4 ? 12u : 15u);  // c = 4: whole pixels
        any[m] = any[m] && (u == 0 || 16 * u - mis < rowbytes);
        uint32_t o = u ? 16 * u - mis : 0;  // vectors inside a row start at 16-byte addresses
        if (o > rowbytes - 16) o = rowbytes - 16;
        pos[m] = y * p.rowbytes + o;
        t[m] = row_vec<C>(p, y, o);
        direct = row_direct<C>(p, t[m], &at[m], &shift[m]) && any[m] && direct;
    }
    if (__all(direct)) {
        uint32_t d[UNR][ND];
#pragma unroll
        for (int m = 0; m < UNR; ++m) {
            v[m] = load16<NT>(p.src + pos[m]);
            const u32_any *q = reinterpret_cast<const u32_any *>(at[m]);
#pragma unroll
            for (int w = 0; w < ND; ++w) d[m][w] = q[w];
        }
#pragma unroll
        for (int m = 0; m < UNR; ++m) {
            uint32_t kp[ND];
#pragma unroll
            for (int w = 0; w < ND; ++w) {
                d[m][w] = (d[m][w] >> shift[m]) & 0x03030303u;
                kp[w] = 0x03030303u;
            }
            store16<NTS>(p.dst + pos[m], place_pairs<C>(p, v[m], d[m], kp, t[m].r));
        }
        return;
    }
#pragma unroll
    for (int m = 0; m < UNR; ++m)
        if (any[m]) v[m] = load16<NT>(p.src + pos[m]);
#pragma unroll
    for (int m = 0; m < UNR; ++m)
        if (any[m]) store16<NTS>(p.dst + pos[m], row_general<C>(p, t[m], v[m]));
}

// Four plane bytes of the four pixels whose C * 4 bytes are in d (Section VII
// step 6 masks their low two bits later).
template <int C>
__device__ __forceinline__ uint32_t plane4(const uint32_t *d, uint32_t plane) {
    if constexpr (C == 1) {
        return d[0];
    } else {
        const uint32_t sh = 8 * plane;
        uint32_t v = 0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {  // byte C*m + plane: within dword C*m/4 or the next
            const int b = C * m;
            const uint64_t pair = (uint64_t)(b / 4 + 1 < C ? d[b / 4 + 1] : 0u) << 32 | d[b / 4];
            v |= ((uint32_t)(pair >> (8 * (b % 4) + sh)) & 0xFFu) << (8 * m);
        }
        return v;
    }
}

// Extract, a run of N data bytes of a row per thread (N = 16 for one channel,
// else 4): bit pair i of the run is in the low bits of the plane bytes of
// pixels L*i + j .., which are contiguous, so each quarter is one load of
// N * C bytes and neighbouring threads read neighbouring bytes.  Against one
// byte and four gathers per thread: 8192x8192x3 50.7 -> 35 us (5.6 TB/s of the
// lines touched), one channel 23.5 -> 12 us.
template <int C, bool SHORT>
__global__ void __launch_bounds__(1024) lsb_paper_extract_units_kernel(PaperSpan p, RowMap map, uint64_t n_rows) {
    constexpr int N = C == 1 ? 16 : 4, ND = N / 4;  // data bytes and dwords
    uint64_t y;
    uint32_t u;
    if (!row_unit<SHORT>(map, n_rows, threadIdx.x, &y, &u)) return;
    const uint64_t first = y * p.q;
    const uint64_t left = p.len - first;  // n_rows rows carry data
    const uint32_t L = left < p.q ? (uint32_t)left : p.q;
    if (N * u >= L) return;  // the last row may be short
    const uint8_t *row = p.src + y * p.rowbytes;
    uint8_t *out = p.out + first;
    if (L < N) {
        for (uint32_t j = 0; j < L; ++j) {
            uint32_t v = 0;
            for (uint32_t i = 0; i < 4; ++i)
                v |= ((uint32_t)row[(uint64_t)(L * i + j) * C + p.plane] & 3u) << (2 * i);
            out[j] = (uint8_t)v;
        }
        return;
    }
    const uint32_t j = N * u + N <= L ? N * u : L - N;
    uint32_t d[4][ND * C];
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        const u32_any *q = reinterpret_cast<const u32_any *>(row + (uint64_t)(L * i + j) * C);
#pragma unroll
        for (int w = 0; w < ND * C; ++w) d[i][w] = q[w];
    }
    u32_any *o = reinterpret_cast<u32_any *>(out + j);
#pragma unroll
    for (int w = 0; w < ND; ++w) {
        uint32_t v = 0;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) v |= (plane4<C>(d[i] + w * C, p.plane) & 0x03030303u) << (2 * i);
        o[w] = v;
    }
}

}  // namespace lsb
