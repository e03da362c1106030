// lsb_plane_device.hpp -- device code for one colour plane with the general
// method (arXiv:0912.0947, Section VI step 2 / Section VII step 2 select the
// plane; steps VI.7 / VII.6 place and gather the bits).  Included by
// lsb_plane.hip.
#pragma once

#include "../../include/lsb.h"
#include "lsb_device.hpp"

namespace lsb {

// Buffer byte of field t in a plane view.
__device__ __forceinline__ uint64_t plane_byte(uint64_t t, uint32_t c, uint32_t plane) {
    return t * c + plane;
}

// Embed field t of the plane view (Section VI step 7, k-bit fields).
__device__ __forceinline__ void plane_embed_field(const Span &s, uint64_t t, uint32_t c, uint32_t plane) {
    const uint32_t k = (uint32_t)s.k;
    const uint64_t first = (uint64_t)k * t;
    if (first >= s.bits) return;
    const uint64_t left = s.bits - first;
    const uint32_t nb = left < k ? (uint32_t)left : k;
    const uint64_t byte = first >> 3;
    const uint32_t bit = (uint32_t)(first & 7);
    uint32_t pair = stream_byte(s, byte) << 8;
    if (bit + nb > 8) pair |= stream_byte(s, byte + 1);
    const uint32_t v = (pair >> (16 - bit - nb)) & ((1u << nb) - 1u);
    const uint32_t shift = k - nb;
    const uint32_t mask = ((1u << nb) - 1u) << shift;
    const uint64_t at = plane_byte(t, c, plane);
    s.dst[at] = (uint8_t)((s.src[at] & ~mask) | (v << shift));
}

// Stream byte i (>= 4) of a plane view from its fields (Section VII step 6).
__device__ __forceinline__ uint32_t plane_stream_byte(const Span &s, uint64_t i, uint32_t c, uint32_t plane) {
    const uint32_t k = (uint32_t)s.k;
    const uint32_t low = (1u << k) - 1u;
    const uint64_t b0 = 8 * i;
    const uint64_t b1 = (b0 + 8 < s.bits) ? b0 + 8 : s.bits;
    const uint64_t g_first = b0 / k, g_last = (b1 - 1) / k;
    uint32_t acc = 0, nbits = 0;
    for (uint64_t g = g_first; g <= g_last; ++g) {
        acc = (acc << k) | (s.src[plane_byte(g, c, plane)] & low);
        nbits += k;
    }
    const uint32_t skip = (uint32_t)(b0 - (uint64_t)k * g_first);
    const uint32_t v = ((acc << (32 - nbits)) << skip) >> 24;
    const uint32_t valid = (uint32_t)(b1 - b0);
    return v & ((0xFF00u >> valid) & 0xFFu);
}

__global__ void __launch_bounds__(256) lsb_copy_kernel(const uint8_t *src, uint8_t *dst, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t nv = n / 16;
    for (uint64_t u = gid; u < nv; u += stride) store16<true>(dst + 16 * u, load16<true>(src + 16 * u));
    for (uint64_t t = 16 * nv + gid; t < n; t += stride) dst[t] = src[t];
}

__global__ void __launch_bounds__(256) lsb_plane_embed_kernel(Span s, uint64_t fields, uint32_t c, uint32_t plane) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < fields; t += stride)
        plane_embed_field(s, t, c, plane);
}

// Header decode on the plane view (lane j < 32 reads stream bit j), status
// through block 0, then one lane per message byte.
__global__ void __launch_bounds__(256) lsb_plane_extract_kernel(Span s, uint32_t c, uint32_t plane, uint64_t out_cap,
                                                                uint32_t *len_out, int32_t *status_out) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t k = (uint32_t)s.k;
    uint32_t len = 0;
    int status = LSB_E_HEADER;
    if ((uint64_t)k * s.n >= 32) {
        uint32_t bit = 0;
        if (lane < 32) bit = (s.src[plane_byte(lane / k, c, plane)] >> (k - 1 - lane % k)) & 1u;
        len = __builtin_bitreverse32((uint32_t)__ballot(bit));
        if (4 + (uint64_t)len > room_bytes(s.n, (int)k)) status = LSB_E_HEADER;
        else if ((uint64_t)len > out_cap) status = LSB_E_BUFFER;
        else status = LSB_OK;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *len_out = len;
        *status_out = status;
    }
    if (status != LSB_OK) return;
    s.bits = 8 * (4 + (uint64_t)len);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t m = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; m < len; m += stride)
        s.out[m] = (uint8_t)plane_stream_byte(s, m + 4, c, plane);
}

// ---------------------------------------------------------------------------
// Extract for C in {2, 3, 4} channels: a lane takes 16 pixels = C 16-byte
// vectors, gathers their plane bytes into one 16-field vector and runs the
// plain vector extract on it.  All byte positions are compile-time constants
// (C and PLANE are template parameters), so the gather is register bit-field
// moves.
template <int C, int PLANE>
__device__ __forceinline__ u32x4 plane_gather(const u32x4 *v) {
    u32x4 p = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int f = 0; f < 16; ++f) {
        const int b = f * C + PLANE;
        const uint32_t byte = (v[b >> 4][(b & 15) >> 2] >> (8 * (b & 3))) & 0xFFu;
        p[f >> 2] |= byte << (8 * (f & 3));
    }
    return p;
}

template <int K, int C>
__device__ __forceinline__ u32x4 plane_gather_any(const u32x4 *v, uint32_t plane) {
    switch (plane) {
        case 0: return plane_gather<C, 0>(v);
        case 1: return plane_gather<C, 1>(v);
        case 2: if constexpr (C > 2) return plane_gather<C, 2>(v); break;
        default: if constexpr (C > 3) return plane_gather<C, 3>(v); break;
    }
    return u32x4{0u, 0u, 0u, 0u};
}

// Wave groups: a wave takes 64 consecutive 16-pixel units (64*C vectors,
// C KiB of the interleaved buffer).  When the whole group is fast, the wave
// loads it with C contiguous 1 KiB accesses into LDS and each lane reads back
// its own C vectors (16 pixels): every global access of the wave covers one
// contiguous span, instead of 64 lanes touching C-vector runs at a stride of
// 16*C bytes.  Other groups (header, stream end, buffer tail) go lane by lane.

// stage[64*i + lane] = vector 64*i + lane of the group.
template <int C, bool NT>
__device__ __forceinline__ void plane_group_load(const uint8_t *src, u32x4 *stage, uint32_t lane) {
#pragma unroll
    for (int i = 0; i < C; ++i) stage[64 * i + lane] = load16<NT>(src + 16 * (64 * i + lane));
}

// Embed of a plane, 16-byte vectors of the interleaved buffer.  A vector holds
// W = 4 to 8 plane bytes (every C-th byte, from byte r on), so its fields are
// at most 64 stream bits from any bit on: one unaligned 8-byte read.  The
// fields are unpacked to one byte each and spread to every C-th byte.  Nothing
// is shared between lanes: memory is read and written as a plain copy.
template <int C>
struct PlaneVec {
    static constexpr int W = C == 2 ? 8 : (C == 3 ? 6 : 4);
};

// W fields of K bits, the first in the top bits of x, to one byte each.
template <int K, int W>
__device__ __forceinline__ uint64_t unpack_fields(uint64_t x) {
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int m = 0; m < W; ++m) {
        const uint32_t f = (uint32_t)(x >> (64 - K * (m + 1))) & ((1u << K) - 1u);
        if (m < 4) lo |= f << (8 * m);
        else hi |= f << (8 * (m - 4));
    }
    return (uint64_t)hi << 32 | lo;
}

// Bytes 0.. of f to bytes r, r + C, ... of a 16-byte vector (r < C).
template <int C>
__device__ __forceinline__ u32x4 spread_fields(uint64_t f, uint32_t r) {
    const uint32_t lo = (uint32_t)f, hi = (uint32_t)(f >> 32);
    uint32_t t[4];
    if constexpr (C == 2) {
        const uint32_t h[4] = {lo & 0xFFFFu, lo >> 16, hi & 0xFFFFu, hi >> 16};
#pragma unroll
        for (int d = 0; d < 4; ++d) t[d] = ((h[d] & 0xFFu) | ((h[d] & 0xFF00u) << 8)) << (8 * r);
    } else if constexpr (C == 3) {
        t[0] = (lo & 0xFFu) | ((lo & 0xFF00u) << 16);
        t[1] = lo & 0xFF0000u;
        t[2] = (lo >> 16) & 0xFF00u;
        t[3] = (hi & 0xFFu) | ((hi & 0xFF00u) << 16);
        const uint32_t sh = 32 - 8 * r;
#pragma unroll
        for (int d = 3; d >= 0; --d) t[d] = (uint32_t)((((uint64_t)t[d] << 32) | (d ? t[d - 1] : 0u)) >> sh);
    } else {
#pragma unroll
        for (int d = 0; d < 4; ++d) t[d] = ((lo >> (8 * d)) & 0xFFu) << (8 * r);
    }
    return u32x4{t[0], t[1], t[2], t[3]};
}

// The stream bits of fields x .. x + W - 1 (first in the top bit), masked to
// the stream's end, byte by byte: header bytes come from the header value and
// no byte past the stream is read.  *nb_out: how many of the bits are stream.
template <int K, int W>
__device__ __forceinline__ uint64_t plane_bits_edge(const Span &s, uint64_t x, uint32_t *nb_out) {
    const uint64_t first = (uint64_t)K * x;
    const uint64_t left = s.bits > first ? s.bits - first : 0;
    const uint32_t nb = left < K * W ? (uint32_t)left : K * W;
    const uint32_t r = (uint32_t)(first & 7), bytes = nb ? (r + nb + 7) / 8 : 0;
    uint64_t v = 0;
#pragma unroll
    for (uint32_t i = 0; i < 8; ++i)
        if (i < bytes) v |= (uint64_t)stream_byte(s, (first >> 3) + i) << (56 - 8 * i);
    *nb_out = nb;
    v <<= r;
    return nb < 64 ? v & ~(~0ull >> nb) : v;
}

// Embed over the plane view; s.n = pixels, s.src/s.dst the interleaved
// cover/stego, header mode (t0 = 0), `bytes` = s.n * C, `count` vectors.  A
// block takes 512 vectors per step, two per thread.  HBM bounds it, as the
// plain embed.  Against 16 pixels per lane exchanged through LDS (the first
// and last of them byte by byte): 512x512x3 11.1 -> 4.2 us, 3000x4000x3 18.8
// -> 13.7 us, 8192x8192x3 74.2 -> 64.1 us (6.5 TB/s).
template <int K, int C, int ACC>
__global__ void __launch_bounds__(256)
    lsb_plane_embed_vec_kernel(Span s, uint32_t plane, uint64_t bytes, uint64_t count) {
    constexpr bool NT = ACC != CACHED, NTS = ACC == STREAM;
    constexpr int UNR = 2, W = PlaneVec<C>::W;
    const uint8_t *body = s.body - s.hdr_len;  // stream byte i at body + i
    const uint64_t end = s.bits / 8;           // whole stream bytes (header mode: bits is a multiple of 8)
    const uint64_t blocks = ceil_div(count, 256 * UNR);
    for (uint64_t b = xcd_run_block(blockIdx.x, gridDim.x); b < blocks; b += gridDim.x) {
        const uint64_t u0 = b * (256 * UNR), px0 = 16 * u0 / C;
        const uint32_t rem = (uint32_t)(16 * u0 - px0 * C);
        uint64_t at[UNR], x[UNR];
        uint32_t r[UNR];
        bool any[UNR], direct = true;
#pragma unroll
        for (int m = 0; m < UNR; ++m) {
            const uint32_t t = threadIdx.x + 256 * m;
            at[m] = 16 * (u0 + t);
            any[m] = u0 + t < count;
            // first plane byte at or past the vector's start
            const uint32_t o = rem + 16 * t;
            const uint32_t q = (o + (uint32_t)C - 1 - plane) / C;
            x[m] = px0 + q;
            r[m] = q * C + plane - o;
            const uint64_t byte = ((uint64_t)K * x[m]) >> 3;
            direct = direct && any[m] && at[m] + 16 <= bytes && byte >= s.hdr_len && byte + 8 <= end;
        }
        if (__all(direct)) {
            u32x4 v[UNR];
            uint64_t w[UNR];
#pragma unroll
            for (int m = 0; m < UNR; ++m) {
                v[m] = load16<NT>(s.src + at[m]);
                const u32_any *p = reinterpret_cast<const u32_any *>(body + (((uint64_t)K * x[m]) >> 3));
                w[m] = (uint64_t)bswap32(p[0]) << 32 | bswap32(p[1]);
            }
#pragma unroll
            for (int m = 0; m < UNR; ++m) {
                const uint32_t sh = (uint32_t)((uint64_t)K * x[m]) & 7u;
                const u32x4 f = spread_fields<C>(unpack_fields<K, W>(w[m] << sh), r[m]);
                const u32x4 keep = spread_fields<C>(((1u << K) - 1u) * 0x0101010101010101ull, r[m]);
                store16<NTS>(s.dst + at[m], (v[m] & ~keep) | f);
            }
        } else {
#pragma unroll 1
            for (int m = 0; m < UNR; ++m) {
                if (!any[m]) continue;
                uint32_t nb;
                const uint64_t w = plane_bits_edge<K, W>(s, x[m], &nb);
                if (nb == 0 && s.inplace) continue;
                const uint32_t nbytes = bytes - at[m] < 16 ? (uint32_t)(bytes - at[m]) : 16;
                const u32x4 v = load_bytes<NT>(s.src + at[m], nbytes);
                const u32x4 f = spread_fields<C>(unpack_fields<K, W>(w), r[m]);
                const u32x4 keep = spread_fields<C>(
                    unpack_fields<K, W>(nb >= 64 ? ~0ull : ~(~0ull >> nb)), r[m]);
                const u32x4 o = (v & ~keep) | f;
                // in place nothing past the last stream-carrying byte is written
                const uint32_t carry = r[m] + C * ((nb + K - 1) / K) - (C - 1);
                const uint32_t hi = s.inplace && carry < nbytes ? carry : nbytes;
                if (hi == 16) store16<NTS>(s.dst + at[m], o);
                else store_bytes<16>(s.dst + at[m], o, 0, hi);
            }
        }
    }
}

// Extract unit u from its C vectors v (fast units).
template <int K, int C>
__device__ __forceinline__ void plane_extract_vec_out(const Span &s, const u32x4 *v, uint64_t u, uint32_t plane) {
    const uintptr_t out_base = (uintptr_t)s.out - s.hdr_len;
    uint32_t w[Chunk<K>::NW];
    extract_vec<K>(plane_gather_any<K, C>(v, plane), w);
    uint8_t *p = reinterpret_cast<uint8_t *>(out_base + 2 * K * u);
    store_chunk<K>(p, w);
}

template <int K, int C>
__device__ __forceinline__ void plane_group_extract(const Span &s, const u32x4 *stage, uint64_t u, uint32_t lane,
                                                    uint32_t plane) {
    u32x4 v[C];
#pragma unroll
    for (int i = 0; i < C; ++i) v[i] = stage[C * lane + i];
    plane_extract_vec_out<K, C>(s, v, u, plane);
}

template <int K, int C>
__device__ __forceinline__ void plane_extract_unit(const Span &s, const Ranges &r, uint64_t u, uint32_t plane) {
    if (u >= r.fast_begin && u < r.fast_end) {
        u32x4 v[C];
#pragma unroll
        for (int i = 0; i < C; ++i) v[i] = load16<true>(s.src + 16 * (C * u + i));
        plane_extract_vec_out<K, C>(s, v, u, plane);
    } else {
        const uint64_t end_byte = ceil_div(s.bits, 8);
        const uint64_t i0 = 2 * K * u;
        for (uint64_t i = i0; i < i0 + 2 * K && i < end_byte; ++i)
            if (i >= s.hdr_len) s.out[i - s.hdr_len] = (uint8_t)plane_stream_byte(s, i, C, plane);
    }
}

// Extract over the plane view: header decode per wave (lane j < 32 reads
// stream bit j), status through block 0, then 2K message bytes per lane.
template <int K, int C, bool NT>
__global__ void __launch_bounds__(256)
    lsb_plane_extract_vec_kernel(Span s, uint32_t plane, uint64_t out_cap, uint32_t *len_out, int32_t *status_out) {
    __shared__ u32x4 stage_all[4][64 * C];
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t len = 0;
    int status = LSB_E_HEADER;
    if ((uint64_t)K * s.n >= 32) {
        uint32_t bit = 0;
        if (lane < 32) bit = (s.src[plane_byte(lane / K, C, plane)] >> (K - 1 - lane % K)) & 1u;
        len = __builtin_bitreverse32((uint32_t)__ballot(bit));
        if (4 + (uint64_t)len > room_bytes(s.n, K)) status = LSB_E_HEADER;
        else if ((uint64_t)len > out_cap) status = LSB_E_BUFFER;
        else status = LSB_OK;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *len_out = len;
        *status_out = status;
    }
    if (status != LSB_OK) return;
    s.bits = 8 * (4 + (uint64_t)len);
    const Ranges r = extract_ranges<K>(s);
    u32x4 *stage = stage_all[threadIdx.x >> 6];
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint64_t n_waves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    const uint64_t groups = ceil_div(r.count, 64);
    for (uint64_t g = wave; g < groups; g += n_waves) {
        const uint64_t u0 = 64 * g;
        if (u0 >= r.fast_begin && u0 + 64 <= r.fast_end) {
            plane_group_load<C, NT>(s.src + 16 * C * u0, stage, lane);
            __builtin_amdgcn_wave_barrier();
            plane_group_extract<K, C>(s, stage, u0 + lane, lane, plane);
            __builtin_amdgcn_wave_barrier();
        } else if (u0 + lane < r.count) {
            plane_extract_unit<K, C>(s, r, u0 + lane, plane);
        }
    }
}

}  // namespace lsb
