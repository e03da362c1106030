// lsb_device.hpp -- device-side building blocks of k-bit LSB embed/extract
// for gfx950 (CDNA4, wave64).
//
// Operation (arXiv:0912.0947): embedding, Section VI step 7 -- a cover byte
// keeps its bits above the field and takes k stream bits in the field;
// extraction, Section VII step 6 -- the field is masked out of the stego byte
// and its bits are placed back into the zero-initialised data byte.
//
// Stream: S = BE32(len) || msg in header mode, or a caller stream in raw
// mode, read most-significant bit first.  Buffer byte t is logical field
// g = t0 + t and carries stream bits k*g .. k*g+k-1, first bit highest.
//
// Work unit: one "vector" = 16 consecutive buffer bytes = 16 fields = 16k
// stream bits = 2k whole stream bytes (16k is a multiple of 8, so when k*t0
// is byte aligned every vector starts on a stream byte).  A lane moves one
// 16-byte vector of cover/stego per step with a single dwordx4 access and the
// matching 2k stream bytes with dwords (and a short for odd k), all at any
// byte address.
// Vectors are grouped 64 per wave access so that every load and store
// instruction of a wave touches one contiguous 1 KiB span.
//
// Each span of vectors splits into (computed once per wave, in scalars):
//   fast  -- all 16 fields full and every stream byte past the header,
//   copy  -- no stream bits at all (embed copies the cover),
//   edge  -- the rest (header bytes, the partial last field, the buffer tail),
//            masked; only a few vectors per buffer are edges.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lsb {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Memory forms of a vector, a dword and a short at any byte address: gfx950
// takes unaligned global accesses of every width (the compiler emits the same
// instructions as for aligned ones), so buffers need no alignment at all.
// A 36 MB cover behind a 54-byte file header at k = 2, embed + extract pass:
// 23.5 us, against 88 through the per-byte kernels that misaligned buffers used to
// take.  Kernels at byte 0 / 4 / 54, us: 201 MB k = 1 embed 63.8 / 69.2 / 73.3,
// extract 35.6 / 34.5 / 44.5, k = 4 78.2 / 77.9 / 77.8 and 45.6 / 45.9 / 50.6; 36 MB
// k = 2, read from the caches, 12.4 / 12.4 / 13.0 and 7.5 / 9.5 / 12.4; 0.8 MB no
// difference.
typedef u32x4 u32x4_any __attribute__((aligned(1)));
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint16_t u16_any __attribute__((aligned(1)));

__host__ __device__ inline uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

// -------------------------------------------------------------------------
// Description of one embed or extract over one buffer.
struct Span {
    const uint8_t *src;   // embed: cover; extract: stego
    uint8_t *dst;         // embed: stego; extract: unused
    const uint8_t *body;  // embed: stream source (msg in header mode)
    uint8_t *out;         // extract: destination of stream bytes >= hdr_len
    uint64_t n;           // buffer bytes
    uint64_t t0;          // logical field index of buffer byte 0
    uint64_t bits;        // embed: stream bits; extract: end bit e (exclusive)
    uint32_t hdr;         // header value (header mode)
    uint32_t hdr_len;     // 4 in header mode, 0 in raw mode
    int k;
    int inplace;          // embed: dst == src, skip copy-only bytes
    int block_order;      // plain kernels: 1 = blocks in runs of 16 per XCD
};

// Vector classes of a span (all in the span's own vector index space).
struct Ranges {
    uint64_t fast_begin, fast_end;  // fast vectors: [fast_begin, fast_end)
    uint64_t copy_begin, copy_end;  // copy vectors: [copy_begin, copy_end)
    uint64_t count;                 // vectors to visit: [0, count)
};

__host__ __device__ inline uint64_t stream_byte0(const Span &s) {
    return ((uint64_t)s.k * s.t0) >> 3;  // stream byte holding field t0's first bit
}

// The range functions take k as a compile-time constant on the device
// (KC > 0), so that their divisions by k and 2k become shifts or constant
// multiplies instead of 64-bit division sequences; KC = 0 reads s.k (host).
template <int KC = 0>
__host__ __device__ inline Ranges embed_ranges(const Span &s) {
    Ranges r;
    const uint64_t k = KC > 0 ? (uint64_t)KC : (uint64_t)s.k;
    const uint64_t full = s.bits / k;            // fields fully inside the stream
    const uint64_t any = ceil_div(s.bits, k);    // fields carrying any stream bit
    const uint64_t whole = s.n / 16;             // vectors fully inside the buffer
    const uint64_t sb = stream_byte0(s);
    r.fast_begin = sb >= s.hdr_len ? 0 : ceil_div(s.hdr_len - sb, 2 * k);
    const uint64_t f_end = full > s.t0 ? (full - s.t0) / 16 : 0;
    r.fast_end = f_end < whole ? f_end : whole;
    r.copy_begin = any > s.t0 ? ceil_div(any - s.t0, 16) : 0;
    r.copy_end = whole;
    const uint64_t all = ceil_div(s.n, 16);
    r.count = s.inplace ? (r.copy_begin < all ? r.copy_begin : all) : all;
    return r;
}

// For extract, s.bits is the end bit e <= k*(t0+n), and k*t0 % 8 == 0.
template <int KC = 0>
__host__ __device__ inline Ranges extract_ranges(const Span &s) {
    Ranges r;
    const uint64_t k = KC > 0 ? (uint64_t)KC : (uint64_t)s.k;
    const uint64_t full = s.bits / k;
    const uint64_t whole = s.n / 16;
    const uint64_t sb = stream_byte0(s);
    r.fast_begin = sb >= s.hdr_len ? 0 : ceil_div(s.hdr_len - sb, 2 * k);
    const uint64_t f_end = full > s.t0 ? (full - s.t0) / 16 : 0;
    r.fast_end = f_end < whole ? f_end : whole;
    r.copy_begin = r.copy_end = 0;
    const uint64_t end_byte = ceil_div(s.bits, 8);  // exclusive
    const uint64_t by_stream = end_byte > sb ? ceil_div(end_byte - sb, 2 * k) : 0;
    const uint64_t all = ceil_div(s.n, 16);
    r.count = by_stream < all ? by_stream : all;
    return r;
}

// -------------------------------------------------------------------------
// Memory access helpers.
template <bool NT>
__device__ __forceinline__ u32x4 load16(const uint8_t *p) {
    const u32x4_any *q = reinterpret_cast<const u32x4_any *>(p);
    if constexpr (NT) return __builtin_nontemporal_load(q);
    else return *q;
}

template <bool NT>
__device__ __forceinline__ void store16(uint8_t *p, u32x4 v) {
    u32x4_any *q = reinterpret_cast<u32x4_any *>(p);
    if constexpr (NT) __builtin_nontemporal_store(v, q);
    else *q = v;
}

// Access kinds of the layout kernels.
enum Access { CACHED = 0, STREAM_LOADS = 1, STREAM = 2 };

__device__ __forceinline__ uint32_t bswap32(uint32_t x) { return __builtin_bswap32(x); }

// Logical stream byte s (header bytes come from the header value).
__device__ __forceinline__ uint32_t stream_byte(const Span &s, uint64_t i) {
    if (i < s.hdr_len) return (s.hdr >> (8 * (3 - (uint32_t)i))) & 0xFFu;
    return s.body[i - s.hdr_len];
}

// Number of 32-bit words holding one vector's 16k stream bits.
template <int K> struct Chunk { static constexpr int NW = (K + 1) / 2; };

// Load one vector's 2K stream bytes that start at `p` (any alignment) as
// big-endian words (bit 31 of w[0] is the vector's first stream bit).
template <int K>
__device__ __forceinline__ void load_chunk(const uint8_t *p, uint32_t *w) {
    const u32_any *q = reinterpret_cast<const u32_any *>(p);
#pragma unroll
    for (int i = 0; i < K / 2; ++i) w[i] = bswap32(q[i]);
    if constexpr (K % 2 == 1) w[K / 2] = bswap32((uint32_t)*reinterpret_cast<const u16_any *>(p + 2 * K - 2));
}

// Same where the vector's first stream bit is bit r (1..7) of byte p[0]
// (k*t0 not byte aligned): reads 2K + 1 bytes, all of which hold bits of the
// vector.
template <int K>
__device__ __forceinline__ void load_chunk_shifted(const uint8_t *p, uint32_t r, uint32_t *w) {
    constexpr int NW = Chunk<K>::NW;
    uint32_t W[NW + 1];
    load_chunk<K>(p, W);
    const uint32_t last = p[2 * K];
    if constexpr (K % 2 == 0) {
        W[NW] = last << 24;
    } else {
        W[NW - 1] |= last << 8;
        W[NW] = 0;
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = (W[i] << r) | (W[i + 1] >> (32 - r));
}

// Field f (0..15) of a vector: K bits at chunk bit offset K*f.
template <int K>
__device__ __forceinline__ uint32_t get_field(const uint32_t *w, int f) {
    constexpr uint32_t low = (1u << K) - 1u;
    const int off = K * f;
    const int i = off >> 5, sh = off & 31;
    if (sh + K <= 32) return (w[i] >> (32 - sh - K)) & low;
    return ((w[i] << (sh + K - 32)) | (w[i + 1] >> (64 - sh - K))) & low;
}

template <int K>
__device__ __forceinline__ void put_field(uint32_t *w, int f, uint32_t v) {
    const int off = K * f;
    const int i = off >> 5, sh = off & 31;
    if (sh + K <= 32) {
        w[i] |= v << (32 - sh - K);
    } else {
        w[i] |= v >> (sh + K - 32);
        w[i + 1] |= v << (64 - sh - K);
    }
}

// Embed 16 fields: byte f of the vector keeps its bits above the field and
// takes field f of the chunk (Section VI step 7f, k-bit masks).
template <int K>
__device__ __forceinline__ u32x4 embed_vec(u32x4 c, const uint32_t *w) {
    u32x4 o;
    if constexpr (K == 1) {
        // The 16 stream bits sit in w[0] bits 31..16.  Reverse them so stream
        // bit f is bit f, then spread each nibble to the LSBs of 4 bytes with
        // one 24-bit multiply (shifts 0, 7, 14, 21 never overlap).
        const uint32_t r = __builtin_bitreverse32(w[0]);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t nib = (r >> (4 * d)) & 0xFu;
            const uint32_t spread = (nib * 0x204081u) & 0x01010101u;
            o[d] = (c[d] & 0xFEFEFEFEu) | spread;
        }
    } else if constexpr (K == 8) {
#pragma unroll
        for (int d = 0; d < 4; ++d) o[d] = bswap32(w[d]);
    } else {
        constexpr uint32_t low = (1u << K) - 1u;
        constexpr uint32_t keep = ~(low * 0x01010101u);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t f = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) f |= get_field<K>(w, 4 * d + j) << (8 * j);
            o[d] = (c[d] & keep) | f;
        }
    }
    return o;
}

// Extract 16 fields into the chunk's big-endian words (Section VII step 6:
// mask the field, shift it to its place, OR into zeroed data).
template <int K>
__device__ __forceinline__ void extract_vec(u32x4 c, uint32_t *w) {
#pragma unroll
    for (int i = 0; i < Chunk<K>::NW; ++i) w[i] = 0;
    if constexpr (K == 1) {
        // Gather the 4 LSBs of a dword into a nibble, first byte highest:
        // one multiply moves byte j's LSB (bit 8j) to bit 31-j.
        uint32_t v = 0;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t nib = ((c[d] & 0x01010101u) * 0x80402010u) >> 28;
            v |= nib << (28 - 4 * d);
        }
        w[0] = v;
    } else if constexpr (K == 8) {
#pragma unroll
        for (int d = 0; d < 4; ++d) w[d] = bswap32(c[d]);
    } else {
        constexpr uint32_t low = (1u << K) - 1u;
#pragma unroll
        for (int f = 0; f < 16; ++f) put_field<K>(w, f, (c[f >> 2] >> (8 * (f & 3))) & low);
    }
}

// Store one vector's 2K stream bytes from big-endian words at `p` (any
// alignment).
template <int K>
__device__ __forceinline__ void store_chunk(uint8_t *p, const uint32_t *w) {
    u32_any *q = reinterpret_cast<u32_any *>(p);
#pragma unroll
    for (int i = 0; i < K / 2; ++i) q[i] = bswap32(w[i]);
    if constexpr (K % 2 == 1) *reinterpret_cast<u16_any *>(p + 2 * K - 2) = (uint16_t)bswap32(w[K / 2]);
}

// -------------------------------------------------------------------------
// Edge vectors: those with header bytes, the stream's end or the buffer's
// end.  Each is handled as a whole like the others: all of its loads are
// issued together, the bits past the stream are masked off, and only bytes of
// the buffer (and of the message) are touched.  Walking such a vector byte by
// byte waits for memory sixteen times in a row, about 2 us, which was half
// the time of a small cover's embed (512 x 512 x 3 at k = 1: 4.4 us).

// Stream bits that vector u's fields hold (0 past the stream's end).
template <int K>
__device__ __forceinline__ uint32_t vector_bits(const Span &s, uint64_t u) {
    const uint64_t first = (uint64_t)K * (s.t0 + 16 * u);
    const uint64_t left = s.bits > first ? s.bits - first : 0;
    return left < 16 * K ? (uint32_t)left : 16 * K;
}

// Bytes of vector u inside the buffer.
__device__ __forceinline__ uint32_t vector_bytes(const Span &s, uint64_t u) {
    const uint64_t left = s.n - 16 * u;
    return left < 16 ? (uint32_t)left : 16;
}

// The first m bytes at p (the rest repeat the first).
template <bool NT>
__device__ __forceinline__ u32x4 load_bytes(const uint8_t *p, uint32_t m) {
    if (m == 16) return load16<NT>(p);
    uint32_t b[16];
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) b[i] = p[i < m ? i : 0];
    u32x4 v;
#pragma unroll
    for (int d = 0; d < 4; ++d) v[d] = b[4 * d] | (b[4 * d + 1] << 8) | (b[4 * d + 2] << 16) | (b[4 * d + 3] << 24);
    return v;
}

// Store bytes [lo, hi) of NB bytes given as little-endian dwords.
template <int NB, typename V>
__device__ __forceinline__ void store_bytes(uint8_t *p, const V &v, uint32_t lo, uint32_t hi) {
#pragma unroll
    for (uint32_t i = 0; i < NB; ++i)
        if (i >= lo && i < hi) p[i] = (uint8_t)(v[i >> 2] >> (8 * (i & 3)));
}

// Keep the first nb bits of a chunk's big-endian words.
template <int K>
__device__ __forceinline__ void keep_bits(uint32_t *w, uint32_t nb) {
#pragma unroll
    for (int i = 0; i < Chunk<K>::NW; ++i) {
        const uint32_t left = nb > 32u * i ? nb - 32u * i : 0;
        w[i] = left >= 32 ? w[i] : w[i] & ~(0xFFFFFFFFu >> left);
    }
}

// Chunk words of any vector u whose m bytes hold nb > 0 stream bits.  Header
// bytes come from the header value; only the stream bytes that these fields
// need are read, the rest are zero.
template <int K>
__device__ __forceinline__ void load_chunk_edge(const Span &s, uint64_t u, uint32_t nb, uint32_t m, uint32_t *w) {
    constexpr int NB = 2 * K + 1;
    const uint64_t at = stream_byte0(s) + 2 * K * u;  // first stream byte
    const uint32_t r = (uint32_t)(((uint64_t)K * s.t0) & 7);
    const uint32_t lo = at < s.hdr_len ? s.hdr_len - (uint32_t)at : 0;
    const uint32_t hi = (r + (nb < K * m ? nb : K * m) + 7) >> 3;
    uint32_t b[NB] = {};
    if (lo < hi) {
        const uint8_t *p = s.body + (at + lo - s.hdr_len) - lo;
#pragma unroll
        for (uint32_t i = 0; i < NB; ++i) b[i] = p[i >= lo && i < hi ? i : lo];
    }
#pragma unroll
    for (uint32_t i = 0; i < NB; ++i) {
        const uint32_t h = i < 4 && i < lo ? (s.hdr >> (8 * (3 - ((uint32_t)at + i)))) & 0xFFu : 0u;
        b[i] = i < lo ? h : (i < hi ? b[i] : 0u);
    }
    uint32_t W[Chunk<K>::NW + 1];
#pragma unroll
    for (int i = 0; i <= Chunk<K>::NW; ++i) {
        W[i] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) W[i] = (W[i] << 8) | (4 * i + j < NB ? b[4 * i + j] : 0u);
    }
#pragma unroll
    for (int i = 0; i < Chunk<K>::NW; ++i) w[i] = (uint32_t)((((uint64_t)W[i] << 32 | W[i + 1]) << r) >> 32);
}

// Embed any vector u of the span and store it; an in-place span writes
// stream-carrying bytes only.  Returns the new vector, with the cover's in *c
// and the chunk in w (for the check of what was written).
template <int K, bool NT>
__device__ __forceinline__ u32x4 embed_any(const Span &s, uint64_t u, uint32_t nb, uint32_t m, u32x4 *c, uint32_t *w) {
    *c = load_bytes<NT>(s.src + 16 * u, m);
    uint32_t ones[Chunk<K>::NW];
#pragma unroll
    for (int i = 0; i < Chunk<K>::NW; ++i) {
        w[i] = 0;
        ones[i] = ~0u;
    }
    if (nb) load_chunk_edge<K>(s, u, nb, m, w);
    keep_bits<K>(ones, nb);
    const u32x4 mask = embed_vec<K>(u32x4{0u, 0u, 0u, 0u}, ones);
    const u32x4 o = (*c & ~mask) | (embed_vec<K>(*c, w) & mask);
    const uint32_t carry = (nb + K - 1) / K;
    const uint32_t hi = s.inplace && carry < m ? carry : m;
    if (hi == 16) store16<NT>(s.dst + 16 * u, o);
    else store_bytes<16>(s.dst + 16 * u, o, 0, hi);
    return o;
}

// Extract any vector u that holds stream bits; writes message bytes only.
template <int K, bool NT>
__device__ __forceinline__ void extract_any(const Span &s, uint64_t u) {
    const uint32_t nb = vector_bits<K>(s, u);
    uint32_t w[Chunk<K>::NW];
    extract_vec<K>(load_bytes<NT>(s.src + 16 * u, vector_bytes(s, u)), w);
    keep_bits<K>(w, nb);
    const uint64_t at = stream_byte0(s) + 2 * K * u;
    const uint32_t lo = at < s.hdr_len ? s.hdr_len - (uint32_t)at : 0;
    const uint32_t hi = (nb + 7) / 8;
    uint8_t *p = reinterpret_cast<uint8_t *>((uintptr_t)s.out + at - s.hdr_len);
    if (lo == 0 && hi == 2 * K) {
        store_chunk<K>(p, w);
    } else {
#pragma unroll
        for (int i = 0; i < Chunk<K>::NW; ++i) w[i] = bswap32(w[i]);
        store_bytes<2 * K>(p, w, lo, hi);
    }
}

// -------------------------------------------------------------------------
// Span walkers.  A team of `n_waves` waves (a whole grid, or one block) walks
// vectors [v_begin, v_end) of a span in groups of 64*UNR vectors; wave
// `wave` takes groups wave, wave + n_waves, ...

template <int K, int UNR, bool NT>
__device__ __forceinline__ void embed_walk(const Span &s, const Ranges &r, uint64_t v_begin,
                                           uint64_t v_end, uint64_t wave, uint64_t n_waves,
                                           uint32_t lane) {
    constexpr uint64_t G = 64 * UNR;
    const uint64_t sb = stream_byte0(s);
    const uint32_t rbit = (uint32_t)(((uint64_t)K * s.t0) & 7);
    // address of stream byte sb + 2K*u is body_base + 2K*u, valid for fast u
    const uintptr_t body_base = (uintptr_t)s.body + sb - s.hdr_len;
    for (uint64_t u0 = v_begin + wave * G; u0 < v_end; u0 += n_waves * G) {
        const uint64_t u_hi = u0 + G;
        if (u0 >= r.fast_begin && u_hi <= r.fast_end && u_hi <= v_end) {
            u32x4 c[UNR];
            uint32_t w[UNR][Chunk<K>::NW];
#pragma unroll
            for (int j = 0; j < UNR; ++j) {
                const uint64_t u = u0 + (uint64_t)j * 64 + lane;
                c[j] = load16<NT>(s.src + 16 * u);
                const uint8_t *p = reinterpret_cast<const uint8_t *>(body_base + 2 * K * u);
                if (rbit == 0) load_chunk<K>(p, w[j]);
                else load_chunk_shifted<K>(p, rbit, w[j]);
            }
#pragma unroll
            for (int j = 0; j < UNR; ++j) {
                const uint64_t u = u0 + (uint64_t)j * 64 + lane;
                store16<NT>(s.dst + 16 * u, embed_vec<K>(c[j], w[j]));
            }
        } else if (u0 >= r.copy_begin && u_hi <= r.copy_end && u_hi <= v_end) {
            if (!s.inplace) {
                u32x4 c[UNR];
#pragma unroll
                for (int j = 0; j < UNR; ++j)
                    c[j] = load16<NT>(s.src + 16 * (u0 + (uint64_t)j * 64 + lane));
#pragma unroll
                for (int j = 0; j < UNR; ++j)
                    store16<NT>(s.dst + 16 * (u0 + (uint64_t)j * 64 + lane), c[j]);
            }
        } else {
#pragma unroll 1
            for (int j = 0; j < UNR; ++j) {
                const uint64_t u = u0 + (uint64_t)j * 64 + lane;
                if (u >= v_end) continue;
                const uint32_t nb = vector_bits<K>(s, u);
                if (nb == 0 && s.inplace) continue;
                u32x4 c;
                uint32_t w[Chunk<K>::NW];
                embed_any<K, NT>(s, u, nb, vector_bytes(s, u), &c, w);
            }
        }
    }
}

// Store the stream bytes of one fast wave group whose stego vectors are in c.
// Every vector of the group is extracted before the first store.
template <int K, int UNR>
__device__ __forceinline__ void extract_store_group(const Span &s, uintptr_t out_base, uint64_t u0,
                                                    const u32x4 *c, uint32_t lane) {
    uint32_t w[UNR][Chunk<K>::NW];
#pragma unroll
    for (int j = 0; j < UNR; ++j) extract_vec<K>(c[j], w[j]);
    uint8_t *p0 = reinterpret_cast<uint8_t *>(out_base + 2 * K * (u0 + lane));
#pragma unroll
    for (int j = 0; j < UNR; ++j) store_chunk<K>(p0 + 2 * K * 64 * j, w[j]);
}

// Same for k = 1 with wavefront ballots.  The wave's 1 KiB of stego bytes
// per vector set is staged in LDS so that lane L can read bytes L, L+64, ...,
// L+960; ballot m over their LSBs then holds 64 consecutive stream bits
// (bit L = stream bit 64m + L), i.e. 8 output bytes, which a per-byte bit
// reversal puts in MSB-first order.  Lanes 0..15 store the 16 ballots.
// `stage` is this wave's 1 KiB of LDS.  Must be called by all 64 lanes.
template <int UNR>
__device__ __forceinline__ void extract_store_group_ballot(const Span &s, uintptr_t out_base, uint64_t u0,
                                                           const u32x4 *c, uint32_t lane, uint8_t *stage) {
#pragma unroll
    for (int j = 0; j < UNR; ++j) {
        *reinterpret_cast<u32x4 *>(stage + 16 * lane) = c[j];
        uint32_t bits = 0;
#pragma unroll
        for (int m = 0; m < 16; ++m) bits |= ((uint32_t)stage[lane + 64 * m] & 1u) << m;
        uint64_t mine = 0;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const uint64_t mask = __ballot((bits >> m) & 1u);
            mine = lane == (uint32_t)m ? mask : mine;
        }
        if (lane < 16) {
            const uint64_t v = __builtin_bswap64(__builtin_bitreverse64(mine));
            uint8_t *p = reinterpret_cast<uint8_t *>(out_base + 2 * (u0 + (uint64_t)j * 64) + 8 * lane);
            reinterpret_cast<u32_any *>(p)[0] = (uint32_t)v;
            reinterpret_cast<u32_any *>(p)[1] = (uint32_t)(v >> 32);
        }
    }
}

__host__ __device__ inline uintptr_t extract_out_base(const Span &s) {
    return (uintptr_t)s.out + stream_byte0(s) - s.hdr_len;
}

// BALLOT (k = 1 only): pack fast groups with wavefront ballots through the
// wave's 1 KiB LDS `stage` instead of per-lane multiplies.
template <int K, int UNR, bool NT, bool BALLOT = false>
__device__ __forceinline__ void extract_walk(const Span &s, const Ranges &r, uint64_t v_begin,
                                             uint64_t v_end, uint64_t wave, uint64_t n_waves,
                                             uint32_t lane, uint8_t *stage = nullptr) {
    constexpr uint64_t G = 64 * UNR;
    const uintptr_t out_base = extract_out_base(s);
    for (uint64_t u0 = v_begin + wave * G; u0 < v_end; u0 += n_waves * G) {
        const uint64_t u_hi = u0 + G;
        if (u0 >= r.fast_begin && u_hi <= r.fast_end && u_hi <= v_end) {
            u32x4 c[UNR];
#pragma unroll
            for (int j = 0; j < UNR; ++j)
                c[j] = load16<NT>(s.src + 16 * (u0 + (uint64_t)j * 64 + lane));
            if constexpr (BALLOT && K == 1)
                extract_store_group_ballot<UNR>(s, out_base, u0, c, lane, stage);
            else
                extract_store_group<K, UNR>(s, out_base, u0, c, lane);
        } else {
#pragma unroll 1
            for (int j = 0; j < UNR; ++j) {
                const uint64_t u = u0 + (uint64_t)j * 64 + lane;
                if (u < v_end) extract_any<K, NT>(s, u);
            }
        }
    }
}

// Decode the 32-bit length header from the first ceil(32/k) stego bytes with
// one ballot: lane j (< 32) reads stream bit j, the ballot's low 32 bits are
// the header bits in reverse order.  Caller guarantees n*k >= 32.
__device__ __forceinline__ uint32_t decode_header(const uint8_t *stego, int k, uint32_t lane) {
    uint32_t bit = 0;
    if (lane < 32) {
        const uint32_t t = lane / (uint32_t)k, q = lane % (uint32_t)k;
        bit = (stego[t] >> ((uint32_t)k - 1 - q)) & 1u;
    }
    const uint64_t m = __ballot(bit);
    return __builtin_bitreverse32((uint32_t)m);
}

// Block order of the embed and extract kernels (launch configuration field
// `order`; Span.block_order).  Workgroups go to the eight XCDs in turn, so
// neighbouring blocks sit on different XCDs (each with its own L2), and a
// line that two neighbours share is moved by both: the embed's
// stream bytes straddle a line at each end of a block (the 4-byte header sits
// in front of the message), and an extract block's 2k-byte outputs end
// inside a line.  Logical blocks are therefore handed out in runs of 16 per
// XCD (physical block b on XCD b % 8 takes logical block
// 128 (s / 16) + 16 x + s % 16, s = b / 8): the neighbours inside a run share
// an L2, and the XCDs still interleave at 16-block granularity (handing each
// XCD one contiguous eighth removed the shared lines too, but made every
// XCD stream its own distant region and slowed the grid-stride launches).
// Blocks past the last whole round of 128 keep their index.  (The batched
// kernel takes longer runs, kRun.)
template <uint32_t kRun = 16>
__device__ __forceinline__ uint32_t xcd_run_block(uint32_t b, uint32_t grid) {
    constexpr uint32_t kXcds = 8, kRound = kXcds * kRun;
    if (b >= grid / kRound * kRound) return b;
    const uint32_t x = b % kXcds, slot = b / kXcds;
    return (slot / kRun) * kRound + x * kRun + slot % kRun;
}

// floor(n*k/8) without overflow.
__host__ __device__ inline uint64_t room_bytes(uint64_t n, int k) {
    return (n / 8) * (uint64_t)k + ((n % 8) * (uint64_t)k) / 8;
}

}  // namespace lsb
