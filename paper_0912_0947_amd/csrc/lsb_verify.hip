// lsb_verify.hip -- round-trip checks of a stego buffer in one launch
// (arXiv:0912.0947: embedding is Section VI step 7, extraction Section VII
// step 6; extraction reverses embedding).
//
// A stego byte t is right when
//   - the bits of its field that carry stream bits, read back as extraction
//     reads them (mask the field, shift it down), equal those stream bits, and
//   - every other bit (above the field; the low bits of a partial last field;
//     all bits of a byte past the stream) equals the cover's.
// Both checks go through the extraction side of the method (extract_vec),
// never through the embedding arithmetic, so an embedding mistake shows up as
// a mismatch.
//
// lsb_verify reads cover, stego and stream once (2n + |S| bytes) and counts
// wrong stego bytes.  lsb_embed_verify embeds (as lsb_embed) and, in the same
// launch, checks every byte it writes in this way: the round trip of each
// vector happens in registers, so the check costs no memory traffic beyond
// the embed's own 2n + |S| bytes.
#include <hip/hip_ext.h>

#include "lsb_host.hpp"

namespace lsb {

// Wrong bytes of a fast vector (all 16 fields carry K stream bits): extract
// the stego vector's fields into stream words, compare them with the stream
// chunk w, and compare the bits above the fields with the cover's.  Whole
// words first: when every word reads back and no kept bit changed (a
// correct embedding) the vector costs a few compares; only a vector with a
// difference is counted field by field and byte by byte.
template <int K>
__device__ __forceinline__ uint32_t vec_wrong(u32x4 c, u32x4 g, const uint32_t *w) {
    uint32_t got[Chunk<K>::NW];
    extract_vec<K>(g, got);
    uint32_t diff[Chunk<K>::NW];
    uint32_t any = 0;
#pragma unroll
    for (int i = 0; i < Chunk<K>::NW; ++i) {
        diff[i] = got[i] ^ w[i];
        any |= diff[i];
    }
    if constexpr (K < 8) {
        constexpr uint32_t keep_bits = ~(((1u << K) - 1u) * 0x01010101u);
#pragma unroll
        for (int d = 0; d < 4; ++d) any |= (c[d] ^ g[d]) & keep_bits;
    }
    if (!any) return 0;
    uint32_t bad = 0;  // bit f: byte f of the vector is wrong
#pragma unroll
    for (int f = 0; f < 16; ++f) bad |= (get_field<K>(diff, f) != 0 ? 1u : 0u) << f;
    if constexpr (K < 8) {
        constexpr uint32_t keep = ~(((1u << K) - 1u) * 0x01010101u);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t x = (c[d] ^ g[d]) & keep;
#pragma unroll
            for (int j = 0; j < 4; ++j) bad |= (((x >> (8 * j)) & 0xFFu) != 0 ? 1u : 0u) << (4 * d + j);
        }
    }
    return (uint32_t)__builtin_popcount(bad);
}

__device__ __forceinline__ uint32_t bytes_differ(u32x4 a, u32x4 b) {
    uint32_t n = 0;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t x = a[d] ^ b[d];
#pragma unroll
        for (int j = 0; j < 4; ++j) n += ((x >> (8 * j)) & 0xFFu) != 0;
    }
    return n;
}

// Wrong bytes of any vector whose first m bytes are in the buffer and whose
// fields hold nb stream bits, the chunk w: a field's stream bits are read back
// through extraction, every other bit of its byte is compared with the cover.
template <int K>
__device__ __forceinline__ uint32_t any_wrong(u32x4 c, u32x4 g, uint32_t *w, uint32_t nb, uint32_t m) {
    uint32_t diff[Chunk<K>::NW];
    extract_vec<K>(g, diff);
#pragma unroll
    for (int i = 0; i < Chunk<K>::NW; ++i) diff[i] ^= w[i];
    keep_bits<K>(diff, nb);
    uint32_t bad = 0;
#pragma unroll
    for (uint32_t f = 0; f < 16; ++f) {
        const uint32_t left = nb > K * f ? nb - K * f : 0;
        const uint32_t vb = left < K ? left : K;  // the field's stream bits, its highest
        const uint32_t mask = ((1u << vb) - 1u) << (K - vb);
        const uint32_t kept = ((c[f >> 2] ^ g[f >> 2]) >> (8 * (f & 3))) & 0xFFu & ~mask;
        bad += f < m && (get_field<K>(diff, (int)f) | kept) != 0;
    }
    return bad;
}

// Sum `bad` over the block (256 threads) and add it to the counter.
__device__ __forceinline__ void add_block_count(uint32_t bad, unsigned long long *mismatches) {
    for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off);
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63u) == 0) part[threadIdx.x >> 6] = bad;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t sum = part[0] + part[1] + part[2] + part[3];
        if (sum) atomicAdd(mismatches, (unsigned long long)sum);
    }
}

// Check only: s.src = cover, s.dst = stego (read only here).  One vector u
// of the span (any class).
template <int K, bool NT>
__device__ __forceinline__ uint32_t verify_one(const Span &s, const Ranges &r, uintptr_t body_base, uint64_t u) {
    if (u >= r.fast_begin && u < r.fast_end) {
        uint32_t w[Chunk<K>::NW];
        const uint8_t *p = reinterpret_cast<const uint8_t *>(body_base + 2 * K * u);
        load_chunk<K>(p, w);
        return vec_wrong<K>(load16<NT>(s.src + 16 * u), load16<NT>(s.dst + 16 * u), w);
    }
    if (u >= r.copy_begin && u < r.copy_end)
        return bytes_differ(load16<NT>(s.src + 16 * u), load16<NT>(s.dst + 16 * u));
    const uint32_t nb = vector_bits<K>(s, u), m = vector_bytes(s, u);
    uint32_t w[Chunk<K>::NW] = {};
    if (nb) load_chunk_edge<K>(s, u, nb, m, w);
    return any_wrong<K>(load_bytes<NT>(s.src + 16 * u, m), load_bytes<NT>(s.dst + 16 * u, m), w, nb, m);
}

// A block covers 512 vectors per pass, two per thread (vectors v and v + 256
// of the pass), as in the embedding form below.
template <int K, bool NT>
__global__ void __launch_bounds__(256) lsb_verify_kernel(Span s, unsigned long long *mismatches) {
    const Ranges r = embed_ranges<K>(s);  // inplace = 0: every vector is visited
    const uint64_t stride = (uint64_t)gridDim.x * 512;
    const uintptr_t body_base = (uintptr_t)s.body - s.hdr_len;
    uint32_t bad = 0;
    for (uint64_t u0 = (uint64_t)xcd_run_block(blockIdx.x, gridDim.x) * 512 + threadIdx.x; u0 < r.count; u0 += stride) {
        const uint64_t u1 = u0 + 256;
        if (u0 >= r.fast_begin && u1 < r.fast_end) {
            uint32_t w0[Chunk<K>::NW], w1[Chunk<K>::NW];
            const uint8_t *p0 = reinterpret_cast<const uint8_t *>(body_base + 2 * K * u0);
            const uint8_t *p1 = reinterpret_cast<const uint8_t *>(body_base + 2 * K * u1);
            load_chunk<K>(p0, w0);
            load_chunk<K>(p1, w1);
            const u32x4 c0 = load16<NT>(s.src + 16 * u0), g0 = load16<NT>(s.dst + 16 * u0);
            const u32x4 c1 = load16<NT>(s.src + 16 * u1), g1 = load16<NT>(s.dst + 16 * u1);
            bad += vec_wrong<K>(c0, g0, w0) + vec_wrong<K>(c1, g1, w1);
        } else {
            bad += verify_one<K, NT>(s, r, body_base, u0);
            if (u1 < r.count) bad += verify_one<K, NT>(s, r, body_base, u1);
        }
    }
    add_block_count(bad, mismatches);
}

// Embed and check one vector u of the span (any class).  A fast vector is
// embedded in registers, stored, and its stored value is checked against
// the stream through extraction; an edge vector likewise, masked.
template <int K, bool NT>
__device__ __forceinline__ uint32_t embed_verify_one(const Span &s, const Ranges &r, uintptr_t body_base,
                                                     uint64_t u) {
    if (u >= r.fast_begin && u < r.fast_end) {
        uint32_t w[Chunk<K>::NW];
        const uint8_t *p = reinterpret_cast<const uint8_t *>(body_base + 2 * K * u);
        load_chunk<K>(p, w);
        const u32x4 c = load16<NT>(s.src + 16 * u);
        const u32x4 g = embed_vec<K>(c, w);
        store16<NT>(s.dst + 16 * u, g);
        return vec_wrong<K>(c, g, w);
    }
    if (u >= r.copy_begin && u < r.copy_end) {
        if (!s.inplace) store16<NT>(s.dst + 16 * u, load16<NT>(s.src + 16 * u));
        return 0;
    }
    const uint32_t nb = vector_bits<K>(s, u), m = vector_bytes(s, u);
    if (nb == 0 && s.inplace) return 0;
    u32x4 c;
    uint32_t w[Chunk<K>::NW];
    const u32x4 g = embed_any<K, NT>(s, u, nb, m, &c, w);
    return any_wrong<K>(c, g, w, nb, m);
}

// Embed and check in one launch: s.src = cover, s.dst = stego (may equal
// cover).  A block covers 512 vectors per pass, two per thread (vectors v
// and v + 256 of the pass, so each load instruction of a wave stays
// contiguous); when both are fast their loads are issued before either is
// embedded.
template <int K, bool NT>
__global__ void __launch_bounds__(256) lsb_embed_verify_kernel(Span s, unsigned long long *mismatches) {
    const Ranges r = embed_ranges<K>(s);
    const uint64_t stride = (uint64_t)gridDim.x * 512;
    const uintptr_t body_base = (uintptr_t)s.body - s.hdr_len;
    uint32_t bad = 0;
    for (uint64_t u0 = (uint64_t)xcd_run_block(blockIdx.x, gridDim.x) * 512 + threadIdx.x; u0 < r.count; u0 += stride) {
        const uint64_t u1 = u0 + 256;
        if (u0 >= r.fast_begin && u1 < r.fast_end) {
            uint32_t w0[Chunk<K>::NW], w1[Chunk<K>::NW];
            const uint8_t *p0 = reinterpret_cast<const uint8_t *>(body_base + 2 * K * u0);
            const uint8_t *p1 = reinterpret_cast<const uint8_t *>(body_base + 2 * K * u1);
            load_chunk<K>(p0, w0);
            load_chunk<K>(p1, w1);
            const u32x4 c0 = load16<NT>(s.src + 16 * u0);
            const u32x4 c1 = load16<NT>(s.src + 16 * u1);
            const u32x4 g0 = embed_vec<K>(c0, w0);
            const u32x4 g1 = embed_vec<K>(c1, w1);
            store16<NT>(s.dst + 16 * u0, g0);
            store16<NT>(s.dst + 16 * u1, g1);
            bad += vec_wrong<K>(c0, g0, w0) + vec_wrong<K>(c1, g1, w1);
        } else {
            bad += embed_verify_one<K, NT>(s, r, body_base, u0);
            if (u1 < r.count) bad += embed_verify_one<K, NT>(s, r, body_base, u1);
        }
    }
    add_block_count(bad, mismatches);
}

// The counter is cleared by a kernel (not a memset node), so that the call
// can sit in a captured graph.
__global__ void lsb_verify_zero_kernel(unsigned long long *p) { *p = 0; }

typedef void (*VerifyFn)(Span, unsigned long long *);

// [embed][streaming accesses]
template <int K>
struct VerifyTable {
    static constexpr VerifyFn fn[2][2] = {{lsb_verify_kernel<K, false>, lsb_verify_kernel<K, true>},
                                          {lsb_embed_verify_kernel<K, false>, lsb_embed_verify_kernel<K, true>}};
};

static VerifyFn verify_fn(int k, bool embed, bool nt) {
    switch (k) {
        case 1: return VerifyTable<1>::fn[embed][nt];
        case 2: return VerifyTable<2>::fn[embed][nt];
        case 3: return VerifyTable<3>::fn[embed][nt];
        case 4: return VerifyTable<4>::fn[embed][nt];
        case 5: return VerifyTable<5>::fn[embed][nt];
        case 6: return VerifyTable<6>::fn[embed][nt];
        case 7: return VerifyTable<7>::fn[embed][nt];
        default: return VerifyTable<8>::fn[embed][nt];
    }
}

// Shared argument checks and launch of both entry points.
static int verify_call(const char *name, bool embed, const uint8_t *cover, uint8_t *stego, uint64_t n,
                       const uint8_t *msg, uint32_t len, int k, uint64_t *mismatches_dev, void *stream) {
    if (k < 1 || k > 8) return fail(LSB_E_ARG, "%s: k=%d outside 1..8", name, k);
    const int64_t cap = lsb_capacity(n, k);
    if (cap < 0) return (int)cap;
    if ((uint64_t)len > (uint64_t)cap)
        return fail(LSB_E_CAPACITY, "%s: message of %u bytes exceeds capacity %lld", name, len, (long long)cap);
    if (!cover || !stego || !mismatches_dev) return fail(LSB_E_ARG, "%s: null pointer", name);
    if (len && !msg) return fail(LSB_E_ARG, "%s: null msg", name);
    if (overlaps(mismatches_dev, 8, cover, n) || overlaps(mismatches_dev, 8, stego, n) ||
        overlaps(mismatches_dev, 8, msg, len))
        return fail(LSB_E_ARG, "%s: counter overlaps a buffer", name);
    if (embed) {
        if (cover != stego && overlaps(cover, n, stego, n))
            return fail(LSB_E_ARG, "%s: cover and stego overlap (only stego == cover is allowed)", name);
        if (overlaps(msg, len, stego, n)) return fail(LSB_E_ARG, "%s: msg overlaps stego", name);
    }
    Span s{};
    s.src = cover;
    s.dst = stego;
    s.body = msg;
    s.n = n;
    s.bits = 8 * (4 + (uint64_t)len);
    s.hdr = len;
    s.hdr_len = 4;
    s.k = k;
    s.inplace = embed && cover == stego;
    hipStream_t st = (hipStream_t)stream;
    unsigned long long *cnt = (unsigned long long *)mismatches_dev;
    hipLaunchKernelGGL(lsb_verify_zero_kernel, dim3(1), dim3(1), 0, st, cnt);
    uint64_t items = ceil_div(n, 16);
    if (s.inplace) items = embed_ranges(s).count;  // in place: bytes past the stream stay untouched
    // The kernels' blocks cover 512 vectors per pass, and the grid
    // gives every pair of vectors a thread: on a grid capped at 8 blocks
    // per CU the waves loop, and a looping wave's wait for its next loads
    // also waits for its previous stores (one counter covers both).  The
    // capped grid measured slower for the check alone too.  A correct
    // embedding adds nothing to the counter, so the larger grid costs no
    // atomics.
    uint64_t blocks = ceil_div(items ? items : 1, 512);
    if (blocks > (uint64_t)INT32_MAX) blocks = (uint64_t)INT32_MAX;
    // Streaming accesses from 128 MB on, where cover and stego no longer stay
    // in the caches for the call that reads them next (checked embed, verify
    // and squared error in turn: 36 MB 44.1 us cached, 45.9 streaming; 201 MB
    // 222 against 196 us).
    VerifyFn fn = verify_fn(k, embed, access_kind(n) == STREAM);
    hipEvent_t e0, e1;
    take_launch_events(&e0, &e1);
    hipExtLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(256), 0, st, e0, e1, 0, s, cnt);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? LSB_OK : hip_fail(e, "verify kernel launch");
}

}  // namespace lsb

using namespace lsb;

extern "C" int lsb_verify(const uint8_t *cover, const uint8_t *stego, uint64_t n, const uint8_t *msg, uint32_t len,
                          int k, uint64_t *mismatches_dev, void *stream) {
    const TimedCall timed_call;
    return verify_call("lsb_verify", false, cover, const_cast<uint8_t *>(stego), n, msg, len, k, mismatches_dev,
                       stream);
}

extern "C" int lsb_embed_verify(const uint8_t *cover, uint8_t *stego, uint64_t n, const uint8_t *msg, uint32_t len,
                                int k, uint64_t *mismatches_dev, void *stream) {
    const TimedCall timed_call;
    return verify_call("lsb_embed_verify", true, cover, stego, n, msg, len, k, mismatches_dev, stream);
}
