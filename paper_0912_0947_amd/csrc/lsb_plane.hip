// lsb_plane.hip -- one colour plane with the general method, and the squared
// error behind the paper's PSNR figures (arXiv:0912.0947).
//
// Section VI step 2 / Section VII step 2 separate one plane of the image
// before embedding.  Here the fields are the bytes of plane `plane` of an
// HWC image (byte p*c + plane for pixel p), in raster order; the stream, bit
// order, header and partial last field are those of lsb_embed.  Images of up
// to 4 channels take one pass over their vectors; others (and misaligned ones in
// place) a vector copy (out of place), then a strided kernel over the plane bytes
// that carry stream bits.
//
// Section VIII reports PSNR = 10*log10(255^2 / MSE).  lsb_sse sums the
// squared byte differences of two buffers on the device (16 bytes per lane,
// block reduction, one 64-bit atomic per block).
#include <hip/hip_ext.h>

#include <algorithm>

#include "lsb_host.hpp"

#include "lsb_plane_device.hpp"

namespace lsb {

__global__ void lsb_zero_u64_kernel(uint64_t *p) { *p = 0; }

// Sum of squared differences of four byte pairs, a.a + b.b - 2 a.b in three
// dot products (each at most 4 * 255^2).
__device__ __forceinline__ uint32_t sq_diff4(uint32_t a, uint32_t b, uint32_t acc) {
    acc = __builtin_amdgcn_udot4(a, a, acc, false);
    acc = __builtin_amdgcn_udot4(b, b, acc, false);
    return acc - 2 * __builtin_amdgcn_udot4(a, b, 0u, false);
}

__device__ __forceinline__ uint32_t sq_diff16(u32x4 x, u32x4 y, uint32_t acc) {
#pragma unroll
    for (int d = 0; d < 4; ++d) acc = sq_diff4(x[d], y[d], acc);
    return acc;
}

// Sum of squared byte differences; one 64-bit atomic per block.  The atomics
// on the one result word run one after the other, about 10 ns each, so the
// grid is one block per CU; a block covers kSseUnroll * kSseBlock vectors of
// both buffers per pass, all of a thread's loads issued before any is used.
// Nothing is stored, so the passes do not wait for each other.  Against 1024
// blocks of 256 threads with one pair in flight: 2 x 6.2 MB 14.6 -> 5.7 us, 2
// x 36 MB 22.6 -> 14.1 us, 2 x 201 MB 65.0 -> 60.3 us (6.7 TB/s); 256 blocks
// of 1024 threads 5.8 / 15.7 / 61.4 us, 512 blocks of 512 5.7 / 16.3 / 61.6 us.
constexpr int kSseUnroll = 4, kSseBlocksPerCu = 1, kSseBlock = 512;
template <bool NT>
__global__ void __launch_bounds__(kSseBlock) lsb_sse_kernel(const uint8_t *a, const uint8_t *b, uint64_t n,
                                                     unsigned long long *out) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t acc = 0;
    const uint64_t nv = n / 16;
    for (uint64_t u0 = (uint64_t)blockIdx.x * (kSseBlock * kSseUnroll) + threadIdx.x; u0 < nv; u0 += stride * kSseUnroll) {
        uint32_t sum = 0;
        if (u0 + kSseBlock * (kSseUnroll - 1) < nv) {
            u32x4 x[kSseUnroll], y[kSseUnroll];
#pragma unroll
            for (int j = 0; j < kSseUnroll; ++j) {
                x[j] = load16<NT>(a + 16 * (u0 + kSseBlock * j));
                y[j] = load16<NT>(b + 16 * (u0 + kSseBlock * j));
            }
#pragma unroll
            for (int j = 0; j < kSseUnroll; ++j) sum = sq_diff16(x[j], y[j], sum);
        } else {
            for (uint64_t u = u0; u < nv && u < u0 + kSseBlock * kSseUnroll; u += kSseBlock)
                sum = sq_diff16(load16<NT>(a + 16 * u), load16<NT>(b + 16 * u), sum);
        }
        acc += sum;
    }
    for (uint64_t t = 16 * nv + gid; t < n; t += stride) {
        const int d = (int)a[t] - (int)b[t];
        acc += (uint64_t)(d * d);
    }
    // wave reduction of the 64-bit partial sums, then across the block's
    // waves in LDS, then one atomic per block
    uint32_t lo = (uint32_t)acc, hi = (uint32_t)(acc >> 32);
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t olo = __shfl_xor(lo, off), ohi = __shfl_xor(hi, off);
        const uint64_t sum = ((uint64_t)hi << 32 | lo) + ((uint64_t)ohi << 32 | olo);
        lo = (uint32_t)sum;
        hi = (uint32_t)(sum >> 32);
    }
    __shared__ unsigned long long part[kSseBlock / 64];
    if ((threadIdx.x & 63u) == 0) part[threadIdx.x >> 6] = (unsigned long long)hi << 32 | lo;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long sum = 0;
        for (int i = 0; i < kSseBlock / 64; ++i) sum += part[i];
        atomicAdd(out, sum);
    }
}

typedef void (*PlaneEmbedFn)(Span, uint32_t, uint64_t, uint64_t);
typedef void (*PlaneExtractFn)(Span, uint32_t, uint64_t, uint32_t *, int32_t *);

// [access kind or streaming loads][channels - 2]
template <int K>
struct PlaneTable {
    static constexpr PlaneEmbedFn embed[3][3] = {
        {lsb_plane_embed_vec_kernel<K, 2, CACHED>, lsb_plane_embed_vec_kernel<K, 3, CACHED>,
         lsb_plane_embed_vec_kernel<K, 4, CACHED>},
        {lsb_plane_embed_vec_kernel<K, 2, STREAM_LOADS>, lsb_plane_embed_vec_kernel<K, 3, STREAM_LOADS>,
         lsb_plane_embed_vec_kernel<K, 4, STREAM_LOADS>},
        {lsb_plane_embed_vec_kernel<K, 2, STREAM>, lsb_plane_embed_vec_kernel<K, 3, STREAM>,
         lsb_plane_embed_vec_kernel<K, 4, STREAM>}};
    static constexpr PlaneExtractFn extract[2][3] = {
        {lsb_plane_extract_vec_kernel<K, 2, false>, lsb_plane_extract_vec_kernel<K, 3, false>,
         lsb_plane_extract_vec_kernel<K, 4, false>},
        {lsb_plane_extract_vec_kernel<K, 2, true>, lsb_plane_extract_vec_kernel<K, 3, true>,
         lsb_plane_extract_vec_kernel<K, 4, true>}};
};

static PlaneEmbedFn plane_embed_fn(int k, uint32_t c, Access a) {
    const int ci = (int)c - 2;
    switch (k) {
        case 1: return PlaneTable<1>::embed[a][ci];
        case 2: return PlaneTable<2>::embed[a][ci];
        case 3: return PlaneTable<3>::embed[a][ci];
        case 4: return PlaneTable<4>::embed[a][ci];
        case 5: return PlaneTable<5>::embed[a][ci];
        case 6: return PlaneTable<6>::embed[a][ci];
        case 7: return PlaneTable<7>::embed[a][ci];
        default: return PlaneTable<8>::embed[a][ci];
    }
}

static PlaneExtractFn plane_extract_fn(int k, uint32_t c, bool nt) {
    const int ci = (int)c - 2;
    switch (k) {
        case 1: return PlaneTable<1>::extract[nt][ci];
        case 2: return PlaneTable<2>::extract[nt][ci];
        case 3: return PlaneTable<3>::extract[nt][ci];
        case 4: return PlaneTable<4>::extract[nt][ci];
        case 5: return PlaneTable<5>::extract[nt][ci];
        case 6: return PlaneTable<6>::extract[nt][ci];
        case 7: return PlaneTable<7>::extract[nt][ci];
        default: return PlaneTable<8>::extract[nt][ci];
    }
}

// Grid of the strided and extract kernels: a thread per item.  They are
// grid-stride loops, and a looping wave's wait for its next loads also waits
// for its previous stores; capped at 16 blocks per CU, the extract of an
// 8192x8192x3 image took 37.8-38.2 us against 37.3-37.6 us uncapped.
static unsigned grid_cap(uint64_t items) {
    const uint64_t blocks = ceil_div(items ? items : 1, 256);
    return (unsigned)(blocks < (uint64_t)INT32_MAX ? blocks : (uint64_t)INT32_MAX);
}

}  // namespace lsb

using namespace lsb;

extern "C" {

int lsb_embed_plane(const uint8_t *cover, uint8_t *stego, uint64_t pixels, uint32_t c, uint32_t plane,
                    const uint8_t *msg, uint32_t len, int k, void *stream) {
    const TimedCall timed_call;
    if (k < 1 || k > 8) return fail(LSB_E_ARG, "lsb_embed_plane: k=%d outside 1..8", k);
    if (c == 0 || plane >= c) return fail(LSB_E_ARG, "lsb_embed_plane: plane %u outside 0..%u", plane, c ? c - 1 : 0);
    if (pixels > (1ull << 48) || c > 65536) return fail(LSB_E_ARG, "lsb_embed_plane: pixels or channels out of range");
    const int64_t cap = lsb_capacity(pixels, k);
    if (cap < 0) return (int)cap;
    if ((uint64_t)len > (uint64_t)cap)
        return fail(LSB_E_CAPACITY, "lsb_embed_plane: message of %u bytes exceeds capacity %lld", len, (long long)cap);
    const uint64_t n = pixels * c;
    if (!cover || !stego) return fail(LSB_E_ARG, "lsb_embed_plane: null cover/stego");
    if (len && !msg) return fail(LSB_E_ARG, "lsb_embed_plane: null msg");
    if (cover != stego && overlaps(cover, n, stego, n))
        return fail(LSB_E_ARG, "lsb_embed_plane: cover and stego overlap (only stego == cover is allowed)");
    if (overlaps(msg, len, stego, n)) return fail(LSB_E_ARG, "lsb_embed_plane: msg overlaps stego");
    hipStream_t st = (hipStream_t)stream;
    if (c == 1) return lsb_embed(cover, stego, pixels, msg, len, k, stream);  // the plane is the image
    // The vector kernel rewrites whole vectors, other planes' bytes with what it
    // read.  In place on an image off a 16-byte boundary, as the pixels behind a
    // file header are, the strided kernel writes plane bytes only, so that streams
    // may embed the planes of one image at once (36 MB at byte 54: 30 us against
    // 15; whole vectors with byte stores 24, and 23 against 12 where aligned).
    const bool plane_bytes_only = cover == stego && ((uintptr_t)stego & 15u) != 0;
    if (c <= 4 && !plane_bytes_only) {
        // one pass over the image's vectors
        Span s{};
        s.src = cover;
        s.dst = stego;
        s.body = msg;
        s.n = pixels;
        s.bits = 8 * (4 + (uint64_t)len);
        s.hdr = len;
        s.hdr_len = 4;
        s.k = k;
        s.inplace = cover == stego;
        // in place: up to the last vector that carries stream bits
        const uint64_t fields = ceil_div(s.bits, (uint64_t)k);
        const uint64_t count = ceil_div(s.inplace && fields < pixels ? fields * c : n, 16);
        const uint64_t blocks = std::min<uint64_t>(ceil_div(count, 512), 0xFFFFFFFFull / 256);
        hipEvent_t e0, e1;
        take_launch_events(&e0, &e1);
        hipExtLaunchKernelGGL(plane_embed_fn(k, c, access_kind(n)), dim3((unsigned)blocks), dim3(256), 0, st, e0, e1,
                              0, s, plane, n, count);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? LSB_OK : hip_fail(e, "plane embed kernel launch");
    }
    // others: copy, then rewrite the plane bytes
    if (cover != stego)
        hipLaunchKernelGGL(lsb_copy_kernel, dim3(grid_cap(n / 16)), dim3(256), 0, st, cover, stego, n);
    Span s{};
    s.src = stego;  // after the copy the plane bytes are read back from stego
    s.dst = stego;
    s.body = msg;
    s.n = pixels;
    s.bits = 8 * (4 + (uint64_t)len);
    s.hdr = len;
    s.hdr_len = 4;
    s.k = k;
    const uint64_t fields = ceil_div(s.bits, (uint64_t)k);
    hipEvent_t e0, e1;
    take_launch_events(&e0, &e1);
    hipExtLaunchKernelGGL(lsb_plane_embed_kernel, dim3(grid_cap(fields)), dim3(256), 0, st, e0, e1, 0, s, fields, c,
                          plane);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? LSB_OK : hip_fail(e, "plane embed kernel launch");
}

int lsb_extract_plane(const uint8_t *stego, uint64_t pixels, uint32_t c, uint32_t plane, int k, uint8_t *msg_out,
                      uint64_t out_cap, uint32_t *len_out_dev, int32_t *status_out_dev, void *stream) {
    const TimedCall timed_call;
    if (k < 1 || k > 8) return fail(LSB_E_ARG, "lsb_extract_plane: k=%d outside 1..8", k);
    if (c == 0 || plane >= c) return fail(LSB_E_ARG, "lsb_extract_plane: plane %u outside 0..%u", plane, c ? c - 1 : 0);
    if (!len_out_dev || !status_out_dev) return fail(LSB_E_ARG, "lsb_extract_plane: null len/status pointer");
    if (pixels && !stego) return fail(LSB_E_ARG, "lsb_extract_plane: null stego");
    if (out_cap && !msg_out) return fail(LSB_E_ARG, "lsb_extract_plane: null msg_out with out_cap > 0");
    if (pixels > (1ull << 48) || c > 65536)
        return fail(LSB_E_ARG, "lsb_extract_plane: pixels or channels out of range");
    const uint64_t n = pixels * c;
    const uint64_t room = room_bytes(pixels, k);
    const uint64_t cap = room >= 4 ? room - 4 : 0;
    const uint64_t max_len = out_cap < cap ? out_cap : cap;
    if (overlaps(msg_out, max_len, stego, n)) return fail(LSB_E_ARG, "lsb_extract_plane: msg_out overlaps stego");
    if (overlaps(len_out_dev, 4, stego, n) || overlaps(status_out_dev, 4, stego, n) ||
        overlaps(len_out_dev, 4, msg_out, max_len) || overlaps(status_out_dev, 4, msg_out, max_len))
        return fail(LSB_E_ARG, "lsb_extract_plane: len/status overlap a data buffer");
    if (c == 1) return lsb_extract(stego, pixels, k, msg_out, out_cap, len_out_dev, status_out_dev, stream);
    Span s{};
    s.src = stego;
    s.out = msg_out;
    s.n = pixels;
    s.hdr_len = 4;
    s.k = k;
    hipEvent_t e0, e1;
    take_launch_events(&e0, &e1);
    if (c <= 4) {
        uint64_t vectors = 0;  // bound on the vectors a decodable stream can need
        if ((uint64_t)k * pixels >= 32) {
            const uint64_t v_stream = ceil_div(4 + max_len, 2 * (uint64_t)k);
            const uint64_t v_buf = ceil_div(pixels, 16);
            vectors = v_stream < v_buf ? v_stream : v_buf;
        }
        hipExtLaunchKernelGGL(plane_extract_fn(k, c, access_kind(n) != CACHED), dim3(grid_cap(vectors)), dim3(256), 0,
                              (hipStream_t)stream, e0, e1, 0, s, plane, out_cap, len_out_dev, status_out_dev);
    } else {
        hipExtLaunchKernelGGL(lsb_plane_extract_kernel, dim3(grid_cap(max_len)), dim3(256), 0, (hipStream_t)stream,
                              e0, e1, 0, s, c, plane, out_cap, len_out_dev, status_out_dev);
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? LSB_OK : hip_fail(e, "plane extract kernel launch");
}

int lsb_sse(const uint8_t *a, const uint8_t *b, uint64_t n, uint64_t *sse_dev, void *stream) {
    const TimedCall timed_call;
    if (!sse_dev) return fail(LSB_E_ARG, "lsb_sse: null result pointer");
    if (n && (!a || !b)) return fail(LSB_E_ARG, "lsb_sse: null buffer");
    if (overlaps(sse_dev, 8, a, n) || overlaps(sse_dev, 8, b, n))
        return fail(LSB_E_ARG, "lsb_sse: result overlaps an input");
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(lsb_zero_u64_kernel, dim3(1), dim3(1), 0, st, sse_dev);
    hipEvent_t e0, e1;
    take_launch_events(&e0, &e1);
    uint64_t blocks = ceil_div(n / 16 + 1, kSseBlock * kSseUnroll);
    const uint64_t cap = (uint64_t)device_cus() * kSseBlocksPerCu;
    if (blocks > cap) blocks = cap;
    // cached loads while the buffers may still be in the caches (a checked embed,
    // verify and squared error in turn, cached / streaming: 36 MB 42.9 / 44.4 us;
    // images that are new each time 42 MB 49.5 / 48.5, 60 MB 64.0 / 63.5)
    const auto fn = access_kind(n) == CACHED ? lsb_sse_kernel<false> : lsb_sse_kernel<true>;
    hipExtLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(kSseBlock), 0, st, e0, e1, 0, a, b, n,
                          (unsigned long long *)sse_dev);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? LSB_OK : hip_fail(e, "sse kernel launch");
}

}  // extern "C"
