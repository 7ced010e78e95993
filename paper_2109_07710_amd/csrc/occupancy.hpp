// Device bodies shared by the stand-alone integer launches and the combined
// preparation launch of both gradients: the non-zero test of 16-byte
// vectors, and the dY block occupancy (with the X-window liveness).
#pragma once

#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "footprint.hpp"

namespace cbw {

// Bit per element: relu ? (value > 0) : (value != 0), over 16-byte vectors.
template <typename T>
__device__ __forceinline__ uint32_t vec_bits(const uint4& v, bool relu)
{
    constexpr int E = Elem<T>::E;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t b = 0;
#pragma unroll
    for (int i = 0; i < E; ++i) {
        uint32_t u;
        if (sizeof(T) == 2) u = (w[i >> 1] >> ((i & 1) * 16)) & 0xffffu;
        else u = w[i];
        bool on;
        if (sizeof(T) == 2) {
            const uint32_t mag = u & 0x7fffu;
            on = relu ? ((u & 0x8000u) == 0 && mag != 0 && mag <= 0x7f80u) : (mag != 0);
        } else {
            const uint32_t mag = u & 0x7fffffffu;
            on = relu ? ((u >> 31) == 0 && mag != 0 && mag <= 0x7f800000u) : (mag != 0);
        }
        b |= (on ? 1u : 0u) << i;
    }
    return b;
}

// Workgroup `block` of the occupancy pass (256 threads):
// occ[chunk][kt] = 1 iff dY has a non-zero in pixels of the chunk and
// channels of k-tile kt (from the packed footprint when given: one (pixel,
// k-tile) pair per thread and round, eight rounds' loads issued together,
// the tile's words read as one or two vectors when K is a multiple of the
// tile width).  A workgroup covers p.cpw consecutive chunks, about four
// pairs per thread, so narrow layers do not launch one nearly idle workgroup
// per 64-pixel chunk.
__device__ __forceinline__ void occupancy_block(const OccParams& p, int block)
{
    // Per (chunk of the group, k tile) block a flag, set by the non-zeros it
    // holds -- or, where the live pixels are recorded (64-pixel chunks, packed
    // footprint), the block's dead pixels, a bit each: an element-wise
    // footprint has none and marks nothing.
    __shared__ uint32_t marks[2048];
    __shared__ int found_s;                      // 1: a dead block, 2: one with more dead pixels than live ones
    if (threadIdx.x == 0) found_s = 0;
    int* const flags = reinterpret_cast<int*>(marks);
    uint32_t* const dead_s = marks;
    const bool pixels = p.pmask != nullptr && p.bits != nullptr;
    const int chunk0 = block * p.cpw;
    const int nloc = min(p.cpw, p.nchunks - chunk0);
    const int px0 = chunk0 * p.chunk;
    const int npx = min(nloc * p.chunk, p.npq - px0);   // pixels of the group
    for (int i = threadIdx.x; i < nloc * p.ktiles * (pixels ? 2 : 1); i += blockDim.x) marks[i] = 0u;
    __syncthreads();
    auto mark_dead = [&](int i) {   // pair i of the group
        const int j = (int)fdiv((uint32_t)i, p.div_ktiles), kt = i - j * p.ktiles;
        atomicOr(&dead_s[2 * ((j >> 6) * p.ktiles + kt) + ((j >> 5) & 1)], 1u << (j & 31));
    };
    if (p.bits) {
        // whole 8-, 16- or 32-byte aligned word runs per (pixel, k tile) when
        // K is a multiple of the tile width (64, 128 or 256 channels)
        const int vw = (p.K % p.BNk) == 0 ? (p.BNk == 256 ? 8 : p.BNk == 128 ? 4 : p.BNk == 64 ? 2 : 0) : 0;
        const int pairs = npx * p.ktiles;
        const int64_t bits_bytes = ((int64_t)p.npq * p.K + 31) / 32 * 4;
        const int lane = threadIdx.x & 63;
        // eight (pixel, k tile) pairs per thread and round; consecutive
        // threads read consecutive runs.  The runs go through a buffer
        // descriptor, so every load is issued unconditionally (a pair past
        // the group gets offset kOOB and reads zeros) and the eight of a
        // round are in flight together.  A lane marks its pair's flag only
        // when the lane before it does not mark the same one, so a wave
        // whose pairs share a chunk writes that flag once.
        auto rounds = [&](auto vw_tag) {
            constexpr int VW = decltype(vw_tag)::value;
            const __amdgpu_buffer_rsrc_t rs = make_rsrc(p.bits, (uint32_t)bits_bytes);
            for (int i0 = threadIdx.x; i0 < pairs; i0 += 8 * blockDim.x) {
                int idx[8];
                uint32_t off[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = i0 + u * blockDim.x;
                    const int j = (int)fdiv((uint32_t)i, p.div_ktiles), kt = i - j * p.ktiles;   // pixel of the group, k tile
                    idx[u] = (int)fdiv((uint32_t)j, p.div_chunk) * p.ktiles + kt;
                    off[u] = i < pairs ? (uint32_t)(((int64_t)(px0 + j) * p.K + kt * p.BNk) >> 3) : kOOB;
                }
                uint32_t w[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if constexpr (VW == 2) {
                        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, off[u], 0, 0);
                        w[u] = v.x | v.y;
                    } else if constexpr (VW == 4) {
                        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, off[u], 0, 0);
                        w[u] = v.x | v.y | v.z | v.w;
                    } else {
                        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, off[u], 0, 0);
                        const u32x4 v2 = __builtin_amdgcn_raw_buffer_load_b128(rs, off[u] + 16u, 0, 0);
                        w[u] = (v.x | v.y | v.z | v.w) | (v2.x | v2.y | v2.z | v2.w);
                    }
                }
                if (!pixels) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int key = w[u] != 0u ? idx[u] : -1;
                        const int prev = __shfl_up(key, 1, 64);
                        if (key >= 0 && (lane == 0 || prev != key)) flags[idx[u]] = 1;   // every writer stores 1
                    }
                } else {
                    uint32_t least = w[0];   // zero iff some pair is dead (or past the group)
#pragma unroll
                    for (int u = 1; u < 8; ++u) least = min(least, w[u]);
                    if (least == 0u) {
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            if (w[u] == 0u && off[u] != kOOB) mark_dead(i0 + u * blockDim.x);
                    }
                }
            }
        };
        if (vw == 2 && bits_bytes < (int64_t)kOOB) rounds(std::integral_constant<int, 2>{});
        else if (vw == 4 && bits_bytes < (int64_t)kOOB) rounds(std::integral_constant<int, 4>{});
        else if (vw == 8 && bits_bytes < (int64_t)kOOB) rounds(std::integral_constant<int, 8>{});
        else {
            for (int i = threadIdx.x; i < pairs; i += blockDim.x) {
                const int j = (int)fdiv((uint32_t)i, p.div_ktiles), kt = i - j * p.ktiles;
                const int64_t base = (int64_t)(px0 + j) * p.K;
                const int lo = kt * p.BNk, hi = min(p.K, lo + p.BNk);
                const bool any = any_bits(p.bits, base + lo, base + hi);
                if (pixels) {
                    if (!any) mark_dead(i);
                } else if (any) {
                    flags[(int)fdiv((uint32_t)j, p.div_chunk) * p.ktiles + kt] = 1;   // every writer stores 1
                }
            }
        }
    } else {
        const int E = p.dtype == 1 ? 8 : 4;
        const int vpp = p.K / E;  // vectors per pixel
        const int nv = npx * vpp;
        const uint4* v4 = reinterpret_cast<const uint4*>(static_cast<const char*>(p.dy) +
                                                         (int64_t)px0 * p.K * (p.dtype == 1 ? 2 : 4));
        for (int i = threadIdx.x; i < nv; i += blockDim.x) {
            const uint4 v = v4[i];
            const uint32_t b = p.dtype == 1 ? vec_bits<uint16_t>(v, false) : vec_bits<float>(v, false);
            const int j = i / vpp;
            if (b) flags[(int)fdiv((uint32_t)j, p.div_chunk) * p.ktiles + ((i - j * vpp) * E) / p.BNk] = 1;
        }
    }
    __syncthreads();
    bool dead = false, sparse = false;
    for (int i = threadIdx.x; i < nloc * p.ktiles; i += blockDim.x) {
        bool any;
        if (pixels) {
            const int cl = (int)fdiv((uint32_t)i, p.div_ktiles), kt = i - cl * p.ktiles;
            const int left = npx - cl * 64;   // pixels of the block (at least one)
            const uint64_t valid = left >= 64 ? ~0ull : (1ull << left) - 1;
            const uint64_t live = valid & ~(((uint64_t)dead_s[2 * i + 1] << 32) | dead_s[2 * i]);
            p.pmask[(int64_t)kt * p.nchunks + chunk0 + cl] = live;
            any = live != 0;
            sparse |= any && 2 * __popcll(live) <= 64;
        } else {
            any = flags[i] != 0;
        }
        dead |= !any;
        p.occ[(int64_t)chunk0 * p.ktiles + i] = any ? 1 : 0;
    }
    // the call's flags (every writer stores the same number)
    if (dead || sparse) atomicOr(&found_s, (dead ? 1 : 0) | (sparse ? 2 : 0));
    __syncthreads();
    const int found = found_s;
    if ((found & 1) && p.any_dead && threadIdx.x == 0) p.any_dead[0] = (int)p.gen;
    if ((found & 2) && p.any_dead) {
        // A k tile whose live pixels fit half its live blocks has a workgroup
        // where they do, so the GEMM's count over the whole tile (two passes
        // of its ranking, 4 us) runs only if one says so: footprints of
        // clustered pixels have sparse blocks at densities where nothing can
        // be gained.  Per k tile the sum of 2 live - 64 over the live blocks,
        // scaled so that a sum of zero with a live block counts.
        __shared__ int sum[1024];
        for (int i = threadIdx.x; i < p.ktiles; i += blockDim.x) sum[i] = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < nloc * p.ktiles; i += blockDim.x) {
            const int cl = (int)fdiv((uint32_t)i, p.div_ktiles);
            const int n = min(64, npx - cl * 64) - __popc(dead_s[2 * i]) - __popc(dead_s[2 * i + 1]);
            if (n > 0) atomicAdd(&sum[i - cl * p.ktiles], 2048 * (2 * n - 64) - 1);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < p.ktiles; i += blockDim.x)
            if (sum[i] < 0) p.any_dead[1] = (int)p.gen;
    }

    // X-window liveness for every (tap group, channel tile) of the weight
    // gradient's tiling: 1 iff some pixel of the chunk has, at one of the
    // group's taps, an X pixel inside the image with a non-zero among the
    // tile's channels (from the packed X footprint).
    if (p.xlive) {
        __shared__ int xflags[1024];             // [chunk of the group][combo]
        const int ncombo = p.tgroups * p.ctiles;
        for (int i = threadIdx.x; i < nloc * ncombo; i += blockDim.x) xflags[i] = 0;
        __syncthreads();
        const int pairs = ncombo * npx;
        for (int i = threadIdx.x; i < pairs; i += blockDim.x) {
            const int combo = i / npx, j = i - combo * npx;
            const int tg = combo / p.ctiles, ct = combo - tg * p.ctiles;
            const uint32_t pix = (uint32_t)(px0 + j);
            const uint32_t nq = fdiv(pix, p.div_q);
            const int qq = (int)pix - (int)nq * p.Q;
            const uint32_t nn = fdiv(nq, p.div_p);
            const int pp = (int)nq - (int)nn * p.P;
            const int lo = ct * p.ctw, hi = min(p.C, lo + p.ctw);
            // whole 256-channel tiles on 128-bit boundaries: two vector loads
            const bool vec = hi - lo == 256 && (p.C & 127) == 0;
            bool any = false;
            for (int tl = 0; tl < p.tpg && !any; ++tl) {
                const int tap = tg * p.tpg + tl;
                if (tap >= p.RS) break;
                const int r = tap / p.S, s = tap - r * p.S;
                const int h = pp * p.stride_h - p.pad_h + r, w = qq * p.stride_w - p.pad_w + s;
                if (h < 0 || h >= p.H || w < 0 || w >= p.W) continue;
                const int64_t base = (((int64_t)nn * p.H + h) * p.W + w) * p.C;
                if (vec) {
                    const uint4* v = reinterpret_cast<const uint4*>(p.xbits + ((base + lo) >> 5));
                    const uint4 a = v[0], b = v[1];
                    any = ((a.x | a.y | a.z | a.w) | (b.x | b.y | b.z | b.w)) != 0;
                } else {
                    any = any_bits(p.xbits, base + lo, base + hi);
                }
            }
            if (any) xflags[(int)fdiv((uint32_t)j, p.div_chunk) * ncombo + combo] = 1;   // every writer stores 1
        }
        __syncthreads();
        bool xdead = false;
        for (int i = threadIdx.x; i < nloc * ncombo; i += blockDim.x) {
            p.xlive[(int64_t)chunk0 * ncombo + i] = (uint8_t)(xflags[i] != 0);
            xdead |= xflags[i] == 0;
        }
        if (__syncthreads_or(xdead) && p.any_dead && threadIdx.x == 0) *p.any_dead = (int)p.gen;
    }
}

}  // namespace cbw
