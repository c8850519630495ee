// rfi_item.hpp -- what the int8 and int16 kernels of librfimad share: window
// parameters, the digital noise and its pools, sample loads of generic
// windows, the item loop and the launch of an item kernel.
#pragma once

#include "rfi_device.hpp"
#include "rfi_internal.hpp"

namespace rfi {

static __constant__ int16_t c_q8[4096] = {
#include "q8_table.inc"
};

struct WinParams {
    int32_t lo;   // lowest unflagged value, m - floor(t) saturated
    int32_t hi;   // highest unflagged value, m + floor(t) saturated
    int32_t m;    // median
    int32_t sq8;  // (int)(1.4826f * D * 256), Q8 robust sigma for noise
};

__device__ __forceinline__ uint64_t pick4(const Philox4x64& r, int i)
{
    const uint64_t a = (i & 1) ? r.w[1] : r.w[0];
    const uint64_t b = (i & 1) ? r.w[3] : r.w[2];
    return (i & 2) ? b : a;
}

// Robust sigma, threshold and the integer bounds of one window (Eq. (1)).
__device__ __forceinline__ float threshold_of(int D, float k, float& sig)
{
    sig = __fmul_rn(1.4826f, (float)D);
    return __fmul_rn(k, sig);
}

// ---------------------------------------------------------------------------
// Noise.  One Philox4x64-10 block (counter j >> 2) serves 4 consecutive
// samples: sample j takes word j & 3 and indexes the Q8 table with its 12
// most significant bits.
// ---------------------------------------------------------------------------
// 4 int8 noise samples starting at absolute index j0 (a multiple of 4):
// byte c is sample j0 + c.
__device__ __forceinline__ uint32_t noise_quad_i8(uint64_t j0, uint64_t seed, uint32_t key, int m,
                                                  int sq8)
{
    const Philox4x64 r = philox4x64_10(j0 >> 2, seed, key);
    uint32_t nb = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int g = c_q8[(uint32_t)(r.w[c] >> 52)];
        const int q = (sq8 * g + 32768) >> 16;  // |sq8 * g| < 2^31 for int8
        nb |= ((uint32_t)min(max(m + q, -128), 127) & 0xFFu) << (8 * c);
    }
    return nb;
}

// The flagged 4-sample parts (one Philox block each) of a workgroup's tile
// are pooled into one list, and one thread turns each entry into its
// merged part (noise in the flagged samples), so the draws of a workgroup
// occupy as few waves as the list needs and an isolated flagged sample
// costs one block.  int8: a lane holds load slots of four parts, one dword
// each; cf bit (slot * 4 + part) marks a part holding a flagged sample;
// merged(wave, lane, slot, part, x) returns the merged part from the input
// part x.  The list and the parts (1 KiB each) live in LDS that the tile no
// longer needs once its windows' parameters are known (its histograms):
// nothing is written there before the first barrier below, which every
// wave reaches only after its selection.  The per-wave counts have storage
// of their own, as they are written before that barrier.
struct NoiseScratch {
    uint32_t* counts;  // [4]
    uint32_t* list;    // [256]
    uint4* data;       // the parts, 16-byte aligned
};
constexpr int kNoiseAliasWords = 256 + 4 * 256;

// A workgroup of kBlock threads; the list holds as many parts a round.
template <int NQ, class PartFn>
__device__ __forceinline__ void pool_noise(uint32_t (&v)[NQ], uint32_t cf, const NoiseScratch& ns, PartFn merged)
{
    constexpr int C = kBlock;  // parts per round
    uint32_t* data = reinterpret_cast<uint32_t*>(ns.data);
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    const uint32_t cnt = __popc(cf);
    const uint32_t incl = group_incl_scan<64>(cnt);
    if (lane == 63) ns.counts[wave] = incl;
    __syncthreads();
    int wbase = 0, F = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        const int c = (int)ns.counts[w];
        wbase += w < wave ? c : 0;
        F += c;
    }
    const int base = wbase + (int)(incl - cnt);
    // With no entries the loop below has no barrier: close the counts reads
    // here so no wave reuses the scratch while another still reads it.
    if (F == 0) __syncthreads();
    for (int r0 = 0; r0 < F; r0 += C) {
        int e = base - r0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if ((cf >> q) & 1u) {
                if (e >= 0 && e < C) {
                    ns.list[e] = (uint32_t)(q / 4 << 10 | wave << 8 | lane << 2 | (q % 4));
                    data[e] = v[q];
                }
                ++e;
            }
        }
        __syncthreads();
        const int k = (int)threadIdx.x;
        if (k < min(C, F - r0)) {
            const uint32_t ent = ns.list[k];
            data[k] = merged((int)((ent >> 8) & 3u), (int)((ent >> 2) & 63u), (int)(ent >> 10), (int)(ent & 3u),
                             data[k]);
        }
        __syncthreads();
        e = base - r0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if ((cf >> q) & 1u) {
                if (e >= 0 && e < C) v[q] = data[e];
                ++e;
            }
        }
        __syncthreads();
    }
}

// Orders the LDS accesses of NT cooperating threads: one wave by itself, or
// the workgroup.
template <int NT>
__device__ __forceinline__ void group_sync()
{
    if constexpr (NT == 64) wave_sync();
    else __syncthreads();
}

// pool_noise for int16 (a part is two dwords, two parts to a load slot) and
// without its first barrier: each wave reserves its slots with
// one LDS atomic add on ns.counts[0], which the caller has zeroed before a
// workgroup barrier that precedes the call (the waves' slots then follow
// in the order of their adds).  The total is read after the barrier that
// closes the list writes.  A wave writes its list entries and parts as soon
// as it arrives, so the list and the parts must have storage of their own:
// unlike pool_noise's, they cannot alias memory that another wave of the
// workgroup may still be reading.  NT = 64: one wave by itself, with no
// barriers and no counter, whose list may take the place of what the wave
// no longer needs.  tid: the thread's index among the NT.
template <int NT, int NV, class PartFn>
__device__ __forceinline__ void pool_noise_reserved(uint32_t (&v)[NV], uint32_t cf, const NoiseScratch& ns, int tid,
                                                    int wave, PartFn merged)
{
    constexpr int C = NT;
    uint2* data = reinterpret_cast<uint2*>(ns.data);
    const int lane = lane_id();
    const uint32_t cnt = __popc(cf);
    const uint32_t incl = group_incl_scan<64>(cnt);
    uint32_t wb = 0;
    int F = __builtin_amdgcn_readlane((int)incl, 63);
    if constexpr (NT == 64) {
        if (F == 0) return;
    } else {
        if (lane == 0 && F) wb = atomicAdd(&ns.counts[0], (uint32_t)F);
        wb = (uint32_t)__builtin_amdgcn_readfirstlane((int)wb);
    }
    const int base = (int)(wb + incl - cnt);
    for (int r0 = 0;; r0 += C) {
        int e = base - r0;
#pragma unroll
        for (int q = 0; q < NV / 2; ++q) {
            if ((cf >> q) & 1u) {
                if (e >= 0 && e < C) {
                    ns.list[e] = (uint32_t)(q / 2 << 12 | wave << 8 | lane << 2 | (q % 2));
                    data[e] = make_uint2(v[2 * q], v[2 * q + 1]);
                }
                ++e;
            }
        }
        group_sync<NT>();
        if constexpr (NT > 64) F = (int)ns.counts[0];  // every wave has added its count
        const int k = tid;
        if (k < min(C, F - r0)) {
            const uint32_t ent = ns.list[k];
            data[k] = merged((int)((ent >> 8) & 15u), (int)((ent >> 2) & 63u), (int)(ent >> 12), (int)(ent & 3u),
                             data[k]);
        }
        group_sync<NT>();
        e = base - r0;
#pragma unroll
        for (int q = 0; q < NV / 2; ++q) {
            if ((cf >> q) & 1u) {
                if (e >= 0 && e < C) {
                    const uint2 t = data[e];
                    v[2 * q] = t.x;
                    v[2 * q + 1] = t.y;
                }
                ++e;
            }
        }
        group_sync<NT>();
        if (r0 + C >= F) break;
    }
}

template <typename T>
__device__ __forceinline__ int load_logical(const StreamView& d, int64_t i)
{
    return i < d.head_len ? (int)gload(static_cast<const T*>(d.x_head) + i)
                          : (int)gload(static_cast<const T*>(d.x) + (i - d.head_len));
}

// Noise sample for absolute index j (one Philox block per 4 samples).
__device__ __forceinline__ int noise_sample(int64_t j, uint64_t seed, uint32_t key, int m, int sq8,
                                            int vmin, int vmax)
{
    const Philox4x64 r = philox4x64_10((uint64_t)j >> 2, seed, key);
    const uint64_t word = pick4(r, (int)(j & 3));
    const int g = c_q8[(uint32_t)(word >> 52)];
    const int64_t q = ((int64_t)sq8 * g + 32768) >> 16;
    return (int)min(max((int64_t)m + q, (int64_t)vmin), (int64_t)vmax);
}

// A carry update by one workgroup.  The usual carry is one run of whole
// 16-byte units (a block's tail).  The item is taken by value: through a
// reference its fields are read again after every store.
__device__ __forceinline__ void carry_copy(CarryItem c)
{
    const uint64_t bytes = (uint64_t)c.count * (uint64_t)c.elem;
    if (c.from == 0 && c.count <= c.head_len && ((c.head | c.dst | bytes) & 15u) == 0) {
        for (uint64_t i = threadIdx.x; i < bytes / 16; i += kBlock)
            gstore16(reinterpret_cast<void*>(c.dst + 16 * i), gload16(reinterpret_cast<const void*>(c.head + 16 * i)));
        return;
    }
    for (int i = (int)threadIdx.x; i < c.count; i += kBlock) {
        const int j = c.from + i;
        const uint64_t src = j < c.head_len ? c.head + (uint64_t)j * c.elem
                                            : c.body + (uint64_t)(j - c.head_len) * c.elem;
        const uint64_t dst = c.dst + (uint64_t)i * c.elem;
        if (c.elem == 1)
            gstore(reinterpret_cast<uint8_t*>(dst), gload(reinterpret_cast<const uint8_t*>(src)));
        else
            gstore(reinterpret_cast<uint16_t*>(dst), gload(reinterpret_cast<const uint16_t*>(src)));
    }
}

// Runs body(item_index) for this workgroup's items.  PERSIST: grid-stride
// loop; otherwise exactly one item per workgroup (no loop, so nothing is
// kept live across items).
template <bool PERSIST, class Body>
__device__ __forceinline__ void for_items(const LaunchArgs& a, Body body)
{
    if constexpr (PERSIST) {
        for (int64_t it = blockIdx.x; it < a.n_items; it += gridDim.x) body(it);
    } else {
        if ((int64_t)blockIdx.x < a.n_items) body((int64_t)blockIdx.x);
    }
}

// ---------------------------------------------------------------------------
// Launches.
// ---------------------------------------------------------------------------
// wg_per_cu > 0 caps the workgroups resident on one CU by padding each
// workgroup's LDS allocation (160 KiB per CU), an occupancy limit the
// autotuner can choose.
static hipError_t launch(void (*k)(LaunchArgs), const LaunchArgs& a, int grid, hipStream_t s)
{
    if (a.n_items <= 0) return hipSuccess;
    if (grid < 1) grid = 1;
    size_t dyn = 0;
    if (wg_per_cu() > 0) {
        hipFuncAttributes fa;
        if (hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(k)) == hipSuccess) {
            const size_t want = (160u * 1024u) / (size_t)wg_per_cu();
            if (want > fa.sharedSizeBytes) dyn = ((want - fa.sharedSizeBytes) + 255) & ~(size_t)255;
            if (dyn + fa.sharedSizeBytes > 160u * 1024u) dyn = 0;
        }
    }
    LaunchArgs args = a;
    void* kargs[] = {&args};
    return hipLaunchKernel(reinterpret_cast<const void*>(k), dim3(grid), dim3(kBlock), kargs, dyn, s);
}

// Workgroups of kernel k that are resident on the device at once.
static int resident_grid(void (*k)(LaunchArgs))
{
    int per_cu = 0;
    if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kBlock, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    return per_cu * cus;
}

}  // namespace rfi
