// rfi_internal.hpp -- structures shared by the host runtime and the kernels
// of librfimad (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rfi_mad.h"

namespace rfi {

// Samples of one workgroup tile: 16 KiB (4 waves x 64 lanes x 64 bytes).
constexpr int kTileBytes = 16384;
constexpr int kBlock = 256;

// Per-stream parameters, resident in device memory for the life of a plan.
// Addresses are byte offsets added to the base addresses of LaunchArgs, so
// one table serves any buffers (plans) or holds absolute addresses with
// zero bases (serving).
struct StreamDesc {
    uint64_t x_off;      // first input element
    uint64_t y_off;      // first output element (logical index 0)
    uint64_t stats_off;  // stats entry of window 0
    uint64_t head_off;   // carry samples that precede x (serving)
    int64_t length;      // logical samples: head_len + body samples
    int64_t abs_base;    // absolute stream index of logical sample 0
    int32_t window;      // W
    float k;             // threshold multiple
    int32_t mode;        // rfi_mode
    uint32_t key;        // Philox key word 1 (stream index or stream id)
    int32_t head_len;    // carry samples at head_off
    int32_t flags;       // kNoStats, kPadded
};
constexpr int32_t kNoStats = 1;
// The stream lies in the packed batch layout, whose buffers extend to a
// multiple of 64 elements past its end (reads may round up to 16 bytes).
constexpr int32_t kPadded = 2;

// A stream as the kernels see it, with addresses resolved.
struct StreamView {
    const void* x;
    void* y;
    rfi_window_stats* stats;  // NULL: no statistics
    uint8_t* mads;            // statistics-only launches: MADs, or NULL
    const void* x_head;
    int64_t length;
    int64_t abs_base;
    int32_t window;
    float k;
    int32_t mode;
    uint32_t key;
    int32_t head_len;
    int32_t padded;  // kPadded
};

// One unit of work for a workgroup.
//   kind == kItemTile:    a 16 KiB tile of whole, aligned windows of a stream
//                         whose W is a tile class; `first` = first sample.
//   kind == kItemGeneric: one window of any size/alignment; `first` = its
//                         window index.
struct Item {
    int32_t stream;
    int32_t kind;
    int64_t first;
};
//   kind == kItemCarry:   a serving carry update (fused kernels); `stream` =
//                         its index in LaunchArgs::carries.
constexpr int32_t kItemTile = 0;
constexpr int32_t kItemGeneric = 1;
constexpr int32_t kItemCarry = 2;

// Window classes with a register-resident tile path.
//   int8:  512, 1024, 2048, 4096 (one wave per window or less),
//          8192, 16384 (2 or 4 waves per window);
//   int16: 8192 (four waves per window).
inline __host__ __device__ int i8_tile_class(int32_t w)
{
    switch (w) {
        case 512: return 0;
        case 1024: return 1;
        case 2048: return 2;
        case 4096: return 3;
        case 8192: return 4;
        case 16384: return 5;
        default: return -1;
    }
}
constexpr int kI8Classes = 6;
inline __host__ __device__ int i16_tile_class(int32_t w) { return w == 8192 ? 0 : -1; }
constexpr int kI16Classes = 1;

// Internal mode: compute window statistics only (median, MAD, and the flag
// count and threshold of the window's own MAD); write no samples.  Used by
// the median-of-MAD path's first pass.
constexpr int32_t kModeStats = 3;

// Serving carry update: copies logical elements [from, from + count) of the
// concatenation (head[0 .. head_len), body[...]) to dst.  Addresses are
// absolute device addresses.
struct CarryItem {
    uint64_t head;
    uint64_t body;
    uint64_t dst;
    int32_t head_len;
    int32_t from;
    int32_t count;
    int32_t elem;  // 1 or 2 bytes
};

// Kernel launch requests issued by the host runtime.
struct LaunchArgs {
    const StreamDesc* streams;
    const Item* items;
    int64_t n_items;
    uint64_t seed;
    uint64_t x_base;      // added to StreamDesc::x_off / head_off
    uint64_t y_base;      // added to StreamDesc::y_off
    uint64_t stats_base;  // added to StreamDesc::stats_off
    int32_t no_stats;     // 1: write no statistics at all
    int32_t pad;
    const CarryItem* carries;  // of kItemCarry items
    // statistics-only launches: byte g receives window g's MAD (g in the
    // packed stats order); 0: none
    uint64_t mad_base;
};

__host__ __device__ inline StreamView resolve(const StreamDesc& d, const LaunchArgs& a)
{
    StreamView v;
    v.x = reinterpret_cast<const void*>(static_cast<uintptr_t>(a.x_base + d.x_off));
    v.y = reinterpret_cast<void*>(static_cast<uintptr_t>(a.y_base + d.y_off));
    v.stats = (a.no_stats || (d.flags & kNoStats))
                  ? nullptr
                  : reinterpret_cast<rfi_window_stats*>(static_cast<uintptr_t>(a.stats_base + d.stats_off));
    v.mads = a.mad_base ? reinterpret_cast<uint8_t*>(static_cast<uintptr_t>(
                              a.mad_base + d.stats_off / sizeof(rfi_window_stats)))
                        : nullptr;
    v.x_head = reinterpret_cast<const void*>(static_cast<uintptr_t>(a.x_base + d.head_off));
    v.length = d.length;
    v.abs_base = d.abs_base;
    v.window = d.window;
    v.k = d.k;
    v.mode = d.mode;
    v.key = d.key;
    v.head_len = d.head_len;
    v.padded = (d.flags & kPadded) != 0;
    return v;
}

// Host wrappers around the kernels (defined in rfi_kernels.hip).
// cls: tile class (-1 = generic items); modes: bit m set if mode m occurs;
// fused: one kernel for all kinds.
hipError_t launch_i8_tiles(int cls, int modes, int tpw, const LaunchArgs& a, int grid, hipStream_t s);
// modes: bit m set if some window of the launch uses mode m.
// small_nt: kShortWindows if every stream of the launch has short windows,
// else i8_window_threads of its longest window, if its streams are padded and
// start at absolute index 0, used when the grid covers every item; 0: windows
// of any kind, 256 threads each.
// i8_window_threads: threads per window for `count` windows of up to n
// samples: four 16-byte chunks per thread, or eight (kWideThreads), which
// need fewer waves per window; n + 30 <= 16 * chunks * threads keeps a window
// within them at any alignment.  A launch of few windows leaves the device
// idle and takes as long as one window, so it gives each more threads (60
// streams, noise, microseconds, 256 threads against the fewest: 60 windows of
// 3000 samples 6.8 / 8.3, 480 of 4067 7.2 / 10.0; 128 threads of four chunks
// against 64 of eight, 960 of 6000 8.7 / 10.3, 3840 16.8 / 17.8, 15360 45.1 /
// 42.8), and so does one whose chunks nearly fill them (15360 windows, 256
// threads of four against 128 of eight, clip: 9000 samples 54 / 53, 12000 65 /
// 67, 14001 77 / 86, 16354 88 / 101; noise: 12000 79 / 75, 14001 92 / 89, 15000 95
// / 93, 16354 99 / 100).  noise: some window of the launch may be in noise
// mode.  no_scratch: only kernels without private memory
// (eight chunks of 64 or 128 threads spill in noise mode).
constexpr int kWideThreads = 1;
constexpr int kShortWindows = 2;
inline int i8_window_threads(int64_t n, int64_t count, bool noise, bool no_scratch = false)
{
    if (n > 32738) return 0;
    if (n > 16354) return 256 | kWideThreads;
    if (count <= 512) return 256;
    if (n <= 4066) return 64;
    const bool few = count <= 4096 || no_scratch;
    if (n <= 8162) return few ? 128 : 64 | kWideThreads;
    return few || n > (noise ? 15000 : 11000) ? 256 : 128 | kWideThreads;
}
// Whether a stream's windows are short: counting them into one plain
// histogram by one wave, sample by sample, beats holding 16-byte chunks in
// registers and four replicas of the histogram, which cost the same for any
// length (61440 windows, noise, W 1 26 / 63 us, 100 40 / 63, 200 56 / 64, 300 69
// / 65; clip, W 100 31 / 36, 150 36 / 38, 200 40 / 37).  noise: some stream of
// the batch is in noise mode.  In a batch that also has longer windows, short
// ones take a launch of their own (3 us) if they are this many: below, they
// cost no more than that in the longer ones' kernel.
inline bool i8_short_windows(int32_t W, int64_t L, bool noise) { return (L < W ? L : W) <= (noise ? 256 : 160); }
constexpr int64_t kShortLaunch = 4096;
hipError_t launch_i8_generic(const LaunchArgs& a, int modes, int grid, hipStream_t s, int small_nt = 0);
hipError_t launch_i8_fused(int modes, const LaunchArgs& a, int grid, hipStream_t s);
hipError_t launch_i16_tiles(int cls, int modes, const LaunchArgs& a, int grid, hipStream_t s);
// nt: threads per window (64, 128 or 512 with four 16-byte chunks each, 128 or
// 256 with eight: kWideThreads) if they hold every window of the launch, its
// streams are padded and start at absolute index 0, used when the grid covers
// every item; 0: 256-thread workgroups for windows of any kind.
hipError_t launch_i16_generic(const LaunchArgs& a, int modes, int grid, hipStream_t s, int nt = 0);
hipError_t launch_i16_fused(const LaunchArgs& a, int grid, hipStream_t s);
// One workgroup of each fused kernel that a server's batch may take, with no
// items.  A kernel that needs private (scratch) memory has it set up by the
// runtime at its first dispatch on a hardware queue, which can hold that queue
// for milliseconds; a server runs this once per lane when it is created, so
// that no block's latency pays for it.
hipError_t warm_i8_fused(bool persist, hipStream_t s);
hipError_t warm_i16_fused(bool persist, hipStream_t s);

// Several outputs from one read (int8 tile items): output o uses the
// descriptors desc[o] (its k and mode; offsets as a.streams) and the bases
// y_base[o], stats_base[o] (0: no statistics).  a.items: tiles of one class.
struct MultiArgs {
    LaunchArgs a;
    const StreamDesc* desc[3];
    uint64_t y_base[3];
    uint64_t stats_base[3];
    int32_t n_out;
    int32_t pad;
};
// Outputs in zero or clip mode only.
hipError_t launch_i8_multi(int cls, const MultiArgs& ma, int grid, hipStream_t s);

// Median of MAD (int8).  Windows of all streams are numbered globally in
// the packed stats order; mad[g] is window g's own MAD (written by the
// statistics pass), dm[g] receives the lower median of the MADs of its
// stream's last K windows.  Each stream's MAD sequence is `pre` history
// slots (hist[s * pre ..]: the MADs of earlier calls, right-aligned,
// hist_len[s] of them valid) followed by its windows; pre = 0 when there is
// no history.
struct MomStream {
    int64_t woff;  // first window of the stream in the stats order
    int64_t nw;    // windows of the stream in this call
    int64_t pre;   // history slots before its first window (0 or K - 1)
};
// One wave's windows of the median search: `first` .. first + n - 1 of a
// stream.
struct MomSeg {
    int32_t stream;
    int32_t n;
    int64_t first;
};
hipError_t launch_mom_select(const MomStream* streams, const MomSeg* segs, int64_t n_segs, int32_t mom_k,
                             const uint8_t* mad, const uint8_t* hist, const int32_t* hist_len, int32_t* dm,
                             hipStream_t s);
// Replacement pass: items of up to 256 windows (<= 16 KiB) of one stream;
// window params from stats (median) and dm; rewrites n_flagged and threshold.
struct MomItem {
    int32_t stream;
    int32_t n_windows;
    int64_t first_window;  // within the stream
};
// abs_add: NULL, or per stream an offset added to its absolute sample index.
// n_hist streams (0 without a carried history): one workgroup each writes the
// new history, the last min(pre, hist_len + nw) entries of the stream's MAD
// sequence, right-aligned in hist[s * pre ..], and hist_len.
struct MomHistory {
    const MomStream* streams;
    const uint8_t* mad;
    uint8_t* hist;
    int32_t* hist_len;
    int32_t n_hist;
};
hipError_t launch_mom_apply(const LaunchArgs& a, const MomItem* items, int64_t n_items,
                            const int32_t* dm, const int64_t* stream_woff, const int64_t* abs_add,
                            rfi_window_stats* stats, const MomHistory& h, hipStream_t s);
// Copies n16 16-byte units from pinned host memory to device memory.
hipError_t launch_stage(void* dst, const void* src_host, int64_t n16, hipStream_t s);

// Launches k and returns this launch's own status (hipGetLastError would also
// report an error that the program left before).
template <class T> struct SameType { using type = T; };
template <class... P>
hipError_t launch_kernel(void (*k)(P...), dim3 grid, dim3 block, hipStream_t s, typename SameType<P>::type... args)
{
    void* kargs[] = {const_cast<void*>(static_cast<const volatile void*>(&args))...};
    return hipLaunchKernel(reinterpret_cast<const void*>(k), grid, block, kargs, 0, s);
}

// Occupancy cap for the launches issued by this thread (0: none).
void set_wg_per_cu(int n);
int wg_per_cu();

// Occupancy-derived persistent grid size for a kernel choice.
int persistent_grid(int elem_size, int cls, int modes, bool fused);
int i8_persistent_grid(int cls, int modes, bool fused);
int i16_persistent_grid(int cls, int modes, bool fused);

}  // namespace rfi
