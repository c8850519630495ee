// rfi_kernels.hip -- gfx950 kernels of librfimad.
//
// Method (Buch et al., Sec. II-D): per non-overlapping window, the median
// M(x), the MAD D, the thresholds M(x) +/- k * (1.4826 * D) of Eq. (1) and the
// replacement of Eq. (2).  The work is a pure stream: every sample is read
// once from HBM and written once, so the kernels are built around 128-bit
// coalesced loads into registers and keep all per-window work in LDS.
//
// int8 windows: one 256-bin LDS histogram of x + 128 per window; a
//   segmented wave scan turns it into cumulative counts C[v]; the median is
//   the first bin with C >= r + 1 (r = floor((N-1)/2)); the MAD is the first
//   d with C[m+d] - C[m-d-1] >= r + 1, i.e. the |x - m| histogram folded out
//   of the same counts, so the samples are histogrammed once.  The flag
//   count is N - (C[hi] - C[lo-1]) and needs no extra pass.
// int16 windows of up to 16384 samples stay in registers: a histogram of one
//   value (or 2^s values, by the samples' spread) per slot around a sampled
//   estimate of the median gives the median and the MAD, with a pass over
//   the samples for the last s bits of each.  Longer ones, and windows with
//   a carried head: an 8+8-bit radix select over global memory.
// Replacement: the per-sample test |x - m| > t equals x < m - floor(t) or
//   x > m + floor(t) because |x - m| is an integer, so after one binary32
//   threshold per window everything is integer; int8 samples are clamped
//   four to a dword with packed 16-bit max/min.
// Noise: the flagged 4-sample parts of a workgroup's tile are pooled into
//   one list, one thread draws one Philox4x64-10 block per entry, and the
//   owners merge the noise bytes back, so the cost follows the number of
//   flagged parts, not the worst lane.
// Also here: the several-outputs kernels, the median-of-MAD search and
//   replacement, and the copy that brings a serving batch's tables in.
#include "rfi_item.hpp"

namespace rfi {

// ---------------------------------------------------------------------------
// int8: selection from a 256-bin histogram owned by an aligned group of G
// lanes (G = 8..64, 256 / G bins per lane).  On return the bins hold
// inclusive cumulative counts and every lane of the group has mb (median
// + 128) and D.  Used when a wave holds several windows.
// ---------------------------------------------------------------------------
// Smallest d in [0, 256) with f(d) >= need, for f non-decreasing with
// f(255) >= need, i.e. the number of d with f(d) < need.  The G lanes of a
// group test G evenly spaced candidates per step (a G-ary search), so the
// answer takes log_G(256) steps instead of a test of every d.
template <int G, int SPAN, class F>
__device__ __forceinline__ int group_search(int lo, uint32_t need, const F& f)
{
    if constexpr (SPAN <= 1) {
        return lo;
    } else {
        constexpr int STEP = SPAN >= G ? SPAN / G : 1;
        constexpr int NC = SPAN >= G ? G : SPAN;  // candidates tested
        const int sl = lane_id() & (G - 1);
        const int d = min(lo + (sl + 1) * STEP - 1, 255);
        const bool below = (NC == G || sl < NC) && f(d) < need;
        return group_search<G, STEP>(lo + group_count<G>(below) * STEP, need, f);
    }
}

// Narrow histograms are scanned by groups of G lanes, each lane over 256 / G
// consecutive bins read as 16-byte chunks.  With G = 16 (16 bins, four
// chunks per lane) bin v lives in word nphys(v): the chunks inside a lane's
// run are permuted by XOR with bits 6-7 of v, so that the group's 16-byte
// reads of the same chunk fall in different banks (without it the 16 lanes
// of a group meet in four).  Measured 4-6 % faster at W 512 and 1024; at
// G = 32 (W 2048) it did not pay, and G = 64 has a single chunk: identity.
template <int G>
__device__ __forceinline__ int nphys(int v)
{
    return G == 16 ? (v ^ (((v >> 6) & 3) << 2)) : v;
}
// nphys of the four bytes of u at once.
template <int G>
__device__ __forceinline__ uint32_t nphys4(uint32_t u)
{
    return G == 16 ? (u ^ ((u >> 4) & 0x0C0C0C0Cu)) : u;
}

// Median bin and MAD of one window from its 256-bin histogram hw (bin v
// counts samples x = v - 128), by the G lanes of a group.  Leaves the
// cumulative counts C[v] = #{x <= v - 128} in hw.
template <int G>
__device__ __forceinline__ void select_i8(uint32_t* hw, uint32_t need, int& mb, int& D)
{
    constexpr int BPL = 256 / G;
    const int sl = lane_id() & (G - 1);
    uint32_t* my = hw + sl * BPL;
    const int key = G == 16 ? (((sl >> 2) & 3) << 2) : 0;  // chunk permutation of nphys
    uint32_t c[BPL];
#pragma unroll
    for (int j = 0; j < BPL; j += 4) {
        const uint4 t = *reinterpret_cast<const uint4*>(my + (j ^ key));
        c[j] = t.x;
        c[j + 1] = t.y;
        c[j + 2] = t.z;
        c[j + 3] = t.w;
    }
#pragma unroll
    for (int j = 1; j < BPL; ++j) c[j] += c[j - 1];
    const uint32_t incl = group_incl_scan<G>(c[BPL - 1]);
    const uint32_t excl = incl - c[BPL - 1];
#pragma unroll
    for (int j = 0; j < BPL; ++j) c[j] += excl;
#pragma unroll
    for (int j = 0; j < BPL; j += 4)
        *reinterpret_cast<uint4*>(my + (j ^ key)) = make_uint4(c[j], c[j + 1], c[j + 2], c[j + 3]);
    wave_sync();
    // The median bin is the first v with C[v] >= need.
    mb = group_search<G, 256>(0, need, [&](int v) { return hw[nphys<G>(v)]; });
    // #{|x - m| <= d} = C[min(mb + d, 255)] - C[mb - d - 1] is non-decreasing
    // in d and reaches the window size at d = 255; D is its first d >= need.
    const int m0 = mb;
    D = group_search<G, 256>(0, need, [&](int d) {
        const int dn = m0 - d - 1;
        return hw[nphys<G>(min(m0 + d, 255))] - (dn >= 0 ? hw[nphys<G>(max(dn, 0))] : 0u);
    });
}

// The same for two windows that share a histogram, one in each 16-bit half of
// a bin: GA lanes turn it into cumulative
// counts, both windows at once; then the first half of the lanes finds the
// median bin and the MAD of the window in the low halves, the second half
// those of the other.  C(v): this lane's window's count at bin v afterwards.
template <int GA>
__device__ __forceinline__ uint32_t pair_count(const uint32_t* hw, int shift, int v)
{
    return (hw[nphys<GA>(v)] >> shift) & 0xFFFFu;
}

template <int GA>
__device__ __forceinline__ void select_i8_pair(uint32_t* hw, int shift, uint32_t need, int& mb, int& D)
{
    constexpr int BPL = 256 / GA;
    const int sl = lane_id() & (GA - 1);
    uint32_t* my = hw + sl * BPL;
    const int key = GA == 16 ? (((sl >> 2) & 3) << 2) : 0;  // chunk permutation of nphys
    uint32_t c[BPL];
#pragma unroll
    for (int j = 0; j < BPL; j += 4) {
        const uint4 t = *reinterpret_cast<const uint4*>(my + (j ^ key));
        c[j] = t.x;
        c[j + 1] = t.y;
        c[j + 2] = t.z;
        c[j + 3] = t.w;
    }
#pragma unroll
    for (int j = 1; j < BPL; ++j) c[j] += c[j - 1];
    const uint32_t excl = group_incl_scan<GA>(c[BPL - 1]) - c[BPL - 1];
#pragma unroll
    for (int j = 0; j < BPL; ++j) c[j] += excl;
#pragma unroll
    for (int j = 0; j < BPL; j += 4)
        *reinterpret_cast<uint4*>(my + (j ^ key)) = make_uint4(c[j], c[j + 1], c[j + 2], c[j + 3]);
    wave_sync();
    mb = group_search<GA / 2, 256>(0, need, [&](int v) { return pair_count<GA>(hw, shift, v); });
    const int m0 = mb;
    D = group_search<GA / 2, 256>(0, need, [&](int d) {
        const int dn = m0 - d - 1;
        return pair_count<GA>(hw, shift, min(m0 + d, 255)) - (dn >= 0 ? pair_count<GA>(hw, shift, max(dn, 0)) : 0u);
    });
}

// Window parameters and statistics from the cumulative counts C(v).
template <class Count>
__device__ __forceinline__ void params_i8(const Count& C, int mb, int D, float k, int n, WinParams& p,
                                          rfi_window_stats& s)
{
    float sig;
    const float t = threshold_of(D, k, sig);
    const int T = (int)floorf(t);
    const int m = mb - 128;
    const int lo = max(m - T, -128), hi = min(m + T, 127);
    const int lob = lo + 128, hib = hi + 128;
    const uint32_t inside = C(hib) - (lob > 0 ? C(max(lob - 1, 0)) : 0u);
    p.lo = lo;
    p.hi = hi;
    p.m = m;
    p.sq8 = (int)__fmul_rn(sig, 256.0f);
    s.median = m;
    s.mad = D;
    s.n_flagged = (uint32_t)n - inside;
    s.threshold = t;
}

// ---------------------------------------------------------------------------
// Wide windows (W >= 4096, whole waves per window).  Each wave keeps four
// replicas of a 256-bin histogram (lane & 3 picks one; replicas start eight
// banks apart, which spreads same-bin atomics of a wave), indexed by the raw
// byte so a sample costs one bit-field extract and one address add.
// ---------------------------------------------------------------------------
constexpr int kRepStride = 264;                // 256 bins + 8 words
constexpr int kWaveHistWords = 4 * kRepStride;  // per wave
// Padded cumulative array (264 words): pc[0..3] = 0 (C[-4..-1]), pc[4 + v] =
// C[v] for the biased value v = 0..255, pc[260..263] = N.

__device__ __forceinline__ void wide_hist_zero(uint32_t* h)
{
    const int lane = lane_id();
    uint4* p = reinterpret_cast<uint4*>(h);
#pragma unroll
    for (int i = 0; i < (kWaveHistWords / 4 + 63) / 64; ++i) {
        const int idx = i * 64 + lane;
        if (idx < kWaveHistWords / 4) p[idx] = make_uint4(0, 0, 0, 0);
    }
}

// hl: this lane's replica.
__device__ __forceinline__ void wide_hist_add(uint32_t* hl, uint32_t x)
{
    atomicAdd(hl + (x & 0xFFu), 1u);
    atomicAdd(hl + ((x >> 8) & 0xFFu), 1u);
    atomicAdd(hl + ((x >> 16) & 0xFFu), 1u);
    atomicAdd(hl + (x >> 24), 1u);
}

// Counts of the biased bins 4*lane .. 4*lane+3 (biased bin v holds the raw
// byte (v + 128) & 255), summed over the four replicas.
__device__ __forceinline__ void wide_hist_totals(const uint32_t* h, uint32_t (&c)[4])
{
    const int rb = (4 * lane_id() + 128) & 255;
    c[0] = c[1] = c[2] = c[3] = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint4 t = *reinterpret_cast<const uint4*>(h + r * kRepStride + rb);
        c[0] += t.x;
        c[1] += t.y;
        c[2] += t.z;
        c[3] += t.w;
    }
}

// Selection over a whole wave holding the counts of bins 4*lane.. in c:
// writes the padded cumulative array pc and returns the wave-uniform mb
// (median + 128) and D.  The padding lets every lane read four consecutive
// counts without clamping its indices.
__device__ __forceinline__ void wide_select(uint32_t (&c)[4], uint32_t* pc, uint32_t need, int& mb,
                                            int& D)
{
    const int lane = lane_id();
    c[1] += c[0];
    c[2] += c[1];
    c[3] += c[2];
    const uint32_t incl = group_incl_scan<64>(c[3]);
    const uint32_t excl = incl - c[3];
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] += excl;
    *reinterpret_cast<uint4*>(pc + 4 + 4 * lane) = make_uint4(c[0], c[1], c[2], c[3]);
    if (lane == 0) *reinterpret_cast<uint4*>(pc) = make_uint4(0, 0, 0, 0);
    if (lane == 63) *reinterpret_cast<uint4*>(pc + 260) = make_uint4(c[3], c[3], c[3], c[3]);
    int below = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) below += group_count<64>(c[j] < need);
    mb = below;
    wave_sync();
    // d = 4*lane + j: C[min(mb + d, 255)] - C[mb - d - 1]
    const int t = min(mb + 4 * lane, 255) + 4;
    const int s = max(mb - 4 * lane - 1, -1) + 4;
    int dbelow = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) dbelow += group_count<64>(pc[t + j] - pc[s - j] < need);
    D = dbelow;
}

__device__ __forceinline__ void wide_params(const uint32_t* pc, int mb, int D, float k, int n,
                                            WinParams& p, rfi_window_stats& s)
{
    float sig;
    const float t = threshold_of(D, k, sig);
    const int T = (int)floorf(t);
    const int m = mb - 128;
    const int lo = max(m - T, -128), hi = min(m + T, 127);
    const uint32_t inside = pc[4 + hi + 128] - pc[3 + lo + 128];
    p.lo = lo;
    p.hi = hi;
    p.m = m;
    p.sq8 = (int)__fmul_rn(sig, 256.0f);
    s.median = m;
    s.mad = D;
    s.n_flagged = (uint32_t)n - inside;
    s.threshold = t;
}

// ---------------------------------------------------------------------------
// int8 tiles: 16 KiB of whole windows of one class W, 64 bytes per lane.
// ---------------------------------------------------------------------------
// Narrow windows: one 256-bin histogram per window, 12 words apart in bank
// order, so the same bin of the windows of a wave falls in different banks
// (12 measured 2-3 % faster than 8 at W 512, the same at W 1024 and 2048).
constexpr int kNarrowStride = 268;

template <int W, bool NS>
struct I8TileSmem {
    static constexpr int kWin = 16384 / W;
    static constexpr bool kWide = W >= 4096;
    static constexpr int kWPW = kWide ? W / 4096 : 1;  // waves per window
    // wide: per-wave replicated histograms; W = 4096 keeps its cumulative
    // counts in replica 0 of its wave, larger W in pc.
    // W = 512: two windows share a histogram, one in each half of its bins
    // (counts of at most 512), so that clearing, adding up and scanning it
    // serve both.  Against one histogram per window in two rounds, 60 x 2^22
    // samples, zero / clip / noise: 129 / 127 / 142 -> 105 / 104 / 117 us
    // (4.86 TB/s, LDS and VALU); sharing at W 1024 puts more lanes on one
    // address and gains nothing (101 / 100 / 115 -> 103 / 101 / 116).
    static constexpr bool kPair = W == 512;
    static constexpr int kHists = kPair ? kWin / 2 : kWin;
    static constexpr int kHistWords = kWide ? 4 * kWaveHistWords
                                      : kHists * kNarrowStride > kNoiseAliasWords ? kHists * kNarrowStride
                                                                                   : kNoiseAliasWords;
    static_assert(kHistWords >= kNoiseAliasWords, "noise scratch aliases the histograms");
    __align__(16) uint32_t hist[kHistWords];
    __align__(16) uint32_t tot[kWPW > 1 ? 4 * 256 : 0];  // each wave's bin totals
    WinParams prm[kWin];
    int32_t mad[kWin];  // statistics-only mode: each window's MAD
    uint32_t noise_counts[NS ? 4 : 0];
    __device__ NoiseScratch noise()
    {
        return NoiseScratch{noise_counts, hist, reinterpret_cast<uint4*>(hist + 256)};
    }
};

// Statistics record of one window produced by a tile, written by the caller
// once the tile's samples are stored.
struct TileStats {
    rfi_window_stats s;
    rfi_window_stats* dst;  // NULL: this lane writes nothing
};

__device__ __forceinline__ void write_stats(const TileStats& t)
{
    if (t.dst)
        gstore16(t.dst, make_uint4((uint32_t)t.s.median, (uint32_t)t.s.mad, t.s.n_flagged,
                                   __float_as_uint(t.s.threshold)));
}

// This lane's 64 bytes of a 16 KiB tile: four 16-byte loads at a 1 KiB
// stride, so each load instruction of the wave covers 1 KiB contiguously.
// AGAIN: the samples are read a second time soon (the statistics pass of the
// median of MAD: with non-temporal loads its call took 142 against 134 us
// for 60 x 2^22 samples, 296 against 291 for 60 x 2^23).
template <bool AGAIN = false>
__device__ __forceinline__ void tile_load(const StreamView& d, int64_t first_byte, uint32_t (&v)[16])
{
    const uint8_t* xt = static_cast<const uint8_t*>(d.x) + first_byte + (threadIdx.x >> 6) * 4096 +
                        lane_id() * 16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint4 t = AGAIN ? gload16(xt + i * 1024) : gload16_nt(xt + i * 1024);
        v[4 * i] = t.x;
        v[4 * i + 1] = t.y;
        v[4 * i + 2] = t.z;
        v[4 * i + 3] = t.w;
    }
}

// Replacement of one lane's 16 dwords.  bounds(i) returns the window
// parameters of load slot i.  NOISE needs the pooled scratch.
template <int W, bool NS, int MODE, class Bounds>
__device__ __forceinline__ void i8_replace(const StreamView& d, int64_t first, uint64_t seed,
                                           I8TileSmem<W, NS>& sm, uint32_t (&v)[16], Bounds bounds)
{
    if constexpr (MODE == RFI_MODE_CLIP) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const WinParams p = bounds(i);
            const uint32_t lo = rep_i16(p.lo * 256), hi = rep_i16(p.hi * 256);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[4 * i + j] = clamp_i8x4(v[4 * i + j], lo, hi);
                sched_fence();
            }
        }
    } else if constexpr (MODE == RFI_MODE_ZERO) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const WinParams p = bounds(i);
            const uint32_t lo_u = rep_i16((p.lo + 128) * 256), hi_u = rep_i16((p.hi + 128) * 256);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[4 * i + j] = byte_perm(0u, v[4 * i + j], flag_sel_i8x4(v[4 * i + j], lo_u, hi_u));
                sched_fence();
            }
        }
    } else {
        static_assert(NS, "noise needs its LDS scratch");
        uint32_t cf = 0;  // bit 4i + j: dword j of slot i holds a flagged sample
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const WinParams p = bounds(i);
            const uint32_t lo4 = rep_i8(p.lo + 128), hi4 = rep_i8(p.hi + 128), span4 = 4u * (uint32_t)(p.hi - p.lo);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                cf |= (outside_i8x4(v[4 * i + j], lo4, hi4, span4) ? 1u : 0u) << (4 * i + j);
            sched_fence();
        }
        if constexpr (NS) {
            const int64_t abs0 = d.abs_base + first;
            const uint32_t key1 = d.key;
            auto merged = [&](int wv, int ln, int slot, int part, uint32_t x) -> uint32_t {
                const int off = wv * 4096 + slot * 1024 + ln * 16 + part * 4;
                const WinParams p = sm.prm[off / W];
                const uint32_t lo_u = rep_i16((p.lo + 128) * 256), hi_u = rep_i16((p.hi + 128) * 256);
                const uint32_t nz = noise_quad_i8((uint64_t)(abs0 + off), seed, key1, p.m, p.sq8);
                return byte_perm(nz, x, flag_sel_i8x4(x, lo_u, hi_u));
            };
            pool_noise(v, cf, sm.noise(), merged);
        }
    }
}

// Median bin mb (median + 128) and MAD D of the wide windows (W >= 4096) of
// a tile, from each wave's own histogram of its 4 KiB.  pc: the window's
// padded cumulative counts.  W 16384: mb, D and pc are wave 0's alone.
template <int W, bool NS>
__device__ __forceinline__ void i8_wide_tile_select(I8TileSmem<W, NS>& sm, const uint32_t (&v)[16], int& mb, int& D,
                                                    uint32_t*& pc)
{
    using Smem = I8TileSmem<W, NS>;
    constexpr uint32_t need = (W - 1) / 2 + 1;
    constexpr int WPW = Smem::kWPW;
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    const int wl = wave / WPW;
    uint32_t* h = sm.hist + wave * kWaveHistWords;
    if constexpr (WPW > 1) __syncthreads();  // the previous tile is done with tot and prm
    wide_hist_zero(h);
    wave_sync();
    uint32_t* hl = h + (lane & 3) * kRepStride;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        wide_hist_add(hl, v[q]);
        sched_fence();
    }
    wave_sync();
    uint32_t c[4];
    wide_hist_totals(h, c);
    // The cumulative counts overwrite replica 0 of the selecting wave,
    // whose reads were all issued above.
    pc = h;
    if constexpr (WPW == 2) {
        // W 8192: both waves publish their totals; after one barrier each
        // wave adds its window's two and selects by itself (the same
        // values in both, no second exchange).
        *reinterpret_cast<uint4*>(sm.tot + wave * 256 + lane * 4) = make_uint4(c[0], c[1], c[2], c[3]);
        __syncthreads();
        const uint4 t0 = *reinterpret_cast<const uint4*>(sm.tot + (wl * 2) * 256 + lane * 4);
        const uint4 t1 = *reinterpret_cast<const uint4*>(sm.tot + (wl * 2 + 1) * 256 + lane * 4);
        c[0] = t0.x + t1.x;
        c[1] = t0.y + t1.y;
        c[2] = t0.z + t1.z;
        c[3] = t0.w + t1.w;
    } else if constexpr (WPW == 4) {
        // W 16384: the four waves' totals are added in LDS and one wave
        // selects (selecting in all four measured slower).
        if (threadIdx.x < 64) reinterpret_cast<uint4*>(sm.tot)[threadIdx.x] = make_uint4(0, 0, 0, 0);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) atomicAdd(&sm.tot[lane * 4 + j], c[j]);
        __syncthreads();
        if (wave == 0) {
            const uint4 t = *reinterpret_cast<const uint4*>(sm.tot + lane * 4);
            c[0] = t.x;
            c[1] = t.y;
            c[2] = t.z;
            c[3] = t.w;
        }
    }
    mb = D = 0;
    if (WPW < 4 || wave == 0) wide_select(c, pc, need, mb, D);
}

// Six consecutive counts of a wave's 2048 samples u (8 dwords per lane,
// biased bytes): e[j] = 2 #{u > t + j}, 0 <= t, t + 6 <= 255.
//
// |u - t| - |u - t - 1| is 1 for u > t and -1 otherwise, so the difference of
// two neighbouring sums of distances, one v_sad_u8 per dword each, counts
// the samples above t.
__device__ __forceinline__ void sad_counts(const uint32_t (&u)[8], int t, uint32_t (&e)[6])
{
    uint32_t S[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        S[j] = 32u * (uint32_t)(6 - j);  // each difference gains 32: 2 #{u > t} of 32 samples, never negative
        const uint32_t t4 = (uint32_t)__builtin_amdgcn_readfirstlane((int)rep_i8(t + j));
#pragma unroll
        for (int q = 0; q < 8; ++q) S[j] = __builtin_amdgcn_sad_u8(u[q], t4, S[j]);
    }
#pragma unroll
    for (int j = 0; j < 6; ++j) e[j] = S[j] - S[j + 1];
}

// Sums over the wave of six per-lane values of at most 64 each, two to a
// register (sums of at most 4096 fit 16 bits).
__device__ __forceinline__ void wave_sums6(const uint32_t (&e)[6], int (&sum)[6])
{
#pragma unroll
    for (int j = 0; j < 6; j += 2) {
        const uint32_t t = (uint32_t)__builtin_amdgcn_readlane((int)group_incl_scan<64>(e[j] | e[j + 1] << 16), 63);
        sum[j] = (int)(t & 0xFFFFu);
        sum[j + 1] = (int)(t >> 16);
    }
}

// Median bin and MAD of a 4096-sample window from half the atomics, for the
// statistics-only pass, which nothing but the histogram's LDS atomics bounds
// (its samples are read once and not written).  Half of the window's samples
// are counted into the histogram; its median and MAD are within a value or
// two of the window's.  The other half is counted at the six values around
// each place that decides the result, the median and m + D and m - D, by
// sums of distances, and added to the histogram's cumulative counts there.
// False if the result is not among those values; the counts are then taken
// from all samples.  60 x 2^21 samples: 44 -> 32 us (3.9 TB/s read), 60 x
// 2^20 23.6 -> 18.  Only for W 4096, whose window is one wave's: the narrow
// classes have other histograms, and the waves of a W 8192 or 16384 window
// would have to add up their counts twice more between barriers (not tried).
template <bool NS>
__device__ __forceinline__ bool i8_stats_select_4096(I8TileSmem<4096, NS>& sm, const uint32_t (&v)[16], int& mb_out,
                                                     int& D_out)
{
    constexpr int need = 2048;  // rank floor((4096 - 1) / 2), 1-based
    const int lane = lane_id();
    uint32_t* h = sm.hist + (threadIdx.x >> 6) * kWaveHistWords;
    wide_hist_zero(h);
    wave_sync();
    uint32_t* hl = h + (lane & 3) * kRepStride;
    // the first two dwords of every 16 bytes: both halves see the same signal
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        wide_hist_add(hl, v[4 * (q >> 1) + (q & 1)]);
        sched_fence();
    }
    wave_sync();
    uint32_t c[4];
    wide_hist_totals(h, c);
    int m, D;
    wide_select(c, h, 1024, m, D);
    m = __builtin_amdgcn_readfirstlane(m);
    D = __builtin_amdgcn_readfirstlane(D);
    const uint32_t* C = h + 4;  // cumulative counts of the histogram's half
    uint32_t u[8], e[6];
    int s[6];
#pragma unroll
    for (int q = 0; q < 8; ++q) u[q] = v[4 * (q >> 1) + 2 + (q & 1)] ^ 0x80808080u;
    // The median: the first value whose count reaches the rank, among the
    // five above t.
    const int t = m - 3;
    if (t < 0 || t + 6 > 255) return false;
    sad_counts(u, t, e);
    wave_sums6(e, s);
    int cv = (int)C[min(t + lane, 255)];
    int below = 0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        s[j] = __builtin_amdgcn_readlane(cv, j) + 2048 - (s[j] >> 1);
        below += s[j] < need ? 1 : 0;
    }
    if (below == 0 || below == 6) return false;
    m = t + below;
    // The MAD: the first d with C(m + d) - C(m - d - 1) >= need, among d0 ..
    // d0 + 5.
    const int d0 = max(D - 3, 0);
    const int hi = m + d0, lo = m - d0 - 6;  // lo + 5 - j goes with hi + j
    if (lo < 0 || hi + 6 > 255) return false;
    uint32_t el[6];
    sad_counts(u, lo, el);
    sad_counts(u, hi, e);
#pragma unroll
    for (int j = 0; j < 6; ++j) e[j] = el[5 - j] - e[j];
    wave_sums6(e, s);
    cv = (int)C[min(hi + lane, 255)] - (int)C[max(lo + 5 - lane, 0)];
    below = 0;
#pragma unroll
    for (int j = 0; j < 6; ++j) below += __builtin_amdgcn_readlane(cv, j) + (s[j] >> 1) < need ? 1 : 0;
    if (below == 6 || (below == 0 && d0 > 0)) return false;
    mb_out = m;
    D_out = d0 + below;
    return true;
}

// Processes one int8 tile whose samples this lane already holds in v
// (tile_load), stores the output, and returns the statistics record this
// lane must write (see write_stats).
template <int W, bool NS, int MODE>
__device__ __forceinline__ TileStats i8_tile(const StreamView& d, int64_t first, uint64_t seed,
                                             I8TileSmem<W, NS>& sm, uint32_t (&v)[16])
{
    using Smem = I8TileSmem<W, NS>;
    constexpr uint32_t need = (W - 1) / 2 + 1;
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    const int wbase = wave * 4096;
    TileStats ts;
    ts.dst = nullptr;

    if constexpr (Smem::kWide) {
        constexpr int WPW = Smem::kWPW;
        const int wl = wave / WPW;
        uint32_t* pc;
        int mb, D;
        WinParams p;
        rfi_window_stats ws;
        if constexpr (W == 4096 && MODE == kModeStats) {
            if (i8_stats_select_4096(sm, v, mb, D)) {
                // flag count and threshold are the replacement pass's
                ws.median = mb - 128;
                ws.mad = D;
                ws.n_flagged = 0;
                ws.threshold = 0.0f;
                p.m = ws.median;
            } else {
                wave_sync();  // the histogram is taken again
                i8_wide_tile_select(sm, v, mb, D, pc);
                wide_params(pc, mb, D, d.k, W, p, ws);
            }
        } else {
            i8_wide_tile_select(sm, v, mb, D, pc);
            if (WPW < 4 || wave == 0) wide_params(pc, mb, D, d.k, W, p, ws);
        }
        if (wave % WPW == 0) {
            if (lane == 0) {
                sm.prm[wl] = p;
                if constexpr (MODE == kModeStats) {
                    sm.mad[wl] = D;
                    if (d.mads) gstore(d.mads + first / W + wl, (uint8_t)D);
                }
            }
            ts.s = ws;
            ts.dst = (lane == 0 && d.stats) ? d.stats + first / W + wl : nullptr;
        }
        if constexpr (WPW == 4) {
            __syncthreads();
            p = sm.prm[0];
        }
        // The record is complete: write it now rather than keep it in
        // registers through the replacement (the noise draws' peak).
        write_stats(ts);
        ts.dst = nullptr;
        if constexpr (MODE != kModeStats) i8_replace<W, NS, MODE>(d, first, seed, sm, v, [&](int) { return p; });
    } else {
        // Several windows per wave: one 256-bin histogram of x + 128 per
        // window, or per two windows (Smem::kPair) in the halves of its bins.
        constexpr int NWW = 4096 / W;            // windows per wave
        constexpr bool PAIR = Smem::kPair;
        constexpr int NH = PAIR ? NWW / 2 : NWW;  // histograms per wave
        constexpr int GA = 64 / NH;               // lanes per histogram in the scan
        constexpr int G = 64 / NWW;               // lanes per window in the search
        uint32_t* hwave = sm.hist + wave * NH * kNarrowStride;
        // A load's 1 KiB lies in at most two windows, so counting load i in
        // step i would send 32 or 64 lanes of a wave to one histogram and
        // serialise their same-bin atomics.  Lane groups count the loads in
        // rotated order instead (lanes 8g .. 8g+7 mod 32 start at load g), so
        // each step spreads the wave over more histograms.  The rotation uses
        // masked selects with opaque masks, so it stays bit-field inserts
        // instead of becoming a per-lane indexed read.
        const int g = (lane >> 3) & 3;
        uint32_t m1 = (g & 1) ? ~0u : 0u, m2 = (g & 2) ? ~0u : 0u;
        asm volatile("" : "+v"(m1), "+v"(m2));
#pragma unroll
        for (int j = 0; j < NH; ++j)
            reinterpret_cast<uint4*>(hwave + j * kNarrowStride)[lane] = make_uint4(0, 0, 0, 0);
        wave_sync();
        uint32_t q[16], q2[16];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) q2[4 * t + j] = bit_select(m1, v[4 * ((t + 1) & 3) + j], v[4 * t + j]);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) q[4 * t + j] = bit_select(m2, q2[4 * ((t + 2) & 3) + j], q2[4 * t + j]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int li = (t + g) & 3;
            const int win = (li * 1024 + lane * 16) / W;  // of the wave
            uint32_t* hh = hwave + (PAIR ? win >> 1 : win) * kNarrowStride;
            const uint32_t one = PAIR ? ((win & 1) ? 0x10000u : 1u) : 1u;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t u = nphys4<GA>(q[4 * t + j] ^ 0x80808080u);
                atomicAdd(&hh[u & 0xFFu], one);
                atomicAdd(&hh[(u >> 8) & 0xFFu], one);
                atomicAdd(&hh[(u >> 16) & 0xFFu], one);
                atomicAdd(&hh[u >> 24], one);
                sched_fence();
            }
        }
        wave_sync();
        const int wl = wave * NWW + lane / G;
        uint32_t* hw = hwave + (lane / GA) * kNarrowStride;
        const int shift = PAIR ? (lane & G ? 16 : 0) : 0;
        int mb, D;
        if constexpr (PAIR) select_i8_pair<GA>(hw, shift, need, mb, D);
        else select_i8<GA>(hw, need, mb, D);
        WinParams p;
        rfi_window_stats ws;
        params_i8([&](int v) { return PAIR ? pair_count<GA>(hw, shift, v) : hw[nphys<GA>(v)]; }, mb, D, d.k, W, p, ws);
        if ((lane & (G - 1)) == 0) {
            sm.prm[wl] = p;
            if constexpr (MODE == kModeStats) {
                sm.mad[wl] = D;
                if (d.mads) gstore(d.mads + first / W + wl, (uint8_t)D);
            }
            ts.s = ws;
            ts.dst = d.stats ? d.stats + first / W + wl : nullptr;
        }
        wave_sync();
        write_stats(ts);
        ts.dst = nullptr;
        if constexpr (MODE != kModeStats)
            i8_replace<W, NS, MODE>(d, first, seed, sm, v, [&](int i) {
                return sm.prm[(wbase + i * 1024 + lane * 16) / W];
            });
    }

    if constexpr (MODE != kModeStats) {
        uint8_t* yt = static_cast<uint8_t*>(d.y) + first + wbase + lane * 16;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            gstore16_nt(yt + i * 1024, make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]));
    }
    return ts;
}

// Mode dispatch: MODES is the set (bit m = mode m) compiled into a kernel.
template <int W, bool NS, int MODES>
__device__ __forceinline__ TileStats i8_tile_any(const StreamView& d, int64_t first, uint64_t seed,
                                                 I8TileSmem<W, NS>& sm, uint32_t (&v)[16])
{
    static_assert(!(MODES & 4) || NS, "noise needs its LDS scratch");
    if constexpr (MODES == (1 << kModeStats)) {
        return i8_tile<W, false, kModeStats>(d, first, seed, sm, v);
    } else if constexpr (MODES == 1) {
        return i8_tile<W, NS, RFI_MODE_ZERO>(d, first, seed, sm, v);
    } else if constexpr (MODES == 2) {
        return i8_tile<W, NS, RFI_MODE_CLIP>(d, first, seed, sm, v);
    } else if constexpr (MODES == 4) {
        return i8_tile<W, NS, RFI_MODE_NOISE>(d, first, seed, sm, v);
    } else {
        if ((MODES & 2) && d.mode == RFI_MODE_CLIP) return i8_tile<W, NS, RFI_MODE_CLIP>(d, first, seed, sm, v);
        if ((MODES & 1) && d.mode == RFI_MODE_ZERO) return i8_tile<W, NS, RFI_MODE_ZERO>(d, first, seed, sm, v);
        if constexpr ((MODES & 4) != 0) return i8_tile<W, NS, RFI_MODE_NOISE>(d, first, seed, sm, v);
        TileStats none;
        none.dst = nullptr;
        return none;
    }
}

// ---------------------------------------------------------------------------
// int8 generic window: any length, any alignment, optional head segment.
// ---------------------------------------------------------------------------
// Scratch of a workgroup that holds kBlock / NT windows of NT threads each.
template <int NT>
struct I8WinSmem {
    static constexpr int PER = kBlock / NT;
    union {
        uint32_t hist[256];                                // two-pass path
        __align__(16) uint32_t whist[4 * kWaveHistWords];  // per-wave replicated histograms
    };
    WinParams prm[PER];
    int64_t j0[PER];     // absolute index of each window's first chunk
    uint32_t key[PER];   // and its stream's Philox key word
    uint32_t noise_counts[4];
    __device__ NoiseScratch noise()
    {
        return NoiseScratch{noise_counts, whist, reinterpret_cast<uint4*>(whist + 256)};
    }
};
using GenericSmem = I8WinSmem<kBlock>;

__device__ __forceinline__ uint32_t byte_of(uint32_t v, int b) { return (v >> (8 * b)) & 0xFFu; }

// Whether a window qualifies for i8_window in a launch of windows of any kind:
// not a short one, 16-byte aligned input and output, no head segment (HEAD: or one of whole chunks, as a serving
// stream's carry whose blocks start and end on 16 samples), at most K chunks
// per thread.  NOISE: noise windows too, where each dword of the
// stream holds one Philox block (absolute index of the stream's first
// sample a multiple of 4).
template <bool NOISE, int NT, int K, bool HEAD>
__device__ __forceinline__ bool i8_window_ok(const StreamView& d, int64_t a, int n)
{
    if (n < 512) return false;
    if (d.head_len != 0 && (!HEAD || ((d.head_len | (uint32_t)(uintptr_t)d.x_head) & 15u) != 0)) return false;
    if (d.mode == RFI_MODE_NOISE && (!NOISE || (d.abs_base & 3) != 0)) return false;
    if (((uintptr_t)d.x | (uintptr_t)d.y) & 15u) return false;
    // the last chunk may reach up to 15 bytes past the window: inside the
    // stream, or inside the packed layout's padding
    if (!d.padded && ((a + n + 15) & ~(int64_t)15) > d.length) return false;
    return ((a + n + 15) >> 4) - (a >> 4) <= K * NT;
}

// One window [a, a + n) in registers, by the NT threads `tid` of the
// workgroup's window `sub` (n = 0: no window, which takes part in the
// barriers).  The 16-byte chunks covering it are loaded, K per thread,
// and counted into per-wave replicated histograms; the samples of the edge
// chunks outside the window are counted as the largest value and taken out
// of its count again.  The counts are summed and selected as the wide tiles
// do; whole chunks are stored as one, the dwords and bytes of the edge
// chunks one by one, so that a neighbouring window's bytes are never
// written.
//
// The flagged dwords of every window of the workgroup are pooled for the
// draws.  With one window per workgroup of 64 or 128 threads, a window of
// 5000 samples took a wave's draws for its 28 flagged dwords, one of 1000
// for its 6.
//
// MODES: bit m set if the launch has windows in mode m (one bit: the mode is
// fixed at compile time).
template <int NT, int K, int MODES, bool HEAD>
__device__ __forceinline__ void i8_window(const StreamView& d, int64_t w, int64_t a, int n, uint64_t seed, int sub,
                                          int tid, I8WinSmem<NT>& sm)
{
    constexpr bool NOISE = (MODES & 4) != 0;
    const int mode = MODES == 1   ? RFI_MODE_ZERO
                     : MODES == 2 ? RFI_MODE_CLIP
                     : MODES == 4 ? RFI_MODE_NOISE
                     : MODES == 8 ? kModeStats
                                  : d.mode;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // of the workgroup
    const int lead = (int)(a & 15);
    const int nch = n > 0 ? (lead + n + 15) >> 4 : 0;
    const int tail = ((lead + n - 1) & 15) + 1;
    const int64_t base = a - lead;  // first byte of chunk 0
    const uint8_t* xb = static_cast<const uint8_t*>(d.x) + base;
    const bool edges = lead != 0 || tail != 16;
    uint32_t v[4 * K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int c = tid + i * NT;
        uint4 t = make_uint4(0, 0, 0, 0);
        if (c < nch) {
            const uint8_t* at = xb + c * 16;
            if constexpr (HEAD) {
                const int64_t p = base + c * 16;
                at = p < d.head_len ? static_cast<const uint8_t*>(d.x_head) + p : at - d.head_len;
            }
            t = gload16_nt(at);
        }
        v[4 * i] = t.x;
        v[4 * i + 1] = t.y;
        v[4 * i + 2] = t.z;
        v[4 * i + 3] = t.w;
    }
    if constexpr (NT == kBlock) __syncthreads();  // the previous item is done with the scratch
    uint32_t* h = sm.whist + wave * kWaveHistWords;
    wide_hist_zero(h);
    wave_sync();
    uint32_t* hl = h + (lane & 3) * kRepStride;
    // bytes of dword j of chunk c that belong to the window
    auto inside = [&](int c, int j) -> uint32_t {
        const int f = (c == 0 ? lead : 0) - 4 * j, e = (c == nch - 1 ? tail : 16) - 4 * j;
        const uint32_t lo = f <= 0 ? ~0u : f >= 4 ? 0u : ~0u << (8 * f);
        const uint32_t hi = e >= 4 ? ~0u : e <= 0 ? 0u : (1u << (8 * e)) - 1u;
        return lo & hi;
    };
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int c = tid + i * NT;
        if (c < nch) {
            uint32_t x[4] = {v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]};
            if (edges && (c == 0 || c == nch - 1)) {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = bit_select(inside(c, j), x[j], 0x7F7F7F7Fu);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                wide_hist_add(hl, x[j]);
                sched_fence();
            }
        }
    }
    wave_sync();
    uint32_t cnt[4];
    wide_hist_totals(h, cnt);
    const int wv = NT == 64 ? 0 : wave & (NT / 64 - 1);  // wave of the window
    if constexpr (NT > 64) {
        // Each wave leaves its totals in its second replica, which only it
        // has read.  Two waves both add and select (no second exchange);
        // four leave that to the first.
        *reinterpret_cast<uint4*>(h + kRepStride + 4 * lane) = make_uint4(cnt[0], cnt[1], cnt[2], cnt[3]);
        __syncthreads();
        if (NT == 128 || wv == 0) {
            const uint32_t* t0 = sm.whist + (wave - wv) * kWaveHistWords + kRepStride + 4 * lane;
            cnt[0] = cnt[1] = cnt[2] = cnt[3] = 0;
#pragma unroll
            for (int q = 0; q < NT / 64; ++q) {
                const uint4 t = *reinterpret_cast<const uint4*>(t0 + q * kWaveHistWords);
                cnt[0] += t.x;
                cnt[1] += t.y;
                cnt[2] += t.z;
                cnt[3] += t.w;
            }
        }
    }
    WinParams p;
    if (n > 0 && (NT <= 128 || wv == 0)) {
        if (lane == 63) cnt[3] -= (uint32_t)(nch * 16 - n);  // the edge chunks' other samples
        int mb, D;
        rfi_window_stats s;
        // the cumulative counts take the place of the wave's first replica
        wide_select(cnt, h, (uint32_t)((n - 1) / 2 + 1), mb, D);
        wide_params(h, mb, D, d.k, n, p, s);
        if (lane == 0 && wv == 0) {
            if (NOISE || NT == kBlock) sm.prm[sub] = p;
            if (d.stats) d.stats[w] = s;
            if (mode == kModeStats && d.mads) gstore(d.mads + w, (uint8_t)D);
            if constexpr (NOISE) {
                sm.j0[sub] = d.abs_base + base;
                sm.key[sub] = d.key;
            }
        }
    }
    if constexpr (NT == kBlock) {
        __syncthreads();
        p = sm.prm[0];
    }
    const uint32_t lo = rep_i16(p.lo * 256), hi = rep_i16(p.hi * 256);
    const uint32_t lo_u = rep_i16((p.lo + 128) * 256), hi_u = rep_i16((p.hi + 128) * 256);
    const bool noise = NOISE && mode == RFI_MODE_NOISE;
    if constexpr (NOISE) {
        const uint32_t lo4 = rep_i8(p.lo + 128), hi4 = rep_i8(p.hi + 128), span4 = 4u * (uint32_t)(p.hi - p.lo);
        uint32_t cf = 0;  // bit q: dword q holds a flagged sample
        if (noise) {
#pragma unroll
            for (int q = 0; q < 4 * K; ++q)
                if (tid + (q >> 2) * NT < nch) cf |= (outside_i8x4(v[q], lo4, hi4, span4) ? 1u : 0u) << q;
        }
        auto merged = [&](int wvs, int ln, int slot, int part, uint32_t x) -> uint32_t {
            const int s = NT == kBlock ? 0 : wvs / (NT / 64);
            const int t = NT == 64 ? ln : (wvs & (NT / 64 - 1)) * 64 + ln;
            const int64_t j0 = sm.j0[s] + (int64_t)(t + slot * NT) * 16 + 4 * part;
            const WinParams q = sm.prm[s];
            const uint32_t ql = rep_i16((q.lo + 128) * 256), qh = rep_i16((q.hi + 128) * 256);
            const uint32_t nz = noise_quad_i8((uint64_t)j0, seed, NT == kBlock ? d.key : sm.key[s], q.m, q.sq8);
            return byte_perm(nz, x, flag_sel_i8x4(x, ql, qh));
        };
        static_assert(sizeof(sm.whist) >= kNoiseAliasWords * 4, "noise list in the histograms");
        // every thread of the workgroup, whatever its window's mode
        pool_noise(v, cf, sm.noise(), merged);
    }
    if (mode == kModeStats) return;
    uint8_t* yb = static_cast<uint8_t*>(d.y) + base;
    const bool clip = mode == RFI_MODE_CLIP;
    // A fresh index, so that offsets and bounds are not kept over the draws
    // (64 threads of eight chunks spilled 36 bytes per lane for them, 16 % more
    // HBM traffic, now 8; noise, 60 x 2^22: W 1000 280 -> 273 us, 5000 128 ->
    // 122, 20000 112 -> 104).
    uint32_t ts = (uint32_t)tid;
    if constexpr (NOISE) pin_vgpr(ts);
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int c = (int)ts + i * NT;
        if (c >= nch) continue;
        uint32_t r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t x = v[4 * i + j];
            r[j] = noise ? x : clip ? clamp_i8x4(x, lo, hi) : byte_perm(0u, x, flag_sel_i8x4(x, lo_u, hi_u));
        }
        uint8_t* at = yb + c * 16;
        if (edges && (c == 0 || c == nch - 1)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t m = inside(c, j);
                if (m == ~0u) {
                    gstore(reinterpret_cast<uint32_t*>(at) + j, r[j]);
                } else if (m != 0) {
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        if (byte_of(m, b)) gstore(at + 4 * j + b, (uint8_t)byte_of(r[j], b));
                }
            }
        } else {
            gstore16_nt(at, make_uint4(r[0], r[1], r[2], r[3]));
        }
    }
}

// A generic window in a workgroup of NT threads: in registers if it
// qualifies, else by two passes over the samples in global memory.
// REG: zero/clip windows may stay in registers; REG_NOISE: noise windows too
// (kept out of the fused kernels, whose register budget the inlined draw
// would raise).
template <bool REG = true, bool REG_NOISE = false, int NT = kBlock, class Smem = GenericSmem>
__device__ void i8_generic(const StreamView& d, int64_t w, uint64_t seed, Smem& sm)
{
    const int W = d.window;
    const int64_t a = w * (int64_t)W;
    const int n = (int)min((int64_t)W, d.length - a);
    if constexpr (REG) {
        if (i8_window_ok<REG_NOISE, NT, 4, true>(d, a, n)) {
            i8_window<NT, 4, REG_NOISE ? 15 : 11, true>(d, w, a, n, seed, 0, (int)threadIdx.x, sm);
            return;
        }
    }
    const int tid = (int)threadIdx.x;
    int8_t* y = static_cast<int8_t*>(d.y);
    __syncthreads();
    for (int i = tid; i < 256; i += NT) sm.hist[i] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += NT) atomicAdd(&sm.hist[load_logical<int8_t>(d, a + i) + 128], 1u);
    __syncthreads();
    if (tid < 64) {
        int mb, D;
        select_i8<64>(sm.hist, (uint32_t)((n - 1) / 2 + 1), mb, D);
        WinParams p;
        rfi_window_stats s;
        params_i8([&](int v) { return sm.hist[v]; }, mb, D, d.k, n, p, s);
        if (tid == 0) {
            sm.prm[0] = p;
            if (d.stats) d.stats[w] = s;
            if (d.mode == kModeStats && d.mads) gstore(d.mads + w, (uint8_t)D);
        }
    }
    __syncthreads();
    if (d.mode == kModeStats) return;
    const WinParams p = sm.prm[0];
    for (int i = tid; i < n; i += NT) {
        const int x = load_logical<int8_t>(d, a + i);
        int yv = x;
        if (x < p.lo || x > p.hi) {
            if (d.mode == RFI_MODE_ZERO) yv = 0;
            else if (d.mode == RFI_MODE_CLIP) yv = min(max(x, p.lo), p.hi);
            else yv = noise_sample(d.abs_base + a + i, seed, d.key, p.m, p.sq8, -128, 127);
        }
        gstore(y + a + i, (int8_t)yv);
    }
}

// ---------------------------------------------------------------------------
// Kernels.  Those with a PERSIST parameter serve launches of one workgroup per
// item and, with a grid-stride loop over the items, persistent ones.
// ---------------------------------------------------------------------------
// One or two tiles per workgroup.  With two, the second tile's loads are
// issued before the first tile is processed, so they are in flight while
// the first tile's histogram, selection and replacement run.
template <int CLS, int MODES, bool PERSIST, int TPW>
__global__ __launch_bounds__(kBlock) void k_i8_tiles(LaunchArgs a)
{
    constexpr int W = 512 << CLS;
    constexpr bool NOISE = (MODES & 4) != 0;
    __shared__ I8TileSmem<W, NOISE> sm;
    if constexpr (TPW == 1) {
        for_items<PERSIST>(a, [&](int64_t it) {
            const Item item = a.items[it];
            const StreamView d = resolve(a.streams[item.stream], a);
            uint32_t v[16];
            tile_load<MODES == (1 << kModeStats)>(d, item.first, v);
            write_stats(i8_tile_any<W, NOISE, MODES>(d, item.first, a.seed, sm, v));
        });
    } else {
        const int64_t it = 2 * (int64_t)blockIdx.x;
        if (it >= a.n_items) return;
        const bool two = it + 1 < a.n_items;
        const Item ia = a.items[it];
        const Item ib = a.items[two ? it + 1 : it];
        const StreamView da = resolve(a.streams[ia.stream], a);
        const StreamView db = resolve(a.streams[ib.stream], a);
        uint32_t va[16], vb[16];
        // Both loads are unconditional (the second repeats the first tile
        // when there is no second item): a branch around them would make
        // the first tile's waits cover the second tile's loads too.
        tile_load(da, ia.first, va);
        tile_load(db, ib.first, vb);
        const TileStats sa = i8_tile_any<W, NOISE, MODES>(da, ia.first, a.seed, sm, va);
        if (two) {
            if constexpr (W > 4096) __syncthreads();
            write_stats(i8_tile_any<W, NOISE, MODES>(db, ib.first, a.seed, sm, vb));
        }
        write_stats(sa);
    }
}

// Windows of at most K * NT chunks of padded streams (plans), kBlock / NT of
// them per workgroup.  Bound by the VALU (a window's fixed work: clearing and
// adding up the replicas, the search) below 3000 samples, near HBM from
// there on.  K = 8 (windows of more than 4066 samples): half the waves per
// window, so half its fixed work, and one wave up to 8162.  60 x 2^22 samples,
// zero / clip / noise, against one window per workgroup of 64, 128 or 256
// threads with the edge chunks counted and stored byte by byte, in batches
// that fill the device (i8_window_threads has the others): W 1000 210 /
// 203 / 342 -> 172 / 167 / 273 us, 3000 121 / 114 / 176 -> 107 / 101 / 133,
// 5000 119 / 112 / 160 -> 100 / 95 / 122 (K = 4: 110 / 105 / 146), 9000 117 /
// 109 / 163 -> 100 / 96 / 127, 12000 94 / 90 / 126 -> 93 / 90 / 106.  Noise
// with K = 8: seven waves per SIMD (W 5000, before the offsets were formed again
// after the draws, 124 us; six 132, five 143).
template <int NT, int K, int MODES>
__global__ __launch_bounds__(kBlock, K == 8 && (MODES & 4) ? 7 : 8) void k_i8_windows(LaunchArgs a)
{
    __shared__ I8WinSmem<NT> sm;
    constexpr int PER = kBlock / NT;
    const int sub = __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
    const int64_t it = (int64_t)blockIdx.x * PER + sub;
    if (PER == 1 && it >= a.n_items) return;
    const bool has = it < a.n_items;
    const Item item = a.items[has ? it : 0];
    const StreamView d = resolve(a.streams[item.stream], a);
    const int64_t first = item.first * (int64_t)d.window;
    const int n = has ? (int)min((int64_t)d.window, d.length - first) : 0;
    i8_window<NT, K, MODES, false>(d, item.first, first, n, a.seed, sub, (int)threadIdx.x & (NT - 1), sm);
}

// Short windows (i8_short_windows) of any kind of stream, one wave each.
struct I8ShortSmem {
    __align__(16) uint32_t hist[256];
    WinParams prm[1];
};
__global__ __launch_bounds__(64) void k_i8_short(LaunchArgs a)
{
    __shared__ I8ShortSmem sm;
    if ((int64_t)blockIdx.x >= a.n_items) return;
    const Item item = a.items[blockIdx.x];
    const StreamView d = resolve(a.streams[item.stream], a);
    i8_generic<false, false, 64>(d, item.first, a.seed, sm);
}

// NOISE: noise windows may take the register path (launched only for items
// that include noise streams: the draw costs registers the other modes'
// small windows would pay for in occupancy).
template <bool PERSIST, bool NOISE>
__global__ __launch_bounds__(kBlock, NOISE ? (PERSIST ? 4 : 8) : 0) void k_i8_generic(LaunchArgs a)
{
    __shared__ GenericSmem sm;
    for_items<PERSIST>(a, [&](int64_t it) {
        const Item item = a.items[it];
        const StreamView d = resolve(a.streams[item.stream], a);
        i8_generic<true, NOISE>(d, item.first, a.seed, sm);
    });
}

template <bool NS>
union I8FusedSmem {
    I8TileSmem<512, NS> c0;
    I8TileSmem<1024, NS> c1;
    I8TileSmem<2048, NS> c2;
    I8TileSmem<4096, NS> c3;
    I8TileSmem<8192, NS> c4;
    I8TileSmem<16384, NS> c5;
    GenericSmem g;
};

// Generic items of the all-modes fused kernel, which is too large for the
// compiler to inline the generic path: out of line, taking the descriptor's
// address and the launch's base addresses as scalars and resolving the
// stream itself.  Handing over the resolved stream (by reference, or by
// value, which the calling convention also passes through memory) made
// the caller store it to private memory before every item, tiles included:
// about 5 KiB of writes per wave.
template <bool REG, class Smem>
__device__ __noinline__ void i8_generic_item(const StreamDesc* sd, uint64_t x_base, uint64_t y_base,
                                             uint64_t stats_base, int32_t no_stats, int64_t w, uint64_t seed,
                                             Smem& sm)
{
    LaunchArgs la;
    la.x_base = x_base;
    la.y_base = y_base;
    la.stats_base = stats_base;
    la.no_stats = no_stats;
    la.mad_base = 0;
    const StreamView d = resolve(*sd, la);
    i8_generic<REG>(d, w, seed, sm);
}

// Every item kind and window class in one launch.  MODES: the modes of the
// launch's tiles (a kernel compiled for one mode needs fewer registers than
// one that branches over all three, and registers bound its occupancy);
// generic items take any mode.  The all-modes instance is bounded to four
// workgroups per CU (120 VGPRs, against 132 and three workgroups unbounded,
// a count set by the out-of-line generic item, which under the bound saves
// four callee-saved registers to private memory): on the 64-stream mixed
// batch 0.232 -> 0.214 ms in one launch; five workgroups (96 VGPRs)
// spilled in the tile code and lost it again.
// The one-mode instances keep the unbounded budget, which measured faster
// than five or seven workgroups per CU.
template <bool PERSIST, int MODES>
__global__ __launch_bounds__(kBlock, MODES == 7 ? 4 : 0) void k_i8_fused(LaunchArgs a)
{
    constexpr bool NS = (MODES & 4) != 0;
    __shared__ I8FusedSmem<NS> sm;
    for_items<PERSIST>(a, [&](int64_t it) {
        const Item item = a.items[it];
        if (item.kind == kItemCarry) {
            carry_copy(a.carries[item.stream]);
            return;
        }
        if constexpr (MODES == 7) {
            if (item.kind == kItemGeneric) {
                i8_generic_item<true>(a.streams + item.stream, a.x_base, a.y_base, a.stats_base, a.no_stats,
                                      item.first, a.seed, sm.g);
                return;
            }
        }
        const StreamView d = resolve(a.streams[item.stream], a);
        if (item.kind == kItemGeneric) {
            i8_generic<(MODES & 3) != 0>(d, item.first, a.seed, sm.g);
            return;
        }
        // Items of different classes may follow each other: keep the LDS
        // of the previous item alive until every wave is done with it.
        __syncthreads();
        uint32_t v[16];
        tile_load(d, item.first, v);
        switch (i8_tile_class(d.window)) {
            case 0: write_stats(i8_tile_any<512, NS, MODES>(d, item.first, a.seed, sm.c0, v)); break;
            case 1: write_stats(i8_tile_any<1024, NS, MODES>(d, item.first, a.seed, sm.c1, v)); break;
            case 2: write_stats(i8_tile_any<2048, NS, MODES>(d, item.first, a.seed, sm.c2, v)); break;
            case 3: write_stats(i8_tile_any<4096, NS, MODES>(d, item.first, a.seed, sm.c3, v)); break;
            case 4: write_stats(i8_tile_any<8192, NS, MODES>(d, item.first, a.seed, sm.c4, v)); break;
            default: write_stats(i8_tile_any<16384, NS, MODES>(d, item.first, a.seed, sm.c5, v)); break;
        }
    });
}

// ---------------------------------------------------------------------------
// Several outputs from one read (int8 tiles): the tile's windows are
// selected once (statistics-only mode), then each output's parameters
// (its own k) are derived from the window's median and MAD and its
// replacement (its own mode) is applied to a copy of the tile and stored.
// Output o is the same as a single call with that output's k and mode.
// ---------------------------------------------------------------------------
// Wide windows (W >= 4096): every wave holds one window or a part of one, and
// an output's parameters and its flag count are read off the window's
// cumulative counts, so the outputs follow each other without a barrier, a
// count of flagged samples or a table of parameters.  60 x 2^22 samples, W
// 4096, three outputs: 198 us with those, 182 without (the bytes moved take
// 164 at the copy rate).
template <int CLS>
__global__ __launch_bounds__(kBlock, CLS == 3 ? 8 : 7) void k_i8_multi_wide(MultiArgs ma)
{
    constexpr int W = 512 << CLS;
    using Smem = I8TileSmem<W, false>;
    constexpr int WPW = Smem::kWPW;
    __shared__ Smem sm;
    const LaunchArgs& a = ma.a;
    const Item item = a.items[blockIdx.x];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t v[16];
    tile_load(resolve(a.streams[item.stream], a), item.first, v);
    int mb, D;
    uint32_t* pc;
    i8_wide_tile_select(sm, v, mb, D, pc);
    if constexpr (WPW == 4) {
        if (threadIdx.x == 0) {
            sm.prm[0].m = mb;
            sm.mad[0] = D;
        }
        __syncthreads();
        mb = sm.prm[0].m;
        D = sm.mad[0];
        pc = sm.hist;
    }
    const int64_t off = item.first + wave * 4096 + lane * 16;
#pragma unroll 1
    for (int o = 0; o < ma.n_out; ++o) {
        const StreamDesc& sd = ma.desc[o][item.stream];
        WinParams p;
        rfi_window_stats s;
        wide_params(pc, mb, D, sd.k, W, p, s);
        if (lane == 0 && wave % WPW == 0 && ma.stats_base[o] != 0) {
            TileStats ts;
            ts.s = s;
            ts.dst = reinterpret_cast<rfi_window_stats*>(ma.stats_base[o] + sd.stats_off) + item.first / W + wave / WPW;
            write_stats(ts);
        }
        uint8_t* yt = reinterpret_cast<uint8_t*>(ma.y_base[o] + sd.y_off) + off;
        const uint32_t lo = rep_i16(p.lo * 256), hi = rep_i16(p.hi * 256);
        const uint32_t lo_u = rep_i16((p.lo + 128) * 256), hi_u = rep_i16((p.hi + 128) * 256);
        const bool clip = sd.mode == RFI_MODE_CLIP;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t r[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // opaque: the parts of the replacement that no output
                // changes are not kept in registers over the loop
                uint32_t x = v[4 * i + j];
                pin_vgpr(x);
                r[j] = clip ? clamp_i8x4(x, lo, hi) : byte_perm(0u, x, flag_sel_i8x4(x, lo_u, hi_u));
            }
            gstore16_nt(yt + i * 1024, make_uint4(r[0], r[1], r[2], r[3]));
        }
    }
}

// Narrow windows: the flags are counted, since the histograms of one round of
// windows make room for the next.
template <int W>
struct I8MultiSmem {
    I8TileSmem<W, false> t;
    int32_t med[16384 / W];
    float thr[16384 / W];
    uint32_t nfl[16384 / W];
};

// Zero and clip outputs only: a noise output would keep a second copy of
// the tile and the pooled draws in registers, which costs more occupancy
// than a second read of the input (noise outputs are separate passes).
template <int CLS>
__global__ __launch_bounds__(kBlock) void k_i8_multi(MultiArgs ma)
{
    constexpr int W = 512 << CLS;
    constexpr int kWin = 16384 / W;
    __shared__ I8MultiSmem<W> sm;
    const LaunchArgs& a = ma.a;
    const Item item = a.items[blockIdx.x];
    const int tid = (int)threadIdx.x, lane = lane_id();
    const int wbase = (tid >> 6) * 4096;
    const StreamView d0 = resolve(a.streams[item.stream], a);
    uint32_t v[16];
    tile_load(d0, item.first, v);
    (void)i8_tile<W, false, kModeStats>(d0, item.first, a.seed, sm.t, v);
    __syncthreads();
    if (tid < kWin) sm.med[tid] = sm.t.prm[tid].m;
#pragma unroll 1
    for (int o = 0; o < ma.n_out; ++o) {
        LaunchArgs ao = a;
        ao.streams = ma.desc[o];
        ao.y_base = ma.y_base[o];
        ao.stats_base = ma.stats_base[o];
        ao.no_stats = ma.stats_base[o] == 0 ? 1 : 0;
        const StreamView d = resolve(ao.streams[item.stream], ao);
        __syncthreads();  // the previous output is done with prm and the scratch
        if (tid < kWin) {
            const int m = sm.med[tid];
            float sig;
            const float t = threshold_of(sm.t.mad[tid], d.k, sig);
            const int T = (int)floorf(t);
            WinParams p;
            p.lo = max(m - T, -128);
            p.hi = min(m + T, 127);
            p.m = m;
            p.sq8 = (int)__fmul_rn(sig, 256.0f);
            sm.t.prm[tid] = p;
            sm.thr[tid] = t;
            sm.nfl[tid] = 0;
        }
        __syncthreads();
        uint8_t* yt = static_cast<uint8_t*>(d.y) + item.first + wbase + lane * 16;
        {
            // zero / clip: slot by slot, four registers at a time
            const bool clip = d.mode == RFI_MODE_CLIP;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int win = (wbase + i * 1024 + lane * 16) / W;
                const WinParams p = sm.t.prm[win];
                const uint32_t lo = rep_i16(p.lo * 256), hi = rep_i16(p.hi * 256);
                const uint32_t lo_u = rep_i16((p.lo + 128) * 256), hi_u = rep_i16((p.hi + 128) * 256);
                uint32_t r[4], nf = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t xw = v[4 * i + j];
                    pin_vgpr(xw);  // as in k_i8_multi_wide
                    const uint32_t c = clamp_i8x4(xw, lo, hi);
                    nf += __popc(nonzero_byte_mask(c ^ xw)) >> 3;
                    r[j] = clip ? c : byte_perm(0u, xw, flag_sel_i8x4(xw, lo_u, hi_u));
                }
                if (nf) atomicAdd(&sm.nfl[win], nf);
                gstore16_nt(yt + i * 1024, make_uint4(r[0], r[1], r[2], r[3]));
            }
        }
        __syncthreads();
        if (tid < kWin && d.stats) {
            rfi_window_stats st;
            st.median = sm.med[tid];
            st.mad = sm.t.mad[tid];
            st.n_flagged = sm.nfl[tid];
            st.threshold = sm.thr[tid];
            d.stats[item.first / W + tid] = st;
        }
    }
}

// ---------------------------------------------------------------------------
// Median of MAD (Eq. (3)), int8: the statistics pass leaves each window's
// MAD as a byte; each window's lower median of the MADs of its K-window
// history is found 64 windows at a time; a last pass applies Eqs. (1)-(2)
// with it.
// ---------------------------------------------------------------------------
// One wave per segment, one lane per window, 64 windows at a time.  The MADs
// [a0, p0) that precede the group's first window in its history are counted
// into a 256-value histogram; window i of the group then differs from that
// by its predecessors' and its own MAD added and by the entries from a0 on
// that its history no longer holds (for K < 64 the group's own among them),
// which for one value v are two ballots and their popcounts for all 64
// windows at once.  The medians are found by trying the values in order from
// the first that any window can reach; MADs of neighbouring windows differ
// little, so a few values do.  From group to group the histogram takes up 64
// entries and drops as many.
//
// The counts have 16 replicas (lane & 15): MADs cluster on a few values, on
// which the atomics of a wave would meet.  Latency-bound: 60 streams of 256
// windows with 4095 MADs of history 34 us before, as five kernels (gather,
// concatenate, count in blocks of 64, add up, search), 6 us now.
constexpr int kMomReps = 16;

__global__ __launch_bounds__(64) void k_mom_select(const MomStream* __restrict__ streams,
                                                   const MomSeg* __restrict__ segs, int32_t K,
                                                   const uint8_t* __restrict__ mad,
                                                   const uint8_t* __restrict__ hist,
                                                   const int32_t* __restrict__ hist_len, int32_t* __restrict__ dm)
{
    __shared__ __align__(16) uint32_t rep[256 * kMomReps];  // value v, replica r at v * 16 + r
    __shared__ __align__(16) uint32_t cum[256];             // #{entries <= v}
    const MomSeg sg = segs[blockIdx.x];
    const MomStream st = streams[sg.stream];
    const int lane = lane_id();
    const uint8_t* hs = hist ? hist + sg.stream * st.pre : nullptr;
    const uint8_t* ms = mad + st.woff;
    auto entry = [&](int64_t p) -> uint32_t { return p < st.pre ? hs[p] : ms[p - st.pre]; };
    // sequence position of the first valid entry
    const int64_t H = st.pre > 0 ? min(max((int64_t)hist_len[sg.stream], (int64_t)0), st.pre) : 0;
    const int64_t lb = st.pre - H;
    int64_t p0 = st.pre + sg.first;  // sequence position of the group's first window
    int64_t a0 = max(lb, p0 + 1 - (int64_t)K);
    for (int i = lane; i < 256 * kMomReps / 4; i += 64) reinterpret_cast<uint4*>(rep)[i] = make_uint4(0, 0, 0, 0);
    wave_sync();
    uint32_t* mine = rep + (lane & (kMomReps - 1));
    // 32 loads of a lane in flight: a history of 4096 takes two round trips
    for (int64_t p = a0 + lane; p < p0; p += 32 * 64) {
        uint32_t e[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) e[u] = p + 64 * u < p0 ? entry(p + 64 * u) : 256u;
#pragma unroll
        for (int u = 0; u < 32; ++u)
            if (e[u] < 256u) atomicAdd(mine + e[u] * kMomReps, 1u);
    }
    for (int done = 0; done < sg.n; done += 64) {
        const int n = min(64, sg.n - done);
        const bool has = lane < n;
        const int64_t p = p0 + lane;  // this lane's window
        const int64_t a = max(lb, p + 1 - (int64_t)K);
        const int gone = has ? (int)(a - a0) : 0;  // entries from a0 on that it has dropped, at most lane
        const uint32_t mine_e = has ? entry(p) : 255u;
        // lane r holds the r-th entry to be dropped
        const int dropped = __builtin_amdgcn_readlane(gone, n - 1);
        const uint32_t old_e = lane < dropped ? entry(a0 + lane) : 255u;
        const uint32_t need = (uint32_t)((p - a) / 2 + 1);  // rank floor((N - 1) / 2) of N = p + 1 - a, 1-based
        // Sums of the replicas: 4 lanes per value, 16 values at a time, then
        // cumulative counts, four values per lane.
        wave_sync();
#pragma unroll 4
        for (int i = 0; i < 16; ++i) {
            const uint4 t = reinterpret_cast<const uint4*>(rep)[i * 64 + lane];
            uint32_t c = t.x + t.y + t.z + t.w;
            c += dpp0<0xB1>(c);  // quad_perm [1, 0, 3, 2]
            c += dpp0<0x4E>(c);  // quad_perm [2, 3, 0, 1]
            if ((lane & 3) == 0) cum[i * 16 + (lane >> 2)] = c;
        }
        wave_sync();
        uint4 t = reinterpret_cast<const uint4*>(cum)[lane];
        t.y += t.x;
        t.z += t.y;
        t.w += t.z;
        const uint32_t excl = group_incl_scan<64>(t.w) - t.w;
        t.x += excl;
        t.y += excl;
        t.z += excl;
        t.w += excl;
        reinterpret_cast<uint4*>(cum)[lane] = t;
        // No window can reach its rank at values whose count is more than 64
        // below the smallest rank (ranks grow with the window index).
        const uint32_t least = (uint32_t)__builtin_amdgcn_readfirstlane((int)need);
        int v = group_count<64>(t.x + 64 < least) + group_count<64>(t.y + 64 < least) +
                group_count<64>(t.z + 64 < least) + group_count<64>(t.w + 64 < least);
        wave_sync();
        const uint64_t upto = lane == 63 ? ~0ull : (1ull << (lane + 1)) - 1;  // windows 0 .. lane
        const uint64_t first = (1ull << gone) - 1;                            // gone <= lane <= 63
        int res = 255;
        bool found = !has;
        for (; v < 255; ++v) {
            const uint64_t in = __ballot(mine_e <= (uint32_t)v), out = __ballot(old_e <= (uint32_t)v);
            const uint32_t N = cum[v] + (uint32_t)__popcll(in & upto) - (uint32_t)__popcll(out & first);
            if (!found && N >= need) {
                found = true;
                res = v;
            }
            if (__ballot(!found) == 0) break;
        }
        if (has) dm[st.woff + (p - st.pre)] = res;
        if (done + 64 < sg.n) {
            // the next group: this one's entries join, those before its start leave
            wave_sync();
            atomicAdd(mine + mine_e * kMomReps, 1u);
            const int64_t na = max(lb, p0 + 64 + 1 - (int64_t)K);
            for (int64_t q = a0 + lane; q < na; q += 64) atomicSub(mine + entry(q) * kMomReps, 1u);
            p0 += 64;
            a0 = na;
        }
    }
}

// The new right-aligned history of a stream, in place, then its length, by
// one workgroup.  Slot i takes sequence entry nw + i, so the slots move
// towards the front: a pass reads its entries before any of its slots is
// written, and later passes read only from later slots on.
__device__ __forceinline__ void mom_history(const MomHistory& h, int s)
{
    const MomStream st = h.streams[s];
    if (st.pre == 0) return;
    uint8_t* hs = h.hist + s * st.pre;
    const uint8_t* ms = h.mad + st.woff;
    const int64_t H = min(max((int64_t)h.hist_len[s], (int64_t)0), st.pre);
    const int64_t Hn = min(st.pre, H + st.nw);
    constexpr int U = 16;
    for (int64_t i0 = st.pre - Hn; i0 < st.pre; i0 += U * kBlock) {
        uint8_t e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + u * kBlock + threadIdx.x;
            const int64_t p = st.nw + i;
            e[u] = i >= st.pre ? 0 : p < st.pre ? hs[p] : ms[p - st.pre];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + u * kBlock + threadIdx.x;
            if (i < st.pre) hs[i] = e[u];
        }
        __syncthreads();
    }
    __syncthreads();  // every thread has read hist_len
    if (threadIdx.x == 0) h.hist_len[s] = (int32_t)Hn;
}

struct MomSmem {
    WinParams prm[256];
    float thr[256];
    uint32_t flagged[256];
    uint32_t noise_counts[4];
    __align__(16) uint32_t noise_list[256];
    __align__(16) uint32_t noise_data[256];
    __device__ NoiseScratch noise()
    {
        return NoiseScratch{noise_counts, noise_list, reinterpret_cast<uint4*>(noise_data)};
    }
};

// One item: up to 256 whole windows (<= 16 KiB, or one window) of a stream,
// compiled per mode (the stream's mode is uniform over the workgroup).
template <int MODE>
__device__ __forceinline__ void mom_apply_item(const LaunchArgs& a, const MomItem& it, const StreamView& d,
                                               const int32_t* __restrict__ dm,
                                               const int64_t* __restrict__ stream_woff,
                                               rfi_window_stats* __restrict__ stats, MomSmem& sm)
{
    const int tid = (int)threadIdx.x;
    const int W = d.window;
    const int64_t g0 = stream_woff[it.stream] + it.first_window;
    if (tid < it.n_windows) {
        const int m = stats[g0 + tid].median;
        float sig;
        const float t = threshold_of(dm[g0 + tid], d.k, sig);
        const int T = (int)floorf(t);
        WinParams p;
        p.m = m;
        p.lo = max(m - T, -128);
        p.hi = min(m + T, 127);
        p.sq8 = (int)__fmul_rn(sig, 256.0f);
        sm.prm[tid] = p;
        sm.thr[tid] = t;
        sm.flagged[tid] = 0;
    }
    __syncthreads();
    const int64_t s0 = it.first_window * (int64_t)W;
    const int64_t s1 = min((it.first_window + it.n_windows) * (int64_t)W, d.length);
    const int8_t* x = static_cast<const int8_t*>(d.x);
    int8_t* y = static_cast<int8_t*>(d.y);
    // Noise is drawn four samples (one Philox block) at a time where the
    // stream's dwords are whole blocks.
    const bool quads = MODE != RFI_MODE_NOISE || (d.abs_base & 3) == 0;
    if (s1 - s0 == 16384 && (W & 15) == 0 && (W & (W - 1)) == 0 && quads) {
        // A whole 16 KiB tile of windows of a power of two of samples, at
        // least 16: every 16-byte chunk lies in one window.  (Another W above
        // 16384 may end a stream with a window of 16384 samples.)  All four
        // loads of a lane are issued before any store; noise goes through the
        // workgroup pool.
        const int lane = tid & 63, wave = tid >> 6;
        const int64_t base = s0 + wave * 4096 + lane * 16;
        const int sh = __builtin_ctz((unsigned)W);
        uint32_t v[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 t = gload16_nt(x + base + i * 1024);
            v[4 * i] = t.x;
            v[4 * i + 1] = t.y;
            v[4 * i + 2] = t.z;
            v[4 * i + 3] = t.w;
        }
        uint32_t cf = 0;  // bit 4i + q: dword q of chunk i holds a flagged sample
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int lw = (wave * 4096 + i * 1024 + lane * 16) >> sh;
            const WinParams p = sm.prm[lw];
            const uint32_t lo = rep_i16(p.lo * 256), hi = rep_i16(p.hi * 256);
            const uint32_t lo_u = rep_i16((p.lo + 128) * 256), hi_u = rep_i16((p.hi + 128) * 256);
            uint32_t nf = 0;
            if constexpr (MODE == RFI_MODE_NOISE) {
                // the flags are counted where they are drawn
                const uint32_t lo4 = rep_i8(p.lo + 128), hi4 = rep_i8(p.hi + 128), span4 = 4u * (uint32_t)(p.hi - p.lo);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    cf |= (outside_i8x4(v[4 * i + q], lo4, hi4, span4) ? 1u : 0u) << (4 * i + q);
                continue;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t xw = v[4 * i + q];
                const uint32_t clipped = clamp_i8x4(xw, lo, hi);
                const uint32_t diff = clipped ^ xw;
                nf += __popc(nonzero_byte_mask(diff)) >> 3;
                cf |= (diff != 0 ? 1u : 0u) << (4 * i + q);
                if constexpr (MODE == RFI_MODE_CLIP) v[4 * i + q] = clipped;
                else if constexpr (MODE == RFI_MODE_ZERO)
                    v[4 * i + q] = byte_perm(0u, xw, flag_sel_i8x4(xw, lo_u, hi_u));
            }
            if (nf) atomicAdd(&sm.flagged[lw], nf);
        }
        if constexpr (MODE == RFI_MODE_NOISE) {
            const int64_t t0 = s0;
            auto merged = [&](int wv, int ln, int slot, int part, uint32_t xw) -> uint32_t {
                const int rel = wv * 4096 + slot * 1024 + ln * 16 + part * 4;
                const int64_t c = t0 + rel;
                const WinParams p = sm.prm[rel >> sh];
                const uint32_t lo_u = rep_i16((p.lo + 128) * 256), hi_u = rep_i16((p.hi + 128) * 256);
                const uint32_t nz = noise_quad_i8((uint64_t)(d.abs_base + c), a.seed, d.key, p.m, p.sq8);
                const uint32_t sel = flag_sel_i8x4(xw, lo_u, hi_u);
                atomicAdd(&sm.flagged[rel >> sh], (uint32_t)__popc(sel ^ 0x03020100u));  // one bit per flagged byte
                return byte_perm(nz, xw, sel);
            };
            pool_noise(v, cf, sm.noise(), merged);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            gstore16_nt(y + base + i * 1024, make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]));
    } else if (W >= 16 && quads) {
        // Other items (irregular W, stream tails): 16-byte chunks of the
        // stream, 16 KiB a pass.  A chunk holds samples of at most two of the
        // item's windows, the second from its byte t on; the edge chunks hold
        // other items' samples too, which are neither counted nor stored.
        // (The last chunk may read into the packed layout's padding.)
        const int lead = (int)(s0 & 15);
        const int64_t base = s0 - lead;
        const int len = (int)(s1 - s0);
        const float rW = __builtin_amdgcn_rcpf((float)W);
        auto window_of = [&](int rel) {  // rel / W
            int w = (int)((float)rel * rW);
            w -= w * W > rel ? 1 : 0;
            return w + ((w + 1) * W <= rel ? 1 : 0);
        };
        auto below = [](int t) -> uint32_t { return t >= 4 ? ~0u : t <= 0 ? 0u : (1u << (8 * t)) - 1u; };  // bytes < t
        const int last = it.n_windows - 1;
#pragma unroll 1
        for (int p = 0; p < lead + len; p += 16384) {
            uint32_t v[16];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = p + i * 4096 + tid * 16;
                uint4 t = make_uint4(0, 0, 0, 0);
                if (at < lead + len) t = gload16_nt(x + base + at);
                v[4 * i] = t.x;
                v[4 * i + 1] = t.y;
                v[4 * i + 2] = t.z;
                v[4 * i + 3] = t.w;
            }
            uint32_t cf = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int rel = p + i * 4096 + tid * 16 - lead;  // first sample of the chunk, from s0
                if (rel < len) {
                    const int w0 = min(window_of(max(rel, 0)), last);
                    const int w1 = min(w0 + 1, last);
                    const int t = (w0 + 1) * W - rel;
                    auto apply = [&](int w, bool second) {
                        const WinParams pw = sm.prm[w];
                        const uint32_t lo = rep_i16(pw.lo * 256), hi = rep_i16(pw.hi * 256);
                        const uint32_t lo_u = rep_i16((pw.lo + 128) * 256), hi_u = rep_i16((pw.hi + 128) * 256);
                        uint32_t nf = 0;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t xw = v[4 * i + q];
                            uint32_t mask = below(t - 4 * q);
                            if (second) mask = ~mask;
                            const uint32_t clipped = clamp_i8x4(xw, lo, hi);
                            const uint32_t diff = (clipped ^ xw) & mask & below(len - rel - 4 * q) & ~below(-rel - 4 * q);
                            nf += __popc(nonzero_byte_mask(diff)) >> 3;
                            cf |= (diff != 0 ? 1u : 0u) << (4 * i + q);
                            if constexpr (MODE == RFI_MODE_CLIP) v[4 * i + q] = bit_select(mask, clipped, xw);
                            else if constexpr (MODE == RFI_MODE_ZERO)
                                v[4 * i + q] = bit_select(mask, byte_perm(0u, xw, flag_sel_i8x4(xw, lo_u, hi_u)), xw);
                        }
                        if (nf) atomicAdd(&sm.flagged[w], nf);
                    };
                    apply(w0, false);
                    if (t < 16 && w1 != w0) apply(w1, true);
                }
            }
            if constexpr (MODE == RFI_MODE_NOISE) {
                const int64_t j0 = d.abs_base + base + p;
                auto merged = [&](int wv, int ln, int slot, int part, uint32_t xw) -> uint32_t {
                    const int off = slot * 4096 + (wv * 64 + ln) * 16 + part * 4;
                    const int rel = p + off - lead;
                    const int w0 = min(window_of(max(rel, 0)), last);
                    const int w1 = min(w0 + 1, last);
                    uint32_t r = xw;
                    // the two windows of a part share its Philox block, not
                    // their parameters
                    for (int w = w0; w <= ((w0 + 1) * W - rel < 4 ? w1 : w0); ++w) {
                        const WinParams pw = sm.prm[w];
                        const uint32_t mask = w == w0 ? below((w0 + 1) * W - rel) : ~below((w0 + 1) * W - rel);
                        const uint32_t lo_u = rep_i16((pw.lo + 128) * 256), hi_u = rep_i16((pw.hi + 128) * 256);
                        const uint32_t nz = noise_quad_i8((uint64_t)(j0 + off), a.seed, d.key, pw.m, pw.sq8);
                        r = bit_select(mask, byte_perm(nz, xw, flag_sel_i8x4(xw, lo_u, hi_u)), r);
                    }
                    return r;
                };
                pool_noise(v, cf, sm.noise(), merged);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int rel = p + i * 4096 + tid * 16 - lead;
                if (rel >= len) continue;
                if (rel >= 0 && rel + 16 <= len) {
                    gstore16_nt(y + s0 + rel, make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]));
                } else {
#pragma unroll
                    for (int b = 0; b < 16; ++b)
                        if (rel + b >= 0 && rel + b < len)
                            gstore(reinterpret_cast<uint8_t*>(y) + s0 + rel + b, (uint8_t)byte_of(v[4 * i + b / 4], b % 4));
                }
            }
        }
    } else {
        // Windows of a few samples, and noise on streams whose dwords are not
        // whole Philox blocks: sample by sample.
#pragma unroll 1
        for (int64_t j = s0 + tid; j < s1; j += kBlock) {
            const int wl = (int)(j - s0) / W;
            const WinParams p = sm.prm[wl];
            const int xv = gload(x + j);
            int yv = xv;
            if (xv < p.lo || xv > p.hi) {
                atomicAdd(&sm.flagged[wl], 1u);
                if constexpr (MODE == RFI_MODE_ZERO) yv = 0;
                else if constexpr (MODE == RFI_MODE_CLIP) yv = min(max(xv, p.lo), p.hi);
                else yv = noise_sample(d.abs_base + j, a.seed, d.key, p.m, p.sq8, -128, 127);
            }
            gstore(y + j, (int8_t)yv);
        }
    }
    __syncthreads();
    if (tid < it.n_windows) {
        stats[g0 + tid].n_flagged = sm.flagged[tid];
        stats[g0 + tid].threshold = sm.thr[tid];
    }
}

// One 16-byte unit per thread from pinned host memory: tables of a few tens
// of KiB reach the device in about 3 us, ordered before the next kernel of
// the stream without the signals a DMA copy waits for (7 us and a gap of 17
// before the kernel that follows it).
__global__ __launch_bounds__(kBlock) void k_stage(void* dst, const void* src, int64_t n16)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n16) gstore16(static_cast<uint8_t*>(dst) + 16 * i, gload16(static_cast<const uint8_t*>(src) + 16 * i));
}

// ---------------------------------------------------------------------------
// Host launch wrappers.
// ---------------------------------------------------------------------------
template <int MODES, bool PERSIST, int T>
static void (*i8_tile_kernel_t(int cls))(LaunchArgs)
{
    switch (cls) {
        case 0: return k_i8_tiles<0, MODES, PERSIST, T>;
        case 1: return k_i8_tiles<1, MODES, PERSIST, T>;
        case 2: return k_i8_tiles<2, MODES, PERSIST, T>;
        case 3: return k_i8_tiles<3, MODES, PERSIST, T>;
        case 4: return k_i8_tiles<4, MODES, PERSIST, T>;
        case 5: return k_i8_tiles<5, MODES, PERSIST, T>;
        default: return nullptr;
    }
}

// Loop-free launches take one or two tiles per workgroup, persistent ones one.
template <int MODES, bool PERSIST>
static void (*i8_tile_kernel_m(int cls, int tpw))(LaunchArgs)
{
    if constexpr (PERSIST) return i8_tile_kernel_t<MODES, true, 1>(cls);
    else return tpw == 2 ? i8_tile_kernel_t<MODES, false, 2>(cls) : i8_tile_kernel_t<MODES, false, 1>(cls);
}

// modes: bit m set if some stream of the launch uses mode m.
template <bool PERSIST>
static void (*i8_tile_kernel_p(int cls, int modes, int tpw))(LaunchArgs)
{
    switch (modes) {
        case 1: return i8_tile_kernel_m<1, PERSIST>(cls, tpw);
        case 2: return i8_tile_kernel_m<2, PERSIST>(cls, tpw);
        case 3: return i8_tile_kernel_m<3, PERSIST>(cls, tpw);
        case 4: return i8_tile_kernel_m<4, PERSIST>(cls, tpw);
        case 1 << kModeStats: return i8_tile_kernel_m<1 << kModeStats, PERSIST>(cls, tpw);
        default: return i8_tile_kernel_m<7, PERSIST>(cls, tpw);
    }
}

static void (*i8_tile_kernel(int cls, int modes, bool persist, int tpw))(LaunchArgs)
{
    return persist ? i8_tile_kernel_p<true>(cls, modes, 1) : i8_tile_kernel_p<false>(cls, modes, tpw);
}

hipError_t launch_i8_tiles(int cls, int modes, int tpw, const LaunchArgs& a, int grid, hipStream_t s)
{
    // A grid that covers every item runs a loop-free variant with tpw
    // items per workgroup; a smaller grid runs the persistent variant.
    const bool persist = grid < a.n_items;
    if (tpw != 1 && tpw != 2) return hipErrorInvalidValue;
    auto k = i8_tile_kernel(cls, modes, persist, tpw);
    if (!k) return hipErrorInvalidValue;
    return launch(k, a, persist ? grid : (int)((a.n_items + tpw - 1) / tpw), s);
}
template <int NT, int K>
static void (*i8_window_kernel(int modes))(LaunchArgs)
{
    switch (modes) {
        case 1: return k_i8_windows<NT, K, 1>;
        case 2: return k_i8_windows<NT, K, 2>;
        case 3: return k_i8_windows<NT, K, 3>;
        case 4: return k_i8_windows<NT, K, 4>;
        case 1 << kModeStats: return k_i8_windows<NT, K, 1 << kModeStats>;
        default: return k_i8_windows<NT, K, 7>;
    }
}

hipError_t launch_i8_generic(const LaunchArgs& a, int modes, int grid, hipStream_t s, int small_nt)
{
    const bool persist = grid < a.n_items;
    if (small_nt != 0 && !persist && a.n_items > 0) {
        if (small_nt == kShortWindows) return launch_kernel(k_i8_short, dim3((unsigned)a.n_items), dim3(64), s, a);
        const int nt = small_nt & ~kWideThreads;
        void (*k)(LaunchArgs) = small_nt == 64                   ? i8_window_kernel<64, 4>(modes)
                                : small_nt == (64 | kWideThreads)  ? i8_window_kernel<64, 8>(modes)
                                : small_nt == 128                  ? i8_window_kernel<128, 4>(modes)
                                : small_nt == (128 | kWideThreads) ? i8_window_kernel<128, 8>(modes)
                                : small_nt == 256                  ? i8_window_kernel<256, 4>(modes)
                                : small_nt == (256 | kWideThreads) ? i8_window_kernel<256, 8>(modes)
                                                                   : nullptr;
        if (!k) return hipErrorInvalidValue;
        const int64_t per = kBlock / nt;
        const int64_t blocks = (a.n_items + per - 1) / per;
        if (blocks > (1 << 30)) return hipErrorInvalidValue;
        return launch_kernel(k, dim3((unsigned)blocks), dim3(kBlock), s, a);
    }
    void (*k)(LaunchArgs) = (modes & 4) ? (persist ? k_i8_generic<true, true> : k_i8_generic<false, true>)
                                        : (persist ? k_i8_generic<true, false> : k_i8_generic<false, false>);
    return launch(k, a, grid, s);
}
template <bool PERSIST>
static void (*i8_fused_kernel(int modes))(LaunchArgs)
{
    switch (modes) {
        case 1: return k_i8_fused<PERSIST, 1>;
        case 2: return k_i8_fused<PERSIST, 2>;
        case 4: return k_i8_fused<PERSIST, 4>;
        default: return k_i8_fused<PERSIST, 7>;
    }
}

hipError_t launch_i8_fused(int modes, const LaunchArgs& a, int grid, hipStream_t s)
{
    return launch(grid < a.n_items ? i8_fused_kernel<true>(modes) : i8_fused_kernel<false>(modes), a, grid, s);
}

// Six waves per SIMD (80 VGPRs; unbounded 97 and five: 60 x 2^22 samples, W
// 5000, 258 against 239 us for the whole call, W 4096 unchanged).
__global__ __launch_bounds__(kBlock, 6) void k_mom_apply(LaunchArgs a, const MomItem* __restrict__ items,
                                                      const int32_t* __restrict__ dm,
                                                      const int64_t* __restrict__ stream_woff,
                                                      const int64_t* __restrict__ abs_add,
                                                      rfi_window_stats* __restrict__ stats, MomHistory h)
{
    __shared__ MomSmem sm;
    // the first workgroups carry the streams' histories on
    if ((int)blockIdx.x < h.n_hist) {
        mom_history(h, (int)blockIdx.x);
        return;
    }
    const MomItem it = items[blockIdx.x - h.n_hist];
    StreamView d = resolve(a.streams[it.stream], a);
    if (abs_add) d.abs_base += abs_add[it.stream];
    if (d.mode == RFI_MODE_CLIP) mom_apply_item<RFI_MODE_CLIP>(a, it, d, dm, stream_woff, stats, sm);
    else if (d.mode == RFI_MODE_ZERO) mom_apply_item<RFI_MODE_ZERO>(a, it, d, dm, stream_woff, stats, sm);
    else mom_apply_item<RFI_MODE_NOISE>(a, it, d, dm, stream_woff, stats, sm);
}

hipError_t launch_i8_multi(int cls, const MultiArgs& ma, int grid, hipStream_t s)
{
    if (ma.a.n_items <= 0) return hipSuccess;
    void (*k)(MultiArgs) = nullptr;
    switch (cls) {
        case 0: k = k_i8_multi<0>; break;
        case 1: k = k_i8_multi<1>; break;
        case 2: k = k_i8_multi<2>; break;
        case 3: k = k_i8_multi_wide<3>; break;
        case 4: k = k_i8_multi_wide<4>; break;
        case 5: k = k_i8_multi_wide<5>; break;
        default: return hipErrorInvalidValue;
    }
    MultiArgs args = ma;
    void* kargs[] = {&args};
    return hipLaunchKernel(reinterpret_cast<const void*>(k), dim3(grid), dim3(kBlock), kargs, 0, s);
}

hipError_t launch_mom_select(const MomStream* streams, const MomSeg* segs, int64_t n_segs, int32_t mom_k,
                             const uint8_t* mad, const uint8_t* hist, const int32_t* hist_len, int32_t* dm,
                             hipStream_t s)
{
    if (n_segs <= 0) return hipSuccess;
    if (n_segs > (1 << 30)) return hipErrorInvalidValue;
    return launch_kernel(k_mom_select, dim3((unsigned)n_segs), dim3(64), s, streams, segs, mom_k, mad, hist, hist_len, dm);
}

hipError_t launch_mom_apply(const LaunchArgs& a, const MomItem* items, int64_t n_items, const int32_t* dm,
                            const int64_t* stream_woff, const int64_t* abs_add, rfi_window_stats* stats,
                            const MomHistory& h, hipStream_t s)
{
    if (n_items + h.n_hist <= 0) return hipSuccess;
    if (n_items > (1 << 30)) return hipErrorInvalidValue;
    return launch_kernel(k_mom_apply, dim3((unsigned)(n_items + h.n_hist)), dim3(kBlock), s, a, items, dm, stream_woff,
                         abs_add, stats, h);
}

hipError_t launch_stage(void* dst, const void* src_host, int64_t n16, hipStream_t s)
{
    if (n16 <= 0) return hipSuccess;
    return launch_kernel(k_stage, dim3((unsigned)((n16 + kBlock - 1) / kBlock)), dim3(kBlock), s, dst, src_host, n16);
}

// Every instance that a batch may take (one mode, or mixed; persistent ones
// mixed): a kernel's first dispatch pays for bringing its code in.
hipError_t warm_i8_fused(bool persist, hipStream_t s)
{
    LaunchArgs a{};  // no items: the workgroup returns at once
    void* kargs[] = {&a};
    for (int modes : {1, 2, 4, 7}) {
        if (persist && modes != 7) continue;
        void (*k)(LaunchArgs) = persist ? i8_fused_kernel<true>(modes) : i8_fused_kernel<false>(modes);
        hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(k), dim3(1), dim3(kBlock), kargs, 0, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

int i8_persistent_grid(int cls, int modes, bool fused)
{
    if (fused) return resident_grid(i8_fused_kernel<true>(modes));
    if (cls < 0) return resident_grid((modes & 4) ? k_i8_generic<true, true> : k_i8_generic<true, false>);
    return resident_grid(i8_tile_kernel(cls, modes, true, 1));
}

}  // namespace rfi
