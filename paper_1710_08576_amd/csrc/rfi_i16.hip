// rfi_i16.hip -- the int16 kernels of librfimad: windows of up to 16384
// samples held in registers (one window per 64 to 512 threads, 8192-sample
// tiles among them) and an 8+8-bit radix select over global memory for the
// others (longer windows, windows with a carried head).
#include <type_traits>

#include "rfi_item.hpp"

namespace rfi {

// Scratch of the radix select: four digit histograms.
struct I16RadixSmem {
    __align__(16) uint32_t hist[4 * 256];
    int32_t sel[4];
    uint32_t flagged;
};

// ---------------------------------------------------------------------------
// int16: radix select over two 8-bit digits.
// ---------------------------------------------------------------------------
// Find the bucket of rank `need` (1-based) in a 256-bin histogram.  Every lane
// of the wave gets the bucket and the count below it.  hw is left unchanged.
__device__ __forceinline__ void bucket_of(const uint32_t* hw, uint32_t need, int& bucket, uint32_t& below)
{
    const int lane = lane_id();
    uint32_t c[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] = hw[lane * 4 + j];
#pragma unroll
    for (int j = 1; j < 4; ++j) c[j] += c[j - 1];
    const uint32_t incl = group_incl_scan<64>(c[3]);
    const uint32_t excl = incl - c[3];
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] += excl;
    // Bins run in lane order and C is non-decreasing: the bucket holding
    // rank `need` is the number of bins with C < need.
    int nb = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) nb += group_count<64>(c[j] < need);
    bucket = min(nb, 255);  // 255 only if the histogram held fewer than `need`
    const int prev = bucket - 1;
    const int pj = prev & 3;
    const uint32_t mine = pj == 0 ? c[0] : pj == 1 ? c[1] : pj == 2 ? c[2] : c[3];
    const uint32_t got = (uint32_t)__builtin_amdgcn_readlane((int)mine, max(prev, 0) >> 2);
    below = prev >= 0 ? got : 0u;
}

// 4 int16 noise samples starting at absolute index j0 (a multiple of 4):
// dword k holds samples j0 + 2k (low half) and j0 + 2k + 1.
__device__ __forceinline__ uint2 noise_quad_i16(uint64_t j0, uint64_t seed, uint32_t key, int m,
                                                int sq8)
{
    make_opaque(seed, key);
    const Philox4x64 r = philox4x64_10(j0 >> 2, seed, key);
    uint32_t o[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        uint32_t nb = 0;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int g = c_q8[(uint32_t)(r.w[2 * k + b] >> 52)];
            const int64_t q = ((int64_t)sq8 * g + 32768) >> 16;
            const int val = (int)min(max((int64_t)m + q, (int64_t)-32768), (int64_t)32767);
            nb |= ((uint32_t)val & 0xFFFFu) << (16 * b);
        }
        o[k] = nb;
    }
    return make_uint2(o[0], o[1]);
}

// ---------------------------------------------------------------------------
// int16 windows in registers: one window of at most 8 * K * NT samples per NT
// threads (K 16-byte chunks per thread).
// ---------------------------------------------------------------------------
// A window is one contiguous run of 16-byte chunks; the samples of the edge
// chunks outside the window are set to the largest value, whose count in
// excess is known (`pad` below), so that the counting has no per-sample
// bounds test.  Chunks past the window's end are skipped: counted too, they
// would all meet in one slot (W 5000 by 256 threads of four chunks, 19 % of
// them: 180 us against 110 for 60 x 2^21 samples).
constexpr uint32_t kI16Pad = 0x7FFF7FFFu;

// Slots of the window's histogram: 16 per thread.
template <int NT, bool NOISE>
struct I16WinSmem {
    static constexpr int NW = NT / 64;
    static constexpr int kSlots = 16 * NT;
    static constexpr int kMaxShift = NT == 64 ? 6 : NT == 128 ? 5 : NT == 256 ? 4 : 3;
    static_assert((kSlots << kMaxShift) == 65536, "the widest slots cover every value");
    __align__(16) uint32_t h[kSlots];
    __align__(16) uint32_t fine[2][64];  // digits inside the median's slot, inside the MAD's bracket
    uint32_t part[NW];                   // per-wave totals of the scan
    int32_t est[NW];                     // per-wave median estimates (-1: no sample)
    int32_t shift[NW];                   // per-wave slot widths
    int32_t sel[2];                      // the median's slot, the count below it
    uint32_t below;                      // samples below the MAD's bracket
    uint32_t flagged;
    // With several waves the noise pool writes its list while other waves
    // may still be searching the counts in h, so it has storage of its own;
    // one wave orders its own accesses and reuses h.
    uint32_t noise_counts[4];
    __align__(16) uint32_t noise_list[NOISE && NT > 64 ? NT : 0];
    __align__(16) uint2 noise_data[NOISE && NT > 64 ? NT : 0];
    __device__ NoiseScratch noise()
    {
        if constexpr (NT == 64) return NoiseScratch{noise_counts, h, reinterpret_cast<uint4*>(h + 64)};
        else return NoiseScratch{noise_counts, noise_list, reinterpret_cast<uint4*>(noise_data)};
    }
};

// A wave's estimate of the median of u = x + 32768 (the lower median of 64
// of its samples to 32 values, by ballot counts), and the slot width 2^s at
// which the histogram reaches 1.5 of the samples' MAD on either side of it.
// -1 if the wave holds no sample.  Only the place and the width of the
// histogram depend on it, not the results.
template <int NT, int K>
__device__ __forceinline__ void i16_estimate(const uint32_t (&v)[4 * K], int nch, int& est, int& shift)
{
    constexpr int kSlots = 16 * NT;
    constexpr int kMaxShift = I16WinSmem<NT, false>::kMaxShift;
    const int lane = lane_id();
    uint32_t pick = v[0];
    if (nch > 3 * NT) pick = lane < 16 ? v[0] : lane < 32 ? v[5] : lane < 48 ? v[10] : v[15];  // of the first four chunks
    const uint32_t us = (pick ^ 0x8000u) & 0xFFFFu;
    const uint64_t vm = __ballot(us != 0xFFFFu);  // not padding
    const int half = ((int)__popcll(vm) + 1) >> 1;
    est = -1;
    shift = 0;
    if (vm == 0) return;
    uint32_t e = 0;
#pragma unroll
    for (int b = 15; b >= 5; --b) {
        const uint32_t t = e | (1u << b);
        e = (int)__popcll(__ballot(us < t)) < half ? t : e;
    }
    e += 16;
    est = (int)e;
    const uint32_t dv = us > e ? us - e : e - us;
    int s = 0;
    while (s < kMaxShift && (int)__popcll(__ballot(dv < ((uint32_t)(kSlots / 3) << s)) & vm) < half) ++s;
    shift = s;
}

// Exact lower median m and MAD D of a window.  v: its samples, kI16Pad where
// there is none; nch: its chunks, pad: the padding samples in them.
//
// One histogram of kSlots slots of 2^s values is counted around the
// estimated median (slot 0 also takes everything below, the last slot
// everything above), and turned into cumulative counts.  With s = 0 the
// median and the MAD are read off the counts; N(d) = #{|x - m| <= d} is
// C(m + d) - C(m - d - 1), searched 64-way.  With wider slots a pass over
// the samples in the median's slot gives its last s bits; the MAD is
// bracketed to 2^s values by the counts of the slots that touch
// [m - d, m + d], and a pass over |x - m| gives its place in the bracket.
// If the median or the MAD lies outside the counted values (every thread
// alike), the histogram is taken again over all 65536 values.
template <int NT, int K, bool NOISE, bool WHOLE>
__device__ __forceinline__ void i16_select(const uint32_t (&v)[4 * K], int nch, int pad, int n, int tid, int wave,
                                           I16WinSmem<NT, NOISE>& sm, int& m_out, int& D_out)
{
    using Smem = I16WinSmem<NT, NOISE>;
    constexpr int NW = Smem::NW;
    constexpr int NS = Smem::kSlots;
    constexpr int SW = 1024;  // slots per wave
    const int lane = lane_id();
    const uint32_t need = (uint32_t)((n - 1) / 2 + 1);
    int est, s;
    i16_estimate<NT, K>(v, nch, est, s);
    auto have = [&](int q) { return WHOLE || tid + (q >> 2) * NT < nch; };  // dword q of this thread
    for (bool full = false;; full = true) {
        group_sync<NT>();  // the previous use of the scratch is over
        uint32_t* hw = sm.h + wave * SW;
#pragma unroll
        for (int q = 0; q < 4; ++q) reinterpret_cast<uint4*>(hw)[q * 64 + lane] = make_uint4(0, 0, 0, 0);
        if (tid < 32) reinterpret_cast<uint4*>(&sm.fine[0][0])[tid] = make_uint4(0, 0, 0, 0);
        if (tid == 0) {
            sm.below = 0;
            sm.flagged = 0;
            sm.noise_counts[0] = 0;  // the noise pool's slot reservations
        }
        if constexpr (NW > 1) {
            if (lane == 0) {
                sm.est[wave] = est;
                sm.shift[wave] = s;
            }
        }
        group_sync<NT>();
        int mid = est, sh = s;
        if constexpr (NW > 1) {
            // mean of the waves' estimates, without the lowest and highest
            int cnt = 0, sum = 0, lo = 1 << 20, hi = 0;
            sh = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const int e = sm.est[w];
                if (e >= 0) {
                    ++cnt;
                    sum += e;
                    lo = min(lo, e);
                    hi = max(hi, e);
                }
                sh = max(sh, sm.shift[w]);
            }
            if (cnt > 2) {
                sum -= lo + hi;
                cnt -= 2;
            }
            mid = cnt > 0 ? (int)((float)sum * __builtin_amdgcn_rcpf((float)cnt)) : -1;
        }
        if (mid < 0) mid = 32768;
        sh = __builtin_amdgcn_readfirstlane(full ? Smem::kMaxShift : sh);
        // first value of slot 0, as a sample
        const int base = __builtin_amdgcn_readfirstlane(
            min(max(mid - ((NS / 2) << sh), 0), 65536 - (NS << sh)) - 32768);
        const bool lo_all = base == -32768;                    // slot 0 holds its own values only
        const bool hi_all = base + (NS << sh) >= 32768;        // and so does the last slot
        const uint32_t b2 = rep_i16(base);
        // opaque, so that v ^ bias of the rare paths is not kept in
        // registers across the loop
        uint32_t bias = 0x80008000u;
        pin_sgpr(bias);
        char* hb = reinterpret_cast<char*>(sm.h);
        auto count = [&](uint32_t x, auto shifted) {
            uint32_t t = pk_subsat_i16(x, b2);
            if constexpr (decltype(shifted)::value) t = pk_ashr_i16(t, sh);
            t = pk_shl2_u16(pk_clamp_i16(t, 0u, (uint32_t)(NS - 1) * 0x10001u));
            atomicAdd(reinterpret_cast<uint32_t*>(hb + (t & 0xFFFFu)), 1u);
            atomicAdd(reinterpret_cast<uint32_t*>(hb + (t >> 16)), 1u);
            sched_fence();
        };
        // Saturation: x - base is at most 32767, which an unshifted or
        // narrow slot number already exceeds; shifted slots of the full
        // range are counted from x + 32768 as unsigned halves.
        if (sh == Smem::kMaxShift) {
#pragma unroll
            for (int q = 0; q < 4 * K; ++q) {
                if (have(q)) {
                    const uint32_t u = v[q] ^ bias;
                    atomicAdd(sm.h + ((u & 0xFFFFu) >> Smem::kMaxShift), 1u);
                    atomicAdd(sm.h + (u >> (16 + Smem::kMaxShift)), 1u);
                    sched_fence();
                }
            }
        } else if (sh == 0) {
#pragma unroll
            for (int q = 0; q < 4 * K; ++q)
                if (have(q)) count(v[q], std::false_type{});
        } else {
#pragma unroll
            for (int q = 0; q < 4 * K; ++q)
                if (have(q)) count(v[q], std::true_type{});
        }
        group_sync<NT>();
        // Cumulative counts.  Lane l of a wave holds slots 4 (64 q + l) ..
        // + 3 of the wave's 1024 (consecutive lanes read consecutive chunks:
        // no bank conflicts), q = 0..3; four scans instead of one, but the
        // reads and writes of a 64-byte run per lane would meet four deep.
        uint32_t c[16], tot[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 t = reinterpret_cast<const uint4*>(hw)[q * 64 + lane];
            c[4 * q] = t.x;
            c[4 * q + 1] = t.y + c[4 * q];
            c[4 * q + 2] = t.z + c[4 * q + 1];
            c[4 * q + 3] = t.w + c[4 * q + 2];
        }
        uint32_t run = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t incl = group_incl_scan<64>(c[4 * q + 3]);
            const uint32_t excl = run + incl - c[4 * q + 3];
            run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            tot[q] = run;
#pragma unroll
            for (int j = 0; j < 4; ++j) c[4 * q + j] += excl;
        }
        uint32_t off = 0;
        if constexpr (NW > 1) {
            if (lane == 0) sm.part[wave] = run;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) off += w < wave ? sm.part[w] : 0u;
            off = (uint32_t)__builtin_amdgcn_readfirstlane((int)off);
        }
        // The padding is counted with the largest value: cap at n.
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int j = 0; j < 4; ++j) c[4 * q + j] = WHOLE ? c[4 * q + j] + off : min(c[4 * q + j] + off, (uint32_t)n);
            reinterpret_cast<uint4*>(hw)[q * 64 + lane] =
                make_uint4(c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]);
        }
        // The median's slot: the number of slots whose count is below need.
        int mt = 0;
        if (off < need && need <= off + run) {
            int found = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (off + tot[q] < need) {
                    found += 256;
                } else if (q == 0 || off + tot[q > 0 ? q - 1 : 0] < need) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) found += group_count<64>(c[4 * q + j] < need);
                }
            }
            mt = wave * SW + found;
            if constexpr (NW > 1)
                if (lane == 0) sm.sel[0] = mt;
        }
        group_sync<NT>();
        if constexpr (NW > 1) mt = __builtin_amdgcn_readfirstlane(sm.sel[0]);
        const bool med_ok = (mt > 0 || lo_all) && (mt < NS - 1 || hi_all);
        if (!med_ok) continue;
        // count of the values of slots 0..t
        auto H = [&](int t) -> uint32_t { return t < 0 ? 0u : sm.h[min(t, NS - 1)]; };
        int m = base + (mt << sh);
        if (sh > 0) {
            // the median's last sh bits, from the samples of its slot
            const uint32_t lowmask = (1u << sh) - 1u;
            const uint32_t mtu = (uint32_t)(m + 32768), topmask = 0xFFFFu & ~lowmask;
            // slots start at base, which need not be a multiple of 2^sh
            const uint32_t bu = mtu * 0x10001u;
#pragma unroll
            for (int q = 0; q < 4 * K; ++q) {
                if ((q >> 2) * NT < nch) {
                    const uint32_t r = pk_sub_u16(v[q] ^ bias, bu);
                    const bool in0 = have(q) && (r & topmask) == 0, in1 = have(q) && (r & (topmask << 16)) == 0;
                    if (__ballot(in0 || in1) != 0) {
                        if (in0) atomicAdd(&sm.fine[0][r & lowmask], 1u);
                        if (in1) atomicAdd(&sm.fine[0][(r >> 16) & lowmask], 1u);
                    }
                }
            }
            group_sync<NT>();
            const uint32_t fc = group_incl_scan<64>(sm.fine[0][lane]);
            m += min(group_count<64>(fc < need - H(mt - 1)), (int)lowmask);
        }
        // Largest d whose counts are known on both sides of the median.
        const int one = 1 << sh;
        const int dlo_max = lo_all ? 65535 : m - (base + one);
        const int dhi_max = hi_all ? 65535 : base + ((NS - 1) << sh) - 1 - m;
        const int dwin = min(dlo_max, dhi_max);
        // samples in the slots that touch [m - d, m + d]
        auto N = [&](int d) -> uint32_t { return H((m + d - base) >> sh) - H(((m - d - base) >> sh) - 1); };
        if (dwin < 0 || N(dwin) < need) continue;
        // smallest d in [0, dwin] with N(d) >= need: 64-way search, each lane
        // testing the right end of its sub-range
        int lo = 0, span = dwin + 1;
        while (span > 1) {
            const int step = (span + 63) >> 6;
            const int right = min(lo + (lane + 1) * step - 1, lo + span - 1);
            const bool ok = lo + lane * step < lo + span && N(right) >= need;
            const int f = (int)__builtin_ctzll(__ballot(ok));  // the last sub-range always qualifies
            const int nlo = lo + f * step;
            span = min(step, lo + span - nlo);
            lo = nlo;
        }
        if (sh > 0) {
            // D is in [lo, lo + 2^sh - 1]
            const uint32_t m2 = rep_i16(m), l2 = rep_i16(lo);
            uint32_t nbelow = 0;
#pragma unroll
            for (int q = 0; q < 4 * K; ++q) {
                if ((q >> 2) * NT < nch) {
                    const uint32_t dq = pk_absdiff_i16(v[q], m2);
                    nbelow += (uint32_t)__popcll(__ballot(have(q) && (dq & 0xFFFFu) < (uint32_t)lo)) +
                              (uint32_t)__popcll(__ballot(have(q) && dq < ((uint32_t)lo << 16)));
                    pin_sgpr(nbelow);
                    const uint32_t r = pk_sub_u16(dq, l2);  // wraps when below
                    const bool in0 = have(q) && (r & 0xFFFFu) < (uint32_t)one;
                    const bool in1 = have(q) && r < ((uint32_t)one << 16);
                    if (__ballot(in0 || in1) != 0) {
                        if (in0) atomicAdd(&sm.fine[1][r & 0x3Fu], 1u);
                        if (in1) atomicAdd(&sm.fine[1][(r >> 16) & 0x3Fu], 1u);
                    }
                }
            }
            if constexpr (NW > 1) {
                if (lane == 0) atomicAdd(&sm.below, nbelow);
            }
            group_sync<NT>();
            if constexpr (NW > 1) nbelow = sm.below;
            // take the padding out again: all of it lies dp from the median
            const int dp = 32767 - m;
            if (dp < lo) nbelow -= (uint32_t)pad;
            uint32_t f = sm.fine[1][lane];
            if (dp - lo == lane && lane < one) f -= (uint32_t)pad;
            const uint32_t fc = group_incl_scan<64>(f);
            lo += min(group_count<64>(fc < need - nbelow), one - 1);
        }
        m_out = m;
        D_out = lo;
        return;
    }
}

// One window of NT threads (tid: the thread's index among them).  WHOLE:
// the window is 8 * K * NT samples and starts on a chunk (tiles); otherwise
// any length and position that spans at most K * NT chunks.  MODES: bit m
// set if the launch has windows in mode m (one bit: the mode is fixed at
// compile time).
template <int NT, int K, int MODES, bool WHOLE>
__device__ __forceinline__ void i16_window(const StreamView& d, int64_t w, int64_t a, int n, uint64_t seed, int tid,
                                           I16WinSmem<NT, (MODES & 4) != 0>& sm)
{
    const int lane = lane_id();
    const int wave = NT == 64 ? 0 : tid >> 6;
    const int64_t c0 = a >> 3;
    const int lead = WHOLE ? 0 : (int)(a & 7);       // first sample of the window in chunk 0
    const int nch = WHOLE ? K * NT : __builtin_amdgcn_readfirstlane((lead + n + 7) >> 3);
    const int tail = WHOLE ? 8 : ((lead + n - 1) & 7) + 1;  // end of the window in the last chunk
    // first byte of this thread's chunk 0
    const uint8_t* xt = static_cast<const uint8_t*>(d.x) + (c0 + tid) * 16;
    // valid halves of dword j of chunk c, as a mask
    auto inside = [&](int c, int j) -> uint32_t {
        const int f = c == 0 ? lead : 0, e = c == nch - 1 ? tail : 8;
        return (2 * j >= f && 2 * j < e ? 0xFFFFu : 0u) | (2 * j + 1 >= f && 2 * j + 1 < e ? 0xFFFF0000u : 0u);
    };
    uint32_t v[4 * K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        uint4 t = make_uint4(kI16Pad, kI16Pad, kI16Pad, kI16Pad);
        if (WHOLE || tid + i * NT < nch) t = gload16_nt(xt + i * NT * 16);
        v[4 * i] = t.x;
        v[4 * i + 1] = t.y;
        v[4 * i + 2] = t.z;
        v[4 * i + 3] = t.w;
    }
    const bool edges = !WHOLE && (lead != 0 || tail != 8);
    if (edges) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const int c = tid + i * NT;
            if (c == 0 || c == nch - 1) {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[4 * i + j] = bit_select(inside(c, j), v[4 * i + j], kI16Pad);
            }
        }
    }
    const int pad = nch * 8 - n;
    int m, D;
    i16_select<NT, K, (MODES & 4) != 0, WHOLE>(v, nch, pad, n, tid, wave, sm, m, D);

    float sig;
    const float t = threshold_of(D, d.k, sig);
    const int T = (int)floorf(t);
    const int lo = max(m - T, -32768), hi = min(m + T, 32767);
    const uint32_t lo2 = rep_i16(lo), hi2 = rep_i16(hi);
    const int sq8 = (int)__fmul_rn(sig, 256.0f);
    const int mode = MODES == 1 ? RFI_MODE_ZERO : MODES == 2 ? RFI_MODE_CLIP : MODES == 4 ? RFI_MODE_NOISE : d.mode;
    uint32_t nflag = 0;
    if (mode != RFI_MODE_NOISE) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
            if (WHOLE || tid + i * NT < nch) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int q = 4 * i + j;
                    const uint32_t x = v[q];
                    const uint32_t c = pk_clamp_i16(x, lo2, hi2);
                    const uint32_t bit = pk_umin1(c ^ x);  // 1 in the halves of flagged samples
                    nflag = udot2_u16(bit, 0x00010001u, nflag);
                    pin_vgpr(nflag);
                    v[q] = mode == RFI_MODE_CLIP ? c : x & ~pk_sub_u16(0u, bit);
                }
            }
        }
    }
    if constexpr ((MODES & 4) != 0) {
        if (mode == RFI_MODE_NOISE) {
            const int64_t abs0 = d.abs_base + c0 * 8;
            const uint32_t key1 = d.key;
            auto merged = [&](int wv, int ln, int slot, int part, uint2 x) -> uint2 {
                const int64_t off = (int64_t)(slot * NT + wv * 64 + ln) * 8 + part * 4;
                const uint2 nz = noise_quad_i16((uint64_t)(abs0 + off), seed, key1, m, sq8);
                const uint32_t m0 = nonzero_half_mask(pk_clamp_i16(x.x, lo2, hi2) ^ x.x);
                const uint32_t m1 = nonzero_half_mask(pk_clamp_i16(x.y, lo2, hi2) ^ x.y);
                // every flagged sample is in one part, drawn once
                nflag += (__popc(m0) + __popc(m1)) >> 4;
                return make_uint2((x.x & ~m0) | (nz.x & m0), (x.y & ~m1) | (nz.y & m1));
            };
            if constexpr (NT == 64) wave_sync();  // the counts in h are dead: the list takes their place
            const uint32_t lob = rep_i16(lo + 32768), hib = rep_i16(hi + 32768), span4 = 4u * (uint32_t)(hi - lo);
            uint32_t cf = 0;  // bit q: dwords 2q, 2q + 1 hold a flagged sample
#pragma unroll
            for (int q = 0; q < 2 * K; ++q)
                if (WHOLE || tid + (q >> 1) * NT < nch)
                    cf |= (outside_i16x4(v[2 * q], v[2 * q + 1], lob, hib, span4) ? 1u : 0u) << q;
            pool_noise_reserved<NT>(v, cf, sm.noise(), tid, wave, merged);
        }
    }
    // The store address is formed here from a fresh copy of the thread
    // index: kept live from the loads, its offsets were spilled to private
    // memory and reloaded right before the stores.
    uint32_t t2 = (uint32_t)tid;
    asm volatile("" : "+v"(t2));
    uint8_t* yt = static_cast<uint8_t*>(d.y) + c0 * 16 + (uint64_t)t2 * 16;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int c = (int)t2 + i * NT;
        if (!WHOLE && c >= nch) continue;
        if (edges && (c == 0 || c == nch - 1)) {
            // an edge chunk holds samples of the neighbouring window
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t ok = inside(c, j);
                if (ok & 0xFFFFu) gstore(reinterpret_cast<uint16_t*>(yt + i * NT * 16) + 2 * j, (uint16_t)(v[4 * i + j] & 0xFFFFu));
                if (ok >> 16) gstore(reinterpret_cast<uint16_t*>(yt + i * NT * 16) + 2 * j + 1, (uint16_t)(v[4 * i + j] >> 16));
            }
        } else {
            gstore16_nt(yt + i * NT * 16, make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]));
        }
    }
    nflag = group_incl_scan<64>(nflag);
    if constexpr (NT > 64) {
        if (lane == 63) atomicAdd(&sm.flagged, nflag);
        __syncthreads();
        nflag = sm.flagged;
    }
    if (tid == NT - 1 && d.stats) {
        rfi_window_stats s;
        s.median = m;
        s.mad = D;
        // the padding samples are flagged too unless the bound is their value
        s.n_flagged = nflag - (hi < 32767 ? (uint32_t)pad : 0u);
        s.threshold = t;
        d.stats[w] = s;
    }
}

// Whether a window qualifies for i16_window: no head segment,
// 16-byte aligned buffers, noise quads that are whole (the stream's first
// absolute index a multiple of 4), a last chunk that ends inside the stream
// or the packed layout's padding, at most K * NT chunks.
template <int NT, int K>
__device__ __forceinline__ bool i16_window_ok(const StreamView& d, int64_t a, int n)
{
    if (d.head_len != 0) return false;
    if (d.mode == RFI_MODE_NOISE && (d.abs_base & 3) != 0) return false;
    if (((uintptr_t)d.x | (uintptr_t)d.y) & 15u) return false;
    if (!d.padded && ((a + n + 7) & ~(int64_t)7) > d.length) return false;
    return ((a + n + 7) >> 3) - (a >> 3) <= K * NT;
}

// Generic int16 window: radix passes over global memory.
__device__ void i16_generic(const StreamView& d, int64_t w, uint64_t seed, I16RadixSmem& sm)
{
    const int W = d.window;
    const int64_t a = w * (int64_t)W;
    const int n = (int)min((int64_t)W, d.length - a);
    const int tid = (int)threadIdx.x;
    int16_t* y = static_cast<int16_t*>(d.y);
    uint32_t* h = sm.hist;
    const uint32_t need = (uint32_t)((n - 1) / 2 + 1);
    __syncthreads();
    for (int i = tid; i < 4 * 256; i += kBlock) h[i] = 0;
    if (tid == 0) sm.flagged = 0;
    __syncthreads();
    for (int i = tid; i < n; i += kBlock)
        atomicAdd(&h[(uint32_t)(load_logical<int16_t>(d, a + i) + 32768) >> 8], 1u);
    __syncthreads();
    if (tid < 64) {
        int b;
        uint32_t below;
        bucket_of(h, need, b, below);
        if (tid == 0) {
            sm.sel[0] = b;
            sm.sel[1] = (int)below;
        }
    }
    __syncthreads();
    const int b1 = sm.sel[0];
    const uint32_t below1 = (uint32_t)sm.sel[1];
    for (int i = tid; i < n; i += kBlock) {
        const uint32_t u = (uint32_t)(load_logical<int16_t>(d, a + i) + 32768);
        if ((int)(u >> 8) == b1) atomicAdd(&h[256 + (u & 0xFFu)], 1u);
    }
    __syncthreads();
    if (tid < 64) {
        int b;
        uint32_t below;
        bucket_of(h + 256, need - below1, b, below);
        if (tid == 0) sm.sel[2] = ((b1 << 8) | b) - 32768;
    }
    __syncthreads();
    const int m = sm.sel[2];
    for (int i = tid; i < n; i += kBlock) {
        const uint32_t dv = (uint32_t)abs(load_logical<int16_t>(d, a + i) - m);
        atomicAdd(&h[512 + (dv >> 8)], 1u);
    }
    __syncthreads();
    if (tid < 64) {
        int b;
        uint32_t below;
        bucket_of(h + 512, need, b, below);
        if (tid == 0) {
            sm.sel[0] = b;
            sm.sel[1] = (int)below;
        }
    }
    __syncthreads();
    const int b3 = sm.sel[0];
    const uint32_t below3 = (uint32_t)sm.sel[1];
    for (int i = tid; i < n; i += kBlock) {
        const uint32_t dv = (uint32_t)abs(load_logical<int16_t>(d, a + i) - m);
        if ((int)(dv >> 8) == b3) atomicAdd(&h[768 + (dv & 0xFFu)], 1u);
    }
    __syncthreads();
    if (tid < 64) {
        int b;
        uint32_t below;
        bucket_of(h + 768, need - below3, b, below);
        if (tid == 0) sm.sel[3] = (b3 << 8) | b;
    }
    __syncthreads();
    const int D = sm.sel[3];
    float sig;
    const float t = threshold_of(D, d.k, sig);
    const int T = (int)floorf(t);
    const int lo = max(m - T, -32768), hi = min(m + T, 32767);
    const int sq8 = (int)__fmul_rn(sig, 256.0f);
    uint32_t nflag = 0;
    for (int i = tid; i < n; i += kBlock) {
        const int x = load_logical<int16_t>(d, a + i);
        int yv = x;
        if (x < lo || x > hi) {
            ++nflag;
            if (d.mode == RFI_MODE_ZERO) yv = 0;
            else if (d.mode == RFI_MODE_CLIP) yv = min(max(x, lo), hi);
            else yv = noise_sample(d.abs_base + a + i, seed, d.key, m, sq8, -32768, 32767);
        }
        gstore(y + a + i, (int16_t)yv);
    }
    nflag = group_sum<64>(nflag);
    if (lane_id() == 0) atomicAdd(&sm.flagged, nflag);
    __syncthreads();
    if (tid == 0 && d.stats) {
        rfi_window_stats s;
        s.median = m;
        s.mad = D;
        s.n_flagged = sm.flagged;
        s.threshold = t;
        d.stats[w] = s;
    }
}

// One tile per workgroup: eight workgroups per CU, seven in noise mode (72
// VGPRs; at eight the draws spill, 105 us against 96 for 60 x 2^21 samples).
// The persistent loop keeps more live and keeps the unbounded budget.
template <bool PERSIST, int MODES>
__global__ __launch_bounds__(kBlock, PERSIST ? 0 : (MODES & 4) ? 7 : 8) void k_i16_tiles(LaunchArgs a)
{
    __shared__ I16WinSmem<kBlock, (MODES & 4) != 0> sm;
    for_items<PERSIST>(a, [&](int64_t it) {
        const Item item = a.items[it];
        const StreamView d = resolve(a.streams[item.stream], a);
        i16_window<kBlock, 4, MODES, true>(d, item.first / 8192, item.first, 8192, a.seed, (int)threadIdx.x, sm);
    });
}

// Windows of at most K * NT chunks, NT threads each, of padded streams
// (plans).  NT = 64: four windows per workgroup, one per wave, which never
// wait for each other.  Bound by the selection's VALU and LDS work below
// 2048 samples (the fixed cost of a window: 1024 slots to clear, add up and
// search), by HBM from there on.  60 x 2^21 samples, clip, against the
// radix select over global memory that took every window but 8192 before:
// W 512 953 -> 196 us, 1000 762 -> 120, 2048 665 -> 96, 4096 630 -> 85,
// 5000 632 -> 91, 16384 655 -> 90 (5.6 TB/s); noise W 4096 710 -> 102.
// Eight waves per SIMD; the noise kernel of 128 threads and those with eight
// chunks take seven, so as not to spill.
template <int NT, int K, bool NOISE>
__global__ __launch_bounds__(NT == 64 ? kBlock : NT, K == 8 || (NOISE && NT == 128) ? 7 : 8) void k_i16_windows(LaunchArgs a)
{
    constexpr int PER = NT == 64 ? kBlock / 64 : 1;
    __shared__ I16WinSmem<NT, NOISE> sm[PER];
    const int sub = PER > 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    const int64_t it = (int64_t)blockIdx.x * PER + sub;
    if (it >= a.n_items) return;
    const Item item = a.items[it];
    const StreamView d = resolve(a.streams[item.stream], a);
    // a tile item is one window, given by its first sample
    const int64_t win = item.kind == kItemTile ? item.first / d.window : item.first;
    const int64_t first = win * (int64_t)d.window;
    const int n = (int)min((int64_t)d.window, d.length - first);
    i16_window<NT, K, NOISE ? 7 : 3, false>(d, win, first, n, a.seed, (int)threadIdx.x & (NT - 1), sm[sub]);
}

union I16FusedSmem {
    I16WinSmem<kBlock, true> t;
    I16RadixSmem g;
};

// A generic item in a launch of 256-thread workgroups.
__device__ __forceinline__ void i16_generic_any(const StreamView& d, int64_t w, uint64_t seed, I16FusedSmem& sm)
{
    const int64_t first = w * (int64_t)d.window;
    const int n = (int)min((int64_t)d.window, d.length - first);
    if (i16_window_ok<kBlock, 4>(d, first, n)) {
        i16_window<kBlock, 4, 7, false>(d, w, first, n, seed, (int)threadIdx.x, sm.t);
        __syncthreads();  // a following item may use the scratch as the other kind
    } else {
        i16_generic(d, w, seed, sm.g);
    }
}

template <bool PERSIST>
__global__ __launch_bounds__(kBlock, PERSIST ? 0 : 7) void k_i16_generic(LaunchArgs a)
{
    __shared__ I16FusedSmem sm;
    for_items<PERSIST>(a, [&](int64_t it) {
        const Item item = a.items[it];
        const StreamView d = resolve(a.streams[item.stream], a);
        i16_generic_any(d, item.first, a.seed, sm);
    });
}

template <bool PERSIST>
__global__ __launch_bounds__(kBlock, PERSIST ? 0 : 7) void k_i16_fused(LaunchArgs a)
{
    __shared__ I16FusedSmem sm;
    for_items<PERSIST>(a, [&](int64_t it) {
        const Item item = a.items[it];
        if (item.kind == kItemCarry) {
            carry_copy(a.carries[item.stream]);
            return;
        }
        const StreamView d = resolve(a.streams[item.stream], a);
        // a tile is one window: the same code serves both kinds
        i16_generic_any(d, item.kind == kItemGeneric ? item.first : item.first / 8192, a.seed, sm);
    });
}

// ---------------------------------------------------------------------------
// Host launch wrappers.
// ---------------------------------------------------------------------------
#define RFI_PICK(K, a, grid) ((grid) < (a).n_items ? K<true> : K<false>)
template <bool PERSIST>
static void (*i16_tile_kernel(int modes))(LaunchArgs)
{
    switch (modes) {
        case 1: return k_i16_tiles<PERSIST, 1>;
        case 2: return k_i16_tiles<PERSIST, 2>;
        case 4: return k_i16_tiles<PERSIST, 4>;
        default: return k_i16_tiles<PERSIST, 7>;
    }
}

hipError_t launch_i16_tiles(int cls, int modes, const LaunchArgs& a, int grid, hipStream_t s)
{
    if (cls != 0) return hipErrorInvalidValue;
    return launch(grid < a.n_items ? i16_tile_kernel<true>(modes) : i16_tile_kernel<false>(modes), a, grid, s);
}
hipError_t launch_i16_generic(const LaunchArgs& a, int modes, int grid, hipStream_t s, int nt)
{
    if (a.n_items > 0 && grid >= a.n_items && nt != 0) {
        const bool noise = (modes & 4) != 0;
        void (*k)(LaunchArgs) = nullptr;
        switch (nt) {
            case 64: k = noise ? k_i16_windows<64, 4, true> : k_i16_windows<64, 4, false>; break;
            case 128: k = noise ? k_i16_windows<128, 4, true> : k_i16_windows<128, 4, false>; break;
            case 128 | kWideThreads: k = noise ? k_i16_windows<128, 8, true> : k_i16_windows<128, 8, false>; break;
            case 256 | kWideThreads: k = noise ? k_i16_windows<256, 8, true> : k_i16_windows<256, 8, false>; break;
            case 512: k = noise ? k_i16_windows<512, 4, true> : k_i16_windows<512, 4, false>; break;
            default: return hipErrorInvalidValue;
        }
        const int threads = nt & ~kWideThreads;
        const int64_t blocks = threads == 64 ? (a.n_items + 3) / 4 : a.n_items;
        if (blocks > (1 << 30)) return hipErrorInvalidValue;
        return launch_kernel(k, dim3((unsigned)blocks), dim3(threads == 64 ? kBlock : (unsigned)threads), s, a);
    }
    return launch(RFI_PICK(k_i16_generic, a, grid), a, grid, s);
}
hipError_t launch_i16_fused(const LaunchArgs& a, int grid, hipStream_t s)
{
    return launch(RFI_PICK(k_i16_fused, a, grid), a, grid, s);
}
#undef RFI_PICK

hipError_t warm_i16_fused(bool persist, hipStream_t s)
{
    LaunchArgs a{};  // no items: the workgroup returns at once
    void (*k)(LaunchArgs) = persist ? k_i16_fused<true> : k_i16_fused<false>;
    void* kargs[] = {&a};
    return hipLaunchKernel(reinterpret_cast<const void*>(k), dim3(1), dim3(kBlock), kargs, 0, s);
}

int i16_persistent_grid(int cls, int modes, bool fused)
{
    if (fused) return resident_grid(k_i16_fused<true>);
    if (cls < 0) return resident_grid(k_i16_generic<true>);
    return resident_grid(i16_tile_kernel<true>(modes));
}

}  // namespace rfi
