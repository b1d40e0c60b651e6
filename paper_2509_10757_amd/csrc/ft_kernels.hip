// HIP kernels of the tracking correspondence search for gfx950 (MI355X).
//
// Every kernel is written as phase functions over one frame job, so the
// single-frame calls and the batched submissions execute the very same code.
// Workgroups have 256 threads (four 64-wide waves), but for the set-up sorts and the
// stereo resolve (1024, or 256 by the launch shapes), the one-workgroup last-frame
// resolve (1024) and the record-dealt searches (one wave).  Build flags:
// -ffp-contract=off (no fused multiply-add: every float expression rounds
// exactly as written) with correctly rounded fp32 divide and sqrt.
//
// Phases per frame (Section IV-C and IV-E of the paper):
//   setup      counting sort of right keypoints by row (pinhole) | overlap
//              lists + packed target descriptors (fisheye); counting sort of
//              each view's keypoints by grid cell into packed records; clears
//              claim tables and counters
//   stereo_a   pinhole best match: G lanes per left keypoint stream the
//              row-sorted records of the rows that can hold a match
//              | fisheye all-pairs top-2 on the matrix cores (int8 MFMA over the
//              descriptors' bits)
//   refine     pinhole SAD refinement: sixteen lanes per match, a window row per
//              lane in registers (11x11, +-5 shifts); other windows one wave per
//              match, patches in LDS
//   tri        fisheye ratio + triangulation check (float64; its own kernel
//              so that its register demand does not cap the refinement's
//              occupancy)
//   stereo_c   pinhole duplicate resolution + median filter + outputs
//              | fisheye duplicate resolution + outputs
//   search     projection + window search: G lanes per map point stream the
//              cell-sorted keypoint records of the window's cells
//   search_fin duplicate resolution + outputs
//
// Batched submissions flatten every phase's tiles over the jobs; the flat
// block index is first remapped so that consecutive tiles (one frame's data)
// land on the same XCD and share its L2.

#include <hip/hip_runtime.h>

#include <algorithm>

#define FT_KERNELS 1
#include "ft_internal.h"

namespace ft {

typedef int v4i __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ helpers
struct Desc {
    uint4 a, b;
};

// 16-byte vector for copying descriptor halves through registers (a native
// vector type: arrays of it stay in registers, unlike arrays of uint4).
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// A dword at any byte address; four dwords from a dword boundary.
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef v4u v4u_dw __attribute__((aligned(4)));

// Constant address space: memory that no kernel running with the reader writes.
#if defined(__HIP_DEVICE_COMPILE__)
#define FT_C __attribute__((address_space(4)))
#else
#define FT_C
#endif

// Keypoints per thread whose loads are issued together in the setup sorts and
// the median pass (a strided loop body unrolled; surplus entries masked).
constexpr int kSortUnroll = 4;

// Candidates whose loads are issued together in the best-match and search scans.
constexpr int kBestUnroll = 2;
constexpr int kSearchUnroll = 2;

__device__ __forceinline__ Desc load_desc(const uint8_t *base, int idx)
{
    const uint4 *p = reinterpret_cast<const uint4 *>(base + 32 * (size_t)idx);
    Desc d;
    d.a = p[0];
    d.b = p[1];
    return d;
}

__device__ __forceinline__ int hamming(const Desc &u, const Desc &v)
{
    return __popc(u.a.x ^ v.a.x) + __popc(u.a.y ^ v.a.y) + __popc(u.a.z ^ v.a.z) +
           __popc(u.a.w ^ v.a.w) + __popc(u.b.x ^ v.b.x) + __popc(u.b.y ^ v.b.y) +
           __popc(u.b.z ^ v.b.z) + __popc(u.b.w ^ v.b.w);
}

__host__ __device__ inline int div_up(int n, int d) { return (n + d - 1) / d; }

// The refinement runs four matches per wave for the 11x11 window and +-5 shifts.
__host__ __device__ inline bool refine_quarter(const DevJob &J) { return J.half_win == 5 && J.half_range == 5; }

__host__ __device__ inline int view_kp(const DevJob &J, int v) { return J.view[v].side ? J.R.n : J.L.n; }
// Entry l of a per-level table, selected from values loaded for every level
// (the loads do not wait for l; a select chain instead of a dependent load).
template <class T>
__device__ __forceinline__ T pick_level(const T (&t)[kLevels], int l)
{
    T v[kLevels];
    _Pragma("unroll") for (int k = 0; k < kLevels; ++k) v[k] = t[k];
    T r = v[0];
    _Pragma("unroll") for (int k = 1; k < kLevels; ++k) r = l == k ? v[k] : r;
    return r;
}

// Pyramid level of a keypoint as a table index (levels are 0..7 by contract;
// the clamp only keeps a malformed octave byte inside the tables).
__device__ __forceinline__ int lvl(uint32_t o) { return o < (uint32_t)kLevels ? (int)o : kLevels - 1; }

__device__ __forceinline__ uint64_t shfl_xor64(uint64_t v, int m)
{
    const uint32_t lo = __shfl_xor((uint32_t)v, m);
    const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), m);
    return ((uint64_t)hi << 32) | lo;
}

// The two smallest keys seen so far (by value, so they stay in registers).
template <class T>
struct Top2 {
    T a, b;
};

template <class T>
__device__ __forceinline__ Top2<T> top2_insert(Top2<T> t, T key)
{
    const bool lt1 = key < t.a, lt2 = key < t.b;
    Top2<T> r;
    r.b = lt1 ? t.a : (lt2 ? key : t.b);
    r.a = lt1 ? key : t.a;
    return r;
}

template <class T>
__device__ __forceinline__ Top2<T> top2_merge(Top2<T> t, T o1, T o2)
{
    Top2<T> r;
    const T hi = t.a < o1 ? o1 : t.a;
    const T m2 = t.b < o2 ? t.b : o2;
    r.a = t.a < o1 ? t.a : o1;
    r.b = hi < m2 ? hi : m2;
    return r;
}

// Inclusive prefix across the 64 lanes of a wave (every lane active) with DPP
// lane moves: shifts by 1, 2, 4 and 8 inside each row of 16 lanes (lanes whose
// source lies in another row read 0), then lane 15 of rows 0 and 2 into rows
// 1 and 3, then lane 31 into rows 2 and 3.  Six VALU steps, no LDS traffic;
// 0 is the identity of both operations used (sum, and max of values >= 0).
template <bool kMax>
__device__ __forceinline__ int wave_inclusive_dpp(int v)
{
    auto op = [](int a, int b) { return kMax ? max(a, b) : a + b; };
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false));   // row_shr:1
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false));   // row_shr:2
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false));   // row_shr:4
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false));   // row_shr:8
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));   // row_bcast:15
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));   // row_bcast:31
    return v;
}

// Inclusive prefix sum across the 64 lanes of a wave.
__device__ __forceinline__ int wave_inclusive_scan(int v) { return wave_inclusive_dpp<false>(v); }

// Inclusive prefix maximum of non-negative values across the 64 lanes of a wave.
__device__ __forceinline__ int wave_inclusive_max(int v) { return wave_inclusive_dpp<true>(v); }

// Value of lane 63 (the total of an inclusive scan), wave-uniform.
__device__ __forceinline__ int wave_last(int v) { return __builtin_amdgcn_readlane(v, 63); }

// Workgroup-wide exclusive scan, from `base` up, of a[0..n) in LDS (16-byte
// aligned, room for n rounded up to 4, zero past n); returns base + the total.
// Each thread owns a contiguous run of whole 16-byte groups (one LDS read per
// four entries, no bank conflicts), the runs' sums are scanned inside each wave,
// and the waves' totals (tmp[0..NT/64)) are combined after one barrier.  `emit`
// receives every group (index, its four prefixes) as it is written back.  `add`
// is summed over the threads into every prefix (records before the first bin).
template <int NT, class Emit>
__device__ __forceinline__ int wg_exclusive_scan(int *a, int n, int *tmp, int add, Emit emit)
{
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = ((n + 4 * NT - 1) / (4 * NT)) * 4;
    const int beg = min(tid * per, n), end = min(beg + per, n);
    int s = 0;
    for (int i = beg; i < end; i += 4) {
        const v4i v = *reinterpret_cast<const v4i *>(a + i);
        s += (v[0] + v[1]) + (v[2] + v[3]);
    }
    const int inc = wave_inclusive_scan(s);
    const int before = wave_last(wave_inclusive_scan(add));
    if (lane == 63) {
        tmp[wave] = inc;
        tmp[NW + wave] = before;
    }
    __syncthreads();
    int run = inc - s, total = 0;
    _Pragma("unroll") for (int w = 0; w < NW; ++w)
    {
        const int t = tmp[w], u = tmp[NW + w];
        run += (w < wave ? t : 0) + u;
        total += t + u;
    }
    for (int i = beg; i < end; i += 4) {
        const v4i v = *reinterpret_cast<const v4i *>(a + i);
        v4i e;
        _Pragma("unroll") for (int k = 0; k < 4; ++k)
        {
            e[k] = run;
            run += v[k];
        }
        *reinterpret_cast<v4i *>(a + i) = e;
        emit(i, e);
    }
    __syncthreads();
    return total;
}

// Zeroes a[0..n rounded up to 4) (LDS, 16-byte aligned).
template <int NT>
__device__ __forceinline__ void lds_zero(int *a, int n)
{
    for (int i = 4 * (int)threadIdx.x; i < n; i += 4 * NT) *reinterpret_cast<v4i *>(a + i) = v4i{0, 0, 0, 0};
}

__device__ __forceinline__ int cell_coord(float v, float lo, float inv, int n)
{
    const float f = (v - lo) * inv;
    if (!(f >= 0.0f)) return 0;           // negative or NaN
    if (!(f < (float)n)) return n - 1;
    return (int)f;
}

// ------------------------------------------------------ image pyramid
// Level l of a pyramid is a bilinear resample of level 0 (Section IV-B: the
// pyramid is built on the device and kept for stereo; every level is computed
// from the image at once, so one launch builds them all).  Output index x of a
// level n_out wide samples s = ((2x + 1) * n_in - n_out) / (2 * n_out) of the
// level-0 axis n_in long: source pixel floor(s) and weight floor(256 * frac(s)),
// clamped to the first and last pixel.  Returns pixel | weight << 16.
//
// Both come from one quotient, t = floor(256 num / den): pixel t >> 8, weight
// t & 255.  num < 2^26, den <= 2^13 and t <= 2^20, so the reciprocal estimate is
// off by at most one, and the remainder, at most a few den in size, is exact
// modulo 2^32.
__device__ __forceinline__ uint32_t pyr_tap(int x, int n_in, int n_out)
{
    const int num = (2 * x + 1) * n_in - n_out;
    if (num <= 0) return 0u;
    const uint32_t den = 2u * (uint32_t)n_out;
    uint32_t t = (uint32_t)floorf((float)num * 256.0f * __builtin_amdgcn_rcpf((float)den));
    const int r = (int)(((uint32_t)num << 8) - t * den);
    t = r < 0 ? t - 1u : r >= (int)den ? t + 1u : t;
    const uint32_t q = t >> 8;
    return q >= (uint32_t)(n_in - 1) ? (uint32_t)(n_in - 1) : q | ((t & 255u) << 16);
}

// A wave's strip: 64 lanes of 4 output columns (level 0: 1024 bytes of a row,
// which may start up to 3 bytes past a dword boundary) by 2^pyr_rows_log2 rows.
// Sets the strips of each level as prefix sums.
constexpr int kPyrCols = 4, kPyrStripW = 64 * kPyrCols, kPyrCopyW = 1024;
void pyr_plan(DevJob &J, int rows_log2)
{
    J.pyr_rows_log2 = rows_log2;
    J.pyr_first[0] = 0;
    for (int l = 0; l < kLevels; ++l) {
        const int nx = l == 0 ? div_up(J.lv_w[0] + 3, kPyrCopyW) : div_up(J.lv_w[l], kPyrStripW);
        J.pyr_first[l + 1] = J.pyr_first[l] + nx * div_up(J.lv_h[l], 1 << rows_log2);
    }
}

// How a lane reads the taps of four neighbouring columns of a level that is
// 1 / s of the image.  From a dword boundary at or below the first tap, 16 bytes
// hold all four pixel pairs while s <= 11/3; realigned to the first tap, column
// k's pair starts floor(k s) or one more bytes in, so it lies in a fixed pair of
// dwords: the first two for every column while s <= 2 (kNear), later ones for
// columns 2 and 3 beyond (kMid, kFar); past 11/3 each column reads the dword pair
// that holds its own (kPairs).  kAny, for a strip that reaches the image's last
// bytes, reads the pixels one by one.
enum PyrReach { kNear, kMid, kFar, kPairs, kAny };

// Columns x .. x + 3 of output rows [ylo, yhi) of one level; `row_taps`: lane r
// holds the row tap of output row ylo + r.  A lane reads one aligned dwordx4
// per source row, realigns it (v_alignbyte), and blends a pixel pair per column
// with a byte permute and a 16-bit dot product; the two blended rows of an
// output row are combined by 24-bit multiply-adds.  All arithmetic is exact, so
// the order of the blends does not matter.  Up to s = 2 neighbouring output rows
// share source rows, so those are walked one after another and blended once;
// beyond, each output row takes its two.  (Misaligned vector loads take one
// lane per cycle here: a wave's dwordx2 33 cycles, its dwordx4 65, against 17
// aligned.)  Every dword read holds at least one byte of the image.
template <PyrReach kReach>
__device__ __forceinline__ void pyr_resample(const FT_G uint8_t *src, int W, int H, int pitch, FT_G uint8_t *dst, int wl,
                                             int x, int ylo, int yhi, uint32_t row_taps, bool full)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    constexpr bool kShared = kReach == kNear;
    uint32_t wgt[kPyrCols], sel[kPyrCols];
    int x0[kPyrCols];
    _Pragma("unroll") for (int k = 0; k < kPyrCols; ++k)
    {
        const uint32_t c = pyr_tap(min(x + k, wl - 1), W, wl);
        x0[k] = (int)(c & 0xFFFFu);
        const uint32_t a = c >> 16;
        wgt[k] = (256u - a) | (a << 16);
        const int first = kReach == kFar && k == 3 ? 8 : kReach >= kMid && k >= 2 ? 4 : 0;
        // bytes o and o + 1 of the dword pair as a 16-bit pair (0x0C: zero)
        sel[k] = 0x0C010C00u + 0x00010001u * (uint32_t)(x0[k] - x0[0] - first);
    }
    struct Row {
        uint32_t d[kReach == kPairs ? 2 * kPyrCols : 4];
    };
    auto load = [&](const FT_G uint8_t *row) {
        Row v;
        if constexpr (kReach == kAny) {   // (a pixel pair per column, in place)
            _Pragma("unroll") for (int k = 0; k < kPyrCols; ++k)
                v.d[k] = (uint32_t)row[x0[k]] | ((uint32_t)row[min(x0[k] + 1, W - 1)] << 16);
        } else if constexpr (kReach == kPairs) {
            typedef uint32_t v2u_dw __attribute__((ext_vector_type(2), aligned(4)));
            const uint32_t sh = (uint32_t)reinterpret_cast<uintptr_t>(row) & 3u;
            _Pragma("unroll") for (int k = 0; k < kPyrCols; ++k)
            {
                const v2u_dw q = *reinterpret_cast<const FT_G v2u_dw *>(row - sh + (((uint32_t)x0[k] + sh) & ~3u));
                v.d[2 * k] = q[0];
                v.d[2 * k + 1] = q[1];
            }
        } else {
            // (past the row's end lie the next row's bytes, whose weights are 0)
            const uint32_t sh = (uint32_t)reinterpret_cast<uintptr_t>(row) & 3u;
            const uint32_t off = ((uint32_t)x0[0] + sh) & ~3u;
            const v4u q = *reinterpret_cast<const FT_G v4u_dw *>(row - sh + off);
            _Pragma("unroll") for (int i = 0; i < 4; ++i) v.d[i] = q[i];
        }
        return v;
    };
    auto blend = [&](const Row &v, uint32_t sh, uint32_t h[kPyrCols]) {
        uint32_t e[4] = {v.d[0], v.d[1], v.d[2], v.d[3]};
        if constexpr (kReach < kPairs) {
            const uint32_t a = (uint32_t)x0[0] + sh;   // (v_alignbyte takes it modulo 4)
            _Pragma("unroll") for (int i = 0; i < 3; ++i) e[i] = __builtin_amdgcn_alignbyte(v.d[i + 1], v.d[i], a);
            e[3] = __builtin_amdgcn_alignbyte(0u, v.d[3], a);
        }
        _Pragma("unroll") for (int k = 0; k < kPyrCols; ++k)
        {
            const int j = kReach == kFar && k == 3 ? 2 : kReach >= kMid && k >= 2 ? 1 : 0;
            uint32_t pr;
            if constexpr (kReach == kAny) pr = e[k];
            else if constexpr (kReach == kPairs)   // bytes o and o + 1 of the pair, o the first one's place in its dword
                pr = __builtin_amdgcn_perm(v.d[2 * k + 1], v.d[2 * k], 0x0C010C00u + 0x00010001u * (((uint32_t)x0[k] + sh) & 3u));
            else pr = __builtin_amdgcn_perm(e[j + 1], e[j], sel[k]);
            h[k] = __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, pr), __builtin_bit_cast(u16x2, wgt[k]), 0u, false);
        }
    };
    FT_G uint8_t *d = dst + (size_t)ylo * wl + x;
    auto write = [&](const uint32_t top[kPyrCols], const uint32_t bot[kPyrCols], uint32_t b) {
        uint32_t o[kPyrCols];
        _Pragma("unroll") for (int k = 0; k < kPyrCols; ++k)
            o[k] = __umul24(bot[k], b) + (__umul24(top[k], 256u - b) + 32768u);
        // bits 16..23 of the four sums
        const uint32_t px = __builtin_amdgcn_perm(__builtin_amdgcn_perm(o[3], o[2], 0x0C0C0602u),
                                                  __builtin_amdgcn_perm(o[1], o[0], 0x0C0C0602u), 0x05040100u);
        if (full) {
            *reinterpret_cast<FT_G u32_any *>(d) = px;
        } else if (wl - x >= kPyrCols) {
            *reinterpret_cast<FT_G u32_any *>(d) = px;
        } else {
            _Pragma("unroll") for (int k = 0; k < kPyrCols - 1; ++k) if (k < wl - x) d[k] = (uint8_t)(px >> (8 * k));
        }
        d += wl;
    };
    auto tap_of = [&](int r) { return (uint32_t)__builtin_amdgcn_readlane((int)row_taps, r); };
    auto mod4 = [](const FT_G uint8_t *q) { return (uint32_t)reinterpret_cast<uintptr_t>(q) & 3u; };
    const int n_rows = yhi - ylo;
    uint32_t t = tap_of(0);
    if constexpr (kShared) {
        // every source row from the first tap to the one below the last; a row
        // whose predecessor is the next output row's tap completes that row
        constexpr int kChunk = 4;   // source rows whose loads are issued together
        const int y0 = (int)(t & 0xFFFFu), y1 = min((int)(tap_of(n_rows - 1) & 0xFFFFu) + 1, H - 1);
        uint32_t top[kPyrCols] = {};
        int r = 0;
        const FT_G uint8_t *row = src + (size_t)y0 * pitch;
        for (int y = y0; y <= y1; y += kChunk) {
            Row v[kChunk];
            const FT_G uint8_t *q = row;
            _Pragma("unroll") for (int u = 0; u < kChunk; ++u)
            {
                v[u] = load(q);
                if (y + u < y1) q += pitch;
            }
            _Pragma("unroll") for (int u = 0; u < kChunk; ++u)
            {
                if (y + u > y1) break;
                uint32_t bot[kPyrCols];
                blend(v[u], mod4(row), bot);
                row += pitch;
                if (y + u == (int)(t & 0xFFFFu) + 1) {
                    write(top, bot, t >> 16);
                    t = tap_of(min(++r, n_rows - 1));
                }
                _Pragma("unroll") for (int k = 0; k < kPyrCols; ++k) top[k] = bot[k];
            }
        }
        // the last output row's tap is the image's last row (its other weight is 0)
        if (r < n_rows) write(top, top, 0u);
    } else {
        // two source rows per output row
        constexpr int kChunk = 2;   // output rows whose loads are issued together
        for (int r0 = 0; r0 < n_rows; r0 += kChunk) {
            Row v[kChunk], w[kChunk];
            uint32_t sv[kChunk], sw[kChunk], b[kChunk];
            _Pragma("unroll") for (int u = 0; u < kChunk; ++u)
            {
                t = tap_of(min(r0 + u, n_rows - 1));
                const int ys = (int)(t & 0xFFFFu);
                const FT_G uint8_t *p0 = src + (size_t)ys * pitch, *p1 = ys < H - 1 ? p0 + pitch : p0;
                v[u] = load(p0);
                w[u] = load(p1);
                sv[u] = mod4(p0);
                sw[u] = mod4(p1);
                b[u] = t >> 16;
            }
            _Pragma("unroll") for (int u = 0; u < kChunk; ++u)
            {
                if (r0 + u >= n_rows) break;
                uint32_t top[kPyrCols], bot[kPyrCols];
                blend(v[u], sv[u], top);
                blend(w[u], sw[u], bot);
                write(top, bot, b[u]);
            }
        }
    }
}

// Rows [ylo, yhi) of a level at most 64 columns wide, a column per lane and byte
// loads: with four columns per lane most lanes idle, and a tall image's strips are
// bound by their number of instructions (16x4096: 7.2 us with four columns per lane,
// 5.3 with one).  Level 0 too: its taps are the pixels themselves.
__device__ __forceinline__ void pyr_narrow(const FT_G uint8_t *src, int W, int H, int pitch, FT_G uint8_t *dst, int wl,
                                           int ylo, int yhi, uint32_t row_taps)
{
    const int lane = threadIdx.x & 63;
    const uint32_t c = pyr_tap(min(lane, wl - 1), W, wl);
    const uint32_t a = c >> 16;
    const FT_G uint8_t *s0 = src + (c & 0xFFFFu), *s1 = src + min((int)(c & 0xFFFFu) + 1, W - 1);
    FT_G uint8_t *d = dst + (size_t)ylo * wl + lane;
    constexpr int kChunk = 4;   // output rows whose loads are issued together
    for (int r0 = 0; r0 < yhi - ylo; r0 += kChunk) {
        uint32_t p[kChunk][4], b[kChunk];
        _Pragma("unroll") for (int u = 0; u < kChunk; ++u)
        {
            const uint32_t t = (uint32_t)__builtin_amdgcn_readlane((int)row_taps, min(r0 + u, yhi - ylo - 1));
            const int ys = (int)(t & 0xFFFFu);
            const int64_t o0 = (int64_t)ys * pitch, o1 = (int64_t)min(ys + 1, H - 1) * pitch;
            p[u][0] = s0[o0];
            p[u][1] = s1[o0];
            p[u][2] = s0[o1];
            p[u][3] = s1[o1];
            b[u] = t >> 16;
        }
        _Pragma("unroll") for (int u = 0; u < kChunk; ++u)
        {
            const uint32_t top = p[u][0] * (256u - a) + p[u][1] * a, bot = p[u][2] * (256u - a) + p[u][3] * a;
            const uint32_t o = __umul24(bot, b[u]) + (__umul24(top, 256u - b[u]) + 32768u);
            if (r0 + u < yhi - ylo && lane < wl) d[0] = (uint8_t)(o >> 16);
            d += wl;
        }
    }
}

// Rows [ylo, yhi) of level 0: a lane takes dwords lane, lane + 64, .. of the
// 1024-byte strip bx of each destination row, counted from the row's dword
// boundary (neighbouring lanes on neighbouring dwords), realigned from the
// source's dwords, every one of which holds at least one byte of the row; the
// dwords at a row's two ends are written byte by byte.
__device__ __forceinline__ void pyr_copy(const FT_G uint8_t *src, int W, int pitch, FT_G uint8_t *dst, int bx, int ylo, int yhi)
{
    const int lane = threadIdx.x & 63;
    constexpr int kRows = 4, kDw = 4;   // rows and dwords per lane whose loads are issued together
    for (int y0 = ylo; y0 < yhi; y0 += kRows) {
        uint32_t lo[kRows][kDw], hi[kRows][kDw] = {};
        _Pragma("unroll") for (int r = 0; r < kRows; ++r)
        {
            const int y = min(y0 + r, yhi - 1);
            const FT_G uint8_t *s = src + (size_t)y * pitch;
            const int da = (int)(reinterpret_cast<uintptr_t>(dst + (size_t)y * W) & 3u);
            const int sa = (int)(reinterpret_cast<uintptr_t>(s) & 3u);
            const int sh = (sa - da) & 3;
            const FT_G uint32_t *dw = reinterpret_cast<const FT_G uint32_t *>(s - sa);
            const int last = (sa + W - 1) >> 2;
            const int d0 = (sa - da - sh) >> 2;   // source dword of the row's destination dword 0 (-1 or 0)
            _Pragma("unroll") for (int i = 0; i < kDw; ++i)
            {
                const int q = d0 + kPyrCopyW / 4 * bx + 64 * i + lane;
                lo[r][i] = dw[min(max(q, 0), last)];
                if (sh) hi[r][i] = dw[min(max(q + 1, 0), last)];
            }
        }
        _Pragma("unroll") for (int r = 0; r < kRows; ++r)
        {
            if (y0 + r >= yhi) break;
            FT_G uint8_t *row = dst + (size_t)(y0 + r) * W;
            const int da = (int)(reinterpret_cast<uintptr_t>(row) & 3u);
            const uint32_t sh = (uint32_t)(reinterpret_cast<uintptr_t>(src + (size_t)(y0 + r) * pitch) - (uintptr_t)da) & 3u;
            _Pragma("unroll") for (int i = 0; i < kDw; ++i)
            {
                const int p = 4 * (kPyrCopyW / 4 * bx + 64 * i + lane) - da;   // row offset of the dword
                const uint32_t e = __builtin_amdgcn_alignbyte(hi[r][i], lo[r][i], sh);
                if (p >= 0 && p + 4 <= W) {
                    *reinterpret_cast<FT_G uint32_t *>(row + p) = e;
                } else if (p < W) {
                    _Pragma("unroll") for (int k = 0; k < 4; ++k)
                        if (p + k >= 0 && p + k < W) row[p + k] = (uint8_t)(e >> (8 * k));
                }
            }
        }
    }
}

// One wave's strip of image `side` (0 left, 1 right) of the frame.  The strips
// read level 0 straight from memory (it stays in L2; up to seven levels read
// it), so there is no staging, no barrier and no shared tile: what bounds the
// build is vector issue and the strips' chains of loads, and a single image
// needs many short waves rather than few workgroups.  (1281x719, one image: 42.5
// us as 16-row workgroups with the rows staged in LDS, 7.2 us as strips; 16
// images of 752x480 in a batch: 29 us and 17 us.)
__device__ __forceinline__ void ph_pyramid(const DevJob &J, int tile)
{
    const int lane = threadIdx.x & 63;
    int u = tile * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int per = J.pyr_first[kLevels];
    const int side = u >= per ? 1 : 0;
    u -= side * per;
    const FT_G uint8_t *src = side ? J.imgR : J.imgL;
    FT_G uint8_t *dst = side ? J.pyr_outR : J.pyr_outL;
    if (u >= per || !src) return;
    const int W = J.img_w, H = J.img_h, pitch = J.img_pitch, rl = J.pyr_rows_log2;
    int l = 0, first = 0, wl = W, hl = H;
    int64_t off = 0;
    _Pragma("unroll") for (int k = 1; k < kLevels; ++k)
    {
        const bool in = u >= J.pyr_first[k];
        l = in ? k : l;
        first = in ? J.pyr_first[k] : first;
        wl = in ? J.lv_w[k] : wl;
        hl = in ? J.lv_h[k] : hl;
        off = in ? J.lv_off[k] : off;
    }
    // strips of a level column by column
    const int ny = (hl + (1 << rl) - 1) >> rl;
    int by = u - first, bx = 0;
    while (by >= ny) {
        by -= ny;
        ++bx;
    }
    const int ylo = by << rl, yhi = min(ylo + (1 << rl), hl);
    if (l == 0 && W > 64) {
        pyr_copy(src, W, pitch, dst, bx, ylo, yhi);
        return;
    }
    // Every lane stays active (lanes past the last column repeat it and write
    // nothing): lane r's tap is read by all.
    const uint32_t taps = pyr_tap(min(ylo + lane, hl - 1), H, hl);   // lane r: output row ylo + r (at most 64 rows)
    const int x = kPyrStripW * bx + kPyrCols * lane;
    FT_G uint8_t *out = dst + off;
    // (column 3's pair ends ceil(3 s) + 1 bytes after the first tap, which is up
    // to 3 past its dword: 16 bytes while 3 s <= 11; columns 2 and 3 start at
    // least 4 bytes in from s = 2, column 3 at least 9 from s = 10/3).  Beyond, two
    // dwords a column: with a scale factor of 2 a 1536x4096 image takes 8.6 us, read
    // pixel by pixel 17.5, and 1536x1080 6.3 and 11.4.
    const bool full = kPyrStripW * (bx + 1) <= wl;
    // a strip that reads the image's last row (its own last row's taps, or the one
    // before where the level is as tall as the image) and, with 16 bytes per
    // lane, past that row's end (the last lane within 24 columns of it)
    const bool corner = yhi >= hl - 1 && kPyrStripW * (bx + 1) + 20 >= wl;
    if (wl <= 64) pyr_narrow(src, W, H, pitch, out, wl, ylo, yhi, taps);
    else if (corner) pyr_resample<kAny>(src, W, H, pitch, out, wl, x, ylo, yhi, taps, full);
    else if (W <= 2 * wl) pyr_resample<kNear>(src, W, H, pitch, out, wl, x, ylo, yhi, taps, full);
    else if (3 * W <= 10 * wl) pyr_resample<kMid>(src, W, H, pitch, out, wl, x, ylo, yhi, taps, full);
    else if (3 * W > 11 * wl) pyr_resample<kPairs>(src, W, H, pitch, out, wl, x, ylo, yhi, taps, full);
    else pyr_resample<kFar>(src, W, H, pitch, out, wl, x, ylo, yhi, taps, full);
}

// ------------------------------------------------ setup: rows (pinhole)
// Row bin of a right keypoint (clamped; non-finite rows go to bin 0).
__device__ __forceinline__ int row_bin(float y, int rows)
{
    if (!(y >= 0.0f)) return 0;
    if (!(y < (float)rows)) return rows - 1;
    return (int)y;
}

// Packed rows [lo, hi] of the epipolar band of a right keypoint, or an empty
// range (lo > hi).
__device__ __forceinline__ uint32_t band_rows(const DevJob &J, float y, int oct)
{
    const float r = J.band * J.sf[lvl(oct)];
    const float flo = floorf(y - r);
    const float fhi = ceilf(y + r);
    if (!(fhi >= 0.0f) || !(flo <= (float)(J.rows - 1))) return 0xFFFFu;  // lo = 65535 > hi = 0
    const int lo = flo < 0.0f ? 0 : (int)flo;
    const int hi = fhi > (float)(J.rows - 1) ? J.rows - 1 : (int)fhi;
    return (uint32_t)lo | ((uint32_t)hi << 16);
}

// Levels [part * kLevels / parts, ..) of the row sort, one workgroup each
// (`parts` = 1: the one bin of every level).  A workgroup reads every right
// keypoint and keeps its own levels'; the records of lower levels are counted
// on the way, so the parts need nothing from each other.
template <int NT>
__device__ __forceinline__ void ph_rowsort(const DevJob &J, int part, int parts, int *cnt, int *tmp)
{
    const int tid = threadIdx.x;
    const int rows = J.rows, nR = J.R.n;
    const int b0 = part * J.n_lb / parts, b1 = (part + 1) * J.n_lb / parts, nb = (b1 - b0) * rows;
    const bool per_level = J.n_lb > 1;
    lds_zero<NT>(cnt, nb);
    for (int j = part * NT + tid; j < nR; j += parts * NT) J.claimR[j] = 0xFFFFFFFFu;
    for (int i = part * NT + tid; i < J.L.n; i += parts * NT) J.flag[i] = 0;   // the refinement flags matches only
    if (part == 0 && tid == 0) J.counts[2] = 0;                                // length of the match list
    __syncthreads();
    // A chunk of kSortUnroll right keypoints per thread; the first chunk stays
    // in registers from the counting pass to the scatter.
    auto load = [&](int j0, float *x, float *y, int *oc) {
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
        {
            const int j = min(j0 + e * NT, nR - 1);
            x[e] = J.R.x[j];
            y[e] = J.R.y[j];
            oc[e] = J.R.oct[j];
        }
    };
    // bin of this part, or -1 (a lower level: -2)
    auto bin_of = [&](float y, int oc) {
        const int lb = per_level ? lvl(oc) : 0;
        return lb < b0 ? -2 : lb >= b1 ? -1 : (lb - b0) * rows + row_bin(y, rows);
    };
    int lower = 0;
    auto count = [&](int j0, const float *y, const int *oc) {
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
        {
            if (j0 + e * NT < nR) {
                const int b = bin_of(y[e], oc[e]);
                if (b >= 0) atomicAdd(&cnt[b], 1);
                lower += b == -2 ? 1 : 0;
            }
        }
    };
    auto scatter = [&](int j0, const float *x, const float *y, const int *oc) {
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
        {
            const int j = j0 + e * NT;
            const int b = j < nR ? bin_of(y[e], oc[e]) : -1;
            if (b >= 0) {
                const int pos = atomicAdd(&cnt[b], 1);
                RowRec rec;
                rec.x = x[e];
                rec.band = band_rows(J, y[e], oc[e]);
                rec.meta = (uint32_t)oc[e] | ((uint32_t)j << 16);
                rec.pad = 0;
                J.rrec[pos] = rec;
            }
        }
    };
    float x0[kSortUnroll], y0[kSortUnroll];
    int oc0[kSortUnroll];
    if (tid < nR) {
        load(tid, x0, y0, oc0);
        count(tid, y0, oc0);
    }
    for (int j0 = tid + kSortUnroll * NT; j0 < nR; j0 += kSortUnroll * NT) {
        float x[kSortUnroll], y[kSortUnroll];
        int oc[kSortUnroll];
        load(j0, x, y, oc);
        count(j0, y, oc);
    }
    __syncthreads();
    const int total = wg_exclusive_scan<NT>(cnt, nb, tmp, lower, [](int, v4i) {});
    // row_start[lb][r] = first record of (lb, r); row_start[lb][rows] = end of level bin lb
    for (int e = tid; e < (b1 - b0) * (rows + 1); e += NT) {
        const int lb = e / (rows + 1), r = e - lb * (rows + 1);
        const int bin = lb * rows + r;
        J.row_start[b0 * (rows + 1) + e] = bin < nb ? cnt[bin] : total;
    }
    __syncthreads();
    if (tid < nR) scatter(tid, x0, y0, oc0);
    for (int j0 = tid + kSortUnroll * NT; j0 < nR; j0 += kSortUnroll * NT) {
        float x[kSortUnroll], y[kSortUnroll];
        int oc[kSortUnroll];
        load(j0, x, y, oc);
        scatter(j0, x, y, oc);
    }
}

// ------------------------------------------- setup: overlap lists (fisheye)
// Indices i < n with a <= x[i] <= b, in order, into out[]; with `desc`, their
// descriptors in the same order into tdesc and their all-pairs keys (256 +
// popcount) << 16 | position into tkey.  U keypoints per thread
// and round, their loads together; a round's counts per (keypoint, wave) are
// scanned by every wave after one barrier.
template <int NT, int U>
__device__ __forceinline__ int compact_range(const FT_G float *x, int n, float a, float b, FT_G int32_t *out,
                                             const FT_G uint8_t *desc, FT_G uint8_t *tdesc, FT_G uint32_t *tkey, int *wcnt)
{
    constexpr int NW = NT / 64;
    static_assert(U * NW <= 64, "one lane per (keypoint, wave) count");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const FT_G v4u *src = reinterpret_cast<const FT_G v4u *>(desc);
    FT_G v4u *dst = reinterpret_cast<FT_G v4u *>(tdesc);
    int base = 0;
    for (int s = 0; s < n; s += U * NT) {
        bool p[U];
        int rank[U];
        v4u d[U][2];
        _Pragma("unroll") for (int e = 0; e < U; ++e)
        {
            const int i = s + e * NT + tid;
            const float v = x[min(i, n - 1)];
            p[e] = i < n && v >= a && v <= b;
            if (desc && p[e]) {
                d[e][0] = src[2 * (size_t)i];
                d[e][1] = src[2 * (size_t)i + 1];
            }
        }
        _Pragma("unroll") for (int e = 0; e < U; ++e)
        {
            const unsigned long long m = __ballot(p[e]);
            rank[e] = __popcll(m & ((1ull << lane) - 1ull));
            if (lane == 0) wcnt[e * NW + wave] = __popcll(m);
        }
        __syncthreads();
        const int inc = wave_inclusive_scan(lane < U * NW ? wcnt[lane] : 0);
        _Pragma("unroll") for (int e = 0; e < U; ++e)
        {
            const int j = e * NW + wave;
            const int pos = base + rank[e] + (j ? __builtin_amdgcn_readlane(inc, (j - 1) & 63) : 0);
            if (p[e]) {
                out[pos] = s + e * NT + tid;
                if (desc) {
                    dst[2 * (size_t)pos] = d[e][0];
                    dst[2 * (size_t)pos + 1] = d[e][1];
                    int pop = 0;
                    _Pragma("unroll") for (int w = 0; w < 4; ++w) pop += __popc(d[e][0][w]) + __popc(d[e][1][w]);
                    tkey[pos] = ((256u + (uint32_t)pop) << 16) | (uint32_t)pos;
                }
            }
        }
        base += wave_last(inc);
        __syncthreads();   // the counts are free for the next round
    }
    return base;
}

// Part 0: the query list; part 1: the target list and the targets' descriptors
// in its order.
template <int NT>
__device__ __forceinline__ void ph_overlap(const DevJob &J, int part, int *wcnt)
{
    const int tid = threadIdx.x;
    if (part == 0) {
        for (int i = tid; i < J.L.n; i += NT) J.flag[i] = 0;
        const int nQ = compact_range<NT, kSortUnroll>(J.L.x, J.L.n, J.ovl[0], J.ovl[1], J.qlist, nullptr, nullptr, nullptr, wcnt);
        if (tid == 0) {
            J.counts[0] = nQ;
            *J.o_nmatch = 0;
        }
    } else {
        for (int j = tid; j < J.R.n; j += NT) J.claimR[j] = 0xFFFFFFFFu;
        const int nT = compact_range<NT, 2>(J.R.x, J.R.n, J.ovr[0], J.ovr[1], J.tlist, J.R.desc, J.tdesc, J.tkey, wcnt);
        if (tid == 0) J.counts[1] = nT;
    }
}

// ------------------------------------------------ setup: keypoint grid
// Level bins of the cell index that hold a keypoint of octave o: the bins p
// whose octave window p - lv_lo .. p + lv_hi contains o, i.e. the predicted
// levels of the map points that may match it; one bin when the index is not
// binned.
__device__ __forceinline__ void cell_bins(const DevView &V, int o, int lv_lo, int lv_hi, int &p0, int &p1)
{
    if (V.n_pb == 1) {
        p0 = p1 = 0;
        return;
    }
    p0 = max(o - lv_hi, 0);
    p1 = min(o + lv_lo, kLevels - 1);
}

// Counting sort of the view's keypoints by (level bin, row, column) into
// 16-byte records; a keypoint is copied into every bin that holds its octave.
// One workgroup per part: level bins [part * n_pb / parts, ..), each reading
// every keypoint and counting the copies that go to lower bins, so the parts
// need nothing from each other.
template <int NT>
__device__ __forceinline__ void ph_cellsort(const DevView &V, const DevKps &K, int lv_lo, int lv_hi, int part, int parts,
                                            int *cnt, int *tmp)
{
    const int tid = threadIdx.x;
    const int cells = V.cols * V.rows;
    const int b0 = part * V.n_pb / parts, b1 = (part + 1) * V.n_pb / parts, nb = (b1 - b0) * cells;
    lds_zero<NT>(cnt, nb);
    for (int k = part * NT + tid; k < K.n; k += parts * NT) V.claim[k] = 0xFFFFFFFFu;
    if (part == 0) {
        for (int b = tid; b < kRotBinsMax; b += NT) V.hist[b] = 0;
        if (tid == 0) *V.n_matches = 0;
    }
    __syncthreads();
    // A chunk of kSortUnroll keypoints per thread: the position and record meta
    // of each (load), its counts (count) and its records (scatter).  The first
    // chunk stays in registers from the counting pass to the scatter, so a view
    // of up to kSortUnroll * NT keypoints is read once per part.
    auto load = [&](int k0, float *x, float *y, uint32_t *meta) {
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
        {
            const int k = min(k0 + e * NT, K.n - 1);
            x[e] = K.x[k];
            y[e] = K.y[k];
            const uint32_t pre = (V.preassigned && V.preassigned[k]) ? 1u : 0u;
            meta[e] = (uint32_t)K.oct[k] | (pre << 8) | ((uint32_t)k << 16);
        }
    };
    auto cell_of = [&](float x, float y) {
        return cell_coord(y, V.min_y, V.inv_ch, V.rows) * V.cols + cell_coord(x, V.min_x, V.inv_cw, V.cols);
    };
    int lower = 0;
    auto count = [&](int k0, const float *x, const float *y, const uint32_t *meta) {
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
        {
            if (k0 + e * NT < K.n) {
                int q0, q1;
                cell_bins(V, (int)(meta[e] & 0xFFu), lv_lo, lv_hi, q0, q1);
                lower += max(min(q1 + 1, b0) - q0, 0);
                const int p0 = max(q0, b0), p1 = min(q1, b1 - 1);
                int c = (p0 - b0) * cells + cell_of(x[e], y[e]);
                for (int p = p0; p <= p1; ++p, c += cells) atomicAdd(&cnt[c], 1);
            }
        }
    };
    auto scatter = [&](int k0, const float *x, const float *y, const uint32_t *meta) {
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
        {
            if (k0 + e * NT < K.n) {
                CellRec rec;
                rec.x = x[e];
                rec.y = y[e];
                rec.meta = meta[e];
                rec.pad = 0;
                int q0, q1;
                cell_bins(V, (int)(meta[e] & 0xFFu), lv_lo, lv_hi, q0, q1);
                const int p0 = max(q0, b0), p1 = min(q1, b1 - 1);
                int c = (p0 - b0) * cells + cell_of(x[e], y[e]);
                for (int p = p0; p <= p1; ++p, c += cells) V.crec[atomicAdd(&cnt[c], 1)] = rec;
            }
        }
    };
    float x0[kSortUnroll], y0[kSortUnroll];
    uint32_t meta0[kSortUnroll];
    if (tid < K.n) {
        load(tid, x0, y0, meta0);
        count(tid, x0, y0, meta0);
    }
    for (int k0 = tid + kSortUnroll * NT; k0 < K.n; k0 += kSortUnroll * NT) {
        float x[kSortUnroll], y[kSortUnroll];
        uint32_t meta[kSortUnroll];
        load(k0, x, y, meta);
        count(k0, x, y, meta);
    }
    __syncthreads();
    FT_G int32_t *off = V.cell_off + b0 * cells;
    const int total = wg_exclusive_scan<NT>(cnt, nb, tmp, lower, [&](int i, v4i e) {
        if (i + 4 <= nb) {
            *reinterpret_cast<FT_G v4u_dw *>(off + i) = __builtin_bit_cast(v4u, e);
        } else {
            _Pragma("unroll") for (int k = 0; k < 3; ++k) if (i + k < nb) off[i + k] = e[k];
        }
    });
    if (part == parts - 1 && tid == 0) off[nb] = total;
    if (tid < K.n) scatter(tid, x0, y0, meta0);
    for (int k0 = tid + kSortUnroll * NT; k0 < K.n; k0 += kSortUnroll * NT) {
        float x[kSortUnroll], y[kSortUnroll];
        uint32_t meta[kSortUnroll];
        load(k0, x, y, meta);
        scatter(k0, x, y, meta);
    }
}

// ------------------------------------- stereo_a (pinhole): row-band best match
// Level bins of the row index a left keypoint of octave oi scans: the bins of
// octaves oi - level_window .. oi + level_window (clamped into the table;
// octaves above the last level share its bin), or the one bin of all levels.
__device__ __forceinline__ void level_bins(const DevJob &J, int oi, int &lb0, int &lb1)
{
    if (J.n_lb == 1) {
        lb0 = lb1 = 0;
        return;
    }
    lb0 = min(max(oi - J.level_window, 0), kLevels - 1);
    lb1 = min(max(oi + J.level_window, 0), kLevels - 1);
}

// G lanes per left keypoint.  The candidates of row r are the right keypoints
// whose band covers r; their integer rows lie within J.row_reach of r, so the
// lanes stream the row-sorted records of those bins and test the band exactly.
// Appends the wave's accepted pinhole matches to the frame's match list, one
// counter update per wave; the list order does not matter (the refinement
// writes by left keypoint).  Every lane of the wave calls it.
__device__ __forceinline__ void append_match(const DevJob &J, bool take, const MatchRec &r)
{
    const unsigned long long bal = __ballot(take);
    if (bal == 0ull) return;
    const int lane = threadIdx.x & 63;
    const int leader = __ffsll((long long)bal) - 1;
    int base = 0;
    if (lane == leader) base = atomicAdd(&J.counts[2], (int)__popcll(bal));
    base = __shfl(base, leader);
    if (take) J.mrec[base + (int)__popcll(bal & ((1ull << lane) - 1ull))] = r;
}

__device__ __forceinline__ MatchRec match_rec(int i, uint32_t best, float bx, float x, float y, int oi)
{
    MatchRec r;
    r.i = i;
    r.j = (int)(best & 0xFFFFu);
    r.h = (int)(best >> 16);
    r.bx = bx;
    r.x = x;
    r.y = y;
    r.oct = oi;
    r.pad = 0;
    return r;
}

// Records [s, s + n) of level bin lb whose integer rows lie within that bin's
// reach of row.
__device__ __forceinline__ void bin_range(const DevJob &J, int lb, int row, int &s, int &n)
{
    const int reach = pick_level(J.lv_reach, lb);
    const FT_G int32_t *rs = J.row_start + lb * (J.rows + 1);
    s = rs[max(row - reach, 0)];
    n = rs[min(row + reach, J.rows - 1) + 1] - s;
}

template <int G>
__device__ __forceinline__ void ph_best(const DevJob &J, int tile)
{
    const int sub = threadIdx.x % G;
    const int i = tile * (kWG / G) + threadIdx.x / G;
    uint32_t best = 0xFFFFFFFFu;   // Hamming << 16 | right index
    float bx = 0.0f;               // x of that right keypoint (for the refinement)
    float x = 0.0f, y = 0.0f;
    int oi = 0;
    if (i < J.L.n) {
        y = J.L.y[i];
        x = J.L.x[i];
        oi = J.L.oct[i];
        const float minU = x - J.maxD;
        const float maxU = x - 0.0f;
        if (y > -1.0f && y < (float)J.rows && !(maxU < 0.0f)) {
            const int row = (int)y;
            const Desc di = load_desc(J.L.desc, i);
            int lb0, lb1;
            level_bins(J, oi, lb0, lb1);
            auto test = [&](const RowRec &rec) {
                const int lo = (int)(rec.band & 0xFFFFu), hi = (int)(rec.band >> 16);
                const int oj = (int)(rec.meta & 0xFFu);
                return row >= lo && row <= hi && oj >= oi - J.level_window && oj <= oi + J.level_window &&
                       rec.x >= minU && rec.x <= maxU;
            };
            auto push = [&](const RowRec &rec, const Desc &d) {
                const uint32_t key = ((uint32_t)hamming(di, d) << 16) | (rec.meta >> 16);
                if (key < best) {
                    best = key;
                    bx = rec.x;
                }
            };
            if (lb1 - lb0 < 3) {
                // Up to three bins: their ranges are read together, positions
                // 0 .. total - 1 run over them in order, lane `sub` taking every
                // G-th, kBestUnroll per step; a step's descriptors load together
                // with the next step's records.  (The minimum over distinct
                // keys does not depend on the order.)
                int s0, n0, s1 = 0, n1 = 0, s2 = 0, n2 = 0;
                bin_range(J, lb0, row, s0, n0);
                if (lb0 + 1 <= lb1) bin_range(J, lb0 + 1, row, s1, n1);
                if (lb0 + 2 <= lb1) bin_range(J, lb0 + 2, row, s2, n2);
                const int n01 = n0 + n1, total = n01 + n2;
                auto at = [&](int p) {
                    p = min(p, total - 1);   // past the end: a record loaded and never used
                    return J.rrec[p < n0 ? s0 + p : p < n01 ? s1 + (p - n0) : s2 + (p - n01)];
                };
                RowRec rec[kBestUnroll];
                if (total > 0) {
                    _Pragma("unroll") for (int u = 0; u < kBestUnroll; ++u) rec[u] = at(sub + u * G);
                }
                for (int p0 = sub; p0 < total; p0 += kBestUnroll * G) {
                    bool cand[kBestUnroll];
                    Desc d[kBestUnroll];
                    _Pragma("unroll") for (int u = 0; u < kBestUnroll; ++u)
                    {
                        cand[u] = p0 + u * G < total && test(rec[u]);
                        if (cand[u]) d[u] = load_desc(J.R.desc, (int)(rec[u].meta >> 16));
                    }
                    RowRec nx[kBestUnroll];
                    _Pragma("unroll") for (int u = 0; u < kBestUnroll; ++u) nx[u] = at(p0 + (kBestUnroll + u) * G);
                    _Pragma("unroll") for (int u = 0; u < kBestUnroll; ++u) if (cand[u]) push(rec[u], d[u]);
                    _Pragma("unroll") for (int u = 0; u < kBestUnroll; ++u) rec[u] = nx[u];
                }
            } else {
                // any number of bins, one after another
                for (int lb = lb0; lb <= lb1; ++lb) {
                    int s, n;
                    bin_range(J, lb, row, s, n);
                    const int p1 = s + n;
                    // kBestUnroll records per step are loaded together (indices
                    // clamped into the range, surplus entries masked); then the
                    // descriptors of the candidates among them.
                    for (int p0 = s + sub; p0 < p1; p0 += kBestUnroll * G) {
                        RowRec rec[kBestUnroll];
                        bool cand[kBestUnroll];
                        Desc d[kBestUnroll];
                        _Pragma("unroll") for (int u = 0; u < kBestUnroll; ++u) rec[u] = J.rrec[min(p0 + u * G, p1 - 1)];
                        _Pragma("unroll") for (int u = 0; u < kBestUnroll; ++u)
                        {
                            cand[u] = p0 + u * G < p1 && test(rec[u]);
                            if (cand[u]) d[u] = load_desc(J.R.desc, (int)(rec[u].meta >> 16));
                        }
                        _Pragma("unroll") for (int u = 0; u < kBestUnroll; ++u) if (cand[u]) push(rec[u], d[u]);
                    }
                }
            }
        }
    }
    for (int m = 1; m < G; m <<= 1) {
        const uint32_t o = __shfl_xor(best, m);
        const float ox = __shfl_xor(bx, m);
        if (o < best) {
            best = o;
            bx = ox;
        }
    }
    const int h = (int)(best >> 16);
    const bool ok = best != 0xFFFFFFFFu && h < J.th_orb;
    if (sub == 0 && i < J.L.n) {
        J.best_j[i] = ok ? (int)(best & 0xFFFFu) : -1;
        J.best_h[i] = ok ? h : -1;
    }
    append_match(J, sub == 0 && i < J.L.n && ok, match_rec(i, best, bx, x, y, oi));
}

// ----------------------------- stereo_a (fisheye): all-pairs top-2 on MFMA
// H(a, b) = popcount(a) + popcount(b) - 2 popcount(a & b), the last term an int8
// dot product over the descriptors' bits.  An operand byte need not be 0 or 1: a
// target's bit t of a byte enters as that bit in place, 2^t (bit 7 as -128), so
// that four operand bytes are one masked descriptor word; a query's bit t enters
// as -2^(7 - t) (bit 7 as 1), so every pair of set bits adds -128, exactly.  (A
// +-1 expansion of both operands takes a table lookup per byte, 8 conflicting
// LDS reads and their indices per lane and tile, against 16 masks.)
// Each lane group g (lanes 16g..16g+15) supplies descriptor bytes 8g..8g+7 over
// the four K-steps of v_mfma_i32_16x16x64_i8 (bits 4h .. 4h + 3 of the bytes of
// one word per step); the A and B operands use the same bit-to-K assignment, so
// the dot product is the full 256-term sum whatever order the hardware sums K in.
// Top-2 of 32-bit keys by value (keys are distinct: they carry the target
// index).  a <= b always holds, so the new second is the median of a, b and
// the key, one v_med3_u32; the new best is min(a, key).
__device__ __forceinline__ void top2_push(uint32_t &a, uint32_t &b, uint32_t key)
{
    uint32_t m;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(m) : "v"(a), "v"(b), "v"(key));
    b = m;
    a = min(a, key);
}

// Target operand: bits 4 half .. 4 half + 3 of the word's bytes, in place.
__device__ __forceinline__ v4i target_bits(uint32_t word, int half)
{
    v4i v;
    _Pragma("unroll") for (int k = 0; k < 4; ++k) v[k] = (int)(word & (0x01010101u << (4 * half + k)));
    return v;
}

// Query operand of the same bits: bit t as -2^(7 - t), bit 7 as 1 (a byte holds
// 0 or 1 times 256 - 2^(7 - t), so the product never carries).
__device__ __forceinline__ v4i query_bits(uint32_t word, int half)
{
    v4i v;
    _Pragma("unroll") for (int k = 0; k < 4; ++k)
    {
        const int t = 4 * half + k;
        v[k] = (int)(((word >> t) & 0x01010101u) * (t == 7 ? 1u : 256u - (128u >> t)));
    }
    return v;
}

// One halving step of the top-2 lists of 2 N rows over a row of 16 lanes: a lane
// keeps N of them (the upper N when `upper`), gives the others to its partner
// (DPP control kCtrl, an exchange with a lane of the other half) and merges what
// the partner gives.
template <int N, int kCtrl>
__device__ __forceinline__ void top2_halve(uint32_t *ta, uint32_t *tb, bool upper)
{
    _Pragma("unroll") for (int i = 0; i < N; ++i)
    {
        const uint32_t ka = upper ? ta[i + N] : ta[i], kb = upper ? tb[i + N] : tb[i];
        const uint32_t sa = upper ? ta[i] : ta[i + N], sb = upper ? tb[i] : tb[i + N];
        const uint32_t oa = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sa, kCtrl, 0xF, 0xF, false);
        const uint32_t ob = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sb, kCtrl, 0xF, 0xF, false);
        const Top2<uint32_t> t = top2_merge(Top2<uint32_t>{ka, kb}, oa, ob);
        ta[i] = t.a;
        tb[i] = t.b;
    }
}

// Fisheye all-pairs top-2 on the matrix cores.  A workgroup subgroup (256
// threads) owns kKnnQueriesPerWG queries; its four waves split the target
// tiles, and the partial top-2 lists are merged in LDS (`part`: 4 x
// kKnnQueriesPerWG x 2 words per subgroup).  Each wave holds the operands of all
// its queries (QB blocks of 16) and expands every 16-target tile once for all QB
// blocks.  Every thread reaches the barrier.
// Bound by vector instructions (32 keys and 16 masks per lane and tile beside 8
// MFMAs): 64 fisheye frames of 1500 keypoints 44.0 us with +-1 operands from a
// table, a key assembled per column and shuffles at the end, 38.9 now; the mixed
// 64-frame batch 167.4 -> 165.2.  Pushing a tile's keys while the next one's
// MFMAs run takes 25 registers more and loses in the batch (168.5).
template <int NT>
__device__ __forceinline__ void ph_knn(const DevJob &J, int tile, uint32_t *part)
{
    constexpr int QB = kKnnQueriesPerWG / 16;
    const int tid = threadIdx.x, ltid = tid & 255, sg = tid >> 8;
    const int nQ = J.counts[0], nT = J.counts[1];
    const int q0 = (tile * (NT / 256) + sg) * kKnnQueriesPerWG;
    part += sg * (4 * kKnnQueriesPerWG * 2);
    const bool active = q0 < nQ && nT >= 2;   // uniform over the subgroup
    const int lane = ltid & 63, wave = ltid >> 6, g = lane >> 4, c = lane & 15;
    if (active) {
    v4i A[QB][4];
    _Pragma("unroll") for (int qb = 0; qb < QB; ++qb)
    {
        // (queries past the last: no bits)
        const int qa = q0 + 16 * qb + c;
        uint2 w = make_uint2(0, 0);
        if (qa < nQ) w = *reinterpret_cast<const uint2 *>(J.L.desc + 32 * (size_t)J.qlist[qa] + 8 * g);
        _Pragma("unroll") for (int s = 0; s < 4; ++s) A[qb][s] = query_bits(s < 2 ? w.x : w.y, s & 1);
    }
    uint32_t ta[QB * 4], tb[QB * 4];
    _Pragma("unroll") for (int r = 0; r < QB * 4; ++r) ta[r] = tb[r] = 0xFFFFFFFFu;
    // (wave-uniform, so that the loop below branches on scalars)
    const int n_tiles = __builtin_amdgcn_readfirstlane((nT + 15) >> 4);
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    // A ring of kKnnTilesInFlight target tiles' descriptor bytes and keys per
    // wave: the loop is unrolled over the ring, and a slot is reloaded with the
    // tile kKnnTilesInFlight steps ahead as soon as its bytes are expanded, so
    // that several loads are in flight while the matrix cores work.
    constexpr int D = kKnnTilesInFlight;
    const FT_G uint8_t *tdesc = J.tdesc + 8 * g;
    struct Slot {
        uint2 w;
        uint32_t key;
    };
    auto load = [&](int tj) {
        tj = min(tj, nT - 1);
        typedef uint32_t v2u __attribute__((ext_vector_type(2)));
        const v2u w = *reinterpret_cast<const FT_G v2u *>(tdesc + 32 * (size_t)tj);
        return Slot{make_uint2(w[0], w[1]), J.tkey[tj]};
    };
    Slot ring[D];
    _Pragma("unroll") for (int d = 0; d < D; ++d) ring[d] = load(((wv + 4 * d) << 4) + c);
    // one tile: expand its bytes from ring slot d (then refill the slot with
    // the tile D steps ahead), run the MFMAs, push the column's keys
    auto step = [&](Slot &slot, int t, bool refill) {
        // (a column past the end holds the last target's bytes; its keys are above
        // every other, and at least two targets are valid, so they never survive)
        const uint32_t key = (t << 4) + c < nT ? slot.key : 0xC0000000u;
        v4i B[4], acc[QB];
        _Pragma("unroll") for (int s = 0; s < 4; ++s) B[s] = target_bits(s < 2 ? slot.w.x : slot.w.y, s & 1);
        if (refill) slot = load((t << 4) + c + 64 * D);
        // acc[r] = -128 popcount(a & b) of query row 4g + r of block qb and target
        // column c, so key + (acc << 10) = (256 + H - popcount(a)) << 16 | position,
        // one shift-add; the query's own count is added at the end.  The blocks'
        // MFMA chains are interleaved so that each hides the other's latency.
        _Pragma("unroll") for (int qb = 0; qb < QB; ++qb) acc[qb] = v4i{0, 0, 0, 0};
        _Pragma("unroll") for (int s = 0; s < 4; ++s)
            _Pragma("unroll") for (int qb = 0; qb < QB; ++qb)
                acc[qb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[qb][s], B[s], acc[qb], 0, 0, 0);
        _Pragma("unroll") for (int qb = 0; qb < QB; ++qb)
            _Pragma("unroll") for (int r = 0; r < 4; ++r)
                top2_push(ta[4 * qb + r], tb[4 * qb + r], key + ((uint32_t)acc[qb][r] << 10));
    };
    // whole turns of the ring (no exit inside, so the loads' waits stay
    // counted), then the last tiles with no refill
    int t0 = wv;
    for (; t0 + 4 * (D - 1) < n_tiles; t0 += 4 * D)
        _Pragma("unroll") for (int d = 0; d < D; ++d) step(ring[d], t0 + 4 * d, true);
    _Pragma("unroll") for (int d = 0; d < D - 1; ++d)
        if (t0 + 4 * d < n_tiles) step(ring[d], t0 + 4 * d, false);
    // The lists of the 8 rows (4 qb + r) merged over the 16 columns: lanes halve
    // the rows they hold with the lane at c ^ 8, c ^ 7 and c ^ 3, so that lane c
    // ends with row c >> 1, then merge with the lane at c ^ 1.
    static_assert(QB == 2, "eight rows per lane");
    top2_halve<4, 0x128>(ta, tb, c & 8);   // row_ror:8
    top2_halve<2, 0x141>(ta, tb, c & 4);   // row_half_mirror
    top2_halve<1, 0x1B>(ta, tb, c & 2);    // quad_perm 3,2,1,0
    {
        const uint32_t oa = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ta[0], 0xB1, 0xF, 0xF, false);   // quad_perm 1,0,3,2
        const uint32_t ob = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)tb[0], 0xB1, 0xF, 0xF, false);
        const Top2<uint32_t> t = top2_merge(Top2<uint32_t>{ta[0], tb[0]}, oa, ob);
        const int r = c >> 1;
        if ((c & 1) == 0) {
            uint32_t *pw = part + (wave * kKnnQueriesPerWG + 16 * (r >> 2) + 4 * g + (r & 3)) * 2;
            pw[0] = t.a;
            pw[1] = t.b;
        }
    }
    }
    __syncthreads();
    if (active && ltid < kKnnQueriesPerWG && q0 + ltid < nQ) {
        Top2<uint32_t> t = {part[ltid * 2], part[ltid * 2 + 1]};
        for (int w = 1; w < 4; ++w)
            t = top2_merge(t, part[(w * kKnnQueriesPerWG + ltid) * 2], part[(w * kKnnQueriesPerWG + ltid) * 2 + 1]);
        const int i = J.qlist[q0 + ltid];
        const Desc d = load_desc(J.L.desc, i);
        const int pop = hamming(d, Desc{make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0)}) - 256;
        J.best_j[i] = J.tlist[t.a & 0xFFFFu];
        J.best_h[i] = (int)(t.a >> 16) + pop;
        J.h2[i] = (int)(t.b >> 16) + pop;
    }
}

// ------------------------------------- stereo_b (pinhole): SAD refinement
// One wave per match.  The wave stages the left patch and the right strip of
// the left keypoint's level in LDS, then 64 lanes split the (shift, row) sums.
// General window sizes: one wave per match, lanes split the (shift, row) sums.
__device__ __forceinline__ void ph_refine_wave(const DevJob &J, int tile, uint8_t *lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int idx = tile * kRefinePerWG + wave;   // position in the frame's match list
    const bool has = idx < J.counts[2];
    const MatchRec mr = J.mrec[min(idx, max(J.L.n - 1, 0))];   // loaded with the list length
    const int i = mr.i;
    const int w = J.half_win, L = J.half_range;
    const int side = 2 * w + 1, strip = 2 * (L + w) + 1, nS = 2 * L + 1;
    int j = -1, l = 0, su = 0, sv = 0, su0 = 0, Wl = 0, bh = 0;
    float xi = 0.0f, sfl = 0.0f;
    int64_t off = 0;
    bool act = false;
    if (has) {
        // everything the match needs is in its list record: one round of loads
        j = mr.j;
        bh = mr.h;
        const float xj = mr.bx;
        xi = mr.x;
        const float yi = mr.y;
        l = lvl(mr.oct);
        const float s = pick_level(J.inv_sf, l);
        sfl = pick_level(J.sf, l);
        su = (int)roundf(xi * s);
        sv = (int)roundf(yi * s);
        su0 = (int)roundf(xj * s);
        Wl = pick_level(J.lv_w, l);
        const int Hl = pick_level(J.lv_h, l);
        off = pick_level(J.lv_off, l);
        act = su - w >= 0 && su + w < Wl && sv - w >= 0 && sv + w < Hl && su0 - L - w >= 0 &&
              su0 + L + w < Wl;
    }
    uint8_t *P = lds + wave * kRefineLds;          // left patch [side][side]
    uint8_t *S = P + side * side;                  // right strip [side][strip]
    if (act) {
        const uint8_t *IL = J.pyrL + off;
        const uint8_t *IR = J.pyrR + off;
        const int nP = side * side, n = nP + side * strip;
        for (int e = lane; e < n; e += 64) {
            if (e < nP) {
                const int r = e / side, c = e - r * side;
                P[e] = IL[(size_t)(sv - w + r) * Wl + su - w + c];
            } else {
                const int e2 = e - nP, r = e2 / strip, c = e2 - r * strip;
                P[e] = IR[(size_t)(sv - w + r) * Wl + su0 - L - w + c];
            }
        }
    }
    __syncthreads();
    const int parts = 64 / nS;
    const int k_idx = lane / parts, part = lane - k_idx * parts;
    int acc = 0;
    if (act && k_idx < nS) {
        const int cL = P[w * side + w];
        const int cR = S[w * strip + k_idx + w];
        for (int r = part; r < side; r += parts) {
            const uint8_t *pl = P + r * side;
            const uint8_t *pr = S + r * strip + k_idx;
            for (int dx = 0; dx < side; ++dx) acc += abs(((int)pl[dx] - cL) - ((int)pr[dx] - cR));
        }
    }
    int tot = acc;
    for (int p = 1; p < parts; ++p) tot += __shfl(acc, min(lane + p, 63));
    // every lane takes part in the shuffles; ties go to the smaller shift
    int best = 0x7FFFFFFF, kb = -L;
    for (int kk = 0; kk < nS; ++kk) {
        const int v = __shfl(tot, kk * parts);
        if (v < best) {
            best = v;
            kb = kk - L;
        }
    }
    const int a = __shfl(tot, max(kb + L - 1, 0) * parts);
    const int e = __shfl(tot, min(kb + L + 1, nS - 1) * parts);
    if (lane != 0 || !has) return;
    if (!act || kb == -L || kb == L) {
        J.flag[i] = 0;
        return;
    }
    const int c = best;
    const float num = (float)(a - e);
    const float den = (float)(2 * (a + e - 2 * c));
    const float delta = num / den;
    if (delta < -1.0f || delta > 1.0f) {
        J.flag[i] = 0;
        return;
    }
    float uR = sfl * (((float)su0 + (float)kb) + delta);
    float disp = xi - uR;
    if (!(disp >= 0.0f && disp < J.maxD)) {
        J.flag[i] = 0;
        return;
    }
    if (disp <= 0.0f) {
        disp = 0.01f;
        uR = (float)((double)xi - 0.01);
    }
    J.sad[i] = c;
    J.uR[i] = uR;
    J.depth[i] = J.bf / disp;
    J.flag[i] = 1;
    atomicMin(&J.claimR[j], ((uint32_t)bh << 23) | (uint32_t)i);
}

// Sum of two lanes' packed 16-bit partial sums, halving the dwords a lane holds:
// the upper N when `upper`; the others go to the partner of DPP control kCtrl.
template <int N, int kCtrl>
__device__ __forceinline__ void sums_halve(uint32_t *s, bool upper)
{
    _Pragma("unroll") for (int i = 0; i < N; ++i)
    {
        const uint32_t keep = upper ? s[i + N] : s[i], give = upper ? s[i] : s[i + N];
        s[i] = keep + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)give, kCtrl, 0xF, 0xF, false);
    }
}

template <int kCtrl>
__device__ __forceinline__ uint32_t min_dpp(uint32_t v)
{
    return min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xF, 0xF, false));
}

// The usual 11x11 window and +-5 shifts: four matches per wave, sixteen lanes
// each.  Lane r < 11 holds row r of the patch and of the strip in registers (two
// pixels per dword) and sums its row for all 11 shifts; the sums of the rows are
// added by halving exchanges that leave lane k with the SAD of shift k - 5.
// Two pixels per instruction, no LDS and no barrier, about 450 vector instructions
// a wave (768 with the rows staged in LDS as 16-bit pairs, read back per shift).
// One frame of 1200 keypoints 39.2 -> 36.9 us, the mixed 64-frame batch 154.2 ->
// 151.2; in 64 pinhole frames the kernel takes 32 us (36.7 before), where the
// window rows, a cache line each, fetch 106 MB.
__device__ __forceinline__ void ph_refine_quarter(const DevJob &J, int tile)
{
    constexpr int w = 5, L = 5, side = 2 * w + 1, nS = 2 * L + 1;
    static_assert(side == 11 && nS == 11, "a row of 16 lanes: 11 window rows, then 11 shifts");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ql = lane & 15, slot = wave * 4 + (lane >> 4);
    const int idx = tile * kRefineQPerWG + slot;   // position in the frame's match list
    const bool has = idx < J.counts[2];
    const MatchRec mr = J.mrec[min(idx, max(J.L.n - 1, 0))];   // loaded with the list length
    if (__ballot(has) == 0) return;   // (whole waves past the list's end)
    // the level tables, a level per lane, read by the match's level from there
    // (a select chain over 8 levels of 6 dwords takes 150 instructions)
    static_assert(kLevels == 8, "a level table per 8 lanes");
    const int tl = lane & 7;
    const float t_inv = J.inv_sf[tl], t_sf = J.sf[tl];
    const int t_w = J.lv_w[tl], t_h = J.lv_h[tl];
    const int64_t t_off = J.lv_off[tl];
    // everything the match needs is in its list record: one round of loads
    const int i = mr.i, j = mr.j, bh = mr.h;
    const float xi = mr.x;
    const int l = lvl(mr.oct);
    const float s = __shfl(t_inv, l), sfl = __shfl(t_sf, l);
    const int Wl = __shfl(t_w, l), Hl = __shfl(t_h, l);
    const int64_t off = ((int64_t)__shfl((int)(t_off >> 32), l) << 32) | (uint32_t)__shfl((int)t_off, l);
    const int su = (int)roundf(xi * s), sv = (int)roundf(mr.y * s), su0 = (int)roundf(mr.bx * s);
    const bool act = has && su - w >= 0 && su + w < Wl && sv - w >= 0 && sv + w < Hl && su0 - L - w >= 0 &&
                     su0 + L + w < Wl;
    // For shift k the centre-subtracted difference |(P - cL) - (S - cR)| equals
    // |(P + 255) - (S + off_k)| with off_k = cL - cR + 255 in [0, 510]; both terms
    // lie in [0, 765], so v_sad_u16 sums two pixels per instruction.
    uint32_t sums[8];   // of shifts 2d, 2d + 1: each at most 120 * 510 over the window, 16 bits
    _Pragma("unroll") for (int d = 0; d < 8; ++d) sums[d] = 0;
    if (act && ql < side) {
        const int64_t row = off + (int64_t)(sv - w + ql) * Wl;
        const FT_G uint8_t *p = J.pyrL + row + (su - w);
        const FT_G uint8_t *q = J.pyrR + row + (su0 - L - w);
        // The aligned dwords that hold the row (misaligned loads take two to four
        // times as long).  The strip's 21 bytes lie in six of them.  The patch's 11
        // lie in three or four; a load of four begins with the first of them, so it
        // may end up to 4 bytes behind the row's last dword, inside the next row of
        // the window; the last row's load ends with its last dword and begins up to
        // 5 bytes before the row, inside the row above.
        const uint32_t ap = (uint32_t)reinterpret_cast<uintptr_t>(p) & 3u;
        const uint32_t aq = (uint32_t)reinterpret_cast<uintptr_t>(q) & 3u;
        const bool back = ql == side - 1 && ap < 2;
        const v4u pd = *reinterpret_cast<const FT_G v4u_dw *>(p - ap - (back ? 4 : 0));
        const v4u qd = *reinterpret_cast<const FT_G v4u_dw *>(q - aq);
        typedef uint32_t v2u_dw __attribute__((ext_vector_type(2), aligned(4)));
        const v2u_dw qe = *reinterpret_cast<const FT_G v2u_dw *>(q - aq + 16);
        const uint32_t p0 = back ? pd[1] : pd[0], p1 = back ? pd[2] : pd[1], p2 = back ? pd[3] : pd[2];
        const uint32_t pb[3] = {__builtin_amdgcn_alignbyte(p1, p0, ap), __builtin_amdgcn_alignbyte(p2, p1, ap),
                                __builtin_amdgcn_alignbyte(pd[3], p2, ap)};
        const uint32_t sd[7] = {qd[0], qd[1], qd[2], qd[3], qe[0], qe[1], 0u};
        uint32_t sb[6];
        _Pragma("unroll") for (int k = 0; k < 6; ++k) sb[k] = __builtin_amdgcn_alignbyte(sd[k + 1], sd[k], aq);
        // pixel pairs: P of columns 2t, 2t + 1 plus 255 (the last of column 10 alone),
        // E of strip columns 2t, 2t + 1, O of 2t + 1, 2t + 2
        constexpr uint32_t kLo = 0x0C010C00u, kHi = 0x0C030C02u, kMid = 0x0C020C01u, kNext = 0x0C040C03u;
        constexpr uint32_t k255 = 0x00FF00FFu;
        const uint32_t P[6] = {__builtin_amdgcn_perm(0u, pb[0], kLo) + k255, __builtin_amdgcn_perm(0u, pb[0], kHi) + k255,
                               __builtin_amdgcn_perm(0u, pb[1], kLo) + k255, __builtin_amdgcn_perm(0u, pb[1], kHi) + k255,
                               __builtin_amdgcn_perm(0u, pb[2], kLo) + k255, ((pb[2] >> 16) & 255u) + 255u};
        uint32_t E[11], O[10];
        _Pragma("unroll") for (int t = 0; t < 5; ++t)
        {
            E[2 * t] = __builtin_amdgcn_perm(0u, sb[t], kLo);
            E[2 * t + 1] = __builtin_amdgcn_perm(0u, sb[t], kHi);
            O[2 * t] = __builtin_amdgcn_perm(0u, sb[t], kMid);
            O[2 * t + 1] = __builtin_amdgcn_perm(sb[t + 1], sb[t], kNext);
        }
        E[10] = sb[5] & 255u;
        // the centre row's pixels 5..15, one per shift, from lane 5 (row_newbcast:5)
        auto centre = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x155, 0xF, 0xF, false); };
        constexpr uint32_t kLoLo = 0x01000100u, kHiHi = 0x03020302u;
        const uint32_t cl = centre(P[2]);
        const uint32_t cL = __builtin_amdgcn_perm(cl, cl, kHiHi);   // cL + 255 in both halves
        uint32_t c[6];
        _Pragma("unroll") for (int t = 0; t < 6; ++t) c[t] = centre(E[t + 2]);
        _Pragma("unroll") for (int k = 0; k < nS; ++k)
        {
            const uint32_t cc = c[(k + 1) >> 1];
            const uint32_t o = cL - __builtin_amdgcn_perm(cc, cc, (k & 1) ? kLoLo : kHiHi);
            const uint32_t *S = (k & 1) ? O + (k >> 1) : E + (k >> 1);
            uint32_t acc = 0;
            _Pragma("unroll") for (int t = 0; t < 5; ++t) acc = __builtin_amdgcn_sad_u16(P[t], S[t] + o, acc);
            acc = __builtin_amdgcn_sad_u16(P[5], (uint32_t)(uint16_t)(S[5] + o), acc);   // column 10
            if (k & 1) sums[k >> 1] |= acc << 16;
            else sums[k >> 1] = acc;
        }
    }
    // rows added with the lane at ql ^ 8, ^ 7, ^ 3 and ^ 1; lane ql ends with the
    // dword of shifts ql & ~1, ql | 1
    sums_halve<4, 0x128>(sums, ql & 8);   // row_ror:8
    sums_halve<2, 0x141>(sums, ql & 4);   // row_half_mirror
    sums_halve<1, 0x1B>(sums, ql & 2);    // quad_perm 3,2,1,0
    const uint32_t both = sums[0] + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sums[0], 0xB1, 0xF, 0xF, false);   // quad_perm 1,0,3,2
    const int sad = (int)((ql & 1) ? both >> 16 : both & 0xFFFFu);
    // SAD << 4 | lane: ties go to the smaller shift
    uint32_t key = act && ql < nS ? ((uint32_t)sad << 4) | (uint32_t)ql : 0xFFFFFFFFu;
    key = min_dpp<0xB1>(min_dpp<0x1B>(min_dpp<0x141>(min_dpp<0x128>(key))));
    const int kb = (int)(key & 15u) - L;
    const int base = lane & ~15;
    const int a = __shfl(sad, base + max(kb + L - 1, 0));
    const int e = __shfl(sad, base + min(kb + L + 1, nS - 1));
    if (ql != 0 || !has) return;
    if (!act || kb == -L || kb == L) {
        J.flag[i] = 0;
        return;
    }
    const int c = (int)(key >> 4);
    const float num = (float)(a - e);
    const float den = (float)(2 * (a + e - 2 * c));
    const float delta = num / den;
    if (delta < -1.0f || delta > 1.0f) {
        J.flag[i] = 0;
        return;
    }
    float uR = sfl * (((float)su0 + (float)kb) + delta);
    float disp = xi - uR;
    if (!(disp >= 0.0f && disp < J.maxD)) {
        J.flag[i] = 0;
        return;
    }
    if (disp <= 0.0f) {
        disp = 0.01f;
        uR = (float)((double)xi - 0.01);
    }
    J.sad[i] = c;
    J.uR[i] = uR;
    J.depth[i] = J.bf / disp;
    J.flag[i] = 1;
    atomicMin(&J.claimR[j], ((uint32_t)bh << 23) | (uint32_t)i);
}

__device__ __forceinline__ void ph_refine(const DevJob &J, int tile, uint8_t *lds)
{
    if (refine_quarter(J)) ph_refine_quarter(J, tile);
    else ph_refine_wave(J, tile, lds);
}

// ------------------------------- stereo_b (fisheye): ratio + triangulation
__device__ __forceinline__ double kb_distort(const float *kb, double th)
{
    const double k1 = kb[4], k2 = kb[5], k3 = kb[6], k4 = kb[7];
    const double t2 = th * th, t4 = t2 * t2, t6 = t4 * t2, t8 = t4 * t4;
    return th * ((((1.0 + k1 * t2) + k2 * t4) + k3 * t6) + k4 * t8);
}

__device__ __forceinline__ void kb_project(const float *kb, const double X[3], double uv[2])
{
    const double fx = kb[0], fy = kb[1], cx = kb[2], cy = kb[3];
    const double rho = sqrt(X[0] * X[0] + X[1] * X[1]);
    if (rho == 0.0) {
        uv[0] = cx;
        uv[1] = cy;
        return;
    }
    const double th = atan2(rho, X[2]);
    const double thd = kb_distort(kb, th);
    uv[0] = fx * ((thd * X[0]) / rho) + cx;
    uv[1] = fy * ((thd * X[1]) / rho) + cy;
}

__device__ __forceinline__ bool kb_unproject(const float *kb, float u, float v, int iters, double tol,
                             double max_theta, double ray[3])
{
    const double fx = kb[0], fy = kb[1], cx = kb[2], cy = kb[3];
    const double k1 = kb[4], k2 = kb[5], k3 = kb[6], k4 = kb[7];
    const double xp = ((double)u - cx) / fx;
    const double yp = ((double)v - cy) / fy;
    double thd = sqrt(xp * xp + yp * yp);
    const double half_pi = 1.5707963267948966;
    if (thd > half_pi) thd = half_pi;
    if (!(thd > 1e-8)) {
        ray[0] = xp;
        ray[1] = yp;
        ray[2] = 1.0;
        return true;
    }
    double th = thd;
    for (int it = 0; it < iters; ++it) {
        const double t2 = th * th, t4 = t2 * t2, t6 = t4 * t2, t8 = t4 * t4;
        const double f = th * ((((1.0 + k1 * t2) + k2 * t4) + k3 * t6) + k4 * t8) - thd;
        const double fp = (((1.0 + 3.0 * k1 * t2) + 5.0 * k2 * t4) + 7.0 * k3 * t6) + 9.0 * k4 * t8;
        const double step = f / fp;
        th = th - step;
        if (fabs(step) < tol) break;
    }
    if (!(th < max_theta)) return false;
    const double scale = tan(th) / thd;
    ray[0] = xp * scale;
    ray[1] = yp * scale;
    ray[2] = 1.0;
    return true;
}

__device__ __forceinline__ double det3(const double m[3][3])
{
    return m[0][0] * (m[1][1] * m[2][2] - m[1][2] * m[2][1]) -
           m[0][1] * (m[1][0] * m[2][2] - m[1][2] * m[2][0]) +
           m[0][2] * (m[1][0] * m[2][1] - m[1][1] * m[2][0]);
}

// Linear least-squares triangulation with the homogeneous coordinate fixed to
// one; 3x3 normal equations solved by Cramer's rule (float64).
__device__ __forceinline__ bool triangulate(const double r1[3], const double r2[3], const float *R_lr,
                            const float *t_lr, double X[3])
{
    double Rrl[3][3], trl[3];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) Rrl[r][c] = (double)R_lr[3 * c + r];
    for (int r = 0; r < 3; ++r)
        trl[r] = -(((Rrl[r][0] * (double)t_lr[0]) + Rrl[r][1] * (double)t_lr[1]) +
                   Rrl[r][2] * (double)t_lr[2]);
    const double p1x = r1[0] / r1[2], p1y = r1[1] / r1[2];
    const double p2x = r2[0] / r2[2], p2y = r2[1] / r2[2];
    double A[4][3], bb[4];
    A[0][0] = -1.0; A[0][1] = 0.0; A[0][2] = p1x; bb[0] = 0.0;
    A[1][0] = 0.0; A[1][1] = -1.0; A[1][2] = p1y; bb[1] = 0.0;
    for (int c = 0; c < 3; ++c) {
        A[2][c] = p2x * Rrl[2][c] - Rrl[0][c];
        A[3][c] = p2y * Rrl[2][c] - Rrl[1][c];
    }
    bb[2] = -(p2x * trl[2] - trl[0]);
    bb[3] = -(p2y * trl[2] - trl[1]);
    double M[3][3], v[3];
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) {
            double acc = 0.0;
            for (int k = 0; k < 4; ++k) acc = acc + A[k][r] * A[k][c];
            M[r][c] = acc;
        }
        double acc = 0.0;
        for (int k = 0; k < 4; ++k) acc = acc + A[k][r] * bb[k];
        v[r] = acc;
    }
    const double D = det3(M);
    if (D == 0.0 || !isfinite(D)) return false;
    for (int c = 0; c < 3; ++c) {
        double Mc[3][3];
        for (int r = 0; r < 3; ++r)
            for (int q = 0; q < 3; ++q) Mc[r][q] = q == c ? v[r] : M[r][q];
        X[c] = det3(Mc) / D;
    }
    return true;
}

__device__ __forceinline__ void ph_tri(const DevJob &J, int tile)
{
    const int nQ = J.counts[0], nT = J.counts[1];
    const int q = tile * kWG + threadIdx.x;
    if (q >= nQ || nT < 2) return;
    const int i = J.qlist[q];
    const int j1 = J.best_j[i], h1 = J.best_h[i], h2 = J.h2[i];
    if (!(J.ratio_den * h1 < J.ratio_num * h2)) return;
    double r1[3], r2[3];
    if (!kb_unproject(J.kbL, J.L.x[i], J.L.y[i], J.newton_iters, J.newton_tol, J.max_theta, r1)) return;
    if (!kb_unproject(J.kbR, J.R.x[j1], J.R.y[j1], J.newton_iters, J.newton_tol, J.max_theta, r2)) return;
    double r21[3];
    for (int r = 0; r < 3; ++r)
        r21[r] = (((double)J.R_lr[3 * r] * r2[0]) + (double)J.R_lr[3 * r + 1] * r2[1]) +
                 (double)J.R_lr[3 * r + 2] * r2[2];
    const double n1 = sqrt((r1[0] * r1[0] + r1[1] * r1[1]) + r1[2] * r1[2]);
    const double n2 = sqrt((r21[0] * r21[0] + r21[1] * r21[1]) + r21[2] * r21[2]);
    const double cosp = ((r1[0] * r21[0] + r1[1] * r21[1]) + r1[2] * r21[2]) / (n1 * n2);
    if (!(cosp <= J.cos_max)) return;
    double X[3];
    if (!triangulate(r1, r2, J.R_lr, J.t_lr, X)) return;
    if (!(X[2] > 0.0)) return;
    double X2[3];
    for (int r = 0; r < 3; ++r)
        X2[r] = (((double)J.R_lr[r] * (X[0] - (double)J.t_lr[0])) +
                 (double)J.R_lr[3 + r] * (X[1] - (double)J.t_lr[1])) +
                (double)J.R_lr[6 + r] * (X[2] - (double)J.t_lr[2]);
    if (!(X2[2] > 0.0)) return;
    double uv[2];
    kb_project(J.kbL, X, uv);
    double ex = uv[0] - (double)J.L.x[i], ey = uv[1] - (double)J.L.y[i];
    if (!(ex * ex + ey * ey <= J.chi2 * (double)J.sigma2[lvl(J.L.oct[i])])) return;
    kb_project(J.kbR, X2, uv);
    ex = uv[0] - (double)J.R.x[j1];
    ey = uv[1] - (double)J.R.y[j1];
    if (!(ex * ex + ey * ey <= J.chi2 * (double)J.sigma2[lvl(J.R.oct[j1])])) return;
    J.depth[i] = (float)X[2];
    J.xyz[3 * i] = (float)X[0];
    J.xyz[3 * i + 1] = (float)X[1];
    J.xyz[3 * i + 2] = (float)X[2];
    J.flag[i] = 1;
    atomicMin(&J.claimR[j1], ((uint32_t)h1 << 23) | (uint32_t)i);
}

// ---------------------- stereo_c (pinhole): conflicts + median + outputs
// The median is the value at rank n/2 of the survivors' 16-bit SADs, found by
// a two-pass 8-bit radix select.  Every wave reads the 256 counts (four bins per
// lane) and selects by itself, so a pass costs one barrier: what bounds the
// phase is its chain of barriers and loads in one workgroup.

// Bin of hist[256] that holds rank `target` (the total's half when negative),
// the rank inside it, and the total; wave-uniform.
__device__ __forceinline__ int select_bin(const int *hist, int target, int &rank, int &total)
{
    const int lane = threadIdx.x & 63;
    const v4i h = *reinterpret_cast<const v4i *>(hist + 4 * lane);
    const int s = (h[0] + h[1]) + (h[2] + h[3]);
    const int inc = wave_inclusive_scan(s);
    total = wave_last(inc);
    const int t = target < 0 ? total / 2 : target;
    int run = inc - s, bin = 4 * lane, left = 0;
    const bool here = run <= t && t < inc;
    _Pragma("unroll") for (int k = 0; k < 4; ++k)
    {
        const bool in = run <= t && t < run + h[k];
        bin = in ? 4 * lane + k : bin;
        left = in ? t - run : left;
        run += h[k];
    }
    const int at = max(__ffsll((long long)__ballot(here)) - 1, 0);   // (no lane when the total is 0)
    rank = __builtin_amdgcn_readlane(left, at);
    return __builtin_amdgcn_readlane(bin, at);
}

__device__ __forceinline__ bool bit(const uint32_t *b, int i) { return (b[i >> 5] >> (i & 31)) & 1u; }

constexpr int kMedianLds = (256 + 256 + 16) * 4 + (kMaxKp + 32) / 32 * 4;   // counts, kept per wave, survivor bits

template <int NT>
__device__ __forceinline__ void ph_median(const DevJob &J, unsigned char *smem)
{
    int *hist = reinterpret_cast<int *>(smem), *hist2 = hist + 256, *wkept = hist + 512;
    uint32_t *surv = reinterpret_cast<uint32_t *>(hist + 528);
    const int tid = threadIdx.x, nL = J.L.n;
    // Up to kSortUnroll * NT keypoints, every field a thread needs stays in
    // its registers from the first pass to the outputs; larger frames re-read.
    const bool held = nL <= kSortUnroll * NT;
    for (int b = tid; b < 512; b += NT) hist[b] = 0;
    if (!held)
        for (int w = tid; w < (nL + 31) / 32; w += NT) surv[w] = 0;
    __syncthreads();
    int bj[kSortUnroll], bh[kSortUnroll], sd[kSortUnroll];
    float ur[kSortUnroll], dp[kSortUnroll];
    bool sv[kSortUnroll] = {};
    for (int i0 = tid; i0 < nL; i0 += kSortUnroll * NT) {
        int fl[kSortUnroll];
        uint32_t cl[kSortUnroll];
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
        {
            const int i = min(i0 + e * NT, nL - 1);
            fl[e] = J.flag[i];
            bj[e] = J.best_j[i];
            bh[e] = J.best_h[i];
            sd[e] = J.sad[i];
            ur[e] = J.uR[i];
            dp[e] = J.depth[i];
        }
        // a flagged keypoint has a valid right index; others read index 0
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e) cl[e] = J.claimR[fl[e] ? bj[e] : 0];
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
        {
            const int i = i0 + e * NT;
            sv[e] = i < nL && fl[e] && cl[e] == (((uint32_t)bh[e] << 23) | (uint32_t)i);
            if (sv[e]) {
                if (!held) atomicOr(&surv[i >> 5], 1u << (i & 31));
                atomicAdd(&hist[(sd[e] >> 8) & 0xFF], 1);
            }
        }
    }
    __syncthreads();
    int rank, n, m = 0;
    const int hb = select_bin(hist, -1, rank, n);
    if (n > 0) {   // (uniform)
        if (held) {
            _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
                if (tid + e * NT < nL && sv[e] && ((sd[e] >> 8) & 0xFF) == hb) atomicAdd(&hist2[sd[e] & 0xFF], 1);
        } else {
            for (int i = tid; i < nL; i += NT)
                if (bit(surv, i) && ((J.sad[i] >> 8) & 0xFF) == hb) atomicAdd(&hist2[J.sad[i] & 0xFF], 1);
        }
        __syncthreads();
        int rank2, n2;
        m = (hb << 8) | select_bin(hist2, rank, rank2, n2);
    }
    int kept = 0;
    for (int i0 = tid; i0 < nL; i0 += kSortUnroll * NT) {
        if (!held) {
            _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
            {
                const int i = min(i0 + e * NT, nL - 1);
                bj[e] = J.best_j[i];
                bh[e] = J.best_h[i];
                sd[e] = J.sad[i];
                ur[e] = J.uR[i];
                dp[e] = J.depth[i];
                sv[e] = bit(surv, i);
            }
        }
        _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
        {
            const int i = i0 + e * NT;
            if (i >= nL) continue;
            const bool keep = sv[e] && (long long)J.med_den * sd[e] < (long long)J.med_num * m;
            J.o_right_idx[i] = keep ? bj[e] : -1;
            J.o_dist[i] = keep ? bh[e] : -1;
            J.o_uR[i] = keep ? ur[e] : -1.0f;
            J.o_depth[i] = keep ? dp[e] : -1.0f;
            J.o_sad[i] = keep ? sd[e] : -1;
            kept += keep ? 1 : 0;
        }
    }
    kept = wave_last(wave_inclusive_scan(kept));
    if ((tid & 63) == 0) wkept[tid >> 6] = kept;
    __syncthreads();
    if (tid < 64) {
        const int all = wave_last(wave_inclusive_scan(tid < NT / 64 ? wkept[tid] : 0));
        if (tid == 0) *J.o_nmatch = all;
    }
}

// ---------------------- stereo_c (fisheye): conflicts + outputs
template <int NT>
__device__ __forceinline__ void ph_fish_final(const DevJob &J, int tile)
{
    const int i = tile * NT + threadIdx.x;
    bool keep = false;
    if (i < J.L.n) {
        keep = J.flag[i] &&
               J.claimR[J.best_j[i]] == (((uint32_t)J.best_h[i] << 23) | (uint32_t)i);
        if (keep) {
            J.o_right_idx[i] = J.best_j[i];
            J.o_dist[i] = J.best_h[i];
            J.o_depth[i] = J.depth[i];
            J.o_xyz[3 * i] = J.xyz[3 * i];
            J.o_xyz[3 * i + 1] = J.xyz[3 * i + 1];
            J.o_xyz[3 * i + 2] = J.xyz[3 * i + 2];
        } else {
            J.o_right_idx[i] = -1;
            J.o_dist[i] = -1;
            J.o_depth[i] = -1.0f;
            J.o_xyz[3 * i] = 0.0f;
            J.o_xyz[3 * i + 1] = 0.0f;
            J.o_xyz[3 * i + 2] = 0.0f;
        }
    }
    const unsigned long long m = __ballot(keep);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(J.o_nmatch, (int)__popcll(m));
}

// ------------------------------------------------ search by projection
// G lanes per map point.  Every lane of the group evaluates the projection and
// the visibility tests (identical results), then the group streams the
// cell-sorted records of the window's cells (one cell of margin on each side
// covers the rounding of the cell arithmetic) and merges its top-2 lists.
// Keys order candidates by (distance, keypoint index): distance << 40 |
// index << 8 | level.
// What one map point looks for in one view: its projection, the search
// window (radius, levels, cells) and its descriptor.
struct Query {
    bool vis;
    bool gate;          // stereo right-coordinate gate applies
    float u, v, Rm, uR;
    int cx0, cx1, cy0, cy1, plo, phi;
    int cb;             // first cell offset of the level bin of the predicted level
    Desc dm;
};

__device__ __forceinline__ Query make_query(const DevJob &J, const DevView &V, int m)
{
    Query q;
    // every field of the map point record is issued up front (one round trip)
    const float X = J.pos[3 * m], Y = J.pos[3 * m + 1], Z = J.pos[3 * m + 2];
    const float nx = J.normal[3 * m], ny = J.normal[3 * m + 1], nz = J.normal[3 * m + 2];
    const float dmin = J.dmin[m], dmax = J.dmax[m];
    q.dm = load_desc(J.mdesc, m);
    const float xc = ((V.R[0] * X + V.R[1] * Y) + V.R[2] * Z) + V.t[0];
    const float yc = ((V.R[3] * X + V.R[4] * Y) + V.R[5] * Z) + V.t[1];
    const float zc = ((V.R[6] * X + V.R[7] * Y) + V.R[8] * Z) + V.t[2];
    float u = 0.0f, v = 0.0f;
    bool vis = false;
    if (zc > 0.0f) {
        if (V.model == FT_CAMERA_PINHOLE) {
            u = ((V.fx * xc) / zc) + V.cx;
            v = ((V.fy * yc) / zc) + V.cy;
        } else {
            const float kb[8] = {V.fx, V.fy, V.cx, V.cy, V.k[0], V.k[1], V.k[2], V.k[3]};
            const double Pc[3] = {(double)xc, (double)yc, (double)zc};
            double uv[2];
            kb_project(kb, Pc, uv);
            u = (float)uv[0];
            v = (float)uv[1];
        }
        vis = u >= V.min_x && u <= V.max_x && v >= V.min_y && v <= V.max_y;
    }
    const float pox = X - V.O[0], poy = Y - V.O[1], poz = Z - V.O[2];
    const float dist = sqrtf((pox * pox + poy * poy) + poz * poz);
    vis = vis && dist >= J.dist_lo * dmin && dist <= J.dist_hi * dmax;
    const float vcos = ((pox * nx + poy * ny) + poz * nz) / dist;
    q.vis = vis && vcos >= J.cos_lim;
    q.u = u;
    q.v = v;
    if (!q.vis) return q;
    const float ratio = dmax / dist;
    int pred = kLevels - 1;
    for (int l = 0; l < kLevels; ++l)
        if (J.sf[l] >= ratio) {
            pred = l;
            break;
        }
    const float rbase = (vcos > J.cos_narrow ? J.r_narrow : J.r_wide) * J.th;
    q.Rm = rbase * J.sf[pred];
    q.gate = V.u_right != nullptr;
    q.uR = q.gate ? u - V.bf * (1.0f / zc) : 0.0f;
    // A candidate has |x - u| < Rm up to one rounding of the subtraction, so x
    // lies within Rm + 0.01 px of u; cell_coord is monotone, so the cells of
    // u -+ (Rm + 0.01) bracket the cells of every candidate.
    const float Rc = q.Rm + 0.01f;
    q.cx0 = cell_coord(u - Rc, V.min_x, V.inv_cw, V.cols);
    q.cx1 = cell_coord(u + Rc, V.min_x, V.inv_cw, V.cols);
    q.cy0 = cell_coord(v - Rc, V.min_y, V.inv_ch, V.rows);
    q.cy1 = cell_coord(v + Rc, V.min_y, V.inv_ch, V.rows);
    q.plo = pred - J.lv_lo;
    q.phi = pred + J.lv_hi;
    q.cb = (V.n_pb > 1 ? pred : 0) * (V.cols * V.rows);
    return q;
}

// A keypoint record (level, position) is a candidate of the query, before the
// stereo gate.
__device__ __forceinline__ bool in_window(const Query &q, float x, float y, uint32_t meta)
{
    const int ok = (int)(meta & 0xFFu);
    return ok >= q.plo && ok <= q.phi && fabsf(x - q.u) < q.Rm && fabsf(y - q.v) < q.Rm && !(meta & 0x100u);
}

__device__ __forceinline__ bool gate_rejects(const Query &q, float ur)
{
    return q.gate && ur > 0.0f && !(fabsf(q.uR - ur) <= q.Rm);
}

__device__ __forceinline__ uint64_t cand_key(int h, uint32_t meta)
{
    return ((uint64_t)h << 40) | ((uint64_t)(meta >> 16) << 8) | (uint64_t)(meta & 0xFFu);
}

// Scan of the window over the sorted records in global memory; lane `sub` of
// G takes every G-th record.  One record range per window row; the next row's
// bounds are loaded before the current row is scanned, and kSearchUnroll
// records are loaded together (indices clamped into the range, surplus
// entries masked), then the descriptors of the candidates among them.
template <int G>
__device__ __forceinline__ Top2<uint64_t> scan_global(const DevView &V, const Query &q, int sub)
{
    Top2<uint64_t> top = {~0ull, ~0ull};
    const FT_G int32_t *off = V.cell_off + q.cb;
    int c0 = off[q.cy0 * V.cols + q.cx0];
    int c1 = off[q.cy0 * V.cols + q.cx1 + 1];
    for (int cy = q.cy0; cy <= q.cy1; ++cy) {
        int n0 = 0, n1 = 0;
        if (cy < q.cy1) {
            n0 = off[(cy + 1) * V.cols + q.cx0];
            n1 = off[(cy + 1) * V.cols + q.cx1 + 1];
        }
        for (int p0 = c0 + sub; p0 < c1; p0 += kSearchUnroll * G) {
            CellRec rec[kSearchUnroll];
            bool cand[kSearchUnroll];
            Desc d[kSearchUnroll];
            float ur[kSearchUnroll];
            _Pragma("unroll") for (int e = 0; e < kSearchUnroll; ++e) rec[e] = V.crec[min(p0 + e * G, c1 - 1)];
            _Pragma("unroll") for (int e = 0; e < kSearchUnroll; ++e)
            {
                cand[e] = p0 + e * G < c1 && in_window(q, rec[e].x, rec[e].y, rec[e].meta);
                ur[e] = 0.0f;
                if (cand[e]) {
                    d[e] = load_desc(V.kdesc, (int)(rec[e].meta >> 16));
                    if (q.gate) ur[e] = V.u_right[rec[e].meta >> 16];
                }
            }
            _Pragma("unroll") for (int e = 0; e < kSearchUnroll; ++e)
            {
                if (cand[e] && !gate_rejects(q, ur[e]))
                    top = top2_insert(top, cand_key(hamming(q.dm, d[e]), rec[e].meta));
            }
        }
        c0 = n0;
        c1 = n1;
    }
    return top;
}

// Merge of the G lanes' lists, acceptance, outputs and the claim on the
// matched keypoint.  Every lane of the wave calls it (shuffles).
template <int G>
__device__ __forceinline__ void finish_query(const DevJob &J, const DevView &V, int m, int sub,
                                             Top2<uint64_t> top)
{
    for (int o = 1; o < G; o <<= 1) top = top2_merge(top, shfl_xor64(top.a, o), shfl_xor64(top.b, o));
    if (sub != 0 || m >= J.nM) return;
    const uint64_t k1 = top.a, k2 = top.b;
    int kk1 = -1, b1 = -1;
    if (k1 != ~0ull) {
        const int h1 = (int)(k1 >> 40), l1 = (int)(k1 & 0xFFu);
        const int h2 = k2 != ~0ull ? (int)(k2 >> 40) : 256;
        const int l2 = k2 != ~0ull ? (int)(k2 & 0xFFu) : -1;
        const bool fails = J.s_ratio_den * h1 > J.s_ratio_num * h2;
        if (h1 <= J.th_high && !(J.same_level_only ? (l1 == l2 && fails) : fails)) {
            kk1 = (int)((k1 >> 8) & 0xFFFFu);
            b1 = h1;
        }
    }
    V.mp_k[m] = kk1;
    V.mp_h[m] = b1;
    if (kk1 >= 0) atomicMin(&V.claim[kk1], ((uint32_t)b1 << 23) | (uint32_t)m);
}

// Candidate keys of the record-dealt search are 32 bits: distance (9 bits),
// keypoint (16), level (4; octaves are 0..7 by contract), in the same order as
// cand_key; each map point's best two keys are kept in LDS by atomic minima: a
// key goes to the best slot, and whichever of it and the displaced best is
// larger goes to the second slot, which leaves the two smallest distinct keys.
__device__ __forceinline__ uint64_t key32_to_64(uint32_t k)
{
    if (k == 0xFFFFFFFFu) return ~0ull;
    return ((uint64_t)(k >> 20) << 40) | ((uint64_t)((k >> 4) & 0xFFFFu) << 8) | (uint64_t)(k & 15u);
}

// Orders one wave's LDS accesses (its lanes read what other lanes wrote); the
// record-dealt search syncs only within a wave, whose chunk and round counts
// are wave-uniform but may differ between the waves of a workgroup.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// --------------------------------- last-frame search by projection
// Initial Pose Estimation projects the last frame's matched map points into
// the current frame and searches its keypoints (Section II-C); the same
// search by projection as the local-map search (Section IV-E), with the
// window taken from the last-frame keypoint (radius th * sf[octave], levels
// by the direction of motion) instead of the predicted level, no ratio test,
// and a rotation-consistency check over the frame's matches.
//
// Camera projection of a world point into view V (pinhole binary32, KB
// binary64 rounded to binary32); false when the point is behind the camera
// or outside the image bounds.
__device__ __forceinline__ bool project_point(const DevView &V, float X, float Y, float Z, float &u, float &v,
                                              float &zc)
{
    const float xc = ((V.R[0] * X + V.R[1] * Y) + V.R[2] * Z) + V.t[0];
    const float yc = ((V.R[3] * X + V.R[4] * Y) + V.R[5] * Z) + V.t[1];
    zc = ((V.R[6] * X + V.R[7] * Y) + V.R[8] * Z) + V.t[2];
    u = 0.0f;
    v = 0.0f;
    if (!(zc > 0.0f)) return false;
    if (V.model == FT_CAMERA_PINHOLE) {
        u = ((V.fx * xc) / zc) + V.cx;
        v = ((V.fy * yc) / zc) + V.cy;
    } else {
        const float kb[8] = {V.fx, V.fy, V.cx, V.cy, V.k[0], V.k[1], V.k[2], V.k[3]};
        const double Pc[3] = {(double)xc, (double)yc, (double)zc};
        double uv[2];
        kb_project(kb, Pc, uv);
        u = (float)uv[0];
        v = (float)uv[1];
    }
    return u >= V.min_x && u <= V.max_x && v >= V.min_y && v <= V.max_y;
}

// What one last-frame point looks for: its projection and window.  The index's
// level bins are those of the points' octaves (when it has them).
__device__ __forceinline__ Query make_last_query(const DevJob &J, const DevView &V, int i)
{
    Query q;
    const float X = J.pos[3 * i], Y = J.pos[3 * i + 1], Z = J.pos[3 * i + 2];
    const int ol = lvl(J.l_oct[i]);
    q.dm = load_desc(J.mdesc, i);
    float zc;
    q.vis = project_point(V, X, Y, Z, q.u, q.v, zc);
    if (!q.vis) return q;
    q.Rm = J.th * J.sf[ol];
    q.plo = J.direction > 0 ? ol : J.direction < 0 ? 0 : ol - 1;
    q.phi = J.direction > 0 ? kLevels - 1 : J.direction < 0 ? ol : ol + 1;
    q.gate = V.u_right != nullptr;
    q.uR = q.gate ? q.u - V.bf * (1.0f / zc) : 0.0f;
    // cells of u -+ (r + 0.01) bracket every candidate (as in the local search)
    const float Rc = q.Rm + 0.01f;
    q.cx0 = cell_coord(q.u - Rc, V.min_x, V.inv_cw, V.cols);
    q.cx1 = cell_coord(q.u + Rc, V.min_x, V.inv_cw, V.cols);
    q.cy0 = cell_coord(q.v - Rc, V.min_y, V.inv_ch, V.rows);
    q.cy1 = cell_coord(q.v + Rc, V.min_y, V.inv_ch, V.rows);
    q.cb = (V.n_pb > 1 ? ol : 0) * (V.cols * V.rows);
    return q;
}

// Acceptance and claim of a last-frame point's best candidate key (distance,
// keypoint, level: 32 bits).
__device__ __forceinline__ void finish_last(const DevJob &J, const DevView &V, int i, uint32_t key)
{
    if (i >= J.nM) return;
    int k = -1, h = -1;
    if (key != 0xFFFFFFFFu && (int)(key >> 20) <= J.th_high) {
        h = (int)(key >> 20);
        k = (int)((key >> 4) & 0xFFFFu);
    }
    V.mp_k[i] = k;
    V.mp_h[i] = h;
    if (k >= 0) atomicMin(&V.claim[k], ((uint32_t)h << 23) | (uint32_t)i);
}

// Record-dealt search (one lane per map point).  Every lane projects its map
// point and loads the record ranges of up to kDealRows window rows at once;
// the wave then lays the records of all 64 windows end to end and deals them
// out in rounds of 64 * kDealRecs positions, lane d taking positions d, d + 64,
// d + 128, ..., so every lane issues all its record loads together whatever
// the window sizes and each load instruction reads 64 consecutive positions.
// Records that pass the window test become candidates in one wave-wide list,
// which is again dealt evenly for the descriptor reads; each map point's best
// two keys are kept in LDS by 32-bit atomic minima.
constexpr int kDealRows = 4;    // window rows per lane and chunk
constexpr int kDealRecs = 4;    // records per lane and round
constexpr int kDealFlush = 1;   // candidates per lane and descriptor batch
constexpr int kDealQp = 0;                                // float4 u, v, Rm, level window [64]
constexpr int kDealUr = kDealQp + 64 * 16;                // float uR [64]
constexpr int kDealQd = kDealUr + 64 * 4;                 // Desc [64]
constexpr int kDealTb = kDealQd + 64 * 32;                // best [64], second [64]
constexpr int kDealSeg = kDealTb + 128 * 4;               // record offset of each segment [64][kDealRows]
constexpr int kDealCands = kDealSeg + 64 * kDealRows * 4;  // candidate list [64 * kDealRecs], or the round's marks
constexpr int kDealLdsPerWave = kDealCands + 64 * kDealRecs * 4;

// The wave takes map points (kLast: last-frame points) m0 .. m0 + 63 of the view;
// `base` is its LDS.
template <bool kLast>
__device__ __forceinline__ void ph_search_deal(const DevJob &J, const DevView &V, int m0, unsigned char *base)
{
    const int lane = threadIdx.x & 63;
    const int m = m0 + lane;
    float4 *qp = reinterpret_cast<float4 *>(base + kDealQp);
    float *quR = reinterpret_cast<float *>(base + kDealUr);
    Desc *qd = reinterpret_cast<Desc *>(base + kDealQd);
    uint32_t *tb = reinterpret_cast<uint32_t *>(base + kDealTb);
    uint32_t *seg = reinterpret_cast<uint32_t *>(base + kDealSeg);
    uint32_t *cl = reinterpret_cast<uint32_t *>(base + kDealCands);
    uint32_t *mark = cl;

    Query q;
    q.vis = false;
    if (m < J.nM) q = kLast ? make_last_query(J, V, m) : make_query(J, V, m);
    const int cx0 = q.vis ? q.cx0 : 0, cx1 = q.vis ? q.cx1 : 0;
    const int cy0 = q.vis ? q.cy0 : 0, cy1 = q.vis ? q.cy1 : -1;
    const FT_G int32_t *off = V.cell_off + (q.vis ? q.cb : 0);
    // the octave window's two ends as signed 16-bit halves (-kMaxWindow .. kLevels - 1 + kMaxWindow)
    static_assert(kMaxWindow + kLevels <= 0x7FFF, "16-bit halves");
    const int lv = q.vis ? (q.plo & 0xFFFF) | (int)((uint32_t)q.phi << 16) : (int)0xFFFF0000u;   // (else 0 .. -1: none)
    qp[lane] = make_float4(q.u, q.v, q.vis ? q.Rm : 0.0f, __int_as_float(lv));
    quR[lane] = q.vis ? q.uR : 0.0f;
    qd[lane] = q.dm;
    tb[lane] = 0xFFFFFFFFu;
    tb[64 + lane] = 0xFFFFFFFFu;
    const bool gate = V.u_right != nullptr;
    const int chunks = wave_last(wave_inclusive_max((cy1 - cy0 + kDealRows) / kDealRows));
    for (int ch = 0; ch < chunks; ++ch) {
        // record ranges of this lane's rows of the chunk: one round of loads
        const int r0 = cy0 + ch * kDealRows;
        int sa[kDealRows], sn[kDealRows];
        int mine = 0;
        _Pragma("unroll") for (int e = 0; e < kDealRows; ++e)
        {
            const bool in = r0 + e <= cy1;
            const int row = in ? r0 + e : 0;
            sa[e] = off[row * V.cols + cx0];
            const int b = off[row * V.cols + cx1 + 1];
            sn[e] = in ? b - sa[e] : 0;
            mine += sn[e];
        }
        const int incl = wave_inclusive_scan(mine);
        const int total = wave_last(incl);
        // the records of all segments (lane, row) end to end: a segment's first
        // position in the chunk, and the offset from a position to its record
        int st[kDealRows];
        st[0] = incl - mine;
        _Pragma("unroll") for (int e = 1; e < kDealRows; ++e) st[e] = st[e - 1] + sn[e - 1];
        wave_lds_sync();   // the previous chunk's readers are done with seg
        _Pragma("unroll") for (int e = 0; e < kDealRows; ++e) seg[lane * kDealRows + e] = (uint32_t)(sa[e] - st[e]);
        for (int g_lo = 0; g_lo < total; g_lo += 64 * kDealRecs) {
            const int cnt = min(total - g_lo, 64 * kDealRecs);
            // Position g_lo + 64k + d of the chunk goes to lane d.  Each
            // non-empty segment writes its id + 1 at its first position of the
            // round (position 0 for the one begun in an earlier round); no two
            // segments share a position and ids grow with positions, so the
            // prefix maximum over positions names every position's segment.
            // The marks use the candidate list's memory.
            *reinterpret_cast<uint4 *>(mark + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
            wave_lds_sync();
            _Pragma("unroll") for (int e = 0; e < kDealRows; ++e)
            {
                const int A = st[e] - g_lo;
                if (sn[e] > 0 && A < cnt && A + sn[e] > 0) mark[max(A, 0)] = (uint32_t)(lane * kDealRows + e + 1);
            }
            wave_lds_sync();
            int own[kDealRecs];
            int carry = 0;
            _Pragma("unroll") for (int k = 0; k < kDealRecs; ++k)
            {
                own[k] = max(wave_inclusive_max((int)mark[k * 64 + lane]), carry) - 1;
                carry = wave_last(own[k]) + 1;
            }
            // the records: position + its segment's offset, 64 consecutive
            // positions per load instruction
            CellRec rec[kDealRecs];
            _Pragma("unroll") for (int k = 0; k < kDealRecs; ++k)
            {
                const int p = k * 64 + lane;
                if (p < cnt) rec[k] = V.crec[g_lo + p + (int)seg[max(own[k], 0)]];
            }
            // window test; candidates as keypoint | level << 16 | map lane << 20
            uint32_t cand[kDealRecs];
            int nc = 0;
            _Pragma("unroll") for (int k = 0; k < kDealRecs; ++k)
            {
                cand[k] = 0xFFFFFFFFu;
                if (k * 64 + lane < cnt) {
                    const int ml = max(own[k], 0) / kDealRows;
                    const float4 qq = qp[ml];
                    const int l = __float_as_int(qq.w);
                    Query iq;
                    iq.u = qq.x;
                    iq.v = qq.y;
                    iq.Rm = qq.z;
                    iq.plo = (int16_t)l;
                    iq.phi = l >> 16;
                    if (in_window(iq, rec[k].x, rec[k].y, rec[k].meta)) {
                        cand[k] = (rec[k].meta >> 16) | ((rec[k].meta & 15u) << 16) | ((uint32_t)ml << 20);
                        ++nc;
                    }
                }
            }
            const int cincl = wave_inclusive_scan(nc);
            const int ctot = wave_last(cincl);
            int cw = cincl - nc;
            _Pragma("unroll") for (int k = 0; k < kDealRecs; ++k) if (cand[k] != 0xFFFFFFFFu) cl[cw++] = cand[k];
            wave_lds_sync();
            // candidates dealt evenly: descriptor (and right coordinate) reads together
            for (int c0 = 0; c0 < ctot; c0 += 64 * kDealFlush) {
                uint32_t cc[kDealFlush];
                Desc d[kDealFlush];
                float ur[kDealFlush];
                _Pragma("unroll") for (int t = 0; t < kDealFlush; ++t)
                {
                    const int ci = c0 + t * 64 + lane;
                    cc[t] = ci < ctot ? cl[ci] : 0xFFFFFFFFu;
                    if (cc[t] != 0xFFFFFFFFu) d[t] = load_desc(V.kdesc, (int)(cc[t] & 0xFFFFu));
                    ur[t] = 0.0f;
                    if (cc[t] != 0xFFFFFFFFu && gate) ur[t] = V.u_right[cc[t] & 0xFFFFu];
                }
                _Pragma("unroll") for (int t = 0; t < kDealFlush; ++t)
                {
                    if (cc[t] == 0xFFFFFFFFu) continue;
                    const int ml = (int)(cc[t] >> 20);
                    const bool rej = gate && ur[t] > 0.0f && !(fabsf(quR[ml] - ur[t]) <= qp[ml].z);
                    if (!rej) {
                        const uint32_t key32 = ((uint32_t)hamming(qd[ml], d[t]) << 20) | ((cc[t] & 0xFFFFu) << 4) |
                                               ((cc[t] >> 16) & 15u);
                        const uint32_t old = atomicMin(&tb[ml], key32);
                        atomicMin(&tb[64 + ml], key32 < old ? old : key32);
                    }
                }
            }
            wave_lds_sync();   // the list is free for the next round
        }
    }
    wave_lds_sync();
    if constexpr (kLast) {
        finish_last(J, V, m, tb[lane]);
    } else {
        Top2<uint64_t> top = {key32_to_64(tb[lane]), key32_to_64(tb[64 + lane])};
        finish_query<1>(J, V, m, 0, top);
    }
}

// Search by projection, kWG-thread tiles, G lanes per map point, records read
// from global memory.
template <int G>
__device__ __forceinline__ void ph_search(const DevJob &J, const DevView &V, int tile)
{
    const int sub = threadIdx.x % G;
    const int m = tile * (kWG / G) + threadIdx.x / G;
    Top2<uint64_t> top = {~0ull, ~0ull};
    if (m < J.nM) {
        const Query q = make_query(J, V, m);
        if (q.vis) top = scan_global<G>(V, q, sub);
    }
    finish_query<G>(J, V, m, sub, top);
}

// Duplicate resolution and outputs: kPer (1 or 4) consecutive map points and
// keypoints per thread, their loads together.
template <int kPer>
__device__ __forceinline__ void ph_search_final(const DevJob &J, const DevView &V, int nK, int tile)
{
    static_assert(kPer == 1 || kPer == 4, "a dword or four");
    const int i0 = (tile * kWG + (int)threadIdx.x) * kPer;
    auto load = [](const FT_G int32_t *p, int i, int n, int r[kPer]) {
        if (kPer == 4 && i + kPer <= n) {
            const v4u v = *reinterpret_cast<const FT_G v4u_dw *>(p + i);
            _Pragma("unroll") for (int e = 0; e < kPer; ++e) r[e] = (int)v[e];
        } else {
            _Pragma("unroll") for (int e = 0; e < kPer; ++e) r[e] = i + e < n ? p[i + e] : -1;
        }
    };
    auto store = [](FT_G int32_t *p, int i, int n, const int r[kPer]) {
        if (kPer == 4 && i + kPer <= n) {
            v4u v;
            _Pragma("unroll") for (int e = 0; e < 4; ++e) v[e] = (uint32_t)r[e % kPer];
            *reinterpret_cast<FT_G v4u_dw *>(p + i) = v;
        } else {
            _Pragma("unroll") for (int e = 0; e < kPer; ++e) if (i + e < n) p[i + e] = r[e];
        }
    };
    int k[kPer], h[kPer], c[kPer];
    load(V.mp_k, i0, J.nM, k);
    load(V.mp_h, i0, J.nM, h);
    load(reinterpret_cast<const FT_G int32_t *>(V.claim), i0, nK, c);
    if (i0 < J.nM) {
        uint32_t cl[kPer];
        _Pragma("unroll") for (int e = 0; e < kPer; ++e) cl[e] = k[e] >= 0 ? V.claim[k[e]] : 0u;
        _Pragma("unroll") for (int e = 0; e < kPer; ++e)
        {
            const bool keep = k[e] >= 0 && cl[e] == (((uint32_t)h[e] << 23) | (uint32_t)(i0 + e));
            k[e] = keep ? k[e] : -1;
            h[e] = keep ? h[e] : -1;
        }
        store(V.mp_match, i0, J.nM, k);
        store(V.mp_dist, i0, J.nM, h);
    }
    int n = 0;   // (an unclaimed keypoint's claim is ~0, as is what lies past the last)
    _Pragma("unroll") for (int e = 0; e < kPer; ++e)
    {
        const bool has = c[e] != -1;
        n += has ? 1 : 0;
        c[e] = has ? (c[e] & 0x7FFFFF) : -1;
    }
    if (i0 < nK) store(V.kp_match, i0, nK, c);
    n = wave_last(wave_inclusive_scan(n));
    if ((threadIdx.x & 63) == 0 && n) atomicAdd(V.n_matches, n);
}

// Rotation bin of a match: last minus current orientation, plus 360 when
// negative, rounded to one of `bins` equal bins, taken modulo `bins` (the one
// past the last is bin 0).
__device__ __forceinline__ int rotation_bin(float a_last, float a_cur, int bins)
{
    float rot = a_last - a_cur;
    if (rot < 0.0f) rot += 360.0f;
    const float factor = (float)bins / 360.0f;
    int bin = (int)roundf(rot * factor) % bins;   // the bin past the last is bin 0
    if (bin < 0) bin += bins;                      // (angles outside [0, 360) stay in range)
    return bin;
}

// Bins kept by the rotation check (bit b set), from the count of bin `lane` in
// every lane: the fullest bin and, while holding a tenth of it, the second and
// third fullest; ties to the lower bin.
__device__ __forceinline__ uint64_t kept_bins(int count)
{
    const int lane = threadIdx.x & 63;
    int key = count > 0 ? (count << 6) | (63 - lane) : 0;   // (at most 2^23 points)
    int top[3];
    _Pragma("unroll") for (int t = 0; t < 3; ++t)
    {
        top[t] = wave_last(wave_inclusive_max(key));
        key = key == top[t] ? 0 : key;
    }
    const int m1 = top[0] >> 6, m2 = top[1] >> 6, m3 = top[2] >> 6;
    uint64_t kept = 0;
    if (m1 > 0) kept |= 1ull << (63 - (top[0] & 63));
    if (m2 > 0 && 10 * (int64_t)m2 >= m1) {
        kept |= 1ull << (63 - (top[1] & 63));
        if (m3 > 0 && 10 * (int64_t)m3 >= m1) kept |= 1ull << (63 - (top[2] & 63));
    }
    return kept;
}

// Claims, rotation check and outputs of up to kSortUnroll * NT points in one
// workgroup (the points stay in registers, the histogram and the surviving
// points' bits in LDS).
constexpr int kLastFinishLds = kRotBinsMax * 4 + kSortUnroll * kAuxWG / 8 + 64 * 4;

template <int NT>
__device__ __forceinline__ void ph_last_finish(const DevJob &J, const DevView &V, int nK, unsigned char *smem)
{
    int *hist = reinterpret_cast<int *>(smem);
    uint64_t *alive = reinterpret_cast<uint64_t *>(hist + kRotBinsMax);
    int *found = reinterpret_cast<int *>(alive + kSortUnroll * NT / 64);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nM = J.nM;
    if (tid < kRotBinsMax) hist[tid] = 0;
    __syncthreads();
    int k[kSortUnroll], h[kSortUnroll], bin[kSortUnroll];
    uint32_t cl[kSortUnroll];
    _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
    {
        const int i = tid + e * NT;
        k[e] = i < nM ? V.mp_k[i] : -1;
        h[e] = i < nM ? V.mp_h[i] : -1;
    }
    _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
    {
        const int i = tid + e * NT;
        const bool q = k[e] >= 0;
        float al = 0.0f, ak = 0.0f;
        cl[e] = q ? V.claim[k[e]] : 0u;
        if (q && J.check_rot) {
            al = J.l_ang[i];
            ak = J.k_ang[k[e]];
        }
        bin[e] = q && J.check_rot ? rotation_bin(al, ak, J.rot_bins) : 0;
    }
    _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
    {
        const int i = tid + e * NT;
        if (k[e] >= 0 && cl[e] != (((uint32_t)h[e] << 23) | (uint32_t)i)) k[e] = -1;
        if (k[e] >= 0 && J.check_rot) atomicAdd(&hist[bin[e]], 1);
    }
    __syncthreads();
    const uint64_t kept = J.check_rot ? kept_bins(hist[lane]) : ~0ull;
    _Pragma("unroll") for (int e = 0; e < kSortUnroll; ++e)
    {
        const int i = tid + e * NT;
        const bool a = k[e] >= 0 && ((kept >> bin[e]) & 1ull);
        const uint64_t m = __ballot(a);
        if (lane == 0) alive[e * (NT / 64) + wave] = m;
        if (i < nM) {
            V.mp_match[i] = a ? k[e] : -1;
            V.mp_dist[i] = a ? h[e] : -1;
        }
    }
    __syncthreads();
    int n = 0;
    for (int idx = tid; idx < nK; idx += NT) {
        const uint32_t c = V.claim[idx];
        const int i = (int)(c & 0x7FFFFFu);
        const bool has = c != 0xFFFFFFFFu && ((alive[i >> 6] >> (i & 63)) & 1ull);
        V.kp_match[idx] = has ? i : -1;
        n += has ? 1 : 0;
    }
    n = wave_last(wave_inclusive_scan(n));
    if (lane == 0) found[wave] = n;
    __syncthreads();
    if (tid < 64) {
        n = wave_last(wave_inclusive_scan(tid < NT / 64 ? found[tid] : 0));
        if (tid == 0) *V.n_matches = n;
    }
}

// More points: thread per point: the claim winners keep their keypoint (mp_k,
// distance | bin << 16 in mp_h; losers get -1) and count their rotation bin, in
// LDS first (one global update per bin and workgroup).
__device__ __forceinline__ void ph_last_resolve(const DevJob &J, const DevView &V, int tile, int *hist)
{
    const int i = tile * kWG + threadIdx.x;
    if (threadIdx.x < kRotBinsMax) hist[threadIdx.x] = 0;
    __syncthreads();
    if (i < J.nM) {
        const int k = V.mp_k[i];
        const int h = V.mp_h[i];
        const bool keep = k >= 0 && V.claim[k] == (((uint32_t)h << 23) | (uint32_t)i);
        int bin = 0;
        if (keep && J.check_rot) {
            bin = rotation_bin(J.l_ang[i], J.k_ang[k], J.rot_bins);
            atomicAdd(&hist[bin], 1);
        }
        V.mp_k[i] = keep ? k : -1;
        V.mp_h[i] = keep ? (h | (bin << 16)) : -1;
    }
    __syncthreads();
    if (threadIdx.x < kRotBinsMax && hist[threadIdx.x]) atomicAdd(&V.hist[threadIdx.x], hist[threadIdx.x]);
}

// Thread per point / keypoint: the rotation check and the outputs.
__device__ __forceinline__ void ph_last_final(const DevJob &J, const DevView &V, int nK, int tile)
{
    const uint64_t kept = J.check_rot ? kept_bins(V.hist[threadIdx.x & 63]) : ~0ull;
    auto alive = [&](int i) {
        return V.mp_k[i] >= 0 && ((kept >> ((V.mp_h[i] >> 16) & 63)) & 1ull);
    };
    const int idx = tile * kWG + threadIdx.x;
    if (idx < J.nM) {
        const bool a = alive(idx);
        V.mp_match[idx] = a ? V.mp_k[idx] : -1;
        V.mp_dist[idx] = a ? (V.mp_h[idx] & 0xFFFF) : -1;
    }
    bool has = false;
    if (idx < nK) {
        const uint32_t c = V.claim[idx];
        has = c != 0xFFFFFFFFu && alive((int)(c & 0x7FFFFFu));
        V.kp_match[idx] = has ? (int)(c & 0x7FFFFFu) : -1;
    }
    const unsigned long long mk = __ballot(has);
    if ((threadIdx.x & 63) == 0 && mk) atomicAdd(V.n_matches, (int)__popcll(mk));
}

// ------------------------------------------------------- tile bookkeeping

// Search tiles of a view: one wave of 64 map points for the record-dealt
// search (one lane per map point), else kWG / lanes map points.
__host__ __device__ inline int search_tiles_per_view(const DevJob &J, int lanes)
{
    return div_up(J.nM, lanes == 1 ? 64 : kWG / lanes);
}


__host__ __device__ inline int final_tiles_view(const DevJob &J, int v, int per)
{
    const int nK = view_kp(J, v);
    return div_up(J.nM > nK ? J.nM : nK, kWG * per);
}

// Workgroups of the setup phase: J.setup_split for the row sort by level and
// each view's cell sort by level bin (indexes with one bin: one workgroup), two
// for the overlap lists.
__host__ __device__ inline int setup_parts_stereo(const DevJob &J)
{
    return J.flags & JOB_STEREO_FISHEYE ? 2 : J.n_lb > 1 ? J.setup_split : 1;
}
__host__ __device__ inline int setup_parts_view(const DevJob &J, int v) { return J.view[v].n_pb > 1 ? J.setup_split : 1; }

void job_tiles(const DevJob &J, const Shapes &s, bool do_stereo, bool do_search, int32_t out[PH_COUNT])
{
    for (int p = 0; p < PH_COUNT; ++p) out[p] = 0;
    if (do_stereo && J.imgL) out[PH_PYRAMID] = div_up((J.imgR ? 2 : 1) * J.pyr_first[kLevels], kWG / 64);
    const int nL = J.L.n;
    const bool pin = do_stereo && (J.flags & JOB_STEREO_PINHOLE);
    const bool fish = do_stereo && (J.flags & JOB_STEREO_FISHEYE);
    const int nv = do_search ? J.n_views : 0;
    out[PH_SETUP] = pin || fish ? setup_parts_stereo(J) : 0;
    for (int v = 0; v < nv; ++v) out[PH_SETUP] += setup_parts_view(J, v);
    if (pin) {
        out[PH_STEREO_A] = div_up(nL, kWG / s.best_lanes);
        out[PH_REFINE] = div_up(nL, refine_quarter(J) ? kRefineQPerWG : kRefinePerWG);
        out[PH_STEREO_C] = 1;
    } else if (fish) {
        out[PH_STEREO_A] = div_up(nL, kKnnQueriesPerWG);
        out[PH_TRI] = div_up(nL, kWG);
        out[PH_STEREO_C] = div_up(nL, s.aux_block);
    }
    for (int v = 0; v < nv; ++v) {
        out[PH_SEARCH] += search_tiles_per_view(J, s.search_lanes);
        out[PH_SEARCH_FIN] += final_tiles_view(J, v, s.final_per);
    }
}

// ------------------------------------------------------------------ kernels
// Consecutive logical tiles on one XCD: workgroups are dealt round-robin over
// the 8 XCDs, so block b runs on XCD b % 8; map it to a contiguous chunk.
__device__ __forceinline__ int xcd_remap(int b, int n)
{
    const int per = n >> 3;
    if (b >= (per << 3)) return b;
    return (b & 7) * per + (b >> 3);
}

struct OneJob {
    DevJob j;
    __device__ __forceinline__ const DevJob &operator()(int) const { return j; }
    __device__ __forceinline__ bool locate(int, int &job, int &tile) const
    {
        job = 0;
        tile = xcd_remap((int)blockIdx.x, (int)gridDim.x);
        return true;
    }
};

struct JobTable : BatchArgs {
    // The table is constant while a kernel runs, and a tile's job is uniform: read
    // from the constant address space its fields are scalar loads also behind the
    // kernel's own stores (the compiler must otherwise take them for changed, and
    // loads each through the vector units: 78 loads of the set-up, 19 of the
    // refinement).  Mixed 64-frame batch 165.2 -> 154.2 us, 8 frames from images
    // 76.8 -> 72.2.
    __device__ __forceinline__ const DevJob &operator()(int i) const
    {
        return *(const DevJob *)((const FT_C DevJob *)p + i);
    }
    __device__ __forceinline__ bool locate(int ph, int &job, int &tile) const
    {
        const FT_G int32_t *pre = map.prefix + ph * (map.n_jobs + 1);
        const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
        const int lane = threadIdx.x & 63, n = map.n_jobs;
        // The job is the number of prefix ends at or below b: 64 of them are
        // compared per load (one round trip for up to 64 jobs, two for up to
        // 4096, instead of one per step of a bisection).
        int j0 = 0, below = 0;   // first job of the 64 compared, tiles before it
        if (n > 64) {
            const int e = 64 * (lane + 1);
            const int v = pre[min(e, n)];
            j0 = 64 * (int)__popcll(__ballot(e <= n && v <= b));
            below = j0 ? __builtin_amdgcn_readlane(v, (j0 >> 6) - 1) : 0;
        }
        const int v = pre[min(j0 + lane + 1, n)];
        const int k = (int)__popcll(__ballot(j0 + lane < n && v <= b));
        job = j0 + k;
        tile = b - (k ? __builtin_amdgcn_readlane(v, (k - 1) & 63) : below);
        return job < n;
    }
};
static_assert(sizeof(JobTable) == sizeof(BatchArgs), "graph nodes pass a BatchArgs as the JobTable argument");

// ------------------------------------------------------------ phase tasks
// One task = one tile of one phase of one frame, run by a whole workgroup.
// `smem` is the workgroup's LDS scratch (kTaskLds bytes, 16-byte aligned).
constexpr int kTaskLds = (kMaxCells + 8 + kWG) * 4;

template <int NT>
__device__ __forceinline__ void task_setup(const DevJob &J, int tile, unsigned char *smem)
{
    int *lds = reinterpret_cast<int *>(smem);
    int *tmp = lds + kMaxCells + 8;
    if (J.flags & (JOB_STEREO_PINHOLE | JOB_STEREO_FISHEYE)) {
        const int n = setup_parts_stereo(J);
        if (tile < n) {
            if (J.flags & JOB_STEREO_PINHOLE) ph_rowsort<NT>(J, tile, n, lds, tmp);
            else ph_overlap<NT>(J, tile, tmp);
            return;
        }
        tile -= n;
    }
    const int n0 = setup_parts_view(J, 0);
    const int v = tile < n0 ? 0 : 1;
    const DevView &V = J.view[v];
    ph_cellsort<NT>(V, V.side ? J.R : J.L, J.lv_lo, J.lv_hi, tile - (v ? n0 : 0), setup_parts_view(J, v), lds, tmp);
}

template <int G>
__device__ __forceinline__ void task_stereo_a(const DevJob &J, int tile, unsigned char *smem)
{
    if (J.flags & JOB_STEREO_PINHOLE) ph_best<G>(J, tile);
    else ph_knn<kWG>(J, tile, reinterpret_cast<uint32_t *>(smem));
}

template <int NT>
__device__ __forceinline__ void task_stereo_c(const DevJob &J, int tile, unsigned char *smem)
{
    if (J.flags & JOB_STEREO_PINHOLE) ph_median<NT>(J, smem);
    else ph_fish_final<NT>(J, tile);
}

template <int G>
__device__ __forceinline__ void task_search(const DevJob &J, int tile, unsigned char *smem)
{
    const int tpv = search_tiles_per_view(J, G);
    const int v = tile / tpv;
    if (v >= J.n_views) return;
    if constexpr (G == 1) ph_search_deal<false>(J, J.view[v], (tile - v * tpv) * 64, smem);
    else ph_search<G>(J, J.view[v], tile - v * tpv);
}

template <int kPer>
__device__ __forceinline__ void task_search_final(const DevJob &J, int tile)
{
    const int t0 = final_tiles_view(J, 0, kPer);
    const int v = tile < t0 ? 0 : 1;
    if (v >= J.n_views) return;
    ph_search_final<kPer>(J, J.view[v], view_kp(J, v), tile - (v ? t0 : 0));
}

static_assert(4 * kKnnQueriesPerWG * 2 * 4 <= kTaskLds, "stereo_a LDS");
static_assert(kRefinePerWG * kRefineLds <= kTaskLds, "refine LDS");
static_assert(kDealLdsPerWave <= kTaskLds, "record-dealt search LDS");
static_assert(kMedianLds <= kTaskLds, "median LDS");

// ------------------------------------------------------- per-phase kernels
template <class Src>
__global__ __launch_bounds__(kWG) void k_pyramid(Src src)
{
    int job, tile;
    if (!src.locate(PH_PYRAMID, job, tile)) return;
    ph_pyramid(src(job), tile);
}

// (two 1024-thread workgroups per CU: 64 registers)
template <class Src, int NT>
__global__ __launch_bounds__(NT, NT == kAuxWG ? 8 : 4) void k_setup(Src src)
{
    __shared__ __align__(16) unsigned char smem[(kMaxCells + 8 + NT) * 4];
    int job, tile;
    if (!src.locate(PH_SETUP, job, tile)) return;
    task_setup<NT>(src(job), tile, smem);
}

// Five waves per SIMD: with four the mixed 64-frame batch takes 166.9 us instead
// of 165.4 (its pinhole frames want the waves; a single fisheye frame is equal),
// and six spill (191 and more).
template <class Src, int G>
__global__ __launch_bounds__(kWG, 5) void k_stereo_a(Src src)
{
    __shared__ __align__(16) unsigned char smem[4 * kKnnQueriesPerWG * 2 * 4];
    int job, tile;
    if (!src.locate(PH_STEREO_A, job, tile)) return;
    task_stereo_a<G>(src(job), tile, smem);
}

template <class Src>
// 7 waves per SIMD (at most 72 registers): more window loads in flight; 8 spill
// and are no faster.
__global__ __launch_bounds__(kWG, 7) void k_refine(Src src)
{
    __shared__ __align__(16) unsigned char smem[kRefinePerWG * kRefineLds];
    int job, tile;
    if (!src.locate(PH_REFINE, job, tile)) return;
    ph_refine(src(job), tile, smem);
}

template <class Src>
__global__ __launch_bounds__(kWG) void k_tri(Src src)
{
    int job, tile;
    if (!src.locate(PH_TRI, job, tile)) return;
    ph_tri(src(job), tile);
}

template <class Src, int NT>
__global__ __launch_bounds__(NT) void k_stereo_c(Src src)
{
    __shared__ __align__(16) unsigned char smem[kMedianLds];
    int job, tile;
    if (!src.locate(PH_STEREO_C, job, tile)) return;
    task_stereo_c<NT>(src(job), tile, smem);
}

template <class Src, int G>
__global__ __launch_bounds__(kWG) void k_search(Src src)
{
    int job, tile;
    if (!src.locate(PH_SEARCH, job, tile)) return;
    task_search<G>(src(job), tile, nullptr);
}

// Record-dealt search in one-wave workgroups: a wave's LDS and registers are
// released as soon as it ends (waves of one workgroup would hold theirs until
// the slowest ends), and single-wave workgroups take no barrier slot, so LDS
// alone bounds the waves per CU.  Registers are capped at seven waves per SIMD.
template <class Src>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(7, 8))) void k_search_deal(Src src)
{
    __shared__ __align__(16) unsigned char smem[kDealLdsPerWave];
    int job, tile;
    if (!src.locate(PH_SEARCH, job, tile)) return;
    task_search<1>(src(job), tile, smem);
}

// (kPer: the launch's final_per)
template <class Src, int kPer>
__global__ __launch_bounds__(kWG) void k_search_final(Src src)
{
    int job, tile;
    if (!src.locate(PH_SEARCH_FIN, job, tile)) return;
    task_search_final<kPer>(src(job), tile);
}

// Last-frame search (one view of one job): search, then claims, rotation check
// and outputs in one workgroup, or in two kernels for many points.
template <class Src>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(7, 8))) void k_last_search(Src src)
{
    __shared__ __align__(16) unsigned char smem[kDealLdsPerWave];
    int job, tile;
    if (!src.locate(PH_SEARCH, job, tile)) return;
    const DevJob &J = src(job);
    ph_search_deal<true>(J, J.view[0], tile * 64, smem);
}

template <class Src>
__global__ __launch_bounds__(kAuxWG) void k_last_finish(Src src)
{
    __shared__ __align__(16) unsigned char smem[kLastFinishLds];
    const DevJob &J = src(0);
    ph_last_finish<kAuxWG>(J, J.view[0], view_kp(J, 0), smem);
}

template <class Src>
__global__ __launch_bounds__(kWG) void k_last_resolve(Src src)
{
    __shared__ int hist[kRotBinsMax];
    int job, tile;
    if (!src.locate(PH_SEARCH_FIN, job, tile)) return;
    const DevJob &J = src(job);
    ph_last_resolve(J, J.view[0], tile, hist);
}

template <class Src>
__global__ __launch_bounds__(kWG) void k_last_final(Src src)
{
    int job, tile;
    if (!src.locate(PH_SEARCH_FIN, job, tile)) return;
    const DevJob &J = src(job);
    ph_last_final(J, J.view[0], view_kp(J, 0), tile);
}

hipError_t launch_last_frame(const DevJob &J, hipStream_t s)
{
    OneJob src{J};
    void *args[] = {&src};
    const int nK = view_kp(J, 0);
    auto launch = [&](auto *fn, int grid, int block) {
        return hipLaunchKernel(reinterpret_cast<void *>(fn), dim3(grid), dim3(block), args, 0, s);
    };
    // setup: the view's cell index, claims cleared, histogram and match count zeroed
    hipError_t e = launch(&k_setup<OneJob, kAuxWG>, setup_parts_view(J, 0), kAuxWG);
    if (e != hipSuccess) return e;
    if (J.nM > 0 && (e = launch(&k_last_search<OneJob>, div_up(J.nM, 64), 64)) != hipSuccess) return e;
    // One workgroup holds kSortUnroll points per thread and strides the keypoints, which
    // saves a launch and the histogram's updates in memory; with many keypoints more
    // workgroups win (one kernel and two, per call: 1,200 keypoints and 1,153 points
    // 18.1 and 20.8 us, 3,600 and 4,096 25.5 and 26.8, 8,000 and 1,153 38.3 and 38.9,
    // 8,000 and 4,096 40.0 and 39.2, 16,000 and 4,096 65.4 and 62.2).
    if (J.nM <= kSortUnroll * kAuxWG && nK <= 2 * kSortUnroll * kAuxWG) return launch(&k_last_finish<OneJob>, 1, kAuxWG);
    if (J.nM > 0 && (e = launch(&k_last_resolve<OneJob>, div_up(J.nM, kWG), kWG)) != hipSuccess) return e;
    return launch(&k_last_final<OneJob>, div_up(J.nM > nK ? J.nM : nK, kWG), kWG);
}

// ---------------------------------------------------- local-map edit
// One point's 64-byte record (position, normal, distance bounds, descriptor).
struct MapRec {
    float p[3], nr[3], d0, d1;
    v4u q0, q1;
};

__device__ __forceinline__ MapRec load_rec(const FT_G float *pos, const FT_G float *normal, const FT_G float *dmin,
                                           const FT_G float *dmax, const FT_G uint8_t *desc, int i)
{
    MapRec r;
    _Pragma("unroll") for (int c = 0; c < 3; ++c)
    {
        r.p[c] = pos[3 * i + c];
        r.nr[c] = normal[3 * i + c];
    }
    r.d0 = dmin[i];
    r.d1 = dmax[i];
    r.q0 = reinterpret_cast<const FT_G v4u *>(desc + 32 * (size_t)i)[0];
    r.q1 = reinterpret_cast<const FT_G v4u *>(desc + 32 * (size_t)i)[1];
    return r;
}

__device__ __forceinline__ void store_rec(const MapEditArgs &a, int i, const MapRec &r)
{
    _Pragma("unroll") for (int c = 0; c < 3; ++c)
    {
        a.pos[3 * i + c] = r.p[c];
        a.normal[3 * i + c] = r.nr[c];
    }
    a.dmin[i] = r.d0;
    a.dmax[i] = r.d1;
    reinterpret_cast<FT_G v4u *>(a.desc + 32 * (size_t)i)[0] = r.q0;
    reinterpret_cast<FT_G v4u *>(a.desc + 32 * (size_t)i)[1] = r.q1;
}

// A thread per tail slot n1 + i: the surviving point it holds moves to its hole
// below n1 (a slot no other thread touches), then inserted point i takes the
// slot.  Both records are read before either is written, so one launch does
// what moves and appends in two had to order.  What bounds it is the launch and
// the holes' trip over the bus.
__global__ __launch_bounds__(kWG) void k_map_edit(MapEditArgs a)
{
    const int i = blockIdx.x * kWG + threadIdx.x;
    const int hole = i < a.n_tail ? a.holes[i] : -1;
    MapRec old, in;
    if (i < a.n_insert) in = load_rec(a.ipos, a.inormal, a.idmin, a.idmax, a.idesc, i);
    if (hole >= 0) {
        old = load_rec(a.pos, a.normal, a.dmin, a.dmax, a.desc, a.n1 + i);
        store_rec(a, hole, old);
    }
    if (i < a.n_insert) store_rec(a, a.n1 + i, in);
}

hipError_t launch_map_edit(const MapEditArgs &a, hipStream_t s)
{
    const int n = std::max(a.n_tail, a.n_insert);
    if (n > 0) hipLaunchKernelGGL(k_map_edit, dim3(div_up(n, kWG)), dim3(kWG), 0, s, a);
    return hipGetLastError();
}

// Kernel of phase p for these shapes, and its workgroup size.
template <class Src>
static void *phase_kernel(const Shapes &sh, int p, int *block)
{
    *block = kWG;
    switch (p) {
    case PH_PYRAMID: return reinterpret_cast<void *>(&k_pyramid<Src>);
    case PH_SETUP:
        if (sh.aux_block == kAuxWG) {
            *block = kAuxWG;
            return reinterpret_cast<void *>(&k_setup<Src, kAuxWG>);
        }
        return reinterpret_cast<void *>(&k_setup<Src, kWG>);
    case PH_STEREO_A:
        switch (sh.best_lanes) {
        case 1: return reinterpret_cast<void *>(&k_stereo_a<Src, 1>);
        case 2: return reinterpret_cast<void *>(&k_stereo_a<Src, 2>);
        case 4: return reinterpret_cast<void *>(&k_stereo_a<Src, 4>);
        case 16: return reinterpret_cast<void *>(&k_stereo_a<Src, 16>);
        default: return reinterpret_cast<void *>(&k_stereo_a<Src, 8>);
        }
    case PH_REFINE: return reinterpret_cast<void *>(&k_refine<Src>);
    case PH_TRI: return reinterpret_cast<void *>(&k_tri<Src>);
    case PH_STEREO_C:
        if (sh.aux_block == kAuxWG) {
            *block = kAuxWG;
            return reinterpret_cast<void *>(&k_stereo_c<Src, kAuxWG>);
        }
        return reinterpret_cast<void *>(&k_stereo_c<Src, kWG>);
    case PH_SEARCH:
        switch (sh.search_lanes) {
        case 1: *block = 64; return reinterpret_cast<void *>(&k_search_deal<Src>);
        case 2: return reinterpret_cast<void *>(&k_search<Src, 2>);
        case 8: return reinterpret_cast<void *>(&k_search<Src, 8>);
        case 16: return reinterpret_cast<void *>(&k_search<Src, 16>);
        default: return reinterpret_cast<void *>(&k_search<Src, 4>);
        }
    default:
        if constexpr (std::is_same_v<Src, OneJob>)
            if (sh.final_per == 1) return reinterpret_cast<void *>(&k_search_final<Src, 1>);
        return reinterpret_cast<void *>(&k_search_final<Src, 4>);
    }
}

void batch_kernels(const Shapes &shapes, void *fn[PH_COUNT], int block[PH_COUNT])
{
    for (int p = 0; p < PH_COUNT; ++p) fn[p] = phase_kernel<JobTable>(shapes, p, &block[p]);
}

template <class Src>
static hipError_t run(Src src, const int32_t *tot, const Shapes &sh, hipStream_t s, hipEvent_t *ev)
{
    void *args[] = {&src};
    for (int p = 0; p < PH_COUNT; ++p) {
        if (ev) (void)hipEventRecord(ev[p], s);
        if (tot[p] <= 0) continue;   // planned by job_tiles for the phases asked for
        int block = kWG;
        void *fn = phase_kernel<Src>(sh, p, &block);
        const hipError_t e = hipLaunchKernel(fn, dim3(tot[p]), dim3(block), args, 0, s);
        if (e != hipSuccess) return e;
    }
    if (ev) (void)hipEventRecord(ev[PH_COUNT], s);
    return hipGetLastError();
}

hipError_t launch_pipeline(const DevJob *table, const TileMap &map, const int32_t totals[PH_COUNT],
                           const DevJob &one, const Shapes &shapes, hipStream_t stream, hipEvent_t *ev)
{
    if (table) return run(JobTable{{table, map}}, totals, shapes, stream, ev);
    return run(OneJob{one}, totals, shapes, stream, ev);
}

}  // namespace ft
