// ORB extraction on the device-resident image pyramid (Section II-A: keypoints
// are extracted on every scale and described; Section IV-B: the extraction
// runs next to the pyramid on the device).
//
//  * k_orb_detect: one workgroup per tile of kOrbRows rows of one level.  The
//    tile's level rows and kOrbHalo rows above and below are staged in LDS;
//    FAST-9 scores, four pixels per lane, fill a score band one row larger on
//    each side; strict 3x3 suppression collects the tile's corners in (row,
//    column) order in LDS; the tile publishes its count, and its first output
//    index is the sum of the counts of the tiles before it (tiles are in (level,
//    row) order and taken by ticket), so the corners are written contiguously;
//    the descriptor's binomial smoothing of the tile's rows is written from the
//    same staged rows.
//  * k_orb_describe: one wave per keypoint: the intensity-centroid moments
//    over the radius-15 disc (byte dot products, one wave reduction), then four
//    tests per lane on the smoothed window in LDS with the pattern turned exactly
//    by the moments (integer rounding decisions), and one ballot per 64 tests
//    gives 8 descriptor bytes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#define FT_KERNELS 1
#include "ft_internal.h"

namespace ft {

namespace {

constexpr int kThreads = 256;      // description: one wave per keypoint, 4 waves per workgroup
constexpr int kDetThreads = 512;   // detection: one tile per workgroup, two workgroups per CU
constexpr int kDetWaves = kDetThreads / 64;
constexpr int kStaged = kOrbRows + 2 * kOrbHalo;   // level rows staged per tile
constexpr int kScoreRows = kOrbRows + 2;           // score rows: the tile and one row each side
static_assert(kOrbRows % 2 == 0 && kOrbRows <= 8 && kMaxPyrW < 2048, "emitted corners pack column, row, score");

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef v4u v4u_dw __attribute__((aligned(4)));       // four dwords from a dword boundary
typedef uint32_t u32_any __attribute__((aligned(1)));  // a dword at any byte address

// The 16 ring pixels at distance 3 (clockwise from straight above).
constexpr int kRingDx[16] = {0, 1, 2, 3, 3, 3, 2, 1, 0, -1, -2, -3, -3, -3, -2, -1};
constexpr int kRingDy[16] = {-3, -3, -2, -1, 0, 1, 2, 3, 3, 3, 2, 1, 0, -1, -2, -3};

__device__ __forceinline__ int level_of_tile(const OrbDetectArgs &a, int tile)
{
    int l = 0;
    while (l + 1 < kLevels && tile >= a.tile0[l + 1]) ++l;
    return l;
}

// Inclusive prefix sum over the 64 lanes of a wave (every lane active) by DPP
// moves: shifts by 1, 2, 4 and 8 inside rows of 16 lanes, then lane 15 of rows 0
// and 2 into rows 1 and 3, then lane 31 into rows 2 and 3.
__device__ __forceinline__ int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31
    return v;
}

// Sum over the 64 lanes, wave-uniform.
__device__ __forceinline__ int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_scan(v), 63); }

// LDS rows of a level W wide: 4 bytes, the W pixels, at least 8 bytes; whole
// dwords, so pixel x of a row lies at byte 4 + x and groups of four pixels on
// dword boundaries.
__host__ __device__ inline int row_stride(int W) { return (W + 15) & ~3; }

// it / n for 0 <= it < 2^15, 0 < n < 2^11 (inv = 1 / n in binary32): the exact
// quotient is at least 1 / (2n) away from an integer, far above the rounding.
__device__ __forceinline__ int div_items(int it, float inv) { return (int)(((float)it + 0.5f) * inv); }

__device__ __forceinline__ u16x2 pk(uint32_t v) { return __builtin_bit_cast(u16x2, v); }

// Bytes j and j + 1 of the twelve in w as a pair of 16-bit values (j constant).
__device__ __forceinline__ u16x2 byte_pair(const uint32_t w[3], int j)
{
    const int k = j < 7 ? j : j - 4;
    const uint32_t sel = 0x0C000C00u | (uint32_t)k | ((uint32_t)(k + 1) << 16);
    return pk(j < 7 ? __builtin_amdgcn_perm(w[1], w[0], sel) : __builtin_amdgcn_perm(w[2], w[1], sel));
}

// Twelve bytes x - 4 .. x + 7 of an LDS row (x a multiple of 4).
__device__ __forceinline__ void row_window(const unsigned char *row, int x, uint32_t w[3])
{
    const uint32_t *q = reinterpret_cast<const uint32_t *>(row + x);   // (the row's pixels start 4 bytes in)
    w[0] = q[0];
    w[1] = q[1];
    w[2] = q[2];
}

// FAST-9 scores of the four pixels x .. x + 3 whose ring's top row is the LDS
// row `top`, one byte each: the largest, over the 16 arcs of nine ring pixels,
// of (smallest ring pixel - centre) and (centre - largest ring pixel), minus
// one; 0 unless it reaches t.  Two pixels per packed 16-bit operation.  The two
// arcs that start at ring pixels k and k + 1 share the eight pixels k + 1 ..
// k + 8, so eight windows of eight pixels (by doubling) and one more pixel from
// either side give all 16: max(min(m, e[k]), min(m, e[k + 9])) =
// min(m, max(e[k], e[k + 9])).
__device__ __forceinline__ uint32_t fast_scores(const unsigned char *top, int S, int x, uint32_t t)
{
    uint32_t w[7][3];
    _Pragma("unroll") for (int r = 0; r < 7; ++r) row_window(top + r * S, x, w[r]);
    uint32_t out[2];
    _Pragma("unroll") for (int h = 0; h < 2; ++h)
    {
        u16x2 e[16];
        _Pragma("unroll") for (int k = 0; k < 16; ++k) e[k] = byte_pair(w[3 + kRingDy[k]], 4 + 2 * h + kRingDx[k]);
        const u16x2 c = byte_pair(w[3], 4 + 2 * h);
        auto lo = [](u16x2 a, u16x2 b) { return __builtin_elementwise_min(a, b); };
        auto hi = [](u16x2 a, u16x2 b) { return __builtin_elementwise_max(a, b); };
        u16x2 bright = {0, 0}, dark = {255, 255};   // best arc minimum; smallest arc maximum
        {
            u16x2 a2[16], a4[16];
            _Pragma("unroll") for (int k = 1; k < 16; k += 2) a2[k] = lo(e[k], e[(k + 1) & 15]);
            _Pragma("unroll") for (int k = 1; k < 16; k += 2) a4[k] = lo(a2[k], a2[(k + 2) & 15]);
            _Pragma("unroll") for (int k = 1; k < 16; k += 2)
                bright = hi(bright, lo(lo(a4[k], a4[(k + 4) & 15]), hi(e[k - 1], e[(k + 8) & 15])));
        }
        {
            u16x2 a2[16], a4[16];
            _Pragma("unroll") for (int k = 1; k < 16; k += 2) a2[k] = hi(e[k], e[(k + 1) & 15]);
            _Pragma("unroll") for (int k = 1; k < 16; k += 2) a4[k] = hi(a2[k], a2[(k + 2) & 15]);
            _Pragma("unroll") for (int k = 1; k < 16; k += 2)
                dark = lo(dark, hi(hi(a4[k], a4[(k + 4) & 15]), lo(e[k - 1], e[(k + 8) & 15])));
        }
        const i16x2 d = __builtin_elementwise_max(__builtin_bit_cast(i16x2, (u16x2)(bright - c)),
                                                  __builtin_bit_cast(i16x2, (u16x2)(c - dark)));
        // d = score + 1 >= t + 1, else 0 (t < 255, so t + 1 fits)
        const u16x2 sp = __builtin_bit_cast(u16x2, __builtin_elementwise_max(d, i16x2{0, 0}));
        const u16x2 over = __builtin_elementwise_sub_sat(sp, u16x2{(unsigned short)t, (unsigned short)t});
        const u16x2 keep = __builtin_elementwise_min(over, u16x2{1, 1});
        out[h] = __builtin_bit_cast(uint32_t, (u16x2)((sp - keep) * keep));
    }
    return __builtin_amdgcn_perm(out[1], out[0], 0x06040200u);
}

// Look-back state of a tile: epoch << 32 | published << 30 | corners.
constexpr unsigned long long kPublished = 1ull << 30;
constexpr uint32_t kValueMask = (1u << 30) - 1u;
constexpr int kMaxSpins = 1 << 16;       // bounds every wait (a tile found stuck poisons the prefix)
constexpr int kPoison = 1 << 29;         // prefix of a tile whose predecessors never published

// One tile.  What bounds it is the chain ticket, staging, scores, suppression,
// look-back, output of a single tile (277 tiles of a 752x480 pyramid on 256
// CUs, one round), so the work per pixel is cut where it is vector issue: four
// pixels per lane from dword LDS reads, two per packed 16-bit operation (about
// 60 instructions per pixel against 220 one pixel at a time), the smoothing by
// byte dot products, and the tile's count is published before the smoothing so
// that the other tiles' counts arrive meanwhile.
__global__ __launch_bounds__(kDetThreads, 4) void k_orb_detect(OrbDetectArgs a)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int kItems = (kOrbRows * ((kMaxPyrW + 3) / 4) + kDetThreads - 1) / kDetThreads;   // four-pixel items per thread
    static_assert(kItems * kDetWaves <= 64, "one lane per (round, wave) count");
    __shared__ int wave_n[kItems * kDetWaves];
    __shared__ int shared_tile, wave_prefix[kDetWaves];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // tiles by ticket: every lower tile has been taken by a running workgroup,
    // and none waits on a higher one, so each wait below ends
    if (tid == 0) shared_tile = (int)(atomicAdd(a.ticket, 1u) - a.ticket_base);
    if (tid < kItems * kDetWaves) wave_n[tid] = 0;
    __syncthreads();
    const int tile = __builtin_amdgcn_readfirstlane(shared_tile);
    const int tiles = a.tile0[kLevels];
    const int l = level_of_tile(a, tile);
    const int W = a.w[l], H = a.h[l], S = row_stride(W), E = a.edge;
    const int y0 = (tile - a.tile0[l]) * kOrbRows;
    const int rows = min(kOrbRows, H - y0);
    unsigned char *px = lds;                                // staged rows
    unsigned char *sc = lds + kStaged * row_stride(a.lds_w);  // scores: rows y0 - 1 .. y0 + rows
    uint32_t *tc = reinterpret_cast<uint32_t *>(sc + kScoreRows * row_stride(a.lds_w));
    const FT_G uint8_t *img = a.pyr + a.off[l];
    // Stage rows y0 - 4 .. y0 + rows + 3 (clamped), each from 4 pixels before
    // its first to 8 past its last (clamped), as dwords realigned from the
    // level's (every dword read holds a byte of the row); the ones that hold a
    // clamped pixel byte by byte.
    {
        const int nd = S >> 2, n = (rows + 2 * kOrbHalo) * nd;
        const float inv = 1.0f / (float)nd;
        constexpr int kPer = (kStaged * ((kMaxPyrW + 15) / 4) + kDetThreads - 1) / kDetThreads;
        constexpr int kBatch = 4;   // dwords per thread whose loads are issued together
        for (int k0 = 0; k0 < kPer; k0 += kBatch) {
            if (k0 * kDetThreads >= n) break;
            uint32_t v[kBatch];
            _Pragma("unroll") for (int k = 0; k < kBatch; ++k)
            {
                const int it = min((k0 + k) * kDetThreads + tid, n - 1);
                const int sr = div_items(it, inv), x = 4 * (it - sr * nd) - 4;
                const int yy = min(max(y0 - kOrbHalo + sr, 0), H - 1);
                const FT_G uint8_t *row = img + (int64_t)yy * W;
                if (x >= 0 && x + 4 <= W) {
                    const uint32_t sh = (uint32_t)reinterpret_cast<uintptr_t>(row + x) & 3u;
                    const FT_G uint32_t *q = reinterpret_cast<const FT_G uint32_t *>(row + x - sh);
                    v[k] = __builtin_amdgcn_alignbyte(q[sh ? 1 : 0], q[0], sh);
                } else {
                    uint32_t e[4];
                    _Pragma("unroll") for (int j = 0; j < 4; ++j) e[j] = row[min(max(x + j, 0), W - 1)];
                    v[k] = e[0] | (e[1] << 8) | (e[2] << 16) | (e[3] << 24);
                }
            }
            _Pragma("unroll") for (int k = 0; k < kBatch; ++k)
            {
                const int it = (k0 + k) * kDetThreads + tid;
                if (it < n) reinterpret_cast<uint32_t *>(px)[it] = v[k];
            }
        }
    }
    __syncthreads();
    const int G = (W + 3) >> 2;            // four-pixel groups of a row
    const float inv_g = 1.0f / (float)G;
    for (int it = tid; it < (rows + 2) * G; it += kDetThreads) {
        const int r = div_items(it, inv_g), x = 4 * (it - r * G);
        const int yy = y0 - 1 + r;
        uint32_t s4 = 0;
        if (yy >= E && yy < H - E && x + 3 >= E && x < W - E) {
            s4 = fast_scores(px + r * S, S, x, (uint32_t)a.t);
            // pixels of the window only
            _Pragma("unroll") for (int j = 0; j < 4; ++j)
                if (x + j < E || x + j >= W - E) s4 &= ~(0xFFu << (8 * j));
        }
        *reinterpret_cast<uint32_t *>(sc + r * S + 4 + x) = s4;
    }
    __syncthreads();
    // strict suppression (a group's window pixels lie >= 19 from every border,
    // so what the band's row ends hold never matters); the kept corners of
    // round k of this thread as four bits and the counts of every wave
    uint32_t kept[kItems], cen[kItems];
    const uint64_t below = (1ull << lane) - 1ull;
    int rank[kItems];
    _Pragma("unroll") for (int k = 0; k < kItems; ++k)
    {
        kept[k] = cen[k] = 0;
        rank[k] = 0;
        if (k * kDetThreads >= rows * G) continue;   // (uniform)
        const int it = k * kDetThreads + tid;
        if (it < rows * G) {
            const int r = div_items(it, inv_g), x = 4 * (it - r * G);
            uint32_t w[3][3];
            _Pragma("unroll") for (int d = 0; d < 3; ++d) row_window(sc + (r + d) * S, x, w[d]);
            cen[k] = w[1][1];
            _Pragma("unroll") for (int h = 0; h < 2; ++h)
            {
                u16x2 m = byte_pair(w[1], 3 + 2 * h);
                m = __builtin_elementwise_max(m, byte_pair(w[1], 5 + 2 * h));
                _Pragma("unroll") for (int d = 0; d < 3; d += 2)
                    _Pragma("unroll") for (int j = 3; j < 6; ++j) m = __builtin_elementwise_max(m, byte_pair(w[d], j + 2 * h));
                const u16x2 over = __builtin_elementwise_sub_sat(byte_pair(w[1], 4 + 2 * h), m);
                kept[k] |= (over[0] ? 1u : 0u) << (2 * h) | (over[1] ? 2u : 0u) << (2 * h);
            }
        }
        const int cnt = __popc(kept[k]);             // 0, 1 or 2 (no two neighbours)
        const uint64_t m1 = __ballot(cnt & 1), m2 = __ballot(cnt & 2);
        rank[k] = __popcll(m1 & below) + 2 * __popcll(m2 & below);
        if (lane == 0) wave_n[k * kDetWaves + wave] = __popcll(m1) + 2 * __popcll(m2);
    }
    __syncthreads();
    int n;
    {
        int v = lane < kItems * kDetWaves ? wave_n[lane] : 0;
        v = wave_scan(v);
        n = __builtin_amdgcn_readlane(v, 63);
        _Pragma("unroll") for (int k = 0; k < kItems; ++k)
        {
            const int j = k * kDetWaves + __builtin_amdgcn_readfirstlane(wave);
            rank[k] += j ? __builtin_amdgcn_readlane(v, (j - 1) & 63) : 0;
        }
    }
    // the tile's count, before anything that does not depend on the others
    const unsigned long long ep = (unsigned long long)a.epoch << 32;
    if (tid == 0)
        __hip_atomic_store(&a.tile_state[tile], ep | kPublished | (unsigned long long)n, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    // the tile's corners in (row, column) order: column | row << 11 | score << 14
    _Pragma("unroll") for (int k = 0; k < kItems; ++k)
    {
        if (k * kDetThreads >= rows * G) continue;
        const int it = k * kDetThreads + tid;
        const int r = div_items(it, inv_g), x = 4 * (it - r * G);
        int at = rank[k];
        _Pragma("unroll") for (int j = 0; j < 4; ++j)
            if ((kept[k] >> j) & 1u)
                tc[at++] = (uint32_t)(x + j) | ((uint32_t)r << 11) | (((cen[k] >> (8 * j)) & 0xFFu) << 14);
    }
    if (a.blurred) {
        // Smoothing, four columns by two rows per item: horizontal sums of the
        // eight staged rows by byte dot products, then the vertical taps.
        FT_G uint8_t *dst = a.blurred + a.off[l];
        const int pairs = (rows + 1) >> 1;
        for (int it = tid; it < pairs * G; it += kDetThreads) {
            const int rp = div_items(it, inv_g), x = 4 * (it - rp * G), r0 = 2 * rp;
            uint32_t hs[8][4];
            _Pragma("unroll") for (int k = 0; k < 8; ++k)
            {
                uint32_t w[3];
                row_window(px + (r0 + k + 1) * S, x, w);
                _Pragma("unroll") for (int j = 0; j < 4; ++j)
                {
                    // bytes x + j - 3 .. x + j and x + j + 1 .. x + j + 4
                    const uint32_t p = j < 3 ? __builtin_amdgcn_alignbyte(w[1], w[0], 1 + j) : w[1];
                    const uint32_t q = j < 3 ? __builtin_amdgcn_alignbyte(w[2], w[1], 1 + j) : w[2];
                    hs[k][j] = __builtin_amdgcn_udot4(p, 0x140F0601u, __builtin_amdgcn_udot4(q, 0x0001060Fu, 0u, false), false);
                }
            }
            _Pragma("unroll") for (int r = 0; r < 2; ++r)
            {
                if (r0 + r >= rows) break;
                uint32_t o[4];
                _Pragma("unroll") for (int j = 0; j < 4; ++j)
                    o[j] = (hs[r][j] + hs[r + 6][j] + 6u * (hs[r + 1][j] + hs[r + 5][j]) + 15u * (hs[r + 2][j] + hs[r + 4][j]) +
                            20u * hs[r + 3][j] + 2048u) >> 12;
                const uint32_t v = o[0] | (o[1] << 8) | (o[2] << 16) | (o[3] << 24);
                FT_G uint8_t *d = dst + (int64_t)(y0 + r0 + r) * W + x;
                if (x + 4 <= W) {
                    *reinterpret_cast<FT_G u32_any *>(d) = v;
                } else {
                    _Pragma("unroll") for (int j = 0; j < 3; ++j) if (x + j < W) d[j] = (uint8_t)(v >> (8 * j));
                }
            }
        }
    }
    // Look-back: the counts of every lower tile, one per thread and round (each
    // state is one self-contained 64-bit word, so no other ordering is needed).
    int prefix = 0;
    for (int k = tid; k < tile; k += kDetThreads) {
        unsigned long long v;
        int spins = 0;
        do
            v = __hip_atomic_load(&a.tile_state[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        while (!((v >> 32) == a.epoch && (v & kPublished)) && ++spins <= kMaxSpins);
        prefix = min(prefix + (spins > kMaxSpins ? kPoison : (int)(v & kValueMask)), kPoison);
    }
    // (at most 2^29 + 2^29 per addition: clamped to the poison value before each)
    _Pragma("unroll") for (int o = 32; o > 0; o >>= 1) prefix = min(prefix + __shfl_xor(prefix, o), kPoison);
    if (lane == 0) wave_prefix[wave] = prefix;
    __syncthreads();
    int before = 0;
    _Pragma("unroll") for (int w = 0; w < kDetWaves; ++w) before = min(before + wave_prefix[w], kPoison);
    if (tid == 0 && tile == tiles - 1) a.count[0] = before >= kPoison ? -1 : before + n;
    const float sf = a.sf[l];
    for (int k = tid; k < n; k += kDetThreads) {
        const int i = before + k;
        if (i >= a.capacity) break;
        const uint32_t e = tc[k];
        const int x = (int)(e & 2047u), yy = y0 + (int)((e >> 11) & 7u);
        a.lx[i] = (int16_t)x;
        a.ly[i] = (int16_t)yy;
        a.oct[i] = (uint8_t)l;
        a.score[i] = (uint8_t)(e >> 14);
        a.x[i] = (float)x * sf;
        a.y[i] = (float)yy * sf;
    }
}

// The integer nearest num / sqrt(m2), halves away from zero, decided exactly:
// the largest k >= 0 with k = 0 or (2k - 1)^2 m2 <= 4 num^2, with num's sign;
// found from a binary64 estimate by exact integer corrections.
__device__ __forceinline__ int round_ratio_exact(int num, int64_t m2)
{
    const int64_t a = num < 0 ? -(int64_t)num : (int64_t)num;
    const int64_t a4 = 4 * a * a;
    int k = (int)floor((double)a / sqrt((double)m2) + 0.5);
    if (k < 0) k = 0;
    while (k > 0 && (int64_t)(2 * k - 1) * (2 * k - 1) * m2 > a4) --k;
    while ((int64_t)(2 * k + 1) * (2 * k + 1) * m2 <= a4) ++k;
    return num < 0 ? -k : k;
}

// Orders one wave's LDS accesses (its lanes read what other lanes wrote).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ float angle_deg(int m10, int m01)
{
    double ang = atan2((double)m01, (double)m10) * (180.0 / 3.14159265358979323846);
    if (ang < 0.0) ang += 360.0;
    return (float)ang;
}

constexpr int kDescSlots = 16;        // most keypoints of a wave (its workgroup's angles: one per lane of a wave)
constexpr int kDescWaves = kThreads / 64;
constexpr int kTurnR = 13;            // turned pattern points lie within radius 13
constexpr int kWinRows = 2 * kTurnR + 1, kWinStride = 32;   // the smoothed window in LDS
static_assert(kDescSlots * kDescWaves == 64 && kWinRows * 2 <= 64, "one lane per angle and per window half row");

// The disc dx^2 + dy^2 <= 225 over the lanes of a wave: lane = (row dy, half of
// the 29 columns -14 .. 14), 16 or 13 columns each, and the two pixels (-15, 0)
// and (15, 0) in lanes 62 and 63 (no other row reaches column 15).  Per lane the
// column weights dx and the 0 / 1 weights of its 16 bytes.
struct DiscWeights {
    uint32_t v[64][8];
    constexpr DiscWeights() : v{}
    {
        for (int lane = 0; lane < 62; ++lane) {
            const int dy = (lane >> 1) - 15;
            for (int c = 0; c < 16; ++c) {
                const int dx = (lane & 1 ? 2 : -14) + c;
                if (dx > 14 || dx * dx + dy * dy > 225) continue;
                v[lane][c >> 2] |= ((uint32_t)dx & 0xFFu) << (8 * (c & 3));
                v[lane][4 + (c >> 2)] |= 1u << (8 * (c & 3));
            }
        }
        v[62][0] = (uint32_t)-15 & 0xFFu;
        v[63][0] = 15u;
    }
};
__constant__ const DiscWeights kDisc;

// One wave per keypoint.  Both windows are read as aligned dwordx4 (misaligned
// vector loads take one lane per cycle) and realigned in registers, a half
// row's last bytes coming from the other half's lane:
//  * the disc: moments by byte dot products with the lane's column weights
//    (signed, on pixel - 128: the weights of a row of the disc cancel) and 0 / 1
//    weights;
//  * the 27 smoothed rows that turned points can reach, staged in LDS, where the
//    tests' 512 pixels per keypoint are gathered.
// The next keypoint's loads are issued before the current one's arithmetic.
// What bounds it is vector issue (about 240 instructions per keypoint against 600
// one byte load per disc pixel and one gather from memory per test point: 76 ->
// 36 us at 47,700 keypoints), then the window rows' trips through L1.
__global__ __launch_bounds__(kThreads, 4) void k_orb_describe(OrbDescribeArgs a)
{
    __shared__ __align__(16) unsigned char win[kDescWaves * 64 * 16];
    __shared__ float4 pattern[kOrbTests];
    __shared__ int list_i[64], list_m10[64], list_m01[64];
    static_assert(kOrbTests == kThreads, "a test per thread");
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wave = (int)blockIdx.x * kDescWaves + w;
    const int waves = (int)gridDim.x * kDescWaves;
    int n = a.n_max;
    if (a.count) {
        const int c = a.count[0];
        n = c < n ? c : n;
    }
    if ((int)blockIdx.x * kDescWaves >= n) return;
    // slot s is keypoint s * waves + wave; lane s reads its record
    const int mine = (lane & (kDescSlots - 1)) * waves + wave;
    const int rec = min(mine, n - 1);
    const int l = a.oct[rec], u = a.lx[rec], v = a.ly[rec];
    // the tests' points
    {
        const int t = (int)threadIdx.x;
        pattern[t] = make_float4((float)a.pattern[t][0], (float)a.pattern[t][1], (float)a.pattern[t][2], (float)a.pattern[t][3]);
        __syncthreads();
    }
    uint32_t wdx[4], wone[4];
    _Pragma("unroll") for (int i = 0; i < 4; ++i)
    {
        wdx[i] = kDisc.v[lane][i];
        wone[i] = kDisc.v[lane][4 + i];
    }
    const int half = lane & 1;
    const bool tip = lane >= 62;
    const int drow = tip ? 15 : lane >> 1, dcol = lane == 62 ? 0 : lane == 63 ? 30 : 1;   // from (-15, -15)
    const int dy = drow - 15;
    const uint32_t dhalf = tip ? 0u : 16u * (uint32_t)half;
    const int wrow = min(lane >> 1, kWinRows - 1);   // window row of this lane
    struct Pre {
        v4u d, b;
        uint32_t sh_d, sh_b;
    };
    // Slot records, one per lane: the level's width (0: the keypoint
    // is closer than 15 pixels to its level's border, or has no level) and the
    // keypoint's byte offset in the pyramid.
    int m_w, m_lo, m_hi;
    {
        int W = a.w[0], H = a.h[0];
        int64_t off = a.off[0];
        _Pragma("unroll") for (int k = 1; k < kLevels; ++k)
        {
            W = l == k ? a.w[k] : W;
            H = l == k ? a.h[k] : H;
            off = l == k ? a.off[k] : off;
        }
        const bool ok = l < kLevels && u >= 15 && v >= 15 && u < W - 15 && v < H - 15;
        const int64_t at = off + (int64_t)v * W + u;
        m_w = ok ? W : 0;
        m_lo = (int)(uint32_t)at;
        m_hi = (int)(at >> 32);
    }
    auto fetch = [&](int s) {
        Pre p{};
        const int W = __builtin_amdgcn_readlane(m_w, s);
        if (W) {
            const int64_t at = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(m_hi, s) << 32) |
                                         (uint32_t)__builtin_amdgcn_readlane(m_lo, s));
            // Every dword read holds a byte of the keypoint's 31 x 31 square, but
            // for the last three of lane 63's (15, 0), which lie in rows below.
            const FT_G uint8_t *img = a.pyr + at - 15 * (int64_t)W - 15;
            const uint32_t si = (uint32_t)reinterpret_cast<uintptr_t>(img) & 3u;
            const uint32_t od = (uint32_t)(drow * W + dcol) + si;
            p.sh_d = od & 3u;
            p.d = *reinterpret_cast<const FT_G v4u_dw *>(img - si + ((od & ~3u) + dhalf));
            const FT_G uint8_t *B = a.blurred + at - kTurnR * (int64_t)W - kTurnR;
            const uint32_t sb = (uint32_t)reinterpret_cast<uintptr_t>(B) & 3u;
            const uint32_t ob = (uint32_t)(wrow * W) + sb;
            p.sh_b = ob & 3u;
            p.b = *reinterpret_cast<const FT_G v4u_dw *>(B - sb + ((ob & ~3u) + 16u * (uint32_t)half));
        }
        return p;
    };
    // e[k]: bytes 4 k .. 4 k + 3 of the lane's 16, from the pixel at shift sh
    auto realign = [](const v4u &d, uint32_t sh, uint32_t e[4]) {
        const uint32_t over = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d[0], 0xF5, 0xF, 0xF, false);   // quad_perm 1,1,3,3
        _Pragma("unroll") for (int k = 0; k < 4; ++k) e[k] = __builtin_amdgcn_alignbyte(k < 3 ? d[k + 1] : over, d[k], sh);
    };
    unsigned char *wl = win + 64 * 16 * w;
    const float mid = (float)(64 * 16 * w + kTurnR * kWinStride + kTurnR);   // the keypoint's byte in `win`
    if (lane < kDescSlots) list_i[w * kDescSlots + lane] = mine < n ? mine : -1;
    const int slots = n - wave <= 0 ? 0 : min(kDescSlots, (n - wave + waves - 1) / waves);
    Pre cur{};
    if (slots > 0) cur = fetch(0);
    for (int s = 0; s < slots; ++s) {
        const int i = s * waves + wave;
        Pre nxt{};
        if (s + 1 < slots) nxt = fetch(s + 1);
        const bool ok = __builtin_amdgcn_readlane(m_w, s) != 0;
        FT_G uint8_t *d = a.desc + 32 * (int64_t)i;
        if (!ok) {   // outside the window the disc and the turned pattern need
            if (lane < 8) reinterpret_cast<FT_G uint32_t *>(d)[lane] = 0u;
            if (lane == 0) list_m10[w * kDescSlots + s] = INT_MIN;
            cur = nxt;
            continue;
        }
        // moments (exact integers, |m| <= 577,320)
        int m10 = 0;
        uint32_t row_sum = 0, e[4];
        realign(cur.d, cur.sh_d, e);
        _Pragma("unroll") for (int k = 0; k < 4; ++k)
        {
            m10 = __builtin_amdgcn_sdot4((int)(e[k] ^ 0x80808080u), (int)wdx[k], m10, false);
            row_sum = __builtin_amdgcn_udot4(e[k], wone[k], row_sum, false);
        }
        int m01 = dy * (int)row_sum;
        m10 = wave_sum(m10);
        m01 = wave_sum(m01);
        if (lane == 0) {
            list_m10[w * kDescSlots + s] = m10;
            list_m01[w * kDescSlots + s] = m01;
        }
        // the smoothed window: row wrow at byte 32 wrow of the wave's LDS
        realign(cur.b, cur.sh_b, e);
        *reinterpret_cast<v4u *>(wl + 16 * lane) = v4u{e[0], e[1], e[2], e[3]};
        wave_lds_sync();
        // per test: the two turned points, then their smoothed pixels.  A
        // turned coordinate is (x m10 - y m01) / |m| or (x m01 + y m10) / |m|, at
        // most 13 in size; in binary32 from the direction (m10, m01) / |m| (half a
        // unit for each square, their sum, both products and the two terms, one
        // for the reciprocal root) it is off by less than 4.5e-6, so unless it
        // lies within 1e-5 of a half it rounds to the exact integer, and else is
        // decided in integers.  m = 0: no turn.
        const bool turned = (m10 | m01) != 0;
        const float f10 = (float)m10, f01 = (float)m01;   // exact: |m| < 2^24
        const float inv_r = turned ? rsqrtf(f10 * f10 + f01 * f01) : 0.0f;
        const float cs = turned ? f10 * inv_r : 1.0f, sn = f01 * inv_r;
        int p1[4], p2[4];    // bytes of the test's points in `win`
        float far[4];        // largest distance of a turned coordinate from its integer
        auto place = [&](float c, float r) { return (int)fmaf(r, (float)kWinStride, c + mid); };
        _Pragma("unroll") for (int q = 0; q < 4; ++q)
        {
            const float4 t = pattern[64 * q + lane];
            far[q] = 0.0f;
            auto turn = [&](float x) {
                const float r = __builtin_rintf(x);
                far[q] = fmaxf(far[q], fabsf(x - r));
                return r;
            };
            const float c1 = turn(fmaf(-t.y, sn, t.x * cs)), r1 = turn(fmaf(t.y, cs, t.x * sn));
            const float c2 = turn(fmaf(-t.w, sn, t.z * cs)), r2 = turn(fmaf(t.w, cs, t.z * sn));
            p1[q] = place(c1, r1);
            p2[q] = place(c2, r2);
        }
        constexpr float kNear = 0.5f - 1e-5f;
        if (!(fmaxf(fmaxf(far[0], far[1]), fmaxf(far[2], far[3])) < kNear)) {
            // (the moments made opaque here, so that nothing of this rare path is
            // computed outside it)
            int a10 = turned ? m10 : 1, a01 = m01;
            asm volatile("" : "+v"(a10), "+v"(a01));
            const int64_t m2 = (int64_t)a10 * a10 + (int64_t)a01 * a01;
            _Pragma("unroll 1") for (int q = 0; q < 4; ++q)
            {
                const float f = q == 0 ? far[0] : q == 1 ? far[1] : q == 2 ? far[2] : far[3];
                if (f < kNear) continue;
                const float4 t = pattern[64 * q + lane];
                int at[2];
                _Pragma("unroll 1") for (int k = 0; k < 2; ++k)
                {
                    const int x = (int)(k ? t.z : t.x), y = (int)(k ? t.w : t.y);
                    const int v = place((float)round_ratio_exact(x * a10 - y * a01, m2),
                                        (float)round_ratio_exact(x * a01 + y * a10, m2));
                    at[0] = k ? at[0] : v;
                    at[1] = v;
                }
                _Pragma("unroll") for (int j = 0; j < 4; ++j)
                {
                    p1[j] = q == j ? at[0] : p1[j];
                    p2[j] = q == j ? at[1] : p2[j];
                }
            }
        }
        uint64_t bits = 0;   // lane q: tests 64 q .. 64 q + 63
        uint32_t g1[4], g2[4];
        _Pragma("unroll") for (int q = 0; q < 4; ++q)
        {
            g1[q] = win[p1[q]];
            g2[q] = win[p2[q]];
        }
        _Pragma("unroll") for (int q = 0; q < 4; ++q)
        {
            const uint64_t m = __ballot(g1[q] < g2[q]);
            bits = lane == q ? m : bits;
        }
        wave_lds_sync();   // the window is free for the next keypoint
        if (lane < 4) reinterpret_cast<FT_G uint64_t *>(d)[lane] = bits;
        cur = nxt;
    }
    // the workgroup's angles, one per lane of one wave
    __syncthreads();
    if (w == 0) {
        const int i = list_i[lane], m10 = list_m10[lane], m01 = list_m01[lane];
        if (i >= 0) a.angle[i] = m10 == INT_MIN ? -1.0f : angle_deg(m10, m01);
    }
}

}  // namespace

size_t orb_detect_lds(int lds_w)
{
    // staged rows, scores, and the tile's kept corners: strict suppression never
    // keeps two 8-neighbours, so at most (kOrbRows / 2) x ceil(W / 2) of them
    return (size_t)(kStaged + kScoreRows) * (size_t)row_stride(lds_w) + 4 * (size_t)(kOrbRows / 2) * (size_t)(lds_w / 2);
}

hipError_t launch_orb_detect(const OrbDetectArgs &a, hipStream_t s)
{
    const int tiles = a.tile0[kLevels];
    if (tiles <= 0) return hipSuccess;
    const size_t lds = orb_detect_lds(a.lds_w);
    hipLaunchKernelGGL(k_orb_detect, dim3(tiles), dim3(kDetThreads), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_orb_describe(const OrbDescribeArgs &a, hipStream_t s)
{
    if (a.n_max <= 0) return hipSuccess;
    // One wave per keypoint up to four waves per SIMD of the chip's 256 CUs, then
    // up to kDescSlots keypoints per wave (so a wave's set-up and its share of
    // the binary64 angles are paid less often), then more workgroups.
    const int most = kDescWaves * kDescSlots;
    int blocks = (a.n_max + kDescWaves - 1) / kDescWaves;
    blocks = std::max(std::min(blocks, 1024), (a.n_max - 1) / most + 1);
    hipLaunchKernelGGL(k_orb_describe, dim3(blocks), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace ft
