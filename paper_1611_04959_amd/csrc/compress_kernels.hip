// compress_kernels.hip -- gfx950 kernels of libdaqisland: lossless
// compression of the chopped islands.
//
// Section 3: the frontend compresses the chopped data losslessly before the
// event builder (the algorithm is not named). The format is the one stated in
// include/daq.h: each channel's packed row of L samples in blocks of 64; per
// block a header word (first sample, bit width w) and the zigzag-coded
// differences of consecutive samples as a little-endian bit stream of w bits
// each, the blocks' payloads back to back.
//
// A wave takes groups of 8 consecutive blocks of one row: lane l holds the 8
// samples 8 l .. 8 l + 7 of a group (one 16-byte load), so block j of the
// group is lanes 8 j .. 8 j + 7. The launch's work-groups are shared out to the
// fills by their groups, and a fill's groups cut into one contiguous range per
// wave. Two kernels:
// the size pass writes the block headers and the payload words of each wave and
// work-group; the pack pass starts each wave at the sum of the sizes before it,
// walks its groups in order, ORs each lane's codes into the group's payload
// in LDS (all eight as one or two 64-bit values, three atomics each) and stores
// the payload with coalesced writes. Every wave touches only its own LDS, so
// there are no work-group barriers but the one behind the size pass's sums.
//
// These kernels are bound by the vector instructions a sample takes and by
// each wave's chain of loads. So codes are computed two at a time in 16-bit
// halves wherever the differences fit them (widths up to 16: always, for the
// digitizers' 12-bit samples; rows' ends and wider blocks take the general
// path, one 32-bit code at a time), and the next groups' loads are in flight
// while one is worked on, at clamped indices rather than behind branches.
// 16 fills of 54 rows of 11,000 to 61,000 samples (31 M samples, 62 MB, 21 MB
// of payload): size pass 16.6 -> 14.5 us (4.3 TB/s), pack pass 32.7 -> 22.3 us
// (4.0 TB/s), decoding 35.3 -> 22.8 us a call (3.7 TB/s).
#include "chop_internal.h"

namespace daqk {
namespace {

constexpr int kZBlock = 64;     // samples per block
constexpr int kZGroup = 8;      // blocks per wave
constexpr int kZMaxWords = 34;  // ceil(63 * 17 / 32): the widest block's payload
constexpr int kZGroupWords = kZGroup * kZMaxWords;
// Groups a wave loads before it uses them, in the size and the pack pass.
#ifndef DAQ_Z_UNROLL
#define DAQ_Z_UNROLL 4
#endif
#ifndef DAQ_Z_PACK_UNROLL
#define DAQ_Z_PACK_UNROLL 1
#endif
constexpr int kZUnroll = DAQ_Z_UNROLL;
constexpr int kZPackUnroll = DAQ_Z_PACK_UNROLL;
constexpr int kZSums = 2;
// LDS words of a group's payload: a spare word in front (a block's first lane
// starts its codes one width early, with zeros) and three behind.
constexpr int kZLdsWords = kZGroupWords + 4;

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ s16x2 as_s(uint32_t v) { return __builtin_bit_cast(s16x2, v); }
__device__ __forceinline__ u16x2 as_u(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
template <class T>
__device__ __forceinline__ uint32_t as_word(T v) {
    return __builtin_bit_cast(uint32_t, v);
}

// Rows of L samples (at most DAQ_MAX_SAMPLES) in blocks and groups.
struct ZGeom {
    int32_t L;    // samples per row
    int32_t nb;   // blocks per row
    int32_t gpr;  // groups per row
};
__device__ __forceinline__ ZGeom z_geom_of(int64_t L) {
    ZGeom g;
    g.L = (int32_t)L;
    g.nb = (int32_t)((L + kZBlock - 1) / kZBlock);
    g.gpr = (g.nb + kZGroup - 1) / kZGroup;
    return g;
}

// A DPP lane move, zero where a lane has no source. The empty asm keeps it
// apart from the arithmetic that uses it (a row shift folded into a reverse
// subtract gave wrong differences on gfx950).
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
    int r = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
    asm("" : "+v"(r));
    return (uint32_t)r;
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int64_t dpp_or_zero64(int64_t v) {
    return (int64_t)(((uint64_t)dpp_or_zero<CTRL, ROWS>((uint32_t)((uint64_t)v >> 32)) << 32) |
                     dpp_or_zero<CTRL, ROWS>((uint32_t)v));
}

__device__ __forceinline__ int64_t lane_i64(int64_t v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The sum over the wave's lanes, in every lane.
__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
    v += dpp_or_zero64<0x111>(v);       // the lanes 1, 2, 4, 8 below, within rows of 16
    v += dpp_or_zero64<0x112>(v);
    v += dpp_or_zero64<0x114>(v);
    v += dpp_or_zero64<0x118>(v);
    v += dpp_or_zero64<0x142, 0xA>(v);  // the last lane of the row before
    v += dpp_or_zero64<0x143, 0xC>(v);  // the last lane of the first half
    return lane_i64(v, 63);
}

// a / b of wave-uniform non-negative values: 32-bit where they fit, which
// takes a fifth of the instructions.
__device__ __forceinline__ int64_t udiv(int64_t a, int64_t b) {
    if ((((uint64_t)a | (uint64_t)b) >> 32) == 0) return (int64_t)((uint32_t)a / (uint32_t)b);
    return a / b;
}

// A wave's contiguous range of a fill's groups, and where it starts.
struct ZRange {
    int64_t lo, hi;
    int32_t c, gr;  // row and group in the row of group lo
};
__device__ __forceinline__ ZRange z_range(int64_t groups, int32_t gpr, int v, int W) {
    ZRange r;
    const int64_t each = udiv(groups, W);
    const int more = (int)(groups - each * W);  // the first `more` waves take one more
    r.lo = each * v + (v < more ? v : more);
    r.hi = r.lo + each + (v < more ? 1 : 0);
    r.c = gpr ? (int32_t)udiv(r.lo, gpr) : 0;
    r.gr = (int32_t)(r.lo - (int64_t)r.c * gpr);
    return r;
}

// A wave's part of a compression launch: its fill, its number in the launch
// and that of its fill's first wave, whether it has the fill's last group (or is
// the first wave of a fill without any).
struct ZPart {
    int fill;
    bool last;
    ZGeom g;
    ZRange r;
    int wave0, wave;
};

// The shares of the launch's work-groups: fill j gets one, and its part by
// groups of the rest. The fills' lengths are on the device, so every wave works
// this out: lane j for fill j, then the fill whose work-groups include this
// one. (With equal shares the waves of 16 fills of 11,000 to 61,000 samples a
// row had between a fifth and all of the longest one's work; in the scalar unit,
// fill by fill, this took 10 us of the kernel.) False for a work-group that the
// rounding left over.
__device__ __forceinline__ bool z_part(const ZArgs &a, ZPart *p) {
    const int lane = threadIdx.x & 63;
    const int wl = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t L = 0, groups = 0;
    if (lane < a.n) {
        const ZFillDev &f = a.f[lane];
        const int64_t tl = f.counts->total_len;
        L = tl < f.max_len ? (tl > 0 ? tl : 0) : f.max_len;
        groups = (int64_t)z_geom_of(L).gpr * f.C;
    }
    const int64_t all = wave_sum_i64(groups);
    // 1 + floor(groups * spare / all), rounded down further, in 32 bits: all of
    // them together never exceed the launch
    const uint32_t spare = gridDim.x - (uint32_t)a.n;
    const int bits = 64 - __clzll(all | 1);
    const int sh = bits > 20 ? bits - 20 : 0;
    const uint32_t recip = 0xFFFFFFFFu / (uint32_t)((all >> sh) + 1);
    const int mine = lane < a.n ? 1 + (int)__umulhi((uint32_t)(groups >> sh) * spare, recip) : 0;
    uint32_t end = (uint32_t)mine;  // work-groups of the fills up to lane's
    end += dpp_or_zero<0x111>(end);
    end += dpp_or_zero<0x112>(end);
    end += dpp_or_zero<0x114>(end);
    end += dpp_or_zero<0x118>(end);
    const uint64_t after = __ballot(lane < a.n && blockIdx.x < end);
    if (after == 0) return false;
    const int j = __ffsll((unsigned long long)after) - 1;
    const int wgs = __builtin_amdgcn_readlane(mine, j);
    const int wg0 = __builtin_amdgcn_readlane((int)end, j) - wgs;
    p->g = z_geom_of(lane_i64(L, j));
    const int v = ((int)blockIdx.x - wg0) * kZWaves + wl, W = wgs * kZWaves;
    p->r = z_range(lane_i64(groups, j), p->g.gpr, v, W);
    p->fill = j;
    p->last = p->r.hi == lane_i64(groups, j) && (p->r.lo < p->r.hi || v == 0);
    p->wave0 = wg0 * kZWaves;
    p->wave = p->wave0 + v;
    return true;
}

// Where a group sits: its row and its index in the row (wave-uniform).
struct ZAt {
    int32_t c, gr;
};

// The lane's 8 samples of the group at `at` (past the row's end: samples that
// are not used; the load has no branch around it so that several can be in
// flight). L >= 1.
__device__ __forceinline__ int4 z_load(const ZFillDev &f, const ZGeom &g, ZAt at, int lane) {
    uint32_t t = (uint32_t)lane * kVec;
    const uint32_t last = ((uint32_t)g.L - 1) / kVec * kVec - (uint32_t)at.gr * (kZGroup * kZBlock);
    t = t < last ? t : last;
    const int16_t *row = f.packed + (int64_t)at.c * f.stride + (int64_t)at.gr * (kZGroup * kZBlock);
    return *reinterpret_cast<const int4 *>(row + t);
}

// The block in the group that lane's samples belong to, or the row's last one.
__device__ __forceinline__ int z_block_at(const ZGeom &g, int32_t gr, int lane) {
    const int last = g.nb - 1 - gr * kZGroup;
    return (lane >> 3) < last ? lane >> 3 : last;
}

// The next group, or the same one again where there is none.
__device__ __forceinline__ ZAt z_next(const ZGeom &g, ZAt at, bool more) {
    ZAt n = at;
    if (more && ++n.gr == g.gpr) {
        n.gr = 0;
        n.c++;
    }
    return n;
}

// Whether every block of the group holds 64 samples.
__device__ __forceinline__ bool z_full(const ZGeom &g, ZAt at) {
    return (int64_t)(at.gr + 1) * (kZGroup * kZBlock) <= g.L;
}

// Lane-to-lane moves within rows of 16 lanes (DPP): the value of lane l - 1
// (lanes 16 k keep their own), and an OR over the 8 lanes of a block. The
// moves keep the lane's own value as the fallback, which stops the compiler
// from folding them into the arithmetic that uses them: a row shift folded
// into a reverse subtract gave wrong differences on gfx950.
__device__ __forceinline__ int32_t dpp_prev(int32_t v) { return __builtin_amdgcn_update_dpp(v, v, 0x111, 0xF, 0xF, false); }
__device__ __forceinline__ uint32_t or8(uint32_t m) {
    m |= (uint32_t)__builtin_amdgcn_update_dpp((int)m, (int)m, 0xB1, 0xF, 0xF, false);   // lanes 1 0 3 2
    m |= (uint32_t)__builtin_amdgcn_update_dpp((int)m, (int)m, 0x4E, 0xF, 0xF, false);   // lanes 2 3 0 1
    m |= (uint32_t)__builtin_amdgcn_update_dpp((int)m, (int)m, 0x141, 0xF, 0xF, false);  // 7 - i within 8
    return m;
}

// Samples in the lane's block (lane >> 3 of the group at `at`): 0 past the row.
__device__ __forceinline__ int z_block_len(const ZGeom &g, ZAt at, int lane) {
    const int64_t left = g.L - ((int64_t)at.gr * kZGroup + (lane >> 3)) * kZBlock;
    return left <= 0 ? 0 : (left < kZBlock ? (int)left : kZBlock);
}

__device__ __forceinline__ uint32_t zigzag(int32_t r) { return ((uint32_t)r << 1) ^ (uint32_t)(r >> 31); }

// Zigzag codes of the lane's 8 samples, sample i = 8 sub + e of its block of
// n samples; 0 where there is no code (i = 0 or i >= n).
__device__ __forceinline__ void z_codes(int4 q, int sub, int n, uint32_t z[kVec]) {
    const int16_t *h = reinterpret_cast<const int16_t *>(&q);
    int32_t s[kVec];
#pragma unroll
    for (int e = 0; e < kVec; e++) s[e] = h[e];
    // lanes 16 k have no previous lane in their DPP row: they start a block
    const int32_t prev = dpp_prev(s[kVec - 1]);
#pragma unroll
    for (int e = 0; e < kVec; e++) {
        const int i = sub * kVec + e;
        z[e] = (i >= 1 && i < n) ? zigzag(s[e] - (e ? s[e - 1] : prev)) : 0u;
    }
}

__device__ __forceinline__ uint32_t z_width(const uint32_t z[kVec]) {
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < kVec; e++) m |= z[e];
    m = or8(m);  // the bit length of the OR is that of the largest code
    return m ? 32u - (uint32_t)__clz(m) : 0u;
}

// The same for a full group whose differences fit int16, two codes to a word
// (sample 2 k of the lane in the low half of z[k]). `first`: 0xFFFF0000 on a
// block's first lane, which has no code for its first sample, else all ones.
__device__ __forceinline__ void z_codes2(int4 q, uint32_t first, uint32_t z[kVec / 2]) {
    const uint32_t w[4] = {(uint32_t)q.x, (uint32_t)q.y, (uint32_t)q.z, (uint32_t)q.w};
    uint32_t before = (uint32_t)dpp_prev((int32_t)w[3]);  // the pair before the lane's first
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const uint32_t prev = __builtin_amdgcn_alignbit(w[k], before, 16);
        const uint32_t d = as_word(as_u(w[k]) - as_u(prev)) & (k ? ~0u : first);
        z[k] = as_word(as_s(d) << (short)1) ^ as_word(as_s(d) >> (short)15);
        before = w[k];
    }
}

// Whether some sample of the lane lies outside [-16384, 16383], so that a
// difference might not fit int16.
__device__ __forceinline__ bool z_wide(int4 q) {
    const u16x2 h = {16384, 16384};
    const uint32_t t = as_word(as_u((uint32_t)q.x) + h) | as_word(as_u((uint32_t)q.y) + h) |
                       as_word(as_u((uint32_t)q.z) + h) | as_word(as_u((uint32_t)q.w) + h);
    return (t & 0x80008000u) != 0;
}

__device__ __forceinline__ uint32_t z_words(int n, uint32_t w) {
    return n > 0 ? ((uint32_t)(n - 1) * w + 31u) >> 5 : 0u;
}

__global__ void __launch_bounds__(kZWaves * 64) k_z_size(ZArgs a) {
    ZPart p;
    if (!z_part(a, &p)) return;
    const ZFillDev &f = a.f[p.fill];
    const ZGeom g = p.g;
    const int lane = threadIdx.x & 63, sub = lane & 7;
    const uint32_t first = sub ? ~0u : 0xFFFF0000u;
    ZAt at{p.r.c, p.r.gr};
    int64_t mine = 0;  // payload words of the lane's blocks (on each block's first lane)
    for (int64_t g0 = p.r.lo; g0 < p.r.hi; g0 += kZUnroll) {
        int4 q[kZUnroll];
        ZAt ats[kZUnroll];
#pragma unroll
        for (int u = 0; u < kZUnroll; u++) {
            ats[u] = at;
            q[u] = z_load(f, g, at, lane);
            at = z_next(g, at, g0 + u + 1 < p.r.hi);
        }
#pragma unroll
        for (int u = 0; u < kZUnroll; u++) {
            if (g0 + u >= p.r.hi) break;
            const bool full = z_full(g, ats[u]);
            int n = kZBlock;
            uint32_t w;
            if (full && __ballot(z_wide(q[u])) == 0) {
                uint32_t z[kVec / 2];
                z_codes2(q[u], first, z);
                uint32_t m = or8(z[0] | z[1] | z[2] | z[3]);
                m = (m | (m >> 16)) & 0xFFFFu;
                w = m ? 32u - (uint32_t)__clz(m) : 0u;
            } else {
                uint32_t z[kVec];
                if (!full) n = z_block_len(g, ats[u], lane);
                z_codes(q[u], sub, n, z);
                w = z_width(z);
            }
            if (sub == 0 && n > 0) {
                uint32_t *hdr = f.hdr + (int64_t)ats[u].c * g.nb + ats[u].gr * kZGroup;
                hdr[lane >> 3] = ((uint32_t)q[u].x & 0xFFFFu) | (w << 16);
                mine += z_words(n, w);
            }
        }
    }
    // the wave's payload words, and those of the work-group's waves together
    __shared__ int64_t s_tot[kZWaves];
    const int64_t tot = wave_sum_i64(mine);
    if (lane == 0) {
        a.gofs[gridDim.x + p.wave] = tot;
        s_tot[p.wave & (kZWaves - 1)] = tot;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t all = 0;
#pragma unroll
        for (int w = 0; w < kZWaves; w++) all += s_tot[w];
        a.gofs[blockIdx.x] = all;
    }
}

// Ordering of one wave's own LDS accesses (clear, OR, read back, clear).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ORs the 64-bit value v into the payload from bit `pos` on (pos >= -16).
__device__ __forceinline__ void z_or64(uint32_t *acc, int pos, uint64_t v) {
    const uint32_t r = (uint32_t)pos & 31u;
    const uint64_t low = v << r;
    const uint32_t high = ((uint32_t)(v >> 32) >> 1) >> (31u - r);
    uint32_t *at = acc + 1 + (pos >> 5);
    atomicOr(at, (uint32_t)low);
    atomicOr(at + 1, (uint32_t)(low >> 32));
    atomicOr(at + 2, high);
}

// The pack pass. Besides the loads and stores, a group costs its codes, three
// or six LDS atomics a lane (up to two per pair of codes when each pair was put
// in by itself) and one exchange per word, which also clears it.
__global__ void __launch_bounds__(kZWaves * 64) k_z_pack(ZArgs a) {
    __shared__ uint32_t s_words[kZWaves][kZLdsWords];
    ZPart p;
    if (!z_part(a, &p)) return;
    const ZFillDev &f = a.f[p.fill];
    const ZGeom g = p.g;
    const int lane = threadIdx.x & 63;
    if (p.r.lo >= p.r.hi) {  // an empty fill, or more waves than groups
        if (p.last && lane == 0) *f.n_words = 0;
        return;
    }
    const int sub = lane & 7, jb = lane >> 3;
    const uint32_t first = sub ? ~0u : 0xFFFF0000u;
    const int wl = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t *acc = s_words[wl];  // payload word k of the group in flight at acc[1 + k]; zero between groups
    for (int k = lane; k < kZLdsWords; k += 64) acc[k] = 0u;
    const int64_t lo = p.r.lo, hi = p.r.hi;
    // kZPackUnroll groups' samples and headers, loaded while the ones before
    // them are packed
    struct Batch {
        int4 q[kZPackUnroll];
        uint32_t hw[kZPackUnroll];
        ZAt at[kZPackUnroll];
    };
    ZAt next{p.r.c, p.r.gr};
    int64_t gn = lo;
    auto load = [&](Batch &b) {
#pragma unroll
        for (int u = 0; u < kZPackUnroll; u++) {
            b.at[u] = next;
            b.q[u] = z_load(f, g, next, lane);
            b.hw[u] = (f.hdr + (int64_t)next.c * g.nb + next.gr * kZGroup)[(uint32_t)z_block_at(g, next.gr, lane)];
            next = z_next(g, next, ++gn < hi);
        }
    };
    Batch b0, b1;
    load(b0);
    // where this wave's payload starts: the sizes of the fill's work-groups before
    // its own, kZSums of them per lane at a time, and of the waves before it in
    // that one. (A lone fill has up to 8,192 waves: with the sizes of all those
    // before it to add up, four loads in flight, the last ones had 32 rounds to
    // wait for; 54 x 20,000 samples took 25.6 us, 11.4 so. More loads at a time
    // gain up to 0.3 us there and cost 16 fills of 61,000 up to 0.7.)
    const int wg0 = p.wave0 / kZWaves, wg = (int)blockIdx.x;
    int64_t before = lane < (p.wave & (kZWaves - 1)) ? a.gofs[gridDim.x + wg * kZWaves + lane] : 0;
    for (int k0 = wg0; k0 < wg; k0 += 64 * kZSums) {
        int64_t v[kZSums];
#pragma unroll
        for (int u = 0; u < kZSums; u++) {
            const int k = k0 + 64 * u + lane;
            v[u] = k < wg ? a.gofs[k] : 0;
        }
#pragma unroll
        for (int u = 0; u < kZSums; u++) before += v[u];
    }
    int64_t carry = wave_sum_i64(before);
    auto pack = [&](const Batch &b, int64_t g0) {
#pragma unroll
        for (int u = 0; u < kZPackUnroll; u++) {
            if (g0 + u >= hi) break;
            const bool full = z_full(g, b.at[u]);
            const int n = full ? kZBlock : z_block_len(g, b.at[u], lane);
            const uint32_t w = b.hw[u] >> 16;
            const uint32_t nw = z_words(n, w);
            // the group's blocks' payload sizes: where the lane's block
            // starts, and the total (nw is the same in a block's 8 lanes)
            uint32_t upto = nw + dpp_or_zero<0x118>(nw);
            upto += dpp_or_zero<0x142, 0xA>(upto);
            upto += dpp_or_zero<0x143, 0xC>(upto);
            const uint32_t base = upto - nw;
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
            if (f.offsets && sub == 0 && n > 0)
                (f.offsets + (int64_t)b.at[u].c * g.nb + b.at[u].gr * kZGroup)[jb] = carry + base;
            // code i of the block sits at bit (i - 1) w of its payload
            if (full && __ballot(w > 16u) == 0) {
                uint32_t z[kVec / 2], pr[kVec / 2];
                z_codes2(b.q[u], first, z);
#pragma unroll
                for (int k = 0; k < 4; k++) pr[k] = (z[k] & 0xFFFFu) | ((z[k] >> 16) << w);
                const int pos = (int)(base * 32u) + (sub * kVec - 1) * (int)w;
                const uint64_t va = (uint64_t)pr[0] | ((uint64_t)pr[1] << (2 * w));
                const uint64_t vb = (uint64_t)pr[2] | ((uint64_t)pr[3] << (2 * w));
                if (__ballot(w > 8u) == 0) {
                    z_or64(acc, pos, va | (vb << (4 * w)));
                } else {
                    z_or64(acc, pos, va);
                    z_or64(acc, pos + 4 * (int)w, vb);
                }
            } else {
                uint32_t z[kVec];
                z_codes(b.q[u], sub, n, z);
#pragma unroll
                for (int e = 0; e < kVec; e++) {
                    if (z[e]) {
                        const uint32_t pos = base * 32u + (uint32_t)(sub * kVec + e - 1) * w;
                        const uint64_t val = (uint64_t)z[e] << (pos & 31u);
                        atomicOr(&acc[1 + (pos >> 5)], (uint32_t)val);
                        if ((uint32_t)(val >> 32)) atomicOr(&acc[2 + (pos >> 5)], (uint32_t)(val >> 32));
                    }
                }
            }
            wave_lds_order();
            const int64_t room = f.cap - carry;
            const uint32_t lim = room < (int64_t)total ? (uint32_t)(room < 0 ? 0 : room) : total;
            uint32_t *out = f.words + carry;
            for (uint32_t k = lane; k < total; k += 64) {
                const uint32_t x = atomicExch(&acc[1 + k], 0u);  // read, and cleared for the next group
                if (k < lim) out[k] = x;
            }
            wave_lds_order();
            carry += total;
        }
    };
    // (two batches per round, with their roles swapped: carried through a loop,
    // a batch's loads would be copied, and so waited for, in every turn)
    for (int64_t g0 = lo; g0 < hi;) {
        load(b1);
        pack(b0, g0);
        if ((g0 += kZPackUnroll) >= hi) break;
        load(b0);
        pack(b1, g0);
        g0 += kZPackUnroll;
    }
    if (p.last && lane == 0) *f.n_words = carry;
}

// ---- decompression ------------------------------------------------------------
//
// The same 8-block groups: a wave copies the group's payload words (contiguous
// in the stream) into its LDS, then lane l decodes the codes of samples
// 8 l .. 8 l + 7 of the group, undoes the zigzag, and adds the differences up: a
// prefix within the lane, then across the block's 8 lanes, plus the block's
// first sample. Words past n_words are read as zero, so a damaged stream cannot
// make the kernel read out of bounds. Samples are int16, so all sums are modulo
// 2^16: groups whose codes are at most 16 bits wide are decoded two samples to
// a word. ONE: every stream (blockIdx.y) has a wave for each of its groups. Else
// the streams share the work-groups out, and a wave takes a range of groups, the
// next one's loads in flight while one is decoded.

// 64 bits of the payload from bit `pos` on (pos >= -16; three words).
__device__ __forceinline__ uint64_t z_get64(const uint32_t *buf, int pos) {
    const uint32_t *at = buf + 1 + (pos >> 5);
    const uint32_t r = (uint32_t)pos & 31u;
    const uint32_t a = at[0], b = at[1], c = at[2];
    return ((uint64_t)__builtin_amdgcn_alignbit(c, b, r) << 32) | __builtin_amdgcn_alignbit(b, a, r);
}

// Eight decoded samples, stored non-temporally: left dirty in the L2 caches the
// rows are written back when the kernel ends (62 MB 23.2 us, with plain stores
// 29.6; 26 MB 14.4 and 15.7; 8.6 MB 7.1 and 7.6).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store16_out(int16_t *p, u32x4 v) {
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(p));
}

// Two codes of w <= 16 bits at the low end of v, to the halves of a word.
__device__ __forceinline__ uint32_t z_pair(uint32_t v, uint32_t w, uint32_t mask) {
    return (v & mask) | (((v >> w) & mask) << 16);
}

template <bool ONE>
__global__ void __launch_bounds__(kZWaves * 64) k_unz(ZDecArgs a) {
    // a lane's clamped start, the 34 words of its block and the spare words
    constexpr int kBuf = kZGroupWords + kZMaxWords + 8;
    __shared__ uint32_t s_words[kZWaves][kBuf];
    // the stream whose work-groups include this one (all bounds in one load)
    int si = 0, wg0 = 0, wg1 = 0;
    if constexpr (ONE) {
        si = blockIdx.y;
    } else {
        wg1 = a.wg0[1];
#pragma unroll
        for (int j = 1; j < kZMaxFills; j++) {
            const bool at_or_after = (int)blockIdx.x >= a.wg0[j];
            si = at_or_after ? j : si;
            wg0 = at_or_after ? a.wg0[j] : wg0;
            wg1 = at_or_after ? a.wg0[j + 1] : wg1;
        }
    }
    const ZStreamDev &f = a.f[si];
    const uint32_t lane = threadIdx.x & 63;
    const int sub = lane & 7;
    const uint32_t not_first = sub ? ~0u : 0xFFFF0000u;
    const int wl = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t *buf = s_words[wl];  // payload word k of the group at buf[1 + k]
    for (int k = lane; k < kBuf; k += 64) buf[k] = 0u;
    const ZGeom g = z_geom_of(f.L);
    const int v = ((int)blockIdx.x - wg0) * kZWaves + wl;
    ZRange r;
    if constexpr (ONE) {
        const int64_t groups = (int64_t)g.gpr * f.C;
        r.lo = v;
        r.hi = v < groups ? v + 1 : v;
        r.c = g.gpr ? (int32_t)udiv(v, g.gpr) : 0;
        r.gr = v - r.c * g.gpr;
    } else {
        r = z_range((int64_t)g.gpr * f.C, g.gpr, v, (wg1 - wg0) * kZWaves);
    }
    if (r.lo >= r.hi) return;
    // payload words are read at clamped indices, without branches around the
    // loads (a stream without words reads a header instead, and drops it)
    const uint32_t *words = f.n_words > 0 ? f.words : f.hdr;
    const int64_t most = f.n_words > 0 ? f.n_words - 1 : 0;
    // a group: its block headers and payload offsets (lane: block lane / 8),
    // then its payload, from its first block's offset to the end of its last
    // block, of which the first 128 words are loaded ahead
    struct Group {
        ZAt at;
        uint32_t hw;
        int64_t off;
        int64_t start;
        int span;
        uint32_t x0, x1;
    };
    ZAt next{r.c, r.gr};
    int64_t gn = r.lo;
    auto load_head = [&](Group &p) {
        p.at = next;
        const int64_t b = (int64_t)next.c * g.nb + next.gr * kZGroup;
        const uint32_t k = (uint32_t)z_block_at(g, next.gr, lane);
        p.hw = (f.hdr + b)[k];
        p.off = (f.offsets + b)[k];
        next = z_next(g, next, ++gn < r.hi);
    };
    auto load_payload = [&](Group &p) {
        uint32_t w = p.hw >> 16;
        w = w > 17u ? 17u : w;
        const uint32_t nw = z_words(z_full(g, p.at) ? kZBlock : z_block_len(g, p.at, lane), w);
        const int blocks = g.nb - p.at.gr * kZGroup;
        const int last = 8 * ((blocks < kZGroup ? blocks : kZGroup) - 1);
        p.start = lane_i64(p.off, 0);
        // (a damaged stream's offsets can be anything: unsigned, so that nothing overflows)
        const int64_t span = (int64_t)((uint64_t)lane_i64(p.off, last) + (uint64_t)__builtin_amdgcn_readlane((int)nw, last) -
                                       (uint64_t)p.start);
        p.span = (int)(span < 0 ? 0 : (span > kZGroupWords ? kZGroupWords : span));
        int64_t k0 = p.start < most ? p.start : most;
        k0 = k0 < 0 ? 0 : k0;
        const uint32_t most32 = (uint32_t)(most - k0 < 127 ? most - k0 : 127);
        p.x0 = (words + k0)[lane < most32 ? lane : most32];
        p.x1 = (words + k0)[lane + 64 < most32 ? lane + 64 : most32];
    };
    // p: the group in hand; q: the next one, whose payload is loaded while p is
    // decoded, as are the headers of the one after it (into p)
    auto turn = [&](Group &p, Group &q) {
        const uint32_t hw = p.hw;
        const ZAt at = p.at;
        const uint32_t rel = (uint32_t)p.off - (uint32_t)p.start;  // the block's first word (clamped below)
        const int span = p.span;
        if (p.start >= 0 && p.start <= f.n_words - span) {  // (no sum that could wrap)
            buf[1 + lane] = p.x0;
            buf[1 + 64 + lane] = p.x1;
            for (int k = (int)lane + 128; k < span; k += 64) buf[1 + k] = (words + p.start)[k];
        } else {  // a damaged stream: words outside it are zero
            for (int k = lane; k < span + 2; k += 64) {
                const int64_t i = (int64_t)((uint64_t)p.start + (uint64_t)k);
                buf[1 + k] = i >= 0 && i < f.n_words ? words[i] : 0u;
            }
        }
        if constexpr (!ONE) {
            load_payload(q);
            load_head(p);
        }
        wave_lds_order();
        uint32_t w = hw >> 16;
        w = w > 17u ? 17u : w;
        const int base = 32 * (int)(rel < (uint32_t)kZGroupWords ? rel : (uint32_t)kZGroupWords);
        int16_t *row = f.out + (int64_t)at.c * f.out_stride + (int64_t)at.gr * (kZGroup * kZBlock);
        if (z_full(g, at) && __ballot(w > 16u) == 0) {
            // every block of the group holds 64 samples, with codes of at most
            // 16 bits: the lane's 8 codes start one width before its second
            // sample's (the first lane of a block drops what it finds there)
            const uint32_t mask = (1u << w) - 1u;  // 0 for a constant block
            const int pos = base + (sub * kVec - 1) * (int)w;
            const uint64_t va = z_get64(buf, pos);
            uint64_t vb;
            if (__ballot(w > 8u) == 0) vb = va >> (4 * w);
            else vb = z_get64(buf, pos + 4 * (int)w);
            uint32_t d[4];
            d[0] = z_pair((uint32_t)va, w, mask) & not_first;
            d[1] = z_pair((uint32_t)(va >> (2 * w)), w, mask);
            d[2] = z_pair((uint32_t)vb, w, mask);
            d[3] = z_pair((uint32_t)(vb >> (2 * w)), w, mask);
            uint32_t run = 0;  // sum of the lane's differences so far, in both halves
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t half = as_word(as_u(d[k]) >> (unsigned short)1);
                const uint32_t sign = as_word(as_u(0u) - as_u(d[k] & 0x00010001u));
                const uint32_t x = half ^ sign;  // the two differences
                d[k] = as_word(as_u(as_word(as_u(x) + as_u(x << 16))) + as_u(run));
                run = __builtin_amdgcn_perm(d[k], d[k], 0x03020302u);  // the later one, twice
            }
            // exclusive prefix of the lanes' sums over the block's 8 lanes (a
            // row of 16 lanes holds two blocks), plus the block's first sample
            const uint32_t mine = run & 0xFFFFu;
            uint32_t inc = mine;
            uint32_t below = dpp_or_zero<0x111>(inc);  // (moved by every lane, used by some)
            inc += sub >= 1 ? below : 0u;
            below = dpp_or_zero<0x112>(inc);
            inc += sub >= 2 ? below : 0u;
            below = dpp_or_zero<0x114>(inc);
            inc += sub >= 4 ? below : 0u;
            const uint32_t before = (inc - mine + hw) & 0xFFFFu;
            const uint32_t both = before | (before << 16);
            u32x4 o;
            o.x = as_word(as_u(d[0]) + as_u(both));
            o.y = as_word(as_u(d[1]) + as_u(both));
            o.z = as_word(as_u(d[2]) + as_u(both));
            o.w = as_word(as_u(d[3]) + as_u(both));
            store16_out(row + lane * kVec, o);
        } else {
            const int n = z_block_len(g, at, lane);
            int32_t x[kVec];
            int32_t run = 0;
#pragma unroll
            for (int e = 0; e < kVec; e++) {
                const int i = sub * kVec + e;
                int32_t d = 0;
                if (i >= 1 && i < n && w > 0) {
                    const int pos = base + (i - 1) * (int)w;
                    const uint32_t z =
                        __builtin_amdgcn_alignbit(buf[2 + (pos >> 5)], buf[1 + (pos >> 5)], (uint32_t)pos & 31u) &
                        ((1u << w) - 1u);
                    d = (int32_t)(z >> 1) ^ -(int32_t)(z & 1u);
                }
                run += d;
                x[e] = run;
            }
            int32_t inc = run;
#pragma unroll
            for (int dd = 1; dd < 8; dd <<= 1) {
                const int32_t t = __shfl_up(inc, dd, 64);
                if (sub >= dd) inc += t;
            }
            const int32_t before = inc - run + (int32_t)(int16_t)(hw & 0xFFFFu);
            const int valid = n - sub * kVec;
            int16_t *to = row + lane * kVec;
            if (valid >= kVec) {
                uint4 o;
                o.x = (uint32_t)(uint16_t)(before + x[0]) | ((uint32_t)(uint16_t)(before + x[1]) << 16);
                o.y = (uint32_t)(uint16_t)(before + x[2]) | ((uint32_t)(uint16_t)(before + x[3]) << 16);
                o.z = (uint32_t)(uint16_t)(before + x[4]) | ((uint32_t)(uint16_t)(before + x[5]) << 16);
                o.w = (uint32_t)(uint16_t)(before + x[6]) | ((uint32_t)(uint16_t)(before + x[7]) << 16);
                *reinterpret_cast<uint4 *>(to) = o;
            } else {
                for (int e = 0; e < valid; e++) to[e] = (int16_t)(before + x[e]);
            }
        }
        wave_lds_order();
    };
    Group p, q;
    load_head(p);
    if constexpr (ONE) {
        load_payload(p);
        turn(p, q);
        return;
    }
    load_head(q);
    load_payload(p);
    // (two turns per round, with the groups' roles swapped: carried through a
    // loop, a group's loads would be copied, and so waited for, in every turn)
    for (int64_t gi = r.lo;;) {
        turn(p, q);
        if (++gi >= r.hi) break;
        turn(q, p);
        if (++gi >= r.hi) break;
    }
}

}  // namespace

hipError_t launch_unz(const ZDecArgs &a, int n, bool one, int grid, hipStream_t s) {
    if (grid < 1 || n < 1 || n > kZMaxFills) return hipErrorInvalidValue;
    if (one) hipLaunchKernelGGL(k_unz<true>, dim3(grid, n), dim3(kZWaves * 64), 0, s, a);
    else hipLaunchKernelGGL(k_unz<false>, dim3(grid), dim3(kZWaves * 64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_z(const ZArgs &a, int grid, hipStream_t s) {
    if (a.n < 1 || a.n > kZMaxFills || grid < a.n || grid > kZMaxGrid) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_z_size, dim3(grid), dim3(kZWaves * 64), 0, s, a);
    hipLaunchKernelGGL(k_z_pack, dim3(grid), dim3(kZWaves * 64), 0, s, a);
    return hipGetLastError();
}

}  // namespace daqk
