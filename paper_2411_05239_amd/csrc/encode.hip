// Encode kernels of the gfx950 ZipNN codec.
//
//   k_analyze  one workgroup of 8 or 16 waves per chunk: reads the chunk (16-byte
//              loads, XOR with the base for a delta, paper §IV-B, exponent
//              extraction when asked, §III-A), splits every word into its B
//              byte groups (paper §III-A/§III-B) and histograms each group in
//              LDS; one wave per code then builds the optimal lengths <= L by
//              package-merge (Larmore & Hirschberg, lists merged in
//              registers, see package_merge) and canonical codes (RFC 1951
//              §3.2.2).  A group with one value becomes RLE (paper §III-B);
//              a group whose most frequent byte fills half of it is also a ZG
//              candidate (zero-aware coding, §IV-B).  For every candidate the
//              waves sum each lane's code bits, each over a range of steps of
//              a lane group, which gives the exact payload sizes, so AUTO
//              keeps the smallest of RAW, HUF and ZG (paper §III-B, §V-A).
//              With a probe interval the probe chunks run first
//              (compressibility probing, §III-B).
//   k_place    one workgroup per tensor: exclusive scan of the 128-byte aligned
//              payload sizes in chunk-major order (the map that enables
//              parallel decode, paper §V-A), and whether the map holds ZG
//              entries (a header flag); the last workgroup places the
//              containers in the arena and writes their headers.
//   k_pack     one workgroup per chunk: a wave writes a lane group's words of
//              every coded stream (few chunks: a range of its steps) in
//              lock-step over the layout's steps and pairs; a word's place
//              follows from the rank among the lanes that take one (ballot +
//              prefix popcount).  Raw groups are copied on the same pass.
//              Every byte of the payload extent, padding included, is
//              written; no atomics.
//   k_compact  large launches with an XOR base: their words were packed into
//              staging slots and counted there, and move to their places.
#include <type_traits>

#include "zipnn_internal.h"

namespace zipnn {
namespace {

constexpr int kWaves = kBlock / 64;
// The analysis runs one workgroup of NT = 512 or 1024 threads per chunk, full
// CUs of 32 waves at 64 VGPRs: a chunk's bytes are spread over all its waves,
// and the chunks of a CU are in different phases.
// The counting pass's histograms: kCopies copies of every bin, side by side;
// a lane adds to copy (lane mod 32), so the lanes of half a wave always hit
// 32 different banks, whatever the values (LDS atomics on one bank, let alone
// one address, serialise).  Two byte groups share a copy's 32-bit counter
// (16 bits each), so the counts are reduced every kPartVec 16-byte vectors,
// before a half can overflow: a copy sees at most 32 threads x 128 vectors x 8
// elements = 32768 values of a group in a part.
constexpr uint32_t kCopies = 32;
constexpr uint32_t kPartVec = (2u << 20) / 16;

// Sized by the word width B.
template <int B, int NT>
union AnalyzeLds {
    uint32_t copies[B == 4 ? 2 : 1][256][kCopies];   // the counting pass
    uint32_t pm[3 * B][256];                         // the code constructions, one wave each
    uint32_t seg[2][B][NT];                          // the size pass: bits << 5 | last pair, HUF and ZG
};

// Reductions over a full wave in the vector unit (DPP row shifts, then row
// broadcasts; lane 63 ends with the result): shuffles through LDS would queue
// behind the counting passes' atomics.
template <class F>
__device__ __attribute__((always_inline)) inline uint32_t wave_reduce(uint32_t v, F op)   // op(0, x) = x
{
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true));   // row_shr:1
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true));
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true));
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true));
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ inline uint32_t wave_sum(uint32_t v)
{
    return wave_reduce(v, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ inline uint32_t wave_max(uint32_t v)
{
    return wave_reduce(v, [](uint32_t a, uint32_t b) { return max(a, b); });
}
__device__ inline float wave_fsum(float v)
{
    return __uint_as_float(wave_reduce(__float_as_uint(v), [](uint32_t a, uint32_t b) {
        return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
    }));
}

// x of lane (lane ^ D), for the compare-exchange steps below
template <int D>
__device__ inline uint32_t lane_xor(uint32_t x)
{
    static_assert(D == 1 || D == 2 || D == 4 || D == 8 || D == 16 || D == 32, "one bit of the lane");
    if constexpr (D == 1) return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);        // quad_perm 1,0,3,2
    else if constexpr (D == 2) return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);   // quad_perm 2,3,0,1
    else if constexpr (D == 4)   // mirrored in halves of a row, then in quads
        return __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
    else if constexpr (D == 8) return __builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true);  // row_ror:8
    else if constexpr (D == 16) {
        const auto y = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (threadIdx.x & 16) ? y[0] : y[1];
    } else {
        const auto y = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (threadIdx.x & 32) ? y[0] : y[1];
    }
}

// One step of a bitonic sort of the wave's 64 R keys (key e = R lane + r in
// x[r]): keys e and e ^ DIST, ascending where bit SIZE of e is clear.
template <int R, int SIZE, int DIST>
__device__ inline void sort_step(uint32_t* x)
{
    const uint32_t lane = threadIdx.x & 63;
    if constexpr (DIST >= R) {
        constexpr uint32_t D = DIST / R;
        const bool keep_min = (SIZE == 64 * R || ((R * lane) & SIZE) == 0) == ((lane & D) == 0);
#pragma unroll
        for (int r = 0; r < R; r++) {
            const uint32_t y = lane_xor<int(D)>(x[r]);
            x[r] = keep_min ? min(x[r], y) : max(x[r], y);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (r & DIST) continue;
            const bool asc = SIZE < R ? (r & SIZE) == 0 : ((R * lane) & SIZE) == 0;
            const uint32_t a = min(x[r], x[r | DIST]), b = max(x[r], x[r | DIST]);
            x[r] = asc ? a : b;
            x[r | DIST] = asc ? b : a;
        }
    }
    if constexpr (DIST > 1) sort_step<R, SIZE, DIST / 2>(x);
}
template <int R, int SIZE = 2>
__device__ inline void sort_keys(uint32_t* x)
{
    sort_step<R, SIZE, SIZE / 2>(x);
    if constexpr (SIZE < 64 * R) sort_keys<R, SIZE * 2>(x);
}

// One step of a merge over the lanes: every register's keys of lanes l and
// l ^ D, the smaller to the lower lane.  Across rows two registers at a time:
// the swap puts the lower lanes' keys of both in one and the upper lanes' in
// the other, so minimum and maximum need no select.
template <int N, int D>
__device__ inline void merge_step(uint32_t* x)
{
    if constexpr (D >= 16) {
#pragma unroll
        for (int r = 0; r < N; r += 2) {
            const auto y = D == 32 ? __builtin_amdgcn_permlane32_swap(x[r], x[r + 1], false, false)
                                   : __builtin_amdgcn_permlane16_swap(x[r], x[r + 1], false, false);
            const uint32_t a = min(y[0], y[1]), b = max(y[0], y[1]);
            const auto z = D == 32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false)
                                   : __builtin_amdgcn_permlane16_swap(a, b, false, false);
            x[r] = z[0];
            x[r + 1] = z[1];
        }
    } else {
        const bool upper = (threadIdx.x & D) != 0;
#pragma unroll
        for (int r = 0; r < N; r++) {
            const uint32_t y = lane_xor<D>(x[r]);
            x[r] = upper ? max(x[r], y) : min(x[r], y);
        }
    }
    if constexpr (D > 1) merge_step<N, D / 2>(x);
}

// Optimal code lengths <= L of the n symbols whose sort keys (f << 8 |
// symbol; f < 2^24) lie in buf[0, n), n <= 64 R, into len[256] (zero for the
// others, cleared by the caller), by one wave; returns the coded bits.
//
// Package-merge with lists made of leaves and packages: list 0 = the leaves
// sorted by (f, symbol); list d = the leaves merged with the packages of
// consecutive pairs of list d-1, a leaf before a package of equal weight.
// The 2n-2 first items of the top list are selected; the packages among the
// first m items of a list select the first 2*(their count) items of the list
// below; leaf i is selected at a level iff fewer than (leaves among the
// selected items) leaves precede it, so its length is the number of such
// levels.  Only the weights and kinds of a list's items matter, not which
// package is which: an item is the key weight * 2 + (1 for a package), and a
// list is a bitonic merge of two sorted runs in registers, R keys of each per
// lane (lower and upper half of the list).  The packages pass through LDS to
// come out in reverse order, as the merge wants them.  A level takes about
// 700 (R = 1) to 1500 cycles; with the ranks taken by searches in LDS over
// the whole workgroup a code took 22000 cycles, and LDS time is what the
// counting pass next to it is short of.
template <int R>
__device__ __attribute__((always_inline)) uint32_t package_merge(uint32_t* buf, uint32_t n, uint32_t L, uint8_t* len)
{
    const uint32_t lane = threadIdx.x & 63;
    uint32_t leaf[R], sym[R];
#pragma unroll
    for (int r = 0; r < R; r++) leaf[r] = R * lane + r < n ? buf[R * lane + r] : ~0u;
    sort_keys<R>(leaf);
#pragma unroll
    for (int r = 0; r < R; r++) {
        sym[r] = leaf[r] & 0xFFu;
        leaf[r] = leaf[r] == ~0u ? ~0u : (leaf[r] >> 8) << 1;
    }
    uint32_t x[2 * R];   // the list: items R lane + r, then 64 R + R lane + r
#pragma unroll
    for (int r = 0; r < R; r++) x[r] = leaf[r], x[R + r] = ~0u;
    // per level, which of this lane's items are leaves (2 R bits), the last
    // level lowest
    uint64_t kind0 = 0, kind1 = 0;
    for (uint32_t lev = 1; lev < L; lev++) {
        __builtin_amdgcn_wave_barrier();
        if constexpr (R == 1) {
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const uint32_t y = lane_xor<1>(x[h]);   // even lanes: the pair's second item
                const uint32_t pk = y == ~0u ? ~0u : ((x[h] & ~1u) + (y & ~1u)) | 1u;
                if (!(lane & 1)) buf[32 * h + lane / 2] = pk;
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int r = 0; r < R; r += 2) {
                    const uint32_t a = x[R * h + r], b = x[R * h + r + 1];
                    buf[32 * R * h + R / 2 * lane + r / 2] = b == ~0u ? ~0u : ((a & ~1u) + (b & ~1u)) | 1u;
                }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < R; r++) {
            const uint32_t pk = buf[64 * R - 1 - (R * lane + r)];
            x[r] = min(leaf[r], pk);
            x[R + r] = max(leaf[r], pk);
        }
        merge_step<2 * R, 32>(x);
#pragma unroll
        for (int dist = R / 2; dist >= 1; dist /= 2)
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int r = 0; r < R; r++) {
                    if (r & dist) continue;
                    uint32_t &a = x[R * h + r], &b = x[R * h + (r | dist)];
                    const uint32_t lo = min(a, b), hi = max(a, b);
                    a = lo;
                    b = hi;
                }
        uint32_t f = 0;
#pragma unroll
        for (int r = 0; r < 2 * R; r++) f |= ((x[r] & 1u) ^ 1u) << r;
        if constexpr (R > 1) kind1 = (kind1 << (2 * R)) | (kind0 >> (64 - 2 * R));
        kind0 = (kind0 << (2 * R)) | f;
    }
    uint32_t ln[R];
#pragma unroll
    for (int r = 0; r < R; r++) ln[r] = 0;
    uint32_t sel = 2 * n - 2;
    for (uint32_t lev = L - 1; lev >= 1; lev--) {
        uint32_t c = 0;   // leaves among the first sel items
#pragma unroll
        for (int r = 0; r < 2 * R; r++) {
            const uint32_t item = (r >= R ? 64 * R : 0) + R * lane + (r % R);
            c += uint32_t(__popcll(__ballot(((kind0 >> r) & 1) != 0 && item < sel)));
        }
        kind0 >>= 2 * R;
        if constexpr (R > 1) {
            kind0 |= kind1 << (64 - 2 * R);
            kind1 >>= 2 * R;
        }
#pragma unroll
        for (int r = 0; r < R; r++) ln[r] += R * lane + r < c ? 1u : 0u;
        sel = 2 * (sel - c);
    }
    const uint32_t c = min(sel, n);   // list 0 holds the leaves alone
    uint32_t bits = 0;
#pragma unroll
    for (int r = 0; r < R; r++)
        if (R * lane + r < n) {
            ln[r] += R * lane + r < c ? 1u : 0u;
            len[sym[r]] = uint8_t(ln[r]);
            bits += (leaf[r] >> 1) * ln[r];
        }
    return wave_sum(bits);
}

// The code lengths of the histogram fv[r] = f[lane + 64 r] (at least two
// symbols with f > 0), by one wave, with 256 words of LDS; returns the coded bits.
__device__ __attribute__((always_inline)) uint32_t build_lengths(const uint32_t* fv, uint32_t* buf, uint32_t L,
                                                                 uint8_t* len)
{
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t n = 0;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const uint64_t msk = __ballot(fv[r] > 0);
        const uint32_t s = lane + 64 * r;
        if (fv[r]) buf[n + uint32_t(__popcll(msk & lt_mask))] = (fv[r] << 8) | s;
        len[s] = 0;
        n += uint32_t(__popcll(msk));
    }
    __builtin_amdgcn_wave_barrier();
    return n <= 64 ? package_merge<1>(buf, n, L, len) : package_merge<4>(buf, n, L, len);
}

// Whether even the empirical entropy of a histogram held by one wave (fv[r] =
// f[lane + 64 r], sum tot) leaves a payload of `head` bytes and coded bits no
// smaller than the raw bytes: any prefix code spends at least
// sum f log2(tot/f) bits, so AUTO cannot keep this code (the decision is the
// one the exact size would give), and it need not be built.  In single
// precision (v_log_f32): each log2 of a count below 2^23 is within about
// 2^-18 of the truth, so the terms err by under 10^-5 bits per symbol in all,
// and rounding the products and the sum errs by under 10^-6 of the sum; the
// margins below (10^-4 relative, 10^-4 bits per symbol) keep the bound a lower
// bound.
//
// Near the boundary (within 1/32 of the raw bytes) whole code lengths give a
// closer bound, by weak duality: for any price mu of code space, lengths l in
// 1..L with sum 2^-l <= 1 cost sum f l >= sum min_l (f l + mu 2^-l) - mu.  The
// best mu lies between tot and 2 tot (each term's best l has mu 2^-(l+1) <= f <
// mu 2^-l) and is bisected on the sum of 2^-l; every mu tried gives a valid
// bound, in whole numbers (mu a multiple of 2^L).  The fraction byte of BF16
// weights, whose best code is 46 bytes under 128 KiB, is settled here in about
// 3000 cycles instead of a construction of 20000.  What is still open is
// built and sized exactly.
__device__ __attribute__((always_inline)) inline bool lengths_say_raw(const uint32_t* fv, uint32_t tot, uint32_t head,
                                                                      uint32_t raw, uint32_t L)
{
    float lf[4];
#pragma unroll
    for (int r = 0; r < 4; r++) lf[r] = __log2f(float(fv[r]));
    uint32_t lo = tot, hi = 2 * tot;
    for (int it = 0; it < 10 && hi - lo > 2 << kMaxL; it++) {
        const uint32_t mu = ((lo + hi) / 2) & ~((1u << kMaxL) - 1);
        const float lm = __log2f(float(mu));
        uint32_t v = 0, space = 0;   // space: sum of 2^(kMaxL - l)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            if (!fv[r]) continue;
            // the best length is the quotient's logarithm rounded down, or
            // one off where the logarithms round
            const int l0 = int(lm - lf[r]);
            uint32_t best = ~0u, bl = 1;
#pragma unroll
            for (int d = -1; d <= 1; d++) {
                const uint32_t l = uint32_t(min(max(l0 + d, 1), int(L)));
                const uint32_t c = fv[r] * l + (mu >> l);
                if (c < best) best = c, bl = l;
            }
            v += best;
            space += (1u << kMaxL) >> bl;
        }
        v = wave_sum(v);
        space = wave_sum(space);
        if (v > mu && uint64_t(head) + (v - mu + 7) / 8 >= raw) return true;
        if (space > 1u << kMaxL) lo = mu;
        else hi = mu;
    }
    return false;
}
__device__ inline bool entropy_says_raw(const uint32_t* fv, uint32_t tot, uint32_t head, uint32_t raw, uint32_t L)
{
    const float lt = __log2f(float(tot));
    float h = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; r++)
        if (fv[r]) h += float(fv[r]) * (lt - __log2f(float(fv[r])));
    h = wave_fsum(h);
    const float lb = h * (1.0f - 1e-4f) - 1e-4f * float(tot) - 1.0f;
    const uint64_t words_lb = lb > 0.0f ? uint64_t(lb / 32.0f) : 0u;   // floor: a lower bound too
    const uint64_t bound = uint64_t(head) + 4 * words_lb;
    if (bound >= raw) return true;
    return bound + raw / 32 >= raw && lengths_say_raw(fv, tot, head, raw, L);
}

// One workgroup per chunk over a two-dimensional grid (chunk_grid).  A loop
// over chunks in the kernel has the compiler compute every address that does
// not depend on the chunk before it and keep it in scratch memory: 27 spilled
// registers of the analysis, 1 GB written per 5 GB of input.
__device__ inline uint32_t chunk_of_block() { return blockIdx.y * gridDim.x + blockIdx.x; }
inline dim3 chunk_grid(uint32_t chunks)
{
    const uint32_t x = min(max(chunks, 1u), 1u << 16);
    return dim3(x, (max(chunks, 1u) + x - 1) / x);
}

// The tensor holding chunk g: the last i with prefix[i] <= g, by a whole wave
// (64 candidates a step: one dependent load for up to 64 tensors, two for
// 4096, where a binary search made six and twelve).
__device__ inline int find_desc(const uint32_t* prefix, int n_desc, uint32_t g)
{
    const int lane = int(threadIdx.x & 63);
    int lo = 0, n = n_desc;   // it is in [lo, lo + n)
    while (n > 1) {
        const int step = (n + 63) / 64;
        const int i = lane * step;
        const int c = __popcll(__ballot(i < n && prefix[lo + min(i, n - 1)] <= g)) - 1;
        lo += c * step;
        n = min(step, n - c * step);
    }
    return lo;
}

// Load NB bytes (NB in {2,4,8,16,32,64}) of device memory into 32-bit words
// (global loads: a generic pointer's flat loads would also wait for LDS).
template <class T>
using global_ptr = const T __attribute__((address_space(1)))*;
// A flat access also leaves the compiler unsure which later wait covers it:
// one pending before the packer's loop made every step wait for all memory
// operations, stores included.
__device__ inline uint32_t gld8(const uint8_t* p)
{
    return *(global_ptr<uint8_t>)reinterpret_cast<uint64_t>(p);
}
template <class T>
__device__ inline void gst(uint8_t* p, T v)
{
    *(T __attribute__((address_space(1)))*)reinterpret_cast<uint64_t>(p) = v;
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <int NB>
__device__ inline void loadNB(const uint8_t* p, uint32_t* w)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    if constexpr (NB == 2) w[0] = *(global_ptr<uint16_t>)a;
    else if constexpr (NB == 4) w[0] = *(global_ptr<uint32_t>)a;
    else if constexpr (NB == 8) {
        const u32x2 v = *(global_ptr<u32x2>)a;
        w[0] = v.x;
        w[1] = v.y;
    } else {
#pragma unroll
        for (int i = 0; i < NB / 16; i++) {
            const u32x4 v = *(global_ptr<u32x4>)(a + 16 * i);
            w[4 * i] = v.x;
            w[4 * i + 1] = v.y;
            w[4 * i + 2] = v.z;
            w[4 * i + 3] = v.w;
        }
    }
}

// A chunk's bytes as a buffer resource: a load's address is a lane offset
// and a scalar offset (no 64-bit address per load in vector registers).
// Reads whose lane offset is past the end give zero; the scalar offset is
// not part of that check, so it is used only where every lane is in range.
__device__ inline __amdgpu_buffer_rsrc_t in_rsrc(const uint8_t* p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p), (short)0, int(bytes), 0x00020000);
}
// Non-temporal (the cache policy bits of the buffer builtins): bytes touched
// once and not again soon.  The packer's input and raw stores so: 256 MiB of
// FP32 243 -> 227 us a pass, a 5 GB checkpoint 3306 -> 3216, a 1.7 GB delta
// 1733 -> 1665; its words complete in scattered order, and their partly
// written lines must stay (non-temporal: 4530 us).  The analysis' size pass
// too (checkpoint 3216 -> 3101), but not its counting pass, which the size
// pass follows (3320) -- unless there is an XOR base, where large launches
// need no size pass (delta 1663 -> 1612).
constexpr int kNt = 2;
template <int NB, int AUX = 0>
__device__ __attribute__((always_inline)) inline void buf_in(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff,
                                                             uint32_t* w)
{
    if constexpr (NB == 2) w[0] = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, AUX);
    else if constexpr (NB == 4) w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, AUX);
    else if constexpr (NB == 8) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, AUX);
        w[0] = v.x;
        w[1] = v.y;
    } else {
#pragma unroll
        for (int i = 0; i < NB / 16; i++) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff + 16 * i, soff, AUX);
            w[4 * i] = v.x;
            w[4 * i + 1] = v.y;
            w[4 * i + 2] = v.z;
            w[4 * i + 3] = v.w;
        }
    }
}
// The same of the chunk XORed with its base, exponent extracted when xf.
struct ChunkIn {
    __amdgpu_buffer_rsrc_t src, base;
    bool delta, xf;
};
template <int B, int NB, int AUX = 0>
__device__ __attribute__((always_inline)) inline void chunk_in(const ChunkIn& in, uint32_t voff, uint32_t soff,
                                                               uint32_t* w)
{
    constexpr int NW = NB >= 4 ? NB / 4 : 1;
    buf_in<NB, AUX>(in.src, voff, soff, w);
    if (in.delta) {
        uint32_t y[NW];
        buf_in<NB, AUX>(in.base, voff, soff, y);
#pragma unroll
        for (int x = 0; x < NW; x++) w[x] ^= y[x];
    }
    if (in.xf)
#pragma unroll
        for (int x = 0; x < NW; x++) w[x] = exp_fwd<B>(w[x]);
}

// The words of group q of a chunk (g elements, XORed with the base, then with
// the exponent extracted when xf), or of the partial last group (zero beyond
// the chunk's m elements).
template <int B, int G>
__device__ inline void group_words(const uint8_t* src, const uint8_t* base, uint32_t q, uint32_t m, uint32_t* wd,
                                   bool xf)
{
    constexpr int NB = B * G;
    constexpr int NW = NB >= 4 ? NB / 4 : 1;
    const uint32_t e = q * G;
    if (e + G <= m) {
        loadNB<NB>(src + uint64_t(e) * B, wd);
        if (base) {
            uint32_t bw[NW];
            loadNB<NB>(base + uint64_t(e) * B, bw);
#pragma unroll
            for (int x = 0; x < NW; x++) wd[x] ^= bw[x];
        }
    } else {
        // the partial last group: bytes past the chunk's m elements are zero
        const uint32_t nb = (m - e) * B;
#pragma unroll
        for (int x = 0; x < NW; x++) {
            wd[x] = 0;
#pragma unroll
            for (int b = 0; b < 4; b++) {
                const uint32_t jb = 4 * x + b;
                if (jb < nb) {
                    const uint32_t v = gld8(src + uint64_t(e) * B + jb) ^ (base ? gld8(base + uint64_t(e) * B + jb) : 0u);
                    wd[x] |= v << (8 * b);
                }
            }
        }
    }
    if (xf)
#pragma unroll
        for (int x = 0; x < NW; x++) wd[x] = exp_fwd<B>(wd[x]);
}

// Element e of a chunk as a little-endian word (XORed with the base, exponent
// extracted when xf), read byte by byte.
template <int B>
__device__ inline uint32_t element_word(const uint8_t* src, const uint8_t* base, uint32_t e, bool xf)
{
    uint32_t v = 0;
#pragma unroll
    for (int b = 0; b < B; b++) {
        const uint64_t o = uint64_t(e) * B + b;
        v |= (gld8(src + o) ^ (base ? gld8(base + o) : 0u)) << (8 * b);
    }
    return xf ? exp_fwd<B>(v) : v;
}

// byte of stream k of element i of a group's words
template <int B>
__device__ inline uint32_t sym_of(const uint32_t* wd, int k, int i)
{
    const int jb = i * B + (B - 1 - k);
    return (wd[jb >> 2] >> (8 * (jb & 3))) & 0xFFu;
}

// The bytes of stream k in a 32-bit word of B-byte elements (in its first
// `nb` bytes).
template <int B>
__device__ inline constexpr uint32_t stream_bytes(int k, int nb)
{
    uint32_t m = 0;
    for (int jb = B - 1 - k; jb < nb; jb += B) m |= 0xFFu << (8 * jb);
    return m;
}

// Whether a group of gcnt symbols of stream k holds a value other than z.
template <int B, int G>
__device__ inline bool marked(const uint32_t* wd, int k, uint32_t gcnt, uint32_t z)
{
    bool mk = false;
#pragma unroll
    for (int i = 0; i < G; i++) mk |= uint32_t(i) < gcnt && sym_of<B>(wd, k, i) != z;
    return mk;
}

// The symbols of stream k that lie in groups of g made of z[k] alone, for the
// streams in zc, summed over the wave.  Every value other than z lies in a
// marked group, so the histogram over the marked groups is the main one with
// this many taken off the count of z.
template <int B, int G, int NT>
__device__ __attribute__((always_inline)) void zg_unmarked(const uint8_t* src, const uint8_t* base, uint32_t zc,
                                                           const uint32_t* z, uint32_t m, uint32_t* un, bool xf)
{
    constexpr int NB = B * G;
    constexpr int NW = NB >= 4 ? NB / 4 : 1;
    constexpr uint32_t CB = NB >= 16 ? 2 : 4;   // groups in flight per thread
    const uint32_t Gtot = (m + G - 1) / G;
#pragma unroll
    for (int k = 0; k < B; k++) un[k] = 0;
    for (uint32_t q0 = threadIdx.x; q0 < Gtot; q0 += CB * NT) {
        uint32_t wds[CB][NW];
#pragma unroll
        for (uint32_t u = 0; u < CB; u++)
            if (q0 + u * NT < Gtot) group_words<B, G>(src, base, q0 + u * NT, m, wds[u], xf);
#pragma unroll
        for (uint32_t u = 0; u < CB; u++) {
            const uint32_t q = q0 + u * NT;
            if (q >= Gtot) continue;
            const uint32_t gcnt = min(uint32_t(G), m - q * G);
#pragma unroll
            for (int k = 0; k < B; k++)
                if (((zc >> k) & 1) && !marked<B, G>(wds[u], k, gcnt, z[k])) un[k] += gcnt;
        }
    }
#pragma unroll
    for (int k = 0; k < B; k++) un[k] = wave_sum(un[k]);
}

// Bytes of stream k of the g elements of a group's words, packed little-endian
// into one register (groups of at most 4 bytes per stream): v_perm_b32 picks
// byte B-1-k of each word (selector 0-3: the second operand, 4-7: the first,
// 0x0C: zero).
template <int B, int G>
__device__ inline uint32_t gather_stream(const uint32_t* wd, int k)
{
    if constexpr (B == 2) {
        const uint32_t b = uint32_t(1 - k);   // byte of the 16-bit element
        if constexpr (G == 2) return __builtin_amdgcn_perm(0u, wd[0], 0x0C0C0000u | ((b + 2) << 8) | b);
        else return __builtin_amdgcn_perm(wd[1], wd[0], ((b + 6) << 24) | ((b + 4) << 16) | ((b + 2) << 8) | b);
    } else if constexpr (B == 4) {
        const uint32_t b = uint32_t(3 - k);
        const uint32_t lo = __builtin_amdgcn_perm(wd[1], wd[0], 0x0C0C0000u | ((b + 4) << 8) | b);
        if constexpr (G == 2) return lo;
        else return lo | __builtin_amdgcn_perm(wd[3], wd[2], ((b + 4) << 24) | (b << 16) | 0x0C0Cu);
    } else {
        uint32_t v = 0;
#pragma unroll
        for (int i = 0; i < G; i++) v |= sym_of<B>(wd, k, i) << (8 * i);
        return v;
    }
}

// Code bits of steps [s0, s1) of lane group j of one chunk, per lane and
// candidate: HUF candidates (bit k of hc, lengths lens[k]) over every group,
// ZG candidates (bit k of zgc, lengths lens2[k], fill value z[k]) over the
// groups holding another value.  out[v][k] = bits << 5 | bits of the last
// pair coded here (at most 4096 * 11 bits in all, 22 in a pair).
template <int B, int G>
__device__ __attribute__((always_inline)) void count_steps(const ChunkIn& in, const uint8_t* src, const uint8_t* base, uint32_t hc,
                                                           uint32_t zgc, const uint8_t (*lens)[256],
                                                           const uint8_t (*lens2)[256], const uint32_t* z, uint32_t j,
                                                           uint32_t s0, uint32_t s1, uint32_t W, uint32_t m,
                                                           uint32_t (*out)[B], bool xf)
{
    constexpr int NB = B * G;
    constexpr int NW = NB >= 4 ? NB / 4 : 1;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t w = 64 * j + lane;
    const uint32_t Gtot = (m + G - 1) / G, Gfull = m / G, rem = m - Gfull * G;
    const uint32_t ng = (w < W && w < Gtot) ? (Gtot - 1 - w) / W + 1 : 0;
    const uint32_t end = min(ng, s1);
    uint32_t bits[2][B], last[2][B];
#pragma unroll
    for (int k = 0; k < B; k++) bits[0][k] = bits[1][k] = last[0][k] = last[1][k] = 0;
    if (zgc == 0 && s1 > s0 && min(W, 64 * j + 64) - 1 + (s1 - 1) * W < Gfull) {
        // HUF alone and a full group for every lane at every step: no
        // conditions, so the table reads of several groups are in flight
        constexpr uint32_t FB = NB >= 32 ? 2 : (NB >= 16 ? 4 : 8);
        if (w < W) {
            uint32_t lw[NW];
            auto add = [&](auto n_const, uint32_t jj) __attribute__((always_inline)) {
                constexpr uint32_t N = decltype(n_const)::value;
                uint32_t wds[N][NW];
#pragma unroll
                for (uint32_t u = 0; u < N; u++) chunk_in<B, NB, kNt>(in, w * NB, (jj + u) * W * NB, wds[u]);
#pragma unroll
                for (int k = 0; k < B; k++) {
                    if (!((hc >> k) & 1)) continue;
                    // 8 reads in flight (left alone, the compiler waits for
                    // every two)
                    constexpr uint32_t U = N * G > 8 ? 8 / G : N;
#pragma unroll
                    for (uint32_t u0 = 0; u0 < N; u0 += U) {
                        uint32_t e[U * G];
#pragma unroll
                        for (uint32_t i = 0; i < U * G; i++)
                            e[i] = lens[k][sym_of<B>(wds[u0 + i / G], k, int(i % G))];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (uint32_t i = 0; i < U * G; i++) bits[0][k] += e[i];
                    }
                }
#pragma unroll
                for (int x = 0; x < NW; x++) lw[x] = wds[N - 1][x];
            };
            uint32_t jj = s0;
            for (; (s1 - jj) % FB; jj++) add(std::integral_constant<uint32_t, 1>{}, jj);
            for (; jj < s1; jj += FB) add(std::integral_constant<uint32_t, FB>{}, jj);
#pragma unroll
            for (int k = 0; k < B; k++)
                if ((hc >> k) & 1)
                    last[0][k] = uint32_t(lens[k][sym_of<B>(lw, k, G - 2)]) + lens[k][sym_of<B>(lw, k, G - 1)];
        }
#pragma unroll
        for (int k = 0; k < B; k++) {
            out[0][k] = (bits[0][k] << 5) | last[0][k];
            out[1][k] = 0;
        }
        return;
    }
    constexpr uint32_t CB = NB >= 32 ? 1 : (NB >= 16 ? 2 : 4);   // groups in flight per lane
    for (uint32_t j0 = s0; j0 < end; j0 += CB) {
        uint32_t wds[CB][NW];
#pragma unroll
        for (uint32_t u = 0; u < CB; u++)
            if (j0 + u < end) group_words<B, G>(src, base, w + (j0 + u) * W, m, wds[u], xf);
#pragma unroll
        for (uint32_t u = 0; u < CB; u++) {
            const uint32_t jj = j0 + u;
            const uint32_t q = w + jj * W;
            const uint32_t gcnt = jj >= end ? 0u : (q < Gfull ? G : rem);
            const uint32_t* wd = wds[u];
#pragma unroll
            for (int k = 0; k < B; k++) {
#pragma unroll
                for (int v = 0; v < 2; v++) {
                    if (!(((v ? zgc : hc) >> k) & 1)) continue;
                    const uint8_t* ln = v ? lens2[k] : lens[k];
                    const uint32_t gc = (v && !marked<B, G>(wd, k, gcnt, z[k])) ? 0u : gcnt;
#pragma unroll
                    for (int pr = 0; pr < G / 2; pr++) {
                        if (2u * pr < gc) {
                            uint32_t c = ln[sym_of<B>(wd, k, 2 * pr)];
                            if (2u * pr + 1 < gc) c += ln[sym_of<B>(wd, k, 2 * pr + 1)];
                            bits[v][k] += c;
                            last[v][k] = c;
                        }
                    }
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < B; k++) {
        out[0][k] = (bits[0][k] << 5) | last[0][k];
        out[1][k] = (bits[1][k] << 5) | last[1][k];
    }
}

template <int B>
struct AnalyzeTail {
    alignas(4) uint8_t lens[B][256];    // HUF code lengths
    alignas(4) uint8_t lens2[B][256];   // ZG code lengths
    uint32_t z[4];           // ZG fill value: the most frequent byte (smallest on ties)
    uint32_t zn[4];          // its count over the marked groups
    uint32_t open;           // bit k: mode still to be decided (neither forced RAW nor RLE)
    uint32_t build[3];       // bit k: codes to build: HUF, ZG, HUF where a forced ZG falls back to it
    uint32_t hc;             // bit k: HUF candidate
    uint32_t zc;             // bit k: ZG considered (its histogram is needed)
    uint32_t zgc;            // bit k: ZG candidate
    uint32_t fin;            // bit k: ZG chosen (else HUF) for a coded stream
    uint32_t coded;          // bit k: coded (HUF or ZG chosen)
    uint32_t words[2][4];    // words over all lane groups, per stream: HUF, ZG
    uint32_t T[2][4];        // coded bits of the candidates: HUF, ZG
    int pol[4];              // policy of each group in this chunk (RAW where probing skips it)
    uint32_t specok;         // bit k: the main pass's count of zeros in unmarked groups holds (z = 0)
    uint32_t amb;            // staged packing: bit k, the mode decision needs exact sizes
};

// One workgroup per chunk (phase -1: every chunk; with a probe interval K,
// phase 0: the probe chunks c mod (K+1) = 0 of each tensor, phase 1: the
// others, where a byte group that the run's probe chunk stored raw is stored
// raw without analysis under AUTO: compressibility probing, paper §III-B):
//   1. histogram f of every byte group;
//   2. wave k classifies group k: forced RAW, RLE (one value), else a HUF
//      candidate (unless ZG is forced) and, when ZG is forced or (AUTO) the
//      most frequent value z fills half the group, a ZG candidate, whose
//      histogram counts only the groups of g symbols that hold another value;
//   3. the workgroup builds the candidates' code lengths;
//   4. its waves sum the code bits of every candidate, each wave a range of
//      steps of a lane group, which gives the exact sizes;
//   5. the mode of each group (AUTO: the smallest of RAW, HUF, ZG, ties to
//      RAW then HUF), its entry, its lane-group word counts and its canonical
//      code table.

// Shared memory of the analysis of one chunk.
template <int BB, int NT>
struct AnalyzeShared {
    AnalyzeLds<BB, NT> S;
    uint32_t hist[BB][256];
    uint32_t lgw[2][BB][64];        // words per lane group: HUF, ZG
    AnalyzeTail<BB> A;
    uint32_t zsum[NT / 64][4];      // symbols in unmarked groups, per wave
};

// The analysis of chunk gc by one workgroup (steps 1-5 above); a chunk that
// the probing phase leaves to the other launch is passed over.
template <int BB, int NT, int HOLD>
__device__ __attribute__((always_inline)) void analyze_chunk(uint32_t gc, const EncDesc& d, uint32_t c,
                                                             const EncParams& p, int phase,
                                                             EncEntry* __restrict__ entries, uint8_t* __restrict__ lens,
                                                             uint32_t* __restrict__ nwords, AnalyzeShared<BB, NT>& sh)
{
    constexpr int kWavesA = NT / 64;
    AnalyzeLds<BB, NT>& S = sh.S;
    auto& hist = sh.hist;
    AnalyzeTail<BB>& A = sh.A;
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    constexpr uint32_t B = BB;
    const uint32_t run = p.skip + 1;
    const bool probe = c % run == 0;
    if ((phase == 0 && !probe) || (phase == 1 && probe)) return;
    // the groups this chunk analyses (uniform: every thread reads the same entries)
    uint32_t live = (1u << B) - 1;
    if (!probe)
        for (uint32_t k = 0; k < B; k++)
            if (p.policy[k] == ZIPNN_AUTO && entries[uint64_t(gc - c % run) * B + k].mode == kModeRaw)
                live &= ~(1u << k);
    const uint32_t E = p.chunk / B;
    const uint64_t e0 = uint64_t(c) * E;
    const uint32_t m = uint32_t(min(uint64_t(E), d.n - e0));
    const uint32_t W = (m + p.S - 1) / p.S;
    const uint32_t NG = (W + 63) / 64;
    const uint32_t head = huf_head(W), head_z = head + zg_bitmap(m, p.g);
    if (live == 0) {
        if (uint32_t(t) < B) {
            EncEntry e;
            e.pad = 0;
            e.mode = kModeRaw;
            e.rle = 0;
            e.bytes = m;
            entries[uint64_t(gc) * B + t] = e;
        }
        return;
    }
    constexpr uint32_t kCopyWords = sizeof(S.copies) / 4;
    for (uint32_t i = t; i < kCopyWords / 4; i += NT)
        reinterpret_cast<uint4*>(&S.copies[0][0][0])[i] = make_uint4(0, 0, 0, 0);
    for (uint32_t i = t; i < B * 256; i += NT) (&hist[0][0])[i] = 0;
    if (t == 0) A.open = A.build[0] = A.build[1] = A.build[2] = A.hc = A.zc = A.zgc = A.fin = A.coded = A.specok = A.amb = 0;
    if (t < 8) (&A.words[0][0])[t] = 0;
    if (t < 4) A.pol[t] = ((live >> t) & 1) ? int(p.policy[t]) : ZIPNN_RAW;
    __syncthreads();
    const uint8_t* src = d.src + e0 * B;
    const uint8_t* base = d.base ? d.base + e0 * B : nullptr;
    const uint32_t nbytes = m * B;
    const bool xf = (p.flags & kFlagExp) != 0;
    // 16-byte vectors; the element boundary is aligned since 16 % B == 0
    const uint32_t nvec = nbytes / 16;
    const ChunkIn in{in_rsrc(src, nbytes), in_rsrc(base ? base : src, nbytes), base != nullptr, xf};
    // this lane's copy of the counters: B = 1 counts in 32 bits, else byte
    // groups 2a and 2a+1 in the halves of array a
    const uint32_t copy = uint32_t(lane) % kCopies;
    // counts byte jb (of a run of whole little-endian words starting at x)
    auto add = [&](const uint32_t* x, int jb) __attribute__((always_inline)) {
        const uint32_t k = B - 1 - uint32_t(jb) % B;   // byte jb%B of a word -> stream B-1-jb%B
        atomicAdd(&S.copies[k / 2][(x[jb >> 2] >> (8 * (jb & 3))) & 0xFFu][copy], (B > 1 && (k & 1)) ? 0x10000u : 1u);
    };
    // Delta-like groups (zero bytes in at least half of the first 64 vectors;
    // the same vectors in every wave, so the choice is uniform) also count, in
    // this pass, the groups of g zero bytes.  If 0 turns out to be the most
    // frequent value, that gives the ZG histogram without a pass of its own.
    const uint32_t gB = p.g * B;
    uint32_t spec = 0;
    if (nbytes % 16 == 0 && gB <= 16) {
        uint32_t x0 = 0;
        if (uint32_t(lane) < nvec) {
            loadNB<4>(src + 16 * lane, &x0);
            if (base) {
                uint32_t y0;
                loadNB<4>(base + 16 * lane, &y0);
                x0 ^= y0;
            }
            if (xf) x0 = exp_fwd<B>(x0);
        }
        for (uint32_t k = 0; k < B; k++) {
            const uint32_t byte = (x0 >> (8 * (B - 1 - k))) & 0xFFu;
            const bool zg_policy = A.pol[k] == ZIPNN_AUTO || A.pol[k] == ZIPNN_ZG;
            if (zg_policy && __popcll(__ballot(uint32_t(lane) < nvec && byte == 0)) >= 32) spec |= 1u << k;
        }
    }
    spec = __builtin_amdgcn_readfirstlane(spec);
    uint32_t ung[B];   // unmarked groups (of zeros)
#pragma unroll
    for (uint32_t k = 0; k < B; k++) ung[k] = 0;
    // LV: every group is live (no per-byte test); SP: count the groups of
    // zeros of the streams in `spec`; DL: there is an XOR base
    auto count = [&](auto lv_const, auto sp_const, auto dl_const, uint32_t v_begin, uint32_t v_end) {
        constexpr bool LV = decltype(lv_const)::value;
        constexpr bool SP = decltype(sp_const)::value;
        ChunkIn cin = in;
        cin.delta = decltype(dl_const)::value;
        // vectors in flight per lane (loading the next batch ahead of this
        // one's atomics took registers and measured 5% slower)
        constexpr uint32_t HB = decltype(dl_const)::value ? 2 : 4;
        auto one = [&](const uint32_t* x) __attribute__((always_inline)) {
#pragma unroll
            for (int jb = 0; jb < 16; jb++) {
                if (!LV && !((live >> (int(B) - 1 - (jb % int(B)))) & 1)) continue;
                add(x, jb);
            }
            if constexpr (SP) {
#pragma unroll
                for (int k = 0; k < int(B); k++) {
                    if (!((spec >> k) & 1)) continue;
                    // the stream's bytes of the four words
                    constexpr uint32_t kAll = B == 1 ? 0xFFFFFFFFu : (B == 2 ? 0x00FF00FFu : 0x000000FFu);
                    const uint32_t km = B == 1 ? kAll : kAll << (8 * (int(B) - 1 - k));
                    uint32_t un = 0;   // groups of zeros in this vector
                    if (gB == 8) {
                        un += uint32_t(((x[0] | x[1]) & km) == 0) + uint32_t(((x[2] | x[3]) & km) == 0);
                    } else if (gB == 4) {
#pragma unroll
                        for (int y = 0; y < 4; y++) un += uint32_t((x[y] & km) == 0);
                    } else if (gB == 2) {
#pragma unroll
                        for (int y = 0; y < 4; y++)
                            un += uint32_t((x[y] & km & 0xFFFFu) == 0) + uint32_t((x[y] & km & 0xFFFF0000u) == 0);
                    } else {
                        un += uint32_t(((x[0] | x[1] | x[2] | x[3]) & km) == 0);
                    }
                    ung[k] += un;
                }
            }
        };
        for (uint32_t v0 = v_begin; v0 < v_end; v0 += HB * NT) {
            uint32_t xs[HB][4];
#pragma unroll
            for (uint32_t i = 0; i < HB; i++) chunk_in<B, 16, decltype(dl_const)::value ? kNt : 0>(cin, (v0 + i * NT + t) * 16, 0, xs[i]);
#pragma unroll
            for (uint32_t i = 0; i < HB; i++)
                if (v0 + i * NT + t < v_end) one(xs[i]);
        }
    };
    // HOLD > 0: a full chunk of HOLD groups of 4 per thread, which its size
    // pass would give to the same threads (wave wv: range wv / NG of the steps
    // of lane group wv % NG), is read in that order, and the bytes of its
    // first streams stay in registers for the size pass.
    constexpr int kHeld = HOLD ? (BB == 4 ? 2 : 1) : 1;
    constexpr int kHoldN = HOLD ? HOLD : 1;
    uint32_t hold[kHeld][kHoldN];
    bool held = false;
    if constexpr (HOLD > 0) {
        held = m == uint32_t(HOLD) * 4 * NT && W % 64 == 0 && NG <= uint32_t(kWavesA) && kWavesA % NG == 0 &&
               live == (1u << B) - 1 && spec == 0 && !in.delta && !xf;
        if (held) {
            constexpr int NB = BB * 4, NW = NB / 4;
            constexpr int FB = 16 / NW;   // groups in flight
            const uint32_t q0 = 64 * (uint32_t(wv) % NG) + (uint32_t(wv) / NG) * HOLD * W;
            uint32_t wd[2][FB][NW];
            auto fetch = [&](int i0, uint32_t (*x)[NW]) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < FB; u++) buf_in<NB, kNt>(in.src, lane * NB, (q0 + (i0 + u) * W) * NB, x[u]);
            };
            fetch(0, wd[0]);
#pragma unroll
            for (int i0 = 0; i0 < HOLD; i0 += FB) {
                uint32_t(*x)[NW] = wd[(i0 / FB) & 1];
                if (i0 + FB < HOLD) fetch(i0 + FB, wd[(i0 / FB + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);   // the next batch is on its way, and no more than that
#pragma unroll
                for (int u = 0; u < FB; u++) {
#pragma unroll
                    for (int jb = 0; jb < NB; jb++) add(x[u], jb);
#pragma unroll
                    for (int k = 0; k < kHeld; k++) hold[k][i0 + u] = gather_stream<BB, 4>(x[u], k);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    for (uint32_t part = 0;; part += kPartVec) {
        const uint32_t v_end = min(nvec, part + kPartVec);
        using T = std::integral_constant<bool, true>;
        using F = std::integral_constant<bool, false>;
        if (held) ;
        else if (live != (1u << B) - 1) in.delta ? count(F{}, T{}, T{}, part, v_end) : count(F{}, T{}, F{}, part, v_end);
        else if (spec) in.delta ? count(T{}, T{}, T{}, part, v_end) : count(T{}, T{}, F{}, part, v_end);
        else in.delta ? count(T{}, F{}, T{}, part, v_end) : count(T{}, F{}, F{}, part, v_end);
        const bool done = v_end == nvec;
        if (done)   // the elements after the last whole vector
            for (uint32_t e = nvec * 16 / B + t; e < m; e += NT) {
                const uint32_t v = element_word<B>(src, base, e, xf);
                for (uint32_t b = 0; b < B; b++)
                    if ((live >> (B - 1 - b)) & 1) add(&v, int(b));
            }
        __syncthreads();
        // the copies of a bin: kPer neighbouring threads sum kEach counters each
        constexpr uint32_t kPer = NT / 256, kEach = kCopies / kPer;
        static_assert(kPer >= 1 && kPer <= 4 && kEach % 4 == 0, "threads per bin");
        const uint32_t s = uint32_t(t) / kPer, q = uint32_t(t) % kPer;
        for (uint32_t a = 0; a < (B == 4 ? 2u : 1u); a++) {
            uint4* cp = reinterpret_cast<uint4*>(&S.copies[a][s][kEach * q]);
            uint32_t lo = 0, hi = 0;
#pragma unroll
            for (uint32_t i = 0; i < kEach / 4; i++) {
                const uint4 x = cp[i];
                if (!done) cp[i] = make_uint4(0, 0, 0, 0);
                if (B == 1) {
                    lo += x.x + x.y + x.z + x.w;
                } else {
                    lo += (x.x & 0xFFFFu) + (x.y & 0xFFFFu) + (x.z & 0xFFFFu) + (x.w & 0xFFFFu);
                    hi += (x.x >> 16) + (x.y >> 16) + (x.z >> 16) + (x.w >> 16);
                }
            }
            if (kPer >= 2) lo += lane_xor<1>(lo), hi += lane_xor<1>(hi);
            if (kPer >= 4) lo += lane_xor<2>(lo), hi += lane_xor<2>(hi);
            if (q == 0) {
                hist[2 * a][s] += lo;
                if (B > 1) hist[2 * a + 1][s] += hi;
            }
        }
        __syncthreads();
        if (done) break;
    }
    if (spec) {
#pragma unroll
        for (uint32_t k = 0; k < B; k++) {
            const uint32_t un = wave_sum(ung[k]) * p.g;
            if (lane == 0) sh.zsum[wv][k] = un;
        }
    }
    // 2. classification, wave k for group k
    if (uint32_t(wv) < B) {
        __builtin_amdgcn_s_setprio(3);
        const int k = wv;
        const int policy = A.pol[k];
        uint32_t fv[4], nd = 0, best = 0;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            fv[r] = hist[k][lane + 64 * r];
            nd += __popcll(__ballot(fv[r] > 0));
            // most frequent value, smallest on ties: key f << 8 | (255 - s)
            best = max(best, (fv[r] << 8) | uint32_t(255 - (lane + 64 * r)));
        }
        best = wave_max(best);
        const uint32_t arg = 255 - (best & 0xFFu);
        if (policy == ZIPNN_RAW || nd <= 1) {
            if (lane == 0) {
                EncEntry e;
                e.pad = 0;
                const bool rle = policy != ZIPNN_RAW && nd == 1;
                e.mode = rle ? kModeRle : kModeRaw;
                e.rle = rle ? uint8_t(arg) : 0;
                e.bytes = rle ? 0 : m;
                entries[uint64_t(gc) * B + k] = e;
            }
        } else {
            const bool huf = policy == ZIPNN_HUF || (policy == ZIPNN_AUTO && !entropy_says_raw(fv, m, head, m, p.L));
            const bool zc = policy == ZIPNN_ZG || (policy == ZIPNN_AUTO && 2 * (best >> 8) >= m);
            if (lane == 0) {
                atomicOr(&A.open, 1u << k);
                if (huf) atomicOr(&A.build[0], 1u << k);
                if (zc) atomicOr(&A.zc, 1u << k);
                if (zc && ((spec >> k) & 1) && arg == 0) atomicOr(&A.specok, 1u << k);
                A.z[k] = arg;
            }
        }
    }
    __syncthreads();
    // the ZG histograms
    if (A.zc) {
        // groups whose count of unmarked symbols the main pass could not
        // give: one more pass over the data
        const uint32_t need = A.zc & ~A.specok;
        if (need) {
            uint32_t un[B];
            switch (p.g) {
            case 2: zg_unmarked<BB, 2, NT>(src, base, need, A.z, m, un, xf); break;
            case 4: zg_unmarked<BB, 4, NT>(src, base, need, A.z, m, un, xf); break;
            default: zg_unmarked<BB, 8, NT>(src, base, need, A.z, m, un, xf); break;
            }
#pragma unroll
            for (uint32_t k = 0; k < B; k++)
                if (lane == 0 && ((need >> k) & 1)) sh.zsum[wv][k] = un[k];
            __syncthreads();
        }
        if (uint32_t(wv) < B && ((A.zc >> wv) & 1)) {
            const int k = wv;
            const uint32_t z = A.z[k];
            uint32_t zn = hist[k][z];
            for (int i = 0; i < kWavesA; i++) zn -= sh.zsum[i][k];
            uint32_t fv[4], tot = 0, nd = 0;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                fv[r] = uint32_t(lane + 64 * r) == z ? zn : hist[k][lane + 64 * r];
                tot += fv[r];
                nd += __popcll(__ballot(fv[r] > 0));
            }
            tot = wave_sum(tot);
            const bool zg = nd >= 2 && !(A.pol[k] == ZIPNN_AUTO && entropy_says_raw(fv, tot, head_z, m, p.L));
            if (lane == 0) {
                A.zn[k] = zn;
                if (zg) atomicOr(&A.build[1], 1u << k);
                // the marked groups hold a single value: forced ZG falls back to HUF
                if (nd < 2 && A.pol[k] == ZIPNN_ZG) atomicOr(&A.build[2], 1u << k);
            }
        }
        __syncthreads();
    }
    // 3. the code lengths, one wave per code: HUF, ZG, fallback HUF
    if (uint32_t(wv) < 3 * B) {
        const int v = wv / int(B), k = wv % int(B);
        if ((A.build[v] >> k) & 1) {
            __builtin_amdgcn_s_setprio(3);
            uint32_t fv[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const uint32_t s = uint32_t(lane) + 64 * r;
                fv[r] = v == 1 && s == A.z[k] ? A.zn[k] : hist[k][s];
            }
            const uint32_t bits = build_lengths(fv, S.pm[wv], p.L, v == 1 ? A.lens2[k] : A.lens[k]);
            // under AUTO a payload of at least its head and coded bits that
            // is no smaller than the raw bytes is out
            if (lane == 0) {
                A.T[v == 1][k] = bits;
                if (A.pol[k] != ZIPNN_AUTO || (v == 1 ? head_z : head) + (bits + 7) / 8 < m)
                    atomicOr(v == 1 ? &A.zgc : &A.hc, 1u << k);
            }
        }
    }
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    // AUTO with both candidates: a candidate that loses even at its best
    // (head + coded bits) against the other at its worst (plus two words
    // of padding per sub-stream) needs no count; ties go to HUF
    if (uint32_t(t) < B && A.pol[t] == ZIPNN_AUTO && ((A.hc & A.zgc) >> t & 1)) {
        const uint64_t h_lo = head + (A.T[0][t] + 7) / 8, h_hi = h_lo + 8 * W;
        const uint64_t z_lo = head_z + (A.T[1][t] + 7) / 8, z_hi = z_lo + 8 * W;
        if (z_hi < h_lo) atomicAnd(&A.hc, ~(1u << t));
        else if (h_hi <= z_lo) atomicAnd(&A.zgc, ~(1u << t));
    }
    __syncthreads();
    // Staged packing: the packer counts the words, so the sizes are needed
    // here only where the bounds of the candidates (head + coded bits, plus
    // two words of padding per sub-stream) leave AUTO's choice open.
    const bool staged = p.stage != nullptr;
    if (staged && uint32_t(t) < B && ((A.open >> t) & 1) && A.pol[t] == ZIPNN_AUTO) {
        const bool hc = (A.hc >> t) & 1, zgc = (A.zgc >> t) & 1;
        const uint64_t h_lo = head + (A.T[0][t] + 7) / 8, h_hi = h_lo + 8 * W;
        const uint64_t z_lo = head_z + (A.T[1][t] + 7) / 8, z_hi = z_lo + 8 * W;
        bool amb = false;
        uint64_t best_lo = m, best_hi = m;   // RAW
        if (hc) {
            if (h_hi < m) best_lo = h_lo, best_hi = h_hi;
            else if (h_lo < m) amb = true;
        }
        if (zgc && z_hi >= best_lo && z_lo < best_hi) amb = true;
        if (amb) atomicOr(&A.amb, 1u << t);
    }
    __syncthreads();
    const bool exact = !staged || A.amb != 0;
    // 4. the words of every candidate.  A lane group's steps are cut into
    // nseg ranges, one wave each, when there are fewer lane groups than waves.
    const uint32_t hc = __builtin_amdgcn_readfirstlane(A.hc), zgc = __builtin_amdgcn_readfirstlane(A.zgc);
    if ((hc | zgc) && exact) {
        const uint32_t Gtot = (m + p.g - 1) / p.g;
        const uint32_t steps = (Gtot - 1) / W + 1;   // of lane 0 of the first lane group, the most
        const uint32_t nseg = NG < uint32_t(kWavesA) ? uint32_t(kWavesA) / NG : 1u;
        const uint32_t per = (steps + nseg - 1) / nseg;
        auto steps_of = [&](uint32_t j, uint32_t s0, uint32_t s1, uint32_t (*out)[BB]) __attribute__((always_inline)) {
            switch (p.g) {
            case 2: count_steps<BB, 2>(in, src, base, hc, zgc, A.lens, A.lens2, A.z, j, s0, s1, W, m, out, xf); break;
            case 4: count_steps<BB, 4>(in, src, base, hc, zgc, A.lens, A.lens2, A.z, j, s0, s1, W, m, out, xf); break;
            default: count_steps<BB, 8>(in, src, base, hc, zgc, A.lens, A.lens2, A.z, j, s0, s1, W, m, out, xf); break;
            }
        };
        // the sums of the streams held in registers, if they are all there is
        bool from_held = false;
        uint32_t hsum[kHeld];
#pragma unroll
        for (int k = 0; k < kHeld; k++) hsum[k] = 0;
        if constexpr (HOLD > 0) {
            from_held = held && zgc == 0 && (hc >> kHeld) == 0;
            if (from_held) {
#pragma unroll
                for (int k = 0; k < kHeld; k++) {
                    if (!((hc >> k) & 1)) continue;
                    uint32_t bits = 0, last = 0;
#pragma unroll
                    for (int i0 = 0; i0 < HOLD; i0 += 4) {
                        uint32_t e[16];
#pragma unroll
                        for (int i = 0; i < 16; i++)
                            e[i] = A.lens[k][(hold[k][i0 + i / 4] >> (8 * (i % 4))) & 0xFFu];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int i = 0; i < 16; i++) bits += e[i];
                        last = e[14] + e[15];
                    }
                    hsum[k] = (bits << 5) | last;
                }
            }
        }
        // wave wv: range wv / NG of lane group wv % NG, or (nseg = 1) all of
        // lane groups wv, wv + kWavesA, ...
        for (uint32_t j0 = 0; j0 < NG; j0 += kWavesA) {
            const uint32_t sg = nseg > 1 ? uint32_t(wv) / NG : 0u, j = nseg > 1 ? uint32_t(wv) % NG : j0 + wv;
            uint32_t out[2][BB];
            const bool mine = nseg > 1 ? sg < nseg : j < NG;
            if (from_held) {
#pragma unroll
                for (int k = 0; k < BB; k++) out[0][k] = k < kHeld ? hsum[k < kHeld ? k : 0] : 0u, out[1][k] = 0;
            }
            if (mine && !from_held) steps_of(j, sg * per, min(steps, (sg + 1) * per), out);
            if (nseg > 1) {
                if (mine) {
#pragma unroll
                    for (uint32_t k = 0; k < B; k++) {
                        S.seg[0][k][t] = out[0][k];
                        S.seg[1][k][t] = out[1][k];
                    }
                }
                __syncthreads();
            }
            const uint32_t jw = j0 + wv;   // this wave sums up lane group jw
            if (jw >= NG) continue;
#pragma unroll
            for (int k = 0; k < BB; k++) {
#pragma unroll
                for (int v = 0; v < 2; v++) {
                    if (!(((v ? zgc : hc) >> k) & 1)) continue;
                    uint32_t bits = 0, last = 0;
                    if (nseg == 1) {
                        bits = out[v][k] >> 5;
                        last = out[v][k] & 31;
                    } else {
#pragma unroll 4
                        for (uint32_t g = 0; g < nseg; g++) {
                            const uint32_t x = S.seg[v][k][64 * (g * NG + jw) + lane];
                            bits += x >> 5;
                            last = x ? x & 31 : last;
                        }
                    }
                    // before each pair a lane holding fewer than 2L bits takes
                    // a word, so after that check 32 * taken - consumed lies in
                    // [2L, 2L + 31]: a lane takes ceil((consumed before its
                    // last pair + 2L) / 32) words in all, none without a pair
                    const uint32_t tot = wave_sum(bits ? (bits - last + 2 * p.L + 31) / 32 : 0u);
                    if (lane == 0) {
                        sh.lgw[v][k][jw] = tot;
                        atomicAdd(&A.words[v][k], tot);
                    }
                }
            }
        }
    }
    __syncthreads();
    // 5. the decision, the entry and the word counts of every open group.
    // Without exact sizes (staged, no open choice) the lower bounds decide
    // as the sizes would, and the entry's bytes are left to the packer's
    // counts.
    if (uint32_t(t) < B && ((A.open >> t) & 1)) {
        const int policy = A.pol[t];
        const bool hc1 = (A.hc >> t) & 1, zgc1 = (A.zgc >> t) & 1;
        const uint32_t size_h = exact ? head + 4 * A.words[0][t] : head + (A.T[0][t] + 7) / 8;
        const uint32_t size_z = exact ? head_z + 4 * A.words[1][t] : head_z + (A.T[1][t] + 7) / 8;
        int mode = kModeRaw;
        uint32_t bytes = m;
        if (policy == ZIPNN_AUTO) {
            if (hc1 && size_h < bytes) mode = kModeHuf, bytes = size_h;
            if (zgc1 && size_z < bytes) mode = kModeZg, bytes = size_z;
        } else if (zgc1) {
            mode = kModeZg, bytes = size_z;
        } else {
            mode = kModeHuf, bytes = size_h;
        }
        EncEntry e;
        e.pad = 0;
        e.mode = uint8_t(mode);
        e.rle = mode == kModeZg ? uint8_t(A.z[t]) : 0;
        e.bytes = (staged && mode != kModeRaw) ? 0u : bytes;
        entries[uint64_t(gc) * B + t] = e;
        if (mode != kModeRaw) atomicOr(&A.coded, 1u << t);
        if (mode == kModeZg) atomicOr(&A.fin, 1u << t);
    }
    __syncthreads();
    if (uint32_t(wv) < B && ((A.coded >> wv) & 1)) {
        const uint64_t ei = uint64_t(gc) * B + wv;
        const int v = (A.fin >> wv) & 1;
        reinterpret_cast<uint32_t*>(lens + ei * 256)[lane] =
            reinterpret_cast<const uint32_t*>(v ? A.lens2[wv] : A.lens[wv])[lane];
        if (!staged && uint32_t(lane) < NG) nwords[ei * 64 + lane] = sh.lgw[v][wv][lane];
    }
    // the ranges' sums of the chosen codes, for the packer (its ranges are these)
    if (p.segs && NT == kSegWords && NG < uint32_t(kWavesA)) {
#pragma unroll
        for (uint32_t k = 0; k < B; k++)
            if ((A.coded >> k) & 1)
                p.segs[(uint64_t(gc) * B + k) * kSegWords + t] = S.seg[(A.fin >> k) & 1][k][t];
    }
    __syncthreads();
}

// What bounds it: on full launches without HOLD the two reads of every chunk
// (the counting and the size pass; the second one misses L2, and the
// last-level cache serves it at 7.5 TB/s against HBM's 6.2): 5 GB of an 8B
// checkpoint (BF16, 256 KiB chunks) 1.37 ms, 7.3 TB/s of both reads.  With
// HOLD one read, 1.13 ms, and the waves of a CU halved by the registers: the
// chain of a chunk's phases shows.  (Four waves per chunk, one wave building
// each code in LDS, took 3.45 ms.)  256 MiB of FP32: 240, 108 and 72 us.  On
// small launches the chain count - code - sizes of one chunk: an 8 KiB tensor
// 98 -> 14 us, 32 chunks 146 -> 26 us.  The waves that classify and build
// codes run at raised priority: the others wait for them.
// A single tensor's descriptor comes in `one`, and the first workgroup writes
// it and its prefix to own[0] and own_prefix[0, 2) for the kernels that
// follow (own not null); by a kernel of its own before this one, an 8 KiB
// tensor's compress took 57 us, so 54.5 (8 MiB of BF16: 76.5, 73.1).
template <int BB, int NT, int HOLD>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(HOLD ? 4 : 8, 8))) void k_analyze(
    const EncDesc* __restrict__ descs, int n_desc, const uint32_t* __restrict__ chunk_prefix, uint32_t total_chunks,
    EncParams p, int phase, EncEntry* __restrict__ entries, uint8_t* __restrict__ lens, uint32_t* __restrict__ nwords,
    EncDesc one, EncDesc* own, uint32_t* own_prefix)
{
    __shared__ AnalyzeShared<BB, NT> sh;
    const uint32_t gc = chunk_of_block();
    if (gc >= total_chunks) return;
    uint32_t c = gc;
    if (own) {
        if (gc == 0 && threadIdx.x == 0) {
            *own = one;
            own_prefix[0] = 0;
            own_prefix[1] = total_chunks;
        }
    } else {
        const int di = find_desc(chunk_prefix, n_desc, gc);
        one = descs[di];
        c = gc - chunk_prefix[di];
    }
    analyze_chunk<BB, NT, HOLD>(gc, one, c, p, phase, entries, lens, nwords, sh);
}

constexpr int kPlaceThreads = 1024;
constexpr int kPlaceVec = 4;   // neighbouring entries per thread

// Exclusive scan over the workgroup: this thread's start, `carry` advanced by
// the total (both in every thread).
__device__ inline uint64_t block_scan(uint64_t v, uint64_t& carry, uint64_t* red)
{
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint64_t inc = v;
#pragma unroll
    for (int dd = 1; dd < 64; dd <<= 1) {
        const uint64_t o = __shfl_up(inc, dd, 64);
        if (lane >= dd) inc += o;
    }
    if (lane == 63) red[wv] = inc;
    __syncthreads();
    uint64_t pre = carry, tot = carry;
    for (int i = 0; i < kPlaceThreads / 64; i++) {
        pre += i < wv ? red[i] : 0;
        tot += red[i];
    }
    __syncthreads();
    carry = tot;
    return pre + inc - v;
}

// One workgroup per tensor: offsets of its entries (128-byte aligned, in
// chunk-major order) and the tensor's container size.  The last workgroup to
// finish then lays the tensors' containers out back to back in the arena
// (each at a kPayAlign-aligned offset, in tensor order): it sets each
// descriptor's dst, writes every header, and records the arena offsets (n+1
// of them, in host_off too unless null: host memory).  If the arena is too
// small nothing is written and the recorded end says so.  descs[0].pad
// counts the workgroups; it is zero before and after.  4096 entries a round:
// the 8016 of a checkpoint's embedding, 256 a round, took 33 us and the
// arena 5 us in a launch of its own; now 21 us together.
__global__ __launch_bounds__(kPlaceThreads) void k_place(EncDesc* descs, int n_desc, EncParams p, EncEntry* entries,
                                                         uint64_t* offsets, uint64_t* totals, const uint32_t* nwords,
                                                         uint8_t* arena, uint64_t cap, uint64_t* arena_off,
                                                         uint64_t* host_off)
{
    __shared__ uint64_t red[kPlaceThreads / 64];
    __shared__ uint32_t zg, last;
    const EncDesc d = descs[blockIdx.x];
    const int t = threadIdx.x;
    const uint32_t B = p.B;
    const uint64_t ne = uint64_t(d.n_chunks) * B;
    const uint64_t e_first = uint64_t(d.chunk0) * B;
    uint64_t carry = 0;
    if (t == 0) zg = 0;
    __syncthreads();
    for (uint64_t b0 = 0; b0 < ne; b0 += kPlaceThreads * kPlaceVec) {
        const uint64_t e0 = b0 + uint64_t(t) * kPlaceVec;
        uint64_t sz[kPlaceVec], sum = 0;
#pragma unroll
        for (int v = 0; v < kPlaceVec; v++) {
            const uint64_t e = e0 + v;
            sz[v] = 0;
            if (e < ne) {
                EncEntry en = entries[e_first + e];
                if (p.stage && (en.mode == kModeHuf || en.mode == kModeZg)) {
                    // staged: the payload's size from the packer's word counts
                    const uint32_t E = p.chunk / B;
                    const uint32_t m = uint32_t(min(uint64_t(E), d.n - uint64_t(e / B) * E));
                    const uint32_t W = (m + p.S - 1) / p.S, NG = (W + 63) / 64;
                    uint32_t words = 0;
                    for (uint32_t j = 0; j < NG; j++) words += nwords[(e_first + e) * 64 + j];
                    en.bytes = huf_head(W) + (en.mode == kModeZg ? zg_bitmap(m, p.g) : 0u) + 4 * words;
                    entries[e_first + e].bytes = en.bytes;
                }
                sz[v] = align_pay(en.bytes);
                if (en.mode == kModeZg) zg = 1;
            }
            sum += sz[v];
        }
        uint64_t at = block_scan(sum, carry, red);
#pragma unroll
        for (int v = 0; v < kPlaceVec; v++) {
            if (e0 + v < ne) offsets[e_first + e0 + v] = at;
            at += sz[v];
        }
    }
    __syncthreads();
    const uint64_t total1 = payload_base_of(d.n_chunks, B) + carry;
    if (t == 0) {
        totals[blockIdx.x] = total1;
        if (n_desc > 1) {
            descs[blockIdx.x].has_zg = zg;
            __threadfence();
            last = atomicAdd(&descs[0].pad, 1u) == uint32_t(n_desc) - 1;
        }
    }
    // a tensor's container: descriptor and header
    auto write_header = [&](int i, EncDesc x, uint64_t total, uint64_t at, bool fits) {
        x.dst = arena + at;
        x.dst_cap = fits ? total : 0;   // pack skips tensors whose dst_cap is short
        x.pad = 0;
        descs[i] = x;
        if (!fits) return;
        uint32_t h[16];
        h[0] = 0x314E4E5Au;
        h[1] = 1u | (p.dtype << 16) | (B << 24);
        h[2] = uint32_t(x.n);
        h[3] = uint32_t(x.n >> 32);
        h[4] = p.chunk;
        h[5] = p.S | (p.g << 16) | (p.L << 24);
        h[6] = (x.base ? kFlagDelta : 0u) | (x.has_zg ? kFlagZg : 0u) | (p.flags & kFlagExp);
        h[7] = x.n_chunks;
        h[8] = uint32_t(total);
        h[9] = uint32_t(total >> 32);
        h[10] = 0;
        for (uint32_t k = 0; k < B; k++) h[10] |= uint32_t(p.policy[k]) << (8 * k);
        h[11] = p.skip;   // byte 44: the probe interval
        for (int y = 12; y < 16; y++) h[y] = 0;
        uint4* o = (uint4*)x.dst;
        for (int y = 0; y < 4; y++) o[y] = make_uint4(h[4 * y], h[4 * y + 1], h[4 * y + 2], h[4 * y + 3]);
        // zero padding between the map and the aligned payload area
        const uint64_t map_end = 64 + 16ull * x.n_chunks * B, pb = payload_base_of(x.n_chunks, B);
        for (uint64_t y = map_end / 16; y < pb / 16; y++) o[y] = make_uint4(0, 0, 0, 0);
    };
    if (n_desc == 1) {   // nothing to wait for or read back
        if (t == 0) {
            arena_off[0] = 0;
            arena_off[1] = total1;
            if (host_off) host_off[0] = 0, host_off[1] = total1;
            EncDesc x = d;
            x.has_zg = zg;
            write_header(0, x, total1, 0, total1 <= cap);
        }
        return;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    carry = 0;
    uint64_t end = 0;   // the last container needs only its own bytes, not the alignment
    for (int b0 = 0; b0 < n_desc; b0 += kPlaceThreads) {
        const int i = b0 + t;
        const uint64_t total = i < n_desc ? totals[i] : 0;
        const uint64_t at = block_scan(align_pay(total), carry, red);
        if (i < n_desc) {
            arena_off[i] = at;
            if (host_off) host_off[i] = at;
        }
        if (i == n_desc - 1) red[0] = at + total;
        __syncthreads();
        if (b0 + kPlaceThreads >= n_desc) end = red[0];
        __syncthreads();
    }
    if (t == 0) {
        arena_off[n_desc] = end;
        if (host_off) host_off[n_desc] = end;
    }
    const bool fits = end <= cap;
    for (int i = t; i < n_desc; i += kPlaceThreads) {
        write_header(i, descs[i], totals[i], arena_off[i], fits);
    }
}

struct PackLds {
    uint32_t rcode[4][256];     // reversed code | length << 27 (0 for absent symbols)
    uint64_t pay[4];            // absolute payload offset of each stream
    uint32_t mode[4];
    uint32_t bytes[4];
    uint32_t z[4];              // ZG fill value
    uint32_t wpre[4][65];       // lane-group word prefix per stream
    alignas(16) uint32_t cnt[4][kMaxL + 1][kWaves];   // symbols of each code length, per wave
};

constexpr uint32_t kLenShift = 27;              // code length's place in a packer code entry

// f(integral_constant<int, k>) for k = 0 .. N-1: per-stream state is then
// picked at compile time and stays in registers
template <int N, class F>
__device__ __attribute__((always_inline)) inline void for_streams(F&& f)
{
    if constexpr (N > 0) {
        for_streams<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}
constexpr int kNever = -0x7FFFFFFF;             // packer: no lane holds fewer bits
constexpr uint32_t kNoStore = 0x80000000u;      // buffer offset past every resource: the store is dropped

// Write the words of lane group j of every coded stream of one chunk (bit k
// of cm; with bit k of zm a ZG stream with fill value P.z[k], whose unmarked
// groups are not coded) in one pass over the chunk's groups, in lock-step
// over the steps and pairs of the layout.  Per stream, at every pair of its
// coded groups a lane first takes a word if it holds fewer than 2L bits: the
// word's place is the lane group's cursor plus the lane's rank among the
// pair's takers.  Then the pair's codes join the lane's bits, and a word that
// is complete is stored at the oldest place taken for it.  With held =
// 32 * taken - consumed and nacc the coded bits not yet stored, held + nacc is
// 32 times the words taken and not yet stored: a taken word lies wholly past
// what the lane has consumed, so it is finished later, and at most two are
// ever unfinished (after each take held lies in [2L, 2L + 31]).  After the
// lane's last pair the unfinished words are stored: the partial one, then
// zero.  The stores go through a buffer resource over the lane group's words,
// so a place past them (which the analysis's counts never give) is dropped.
// Steps in which every lane has a full group run without per-lane group
// counts; the raw byte groups of small groups are copied on the same pass.
// Staged (stage_lg > 0): stream k's payload area is the staging slot at
// P.pay[k], lane group j's words start at stage_bm + j * stage_lg, a ZG
// bitmap at the slot's start; the lane group's word count goes to
// nw_out[k * 64 + j].
// A range [s0, s1) of the lane group's steps can be packed on its own: with c
// a lane's code bits and l those of its last pair before the range (summed
// here from the ranges' sums in `seg`, this being range sg), it has taken
// ceil((c - l + 2L) / 32) words, c mod 32 bits lie in its first unfinished
// one, and the lanes' words add up to the cursor.  A word belongs to the range
// that takes it: the words taken before are completed but not stored here,
// and after s1 the lanes go on, taking none, until theirs are complete.
template <int B, int G, bool XB, bool SPEC>
__device__ __attribute__((always_inline)) void pack_lane_group(const uint8_t* src, const uint8_t* base, uint32_t cm,
                                                               uint32_t zm, const PackLds& P, uint32_t L, uint32_t j,
                                                               uint32_t W, uint32_t m, bool xf, bool fuse_bitmap,
                                                               uint32_t rawmask, uint8_t* dst, uint32_t stage_lg,
                                                               uint32_t stage_bm, uint32_t* nw_out, uint32_t s0,
                                                               uint32_t s1, uint32_t sg, const uint32_t* seg)
{
    constexpr int NB = B * G;
    constexpr int NW = NB >= 4 ? NB / 4 : 1;
    // groups of input prefetched ahead (two for 4-byte words: fewer registers)
    constexpr uint32_t kPf = B == 4 ? 2 : 4;
    cm = __builtin_amdgcn_readfirstlane(cm);
    zm = __builtin_amdgcn_readfirstlane(zm);
    // the lane group is the wave's: uniform, so every value derived from it
    // (a buffer resource above all) stays in scalar registers
    j = __builtin_amdgcn_readfirstlane(j);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t w = 64 * j + lane;
    const int twoL = int(2 * L);
    const uint32_t Gtot = (m + G - 1) / G, Gfull = m / G, rem = m - Gfull * G;
    const uint32_t ng = (w < W && w < Gtot) ? (Gtot - 1 - w) / W + 1 : 0;
    const uint32_t ng_max = __builtin_amdgcn_readfirstlane(ng);   // lane 0 has the most
    // full groups of the lane group's last lane: every lane has at least these
    const uint32_t w_last = min(W, 64 * j + 64) - 1;
    const uint32_t nfull_all = w_last < Gfull ? (Gfull - 1 - w_last) / W + 1 : 0;
    s0 = __builtin_amdgcn_readfirstlane(s0);
    s1 = min(uint32_t(__builtin_amdgcn_readfirstlane(s1)), ng_max);
    const uint32_t n_fast = min(s1, nfull_all) > s0 ? s0 + (min(s1, nfull_all) - s0) / kPf * kPf : s0;
    const uint32_t head = huf_head(W), bm = zg_bitmap(m, G);
    // lanes past the last sub-stream: their loads and stores are out of range
    // and they never need a word
    const bool act = w < W;
    uint32_t zrep[B];   // a ZG stream's fill value in every byte
#pragma unroll
    for (int k = 0; k < B; k++) zrep[k] = __builtin_amdgcn_readfirstlane(P.z[k] * 0x01010101u);
    const uint32_t w_in = act ? w * NB : kNoStore, w_raw = act ? w * G : kNoStore;
    const __amdgpu_buffer_rsrc_t rsrc = in_rsrc(src, m * B);
    const __amdgpu_buffer_rsrc_t rbase = in_rsrc(base ? base : src, base ? m * B : 0u);   // no base: zeros
    auto uni64 = [](uint64_t v) {
        return uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v)))) |
               (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v >> 32)))) << 32);
    };
    // per coded stream: its words of this lane group (a buffer resource), the
    // fused bitmap, and the lock-step state
    struct Stream {
        __amdgpu_buffer_rsrc_t out;
        uint8_t* bmw;   // the fused bitmap
        uint32_t cur, alo, ahi, nacc, s0, s1;
        int held;
    };
    Stream st0, st1, st2, st3;
    auto S = [&](auto kc) __attribute__((always_inline)) -> Stream& {
        constexpr int k = decltype(kc)::value;
        if constexpr (k == 0) return st0;
        else if constexpr (k == 1) return st1;
        else if constexpr (k == 2) return st2;
        else return st3;
    };
    for_streams<B>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        Stream& x = S(kc);
        const uint32_t zb = (zm >> k) & 1;
        const uint64_t pk = uni64(P.pay[k]);
        const bool staged = stage_lg != 0;
        const uint32_t w0 = staged ? j * (stage_lg / 4) : __builtin_amdgcn_readfirstlane(P.wpre[k][j]);
        const uint32_t nw = staged ? stage_lg / 4 : __builtin_amdgcn_readfirstlane(P.wpre[k][j + 1]) - w0;
        const uint32_t lead = staged ? stage_bm : head + (zb ? bm : 0u);   // bytes before the words
        const uint64_t wa = uni64(uint64_t(dst + pk + lead) + 4ull * w0);
        x.out = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(wa), (short)0,
                                                  int(((cm >> k) & 1) ? 4 * nw : 0u), 0x00020000);
        x.bmw = (zb && fuse_bitmap) ? dst + pk + (staged ? 0u : head) : nullptr;
        x.cur = x.alo = x.ahi = x.nacc = 0;
        x.s0 = x.s1 = kNoStore;
        x.held = 0;
        if (sg && ((cm >> k) & 1)) {
            const uint32_t NG = (W + 63) / 64;
            uint32_t c = 0, last = 0;
            for (uint32_t g = 0; g < sg; g++) {
                const uint32_t y = seg[k * kSegWords + 64 * (g * NG + j) + lane];
                c += y >> 5;
                last = y ? y & 31 : last;
            }
            const uint32_t taken = c ? (c - last + 2 * L + 31) / 32 : 0u;
            x.cur = wave_sum(taken);
            x.nacc = c & 31;
            x.held = int(32 * taken - c);
        }
        if (!act) x.held = 1 << 30;
    });
    // raw byte groups copied here (groups of at most 4 bytes: b16 / b32
    // stores through one resource over the chunk's payloads, which are
    // consecutive, and a scalar offset per raw group)
    constexpr bool kFuseRaw = G <= 4 && B * G <= 16;
    const uint64_t raw0 = uni64(uint64_t(dst + P.pay[0]));
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(raw0), (short)0,
        int(__builtin_amdgcn_readfirstlane(rawmask ? uint32_t(P.pay[B - 1] - P.pay[0]) + m : 0u)), 0x00020000);
    // one pair of stream k: entries c0, c1 (zero for a symbol that is not
    // coded); a lane takes a word if it holds fewer than thr bits (2L, or
    // kNever where it takes no part)
    auto pair = [&](auto kc, uint32_t c0, uint32_t c1, int thr, auto take_c) __attribute__((always_inline)) {
        constexpr bool TAKE = decltype(take_c)::value;
        Stream& x = S(kc);
        if constexpr (TAKE) {
            const bool need = x.held < thr;
            const uint64_t msk = __ballot(need);
            const uint32_t place = 4u * __builtin_amdgcn_mbcnt_hi(uint32_t(msk >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo(uint32_t(msk), x.cur));
            // nothing pending: held + nacc = 0, i.e. held = 0 (nacc < 32)
            const bool empty = x.held == 0;
            x.s0 = (need && empty) ? place : x.s0;
            x.s1 = need ? place : x.s1;
            x.held += need ? 32 : 0;
            x.cur += uint32_t(__popcll(msk));
        }
        // the two codes side by side (the lengths sit in bits 27..31 of an
        // entry, so the entries' sum carries the sum of the lengths, <= 2L)
        const uint32_t l0 = c0 >> kLenShift, l = (c0 + c1) >> kLenShift;
        const uint32_t pc = (c0 | (c1 << l0)) & ((1u << kLenShift) - 1);
        const uint64_t v = uint64_t(pc) << x.nacc;
        x.alo |= uint32_t(v);
        x.ahi |= uint32_t(v >> 32);
        x.nacc += l;
        x.held -= int(l);
        // at most one word completes per pair (nacc < 32 + 2L)
        const bool full = x.nacc >= 32;
        __builtin_amdgcn_raw_buffer_store_b32(x.alo, x.out, full ? x.s0 : kNoStore, 0, 0);
        x.alo = full ? x.ahi : x.alo;
        x.ahi = 0;   // fewer than 32 bits left: none above the low word
        x.nacc &= 31u;
        x.s0 = full ? x.s1 : x.s0;
        if constexpr (!TAKE) x.s1 = full ? kNoStore : x.s1;
    };
    // one step (group e of every lane); FAST: every lane has a full group
    auto step = [&](uint32_t e, const uint32_t* wd, auto fast_c, auto take_c, auto cm_c, auto zm_c)
                    __attribute__((always_inline)) {
        // the coded and the ZG streams, known here or (-1) not
        constexpr int CM = decltype(cm_c)::value, ZM = decltype(zm_c)::value;
        const uint32_t cms = CM >= 0 ? uint32_t(CM) : cm, zms = ZM >= 0 ? uint32_t(ZM) : zm;
        constexpr bool FAST = decltype(fast_c)::value;
        constexpr bool TAKE = decltype(take_c)::value;   // else only words already taken are completed
        const bool has = FAST || e < ng;
        const uint32_t ecnt = FAST ? uint32_t(G) : (has ? (w + e * W < Gfull ? G : rem) : 0u);
        if constexpr (kFuseRaw && TAKE) {
            if (rawmask && has) {
                const uint32_t q0 = w_raw + e * W * G;
                for_streams<B>([&](auto rc) __attribute__((always_inline)) {
                    constexpr int r = decltype(rc)::value;
                    if (!((rawmask >> r) & 1)) return;
                    const uint32_t roff = __builtin_amdgcn_readfirstlane(uint32_t(P.pay[r] - P.pay[0]));
                    if (FAST || ecnt == G) {
                        const uint32_t v = gather_stream<B, G>(wd, r);
                        if constexpr (G == 2) __builtin_amdgcn_raw_buffer_store_b16(uint16_t(v), rr, q0, roff, kNt);
                        else __builtin_amdgcn_raw_buffer_store_b32(v, rr, q0, roff, kNt);
                    } else {
                        for (uint32_t i = 0; i < ecnt; i++)
                            __builtin_amdgcn_raw_buffer_store_b8(uint8_t(sym_of<B>(wd, r, int(i))), rr, q0 + i, roff,
                                                                 0);
                    }
                });
            }
        }
        for_streams<B>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            if (!((cms >> k) & 1)) return;
            // the pairs of a group of gcnt coded symbols; in a fast step, all
            // G of them, or none where `on` (all ones or zero) is zero.  The
            // table is read in either case and the entries are masked: no
            // branch per pair, no flag turned into a number for the ballot.
            auto pairs = [&](uint32_t gcnt, uint32_t on) __attribute__((always_inline)) {
                const int thr_on = on ? twoL : kNever;
#pragma unroll
                for (int pr = 0; pr < G / 2; pr++) {
                    const uint32_t c0 = P.rcode[k][sym_of<B>(wd, k, 2 * pr)];
                    const uint32_t c1 = P.rcode[k][sym_of<B>(wd, k, 2 * pr + 1)];
                    if constexpr (FAST) {
                        pair(kc, c0 & on, c1 & on, thr_on, take_c);
                    } else {
                        const bool p0 = 2u * pr < gcnt, p1 = 2u * pr + 1 < gcnt;
                        pair(kc, p0 ? c0 : 0u, p1 ? c1 : 0u, p0 ? twoL : kNever, take_c);
                    }
                }
            };
            if ((zms >> k) & 1) {
                bool mk;
                if constexpr (FAST) {
                    // lanes past the last sub-stream may count as marked:
                    // they take no word and their stores are out of range
                    // (a fused bitmap has no such lanes)
                    uint32_t diff = 0;
#pragma unroll
                    for (int x = 0; x < NW; x++) diff |= (wd[x] ^ zrep[k]) & stream_bytes<B>(k, NB < 4 ? NB : 4);
                    mk = diff != 0;
                } else {
                    mk = has && marked<B, G>(wd, k, ecnt, P.z[k]);
                }
                const uint64_t bits = __ballot(mk);
                // ZG with W a multiple of 64: the 64 bits of this lane
                // group's step e are one aligned word of the bitmap
                if (TAKE && fuse_bitmap && lane == 0) gst(S(kc).bmw + 8 * (j + e * (W / 64)), bits);
                // where no lane of the wave holds a marked group, the pairs
                // would take no word and add no bits: they are skipped
                if (bits) pairs(mk ? ecnt : 0u, mk ? ~0u : 0u);
            } else {
                pairs(ecnt, ~0u);   // in a fast step, G: no per-lane conditions
            }
        });
    };
    // step e's bytes of every lane (zeros past the end), fetched kPf steps
    // ahead; taken into words when the step comes, so that nothing waits for
    // them before.  The tensor's partial last group is read element by element.
    struct Fetch {
        uint32_t x[NW], y[XB ? NW : 1];
    };
    Fetch pf[kPf];
    auto load = [&](uint32_t e, Fetch& f) __attribute__((always_inline)) {
        buf_in<NB, kNt>(rsrc, w_in + e * W * NB, 0, f.x);
        if constexpr (XB) buf_in<NB, kNt>(rbase, w_in + e * W * NB, 0, f.y);
    };
    auto words = [&](const Fetch& f, uint32_t* wd) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NW; x++) {
            wd[x] = f.x[x];
            if constexpr (XB) wd[x] ^= f.y[x];
        }
        if (xf) {
            asm volatile("");   // a branch: computed and selected, it is 12 instructions of every step
#pragma unroll
            for (int x = 0; x < NW; x++) wd[x] = exp_fwd<B>(wd[x]);
        }
    };
    auto last_words = [&](uint32_t e, uint32_t* wd) __attribute__((always_inline)) {
        if (rem && act && w + e * W == Gfull) group_words<B, G>(src, base, Gfull, m, wd, xf);
    };
    using T = std::integral_constant<bool, true>;
    using F = std::integral_constant<bool, false>;
#pragma unroll
    for (uint32_t u = 0; u < kPf; u++) load(s0 + u, pf[u]);
    // the first loads are waited for once, here: left pending, their order
    // would set how far back the loop's waits reach
#pragma unroll
    for (uint32_t u = 0; u < kPf; u++) {
#pragma unroll
        for (int x = 0; x < NW; x++) {
            asm volatile("" : "+v"(pf[u].x[x]));
            if constexpr (XB) asm volatile("" : "+v"(pf[u].y[x]));
        }
    }
    // A copy of the loop for a BF16 chunk's common set (exponent coded, the
    // other byte group raw): with the set known only at run time every stream's
    // state is moved at the ends of its branches (a 5 GB shard's encode, us:
    // 2880 without, 2869 with). On a delta such a copy for both byte groups
    // coded and unmarked spills: 1590 without, 1605 with.
    auto fast = [&](auto cm_c, auto zm_c) __attribute__((always_inline)) {
        for (uint32_t j0 = s0; j0 < n_fast; j0 += kPf) {
#pragma unroll
            for (uint32_t u = 0; u < kPf; u++) {
                uint32_t cw[NW];
                words(pf[u], cw);
                load(j0 + u + kPf, pf[u]);
                step(j0 + u, cw, T{}, T{}, cm_c, zm_c);
            }
        }
    };
    using Any = std::integral_constant<int, -1>;
    bool done = false;
    if constexpr (SPEC && B == 2 && !XB) {
        if (cm == 1 && zm == 0) {
            fast(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{});
            done = true;
        }
    }
    if (!done) fast(Any{}, Any{});
    // the steps without a full group in every lane, then (after s1) those that
    // complete the words taken in this range
    bool ended = false;
    for (uint32_t j0 = n_fast; j0 < ng_max && !ended; j0 += kPf) {
#pragma unroll
        for (uint32_t u = 0; u < kPf; u++) {
            const uint32_t jj = j0 + u;
            if (jj >= ng_max || ended) continue;
            if (jj == s1)
                for_streams<B>([&](auto kc) __attribute__((always_inline)) {
                    Stream& x = S(kc);
                    const int pend = act ? (x.held + int(x.nacc)) >> 5 : 0;
                    x.s0 = pend > 0 ? x.s0 : kNoStore;
                    x.s1 = pend > 1 ? x.s1 : kNoStore;
                });
            if (jj >= s1) {
                bool open = false;
                for_streams<B>([&](auto kc) __attribute__((always_inline)) {
                    constexpr int k = decltype(kc)::value;
                    const Stream& x = S(kc);
                    if ((cm >> k) & 1) open |= act && (x.held + int(x.nacc)) >> 5 > 0;
                });
                if (__ballot(open) == 0) {
                    ended = true;
                    continue;
                }
            }
            uint32_t cw[NW];
            words(pf[u], cw);
            last_words(jj, cw);
            load(jj + kPf, pf[u]);
            if (jj < s1) step(jj, cw, F{}, T{}, Any{}, Any{});
            else step(jj, cw, F{}, F{}, Any{}, Any{});
        }
    }
    // the lane's unfinished words: the partial one (zero bits if none), then zero
    for_streams<B>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        if (!((cm >> k) & 1)) return;
        const Stream& x = S(kc);
        const int pend = (x.held + int(x.nacc)) >> 5;
        __builtin_amdgcn_raw_buffer_store_b32(x.alo, x.out, pend > 0 ? x.s0 : kNoStore, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(0u, x.out, pend > 1 ? x.s1 : kNoStore, 0, 0);
        // staged: the words this lane group took (the cursor is uniform)
        if (nw_out && lane == 0) gst(reinterpret_cast<uint8_t*>(nw_out + k * 64 + j), x.cur);
    });
}

// The group bitmap of a ZG stream: wave v writes 64-bit words x = v, v+4, ...
// of the bm bytes (lane l tests group 64x + l); bits past the last group and
// the padding are zero.
template <int B, int G, int NT>
__device__ void pack_bitmap(const uint8_t* src, const uint8_t* base, int k, uint32_t z, uint32_t m, uint32_t bm,
                            uint8_t* dst, bool xf)
{
    constexpr int NB = B * G;
    constexpr int NW = NB >= 4 ? NB / 4 : 1;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t Gtot = (m + G - 1) / G;
    for (uint32_t x = threadIdx.x >> 6; x < bm / 8; x += NT / 64) {
        const uint32_t q = 64 * x + lane;
        bool mk = false;
        if (q < Gtot) {
            uint32_t wd[NW];
            group_words<B, G>(src, base, q, m, wd, xf);
            mk = marked<B, G>(wd, k, min(uint32_t(G), m - q * G), z);
        }
        const uint64_t bits = __ballot(mk);
        if (lane == 0) gst(dst + 8 * x, bits);
    }
}

// Raw groups of one chunk: thread t copies elements [16u, 16u+16) of every
// RAW stream with one 16-byte store each, then the zero padding.  With
// pad_only the packer of a coded group copies the elements, and only the
// padding is written here.
template <int B, int NT>
__device__ void pack_raw(const uint8_t* src, const uint8_t* base, uint8_t* dst, const PackLds& P, uint32_t m, bool xf,
                         bool pad_only)
{
    uint32_t rawmask = 0;
    for (int k = 0; k < B; k++)
        if (P.mode[k] == kModeRaw) rawmask |= 1u << k;
    if (!rawmask) return;
    if (pad_only) {
        for (uint32_t e = m + threadIdx.x; e < uint32_t(align_pay(m)); e += NT)
#pragma unroll
            for (int k = 0; k < B; k++)
                if ((rawmask >> k) & 1) gst(dst + P.pay[k] + e, uint8_t(0));
        return;
    }
    const uint32_t units = m / 16;
    constexpr uint32_t RB = B == 4 ? 2 : (B == 2 ? 4 : 8);   // units in flight per thread
    for (uint32_t u0 = threadIdx.x; u0 < units; u0 += RB * NT) {
        uint32_t wds[RB][4 * B];
#pragma unroll
        for (uint32_t r = 0; r < RB; r++) {
            const uint32_t u = u0 + r * NT;
            if (u < units) {
                loadNB<16 * B>(src + uint64_t(u) * 16 * B, wds[r]);
                if (base) {
                    uint32_t bw[4 * B];
                    loadNB<16 * B>(base + uint64_t(u) * 16 * B, bw);
#pragma unroll
                    for (int x = 0; x < 4 * B; x++) wds[r][x] ^= bw[x];
                }
                if (xf)
#pragma unroll
                    for (int x = 0; x < 4 * B; x++) wds[r][x] = exp_fwd<B>(wds[r][x]);
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < RB; r++) {
            const uint32_t u = u0 + r * NT;
#pragma unroll
            for (int k = 0; k < B; k++) {
                if (!((rawmask >> k) & 1) || u >= units) continue;
                uint32_t o[4] = {0, 0, 0, 0};
#pragma unroll
                for (int i = 0; i < 16; i++) o[i >> 2] |= sym_of<B>(wds[r], k, i) << (8 * (i & 3));
                gst(dst + P.pay[k] + 16 * u, u32x4{o[0], o[1], o[2], o[3]});
            }
        }
    }
    // tail elements, then zero padding to the payload alignment
    for (uint32_t e = units * 16 + threadIdx.x; e < uint32_t(align_pay(m)); e += NT) {
        const uint32_t v = e < m ? element_word<B>(src, base, e, xf) : 0u;
#pragma unroll
        for (int k = 0; k < B; k++)
            if ((rawmask >> k) & 1) gst(dst + P.pay[k] + e, uint8_t(v >> (8 * (B - 1 - k))));
    }
}

// The packing of chunk gc by one workgroup (into its container, or staged
// into its staging slots with the word counts).
template <int BB, int GG, bool XB, int NT>
__device__ __attribute__((always_inline)) void pack_chunk(uint32_t gc, const EncDesc* __restrict__ descs, int n_desc,
                                                          const uint32_t* __restrict__ chunk_prefix, const EncParams& p,
                                                          const EncEntry* __restrict__ entries,
                                                          const uint8_t* __restrict__ lens,
                                                          const uint64_t* __restrict__ offsets,
                                                          const uint64_t* __restrict__ totals,
                                                          uint32_t* __restrict__ nwords, PackLds& P)
{
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    constexpr uint32_t B = BB;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t len[B], rank[B];   // this thread's symbol: code length, place among its length in the wave
#pragma unroll
    for (uint32_t k = 0; k < B; k++) len[k] = rank[k] = 0;
    // staged: the payloads go to the staging slots (their places in the
    // container are not known yet) and the word counts come out
    const bool staged = p.stage != nullptr;
    const int di = find_desc(chunk_prefix, n_desc, gc);
    const EncDesc d = descs[di];
    if (!staged && totals[di] > d.dst_cap) return;   // too small: the host reports it
    const uint32_t c = gc - chunk_prefix[di];
    const uint32_t E = p.chunk / B;
    const uint64_t e0 = uint64_t(c) * E;
    const uint32_t m = uint32_t(min(uint64_t(E), d.n - e0));
    const uint32_t W = (m + p.S - 1) / p.S;
    const uint32_t NG = (W + 63) / 64;
    const uint32_t head = huf_head(W);
    const uint64_t payload_base = payload_base_of(d.n_chunks, B);
#pragma unroll
    for (uint32_t k = 0; k < B; k++) {
        const uint64_t ei = uint64_t(gc) * B + k;
        const EncEntry en = entries[ei];
        if (t == 0 && staged) {
            P.mode[k] = en.mode;
            P.bytes[k] = en.bytes;
            P.pay[k] = ei * p.stage_chunk;
        } else if (t == 0) {
            P.mode[k] = en.mode;
            P.bytes[k] = en.bytes;
            P.pay[k] = payload_base + offsets[ei];
            // this chunk's map entry
            gst(d.dst + 64 + 16 * (uint64_t(c) * B + k),
                u32x4{uint32_t(offsets[ei]), uint32_t(offsets[ei] >> 32), en.bytes,
                      uint32_t(en.mode) | (uint32_t(en.rle) << 8)});
        }
        if (t == 0) P.z[k] = en.rle;
        if (en.mode == kModeHuf || en.mode == kModeZg) {
            len[k] = t < 256 ? lens[ei * 256 + t] : 0u;
            // symbols of each length in this wave; rank: equal lengths below
            for (uint32_t l = 1; l <= p.L; l++) {
                const uint64_t msk = __ballot(len[k] == l);
                if (len[k] == l) rank[k] = __popcll(msk & lt_mask);
                if (lane == 0 && wv < 4) P.cnt[k][l][wv] = uint32_t(__popcll(msk));
            }
            if (t < 64 && !staged) {
                const uint32_t nw = uint32_t(t) < NG ? nwords[ei * 64 + t] : 0u;
                uint32_t inc = nw;
#pragma unroll
                for (int dd = 1; dd < 64; dd <<= 1) {
                    uint32_t o = __shfl_up(inc, dd, 64);
                    if (t >= dd) inc += o;
                }
                P.wpre[k][t + 1] = inc;
                if (t == 0) P.wpre[k][0] = 0;
            }
        }
    }
    __syncthreads();
    // canonical codes (RFC 1951 §3.2.2): the first code of each length follows
    // from the counts of the shorter ones; within a length the codes follow
    // the symbol order
#pragma unroll
    for (uint32_t k = 0; k < B; k++) {
        if (P.mode[k] != kModeHuf && P.mode[k] != kModeZg) continue;
        uint32_t first = 0, prev = 0, code = 0;
        for (uint32_t l = 1; l <= p.L; l++) {
            const uint4 c4 = *reinterpret_cast<const uint4*>(P.cnt[k][l]);
            first = (first + prev) << 1;
            prev = c4.x + c4.y + c4.z + c4.w;
            if (len[k] == l)
                code = first + rank[k] + (wv > 0 ? c4.x : 0u) + (wv > 1 ? c4.y : 0u) + (wv > 2 ? c4.z : 0u);
        }
        if (t < 256) P.rcode[k][t] = len[k] ? ((__brev(code) >> (32 - len[k])) | (len[k] << kLenShift)) : 0u;
    }
    __syncthreads();
    const uint8_t* src = d.src + e0 * B;
    const uint8_t* base = d.base ? d.base + e0 * B : nullptr;
    uint8_t* dst = staged ? p.stage : d.dst;
    const bool xf = (p.flags & kFlagExp) != 0;
    // the coded groups (HUF and ZG) are packed in one pass, which also
    // copies the raw groups when groups are small (at most 4 bytes)
    uint32_t rawmask = 0, cm = 0, zm = 0;
    for (uint32_t k = 0; k < B; k++) {
        if (P.mode[k] == kModeRaw) rawmask |= 1u << k;
        if (P.mode[k] == kModeHuf || P.mode[k] == kModeZg) cm |= 1u << k;
        if (P.mode[k] == kModeZg) zm |= 1u << k;
    }
    const bool fuse_raw = GG <= 4 && BB * GG <= 16 && cm != 0;
    pack_raw<BB, NT>(src, base, dst, P, m, xf, fuse_raw);
    // with W a multiple of 64 the packer writes a ZG bitmap's words as it
    // marks the groups
    const bool fuse_bitmap = W % 64 == 0;
    for (uint32_t k = 0; k < B; k++) {
        const bool zg = P.mode[k] == kModeZg;
        if (P.mode[k] != kModeHuf && !zg) continue;
        uint8_t* pay = dst + P.pay[k];
        // head: nibble table, word counts, zero pad; ZG bitmap; zero pad
        // after words (staged: the compaction writes all but the bitmap)
        if (!staged) {
            if (t < 128)
                gst(pay + t, uint8_t((P.rcode[k][2 * t] >> kLenShift) | ((P.rcode[k][2 * t + 1] >> kLenShift) << 4)));
            if (uint32_t(t) < NG) gst(pay + 128 + 4 * t, P.wpre[k][t + 1] - P.wpre[k][t]);
            for (uint32_t i = 128 + 4 * NG + t; i < head; i += NT) gst(pay + i, uint8_t(0));
            for (uint32_t i = P.bytes[k] + t; i < uint32_t(align_pay(P.bytes[k])); i += NT) gst(pay + i, uint8_t(0));
        }
        const uint32_t lead = staged ? 0u : head;   // where the bitmap starts
        if (zg) {
            const uint32_t bm = zg_bitmap(m, GG);
            if (fuse_bitmap) {   // only the words past the last group are zeroed here
                const uint32_t Gtot = (m + GG - 1) / GG;
                for (uint32_t x = (Gtot + 63) / 64 + t; x < bm / 8; x += NT) gst(pay + lead + 8 * x, uint64_t(0));
            } else {
                pack_bitmap<BB, GG, NT>(src, base, int(k), P.z[k], m, bm, pay + lead, xf);
            }
        }
    }
    // one wave per lane group, or (ranges of steps summed by the analysis,
    // fewer lane groups than waves) per range of one
    const uint32_t nseg = p.segs && NG < uint32_t(NT / 64) ? uint32_t(NT / 64) / NG : 1u;
    const uint32_t steps = ((m + GG - 1) / GG - 1) / W + 1, per = (steps + nseg - 1) / nseg;
    if (cm)
        for (uint32_t x = wv; x < NG * nseg; x += NT / 64) {
            const uint32_t j = x % NG, sg = x / NG;
            if (sg * per >= steps) continue;
            pack_lane_group<BB, GG, XB, NT == 256>(src, base, cm, zm, P, p.L, j, W, m, xf, fuse_bitmap,
                                                   fuse_raw ? rawmask : 0u, dst, staged ? p.stage_lg : 0u, p.stage_bm,
                                                   staged ? nwords + uint64_t(gc) * B * 64 : nullptr, sg * per,
                                                   min(steps, (sg + 1) * per), sg, p.segs + uint64_t(gc) * B * kSegWords);
        }
}

// NT = 256 for full launches, which the bytes read and written bound: 5 GB of
// an 8B checkpoint 1.72 ms, 4.9 TB/s, a copy's rate.  NT = 1024 for few
// chunks, where a lane group's serial steps bound: with its steps cut into 16
// / (lane groups) ranges, an 8 KiB tensor 58 -> 16 us, 32 chunks of 256 KiB 61
// -> 30 us.  XB: some tensor has an XOR base, whose bytes are fetched ahead
// with the tensor's (against the XOR at the fetch, which waited for both).
// Vector instructions bound it (93% of its issue slots): with 128 a step of a
// wave instead of 150, a 1.7 GB delta's pass 858 -> 826 us.
template <int BB, int GG, bool XB, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 256 && BB == 2 ? (XB ? 6 : 5) : 4, 8))) void k_pack(
    const EncDesc* __restrict__ descs, int n_desc, const uint32_t* __restrict__ chunk_prefix, uint32_t total_chunks,
    EncParams p, const EncEntry* __restrict__ entries, const uint8_t* __restrict__ lens,
    const uint64_t* __restrict__ offsets, const uint64_t* __restrict__ totals, uint32_t* __restrict__ nwords)
{
    __shared__ PackLds P;
    const uint32_t gc = chunk_of_block();
    if (gc < total_chunks)
        pack_chunk<BB, GG, XB, NT>(gc, descs, n_desc, chunk_prefix, p, entries, lens, offsets, totals, nwords, P);
}

// Staged packing, last step: for each chunk, its map entries, and for each
// coded stream the head (nibble table, word counts, padding), the ZG bitmap
// and the lane groups' words copied from their staging slots to their places;
// raw streams are copied whole; then the zero padding to the payload
// alignment.  Tensors whose container did not fit the arena are skipped.
template <int BB, int GG>
__global__ __launch_bounds__(kBlock) void k_compact(const EncDesc* __restrict__ descs, int n_desc,
                                                    const uint32_t* __restrict__ chunk_prefix, uint32_t total_chunks,
                                                    EncParams p, const EncEntry* __restrict__ entries,
                                                    const uint8_t* __restrict__ lens,
                                                    const uint64_t* __restrict__ offsets,
                                                    const uint64_t* __restrict__ totals,
                                                    const uint32_t* __restrict__ nwords)
{
    __shared__ uint32_t wpre[65];
    const int t = threadIdx.x;
    constexpr uint32_t B = BB;
    {
        const uint32_t gc = chunk_of_block();
        if (gc >= total_chunks) return;
        const int di = find_desc(chunk_prefix, n_desc, gc);
        const EncDesc d = descs[di];
        if (totals[di] > d.dst_cap) return;   // too small: the host reports it
        const uint32_t c = gc - chunk_prefix[di];
        const uint32_t E = p.chunk / B;
        const uint32_t m = uint32_t(min(uint64_t(E), d.n - uint64_t(c) * E));
        const uint32_t W = (m + p.S - 1) / p.S;
        const uint32_t NG = (W + 63) / 64;
        const uint32_t head = huf_head(W);
        const uint64_t payload_base = payload_base_of(d.n_chunks, B);
        for (uint32_t k = 0; k < B; k++) {
            const uint64_t ei = uint64_t(gc) * B + k;
            const EncEntry en = entries[ei];
            if (t == 0) {
                uint4 ent;
                ent.x = uint32_t(offsets[ei]);
                ent.y = uint32_t(offsets[ei] >> 32);
                ent.z = en.bytes;
                ent.w = uint32_t(en.mode) | (uint32_t(en.rle) << 8);
                *(uint4*)(d.dst + 64 + 16 * (uint64_t(c) * B + k)) = ent;
            }
            uint8_t* pay = d.dst + payload_base + offsets[ei];
            const uint8_t* slot = p.stage + ei * p.stage_chunk;
            if (en.mode == kModeRaw) {
                // 16-byte pieces (both ends are 16-byte aligned), then the tail
                for (uint32_t i = t; i < m / 16; i += kBlock)
                    reinterpret_cast<uint4*>(pay)[i] = reinterpret_cast<const uint4*>(slot)[i];
                for (uint32_t i = m / 16 * 16 + t; i < m; i += kBlock) pay[i] = slot[i];
            } else if (en.mode == kModeHuf || en.mode == kModeZg) {
                const bool zg = en.mode == kModeZg;
                const uint32_t bm = zg ? zg_bitmap(m, GG) : 0u;
                if (t < 128)
                    pay[t] = uint8_t(lens[ei * 256 + 2 * t] | (lens[ei * 256 + 2 * t + 1] << 4));
                if (t < 64) {
                    const uint32_t nw = uint32_t(t) < NG ? nwords[ei * 64 + t] : 0u;
                    if (uint32_t(t) < NG) reinterpret_cast<uint32_t*>(pay + 128)[t] = nw;
                    uint32_t inc = nw;
#pragma unroll
                    for (int dd = 1; dd < 64; dd <<= 1) {
                        uint32_t o = __shfl_up(inc, dd, 64);
                        if (t >= dd) inc += o;
                    }
                    wpre[t + 1] = inc;
                    if (t == 0) wpre[0] = 0;
                }
                for (uint32_t i = 128 + 4 * NG + t; i < head; i += kBlock) pay[i] = 0;
                for (uint32_t i = t; i < bm / 16; i += kBlock)
                    reinterpret_cast<uint4*>(pay + head)[i] = reinterpret_cast<const uint4*>(slot)[i];
                __syncthreads();
                uint32_t* words = reinterpret_cast<uint32_t*>(pay + head + bm);
                for (uint32_t j = 0; j < NG; j++) {
                    const uint32_t* from = reinterpret_cast<const uint32_t*>(slot + p.stage_bm + uint64_t(j) * p.stage_lg);
                    const uint32_t w0 = wpre[j], nw = wpre[j + 1] - w0;
                    for (uint32_t i = t; i < nw; i += kBlock) words[w0 + i] = from[i];
                }
            }
            for (uint32_t i = en.bytes + t; i < uint32_t(align_pay(en.bytes)); i += kBlock) pay[i] = 0;
            __syncthreads();
        }
    }
}

// An empty tensor's descriptor and chunk prefix, written from kernel arguments
// (no analysis runs that would).
__global__ void k_fill_desc(EncDesc one, uint32_t total_chunks, EncDesc* __restrict__ d, uint32_t* __restrict__ prefix)
{
    if (threadIdx.x == 0) {
        *d = one;
        prefix[0] = 0;
        prefix[1] = total_chunks;
    }
}

}  // namespace

hipError_t launch_encode(const EncDesc* single, EncDesc* d_descs, int n_desc, uint32_t* d_chunk_prefix,
                         uint32_t total_chunks, const EncParams& p, uint8_t* arena, uint64_t cap, EncEntry* entries, uint8_t* lens,
                         uint32_t* nwords, uint64_t* offsets, uint64_t* totals, uint64_t* arena_off,
                         uint64_t* host_off, hipStream_t s)
{
    const dim3 grid = chunk_grid(total_chunks);
    const bool xb = (p.flags & kFlagDelta) != 0;   // some tensor has an XOR base
    const bool staged = p.stage != nullptr;
    const EncDesc one = single ? *single : EncDesc{};
    if (single && !total_chunks) {
        k_fill_desc<<<1, 64, 0, s>>>(one, total_chunks, d_descs, d_chunk_prefix);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    }
    if (total_chunks) {
        // with probing, the probe chunks first: the others read their entries
        for (int phase = p.skip ? 0 : -1; phase <= (p.skip ? 1 : -1); phase++) {
            bool launched = true;
            // one chunk's latency counts until two workgroups of 1024 threads
            // per CU are full; then 512 threads a chunk, four workgroups per
            // CU, overlap more phases (5 GB of BF16: 3.27 against 3.39 ms a
            // pass; 32 chunks: equal within 1%)
            const bool many = p.segs == nullptr;
            // plain launches at the default group: chunks of 64 (4-byte words:
            // 32) groups a thread, 256 KiB, keep their coded streams in
            // registers (a pass over 5 GB of BF16 2.88 against 3.09 ms, 256
            // MiB of FP32 202 against 218 us).  At 512 KiB it would take 1024
            // threads, one workgroup per CU, whose phases nothing overlaps:
            // 3.08 against 3.11 ms, so no instance.
            const bool hold = many && !staged && p.g == 4 && p.skip == 0 && p.chunk == 512 * 512;
#define ZIPNN_ANALYZE(B_, NT_, H_)                                                                                  \
    k_analyze<B_, NT_, H_><<<grid, NT_, 0, s>>>(d_descs, n_desc, d_chunk_prefix, total_chunks, p, phase, entries,   \
                                                lens, nwords, one, single ? d_descs : nullptr, d_chunk_prefix)
            if (p.B == 1 && many) ZIPNN_ANALYZE(1, 512, 0);
            else if (p.B == 1) ZIPNN_ANALYZE(1, 1024, 0);
            else if (p.B == 2 && hold) ZIPNN_ANALYZE(2, 512, 64);
            else if (p.B == 2 && many) ZIPNN_ANALYZE(2, 512, 0);
            else if (p.B == 2) ZIPNN_ANALYZE(2, 1024, 0);
            else if (p.B == 4 && hold) ZIPNN_ANALYZE(4, 512, 32);
            // (its counters leave LDS for two workgroups per CU)
            else if (p.B == 4) ZIPNN_ANALYZE(4, 1024, 0);
            else launched = false;
#undef ZIPNN_ANALYZE
            if (!launched) return hipErrorInvalidValue;
            if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
        }
    }
    // exact: analysis, placement, arena, then packing into the containers;
    // staged: analysis, packing into the staging slots, placement from the
    // word counts, arena, then the compaction into the containers
    auto pack_or_compact = [&](bool compact) -> hipError_t {
        if (!total_chunks) return hipSuccess;
        bool launched = false;
#define ZIPNN_PACK(B_, G_)                                                                                           \
    if (!launched && p.B == B_ && p.g == G_) {                                                                      \
        if (compact)                                                                                                \
            k_compact<B_, G_><<<grid, kBlock, 0, s>>>(d_descs, n_desc, d_chunk_prefix, total_chunks, p, entries,   \
                                                      lens, offsets, totals, nwords);                             \
        else if (p.segs)                                                                                            \
            (xb ? k_pack<B_, G_, true, 1024> : k_pack<B_, G_, false, 1024>)<<<grid, 1024, 0, s>>>(                  \
                d_descs, n_desc, d_chunk_prefix, total_chunks, p, entries, lens, offsets, totals, nwords);          \
        else                                                                                                        \
            (xb ? k_pack<B_, G_, true, 256> : k_pack<B_, G_, false, 256>)<<<grid, 256, 0, s>>>(                     \
                d_descs, n_desc, d_chunk_prefix, total_chunks, p, entries, lens, offsets, totals, nwords);          \
        launched = true;                                                                                            \
    }
        ZIPNN_PACK(1, 2) ZIPNN_PACK(1, 4) ZIPNN_PACK(1, 8)
        ZIPNN_PACK(2, 2) ZIPNN_PACK(2, 4) ZIPNN_PACK(2, 8)
        ZIPNN_PACK(4, 2) ZIPNN_PACK(4, 4) ZIPNN_PACK(4, 8)
#undef ZIPNN_PACK
        if (!launched) return hipErrorInvalidValue;
        return hipGetLastError() == hipSuccess ? hipSuccess : hipErrorLaunchFailure;
    };
    if (staged) {
        const hipError_t e = pack_or_compact(false);
        if (e != hipSuccess) return e;
    }
    k_place<<<n_desc, kPlaceThreads, 0, s>>>(d_descs, n_desc, p, entries, offsets, totals, nwords, arena, cap,
                                             arena_off, host_off);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    return pack_or_compact(staged);
}

}  // namespace zipnn
