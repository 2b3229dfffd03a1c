// GPU compressor for 32^3 bricks: the container of csv_encode_volume, byte
// for byte, built on the device from a label volume resident in HBM.
//
//   reuse kernel (a 1024-thread workgroup per brick, one per CU, persistent):
//     resolution pyramid (Sec. 3.1)    level 1 from the volume, levels 2..5
//                                      in LDS
//     reuse operations (Sec. 3.2,      a lane per expanded parent: its eight
//       Alg. 2)                        children against the parent and the
//                                      neighbours, all levels alike; the
//                                      children left over (they need the
//                                      palette) listed in stream order
//   palette kernel (a wavefront per brick): the palette operations of those
//     children one by one, the last 17 palette entries in its lanes; then
//     the symbol stream as packed nibbles (per level the deltas, then the
//     operations), and the histograms of the sampled bricks
//   rANS kernel (a wavefront per brick): the frequency tables (Sec. 3.3/3.4)
//     from the histograms, interleaved rANS, one state per lane, symbols
//     from last to first; the record into an arena
//   packing: a device scan of record sizes, a kernel that gathers the
//     records, and one that takes the state and the container to the host
//     (one launch for all three where the bricks are few)
//
// The kernels pass their results through arenas in global memory; a brick
// takes its part of arena 1 by an atomic add (its part of arena 2 follows
// from it), and a part that does not fit makes the host repeat the launches
// with the sizes they report.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>
#include <type_traits>

#include "csv.h"
#include "csv_format.hpp"

namespace {

constexpr int kN = 5;
constexpr uint32_t kThreads = 256;
constexpr uint32_t kWaves = kThreads / 64;
constexpr uint32_t kNodes = 4681;           // levels 1..5 of a 32^3 brick
constexpr uint32_t kMaxChildren = 37448;    // 8 * (1 + 8 + 64 + 512 + 4096)
constexpr uint32_t kMaxSym = 2 * kMaxChildren;  // operations and deltas
// per-workgroup scratch of the reuse kernel (dwords): the operations of the
// expanded parents of levels 5..2 (at most 585) and of level 1, then per
// chunk of 64 parents (10 and 64 chunks) the labels of its left-over children
constexpr uint32_t kReuseThreads = 1024;
constexpr uint32_t kChunksA = 10, kChunks = kChunksA + 64, kOpsA = 640;
constexpr uint32_t kOffCand = kOpsA + 4096;
constexpr size_t kScratch = 4 * ((size_t)kOffCand + 512 * kChunks);
// per-wavefront scratch of the rANS kernel: the words of one brick (filled
// from the end, 512 at a time), a multiple of 16 bytes
constexpr size_t kWordsScratch = (2 * (size_t)kMaxSym + 1024 + 64 + 15) & ~(size_t)15;

__device__ __forceinline__ uint32_t lane() { return __lane_id(); }
__device__ __forceinline__ uint32_t mbcnt(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// offset of level l (1..5) in the LDS node arrays
__device__ __forceinline__ uint32_t lvl_off(int l) {
    return l == 1 ? 0u : (l == 2 ? 4096u : (l == 3 ? 4608u : (l == 4 ? 4672u : 4680u)));
}

// 2-bit coordinate (bits 0 and 3)
__device__ __forceinline__ uint32_t coord2(uint32_t p) { return (p & 1u) | ((p >> 2) & 2u); }
// 4-bit coordinate (bits 0, 3, 6, 9)
__device__ __forceinline__ uint32_t coord4(uint32_t p) { return coord2(p) | (coord2(p >> 6) << 2); }
__device__ __forceinline__ uint32_t morton_inc(uint32_t m, uint32_t mask) { return (((m | ~mask) + 1u) & mask) | (m & ~mask); }
__device__ __forceinline__ uint32_t morton_dec(uint32_t m, uint32_t mask) { return (((m & mask) - 1u) & mask) | (m & ~mask); }
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint32_t readlane(uint32_t v, uint32_t k) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)k); }
// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}
// this wave's global stores before its own loads of them
__device__ __forceinline__ void own_stores() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
// order a wave's own LDS operations
__device__ __forceinline__ void wsync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// A device address as a pointer into the global address space, so that the
// accesses compile to global (not flat) instructions
template <class T>
__device__ __forceinline__ T *glob(T *p) {
    return (T *)(__attribute__((address_space(1))) T *)p;
}
// position of the n-th set bit of b (n below its count)
__device__ __forceinline__ uint32_t select_bit(uint64_t b, uint32_t n) {
    uint32_t pos = 0, x = (uint32_t)b;
    const uint32_t c = (uint32_t)__builtin_popcount(x);
    if (n >= c) {
        n -= c;
        pos = 32;
        x = (uint32_t)(b >> 32);
    }
#pragma unroll
    for (uint32_t h = 16; h; h >>= 1) {
        const uint32_t k = (uint32_t)__builtin_popcount(x & ((1u << h) - 1u));
        const bool up = n >= k;
        n -= up ? k : 0u;
        pos += up ? h : 0u;
        x = up ? x >> h : x;
    }
    return pos;
}
// bits 0..7 of v to bits 0, 4, .., 28
__device__ __forceinline__ uint32_t spread_nibbles(uint32_t v) {
    v = (v | (v << 12)) & 0x000F000Fu;
    v = (v | (v << 6)) & 0x03030303u;
    return (v | (v << 3)) & 0x11111111u;
}
// nibble k of z is zero -> bit 4k of the result
__device__ __forceinline__ uint32_t zero_nibbles(uint32_t z) { return ~(z | (z >> 1) | (z >> 2) | (z >> 3)) & 0x11111111u; }

// Per-workgroup phase clocks of the reuse kernel, only in builds with
// CSV_PHASE_TIMING: 8 u64 per workgroup, the shader clocks its thread 0
// spent in each phase.
#ifdef CSV_PHASE_TIMING
__device__ uint64_t *g_enc_phase = nullptr;
struct PhaseClock {
    uint64_t acc[8] = {}, t0 = 0;
    __device__ void start() { t0 = __builtin_amdgcn_s_memtime(); }
    __device__ void stop(int i) {
        const uint64_t t = __builtin_amdgcn_s_memtime();
        acc[i] += t - t0;
        t0 = t;
    }
    __device__ void flush() {
        if (g_enc_phase && threadIdx.x == 0)
            for (int i = 0; i < 8; i++) g_enc_phase[8 * (size_t)blockIdx.x + i] += acc[i];
    }
};
#else
struct PhaseClock {
    __device__ void start() {}
    __device__ void stop(int) {}
    __device__ void flush() {}
};
#endif

// What the kernels know of a brick
struct BrickMeta {
    uint64_t off1;   // arena 1: operations of the expanded parents (stream order), then left-over children's labels
    uint64_t pad;
    uint32_t E[kN];  // expanded parents whose children are on level m
    uint32_t NC[kN]; // children on level m that need the palette
    uint32_t root;   // label of the root
    uint32_t ok;     // 1: arena 1 holds the brick
    uint32_t n, P;   // symbols, palette entries
    uint32_t pal;    // dwords before the palette in arena 2
    uint32_t cum[kN];
};
static_assert(sizeof(BrickMeta) == 96, "brick meta");

// counters of a compression, cleared before its first kernel
struct EncCtl {
    unsigned long long hist[2][16];  // symbols of the sampled bricks
    unsigned long long top1, top3;   // bytes asked of arenas 1 and 3
    unsigned long long total;        // bytes of the records
    uint16_t freq[2][16];            // the tables, for the header
};

// A brick's part of arena 2 lies at three times its place in arena 1 (no
// counter: thousands of waves that start at once would queue for it): packed
// nibbles, palette, then its record if that is not larger than the nibbles,
// palette, header and 64 states (8 E + 9 c + 314 bytes for E parents and c
// left-over children; before the record is written, a byte for each outcome
// and delta).  In arena 1 it takes 4 (E + c) bytes and a pad that keeps the
// parts three times that apart.
constexpr uint32_t kPad1 = 128;
static_assert(3 * kPad1 >= 314, "a brick's part of arena 2");
__host__ __device__ constexpr uint64_t part2(uint64_t off1) { return 3 * off1; }

struct EncArgs {
    const uint32_t *vol;
    uint32_t nx, ny, nz, nbx, nby;
    uint32_t first, step;      // the bricks: first, first + step, ..
    uint32_t n_items;          // how many
    uint32_t sample_stride;    // the frequency tables count every sample_stride-th brick (0: none of these)
    uint32_t bits, lane_k, lane_max, one_table;
    EncCtl *ctl;
    BrickMeta *meta;
    uint8_t *scratch;          // reuse kernel: per workgroup
    uint8_t *wscratch;         // rANS kernel: per wavefront
    uint8_t *arena1, *arena2, *arena3;
    uint64_t cap1, cap3;
    uint32_t *sizes;  // per brick: record bytes
    uint64_t *aoff;   // per brick: record address
};

// four labels in x from any 4-byte aligned address
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ uint32_t lanes_for(uint32_t n, uint32_t K, uint32_t Wmax) {
    if (n == 0) return 0;
    uint32_t W = 1;
    while (2 * W <= Wmax && (uint64_t)2 * W * K <= n) W *= 2;
    return W;
}

// the most frequent of 8 children, the earliest winning a tie; same: all equal
__device__ __forceinline__ uint32_t mode8(const uint32_t ch[8], bool &same) {
    uint32_t n[8] = {};
#pragma unroll
    for (int i = 0; i < 8; i++)
#pragma unroll
        for (int j = i + 1; j < 8; j++) {
            const uint32_t e = ch[i] == ch[j] ? 1u : 0u;
            n[i] += e;
            n[j] += e;
        }
    same = n[0] == 7u;
    uint32_t best = 8 * n[0] + 7, v = ch[0];
#pragma unroll
    for (uint32_t k = 1; k < 8; k++) best = max(best, 8 * n[k] + 7 - k);
#pragma unroll
    for (uint32_t k = 1; k < 8; k++) v = (best & 7u) == 7 - k ? ch[k] : v;
    return v;
}

// A parent's children c, its value p and the neighbours its children may
// refer to: at child 0 on an axis the same-level nodes at -1 (xm by ky + 2
// kz, ym by kx + 2 kz, zm by kx + 2 ky), at child 1 the parent level's node
// at +1.  low / high: bit a set if there is a node at -1 / +1 on axis a.
struct Family {
    uint32_t c[8], p, xm[4], ym[4], zm[4], xp, yp, zp, low, high;
};
// the reuse operations (bestOperation's order: parent, x, y, z), a nibble
// per child, 6 where none applies; left: those children (bit k)
__device__ __forceinline__ uint32_t reuse_ops(const Family &f, uint32_t &left) {
    uint32_t mp = 0, mx = 0, my = 0, mz = 0;
#pragma unroll
    for (uint32_t k = 0; k < 8; k++) {
        const uint32_t c = f.c[k];
        mp |= c == f.p ? 1u << k : 0u;
        mx |= c == ((k & 1) ? f.xp : f.xm[k >> 1]) ? 1u << k : 0u;
        my |= c == ((k & 2) ? f.yp : f.ym[(k & 1) | ((k >> 2) << 1)]) ? 1u << k : 0u;
        mz |= c == ((k & 4) ? f.zp : f.zm[k & 3]) ? 1u << k : 0u;
    }
    mx &= ((f.low & 1u) ? 0x55u : 0u) | ((f.high & 1u) ? 0xAAu : 0u);
    my &= ((f.low & 2u) ? 0x33u : 0u) | ((f.high & 2u) ? 0xCCu : 0u);
    mz &= ((f.low & 4u) ? 0x0Fu : 0u) | ((f.high & 4u) ? 0xF0u : 0u);
    mx &= ~mp;
    my &= ~(mp | mx);
    mz &= ~(mp | mx | my);
    left = 0xFFu & ~(mp | mx | my | mz);
    static_assert(csv::kRp == 0 && csv::kRx == 1 && csv::kRy == 2 && csv::kRz == 3 && csv::kPa == 6, "operation codes");
    return spread_nibbles(mx | mz) | (spread_nibbles(my | mz | left) << 1) | (spread_nibbles(left) << 2);
}

// LDS of a reuse workgroup: the brick's labels, levels 1..5 in Morton order
// (see lvl_off), their constant-subtree flags, what finds an expanded node of
// a given rank, per chunk of 64 parents its left-over children
struct ReuseLds {
    uint32_t vox[32768];          // see vox_at
    uint32_t lab[kNodes + 7];
    uint64_t cst[74];             // level 1, 2, 3 from words 0, 64, 72; level 4 and 5 in bits 0..7 and 8 of 73
    uint64_t wA[16];              // expanded nodes of levels 5, 4, 3 and 2 (8 words)
    uint64_t share;
    uint32_t nE[kN], nC[kN];
    uint32_t before[kChunks + 6]; // left-over children before a chunk's (first: the chunk's own)
    uint16_t preA[16];            // expanded nodes before each word of wA
    uint16_t pre1[64];            // ... of level 1 before each of its words
};
static_assert(sizeof(ReuseLds) <= 160 * 1024, "one workgroup per CU");

// Dword of voxel (x, y, z) of the brick.  Rows of four groups of 8 dwords,
// exchanged so that the 4 x 4 cells in x and y that a wave reads at once
// lie in different banks (groups of 4 dwords in x stay together).
__device__ __forceinline__ uint32_t vox_at(uint32_t x, uint32_t y, uint32_t z) {
    return 1024 * z + 32 * y + (x ^ ((y & 6u) << 2));
}

// Pyramid and reuse operations of one brick per workgroup of 16 waves, one
// workgroup per CU: the brick's 128 KB of labels are read once, into
// registers while the brick before is worked on, and kept in LDS for the
// operations, which look at every expanded node's eight children and twelve
// neighbours.  Bound by vector issue (20 k wave-instructions per brick, 49 %
// of the time) and the steps of few waves between barriers; 307 us for the
// 512^3 cells volume (1.75 TB/s of labels).  Reading the labels again from
// memory, with six smaller workgroups per CU, exceeded the L2 and took 625
// us; a thread per child with its own addresses for every neighbour, and the
// palette operations in the same workgroup, 1.19 ms.
__global__ __launch_bounds__(kReuseThreads) __attribute__((amdgpu_waves_per_eu(4))) void reuse_kernel(EncArgs a) {
    extern __shared__ __align__(16) uint8_t smem[];
    ReuseLds &S = *reinterpret_cast<ReuseLds *>(smem);
    constexpr uint32_t kW = kReuseThreads / 64;
    const uint32_t t = threadIdx.x, L = lane(), w = uniform(t >> 6);
    uint32_t *opw = glob(reinterpret_cast<uint32_t *>(a.scratch + (size_t)blockIdx.x * kScratch));
    const uint32_t lx = coord2(L), ly = coord2(L >> 1), lz = coord2(L >> 2);
    const uint64_t row = a.nx, plane = (uint64_t)a.nx * a.ny;
    // this thread's voxels: 4 in x of row (t >> 3) & 31 in the planes t >> 8, + 4, ..
    const uint32_t vx = 4 * (t & 7u), vy = (t >> 3) & 31u, vz = t >> 8;
    uint4 pre[8];
    auto fetch = [&](uint32_t item) {
        const uint32_t id = a.first + item * a.step;
        const uint64_t x = (uint64_t)(id % a.nbx) * 32 + vx, y = (uint64_t)((id / a.nbx) % a.nby) * 32 + vy;
        const uint64_t z0 = (id / ((uint64_t)a.nbx * a.nby)) * 32;
        const uint32_t *v = glob(a.vol) + x + row * y + plane * (z0 + vz);
        if ((x | 31u) < a.nx && (y | 31u) < a.ny && z0 + 32 <= a.nz) {  // (the same for the whole brick)
#pragma unroll
            for (uint32_t k = 0; k < 8; k++) {
                const u32x4 r = *reinterpret_cast<const u32x4 *>(v + 4 * k * plane);
                pre[k] = make_uint4(r.x, r.y, r.z, r.w);
            }
        } else {  // labels beyond the volume are 0 (padding)
#pragma unroll
            for (uint32_t k = 0; k < 8; k++) {
                const bool in = y < a.ny && z0 + vz + 4 * k < a.nz;
                const uint32_t *u = v + 4 * k * plane;
                pre[k].x = in && x < a.nx ? u[0] : 0u;
                pre[k].y = in && x + 1 < a.nx ? u[1] : 0u;
                pre[k].z = in && x + 2 < a.nx ? u[2] : 0u;
                pre[k].w = in && x + 3 < a.nx ? u[3] : 0u;
            }
        }
    };
    PhaseClock pc;
    if (blockIdx.x < a.n_items) fetch(blockIdx.x);
    for (uint32_t id = blockIdx.x; id < a.n_items; id += gridDim.x) {
        pc.start();
#pragma unroll
        for (uint32_t k = 0; k < 8; k++) *reinterpret_cast<uint4 *>(&S.vox[vox_at(vx, vy, vz + 4 * k)]) = pre[k];
        if (t < kN) S.nC[t] = 0;
        __syncthreads();
        if (a.n_items - id > gridDim.x) fetch(id + gridDim.x);
        pc.stop(0);  // labels
        // level 1 (every level-0 node is a constant subtree): a wave takes
        // 4 x 4 x 4 nodes, one flag word
        for (uint32_t g = w; g < 64; g += kW) {
            const uint32_t X = 4 * coord2(g) + lx, Y = 4 * coord2(g >> 1) + ly, Z = 4 * coord2(g >> 2) + lz;
            uint32_t ch[8];
#pragma unroll
            for (uint32_t k = 0; k < 4; k++) {
                const uint2 r = *reinterpret_cast<const uint2 *>(&S.vox[vox_at(2 * X, 2 * Y + (k & 1), 2 * Z + (k >> 1))]);
                ch[2 * k] = r.x;
                ch[2 * k + 1] = r.y;
            }
            bool same;
            S.lab[64 * g + L] = mode8(ch, same);
            const uint64_t bm = __ballot(same);
            if (L == 0) S.cst[g] = bm;
        }
        __syncthreads();
        // levels 2..5
        auto coarser = [&](int l, uint32_t q, bool act) -> uint64_t {
            const uint32_t lo = lvl_off(l - 1) + 8 * (act ? q : 0u);
            uint32_t ch[8];
#pragma unroll
            for (int k = 0; k < 8; k++) ch[k] = S.lab[lo + k];
            bool same;
            const uint32_t v = mode8(ch, same);
            if (act) S.lab[lvl_off(l) + q] = v;
            // the 8 children's flags: one byte
            return __ballot(act && same && reinterpret_cast<const uint8_t *>(S.cst)[lo >> 3] == 0xFFu);
        };
        if (w < 8) {
            const uint64_t m = coarser(2, 64 * w + L, true);
            if (L == 0) S.cst[64 + w] = m;
        } else if (w == 8) {  // the expanded nodes (not constant) of level 1
            const uint32_t c = (uint32_t)__popcll(~S.cst[L]), inc = wave_incl_scan(c);
            S.pre1[L] = (uint16_t)(inc - c);
            if (L == 63) S.nE[0] = inc;
        }
        __syncthreads();
        pc.stop(1);  // levels 1 and 2
        const uint32_t EB = S.nE[0], nchB = (EB + 63) / 64;
        // a chunk's operations to opw[r] and its left-over children, counted
        // and listed in the chunk's own place
        auto put = [&](const Family &f, bool act, uint32_t r, uint32_t stops, uint32_t ch) -> uint32_t {
            uint32_t left = 0;
            const uint32_t o = reuse_ops(f, left) | (spread_nibbles(stops) << 3);
            if (!act) left = 0;
            if (act) opw[r] = o;
            const uint32_t c = (uint32_t)__builtin_popcount(left), inc = wave_incl_scan(c);
            uint32_t *to = opw + kOffCand + 512 * ch + inc - c;
#pragma unroll
            for (uint32_t k = 0; k < 8; k++)
                if ((left >> k) & 1u) *to++ = f.c[k];
            if (L == 63) S.before[ch] = inc;
            return c;
        };
        if (w == kW - 1) {
            // levels 3..5, and their and level 2's expanded nodes in stream order
            const uint64_t m3 = coarser(3, L, true);
            if (L == 0) S.cst[72] = m3;
            wsync();
            const uint64_t m4 = coarser(4, L, L < 8);
            if (L == 0) S.cst[73] = m4;
            wsync();
            const uint64_t m5 = coarser(5, L, L == 0);
            if (L == 0) S.cst[73] = m4 | (m5 << 8);
            uint64_t x = 0;
            if (L == 0) x = ~m5 & 1u;
            else if (L == 1) x = ~m4 & 0xFFu;
            else if (L == 2) x = ~m3;
            else if (L < 11) x = ~S.cst[61 + L];
            const uint32_t c = (uint32_t)__popcll(x), inc = wave_incl_scan(c);
            if (L < 16) {
                S.wA[L] = x;
                S.preA[L] = L < 11 ? (uint16_t)(inc - c) : (uint16_t)0xFFFFu;
            }
            if (L < 3) S.nE[4 - L] = c;
            const uint32_t up = readlane(inc, 2);
            if (L == 10) S.nE[1] = inc - up;
        } else {
            // children on level 0
            for (uint32_t ch = w; ch < nchB; ch += kW - 1) {
                const uint32_t r = 64 * ch + L;
                const bool act = r < EB;
                const uint32_t rr = act ? r : 0u;
                uint32_t wd = 0;
#pragma unroll
                for (uint32_t h = 32; h; h >>= 1) wd += S.pre1[wd + h] <= rr ? h : 0u;
                const uint32_t q = 64 * wd + select_bit(~S.cst[wd], rr - S.pre1[wd]);
                const uint32_t X = coord4(q), Y = coord4(q >> 1), Z = coord4(q >> 2);
                Family f;
                f.low = (X ? 1u : 0u) | (Y ? 2u : 0u) | (Z ? 4u : 0u);
                f.high = (X < 15 ? 1u : 0u) | (Y < 15 ? 2u : 0u) | (Z < 15 ? 4u : 0u);
                // (a neighbour outside the brick: any value)
                const uint32_t x1 = X ? 2 * X - 1 : 0u, y1 = Y ? 2 * Y - 1 : 0u, z1 = Z ? 2 * Z - 1 : 0u;
#pragma unroll
                for (uint32_t k = 0; k < 4; k++) {  // k: ky + 2 kz
                    const uint32_t y = 2 * Y + (k & 1), z = 2 * Z + (k >> 1);
                    const uint2 c = *reinterpret_cast<const uint2 *>(&S.vox[vox_at(2 * X, y, z)]);
                    f.c[2 * k] = c.x;
                    f.c[2 * k + 1] = c.y;
                    f.xm[k] = S.vox[vox_at(x1, y, z)];
                }
#pragma unroll
                for (uint32_t k = 0; k < 2; k++) {
                    const uint2 c = *reinterpret_cast<const uint2 *>(&S.vox[vox_at(2 * X, y1, 2 * Z + k)]);
                    f.ym[2 * k] = c.x;
                    f.ym[2 * k + 1] = c.y;
                    const uint2 d = *reinterpret_cast<const uint2 *>(&S.vox[vox_at(2 * X, 2 * Y + k, z1)]);
                    f.zm[2 * k] = d.x;
                    f.zm[2 * k + 1] = d.y;
                }
                f.p = S.lab[q];
                f.xp = S.lab[X < 15 ? morton_inc(q, 0x249u) : q];
                f.yp = S.lab[Y < 15 ? morton_inc(q, 0x492u) : q];
                f.zp = S.lab[Z < 15 ? morton_inc(q, 0x924u) : q];
                put(f, act, kOpsA + r, 0u, kChunksA + ch);
            }
        }
        __syncthreads();
        pc.stop(2);  // operations of level 0
        const uint32_t EA = S.nE[1] + S.nE[2] + S.nE[3] + S.nE[4], nchA = (EA + 63) / 64;
        // children on levels 4..1
        if (w < nchA) {
            const uint32_t r = 64 * w + L;
            const bool act = r < EA;
            const uint32_t rr = act ? r : 0u;
            uint32_t wd = 0;
#pragma unroll
            for (uint32_t h = 8; h; h >>= 1) wd += S.preA[wd + h] <= rr ? h : 0u;
            const uint32_t pos = select_bit(S.wA[wd], rr - S.preA[wd]);
            const int l = wd == 0 ? 5 : (wd == 1 ? 4 : (wd == 2 ? 3 : 2));
            const uint32_t q = wd >= 3 ? 64 * (wd - 3) + pos : pos;
            const uint32_t lo = lvl_off(l - 1), lp = lvl_off(l);
            const uint32_t pm = 0x49249249u & ((1u << (3 * (5 - l))) - 1u);
            Family f;
            f.low = f.high = 0;
            uint32_t at[3], up[3];
#pragma unroll
            for (int x = 0; x < 3; x++) {
                const uint32_t am = pm << x;
                f.low |= (q & am) ? 1u << x : 0u;
                f.high |= (q & am) != am ? 1u << x : 0u;
                at[x] = lo + 8 * ((q & am) ? morton_dec(q, am) : q);
                up[x] = S.lab[lp + ((q & am) != am ? morton_inc(q, am) : q)];
            }
            f.p = S.lab[lp + q];
            f.xp = up[0];
            f.yp = up[1];
            f.zp = up[2];
#pragma unroll
            for (uint32_t k = 0; k < 8; k++) f.c[k] = S.lab[lo + 8 * q + k];
#pragma unroll
            for (uint32_t k = 0; k < 4; k++) {
                f.xm[k] = S.lab[at[0] + 2 * k + 1];
                f.ym[k] = S.lab[at[1] + (k & 1) + 2 + 4 * (k >> 1)];
                f.zm[k] = S.lab[at[2] + k + 4];
            }
            const uint32_t stops = reinterpret_cast<const uint8_t *>(S.cst)[(lo >> 3) + q];
            const uint32_t c = put(f, act, r, stops, w);
            if (c) atomicAdd(&S.nC[l - 1], c);
        }
        __syncthreads();
        // operations and left-over labels to arena 1
        const uint32_t Et = EA + EB;
        if (w == 0) {
            // chunks of levels 4..1, then of level 0: the left-over children
            // before each
            const uint32_t cA = L < nchA ? S.before[L] : 0u, cB = L < nchB ? S.before[kChunksA + L] : 0u;
            const uint32_t iA = wave_incl_scan(cA), iB = wave_incl_scan(cB);
            const uint32_t tA = readlane(iA, 63), tB = readlane(iB, 63);
            if (L < nchA) S.before[L] = iA - cA;
            if (L < nchB) S.before[kChunksA + L] = tA + iB - cB;
            const uint64_t bytes = 4ull * (Et + tA + tB) + kPad1;
            if (L == 0) {
                const uint64_t off = atomicAdd(&glob(a.ctl)->top1, (unsigned long long)bytes);
                const bool ok = off + bytes <= a.cap1;
                S.share = ok ? off : ~0ull;
                S.nC[0] = tB;
                BrickMeta *m = glob(a.meta) + id;
                m->off1 = off;
                m->ok = ok ? 1u : 0u;
                m->root = S.lab[lvl_off(kN)];
                for (int k = 0; k < kN; k++) {
                    m->E[k] = S.nE[k];
                    m->NC[k] = S.nC[k];
                }
            }
        }
        __syncthreads();
        const uint64_t off = S.share;
        if (off != ~0ull) {
            uint32_t *d = glob(reinterpret_cast<uint32_t *>(a.arena1 + off));
            for (uint32_t i = t; i < Et; i += kReuseThreads) d[i] = opw[i < EA ? i : kOpsA - EA + i];
            d += Et;
            const uint32_t tot = S.nC[0] + S.nC[1] + S.nC[2] + S.nC[3] + S.nC[4];
            for (uint32_t k = w; k < nchA + nchB; k += kW) {
                const uint32_t ch = k < nchA ? k : kChunksA + k - nchA;
                const uint32_t at = S.before[ch];
                const uint32_t to = k + 1 == nchA + nchB ? tot : S.before[k + 1 < nchA ? k + 1 : kChunksA + k + 1 - nchA];
                for (uint32_t i = L; i < to - at; i += 64) d[at + i] = opw[kOffCand + 512 * ch + i];
            }
        }
        __syncthreads();
        pc.stop(3);  // levels 4..1, arena
    }
    pc.flush();
}

// Palette operations (P_0, else the smallest delta among the 16 entries
// before it, else append; Alg. 2) of one brick's left-over children per
// wavefront, then its symbol stream.  An append moves the window that the
// next child searches, so appends are a chain, but only they: lanes hold 64
// children and the place of each one's label among the last 17 entries; the
// first child without a place is appended, which moves the places behind it
// by one (or to 0), and those before it are final.  A brick of the 512^3
// cells volume of the performance cases has about 300 left-over children and
// 100 appends; 60 us for its 4,096 bricks (155 us with a step per child and
// outcomes in global memory, 113 us with a counter for places in arena 2); 51
// us for those of the benchmark's 512^3 cells.
constexpr uint32_t kOutcomes = 2048;  // left-over children whose outcome fits LDS
__global__ __launch_bounds__(kThreads) void palette_kernel(EncArgs a) {
    __shared__ __align__(8) uint8_t cop_l[kWaves][kOutcomes + 16];
    __shared__ __align__(8) uint8_t del_l[kWaves][kOutcomes + 8 * kN + 8];
    const uint32_t L = lane(), w = uniform(threadIdx.x >> 6);
    for (uint32_t id = blockIdx.x * kWaves + w; id < a.n_items; id += gridDim.x * kWaves) {
        BrickMeta *m = glob(a.meta) + id;
        if (uniform(m->ok) == 0) continue;
        uint32_t E[kN], NC[kN], Et = 0, nc = 0;
#pragma unroll
        for (int k = 0; k < kN; k++) {
            E[k] = uniform(m->E[k]);
            NC[k] = uniform(m->NC[k]);
            Et += E[k];
            nc += NC[k];
        }
        const uint32_t *opw = glob(reinterpret_cast<const uint32_t *>(a.arena1 + m->off1));
        const uint32_t *cand = opw + Et;
        uint32_t win = uniform(m->root), P = 1;  // lane i: entry P - 1 - i
        uint32_t lbn = L < nc ? cand[L] : 0u;    // labels from the next child on
        uint32_t xn = L < Et ? opw[L] : 0u;      // operations from the next parent on
        // arena 2: nibbles, palette, then, for bricks with many left-over
        // children, a byte per child and its level's deltas from a multiple
        // of 8 bytes on (else in LDS)
        const bool small = nc <= kOutcomes;
        const uint32_t ndw = (8 * Et + nc + 7) / 8 + 1;
        uint32_t *nib = glob(reinterpret_cast<uint32_t *>(a.arena2 + part2(m->off1)));
        uint32_t *pal = nib + ndw;
        if (L == 0) pal[0] = win;
        uint32_t n = 0;
        uint32_t D[kN], d0[kN];
        auto work = [&](auto *cop, auto *del) {
            uint32_t c0 = 0, dp = 0;
#pragma unroll
            for (int lv = kN - 1; lv >= 0; lv--) {
                d0[lv] = dp;
                uint32_t d = 0;
                for (uint32_t i0 = 0; i0 < NC[lv]; i0 += 64) {
                    const uint32_t cn = min(64u, NC[lv] - i0), at = c0 + i0;
                    const uint32_t lb = lbn;
                    lbn = at + cn + L < nc ? cand[at + cn + L] : 0u;
                    // each child's place in the window: 0 the last entry, 17
                    // and more: none
                    uint32_t pos = 32;
#pragma unroll
                    for (int i = 16; i >= 0; i--) {
                        const uint32_t e = readlane(win, (uint32_t)i);
                        pos = (uint32_t)i < P && lb == e ? (uint32_t)i : pos;
                    }
                    const uint32_t P0 = P;
                    uint64_t ma = 0, todo = cn == 64 ? ~0ull : (1ull << cn) - 1ull;
                    for (uint64_t miss; (miss = __ballot(pos > 16u) & todo) != 0;) {
                        const uint32_t k = (uint32_t)__builtin_ctzll(miss), lc = readlane(lb, k);
                        todo &= ~((2ull << k) - 1ull);
                        ma |= 1ull << k;
                        // (appended entries move through the lanes: DPP wave shift right by one)
                        win = (uint32_t)__builtin_amdgcn_update_dpp((int)lc, (int)win, 0x138, 0xF, 0xF, false);
                        P++;
                        const uint32_t moved = lb == lc ? 0u : pos + 1u;
                        pos = L > k ? moved : pos;
                    }
                    const bool in = L < cn, ap = (ma >> L) & 1u, dl = in && !ap && pos > 0;
                    const uint64_t md = __ballot(dl);
                    if (ap) pal[P0 + mbcnt(ma)] = lb;
                    if (dl) del[dp + d + mbcnt(md)] = (uint8_t)(pos - 1u);
                    // what turns the placeholder (P_a) into the operation
                    if (in) cop[at + L] = (uint8_t)(ap ? 0u : (dl ? (csv::kPa ^ csv::kPd) : (csv::kPa ^ csv::kP0)));
                    d += (uint32_t)__popcll(md);
                }
                c0 += NC[lv];
                D[lv] = d;
                dp = (dp + d + 7u) & ~7u;
            }
            own_stores();
            // the stream: words of 8 nibbles appended behind sh pending ones,
            // which are the top nibbles of cw
            uint32_t op = 0, sh = 0, cw = 0, rk = 0, eb = 0;
            auto append = [&](uint32_t x, uint32_t k) {  // k words, lane i holds word i
                const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp((int)cw, (int)x, 0x138, 0xF, 0xF, false);
                const uint32_t o = sh ? __builtin_amdgcn_alignbit(x, prev, 32 - 4 * sh) : x;
                if (L < k) nib[op + L] = o;
                op += k;
                cw = readlane(x, k - 1);
            };
#pragma unroll
            for (int lv = kN - 1; lv >= 0; lv--) {
                for (uint32_t i0 = 0; i0 < D[lv]; i0 += 512) {
                    const uint32_t left = min(512u, D[lv] - i0), i = 8 * L;
                    uint32_t x = 0;
                    if (i < left) {
                        const auto *b = reinterpret_cast<const uint32_t *>(del + d0[lv] + i0 + i);
                        const uint32_t bx = b[0], by = b[1];
                        const uint32_t lo = (bx | (bx >> 4)) & 0x00FF00FFu, hi = (by | (by >> 4)) & 0x00FF00FFu;
                        x = ((lo | (lo >> 8)) & 0xFFFFu) | (((hi | (hi >> 8)) & 0xFFFFu) << 16);
                    }
                    const uint32_t k = left / 8, rem = left & 7u;
                    if (k) append(x, k);
                    if (rem) {  // (the last deltas of the level)
                        const uint32_t v = readlane(x, k) & ((1u << (4 * rem)) - 1u);
                        const uint32_t both = sh ? (cw >> (32 - 4 * sh)) | (v << (4 * sh)) : v;
                        if (sh + rem >= 8) {
                            if (L == 0) nib[op] = both;
                            op++;
                            const uint32_t over = sh + rem - 8;
                            cw = over ? (v >> (4 * (8 - sh))) << (32 - 4 * over) : 0u;
                            sh = over;
                        } else {
                            sh += rem;
                            cw = both << (32 - 4 * sh);
                        }
                    }
                }
                for (uint32_t r0 = 0; r0 < E[lv]; r0 += 64) {
                    const uint32_t k = min(64u, E[lv] - r0), nx = eb + r0 + k + L;
                    uint32_t x = L < k ? xn : 0u;
                    xn = nx < Et ? opw[nx] : 0u;
                    // the placeholders, in the order of their children
                    uint32_t left = zero_nibbles((x & 0x77777777u) ^ 0x66666666u);
                    const uint32_t c = (uint32_t)__builtin_popcount(left), inc = wave_incl_scan(c);
                    const uint32_t at = rk + inc - c;
                    // (at most 8, read at once: the bytes behind them are not used)
                    const auto *cw4 = reinterpret_cast<const uint32_t *>(cop + (at & ~3u));
                    const uint32_t w0 = cw4[0], w1 = cw4[1], w2 = cw4[2];
                    uint64_t got = (uint64_t)__builtin_amdgcn_alignbyte(w2, w1, at & 3u) << 32 |
                                   __builtin_amdgcn_alignbyte(w1, w0, at & 3u);
                    while (left) {
                        const uint32_t b = (uint32_t)__builtin_ctz(left);
                        left &= left - 1u;
                        x ^= ((uint32_t)got & 0xFFu) << b;
                        got >>= 8;
                    }
                    rk += readlane(inc, 63);
                    append(x, k);
                }
                eb += E[lv];
                n += D[lv] + 8 * E[lv];
                if (L == 0) m->cum[lv] = n;
            }
            if (sh && L == 0) nib[op] = cw >> (32 - 4 * sh);
        };
        if (small) {
            work(cop_l[w], del_l[w]);
        } else {
            uint8_t *cop = glob(reinterpret_cast<uint8_t *>((reinterpret_cast<uintptr_t>(pal + 1 + nc) + 7) & ~(uintptr_t)7));
            work(cop, cop + ((nc + 7u) & ~7u));
        }
        wsync();  // the LDS is reused for this wave's next brick
        if (L == 0) {
            m->pal = ndw;
            m->n = n;
            m->P = P;
        }
        // the sampled bricks' symbols (the frequency tables, Sec. 3.4)
        if (a.sample_stride && (a.first + id * a.step) % a.sample_stride == 0) {
            own_stores();
            const uint32_t leaf = n - D[0] - 8 * E[0];
            for (uint32_t tb = 0; tb < 2; tb++) {
                const uint32_t i0 = tb ? leaf : 0u, i1 = tb ? n : leaf;
                uint32_t cnt[16] = {};
#pragma unroll 4
                for (uint32_t d = (i0 >> 3) + L; 8 * d < i1; d += 64) {
                    const uint32_t x = nib[d];
                    // a bit per symbol of the range
                    uint32_t in = 0x11111111u;
                    if (8 * d < i0) in &= ~0u << (4 * (i0 - 8 * d));
                    if (8 * d + 8 > i1) in &= (1u << (4 * (i1 - 8 * d))) - 1u;
                    const uint32_t b0 = x, b1 = x >> 1, b2 = x >> 2, b3 = x >> 3;
                    const uint32_t lo[4] = {~b0 & ~b1, b0 & ~b1, ~b0 & b1, b0 & b1};
                    const uint32_t hi[4] = {in & ~b2 & ~b3, in & b2 & ~b3, in & ~b2 & b3, in & b2 & b3};
#pragma unroll
                    for (int v = 0; v < 16; v++) cnt[v] += (uint32_t)__builtin_popcount(lo[v & 3] & hi[v >> 2]);
                }
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const uint32_t c = readlane(wave_incl_scan(cnt[v]), 63);
                    if (L == 0 && c) atomicAdd(&glob(a.ctl)->hist[tb][v], (unsigned long long)c);
                }
            }
        }
    }
}

// Interleaved rANS and the record of one brick per wavefront (Sec. 3.3):
// symbol i to state i mod W, from the last symbol to the first; the words
// of a step go to descending lanes, so they are placed from the end of the
// wave's scratch towards its start, where the decoder's order begins.
// Division by a frequency is a multiply by its 32-bit reciprocal with one
// correction.  The chain of a step is a dozen operations (the symbols and
// table entries of 16 steps are fetched ahead, the words gathered in LDS);
// bound by vector issue: 71 us for the 4,096 bricks (122 us with a store per
// word, tables unpacked in every step and a double reciprocal; 81 us with a
// look at the kept words after every step and the tables normalised by one
// thread each).  The few bricks of a small volume are bound by the chain: 36
// us for 140, 46 us before the latter two.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void rans_kernel(EncArgs a) {
    // per table and symbol: the reciprocal m, f | s << 24, 2^bits - f and the
    // start c of its slots; with 2^s < f <= 2^(s + 1), v / f is
    // (v m >> 32 >> s) or one more
    __shared__ uint4 tab[32];
    // per wave: the packed symbols of a block of 16 steps, the last 1024 words
    __shared__ uint32_t sym_l[kWaves][128];
    __shared__ __align__(16) uint16_t word_l[kWaves][1024];
    const uint32_t t = threadIdx.x, L = lane(), w = uniform(t >> 6), bits = a.bits, M = 1u << bits;
    if (w == 0) {  // the host compressor's normalisation of the counts, 16 lanes per table
        const uint32_t k = (L >> 4) & 1u, q = L & 15u;
        const unsigned long long h0 = glob(a.ctl)->hist[0][q], h1 = glob(a.ctl)->hist[1][q];
        const uint64_t c = (a.one_table ? h0 + h1 : (k ? h1 : h0)) + 1;
        uint64_t tot = c;
        for (int d = 1; d < 16; d *= 2) tot += __shfl_xor((unsigned long long)tot, d);
        const uint64_t v = c * M / tot;
        uint32_t f = v ? (uint32_t)v : 1u, sum = f;
        for (int d = 1; d < 16; d *= 2) sum += __shfl_xor(sum, d);
        // the first of the largest frequencies (of those above 1) takes what
        // is missing, or gives back what is too much one by one
        auto is_best = [&](bool on) {
            const uint32_t key = on ? f << 4 | (15u - q) : 0u;
            uint32_t top = key;
            for (int d = 1; d < 16; d *= 2) top = max(top, (uint32_t)__shfl_xor(top, d));
            return on && key == top;
        };
        if (is_best(true) && sum < M) f += M - sum;
        while (__any(sum > M)) {
            const bool best = is_best(f > 1);
            if (sum > M) {
                f -= best ? 1u : 0u;
                sum--;
            }
        }
        uint32_t c0 = f;
        for (int d = 1; d < 16; d *= 2) {
            const uint32_t lower = __shfl_up(c0, d, 16);
            c0 += q >= (uint32_t)d ? lower : 0u;
        }
        const uint32_t sh = f > 2 ? 31u - (uint32_t)__builtin_clz(f - 1) : 0u;
        const uint64_t m = ((uint64_t)1 << (32 + sh)) / f;
        if (L < 32) {
            tab[L] = make_uint4(m >> 32 ? 0xFFFFFFFFu : (uint32_t)m, f | (sh << 24), M - f, c0 - f);
            if (blockIdx.x == 0) glob(a.ctl)->freq[k][q] = (uint16_t)f;
        }
    }
    __syncthreads();
    // word i of a brick goes to LDS place 1023 - (i mod 1024), and each 512 of
    // them in one store per lane to the scratch, which fills downwards
    uint8_t *wend = glob(a.wscratch) + ((size_t)blockIdx.x * kWaves + w + 1) * kWordsScratch - 64;
    uint16_t *words = word_l[w];
    uint32_t *syms = sym_l[w];
    const uint32_t hdr = csv::record_header_words(kN);
    for (uint32_t id = blockIdx.x * kWaves + w; id < a.n_items; id += gridDim.x * kWaves) {
        const BrickMeta *bm = glob(a.meta) + id;
        if (uniform(bm->ok) == 0u) continue;
        const uint32_t n = uniform(bm->n), Pn = uniform(bm->P), leaf = uniform(bm->cum[1]);
        const uint32_t *nib = glob(reinterpret_cast<const uint32_t *>(a.arena2 + part2(bm->off1)));
        const uint32_t *pal = nib + bm->pal;
        const uint32_t W = lanes_for(n, a.lane_k, a.lane_max);
        uint32_t x = csv::kRansLower, pushed = 0, kept = 0;
        auto flush = [&]() {  // words kept .. kept + 511
            wsync();
            const uint4 v = *reinterpret_cast<const uint4 *>(words + 512 - (kept & 1023u) + 8 * L);
            kept += 512;
            *reinterpret_cast<uint4 *>(wend - 2 * (size_t)kept + 16 * L) = v;
            wsync();
        };
        if (n) {
            // blocks of 16 steps from a multiple of 16 steps on, the last
            // first; their symbols are 2 W dwords, loaded a block ahead
            constexpr int kBlk = 16;
            const uint32_t steps = (n + W - 1) / W, ndw = (n + 7) / 8;
            uint32_t blk = (steps - 1) / kBlk;
            auto fetch = [&](uint32_t b) -> uint2 {
                const uint32_t d = 2 * W * b + L;
                return make_uint2(L < 2 * W && d < ndw ? nib[d] : 0u, L + 64 < 2 * W && d + 64 < ndw ? nib[d + 64] : 0u);
            };
            const uint64_t lanes = W == 64 ? ~0ull : (1ull << W) - 1ull;
            uint2 next = fetch(blk);
            // all: every state of the block has a symbol in every step
            auto block = [&](auto all) {
                wsync();
                syms[L] = next.x;
                syms[L + 64] = next.y;
                wsync();
                if (blk) next = fetch(blk - 1);
                uint4 te[kBlk];
#pragma unroll
                for (int k = 0; k < kBlk; k++) {
                    const uint32_t j = (uint32_t)(kBlk - 1 - k) * W + L, i = kBlk * W * blk + j;
                    const uint32_t sy = (syms[(j >> 3) & 127u] >> (4 * (j & 7u))) & 15u;
                    te[k] = tab[sy + (i >= leaf ? 16u : 0u)];
                }
#pragma unroll
                for (int k = 0; k < kBlk; k++) {
                    const uint4 e = te[k];
                    bool act = true;
                    if constexpr (!decltype(all)::value)
                        act = kBlk * W * blk + (uint32_t)(kBlk - 1 - k) * W + L < n && L < W;
                    // (the shift leaves f alone of e.y)
                    const bool full = x >= e.y << (32 - bits) && act;
                    const uint64_t em = __ballot(full) & lanes;
                    const uint32_t v = full ? x >> 16 : x;
                    // the host order within a step is descending lanes
                    const uint32_t cnt = (uint32_t)__popcll(em);
                    if ((em >> L) & 1ull) words[(mbcnt(em) - pushed - cnt) & 1023u] = (uint16_t)x;
                    pushed += cnt;
                    uint32_t q = __umulhi(v, e.x) >> (e.y >> 24);
                    q += v - __umul24(q, e.y) >= (e.y & 0xFFFFFFu) ? 1u : 0u;
                    const uint32_t y = __umul24(q, e.z) + v + e.w;
                    x = act ? y : x;
                    // (8 steps emit up to 512 words, behind up to 511 kept)
                    if (k % 8 == 7 && pushed - kept >= 512) flush();
                }
            };
            if (n % (kBlk * W)) {
                block(std::false_type{});
                if (blk-- == 0) blk = 0xFFFFFFFFu;
            }
            for (; blk != 0xFFFFFFFFu; blk--) block(std::true_type{});
            // the rest (up to 511 words), in a whole store: what lies before
            // them is not read
            if (pushed != kept) flush();
        }
        const uint32_t nw = pushed;
        const uint32_t size = (4 * (hdr + Pn + W) + 2 * nw + 3) & ~3u;
        // behind the palette in arena 2; a record larger than its nibbles
        // (symbols unlike the sampled ones) takes a part of arena 3
        uint64_t at = reinterpret_cast<uintptr_t>(pal + Pn);
        bool room = 2 * (uint64_t)nw <= 4ull * bm->pal;
        if (!room) {
            uint64_t off = 0;
            if (L == 0) off = atomicAdd(&glob(a.ctl)->top3, (unsigned long long)size);
            off = (uint64_t)readlane((uint32_t)off, 0) | ((uint64_t)readlane((uint32_t)(off >> 32), 0) << 32);
            room = off + size <= a.cap3;
            at = reinterpret_cast<uintptr_t>(a.arena3) + off;
        }
        if (L == 0) {
            a.sizes[id] = size;
            a.aoff[id] = at;
        }
        own_stores();
        if (room) {
            uint32_t *r = glob(reinterpret_cast<uint32_t *>(at));
            if (L == 0) {
                r[0] = Pn;
                r[1] = W;
                r[2] = nw;
                for (int m = 0; m < kN; m++) r[3 + m] = bm->cum[m];
            }
            // eight loads in flight per lane
            auto copy = [&](uint32_t *to, uint32_t cnt, auto get) {
                for (uint32_t q0 = 0; q0 < cnt; q0 += 512) {
                    uint32_t v[8];
#pragma unroll
                    for (uint32_t k = 0; k < 8; k++) {
                        const uint32_t q = q0 + 64 * k + L;
                        v[k] = q < cnt ? get(q) : 0u;
                    }
#pragma unroll
                    for (uint32_t k = 0; k < 8; k++) {
                        const uint32_t q = q0 + 64 * k + L;
                        if (q < cnt) to[q] = v[k];
                    }
                }
            };
            copy(r + hdr, Pn, [&](uint32_t q) -> uint32_t { return pal[q]; });
            if (L < W) r[hdr + Pn + L] = x;
            // the words lie in order from -nw on; dwords from an even place
            uint32_t *wr = r + hdr + Pn + W;
            const uint32_t *src = reinterpret_cast<const uint32_t *>(wend) - (nw + 1) / 2;
            if (nw & 1u)
                copy(wr, (nw + 1) / 2, [&](uint32_t q) -> uint32_t {
                    const uint32_t hi = 2 * q + 1 < nw ? src[q + 1] : 0u;
                    return (src[q] >> 16) | (hi << 16);
                });
            else
                copy(wr, nw / 2, [&](uint32_t q) -> uint32_t { return src[q]; });
        }
        // the words region is reused by this wavefront's next brick
        own_stores();
    }
}

// whether every arena held what was asked of it (else the host repeats the
// launches, and the sizes and offsets of some bricks are not written)
__device__ __forceinline__ bool arenas_held(const EncArgs &a) {
    const EncCtl *c = glob(a.ctl);
    return c->top1 <= a.cap1 && c->top3 <= a.cap3;
}

// exclusive scan of the record sizes into the container's u64 index: four
// sizes per thread and round, a wave scan, the waves' sums in LDS
__global__ __launch_bounds__(1024) void scan_kernel(EncArgs a, uint64_t *index) {
    __shared__ uint64_t part[16];
    if (!arenas_held(a)) return;
    const uint32_t t = threadIdx.x, L = lane(), w = t >> 6, n = a.n_items;
    uint64_t carry = 0;
    for (uint32_t b0 = 0; b0 < n; b0 += 4096) {
        const uint32_t i = b0 + 4 * t;
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            v[k] = i + k < n && i + k >= i ? a.sizes[i + k] : 0u;
            sum += v[k];  // (a record is below 2^20 bytes)
        }
        const uint32_t inc = wave_incl_scan(sum);
        if (L == 63) part[w] = inc;
        __syncthreads();
        uint64_t before = carry, all = carry;
#pragma unroll
        for (uint32_t k = 0; k < 16; k++) {
            before += k < w ? part[k] : 0ull;
            all += part[k];
        }
        uint64_t o = before + inc - sum;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            if (i + k < n && i + k >= i) index[i + k] = o;
            o += v[k];
        }
        carry = all;
        __syncthreads();
    }
    if (t == 0) {
        index[n] = carry;
        glob(a.ctl)->total = carry;
    }
}

// records from the arenas to their place in the container's record area of
// cap bytes
__global__ __launch_bounds__(256) void pack_kernel(EncArgs a, const uint64_t *index, uint8_t *records,
                                                   uint64_t cap) {
    if (!arenas_held(a)) return;
    for (uint32_t id = blockIdx.x; id < a.n_items; id += gridDim.x) {
        const uint32_t *src = glob(reinterpret_cast<const uint32_t *>(a.aoff[id]));
        const uint64_t at = index[id], size = a.sizes[id];
        if (at + size > cap) return;  // (the host repeats the copy)
        uint32_t *dst = glob(reinterpret_cast<uint32_t *>(records + at));
        for (uint32_t i = threadIdx.x; i < size / 4; i += 256) dst[i] = src[i];
    }
}

// bytes of device memory to pinned host memory, 16 per lane; src and dst
// 16-byte aligned
__device__ __forceinline__ void copy_out(const uint8_t *src, uint8_t *dst, uint64_t bytes) {
    const uint4 *s4 = glob(reinterpret_cast<const uint4 *>(src));
    uint4 *d4 = glob(reinterpret_cast<uint4 *>(dst));
    const uint64_t n = bytes / 16;
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < n; i += gridDim.x * 256ull) d4[i] = s4[i];
    const uint64_t at = 16 * n + threadIdx.x;
    if (blockIdx.x == 0 && at < bytes) dst[at] = src[at];
}

// The end of a compression: the state to host memory, and the container as
// well when it has fewer than cap bytes, which is the room there.  Bound by
// the link to the host.  One kernel and one wait of the host, without a copy of
// the state, a wait and a copy of the container: 12 us less for a container of
// 0.2 MB.
__global__ __launch_bounds__(256) void leave_kernel(EncArgs a, EncCtl *h_ctl, const uint8_t *blob, uint64_t rs,
                                                    uint8_t *h_blob, uint64_t cap) {
    constexpr uint32_t words = sizeof(EncCtl) / 4;
    static_assert(sizeof(EncCtl) % 4 == 0 && words <= 256, "one word per thread");
    if (blockIdx.x == 0 && threadIdx.x < words)
        reinterpret_cast<uint32_t *>(h_ctl)[threadIdx.x] = reinterpret_cast<const uint32_t *>(a.ctl)[threadIdx.x];
    if (!arenas_held(a)) return;
    const uint64_t total = rs + glob(a.ctl)->total;
    if (total < cap) copy_out(blob, h_blob, total);
}

// The scan, the packing and the end in one launch, for volumes of at most
// kFinishMax bricks: every workgroup scans all the sizes itself, four per
// thread, and the records of a container of fewer than cap bytes go straight
// to the host, those of a larger one to blob.  A small volume's call is bound
// by latency: 140 bricks take 9 us here, 17 in three launches; the whole call
// of 1 brick 98 -> 93 us, of 125 133 -> 128, of 1,000 385 -> 374 to 381.
// Beyond that a thread would scan more than four sizes in every workgroup
// for a gain of 2 %.
constexpr uint32_t kFinishMax = 1024;
__global__ __launch_bounds__(256) void finish_kernel(EncArgs a, EncCtl *h_ctl, uint8_t *blob, uint64_t blob_cap,
                                                     uint64_t rs, uint8_t *h_blob, uint64_t cap) {
    __shared__ uint32_t off[kFinishMax], part[4];
    constexpr uint32_t words = sizeof(EncCtl) / 4, total_at = offsetof(EncCtl, total) / 4;
    const uint32_t t = threadIdx.x, L = lane(), w = t >> 6, n = a.n_items;
    // the state but for its total, which is written below
    if (blockIdx.x == 0 && t < words && t / 2 != total_at / 2)
        reinterpret_cast<uint32_t *>(h_ctl)[t] = reinterpret_cast<const uint32_t *>(a.ctl)[t];
    if (!arenas_held(a)) return;
    uint32_t v[4], sum = 0;  // (a record is below 2^20 bytes)
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) {
        v[k] = 4 * t + k < n ? a.sizes[4 * t + k] : 0u;
        sum += v[k];
    }
    const uint32_t inc = wave_incl_scan(sum);
    if (L == 63) part[w] = inc;
    __syncthreads();
    uint32_t o = inc - sum, records = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) {
        o += k < w ? part[k] : 0u;
        records += part[k];
    }
    const bool direct = rs + records < cap;
    uint8_t *to = direct ? h_blob : blob;
    uint64_t *index = glob(reinterpret_cast<uint64_t *>(to + csv::kHeaderBytes));
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) {
        off[4 * t + k] = o;
        if (blockIdx.x == 0 && 4 * t + k < n) index[4 * t + k] = o;
        o += v[k];
    }
    __syncthreads();
    if (blockIdx.x == 0 && t == 0) {
        index[n] = records;
        h_ctl->total = records;
    }
    for (uint32_t id = blockIdx.x; id < n; id += gridDim.x) {
        const uint32_t *src = glob(reinterpret_cast<const uint32_t *>(a.aoff[id]));
        const uint64_t at = rs + off[id], size = a.sizes[id];
        if (!direct && at + size > blob_cap) return;  // (the host repeats the copy)
        uint32_t *dst = glob(reinterpret_cast<uint32_t *>(to + at));
        for (uint32_t i = t; i < size / 4; i += 256) dst[i] = src[i];
    }
}

// a piece of a large container
__global__ __launch_bounds__(256) void piece_kernel(const uint8_t *src, uint8_t *dst, uint64_t bytes) {
    copy_out(src, dst, bytes);
}

// keep_hist: all but the histograms
__global__ __launch_bounds__(256) void begin_kernel(EncCtl *ctl, bool keep_hist) {
    const uint32_t from = keep_hist ? sizeof(EncCtl::hist) / 4 : 0u;
    if (threadIdx.x >= from && threadIdx.x < sizeof(EncCtl) / 4) reinterpret_cast<uint32_t *>(ctl)[threadIdx.x] = 0;
}

// a device buffer that grows on demand
struct DevBuf {
    void *p = nullptr;
    size_t bytes = 0;
    bool ensure(size_t need) {
        need = std::max<size_t>(need, 256);
        if (bytes >= need) return true;
        if (p) (void)hipFree(p);
        p = nullptr;
        bytes = 0;
        if (hipMalloc(&p, need) != hipSuccess) {
            (void)hipGetLastError();  // (the caller goes on without it)
            p = nullptr;
            return false;
        }
        bytes = need;
        return true;
    }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
        bytes = 0;
    }
    template <class T>
    T *as() const {
        return reinterpret_cast<T *>(p);
    }
};

// A container of at least kPiecewise bytes leaves in kPieces copies, which
// kCopyThreads threads move from the pinned buffer to the caller's memory as
// they arrive, kParts parts each: the call ends shortly after the transfer.
// A kernel per piece: 17.8 us for 0.92 MB (52 GB/s, the link's rate) and 5.5 us
// to the next, where the copy engine takes 17.1 us and stops for 10.6.
// 512^3 cells (14.7 MB): 1052 -> 894 us for the whole call.
constexpr unsigned kPieces = 8, kParts = 8, kCopyThreads = 8;
constexpr size_t kPiecewise = 8u << 20;
constexpr unsigned kCopyGroups = 128;
constexpr size_t kPinFirst = 1u << 20;  // pinned memory of a device's first call

// per device: the buffers of the last call, kept for the next one
struct EncCache {
    std::mutex mu;
    DevBuf scratch, wscratch, ctl, meta, sizes, aoff, arena1, arena2, arena3, dblob;
    EncCtl *h_ctl = nullptr;   // pinned
    uint8_t *h_pin = nullptr;  // pinned staging of the container on its way to host memory
    size_t h_pin_bytes = 0;
    hipEvent_t arrived[kPieces] = {};  // the pieces of a large container
    void release_device() {
        scratch.release();
        wscratch.release();
        ctl.release();
        meta.release();
        sizes.release();
        aoff.release();
        arena1.release();
        arena2.release();
        arena3.release();
        dblob.release();
    }
    void release() {
        release_device();
        if (h_ctl) (void)hipHostFree(h_ctl);
        h_ctl = nullptr;
        if (h_pin) (void)hipHostFree(h_pin);
        h_pin = nullptr;
        h_pin_bytes = 0;
        for (auto &e : arrived) {
            if (e) (void)hipEventDestroy(e);
            e = nullptr;
        }
    }
    // arenas 1 and 2 for cap1 bytes of operations and labels; if one cannot
    // be had, neither is kept
    bool arenas(uint64_t cap1) {
        if (arena1.ensure(cap1) && arena2.ensure(part2(cap1))) return true;
        arena1.release();
        arena2.release();
        return false;
    }
    uint64_t cap1() const { return std::min<uint64_t>(arena1.bytes, arena2.bytes / part2(1)); }
    // at least bytes of pinned memory
    bool pin(size_t bytes) {
        if (h_pin_bytes >= bytes) return true;
        if (h_pin) (void)hipHostFree(h_pin);
        h_pin = nullptr;
        h_pin_bytes = 0;
        if (hipHostMalloc(reinterpret_cast<void **>(&h_pin), bytes, hipHostMallocDefault) != hipSuccess) return false;
        h_pin_bytes = bytes;
        return true;
    }
    // bytes of device memory src through h_pin to dst, on stream s
    int bring(uint8_t *dst, const uint8_t *src, size_t bytes, hipStream_t s) {
        bool pieces = bytes >= kPiecewise;
        for (unsigned k = 0; pieces && k < kPieces; k++)
            if (!arrived[k] && hipEventCreateWithFlags(&arrived[k], hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                arrived[k] = nullptr;
                pieces = false;
            }
        const dim3 grid(kCopyGroups), threads(256);
        if (!pieces) {
            hipLaunchKernelGGL(piece_kernel, grid, threads, 0, s, src, h_pin, (uint64_t)bytes);
            if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return CSV_EHIP;
            std::memcpy(dst, h_pin, bytes);
            return CSV_OK;
        }
        constexpr size_t kAlign = 4096 * kParts;
        const size_t piece = ((bytes + kPieces - 1) / kPieces + kAlign - 1) & ~(kAlign - 1), part = piece / kParts;
        bool ok = true;
        for (unsigned k = 0; ok && k < kPieces; k++) {
            const size_t at = std::min(bytes, k * piece), m = std::min(bytes, at + piece) - at;
            if (m) hipLaunchKernelGGL(piece_kernel, grid, threads, 0, s, src + at, h_pin + at, (uint64_t)m);
            ok = hipGetLastError() == hipSuccess && hipEventRecord(arrived[k], s) == hipSuccess;
        }
        if (!ok) return CSV_EHIP;
        std::atomic<unsigned> next{0};
        std::atomic<bool> failed{false};
        auto work = [&] {
            for (unsigned k; (k = next.fetch_add(1)) < kPieces * kParts;) {
                const size_t at = std::min(bytes, k * part), m = std::min(bytes, at + part) - at;
                if (hipEventSynchronize(arrived[k / kParts]) != hipSuccess) failed = true;
                else std::memcpy(dst + at, h_pin + at, m);
            }
        };
        std::thread th[kCopyThreads - 1];
        for (auto &x : th) {
            try {
                x = std::thread(work);
            } catch (...) {  // fewer threads then
                break;
            }
        }
        work();
        for (auto &x : th)
            if (x.joinable()) x.join();
        return failed ? CSV_EHIP : CSV_OK;
    }
};
constexpr int kMaxDevices = 64;
EncCache *g_cache[kMaxDevices] = {};
std::mutex g_cache_mu;

EncCache *cache_for(int device) {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    if (!g_cache[device]) g_cache[device] = new (std::nothrow) EncCache;
    return g_cache[device];
}

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) (void)hipSetDevice(dev);
    }
    ~DeviceGuard() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

// A call that fails waits for its launches before the buffers, which the next
// call uses on another stream, are free again, and takes the runtime's error
// with it (its code says what failed).
struct InFlight {
    hipStream_t s;
    bool finished = false;
    explicit InFlight(hipStream_t stream) : s(stream) {}
    ~InFlight() {
        if (finished) return;
        (void)hipStreamSynchronize(s);
        (void)hipGetLastError();
    }
};

// The most that a brick can ask for: all of its 4,681 parents expanded, a
// palette entry for each child; a record of two words per child and delta
constexpr uint64_t kMostOps = 4ull * (kNodes + kMaxChildren) + kPad1;
constexpr uint64_t kMostRecord = 4ull * (csv::record_header_words(kN) + kMaxChildren + 1 + 64) + 2ull * kMaxSym + 4;
// Bricks per CU of a batch where the device has no room for all at once, at
// most (1.28 MB each)
constexpr uint32_t kBatchPerCu = 16;

// The kernels of a compression on stream s with the buffers of ec; a: the
// volume and the options, then the bricks and buffers of the launches
struct Compression {
    EncCache *ec;
    hipStream_t s;
    uint32_t cu;
    EncArgs a;
    bool there = false;  // the last run's container is in the pinned buffer
    uint64_t bytes = 0;  // ... its bytes

    // reuse kernel: a workgroup per CU
    uint32_t grid(uint32_t n) const { return std::min(n, cu); }
    uint32_t grid2(uint32_t n) const {
        return (uint32_t)std::min<uint64_t>(((uint64_t)n + kWaves - 1) / kWaves, (uint64_t)cu * 4);
    }
    // what n bricks need apart from the arenas and the container
    bool room(uint32_t n) {
        return ec->scratch.ensure(kScratch * grid(n)) && ec->wscratch.ensure(kWordsScratch * grid2(n) * kWaves) &&
               ec->ctl.ensure(sizeof(EncCtl)) && ec->meta.ensure(sizeof(BrickMeta) * (size_t)n) &&
               ec->sizes.ensure(4ull * n) && ec->aoff.ensure(8ull * n);
    }
    void bind() {
        a.ctl = ec->ctl.as<EncCtl>();
        a.meta = ec->meta.as<BrickMeta>();
        a.scratch = ec->scratch.as<uint8_t>();
        a.wscratch = ec->wscratch.as<uint8_t>();
        a.sizes = ec->sizes.as<uint32_t>();
        a.aoff = ec->aoff.as<uint64_t>();
        a.arena1 = ec->arena1.as<uint8_t>();
        a.arena2 = ec->arena2.as<uint8_t>();
        a.arena3 = ec->arena3.as<uint8_t>();
        a.cap1 = ec->cap1();
        a.cap3 = ec->arena3.bytes;
    }
    void symbols(bool keep_hist) {
        hipLaunchKernelGGL(begin_kernel, dim3(1), dim3(256), 0, s, a.ctl, keep_hist);
        hipLaunchKernelGGL(reuse_kernel, dim3(grid(a.n_items)), dim3(kReuseThreads), sizeof(ReuseLds), s, a);
        hipLaunchKernelGGL(palette_kernel, dim3(grid2(a.n_items)), dim3(kThreads), 0, s, a);
    }
    void gather(uint64_t rs) {
        uint64_t *index = reinterpret_cast<uint64_t *>(ec->dblob.as<uint8_t>() + csv::kHeaderBytes);
        hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, s, a, index);
        hipLaunchKernelGGL(pack_kernel, dim3(std::min<uint32_t>(a.n_items, cu * 8)), dim3(256), 0, s, a,
                           (const uint64_t *)index, ec->dblob.as<uint8_t>() + rs, ec->dblob.bytes - rs);
    }
    // The container of the a.n_items bricks (its header is not written),
    // there or in ec->dblob.  CSV_ENOMEM: the device's memory is short.  All
    // launches in one go, repeated with larger arenas if one was short
    // (arena 3's demand is only known once arena 1 held).
    int run(bool keep_hist) {
        const uint32_t n = a.n_items;
        const uint64_t rs = csv::record_area_offset(n);
        for (int pass = 0;; pass++) {
            bind();
            const uint64_t cap = std::min<uint64_t>(std::min<uint64_t>(ec->h_pin_bytes, ec->dblob.bytes), kPiecewise);
            symbols(keep_hist);
            hipLaunchKernelGGL(rans_kernel, dim3(grid2(n)), dim3(kThreads), 0, s, a);
            if (n <= kFinishMax) {
                hipLaunchKernelGGL(finish_kernel, dim3(std::min<uint32_t>(n, cu * 8)), dim3(256), 0, s, a, ec->h_ctl,
                                   ec->dblob.as<uint8_t>(), (uint64_t)ec->dblob.bytes, rs, ec->h_pin, cap);
            } else {
                gather(rs);
                hipLaunchKernelGGL(leave_kernel, dim3(kCopyGroups), dim3(256), 0, s, a, ec->h_ctl,
                                   (const uint8_t *)ec->dblob.as<uint8_t>(), rs, ec->h_pin, cap);
            }
            if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return CSV_EHIP;
            const EncCtl &c = *ec->h_ctl;
            if (c.top1 <= a.cap1 && c.top3 <= a.cap3) {
                bytes = rs + c.total;
                there = bytes < cap;
                if (bytes <= ec->dblob.bytes) return CSV_OK;
                // the records did not fit the container's buffer
                if (!ec->dblob.ensure(bytes)) return CSV_ENOMEM;
                gather(rs);
                return hipGetLastError() == hipSuccess ? CSV_OK : CSV_EHIP;
            }
            if (pass == 2 || !ec->arenas(c.top1) || !ec->arena3.ensure(c.top3)) return CSV_ENOMEM;
        }
    }
    // the last run's container, to host memory
    int take(uint8_t *to) {
        if (!there) return ec->bring(to, ec->dblob.as<uint8_t>(), bytes, s);
        std::memcpy(to, ec->h_pin, bytes);
        return CSV_OK;
    }
};

// containers of batches in host memory (the header of each unused)
struct Batches {
    struct Piece {
        Piece *next;
        uint32_t n;
        uint64_t bytes;
        uint8_t *at() { return reinterpret_cast<uint8_t *>(this + 1); }
    };
    Piece *head = nullptr, **tail = &head;
    uint64_t records = 0;
    ~Batches() {
        for (Piece *p = head; p;) {
            Piece *q = p->next;
            std::free(p);
            p = q;
        }
    }
    uint8_t *add(uint32_t n, uint64_t bytes) {
        Piece *p = static_cast<Piece *>(std::malloc(sizeof(Piece) + bytes));
        if (!p) return nullptr;
        p->next = nullptr;
        p->n = n;
        p->bytes = bytes;
        *tail = p;
        tail = &p->next;
        records += bytes - csv::record_area_offset(n);
        return p->at();
    }
    // the index and the records of the B bricks
    void join(uint8_t *out, uint32_t B) {
        uint8_t *to = out + csv::record_area_offset(B), *index = out + csv::kHeaderBytes;
        uint64_t at = 0;
        auto put = [&](uint64_t v) {  // (the caller's memory may have any alignment)
            std::memcpy(index, &v, 8);
            index += 8;
        };
        for (Piece *p = head; p; p = p->next) {
            const uint64_t rs = csv::record_area_offset(p->n), m = p->bytes - rs;
            const uint64_t *from = reinterpret_cast<const uint64_t *>(p->at() + csv::kHeaderBytes);
            for (uint32_t i = 0; i < p->n; i++) put(at + from[i]);
            std::memcpy(to + at, p->at() + rs, m);
            at += m;
        }
        put(at);
    }
};

// A compression in batches of bricks, for volumes that the device has no room
// for at once: the symbols of the sampled bricks first, for the frequency
// tables, then batch after batch, each of as many bricks as there is room for
// whatever they ask for (so that no launch has to be repeated).  All 4,096
// bricks of the 512^3 cells volume at once need 0.9 GB besides the container.
int in_batches(Compression &c, uint32_t B, uint32_t stride, Batches &out) {
    EncCache *ec = c.ec;
    uint32_t nb = (uint32_t)std::min<uint64_t>(B, (uint64_t)c.cu * kBatchPerCu);
    for (;; nb = (nb + 1) / 2) {
        ec->release_device();
        if (c.room(nb) && ec->arenas(kMostOps * nb) && ec->arena3.ensure(kMostRecord * nb) &&
            ec->dblob.ensure(csv::record_area_offset(nb) + kMostRecord * nb))
            break;
        if (nb == 1) return CSV_ENOMEM;
    }
    c.bind();
    c.a.step = stride;
    c.a.sample_stride = 1;
    const uint32_t samples = (uint32_t)(((uint64_t)B + stride - 1) / stride);
    for (uint64_t i = 0; i < samples; i += nb) {
        c.a.first = (uint32_t)(i * stride);
        c.a.n_items = (uint32_t)std::min<uint64_t>(nb, samples - i);
        c.symbols(i > 0);
    }
    c.a.step = 1;
    c.a.sample_stride = 0;
    for (uint64_t at = 0; at < B; at += nb) {
        c.a.first = (uint32_t)at;
        c.a.n_items = (uint32_t)std::min<uint64_t>(nb, B - at);
        int rc = c.run(true);
        if (rc) return rc;
        uint8_t *to = out.add(c.a.n_items, c.bytes);
        if (!to || (!c.there && !ec->pin(c.bytes))) return CSV_ENOMEM;
        rc = c.take(to);
        if (rc) return rc;
    }
    return CSV_OK;
}

}  // namespace

extern "C" int csv_encode_volume_gpu_alloc(const uint32_t *labels, uint32_t nx, uint32_t ny, uint32_t nz,
                                           const csv_encode_opts *opts, int device, void *stream,
                                           void *(*alloc)(size_t bytes, void *ctx), void *ctx, size_t *blob_bytes) {
    if (!labels || !alloc || !blob_bytes || !nx || !ny || !nz) return CSV_EINVAL;
    csv_encode_opts o;
    csv_encode_opts_default(&o);
    if (opts) o = *opts;
    if (o.brick_log2 != (uint32_t)kN || o.scale_bits < 8 || o.scale_bits > 12 || o.lane_k < 1 || o.lane_max < 1 ||
        o.lane_max > 64 || (o.lane_max & (o.lane_max - 1)) || o.tables > 2 || o.coding != 0)
        return CSV_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev || device >= kMaxDevices)
        return CSV_EINVAL;
    const uint32_t nbx = (nx + 31) / 32, nby = (ny + 31) / 32, nbz = (nz + 31) / 32;
    const uint64_t B64 = (uint64_t)nbx * nby * nbz;
    if (B64 >= (1ull << 32)) return CSV_ERANGE;
    const uint32_t B = (uint32_t)B64;
    const uint32_t stride = o.sample_stride ? o.sample_stride : (B64 > (1ull << 20) ? 4096u : 512u);
    DeviceGuard g(device);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int cu = 0;
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cu < 1) cu = 1;
    const uint64_t raw = (uint64_t)nx * ny * nz * 4;
    const uint64_t rs = csv::record_area_offset(B);
    EncCache *ec = cache_for(device);
    if (!ec) return CSV_ENOMEM;
    std::lock_guard<std::mutex> lk(ec->mu);  // one compression per device at a time
    InFlight flight(s);
    if (!ec->h_ctl &&
        hipHostMalloc(reinterpret_cast<void **>(&ec->h_ctl), sizeof(EncCtl), hipHostMallocDefault) != hipSuccess)
        return CSV_ENOMEM;
    if (!ec->pin(kPinFirst)) return CSV_ENOMEM;
    static std::once_flag once;
    std::call_once(once, [] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(reuse_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(ReuseLds));
    });
    Compression c;
    c.ec = ec;
    c.s = s;
    c.cu = (uint32_t)cu;
    EncArgs &a = c.a;
    std::memset(&a, 0, sizeof(a));
    a.vol = labels;
    a.nx = nx;
    a.ny = ny;
    a.nz = nz;
    a.nbx = nbx;
    a.nby = nby;
    a.step = 1;
    a.n_items = B;
    a.sample_stride = stride;
    a.bits = o.scale_bits;
    a.lane_k = o.lane_k;
    a.lane_max = o.lane_max;
    a.one_table = o.tables == 1 ? 1u : 0u;
    // arena 1 at first for a part of 1/12 of the labels (dense cells take
    // 1/15), or of 1/64 where that does not fit the device
    const bool fits = c.room(B) && ec->arena3.ensure(1ull << 20) &&
                      (ec->arenas(std::max<uint64_t>(16ull << 20, raw / 12)) ||
                       ec->arenas(std::max<uint64_t>(16ull << 20, raw / 64))) &&
                      ec->dblob.ensure(rs + std::max<uint64_t>(16ull << 20, raw / 32));
    int rc = fits ? c.run(false) : CSV_ENOMEM;
    Batches batches;
    const bool parts = rc == CSV_ENOMEM;
    if (parts) rc = in_batches(c, B, stride, batches);
    if (rc) return rc;
    const uint64_t total = parts ? rs + batches.records : c.bytes;
    if (!parts && !ec->pin(total)) return CSV_ENOMEM;
    uint8_t *out = static_cast<uint8_t *>(alloc(total, ctx));
    if (!out) return CSV_ENOMEM;
    if (parts) batches.join(out, B);
    else rc = c.take(out);
    if (rc) return rc;
    csv::VolumeHeader h;
    std::memset(&h, 0, sizeof(h));
    h.magic = csv::kMagic;
    h.version = csv::kVersion;
    h.nx = nx;
    h.ny = ny;
    h.nz = nz;
    h.brick_log2 = (uint32_t)kN;
    h.nbx = nbx;
    h.nby = nby;
    h.nbz = nbz;
    h.n_bricks = B;
    h.scale_bits = o.scale_bits;
    h.lane_k = o.lane_k;
    h.lane_max = o.lane_max;
    h.sample_stride = stride;
    for (int k = 0; k < 2; k++)
        for (int q = 0; q < 16; q++) h.freq[k][q] = ec->h_ctl->freq[k][q];
    std::memcpy(out, &h, sizeof(h));
    const uint64_t idx_end = csv::kHeaderBytes + 8ull * (B + 1);
    std::memset(out + idx_end, 0, rs - idx_end);  // padding before the record area
    *blob_bytes = total;
    flight.finished = true;
    return CSV_OK;
}

extern "C" int csv_encode_volume_gpu(const uint32_t *labels, uint32_t nx, uint32_t ny, uint32_t nz,
                                     const csv_encode_opts *opts, int device, void *stream, uint8_t **blob,
                                     size_t *blob_bytes) {
    if (!blob) return CSV_EINVAL;
    void *out = nullptr;
    const int rc = csv_encode_volume_gpu_alloc(
        labels, nx, ny, nz, opts, device, stream,
        [](size_t bytes, void *ctx) -> void * { return *static_cast<void **>(ctx) = std::malloc(bytes); }, &out,
        blob_bytes);
    if (rc) std::free(out);
    else *blob = static_cast<uint8_t *>(out);
    return rc;
}

extern "C" int csv_encode_gpu_release(int device) {
    if (device < 0 || device >= kMaxDevices) return CSV_EINVAL;
    EncCache *ec;
    {
        std::lock_guard<std::mutex> lk(g_cache_mu);
        ec = g_cache[device];
    }
    if (!ec) return CSV_OK;
    DeviceGuard g(device);
    std::lock_guard<std::mutex> lk(ec->mu);
    (void)hipDeviceSynchronize();
    ec->release();
    return CSV_OK;
}

#ifdef CSV_PHASE_TIMING
// install (or clear, with NULL) a device buffer of 8 u64 clocks per workgroup
extern "C" int csv_debug_enc_phase_buffer(uint64_t *dev_buf) {
    return hipMemcpyToSymbol(HIP_SYMBOL(g_enc_phase), &dev_buf, sizeof(dev_buf)) == hipSuccess ? CSV_OK : CSV_EHIP;
}
#endif
