// Decoder for 64^3 bricks with palettes of fewer than k64PalMax entries,
// rANS or raw nibbles; part of csv_decode.hip, whose helpers it uses.  The
// launches of a decode:
//   entropy64_kernel  (pools with rANS volumes) one wave per brick: the
//                     symbols as packed nibbles in the request's slot (few
//                     requests or symbols: a wave of upper64_kernel instead);
//                     raw bricks are read where they lie in the record;
//   front_kernel      (of csv_decode.hip; many requests of t >= 2) a wave per
//                     brick, which is a 32^3 brick of level t - 1 then;
//   split64_kernel    (levels by request, more requests than slots) a list of
//                     those of levels 0 and 1, for the kernels below;
//   upper64_kernel    a workgroup per brick: levels 5 .. max(t, 1) in LDS
//                     (u16 palette indices, Morton order), one lane per
//                     parent; t >= 1: the output.  t = 0: level 1, its
//                     expansion bits and, per expanded level-1 node, the P_a
//                     and P_delta operations before it go to the slot, and
//                     everything that could be malformed in level 0 is
//                     checked here;
//   leaf64_kernel     one wave per block of 32 x 8 x 8 voxels: its expanded
//                     parents 64 at a time, in no order that matters (each
//                     has its own counts), the block in LDS, the output in
//                     rows of 128 bytes.  References out of the block are
//                     evaluated on the other block's operations.
// The finest level of a 64^3 brick (512 KB of u16) does not fit LDS; blocks
// that need nothing of each other's results keep it out of global memory
// and give 128 waves of work per brick.  512 raw bricks of the 512^3 cells
// volume, full LOD: 267 us for the call (2.01 TB/s of labels); with a
// workgroup per brick and its levels in global scratch 2.73 ms.

constexpr uint32_t k64PalMax = 1u << 14;  // P_a counts of a slot have 14 bits
constexpr int k64Threads = 512;           // of an upper workgroup
constexpr uint32_t k64Waves = k64Threads / 64;

// The slot of a request (bytes): level 1, its expansion bits, the expanded
// nodes before each 64 of them, Head64, per expanded node its counts, the
// nibbles (pools with rANS volumes)
constexpr uint32_t k64Bits = 2 * 32768, k64Pre = k64Bits + 4096, k64Head = k64Pre + 1024, k64Info = k64Head + 256;

struct Head64 {
    uint32_t leaf;  // 1: a full-LOD request for leaf64_kernel
    uint32_t bad;   // 1: the entropy decode failed
    uint32_t P, ops0, seg, ipl;
    uint64_t pal, nib, dst;
};
static_assert(sizeof(Head64) <= 256, "slot layout");

// nibble dwords of a wave's slot for levels 5 .. 2 (585 parents at most, 16
// symbols each), and the 16 that entropy_decode may write past them
constexpr uint32_t k64CoarseDw = 585 * 16 / 8 + 14;
static_assert(k64CoarseDw % 4 == 0, "levels behind it");
static_assert(k64Info >= kWavesGen * (4 * k64CoarseDw + kSlotLv), "a request's slot holds those of a front workgroup");

struct Launch64 {
    uint8_t *slots;
    uint64_t slot_bytes;
    uint32_t nib_off;        // nibbles in a slot
    uint32_t nib_dw;         // dwords they may take
    uint32_t lut_lds_words;  // decode-table words in LDS (entropy kernel; 0: read from global memory)
    // levels by request in more than one chunk: the requests of levels 0 and 1
    // (nullptr: requests 0 .. n - 1), how many there are, the chunk's first one
    const uint32_t *list, *count;
    uint32_t base;
};

// requests of a launch, and the i-th of them
__device__ __forceinline__ uint32_t requests64(const DecodeArgs &a, const Launch64 &l) {
    if (!l.list) return a.n;
    const uint32_t c = ld_s(l.count);
    return c > l.base ? min(a.n, c - l.base) : 0u;
}
__device__ __forceinline__ uint32_t request64(const Launch64 &l, uint32_t i) {
    return l.list ? ld_s(l.list + l.base + i) : i;
}

// Lists the requests of levels 0 and 1 (list, *count from zero), in no order:
// a counter step per workgroup.  Without it a chunk of a batch with mostly
// coarser levels holds few of these, and every chunk takes as long as one
// full-LOD brick: 200,000 requests, one in 200 at full LOD, 57 ms.
__global__ __launch_bounds__(256) void split64_kernel(const uint8_t *lods, uint32_t n, uint32_t *list, uint32_t *count) {
    __shared__ uint32_t part[4], first;
    const uint32_t i = blockIdx.x * 256u + threadIdx.x, w = threadIdx.x >> 6;
    const uint64_t m = __ballot(i < n && lods[i] < 2);
    if (lane() == 0) part[w] = (uint32_t)__popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) first = atomicAdd(count, part[0] + part[1] + part[2] + part[3]);
    __syncthreads();
    uint32_t at = first;
#pragma unroll
    for (uint32_t v = 0; v < 4; v++) at += v < w ? part[v] : 0u;
    if ((m >> lane()) & 1u) list[at + mbcnt(m)] = i;
}

struct Hdr64 {
    const uint32_t *rec;
    uint32_t P, W, nw, t, vol, id;
    bool raw;
    uint32_t c[6];  // c[m]: symbols in the segments of child levels 5 .. m
};

__device__ __forceinline__ ReqKind load_request64(const DecodeArgs &a, uint32_t rq, Hdr64 &h, uint32_t *&dst,
                                                  uint32_t &count, uint32_t &fill) {
    h.id = ld_s(a.ids + rq);
    h.t = a.lods ? ld_s_u8(a.lods + rq) : a.lod_scalar;
    dst = nullptr;
    count = 0;
    fill = 0;
    if (h.t > 6u) return kReqBadLod;
    const uint32_t G = 64u >> h.t;
    count = G * G * G;
    dst = a.out + (a.out_off ? ld_s(a.out_off + rq) : (uint64_t)rq * count);
    if (h.id >= a.n_bricks) return kReqBadId;
    h.rec = rec_at(ld_s(a.rec_ptr + h.id));
    const uint32_t size = ld_s(a.rec_size + h.id);
    h.vol = ld_s_u16(a.rec_vol + h.id);
    h.raw = ld_s_u8(a.vol_raw + h.vol) != 0;
    h.P = ld_s(h.rec + 0);
    h.W = ld_s(h.rec + 1);
    h.nw = ld_s(h.rec + 2);
    bool ok = true;
#pragma unroll
    for (int m = 0; m < 6; m++) {
        h.c[m] = ld_s(h.rec + 3 + m);
        if (m > 0) ok = ok && h.c[m] <= h.c[m - 1];
    }
    const uint32_t c0 = h.c[0], hdr = csv::record_header_words(6);
    ok = ok && h.P < k64PalMax && (c0 == 0 ? h.P == 1 : h.P >= 2);
    ok = ok && (h.raw ? (h.W == 0 && h.nw == (c0 + 3) / 4)
                      : (h.W <= 64 && (h.W & (h.W - 1)) == 0 && (c0 > 0) == (h.W > 0)));
    ok = ok && 4ull * ((uint64_t)hdr + h.P + h.W) + 2ull * h.nw <= size;
    if (!ok) return kReqCorrupt;
    if (h.t == 6u || c0 == 0) {
        fill = ld_s(h.rec + hdr);
        return kReqFill;
    }
    return kReqDecode;
}

// 5-bit coordinate -> Morton bit positions 0, 3, .., 12, and back
__device__ __forceinline__ uint32_t spread5(uint32_t v) { return spread4(v) | ((v & 16u) << 8); }
__device__ __forceinline__ uint32_t coord5(uint32_t p) {
    return (p & 1u) | ((p >> 2) & 2u) | ((p >> 4) & 4u) | ((p >> 6) & 8u) | ((p >> 8) & 16u);
}

// Children of one expanded parent (its 8 nibbles wd) as u16 indices: pv the
// parent's index, nb the parent level's +1 neighbours, ipb the palette
// position before the first child, pam / pdm its P_a / P_delta children
// (bit 4k), dl its deltas.  As replay_children_u8, with low and high bytes
// selected apart and then paired; nothing is checked here.
__device__ __forceinline__ uint4 replay_children_u16(uint32_t wd, uint32_t pv, const uint32_t nb[3], uint32_t ipb,
                                                     uint32_t pam, uint32_t pdm, uint32_t dl) {
    auto perm = [](uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); };
    // selector bytes (child_selectors): marks 0..2, parent 4, neighbours 5..7, zero 12
    const uint32_t ye = wd & 0x07070707u, yo = (wd >> 4) & 0x07070707u;
    const uint32_t be = perm(0x0C0C0C0Cu, 0x02010004u, ye), bo = perm(0x0C0C0C0Cu, 0x02010004u, yo);
    const uint32_t f2e = perm(0u, 0x00050000u, ye), f3e = perm(0u, 0x05000000u, ye);
    const uint32_t f1o = perm(0u, 0x00000500u, yo), f2o = perm(0u, 0x00050000u, yo), f3o = perm(0u, 0x05000000u, yo);
    const uint32_t se = be + ((f2e & 0xFF00FF00u) | (f3e & 0xFFFF0000u));
    const uint32_t so = bo + (f1o | (f2o & 0xFF00FF00u) | (f3o & 0xFFFF0000u));
    const uint32_t sel_lo = perm(so, se, 0x05010400u), sel_hi = perm(so, se, 0x07030602u);
    // low and high bytes of {parent, neighbours}; the marks are 0xFFFD .. 0xFFFF
    const uint32_t t01 = perm(nb[0], pv, 0x05010400u), t23 = perm(nb[2], nb[1], 0x05010400u);
    const uint32_t cl = perm(t23, t01, 0x05040100u), ch = perm(t23, t01, 0x07060302u);
    const uint32_t l0 = perm(cl, 0x00FFFEFDu, sel_lo), h0 = perm(ch, 0x00FFFFFFu, sel_lo);
    const uint32_t l1 = perm(cl, 0x00FFFEFDu, sel_hi), h1 = perm(ch, 0x00FFFFFFu, sel_hi);
    // palette positions after the parent's first one: P_a children so far
    // (itself included), on the P operations' bytes
    const uint32_t y = wd & 0x77777777u, wp = (y >> 2) & 0x11111111u;
    const uint32_t pa0 = nib_to_bytes(pam), pa1 = nib_to_bytes(pam >> 16), pb0 = nib_to_bytes(wp),
                   pb1 = nib_to_bytes(wp >> 16);
    const uint32_t m0 = (pb0 << 8) - pb0, m1 = (pb1 << 8) - pb1;
    const uint32_t c0 = pa0 * 0x01010101u, c1 = pa1 * 0x01010101u + (c0 >> 24) * 0x01010101u;
    const uint32_t p0 = c0 & m0, p1 = c1 & m1, ip2 = ipb * 0x00010001u;
    uint4 v;
    v.x = perm(h0, l0, 0x05010400u) + perm(0u, p0, 0x0C010C00u) + (ip2 & perm(0u, m0, 0x01010000u));
    v.y = perm(h0, l0, 0x07030602u) + perm(0u, p0, 0x0C030C02u) + (ip2 & perm(0u, m0, 0x03030202u));
    v.z = perm(h1, l1, 0x05010400u) + perm(0u, p1, 0x0C010C00u) + (ip2 & perm(0u, m1, 0x01010000u));
    v.w = perm(h1, l1, 0x07030602u) + perm(0u, p1, 0x0C030C02u) + (ip2 & perm(0u, m1, 0x03030202u));
    while (pdm) {  // delta d: the entry d + 1 before
        const uint32_t k4 = (uint32_t)__builtin_ctz(pdm), j = k4 >> 3;
        const uint32_t sub = ((dl & 15u) + 1u) << (4 * (k4 & 4u));
        pdm &= pdm - 1u;
        dl >>= 4;
        v.x -= j == 0 ? sub : 0u;
        v.y -= j == 1 ? sub : 0u;
        v.z -= j == 2 ? sub : 0u;
        v.w -= j == 3 ? sub : 0u;
    }
    return v;
}
// nibbles of wd whose reference leaves the brick: q on a low or high face of
// the grid with axis mask pm
__device__ __forceinline__ uint32_t leaving(uint32_t wd, uint32_t q, uint32_t pm) {
    const uint32_t y = wd & 0x77777777u;
    uint32_t out = 0;
#pragma unroll
    for (int x = 0; x < 3; x++) {
        const uint32_t side = x == 0 ? 0x01010101u : x == 1 ? 0x00110011u : 0x00001111u;  // children at 0 on the axis
        const uint32_t am = pm << x, v = q & am;
        const uint32_t face = (v == 0 ? side : 0u) | (v == am ? 0x11111111u ^ side : 0u);
        out |= zero_nibbles(y ^ (0x11111111u * (uint32_t)(x + 1))) & face;
    }
    return out;
}

// a delta past the first palette entry (dl: the deltas of the P_delta
// children pdm); positions from 16 on hold any
__device__ __forceinline__ bool short_delta(uint32_t ipb, uint32_t pam, uint32_t pdm, uint32_t dl) {
    bool bad = false;
    if (ipb < 16u)
        for (; pdm; dl >>= 4) {
            const uint32_t k4 = (uint32_t)__builtin_ctz(pdm);
            pdm &= pdm - 1u;
            bad |= ipb + (uint32_t)__builtin_popcount(pam & ((1u << k4) - 1u)) < (dl & 15u) + 1u;
        }
    return bad;
}

// The symbols of request g as packed nibbles in its slot, by one wave with wl
// (kWaveLds bytes) of LDS; false on a malformed stream
template <bool kLutLds>
__device__ __forceinline__ bool entropy64(const DecodeArgs &a, const Launch64 &l, const Hdr64 &g, uint8_t *slot,
                                          const uint32_t *slut, uint8_t *wl) {
    const uint32_t n = g.t == 0   ? g.c[0]
                       : g.t == 1 ? g.c[1]
                       : g.t == 2 ? g.c[2]
                       : g.t == 3 ? g.c[3]
                       : g.t == 4 ? g.c[4]
                                  : g.c[5];
    if (n + 16 > 8 * l.nib_dw) return false;
    Hdr h;
    h.rec = g.rec;
    h.sfx = nullptr;
    h.pdw = 0xFFFFFFFFu;
    h.P = g.P;
    h.W = g.W;
    h.nw = g.nw;
    h.vol = g.vol;
    h.t = g.t - 1u;  // (levels of a 64^3 brick are one above those of Hdr)
    h.c0 = g.c[1];
    h.c1 = 0;
    uint32_t words = 0;
    return entropy_decode<kLutLds, -1, true>(a, h, slut, reinterpret_cast<uint32_t *>(wl),
                                             reinterpret_cast<uint32_t *>(slot + l.nib_off),
                                             reinterpret_cast<uint32_t *>(wl + kWPal), n, words);
}

// One wave per rANS request; a serial chain of c_t / 64 steps (a brick of
// the 512^3 cells volume has 100,000 symbols), so a launch of 512 bricks is
// bound by that chain's latency, not by the machine.
template <bool kLutLds>
__global__ __launch_bounds__(64 * kWavesGen) void entropy64_kernel(DecodeArgs a, Launch64 l) {
    extern __shared__ __align__(16) uint8_t smem[];
    uint32_t *slut = reinterpret_cast<uint32_t *>(smem);
    if (kLutLds)
        for (uint32_t e = threadIdx.x; e < l.lut_lds_words; e += blockDim.x) slut[e] = a.luts[e];
    __syncthreads();
    const uint32_t wave = uniform(threadIdx.x >> 6);
    uint8_t *wl = smem + align16(4 * l.lut_lds_words) + wave * kWaveLds;
    const uint32_t n = requests64(a, l);
    for (uint32_t i = blockIdx.x * kWavesGen + wave; i < n; i += gridDim.x * kWavesGen) {
        Hdr64 g;
        uint32_t *dst, count, fill;
        const ReqKind kind = load_request64(a, request64(l, i), g, dst, count, fill);
        if (kind != kReqDecode || g.raw) continue;
        uint8_t *slot = glob(l.slots) + (size_t)i * l.slot_bytes;
        const bool ok = entropy64<kLutLds>(a, l, g, slot, slut, wl);
        wsync();
        if (lane() == 0) reinterpret_cast<Head64 *>(slot + k64Head)->bad = ok ? 0u : 1u;
    }
}

// Who decodes the symbols before upper64_kernel replays them: a launch of
// entropy64_kernel, or the workgroup's own first wave, with the tables in LDS
// (in the place of level 1, which comes later) or in global memory
enum class Symbols64 { kLaunch, kOwnLds, kOwnGlobal };

// LDS of an upper workgroup: levels 2..5 and the root (u16), level 1, the
// expansion bits of levels 1..5 and of the root (64-bit words), expanded
// nodes before each word of the parent level, per-wave counts
__device__ constexpr uint32_t k64Lv[7] = {0, 0, 0, 4096, 4608, 4672, 4680};
__device__ constexpr uint32_t k64Bm[7] = {0, 0, 512, 576, 584, 585, 586};  // words of level m
constexpr uint32_t kU64L1 = 2 * 4688, kU64Bm = kU64L1 + 65536, kU64Pre = kU64Bm + 8 * 588, kU64Sm = kU64Pre + 1024,
                   kU64Lds = kU64Sm + 96;
static_assert(kLutLdsCap + kWaveLds <= 65536, "tables and a decoding wave in the place of level 1");

// What bounds it: latency (a chain of six levels with a few barriers and
// dependent loads each, at the two workgroups per CU that 80 KB of LDS
// allow) and vector issue (6.6 k wave-instructions per wave, 60 % of the
// time).  512 bricks of the 512^3 cells volume take 82 us; with a lane per
// parent instead of per expanded parent, the counts of level 0 scanned 64 at
// a time and deltas read child by child it was 118 us.
template <Symbols64 kSym>
__global__ __launch_bounds__(k64Threads) __attribute__((amdgpu_waves_per_eu(4))) void upper64_kernel(DecodeArgs a,
                                                                                                   Launch64 l) {
    extern __shared__ __align__(16) uint8_t smem[];
    uint16_t *lv = reinterpret_cast<uint16_t *>(smem);
    uint16_t *l1 = reinterpret_cast<uint16_t *>(smem + kU64L1);
    uint64_t *bmw = reinterpret_cast<uint64_t *>(smem + kU64Bm);
    uint16_t *pre = reinterpret_cast<uint16_t *>(smem + kU64Pre);
    uint32_t *wt = reinterpret_cast<uint32_t *>(smem + kU64Sm);  // per wave: P_a, P_delta counts
    uint32_t *tot = wt + 2 * k64Waves;                           // expanded parents
    uint32_t *bad = tot + 1;
    const uint32_t tid = threadIdx.x, L = lane(), w = uniform(tid >> 6), hdr = csv::record_header_words(6);
    constexpr uint32_t kMark = 65533u;
    using V = Vec8<uint16_t>;
    const uint32_t n = requests64(a, l);
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
        const uint32_t rq = request64(l, i);
        uint8_t *slot = glob(l.slots) + (size_t)i * l.slot_bytes;
        Head64 *head = reinterpret_cast<Head64 *>(slot + k64Head);
        Hdr64 h;
        uint32_t *dst, count, fill;
        const ReqKind kind = load_request64(a, rq, h, dst, count, fill);
        __syncthreads();  // LDS of the request before
        if (tid == 0) {
            head->leaf = 0;
            *bad = (kSym == Symbols64::kLaunch && kind == kReqDecode && !h.raw) ? head->bad : 0u;
            bmw[k64Bm[6]] = 1;
            bmw[k64Bm[5]] = 0;  // (8 of the word's bits are nodes)
            lv[k64Lv[6]] = 0;
        }
        if (kind == kReqBadLod) {
            if (tid == 0) fail(a, rq, CSV_ERANGE, a.rq_base + rq);
            continue;
        }
        if (kind != kReqDecode) {
            if (kind != kReqFill && tid == 0)
                fail(a, rq, kind == kReqBadId ? CSV_ERANGE : CSV_ECORRUPT, kind == kReqBadId ? a.rq_base + rq : h.id);
            fill_labels<k64Threads>(dst, count, kind == kReqFill ? fill : 0u, tid);
            continue;
        }
        const uint32_t t = h.t, P = h.P;
        const uint32_t *nib = h.raw ? h.rec + hdr + P : reinterpret_cast<const uint32_t *>(slot + l.nib_off);
        if (h.raw && t == 0 && (h.c[0] & 3u) && tid == 0) {
            // a complete decode finds the last word's unused nibbles zero
            const uint32_t last = (nib[(h.nw - 1) / 2] >> (16 * ((h.nw - 1) & 1u))) & 0xFFFFu;
            if ((last >> (4 * (h.c[0] & 3u))) != 0) *bad = 1;
        }
        uint32_t ipl = 0;
        bool ok = true;
        if constexpr (kSym != Symbols64::kLaunch) {
            constexpr bool kLds = kSym == Symbols64::kOwnLds;
            uint32_t *slut = reinterpret_cast<uint32_t *>(smem + kU64L1);
            if (!h.raw) {
                if (kLds)
                    for (uint32_t e = tid; e < l.lut_lds_words; e += k64Threads) slut[e] = a.luts[e];
                __syncthreads();
                if (w == 0 && !entropy64<kLds>(a, l, h, slot, slut, smem + kU64L1 + kLutLdsCap) && L == 0) *bad = 1;
            }
        }
        __syncthreads();
        if (*bad) ok = false;
        // node of rank r among the expanded nodes whose bits are pb and
        // whose counts before each of 2^lw words are pre: the word by binary
        // search, the bit by halving
        auto node_of = [&](const uint64_t *pb, uint32_t lw, uint32_t r) -> uint32_t {
            uint32_t word = 0;
            for (uint32_t h = (1u << lw) >> 1; h; h >>= 1) word += pre[word + h] <= r ? h : 0u;
            const uint64_t b = pb[word];
            uint32_t n = r - pre[word], pos = 0, x = (uint32_t)b;
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
            return 64 * word + pos;
        };
        // child level m from the 8^(5 - m) nodes of level m + 1.  The
        // expanded ones go to the waves in runs of chunks of 64, so that no
        // lane idles at nodes that are not (two of three in the cells volume).
        auto level = [&](uint32_t m, uint32_t seg, uint32_t seg_end) __attribute__((always_inline)) -> bool {
            const uint32_t Bp = 5 - m, np = 1u << (3 * Bp), lw = Bp > 2 ? 3 * Bp - 6 : 0u, nw = 1u << lw;
            const uint64_t *pb = bmw + k64Bm[m + 1];
            const uint16_t *up = lv + k64Lv[m + 1];
            uint16_t *cur = m == 1 ? l1 : lv + k64Lv[m];
            uint8_t *cb = reinterpret_cast<uint8_t *>(bmw + k64Bm[m]);
            if (w == 0) {
                const uint32_t c = L < nw ? (uint32_t)__popcll(pb[L]) : 0u;
                const uint32_t inc = wave_incl_scan(c);
                pre[L] = (uint16_t)(inc - c);
                if (L == 63) *tot = inc;
            }
            // every child its parent's value; those of expanded nodes are
            // overwritten below
            for (uint32_t q = tid; q < np; q += k64Threads) {
                *reinterpret_cast<typename V::T *>(cur + 8 * q) = V::splat(up[q]);
                cb[q] = 0;
            }
            __syncthreads();
            const uint32_t E = *tot;
            if ((uint64_t)seg + 8ull * E > seg_end) return false;
            const uint32_t D = seg_end - seg - 8 * E, ops0 = seg + D;  // deltas precede the operations
            const uint32_t nch = (E + 63) / 64, cpw = (nch + k64Waves - 1) / k64Waves;
            const uint32_t c0 = min(w * cpw, nch), c1 = min(c0 + cpw, nch);
            uint32_t sum = 0;
#pragma unroll 4
            for (uint32_t c = c0; c < c1; c++) {
                const uint32_t r = 64 * c + L, y = (r < E ? nib8(nib, ops0 + 8 * r) : 0u) & 0x77777777u;
                sum += (uint32_t)__builtin_popcount(zero_nibbles(y ^ 0x66666666u)) |
                       ((uint32_t)__builtin_popcount(zero_nibbles(y ^ 0x55555555u)) << 16);
            }
            sum = uniform(__builtin_amdgcn_readlane(wave_incl_scan(sum), 63));
            if (L == 0) wt[w] = sum;
            __syncthreads();
            uint32_t bpa = 0, bpd = 0, tpa = 0, tpd = 0;
#pragma unroll
            for (uint32_t v = 0; v < k64Waves; v++) {
                const uint32_t s = wt[v];
                if (v < w) {
                    bpa += s & 0xFFFFu;
                    bpd += s >> 16;
                }
                tpa += s & 0xFFFFu;
                tpd += s >> 16;
            }
            if (tpd != D) return false;
            const uint32_t pm = axis_mask(0, Bp);
            bool wrong = ipl + tpa >= P;  // the last new palette entry
#pragma unroll 1
            for (uint32_t c = c0; c < c1; c++) {
                const uint32_t r = 64 * c + L;
                const bool act = r < E;
                const uint32_t wd = act ? nib8(nib, ops0 + 8 * r) : 0u;
                uint32_t pam, pdm, exm, cnt;
                nibble_counts(wd, act, pam, pdm, exm, cnt);
                const uint32_t inc = wave_incl_scan(cnt & 0xFFFFFu), exc = inc - (cnt & 0xFFFFFu);
                const uint32_t all = uniform(__builtin_amdgcn_readlane(inc, 63));
                if (act) {
                    const uint32_t dl = pdm ? nib8(nib, seg + bpd + (exc >> 10)) : 0u;
                    const uint32_t q = node_of(pb, lw, r);
                    uint32_t nb[3];
#pragma unroll
                    for (int x = 0; x < 3; x++) {  // (on a high face: any value)
                        const uint32_t am = pm << x;
                        nb[x] = up[morton_inc(q, am)];
                    }
                    const uint32_t ipb = ipl + bpa + (exc & 1023u);
                    *reinterpret_cast<typename V::T *>(cur + 8 * q) =
                        replay_children_u16(wd, up[q], nb, ipb, pam, pdm, dl);
                    cb[q] = (uint8_t)compact_nibble_bits(exm);
                    wrong |= leaving(wd, q, pm) != 0 || zero_nibbles((wd & 0x77777777u) ^ 0x77777777u) != 0 ||
                             short_delta(ipb, pam, pdm, dl);
                }
                bpa += all & 1023u;
                bpd += all >> 10;
            }
            if (__ballot(wrong) && L == 0) atomicOr(bad, 1u);
            __syncthreads();
            if (*bad) return false;
            // references to the same-level node at -1, followed to their
            // values (at most three links; a reader sees a reference or its
            // final value, and both lead to the value)
#pragma unroll 1
            for (uint32_t c = c0; c < c1; c++) {
                const uint32_t r = 64 * c + L;
                if (r >= E) continue;
                const uint32_t wd = nib8(nib, ops0 + 8 * r);
                uint32_t open = ref_children(wd, 7u);
                const uint32_t q = node_of(pb, lw, r);
                while (open) {
                    uint32_t kk = (uint32_t)__builtin_ctz(open) >> 2, qq = q;
                    const uint32_t at = 8 * q + kk;
                    open &= open - 1u;
                    uint32_t v = cur[at];
                    while (v >= kMark) {
                        const uint32_t x = v - kMark;
                        qq = morton_dec(qq, pm << x);
                        kk |= 1u << x;
                        v = cur[8 * qq + kk];
                    }
                    cur[at] = (uint16_t)v;
                }
            }
            ipl += tpa;
            __syncthreads();
            return true;
        };
        const uint32_t tl = t > 1 ? t : 1u;
        auto cum = [&](uint32_t m) -> uint32_t {
            return m == 5 ? h.c[5] : m == 4 ? h.c[4] : m == 3 ? h.c[3] : m == 2 ? h.c[2] : m == 1 ? h.c[1] : 0u;
        };
#pragma unroll 1
        for (uint32_t m = 5; ok && m >= tl; m--) ok = level(m, cum(m + 1), cum(m));
        const uint32_t *pal = h.rec + hdr;
        if (ok && t >= 1) {  // level t to the output (every index has been checked against P)
            const uint32_t lg = 6 - t, G = 1u << lg;
            const uint16_t *res = t == 1 ? l1 : lv + (t == 2 ? 0u : t == 3 ? 4096u : t == 4 ? 4608u : 4672u);
            if (t == 5) {
                if (tid < 8) dst[tid] = pal[res[tid]];  // Morton order equals dense order on 2^3
            } else {
                const bool al = (reinterpret_cast<uintptr_t>(dst) & 15) == 0;
                for (uint32_t e = 4 * tid; e < count; e += 4 * k64Threads) {
                    const uint32_t x = e & (G - 1), y = (e >> lg) & (G - 1), z = e >> (2 * lg);
                    const uint32_t m0 = spread5(x) | (spread5(y) << 1) | (spread5(z) << 2);
                    const uint4 o = make_uint4(pal[res[m0]], pal[res[m0 | 1u]], pal[res[m0 | 8u]], pal[res[m0 | 9u]]);
                    if (al) store4<true>(dst + e, o);
                    else store4<false>(dst + e, o);
                }
            }
            continue;
        }
        // t = 0: what leaf64_kernel needs of the levels above
        const uint64_t *b1 = bmw + k64Bm[1];
        uint32_t ops0 = 0;
        const uint32_t seg = h.c[1], seg_end = h.c[0];
        if (ok) {
            const uint32_t c = (uint32_t)__popcll(b1[tid]), inc = wave_incl_scan(c);
            if (L == 63) wt[w] = inc;
            __syncthreads();
            uint32_t before = 0, E = 0;
#pragma unroll
            for (uint32_t v = 0; v < k64Waves; v++) {
                before += v < w ? wt[v] : 0u;
                E += wt[v];
            }
            pre[tid] = (uint16_t)(before + inc - c);
            __syncthreads();
            ok = (uint64_t)seg + 8ull * E <= seg_end;
            if (ok) {
                // per expanded node the P_a and P_delta operations before it:
                // a wave takes a run of nodes in stream order, 512 at a time
                // (8 per lane, one scan), its totals first.  The operations
                // are checked: no stop bit, no code 7, deltas and palette
                // positions in range.
                const uint32_t D = seg_end - seg - 8 * E;
                ops0 = seg + D;
                const uint32_t nch = (E + 511) / 512, cpw = (nch + k64Waves - 1) / k64Waves;
                const uint32_t cb = min(w * cpw, nch), ce = min(cb + cpw, nch);
                // node r's operations (none past the end); P_a | P_delta << 16
                auto ops_at = [&](uint32_t r) -> uint32_t { return r < E ? nib8(nib, ops0 + 8 * r) : 0u; };
                auto counts = [&](uint32_t wd) -> uint32_t {
                    const uint32_t y = wd & 0x77777777u;
                    return (uint32_t)__builtin_popcount(zero_nibbles(y ^ 0x66666666u)) |
                           ((uint32_t)__builtin_popcount(zero_nibbles(y ^ 0x55555555u)) << 16);
                };
                uint32_t sum = 0;
                bool wrong = false;
                for (uint32_t ch = cb; ch < ce; ch++) {
                    uint32_t part = 0;
#pragma unroll
                    for (uint32_t k = 0; k < 8; k++) {
                        const uint32_t wd = ops_at(512 * ch + 64 * k + L);
                        part += counts(wd);
                        wrong |= (wd & 0x88888888u) != 0 || zero_nibbles((wd & 0x77777777u) ^ 0x77777777u) != 0;
                    }
                    sum += part;
                }
                uint32_t spa = uniform(__builtin_amdgcn_readlane(wave_incl_scan(sum & 0xFFFFu), 63));
                uint32_t spd = uniform(__builtin_amdgcn_readlane(wave_incl_scan(sum >> 16), 63));
                if (L == 0) {
                    wt[2 * w] = spa;
                    wt[2 * w + 1] = spd;
                }
                __syncthreads();
                uint32_t bpa = 0, bpd = 0, tpa = 0, tpd = 0;
#pragma unroll
                for (uint32_t v = 0; v < k64Waves; v++) {
                    const uint32_t s0 = wt[2 * v], s1 = wt[2 * v + 1];
                    if (v < w) {
                        bpa += s0;
                        bpd += s1;
                    }
                    tpa += s0;
                    tpd += s1;
                }
                ok = tpd == D && ipl + tpa < P;
                if (ok) {
                    uint32_t *info = reinterpret_cast<uint32_t *>(slot + k64Info);
                    for (uint32_t ch = cb; ch < ce; ch++) {
                        const uint32_t r0 = 512 * ch + 8 * L;
                        uint32_t cnt[8], part = 0;
#pragma unroll
                        for (uint32_t k = 0; k < 8; k++) {
                            const uint32_t c = counts(ops_at(r0 + k));
                            cnt[k] = part;
                            part += c;
                        }
                        const uint32_t inc = wave_incl_scan(part), exc = inc - part;
                        const uint32_t all = uniform(__builtin_amdgcn_readlane(inc, 63));
                        uint32_t o[8];
#pragma unroll
                        for (uint32_t k = 0; k < 8; k++) {
                            const uint32_t e = exc + cnt[k];
                            o[k] = (bpa + (e & 0xFFFFu)) | ((bpd + (e >> 16)) << 14);
                        }
                        // (the slot has room for whole groups of 8)
                        if (r0 < E) {
                            reinterpret_cast<uint4 *>(info + r0)[0] = make_uint4(o[0], o[1], o[2], o[3]);
                            reinterpret_cast<uint4 *>(info + r0)[1] = make_uint4(o[4], o[5], o[6], o[7]);
                        }
                        if (ipl + bpa < 16u)
                            for (uint32_t k = 0; k < 8; k++) {
                                const uint32_t wd = ops_at(r0 + k), y = wd & 0x77777777u;
                                const uint32_t in = o[k], pdm = zero_nibbles(y ^ 0x55555555u);
                                if (pdm)
                                    wrong |= short_delta(ipl + (in & (k64PalMax - 1u)), zero_nibbles(y ^ 0x66666666u),
                                                         pdm, nib8(nib, seg + (in >> 14)));
                            }
                        bpa += all & 0xFFFFu;
                        bpd += all >> 16;
                    }
                    // references of nodes on the brick's six faces must stay inside
#pragma unroll 4
                    for (uint32_t e = tid; e < 6 * 1024; e += k64Threads) {
                        const uint32_t x = e >> 11, u = spread5(e & 31u), v = spread5((e >> 5) & 31u);
                        const uint32_t am = 0x1249u << x, fixed = (e & 1024u) ? am : 0u;
                        const uint32_t q = fixed | (x == 0 ? (u << 1) | (v << 2) : x == 1 ? u | (v << 2) : u | (v << 1));
                        const uint64_t b = b1[q >> 6];
                        if ((b >> (q & 63u)) & 1u) {
                            const uint32_t r = pre[q >> 6] + (uint32_t)__popcll(b & ((1ull << (q & 63u)) - 1ull));
                            wrong |= leaving(nib8(nib, ops0 + 8 * r), q, 0x1249u) != 0;
                        }
                    }
                }
                if (__ballot(wrong) && L == 0) atomicOr(bad, 1u);
            }
            __syncthreads();
            if (*bad) ok = false;
        }
        if (!ok) {
            if (tid == 0) fail(a, rq, CSV_ECORRUPT, h.id);
            fill_labels<k64Threads>(dst, count, 0u, tid);
            continue;
        }
        uint4 *s4 = reinterpret_cast<uint4 *>(slot);
        const uint4 *l4 = reinterpret_cast<const uint4 *>(l1);
#pragma unroll
        for (int q = 0; q < 8; q++) s4[tid + k64Threads * q] = l4[tid + k64Threads * q];
        reinterpret_cast<uint64_t *>(slot + k64Bits)[tid] = b1[tid];
        reinterpret_cast<uint16_t *>(slot + k64Pre)[tid] = pre[tid];
        if (tid == 0) {
            head->P = P;
            head->ops0 = ops0;
            head->seg = seg;
            head->ipl = ipl;
            head->pal = reinterpret_cast<uintptr_t>(pal);
            head->nib = reinterpret_cast<uintptr_t>(nib);
            head->dst = reinterpret_cast<uintptr_t>(dst);
            head->leaf = 1;
        }
    }
}

// A block of a leaf wave: 16 x 4 x 4 parents (4 words of 4 x 4 x 4), 32 x 8 x
// 8 voxels.  5 KB of LDS per wave let 28 waves run on a CU; blocks of
// twice the height issue 18 % fewer instructions, but at 12 waves per CU
// took 216 us instead of 164 us (512 bricks of the 512^3 cells volume).
constexpr uint32_t k64Words = 4, k64Blocks = 512 / k64Words;  // words of a block, blocks of a brick
// LDS of a leaf wave: the block's voxels as u16 (planes of 8 rows of 16
// dwords, plus 8), its expanded parents (word and lane), per word the rank of
// its first parent less its place in that list, voxels with a reference
constexpr uint32_t kV64Plane = 136, kV64List = 4 * 8 * kV64Plane, kV64Delta = kV64List + 256, kV64Ref = kV64Delta + 16,
                   kV64RefCap = 192, kV64Wave = kV64Ref + 2 * kV64RefCap;
constexpr uint32_t k64LeafWaves = 4;
constexpr uint32_t k64PalLds = 752;  // palette entries kept in LDS

// Dword of voxels (x, x + 1), x even, of a block row.  The exclusive or
// spreads the four y-rows of parents that a store touches over the banks, the
// planes' 8 extra dwords spread z.
__device__ __forceinline__ uint32_t v64_dw(uint32_t x, uint32_t y, uint32_t z) {
    return kV64Plane * z + 16 * y + ((x >> 1) ^ (((y >> 1) & 3u) << 2));
}
// 2-bit coordinate of a parent in its word
__device__ __forceinline__ uint32_t coord2(uint32_t p) { return (p & 1u) | ((p >> 2) & 2u); }
// 4 * half H of q
template <int H>
__device__ __forceinline__ uint32_t half_x4(uint32_t q) {
    uint32_t r;
    __asm__("v_lshlrev_b32_sdwa %0, 2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_%c2"
            : "=v"(r)
            : "v"(q), "n"(H));
    return r;
}

// What bounds the leaf kernel: vector issue (1,030 wave-instructions per
// block, 80 % of its time) and the latency of its dependent gathers.  The 512
// bricks take 144 us (3.8 TB/s of labels written).  Before, 338 us: children
// one at a time with a delta load each, references followed in the output
// loop, 12 waves per CU.
struct Leaf64 {
    const uint16_t *l1;
    const uint64_t *bits;
    const uint16_t *pre;
    const uint32_t *info, *nib;
    uint32_t ops0, seg, ipl;
};

// value of child k of level-1 node q, from the brick's operations
__device__ __forceinline__ uint32_t eval64(const Leaf64 &f, uint32_t q, uint32_t k) {
    for (;;) {
        const uint64_t b = f.bits[q >> 6];
        if (!((b >> (q & 63u)) & 1u)) return f.l1[q];
        const uint32_t r = f.pre[q >> 6] + (uint32_t)__popcll(b & ((1ull << (q & 63u)) - 1ull));
        const uint32_t wd = nib8(f.nib, f.ops0 + 8 * r), op = (wd >> (4 * k)) & 7u;
        if (op == csv::kRp) return f.l1[q];
        if (op <= csv::kRz) {
            const uint32_t x = op - 1u, am = 0x1249u << x;
            if ((k >> x) & 1u) return f.l1[morton_inc(q, am)];
            q = morton_dec(q, am);
            k |= 1u << x;
            continue;
        }
        const uint32_t in = f.info[r], y = wd & 0x77777777u, below = (1u << (4 * k)) - 1u;
        const uint32_t ip =
            f.ipl + (in & (k64PalMax - 1u)) + (uint32_t)__builtin_popcount(zero_nibbles(y ^ 0x66666666u) & below);
        if (op == csv::kP0) return ip;
        if (op == csv::kPa) return ip + 1u;
        const uint32_t d =
            nib1(f.nib, f.seg + (in >> 14) + (uint32_t)__builtin_popcount(zero_nibbles(y ^ 0x55555555u) & below));
        return ip - 1u - d;
    }
}

// kRuns: workgroups' blocks that one workgroup takes in turn: 8 for the later
// chunks of a batch with levels by request, which mostly find nothing to do and
// are then bound by the rate at which workgroups are handed out (12 us for
// those of 1,024 requests); else 1, which balances better.
template <uint32_t kRuns>
__global__ __launch_bounds__(64 * k64LeafWaves) __attribute__((amdgpu_waves_per_eu(7))) void leaf64_kernel(DecodeArgs a,
                                                                                                           Launch64 l) {
    extern __shared__ __align__(16) uint8_t smem[];
    uint32_t *spal = reinterpret_cast<uint32_t *>(smem);
    const uint32_t L = lane(), w = uniform(threadIdx.x >> 6);
    uint8_t *wl = smem + 4 * k64PalLds + w * kV64Wave;
    uint32_t *D32 = reinterpret_cast<uint32_t *>(wl);
    uint16_t *D = reinterpret_cast<uint16_t *>(wl);
    uint8_t *list = wl + kV64List;
    uint32_t *delta = reinterpret_cast<uint32_t *>(wl + kV64Delta);
    uint16_t *refs = reinterpret_cast<uint16_t *>(wl + kV64Ref);
    constexpr uint32_t kMark = 65533u, kGroups = k64Blocks / k64LeafWaves / kRuns;  // workgroups per brick
    // workgroups go to the 8 XCDs in turn: those of a brick on the XCD of its
    // upper workgroup, whose L2 holds the slot
    const uint32_t g = blockIdx.x >> 3, i = (g / kGroups) * 8 + (blockIdx.x & 7u);
    if (i >= requests64(a, l)) return;
    const uint8_t *slot = glob(l.slots) + (size_t)i * l.slot_bytes;
    const Head64 *head = reinterpret_cast<const Head64 *>(slot + k64Head);
    if (!ld_s(&head->leaf)) return;
    const uint32_t P = ld_s(&head->P);
    const uint32_t *pal = rec_at(ld_s(&head->pal));
    uint32_t *const brick = reinterpret_cast<uint32_t *>(ld_s(&head->dst));
    Leaf64 f;
    f.l1 = reinterpret_cast<const uint16_t *>(slot);
    f.bits = reinterpret_cast<const uint64_t *>(slot + k64Bits);
    f.pre = reinterpret_cast<const uint16_t *>(slot + k64Pre);
    f.info = reinterpret_cast<const uint32_t *>(slot + k64Info);
    f.nib = rec_at(ld_s(&head->nib));
    f.ops0 = ld_s(&head->ops0);
    f.seg = ld_s(&head->seg);
    f.ipl = ld_s(&head->ipl);
    const bool plds = P <= k64PalLds;
    if (plds)
        for (uint32_t e = threadIdx.x; e < P; e += 64 * k64LeafWaves) spal[e] = pal[e];
    for (uint32_t run = 0; run < kRuns; run++) {
        // the block's first parent, and its Morton index
        const uint32_t blk = ((g % kGroups) * kRuns + run) * k64LeafWaves + w;
        const uint32_t PX = 16 * (blk & 1u), PY = 4 * ((blk >> 1) & 7u), PZ = 4 * (blk >> 4);
        const uint32_t Q0 = spread5(PX) | (spread5(PY) << 1) | (spread5(PZ) << 2);
        const uint32_t lx = coord2(L), ly = coord2(L >> 1), lz = coord2(L >> 2);
        // every voxel its parent's value; the expanded parents listed
        uint32_t E = 0;
    #pragma unroll
        for (uint32_t j = 0; j < k64Words; j++) {
            const uint32_t q0 = Q0 + 64 * (j & 1u) + 512 * (j >> 1), word = q0 >> 6;
            const uint64_t b = ld_s(f.bits + word);
            const uint32_t pv = f.l1[q0 + L] * 0x00010001u;
            const uint32_t d = v64_dw(8 * j + 2 * lx, 2 * ly, 2 * lz);  // (the rows y and y + 1 share it)
            D32[d] = pv;
            D32[d + 16] = pv;
            D32[d + kV64Plane] = pv;
            D32[d + kV64Plane + 16] = pv;
            if ((b >> L) & 1u) list[E + mbcnt(b)] = (uint8_t)(64 * j + L);
            if (L == 0) delta[j] = ld_s_u16(f.pre + word) - E;
            E += (uint32_t)__popcll(b);
        }
        __syncthreads();  // the palette, for every wave
        // the children of the expanded parents; those that refer to a same-level
        // node are listed
        struct Ops {
            uint32_t idx, wd, in, pv, nb[3];
        };
        // what a lane needs of the expanded parent at place 64 c + L, loaded
        // while the chunk before is replayed
        auto load = [&](uint32_t c) -> Ops {
            Ops o;
            const uint32_t pos = min(64 * c + L, E - 1);
            o.idx = list[pos];
            const uint32_t j = o.idx >> 6, q = Q0 + (o.idx & 63u) + 64 * (j & 1u) + 512 * (j >> 1), r = pos + delta[j];
            o.wd = nib8(f.nib, f.ops0 + 8 * r);
            o.in = f.info[r];
            o.pv = f.l1[q];
    #pragma unroll
            for (int x = 0; x < 3; x++) o.nb[x] = f.l1[morton_inc(q, 0x1249u << x)];  // (on a high face: any value)
            return o;
        };
        uint32_t nref = 0;
        const uint32_t chunks = (E + 63) / 64;
        Ops next{};
        if (chunks) next = load(0);
        for (uint32_t c = 0; c < chunks; c++) {
            const Ops o = next;
            if (c + 1 < chunks) next = load(c + 1);
            uint32_t open = 0, v0 = 0;
            if (64 * c + L < E) {
                const uint32_t j = o.idx >> 6, i = o.idx & 63u;
                const uint32_t bx = 4 * j + coord2(i), by = coord2(i >> 1), bz = coord2(i >> 2);
                const uint32_t y = o.wd & 0x77777777u;
                const uint32_t pam = zero_nibbles(y ^ 0x66666666u), pdm = zero_nibbles(y ^ 0x55555555u);
                const uint32_t dl = pdm ? nib8(f.nib, f.seg + (o.in >> 14)) : 0u;
                const uint4 v = replay_children_u16(o.wd, o.pv, o.nb, f.ipl + (o.in & (k64PalMax - 1u)), pam, pdm, dl);
                const uint32_t d = v64_dw(2 * bx, 2 * by, 2 * bz);
                D32[d] = v.x;
                D32[d + 16] = v.y;
                D32[d + kV64Plane] = v.z;
                D32[d + kV64Plane + 16] = v.w;
                open = ref_children(o.wd, 7u);
                v0 = 2 * bx + 64 * by + 512 * bz;  // x + 32 y + 256 z
            }
            for (uint64_t m; (m = __ballot(open != 0)) != 0;) {
                const uint32_t k = (uint32_t)__builtin_ctz(open) >> 2, to = nref + mbcnt(m);
                if (open && to < kV64RefCap) refs[to] = (uint16_t)(v0 + (k & 1u) + 16 * (k & 2u) + 64 * (k & 4u));
                open &= open - 1u;
                nref += (uint32_t)__popcll(m);
            }
        }
        wsync();
        // a voxel's value: references followed inside the block, and out of it on
        // the other block's operations (concurrent chases see a reference or its
        // value, both of which lead to the value)
        auto at = [&](uint32_t x, uint32_t y, uint32_t z) -> uint32_t { return 2 * v64_dw(x, y, z) + (x & 1u); };
        auto chase = [&](uint32_t x, uint32_t y, uint32_t z, uint32_t v) -> uint32_t {
            while (v >= kMark) {
                const uint32_t ax = v - kMark, c = ax == 0 ? x : ax == 1 ? y : z;
                if (c == 0) {
                    const uint32_t q = spread5(PX + (x >> 1)) | (spread5(PY + (y >> 1)) << 1) | (spread5(PZ + (z >> 1)) << 2);
                    return eval64(f, morton_dec(q, 0x1249u << ax), (x & 1u) | ((y & 1u) << 1) | ((z & 1u) << 2) | (1u << ax));
                }
                x -= ax == 0 ? 1u : 0u;
                y -= ax == 1 ? 1u : 0u;
                z -= ax == 2 ? 1u : 0u;
                v = D[at(x, y, z)];
            }
            return v;
        };
        const bool listed = nref <= kV64RefCap;
        for (uint32_t e = L; listed && e < nref; e += 64) {
            const uint32_t v = refs[e], x = v & 31u, y = (v >> 5) & 7u, z = v >> 8, p = at(x, y, z);
            D[p] = (uint16_t)chase(x, y, z, D[p]);
        }
        wsync();
        // the block through the palette: 8 rows of 32 voxels per store
        const uint32_t x = 4 * (L & 7u), y = L >> 3;
        uint32_t *dst = brick + 2 * PX + 128 * PY + 8192 * PZ + x + 64 * y;
        auto rows = [&](auto al16, auto p, auto refs_left) {
    #pragma unroll 2
            for (uint32_t z = 0; z < 8; z++) {
                uint2 v = *reinterpret_cast<const uint2 *>(D32 + v64_dw(x, y, z));
                if constexpr (decltype(refs_left)::value) {  // more references than the list holds
                    v.x = chase(x, y, z, v.x & 0xFFFFu) | (chase(x + 1, y, z, v.x >> 16) << 16);
                    v.y = chase(x + 2, y, z, v.y & 0xFFFFu) | (chase(x + 3, y, z, v.y >> 16) << 16);
                }
                store4<decltype(al16)::value>(dst + 4096 * z, make_uint4(p(half_x4<0>(v.x)), p(half_x4<1>(v.x)),
                                                                         p(half_x4<0>(v.y)), p(half_x4<1>(v.y))));
            }
        };
        const bool al = (reinterpret_cast<uintptr_t>(dst) & 15) == 0;
        const uint8_t *sp = smem, *gp = reinterpret_cast<const uint8_t *>(pal);
        auto in_lds = [&](uint32_t o) -> uint32_t { return *reinterpret_cast<const uint32_t *>(sp + o); };
        auto in_mem = [&](uint32_t o) -> uint32_t { return *reinterpret_cast<const uint32_t *>(gp + o); };
        if (plds && al && listed) rows(std::true_type{}, in_lds, std::false_type{});
        else if (al && listed) rows(std::true_type{}, in_mem, std::false_type{});
        else if (al) rows(std::true_type{}, in_mem, std::true_type{});
        else rows(std::false_type{}, in_mem, std::true_type{});
    }
}
