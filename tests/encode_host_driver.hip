// The GPU compressor's host code on the CPU: csv_encode_gpu.hip compiled for
// the host only and linked with the stand-in below for the HIP runtime, which
// has a limit on device memory, fails calls on demand and runs a kernel's
// stand-in when its stream is waited for.  Usage: encode_host_driver SCENARIO
#include "../paper_2308_16619_amd/csrc/csv_encode_gpu.hip"

#include <cstdio>
#include <functional>
#include <map>
#include <string>
#include <vector>

namespace fake {

size_t limit = ~(size_t)0, used = 0;      // device memory
std::map<uint8_t *, size_t> blocks;       // its allocations
std::map<const void *, std::string> name; // kernels
std::vector<std::function<void()>> queue; // launched, not yet run
hipError_t last = hipSuccess;
int calls = 0, fail_at = -1;              // calls that can fail; the one that does
uint64_t ops = 9000, extra = 0;           // bytes of arenas 1 and 3 per brick
uint32_t rec = 64;                        // ... of a record, at least
uint64_t samples = 0;                     // bricks that the frequency tables count
dim3 grid, block;
std::mutex mu;

void check(bool ok, const char *what) {
    if (ok) return;
    std::printf("FAILED: %s\n", what);
    std::exit(1);
}
hipError_t done(hipError_t e) {
    if (e != hipSuccess) last = e;
    return e;
}
bool fails() {
    std::lock_guard<std::mutex> lk(mu);
    return calls++ == fail_at;
}
// bytes from p to the end of its allocation
size_t room(const void *p) {
    auto it = blocks.upper_bound((uint8_t *)p);
    check(it != blocks.begin(), "a device pointer of no allocation");
    --it;
    check((uint8_t *)p < it->first + it->second, "a device pointer past its allocation");
    return it->first + it->second - (uint8_t *)p;
}
void run() {
    std::vector<std::function<void()>> q;
    q.swap(queue);
    for (auto &f : q) f();
}

uint32_t record_bytes(uint32_t id) { return rec + 4 * (id % 7); }
bool held(const EncArgs &a) { return a.ctl->top1 <= a.cap1 && a.ctl->top3 <= a.cap3; }

template <class T>
T arg(void **args, int k) { return *static_cast<T *>(args[k]); }

void copy_out(const EncArgs &a, EncCtl *h, const uint8_t *blob, uint64_t rs, uint8_t *pin, uint64_t cap) {
    *h = *a.ctl;
    if (held(a) && rs + a.ctl->total < cap) std::memcpy(pin, blob, rs + a.ctl->total);
}
void scan(const EncArgs &a, uint64_t *index) {
    if (!held(a)) return;
    uint64_t at = 0;
    for (uint32_t i = 0; i < a.n_items; i++) {
        index[i] = at;
        at += a.sizes[i];
    }
    index[a.n_items] = a.ctl->total = at;
}
void pack(const EncArgs &a, const uint64_t *index, uint8_t *to, uint64_t cap) {
    check(cap <= room(to), "packing past the container's buffer");
    for (uint32_t i = 0; held(a) && i < a.n_items && index[i] + a.sizes[i] <= cap; i++)
        std::memset(to + index[i], (int)(a.aoff[i] & 255), a.sizes[i]);
}
// what a launch does, by the kernel's name
std::function<void()> effect(const std::string &k, void **args, uint32_t groups) {
    auto is = [&](const char *s) { return k.find(s) != std::string::npos; };
    if (is("begin_kernel")) {
        EncCtl *c = arg<EncCtl *>(args, 0);
        const size_t keep = arg<bool>(args, 1) ? sizeof(c->hist) : 0;
        return [c, keep] { std::memset((char *)c + keep, 0, sizeof(*c) - keep); };
    }
    if (is("piece_kernel")) {
        auto src = arg<const uint8_t *>(args, 0);
        auto dst = arg<uint8_t *>(args, 1);
        const auto n = arg<uint64_t>(args, 2);
        return [=] {
            check(n <= room(src), "a piece past the container's buffer");
            std::memcpy(dst, src, n);
        };
    }
    const EncArgs a = arg<EncArgs>(args, 0);
    if (is("reuse_kernel"))
        return [a, groups] {
            check(kScratch * groups <= room(a.scratch), "reuse kernel's scratch");
            check(a.cap1 <= room(a.arena1) && part2(a.cap1) <= room(a.arena2), "arenas 1 and 2");
            check(sizeof(BrickMeta) * (size_t)a.n_items <= room(a.meta), "bricks' states");
            a.ctl->top1 += ops * a.n_items;
        };
    if (is("palette_kernel"))
        return [a] {
            for (uint32_t i = 0; i < a.n_items; i++)
                if (a.sample_stride && (a.first + i * a.step) % a.sample_stride == 0) a.ctl->hist[0][0]++;
        };
    if (is("rans_kernel"))
        return [a, groups] {
            check(kWordsScratch * kWaves * groups <= room(a.wscratch), "rANS kernel's scratch");
            check(a.cap3 <= room(a.arena3), "arena 3");
            check(fail_at >= 0 || a.ctl->hist[0][0] == samples, "the sampled bricks, each once");
            check(4ull * a.n_items <= room(a.sizes) && 8ull * a.n_items <= room(a.aoff), "records' places");
            if (a.ctl->top1 > a.cap1) return;  // (some bricks have no operations)
            a.ctl->top3 += extra * a.n_items;
            for (uint32_t i = 0; i < a.n_items; i++) {
                a.sizes[i] = record_bytes(a.first + i * a.step);
                a.aoff[i] = a.first + i * a.step;
            }
        };
    if (is("scan_kernel")) {
        auto index = arg<uint64_t *>(args, 1);
        return [a, index] { scan(a, index); };
    }
    if (is("pack_kernel")) {
        auto index = arg<const uint64_t *>(args, 1);
        auto to = arg<uint8_t *>(args, 2);
        const auto cap = arg<uint64_t>(args, 3);
        return [=] { pack(a, index, to, cap); };
    }
    if (is("leave_kernel")) {
        auto h = arg<EncCtl *>(args, 1);
        auto blob = arg<const uint8_t *>(args, 2);
        const auto rs = arg<uint64_t>(args, 3), cap = arg<uint64_t>(args, 5);
        auto pin = arg<uint8_t *>(args, 4);
        return [=] { copy_out(a, h, blob, rs, pin, cap); };
    }
    check(is("finish_kernel"), "a kernel without a stand-in");
    auto h = arg<EncCtl *>(args, 1);
    auto blob = arg<uint8_t *>(args, 2);
    const auto cap = arg<uint64_t>(args, 3), rs = arg<uint64_t>(args, 4), hcap = arg<uint64_t>(args, 6);
    auto pin = arg<uint8_t *>(args, 5);
    return [=] {
        auto index = reinterpret_cast<uint64_t *>(blob + csv::kHeaderBytes);
        scan(a, index);
        if (held(a)) pack(a, index, blob + rs, cap - rs);
        copy_out(a, h, blob, rs, pin, hcap);
    };
}

}  // namespace fake

using namespace fake;

extern "C" {
void **__hipRegisterFatBinary(const void *) {
    static void *p;
    return &p;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *,
                           void *, int *) {
    name[host] = device;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) {
    grid = g;
    block = b;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
    *g = grid;
    *b = block;
    *lds = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3, void **args, size_t, hipStream_t) {
    if (fails()) return done(hipErrorLaunchFailure);
    queue.push_back(effect(name[f], args, g.x));
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes) {
    if (fails() || bytes > limit - used) return done(hipErrorOutOfMemory);
    *p = std::malloc(bytes);
    check(*p != nullptr, "memory of the test's own");
    blocks[(uint8_t *)*p] = bytes;
    used += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    run();  // (as the runtime does, it waits for the device)
    check(blocks.count((uint8_t *)p), "free of no allocation");
    used -= blocks[(uint8_t *)p];
    blocks.erase((uint8_t *)p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
    if (fails()) return done(hipErrorOutOfMemory);
    *p = std::malloc(bytes);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    if (p) run();
    std::free(p);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    run();
    return fails() ? done(hipErrorUnknown) : hipSuccess;
}
hipError_t hipDeviceSynchronize() {
    run();
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    if (fails()) return done(hipErrorOutOfMemory);
    *e = (hipEvent_t)e;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return fails() ? done(hipErrorUnknown) : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) {
    if (fails()) return hipErrorUnknown;  // (the pieces behind it have not arrived)
    std::lock_guard<std::mutex> lk(mu);
    run();
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
void csv_encode_opts_default(csv_encode_opts *o) {
    std::memset(o, 0, sizeof(*o));
    o->brick_log2 = 5;
    o->scale_bits = 10;
    o->lane_k = 64;
    o->lane_max = 64;
}
}

// one call on an edge^3 volume; what it leaves is checked, and so is the container
static int call(uint32_t edge) {
    static const uint32_t label = 0;  // (never read: the kernels do not run)
    uint8_t *blob = nullptr;
    size_t n = 0;
    const uint32_t e = (edge + 31) / 32, B = e * e * e;
    samples = (B + 511) / 512;
    const int rc = csv_encode_volume_gpu(&label, edge, edge, edge, nullptr, 0, nullptr, &blob, &n);
    check(queue.empty(), "the call returned with kernels in flight");
    check((rc == CSV_OK) == (blob != nullptr), "a container if and only if the call succeeds");
    if (rc == CSV_OK) {
        const uint64_t rs = csv::record_area_offset(B);
        auto index = reinterpret_cast<const uint64_t *>(blob + csv::kHeaderBytes);
        uint64_t at = 0;
        bool ok = true;
        for (uint32_t i = 0; ok && i < B; i++) {
            ok = index[i] == at && rs + at + record_bytes(i) <= n && blob[rs + at] == (i & 255) &&
                 blob[rs + at + record_bytes(i) - 1] == (i & 255);
            at += record_bytes(i);
        }
        check(ok && index[B] == at && n == rs + at, "the container");
    }
    std::free(blob);
    return rc;
}

static constexpr size_t MiB = 1u << 20;

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "plain") {
        for (uint32_t e : {1u, 100u, 512u, 600u}) check(call(e) == CSV_OK, "a call");
        extra = 200;  // records larger than arena 3 at first
        check(call(600) == CSV_OK, "a call with a larger arena 3");
    } else if (what == "smaller arenas") {
        // arena 1 for a twelfth of the labels fits, arena 2 beside it does not
        ops = 1000;
        limit = 3000 * MiB;
        check(call(1536) == CSV_OK, "a call on 64ths of the labels");
        check(call(64) == CSV_OK, "a small call after it");
    } else if (what == "small after too large") {
        ops = 100000;
        limit = 1500 * MiB;
        (void)call(1536);
        ops = 9000;
        check(call(64) == CSV_OK, "a small call after one that did not fit");
        check(call(512) == CSV_OK, "a middle-sized call");
    } else if (what == "every failure") {
        // call k of the runtime fails, for every k: nothing stays in flight,
        // and the next call succeeds
        for (uint32_t e : {64u, 260u, 700u}) {
            limit = e == 260 ? 150 * MiB : ~(size_t)0;  // (in batches)
            if (e == 700) extra = 400, rec = 5000;  // larger than the container's buffer at first
            fail_at = -1;
            calls = 0;
            check(csv_encode_gpu_release(0) == CSV_OK && call(e) == CSV_OK, "a call");
            const int n = calls;
            for (int k = 0; k < n; k++) {
                check(csv_encode_gpu_release(0) == CSV_OK, "release");
                calls = 0;
                fail_at = k;
                (void)call(e);
                fail_at = -1;
                check(call(e) == CSV_OK, "a call after a failed one");
            }
        }
    } else if (what == "batches") {
        // noise: the most that bricks can ask for
        ops = kMostOps;
        extra = rec = 160000;
        for (size_t m : {3000, 800, 300, 100, 40}) {
            check(csv_encode_gpu_release(0) == CSV_OK, "release");
            limit = m * MiB;
            check(call(256) == CSV_OK, "noise in little memory");
        }
        check(call(64) == CSV_OK && call(256) == CSV_OK, "calls after it");
        limit = 2 * MiB;  // a brick at a time
        check(csv_encode_gpu_release(0) == CSV_OK && call(128) == CSV_OK, "noise, brick by brick");
        limit = MiB / 2;
        check(csv_encode_gpu_release(0) == CSV_OK && call(64) == CSV_ENOMEM, "no room for a brick");
        limit = ~(size_t)0;
        check(call(256) == CSV_OK, "a call with enough memory");
        // more than three batches of sampled bricks, the last one ragged
        ops = 3000;
        extra = 0;
        rec = 64;
        limit = 4 * MiB;
        check(csv_encode_gpu_release(0) == CSV_OK && call(700) == CSV_OK, "many sampled bricks");
    } else {
        check(false, "no such scenario");
    }
    check(csv_encode_gpu_release(0) == CSV_OK && used == 0, "everything released");
    std::printf("ok\n");
    return 0;
}
