// The host half of packing a state, run on the CPU with a stand-in for the
// GPU runtime: this program defines the few HIP calls that fate_host.cpp makes
// and the launch of the completed-parent kernel, so that the library's own
// references resolve here.  "Device" memory is host memory registered with a
// GPU number, and work enqueued on the stream runs when the stream is waited
// for, from whatever the sources hold then.
//
//   pack_runtime devices      which GPUs the packing may launch its kernel on,
//                             and the image it leaves, against the host layout
//   pack_runtime shapes       up to how many models the row kernels take a cluster
//   pack_runtime memory       an allocation that fails, on the caller's thread or
//                             on one that validates a part of the batch
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <functional>
#include <new>
#include <random>
#include <vector>

#include "fate.h"
#include "fate_internal.h"

namespace {

// ---- the stand-in runtime ----------------------------------------------------

struct Range {
    const uint8_t *lo, *hi;
    int device;
};
std::vector<Range> ranges;
std::vector<std::function<void()>> queue;
int stream_device = 0, current_device = 0;
int launches = 0, launched_on = -1;
bool bad_access = false;

const Range *range_of(const void *p) {
    for (const Range &r : ranges)
        if (p >= r.lo && p < r.hi) return &r;
    return nullptr;
}

#define CHECK(x)                                                     \
    do {                                                             \
        if (!(x)) {                                                  \
            printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #x);    \
            fflush(stdout);                                          \
            exit(1);                                                 \
        }                                                            \
    } while (0)

}  // namespace

extern "C" {
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    const Range *r = range_of(p);
    if (!r) return hipErrorInvalidValue;
    memset(a, 0, sizeof(*a));
    a->type = hipMemoryTypeDevice;
    a->device = r->device;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    queue.push_back([=] { memcpy(d, s, n); });
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
    queue.push_back([=] { memset(d, v, n); });
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    for (auto &f : queue) f();
    queue.clear();
    return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) {
    *d = stream_device;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = current_device;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

namespace fate {
// The kernel's rule on the host; it may only touch memory of the GPU it runs on.
int launch_lists(const ListsLaunch &a, void *) {
    ++launches;
    launched_on = stream_device;
    for (const void *p : {(const void *)a.rec, (const void *)a.par_idx, (const void *)a.stage_off, (const void *)a.holders,
                          (const void *)a.tnow, (const void *)a.done_n, (const void *)a.done}) {
        const Range *r = range_of(p);
        if (!r || r->device != stream_device || stream_device != current_device) bad_access = true;
    }
    queue.push_back([a] {
        for (int b = 0; b < a.B; ++b)
            for (int64_t s = a.stage_off[b]; s < a.stage_off[b + 1]; ++s) {
                const StageRec &r = a.rec[s];
                uint32_t n = 0;
                for (uint32_t q = 0; a.done_n[s] && q < r.npar; ++q) {
                    const uint32_t u = a.par_idx[r.par_begin + q];
                    if (a.holders[u]) a.done[r.par_begin + n++] = DoneParent{a.holders[u], a.rec[u].sigma, 0u};
                }
                for (uint32_t q = n; q < r.npar; ++q) a.done[r.par_begin + q] = DoneParent{0ull, 0.0f, 0u};
                a.done_n[s] = n;
                if (a.finish) a.finish[s] = a.holders[s] ? a.tnow[b] : 0.0f;
            }
    });
    return 0;
}
}  // namespace fate

namespace {

// ---- allocations that fail -----------------------------------------------------

std::atomic<long> fail_at{-1}, allocated{0};  // fail the allocation of this number (counted from 0)

}  // namespace

void *operator new(size_t n) {
    if (fail_at.load() >= 0 && allocated.fetch_add(1) == fail_at.load()) throw std::bad_alloc();
    if (void *p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

namespace {

// ---- a batch -----------------------------------------------------------------

struct Batch {
    static constexpr int D = 4, M = 3, K = 2;
    std::vector<float> exec, sw, beta, tokens, sigma, tau, tnow;
    std::vector<int64_t> weight, cap, stage_off, par_off;
    std::vector<int32_t> par, model, shard;
    std::vector<uint64_t> elig, hash, resident, cache, holders;
    std::vector<uint8_t> status;
    fate_cluster_t c;
    fate_dag_batch_t g;
    fate_state_t st;

    Batch(const std::vector<int> &sizes, unsigned seed) {
        std::mt19937 rng(seed);
        exec.assign(M * D, 1.0f);
        sw.assign(M * D, 0.5f);
        weight.assign(M, 10);
        cap.assign(D, 25);
        beta.assign(D * D, 1e-9f);
        stage_off.push_back(0);
        par_off.push_back(0);
        for (int n : sizes) {
            const int64_t base = stage_off.back();
            for (int v = 0; v < n; ++v) {
                std::vector<int> ps;
                for (int u = std::max(0, v - 12); u < v; ++u)
                    if (rng() % 4 == 0) ps.push_back(u);
                bool done = true;
                for (int u : ps) {
                    par.push_back(u);
                    done &= status[base + u] == FATE_COMPLETED;
                }
                par_off.push_back((int64_t)par.size());
                const bool completed = done && rng() % 3 != 0;
                status.push_back(completed ? FATE_COMPLETED : done && rng() % 4 == 0 ? FATE_RUNNING : FATE_PENDING);
                holders.push_back(completed ? 1 + rng() % 15 : 0);
                model.push_back((int32_t)(rng() % M));
                shard.push_back(1 + (int32_t)(rng() % 3));
                elig.push_back(15);
                hash.push_back(rng() % 5);
                tokens.push_back((float)(rng() % 100));
                sigma.push_back((float)(1 + rng() % 1000));
            }
            stage_off.push_back(base + n);
            tnow.push_back((float)(rng() % 10) * 0.5f);
            for (int d = 0; d < D; ++d) {
                resident.push_back(rng() % 8);
                tau.push_back((float)(rng() % 10) * 0.25f);
                for (int k = 0; k < K; ++k) cache.push_back(rng() % 5);
            }
        }
        c = fate_cluster_t{D, M, exec.data(), sw.data(), weight.data(), cap.data(), beta.data()};
        g = fate_dag_batch_t{(int32_t)sizes.size(), stage_off.data(), par_off.data(), par.data(), model.data(), elig.data(),
                             shard.data(), hash.data(), tokens.data(), sigma.data()};
        st = fate_state_t{K, resident.data(), cache.data(), holders.data(), status.data(), tau.data(), tnow.data()};
    }
};

struct Buffer {  // memory of a GPU (or, with device < 0, of the host), filled with a pattern
    std::vector<uint64_t> mem;
    size_t bytes;
    Buffer(size_t n, int device) : mem(n / 8 + 2, 0xa5a5a5a5a5a5a5a5ull), bytes(n) {
        const uint8_t *p = reinterpret_cast<const uint8_t *>(mem.data());
        if (device >= 0) ranges.push_back({p, p + mem.size() * 8, device});
    }
    ~Buffer() {
        const void *p = mem.data();
        ranges.erase(std::remove_if(ranges.begin(), ranges.end(), [&](const Range &r) { return r.lo == p; }), ranges.end());
    }
    void *data() { return mem.data(); }
};

// Packing launches the kernel where the DAGs, the buffer, the stream and the
// current device are one GPU and the image is not small, and gathers the lists
// on the host otherwise; the image is the same.
void devices() {
    std::vector<int> sizes{0, 1, 30000, 0, 7, 9000, 1};
    const std::vector<int> small{5, 0, 40};
    for (const std::vector<int> &ns : {sizes, small}) {
        const bool large = ns.size() > 3;
        Batch b(ns, 7);
        size_t db = 0, sb = 0, ab = 0;
        CHECK(fate_pack_dags_size(&b.c, &b.g, 1, &db) == FATE_OK);
        for (int dag = -1; dag < 2; ++dag) {
            Buffer dags(db, dag);
            fate_dags_t pk;
            CHECK(fate_layout_dags(&b.c, &b.g, 1, dags.data(), db, &pk) == FATE_OK);
            int64_t nf = 0, nc = 0;
            CHECK(fate_pack_state_size(&pk, &b.g, &b.st, 4, &sb, &nf, &nc) == FATE_OK);
            CHECK(fate_pack_state_advance_size(&pk, &b.g, &b.st, 4, &ab) == FATE_OK);
            Buffer want(sb, -1);
            fate_state_h h, hw;
            CHECK(fate_layout_state(&pk, &b.g, &b.st, 4, want.data(), sb, &hw) == FATE_OK);
            std::vector<uint64_t> first;
            for (int buf = 0; buf < 2; ++buf)
                for (stream_device = 0; stream_device < 2; ++stream_device)
                    for (current_device = 0; current_device < 2; ++current_device) {
                        const bool kernel = large && dag == buf && buf == stream_device && stream_device == current_device;
                        Buffer out(sb, buf), adv(ab, buf);
                        launches = 0;
                        CHECK(fate_pack_state(&pk, &b.g, &b.st, 4, out.data(), sb, nullptr, &h) == FATE_OK);
                        CHECK(queue.empty());
                        CHECK(!bad_access);
                        CHECK(launches == (kernel ? 1 : 0));
                        CHECK(memcmp(out.data(), want.data(), sb) == 0);
                        CHECK(h.n_frontier == nf && h.n_cand == nc && h.n_slices == hw.n_slices);
                        launches = 0;
                        CHECK(fate_pack_state_advance(&pk, &b.g, &b.st, 4, adv.data(), ab, nullptr, &h) == FATE_OK);
                        CHECK(queue.empty() && !bad_access && launches == (kernel ? 1 : 0));
                        const uint64_t *a = static_cast<const uint64_t *>(adv.data());
                        if (first.empty()) first.assign(a, a + ab / 8);
                        CHECK(memcmp(a, first.data(), first.size() * 8) == 0);
                    }
        }
    }
    printf("devices ok\n");
}

// A failed allocation leaves each call by std::bad_alloc, on the caller's
// thread and with every other thread ended, whichever thread it failed on (or
// the call does without: a range whose thread cannot be started runs on the
// caller's); the outputs are as they were, and the next call succeeds.
void memory() {
    Batch b(std::vector<int>{40000, 1, 30000, 0, 33000, 20000, 25000}, 11);
    size_t db = 0, sb = 0;
    CHECK(fate_pack_dags_size(&b.c, &b.g, 0, &db) == FATE_OK);
    Buffer dags(db, -1);
    fate_dags_t pk;
    CHECK(fate_layout_dags(&b.c, &b.g, 0, dags.data(), db, &pk) == FATE_OK);
    int64_t nf = 0, nc = 0;
    CHECK(fate_pack_state_size(&pk, &b.g, &b.st, 4, &sb, &nf, &nc) == FATE_OK);
    Buffer want(sb, -1), out(sb, -1);
    fate_state_h h;
    CHECK(fate_layout_state(&pk, &b.g, &b.st, 4, want.data(), sb, &h) == FATE_OK);
    const std::vector<uint64_t> before(out.mem);
    for (int call = 0; call < 2; ++call) {
        long thrown = 0;
        for (long n = 0;; ++n) {
            size_t bytes = 1;
            int64_t f = 2, c = 3;
            fate_state_h x;
            memset(&x, 0x5a, sizeof(x));
            const fate_state_h x0 = x;
            bool failed = false;
            fate_status_t st = FATE_OK;
            allocated = 0;
            fail_at = n;
            try {
                st = call ? fate_layout_state(&pk, &b.g, &b.st, 4, out.data(), sb, &x)
                          : fate_pack_state_size(&pk, &b.g, &b.st, 4, &bytes, &f, &c);
            } catch (const std::bad_alloc &) {
                failed = true;
            }
            fail_at = -1;
            const bool reached = allocated.load() > n;
            if (failed) {
                ++thrown;
                CHECK(bytes == 1 && f == 2 && c == 3 && memcmp(&x, &x0, sizeof(x)) == 0 && out.mem == before);
            } else {
                CHECK(st == FATE_OK);
                if (call) {
                    CHECK(memcmp(out.data(), want.data(), sb) == 0);
                    out.mem = before;
                } else {
                    CHECK(bytes == sb && f == nf && c == nc);
                }
            }
            if (!reached) break;  // every allocation of the call has failed once
        }
        CHECK(thrown > 0);
    }
    printf("memory ok\n");
}

// The models up to which a row kernel's tables fit, by devices and prefix slots
// (a shape past them takes the general kernel, several times slower).
void shapes() {
    const int most[][3] = {{1, 32, 32}, {16, 0, 32}, {16, 32, 32}, {17, 16, 64}, {32, 16, 64}, {32, 32, 53},
                           {33, 31, 53}, {33, 32, 26}, {48, 32, 26}, {64, 16, 53}, {64, 17, 26}, {64, 32, 26}};
    for (const auto &x : most) {
        int m = 0;
        while (m < FATE_MAX_MODELS && fate::rows_kernel_fits(x[0], x[1], m + 1)) ++m;
        if (m != x[2]) printf("%d devices, %d slots: %d models\n", x[0], x[1], m);
        CHECK(m == x[2]);
    }
    printf("shapes ok\n");
}

}  // namespace

int main(int argc, char **argv) {
    if (argc > 1 && !strcmp(argv[1], "devices")) devices();
    else if (argc > 1 && !strcmp(argv[1], "memory")) memory();
    else if (argc > 1 && !strcmp(argv[1], "shapes")) shapes();
    else return 2;
    return 0;
}
