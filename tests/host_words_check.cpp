// Check of the page-locked result words (csrc/host_words.h) on the CPU, with a
// stand-in for the HIP runtime's calls: slots are disjoint and bounded, also
// with many threads; a page that a device reset has freed, or whose address
// another allocation has taken, is replaced and never handed out again; slots
// of a lost page do not come back into the new one; no slot is given on
// another device, on a capturing stream or without memory, and the
// runtime's last error is left clean.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <thread>
#include <vector>

#include "host_words.h"

static int g_device = 0;
static hipStreamCaptureStatus g_capture = hipStreamCaptureStatusNone;
static bool g_no_memory = false;
static hipError_t g_last = hipSuccess;
static uint64_t g_next_id = 1, g_id = 0;
static void *g_live = nullptr;   // the one live allocation
static void *g_force = nullptr;  // address the next allocation gets
static hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal;
static int g_allocs = 0;

extern "C" {
hipError_t hipGetDevice(int *d) { return *d = g_device, hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    return *s = g_capture, hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m)
{
    return std::swap(*m, g_mode), hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    if (g_mode != hipStreamCaptureModeRelaxed) abort();
    if (g_no_memory) return g_last = hipErrorOutOfMemory;
    ++g_allocs;
    g_live = *p = g_force ? g_force : malloc(n);
    g_force = nullptr;
    g_id = g_next_id++;
    return hipSuccess;
}
hipError_t hipHostFree(void *) { return hipSuccess; }
hipError_t hipPointerGetAttribute(void *out, hipPointer_attribute a, hipDeviceptr_t p)
{
    if (a != HIP_POINTER_ATTRIBUTE_BUFFER_ID || p != g_live) return g_last = hipErrorInvalidValue;
    return *(uint64_t *)out = g_id, hipSuccess;
}
hipError_t hipGetLastError() { const hipError_t e = g_last; return g_last = hipSuccess, e; }
}

using lbm_host::HostWords;
#define CHECK(c) \
    do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

int main()
{
    {   // no memory: no slot; then one
        g_no_memory = true;
        HostWords a(0, nullptr);
        CHECK(!a.w && g_last == hipSuccess && g_mode == hipStreamCaptureModeGlobal);
        g_no_memory = false;
        HostWords b(0, nullptr);
        CHECK(b.w && g_allocs == 1 && g_mode == hipStreamCaptureModeGlobal);
        b.give_back();
        CHECK(!b.w);
    }
    {   // another device, a capturing stream
        HostWords a(1, nullptr);
        g_capture = hipStreamCaptureStatusActive;
        HostWords b(0, nullptr);
        g_capture = hipStreamCaptureStatusNone;
        CHECK(!a.w && !b.w);
    }
    {   // all slots, disjoint; the next call gets none; a slot given back is used again
        std::vector<HostWords *> v;
        std::set<unsigned long long *> at;
        for (int k = 0; k < lbm_host::kHostSlots; ++k) {
            v.push_back(new HostWords(0, nullptr));
            CHECK(v.back()->w && at.insert(v.back()->w).second);
        }
        for (auto *p : at) CHECK((*at.begin() <= p) && (p - *at.begin()) % lbm_host::kHostWords == 0);
        HostWords full(0, nullptr);
        CHECK(!full.w);
        unsigned long long *third = v[3]->w;
        v[3]->give_back();
        HostWords again(0, nullptr);
        CHECK(again.w == third);
        again.give_back();
        // a device reset frees the page: a new one, with every slot, and the
        // old one's slots do not free any of the new one's
        g_live = nullptr;
        std::vector<HostWords *> n;
        for (int k = 0; k < lbm_host::kHostSlots; ++k) n.push_back(new HostWords(0, nullptr));
        CHECK(g_allocs == 2 && g_last == hipSuccess);
        for (auto *x : n) CHECK(x->w && !at.count(x->w));
        for (auto *x : v) x->give_back();
        HostWords none(0, nullptr);
        CHECK(!none.w);
        for (auto *x : n) x->give_back();
        // the page is freed and its address belongs to another allocation
        g_id = g_next_id++;
        HostWords other(0, nullptr);
        CHECK(other.w && g_allocs == 3);
        // a slot whose wait failed (never given back) stays taken
        HostWords b(0, nullptr);
        CHECK(b.w && b.w != other.w);
        b.give_back();
        for (auto *x : v) delete x;
        for (auto *x : n) delete x;
    }
    {   // threads: nobody else writes a slot while it is held
        std::vector<std::thread> ts;
        std::vector<int> bad(24, 0);
        for (int t = 0; t < 24; ++t)
            ts.emplace_back([&, t] {
                for (int k = 0; k < 2000; ++k) {
                    HostWords a(0, nullptr);
                    if (!a.w) continue;
                    *(volatile unsigned long long *)a.w = (unsigned long long)t * 10000 + k;
                    std::this_thread::yield();
                    if (*(volatile unsigned long long *)a.w != (unsigned long long)t * 10000 + k) ++bad[t];
                    a.give_back();
                }
            });
        for (auto &t : ts) t.join();
        for (int b : bad) CHECK(b == 0);
    }
    printf("ok\n");
    return 0;
}
