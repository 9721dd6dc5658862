// A host-only stand-in for the HIP runtime calls that libttcross.so makes, to
// be loaded before the real runtime: device memory is host memory, every
// launch runs at once on the calling thread.  Kernels do nothing, but
//   k_commit      ends the run at rank fake_ranks, as far as the capacities go
//                 (it writes the host mirror),
//   k_cores(_t)   fills the cores with 1, 2, 3, ... and leaves a clean state,
//   k_copy_one    copies and raises its flag,
//   k_commit_b    lets every problem of the launch grow by one rank a sweep, to
//                 fake_sweeps sweeps, and k_state_out_b leaves clean states.
// So a test can follow which memory, stream and device a call uses, make a
// runtime call fail, and stop one thread inside a call while another goes on.
// Faults (a dead stream or freed memory used, memory of another device
// touched by a kernel) are counted and kept as text.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "tt_device.h"

namespace {
struct Block { size_t size; int dev; bool host, freed; };
struct Stream { int dev; bool dead; };
std::recursive_mutex mu;
std::map<char *, Block> blocks;
std::set<Stream *> streams;
std::map<const void *, std::string> names;
std::vector<std::string> log_, faults;
std::map<std::string, int> fail_at;              // calls left until the call of that name fails
size_t in_use = 0, limit = ~(size_t)0;
thread_local int cur = 0;
thread_local hipError_t last = hipSuccess;
void (*hook)(const char *, const void *) = nullptr;
// a batched launch's problems (as in tt_kernels.h)
struct Batch { int na; int boff[513]; uint16_t p[512]; };
int batch_sweeps = 1, run_rank = 1;
struct Config { dim3 g, b; size_t lds; hipStream_t s; };
thread_local std::vector<Config> configs;

void note(const std::string &s) { std::lock_guard<std::recursive_mutex> l(mu); log_.push_back(s); }
void fault(const std::string &s) { std::lock_guard<std::recursive_mutex> l(mu); faults.push_back(s); }

// Called first by every entry point that a test can stop or make fail.
bool fails(const char *name, const void *arg = nullptr)
{
    if (hook) hook(name, arg);
    std::lock_guard<std::recursive_mutex> l(mu);
    auto it = fail_at.find(name);
    return it != fail_at.end() && it->second > 0 && --it->second == 0;
}

const Block *find(const void *p)
{
    auto it = blocks.upper_bound((char *)p);
    if (it == blocks.begin()) return nullptr;
    --it;
    return (char *)p < it->first + it->second.size ? &it->second : nullptr;
}

int stream_dev(hipStream_t s, const char *who)
{
    if (!s) return cur;
    std::lock_guard<std::recursive_mutex> l(mu);
    Stream *x = (Stream *)s;
    if (!streams.count(x)) return cur;           // a caller's stream
    if (x->dead) fault(std::string(who) + " on a destroyed stream");
    return x->dev;
}

// A kernel on device dev touches n bytes at p.
bool touch(const void *p, size_t n, int dev, const char *what)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    const Block *b = find(p);
    if (!b) return fault(std::string(what) + ": memory the device does not know"), false;
    if (b->freed) return fault(std::string(what) + ": freed memory"), false;
    if (!b->host && b->dev != dev) return fault(std::string(what) + ": another device's memory"), false;
    if (!find((const char *)p + n - 1)) return fault(std::string(what) + ": past the end"), false;
    return true;
}

hipError_t alloc(void **p, size_t n, bool host)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    *p = nullptr;
    if (!host && (n > ((size_t)1 << 40) || in_use + n > limit)) return hipErrorOutOfMemory;
    char *q = (char *)calloc(1, n + 64);
    if (!q) return hipErrorOutOfMemory;
    blocks[q] = Block{n, cur, host, false};
    if (!host) in_use += n;
    *p = q;
    return hipSuccess;
}

hipError_t release(void *p, const char *who)
{
    if (!p) return hipSuccess;
    std::lock_guard<std::recursive_mutex> l(mu);
    auto it = blocks.find((char *)p);
    if (it == blocks.end() || it->second.freed) return fault(std::string(who) + ": not allocated"), hipErrorInvalidValue;
    it->second.freed = true;                     // the memory itself stays, so that late uses are seen
    if (!it->second.host) in_use -= it->second.size;
    return hipSuccess;
}

hipError_t launch(const void *fn, dim3 grid, void **args, hipStream_t s)
{
    std::string name = names.count(fn) ? names[fn] : "?";
    if (fails("hipLaunchKernel", name.c_str())) return last = hipErrorLaunchFailure;
    const int dev = stream_dev(s, "launch");
    char line[256];
    snprintf(line, sizeof line, "launch %.60s dev %d stream %p grid %u", name.c_str(), dev, (void *)s, grid.x);
    note(line);
    using namespace ttc;
    if (name.find("k_commit") != std::string::npos && name.find("k_commit_b") == std::string::npos) {
        const ProbDev *P = *(const ProbDev **)args[0];
        HostMirror *hm = P->hm;
        hm->r[0] = hm->r[P->d] = 1;
        for (int k = 1; k < P->d; ++k) hm->r[k] = run_rank < P->kd[k - 1].rk_cap ? run_rank : P->kd[k - 1].rk_cap;
        hm->stop = 1;
        hm->sweeps_done = ((const SweepArgs *)args[1])->sweep + 1;
    } else if (name.find("k_commit_b") != std::string::npos) {
        const ProbDev *Pa = *(const ProbDev **)args[0];
        const Batch &bm = *(const Batch *)args[1];
        for (int b = 0; b < bm.na; ++b) {
            const ProbDev &P = Pa[bm.p[b]];
            HostMirror *hm = P.hm;
            if (hm->stop) continue;
            ++hm->sweeps_done;
            hm->r[0] = hm->r[P.d] = 1;
            hm->stop = hm->sweeps_done >= batch_sweeps;
            for (int k = 1; k < P.d; ++k) hm->r[k] = hm->sweeps_done + (hm->stop ? 0 : 1);
        }
    } else if (name.find("k_state_out_b") != std::string::npos) {
        ProbState *hS = *(ProbState **)args[1];
        const Batch &bo = *(const Batch *)args[2];
        for (int b = 0; b < bo.na; ++b) {
            memset(hS + bo.p[b], 0, sizeof *hS);
            hS[bo.p[b]].sweeps = batch_sweeps;
        }
    } else if (name.find("7k_cores") != std::string::npos || name.find("k_cores_t") != std::string::npos) {
        const ProbDev *P = *(const ProbDev **)args[0];
        double *G = *(double **)args[2];
        int64_t len = 0;
        for (int j = 0; j < P->d; ++j) len += P->F.n[j];
        if (touch(G, 8 * len, dev, "k_cores"))
            for (int64_t i = 0; i < len; ++i) G[i] = (double)(i + 1);
        ProbState *hS = *(ProbState **)args[name.find("k_cores_t") != std::string::npos ? 4 : 3];
        memset(hS, 0, sizeof *hS);
        hS->sweeps = 1;
    } else if (name.find("k_copy_one") != std::string::npos) {
        const double *src = *(const double **)args[0];
        double *dst = *(double **)args[1];
        const int m = *(int *)args[2];
        int *done = *(int **)args[3];
        const int number = *(int *)args[4];
        bool ok = touch(src, 8 * (size_t)m, dev, "core copy, source");
        ok = touch(dst, 8 * (size_t)m, dev, "core copy, target") && ok;
        if (((uintptr_t)dst & 7) != 0) fault("core copy, target: misaligned");
        ok = touch(done, 4, dev, "core copy, flag") && ok;
        if (ok) {
            memcpy(dst, src, 8 * (size_t)m);
            __atomic_store_n(done, number, __ATOMIC_RELEASE);
        }
    }
    return hipSuccess;
}

// As the runtime does it: the range of a known allocation is checked.
hipError_t copy(void *d, const void *s, size_t n)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    for (const void *p : {(const void *)d, s})
        if (find(p) && !find((const char *)p + n - 1)) return hipErrorInvalidValue;
    memcpy(d, s, n);
    return hipSuccess;
}
}  // namespace

extern "C" {

// --- for the tests ---------------------------------------------------------
void fake_hook(void (*f)(const char *, const void *)) { hook = f; }
void fake_set_device(int d) { cur = d; }
void fake_sweeps(int n) { batch_sweeps = n; }
void fake_ranks(int r) { run_rank = r; }
void fake_limit(size_t bytes) { std::lock_guard<std::recursive_mutex> l(mu); limit = bytes ? in_use + bytes : ~(size_t)0; }
void fake_fail(const char *name, int nth) { std::lock_guard<std::recursive_mutex> l(mu); fail_at[name] = nth; }
size_t fake_in_use() { std::lock_guard<std::recursive_mutex> l(mu); return in_use; }
void fake_clear() { std::lock_guard<std::recursive_mutex> l(mu); log_.clear(); faults.clear(); }
static int out(const std::vector<std::string> &v, char *buf, int n)
{
    std::string s;
    for (auto &x : v) s += x + "\n";
    snprintf(buf, n, "%s", s.c_str());
    return (int)v.size();
}
int fake_log(char *buf, int n) { std::lock_guard<std::recursive_mutex> l(mu); return out(log_, buf, n); }
int fake_faults(char *buf, int n) { std::lock_guard<std::recursive_mutex> l(mu); return out(faults, buf, n); }
void *fake_malloc(size_t n, int host) { void *p; return alloc(&p, n, host != 0) == hipSuccess ? p : nullptr; }

// --- the runtime's names ---------------------------------------------------
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s)
{
    configs.push_back(Config{g, b, lds, s});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s)
{
    const Config c = configs.back();
    configs.pop_back();
    *g = c.g; *b = c.b; *lds = c.lds; *s = c.s;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *x; return &x; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *dev, unsigned, void *, void *, void *, void *, int *)
{
    names[host] = dev;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

hipError_t hipGetDevice(int *d) { *d = cur; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 163840; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) { memset(a, 0, sizeof *a); return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) { return alloc(p, 16 << 20, false); }

hipError_t hipMalloc(void **p, size_t n)
{
    note("hipMalloc " + std::to_string(n));
    if (fails("hipMalloc")) { *p = nullptr; return hipErrorOutOfMemory; }
    return alloc(p, n, false);
}
hipError_t hipFree(void *p) { fails("hipFree", p); return release(p, "hipFree"); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return alloc(p, n, true); }
hipError_t hipHostFree(void *p) { fails("hipHostFree", p); return release(p, "hipHostFree"); }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return copy(d, s, n); }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    if (fails("hipMemcpyAsync")) return hipErrorUnknown;
    const int dev = stream_dev(st, "hipMemcpyAsync");
    char line[128];
    snprintf(line, sizeof line, "hipMemcpyAsync %zu dev %d stream %p", n, dev, (void *)st);
    note(line);
    return copy(d, s, n);
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    const Block *b = find(p);
    memset(a, 0, sizeof *a);
    if (!b || b->freed) return hipErrorInvalidValue;
    a->type = b->host ? hipMemoryTypeHost : hipMemoryTypeDevice;
    a->device = b->dev;
    a->devicePointer = const_cast<void *>(p);
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    auto it = blocks.upper_bound((char *)p);
    if (it == blocks.begin()) return hipErrorInvalidValue;
    --it;
    if ((char *)p >= it->first + it->second.size || it->second.freed) return hipErrorInvalidValue;
    *base = it->first;
    *size = it->second.size;
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    std::lock_guard<std::recursive_mutex> l(mu);
    Stream *x = new Stream{cur, false};
    streams.insert(x);
    *s = (hipStream_t)x;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    fails("hipStreamDestroy", s);
    stream_dev(s, "hipStreamDestroy");
    std::lock_guard<std::recursive_mutex> l(mu);
    ((Stream *)s)->dead = true;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    char line[64];
    snprintf(line, sizeof line, "hipStreamSynchronize %p", (void *)s);
    note(line);
    stream_dev(s, "hipStreamSynchronize");
    return fails("hipStreamSynchronize", s) ? hipErrorUnknown : hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) { stream_dev(s, "hipStreamQuery"); return hipSuccess; }

// an event's time is the number of records and attached launches before it
static float clock_ms = 0.0f;
struct Event { float ms; };
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t) new Event{-1.0f}; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { ((Event *)e)->ms = ++clock_ms; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b)
{
    if (((Event *)a)->ms < 0 || ((Event *)b)->ms < 0) return hipErrorInvalidHandle;
    *ms = ((Event *)b)->ms - ((Event *)a)->ms;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *fn, dim3 g, dim3, void **args, size_t, hipStream_t s) { return launch(fn, g, args, s); }
hipError_t hipExtLaunchKernel(const void *fn, dim3 g, dim3, void **args, size_t, hipStream_t s, hipEvent_t a, hipEvent_t b, int)
{
    const hipError_t e = launch(fn, g, args, s);
    // a launch of g workgroups takes g milliseconds
    if (a) ((Event *)a)->ms = clock_ms;
    if (b) ((Event *)b)->ms = clock_ms + (float)g.x;
    return e;
}

}  // extern "C"
