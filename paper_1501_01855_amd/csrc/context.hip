// Context life cycle, workspace, profiling events.
#include <cstring>

#include <algorithm>

#include <thread>

#include "context.h"
#include "kernels.h"

namespace ovl {

static thread_local std::string g_last_error;

void set_error(const std::string &msg) { g_last_error = msg; }
const char *last_error() { return g_last_error.c_str(); }

size_t Context::room() const
{
    size_t avail = 0, total = 0;
    OVL_HIP(hipMemGetInfo(&avail, &total));
    if (ws_limit) avail = std::min(avail, ws_limit > (size_t)bytes_held ? ws_limit - (size_t)bytes_held : 0);
    return avail;
}

// Gives back memory the context can do without: buffers that hold nothing any
// more (level 0), a running solver's spare basis vectors (1), the FP64 two-row
// links (2: the full links are always there and give the same values).
bool Context::reclaim(int level)
{
    const int64_t before = bytes_held;
    if (level == 0) {
        for (auto &kv : pool)
            if (kv.second.idle) release(kv.first);
    } else if (level == 1) {
        if (shrink) shrink();
    } else if (U64r) {
        OVL_HIP(hipStreamSynchronize(stream));
        OVL_HIP(hipFree(U64r));
        U64r = nullptr;
        bytes_held -= two_row64_bytes(g);
        update_link_form(*this);
    }
    return bytes_held < before;
}

hipError_t Context::device_alloc(void **p, size_t bytes)
{
    hipError_t e = hipErrorOutOfMemory;
    bool limited = false;
    for (int level = -1; level < 3; ++level) {
        if (level >= 0 && !reclaim(level)) continue;
        limited = ws_limit && (size_t)bytes_held + bytes > ws_limit;
        if (limited) continue;
        e = hipMalloc(p, bytes);
        if (e == hipSuccess) return e;
        (void)hipGetLastError();   // reported by the caller, not by the next launch
    }
    *p = nullptr;
    OVL_REQUIRE(!limited, OVL_ERR_NOMEM,
                "the workspace limit leaves no room for " + std::to_string(bytes) + " bytes more");
    return e;
}

void Context::release(const std::string &name)
{
    DevBuf &b = pool[name];
    if (b.p) {
        OVL_HIP(hipStreamSynchronize(stream));
        OVL_HIP(hipFree(b.p));
        bytes_held -= (int64_t)b.bytes;
    }
    b = DevBuf{};
}

void Context::idle(std::initializer_list<const char *> names)
{
    for (const char *n : names) pool[n].idle = true;
}

size_t Context::idle_bytes() const
{
    size_t s = 0;
    for (const auto &kv : pool)
        if (kv.second.idle) s += kv.second.bytes;
    return s;
}

void *Context::buf(const std::string &name, size_t bytes)
{
    DevBuf &b = pool[name];
    b.idle = false;
    if (b.bytes < bytes) {
        release(name);
        if (device_alloc(&b.p, bytes) != hipSuccess)
            throw Error{OVL_ERR_NOMEM, "workspace '" + name + "': hipMalloc of " + std::to_string(bytes) +
                                           " bytes failed"};
        b.bytes = bytes;
        bytes_held += (int64_t)bytes;
    }
    return b.p;
}

void *Context::opt_buf(const std::string &name, size_t bytes)
{
    DevBuf &b = pool[name];
    if (b.bytes < bytes) {
        release(name);
        if (ws_limit && (size_t)bytes_held + bytes > ws_limit) return nullptr;
        if (hipMalloc(&b.p, bytes) != hipSuccess) {
            (void)hipGetLastError();
            b.p = nullptr;
            return nullptr;
        }
        b.bytes = bytes;
        bytes_held += (int64_t)bytes;
    }
    b.idle = false;
    return b.p;
}

double *Context::host_results(size_t n, double **dev)
{
    if (hres_n < n) {
        if (hres) {
            OVL_HIP(hipStreamSynchronize(stream));
            OVL_HIP(hipHostFree(hres));
            hres = nullptr;
        }
        const size_t cap = std::max<size_t>(n, 4096);
        OVL_HIP(hipHostMalloc((void **)&hres, cap * sizeof(double), hipHostMallocMapped | hipHostMallocCoherent));
        OVL_HIP(hipHostGetDevicePointer((void **)&hres_dev, hres, 0));
        hres_n = cap;
    }
    *dev = hres_dev;
    return hres;
}

void Context::spin_wait(hipEvent_t e)
{
    while (true) {
        const hipError_t r = hipEventQuery(e);
        if (r == hipSuccess) return;
        if (r != hipErrorNotReady) OVL_HIP(r);
        std::this_thread::yield();   // several contexts may be polled by threads sharing the cores
    }
}

void *Context::host_stage(size_t bytes)
{
    if (pinned_bytes < bytes) {
        if (pinned) {
            OVL_HIP(hipStreamSynchronize(stream));
            OVL_HIP(hipHostFree(pinned));
            pinned = nullptr;
        }
        OVL_HIP(hipHostMalloc(&pinned, bytes, hipHostMallocDefault));
        pinned_bytes = bytes;
    }
    return pinned;
}

hipEvent_t Context::event()
{
    hipEvent_t e;
    OVL_HIP(hipEventCreate(&e));
    free_events.push_back(e);   // owned by the context; destroyed at exit
    return e;
}

void Context::lowmodes_changed()
{
    OVL_HIP(hipStreamSynchronize(stream));
    for (int p = 1; p < 3; ++p)
        if (low_lp[p]) {
            OVL_HIP(hipFree(low_lp[p]));
            bytes_held -= (int64_t)field_bytes(g, p) * n_low;
            low_lp[p] = nullptr;
        }
    if (low_sgn) {
        OVL_HIP(hipFree(low_sgn));
        low_sgn = nullptr;
    }
}

const void *Context::low_basis(int prec)
{
    if (prec == OVL_F64 || n_low == 0) return low;
    if (!low_lp[prec]) {
        const size_t B = field_bytes(g, prec) * n_low;
        OVL_HIP(device_alloc(&low_lp[prec], B));
        bytes_held += (int64_t)B;
        convert_spinor(*this, low, OVL_F64, low_lp[prec], prec, n_low);
    }
    return low_lp[prec];
}

const double *Context::low_signs()
{
    if (!low_sgn && n_low > 0) {
        std::vector<double> sg(n_low);
        for (int j = 0; j < n_low; ++j) sg[j] = low_evals[j] >= 0.0 ? 1.0 : -1.0;
        OVL_HIP(hipMalloc(&low_sgn, sizeof(double) * n_low));
        OVL_HIP(hipMemcpyAsync(low_sgn, sg.data(), sizeof(double) * n_low, hipMemcpyHostToDevice, stream));
        OVL_HIP(hipStreamSynchronize(stream));   // sg is released on return
    }
    return low_sgn;
}

void Context::prof_begin(PendingEvent &pe, int kern, int prec, double bytes)
{
    pe.kern = kern;
    pe.prec = prec;
    pe.bytes = bytes;
    if (event_pool.size() < 2) {
        for (int i = 0; i < 64; ++i) {
            hipEvent_t e;
            OVL_HIP(hipEventCreate(&e));
            event_pool.push_back(e);
        }
    }
    pe.a = event_pool.back();
    event_pool.pop_back();
    pe.b = event_pool.back();
    event_pool.pop_back();
}

void Context::prof_end(PendingEvent &pe)
{
    pending.push_back(pe);
    if (pending.size() > 32768) prof_collect();
}

void Context::prof_collect()
{
    if (pending.empty()) return;
    OVL_HIP(hipEventSynchronize(pending.back().b));
    for (auto &pe : pending) {
        float ms = 0.f;
        OVL_HIP(hipEventElapsedTime(&ms, pe.a, pe.b));
        ProfileSlot &s = slots[pe.kern][pe.prec];
        s.launches += 1;
        s.ms += ms;
        s.bytes += pe.bytes;
        event_pool.push_back(pe.a);
        event_pool.push_back(pe.b);
    }
    pending.clear();
}

Context::~Context()
{
    hipStreamSynchronize(stream);
    for (auto &pe : pending) {
        hipEventDestroy(pe.a);
        hipEventDestroy(pe.b);
    }
    for (auto e : event_pool) hipEventDestroy(e);
    for (auto e : free_events) hipEventDestroy(e);
    for (auto &kv : pool)
        if (kv.second.p) hipFree(kv.second.p);
    if (U64) hipFree(U64);
    if (U64r) hipFree(U64r);
    if (U32) hipFree(U32);
    if (U16) hipFree(U16);
    if (U32r) hipFree(U32r);
    if (U16r) hipFree(U16r);
    if (low) hipFree(low);
    for (int p = 1; p < 3; ++p)
        if (low_lp[p]) hipFree(low_lp[p]);
    if (low_sgn) hipFree(low_sgn);
    if (ms_pin) hipHostFree(ms_pin);
    for (auto e : ms_ev)
        if (e) hipEventDestroy(e);
    if (sync_ev) hipEventDestroy(sync_ev);
    for (auto &kv : graphs) hipGraphExecDestroy(kv.second);
    if (pinned) hipHostFree(pinned);
    if (hres) hipHostFree(hres);
}

}  // namespace ovl
