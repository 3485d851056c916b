// Device memory cache behind DBuf.  Large hipMalloc/hipFree pairs become slow
// (tens of milliseconds each) once several multi-GB buffers are alive, and the
// setup allocates and frees such buffers at every cascade step; cached blocks
// are reused instead.  A freed block keeps hipFree's ordering guarantee: the
// device is synchronised before the block becomes reusable.  Inside a PoolScope
// (a setup, which works on one stream from one thread) that wait is put off to
// the scope's end: blocks allocated in the scope are reused in stream order
// without it, others wait for the end.  (A setup frees about ten buffers per
// fit step; 576 waits in the setup of the 64^2 SIPG problem, each of which left
// the GPU idle until the next launch.)
#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "cs_internal.h"

namespace cs {
namespace {

constexpr size_t CACHE_CAP = size_t(96) << 30;   // cached bytes per device

struct DevicePool {
    std::multimap<size_t, void *> cached;   // size -> block
    std::unordered_map<void *, size_t> sizes;
    size_t cached_bytes = 0;
};

std::mutex g_mu;
std::map<int, DevicePool> g_pools;
int g_users = 0;

struct ScopeState {
    int dev = 0;
    std::unordered_map<void *, size_t> own;        // allocated in the scope, in use
    std::multimap<size_t, void *> free;            // allocated in the scope, free again
    std::vector<void *> deferred;                  // older blocks, freed in the scope
};
thread_local ScopeState *t_scope = nullptr;

size_t round_size(size_t b) {
    const size_t g = b <= (size_t(1) << 20) ? 4096 : (size_t(2) << 20);
    return (b + g - 1) / g * g;
}

// An unused block into the cache (or back to the device above the cap); the
// device no longer works on it.
void cache_block(DevicePool &pool, void *p) {
    auto s = pool.sizes.find(p);
    if (s == pool.sizes.end()) {   // not ours (cannot happen): plain free
        (void)hipFree(p);
        return;
    }
    if (pool.cached_bytes + s->second > CACHE_CAP) {
        (void)hipFree(p);
        pool.sizes.erase(s);
        return;
    }
    pool.cached.emplace(s->second, p);
    pool.cached_bytes += s->second;
}

void drop_all(int dev, DevicePool &pool) {
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(dev);
    for (auto &kv : pool.cached) {
        (void)hipFree(kv.second);
        pool.sizes.erase(kv.second);
    }
    pool.cached.clear();
    pool.cached_bytes = 0;
    (void)hipSetDevice(cur);
}

}  // namespace

// Give a scope's free blocks back to the cache, after the device has finished.
static void drain_scope(ScopeState &sc) {
    if (sc.free.empty() && sc.deferred.empty()) return;
    (void)hipDeviceSynchronize();
    std::lock_guard<std::mutex> lock(g_mu);
    DevicePool &pool = g_pools[sc.dev];
    for (auto &kv : sc.free) cache_block(pool, kv.second);
    for (void *p : sc.deferred) cache_block(pool, p);
    sc.free.clear();
    sc.deferred.clear();
}

PoolScope::PoolScope() {
    if (t_scope) return;   // nested: the outer scope serves
    ScopeState *sc = new ScopeState;
    if (hipGetDevice(&sc->dev) != hipSuccess) {
        delete sc;
        return;
    }
    state = sc;
    t_scope = sc;
}

PoolScope::~PoolScope() {
    if (!state) return;
    ScopeState *sc = static_cast<ScopeState *>(state);
    t_scope = nullptr;
    drain_scope(*sc);
    delete sc;
}

void *pool_alloc(size_t bytes) {
    const size_t want = round_size(bytes);
    int dev = 0;
    CS_HIP(hipGetDevice(&dev));
    ScopeState *sc = t_scope && t_scope->dev == dev ? t_scope : nullptr;
    if (sc) {
        auto it = sc->free.lower_bound(want);
        if (it != sc->free.end() && it->first <= 2 * want) {
            void *p = it->second;
            sc->own.emplace(p, it->first);
            sc->free.erase(it);
            return p;
        }
    }
    std::unique_lock<std::mutex> lock(g_mu);
    DevicePool &pool = g_pools[dev];
    auto it = pool.cached.lower_bound(want);
    if (it != pool.cached.end() && it->first <= 2 * want) {
        void *p = it->second;
        if (sc) sc->own.emplace(p, it->first);
        pool.cached_bytes -= it->first;
        pool.cached.erase(it);
        return p;
    }
    void *p = nullptr;
    if (hipMalloc(&p, want) != hipSuccess) {
        (void)hipGetLastError();
        if (sc) {   // the scope's free blocks too
            lock.unlock();
            drain_scope(*sc);
            lock.lock();
        }
        drop_all(dev, pool);   // give the cache back and retry once
        if (hipMalloc(&p, want) != hipSuccess) {
            (void)hipGetLastError();
            fail(CS_ENOMEM, "hipMalloc of " + std::to_string(want) + " bytes failed");
        }
    }
    pool.sizes[p] = want;
    if (sc) sc->own.emplace(p, want);
    return p;
}

void pool_free(void *p) {
    if (!p) return;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    if (ScopeState *sc = t_scope && t_scope->dev == dev ? t_scope : nullptr) {
        auto it = sc->own.find(p);
        if (it != sc->own.end()) {   // only this scope's stream has used it
            sc->free.emplace(it->second, p);
            sc->own.erase(it);
        } else {
            sc->deferred.push_back(p);
        }
        return;
    }
    std::lock_guard<std::mutex> lock(g_mu);
    // work still queued on any stream may use the block: wait as hipFree would
    (void)hipDeviceSynchronize();
    cache_block(g_pools[dev], p);
}

void pool_user(int delta) {
    std::lock_guard<std::mutex> lock(g_mu);
    g_users += delta;
    if (g_users == 0)
        for (auto &kv : g_pools) drop_all(kv.first, kv.second);
}

}  // namespace cs
