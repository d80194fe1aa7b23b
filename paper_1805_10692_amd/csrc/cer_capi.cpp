// extern "C" boundary of the library: argument checks, handle lifetime, device upload.
#include <algorithm>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "../../include/cer.h"
#include "cer_internal.hpp"

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e) {
    g_last_hip_error = (int)e;
    return CER_E_HIP;
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

int cer::record_hip_error(int hip_error) {
    g_last_hip_error = hip_error;
    return CER_E_HIP;
}

// ---- stream-ordered temporaries from a pool of the library's own ------------------------------------------------
namespace {
struct TempPool {
    std::mutex mu;
    bool tried = false;
    hipMemPool_t pool = nullptr;  // nullptr after a failed creation: the device's default pool serves instead
};
TempPool g_temp_pools[16];

// The library's pool on the current device, created on first use.
hipMemPool_t temp_pool() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return nullptr;
    TempPool& t = g_temp_pools[dev];
    std::lock_guard<std::mutex> lock(t.mu);
    if (!t.tried) {
        t.tried = true;
        hipMemPoolProps props;
        std::memset(&props, 0, sizeof props);
        props.allocType = hipMemAllocationTypePinned;
        props.handleTypes = hipMemHandleTypeNone;
        props.location.type = hipMemLocationTypeDevice;
        props.location.id = dev;
        hipMemPool_t pool = nullptr;
        if (hipMemPoolCreate(&pool, &props) == hipSuccess) {
            uint64_t keep = UINT64_MAX;  // nothing goes back to the system before cer_trim
            if (hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep) == hipSuccess)
                t.pool = pool;
            else
                (void)hipMemPoolDestroy(pool);
        }
        (void)hipGetLastError();  // a failed creation is not an error of the call that asked for memory
    }
    return t.pool;
}
}  // namespace

// Blocks that a product has given back, kept for the next one.  A release to the runtime's pool (hipFreeAsync) waits on
// the host until the stream has drained -- 8 us on an idle stream, the whole product on a busy one: AlexNet-fc6 shape
// batch 99 was enqueued in 66 us per call, its own duration -- so blocks go through this list instead:
//   * a block released on the null stream serves later requests of the null stream, which are ordered behind its last use;
//   * a block released on any other stream carries an event: any stream may take it once the event has passed, the same
//     stream at once, behind a wait for the event (a stream's handle may be that of a new stream at the same address).
// The list is bounded (kBlocksKept blocks, kBytesKept bytes per device; the oldest goes first) and cer_trim empties it.
// Under stream capture the runtime's pool is used directly.
namespace {
struct TempBlock {
    void* p = nullptr;
    size_t bytes = 0;
    hipStream_t stream = nullptr;
    hipEvent_t done = nullptr;  // null: released on the null stream
};
constexpr size_t kBlocksKept = 32, kBlocksOut = 256, kBytesKept = (size_t)2 << 30;
struct TempCache {
    TempCache() {  // never grown later: no allocation, no exception in a product
        kept.reserve(kBlocksKept + 1);
        in_use.reserve(kBlocksOut);
        events.reserve(kBlocksKept + 1);
    }
    void spare(hipEvent_t e) {
        if (events.size() < kBlocksKept) events.push_back(e); else (void)hipEventDestroy(e);
    }
    std::mutex mu;
    std::vector<TempBlock> kept;       // oldest first
    std::vector<TempBlock> in_use;     // handed out through this list
    std::vector<hipEvent_t> events;    // spare ones
    size_t kept_bytes = 0;
};
TempCache g_temp_caches[16];

TempCache* temp_cache() {
    int dev = 0;
    return hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 16 ? &g_temp_caches[dev] : nullptr;
}

bool capturing(hipStream_t s) {
    if (!s) return false;  // the null stream cannot be captured
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone;
}

// Blocks on their way back to the runtime's pool: taken from the list under its lock, released without it (release may
// have to wait for the work that used a block last).
struct TempLeaving {
    TempBlock block[kBlocksKept];
    size_t count = 0;
    void take(TempCache& c, size_t i) {
        block[count++] = c.kept[i];
        c.kept_bytes -= c.kept[i].bytes;
        c.kept.erase(c.kept.begin() + (ptrdiff_t)i);
    }
    void release(TempCache& c) {
        for (size_t i = 0; i < count; ++i) {
            if (block[i].done) (void)hipEventSynchronize(block[i].done);
            (void)hipFreeAsync(block[i].p, nullptr);
        }
        std::lock_guard<std::mutex> lock(c.mu);
        for (size_t i = 0; i < count; ++i)
            if (block[i].done) c.spare(block[i].done);
    }
};
}  // namespace

int cer::temp_alloc(void** p, size_t bytes, void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    TempCache* c = temp_cache();
    const bool listed = c && !capturing(s);
    if (listed) {
        std::lock_guard<std::mutex> lock(c->mu);
        size_t best = SIZE_MAX;
        bool wait = false;
        for (size_t i = 0; i < c->kept.size(); ++i) {
            const TempBlock& b = c->kept[i];
            if (b.bytes < bytes || (best != SIZE_MAX && b.bytes >= c->kept[best].bytes)) continue;
            if (b.bytes > (16u << 20) && b.bytes / 4 > bytes) continue;  // a large block is not spent on a small request
            if (!b.done) {
                if (s) continue;
                wait = false;
            } else if (hipEventQuery(b.done) == hipSuccess) {
                wait = false;
            } else {
                (void)hipGetLastError();  // hipErrorNotReady
                if (b.stream != s) continue;
                wait = true;
            }
            best = i;
        }
        if (best != SIZE_MAX && c->in_use.size() < kBlocksOut) {
            TempBlock b = c->kept[best];
            if (!wait || hipStreamWaitEvent(s, b.done, 0) == hipSuccess) {
                c->kept.erase(c->kept.begin() + (ptrdiff_t)best);
                c->kept_bytes -= b.bytes;
                if (b.done) c->spare(b.done);
                b.done = nullptr;
                c->in_use.push_back(b);
                *p = b.p;
                return (int)hipSuccess;
            }
            (void)hipGetLastError();
        }
    }
    hipMemPool_t pool = temp_pool();
    const size_t rounded = (bytes + 65535) & ~(size_t)65535;
    const hipError_t e = pool ? hipMallocFromPoolAsync(p, rounded, pool, s) : hipMallocAsync(p, rounded, s);
    if (e == hipSuccess && listed) {
        std::lock_guard<std::mutex> lock(c->mu);
        if (c->in_use.size() < kBlocksOut) c->in_use.push_back(TempBlock{*p, rounded, s, nullptr});
    }
    return (int)e;
}

int cer::temp_free(void* p, void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    TempCache* c = temp_cache();
    if (c) {
        std::unique_lock<std::mutex> lock(c->mu);
        for (size_t i = c->in_use.size(); i-- > 0;) {
            if (c->in_use[i].p != p) continue;
            TempBlock b = c->in_use[i];
            c->in_use.erase(c->in_use.begin() + (ptrdiff_t)i);
            b.stream = s;
            bool keep = b.bytes <= kBytesKept;
            if (keep && s) {
                if (c->events.empty()) {
                    keep = hipEventCreateWithFlags(&b.done, hipEventDisableTiming) == hipSuccess;
                } else {
                    b.done = c->events.back();
                    c->events.pop_back();
                }
                if (keep && hipEventRecord(b.done, s) != hipSuccess) {
                    c->spare(b.done);
                    keep = false;
                }
                if (!keep) (void)hipGetLastError();
            }
            if (!keep) break;
            TempLeaving out;
            while (!c->kept.empty() && (c->kept.size() >= kBlocksKept || c->kept_bytes + b.bytes > kBytesKept)) out.take(*c, 0);
            c->kept.push_back(b);
            c->kept_bytes += b.bytes;
            lock.unlock();
            if (out.count) out.release(*c);
            return (int)hipSuccess;
        }
    }
    return (int)hipFreeAsync(p, s);
}

// ---- device memory of handles ------------------------------------------------------------------------------------
namespace {
struct HandleBlock {
    void* p = nullptr;
    size_t bytes = 0;
    bool null_stream_only = false;
    uint64_t returned = 0;  // which block it was that came back, counted from 1; 0: nothing has used it yet
};
constexpr size_t kHandleBlocksKept = 16, kHandleBytesKept = (size_t)1 << 30;
struct HandleCache {
    HandleCache() { kept.reserve(kHandleBlocksKept); }  // never grown later: cer_free does not throw
    HandleBlock take(size_t i) {
        const HandleBlock b = kept[i];
        kept.erase(kept.begin() + (ptrdiff_t)i);
        kept_bytes -= b.bytes;
        return b;
    }
    std::mutex mu;                    // held for the bookkeeping only, never while the device is waited for
    std::vector<HandleBlock> kept;    // oldest first
    std::vector<HandleBlock> in_use;
    size_t kept_bytes = 0;
    uint64_t returned = 0;  // blocks that have come back so far
    uint64_t waited = 0;    // for the first so many of them the device has been waited for since
};
HandleCache g_handle_caches[16];

HandleCache* handle_cache() {
    int dev = 0;
    return hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 16 ? &g_handle_caches[dev] : nullptr;
}

// Sizes in steps of an eighth of their power of two (at least 64 KiB), so that layers of about the same size share blocks.
size_t handle_block_bytes(size_t bytes) {
    size_t step = 65536;
    while (step * 16 <= bytes) step <<= 1;
    return (bytes + step - 1) / step * step;
}
}  // namespace

int cer::handle_alloc(void** p, size_t bytes, void* stream) {
    const size_t want = handle_block_bytes(bytes);
    HandleCache* c = handle_cache();
    if (c) {
        std::unique_lock<std::mutex> lock(c->mu);
        size_t best = SIZE_MAX;
        bool best_waits = true;
        for (size_t i = 0; i < c->kept.size(); ++i) {  // blocks that need no wait come first, then the smallest
            const HandleBlock& b = c->kept[i];
            if (b.bytes < want || b.bytes > want + want / 4) continue;
            const bool waits = b.returned > c->waited && !(b.null_stream_only && !stream);
            if (best != SIZE_MAX && (waits != best_waits ? waits : b.bytes >= c->kept[best].bytes)) continue;
            best = i;
            best_waits = waits;
        }
        if (best != SIZE_MAX) {
            c->in_use.push_back(c->kept[best]);
            const HandleBlock b = c->take(best);
            *p = b.p;
            if (!best_waits) return (int)hipSuccess;
            const uint64_t until = c->returned;
            lock.unlock();
            const hipError_t e = hipDeviceSynchronize();  // what was queued on the blocks that have come back is done
            lock.lock();
            if (e == hipSuccess) {
                c->waited = std::max(c->waited, until);
                return (int)hipSuccess;
            }
            (void)hipGetLastError();  // also under capture: a fresh block then
            for (size_t i = c->in_use.size(); i-- > 0;)
                if (c->in_use[i].p == b.p) {
                    c->in_use.erase(c->in_use.begin() + (ptrdiff_t)i);
                    break;
                }
            if (c->kept.size() < kHandleBlocksKept) {
                c->kept.push_back(b);
                c->kept_bytes += b.bytes;
            } else {
                lock.unlock();
                (void)hipFree(b.p);
            }
        }
    }
    hipError_t e = hipMalloc(p, want);
    if (e == hipErrorOutOfMemory && c) {  // what is kept may be what is missing
        (void)hipGetLastError();
        (void)cer_trim();
        e = hipMalloc(p, want);
    }
    if (e == hipSuccess && c) {
        try {
            std::lock_guard<std::mutex> lock(c->mu);
            c->in_use.push_back(HandleBlock{*p, want, false, 0});
        } catch (...) {
            (void)hipFree(*p);
            throw;
        }
    }
    return (int)e;
}

void cer::handle_free(void* p, bool null_stream_only) {
    if (!p) return;
    // the block may belong to a device that is not the current one
    for (HandleCache& c : g_handle_caches) {
        void* out[kHandleBlocksKept + 1];
        size_t n_out = 0;
        bool found = false;
        {
            std::lock_guard<std::mutex> lock(c.mu);
            for (size_t i = 0; i < c.in_use.size() && !found; ++i) {
                if (c.in_use[i].p != p) continue;
                found = true;
                HandleBlock b = c.in_use[i];
                c.in_use.erase(c.in_use.begin() + (ptrdiff_t)i);
                b.null_stream_only = null_stream_only;
                b.returned = ++c.returned;
                if (b.bytes > kHandleBytesKept) {
                    out[n_out++] = b.p;
                    break;
                }
                while (!c.kept.empty() && (c.kept.size() >= kHandleBlocksKept || c.kept_bytes + b.bytes > kHandleBytesKept))
                    out[n_out++] = c.take(0).p;
                c.kept.push_back(b);
                c.kept_bytes += b.bytes;
            }
        }
        for (size_t i = 0; i < n_out; ++i) (void)hipFree(out[i]);
        if (found) return;
    }
    (void)hipFree(p);
}


namespace {

// The array's values as 32-bit words.
void widen(const cer::HostArray& a, uint32_t* out) {
    const size_t n = (size_t)a.len;
    if (a.bits == 8) std::copy_n(a.bytes.data(), n, out);
    else if (a.bits == 16) std::copy_n(reinterpret_cast<const uint16_t*>(a.bytes.data()), n, out);
    else std::memcpy(out, a.bytes.data(), n * 4);
}

// Pinned host memory through which host-encoded handles go to the device (a copy out of pageable memory waits once per
// array, 48 us each): one block is kept, of at most kStageKept bytes.
constexpr size_t kStageKept = 16u << 20;
std::mutex g_stage_mutex;
void* g_stage = nullptr;
size_t g_stage_bytes = 0;

struct StageBlock {
    void* p = nullptr;
    size_t bytes = 0;
    bool get(size_t need) {
        {
            std::lock_guard<std::mutex> lock(g_stage_mutex);
            std::swap(p, g_stage);
            std::swap(bytes, g_stage_bytes);
        }
        if (p && bytes >= need) return true;
        if (p) (void)hipHostFree(p);
        p = nullptr;
        bytes = 65536;
        while (bytes < need) bytes *= 2;
        if (hipHostMalloc(&p, bytes, hipHostMallocPortable) == hipSuccess) return true;
        (void)hipGetLastError();
        p = nullptr;
        return false;
    }
    ~StageBlock() {
        if (!p) return;
        if (bytes <= kStageKept) {
            std::lock_guard<std::mutex> lock(g_stage_mutex);
            if (!g_stage) {
                g_stage = p;
                g_stage_bytes = bytes;
                return;
            }
        }
        (void)hipHostFree(p);
    }
};

}  // namespace

cer::DeviceLayout cer::DeviceLayout::make(size_t colI_bytes, int64_t G, int64_t m, size_t omegaI_bytes, int32_t K) {
    DeviceLayout l;
    l.colI_bytes = colI_bytes;
    l.omegaI_bytes = omegaI_bytes;
    l.off_colI = 0;
    l.off_optr = align_up(l.off_colI + colI_bytes + 8192, 256);  // the product reads ahead of a row's end
    l.off_rptr = align_up(l.off_optr + (size_t)(G + 1) * 4 + 16, 256);
    l.off_oi = align_up(l.off_rptr + (size_t)(m + 1) * 4 + 16, 256);
    l.off_om = align_up(l.off_oi + omegaI_bytes + 16, 256);
    l.off_ri = align_up(l.off_om + (size_t)std::max(K, 1) * 4, 256);
    l.off_tab = align_up(l.off_ri + (size_t)(m + 1) * 8, 256);
    size_t tab_bytes = 0;
    if (K >= 2 && K <= 256 && m > 0) {  // rank table: 4 .. 256 words per row
        l.tab_shift = 2;
        while ((1 << l.tab_shift) < K) ++l.tab_shift;
        tab_bytes = ((size_t)m << l.tab_shift) * 4 + 256;
    }
    l.total = align_up(l.off_tab + tab_bytes, 256);
    return l;
}

namespace {
// Compute units and LDS per workgroup of a device, read once per device.
struct DeviceProps {
    std::once_flag once;
    int cus = 256;
    size_t lds_per_block = 64 * 1024;
};
DeviceProps g_device_props[16];

const DeviceProps& device_props(int dev) {
    DeviceProps& p = g_device_props[(dev >= 0 && dev < 16) ? dev : 0];
    std::call_once(p.once, [&p, dev] {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) == hipSuccess) {
            p.cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
            p.lds_per_block = std::max<size_t>(prop.sharedMemPerBlock, prop.maxSharedMemoryPerMultiProcessor);
        } else {
            (void)hipGetLastError();
        }
    });
    return p;
}
}  // namespace

namespace {
// bf16 numbers that add up to `x` exactly (csrc/cer_split3.hpp: the same split); 0 if one of them is subnormal.
int value_pieces(float x) {
    auto bits = [](float v) { uint32_t u; std::memcpy(&u, &v, 4); return u; };
    auto value = [](uint32_t u) { float v; std::memcpy(&v, &u, 4); return v; };
    int used = 0;
    for (int i = 1; i <= 3 && x != 0.f; ++i) {
        const uint32_t u = bits(x), mag = u & 0x7FFFFFFFu;
        const uint32_t p = (mag >= 0x7F7F0000u ? u : u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u;  // nearest, ties to even
        if ((p & 0x7F800000u) == 0) return 0;
        x -= value(p);
        used = i;
    }
    return x == 0.f ? std::max(used, 1) : 0;
}

// Whether the values are whole multiples of one number in the sense of csrc/cer_split3.hpp (uniform_pieces): three or more values, zero
// among them, at most 256 steps from it, and what a multiple's rounding leaves at most 2^-22 of the value (two binary32 roundings, the
// value's and the step's, leave 2^-23), so that the bits of that rest which its eight-bit number does not hold are below 2^-31 of the
// value.  The step: the range over the number of smallest distances in it (values that do not occur leave gaps).
// A grid beside zero keeps three pieces: its offset times the sum of X is cancelled by the sum of the integers where X has a mean.
// Codebooks of the uniform quantizer, 44 products, 2-norm errors against fp64 over those of three pieces: X normal 0.64 in the
// mean, cut at 0 up to 1.22, |x| + 1 up to 2.5, constant up to 90.  With zero on the grid, 29 products: 0.56 (at most 0.86), 0.65 (0.95),
// 0.67 (1.00) and 0.66 (1.03).
bool uniform_grid(const std::vector<float>& omega, cer::UniformGrid* grid) {
    if (omega.size() < 3 || omega.size() > 256 || std::find(omega.begin(), omega.end(), 0.f) == omega.end()) return false;
    std::vector<double> v(omega.begin(), omega.end());
    std::sort(v.begin(), v.end());
    const double range = v.back() - v.front(), largest = std::max(std::fabs(v.front()), std::fabs(v.back()));
    double gap = range;
    for (size_t k = 0; k + 1 < v.size(); ++k) gap = std::min(gap, v[k + 1] - v[k]);
    if (!(gap > 0) || !(range / gap < 512.5) || largest > 0x1p100) return false;
    const float s = (float)(range / std::rint(range / gap));
    if (!(s > 0x1p-80f)) return false;
    for (double w : v) {
        const double j = std::rint(w / s), rest = w - s * j;
        if (std::fabs(j) > 256.0 || std::fabs(rest) > 0x1p-22 * std::fabs(w)) return false;
    }
    int e;
    std::frexp(s, &e);
    grid->unit = std::ldexp(1.f, e - 1);
    grid->scale = s / grid->unit;
    grid->inverse = 1.0 / s;
    return true;
}
}  // namespace

void cer::bind_device(cer_matrix* h, int dev, void* base, const DeviceLayout& l) {
    const HostMatrix& A = *h->host;
    auto* b = static_cast<unsigned char*>(base);
    h->device = dev;
    h->d_base = base;
    h->d_bytes = l.total;
    h->stream_bytes = (int64_t)(l.colI_bytes + (size_t)(A.G + 1) * 4 + (size_t)(A.m + 1) * 4 + l.omegaI_bytes +
                                A.omega.size() * 4);
    DeviceView& v = h->view;
    v.colI = b + l.off_colI;
    v.omegaPtr = reinterpret_cast<const uint32_t*>(b + l.off_optr);
    v.rowPtr = reinterpret_cast<const uint32_t*>(b + l.off_rptr);
    v.omegaI = b + l.off_oi;
    v.omega = reinterpret_cast<const float*>(b + l.off_om);
    v.rowInfo = b + l.off_ri;
    v.rank_tab = l.tab_shift ? reinterpret_cast<const uint32_t*>(b + l.off_tab) : nullptr;
    v.rank_tab_shift = l.tab_shift;
    v.colI_bits = A.colI.bits;
    v.omegaI_bits = A.omegaI.bits;
    v.cser = A.cser ? 1 : 0;
    v.K = A.K;
    v.m = A.m;
    v.n = A.n;
    v.max_row_groups = A.max_row_groups;
    v.nnz = A.nnz;
    v.nonempty_groups = A.nonempty_groups;
    v.omega0 = A.K > 0 ? A.omega[0] : 0.f;
    v.pieces = A.K > 0 ? 1 : 0;
    for (float w : A.omega) {
        const int p = value_pieces(w);
        v.pieces = p && v.pieces ? std::max(v.pieces, p) : 0;
        v.omega_max = std::max(v.omega_max, std::fabs(w));
    }
    v.grid = {};
    if (v.pieces > 2 && v.rank_tab) uniform_grid(A.omega, &v.grid);
    const DeviceProps& dp = device_props(dev);
    v.cus = dp.cus;
    v.lds_per_block = dp.lds_per_block;
    h->layout = l;
}

int cer::ensure_host_arrays(const cer_matrix* h) {
    const HostMatrix& A = *h->host;
    if (A.arrays_on_host.load(std::memory_order_acquire)) return CER_OK;
    std::lock_guard<std::mutex> lock(A.fetch_mutex);
    if (A.arrays_on_host.load(std::memory_order_relaxed)) return CER_OK;
    if (h->device < 0 || !h->d_base) return CER_E_INVALID;
    const auto* b = static_cast<const unsigned char*>(h->d_base);
    const DeviceLayout& l = h->layout;
    hipError_t e = hipSuccess;
    auto get = [&](void* dst, size_t off, size_t bytes) {
        if (e == hipSuccess && bytes) e = hipMemcpy(dst, b + off, bytes, hipMemcpyDeviceToHost);
    };
    auto narrow = [](const std::vector<uint32_t>& src, HostArray& dst) {  // dst.len and dst.bits are already set
        dst.bytes.resize(src.size() * (size_t)(dst.bits / 8));
        for (size_t i = 0; i < src.size(); ++i) {
            if (dst.bits == 8) dst.bytes[i] = (uint8_t)src[i];
            else if (dst.bits == 16) reinterpret_cast<uint16_t*>(dst.bytes.data())[i] = (uint16_t)src[i];
            else reinterpret_cast<uint32_t*>(dst.bytes.data())[i] = src[i];
        }
    };
    A.colI.bytes.resize(l.colI_bytes);
    get(A.colI.bytes.data(), l.off_colI, l.colI_bytes);
    A.omegaI.bytes.resize(l.omegaI_bytes);
    get(A.omegaI.bytes.data(), l.off_oi, l.omegaI_bytes);
    std::vector<uint32_t> optr((size_t)A.G + 1), rptr((size_t)A.m + 1);
    get(optr.data(), l.off_optr, optr.size() * 4);
    get(rptr.data(), l.off_rptr, rptr.size() * 4);
    if (e != hipSuccess) return hip_fail(e);
    narrow(optr, A.omegaPtr);
    narrow(rptr, A.rowPtr);
    A.arrays_on_host.store(true, std::memory_order_release);
    return CER_OK;
}

namespace {
// P: positions per part of a long row
uint64_t part_length(uint64_t mean) { return ((std::max<uint64_t>(mean + mean / 2, 2048) + 2047) / 2048) * 2048; }
}  // namespace

bool cer::row_schedule_wanted(uint64_t nnz, uint64_t m, uint64_t longest) {
    if (m == 0 || nnz == 0) return false;
    const uint64_t mean = nnz / m;
    if (longest < 2048 || longest <= 2 * mean) return false;
    // rows of a few dozen indices are bound by their wave's start-up chain, to which the look-up of the row adds a
    // step: 16384 x 4096 with 41 indices per row and three rows of about 3000 measured 8 % slower in order
    return mean >= 256 || longest > 3 * part_length(mean);
}

// Rows of unequal length (pruned layers; matrices of independent elements have none).  One wave serves one row per
// batch tile and a workgroup holds its resources until its longest row is done, so the batched product
//  - takes the rows in descending order of length when the longest row holds more than twice the average (and at
//    least 2048 positions; the average row at least 256, or some row is split): the four rows of a workgroup are
//    then about equally long and the long rows start first;
//  - serves rows in parts when one of them would outlast the launch: if some row holds more than 3 P positions, P =
//    1.5 x the average row rounded up to a multiple of 2048, the rows of more than 2 P positions are split into parts
//    of P positions (the table lists every part but a row's first; the second kernel and the temporary that the parts
//    need cost about 6 us per product, hence the 3 P).
// Device table: [order: m x uint32][parts: {row, first position, end position, 0}][rows: {row, first part, parts, 0}].
int cer::build_row_schedule(cer_matrix* h, const std::vector<uint64_t>& start) {
    const cer::HostMatrix& A = *h->host;
    if (A.m <= 0 || A.nnz <= 0 || h->device < 0) return CER_OK;
    uint64_t longest = 0;
    for (int64_t r = 0; r < A.m; ++r) longest = std::max(longest, start[(size_t)r + 1] - start[(size_t)r]);
    if (!row_schedule_wanted((uint64_t)A.nnz, (uint64_t)A.m, longest)) return CER_OK;
    const uint64_t mean = (uint64_t)(A.nnz / A.m);
    const uint64_t len = part_length(mean);

    std::vector<uint32_t> order((size_t)A.m);
    for (int64_t r = 0; r < A.m; ++r) order[(size_t)r] = (uint32_t)r;
    std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) {
        return start[(size_t)a + 1] - start[a] > start[(size_t)b + 1] - start[b];
    });

    std::vector<uint32_t> parts, rows;
    if (longest > 3 * len && len <= 0x3FFFFFFFull) {
        for (int64_t r = 0; r < A.m; ++r) {
            const uint64_t rs = start[(size_t)r], re = start[(size_t)r + 1];
            if (re - rs <= 2 * len) continue;
            const uint32_t first = (uint32_t)(parts.size() / 4);
            for (uint64_t b = rs + len; b < re; b += len) {
                parts.push_back((uint32_t)r);
                parts.push_back((uint32_t)b);
                parts.push_back((uint32_t)std::min(re, b + len));
                parts.push_back(0u);
            }
            rows.push_back((uint32_t)r);
            rows.push_back(first);
            rows.push_back((uint32_t)(parts.size() / 4) - first);
            rows.push_back(0u);
        }
    }
    const size_t order_bytes = (order.size() * 4 + 15) & ~(size_t)15, part_bytes = parts.size() * 4, row_bytes = rows.size() * 4;
    void* base = nullptr;
    hipError_t e = (hipError_t)handle_alloc(&base, order_bytes + part_bytes + row_bytes + 16, nullptr);
    if (e != hipSuccess) return hip_fail(e);
    auto* b8 = static_cast<unsigned char*>(base);
    e = hipMemcpy(b8, order.data(), order.size() * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess && part_bytes) e = hipMemcpy(b8 + order_bytes, parts.data(), part_bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess && row_bytes) e = hipMemcpy(b8 + order_bytes + part_bytes, rows.data(), row_bytes, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        handle_free(base, true);
        return hip_fail(e);
    }
    h->d_split = base;
    h->view.row_order = base;
    h->view.split_parts = b8 + order_bytes;
    h->view.split_rows = b8 + order_bytes + part_bytes;
    h->view.n_split_parts = (uint32_t)(parts.size() / 4);
    h->view.n_split_rows = (uint32_t)(rows.size() / 4);
    h->view.split_len = (uint32_t)len;
    h->view.split_min = parts.empty() ? 0xFFFFFFFFu : (uint32_t)(2 * len);
    return CER_OK;
}

namespace {

// Copies the host arrays into one fresh device allocation (layout: cer::DeviceLayout).  Everything but the rank table,
// which the device derives, is laid out in host memory first and copied at once.
int upload(cer_matrix* h) {
    const cer::HostMatrix& A = *h->host;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) {
        (void)hipGetLastError();
        h->device = -1;
        return CER_OK;  // host-only handle
    }
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);

    const cer::DeviceLayout l = cer::DeviceLayout::make(A.colI.bytes.size(), A.G, A.m, A.omegaI.bytes.size(), A.K);
    void* base = nullptr;
    e = (hipError_t)cer::handle_alloc(&base, l.total, nullptr);
    if (e != hipSuccess) return hip_fail(e);
    cer::bind_device(h, dev, base, l);  // from here on the caller frees the allocation with the handle

    StageBlock stage;
    std::vector<unsigned char> pageable;
    unsigned char* img = nullptr;
    if (l.off_tab <= kStageKept && stage.get(l.off_tab)) {
        img = static_cast<unsigned char*>(stage.p);
    } else {
        pageable.resize(l.off_tab);
        img = pageable.data();
    }
    auto put = [&](size_t off, const void* src, size_t bytes, size_t end) {  // an array and the zeros behind it
        cer::copy_host(img + off, src, bytes);
        std::memset(img + off + bytes, 0, end - off - bytes);
    };
    put(l.off_colI, A.colI.bytes.data(), l.colI_bytes, l.off_optr);
    auto* optr = reinterpret_cast<uint32_t*>(img + l.off_optr);
    auto* rptr = reinterpret_cast<uint32_t*>(img + l.off_rptr);
    auto* info = reinterpret_cast<uint32_t*>(img + l.off_ri);
    const size_t optr_bytes = (size_t)(A.G + 1) * 4, rptr_bytes = (size_t)(A.m + 1) * 4;
    widen(A.omegaPtr, optr);
    widen(A.rowPtr, rptr);
    std::memset(img + l.off_optr + optr_bytes, 0, l.off_rptr - l.off_optr - optr_bytes);
    std::memset(img + l.off_rptr + rptr_bytes, 0, l.off_oi - l.off_rptr - rptr_bytes);
    put(l.off_oi, A.omegaI.bytes.data(), l.omegaI_bytes, l.off_om);
    put(l.off_om, A.omega.data(), A.omega.size() * 4, l.off_ri);
    for (int64_t r = 0; r <= A.m; ++r) {
        info[(size_t)r * 2] = rptr[(size_t)r];
        info[(size_t)r * 2 + 1] = optr[rptr[(size_t)r]];
    }
    std::memset(img + l.off_ri + 2 * rptr_bytes, 0, l.off_tab - l.off_ri - 2 * rptr_bytes);
    e = hipMemcpyAsync(base, img, l.off_tab, hipMemcpyHostToDevice, nullptr);
    if (e == hipSuccess) e = (hipError_t)cer::build_rank_table(h->view, nullptr);
    const hipError_t f = hipStreamSynchronize(nullptr);  // the image may be used again
    if (e == hipSuccess) e = f;
    if (e != hipSuccess) return hip_fail(e);
    if (A.m <= 0 || A.nnz <= 0) return CER_OK;
    // the row schedule: from the rows' first colI positions, where some row is long enough
    uint64_t longest = 0;
    for (int64_t r = 0; r < A.m; ++r)
        longest = std::max<uint64_t>(longest, info[(size_t)r * 2 + 3] - info[(size_t)r * 2 + 1]);
    h->view.longest_row = (uint32_t)longest;
    if (!cer::row_schedule_wanted((uint64_t)A.nnz, (uint64_t)A.m, longest)) return CER_OK;
    std::vector<uint64_t> start((size_t)A.m + 1);
    for (int64_t r = 0; r <= A.m; ++r) start[(size_t)r] = info[(size_t)r * 2 + 1];
    return cer::build_row_schedule(h, start);
}

// A handle under construction: also an exception (no host memory for the image of its arrays) gives its memory back.
using HandleOwner = std::unique_ptr<cer_matrix, void (*)(cer_handle_t*)>;

int encode_any(const float* W, int64_t m, int64_t n, const float* codebook, int32_t K, bool cser, cer_handle_t** out) {
    if (!out) return CER_E_INVALID;
    *out = nullptr;
    if (m < 0 || n < 0 || K < 0) return CER_E_INVALID;
    if ((m > 0 && n > 0 && !W) || (K > 0 && !codebook)) return CER_E_INVALID;
    if (m > 0 && n > 0 && K == 0) return CER_E_NOT_IN_CODEBOOK;
    if (m > 0x7FFFFFFFll) return CER_E_TOO_LARGE;
    const cer::HostCall call;
    try {
        std::shared_ptr<cer::HostMatrix> host;
        int rc = cer::encode_host(W, m, n, codebook, K, cser, &host);
        if (rc != CER_OK) return rc;
        HandleOwner h(new cer_matrix(), cer_free);
        h->host = std::move(host);
        rc = upload(h.get());
        if (rc != CER_OK) return rc;
        *out = h.release();
        return CER_OK;
    } catch (const std::bad_alloc&) {
        return CER_E_NOMEM;
    } catch (...) {
        return CER_E_INVALID;
    }
}

// cer_matmul_opts_t -> the launchers' options; false: a field holds a value the header does not define.
bool read_options(const cer_matmul_opts_t* in, cer::MatmulOptions* out) {
    *out = cer::MatmulOptions{};
    if (!in) return true;
    constexpr uint32_t known = CER_OPT_SUM_THEN_MULTIPLY | CER_OPT_ROWS_WHOLE | CER_OPT_X_FROM_GLOBAL |
                               CER_OPT_ONE_COLUMN_PER_LANE | CER_OPT_SHORT_CHUNKS | CER_OPT_LONG_CHUNKS |
                               CER_OPT_NO_RANK_TABLE;
    if (in->path < CER_PATH_AUTO || in->path > CER_PATH_STRIP) return false;
    if (in->flags & ~known) return false;
    if ((in->flags & CER_OPT_SHORT_CHUNKS) && (in->flags & CER_OPT_LONG_CHUNKS)) return false;
    switch (in->tile_cols) {
        case 0: case 8: case 16: case 32: case 64: case 128: break;
        default: return false;
    }
    out->path = in->path;
    out->tile_cols = in->tile_cols;
    out->flags = in->flags;
    return true;
}

// Work on `stream` is about to use the handle's device arrays (cer_free wants to know).
void note_stream(const cer_handle_t* h, void* stream) {
    if (stream && !h->off_null_stream.load(std::memory_order_relaxed)) h->off_null_stream.store(true, std::memory_order_relaxed);
}

// The handle's device is the current one and holds its arrays; else the CER_* code to return.
int check_device(const cer_handle_t* h) {
    if (h->device < 0 || !h->d_base) {
        g_last_hip_error = (int)hipErrorNoDevice;
        return CER_E_HIP;
    }
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev != h->device) return hip_fail(hipErrorInvalidDevice);
    return CER_OK;
}

int matmul_any(const cer_handle_t* h, int want_cser /* -1: either */, const float* X, float* Y, int64_t batch, void* stream,
               const cer_matmul_opts_t* opts) {
    if (!h || !X || !Y || batch < 1) return CER_E_INVALID;
    if (want_cser >= 0 && h->host->cser != (want_cser != 0)) return CER_E_FORMAT;
    cer::MatmulOptions o;
    if (!read_options(opts, &o)) return CER_E_INVALID;
    const int dc = check_device(h);
    if (dc != CER_OK) return dc;
    note_stream(h, stream);
    const int rc = cer::launch_matmul(h->view, X, Y, batch, stream, o);
    return rc == 0 ? CER_OK : hip_fail((hipError_t)rc);
}

int decode_any(const cer_handle_t* h, bool want_cser, float* W_out) {
    if (!h) return CER_E_INVALID;
    if (h->host->cser != want_cser) return CER_E_FORMAT;
    if (!W_out && h->host->m * h->host->n > 0) return CER_E_INVALID;
    const cer::HostCall call;
    try {
        const int rc = cer::ensure_host_arrays(h);
        if (rc != CER_OK) return rc;
        return cer::decode_host(*h->host, W_out);
    } catch (...) {
        return CER_E_NOMEM;
    }
}

}  // namespace

extern "C" {

int cer_encode(const float* W, int64_t m, int64_t n, const float* codebook, int32_t K, cer_handle_t** out) {
    return encode_any(W, m, n, codebook, K, false, out);
}
int cser_encode(const float* W, int64_t m, int64_t n, const float* codebook, int32_t K, cer_handle_t** out) {
    return encode_any(W, m, n, codebook, K, true, out);
}

int cer_matmul(const cer_handle_t* h, const float* X, float* Y, int64_t batch, void* stream) {
    return matmul_any(h, 0, X, Y, batch, stream, nullptr);
}
int cser_matmul(const cer_handle_t* h, const float* X, float* Y, int64_t batch, void* stream) {
    return matmul_any(h, 1, X, Y, batch, stream, nullptr);
}
int cer_matmul_ex(const cer_handle_t* h, const float* X, float* Y, int64_t batch, void* stream,
                  const cer_matmul_opts_t* opts) {
    return matmul_any(h, -1, X, Y, batch, stream, opts);
}

int cer_matmul_noalloc(const cer_handle_t* h, const float* X, float* Y, int64_t batch, void* stream) {
    if (!h || !X || !Y || batch < 1) return CER_E_INVALID;
    const int dc = check_device(h);
    if (dc != CER_OK) return dc;
    float* ws = nullptr;
    size_t ws_floats = 0;
    const int we = cer::static_workspace(&ws, &ws_floats);
    if (we != 0) return hip_fail((hipError_t)we);
    const cer::MatmulOptions o;
    if (cer::matmul_workspace_floats(h->view, batch, o) > ws_floats) return CER_E_TOO_LARGE;
    note_stream(h, stream);
    const int rc = cer::launch_matmul(h->view, X, Y, batch, stream, o, ws, ws_floats);
    return rc == 0 ? CER_OK : hip_fail((hipError_t)rc);
}

int cer_matmul_path_ex(const cer_handle_t* h, int64_t batch, const cer_matmul_opts_t* opts) {
    if (!h || batch < 1) return CER_E_INVALID;
    cer::MatmulOptions o;
    if (!read_options(opts, &o)) return CER_E_INVALID;
    if (h->device < 0 || !h->d_base) return CER_E_HIP;
    return cer::matmul_path(h->view, batch, o);
}
int cer_matmul_path(const cer_handle_t* h, int64_t batch) { return cer_matmul_path_ex(h, batch, nullptr); }

int cer_matmul_narrow_columns(const cer_handle_t* h, int64_t batch) {
    if (!h || batch < 1) return CER_E_INVALID;
    if (h->device < 0 || !h->d_base) return CER_E_HIP;
    return cer::matmul_narrow_columns(h->view, batch);
}

int cer_matmul_fused_rows(const cer_handle_t* h, int64_t batch) {
    if (!h || batch < 1) return CER_E_INVALID;
    if (h->device < 0 || !h->d_base) return CER_E_HIP;
    return cer::matmul_fused_rows(h->view, batch);
}

int cer_matmul_tile_columns(const cer_handle_t* h, int64_t batch) {
    if (!h || batch < 1) return CER_E_INVALID;
    if (h->device < 0 || !h->d_base) return CER_E_HIP;
    return cer::matmul_tile_columns(h->view, batch);
}

int cer_encode_sorts_rows(const cer_handle_t* h, int32_t K) {
    if (!h || K < 1 || K > 256) return CER_E_INVALID;
    if (h->device < 0 || !h->d_base) return CER_E_HIP;
    return cer::encode_sorts_rows(h->view, K) ? 1 : 0;
}

int cer_matmul_planes(const cer_handle_t* h) {
    if (!h) return CER_E_INVALID;
    if (h->device < 0 || !h->d_base) return CER_E_HIP;
    return cer::matmul_planes(h->view);
}

int cer_decode(const cer_handle_t* h, float* W_out) { return decode_any(h, false, W_out); }
int cser_decode(const cer_handle_t* h, float* W_out) { return decode_any(h, true, W_out); }

int cer_get_array(const cer_handle_t* h, int which, const void** host_ptr, int64_t* len, int32_t* elem_bits) {
    if (!h || !host_ptr || !len || !elem_bits) return CER_E_INVALID;
    const cer::HostMatrix& A = *h->host;
    const cer::HostArray* a = nullptr;
    switch (which) {
        case CER_ARRAY_OMEGA: *host_ptr = A.omega.data(); *len = A.K; *elem_bits = 32; return CER_OK;
        case CER_ARRAY_COUNT: *host_ptr = A.count.data(); *len = A.K; *elem_bits = 64; return CER_OK;
        case CER_ARRAY_COLI: a = &A.colI; break;
        case CER_ARRAY_OMEGAPTR: a = &A.omegaPtr; break;
        case CER_ARRAY_ROWPTR: a = &A.rowPtr; break;
        case CER_ARRAY_OMEGAI: a = &A.omegaI; break;
        default: return CER_E_INVALID;
    }
    try {
        const int rc = cer::ensure_host_arrays(h);
        if (rc != CER_OK) return rc;
    } catch (...) {
        return CER_E_NOMEM;
    }
    *host_ptr = a->bytes.data();
    *len = a->len;
    *elem_bits = a->bits;
    return CER_OK;
}

int cer_get_dims(const cer_handle_t* h, int64_t* m, int64_t* n, int32_t* K, int64_t* nnz, int64_t* groups,
                 int32_t* is_cser) {
    if (!h) return CER_E_INVALID;
    const cer::HostMatrix& A = *h->host;
    if (m) *m = A.m;
    if (n) *n = A.n;
    if (K) *K = A.K;
    if (nnz) *nnz = A.nnz;
    if (groups) *groups = A.G;
    if (is_cser) *is_cser = A.cser ? 1 : 0;
    return CER_OK;
}

int64_t cer_storage_bits(const cer_handle_t* h) {
    if (!h) return CER_E_INVALID;
    const cer::HostMatrix& A = *h->host;
    int64_t bits = (int64_t)A.K * 32 + A.colI.len * A.colI.bits + A.omegaPtr.len * A.omegaPtr.bits +
                   A.rowPtr.len * A.rowPtr.bits;
    if (A.cser) bits += A.omegaI.len * A.omegaI.bits;
    return bits;
}

int cer_get_stats(const cer_handle_t* h, double* H, double* p0, double* k_bar, double* k_tilde) {
    if (!h) return CER_E_INVALID;
    const cer::HostMatrix& A = *h->host;
    const double N = (double)A.m * (double)A.n;
    double ent = 0.0;
    for (int32_t k = 0; k < A.K; ++k) {
        const double p = N > 0 ? (double)A.count[(size_t)k] / N : 0.0;
        if (p > 0) ent -= p * std::log2(p);
    }
    if (H) *H = ent;
    if (p0) *p0 = (A.K > 0 && N > 0) ? (double)A.count[0] / N : 0.0;
    if (k_bar) *k_bar = A.m > 0 ? (double)A.nonempty_groups / (double)A.m : 0.0;
    if (k_tilde) *k_tilde = A.m > 0 ? (double)(A.G - A.nonempty_groups) / (double)A.m : 0.0;
    return CER_OK;
}

int cer_clone_device(const cer_handle_t* h, cer_handle_t** out) {
    if (!h || !out) return CER_E_INVALID;
    *out = nullptr;
    const cer::HostCall call;
    try {
        int rc = cer::ensure_host_arrays(h);
        if (rc != CER_OK) return rc;
        HandleOwner c(new cer_matrix(), cer_free);
        c->host = h->host;
        rc = upload(c.get());
        if (rc != CER_OK) return rc;
        *out = c.release();
        return CER_OK;
    } catch (const std::bad_alloc&) {
        return CER_E_NOMEM;
    }
}

static int device_front_end(const float* W, int64_t m, int64_t n, const float* codebook, int32_t K, int32_t bits,
                            int32_t format, void* stream, float* codebook_out, int32_t* K_out, cer_handle_t** out) {
    if (!out) return CER_E_INVALID;
    *out = nullptr;
    if (K_out) *K_out = 0;
    if (m < 0 || n < 0 || (format != CER_FORMAT_CER && format != CER_FORMAT_CSER)) return CER_E_INVALID;
    if (m > 0 && n > 0 && !W) return CER_E_INVALID;
    if (m > 0x7FFFFFFFll || n > (int64_t)0xFFFFFFFFll) return CER_E_TOO_LARGE;
    const bool cser = format == CER_FORMAT_CSER;
    if (m == 0 || n == 0) return encode_any(nullptr, m, n, codebook, bits > 0 ? 0 : K, cser, out);  // nothing to read
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) {
        (void)hipGetLastError();
        return hip_fail(hipErrorNoDevice);
    }
    try {
        return cer::encode_device(W, m, n, codebook, K, bits, cser, stream, codebook_out, K_out, out);
    } catch (const std::bad_alloc&) {
        return CER_E_NOMEM;
    } catch (...) {
        return CER_E_INVALID;
    }
}

int cer_encode_device(const float* W, int64_t m, int64_t n, const float* codebook, int32_t K, int32_t format, void* stream,
                      cer_handle_t** out) {
    if (K < 0 || (K > 0 && !codebook)) return CER_E_INVALID;
    if (K > 256) return CER_E_TOO_LARGE;
    if (m > 0 && n > 0 && K == 0) return CER_E_NOT_IN_CODEBOOK;
    return device_front_end(W, m, n, codebook, K, 0, format, stream, nullptr, nullptr, out);
}

int cer_quantize_encode_device(const float* W, int64_t m, int64_t n, int32_t bits, int32_t format, void* stream,
                               float* codebook_out, int32_t* K_out, cer_handle_t** out) {
    if (bits < 1 || bits > 8) return CER_E_INVALID;
    return device_front_end(W, m, n, nullptr, 0, bits, format, stream, codebook_out, K_out, out);
}

int cer_decode_device(const cer_handle_t* h, float* W, void* stream) {
    if (!h) return CER_E_INVALID;
    if (!W && h->host->m * h->host->n > 0) return CER_E_INVALID;
    if (h->device < 0 || !h->d_base) return hip_fail(hipErrorNoDevice);
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev != h->device) return hip_fail(hipErrorInvalidDevice);
    if (h->host->m * h->host->n > 0 && h->host->K < 1) return CER_E_INVALID;
    note_stream(h, stream);
    return cer::decode_device(h->view, W, stream);
}

int cer_quantize_uniform(const float* W, int64_t count, int32_t bits, uint8_t* codes, float* Wq, float* codebook_out,
                         int32_t* K_out, void* stream) {
    if (K_out) *K_out = 0;
    if (bits < 1 || bits > 8 || count < 0 || (count > 0 && !W)) return CER_E_INVALID;
    if (count == 0) return CER_OK;
    if (count > ((int64_t)1 << 42)) return CER_E_TOO_LARGE;
    try {
        return cer::quantize_device(W, count, bits, codes, Wq, codebook_out, K_out, stream);
    } catch (...) {
        return CER_E_NOMEM;
    }
}

int cer_prepare_strips(cer_handle_t* h) {
    if (!h) return CER_E_INVALID;
    if (h->d_strip) return CER_OK;
    const cer::HostMatrix& A = *h->host;
    if (A.K > 64) return CER_E_TOO_LARGE;  // the rank shares 16 bits with the column inside the strip
    if (h->device < 0 || !h->d_base) return hip_fail(hipErrorNoDevice);
    if (A.m <= 0 || A.n <= 0) return CER_OK;
    const int dc = check_device(h);
    if (dc != CER_OK) return dc;
    try {
        const int rc = cer::ensure_host_arrays(h);
        if (rc != CER_OK) return rc;
        // as few strips as 1024 rows each allow, all equally long (4608 columns: five strips of 922, not four of 1024
        // and a half-empty fifth)
        const uint64_t ns = ((uint64_t)A.n + cer::kStripRows - 1) / cer::kStripRows, m = (uint64_t)A.m;
        const uint64_t S = ((uint64_t)A.n + ns - 1) / ns;
        if (ns * (m + 1) > 0x7FFFFFFFull) return CER_E_TOO_LARGE;
        // rank of every raw group (Algorithm 3: position in the row + 1; Algorithm 4: OmegaI)
        std::vector<uint32_t> ptr((size_t)(ns * (m + 1)) + 1, 0u);
        auto for_each = [&](auto&& fn) {
            for (uint64_t r = 0; r < m; ++r) {
                const uint64_t ga = A.rowPtr.at((int64_t)r), gb = A.rowPtr.at((int64_t)r + 1);
                for (uint64_t g = ga; g < gb; ++g) {
                    const uint32_t rank = A.cser ? (uint32_t)A.omegaI.at((int64_t)g) : (uint32_t)(g - ga + 1);
                    const uint64_t pa = A.omegaPtr.at((int64_t)g), pb = A.omegaPtr.at((int64_t)g + 1);
                    for (uint64_t p = pa; p < pb; ++p) fn(r, rank, (uint64_t)A.colI.at((int64_t)p));
                }
            }
        };
        for_each([&](uint64_t r, uint32_t, uint64_t c) { ++ptr[(size_t)((c / S) * (m + 1) + r) + 1]; });
        // entries -> chunks of eight (the last chunk of a (strip, row) is padded with entries of rank 0: weight zero),
        // then counts -> offsets; the entry after each strip's m rows stays a running total, so ptr[s * (m + 1) + m]
        // closes row m - 1
        for (size_t i = 1; i < ptr.size(); ++i) ptr[i] = (ptr[i] + 7u) / 8u;
        for (size_t i = 1; i < ptr.size(); ++i) {
            if ((uint64_t)ptr[i] + ptr[i - 1] >= 0xFFFFFFFFull) return CER_E_TOO_LARGE;
            ptr[i] += ptr[i - 1];
        }
        const uint64_t nchunks = ptr.back();
        std::vector<uint16_t> idx(((size_t)nchunks + 1) * 8, (uint16_t)0);  // one chunk of zeros closes the index
        std::vector<uint64_t> fill(ptr.size() - 1);
        for (size_t i = 0; i + 1 < ptr.size(); ++i) fill[i] = (uint64_t)ptr[i] * 8u;
        for_each([&](uint64_t r, uint32_t rank, uint64_t c) {
            const uint64_t s = c / S;
            idx[(size_t)fill[(size_t)(s * (m + 1) + r)]++] = (uint16_t)((rank << 10) | (uint32_t)(c - s * S));
        });
        const size_t idx_bytes = (idx.size() * 2 + 255) & ~(size_t)255, ptr_bytes = (ptr.size() - 1) * 4;
        // Both indexes, or neither: an error leaves the handle as it was.
        struct Block {
            void* p = nullptr;
            ~Block() { cer::handle_free(p, true); }
            void* release() { return std::exchange(p, nullptr); }
        } strips, tile;
        hipError_t e = (hipError_t)cer::handle_alloc(&strips.p, idx_bytes + ptr_bytes + 256, nullptr);
        if (e != hipSuccess) return hip_fail(e);
        auto* b8 = static_cast<unsigned char*>(strips.p);
        if (!idx.empty()) e = hipMemcpy(b8, idx.data(), idx.size() * 2, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(b8 + idx_bytes, ptr.data(), ptr_bytes, hipMemcpyHostToDevice);
        if (e != hipSuccess) return hip_fail(e);
        cer::DeviceView view = h->view;
        view.strip_idx = strips.p;
        view.strip_ptr = reinterpret_cast<const uint32_t*>(b8 + idx_bytes);
        view.n_strips = (uint32_t)ns;
        view.strip_rows = (uint32_t)S;
        view.strip_chunks = nchunks;
        // The tile index, written by a kernel.  Products do without it where no batch would take it or there is no memory for it, and only there.
        const size_t tile_bytes = cer::tile_index_pays(view) ? cer::tile_index_bytes(view) : 0;
        if (tile_bytes > 0) {
            e = (hipError_t)cer::handle_alloc(&tile.p, tile_bytes, nullptr);
            if (e == hipErrorOutOfMemory) {
                (void)hipGetLastError();
                tile.p = nullptr;
            } else {
                if (e == hipSuccess) e = (hipError_t)cer::build_tile_index(view, tile.p, nullptr);
                const hipError_t f = hipStreamSynchronize(nullptr);
                if (e == hipSuccess) e = f;
                if (e != hipSuccess) return hip_fail(e);
            }
        }
        view.tile_index = tile.p;
        h->view = view;
        h->d_strip = strips.release();
        h->d_tile = tile.release();
        return CER_OK;
    } catch (const std::bad_alloc&) {
        return CER_E_NOMEM;
    } catch (...) {
        return CER_E_INVALID;
    }
}

int64_t cer_device_bytes(const cer_handle_t* h) { return (h && h->device >= 0) ? h->stream_bytes : 0; }

int64_t cer_long_row_parts(const cer_handle_t* h) { return (h && h->device >= 0) ? (int64_t)h->view.n_split_parts : 0; }

void cer_free(cer_handle_t* h) {
    if (!h) return;
    const bool null_only = !h->off_null_stream.load(std::memory_order_relaxed);
    cer::handle_free(h->d_base, null_only);
    cer::handle_free(h->d_split, null_only);
    cer::handle_free(h->d_strip, null_only);
    cer::handle_free(h->d_tile, null_only);
    delete h;
}

int dense_matmul(const float* W, const float* X, float* Y, int64_t m, int64_t n, int64_t batch, void* stream) {
    if (m < 0 || n < 0 || batch < 1) return CER_E_INVALID;
    if (!Y || (n > 0 && m > 0 && !W) || (n > 0 && !X)) return CER_E_INVALID;
    const int rc = cer::launch_dense(W, X, Y, m, n, batch, stream);
    return rc == 0 ? CER_OK : hip_fail((hipError_t)rc);
}

int cer_stream_copy(void* dst, const void* src, int64_t bytes, void* stream) {
    if (!dst || !src || bytes < 0) return CER_E_INVALID;
    if ((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) & 15u) return CER_E_INVALID;
    const int rc = cer::launch_stream_copy(dst, src, bytes, stream);
    return rc == 0 ? CER_OK : hip_fail((hipError_t)rc);
}

int cer_stream_read(const void* src, int64_t bytes, void* sink, void* stream) {
    if (!src || !sink || bytes < 0) return CER_E_INVALID;
    if ((reinterpret_cast<uintptr_t>(src) & 15u) || (reinterpret_cast<uintptr_t>(sink) & 3u)) return CER_E_INVALID;
    const int rc = cer::launch_stream_read(src, bytes, sink, stream);
    return rc == 0 ? CER_OK : hip_fail((hipError_t)rc);
}

int cer_trim(void) {
    cer::stop_host_threads();
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hip_fail(hipGetLastError());
    if (dev < 0 || dev >= 16) return CER_OK;
    {
        TempCache& c = g_temp_caches[dev];
        TempLeaving out;
        {
            std::lock_guard<std::mutex> lock(c.mu);
            for (size_t i = c.kept.size(); i-- > 0;) {
                if (c.kept[i].done && hipEventQuery(c.kept[i].done) != hipSuccess)
                    (void)hipGetLastError();  // still in use
                else
                    out.take(c, i);
            }
        }
        out.release(c);
    }
    {
        std::lock_guard<std::mutex> lock(g_stage_mutex);
        if (g_stage) (void)hipHostFree(g_stage);
        g_stage = nullptr;
        g_stage_bytes = 0;
    }
    {
        HandleCache& c = g_handle_caches[dev];
        void* out[kHandleBlocksKept];
        size_t n_out = 0;
        {
            std::lock_guard<std::mutex> lock(c.mu);
            while (!c.kept.empty()) out[n_out++] = c.take(0).p;
        }
        for (size_t i = 0; i < n_out; ++i) (void)hipFree(out[i]);
    }
    TempPool& t = g_temp_pools[dev];
    std::lock_guard<std::mutex> lock(t.mu);
    if (!t.pool) return CER_OK;
    const hipError_t e = hipMemPoolTrimTo(t.pool, 0);
    return e == hipSuccess ? CER_OK : hip_fail(e);
}

const char* cer_strerror(int code) {
    switch (code) {
        case CER_OK: return "ok";
        case CER_E_INVALID: return "invalid argument";
        case CER_E_NOT_IN_CODEBOOK: return "matrix element not in codebook";
        case CER_E_BAD_CODEBOOK: return "codebook has a duplicate, NaN or infinite value";
        case CER_E_TOO_LARGE: return "matrix too large for 32-bit indices";
        case CER_E_NOMEM: return "out of host memory";
        case CER_E_HIP: return "HIP error or no device copy";
        case CER_E_FORMAT: return "handle has the other format";
        default: return "unknown error";
    }
}

int cer_last_hip_error(void) { return g_last_hip_error; }

}  // extern "C"
