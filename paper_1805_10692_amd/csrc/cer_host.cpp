// Host-side encoder and decoder of the CER / CSER formats (Section III-A of the paper).
//
// The encoder is a row-parallel counting sort; a team of threads goes through all its steps:
//   symbols  element -> codebook symbol through a hash of the fp32 bit pattern; per-row histograms
//   (order)  symbols ranked by count (Section III-A step 1: frequency-major Omega)
//   sizes    per row: number of indexed elements and of groups
//   (scan)   exclusive prefix sums give every row its slice of colI / OmegaPtr / OmegaI
//   fill     per row: scatter the columns into their rank bucket (ascending inside a bucket because
//            columns are visited in order) and write the bucket boundaries as the row's pointers
// Conversion cost is O(m.n), as the paper notes in Section V.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>
#include <numeric>
#include <mutex>
#include <new>
#include <thread>

#include <climits>
#include <emmintrin.h>
#include <linux/futex.h>
#include <pthread.h>
#include <sys/syscall.h>
#include <unistd.h>

#include "../../include/cer.h"
#include "cer_internal.hpp"

namespace cer {
namespace {

inline uint32_t value_bits(float v) {
    uint32_t u;
    std::memcpy(&u, &v, 4);
    return u == 0x80000000u ? 0u : u;  // -0.0 and +0.0 are one value, stored as +0.0
}

// fp32 bit pattern -> position in the caller's codebook: a table without collisions where one of a few multipliers gives
// one (always, in practice, up to a few hundred values: the table may be large, only the K occupied slots are touched), so
// that a look-up is one load and no branch; else a table with open addressing.
class SymbolTable {
public:
    struct Slot {
        uint32_t key, sym;
    };
    static constexpr uint32_t kFree = 0xFFFFFFFFu;  // the pattern of a NaN: no codebook value

    // false: a value occurs twice
    bool build(const float* codebook, int32_t K) {
        uint32_t bits = 4;
        while ((1u << bits) < (uint32_t)K * 4u && bits < 31) ++bits;
        const uint32_t first = bits, last = K <= 1024 ? first + 6 : first - 1;
        for (; bits <= last; ++bits) {
            for (uint32_t t = 0; t < 8; ++t) {
                mul_ = 0x9E3779B1u + t * 0x7F4A7C16u;  // odd
                shift_ = 32 - bits;
                slots_.assign((size_t)1 << bits, Slot{kFree, 0});
                bool ok = true;
                for (int32_t k = 0; k < K && ok; ++k) {
                    Slot& s = slots_[slot(value_bits(codebook[k]))];
                    if (s.key == value_bits(codebook[k])) return false;
                    ok = s.key == kFree;
                    s = Slot{value_bits(codebook[k]), (uint32_t)k};
                }
                if (ok) {
                    perfect_ = true;
                    return true;
                }
            }
        }
        perfect_ = false;
        mul_ = 0x9E3779B1u;
        shift_ = 32 - first;
        slots_.assign((size_t)1 << first, Slot{kFree, 0});
        for (int32_t k = 0; k < K; ++k) {
            const uint32_t key = value_bits(codebook[k]);
            size_t h = slot(key);
            while (slots_[h].key != kFree) {
                if (slots_[h].key == key) return false;
                h = (h + 1) & (slots_.size() - 1);
            }
            slots_[h] = Slot{key, (uint32_t)k};
        }
        return true;
    }
    bool perfect() const { return perfect_; }
    // the slot of a key in a table without collisions; the caller compares the key (kFree is never a codebook value)
    const Slot& at(uint32_t key) const { return slots_[slot(key)]; }
    int32_t find(uint32_t key) const {
        if (key == kFree) return -1;
        size_t h = slot(key);
        while (slots_[h].key != kFree) {
            if (slots_[h].key == key) return (int32_t)slots_[h].sym;
            h = (h + 1) & (slots_.size() - 1);
        }
        return -1;
    }

private:
    size_t slot(uint32_t key) const { return (size_t)((key * mul_) >> shift_); }
    uint32_t mul_ = 1, shift_ = 28;
    bool perfect_ = false;
    std::vector<Slot> slots_;
};

// Threads that wait between calls: starting 15 of them takes 160 us, waking them 20, and until the last one runs 60 to 100 (a 2048 x 2048
// layer is encoded in 250).  At most 15; they sleep on a futex after having looked for work for kAwake: a handle that has been encoded is on its
// way to the device for some 60 us, and what converts a layer often converts it back or goes on with the next (encode and decode in turn,
// looking for 25 / 250 us, with the counters apart: 1172 x 1576, 50 values, 330 -> 263 us, 779 x 1437, 26 values, 186 -> 140).  Behind a call
// that stands alone nobody comes, and 15 threads would spend 4 ms of processor time for nothing: they look for work while a call lasts, and
// afterwards only if it began within kAwake of the one before (HostCall).  A fork leaves the child without them
// (it starts its own).  One call at a time uses them (Crew).
class Workers {
public:
    using Job = void (*)(void* ctx, int t);
    // For the caller alone until it lets go; null: they are busy.
    static Workers* hold() {
        Workers* w = instance();
        return w && w->mu_.try_lock() ? w : nullptr;
    }
    void let_go() { mu_.unlock(); }
    // job(ctx, t) for t = 0 .. threads - 1, 0 on the calling thread, which holds them; returns false (nothing has run) if there are too few
    bool run(int threads, Job job, void* ctx) {
        if (threads > kMost + 1) return false;
        while (started_ < threads - 1) {
            try {
                std::thread(&Workers::loop, this, started_ + 1, turn_.load(std::memory_order_relaxed)).detach();
            } catch (...) {  // no more threads, or no memory for one
                return false;
            }
            ++started_;
        }
        job_ = job;
        ctx_ = ctx;
        members_ = threads;
        linger_.store(true, std::memory_order_relaxed);
        left_.store(started_, std::memory_order_relaxed);
        turn_.fetch_add(1, std::memory_order_seq_cst);
        if (asleep_.load(std::memory_order_seq_cst) > 0) syscall(SYS_futex, &turn_, FUTEX_WAKE_PRIVATE, INT_MAX, nullptr, nullptr, 0);
        job(ctx, 0);
        for (int spins = 0; left_.load(std::memory_order_acquire) > 0; ++spins) {
            if (spins < 4000) _mm_pause(); else std::this_thread::yield();
        }
        return true;
    }

    static constexpr std::chrono::microseconds kAwake{250};
    // The call that has used the threads ends; no other follows at once.
    static void rest() {
        if (Workers* w = slot().load(std::memory_order_acquire)) w->linger_.store(false, std::memory_order_relaxed);
    }

    // Ends the threads (they are started again when needed), unless they are busy.
    static void stop() {
        Workers* w = slot().load(std::memory_order_acquire);
        if (!w || !w->mu_.try_lock()) return;
        std::lock_guard<std::mutex> hold(w->mu_, std::adopt_lock);
        w->quit_ = true;
        w->left_.store(w->started_, std::memory_order_relaxed);
        w->turn_.fetch_add(1, std::memory_order_seq_cst);
        syscall(SYS_futex, &w->turn_, FUTEX_WAKE_PRIVATE, INT_MAX, nullptr, nullptr, 0);
        while (w->left_.load(std::memory_order_acquire) > 0) std::this_thread::yield();
        w->started_ = 0;
        w->quit_ = false;
    }

private:
    static constexpr int kMost = 15;
    static std::atomic<Workers*>& slot() {
        static std::atomic<Workers*> s{nullptr};
        return s;
    }
    static Workers* instance() {
        Workers* w = slot().load(std::memory_order_acquire);
        if (w) return w;
        static std::mutex mu;
        std::lock_guard<std::mutex> hold(mu);
        w = slot().load(std::memory_order_acquire);
        if (w) return w;
        static bool once = pthread_atfork(nullptr, nullptr, [] { slot().store(nullptr); }) == 0;
        if (!once) return nullptr;
        w = new (std::nothrow) Workers();  // never destroyed: its threads wait in it until the process ends
        slot().store(w, std::memory_order_release);
        return w;
    }
    void loop(int t, uint32_t seen) {
        for (;;) {
            uint32_t now = turn_.load(std::memory_order_acquire);
            std::chrono::steady_clock::time_point until{};
            for (int spins = 0; now == seen; now = turn_.load(std::memory_order_acquire)) {
                if (++spins < 1500) {
                    _mm_pause();
                    continue;
                }
                if (spins == 1500) until = std::chrono::steady_clock::now() + kAwake;
                if (linger_.load(std::memory_order_relaxed) && std::chrono::steady_clock::now() < until) {
                    std::this_thread::yield();  // (others that want the processor get it)
                    continue;
                }
                asleep_.fetch_add(1, std::memory_order_seq_cst);
                if (turn_.load(std::memory_order_seq_cst) == seen)
                    syscall(SYS_futex, &turn_, FUTEX_WAIT_PRIVATE, seen, nullptr, nullptr, 0);
                asleep_.fetch_sub(1, std::memory_order_relaxed);
            }
            seen = now;
            const bool quit = quit_;
            if (!quit && t < members_) job_(ctx_, t);
            left_.fetch_sub(1, std::memory_order_acq_rel);
            if (quit) return;
        }
    }
    std::mutex mu_;
    std::atomic<uint32_t> turn_{0};
    std::atomic<int> asleep_{0}, left_{0};
    std::atomic<bool> linger_{false};
    int started_ = 0, members_ = 0;
    bool quit_ = false;
    Job job_ = nullptr;
    void* ctx_ = nullptr;
};

// Who works on `work` elements: the waiting threads, or, where those are busy with another call, threads started for it.  One for every 64 Ki elements;
// the waiting ones, whom it costs nothing to start, one for every 16 Ki, but no more than three quarters of the processors for that: whoever else
// wants one of them (the runtime's threads, another call) stops a thread that all others wait for.  At most 16 and never more than there are rows.
// us there and back on 16 processors, one for every 64 Ki / one for every 16 Ki, up to 16 / up to 12: 300 x 900, 30 values, in turn 250 / 141, one call in
// ten 830 to 990 / 146, in two threads at once 360 / 1540 / 295, in four 690 / 3760 / 720; 498 x 848, 214 values 380 / 230 (740) / 245, in two 610 /
// 1960 / 840, in four 1600 / 4490 / 1840.  (A thread takes 1 to 2 ns per element; waiting for the others costs some us each of five times, starting one
// 10 us.)
class Crew {
public:
    Crew(int64_t rows, int64_t work) {
        const int64_t processors = std::max(1u, std::thread::hardware_concurrency());
        const int64_t few = std::max<int64_t>(1, std::min<int64_t>({16, processors, rows, (work + 65535) / 65536}));
        const int64_t more = std::min<int64_t>({16, processors * 3 / 4, rows, (work + 16383) / 16384});
        size_ = (int)std::max(few, more);
        if (size_ > 1 && !(waiting_ = Workers::hold())) size_ = (int)few;
    }
    ~Crew() {
        if (waiting_) waiting_->let_go();
    }
    Crew(const Crew&) = delete;
    Crew& operator=(const Crew&) = delete;
    int size() const { return size_; }
    Workers* waiting() const { return waiting_; }

private:
    Workers* waiting_ = nullptr;
    int size_ = 1;
};

// A team runs body(t, r0, r1, team) on its threads, each with a contiguous share of m rows; sync() waits for all of them.
// The bodies must not throw (what they need is allocated before).
class Team {
public:
    template <typename F>
    static void run(const Crew& crew, int64_t m, F&& body) {
        const int threads = crew.size();
        Team team;
        auto work = [&](int t) {
            const int n = team.size_.load(std::memory_order_relaxed);
            body(t, m * t / n, m * (t + 1) / n, team);
        };
        team.size_.store(threads, std::memory_order_relaxed);
        if (threads == 1) return work(0);
        using Work = decltype(work);
        if (crew.waiting() && crew.waiting()->run(threads, [](void* ctx, int t) { (*static_cast<Work*>(ctx))(t); }, &work)) return;
        team.size_.store(0, std::memory_order_relaxed);
        std::vector<std::thread> pool;
        pool.reserve((size_t)threads - 1);
        try {
            for (int t = 1; t < threads; ++t)
                pool.emplace_back([&team, &work, t] {
                    while (team.size_.load(std::memory_order_acquire) == 0) std::this_thread::yield();
                    work(t);
                });
        } catch (...) {  // no more threads to be had, or no memory for one: the ones there are share the rows (and are joined)
        }
        team.size_.store((int)pool.size() + 1, std::memory_order_release);
        work(0);
        for (auto& th : pool) th.join();
    }
    void sync() {
        const int n = size_.load(std::memory_order_relaxed);
        const int turn = turn_.load(std::memory_order_relaxed);
        if (arrived_.fetch_add(1, std::memory_order_acq_rel) + 1 == n) {
            arrived_.store(0, std::memory_order_relaxed);
            turn_.store(turn + 1, std::memory_order_release);
            return;
        }
        for (int spins = 0; turn_.load(std::memory_order_acquire) == turn; ++spins) {
            if (spins < 4000) _mm_pause(); else std::this_thread::yield();
        }
    }

private:
    std::atomic<int> size_{0}, arrived_{0}, turn_{0};
};

void store(HostArray& a, uint64_t i, uint32_t v) {
    switch (a.bits) {
        case 8: a.bytes[(size_t)i] = (uint8_t)v; break;
        case 16: reinterpret_cast<uint16_t*>(a.bytes.data())[i] = (uint16_t)v; break;
        default: reinterpret_cast<uint32_t*>(a.bytes.data())[i] = v;
    }
}

void shape(HostArray& a, uint64_t len, int bits) {
    a.len = (int64_t)len;
    a.bits = bits;
    a.bytes.resize((size_t)len * (size_t)(bits / 8));
}

// Symbols of one row and their histogram (four interleaved ones: a value that follows itself does not wait for its own
// last increment); false: an element is no codebook value.  `likely`: the symbol to expect (and its bit pattern): sixteen
// elements are compared with it at once, and only the others are looked up.
template <typename SymT>
bool row_symbols(const SymbolTable& table, const float* W, int64_t n, int32_t K, int32_t likely, uint32_t likely_key, SymT* sym,
                 uint32_t* h4, uint32_t* c) {
    std::fill(h4, h4 + 4 * (size_t)K, 0u);
    uint32_t bad = 0;
    int64_t j = 0;
    if (table.perfect()) {
        auto one = [&](int64_t i, uint32_t* h) {
            const uint32_t key = value_bits(W[i]);
            const SymbolTable::Slot s = table.at(key);
            bad |= (s.key ^ key) | (uint32_t)(key == SymbolTable::kFree);
            sym[i] = (SymT)s.sym;
            ++h[s.sym];
        };
        if (sizeof(SymT) == 1) {
            const __m128i want = _mm_set1_epi32((int)likely_key), fill = _mm_set1_epi8((char)likely);
            int64_t others = 0;
            for (; j + 16 <= n; j += 16) {
                const __m128i* p = reinterpret_cast<const __m128i*>(W + j);
                const __m128i a = _mm_cmpeq_epi32(_mm_loadu_si128(p), want), b = _mm_cmpeq_epi32(_mm_loadu_si128(p + 1), want);
                const __m128i d = _mm_cmpeq_epi32(_mm_loadu_si128(p + 2), want), e = _mm_cmpeq_epi32(_mm_loadu_si128(p + 3), want);
                uint32_t rest = 0xFFFFu ^ (uint32_t)_mm_movemask_epi8(_mm_packs_epi16(_mm_packs_epi32(a, b), _mm_packs_epi32(d, e)));
                _mm_storeu_si128(reinterpret_cast<__m128i*>(sym + j), fill);
                others += __builtin_popcount(rest);
                uint32_t* h = h4;
                for (; rest; rest &= rest - 1u) {
                    one(j + __builtin_ctz(rest), h);
                    h = h == h4 ? h4 + K : h4;
                }
            }
            h4[likely] += (uint32_t)(j - others);
        }
        for (; j + 4 <= n; j += 4) {
            one(j, h4);
            one(j + 1, h4 + K);
            one(j + 2, h4 + 2 * (size_t)K);
            one(j + 3, h4 + 3 * (size_t)K);
        }
        for (; j < n; ++j) one(j, h4);
    } else {
        for (; j < n; ++j) {
            const int32_t s = table.find(value_bits(W[j]));
            if (s < 0) return false;
            sym[j] = (SymT)s;
            ++h4[s];
        }
    }
    for (int32_t k = 0; k < K; ++k) c[k] = h4[k] + h4[(size_t)K + k] + h4[2 * (size_t)K + k] + h4[3 * (size_t)K + k];
    return bad == 0;
}

template <typename SymT>
void row_histogram(const SymT* sym, int64_t n, int32_t K, uint32_t* c) {
    std::fill(c, c + K, 0u);
    for (int64_t j = 0; j < n; ++j) ++c[sym[j]];
}

// Columns of the row's elements that do not hold the symbol `dom`, each to the next slot of its symbol's bucket.
template <typename SymT, typename ColT>
void row_scatter(const SymT* sym, int64_t n, uint32_t dom, uint32_t* fill, ColT* colI) {
    int64_t j = 0;
    if (sizeof(SymT) == 1) {  // 64 symbols at a time; the ones to place come out of a bit mask
        const __m128i d = _mm_set1_epi8((char)dom);
        for (; j + 64 <= n; j += 64) {
            uint64_t mask = 0;
            for (int q = 0; q < 4; ++q) {
                const __m128i v = _mm_loadu_si128(reinterpret_cast<const __m128i*>(sym + j + 16 * q));
                mask |= (uint64_t)(uint16_t)~_mm_movemask_epi8(_mm_cmpeq_epi8(v, d)) << (16 * q);
            }
            while (mask) {
                const int64_t i = j + __builtin_ctzll(mask);
                mask &= mask - 1;
                colI[fill[sym[i]]++] = (ColT)i;
            }
        }
    }
    for (; j < n; ++j)
        if (sym[j] != dom) colI[fill[sym[j]]++] = (ColT)j;
}

template <typename SymT>
int encode_rows(const float* W, int64_t m, int64_t n, const float* codebook, int32_t Kc, const SymbolTable& table,
                HostMatrix& A) {
    const int64_t N = m * n;
    const bool cser = A.cser;
    std::unique_ptr<SymT[]> sym(new SymT[(size_t)std::max<int64_t>(N, 1)]);
    // the rows' histograms are kept unless they would be larger than the matrix (few columns, many values)
    const bool keep = (int64_t)Kc <= n;
    std::unique_ptr<uint32_t[]> rows_c(new uint32_t[keep ? (size_t)m * (size_t)Kc : 1]);
    const Crew crew(m, N);  // (behind the large allocations: others may use the threads meanwhile)
    const int T = crew.size();
    // What a thread counts in has cache lines of its own: with those of a few values next to each other the threads waited for one another at
    // every element (659 x 1121, two values: 356 -> 173 us there and back).
    constexpr size_t kLine = 128;
    auto lines = [](size_t bytes) { return (bytes + kLine - 1) / kLine * kLine + kLine; };
    const size_t Kz = (size_t)std::max(Kc, 1), scratch_of = lines(Kz * 6 * 4) / 4, total_of = lines(Kz * 8) / 8;
    std::vector<uint32_t> scratch((size_t)T * scratch_of);  // per thread: four histograms, counts, bucket positions
    std::vector<int64_t> total((size_t)T * total_of, 0);
    std::vector<uint64_t> row_nnz((size_t)m + 1, 0), row_groups((size_t)m + 1, 0);
    std::vector<int64_t> nonempty_part((size_t)T, 0);
    std::vector<uint32_t> order;  // rank -> symbol
    order.reserve(Kz);
    std::vector<uint32_t> rank_of(Kz, 0);
    std::atomic<bool> missing{false};
    std::atomic<int> rc{CER_OK};

    Team::run(crew, m, [&](int t, int64_t r0, int64_t r1, Team& team) {
        uint32_t* h4 = scratch.data() + (size_t)t * scratch_of;
        uint32_t* own = h4 + 4 * Kz;
        uint32_t* fill = own + Kz;
        int64_t* sum = total.data() + (size_t)t * total_of;
        bool ok = true;
        int32_t likely = 0;  // the most frequent symbol of the rows so far
        for (int64_t r = r0; r < r1 && ok; ++r) {
            uint32_t* c = keep ? rows_c.get() + (size_t)r * Kz : own;
            ok = row_symbols<SymT>(table, W + r * n, n, Kc, likely, Kc > 0 ? value_bits(codebook[likely]) : 0u, sym.get() + r * n, h4, c);
            for (int32_t k = 0; k < Kc; ++k) sum[k] += c[k];
            likely = (int32_t)(std::max_element(sum, sum + Kc) - sum);
        }
        if (!ok) missing.store(true);
        team.sync();
        if (missing.load()) return;

        if (t == 0) {
            // Omega: occurring symbols by count, highest first; stable, so equal counts keep codebook order
            for (int i = 1; i < T; ++i)
                for (int32_t k = 0; k < Kc; ++k) total[(size_t)k] += total[(size_t)i * total_of + (size_t)k];
            for (int32_t k = 0; k < Kc; ++k)
                if (total[(size_t)k] > 0) order.push_back((uint32_t)k);
            std::sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) {
                return total[a] > total[b] || (total[a] == total[b] && a < b);
            });
            for (size_t k = 0; k < order.size(); ++k) rank_of[order[k]] = (uint32_t)k;
        }
        team.sync();
        const int32_t K = (int32_t)order.size();
        int64_t nonempty = 0;

        for (int64_t r = r0; r < r1; ++r) {
            const uint32_t* c = keep ? rows_c.get() + (size_t)r * Kz : own;
            if (!keep) row_histogram(sym.get() + r * n, n, Kc, own);
            uint64_t present = 0, top = 0;
            for (int32_t k = 1; k < K; ++k)
                if (c[order[(size_t)k]]) { ++present; top = (uint64_t)k; }
            row_nnz[(size_t)r] = (uint64_t)n - (K > 0 ? c[order[0]] : 0u);
            row_groups[(size_t)r] = cser ? present : top;
            nonempty += (int64_t)present;
        }
        nonempty_part[(size_t)t] = nonempty;
        team.sync();

        if (t == 0) {
            // exclusive scans
            uint64_t acc_n = 0, acc_g = 0;
            for (int64_t r = 0; r <= m; ++r) {
                const uint64_t a = row_nnz[(size_t)r], g = row_groups[(size_t)r];
                A.max_row_groups = std::max<int64_t>(A.max_row_groups, (int64_t)g);
                row_nnz[(size_t)r] = acc_n;
                row_groups[(size_t)r] = acc_g;
                acc_n += a;
                acc_g += g;
            }
            // the kernels address colI and OmegaPtr with 32-bit offsets and read ahead of a row's end
            const uint64_t limit = 0xFFFFFFFFull - 65536;
            if (acc_n > limit || acc_g > limit) {
                rc.store(CER_E_TOO_LARGE);
            } else {
                try {
                    A.K = K;
                    A.omega.resize((size_t)K);
                    A.count.resize((size_t)K);
                    for (int32_t k = 0; k < K; ++k) {
                        const float v = codebook[order[(size_t)k]];
                        A.omega[(size_t)k] = (v == 0.0f) ? 0.0f : v;
                        A.count[(size_t)k] = total[order[(size_t)k]];
                    }
                    A.nnz = (int64_t)acc_n;
                    A.G = (int64_t)acc_g;
                    A.nonempty_groups = std::accumulate(nonempty_part.begin(), nonempty_part.end(), (int64_t)0);
                    shape(A.colI, acc_n, min_index_bits(n > 0 ? (uint64_t)(n - 1) : 0));
                    shape(A.omegaPtr, acc_g + 1, min_index_bits(acc_n));
                    shape(A.rowPtr, (uint64_t)m + 1, min_index_bits(acc_g));
                    if (cser) shape(A.omegaI, acc_g, min_index_bits(K > 0 ? (uint64_t)(K - 1) : 0));
                    store(A.omegaPtr, 0, 0);
                    store(A.rowPtr, (uint64_t)m, (uint32_t)acc_g);
                } catch (const std::bad_alloc&) {
                    rc.store(CER_E_NOMEM);
                }
            }
        }
        team.sync();
        if (rc.load() != CER_OK) return;

        for (int64_t r = r0; r < r1; ++r) {
            const SymT* s = sym.get() + r * n;
            const uint32_t* c = keep ? rows_c.get() + (size_t)r * Kz : own;
            if (!keep) row_histogram(s, n, Kc, own);
            uint64_t g = row_groups[(size_t)r];
            store(A.rowPtr, (uint64_t)r, (uint32_t)g);
            const uint64_t g_end = row_groups[(size_t)r + 1];
            uint32_t pos = (uint32_t)row_nnz[(size_t)r];
            for (int32_t k = 1; k < K && g < g_end; ++k) {
                const uint32_t len = c[order[(size_t)k]];
                fill[order[(size_t)k]] = pos;
                pos += len;
                if (cser) {
                    if (len == 0) continue;
                    store(A.omegaI, g, (uint32_t)k);
                }
                store(A.omegaPtr, ++g, pos);
            }
            if (K == 0) continue;
            if (A.colI.bits == 8) row_scatter<SymT>(s, n, order[0], fill, A.colI.bytes.data());
            else if (A.colI.bits == 16) row_scatter<SymT>(s, n, order[0], fill, reinterpret_cast<uint16_t*>(A.colI.bytes.data()));
            else row_scatter<SymT>(s, n, order[0], fill, reinterpret_cast<uint32_t*>(A.colI.bytes.data()));
        }
    });
    return missing.load() ? (int)CER_E_NOT_IN_CODEBOOK : rc.load();
}

template <typename ColT>
void decode_rows(const HostMatrix& A, float* W, int64_t r0, int64_t r1) {
    const ColT* colI = reinterpret_cast<const ColT*>(A.colI.bytes.data());
    for (int64_t r = r0; r < r1; ++r) {
        float* row = W + r * A.n;
        std::fill(row, row + A.n, A.omega[0]);
        const int64_t g0 = (int64_t)A.rowPtr.at(r), g1 = (int64_t)A.rowPtr.at(r + 1);
        uint64_t i = A.omegaPtr.at(g0);
        for (int64_t g = g0; g < g1; ++g) {
            const int64_t rank = A.cser ? (int64_t)A.omegaI.at(g) : g - g0 + 1;
            const float v = A.omega[(size_t)rank];
            const uint64_t e = A.omegaPtr.at(g + 1);
            for (; i < e; ++i) row[colI[i]] = v;
        }
    }
}

}  // namespace

void stop_host_threads() { Workers::stop(); }

namespace {
std::atomic<int64_t> g_last_call{INT64_MIN / 2};  // when it ended, ns
int64_t now_ns() { return std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now().time_since_epoch()).count(); }
}  // namespace
HostCall::HostCall() : follows_(now_ns() - g_last_call.load(std::memory_order_relaxed) < std::chrono::nanoseconds(Workers::kAwake).count()) {}
HostCall::~HostCall() {
    g_last_call.store(now_ns(), std::memory_order_relaxed);
    if (!follows_) Workers::rest();
}

// From 256 KiB on the waiting threads share the copy (fifteen layers there and back 0.811 of the time, 0.828 with one thread copying); none are
// started for it (one thread copies 256 KiB in some 20 us, starting 15 takes 160).
void copy_host(void* to, const void* from, size_t bytes) {
    const Crew crew(INT64_MAX, bytes < (size_t)256 << 10 ? 0 : (int64_t)(bytes / 4));
    if (!crew.waiting()) {
        if (bytes) std::memcpy(to, from, bytes);
        return;
    }
    Team::run(crew, (int64_t)(bytes / 64), [&](int, int64_t b0, int64_t b1, Team&) {
        const size_t end = b1 == (int64_t)(bytes / 64) ? bytes : (size_t)b1 * 64;
        std::memcpy(static_cast<char*>(to) + b0 * 64, static_cast<const char*>(from) + b0 * 64, end - (size_t)b0 * 64);
    });
}

int min_index_bits(uint64_t max_value) {
    return max_value <= 0xFFu ? 8 : (max_value <= 0xFFFFu ? 16 : 32);
}

int encode_host(const float* W, int64_t m, int64_t n, const float* codebook, int32_t Kc, bool cser,
                std::shared_ptr<HostMatrix>* out) {
    if (n > (int64_t)0xFFFFFFFFll) return CER_E_TOO_LARGE;
    for (int32_t k = 0; k < Kc; ++k)
        if (!std::isfinite(codebook[k])) return CER_E_BAD_CODEBOOK;
    SymbolTable table;
    if (!table.build(codebook, Kc)) return CER_E_BAD_CODEBOOK;
    auto A = std::make_shared<HostMatrix>();
    A->cser = cser;
    A->m = m;
    A->n = n;
    const int rc = Kc <= 256 ? encode_rows<uint8_t>(W, m, n, codebook, Kc, table, *A)
                             : encode_rows<uint32_t>(W, m, n, codebook, Kc, table, *A);
    if (rc == CER_OK) *out = std::move(A);
    return rc;
}

int decode_host(const HostMatrix& A, float* W) {
    if (A.m * A.n == 0) return CER_OK;
    if (A.K < 1) return CER_E_INVALID;
    Team::run(Crew(A.m, A.m * A.n), A.m, [&](int, int64_t r0, int64_t r1, Team&) {
        if (A.colI.bits == 8) decode_rows<uint8_t>(A, W, r0, r1);
        else if (A.colI.bits == 16) decode_rows<uint16_t>(A, W, r0, r1);
        else decode_rows<uint32_t>(A, W, r0, r1);
    });
    return CER_OK;
}

}  // namespace cer
