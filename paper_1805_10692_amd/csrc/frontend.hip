// Device front-end: a dense fp32 weight matrix that already lives in HBM goes to CER / CSER without a
// trip through the host -- optionally through the uniform quantizer of Section V-B first.
//
//   range     min / max of W (quantizer only)
//   codes     the K = 2^b points of the codebook; element -> codebook position (quantizer: nearest point;
//             otherwise: exact look-up), one byte per element, and a per-row histogram over the positions
//   layout    frequency-major order Omega (Section III-A, step 1); per row: number of indexed elements and of groups;
//             exclusive scans over the rows give every row its slice of colI and of OmegaPtr / OmegaI; the sizes go to
//             the host, which allocates the handle
//   emit      per row: a stable counting sort of the columns by rank writes colI, the bucket ends are
//             the row's pointers (steps 2-4) and its record of the rank table
//
// One wave owns one row in `layout` and `emit`, so no two waves ever write the same output element
// and the result does not depend on scheduling: it is the same array, bit for bit, as the host
// encoder's.  Codebooks of up to 256 values are supported here (one byte per code).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>

#include "../../include/cer.h"
#include "cer_device.hpp"
#include "cer_split3.hpp"
#include "cer_stream.hpp"

namespace {

using cer::kWave;
constexpr int kCodes = 256;  // most codebook positions a byte can name

enum : uint32_t {
    kFlagNonFinite = 1u,  // NaN or infinity among the weights
    kFlagMissing = 2u,    // element that is no codebook value
    kFlagCollide = 4u,    // range too narrow: two of the 2^b points coincide
    kFlagTooLarge = 8u,   // 32-bit offsets do not reach
};

// Small block of device memory the kernels communicate through.
struct FrontState {
    uint32_t flags;
    uint32_t K;         // codebook positions in use (caller's K, or the quantizer's point count)
    uint32_t Kp;        // values that occur = length of Omega
    uint32_t done;      // workgroups of row_layout_kernel that have finished
    unsigned long long count[kCodes];  // occurrences by rank
    float codebook[kCodes];            // value by codebook position
    float omega[kCodes];               // value by rank
    uint32_t rank_of[kCodes];          // codebook position -> rank
    uint32_t pos_of[kCodes];           // rank -> codebook position
};

// What the host needs to know, in pinned host memory: first what the handle's memory and the emitter are chosen by, as soon as the values are
// ranked; then the sizes that the rows add up to; the values with the handle's arrays (read when the stream has been waited for).  Every word
// says for itself that it is there (kWritten), so that nothing orders them: a release for the host writes the L2 back (4096 x 9216, 7 bits, 3 us).
constexpr unsigned long long kWritten = 1ull << 63;
struct FrontResult {
    unsigned long long early[2];   // longest row's indexed elements | K << 32 | Kp << 41 | flags << 50; indexed elements
    unsigned long long totals[3];  // groups; non-empty ones; largest group count of a row | flags << 50
    unsigned long long count[kCodes];
    float codebook[kCodes];
    float omega[kCodes];
};
struct FrontSizes {
    uint32_t flags, K, Kp, longest;
    unsigned long long nnz;
};
__device__ __forceinline__ void tell(unsigned long long* word, unsigned long long value) {
    __hip_atomic_store(word, value | kWritten, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// LDS traffic of one wave is ordered; this only keeps the compiler from moving accesses across.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float canonical(float v) { return v == 0.0f ? 0.0f : v; }

// ------------------------------------------------------------------------------------------------
// range: min / max / finiteness
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void range_take(float w, float& lo, float& hi, uint32_t& bad) {
    bad |= (uint32_t)!(fabsf(w) <= 3.402823466e+38f);
    lo = fminf(lo, w);
    hi = fmaxf(hi, w);
}

// The global histogram is gathered in kHistParts copies (workgroups of codes_kernel add theirs to one of them each), cleared
// by the kernel in front.
// Behind them, in as many copies, lies how often a value occurs in a row at least.
constexpr int kHistParts = 16;
__device__ __forceinline__ uint32_t* least_of(unsigned long long* hist) { return reinterpret_cast<uint32_t*>(hist + kHistParts * kCodes); }
__device__ __forceinline__ void clear_histogram(unsigned long long* hist, FrontState* st) {  // one workgroup of 256 threads
    for (int i = 0; i < kHistParts; ++i) {
        hist[i * kCodes + threadIdx.x] = 0ull;
        least_of(hist)[i * kCodes + threadIdx.x] = 0xFFFFFFFFu;
    }
    if (threadIdx.x == 0) {
        st->flags = 0;
        st->done = 0;
    }
}

constexpr int kRangeParts = 1024;  // most workgroups of range_kernel: four per compute unit, eight loads in flight per thread

// Partial results {min, max, not-finite flag}; the workgroups of codes_kernel finish the reduction themselves (one launch
// less, 16 KiB of L2 reads per workgroup at most).  Bound by the read of W.
__global__ __launch_bounds__(256) void range_kernel(const float* __restrict__ W, int64_t N, float4* __restrict__ part,
                                                    unsigned long long* __restrict__ hist, FrontState* __restrict__ st) {
    if (blockIdx.x == 0 && hist) clear_histogram(hist, st);
    float lo = INFINITY, hi = -INFINITY;
    uint32_t bad = 0;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    // the bulk in 16-byte pieces (W is aligned by the caller's allocator or the scalar loop below takes it all)
    const int64_t N4 = ((reinterpret_cast<uintptr_t>(W) & 15u) == 0) ? N / 4 : 0;
    const float4* W4 = reinterpret_cast<const float4*>(W);
    const auto take = [&](const float4& w) {
        range_take(w.x, lo, hi, bad);
        range_take(w.y, lo, hi, bad);
        range_take(w.z, lo, hi, bad);
        range_take(w.w, lo, hi, bad);
    };
    // Eight loads in flight: 32 KiB in a row per workgroup and round (loads a grid's width apart took 44 us for 4096 x 9216 behind a
    // decoder's writes, 38 this way), or, where that leaves workgroups without work, a grid's width apart.
    constexpr int64_t kTile = 8 * 256;
    if (N4 >= (int64_t)gridDim.x * kTile) {
        for (int64_t b = (int64_t)blockIdx.x * kTile + threadIdx.x; b < N4; b += (int64_t)gridDim.x * kTile) {
            float4 w[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = W4[min(b + 256 * k, N4 - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k) take(w[k]);
        }
    } else if (tid < N4) {
        float4 w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k * stride < N4) w[k] = W4[min(tid + k * stride, N4 - 1)];  // (uniform)
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k * stride < N4) take(w[k]);
    }
    for (int64_t i = N4 * 4 + tid; i < N; i += stride) range_take(W[i], lo, hi, bad);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off, kWave));
        hi = fmaxf(hi, __shfl_xor(hi, off, kWave));
        bad |= (uint32_t)__shfl_xor((int)bad, off, kWave);
    }
    __shared__ float s_lo[4], s_hi[4];
    __shared__ uint32_t s_bad[4];
    const uint32_t wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0) {
        s_lo[wave] = lo;
        s_hi[wave] = hi;
        s_bad[wave] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t any = s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3];
        part[blockIdx.x] = make_float4(fminf(fminf(s_lo[0], s_lo[1]), fminf(s_lo[2], s_lo[3])),
                                       fmaxf(fmaxf(s_hi[0], s_hi[1]), fmaxf(s_hi[2], s_hi[3])), any ? 1.f : 0.f, 0.f);
        if (blockIdx.x == 0 && !hist) st->flags = 0;
    }
}

// The caller's codebook, handed over as a kernel argument, into the state.
struct CodebookArg {
    float v[kCodes];
    uint32_t K;
};
__global__ __launch_bounds__(256) void codebook_kernel(CodebookArg cb, unsigned long long* __restrict__ hist, FrontState* __restrict__ st) {
    const uint32_t t = threadIdx.x;
    clear_histogram(hist, st);
    if (t < cb.K) st->codebook[t] = cb.v[t];
    if (t == 0) st->K = cb.K;
}

// ------------------------------------------------------------------------------------------------
// codes: element -> codebook position; per-row histogram.  One workgroup per row (a flat array is
// cut into rows of row_len elements).
// ------------------------------------------------------------------------------------------------
// Look-up of a value's codebook position: open-addressing hash table in LDS over the bit patterns of the (at most
// 256) codebook values; a free slot holds a pattern no finite value has.
constexpr uint32_t kHashSlots = 1024, kHashFree = 0xFFFFFFFFu;
__device__ __forceinline__ uint32_t hash_slot(uint32_t bits) { return (bits * 2654435761u) >> 22; }

struct CodeCtx {
    uint32_t K;
    float wmin, step, top;
    const float* val;      // LDS: quantizer -> points by position
    const uint32_t* hkey;  // LDS: look-up -> bit pattern stored in each hash slot
    const uint32_t* hpos;  // LDS: look-up -> codebook position of that value
};

template <bool kQuant>
__device__ __forceinline__ uint32_t code_of(float w, const CodeCtx& c, bool& missing) {
#pragma clang fp contract(off)
    if (kQuant) {
        // nearest point, decided in binary32: round-half-even of the scaled coordinate
        float q = 0.f;
        if (c.K > 1) {
            const float d = w - c.wmin;
            q = fminf(fmaxf(rintf(d / c.step), 0.f), c.top);
        }
        return (uint32_t)q;
    }
    const uint32_t bits = __float_as_uint(canonical(w));
    uint32_t h = hash_slot(bits);
    for (;;) {
        const uint32_t key = c.hkey[h];
        if (key == kHashFree) {  // not a codebook value (the table always has free slots)
            missing = true;
            return 0u;
        }
        if (key == bits) return c.hpos[h];
        h = (h + 1u) & (kHashSlots - 1u);
    }
}

// Copies of a long row's histogram: lane l counts in copy l % 4.  Weights have a few frequent values -- of 7-bit codes of Laplace weights one
// in four elements has the first, half of them the first three --, and adds to one address go one after the other: with one copy 4096 x
// 9216, 7 bits, took 48 us instead of 37 (189 MB: what memory delivers; 8 and 4 bits, where fewer meet, took that all along).  Shorter
// rows (`aligned` ones below 4096 elements, others below 1024) keep one: 2836 x 704 11 instead of 13 us, 4096 x 2052 and 2048 x 4096 17
// and 14 either way.  With 16 copies the sum at a row's end took 1 us more.  The copies of a value are 16 banks apart.
constexpr uint32_t kHistCopies = 4, kHistPitch = kCodes + 16;

// Each thread takes four consecutive elements per round: one 16-byte load, four codes, one 4-byte store -- kCopies > 1: wherever the row
// starts, the memory path takes floats and bytes at any address (with singles 4096 x 2050 took 20 us instead of 18, 4096 x 1501 19.4
// instead of 15.3), and only the last one to three of a row come singly; else where `aligned`.
typedef float FourFloats __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t FourBytes __attribute__((aligned(1)));
// kQuant: every workgroup first finishes the min / max reduction from the partial results of range_kernel and lays the
// K = 2^bits points on the range (Section V-B).  Every operation rounds once, to binary32: step = (max - min) / (K - 1),
// point_j = min + j.step, the last point is max itself.  A constant matrix has one point.  Workgroup 0 publishes them.
template <bool kQuant, uint32_t kCopies>
__global__ __launch_bounds__(256) void codes_kernel(const float* __restrict__ W, int64_t total, int64_t rows, int64_t row_len,
                                                    const float4* __restrict__ part, int nparts, int bits,
                                                    FrontState* __restrict__ st, uint8_t* __restrict__ codes,
                                                    uint32_t* __restrict__ cnt, unsigned long long* __restrict__ hist,
                                                    float* __restrict__ Wq, int aligned) {
#pragma clang fp contract(off)
    __shared__ uint32_t s_hist[kCopies][kHistPitch];
    __shared__ float s_val[kCodes];
    __shared__ uint32_t s_hkey[kQuant ? 1 : kHashSlots], s_hpos[kQuant ? 1 : kHashSlots];
    __shared__ float s_lo[4], s_hi[4];
    const uint32_t t = threadIdx.x;
    CodeCtx c;
#pragma unroll
    for (uint32_t i = 0; i < kCopies; ++i) s_hist[i][t] = 0;
    uint32_t* const copy = s_hist[t & (kCopies - 1)];
    if (kQuant) {
        float lo = INFINITY, hi = -INFINITY, bad = 0.f;
        for (int i = (int)t; i < nparts; i += 256) {
            const float4 p = part[i];
            lo = fminf(lo, p.x);
            hi = fmaxf(hi, p.y);
            bad = fmaxf(bad, p.z);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, off, kWave));
            hi = fmaxf(hi, __shfl_xor(hi, off, kWave));
        }
        if ((t & 63u) == 0) {
            s_lo[t >> 6] = lo;
            s_hi[t >> 6] = hi;
        }
        const bool any_bad = __syncthreads_or(bad > 0.f);
        const float wmin = fminf(fminf(s_lo[0], s_lo[1]), fminf(s_lo[2], s_lo[3])) + 0.0f;  // -0.0 -> +0.0
        const float wmax = fmaxf(fmaxf(s_hi[0], s_hi[1]), fmaxf(s_hi[2], s_hi[3])) + 0.0f;
        const uint32_t K = (wmin == wmax) ? 1u : (1u << bits);
        const float step = (K > 1) ? (wmax - wmin) / (float)(K - 1) : 0.0f;
        float p = 0.f;
        if (t < K) {
            const float prod = (float)t * step;
            p = prod + wmin;
            if (t == K - 1) p = wmax;
            if (K == 1) p = wmin;
        }
        s_val[t] = p;
        c.K = K;
        c.wmin = wmin;
        c.step = step;
        __syncthreads();
        if (blockIdx.x == 0) {
            if (t < K) st->codebook[t] = p;
            if (t + 1 < K && !(s_val[t + 1] > s_val[t])) atomicOr(&st->flags, kFlagCollide);
            if (t == 0) {
                st->K = K;
                if (any_bad) atomicOr(&st->flags, kFlagNonFinite);
            }
        }
    } else {
        c.K = st->K;
        c.wmin = c.step = 0.f;
        for (uint32_t i = t; i < kHashSlots; i += 256) s_hkey[i] = kHashFree;
        __syncthreads();
        if (t < c.K) {
            const uint32_t key = __float_as_uint(canonical(st->codebook[t]));
            uint32_t h = hash_slot(key);
            while (atomicCAS(&s_hkey[h], kHashFree, key) != kHashFree) h = (h + 1u) & (kHashSlots - 1u);
            s_hpos[h] = t;
        }
        __syncthreads();
    }
    c.top = (float)(c.K - 1);
    c.val = s_val;
    c.hkey = s_hkey;
    c.hpos = s_hpos;
    bool missing = false;
    unsigned long long total_t = 0;  // occurrences of codebook position t in this workgroup's rows
    uint32_t least_t = 0xFFFFFFFFu;  // ... in the row that has fewest
    for (int64_t r = blockIdx.x; r < rows; r += gridDim.x) {
        const float* row = W + r * row_len;
        uint8_t* crow = codes ? codes + r * row_len : nullptr;
        float* qrow = Wq ? Wq + r * row_len : nullptr;
        const int64_t n = min(row_len, total - r * row_len);  // the last row of a flat array may be short
        const bool any = kCopies > 1 || aligned;  // 16-byte pieces
        // the next round's four elements are requested before this round's are coded
        FourFloats ahead = {0.f, 0.f, 0.f, 0.f};
        if (any && 4 * (int64_t)t + 4 <= n) ahead = *reinterpret_cast<const FourFloats*>(row + 4 * (int64_t)t);
        for (int64_t j0 = 0; j0 < n; j0 += 1024) {
            const int64_t j = j0 + 4 * (int64_t)t;
            uint32_t code[4] = {0, 0, 0, 0};
            const int valid = (int)max((int64_t)0, min((int64_t)4, n - j));
            const FourFloats w = ahead;
            if (any && j + 1024 + 4 <= n) ahead = *reinterpret_cast<const FourFloats*>(row + j + 1024);
            if (valid == 4 && any) {
                code[0] = code_of<kQuant>(w.x, c, missing);
                code[1] = code_of<kQuant>(w.y, c, missing);
                code[2] = code_of<kQuant>(w.z, c, missing);
                code[3] = code_of<kQuant>(w.w, c, missing);
                if (crow) *reinterpret_cast<FourBytes*>(crow + j) = code[0] | (code[1] << 8) | (code[2] << 16) | (code[3] << 24);
                if (kQuant && qrow)
                    *reinterpret_cast<FourFloats*>(qrow + j) = FourFloats{s_val[code[0]], s_val[code[1]], s_val[code[2]], s_val[code[3]]};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (e < valid) {
                        code[e] = code_of<kQuant>(row[j + e], c, missing);
                        if (crow) crow[j + e] = (uint8_t)code[e];
                        if (kQuant && qrow) qrow[j + e] = s_val[code[e]];
                    }
                }
            }
            if (!cnt) continue;  // uniform
            // histogram: everything that equals the first active lane's first code is counted with one add
            const uint64_t act = __ballot(valid > 0);
            if (act) {
                const uint32_t lead = (uint32_t)__builtin_amdgcn_readfirstlane((int)code[0]);
                uint32_t same = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = e < valid;
                    same += (uint32_t)__popcll(__ballot(in && code[e] == lead));
                    if (in && code[e] != lead) atomicAdd(&copy[code[e]], 1u);
                }
                if ((uint32_t)__builtin_ctzll(act) == (t & 63u)) atomicAdd(&copy[lead], same);
            }
        }
        if (cnt) {
            __syncthreads();
            uint32_t sum = 0;
            if (kCopies == 1 || t < c.K) {
                uint32_t h[kCopies];
#pragma unroll
                for (uint32_t i = 0; i < kCopies; ++i) h[i] = s_hist[i][t];
#pragma unroll
                for (uint32_t i = 0; i < kCopies; ++i) {
                    sum += h[i];
                    s_hist[i][t] = 0;
                }
            }
            cnt[r * kCodes + t] = sum;
            total_t += sum;
            least_t = min(least_t, sum);
            __syncthreads();
        }
    }
    if (cnt && t < c.K) {
        const uint32_t at = (blockIdx.x & (kHistParts - 1)) * kCodes + t;
        if (total_t) atomicAdd(&hist[at], total_t);
        atomicMin(&least_of(hist)[at], least_t);
    }
    if (__syncthreads_or(missing) && t == 0) atomicOr(&st->flags, kFlagMissing);
}

// ------------------------------------------------------------------------------------------------
// layout: per row, the number of indexed elements, of groups and of non-empty groups.  One wave per kRows rows, sixteen waves per
// workgroup; every workgroup first ranks the values for itself, and the last one to finish scans the rows (two launches less
// than kernels of their own: 20 of the 70 us that a layer of 300 x 700 took went into such steps).
//
// Frequency-major order: higher count first, equal counts in codebook order; values that never occur are left out
// (Section III-A, step 1).  Each thread finds its own value's position by counting who comes before it.
//
// scan: exclusive prefix sums of the rows' groups and indexed elements (m + 1 entries {groups, elements}), the number of
// non-empty groups and the largest group count of a row; kScanRows consecutive rows per thread and round.
//
// One workgroup more has no rows: it tells the host what follows from the values' counts alone -- the number of indexed elements, of values, and the
// longest row's elements: all but the most frequent value's, of which codes_kernel leaves the least count (looked for here, in one count per row, it
// took 4 us of 4096 rows).
// ------------------------------------------------------------------------------------------------
constexpr int kScanRows = 4;

// Of a wave's lanes up to the own one: sums of 64 bits (cer::wave_inclusive_scan takes 32), and the largest.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long lanes_before(unsigned long long x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), CTRL, ROWS, 0xF, false);
    return (unsigned long long)hi << 32 | lo;
}
__device__ __forceinline__ unsigned long long wave_scan64(unsigned long long x) {
    x += lanes_before<0x111, 0xF>(x);  // row_shr:1, 2, 4, 8
    x += lanes_before<0x112, 0xF>(x);
    x += lanes_before<0x114, 0xF>(x);
    x += lanes_before<0x118, 0xF>(x);
    x += lanes_before<0x142, 0xA>(x);  // row_bcast:15 into rows 1 and 3
    x += lanes_before<0x143, 0xC>(x);  // row_bcast:31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ uint32_t wave_largest(uint32_t x) {  // in the last lane
#define CER_MAX_STEP(CTRL, ROWS) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false));
    CER_MAX_STEP(0x111, 0xF)
    CER_MAX_STEP(0x112, 0xF)
    CER_MAX_STEP(0x114, 0xF)
    CER_MAX_STEP(0x118, 0xF)
    CER_MAX_STEP(0x142, 0xA)
    CER_MAX_STEP(0x143, 0xC)
#undef CER_MAX_STEP
    return x;
}

__device__ void scan_rows(const unsigned long long* rowGN, int64_t m, uint2* __restrict__ rowStart, FrontState* __restrict__ st,
                          FrontResult* __restrict__ out) {
    __shared__ unsigned long long s_g[16], s_n[16], s_p[16];
    __shared__ uint32_t s_mx[16];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    unsigned long long carry_g = 0, carry_n = 0, my_p = 0;
    uint32_t my_mx = 0;
    const uint32_t flags = st->flags;  // on its way with the first rows
    for (int64_t base = 0; base < m; base += 1024 * kScanRows) {
        const int64_t r0 = base + (int64_t)t * kScanRows;
        uint2 v[kScanRows];
        unsigned long long g = 0, nn = 0;
#pragma unroll
        for (int k = 0; k < kScanRows; ++k) {
            const unsigned long long q = r0 + k < m ? rowGN[r0 + k] : 0ull;
            v[k] = make_uint2((uint32_t)q, (uint32_t)(q >> 32));
        }
#pragma unroll
        for (int k = 0; k < kScanRows; ++k) {
            my_p += v[k].x >> 16;
            v[k].x &= 0xFFFFu;
            my_mx = max(my_mx, v[k].x);
            g += v[k].x;
            nn += v[k].y;
        }
        const unsigned long long ig = wave_scan64(g), in_ = wave_scan64(nn);  // inside the wave
        if (lane == 63) {
            s_g[wave] = ig;
            s_n[wave] = in_;
        }
        __syncthreads();
        unsigned long long og = carry_g, on = carry_n;
        for (uint32_t w = 0; w < 16; ++w) {
            if (w < wave) {
                og += s_g[w];
                on += s_n[w];
            }
            carry_g += s_g[w];
            carry_n += s_n[w];
        }
        og += ig - g;
        on += in_ - nn;
#pragma unroll
        for (int k = 0; k < kScanRows; ++k) {
            if (r0 + k < m) rowStart[r0 + k] = make_uint2((uint32_t)og, (uint32_t)on);
            og += v[k].x;
            on += v[k].y;
        }
        __syncthreads();
    }
    my_p = wave_scan64(my_p);
    my_mx = wave_largest(my_mx);
    if (lane == 63) {
        s_p[wave] = my_p;
        s_mx[wave] = my_mx;
    }
    __syncthreads();
    if (t == 0) {
        unsigned long long p = 0;
        uint32_t mx = 0;
        for (int w = 0; w < 16; ++w) {
            p += s_p[w];
            mx = max(mx, s_mx[w]);
        }
        rowStart[m] = make_uint2((uint32_t)carry_g, (uint32_t)carry_n);
        // the product kernels address colI and OmegaPtr with 32-bit offsets and read ahead of a row's end
        const unsigned long long limit = 0xFFFFFFFFull - 65536;
        tell(&out->totals[0], carry_g);
        tell(&out->totals[1], p);
        tell(&out->totals[2], mx | (unsigned long long)(flags | (carry_g > limit || carry_n > limit ? kFlagTooLarge : 0u)) << 50);
    }
}

// Bound by a chain of steps (values ranked, the arrivals, the scan), of which only the arrivals grow with the workgroups (4096 rows 15.2 us
// with 256 workgroups, 10.8 with 64; 300 rows 8.6): beyond kFewRows
// rows a wave takes four (the call for 4096 x 9216, 7 bits, with one / two / four / eight rows per wave 187.0 / 185.5 / 184.5 / 185.0 us; 188.3
// when one row per wave went with shuffles in place of DPP), below one: 2000 x 5000, 8 bits, 110.3 / 110.4 / 110.3 / 111.8, 1024 x 2048, 5 bits, 65.9 /
// 66.2 / 66.7 / 68.6.
constexpr int64_t kFewRows = 2048;
template <int kRows>
__global__ __launch_bounds__(1024) void row_layout_kernel(const uint32_t* __restrict__ cnt, const unsigned long long* __restrict__ hist,
                                                          int64_t m, int64_t n, int cser, FrontState* __restrict__ st, unsigned long long* __restrict__ rowGN,
                                                          uint2* __restrict__ rowStart, FrontResult* __restrict__ out) {
    __shared__ unsigned long long s_sum[4][kCodes];
    __shared__ unsigned long long s_h[kCodes];
    __shared__ uint32_t s_rank[kCodes];
    __shared__ uint32_t s_last;
    const uint32_t t = threadIdx.x, lane = t & 63u, pos = t & 255u, sub = t >> 8, K = st->K;
    const bool tells = blockIdx.x == gridDim.x - 1u;
    // the rows' histograms are on their way while the values are ranked
    const int64_t r0 = ((int64_t)blockIdx.x * 16 + (t >> 6)) * kRows;
    uint32_t c4[kRows][kCodes / kWave];
#pragma unroll
    for (int k = 0; k < kRows; ++k)
#pragma unroll
        for (int i = 0; i < kCodes / kWave; ++i) c4[k][i] = cnt[min(r0 + k, m - 1) * kCodes + lane + 64u * i];
    {
        unsigned long long s = 0;
#pragma unroll
        for (int i = 0; i < kHistParts / 4; ++i) s += hist[(sub + 4 * i) * kCodes + pos];
        s_sum[sub][pos] = s;
    }
    __syncthreads();
    // (count, then the earlier position): no two are equal, so that one comparison tells who comes first
    if (sub == 0) s_h[pos] = (pos < K ? s_sum[0][pos] + s_sum[1][pos] + s_sum[2][pos] + s_sum[3][pos] : 0ull) << 8 | (255u - pos);
    __syncthreads();
    // the four threads of a position compare it with a quarter of the others each
    const unsigned long long key = s_h[pos];
    {
        uint32_t before = 0;
        for (uint32_t j = sub * 64u; j < min(K, sub * 64u + 64u); j += 8u)  // (positions from K on have no count)
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i) before += s_h[j + i] > key ? 1u : 0u;
        s_sum[sub][pos] = before;
    }
    const int occurring = __syncthreads_count(sub == 0 && key >> 8 != 0ull);
    if (sub == 0) {
        const unsigned long long c = key >> 8;
        const uint32_t before = (uint32_t)(s_sum[0][pos] + s_sum[1][pos] + s_sum[2][pos] + s_sum[3][pos]);
        s_rank[pos] = c > 0 ? before : 0u;
        if (blockIdx.x == 0) {
            st->rank_of[pos] = c > 0 ? before : 0u;
            if (c > 0) {
                st->pos_of[before] = pos;
                st->omega[before] = canonical(st->codebook[pos]);
                st->count[before] = c;
            }
        }
    }
    if (blockIdx.x == 0 && t == 0) st->Kp = (uint32_t)occurring;
    if (tells) {
        if (sub == 0 && key >> 8 != 0ull && s_rank[pos] == 0u) {
            s_last = pos;
            s_h[0] = key >> 8;
        }
        __syncthreads();
        if (t < kWave) {
            const uint32_t* least = reinterpret_cast<const uint32_t*>(hist + kHistParts * kCodes) + (occurring ? s_last : 0u);
            const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)wave_largest(~least[(t & (kHistParts - 1)) * kCodes]), 63);
            if (t != 0) return;
            tell(&out->early[0], ((uint32_t)n - ~all) | (unsigned long long)K << 32 | (unsigned long long)(uint32_t)occurring << 41 | (unsigned long long)st->flags << 50);
            tell(&out->early[1], (unsigned long long)(m * n) - (occurring ? s_h[0] : 0ull));
        }
        return;
    }
    __syncthreads();
    uint32_t rank[kCodes / kWave];
#pragma unroll
    for (int i = 0; i < kCodes / kWave; ++i) rank[i] = s_rank[lane + 64u * i];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        uint32_t present = 0, topk = 0, nn = 0;
#pragma unroll
        for (int i = 0; i < kCodes / kWave; ++i)
            if (c4[k][i] > 0 && rank[i] >= 1) {
                ++present;
                topk = max(topk, rank[i]);
                nn += c4[k][i];
            }
        present = cer::wave_inclusive_scan(present);
        nn = cer::wave_inclusive_scan(nn);
        topk = wave_largest(topk);
        // groups (CER keeps the empty groups below the row's highest rank) | non-empty groups << 16, indexed elements
        if (lane == 63u && r0 + k < m) rowGN[r0 + k] = ((unsigned long long)nn << 32) | (cser ? present : topk) | (present << 16);
    }
    // The last workgroup to arrive scans the rows.  Thread 0 publishes what the workgroup's threads have written in front of the
    // barrier and takes what the others have: one release and one acquire per workgroup.  (Each release writes an L2 back: 4096
    // rows 16 -> 18 us against relaxed accesses past the caches, which nothing orders; a fence per wave took 80 us.)
    __syncthreads();
    if (t == 0) s_last = __hip_atomic_fetch_add(&st->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 2u ? 1u : 0u;
    __syncthreads();
    if (s_last) scan_rows(rowGN, m, rowStart, st, out);
}

// ------------------------------------------------------------------------------------------------
// emit: the row's pointers and its columns, grouped by rank.  One wave per row.
// ------------------------------------------------------------------------------------------------
// 64 consecutive columns: lanes with the same rank are found with one ballot per bit of the rank
// and take consecutive slots of that rank's bucket in lane (= column) order.
template <typename ColT>
__device__ __forceinline__ void scatter64(uint32_t k, int64_t j, uint32_t nbits, uint64_t below, uint32_t* fill,
                                          unsigned long long* marks, ColT* __restrict__ colI) {
    const bool act = k >= 1;
    uint64_t peers = __ballot(act);
    if (!peers) return;
    if (nbits > 3) {
        // many ranks: the lanes of a rank meet in that rank's 64-bit word in LDS (all words are zero between calls)
        if (act) atomicOr(&marks[k], below + 1ull);  // below = 2^lane - 1
        wave_lds_sync();
        if (act) peers = marks[k];
    } else {
        for (uint32_t b = 0; b < nbits; ++b) {
            const bool bit = (k >> b) & 1u;
            const uint64_t votes = __ballot(bit);
            peers &= bit ? votes : ~votes;
        }
    }
    if (act) {
        const uint32_t before = (uint32_t)__popcll(peers & below);
        const uint32_t slot = fill[k];
        colI[slot + before] = (ColT)j;
        if (before == 0) {
            fill[k] = slot + (uint32_t)__popcll(peers);
            if (nbits > 3) marks[k] = 0ull;
        }
    }
    wave_lds_sync();
}

constexpr uint32_t kEmitStage = 1024;  // staged entries per wave

// Where the parts of the handle's allocation start, and the gaps between them (cleared: the product reads ahead).
struct EmitTarget {
    unsigned char* base;
    size_t off_optr, off_rptr, off_ri, off_oi, off_om, off_tab;
    int32_t tab_shift;  // rank table: 1 << tab_shift words per row; 0: none
    int32_t ngaps;
    size_t gap_begin[8], gap_end[8];
    uint32_t gap_group[8];  // bytes per group that stand between begin and the gap
};

// What one workgroup of an emitter does besides the rows: Omega, the gaps, and the values for the host.
__device__ __forceinline__ void emit_values(const FrontState* __restrict__ st, const EmitTarget& to, uint32_t groups, FrontResult* __restrict__ out) {
    for (uint32_t t = threadIdx.x; t < kCodes; t += blockDim.x) {
        if (t < st->Kp) {
            const float w = st->omega[t];
            reinterpret_cast<float*>(to.base + to.off_om)[t] = w;
            out->omega[t] = w;
            out->count[t] = st->count[t];
        }
        if (t < st->K) out->codebook[t] = st->codebook[t];
    }
    for (int g = 0; g < to.ngaps; ++g) {
        // (behind the groups there may be room for more of them, which nobody reads but for the first bytes)
        const size_t begin = to.gap_begin[g] + (size_t)to.gap_group[g] * groups, end = to.gap_group[g] ? min(to.gap_end[g], begin + 512) : to.gap_end[g];
        for (size_t o = begin + threadIdx.x; o < end; o += blockDim.x) to.base[o] = 0;
    }
}

// What a wave needs to know of a row: where its groups and indices begin and end, and its values' counts by rank (64 i + lane).
struct RowHead {
    uint2 here, next;
    uint32_t size[kCodes / kWave];
};
// Codebook positions by rank, the same for every row.
__device__ __forceinline__ void load_places(const FrontState* __restrict__ st, uint32_t ranks, uint32_t (&place_of)[kCodes / kWave]) {
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (uint32_t i = 0; i < kCodes / kWave; ++i) place_of[i] = i * kWave < ranks ? st->pos_of[i * kWave + lane] & (kCodes - 1u) : 0u;
}
__device__ __forceinline__ RowHead load_head(int64_t r, const uint32_t* __restrict__ cnt, const uint2* __restrict__ rowStart, uint32_t ranks,
                                             const uint32_t (&place_of)[kCodes / kWave]) {
    RowHead h;
    h.here = rowStart[r];
    h.next = rowStart[r + 1];
#pragma unroll
    for (uint32_t i = 0; i < kCodes / kWave; ++i) h.size[i] = i * kWave < ranks ? cnt[r * kCodes + place_of[i]] : 0u;
    return h;
}

// One wave: everything of row r but its columns -- bucket sizes by rank -> bucket starts (exclusive scan over ranks 1, 2, ...), the
// pointers and the row's record of the rank table.  place(rank, codebook position, first colI position of the bucket).
template <typename OiT, typename Place>
__device__ __forceinline__ void emit_row_pointers(int64_t r, const RowHead& head, const uint32_t (&place_of)[kCodes / kWave], uint32_t Kp, uint32_t ranks,
                                                  int64_t m, int cser, const EmitTarget& to, Place place) {
    uint32_t* omegaPtr = reinterpret_cast<uint32_t*>(to.base + to.off_optr);
    uint32_t* rowPtr = reinterpret_cast<uint32_t*>(to.base + to.off_rptr);
    uint2* rowInfo = reinterpret_cast<uint2*>(to.base + to.off_ri);
    OiT* omegaI = reinterpret_cast<OiT*>(to.base + to.off_oi);
    uint32_t* tab = reinterpret_cast<uint32_t*>(to.base + to.off_tab);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t g0 = head.here.x, off0 = head.here.y;
    const uint32_t groups = head.next.x - g0;
    if (lane == 0) {
        rowPtr[r] = g0;
        rowInfo[r] = head.here;
        if (r == 0) omegaPtr[0] = 0;
        if (r == m - 1) {
            rowPtr[m] = head.next.x;
            rowInfo[m] = head.next;
        }
    }
    uint32_t carry = 0, gcarry = 0;
#pragma unroll
    for (uint32_t i = 0; i < kCodes / kWave; ++i) {
        if (i * kWave >= ranks) break;  // uniform
        const uint32_t k = i * kWave + lane, pos = place_of[i];
        const uint32_t c = (k >= 1 && k < Kp) ? head.size[i] : 0u;
        const uint32_t inc = cer::wave_inclusive_scan(c);
        const uint32_t end = off0 + carry + inc;
        place(k, pos, end - c);
        if (to.tab_shift && (k >> to.tab_shift) == 0) tab[((size_t)r << to.tab_shift) + k] = end;
        const uint64_t pres = __ballot(c > 0);
        if (cser) {
            if (c > 0) {
                const uint32_t idx = gcarry + (uint32_t)__popcll(pres & ((1ull << lane) - 1ull));
                omegaPtr[g0 + idx + 1] = end;
                omegaI[g0 + idx] = (OiT)k;
            }
            gcarry += (uint32_t)__popcll(pres);
        } else if (k >= 1 && k <= groups) {
            omegaPtr[g0 + k] = end;  // an empty group repeats the previous pointer
        }
        carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    }
}

// One row at a time per workgroup of one wave, whose columns are sorted in LDS; the last workgroup does emit_values.
// A lane takes a run of consecutive columns and has a counter of its own per codebook position (16 bits, two lanes to a word), so
// that counting and placing need neither a vote nor an order among the lanes: count the run's elements, turn the counters into
// first slots (a scan over the lanes per position, two positions at a time, on top of the bucket starts), then take the slots one
// after another and write the columns to their places in LDS.  The row goes to memory as it lies there, with 16-byte stores.
// As many workgroups as fit at once take the rows in turn: a row's codes, pointers and counts come while the row before is sorted.
// A row of 9216 columns and 128 positions takes 31 KiB, five of them on a compute unit: 56 us for 4096, against 69 with emit_kernel (60
// with a workgroup per row that loads its codes twice); 3400 clocks of LDS instructions per row (an add 5, a store to any place 6), twice
// that with five waves to hide their latency.  Where all rows run at once the gain is larger: 300 x 9000 115 -> 89 us.
constexpr uint32_t kRowCounters = 32;  // words of counters per codebook position
// 64 runs of a multiple of 16 columns: below 65536, so that slots fit 16 bits (the most frequent value's lie behind all others: a row has
// as many slots as columns).
constexpr int64_t kSortedColumns = 64512;
constexpr int kSortedPieces = 12;  // sixteens of columns per lane that stay in registers
inline uint32_t emit_stage_bytes(uint32_t longest) { return ((longest * 2u + 16u + 15u) & ~15u) + 256u; }

template <int kPieces>
__global__ __launch_bounds__(64) void emit_sorted_kernel(const uint8_t* __restrict__ codes, const uint32_t* __restrict__ cnt,
                                                         const uint2* __restrict__ rowStart, const FrontState* __restrict__ st,
                                                         int64_t m, uint32_t n, int cser, uint32_t positions, uint32_t stage_bytes,
                                                         EmitTarget to, FrontResult* __restrict__ out) {
    // LDS: [the row's columns][a word per lane for what is not indexed][counters: positions x kRowCounters][bucket start by position],
    // positions rounded up to eight
    extern __shared__ __align__(16) unsigned char s_row[];
    if (blockIdx.x == gridDim.x - 1) {
        emit_values(st, to, rowStart[m].x, out);
        return;
    }
    const uint32_t lane = threadIdx.x, eights = (positions + 7u) & ~7u;
    const uint32_t run = ((n + 63u) / 64u + 15u) & ~15u, c0 = lane * run, pieces = run / 16u;
    const uint32_t Kp = st->Kp, ranks = max(Kp, 1u << to.tab_shift), most = st->pos_of[0], blank = most * 0x01010101u;
    uint32_t place_of[kCodes / kWave];
    load_places(st, ranks, place_of);
    // Rows of up to 1024 kPieces columns stay in registers, loaded at once and while the row before is sorted; of longer ones four loads
    // are in flight (a trip to memory per sixteen columns took two thirds of the time).
    constexpr int kAhead = kPieces > 0 ? kPieces : 4;
    const uint32_t stride = gridDim.x - 1u;
    auto row_codes = [&](int64_t r) { return codes + min(r, m - 1) * (int64_t)n; };
    // (sixteen codes from a column in front of the row's end on: up to fifteen of the next row's)
    auto request = [&](const uint8_t* crow, uint32_t p, uint4& q) { __builtin_memcpy(&q, crow + min(c0 + 16u * min(p, pieces - 1u), n - 1u), 16); };
    auto request_first = [&](const uint8_t* crow, uint4 (&q)[kAhead]) {
#pragma unroll
        for (int d = 0; d < kAhead; ++d)
            if (kPieces == 0 || (uint32_t)d < pieces) request(crow, d, q[d]);
    };
    uint32_t* counters = reinterpret_cast<uint32_t*>(s_row + stage_bytes);
    uint32_t* begin = counters + eights * kRowCounters;
    typedef unsigned char __attribute__((address_space(3))) * LdsByte;
    typedef uint32_t __attribute__((address_space(3))) * LdsWord;
    typedef uint16_t __attribute__((address_space(3))) * LdsCol;
    const uint32_t mine = (uint32_t)(uintptr_t)(LdsByte)(unsigned char*)counters + (lane >> 1) * 4u;
    const uint32_t half = 16u * (lane & 1u), one = 1u << half;
    // the lane's counter of the i-th of four codes: one byte times the distance of the counters, a dot product of bytes
    static_assert(kRowCounters * 4u < 256u, "distance of the counters");
    auto counter = [&](uint32_t four, int i) {
        return reinterpret_cast<LdsWord>((uintptr_t)__builtin_amdgcn_udot4(four, (kRowCounters * 4u) << (8 * i), mine, false));
    };
    auto add = [&](LdsWord at) { return __hip_atomic_fetch_add(at, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    uint4 ring[kAhead], ahead[kAhead];
    RowHead head = load_head(min((int64_t)blockIdx.x, m - 1), cnt, rowStart, ranks, place_of);
    request_first(row_codes(blockIdx.x), ring);
    for (int64_t r = blockIdx.x; r < m; r += stride) {
        const uint8_t* crow = row_codes(r);
        uint32_t column0 = c0;
        asm volatile("" : "+v"(column0));  // (columns are counted from here for every row: hoisted, their numbers would take all registers)
        // f(first column, sixteen codes); behind the row's end stands the most frequent value, which takes no part
        auto each_sixteen = [&](auto f) {
            for (uint32_t p0 = 0; p0 < (kPieces > 0 ? 1u : pieces); p0 += kAhead) {
#pragma unroll
                for (int d = 0; d < kAhead; ++d) {
                    const uint32_t p = p0 + d, c = column0 + 16u * p;
                    if (p >= pieces) break;  // uniform
                    uint32_t q[4] = {ring[d].x, ring[d].y, ring[d].z, ring[d].w};
                    if (kPieces == 0) request(crow, p + kAhead, ring[d]);
                    if (__ballot(c + 16u > n) != 0ull) {
                        const int left = (int)n - (int)c;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int bytes = min(max(left - 4 * i, 0), 4);
                            const uint32_t keep = bytes == 4 ? 0xFFFFFFFFu : (1u << (8 * bytes)) - 1u;
                            q[i] = (q[i] & keep) | (blank & ~keep);
                        }
                    }
                    f(c, q);
                }
            }
        };
        for (uint32_t i = lane; i < eights * kRowCounters / 4u; i += kWave) reinterpret_cast<uint4*>(counters)[i] = make_uint4(0, 0, 0, 0);
        const uint32_t off0 = head.here.y, count = head.next.y - off0;
        for (uint32_t i = lane; i < eights; i += kWave) begin[i] = i == most ? count : 0u;  // the most frequent value: behind all others
        emit_row_pointers<uint8_t>(r, head, place_of, Kp, ranks, m, cser, to, [&](uint32_t k, uint32_t pos, uint32_t first) {
            if (k >= 1u && k < Kp) begin[pos] = first - off0;
        });
        wave_lds_sync();
        // the next row is on its way
        head = load_head(min(r + stride, m - 1), cnt, rowStart, ranks, place_of);
        if (kPieces > 0) request_first(row_codes(r + stride), ahead);
        each_sixteen([&](uint32_t, const uint32_t (&q)[4]) {
#pragma unroll
            for (int i = 0; i < 16; ++i) (void)add(counter(q[i >> 2], i & 3));
        });
        wave_lds_sync();
        if (kPieces == 0) request_first(crow, ring);
        // two positions per instruction, four instructions side by side, the next four on their way from LDS
        const uint32_t words = eights * kRowCounters;
        uint32_t word[4], start[4];
        auto read = [&](uint32_t i) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                word[u] = counters[i + u * kWave];
                start[u] = begin[(i + u * kWave) / kRowCounters];
            }
        };
        read(lane);
        for (uint32_t i = lane; i < words; i += 4u * kWave) {
            uint32_t incl[4], now[4], from[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                now[u] = word[u];
                from[u] = start[u];
                incl[u] = (word[u] & 0xFFFFu) + (word[u] >> 16);
            }
            read(i + 4u * kWave < words ? i + 4u * kWave : i);
#define CER_HALF_SCAN(CTRL, ROWS) \
    _Pragma("unroll") for (int u = 0; u < 4; ++u) incl[u] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl[u], CTRL, ROWS, 0xF, false);
            CER_HALF_SCAN(0x111, 0xF)  // row_shr:1, 2, 4, 8
            CER_HALF_SCAN(0x112, 0xF)
            CER_HALF_SCAN(0x114, 0xF)
            CER_HALF_SCAN(0x118, 0xF)
            CER_HALF_SCAN(0x142, 0xA)  // row_bcast:15 into rows 1 and 3
#undef CER_HALF_SCAN
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t lo = now[u] & 0xFFFFu, first = from[u] + incl[u] - lo - (now[u] >> 16);
                counters[i + u * kWave] = first | ((first + lo) << 16);
            }
        }
        wave_lds_sync();
        // the row lies in LDS as far from a multiple of 16 bytes as in memory
        uint16_t* colI = reinterpret_cast<uint16_t*>(to.base) + off0;
        constexpr uint32_t kPer = 8;
        const uint32_t shift = off0 & (kPer - 1u);
        uint16_t* stage = reinterpret_cast<uint16_t*>(s_row) + shift;
        const uint32_t stage_at = (uint32_t)(uintptr_t)(LdsByte)(unsigned char*)stage;
        const uint32_t aside = (uint32_t)(uintptr_t)(LdsByte)s_row + stage_bytes - 256u + lane * 4u;
        each_sixteen([&](uint32_t c, const uint32_t (&q)[4]) {
            uint32_t old[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) old[i] = add(counter(q[i >> 2], i & 3));
#pragma unroll
            for (uint32_t i = 0; i < 16; ++i)
                *reinterpret_cast<LdsCol>((uintptr_t)min(stage_at + ((old[i] >> half) & 0xFFFFu) * 2u, aside)) = (uint16_t)(c | i);
        });
        wave_lds_sync();
        const uint32_t total = shift + count;  // in units of columns, from the 16-byte boundary before the row on
        // whole pieces of 16 bytes, four on their way at a time; what lies in front of the first and behind the last one singly
        const uint32_t v0 = shift != 0u ? 1u : 0u, v1 = total / kPer;
        for (uint32_t v = v0 + lane; v < v1; v += 4u * kWave) {
            uint4 q[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) q[u] = reinterpret_cast<const uint4*>(s_row)[min(v + u * kWave, v1 - 1u)];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u)
                if (v + u * kWave < v1) reinterpret_cast<uint4*>(colI - shift)[v + u * kWave] = q[u];
        }
        const uint32_t head_end = v0 <= v1 ? v0 * kPer : total, tail = max(v0, v1) * kPer;
        if (lane >= shift && lane < min(head_end, total)) colI[lane - shift] = stage[lane - shift];
        if (v0 <= v1 && tail + lane < total) colI[tail + lane - shift] = stage[tail + lane - shift];
        wave_lds_sync();
        if constexpr (kPieces > 0) {
#pragma unroll
            for (int d = 0; d < kAhead; ++d) ring[d] = ahead[d];
        } else {
            request_first(row_codes(r + stride), ring);
        }
    }
}

// Four rows per workgroup; the last workgroup does emit_values.
template <typename ColT, typename OiT>
__global__ __launch_bounds__(256) void emit_kernel(const uint8_t* __restrict__ codes, const uint32_t* __restrict__ cnt,
                                                   const uint2* __restrict__ rowStart, const FrontState* __restrict__ st,
                                                   int64_t m, int64_t n, int cser, int sparse, EmitTarget to,
                                                   FrontResult* __restrict__ out) {
    __shared__ uint32_t s_rank[kCodes];
    __shared__ uint32_t s_fill[4][kCodes];  // next free colI slot of each rank's bucket
    __shared__ uint32_t s_stage[4][kEmitStage];  // (column << 8) | rank of the columns waiting for the scatter
    __shared__ unsigned long long s_marks[4][kCodes];  // per rank: the lanes of the current batch that hold it
    if (blockIdx.x == gridDim.x - 1) {
        emit_values(st, to, rowStart[m].x, out);
        return;
    }
    ColT* colI = reinterpret_cast<ColT*>(to.base);
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    s_rank[threadIdx.x] = st->rank_of[threadIdx.x];
#pragma unroll
    for (int w = 0; w < 4; ++w) s_marks[w][threadIdx.x] = 0ull;
    __syncthreads();
    const int64_t r = (int64_t)blockIdx.x * 4 + wave;
    if (r >= m) return;
    uint32_t* fill = s_fill[wave];
    unsigned long long* marks = s_marks[wave];
    const uint32_t Kp = st->Kp;
    const uint32_t ranks = max(Kp, 1u << to.tab_shift);
    uint32_t place_of[kCodes / kWave];
    load_places(st, ranks, place_of);
    emit_row_pointers<OiT>(r, load_head(r, cnt, rowStart, ranks, place_of), place_of, Kp, ranks, m, cser, to,
                           [&](uint32_t k, uint32_t, uint32_t first) { fill[k] = first; });
    wave_lds_sync();
    // stable scatter of the row's columns into the buckets
    const uint32_t nbits = 32u - (uint32_t)__builtin_clz(Kp > 1 ? Kp - 1 : 1u);
    const uint64_t below = (1ull << lane) - 1ull;
    const uint8_t* crow = codes + r * n;
    if (sparse && (n & 3) == 0 && (reinterpret_cast<uintptr_t>(codes) & 3u) == 0 && n <= (int64_t)1 << 24) {
        // 256 columns per round: each lane loads the codes of four consecutive columns at once (the
        // next round's are requested before this round's are used).  Most columns hold the most
        // frequent value and take no part in the scatter: the others are first packed, in column order,
        // as (column, rank) into a buffer in LDS -- four ballots per 256 columns -- and the scatter with
        // its ballot per rank bit then runs over full batches of 64 buffered entries.
        uint32_t* buf = s_stage[wave];
        uint32_t held = 0;  // wave-uniform
        auto drain = [&](uint32_t keep_below) {
            // scatters buffered entries in batches of 64 until fewer than keep_below remain
            uint32_t done = 0;
            while (held - done >= keep_below && held > done) {
                const uint32_t i = done + lane;
                const uint32_t e = i < held ? buf[i] : 0u;
                scatter64<ColT>(e & 0xFFu, (int64_t)(e >> 8), nbits, below, fill, marks, colI);
                done += kWave;
            }
            if (done >= held) {
                held = 0;
            } else {
                // fewer than 64 left: move them to the front
                const uint32_t rest = held - done;
                const uint32_t e = lane < rest ? buf[done + lane] : 0u;
                wave_lds_sync();
                if (lane < rest) buf[lane] = e;
                wave_lds_sync();
                held = rest;
            }
        };
        const uint32_t* crow4 = reinterpret_cast<const uint32_t*>(crow);
        const int64_t n4 = n >> 2;
        // the code words of four rounds are in flight: a round is short against the memory latency
        constexpr int kAhead = 4;
        uint32_t ring[kAhead];
#pragma unroll
        for (int d = 0; d < kAhead; ++d) ring[d] = 64 * d + lane < n4 ? crow4[64 * d + lane] : 0u;
        for (int64_t jb = 0; jb < n; jb += 256 * kAhead) {
#pragma unroll
            for (int d = 0; d < kAhead; ++d) {
                const int64_t j0 = jb + 256 * d;  // may lie beyond the row: then no lane is inside
                const uint32_t cur = ring[d];
                const int64_t q = ((j0 + 256 * kAhead) >> 2) + lane;
                ring[d] = q < n4 ? crow4[q] : 0u;
                // this lane's four columns are consecutive, so lane order is column order
                const uint32_t c0 = (uint32_t)j0 + 4u * lane;
                const bool inside = j0 + 4 * (int64_t)lane < n;
                uint32_t k[4];
                uint32_t pos = held, total = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    k[i] = inside ? s_rank[(cur >> (8 * i)) & 0xFFu] : 0u;
                    const uint64_t some = __ballot(k[i] >= 1);
                    pos += (uint32_t)__popcll(some & below);
                    total += (uint32_t)__popcll(some);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (k[i] >= 1) buf[pos++] = ((c0 + (uint32_t)i) << 8) | k[i];
                }
                held += total;
                if (held > kEmitStage - 256) {
                    wave_lds_sync();
                    drain(kWave);
                }
            }
        }
        wave_lds_sync();
        drain(1);
    } else if ((n & 3) == 0 && (reinterpret_cast<uintptr_t>(codes) & 3u) == 0) {
        // as above without the buffer (most columns take part): a shuffle hands every lane the code of its own
        // column, 64 consecutive columns per scatter
        const uint32_t* crow4 = reinterpret_cast<const uint32_t*>(crow);
        const int64_t n4 = n >> 2;
        constexpr int kAhead = 4;
        uint32_t ring[kAhead];
#pragma unroll
        for (int d = 0; d < kAhead; ++d) ring[d] = 64 * d + lane < n4 ? crow4[64 * d + lane] : 0u;
        for (int64_t jb = 0; jb < n; jb += 256 * kAhead) {
#pragma unroll
            for (int d = 0; d < kAhead; ++d) {
                const int64_t j0 = jb + 256 * d;
                const uint32_t cur = ring[d];
                const int64_t q = ((j0 + 256 * kAhead) >> 2) + lane;
                ring[d] = q < n4 ? crow4[q] : 0u;
                if (j0 >= n) break;  // uniform
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int64_t j = j0 + 64 * s + lane;
                    const uint32_t v = (uint32_t)__shfl((int)cur, 16 * s + (int)(lane >> 2), kWave);
                    const uint32_t code = (v >> (8u * (lane & 3u))) & 0xFFu;
                    scatter64<ColT>(j < n ? s_rank[code] : 0u, j, nbits, below, fill, marks, colI);
                }
            }
        }
    } else {
        for (int64_t j0 = 0; j0 < n; j0 += kWave) {
            const int64_t j = j0 + lane;
            scatter64<ColT>(j < n ? s_rank[crow[j]] : 0u, j, nbits, below, fill, marks, colI);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// decode: format arrays -> dense matrix (Section III-A: M is reconstructed uniquely), as fp32 or as bf16 pieces for the
// matrix cores.  One workgroup per (row, every gridDim.y-th segment of its columns).  A segment is assembled in LDS as one
// byte per column, the element's rank (codebooks of more than 256 values: as its value), and written out with 16-byte
// stores, so that HBM sees every line of the output once.  A thread takes eight consecutive positions of colI per step with
// one load (the next step's is in flight), finds the group of the first one by a binary search in the row's pointers
// (kThreads groups at a time in LDS; repeated pointers, CER's empty groups, fall to the last of them) and walks on from
// there.  A row with several segments is read once per segment.
// Bound by the bytes written and the indices read: 4096 x 9216, 75 % indexed, 83 -> 33 us (one position per thread and
// search, values of a segment in LDS as fp32, before).
// ------------------------------------------------------------------------------------------------
struct DecodeArgs {
    const uint32_t* omegaPtr;
    const uint32_t* rowPtr;
    const uint8_t* omegaI;
    const float* omega;
    int oi_bits, cser;
    uint32_t K;
    int64_t n;
    uint32_t seg, nseg;  // columns per segment: a multiple of 8
    const uint32_t* tab;  // rank table
    uint32_t tab_shift;
    uint32_t rows;        // decode_tiles_kernel: rows per workgroup, 8, 4 or 2
    cer::UniformGrid grid;  // ... and the grid of the values
};

__device__ __forceinline__ void load_eight(const uint8_t* p, uint32_t v[8]) {
    const uint2 q = *reinterpret_cast<const uint2*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = (q.x >> (8 * i)) & 0xFFu;
        v[4 + i] = (q.y >> (8 * i)) & 0xFFu;
    }
}
__device__ __forceinline__ void load_eight(const uint16_t* p, uint32_t v[8]) {
    const uint4 q = *reinterpret_cast<const uint4*>(p);
    v[0] = q.x & 0xFFFFu; v[1] = q.x >> 16; v[2] = q.y & 0xFFFFu; v[3] = q.y >> 16;
    v[4] = q.z & 0xFFFFu; v[5] = q.z >> 16; v[6] = q.w & 0xFFFFu; v[7] = q.w >> 16;
}
__device__ __forceinline__ void load_eight(const uint32_t* p, uint32_t v[8]) {
    const uint4 a = reinterpret_cast<const uint4*>(p)[0], b = reinterpret_cast<const uint4*>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// Ranks (CodeT = uint8_t) or values (float) of columns c0 .. c0 + len - 1 of row r -> code, by T threads: a workgroup, or
// (kWave) one wave of it with its own LDS.  Only indexed elements are written.
template <bool kWave>
__device__ __forceinline__ void team_sync() {
    if constexpr (kWave) wave_lds_sync(); else __syncthreads();
}
template <typename ColT, typename CodeT, uint32_t T, bool kWave>
__device__ __forceinline__ void scatter_row(const ColT* __restrict__ colI, const DecodeArgs& a, uint32_t g0, uint32_t g1, uint32_t tid,
                                            int64_t c0, uint32_t len, uint32_t* s_ptr /* T + 1 */, CodeT* s_grp /* T */, CodeT* code) {
    for (uint32_t gb = g0; gb < g1; gb += T) {
        // pointers and ranks (values) of the groups gb .. gb + cnt - 1 of this row -> LDS
        const uint32_t cnt = min(g1 - gb, T);
        team_sync<kWave>();
        if (tid < cnt) {
            const uint32_t g = gb + tid;
            uint32_t rank = g - g0 + 1u;  // Algorithm 3: position in the row; Algorithm 4: OmegaI
            if (a.cser) {
                rank = a.oi_bits == 8 ? a.omegaI[g]
                                      : (a.oi_bits == 16 ? reinterpret_cast<const uint16_t*>(a.omegaI)[g]
                                                         : reinterpret_cast<const uint32_t*>(a.omegaI)[g]);
            }
            s_ptr[tid] = a.omegaPtr[g];
            if constexpr (sizeof(CodeT) == 1) s_grp[tid] = (uint8_t)rank; else s_grp[tid] = a.omega[rank];
        }
        if (tid == 0) s_ptr[cnt] = a.omegaPtr[gb + cnt];
        team_sync<kWave>();
        const uint32_t pb = s_ptr[0], pe = s_ptr[cnt];
        uint32_t lo = 0;
        uint32_t v = (pb & ~7u) + tid * 8u;
        uint32_t ahead[8];
        if (v < pe) load_eight(colI + v, ahead);  // up to seven positions on either side belong to others
        for (; v < pe; v += T * 8u) {
            uint32_t col[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) col[i] = ahead[i];
            if (v + T * 8u < pe) load_eight(colI + v + T * 8u, ahead);
            const uint32_t first = max(v, pb);
            uint32_t hi = cnt;  // s_ptr[lo] <= first < s_ptr[hi]
            while (hi - lo > 1u) {
                const uint32_t mid = (lo + hi) >> 1;
                if (s_ptr[mid] <= first) lo = mid; else hi = mid;
            }
            uint32_t end = s_ptr[lo + 1u];
            CodeT c = s_grp[lo];
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i) {
                const uint32_t p = v + i;
                if (p >= pb && p < pe) {
                    if (p >= end) {
                        do end = s_ptr[++lo + 1u]; while (end <= p);
                        c = s_grp[lo];
                    }
                    const uint64_t rel = (uint64_t)col[i] - (uint64_t)c0;  // huge when left of the segment
                    if (rel < len) code[rel] = c;
                }
            }
        }
    }
}

typedef uint32_t Words4 __attribute__((ext_vector_type(4), aligned(4)));  // (the memory path takes them at any such address)

// fp32 output.  kPast: large outputs go past the caches (kPastCaches), where nothing puts the halves of a line together: the stores begin at
// whole lines (4096 x 12300 49 -> 40 us, 4096 x 10250, 3 bits, 42 -> 33; rows of whole lines take the same either way).
template <typename ColT, typename CodeT, uint32_t kThreads, bool kPast>
__global__ __launch_bounds__(kThreads) void decode_kernel(const ColT* __restrict__ colI, DecodeArgs a, float* __restrict__ out) {
    constexpr bool kRanks = sizeof(CodeT) == 1;
    constexpr uint32_t T = kThreads;
    extern __shared__ __align__(16) unsigned char s_seg[];  // seg codes
    __shared__ uint32_t s_ptr[T + 1];
    __shared__ CodeT s_grp[T];
    __shared__ uint32_t s_val[kRanks ? kCodes : 1];  // fp32 value by rank
    constexpr bool kLines = kRanks && kPast;
    const uint32_t tid = threadIdx.x;
    const int64_t r = blockIdx.x;
    const uint32_t g0 = a.rowPtr[r], g1 = a.rowPtr[r + 1];
    if constexpr (kRanks)
        for (uint32_t k = tid; k < a.K; k += T) s_val[k] = __float_as_uint(a.omega[k]);
    const float w0 = kRanks ? 0.f : a.omega[0];

    for (uint32_t si = blockIdx.y; si < a.nseg; si += gridDim.y) {  // uniform over the workgroup
        const int64_t c0 = (int64_t)si * a.seg;
        const uint32_t len = (uint32_t)min((int64_t)a.seg, a.n - c0);  // 1 .. seg
        float* o = out + r * a.n + c0;
        // columns in front of the first whole line, and as many bytes in front of their codes that the others begin at a word
        const uint32_t front = kLines ? min(len, (uint32_t)(-(reinterpret_cast<uintptr_t>(o) >> 2)) & 31u) : 0u, pad = (0u - front) & 3u;
        CodeT* code = reinterpret_cast<CodeT*>(s_seg) + pad;
        if constexpr (kRanks) {
            for (uint32_t j = tid; j < (len + pad + 15u) / 16u; j += T) reinterpret_cast<uint4*>(s_seg)[j] = make_uint4(0, 0, 0, 0);
        } else {
            for (uint32_t j = tid; j < (len + 3u) / 4u; j += T) reinterpret_cast<float4*>(s_seg)[j] = make_float4(w0, w0, w0, w0);
        }
        scatter_row<ColT, CodeT, T, false>(colI, a, g0, g1, tid, c0, len, s_ptr, s_grp, code);
        __syncthreads();
        if constexpr (kRanks) {
            const uint32_t n4 = (len - front) >> 2;
            const uint32_t* words = reinterpret_cast<const uint32_t*>(s_seg + front + pad);
            if (kLines && tid < front) o[tid] = __uint_as_float(s_val[code[tid]]);
            for (uint32_t j = tid; j < n4; j += T) {
                const uint32_t q = words[j];
                const Words4 v = {s_val[q & 0xFFu], s_val[(q >> 8) & 0xFFu], s_val[(q >> 16) & 0xFFu], s_val[q >> 24]};
                if constexpr (kPast) __builtin_nontemporal_store(v, reinterpret_cast<Words4*>(o + front) + j);
                else reinterpret_cast<Words4*>(o)[j] = v;
            }
            for (uint32_t j = front + (n4 << 2) + tid; j < len; j += T) o[j] = __uint_as_float(s_val[code[j]]);
        } else {
            const uint32_t n4 = (reinterpret_cast<uintptr_t>(o) & 15u) == 0 ? len >> 2 : 0u;
            for (uint32_t j = tid; j < n4; j += T) reinterpret_cast<float4*>(o)[j] = reinterpret_cast<const float4*>(s_seg)[j];
            for (uint32_t j = (n4 << 2) + tid; j < len; j += T) o[j] = (float)code[j];
        }
        __syncthreads();  // the segment has been read before the next one is filled
    }
}

// bf16 pieces (kPieces 0: ranks, a byte each, see decode_ranks) in the operand order of v_mfma_f32_32x32x16_bf16: tiles of 32 rows x 16 columns, 1 KiB each, [row / 32]
// [column / 16][column / 8 % 2][row % 32][column % 8], rows padded with zeros to a multiple of 32 columns (pitch).  Eight
// rows per workgroup, so that a store of the workgroup covers whole 128-byte lines; four where eight would leave compute
// units without work (reading the rows' indices is what takes time, and segments do not divide it).
// Ranks: the rows' records of the rank table come with one load, and their positions -- consecutive in colI -- are
// dealt to all T threads, eight at a time, two vectors in flight.  A position's group is the number of groups that begin at or
// before it: a bitmap of the beginnings, counted up per word, as in the batch-1 kernel -- no search, no branch (a binary search
// and a walk over the boundaries waited for LDS at every step: 633 x 5106, 112 values, 22 us, now 11; 986 x 16765, three
// values, 42 against 28).  Bound by the phases of a workgroup -- records, list, bitmap, positions, output -- that follow one another
// (512 x 4608, 128 workgroups, 6.7 us: vector ALU busy 16 % of the launch, LDS 9 %, a wave waits for data or at a barrier 60 %).  So the first
// positions are requested as soon as the records tell where they are, the pieces of the values are made and the bitmap is filled
// beside the list meanwhile, and the counts are summed by lane moves: 0.4 to 0.8 us of 5.6 to 11.3, 0.985 of the call in the geometric mean of
// 50 products (2067 x 521, batch 1638, 38.7 -> 37.3 us).  Eight rows in more segments instead of four rows: 1.03 times the call; four rows in more
// segments 1.01; two rows 1.005 (rows of up to 6144 columns).  Stores past the L2 (what a launch leaves there is written back behind it): 0.97 with eight rows and up to
// 16 MB, but 1.02 - 1.06 with four rows or larger matrices.
constexpr uint32_t kStretch = 32768;  // positions per bitmap
template <typename ColT, typename CodeT, int kPieces, uint32_t T>
__global__ __launch_bounds__(T) void decode_tiles_kernel(const ColT* __restrict__ colI, DecodeArgs a, int64_t m, int64_t pitch,
                                                         int64_t plane, uint16_t* __restrict__ out) {
    constexpr bool kRanks = sizeof(CodeT) == 1;
    constexpr uint32_t kPer = kStretch / 32 / T;  // words of the bitmap per thread
    extern __shared__ __align__(16) unsigned char s_seg[];  // eight rows of seg + 8 codes
    __shared__ uint32_t s_ptr[kRanks ? 8 * kCodes : 8 * (kWave + 1)];
    __shared__ uint32_t s_list[kRanks ? 8 * kCodes + 1 : 1];
    __shared__ uint32_t s_bits[kRanks ? kStretch / 32 : 1], s_pre[kRanks ? kStretch / 32 : 1];
    __shared__ uint32_t s_cnt[T / kWave], s_sum[T / kWave];
    __shared__ CodeT s_grp[8][kRanks ? 1 : kWave];
    __shared__ uint32_t s_val[kRanks && kPieces > 0 ? kCodes : 1];  // pieces 0 | 1 << 16, by rank
    __shared__ uint32_t s_val2[kRanks && kPieces == 3 ? kCodes : 1];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * a.rows;
    const int64_t c0 = (int64_t)blockIdx.y * a.seg;
    const uint32_t len = (uint32_t)min((int64_t)a.seg, a.n - c0);
    const uint32_t stride = a.seg + 8u;
    CodeT* code = reinterpret_cast<CodeT*>(s_seg);
    if constexpr (kRanks) {
        const uint32_t rows = (uint32_t)min((int64_t)a.rows, m - row0), words = rows << a.tab_shift;
        const float own = kPieces > 0 ? a.omega[min(tid, a.K - 1u)] : 0.f;  // (at most 256 values)
        for (uint32_t i = tid; i < words; i += T) s_ptr[i] = a.tab[((size_t)row0 << a.tab_shift) + i];
        for (uint32_t j = tid; j < a.rows * stride >> 3; j += T) reinterpret_cast<uint2*>(s_seg)[j] = make_uint2(0, 0);
        for (uint32_t i = 0; i < kPer; ++i) s_bits[kPer * tid + i] = 0u;
        __syncthreads();
        // the first positions are on their way while what tells their groups is made
        const uint32_t pb = s_ptr[0], pe = s_ptr[words - 1u];
        uint32_t ahead[2][8];
        auto request = [&](uint32_t v, uint32_t stop, uint32_t (&to)[8]) {
            if (v < stop) load_eight(colI + v, to);  // up to seven positions on either side of the rows belong to others
        };
        const uint32_t first = pb & ~7u;
        request(first + tid * 8u, min(pe, first + kStretch), ahead[0]);
        request(first + tid * 8u + 8u * T, min(pe, first + kStretch), ahead[1]);
        if constexpr (kPieces > 0)
            if (tid < a.K) {
                if (kPieces == 2 && a.grid.scale != 0.f) {
                    s_val[tid] = cer::uniform_pieces(own, a.grid);
                } else {
                    uint32_t p[3];
                    cer::split3_finite(own, p);
                    s_val[tid] = p[0] | (p[1] << 16);
                    if constexpr (kPieces == 3) s_val2[tid] = p[2];
                }
            }
        // list of the non-empty groups, in order of their positions: the row's place in s_seg | rank << 24; entry 0 is unused; and a bitmap of
        // the positions that begin a group, of the first stretch of positions
        auto begins = [&](uint32_t i, uint32_t& at) {  // boundary i closes a group that begins at position `at`
            if (i == 0 || i >= words) return false;
            at = s_ptr[i - 1u];
            return s_ptr[i] > at;
        };
        auto mark = [&](uint32_t at, uint32_t base) {
            if (at - base < kStretch) atomicOr(&s_bits[(at - base) >> 5], 1u << ((at - base) & 31u));
        };
        uint32_t groups = 1;
        for (uint32_t c = 0; c < words; c += T) {
            uint32_t at;
            const uint32_t i = c + tid;
            const bool some = begins(i, at);
            if (some) mark(at, first);
            const uint64_t votes = __ballot(some);
            if (lane == 0) s_cnt[wave] = (uint32_t)__popcll(votes);
            __syncthreads();
            uint32_t pos = groups + (uint32_t)__popcll(votes & ((1ull << lane) - 1ull));
            for (uint32_t w = 0; w < T / kWave; ++w) {
                if (w < wave) pos += s_cnt[w];
                groups += s_cnt[w];
            }
            if (some) s_list[pos] = (i >> a.tab_shift) * stride | ((i & ((1u << a.tab_shift) - 1u)) << 24);
            if (c + T < words) __syncthreads();  // (uniform)
        }
        uint32_t seen = 0;  // groups that begin before the current stretch of positions
        for (uint32_t base = first; base < pe; base += kStretch) {  // uniform over the workgroup
            if (base != first) {
                request(base + tid * 8u, min(pe, base + kStretch), ahead[0]);
                request(base + tid * 8u + 8u * T, min(pe, base + kStretch), ahead[1]);
                for (uint32_t i = 0; i < kPer; ++i) s_bits[kPer * tid + i] = 0u;
                __syncthreads();
                for (uint32_t i = tid; i < words; i += T) {
                    uint32_t at;
                    if (begins(i, at)) mark(at, base);
                }
                __syncthreads();
            }
            // the number of beginnings in front of every word
            uint32_t ones[kPer], all = 0;
#pragma unroll
            for (uint32_t i = 0; i < kPer; ++i) all += ones[i] = (uint32_t)__builtin_popcount(s_bits[kPer * tid + i]);
            const uint32_t incl = cer::wave_inclusive_scan(all);
            if (lane == 63u) s_sum[wave] = incl;
            __syncthreads();
            uint32_t before = seen + incl - all;
            for (uint32_t w = 0; w < T / kWave; ++w) {
                if (w < wave) before += s_sum[w];
                seen += s_sum[w];
            }
#pragma unroll
            for (uint32_t i = 0; i < kPer; ++i) {
                s_pre[kPer * tid + i] = before;
                before += ones[i];
            }
            __syncthreads();
            auto take = [&](uint32_t v, const uint32_t (&col)[8]) {
                const uint32_t rel0 = v - base, word = s_bits[rel0 >> 5], sh = rel0 & 31u;
                uint32_t g = s_pre[rel0 >> 5] + (uint32_t)__builtin_popcount(word & ((1u << sh) - 1u));
                uint32_t e[8];
#pragma unroll
                for (uint32_t i = 0; i < 8; ++i) {
                    g += (word >> (sh + i)) & 1u;
                    e[i] = s_list[g];
                }
#pragma unroll
                for (uint32_t i = 0; i < 8; ++i) {
                    const uint32_t rel = col[i] - (uint32_t)c0;  // huge when left of the segment
                    if (v + i >= pb && v + i < pe && rel < len) code[(e[i] & 0xFFFFFFu) + rel] = (CodeT)(e[i] >> 24);
                }
            };
            const uint32_t stop = min(pe, base + kStretch);
            for (uint32_t v = base + tid * 8u; v < stop; v += 16u * T) {
                uint32_t col[2][8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    col[0][i] = ahead[0][i];
                    col[1][i] = ahead[1][i];
                }
                request(v + 16u * T, stop, ahead[0]);
                request(v + 24u * T, stop, ahead[1]);
                take(v, col[0]);
                if (v + 8u * T < stop) take(v + 8u * T, col[1]);
            }
            __syncthreads();
        }
    } else {
        const int64_t r = row0 + wave;
        const float w0 = a.omega[0];
        CodeT* mine = code + min(wave, a.rows - 1u) * stride;
        for (uint32_t j = lane * 2u; wave < a.rows && j < len; j += kWave * 2u) *reinterpret_cast<float2*>(mine + j) = make_float2(w0, w0);
        if (wave < a.rows && r < m)
            scatter_row<ColT, CodeT, kWave, true>(colI, a, a.rowPtr[r], a.rowPtr[r + 1], lane, c0, len, s_ptr + wave * (kWave + 1), s_grp[wave], mine);
    }
    __syncthreads();
    const uint32_t wlen = c0 + a.seg >= a.n ? (uint32_t)(pitch - c0) : a.seg;  // the last segment also writes the padding
    const uint32_t rr = tid & (a.rows - 1u), columns = 8u * T / a.rows;  // columns per step of the workgroup
    if (row0 + rr >= m) return;
    if constexpr (kPieces == 0) {
        // 16 bytes per thread: columns 16 s + 8 half .. + 7 of 32, s = 0, 1 (a multiple of 32 columns lies in s_seg whole, zeros behind len)
        const uint32_t half = tid / a.rows & 1u;
        uint4* o = reinterpret_cast<uint4*>(reinterpret_cast<uint8_t*>(out) + ((row0 >> 5) * pitch + c0) * 32) + 32u * half + ((uint32_t)row0 & 31u) + rr;
        const CodeT* mine = code + rr * stride + 8u * half;
        for (uint32_t j = tid / a.rows / 2u * 32u; j < wlen; j += 2u * columns) {
            uint2 q0 = make_uint2(0u, 0u), q1 = q0;
            if (j < a.seg) {
                q0 = *reinterpret_cast<const uint2*>(mine + j);
                q1 = *reinterpret_cast<const uint2*>(mine + j + 16u);
            }
            o[2u * j] = make_uint4(q0.x, q0.y, q1.x, q1.y);
        }
        return;
    }
    uint16_t* o = out + (row0 >> 5) * 32 * pitch + ((row0 & 31) + rr) * 8;
    const CodeT* mine = code + rr * stride;
    for (uint32_t j = tid / a.rows * 8u; j < wlen; j += columns) {
        uint32_t p01[8], p2[8];
        if constexpr (kRanks) {
            const uint2 q = *reinterpret_cast<const uint2*>(mine + j);  // (behind len: anything, up to what launch_decode_tiles leaves behind the last row)
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i) {
                const uint32_t k = ((i < 4 ? q.x : q.y) >> (8 * (i & 3u))) & 0xFFu;
                p01[i] = s_val[k];
                p2[i] = kPieces == 3 ? s_val2[k] : 0u;
            }
        } else {
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i) {
                uint32_t p[3];
                cer::split3_finite((float)mine[min(j + i, len - 1u)], p);
                p01[i] = p[0] | (p[1] << 16);
                p2[i] = p[2];
            }
        }
        if (j + 8u > len) {
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i)
                if (j + i >= len) p01[i] = p2[i] = 0u;
        }
        uint32_t w[3][4];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            w[0][i] = __builtin_amdgcn_perm(p01[2 * i + 1], p01[2 * i], 0x05040100u);
            w[1][i] = __builtin_amdgcn_perm(p01[2 * i + 1], p01[2 * i], 0x07060302u);
            w[2][i] = p2[2 * i] | (p2[2 * i + 1] << 16);
        }
        const int64_t at = (c0 + j) * 32;  // (column / 8) . 32 rows . 8
#pragma unroll
        for (int q = 0; q < kPieces; ++q)
            *reinterpret_cast<uint4*>(o + q * plane + at) = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
    }
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
// Temporary device memory from the stream-ordered pool: released when the work queued before the
// release has run, so the buffers can be dropped as soon as the last kernel using them is queued.
struct DeviceBuf {
    void* p = nullptr;
    hipStream_t s = nullptr;
    ~DeviceBuf() {
        if (p) (void)cer::temp_free(p, s);
    }
    hipError_t alloc(size_t bytes, hipStream_t stream) {
        s = stream;
        return (hipError_t)cer::temp_alloc(&p, bytes ? bytes : 1, stream);
    }
    template <typename T>
    T* as() const {
        return static_cast<T*>(p);
    }
};

#define HIP_TRY(expr)                                                \
    do {                                                             \
        const hipError_t e_ = (expr);                                \
        if (e_ != hipSuccess) return cer::record_hip_error((int)e_); \
    } while (0)

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Enqueues range (bits > 0) or the caller's codebook, then codes + per-row histograms (cnt != nullptr) over `rows` rows of
// row_len elements (the last one possibly shorter).  `part`: kRangeParts float4.
int run_codes(const float* W, int64_t total, int64_t rows, int64_t row_len, const float* codebook, int32_t K, int32_t bits,
              hipStream_t s, FrontState* st_dev, float4* part, uint8_t* codes, uint32_t* cnt, unsigned long long* hist, float* Wq) {
    // workgroups walk several rows where that still leaves eight of them per compute unit: their prologue is shared
    const unsigned blocks = (unsigned)std::min<int64_t>(rows, 2048);
    const int aligned = row_len % 4 == 0 && aligned16(W) && (!Wq || aligned16(Wq)) && (reinterpret_cast<uintptr_t>(codes) & 3u) == 0;
    const bool copies = cnt && row_len >= (aligned ? 4096 : 1024);
    if (bits > 0) {
        const int nparts = (int)std::min<int64_t>(kRangeParts, (total + 1023) / 1024);
        HIP_TRY(cer::launch_kernel(range_kernel, dim3(nparts), dim3(256), 0, s, W, total, part, hist, st_dev));
        HIP_TRY(cer::launch_kernel(copies ? codes_kernel<true, kHistCopies> : codes_kernel<true, 1>, dim3(blocks), dim3(256), 0, s, W, total, rows, row_len, part, nparts, bits,
                                   st_dev, codes, cnt, hist, Wq, aligned));
    } else {
        // duplicates and non-finite values are refused
        CodebookArg cb;
        std::memset(&cb, 0, sizeof cb);
        for (int32_t k = 0; k < K; ++k) {
            if (!std::isfinite(codebook[k])) return CER_E_BAD_CODEBOOK;
            cb.v[k] = codebook[k] == 0.0f ? 0.0f : codebook[k];
        }
        float sorted[kCodes];
        std::copy(cb.v, cb.v + K, sorted);
        std::sort(sorted, sorted + K);
        if (std::adjacent_find(sorted, sorted + K) != sorted + K) return CER_E_BAD_CODEBOOK;
        cb.K = (uint32_t)K;
        HIP_TRY(cer::launch_kernel(codebook_kernel, dim3(1), dim3(256), 0, s, cb, hist, st_dev));
        HIP_TRY(cer::launch_kernel(copies ? codes_kernel<false, kHistCopies> : codes_kernel<false, 1>, dim3(blocks), dim3(256), 0, s, W, total, rows, row_len, part, 0, 0, st_dev,
                                   codes, cnt, hist, (float*)nullptr, aligned));
    }
    return CER_OK;
}

// Pinned host memory for FrontResult: a few blocks are kept for later calls.
struct Mailboxes {
    std::mutex mu;
    FrontResult* spare[8] = {};
    int count = 0;
};
Mailboxes g_mailboxes;

struct Mailbox {
    FrontResult* p = nullptr;
    bool busy = false;  // a kernel that writes to it may still be running
    ~Mailbox() {
        if (!p || busy) return;
        {
            std::lock_guard<std::mutex> lock(g_mailboxes.mu);
            if (g_mailboxes.count < 8) {
                g_mailboxes.spare[g_mailboxes.count++] = p;
                return;
            }
        }
        (void)hipHostFree(p);
    }
    hipError_t get() {
        {
            std::lock_guard<std::mutex> lock(g_mailboxes.mu);
            if (g_mailboxes.count > 0) p = g_mailboxes.spare[--g_mailboxes.count];
        }
        if (!p) {
            void* q = nullptr;
            const hipError_t e = hipHostMalloc(&q, sizeof(FrontResult), hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent);
            if (e != hipSuccess) return e;
            p = static_cast<FrontResult*>(q);
        }
        for (unsigned long long* word : {&p->early[0], &p->early[1], &p->totals[0], &p->totals[1], &p->totals[2]}) __atomic_store_n(word, 0ull, __ATOMIC_RELEASE);
        return hipSuccess;
    }
    // Returns when the words are there.  A copy and a synchronisation of the stream take 30 us more than looking at them; the stream is asked
    // now and then, so that a failed launch ends the wait.
    template <size_t kWords>
    hipError_t wait(hipStream_t s, const unsigned long long (&words)[kWords]) {
        auto there = [&] {
            for (size_t i = 0; i < kWords; ++i)
                if (!__atomic_load_n(&words[i], __ATOMIC_ACQUIRE)) return false;
            return true;
        };
        for (uint32_t spins = 1; !there(); ++spins) {
            if (spins % 8192u == 0) {
                hipError_t e = spins > (1u << 20) ? hipStreamSynchronize(s) : hipStreamQuery(s);
                if (e == hipErrorNotReady) {
                    (void)hipGetLastError();
                    continue;
                }
                if (e == hipSuccess && !there()) e = hipErrorLaunchFailure;
                if (e != hipSuccess) return e;
                break;
            }
            __builtin_ia32_pause();
        }
        return hipSuccess;
    }
    hipError_t wait_sizes(hipStream_t s, FrontSizes* sizes) {
        const hipError_t e = wait(s, p->early);
        const unsigned long long q = p->early[0];
        *sizes = FrontSizes{(uint32_t)(q >> 50) & 0xFu, (uint32_t)(q >> 32) & 0x1FFu, (uint32_t)(q >> 41) & 0x1FFu, (uint32_t)q, p->early[1] & ~kWritten};
        return e;
    }
    hipError_t wait_totals(hipStream_t s) {  // the last that a kernel writes before the emitter
        const hipError_t e = wait(s, p->totals);
        if (e == hipSuccess) busy = false;
        return e;
    }
    unsigned long long groups() const { return p->totals[0] & ~kWritten; }
    unsigned long long nonempty() const { return p->totals[1] & ~kWritten; }
    uint32_t max_row_groups() const { return (uint32_t)p->totals[2]; }
    uint32_t flags() const { return (uint32_t)(p->totals[2] >> 50) & 0xFu; }
};

int flags_to_error(uint32_t flags) {
    if (flags & kFlagNonFinite) return CER_E_INVALID;
    if (flags & kFlagMissing) return CER_E_NOT_IN_CODEBOOK;
    if (flags & kFlagCollide) return CER_E_BAD_CODEBOOK;
    if (flags & kFlagTooLarge) return CER_E_TOO_LARGE;
    return CER_OK;
}

bool mostly_implicit(int64_t nnz, int64_t m, int64_t n) { return (double)nnz * 2.0 < (double)m * (double)n; }

// Whether emit_sorted_kernel is expected to be ahead.  Clocks, where half or more is indexed: a row sorted in LDS takes 125 per 64 columns, 60
// per codebook position and 10000 (its start, the pointers, the way out), and its LDS limits how many of them a compute unit holds;
// emit_kernel takes 800 per 64 columns of a row, one after another, or 72 of a compute unit's time.  Whole calls, emit_kernel / emit_sorted_kernel,
// us: 300 x 9000, 7 bits 90 / 65, 8 bits 91 / 70; 1000 x 2000, 6 bits 59 / 54; 4096 x 9216, 7 bits 158 / 148, 8 bits 173 / 192; 2048 x 4096,
// 7 bits 80 / 76, 8 bits 82 / 96; 4096 x 2050, 7 bits 84 / 86.  Of 165 such matrices it takes the slower one for eight, by up to 11 % (2092 x 2716, 98
// values, 81 / 73).  Where large matrices have many equally frequent values emit_kernel takes far longer, which the sizes do not tell: 4096 x
// 9216, 100 of them 313 / 193, but 256 474 / 245, where emit_kernel serves.
// Where fewer are, emit_kernel packs a row's elements first, which takes 160 per 64 columns, and 640 per 64 elements behind it; the terms are
// fitted to 68 such matrices (256 to 4096 rows of 1024 to 25088 columns, 2 to 49 % indexed, 4 to 256 values), compressed by either kernel: the
// one taken is 0.4 % slower than the better one in the mean, always emit_kernel 11 %.  Whole calls: 1024 x 9216, 5 bits 106 / 79; 4096 x 9216, 5
// bits 182 / 155, 3 bits (2 % indexed) 142 / 147; 1024 x 2048, 5 bits 64.7 / 60.8; 2048 x 1024, 5 bits 64.9 / 67.4; 400 x 25088, 4 values, 40 %
// indexed 146 / 89; 4096 x 12000, 200 values, 10 % 131 / 171.  With the factor of 0.93 none of the 68 is slower than with emit_kernel (with 1 and 4000 in
// place of 2500 five of them, by up to 5 %).
bool sorted_rows_pay(int64_t m, int64_t n, uint32_t positions, size_t lds, double indexed) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 256;
    const double columns = (double)n / 64.0, share = std::max((double)m / std::max(cus, 1), 1.0);  // rows per compute unit
    const double rounds = std::ceil(share / std::floor(160.0 * 1024.0 / (double)lds));
    if (indexed >= 0.5) return rounds * (125.0 * columns + 60.0 * positions + 10000.0) < std::max(800.0 * columns, 72.0 * columns * share) + 6000.0;
    const double eights = (double)((positions + 7u) & ~7u);
    const double sorted = std::max(rounds * (45.0 * columns + 72.0 * eights + 8000.0), share * (15.5 * columns + 10.0 * eights + 1000.0));
    return sorted < 0.93 * (std::max((160.0 + 640.0 * indexed) * columns, share * 110.0 * indexed * columns) + 2500.0);
}

// LDS per row of emit_sorted_kernel, 0 where emit_kernel serves.  longest: indexed elements of the longest row; nnz: of the matrix.
size_t sorted_lds(int64_t m, int64_t n, uint32_t positions, uint32_t longest, uint64_t nnz) {
    const size_t lds = emit_stage_bytes(longest) + (size_t)((positions + 7u) & ~7u) * (kRowCounters + 1u) * 4u;
    return n >= 1024 && n <= kSortedColumns && lds <= 64 * 1024 && sorted_rows_pay(m, n, positions, lds, (double)nnz / ((double)m * (double)n)) ? lds : 0;
}

// Waves of emit_sorted_kernel that run at once.
int64_t sorted_waves(size_t lds) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 256;
    return (int64_t)std::max(cus, 1) * (int64_t)(160 * 1024 / lds);
}

template <typename ColT>
hipError_t launch_emit(hipStream_t s, const uint8_t* codes, const uint32_t* cnt, const uint2* rowStart, const FrontState* st,
                       int64_t m, int64_t n, int cser, int sparse, const EmitTarget& to, const FrontSizes& sizes, FrontResult* out) {
    if constexpr (sizeof(ColT) == 2) {
        if (const size_t lds = sorted_lds(m, n, sizes.K, sizes.longest, sizes.nnz))
            return cer::launch_kernel(n <= 1024 * kSortedPieces ? emit_sorted_kernel<kSortedPieces> : emit_sorted_kernel<0>, dim3((unsigned)std::min<int64_t>(m, sorted_waves(lds)) + 1u), dim3(64), lds, s, codes, cnt, rowStart, st, m, (uint32_t)n, cser,
                                      sizes.K, emit_stage_bytes(sizes.longest), to, out);
    }
    // rank < K <= 256, so OmegaI is always one byte wide here
    return cer::launch_kernel(emit_kernel<ColT, uint8_t>, dim3((unsigned)((m + 3) / 4 + 1)), dim3(256), 0, s, codes, cnt, rowStart,
                              st, m, n, cser, sparse, to, out);
}

}  // namespace

namespace cer {

namespace {
DecodeArgs decode_args(const DeviceView& v, int64_t nseg, uint32_t multiple) {
    DecodeArgs a;
    a.omegaPtr = v.omegaPtr;
    a.rowPtr = v.rowPtr;
    a.omegaI = static_cast<const uint8_t*>(v.omegaI);
    a.omega = v.omega;
    a.oi_bits = v.omegaI_bits;
    a.cser = v.cser;
    a.K = (uint32_t)v.K;
    a.n = v.n;
    a.tab = v.rank_tab;
    a.tab_shift = (uint32_t)v.rank_tab_shift;
    a.grid = v.grid;
    nseg = std::min<int64_t>(std::max<int64_t>(nseg, 1), 65535);
    a.seg = (uint32_t)(((v.n + nseg - 1) / nseg + multiple - 1) / multiple * multiple);
    a.nseg = (uint32_t)((v.n + a.seg - 1) / a.seg);
    return a;
}

// From half of the 256 MB cache in front of the memory on, the decoder's stores go past the caches: what they would leave there is written
// back while the next kernels read.  us without / with, 7 bits: 4096 x 9216 (151 MB), into several results in turn 52 / 41, compressed and decoded
// 222 / 206, one layer after the other 206 / 190 (the next matrix's range_kernel 38 / 27), and reduced 256 / 257; 4096 x 25088 (411 MB) 567 / 531, 549 / 513,
// 663 / 641.  Programs that only decode and read the result at once lose where it would have stayed: decoded in turn and reduced 4096 x 9216
// 92 / 93, 4096 x 12288 (201 MB) 98 / 116, 4096 x 25088 254 / 241; into the same memory each time 4096 x 9216 70 / 86.  Smaller results are read from
// that cache (67 MB, decoder and reduction: 42 us, 47 past it).
constexpr int64_t kPastCaches = 128 << 20;

template <typename ColT, typename CodeT>
hipError_t launch_decode(const DeviceView& v, float* out, hipStream_t s) {
    // Segments of equal length, at most 32 KiB of LDS; more of them where the rows alone give fewer than eight workgroups
    // per compute unit, but not below 1024 columns (every segment reads the whole row's indices).
    const int64_t most = 32768 / (int64_t)sizeof(CodeT);
    const DecodeArgs a = decode_args(v, std::max<int64_t>((v.n + most - 1) / most, std::min<int64_t>((2048 + v.m - 1) / v.m, v.n / 1024)), 8);
    const dim3 grid((unsigned)v.m, a.nseg);
    const size_t lds = ((size_t)a.seg * sizeof(CodeT) + 18) & ~(size_t)15;  // (up to three bytes in front of the codes)
    const ColT* colI = static_cast<const ColT*>(v.colI);
    const bool past = v.m * v.n * 4 >= kPastCaches;
    // short rows: one wave per row, four times as many workgroups in flight
    if (v.n <= 1024)
        return launch_kernel(past ? decode_kernel<ColT, CodeT, 64, true> : decode_kernel<ColT, CodeT, 64, false>, grid, dim3(64), lds, s, colI, a, out);
    return launch_kernel(past ? decode_kernel<ColT, CodeT, 256, true> : decode_kernel<ColT, CodeT, 256, false>, grid, dim3(256), lds, s, colI, a, out);
}

// kPieces == 0: ranks, one byte each (decode_ranks).
template <typename ColT, typename CodeT, int kPieces>
hipError_t launch_decode_tiles(const DeviceView& v, uint16_t* out, int64_t pitch, int64_t plane, hipStream_t s) {
    uint32_t rows = 8;
    while (rows > 4 && (v.m + rows - 1) / rows < v.cus) rows >>= 1;
    // Every segment reads all indices of its rows, so there are as few as the LDS allows: two workgroups of 512 threads per compute unit with 48
    // KiB each for rows of up to 6144 columns, one of 1024 threads with up to 132 for longer ones (33792 columns in one segment).  2780 x 19849, 40 %
    // indexed, ranks: eight rows in four segments of 6 K columns 50 us, in two of 10 K 36, four rows in one 20 (whole call 136 / 119 / 101); 2150 x 19579,
    // one piece, 69 -> 42 us; two workgroups of 512 threads and four rows 2 - 10 % slower in the call from 11000 columns on, 5 - 10 % faster below
    // 9000 and large batches of rows.  Two rows where four leave half of the compute units without any: 358 x 22120, batch 329 72 -> 67, 264 x 9255, 29 25 -> 21.
    int64_t most = 48 * 1024;
    bool wide = false;
    if (sizeof(CodeT) == 1 && v.n > most / 8) {
        rows = kPieces == 0 && v.m <= 2 * v.cus ? 2 : 4;
        wide = rows == 2 || v.n > most / 4;
        if (wide) most = 132 * 1024;
    }
    most /= sizeof(CodeT) * rows;
    const int64_t groups = (v.m + rows - 1) / rows;
    DecodeArgs a = decode_args(v, (v.n + most - 1) / most, 32);
    a.rows = rows;
    const dim3 grid((unsigned)groups, a.nseg);
    // The last segment's rows are read up to the pitch, the last of them behind all others.
    const size_t behind = (size_t)std::max<int64_t>(pitch - (int64_t)(a.nseg - 1) * a.seg - (int64_t)(a.seg + 8), 0);
    const size_t lds = ((size_t)(a.seg + 8) * rows + behind) * sizeof(CodeT);
    auto* kern = decode_tiles_kernel<ColT, CodeT, kPieces, 512>;
    if constexpr (sizeof(CodeT) == 1)
        if (wide) kern = decode_tiles_kernel<ColT, CodeT, kPieces, 1024>;
    {   // with the static part more than 64 KiB
        static cer::LdsGrant<2> grant;
        const hipError_t e = grant.ensure(wide, (const void*)kern, 133 * 1024);
        if (e != hipSuccess) return e;
    }
    return launch_kernel(kern, grid, dim3(wide ? 1024 : 512), lds, s, static_cast<const ColT*>(v.colI), a, v.m, pitch, plane, out);
}

// The pieces of the values, or (pieces 0) their ranks.
template <typename ColT>
hipError_t decode_tiles_by(const DeviceView& v, int pieces, uint16_t* out, int64_t pitch, int64_t plane, hipStream_t s) {
    if (v.rank_tab) {
        switch (pieces) {
            case 0: return launch_decode_tiles<ColT, uint8_t, 0>(v, out, pitch, plane, s);
            case 1: return launch_decode_tiles<ColT, uint8_t, 1>(v, out, pitch, plane, s);
            case 2: return launch_decode_tiles<ColT, uint8_t, 2>(v, out, pitch, plane, s);
            default: return launch_decode_tiles<ColT, uint8_t, 3>(v, out, pitch, plane, s);
        }
    }
    switch (pieces) {
        case 1: return launch_decode_tiles<ColT, float, 1>(v, out, pitch, plane, s);
        case 2: return launch_decode_tiles<ColT, float, 2>(v, out, pitch, plane, s);
        default: return launch_decode_tiles<ColT, float, 3>(v, out, pitch, plane, s);
    }
}
int decode_tiles(const DeviceView& v, int pieces, uint16_t* out, int64_t pitch, int64_t plane, void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (v.colI_bits) {
        case 8: return (int)decode_tiles_by<uint8_t>(v, pieces, out, pitch, plane, s);
        case 16: return (int)decode_tiles_by<uint16_t>(v, pieces, out, pitch, plane, s);
        default: return (int)decode_tiles_by<uint32_t>(v, pieces, out, pitch, plane, s);
    }
}
}  // namespace

int decode_device(const DeviceView& v, float* W, void* stream) {
    if (v.m == 0 || v.n == 0) return CER_OK;
    if (v.m > 0x7FFFFFFFll) return CER_E_INVALID;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool ranks = v.K <= kCodes;
    hipError_t e;
    switch (v.colI_bits) {
        case 8: e = ranks ? launch_decode<uint8_t, uint8_t>(v, W, s) : launch_decode<uint8_t, float>(v, W, s); break;
        case 16: e = ranks ? launch_decode<uint16_t, uint8_t>(v, W, s) : launch_decode<uint16_t, float>(v, W, s); break;
        default: e = ranks ? launch_decode<uint32_t, uint8_t>(v, W, s) : launch_decode<uint32_t, float>(v, W, s);
    }
    HIP_TRY(e);
    return CER_OK;
}

int decode_pieces(const DeviceView& v, uint16_t* W, int64_t pitch, int64_t plane, void* stream) {
    return decode_tiles(v, v.grid.scale != 0.f ? 2 : v.pieces, W, pitch, plane, stream);
}

int decode_ranks(const DeviceView& v, uint8_t* W, int64_t pitch, void* stream) {
    return decode_tiles(v, 0, reinterpret_cast<uint16_t*>(W), pitch, 0, stream);
}

int quantize_device(const float* W, int64_t count, int32_t bits, uint8_t* codes, float* Wq, float* codebook_out,
                    int32_t* K_out, void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t row_len = 4096, rows = (count + row_len - 1) / row_len;
    DeviceBuf tmp;
    HIP_TRY(tmp.alloc(kRangeParts * sizeof(float4) + sizeof(FrontState), s));
    float4* part = tmp.as<float4>();
    FrontState* st = reinterpret_cast<FrontState*>(part + kRangeParts);
    int rc = run_codes(W, count, rows, row_len, nullptr, 0, bits, s, st, part, codes, nullptr, nullptr, Wq);
    if (rc != CER_OK) return rc;
    FrontState h;
    HIP_TRY(hipMemcpyAsync(&h, st, sizeof h, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    rc = flags_to_error(h.flags);
    if (rc != CER_OK) return rc;
    if (K_out) *K_out = (int32_t)h.K;
    if (codebook_out) std::memcpy(codebook_out, h.codebook, (size_t)h.K * 4);
    return CER_OK;
}

bool encode_sorts_rows(const DeviceView& v, int32_t K) {
    return v.colI_bits == 16 && v.m > 0 && sorted_lds(v.m, v.n, (uint32_t)K, v.longest_row, (uint64_t)v.nnz) != 0;
}

int encode_device(const float* W, int64_t m, int64_t n, const float* codebook, int32_t K, int32_t bits, bool cser,
                  void* stream, float* codebook_out, int32_t* K_out, cer_matrix** out) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t N = m * n;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));

    // one stream-ordered temporary: [state][codes: N bytes][per-row histograms][{groups, elements} per row: m][their prefix
    // sums: m + 1][partial histograms and least counts][partial ranges]
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t off_codes = up(sizeof(FrontState)), off_cnt = off_codes + up((size_t)N);
    const size_t off_gn = off_cnt + up((size_t)m * kCodes * 4), off_start = off_gn + up((size_t)m * 8);
    const size_t off_hist = off_start + up((size_t)(m + 1) * 8), off_part = off_hist + (size_t)kHistParts * kCodes * (8 + 4);
    Mailbox box;
    HIP_TRY(box.get());
    DeviceBuf tmp;
    HIP_TRY(tmp.alloc(off_part + kRangeParts * sizeof(float4), s));
    unsigned char* tp = tmp.as<unsigned char>();
    FrontState* sd = reinterpret_cast<FrontState*>(tp);
    uint8_t* codes_d = tp + off_codes;
    uint32_t* cnt_d = reinterpret_cast<uint32_t*>(tp + off_cnt);
    auto* rowGN = reinterpret_cast<unsigned long long*>(tp + off_gn);
    uint2* rowStart = reinterpret_cast<uint2*>(tp + off_start);
    auto* hist = reinterpret_cast<unsigned long long*>(tp + off_hist);

    int rc = run_codes(W, N, m, n, codebook, K, bits, s, sd, reinterpret_cast<float4*>(tp + off_part), codes_d, cnt_d, hist, nullptr);
    if (rc != CER_OK) return rc;
    box.busy = true;
    const int64_t rows_each = m > kFewRows ? 4 : 1;
    HIP_TRY(launch_kernel(rows_each > 1 ? row_layout_kernel<4> : row_layout_kernel<1>, dim3((unsigned)((m + 16 * rows_each - 1) / (16 * rows_each)) + 1u),
                          dim3(1024), 0, s, cnt_d, hist, m, n, cser ? 1 : 0, sd, rowGN, rowStart, box.p));
    // what can be done before the sizes are here
    auto A = std::make_shared<HostMatrix>();
    A->cser = cser;
    A->m = m;
    A->n = n;
    A->colI.bits = min_index_bits(n > 0 ? (uint64_t)(n - 1) : 0);
    A->rowPtr.len = m + 1;
    A->omega.reserve(kCodes);
    A->count.reserve(kCodes);
    A->arrays_on_host.store(false);  // the index arrays stay on the device until somebody asks for them on the host
    std::unique_ptr<cer_matrix, void (*)(cer_handle_t*)> hnd(new cer_matrix(), cer_free);
    hnd->host = A;
    if (s) hnd->off_null_stream.store(true, std::memory_order_relaxed);
    EmitTarget to;
    std::memset(&to, 0, sizeof to);

    FrontSizes sizes;
    HIP_TRY(box.wait_sizes(s, &sizes));
    const FrontResult& h = *box.p;
    rc = flags_to_error(sizes.flags);
    // The emitter is launched while the rows are added up -- the host's and the launch's time were between the two: compressed and decoded 256 x 512, 5
    // bits, 53 -> 49 us, 1024 x 2048, 6 bits, 61.7 -> 58.9, 4096 x 9216, 7 bits, 182 -> 177 --, with room for as many groups as there may be: a row has at
    // most one per value but one.  Where that room could be more than half of all other parts (few indexed elements per value and
    // row), their number is waited for.
    const uint64_t limit = 0xFFFFFFFFull - 65536;
    uint64_t room = (uint64_t)m * (sizes.Kp > 0 ? sizes.Kp - 1u : 0u);
    if (cser) room = std::min<uint64_t>(room, sizes.nnz);
    const size_t colI_bytes = (size_t)sizes.nnz * (size_t)(A->colI.bits / 8), oi_width = cser ? 1 : 0;  // (ranks below 256)
    auto layout = [&] { return DeviceLayout::make(colI_bytes, (int64_t)room, m, (size_t)room * oi_width, (int32_t)sizes.Kp); };
    bool known = rc != CER_OK || sizes.nnz > limit || room > limit;
    DeviceLayout l;
    if (!known) {
        l = layout();
        const size_t room_bytes = room * (4 + oi_width);
        known = (l.total - room_bytes) / 2 < room_bytes;
    }
    auto exact = [&]() -> int {  // waits for the number of groups
        HIP_TRY(box.wait_totals(s));
        if (rc == CER_OK) rc = flags_to_error(box.flags());
        if (rc != CER_OK) return rc;
        known = true;
        room = box.groups();
        l = layout();
        return CER_OK;
    };
    if (known && (rc = exact()) != CER_OK) return rc;

    // the handle's own allocation, filled in place by the emit kernel
    void* base = nullptr;
    int got = handle_alloc(&base, l.total, s);
    if (got == (int)hipErrorOutOfMemory && !known) {  // there may be enough for the handle without the room
        (void)hipGetLastError();
        if ((rc = exact()) != CER_OK) return rc;
        got = handle_alloc(&base, l.total, s);
    }
    if (got != (int)hipSuccess) {
        (void)box.wait_totals(s);
        HIP_TRY((hipError_t)got);
    }
    hnd->d_base = base;

    to.base = static_cast<unsigned char*>(base);
    to.off_optr = l.off_optr;
    to.off_rptr = l.off_rptr;
    to.off_ri = l.off_ri;
    to.off_oi = l.off_oi;
    to.off_om = l.off_om;
    to.off_tab = l.off_tab;
    to.tab_shift = l.tab_shift;
    // the read-ahead padding and the gaps are cleared; the arrays themselves are written completely
    auto gap = [&](size_t begin, size_t end, size_t per_group = 0) {
        to.gap_begin[to.ngaps] = begin;
        to.gap_group[to.ngaps] = (uint32_t)per_group;
        to.gap_end[to.ngaps++] = end;
    };
    gap(colI_bytes, l.off_optr);
    gap(l.off_optr + 4, l.off_rptr, 4);
    gap(l.off_rptr + (size_t)(m + 1) * 4, l.off_oi);
    gap(l.off_oi, l.off_om, oi_width);
    gap(l.off_om + (size_t)sizes.Kp * 4, l.off_ri);
    gap(l.off_ri + (size_t)(m + 1) * 8, l.off_tab);
    gap(l.off_tab + (l.tab_shift ? ((size_t)m << l.tab_shift) * 4 : 0), l.total);
    const int cs = cser ? 1 : 0;
    // with fewer than half of the elements indexed emit_kernel packs them in LDS before it scatters them
    const int sp = mostly_implicit((int64_t)sizes.nnz, m, n) ? 1 : 0;
    hipError_t e = hipSuccess;
    switch (hnd->host->colI.bits) {
        case 8: e = launch_emit<uint8_t>(s, codes_d, cnt_d, rowStart, sd, m, n, cs, sp, to, sizes, box.p); break;
        case 16: e = launch_emit<uint16_t>(s, codes_d, cnt_d, rowStart, sd, m, n, cs, sp, to, sizes, box.p); break;
        default: e = launch_emit<uint32_t>(s, codes_d, cnt_d, rowStart, sd, m, n, cs, sp, to, sizes, box.p);
    }
    box.busy = true;
    HIP_TRY(e);
    A->K = (int32_t)sizes.Kp;
    A->nnz = (int64_t)sizes.nnz;
    A->colI.len = A->nnz;
    A->omegaPtr.bits = min_index_bits((uint64_t)A->nnz);
    if (cser) A->omegaI.bits = min_index_bits(A->K > 0 ? (uint64_t)(A->K - 1) : 0);
    A->omega.resize(sizes.Kp);
    A->count.resize(sizes.Kp);
    HIP_TRY(hipStreamSynchronize(s));  // the handle is complete for every stream; errors surface here
    box.busy = false;
    if (!known && (rc = flags_to_error(box.flags())) != CER_OK) return rc;
    A->G = (int64_t)box.groups();
    A->nonempty_groups = (int64_t)box.nonempty();
    A->max_row_groups = (int64_t)box.max_row_groups();
    A->omegaPtr.len = A->G + 1;
    A->rowPtr.bits = min_index_bits((uint64_t)A->G);
    if (cser) A->omegaI.len = A->G;
    l.omegaI_bytes = (size_t)A->G * oi_width;
    std::copy_n(h.omega, sizes.Kp, A->omega.begin());
    std::copy_n(h.count, sizes.Kp, A->count.begin());
    bind_device(hnd.get(), dev, base, l);
    hnd->view.longest_row = sizes.longest;
    if (K_out) *K_out = (int32_t)sizes.K;
    if (codebook_out) std::memcpy(codebook_out, h.codebook, (size_t)sizes.K * 4);
    // rows of unequal length: the batched product wants them ordered (and the longest in parts); the row starts
    // come back from the device only when the longest row says that the table will be built
    if (row_schedule_wanted((uint64_t)sizes.nnz, (uint64_t)m, (uint64_t)sizes.longest)) {
        std::vector<uint32_t> info((size_t)(m + 1) * 2);
        HIP_TRY(hipMemcpy(info.data(), to.base + l.off_ri, info.size() * 4, hipMemcpyDeviceToHost));
        std::vector<uint64_t> start((size_t)m + 1);
        for (int64_t r = 0; r <= m; ++r) start[(size_t)r] = info[(size_t)r * 2 + 1];
        rc = build_row_schedule(hnd.get(), start);
        if (rc != CER_OK) return rc;
    }
    *out = hnd.release();
    return CER_OK;
}

}  // namespace cer
