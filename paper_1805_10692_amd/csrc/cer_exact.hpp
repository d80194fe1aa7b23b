// Decoded rows of W in LDS, pieces of X, and outputs formed once more in binary32: what the kernels that decode and multiply in one
// launch share (cer_fused.hip, cer_tile.hip).
#pragma once

#include "cer_split3.hpp"
#include "cer_stream.hpp"

namespace cer {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx3 __attribute__((ext_vector_type(3)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

using Shape = GemvShape<uint16_t>;  // windows of 512 positions, three per batch

struct ExactArgs {
    float* Out;
    const uint32_t* tab;
    const uint16_t* colI;
    const float* omega;
    const float* X;
    float scale;
    uint32_t m, n, L, tab_shift, entry;
    uint32_t row0, rows, col0, cols, k_begin, k_end;   // the workgroup's outputs
    uint32_t seg, stride, codes, values, row_values;
};

// LDS:
//   [prefix: 256 x 8 bytes]  byte k of entry f = number of set bits of f below bit k
//   [flags, cleared at the kernel's start, a bit per row: sums that are not finite, faint ones, rows without elements, rows with elements in
//    this part of W's columns; and: lossy inputs]
//   [arguments of the functions for those rows]
//   [per wave: bitmap | counts per word]
//   [pieces of the codebook's values, by rank]
//   [per row: values of its groups, in list order (kEntry bytes each): entry 0 = the most frequent value]
//   [per row: one byte per column of the segment, the entry its element has in that list]; later the waves' sums
constexpr uint32_t kPrefixBytes = 2048, kCallAt = kPrefixBytes + 32, kListsAt = kCallAt + 112;
constexpr int kOdd = 0, kFaint = 1, kEmpty = 2, kHolds = 3, kLossy = 4;  // the flags
__host__ __device__ constexpr uint32_t table_at(uint32_t waves) { return kListsAt + waves * 2u * (uint32_t)Shape::NWORDS * 4u; }
__host__ __device__ constexpr uint32_t entry_bytes(int form) { return form == 1 ? 2u : (form == kUniform ? 4u : 8u); }
__host__ __device__ __forceinline__ uint32_t values_at(uint32_t waves, uint32_t tab_shift, uint32_t entry) { return table_at(waves) + (entry << tab_shift); }

__device__ __forceinline__ uint32_t& flag(unsigned char* smem, int which) { return reinterpret_cast<uint32_t*>(smem + kPrefixBytes)[which]; }

// The prefix table's entry f.
__device__ __forceinline__ void prefix_entry(unsigned char* smem, uint32_t f) {
    uint32_t lo8 = 0, hi8 = 0;
#pragma unroll
    for (uint32_t k = 1; k < 8; ++k) {
        const uint32_t below = (uint32_t)__builtin_popcount(f & ((1u << k) - 1u));
        if (k < 4) lo8 |= below << (8 * k); else hi8 |= below << (8 * (k - 4));
    }
    reinterpret_cast<uint2*>(smem)[f] = make_uint2(lo8, hi8);
}

__device__ __forceinline__ void request_batch(const uint16_t* colI, uint4 (&q)[Shape::NW], uint32_t b, uint32_t te, uint32_t lane) {
    const uint4* p = reinterpret_cast<const uint4*>(colI + b) + lane;
#pragma unroll
    for (int W = 0; W < Shape::NW; ++W) q[W] = p[(b + (uint32_t)W * Shape::WIN < te ? W : 0) * kWave];
}

// Position behind the row's last one, from its record.
__device__ __forceinline__ uint32_t row_end(const uint32_t (&rec)[4], uint32_t last_word) {
    uint32_t te = (uint32_t)__builtin_amdgcn_readlane((int)rec[0], (int)(last_word & 63u));
#pragma unroll
    for (uint32_t t = 1; t < 4; ++t)
        if (t <= (last_word >> 6)) te = (uint32_t)__builtin_amdgcn_readlane((int)rec[t], 63);
    return te;
}

typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));

// The elements of one row, pair by pair: sink(pair, numbers) gets two positions' columns (65535: a position of another row) and in the
// lower half of `numbers`, a byte each, the numbers of their groups among the row's non-empty ones (from 1).  store(entry, tile): what
// belongs to group 64 tile + lane + 1 goes to that entry.  first_batch: the row's first indices, already requested.
// Per window of eight positions and lane: the bitmap's byte says which positions end a group, a table how many do before each
// of them, and the eight numbers come from two additions.
template <typename Store, typename Sink>
__device__ __forceinline__ void walk_row(const uint16_t* colI, const uint32_t (&rec)[4], const uint4 (&first_batch)[Shape::NW], uint32_t tab_shift,
                                         unsigned char* smem, uint32_t wave, uint32_t lane, Store store, Sink sink) {
    using S = Shape;
    const uint32_t last_word = (1u << tab_shift) - 1u, ntiles = (last_word >> 6) + 1u;
    uint32_t* bmp = reinterpret_cast<uint32_t*>(smem + kListsAt) + wave * (2u * (uint32_t)S::NWORDS);
    uint32_t* wpre = bmp + S::NWORDS;
    const uint32_t rs = (uint32_t)__builtin_amdgcn_readlane((int)rec[0], 0), te = row_end(rec, last_word);
    uint32_t b0 = rs & ~((uint32_t)S::PPL - 1u);
    uint32_t ends[4];  // of the lane's groups; kNoEnd: an empty one
    uint32_t count = 1;
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) {
        ends[t] = kNoEnd;
        if (t >= ntiles) continue;
        uint32_t e = (uint32_t)__builtin_amdgcn_update_dpp((int)rec[t], (int)rec[t], 0x130 /* wave_shl:1 */, 0xF, 0xF, false);
        if (t + 1 < ntiles && lane == kWave - 1u) e = (uint32_t)__builtin_amdgcn_readlane((int)rec[t < 3 ? t + 1 : 3], 0);
        const bool some = t * kWave + lane < last_word && e > rec[t];
        const uint64_t votes = __ballot(some);
        const uint32_t at = count + __builtin_amdgcn_mbcnt_hi((uint32_t)(votes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)votes, 0u));
        if (some) ends[t] = e;
        store(some ? at : 1u << tab_shift, t);  // (the entry behind all others)
        count += (uint32_t)__popcll(votes);
    }
    if (b0 >= te || count <= 1) return;  // wave-uniform
    // bit p of the bitmap: position b + p is the last one of a group (or of what lies in front of the row); wpre: how many of them
    // are in front of a word, and of the batch
    auto boundaries = [&](uint32_t b, uint32_t& before) {
        if (lane < (uint32_t)S::NWORDS) bmp[lane] = 0u;
        wave_lds_sync();
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
            if (t >= ntiles) break;
            const uint32_t rel = ends[t] - b - 1u;
            if (rel < (uint32_t)S::BATCH) atomicOr(&bmp[rel >> 5], 1u << (rel & 31u));
        }
        wave_lds_sync();
        uint32_t word = bmp[min(lane, (uint32_t)S::NWORDS - 1u)];
        const uint32_t front = rs - b - 1u;  // (only in the row's first batch, and if the row does not begin with it)
        if (front < 8u && lane == 0) { word |= 1u << front; bmp[0] = word; }
        const uint32_t pc = lane < (uint32_t)S::NWORDS ? (uint32_t)__builtin_popcount(word) : 0u, incl = wave_inclusive_scan(pc);
        if (lane < (uint32_t)S::NWORDS) wpre[lane] = before + incl - pc;
        before += __builtin_amdgcn_readlane(incl, kWave - 1);
        wave_lds_sync();
    };
    auto batch = [&](const uint4 (&q)[S::NW], uint32_t b, uint32_t& first) {
        boundaries(b, first);
#pragma unroll
        for (int W = 0; W < S::NW; ++W) {
            const uint32_t w0 = b + (uint32_t)W * S::WIN;
            if (W > 0 && w0 >= te) break;  // wave-uniform
            uint32_t col[4] = {q[W].x, q[W].y, q[W].z, q[W].w};
            if (w0 < rs || w0 + S::WIN > te) {  // wave-uniform: positions in front of the row or behind it get a column behind all
                const uint32_t p = w0 + 8u * lane;
                const int lo = min(max((int)(rs - p), 0), 8), hi = min(max((int)(te - p), 0), 8);
                const uint32_t out = ~((1u << hi) - 1u) | ((1u << lo) - 1u);
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    col[d] |= ((out >> (2 * d)) & 1u ? 0xFFFFu : 0u) | ((out >> (2 * d + 1)) & 1u ? 0xFFFF0000u : 0u);
            }
            const uint32_t bit0 = 8u * lane, wj = (uint32_t)W * S::WPW + (bit0 >> 5), sh = bit0 & 31u, word = bmp[wj];
            const uint32_t before = wpre[wj] + (uint32_t)__builtin_popcount(word & ((1u << sh) - 1u));
            const uint2 steps = reinterpret_cast<const uint2*>(smem)[(word >> sh) & 0xFFu];
            const uint32_t all = __builtin_amdgcn_perm(before, before, 0u);  // the byte four times
            const uint32_t num[2] = {all + steps.x, all + steps.y};  // beyond the row's last group bytes may carry, into others beyond it
#pragma unroll
            for (int d = 0; d < 4; ++d) sink(col[d], num[d >> 1] >> (16 * (d & 1)));
        }
    };
    uint4 ix[2][S::NW];
#pragma unroll
    for (int W = 0; W < S::NW; ++W) ix[0][W] = first_batch[W];
    uint32_t first = rs > b0 ? 0u : 1u;
    for (;;) {
        const uint32_t b1 = b0 + S::BATCH, b2 = b1 + S::BATCH;
        request_batch(colI, ix[1], b1 < te ? b1 : b0, te, lane);
        batch(ix[0], b0, first);
        if (b1 >= te) break;
        request_batch(colI, ix[0], b2 < te ? b2 : b1, te, lane);
        batch(ix[1], b1, first);
        if (b2 >= te) break;
        b0 = b2;
    }
    wave_lds_sync();  // the bitmap serves the next row
}

// The elements of one row in columns c0 .. c0 + seg - 1: row[column - c0] = the number of their group (walk_row); row[seg] takes what
// lies elsewhere.  Two positions' columns are moved and clamped by one instruction: 27 vector instructions and 10 of LDS per window --
// with a look-up of the rank, comparison and selection per position there were 64 and 18, and the scatter of 16 rows of 1380 elements took
// 7900 clocks in 8 waves instead of 6200 (5300 in 16); now the writes bound it.
template <typename Store>
__device__ __forceinline__ void scatter_row(const uint16_t* colI, const uint32_t (&rec)[4], const uint4 (&first_batch)[Shape::NW], uint32_t tab_shift,
                                            unsigned char* smem, uint32_t wave, uint32_t c0, uint32_t seg, unsigned char* row, uint32_t lane, Store store) {
    const uint32_t row_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)row;
    const ushortx2 shift = {(unsigned short)c0, (unsigned short)c0}, dump = {(unsigned short)seg, (unsigned short)seg};
    walk_row(colI, rec, first_batch, tab_shift, smem, wave, lane, store, [&](uint32_t cols, uint32_t two) {
        const ushortx2 at = __builtin_elementwise_min(__builtin_bit_cast(ushortx2, cols) - shift, dump);
        typedef unsigned char __attribute__((address_space(3))) * LdsByte;
        const uint32_t pair = __builtin_bit_cast(uint32_t, at);
        *reinterpret_cast<LdsByte>((uintptr_t)(row_at + (pair & 0xFFFFu))) = (unsigned char)two;
        *reinterpret_cast<LdsByte>((uintptr_t)(row_at + (pair >> 16))) = (unsigned char)(two >> 8);
    });
}

template <int CT>
__device__ __forceinline__ void load_columns(__amdgpu_buffer_rsrc_t x, uint32_t off, float (&v)[CT]) {
    if constexpr (CT >= 4) {
        const uintx4 q = __builtin_amdgcn_raw_buffer_load_b128(x, off, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = __uint_as_float(q[j]);
    }
    constexpr int kDone = CT >= 4 ? 4 : 0, kRest = CT - kDone;
    if constexpr (kRest == 4) {
        const uintx4 q = __builtin_amdgcn_raw_buffer_load_b128(x, off + kDone * 4, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[kDone + j] = __uint_as_float(q[j]);
    } else if constexpr (kRest == 3) {
        const uintx3 q = __builtin_amdgcn_raw_buffer_load_b96(x, off + kDone * 4, 0, 0);
#pragma unroll
        for (int j = 0; j < 3; ++j) v[kDone + j] = __uint_as_float(q[j]);
    } else if constexpr (kRest == 2) {
        const uintx2 q = __builtin_amdgcn_raw_buffer_load_b64(x, off + kDone * 4, 0, 0);
        v[kDone] = __uint_as_float(q[0]);
        v[kDone + 1] = __uint_as_float(q[1]);
    } else if constexpr (kRest == 1) {
        v[kDone] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x, off + kDone * 4, 0, 0));
    }
}

__device__ __forceinline__ floatx4 mfma16(uint4 a, uint4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// x - p of eight numbers and their pieces p, paired: the dot product of a pair (p, p') with (-1, 0) or (0, -1), added to x.  One
// instruction where unpacking and subtracting take two; exact, as the difference is.  Written out: the compiler's choice is the
// two-address form, which costs a move for every number of a wide load.  Results of dot products may be read by other
// instructions three wait states later: the block ends with them, or with the instructions that take the bits, in the order of the results.
// lost: takes the bits of the remainders.  Those of the second pieces have eight significant bits at most, so that the lower half of their
// binary32 form is zero unless they reach below 2^-133, the smallest bf16 number: then the third piece loses something.  (0.5 to 1 us
// of 11 to 30; looking at the inputs instead, three instructions per two, took 24 -> 27 us for 4096 x 9216, 15 % indexed, batch 32, and
// reading them again where a sum is faint 24 -> 37 with a column of zeros in X.)
__device__ __forceinline__ void remainders8(const uint32_t p[4], const float x[8], float r[8], uint32_t* lost) {
    const uint32_t lo = 0x0000BF80u, hi = 0xBF800000u;  // (-1, 0), (0, -1)
    if (lost != nullptr) {
        asm("v_dot2_f32_bf16 %0, %9, %21, %13\n\tv_dot2_f32_bf16 %1, %9, %22, %14\n\t"
            "v_dot2_f32_bf16 %2, %10, %21, %15\n\tv_dot2_f32_bf16 %3, %10, %22, %16\n\t"
            "v_dot2_f32_bf16 %4, %11, %21, %17\n\tv_dot2_f32_bf16 %5, %11, %22, %18\n\t"
            "v_dot2_f32_bf16 %6, %12, %21, %19\n\tv_dot2_f32_bf16 %7, %12, %22, %20\n\t"
            "v_or3_b32 %8, %8, %0, %1\n\tv_or3_b32 %8, %8, %2, %3\n\tv_or3_b32 %8, %8, %4, %5\n\tv_or3_b32 %8, %8, %6, %7"
            : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]), "+&v"(*lost)
            : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]),
              "s"(lo), "s"(hi));
        return;
    }
    asm("v_dot2_f32_bf16 %0, %8, %20, %12\n\tv_dot2_f32_bf16 %1, %8, %21, %13\n\t"
        "v_dot2_f32_bf16 %2, %9, %20, %14\n\tv_dot2_f32_bf16 %3, %9, %21, %15\n\t"
        "v_dot2_f32_bf16 %4, %10, %20, %16\n\tv_dot2_f32_bf16 %5, %10, %21, %17\n\t"
        "v_dot2_f32_bf16 %6, %11, %20, %18\n\tv_dot2_f32_bf16 %7, %11, %21, %19\n\ts_nop 2"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
        : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]),
          "s"(lo), "s"(hi));
}

// Pieces of eight numbers as split3_8 has them, for numbers that are finite and round to finite bf16 numbers; others leave a NaN.
__device__ __forceinline__ void split3_8_dot(const float x[8], uint4 out[3], uint32_t& lost) {
    float a[8], b[8];
    uint32_t p[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[0][i] = bf16_pair(x[2 * i], x[2 * i + 1]);
    remainders8(p[0], x, a, nullptr);
#pragma unroll
    for (int i = 0; i < 4; ++i) p[1][i] = bf16_pair(a[2 * i], a[2 * i + 1]);
    remainders8(p[1], a, b, &lost);
#pragma unroll
    for (int i = 0; i < 4; ++i) p[2][i] = bf16_pair(b[2 * i], b[2 * i + 1]);
#pragma unroll
    for (int j = 0; j < 3; ++j) out[j] = make_uint4(p[j][0], p[j][1], p[j][2], p[j][3]);
}

// Pointers of a function that is not inlined: told to be to memory or to LDS, or its loads would be of the kind that may be to either.
template <typename T>
__device__ __forceinline__ T* uniform_pointer(T* p) {
    const uint64_t u = (uint64_t)(uintptr_t)p;
    return (T*)reinterpret_cast<__attribute__((address_space(1))) T*>((uintptr_t)((uint64_t)uniform((uint32_t)(u >> 32)) << 32 | uniform((uint32_t)u)));
}
__device__ __forceinline__ unsigned char* lds_pointer(uint32_t at) {
    return (unsigned char*)reinterpret_cast<__attribute__((address_space(3))) unsigned char*>((uintptr_t)at);
}

// What the functions below know of the workgroup's outputs.
struct ExactCtx {
    uint32_t lane, wave, waves, m, n, L, row0, col0, cols, k_begin, k_end, shift, last_word;
    const float* X;
    const uint32_t* tab;
    const uint16_t* colI;
    __device__ __forceinline__ explicit ExactCtx(const unsigned char* smem) {
        const ExactArgs& a = *reinterpret_cast<const ExactArgs*>(smem + kCallAt);
        lane = threadIdx.x & 63u; wave = uniform(threadIdx.x >> 6); waves = uniform(blockDim.x / kWave);
        m = uniform(a.m); n = uniform(a.n); L = uniform(a.L);
        row0 = uniform(a.row0); col0 = uniform(a.col0); cols = uniform(a.cols); k_begin = uniform(a.k_begin); k_end = uniform(a.k_end);
        shift = uniform(a.tab_shift); last_word = (1u << shift) - 1u;
        X = uniform_pointer(a.X); tab = uniform_pointer(a.tab); colI = uniform_pointer(a.colI);
    }
};

// A lane's share of the tile's columns where rows of X are loaded four columns per lane: rows of X per load (a power of two), the lane's
// row and column.  (48 columns: 16 lanes idle.  Columns behind the batch: the next row's, not used for outputs.)
struct FourColumns {
    uint32_t lanes, at_once, row, col;
    __device__ __forceinline__ FourColumns(uint32_t lane, uint32_t cols)
        : lanes(cols / 4u), at_once(cols == 48u ? 4u : kWave / lanes), row(lane / lanes), col(4u * (lane - row * lanes)) {}
    __device__ __forceinline__ bool idle() const { return row >= at_once; }
};

// Of the rows of faint sums, where an input has lost bits: those with elements in these columns of W (or a most frequent value).  The
// others' sums are zero and lose nothing.
__device__ __attribute__((noinline)) uint32_t lossy_rows(uint32_t lds, uint32_t faint) {
    unsigned char* smem = lds_pointer(lds);
    const ExactCtx a(smem);
    if (uniform_pointer(reinterpret_cast<const ExactArgs*>(smem + kCallAt)->omega)[0] != 0.f) return faint;
    for (uint32_t r = a.wave; r < 32u; r += a.waves) {
        if (((faint >> r) & 1u) == 0u) continue;
        const uint32_t* record = a.tab + ((size_t)(a.row0 + r) << a.shift);
        const uint32_t te = uniform(record[a.last_word]);
        bool some = false;
        for (uint32_t p = uniform(record[0]); p < te && __ballot(some) == 0ull; p += kWave) {
            const uint32_t k = a.colI[min(p + a.lane, te - 1u)];
            some = k >= a.k_begin && k < a.k_end;
        }
        if (__ballot(some) != 0ull && a.lane == 0) atomicOr(&flag(smem, kHolds), 1u << r);
    }
    __syncthreads();
    return faint & uniform(flag(smem, kHolds));
}

// Rows of the outputs once more, in binary32, as the gathers have them: the sum over the row's indices of (value - most frequent value) . x,
// and that value times the column sum.  A wave takes a row, 256 positions at a time, and four columns of as many inputs per load as it has
// lanes for, eight loads in flight.  Calls that repeat every row (all of X near 2^-120, or a column with an infinity): 4096 x 9216, 15 %
// indexed, batch 32 65 us (25 without, 28 with the gathers), 2048 x 2048, 256 values, batch 16 34 (9.4; 12); with the outputs one per thread,
// each along W's columns, 1200 and 360.
__device__ __attribute__((noinline)) void exact_gathered(uint32_t lds, uint32_t rows) {
    unsigned char* smem = lds_pointer(lds);
    const ExactCtx a(smem);
    const ExactArgs& args = *reinterpret_cast<const ExactArgs*>(smem + kCallAt);
    const FourColumns mine(a.lane, a.cols);
    const __amdgpu_buffer_rsrc_t xbuf = x_rows(a.X, a.L, 0, a.n);
    const uint32_t end = min(a.k_end, a.n), columns = (a.col0 + mine.col) * 4u;
    constexpr uint32_t kNone = 0xFFFFFF00u;  // behind X: loads return zero
    float* factor = reinterpret_cast<float*>(smem + args.codes);  // by rank
    double* s_sum = reinterpret_cast<double*>(factor + 256);      // of X's columns: the waves' shares
    const float* omega = uniform_pointer(args.omega);
    float* out = uniform_pointer(args.Out);
    const float omega0 = omega[0];
    auto lanes_sum = [&](float v) {  // of the lanes that have the same columns
        double t = 0;
        for (uint32_t e = 0; e < mine.at_once; ++e) t += __shfl(v, (int)(mine.col / 4u + e * mine.lanes), kWave);
        return t;
    };
    __syncthreads();
    if (threadIdx.x <= a.last_word) factor[threadIdx.x] = omega[threadIdx.x] - omega0;  // (behind omega's end lies the rest of the handle)
    float column[4] = {};
    if (omega0 != 0.f) {
        float sum[4] = {};
        constexpr uint32_t kAhead = 8;
        const uint32_t step = a.waves * mine.at_once;
        for (uint32_t k = a.k_begin + a.wave * mine.at_once + mine.row; k < end; k += kAhead * step) {
            uintx4 x[kAhead];
#pragma unroll
            for (uint32_t u = 0; u < kAhead; ++u)
                x[u] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, mine.idle() || k + u * step >= end ? kNone : (k + u * step) * a.L * 4u + columns, 0, 0);
#pragma unroll
            for (uint32_t u = 0; u < kAhead; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += __uint_as_float(x[u][e]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double t = lanes_sum(sum[e]);
            if (mine.row == 0) s_sum[a.wave * a.cols + mine.col + e] = t;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double t = 0;
            for (uint32_t w = 0; w < a.waves; ++w) t += s_sum[w * a.cols + mine.col + e];
            column[e] = (float)t;
        }
    }
    __syncthreads();
    for (uint32_t r = a.wave; r < 32u; r += a.waves) {
        if (((rows >> r) & 1u) == 0u) continue;
        const uint32_t* record = a.tab + ((size_t)(a.row0 + r) << a.shift);
        const uint32_t rs = uniform(record[0]), count = uniform(record[a.last_word]) - rs;
        uint16_t* ends = reinterpret_cast<uint16_t*>(smem + args.values + r * args.row_values);  // of the row's groups, in its values' place
        for (uint32_t i = a.lane; i <= a.last_word; i += kWave) ends[i] = (uint16_t)(record[i] - rs);
        wave_lds_sync();
        float sum[4] = {};
        constexpr uint32_t kParts = 4, kAhead = 8;  // of 64 positions; loads
        for (uint32_t p0 = 0; p0 < count; p0 += kParts * kWave) {
            uint32_t at[kParts], rank[kParts] = {};  // where the input begins; the last of the row's boundaries at or before the position
            float f[kParts];
#pragma unroll
            for (uint32_t q = 0; q < kParts; ++q) {
                const uint32_t p = p0 + q * kWave + a.lane, k = p < count ? a.colI[rs + p] : ~0u;
                at[q] = k >= a.k_begin && k < end ? k * a.L * 4u : kNone;
            }
            for (uint32_t half = (a.last_word + 1u) >> 1; half != 0u; half >>= 1)
#pragma unroll
                for (uint32_t q = 0; q < kParts; ++q)
                    if (ends[rank[q] + half] <= p0 + q * kWave + a.lane) rank[q] += half;
#pragma unroll
            for (uint32_t q = 0; q < kParts; ++q) f[q] = factor[min(rank[q] + 1u, a.last_word)];
            const uint32_t here = min(count - p0, kParts * kWave);
            for (uint32_t i0 = 0; i0 < here; i0 += kAhead * mine.at_once) {
                uintx4 x[kAhead];
                float w[kAhead];
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u) {
                    const uint32_t i = i0 + u * mine.at_once, q = i >> 6;  // (uniform: at_once divides 64)
                    const int lane = (int)((i + mine.row) & 63u);
                    const uint32_t from = (uint32_t)__shfl((int)(q == 0u ? at[0] : (q == 1u ? at[1] : (q == 2u ? at[2] : at[3]))), lane, kWave);
                    w[u] = __shfl(q == 0u ? f[0] : (q == 1u ? f[1] : (q == 2u ? f[2] : f[3])), lane, kWave);
                    x[u] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, i >= kParts * kWave || mine.idle() || from == kNone ? kNone : from + columns, 0, 0);
                }
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] = fmaf(w[u], __uint_as_float(x[u][e]), sum[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double t = lanes_sum(sum[e]);
            if (omega0 != 0.f) t = fma((double)omega0, (double)column[e], t);
            const uint32_t c = a.col0 + mine.col + e;
            if (mine.row == 0 && c < a.L) out[(size_t)(a.row0 + r) * a.L + c] = (float)t;
        }
    }
}

// The same with every element of W, a zero weight times an infinity too: the rows are decoded once more and multiplied by the fp32 matrix
// instruction, 32 columns after the other.  1500 x 9000, 16 values, batch 40: 94 us (25 without, 82 with the decoded matrix), 786 x 1952, 32
// values, batch 113 39 (11; 48); one output per thread: 1970 and 367.
__device__ __attribute__((noinline)) void exact_dense(uint32_t lds, uint32_t rows) {
    unsigned char* smem = lds_pointer(lds);
    const ExactCtx a(smem);
    const ExactArgs& args = *reinterpret_cast<const ExactArgs*>(smem + kCallAt);
    const uint32_t tid = threadIdx.x, lane = a.lane, n = a.n, L = a.L, tiles = uniform(args.rows) / 16u, seg = uniform(args.seg), stride = uniform(args.stride);
    const uint32_t entry = uniform(args.entry), row_values = uniform(args.row_values);
    const float scale = args.scale;
    float* out = uniform_pointer(args.Out);
    unsigned char *codes = smem + uniform(args.codes), *values = smem + uniform(args.values);
    const uint32_t c16 = lane & 15u, g = lane >> 4;
    // the value of a weight from its pieces
    auto value_of = [&](const unsigned char* row, uint32_t code) {
        if (entry == 2u) return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(row)[code] << 16);
        if (entry == 4u) {
            const uint32_t v = reinterpret_cast<const uint32_t*>(row)[code];
            return fmaf(scale, __uint_as_float(v << 16), scale * __uint_as_float(v & 0xFFFF0000u));
        }
        const uint32_t v = reinterpret_cast<const uint32_t*>(row)[2u * code], w = reinterpret_cast<const uint32_t*>(row)[2u * code + 1u];
        return __uint_as_float(v << 16) + (__uint_as_float(v & 0xFFFF0000u) + __uint_as_float(w << 16));
    };
    const uint32_t col_end = min(a.col0 + a.cols, L);
#pragma unroll 1
    for (uint32_t c0 = a.col0; c0 < col_end; c0 += 32u) {
        floatx4 sum[2][2] = {}, acc[2][2] = {};
        const bool two = c0 + 16u < col_end;
        const uint32_t c[2] = {min(c0 + c16, L - 1u), min(c0 + 16u + c16, L - 1u)};
        uint32_t held = 0;
#pragma unroll 1
        for (uint32_t s0 = a.k_begin; s0 < a.k_end; s0 += seg) {
            const uint32_t steps = (min(a.k_end, s0 + seg) - s0) >> 5;
            __syncthreads();
            for (uint32_t i = tid; i < tiles * stride; i += blockDim.x) reinterpret_cast<uint4*>(codes)[i] = make_uint4(0, 0, 0, 0);
            __syncthreads();
#pragma unroll 1
            for (uint32_t r = a.wave; r < 16u * tiles && a.row0 + r < a.m; r += a.waves) {
                uint32_t rec[4] = {};
#pragma unroll
                for (uint32_t t = 0; t < 4; ++t)
                    if (t <= (a.last_word >> 6)) rec[t] = a.tab[((size_t)(a.row0 + r) << a.shift) + min(t * kWave + lane, a.last_word)];
                uint4 first[Shape::NW];
                request_batch(a.colI, first, uniform(rec[0]) & ~((uint32_t)Shape::PPL - 1u), row_end(rec, a.last_word), lane);
                scatter_row(a.colI, rec, first, a.shift, smem, a.wave, s0, seg, codes + r * stride, lane, [](uint32_t, uint32_t) {});
            }
            __syncthreads();
            float x[2][2][8];
            auto load = [&](uint32_t t, float (&v)[2][8]) {
                const __amdgpu_buffer_rsrc_t xbuf = x_rows(a.X, L, s0 + min(t, steps - 1u) * 32u, n);
#pragma unroll
                for (uint32_t j = 0; j < 2; ++j)
#pragma unroll
                    for (uint32_t i = 0; i < 8; ++i) v[j][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xbuf, ((8u * g + i) * L + c[j]) * 4u, 0, 0));
            };
            auto multiply = [&](uint32_t t, const float (&v)[2][8]) {
#pragma unroll
                for (uint32_t r = 0; r < 2; ++r) {
                    if (r >= tiles) break;
                    const unsigned char* row = values + (16u * r + c16) * row_values;
                    const uint2 q = *reinterpret_cast<const uint2*>(codes + (16u * r + c16) * stride + 32u * t + 8u * g);
                    float w[8];
#pragma unroll
                    for (uint32_t i = 0; i < 8; ++i) w[i] = value_of(row, ((i < 4 ? q.x : q.y) >> (8 * (i & 3))) & 0xFFu);
#pragma unroll
                    for (uint32_t i = 0; i < 8; ++i) {
                        acc[r][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], v[0][i], acc[r][0], 0, 0, 0);
                        if (two) acc[r][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], v[1][i], acc[r][1], 0, 0, 0);
                    }
                }
                if (++held == 2u) {  // sums of 64 columns
                    held = 0;
#pragma unroll
                    for (uint32_t r = 0; r < 2; ++r)
#pragma unroll
                        for (uint32_t j = 0; j < 2; ++j) {
                            sum[r][j] += acc[r][j];
                            acc[r][j] = floatx4{};
                        }
                }
            };
            if (a.wave < steps) load(a.wave, x[0]);
            for (uint32_t t = a.wave; t < steps; t += 2u * a.waves) {
                load(t + a.waves, x[1]);
                multiply(t, x[0]);
                if (t + a.waves >= steps) break;
                load(t + 2u * a.waves, x[0]);
                multiply(t + a.waves, x[1]);
            }
        }
        // the waves' sums meet in LDS as below, 16 columns after the other: [wave][row tile][element][lane]
        float* s_sum = reinterpret_cast<float*>(codes);
        const uint32_t half = a.waves / 2u;
#pragma unroll
        for (uint32_t j = 0; j < 2; ++j) {
            if (j == 1 && !two) break;
#pragma unroll
            for (int upper = 1; upper >= 0; --upper) {
                __syncthreads();
                if ((a.wave >= half) == (upper == 1))
#pragma unroll
                    for (uint32_t r = 0; r < 2; ++r)
#pragma unroll
                        for (uint32_t e = 0; e < 4; ++e)
                            if (r < tiles) {
                                float* at = s_sum + ((a.wave % half * tiles + r) * 4u + e) * kWave + lane;
                                *at = sum[r][j][e] + acc[r][j][e] + (upper == 1 ? 0.f : *at);
                            }
            }
            __syncthreads();
            const uint32_t row = 16u * (tid >> 8) + 4u * g + ((tid >> 6) & 3u), col = c0 + 16u * j + c16;
            if (tid < 256u * tiles && ((rows >> row) & 1u) && a.row0 + row < a.m && col < L) {
                double total = 0;
                for (uint32_t w = 0; w < half; ++w) total += s_sum[w * tiles * 256u + tid];
                out[(size_t)(a.row0 + row) * L + col] = (float)total;
            }
        }
    }
}

}  // namespace
}  // namespace cer
