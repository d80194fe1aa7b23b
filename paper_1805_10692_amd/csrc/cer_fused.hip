// Decode + product in one launch: Y = W.X on the bf16 matrix cores with the decoded rows of W in LDS.
//
// Workgroup of 8 or 16 waves: R = 16 RT rows x BN = 16 CT columns of Y over a range of W's columns.  The waves first write, for
// their rows, one byte per element of W into LDS: the number of the element's group among the row's non-empty ones (0: the most
// frequent value).  16 rows of 9216 columns are 144 KiB; a range that does not fit is taken in segments, for each of which the rows'
// indices are read again.  Then the waves share the columns of W, 32 at a time in turn, and multiply: a lane reads eight bytes of one
// row with one LDS read, looks up each one's value as bf16 pieces (cer_split3.hpp) in the row's table in LDS, and loads the same
// eight rows of X straight from memory, CT consecutive columns of each -- column c of the tile is accumulator c % CT of lane c / CT, so
// that the loads are as wide as CT allows and need no transposition.  No barrier and no X in LDS on the way; the waves' sums meet in
// LDS at the end.
//
// Against the two or three launches of decode_tiles_kernel + mfma_product_kernel (+ the sum of the parts) it saves the launches, 2 to 6
// bytes of memory per element of W written and read, and a decoder that waits for its phases (786 x 1952, 32 values, batch 113: 18.9
// -> 11.4 us; 842 x 3509, 190 values, batch 161: 37 -> 23), against the gathers the lines (4096 x 9216, 15 % indexed, batch 32: 28.4 ->
// 23.7; 2048 x 2048, 256 values, batch 16, four passes of the narrow kernel: 12.0 -> 9.2).  What it pays: every workgroup loads and
// splits all of its X, so that products of many rows and columns stay with the large tiles.
// What a product lasts (4096 x 9216, 32 values, batch 32; 256 workgroups, clocks): arguments and records 3000, X and indices requested,
// bytes cleared 3500, scatter 5300, product 38000 -- X alone, 1.2 MB per compute unit at 36 bytes per clock, takes 33000 --, sums 2000.
// The small ones (786 x 1952, batch 113) are half launch and start-up: 1300, 3000, 4500, 10000, 1000.
#include "cer_split3.hpp"
#include "cer_stream.hpp"

namespace cer {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx3 __attribute__((ext_vector_type(3)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

// Steps of a running sum; the waves' sums are added up in binary64.  Against the decoded route, 31 products, 2-norm of the error, X
// normal and cut at 0: at most 0.92 and 0.93 of its error; with eight steps and a binary32 sum up to 1.11 and 1.07.  Same time.
constexpr uint32_t kFlush = 4;
using Shape = GemvShape<uint16_t>;  // windows of 512 positions, three per batch

// What a wave needs first comes as the kernel's first fourteen dwords of arguments, which are in registers when it starts;
// the rest is loaded meanwhile.
struct FusedRest {
    float* Out;
    size_t split_stride;
    uint32_t seg, stride;        // columns of W per segment (a multiple of 32), bytes per row of them
    uint32_t codes, row_values;  // offset of the bytes in LDS, bytes per row of values
    float faint;
    uint32_t dense;              // a zero weight times an infinity counts (exact_dense)
};
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

// The elements of one row in columns c0 .. c0 + seg - 1: row[column - c0] = the number of their group among the row's non-empty ones
// (from 1); row[seg] takes what lies elsewhere.  store(entry, tile): what belongs to group 64 tile + lane + 1 goes to that entry.
// first_batch: the row's first indices, already requested.
// Per window of eight positions and lane: the bitmap's byte says which positions end a group, a table how many do before each
// of them, and the eight numbers come from two additions; two positions' columns are moved and clamped by one instruction.
// 27 vector instructions and 10 of LDS per window -- with a look-up of the rank, comparison and selection per position there were 64 and
// 18, and the scatter of 16 rows of 1380 elements took 7900 clocks in 8 waves instead of 6200 (5300 in 16); now the writes bound it.
template <typename Store>
__device__ __forceinline__ void scatter_row(const uint16_t* colI, const uint32_t (&rec)[4], const uint4 (&first_batch)[Shape::NW], uint32_t tab_shift,
                                            unsigned char* smem, uint32_t wave, uint32_t c0, uint32_t seg, unsigned char* row, uint32_t lane, Store store) {
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
    const uint32_t row_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)row;
    const ushortx2 shift = {(unsigned short)c0, (unsigned short)c0}, dump = {(unsigned short)seg, (unsigned short)seg};
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
            for (int d = 0; d < 4; ++d) {
                const ushortx2 at = __builtin_elementwise_min(__builtin_bit_cast(ushortx2, col[d]) - shift, dump);
                typedef unsigned char __attribute__((address_space(3))) * LdsByte;
                const uint32_t pair = __builtin_bit_cast(uint32_t, at), two = num[d >> 1] >> (16 * (d & 1));
                *reinterpret_cast<LdsByte>((uintptr_t)(row_at + (pair & 0xFFFFu))) = (unsigned char)two;
                *reinterpret_cast<LdsByte>((uintptr_t)(row_at + (pair >> 16))) = (unsigned char)(two >> 8);
            }
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

template <int kForm, int RT, int CT, int NW>
__global__ __launch_bounds__(NW * kWave) void cer_fused_kernel(
    const uint32_t* tab, const float* X, const uint16_t* colI, const float* omega, uint32_t m, uint32_t n, uint32_t L, uint32_t row_magic,
    uint32_t eighth, uint32_t packed, FusedRest rest, UniformGrid grid) {
    constexpr int PW = weight_planes(kForm), kWords = kForm == 3 ? 2 : 1;  // bf16 numbers and dwords per value
    constexpr uint32_t kWaves = NW, kThreads = NW * kWave;
    constexpr uint32_t R = 16 * RT, RW = R / kWaves, BN = 16 * CT;
    constexpr int D = NW == 16 ? 2 : (CT == 1 ? 4 : (CT == 2 ? 3 : 2));  // steps of X in registers: the current one and what is on its way
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid >> 6);
    const uint32_t c16 = lane & 15u, g = lane >> 4;
    // Workgroups are dealt round-robin to the eight XCDs; every XCD takes a contiguous eighth of the items, in which those that
    // share columns of X are neighbours.  packed: columns of W per workgroup / 32 | log2 of the rank table's words per row << 12 |
    // splits << 16; item / row_blocks by multiplication (row_magic = 2^32 / row_blocks rounded up; 0: one block).
    const uint32_t item = (blockIdx.x & 7u) * eighth + (blockIdx.x >> 3), row_blocks = (m + R - 1u) / R;
    const uint32_t over = row_magic ? (uint32_t)(((uint64_t)item * row_magic) >> 32) : item, rt = item - over * row_blocks;
    const uint32_t splits = packed >> 16, tab_shift = (packed >> 12) & 15u, kchunk = (packed & 0xFFFu) * 32u;
    const uint32_t ct = splits == 1u ? over : over / splits, sp = over - ct * splits;
    const uint32_t row0 = rt * R, col0 = ct * BN, k_begin = sp * kchunk, k_end = min((n + 31u) & ~31u, k_begin + kchunk);
    if ((blockIdx.x >> 3) >= eighth || col0 >= L) return;

    // the wave's rows: row0 + RW wave + i; a record has one word per lane and 64 ranks
    const uint32_t last_word = (1u << tab_shift) - 1u, ntiles = (last_word >> 6) + 1u;
    const uint32_t my_row = row0 + RW * wave;
    uint32_t rec[RW][4] = {};
#pragma unroll
    for (uint32_t i = 0; i < RW; ++i)
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t)
            if (t < ntiles) rec[i][t] = tab[((size_t)min(my_row + i, m - 1u) << tab_shift) + min(t * kWave + lane, last_word)];
    const float omega0 = omega[0], value = omega[min(tid, last_word)];  // (behind omega's end lies the rest of the handle)

    // X: a lane takes the rows 8 g .. 8 g + 7 of a step and CT columns of each; the last lanes' columns move back where the batch
    // ends (the same numbers once more, not stored)
    const uint32_t xcol = min(col0 + CT * c16, L - (uint32_t)CT);
    uint32_t xoff[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) xoff[i] = ((8u * g + i) * L + xcol) * 4u;
    float x[D][8][CT];
    auto load_x = [&](uint32_t k0, float (&v)[8][CT]) {
        const __amdgpu_buffer_rsrc_t xbuf = x_rows(X, L, k0, n);
#pragma unroll
        for (int i = 0; i < 8; ++i) load_columns<CT>(xbuf, xoff[i], v[i]);
    };
    floatx4 sum[RT][CT] = {}, acc[RT][CT] = {}, lo[RT][CT] = {};
    uint32_t lost = 0;  // lower half: inputs have bits that their pieces do not reach
    auto joined = [&](int r, int c) {
        floatx4 v = acc[r][c] + lo[r][c];
        if constexpr (kForm == kUniform)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(grid.scale, acc[r][c][e], grid.scale * lo[r][c][e]);
        return v;
    };
    typedef const uintx2 __attribute__((address_space(3))) * LdsU2;
    typedef const typename std::conditional<kForm == 1, uint16_t, uint32_t>::type __attribute__((address_space(3))) * LdsOne;
    unsigned char *codes = nullptr, *values = nullptr;
    uint32_t codes0 = 0, values0 = 0;

    for (uint32_t s0 = k_begin; s0 < k_end;) {
        // the first steps of X and the rows' first indices are requested before the bytes' place in LDS is cleared
        const uint32_t seg = rest.seg, s1 = min(k_end, s0 + seg), steps = (s1 - s0) >> 5;
        // the wave's steps: wave, wave + kWaves, ...
        uint32_t t_load = wave;
        t_load -= t_load >= steps ? steps : 0u;
        const uint32_t mine = wave < steps ? (steps - wave + kWaves - 1u) / kWaves : 0u;
        uint32_t t_read = t_load;
        auto advance = [&](uint32_t t) {  // (behind the end: some step of the segment)
            t += kWaves;
            t -= t >= steps ? steps : 0u;
            return min(t, steps - 1u);
        };
        t_load = t_read = min(t_load, steps - 1u);
        if (s0 == k_begin) {
            if (tid < 256u) {
                uint32_t lo8 = 0, hi8 = 0;
#pragma unroll
                for (uint32_t k = 1; k < 8; ++k) {
                    const uint32_t below = (uint32_t)__builtin_popcount(tid & ((1u << k) - 1u));
                    if (k < 4) lo8 |= below << (8 * k); else hi8 |= below << (8 * (k - 4));
                }
                reinterpret_cast<uint2*>(smem)[tid] = make_uint2(lo8, hi8);
            }
            if (tid < 8u) flag(smem, (int)tid) = 0u;
            codes = smem + rest.codes;
            values = smem + values_at(kWaves, tab_shift, entry_bytes(kForm));
            codes0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)codes + c16 * rest.stride + 8u * g;
            values0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)values + c16 * rest.row_values;
        } else {
            __syncthreads();  // the bytes of the segment before have been read
        }
        const double inverse = grid.inverse;
        if constexpr (kForm == kUniform) asm volatile("" ::"s"(inverse));  // (loaded with the other arguments)
        for (uint32_t i = tid; i < R * rest.stride / 16u; i += kThreads) reinterpret_cast<uint4*>(codes)[i] = make_uint4(0, 0, 0, 0);
        uint4 first[RW][Shape::NW];
#pragma unroll
        for (uint32_t i = 0; i < RW; ++i)
            request_batch(colI, first[i], uniform(rec[i][0]) & ~((uint32_t)Shape::PPL - 1u), row_end(rec[i], last_word), lane);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s + 1 < D; ++s) {
            load_x(s0 + t_load * 32u, x[s]);
            t_load = advance(t_load);
        }
        __builtin_amdgcn_sched_barrier(0);
        unsigned char* table = smem + table_at(kWaves);
        if (s0 == k_begin && tid <= last_word) {
            uint32_t p[3];
            if constexpr (kForm != kUniform) split3_finite(value, p);
            if constexpr (kForm == 1) reinterpret_cast<uint16_t*>(table)[tid] = (uint16_t)p[0];
            else if constexpr (kForm == kUniform) reinterpret_cast<uint32_t*>(table)[tid] = uniform_pieces(value, grid);
            else reinterpret_cast<uint2*>(table)[tid] = make_uint2(p[0] | (p[1] << 16), p[2]);
        }
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < RW; ++i)
            if (my_row + i < m) {
                const uint32_t r = RW * wave + i;
                // (the values are read before any is stored: one trip to LDS)
                unsigned char* v = values + r * rest.row_values;
                typedef typename std::conditional<kForm == 1, uint16_t, typename std::conditional<kForm == kUniform, uint32_t, uint2>::type>::type Entry;
                Entry own[4] = {}, zero = reinterpret_cast<const Entry*>(table)[0];
#pragma unroll
                for (uint32_t t = 0; t < 4; ++t)
                    if (t < ntiles) own[t] = reinterpret_cast<const Entry*>(table)[min(t * kWave + lane + 1u, last_word)];
                if (lane == 0) {
                    reinterpret_cast<Entry*>(v)[0] = zero;
                    if (omega0 == 0.f && uniform(rec[i][0]) == row_end(rec[i], last_word)) atomicOr(&flag(smem, kEmpty), 1u << r);
                }
                scatter_row(colI, rec[i], first[i], tab_shift, smem, wave, s0, seg, codes + r * rest.stride, lane,
                            [&](uint32_t at, uint32_t t) { reinterpret_cast<Entry*>(v)[at] = own[t]; });
            }
        __syncthreads();
        // Weights take two trips to LDS, the eight ranks and their values: the ranks are read two steps ahead, the values one.
        auto ranks_of = [&](uintx2 (&q)[RT]) {
#pragma unroll
            for (int r = 0; r < RT; ++r) q[r] = *reinterpret_cast<LdsU2>((uintptr_t)(codes0 + (uint32_t)r * 16u * rest.stride + t_read * 32u));
            t_read = advance(t_read);
        };
        auto values_of = [&](const uintx2 (&q)[RT], uint32_t (&e)[RT][8][kWords]) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    // the entry's address: one byte times the size of an entry, plus the row's base (a dot product of bytes)
                    const uint32_t at = __builtin_amdgcn_udot4(q[r][i >> 2], entry_bytes(kForm) << (8 * (i & 3)), values0 + (uint32_t)r * 16u * rest.row_values, false);
                    if constexpr (kWords == 1) {
                        e[r][i][0] = *reinterpret_cast<LdsOne>((uintptr_t)at);
                    } else {
                        const uintx2 v = *reinterpret_cast<LdsU2>((uintptr_t)at);
                        e[r][i][0] = v[0];
                        e[r][i][1] = v[1];
                    }
                }
            }
        };
        auto pack = [&](const uint32_t (&e)[RT][8][kWords], uint4 (&w)[RT][PW]) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                uint32_t o[PW][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (kForm == 1) {
                        o[0][i] = e[r][2 * i][0] | e[r][2 * i + 1][0] << 16;
                    } else {
                        o[0][i] = __builtin_amdgcn_perm(e[r][2 * i + 1][0], e[r][2 * i][0], 0x05040100u);
                        o[1][i] = __builtin_amdgcn_perm(e[r][2 * i + 1][0], e[r][2 * i][0], 0x07060302u);
                        if constexpr (kForm == 3) o[2][i] = __builtin_amdgcn_perm(e[r][2 * i + 1][kWords - 1], e[r][2 * i][kWords - 1], 0x05040100u);
                    }
                }
#pragma unroll
                for (int p = 0; p < PW; ++p) w[r][p] = make_uint4(o[p][0], o[p][1], o[p][2], o[p][3]);
            }
        };
        auto multiply = [&](const uint4 (&w)[RT][PW], const float (&v)[8][CT]) {
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                float xc[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) xc[i] = v[i][c];
                uint4 b[3];
                split3_8_dot(xc, b, lost);
                // as mfma_pieces: the small products have a sum of their own
#pragma unroll
                for (int s = 2; s >= 0; --s)
#pragma unroll
                    for (int i = 0; i < PW; ++i)
                        if (s - i >= 0 && !(kForm == kUniform && i == 1 && s == 2))
#pragma unroll
                            for (int r = 0; r < RT; ++r) {
                                floatx4& to = s > 0 ? lo[r][c] : acc[r][c];
                                to = mfma16(w[r][i], b[s - i], to);
                            }
            }
        };
        if (mine > 0) {
            uintx2 q[RT];
            uint32_t e[RT][8][kWords];
            uint4 w[RT][PW];
            ranks_of(q);
            values_of(q, e);
            ranks_of(q);
            pack(e, w);
            uint32_t left = mine, held = 0;
            for (;;) {
#pragma unroll
                for (int s = 0; s < D; ++s) {
                    load_x(s0 + t_load * 32u, x[(s + D - 1) % D]);
                    t_load = advance(t_load);
                    values_of(q, e);
                    ranks_of(q);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(w, x[s]);
                    __builtin_amdgcn_sched_barrier(0);
                    pack(e, w);
                    if (--left == 0) break;
                }
                if (left == 0) break;
                if (PW > 1 && (held += D) >= kFlush) {
                    held = 0;
#pragma unroll
                    for (int r = 0; r < RT; ++r)
#pragma unroll
                        for (int c = 0; c < CT; ++c) {
                            sum[r][c] += joined(r, c);
                            acc[r][c] = lo[r][c] = floatx4{};
                        }
                }
            }
        }
        s0 = s1;
    }
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[r][c] = sum[r][c] + joined(r, c);

    // the waves' sums meet in LDS, first the upper half's, then all: [wave][row tile][element][column of CT][lane]
    float* s_sum = reinterpret_cast<float*>(codes);
    constexpr uint32_t kPer = RT * CT * 4 * kWave;
    if (__ballot((lost & 0xFFFFu) != 0u) != 0ull && lane == 0) atomicOr(&flag(smem, kLossy), 1u);
    __syncthreads();
    constexpr uint32_t kHalf = kWaves / 2;
    if (wave >= kHalf) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < CT; ++c) s_sum[(wave - kHalf) * kPer + ((r * 4 + e) * CT + c) * kWave + lane] = acc[r][c][e];
    }
    __syncthreads();
    if (wave < kHalf) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < CT; ++c) s_sum[wave * kPer + ((r * 4 + e) * CT + c) * kWave + lane] += acc[r][c][e];
    }
    __syncthreads();
    // accumulator element e of lane l: row 4 (l / 16) + e, column l % 16
    constexpr uint32_t kVec = RT * 4 * kWave / kThreads > 0 ? RT * 4 * kWave / kThreads : 1;
    // What is formed once more: sums that are not finite, subnormal ones (the pieces' products are rounded apart there), and where an input
    // has lost bits the faint ones, but of rows without elements.
    const uint32_t empty = flag(smem, kEmpty);
    const float least = flag(smem, kLossy) != 0u ? rest.faint : 0.f;
    float y[kVec][CT];
#pragma unroll
    for (uint32_t q = 0; q < kVec; ++q) {
        const uint32_t i = tid + q * kThreads, re = i >> 6, r = 16u * (re >> 2) + 4u * g + (re & 3u);
        if (i < RT * 4u * kWave) {
            bool odd = false, faint = false;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const float* s = s_sum + (re * CT + c) * kWave + lane;
                float part[kHalf];
#pragma unroll
                for (uint32_t h = 0; h < kHalf; ++h) part[h] = s[h * kPer];
                double total = part[0];
#pragma unroll
                for (uint32_t h = 1; h < kHalf; ++h) total += part[h];
                y[q][c] = (float)total;
                const float size = fabsf(y[q][c]);
                odd |= !(size < INFINITY);
                faint |= size < least || (size < 0x1p-126f && size > 0.f);
            }
            if (odd && row0 + r < m) atomicOr(&flag(smem, kOdd), 1u << r);
            if (faint && row0 + r < m && !((empty >> r) & 1u)) atomicOr(&flag(smem, kFaint), 1u << r);
        }
    }
    __syncthreads();
    const uint32_t odd = flag(smem, kOdd), faint = flag(smem, kFaint);
    float* out = rest.Out + sp * rest.split_stride;
#pragma unroll
    for (uint32_t q = 0; q < kVec; ++q) {
        const uint32_t i = tid + q * kThreads, re = i >> 6, r = 16u * (re >> 2) + 4u * g + (re & 3u), row = row0 + r;
        if (i < RT * 4u * kWave && row < m) {
            const uint32_t first = col0 + CT * c16;
#pragma unroll
            for (int c = 0; c < CT; ++c)
                if (xcol + c >= first) out[(size_t)row * L + xcol + c] = y[q][c];
        }
    }
    if ((odd | faint) != 0u) {
        static_assert(sizeof(ExactArgs) <= kListsAt - kCallAt, "place of the arguments");
        if (tid == 0)
            *reinterpret_cast<ExactArgs*>(smem + kCallAt) =
                ExactArgs{out, tab, colI, omega, X, grid.scale, m, n, L, tab_shift, entry_bytes(kForm), row0, R, col0, BN, k_begin, k_end,
                          rest.seg, rest.stride, rest.codes, values_at(kWaves, tab_shift, entry_bytes(kForm)), rest.row_values};
        __syncthreads();
        const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
        uint32_t rows = uniform(odd);
        if (faint != 0u) rows |= lossy_rows(lds, uniform(faint));
        if (rows != 0u) {
            if (rest.dense) exact_dense(lds, rows); else exact_gathered(lds, rows);
        }
    }
}

// The sums of the parts of W's columns, in their order.
__global__ __launch_bounds__(256) void fused_sum_kernel(const float* __restrict__ part, float* __restrict__ Y, size_t count, uint32_t splits) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    float a = 0.f;
    for (uint32_t s = 0; s < splits; ++s) a += part[(size_t)s * count + i];
    Y[i] = a;
}

typedef void (*FusedKernel)(const uint32_t*, const float*, const uint16_t*, const float*, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t,
                            uint32_t, FusedRest, UniformGrid);

// The variants, and the terms of their duration in microseconds, fitted to 450 random products of 2 to 800 columns (the typical
// deviation is 3 %, one in ten is off by more than 8 %).  A launch takes `fixed`; then the busiest compute unit's workgroups follow
// one another, each `round`, `list` per row, 64 ranks and wave, `batch` per wave and 1536 positions (rows of several segments are read
// several times), `pos` per 64 positions and `step` per 32 columns of W.
// The uniform form's steps are 7 % shorter than three pieces' (two tables' words and six products become one and four: 1972 x 4004, 135
// values, batch 55: 23.0 -> 21.7 us, 883 x 11262, batch 35: 25.8 -> 24.5).
// Which of them are worth having: without 16 waves for 16 columns 3 % are lost on average, without the tile of 48 columns 4 %,
// of 64 3 %, of 32 2 %, without the two tiles of 32 rows 0.8 %.
struct Variant {
    uint8_t form, rt, ct, waves;
    float fixed, round, list, batch, pos, step;
    FusedKernel kernel;
};
const Variant kVariants[] = {
    {1, 1, 1, 16, 1.11f, 3.74f, 0.404f, 0.260f, 0.00290f, 0.0344f, cer_fused_kernel<1, 1, 1, 16>},
    {1, 1, 2, 16, 1.38f, 4.77f, 0.212f, 0.364f, 0.00232f, 0.0640f, cer_fused_kernel<1, 1, 2, 16>},
    {1, 1, 3, 8, 1.46f, 4.13f, 0.216f, 0.114f, 0.00409f, 0.0816f, cer_fused_kernel<1, 1, 3, 8>},
    {1, 1, 4, 8, 1.35f, 4.75f, 0.159f, 0.227f, 0.00360f, 0.0977f, cer_fused_kernel<1, 1, 4, 8>},
    {1, 2, 2, 8, 1.88f, 5.47f, 0.231f, 0.154f, 0.00401f, 0.0945f, cer_fused_kernel<1, 2, 2, 8>},
    {1, 2, 4, 8, 1.73f, 5.94f, 0.250f, 0.178f, 0.00407f, 0.1341f, cer_fused_kernel<1, 2, 4, 8>},
    {3, 1, 1, 16, 1.27f, 3.55f, 0.356f, 0.239f, 0.00310f, 0.0467f, cer_fused_kernel<3, 1, 1, 16>},
    {3, 1, 2, 8, 1.30f, 4.15f, 0.257f, 0.292f, 0.00309f, 0.0785f, cer_fused_kernel<3, 1, 2, 8>},
    {3, 1, 3, 8, 1.25f, 4.23f, 0.232f, 0.204f, 0.00360f, 0.1010f, cer_fused_kernel<3, 1, 3, 8>},
    {3, 1, 4, 8, 1.33f, 4.55f, 0.240f, 0.248f, 0.00356f, 0.1232f, cer_fused_kernel<3, 1, 4, 8>},
    {3, 2, 2, 8, 1.34f, 4.84f, 0.271f, 0.403f, 0.00262f, 0.1261f, cer_fused_kernel<3, 2, 2, 8>},
    {kUniform, 1, 1, 16, 1.27f, 3.55f, 0.356f, 0.239f, 0.00310f, 0.0434f, cer_fused_kernel<kUniform, 1, 1, 16>},
    {kUniform, 1, 2, 8, 1.30f, 4.15f, 0.257f, 0.292f, 0.00309f, 0.0730f, cer_fused_kernel<kUniform, 1, 2, 8>},
    {kUniform, 1, 3, 8, 1.25f, 4.23f, 0.232f, 0.204f, 0.00360f, 0.0939f, cer_fused_kernel<kUniform, 1, 3, 8>},
    {kUniform, 1, 4, 8, 1.33f, 4.55f, 0.240f, 0.248f, 0.00356f, 0.1146f, cer_fused_kernel<kUniform, 1, 4, 8>},
    {kUniform, 2, 2, 8, 1.34f, 4.84f, 0.271f, 0.403f, 0.00262f, 0.1173f, cer_fused_kernel<kUniform, 2, 2, 8>},
};
constexpr int kVariantCount = sizeof(kVariants) / sizeof(kVariants[0]);

// Products of fewer workgroups leave four fifths of the compute units without work and are left to the other kernels: of 450 random
// products one would gain (371 x 1668, batch 20: 13.6 -> 7.6 us).
constexpr uint32_t kFewestTiles = 48;

struct FusedPlan {
    int variant = -1;
    uint32_t row_blocks = 0, col_tiles = 0, splits = 1, kchunk = 0, seg = 0, codes = 0, row_values = 0;
    size_t lds = 0;
    double us = 1e30;
};

// The best plan of less than `below` microseconds.
FusedPlan plan_fused(const DeviceView& d, uint32_t L, bool temporaries, double below) {
    FusedPlan best;
    best.us = below;
    // 16-bit column indices, one of which (65535) stands for none; X is addressed with 32-bit offsets
    if (!d.rank_tab || d.pieces < 1 || d.colI_bits != 16 || d.n < 1 || d.n > 65000 || d.m < 1 || d.m > (1 << 24) || L < 2 || L > (1u << 20) ||
        ((uint64_t)d.n + 64) * L * 4u >= (1ull << 32))
        return best;
    const int form = d.grid.scale != 0.f ? kUniform : (d.pieces == 1 ? 1 : 3);
    const uint32_t entry = entry_bytes(form), shift = (uint32_t)d.rank_tab_shift;
    const uint32_t row_values = (((1u << shift) + 1u) * entry + 3u) & ~3u;
    const uint32_t steps = (uint32_t)((d.n + 31) / 32), budget = (uint32_t)std::min<size_t>(d.lds_per_block - 256, 160 * 1024);
    const double row = (double)d.nnz / (double)d.m, batches = std::ceil((row + 8.0) / Shape::BATCH), lists = std::max(1u, (1u << shift) / 64u);
    for (int v = 0; v < kVariantCount; ++v) {
        const Variant& k = kVariants[v];
        if (k.form != form || k.fixed + k.round > best.us || k.ct > L || (k.ct > 1 && 8u * k.ct >= L)) continue;  // a tile of half the width holds the batch
        FusedPlan p;
        p.variant = v;
        const uint32_t R = 16u * k.rt;
        p.row_blocks = (uint32_t)((d.m + R - 1) / R);
        p.col_tiles = (L + 16u * k.ct - 1) / (16u * k.ct);
        p.row_values = row_values;
        p.codes = (values_at(k.waves, shift, entry) + R * row_values + 15u) & ~15u;
        const size_t sums = (size_t)k.rt * k.ct * 512u * k.waves;
        if (p.codes + std::max<size_t>(R * 48u, sums) > budget) continue;
        const uint32_t most = ((budget - p.codes) / R - 16u) / 32u;  // steps per segment
        const uint64_t tiles = (uint64_t)p.row_blocks * p.col_tiles;
        if (tiles < kFewestTiles) continue;
        if (tiles * 8u * p.row_blocks >= (1ull << 32)) continue;  // (the kernel divides by multiplication)
        for (uint32_t sp = 1; sp <= (temporaries ? 8u : 1u); ++sp) {
            if (sp > 1 && (steps < 16u * sp || tiles * (sp - 1) >= (uint64_t)d.cus)) break;
            const uint32_t per = (steps + sp - 1) / sp;
            p.splits = (steps + per - 1) / per;
            const double part_bytes = (double)p.splits * (double)d.m * L * 4.0;
            if (p.splits > 1 && part_bytes > (double)(1ull << 30)) break;
            const uint32_t segs = (per + most - 1) / most;
            p.kchunk = per * 32u;
            p.seg = (per + segs - 1) / segs * 32u;
            p.lds = p.codes + std::max<size_t>((size_t)R * (p.seg + 16u), sums);
            const double rounds = std::ceil((double)(tiles * p.splits) / std::max(d.cus, 1));
            const double rows = (double)R * segs;
            // (a row is one wave's: rows of unequal length wait for the longest)
            const double positions = std::max(rows * row / 64.0 * k.pos, segs * d.longest_row / 64.0 * 0.035);
            p.us = k.fixed + rounds * (k.round + rows / k.waves * (lists * k.list + batches * k.batch) + positions + per * k.step);
            if (p.splits > 1) p.us += 2.1 + (part_bytes + (double)d.m * L * 4.0) * 0.9e-6;  // the second launch
            if (p.us < best.us) best = p;
        }
    }
    return best;
}

}  // namespace

int fused_rows(const DeviceView& d, uint32_t L, bool temporaries, double below) {
    const FusedPlan p = plan_fused(d, L, temporaries, below);
    return p.variant >= 0 ? 16 * kVariants[p.variant].rt : 0;
}

hipError_t launch_fused(const DeviceView& d, const float* X, float* Y, uint32_t L, bool temporaries, bool dense_zeros, hipStream_t stream) {
    const FusedPlan p = plan_fused(d, L, temporaries, 1e30);
    if (p.variant < 0) return hipErrorInvalidValue;
    const Variant& k = kVariants[p.variant];
    {
        static LdsGrant<kVariantCount> grant;
        const hipError_t e = grant.ensure(p.variant, reinterpret_cast<const void*>(k.kernel), d.lds_per_block);
        if (e != hipSuccess) return e;
    }
    FusedRest a;
    a.seg = p.seg;
    a.stride = p.seg + 16u;
    a.codes = p.codes;
    a.row_values = p.row_values;
    a.split_stride = (size_t)d.m * L;
    // as in launch_mfma: less than 2^-26 of a sum from here on
    a.faint = (float)std::min((double)d.n * d.omega_max * 0x1p-108, 1e38);
    a.dense = dense_zeros ? 1u : 0u;
    float* part = nullptr;
    if (p.splits > 1) {
        const hipError_t e = (hipError_t)temp_alloc(reinterpret_cast<void**>(&part), a.split_stride * p.splits * 4u, stream);
        if (e != hipSuccess) return e;
    }
    a.Out = part ? part : Y;
    const uint32_t items = p.row_blocks * p.col_tiles * p.splits, eighth = (items + 7u) / 8u;
    const uint32_t magic = p.row_blocks == 1 ? 0u : (uint32_t)(((1ull << 32) + p.row_blocks - 1) / p.row_blocks);
    const uint32_t packed = p.kchunk / 32u | (uint32_t)d.rank_tab_shift << 12 | p.splits << 16;
    hipError_t e = launch_kernel(k.kernel, dim3(eighth * 8u), dim3(k.waves * kWave), p.lds, stream, d.rank_tab, X,
                                 static_cast<const uint16_t*>(d.colI), d.omega, (uint32_t)d.m, (uint32_t)d.n, L, magic, eighth, packed, a, d.grid);
    if (part) {
        if (e == hipSuccess)
            e = launch_kernel(fused_sum_kernel, dim3((uint32_t)((a.split_stride + 255) / 256)), dim3(256), 0, stream, part, Y, a.split_stride,
                              p.splits);
        const hipError_t f = (hipError_t)temp_free(part, stream);
        if (e == hipSuccess) e = f;
    }
    return e;
}

}  // namespace cer
