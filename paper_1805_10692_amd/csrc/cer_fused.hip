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
// 24.1; 2048 x 2048, 256 values, batch 16, four passes of the narrow kernel: 12.0 -> 9.2).  What it pays: every workgroup loads and
// splits all of its X, so that products of many rows and columns stay with the large tiles.
// What a product lasts (4096 x 9216, 32 values, batch 32; 256 workgroups, clocks): arguments and records 3000, X and indices requested,
// bytes cleared 3500, scatter 5300, product 38000 -- X alone, 1.2 MB per compute unit at 36 bytes per clock, takes 33000 --, sums 2000.
// The small ones (786 x 1952, batch 113) are half launch and start-up: 1300, 3000, 4500, 10000, 1000.
#include "cer_exact.hpp"

namespace cer {
namespace {

// Steps of a running sum; the waves' sums are added up in binary64.  Against the decoded route, 31 products, 2-norm of the error, X
// normal and cut at 0: at most 0.92 and 0.93 of its error; with eight steps and a binary32 sum up to 1.11 and 1.07.  Same time.
constexpr uint32_t kFlush = 4;

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

// kTurns: matrix and LDS instructions by turns (the compiler's hint for such loops instead of the fences).  One piece, 16 rows x 32 columns and 16 waves:
// 26 products 0.966 times the time, 0.984 at most (4096 x 9216, 32 values, batch 32 24.5 -> 24.1 us).  Uniform grids, 16 x 48 and 16 x 64: 0.97 to 1.00
// where a workgroup multiplies few columns of W (2994 x 2804, 36 values, 72 31.4 -> 30.6), 1.01 to 1.03 where they are many (1360 x 13925, 12 values,
// 136 65.9 -> 68.0); launch_fused draws the line.  Elsewhere, 26 products of each: one piece 16 x 64 1.026 (1666 x 2968, 4 values, 124 17.8 -> 18.6),
// 32 x 64 1.02, up to 1.08 (1921 x 4736, 32 values, 210 28.7 -> 30.9), 16 x 48 and 32 x 32 1.00; uniform grids 16 x 32 and 32 x 32 1.005; three pieces
// up to 1.07.
template <int kForm, int RT, int CT, int NW, bool kTurns = kForm == 1 && RT == 1 && CT == 2 && NW == 16>
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
                    if constexpr (kTurns) __builtin_amdgcn_iglp_opt(0);
                    else __builtin_amdgcn_sched_barrier(0);
                    multiply(w, x[s]);
                    if constexpr (!kTurns) __builtin_amdgcn_sched_barrier(0);
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

// The sums of the parts of W's columns, in their order, in binary64 (300 x 40000, three pieces, batch 41, X of one
// sign: 3.0e-8 of the 2-norm from fp64 instead of 4.3e-8 when added in binary32).
__global__ __launch_bounds__(256) void fused_sum_kernel(const float* __restrict__ part, float* __restrict__ Y, size_t count, uint32_t splits) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    double a = 0;
    for (uint32_t s = 0; s < splits; ++s) a += part[(size_t)s * count + i];
    Y[i] = (float)a;
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
    FusedKernel turns = nullptr;  // kTurns, where launch_fused chooses between the two
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
    {kUniform, 1, 3, 8, 1.25f, 4.23f, 0.232f, 0.204f, 0.00360f, 0.0939f, cer_fused_kernel<kUniform, 1, 3, 8>, cer_fused_kernel<kUniform, 1, 3, 8, true>},
    {kUniform, 1, 4, 8, 1.33f, 4.55f, 0.240f, 0.248f, 0.00356f, 0.1146f, cer_fused_kernel<kUniform, 1, 4, 8>, cer_fused_kernel<kUniform, 1, 4, 8, true>},
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

int fused_rows(const DeviceView& d, uint32_t L, bool temporaries, double below, double* us) {
    const FusedPlan p = plan_fused(d, L, temporaries, below);
    if (us && p.variant >= 0) *us = p.us;
    return p.variant >= 0 ? 16 * kVariants[p.variant].rt : 0;
}

hipError_t launch_fused(const DeviceView& d, const float* X, float* Y, uint32_t L, bool temporaries, bool dense_zeros, hipStream_t stream) {
    const FusedPlan p = plan_fused(d, L, temporaries, 1e30);
    if (p.variant < 0) return hipErrorInvalidValue;
    const Variant& k = kVariants[p.variant];
    // Turns / fences by columns per workgroup: 16 x 48 854 to 6957 0.976 to 1.000, 12431 and more 1.03; 16 x 64 1195 to 4986 0.973 to 1.000, 5057 to
    // 9448 1.00 to 1.03.
    const bool turns = k.turns != nullptr && std::min<int64_t>(p.kchunk, d.n) <= (k.ct == 3 ? 7000 : 5000);
    const auto kernel = turns ? k.turns : k.kernel;
    {
        static LdsGrant<2 * kVariantCount> grant;
        const hipError_t e = grant.ensure(p.variant + (turns ? kVariantCount : 0), reinterpret_cast<const void*>(kernel), d.lds_per_block);
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
    hipError_t e = launch_kernel(kernel, dim3(eighth * 8u), dim3(k.waves * kWave), p.lds, stream, d.rank_tab, X,
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
