// Decode + matrix-core product: Y = W.X with the decoded matrix as bf16 pieces (cer_split3.hpp) and X split into its three
// pieces on the way into LDS.
//
// Workgroup of 256 rows x BN columns of Y, k steps of BK = 2048 / BN: four waves of 64 rows each (codebooks of one piece), or eight of 32.
// W's pieces go from memory straight into the registers of the wave that owns the rows: the decoder has left them in operand
// order, a tile of 32 rows x 16 columns in 1 KiB (row-major pieces cost four times as many cache lines per load and ran at 40 %
// of this speed) -- or its ranks, which the wave looks up in LDS (multiplies_ranks).  X is loaded as fp32, eight or four rows of one column per thread, split, and stored to LDS as
// [piece][k / 8][column][8], so that the operand reads are 16 bytes per lane at consecutive addresses.  X is loaded several steps
// ahead, W one step, and the LDS stores go one or two steps ahead into other buffers: one barrier per step, no branch in between
// (rows of X behind the last one read as zeros: buffer loads with bounds).
// Counters for 512 x 4608, batch 3136, one piece (42 us, 1050 TFLOP/s of bf16; 10 TB/s from L2): matrix pipes busy 59 % of the launch,
// vector ALU 28 % (the splitting), LDS 22 %, no bank conflicts; a wave waits 48 % of its time to issue and 16 % for data -- two waves
// per SIMD that meet at the matrix pipe, and a barrier per step.  Two workgroups of four waves, whose barriers do not meet, are
// worth 10 us there against one of eight waves of 32 rows (52 us: the operands of X are read twice as often), and as much as one of
// 512 rows (42 us; but 481 x 6989, batch 1415, 61 us the call instead of 45).  With more pieces the sums take twice the registers, and a
// SIMD held one wave of 64 rows: two of 32 took 4 - 14 % off the call (703 x 12909, 72 values, batch 449, 70 -> 64 us; 1549 x 4734, 203
// values, batch 548, 60 -> 54; 2271 x 744, three pieces, batch 2961, 87 -> 78).
#include "cer_device.hpp"
#include "cer_split3.hpp"

namespace cer {
namespace {

constexpr uint32_t kFlush = 256;  // (kUniform twice that: its flush rounds once more, its large products are short; 2-norm of the error 2 - 5 % less)

// The two sums of mfma_pieces together.  kUniform: times the scale, with one rounding of the larger.
template <int kForm>
__device__ __forceinline__ floatx16 joined(floatx16 hi, floatx16 lo, float scale) {
    if constexpr (kForm == 1) return hi;
    if constexpr (kForm != kUniform) return hi + lo;
#pragma unroll
    for (int e = 0; e < 16; ++e) hi[e] = fmaf(scale, hi[e], scale * lo[e]);
    return hi;
}

// kByRank: W comes as one byte per element, and what the matrix cores multiply is looked up in LDS: a word per rank (two pieces; one in the
// lower half) or two (three), a copy of the table per bank, so that 64 lanes with any ranks read without conflicts.
// The table of 256 ranks takes 32 KiB: 32 copies of words, 16 of pairs of words.
constexpr uint32_t kTableWords = 256 * 32, kTableStep = 128;  // bytes from one rank to the next
template <int kForm>
__device__ __forceinline__ void fill_table(uint32_t* table, const float* __restrict__ omega, uint32_t K, const UniformGrid& grid, uint32_t tid, uint32_t threads) {
    // eight threads per rank, 16 bytes each
    for (uint32_t i = tid; i < 8u * K; i += threads) {
        const float w = omega[i >> 3];
        uint32_t p[3];
        uint4 q;
        if constexpr (kForm == kUniform) {
            p[0] = uniform_pieces(w, grid);
            q = make_uint4(p[0], p[0], p[0], p[0]);
        } else {
            split3_finite(w, p);
            const uint32_t two = p[0] | (p[1] << 16);
            if constexpr (weight_planes(kForm) == 3) q = make_uint4(two, p[2], two, p[2]);
            else q = make_uint4(two, two, two, two);
        }
        reinterpret_cast<uint4*>(table)[i] = q;
    }
}
// Address of this lane's copy.
template <int kForm>
__device__ __forceinline__ uint32_t table_of(const uint32_t* table, uint32_t lane) {
    typedef const uint32_t __attribute__((address_space(3))) * LdsWord;
    return (uint32_t)(uintptr_t)(LdsWord)table + (weight_planes(kForm) == 3 ? (lane & 15u) * 8u : (lane & 31u) * 4u);
}
// Eight ranks -> the operand registers.
template <int kForm>
__device__ __forceinline__ void look_up(uint32_t mine, uint32_t four0, uint32_t four1, uint4 (&a)[weight_planes(kForm)]) {
    typedef const uint32_t __attribute__((address_space(3))) * LdsWord;
    typedef uint32_t Pair __attribute__((ext_vector_type(2)));
    typedef const Pair __attribute__((address_space(3))) * LdsPair;
    constexpr int PW = weight_planes(kForm);
    uint32_t e[8], f[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // (one byte times the distance of the entries, a dot product of bytes)
        const uint32_t at = __builtin_amdgcn_udot4(i < 4 ? four0 : four1, kTableStep << (8 * (i & 3)), mine, false);
        if constexpr (PW == 3) {
            const Pair q = *reinterpret_cast<LdsPair>((uintptr_t)at);
            e[i] = q.x;
            f[i] = q.y;
        } else {
            e[i] = *reinterpret_cast<LdsWord>((uintptr_t)at);
        }
    }
    uint32_t w[PW][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[0][i] = __builtin_amdgcn_perm(e[2 * i + 1], e[2 * i], 0x05040100u);
        if constexpr (PW > 1) w[1][i] = __builtin_amdgcn_perm(e[2 * i + 1], e[2 * i], 0x07060302u);
        if constexpr (PW > 2) w[2][i] = __builtin_amdgcn_perm(f[2 * i + 1], f[2 * i], 0x05040100u);
    }
#pragma unroll
    for (int p = 0; p < PW; ++p) a[p] = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
}

// What a workgroup of either kernel below was given.
struct Block {
    const uint16_t* W;
    const float* X;
    float* Out;
    size_t plane;
    uint32_t m, n, L, pitch, row0, rows, col0, cols, k_begin, k_end, threads;
    float scale;  // kUniform
    const float* omega;  // kByRank
    uint32_t K;
};

// Products in binary32, the pieces of W added up again: the workgroup's outputs once more, over the ones from the matrix cores.
// Called (by all threads, through a barrier) where X holds infinities, NaNs or numbers that round to infinity (must: some thread
// has met one), and where a sum is faint -- so small that what the pieces of small inputs lose can show.  Faint sums alone
// are mostly those of empty rows: the inputs are looked at first (odd: this thread's inputs had third pieces; without them nothing
// is lost), those of the columns with faint sums (small: a bit per 32 columns, this lane's; looking at all of the workgroup's for a
// single sum took 10 of 48 us: 1204 x 10213, 224 values, batch 245).  A function of its own, and behind the stores, so that nothing of it is
// held in registers while the matrix cores work, nor fetched by those who do not come here (2 of 19 us: 506 x 987, batch 1870).  Small inputs could also be caught on their way: a tenth more for
// 512 x 4608, batch 3136.
// A wave takes tiles of 32 x 32 outputs, 64 or 32 columns of W per step, straight from memory; sums of kFlush columns as below.  Product of
// 512 x 4608, batch 3136, one-piece codebook: 68 us, 80 with empty rows, 247 with an infinity in X, 331 with X of about 2^-120.
template <int kForm, bool kByRank>
__device__ __attribute__((noinline)) void exact_block(const Block b, bool must, bool odd, uint32_t small) {
    constexpr int PW = weight_planes(kForm), NS = kForm == kUniform ? 2 : 4, PR = kByRank ? 1 : PW;  // 16 NS columns of W per step
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
    if (!__syncthreads_or(must)) {
        if (!__syncthreads_or(odd)) return;
        uint32_t at = tid % b.cols, step = b.threads / b.cols, begin = tid / b.cols;
        if (__syncthreads_count(small != 0u) < 16) {
            // few columns: those alone, by all threads (a few sums in a hundred million come out as zero by themselves: most launches
            // meet none, some one)
            __shared__ uint32_t s_small[2];
            if (tid < 2u) s_small[tid] = 0u;
            __syncthreads();
#pragma unroll
            for (uint32_t j = 0; j < 2; ++j)
                if ((small >> j) & 1u) atomicOr(&s_small[j], 1u << (lane & 31u));
            __syncthreads();
            uint64_t columns = s_small[0] | (uint64_t)s_small[1] << 32;
            const uint32_t count = (uint32_t)__popcll(columns), across = pow2_ceil(count);
            for (uint32_t i = tid % across % count; i > 0u; --i) columns &= columns - 1u;
            at = (uint32_t)__builtin_ctzll(columns);
            step = b.threads / across;
            begin = tid / across;
        }
        const uint32_t xcol = min(b.col0 + at, b.L - 1u), last = min(b.k_end, b.n) - 1u;
        bool some = false;
        for (uint32_t k0 = b.k_begin + begin; k0 < b.k_end; k0 += 16u * step) {
            float x[16];
#pragma unroll
            for (uint32_t i = 0; i < 16; ++i) x[i] = b.X[(size_t)min(k0 + i * step, last) * b.L + xcol];
#pragma unroll
            for (int i = 0; i < 16; ++i) some |= split_lossy(x[i]);
        }
        if (!__syncthreads_or(some)) return;
    }
    const uint32_t across = b.cols / 32u;
    for (uint32_t t = wave; t < b.rows / 32u * across; t += b.threads / kWave) {
        const uint32_t row32 = b.row0 + t / across * 32u, c = b.col0 + t % across * 32u + (lane & 31u);
        if (row32 >= b.m) break;
        const uint16_t* w = b.W + (size_t)(row32 >> 5) * (kByRank ? 16 : 32) * b.pitch;
        const uint32_t xoff = (8u * half * b.L + min(c, b.L - 1u)) * 4u;
        floatx16 sum = {}, acc = {};
        uint32_t held = 0;
        for (uint32_t k0 = b.k_begin; k0 < b.k_end; k0 += 16u * NS) {  // behind the end: zeros of X, W's last columns once more
            float x[NS][8];
            uint4 q[NS][PR];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const __amdgpu_buffer_rsrc_t xbuf = x_rows(b.X, b.L, k0 + 16 * s, min(b.n, b.k_end));
#pragma unroll
                for (int i = 0; i < 8; ++i) x[s][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xbuf, xoff + i * b.L * 4u, 0, 0));
                if constexpr (kByRank) {
                    if (s % 2 == 0) q[s][0] = reinterpret_cast<const uint4*>(w + (size_t)min(k0 + 16 * s, b.pitch - 32u) * 16)[lane];
                } else {
#pragma unroll
                    for (int p = 0; p < PW; ++p) q[s][p] = reinterpret_cast<const uint4*>(w + p * b.plane + (size_t)min(k0 + 16 * s, b.pitch - 16u) * 32)[lane];
                }
            }
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    float v = 0.f;  // the codebook's value: a binary32 number
                    if constexpr (kByRank) {
                        const uint4& r = q[s & ~1][0];
                        const uint32_t u = i < 4 ? (s & 1 ? r.z : r.x) : (s & 1 ? r.w : r.y);
                        v = b.omega[min((u >> (8 * (i & 3))) & 0xFFu, b.K - 1u)];  // (rows behind the last one: any byte)
                    } else {
#pragma unroll
                        for (int p = PW - 1; p >= 0; --p) {
                            const uint32_t u = i < 4 ? (i < 2 ? q[s][p].x : q[s][p].y) : (i < 6 ? q[s][p].z : q[s][p].w);
                            const float piece = __uint_as_float(i & 1 ? u & 0xFFFF0000u : u << 16);
                            v = kForm == kUniform ? fmaf(b.scale, piece, v) : v + piece;
                        }
                    }
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v, x[s][i], acc, 0, 0, 0);
                }
            if ((held += 16u * NS) >= kFlush) {
                held = 0;
                sum += acc;
                acc = floatx16{};
            }
        }
        sum += acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t r = row32 + 8 * (e / 4) + 4 * half + (e % 4);
            if (r < b.m && c < b.L) b.Out[(size_t)r * b.L + c] = sum[e];
        }
    }
}

constexpr int mfma_waves(int form) { return form == 1 ? 4 : 8; }

template <int kForm, bool kByRank, int TN>
struct MfmaTile {
    static constexpr int PW = weight_planes(kForm), NW = mfma_waves(kForm);
    static constexpr int TM = kForm == 1 ? 2 : 1, BM = 32 * TM * NW, BN = 32 * TN, BK = 2048 / BN, KG = BK / 8, KS = BK / 16;
    // Steps of X in registers; steps that its stores are ahead (two: the next step's first operands are read before the barrier, where there
    // are registers for them) and its loads; rows of X per thread and step, threads per eight of them.
    static constexpr int D = 4, kAhead = kForm == 1 ? 1 : 2, kFetch = D - 3 + 2 * kAhead, kBuffers = 2 * kAhead, XR = 32 / NW, XP = 8 / XR;
    uint4 b[kBuffers][3][KG][BN];
    uint32_t table[kByRank ? kTableWords : 1];

    // sum: what is finished; acc: the sum over the current kFlush columns or so (a running sum of thousands of terms would
    // round each of them to the size of the whole).  Returns a NaN if this thread's share of X holds numbers without pieces, and
    // 0 if none of them has a third piece.
    __device__ __forceinline__ float run(const uint16_t* const (&wtile)[TM], size_t plane, const float* X, uint32_t n, uint32_t L,
                                         uint32_t col0, uint32_t k_begin, uint32_t k_end, floatx16 (&sum)[TM][TN], float scale) {
        const uint32_t tid = threadIdx.x, lane = tid & 63u;
        // this thread's share of X: rows 8 xg + XR xp .. of a step, one column
        const uint32_t xp = tid % XP, xc = tid / XP % BN, xg = tid / XP / BN, xcol = min(col0 + xc, L - 1u);
        uint32_t xoff[XR];
#pragma unroll
        for (int i = 0; i < XR; ++i) xoff[i] = ((8u * xg + XR * xp + i) * L + xcol) * 4u;
        float xr[D][XR];
        uint4 a[2][kByRank ? 1 : KS][TM][PW], bb[kAhead][TN][3];
        uint4 raw[kByRank ? D : 1][kByRank ? KS / 2 : 1][TM];  // kByRank: 32 columns per 16 bytes of a lane, two steps ahead
        const uint32_t mine = table_of<kForm>(table, lane);
        float odd = 0.f;
        auto load_x = [&](uint32_t k0, int slot) {
            const __amdgpu_buffer_rsrc_t xbuf = x_rows(X, L, k0, n);
#pragma unroll
            for (int i = 0; i < XR; ++i) xr[slot][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xbuf, xoff[i], 0, 0));
        };
        auto load_w = [&](uint32_t k0, int slot) {
            if constexpr (kByRank) {
#pragma unroll
                for (int s = 0; s < KS / 2; ++s)
#pragma unroll
                    for (int i = 0; i < TM; ++i) raw[slot][s][i] = reinterpret_cast<const uint4*>(wtile[i] + (size_t)(k0 + 32 * s) * 16)[lane];
            } else {
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int p = 0; p < PW; ++p)
                            a[slot][s][i][p] = reinterpret_cast<const uint4*>(wtile[i] + p * plane + (size_t)(k0 + 16 * s) * 32)[lane];
            }
        };
        auto expand = [&](int slot, int s, int to) {
            if constexpr (kByRank)
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const uint4& r = raw[slot][s / 2][i];
                    look_up<kForm>(mine, s & 1 ? r.z : r.x, s & 1 ? r.w : r.y, a[to][0][i]);
                }
        };
        auto store_x = [&](int slot, int buf) {
            if constexpr (XP == 1) {
                uint4 o[3];
                odd += split3_8(xr[slot], o);
#pragma unroll
                for (int p = 0; p < 3; ++p) b[buf][p][xg][xc] = o[p];
            } else {
                uint32_t p0[3], p1[3];
                odd += split3_pair(xr[slot][0], xr[slot][1], p0) + split3_pair(xr[slot][2], xr[slot][3], p1);
#pragma unroll
                for (int p = 0; p < 3; ++p) reinterpret_cast<uint2*>(&b[buf][p][xg][xc])[xp] = make_uint2(p0[p], p1[p]);
            }
        };
        auto read_b = [&](int buf, int s, int to) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int p = 0; p < 3; ++p) bb[to][j][p] = b[buf][p][2 * s + (lane >> 5)][j * 32 + (lane & 31u)];
        };
        floatx16 acc[TM][TN], lo[TM][TN];
        auto clear = [](floatx16 (&v)[TM][TN]) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) v[i][j][e] = 0.f;
        };
        auto flush = [&] {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) sum[i][j] += joined<kForm>(acc[i][j], lo[i][j], scale);
        };
        clear(acc);
        clear(lo);
        clear(sum);
        auto at = [&](uint32_t k) { return min(k, k_end - BK); };  // behind the end: the last step's once more
#pragma unroll
        for (int t = 0; t < (kFetch < D ? kFetch : D); ++t) load_x(at(k_begin + t * BK), t);
        load_w(k_begin, 0);
        if constexpr (kByRank) load_w(at(k_begin + BK), 1);
#pragma unroll
        for (int t = 0; t < kAhead; ++t) store_x(t, t);
#pragma unroll
        for (int t = D; t < kFetch; ++t) load_x(at(k_begin + t * BK), t % D);
        __syncthreads();
        if constexpr (kAhead > 1) read_b(0, 0, 0);
        expand(0, 0, 0);
        // D steps per round, so that the register slots are named at compile time; the last round may be shorter
        uint32_t held = 0;
        for (uint32_t k0 = k_begin; k0 < k_end; k0 += D * BK) {
#pragma unroll
            for (int t = 0; t < D; ++t) {
                if (t > 0 && k0 + t * BK >= k_end) break;
                // (matrix and LDS instructions by turns; left to itself the compiler puts the matrix instructions of a step behind one another: 512 x
                // 4608, batch 3136, 55.7 -> 53.8 us the call, 1509 x 4663, 17 values, 723 59.2 -> 57.3, 2780 x 19849, 117 values, 79 95.5 -> 92.6; the
                // other order of the two 0.5 to 2.5 % less)
                if constexpr (kForm == 1) __builtin_amdgcn_iglp_opt(1);
                else __builtin_amdgcn_iglp_opt(0);
                load_x(at(k0 + (t + kFetch) * BK), (t + kFetch) % D);
                if constexpr (kByRank) load_w(at(k0 + (t + 2) * BK), (t + 2) % D);
                else load_w(at(k0 + (t + 1) * BK), (t + 1) & 1);
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const int q = (t * KS + s) % kAhead;
                    if constexpr (kAhead == 1) read_b(t % kBuffers, s, 0);
                    else if (s + 1 < KS) read_b(t, s + 1, q ^ 1);
                    else read_b((t + 1) % kBuffers, 0, q ^ 1);
                    const int w = (t * KS + s) & 1;
                    if (s + 1 < KS) expand(t, s + 1, w ^ 1);
                    else expand((t + 1) % D, 0, w ^ 1);
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            mfma_pieces<kForm>(a[kByRank ? w : t & 1][kByRank ? 0 : s][i], bb[q][j], acc[i][j], lo[i][j]);
                }
                store_x((t + kAhead) % D, (t + kAhead) % kBuffers);
                __syncthreads();
            }
            held += D * BK;
            if (held >= (kForm == kUniform ? 2u * kFlush : kFlush)) {
                held = 0;
                flush();
                clear(acc);
                clear(lo);
            }
        }
        flush();
        return odd;
    }
};

// Where a part of the columns begins: the parts differ by one unit of columns at most (a compute unit with two long ones is what a launch
// waits for: 512 x 4608, batch 3136, five parts of 8, 8, 8, 8 and 4 rounds of 128 columns 48 us, of 29, 29, 29, 29 and 28 steps of 32 44).
// The first `longer` ones are a unit longer than kchunk.
template <uint32_t kUnit>
__device__ __forceinline__ uint32_t part_begin(uint32_t part, uint32_t kchunk, uint32_t longer) {
    return part * kchunk + min(part, longer) * kUnit;
}

// A workgroup's tile and part: tiles along the shorter side are neighbours.
struct Place {
    uint32_t few, many, part;
};
__device__ __forceinline__ Place place_of(uint32_t item, uint32_t few, uint32_t many, uint32_t splits, uint32_t parts_inside) {
    const uint32_t rest = item / few, next = parts_inside ? splits : many, last = rest / next, middle = rest - last * next;
    return Place{item - rest * few, parts_inside ? last : middle, parts_inside ? middle : last};
}

template <int kForm, bool kByRank, int TN>
__global__ __launch_bounds__(64 * mfma_waves(kForm), 2) void mfma_product_kernel(
    const uint16_t* __restrict__ W, const float* __restrict__ X, float* __restrict__ Out, uint32_t m, uint32_t n, uint32_t L,
    uint32_t pitch, size_t plane, uint32_t row_tiles, uint32_t col_tiles, uint32_t splits, uint32_t kchunk, uint32_t longer, uint32_t parts_inside,
    size_t split_stride, float faint, UniformGrid grid, const float* __restrict__ omega, uint32_t K) {
    using Tile = MfmaTile<kForm, kByRank, TN>;
    __shared__ Tile tile;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups are dealt round-robin to the eight XCDs; every XCD takes a contiguous eighth of the list of work items, in
    // which those that share columns of X (or, with few column tiles, rows of W) are neighbours: they meet in its L2.
    const uint32_t items = row_tiles * col_tiles * splits, eighth = (items + 7u) >> 3;
    const uint32_t item = (blockIdx.x & 7u) * eighth + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= eighth || item >= items) return;
    const uint32_t few = min(row_tiles, col_tiles), many = max(row_tiles, col_tiles);
    const Place at = place_of(item, few, many, splits, parts_inside);
    const uint32_t rt = row_tiles <= col_tiles ? at.few : at.many, ct = row_tiles <= col_tiles ? at.many : at.few, sp = at.part;
    const uint32_t row0 = rt * Tile::BM + wave * 32u * Tile::TM, col0 = ct * Tile::BN;
    const uint32_t k_begin = part_begin<Tile::BK>(sp, kchunk, longer), k_end = part_begin<Tile::BK>(sp + 1u, kchunk, longer);
    Out += sp * split_stride;
    const uint16_t* wtile[Tile::TM];
#pragma unroll
    for (int i = 0; i < Tile::TM; ++i) wtile[i] = W + (size_t)min((row0 >> 5) + i, (m - 1u) >> 5) * (kByRank ? 16 : 32) * pitch;
    floatx16 sum[Tile::TM][TN];
    if constexpr (kByRank) fill_table<kForm>(tile.table, omega, K, grid, tid, 64u * mfma_waves(kForm));
    const float odd = tile.run(wtile, plane, X, n, L, col0, k_begin, k_end, sum, grid.scale);

    // The vote comes before the stores (behind them: 2 us more).
    float least = INFINITY;
#pragma unroll
    for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (row0 + 32 * i + 8 * (e / 4) + 4 * (lane >> 5) + (e % 4) < m)
#pragma unroll
                for (int j = 0; j < TN; ++j) least = fminf(least, fabsf(sum[i][j][e]));
    const int look = __syncthreads_or(odd != odd || least < faint);

    // accumulator element e of lane l: row = 8 (e / 4) + 4 (l / 32) + e % 4, column = l % 32
#pragma unroll
    for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const uint32_t c = col0 + j * 32 + (lane & 31u);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint32_t r = row0 + 32 * i + 8 * (e / 4) + 4 * (lane >> 5) + (e % 4);
                if (r < m && c < L) Out[(size_t)r * L + c] = sum[i][j][e];
            }
        }
    if (look) {
        uint32_t small = 0;  // bit j: a faint sum in column 32 j + lane % 32 (behind the last row at worst one that is none)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float low = INFINITY;
#pragma unroll
            for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) low = fminf(low, fabsf(sum[i][j][e]));
            small |= low < faint ? 1u << j : 0u;
        }
        exact_block<kForm, kByRank>(Block{W, X, Out, plane, m, n, L, pitch, rt * Tile::BM, Tile::BM, col0, Tile::BN, k_begin, k_end, 64u * mfma_waves(kForm), grid.scale, omega, K}, odd != odd, odd != 0.f, small);
    }
}

// The same for small problems: 64 x 32 CT outputs per workgroup, the four waves share its columns of W (32 at a time, in turn)
// and add their sums up in LDS at the end.  A wave loads and splits the part of X that it multiplies straight into operand
// registers, so there is no LDS and no barrier on the way; 128 columns take the workgroup 0.4 - 0.9 us instead of 2.7 (one
// piece), and a matrix of 600 rows wastes 40 of them instead of 168.  This kernel alone, against the large tiles: 700 x 1200, batch
// 60: 9 instead of 19 us, 2048 x 2048, batch 16: 4.6 instead of 9.2, 2728 x 3378, batch 115: 16 instead of 20; 512 x 4608, batch
// 3136: 66 instead of 44.  Bound by the latency of its loads where the chip is not full (2048 x 2048, batch 16, 128 workgroups:
// matrix pipes busy 6 % of the launch, vector ALU 11 %, half of a wave's time is waiting for data), else by what L2 delivers (80
// KiB per 128 columns): the larger tile is the better one where it fills the chip.
template <int kForm, bool kByRank, int CT>
__device__ __forceinline__ float mfma_small_run(const uint16_t* const (&wtile)[2], size_t plane, const float* X, uint32_t n,
                                                uint32_t L, uint32_t col0, uint32_t k_begin, uint32_t k_end, floatx16 (&acc)[2][CT],
                                                float scale, uint32_t mine) {
    constexpr int PW = weight_planes(kForm);
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t xoff[8];  // of the wave's first column tile
#pragma unroll
    for (int i = 0; i < 8; ++i) xoff[i] = ((8u * (lane >> 5) + i) * L + min(col0 + (lane & 31u), L - 1u)) * 4u;
    uint32_t xstep[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) xstep[j] = (min(col0 + 32u * j + (lane & 31u), L - 1u) - min(col0 + (lane & 31u), L - 1u)) * 4u;
    uint4 a[2][kByRank ? 1 : 2][2][kByRank ? 1 : PW];  // kByRank: 32 columns per 16 bytes of a lane
    floatx16 lo[2][CT];
    float x[2][2][CT][8];
    float odd = 0.f;
    auto load = [&](uint32_t k0, int slot) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const __amdgpu_buffer_rsrc_t xbuf = x_rows(X, L, k0 + 16 * s, n);
#pragma unroll
            for (int j = 0; j < CT; ++j)
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    x[slot][s][j][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xbuf, xoff[i] + xstep[j], 0, 0));
            if constexpr (kByRank) {
                if (s == 0)
#pragma unroll
                    for (int i = 0; i < 2; ++i) a[slot][0][i][0] = reinterpret_cast<const uint4*>(wtile[i] + (size_t)k0 * 16)[lane];
            } else {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int p = 0; p < PW; ++p)
                        a[slot][s][i][p] = reinterpret_cast<const uint4*>(wtile[i] + p * plane + (size_t)(k0 + 16 * s) * 32)[lane];
            }
        }
    };
    auto step = [&](int slot) {
        // (as above: 623 x 6257, one piece, batch 1101 58.8 -> 52.4 us the call, 1263 x 652, 8 bits, 501 27.2 -> 24.3; nothing for two pieces)
        if constexpr (kForm == 1 || kForm == 3) __builtin_amdgcn_iglp_opt(0);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            uint4 w[2][PW];
            if constexpr (kByRank) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const uint4& r = a[slot][0][i][0];
                    look_up<kForm>(mine, s ? r.z : r.x, s ? r.w : r.y, w[i]);
                }
            }
#pragma unroll
            for (int j = 0; j < CT; ++j) {
                uint4 b[3];
                odd += split3_8(x[slot][s][j], b);
#pragma unroll
                for (int i = 0; i < 2; ++i) mfma_pieces<kForm>(kByRank ? w[i] : a[slot][kByRank ? 0 : s][i], b, acc[i][j], lo[i][j]);
            }
        }
    };
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = lo[i][j][e] = 0.f;
    uint32_t k0 = k_begin + 32u * wave;
    if (k0 >= k_end) return odd;
    load(k0, 0);
    // (kUniform: the loads of a step stay behind the one before; mixed with it by the compiler they waited for one another: 603 x 6906, three
    // values, batch 1359 77 us instead of 102, 1320 x 5895, 81 values, batch 691 68 instead of 96)
    for (;;) {
        load(min(k0 + 128u, k_end - 32u), 1);  // behind the end: the last columns once more
        step(0);
        if constexpr (kForm == kUniform) __builtin_amdgcn_sched_barrier(0);
        if ((k0 += 128u) >= k_end) break;
        load(min(k0 + 128u, k_end - 32u), 0);
        step(1);
        if constexpr (kForm == kUniform) __builtin_amdgcn_sched_barrier(0);
        if ((k0 += 128u) >= k_end) break;
    }
    if (PW > 1) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) acc[i][j] = joined<kForm>(acc[i][j], lo[i][j], scale);
    }
    return odd;
}

template <int kForm, bool kByRank, int CT>
__global__ __launch_bounds__(256, kForm == 1 || ((kForm == 2 || kForm == kUniform) && CT == 1) ? 2 : 1) void mfma_small_kernel(
    const uint16_t* __restrict__ W, const float* __restrict__ X, float* __restrict__ Out, uint32_t m, uint32_t n, uint32_t L,
    uint32_t pitch, size_t plane, uint32_t row_tiles, uint32_t col_tiles, uint32_t splits, uint32_t kchunk, uint32_t longer, uint32_t,
    size_t split_stride, float faint, UniformGrid grid, const float* __restrict__ omega, uint32_t K) {
    __shared__ float s_acc[4][2 * CT][16][64];
    uint32_t* const table = reinterpret_cast<uint32_t*>(s_acc);  // kByRank: until the sums are made
    static_assert(sizeof s_acc >= kTableWords * 4, "the table lies where the sums meet");
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t items = row_tiles * col_tiles * splits, eighth = (items + 7u) >> 3;
    const uint32_t item = (blockIdx.x & 7u) * eighth + (blockIdx.x >> 3);  // as above
    if ((blockIdx.x >> 3) >= eighth || item >= items) return;
    const uint32_t rt = item % row_tiles, ct = item / row_tiles % col_tiles, sp = item / row_tiles / col_tiles;
    const uint32_t row0 = rt * 64u, col0 = ct * 32u * CT;
    const uint32_t k_begin = part_begin<128>(sp, kchunk, longer), k_end = part_begin<128>(sp + 1u, kchunk, longer);
    Out += sp * split_stride;
    const uint16_t* wtile[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) wtile[i] = W + (size_t)min((row0 >> 5) + i, (m - 1u) >> 5) * (kByRank ? 16 : 32) * pitch;
    if constexpr (kByRank) {
        fill_table<kForm>(table, omega, K, grid, tid, 256u);
        __syncthreads();
    }
    floatx16 acc[2][CT];
    const float odd = mfma_small_run<kForm, kByRank, CT>(wtile, plane, X, n, L, col0, k_begin, k_end, acc, grid.scale, table_of<kForm>(table, lane));
    if constexpr (kByRank) __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) s_acc[wave][i * CT + j][e][lane] = acc[i][j][e];
    __syncthreads();
    // every wave adds up and stores a quarter of the workgroup's accumulators
    constexpr int PER = 2 * CT * 16 / 4;
    float y[PER], least = INFINITY;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t f = wave * PER + q, tile = f >> 4, e = f & 15u;
        y[q] = (s_acc[0][tile][e][lane] + s_acc[1][tile][e][lane]) + (s_acc[2][tile][e][lane] + s_acc[3][tile][e][lane]);
        if (row0 + 32 * (tile / CT) + 8 * (e / 4) + 4 * (lane >> 5) + (e % 4) < m) least = fminf(least, fabsf(y[q]));
    }
    const int look = __syncthreads_or(odd != odd || least < faint);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t f = wave * PER + q, tile = f >> 4, e = f & 15u;
        const uint32_t r = row0 + 32 * (tile / CT) + 8 * (e / 4) + 4 * (lane >> 5) + (e % 4);
        const uint32_t c = col0 + 32 * (tile % CT) + (lane & 31u);
        if (r < m && c < L) Out[(size_t)r * L + c] = y[q];
    }
    if (look)
        exact_block<kForm, kByRank>(Block{W, X, Out, plane, m, n, L, pitch, row0, 64u, col0, 32u * CT, k_begin, k_end, 256u, grid.scale, omega, K}, odd != odd, odd != 0.f, least < faint ? 1u << ((wave * PER >> 4) % CT) : 0u);  // (a wave's share lies in one tile)
}

// The sums of the parts.  Bound by the bytes: four floats per thread and load, four loads in flight; the parts of 512 x 4608, batch 3136
// (five of 6.4 MB) 6.6 us, with one float per load 8.3.
// Many parts (kManyParts) are added in binary64: each addition rounds the sum once more, and from as many as a part's own running sums have
// steps of 16 columns (kFlush) they would round more than those.  The same time; 504 products of 200 to 1024 rows of 4000 to 65000 columns
// end 0.67 times as far from fp64 in the mean (2-norm), 300 x 40000, three pieces, batch 99, X of one sign 2.9e-8 instead of 7.2e-8.
constexpr uint32_t kManyParts = kFlush / 16;
typedef float FourFloats __attribute__((ext_vector_type(4), aligned(4)));
typedef double FourDoubles __attribute__((ext_vector_type(4)));
template <typename Four>
__global__ __launch_bounds__(256) void mfma_sum_kernel(const float* __restrict__ part, float* __restrict__ Y, size_t count,
                                                       uint32_t splits) {
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4u;
    if (i >= count) return;
    const float* p = part + i;
    // (the last thread's four end behind a part by up to three floats: in the next one or in W, which follows the last)
    Four a = {}, b = {};
    uint32_t s = 0;
    for (; s + 4u <= splits; s += 4u) {
        FourFloats v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const FourFloats*>(p + (size_t)(s + k) * count);
        a += __builtin_convertvector(v[0], Four);
        b += __builtin_convertvector(v[1], Four);
        a += __builtin_convertvector(v[2], Four);
        b += __builtin_convertvector(v[3], Four);
    }
    for (; s < splits; ++s) {
        const Four v = __builtin_convertvector(*reinterpret_cast<const FourFloats*>(p + (size_t)s * count), Four);
        if (s & 1u) b += v; else a += v;
    }
    const FourFloats y = __builtin_convertvector(a + b, FourFloats);
    if (i + 4u <= count) {
        *reinterpret_cast<FourFloats*>(Y + i) = y;
    } else {
        for (uint32_t k = 0; i + k < count; ++k) Y[i + k] = y[k];
    }
}

// The parts of a split come one after the other, so that an XCD reads its parts of W and X only (with the parts of a tile next to each
// other, all of W: 707 x 14221, three pieces, batch 452, 109 us the call instead of 90; 727 x 11065, batch 510, 69 instead of 59), but where the decoded
// matrix and X fit the L2s of the chip together (32 MB) and the parts are not many: what an XCD has read alone makes the next call's decoder
// slower (885 x 2357, three pieces, batch 477: 12.0 us instead of 9.1 with the product no faster; 2536 x 963, batch 304, 36.0 us the call instead of 33.5).
// Either order for 53 such products: 0.981 times the time in the mean, 0.92 to 1.05, where the parts are no more than 20 MB; beyond them 1.00 to 1.10
// (1476 x 1476, three pieces, batch 968, 28.6 MB: 50 us, 55 with the parts inside).  The small tiles keep them outermost: 0.97 to 1.09, 1.00 in the mean.
constexpr uint64_t kPartsInside = 26 << 20, kFewParts = 20 << 20;

constexpr uint32_t kPitchStep = 128;  // W's rows are padded to a multiple of this many columns: a round of every variant

int weight_form(const DeviceView& d) { return d.grid.scale != 0.f ? kUniform : d.pieces; }

struct MfmaShape {
    bool small;
    uint32_t BM, BN, row_tiles, col_tiles, splits, unit, per, longer;  // parts of `per` units of columns, the first ones of one more
    bool parts_inside = false;  // next to each other
    double us;  // estimate of the product (without the decode)
};

// The launch lasts as long as the busiest compute unit: its share of the workgroups, one after the other (two resident ones --
// one-piece codebooks with BN = 64 -- overlap, but share the matrix cores: `alone` and `together` scale the time of a round).
// Measured per unit: 4.1 - 4.7 TFLOP/s with BN = 64, bound by the operands' bytes with
// BN = 32; the small tiles 2.4 - 3.5 TFLOP/s.  A split along n costs its partial sums, written and read again.
// each_us: what a workgroup takes besides its rounds, kUniform only, fitted with the rates to 60 products (8.8 us of the large tiles, 6.5
// of the small ones with the launch's; per 64 columns of the large ones 2.05 us, per 128 of the small ones 1.45).
void shape_splits(const DeviceView& d, uint32_t L, uint32_t round, double round_us, double alone, double together,
                  double fixed_us, double each_us, MfmaShape* s) {
    const uint32_t pitch = ((uint32_t)d.n + kPitchStep - 1) / kPitchStep * kPitchStep, units = pitch / s->unit, rounds = pitch / round;
    s->row_tiles = (uint32_t)((d.m + s->BM - 1) / s->BM);
    s->col_tiles = (L + s->BN - 1) / s->BN;
    const double tiles = (double)s->row_tiles * s->col_tiles, cus = std::max(d.cus, 1);
    const uint32_t most = (uint32_t)std::min<double>(std::max(1u, rounds / 4), std::max(1.0, 4.0 * cus / tiles));
    s->us = 1e300;
    for (uint32_t sp = 1; sp <= std::min(most, 64u); ++sp) {
        const double share = std::ceil(tiles * sp / cus);
        // rounds of the busiest one (neighbouring parts, long and short ones, overlap; ones after another may all be long)
        const double own = (together < 1 ? std::ceil(share * units / sp) : share * std::ceil((double)units / sp)) * s->unit / round;
        double us = own * round_us * (share < 2 ? alone : together) + share * each_us + fixed_us;
        if (sp > 1) us += (each_us > 0 ? 4.0 : 3.0) + (double)sp * d.m * L * 8.0 / 6.5e6;
        if (us < s->us) {
            s->us = us;
            s->splits = sp;
            s->per = units / sp;
            s->longer = units % sp;
        }
    }
}

MfmaShape mfma_shape(const DeviceView& d, uint32_t L) {
    const int form = weight_form(d), planes = weight_planes(form);
    const double products = form == 1 ? 3 : (form == kUniform ? 4 : (form == 2 ? 5 : 6));
    MfmaShape big;
    big.small = false;
    big.BN = L <= 32 ? 32 : 64;
    big.BM = 256;
    big.unit = 2048 / big.BN;
    {
        const uint32_t round = (form == 1 && big.BN == 64 ? 4 : 2) * 2048 / big.BN;  // a part has at least four times as many columns
        const double flops = 2.0 * big.BM * big.BN * round * products, bytes = (double)round * (big.BM * 2.0 * planes + big.BN * 4.0);
        shape_splits(d, L, round, big.BN == 32 ? std::max(flops / (form == kUniform ? 4.0e6 : 4.3e6), bytes / 3.0e4) : flops / (form == 1 ? 4.4e6 : (form == kUniform ? 4.2e6 : 4.6e6)),
                     form == 1 ? 1.12 : 1.0, form == 1 ? 0.95 : 1.0, form == kUniform ? 2.5 : 4.0, form == kUniform ? 6.5 : 0.0, &big);
    }
    MfmaShape small;
    small.small = true;
    small.BN = L <= 32 ? 32 : 64;
    small.BM = 64;
    small.unit = 128;
    {
        const double flops = 2.0 * small.BM * small.BN * 128 * products;
        shape_splits(d, L, 128, flops / (form == 1 ? 3.5e6 : (planes == 2 ? 2.9e6 : 2.4e6)), form == 1 && small.BN == 64 ? 1.5 : 1.0, 1.0,
                     form == kUniform ? 3.5 : 3.0, form == kUniform ? 4.0 : 0.0, &small);
    }
    return small.us < big.us ? small : big;
}

// Whether the decoder leaves ranks instead of pieces: one byte per element written and read instead of four or six, but the product looks
// every one up again for each of its tiles of columns (a dot product, an LDS read and an add or two of a permutation each, on a launch bound by the
// matrix cores' power).  Saved, us: 1.5 and 0.14 per million bytes (1419 x 7930, two pieces, 5.1; 1180 x 1489, three, 1.9), twice that where
// few rows keep a decoder of pieces waiting (260 x 8894, batch 264 31.8 / 25.4); added, in shares of the
// product: 0.16 with two pieces (1419 x 7930, batch 242 30.0 -> 34.9), 0.12 with three (1180 x 1489, batch 847 27.4 -> 30.6) and of the small tiles, which
// wait for their loads (1040 x 5160, batch 949 57.2 -> 65.5).  us per call, pieces / ranks: 2780 x 19849, 117 values, batch 79 130 / 104; 2819 x 13862,
// 6 bits, 130 171 / 135; 1252 x 22319, 8 bits, 186 140 / 107; 3054 x 4174, 6 bits, 137 60 / 50; 961 x 3191, 4 bits, 517 43 / 38; but 599 x 19045,
// 3 values, batch 384 70.6 / 73.5; 1509 x 4663, 17 values, 723 73 / 77; 2095 x 1669, 7 bits, 1109 78 / 80.  One piece is two bytes as it is: 0.95 to 1.14
// times the time.
bool multiplies_ranks(const DeviceView& d, const MfmaShape& s) {
    const int planes = weight_planes(weight_form(d));
    if (!d.rank_tab || planes == 1) return false;
    const double bytes = (double)d.m * (double)d.n * (2.0 * planes - 1.0) * (d.m <= 2 * d.cus ? 2.0 : 1.0);
    return 1.5 + bytes / 7e6 > s.us * (s.small || planes == 3 ? 0.12 : 0.16);
}

template <int kForm, bool kByRank>
hipError_t launch_shape(const MfmaShape& s, const uint16_t* W, const float* X, float* out, uint32_t m, uint32_t n, uint32_t L,
                        uint32_t pitch, size_t plane, float faint, const DeviceView& d, hipStream_t stream) {
    const dim3 grid((s.row_tiles * s.col_tiles * s.splits + 7) / 8 * 8);
    const size_t count = (size_t)m * L;
    auto* kern = s.small ? (s.BN == 32 ? mfma_small_kernel<kForm, kByRank, 1> : mfma_small_kernel<kForm, kByRank, 2>)
                         : (s.BN == 32 ? mfma_product_kernel<kForm, kByRank, 1> : mfma_product_kernel<kForm, kByRank, 2>);
    return launch_kernel(kern, grid, dim3(s.small ? 256 : 64 * mfma_waves(kForm)), 0, stream, W, X, out, m, n, L, pitch, plane, s.row_tiles, s.col_tiles, s.splits,
                         s.per * s.unit, s.longer, s.parts_inside ? 1u : 0u, count, faint, d.grid, d.omega, (uint32_t)d.K);
}

}  // namespace

// Whether the codebook and the sizes allow the route at all, and its estimated duration without the decode.
int mfma_planes(const DeviceView& d) { return weight_planes(weight_form(d)); }
bool mfma_applicable(const DeviceView& d, uint32_t L) {
    return d.pieces > 0 && d.m > 0 && d.n > 0 && L > 1 && d.n < (1ll << 31) && d.m < (1ll << 31) && (uint64_t)d.m * L < (1ull << 40) &&
           ((uint64_t)d.n + kPitchStep) * L * 4u < (1ull << 32);  // X is addressed with 32-bit offsets
}
double mfma_estimate_us(const DeviceView& d, uint32_t L) { return mfma_shape(d, L).us; }

hipError_t launch_mfma(const DeviceView& d, const float* X, float* Y, uint32_t L, hipStream_t stream) {
    MfmaShape s = mfma_shape(d, L);
    const int form = weight_form(d);
    const int64_t pitch = (d.n + kPitchStep - 1) / kPitchStep * kPitchStep, plane = pitch * ((d.m + 31) / 32 * 32);
    const bool by_rank = multiplies_ranks(d, s);
    const size_t w_bytes = by_rank ? (size_t)plane : (size_t)plane * 2 * weight_planes(form);
    const size_t count = (size_t)d.m * L;
    s.parts_inside = (uint64_t)w_bytes + (uint64_t)d.n * L * 4 <= kPartsInside && count * s.splits * 4 <= kFewParts;
    // one temporary: the partial sums, then the pieces
    const size_t part_bytes = s.splits > 1 ? (count * s.splits * 4 + 255) & ~(size_t)255 : 0;
    unsigned char* tmp = nullptr;
    hipError_t e = (hipError_t)temp_alloc(reinterpret_cast<void**>(&tmp), part_bytes + w_bytes, stream);
    if (e != hipSuccess) return e;
    auto* W = reinterpret_cast<uint16_t*>(tmp + part_bytes);
    float* out = s.splits > 1 ? reinterpret_cast<float*>(tmp) : Y;
    e = (hipError_t)(by_rank ? decode_ranks(d, reinterpret_cast<uint8_t*>(W), pitch, stream) : decode_pieces(d, W, pitch, plane, stream));
    if (e == hipSuccess) {
        const uint32_t m = (uint32_t)d.m, n = (uint32_t)d.n;
        // An input loses at most half of 2^-133, a sum at most n max|w| 2^-134: less than 2^-26 of itself from here on.
        const float faint = (float)std::min((double)d.n * d.omega_max * 0x1p-108, 1e38);
        auto launch = [&](auto kernels) { return kernels(s, W, X, out, m, n, L, (uint32_t)pitch, (size_t)plane, faint, d, stream); };
        switch (form) {
            case 1: e = launch(launch_shape<1, false>); break;
            case 2: e = launch(by_rank ? launch_shape<2, true> : launch_shape<2, false>); break;
            case 3: e = launch(by_rank ? launch_shape<3, true> : launch_shape<3, false>); break;
            default: e = launch(by_rank ? launch_shape<kUniform, true> : launch_shape<kUniform, false>);
        }
    }
    if (e == hipSuccess && s.splits > 1)
        e = launch_kernel(s.splits < kManyParts ? mfma_sum_kernel<FourFloats> : mfma_sum_kernel<FourDoubles>, dim3((uint32_t)((count + 1023) / 1024)), dim3(256), 0, stream, out, Y, count, s.splits);
    const hipError_t f = (hipError_t)temp_free(tmp, stream);
    return e == hipSuccess ? f : e;
}

}  // namespace cer
