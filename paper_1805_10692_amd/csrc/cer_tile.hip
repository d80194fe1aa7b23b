// Products of some dozens of batch columns and more on the bf16 matrix cores, tiles of W laid out in LDS from a tile index.
//
// The format orders a row's indices by value, then column, so that the elements of a range of columns are scattered over the row's
// groups: cer_fused_kernel lays out 16 or 32 whole rows at a time, and its workgroups load X as often as there are such blocks of rows.
// The tile index (tile_index_kernel; cer_prepare_strips keeps it with the handle) has the elements in buckets of 16 rows and 64 columns, an
// entry each, so that 64 rows can be laid out for 64 columns by reading nothing else.
//
// Workgroup of eight waves: 16 RT rows x 16 CT columns of Y over a range of W's columns.  The waves share that range, 64 columns in turn,
// and never wait for one another: a wave lays out its 64 columns as bf16 numbers in planes of its own in LDS (the most frequent value
// everywhere, then the entries), reads them back as the matrix instructions want them, loads the same 64 rows of X from memory, takes
// them to pieces (cer_split3.hpp) and multiplies; its next entries and rows of X are on their way meanwhile.  The waves' sums meet in LDS
// at the end, parts of W's columns in a second launch.
// One barrier per 512 columns with planes that all waves fill instead: 4096 x 9216, 15 % indexed, batch 99 41 us instead of 38.  128 rows
// (half the loads and splits of X): one wave per SIMD 50 us, two with one step of X in registers 41.
// Against the kernels it takes the place of: that product 56.8 us with the strips -> 35.5; 2593 x 18163, 66 % indexed, batch 41 103
// (decoded matrix) -> 42; 1529 x 862, 38 values, batch 167 19.9 (gathers) -> 11.2; 1103 x 14914, 5 values, batch 42 33.6 (one launch) -> 24.7; of
// 11000 random products of prepared handles a fifth takes it (tile_limit_us in cer_matmul.hip), at 1.28 times the speed in the geometric mean.
// What bounds it: 4096 x 9216, batch 99, 68000 clocks: start-up 7500 (bounds, entries and X one after the other from memory), sums 5300;
// between them the matrix pipes are busy half the time -- while they are, a SIMD issues other vector instructions every nine clocks only and dot
// products (the splitting) every 22.  The variant of 64 rows and 64 columns takes all 256 registers and spills two; the functions for columns
// formed again save theirs in scratch (468 bytes per lane).
// Errors against fp64 are 0.41 of the replaced kernels' in the mean, at most 0.97 (2-norm; 333 products of 4000 to 64990 columns, X normal, cut at
// 0, |x| + 1): short running sums per wave, the small products apart, the waves' and the parts' sums in binary64.
#include "cer_exact.hpp"

#include <type_traits>

namespace cer {
namespace {

constexpr uint32_t kTileWaves = 8, kTileThreads = kTileWaves * kWave;
// A bucket's rows and columns of W; bytes per row of them in LDS (rows 36 banks apart: a wave's 16-byte reads of 16 rows meet no conflict).
constexpr uint32_t kGroupRows = 16, kSegCols = 64, kPitch = 2 * kSegCols + 16, kGroupBytes = kGroupRows * kPitch;

// LDS: [flags, cleared at the kernel's start: columns with sums that are not finite, with faint ones, left for binary32; lossy inputs]
// [arguments of the functions for those][what tile_again learns of rows and columns][pieces of the codebook's values, by rank][per wave: planes of
// 16 RT rows]; later the waves' sums
constexpr uint32_t kTileArgsAt = 32, kTileBitsAt = kTileArgsAt + 128, kTileSizesAt = kTileBitsAt + 512, kTileTableAt = kTileSizesAt + 128;
constexpr int kOddColumns = 0, kFaintColumns = 2, kTileLossy = 4, kSlowColumns = 5;  // the flags' words: 64 columns, 64 columns, a bit per 16 lanes' columns, 64 columns
__host__ __device__ constexpr uint32_t planes_at(int form) { return kTileTableAt + 256u * (form == 1 ? 0u : entry_bytes(form)); }
__host__ __device__ constexpr uint32_t wave_bytes(int form, int rt) { return (uint32_t)weight_planes(form) * rt * kGroupBytes; }

// LDS of tile_index_kernel: [as far as table_at: cer_exact.hpp][counts by segment][per row: payloads of its groups][staged entries]
constexpr uint32_t kCounts = 1028;  // (segments of the widest matrix, 1016, and one more)
__host__ __device__ constexpr uint32_t index_counts_at(uint32_t waves) { return (table_at(waves) + 15u) & ~15u; }
__host__ __device__ constexpr uint32_t index_payload_at(uint32_t waves) { return index_counts_at(waves) + 4u * kCounts; }
__host__ __device__ constexpr uint32_t payload_bytes(uint32_t tab_shift) { return 2u * ((1u << tab_shift) + 2u); }
__host__ __device__ constexpr uint32_t index_stage_at(uint32_t waves, uint32_t tab_shift) {
    return (index_payload_at(waves) + waves * payload_bytes(tab_shift) + 15u) & ~15u;
}
// First entry of a group's buckets: room for its elements and three more in every bucket, whole quads, behind the quad that goes nowhere.
__host__ __device__ constexpr uint32_t group_base(uint32_t first_position, uint32_t group, uint32_t segs) {
    return 4u + ((first_position + 3u * segs * group + 3u) & ~3u);
}

typedef float FourFloats __attribute__((ext_vector_type(4), aligned(4)));

struct TileRest {
    float* Out;
    size_t split_stride;
    const float* omega;
    uint32_t values;  // of the codebook, less one
    float faint, most;
    uint32_t dense;   // a zero weight times an infinity counts
};
struct TileArgs {
    const uint4* quads;
    const uint32_t* ptr;
    const float* X;
    const float* omega;
    float* Out;
    double inverse;
    float scale, unit, least, most;
    uint32_t m, n, L, row0, col0, cols, h0, h1, dense;
};
static_assert(sizeof(TileArgs) <= kTileBitsAt - kTileArgsAt, "place of the arguments");

typedef uint32_t TwoBounds __attribute__((ext_vector_type(2), aligned(4)));

// The most frequent value's pieces, twice each, in every dword of a wave's planes.
template <int kForm>
__device__ __forceinline__ void fill_pieces(float omega0, const UniformGrid& grid, uint32_t (&fill)[weight_planes(kForm)]) {
    uint32_t p[3];
    if constexpr (kForm == kUniform) {
        p[0] = uniform_pieces(omega0, grid);
        p[1] = p[0] >> 16;
        p[0] &= 0xFFFFu;
    } else {
        split3_finite(omega0, p);
    }
#pragma unroll
    for (int i = 0; i < weight_planes(kForm); ++i) fill[i] = uniform(p[i] | p[i] << 16);
}

template <int kForm, int RT>
__device__ __forceinline__ void clear_planes(uint32_t mine, const uint32_t (&fill)[weight_planes(kForm)], uint32_t lane) {
    constexpr uint32_t kPlane = RT * kGroupBytes;
    typedef uintx4 __attribute__((address_space(3))) * Lds4;
#pragma unroll
    for (int p = 0; p < weight_planes(kForm); ++p) {
        const uintx4 f = {fill[p], fill[p], fill[p], fill[p]};
#pragma unroll
        for (uint32_t i = 0; i < (kPlane / 16u + kWave - 1u) / kWave; ++i)
            if ((i + 1u) * kWave * 16u <= kPlane || i * kWave + lane < kPlane / 16u)
                *reinterpret_cast<Lds4>((uintptr_t)(mine + (uint32_t)p * kPlane + (i * kWave + lane) * 16u)) = f;
    }
}

// Four entries into the planes; to: the group's rows of the first one.
template <int kForm, int RT>
__device__ __forceinline__ void place_quad(uint32_t to, const unsigned char* smem, const uint4& quad) {
    constexpr uint32_t kPlane = RT * kGroupBytes;
    typedef uint16_t __attribute__((address_space(3))) * Lds16;
    const uint32_t e[4] = {quad.x, quad.y, quad.z, quad.w};
    if constexpr (kForm == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<Lds16>((uintptr_t)(to + (e[i] & 0xFFFFu))) = (uint16_t)(e[i] >> 16);
    } else {
        uint32_t v[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (kForm == kUniform) {
                v[i][0] = reinterpret_cast<const uint32_t*>(smem + kTileTableAt)[e[i] >> 16];
            } else {
                const uint2 w = reinterpret_cast<const uint2*>(smem + kTileTableAt)[e[i] >> 16];
                v[i][0] = w.x;
                v[i][1] = w.y;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t at = to + (e[i] & 0xFFFFu);
            *reinterpret_cast<Lds16>((uintptr_t)at) = (uint16_t)v[i][0];
            *reinterpret_cast<Lds16>((uintptr_t)(at + kPlane)) = (uint16_t)(v[i][0] >> 16);
            if constexpr (kForm == 3) *reinterpret_cast<Lds16>((uintptr_t)(at + 2u * kPlane)) = (uint16_t)v[i][1];
        }
    }
}

// What the functions below know of the workgroup's outputs, and its wave's planes.
template <int kForm, int RT>
struct TileAgain {
    static constexpr int PW = weight_planes(kForm);
    unsigned char* smem;
    uint32_t lane, wave, m, n, L, row0, col0, cols, h0, h1, segs, mine, fill[PW];
    const uint4* quads;
    const uint32_t* bounds;
    const float* X;
    float* out;
    bool rows;  // of the lane's group
    UniformGrid grid;
    float omega0, least, most;
    bool dense;
    __device__ __forceinline__ explicit TileAgain(uint32_t lds) : smem(lds_pointer(lds)) {
        const TileArgs& a = *reinterpret_cast<const TileArgs*>(smem + kTileArgsAt);
        constexpr uint32_t kLanes = kWave / RT;
        lane = threadIdx.x & 63u; wave = uniform(threadIdx.x >> 6);
        m = uniform(a.m); n = uniform(a.n); L = uniform(a.L);
        row0 = uniform(a.row0); col0 = uniform(a.col0); cols = uniform(a.cols); h0 = uniform(a.h0); h1 = uniform(a.h1);
        segs = (n + kSegCols - 1u) / kSegCols;
        mine = lds + planes_at(kForm) + wave * wave_bytes(kForm, RT);
        quads = uniform_pointer(a.quads); X = uniform_pointer(a.X); out = uniform_pointer(a.Out);
        const uint32_t groups = (m + kGroupRows - 1u) / kGroupRows, group = row0 / kGroupRows + lane / kLanes;
        rows = group < groups;
        bounds = uniform_pointer(a.ptr) + (size_t)min(group, groups - 1u) * (segs + 1u);
        grid.scale = a.scale; grid.unit = a.unit; grid.inverse = a.inverse;
        least = a.least; most = a.most;
        dense = uniform(a.dense) != 0u;
        omega0 = uniform_pointer(a.omega)[0];
        fill_pieces<kForm>(omega0, grid, fill);
    }
    // Segment h's weights into the wave's planes.
    __device__ __forceinline__ void lay_out(uint32_t h) const {
        constexpr uint32_t kLanes = kWave / RT;
        const TwoBounds b = *reinterpret_cast<const TwoBounds*>(bounds + h);
        wave_lds_sync();
        clear_planes<kForm, RT>(mine, fill, lane);
        const uint32_t end = rows ? b[1] : 0u;
        for (uint32_t i = b[0] + lane % kLanes; __ballot(i < end) != 0ull; i += kLanes)
            place_quad<kForm, RT>(mine + lane / kLanes * kGroupBytes, smem, quads[i < end ? i : 0u]);
        wave_lds_sync();
    }
};

// Columns of outputs once more on the matrix cores, 16 CT after the other; the loop is the kernel's.
// Not scaled, columns with sums that are not finite: infinities and NaNs of X count as zeros in the sums, and what they make of an output
// is kept as two bits per row and column (a term that is +infinity, one that is -infinity; a NaN is both), which tells it whatever the
// order of the sum.  As with the gathers the terms are those of a row's indices, (value - most frequent value) . x, and that value . x, or
// (dense) as with the decoded matrix those of every element.
// Scaled, columns with faint sums next to inputs that have lost bits: with X times 2^64 every input has its pieces.  Only where the
// column's largest input leaves room for that (most): a sum of large terms may be faint as well, by cancelling.
// Sums that are not finite all the same, and columns with inputs too large to be scaled, are left to tile_slow.
// 4096 x 9216, 15 % indexed, batch 99 (41 us; without the index 58 for any X): one or eight columns with an infinity 54 us, all of them 88, one
// column near 2^-120 52, all of X 93; 1103 x 14914, 5 values, batch 42 (26; without the index 33, all of these 470 to 490): 43, 68, 45, 79.  Bound by what
// the kernel is bound by, which its own loop does for 16 CT columns with fewer registers.
template <int kForm, int RT, int CT, bool kScaled>
__device__ __attribute__((noinline)) void tile_again(uint32_t lds, uint32_t columns0, uint32_t columns1) {
    using Tile = TileAgain<kForm, RT>;
    const Tile a(lds);
    constexpr int PW = Tile::PW, kQ = 3, kSteps = kSegCols / 32;
    constexpr uint32_t kPlane = RT * kGroupBytes, kLanes = kWave / RT, R = 16 * RT, kPer = RT * CT * 4 * kWave;
    typedef const uintx4 __attribute__((address_space(3))) * Lds4;
    typedef const uint16_t __attribute__((address_space(3))) * Lds16;
    const uint64_t columns = (uint64_t)uniform(columns1) << 32 | uniform(columns0);
    const uint32_t tid = threadIdx.x, lane = a.lane, c16 = lane & 15u, g = lane >> 4;
    uint32_t* const flags = reinterpret_cast<uint32_t*>(a.smem);
    uint32_t* const s_bits = reinterpret_cast<uint32_t*>(a.smem + kTileBitsAt);   // [row][+, -], a bit per column
    uint32_t* const s_size = reinterpret_cast<uint32_t*>(a.smem + kTileSizesAt);  // scaled: the columns' largest inputs; else: whether a lane's have lost bits
    float* const s_sum = reinterpret_cast<float*>(a.smem + planes_at(kForm));
    auto bounds_of = [&](uint32_t h) { return *reinterpret_cast<const TwoBounds*>(a.bounds + min(h, a.segs - 1u)); };
#pragma unroll 1
    for (uint32_t c0 = 0; c0 < a.cols; c0 += 16u * CT) {
        const uint32_t mask = (uint32_t)(columns >> c0) & (CT == 2 ? 0xFFFFFFFFu : 0xFFFFu);
        if (mask == 0u) continue;
        __syncthreads();  // what lies in LDS has been read
        if (tid < 2u * R) s_bits[tid] = 0u;
        if (tid < 32u) s_size[tid] = 0u;
        const uint32_t first = a.col0 + c0 + CT * c16, xcol = min(first, a.L - (uint32_t)CT);
        uint32_t xoff[8];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) xoff[i] = ((8u * g + i) * a.L + xcol) * 4u;
        float x[kSteps][8][CT];
        auto load_x = [&](uint32_t k0, float (&v)[8][CT]) {
            const __amdgpu_buffer_rsrc_t xbuf = x_rows(a.X, a.L, min(k0, a.n), a.n);
#pragma unroll
            for (int i = 0; i < 8; ++i) load_columns<CT>(xbuf, xoff[i], v[i]);
        };
        TwoBounds bound = bounds_of(a.h0 + a.wave);
        uint4 q[kQ];
        uint32_t cb = 0, ce = 0;
        auto request = [&](uint32_t h) {
            cb = bound[0] + lane % kLanes;
            ce = a.rows && h < a.h1 ? bound[1] : 0u;
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                const uint32_t i = cb + (uint32_t)u * kLanes;
                q[u] = a.quads[i < ce ? i : 0u];
            }
        };
        floatx4 sum[RT][CT] = {};
        float largest[CT] = {};
        uint32_t plus = 0, minus = 0, lost = 0;  // plus, minus: of row lane % R, column xcol + c is bit 16 c + c16
        // The inputs of a step among which some are not finite, or round to an infinite bf16 number: their pieces.  (Rows one after the other in
        // a loop: 16 copies of it would be most of the code.)
        auto take_apart = [&](int s, uint4 (&b)[CT][3]) {
            if constexpr (!kScaled)
#pragma unroll 1
                for (uint32_t i = 0; i < 8; ++i) {
                    uint64_t up[CT], down[CT], none[CT], any = 0;
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        float v = x[s][0][c];
#pragma unroll
                        for (uint32_t j = 1; j < 8; ++j) v = i == j ? x[s][j][c] : v;
                        up[c] = __ballot(v == INFINITY);
                        down[c] = __ballot(v == -INFINITY);
                        none[c] = __ballot(v != v);
                        any |= up[c] | down[c] | none[c];
                    }
                    if (any == 0ull) continue;
#pragma unroll 1
                    for (uint32_t k = 0; k < 4; ++k) {  // row 8 k + i of the step: 16 lanes' columns
                        uint32_t bits[3] = {};
#pragma unroll
                        for (int c = 0; c < CT; ++c) {
                            bits[0] |= ((uint32_t)(up[c] >> (16u * k)) & 0xFFFFu) << (16 * c);
                            bits[1] |= ((uint32_t)(down[c] >> (16u * k)) & 0xFFFFu) << (16 * c);
                            bits[2] |= ((uint32_t)(none[c] >> (16u * k)) & 0xFFFFu) << (16 * c);
                        }
                        const uint32_t one_way = bits[0] | bits[2], other_way = bits[1] | bits[2], all = one_way | other_way;
                        if (all == 0u) continue;
                        uint32_t piece[PW];
                        bool indexed = false;
#pragma unroll
                        for (int p = 0; p < PW; ++p) {
                            piece[p] = *reinterpret_cast<Lds16>((uintptr_t)(a.mine + (uint32_t)p * kPlane + lane % R * kPitch + 2u * (32u * s + 8u * k + i)));
                            indexed |= piece[p] != (a.fill[p] & 0xFFFFu);
                            piece[p] <<= 16;
                        }
                        float w = __uint_as_float(piece[0]);
                        if constexpr (kForm == kUniform) w = fmaf(a.grid.scale, w, a.grid.scale * __uint_as_float(piece[PW - 1]));
                        if constexpr (kForm == 3) w += __uint_as_float(piece[PW > 1 ? 1 : 0]) + __uint_as_float(piece[PW - 1]);
                        // the terms' signs: of w, or of w - omega0 where indexed, and of omega0
                        const bool rises = a.dense ? w > 0.f : indexed && w > a.omega0, falls = a.dense ? w < 0.f : indexed && w < a.omega0;
                        const uint32_t nan = a.dense && !rises && !falls ? all : 0u;
                        plus |= (rises ? one_way : 0u) | (falls ? other_way : 0u) | nan;
                        minus |= (rises ? other_way : 0u) | (falls ? one_way : 0u) | nan;
                        if (!a.dense && a.omega0 != 0.f) {
                            plus |= a.omega0 > 0.f ? one_way : other_way;
                            minus |= a.omega0 > 0.f ? other_way : one_way;
                        }
                    }
                }
            uint32_t pieces[CT][3][4];
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    float& v = x[s][i][c];
                    v = fabsf(v) < INFINITY ? v : 0.f;
                    lost |= split_lossy(v) ? 1u : 0u;
                    uint32_t p[3];
                    split3_finite(kScaled ? v * 0x1p64f : v, p);
#pragma unroll
                    for (int j = 0; j < 3; ++j) pieces[c][j][i >> 1] = i & 1 ? pieces[c][j][i >> 1] | p[j] << 16 : p[j];
                }
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int j = 0; j < 3; ++j) b[c][j] = make_uint4(pieces[c][j][0], pieces[c][j][1], pieces[c][j][2], pieces[c][j][3]);
        };
        uint32_t h = a.h0 + a.wave;
        request(h);
        bound = bounds_of(h + kTileWaves);
#pragma unroll
        for (int s = 0; s < kSteps; ++s) load_x(h * kSegCols + 32u * s, x[s]);
        __syncthreads();
#pragma unroll 1
        for (; h < a.h1; h += kTileWaves) {
            wave_lds_sync();
            clear_planes<kForm, RT>(a.mine, a.fill, lane);
            const uint32_t to = a.mine + lane / kLanes * kGroupBytes;
#pragma unroll
            for (int u = 0; u < kQ; ++u) place_quad<kForm, RT>(to, a.smem, q[u]);
            for (uint32_t c = cb + (uint32_t)kQ * kLanes; __ballot(c < ce) != 0ull; c += kLanes) place_quad<kForm, RT>(to, a.smem, a.quads[c < ce ? c : 0u]);
            wave_lds_sync();
            request(h + kTileWaves);
            bound = bounds_of(h + 2u * kTileWaves);
            floatx4 acc[RT][CT] = {}, lo[RT][CT] = {};
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                uint4 w[RT][PW], b[CT][3];
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int p = 0; p < PW; ++p) {
                        const uintx4 v = *reinterpret_cast<Lds4>((uintptr_t)(a.mine + c16 * kPitch + (uint32_t)s * 64u + g * 16u + (uint32_t)p * kPlane + (uint32_t)r * kGroupBytes));
                        w[r][p] = make_uint4(v[0], v[1], v[2], v[3]);
                    }
                uint32_t bits = 0;
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    float xc[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) xc[i] = kScaled ? x[s][i][c] * 0x1p64f : x[s][i][c];
                    split3_8_dot(xc, b[c], bits);
                }
                lost |= bits;
                // an input without pieces leaves a NaN among the remainders (and inputs from 2^17 on what may look like one)
                if (__ballot((bits & 0x7F800000u) == 0x7F800000u) != 0ull) take_apart(s, b);
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    if constexpr (kScaled)
#pragma unroll
                        for (int i = 0; i < 8; ++i) largest[c] = fmaxf(largest[c], fabsf(x[s][i][c]));
#pragma unroll
                    for (int d = 2; d >= 0; --d)
#pragma unroll
                        for (int i = 0; i < PW; ++i)
                            if (d - i >= 0 && !(kForm == kUniform && i == 1 && d == 2))
#pragma unroll
                                for (int r = 0; r < RT; ++r) {
                                    floatx4& into = d > 0 ? lo[r][c] : acc[r][c];
                                    into = mfma16(w[r][i], b[c][d - i], into);
                                }
                }
                load_x((h + kTileWaves) * kSegCols + 32u * s, x[s]);
            }
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        sum[r][c][e] += kForm == kUniform ? fmaf(a.grid.scale, acc[r][c][e], a.grid.scale * lo[r][c][e]) : acc[r][c][e] + lo[r][c][e];
        }
        __syncthreads();
        if (plus != 0u) atomicOr(&s_bits[2u * (lane % R)], plus);
        if (minus != 0u) atomicOr(&s_bits[2u * (lane % R) + 1u], minus);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            if constexpr (kScaled) atomicMax(&s_size[16u * c + c16], __float_as_uint(largest[c]));
            else if ((lost & 0xFFFFu) != 0u) s_size[16u * c + c16] = 1u;
        }
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) s_sum[a.wave * kPer + ((r * 4 + e) * CT + c) * kWave + lane] = sum[r][c][e];
        __syncthreads();
        uint32_t slow = 0, faint = 0;  // of the lane's columns
        for (uint32_t re = a.wave; re < RT * 4u; re += kTileWaves) {
            const uint32_t r = 16u * (re >> 2) + 4u * g + (re & 3u), row = a.row0 + r;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const uint32_t column = xcol + c - a.col0 - c0;  // (the lane's first ones are another lane's where the batch ends)
                if (row >= a.m || xcol + c < first || ((mask >> column) & 1u) == 0u) continue;
                double total = 0;
#pragma unroll
                for (uint32_t k = 0; k < kTileWaves; ++k) total += s_sum[k * kPer + (re * CT + c) * kWave + lane];
                const uint32_t size_x = s_size[16u * c + c16];
                float* at = a.out + (size_t)row * a.L + xcol + c;
                if constexpr (kScaled) {
                    const float size = fabsf(*at);
                    if (size < a.least || (size < 0x1p-126f && size > 0.f)) {
                        if (__uint_as_float(size_x) < a.most) *at = (float)(total * 0x1p-64); else slow |= 1u << c;
                    }
                } else {
                    const float y = (float)total, size = fabsf(y);
                    const bool up = (s_bits[2u * r] >> (16 * c + c16)) & 1u, down = (s_bits[2u * r + 1u] >> (16 * c + c16)) & 1u;
                    if (!(size < INFINITY)) slow |= 1u << c;
                    if (!up && !down && ((size < a.least && size_x != 0u) || (size < 0x1p-126f && size > 0.f))) faint |= 1u << c;
                    *at = up && down ? NAN : (up ? INFINITY : (down ? -INFINITY : y));
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const uint32_t column = xcol + c - a.col0;
            if ((slow >> c) & 1u) atomicOr(&flags[kSlowColumns + (column >> 5)], 1u << (column & 31u));
            if ((faint >> c) & 1u) atomicOr(&flags[kFaintColumns + (column >> 5)], 1u << (column & 31u));
        }
    }
    __syncthreads();
}

// 32 columns at a time where both sixteens have some, else sixteen.
template <int kForm, int RT, int CT, bool kScaled>
__device__ __forceinline__ void tile_again_columns(uint32_t lds, uint32_t columns0, uint32_t columns1) {
    const uint32_t wide0 = (columns0 & 0xFFFFu) != 0u && columns0 >> 16 != 0u ? columns0 : 0u, wide1 = (columns1 & 0xFFFFu) != 0u && columns1 >> 16 != 0u ? columns1 : 0u;
    if constexpr (CT >= 2)
        if ((wide0 | wide1) != 0u) tile_again<kForm, RT, 2, kScaled>(lds, wide0, wide1);
    if (((columns0 ^ wide0) | (columns1 ^ wide1)) != 0u) tile_again<kForm, RT, 1, kScaled>(lds, columns0 ^ wide0, columns1 ^ wide1);
}

// Columns of which nothing else is certain once more, in binary32, four after the other: a lane takes a row and walks along W's columns.  As
// with the gathers the sum is over a row's indices of (value - most frequent value) . x, and that value times the column sum, or
// (dense) as with the decoded matrix over every element.  4096 x 9216, 15 % indexed, batch 99, a column with sums beyond binary32: 104 us (41;
// 58 without the index).
template <int kForm, int RT>
__device__ __attribute__((noinline)) void tile_slow(uint32_t lds, uint32_t columns0, uint32_t columns1) {
    using Tile = TileAgain<kForm, RT>;
    const Tile a(lds);
    constexpr int PW = Tile::PW;
    constexpr uint32_t kPlane = RT * kGroupBytes, R = 16 * RT;
    typedef const uintx4 __attribute__((address_space(3))) * Lds4;
    const bool dense = a.dense;
    uint64_t columns = (uint64_t)uniform(columns1) << 32 | uniform(columns0);
    float* s_sum = reinterpret_cast<float*>(a.smem + planes_at(kForm));  // [wave][column][row], [wave][column][lane] of X
    float* s_x = s_sum + kTileWaves * 4u * kWave;
    const uint32_t row = a.lane % R;
#pragma unroll 1
    while (columns != 0ull) {
        uint32_t c[4], count = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = a.col0 + (columns != 0ull ? (uint32_t)__builtin_ctzll(columns) : 0u);
            count += columns != 0ull ? 1u : 0u;
            columns &= columns - 1ull;
        }
        float y[4] = {}, sum[4] = {};
        __syncthreads();
        auto walk = [&](auto columns_at_once) {
            constexpr int kCols = columns_at_once.value;
#pragma unroll 1
            for (uint32_t h = a.h0 + a.wave; h < a.h1; h += kTileWaves) {
                float x[kCols];
                const uint32_t k0 = h * kSegCols;
#pragma unroll
                for (int j = 0; j < kCols; ++j) {
                    x[j] = k0 + a.lane < a.n && (uint32_t)j < count ? a.X[(size_t)(k0 + a.lane) * a.L + c[j]] : 0.f;
                    sum[j] += x[j];
                }
                a.lay_out(h);
#pragma unroll 1
                for (uint32_t k = 0; k < kSegCols; k += 8u) {
                    uint32_t d[PW][4];
#pragma unroll
                    for (int p = 0; p < PW; ++p) {
                        const uintx4 v = *reinterpret_cast<Lds4>((uintptr_t)(a.mine + (uint32_t)p * kPlane + row * kPitch + 2u * k));
#pragma unroll
                        for (int i = 0; i < 4; ++i) d[p][i] = v[i];
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        float piece[PW];
                        bool indexed = false;
#pragma unroll
                        for (int p = 0; p < PW; ++p) {
                            const uint32_t u = i & 1 ? d[p][i >> 1] & 0xFFFF0000u : d[p][i >> 1] << 16;
                            piece[p] = __uint_as_float(u);
                            indexed |= u != a.fill[p] << 16;
                        }
                        float w = piece[0];
                        if constexpr (kForm == kUniform) w = fmaf(a.grid.scale, piece[0], a.grid.scale * piece[PW - 1]);
                        if constexpr (kForm == 3) w = piece[0] + (piece[PW > 1 ? 1 : 0] + piece[PW - 1]);
                        if (!dense) w -= a.omega0;
#pragma unroll
                        for (int j = 0; j < kCols; ++j) {
                            const float xs = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x[j]), (int)(k + i)));
                            if (dense ? k0 + k + i < a.n : indexed) y[j] = fmaf(w, xs, y[j]);
                        }
                    }
                }
            }
        };
        if (count == 1u) walk(std::integral_constant<int, 1>()); else walk(std::integral_constant<int, 4>());
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            s_sum[(a.wave * 4u + j) * kWave + a.lane] = y[j];
            s_x[(a.wave * 4u + j) * kWave + a.lane] = sum[j];
        }
        __syncthreads();
        const uint32_t j = threadIdx.x >> 6;
        if (j < count && a.lane < R && a.row0 + a.lane < a.m) {
            double total = 0, ones = 0;
            for (uint32_t k = 0; k < kTileWaves; ++k) total += s_sum[(k * 4u + j) * kWave + a.lane];
            if (!dense && a.omega0 != 0.f) {
                for (uint32_t k = 0; k < kTileWaves; ++k)
                    for (uint32_t i = 0; i < kWave; ++i) ones += s_x[(k * 4u + j) * kWave + i];
                total = fma((double)a.omega0, (double)(float)ones, total);
            }
            a.out[(size_t)(a.row0 + a.lane) * a.L + (j == 0u ? c[0] : (j == 1u ? c[1] : (j == 2u ? c[2] : c[3])))] = (float)total;
        }
    }
}

// quads: the buckets, in fours of entries; quad 0 has entries that go nowhere.  ptr[group][segment]: its first quad.
template <int kForm, int RT, int CT, int kQ>
__global__ __launch_bounds__(kTileThreads) void cer_tile_kernel(const uint4* quads, const uint32_t* ptr, const float* X, uint32_t m, uint32_t n,
                                                                uint32_t L, uint32_t row_magic, uint32_t eighth, uint32_t packed, TileRest rest,
                                                                UniformGrid grid) {
    constexpr int PW = weight_planes(kForm);
    constexpr uint32_t R = 16 * RT, BN = 16 * CT, kPlane = RT * kGroupBytes, kLanes = kWave / RT;  // lanes per group of 16 rows
    constexpr int kSteps = kSegCols / 32;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid >> 6);
    const uint32_t c16 = lane & 15u, g = lane >> 4;
    const uint32_t item = (blockIdx.x & 7u) * eighth + (blockIdx.x >> 3), row_blocks = (m + R - 1u) / R;
    const uint32_t over = row_magic ? (uint32_t)(((uint64_t)item * row_magic) >> 32) : item, rt = item - over * row_blocks;
    const uint32_t splits = packed >> 16, per = packed & 0xFFFFu, segs = (n + kSegCols - 1u) / kSegCols;
    const uint32_t ct = splits == 1u ? over : over / splits, sp = over - ct * splits;
    const uint32_t row0 = rt * R, col0 = ct * BN, h0 = sp * per, h1 = min(segs, h0 + per);
    if ((blockIdx.x >> 3) >= eighth || col0 >= L || h0 >= h1) return;

    const uint32_t groups = (m + kGroupRows - 1u) / kGroupRows, group = row0 / kGroupRows + lane / kLanes;
    const uint32_t* bounds = ptr + (size_t)min(group, groups - 1u) * (segs + 1u);
    auto bounds_of = [&](uint32_t h) { return *reinterpret_cast<const TwoBounds*>(bounds + min(h, segs - 1u)); };
    TwoBounds bound = bounds_of(h0 + wave);
    const float* omega = rest.omega;
    const float omega0 = omega[0], value = omega[min(tid, rest.values)];

    const uint32_t xcol = min(col0 + CT * c16, L - (uint32_t)CT);
    uint32_t xoff[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) xoff[i] = ((8u * g + i) * L + xcol) * 4u;
    float x[kSteps][8][CT];
    auto load_x = [&](uint32_t k0, float (&v)[8][CT]) {
        const __amdgpu_buffer_rsrc_t xbuf = x_rows(X, L, min(k0, n), n);
#pragma unroll
        for (int i = 0; i < 8; ++i) load_columns<CT>(xbuf, xoff[i], v[i]);
    };
    // a bucket's first entries; lanes that have none take the quad that goes nowhere
    uint4 q[kQ];
    uint32_t cb = 0, ce = 0;
    auto request = [&](uint32_t h) {
        cb = bound[0] + lane % kLanes;
        ce = group < groups && h < h1 ? bound[1] : 0u;
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            const uint32_t i = cb + (uint32_t)u * kLanes;
            q[u] = quads[i < ce ? i : 0u];
        }
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const uint32_t mine = lds0 + planes_at(kForm) + wave * wave_bytes(kForm, RT);
    uint32_t fill[PW];
    fill_pieces<kForm>(omega0, grid, fill);
    auto scatter = [&]() {
        clear_planes<kForm, RT>(mine, fill, lane);
        const uint32_t to = mine + lane / kLanes * kGroupBytes;
#pragma unroll
        for (int u = 0; u < kQ; ++u) place_quad<kForm, RT>(to, smem, q[u]);
        for (uint32_t c = cb + (uint32_t)kQ * kLanes; __ballot(c < ce) != 0ull; c += kLanes) place_quad<kForm, RT>(to, smem, quads[c < ce ? c : 0u]);
    };
    floatx4 acc[RT][CT] = {}, lo[RT][CT] = {}, sum[kForm == 3 ? RT : 1][kForm == 3 ? CT : 1] = {};
    uint32_t lost = 0;
    auto joined = [&](int r, int c) {
        floatx4 v = acc[r][c] + lo[r][c];
        if constexpr (kForm == kUniform)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(grid.scale, acc[r][c][e], grid.scale * lo[r][c][e]);
        if constexpr (kForm == 3) v += sum[r][c];
        return v;
    };
    auto multiply = [&](uint32_t t, const float (&v)[8][CT]) {
        typedef const uintx4 __attribute__((address_space(3))) * Lds4;
        uint4 w[RT][PW];
        const uint32_t at = mine + c16 * kPitch + t * 64u + g * 16u;
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int p = 0; p < PW; ++p) {
                const uintx4 a = *reinterpret_cast<Lds4>((uintptr_t)(at + (uint32_t)p * kPlane + (uint32_t)r * kGroupBytes));
                w[r][p] = make_uint4(a[0], a[1], a[2], a[3]);
            }
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

    uint32_t h = h0 + wave;
    request(h);
    bound = bounds_of(h + kTileWaves);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) load_x(h * kSegCols + 32u * s, x[s]);
    uint32_t* const flags = reinterpret_cast<uint32_t*>(smem);
    if (tid < 8u) flags[tid] = 0u;
    if (kForm != 1 && tid <= rest.values) {
        uint32_t p[3];
        if constexpr (kForm == kUniform) {
            reinterpret_cast<uint32_t*>(smem + kTileTableAt)[tid] = uniform_pieces(value, grid);
        } else {
            split3_finite(value, p);
            reinterpret_cast<uint2*>(smem + kTileTableAt)[tid] = make_uint2(p[0] | (p[1] << 16), p[2]);
        }
    }
    __syncthreads();
    for (uint32_t it = wave >> 2; h < h1; h += kTileWaves, ++it) {
        if (it & 1u) __builtin_amdgcn_s_setprio(1); else __builtin_amdgcn_s_setprio(0);
        wave_lds_sync();
        scatter();
        wave_lds_sync();
        // (matrix and LDS instructions by turns: 1737 x 8986, 36 values, batch 198 54.3 -> 49.2 us, 4052 x 10595, 9 values, 87 46.2 -> 44.6,
        // 2247 x 10262, 3 values, 63 28.5 -> 27.8; one piece, AlexNet-fc6 shape, 99 36.6 -> 37.8; three pieces 1.00 times the time)
        if constexpr (kForm == kUniform) __builtin_amdgcn_iglp_opt(1);
        request(h + kTileWaves);
        bound = bounds_of(h + 2u * kTileWaves);
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            multiply((uint32_t)s, x[s]);
            load_x((h + kTileWaves) * kSegCols + 32u * s, x[s]);
        }
        if constexpr (kForm == 3)
            if (it & 1u) {  // running sums of four steps, as in cer_fused_kernel
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        sum[r][c] = joined(r, c);
                        acc[r][c] = lo[r][c] = floatx4{};
                    }
            }
    }
    __syncthreads();

    // the waves' sums meet in LDS: [wave][row tile][element][column of CT][lane]
    float* s_sum = reinterpret_cast<float*>(smem + planes_at(kForm));
    constexpr uint32_t kPer = RT * CT * 4 * kWave;
    if ((lost & 0xFFFFu) != 0u) atomicOr(&flags[kTileLossy], 1u << c16);
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const floatx4 v = joined(r, c);
#pragma unroll
            for (int e = 0; e < 4; ++e) s_sum[wave * kPer + ((r * 4 + e) * CT + c) * kWave + lane] = v[e];
        }
    __syncthreads();
    // accumulator element e of lane l: row 4 (l / 16) + e, column l % 16
    constexpr uint32_t kVec = RT * 4 * kWave / kTileThreads;
    static_assert(kVec >= 1, "threads");
    const float least = (flags[kTileLossy] >> c16) & 1u ? rest.faint : 0.f;
    uint32_t odd = 0, faint = 0;  // of the lane's columns
    float* out = rest.Out + sp * rest.split_stride;
#pragma unroll
    for (uint32_t v = 0; v < kVec; ++v) {
        const uint32_t i = tid + v * kTileThreads, re = i >> 6, r = 16u * (re >> 2) + 4u * g + (re & 3u), row = row0 + r;
        const uint32_t first = col0 + CT * c16;
        float y[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const float* s = s_sum + (re * CT + c) * kWave + lane;
            double total = s[0];
#pragma unroll
            for (uint32_t k = 1; k < kTileWaves; ++k) total += s[k * kPer];
            y[c] = (float)total;
            const float size = fabsf(y[c]);
            if (row < m && xcol + c >= first) {
                odd |= size < INFINITY ? 0u : 1u << c;
                faint |= size < least || (size < 0x1p-126f && size > 0.f) ? 1u << c : 0u;
            }
        }
        if (row < m) {
            float* to = out + (size_t)row * L + xcol;
            if (CT == 4 && xcol == first) {
                *reinterpret_cast<FourFloats*>(to) = FourFloats{y[0], y[1], y[CT > 2 ? 2 : 0], y[CT > 3 ? 3 : 0]};
            } else {
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    if (xcol + c >= first) to[c] = y[c];
            }
        }
    }
    if (__ballot((odd | faint) != 0u) != 0ull) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const uint32_t column = xcol + c - col0;
            if ((odd >> c) & 1u) atomicOr(&flags[kOddColumns + (column >> 5)], 1u << (column & 31u));
            if ((faint >> c) & 1u) atomicOr(&flags[kFaintColumns + (column >> 5)], 1u << (column & 31u));
        }
    }
    __syncthreads();
    const uint32_t odd0 = uniform(flags[kOddColumns]), odd1 = uniform(flags[kOddColumns + 1]);
    if ((odd0 | odd1 | flags[kFaintColumns] | flags[kFaintColumns + 1]) == 0u) return;
    // columns with sums that are not finite, and where inputs have lost bits those with faint ones, are formed again
    if (tid == 0)
        *reinterpret_cast<TileArgs*>(smem + kTileArgsAt) =
            TileArgs{quads, ptr, X, omega, out, grid.inverse, grid.scale, grid.unit, rest.faint, rest.most, m, n, L, row0, col0, BN, h0, h1, rest.dense};
    __syncthreads();
    if ((odd0 | odd1) != 0u) tile_again_columns<kForm, RT, CT, false>(lds0, odd0, odd1);
    const uint32_t faint0 = uniform(flags[kFaintColumns]), faint1 = uniform(flags[kFaintColumns + 1]);
    if ((faint0 | faint1) != 0u) tile_again_columns<kForm, RT, CT, true>(lds0, faint0, faint1);
    const uint32_t slow0 = uniform(flags[kSlowColumns]), slow1 = uniform(flags[kSlowColumns + 1]);
    if ((slow0 | slow1) != 0u) tile_slow<kForm, RT>(lds0, slow0, slow1);
}

// The tile index of 16 rows, one per wave: their elements are counted by segment, then placed.  An entry: its place in the group's
// rows of a plane | 16 more bits: its value where that is one bf16 number, else its rank.  Buckets are filled up to whole quads with
// entries that go behind the first row's segment, where nothing is read.
// The order inside a bucket does not matter: every entry has a place of its own.
template <bool kValues>
__global__ __launch_bounds__(kGroupRows* kWave) void tile_index_kernel(const uint32_t* tab, const uint16_t* colI,
                                                                               const float* omega, uint32_t m, uint32_t n, uint32_t tab_shift,
                                                                               uint32_t room, uint32_t* ptr, uint32_t* entries) {
    constexpr uint32_t RW = kGroupRows, SEG = kSegCols, P = kPitch, kThreads = RW * kWave;
    constexpr uint32_t kNowhere = 2u * SEG;  // the place behind a segment of the first row
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid >> 6);
    uint32_t* count = reinterpret_cast<uint32_t*>(smem + index_counts_at(RW));  // of the segments; then the next entry's place
    uint16_t* payload = reinterpret_cast<uint16_t*>(smem + index_payload_at(RW) + wave * payload_bytes(tab_shift));
    uint32_t* stage = reinterpret_cast<uint32_t*>(smem + index_stage_at(RW, tab_shift));
    const uint32_t group = blockIdx.x, row0 = group * RW, row = row0 + wave, segs = (n + SEG - 1u) / SEG;
    const uint32_t last_word = (1u << tab_shift) - 1u, ntiles = (last_word >> 6) + 1u;
    // the rows' positions follow one another; the last row's end is its record's last word
    const uint32_t p0 = uniform(tab[(size_t)row0 << tab_shift]);
    const uint32_t p1 = uniform(row0 + RW < m ? tab[(size_t)(row0 + RW) << tab_shift] : tab[((size_t)(m - 1u) << tab_shift) + last_word]);
    uint32_t rec[4] = {};
    float own[4] = {};
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t)
        if (t < ntiles) {
            rec[t] = tab[((size_t)min(row, m - 1u) << tab_shift) + min(t * kWave + lane, last_word)];
            own[t] = omega[min(t * kWave + lane + 1u, last_word)];
        }
    uint4 first[Shape::NW];
    request_batch(colI, first, uniform(rec[0]) & ~((uint32_t)Shape::PPL - 1u), row_end(rec, last_word), lane);
    if (tid < 256u) prefix_entry(smem, tid);
    if (tid < kCounts - 4u) count[tid] = 0u;
    __syncthreads();
    for (uint32_t p = (p0 & ~7u) + 8u * tid; p < p1; p += 8u * kThreads) {
        const uint4 q = *reinterpret_cast<const uint4*>(colI + p);
        const uint32_t c[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i)
            if (p + i >= p0 && p + i < p1) atomicAdd(&count[(i & 1u ? c[i >> 1] >> 16 : c[i >> 1] & 0xFFFFu) / SEG], 1u);
    }
    __syncthreads();
    const uint32_t base = group_base(p0, group, segs);
    if (wave == 0) {
        constexpr uint32_t kEach = (kCounts - 4u) / kWave;
        uint32_t before[kEach], sum = 0;
#pragma unroll
        for (uint32_t i = 0; i < kEach; ++i) {
            before[i] = sum;
            sum += (count[kEach * lane + i] + 3u) & ~3u;
        }
        const uint32_t incl = wave_inclusive_scan(sum);
#pragma unroll
        for (uint32_t i = 0; i < kEach; ++i) {
            const uint32_t s = kEach * lane + i, at = incl - sum + before[i];
            count[s] = at;
            if (s <= segs) ptr[(size_t)group * (segs + 1u) + s] = (base + at) >> 2;
        }
        if (lane == kWave - 1u) count[kCounts - 4u] = incl;
    }
    if (group == 0 && tid < 4u) entries[tid] = kNowhere;
    __syncthreads();
    const uint32_t total = uniform(count[kCounts - 4u]);
    const bool staged = total <= room;
    if (staged) {
        for (uint32_t i = tid; i < total; i += kThreads) stage[i] = kNowhere;
    } else {
        for (uint32_t i = tid; i < total; i += kThreads) entries[base + i] = kNowhere;
        __threadfence();
    }
    __syncthreads();
    if (row < m) {
        uint32_t to = wave * P;  // the row's place
        auto walk = [&](auto put) {
            walk_row(colI, rec, first, tab_shift, smem, wave, lane,
                     [&](uint32_t at, uint32_t t) {
                         const uint32_t rank = t * kWave + lane + 1u;
                         payload[at] = kValues ? (uint16_t)(__float_as_uint(own[t]) >> 16) : (uint16_t)rank;
                     },
                     [&](uint32_t cols, uint32_t two) {
#pragma unroll
                         for (int i = 0; i < 2; ++i) {
                             const uint32_t col = i ? cols >> 16 : cols & 0xFFFFu;
                             if (col != 0xFFFFu)
                                 put(atomicAdd(&count[col / SEG], 1u), (to + 2u * (col % SEG)) | (uint32_t)payload[(two >> (8 * i)) & 0xFFu] << 16);
                         }
                     });
        };
        if (staged) walk([&](uint32_t at, uint32_t e) { stage[at] = e; });
        else walk([&](uint32_t at, uint32_t e) { entries[base + at] = e; });
    }
    if (!staged) return;
    __syncthreads();
    for (uint32_t i = tid; i < total / 4u; i += kThreads) reinterpret_cast<uint4*>(entries + base)[i] = reinterpret_cast<const uint4*>(stage)[i];
}

// The sums of the parts of W's columns, in their order, four at a time.
__global__ __launch_bounds__(256) void tile_sum_kernel(const float* __restrict__ part, float* __restrict__ Y, size_t count, size_t stride, uint32_t splits) {
    const size_t i = 4u * ((size_t)blockIdx.x * 256 + threadIdx.x);
    if (i >= count) return;
    double a[4] = {};
    uint32_t s = 0;
    for (; s + 4u <= splits; s += 4u) {  // four on their way at a time
        FourFloats b[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) b[k] = *reinterpret_cast<const FourFloats*>(part + (s + k) * stride + i);
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] += b[k][e];
    }
    for (; s < splits; ++s) {
        const FourFloats b = *reinterpret_cast<const FourFloats*>(part + s * stride + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] += b[e];
    }
    if (i + 4u <= count) {
        *reinterpret_cast<FourFloats*>(Y + i) = FourFloats{(float)a[0], (float)a[1], (float)a[2], (float)a[3]};
    } else {
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e)
            if (i + e < count) Y[i + e] = (float)a[e];
    }
}

typedef void (*TileKernel)(const uint4*, const uint32_t*, const float*, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t, TileRest, UniformGrid);
typedef void (*IndexKernel)(const uint32_t*, const uint16_t*, const float*, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t*, uint32_t*);

// The variants, and the terms of their duration in microseconds, fitted to 470 random products of 8 to 1200 columns (typical
// deviation 5 to 11 %).  A launch takes `fixed`; then the busiest compute unit's workgroups follow one another, each `round`, and `seg` +
// `quad` per quad of entries and lane for 64 columns per wave; the second launch `sum` and `traffic` per MB of parts.
struct Variant {
    int form, rt, ct, rounds;
    float fixed, round, seg, quad, sum, traffic;
    TileKernel kernel;
};
const Variant kVariants[] = {
    {1, 4, 1, 1, 0.46f, 1.73f, 1.057f, 0.225f, 4.15f, 0.47f, cer_tile_kernel<1, 4, 1, 1>},
    {1, 4, 1, 3, 0.46f, 1.73f, 1.057f, 0.225f, 4.15f, 0.47f, cer_tile_kernel<1, 4, 1, 3>},
    {1, 4, 2, 1, 0.99f, 2.34f, 1.464f, 0.270f, 3.58f, 0.46f, cer_tile_kernel<1, 4, 2, 1>},
    {1, 4, 2, 3, 0.99f, 2.34f, 1.464f, 0.270f, 3.58f, 0.46f, cer_tile_kernel<1, 4, 2, 3>},
    {1, 4, 3, 1, 0.00f, 3.60f, 2.003f, 0.276f, 3.59f, 0.50f, cer_tile_kernel<1, 4, 3, 1>},
    {1, 4, 3, 3, 0.00f, 3.60f, 2.003f, 0.276f, 3.59f, 0.50f, cer_tile_kernel<1, 4, 3, 3>},
    {1, 4, 4, 1, 0.00f, 4.44f, 2.436f, 0.285f, 3.10f, 0.68f, cer_tile_kernel<1, 4, 4, 1>},
    {1, 4, 4, 3, 0.00f, 4.44f, 2.436f, 0.285f, 3.10f, 0.68f, cer_tile_kernel<1, 4, 4, 3>},
    {kUniform, 4, 1, 1, 1.35f, 0.81f, 1.749f, 0.290f, 4.05f, 0.29f, cer_tile_kernel<kUniform, 4, 1, 1>},
    {kUniform, 4, 1, 3, 1.35f, 0.81f, 1.749f, 0.290f, 4.05f, 0.29f, cer_tile_kernel<kUniform, 4, 1, 3>},
    {kUniform, 4, 2, 1, 0.58f, 2.40f, 2.089f, 0.323f, 4.27f, 0.38f, cer_tile_kernel<kUniform, 4, 2, 1>},
    {kUniform, 4, 2, 3, 0.58f, 2.40f, 2.089f, 0.323f, 4.27f, 0.38f, cer_tile_kernel<kUniform, 4, 2, 3>},
    {kUniform, 4, 3, 1, 0.45f, 2.68f, 2.673f, 0.322f, 4.20f, 0.58f, cer_tile_kernel<kUniform, 4, 3, 1>},
    {kUniform, 4, 3, 3, 0.45f, 2.68f, 2.673f, 0.322f, 4.20f, 0.58f, cer_tile_kernel<kUniform, 4, 3, 3>},
    {3, 2, 2, 1, 0.37f, 2.51f, 1.927f, 0.350f, 4.23f, 0.48f, cer_tile_kernel<3, 2, 2, 1>},
    {3, 2, 2, 3, 0.37f, 2.51f, 1.927f, 0.350f, 4.23f, 0.48f, cer_tile_kernel<3, 2, 2, 3>},
    {3, 2, 4, 1, 0.00f, 3.09f, 2.775f, 0.377f, 3.73f, 0.94f, cer_tile_kernel<3, 2, 4, 1>},
    {3, 2, 4, 3, 0.00f, 3.09f, 2.775f, 0.377f, 3.73f, 0.94f, cer_tile_kernel<3, 2, 4, 3>},
};
constexpr int kVariantCount = sizeof(kVariants) / sizeof(kVariants[0]);

int form_of(const DeviceView& d) { return d.grid.scale != 0.f ? kUniform : (d.pieces == 1 ? 1 : 3); }

bool index_applicable(const DeviceView& d) {
    if (!d.rank_tab || d.pieces < 1 || d.colI_bits != 16 || d.n < 1 || d.n > 65000 || d.m < 1 || d.m > (1 << 24) || d.lds_per_block < 160 * 1024) return false;
    const TileIndexShape s = tile_index_shape(d);
    return (uint64_t)d.nnz + 3ull * s.segs * s.groups + 64u < (1ull << 32);
}

bool tile_applicable(const DeviceView& d, uint32_t L) {
    return index_applicable(d) && L >= 2 && L <= (1u << 20) && ((uint64_t)d.n + 600) * L * 4u < (1ull << 32);
}

}  // namespace

// A call waits for this search (0.1 to 0.2 us): variants, and numbers of parts, that cannot be below the best so far are not
// looked at.  For their rounds times the waves' segments are at least the workgroups' segments by the compute units, and parts cost their sum.
TilePlan plan_tile(const DeviceView& d, uint32_t L, bool temporaries, double below) {
    TilePlan best;
    best.us = below;
    if (!d.tile_index || !tile_applicable(d, L)) return best;
    const int form = form_of(d);
    const TileIndexShape shape = tile_index_shape(d);
    const uint32_t segs = shape.segs, cus = (uint32_t)std::max(d.cus, 1);
    const uint32_t most = temporaries ? std::min((segs + kTileWaves - 1u) / kTileWaves, 16u) : 1u;
    const double quads = (double)d.nnz / ((double)segs * shape.groups) / 4.0, out_bytes = (double)d.m * L * 4.0;
    for (int v = 0; v < kVariantCount; ++v) {
        const Variant& k = kVariants[v];
        if (k.form != form || (uint32_t)k.ct > L) continue;
        const double per_lane = quads * k.rt / kWave;
        if ((k.rounds == 1) != (per_lane <= 0.85)) continue;
        TilePlan p;
        p.variant = v;
        const uint32_t R = 16u * k.rt;
        p.row_blocks = (uint32_t)((d.m + R - 1) / R);
        p.col_tiles = (L + 16u * k.ct - 1) / (16u * k.ct);
        const uint64_t tiles = (uint64_t)p.row_blocks * p.col_tiles;
        const double each = k.seg + k.quad * std::max(per_lane, 0.5);
        const double least = k.fixed + k.round + std::max(1.0, (double)tiles * segs / ((double)kTileWaves * cus)) * each;
        for (uint32_t sp = 1; sp <= most; ++sp) {
            if (least + (sp > 1 ? k.sum + 3.0 * out_bytes * 1e-6 * k.traffic : 0.0) >= best.us) break;
            p.per = (segs + sp - 1) / sp;
            p.splits = (segs + p.per - 1) / p.per;
            const double part_bytes = p.splits * out_bytes;
            if (p.splits > 1 && part_bytes > (double)(1ull << 30)) break;
            if (tiles * p.splits * p.row_blocks >= (1ull << 32)) break;  // (the kernel divides by multiplication)
            const double rounds = (double)((tiles * p.splits + cus - 1u) / cus), waves = (double)((p.per + kTileWaves - 1u) / kTileWaves);
            p.us = k.fixed + rounds * (k.round + waves * each);
            if (p.splits > 1) p.us += k.sum + (part_bytes + out_bytes) * 1e-6 * k.traffic;
            if (p.us < best.us) best = p;
        }
    }
    if (best.variant >= 0) {
        const Variant& k = kVariants[best.variant];
        best.lds = planes_at(form) + std::max<size_t>(kTileWaves * wave_bytes(form, k.rt), (size_t)kTileWaves * k.rt * k.ct * 1024u);
    }
    return best;
}

TileIndexShape tile_index_shape(const DeviceView& d) {
    TileIndexShape s;
    s.segs = (uint32_t)((d.n + kSegCols - 1) / kSegCols);
    s.groups = (uint32_t)((d.m + kGroupRows - 1) / kGroupRows);
    s.ptr_bytes = ((size_t)s.groups * (s.segs + 1u) * 4u + 255u) & ~(size_t)255u;
    s.bytes = s.ptr_bytes + ((size_t)d.nnz + (size_t)3u * s.segs * s.groups + 16u) * 4u;
    return s;
}

hipError_t launch_tile_index(const DeviceView& d, void* index, hipStream_t stream) {
    const TileIndexShape s = tile_index_shape(d);
    const uint32_t shift = (uint32_t)d.rank_tab_shift, stage = index_stage_at(kGroupRows, shift);
    const bool values = form_of(d) == 1;
    const IndexKernel kernel = values ? tile_index_kernel<true> : tile_index_kernel<false>;
    static LdsGrant<2> grant;
    const hipError_t e = grant.ensure(values ? 0 : 1, reinterpret_cast<const void*>(kernel), d.lds_per_block);
    if (e != hipSuccess) return e;
    const double mean = (double)d.nnz / s.groups + 3.0 * s.segs;
    const uint32_t room = (uint32_t)std::min(mean * 1.25 + 512.0, (double)((d.lds_per_block - 1024 - stage) / 4)) & ~3u;
    return launch_kernel(kernel, dim3(s.groups), dim3(kGroupRows * kWave), (size_t)stage + 4u * room, stream, d.rank_tab, static_cast<const uint16_t*>(d.colI),
                         d.omega, (uint32_t)d.m, (uint32_t)d.n, shift, room, static_cast<uint32_t*>(index),
                         reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(index) + s.ptr_bytes));
}

size_t tile_index_bytes(const DeviceView& d) { return index_applicable(d) ? tile_index_shape(d).bytes : 0; }

int build_tile_index(const DeviceView& d, void* index, void* stream) { return (int)launch_tile_index(d, index, static_cast<hipStream_t>(stream)); }

int tile_columns(const TilePlan& p) { return p.variant >= 0 ? 16 * kVariants[p.variant].ct : 0; }

hipError_t launch_tile(const DeviceView& d, const TilePlan& p, const float* X, float* Y, uint32_t L, bool dense_zeros, hipStream_t stream) {
    if (p.variant < 0) return hipErrorInvalidValue;
    const Variant& k = kVariants[p.variant];
    {
        static LdsGrant<kVariantCount> grant;
        const hipError_t e = grant.ensure(p.variant, reinterpret_cast<const void*>(k.kernel), d.lds_per_block);
        if (e != hipSuccess) return e;
    }
    const TileIndexShape s = tile_index_shape(d);
    float* part = nullptr;
    TileRest a;
    a.split_stride = ((size_t)d.m * L + 3u) & ~(size_t)3u;
    hipError_t e = hipSuccess;
    if (p.splits > 1) e = (hipError_t)temp_alloc(reinterpret_cast<void**>(&part), a.split_stride * p.splits * 4u, stream);
    if (e == hipSuccess) {
        a.Out = part ? part : Y;
        a.omega = d.omega;
        a.values = (uint32_t)d.K - 1u;
        a.faint = (float)std::min((double)d.n * d.omega_max * 0x1p-108, 1e38);
        // sums of terms this large times 2^64 stay below 2^126 on their way; and the inputs below 2^62
        a.most = (float)(0x1p62 / std::max((double)d.n * d.omega_max, 1.0));
        a.dense = dense_zeros ? 1u : 0u;
        const uint32_t items = p.row_blocks * p.col_tiles * p.splits, eighth = (items + 7u) / 8u;
        const uint32_t magic = p.row_blocks == 1 ? 0u : (uint32_t)(((1ull << 32) + p.row_blocks - 1) / p.row_blocks);
        e = launch_kernel(k.kernel, dim3(eighth * 8u), dim3(kTileThreads), p.lds, stream,
                          reinterpret_cast<const uint4*>(static_cast<const unsigned char*>(d.tile_index) + s.ptr_bytes), static_cast<const uint32_t*>(d.tile_index), X,
                          (uint32_t)d.m, (uint32_t)d.n, L, magic, eighth, p.per | p.splits << 16, a, d.grid);
    }
    if (part) {
        const size_t count = (size_t)d.m * L;
        if (e == hipSuccess)
            e = launch_kernel(tile_sum_kernel, dim3((uint32_t)((count + 1023u) / 1024u)), dim3(256), 0, stream, part, Y, count, a.split_stride, p.splits);
        const hipError_t f = (hipError_t)temp_free(part, stream);
        if (e == hipSuccess) e = f;
    }
    return e;
}

}  // namespace cer
