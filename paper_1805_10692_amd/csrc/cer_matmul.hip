// cer_matmul / cser_matmul: choice of the product kernel for a handle and a batch width, the column sums of X for
// a non-zero most frequent value (Appendix A-A1), and the decode + dense route.
#include "cer_device.hpp"

// Workspace of the entry point that allocates nothing: one array per GPU, part of the loaded code object, so it
// exists from the moment the library is loaded on a device until the process ends.  Host code never uses the
// array's name as an address: the address on the current device comes from hipGetSymbolAddress, once per device.
// (No `used` attribute: it keeps the symbol local to the code object, where the runtime's look-up by name cannot find it.)
constexpr size_t kStaticWorkspaceFloats = 512 * 1024;  // 2 MiB
static __device__ __align__(256) float scratch[kStaticWorkspaceFloats];

namespace cer {
namespace {

// ------------------------------------------------------------------------------------------------
// Column sums of X (Appendix A-A1): T[l] = sum_i X[i,l], in two stages of short partial sums.
// ------------------------------------------------------------------------------------------------

// block (bx, by): columns [bx*CB, +CB), rows [by*slab, +slab).  CB divides 256.
__global__ __launch_bounds__(256) void colsum_partial_kernel(const float* __restrict__ X, uint32_t n, uint32_t L,
                                                             uint32_t CB, uint32_t slab, float* __restrict__ part) {
    __shared__ float red[256];
    const uint32_t cl = threadIdx.x % CB, rl = threadIdx.x / CB, RPB = 256u / CB;
    const uint32_t col = blockIdx.x * CB + cl;
    const uint32_t i0 = blockIdx.y * slab, i1 = min(n, i0 + slab);
    float a0 = 0.f, a1 = 0.f;
    if (col < L) {
        uint32_t i = i0 + rl;
        for (; i + RPB < i1; i += 2 * RPB) {
            a0 += X[(size_t)i * L + col];
            a1 += X[(size_t)(i + RPB) * L + col];
        }
        if (i < i1) a0 += X[(size_t)i * L + col];
    }
    red[threadIdx.x] = a0 + a1;
    __syncthreads();
    for (uint32_t s = RPB >> 1; s > 0; s >>= 1) {
        if (rl < s) red[threadIdx.x] += red[threadIdx.x + s * CB];
        __syncthreads();
    }
    if (rl == 0 && col < L) part[(size_t)blockIdx.y * L + col] = red[cl];
}

// The same for wide batches (L a multiple of 4, X 16-byte aligned): a thread owns four columns and reads them with
// 16-byte loads, four rows in flight.  block (bx, by): columns [bx*1024, +1024), rows [by*slab, +slab).
__global__ __launch_bounds__(256) void colsum_partial4_kernel(const float* __restrict__ X, uint32_t n, uint32_t L,
                                                              uint32_t slab, float* __restrict__ part) {
    typedef float F4 __attribute__((ext_vector_type(4)));
    const uint32_t col = (blockIdx.x * 256u + threadIdx.x) * 4u;
    if (col >= L) return;
    const uint32_t i0 = blockIdx.y * slab, i1 = min(n, i0 + slab);
    const F4* p = reinterpret_cast<const F4*>(X + col);
    const size_t pitch = L >> 2;
    F4 a0 = F4{0.f, 0.f, 0.f, 0.f}, a1 = a0, a2 = a0, a3 = a0;
    uint32_t i = i0;
    for (; i + 4 <= i1; i += 4) {
        const F4 x0 = p[(size_t)i * pitch], x1 = p[(size_t)(i + 1) * pitch], x2 = p[(size_t)(i + 2) * pitch],
                 x3 = p[(size_t)(i + 3) * pitch];
        a0 += x0; a1 += x1; a2 += x2; a3 += x3;
    }
    for (; i < i1; ++i) a0 += p[(size_t)i * pitch];
    *reinterpret_cast<F4*>(part + (size_t)blockIdx.y * L + col) = (a0 + a1) + (a2 + a3);
}

// block: CB columns (a power of two up to 256), the slabs dealt to its 256 / CB groups of threads, eight in flight each (a
// single thread per column took 15 us for 344 slabs).
__global__ __launch_bounds__(256) void colsum_final_kernel(const float* __restrict__ part, uint32_t nslabs, uint32_t L,
                                                           uint32_t CB, float* __restrict__ T) {
    __shared__ float red[256];
    const uint32_t cl = threadIdx.x % CB, g = threadIdx.x / CB, G = 256u / CB, col = blockIdx.x * CB + cl;
    float a = 0.f;
    if (col < L) {
        const float* p = part + col;
        uint32_t s = g;
        for (; s + 7u * G < nslabs; s += 8u * G) {  // added in slab order
            float b[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) b[k] = p[(size_t)(s + k * G) * L];
#pragma unroll
            for (int k = 0; k < 8; ++k) a += b[k];
        }
        for (; s < nslabs; s += G) a += p[(size_t)s * L];
    }
    red[threadIdx.x] = a;
    __syncthreads();
    for (uint32_t s = G >> 1; s > 0; s >>= 1) {
        if (g < s) red[threadIdx.x] += red[threadIdx.x + s * CB];
        __syncthreads();
    }
    if (g == 0 && col < L) T[col] = red[cl];
}

hipError_t launch_colsum(const float* X, uint32_t n, uint32_t L, float* part, uint32_t nslabs, uint32_t slab,
                         uint32_t CB, float* T, hipStream_t stream) {
    const uint32_t coltiles = (L + CB - 1) / CB;
    hipError_t e;
    if (L >= 1024u && L % 4u == 0 && (reinterpret_cast<uintptr_t>(X) & 15u) == 0 && (reinterpret_cast<uintptr_t>(part) & 15u) == 0)
        e = launch_kernel(colsum_partial4_kernel, dim3((L + 1023u) / 1024u, nslabs), dim3(256), 0, stream, X, n, L, slab, part);
    else
        e = launch_kernel(colsum_partial_kernel, dim3(coltiles, nslabs), dim3(256), 0, stream, X, n, L, CB, slab, part);
    if (e != hipSuccess) return e;
    const uint32_t FB = std::min<uint32_t>(CB, 32u);
    return launch_kernel(colsum_final_kernel, dim3((L + FB - 1) / FB), dim3(256), 0, stream, part, nslabs, L, FB, T);
}

// Large batches of a matrix that is not sparse enough: the gathers move a line of X per indexed element and 32 columns
// (gemm_gather_us), the matrix cores need 2.m.n.batch flops however many elements are indexed.  The matrix is then decoded into a
// stream-ordered temporary (bounded here) and multiplied on the matrix cores: as bf16 pieces (cer_mfma.hip: 2 to 6 bytes per
// element written, three to six products at about 900 TFLOP/s), or, where the values or the sizes rule that out, as fp32 (4 bytes
// per element; 90 - 120 TFLOP/s).  Measured on MI355X, gathers against decode + product: 3x3 convolution shape (60 % zeros)
// batch 3136 391 / 53 us (fp32: 149 us).
//
// Estimated duration (seconds) of the kernel that gathers from L2.
//   * bytes and steps: gemm_gather_us (lines per index, gather instructions, the walk of the longest row: 543 x 7364, batch 28, 4900
//     positions per row, 28 us)
//   * waves: every (row, tile) is a wave whose start-up chain (descriptor -> pointers -> indices -> first gathers) takes about
//     4 us, 4096 of them in flight: what bounds matrices of many short rows (16384 x 512: batch 128 64 - 84 us)
//   * the column sums of X for a non-zero most frequent value: two launches and a pass over X
// A call asks for it several times (0.3 us of the host's time each): gathers_us, gemm_gather_us where that is known already.
double gather_estimate(const DeviceView& d, uint32_t L, double* gathers_us) {
    const double tiles = std::ceil((double)L / 32.0);
    const double t_waves = (double)d.m * tiles * 4e-6 / 4096.0;
    if (*gathers_us < 0) *gathers_us = gemm_gather_us(d, L);
    return 4e-6 + std::max(*gathers_us * 1e-6, t_waves) + (d.omega0 != 0.f ? 5e-6 + (double)d.n * L * 4.0 / 4e12 : 0.0);
}

// Estimated durations (seconds) of the gathers and of decode + dense; false where the dense route is not available.
bool densify_estimates(const DeviceView& d, uint32_t L, double* gathers_us, double* t_gather_out, double* t_dense_out) {
    if (L < 2 || d.m < 128 || d.n < 256) return false;
    const double mn = (double)d.m * (double)d.n;
    if ((double)d.nnz * 10.0 < mn) return false;  // the matrix cores spend ten times the multiply-adds: not worth estimating
    const bool pieces = mfma_applicable(d, L);
    if (mn * (pieces ? 2.0 * mfma_planes(d) : 4.0) > (double)(1ull << 30)) return false;
    const double flops = 2.0 * mn * L;
    const double t_gather = gather_estimate(d, L, gathers_us);
    if (t_gather < 9e-6) return false;  // decoder and product take longer: their shapes need not be looked at
    double t_dense;
    if (pieces) {
        // the decoder where it leaves pieces: 7 us (578 x 1013), 9 us (conv shape), 11 us (633 x 5106, three pieces, 2.3 M indices).  Where it
        // leaves ranks, or rows are long, it takes less (18 us for 1867 x 13028, 9.4 M), but the choice between all kernels is fitted with this:
        // of 600 products nine would change theirs, five by 0.59 to 0.87 times, four by 1.08 to 1.18
        t_dense = mfma_estimate_us(d, L) * 1e-6 + 6e-6 + mn * 2.0 * mfma_planes(d) / 4.4e12 + (double)d.nnz * 0.35e-12;
    } else {
        const double rate = flops < 1.5e10 ? 90e12 : (flops < 1e11 ? 105e12 : 120e12);
        const double t_write = 4.0 * mn / 4.5e12;  // the decoded matrix goes to memory once and is read back at least once
        const double t_decode = t_write + (double)d.nnz * 0.7e-12 + 3e-6;
        t_dense = (flops < 5e9 ? 20e-6 : 12e-6) + std::max(flops / rate, t_write) + t_decode;
    }
    *t_gather_out = t_gather;
    *t_dense_out = t_dense;
    return true;
}

hipError_t launch_densified(const DeviceView& d, const float* X, float* Y, uint32_t L, hipStream_t stream) {
    if (mfma_applicable(d, L)) return launch_mfma(d, X, Y, L, stream);
    float* W = nullptr;
    hipError_t e = (hipError_t)temp_alloc(reinterpret_cast<void**>(&W), (size_t)d.m * (size_t)d.n * sizeof(float), stream);
    if (e != hipSuccess) return e;
    if (decode_device(d, W, stream) != 0) e = hipErrorLaunchFailure;  // a CER_* code: only a failed launch is possible
    if (e == hipSuccess) e = (hipError_t)launch_dense(W, X, Y, d.m, d.n, (int64_t)L, stream);
    const hipError_t f = (hipError_t)temp_free(W, stream);
    return e == hipSuccess ? f : e;
}

// Decode + product in one launch is taken where its estimate is below this share of the other kernel's.  Over 438 random products
// 0.85 / 0.9 / 0.95 / 1 give 1.125 / 1.133 / 1.132 / 1.138 times the speed on average and make 4 / 5 / 9 / 11 of them slower.
constexpr double kFusedMargin = 0.9;

// Whether the LDS variant is expected to beat the kernel that gathers from L2.  Measured on MI355X: for wide
// batches it never does -- gathers of 16- or 32-byte pieces at random LDS addresses are bank-conflict bound at
// 32 - 43 B/clk per CU, while the L2 kernel's gathers of whole 128-byte rows sustain 27 - 48 B/clk per CU and
// amortise the group structure over 32 batch columns instead of 4 or 8 (AlexNet-fc6 shape, batch 32: 62 us against
// 35 us; 3x3 convolution shape, batch 3136: 536 us against 378 us).  For narrow batches it does: the L2 kernel
// still moves a whole 128-byte line per index, the LDS kernel 16 or 32 bytes (AlexNet-fc6 shape, batch 2 / 4 / 8: 27 / 28 / 30 us
// from L2, 15.6 / 12.5 / 22 us from LDS), provided the matrix is large enough for the gathers to dominate the launch (2048 x 2048
// cells with 0.2 - 2 million indices: 6 - 12 us either way, the L2 kernel ahead).  The stream kernel for several columns
// (cer_narrow.hip) is ahead of both there (7.7 / 8.6 / 12.5 us) and takes most of these products.
bool xtile_pays(const DeviceView& d, uint32_t L) { return L <= 8 && d.nnz >= 2500000; }

// Which kernel serves a batch of L > 1 columns (cer_matmul_path's numbering: 1, 2 or 3).  A preferred kernel is
// taken whenever it is applicable; otherwise the estimates decide.  no_temporaries: only kernels that need no
// temporary memory (the decode + dense route and batches of more than one LDS tile are left out).
int choose_batched_path(const DeviceView& d, uint32_t L, const MatmulOptions& o, bool no_temporaries, double* gathers_us, XtilePlan* plan_out,
                        const float* X = nullptr, const float* Y = nullptr) {
    const bool has_elements = d.m > 0 && d.n > 0;
    // strips of X in LDS: on request (and only when the strip-major index was prepared); the partial sums of the strips
    // need a temporary.  X == nullptr: the question is asked without buffers (cer_matmul_path_ex): aligned ones assumed.
    const bool strips_ok = !no_temporaries && strip_applicable(d, X, Y, L);
    if (o.path == kPathStrip && strips_ok) return kPathStrip;
    if (o.path == 3 && has_elements && !no_temporaries) return 3;
    // the strips' estimate against the gathers' (and, below, against decode + dense)
    bool strips_beat_gathers = false;
    double t_strip = 0;
    if (o.path < 0 && strips_ok && has_elements) {
        t_strip = plan_strip(d, L).est_us * 1e-6;
        const double t_gather_l2 = gather_estimate(d, L, gathers_us);
        strips_beat_gathers = t_strip < 0.95 * t_gather_l2;
    }
    // (from 8 columns on the strips are ahead of the LDS tile of all input rows: AlexNet-fc6 shape batch 8 15 against 22 us)
    if (o.path != 1 && o.path != 3 && !(strips_beat_gathers && L >= 8u)) {
        const XtilePlan plan = plan_xtile(d, L);
        if (plan.valid && (o.path == 2 || xtile_pays(d, L)) && (!no_temporaries || plan.ntiles == 1)) {
            if (plan_out) *plan_out = plan;
            return 2;
        }
    }
    // A handle whose strip-major index was prepared takes the strip kernel where its estimate is below 0.95 times that of the
    // gathers from L2 and below that of decode + product, if the latter pays: wide batches of large matrices.  Measured, gathers /
    // strips: AlexNet-fc6 shape, batch 8 / 16 / 32 / 64 / 100 / 128: 30 / 31 / 32 / 57 / 114 / 106 against 15 / 16 / 22 / 34 / 58 / 59
    // us; VGG-fc6 shape, batch 8 / 16 / 64 / 128: 27 / 28 / 53 / 99 against 17 / 18 / 39 / 76 us (batch 32: 30 against 25 us, but the
    // estimate keeps the gathers); 3x3 convolution shape, batch 3136: 191 us against 53 us decoded and multiplied.
    if (o.path < 0 && !no_temporaries && has_elements) {
        double t_gather = 0, t_dense = 0;
        const bool dense_ok = densify_estimates(d, L, gathers_us, &t_gather, &t_dense);
        const bool dense_pays = dense_ok && t_gather > 1.05 * t_dense;
        if (strips_beat_gathers && (!dense_pays || t_strip < t_dense)) return kPathStrip;
        if (dense_pays) return 3;
    }
    return 1;
}

// Estimated duration (microseconds) of the kernel that choose_batched_path has named.
double path_estimate_us(const DeviceView& d, uint32_t L, int path, double* gathers_us) {
    if (path == kPathStrip) return plan_strip(d, L).est_us;
    if (path == 2) return 4.0 + (double)d.nnz * 3.2e-6;  // AlexNet-fc6 shape batch 2 / 4 / 8: 23 / 13 / 28 us
    double t_gather = 0, t_dense = 0;
    if (path == 3 && densify_estimates(d, L, gathers_us, &t_gather, &t_dense)) return t_dense * 1e6;
    return gather_estimate(d, L, gathers_us) * 1e6;
}

// Estimated duration (microseconds) below which products from a prepared handle's tile index are taken, where `path` runs without it, or (one)
// decode + product in one launch or the stream kernel, which are expected to take `us`.  gathers: gemm_gather_us.
// 11000 random products of prepared handles (256 to 4096 rows of 512 to 25088 columns, 2 to 3136 batch columns, 0.5 to 75 % indexed, 2 to 64
// values), each with the tile index and without: a fifth takes it, at 1.28 times the speed in the geometric mean; one in ninety is slower by more than
// 2 %, one in 140 by more than 5 %, 1.25 times at most.  With 0.95 times the estimates that the other choices go by
// one in fourteen was slower, by up to 3.3 times (3135 x 1433, batch 101, 2 % indexed: 5.5 -> 12 us), because
//   * a wave of gather_estimate takes 4 us whatever its row holds; rows of some dozens of elements take less (38 % too much; typical deviation
//     of the terms below 15 %)
//   * plan_strip has 6 us for workgroups with next to nothing to stream, which small matrices do not take
//   * the product of the decoded matrix has become faster for uniform codebooks than densify_estimates has it (14 to 22 % too much from 100
//     columns on).
// (Those estimates are as the choice between the other kernels was fitted with them.)
double tile_limit_us(const DeviceView& d, uint32_t L, int path, bool one, double us, double gathers) {
    const double colsum = d.omega0 != 0.f ? 5.0 + (double)d.n * L * 4.0 / 4e6 : 0.0;
    if (one) return 0.95 * us;
    if (path == kPathStrip && L > 16) return 0.91 * (plan_strip(d, L).fitted_us + colsum);
    if (path == 3 && d.pieces > 1) return (d.grid.scale == 0.f ? 0.925 : (L < 100 ? 0.95 : 0.75)) * us;
    if (path != 1 || d.row_order) return 0.95 * us;
    const double waves = (double)d.m * std::ceil((double)L / 32.0) * std::min(4.0, 0.7 + 0.005 * (double)d.nnz / (double)d.m) / 4096.0;
    return 0.78 * (4.0 + std::max(gathers, waves) + 0.3 * std::min(gathers, waves) + colsum);
}

// What the library's own choice runs instead of `path` (a path, flags or a tile width of the caller's speak of the others):
// the stream kernel for several columns (narrow: its columns per pass), decode + product in one launch (fused: its rows per
// workgroup), or products from the handle's tile index (tile).  temporaries: the last two may have partial sums -- only where the kernel
// they take the place of has a temporary as well.
struct Instead {
    int narrow = 0, fused = 0;
    bool temporaries = false;
    TilePlan tile;  // variant -1: not taken
};
Instead choose_instead(const DeviceView& d, uint32_t L, const MatmulOptions& o, int path, double* gathers_us) {
    Instead r;
    if (L < 2 || o.path >= 0 || o.flags != 0 || o.tile_cols != 0) return r;
    double us = path_estimate_us(d, L, path, gathers_us);
    if (L <= 16) {
        const NarrowEstimate narrow = narrow_estimate(d, L);
        if (narrow.us < us) {
            us = narrow.us;
            r.narrow = narrow.columns;
        }
    }
    r.temporaries = r.narrow == 0 && (path == 3 || path == kPathStrip || d.omega0 != 0.f || d.n_split_parts > 0);
    r.fused = fused_rows(d, L, r.temporaries, kFusedMargin * us, &us);
    if (r.fused > 0) r.narrow = 0;
    if (d.tile_index) {
        r.tile = plan_tile(d, L, r.temporaries, tile_limit_us(d, L, path, r.fused > 0 || r.narrow > 0, us, *gathers_us));
        if (r.tile.variant >= 0) r.narrow = r.fused = 0;
    }
    return r;
}

// What the library runs by its own choice for a batch of L > 1 columns.
Instead choose_all(const DeviceView& d, uint32_t L) {
    const MatmulOptions o;
    double gathers_us = -1;
    const int path = choose_batched_path(d, L, o, false, &gathers_us, nullptr);
    return choose_instead(d, L, o, path, &gathers_us);
}

// Column sums of X for a non-zero most frequent value: shape of the two-stage sum and the floats it needs
// ([T: L rounded to 64][partials: nslabs x L]).
struct ColsumPlan {
    uint32_t CB = 1, nslabs = 1, slab = 1;
    size_t t_floats = 0, floats = 0;
};

// Slabs of 32 rows or more, up to 4096 workgroups: a pass over a large X is bound by how many loads are in flight (3x3
// convolution shape, batch 3136, 58 MB of X: 48 us with slabs of 256 rows).  Where that many partial sums would not fit
// the fixed workspace of the entry point that allocates nothing, slabs of 256 rows and up to 1024 workgroups: both
// entry points sum in the same order.
ColsumPlan plan_colsum(uint32_t n, uint32_t L) {
    ColsumPlan p;
    p.CB = std::min<uint32_t>(256u, pow2_ceil(L));
    const uint32_t coltiles = (L + p.CB - 1) / p.CB;
    p.t_floats = ((size_t)L + 63) & ~(size_t)63;
    for (int wide = 1; wide >= 0; --wide) {
        const uint32_t rows = wide ? 32u : 256u, blocks = wide ? 4096u : 1024u;
        p.nslabs = std::max<uint32_t>(1u, std::min<uint32_t>((n + rows - 1u) / rows, blocks / std::max(coltiles, 1u)));
        p.slab = std::max<uint32_t>((n + p.nslabs - 1) / p.nslabs, 1u);
        p.floats = p.t_floats + (size_t)p.nslabs * L;
        if (p.floats <= kStaticWorkspaceFloats) break;
    }
    return p;
}

}  // namespace

int matmul_path(const DeviceView& d, int64_t L, const MatmulOptions& o) {
    if (L <= 1) return gemv_path(d, o);
    if (L > 0x7FFFFFFFll) return 1;
    double gathers_us = -1;
    return choose_batched_path(d, (uint32_t)L, o, false, &gathers_us, nullptr);
}

int matmul_narrow_columns(const DeviceView& d, int64_t L) {
    return L < 2 || L > 16 ? 0 : choose_all(d, (uint32_t)L).narrow;
}

int matmul_fused_rows(const DeviceView& d, int64_t L) {
    return L < 2 || L > 0x7FFFFFFFll ? 0 : choose_all(d, (uint32_t)L).fused;
}

int matmul_tile_columns(const DeviceView& d, int64_t L) {
    if (L < 2 || L > 0x7FFFFFFFll) return 0;
    return tile_columns(choose_all(d, (uint32_t)L).tile);
}

// Batches that are looked at: every one of up to 128 columns, then multiples of 16, where a workgroup's columns are all used, and one column less,
// which other kernels read in smaller pieces; from 1024 on a 32nd apart.  A query takes 1 to 2 us on the host, the index 4 bytes per element on the
// device.
bool tile_index_pays(const DeviceView& v) {
    if (tile_index_bytes(v) == 0) return false;
    DeviceView d = v;
    d.tile_index = &d;  // (the estimates do not read it)
    auto taken = [&](uint32_t L) { return choose_all(d, L).tile.variant >= 0; };
    for (uint32_t L = 2; L < 128u; ++L)
        if (taken(L)) return true;
    for (uint32_t L = 128; L <= (1u << 20); L += L < 1024u ? 16u : (L / 32u) & ~15u)
        if (taken(L) || taken(L - 1u)) return true;
    return false;
}

int matmul_planes(const DeviceView& d) { return mfma_applicable(d, 2) ? mfma_planes(d) : 0; }

size_t matmul_workspace_floats(const DeviceView& d, int64_t L, const MatmulOptions& o) {
    if (d.m == 0 || L < 1 || L > 0x7FFFFFFFll || d.omega0 == 0.f) return 0;
    if (L == 1 && gemv_sums_x(d, o)) return 0;
    return plan_colsum((uint32_t)d.n, (uint32_t)L).floats;
}

int static_workspace(float** ptr, size_t* floats) {
    static std::mutex mu;
    static float* addr[16] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= 16) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        if (!p) return (int)hipErrorInvalidSymbol;
        addr[dev] = static_cast<float*>(p);
    }
    *ptr = addr[dev];
    *floats = kStaticWorkspaceFloats;
    return (int)hipSuccess;
}

int launch_matmul(const DeviceView& d, const float* X, float* Y, int64_t L64, void* stream_v, const MatmulOptions& o_in,
                  float* workspace, size_t workspace_floats) {
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    if (d.m == 0) return (int)hipSuccess;
    if (L64 > 0x7FFFFFFFll || d.m > 0x7FFFFFFFll) return (int)hipErrorInvalidValue;
    const uint32_t L = (uint32_t)L64;
    const bool no_temporaries = workspace != nullptr;
    MatmulOptions o = o_in;
    if (no_temporaries) o.flags |= kOptRowsWhole;  // the parts of split rows meet in a temporary
    XtilePlan plan;
    double gathers_us = -1;
    const int batched_path = L > 1 ? choose_batched_path(d, L, o, no_temporaries, &gathers_us, &plan, X, Y) : 0;
    if (!no_temporaries && L > 1) {
        const Instead instead = choose_instead(d, L, o, batched_path, &gathers_us);
        if (instead.tile.variant >= 0) return (int)launch_tile(d, instead.tile, X, Y, L, batched_path == 3, stream);
        if (instead.narrow > 0) return (int)launch_narrow(d, X, Y, L, stream);
        if (instead.fused > 0) return (int)launch_fused(d, X, Y, L, instead.temporaries, batched_path == 3, stream);
    }
    if (batched_path == 3) return (int)launch_densified(d, X, Y, L, stream);

    float* T = nullptr;
    float* scratch = nullptr;
    hipError_t e = hipSuccess;
    if (d.omega0 != 0.f && !(L == 1 && gemv_sums_x(d, o))) {
        // T[l] = sum_i X[i,l], in the caller's workspace or in a stream-ordered temporary
        const ColsumPlan cp = plan_colsum((uint32_t)d.n, L);
        float* base = workspace;
        if (no_temporaries) {
            if (cp.floats > workspace_floats) return (int)hipErrorInvalidValue;  // the caller has checked the size
        } else {
            e = (hipError_t)temp_alloc(reinterpret_cast<void**>(&scratch), cp.floats * sizeof(float), stream);
            if (e != hipSuccess) return (int)e;
            base = scratch;
        }
        T = base;
        e = launch_colsum(X, (uint32_t)d.n, L, base + cp.t_floats, cp.nslabs, cp.slab, cp.CB, T, stream);
        if (e != hipSuccess) {
            if (scratch) (void)temp_free(scratch, stream);
            return (int)e;
        }
    }
    if (L == 1)
        e = launch_gemv_any(d, X, Y, T, stream, o);
    else if (batched_path == 2)
        e = launch_xtile_any(d, plan, X, Y, T, L, stream);
    else if (batched_path == kPathStrip)
        e = launch_strip(d, X, Y, T, L, stream);
    else
        e = launch_gemm_any(d, X, Y, T, L, stream, o);
    if (scratch) {
        hipError_t f = (hipError_t)temp_free(scratch, stream);
        if (e == hipSuccess) e = f;
    }
    return (int)e;
}

}  // namespace cer
