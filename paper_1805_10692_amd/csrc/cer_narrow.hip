// Batches of 2 to 8 columns: the stream kernel of batch 1 (cer_gemv.hip) for V columns at once.
//
// V columns of X are staged into LDS as [row][V] and gathered from there, 4 V bytes per indexed element; everything else -- one
// wave per row (or several: matrices of few rows), 16-byte loads of the indices, boundary bitmap, one weight per position -- costs
// the same as for one column and is shared by the V of them.  A launch covers all columns: the workgroups of the second,
// third ... group of V columns follow those of the first.
// Bound by the LDS: a 16-byte gather at 64 random rows takes about 12 clocks of it (four passes of 16 lanes, the busiest of the
// 16 bank groups hit three times), the weight four.  AlexNet-fc6 shape, batch 4: 7.6 us; 12.8 with the tile kernel
// (cer_xtile.hip), 20 gathering from L2.
#include "cer_stream.hpp"

namespace cer {
namespace {

template <int V>
struct alignas(4 * V) Cols {
    float v[V];
};

enum : int32_t { kRowVectors, kInOrder, kScalar };

struct NarrowArgs {
    const uint32_t* tab;
    const float* X;
    const float* omega;
    const void* colI;
    float* Y;
    uint32_t n, m, L, K;
    uint32_t tab_shift, part_shift, row_blocks, rows_per_block;
    uint32_t magic;  // ceil(2^32 / L)
    int32_t how;     // kRowVectors, kInOrder: X is aligned; kScalar: it is not
};

template <typename IdxT, int V>
__global__ __launch_bounds__(1024) void cer_narrow_kernel(NarrowArgs a) {
    using S = GemvShape<IdxT, sizeof(IdxT) == 2 ? 2 : 1>;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t nthreads = blockDim.x, nwaves = nthreads >> 6;
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = uniform(threadIdx.x >> 6);
    const uint32_t last_word = (1u << a.tab_shift) - 1u, ntiles = (last_word >> 6) + 1u;  // 64 ranks per tile
    const uint32_t lcap = max(last_word, 63u) + 5u;  // the pseudo group in front of the row, the groups, two sentinels
    // LDS: [X: n x V][ends | wts: nwaves x lcap][bitmap | word prefix: nwaves x NWORDS][sums: nwaves x V]
    Cols<V>* xs = reinterpret_cast<Cols<V>*>(smem);
    uint32_t* list0 = reinterpret_cast<uint32_t*>(xs + ((a.n + 3u) & ~3u));
    uint32_t* ends = list0 + wave * lcap;
    float* wts = reinterpret_cast<float*>(list0 + nwaves * lcap) + wave * lcap;
    uint32_t* bmp = list0 + 2u * nwaves * lcap + wave * (uint32_t)S::NWORDS;
    uint32_t* wpre = list0 + 2u * nwaves * lcap + (nwaves + wave) * (uint32_t)S::NWORDS;
    float* s_sum = reinterpret_cast<float*>(list0 + 2u * nwaves * lcap + 2u * nwaves * (uint32_t)S::NWORDS);

    const uint32_t parts = 1u << a.part_shift, part = wave & (parts - 1u), rows_at_once = nwaves >> a.part_shift;
    const uint32_t pass = blockIdx.x / a.row_blocks, rb = blockIdx.x % a.row_blocks;
    const uint32_t col0 = pass * V, cols = min((uint32_t)V, a.L - col0);
    const uint32_t row_begin = rb * a.rows_per_block, row_end = min(a.m, row_begin + a.rows_per_block);
    const IdxT* colI = static_cast<const IdxT*>(a.colI);
    uint32_t r = row_begin + (wave >> a.part_shift);  // wave-uniform

    // the row's record (one word per lane and tile) and Omega: lane l of tile t holds the group of rank 64 t + l + 1
    uint32_t rec[4];
    float wq[4];
    auto load_record = [&](uint32_t row) {
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t)
            if (t < ntiles) rec[t] = a.tab[((size_t)row << a.tab_shift) + min(t * kWave + lane, last_word)];
    };
    load_record(min(r, a.m - 1u));
    const float omega0 = a.omega[0];
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t)
        if (t < ntiles) wq[t] = a.omega[min(t * kWave + lane + 1u, a.K - 1u)];

    // X to LDS.  A compute unit's memory pipeline accepts a load about every 26 clocks whatever its width, so 16 bytes at a
    // time: a copy (L == V), one vector per row (L a multiple of V), or all of X in order, each number to its place or nowhere.
    typedef float Vec __attribute__((ext_vector_type(V)));
    if (a.how == kRowVectors) {
        const Vec* src = reinterpret_cast<const Vec*>(a.X + col0);
        Vec* dst = reinterpret_cast<Vec*>(xs);
        const uint32_t step = a.L / V;
        uint32_t i = threadIdx.x;
        for (; i + 3u * nthreads < a.n; i += 4u * nthreads) {
            Vec q[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) q[k] = src[(size_t)(i + k * nthreads) * step];
#pragma unroll
            for (int k = 0; k < 4; ++k) dst[i + k * nthreads] = q[k];
        }
        for (; i < a.n; i += nthreads) dst[i] = src[(size_t)i * step];
    } else {
        const uint32_t total = a.n * a.L, n4 = a.how == kInOrder ? total >> 2 : 0u;  // at most 36000 x 8 numbers
        float* dst = reinterpret_cast<float*>(xs);
        auto place = [&](uint32_t e, float x) {
            const uint32_t row = __umulhi(e, a.magic), c = e - row * a.L - col0;
            if (c < (uint32_t)V) dst[row * V + c] = x;
        };
        auto place4 = [&](uint32_t i, const float4& q) {
            place(4u * i, q.x);
            place(4u * i + 1u, q.y);
            place(4u * i + 2u, q.z);
            place(4u * i + 3u, q.w);
        };
        const float4* src = reinterpret_cast<const float4*>(a.X);
        uint32_t i = threadIdx.x;
        for (; i + 3u * nthreads < n4; i += 4u * nthreads) {
            float4 q[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) q[k] = src[i + k * nthreads];
#pragma unroll
            for (int k = 0; k < 4; ++k) place4(i + k * nthreads, q[k]);
        }
        for (; i < n4; i += nthreads) place4(i, src[i]);
        for (i = (n4 << 2) + threadIdx.x; i < total; i += nthreads) place(i, a.X[i]);
    }
    __syncthreads();
    // Appendix A-A1: the constant term of a non-zero most frequent value
    float t_off[V] = {};
    if (omega0 != 0.f) {  // uniform over the grid
        float part_sum[V] = {};
        for (uint32_t i = threadIdx.x; i < a.n; i += nthreads)
#pragma unroll
            for (int v = 0; v < V; ++v) part_sum[v] += xs[i].v[v];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const float y = wave_sum(part_sum[v]);
            if (lane == 0) s_sum[wave * V + v] = y;
        }
        __syncthreads();
        for (uint32_t w = 0; w < nwaves; ++w)
#pragma unroll
            for (int v = 0; v < V; ++v) t_off[v] += s_sum[w * V + v];
#pragma unroll
        for (int v = 0; v < V; ++v) t_off[v] *= omega0;
        __syncthreads();  // s_sum serves again
    }

    const uint32_t xbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)smem;
    uint32_t shift = V == 1 ? 2u : (V == 2 ? 3u : (V == 4 ? 4u : 5u));
    asm("" : "+v"(shift));  // in a vector register (sub-dword forms take no constants)
    for (; r < row_end; r += rows_at_once) {
        // list of the non-empty groups: the pseudo group in front of the row, then the record's
        const uint32_t rs = (uint32_t)__builtin_amdgcn_readlane((int)rec[0], 0);
        uint32_t re = (uint32_t)__builtin_amdgcn_readlane((int)rec[0], (int)(last_word & 63u));
        if (lane == 0) { ends[0] = rs; wts[0] = 0.f; }
        int count = 1;
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
            if (t >= ntiles) break;
            PtrTile p;
            p.s = rec[t];
            p.e = (uint32_t)__builtin_amdgcn_update_dpp((int)rec[t], (int)rec[t], 0x130 /* wave_shl:1 */, 0xF, 0xF, false);
            if (t + 1 < ntiles && lane == kWave - 1u) p.e = (uint32_t)__builtin_amdgcn_readlane((int)rec[t < 3 ? t + 1 : 3], 0);
            if (t * kWave + lane >= last_word) p.e = p.s;
            if (t > 0) re = (uint32_t)__builtin_amdgcn_readlane((int)rec[t], 63);
            count = list_append(p, wq[t] - omega0, ends, wts, count);
        }
        list_close(ends, wts, count, lane);
        // this wave's share of the row's windows
        uint32_t b0 = rs & ~((uint32_t)S::PPL - 1u), te = re;
        if (parts > 1u) {
            const uint32_t nwin = (re - b0 + (uint32_t)S::WIN - 1u) / (uint32_t)S::WIN;
            const uint32_t share = ((nwin + parts - 1u) >> a.part_shift) * (uint32_t)S::WIN;
            const uint32_t mine = b0 + part * share;
            if (mine < re) { b0 = mine; te = min(re, mine + share); } else { te = b0; }
        }
        float acc[V] = {};
        if (count > 1 && b0 < te) {  // wave-uniform
            // two sets of index registers: the next batch is requested before the current one is summed; a window behind the
            // end asks for the first one again
            uint4 ix[2][S::NW];
            auto request = [&](uint4 (&q)[S::NW], uint32_t b) {
                const uint4* p = reinterpret_cast<const uint4*>(colI + b) + lane;
#pragma unroll
                for (int W = 0; W < S::NW; ++W) q[W] = p[(b + (uint32_t)W * S::WIN < te ? W : 0) * kWave];
            };
            auto batch = [&](const uint4 (&q)[S::NW], uint32_t b, uint32_t& first) {
                bitmap_build<S>(ends, (uint32_t)count + 1u, first, b, bmp, wpre, lane);
#pragma unroll
                for (int W = 0; W < S::NW; ++W) {
                    if (W > 0 && b + (uint32_t)W * S::WIN >= te) break;  // wave-uniform
                    float wl[S::PPL];
                    window_weights<S>(W, bmp, wpre, wts, lane, wl);
#pragma unroll
                    for (int k = 0; k < S::PPL; ++k) {
                        typedef const Vec __attribute__((address_space(3))) * LdsVec;
                        const Cols<V> x = __builtin_bit_cast(Cols<V>, *reinterpret_cast<LdsVec>((uintptr_t)(xbase + packed_offset<IdxT>(q[W], k, shift))));
#pragma unroll
                        for (int v = 0; v < V; ++v) acc[v] = fmaf(x.v[v], wl[k], acc[v]);
                    }
                }
            };
            request(ix[0], b0);
            wave_lds_sync();
            uint32_t first = part > 0u ? list_rank_of(ends, count, b0, lane) : (rs > b0 ? 0u : 1u);
            for (;;) {
                const uint32_t b1 = b0 + S::BATCH, b2 = b1 + S::BATCH;
                request(ix[1], b1 < te ? b1 : b0);
                batch(ix[0], b0, first);
                if (b1 >= te) break;
                request(ix[0], b2 < te ? b2 : b1);
                batch(ix[1], b1, first);
                if (b2 >= te) break;
                b0 = b2;
            }
        }
        const uint32_t next = r + rows_at_once;
        if (next < row_end) load_record(next);
        wave_lds_sync();  // the list is rebuilt by the next row
        float y[V];
#pragma unroll
        for (int v = 0; v < V; ++v) y[v] = wave_sum(acc[v]);
        if (parts == 1u) {
            float mine = 0.f;
#pragma unroll
            for (int v = 0; v < V; ++v) mine = lane == (uint32_t)v ? y[v] + t_off[v] : mine;
            if (lane < cols) a.Y[(size_t)r * a.L + col0 + lane] = mine;
        } else if (lane == 0) {
#pragma unroll
            for (int v = 0; v < V; ++v) s_sum[wave * V + v] = y[v];
        }
    }
    if (parts > 1u) {  // uniform over the grid: every wave had at most one row
        __syncthreads();
        r = row_begin + (wave >> a.part_shift);
        if (part == 0u && r < row_end && lane < cols) {
            float y = 0.f;
            for (uint32_t q = 0; q < parts; ++q) y += s_sum[(wave + q) * V + lane];
            float off = 0.f;
#pragma unroll
            for (int v = 0; v < V; ++v) off = lane == (uint32_t)v ? t_off[v] : off;
            a.Y[(size_t)r * a.L + col0 + lane] = y + off;
        }
    }
}

struct NarrowPlan {
    int V = 0;  // 0: not applicable
    uint32_t waves = 0, part_shift = 0, rows_per_block = 0, row_blocks = 0, passes = 0;
    size_t lds = 0;
    double us = 0;  // estimate
};

template <typename IdxT>
NarrowPlan plan_narrow_t(const DeviceView& d, uint32_t L) {
    using S = GemvShape<IdxT, sizeof(IdxT) == 2 ? 2 : 1>;
    NarrowPlan best;
    const size_t budget = d.lds_per_block - 256, rows4 = ((size_t)d.n + 3) & ~(size_t)3;
    const size_t lcap = std::max<size_t>(63, ((size_t)1 << d.rank_tab_shift) - 1) + 5;
    double best_cost = 1e300;
    for (int V : {8, 4, 2, 1}) {
        if (V > 1 && (uint32_t)V / 2 >= L) continue;  // half of the columns would be repetitions
        NarrowPlan p;
        p.V = V;
        p.passes = (L + V - 1) / V;
        // one workgroup per compute unit stages X once; 16 waves, fewer where their lists leave no room for X
        p.waves = 16;
        auto lds = [&](uint32_t w) { return rows4 * V * 4 + w * (lcap * 8 + S::NWORDS * 8 + V * 4); };
        while (p.waves > 4 && lds(p.waves) > budget) p.waves >>= 1;
        p.lds = lds(p.waves);
        if (p.lds > budget) continue;
        const uint64_t units = std::max<uint64_t>(1, (uint64_t)d.cus / p.passes);
        p.rows_per_block = (uint32_t)std::max<uint64_t>(1, ((uint64_t)d.m + units - 1) / units);
        const uint64_t windows = ((uint64_t)d.nnz / (uint64_t)d.m + S::WIN - 1) / S::WIN;  // average row
        while ((2u << p.part_shift) * p.rows_per_block <= p.waves && (1u << p.part_shift) < 8u && (1u << p.part_shift) < windows) ++p.part_shift;
        p.row_blocks = (uint32_t)(((uint64_t)d.m + p.rows_per_block - 1) / p.rows_per_block);
        // clocks of a compute unit: per 64 indexed elements (18, 19, 20, 52 for 1, 2, 4, 8 columns: the weights and their
        // bookkeeping, and beyond 4 columns the LDS), per row its list, the staging, and what any launch takes.  Measured
        // with the fit: AlexNet-fc6 shape batch 2 / 4 / 5 / 8: 6.6 / 7.6 / 14.2 / 11.6 us; VGG-fc6 shape batch 2 / 4: 10.4 / 17.7 us.
        const double gather = V == 8 ? 52.0 : (V == 4 ? 20.0 : (V == 2 ? 19.0 : 18.0));
        const double row = 150.0 * ((((1u << d.rank_tab_shift) - 1u) >> 6) + 1u);
        const double clk = p.passes * ((double)d.nnz / 64.0 * gather * (p.waves < 16 ? 1.5 : 1.0) + (double)d.m * row) / d.cus +
                           rows4 * V * 4 / 1024.0 * 26.0 + 6000.0;
        p.us = clk / 2400.0;
        const double cost = p.us;
        if (cost < best_cost) {
            best_cost = cost;
            best = p;
        }
    }
    return best;
}

NarrowPlan plan_narrow(const DeviceView& d, uint32_t L) {
    if (!d.rank_tab || L < 2 || L > 8 || d.m < 1 || d.n < 1 || d.nnz < 1) return NarrowPlan{};
    switch (d.colI_bits) {
        case 8: return plan_narrow_t<uint8_t>(d, L);
        case 16: return plan_narrow_t<uint16_t>(d, L);
        default: return NarrowPlan{};  // more than 65536 rows of X do not fit
    }
}

template <typename IdxT>
hipError_t launch_narrow_t(const NarrowPlan& p, const NarrowArgs& a, size_t budget, hipStream_t stream) {
    void (*kern)(NarrowArgs);
    int slot;
    switch (p.V) {
        case 8: kern = cer_narrow_kernel<IdxT, 8>; slot = 3; break;
        case 4: kern = cer_narrow_kernel<IdxT, 4>; slot = 2; break;
        case 2: kern = cer_narrow_kernel<IdxT, 2>; slot = 1; break;
        default: kern = cer_narrow_kernel<IdxT, 1>; slot = 0;
    }
    if (p.lds > 48 * 1024) {
        static LdsGrant<4> grant;
        const hipError_t e = grant.ensure(slot, reinterpret_cast<const void*>(kern), budget);
        if (e != hipSuccess) return e;
    }
    return launch_kernel(kern, dim3(p.row_blocks * p.passes), dim3(p.waves * kWave), p.lds, stream, a);
}

}  // namespace

double narrow_estimate_us(const DeviceView& d, uint32_t L) {
    const NarrowPlan p = plan_narrow(d, L);
    return p.V > 0 ? p.us : 1e30;
}

hipError_t launch_narrow(const DeviceView& d, const float* X, float* Y, uint32_t L, hipStream_t stream) {
    const NarrowPlan p = plan_narrow(d, L);
    NarrowArgs a;
    a.tab = d.rank_tab;
    a.X = X;
    a.omega = d.omega;
    a.colI = d.colI;
    a.Y = Y;
    a.n = (uint32_t)d.n;
    a.m = (uint32_t)d.m;
    a.L = L;
    a.K = (uint32_t)d.K;
    a.tab_shift = (uint32_t)d.rank_tab_shift;
    a.part_shift = p.part_shift;
    a.row_blocks = p.row_blocks;
    a.rows_per_block = p.rows_per_block;
    a.magic = (uint32_t)(((1ull << 32) + L - 1) / L);
    a.how = (reinterpret_cast<uintptr_t>(X) & 15u) != 0 ? kScalar : (L % (uint32_t)p.V == 0 ? kRowVectors : kInOrder);
    const size_t budget = d.lds_per_block - 256;
    return d.colI_bits == 8 ? launch_narrow_t<uint8_t>(p, a, budget, stream) : launch_narrow_t<uint16_t>(p, a, budget, stream);
}

}  // namespace cer
