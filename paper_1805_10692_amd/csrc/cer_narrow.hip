// Batches of 2 to 16 columns: the stream kernel of batch 1 (cer_gemv.hip) for V columns at once.
//
// V columns of X are staged into LDS as [row][V] and gathered from there, 4 V bytes per indexed element; everything else -- one
// wave per row (or several: matrices of few rows), 16-byte loads of the indices, boundary bitmap, one weight per position -- costs
// the same as for one column and is shared by the V of them.  A launch covers all columns: the workgroups of the second,
// third ... group of V columns follow those of the first.
// While it streams it is bound by the LDS and the vector ALU about equally: a 16-byte gather at 64 random rows takes about 12
// clocks of LDS (four passes of 16 lanes, the busiest of the 16 bank groups hit three times), the weight four.  AlexNet-fc6 shape,
// batch 4: 7.8 us (12.6 with the tile kernel, cer_xtile.hip, 29 gathering from L2); over the launch the LDS pipe is busy 42 %
// of the time (its conflicts 19 %), the vector ALU 41 %, and a wave waits for data 62 % of its own: the staging of 147 KB of X per
// compute unit comes before the first gather.  2048 x 2048, 256 values, batch 16 (four passes, 255 groups per row): 12 us, LDS
// 51 %, vector ALU 46 %, a wave's waits 59 %.
#include "cer_stream.hpp"

namespace cer {
namespace {

template <int V>
struct alignas(4 * V) Cols {
    float v[V];
};

struct NarrowArgs {
    const uint32_t* tab;
    const float* X;
    const float* omega;
    const void* colI;
    float* Y;
    uint32_t n, m, L, K;
    uint32_t tab_shift, part_shift, row_blocks, rows_per_block;
};

// kFew: fewer than 16 waves (X and that many lists do not fit LDS) do not cover the latency of LDS and of the loads of X one for another, so
// a wave has more of them on their way: all of a window's reads, eight loads.  us per call before and after: one column, four waves 822 x 38457, 3
// values, batch 3 23.9 -> 18.8, eight 300 x 33000, 130 values, 2 8.8 -> 8.7; two columns, four 1900 x 19872, 3 values, 9 73 -> 55, eight 2303 x
// 19624, 3 values, 4 12.2 -> 10.8; four columns, four 2286 x 9957, 33 values, 8 17.4 -> 16.3, eight 1065 x 9467, 33 values, 8 14.7 -> 13.5.
// Four columns and eight waves gain where a wave has several rows that are long or have short lists, and lose else (plan_narrow_t).
template <typename IdxT, int V, bool kFew>
__global__ __launch_bounds__(kFew ? 512 : 1024) void cer_narrow_kernel(NarrowArgs a) {
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
    // a last group that is not full moves back: its first columns are computed twice, to the same numbers
    const uint32_t col0 = a.L > (uint32_t)V ? min(pass * V, a.L - (uint32_t)V) : 0u, cols = min((uint32_t)V, a.L);
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

    // X to LDS: one vector load per row, at whatever 4-byte address the row has there.  Fewer columns than V: a vector runs
    // into the next row (those sums are not stored), and the last rows are read number by number.
    typedef float Vec __attribute__((ext_vector_type(V)));
    struct __attribute__((packed, aligned(4))) Row {
        Vec v;
    };
    {
        const float* src = a.X + col0;
        Vec* dst = reinterpret_cast<Vec*>(xs);
        const uint32_t behind = (uint32_t)V > a.L ? ((uint32_t)V - 1u) / a.L : 0u, nvec = a.n > behind ? a.n - behind : 0u;
        uint32_t i = threadIdx.x;
        if constexpr (kFew) {  // (what is left four at a time: 192 x 18844, batch 2 5.99 -> 5.80 us)
            for (; i + 7u * nthreads < nvec; i += 8u * nthreads) {
                Vec q[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) q[k] = reinterpret_cast<const Row*>(src + (size_t)(i + k * nthreads) * a.L)->v;
#pragma unroll
                for (int k = 0; k < 8; ++k) dst[i + k * nthreads] = q[k];
            }
        }
        for (; i + 3u * nthreads < nvec; i += 4u * nthreads) {
            Vec q[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) q[k] = reinterpret_cast<const Row*>(src + (size_t)(i + k * nthreads) * a.L)->v;
#pragma unroll
            for (int k = 0; k < 4; ++k) dst[i + k * nthreads] = q[k];
        }
        for (; i < nvec; i += nthreads) dst[i] = reinterpret_cast<const Row*>(src + (size_t)i * a.L)->v;
        for (i = nvec + threadIdx.x; i < a.n; i += nthreads)
#pragma unroll
            for (int v = 0; v < V; ++v) xs[i].v[v] = (uint32_t)v < a.L ? src[(size_t)i * a.L + v] : 0.f;
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
                    // The reads of X in front of their products where that is faster: with both in one loop the compiler waits for every second
                    // read right behind its request.  One or two columns, 16 waves: 1412 x 13527, 10 values, batch 5 11.4 -> 9.8 us, 914 x 11814, 33
                    // values, 12 16.2 -> 14.5, 100 products 0.93 times the time; four or eight columns 0.93 to 1.07, and so they stay in one.
                    constexpr int kTogether = kFew || V <= 2 ? std::min<int>(S::PPL, 64 / V) : 1;
#pragma unroll
                    for (int k0 = 0; k0 < S::PPL; k0 += kTogether) {
                        Vec x[kTogether];
#pragma unroll
                        for (int k = 0; k < kTogether; ++k) {
                            typedef const Vec __attribute__((address_space(3))) * LdsVec;
                            x[k] = *reinterpret_cast<LdsVec>((uintptr_t)(xbase + packed_offset<IdxT>(q[W], k0 + k, shift)));
                        }
                        if constexpr (kFew) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int k = 0; k < kTogether; ++k) {
                            const Cols<V> c = __builtin_bit_cast(Cols<V>, x[k]);
#pragma unroll
                            for (int v = 0; v < V; ++v) acc[v] = fmaf(c.v[v], wl[k0 + k], acc[v]);
                        }
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
    bool few = false;  // cer_narrow_kernel's kFew
    size_t lds = 0;
    double us = 0;  // estimate
};

template <typename IdxT>
NarrowPlan plan_narrow_t(const DeviceView& d, uint32_t L) {
    using S = GemvShape<IdxT, sizeof(IdxT) == 2 ? 2 : 1>;
    NarrowPlan best;
    const size_t budget = d.lds_per_block - 256, rows4 = ((size_t)d.n + 3) & ~(size_t)3;
    const size_t lcap = std::max<size_t>(63, ((size_t)1 << d.rank_tab_shift) - 1) + 5;
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
        if (V == 8 && p.waves < 16) continue;  // by the estimate below four columns and twice the waves are always ahead
        const uint64_t units = std::max<uint64_t>(1, (uint64_t)d.cus / p.passes);
        p.rows_per_block = (uint32_t)std::max<uint64_t>(1, ((uint64_t)d.m + units - 1) / units);
        const uint64_t windows = ((uint64_t)d.nnz / (uint64_t)d.m + S::WIN - 1) / S::WIN;  // average row
        while ((2u << p.part_shift) * p.rows_per_block <= p.waves && (1u << p.part_shift) < 8u && (1u << p.part_shift) < windows) ++p.part_shift;
        p.row_blocks = (uint32_t)(((uint64_t)d.m + p.rows_per_block - 1) / p.rows_per_block);
        // (8-bit indices: an X of 256 rows leaves room for 16 waves.)  Four columns, eight waves, kFew against the other way, 48 products: more than
        // eight rows per workgroup and lists of up to 64 values 0.91 to 0.99, longer lists 0.93 to 0.95 from five windows per row on and 1.00
        // to 1.02 at fewer than four; up to eight rows 0.98 to 1.03
        p.few = sizeof(IdxT) > 1 && p.waves < 16 && (V < 4 || p.waves < 8 || (p.rows_per_block > 8 && (d.rank_tab_shift <= 6 || windows > 4)));
        // Clocks, fitted to 220 random shapes of 2 to 16 columns (the typical deviation is 12 %).  A compute unit: per 64 indexed
        // elements, 13, 15, 23, 58 for 1, 2, 4, 8 columns -- the weights and their bookkeeping, and from 4 columns on the
        // LDS -- and per row its list.  Against that the longest row, walked by its waves alone.  Before either, the staging: 21
        // per load of 64 rows and two per line of X.  AlexNet-fc6 shape batch 2 / 4 / 5 / 8: 6.6 / 7.6 / 14.2 / 11.6 us.
        const double gather = V == 8 ? 58.0 : (V == 4 ? 22.6 : (V == 2 ? 15.2 : 12.7));
        const double lists = ((((1u << d.rank_tab_shift) - 1u) >> 6) + 1u);
        const double work = p.passes * ((double)d.nnz / 64.0 * gather + (double)d.m * lists * 72.0) / d.cus * (p.waves < 16 ? 1.36 : 1.0);
        const double rows_per_wave = (double)((p.rows_per_block << p.part_shift) + p.waves - 1) / p.waves;
        const double walk = 2.06 * d.longest_row / (1u << p.part_shift) + rows_per_wave * lists * 535.0;
        const double loads = (double)d.n * (V == 8 ? 2.0 : 1.0) / 64.0, lines = (double)d.n * std::min(L * 4.0, 128.0) / 128.0;
        double clk = 8300.0 + std::max(work, walk) + loads * 21.0 + lines * 2.0 + (V == 8 ? 1700.0 : 0.0);
        if (d.omega0 != 0.f) clk += 3200.0 + 3.3 * d.n * V / 64.0;
        p.us = clk / 2400.0;
        if (best.V == 0 || p.us < best.us) best = p;
    }
    return best;
}

NarrowPlan plan_narrow(const DeviceView& d, uint32_t L) {
    if (!d.rank_tab || L < 2 || L > 16 || d.m < 1 || d.n < 1 || d.nnz < 1) return NarrowPlan{};
    switch (d.colI_bits) {
        case 8: return plan_narrow_t<uint8_t>(d, L);
        case 16: return plan_narrow_t<uint16_t>(d, L);
        default: return NarrowPlan{};  // more than 65536 rows of X do not fit
    }
}

template <typename IdxT>
hipError_t launch_narrow_t(const NarrowPlan& p, const NarrowArgs& a, size_t budget, hipStream_t stream) {
    void (*kern)(NarrowArgs);
    constexpr bool kWide = sizeof(IdxT) > 1;
    const bool few = p.few;
    int slot;
    switch (p.V) {
        case 8: kern = cer_narrow_kernel<IdxT, 8, false>; slot = 3; break;
        case 4: kern = few ? cer_narrow_kernel<IdxT, 4, kWide> : cer_narrow_kernel<IdxT, 4, false>; slot = 2; break;
        case 2: kern = few ? cer_narrow_kernel<IdxT, 2, kWide> : cer_narrow_kernel<IdxT, 2, false>; slot = 1; break;
        default: kern = few ? cer_narrow_kernel<IdxT, 1, kWide> : cer_narrow_kernel<IdxT, 1, false>; slot = 0;
    }
    if (p.lds > 48 * 1024) {
        static LdsGrant<8> grant;
        const hipError_t e = grant.ensure(slot + (few ? 4 : 0), reinterpret_cast<const void*>(kern), budget);
        if (e != hipSuccess) return e;
    }
    return launch_kernel(kern, dim3(p.row_blocks * p.passes), dim3(p.waves * kWave), p.lds, stream, a);
}

}  // namespace

NarrowEstimate narrow_estimate(const DeviceView& d, uint32_t L) {
    const NarrowPlan p = plan_narrow(d, L);
    return p.V > 0 ? NarrowEstimate{p.V, p.us} : NarrowEstimate{};
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
    const size_t budget = d.lds_per_block - 256;
    return d.colI_bits == 8 ? launch_narrow_t<uint8_t>(p, a, budget, stream) : launch_narrow_t<uint16_t>(p, a, budget, stream);
}

}  // namespace cer
