// Shared by the kernels that stream colI with 16-byte loads (cer_gemv.hip, cer_narrow.hip): the shape of a batch of positions
// and the turning of group boundaries into per-position weights without searches or data-dependent branches.
#pragma once

#include "cer_device.hpp"

namespace cer {

// kNW: windows per batch, 0 = the default (2, 3, 4 for 8-, 16-, 32-bit indices: a batch of 2048, 1536, 1024 positions --
// one batch for the rows of the layer shapes).  Rows of many windows run faster in batches of two windows (the 7-bit
// layer of 7000 indices per row: 15.1 us with 3 windows per batch, 14.2 with 2, 14.9 with 1, 14.7 with 4).
template <typename IdxT, int kNW = 0>
struct GemvShape {
    static constexpr int PPL = 16 / (int)sizeof(IdxT);  // positions per lane and 16-byte load: 16, 8, 4
    static constexpr int WIN = kWave * PPL;             // positions per window (one load per lane)
    static constexpr int NW = kNW ? kNW : (sizeof(IdxT) == 1 ? 2 : (sizeof(IdxT) == 2 ? 3 : 4));  // windows per batch
    static constexpr int BATCH = NW * WIN;              // 2048, 1536, 1024 positions
    static constexpr int NWORDS = BATCH / 32;           // bitmap words per batch: 64, 48, 32 (at most one per lane)
    static constexpr int WPW = WIN / 32;                // bitmap words per window
};

// Inclusive prefix sum over the 64 lanes: four shifted adds inside each row of 16 lanes, then the totals of rows 0
// and 2 are added to rows 1 and 3, then the total of rows 0 - 1 to rows 2 - 3.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
#define CER_SCAN_STEP(CTRL, ROWS) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
    CER_SCAN_STEP(0x111, 0xF)  // row_shr:1
    CER_SCAN_STEP(0x112, 0xF)  // row_shr:2
    CER_SCAN_STEP(0x114, 0xF)  // row_shr:4
    CER_SCAN_STEP(0x118, 0xF)  // row_shr:8
    CER_SCAN_STEP(0x142, 0xA)  // row_bcast:15 into rows 1 and 3
    CER_SCAN_STEP(0x143, 0xC)  // row_bcast:31 into rows 2 and 3
#undef CER_SCAN_STEP
    return v;
}

// Boundary bitmap of the batch [b0, b0 + BATCH): bit p is set when a list entry ends at position b0 + p + 1, i.e.
// position b0 + p is the last one of its group.  `first` = number of list entries that end at or before b0 (the
// list index of the group position b0 belongs to); `last` = index of the list's second sentinel.  Afterwards
// wpre[j] = first + the number of boundary bits in words 0 .. j-1, and `first` has moved past the batch.
template <typename S>
__device__ __forceinline__ void bitmap_build(const uint32_t* ends, uint32_t last, uint32_t& first, uint32_t b0,
                                             uint32_t* bmp, uint32_t* wpre, uint32_t lane) {
    if (lane < (uint32_t)S::NWORDS) bmp[lane] = 0u;
    wave_lds_sync();
    for (uint32_t i = first;; i += kWave) {
        const uint32_t e = ends[min(i + lane, last)];  // the sentinels (2^32 - 1) are beyond every batch
        const uint32_t rel = e - b0 - 1u;
        if (rel < (uint32_t)S::BATCH) atomicOr(&bmp[rel >> 5], 1u << (rel & 31u));  // LDS operations of a wave run in order
        if (__builtin_amdgcn_readlane(e, kWave - 1) - b0 > (uint32_t)S::BATCH) break;  // wave-uniform
    }
    wave_lds_sync();
    const uint32_t pc = lane < (uint32_t)S::NWORDS ? (uint32_t)__builtin_popcount(bmp[min(lane, (uint32_t)S::NWORDS - 1u)]) : 0u;
    const uint32_t incl = wave_inclusive_scan(pc);
    if (lane < (uint32_t)S::NWORDS) wpre[lane] = first + incl - pc;
    first += __builtin_amdgcn_readlane(incl, kWave - 1);
    wave_lds_sync();
}

// Number of entries of the wave's list (count entries, sentinels behind them) that end at or before position b: the
// list index of the group position b belongs to.
__device__ __forceinline__ uint32_t list_rank_of(const uint32_t* ends, int count, uint32_t b, uint32_t lane) {
    uint32_t f = 0;
    for (int i = 0; i < count; i += kWave) {
        const uint32_t e = ends[min(i + (int)lane, count)];
        f += (uint32_t)__popcll(__ballot(i + (int)lane < count && e <= b));
    }
    return f;
}

// Weights of the PPL positions lane l holds in window W of the batch: wl[k] = value - Omega[0] of the group that
// position b0 + W.WIN + PPL.l + k belongs to (0 in front of the row and behind it).
template <typename S>
__device__ __forceinline__ void window_weights(int W, const uint32_t* bmp, const uint32_t* wpre, const float* wts,
                                               uint32_t lane, float (&wl)[S::PPL]) {
    const uint32_t bit0 = (uint32_t)S::PPL * lane;  // the lane's first bit inside the window
    const uint32_t wj = (uint32_t)W * S::WPW + (bit0 >> 5), sh = bit0 & 31u;
    const uint32_t word = bmp[wj];
    const uint32_t pre = wpre[wj] + (uint32_t)__builtin_popcount(word & ((1u << sh) - 1u));
    const uint32_t field = word >> sh;  // bit k: position k is the last one of its group
    // the LDS address of the position's list entry moves on by one entry behind every boundary bit: one bit-field
    // extract and one shift-add per position
    typedef const float __attribute__((address_space(3))) * LdsFloatPtr;
    uint32_t addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const float*)wts + (pre << 2);
#pragma unroll
    for (int k = 0; k < S::PPL; ++k) {
        wl[k] = *reinterpret_cast<LdsFloatPtr>((uintptr_t)addr);
        if (k + 1 < S::PPL) {
            uint32_t bit;  // written out so that it stays one extract (the compiler turns it into shift + and)
            asm("v_bfe_u32 %0, %1, %2, 1" : "=v"(bit) : "v"(field), "n"(k));
            asm("v_lshl_add_u32 %0, %1, 2, %0" : "+v"(addr) : "v"(bit));  // addr += 4 * bit
        }
    }
}

// Column index of the k-th of the positions packed into one 16-byte load.
template <typename IdxT>
__device__ __forceinline__ uint32_t packed_index(const uint4& q, int k) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    if (sizeof(IdxT) == 4) return w[k];
    if (sizeof(IdxT) == 2) return (k & 1) ? (w[k >> 1] >> 16) : (w[k >> 1] & 0xFFFFu);
    return (w[k >> 2] >> (8 * (k & 3))) & 0xFFu;
}

// Appends the non-empty groups among raw groups [j0, tg_end) of the row that starts at group g0 to the wave's list.
// The pointer tiles are requested four at a time (tiles past tg_end read the padding behind the pointer arrays and
// come back empty): a row of 256 raw groups waits for memory once, not four times.
__device__ __forceinline__ int list_append_tiles(const KView& v, bool cser, const float* omega, uint32_t g0, uint32_t j0,
                                                 uint32_t tg_end, uint32_t* ends, float* wts, int count, uint32_t lane) {
    for (; j0 < tg_end; j0 += 4u * kWave) {
        PtrTile p[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) p[t] = load_ptr_tile(v, cser, g0, min(j0 + (uint32_t)t * kWave, tg_end), tg_end, lane);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (j0 + (uint32_t)t * kWave < tg_end)  // wave-uniform
                count = list_append(p[t], omega[p[t].rank < v.K ? p[t].rank : 0u] - v.omega0, ends, wts, count);
    }
    return count;
}

// Byte offset (4 x column index) of the k-th of the positions packed into one 16-byte load: for 8- and 16-bit
// indices one instruction that selects the byte or half-word and shifts it (sub-dword addressing of the vector ALU).
template <typename IdxT>
__device__ __forceinline__ uint32_t packed_offset(const uint4& q, int k, uint32_t two) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    uint32_t r;
    if (sizeof(IdxT) == 4) {
        r = w[k] << 2;
    } else if (sizeof(IdxT) == 2) {
        const uint32_t d = w[k >> 1];
        if (k & 1) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(r) : "v"(two), "v"(d));
        else asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(r) : "v"(two), "v"(d));
    } else {
        const uint32_t d = w[k >> 2];
        switch (k & 3) {
            case 0: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(two), "v"(d)); break;
            case 1: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(two), "v"(d)); break;
            case 2: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(two), "v"(d)); break;
            default: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "v"(two), "v"(d)); break;
        }
    }
    return r;
}

}  // namespace cer
