// What the bf16 prefill and its backward share: 32-row blocks of bf16 rows in
// LDS, their LDS-DMA requests and matrix-core fragments (v_mfma 32x32x16), and
// the plan of the key blocks a tile of query positions reads.
#pragma once

#include <type_traits>

#include "eva_device.hpp"
#include "eva_kernels.hpp"

namespace eva {

constexpr int kTileRows = 32;    // rows per block; each of the kTileWaves waves requests a part of it
constexpr int kFragAhead = 3;    // LDS fragments requested ahead of their product

// A block of 32 rows (D features) in LDS.  One DMA instruction moves 1 KB
// (RPI rows); consecutive instructions' rows lie 64 bytes further apart than
// their size, which with the permutation key_of spreads every fragment read
// over the banks with immediate offsets from one or two lane addresses.
template <int D>
struct Tile {
    static constexpr int ROWB = D * 2;          // bytes per row
    static constexpr int RPI = 1024 / ROWB;     // rows per DMA instruction
    static constexpr int GRP = 1024 + 64;       // LDS bytes from one instruction's rows to the next's
    static constexpr int BLK = kTileRows / RPI * GRP;             // LDS bytes per block
    static constexpr int NI = kTileRows / RPI / kTileWaves;       // DMA instructions per wave and block
    static_assert(NI >= 1, "every wave requests a part of every block");
    static constexpr int NDC = D / 16;          // contraction steps over the features
    static constexpr int NDB = D / 32;          // 32-feature output blocks
    static constexpr int NKC = kTileRows / 16;  // contraction steps over a block's rows
    // LDS byte offset of a row within its block
    static constexpr __host__ __device__ int row_at(int r) { return r / RPI * GRP + r % RPI * ROWB; }
    // Row 8q + 4h + i of a product whose A operand is the block (element
    // 4q + i of a lane of half h) is block row key_of(q, i) + h * KH.  The
    // four rows i of a transposing read then lie 64 bytes apart modulo the
    // 256 bytes of the banks (in other DMA groups, or in the two halves of
    // 256 bytes for 128-byte rows).
    static constexpr int KH = D == 128 ? 1 : 4;
    static constexpr __host__ __device__ int key_of(int q, int i) {
        return 16 * (q >> 1) + 2 * (q & 1) + (D == 128 ? 4 * i : 8 * (i >> 1) + (i & 1));
    }
    // stored 16-B chunk of a row = logical chunk ^ swz(row) (the low two
    // bits): a 16-lane fragment read finds 16 rows on distinct banks.  Rows
    // that are only read transposed need no swizzle.
    static constexpr __host__ __device__ int swz(int r) { return D == 128 ? r & 3 : (r >> 1) & 3; }
};

// Buffer descriptor of `rows` rows at address p: reads past them return zeros
// without a memory access.
template <int D>
__device__ __forceinline__ u32x4 rows_desc(uintptr_t p, int rows) {
    return u32x4{(uint32_t)p, (uint32_t)(p >> 32) & 0xffffu, (uint32_t)(rows * Tile<D>::ROWB), 0x00020000u};
}

__device__ __forceinline__ unsigned lds_addr(const void* p) {
    return (unsigned)(size_t)(__attribute__((address_space(3))) const void*)p;
}

// 16 bytes per lane from desc + voff + soff to LDS dst + 16 lane.  Inline
// assembly, so that the compiler, which cannot see the LDS write, leaves the
// waits to the kernel.  M0 holds the LDS address; the load needs one wait
// state after M0 is written.
__device__ __forceinline__ void dma16(const u32x4& desc, unsigned voff, unsigned soff, unsigned dst) {
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(desc), "s"(soff), "{m0}"(dst)
                 : "memory");
}

// the same with 4 bytes per lane, to LDS dst + 4 lane
__device__ __forceinline__ void dma4(const u32x4& desc, unsigned voff, unsigned dst) {
    asm volatile("s_nop 0\n\tbuffer_load_dword %0, %1, 0 offen lds" ::"v"(voff), "s"(desc), "{m0}"(dst) : "memory");
}

// This lane's source offset in a block's requests: the rows of DMA
// instruction i of wave w are (4 i + w) RPI ..; i adds 4 KB of source and
// 4 GRP of LDS, and keeps the swizzle.
template <int D, bool SWZ>
__device__ __forceinline__ unsigned dma_lane_off(int wave, int lane) {
    typedef Tile<D> T;
    const int row = lane * 16 / T::ROWB, pos = (lane * 16 % T::ROWB) / 16;
    return (wave * T::RPI + row) * T::ROWB + ((SWZ ? pos ^ T::swz(row) : pos) << 4);
}
// the wave's share of a block (base: LDS address of the block + wave * GRP)
template <int D>
__device__ __forceinline__ void dma_block(const u32x4& desc, unsigned lane_off, unsigned base) {
#pragma unroll
    for (int i = 0; i < Tile<D>::NI; ++i) dma16(desc, lane_off, i * kTileWaves * 1024, base + i * kTileWaves * Tile<D>::GRP);
}

// Fragment reads of a block.
template <int D>
struct Frags {
    typedef Tile<D> T;
    int r0, r1;  // 16-byte row fragments, even and odd feature steps (swizzled rows)
    int t0, t1;  // transposing reads: rows of q even / odd; swizzled or plain rows
    __device__ Frags(int lane, bool tr_swizzled) {
        const int c32 = lane & 31, h2 = lane >> 5;
        const int row = T::key_of(c32 >> 3, c32 & 3) + ((c32 >> 2) & 1) * T::KH;
        r0 = T::row_at(row) + ((h2 ^ T::swz(row)) << 4);
        r1 = r0 ^ 32;
        // lane names row i = lane%16 / 4 of half h2, features 16 (lane/16 % 2) + 4 (lane%4) ..
        const int tr = T::key_of(0, (lane >> 2) & 3) + h2 * T::KH;
        const int ch = 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
        t0 = T::row_at(tr) + ((tr_swizzled ? ch ^ T::swz(tr) : ch) << 4) + (lane & 1) * 8;
        t1 = (tr_swizzled ? t0 ^ (((T::swz(tr) ^ T::swz(tr + 2)) & 3) << 4) : t0) + 2 * T::ROWB;
    }
    // A operand: rows of the block (c32 -> row), features 16 dc + 8 h2 ..
    __device__ __forceinline__ bf16x8 row(const unsigned char* blk, int dc) const {
        return *reinterpret_cast<const bf16x8*>(blk + ((dc & 1) ? r1 : r0) + (dc >> 1) * 64);
    }
    // A operand of a transposed product: features 32 db + c32, contraction
    // over the block rows of product elements 8 kc .. +7
    __device__ __forceinline__ bf16x8 tr(const unsigned char* blk, int db, int kc) const {
        const unsigned char* p = blk + db * 64 + T::row_at(kc * 16);
        const shortx4 lo = lds_read_tr16(reinterpret_cast<const bf16*>(p + t0));
        const shortx4 hi = lds_read_tr16(reinterpret_cast<const bf16*>(p + t1));
        return __builtin_bit_cast(
            bf16x8, (short __attribute__((ext_vector_type(8)))){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    }
};

// One wave's 32 rows of a tensor (its columns) as B operands: whole rows go
// through LDS (an area of one block, the wave's own), since a lane per row
// reading 16 bytes straight from memory costs the address unit 64 accesses an
// instruction instead of 16.  Rows past the descriptor are zeros.
template <int D>
__device__ __forceinline__ void stage_cols(const u32x4& desc, int lane, unsigned dst) {
    const unsigned off = dma_lane_off<D, true>(0, lane);
    u32x4 d;  // wave-uniform, also where the compiler computed it in vector registers
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = __builtin_amdgcn_readfirstlane(desc[i]);
#pragma unroll
    for (int i = 0; i < kTileRows / Tile<D>::RPI; ++i) dma16(d, off, i * 1024, dst + i * Tile<D>::GRP);
}
// column c32, features 16 dc + 8 h2 ..
template <int D>
__device__ __forceinline__ void read_cols(const unsigned char* blk, int lane, bf16x8 (&f)[D / 16]) {
    const int c32 = lane & 31, h2 = lane >> 5;
    const unsigned char* p = blk + Tile<D>::row_at(c32);
    const int x = (h2 ^ Tile<D>::swz(c32)) << 4;
#pragma unroll
    for (int dc = 0; dc < D / 16; ++dc)
        f[dc] = *reinterpret_cast<const bf16x8*>(p + ((dc & 1) ? x ^ 32 : x) + (dc >> 1) * 64);
}

// Sum over the lanes that hold one row of 16-byte chunks (D / 8 neighbours).
template <int D>
__device__ __forceinline__ float row_lanes_sum(float x) {
    auto dpp = [](float v, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    x += dpp(x, std::integral_constant<int, 0xB1>{});   // lanes 1 0 3 2
    x += dpp(x, std::integral_constant<int, 0x4E>{});   // lanes 2 3 0 1
    x += dpp(x, std::integral_constant<int, 0x141>{});  // mirrored within 8
    if constexpr (D == 128) x += dpp(x, std::integral_constant<int, 0x140>{});  // mirrored within 16
    return x;
}

// The lane id, computed where it is used: a value that depends on the lane
// kept over the block loop only for the rare masks would take a register.
__device__ __forceinline__ int lane_here() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
    return l;
}

// Elements of a score tile whose block row x (less h2 KH) is above hi / below lo to -inf.
template <int D>
__device__ __forceinline__ void mask_above(floatx16& s, int hi) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = Tile<D>::key_of(i / 4, i % 4) <= hi ? s[i] : -INFINITY;
}
template <int D>
__device__ __forceinline__ void mask_below(floatx16& s, int lo) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = Tile<D>::key_of(i / 4, i % 4) >= lo ? s[i] : -INFINITY;
}

// The key blocks of a workgroup's query positions [n0, n_hi]: summaries
// [0, sum_lo(n_hi)) (non-causal: all), then the band [win_lo(n0),
// win_hi(n_hi)]; block j of the band is rows (j - shift) * 32 ..  And which of
// them a wave's 32 positions from p0 on need (some pair visible) and see in
// full, as ranges of block numbers.
template <int VAR>
struct KeyPlan {
    static constexpr bool NC = VAR == kWinNonCausal;
    static constexpr int BN = kTileRows;
    int nsb, shift, nb;               // summary blocks, shift of the band's numbers, all blocks
    int sn1, sf1, xn0, xf0, xf1;      // summaries: needed j < sn1 (non-causal: or j >= xn0), full j < sf1 (or [xf0, xf1))
    int wn0, wf0;                     // window: needed wn0 .. +wnc-1, full wf0 .. +wfc-1
    unsigned wnc, wfc;
    int whi_min, wlo_max;
    __device__ __forceinline__ KeyPlan(int n0, int n_hi, int p0, int L, const FastDiv& W, const FastDiv& C,
                                       int n_chunks) {
        nsb = ((NC ? n_chunks : sum_lo<VAR>(n_hi, W, C)) + BN - 1) / BN;
        const int kb0 = win_lo<VAR>(n0, W, C) / BN;
        nb = nsb + (win_hi<VAR>(n_hi, W, L) / BN - kb0 + 1);
        shift = nsb - kb0;
        const bool active = p0 < L;
        const int last = min(p0 + 31, L - 1);
        whi_min = win_hi<VAR>(p0, W, L);
        wlo_max = win_lo<VAR>(last, W, C);
        sn1 = active ? (sum_lo<VAR>(last, W, C) + BN - 1) / BN : 0;
        sf1 = sum_lo<VAR>(p0, W, C) / BN;
        xn0 = NC && active ? sum_hi<VAR>(p0, W, C, L) / BN : nsb;
        xf0 = NC ? (sum_hi<VAR>(last, W, C, L) + BN - 1) / BN : nsb;
        xf1 = NC ? n_chunks / BN : 0;
        wn0 = win_lo<VAR>(p0, W, C) / BN + shift;
        wnc = active ? win_hi<VAR>(last, W, L) / BN + shift - wn0 + 1 : 0;
        wf0 = (wlo_max + BN - 1) / BN + shift;
        wfc = max(0, (whi_min + 1) / BN + shift - wf0);
    }
    __device__ __forceinline__ bool needed(int j) const {
        return j < sn1 || (NC && j >= xn0 && j < nsb) || (unsigned)(j - wn0) < wnc;
    }
    __device__ __forceinline__ bool full(int j) const {
        return j < sf1 || (NC && j >= xf0 && j < xf1) || (unsigned)(j - wf0) < wfc;
    }
    // scores of block j (rows: keys, columns: positions p0 + c32) that their
    // column does not see to -inf; for blocks that are not full
    template <int D>
    __device__ __forceinline__ void mask(floatx16& s, int j, int p0, int L, const FastDiv& W, const FastDiv& C,
                                         int n_chunks) const {
        const int l = lane_here();
        const int hk = (l >> 5) * Tile<D>::KH, n = min(p0 + (l & 31), L - 1);
        if (j < nsb) {
            // summary c visible iff c < sum_lo(n) (non-causal: or sum_hi(n) <= c < n_chunks)
            const int rel = j * BN + hk;
            const int hi = sum_lo<VAR>(n, W, C) - 1 - rel;
            if constexpr (NC) {
                const int lo = sum_hi<VAR>(n, W, C, L) - rel, end = n_chunks - rel;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int x = Tile<D>::key_of(i / 4, i % 4);
                    const bool ok = x <= hi || (x >= lo && x < end);
                    s[i] = ok ? s[i] : -INFINITY;
                }
            } else {
                mask_above<D>(s, hi);
            }
        } else {
            const int base = (j - shift) * BN;
            const int rel = base + hk;
            if (base + BN - 1 > whi_min) mask_above<D>(s, win_hi<VAR>(n, W, L) - rel);
            if (base < wlo_max) mask_below<D>(s, win_lo<VAR>(n, W, C) - rel);
        }
    }
};

// The requests of a key plan: descriptors of block j's key and value rows.
// With the band's base pointers shifted back by the summary blocks both are
// "base + j blocks".  The descriptor covers the block's valid rows only: rows
// past the end, and every row of a block past the last one, are zeros in LDS
// without a memory access, so that every wave has the same number of requests
// in flight at every wait.
template <int D>
struct KeySource {
    uintptr_t ks, vs, kw, vw;
    int sum_limit, win_limit, nsb, nb;
    template <int VAR>
    __device__ __forceinline__ KeySource(const KeyPlan<VAR>& p, const void* K, const void* V, const void* Ks,
                                         const void* Vs, size_t bg, int L, int n_chunks) {
        constexpr int ROWB = Tile<D>::ROWB;
        const uintptr_t back = (uintptr_t)((intptr_t)p.shift * kTileRows * ROWB);
        ks = (uintptr_t)Ks + bg * (size_t)n_chunks * ROWB;
        vs = (uintptr_t)Vs + bg * (size_t)n_chunks * ROWB;
        kw = (uintptr_t)K + bg * (size_t)L * ROWB - back;
        vw = (uintptr_t)V + bg * (size_t)L * ROWB - back;
        sum_limit = n_chunks;
        win_limit = L + p.shift * kTileRows;
        nsb = p.nsb;
        nb = p.nb;
    }
    __device__ __forceinline__ void block(int j, u32x4& dk, u32x4& dv) const {
        const bool sum = j < nsb;
        const uintptr_t off = (uintptr_t)j * (kTileRows * Tile<D>::ROWB);
        const int rows = j < nb ? min((sum ? sum_limit : win_limit) - j * kTileRows, kTileRows) : 0;
        dk = rows_desc<D>((sum ? ks : kw) + off, rows);
        dv = rows_desc<D>((sum ? vs : vw) + off, rows);
    }
};

// Tile of a workgroup (PosTiles): consecutive tiles of one (b, kv head) land
// on the same XCD (its L2 then holds the keys they share), heavy (late)
// position tiles first.
struct PosTile {
    int b, kvh, h, n0, p0;  // h and p0: this wave's head and first position
    __device__ __forceinline__ PosTile(const PosTiles& t, int block, int wave) {
        int id = block;
        const int per = t.n_tiles / 8;
        if (id < per * 8) id = (id % 8) * per + id / 8;
        const int q_pos = id / t.f_pos_tiles, q_hg = q_pos / t.f_hg;
        const int pt = t.n_pos_tiles - 1 - (id - q_pos * t.n_pos_tiles);
        const int hg = q_pos - q_hg * t.n_hg;
        b = q_hg / t.f_hkv;
        kvh = q_hg - b * t.Hkv;
        h = kvh * t.G + hg * t.Gt + (wave & (t.Gt - 1));
        n0 = pt * t.pos_per_wg;
        p0 = n0 + (wave >> t.gt_shift) * 32;
    }
};

// 32 rows of a wave (column c32 of the 32x32 accumulators acc, features
// 32 db + 8 q + 4 h2 + i as element 4 q + i) as whole bf16 rows to
// base + r * D for r < n_valid: staged in LDS (stg: 32 rows of kStageRow<D>
// bytes, the wave's own), so that each store instruction writes whole rows
// instead of 32 pieces of 16 bytes.  val(db, i) gives an element's value.
// Stores are non-temporal: nothing reads the rows again soon.
template <int D>
constexpr int kStageRow = 2 * D + 16;  // 16 bytes of skew: fragment writes fall in distinct banks
template <int D, typename F>
__device__ __forceinline__ void store_tile_rows(unsigned char* stg, int lane, bf16* base, int n_valid, F&& pair) {
    constexpr int SROW = kStageRow<D>;
    constexpr int LPR = 2 * D / 16;  // lanes per row (16 bytes each)
    constexpr int RPS = 64 / LPR;    // rows per store instruction
    const int c32 = lane & 31, h2 = lane >> 5;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x2 w = {pair(db, 4 * q), pair(db, 4 * q + 2)};
            *reinterpret_cast<u32x2*>(stg + c32 * SROW + (db * 32 + 8 * q + 4 * h2) * 2) = w;
        }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int i = 0; i < 32 / RPS; ++i) {
        const int r = i * RPS + lane / LPR;
        const u32x4 x = *reinterpret_cast<const u32x4*>(stg + r * SROW + (lane % LPR) * 16);
        if (r < n_valid)
            __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(base + (size_t)r * D + (lane % LPR) * 8));
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace eva
