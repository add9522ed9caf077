// Backward pass of the fused EVA prefill (bf16, every window variant): dQ, dK, dV
// of a loss given dO, through the window keys/values, the summary keys and
// values, and the summaries' own dependence on K and V.
//
// Notation: logits l = q.k / sqrt(d) (+ ln C for a summary), the row's
// softmax P = exp(l - lse) with lse saved by the forward, D = dO . O per row,
// dS = P (dP - D) with dP = dO . v.  Then dq = sum dS k / sqrt(d),
// dk += dS q / sqrt(d), dv += P dO (FlashAttention-style recomputation: no
// attention matrix is stored).
//
// Kernels (all bf16 storage, fp32 arithmetic, v_mfma_f32_16x16x32_bf16):
//   bwd_dq_kernel      per query tile (4 waves x 32 columns, the forward's
//                      tiles): the columns' D = dO . O (stored for the dK/dV
//                      kernels), then key blocks of 32 rows (summaries then
//                      window band) streamed through LDS: S^T = K Q^T,
//                      dP^T = V dO^T, dS^T, and dQ^T += K^T dS^T
//                      (v_mfma 32x32x16; K^T by the transposing LDS read)
//   bwd_dkdv_kernel    per key tile (4 waves x 16 keys, window keys or
//                      summaries of one kv head), query blocks of 32 rows of
//                      every head of the group streamed through LDS:
//                      S = Q K^T, dP = dO V^T, dS, dV^T += dO^T P,
//                      dK^T += Q^T dS.  Summary tiles run first and leave
//                      fp32 summary gradients; window tiles run last and add
//                      each key's share of its chunk's summary gradient
//                      before storing dK, dV as bf16
//   bwd_summary_kernel per chunk, between the two: through khat = mean and
//                      the chunk softmax (vhat = sum_j b_j v_j,
//                      b = softmax(khat . k / sqrt(d))); leaves khat, the
//                      total gradient of khat, and each key's b_j and
//                      logit gradient da_j, from which
//                        dk_j += da_j khat / sqrt(d) + dkhat / C,
//                        dv_j += b_j dvhat
// The fragment layouts are those of the forward kernel: streamed rows are the
// A operand (16-B row reads, or transposing reads for the transposed
// products), the stationary rows are B-operand fragments in registers, and
// the 16x16 score tiles of two key (or query) halves form the next product's
// B operand in place.
#include <type_traits>

#include "summary.hpp"
#include "tile32.hpp"

namespace eva {

namespace {

constexpr int kBwdWaves = 4;
constexpr int kBwdBN = 32;     // rows per streamed block
// dQ: four ring stages (70 KB of LDS, two workgroups per CU; 204 VGPRs), so
// that the ring holds the q and dO rows of the whole workgroup while they are
// staged.  Three stages measured the same.
constexpr int kDqNS = 4;
#ifndef KVPF
#define KVPF 2
#endif
constexpr int kKvRing = 4, kKvPF = KVPF;
// dK/dV: LDS ring stages and blocks requested ahead of the one computed.
// It fits 168 VGPRs, so three stages (50 KB) let three workgroups share a CU
// (measured on MI355X: 631 vs 767 us for the window tiles of the LLM workload)
constexpr int kKvNS = 3, kKvAhead = 2;

// s_waitcnt vmcnt(N) lgkmcnt(0): the kernel's own DMA requests are invisible
// to the compiler, so every wait for them is explicit
template <int N>
__device__ __forceinline__ void bwait_vm() {
    static_assert(N < 64, "vmcnt field is 6 bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}
// wait for a block (LATER DMA instructions issued after it may stay in
// flight), then a workgroup barrier: the block is visible to every wave, and
// every wave is done with the stage the next request refills
template <int LATER>
__device__ __forceinline__ void bsync() {
    asm volatile("" ::: "memory");
    bwait_vm<LATER>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int D>
struct BCfg {
    static constexpr int ROWB = 2 * D;            // bytes per row
    static constexpr int CPR = ROWB / 16;         // 16-B chunks per row
    static constexpr int BLK = kBwdBN * ROWB;     // bytes per block
    static constexpr int NI = BLK / 1024 / kBwdWaves;  // DMA instructions per wave per array
    static constexpr int NDC = D / 32;            // contraction steps over features
    static constexpr int NDB = D / 16;            // 16-feature output blocks
};

// stored 16-B chunk = logical chunk ^ bswz(row): conflict-free 16-B row reads
template <int CPR>
__device__ __forceinline__ int bswz(int r) {
    return CPR >= 16 ? (r & 15) : ((r >> 1) & 7);
}

__device__ __forceinline__ void bdma16(const void* base, unsigned voff, unsigned lds_addr) {
    asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "{m0}"(__builtin_amdgcn_readfirstlane(lds_addr))
                 : "memory");
}

template <int D>
struct Stager {
    typedef BCfg<D> Cfg;
    int row[Cfg::NI], off[Cfg::NI];  // per DMA instruction: source row and chunk byte offset
    __device__ Stager(int wave, int lane) {
#pragma unroll
        for (int i = 0; i < Cfg::NI; ++i) {
            const int byte = (i * kBwdWaves + wave) * 1024 + lane * 16;
            const int r = byte / Cfg::ROWB;
            const int pos = (byte % Cfg::ROWB) / 16;
            row[i] = r;
            off[i] = (pos ^ bswz<Cfg::CPR>(r)) << 4;
        }
    }
    // rows [0, n_valid) of `src` (row-major, D bf16 each) into the LDS block at
    // lds_addr; rows past n_valid repeat the last valid row (finite, masked).
    // With real false the same number of instructions read row 0 of src into
    // the 1-KB area at lds_addr (requests past the last block).
    __device__ void issue(const bf16* src, int n_valid, unsigned lds_addr, int wave, bool real = true) const {
#pragma unroll
        for (int i = 0; i < Cfg::NI; ++i) {
            const int r = real ? min(row[i], n_valid - 1) : 0;
            bdma16(src, (unsigned)(r * Cfg::ROWB + off[i]), real ? lds_addr + (i * kBwdWaves + wave) * 1024 : lds_addr);
        }
    }
};

template <int D>
__device__ __forceinline__ unsigned lds_addr_of(const void* p) {
    return lds_addr(p);
}

// 16-B row fragment: row kb*16 + c16, features dc*32 + 8g .. +7
template <int D>
__device__ __forceinline__ bf16x8 row_frag(const unsigned char* blk, int kb, int dc, int c16, int g) {
    typedef BCfg<D> Cfg;
    const int r = kb * 16 + c16;
    const int chunk = (dc * 4 + g) ^ bswz<Cfg::CPR>(r);
    return *reinterpret_cast<const bf16x8*>(blk + r * Cfg::ROWB + chunk * 16);
}

// transposing fragment (A operand of a transposed product): lane (g, c16)
// receives feature db*16 + c16 of rows 4g .. 4g+3 and 16+4g .. 16+4g+3
template <int D>
__device__ __forceinline__ bf16x8 tr_frag(const unsigned char* blk, int db, int c16, int g) {
    typedef BCfg<D> Cfg;
    const int r = g * 4 + (c16 >> 2);
    const int t = c16 & 3;
    const int chunk = (2 * db + (t >> 1)) ^ bswz<Cfg::CPR>(r);
    const unsigned char* p = blk + r * Cfg::ROWB + chunk * 16 + (t & 1) * 8;
    const shortx4 lo = lds_read_tr16(reinterpret_cast<const bf16*>(p));
    // row r + 16 has the same swizzle (bswz depends on r mod 16)
    const shortx4 hi = lds_read_tr16(reinterpret_cast<const bf16*>(p + 16 * Cfg::ROWB));
    return __builtin_bit_cast(
        bf16x8, (short __attribute__((ext_vector_type(8)))){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
}

// B-operand fragment in the contraction order of tr_frag: element e is tile
// kb = e / 4, row 4g + e % 4 of a pair of 16x16 output tiles
__device__ __forceinline__ bf16x8 pair_to_b(const floatx4& t0, const floatx4& t1) {
    bf16x8 f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[i] = to_bf16(t0[i]);
        f[4 + i] = to_bf16(t1[i]);
    }
    return f;
}

// ---------------------------------------------------------------------------
// dQ
// ---------------------------------------------------------------------------
// The forward's tiles and key blocks (tile32.hpp): a wave owns 32 query
// columns, whose q and dO rows are B operands in registers.  Per block:
// S^T = K Q^T, then dP^T = V dO^T with the exponentials of S between its
// products, then dQ^T += K^T dS^T (K rows read transposed from the same block)
// with the second half's dS between.
// What bounds it (MI355X; B8 H32 L4096 W256 C64 / B4 H32/8 L8192 W512 C128):
// 544 / 651 us with 16 columns per wave of 16x16x32 products (24 KB of LDS
// reads per 24 products of 16 cycles, every key block staged twice as often,
// neighbouring tiles on different XCDs); 515 / 580 with 32 columns, of which
// the scattered loads of q, dO, O and O_lo took 22k of a workgroup's 66k
// cycles (one 16-byte access per row and lane); 411 / 481 with whole rows
// staged.  The first shape's 1.9 GB take ~310 us at the rate of a plain read.
template <int D, int NS, int WPE, int VAR>
__global__ __launch_bounds__(kTileWaves * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void bwd_dq_kernel(BwdParams a) {
    typedef Tile<D> T;
    constexpr int BLK = T::BLK, NKC = T::NKC, NDC = T::NDC, NDB = T::NDB;
    constexpr int NIT = 2 * T::NI;  // requests per wave and block
    constexpr int AHEAD = NS - 1;   // blocks requested ahead of the one computed
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NS][2][BLK];  // [stage][K, V]
    __shared__ float dsh[kTileWaves][2][kTileRows];  // per wave and column: D, -lse in log2 units

    const int L = a.L;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c32 = lane & 31;
    const PosTile tile(a.t, blockIdx.x, wave);
    const int p0 = tile.p0;
    const KeyPlan<VAR> plan(tile.n0, min(tile.n0 + a.t.pos_per_wg, L) - 1, p0, L, a.fW, a.fC, a.n_chunks);
    const int nb = plan.nb;
    const KeySource<D> src(plan, a.K, a.V, a.Ks, a.Vs, (size_t)tile.b * a.Hkv + tile.kvh, L, a.n_chunks);
    const unsigned lane_off = dma_lane_off<D, true>(wave, lane);
    const unsigned lds0 = lds_addr(lds) + wave * T::GRP;
    auto request = [&](int j, int stage) {
        u32x4 dk, dv;
        src.block(j, dk, dv);
        dma_block<D>(dk, lane_off, lds0 + stage * 2 * BLK);
        dma_block<D>(dv, lane_off, lds0 + stage * 2 * BLK + BLK);
    };

    // stationary columns (past L: zeros, whose results are not stored): q and
    // dO as B operands through the ring, lse, and D = dO . O (O + O_lo when the
    // forward kept its output's rounding residual), stored negated for the
    // dK/dV kernels.  The dots run on whole rows: O and O_lo are read into
    // the same chunk layout as the staged dO rows.
    const size_t row0 = ((size_t)tile.b * a.H + tile.h) * L + p0;
    const int n_cols = max(0, min(32, L - p0));
    bf16x8 qf[NDC], gf[NDC];
    float off0, dcol;  // -lse in log2 units; D
    {
        // one block per wave in stages 2 and 3 of the ring: dO, then Q; the
        // first two key blocks land in stages 0 and 1 meanwhile
        static_assert(NS == 4, "stages 2 and 3 hold one block per wave");
        unsigned char* const mine = lds[2 + wave / 2][wave % 2];
        const uintptr_t at = row0 * T::ROWB;
        stage_cols<D>(rows_desc<D>((uintptr_t)a.dO + at, n_cols), lane, lds_addr(mine));
        constexpr int NR = kTileRows / T::RPI;
        const int off = (int)dma_lane_off<D, true>(0, lane);
        u32x4 ov[NR], lv[NR];
        {
            const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<bf16*>(static_cast<const bf16*>(a.O) + row0 * D), 0, n_cols * T::ROWB, 0x00020000);
            const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<bf16*>(static_cast<const bf16*>(a.O_lo ? a.O_lo : a.O) + row0 * D), 0,
                a.O_lo ? n_cols * T::ROWB : 0, 0x00020000);
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                ov[i] = __builtin_amdgcn_raw_buffer_load_b128(ro, off + i * 1024, 0, 2);  // nt: read once
                lv[i] = __builtin_amdgcn_raw_buffer_load_b128(rl, off + i * 1024, 0, 2);
            }
        }
        const float lse = lane < n_cols ? a.lse[row0 + lane] : 0.f;
        __builtin_amdgcn_sched_barrier(0);
        request(0, 0);
        request(1, 1);
        wait_vm_lgkm0<2 * NR + 1 + 2 * NIT>();  // dO landed
        u32x4 gv[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) gv[i] = *reinterpret_cast<const u32x4*>(mine + i * T::GRP + lane * 16);
        read_cols<D>(mine, lane, gf);
        wait_vm_lgkm0<2 * NR + 1 + 2 * NIT>();  // and is read
        stage_cols<D>(rows_desc<D>((uintptr_t)a.Q + at, n_cols), lane, lds_addr(mine));
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            float dot = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dot = fmaf(bf16_lo(gv[i][e]), bf16_lo(ov[i][e]) + bf16_lo(lv[i][e]), dot);
                dot = fmaf(bf16_hi(gv[i][e]), bf16_hi(ov[i][e]) + bf16_hi(lv[i][e]), dot);
            }
            dot = row_lanes_sum<D>(dot);
            if (lane % (D / 8) == 0) dsh[wave][0][i * T::RPI + lane / (D / 8)] = dot;
        }
        if (lane < 32) dsh[wave][1][lane] = lse * -kLog2e;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        dcol = dsh[wave][0][c32];
        off0 = dsh[wave][1][c32];
        wait_vm_lgkm0<0>();  // Q landed
        if (lane < n_cols) a.Dv[row0 + lane] = -dcol;
        read_cols<D>(mine, lane, qf);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        // every wave's rows are read before further blocks overwrite them
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    static_assert(AHEAD == 3, "two blocks are requested above");
    request(2, 2);
    const Frags<D> fr(lane, true);

    floatx16 acc[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[db] = floatx16{};

    // block j landed (the AHEAD - 1 requested after it may be in flight); its
    // own request refills the stage of block j-1
    auto block_step = [&](auto ph_tag, int j) {
        constexpr int PH = decltype(ph_tag)::value;  // j mod NS: the stage as a constant
        bsync<(AHEAD - 1) * NIT>();
        request(j + AHEAD, (PH + AHEAD) % NS);
        if (!plan.needed(j)) return;
        const unsigned char* ks = lds[PH][0];
        const unsigned char* vs = lds[PH][1];
        constexpr int PF = kFragAhead;
        constexpr int N = 2 * NDC + NKC * NDB;  // fragments: K rows, V rows, K^T
        bf16x8 op[PF + 1];
        auto load = [&](int k) {
            op[k % (PF + 1)] = k < NDC       ? fr.row(ks, k)
                               : k < 2 * NDC ? fr.row(vs, k - NDC)
                                             : fr.tr(ks, (k - 2 * NDC) % NDB, (k - 2 * NDC) / NDB);
        };
#pragma unroll
        for (int k = 0; k < PF; ++k) load(k);
        floatx16 s, dp;
#pragma unroll
        for (int k = 0; k < NDC; ++k) {
            load(k + PF);
            s = mfma32_bf16(op[k % (PF + 1)], qf[k], k == 0 ? floatx16{} : s);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!plan.full(j)) plan.template mask<D>(s, j, p0, L, a.fW, a.fC, a.n_chunks);
        const float off = (j < plan.nsb ? a.log2C : 0.f) + off0;
#pragma unroll
        for (int k = 0; k < NDC; ++k) {
            load(k + NDC + PF);
            dp = mfma32_bf16(op[(k + NDC) % (PF + 1)], gf[k], k == 0 ? floatx16{} : dp);
#pragma unroll
            for (int i = k * 16 / NDC; i < (k + 1) * 16 / NDC; ++i)  // P^T (masked entries: 0)
                s[i] = fast_exp2(fmaf(s[i], a.scale_log2, off));
            __builtin_amdgcn_sched_barrier(0);
        }
        u32x4 ds[NKC];
        auto weights = [&](int kc, int e) {  // dS^T = P^T (dP^T - D)
            const int i = 8 * kc + 2 * e;
            ds[kc][e] = pack_bf16x2(s[i] * (dp[i] - dcol), s[i + 1] * (dp[i + 1] - dcol));
        };
#pragma unroll
        for (int e = 0; e < 4; ++e) weights(0, e);
#pragma unroll
        for (int k = 2 * NDC; k < N; ++k) {
            if (k + PF < N) load(k + PF);
            const int db = (k - 2 * NDC) % NDB, kc = (k - 2 * NDC) / NDB;
            acc[db] = mfma32_bf16(op[k % (PF + 1)], __builtin_bit_cast(bf16x8, ds[kc]), acc[db]);
            if (kc + 1 < NKC) {
#pragma unroll
                for (int e = db * 4 / NDB; e < (db + 1) * 4 / NDB; ++e) weights(kc + 1, e);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // NS steps per trip, so that each one's stage index is a constant
    int j = 0;
    for (; j + NS - 1 < nb; j += NS) {
        block_step(std::integral_constant<int, 0>{}, j);
        block_step(std::integral_constant<int, 1>{}, j + 1);
        if constexpr (NS > 2) block_step(std::integral_constant<int, 2 % NS>{}, j + 2);
        if constexpr (NS > 3) block_step(std::integral_constant<int, 3 % NS>{}, j + 3);
    }
    if (j < nb) block_step(std::integral_constant<int, 0>{}, j);
    if (NS > 2 && j + 1 < nb) block_step(std::integral_constant<int, 1>{}, j + 1);
    if (NS > 3 && j + 2 < nb) block_step(std::integral_constant<int, 2 % NS>{}, j + 2);

    wait_vm_lgkm0<0>();  // no request may still be writing LDS when the workgroup ends
    __builtin_amdgcn_s_barrier();  // every wave is done with the ring: it holds the staged rows now
    static_assert(kTileWaves * 32 * kStageRow<D> <= NS * 2 * BLK, "staged rows fit in the ring");
    const float inv_sqrt_d = a.scale_log2 / kLog2e;
    store_tile_rows<D>(&lds[0][0][0] + wave * 32 * kStageRow<D>, lane,
                       static_cast<bf16*>(a.dQ) + row0 * D, L - p0, [&](int db, int i) {
                           return pack_bf16x2(acc[db][i] * inv_sqrt_d, acc[db][i + 1] * inv_sqrt_d);
                       });
}

// ---------------------------------------------------------------------------
// dK, dV of window keys and of summaries
// ---------------------------------------------------------------------------
// Rows that see window key m: [kv_rows_lo(m), kv_rows_hi(m)] (the inverse
// of [win_lo(n), win_hi(n)], both non-decreasing); rows that see summary c
// from the prefix side: n >= sum_rows_lo(c) (win_lo(n) >= (c + 1) C).
// Non-causal summaries are also seen by the rows of the blocks wholly before
// them: their tiles stream every row, masked per element.
template <int VAR, typename TW>
__device__ __forceinline__ int kv_rows_lo(int m, const TW& W) {
    return VAR == kWinNonCausal ? (m / W) * (int)W : m;
}
template <int VAR, typename TW, typename TC>
__device__ __forceinline__ long long kv_rows_hi(int m, const TW& W, const TC& C) {
    if constexpr (VAR == kWinSliding) return (long long)m + (int)W - 1;
    if constexpr (VAR == kWinChunkAligned) return ((long long)(m / C) + 1) * (int)C + (int)W - 2;
    return (long long)(m / W) * (int)W + (int)W - 1;
}
template <int VAR>
__device__ __forceinline__ long long sum_rows_lo(int c, int W, int C) {
    if constexpr (VAR == kWinSliding || VAR == kWinChunkAligned) return ((long long)c + 1) * C + W - 1;
    if constexpr (VAR == kWinBlocked) return (((long long)c + 1) * C + W - 1) / W * W;
    return 0;
}

template <int D, bool SUM, int VAR>
__global__ __launch_bounds__(kBwdWaves * 64) __attribute__((amdgpu_waves_per_eu(3, 3))) void bwd_dkdv_kernel(BwdParams a) {
    typedef BCfg<D> Cfg;
    constexpr int NDC = Cfg::NDC, NDB = Cfg::NDB, BLK = Cfg::BLK;
    constexpr int KT = kBwdWaves * 16;  // keys per workgroup
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kKvNS][2][BLK];  // [stage][Q, dO]
    __shared__ __attribute__((aligned(256))) float rowf[kKvNS][2][64];            // [stage][lse, D] of its rows
    __shared__ __attribute__((aligned(1024))) unsigned char dummy[1024];

    const int L = a.L, W = a.W, C = a.C;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c16 = lane & 15;
    // key tiles per (b, kv head): summaries, or window keys
    constexpr bool sum = SUM;
    // summary tiles: n_split workgroups per tile, each over a part of the
    // query range, leaving partial sums
    const int n_split = SUM ? a.n_split : 1;
    const int per_bg = (SUM ? (a.n_chunks + KT - 1) / KT : (L + KT - 1) / KT) * n_split;
    const int bgi = (int)blockIdx.x / per_bg;
    const int t = (int)blockIdx.x % per_bg / n_split;
    const int sp = (int)blockIdx.x % n_split;
    const size_t bg = (size_t)bgi;
    const int b = bgi / a.Hkv, kvh = bgi % a.Hkv;
    const int G = a.H / a.Hkv;
    const int k0 = t * KT;                        // first key (or summary) of the tile
    const int lim = sum ? a.n_chunks : L;
    const int key = k0 + wave * 16 + c16;         // this lane's key column
    const int key_c = min(key, lim - 1);

    // stationary key/value rows (B operands): features dc*32 + 8g .. +7 of key_c
    const bf16* Kr = static_cast<const bf16*>(sum ? a.Ks : a.K) + (bg * (size_t)lim + key_c) * D;
    const bf16* Vr = static_cast<const bf16*>(sum ? a.Vs : a.V) + (bg * (size_t)lim + key_c) * D;
    bf16x8 kf[NDC], vf[NDC];
#pragma unroll
    for (int dc = 0; dc < NDC; ++dc) {
        kf[dc] = *reinterpret_cast<const bf16x8*>(Kr + dc * 32 + g * 8);
        vf[dc] = *reinterpret_cast<const bf16x8*>(Vr + dc * 32 + g * 8);
    }

    // query rows that can see some key of the tile (and of this wave's keys
    // [wk0, wk1]): window key k is seen by rows [kv_rows_lo(k), kv_rows_hi(k)],
    // summary c by rows from sum_rows_lo(c) on (non-causal: by any row)
    constexpr bool NC = VAR == kWinNonCausal;
    const int k_last = min(k0 + KT, lim) - 1;
    const int r_lo = sum ? (int)min((long long)L, sum_rows_lo<VAR>(k0, W, C)) : kv_rows_lo<VAR>(k0, W);
    const int r_hi = sum ? L - 1 : (int)min((long long)L - 1, kv_rows_hi<VAR>(k_last, W, C));
    const int qb0 = r_lo / kBwdBN;
    const int nqb = r_lo <= r_hi ? r_hi / kBwdBN - qb0 + 1 : 0;
    const int wk0 = k0 + wave * 16, wk1 = min(wk0 + 15, lim - 1);
    const bool w_active = wk0 < lim;
    const int wr_lo = sum ? (int)min((long long)L, sum_rows_lo<VAR>(wk0, W, C)) : kv_rows_lo<VAR>(wk0, W);
    const int wr_hi = sum ? L - 1 : (int)min((long long)L - 1, kv_rows_hi<VAR>(wk1, W, C));

    floatx4 dk[NDB], dv[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) dk[db] = dv[db] = floatx4{0.f, 0.f, 0.f, 0.f};
    const float bias = sum ? a.log2C : 0.f;

    const Stager<D> stg(wave, lane);
    // (head, query block) pairs [j0, j0 + steps) of the nqb * G the tile sees
    const int all_steps = nqb * G;
    const int j0 = (int)((long long)all_steps * sp / n_split);
    const int steps = (int)((long long)all_steps * (sp + 1) / n_split) - j0;
    // request of step j: its Q and dO rows (stage j % NS), and their lse and D
    // (one 4-B DMA instruction each, by waves 0 and 1; waves 2 and 3 issue one
    // into the dummy area so that every wave counts the same instructions)
    constexpr int REQ = 2 * Cfg::NI + 1;
    static_assert(kKvNS == 3, "the step loop below takes three steps per trip");
    auto stage = [&](int j) {
        const bool real = j < steps;
        // past the last step: row 0 of the group's first head (always valid)
        const int hh = real ? (j0 + j) / nqb : 0, qb = real ? qb0 + (j0 + j) % nqb : 0;
        const size_t rowh = ((size_t)b * a.H + kvh * G + hh) * L;
        const size_t rowb = rowh + (size_t)qb * kBwdBN;
        const int nv = min(kBwdBN, L - qb * kBwdBN);
        const int st_i = j % kKvNS;
        stg.issue(static_cast<const bf16*>(a.Q) + rowb * D, nv, lds_addr_of<D>(real ? lds[st_i][0] : dummy), wave, real);
        stg.issue(static_cast<const bf16*>(a.dO) + rowb * D, nv, lds_addr_of<D>(real ? lds[st_i][1] : dummy), wave,
                  real);
        const bool mine = real && wave < 2;
        const float* src = wave == 1 ? a.Dv : a.lse;
        const unsigned voff = (unsigned)(mine ? min(lane, nv - 1) : 0) * 4u;
        const unsigned dst = mine ? lds_addr_of<D>(rowf[st_i][wave]) : lds_addr_of<D>(dummy);
        asm volatile("global_load_lds_dword %0, %1" ::"v"(voff), "s"(src + rowb),
                     "{m0}"(__builtin_amdgcn_readfirstlane(dst))
                     : "memory");
    };
#pragma unroll
    for (int k = 0; k < kKvAhead; ++k) stage(k);
    // see bwd_dq_kernel: the stationary fragments are waited for here
    bwait_vm<0>();
    auto block_step = [&](auto ph_tag, int j) {
        constexpr int PH = decltype(ph_tag)::value;  // j mod NS: the stage as a constant
        // step j's rows landed (the request after it may be in flight); the
        // request below refills the stage of step j-1
        bsync<(kKvAhead - 1) * REQ>();
        stage(j + kKvAhead);
        const int qb = qb0 + (j0 + j) % nqb;
        const int r0 = qb * kBwdBN;
        if (!w_active || r0 > wr_hi || r0 + kBwdBN - 1 < wr_lo) return;
        constexpr int st_i = PH;
        // lse and D of this lane's 8 query rows r0 + 16 kb + 4g + i
        float lse2[2][4], dq[2][4];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const floatx4 l4 = *reinterpret_cast<const floatx4*>(&rowf[st_i][0][kb * 16 + g * 4]);
            const floatx4 d4 = *reinterpret_cast<const floatx4*>(&rowf[st_i][1][kb * 16 + g * 4]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                lse2[kb][i] = l4[i] * kLog2e;
                dq[kb][i] = -d4[i];
            }
        }
        const unsigned char* qs = lds[st_i][0];
        const unsigned char* gs = lds[st_i][1];
        // S and dP: rows = queries r0 + kb*16 + 4g + i, column = key c16
        floatx4 s[2], dp[2];
        s[0] = s[1] = dp[0] = dp[1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dc = 0; dc < NDC; ++dc)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                s[kb] = mfma_bf16(row_frag<D>(qs, kb, dc, c16, g), kf[dc], s[kb]);
                dp[kb] = mfma_bf16(row_frag<D>(gs, kb, dc, c16, g), vf[dc], dp[kb]);
            }
        floatx4 p[2];
        // a step every pair of which is visible (the wave's 16 keys, the
        // block's 32 rows: most window steps) skips the per-element test
        const int r1 = r0 + kBwdBN - 1;
        const bool full = wk0 + 15 < lim && r1 < L &&
                          (sum ? wk0 + 16 <= sum_lo<VAR>(r0, W, C) ||
                                     (NC && wk0 >= sum_hi<VAR>(r1, W, C, L))
                               : win_lo<VAR>(r1, W, C) <= wk0 && wk0 + 15 <= win_hi<VAR>(r0, W, L));
        if (full) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    p[kb][i] = fast_exp2(fmaf(s[kb][i], a.scale_log2, bias - lse2[kb][i]));
                    s[kb][i] = p[kb][i] * (dp[kb][i] - dq[kb][i]);  // dS
                }
        } else {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int n = r0 + kb * 16 + g * 4 + i;
                    const int nc = min(n, L - 1);
                    const bool ok = key < lim && n < L &&
                                    (sum ? key < sum_lo<VAR>(nc, W, C) || (NC && key >= sum_hi<VAR>(nc, W, C, L))
                                         : win_lo<VAR>(nc, W, C) <= key && key <= win_hi<VAR>(nc, W, L));
                    p[kb][i] = ok ? fast_exp2(fmaf(s[kb][i], a.scale_log2, bias - lse2[kb][i])) : 0.f;
                    s[kb][i] = p[kb][i] * (dp[kb][i] - dq[kb][i]);  // dS
                }
        }
        const bf16x8 pf = pair_to_b(p[0], p[1]);
        const bf16x8 dsf = pair_to_b(s[0], s[1]);
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            dv[db] = mfma_bf16(tr_frag<D>(gs, db, c16, g), pf, dv[db]);
            dk[db] = mfma_bf16(tr_frag<D>(qs, db, c16, g), dsf, dk[db]);
        }
    };
    // three steps per trip, so that each one's stage index is a constant
    typedef std::integral_constant<int, 0> P0;
    typedef std::integral_constant<int, 1> P1;
    typedef std::integral_constant<int, 2> P2;
    int j = 0;
    for (; j + 2 < steps; j += 3) {
        block_step(P0{}, j);
        block_step(P1{}, j + 1);
        block_step(P2{}, j + 2);
    }
    if (j < steps) block_step(P0{}, j);
    if (j + 1 < steps) block_step(P1{}, j + 1);

    bwait_vm<0>();  // no request may still be writing LDS when the workgroup ends
    if (key >= lim) return;
    const float inv_sqrt_d = a.scale_log2 / kLog2e;
    if constexpr (SUM) {
        // fp32 partial summary gradients, for the per-chunk pass
        const size_t slot = (size_t)sp * a.B * a.Hkv * lim;
        float* dKo = a.dKs_w + (slot + bg * (size_t)lim + key) * D;
        float* dVo = a.dVs_w + (slot + bg * (size_t)lim + key) * D;
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            *reinterpret_cast<floatx4*>(dKo + db * 16 + g * 4) = dk[db] * inv_sqrt_d;
            *reinterpret_cast<floatx4*>(dVo + db * 16 + g * 4) = dv[db];
        }
    } else {
        // window gradient plus the key's share of its chunk's summary gradient
        // (keys after the last complete chunk have none)
        const int c = key / C;
        const bool in_chunk = c < a.n_chunks;
        float da = 0.f, bj = 0.f;
        const size_t cv = (bg * (size_t)a.n_chunks + (in_chunk ? c : 0)) * D;
        if (in_chunk) {
            da = a.da_w[bg * (size_t)a.n_chunks * C + key] * inv_sqrt_d;
            bj = a.bw_w[bg * (size_t)a.n_chunks * C + key];
        }
        bf16* dKo = static_cast<bf16*>(a.dK) + (bg * (size_t)L + key) * D;
        bf16* dVo = static_cast<bf16*>(a.dV) + (bg * (size_t)L + key) * D;
        const float inv_c = 1.f / (float)C;
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            floatx4 gk = dk[db] * inv_sqrt_d, gv = dv[db];
            if (in_chunk) {
                const int f = db * 16 + g * 4;
                const floatx4 kh = *reinterpret_cast<const floatx4*>(a.khat_w + cv + f);
                const floatx4 dkh = *reinterpret_cast<const floatx4*>(a.dkhat_w + cv + f);
                const floatx4 dvh = *reinterpret_cast<const floatx4*>(a.dVs_w + cv + f);
                gk += da * kh + dkh * inv_c;
                gv += bj * dvh;
            }
            const u32x2 wk = {pack_bf16x2(gk[0], gk[1]), pack_bf16x2(gk[2], gk[3])};
            const u32x2 wv = {pack_bf16x2(gv[0], gv[1]), pack_bf16x2(gv[2], gv[3])};
            *reinterpret_cast<u32x2*>(dKo + db * 16 + g * 4) = wk;
            *reinterpret_cast<u32x2*>(dVo + db * 16 + g * 4) = wv;
        }
    }
}

// Window keys: a wave owns 32 keys (its K and V rows as B operands in
// registers, dK^T and dV^T as accumulators) and the query blocks of every head
// of the group that sees one of the workgroup's 128 keys stream through LDS.
// Per block: S = Q K^T; dP = dO V^T - D (the row dots are the product's
// initial value) with the exponentials of S between its products; dV^T +=
// dO^T P with dS = P dP between; dK^T += Q^T dS.
template <int D, int NS, int WPE, int VAR>
__global__ __launch_bounds__(kTileWaves * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void bwd_window_kernel(BwdParams a) {
    typedef Tile<D> T;
    constexpr int BLK = T::BLK, NKC = T::NKC, NDC = T::NDC, NDB = T::NDB;
    constexpr int NIT = 2 * T::NI + 1;  // requests per wave and block
    constexpr int AHEAD = NS - 1;       // blocks requested ahead of the one computed
    constexpr int KT = kTileWaves * 32; // keys per workgroup
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NS][2][BLK];  // [stage][Q, dO]
    __shared__ __attribute__((aligned(256))) float rowf[NS][2][64];           // [stage][lse, -D], by product row
    __shared__ __attribute__((aligned(256))) float sink[64];

    const int L = a.L;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c32 = lane & 31, h2 = lane >> 5;
    // consecutive key tiles of one (b, kv head), which share query rows, on one XCD
    const int n_kt = (L + KT - 1) / KT;
    int id = blockIdx.x;
    {
        const int per = (int)gridDim.x / 8;
        if (id < per * 8) id = (id % 8) * per + id / 8;
    }
    const int bgi = id / n_kt;
    const int k0 = (id - bgi * n_kt) * KT;  // first key of the tile
    const size_t bg = (size_t)bgi;
    const int b = bgi / a.fHkv, kvh = bgi - b * a.Hkv;
    const int G = a.t.G;
    const int wk0 = k0 + wave * 32;         // the wave's keys wk0 .. wk1
    const int wk1 = min(wk0 + 31, L - 1);
    const int n_keys = max(0, min(32, L - wk0));

    // ---- query rows that see some key of the tile, some key of the wave, and
    // all of the wave's keys: key m is seen by [kv_rows_lo(m), kv_rows_hi(m)]
    auto rows_hi = [&](int m) { return (int)min((long long)L - 1, kv_rows_hi<VAR>(m, a.fW, a.fC)); };
    const int qb0 = kv_rows_lo<VAR>(k0, a.fW) / kTileRows;
    const int nqb = rows_hi(min(k0 + KT, L) - 1) / kTileRows - qb0 + 1;
    const bool w_active = wk0 < L;
    const int wb0 = kv_rows_lo<VAR>(min(wk0, L - 1), a.fW) / kTileRows;       // needed query blocks wb0 .. +wbc-1
    const unsigned wbc = w_active ? rows_hi(wk1) / kTileRows - wb0 + 1 : 0;
    const int full_lo = kv_rows_lo<VAR>(wk1, a.fW);
    const int full_hi = rows_hi(min(wk0, L - 1));
    const int steps = nqb * G;

    // ---- requests: step (head, query block) in that order.  Q and dO rows by
    // all waves; lse and -D by waves 0 and 1, 4 bytes per lane, into the order
    // of the product's rows (waves 2 and 3 issue one without rows into the
    // sink, so that every wave counts the same instructions).
    const unsigned lane_off = dma_lane_off<D, true>(wave, lane);
    const unsigned lds0 = lds_addr(lds) + wave * T::GRP;
    const unsigned row_off =
        lane < 32 ? 4 * (T::key_of(lane >> 3, lane & 3) + ((lane >> 2) & 1) * T::KH) : 0x40000000u;
    int rq_h = 0, rq_b = 0;  // next request's head and block of the range
    const size_t head0 = (size_t)b * a.H + (size_t)kvh * G;
    auto request = [&](int stage) {
        const bool real = rq_h < G;
        const int r0 = (qb0 + rq_b) * kTileRows;
        const int rows = real ? min(L - r0, kTileRows) : 0;
        const size_t row = (head0 + (real ? rq_h : 0)) * L + r0;
        dma_block<D>(rows_desc<D>((uintptr_t)a.Q + row * T::ROWB, rows), lane_off, lds0 + stage * 2 * BLK);
        dma_block<D>(rows_desc<D>((uintptr_t)a.dO + row * T::ROWB, rows), lane_off, lds0 + stage * 2 * BLK + BLK);
        const uintptr_t f = (uintptr_t)(wave == 1 ? a.Dv : a.lse) + row * 4;
        const u32x4 d = {(uint32_t)f, (uint32_t)(f >> 32) & 0xffffu, (uint32_t)(wave < 2 ? rows * 4 : 0), 0x00020000u};
        dma4(d, row_off, wave < 2 ? lds_addr(rowf[stage][wave]) : lds_addr(sink));
        if (++rq_b == nqb) {
            rq_b = 0;
            ++rq_h;
        }
    };

    // ---- the wave's K rows, then its V rows, through one block per wave in
    // stages 2 and 3 of the ring, the first two query blocks beside them
    bf16x8 kf[NDC], vf[NDC];
    {
        static_assert(NS == 4 && AHEAD == 3, "stages 2 and 3 hold one block per wave");
        unsigned char* const mine = lds[2 + wave / 2][wave % 2];
        const uintptr_t at = (bg * (size_t)L + wk0) * T::ROWB;
        stage_cols<D>(rows_desc<D>((uintptr_t)a.K + at, n_keys), lane, lds_addr(mine));
        request(0);
        request(1);
        wait_vm_lgkm0<2 * NIT>();
        read_cols<D>(mine, lane, kf);
        wait_vm_lgkm0<2 * NIT>();
        stage_cols<D>(rows_desc<D>((uintptr_t)a.V + at, n_keys), lane, lds_addr(mine));
        wait_vm_lgkm0<0>();
        read_cols<D>(mine, lane, vf);
        wait_vm_lgkm0<0>();
        __builtin_amdgcn_s_barrier();  // every wave's rows are read before further blocks overwrite them
        asm volatile("" ::: "memory");
    }
    request(2);

    const Frags<D> fr(lane, true);
    floatx16 dk[NDB], dv[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) dk[db] = dv[db] = floatx16{};

    int cur = 0;  // this step's block of the range
    auto block_step = [&](auto ph_tag) {
        constexpr int PH = decltype(ph_tag)::value;  // step mod NS: the stage as a constant
        bsync<(AHEAD - 1) * NIT>();
        request((PH + AHEAD) % NS);
        const int qb = qb0 + cur;
        if (++cur == nqb) cur = 0;
        if ((unsigned)(qb - wb0) >= wbc) return;
        const unsigned char* qs = lds[PH][0];
        const unsigned char* gs = lds[PH][1];
        constexpr int PF = kKvPF;
        constexpr int N = 2 * NDC + 2 * NKC * NDB;  // fragments: Q rows, dO rows, dO^T, Q^T
        bf16x8 op[PF + 1];
        auto load = [&](int k) {
            const int kt = (k - 2 * NDC) % (NKC * NDB);
            op[k % (PF + 1)] = k < NDC                     ? fr.row(qs, k)
                               : k < 2 * NDC               ? fr.row(gs, k - NDC)
                               : k < 2 * NDC + NKC * NDB ? fr.tr(gs, kt % NDB, kt / NDB)
                                                           : fr.tr(qs, kt % NDB, kt / NDB);
        };
        // lse or -D of product rows 8 q + 4 h2 ..
        auto rows4 = [&](int arr, int q) {
            return *reinterpret_cast<const floatx4*>(&rowf[PH][arr][8 * q + 4 * h2]);
        };
#pragma unroll
        for (int k = 0; k < PF; ++k) load(k);
        floatx16 s, dp;
#pragma unroll
        for (int k = 0; k < NDC; ++k) {
            load(k + PF);
            s = mfma32_bf16(op[k % (PF + 1)], kf[k], k == 0 ? floatx16{} : s);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const floatx4 d4 = rows4(1, q);
#pragma unroll
            for (int i = 0; i < 4; ++i) dp[4 * q + i] = d4[i];
        }
        const int r0 = qb * kTileRows;
        if (r0 < full_lo || r0 + kTileRows - 1 > full_hi) {
            const int l = lane_here();
            const int m = min(wk0 + (l & 31), L - 1), rel = r0 + (l >> 5) * T::KH;
            if (r0 + kTileRows - 1 > full_hi) mask_above<D>(s, rows_hi(m) - rel);
            if (r0 < full_lo) mask_below<D>(s, kv_rows_lo<VAR>(m, a.fW) - rel);
        }
        floatx4 l4 = rows4(0, 0);
#pragma unroll
        for (int k = 0; k < NDC; ++k) {
            load(k + NDC + PF);
            dp = mfma32_bf16(op[(k + NDC) % (PF + 1)], vf[k], dp);
#pragma unroll
            for (int i = k * 16 / NDC; i < (k + 1) * 16 / NDC; ++i) {
                s[i] = fast_exp2(fmaf(s[i], a.scale_log2, l4[i % 4] * -kLog2e));  // P (masked entries: 0)
                if (i % 4 == 3 && i < 15) l4 = rows4(0, i / 4 + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        u32x4 pf[NKC], ds[NKC];
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc)
#pragma unroll
            for (int e = 0; e < 4; ++e) pf[kc][e] = pack_bf16x2(s[8 * kc + 2 * e], s[8 * kc + 2 * e + 1]);
#pragma unroll
        for (int k = 2 * NDC; k < N; ++k) {
            if (k + PF < N) load(k + PF);
            const int kv = k - 2 * NDC, kt = kv % (NKC * NDB), db = kt % NDB, kc = kt / NDB;
            if (kv < NKC * NDB) {
                dv[db] = mfma32_bf16(op[k % (PF + 1)], __builtin_bit_cast(bf16x8, pf[kc]), dv[db]);
#pragma unroll
                for (int w = kv * 8 / (NKC * NDB); w < (kv + 1) * 8 / (NKC * NDB); ++w)  // dS
                    ds[w / 4][w % 4] = pack_bf16x2(s[2 * w] * dp[2 * w], s[2 * w + 1] * dp[2 * w + 1]);
            } else {
                dk[db] = mfma32_bf16(op[k % (PF + 1)], __builtin_bit_cast(bf16x8, ds[kc]), dk[db]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // four steps per trip, so that each one's stage index is a constant
    typedef std::integral_constant<int, 0> P0;
    typedef std::integral_constant<int, 1> P1;
    typedef std::integral_constant<int, 2> P2;
    typedef std::integral_constant<int, 3> P3;
    int j = 0;
    for (; j + 3 < steps; j += 4) {
        block_step(P0{});
        block_step(P1{});
        block_step(P2{});
        block_step(P3{});
    }
    if (j < steps) block_step(P0{});
    if (j + 1 < steps) block_step(P1{});
    if (j + 2 < steps) block_step(P2{});

    wait_vm_lgkm0<0>();  // no request may still be writing LDS when the workgroup ends
    __builtin_amdgcn_s_barrier();  // every wave is done with the ring: it holds the staged rows now

    // ---- the window gradient plus the key's share of its chunk's summary
    // gradient (keys after the last complete chunk have none), on whole rows:
    // the accumulators go through LDS in fp32, so that the chunk's vectors are
    // read, and the rows written, D / 8 neighbouring lanes to a row
    constexpr int SROW = 4 * D + 16;  // bytes per staged row; fragment writes fall in distinct banks
    constexpr int LPR = D / 8, RPS = 64 / LPR;
    static_assert(kTileWaves * 32 * SROW <= NS * 2 * BLK, "staged rows fit in the ring");
    unsigned char* const stg = &lds[0][0][0] + wave * 32 * SROW;
    const float inv_sqrt_d = a.scale_log2 / kLog2e, inv_c = 1.f / (float)a.C;
    const int row = lane / LPR, f0 = lane % LPR * 8;
    // the chunks of the wave's 32 keys start at c0; vectors of chunks past the
    // last complete one, and the factors of keys past it, read as zeros
    const int c0 = min(wk0, L - 1) / a.fC;
    const int n_c = max(0, min(a.n_chunks - c0, 33)), n_f = max(0, min(a.n_chunks * a.C - wk0, 32));
    auto vec_rsrc = [&](const float* w) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w + (bg * (size_t)a.n_chunks + c0) * D), 0,
                                                 n_c * D * 4, 0x00020000);
    };
    auto key_rsrc = [&](const float* w) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w + bg * (size_t)a.n_chunks * a.C + wk0), 0,
                                                 n_f * 4, 0x00020000);
    };
    auto load4 = [&](__amdgpu_buffer_rsrc_t r, int off) {
        return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    };
    auto load1 = [&](__amdgpu_buffer_rsrc_t r, int off) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    };
    // row r's byte offset into the chunk vectors
    auto vec_off = [&](int r) { return ((min(wk0 + r, L - 1) / a.fC - c0) * D + f0) * 4; };
    auto stage_acc = [&](const floatx16 (&acc)[NDB]) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<floatx4*>(stg + c32 * SROW + (db * 32 + 8 * q + 4 * h2) * 4) =
                    floatx4{acc[db][4 * q], acc[db][4 * q + 1], acc[db][4 * q + 2], acc[db][4 * q + 3]};
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // rows r = i RPS + row in batches of NBAT, whose vectors are all in flight
    // together (those of the first batch behind the staging)
    constexpr int NROW = 32 / RPS, NBAT = NROW < 4 ? NROW : 4;
    auto store_row = [&](bf16* out, int r, const floatx4& v0, const floatx4& v1) {
        const u32x4 w = {pack_bf16x2(v0[0], v0[1]), pack_bf16x2(v0[2], v0[3]), pack_bf16x2(v1[0], v1[1]),
                         pack_bf16x2(v1[2], v1[3])};
        if (wk0 + r < L)
            __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(out + (bg * (size_t)L + wk0 + r) * D + f0));
    };
    auto staged = [&](int r, int x) { return *reinterpret_cast<const floatx4*>(stg + r * SROW + f0 * 4 + 16 * x); };
    {
        const __amdgpu_buffer_rsrc_t rk = vec_rsrc(a.khat_w), rd = vec_rsrc(a.dkhat_w), ra = key_rsrc(a.da_w);
        floatx4 kh[NBAT][2], dkh[NBAT][2];
        float da[NBAT];
        auto fetch = [&](int i0) {
#pragma unroll
            for (int i = 0; i < NBAT; ++i) {
                const int r = (i0 + i) * RPS + row, off = vec_off(r);
                da[i] = load1(ra, r * 4);
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    kh[i][x] = load4(rk, off + 16 * x);
                    dkh[i][x] = load4(rd, off + 16 * x);
                }
            }
        };
        fetch(0);
        stage_acc(dk);
#pragma unroll
        for (int i0 = 0; i0 < NROW; i0 += NBAT) {
            if (i0) fetch(i0);
#pragma unroll
            for (int i = 0; i < NBAT; ++i) {
                const int r = (i0 + i) * RPS + row;
                const float d = da[i] * inv_sqrt_d;
                store_row(static_cast<bf16*>(a.dK), r, staged(r, 0) * inv_sqrt_d + (d * kh[i][0] + dkh[i][0] * inv_c),
                          staged(r, 1) * inv_sqrt_d + (d * kh[i][1] + dkh[i][1] * inv_c));
            }
        }
    }
    {
        const __amdgpu_buffer_rsrc_t rv = vec_rsrc(a.dVs_w), rb = key_rsrc(a.bw_w);
        floatx4 dvh[NROW][2];
        float bj[NROW];
#pragma unroll
        for (int i = 0; i < NROW; ++i) {
            const int r = i * RPS + row, off = vec_off(r);
            bj[i] = load1(rb, r * 4);
#pragma unroll
            for (int x = 0; x < 2; ++x) dvh[i][x] = load4(rv, off + 16 * x);
        }
        // every lane's reads of the staged dK are done
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        stage_acc(dv);
#pragma unroll
        for (int i = 0; i < NROW; ++i) {
            const int r = i * RPS + row;
            store_row(static_cast<bf16*>(a.dV), r, staged(r, 0) + bj[i] * dvh[i][0], staged(r, 1) + bj[i] * dvh[i][1]);
        }
    }
}

// ---------------------------------------------------------------------------
// through the summaries, plus the window gradients, to dK and dV
// ---------------------------------------------------------------------------
// One 256-thread workgroup per chunk.  Thread t holds features cc*8 ..
// cc*8+7 (cc = t % TPR) of rows r0, r0 + RPS, ... (r0 = t / TPR).  LDS: a_j
// (log2 units), C floats, the reduction scratch, then the chunk's summary
// gradients (2 D floats).
template <int D>
__global__ __launch_bounds__(256) void bwd_summary_kernel(BwdParams a) {
    constexpr int TPR = D / 8;
    constexpr int RPS = 256 / TPR;
    extern __shared__ float smem[];
    float* logit = smem;
    float* red = smem + a.C;
    const int chunk = blockIdx.x;
    const size_t bg = blockIdx.y;
    const int L = a.L, C = a.C;
    const int t = threadIdx.x, cc = t % TPR, r0 = t / TPR;
    const int first = chunk * C;
    const bf16* K = static_cast<const bf16*>(a.K) + (bg * (size_t)L + first) * D;
    const bf16* V = static_cast<const bf16*>(a.V) + (bg * (size_t)L + first) * D;
    auto load8 = [&](const bf16* base, int r, float out[8]) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(base + (size_t)r * D + cc * 8);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = bf16_lo(w[i]);
            out[2 * i + 1] = bf16_hi(w[i]);
        }
    };
    auto row_sum = [&](float x) {
#pragma unroll
        for (int off = 1; off < TPR; off <<= 1) x += __shfl_xor(x, off, 64);
        return x;
    };
    const float sc = a.scale_log2;  // log2(e) / sqrt(d): logits in log2 units
    const float inv_sqrt_d = sc / kLog2e;
    const size_t cv = (bg * (size_t)a.n_chunks + chunk) * D + cc * 8;  // this thread's features of the chunk
    const size_t kv = bg * (size_t)a.n_chunks * C + first;             // the chunk's first key
    float kh[8] = {0, 0, 0, 0, 0, 0, 0, 0}, gvh[8], dkh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    // summary gradients: sums of the partials of the query-range splits,
    // formed once per feature (threads t < 2 D / 4: four features of dK^ or
    // dV^ each) and shared through LDS
    float* gsh = smem + ((a.C + summary_red_floats<D>() + 3) & ~3);  // [dK^ | dV^], 2 D floats, 16-B aligned
    if (t < 2 * D / 4) {
        const float* src = (t < D / 4 ? a.dKs_w : a.dVs_w) + (bg * (size_t)a.n_chunks + chunk) * D + (t % (D / 4)) * 4;
        const size_t slot = (size_t)a.B * a.Hkv * a.n_chunks * D;
        floatx4 acc4 = *reinterpret_cast<const floatx4*>(src);
        // unrolled to the maximum split count so that the loads are in flight together
#pragma unroll
        for (int sp = 1; sp < kMaxBwdSplits; ++sp)
            if (sp < a.n_split) acc4 += *reinterpret_cast<const floatx4*>(src + sp * slot);
        *reinterpret_cast<floatx4*>(gsh + t * 4) = acc4;
    }
    __syncthreads();
    float gkh[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        gkh[i] = gsh[cc * 8 + i];
        gvh[i] = gsh[D + cc * 8 + i];
    }
    // khat = mean key
    for (int r = r0; r < C; r += RPS) {
        float k[8];
        load8(K, r, k);
#pragma unroll
        for (int i = 0; i < 8; ++i) kh[i] += k[i];
    }
    reduce_rows8<TPR>(kh, red);
#pragma unroll
    for (int i = 0; i < 8; ++i) kh[i] *= 1.f / (float)C;
    // a_j and their max
    float mx = -INFINITY;
    for (int r = r0; r < C; r += RPS) {
        float k[8];
        load8(K, r, k);
        float x = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) x += kh[i] * k[i];
        x = row_sum(x) * sc;
        if (cc == 0) logit[r] = x;
        mx = fmaxf(mx, x);
    }
    const float amax = block_max(mx, red);  // also orders the logit writes before the reads
    // vhat = sum_j b_j v_j (unnormalized) and the denominator
    float vh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float psum = 0.f;
    for (int r = r0; r < C; r += RPS) {
        float v[8];
        load8(V, r, v);
        const float p = fast_exp2(logit[r] - amax);
        psum += p;
#pragma unroll
        for (int i = 0; i < 8; ++i) vh[i] += p * v[i];
    }
#pragma unroll
    for (int off = TPR; off < 64; off <<= 1) psum += __shfl_xor(psum, off, 64);
    if ((t & 63) == 0) red[5 * TPR * 8 + (t >> 6)] = psum;
    __syncthreads();
    const float inv_den = 1.f / (red[5 * TPR * 8] + red[5 * TPR * 8 + 1] + red[5 * TPR * 8 + 2] + red[5 * TPR * 8 + 3]);
    __syncthreads();
    reduce_rows8<TPR>(vh, red);
    // dvhat . vhat
    float x = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) x += gvh[i] * vh[i] * inv_den;
    const float gvv = row_sum(x);
    // b_j and da_j = b_j (dvhat . v_j - dvhat . vhat); dkhat = dK^_c + sum_j da_j k_j / sqrt(d)
    for (int r = r0; r < C; r += RPS) {
        float v[8], k[8];
        load8(V, r, v);
        load8(K, r, k);
        float y = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) y += gvh[i] * v[i];
        y = row_sum(y);
        const float bj = fast_exp2(logit[r] - amax) * inv_den;
        const float da = bj * (y - gvv);
        if (cc == 0) {
            a.da_w[kv + r] = da;
            a.bw_w[kv + r] = bj;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) dkh[i] += da * k[i];
    }
    reduce_rows8<TPR>(dkh, red);  // its barriers also order every thread's reads of slot 0 before the write
    if (t < TPR) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            a.khat_w[cv + i] = kh[i];
            a.dkhat_w[cv + i] = gkh[i] + dkh[i] * inv_sqrt_d;
            a.dVs_w[cv + i] = gvh[i];  // the total dvhat, for the window tiles
        }
    }
}

// Register-resident variant for chunks of exactly ROWS * RPS rows: every
// thread loads its key and value rows once, and the passes over the chunk
// run on registers (one memory latency per chunk instead of one per pass).
template <int D, int ROWS>
__global__ __launch_bounds__(256) void bwd_summary_kernel_reg(BwdParams a) {
    constexpr int TPR = D / 8;
    constexpr int RPS = 256 / TPR;
    constexpr int C = ROWS * RPS;
    __shared__ float red[summary_red_floats<D>()];
    __shared__ __attribute__((aligned(16))) float gsh[2 * D];  // [dK^ | dV^] of the chunk
    const int chunk = blockIdx.x;
    const size_t bg = blockIdx.y;
    const int L = a.L;
    const int t = threadIdx.x, cc = t % TPR, r0 = t / TPR;
    const int first = chunk * C;
    const bf16* K = static_cast<const bf16*>(a.K) + (bg * (size_t)L + first + r0) * D + cc * 8;
    const bf16* V = static_cast<const bf16*>(a.V) + (bg * (size_t)L + first + r0) * D + cc * 8;
    // read once: non-temporal loads (measured 183 -> 168 us on the LLM workload)
    u32x4 kw[ROWS], vw[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        kw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(K + (size_t)i * RPS * D));
        vw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(V + (size_t)i * RPS * D));
    }
    auto unpack = [&](const u32x4& w, float out[8]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            out[2 * e] = bf16_lo(w[e]);
            out[2 * e + 1] = bf16_hi(w[e]);
        }
    };
    auto row_sum = [&](float x) {
#pragma unroll
        for (int off = 1; off < TPR; off <<= 1) x += __shfl_xor(x, off, 64);
        return x;
    };
    const float sc = a.scale_log2;  // log2(e) / sqrt(d): logits in log2 units
    const float inv_sqrt_d = sc / kLog2e;
    // summary gradients: sums of the partials of the query-range splits
    if (t < 2 * D / 4) {
        const float* src = (t < D / 4 ? a.dKs_w : a.dVs_w) + (bg * (size_t)a.n_chunks + chunk) * D + (t % (D / 4)) * 4;
        const size_t slot = (size_t)a.B * a.Hkv * a.n_chunks * D;
        floatx4 acc4 = *reinterpret_cast<const floatx4*>(src);
#pragma unroll
        for (int sp = 1; sp < kMaxBwdSplits; ++sp)
            if (sp < a.n_split) acc4 += *reinterpret_cast<const floatx4*>(src + sp * slot);
        *reinterpret_cast<floatx4*>(gsh + t * 4) = acc4;
    }
    // khat = mean key
    float kh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        float k[8];
        unpack(kw[i], k);
#pragma unroll
        for (int e = 0; e < 8; ++e) kh[e] += k[e];
    }
    reduce_rows8<TPR>(kh, red);  // its barriers also publish gsh
#pragma unroll
    for (int e = 0; e < 8; ++e) kh[e] *= 1.f / (float)C;
    float gkh[8], gvh[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        gkh[e] = gsh[cc * 8 + e];
        gvh[e] = gsh[D + cc * 8 + e];
    }
    // logits (log2 units) and their max
    float sl[ROWS];
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        float k[8];
        unpack(kw[i], k);
        float x = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) x += kh[e] * k[e];
        sl[i] = row_sum(x) * sc;
        mx = fmaxf(mx, sl[i]);
    }
    const float amax = block_max(mx, red);
    // vhat = sum_j b_j v_j (unnormalized) and the denominator
    float vh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float psum = 0.f;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        float v[8];
        unpack(vw[i], v);
        sl[i] = fast_exp2(sl[i] - amax);
        psum += sl[i];
#pragma unroll
        for (int e = 0; e < 8; ++e) vh[e] += sl[i] * v[e];
    }
#pragma unroll
    for (int off = TPR; off < 64; off <<= 1) psum += __shfl_xor(psum, off, 64);
    if ((t & 63) == 0) red[5 * TPR * 8 + (t >> 6)] = psum;
    __syncthreads();
    const float inv_den = 1.f / (red[5 * TPR * 8] + red[5 * TPR * 8 + 1] + red[5 * TPR * 8 + 2] + red[5 * TPR * 8 + 3]);
    __syncthreads();
    reduce_rows8<TPR>(vh, red);
    // dvhat . vhat
    float x = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) x += gvh[e] * vh[e] * inv_den;
    const float gvv = row_sum(x);
    // b_j, da_j = b_j (dvhat . v_j - dvhat . vhat); dkhat = dK^_c + sum_j da_j k_j / sqrt(d)
    const size_t kv = bg * (size_t)a.n_chunks * C + first + r0;
    float dkh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        float v[8], k[8];
        unpack(vw[i], v);
        unpack(kw[i], k);
        float y = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) y += gvh[e] * v[e];
        y = row_sum(y);
        const float bj = sl[i] * inv_den;
        const float da = bj * (y - gvv);
        if (cc == 0) {
            a.da_w[kv + (size_t)i * RPS] = da;
            a.bw_w[kv + (size_t)i * RPS] = bj;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) dkh[e] += da * k[e];
    }
    reduce_rows8<TPR>(dkh, red);
    if (t < TPR) {
        const size_t cv = (bg * (size_t)a.n_chunks + chunk) * D + cc * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            a.khat_w[cv + e] = kh[e];
            a.dkhat_w[cv + e] = gkh[e] + dkh[e] * inv_sqrt_d;
            a.dVs_w[cv + e] = gvh[e];  // the total dvhat, for the window tiles
        }
    }
}

// The same per-chunk pass with one wave per chunk: lane (r0, cc) holds
// features cc*8 .. cc*8+7 of rows r0, r0 + RPS, ... (RPS = 64 / (D / 8)), and
// every reduction is a cross-lane shuffle (no workgroup barrier), so many
// chunks' loads are in flight per CU.  The summary gradients are summed over
// the query-range splits by each lane for its own features.
template <int D, int ROWS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(ROWS >= 16 ? 2 : 1))) void bwd_summary_kernel_wave(BwdParams a) {
    constexpr int TPR = D / 8;
    constexpr int RPS = 64 / TPR;
    constexpr int C = ROWS * RPS;
    const int chunk = blockIdx.x;
    const size_t bg = blockIdx.y;
    const int L = a.L;
    const int t = threadIdx.x, cc = t % TPR, r0 = t / TPR;
    const int first = chunk * C;
    const bf16* K = static_cast<const bf16*>(a.K) + (bg * (size_t)L + first + r0) * D + cc * 8;
    const bf16* V = static_cast<const bf16*>(a.V) + (bg * (size_t)L + first + r0) * D + cc * 8;
    u32x4 kw[ROWS], vw[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        kw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(K + (size_t)i * RPS * D));
        vw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(V + (size_t)i * RPS * D));
    }
    // summary gradients of this lane's features: sums of the split partials
    // (at most kMaxBwdSplits); row group r0 loads splits r0, r0 + RPS, ...,
    // all in flight together, and the row groups' sums are added across lanes
    float gkh[8], gvh[8];
    {
        static_assert(kMaxBwdSplits % RPS == 0, "splits spread evenly over the row groups");
        const size_t off = (bg * (size_t)a.n_chunks + chunk) * D + cc * 8;
        const size_t slot = (size_t)a.B * a.Hkv * a.n_chunks * D;
        floatx4 k0 = {0.f, 0.f, 0.f, 0.f}, k1 = k0, v0 = k0, v1 = k0;
#pragma unroll
        for (int q = 0; q < kMaxBwdSplits / RPS; ++q) {
            const int sp = r0 + q * RPS;
            if (sp < a.n_split) {
                k0 += *reinterpret_cast<const floatx4*>(a.dKs_w + off + sp * slot);
                k1 += *reinterpret_cast<const floatx4*>(a.dKs_w + off + sp * slot + 4);
                v0 += *reinterpret_cast<const floatx4*>(a.dVs_w + off + sp * slot);
                v1 += *reinterpret_cast<const floatx4*>(a.dVs_w + off + sp * slot + 4);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            gkh[e] = k0[e];
            gkh[4 + e] = k1[e];
            gvh[e] = v0[e];
            gvh[4 + e] = v1[e];
        }
    }
    auto unpack = [](const u32x4& w, float out[8]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            out[2 * e] = bf16_lo(w[e]);
            out[2 * e + 1] = bf16_hi(w[e]);
        }
    };
    // over the lanes of one row (its TPR feature groups)
    auto row_sum = [](float x) {
#pragma unroll
        for (int off = 1; off < TPR; off <<= 1) x += __shfl_xor(x, off, 64);
        return x;
    };
    // over the lanes holding the same features (the row groups)
    auto rows_sum = [](float x) {
#pragma unroll
        for (int off = TPR; off < 64; off <<= 1) x += __shfl_xor(x, off, 64);
        return x;
    };
    const float sc = a.scale_log2;  // log2(e) / sqrt(d): logits in log2 units
    const float inv_sqrt_d = sc / kLog2e;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        gkh[e] = rows_sum(gkh[e]);
        gvh[e] = rows_sum(gvh[e]);
    }
    // khat = mean key
    float kh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        float k[8];
        unpack(kw[i], k);
#pragma unroll
        for (int e = 0; e < 8; ++e) kh[e] += k[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) kh[e] = rows_sum(kh[e]) * (1.f / (float)C);
    // logits (log2 units) and their max
    float sl[ROWS];
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        float k[8];
        unpack(kw[i], k);
        float x = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) x += kh[e] * k[e];
        sl[i] = row_sum(x) * sc;
        mx = fmaxf(mx, sl[i]);
    }
#pragma unroll
    for (int off = TPR; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    // vhat = sum_j b_j v_j (unnormalized), the denominator, and dvhat . v_j
    // (V is not needed after this loop)
    float vh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float psum = 0.f;
    float yv[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        float v[8];
        unpack(vw[i], v);
        sl[i] = fast_exp2(sl[i] - mx);
        psum += sl[i];
        float y = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            vh[e] += sl[i] * v[e];
            y += gvh[e] * v[e];
        }
        yv[i] = row_sum(y);
    }
    const float inv_den = 1.f / rows_sum(psum);
    // dvhat . vhat
    float x = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) x += gvh[e] * rows_sum(vh[e]) * inv_den;
    const float gvv = row_sum(x);
    // b_j, da_j = b_j (dvhat . v_j - dvhat . vhat); dkhat = dK^_c + sum_j da_j k_j / sqrt(d)
    const size_t kv = bg * (size_t)a.n_chunks * C + first + r0;
    float dkh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        float k[8];
        unpack(kw[i], k);
        const float bj = sl[i] * inv_den;
        const float da = bj * (yv[i] - gvv);
        if (cc == 0) {
            a.da_w[kv + (size_t)i * RPS] = da;
            a.bw_w[kv + (size_t)i * RPS] = bj;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) dkh[e] += da * k[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) dkh[e] = rows_sum(dkh[e]);
    if (r0 == 0) {
        // every lane has read the split partials (slot 0 included) above
        const size_t cv = (bg * (size_t)a.n_chunks + chunk) * D + cc * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            a.khat_w[cv + e] = kh[e];
            a.dkhat_w[cv + e] = gkh[e] + dkh[e] * inv_sqrt_d;
            a.dVs_w[cv + e] = gvh[e];  // the total dvhat, for the window tiles
        }
    }
}

}  // namespace

template <int D, int VAR>
hipError_t launch_backward_var(const BwdParams& p, hipStream_t stream) {
    // dQ, and the row dots D = dO . O the dK/dV kernels read
    hipLaunchKernelGGL((bwd_dq_kernel<D, kDqNS, D == 64 ? 3 : 2, VAR>), dim3(p.t.n_tiles), dim3(kTileWaves * 64), 0,
                       stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int KT = kBwdWaves * 16;
    if (p.n_chunks > 0) {
        // summary gradients, then their per-chunk and per-key factors
        const int st = (p.n_chunks + KT - 1) / KT * p.n_split;
        hipLaunchKernelGGL((bwd_dkdv_kernel<D, true, VAR>), dim3(p.B * p.Hkv * st), dim3(kBwdWaves * 64), 0, stream,
                           p);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        constexpr int RPS = 256 / (D / 8);
        constexpr int RPW = 64 / (D / 8);  // rows per sweep of one wave
        const dim3 grid(p.n_chunks, p.B * p.Hkv);
        // one wave per chunk when the chunk is 4, 8 or 16 rows per lane
        const int wrows = p.C % RPW == 0 ? p.C / RPW : 0;
        if (wrows == 4 || wrows == 8 || wrows == 16) {
            if (wrows == 4) hipLaunchKernelGGL((bwd_summary_kernel_wave<D, 4>), grid, dim3(64), 0, stream, p);
            if (wrows == 8) hipLaunchKernelGGL((bwd_summary_kernel_wave<D, 8>), grid, dim3(64), 0, stream, p);
            if (wrows == 16) hipLaunchKernelGGL((bwd_summary_kernel_wave<D, 16>), grid, dim3(64), 0, stream, p);
        } else switch (p.C % RPS == 0 ? p.C / RPS : 0) {
            case 1: hipLaunchKernelGGL((bwd_summary_kernel_reg<D, 1>), grid, dim3(256), 0, stream, p); break;
            case 2: hipLaunchKernelGGL((bwd_summary_kernel_reg<D, 2>), grid, dim3(256), 0, stream, p); break;
            case 4: hipLaunchKernelGGL((bwd_summary_kernel_reg<D, 4>), grid, dim3(256), 0, stream, p); break;
            case 8: hipLaunchKernelGGL((bwd_summary_kernel_reg<D, 8>), grid, dim3(256), 0, stream, p); break;
            default: {
                const size_t lds = (size_t)(((p.C + summary_red_floats<D>() + 3) & ~3) + 2 * D) * sizeof(float);
                hipLaunchKernelGGL((bwd_summary_kernel<D>), grid, dim3(256), lds, stream, p);
            }
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const int wt = (p.L + kTileWaves * 32 - 1) / (kTileWaves * 32);
    hipLaunchKernelGGL((bwd_window_kernel<D, kKvRing, D == 64 ? 3 : 2, VAR>), dim3(p.B * p.Hkv * wt), dim3(kTileWaves * 64), 0,
                       stream, p);
    return hipGetLastError();
}

template <int D>
hipError_t launch_backward(const BwdParams& p, hipStream_t stream) {
    switch (p.window) {
        case kWinChunkAligned: return launch_backward_var<D, kWinChunkAligned>(p, stream);
        case kWinBlocked: return launch_backward_var<D, kWinBlocked>(p, stream);
        case kWinNonCausal: return launch_backward_var<D, kWinNonCausal>(p, stream);
        default: return launch_backward_var<D, kWinSliding>(p, stream);
    }
}

template hipError_t launch_backward<64>(const BwdParams&, hipStream_t);
template hipError_t launch_backward<128>(const BwdParams&, hipStream_t);

}  // namespace eva
