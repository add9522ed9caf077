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
// Kernels (all bf16 storage, fp32 arithmetic, v_mfma 32x32x16 bf16):
//   bwd_dq_kernel      per query tile (4 waves x 32 columns, the forward's
//                      tiles): the columns' D = dO . O (stored for the dK/dV
//                      kernels), then key blocks of 32 rows (summaries then
//                      window band) streamed through LDS: S^T = K Q^T,
//                      dP^T = V dO^T, dS^T, and dQ^T += K^T dS^T
//                      (K^T by the transposing LDS read)
//   bwd_keys_kernel    per key tile (4 waves x 32 keys, window keys or
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
// a 32x32 score tile, its rows permuted, forms the next product's B operands
// in place.
#include <type_traits>

#include "summary.hpp"
#include "tile32.hpp"

namespace eva {

namespace {

// dQ: four ring stages (70 KB of LDS, two workgroups per CU; 204 VGPRs), so
// that the ring holds the q and dO rows of the whole workgroup while they are
// staged.  Three stages measured the same.
constexpr int kDqNS = 4;
// dK/dV: four ring stages; its accumulators leave registers for two fragments
// ahead of their product (three spill: 640 us against 554)
constexpr int kKvNS = 4, kKvPF = 2;
// Window keys take 64 instead of 128 per workgroup while tiles of 128 do not
// outnumber the CUs: twice the workgroups, each through half the steps.  Whole
// backward on MI355X, captured graph, us, 128 / 64 keys: B1 H32/8 L100 d128 W128
// 43 / 36 (8 tiles), B1 H32/8 L200 60 / 46 (16), B1 H64/16 L512 70 / 52 (64), B2 H8
// L1024 d64 W256 38.5 / 34.2 (128), B1 H32 L1024 d128 W256 60.0 / 58.5 (256); beyond,
// every query block is staged twice as often for nothing: B4 H32 L384 d128 W256
// 71.7 / 76.6 (384).  With fewer than four (head, query block) steps there is
// nothing to share (B1 H8 L40 d128 16.0 / 16.0).
constexpr int kFewKeyTiles = 256;

// wait for a block (LATER DMA instructions issued after it may stay in
// flight), then a workgroup barrier: the block is visible to every wave, and
// every wave is done with the stage the next request refills
template <int LATER>
__device__ __forceinline__ void bsync() {
    asm volatile("" ::: "memory");
    wait_vm_lgkm0<LATER>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
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
// staged, 390 / 470 with the prologue's requests in flight
// together.  The first shape's 1.9 GB take ~310 us at the rate of a plain read.
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
        block_step(std::integral_constant<int, 2>{}, j + 2);
        block_step(std::integral_constant<int, 3>{}, j + 3);
    }
    if (j < nb) block_step(std::integral_constant<int, 0>{}, j);
    if (j + 1 < nb) block_step(std::integral_constant<int, 1>{}, j + 1);
    if (j + 2 < nb) block_step(std::integral_constant<int, 2>{}, j + 2);

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
// from the prefix side: n >= sum_rows_lo(c) (win_lo(n) >= (c + 1) C; L if
// none).  Non-causal summaries are also seen by the rows of the blocks wholly
// before them: their tiles stream every row.
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
__device__ __forceinline__ int sum_rows_lo(int c, const FastDiv& W, int C, int L) {
    const int t = (c + 1) * C;  // the chunk's end, at most L
    if constexpr (VAR == kWinSliding || VAR == kWinChunkAligned) return t > L - (int)W ? L : t + (int)W - 1;
    const int down = t / W * (int)W;  // rounded up to a block start, at most L
    return down == t ? t : down > L - (int)W ? L : down + (int)W;
}

// A wave owns 32 keys (its K and V rows as B operands in registers, dK^T and
// dV^T as accumulators) and the query blocks of every head of the group that
// sees one of the workgroup's keys stream through LDS.  Per block: S = Q K^T;
// dP = dO V^T - D (the row dots are the product's initial value) with the
// exponentials of S between its products; dV^T += dO^T P with dS = P dP
// between; dK^T += Q^T dS.
//
// Window keys (SUM false): 128 keys per workgroup.  Summaries (SUM): n_split
// workgroups per tile, each over a part of the query blocks, leaving partial
// sums.  RW = 2: 64 keys per workgroup, two waves on 32 of them, each on every
// other query block, which add their accumulators at the end: for at most 64
// summaries, and for so few window keys that 128 at a time leave CUs idle.
template <int D, int NS, int WPE, int VAR, bool SUM, int RW>
__global__ __launch_bounds__(kTileWaves * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void bwd_keys_kernel(BwdParams a) {
    typedef Tile<D> T;
    constexpr int BLK = T::BLK, NKC = T::NKC, NDC = T::NDC, NDB = T::NDB;
    constexpr int NIT = 2 * T::NI + 1;  // requests per wave and block
    constexpr int STEP = RW;            // blocks per step (one per row group of waves)
    constexpr int AHEAD = NS - STEP;    // blocks requested ahead of the step computed
    constexpr int KW = kTileWaves / RW; // waves on different keys
    constexpr int KT = KW * 32;         // keys per workgroup
    constexpr bool NC = VAR == kWinNonCausal;
    static_assert(NS == 4 && (RW == 1 || RW == 2), "");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NS][2][BLK];  // [stage][Q, dO]
    __shared__ __attribute__((aligned(256))) float rowf[NS][2][64];           // [stage][lse, -D], by product row
    __shared__ __attribute__((aligned(256))) float sink[64];

    const int L = a.L;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c32 = lane & 31, h2 = lane >> 5;
    const int lim = SUM ? a.n_chunks : L;  // keys
    // consecutive tiles (splits) of one (b, kv head), which share query rows,
    // on one XCD
    const int n_kt = (lim + KT - 1) / KT, per_bg = SUM ? n_kt * a.n_split : n_kt;
    int id = blockIdx.x;
    {
        const int per = (int)gridDim.x / 8;
        if (id < per * 8) id = (id % 8) * per + id / 8;
    }
    const int bgi = id / per_bg;
    const int kt = SUM ? (id - bgi * per_bg) % n_kt : id - bgi * per_bg;
    const int split = SUM ? (id - bgi * per_bg) / n_kt : 0;
    const int k0 = kt * KT;  // first key of the tile
    const size_t bg = (size_t)bgi;
    const int b = bgi / a.fHkv, kvh = bgi - b * a.Hkv;
    const int G = a.t.G;
    const int rg = RW == 1 ? 0 : wave / KW;                // the wave's row group
    const int wk0 = k0 + (RW == 1 ? wave : wave % KW) * 32;  // its keys wk0 .. wk1
    const int wk1 = min(wk0 + 31, lim - 1);
    const int n_keys = max(0, min(32, lim - wk0));
    const bool w_active = wk0 < lim;

    // ---- query rows that see some key of the tile, some key of the wave, and
    // all of the wave's keys: key m is seen by [rows_lo(m), rows_hi(m)], both
    // non-decreasing (non-causal summaries also by the rows before rows_before)
    auto rows_lo = [&](int m) {
        if constexpr (SUM) return sum_rows_lo<VAR>(m, a.fW, a.C, L);
        else return kv_rows_lo<VAR>(m, a.fW);
    };
    auto rows_hi = [&](int m) {
        if constexpr (SUM) return L - 1;
        else return (int)min((long long)L - 1, kv_rows_hi<VAR>(m, a.fW, a.fC));
    };
    auto rows_before = [&](int m) { return SUM && NC ? m * a.C / a.fW * a.W : 0; };
    const int first = SUM && NC ? 0 : rows_lo(k0), last = rows_hi(min(k0 + KT, lim) - 1);
    const int qb0 = first / kTileRows;
    const int nqb = first <= last ? last / kTileRows - qb0 + 1 : 0;
    const int wk0c = min(wk0, lim - 1);
    const int wb0 = SUM && NC ? 0 : rows_lo(wk0c) / kTileRows;  // needed query blocks wb0 .. +wbc-1
    const unsigned wbc = w_active ? max(0, rows_hi(wk1) / kTileRows - wb0 + 1) : 0;
    const int full_lo = rows_lo(wk1), full_hi = rows_hi(wk0c), full_before = rows_before(wk0c);
    // this workgroup's part of the (head, query block) pairs
    const int all_blocks = nqb * G;
    const int j0 = SUM ? (int)((long long)all_blocks * split / a.n_split) : 0;
    const int blocks = SUM ? (int)((long long)all_blocks * (split + 1) / a.n_split) - j0 : all_blocks;

    // ---- requests: step (head, query block) in that order.  Q and dO rows by
    // all waves; lse and -D by waves 0 and 1, 4 bytes per lane, into the order
    // of the product's rows (waves 2 and 3 issue one without rows into the
    // sink, so that every wave counts the same instructions).
    const unsigned lane_off = dma_lane_off<D, true>(wave, lane);
    const unsigned lds0 = lds_addr(lds) + wave * T::GRP;
    const unsigned row_off =
        lane < 32 ? 4 * (T::key_of(lane >> 3, lane & 3) + ((lane >> 2) & 1) * T::KH) : 0x40000000u;
    int rq_h = SUM && nqb > 0 ? j0 / nqb : 0, rq_b = SUM ? j0 - rq_h * nqb : 0;  // next request's head and block
    int rq_left = blocks;
    const size_t head0 = (size_t)b * a.H + (size_t)kvh * G;
    auto request = [&](int stage) {
        const bool real = rq_left-- > 0;
        const int r0 = (qb0 + rq_b) * kTileRows;
        const int rows = real ? min(L - r0, kTileRows) : 0;
        const size_t row = (head0 + rq_h) * L + r0;
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
        static_assert(NS == 4, "stages 2 and 3 hold one block per wave");
        unsigned char* const mine = lds[2 + wave / 2][wave % 2];
        const uintptr_t at = (bg * (size_t)lim + wk0) * T::ROWB;
        stage_cols<D>(rows_desc<D>((uintptr_t)(SUM ? a.Ks : a.K) + at, n_keys), lane, lds_addr(mine));
        request(0);
        request(1);
        wait_vm_lgkm0<2 * NIT>();
        read_cols<D>(mine, lane, kf);
        wait_vm_lgkm0<2 * NIT>();
        stage_cols<D>(rows_desc<D>((uintptr_t)(SUM ? a.Vs : a.V) + at, n_keys), lane, lds_addr(mine));
        wait_vm_lgkm0<0>();
        read_cols<D>(mine, lane, vf);
        wait_vm_lgkm0<0>();
        __builtin_amdgcn_s_barrier();  // every wave's rows are read before further blocks overwrite them
        asm volatile("" ::: "memory");
    }
    if constexpr (AHEAD == 3) request(2);

    const Frags<D> fr(lane, true);
    floatx16 dk[NDB], dv[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) dk[db] = dv[db] = floatx16{};

    const float bias = SUM ? a.log2C : 0.f;
    // the wave's block of this step, as a block of the range (waves of row
    // group rg take blocks rg, rg + RW, ..)
    int cur = (SUM && nqb > 0 ? j0 % nqb : 0) + rg;
    if (cur >= nqb) cur -= nqb;
    int left = blocks - rg;
    auto block_step = [&](auto ph_tag) {
        constexpr int PH = decltype(ph_tag)::value;  // first stage of the step, as a constant
        bsync<(AHEAD - STEP) * NIT>();
#pragma unroll
        for (int i = 0; i < STEP; ++i) request((PH + AHEAD + i) % NS);
        const int qb = qb0 + cur;
        const bool mine = left > 0;
        left -= RW;
        cur += RW;
        if (cur >= nqb) cur -= nqb;
        if (RW > 1 && cur >= nqb) cur -= nqb;
        if (!mine || (unsigned)(qb - wb0) >= wbc) return;
        const int st = RW == 1 ? PH : PH + rg;
        const unsigned char* qs = lds[st][0];
        const unsigned char* gs = lds[st][1];
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
            return *reinterpret_cast<const floatx4*>(&rowf[st][arr][8 * q + 4 * h2]);
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
        const int r0 = qb * kTileRows, r1 = r0 + kTileRows - 1;
        if ((r0 < full_lo || r1 > full_hi) && r1 >= full_before) {
            const int l = lane_here();
            const int m = min(wk0 + (l & 31), lim - 1), rel = r0 + (l >> 5) * T::KH;
            if constexpr (SUM && NC) {
                const int lo = rows_lo(m) - rel, before = rows_before(m) - rel;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int x = T::key_of(i / 4, i % 4);
                    s[i] = x >= lo || x < before ? s[i] : -INFINITY;
                }
            } else {
                if (r1 > full_hi) mask_above<D>(s, rows_hi(m) - rel);
                if (r0 < full_lo) mask_below<D>(s, rows_lo(m) - rel);
            }
        }
        floatx4 l4 = rows4(0, 0);
#pragma unroll
        for (int k = 0; k < NDC; ++k) {
            load(k + NDC + PF);
            dp = mfma32_bf16(op[(k + NDC) % (PF + 1)], vf[k], dp);
#pragma unroll
            for (int i = k * 16 / NDC; i < (k + 1) * 16 / NDC; ++i) {
                s[i] = fast_exp2(fmaf(s[i], a.scale_log2, fmaf(l4[i % 4], -kLog2e, bias)));  // P (masked entries: 0)
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
    // NS / STEP steps per trip, so that each one's stages are constants
    typedef std::integral_constant<int, 0> P0;
    typedef std::integral_constant<int, 1> P1;
    typedef std::integral_constant<int, 2> P2;
    typedef std::integral_constant<int, 3> P3;
    const int steps = (blocks + STEP - 1) / STEP;
    int j = 0;
    if constexpr (STEP == 1) {
        for (; j + 3 < steps; j += 4) {
            block_step(P0{});
            block_step(P1{});
            block_step(P2{});
            block_step(P3{});
        }
        if (j < steps) block_step(P0{});
        if (j + 1 < steps) block_step(P1{});
        if (j + 2 < steps) block_step(P2{});
    } else {
        for (; j + 1 < steps; j += 2) {
            block_step(P0{});
            block_step(P2{});
        }
        if (j < steps) block_step(P0{});
    }

    wait_vm_lgkm0<0>();  // no request may still be writing LDS when the workgroup ends
    __builtin_amdgcn_s_barrier();  // every wave is done with the ring
    asm volatile("" ::: "memory");

    if constexpr (RW == 2) {
        // the second row group's accumulators, added by the first
        static_assert((size_t)KW * 32 * D * 2 * 4 <= NS * 2 * BLK, "the accumulators fit in the ring");
        floatx4* const x = reinterpret_cast<floatx4*>(&lds[0][0][0]) + (size_t)(wave % KW) * (32 * D * 2 / 4) + lane;
        if (rg == 1) {
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x[(db * 4 + q) * 128] = floatx4{dk[db][4 * q], dk[db][4 * q + 1], dk[db][4 * q + 2], dk[db][4 * q + 3]};
                    x[(db * 4 + q) * 128 + 64] =
                        floatx4{dv[db][4 * q], dv[db][4 * q + 1], dv[db][4 * q + 2], dv[db][4 * q + 3]};
                }
        }
        __syncthreads();
        if (rg == 0) {
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const floatx4 xk = x[(db * 4 + q) * 128], xv = x[(db * 4 + q) * 128 + 64];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        dk[db][4 * q + i] += xk[i];
                        dv[db][4 * q + i] += xv[i];
                    }
                }
        }
        __syncthreads();
        if (rg == 1) return;
    }

    // ---- results on whole rows: the accumulators go through LDS in fp32, so
    // that the rows are written (and a chunk's vectors read) D / 8
    // neighbouring lanes to a row
    constexpr int SROW = 4 * D + 16;  // bytes per staged row; fragment writes fall in distinct banks
    constexpr int LPR = D / 8, RPS = 64 / LPR;
    static_assert(kTileWaves * 32 * SROW <= NS * 2 * BLK, "staged rows fit in the ring");
    unsigned char* const stg = &lds[0][0][0] + wave * 32 * SROW;
    const float inv_sqrt_d = a.scale_log2 / kLog2e, inv_c = 1.f / (float)a.C;
    const int row = lane / LPR, f0 = lane % LPR * 8;
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
    auto staged = [&](int r, int x) { return *reinterpret_cast<const floatx4*>(stg + r * SROW + f0 * 4 + 16 * x); };
    if constexpr (SUM) {
        // fp32 partial summary gradients, for the per-chunk pass
        const size_t slot = ((size_t)split * a.B * a.Hkv + bg) * lim + wk0;
        auto store = [&](float* out, float scale) {
#pragma unroll
            for (int i = 0; i < 32 / RPS; ++i) {
                const int r = i * RPS + row;
                if (r < n_keys)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        *reinterpret_cast<floatx4*>(out + (slot + r) * D + f0 + 4 * x) = staged(r, x) * scale;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        stage_acc(dk);
        store(a.dKs_w, inv_sqrt_d);
        stage_acc(dv);
        store(a.dVs_w, 1.f);
        return;
    }

    // ---- the window gradient plus the key's share of its chunk's summary
    // gradient (keys after the last complete chunk have none)
    // the chunks of the wave's 32 keys start at c0; vectors of chunks past the
    // last complete one, and the factors of keys past it, read as zeros
    const int c0 = min(wk0, L - 1) / a.fC;
    const int n_c = max(0, min(a.n_chunks - c0, 33)), n_f = max(0, min(a.n_chunks * a.C - wk0, 32));
    // (their descriptors in scalar registers: the compiler computes the tile in
    // vector registers, and would wrap each of the 56 loads in a loop over the
    // lanes' descriptors, 3 us a workgroup)
    auto rsrc = [](const float* w, int n) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(uniform_ptr(w)), 0,
                                                 __builtin_amdgcn_readfirstlane(n * 4), 0x00020000);
    };
    auto vec_rsrc = [&](const float* w) { return rsrc(w + (bg * (size_t)a.n_chunks + c0) * D, n_c * D); };
    auto key_rsrc = [&](const float* w) { return rsrc(w + bg * (size_t)a.n_chunks * a.C + wk0, n_f); };
    auto load4 = [&](__amdgpu_buffer_rsrc_t r, int off) {
        return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    };
    auto load1 = [&](__amdgpu_buffer_rsrc_t r, int off) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    };
    // row r's byte offset into the chunk vectors
    auto vec_off = [&](int r) { return ((min(wk0 + r, L - 1) / a.fC - c0) * D + f0) * 4; };
    // rows r = i RPS + row in batches of NBAT, whose vectors are all in flight
    // together (those of the first batch behind the staging)
    constexpr int NROW = 32 / RPS, NBAT = NROW < 4 ? NROW : 4;
    auto store_row = [&](bf16* out, int r, const floatx4& v0, const floatx4& v1) {
        const u32x4 w = {pack_bf16x2(v0[0], v0[1]), pack_bf16x2(v0[2], v0[3]), pack_bf16x2(v1[0], v1[1]),
                         pack_bf16x2(v1[2], v1[3])};
        if (wk0 + r < L)
            __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(out + (bg * (size_t)L + wk0 + r) * D + f0));
    };
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

// Register-resident variant for chunks of exactly eight rows per thread: every
// thread loads its key and value rows once, and the passes over the chunk
// run on registers (one memory latency per chunk instead of one per pass).
template <int D>
__global__ __launch_bounds__(256) void bwd_summary_kernel_reg(BwdParams a) {
    constexpr int TPR = D / 8;
    constexpr int RPS = 256 / TPR;
    constexpr int ROWS = 8, C = ROWS * RPS;
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
        kw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(K + i * RPS * D));
        vw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(V + i * RPS * D));
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
template <int D, int ROWS, bool ANY>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(ROWS >= 16 ? 2 : 1))) void bwd_summary_kernel_wave(BwdParams a) {
    constexpr int TPR = D / 8;
    constexpr int RPS = 64 / TPR;
    const int C = ANY ? a.C : ROWS * RPS;
    const int chunk = blockIdx.x;
    const size_t bg = blockIdx.y;
    const int L = a.L;
    const int t = threadIdx.x, cc = t % TPR, r0 = t / TPR;
    const int first = chunk * C;
    const bf16* K = static_cast<const bf16*>(a.K) + (bg * (size_t)L + first + r0) * D + cc * 8;
    const bf16* V = static_cast<const bf16*>(a.V) + (bg * (size_t)L + first + r0) * D + cc * 8;
    const ChunkRows<D, bf16, ANY> src{C, cc};
    u32x4 kw[ROWS], vw[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        kw[i] = src.load(K, i * RPS * D, r0);
        vw[i] = src.load(V, i * RPS * D, r0);
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
        if (ANY && r0 + i * RPS >= C) sl[i] = -INFINITY;
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
        if (cc == 0 && (!ANY || r0 + i * RPS < C)) {
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
    if (p.n_chunks > 0) {
        // summary gradients, then their per-chunk and per-key factors
        if (p.n_chunks <= 64)
            hipLaunchKernelGGL((bwd_keys_kernel<D, kKvNS, D == 64 ? 3 : 2, VAR, true, 2>),
                               dim3(p.B * p.Hkv * p.n_split), dim3(kTileWaves * 64), 0, stream, p);
        else
            hipLaunchKernelGGL((bwd_keys_kernel<D, kKvNS, D == 64 ? 3 : 2, VAR, true, 1>),
                               dim3(p.B * p.Hkv * ((p.n_chunks + 127) / 128) * p.n_split), dim3(kTileWaves * 64), 0,
                               stream, p);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        constexpr int RPS = 256 / (D / 8);
        constexpr int RPW = 64 / (D / 8);  // rows per sweep of one wave
        const dim3 grid(p.n_chunks, p.B * p.Hkv);
        auto wave = [&](auto rows, auto any) {
            hipLaunchKernelGGL((bwd_summary_kernel_wave<D, decltype(rows)::value, decltype(any)::value>), grid, dim3(64),
                               0, stream, p);
        };
        typedef std::integral_constant<int, 2> R2;
        typedef std::integral_constant<int, 4> R4;
        typedef std::integral_constant<int, 8> R8;
        typedef std::integral_constant<int, 16> R16;
        // one wave per chunk for chunks of up to 16 rows per lane (whole backward
        // against the three-pass kernel, us: B8 Hkv32 L4096 d128 C48 1185 ->
        // 1114; B4 Hkv8 L4096 C17 223 -> 192), one workgroup for exactly 8 rows
        // per thread; other lengths take three passes (in registers of 8 rows:
        // B8 Hkv8 L8192 d128 C65 654 -> 671, C100 625 -> 622)
        if (p.C == 4 * RPW) wave(R4{}, std::false_type{});
        else if (p.C == 8 * RPW) wave(R8{}, std::false_type{});
        else if (p.C == 16 * RPW) wave(R16{}, std::false_type{});
        else if (p.C <= 2 * RPW) wave(R2{}, std::true_type{});
        else if (p.C <= 4 * RPW) wave(R4{}, std::true_type{});
        else if (p.C <= 8 * RPW) wave(R8{}, std::true_type{});
        else if (p.C <= 16 * RPW) wave(R16{}, std::true_type{});
        else if (p.C == 8 * RPS) hipLaunchKernelGGL((bwd_summary_kernel_reg<D>), grid, dim3(256), 0, stream, p);
        else {
            const size_t lds = (size_t)(((p.C + summary_red_floats<D>() + 3) & ~3) + 2 * D) * sizeof(float);
            hipLaunchKernelGGL((bwd_summary_kernel<D>), grid, dim3(256), lds, stream, p);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const int bg = p.B * p.Hkv, wt = (p.L + 127) / 128, wt2 = (p.L + 63) / 64;
    if ((long long)p.t.G * ((p.L + 31) / 32) >= 4 && (long long)bg * wt <= kFewKeyTiles)
        hipLaunchKernelGGL((bwd_keys_kernel<D, kKvNS, D == 64 ? 3 : 2, VAR, false, 2>), dim3(bg * wt2),
                           dim3(kTileWaves * 64), 0, stream, p);
    else
        hipLaunchKernelGGL((bwd_keys_kernel<D, kKvNS, D == 64 ? 3 : 2, VAR, false, 1>), dim3(bg * wt),
                           dim3(kTileWaves * 64), 0, stream, p);
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
