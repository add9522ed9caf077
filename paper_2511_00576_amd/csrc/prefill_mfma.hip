// Fused window + summary EVA prefill for gfx950, bf16, on 32x32x16
// matrix-core products.
//
// The attention is the one of the fused FlashEVA formulation (section
// "FlashEVA"): one softmax per query over the exact keys of its local window
// and one key per chunk summary that lies fully before the window, the
// summaries carrying a +ln C logit offset.
//
// Work decomposition: a workgroup is 4 waves sharing one K/V head; each wave
// owns 32 query columns, so the workgroup covers 128 columns = Gt heads x
// (128 / Gt) positions.  K/V blocks of 32 rows are staged HBM -> LDS by
// buffer_load_dwordx4 ... lds into a three-stage ring and read by every wave;
// one workgroup barrier per block.  51 KB of LDS and 168 VGPRs let three
// workgroups (three waves per SIMD) share a CU, so that one wave's products,
// another's exponentials and a third's loads overlap.
//
// What bounds it.  A wave issues at most one instruction every four cycles,
// so beside the matrix core its instruction count sets the pace: 32x32x16
// products (16 a block instead of 34 of 16x16x32), request offsets that are
// the same for every block (the buffer descriptor moves, and its size replaces
// the clamp of rows past the end), block classes as ranges of block numbers,
// two weights per conversion and per addition to the denominator: ~150
// instructions per wave and block and ~1000 per wave beside them (counters;
// ~330 a block with 16x16x32).  Measured on MI355X, us (B8 H32 L4096 W256 C64
// / B4 H32/8 L8192 W512 C128 / B1 H32/8 L32768 W1024 C256): 331 / 388 / 662
// with 16x16x32 products, two waves per SIMD and the products of one block
// interleaved with the exponentials of the one before; 316 / 388 / 768
// (spills) the same with 32x32x16; 295 / 329 / 563 with three waves per SIMD
// and each lane loading its own query row; 271 / 327 / 567 as it is here, the
// query rows staged whole through LDS (between 247 / 317 / 553 and that from
// run to run).  Of 263 / 318 / 554, 198 / 169 / 240 remain without the
// arithmetic and 175 / 214 / 376 without the K/V traffic: the first is bound
// by its traffic (1.54 GB past the L2s, 1.42x the algorithmic bytes) about as
// much as by its arithmetic, and their overlap is what is lost; the others by
// their arithmetic (matrix cores busy 34 / 53 / 60% of the time; waves wait
// for data 40 / 21 / 20% and to be issued 30 / 42 / 44% of theirs).
//
// Softmax runs in log2 units with a lazy running maximum: the cross-lane
// maximum and the rescale of the accumulators only run when some lane sees a
// score more than 2^8 above the stored one.
//
// Masks.  Blocks entirely inside every column's visible range need none.  A
// block crossing an edge is masked per element after its product, against the
// lane's own key range (compare and select; only the edge that crosses).
//
// Window variants (template VAR, see win_lo / win_hi / sum_lo / sum_hi): the
// block plan and the per-wave block classification follow each row's window
// [win_lo(n), win_hi(n)] and summary ranges.  The non-causal variant stages
// every summary block (its rows see the chunks on both sides of their block).
#include <type_traits>

#include "tile32.hpp"

namespace eva {

namespace {

constexpr float kTau = 8.f;  // lazy-rescale threshold (log2 units)
constexpr int kNS = 3;       // ring stages

// LO: also store the output's rounding residual (training forward); a
// separate instantiation, since even an untaken branch for it in the epilogue
// measured 6-8% slower in the 4-wave configuration.
template <int D, int WPE, int VAR, bool LO>
__global__ __launch_bounds__(kTileWaves * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void prefill_mfma_kernel(PrefillParams a) {
    typedef Tile<D> T;
    constexpr int NS = kNS, BLK = T::BLK, NKC = T::NKC, NDC = T::NDC, NDB = T::NDB;
    constexpr int NIT = 2 * T::NI;  // requests per wave and block
    constexpr int AHEAD = NS - 1;   // blocks requested ahead of the one computed
    static_assert(NS == 3, "the block loop below takes three steps per trip");

    __shared__ __attribute__((aligned(1024))) unsigned char lds[NS][2][BLK];  // [stage][K, V]

    const int L = a.L;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h2 = lane >> 5, c32 = lane & 31;
    const PosTile tile(a.t, blockIdx.x, wave);
    const int p0 = tile.p0;
    const int col_n = p0 + c32;  // this lane's query position

    const size_t bh = (size_t)tile.b * a.H + tile.h;

    const KeyPlan<VAR> plan(tile.n0, min(tile.n0 + a.t.pos_per_wg, L) - 1, p0, L, a.fW, a.fC, a.n_chunks);
    const int nb = plan.nb;
    const KeySource<D> src(plan, a.K, a.V, a.Ks, a.Vs, (size_t)tile.b * a.Hkv + tile.kvh, L, a.n_chunks);
    const unsigned k_off = dma_lane_off<D, true>(wave, lane), v_off = dma_lane_off<D, false>(wave, lane);
    const unsigned lds0 = lds_addr(lds) + wave * T::GRP;
    auto request = [&](int j, int stage) {
        u32x4 dk, dv;
        src.block(j, dk, dv);
        dma_block<D>(dk, k_off, lds0 + stage * 2 * BLK);
        dma_block<D>(dv, v_off, lds0 + stage * 2 * BLK + BLK);
    };
    const Frags<D> fr(lane, false);  // K rows are swizzled, V rows (only read transposed) are not

    floatx16 acc[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[db] = floatx16{};
    // running maximum (log2 units, the same on both lanes of a column) and
    // this lane's part of the denominator: the bf16-rounded weights its
    // column gives to the keys it holds, summed in fp32.  m_neg: -m_run, or 0
    // while m_run is -inf (a column that has seen no key yet), kept beside it
    // so that each step's exponent offset is one add
    float m_run = -INFINITY, m_neg = 0.f, l_run = 0.f;
    floatx16 sc;                     // scores of a block: element i is key key_of(i / 4, i % 4) + h2 KH of the block

    auto lane_max = [&]() {
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sc[i]);
        return mx;
    };
    // lazy maximum update once the scores of a block are known
    auto update_max = [&](float lm, float bias) {
        const bool need = fmaf(lm, a.scale_log2, bias) > m_run + kTau;
        if (__ballot(need) == 0) return;
        const float bm = fmaf(xhalf_max(lm), a.scale_log2, bias);
        const bool up = bm > m_run + kTau;
        const float alpha = up ? fast_exp2(m_run - bm) : 1.f;
        m_run = up ? bm : m_run;
        m_neg = m_run == -INFINITY ? 0.f : -m_run;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db) acc[db] *= alpha;
    };
    // wait until a block landed (LATER blocks requested after it may stay in
    // flight), then make it visible to the whole workgroup; every wave's
    // reads of the stage about to be refilled are done as well
    auto sync_block = [&](auto later_tag) {
        constexpr int LATER = decltype(later_tag)::value;
        asm volatile("" ::: "memory");
        wait_vm_lgkm0<LATER * NIT>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // ---- prologue: the wave's queries (columns past L: zeros, whose outputs
    //      are not stored) through stages 1 and 2 of the ring as whole rows,
    //      block 0 beside them, then the other blocks requested ahead ----
    bf16x8 qf[NDC];  // B operand of S^T = K Q^T: features dc*16 + 8 h2 .. +7
    {
        unsigned char* const mine = lds[1 + wave / 2][wave % 2];
        const uintptr_t at = (uintptr_t)a.Q + (bh * L + (size_t)p0) * T::ROWB;
        stage_cols<D>(rows_desc<D>(at, max(0, min(32, L - p0))), lane, lds_addr(mine));
        request(0, 0);
        wait_vm_lgkm0<NIT>();
        read_cols<D>(mine, lane, qf);
        wait_vm_lgkm0<NIT>();
        __builtin_amdgcn_s_barrier();  // every wave's queries are read before the stages are filled
        asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int k = 1; k < AHEAD; ++k) request(k, k);

    // ---- iteration j: S^T(j) = K Q^T, its weights, O^T += V^T P^T(j) ----
    auto iteration = [&](auto ph_tag, int j) {
        constexpr int PH = decltype(ph_tag)::value;  // j mod NS: the stages as constants
        // block j landed (the AHEAD-1 blocks after it may stay in flight);
        // the block requested in this iteration refills the stage of block
        // j-1, whose last reads were before this barrier
        sync_block(std::integral_constant<int, AHEAD - 1>{});
        request(j + AHEAD, (PH + AHEAD) % NS);
        if (!plan.needed(j)) return;
        const unsigned char* ks = lds[PH][0];
        const unsigned char* vs = lds[PH][1];
        constexpr int kPF = kFragAhead;
        constexpr int N = NDC + NKC * NDB;  // fragments: NDC of K, then NKC NDB of V^T
        bf16x8 op[kPF + 1];                 // ring of fragments, requested kPF products ahead
        auto load = [&](int k) {
            op[k % (kPF + 1)] = k < NDC ? fr.row(ks, k) : fr.tr(vs, (k - NDC) % NDB, (k - NDC) / NDB);
        };
#pragma unroll
        for (int k = 0; k < kPF; ++k) load(k);
        // fences keep the prefetch distance (and the register count) fixed;
        // the products run at a raised wave priority
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int k = 0; k < NDC; ++k) {
            if (k + kPF < NDC) load(k + kPF);
            sc = mfma32_bf16(op[k % (kPF + 1)], qf[k], k == 0 ? floatx16{} : sc);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
        const float bias = j < plan.nsb ? a.log2C : 0.f;
        if (!plan.full(j)) plan.template mask<D>(sc, j, p0, L, a.fW, a.fC, a.n_chunks);
        update_max(lane_max(), bias);
        // the first V fragments are requested only here (their registers are
        // the masks' before) and land behind the exponentials
#pragma unroll
        for (int k = NDC; k < NDC + kPF; ++k) load(k);
        // contraction slot e of 16-key step kc is score element 8 kc + e (the
        // V read uses the same order); step kc+1's weights are formed between
        // the products of step kc
        const float off = bias + m_neg;
        u32x4 pf[NKC];
        auto weights = [&](int kc, int e) {
            const float w0 = fast_exp2(fmaf(sc[8 * kc + 2 * e], a.scale_log2, off));
            const float w1 = fast_exp2(fmaf(sc[8 * kc + 2 * e + 1], a.scale_log2, off));
            pf[kc][e] = pack_bf16x2(w0, w1);
            l_run = dot2_ones(pf[kc][e], l_run);
        };
#pragma unroll
        for (int e = 0; e < 4; ++e) weights(0, e);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int k = NDC; k < N; ++k) {
            if (k + kPF < N) load(k + kPF);
            const int db = (k - NDC) % NDB, kc = (k - NDC) / NDB;
            acc[db] = mfma32_bf16(op[k % (kPF + 1)], __builtin_bit_cast(bf16x8, pf[kc]), acc[db]);
            if (kc + 1 < NKC) {
#pragma unroll
                for (int e = db * 4 / NDB; e < (db + 1) * 4 / NDB; ++e) weights(kc + 1, e);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    // three steps per trip, so that each one's stage indices are constants
    typedef std::integral_constant<int, 0> P0;
    typedef std::integral_constant<int, 1> P1;
    typedef std::integral_constant<int, 2> P2;
    int j = 0;
    for (; j + 2 < nb; j += 3) {
        iteration(P0{}, j);
        iteration(P1{}, j + 1);
        iteration(P2{}, j + 2);
    }
    if (j < nb) iteration(P0{}, j);
    if (j + 1 < nb) iteration(P1{}, j + 1);

    // No request may still be writing LDS when the workgroup ends: wait for
    // them before the stores, which need not complete before the end.
    wait_vm_lgkm0<0>();

    // ---- epilogue: O = acc / l, staged through LDS so that each store
    // instruction writes whole output rows (measured on MI355X with an earlier
    // layout: whole rows took the LLM workload from 347 to 331 us, the training
    // forward with the residual from 434 to 356 us).  Every wave is done with
    // the ring: it holds the staged rows now.
    __builtin_amdgcn_s_barrier();
    static_assert(kTileWaves * 32 * kStageRow<D> <= NS * 2 * BLK, "staged rows fit in the ring");
    unsigned char* const stg = &lds[0][0][0] + wave * 32 * kStageRow<D>;
    const float l_sum = xhalf_sum(l_run);
    const float inv = 1.f / l_sum;
    // natural log of the softmax denominator: sum 2^(x - m_run) = l
    if (a.lse && h2 == 0 && col_n < L) a.lse[bh * L + col_n] = (m_run + __builtin_amdgcn_logf(l_sum)) * kLn2;
    const size_t out0 = (bh * L + (size_t)p0) * D;
    store_tile_rows<D>(stg, lane, static_cast<bf16*>(a.O) + out0, L - p0,
                       [&](int db, int i) { return pack_bf16x2(acc[db][i] * inv, acc[db][i + 1] * inv); });
    if constexpr (LO) {
        // residual of the rounding: what the bf16 output lost
        store_tile_rows<D>(stg, lane, static_cast<bf16*>(a.O_lo) + out0, L - p0, [&](int db, int i) {
            const float v0 = acc[db][i] * inv, v1 = acc[db][i + 1] * inv;
            const uint32_t w = pack_bf16x2(v0, v1);
            return pack_bf16x2(v0 - bf16_lo(w), v1 - bf16_hi(w));
        });
    }
}

}  // namespace

template <int D, int VAR, bool LO = false>
void launch_prefill_mfma_var(const PrefillParams& p, hipStream_t stream) {
    // waves per SIMD: D = 128 needs 168 VGPRs (three); D = 64 fits 128 (four)
    hipLaunchKernelGGL((prefill_mfma_kernel<D, D == 64 ? 4 : 3, VAR, LO>), dim3(p.t.n_tiles), dim3(kTileWaves * 64), 0,
                       stream, p);
}

template <int D>
hipError_t launch_prefill_mfma(const PrefillParams& p, hipStream_t stream) {
    if (p.O_lo) {
        // the training forward, keeping the output's rounding residual
        switch (p.window) {
            case kWinChunkAligned: launch_prefill_mfma_var<D, kWinChunkAligned, true>(p, stream); break;
            case kWinBlocked: launch_prefill_mfma_var<D, kWinBlocked, true>(p, stream); break;
            case kWinNonCausal: launch_prefill_mfma_var<D, kWinNonCausal, true>(p, stream); break;
            default: launch_prefill_mfma_var<D, kWinSliding, true>(p, stream); break;
        }
        return hipGetLastError();
    }
    switch (p.window) {
        case kWinChunkAligned: launch_prefill_mfma_var<D, kWinChunkAligned>(p, stream); break;
        case kWinBlocked: launch_prefill_mfma_var<D, kWinBlocked>(p, stream); break;
        case kWinNonCausal: launch_prefill_mfma_var<D, kWinNonCausal>(p, stream); break;
        default: launch_prefill_mfma_var<D, kWinSliding>(p, stream); break;
    }
    return hipGetLastError();
}

template hipError_t launch_prefill_mfma<64>(const PrefillParams&, hipStream_t);
template hipError_t launch_prefill_mfma<128>(const PrefillParams&, hipStream_t);

}  // namespace eva
