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
// two weights per conversion and per addition to the denominator: ~165
// instructions per wave and block against ~330 before.  Measured on MI355X, us
// (B8 H32 L4096 W256 C64 / B4 H32/8 L8192 W512 C128 / B1 H32/8 L32768 W1024
// C256): 331 / 388 / 662 with 16x16x32 products, two waves per SIMD and the
// products of one block interleaved with the exponentials of the one before;
// 316 / 388 / 768 (spills) the same with 32x32x16; 295 / 329 / 563 as it is
// here.  Of the first, 215 us remain without the arithmetic (1.08 GB: the
// HBM limit) and 198 without the memory traffic; the last is at 56% of the
// matrix-core cycles.
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

#include "eva_device.hpp"
#include "eva_kernels.hpp"

namespace eva {

namespace {

constexpr float kTau = 8.f;  // lazy-rescale threshold (log2 units)
constexpr int kPF = 3;       // LDS fragments requested ahead of their product
constexpr int kNW = kMfmaWaves, kNS = 3, kBN = 32;  // waves, ring stages, rows per block

template <int D>
struct MCfg {
    static constexpr int ROWB = D * 2;         // bytes per row
    static constexpr int NKC = kBN / 16;       // 16-key steps of the value product
    static constexpr int RPI = 1024 / ROWB;    // rows per DMA instruction
    static constexpr int GRP = 1024 + 64;      // LDS bytes from one instruction's rows to the next's
    static constexpr int BLK = kBN / RPI * GRP;// LDS bytes per block
    static constexpr int NI = kBN / RPI / kNW; // DMA instructions / wave / array
    static_assert(NI >= 1, "block too small for the workgroup");
    static constexpr int NIT = 2 * NI;
    static constexpr int NDC = D / 16;         // contraction steps of S = K Q^T
    static constexpr int NDB = D / 32;         // 32-feature output blocks
    // LDS byte offset of a row within its block
    static constexpr __host__ __device__ int row_at(int r) { return r / RPI * GRP + r % RPI * ROWB; }
    // Score row 8q + 4h + i of a block holds key key_of(q, i) + h * KH.
    // The four rows i of a transposing V read then lie 64 bytes apart modulo
    // the 256 bytes of the banks (in other DMA groups, or in the two halves
    // of 256 bytes for 128-byte rows), without a swizzle: its offsets are
    // immediates of one lane address.
    static constexpr int KH = D == 128 ? 1 : 4;
    static constexpr __host__ __device__ int key_of(int q, int i) {
        return 16 * (q >> 1) + 2 * (q & 1) + (D == 128 ? 4 * i : 8 * (i >> 1) + (i & 1));
    }
    // stored 16-B chunk of a K row = logical chunk ^ kswz(row) (the low two
    // bits): a 16-lane fragment read finds 16 rows on distinct banks, and its
    // offsets are immediates of two lane addresses
    static constexpr __host__ __device__ int kswz(int r) { return D == 128 ? r & 3 : (r >> 1) & 3; }
};

// LO: also store the output's rounding residual (training forward); a
// separate instantiation, since even an untaken branch for it in the epilogue
// measured 6-8% slower in the 4-wave configuration.
template <int D, int WPE, int VAR, bool LO>
__global__ __launch_bounds__(kNW * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void prefill_mfma_kernel(PrefillParams a) {
    typedef MCfg<D> Cfg;
    constexpr int NW = kNW, NS = kNS, BN = kBN;
    constexpr int ROWB = Cfg::ROWB, BLK = Cfg::BLK, GRP = Cfg::GRP, RPI = Cfg::RPI, NIT = Cfg::NIT;
    constexpr int NKC = Cfg::NKC, NDC = Cfg::NDC, NDB = Cfg::NDB;
    constexpr int AHEAD = NS - 1;  // blocks requested ahead of the one computed
    static_assert(NS == 3, "the block loop below takes three steps per trip");

    __shared__ __attribute__((aligned(1024))) unsigned char lds[NS][2][BLK];

    const int L = a.L;
    const FastDiv W = a.fW, C = a.fC;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h2 = lane >> 5, c32 = lane & 31;

    // ---- tile decode: XCD-aware remap, heavy (late) position tiles first ----
    int id = blockIdx.x;
    {
        const int per = a.n_tiles / 8;
        if (id < per * 8) id = (id % 8) * per + id / 8;
    }
    const int q_pos = id / a.f_pos_tiles, q_hg = q_pos / a.f_hg;
    const int pt = a.n_pos_tiles - 1 - (id - q_pos * a.n_pos_tiles);
    const int hg = q_pos - q_hg * a.n_hg;
    const int b = q_hg / a.f_hkv;
    const int kvh = q_hg - b * a.Hkv;

    const int h = kvh * a.G + hg * a.Gt + (wave & (a.Gt - 1));
    const int n0 = pt * a.pos_per_wg;
    const int p0 = n0 + (wave >> a.gt_shift) * 32;
    const int n_hi = min(n0 + a.pos_per_wg - 1, L - 1);
    const int col_n = p0 + c32;           // this lane's query position
    const int n_c = min(col_n, L - 1);

    // ---- Q fragments (B operand of S^T = K Q^T): features dc*16 + 8 h2 .. +7.
    // Columns past L read row L-1: finite, and their outputs are not stored.
    const size_t bh = (size_t)b * a.H + h;
    bf16x8 qf[NDC];
    {
        const bf16* qrow = static_cast<const bf16*>(a.Q) + (bh * L + (size_t)n_c) * D + h2 * 8;
#pragma unroll
        for (int f = 0; f < NDC; ++f) qf[f] = *reinterpret_cast<const bf16x8*>(qrow + f * 16);
    }

    // blocks the workgroup stages: summaries [0, s(n_hi)) (non-causal: all),
    // then the window band; block j of the band is rows (kb0 + j - nsb) * BN ..
    constexpr bool NC = VAR == kWinNonCausal;
    const int nsb = ((NC ? a.n_chunks : sum_lo<VAR>(n_hi, W, C)) + BN - 1) / BN;
    const int kb0 = win_lo<VAR>(n0, W, C) / BN;
    const int nb = nsb + (win_hi<VAR>(n_hi, W, L) / BN - kb0 + 1);

    // what this wave needs: prefix summaries c < ws_hi (all columns: c < ws_lo),
    // non-causal suffix summaries c >= wsx_lo (all columns: c >= wsx_hi), and
    // window keys in [wlo_min, whi_max] (all columns: [wlo_max, whi_min]),
    // as ranges of block numbers
    const bool w_active = p0 < L;
    const int wp_last = min(p0 + 31, L - 1);
    const int whi_min = win_hi<VAR>(p0, W, L), wlo_max = win_lo<VAR>(wp_last, W, C);
    const int sn1 = w_active ? (sum_lo<VAR>(wp_last, W, C) + BN - 1) / BN : 0;  // needed summary blocks: j < sn1
    const int sf1 = sum_lo<VAR>(p0, W, C) / BN;                                 // full ones: j < sf1
    const int xn0 = NC && w_active ? sum_hi<VAR>(p0, W, C, L) / BN : nsb;       // and needed: j >= xn0
    const int xf0 = NC ? (sum_hi<VAR>(wp_last, W, C, L) + BN - 1) / BN : nsb;   // and full: [xf0, xf1)
    const int xf1 = NC ? a.n_chunks / BN : 0;
    const int shift = nsb - kb0;
    const int wn0 = win_lo<VAR>(p0, W, C) / BN + shift;                         // needed window blocks: wn0 .. +wnc-1
    const unsigned wnc = w_active ? win_hi<VAR>(wp_last, W, L) / BN + shift - wn0 + 1 : 0;
    const int wf0 = (wlo_max + BN - 1) / BN + shift;                            // full: wf0 .. +wfc-1
    const unsigned wfc = max(0, (whi_min + 1) / BN + shift - wf0);
    auto needed_of = [&](int j) {
        return j < sn1 || (NC && j >= xn0 && j < nsb) || (unsigned)(j - wn0) < wnc;
    };
    auto full_of = [&](int j) {
        return j < sf1 || (NC && j >= xf0 && j < xf1) || (unsigned)(j - wf0) < wfc;
    };

    // ---- request plan.  Block j's rows come from the summaries (j < nsb) or
    // from the window band; with the band's base pointer shifted back by nsb
    // blocks both are "base + j blocks".  The descriptor covers the block's
    // valid rows only: rows past the end, and every row of a block past the
    // last one, are zeros in LDS without a memory access, so that every wave
    // has the same number of requests in flight at every wait.
    const size_t bg = (size_t)b * a.Hkv + kvh;
    const uintptr_t ks_base = (uintptr_t)a.Ks + bg * (size_t)a.n_chunks * ROWB;
    const uintptr_t vs_base = (uintptr_t)a.Vs + bg * (size_t)a.n_chunks * ROWB;
    const uintptr_t kw_base = (uintptr_t)a.K + bg * (size_t)L * ROWB - (uintptr_t)((intptr_t)shift * BN * ROWB);
    const uintptr_t vw_base = (uintptr_t)a.V + bg * (size_t)L * ROWB - (uintptr_t)((intptr_t)shift * BN * ROWB);
    const int sum_limit = a.n_chunks;
    const int win_limit = L + shift * BN;
    // per lane: instruction i of this wave fills the block's rows
    // (i*NW + wave) * RPI .. + RPI-1 (the swizzle is the same for every i)
    const int d_row = lane * 16 / ROWB, d_pos = (lane * 16 % ROWB) / 16;
    const unsigned dv_off = (wave * RPI + d_row) * ROWB + (d_pos << 4);
    const unsigned dk_off = (wave * RPI + d_row) * ROWB + ((d_pos ^ Cfg::kswz(d_row)) << 4);
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)&lds[0][0][0] + wave * GRP;
    struct Req {
        u32x4 k, v;  // buffer descriptors of the block's rows
    };
    auto request = [&](int j) {
        Req r;
        const bool sum = j < nsb;
        const uintptr_t off = (uintptr_t)j * (BN * ROWB);
        const uintptr_t k = (sum ? ks_base : kw_base) + off;
        const uintptr_t v = (sum ? vs_base : vw_base) + off;
        const int rows = j < nb ? min((sum ? sum_limit : win_limit) - j * BN, BN) : 0;
        r.k = u32x4{(uint32_t)k, (uint32_t)(k >> 32) & 0xffffu, (uint32_t)(rows * ROWB), 0x00020000u};
        r.v = u32x4{(uint32_t)v, (uint32_t)(v >> 32) & 0xffffu, (uint32_t)(rows * ROWB), 0x00020000u};
        return r;
    };
    // part q of a request into stage st: K for even q, V for odd q, instruction q/2
    auto issue_part = [&](const Req& r, int st, int q) {
        const unsigned dst = lds0 + st * 2 * BLK + (q & 1) * BLK + (q >> 1) * NW * GRP;
        const unsigned soff = (q >> 1) * NW * 1024;
        // M0 is the LDS address; one wait state between its write and the load
        asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"((q & 1) ? dv_off : dk_off),
                     "s"((q & 1) ? r.v : r.k), "s"(soff), "{m0}"(dst)
                     : "memory");
    };

    // ---- LDS read offsets ----
    // K fragment dc: score row c32, logical chunk dc*2 + h2.
    // V transposing read (db, kc): the 16-lane group's four score rows
    // i = lane%16 / 4 of half h2, q = 2 (kc%2) (and q + 1), features
    // db*32 + 16 (lane/16 % 2) + 4 (lane%4) ..
    const int k_row = Cfg::key_of(c32 >> 3, c32 & 3) + ((c32 >> 2) & 1) * Cfg::KH;
    const int k0 = Cfg::row_at(k_row) + ((h2 ^ Cfg::kswz(k_row)) << 4);
    const int k1 = k0 ^ 32;
    const int v0 = Cfg::row_at(Cfg::key_of(0, (lane >> 2) & 3) + h2 * Cfg::KH) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    auto kfrag = [&](const unsigned char* ks, int dc) {
        return *reinterpret_cast<const bf16x8*>(ks + ((dc & 1) ? k1 : k0) + (dc >> 1) * 64);
    };
    auto vfrag = [&](const unsigned char* vs, int db, int kc) {
        const unsigned char* vp = vs + v0 + db * 64 + Cfg::row_at(kc * 16);
        const shortx4 lo = lds_read_tr16(reinterpret_cast<const bf16*>(vp));
        const shortx4 hi = lds_read_tr16(reinterpret_cast<const bf16*>(vp + 2 * ROWB));
        return __builtin_bit_cast(
            bf16x8, (short __attribute__((ext_vector_type(8)))){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    };

    floatx16 acc[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[db] = floatx16{};
    // running maximum (log2 units, the same on both lanes of a column) and
    // this lane's part of the denominator: the bf16-rounded weights its
    // column gives to the keys it holds, summed in fp32.  m_neg: -m_run, or 0
    // while m_run is -inf (a column that has seen no key yet), kept beside it
    // so that each step's exponent offset is one add
    float m_run = -INFINITY, m_neg = 0.f, l_run = 0.f;
    floatx16 sc;                     // scores of a block: element i is key key_of(i / 4, i % 4) + h2 KH

    auto lane_max = [&]() {
        float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sc[i]);
        return mx;
    };
    // scores of keys x (within the block, less h2 KH) outside [lo, hi] to -inf
    auto mask_hi = [&](int hi) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int x = Cfg::key_of(i / 4, i % 4);
                sc[i] = x <= hi ? sc[i] : -INFINITY;
            }
    };
    auto mask_lo = [&](int lo) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int x = Cfg::key_of(i / 4, i % 4);
                sc[i] = x >= lo ? sc[i] : -INFINITY;
            }
    };
    // block j straddles an edge of some column's visible range.  The lane's
    // column is recomputed here: kept in a register over the loop it spills,
    // and the reload waits for every request in flight.
    auto mask_block = [&](int j) {
        int l;
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
        const int h2 = l >> 5, n_c = min(p0 + (l & 31), L - 1);
        if (j < nsb) {
            // summary c visible iff c < sum_lo(n) (non-causal: or sum_hi(n) <= c < n_chunks)
            const int rel = j * BN + h2 * Cfg::KH;
            const int hi = sum_lo<VAR>(n_c, W, C) - 1 - rel;
            if constexpr (NC) {
                const int lo = sum_hi<VAR>(n_c, W, C, L) - rel, end = a.n_chunks - rel;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int x = Cfg::key_of(i / 4, i % 4);
                        const bool ok = x <= hi || (x >= lo && x < end);
                        sc[i] = ok ? sc[i] : -INFINITY;
                    }
            } else {
                mask_hi(hi);
            }
        } else {
            const int base = (j - shift) * BN;
            const int rel = base + h2 * Cfg::KH;
            if (base + BN - 1 > whi_min) mask_hi(win_hi<VAR>(n_c, W, L) - rel);
            if (base < wlo_max) mask_lo(win_lo<VAR>(n_c, W, C) - rel);
        }
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

    // ---- prologue: blocks 0 .. AHEAD-1 requested (after the queries) ----
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
        const Req r = request(k);
#pragma unroll
        for (int q = 0; q < NIT; ++q) issue_part(r, k, q);
    }

    // ---- iteration j: S^T(j) = K Q^T, its weights, O^T += V^T P^T(j) ----
    auto iteration = [&](auto ph_tag, int j) {
        constexpr int PH = decltype(ph_tag)::value;  // j mod NS: the stages as constants
        // block j landed (the AHEAD-1 blocks after it may stay in flight);
        // the block requested in this iteration refills the stage of block
        // j-1, whose last reads were before this barrier
        sync_block(std::integral_constant<int, AHEAD - 1>{});
        {
            const Req req = request(j + AHEAD);
#pragma unroll
            for (int q = 0; q < NIT; ++q) issue_part(req, (PH + AHEAD) % NS, q);
        }
        if (!needed_of(j)) return;
        const unsigned char* ks = lds[PH][0];
        const unsigned char* vs = lds[PH][1];
        constexpr int N = NDC + NKC * NDB;  // fragments: NDC of K, then NKC NDB of V^T
        bf16x8 op[kPF + 1];                 // ring of fragments, requested kPF products ahead
        auto load = [&](int k) {
            op[k % (kPF + 1)] = k < NDC ? kfrag(ks, k) : vfrag(vs, (k - NDC) % NDB, (k - NDC) / NDB);
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
        const float bias = j < nsb ? a.log2C : 0.f;
        if (!full_of(j)) mask_block(j);
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
    // instruction writes whole output rows ----
    // Straight from the accumulators a store instruction would write 32
    // pieces of 16 bytes; measured on MI355X (with 16-column pieces of 32
    // bytes), whole rows took the LLM workload from 347 to 331 us, and the
    // training forward with the residual from 434 to 356 us.  Every wave is
    // done with the ring: it holds the staged rows now (a wave's 32 rows with
    // a 16-byte skew between rows, so the fragment writes of one instruction
    // fall in distinct banks).  Stores are non-temporal: nothing here reads
    // the rows again.
    __builtin_amdgcn_s_barrier();
    constexpr int SROW = 2 * D + 16;
    constexpr int LPR = 2 * D / 16;   // lanes per row (16 bytes each)
    constexpr int RPS = 64 / LPR;     // rows per store instruction
    static_assert(NW * 32 * SROW <= NS * 2 * BLK, "staged rows fit in the ring");
    unsigned char* const stg = &lds[0][0][0] + wave * 32 * SROW;
    const float l_sum = xhalf_sum(l_run);
    const float inv = 1.f / l_sum;
    // natural log of the softmax denominator: sum 2^(x - m_run) = l
    if (a.lse && h2 == 0 && col_n < L) a.lse[bh * L + col_n] = (m_run + __builtin_amdgcn_logf(l_sum)) * kLn2;
    // rows p0 + r of this wave's head, r = i RPI + lane / LPR
    auto store_rows = [&](bf16* base) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int i = 0; i < 32 / RPS; ++i) {
            const int r = i * RPS + lane / LPR;
            const u32x4 x = *reinterpret_cast<const u32x4*>(stg + r * SROW + (lane % LPR) * 16);
            const int n = p0 + r;
            bf16* dst = base + (bh * L + (size_t)n) * D + (lane % LPR) * 8;
            if (n < L) __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(dst));
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // accumulator element 4q + i of block db is feature db*32 + 8q + 4 h2 + i
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x2 w = {pack_bf16x2(acc[db][4 * q] * inv, acc[db][4 * q + 1] * inv),
                             pack_bf16x2(acc[db][4 * q + 2] * inv, acc[db][4 * q + 3] * inv)};
            *reinterpret_cast<u32x2*>(stg + c32 * SROW + (db * 32 + 8 * q + 4 * h2) * 2) = w;
        }
    store_rows(static_cast<bf16*>(a.O));
    if constexpr (LO) {
        // residual of the rounding: what the bf16 output lost
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = acc[db][4 * q + i] * inv;
                const u32x2 w = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                const u32x2 r = {pack_bf16x2(v[0] - bf16_lo(w[0]), v[1] - bf16_hi(w[0])),
                                 pack_bf16x2(v[2] - bf16_lo(w[1]), v[3] - bf16_hi(w[1]))};
                *reinterpret_cast<u32x2*>(stg + c32 * SROW + (db * 32 + 8 * q + 4 * h2) * 2) = r;
            }
        store_rows(static_cast<bf16*>(a.O_lo));
    }
}

}  // namespace

template <int D, int VAR, bool LO = false>
void launch_prefill_mfma_var(const PrefillParams& p, hipStream_t stream) {
    // waves per SIMD: D = 128 needs 168 VGPRs (three); D = 64 fits 128 (four)
    hipLaunchKernelGGL((prefill_mfma_kernel<D, D == 64 ? 4 : 3, VAR, LO>), dim3(p.n_tiles), dim3(kNW * 64), 0, stream,
                       p);
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
