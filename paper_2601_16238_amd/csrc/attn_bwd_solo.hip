// dK and dV of the attention backward at D = 65 .. 128, for large launches (dkdv_takes_solo).  The mathematics, the
// statistics, the order of the sums and the form of the stored dS are those of the kernel in attn_bwd.hip, and so are
// the results, bit for bit; the work is divided differently.
//
// There a pair of waves shares 32 keys, and P and dS pass between them through LDS: a slot of 32 query rows moves
// about 1 KB through LDS per key, and the pairs wait for each other at every slot (matrix pipe 58 % busy).  Here four
// waves, one per SIMD, own 64 keys each of a 256-key block and keep a slot's whole chain in their own 512 registers:
// the four 32 x D accumulators in the accumulation half; K and V fragments, scores and dP in the vector half.  Every
// fragment that a wave reads from a slot feeds two MFMAs, one per 32 keys, P and dS go from the scores' registers into
// the next product's operand, and half the LDS traffic is gone.
// With one wave per SIMD nothing hides latencies but the wave's own order.  A slot is 4 KS steps of one fragment and
// its two MFMAs, closed by scheduling fences -- S, dP with most of the exp2, dV with the rest and the first half of
// dS, dK with the second half -- and each step requests the fragment kLead steps further on, across the phases and
// into the next slot.  The barrier that admits the next slot therefore stands before the last phase; a slot's
// transfers are requested after it, kAhead slots ahead, one per step.  (kLead 2 or 4: 1 % slower.)
// us, the kernel alone, storing dS: B=4 H=32 S=4096 D=128 2054 -> 1802 (1.22 PFLOP/s), B=1 H=16 S=16384 causal 1993 ->
// 1882; matrix pipe 68 % busy, at a lower clock than the pairs': the rest is the power that the GPU gives.
#include "attn_device.hpp"
#include "attn_launch.hpp"

namespace attn {

template <int D>
struct DkdvSoloCfg {
    using L = Pieces<D>;
    static constexpr int kWaves = 4, kThreads = kWaves * 64;
    static constexpr int kBlk = kWaves * 64;         // keys owned by the work-group
    static constexpr int kRows = 32;                 // query rows per slot
    static constexpr int kPieces = kRows / L::kRows; // per tensor
    static constexpr int kTensorBytes = L::base(kPieces);    // Q part of a slot; dO follows
    static constexpr int kSlotBytes = 2 * kTensorBytes;
    static constexpr int kStatBytes = 2 * kRows * 4;         // lse2[32], delta[32]
    static constexpr int kAhead = 6, kRing = kAhead + 2;     // (the slot before the one admitted is still read)
    static constexpr int kOffStat = kRing * kSlotBytes;
    static constexpr int kOffZero = kOffStat + kRing * kStatBytes;   // kRows zeros
    static constexpr int kLdsBytes = kOffZero + kRows * 4;
    static constexpr int kDma = 2 * kPieces / kWaves + 1;    // transfers of a slot per wave, the statistics last
    static constexpr int kStage = L::base(kRows / L::kRows); // 32 rows
    static_assert(2 * kPieces % kWaves == 0 && kLdsBytes <= 160 * 1024, "LDS layout");
    static_assert(kWaves * kStage <= (kRing - kAhead) * kSlotBytes, "staging space of the prologue");
};

// x is read only behind this point, which follows the products above it.
__device__ __forceinline__ void after(f32x16 (&x)[2]) { asm volatile("" : "+v"(x[0]), "+v"(x[1])); }

template <int D, int U, bool CAUSAL, bool DS>
__global__ void __launch_bounds__(DkdvSoloCfg<D>::kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
attn_bwd_dkdv_solo_kernel(const BwdArgs a)
{
    using C = DkdvSoloCfg<D>;
    using L = Pieces<D>;
    constexpr int KS = U / 16, DB = U / 32, CPR = D / 8;
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int tid = threadIdx.x, l = tid & 63, r = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = a.S, Sk = a.Sk, Dr = a.Dr;
    const int Hkv = a.H / a.group;
    int bkv, kt;  // causal: key block 0 is the heaviest
    xcd_tile_order<CAUSAL>(blockIdx.x, a.ntile, a.nkv, bkv, kt);
    bkv += a.bkv0;
    const int64_t base_kv = (int64_t)(bkv / Hkv) * a.kv_stride_b + (int64_t)(bkv % Hkv) * a.kv_stride_h;
    const int bh0 = (bkv / Hkv) * a.H + (bkv % Hkv) * a.group;  // first query head of the group
    const int coff = Sk - S;                     // causal: query row i sees keys 0 .. i + coff
    const int k0 = kt * C::kBlk + w * 64;        // first key of this wave
    const int n_slot = (S + C::kRows - 1) / C::kRows;
    // first slot with a row that sees a key of this block (row >= key - coff)
    const int t0 = CAUSAL ? max(0, kt * C::kBlk - coff) / C::kRows : 0;
    const int n_seq = n_slot > t0 ? a.group * (n_slot - t0) : 0;  // slots of all heads of the group

    // ---- global -> LDS streaming (see the kernel above)
    const uint32_t head_bytes = (uint32_t)(((int64_t)(S - 1) * a.stride_s + Dr) * 2);
    const uint32_t row_bytes = (uint32_t)a.stride_s * 2u;
    const uint32_t lds0 = lds_address(smem);
    desc_t Qd, Gd, Wd;  // Q, dO and the row statistics of the query head that is being fetched
    auto set_head = [&](int bh) {
        const int64_t base = (int64_t)(bh / a.H) * a.stride_b + (int64_t)(bh % a.H) * a.stride_h;
        Qd = make_desc(a.Q + base, head_bytes);
        Gd = make_desc(a.dO + base, head_bytes);
        Wd = make_desc(a.delta + (int64_t)bh * 2 * S, (uint32_t)S * 8u);
    };
    const uint32_t voff = L::lane_offset(l, row_bytes, Dr, head_bytes);
    const uint32_t stat_voff = (uint32_t)(h ? r : S + r) * 4u;  // lanes 0-31 lse2, 32-63 delta
    int tf = t0, gqf = 0, rf = 0;  // slot, head and ring position of the next transfers
    // transfer n of the wave's share of slot tf: Q, dO, and the statistics, which every wave requests (the same bytes
    // to the same place), as a branch would end the basic block that the steps below share
    auto dma = [&](int n) __attribute__((always_inline)) {
        if (n == C::kDma - 1) {
            dma4(Wd, lds0 + C::kOffStat + rf * C::kStatBytes, stat_voff, (uint32_t)(tf * C::kRows * 4));
            return;
        }
        const int i = w + n * C::kWaves, tensor = n / (C::kDma / 2), piece = i - tensor * C::kPieces;
        dma16_between(tensor ? Gd : Qd, lds0 + rf * C::kSlotBytes + tensor * C::kTensorBytes + L::base(piece), voff,
                      (uint32_t)((tf * C::kRows + piece * L::kRows) * row_bytes));
    };
    auto dma_slot = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < C::kDma; ++n) dma(n);
    };
    auto step_fetch = [&]() __attribute__((always_inline)) {
        rf = rf + 1 == C::kRing ? 0 : rf + 1;
        ++tf;
    };
    auto wrap_fetch = [&]() __attribute__((always_inline)) {  // to the next query head
        if (tf == n_slot && gqf + 1 < a.group) {
            tf = t0;
            set_head(bh0 + ++gqf);
        }
    };
    // The next slot is in LDS, for every wave: this one's transfers of it are older than those of the kAhead - 1 slots
    // after it (stores in between only make the wait longer).  The transfers behind the barrier go into the ring position
    // of the slot before the current one: its fragments were operands of products that stand before the barrier, so
    // no wave has reads of it left to wait for.
    auto admit = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((C::kAhead - 1) * C::kDma) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // (the first slots before K and V, the others after them: all of it first would keep K and V waiting)
    constexpr int kEarly = 2;
    set_head(bh0);
    if (tid < C::kRows) *(float *)(smem + C::kOffZero + 4 * tid) = 0.f;
#pragma unroll
    for (int i = 0; i < kEarly; ++i) {
        dma_slot();
        step_fetch();
        wrap_fetch();
    }

    // ---- K and V fragments (B operands): block b, lane holds row k0 + 32 b + r, columns 16 ks + 8 h .. +7.  The rows
    // are fetched whole and sorted through ring positions that take a slot only after the first barrier.
    elem8 kf[2][KS], vf[2][KS];
    {
        constexpr int RPI = 64 / CPR, kLoads = 32 / RPI;  // rows per load instruction
        const int lr = l / CPR, lc = l % CPR;
        u32x4 tk[2][kLoads], tv[2][kLoads];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int j = 0; j < kLoads; ++j) {
                const int64_t off = base_kv + (int64_t)min(k0 + 32 * b + RPI * j + lr, Sk - 1) * a.kv_stride_s;
                tk[b][j] = ld_row16(a.K + off, lc * 8, Dr);
                tv[b][j] = ld_row16(a.V + off, lc * 8, Dr);
            }
        char *const mine = smem + C::kAhead * C::kSlotBytes + w * C::kStage;
        auto sort_rows = [&](const u32x4 (&t)[kLoads], elem8 (&f)[KS]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < kLoads; ++j) *(u32x4 *)(mine + L::at(RPI * j + lr, lc)) = t[j];
            asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) f[ks] = *(const elem8 *)(mine + L::at(r, h) + L::step(ks));
            asm volatile("" ::: "memory");
        };
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            sort_rows(tk[b], kf[b]);
            sort_rows(tv[b], vf[b]);
        }
    }
#pragma unroll
    for (int i = kEarly; i < C::kAhead; ++i) {
        dma_slot();
        step_fetch();
        wrap_fetch();
    }

    f32x16 dv[2][DB], dk[2][DB];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) dv[b][db][i] = dk[b][db][i] = 0.f;

    const float c = a.scale_log2e;
    // LDS addresses within a slot: row r's chunk h; transpose reads, rows 4h+e and 8 + 4h+e of the first 32 columns
    int row_at = L::at(r, h), tr_at[2], st_at = C::kOffStat + 16 * h;
#pragma unroll
    for (int j = 0; j < 2; ++j)
        tr_at[j] = L::at(8 * j + 4 * h + ((l & 15) >> 2), 2 * ((l >> 4) & 1) + ((l >> 1) & 1)) + (l & 1) * 8;
    asm volatile("" : "+v"(row_at), "+v"(tr_at[0]), "+v"(tr_at[1]), "+v"(st_at));

    constexpr int kLead = 3, N = 4 * KS;
    static_assert(2 * DB == KS, "phases have one length");
    // fragment of step n of the slot at byte `slot`: rows of Q and dO, then dO^T and Q^T (the first 16 rows of every
    // 32-column block, then the others)
    auto frag = [&](int n, int slot) __attribute__((always_inline)) {
        if (n < 2 * KS)
            return *(const elem8 *)(smem + (n / KS) * C::kTensorBytes + L::step(n % KS) + (row_at + slot));
        const int m = n % KS;
        const char *p = smem + (n < 3 * KS ? C::kTensorBytes : 0) + (m / DB) * L::kRows16 + (m % DB) * L::kBlock;
        return join8(lds_read_tr((const elem *)(p + (tr_at[0] + slot))), lds_read_tr((const elem *)(p + (tr_at[1] + slot))));
    };

    // dS: see the kernel above
    elem *ds_head = DS ? a.dS + ((int64_t)bh0 - (int64_t)a.bkv0 * a.group) * ds_head_blocks(S, Sk, CAUSAL) * kDsBlock : nullptr;
    elem *ds_row = ds_head + (DS ? ds_row_blocks(t0, Sk, coff, CAUSAL) * kDsBlock : 0);
    int ds_len = ds_row_len(t0, Sk, coff, CAUSAL);
    const uint32_t ds_voff = (uint32_t)k0 * 64u + (uint32_t)(((r >> 2) * 16 + h * 4 + (r & 3)) * 16);

    // (after the barrier that admits slot g come the transfers of slot g + kAhead; those of the first two go into the
    // space that K and V were sorted through, whose reads have to be done)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    admit();
    dma_slot();
    step_fetch();
    wrap_fetch();
    int rs = 0, t = t0;  // ring position and rows of the current slot
    int g = 0;
    // wave-uniform: does the slot hold a row that sees some key of the wave
    auto active = [&]() { return !CAUSAL || t * C::kRows + 31 + coff >= k0; };
    auto step_slot = [&]() __attribute__((always_inline)) {
        rs = rs + 1 == C::kRing ? 0 : rs + 1;
        ++t;
        if (DS) {
            ds_row += (CAUSAL ? ds_len : ds_len | 1) * kDsBlock;
            if (CAUSAL) ds_len = ds_row_len(t, Sk, coff, true);
        }
        ++g;
    };
    auto wrap_slot = [&]() __attribute__((always_inline)) {
        wrap_fetch();
        if (t == n_slot) {
            t = t0;
            if (DS) {
                ds_head += ds_head_blocks(S, Sk, CAUSAL) * kDsBlock;
                ds_row = ds_head + ds_row_blocks(t, Sk, coff, CAUSAL) * kDsBlock;
                ds_len = ds_row_len(t, Sk, coff, CAUSAL);
            }
        }
    };
    while (g < n_seq) {
    // (loops of their own: with the two cases as branches of one the compiler spills the accumulators)
    if (CAUSAL)
        for (; g < n_seq && !active(); wrap_slot()) {
            admit();
            dma_slot();
            step_fetch();
            step_slot();
        }
    elem8 lead[kLead];  // the next slot's first fragments
#pragma unroll
    for (int n = 0; n < kLead; ++n) lead[n] = frag(n, rs * C::kSlotBytes);
    for (; g < n_seq && active(); wrap_slot()) {
        const int slot = rs * C::kSlotBytes, next = (rs + 1 == C::kRing ? 0 : rs + 1) * C::kSlotBytes;
        const int q_lo = t * C::kRows;
        const char *const st = smem + rs * C::kStatBytes + st_at;
        f32x16 s[2], dp[2];
        elem8 f[N + kLead], p[2][2], d[2][2];
        rsrc_t row;
        const bool masked = (q_lo + 32 > S) || (CAUSAL && q_lo + coff < k0 + 63);
#pragma unroll
        for (int n = 0; n < kLead; ++n) f[n] = lead[n];
        auto read = [&](int n) __attribute__((always_inline)) { f[n] = n < N ? frag(n, slot) : frag(n - N, next); };
        // the exp2 of score i of block b: numbers 2 i + b
        f32x4 l4[4];
        const char *lse = st;
        float factor = c;
        auto read_lse = [&](int from, int to) __attribute__((always_inline)) {
#pragma unroll
            for (int g4 = from; g4 < to; ++g4) l4[g4] = *(const f32x4 *)(lse + 32 * g4);
        };
        auto exps = [&](int from, int to) __attribute__((always_inline)) {
#pragma unroll
            for (int k = from; k < to; ++k) {
                const int i = k >> 1, b = k & 1;
                s[b][i] = fast_exp2(__builtin_fmaf(s[b][i], factor, -l4[i / 4][i % 4]));
            }
        };
        auto mul = [&](int from, int to) __attribute__((always_inline)) {  // dS = P o (dP - delta)
#pragma unroll
            for (int k = from; k < to; ++k) dp[k & 1][k >> 1] *= s[k & 1][k >> 1];
        };
        auto pack = [](const f32x16 &x, int i0) __attribute__((always_inline)) {
            return pack8(x[i0], x[i0 + 1], x[i0 + 2], x[i0 + 3], x[i0 + 4], x[i0 + 5], x[i0 + 6], x[i0 + 7]);
        };
        auto store = [&](int b, int cc) __attribute__((always_inline)) {
            // (blocks that no row of the slot sees, and keys past the last, lie past the row's end: not stored)
            if (DS) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, d[b][cc]), row, (int)ds_voff, 2048 * b + 128 * cc, 2);
        };
        // Visible rows of block b: >= key - coff - q_lo (causal) and <= S - 1 - q_lo.  What the exp2 take from the scores,
        // the statistics and c is put in the scores' place here, -inf where the row is not visible, whatever its
        // statistics: a row whose LSE is NaN says nothing about keys that it does not see.  The exp2 below then take
        // it times one less zeros: 1.000 .. 1.002 of the time of -inf in the scores alone, whole backward, 1.005 for 104
        // heads on 26 of 1156 rows D = 96.  (Zeros in P behind a branch next to the exp2 of either half: up to 1.010, and
        // 1.018; a loop of its own for such slots: up to 1.006, and 1.023.)
        auto hide = [&]() __attribute__((always_inline)) {
            mfma_settled(s[0], s[1]);
            read_lse(0, 4);
            const int hi = S - 1 - q_lo - 4 * h;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                int lo = (CAUSAL ? k0 + 32 * b + r - coff - q_lo : -64) - 4 * h;
                asm volatile("" : "+v"(lo));  // (not sixteen registers with the loop's constants)
                const unsigned rows = max(hi - lo + 1, 0);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int ro = 8 * (i / 4) + (i % 4);
                    s[b][i] = (unsigned)(ro - lo) < rows ? __builtin_fmaf(s[b][i], c, -l4[i / 4][i % 4]) : -INFINITY;
                }
            }
            lse = smem + C::kOffZero + 16 * h;
            factor = 1.f;
        };
        // ---- S = Q K^T
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks) mfma_v(s[0], f[ks], kf[0][ks]);
            else mfma_v0(s[0], f[ks], kf[0][ks]);
            read(ks + kLead);
            if (ks) mfma_v(s[1], f[ks], kf[1][ks]);
            else mfma_v0(s[1], f[ks], kf[1][ks]);
            if (ks == KS - 2) {  // dP starts from -delta
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int g4 = 0; g4 < 4; ++g4) {
                        const f32x4 d4 = *(const f32x4 *)(st + C::kRows * 4 + 32 * g4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) dp[b][4 * g4 + e] = d4[e];
                        asm volatile("" ::: "memory");
                    }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (masked) hide();
        // ---- dP - delta = dO V^T - delta, with the exp2 of the first 16 rows at least
        constexpr int kFirst = 3 * (KS - 2) < 16 ? 16 : 3 * (KS - 2);  // exp2 before the last step
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            mfma_v(dp[0], f[KS + ks], vf[0][ks]);
            read(KS + ks + kLead);
            mfma_v(dp[1], f[KS + ks], vf[1][ks]);
            if (ks == 0) after(s);
            if (ks == 0) read_lse(0, 2);
            if (ks == KS - 3) read_lse(2, 4);
            if (ks > 0 && ks < KS - 1) exps(kFirst * (ks - 1) / (KS - 2), kFirst * ks / (KS - 2));
            if (ks == KS - 1) { p[0][0] = pack(s[0], 0); p[1][0] = pack(s[1], 0); }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- dV^T += dO^T P, with the other exp2, then the first half of dS
#pragma unroll
        for (int m = 0; m < KS; ++m) {
            const int cc = m / DB, db = m % DB;
            if (m == DB) asm volatile("" : "+v"(dp[0]), "+v"(dp[1]), "+a"(dv[1][0]), "+a"(dv[1][1]));  // (as `after`)
            dv[0][db] = mfma32(f[2 * KS + m], p[0][cc], dv[0][db]);
            read(2 * KS + m + kLead);
            dv[1][db] = mfma32(f[2 * KS + m], p[1][cc], dv[1][db]);
            if (cc == 0) {
                exps(kFirst + (32 - kFirst) * db / DB, kFirst + (32 - kFirst) * (db + 1) / DB);
                if (db == DB - 1) { p[0][1] = pack(s[0], 8); p[1][1] = pack(s[1], 8); }
            } else {
                mul(16 * db / DB, 16 * (db + 1) / DB);
                if (db == DB - 1) { d[0][0] = pack(dp[0], 0); d[1][0] = pack(dp[1], 0); }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        admit();
        row = make_rsrc(ds_row, DS ? (uint32_t)ds_len * (kDsBlock * 2u) : 0u);
        // ---- dK^T += Q^T dS, with the second half of dS
#pragma unroll
        for (int m = 0; m < KS; ++m) {
            const int cc = m / DB, db = m % DB;
            dk[0][db] = mfma32(f[3 * KS + m], d[0][cc], dk[0][db]);
            read(3 * KS + m + kLead);
            dk[1][db] = mfma32(f[3 * KS + m], d[1][cc], dk[1][db]);
            if (m < C::kDma) dma(m);
            if (m == C::kDma) { step_fetch(); step_slot(); }
            if (cc == 0) {
                mul(16 + 16 * db / DB, 16 + 16 * (db + 1) / DB);
                if (db == DB - 1) { d[0][1] = pack(dp[0], 8); d[1][1] = pack(dp[1], 8); }
                if (db < 2) store(db, 0);
            } else if (db < 2) {
                store(db, 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = 0; n < kLead; ++n) lead[n] = f[N + n];
    }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();  // (no transfer in flight, no slot read any more: the LDS is free)

    // The rows leave whole, through a staging area per wave.
    constexpr int RPI = 64 / CPR;  // rows per store instruction
    const int lr = l / CPR, lc = l % CPR;
    char *const stg = smem + w * C::kStage;
    auto rows_out = [&](const f32x16 (&x)[DB], elem *out, float sc, int key0) __attribute__((always_inline)) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *(elem4 *)(stg + L::at(r, 4 * db + g) + 8 * h) =
                    pack4(x[db][4 * g] * sc, x[db][4 * g + 1] * sc, x[db][4 * g + 2] * sc, x[db][4 * g + 3] * sc);
        asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
        for (int j = 0; j < 32 / RPI; ++j) {
            const u32x4 v = *(const u32x4 *)(stg + L::at(RPI * j + lr, lc));
            const int key = key0 + RPI * j + lr;
            if (key < Sk && lc * 8 < Dr) *(u32x4 *)(out + base_kv + (int64_t)key * a.kv_stride_s + lc * 8) = v;
        }
        asm volatile("" ::: "memory");
    };
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        rows_out(dv[b], a.dV, 1.f, k0 + 32 * b);
        rows_out(dk[b], a.dK, a.scale, k0 + 32 * b);
    }
}

template <int D, int U, bool CAUSAL, bool DS>
static int launch_solo(BwdArgs a, hipStream_t st)
{
    using C = DkdvSoloCfg<D>;
    a.ntile = (a.Sk + C::kBlk - 1) / C::kBlk;
    if (hipFuncSetAttribute((const void *)attn_bwd_dkdv_solo_kernel<D, U, CAUSAL, DS>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, C::kLdsBytes) != hipSuccess)
        return -1;
    hipLaunchKernelGGL((attn_bwd_dkdv_solo_kernel<D, U, CAUSAL, DS>), dim3(a.ntile * a.nkv), dim3(C::kThreads),
                       C::kLdsBytes, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int U>
static int launch_solo_u(const BwdArgs &a, bool causal, bool ds, hipStream_t st)
{
    if (causal) return ds ? launch_solo<128, U, true, true>(a, st) : launch_solo<128, U, true, false>(a, st);
    return ds ? launch_solo<128, U, false, true>(a, st) : launch_solo<128, U, false, false>(a, st);
}

int launch_bwd_dkdv_solo(const BwdArgs &a, bool causal, bool ds, hipStream_t st)
{
    constexpr int U = narrow_columns(128);
    return a.Dr <= U ? launch_solo_u<U>(a, causal, ds, st) : launch_solo_u<128>(a, causal, ds, st);
}

}  // namespace attn
