// Fused attention backward for gfx950.  P is recomputed from Q, K and the forward's LSE;
// three kernels on one stream, no atomics, deterministic:
//   1. delta_i = sum_d dO_id O_id                                  (HBM-bound preprocess)
//   2. dK, dV : one work-group per block of keys, loops over query tiles, dK^T / dV^T
//               accumulate in registers                            (4 GEMMs per tile pair)
//   3. dQ     : one work-group per block of queries, loops over key tiles, dQ^T
//               accumulates in registers                           (3 GEMMs per tile pair)
// or, above D = 64 where the workspace holds dS: 1, 2 (which also stores dS), and
//   3b. dQ    : the same from the stored dS                        (1 GEMM per tile pair; waits for dS)
// (2 in attn_bwd_solo.hip for launches that dkdv_takes_solo names)
// or, for calls of few work-groups: 1, then 2 and 3 side by side in one launch.
// With dP = dO V^T and dS = P o (dP - delta):
//   dV = P^T dO,  dK = scale * dS^T Q,  dQ = scale * dS K.
//
// Layout trick shared with the forward: every 32x32 score block is produced in the
// orientation whose accumulator layout IS the B-operand layout of the GEMM that consumes
// it (contraction index enumerated in accumulator order), so P and dS never leave
// registers; the other operand of those GEMMs is a transposed tile read from LDS with
// the LDS transpose read.
//   kernel 2: S = Q K^T (queries x keys): lane owns a key; dV^T += dO^T P, dK^T += Q^T dS
//   kernel 3: S^T = K Q^T (keys x queries): lane owns a query; dQ^T += K^T dS^T
#include "attn_device.hpp"
#include "attn_launch.hpp"

#include <algorithm>
#include <type_traits>

namespace attn {

// ---------------------------------------------------------------------------------------
// 1. Row statistics, fp32, workspace layout [B*H][2][S]: -delta = -rowsum(dO * O), then
// lse2 = LSE * log2(e) (the main kernels run the softmax on exp2).  delta is stored negated
// because the main kernels start the dP = dO V^T accumulation from it, which yields
// dP - delta without a subtraction per element.  D/8 lanes per row,
// 16-byte loads.
// ---------------------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(256) attn_bwd_delta_kernel(const BwdArgs a)
{
    constexpr int LPR = D / 8;          // lanes per row
    constexpr int RPB = 256 / LPR;      // rows per block
    const int64_t rows = (int64_t)a.BH * a.S;
    const int64_t row = (int64_t)blockIdx.x * RPB + threadIdx.x / LPR;
    const int sub = threadIdx.x % LPR;
    float acc = 0.f;
    if (row < rows) {
        const int bh = (int)(row / a.S), i = (int)(row % a.S);
        const int64_t off = (int64_t)(bh / a.H) * a.stride_b + (int64_t)(bh % a.H) * a.stride_h +
                            (int64_t)i * a.stride_s + sub * 8;
        if (sub * 8 < a.Dr) {  // lanes past the tensors' head dimension add nothing
            const elem8 o = as_elem8(ld_global16(a.O + off));
            const elem8 g = as_elem8(ld_global16(a.dO + off));
#pragma unroll
            for (int t = 0; t < 8; ++t) acc += (float)o[t] * (float)g[t];
        }
    }
#pragma unroll
    for (int s = LPR / 2; s >= 1; s >>= 1) acc += __shfl_xor(acc, s);
    if (row < rows && sub == 0) {
        const int64_t bh = row / a.S, i = row % a.S;
        a.delta[(2 * bh) * a.S + i] = -acc;  // negated: it seeds the dP accumulators
        a.delta[(2 * bh + 1) * a.S + i] = a.LSE[row] * kLog2e;
    }
}

// ---------------------------------------------------------------------------------------
// 2. dK, dV.  Work-group = 2P waves = P producers (waves 0 .. P-1) + P consumers (P = 4: two
// waves per SIMD; P = 6 at D = 128: three); it owns 32 P keys and streams the head's Q and dO
// rows through LDS in slots of 32 rows.
// The K/V fragments plus two 32 x D fp32 accumulators do not fit one wave's registers, and a
// wave alternating between the exp-heavy and the accumulate-heavy half cannot overlap them, so
// the halves go to different waves:
//   producer p, slot t:   32 keys; S = Q K^T, dP = dO V^T, P = exp2(c S - lse2),
//                         dS = P o (dP - delta); elem P and dS -> LDS exchange
//   consumer, slot t-1:   64 keys (two producers) and ONE output: even consumers
//                         dV^T += dO^T P, odd ones dK^T += Q^T dS; every transposed
//                         LDS fragment feeds two MFMAs (one per 32-key block)
// Both issue 16 MFMAs per slot (D = 128); the producers' VALU work overlaps the consumers'
// MFMAs on the shared SIMD.  One barrier per slot.
//
// Q/dO slots go global -> LDS directly, kAhead slots ahead, into a ring of kAhead + 2 slots
// (the producer's, the consumer's, and those in flight), requested by the consumers; rows are
// stored unpadded with the 16-byte chunk index XOR-swizzled by the row so that both the
// producer's row reads and the consumer's transpose reads are bank-conflict free.
// ---------------------------------------------------------------------------------------
template <int D, int P>
struct DkdvCfg {
    static constexpr int kPairs = P;                 // producer/consumer pairs: 4, or 6 (three waves per SIMD)
    static constexpr int kWaves = 2 * kPairs;
    static constexpr int kThreads = kWaves * 64;
    static constexpr int kBlk = kPairs * 32;         // keys owned by the work-group
    static constexpr int kRows = 32;                 // query rows per slot
    // slots requested ahead of the producer (a slot of D = 256 is 32 KB: one fewer fits)
    static constexpr int kAhead = D > 128 ? 2 : 3;
    static constexpr int kRing = kAhead + 2;
    static constexpr int kRowBytes = D * 2;
    static constexpr int kTensorBytes = kRows * kRowBytes;   // Q part of a slot; dO follows
    static constexpr int kSlotBytes = 2 * kTensorBytes;
    static constexpr int kStatBytes = 2 * kRows * 4;         // lse2[32], delta[32]
    static constexpr int kXchgBytes = 2 * kPairs * 4 * 1024; // [2][pair][P0,P1,dS0,dS1][64] x 16 B
    static constexpr int kOffStat = kRing * kSlotBytes;
    static constexpr int kOffXchg = kOffStat + kRing * kStatBytes;
    static constexpr int kLdsBytes = kOffXchg + kXchgBytes;
    static constexpr int kDmaPerTensor = kTensorBytes / 1024; // wave-wide 1 KB transfers
    // transfers of a slot that one consumer requests: its share of the Q pieces, then of the dO pieces
    static constexpr int kDmaPerWave = 2 * ((kDmaPerTensor + kPairs - 1) / kPairs);
    // the producer that also fetches the stats (six pairs: waves 2 and 3 are the only producers on
    // their SIMDs, waves 0/4 and 1/5 share one; -0.3..0.6 %)
    static constexpr int kStatWave = kPairs == 6 ? 3 : kPairs - 1;
    static_assert(kOffXchg % 16 == 0 && kLdsBytes <= 160 * 1024, "LDS layout");
};

// Chunk `item` of a K/V head's chunks (see dkdv_split_plan), ordered by key block: its key block and
// its place among that block's chunks.  Every wave finds it for itself, 64 key blocks at a time: a
// prefix sum of the blocks' chunk counts over the lanes.
__device__ __forceinline__ int dkdv_chunks(const BwdArgs &a, int kt, int keys, bool causal)
{
    return max(1, (dkdv_slots(kt, keys, a.group, a.S, a.Sk, causal) + a.dkdv_chunk - 1) / a.dkdv_chunk);
}
__device__ __forceinline__ void dkdv_find_item(const BwdArgs &a, int item, int keys, int n_block, bool causal,
                                               int &kt, int &z)
{
    const int l = threadIdx.x & 63;
    for (int k0 = 0;; k0 += 64) {
        const int c = k0 + l < n_block ? dkdv_chunks(a, k0 + l, keys, causal) : 0;
        int upto = c;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
            const int o = __shfl_up(upto, s);
            if (l >= s) upto += o;
        }
        const int total = __builtin_amdgcn_readlane(upto, 63);
        if (item < total || k0 + 64 >= n_block) {
            const int at = __builtin_ctzll(__builtin_amdgcn_ballot_w64(upto > item) | (1ull << 63));
            kt = k0 + at;
            z = item - (__builtin_amdgcn_readlane(upto, at) - __builtin_amdgcn_readlane(c, at));
            return;
        }
        item -= total;
    }
}

// SPLIT: the work-group takes one chunk of its key block's slots (see dkdv_split_plan).
// DS: the producers also store dS, for attn_bwd_dq_ds_kernel.
// U: columns that the products run over (a multiple of 32 up to D; the others are zeros).
// block, ntile: the work-group among those of the kernel, and its key blocks (or chunks) per K/V head.
template <int D, int U, int P, bool CAUSAL, bool SPLIT, bool DS>
__device__ __forceinline__ void bwd_dkdv(const BwdArgs &a, int block, int ntile)
{
    using C = DkdvCfg<D, P>;
    constexpr int KS = U / 16, DB = U / 32, CPR = D / 8, RB = C::kRowBytes;
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int tid = threadIdx.x, l = tid & 63, r = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool producer = w < C::kPairs;
    const int pair = w < C::kPairs ? w : w - C::kPairs;
    const int S = a.S;
    // The work-group owns 128 keys of one K/V head and sums over the `group` query heads that
    // read it (grouped-query attention; group == 1 is multi-head attention).
    const int Hkv = a.H / a.group;
    int bkv, kt;  // causal: key block 0 is the heaviest
    xcd_tile_order<CAUSAL, D == 64>(block, ntile, a.nkv, bkv, kt);
    bkv += a.bkv0;
    int item = 0, z = 0;  // SPLIT: chunk of the head, and of the key block
    if (SPLIT) {
        item = __builtin_amdgcn_readfirstlane(kt);
        dkdv_find_item(a, item, C::kBlk, (a.Sk + C::kBlk - 1) / C::kBlk, CAUSAL, kt, z);
    }
    const int64_t base_kv = (int64_t)(bkv / Hkv) * a.kv_stride_b + (int64_t)(bkv % Hkv) * a.kv_stride_h;
    const int bh0 = (bkv / Hkv) * a.H + (bkv % Hkv) * a.group;  // first query head of the group

    const int Sk = a.Sk;          // key/value rows; S is the number of query rows
    const int coff = Sk - S;      // causal: query row i sees keys 0 .. i + coff
    const int k0 = kt * C::kBlk + pair * 32;  // first key of this pair
    const int key = k0 + r;
    const int n_slot = (S + C::kRows - 1) / C::kRows;
    // first slot with a row that sees a key of this block (row >= key - coff)
    const int t0 = CAUSAL ? max(0, kt * C::kBlk - coff) / C::kRows : 0;
    const int n_all = n_slot > t0 ? a.group * (n_slot - t0) : 0;  // slots of all heads of the group
    // the slots this work-group walks: n_seq of them from t_first of query head g_first of the group on
    int n_seq = n_all, t_first = t0, g_first = 0;
    if (SPLIT && n_all > 0) {
        const int begin = z * a.dkdv_chunk;
        n_seq = min(a.dkdv_chunk, n_all - begin);
        g_first = begin / (n_slot - t0);
        t_first = t0 + begin % (n_slot - t0);
    }

    // chunk position swizzle: rows 0..15 get 16 distinct values (row reads of 16 lanes hit 16
    // different 16-byte bank groups) and 4 consecutive rows differ in the upper two bits (the
    // 4 rows x 64 bytes of a transpose read spread over all banks)
    auto swz = [](int row) {
        return CPR >= 16 ? (((row & 3) << 2) | ((row >> 2) & 3))
                         : ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));
    };

    // ---- global -> LDS streaming of slot t into ring position rs.  Rows past S-1 lie
    // outside the head's buffer resource and read as zero.
    // Columns Dr..D-1 (head dimensions below the kernel's D) are fetched at an offset past
    // the end of the resource, so they read as zero like everything else outside it.
    const int Dr = a.Dr;
    const uint32_t head_bytes = (uint32_t)(((int64_t)(S - 1) * a.stride_s + Dr) * 2);
    desc_t Qd, Gd;  // Q and dO of the current query head
    rsrc_t Wr;      // its row statistics
    desc_t Wd;      // (DS: issued from assembly, as the compiler would wait for the stores with it)
    const uint32_t lds0 = lds_address(smem);
    auto set_head = [&](int bh) {
        const int64_t base = (int64_t)(bh / a.H) * a.stride_b + (int64_t)(bh % a.H) * a.stride_h;
        Qd = make_desc(a.Q + base, head_bytes);
        Gd = make_desc(a.dO + base, head_bytes);
        if (DS) Wd = make_desc(a.delta + (int64_t)bh * 2 * S, (uint32_t)S * 8u);
        else Wr = make_rsrc(a.delta + (int64_t)bh * 2 * S, (uint32_t)S * 8u);
    };
    const uint32_t row_bytes = (uint32_t)a.stride_s * 2u;
    uint32_t dma_voff[C::kDmaPerWave];
#pragma unroll
    for (int n = 0; n < C::kDmaPerWave; ++n) {
        // (with a pair count that does not divide the pieces the last index wraps; dma_piece skips it)
        const int grp = (pair + (n % (C::kDmaPerWave / 2)) * C::kPairs) % C::kDmaPerTensor;
        const int row = grp * (64 / CPR) + l / CPR;
        const int chunk = (l % CPR) ^ swz(row);
        dma_voff[n] = chunk * 8 < Dr ? row * row_bytes + (chunk << 4) : head_bytes;
    }
    // stats: lanes 0-31 fetch lse2 (second half of the head's workspace), 32-63 delta
    const uint32_t stat_voff = (uint32_t)(h ? r : S + r) * 4u;
    // The Q and dO pieces of a slot are requested by the CONSUMERS, consumer c taking the pieces that
    // pair c is assigned (they have no other vector memory traffic and are the shorter chain of a
    // slot; with the producers issuing them between their MFMAs the kernel was 2-5 % slower), into a
    // ring position that nobody reads before a later barrier: at D <= 128 right after the slot barrier
    // (spread between the consumers' MFMAs the same or up to 2.5 % slower), at D = 256 between their MFMAs
    // (see consume).  Its statistics are requested by one producer, or where the producers store dS, which
    // nobody waits for, by the last pair's consumer.
    auto dma_stat = [&](int t, int rs) __attribute__((always_inline)) {
        if (DS)
            dma4(Wd, lds0 + C::kOffStat + rs * C::kStatBytes, stat_voff, (uint32_t)(t * C::kRows * 4));
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                Wr, (void __attribute__((address_space(3))) *)(smem + C::kOffStat + rs * C::kStatBytes),
                4, (int)stat_voff, t * C::kRows * 4, 0, 0);
    };
    // (With a pair count that does not divide the pieces of a tensor -- six pairs, eight pieces --
    // the first producers take two pieces of each tensor and the others one: `extra`.)
    const bool extra = pair + (C::kDmaPerWave / 2 - 1) * C::kPairs < C::kDmaPerTensor;
    auto dma_piece = [&](int t, int rs, int n) __attribute__((always_inline)) {
        const int tensor = n / (C::kDmaPerWave / 2);  // Q transfers first, then dO
        if (C::kDmaPerTensor % C::kPairs != 0 && n % (C::kDmaPerWave / 2) == C::kDmaPerWave / 2 - 1 && !extra) return;
        const int grp = (pair + (n % (C::kDmaPerWave / 2)) * C::kPairs) % C::kDmaPerTensor;  // 1 KB piece
        const uint32_t dst = lds0 + rs * C::kSlotBytes + tensor * C::kTensorBytes + grp * 1024;
        dma16_between(tensor == 0 ? Qd : Gd, dst, dma_voff[n], (uint32_t)(t * C::kRows * row_bytes));
    };
    auto dma_pieces = [&](int t, int rs) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < C::kDmaPerWave; ++n) dma_piece(t, rs, n);
    };
    // Before slot t is used: this wave's transfers of slot t must have landed (those of the
    // kAhead-1 newer slots may stay in flight) and everyone must be done with slot t-2.
    auto slot_barrier = [&]() {
        if (producer) {
            // (DS: nobody waits for a producer's stores)
            if (DS) wait_vm_and_barrier<63>();
            else if (w == C::kStatWave) wait_vm_and_barrier<C::kAhead - 1>();
            else wait_vm_and_barrier<0>();
        } else if (DS && pair == C::kPairs - 1) {
            constexpr int own = C::kDmaPerTensor % C::kPairs != 0 ? C::kDmaPerWave - 2 : C::kDmaPerWave;
            wait_vm_and_barrier<(C::kAhead - 1) * (own + 1)>();
        } else if (C::kDmaPerTensor % C::kPairs != 0 && !extra) {
            wait_vm_and_barrier<(C::kAhead - 1) * (C::kDmaPerWave - 2)>();
        } else {
            wait_vm_and_barrier<(C::kAhead - 1) * C::kDmaPerWave>();
        }
    };
    // slot and head of the next transfer (both roles keep count: the producers, unless they store dS,
    // for the statistics, the consumers for the rows): the slots of the group's query heads form ONE sequence (head
    // after head, slots t0 .. n_slot-1 of each), so that the ring stays full across the change of
    // head; past the last head the rows lie beyond S and read as zero
    int tf = t_first, gqf = g_first;
    auto advance_fetch = [&]() __attribute__((always_inline)) {
        ++tf;
        if (tf == n_slot && gqf + 1 < a.group) {
            tf = t0;
            set_head(bh0 + ++gqf);
        }
    };
    // wave-uniform: does slot t hold a real row that sees some key of the pair
    auto active = [&](int t) {
        return t * C::kRows < S && (!CAUSAL || t * C::kRows + 31 + coff >= k0);
    };
    auto ring_next = [](int x) { return x + 1 == C::kRing ? 0 : x + 1; };

    elem8 *const Xs = reinterpret_cast<elem8 *>(smem + C::kOffXchg) + pair * 256 + l;

    if (producer) {
        // The statistics of the first kAhead slots are requested before anything else (the
        // consumers request the rows meanwhile).
        if (!DS) {
            set_head(bh0 + g_first);
#pragma unroll
            for (int i = 0; i < C::kAhead; ++i) {
                if (w == C::kStatWave) dma_stat(tf, i);
                advance_fetch();
            }
        }
        // K and V fragments (B operands): lane holds K[key][16ks + 8h .. +7].
        // The 32 rows are fetched whole (an instruction covers 64 / (D/8) consecutive rows instead
        // of 16 bytes of each of 32) and sorted into the fragment layout through LDS that nobody
        // else touches before the first barrier of the slot loop: at D <= 128 the producer's own
        // two slices of the exchange buffer (2 x 4 KB: rows 0-15 and 16-31), at D = 256 (two
        // producers, 16 KB each) the two tensors of the first ring slot that no transfer has been
        // issued for; chunks XOR-swizzled by the row like the slots.
        elem8 kf[KS], vf[KS];
        {
            constexpr int RPI = 64 / CPR, kLoads = 32 / RPI;  // rows per load instruction
            const int lr = l / CPR, lc = l % CPR;
            u32x4 tk[kLoads], tv[kLoads];
#pragma unroll
            for (int j = 0; j < kLoads; ++j) {
                const int64_t off = base_kv + (int64_t)min(k0 + RPI * j + lr, Sk - 1) * a.kv_stride_s;
                tk[j] = ld_row16(a.K + off, lc * 8, Dr);
                tv[j] = ld_row16(a.V + off, lc * 8, Dr);
            }
            static_assert(D <= 128 || C::kPairs <= 2, "staging space of the producers");
            char *const mine = D <= 128 ? smem + C::kOffXchg + pair * 4096
                                        : smem + C::kAhead * C::kSlotBytes + pair * C::kTensorBytes;
            auto slot_of = [&](int row, int chunk) {  // byte offset of a chunk of a staged row
                return D <= 128 ? (row >> 4) * (C::kPairs * 4096) + (row & 15) * RB + ((chunk ^ swz(row & 15)) << 4)
                                : row * RB + ((chunk ^ swz(row)) << 4);
            };
            auto sort_rows = [&](const u32x4 (&t)[kLoads], elem8 (&f)[KS]) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < kLoads; ++j) *(u32x4 *)(mine + slot_of(RPI * j + lr, lc)) = t[j];
                asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) f[ks] = *(const elem8 *)(mine + slot_of(r, 2 * ks + h));
                asm volatile("" ::: "memory");
            };
            sort_rows(tk, kf);
            sort_rows(tv, vf);
        }
        // make sure no register load is counted among the streamed transfers any more
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const float c = a.scale_log2e;
        const int lane_off = r * RB + ((h ^ swz(r)) << 4);  // chunk 2ks+h of row r: ^ (ks*32)

        int rs = 0;  // ring position of the current slot
        int t = t_first;  // its rows: slot t of the current head
        // DS: the 2 KB block of (slot, 32 keys), see ds_row_blocks; the row of blocks of slot t starts at
        // ds_row and has ds_len of them.  One store holds 16 queries of every key: 128-byte runs.
        elem *ds_head = DS ? a.dS + ((int64_t)(bh0 + g_first) - (int64_t)a.bkv0 * a.group) *
                                        ds_head_blocks(S, Sk, CAUSAL) * kDsBlock : nullptr;
        elem *ds_row = ds_head + (DS ? ds_row_blocks(t, Sk, coff, CAUSAL) * kDsBlock : 0);
        int ds_len = ds_row_len(t, Sk, coff, CAUSAL);
        const uint32_t ds_voff = (uint32_t)k0 * 64u + (uint32_t)(((r >> 2) * 16 + h * 4 + (r & 3)) * 16);
        constexpr int kNt = 2;  // non-temporal (plain: dQ 3 .. 10 % longer)
        auto ds_rsrc = [&]() __attribute__((always_inline)) {
            return make_rsrc(ds_row, DS ? (uint32_t)ds_len * (kDsBlock * 2u) : 0u);
        };
        auto store_ds = [&](rsrc_t row, elem8 d0, elem8 d1) __attribute__((always_inline)) {
            // (blocks that no row of the slot sees, and keys past the last, lie past the row's end: not stored)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, d0), row, (int)ds_voff, 0, kNt);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, d1), row, (int)ds_voff, 128, kNt);
        };
        auto next_slot = [&]() __attribute__((always_inline)) {
            if (!DS) advance_fetch();
            rs = ring_next(rs);
            ++t;
            if (DS) {
                ds_row += (CAUSAL ? ds_len : ds_len | 1) * kDsBlock;
                if (CAUSAL) ds_len = ds_row_len(t, Sk, coff, true);
            }
        };
        for (int g = 0; g < n_seq; ++g) {
            slot_barrier();
            int rd = rs + C::kAhead;
            rd = rd >= C::kRing ? rd - C::kRing : rd;
            if (!DS && w == C::kStatWave) dma_stat(tf, rd);
            if (active(t)) {
                const char *Qt = smem + rs * C::kSlotBytes;
                const float *st = reinterpret_cast<const float *>(smem + C::kOffStat + rs * C::kStatBytes);
                const int q_lo = t * C::kRows;
                const rsrc_t row = ds_rsrc();
                f32x16 s, dp;
                // register i <-> query row q_lo + 8*(i/4) + 4h + i%4.  The dP accumulator starts
                // from -delta of its row, so that it ends as dP - delta.  The lane's key is fixed;
                // P = exp2(c S - lse2) per row.
                const bool masked = (q_lo + 32 > S) || (CAUSAL && q_lo + coff < k0 + 31);
                // P = 0 unless the row is visible: row offsets >= key - coff - q_lo (causal), <= S - 1 - q_lo.  (P, not S:
                // a row whose statistics are NaN says nothing about keys that it does not see.)
                auto hide = [&]() __attribute__((always_inline)) {
                    const int lo = (CAUSAL ? key - coff - q_lo : -64) - 4 * h;
                    const int hi = S - 1 - q_lo - 4 * h;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int ro = 8 * (i / 4) + (i % 4);
                        if (ro < lo || ro > hi) s[i] = 0.f;
                    }
                };
                if constexpr (D > 128) {
                    // One wave per SIMD: the scores in the vector half of the register file, the next slot's scalar work
                    // between the MFMAs of S: in this order P is packed while the last MFMA of dP runs, and
                    // nothing but dS is left behind it.
                    constexpr int kAhead = 4;
                    elem8 f[2 * KS];
                    auto fetch = [&](int n) __attribute__((always_inline)) {
                        if (n < 2 * KS)
                            f[n] = *(const elem8 *)(Qt + (n / KS) * C::kTensorBytes + (lane_off ^ ((n % KS) * 32)));
                    };
                    f32x4 l4[4];
#pragma unroll
                    for (int n = 0; n < kAhead; ++n) fetch(n);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        if (ks) mfma_v(s, f[ks], kf[ks]);
                        else mfma_v0(s, f[ks], kf[ks]);
                        fetch(ks + kAhead);
                        if (ks == 2) next_slot();
                        if (ks == KS - 4) {
#pragma unroll
                            for (int g4 = 0; g4 < 4; ++g4) {
                                l4[g4] = *(const f32x4 *)(st + 8 * g4 + 4 * h);
                                const f32x4 d4 = *(const f32x4 *)(st + 32 + 8 * g4 + 4 * h);
#pragma unroll
                                for (int e = 0; e < 4; ++e) dp[4 * g4 + e] = d4[e];
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        mfma_v(dp, f[KS + ks], vf[ks]);
                        fetch(KS + ks + kAhead);
                        if (ks == 1) asm volatile("" : "+v"(s));  // (read two products after its last, see mfma_v)
#pragma unroll
                        for (int i = exps_before(ks, KS); i < exps_before(ks + 1, KS); ++i)
                            s[i] = fast_exp2(__builtin_fmaf(s[i], c, -l4[i / 4][i % 4]));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (masked) hide();
                    elem8 *x = Xs + (g & 1) * (C::kPairs * 256);
                    x[0] = pack8(s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7]);
                    x[64] = pack8(s[8], s[9], s[10], s[11], s[12], s[13], s[14], s[15]);
                    mfma_settled(dp);
                } else {
                    f32x16 zero, nd;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 d4 = *(const f32x4 *)(st + 32 + 8 * g + 4 * h);
#pragma unroll
                        for (int e = 0; e < 4; ++e) nd[4 * g + e] = d4[e];
                    }
#pragma unroll
                    for (int i = 0; i < 16; ++i) zero[i] = 0.f;
                    {
                        // Every MFMA is a step of its own, closed by a scheduling fence, with the read of
                        // the fragment four MFMAs further on (the compiler reads a fragment right
                        // before its MFMA and waits); S first, so that its exp2 run next to the
                        // MFMAs of dP.  us: B=4 H=16 S=4096 D=256 causal 1216 -> 1118 (with the
                        // consumers' steps), B=1 H=16 S=4096 D=128 causal 142 -> 135 (S=16384 the same within noise);
                        // two or six MFMAs ahead are the same
                        constexpr int kAhead = 4;
                        elem8 f[2 * KS];
                        auto fetch = [&](int n) __attribute__((always_inline)) {
                            if (n < 2 * KS)
                                f[n] = *(const elem8 *)(Qt + (n / KS) * C::kTensorBytes + (lane_off ^ ((n % KS) * 32)));
                        };
                        f32x4 l4[4];
#pragma unroll
                        for (int g = 0; g < 4; ++g) l4[g] = *(const f32x4 *)(st + 8 * g + 4 * h);
#pragma unroll
                        for (int n = 0; n < kAhead; ++n) fetch(n);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            s = mfma32(f[ks], kf[ks], ks ? s : zero);
                            fetch(ks + kAhead);
                            __builtin_amdgcn_sched_barrier(0);
                        }
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            dp = mfma32(f[KS + ks], vf[ks], ks ? dp : nd);
                            fetch(KS + ks + kAhead);
#pragma unroll
                            for (int i = exps_before(ks, KS); i < exps_before(ks + 1, KS); ++i)
                                s[i] = fast_exp2(__builtin_fmaf(s[i], c, -l4[i / 4][i % 4]));
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    if (masked) hide();
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) dp[i] *= s[i];  // dS = P o (dP - delta)
                elem8 *x = Xs + (g & 1) * (C::kPairs * 256);
                if (D <= 128) {
                    x[0] = pack8(s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7]);
                    x[64] = pack8(s[8], s[9], s[10], s[11], s[12], s[13], s[14], s[15]);
                }
                const elem8 d0 = pack8(dp[0], dp[1], dp[2], dp[3], dp[4], dp[5], dp[6], dp[7]);
                const elem8 d1 = pack8(dp[8], dp[9], dp[10], dp[11], dp[12], dp[13], dp[14], dp[15]);
                x[128] = d0;
                x[192] = d1;
                if (DS) store_ds(D > 128 ? row : ds_rsrc(), d0, d1);
            } else if (D > 128) {
                next_slot();
            }
            if (D <= 128) next_slot();
            if (t == n_slot) {
                t = t0;
                if (DS) {
                    ds_head += ds_head_blocks(S, Sk, CAUSAL) * kDsBlock;
                    ds_row = ds_head + ds_row_blocks(t, Sk, coff, CAUSAL) * kDsBlock;
                    ds_len = ds_row_len(t, Sk, coff, CAUSAL);
                }
            }
        }
        wait_vm_and_barrier<DS ? 63 : 0>();  // the consumers' last slot
    } else {
        // Consumers.  Wave 4+cw accumulates ONE output for the 64 keys of two producers
        // (2*(cw>>1) and the next): dV^T += dO^T P for even cw, dK^T += Q^T dS for odd cw.
        // Each transposed fragment read from LDS then feeds two MFMAs (one per key block),
        // which halves the consumers' LDS traffic against one wave per 32 keys and both
        // outputs.
        const int cw = w - C::kPairs;
        const int kind = cw & 1, half = cw >> 1;
        const int kA = kt * C::kBlk + half * 64, kB = kA + 32;  // first keys of the two blocks
        f32x16 acc[2][DB];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[kb][db][i] = 0.f;
        // transpose-read addresses: the 16-lane group reads rows 4h+e (e = 0..3), +8 for the
        // second read, 64 bytes of d block db per row; byte offset within a slot tensor
        int tr_off[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = 8 * j + 4 * h + ((l & 15) >> 2);
            const int chunk = 2 * ((l >> 4) & 1) + ((l >> 1) & 1);
            tr_off[j] = row * RB + ((chunk ^ swz(row)) << 4) + (l & 1) * 8;
        }
        // wave-uniform: does slot t hold a real row that sees some key of the block at kfirst
        auto block_active = [&](int t, int kfirst) {
            return t * C::kRows < S && (!CAUSAL || t * C::kRows + 31 + coff >= kfirst);
        };
        const elem8 *const Xc = reinterpret_cast<const elem8 *>(smem + C::kOffXchg) +
                                 (2 * half) * 256 + kind * 128 + l;
        // (D > 128: with the transfers of slot tf into ring position rd between the products, if `fetch`)
        auto consume = [&](int t, int g, int rs, int rd, auto fetch) {
            const bool actA = block_active(t, kA), actB = block_active(t, kB);
            if (!actA) {  // kA < kB: then the second block is not active either
                if (D > 128 && fetch()) dma_pieces(tf, rd);
                return;
            }
            const char *Tt = smem + rs * C::kSlotBytes + (kind ? 0 : C::kTensorBytes);
            const elem8 *x = Xc + (g & 1) * (C::kPairs * 256);
            const elem8 opA[2] = {x[0], x[64]};
            // Slots above the diagonal of the second key block: its producer wrote nothing,
            // so the block gets zero operands (a second code path without its MFMAs makes
            // the compiler spill the accumulators).
            elem8 opB[2];
#pragma unroll
            for (int i = 0; i < 8; ++i) opB[0][i] = opB[1][i] = 0;
            if (actB) { opB[0] = x[256]; opB[1] = x[256 + 64]; }
            // MFMA pair n: 16-row step n / DB, d block n % DB (chunks 4db..4db+3: flips bits 6.. of the
            // swizzled offset)
            auto frag = [&](int n) __attribute__((always_inline)) {
                const int o = (n / DB) * 16 * RB, x = (n % DB) << 6;
                return join8(lds_read_tr((const elem *)(Tt + ((tr_off[0] ^ x) + o))),
                             lds_read_tr((const elem *)(Tt + ((tr_off[1] ^ x) + o))));
            };
            if constexpr (D > 128) {
                // one wave per SIMD: fenced steps as in the producers (no gain at D <= 128), with the
                // transfers between them (in front of them they cost the D = 256 consumers 300 cycles a slot)
                constexpr int kAhead = 4;
                elem8 T[2 * DB];
#pragma unroll
                for (int n = 0; n < kAhead; ++n) T[n] = frag(n);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int n = 0; n < 2 * DB; ++n) {
                    acc[0][n % DB] = mfma32(T[n], opA[n / DB], acc[0][n % DB]);
                    if (n + kAhead < 2 * DB) T[n + kAhead] = frag(n + kAhead);
                    acc[1][n % DB] = mfma32(T[n], opB[n / DB], acc[1][n % DB]);
                    constexpr int kN = fetch() ? C::kDmaPerWave : 0;
#pragma unroll
                    for (int i = kN * n / (2 * DB); i < kN * (n + 1) / (2 * DB); ++i) dma_piece(tf, rd, i);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int n = 0; n < 2 * DB; ++n) {
                    const elem8 T = frag(n);
                    acc[0][n % DB] = mfma32(T, opA[n / DB], acc[0][n % DB]);
                    acc[1][n % DB] = mfma32(T, opB[n / DB], acc[1][n % DB]);
                }
            }
        };

        // the rows of the first kAhead slots
        set_head(bh0 + g_first);
#pragma unroll
        for (int i = 0; i < C::kAhead; ++i) {
            dma_pieces(tf, i);
            if (DS && pair == C::kPairs - 1) dma_stat(tf, i);
            advance_fetch();
        }
        int rs = 0;  // ring position of the producers' slot; the consumers' is one behind
        int t = t_first, tp = t_first;  // rows of the producers' slot and of the one before it
        for (int g = 0; g < n_seq; ++g) {
            slot_barrier();
            // slot g + kAhead goes into the ring position that slot g - 2 has left
            int rd = rs + C::kAhead;
            rd = rd >= C::kRing ? rd - C::kRing : rd;
            if (D <= 128 || g == 0) dma_pieces(tf, rd);
            auto requested = [&]() __attribute__((always_inline)) {
                if (DS && pair == C::kPairs - 1) dma_stat(tf, rd);
                advance_fetch();
            };
            if (D <= 128) requested();
            if (g > 0) consume(tp, g - 1, rs == 0 ? C::kRing - 1 : rs - 1, rd, std::true_type());
            if (D > 128) requested();
            rs = ring_next(rs);
            tp = t;
            if (++t == n_slot) t = t0;
        }
        wait_vm_and_barrier<0>();
        if (n_seq > 0) consume(tp, n_seq - 1, rs == 0 ? C::kRing - 1 : rs - 1, 0, std::false_type());

        // The accumulators hold 4 consecutive columns of one key per register group: stored
        // directly, every instruction writes 8-byte pieces of 32 rows (32 such stores per wave).
        // The rows of a key block go through LDS instead and leave whole, 16 bytes per lane: each
        // consumer takes one tensor's worth of a ring slot other than the last one, which other
        // consumers may still be reading (the producers have issued their last transfer and all
        // of them have landed), in the slots' swizzled row layout.
        elem *const out = kind ? a.dK : a.dV;
        const float sc = kind ? a.scale : 1.f;
        const int64_t row_stride = D > 128 ? in_sgpr(a.kv_stride_s) : a.kv_stride_s;
        {
            constexpr int RPI = 64 / CPR;  // rows per store instruction
            const int last = rs == 0 ? C::kRing - 1 : rs - 1;  // ring position of the last slot
            int slot = cw >> 1;
            slot += slot >= last ? 1 : 0;
            char *stg = smem + slot * C::kSlotBytes + (cw & 1) * C::kTensorBytes;
            const int lr = l / CPR, lc = l % CPR;
            if (SPLIT && n_all > a.dkdv_chunk) {
                // unscaled fp32 partial of this chunk; an fp32 row is twice as long as the
                // staging area's, so it goes in two halves
                float *const part = a.dKVpart + ((int64_t)(bkv * a.dkdv_items + item) * 2 + kind) * (C::kBlk * D);
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int hp = 0; hp < 2; ++hp) {  // (columns past U: anything; the merge drops them)
                        constexpr int HB = D / 64;
#pragma unroll
                        for (int db = hp * HB; db < (hp + 1) * HB && db < DB; ++db)
#pragma unroll
                            for (int g = 0; g < 4; ++g) {
                                f32x4 v;
#pragma unroll
                                for (int e = 0; e < 4; ++e) v[e] = acc[kb][db][4 * g + e];
                                const int chunk = (db % HB) * 8 + 2 * g + h;
                                *(f32x4 *)(stg + r * RB + ((chunk ^ swz(r)) << 4)) = v;
                            }
                        asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
                        for (int j = 0; j < 32 / RPI; ++j) {
                            const int row = RPI * j + lr;
                            const f32x4 v = *(const f32x4 *)(stg + row * RB + ((lc ^ swz(row)) << 4));
                            const int okey = half * 64 + 32 * kb + row;
                            if (kt * C::kBlk + okey < Sk)
                                *(f32x4 *)(part + okey * D + hp * (D / 2) + lc * 4) = v;
                        }
                        asm volatile("" ::: "memory");
                    }
                return;
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        *(elem4 *)(stg + r * RB + (((4 * db + g) ^ swz(r)) << 4) + 8 * h) =
                            pack4(acc[kb][db][4 * g] * sc, acc[kb][db][4 * g + 1] * sc,
                                  acc[kb][db][4 * g + 2] * sc, acc[kb][db][4 * g + 3] * sc);
                asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
                for (int j = 0; j < 32 / RPI; ++j) {
                    const int row = RPI * j + lr;
                    const u32x4 v = *(const u32x4 *)(stg + row * RB + ((lc ^ swz(row)) << 4));
                    const int okey = kA + 32 * kb + row;
                    if (okey < Sk && lc * 8 < Dr)
                        *(u32x4 *)(out + base_kv + (int64_t)okey * row_stride + lc * 8) = v;
                }
                asm volatile("" ::: "memory");
            }
        }
    }
}

template <int D, int U, int P, bool CAUSAL, bool SPLIT, bool DS>
__global__ void __launch_bounds__(P * 128) __attribute__((amdgpu_waves_per_eu(P >= 4 ? P / 2 : 1)))
attn_bwd_dkdv_kernel(const BwdArgs a)
{
    bwd_dkdv<D, U, P, CAUSAL, SPLIT, DS>(a, blockIdx.x, a.ntile);
}

// Sum of the partial dK and dV of the key blocks that were cut into several chunks, in the order of
// the chunks, dK times scale, rounded.  A work-group owns 1024 / D keys of one block and tensor,
// a thread 4 consecutive columns of one key; HBM-bound and small.
template <int D, bool CAUSAL>
__device__ __forceinline__ void bwd_dkdv_merge(const BwdArgs &a, int block, int kind)
{
    constexpr int keys = dkdv_split_keys(D), kRows = 1024 / D, kSub = keys / kRows;
    const int n_block = (a.Sk + keys - 1) / keys;
    const int sub = block % kSub;
    const int kt = (block / kSub) % n_block, bkv = block / (kSub * n_block);
    const int n = dkdv_chunks(a, kt, keys, CAUSAL);
    if (n < 2) return;  // (written by its one work-group)
    int first = 0;  // the block's first chunk: the chunks of the blocks before it, summed over the lanes
    for (int k = threadIdx.x & 63; k < kt; k += 64) first += dkdv_chunks(a, k, keys, CAUSAL);
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) first += __shfl_xor(first, s);
    const int row = sub * kRows + threadIdx.x / (D / 4), d0 = (threadIdx.x % (D / 4)) * 4;
    const int key = kt * keys + row;
    if (key >= a.Sk || d0 >= a.Dr) return;
    const float *part = a.dKVpart + ((int64_t)(bkv * a.dkdv_items + first) * 2 + kind) * (keys * D) + row * D + d0;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int z0 = 0; z0 < n; z0 += 4) {  // four chunks' loads in flight together
        f32x4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            v[k] = *(const f32x4 *)(part + (int64_t)(z0 + k < n ? z0 + k : z0) * (2 * keys * D));
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (z0 + k < n) {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += v[k][e];
            }
    }
    const int Hkv = a.H / a.group;
    const float sc = kind ? a.scale : 1.f;
    elem *out = (kind ? a.dK : a.dV) + (int64_t)(bkv / Hkv) * a.kv_stride_b + (int64_t)(bkv % Hkv) * a.kv_stride_h +
                (int64_t)key * a.kv_stride_s + d0;
    *(elem4 *)out = pack4(acc[0] * sc, acc[1] * sc, acc[2] * sc, acc[3] * sc);
}

template <int D, bool CAUSAL>
__global__ void __launch_bounds__(256) attn_bwd_dkdv_merge_kernel(const BwdArgs a)
{
    bwd_dkdv_merge<D, CAUSAL>(a, blockIdx.x, blockIdx.y);
}

// ---------------------------------------------------------------------------------------
// 3. dQ.  Work-group = NW waves, wave = 32 queries (Q, dO fragments and the 32 x D fp32
// accumulator in registers), loop over key tiles of 64 rows.  K and V tiles go global -> LDS
// directly, two tiles ahead, into a ring of three.
//
// LDS layout of a tile tensor: pieces (see Pieces).  The address of a fragment is a per-lane constant
// plus compile-time terms for the contraction step, the d block, the sub-tile and the ring position: with
// the loop unrolled over the ring positions every LDS access is one register plus an immediate offset and
// the loop has no vector instruction for addressing (it had 16 per sub-tile with a row-major,
// XOR-swizzled tile).
// ---------------------------------------------------------------------------------------
template <int D, int NW>
struct DqCfg {
    static constexpr int kThreads = NW * 64;
    static constexpr int kBlk = NW * 32;             // queries owned by the work-group
    static constexpr int kTile = D > 128 ? 32 : 64;  // keys per tile (a ring of three must fit the LDS)
    static constexpr int kSub = kTile / 32;          // 32-key sub-tiles per tile
    static constexpr int kRing = 3;
    static constexpr int kRowBytes = D * 2;
    using L = Pieces<D>;
    static constexpr int kPieceRows = L::kRows;               // rows one 1 KB transfer fills
    static constexpr int kPieces = kTile / kPieceRows;        // per tensor
    static constexpr int kTensorBytes = L::base(kPieces);        // K part of a tile; V follows
    static constexpr int kTileBytes = 2 * kTensorBytes;
    // D <= 128: the rows of Q, dO and O reach the fragment registers through a per-wave staging
    // area of 32 rows in the tile tensors' layout (see the kernel's prologue).  The areas start
    // at ring position 2, which is free until the first barrier of the key loop.
    static constexpr bool kStageRows = true;
    static constexpr int kStageBytes = kStageRows ? L::base(32 / kPieceRows) : 0;
    static constexpr int kLdsBytes = kRing * kTileBytes > 2 * kTileBytes + NW * kStageBytes
                                         ? kRing * kTileBytes : 2 * kTileBytes + NW * kStageBytes;
    static constexpr int kDmaPerTile = 2 * kPieces;           // wave-wide 1 KB transfers
    static constexpr int kDmaPerWave = (kDmaPerTile + NW - 1) / NW;
    static constexpr int kRows16 = L::kRows16;                // 16 rows further
    static_assert(16 % kPieceRows == 0, "sub-tiles start at piece boundaries");
    static_assert(kLdsBytes <= 160 * 1024, "LDS budget of a gfx950 CU exceeded");
};

// A wave's 32 finished dQ rows from row q0 on (accumulators dq, in the layout of the MFMA), scaled, to
// memory through its staging area stg.
template <typename C, int D, int U>
__device__ __forceinline__ void dq_rows_out(const BwdArgs &a, f32x16 (&dq)[U / 32], char *stg, int64_t base, int q0, int l)
{
    constexpr int DB = U / 32, CPR = D / 8, RPI = 64 / CPR;
    const int r = l & 31, h = l >> 5, lr = l / CPR, lc = l % CPR, S = a.S, Dr = a.Dr;
    const int qc = min(q0 + r, S - 1);
    auto at = [](int row, int chunk) { return Pieces<D>::at(row, chunk); };
    if (U == D && a.rope_cos) {
        // Q was rotated before the forward: what has been accumulated is the gradient of the
        // rotated rows; the gradient of the unrotated ones is its image under the transpose of
        // the rotation (head dimension == D only; column d pairs with d + D/2, i.e. d block db
        // with db + DB/2, same register).
        const int64_t pos = (int64_t)(qc + a.rope_pos0) * (D / 2);
#pragma unroll
        for (int db = 0; db < DB / 2; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 c4 = *(const f32x4 *)(a.rope_cos + pos + 32 * db + 8 * g + 4 * h);
                const f32x4 s4 = *(const f32x4 *)(a.rope_sin + pos + 32 * db + 8 * g + 4 * h);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float y1 = dq[db][4 * g + e], y2 = dq[db + DB / 2][4 * g + e];
                    dq[db][4 * g + e] = __builtin_fmaf(y1, c4[e], y2 * s4[e]);
                    dq[db + DB / 2][4 * g + e] = __builtin_fmaf(y2, c4[e], -(y1 * s4[e]));
                }
            }
    }
    {
        // The accumulator holds 4 consecutive columns of one row per register group: stored
        // directly, every instruction writes 8-byte pieces of 32 rows.  The rows go through the
        // wave's staging area stg instead and leave whole, 16 bytes per lane.  (From dQ's ring the areas that
        // lie in ring position 2 have moved to the position that the last two tiles did not use: other
        // waves may still be reading those.)
        const float sc = a.scale;
        const int64_t row_stride = D > 128 ? in_sgpr(a.stride_s) : a.stride_s;
        elem *const out = (D > 128 ? in_sgpr(a.dQ) : a.dQ) + base;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *(elem4 *)(stg + at(r, 4 * db + g) + 8 * h) =
                    pack4(dq[db][4 * g] * sc, dq[db][4 * g + 1] * sc, dq[db][4 * g + 2] * sc, dq[db][4 * g + 3] * sc);
        asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
        for (int j = 0; j < 32 / RPI; ++j) {
            const u32x4 v = *(const u32x4 *)(stg + at(RPI * j + lr, lc));
            const int row = q0 + RPI * j + lr;
            if (row < S && lc * 8 < Dr) *(u32x4 *)(out + (int64_t)row * row_stride + lc * 8) = v;
        }
    }
}

// block, ntile: the work-group among those of a split, and its query tiles per head; part: the split.
template <int D, int U, int NW, bool CAUSAL, bool SPLIT>
__device__ __forceinline__ void bwd_dq(const BwdArgs &a, int block, int ntile, int part)
{
    using C = DqCfg<D, NW>;
    using L = Pieces<D>;
    constexpr int KS = U / 16, DB = U / 32, PR = C::kPieceRows;
    // A wave's transfers per tile are issued between the MFMAs of the tile's first step instead of
    // in a burst after the barrier wherever their number divides that of the MFMAs (measured at
    // D = 128: long causal shapes 2-3 % faster)
    constexpr bool kBetween = KS % C::kDmaPerWave == 0 || (U < D && KS >= C::kDmaPerWave);
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int tid = threadIdx.x, l = tid & 63, r = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = a.S;
    int bh, rank;
    xcd_tile_order<CAUSAL, D == 64 && NW == 4, (D == 64 && NW == 4 ? 8 : 4)>(block, ntile, a.BH, bh, rank);
    const int qt = CAUSAL ? ntile - 1 - rank : rank;  // heaviest first
    const int64_t base = (int64_t)(bh / a.H) * a.stride_b + (int64_t)(bh % a.H) * a.stride_h;
    // grouped-query heads: query head h reads K/V head h / group
    const int64_t base_kv = (int64_t)(bh / a.H) * a.kv_stride_b +
                            (int64_t)((bh % a.H) / a.group) * a.kv_stride_h;

    const int q0 = qt * C::kBlk + w * 32;
    const int q = q0 + r;
    const int qc = q < S ? q : S - 1;
    // Keys seen by this work-group: all Sk of them, or one split's range (then K and V are
    // simply re-based to the range and the causal offset moves with them; the row statistics
    // belong to the whole row, so the partial dQ of the ranges just add up).
    int Sk = a.Sk;      // key/value rows; S is the number of query rows
    int coff = Sk - S;  // causal: query row i sees keys 0 .. i + coff
    int64_t kv_first = 0;
    if (SPLIT) {
        const int k_begin = part * a.dq_kps;  // < Sk by the launcher's plan
        kv_first = (int64_t)k_begin * a.kv_stride_s;
        Sk = min(Sk - k_begin, a.dq_kps);
        coff -= k_begin;
    }
    const int q0e = q0 + coff;
    const int q_end = min(S, (qt + 1) * C::kBlk);
    // (a split that lies wholly above the work-group's diagonal has no tile)
    const int n_kt = max(0, (CAUSAL ? min(Sk, q_end + coff) : Sk) + C::kTile - 1) / C::kTile;

    // byte offset of 16-byte chunk `chunk` of row `row` within a tile tensor
    auto at = [](int row, int chunk) { return L::at(row, chunk); };

    // ---- streaming of tile kt into ring position pos; rows past S-1 read as zero
    const int Dr = a.Dr;  // columns Dr..D-1 read as zero (offset past the end of the resource)
    const uint32_t head_bytes = (uint32_t)(((int64_t)(Sk - 1) * a.kv_stride_s + Dr) * 2);
    const desc_t Kd0 = make_desc(a.K + base_kv + kv_first, head_bytes),
                 Vd0 = make_desc(a.V + base_kv + kv_first, head_bytes);
    const uint32_t row_bytes = (uint32_t)a.kv_stride_s * 2u;
    const uint32_t lds0 = lds_address(smem);
    // (the descriptors are passed by value: captured by reference through two levels of
    // lambdas the compiler no longer proves them wave-uniform)
    // lane l lands at byte 16 * l of a piece.  The piece's first row goes into the scalar offset (which takes part in the range check like
    // the per-lane one), so one per-lane offset serves every transfer.
    const uint32_t voff = Pieces<D>::lane_offset(l, row_bytes, Dr, head_bytes);
    auto dma_piece = [&](int kt, int pos, int n, desc_t Kd, desc_t Vd) __attribute__((always_inline)) {
        // wave-uniform 1 KB piece; a wave with nothing left repeats an earlier piece so
        // that every wave has the same number of transfers in flight
        const int i = (w + n * NW) % C::kDmaPerTile;
        const int tensor = i / C::kPieces, piece = i % C::kPieces;
        const uint32_t dst = lds0 + pos * C::kTileBytes + tensor * C::kTensorBytes + L::base(piece);
        const uint32_t soff = (kt * C::kTile + piece * PR) * row_bytes;
        if (kBetween) dma16_between(tensor ? Vd : Kd, dst, voff, soff);
        else dma16(tensor ? Vd : Kd, dst, voff, soff);
    };
    auto dma_tile = [&](int kt, int pos, desc_t Kd, desc_t Vd) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < C::kDmaPerWave; ++n) dma_piece(kt, pos, n, Kd, Vd);
    };
    if (n_kt > 0) dma_tile(0, 0, Kd0, Vd0);
    if (n_kt > 1) dma_tile(1, 1, Kd0, Vd0);

    // Q and dO fragments (B operands: lane holds row q, columns 16 ks + 8 h .. +7) and, in a full
    // backward, the O rows for the row statistics.  A load in which every lane fetches 16 bytes
    // of its own row touches 32 rows per instruction, and a work-group issues 192 of them here:
    // measured in the forward, 64 such loads alone took the last wave 5000-7000 cycles to get
    // issued, with the compute unit idle.  At D <= 128 the rows are therefore fetched whole (an
    // instruction covers 64 / (D/8) consecutive rows), all in flight together, and sorted into
    // the fragment layout through the wave's staging area in LDS, one tensor after the other.
    elem8 qf[KS], gf[KS], of[KS];
    if constexpr (C::kStageRows) {
        constexpr int CPR = D / 8, RPI = 64 / CPR, kLoads = 32 / RPI;  // chunks per row; rows per load instruction
        const int lr = l / CPR, lc = l % CPR;
        u32x4 tq[kLoads], tg[kLoads], to[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int64_t off = base + (int64_t)min(q0 + RPI * j + lr, S - 1) * a.stride_s;
            tq[j] = ld_row16(a.Q + off, lc * 8, Dr);
            tg[j] = ld_row16(a.dO + off, lc * 8, Dr);
            if (a.stats_in_dq) to[j] = ld_row16(a.O + off, lc * 8, Dr);
        }
        char *stage = smem + 2 * C::kTileBytes + w * C::kStageBytes;
        const int rd = at(r, h);  // chunk h of row r
        auto sort_rows = [&](const u32x4 (&t)[kLoads], elem8 (&f)[KS]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < kLoads; ++j) *(u32x4 *)(stage + at(RPI * j + lr, lc)) = t[j];
            asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) f[ks] = *(const elem8 *)(stage + rd + L::step(ks));
            asm volatile("" ::: "memory");
        };
        sort_rows(tq, qf);
        sort_rows(tg, gf);
        if (a.stats_in_dq) sort_rows(to, of);
    } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qf[ks] = as_elem8(ld_row16(a.Q + base + (int64_t)qc * a.stride_s, ks * 16 + 8 * h, Dr));
            gf[ks] = as_elem8(ld_row16(a.dO + base + (int64_t)qc * a.stride_s, ks * 16 + 8 * h, Dr));
        }
        if (a.stats_in_dq) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                of[ks] = as_elem8(ld_row16(a.O + base + (int64_t)qc * a.stride_s, ks * 16 + 8 * h, Dr));
        }
    }
    // Row statistics of this lane's query: lse2 = LSE * log2(e) and -delta = -rowsum(dO * O).
    // In a full backward this kernel runs first and forms them itself (the dO row is in
    // registers anyway; lanes l and l^32 hold the two halves of a row) and stores them for the
    // dK/dV kernel, which saves the separate kernel's launch; called alone it reads them.
    float lse2, ndelta;
    if (a.stats_in_dq) {
        float acc = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int t = 0; t < 8; ++t) acc += (float)of[ks][t] * (float)gf[ks][t];
        }
        ndelta = -xhalf_sum(acc);
        lse2 = a.LSE[(int64_t)bh * S + qc] * kLog2e;
        if (q < S && h == 0 && (!SPLIT || part == 0)) {
            a.delta[(int64_t)bh * 2 * S + q] = ndelta;
            a.delta[(int64_t)bh * 2 * S + S + q] = lse2;
        }
    } else {
        lse2 = a.delta[(int64_t)bh * 2 * S + S + qc];
        ndelta = a.delta[(int64_t)bh * 2 * S + qc];
    }
    // -delta replicated: the dP accumulators start from it
    f32x16 nd;
#pragma unroll
    for (int i = 0; i < 16; ++i) nd[i] = ndelta;

    f32x16 dq[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dq[db][i] = 0.f;

    const float c = a.scale_log2e;
    // Per-lane LDS addresses within ring position 0 (lo) and 2 (hi): row fragment = chunk h of
    // row r; transpose reads = rows 4h+e (+8), the 64 bytes of d block 0 of each row.  Everything else --
    // ring position, tensor, sub-tile, 16-row step -- is a compile-time offset.  Position 2
    // gets registers of its own because an LDS instruction's immediate reaches 64 KB and the
    // ring is longer than that at D = 128.  The values are made opaque so that the compiler
    // keeps exactly these six registers instead of re-deriving addresses in the loop.
    int row_lo = at(r, h), tr_lo[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
        tr_lo[j] = at(8 * j + 4 * h + ((l & 15) >> 2), 2 * ((l >> 4) & 1) + ((l >> 1) & 1)) + (l & 1) * 8;
    int row_hi = row_lo + 2 * C::kTileBytes, tr_hi[2] = {tr_lo[0] + 2 * C::kTileBytes,
                                                          tr_lo[1] + 2 * C::kTileBytes};
    asm volatile("" : "+v"(row_lo), "+v"(tr_lo[0]), "+v"(tr_lo[1]));
    if (NW == 8) asm volatile("" : "+v"(row_hi), "+v"(tr_hi[0]), "+v"(tr_hi[1]));

    // All register loads above must be complete before the loop: the compiler would otherwise
    // place its own vmcnt waits for them at their first use inside the loop, where they would
    // also wait for the tile transfers (which it does not see) in every iteration.
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)

    // One tile of 64 keys at ring position `pos`; Kt + rowa / tra0 / tra1 address its K tensor.
    // The steps of one 32-key sub-tile kb2 of the tile whose K tensor Kt + rowa / tra0 / tra1
    // address; register i of s and dp <-> key k_lo + 8*(i/4) + 4h + i%4 (this lane's query is
    // fixed).
    auto step_s = [&](const char *Kt, int rowa, int kb2, f32x16 &s) __attribute__((always_inline)) {
        f32x16 zero;
#pragma unroll
        for (int i = 0; i < 16; ++i) zero[i] = 0.f;
        s = mfma32(*(const elem8 *)(Kt + kb2 * 2 * C::kRows16 + rowa), qf[0], zero);
#pragma unroll
        for (int ks = 1; ks < KS; ++ks)
            s = mfma32(*(const elem8 *)(Kt + kb2 * 2 * C::kRows16 + L::step(ks) + rowa), qf[ks], s);
    };
    // the same with the transfers of tile kt_next (into ring position pos_next) between the MFMAs
    auto step_s_fetch = [&](const char *Kt, int rowa, f32x16 &s, int kt_next, int pos_next, desc_t Kd,
                            desc_t Vd) __attribute__((always_inline)) {
        constexpr int kEvery = kBetween ? KS / C::kDmaPerWave : 1;
        f32x16 zero;
#pragma unroll
        for (int i = 0; i < 16; ++i) zero[i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            s = mfma32(*(const elem8 *)(Kt + L::step(ks) + rowa), qf[ks], ks ? s : zero);
            if ((ks + 1) % kEvery == 0 && (ks + 1) / kEvery <= C::kDmaPerWave) dma_piece(kt_next, pos_next, (ks + 1) / kEvery - 1, Kd, Vd);
        }
    };
    auto step_dp = [&](const char *Kt, int rowa, int kb2, f32x16 &dp) __attribute__((always_inline)) {
        const char *Vt = Kt + C::kTensorBytes;
        dp = mfma32(*(const elem8 *)(Vt + kb2 * 2 * C::kRows16 + rowa), gf[0], nd);  // ends as dP - delta
#pragma unroll
        for (int ks = 1; ks < KS; ++ks)
            dp = mfma32(*(const elem8 *)(Vt + kb2 * 2 * C::kRows16 + L::step(ks) + rowa), gf[ks], dp);
    };
    auto step_p = [&](int k_lo, f32x16 &s) __attribute__((always_inline)) {  // S -> P
        const bool need_mask = (k_lo + 32 > Sk) || (CAUSAL && k_lo + 31 > q0e);
        const int lim = (CAUSAL ? qc + coff : Sk - 1) - k_lo - 4 * h;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = fast_exp2(__builtin_fmaf(s[i], c, -lse2));
        if (need_mask) {  // wave-uniform: only blocks on the diagonal or at the ragged end
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (8 * (i / 4) + (i % 4) > lim) s[i] = 0.f;
        }
    };
    auto step_ds = [&](const f32x16 &s, f32x16 &dp, elem8 (&sb)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) dp[i] *= s[i];  // dS = P o (dP - delta)
        sb[0] = pack8(dp[0], dp[1], dp[2], dp[3], dp[4], dp[5], dp[6], dp[7]);
        sb[1] = pack8(dp[8], dp[9], dp[10], dp[11], dp[12], dp[13], dp[14], dp[15]);
    };
    auto step_dq = [&](const char *Kt, int tra0, int tra1, int kb2, const elem8 (&sb)[2])
                       __attribute__((always_inline)) {
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const int off = (kb2 * 2 + cc) * C::kRows16 + db * L::kBlock;
                const elem8 kT = join8(lds_read_tr((const elem *)(Kt + off + tra0)),
                                       lds_read_tr((const elem *)(Kt + off + tra1)));
                dq[db] = mfma32(kT, sb[cc], dq[db]);
            }
        }
    };
    // A sub-tile as one step per MFMA, closed by a scheduling fence, with the LDS read of the fragment
    // kAhead MFMAs further on: S^T with the transfers of tile kt + 2, dP^T with the exp2 of S, dQ^T, whose
    // second half waits for the second half of dS next to the MFMAs of the first.  For the forms that
    // mostly run one wave per SIMD, where nothing else hides the wave's LDS latency, and for eight waves
    // at D = 64; eight waves at D = 128 are 1 % slower with it.  us: B=4 H=16 S=4096 D=256 causal
    // 831 -> 802, B=2 H=5 S=3607 310 -> 292; four waves B=1 H=8 S=2048 D=128 50.7 -> 48.0, B=8 H=8 S=1024
    // D=64 causal 28.9 -> 27.7; B=4 H=16 S=8192 D=64 causal 813 -> 784.
    constexpr bool kSteps = D > 128 || NW == 4 || (NW == 8 && D == 64);
    auto tile_steps = [&](int kt, int kb2, int pos, const char *Kt, int rowa, int tra0, int tra1, desc_t Kd, desc_t Vd,
                          bool fetch) __attribute__((always_inline)) {
        constexpr int kAhead = 4, N = 2 * KS + 2 * DB;
        elem8 f[N];
        auto read = [&](int n) __attribute__((always_inline)) {
            if (n < 2 * KS) {
                f[n] = *(const elem8 *)(Kt + (n / KS) * C::kTensorBytes + kb2 * 2 * C::kRows16 +
                                        L::step(n % KS) + rowa);
            } else if (n < N) {
                const int off = (kb2 * 2 + (n - 2 * KS) / DB) * C::kRows16 + ((n - 2 * KS) % DB) * L::kBlock;
                f[n] = join8(lds_read_tr((const elem *)(Kt + off + tra0)), lds_read_tr((const elem *)(Kt + off + tra1)));
            }
        };
        const int k_lo = kt * C::kTile + kb2 * 32;
        constexpr int kEvery = kBetween ? KS / C::kDmaPerWave : 1;
        f32x16 s, dp, zero;
#pragma unroll
        for (int i = 0; i < 16; ++i) zero[i] = 0.f;
#pragma unroll
        for (int n = 0; n < kAhead; ++n) read(n);
        __builtin_amdgcn_sched_barrier(0);
        if (fetch) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                s = mfma32(f[ks], qf[ks], ks ? s : zero);
                read(ks + kAhead);
                if ((ks + 1) % kEvery == 0 && (ks + 1) / kEvery <= C::kDmaPerWave) dma_piece(kt + 2, pos == 0 ? 2 : pos - 1, (ks + 1) / kEvery - 1, Kd, Vd);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                s = mfma32(f[ks], qf[ks], ks ? s : zero);
                read(ks + kAhead);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            dp = mfma32(f[KS + ks], gf[ks], ks ? dp : nd);  // ends as dP - delta
            read(KS + ks + kAhead);
#pragma unroll
            for (int i = exps_before(ks, KS); i < exps_before(ks + 1, KS); ++i)
                s[i] = fast_exp2(__builtin_fmaf(s[i], c, -lse2));
            __builtin_amdgcn_sched_barrier(0);
        }
        if ((k_lo + 32 > Sk) || (CAUSAL && k_lo + 31 > q0e)) {  // wave-uniform
            const int lim = (CAUSAL ? qc + coff : Sk - 1) - k_lo - 4 * h;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (8 * (i / 4) + (i % 4) > lim) s[i] = 0.f;
        }
        elem8 sb[2];
        auto half = [&](int i0) __attribute__((always_inline)) {  // dS = P o (dP - delta)
#pragma unroll
            for (int i = i0; i < i0 + 8; ++i) dp[i] *= s[i];
            return pack8(dp[i0], dp[i0 + 1], dp[i0 + 2], dp[i0 + 3], dp[i0 + 4], dp[i0 + 5], dp[i0 + 6], dp[i0 + 7]);
        };
        sb[0] = half(0);
#pragma unroll
        for (int n = 0; n < 2 * DB; ++n) {
            dq[n % DB] = mfma32(f[2 * KS + n], sb[n / DB], dq[n % DB]);
            read(2 * KS + n + kAhead);
            if (n == 0) sb[1] = half(8);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // One tile at ring position `pos`.
    auto tile = [&](int kt, int pos, const char *Kt, int rowa, int tra0, int tra1, desc_t Kd,
                    desc_t Vd) __attribute__((always_inline)) {
        // tile kt must have landed; tile kt+1 (if any) may stay in flight
        if (kt + 1 < n_kt) wait_vm_and_barrier<C::kDmaPerWave>();
        else wait_vm_and_barrier<0>();
        const bool fetch = kt + 2 < n_kt;  // tile kt + 2 goes into the ring position freed by the barrier
        if (fetch && !kBetween) dma_tile(kt + 2, pos == 0 ? 2 : pos - 1, Kd, Vd);

        const int k0 = kt * C::kTile;
        // wave-uniform: does this wave see any key of the first / second sub-tile
        const bool act0 = k0 < Sk && (!CAUSAL || k0 <= q0e + 31);
        const bool act1 = k0 + 32 < Sk && (!CAUSAL || k0 + 32 <= q0e + 31);
        if (kBetween && fetch && !act0) dma_tile(kt + 2, pos == 0 ? 2 : pos - 1, Kd, Vd);
#pragma unroll
        for (int kb2 = 0; kb2 < C::kSub; ++kb2) {
            if (!(kb2 ? act1 : act0)) continue;
            f32x16 s, dp;
            elem8 sb[2];
            if constexpr (kSteps) {
                tile_steps(kt, kb2, pos, Kt, rowa, tra0, tra1, Kd, Vd, fetch && kb2 == 0);
                continue;
            }
            if (kBetween && kb2 == 0 && fetch) step_s_fetch(Kt, rowa, s, kt + 2, pos == 0 ? 2 : pos - 1, Kd, Vd);
            else step_s(Kt, rowa, kb2, s);
            step_dp(Kt, rowa, kb2, dp);
            step_p(k0 + kb2 * 32, s);
            step_ds(s, dp, sb);
            step_dq(Kt, tra0, tra1, kb2, sb);
        }
    };
    if constexpr (NW == 8) {
        // unrolled over the three ring positions, which makes them compile-time constants;
        // n_kt is the same for every wave of the work-group
        for (int kt = 0; kt < n_kt; kt += 3) {
            tile(kt, 0, smem, row_lo, tr_lo[0], tr_lo[1], Kd0, Vd0);
            if (kt + 1 < n_kt)
                tile(kt + 1, 1, smem + C::kTileBytes, row_lo, tr_lo[0], tr_lo[1], Kd0, Vd0);
            if (kt + 2 < n_kt) tile(kt + 2, 2, smem, row_hi, tr_hi[0], tr_hi[1], Kd0, Vd0);
        }
    } else {
        // fewer waves issue more transfers each and have no registers to spare for the unrolled
        // form: the ring position advances at run time (three additions per tile)
        int pos = 0;
        for (int kt = 0; kt < n_kt; ++kt) {
            const int o = pos * C::kTileBytes;
            tile(kt, pos, smem, row_lo + o, tr_lo[0] + o, tr_lo[1] + o, Kd0, Vd0);
            pos = pos == 2 ? 0 : pos + 1;
        }
    }
    // no transfer may still be in flight when the work-group's LDS is released
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // Output rows leave through the wave's staging area in LDS (see the end of the kernel).  The
    // areas that lie in ring position 2 move to the position that the last two tiles did not use
    // (other waves may still be reading those).
    constexpr int CPR = D / 8, RPI = 64 / CPR;  // chunks per bf16 row; rows per store instruction
    char *const stg = smem + ((w + 1) * C::kStageBytes <= C::kTileBytes
                                  ? (n_kt % 3) * C::kTileBytes + w * C::kStageBytes
                                  : 2 * C::kTileBytes + w * C::kStageBytes);
    const int lr = l / CPR, lc = l % CPR;
    if (SPLIT) {
        // unscaled fp32 partial of this key range (zeros if the range had no visible key); an
        // fp32 row is twice as long as the staging area's, so it goes in two halves
        const int64_t row0 = ((int64_t)part * a.BH + bh) * S;
#pragma unroll
        for (int hp = 0; hp < 2; ++hp) {  // (columns past U: anything; the merge drops them)
            constexpr int HB = D / 64;
#pragma unroll
            for (int db = hp * HB; db < (hp + 1) * HB && db < DB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = dq[db][4 * g + e];
                    *(f32x4 *)(stg + at(r, (db % HB) * 8 + 2 * g + h)) = v;
                }
            asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
            for (int j = 0; j < 32 / RPI; ++j) {
                const f32x4 v = *(const f32x4 *)(stg + at(RPI * j + lr, lc));
                const int row = q0 + RPI * j + lr;
                if (row < S) *(f32x4 *)(a.dQpart + (row0 + row) * D + hp * (D / 2) + lc * 4) = v;
            }
            asm volatile("" ::: "memory");
        }
        return;
    }
    dq_rows_out<C, D, U>(a, dq, stg, base, q0, l);
}

template <int D, int U, int NW, bool CAUSAL, bool SPLIT>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(D > 128 ? 1 : 2)))
attn_bwd_dq_kernel(const BwdArgs a)
{
    bwd_dq<D, U, NW, CAUSAL, SPLIT>(a, blockIdx.x, a.ntile, blockIdx.y);
}

// ---------------------------------------------------------------------------------------
// 3b. dQ from the dS that the dK/dV kernel stored: one product instead of three, bound by reading dS
// (2 bytes a score) from HBM where the launch is long (rates: see ds_plan).  Work-group = NW waves, wave = RB
// blocks of 32 queries, loop over tiles of 32 keys; one MFMA (per row block) a step, closed by a scheduling fence,
// with the fragment of K four steps further on requested in it (128 heads of 4096 rows, D = 128, 826 -> 807 us).
// With two row blocks a wave reads every fragment of K once for two products, and a unit half the K tiles (807 -> 734).
// The K tile (in the layout above, shared) and the waves' dS blocks (each read by its wave alone) go
// global -> LDS directly, kRing - 1 tiles ahead: about 100 KB in flight per unit.
// A dS block holds 8-byte groups of 4 consecutive queries of a key; in the order in which the producers
// store them the 64 lanes of a transpose read (8 keys x 32 queries) cover 512 contiguous bytes.
// ---------------------------------------------------------------------------------------
template <int D, int NW, int RB>
struct DqsCfg : DqCfg<D, 4> {
    using L = Pieces<D>;
    static constexpr int kBlk = NW * RB * 32;
    static constexpr int kTile = 32;
    static constexpr int kPieces = kTile / L::kRows;
    static constexpr int kKBytes = L::base(kPieces);
    static constexpr int kTileBytes = kKBytes + NW * RB * kDsBlock * 2;
    static constexpr int kRing = 160 * 1024 / kTileBytes < 6 ? 160 * 1024 / kTileBytes : 6;
    static constexpr int kStage = L::base(32 / L::kRows);
    static constexpr int kLdsBytes = kRing * kTileBytes > NW * kStage ? kRing * kTileBytes : NW * kStage;
    static constexpr int kDmaK = (kPieces + NW - 1) / NW;     // transfers of a wave per tile: K, then dS
    static constexpr int kDma = kDmaK + 2 * RB;
    static_assert(kPieces % NW == 0, "every wave has the same number of transfers in flight");
    static_assert(kRing >= 3 && kLdsBytes <= 160 * 1024, "LDS layout");
};

template <int D, int U, int NW, int RB, bool CAUSAL>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW > 4 ? 2 : 1)))
attn_bwd_dq_ds_kernel(const BwdArgs a)
{
    using C = DqsCfg<D, NW, RB>;
    using L = Pieces<D>;
    constexpr int DB = U / 32, PR = C::kPieceRows;
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int tid = threadIdx.x, l = tid & 63, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = a.S, Sk = a.Sk, coff = Sk - S;
    int bh, rank;
    xcd_tile_order<CAUSAL>(blockIdx.x, a.ntile, a.nkv * a.group, bh, rank);
    const int qt = CAUSAL ? a.ntile - 1 - rank : rank;  // heaviest first
    const int64_t ds_head = bh * ds_head_blocks(S, Sk, CAUSAL);  // (of the launch's heads)
    bh += a.bkv0 * a.group;
    const int64_t base = (int64_t)(bh / a.H) * a.stride_b + (int64_t)(bh % a.H) * a.stride_h;
    const int64_t base_kv = (int64_t)(bh / a.H) * a.kv_stride_b + (int64_t)((bh % a.H) / a.group) * a.kv_stride_h;
    const int t0 = (qt * NW + w) * RB;  // the wave's slots: t0 .. t0 + RB - 1
    const int q_end = min(S, (qt + 1) * C::kBlk);
    const int n_kt = ((CAUSAL ? min(Sk, q_end + coff) : Sk) + 31) / 32;  // key blocks that some wave sees
    int n_row[RB];  // ... and each slot (never more; every wave passes the barriers of n_kt tiles)
    desc_t Sd[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int t = t0 + rb;
        n_row[rb] = t * 32 < S ? min(n_kt, ds_row_len(t, Sk, coff, CAUSAL)) : 0;
        Sd[rb] = make_desc(a.dS + (ds_head + ds_row_blocks(min(t, (S + 31) / 32 - 1), Sk, coff, CAUSAL)) * kDsBlock,
                           (uint32_t)n_row[rb] * (kDsBlock * 2u));
    }

    const int Dr = a.Dr;
    const uint32_t head_bytes = (uint32_t)(((int64_t)(Sk - 1) * a.kv_stride_s + Dr) * 2);
    const desc_t Kd = make_desc(a.K + base_kv, head_bytes);
    const uint32_t row_bytes = (uint32_t)a.kv_stride_s * 2u;
    const uint32_t lds0 = lds_address(smem);
    const uint32_t voff = L::lane_offset(l, row_bytes, Dr, head_bytes);
    // (tiles past the last read as zero, or are keys that nobody uses)
    auto fetch = [&](int kt, int pos) __attribute__((always_inline)) {
        const uint32_t dst = lds0 + pos * C::kTileBytes;
#pragma unroll
        for (int n = 0; n < 2 * RB; ++n)
            dma16_between_nt(Sd[n >> 1], dst + C::kKBytes + (w * RB + (n >> 1)) * (kDsBlock * 2) + (n & 1) * 1024, l * 16,
                             kt * (kDsBlock * 2) + (n & 1) * 1024);
#pragma unroll
        for (int n = 0; n < C::kDmaK; ++n) {
            const int piece = w + n * NW;
            dma16_between(Kd, dst + L::base(piece), voff, (kt * 32 + piece * PR) * row_bytes);
        }
    };
#pragma unroll
    for (int i = 0; i < C::kRing - 1; ++i) fetch(i, i);

    // transpose reads: of K, rows 4h+e (+8) and the 64 bytes of d block 0; of dS, the same keys and
    // the 4 queries of the lane's chunk
    int tr[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = 8 * j + 4 * h + ((l & 15) >> 2), chunk = 2 * ((l >> 4) & 1) + ((l >> 1) & 1);
        tr[j] = L::at(row, chunk) + (l & 1) * 8;
    }
    int ds = C::kKBytes + w * RB * (kDsBlock * 2) + h * 256 + (((l >> 4) & 1) * 2 + (l & 1)) * 64 + ((l & 15) >> 2) * 16 +
             ((l >> 1) & 1) * 8;
    asm volatile("" : "+v"(tr[0]), "+v"(tr[1]), "+v"(ds));

    f32x16 dq[RB][DB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) dq[rb][db][i] = 0.f;

    // row blocks B0 .. B1 - 1 of the wave
    auto step = [&](const char *T, auto B0, auto B1) __attribute__((always_inline)) {
        constexpr int kAhead = 4;
        elem8 b[RB][2], f[2 * DB];
        auto read = [&](int n) __attribute__((always_inline)) {
            const int off = (n / DB) * C::kRows16 + (n % DB) * L::kBlock;
            if (n < 2 * DB)
                f[n] = join8(lds_read_tr((const elem *)(T + off + tr[0])), lds_read_tr((const elem *)(T + off + tr[1])));
        };
#pragma unroll
        for (int rb = B0; rb < B1; ++rb)
#pragma unroll
            for (int cc = 0; cc < 2; ++cc)
                b[rb][cc] = join8(lds_read_tr((const elem *)(T + ds + rb * (kDsBlock * 2) + cc * 1024)),
                                  lds_read_tr((const elem *)(T + ds + rb * (kDsBlock * 2) + cc * 1024 + 512)));
#pragma unroll
        for (int n = 0; n < kAhead; ++n) read(n);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < 2 * DB; ++n) {
#pragma unroll
            for (int rb = B0; rb < B1; ++rb) dq[rb][n % DB] = mfma32(f[n], b[rb][n / DB], dq[rb][n % DB]);
            read(n + kAhead);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using std::integral_constant;
    int kt = 0, pos = 0;
    // tiles kt .. end - 1 with the wave's row blocks B0 .. B1 - 1 (the others see none of these keys)
    auto walk = [&](int end, auto B0, auto B1) __attribute__((always_inline)) {
        for (; kt < end; ++kt) {
            wait_vm_and_barrier<(C::kRing - 2) * C::kDma>();
            fetch(kt + C::kRing - 1, pos == 0 ? C::kRing - 1 : pos - 1);
            if constexpr (B0 < B1) step(smem + pos * C::kTileBytes, B0, B1);
            pos = pos + 1 == C::kRing ? 0 : pos + 1;
        }
    };
    typedef integral_constant<int, 0> I0;
    typedef integral_constant<int, 1> I1;
    typedef integral_constant<int, RB> IR;
    if constexpr (RB > 1) {
        walk(min(n_row[0], n_row[1]), I0(), IR());
        walk(n_row[1], I1(), IR());
    }
    walk(n_row[0], I0(), I1());
    walk(n_kt, I0(), I0());
    wait_vm_and_barrier<0>();  // (everyone's transfers have landed: the LDS is free)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        dq_rows_out<C, D, U>(a, dq[rb], smem + w * C::kStage, base, (t0 + rb) * 32, l);
        asm volatile("" ::: "memory");
    }
}

// Sum of the per-split partial dQ, times scale, rounded: one thread per (row, 4 consecutive d);
// HBM-bound and small.
template <int D>
__device__ __forceinline__ void bwd_dq_merge(const BwdArgs &a, int block)
{
    constexpr int TPR = D / 4;  // threads per row
    const int64_t rows = (int64_t)a.BH * a.S;
    const int64_t row = (int64_t)block * (256 / TPR) + threadIdx.x / TPR;
    if (row >= rows) return;
    const int d0 = (threadIdx.x % TPR) * 4;
    // four splits per step, their loads issued together (one dependent load per split costs a
    // memory latency each); added in the order of the splits
    const int n = a.dq_nsplit;
    auto sum = [&](int d) __attribute__((always_inline)) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int z0 = 0; z0 < n; z0 += 4) {
            f32x4 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[k] = *(const f32x4 *)(a.dQpart + ((int64_t)(z0 + k < n ? z0 + k : z0) * rows + row) * D + d);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (z0 + k < n) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] += v[k][e];
                }
        }
        return acc;
    };
    f32x4 acc = sum(d0);
    const int bh = (int)(row / a.S), q = (int)(row % a.S);
    if (a.rope_cos) {  // rotated back, as in dq_rows_out; d0 pairs with d0 -+ D/2
        const f32x4 other = sum(d0 ^ (D / 2));
        const int64_t pos = (int64_t)(q + a.rope_pos0) * (D / 2) + d0 % (D / 2);
        const f32x4 c4 = *(const f32x4 *)(a.rope_cos + pos), s4 = *(const f32x4 *)(a.rope_sin + pos);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc[e] = __builtin_fmaf(acc[e], c4[e], d0 < D / 2 ? other[e] * s4[e] : -(other[e] * s4[e]));
    }
    elem *dQp = a.dQ + (int64_t)(bh / a.H) * a.stride_b + (int64_t)(bh % a.H) * a.stride_h +
                (int64_t)q * a.stride_s + d0;
    const float sc = a.scale;
    if (d0 < a.Dr) *(elem4 *)dQp = pack4(acc[0] * sc, acc[1] * sc, acc[2] * sc, acc[3] * sc);
}

template <int D>
__global__ void __launch_bounds__(256) attn_bwd_dq_merge_kernel(const BwdArgs a) { bwd_dq_merge<D>(a, blockIdx.x); }

// ---------------------------------------------------------------------------------------
// 2 + 3. dK/dV and dQ in one launch, for calls whose work-groups leave compute units idle: the first
// pair_dkdv work-groups are those of the dK/dV kernel, the others those of the dQ kernel (the statistics,
// which both read, come from the kernel above).  Bound by the longest work-group, so both are cut until
// the units are taken (see pair_plan), and one launch merges both.
// ---------------------------------------------------------------------------------------
template <int D>
struct PairCfg {  // as many waves for dQ as for dK/dV; above D = 128 one per SIMD
    static constexpr int kPairs = D > 128 ? 2 : 4, kWaves = 2 * kPairs;
    using Dkdv = DkdvCfg<D, kPairs>;
    using Dq = DqCfg<D, kWaves>;
    static constexpr int kLdsBytes = Dkdv::kLdsBytes > Dq::kLdsBytes ? Dkdv::kLdsBytes : Dq::kLdsBytes;
    static constexpr int kMergeRows = 256 / (D / 4);  // dQ rows of a merging work-group
    static_assert(Dkdv::kThreads == Dq::kThreads, "one launch");
};

template <int D, int U, bool CAUSAL, bool SPLIT>
__global__ void __launch_bounds__(PairCfg<D>::Dq::kThreads) __attribute__((amdgpu_waves_per_eu(D > 128 ? 1 : 2)))
attn_bwd_pair_kernel(const BwdArgs a)
{
    using C = PairCfg<D>;
    if ((int)blockIdx.x < a.pair_dkdv) {
        bwd_dkdv<D, U, C::kPairs, CAUSAL, SPLIT, false>(a, blockIdx.x, a.ntile);
    } else {
        const int i = (int)blockIdx.x - a.pair_dkdv, n = a.pair_dq * a.BH;
        // (above D = 128 dQ is not split)
        bwd_dq<D, U, C::kWaves, CAUSAL, SPLIT && D <= 128>(a, D > 128 ? i : i % n, a.pair_dq, D > 128 ? 0 : i / n);
    }
}

template <int D, bool CAUSAL>
__global__ void __launch_bounds__(256) attn_bwd_pair_merge_kernel(const BwdArgs a)
{
    const int i = (int)blockIdx.x - a.pair_dkdv;  // first the two tensors of the key blocks, then dQ
    if (i < 0) bwd_dkdv_merge<D, CAUSAL>(a, blockIdx.x >> 1, blockIdx.x & 1);
    else bwd_dq_merge<D>(a, i);
}

// ---------------------------------------------------------------------------------------
// Launch
// ---------------------------------------------------------------------------------------
template <typename K>
static bool allow_lds(K kernel, int bytes)
{
    return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               bytes) == hipSuccess;
}

template <int D, int U, int P, bool CAUSAL, bool DS>
static int launch_dkdv_p(BwdArgs a, hipStream_t st)
{
    using C = DkdvCfg<D, P>;
    a.ntile = (a.Sk + C::kBlk - 1) / C::kBlk;
    if (!allow_lds(attn_bwd_dkdv_kernel<D, U, P, CAUSAL, false, DS>, C::kLdsBytes)) return -1;
    hipLaunchKernelGGL((attn_bwd_dkdv_kernel<D, U, P, CAUSAL, false, DS>), dim3(a.ntile * a.nkv),
                       dim3(C::kThreads), C::kLdsBytes, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Split over the query slots: one work-group per chunk, then the merge.
template <int D, int U, bool CAUSAL, bool DS>
static int launch_dkdv_split(BwdArgs a, hipStream_t st)
{
    constexpr int P = D > 128 ? 2 : 4, keys = dkdv_split_keys(D);
    using C = DkdvCfg<D, P>;
    static_assert(C::kBlk == keys, "keys per work-group");
    const int BHkv = a.BH / a.group;
    a.ntile = a.dkdv_items;
    if (!allow_lds(attn_bwd_dkdv_kernel<D, U, P, CAUSAL, true, DS>, C::kLdsBytes)) return -1;
    hipLaunchKernelGGL((attn_bwd_dkdv_kernel<D, U, P, CAUSAL, true, DS>), dim3(a.ntile * BHkv), dim3(C::kThreads),
                       C::kLdsBytes, st, a);
    if (hipGetLastError() != hipSuccess) return -1;
    const int n_block = (a.Sk + keys - 1) / keys;
    hipLaunchKernelGGL((attn_bwd_dkdv_merge_kernel<D, CAUSAL>), dim3(BHkv * n_block * (keys * D / 1024), 2),
                       dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Work-groups of four producer/consumer pairs (128 keys, two waves per SIMD), or, at D = 128
// on launches of at least two rounds of work-groups, of six (192 keys, 12 waves at 168
// registers: three per SIMD hide more of each other's latencies).  Measured: -2.5..4 % on the
// large shapes; slower on small launches (more of a 192-key block is padding) and at D = 64
// (the larger work-group no longer fits a compute unit twice).  Or, at D = 128 too, the kernel of
// attn_bwd_solo.hip (256 keys), where dkdv_takes_solo says so.
template <int D, int U, bool CAUSAL, bool DS>
static int launch_dkdv_u(const BwdArgs &a, hipStream_t st)
{
    if (a.dkdv_chunk) return launch_dkdv_split<D, U, CAUSAL, DS>(a, st);
    // D = 256: two pairs, one wave per SIMD (a consumer's two 32 x 256 accumulators alone are
    // 256 registers), 64 keys per work-group
    if constexpr (D > 128) return launch_dkdv_p<D, U, 2, CAUSAL, DS>(a, st);
    else {
        if constexpr (D == 128) {
            const int64_t wgs6 = (int64_t)a.nkv * ((a.Sk + 191) / 192);
            if (dkdv_takes_solo(a.nkv, a.group, a.S, a.Sk, CAUSAL, DS)) return launch_bwd_dkdv_solo(a, CAUSAL, DS, st);
            if (wgs6 >= 512) return launch_dkdv_p<D, U, 6, CAUSAL, DS>(a, st);
        }
        return launch_dkdv_p<D, U, 4, CAUSAL, DS>(a, st);
    }
}

template <int D, bool CAUSAL, bool DS = false>
static int launch_dkdv(const BwdArgs &a, hipStream_t st)
{
    constexpr int U = narrow_columns(D);
    return a.Dr <= U ? launch_dkdv_u<D, U, CAUSAL, DS>(a, st) : launch_dkdv_u<D, D, CAUSAL, DS>(a, st);
}

#ifndef ATTN_F16
// Work-groups of one wave (at most 32 rows), of which three fit a unit: 769 .. 1024 take two rounds anyway, and two of
// two a unit are quicker than one of three and the rest.  us, whole backward, 1024 heads on 512 of 32 rows and 4000 keys 395 | 434
// (960 375 | 413, 800 338 | 352), of 18 and 1000 102 | 107; outside 1.04 .. 1.34 times as long.  Not so with more waves.
bool dq_takes_two(int nw, int wgs) { return nw == 1 && wgs > 768 && wgs <= 1024; }
#endif

template <int D, int U, int NW, bool CAUSAL>
static int launch_dq(BwdArgs a, hipStream_t st)
{
    using C = DqCfg<D, NW>;
    a.ntile = (a.S + C::kBlk - 1) / C::kBlk;
    constexpr int kMost = D == 64 && NW == 1 ? std::max(C::kLdsBytes, kLdsTwoPerUnit) : C::kLdsBytes;
    const int lds = D == 64 && dq_takes_two(NW, a.ntile * a.BH) ? kMost : C::kLdsBytes;
    // (one limit for every launch of the kernel: another thread may be between its own call here and its launch)
    if (!allow_lds(attn_bwd_dq_kernel<D, U, NW, CAUSAL, false>, kMost)) return -1;
    hipLaunchKernelGGL((attn_bwd_dq_kernel<D, U, NW, CAUSAL, false>), dim3(a.ntile * a.BH),
                       dim3(C::kThreads), lds, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Split over the keys: 256-row work-groups, one grid row per split, then the merge.
template <int D, int U, bool CAUSAL>
static int launch_dq_split(BwdArgs a, hipStream_t st)
{
    using C = DqCfg<D, 8>;
    a.ntile = (a.S + C::kBlk - 1) / C::kBlk;
    if (!allow_lds(attn_bwd_dq_kernel<D, U, 8, CAUSAL, true>, C::kLdsBytes)) return -1;
    hipLaunchKernelGGL((attn_bwd_dq_kernel<D, U, 8, CAUSAL, true>), dim3(a.ntile * a.BH, a.dq_nsplit),
                       dim3(C::kThreads), C::kLdsBytes, st, a);
    if (hipGetLastError() != hipSuccess) return -1;
    const int64_t rows = (int64_t)a.BH * a.S;
    constexpr int RPB = 256 / (D / 4);
    hipLaunchKernelGGL((attn_bwd_dq_merge_kernel<D>), dim3((unsigned)((rows + RPB - 1) / RPB)),
                       dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

#ifndef ATTN_F16
// Waves per work-group of the unsplit dQ kernel (D = 64 or 128).  At D = 128 eight, i.e. 256 rows, unless they would
// leave compute units (256) idle while 128-row ones would not (few heads and rows against many keys, e.g.
// chunked prefill); without a mask also where the 128-row ones would need a second round (32 heads of 1537 rows
// 84 -> 64 us, 48 of 1024 61 -> 43).  Under a causal mask 128-row work-groups also balance the unequal tiles better as
// long as the launch is small: up to one 256-row work-group per unit (B=1 H=16 S=4096: 135 -> 117 us, B=1 H=8 S=8192:
// 256 -> 220 us; with 1.25 per unit already 15 % slower).
// At D = 64 from 225 rows on: without a mask see WaveRule; causal four, except for narrow tensors in large launches.  us,
// four | eight: 14 heads of 3820 rows 88 | 82, 102 of 869 38 | 46, 316 of 318 23 | 32, 23 of 5113 210 | 203, but 147 of
// 766 40 | 41; causal 860 of 330 42 | 65, 364 of 1230 140 | 159, 102 of 4484 391 | 422, D = 32 136 of 2198 109 | 102, 1229 of
// 453 72 | 65, 76 of 3367 142 | 114.  Without a mask, over 340 problems of 228 .. 6200 rows and 200 .. 5000 work-groups of
// four, 1.000 of the time of the better of the two on average, none above 1.013; causal and above 32 columns, over 171 from
// 1024 work-groups of eight on, 0.80 of the time of eight, none above 1.025 (64 of 4075 207 | 202).
int dq_waves(int BH, int S, int Sk, int D, bool causal, bool narrow)
{
    const int blocks32 = (S + 31) / 32;
    const int64_t wgs8 = (int64_t)BH * ((S + 255) / 256), wgs4 = (int64_t)BH * ((S + 127) / 128);
    if (D == 64 && blocks32 >= 8) {
        static const WaveRule rule = {{5.9f, 3.4f, {0.49f, 0.91f, 1.29f}, 3}, {5.65f, 3.7f, {0.85f, 1.52f}, 2}, 1280};
        return (causal ? narrow && wgs8 >= 1024 : takes_eight_waves(rule, BH, S, Sk, narrow)) ? 8 : 4;
    }
    const bool prefer4 = causal && wgs8 <= 256;
    const bool fill8 = wgs8 >= 256 || (!causal && wgs4 > 256);
    if (blocks32 >= 8 && fill8 && !prefer4) return 8;
    if (blocks32 >= 3) return std::min(blocks32, 4);
    // (one wave: only D = 64; with D = 128 a lone wave would spill while it streams tiles)
    return D == 128 ? 2 : blocks32;
}
#endif

template <int D, int U, bool CAUSAL>
static int launch_dq_u(const BwdArgs &a, hipStream_t st)
{
    // D = 256: always four waves, one per SIMD (Q and dO fragments plus the accumulator are
    // 256 registers); never split
    if constexpr (D > 128) return a.dq_nsplit > 1 ? -1 : launch_dq<D, U, 4, CAUSAL>(a, st);
    else {
    if (a.dq_nsplit > 1) return launch_dq_split<D, U, CAUSAL>(a, st);
    const int nw = dq_waves(a.BH, a.S, a.Sk, D, CAUSAL, U < D);
    if (nw == 8) return launch_dq<D, U, 8, CAUSAL>(a, st);
    if (nw == 4) return launch_dq<D, U, 4, CAUSAL>(a, st);
    if (nw == 3) return launch_dq<D, U, 3, CAUSAL>(a, st);
    if (nw == 2) return launch_dq<D, U, 2, CAUSAL>(a, st);
    if constexpr (D < 128) return launch_dq<D, U, 1, CAUSAL>(a, st);
    return -1;
    }
}

template <int D, bool CAUSAL>
static int launch_dq_for(const BwdArgs &a, hipStream_t st)
{
    constexpr int U = narrow_columns(D);
    return a.Dr <= U ? launch_dq_u<D, U, CAUSAL>(a, st) : launch_dq_u<D, D, CAUSAL>(a, st);
}

template <int D, int U, int NW, int RB, bool CAUSAL>
static int launch_dq_ds_u(BwdArgs a, hipStream_t st)
{
    using C = DqsCfg<D, NW, RB>;
    a.ntile = (a.S + C::kBlk - 1) / C::kBlk;
    if (!allow_lds(attn_bwd_dq_ds_kernel<D, U, NW, RB, CAUSAL>, C::kLdsBytes)) return -1;
    hipLaunchKernelGGL((attn_bwd_dq_ds_kernel<D, U, NW, RB, CAUSAL>), dim3(a.ntile * a.nkv * a.group), dim3(NW * 64),
                       C::kLdsBytes, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int D, int NW, bool CAUSAL>
static int launch_dq_ds(const BwdArgs &a, hipStream_t st)
{
    constexpr int U = narrow_columns(D);
    return a.Dr <= U ? launch_dq_ds_u<D, U, NW, 1, CAUSAL>(a, st) : launch_dq_ds_u<D, D, NW, 1, CAUSAL>(a, st);
}

// Eight waves of two row blocks (see dq_ds_blocks).
template <int D, bool CAUSAL>
static int launch_dq_ds_two(const BwdArgs &a, hipStream_t st)
{
    if constexpr (D > 128) return -1;
    else return launch_dq_ds_u<D, D, 8, 2, CAUSAL>(a, st);
}

#ifndef ATTN_F16
// Row blocks (of 32 rows) per work-group: eight, one a wave, which read K less often, unless smaller work-groups
// still fill the compute units in one round.  us, whole backward, 8 | 4 | 2: 11 heads of 1166 rows 61 | 55 | 53,
// 4 of 5599 causal 173 | 147 | 152, 10 of 1876 D=256 causal 116 | 105 | 105; 8 of 4384 248 | 267 | 284,
// 32 of 4096 and 16384 five per cent faster with eight.  Long causal heads, whose eight-wave work-groups
// are the most unequal, take four for longer: 4 of 10802 460 | 427 | 458, 4 of 12527 550 | 530 | 569, but
// 114 of 321 46 | 51.
// At D = 128 sixteen, two a wave, in launches of two rounds of them: half the K tiles, and every fragment of K feeds
// two products.  us, this kernel alone, 8 | 16: 128 heads of 4096 rows 807 | 734; whole backward: 128 of 2048 causal
// 470 | 455, 192 of 2048 1258 | 1228.  Not
//  - with fewer work-groups, when the launch ends on a long one (64 of 2048 causal 227 | 240, 16 of 4096 causal 220 | 248),
//    which from 4097 rows on takes two and a half rounds to hide;
//  - where the rows that only pad them cost more: a ninth more rows without a mask (1.00 of the time there, 1.02 with a
//    fifth), a seventeenth under one (1.00, and 1.01 with a ninth);
//  - under a mask below 1600 rows, of which a work-group of 512 sees too unequal parts (1.004 on average, 442 of 935 1.037);
//  - at 96 columns (249 of 1076 286 | 288).
// Over 560 whole backwards of 370 .. 9400 rows and 640 .. 4100 blocks of 256 the rule takes sixteen in 190: 0.988 of the
// time of eight on average, one of them above 1.02; over 260 others in 95: 0.988, none above 1.019.
int dq_ds_blocks(int heads, int S, int Dr, bool causal)
{
    const int blocks256 = (S + 255) / 256, padded = (blocks256 + 1) / 2 * 2;  // in blocks of 256 rows
    if (Dr > narrow_columns(128) && Dr <= 128 && (int64_t)heads * blocks256 >= (S > 4096 ? 1280 : 1024) &&
        (causal ? S >= 1600 && 17 * padded <= 18 * blocks256 : 9 * padded <= 10 * blocks256))
        return 16;
    if ((int64_t)heads * ((S + 127) / 128) > (causal && S > 4096 ? 512 : 256)) return 8;
    return (int64_t)heads * ((S + 63) / 64) > 256 ? 4 : 2;
}
#endif

template <int D>
static int launch_delta(const BwdArgs &a, hipStream_t st)
{
    constexpr int RPB = 256 / (D / 8);
    const int64_t rows = (int64_t)a.BH * a.S;
    hipLaunchKernelGGL((attn_bwd_delta_kernel<D>), dim3((unsigned)((rows + RPB - 1) / RPB)), dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// The backward with dS kept: statistics, then dK/dV and dQ for as many K/V heads at a time as the
// workspace holds dS of.
template <int D, bool CAUSAL>
static int launch_bwd_ds(BwdArgs a, hipStream_t st)
{
    if (launch_delta<D>(a, st)) return -1;
    const int BHkv = a.BH / a.group, n_chunk = (BHkv + a.ds_heads - 1) / a.ds_heads;
    for (int i = 0; i < n_chunk; ++i) {
        a.bkv0 = (int)((int64_t)BHkv * i / n_chunk);
        a.nkv = (int)((int64_t)BHkv * (i + 1) / n_chunk) - a.bkv0;
        if (launch_dkdv<D, CAUSAL, true>(a, st)) return -1;
        const int blocks = dq_ds_blocks(a.nkv * a.group, a.S, a.Dr, CAUSAL);
        if (blocks == 16 ? launch_dq_ds_two<D, CAUSAL>(a, st) : blocks == 8 ? launch_dq_ds<D, 8, CAUSAL>(a, st)
                         : blocks == 4 ? launch_dq_ds<D, 4, CAUSAL>(a, st) : launch_dq_ds<D, 2, CAUSAL>(a, st)) return -1;
    }
    return 0;
}

// dK/dV and dQ in one launch.
template <int D, int U, bool CAUSAL, bool SPLIT>
static int launch_bwd_pair_u(BwdArgs a, hipStream_t st)
{
    using C = PairCfg<D>;
    const int n_block = (a.Sk + C::Dkdv::kBlk - 1) / C::Dkdv::kBlk, nsplit = SPLIT && D <= 128 ? a.dq_nsplit : 1;
    a.ntile = SPLIT ? a.dkdv_items : n_block;
    a.pair_dkdv = a.ntile * a.nkv;
    a.pair_dq = (a.S + C::Dq::kBlk - 1) / C::Dq::kBlk;
    a.stats_in_dq = 0;
    if (!allow_lds(attn_bwd_pair_kernel<D, U, CAUSAL, SPLIT>, C::kLdsBytes)) return -1;
    hipLaunchKernelGGL((attn_bwd_pair_kernel<D, U, CAUSAL, SPLIT>), dim3(a.pair_dkdv + a.pair_dq * a.BH * nsplit),
                       dim3(C::Dq::kThreads), C::kLdsBytes, st, a);
    if (hipGetLastError() != hipSuccess) return -1;
    if (!SPLIT) return 0;
    const int64_t rows = D <= 128 ? (int64_t)a.BH * a.S : 0;
    a.pair_dkdv = 2 * a.nkv * n_block * (C::Dkdv::kBlk * D / 1024);
    hipLaunchKernelGGL((attn_bwd_pair_merge_kernel<D, CAUSAL>),
                       dim3((unsigned)(a.pair_dkdv + (rows + C::kMergeRows - 1) / C::kMergeRows)), dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int D, bool CAUSAL>
static int launch_bwd_pair(const BwdArgs &a, hipStream_t st)
{
    constexpr int U = narrow_columns(D);
    if (launch_delta<D>(a, st)) return -1;
    if (a.dkdv_chunk)
        return a.Dr <= U ? launch_bwd_pair_u<D, U, CAUSAL, true>(a, st) : launch_bwd_pair_u<D, D, CAUSAL, true>(a, st);
    return a.Dr <= U ? launch_bwd_pair_u<D, U, CAUSAL, false>(a, st) : launch_bwd_pair_u<D, D, CAUSAL, false>(a, st);
}

// Order of a full backward: dQ (which also forms the row statistics and stores them), then
// dK/dV (which reads them).  The separate statistics kernel runs only when they are asked for
// without dQ.
template <int D>
static int launch_bwd_d(BwdArgs a, bool causal, hipStream_t st, unsigned stages)
{
    a.bkv0 = 0;
    a.nkv = a.BH / a.group;
    if (stages == 7u && a.pair) return causal ? launch_bwd_pair<D, true>(a, st) : launch_bwd_pair<D, false>(a, st);
    if constexpr (D >= 128) {
        if (stages == 7u && a.ds_heads) return causal ? launch_bwd_ds<D, true>(a, st) : launch_bwd_ds<D, false>(a, st);
    }
    a.stats_in_dq = (stages & 5u) == 5u;
    if (stages & 4u) {
        if (causal ? launch_dq_for<D, true>(a, st) : launch_dq_for<D, false>(a, st)) return -1;
    } else if (stages & 1u) {
        if (launch_delta<D>(a, st)) return -1;
    }
    if (stages & 2u) return causal ? launch_dkdv<D, true>(a, st) : launch_dkdv<D, false>(a, st);
    return 0;
}

// Short heads, the full backward: one fused launch.  With grouped-query heads its work-group
// walks the query heads of a K/V head one after the other, which pays once there is a K/V
// head for every compute unit (measured: 10-26 % faster from 256 K/V heads on, slower below,
// where the two-kernel form spreads the query heads over the chip)
static bool takes_bwd_small(int BHkv, int group, int S, int Sk, int D)
{
    return std::max(S, Sk) <= bwd_small_max_rows(D) && (group == 1 || BHkv >= 256);
}

// Split of the dQ kernel over the keys, by an estimate of the launch, in us, with n splits of the key tiles:
//   - no mask: fixed + tiles / n * per-tile time, `alone` unsplit and `full` (the rate of a full chip) in
//     any split, of at most one work-group per compute unit;
//   - causal: the longest work-group, fixed + tiles / n * alone, or the whole work spread evenly over the
//     compute units, work-groups * (average tiles * full + n * fixed) / 256, whichever is more; and 0.3 of
//     the longest where not all work-groups with keys to walk (a query tile has one per started share of its
//     keys) are resident at once, so that some long ones start late.  Unsplit launches, of unsplit_wgs
//     work-groups heaviest first, take at least twice (three times, ..) the one at one (two, ..) times the
//     resident number;
//   - the partial results: 5 us and 0.4 us per MB.
// The number of splits of which it is least is taken if that is a twentieth below the unsplit launch.
// D = 128, causal, unsplit -> split, us: 4 heads of 2048 rows 50 -> 35 (8 splits), 8 of 2048 50 -> 37 (4),
// but 32 of 1024 34 -> 39 (2), 16 of 1024 29 -> 34 (4).  Whole backward of 8 heads of 2319 rows 53 -> 39 with
// 4, 44 with 3; of 12 heads of 3358 on 13519 keys 880 -> 797 with 2.  Over 691 problems of 256 .. 4096 rows
// and up to 20000 keys the splits taken are 1.1 % above the best ones.  Needs at least 256 query rows per
// head (a 256-row work-group must have rows to work on) -- decoding shapes have one row per head and many
// heads, and are not split.
#ifndef ATTN_F16  // functions of the shape only: defined once, by the bf16 build
int longest_split_plan(const LongestCost &c, int64_t wgs, int tiles, float average, size_t part_bytes, bool causal,
                       int most, int S, int64_t unsplit_wgs)
{
    auto estimate = [&](int n) {
        const float alone = n > 1 ? c.alone_split : c.alone;
        const int per = (tiles + n - 1) / n;
        const float merge = n > 1 ? 5.0f + 0.4e-6f * (float)part_bytes * n : 0.0f;
        if (!causal) return c.fixed + per * (n > 1 ? c.full : alone) + merge;
        const float longest = c.fixed + per * alone, load = wgs * (average * c.full + n * c.fixed) / 256.0f;
        float t = std::max(longest, load);
        if (!unsplit_wgs) {
            if (n * wgs > c.resident) t += 0.3f * longest;
        } else if (n > 1) {
            if (wgs * std::min((float)n, average / per + 0.5f) > c.resident) t += 0.3f * longest;
        } else {
            for (int64_t j = c.resident, rounds = 2; j < unsplit_wgs; j += c.resident, ++rounds)
                t = std::max(t, rounds * (c.fixed + alone * (tiles - S / 64.0f * j / unsplit_wgs)));
        }
        return t + merge;
    };
    int best = 1;
    float least = 0.95f * estimate(1);
    for (int n = 2; n <= most && 4 * n <= tiles && n * wgs <= (causal ? 1024 : 256); ++n) {
        const float t = estimate(n);
        if (t < least) { least = t; best = n; }
    }
    return best;
}

int dq_split_plan(int BH, int S, int Sk, int D, bool causal, int *kps, int most)
{
    if (D > 128) {  // the kernel for head dimensions above 128 is not split
        if (kps) *kps = (Sk + 63) / 64 * 64;
        return 1;
    }
    const int64_t wgs = (int64_t)BH * ((S + 255) / 256);
    const int tiles = (Sk + 63) / 64;
    int nsplit = 1;
    if (S >= 256)
        // (the unsplit launch mostly has work-groups of 128 rows, the split one of 256)
        nsplit = longest_split_plan(D > 64 ? LongestCost{7.0f, 1.38f, 1.6f, 2.2f, 256} : LongestCost{7.0f, 0.94f, 1.0f, 1.6f, 512},
                                    wgs, tiles, tiles - S / 128.0f, (size_t)BH * S * D * 4, causal, std::min(most, 16),
                                    S, dq_waves(BH, S, Sk, D, causal, false) == 8 ? wgs : (int64_t)BH * ((S + 127) / 128));
    const int tiles_per = (tiles + nsplit - 1) / nsplit;
    nsplit = (tiles + tiles_per - 1) / tiles_per;  // no empty split
    if (kps) *kps = tiles_per * 64;
    return nsplit;
}

// Sum of floor((a i + b) / m) for i = 0 .. n - 1 (all of them >= 0, m > 0): the whole parts of the quotients at
// once, and of what is left, below the line, the lattice points counted the other way round.
static int64_t floor_sum(int64_t n, int64_t m, int64_t a, int64_t b)
{
    if (n <= 0) return 0;
    const int64_t whole = n * (n - 1) / 2 * (a / m) + n * (b / m);
    a %= m; b %= m;
    const int64_t top = (a * (n - 1) + b) / m;  // the last term
    // (value j is reached from i = ceil((m j - b) / a) on)
    return top ? whole + top * n - floor_sum(top, a, m, m - b + a - 1) : whole;
}

// Chunks of at most L slots that the key blocks of a K/V head are cut into.  The plans try many L: a loop over the
// blocks for each took up to 48 us (one head of 471 rows on 16714 keys), this 1.
struct BlockChunks {
    int64_t flat, falling, longest, shortest, step;  // blocks with all slots, and with `step` fewer each to the last
    BlockChunks(int n_block, int keys, int group, int S, int Sk, bool causal)
        : longest(dkdv_slots(0, keys, group, S, Sk, causal)), shortest(dkdv_slots(n_block - 1, keys, group, S, Sk, causal)),
          step((int64_t)group * (keys / 32))
    {
        // (causal: block kt starts at slot (kt * keys - (Sk - S)) / 32, keys being a multiple of 32)
        flat = causal ? std::min<int64_t>(n_block, (Sk - S) / keys + 1) : n_block;
        falling = n_block - flat;
    }
    int64_t of(int64_t L) const
    {
        return flat * ((longest + L - 1) / L) + floor_sum(falling, L, step, shortest + L - 1);
    }
};

// Whether the unsplit dK/dV kernel at D = 65 .. 128 is that of attn_bwd_solo.hip: where an estimate of the launch is
// below that of the pairs.  A work-group takes a fixed time and one per slot.  Without a mask all of them are equal and
// run in rounds of one per unit.  Under one the launch takes as long as the work spread evenly, and no less than r
// times its work-group number 256 (r - 1) for any r, longest first, as some unit runs r of those up to it: with more
// keys than rows most key blocks see every slot, and these run in rounds too.  (Per key a slot of 256 takes 0.84 of the
// time of one of 128 or 192, but its rounds are coarser, more of the last key block and of the diagonal is idle, and
// one wave per SIMD waits for its K and V alone.)  The constants, relative ones, are fits to the difference of the two in
// whole backwards of D = 80 .. 128.  Without a mask: of 412 of 1 .. 4096 rows the rule takes 0.921 of the time of the
// pairs on average (the better of the two 0.920), none more than 1.041.  Causal, 984 of 1 .. 16384 rows, a third of them
// square: 0.980 (0.975), 25 more than 1.02, the most 1.19 (152 heads on 76 of 212 rows on 804 keys); with the work spread
// evenly alone, and the constants of the other mask, 95 of the first 698 were, one 1.30 (88 heads on 22 of 583 rows on 2989
// keys 235 | 306 us).  Where dS is not stored this kernel gains more, 320 heads of 2048 rows 1247 | 1207 us (stored 1165 |
// 1172), 256 of 3000 2002 | 1919: 3 % more may be estimated for it there.
// 150 more causal ones, drawn among those that take this kernel: 0.967 of the pairs, 22 above 1.02, the most 1.24 (9 heads of
// 958 rows on 7320 keys 86 | 106).
// us, whole backward: B=4 H=32 S=4096 2921 -> 2735, causal 1625 -> 1580; B=1 H=16 S=16384 causal 2835 -> 2690; 104 heads
// on 26 of 1156 rows D = 96 271 -> 232; but 256 of 372 causal 65 | 77.
bool dkdv_takes_solo(int BHkv, int group, int S, int Sk, bool causal, bool stored)
{
    const int64_t units = 256;
    auto time = [&](int keys, float fixed, float slot) {
        const int n_block = (Sk + keys - 1) / keys;
        const int64_t wgs = (int64_t)BHkv * n_block;
        auto length = [&](int64_t wg) { return fixed + slot * dkdv_slots((int)(wg / BHkv), keys, group, S, Sk, causal); };
        if (!causal) return (wgs + units - 1) / units * length(0);
        const BlockChunks head(n_block, keys, group, S, Sk, causal);
        float t = BHkv * (fixed * n_block + slot * head.of(1)) / units;
        for (int r = 0; r < 16 && r * units < wgs; ++r) t = std::max(t, (r + 1) * length(r * units));
        return t;
    };
    if ((int64_t)BHkv * ((Sk + 127) / 128) < units) return false;
    const bool six = (int64_t)BHkv * ((Sk + 191) / 192) >= 512;
    if (!causal) return time(256, 7.7f, 1.026f) < 0.98f * (six ? time(192, 2.0f, 0.916f) : time(128, 3.6f, 0.611f));
    return time(256, 6.2f, 1.026f) < (stored ? 1.0f : 1.03f) * (six ? time(192, 2.9f, 0.82f) : time(128, 4.2f, 0.475f));
}

// Split the dK/dV kernel over the query slots when its work-groups (one per key block of a K/V head)
// leave compute units idle: few K/V heads, e.g. grouped-query heads, whose one work-group per block
// walks the slots of every query head of the group.  The slots of a key block are cut into chunks of
// equal length, the shortest for which all chunks of the launch are resident at once (256 compute
// units; two work-groups fit one at D = 64), at least 16 slots each; blocks of one chunk write their
// result directly.  Whole backward, unsplit -> split, us: B=2 Hq=16 Hkv=4 S=1537 D=96 causal (104
// blocks, the first with 196 slots) 208 -> 129, without mask 226 -> 176; B=1 H=8 S=2048 D=128 causal
// 89 -> 74; B=1 H=4 S=8192 D=64 causal 235 -> 192; B=1 H=8 S=2048 D=64 71 -> 67.  Not below 48 slots in
// the longest block, where the merge (about 5 us) takes most of what is gained and dK and dV keep
// the one order of their sums that does not depend on the workspace; nor unless a chunk is at most
// three quarters of the longest block.  At D = 64, where chunks share a unit two by two (each takes 1.7
// times as long; two unsplit blocks, of unequal length under a mask, 1.1 times), nor unless a chunk and the
// merge (3 us and 0.4 us per MB of partial results) take less than the longest block, at 0.65 us a slot: split
// in two, 208 blocks of 50 slots 57 -> 68 us, 240 of 96 101 -> 107; 174 of 640 510 -> 470 (whole backwards).
// Of 700 problems of 90 blocks and more, timed both ways, two are 3 .. 4 % slower for the choice; split
// whenever it could be, the 700 were 0.9 % slower on average and single ones up to 19 %.
int dkdv_split_plan(int BHkv, int group, int S, int Sk, int D, bool causal, int *chunk, int64_t most)
{
    const int keys = dkdv_split_keys(D), n_block = (Sk + keys - 1) / keys;
    const int64_t resident = D == 64 ? 512 : 256;
    *chunk = 0;
    if ((int64_t)BHkv * n_block >= resident) return n_block;
    const int longest = dkdv_slots(0, keys, group, S, Sk, causal);
    if (longest < 48) return n_block;
    const BlockChunks head(n_block, keys, group, S, Sk, causal);
    int64_t L = (head.of(1) * BHkv + resident - 1) / resident;
    if (L < 16) L = 16;
    for (; 4 * L <= 3 * (int64_t)longest; L += (L + 31) / 32) {
        const int64_t items = head.of(L);
        if (items * BHkv <= std::min(resident, most)) {
            const int64_t chunks = items * BHkv;
            if (D == 64 && 0.65f * L * (chunks > 256 ? 1.7f : 1.0f) + 3.0f + 0.4e-6f * chunks * (2 * 128 * 64 * 4) >=
                               0.65f * longest * ((int64_t)BHkv * n_block > 256 ? 1.1f : 1.0f))
                return n_block;
            *chunk = (int)L;
            return (int)items;
        }
    }
    return n_block;
}

bool bwd_is_small(int BHkv, int group, int S, int Sk, int D) { return takes_bwd_small(BHkv, group, S, Sk, D); }

// dS kept for dQ (above D = 64): K/V heads whose dS is held at a time in `room` bytes, 0: dS is not kept.
// The dK/dV kernel stores it once (11 .. 15 % longer: the stores) and the dQ kernel then has one product per
// tile instead of three and waits for dS: by the counters it reads 6.1 TB/s with 16 heads of 16384 rows, 4.4 .. 5.2 with
// many of 2048 .. 4096 (D = 256: 4.8), 3.0 .. 3.5 in the short launches of few rows on long keys.  Whole backward, before ->
// after, us: B=4 H=32 S=4096 D=128 3322 -> 3186, causal 1818 -> 1722; B=1 H=16 S=16384 causal 3270 -> 3083; B=4 H=16
// S=4096 D=256 causal 2046 -> 1707; 8 heads of 1683 rows 78 -> 62; 4 of 2415 D=256 161 -> 102.
// At D = 64 dQ's products are half as long and dS as large: 64 heads of 8192 rows causal have 4.3 GB of
// it, 0.75 ms to read against 0.78 for the whole dQ kernel that does not.
// Not for one or two long heads at D <= 128, whose dQ is better split over the keys (one of 12784 rows
// causal 181 -> 212, two of 4842 108 -> 110), nor in parts of fewer than 1024 key blocks (four rounds): each
// part ends with a launch's tail, two launches over (16 heads of 16384 rows, causal, eight at a time 3055,
// four 3350; 128 heads of 4096 32 at a time 3115, causal 1710, sixteen 3050 and 1900).
int ds_plan(int BHkv, int group, int S, int Sk, int D, bool causal, size_t room)
{
    if (D < 128 || takes_bwd_small(BHkv, group, S, Sk, D)) return 0;
    if (D == 128 && S >= 2048 && (int64_t)BHkv * group * ((S + 127) / 128) <= 128) return 0;
    const size_t n = std::min<size_t>(BHkv, room / ((size_t)group * ds_head_blocks(S, Sk, causal) * (kDsBlock * 2)));
    if (n == 0 || n == (size_t)BHkv) return (int)n;
    const int parts = (int)((BHkv + n - 1) / n), keys = dkdv_split_keys(D);
    return (int64_t)(BHkv / parts) * ((Sk + keys - 1) / keys) < 1024 ? 0 : (BHkv + parts - 1) / parts;
}

// dK/dV and dQ in one launch, when all work-groups of both kernels find a compute unit of their own: one
// kernel after the other leaves most units idle twice, and three launches (four with the statistics where
// dS is kept, two merges) cost more than the products of such calls.  Both are cut, dQ over the keys and
// dK/dV over the query slots, as long as the chunks still have a unit each.  The launch takes as long as its
// longest work-group: fixed + slots * slot or dq_fixed + tiles * dq_tile us, and, cut, a merge; the cut
// with the least is compared with the same estimate of the two kernels one after the other (constants of
// both: a fit to 160 problems of up to 256 work-groups, 3 .. 9 % rms).  Whole backward, us: 6 heads of 940
// rows D = 64 causal 35 -> 19, 12 of 1037 44 -> 33, 1 of 1181 D = 96 45 -> 23, 3 of 2099 D = 128 causal 58 ->
// 36, 9 of 329 D = 64 causal 22 -> 15, 3 of 134 D = 256 causal 23 -> 16; 0.75 on average over 200 random
// problems; against dS kept one of them is slower by more than 2 % (36 -> 9 heads of 75 rows D = 256: 30.5 -> 33), against
// dQ, then dK/dV none of 1600 by more than 1.3 %.  Not beyond a
// work-group per unit: 26 heads of 1776 rows D = 128 causal 101 -> 110, 13 of 4773 D = 64 175 -> 198 (uncut).
PairPlan pair_plan(int BHkv, int group, int S, int Sk, int D, bool causal, size_t room)
{
    PairPlan best = {};
    if (takes_bwd_small(BHkv, group, S, Sk, D)) return best;
    constexpr int64_t units = 256;
    const int keys = dkdv_split_keys(D), n_block = (Sk + keys - 1) / keys;
    const int dq_rows = D > 128 ? 128 : 256, dq_keys = D > 128 ? 32 : 64, tiles = (Sk + dq_keys - 1) / dq_keys;
    const int64_t heads = (int64_t)BHkv * group, wgs = (int64_t)BHkv * n_block, dq_wgs = heads * ((S + dq_rows - 1) / dq_rows);
    if (wgs + dq_wgs > units) return best;
    const BlockChunks head(n_block, keys, group, S, Sk, causal);
    const size_t dq_bytes = (size_t)heads * S * D * 4, chunk_bytes = (size_t)2 * keys * D * 4;
    const PairCost c = D > 128  ? PairCost{11.0f, 0.87f, 11.0f, 1.10f, 3.0f, 0.35e-6f}
                       : D > 64 ? PairCost{9.1f, 0.67f, 9.5f, 1.65f, 3.7f, 0.34e-6f}
                                : PairCost{7.9f, 0.57f, 8.0f, 1.03f, 3.1f, 0.43e-6f};
    best.items = n_block; best.dq_nsplit = 1; best.dq_kps = tiles * dq_keys;
    const int longest = (int)head.longest;
    const int64_t slots = BHkv * head.of(1);
    float least = std::max(c.fixed + longest * c.slot, c.dq_fixed + tiles * c.dq_tile);
    for (int n = 1; n <= (D > 128 ? 1 : 16) && (n == 1 || 4 * n <= tiles) && n * dq_wgs < units; ++n) {
        const int per = (tiles + n - 1) / n;
        if ((tiles + per - 1) / per != n) continue;
        const float dq_us = c.dq_fixed + per * c.dq_tile + c.merge;
        if (dq_us >= least) continue;
        const int64_t left = units - n * dq_wgs;
        if (left < wgs) break;  // (not a chunk for every block)
        int L = (int)std::max<int64_t>((slots + left - 1) / left, std::min(8, longest));
        int64_t items = 0;
        auto walk_us = [&] { return c.fixed + L * c.slot + c.merge; };
        for (; L <= longest && walk_us() < least; L += (L + 15) / 16) {
            items = BHkv * head.of(L);
            if (items <= left) break;
        }
        if (L > longest || walk_us() >= least) continue;
        const size_t part = (D > 128 ? 0 : (n * dq_bytes + 255) / 256 * 256) + items * chunk_bytes;
        const float t = std::max(walk_us(), dq_us) + c.byte * part;
        if (part > room || t >= least) continue;
        least = t;
        best.dq_nsplit = n; best.dq_kps = per * dq_keys;
        best.dkdv_chunk = L; best.items = (int)(items / BHkv);
    }
    // the two kernels one after the other
    int chunk = 0, kps = 0;
    const int64_t items = (int64_t)BHkv * dkdv_split_plan(BHkv, group, S, Sk, D, causal, &chunk);
    const float walk = chunk ? chunk : longest;
    size_t part = chunk ? items * chunk_bytes : 0;
    int merges = chunk ? 1 : 0;
    float t;
    if (ds_plan(BHkv, group, S, Sk, D, causal, ~(size_t)0)) {  // (not by the room: the same choice in the best size)
        t = D > 128 ? 16.5f + 0.87f * walk + 9.9f * merges + 0.47f * ((Sk + 31) / 32)
                    : 12.2f + 0.75f * walk + 9.3f * merges + 0.23e-6f * part + 0.256f * ((Sk + 31) / 32);
    } else {
        const int n = dq_split_plan((int)heads, S, Sk, D, causal, &kps);
        const float per = n > 1 ? kps / dq_keys : tiles;
        if (n > 1) { ++merges; part += n * dq_bytes; }
        t = D > 64 ? 8.7f + 0.39f * walk + 7.9f * merges + 0.24e-6f * part + 2.95f * per
                   : 9.9f + 0.59f * walk * (items > 256 ? 1.4f : 1.0f) + 4.1f * merges + 0.47e-6f * part + 0.8f * per;
    }
    best.taken = least < 0.95f * t;
    return best;
}
#endif

int launch_bwd(const BwdArgs &a, int D, bool causal, hipStream_t st, unsigned stages)
{
    if (stages == 7u && takes_bwd_small(a.BH / a.group, a.group, a.S, a.Sk, D)) return launch_bwd_small(a, D, causal, st);
    return D == 256 ? launch_bwd_d<256>(a, causal, st, stages)
         : D == 128 ? launch_bwd_d<128>(a, causal, st, stages)
                    : launch_bwd_d<64>(a, causal, st, stages);
}

}  // namespace attn
