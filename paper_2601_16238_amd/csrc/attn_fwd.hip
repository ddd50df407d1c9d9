// Fused attention forward for gfx950: O = softmax(scale * Q K^T [+ causal mask]) V and the
// per-row natural-log LSE, one pass over K/V with an online softmax (the
// "flash-attention-style formulation" the paper's debugging table refers to).
//
// Work decomposition
//   work-group = NW waves, one tile of BR = 32*NW query rows of one (batch, head);
//   wave       = 32 query rows; loops over key tiles of BC = 64 rows staged in LDS.
// The score tile is computed TRANSPOSED, S^T = K Q^T (keys x queries), with the
// 32x32x16 elem MFMA.  Its accumulator layout puts one query per lane (column l%32) and
// 16 keys per lane and 32-key block, so
//   - row max / row sum are in-lane reductions plus ONE exchange with lane l^32,
//   - the rescale factor alpha is a per-lane scalar,
//   - elem(P^T) is already in the B-operand layout of the second MFMA,
//     O^T = V^T P^T (d x queries), once the contraction index is enumerated in the order
//     the accumulator holds it (key = 8*(t/4) + 4*(l/32) + t%4 within 16 keys).
// K and V tiles reach LDS by direct global -> LDS transfers, both row-major.  The K operand is a
// plain 16-byte read; V^T is produced by the reads themselves (two LDS transpose reads per
// fragment, which deliver the keys in exactly that order).  Staging V through registers with a
// 4x4 register transpose, so that its operand is a plain read as well, costs more vector
// instructions than the slower transpose reads do (measured in the kernel: 3-5 % slower).
//
// Software pipeline (per wave): the MFMAs of S^T(j+1) are issued in the same block as the
// softmax arithmetic of tile j, so the matrix pipe and the vector ALU overlap inside one
// wave as well as across the two waves of a SIMD.  The vector ALU issue port is the scarce
// resource (it also carries the MFMA issue and the LDS read returns), so the common path
// does no max reduction at all: probabilities are taken relative to a reference max that is
// only moved when a partial row sum shows that some probability outgrew 2^10 (the O
// accumulator and row sum are then rescaled and the sub-tile redone).  Any reference gives
// the same O and LSE after the final division by the row sum.
#include "attn_device.hpp"
#include "attn_launch.hpp"

#include <algorithm>
#include <cmath>

namespace attn {

// MAIN: the form with the pipelined main loop (eight waves always; four waves at D = 64 in launches that
// fwd_takes_main chooses).
template <int D, int NW, bool MAIN>
struct FwdCfg {
    static constexpr int kThreads = NW * 64;
    static constexpr int kBR = NW * 32;
    static constexpr int kBC = 64;
    // K tile: in pieces (see Pieces), one wave-wide transfer each.  The fragment a lane needs for
    // contraction step ks is at a per-lane constant plus a distance that is known at compile time --
    // one address register instead of one per step.
    using L = Pieces<D>;
    static constexpr int kKDmas = kBC / L::kRows;              // transfers per tile
    static constexpr int kKTile = L::base(kKDmas) / 2;         // in elements
    static constexpr int kKHalf = kKTile / 2;                  // 32 rows further
    static constexpr int kKDmaPerWave = (kKDmas + NW - 1) / NW;
    // V tile: the same transfers and layout as the K tile; it is transposed by the reads (LDS transpose
    // read).
    static constexpr int kVTile = kKTile;                      // in elements
    static constexpr int kVRows16 = L::kRows16;                // 16 rows further, in bytes
    static constexpr bool kMain = MAIN;
    // V tiles: two, or three for the main loop, which multiplies P of a sub-tile by V one sub-tile
    // later and therefore still reads tile kt-1 while tile kt+1 is arriving
    static constexpr int kVBufs = kMain ? 3 : 2;
    // The query rows reach the registers through LDS (see the kernel's prologue):
    // the 64 rows of a pair of waves are staged like a K tile, pair 0 in K buffer 2, pair 1 in
    // V buffer 1 (both free until the first tile barrier), pairs 2 and 3 behind the V buffers.
    static constexpr int kQStage = NW == 8 ? 2 * kKTile : 0;
    static constexpr int kLdsBytes = (3 * kKTile + kVBufs * kVTile + kQStage) * 2;
    static_assert(kLdsBytes <= 160 * 1024, "LDS budget of a gfx950 CU exceeded");
};

// A sub-tile's probabilities are taken relative to a reference max that is only moved when
// one lane's partial row sum (16 keys) exceeds this bound, i.e. some exp2 argument > ~10.
constexpr float kOverflow = 1024.0f;
constexpr float kMinusHuge = -1.0e30f;  // initial reference: finite, so masked -inf scores give 0

// U: columns that the products run over, a multiple of 32 up to D; the others are zeros (tensors of a
// smaller head dimension).  The layouts are those of D.
template <int D, int U, int NW, bool CAUSAL, bool SPLIT, bool MAIN>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
attn_fwd_kernel(const FwdArgs a)
{
    using C = FwdCfg<D, NW, MAIN>;
    constexpr int KS = U / 16;  // contraction steps of K Q^T
    constexpr int DB = U / 32;  // 32-row blocks of O^T
    extern __shared__ __attribute__((aligned(16))) char smem[];
    elem *Ks = reinterpret_cast<elem *>(smem);  // [3][64][D] swizzled
    elem *Vs = Ks + 3 * C::kKTile;              // [kVBufs] tiles in the K tile's layout

    const int tid = threadIdx.x, l = tid & 63, r = l & 31, h = l >> 5;
    const int w = tid >> 6;
    const int S = a.S, Dr = a.Dr;

    // (head, query tile) of this work-group; causal tiles are issued heaviest first.
    int bh, rank;
    xcd_tile_order<CAUSAL, MAIN && NW == 4, (MAIN && NW == 4 ? 8 : 4)>(blockIdx.x, a.nqt, a.BH, bh, rank);
    const int qt = CAUSAL ? a.nqt - 1 - rank : rank;
    const int64_t base = (int64_t)(bh / a.H) * a.stride_b + (int64_t)(bh % a.H) * a.stride_h;
    // grouped-query heads: query head h reads K/V head h / group
    const int64_t base_kv = (int64_t)(bh / a.H) * a.kv_stride_b +
                            (int64_t)((bh % a.H) / a.group) * a.kv_stride_h;
    const elem *Qp = a.Q + base, *Kp = a.K + base_kv, *Vp = a.V + base_kv;
    // Keys seen by this work-group: all Sk of them, or one split's range (then K and V are
    // simply re-based to the range and the causal offset moves with them).  Query row i sees
    // key j iff j <= i + coff.
    int Sk = a.Sk, coff = a.Sk - S;
    if (SPLIT) {
        const int k_begin = blockIdx.y * a.kps;  // < Sk by the launcher's plan
        Kp += (int64_t)k_begin * a.kv_stride_s;
        Vp += (int64_t)k_begin * a.kv_stride_s;
        Sk = min(Sk - k_begin, a.kps);
        coff -= k_begin;
    }

    const int q0 = qt * C::kBR + w * 32;  // first query row of this wave
    const int q = q0 + r;                 // this lane's query row
    const int qc = q < S ? q : S - 1;     // clamped for loads; rows >= S are never stored

    // Q fragments, B operand of K Q^T: lane holds Q[q][16*ks + 8h .. +7].  A lone wave loads them
    // straight from memory.  Others take them through LDS (below): a load in which every lane
    // fetches 16 bytes of its own row touches 32 rows per instruction, and the 64 such instructions of
    // a work-group of eight waves took its last wave 5000-7000 cycles to get issued (measured) -- time
    // in which the compute unit, which holds one such work-group, does nothing.  With fewer waves
    // (this and the rows of O below; us): 2 heads of 128 rows D = 64 5.3 -> 4.7, 512 of 200 causal 18.2 ->
    // 16.4, 64 of 1024 causal 19.2 -> 18.5, 768 of 65 the same.  Not for narrow tensors, whose rows are half (three
    // quarters) of what is then moved: 512 of 41 rows D = 16 4.4, 4.9 through LDS, 4096 of 41 D = 32 causal 19.9 and 21.2, 32 of
    // 214 D = 80 causal 8.3 and 8.7.
    constexpr bool kNarrow = U < D && NW < 8;
    constexpr bool kStageQ = NW > 1 && !kNarrow;
    elem8 qf[KS];
    if constexpr (!kStageQ) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qf[ks] = as_elem8(ld_row16(Qp + (int64_t)qc * a.stride_s, ks * 16 + 8 * h, Dr));
    }

    // Key tiles this work-group visits.
    const int q_end = min(S, (qt + 1) * C::kBR);
    const int k_end = CAUSAL ? min(Sk, q_end + coff) : Sk;  // <= 0: nothing visible (splits only)
    const int n_kt = k_end > 0 ? (k_end + C::kBC - 1) / C::kBC : 0;
    const int q0e = q0 + coff;  // the wave's first row in key coordinates

    // ---- staging: global -> LDS.  Rows past S-1 and tiles past the last one
    // lie outside the head's buffer resource and read as zero (masked to probability 0).
    // Columns Dr..D-1 (head dimensions below the kernel's D) are fetched at an offset past the
    // end of the resource, so they read as zero like everything else outside it.
    const uint32_t head_bytes = (uint32_t)(((int64_t)(Sk - 1) * a.kv_stride_s + Dr) * 2);
    const desc_t Kd = make_desc(Kp, head_bytes), Vd = make_desc(Vp, head_bytes);
    const uint32_t lds0 = lds_address(smem);
    const uint32_t row_bytes = (uint32_t)a.kv_stride_s * 2u;
    const uint32_t tile_bytes = C::kBC * row_bytes;
    // K and V go global -> LDS directly (no registers): one wave-wide transfer of 16 B per lane
    // fills 1 KB of LDS in lane order; lane l fetches the chunk that belongs at its position of the
    // piece.  The piece's first row goes into the scalar
    // offset (which takes part in the range check like the per-lane one).  The transfers are
    // issued from assembly, out of the compiler's sight (it would otherwise make the wave wait for
    // all of them before its next transpose read of LDS); tile_barrier() orders them against the
    // reads.  They fill buffers that nobody reads before the next barrier.
    using L = typename C::L;
    constexpr int PR = L::kRows;
    const uint32_t k_voff = L::lane_offset(l, row_bytes, Dr, head_bytes);
    auto dma_tile = [&](desc_t desc, uint32_t lds_tile, int kt) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < C::kKDmaPerWave; ++n) {
            // which 1 KB piece of the tile: wave-uniform
            const int ii = __builtin_amdgcn_readfirstlane(w) + n * NW;
            if (C::kKDmas % NW == 0 || ii < C::kKDmas)
                dma16_between(desc, lds_tile + L::base(ii), k_voff, kt * tile_bytes + ii * PR * row_bytes);
        }
    };
    auto dma_k = [&](int kt, int buf) __attribute__((always_inline)) {
        dma_tile(Kd, lds0 + buf * (C::kKTile * 2), kt);
    };
    auto dma_v = [&](int kt, int buf) __attribute__((always_inline)) {
        dma_tile(Vd, lds0 + (3 * C::kKTile + buf * C::kVTile) * 2, kt);
    };

    float m = kMinusHuge;  // reference max of c*s (log2 units), identical in lanes l and l^32
    float lsum = 0.f;     // running sum of this lane's half of the keys
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
    const float c = a.scale_log2e;

    // ---- MFMA steps and their LDS operand fetches.  Work proceeds in sub-tiles of 32 keys
    // (one 32x32 score block per wave).  One step is four (D=128) MFMAs whose A fragments
    // are fetched a step ahead into the other of two fragment sets, so the LDS latency hides
    // behind the previous step's MFMAs.
    constexpr int NKQ = (KS + 3) / 4;  // K Q^T steps per sub-tile, up to four contraction steps each
    // element offset of this lane's fragment for contraction step 0 within a 32-row half
    // tile: chunk h of row r
    // The per-lane parts of the LDS addresses are kept in one register each and made opaque to
    // the compiler, so that buffer, sub-tile and step are folded into the 16-bit immediate
    // offset of the LDS instruction instead of into further address registers.  (The V region
    // starts beyond what an immediate reaches from zero, so its registers include its base.)
    int k_lane = L::at(r, h);
    // transpose reads of a V tile: the 16-lane group reads rows 4h + e (e = 0..3; +8 for the
    // second read), 64 bytes of d block 0 of each row -- the keys of contraction half h in the
    // order the accumulator of S^T holds them
    int v_lane0 = 3 * C::kKTile * 2 + L::at(4 * h + ((l & 15) >> 2), 2 * ((l >> 4) & 1) + ((l >> 1) & 1)) + (l & 1) * 8;
    int v_lane1 = 3 * C::kKTile * 2 + L::at(8 + 4 * h + ((l & 15) >> 2), 2 * ((l >> 4) & 1) + ((l >> 1) & 1)) + (l & 1) * 8;
    asm volatile("" : "+v"(k_lane), "+v"(v_lane0), "+v"(v_lane1));
    auto ld_k = [&](const elem *Kt, int kq, elem8 (&f)[4]) {
#pragma unroll
        for (int t = 0; t < 4 && 4 * kq + t < KS; ++t)
            f[t] = *(const elem8 *)((const char *)Kt + L::step(4 * kq + t) + k_lane);
    };
    auto mm_k = [&](int kq, const elem8 (&f)[4], f32x16 &t0) {
#pragma unroll
        for (int t = 0; t < 4 && 4 * kq + t < KS; ++t) t0 = mfma32(f[t], qf[4 * kq + t], t0);
    };
    // V^T fragment: lane (d = 32*db + l%32, half h) gets the 8 keys of contraction step cc
    // that its half owns, from two transpose reads.  Vt: byte offset of tile and sub-tile
    // within the V region.
    auto ld_v = [&](int Vt, int cc, elem8 (&f)[4]) {
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const char *p = smem + Vt + cc * C::kVRows16 + db * L::kBlock;
            f[db] = join8(lds_read_tr((const elem *)(p + v_lane0)), lds_read_tr((const elem *)(p + v_lane1)));
        }
    };
    // Row sums of the ROUNDED probabilities (one packed dot product with a vector of ones per
    // element pair; this lane's half of the keys, both halves are added at the end like the
    // exact sum).  O is divided by this sum, so that the rounding of P cancels between
    // numerator and denominator: the reference max is not the true row max, so the dominant
    // probability of a peaked row is in general not exactly representable, and dividing by the
    // exact sum would leave its rounding error (up to 2^-9 relative) in O.  LSE is still made
    // from the exact fp32 sum.
    float hsum = 0.f;
    auto mm_v = [&](const elem8 (&f)[4], elem8 p) {
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] = mfma32(f[db], p, o[db]);
#pragma unroll
        for (int i = 0; i < 4; ++i) hsum = dot2_acc(p[2 * i], p[2 * i + 1], hsum);
    };
    // exp2 of eight scores against the reference max, fp32 row-sum, and elem pack
    auto softmax8 = [&](const f32x16 &t, int i0, float &psum) -> elem8 {
        float e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            e[i] = fast_exp2(__builtin_fmaf(t[i0 + i], c, -m));
            psum += e[i];
        }
        return pack8(e[0], e[1], e[2], e[3], e[4], e[5], e[6], e[7]);
    };
#define ATTN_FENCE() __builtin_amdgcn_sched_barrier(0)

    // One 32-key sub-tile g = 2*kt + u for an active wave: softmax and P V of sub-tile g
    // (scores in cur) overlapped with S^T of sub-tile g+1 (into nxt; one sub-tile past the
    // end reads zero rows and is unused).  Four fragment sets rotate through the steps
    //   K0 (f0), K1 (f1): S^T(g+1) += K Q^T      V0 (f2), V1 (f3): O^T += V^T P^T(g)
    // and every set is fetched two steps before it is consumed; the K fragments of sub-tile
    // g+2 (tile kt+1, resident since the previous iteration) are fetched during V0/V1.
    elem8 f0[4], f1[4], f2[4], f3[4];
    // The reference max moves to the true running max: rescale what has been accumulated and
    // redo the probabilities of the sub-tile whose scores are in cur.
    auto move_reference = [&](const f32x16 &cur, elem8 &p0, elem8 &p1, float &psum)
                              __attribute__((always_inline)) {
        float mx = cur[0];
#pragma unroll
        for (int i = 1; i < 16; i += 3)
            mx = fmaxf(mx, fmaxf(cur[i], fmaxf(cur[i + 1], cur[i + 2])));
        mx = xhalf_max(mx) * c;
        const float m_new = fmaxf(m, mx);
        const float alpha = fast_exp2(m - m_new);
        m = m_new;
        lsum *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
        hsum *= alpha;
        psum = 0.f;
        p0 = softmax8(cur, 0, psum);
        p1 = softmax8(cur, 8, psum);
    };
    // vb: buffer of V(kt); vb_fill: buffer that takes V(kt+1)
    auto subtile = [&](int kt, int u, int kbuf_next, int kbuf_fill, int vb, int vb_fill, bool masked,
                       f32x16 &cur, f32x16 &nxt) __attribute__((always_inline)) {
        const elem *Kn = Ks + kbuf_next * C::kKTile + u * C::kKHalf;  // rows of sub-tile g+2
        const int Vt = vb * (C::kVTile * 2) + 2 * u * C::kVRows16;
        // ---- K0
        ld_v(Vt, 0, f2);
        if (NKQ == 1) ld_v(Vt, 1, f3);
        if (u == 0) dma_k(kt + 2, kbuf_fill);  // K(kt+2) -> the buffer freed at the last barrier
#pragma unroll
        for (int i = 0; i < 16; ++i) nxt[i] = 0.f;
        if (masked) {
            // Ragged tail and causal mask: only sub-tiles that touch the end or the diagonal.
            const int lim = (CAUSAL ? min(qc + coff, Sk - 1) : Sk - 1) - (kt * C::kBC + 32 * u) - 4 * h;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (8 * (i / 4) + (i % 4) > lim) cur[i] = -INFINITY;
        }
        float psum = 0.f;
        elem8 p0 = softmax8(cur, 0, psum);
        mm_k(0, f0, nxt);
        ATTN_FENCE();
        // ---- K1
        if (NKQ > 1) {
            ld_v(Vt, 1, f3);
            mm_k(1, f1, nxt);
        }
        elem8 p1 = softmax8(cur, 8, psum);
        // Rare path: some probability outgrew 2^10 relative to the reference max (always so
        // for a wave's first sub-tile).  Move the reference to the true running max, rescale
        // what has been accumulated, and redo this sub-tile's probabilities.
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(psum > kOverflow) != 0, 0)) move_reference(cur, p0, p1, psum);
        ATTN_FENCE();
        // ---- V0 (first sub-tile: V(kt+1) -> the buffer freed at the last barrier)
        ld_k(Kn, 0, f0);
        mm_v(f2, p0);
        if (u == 0 && (NW == 8 || kt + 1 < n_kt)) dma_v(kt + 1, vb_fill);
        ATTN_FENCE();
        // ---- V1
        if (NKQ > 1) ld_k(Kn, 1, f1);
        mm_v(f3, p1);
        lsum += psum;
        ATTN_FENCE();
    };

    // ---- prologue: K(0), K(1), V(0) resident; V(1) in flight; first S^T block computed and
    // the K fragments of the second sub-tile on their way.
    // The wave's 32 query rows as half of a K-layout tile, by the same direct
    // transfers (whole rows of four per instruction), issued before those of K and V.  Rows past
    // S-1 and columns Dr..D-1 read as zero.
    uint32_t q_stage = 0;
    if constexpr (kStageQ) {
        const int pair = __builtin_amdgcn_readfirstlane(w) >> 1, half = __builtin_amdgcn_readfirstlane(w) & 1;
        q_stage = (pair == 0 ? 2 * C::kKTile : pair == 1 ? 3 * C::kKTile + C::kVTile
                                                          : 3 * C::kKTile + 3 * C::kVTile + (pair - 2) * C::kKTile) * 2 +
                  half * (C::kKHalf * 2);
        const int row0 = qt * C::kBR + pair * 64;
        const int rows = min(64, S - row0);
        const uint32_t q_bytes = rows > 0 ? (uint32_t)(((int64_t)(rows - 1) * a.stride_s + Dr) * 2) : 0u;
        const desc_t Qd = make_desc(Qp + (int64_t)(rows > 0 ? row0 : 0) * a.stride_s, q_bytes);
        const uint32_t q_row_bytes = (uint32_t)a.stride_s * 2u;
        const uint32_t q_voff = L::lane_offset(l, q_row_bytes, Dr, q_bytes);
#pragma unroll
        for (int n = 0; n < C::kKDmas / 2; ++n)
            dma16_between(Qd, lds0 + q_stage + L::base(n), q_voff,
                          (half * (C::kKDmas / 2) + n) * PR * q_row_bytes);
    }
    dma_k(0, 0);
    dma_k(1, 1);
    dma_v(0, 0);
    // Rotary embedding of the query rows, fused into their load (head dimension == D only):
    // column d pairs with d + D/2, i.e. fragment ks with ks + KS/2, element by element, in this
    // lane; fp32 arithmetic on the widened values, rounded once -- what a separate rotary pass
    // would have written to memory as bf16.  The table rows are requested here, after the first
    // K and V tiles, so that all of them are in flight together, and used further down.
    f32x4 rc[KS][2], rs[KS][2];  // [ks][half of the 8 columns]; only ks < KS/2 is used
    const bool rope = U == D && a.rope_cos;
    if (rope) {
        const int64_t pos = (int64_t)(qc * a.rope_row_step + a.rope_pos0) * (D / 2);
#pragma unroll
        for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                rc[ks][j] = *(const f32x4 *)(a.rope_cos + pos + 16 * ks + 8 * h + 4 * j);
                rs[ks][j] = *(const f32x4 *)(a.rope_sin + pos + 16 * ks + 8 * h + 4 * j);
            }
    }
    if constexpr (kStageQ) {
        // the wave's own query rows have landed once at most the later transfers (K(0), K(1),
        // V(0)) are outstanding; with the rotary table rows in flight as well, whose place in the
        // order of issue is the compiler's choice, everything is awaited
        if (rope) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * C::kKDmaPerWave) : "memory");
        const char *Qs = smem + q_stage + L::at(r, h);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const elem8 *)(Qs + L::step(ks));
        // ... and are in registers before anybody may overwrite the staging space
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    if (rope) {
        elem *qr = a.Qrot ? a.Qrot + base + (int64_t)qc * a.stride_s : nullptr;
#pragma unroll
        for (int ks = 0; ks < KS / 2; ++ks) {
            float lo[8], hi[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float x1 = (float)qf[ks][t], x2 = (float)qf[ks + KS / 2][t];
                const float cc = rc[ks][t >> 2][t & 3], ss = rs[ks][t >> 2][t & 3];
                lo[t] = __builtin_fmaf(x1, cc, -(x2 * ss));
                hi[t] = __builtin_fmaf(x2, cc, x1 * ss);
            }
            qf[ks] = pack8(lo[0], lo[1], lo[2], lo[3], lo[4], lo[5], lo[6], lo[7]);
            qf[ks + KS / 2] = pack8(hi[0], hi[1], hi[2], hi[3], hi[4], hi[5], hi[6], hi[7]);
            if (qr && q < S && (!SPLIT || blockIdx.y == 0)) {
                *(elem8 *)(qr + 16 * ks + 8 * h) = qf[ks];
                *(elem8 *)(qr + 16 * (ks + KS / 2) + 8 * h) = qf[ks + KS / 2];
            }
        }
    }
    if (C::kMain && (NW == 8 || n_kt > 2)) {
        // The main loop's first iteration multiplies an all-zero P by the second half of V
        // buffer 2, which nothing has written yet: give it finite contents.
        const u32x4 z = {0u, 0u, 0u, 0u};
        for (int i = tid; i < C::kVTile / 8; i += C::kThreads)
            *(u32x4 *)(Vs + 2 * C::kVTile + 8 * i) = z;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // K(0), K(1), V(0) have landed
    __syncthreads();
    f32x16 sa, sb;
    {
#pragma unroll
        for (int i = 0; i < 16; ++i) sa[i] = 0.f;
        ld_k(Ks, 0, f0);
        if (NKQ > 1) ld_k(Ks, 1, f1);
        mm_k(0, f0, sa);
        if (NKQ > 1) mm_k(1, f1, sa);
        ATTN_FENCE();
        ld_k(Ks + C::kKHalf, 0, f0);
        if (NKQ > 1) ld_k(Ks + C::kKHalf, 1, f1);
    }

    // Main-loop form of a sub-tile (kMain, sub-tiles that the wave sees in full):
    // the probabilities of sub-tile g are multiplied by V one sub-tile LATER.  The iteration
    // then holds three independent pieces of work -- S^T(g+1) = K Q^T, the softmax arithmetic
    // of g, and O^T += V^T P^T(g-1) -- in one basic block with nothing to mask, and the test
    // whether the reference max must move sits at its end instead of between the softmax and
    // the second MFMA phase, where it made every wave wait for its last exp2 before it could
    // issue the next MFMA (measured: the same arithmetic without that branch in the middle
    // runs 15 % faster).  pp0/pp1 carry P(g-1) into the iteration; vprev is the buffer that
    // holds the V rows of sub-tile g-1 (tile kt-1 for u == 0, tile kt for u == 1).
    elem8 pp0, pp1;
#pragma unroll
    for (int i = 0; i < 8; ++i) pp0[i] = pp1[i] = (elem)0.f;
    auto subtile_main = [&](int kt, int u, int kbuf_next, int kbuf_fill, int vprev, int vb_fill,
                            f32x16 &cur, f32x16 &nxt) __attribute__((always_inline)) {
        const elem *Kn = Ks + kbuf_next * C::kKTile + u * C::kKHalf;  // rows of sub-tile g+2
        const int Vt = vprev * (C::kVTile * 2) + 2 * (1 - u) * C::kVRows16;  // rows of sub-tile g-1
        // The softmax arithmetic of g is spread evenly over the four MFMA steps (four scores
        // each), so that every step has about three quarters as many vector-ALU cycles as
        // matrix-pipe cycles.
        float e[16], psum = 0.f;
        auto exp4 = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
            for (int i = i0; i < i0 + 4; ++i) {
                e[i] = fast_exp2(__builtin_fmaf(cur[i], c, -m));
                psum += e[i];
            }
        };
        auto hsum4 = [&](elem8 p) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) hsum = dot2_acc(p[2 * i], p[2 * i + 1], hsum);
        };
        auto mm_o = [&](const elem8 (&f)[4], elem8 p) __attribute__((always_inline)) {
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] = mfma32(f[db], p, o[db]);
        };
        // ---- K0
        ld_v(Vt, 0, f2);
        if (NKQ == 1) ld_v(Vt, 1, f3);
        // (both tiles' transfers right after the barrier: the V buffer being filled was last read
        // before the previous barrier; measured the same or up to 1 % faster than V two steps later)
        if (u == 0) {
            dma_k(kt + 2, kbuf_fill);
            dma_v(kt + 1, vb_fill);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) nxt[i] = 0.f;
        exp4(0);
        hsum4(pp0);
        mm_k(0, f0, nxt);
        ATTN_FENCE();
        // ---- K1
        if (NKQ > 1) {
            ld_v(Vt, 1, f3);
            mm_k(1, f1, nxt);
        }
        exp4(4);
        hsum4(pp1);
        elem8 p0 = pack8(e[0], e[1], e[2], e[3], e[4], e[5], e[6], e[7]);
        ATTN_FENCE();
        // ---- V0
        ld_k(Kn, 0, f0);
        mm_o(f2, pp0);
        exp4(8);
        ATTN_FENCE();
        // ---- V1
        if (NKQ > 1) ld_k(Kn, 1, f1);
        mm_o(f3, pp1);
        exp4(12);
        elem8 p1 = pack8(e[8], e[9], e[10], e[11], e[12], e[13], e[14], e[15]);
        ATTN_FENCE();
        // rare: some probability of g outgrew 2^10 (always so for a wave's first sub-tile);
        // what has been accumulated (up to g-1) is rescaled, P(g) redone
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(psum > kOverflow) != 0, 0)) move_reference(cur, p0, p1, psum);
        lsum += psum;
        pp0 = p0;
        pp1 = p1;
    };
    // Every transfer this wave issued during the tile (its pieces of K(kt+2) and V(kt+1)) must
    // have landed before the other waves are let past the barrier to read them.
    auto tile_barrier = [&]() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };

    // One loop iteration = one staged tile of 64 keys = two sub-tiles.  Staging is folded
    // into the first sub-tile's steps.  During iteration kt the waves read K(kt) (second
    // half) and K(kt+1) (first half), so K is triple-buffered and K(kt+2) streams into the
    // third buffer; V(kt+1) replaces the oldest V tile, whose last readers finished before the
    // previous barrier.
    int kt0 = 0;  // first tile of the generic loop below
    if constexpr (C::kMain) {
        // Tiles that this wave sees in full (no key past the end, none above its diagonal), in
        // whole groups of three: the loop is unrolled over the three K (and V) buffers so that
        // the buffer of every access is a compile-time constant and the LDS addresses of the
        // fragments are a loop-invariant register plus an immediate offset.
        const int seen = CAUSAL ? min(Sk, q0e + 1) : Sk;  // keys 0 .. seen-1 are visible to every row of the wave
        // (rows past S: never more than n_kt; the same in every lane of the wave, and said so,
        // so that the loop is controlled by scalar registers)
        const int n_main = __builtin_amdgcn_readfirstlane(min(max(seen, 0) / C::kBC, n_kt) / 3 * 3);
        for (int kt = 0; kt < n_main; kt += 3) {
            subtile_main(kt, 0, 1, 2, 2, 1, sa, sb);
            subtile_main(kt, 1, 1, 2, 0, 1, sb, sa);
            tile_barrier();
            subtile_main(kt + 1, 0, 2, 0, 0, 2, sa, sb);
            subtile_main(kt + 1, 1, 2, 0, 1, 2, sb, sa);
            tile_barrier();
            subtile_main(kt + 2, 0, 0, 1, 1, 0, sa, sb);
            subtile_main(kt + 2, 1, 0, 1, 2, 0, sb, sa);
            tile_barrier();
        }
        if (n_main > 0) {
            // the last sub-tile's P V is still owed: second half of V(n_main - 1), buffer 2
            const int Vt = 2 * (C::kVTile * 2) + 2 * C::kVRows16;
            ld_v(Vt, 0, f2);
            ld_v(Vt, 1, f3);
            mm_v(f2, pp0);
            mm_v(f3, pp1);
        }
        kt0 = n_main;  // a multiple of three: K(kt0) and V(kt0) are in buffer 0 again
    }
    // Generic form of a tile (the tiles at the diagonal and the ragged end of the eight-wave
    // kernel; every tile with fewer waves).  kb1, kb2: buffers of K(kt+1), K(kt+2); vb, vb1:
    // buffers of V(kt), V(kt+1).
    auto tile = [&](int kt, int kb1, int kb2, int vb, int vb1) __attribute__((always_inline)) {
        const int kb = kt * C::kBC;
        // wave-uniform: does the wave see any key of the sub-tile / must it mask some
        if (!CAUSAL || kb <= q0e + 31) {
            subtile(kt, 0, kb1, kb2, vb, vb1, (kb + 32 > Sk) || (CAUSAL && kb + 31 > q0e), sa, sb);
        } else {
            dma_k(kt + 2, kb2);
            if (NW == 8 || kt + 1 < n_kt) dma_v(kt + 1, vb1);
        }
        if (!CAUSAL || kb + 32 <= q0e + 31)
            subtile(kt, 1, kb1, kb2, vb, vb1, (kb + 64 > Sk) || (CAUSAL && kb + 63 > q0e), sb, sa);
        tile_barrier();
    };
    if constexpr (C::kMain) {
        // unrolled over the three buffers like the main loop (kt0 is a multiple of three)
        for (int kt = kt0; kt < n_kt; kt += 3) {  // n_kt is the same for every wave of the work-group
            tile(kt, 1, 2, 0, 1);
            if (kt + 1 < n_kt) tile(kt + 1, 2, 0, 1, 2);
            if (kt + 2 < n_kt) tile(kt + 2, 0, 1, 2, 0);
        }
    } else {
        // fewer waves stage more of each tile per wave and have no registers to spare for the
        // unrolled form: the buffer indices rotate at run time
        int kb1 = 1, kb2 = 2, kb0 = 0;
        for (int kt = kt0; kt < n_kt; ++kt) {
            tile(kt, kb1, kb2, kt & 1, (kt + 1) & 1);
            const int t = kb0; kb0 = kb1; kb1 = kb2; kb2 = t;
        }
    }
#undef ATTN_FENCE

    // Epilogue: O = O_acc / l, LSE = ln2 * (m + log2 l).
    const float lt = xhalf_sum(lsum);
    const float lr = xhalf_sum(hsum);  // sum of the rounded probabilities
    // (Narrow tensors, see above: directly.)  The accumulator holds 4 consecutive columns of one row per register group, so
    // a direct store writes 16 bytes to each of 32 rows per instruction, sixteen times per wave.
    // The rows go through LDS instead and leave whole, 16 bytes per lane and four (D = 128) or
    // eight rows per instruction: half as many stores, each over contiguous memory.  The wave's
    // staging space (32 rows in the K tile's layout) lies in the K buffers and the query staging
    // space, which nobody reads after the last tile barrier.
    constexpr int kWaveBytes = C::kKHalf * 2;
    char *const stg = smem + (w < 6 ? w * kWaveBytes
                                                  : (3 * C::kKTile + 3 * C::kVTile) * 2 + (w - 6) * kWaveBytes);
    auto at = [](int row, int chunk) { return L::at(row, chunk); };
    if (SPLIT) {
        // normalised fp32 partial result of this key range; a row that saw no key of the
        // range contributes O = 0 with LSE = -inf
        const float inv = lr > 0.f ? 1.0f / lr : 0.f;
        const int64_t row0 = ((int64_t)blockIdx.y * a.BH + bh) * S;
        {
            // through LDS like O below; an fp32 row is twice as long, so it goes in two halves
            constexpr int CPR = D / 8, RPI = 64 / CPR;
            const int lr_ = l / CPR, lc = l % CPR;
            // (columns past U are not written, the merge drops them: 8 heads of 4471 rows D = 32 causal 44 -> 37 us)
            constexpr int HB = D / 64;
#pragma unroll
            for (int hp = 0; hp < 2 && hp * HB < DB; ++hp) {
#pragma unroll
                for (int db = hp * HB; db < (hp + 1) * HB && db < DB; ++db)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        f32x4 ov;
#pragma unroll
                        for (int e = 0; e < 4; ++e) ov[e] = o[db][4 * g + e] * inv;
                        *(f32x4 *)(stg + at(r, (db % HB) * 8 + 2 * g + h)) = ov;
                    }
                asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
#pragma unroll
                for (int j = 0; j < 32 / RPI; ++j) {
                    const f32x4 v = *(const f32x4 *)(stg + at(RPI * j + lr_, lc));
                    const int row = q0 + RPI * j + lr_, col = hp * (D / 2) + lc * 4;
                    if (row < S && col < U) *(f32x4 *)(a.Opart + (row0 + row) * D + col) = v;
                }
                asm volatile("" ::: "memory");
            }
            if (q < S && h == 0) a.LSEpart[row0 + q] = lt > 0.f ? (m + fast_log2(lt)) * kLn2 : -INFINITY;
        }
        return;
    }
    const float inv = 1.0f / lr;
    if constexpr (kNarrow) {
        if (q >= S) return;
        elem *const Op = a.O + base + (int64_t)q * a.stride_s;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                if (32 * db + 8 * g + 4 * h < Dr)
                    *(elem4 *)(Op + 32 * db + 8 * g + 4 * h) = pack4(o[db][4 * g] * inv, o[db][4 * g + 1] * inv,
                                                                     o[db][4 * g + 2] * inv, o[db][4 * g + 3] * inv);
        if (h == 0) a.LSE[(int64_t)bh * S + q] = (m + fast_log2(lt)) * kLn2;
    } else {
        constexpr int CPR = D / 8, RPI = 64 / CPR;  // chunks per row; rows per store instruction
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *(elem4 *)(stg + at(r, 4 * db + g) + 8 * h) =
                    pack4(o[db][4 * g] * inv, o[db][4 * g + 1] * inv, o[db][4 * g + 2] * inv, o[db][4 * g + 3] * inv);
        asm volatile("" ::: "memory");  // a wave's LDS accesses execute in order
        const int lr = l / CPR, lc = l % CPR;
#pragma unroll
        for (int j = 0; j < 32 / RPI; ++j) {
            const u32x4 v = *(const u32x4 *)(stg + at(RPI * j + lr, lc));
            const int row = q0 + RPI * j + lr;
            if (row < S && lc * 8 < Dr) *(u32x4 *)(a.O + base + (int64_t)row * a.stride_s + lc * 8) = v;
        }
        if (q < S && h == 0) a.LSE[(int64_t)bh * S + q] = (m + fast_log2(lt)) * kLn2;
    }
}

// Combine the per-split partial results: LSE = log sum_z exp(LSE_z), O = sum_z exp(LSE_z - LSE) O_z.
// A thread owns 4 consecutive d of one row and every ZG-th split, four splits per step with their
// loads issued together (a thread that walks all splits one load after the other spends a memory
// latency per split: 21 us for 32 splits of 32 rows), as a running (max, sum, weighted O) triple;
// the ZG triples of a row are then combined through LDS.  The order of the sums is a function of
// the shape only.  HBM-bound and small.
template <int D, int ZG>
__global__ void __launch_bounds__(256) attn_fwd_merge_kernel(const FwdArgs a)
{
    constexpr int TPR = D / 4;               // threads per row and split group
    constexpr int RPB = 256 / (TPR * ZG);    // rows per work-group
    static_assert(RPB >= 1, "a row's threads fit the work-group");
    const int64_t rows = (int64_t)a.BH * a.S;
    const int t = threadIdx.x;
    const int d0 = (t % TPR) * 4, zg = (t / TPR) % ZG;
    const int64_t row_raw = (int64_t)blockIdx.x * RPB + t / (TPR * ZG);
    const bool live = row_raw < rows;
    const int64_t row = live ? row_raw : rows - 1;  // clamped: every thread reaches the barrier
    const int nsplit = a.nsplit;
    float m = -INFINITY, den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int z0 = zg; z0 < nsplit; z0 += 4 * ZG) {
        float lz[4];
        f32x4 oz[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int z = z0 + k * ZG;
            const int64_t at = (int64_t)(z < nsplit ? z : z0) * rows + row;
            lz[k] = a.LSEpart[at];
            oz[k] = *(const f32x4 *)(a.Opart + at * D + d0);
            if (z >= nsplit) lz[k] = -INFINITY;
        }
        const float mk = fmaxf(fmaxf(m, fmaxf(lz[0], lz[1])), fmaxf(lz[2], lz[3]));
        if (mk > -INFINITY) {  // (an empty split has LSE = -inf and weight 0)
            const float sc = expf(m - mk);
            den *= sc;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] *= sc;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float wz = expf(lz[k] - mk);
                den += wz;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += wz * oz[k][e];
            }
            m = mk;
        }
    }
    if constexpr (ZG > 1) {
        __shared__ float red[256 * 6];
        red[t] = m;
        red[256 + t] = den;
#pragma unroll
        for (int e = 0; e < 4; ++e) red[(2 + e) * 256 + t] = acc[e];
        __syncthreads();
        if (zg != 0) return;
        float mm = m;
#pragma unroll
        for (int g = 1; g < ZG; ++g) mm = fmaxf(mm, red[t + g * TPR]);
        const float s0 = mm > -INFINITY ? expf(m - mm) : 0.f;
        den *= s0;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] *= s0;
#pragma unroll
        for (int g = 1; g < ZG; ++g) {
            const int u = t + g * TPR;
            const float sg = mm > -INFINITY ? expf(red[u] - mm) : 0.f;
            den += sg * red[256 + u];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += sg * red[(2 + e) * 256 + u];
        }
        m = mm;
    }
    if (!live) return;
    const float inv = 1.0f / den;
    const int bh = (int)(row / a.S), q = (int)(row % a.S);
    elem *Op = a.O + (int64_t)(bh / a.H) * a.stride_b + (int64_t)(bh % a.H) * a.stride_h +
               a.row_offset(q) + d0;
    if (d0 < a.Dr) *(elem4 *)Op = pack4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
    if (d0 == 0) a.LSE[row] = m + logf(den);
}

template <int D, int ZG>
static int launch_fwd_merge_zg(const FwdArgs &a, hipStream_t st)
{
    const int64_t rows = (int64_t)a.BH * a.S;
    constexpr int RPB = 256 / ((D / 4) * ZG);
    hipLaunchKernelGGL((attn_fwd_merge_kernel<D, ZG>), dim3((unsigned)((rows + RPB - 1) / RPB)),
                       dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Up to four splits: one thread per (row, 4 d) takes them all in one step.  More: a row's splits
// are spread over as many thread groups as fit the work-group with it.
template <int D>
static int launch_fwd_merge(const FwdArgs &a, hipStream_t st)
{
    if (a.nsplit <= 4) return launch_fwd_merge_zg<D, 1>(a, st);
    return launch_fwd_merge_zg<D, (D > 128 ? 4 : 8)>(a, st);
}

#ifndef ATTN_F16
// Three work-groups of four waves fit a unit.  Unsplit, where all of them are resident, from 2000 rows on two are
// quicker, as heavy ones then do not meet three to a unit (0.97 of the time on average, D <= 32 0.98, never more than 1.09;
// over 70 problems.  With more work-groups three, 0.83 .. 1.01 of the time on average in every class of 270).  Split, under a mask, the work-groups of a split that lies behind their rows end
// at once, and the heavy ones among the others are better spread: two on a unit, as with the larger tiles in LDS before, with
// up to 612 of the others in two or three splits and 500 in more (8 heads of 4471 rows, 3 splits, 54 | 47 us, D = 32 43 | 37);
// three with more of them (22 of 2682, 2 splits, D = 32 37 | 43; on average 1.05 with 3 or 4 splits, 1.12 with 2).  Over 408
// problems; with few of either the same.
bool fwd_takes_two(int BH, int S, int Sk, int nsplit, int kps)
{
    const int64_t wgs = (int64_t)BH * ((S + 127) / 128);
    if (nsplit <= 1) return S >= 2000 && wgs > 512 && wgs <= 768;
    const float splits_seen = ((Sk + 63) / 64 - S / 128.0f) * 64 / kps + 0.5f;  // of a query tile, on average
    return wgs * std::min((float)nsplit, splits_seen) <= (nsplit > 3 ? 500 : 612);
}
#endif

template <int D, int U, int NW, bool CAUSAL, bool SPLIT, bool MAIN>
static int launch_fwd_kernel(const FwdArgs &a, hipStream_t st)
{
    using C = FwdCfg<D, NW, MAIN>;
    constexpr bool kTwo = D == 64 && NW == 4 && CAUSAL && MAIN;  // the launches that may ask for more
    constexpr int kMost = kTwo ? std::max(C::kLdsBytes, kLdsTwoPerUnit) : C::kLdsBytes;
    const int lds = kTwo && fwd_takes_two(a.BH, a.S, a.Sk, a.nsplit, a.kps) ? kMost : C::kLdsBytes;
    // (one limit for every launch of the kernel: another thread may be between its own call here and its launch)
    if (hipFuncSetAttribute((const void *)attn_fwd_kernel<D, U, NW, CAUSAL, SPLIT, MAIN>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, kMost) != hipSuccess)
        return -1;
    hipLaunchKernelGGL((attn_fwd_kernel<D, U, NW, CAUSAL, SPLIT, MAIN>),
                       dim3(a.nqt * a.BH, SPLIT ? a.nsplit : 1), dim3(C::kThreads),
                       lds, st, a);
    if (hipGetLastError() != hipSuccess) return -1;
    if (SPLIT) return launch_fwd_merge<D>(a, st);
    return 0;
}

template <int D, int U, int NW, bool MAIN>
static int launch_fwd_nw(const FwdArgs &a, bool causal, hipStream_t st)
{
    // (four waves at D = 64 are split in the form with the main loop only, see fwd_takes_main)
    if constexpr (MAIN || NW != 4 || D != 64)
        if (a.nsplit > 1)
            return causal ? launch_fwd_kernel<D, U, NW, true, true, MAIN>(a, st)
                          : launch_fwd_kernel<D, U, NW, false, true, MAIN>(a, st);
    return causal ? launch_fwd_kernel<D, U, NW, true, false, MAIN>(a, st)
                  : launch_fwd_kernel<D, U, NW, false, false, MAIN>(a, st);
}

#ifndef ATTN_F16
// Whether four waves at D = 64 take the form with the pipelined main loop: from four tiles on.  (It is entered from
// three whole tiles on, and its third V buffer and registers still let three work-groups share a compute unit.)  Over
// 150 problems of 64 .. 3300 rows, up to 4000 work-groups, time relative to the generic form: 0.79 .. 1.04 from 256 keys on,
// 0.94 on average (36 heads of 900 rows causal 19.6 -> 16.8 us, 275 of 349 rows on 1104 keys 39.4 -> 34.1), 0.96 .. 1.04 with
// 192 .. 255, 1.0 .. 1.05 with fewer (347 of 95 7.6 -> 8.0).  For narrow tensors without a mask from three tiles on in launches
// of at most two work-groups per unit: 64 of 195 rows D = 32 6.5 -> 6.1, 250 of 200 9.0 -> 8.8, the same with more.
bool fwd_takes_main(int wgs, int Sk, int nsplit, bool causal, bool narrow)
{
    return nsplit > 1 || Sk >= 256 || (narrow && !causal && Sk >= 192 && wgs <= 512);
}
#endif

// Waves per work-group: 8 (256 query rows) unless the sequence is too short to fill them.
// With D = 128 at least 4 (waves whose rows lie past the end compute and store nothing useful,
// but still take part in the staging): the one- and two-wave forms are only built for D = 64,
// and short problems at D = 128 go to the kernel of attn_fwd_wide.hip unless the rotary
// embedding is fused into the call.
// split_keys: the keys of a launch that may be split, else 0.
static int fwd_waves_for(int S, int D, int BH, bool causal, int split_keys)
{
    const int blocks32 = (S + 31) / 32;
    // D = 64 under a causal mask with fewer than four 256-row work-groups per compute unit:
    // 128-row work-groups (two or three fit a compute unit at D = 64) balance the unequal tiles
    // better.  Measured: B=8 H=8 S=1024 26.5 -> 24.3 us, B=16 H=16 S=512 29.5 -> 27.6 us; not
    // so at D = 128 (+4..33 % on mid-size shapes).  (Split launches; unsplit ones: fwd_waves_unsplit.)
    if (blocks32 >= 8 && D == 64 && causal && (int64_t)BH * ((S + 255) / 256) < 1024) return 4;
    if (blocks32 >= 8) return 8;
    // Five to seven blocks at D = 128, where a work-group fills a unit whatever its waves: two work-groups of
    // four waves per head stage K and V twice and half fill the second, one of eight has the pipelined main
    // loop.  Eight where the heads' pairs do not fit the units at once, or the split of long keys makes as many
    // of them; us, four -> eight: 140 heads of 150 rows on 998 keys 53 -> 33, 176 of 154 causal 18 -> 13, 224 of
    // 215 on 3497 causal 156 -> 102, 64 of 190 on 3243 causal 49 -> 40, 120 of 179 on 5326 D = 96 93 -> 75; with fewer
    // four waves are quicker (100 of 148 causal 10 | 13, 32 of 132 on 1776 23 | 25).  At D = 64, where two or
    // three of the smaller ones share a unit, eight take 1.1 times as long on average.
    if (D == 128 && blocks32 >= 5 && (BH > 128 || (int64_t)BH * split_keys >= 131072)) return 8;
    // Three 32-row blocks also take four waves; the fourth has no rows and only stages K and V.
    // Measured at B=128 H=6 S=65: 13.6 -> 10.4 us, S=96: 15.4 -> 12.5 us.  The three-wave
    // kernel needs 177 registers at D = 64 (two waves per SIMD, two work-groups per compute
    // unit) against 150 for four waves (three work-groups), but capping it at 168 registers
    // (with 48 bytes of spills) did not make it faster, so the shorter staging per wave counts
    // as well.  Four waves for two blocks change nothing.
    if (blocks32 >= 3 || D == 128) return 4;
    return blocks32;  // 1 or 2
}

#ifndef ATTN_F16
// ... of an unsplit launch at D = 64 from 225 rows on (split ones, and the plan that splits them: the rule above; the
// rule without a mask: see WaveRule).  us, four | eight: 32 heads of 1957 rows 41 | 39, 65 of 817 20 | 34, 454 of 388
// 40 | 47, 22 of 4747 163 | 157, 39 of 2809 99 | 97, but 159 of 700 32 | 34; D = 32: 1272 of 234 29 | 27, 80 of
// 3047 155 | 145, 134 of 583 20 | 23, 250 of 291 12 | 13.  Over 600 problems of 228 .. 6200 rows and 200 .. 5000
// work-groups of four it takes 1.000 of the time of the better of the two on average, none above 1.04 (1.01 above 32
// columns).  Causal, where work-groups are unequal and a round has no sharp end, four: 2473 of 282 94 | 174, 675 of 703
// 77 | 95, 72 of 3851 184 | 207; of 286 problems from 1024 work-groups of eight on (below, the rule above takes four as
// well) 0.77 of the time of eight on average and none above it, up to 32 columns 0.92 and up to 1.09 in two rounds that eight
// just fill (53 of 5231 165 | 151).
int fwd_waves_unsplit(int BH, int S, int Sk, bool causal, bool narrow)
{
    static const WaveRule rule = {{6.2f, 2.2f, {0.41f, 0.77f, 1.10f}, 3}, {6.2f, 2.6f, {0.71f, 1.39f}, 2}, 1792};
    return !causal && takes_eight_waves(rule, BH, S, Sk, narrow) ? 8 : 4;
}
#endif

template <int D, int U = D>
static int launch_fwd_d(FwdArgs a, bool causal, hipStream_t st)
{
    const int nw = D == 64 && a.nsplit <= 1 && a.S > 224 ? fwd_waves_unsplit(a.BH, a.S, a.Sk, causal, U < D)
                                                         : fwd_waves_for(a.S, D, a.BH, causal, a.nsplit > 1 ? a.Sk : 0);
    a.nqt = (a.S + nw * 32 - 1) / (nw * 32);
    if (nw == 8) return launch_fwd_nw<D, U, 8, true>(a, causal, st);
    if constexpr (D < 128) {
        if (nw == 4 && fwd_takes_main(a.BH * a.nqt, a.Sk, a.nsplit, causal, U < D)) return launch_fwd_nw<D, U, 4, true>(a, causal, st);
        if (nw == 2) return launch_fwd_nw<D, U, 2, false>(a, causal, st);
        if (nw == 1) return launch_fwd_nw<D, U, 1, false>(a, causal, st);
    }
    if (nw == 4) return launch_fwd_nw<D, U, 4, false>(a, causal, st);
    return -1;
}

// Which problems go to the kernel of attn_fwd_wide.hip (128-row work-groups, two K/V buffers, two
// work-groups per compute unit at D <= 128) instead of the one above: head dimensions above 128 and packed
// rows, whose positions only that kernel knows, and, measured, forward only, graph replay, same box:
//  - at most 32 query rows per head (decoding; one wave of four has rows, the problem is K/V
//    streaming): B=8 Hq=32 Hkv=8 Sk=8192 66.7 -> 49.7 us, B=16 H=16 Sk=4096 143 -> 103;
//  - D = 128 and at most 128 rows: S=96 causal 18.8 -> 14.3 us (the kernel above needs four waves
//    at D = 128 whatever the length); 128 rows on 1024 keys the same either way.
// Everything else is faster above: mid-size causal D = 64 launches by 3-5 % (B=8 H=8 S=1024 22.5
// against 23.6 us), large launches by 7-12 %.
static bool streams(int S, int D, bool packed) { return D > 128 || S <= 32 || packed || (D == 128 && S <= 128); }

#ifndef ATTN_F16  // functions of the shape only: defined once, by the bf16 build
// Split over the keys.  A launch of few work-groups lasts as long as its longest one; a split shortens
// that, but every split writes an fp32 partial result that the merge reads.  The launch's time is estimated
// for every number of splits and the best is taken if it is at least 3 % below the unsplit one (below it, where that is
// another kernel's).  SplitCost:
// us that a launch takes besides its tiles, that a further work-group on the same unit takes besides its
// own; a 64-key tile of a work-group alone on its compute unit, and its share of the unit when several are
// (no tile takes less than the shares of all of them); work-groups that fit a unit.
//   - Work-groups of equal length (no mask, or one query tile per head): as many rounds as they need.
//   - Causal, unsplit: the longest, the whole work spread evenly, or, heaviest first, two (three, ..) of the
//     length at one (two, ..) launches' worth of resident work-groups.
//   - Causal, split: the work-groups of a split that lies behind their rows end at once; the others (a query
//     tile has one per started share of its keys) are dispatched split by split, heaviest first.  Those
//     that are not resident at once, the lightest of the last split, start when earlier ones end: early
//     while there are ones that end at their diagonal in an earlier split, else after a whole one.
// The constants are a fit of this model to the forward's time at every number of splits of 1674 problems
// (1 .. 96 heads and packed rows, 33 .. 4096 rows, up to 32768 keys, both masks; 9 % rms): the splits it
// takes are 2.1 % above the best ones on average, against 8.5 % with at least one work-group per compute
// unit.  us, D = 128 causal: 12 heads of 3143 rows 75 unsplit, 57 with its 2 splits, 74 with 3; 8 heads of
// 2895 67, 52 with 3; 32 of 512 stay unsplit (19; 27 with 2).  D = 256 causal: 4 of 2524 69, 41 with 4; 12
// of 3430 unsplit 98 (133 with 2).  D = 64 without mask: 96 heads of 118 rows on 6729 keys 93, 40 with 4.
struct SplitCost { float fixed, start, tile, share; int per_cu; };

// unsplit: us of the launch without a split where it is another kernel's, else 0.
static int fwd_splits(const SplitCost &c, int64_t wgs, int tiles, int S, float part_mb, bool equal, int most, float unsplit)
{
    const int64_t resident = 256 * c.per_cu;
    auto tile_us = [&](int64_t on_a_unit) { return std::max(c.tile, std::min<int64_t>(on_a_unit, c.per_cu) * c.share); };
    const float diagonal = S / 64.0f;  // tiles over which the rows of a head end
    const float average = tiles - diagonal / 2, spread = wgs * average * std::max(c.tile / c.per_cu, c.share) / 256;
    auto unsplit_causal = [&]() {
        const float on_a_unit = std::min(std::max(wgs / 256.0f, 1.0f), (float)c.per_cu);
        float t = std::max(c.fixed + tiles * std::max(c.tile, on_a_unit * c.share), spread);
        for (int64_t j = resident, rounds = 2; j < wgs; j += resident, ++rounds)
            t = std::max(t, rounds * (c.fixed + tile_us(c.per_cu) * (tiles - diagonal * j / wgs)));
        return t;
    };
    auto estimate = [&](int n) {
        const int per = (tiles + n - 1) / n;
        n = (tiles + per - 1) / per;
        // (the merge of more than four splits: a thread group per row and eight splits, see launch_fwd_merge)
        const float merge = n == 1 ? 0.0f : n <= 4 ? 2.7f + 0.46f * part_mb * n : 3.5f + (0.43f * n + 1.1f) * part_mb;
        if (equal) {
            const int64_t rounds = (n * wgs + resident - 1) / resident, last = n * wgs - (rounds - 1) * resident;
            return (rounds - 1) * (c.start + per * tile_us(c.per_cu)) + c.fixed + per * tile_us((last + 255) / 256) + merge;
        }
        if (n == 1) return unsplit_causal();
        const float busy = wgs * std::min((float)n, average / per + 0.5f), late = busy - resident;
        const float tile = tile_us((int64_t)std::ceil(busy / 256));
        float t = c.fixed + per * tile;
        if (late > 0) {
            const float ends = wgs * std::max(0.0f, 1 - per / diagonal), rest = late - ends;
            const int last = tiles - (n - 1) * per;
            const float in_last = wgs * std::min(1.0f, last / diagonal);
            if (rest <= 0) t *= 1 + 0.3f * late / ends;
            else if (rest > in_last) t *= 1 + std::ceil(late / resident);
            else t += c.start + tile * (diagonal >= last ? last * rest / in_last : last - diagonal * (1 - rest / in_last));
        }
        return std::max(t, spread + busy * c.start / 256) + merge;
    };
    int best = 1;
    // Causal rows beyond those of the fit, one work-group per unit: two splits whose heavy work-groups nearly fill
    // the chip run longer than estimated.  us, unsplit | two | three: 13 heads of 4335 rows D = 96 (221 work-groups)
    // 84 | 108 | 97, 9 of 6061 D = 128 (216) 142 | 172 | 143, 5 of 5535 D = 256 (220) 144 | 161 | 147.  Over 340
    // problems of 120 .. 512 work-groups at D = 80 .. 128 the plan without two splits here takes 0.977 of the time
    // that it takes with them, over 200 above D = 128 0.989, none more than 1.12.  With fewer two splits pay, 5 of
    // 9329 D = 96 (185) 172 | 117, and with more, where the unsplit launch takes a second round: 8 of 8394 D = 128
    // (264) 201 | 175; three pay for longer, 4 of 13775 D = 128 (216) 309 | 304 | 259.
    const bool no_two = !equal && S > 4096 && c.per_cu == 1 && wgs > 188 && wgs <= 256;
    float least = unsplit > 0 ? unsplit : 0.97f * estimate(1);
    for (int n = no_two ? 3 : 2; n <= most && 4 * n <= tiles && n * wgs <= 1024; ++n) {
        const float t = estimate(n);
        if (t < least) { least = t; best = n; }
    }
    return best;
}

// The forward.  Decoding (at most 32 rows per head) runs in the streaming kernel and is bound by
// memory, not by its longest work-group: at least one work-group per compute unit (256 with long key
// ranges beat 512 or 1024 shorter ones there, 0.060 ms against 0.071 and 0.086 on the decode shape),
// every split at least four tiles.  `rule`: the plan, or the smaller workspaces that are accepted: that
// rule for any number of rows, the estimate that dQ uses, or the plan for work-groups of four waves.
int fwd_split_plan(int BH, int S, int Sk, int D, bool causal, bool packed, int *kps, int most, SplitRule rule)
{
    const bool wide = streams(S, D, packed);
    // (rows per work-group: 128 in the streaming kernel)
    // (the smaller workspaces of heads of five to seven blocks at D = 128: those of four waves)
    const int nw = D > 128 || (rule != SplitRule::plan && D == 128 && S <= 224) ? 4 : fwd_waves_for(S, D, BH, causal, Sk);
    const int tile_rows = wide ? 128 : nw * 32;
    const int64_t wgs = (int64_t)BH * ((S + tile_rows - 1) / tile_rows);
    const int64_t target = 256;
    const int tiles = (Sk + 63) / 64;
    int nsplit = 1;
    if (S > 32 && (rule == SplitRule::plan || rule == SplitRule::four_waves)) {
        const SplitCost cost = D > 128           ? SplitCost{8.2f, 9.8f, 1.70f, 1.70f, 1}
                               : D > 64          ? (wide ? SplitCost{4.6f, 1.7f, 1.25f, 1.06f, 2}
                                                         : SplitCost{6.0f, 1.0f, 1.45f, 1.27f, 1})
                               : nw == 8         ? SplitCost{6.0f, 0.9f, 0.97f, 0.97f, 2}
                               : nw == 4 || wide ? SplitCost{4.9f, 1.0f, 0.73f, 0.58f, 2}
                                                 : SplitCost{4.1f, 0.2f, 0.84f, 0.56f, 3};
        // D = 64 without a mask from 225 rows on: the split launch has eight waves, the unsplit one mostly four (see
        // fwd_waves_unsplit) and is the quicker one for longer.  us, split as if it had eight too | unsplit: 20 heads of
        // 1119 rows 24 | 17, 21 of 1353 28 | 19, 34 of 572 on 1393 keys 23 | 16; split still: 5 of 5391 on 8474 84 | 95, 43 of
        // 706 on 3476 42 | 48.  Of 381 problems that were split 230 still are; 1.004 of the time of the better of the two
        // on average (1.09 before).  (The costs are a few per cent above the average measured, so that a split that
        // pays stays: over 260 other problems whose plan changed 0.84 of the time before, none above 1.013.)
        // Where the unsplit launch has eight waves as well, its estimate by rounds is taken for long keys and one round
        // of four-wave work-groups only: 40 problems that it splits take 0.86 .. 0.99 of the unsplit time (17 heads of
        // 2630 on 7291 133 | 126, 16 of 2710 on 6866 D = 32 92 | 80).  With more rounds it splits what is quicker
        // unsplit (16 heads of 6479 on 12904 D = 32 305 | 289), with fewer keys the two are alike.
        float unsplit = 0.0f;
        if (D == 64 && !causal && !wide && S > 224) {
            const bool eight = fwd_waves_unsplit(BH, S, Sk, false, false) == 8;
            if (!eight || (tiles > 64 && BH * ((S + 127) / 128) <= 512))
                unsplit = rounds_us(eight ? RoundCost{6.0f, 7.9f, {0.97f, 2.08f}, 2} : RoundCost{4.8f, 2.6f, {0.65f, 1.1f, 1.65f}, 3},
                                    (int64_t)BH * ((S + (eight ? 255 : 127)) / (eight ? 256 : 128)), tiles);
        }
        nsplit = fwd_splits(cost, wgs, tiles, S, (float)BH * S * D * 4e-6f, !causal || S <= tile_rows, std::min(most, 128), unsplit);
    } else if (S > 32 && rule == SplitRule::longest) {
        const LongestCost cost = D > 128 ? LongestCost{10.0f, 4.3f, 4.3f, 5.0f, 256}
                                 : D > 64 ? LongestCost{7.0f, 1.38f, 1.38f, 1.8f, 256}
                                 : nw == 8 ? LongestCost{7.0f, 0.94f, 0.94f, 1.17f, 256}
                                           : LongestCost{7.0f, 0.67f, 0.67f, 0.69f, 512};
        nsplit = longest_split_plan(cost, wgs, tiles, tiles - S / 128.0f, (size_t)BH * S * D * 4, causal, 128);
    } else if (wgs < target && tiles >= 8) {
        nsplit = (int)((target + wgs - 1) / wgs);
        if (nsplit > tiles / 4) nsplit = tiles / 4;
        if (nsplit > 128) nsplit = 128;
    }
    // Two work-groups of the streaming kernel fit a compute unit: aim at two per unit as far as that
    // leaves every split 8 tiles or more
    // (B=8 Hkv=8 Sk=8192: 8 splits, 55.0 -> 49.5 us; B=16 H=16 Sk=4096: 2 splits, 111 -> 103 us;
    // B=1 Hkv=8 Sk=32768: 64 splits of 8 tiles 28.2 us against 30.0 with 32 of 16; four work-groups
    // per unit are 4-5 % slower again).
    if (S <= 32 && D <= 128 && wgs < 512) {
        int n2 = (int)((512 + wgs - 1) / wgs);
        if (n2 > tiles / 8) n2 = tiles / 8;
        if (n2 > 128) n2 = 128;
        if (n2 > nsplit) nsplit = n2;
    }
    const int tiles_per = (tiles + nsplit - 1) / nsplit;
    nsplit = (tiles + tiles_per - 1) / tiles_per;  // no empty split
    if (kps) *kps = tiles_per * 64;
    return nsplit;
}
#endif

int launch_fwd(const FwdArgs &a, int D, bool causal, hipStream_t st)
{
    if (streams(a.S, D, a.pack_sq != 0)) {
        if (launch_fwd_wide(a, D, causal, st)) return -1;
        if (a.nsplit <= 1) return 0;
        return D == 256 ? launch_fwd_merge<256>(a, st)
             : D == 128 ? launch_fwd_merge<128>(a, st) : launch_fwd_merge<64>(a, st);
    }
    constexpr int U128 = narrow_columns(128), U64 = narrow_columns(64);
    if (D == 128) return a.Dr <= U128 ? launch_fwd_d<128, U128>(a, causal, st) : launch_fwd_d<128>(a, causal, st);
    return a.Dr <= U64 ? launch_fwd_d<64, U64>(a, causal, st) : launch_fwd_d<64>(a, causal, st);
}

}  // namespace attn
