// Host-side kernel argument blocks and launch entry points (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace attn {

// The library is built twice from the same kernel sources: once with bf16 elements (the
// default) and once with IEEE fp16 (-DATTN_F16).  `elem` is the element type of the
// translation unit; the argument blocks are templates so that both builds can live in one
// library (kernels and launchers are distinguished by their argument type).
#ifdef ATTN_F16
typedef _Float16 elem;
#else
typedef __bf16 elem;
#endif

// One small block of arguments per kernel, passed by value: no per-tensor stride lists
// (the paper's debugging table records a crash from too many explicit stride arguments).
// Q, O, dO, dQ have H heads, S rows and the strides stride_*; K, V, dK, dV have H / group
// heads, Sk rows and the strides kv_stride_* (grouped-query attention; group == 1 is
// multi-head attention; Sk == S is the square problem).  With a causal mask query row i sees
// keys 0 .. i + Sk - S (aligned to the bottom-right corner).
template <typename E>
struct FwdArgsT {
    const E *Q, *K, *V;
    E *O;
    float *LSE;
    int64_t stride_b, stride_h, stride_s;
    int64_t kv_stride_b, kv_stride_h, kv_stride_s;
    int S, H, BH;
    int Sk;             // key/value rows
    int Dr;             // head dimension of the tensors (a multiple of 8); the kernels run at
                        // D = 64, 128 or 256 and treat columns Dr..D-1 as zeros
    int group;          // query heads per K/V head
    int pack_sq;        // 0, or: the S rows of a head are G query heads x pack_sq positions of one
                        // K/V head (row r is position r % pack_sq of S_q = pack_sq new rows); only
                        // the mask needs to know
    int64_t pack_stride_g;  // packed rows that are NOT at one distance (e.g. [B,S,H,D] tensors): row r lies
                        // (r / pack_sq) * pack_stride_g + (r % pack_sq) * stride_s past the head; 0: r * stride_s
    int nqt;            // query tiles per head (set by the launcher)
    float scale_log2e;  // scale * log2(e): the softmax runs on exp2
    // Split over the keys (small problems that would leave most of the chip idle): split z
    // (grid y) covers keys [z*kps, (z+1)*kps) and writes a normalised fp32 partial O and its
    // LSE; attn_fwd_merge_kernel combines them.  nsplit == 1: O and LSE are written directly.
    int nsplit, kps;    // kps is a multiple of the 64-key tile
    float *Opart;       // [nsplit][B*H][S][D]
    float *LSEpart;     // [nsplit][B*H][S]
    // Rotary embedding fused into the Q load (NULL tables: none).  Query row i is rotated by the
    // table row i * rope_row_step + rope_pos0 (step 1; step 0 when the rows of a head are the query
    // heads of one decoding position, which all sit at position rope_pos0) ("rotate-half" pairing of column d with d + D/2; tables fp32
    // [positions][D/2]); Qrot, if not NULL, receives the rotated rows (same strides as Q).
    const float *rope_cos, *rope_sin;
    E *Qrot;
    int rope_pos0, rope_row_step;
    // element offset of query row r from its head's first row (Q, O, Qrot share the strides)
    __host__ __device__ int64_t row_offset(int r) const
    {
        return pack_stride_g ? (int64_t)(r / pack_sq) * pack_stride_g + (int64_t)(r % pack_sq) * stride_s
                             : (int64_t)r * stride_s;
    }
};

template <typename E>
struct BwdArgsT {
    const E *Q, *K, *V, *O, *dO;
    const float *LSE;
    float *delta;       // workspace [B*H][2][S]: -delta, then LSE * log2(e)
    E *dQ, *dK, *dV;
    int64_t stride_b, stride_h, stride_s;
    int64_t kv_stride_b, kv_stride_h, kv_stride_s;
    int S, H, BH;
    int Sk;             // key/value rows
    int Dr;             // head dimension of the tensors; columns Dr..D-1 are zeros (see FwdArgsT)
    int group;          // query heads per K/V head
    int ntile;          // tiles per head of the launched kernel (set by the launcher)
    int stats_in_dq;    // the dQ kernel forms the row statistics itself and stores them to
                        // `delta` for the dK/dV kernel (set by the launcher)
    float scale, scale_log2e;
    // dQ kernel split over the keys (few query tiles against many keys would leave most of the
    // chip idle): split z (grid y) covers keys [z*dq_kps, (z+1)*dq_kps) and writes an unscaled
    // fp32 partial dQ; attn_bwd_dq_merge_kernel adds the splits, scales and rounds.
    // dq_nsplit == 1: dQ is written directly.
    int dq_nsplit, dq_kps;   // dq_kps is a multiple of the 64-key tile
    float *dQpart;           // [dq_nsplit][B*H][S][D]
    // dK/dV kernel split over the query slots (see dkdv_split_plan): a key block's slots are cut
    // into chunks of dkdv_chunk, dkdv_items chunks per K/V head in all; a block of several chunks
    // writes unscaled fp32 partial results, item by item, which attn_bwd_dkdv_merge_kernel adds.
    // dkdv_chunk == 0: not split.
    int dkdv_chunk, dkdv_items;
    float *dKVpart;          // [B*Hkv][dkdv_items][dV, dK][keys of a block][D]
    // dS kept from the dK/dV kernel for dQ (see ds_row_blocks): K/V heads that the region holds
    // at a time (0: not kept), and the K/V heads bkv0 .. bkv0 + nkv - 1 of the launch
    E *dS;
    int ds_heads, bkv0, nkv;
    // dK/dV and dQ in one launch (see pair_plan), if `pair`: the work-groups of dK/dV, which come first,
    // and the query tiles per head
    int pair, pair_dkdv, pair_dq;
    // Rotary embedding: Q holds ROTATED rows; dQ is rotated back (by the transpose of the
    // rotation) before it is stored, so that it is the gradient of the unrotated rows.  NULL
    // tables: none.
    const float *rope_cos, *rope_sin;
    int rope_pos0;
};

typedef FwdArgsT<elem> FwdArgs;
typedef BwdArgsT<elem> BwdArgs;

// Each returns 0 on success, -1 if the HIP runtime reported a launch error.  One overload per
// element type; each is defined by the build of the kernel sources for that type.
int launch_fwd(const FwdArgsT<__bf16> &a, int D, bool causal, hipStream_t st);
int launch_fwd(const FwdArgsT<_Float16> &a, int D, bool causal, hipStream_t st);
// The forward that streams both K and V by direct transfers (attn_fwd_wide.hip; D = 64, 128 or
// 256; called by launch_fwd, which also launches the merge of a split).
int launch_fwd_wide(const FwdArgsT<__bf16> &a, int D, bool causal, hipStream_t st);
int launch_fwd_wide(const FwdArgsT<_Float16> &a, int D, bool causal, hipStream_t st);
// Number of key splits the forward would use for this problem (1: none; at most `most`), and the keys per
// split; packed: rows packed as pack_sq says.  A pure host function of the shape.  SplitRule: the plan, and
// three rules whose smaller workspaces are accepted as well (see attn_fwd.hip).
enum class SplitRule { plan, longest, one_per_unit, four_waves };
int fwd_split_plan(int BH, int S, int Sk, int D, bool causal, bool packed, int *kps, int most = 128,
                   SplitRule rule = SplitRule::plan);
// Number of splits over `tiles` key tiles (`average` over the query rows) with which a launch of `wgs`
// work-groups ends soonest (1: none); part_bytes: the partial results of one split.  Times in us: what a
// work-group costs besides its tiles, a tile with the compute unit to itself (unsplit, and in the split
// kernel), a tile on a full chip; and the work-groups resident at once.  S rows in unsplit_wgs work-groups:
// see attn_bwd.hip (0: not counted).
struct LongestCost { float fixed, alone, alone_split, full; int resident; };
int longest_split_plan(const LongestCost &c, int64_t wgs, int tiles, float average, size_t part_bytes, bool causal,
                       int most, int S = 0, int64_t unsplit_wgs = 0);
// Four or eight waves (128 or 256 rows) per work-group at D = 64 without a mask, where all work-groups are equal.  Of four
// waves three work-groups share a compute unit, 768 are resident, of eight two: a launch that just passes its last round
// pays for a whole one.  RoundCost: us of a launch besides its rounds, of a further round besides its tiles, and of a
// 64-key tile with one, two, three work-groups on a unit.
//  - Above 32 columns four, except where eight find a unit each and twice as many of four do not, or (from `keys` on)
//    where those of eight are resident at once and those of four are not.
//  - Up to 32 columns two of eight waves fill a unit as well as three of four, and it is the rounds that decide: the lesser of the
//    two estimates.
struct RoundCost { float fixed, round, tile[3]; int per_cu; };
struct WaveRule { RoundCost four, eight; int keys; };
inline float rounds_us(const RoundCost &c, int64_t wgs, int tiles)
{
    const int64_t resident = 256 * c.per_cu, before = (wgs - 1) / resident, last = wgs - before * resident;
    return c.fixed + before * (c.round + tiles * c.tile[c.per_cu - 1]) + tiles * c.tile[(last + 255) / 256 - 1];
}
inline bool takes_eight_waves(const WaveRule &c, int BH, int S, int Sk, bool narrow)
{
    const int64_t w8 = (int64_t)BH * ((S + 255) / 256), w4 = (int64_t)BH * ((S + 127) / 128);
    if (narrow) return rounds_us(c.eight, w8, (Sk + 63) / 64) < rounds_us(c.four, w4, (Sk + 63) / 64);
    return w4 > 256 && (w8 <= 256 || (w4 > 768 && w8 <= 512 && Sk >= c.keys));
}
// Waves per work-group of the unsplit forward at D = 64 from 225 rows on, and of the unsplit dQ kernel at D = 64 and 128
// (narrow: tensors of at most narrow_columns(D)); pure host functions of the shape.
int fwd_waves_unsplit(int BH, int S, int Sk, bool causal, bool narrow);
int dq_waves(int BH, int S, int Sk, int D, bool causal, bool narrow);
// Whether the forward of `wgs` work-groups of four waves at D = 64 has the pipelined main loop; likewise.
bool fwd_takes_main(int wgs, int Sk, int nsplit, bool causal, bool narrow);
// Blocks of 32 rows per work-group of dQ from the stored dS (tensors of Dr columns); a pure host function of the shape.
int dq_ds_blocks(int heads, int S, int Dr, bool causal);
// LDS with which two work-groups share a compute unit (160 KB) and not three, for launches that are quicker that way.
constexpr int kLdsTwoPerUnit = 54784;
// Whether the causal forward of four waves at D = 64 is one (BH heads, nsplit splits of kps keys); a pure host function
// of the shape.
bool fwd_takes_two(int BH, int S, int Sk, int nsplit, int kps);
// Whether the unsplit dQ launch of `wgs` work-groups of nw waves at D = 64 is one; a pure host function of the shape.
bool dq_takes_two(int nw, int wgs);
// `stages`: bit 0 row statistics, bit 1 dK/dV, bit 2 dQ.  With bits 0 and 2 the dQ kernel
// forms the statistics (and runs first); bit 0 without bit 2 runs the separate kernel.
// Number of key splits the dQ kernel would use for this problem (1: none) and the keys per
// split; a pure host function of the shape.
// At most `most` splits.
int dq_split_plan(int BH, int S, int Sk, int D, bool causal, int *kps, int most = 16);
// Split of the dK/dV kernel over the query slots: returns the chunks (work-groups) per K/V head and
// the slots per chunk (0: not split, one work-group per key block), at most `most` chunks in all; a pure
// host function of the shape.
int dkdv_split_plan(int BHkv, int group, int S, int Sk, int D, bool causal, int *chunk, int64_t most = 512);
// Whether the unsplit dK/dV kernel for D = 128 is that of attn_bwd_solo.hip; a pure host function of the shape.
bool dkdv_takes_solo(int BHkv, int group, int S, int Sk, bool causal, bool stored);
// K/V heads whose dS the backward keeps at a time in `room` bytes (0: it recomputes it for dQ); a pure host
// function of the shape and the room.
int ds_plan(int BHkv, int group, int S, int Sk, int D, bool causal, size_t room);
// dK/dV and dQ in one launch, with both splits (dkdv_chunk == 0: neither is split) in `room` bytes: first the
// partial results of dQ, rounded up to 256 bytes, then those of dK/dV.
struct PairPlan { bool taken; int dq_nsplit, dq_kps, dkdv_chunk, items; };
// PairCost: us (see attn_bwd.hip).
struct PairCost { float fixed, slot, dq_fixed, dq_tile, merge, byte; };
PairPlan pair_plan(int BHkv, int group, int S, int Sk, int D, bool causal, size_t room);
// Columns that the products run over in the narrow instances of the kernels for D columns, for tensors of at
// most that many; the columns past them are zeros and cost their share of the matrix instructions, LDS
// reads and registers.  The products summed are the same.  us, all columns -> narrow, forward |
// backward: 140 heads of 1477 rows D = 80 causal 104 -> 90 | 289 -> 275, 68 of 2529 D = 96 208 -> 181 |
// 737 -> 637 (with dS kept in both); 240 of 1226 D = 32 causal 88 -> 61 | 227 -> 173.  (No further steps:
// at D = 64 an instance of 48 columns would leave the 32-column blocks of dQ, dK, dV and O as they are.)
constexpr int narrow_columns(int D) { return D > 64 ? D / 4 * 3 : D / 2; }
// Keys per work-group of the split dK/dV kernel, and the 32-row query slots (over all query heads of
// the group) that key block kt has to walk: all of them, or under a causal mask those from the
// block's diagonal on.
__host__ __device__ inline constexpr int dkdv_split_keys(int D) { return D > 128 ? 64 : 128; }
__host__ __device__ inline int dkdv_slots(int kt, int keys, int group, int S, int Sk, bool causal)
{
    const int n_slot = (S + 31) / 32, first = kt * keys - (Sk - S);
    const int t0 = causal && first > 0 ? first / 32 : 0;
    return n_slot > t0 ? group * (n_slot - t0) : 0;
}
// Stored dS: 2 KB blocks of 32 query rows (a slot) x 32 keys; per query head, for slot 0, 1, .. the row of its
// key blocks.  Under a causal mask (Sk >= S, coff = Sk - S) a row has only the blocks that hold a visible
// pair, one more than the row before; without one an odd number, so that the rows, which the dQ kernel's
// waves read side by side, start in different memory channels.  ds_row_len: blocks that slot t sees;
// ds_row_blocks: blocks before its row.
constexpr int kDsBlock = 1024;  // elements
__host__ __device__ inline int ds_row_len(int t, int Sk, int coff, bool causal)
{
    const int all = (Sk + 31) / 32, seen = t + (coff + 31) / 32 + 1;
    return causal && seen < all ? seen : all;
}
__host__ __device__ inline int64_t ds_row_blocks(int t, int Sk, int coff, bool causal)
{
    // (only the last slot's row can be cut at the last key)
    return causal ? (int64_t)t * ((coff + 31) / 32 + 1) + (int64_t)t * (t - 1) / 2 : (int64_t)t * ((Sk + 31) / 32 | 1);
}
__host__ __device__ inline int64_t ds_head_blocks(int S, int Sk, bool causal)
{
    const int last = (S + 31) / 32 - 1;
    return ds_row_blocks(last, Sk, Sk - S, causal) + ds_row_len(last, Sk, Sk - S, causal);
}
// The whole backward in one launch for heads of at most bwd_small_max_rows(D) query rows and keys
// (attn_bwd_small.hip; called by launch_bwd when all three stages are asked for).
int bwd_small_max_rows(int D);
bool bwd_is_small(int BHkv, int group, int S, int Sk, int D);  // whether a whole backward is that launch
int launch_bwd_small(const BwdArgsT<__bf16> &a, int D, bool causal, hipStream_t st);
int launch_bwd_small(const BwdArgsT<_Float16> &a, int D, bool causal, hipStream_t st);
// dK and dV of the K/V heads bkv0 .. bkv0 + nkv - 1 by work-groups of 256 keys (attn_bwd_solo.hip; kernels for D = 128),
// storing dS if `ds`.
int launch_bwd_dkdv_solo(const BwdArgsT<__bf16> &a, bool causal, bool ds, hipStream_t st);
int launch_bwd_dkdv_solo(const BwdArgsT<_Float16> &a, bool causal, bool ds, hipStream_t st);
int launch_bwd(const BwdArgsT<__bf16> &a, int D, bool causal, hipStream_t st, unsigned stages);
int launch_bwd(const BwdArgsT<_Float16> &a, int D, bool causal, hipStream_t st, unsigned stages);

}  // namespace attn
