// C ABI of the attention library: host-side validation and dispatch only.
#include "../../include/attn.h"
#include "attn_launch.hpp"

#include <algorithm>
#include <cmath>
#include <limits>
#include <mutex>

namespace {

constexpr size_t kWsAlign = 256;

int check_strides(int32_t S, int32_t D, int64_t sb, int64_t sh, int64_t ss)
{
    if (ss < D || sh < 1 || sb < 1) return ATTN_ERR_STRIDE;
    if (ss % 8 || sh % 8 || sb % 8) return ATTN_ERR_STRIDE;
    // One head's rows (plus the look-ahead tiles the kernels fetch past the end, which read
    // as zero) are addressed with 32-bit byte offsets.
    // (half the 32-bit range: an offset one resource length past a row must not wrap either)
    if (((int64_t)S + 512) * ss * 2 >= ((int64_t)1 << 31)) return ATTN_ERR_STRIDE;
    return ATTN_OK;
}

// Every entry point funnels into the rectangular, grouped-query form.
int check_params(const attn_rect_params_t *p)
{
    if (!p) return ATTN_ERR_NULL;
    if (p->B < 1 || p->Hq < 1 || p->Hkv < 1 || p->Sq < 1 || p->Sk < 1) return ATTN_ERR_SHAPE;
    if (p->Hq % p->Hkv != 0) return ATTN_ERR_SHAPE;
    if (p->D < 8 || p->D > 256 || p->D % 8 != 0) return ATTN_ERR_SHAPE;
    // the causal mask is aligned bottom-right: with fewer keys than rows some rows see none
    if (p->causal && p->Sk < p->Sq) return ATTN_ERR_SHAPE;
    // B*Hq*Sq and B*Hkv*Sk rows must be indexable with int32 (LSE / workspace offsets, grids).
    const int64_t lim = (int64_t)std::numeric_limits<int32_t>::max();
    if ((int64_t)p->B * p->Hq * p->Sq > lim || (int64_t)p->B * p->Hkv * p->Sk > lim)
        return ATTN_ERR_SHAPE;
    int rc = check_strides(p->Sq, p->D, p->q_stride_b, p->q_stride_h, p->q_stride_s);
    if (rc != ATTN_OK) return rc;
    rc = check_strides(p->Sk, p->D, p->kv_stride_b, p->kv_stride_h, p->kv_stride_s);
    if (rc != ATTN_OK) return rc;
    if (!std::isfinite(p->scale) || !(p->scale > 0.0f)) return ATTN_ERR_SCALE;
    return ATTN_OK;
}

attn_rect_params_t as_rect(const attn_gqa_params_t &p)
{
    attn_rect_params_t g;
    g.B = p.B; g.Hq = p.Hq; g.Hkv = p.Hkv; g.Sq = p.S; g.Sk = p.S; g.D = p.D;
    g.q_stride_b = p.q_stride_b; g.q_stride_h = p.q_stride_h; g.q_stride_s = p.q_stride_s;
    g.kv_stride_b = p.kv_stride_b; g.kv_stride_h = p.kv_stride_h; g.kv_stride_s = p.kv_stride_s;
    g.scale = p.scale; g.causal = p.causal;
    return g;
}

// Multi-head parameters as the grouped-query ones with one query head per K/V head.
attn_gqa_params_t as_gqa(const attn_params_t &p)
{
    attn_gqa_params_t g;
    g.B = p.B; g.Hq = p.H; g.Hkv = p.H; g.S = p.S; g.D = p.D;
    g.q_stride_b = g.kv_stride_b = p.stride_b;
    g.q_stride_h = g.kv_stride_h = p.stride_h;
    g.q_stride_s = g.kv_stride_s = p.stride_s;
    g.scale = p.scale; g.causal = p.causal;
    return g;
}

// The kernels exist for D = 64, 128 and 256; other head dimensions (multiples of 8) run in the
// next larger one with the missing columns read as zeros.
int kernel_d(int D) { return D <= 64 ? 64 : D <= 128 ? 128 : 256; }

size_t round_ws(size_t bytes) { return (bytes + kWsAlign - 1) / kWsAlign * kWsAlign; }

// The forward's view of a problem: (B*H) independent heads of S query rows each.
struct FwdView {
    int BH, H, S, group;
    bool packed;  // decoding: the rows of a head are the query heads of one K/V head
    int pack_sq;  // ... times this many new positions each (0: not packed, or one position)
    int64_t pack_stride_g;  // distance between the packed query heads when their rows are not at one distance
    int64_t stride_b, stride_h, stride_s;
    bool causal;
};

// Decoding (Sq == 1) with grouped-query heads: the G query heads that share a K/V head are
// G rows at a uniform distance (the head stride), so they are presented to the kernel as ONE
// head of G rows.  K and V are then streamed once per K/V head instead of once per query
// head.  A single row sees every key, so the mask drops out.  LSE [B,Hq,1] is the same
// memory as [B,Hkv,G].
// A few new positions per sequence (Sq = 2 .. 32, G x Sq <= 128 rows: one query tile, e.g. speculative decoding): with the rows of
// a query head contiguous to the next head's (q_stride_h == Sq * q_stride_s) the G x Sq rows of
// a K/V head are again rows at one uniform distance and are packed the same way; row r is
// position r % Sq, which the causal mask and the fused rotary embedding need to know.
FwdView fwd_view(const attn_rect_params_t &p, bool rope)
{
    (void)rope;  // the plan is the same with and without the fused rotary embedding
    FwdView v;
    v.pack_sq = 0; v.pack_stride_g = 0;
    const int G = p.Hq / p.Hkv;
    if (p.Sq == 1 && G > 1 &&
        check_strides(G, p.D, p.q_stride_b, G * p.q_stride_h, p.q_stride_h) == ATTN_OK) {
        v.BH = p.B * p.Hkv; v.H = p.Hkv; v.S = G; v.group = 1;
        v.stride_b = p.q_stride_b; v.stride_h = G * p.q_stride_h; v.stride_s = p.q_stride_h;
        v.causal = false; v.packed = true;
    } else if (p.Sq > 1 && p.Sq <= 32 && G > 1 &&
               G * p.Sq <= 128 &&  // one query tile of the streaming kernel
               // rows of a head contiguous to the next head's: one distance; otherwise (e.g. [B,S,H,D]
               // tensors) the kernels address a packed row by (head, position); not at D = 256, whose
               // query rows arrive by direct transfers of whole tiles
               (p.q_stride_h == (int64_t)p.Sq * p.q_stride_s || kernel_d(p.D) <= 128) &&
               check_strides(G * p.Sq, p.D, p.q_stride_b, G * p.q_stride_h, p.q_stride_s) == ATTN_OK) {
        v.BH = p.B * p.Hkv; v.H = p.Hkv; v.S = G * p.Sq; v.group = 1;
        v.stride_b = p.q_stride_b; v.stride_h = G * p.q_stride_h; v.stride_s = p.q_stride_s;
        v.causal = p.causal != 0; v.packed = true; v.pack_sq = p.Sq;
        if (p.q_stride_h != (int64_t)p.Sq * p.q_stride_s) v.pack_stride_g = p.q_stride_h;
    } else {
        v.BH = p.B * p.Hq; v.H = p.Hq; v.S = p.Sq; v.group = G;
        v.stride_b = p.q_stride_b; v.stride_h = p.q_stride_h; v.stride_s = p.q_stride_s;
        v.causal = p.causal != 0; v.packed = false;
    }
    return v;
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

}  // namespace

// E: element type of Q, K, V, O (__bf16 or _Float16)
// The fp32 partial results (O and LSE) of one split of the forward over the keys.
static size_t fwd_part_bytes(const attn_rect_params_t *p)
{
    return (size_t)p->B * p->Hq * p->Sq * (kernel_d(p->D) + 1) * sizeof(float);
}
// Workspace that the forward's split over the keys takes with this problem's mask (0: it does not split).
static size_t fwd_split_bytes(const attn_rect_params_t *p, bool rope, attn::SplitRule rule = attn::SplitRule::plan)
{
    const FwdView v = fwd_view(*p, rope);
    const int nsplit = attn::fwd_split_plan(v.BH, v.S, p->Sk, kernel_d(p->D), v.causal, v.pack_sq != 0, nullptr, 128, rule);
    return nsplit > 1 ? round_ws(nsplit * fwd_part_bytes(p)) : 0;
}

// What is asked of the caller: enough for the problem with and without a causal mask, so that a
// workspace sized with one serves the other.
static size_t fwd_workspace_bytes(const attn_rect_params_t *p, bool rope)
{
    if (check_params(p) != ATTN_OK) return 0;
    attn_rect_params_t masked = *p, unmasked = *p;
    masked.causal = p->Sk >= p->Sq;
    unmasked.causal = 0;
    return std::max(fwd_split_bytes(&masked, rope), fwd_split_bytes(&unmasked, rope));
}

// The backward's row statistics: two fp32 values per query row.
static size_t bwd_stats_bytes(const attn_rect_params_t *p)
{
    return round_ws(2 * (size_t)p->B * p->Hq * p->Sq * sizeof(float));
}

// The fp32 partial results of the dQ kernel's split over the keys and of the dK/dV kernel's split
// over the query slots (0: not split).  The two kernels run one after the other, each with its
// merge, so their partial results share one region behind the statistics.
static size_t dq_split_bytes(const attn_rect_params_t *p)  // of one split
{
    return (size_t)p->B * p->Hq * p->Sq * kernel_d(p->D) * sizeof(float);
}
static size_t dq_part_bytes(const attn_rect_params_t *p, bool causal)
{
    const int nsplit = attn::dq_split_plan(p->B * p->Hq, p->Sq, p->Sk, kernel_d(p->D), causal, nullptr);
    return nsplit > 1 ? round_ws(nsplit * dq_split_bytes(p)) : 0;
}
static size_t dkdv_chunk_bytes(const attn_rect_params_t *p)  // of one chunk
{
    return (size_t)2 * attn::dkdv_split_keys(kernel_d(p->D)) * kernel_d(p->D) * sizeof(float);
}
static size_t dkdv_part_bytes(const attn_rect_params_t *p, bool causal)
{
    int chunk = 0;
    const int items = attn::dkdv_split_plan(p->B * p->Hkv, p->Hq / p->Hkv, p->Sq, p->Sk, kernel_d(p->D), causal, &chunk);
    return chunk ? round_ws((size_t)p->B * p->Hkv * items * dkdv_chunk_bytes(p)) : 0;
}

// K/V heads whose dS is kept at a time in `room` bytes (see ds_plan), and the bytes for n heads.
static int ds_heads_in(const attn_rect_params_t *p, size_t room)
{
    return attn::ds_plan(p->B * p->Hkv, p->Hq / p->Hkv, p->Sq, p->Sk, kernel_d(p->D), p->causal != 0, room);
}
static size_t ds_bytes(const attn_rect_params_t *p, int n)
{
    return (size_t)n * (p->Hq / p->Hkv) * attn::ds_head_blocks(p->Sq, p->Sk, p->causal != 0) * (attn::kDsBlock * 2);
}

// dK/dV and dQ in one launch, in `room` bytes (see pair_plan), and the bytes of its partial results.
static attn::PairPlan pair_in(const attn_rect_params_t *p, size_t room)
{
    return attn::pair_plan(p->B * p->Hkv, p->Hq / p->Hkv, p->Sq, p->Sk, kernel_d(p->D), p->causal != 0, room);
}
static size_t pair_bytes(const attn_rect_params_t *p, const attn::PairPlan &plan)
{
    if (!plan.dkdv_chunk) return 0;
    return (kernel_d(p->D) > 128 ? 0 : round_ws(plan.dq_nsplit * dq_split_bytes(p))) +
           round_ws((size_t)p->B * p->Hkv * plan.items * dkdv_chunk_bytes(p));
}

// Rotary embedding fused into the call (both tables NULL: none).
struct Rope {
    const float *cos_table = nullptr, *sin_table = nullptr;
    void *Qrot = nullptr;  // forward only, optional
};

// The fused rotary embedding pairs column d with d + D/2 inside one lane's registers, which
// the kernels can do at their native head dimensions only; positions need Sk >= Sq.
static int check_rope(const attn_rect_params_t *p, const Rope &r)
{
    if (!r.cos_table || !r.sin_table) return ATTN_ERR_NULL;
    if ((p->D != 64 && p->D != 128) || p->Sk < p->Sq) return ATTN_ERR_SHAPE;
    if (!aligned(r.cos_table, 16) || !aligned(r.sin_table, 16) || !aligned(r.Qrot, 16))
        return ATTN_ERR_ALIGN;
    return ATTN_OK;
}

template <typename E>
static int fwd_impl(const void *Q, const void *K, const void *V, void *O, float *LSE,
                    void *workspace, size_t workspace_bytes,
                    const attn_rect_params_t *p, void *hip_stream, const Rope *rope = nullptr)
{
    if (!Q || !K || !V || !O || !LSE) return ATTN_ERR_NULL;
    int rc = check_params(p);
    if (rc != ATTN_OK) return rc;
    if (rope && (rc = check_rope(p, *rope)) != ATTN_OK) return rc;
    if (!aligned(Q, 16) || !aligned(K, 16) || !aligned(V, 16) || !aligned(O, 16) ||
        !aligned(LSE, 4))
        return ATTN_ERR_ALIGN;
    // No workspace at all: run unsplit.  A workspace that is there must be usable: it holds the plan's
    // partial results, or at least those that one of the other rules asks for; then the plan is the best
    // of those that fit.
    const FwdView v = fwd_view(*p, rope != nullptr);
    int kps = 0, nsplit = 1;
    if (workspace) {
        auto plan = [&](int most) {
            return attn::fwd_split_plan(v.BH, v.S, p->Sk, kernel_d(p->D), v.causal, v.pack_sq != 0, &kps, most);
        };
        if (!aligned(workspace, kWsAlign)) return ATTN_ERR_WORKSPACE;
        nsplit = plan(128);
        if (nsplit > 1 && workspace_bytes < round_ws(nsplit * fwd_part_bytes(p))) {
            if (workspace_bytes < std::min({fwd_split_bytes(p, rope != nullptr, attn::SplitRule::longest),
                                            fwd_split_bytes(p, rope != nullptr, attn::SplitRule::one_per_unit),
                                            fwd_split_bytes(p, rope != nullptr, attn::SplitRule::four_waves)}))
                return ATTN_ERR_WORKSPACE;
            nsplit = plan((int)(workspace_bytes / fwd_part_bytes(p)));
        }
    }
    attn::FwdArgsT<E> a;
    a.nsplit = nsplit; a.kps = kps;
    a.Opart = static_cast<float *>(workspace);
    a.LSEpart = a.Opart ? a.Opart + (size_t)nsplit * p->B * p->Hq * p->Sq * kernel_d(p->D) : nullptr;
    a.Q = static_cast<const E *>(Q);
    a.K = static_cast<const E *>(K);
    a.V = static_cast<const E *>(V);
    a.O = static_cast<E *>(O);
    a.LSE = LSE;
    a.stride_b = v.stride_b; a.stride_h = v.stride_h; a.stride_s = v.stride_s;
    a.kv_stride_b = p->kv_stride_b; a.kv_stride_h = p->kv_stride_h; a.kv_stride_s = p->kv_stride_s;
    a.S = v.S; a.Sk = p->Sk; a.H = v.H; a.BH = v.BH; a.group = v.group; a.pack_sq = v.pack_sq; a.pack_stride_g = v.pack_stride_g;
    a.Dr = p->D;
    a.nqt = 0;
    a.scale_log2e = p->scale * 1.4426950408889634f;
    a.rope_cos = rope ? rope->cos_table : nullptr;
    a.rope_sin = rope ? rope->sin_table : nullptr;
    a.Qrot = rope ? static_cast<E *>(rope->Qrot) : nullptr;
    a.rope_pos0 = p->Sk - p->Sq;
    a.rope_row_step = v.packed ? 0 : 1;  // packed decoding heads all sit at the last position
    return attn::launch_fwd(a, kernel_d(p->D), v.causal, static_cast<hipStream_t>(hip_stream)) == 0
               ? ATTN_OK : ATTN_ERR_LAUNCH;
}

// The kernels of a backward call: what a workspace has room for beyond the row statistics bounds the splits.  (A
// plan that is dropped where it does not fit whole costs, in the 8 MiB of the call without workspace, us: one head
// of 1024 rows on 4096 keys, D = 128, causal 112 against 55 with the splits that fit; 4 -> 1 heads of 2048,
// D = 64, causal 180 against 51.)  dQ with rotary tables is split only where it runs next to dK/dV.
struct BwdPlan {
    int dq_nsplit, dq_kps, dkdv_chunk, dkdv_items, ds_heads;
    size_t dkdv_bytes;
    attn::PairPlan pair;
};
static BwdPlan bwd_plan(const attn_rect_params_t *p, size_t workspace_bytes, bool rope, uint32_t stages)
{
    const size_t room = workspace_bytes - bwd_stats_bytes(p);
    BwdPlan r = {};
    r.dq_nsplit = attn::dq_split_plan(p->B * p->Hq, p->Sq, p->Sk, kernel_d(p->D), p->causal != 0, &r.dq_kps,
                                      rope ? 1 : (int)std::min<size_t>(16, room / dq_split_bytes(p)));
    r.dkdv_items = attn::dkdv_split_plan(p->B * p->Hkv, p->Hq / p->Hkv, p->Sq, p->Sk, kernel_d(p->D),
                                         p->causal != 0, &r.dkdv_chunk,
                                         (int64_t)std::min<size_t>(512, room / dkdv_chunk_bytes(p)));
    r.dkdv_bytes = r.dkdv_chunk ? round_ws((size_t)p->B * p->Hkv * r.dkdv_items * dkdv_chunk_bytes(p)) : 0;
    // (a workspace of the size that attn_bwd_rect_workspace_bytes asks for, or less, keeps the form without dS,
    // and with one kernel after the other)
    if (stages == 7u && workspace_bytes > attn_bwd_rect_workspace_bytes(p)) {
        r.ds_heads = ds_heads_in(p, room - r.dkdv_bytes);
        r.pair = pair_in(p, room);
    }
    return r;
}

template <typename E>
static int bwd_impl(const void *Q, const void *K, const void *V, const void *O, const void *dO,
                    const float *LSE, void *dQ, void *dK, void *dV,
                    void *workspace, size_t workspace_bytes,
                    const attn_rect_params_t *p, void *hip_stream, uint32_t stages,
                    const Rope *rope = nullptr)
{
    if (!Q || !K || !V || !O || !dO || !LSE || !dQ || !dK || !dV) return ATTN_ERR_NULL;
    int rc = check_params(p);
    if (rc != ATTN_OK) return rc;
    if (rope && (rc = check_rope(p, *rope)) != ATTN_OK) return rc;
    if (!aligned(Q, 16) || !aligned(K, 16) || !aligned(V, 16) || !aligned(O, 16) ||
        !aligned(dO, 16) || !aligned(dQ, 16) || !aligned(dK, 16) || !aligned(dV, 16) ||
        !aligned(LSE, 4))
        return ATTN_ERR_ALIGN;
    const size_t stats_bytes = bwd_stats_bytes(p);
    if (!workspace || !aligned(workspace, kWsAlign) || workspace_bytes < stats_bytes)
        return ATTN_ERR_WORKSPACE;
    if (stages == 0 || (stages & ~7u)) return ATTN_ERR_SHAPE;
    const BwdPlan plan = bwd_plan(p, workspace_bytes, rope != nullptr, stages);
    const attn::PairPlan &pair = plan.pair;
    attn::BwdArgsT<E> a;
    a.Q = static_cast<const E *>(Q);
    a.K = static_cast<const E *>(K);
    a.V = static_cast<const E *>(V);
    a.O = static_cast<const E *>(O);
    a.dO = static_cast<const E *>(dO);
    a.LSE = LSE;
    a.delta = static_cast<float *>(workspace);
    a.dq_nsplit = plan.dq_nsplit; a.dq_kps = plan.dq_kps;
    a.dQpart = reinterpret_cast<float *>(static_cast<char *>(workspace) + stats_bytes);
    a.dkdv_chunk = plan.dkdv_chunk; a.dkdv_items = plan.dkdv_items;
    a.dKVpart = a.dQpart;
    a.dS = reinterpret_cast<E *>(reinterpret_cast<char *>(a.dQpart) + plan.dkdv_bytes);
    a.ds_heads = plan.ds_heads; a.bkv0 = 0; a.nkv = p->B * p->Hkv;
    a.pair = pair.taken; a.pair_dkdv = a.pair_dq = 0;
    if (pair.taken) {
        a.dq_nsplit = pair.dq_nsplit; a.dq_kps = pair.dq_kps;
        a.dkdv_chunk = pair.dkdv_chunk; a.dkdv_items = pair.items;
        if (kernel_d(p->D) <= 128) a.dKVpart += round_ws(pair.dq_nsplit * dq_split_bytes(p)) / sizeof(float);
    }
    a.dQ = static_cast<E *>(dQ);
    a.dK = static_cast<E *>(dK);
    a.dV = static_cast<E *>(dV);
    a.stride_b = p->q_stride_b; a.stride_h = p->q_stride_h; a.stride_s = p->q_stride_s;
    a.kv_stride_b = p->kv_stride_b; a.kv_stride_h = p->kv_stride_h; a.kv_stride_s = p->kv_stride_s;
    a.S = p->Sq; a.Sk = p->Sk; a.H = p->Hq; a.BH = p->B * p->Hq; a.group = p->Hq / p->Hkv;
    a.Dr = p->D;
    a.ntile = 0;
    a.scale = p->scale;
    a.scale_log2e = p->scale * 1.4426950408889634f;
    a.rope_cos = rope ? rope->cos_table : nullptr;
    a.rope_sin = rope ? rope->sin_table : nullptr;
    a.rope_pos0 = p->Sk - p->Sq;
    return attn::launch_bwd(a, kernel_d(p->D), p->causal != 0, static_cast<hipStream_t>(hip_stream),
                            stages) == 0
               ? ATTN_OK : ATTN_ERR_LAUNCH;
}

extern "C" {

void attn_params_contiguous(attn_params_t *p, int32_t B, int32_t H, int32_t S, int32_t D,
                            float scale, int32_t causal)
{
    if (!p) return;
    p->B = B; p->H = H; p->S = S; p->D = D;
    p->stride_s = D;
    p->stride_h = (int64_t)S * D;
    p->stride_b = (int64_t)H * S * D;
    p->scale = scale;
    p->causal = causal;
}

void attn_gqa_params_contiguous(attn_gqa_params_t *p, int32_t B, int32_t Hq, int32_t Hkv,
                                int32_t S, int32_t D, float scale, int32_t causal)
{
    if (!p) return;
    p->B = B; p->Hq = Hq; p->Hkv = Hkv; p->S = S; p->D = D;
    p->q_stride_s = p->kv_stride_s = D;
    p->q_stride_h = p->kv_stride_h = (int64_t)S * D;
    p->q_stride_b = (int64_t)Hq * S * D;
    p->kv_stride_b = (int64_t)Hkv * S * D;
    p->scale = scale;
    p->causal = causal;
}

void attn_rect_params_contiguous(attn_rect_params_t *p, int32_t B, int32_t Hq, int32_t Hkv,
                                 int32_t Sq, int32_t Sk, int32_t D, float scale, int32_t causal)
{
    if (!p) return;
    p->B = B; p->Hq = Hq; p->Hkv = Hkv; p->Sq = Sq; p->Sk = Sk; p->D = D;
    p->q_stride_s = p->kv_stride_s = D;
    p->q_stride_h = (int64_t)Sq * D;
    p->kv_stride_h = (int64_t)Sk * D;
    p->q_stride_b = (int64_t)Hq * Sq * D;
    p->kv_stride_b = (int64_t)Hkv * Sk * D;
    p->scale = scale;
    p->causal = causal;
}

size_t attn_fwd_rect_workspace_bytes(const attn_rect_params_t *p) { return fwd_workspace_bytes(p, false); }

size_t attn_fwd_rope_workspace_bytes(const attn_rect_params_t *p) { return fwd_workspace_bytes(p, true); }

int attn_fwd_rope(const void *Q, const void *K_rot, const void *V, const float *cos_table,
                  const float *sin_table, void *O, float *LSE, void *Q_rot, void *workspace,
                  size_t workspace_bytes, const attn_rect_params_t *p, void *hip_stream)
{
    Rope r;
    r.cos_table = cos_table; r.sin_table = sin_table; r.Qrot = Q_rot;
    return fwd_impl<__bf16>(Q, K_rot, V, O, LSE, workspace, workspace_bytes, p, hip_stream, &r);
}

int attn_bwd_rope(const void *Q_rot, const void *K_rot, const void *V, const void *O,
                  const void *dO, const float *LSE, const float *cos_table, const float *sin_table,
                  void *dQ, void *dK_rot, void *dV, void *workspace, size_t workspace_bytes,
                  const attn_rect_params_t *p, void *hip_stream)
{
    Rope r;
    r.cos_table = cos_table; r.sin_table = sin_table;
    return bwd_impl<__bf16>(Q_rot, K_rot, V, O, dO, LSE, dQ, dK_rot, dV, workspace, workspace_bytes, p,
                            hip_stream,
                            ATTN_BWD_STAGE_DELTA | ATTN_BWD_STAGE_DKDV | ATTN_BWD_STAGE_DQ, &r);
}

int attn_fwd_rect(const void *Q, const void *K, const void *V, void *O, float *LSE,
                  void *workspace, size_t workspace_bytes,
                  const attn_rect_params_t *p, void *hip_stream)
{
    return fwd_impl<__bf16>(Q, K, V, O, LSE, workspace, workspace_bytes, p, hip_stream);
}

int attn_fwd_rect_f16(const void *Q, const void *K, const void *V, void *O, float *LSE,
                      void *workspace, size_t workspace_bytes,
                      const attn_rect_params_t *p, void *hip_stream)
{
    return fwd_impl<_Float16>(Q, K, V, O, LSE, workspace, workspace_bytes, p, hip_stream);
}

int attn_fwd_gqa(const void *Q, const void *K, const void *V, void *O, float *LSE,
                 const attn_gqa_params_t *p, void *hip_stream)
{
    if (!p) return ATTN_ERR_NULL;
    const attn_rect_params_t g = as_rect(*p);
    return attn_fwd_rect(Q, K, V, O, LSE, nullptr, 0, &g, hip_stream);
}

int attn_fwd(const void *Q, const void *K, const void *V, void *O, float *LSE,
             const attn_params_t *p, void *hip_stream)
{
    if (!p) return ATTN_ERR_NULL;
    const attn_gqa_params_t g = as_gqa(*p);
    return attn_fwd_gqa(Q, K, V, O, LSE, &g, hip_stream);
}

size_t attn_bwd_rect_workspace_bytes(const attn_rect_params_t *p)
{
    if (check_params(p) != ATTN_OK) return 0;
    // (enough with and without a causal mask, as for the forward)
    size_t part = std::max(dq_part_bytes(p, false), dkdv_part_bytes(p, false));
    if (p->Sk >= p->Sq) part = std::max(part, std::max(dq_part_bytes(p, true), dkdv_part_bytes(p, true)));
    return bwd_stats_bytes(p) + part;
}

// dS grows with Sq * Sk: at most 1/64 of the card's 288 GB are asked for it.
size_t attn_bwd_rect_best_workspace_bytes(const attn_rect_params_t *p)
{
    if (check_params(p) != ATTN_OK) return 0;
    constexpr size_t kMost = ((size_t)288 << 30) / 64;
    const size_t plain = attn_bwd_rect_workspace_bytes(p);
    const attn::PairPlan pair = pair_in(p, kMost);
    if (pair.taken) return std::max(bwd_stats_bytes(p) + pair_bytes(p, pair), plain + kWsAlign);
    const int n = ds_heads_in(p, kMost);
    if (!n) return plain;  // (a workspace of that size would not be taken as one for dS)
    return std::max(bwd_stats_bytes(p) + dkdv_part_bytes(p, p->causal != 0) + ds_bytes(p, n), plain + kWsAlign);
}

int attn_bwd_rect_form(const attn_rect_params_t *p, size_t workspace_bytes)
{
    const int rc = check_params(p);
    if (rc != ATTN_OK) return rc;
    if (workspace_bytes < bwd_stats_bytes(p)) return ATTN_ERR_WORKSPACE;
    if (attn::bwd_is_small(p->B * p->Hkv, p->Hq / p->Hkv, p->Sq, p->Sk, kernel_d(p->D))) return ATTN_BWD_FORM_SHORT;
    const BwdPlan plan = bwd_plan(p, workspace_bytes, false, 7u);
    if (plan.pair.taken)
        return ATTN_BWD_FORM_SIDE_BY_SIDE | (plan.pair.dkdv_chunk ? ATTN_BWD_FORM_DKDV_CUT : 0) |
               (plan.pair.dq_nsplit > 1 ? ATTN_BWD_FORM_DQ_CUT : 0);
    const int cut = plan.dkdv_chunk ? ATTN_BWD_FORM_DKDV_CUT : 0;
    if (plan.ds_heads) return ATTN_BWD_FORM_STORED_DS | cut;
    return ATTN_BWD_FORM_APART | cut | (plan.dq_nsplit > 1 ? ATTN_BWD_FORM_DQ_CUT : 0);
}

size_t attn_bwd_gqa_workspace_bytes(const attn_gqa_params_t *p)
{
    if (!p) return 0;
    const attn_rect_params_t g = as_rect(*p);
    return attn_bwd_rect_workspace_bytes(&g);
}

size_t attn_bwd_workspace_bytes(const attn_params_t *p)
{
    if (!p) return 0;
    const attn_gqa_params_t g = as_gqa(*p);
    return attn_bwd_gqa_workspace_bytes(&g);
}

int attn_bwd_rect(const void *Q, const void *K, const void *V, const void *O, const void *dO,
                  const float *LSE, void *dQ, void *dK, void *dV,
                  void *workspace, size_t workspace_bytes,
                  const attn_rect_params_t *p, void *hip_stream)
{
    return bwd_impl<__bf16>(Q, K, V, O, dO, LSE, dQ, dK, dV, workspace, workspace_bytes, p,
                            hip_stream,
                            ATTN_BWD_STAGE_DELTA | ATTN_BWD_STAGE_DKDV | ATTN_BWD_STAGE_DQ);
}

int attn_bwd_rect_f16(const void *Q, const void *K, const void *V, const void *O, const void *dO,
                      const float *LSE, void *dQ, void *dK, void *dV,
                      void *workspace, size_t workspace_bytes,
                      const attn_rect_params_t *p, void *hip_stream)
{
    return bwd_impl<_Float16>(Q, K, V, O, dO, LSE, dQ, dK, dV, workspace, workspace_bytes, p,
                              hip_stream,
                              ATTN_BWD_STAGE_DELTA | ATTN_BWD_STAGE_DKDV | ATTN_BWD_STAGE_DQ);
}

int attn_bwd_gqa(const void *Q, const void *K, const void *V, const void *O, const void *dO,
                 const float *LSE, void *dQ, void *dK, void *dV,
                 void *workspace, size_t workspace_bytes,
                 const attn_gqa_params_t *p, void *hip_stream)
{
    return attn_bwd_gqa_stages(Q, K, V, O, dO, LSE, dQ, dK, dV, workspace, workspace_bytes, p,
                               hip_stream,
                               ATTN_BWD_STAGE_DELTA | ATTN_BWD_STAGE_DKDV | ATTN_BWD_STAGE_DQ);
}

int attn_bwd_gqa_stages(const void *Q, const void *K, const void *V, const void *O,
                        const void *dO, const float *LSE, void *dQ, void *dK, void *dV,
                        void *workspace, size_t workspace_bytes,
                        const attn_gqa_params_t *p, void *hip_stream, uint32_t stages)
{
    if (!p) return ATTN_ERR_NULL;
    const attn_rect_params_t g = as_rect(*p);
    return bwd_impl<__bf16>(Q, K, V, O, dO, LSE, dQ, dK, dV, workspace, workspace_bytes, &g,
                            hip_stream, stages);
}

int attn_bwd(const void *Q, const void *K, const void *V, const void *O, const void *dO,
             const float *LSE, void *dQ, void *dK, void *dV,
             void *workspace, size_t workspace_bytes,
             const attn_params_t *p, void *hip_stream)
{
    return attn_bwd_stages(Q, K, V, O, dO, LSE, dQ, dK, dV, workspace, workspace_bytes, p,
                           hip_stream,
                           ATTN_BWD_STAGE_DELTA | ATTN_BWD_STAGE_DKDV | ATTN_BWD_STAGE_DQ);
}

int attn_bwd_stages(const void *Q, const void *K, const void *V, const void *O, const void *dO,
                    const float *LSE, void *dQ, void *dK, void *dV,
                    void *workspace, size_t workspace_bytes,
                    const attn_params_t *p, void *hip_stream, uint32_t stages)
{
    if (!p) return ATTN_ERR_NULL;
    const attn_gqa_params_t g = as_gqa(*p);
    return attn_bwd_gqa_stages(Q, K, V, O, dO, LSE, dQ, dK, dV, workspace, workspace_bytes, &g,
                               hip_stream, stages);
}

}  // extern "C"

// Scratch of attn_bwd_rect_noalloc: the workspace of the call, in an array that lives in
// the library's device image instead of in memory the caller allocates.  Every GPU the library
// runs on holds its own copy at its own address, so the address is looked up once per device
// (with that device current) and kept; host code uses that pointer, never the array's name.
static __device__ __align__(256) unsigned char scratch[ATTN_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices];  // guarded by g_scratch_mutex; nullptr = not looked up yet
std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device, or nullptr if the runtime refuses.
void *scratch_of_current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

extern "C" {

int attn_bwd_rect_noalloc(const void *Q, const void *K, const void *V, const void *O,
                          const void *dO, const float *LSE, void *dQ, void *dK, void *dV,
                          const attn_rect_params_t *p, void *hip_stream)
{
    // the same checks as attn_bwd_rect, before anything touches the device
    if (!Q || !K || !V || !O || !dO || !LSE || !dQ || !dK || !dV) return ATTN_ERR_NULL;
    const int rc = check_params(p);
    if (rc != ATTN_OK) return rc;
    const size_t need = bwd_stats_bytes(p);
    if (need > (size_t)ATTN_NOALLOC_SCRATCH_BYTES) return ATTN_ERR_WORKSPACE;
    void *ws = scratch_of_current_device();
    if (!ws) return ATTN_ERR_LAUNCH;
    // Every value of the scratch that a kernel reads is written earlier in the same call (the statistics of every
    // query row by the dQ kernel or, in the forms with dS kept or both kernels side by side, by their own; partial
    // results and dS by the kernel before the one that reads them), so nothing has to be cleared although the array
    // keeps the last call's contents.
    return bwd_impl<__bf16>(Q, K, V, O, dO, LSE, dQ, dK, dV, ws, ATTN_NOALLOC_SCRATCH_BYTES, p,
                            hip_stream,
                            ATTN_BWD_STAGE_DELTA | ATTN_BWD_STAGE_DKDV | ATTN_BWD_STAGE_DQ);
}

const char *attn_status_string(int status)
{
    switch (status) {
        case ATTN_OK: return "ok";
        case ATTN_ERR_NULL: return "a required pointer is NULL";
        case ATTN_ERR_SHAPE: return "unsupported shape (B,H,S >= 1, D a multiple of 8 up to 256, Hkv divides Hq, B*H*S < 2^31, causal needs Sk >= Sq)";
        case ATTN_ERR_STRIDE: return "bad stride (D contiguous, strides multiples of 8 elements, stride_s >= D)";
        case ATTN_ERR_ALIGN: return "tensor pointer not 16-byte aligned";
        case ATTN_ERR_WORKSPACE: return "workspace missing, misaligned (256 B) or too small";
        case ATTN_ERR_SCALE: return "scale must be finite and > 0";
        case ATTN_ERR_LAUNCH: return "HIP kernel launch failed";
        default: return "unknown status";
    }
}

int attn_version(void) { return 1005; }

}  // extern "C"
