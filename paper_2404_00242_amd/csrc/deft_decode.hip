// Device side of libdeft: the Attention Calculation Phase of DeFT-Flatten (Algorithm 4) for gfx950.
//
// Stage 1 (deft_stage1): one workgroup of four waves per task = (chunk or run of short chunks, KV head, up to eight
// 16-row tiles).  Short chunks are held in registers whole (resident_task), the others stream (streaming_task).  The
// rows of a tile are (query of the chunk's group) x (query head reading this KV head).
// A wave streams 32 tokens at a time straight from HBM into MFMA operand registers:
//
//   S^T[token, row] = K[token, :] . Q[row, :]      v_mfma_f32_16x16x32_bf16, A = K tile (a lane holds
//                                                   8 consecutive d of one token = one 128-bit load),
//                                                   B = Q (resident in registers for the whole chunk)
//   online softmax over tokens, per row             a row lives in the 4 lanes {n, n+16, n+32, n+48}
//   O^T[d, row]  += V^T[d, token] . P^T[token, row] A = V^T, built from 128-bit row loads by a 2x2
//                                                   16-bit interleave in registers (v_perm_b32),
//                                                   B = P^T, which is S^T's accumulator layout as is
//
// Each token row of one head (2*d bytes, contiguous) is fetched from HBM exactly once per task and every
// byte of every 64-byte sector requested is used.  A narrow group (one row tile) splits the chunk's
// tokens over the four waves, each keeping a block of loads in flight in registers.  A wider group
// gives each wave its own row tile (two tiles for tasks of more than four); the waves that need the same
// block each fetch a share of it and pass the operand registers to the others through LDS.  The waves' partial results
// are merged in LDS before one (m, l, acc) triple per (chunk, row) is written.
//
// Stage 2 (deft_stage2_few, deft_stage2_many): one, two or four waves per (query, query head) merge that query's partial
// results with the log-sum-exp weights of eq. 1.  Small whole calls have both stages in one launch (reduce_rows).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>

#include "deft_internal.h"

// Partial-result workspace of deft_tree_attn_decode_static: device memory inside the code object, one copy
// per GPU at its own address, held until the process ends.  Host code never uses this name as an address;
// it asks the runtime for the device address once per device (static_scratch below).
static __device__ __align__(256) unsigned char scratch[DEFT_STATIC_SCRATCH_BYTES];

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) int32_t i32x4;

struct Stage1Args {
    const uint16_t *q, *k, *v;
    float *part_acc, *part_m, *part_l;
    const int32_t *seg_tok_begin, *seg_len, *seg_qlo, *seg_qhi, *seg_off;
    const int32_t *q_order;
    int32_t n_items, Hq, Hkv, G;
    uint32_t inv_G;  // see divide
    int32_t resident_one, resident_many;  // most row tiles of a task on the resident path, see is_resident
    int32_t table_len;  // entries of the LDS per-token table: longest multi-piece chunk, in whole blocks
    float c;  // scale * log2(e): probabilities are 2^((s - m) * c)
    // A whole call in one launch: a record of 16 bytes per row of partial results, {m, l, mark}, and what this call writes
    // into the marks (publish_rows).  The records of a KV head lie together, in the order of slots and its query heads, so
    // that no two workgroups write to one line at a time (in the order of slots and all heads: 10 % on a call of 4000 rows
    // under 32 heads).
    float *marks;
    uint64_t ticket;
    int32_t n_slots;
};

struct Stage2Args {
    const float *part_acc, *part_m, *part_l;
    const int32_t *q_head, *q_part_slot;
    void *out;
    int32_t nq, Hq, out_f32;
    int32_t head_ints;  // int32 per query record
    uint32_t inv_Hq;
    float c;
};

// What a workgroup needs to ask for its first record is passed ahead of the structures, as plain arguments: the compiler
// has those loaded into registers before the first wave starts (build.py), which takes one round trip out of the chain
// that every workgroup begins with.  Whole call, us: 37 MB over 16-token pages 16.2 -> 15.7, the decode iteration of the
// same tree 170.8 -> 166.0, 21 MB with d = 64 12.4 -> 12.1.

// A whole call in one launch: stage 1's workgroups first, then those of stage 2
struct CallArgs {
    Stage1Args s1;
    Stage2Args s2;
    int32_t polls;  // most looks at a mark before stage 2 leaves a row to stage 1 (reduce_rows)
};

// floor(n / d) for any n and d > 0, given inverse(d); a division by a run-time number costs a workgroup 0.3 us otherwise
uint32_t inverse(uint32_t d) { return d == 1 ? 0xffffffffu : (uint32_t)((uint64_t(1) << 32) / d); }
__device__ __forceinline__ uint32_t divide(uint32_t n, uint32_t d, uint32_t inv) {
    const uint32_t q = __umulhi(n, inv);  // floor(n / d) or one less
    return n - q * d >= d ? q + 1 : q;
}

__device__ __forceinline__ u32x4 load16(const uint16_t *p) { return *reinterpret_cast<const u32x4 *>(p); }
// K/V rows of streaming tasks of one or two row tiles are loaded without being kept in the caches (non-temporal): as a
// rule such a task is its chunk's whole group and no other workgroup will read them; measured 2 % faster on the few-shot
// trees, 5 % where two tiles are all of a group over a long prefix (28644 tokens under 6 queries x 4 heads 33.1 -> 31.2 us
// per call).  Wide groups that the schedule cuts down to two tiles do re-read their rows and would be faster with cached
// loads (478-token root under 256 queries 29.2 -> 24.8 us, 3859 tokens under 44 queries x 6 heads 22.8 -> 22.4), but a
// kernel that holds both kinds of loads pays for it in its wide loops (12345 tokens under 26 queries x 4 heads 28.9 ->
// 29.9, 256-query reasoning tree 119.7 -> 122.5).  Wider tasks and resident ones load through the caches.
__device__ __forceinline__ u32x4 load16_once(const uint16_t *p) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
}
template <bool ONCE>
__device__ __forceinline__ u32x4 load16_kv(const uint16_t *p) {
    return ONCE ? load16_once(p) : load16(p);
}

// Partial results.  SHARED: in a call of one launch they are stored past the L2 of their XCD, and read past the reader's,
// because the workgroup that reads them runs while others still write (publish_rows).  Elsewhere such stores only cost
// time (17 MB of them 1.9 us of 22).
typedef __attribute__((address_space(1))) u32x4 *global_u32x4;
template <bool SHARED>
__device__ __forceinline__ void store_partial(float *p, f32x4 x) {
    if (SHARED)
        __builtin_amdgcn_global_store_b128((global_u32x4)p, __builtin_bit_cast(u32x4, x), "agent");
    else
        *reinterpret_cast<f32x4 *>(p) = x;
}
__device__ __forceinline__ f32x4 load_shared4(const float *p) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_global_load_b128((global_u32x4)p, "agent"));
}

__device__ __forceinline__ float wave_row_max(float x) {
    // a row of a 16-row tile lives in lanes {n, n+16, n+32, n+48}
    // (a swap of rows of 16 lanes, then of halves, between two copies: no LDS round trip)
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t a0 = a[0], a1 = a[1];
    const uint32_t w = __builtin_bit_cast(uint32_t, fmaxf(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1)));
    const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    const uint32_t b0 = b[0], b1 = b[1];
    return fmaxf(__builtin_bit_cast(float, b0), __builtin_bit_cast(float, b1));
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    bf16x2 r = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, r);
}

// In a whole call of one launch, stage 2 may not read a row of partial results before the row is complete.  The wave that
// wrote it waits until its stores have arrived and then puts the call's ticket into the row's mark, for which stage 2's wave
// waits.  Every call has a ticket of its own, 64 bits, so a mark needs no value to start from: whatever a workspace holds,
// it is not the ticket.  (Not so in the replays of a captured call, which would all have one ticket: see one_launch.)
// The mark is exchanged and not just stored, for a wave of stage 2 that would not wait any longer has left word in it, the
// ticket's complement: see reduce_rows.
__device__ __forceinline__ uint64_t *mark_of(float *record) { return reinterpret_cast<uint64_t *>(record) + 1; }
struct LeftRows {
    bool left = false;  // whether stage 2 has left this lane's row to this wave,
    int row = 0;        // which is this one of the task
};
__device__ __forceinline__ LeftRows publish_rows(const Stage1Args &a, bool mine, int row, size_t record) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    LeftRows x;
    x.row = row;
    if (mine) x.left = __hip_atomic_exchange(mark_of(a.marks + 4 * record), a.ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ~a.ticket;
    return x;
}
typedef __attribute__((ext_vector_type(2))) float f32x2;
__device__ __forceinline__ void store_record(const Stage1Args &a, size_t record, float m, float l) {
    __hip_atomic_store(reinterpret_cast<uint64_t *>(a.marks + 4 * record), __builtin_bit_cast(uint64_t, (f32x2{m, l})),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kWaves = 4;              // waves per stage-1 workgroup
constexpr int kXbufBytes = 64 * 1024;  // LDS register-exchange area: 2 token parts x 2 stages x 16 KB
static_assert(4 * DEFT_MAX_CHUNK * sizeof(int32_t) <= kXbufBytes, "piece records are parked in the exchange area");

// What a wave needs to know about its chunk to address tokens.
struct ChunkCtx {
    const uint16_t *kbase, *vbase;  // K/V pointers already offset to this head and this lane's d slice
    const uint16_t *khead, *vhead;  // the same without the lane's slice (wave-uniform), and the slices in bytes
    uint32_t klane, vlane;
    size_t row_stride;              // elements between consecutive token rows
    const int32_t *s_row, *s_qlo, *s_qhi;  // LDS per-token table (only when !uniform), padded to whole blocks
    int clen;                       // tokens in the chunk
    int uniform;                    // the chunk is one piece of one node: rows are begin0 + x
    int begin0, qlo0, qhi0;
    int fresh;                      // blocks after which a new reference is taken (RowState), less one; -1: never
    int n16, g;
};

// One 32-token block as MFMA operands: K as the A operand of S^T = K Q^T (token 16a + n16, d = 32kk + 8g..+7),
// V as loaded, row-major (token 16a + 4g + i, d = 8*n16..+7).  The layout is the same in every wave, whatever
// row tile the wave works on, which is what lets waves exchange these registers through LDS unchanged.
template <int D>
struct KVRegs {
    bf16x8 k[2][D / 32];
    u32x4 v[8];
};

// physical row of chunk position x; positions past the chunk's end give a row that exists (their scores are masked)
__device__ __forceinline__ int tok_row(const ChunkCtx &c, int x) {
    return c.uniform ? c.begin0 + min(x, c.clen - 1) : c.s_row[x];
}

// Loads are issued unconditionally: a block past the end of the wave's work (valid == false) re-reads the
// chunk's first row instead (one cached row, no HBM traffic).  With the same sequence of memory
// instructions on every path the compiler can count exactly how many younger loads may stay in flight when
// an older block is consumed, which is what keeps the software pipeline full.
template <int D>
__device__ __forceinline__ void load_k(KVRegs<D> &r, const ChunkCtx &c, int x0, bool valid) {
    if (!valid) x0 = 0;
#pragma unroll
    for (int aa = 0; aa < 2; ++aa) {
        const int rowk = valid ? tok_row(c, x0 + 16 * aa + c.n16) : c.begin0;
        const uint16_t *kp = c.kbase + (size_t)rowk * c.row_stride;
#pragma unroll
        for (int kk = 0; kk < D / 32; ++kk) r.k[aa][kk] = __builtin_bit_cast(bf16x8, load16_once(kp + 32 * kk));
    }
}
template <int D>
__device__ __forceinline__ void load_v(KVRegs<D> &r, const ChunkCtx &c, int x0, bool valid) {
    if (!valid) x0 = 0;
#pragma unroll
    for (int aa = 0; aa < 2; ++aa)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rowv = valid ? tok_row(c, x0 + 16 * aa + 4 * c.g + i) : c.begin0;
            r.v[4 * aa + i] = load16_once(c.vbase + (size_t)rowv * c.row_stride);
        }
}

// Running softmax state of one row (held redundantly by the row's four lanes).
//   mc  : the reference subtracted inside the exponential, in units of the exponent: the weights are
//         2^(s * cs - mc).  The row's reference maximum in units of the scores is mc / cs.
//   thr : what an exponent s * cs - mc must exceed for the reference to be raised: kLazyLog2, or -inf while
//         the row has seen no visible token (mc is 0 then and stands for "no reference yet")
//   l   : sum over all tokens so far of the bf16-rounded weights, i.e. of exactly the numbers that enter the
//         P.V product.  It is accumulated by one more MFMA per block whose A operand is all ones (every row
//         of that product is the column sum of P^T), which costs the idle matrix pipe 16 cycles instead of 8
//         VALU adds and leaves the total in every lane of the row.
// The reference is only raised when some score exceeds it by more than kLazyLog2 / cs (probabilities may
// then reach 2^kLazyLog2, harmless in bf16 and fp32); otherwise a block costs no cross-lane traffic and
// no rescaling of the accumulators.  Any reference gives the same (m, l, acc) up to rounding, because the
// merge of eq. 1 only needs the three to be consistent.
// The rounding is the smaller the more tokens were the reference once: such a token is among the heaviest of its row, and its
// weight is exactly 1.  A stream that replaces several shorter ones therefore takes a new reference where each of them would
// have begun (kItFresh): the largest exponent of that block, also if it is below the old one, but by no more than kFreshLog2,
// which keeps the sums in range whatever the scores do (2^48 times larger after 6000 tokens in steps of 128).  Only with bf16
// weights: asked in the loops of two-term weights too, it cost trees of both kinds 0.7 % (40.8 -> 41.1 us).
struct RowState {
    float mc, thr;
    f32x4 l;  // four identical copies (rows 4g..4g+3 of the all-ones product)
    // reference maximum in units of the scores, as the partial result states it
    __device__ __forceinline__ float m(float inv_cs) const { return thr == -INFINITY ? -INFINITY : mc * inv_cs; }
};
constexpr float kLazyLog2 = 8.0f;
constexpr float kFreshLog2 = 1.0f;

// Everything a wave keeps for one of its 16-row tiles: Q as the B operand of S^T = K Q^T (resident for the
// whole chunk), the plan position of this lane's row (-1: no such row), the softmax state and the O^T
// accumulators (oacc[c'][i] is d = 32g + 8i + c' of row n16).
template <int D>
struct TileState {
    bf16x8 q[D / 32];
    int qpos;
    RowState rs;
    f32x4 o[8];
};

// Online-softmax step of one wave over one 32-token block, for its NT row tiles.  The K and V operands are
// shared by the tiles, so the loads (or LDS reads) and the V interleave are paid once per block.
//
// PRECISE: every weight enters the P.V product and the denominator as the sum of two bf16 numbers, hi =
// bf16(p) and lo = bf16(p - hi), through a second set of MFMAs, so it carries a relative error of 2^-17
// instead of bf16's 2^-9.  The plan asks for it where some query of the group has a short path: there a
// handful of rounded weights does not average out and an output element would be off by up to
// 2^-7 * sum_t w_t |V_t|.  The matrix pipe has the room (a bandwidth-bound block keeps it busy for a sixth
// of its time).
//
// The pieces of a block's work, in the order compute_block strings them together.  The pipelined loop of the
// wide tasks (WidePipe) calls them separately so that one block's weights and the next block's scores can be
// issued side by side.

// S^T = K Q^T : sacc[t][a][i] is the score of token 16a + 4g + i against row n16 of tile t
template <int D, int NT>
__device__ __forceinline__ void qk_block(const bf16x8 (&k)[2][D / 32], const TileState<D> (&ts)[NT], f32x4 (&sacc)[NT][2]) {
    constexpr int KK = D / 32;
#pragma unroll
    for (int aa = 0; aa < 2; ++aa)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[aa][kk], ts[t].q[kk], acc, 0, 0, 0);
            sacc[t][aa] = acc;
        }
}

// mask: a token is visible to plan position qpos iff qlo <= qpos < qhi of the node piece it belongs to.
// A full block of a single-piece chunk is visible to every row of the chunk's group: nothing to mask
// (rows past the group's end have Q = 0, finite scores, and are never written).
template <int D, int NT>
__device__ __forceinline__ void mask_block(const ChunkCtx &c, int x0, const TileState<D> (&ts)[NT], f32x4 (&sacc)[NT][2]) {
    if (!(c.uniform && x0 + 32 <= c.clen)) {
#pragma unroll
        for (int aa = 0; aa < 2; ++aa) {
            const int xv = x0 + 16 * aa + 4 * c.g;
            i32x4 qlo, qhi;
            if (c.uniform) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool in = xv + i < c.clen;
                    qlo[i] = in ? c.qlo0 : 0;
                    qhi[i] = in ? c.qhi0 : 0;
                }
            } else {
                qlo = *reinterpret_cast<const i32x4 *>(&c.s_qlo[xv]);
                qhi = *reinterpret_cast<const i32x4 *>(&c.s_qhi[xv]);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool on = (ts[t].qpos >= qlo[i]) && (ts[t].qpos < qhi[i]);
                    sacc[t][aa][i] = on ? sacc[t][aa][i] : -INFINITY;
                }
        }
    }
}

// scores -> exponents of the weights: e = s * cs - mc, in place
template <int D, int NT>
__device__ __forceinline__ void shift_block(const TileState<D> (&ts)[NT], f32x4 (&sacc)[NT][2], const float cs) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int aa = 0; aa < 2; ++aa)
#pragma unroll
            for (int i = 0; i < 4; ++i) sacc[t][aa][i] = fmaf(sacc[t][aa][i], cs, -ts[t].rs.mc);
}

// lazy reference, on the shifted scores of shift_block: it is raised (for every tile of the wave) only when
// some exponent exceeds kLazyLog2, i.e. some score exceeds the reference by more than kLazyLog2 / cs.  The
// exponents come out of an fma, so their maximum needs no canonicalisation and takes four instructions per tile.
// fresh: the block takes a new reference.
template <int D, int NT>
__device__ __forceinline__ void raise_block(TileState<D> (&ts)[NT], f32x4 (&sacc)[NT][2], bool fresh = false) {
    float mx[NT];
    bool need = false;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        mx[t] = fmaxf(fmaxf(fmaxf(sacc[t][0][0], sacc[t][0][1]), fmaxf(sacc[t][0][2], sacc[t][0][3])),
                      fmaxf(fmaxf(sacc[t][1][0], sacc[t][1][1]), fmaxf(sacc[t][1][2], sacc[t][1][3])));
        need = need || (mx[t] > ts[t].rs.thr);
    }
    if (__any(need) || fresh) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            // move the reference of every row up to its running maximum (down only for a new one), rescale what was
            // accumulated and move this block's exponents to the new reference
            RowState &st = ts[t].rs;
            const float r = wave_row_max(mx[t]);  // largest exponent of the row in this block, -inf if all masked
            const bool had = st.thr != -INFINITY;
            const float d = had ? fmaxf(r, fresh ? -kFreshLog2 : 0.f) : (r == -INFINITY ? 0.f : r);
            const float alpha = had ? __builtin_amdgcn_exp2f(-d) : 0.f;  // nothing was accumulated before the first
            st.mc += d;
            st.thr = (had || r != -INFINITY) ? kLazyLog2 : -INFINITY;
            st.l *= alpha;
#pragma unroll
            for (int cc = 0; cc < 8; ++cc) ts[t].o[cc] *= alpha;
#pragma unroll
            for (int aa = 0; aa < 2; ++aa)
#pragma unroll
                for (int i = 0; i < 4; ++i) sacc[t][aa][i] -= d;
        }
    }
}

// weights of the block, 2^(shifted score), as bf16 B operands (PRECISE: plus what the rounding to bf16 dropped, itself rounded to
// bf16; hi widens to fp32 by a 16-bit shift)
template <int D, int NT, bool PRECISE>
__device__ __forceinline__ void weights_block(const TileState<D> (&ts)[NT], const f32x4 (&sacc)[NT][2], const float cs,
                                              bf16x8 (&preg)[NT], bf16x8 (&plo)[NT]) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float pv[8];
#pragma unroll
        for (int aa = 0; aa < 2; ++aa)
#pragma unroll
            for (int i = 0; i < 4; ++i) pv[4 * aa + i] = __builtin_amdgcn_exp2f(sacc[t][aa][i]);
        const u32x4 pk = {pack_bf16(pv[0], pv[1]), pack_bf16(pv[2], pv[3]), pack_bf16(pv[4], pv[5]),
                          pack_bf16(pv[6], pv[7])};
        preg[t] = __builtin_bit_cast(bf16x8, pk);
        if (PRECISE) {
            u32x4 lk;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float h0 = __builtin_bit_cast(float, pk[j] << 16);
                const float h1 = __builtin_bit_cast(float, pk[j] & 0xffff0000u);
                lk[j] = pack_bf16(pv[2 * j] - h0, pv[2 * j + 1] - h1);
            }
            plo[t] = __builtin_bit_cast(bf16x8, lk);
        }
    }
}

// l += column sums of P^T;  O^T += V^T P^T
// READY: v[2*c2] and v[2*c2 + 1] already are the interleaved operands vt_lo and vt_hi described below (the
// waves that fetched V interleaved it before passing it on).
template <int D, int NT, bool PRECISE, bool READY = false>
__device__ __forceinline__ void pv_block(const u32x4 (&v)[8], const bf16x8 (&preg)[NT], const bf16x8 (&plo)[NT],
                                         TileState<D> (&ts)[NT]) {
    {
        const u32x4 one4 = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};  // eight bf16 1.0
        const bf16x8 ones = __builtin_bit_cast(bf16x8, one4);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            ts[t].rs.l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, preg[t], ts[t].rs.l, 0, 0, 0);
            if (PRECISE) ts[t].rs.l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, plo[t], ts[t].rs.l, 0, 0, 0);
        }
    }
    // The V^T operand of product c' = 2*c2 + {0,1} is a 16-bit interleave of token pairs:
    // vt[p] = {V[tok 2p][8*n16 + c'], V[tok 2p+1][8*n16 + c']}
#pragma unroll
    for (int c2 = 0; c2 < 4; ++c2) {
        u32x4 vt_lo, vt_hi;
        if (READY) {
            vt_lo = v[2 * c2];
            vt_hi = v[2 * c2 + 1];
        } else {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const uint32_t lo = v[2 * p][c2], hi = v[2 * p + 1][c2];
                vt_lo[p] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                vt_hi[p] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
            }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            ts[t].o[2 * c2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt_lo), preg[t],
                                                                       ts[t].o[2 * c2], 0, 0, 0);
            ts[t].o[2 * c2 + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt_hi), preg[t],
                                                                           ts[t].o[2 * c2 + 1], 0, 0, 0);
            if (PRECISE) {
                ts[t].o[2 * c2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt_lo), plo[t],
                                                                           ts[t].o[2 * c2], 0, 0, 0);
                ts[t].o[2 * c2 + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt_hi), plo[t],
                                                                               ts[t].o[2 * c2 + 1], 0, 0, 0);
            }
        }
    }
}

template <int D, int NT, bool PRECISE>
__device__ __forceinline__ void compute_block(const KVRegs<D> &r, const ChunkCtx &c, int x0, TileState<D> (&ts)[NT],
                                              const float cs, const float inv_cs) {
    f32x4 sacc[NT][2];
    qk_block<D, NT>(r.k, ts, sacc);
    mask_block<D, NT>(c, x0, ts, sacc);
    shift_block<D, NT>(ts, sacc, cs);
    raise_block<D, NT>(ts, sacc);
    bf16x8 preg[NT], plo[NT];
    weights_block<D, NT, PRECISE>(ts, sacc, cs, preg, plo);
    pv_block<D, NT, PRECISE>(r.v, preg, plo, ts);
}

// ---- token-split path (groups of one row tile): every wave streams its own blocks.  K of the next block is asked for
//      as soon as the scores are formed, V as soon as the products are, each into the registers it replaces ----
// wave w takes blocks w, w+4, w+8, ... (neighbouring waves read neighbouring rows at the same time).
// Bound by HBM.  One block of 16 KB per wave, 128 KB per compute unit, is nine times what the unit's share of the
// bandwidth needs at the latency of a loaded chip (24 GB/s x 0.6 us); a second block per wave only made the queue in
// front of the other workgroup's loads longer.  Stage 1, two blocks -> one reloaded whole -> in halves: sixteen
// sequences (148 MB) 29.9 -> 28.8 -> 27.8 us, few-shot prefix (149 MB) 28.7 -> 28.7 -> 27.7, reasoning tree of 256
// queries (456 MB) 96.2 -> 94.5 -> 93.6.
template <int D>
struct SplitPipe {
    KVRegs<D> r;
    __device__ __forceinline__ void prime(const ChunkCtx &ctx, int wave, int nblk) {
        load_k<D>(r, ctx, wave * 32, wave < nblk);
        load_v<D>(r, ctx, wave * 32, wave < nblk);
    }
    template <bool PRECISE>
    __device__ __forceinline__ void run(const ChunkCtx &ctx, int wave, int nblk, TileState<D> (&ts)[1], float cs) {
        for (int blk = wave; blk < nblk; blk += kWaves) {
            const int next = blk + kWaves;
            f32x4 sacc[1][2];
            bf16x8 preg[1], plo[1];
            qk_block<D, 1>(r.k, ts, sacc);
            load_k<D>(r, ctx, next * 32, next < nblk);
            __builtin_amdgcn_sched_barrier(0);  // the loads go out here, not behind the softmax
            mask_block<D, 1>(ctx, blk * 32, ts, sacc);
            shift_block<D, 1>(ts, sacc, cs);
            raise_block<D, 1>(ts, sacc);
            weights_block<D, 1, PRECISE>(ts, sacc, cs, preg, plo);
            pv_block<D, 1, PRECISE>(r.v, preg, plo, ts);
            load_v<D>(r, ctx, next * 32, next < nblk);
        }
    }
};

// ---- row-split path (groups of TR = 2 or 4 row tiles): the TR waves that work on the same blocks each
//      fetch 1/TR of a block from HBM and pass it to the others through LDS, so the block is read once.
// A block is 2*KK + 8 register images of 1 KB (K tile a, step kk -> image a*KK + kk; V token j -> image
// 2*KK + j).  With TR = 2 wave t fetches K tile t and V tokens 4t..4t+3; with TR = 4 waves 0 and 1 fetch the
// two K tiles and waves 2 and 3 four V tokens each.  Either way every 2*d-byte token row is read whole, by
// one wave, in back-to-back loads.
template <int D, int TR>
struct Share {
    static constexpr int KK = D / 32;
    static constexpr int NSLOT = 2 * KK + 8;
    static constexpr int NX = TR == 2 ? KK + 4 : (KK > 4 ? KK : 4);
    u32x4 x[NX];
};

template <int D, int TR>
__device__ __forceinline__ void share_issue(Share<D, TR> &s, const ChunkCtx &c, int t, int x0, bool valid) {
    constexpr int KK = D / 32;
    if (!valid) x0 = 0;
    if (TR == 2 || t < 2) {
        const int rowk = valid ? tok_row(c, x0 + 16 * t + c.n16) : c.begin0;
        const uint16_t *kp = c.kbase + (size_t)rowk * c.row_stride;
#pragma unroll
        for (int q = 0; q < KK; ++q) s.x[q] = load16_kv<TR == 2>(kp + 32 * q);
    }
    if (TR == 2) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int rowv = valid ? tok_row(c, x0 + 16 * t + 4 * c.g + q) : c.begin0;
            s.x[KK + q] = load16_once(c.vbase + (size_t)rowv * c.row_stride);
        }
    } else if (t >= 2) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int rowv = valid ? tok_row(c, x0 + 16 * (t - 2) + 4 * c.g + q) : c.begin0;
            s.x[q] = load16(c.vbase + (size_t)rowv * c.row_stride);
        }
    }
}

template <int D, int TR, int NT, bool PRECISE>
__device__ __forceinline__ void share_step(Share<D, TR> &s, const ChunkCtx &c, u32x4 *xs, int t, int lane, int blk,
                                           int next_blk, int nblk, TileState<D> (&ts)[NT], float cs, float inv_cs) {
    constexpr int KK = D / 32;
    const bool live = blk < nblk;
    if (live) {
        if (TR == 2 || t < 2) {
#pragma unroll
            for (int q = 0; q < KK; ++q) xs[(t * KK + q) * 64 + lane] = s.x[q];
        }
        if (TR == 2) {
#pragma unroll
            for (int q = 0; q < 4; ++q) xs[(2 * KK + 4 * t + q) * 64 + lane] = s.x[KK + q];
        } else if (t >= 2) {
#pragma unroll
            for (int q = 0; q < 4; ++q) xs[(2 * KK + 4 * (t - 2) + q) * 64 + lane] = s.x[q];
        }
    }
    __syncthreads();
    share_issue<D, TR>(s, c, t, next_blk * 32, next_blk < nblk);
    if (live) {
        KVRegs<D> r;
#pragma unroll
        for (int aa = 0; aa < 2; ++aa)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) r.k[aa][kk] = __builtin_bit_cast(bf16x8, xs[(aa * KK + kk) * 64 + lane]);
#pragma unroll
        for (int j = 0; j < 8; ++j) r.v[j] = xs[(2 * KK + j) * 64 + lane];
        compute_block<D, NT, PRECISE>(r, c, blk * 32, ts, cs, inv_cs);
    }
}

// Used for tasks of two row tiles (TR = 2, NT = 1: two waves per tile, the two pairs take alternate blocks);
// wider tasks go through WidePipe below.
template <int D, int TR, int NT>
struct SharedPipe {
    using S = Share<D, TR>;
    static constexpr int NP = kWaves / TR;  // token parts: part p takes blocks p, p+NP, ...
    static constexpr int DEPTH = 2;  // blocks whose shares a wave keeps in flight
    Share<D, TR> st[DEPTH];
    __device__ __forceinline__ void prime(const ChunkCtx &ctx, int wave, int nblk) {
        const int t = wave % TR, part = wave / TR;
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) share_issue<D, TR>(st[u], ctx, t, (part + u * NP) * 32, part + u * NP < nblk);
    }
    template <bool PRECISE>
    __device__ __forceinline__ void run(const ChunkCtx &ctx, u32x4 *xbuf, int wave, int lane, int nblk,
                                        TileState<D> (&ts)[NT], float cs, float inv_cs) {
        const int t = wave % TR, part = wave / TR;
        const int iters = (nblk + NP - 1) / NP;  // the same for every wave: barriers stay aligned
        u32x4 *xb = xbuf + (size_t)part * 2 * S::NSLOT * 64;
        // whole rounds of DEPTH steps; steps past the last block only keep the barrier and a dummy load
        for (int it0 = 0; it0 < iters; it0 += DEPTH) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                const int it = it0 + u;
                const int blk = part + it * NP;
                // LDS exchange stages alternate; stage (it & 1) was last read two steps ago, before the
                // barrier of the previous step
                share_step<D, TR, NT, PRECISE>(st[u], ctx, xb + (it & 1) * S::NSLOT * 64, t, lane, blk, blk + DEPTH * NP, nblk,
                                      ts, cs, inv_cs);
            }
        }
    }
};

// ---- row-split path for groups of 3 to 8 row tiles (TR = 4: the four waves share every block), pipelined
//      across blocks.  A wave's vector work on a block (32 exponentials and their scaling and packing, for two
//      tiles) takes longer than the block's MFMAs, and inside one basic block the matrix pipe and the vector
//      pipe run side by side; so the weights of block b-1 are formed while the scores of block b are
//      multiplied, and the P.V products of block b-1 follow.  Between two barriers a wave therefore holds the
//      scores and V of one block and K of the next.
//      UNIFORM: the chunk is one piece of one node, so its rows are consecutive.  A whole block's share is
//      then addressed as (wave-uniform pointer that moves on by one block per step) + (a byte offset per lane
//      that never changes): no vector arithmetic per load.  The last, partial block and the dummy loads past
//      the end go through the general addressing.
//      DEPTH: blocks whose shares a wave keeps in flight: one where a wave has one tile, two where it has two, whatever
//      the chunk's length.  A task of 5-8 tiles is what its launch waits for, and with one block in flight each of its
//      steps waits for loads that queue behind those of the workgroup beside it.  Whole call, us, one -> two: 120
//      queries x 4 heads over 32768 tokens in chunks of 1024 (equal-token split) 175 -> 163, 20000 tokens under 40
//      branches 89.8 -> 77.3, 32768 under 40 branches, 7 heads a KV head, 104.7 -> 91.0; where such tasks are few among
//      many narrow ones a second block costs 2 % (256-query reasoning tree, balanced split, 97.7 -> 99.9).
template <int D, int NT, bool UNIFORM, int DEPTH>
struct WidePipe {
    static constexpr int KK = D / 32;
    using S = Share<D, 4>;
    S st[DEPTH];
    uint32_t lane_row, lane_col;  // UNIFORM: first row of this lane's loads inside a block, byte offset inside a row

    // UNIFORM: load q of the share is (wave-uniform pointer of the block) + (row of the lane, clamped to the
    // chunk's last row) * row bytes + the lane's column; a K loader reads four 64-byte columns of one row, a V
    // loader one column of four rows.  No branch on any path: blocks past the end repeat the last block, so the same four load instructions are
    // issued whatever happens and the compiler's s_waitcnt vmcnt counts stay exact.
    __device__ __forceinline__ void issue(S &sh, const ChunkCtx &c, int t, int blk, int nblk) {
        if (UNIFORM) {
            static_assert(KK == 4 || !UNIFORM, "a K loader issues four loads");
            const int blk_e = min(blk, nblk - 1);
            const uint32_t row_bytes = (uint32_t)c.row_stride * 2;
            const size_t first = ((size_t)c.begin0 + 32 * (size_t)blk_e) * row_bytes;
            const int lim = min(31, c.clen - 1 - 32 * blk_e);  // last row of the block that exists
            const bool kl = t < 2;
            const char *base = reinterpret_cast<const char *>(kl ? c.khead : c.vhead) + first;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // K loader: four 64-byte columns of row lane_row; V loader: rows lane_row .. lane_row + 3
                const int row = min((int)lane_row + (kl ? 0 : q), lim);
                const uint32_t off = (uint32_t)row * row_bytes + lane_col + (kl ? 64u * q : 0u);
                sh.x[q] = *reinterpret_cast<const u32x4 *>(base + off);
            }
        } else {
            share_issue<D, 4>(sh, c, t, blk * 32, blk < nblk);
        }
    }

    __device__ __forceinline__ void prime(const ChunkCtx &ctx, int wave, int nblk) {
        lane_row = wave < 2 ? 16 * wave + ctx.n16 : 16 * (wave - 2) + 4 * ctx.g;
        lane_col = wave < 2 ? ctx.klane : ctx.vlane;
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) issue(st[u], ctx, wave, u, nblk);
    }

    // pass this wave's share of a block to the others and fetch the share of a later block
    __device__ __forceinline__ void exchange(S &sh, const ChunkCtx &c, u32x4 *xs, int t, int lane, int next_blk, int nblk) {
        if (t < 2) {
#pragma unroll
            for (int q = 0; q < KK; ++q) xs[(t * KK + q) * 64 + lane] = sh.x[q];
        } else {
            // V: this wave holds tokens 16(t-2) + 4g + {0..3}, i.e. the token pairs p = 2(t-2) and 2(t-2) + 1 of
            // every lane's eight; it interleaves them once for all four waves (pv_block, READY) and writes its
            // half (8 bytes) of each of the eight operand images
            uint2 *xh = reinterpret_cast<uint2 *>(xs + 2 * KK * 64) + (t - 2);
#pragma unroll
            for (int c2 = 0; c2 < 4; ++c2) {
                const uint32_t lo0 = sh.x[0][c2], hi0 = sh.x[1][c2], lo1 = sh.x[2][c2], hi1 = sh.x[3][c2];
                xh[((2 * c2) * 64 + lane) * 2] = make_uint2(__builtin_amdgcn_perm(hi0, lo0, 0x05040100u),
                                                            __builtin_amdgcn_perm(hi1, lo1, 0x05040100u));
                xh[((2 * c2 + 1) * 64 + lane) * 2] = make_uint2(__builtin_amdgcn_perm(hi0, lo0, 0x07060302u),
                                                                __builtin_amdgcn_perm(hi1, lo1, 0x07060302u));
            }
        }
        __syncthreads();
        issue(sh, c, t, next_blk, nblk);
    }
    static __device__ __forceinline__ void read_k(const u32x4 *xs, int lane, bf16x8 (&k)[2][KK]) {
#pragma unroll
        for (int aa = 0; aa < 2; ++aa)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) k[aa][kk] = __builtin_bit_cast(bf16x8, xs[(aa * KK + kk) * 64 + lane]);
    }
    static __device__ __forceinline__ void read_v(const u32x4 *xs, int lane, u32x4 (&v)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = xs[(2 * KK + j) * 64 + lane];
    }

    // one steady-state step: block `blk` arrives, block blk-1 (scores in sacc, V in vreg) is finished.  WHOLE: the block
    // is known to need no mask; without a branch in front of them the shift and the check of its scores are issued
    // while the products of block blk-1 are multiplied.  Not with two-term weights: there the second set of products
    // fills the matrix pipe as it is, and what is kept alive across them costs more (64 queries x 4 heads, reasoning tree
    // of two-term weights, 22.6 us with the branch, 24.7 without; 256 queries, 286-token root, 29.5 and 33.3).
    template <bool PRECISE, bool WHOLE>
    __device__ __forceinline__ void step(S &sh, const ChunkCtx &c, u32x4 *xs, int t, int lane, int blk, int nblk,
                                         TileState<D> (&ts)[NT], f32x4 (&sacc)[NT][2], u32x4 (&vreg)[8], float cs,
                                         float inv_cs, bool fresh = false) {
        exchange(sh, c, xs, t, lane, blk + DEPTH, nblk);
        bf16x8 k[2][KK];
        read_k(xs, lane, k);
        bf16x8 preg[NT], plo[NT];
        f32x4 snew[NT][2];
        weights_block<D, NT, PRECISE>(ts, sacc, cs, preg, plo);
        qk_block<D, NT>(k, ts, snew);
        pv_block<D, NT, PRECISE, true>(vreg, preg, plo, ts);
        read_v(xs, lane, vreg);
        if (!WHOLE) mask_block<D, NT>(c, blk * 32, ts, snew);
        shift_block<D, NT>(ts, snew, cs);
        raise_block<D, NT>(ts, snew, fresh);
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
            sacc[tt][0] = snew[tt][0];
            sacc[tt][1] = snew[tt][1];
        }
    }

    template <bool PRECISE>
    __device__ __forceinline__ void run(const ChunkCtx &ctx, u32x4 *xbuf, int wave, int lane, int nblk,
                                        TileState<D> (&ts)[NT], float cs, float inv_cs) {
        const int t = wave;
        constexpr int STAGE = S::NSLOT * 64;  // u32x4 per LDS exchange stage; stage (blk & 1) holds block blk
        f32x4 sacc[NT][2];
        u32x4 vreg[8];
        {   // block 0: scores only
            exchange(st[0], ctx, xbuf, t, lane, DEPTH, nblk);
            bf16x8 k[2][KK];
            read_k(xbuf, lane, k);
            qk_block<D, NT>(k, ts, sacc);
            read_v(xbuf, lane, vreg);
            mask_block<D, NT>(ctx, 0, ts, sacc);
            shift_block<D, NT>(ts, sacc, cs);
            raise_block<D, NT>(ts, sacc);
        }
        // steady state, DEPTH steps per round so that the shares in flight are addressed statically.  Whole
        // rounds only inside the loop (a round that could stop half way would make the compiler assume, for the
        // waits of the next round, that the share it consumes is the youngest one in flight).  kWhole: every block
        // but the last is whole, so the loop leaves that one to the steps behind it.
        constexpr bool kWhole = UNIFORM && !PRECISE;
        const int b_end = kWhole ? nblk - 1 : nblk;
        int b0 = 1;
        for (; b0 + DEPTH <= b_end; b0 += DEPTH) {
            // whether the round begins with a new reference (RowState); asked once a round, because in every step it cost the
            // wide tasks that keep one reference 0.3 to 0.4 %
            const bool fresh = UNIFORM && !PRECISE && (b0 & ctx.fresh) == max(ctx.fresh, 0);
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                const int blk = b0 + u;
                step<PRECISE, kWhole>(st[(1 + u) % DEPTH], ctx, xbuf + (blk & 1) * STAGE, t, lane, blk, nblk, ts, sacc, vreg, cs, inv_cs,
                                      u == 0 && fresh);
            }
        }
#pragma unroll
        for (int u = 0; u < (kWhole ? DEPTH : DEPTH - 1); ++u)
            if (b0 + u < nblk)
                step<PRECISE, false>(st[(1 + u) % DEPTH], ctx, xbuf + ((b0 + u) & 1) * STAGE, t, lane, b0 + u, nblk, ts, sacc, vreg, cs, inv_cs);
        {   // last block: weights and products
            bf16x8 preg[NT], plo[NT];
            weights_block<D, NT, PRECISE>(ts, sacc, cs, preg, plo);
            pv_block<D, NT, PRECISE, true>(vreg, preg, plo, ts);
        }
    }
};

// ---- resident path: chunks short enough to be held in registers ----
// A chunk of at most kResidentTokens<D> tokens is loaded once, all of it at the start, into the registers of the
// four waves (wave w holds blocks w, w+4, ...), and the row tiles of the task then pass over it one after the other:
// Q of the next tile is fetched while the current one is worked on, the softmax of a tile needs no running state
// (every token is there, so the maximum is exact), and the four waves' results of a tile are added in LDS.  A step
// costs one barrier per 16 rows instead of one per 32 tokens, and no K or V byte goes through LDS.
// Bound by latency: the chain descriptor -> rows and pieces -> K/V and Q -> tiles, each link taken once per task.
// Stage 1, before -> after: 64 x 128 tokens x 8 heads, one tile (33.6 MB) 11.5 -> 8.1 us; 288 tasks of 256 tokens over
// 16-token pages (37 MB) 19.9 -> 12.2 us, together with the finer cut of rows in the schedule.  The K/V loads go through
// the caches: non-temporal ones are 10 % faster where the rows come from HBM (6750 tokens of one sequence 12.8 -> 11.4 us
// per call) and 10 to 16 % slower where the memory-side cache still has them (1349 tokens under 4 queries x 4 heads 9.0 ->
// 10.2), as it has for models of few layers and trees of a few MB.
template <int D>
constexpr int kResidentBlocks = 256 / D;  // blocks per wave: 128 registers of K and V
template <int D>
constexpr int kResidentTokens = 32 * kWaves * kResidentBlocks<D>;
constexpr int kTaskRows = 16 * deft::kMaxTilesPerTask;

// LDS of the resident path, in floats / int32: two merge buffers (tiles alternate), the task's rows, the tokens
template <int D>
struct ResidentLds {
    static constexpr int kPitch = D + 4;
    static constexpr int kMerge = kWaves * 16 * kPitch + 2 * kWaves * 16;  // O, then m and l, of one tile
    static constexpr int kRows = 2 * kMerge;
    static constexpr int kTokens = kRows + 4 * kTaskRows;
    static constexpr int kWords = kTokens + 3 * kResidentTokens<D>;
    static_assert(4 * kResidentTokens<D> <= kRows, "piece records are parked in the merge buffers");
};

template <int D>
struct ResidentTask {
    static constexpr int KK = D / 32, VW = D / 16, NB = kResidentBlocks<D>;
    bf16x8 k[NB][2][KK];  // A operand of S^T = K Q^T, as in KVRegs
    u32x4 vt[NB][VW];     // A operand of product c' of O^T += V^T P^T: row n16 of it is d = VW * n16 + c'
    bf16x8 q[KK];
    typedef __attribute__((ext_vector_type(VW / 2))) uint32_t vrow;  // VW values of one token, as loaded

    // Blocks 0..NA-1 of this wave.  Positions past the chunk's end repeat its last row (their scores are masked).
    template <int NA>
    __device__ __forceinline__ void load(vrow (&v)[NA][8], const ChunkCtx &c, const uint16_t *k_lane, const uint16_t *v_lane,
                                         int wave) {
#pragma unroll
        for (int b = 0; b < NA; ++b) {
            const int x0 = 32 * (wave + kWaves * b);
#pragma unroll
            for (int aa = 0; aa < 2; ++aa) {
                const uint16_t *kp = k_lane + (size_t)tok_row(c, min(x0 + 16 * aa + c.n16, c.clen - 1)) * c.row_stride;
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) k[b][aa][kk] = __builtin_bit_cast(bf16x8, load16(kp + 32 * kk));
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int x = min(x0 + 16 * (j >> 2) + 4 * c.g + (j & 3), c.clen - 1);
                v[b][j] = *reinterpret_cast<const vrow *>(v_lane + (size_t)tok_row(c, x) * c.row_stride);
            }
        }
    }
    // 2x2 interleave of token pairs, see pv_block; done once for all tiles
    template <int NA>
    __device__ __forceinline__ void interleave(const vrow (&v)[NA][8]) {
#pragma unroll
        for (int b = 0; b < NA; ++b)
#pragma unroll
            for (int c2 = 0; c2 < VW / 2; ++c2)
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const uint32_t lo = v[b][2 * p][c2], hi = v[b][2 * p + 1][c2];
                    vt[b][2 * c2][p] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                    vt[b][2 * c2 + 1][p] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
                }
    }
    __device__ __forceinline__ void load_q(const uint16_t *q_lane, int row) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) q[kk] = __builtin_bit_cast(bf16x8, load16(q_lane + (size_t)row * D + 32 * kk));
    }

    // One wave's share of one tile: scores of its NA blocks, softmax over them, products, into the merge buffer.
    // `between` runs once the scores are under way: the sum over the waves of the tile before.
    template <int NA, bool MASK, bool PRECISE, typename F>
    __device__ __forceinline__ void tile(const ChunkCtx &c, int wave, int qpos, int vis_lo, int vis_hi, const uint16_t *q_lane,
                                         int next_row, float cs, float *buf, F &&between) {
        const u32x4 one4 = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};  // eight bf16 1.0
        const bf16x8 ones = __builtin_bit_cast(bf16x8, one4);
        f32x4 o[VW], l = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cc = 0; cc < VW; ++cc) o[cc] = f32x4{0.f, 0.f, 0.f, 0.f};
        float mx = -INFINITY;
        f32x4 s[NA][2];
#pragma unroll
        for (int b = 0; b < NA; ++b)
#pragma unroll
            for (int aa = 0; aa < 2; ++aa) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < KK; ++kk)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[b][aa][kk], q[kk], acc, 0, 0, 0);
                s[b][aa] = acc;
            }
        load_q(q_lane, next_row);
        __builtin_amdgcn_sched_barrier(0);  // the loads go out here, not where the registers run short
        between();
        // a tile none of whose rows sees any token of this wave contributes nothing (chunks of several branches)
        if (!MASK || __any(qpos >= vis_lo && qpos < vis_hi)) {
            if (MASK) {
#pragma unroll
                for (int b = 0; b < NA; ++b)
#pragma unroll
                    for (int aa = 0; aa < 2; ++aa) {
                        const int xv = 32 * (wave + kWaves * b) + 16 * aa + 4 * c.g;
                        const i32x4 qlo = *reinterpret_cast<const i32x4 *>(&c.s_qlo[xv]);
                        const i32x4 qhi = *reinterpret_cast<const i32x4 *>(&c.s_qhi[xv]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) s[b][aa][i] = (qpos >= qlo[i] && qpos < qhi[i]) ? s[b][aa][i] : -INFINITY;
                    }
            }
#pragma unroll
            for (int b = 0; b < NA; ++b)
#pragma unroll
                for (int aa = 0; aa < 2; ++aa)
#pragma unroll
                    for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[b][aa][i]);
            mx = wave_row_max(mx);
            const float mc = mx == -INFINITY ? 0.f : mx * cs;
#pragma unroll
            for (int b = 0; b < NA; ++b) {
                float pv[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) pv[j] = __builtin_amdgcn_exp2f(fmaf(s[b][j >> 2][j & 3], cs, -mc));
                u32x4 pk;
#pragma unroll
                for (int j = 0; j < 4; ++j) pk[j] = pack_bf16(pv[2 * j], pv[2 * j + 1]);
                const bf16x8 hi = __builtin_bit_cast(bf16x8, pk);
                l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, hi, l, 0, 0, 0);
#pragma unroll
                for (int cc = 0; cc < VW; ++cc)
                    o[cc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt[b][cc]), hi, o[cc], 0, 0, 0);
                if (PRECISE) {  // what the rounding to bf16 dropped, see weights_block
                    u32x4 lk;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        lk[j] = pack_bf16(pv[2 * j] - __builtin_bit_cast(float, pk[j] << 16),
                                          pv[2 * j + 1] - __builtin_bit_cast(float, pk[j] & 0xffff0000u));
                    const bf16x8 lo = __builtin_bit_cast(bf16x8, lk);
                    l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, lo, l, 0, 0, 0);
#pragma unroll
                    for (int cc = 0; cc < VW; ++cc)
                        o[cc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt[b][cc]), lo, o[cc], 0, 0, 0);
                }
            }
        }
        publish(c, wave, o, mx, l[0], buf);
    }

    // this wave's part of a tile's result: the lane owns d in [D/4 * g, D/4 * (g+1)) of row n16, d = VW * (4g + i) + c'
    __device__ __forceinline__ void publish(const ChunkCtx &c, int wave, const f32x4 (&o)[VW], float m, float l, float *buf) {
        float *dst = buf + (wave * 16 + c.n16) * ResidentLds<D>::kPitch + (D / 4) * c.g;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int cc = 0; cc < VW; cc += 4)
                *reinterpret_cast<f32x4 *>(dst + VW * i + cc) = f32x4{o[cc][i], o[cc + 1][i], o[cc + 2][i], o[cc + 3][i]};
        // the four lanes of a row store the same two numbers
        float *ml = buf + kWaves * 16 * ResidentLds<D>::kPitch + wave * 16 + c.n16;
        ml[0] = m;
        ml[kWaves * 16] = l;
    }

    // The tiles of the task, one barrier each: a wave writes its part of tile t, and adds up four rows of that tile
    // while it works on tile t + 1 in the other buffer.
    template <int NA, bool MASK, bool PRECISE, bool SHARED>
    __device__ __forceinline__ LeftRows run(const Stage1Args &a, const ChunkCtx &c, float *lds, int wave, int lane, int ntiles,
                                            int rows, const uint16_t *q_lane, int vis_lo, int vis_hi) {
        using L = ResidentLds<D>;
        const int32_t *row_q = reinterpret_cast<const int32_t *>(lds + L::kRows), *row_pos = row_q + kTaskRows;
        const uint32_t *row_out = reinterpret_cast<const uint32_t *>(row_pos + kTaskRows), *row_rec = row_out + kTaskRows;
        const int n = 4 * wave + (lane >> 4), dc = lane & 15;
        auto merge = [&](int t, auto final) {
            const float *buf = lds + (t & 1) * L::kMerge, *ml = buf + kWaves * 16 * L::kPitch + n;
            float m[kWaves], M = -INFINITY;
#pragma unroll
            for (int sp = 0; sp < kWaves; ++sp) {
                m[sp] = ml[sp * 16];
                M = fmaxf(M, m[sp]);
            }
            const float ref = M == -INFINITY ? 0.f : M;
            float sum = 0.f;
            f32x4 acc[D / 64];
#pragma unroll
            for (int e = 0; e < D / 64; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sp = 0; sp < kWaves; ++sp) {
                const float w = __builtin_amdgcn_exp2f((m[sp] - ref) * a.c);
                sum += w * ml[(kWaves + sp) * 16];
#pragma unroll
                for (int e = 0; e < D / 64; ++e)
                    acc[e] += w * *reinterpret_cast<const f32x4 *>(buf + (sp * 16 + n) * L::kPitch + 64 * e + 4 * dc);
            }
            // Only the last tile has rows past the end, and only there they are left out: elsewhere no condition, so that
            // the number of stores behind the next Q loads is the same on every path and the wait for those counts them
            // exactly.
            if (decltype(final)::value && 16 * t + n >= rows) return;
            const size_t ro = row_out[16 * t + n];
            *((dc & 1 ? a.part_l : a.part_m) + ro) = dc & 1 ? sum : M;
            if (SHARED && dc == 0) store_record(a, row_rec[16 * t + n], M, sum);
#pragma unroll
            for (int e = 0; e < D / 64; ++e) store_partial<SHARED>(a.part_acc + ro * D + 64 * e + 4 * dc, acc[e]);
        };
        if constexpr (NA == 0) {  // a wave without a block: its part is empty in both buffers from the start
            f32x4 o[VW];
#pragma unroll
            for (int cc = 0; cc < VW; ++cc) o[cc] = f32x4{0.f, 0.f, 0.f, 0.f};
            publish(c, wave, o, -INFINITY, 0.f, lds);
            publish(c, wave, o, -INFINITY, 0.f, lds + L::kMerge);
            for (int t = 0; t < ntiles; ++t) {
                __syncthreads();
                if (t + 1 < ntiles)
                    merge(t, std::false_type());
                else
                    merge(t, std::true_type());
            }
        } else {
            const int last = 16 * (ntiles - 1) + c.n16;
            tile<NA, MASK, PRECISE>(c, wave, MASK ? row_pos[c.n16] : 0, vis_lo, vis_hi, q_lane, row_q[min(16 + c.n16, last)],
                                    a.c, lds, [] {});
            __builtin_amdgcn_s_waitcnt(0);  // nothing but the loop's own loads and stores is in flight inside it
            for (int t = 1; t < ntiles; ++t) {
                __syncthreads();
                tile<NA, MASK, PRECISE>(c, wave, MASK ? row_pos[16 * t + c.n16] : 0, vis_lo, vis_hi, q_lane,
                                        row_q[min(16 * (t + 1) + c.n16, last)], a.c, lds + (t & 1) * L::kMerge,
                                        [&] { merge(t - 1, std::false_type()); });
            }
            __syncthreads();
            merge(ntiles - 1, std::true_type());
        }
        // this wave's rows: 4 * wave .. 4 * wave + 3 of every tile
        const int mine = 16 * (lane >> 2) + 4 * wave + (lane & 3);
        if (SHARED) return publish_rows(a, mine < rows, mine, row_rec[min(mine, rows - 1)]);
        return LeftRows();
    }
};

template <int D, bool PRECISE, bool SHARED>
__device__ __forceinline__ LeftRows resident_task(const Stage1Args &a, const int32_t *it, int h, unsigned char *s_raw) {
    using L = ResidentLds<D>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile0 = it[deft::kItTile0], ntiles = it[deft::kItNTiles];
    const int seg0 = it[deft::kItSeg0], nseg = it[deft::kItPieces];
    const int cqlo = it[deft::kItQlo], width = it[deft::kItWidth];
    const int slot_base = it[deft::kItSlotBase];
    float *lds = reinterpret_cast<float *>(s_raw);
    int32_t *row_q = reinterpret_cast<int32_t *>(lds + L::kRows), *row_pos = row_q + kTaskRows;
    uint32_t *row_out = reinterpret_cast<uint32_t *>(row_pos + kTaskRows), *row_rec = row_out + kTaskRows;
    int32_t *s_row = reinterpret_cast<int32_t *>(lds + L::kTokens), *s_qlo = s_row + kResidentTokens<D>,
            *s_qhi = s_qlo + kResidentTokens<D>;
    ChunkCtx c{};
    c.row_stride = (size_t)a.Hkv * D;
    c.s_row = s_row;
    c.s_qlo = s_qlo;
    c.s_qhi = s_qhi;
    c.clen = it[deft::kItLen];
    c.uniform = nseg == 1;
    c.begin0 = it[deft::kItBegin0];
    c.n16 = lane & 15;
    c.g = lane >> 4;
    const int nblk = (c.clen + 31) >> 5;
    const int rows = min(16 * ntiles, width * a.G - 16 * tile0);  // of this task
    const uint16_t *k_lane = a.k + (size_t)h * D + 8 * c.g, *v_lane = a.v + (size_t)h * D + (D / 16) * c.n16;
    const uint16_t *q_lane = a.q + 8 * c.g;

    // The rows of the task: where Q comes from and where the partial result goes (rows past the end repeat the last).
    // One thread per row; the query index is asked for here and waited for in finish_rows, behind the K/V loads.
    static_assert(kTaskRows <= 64 * kWaves, "one thread per row");
    const int rr = 16 * tile0 + min(tid, rows - 1);
    const int pl = divide(rr, a.G, a.inv_G), gh = rr - pl * a.G;
    const bool row_thread = tid < 16 * ntiles;
    int q_user = 0;
    if (row_thread) q_user = a.q_order[cqlo + pl];
    auto finish_rows = [&] {
        if (row_thread) {
            row_q[tid] = q_user * a.Hq + h * a.G + gh;
            row_pos[tid] = cqlo + pl;
            row_out[tid] = (uint32_t)(slot_base + pl) * (uint32_t)a.Hq + (uint32_t)(h * a.G + gh);
            if (SHARED) row_rec[tid] = (uint32_t)(h * a.n_slots + slot_base + pl) * (uint32_t)a.G + (uint32_t)gh;
        }
    };
    // the tokens: physical row and the interval of plan positions that see it (nobody, past the chunk's end)
    const int mine = (nblk - wave + kWaves - 1) / kWaves;  // blocks of this wave that exist,
    const int taken = mine <= 2 ? mine : kResidentBlocks<D>;  // and that it works on
    const int padded = 32 * kWaves * (nblk <= kWaves ? 1 : nblk <= 2 * kWaves ? 2 : kResidentBlocks<D>);
    const bool ragged = nseg > 1 || (c.clen & 31) || (nblk > 2 * kWaves && padded != c.clen);
    if (nseg > 1) {
        int32_t *p_off = reinterpret_cast<int32_t *>(s_raw), *p_beg = p_off + kResidentTokens<D>,
                *p_lo = p_beg + kResidentTokens<D>, *p_hi = p_lo + kResidentTokens<D>;
        const int flat0 = a.seg_off[seg0];
        for (int s = tid; s < nseg; s += 64 * kWaves) {
            p_off[s] = a.seg_off[seg0 + s] - flat0;
            p_beg[s] = a.seg_tok_begin[seg0 + s];
            p_lo[s] = a.seg_qlo[seg0 + s];
            p_hi[s] = a.seg_qhi[seg0 + s];
        }
        __syncthreads();
        for (int x = tid; x < padded; x += 64 * kWaves) {
            int lo = 0, hi = nseg - 1;  // largest s with p_off[s] <= x
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (p_off[mid] <= x) lo = mid; else hi = mid - 1;
            }
            const bool in = x < c.clen;
            s_row[x] = in ? p_beg[lo] + (x - p_off[lo]) : c.begin0;
            s_qlo[x] = in ? p_lo[lo] : 0;
            s_qhi[x] = in ? p_hi[lo] : 0;
        }
        finish_rows();
        __syncthreads();
    } else if (ragged) {
        for (int x = tid; x < padded; x += 64 * kWaves) {
            s_qlo[x] = 0;
            s_qhi[x] = x < c.clen ? INT32_MAX : 0;
        }
    }

    ResidentTask<D> T;
    LeftRows left;
    auto go = [&](auto na) {
        constexpr int NA = decltype(na)::value;
        typename ResidentTask<D>::vrow v[NA > 0 ? NA : 1][8];
        if constexpr (NA > 0) T.template load<NA>(v, c, k_lane, v_lane, wave);
        if (nseg == 1) {  // (the K/V loads needed no table: they are under way)
            finish_rows();
            __syncthreads();
        }
        // Does every row see every token of this wave's blocks?  Then nothing is masked.
        int vis_lo = INT32_MAX, vis_hi = 0, all = 1;
        if constexpr (NA > 0) {
            T.load_q(q_lane, row_q[c.n16]);
            if (ragged) {
                if (lane < 32) {
                    for (int b = 0; b < taken; ++b) {
                        const int x = 32 * (wave + kWaves * b) + lane;
                        if (s_qhi[x] > s_qlo[x]) vis_lo = min(vis_lo, s_qlo[x]);
                        vis_hi = max(vis_hi, s_qhi[x]);
                        all &= s_qlo[x] <= cqlo && s_qhi[x] >= cqlo + width;
                    }
                }
#pragma unroll
                for (int o = 16; o > 0; o >>= 1) {
                    vis_lo = min(vis_lo, __shfl_xor(vis_lo, o));
                    vis_hi = max(vis_hi, __shfl_xor(vis_hi, o));
                }
                vis_lo = __builtin_amdgcn_readfirstlane(vis_lo);
                vis_hi = __builtin_amdgcn_readfirstlane(vis_hi);
            }
            T.template interleave<NA>(v);
        }
        if (!__all(all))
            left = T.template run<NA, true, PRECISE, SHARED>(a, c, lds, wave, lane, ntiles, rows, q_lane, vis_lo, vis_hi);
        else
            left = T.template run<NA, false, PRECISE, SHARED>(a, c, lds, wave, lane, ntiles, rows, q_lane, vis_lo, vis_hi);
    };
    if (mine <= 0)
        go(std::integral_constant<int, 0>());
    else if (mine == 1)
        go(std::integral_constant<int, 1>());
    else if (D == 128 || mine == 2)
        go(std::integral_constant<int, 2>());
    else
        go(std::integral_constant<int, kResidentBlocks<D>>());
    return left;
}

// Stage 1: one workgroup of four waves per task = (chunk, KV head, up to 128 rows of the chunk's group).
// The rows are (query of the group) x (query head reading this KV head), tiled 16 at a time.  A task of
// 1, 2 or 3-4 tiles splits its rows over TR = 1, 2 or 4 waves and its tokens over the 4 / TR parts that
// remain: wave w works on tile w % TR and token part w / TR.  A task of 5-8 tiles gives every wave two
// tiles.  The parts' partial results are merged in LDS, so one (m, l, acc) triple per (chunk, row)
// reaches the workspace.
//
// PRECISE selects two-term softmax weights (see compute_block).
template <int D, bool PRECISE, bool SHARED>
__device__ __forceinline__ LeftRows streaming_task(const Stage1Args &a, const int32_t *it, int h, unsigned char *s_raw) {
    constexpr int KK = D / 32;  // k-steps of the Q.K^T contraction
    // The P.V product runs as 8 MFMAs per block (a lane loads 8 d of V per token).  With D = 64 lanes
    // n16 >= 8 repeat the loads of n16 - 8 and half of each product is discarded; that shape only occurs
    // in tiny, latency-bound cases.
    static_assert(D == 64 || D == 128, "head dimension");
    constexpr int OP = D + 4;  // padded row pitch (floats) of the merge buffer

    u32x4 *xbuf = reinterpret_cast<u32x4 *>(s_raw);                     // register exchange, kXbufBytes
    float *mO = reinterpret_cast<float *>(s_raw);                       // merge buffer, aliases the exchange
    float *mM = mO + kWaves * 16 * OP;
    float *mL = mM + kWaves * 16;
    int32_t *s_row = reinterpret_cast<int32_t *>(s_raw + kXbufBytes);   // per-token table
    int32_t *s_qlo = s_row + a.table_len;
    int32_t *s_qhi = s_qlo + a.table_len;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps the block loops on scalar branches
    const int n16 = lane & 15;
    const int g = lane >> 4;
    const int tile0 = it[deft::kItTile0], ntiles = it[deft::kItNTiles];
    const int seg0 = it[deft::kItSeg0], nseg = it[deft::kItPieces];
    const int cqlo = it[deft::kItQlo];
    const int R = it[deft::kItWidth] * a.G;
    const int slot_base = it[deft::kItSlotBase];
    const int clen = it[deft::kItLen];
    const int TR = ntiles <= 1 ? 1 : (ntiles == 2 ? 2 : 4);  // waves that split the rows; 4 / TR token parts

    ChunkCtx ctx;
    ctx.row_stride = (size_t)a.Hkv * D;
    ctx.kbase = a.k + (size_t)h * D + 8 * g;
    ctx.vbase = a.v + (size_t)h * D + 8 * (D == 128 ? n16 : (n16 & 7));
    ctx.khead = a.k + (size_t)h * D;
    ctx.vhead = a.v + (size_t)h * D;
    ctx.klane = 16u * g;
    ctx.vlane = 16u * (D == 128 ? n16 : (n16 & 7));
    ctx.s_row = s_row;
    ctx.s_qlo = s_qlo;
    ctx.s_qhi = s_qhi;
    ctx.clen = clen;
    ctx.uniform = (nseg == 1);
    ctx.begin0 = it[deft::kItBegin0];
    ctx.qlo0 = it[deft::kItSegQlo0];
    ctx.qhi0 = it[deft::kItSegQhi0];
    ctx.fresh = SHARED ? -1 : it[deft::kItFresh] - 1;  // (calls of few rows have no such tasks)
    ctx.n16 = n16;
    ctx.g = g;
    const int nblk = (clen + 31) >> 5;

    // ---- chunks made of several node pieces: per-token table (physical row, interval of plan
    //      positions that attend) expanded from the plan's segment table into LDS
    if (nseg > 1) {
        // the piece records are fetched with one thread per piece (one round trip for the whole chunk) and
        // parked in the exchange area, which is idle until the main loop; then one thread per token finds its
        // piece by bisection over the pieces' offsets
        int32_t *p_off = reinterpret_cast<int32_t *>(s_raw);
        int32_t *p_beg = p_off + DEFT_MAX_CHUNK;
        int32_t *p_lo = p_beg + DEFT_MAX_CHUNK;
        int32_t *p_hi = p_lo + DEFT_MAX_CHUNK;
        const int flat0 = a.seg_off[seg0];
        for (int s = tid; s < nseg; s += 64 * kWaves) {
            p_off[s] = a.seg_off[seg0 + s] - flat0;
            p_beg[s] = a.seg_tok_begin[seg0 + s];
            p_lo[s] = a.seg_qlo[seg0 + s];
            p_hi[s] = a.seg_qhi[seg0 + s];
        }
        __syncthreads();
        for (int x = tid; x < nblk * 32; x += 64 * kWaves) {
            if (x < clen) {
                int lo = 0, hi = nseg - 1;  // largest s with p_off[s] <= x
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (p_off[mid] <= x) lo = mid; else hi = mid - 1;
                }
                s_row[x] = p_beg[lo] + (x - p_off[lo]);
                s_qlo[x] = p_lo[lo];
                s_qhi[x] = p_hi[lo];
            } else {  // last block's padding: a real row, masked
                s_row[x] = ctx.begin0;
                s_qlo[x] = 0;
                s_qhi[x] = 0;
            }
        }
        __syncthreads();
    }

    // ---- this wave's rows: tile (wave % TR) of the task and, for tasks of more than four tiles, tile
    //      (wave % TR) + 4 as well.  Q is the B operand, resident for the whole chunk.  The query indices are
    //      fetched first, the first K/V blocks are put in flight while they travel, then Q itself is fetched;
    //      one full wait before the main loop leaves nothing but the block pipeline outstanding inside it.
    const int NTW = ntiles > 4 ? 2 : 1;  // tiles per wave
    TileState<D> ts[2];
    int q_user[2], q_head[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int tile = wave % TR + 4 * u;
        const int r = 16 * (tile0 + tile) + n16;
        const bool ok = (u < NTW) && (tile < ntiles) && (r < R);
        const int pl = divide(r, a.G, a.inv_G);
        q_head[u] = r - pl * a.G;
        ts[u].qpos = ok ? cqlo + pl : -1;
        q_user[u] = 0;
        if (ok) q_user[u] = a.q_order[cqlo + pl];
        ts[u].rs = RowState{0.f, -INFINITY, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) ts[u].o[cc] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto load_q = [&](int ntw) {
        const u32x4 z = {0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (u >= ntw) break;
            const uint16_t *qp = a.q + ((size_t)q_user[u] * a.Hq + (size_t)h * a.G + q_head[u]) * D + 8 * g;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
                ts[u].q[kk] = __builtin_bit_cast(bf16x8, ts[u].qpos >= 0 ? load16(qp + 32 * kk) : z);
        }
        __builtin_amdgcn_s_waitcnt(0);  // vmcnt(0) expcnt(0) lgkmcnt(0)
    };
    const float inv_cs = 1.0f / a.c;  // turns a reference in exponent units back into score units
    TileState<D>(&ts1)[1] = reinterpret_cast<TileState<D>(&)[1]>(ts);  // the one-tile paths use ts[0] only

    if (TR == 1) {
        SplitPipe<D> pipe;
        pipe.prime(ctx, wave, nblk);
        load_q(1);
        pipe.template run<PRECISE>(ctx, wave, nblk, ts1, a.c);
    } else if (TR == 2) {
        SharedPipe<D, 2, 1> pipe;
        pipe.prime(ctx, wave, nblk);
        load_q(1);
        pipe.template run<PRECISE>(ctx, xbuf, wave, lane, nblk, ts1, a.c, inv_cs);
    } else if (NTW == 1 && ctx.uniform) {
        WidePipe<D, 1, D == 128, 1> pipe;
        pipe.prime(ctx, wave, nblk);
        load_q(1);
        pipe.template run<PRECISE>(ctx, xbuf, wave, lane, nblk, ts1, a.c, inv_cs);
    } else if (NTW == 1) {
        WidePipe<D, 1, false, 1> pipe;
        pipe.prime(ctx, wave, nblk);
        load_q(1);
        pipe.template run<PRECISE>(ctx, xbuf, wave, lane, nblk, ts1, a.c, inv_cs);
    } else if (ctx.uniform) {
        WidePipe<D, 2, D == 128, 2> pipe;  // the fast addressing is written for four loads per K loader
        pipe.prime(ctx, wave, nblk);
        load_q(2);
        pipe.template run<PRECISE>(ctx, xbuf, wave, lane, nblk, ts, a.c, inv_cs);
    } else {
        WidePipe<D, 2, false, 2> pipe;
        pipe.prime(ctx, wave, nblk);
        load_q(2);
        pipe.template run<PRECISE>(ctx, xbuf, wave, lane, nblk, ts, a.c, inv_cs);
    }

    // ---- merge the token parts in LDS and write one partial result per (chunk, row):
    //      m = reference maximum of the raw scores, l = sum of exp, acc = un-normalised weighted values.
    //      One round per tile of the wave; the exchange buffer is dead by now and the merge buffer takes its place.
    constexpr int EPL = D / 16;  // floats of a row per lane when 16 lanes share a row
    const int NP = kWaves / TR;  // parts to merge per row
    const int rr = lane >> 4, dc = lane & 15;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (u >= NTW) break;
        const float l_tot = ts[u].rs.l[0];
        __syncthreads();
        if (g == 0) {
            mM[wave * 16 + n16] = ts[u].rs.m(inv_cs);
            mL[wave * 16 + n16] = l_tot;
        }
        if (D == 128 || g < 2) {
            // this lane owns d in [32g, 32g+32) of row n16: d = 32g + 8i + c'
            float *dst = mO + (wave * 16 + n16) * OP + 32 * g;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4 lo4 = {ts[u].o[0][i], ts[u].o[1][i], ts[u].o[2][i], ts[u].o[3][i]};
                const f32x4 hi4 = {ts[u].o[4][i], ts[u].o[5][i], ts[u].o[6][i], ts[u].o[7][i]};
                *reinterpret_cast<f32x4 *>(dst + 8 * i) = lo4;
                *reinterpret_cast<f32x4 *>(dst + 8 * i + 4) = hi4;
            }
        }
        __syncthreads();

        for (int ps = 0; ps < TR; ++ps) {
            const int gr = 4 * TR * wave + 4 * ps + rr;  // row among the tiles of this round: 16 * (wave % TR) + n
            const int wt = gr >> 4, n = gr & 15;
            const int tile = wt + 4 * u;
            const int r = 16 * (tile0 + tile) + n;
            if (tile >= ntiles || r >= R) continue;
            float M = -INFINITY;
            for (int sp = 0; sp < NP; ++sp) M = fmaxf(M, mM[(wt + TR * sp) * 16 + n]);
            const float m_use = (M == -INFINITY) ? 0.f : M;
            float L = 0.f;
            float o[EPL];
#pragma unroll
            for (int e = 0; e < EPL; ++e) o[e] = 0.f;
            for (int sp = 0; sp < NP; ++sp) {
                const int src = wt + TR * sp;
                const float w = __builtin_amdgcn_exp2f((mM[src * 16 + n] - m_use) * a.c);
                L += w * mL[src * 16 + n];
                const float *row = mO + (src * 16 + n) * OP + EPL * dc;
#pragma unroll
                for (int e = 0; e < EPL; e += 4) {
                    const f32x4 x = *reinterpret_cast<const f32x4 *>(row + e);
                    o[e] += w * x[0];
                    o[e + 1] += w * x[1];
                    o[e + 2] += w * x[2];
                    o[e + 3] += w * x[3];
                }
            }
            const int pl = divide(r, a.G, a.inv_G), gh = r - pl * a.G;
            const size_t ro = (size_t)(slot_base + pl) * a.Hq + (size_t)h * a.G + gh;
            if (dc == 0) {
                a.part_m[ro] = M;
                a.part_l[ro] = L;
                if (SHARED) store_record(a, ((size_t)h * a.n_slots + slot_base + pl) * a.G + gh, M, L);
            }
            float *dst = a.part_acc + ro * D + EPL * dc;
#pragma unroll
            for (int e = 0; e < EPL; e += 4) store_partial<SHARED>(dst + e, f32x4{o[e], o[e + 1], o[e + 2], o[e + 3]});
        }
    }
    if (SHARED) {  // this wave's rows: 4 * TR from 4 * TR * wave among the first tiles of the waves, as many among the second
        const int gr = 4 * TR * wave + (lane & 15), tile = (gr >> 4) + 4 * (lane >> 4), r = 16 * (tile0 + tile) + (gr & 15);
        const int pl = divide(r, a.G, a.inv_G);
        return publish_rows(a, (lane & 15) < 4 * TR && lane < 16 * NTW && tile < ntiles && r < R, r - 16 * tile0,
                            ((size_t)h * a.n_slots + slot_base + pl) * a.G + (r - pl * a.G));
    }
    return LeftRows();
}

// One launch for all tasks of a call: a second one would run behind the first, each on a part of the chip (sixteen
// sequences on both sides of 1024 tokens: 29.6 + 16.5 us in two launches, 29.9 us in one).  Plans whose tasks all want
// the same kind of weights, which is most of them, run a kernel that holds that kind alone.
enum Weights { kBf16 = 0, kTwoTerm = 1, kMixed = 2 };

// Which tasks take the resident path, by row tiles.  A resident task costs its loads and then a fixed time per tile (0.4 us
// for 128 tokens, 0.7 us for 256, two workgroups to a compute unit); a streaming task overlaps the two, but takes a step
// per 32 tokens (1.2 us and more where rows are looked up token by token, as in chunks of several pieces, and with d = 64,
// which has no fast addressing).  One piece and d = 128: up to three tiles; four tiles of 256 tokens on a full chip are
// 17.5 us streamed and 20.3 us resident, and seven tiles beside narrow tasks 20.9 and 23.9 us a call (32 queries x 4 heads
// over 7281 tokens).  (Three tiles streamed where they are most of a launch are 0.96 of the time over 256 trees, 0.88 to 1.09,
// but 1.20 to 1.34 times as far from 64 bits: a resident weight is rounded relative to the largest of its wave's tokens, a
// streaming one to that of the first block.)  Several pieces or d = 64: any number.  One such task among tasks of one piece is
// what its launch waits for (2977 tokens under 50 queries x 4 heads, 16 of 712 workgroups, 24.6 -> 22.2 us a call), d = 64 under
// 31 queries x 4 heads 21.0 -> 18.7; on launches of several rounds it is level: 952 workgroups 52.6 -> 51.3, 1696 78.3 -> 77.1,
// 704 37.4 -> 37.8, 896 38.5 -> 38.9, 3064 70.6 -> 70.4.
// (The limits are arguments of the kernel: as constants the compiler lays the kernel's registers out otherwise, and narrow
// streaming tasks take 2 to 8 % longer.)
template <int D>
__device__ __forceinline__ bool is_resident(const Stage1Args &a, const int32_t *it) {
    return it[deft::kItLen] <= kResidentTokens<D> &&
           it[deft::kItNTiles] <= (D == 128 && it[deft::kItPieces] == 1 ? a.resident_one : a.resident_many);
}

template <int D, bool PRECISE, bool SHARED>
__device__ __forceinline__ LeftRows run_task(const Stage1Args &a, const int32_t *it, int h, unsigned char *s_raw) {
    return is_resident<D>(a, it) ? resident_task<D, PRECISE, SHARED>(a, it, h, s_raw) : streaming_task<D, PRECISE, SHARED>(a, it, h, s_raw);
}

// A run of several chunks with the same queries leaves its result in the slots of the first and marks those of the others
// empty, m = -inf and l = 0, so that stage 2 finds the same sum whether it reads the run's slots or the plan's.
__device__ __forceinline__ void mark_empty(const Stage1Args &a, const int32_t *it, int h) {
    static_assert(kTaskRows <= 64 * kWaves, "one thread per row");
    const int width = it[deft::kItWidth], r = 16 * it[deft::kItTile0] + threadIdx.x;
    if (threadIdx.x >= 16 * it[deft::kItNTiles] || r >= width * a.G) return;
    const int pl = divide(r, a.G, a.inv_G), gh = r - pl * a.G;
    for (int k = 1; k < it[deft::kItChunks]; ++k) {
        const size_t ro = (size_t)(it[deft::kItSlotBase] + k * width + pl) * a.Hq + (size_t)h * a.G + gh;
        a.part_m[ro] = -INFINITY;
        a.part_l[ro] = 0.f;
    }
}

// Stage 2: tree-topology-aware global reduction (eq. 1 with the largest maximum subtracted), D/4 lanes to a row of a
// partial result (128-bit loads), 64 / (D/4) rows at a time.  Bound by latency: the query's record, then m, l and rows.
template <int D>
struct Stage2Row {
    static constexpr int kLanes = D / 4;         // lanes per partial row
    static constexpr int kRows = 64 / kLanes;    // rows per load of a wave
    static constexpr int kBatch = 8 * kRows;     // rows a wave keeps in flight in registers
};

// Maximum and sum over the wave, in every lane: within rows of 16 lanes by moves inside the vector unit (lane ^ 1, lane ^ 2,
// then the halves of a row and the row itself mirrored, whose quads hold one value by then), across rows by swaps.  Six
// exchanges through the LDS hardware, one after the other, take 0.3 us each time.
template <int CTRL>
__device__ __forceinline__ float row_move(float x) {
    const int u = __builtin_bit_cast(int, x);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(u, u, CTRL, 0xf, 0xf, false));
}
template <typename Op>
__device__ __forceinline__ float wave_all(float x, Op op) {
    x = op(x, row_move<0xb1>(x));   // quad_perm 1 0 3 2
    x = op(x, row_move<0x4e>(x));   // quad_perm 2 3 0 1
    x = op(x, row_move<0x141>(x));  // row_half_mirror
    x = op(x, row_move<0x140>(x));  // row_mirror
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t a0 = a[0], a1 = a[1];
    const uint32_t w = __builtin_bit_cast(uint32_t, op(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1)));
    const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    const uint32_t b0 = b[0], b1 = b[1];
    return op(__builtin_bit_cast(float, b0), __builtin_bit_cast(float, b1));
}
__device__ __forceinline__ float wave_max(float x) {
    return wave_all(x, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float wave_sum(float x) {
    return wave_all(x, [](float a, float b) { return a + b; });
}

// HOLES: some slots of the list may have been marked empty by a whole call (m = -inf, l = 0).  Their rows of acc were not
// written, so they are dropped and not multiplied by 0; in the place of a weight, which is never negative, such a slot has
// kNoSlot.  A whole call's own list has no such slots, and does without the selection, which costs it 0.3 us.
constexpr float kNoSlot = -1.f;
template <bool HOLES>
__device__ __forceinline__ float row_weight(float w, float m, float l) {
    return HOLES && m == -INFINITY && l == 0.f ? kNoSlot : w;
}
template <bool HOLES>
__device__ __forceinline__ void add_row(f32x4 &acc, float w, const f32x4 &x) {
    if (HOLES && w == kNoSlot) return;
    acc += w * x;
}

__device__ __forceinline__ void store_out(const Stage2Args &a, size_t at, f32x4 x) {
    if (a.out_f32) {
        *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(a.out) + at) = x;
    } else {
        typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
        u32x2 pk = {pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
        *reinterpret_cast<u32x2 *>(reinterpret_cast<uint16_t *>(a.out) + at) = pk;
    }
}

// Every query of the plan has at most kBatch partials: a wave per (query, query head).  The slot ids come with the
// record, so m, l and every row are fetched in the next round trip and the weights are applied to rows that are already
// in registers.  One wave to a workgroup: four cost 0.4 us more on every tree, and two or four heads to a wave gain
// only where there are thousands (0.2 us of 6.3 at 8192).
template <int D, bool HOLES>
__global__ __launch_bounds__(64) void deft_stage2_few(const int32_t *q_head, uint32_t Hq, uint32_t inv_Hq, uint32_t head_ints,
                                                      Stage2Args a) {
    using R = Stage2Row<D>;
    const int lane = threadIdx.x;
    const int p = divide(blockIdx.x, Hq, inv_Hq), qh = blockIdx.x - p * Hq;
    const int rec = q_head[(size_t)p * head_ints + (lane & (deft::kQueryHeadInts - 1))];
    const int n = __builtin_amdgcn_readlane(rec, 0), q_user = __builtin_amdgcn_readlane(rec, 1);
    const int sub = lane / R::kLanes, col = lane - sub * R::kLanes;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float lsum = 0.f;
    if (n > 0) {
        // lanes past the end hold a slot that exists
        const int slot = __shfl(rec, deft::kQueryHeadFixed + (lane < n ? lane : 0));
        const size_t ro = (size_t)slot * a.Hq + qh;
        const float mj = lane < n ? a.part_m[ro] : -INFINITY;
        const float lj = lane < n ? a.part_l[ro] : 0.f;
        f32x4 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int sj = __shfl(slot, u * R::kRows + sub);
            x[u] = *reinterpret_cast<const f32x4 *>(a.part_acc + ((size_t)sj * a.Hq + qh) * D + 4 * col);
        }
        const float mx = wave_max(mj);
        const float w = (lane < n && mx != -INFINITY) ? __builtin_amdgcn_exp2f((mj - mx) * a.c) : 0.f;
        lsum = wave_sum(w * lj);
        const float wr = row_weight<HOLES>(w, mj, lj);
#pragma unroll
        for (int u = 0; u < 8; ++u) add_row<HOLES>(acc, __shfl(wr, u * R::kRows + sub), x[u]);
    }
#pragma unroll
    for (int o = 32; o >= R::kLanes; o >>= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], o);
    if (sub == 0) store_out(a, ((size_t)q_user * a.Hq + qh) * D + 4 * col, acc * (lsum > 0.f ? 1.f / lsum : 0.f));
}

// Any number of partials: one, two or four waves per (query, query head), partial WAVES * i + w with wave w.  Each wave
// merges what it holds as above (64 of its partials at a time, on a running maximum), then their results are merged in LDS.
template <int D, int WAVES, bool HOLES>
__global__ __launch_bounds__(64 * WAVES) void deft_stage2_many(const int32_t *q_head, uint32_t Hq, uint32_t inv_Hq, uint32_t head_ints,
                                                               Stage2Args a) {
    using R = Stage2Row<D>;
    __shared__ __attribute__((aligned(16))) float s_acc[WAVES][D];
    __shared__ float s_m[WAVES], s_l[WAVES];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p = divide(blockIdx.x, Hq, inv_Hq), qh = blockIdx.x - p * Hq;
    const int32_t *rec = q_head + (size_t)p * head_ints;
    int slot = rec[min(deft::kQueryHeadFixed + WAVES * lane + wave, (int)head_ints - 1)];
    const int n = rec[0], q_user = rec[1], s0 = rec[2];
    const int sub = lane / R::kLanes, col = lane - sub * R::kLanes;
    const int mine = (n - wave + WAVES - 1) / WAVES;  // partials of this wave
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float M = -INFINITY, lsum = 0.f;
    for (int base = 0; base < mine; base += 64) {
        const int cnt = min(64, mine - base);
        if (n > (int)head_ints - deft::kQueryHeadFixed)
            slot = a.q_part_slot[s0 + WAVES * (base + min(lane, cnt - 1)) + wave];
        else if (WAVES == 1 && base > 0)  // (two waves or four find all of theirs in the first 64)
            slot = rec[deft::kQueryHeadFixed + base + min(lane, cnt - 1)];
        slot = __shfl(slot, min(lane, cnt - 1));  // lanes past the end hold a slot that exists
        const size_t ro = (size_t)slot * a.Hq + qh;
        const float mj = lane < cnt ? a.part_m[ro] : -INFINITY;
        const float lj = lane < cnt ? a.part_l[ro] : 0.f;
        float w = 0.f;
        for (int j = 0; j < cnt; j += R::kBatch) {
            f32x4 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int sj = __shfl(slot, (j + u * R::kRows + sub) & 63);
                x[u] = *reinterpret_cast<const f32x4 *>(a.part_acc + ((size_t)sj * a.Hq + qh) * D + 4 * col);
            }
            if (j == 0) {
                const float top = fmaxf(M, wave_max(mj));
                const float old = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((M - top) * a.c);
                w = (lane < cnt && top != -INFINITY) ? __builtin_amdgcn_exp2f((mj - top) * a.c) : 0.f;
                lsum = lsum * old + wave_sum(w * lj);
                w = row_weight<HOLES>(w, mj, lj);
                acc *= old;
                M = top;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                add_row<HOLES>(acc, __shfl(w, (j + u * R::kRows + sub) & 63), x[u]);  // weight 0 for rows past the end
            }
        }
    }
#pragma unroll
    for (int o = 32; o >= R::kLanes; o >>= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], o);
    if (sub == 0) *reinterpret_cast<f32x4 *>(&s_acc[wave][4 * col]) = acc;
    if (lane == 0) {
        s_m[wave] = M;
        s_l[wave] = lsum;
    }
    __syncthreads();
    if (wave != 0 || sub != 0) return;
    float top = -INFINITY, total = 0.f;
#pragma unroll
    for (int k = 0; k < WAVES; ++k) top = fmaxf(top, s_m[k]);
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < WAVES; ++k) {
        const float w = top == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((s_m[k] - top) * a.c);
        total += w * s_l[k];
        sum += w * *reinterpret_cast<const f32x4 *>(&s_acc[k][4 * col]);
    }
    store_out(a, ((size_t)q_user * a.Hq + qh) * D + 4 * col, sum * (total > 0.f ? 1.f / total : 0.f));
}

// Stage 2 of a whole call in one launch, at the end of the grid: a wave takes every (kWaves * groups)th row of the output and
// waits for its partial results, kMarkPolls looks at most, about a millisecond.  Workgroups are started in the order of their
// ids, on each XCD for itself, so as a rule what is waited for runs already; but other calls and other work may hold the
// places that stage 1 needs, for any time.  A wave that has waited in vain leaves the row to stage 1: it puts the ticket's
// complement into one of the marks that are still missing, and goes.  The wave of stage 1 that finds it there when it puts its
// ticket in has the row from then on: it leaves it to another in the same way, or, if nothing is missing any more, merges it.
// One wave at a time has a row, so each is merged once.  No result depends on how long anything takes, every wait ends,
// and the at most kReduceGroups workgroups that wait give their places back.
constexpr int kMarkPolls = 1 << 10;
constexpr uint32_t kReduceGroups = 8;
constexpr int kReduceLoads = 16;  // loads of a wave in flight, each of 16 bytes a lane: 32 partial results at d = 128, 64 at d = 64

// Plan query p, query head qh: the list of its partial results.
struct RowParts {
    const CallArgs &call;
    const int32_t *rec;
    int n, q_user, s0, qh, kvh, lane, first;  // first: slot of partial result `lane`, where the record holds one
    __device__ __forceinline__ RowParts(const CallArgs &c, int p, int head, int l) : call(c), qh(head), lane(l) {
        rec = c.s2.q_head + (size_t)p * c.s2.head_ints;
        first = rec[min(deft::kQueryHeadFixed + lane, c.s2.head_ints - 1)];
        n = rec[0], q_user = rec[1], s0 = rec[2];
        kvh = divide(qh, c.s1.G, c.s1.inv_G);
    }
    // of partial results base .. base + cnt - 1, one to a lane; lanes past the end hold the last
    __device__ __forceinline__ int slot(int base, int cnt) const {
        int x = first;
        if (n > call.s2.head_ints - deft::kQueryHeadFixed)
            x = call.s2.q_part_slot[s0 + base + min(lane, cnt - 1)];
        else if (base > 0)
            x = rec[deft::kQueryHeadFixed + base + min(lane, cnt - 1)];
        return __shfl(x, min(lane, cnt - 1));
    }
    __device__ __forceinline__ float *record(int slot) const {
        return call.s1.marks + 4 * (((size_t)kvh * call.s1.n_slots + slot) * call.s1.G + (qh - kvh * call.s1.G));
    }
    // Whether all are there, looking at most `polls` times.
    __device__ __forceinline__ bool complete(int polls) const {
        for (int base = 0; base < n; base += 64) {
            uint64_t *mark = mark_of(record(slot(base, min(64, n - base))));
            for (bool there = false;; __builtin_amdgcn_s_sleep(2)) {
                if (!there) there = __hip_atomic_load(mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == call.s1.ticket;
                if (__all(there)) break;
                if (--polls <= 0) return false;
            }
        }
        asm volatile("" ::: "memory");
        return true;
    }
    // Leaves the row to a wave that writes one of the missing partial results.  False: left; true: nothing is missing.
    __device__ __forceinline__ bool leave() const {
        const uint64_t ticket = call.s1.ticket;
        for (int base = 0; base < n; base += 64) {
            uint64_t *mark = mark_of(record(slot(base, min(64, n - base))));
            for (;;) {
                uint64_t seen = __hip_atomic_load(mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint64_t missing = __ballot(seen != ticket);
                if (!missing) break;
                bool left = false;  // (it fails where the ticket has come meanwhile)
                if (lane == __builtin_ctzll(missing))
                    left = __hip_atomic_compare_exchange_strong(mark, &seen, ~ticket, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__any(left)) return false;
            }
        }
        asm volatile("" ::: "memory");
        return true;
    }
};

// Merges a row whose partial results are all there.
template <int D>
__device__ __forceinline__ void merge_row(const RowParts &row) {
    using R = Stage2Row<D>;
    constexpr int kLoads = kReduceLoads;
    const CallArgs &call = row.call;
    const Stage2Args &a = call.s2;
    const int lane = row.lane, n = row.n, qh = row.qh;
    const int sub = lane / R::kLanes, col = lane - sub * R::kLanes;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float M = -INFINITY, lsum = 0.f;
    for (int base = 0; base < n; base += 64) {
        const int cnt = min(64, n - base);
        const int slot = row.slot(base, cnt);
        float *record = row.record(slot);
        f32x2 ml = {-INFINITY, 0.f};
        if (lane < cnt)
            ml = __builtin_bit_cast(f32x2, __hip_atomic_load(reinterpret_cast<uint64_t *>(record), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const float mj = ml[0], lj = ml[1];
        float w = 0.f;
        for (int j = 0; j < cnt; j += kLoads * R::kRows) {
            f32x4 x[kLoads];
            auto load = [&](int u) {
                const int sj = __shfl(slot, (j + u * R::kRows + sub) & 63);
                x[u] = load_shared4(a.part_acc + ((size_t)sj * a.Hq + qh) * D + 4 * col);
            };
            const bool half = cnt - j <= kLoads / 2 * R::kRows;
#pragma unroll
            for (int u = 0; u < kLoads / 2; ++u) load(u);
            if (!half) {
#pragma unroll
                for (int u = kLoads / 2; u < kLoads; ++u) load(u);
            }
            if (j == 0) {
                const float top = fmaxf(M, wave_max(mj));
                const float old = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((M - top) * a.c);
                w = (lane < cnt && top != -INFINITY) ? __builtin_amdgcn_exp2f((mj - top) * a.c) : 0.f;
                lsum = lsum * old + wave_sum(w * lj);
                acc *= old;
                M = top;
            }
            auto add = [&](int u) {  // (rows past the end repeat the last one, which may hold infinities: no weight of 0 for them)
                const int r = j + u * R::kRows + sub;
                const float wr = __shfl(w, r & 63);
                if (r < cnt) acc += wr * x[u];
            };
#pragma unroll
            for (int u = 0; u < kLoads / 2; ++u) add(u);
            if (!half) {
#pragma unroll
                for (int u = kLoads / 2; u < kLoads; ++u) add(u);
            }
        }
    }
#pragma unroll
    for (int o = 32; o >= R::kLanes; o >>= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], o);
    if (sub == 0) store_out(a, ((size_t)row.q_user * a.Hq + qh) * D + 4 * col, acc * (lsum > 0.f ? 1.f / lsum : 0.f));
}

// Stage 2's waves.
template <int D>
__device__ __forceinline__ void reduce_rows(const CallArgs &call, uint32_t group, uint32_t groups) {
    const Stage2Args &a = call.s2;
    const uint32_t rows = (uint32_t)a.nq * (uint32_t)a.Hq, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (uint32_t r = kWaves * group + wave; r < rows; r += kWaves * groups) {
        const int p = divide(r, a.Hq, a.inv_Hq);
        const RowParts row(call, p, r - p * a.Hq, threadIdx.x & 63);
        if (row.complete(call.polls) || row.leave()) merge_row<D>(row);
    }
}

// A wave of stage 1 to which rows of its task were left.
template <int D>
__device__ __forceinline__ void merge_left_rows(const CallArgs &call, const int32_t *it, int h, const LeftRows &x) {
    const int G = call.s1.G, first = 16 * it[deft::kItTile0];
    for (uint64_t left = __ballot(x.left); left; left &= left - 1) {
        const int r = first + __builtin_amdgcn_readlane(x.row, __builtin_ctzll(left)), pl = divide(r, G, call.s1.inv_G);
        const RowParts row(call, it[deft::kItQlo] + pl, h * G + r - pl * G, threadIdx.x & 63);
        if (row.leave()) merge_row<D>(row);
    }
}

// SHARED: a whole call in one launch, stage 2 included.
//   items   deft::kItemInts int32 per work item, see deft_internal.h
//   tasks   workgroups of stage 1
template <int D, int WEIGHTS, bool SHARED>
__global__ __launch_bounds__(64 * kWaves, 2) void deft_stage1(const int32_t *items, uint32_t Hkv, uint32_t inv_Hkv, uint32_t tasks, CallArgs call) {
    extern __shared__ __attribute__((aligned(16))) unsigned char s_raw[];
    if (SHARED && blockIdx.x >= tasks) {
        reduce_rows<D>(call, blockIdx.x - tasks, gridDim.x - tasks);
        return;
    }
    const Stage1Args &a = call.s1;
    const int item = divide(blockIdx.x, Hkv, inv_Hkv);
    // KV head of this workgroup.  Workgroups b and b + 256 land on the same compute unit (the dispatcher goes
    // round the 256 units), and with Hkv dividing 256 they would stream the same head: K and V rows whose
    // addresses agree in bits 7..12.  A unit whose streams all share those bits reads measurably slower (its
    // L1 keeps fewer lines in flight), so every further round of 256 workgroups is moved on by one head.
    // The shift depends on the task only, so a task still visits every head exactly once.
    const uint32_t turned = blockIdx.x - item * Hkv + ((uint32_t)(item * Hkv) >> 8);
    const int h = turned - divide(turned, Hkv, inv_Hkv) * Hkv;
    const int32_t *it = items + (size_t)item * deft::kItemInts;
    if (it[deft::kItChunks] > 1) mark_empty(a, it, h);  // (first: behind the task its descriptor would have to be read again)
    const LeftRows left = WEIGHTS == kTwoTerm || (WEIGHTS == kMixed && it[deft::kItPrecise]) ? run_task<D, true, SHARED>(a, it, h, s_raw)
                                                                                              : run_task<D, false, SHARED>(a, it, h, s_raw);
    if (SHARED && __any(left.left)) merge_left_rows<D>(call, it, h, left);
}

// Plain read of a buffer with 128-bit loads, every byte once, all compute units busy: the rate this
// reaches is the practical ceiling for a kernel whose job is to read HBM (Section 3.3's premise is that
// the KV read dominates).  Workgroup b leaves the xor of the words it read in sink[b], so that no load
// can be dropped and a caller can check that every word was read exactly once.
constexpr int kProbeGroups = DEFT_PROBE_SINK_BYTES / 4;

__global__ __launch_bounds__(256) void deft_read_probe(const u32x4 *__restrict__ p, size_t n16, uint32_t *sink) {
    __shared__ uint32_t part[4];
    size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const size_t stride = size_t(gridDim.x) * blockDim.x;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (; i < n16; i += stride) acc ^= p[i];
    uint32_t x = acc[0] ^ acc[1] ^ acc[2] ^ acc[3];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x ^= __shfl_xor(x, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) sink[blockIdx.x] = part[0] ^ part[1] ^ part[2] ^ part[3];
}

// A plan's image from pinned host memory into its buffer, one 16-byte word to a thread.  A kernel and not a copy command:
// copies run on an engine of their own, and the compute queue waits some 35 us for it to be told, to copy and to answer.
// Bound by the latency of host memory: 3.4 us for 24 KB.  Decode iteration of 8 layer-calls 166 us with a copy, 147 with the
// kernel.
constexpr int kFetchThreads = 1024;
__global__ __launch_bounds__(kFetchThreads) void deft_fetch_image(const u32x4 *host, u32x4 *image, uint32_t words) {
    const uint32_t i = blockIdx.x * kFetchThreads + threadIdx.x;
    if (i < words) {
        // system scope: no line of an earlier image may be found in a cache
        const u32x4 x = __builtin_amdgcn_global_load_b128((global_u32x4)(host + i), "");
        image[i] = x;
    }
}

// A part of a plan's image that is the kernel's own argument: in a stream that is being captured, what the replays read has
// to live as long as the graph does, and arguments are the one thing that a graph keeps (4 KB of them to a kernel).
constexpr int kPartWords = 224;
struct ImagePart {
    u32x4 word[kPartWords];
};
__global__ __launch_bounds__(256) void deft_store_part(u32x4 *image, uint32_t words, ImagePart part) {
    static_assert(kPartWords <= 256, "a word to a thread");
    if (threadIdx.x < words) image[threadIdx.x] = part.word[threadIdx.x];
}

thread_local std::string g_hip_error;

bool hip_ok(hipError_t e, const char *what) {
    if (e == hipSuccess) return true;
    g_hip_error = std::string(what) + ": " + hipGetErrorString(e);
    return false;
}

// The kernels may use more than the default 64 KB of dynamic LDS: the limit of all variants is raised once
// per device, at the first call that launches one of them.
template <int D>
bool configure_stage1() {
    static std::atomic<uint64_t> configured;  // bit i set: done on device i (one flag per head dimension)
    int dev = 0;
    if (!hip_ok(hipGetDevice(&dev), "hipGetDevice")) return false;
    if (dev >= 0 && dev < 64 && ((configured.load(std::memory_order_acquire) >> dev) & 1)) return true;
    const int bytes = kXbufBytes + 3 * DEFT_MAX_CHUNK * (int)sizeof(int32_t);
    static_assert(ResidentLds<D>::kWords * 4 <= kXbufBytes + 3 * DEFT_MAX_CHUNK * (int)sizeof(int32_t), "LDS limit");
    for (const void *f : {reinterpret_cast<const void *>(&deft_stage1<D, kBf16, false>),
                          reinterpret_cast<const void *>(&deft_stage1<D, kTwoTerm, false>),
                          reinterpret_cast<const void *>(&deft_stage1<D, kMixed, false>),
                          reinterpret_cast<const void *>(&deft_stage1<D, kBf16, true>),
                          reinterpret_cast<const void *>(&deft_stage1<D, kTwoTerm, true>),
                          reinterpret_cast<const void *>(&deft_stage1<D, kMixed, true>)})
        if (!hip_ok(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes), "deft_stage1 LDS size")) return false;
    if (dev >= 0 && dev < 64) configured.fetch_or(1ull << dev, std::memory_order_release);
    return true;
}

template <int D, bool SHARED>
bool launch_stage1(const deft::TaskSet &T, CallArgs a, unsigned reduce_groups, const uint8_t *image, hipStream_t stream) {
    if (T.n_items == 0) return true;
    if (!configure_stage1<D>()) return false;
    Stage1Args &a1 = a.s1;
    const int32_t *items = reinterpret_cast<const int32_t *>(image + T.off_items);
    a1.n_items = T.n_items;
    a1.resident_one = deft::kResidentTiles;
    a1.resident_many = deft::kMaxTilesPerTask;
    const size_t lds = std::max(kXbufBytes + 3 * (size_t)a1.table_len * sizeof(int32_t), (size_t)ResidentLds<D>::kWords * 4);
    const uint32_t Hkv = (uint32_t)a1.Hkv, tasks = (uint32_t)T.n_items * Hkv;
    auto *kernel = T.n_items_precise == 0           ? &deft_stage1<D, kBf16, SHARED>
                   : T.n_items_precise == T.n_items ? &deft_stage1<D, kTwoTerm, SHARED>
                                                    : &deft_stage1<D, kMixed, SHARED>;
    hipLaunchKernelGGL(kernel, dim3(tasks + reduce_groups), dim3(64 * kWaves), lds, stream, items, Hkv, inverse(Hkv), tasks, a);
    return hip_ok(hipGetLastError(), "deft_stage1 launch");
}

template <int D, bool HOLES>
bool launch_stage2(const deft::TaskSet &T, const Stage2Args &a2, hipStream_t stream) {
    if (a2.nq == 0) return true;
    const unsigned rows = (unsigned)a2.nq * (unsigned)a2.Hq;
    const uint32_t Hq = (uint32_t)a2.Hq, ints = (uint32_t)a2.head_ints;
    constexpr int kFew = std::min(Stage2Row<D>::kBatch, deft::kQueryHeadInts - deft::kQueryHeadFixed);
    // Up to kFew partials one wave has them all in flight at once, and more waves cost more to start than they save (16
    // partials, 2048 rows of output: 5.1 us, four waves 7.5).  Beyond that a second batch is a round trip more, which a
    // few rows have the chip to take apart and many do not: the waves of rows with few partials are in the way.  Whole
    // call, us, with one, two and four waves: 32 rows of 64 partials 13.8, 13.0, 12.6; 128 rows, one query in four of 128,
    // 25.4, 24.6, 24.2; 960 of 65 43.9, 43.4, 43.6; 2048 of 32 33.8, 33.5, 35.0; 2048, one query in 64 of 128, 38.9, 38.2,
    // 40.1; 8192, one in 256 of 128, 55.5, 59.1, 65.0.  (One wave to a row beyond 2048 of
    // them also keeps launches of up to 2^26 rows within the 32 bits of grid x block.)
    if (T.max_parts <= kFew)
        hipLaunchKernelGGL((deft_stage2_few<D, HOLES>), dim3(rows), dim3(64), 0, stream, a2.q_head, Hq, a2.inv_Hq, ints, a2);
    else if (rows > 2048)
        hipLaunchKernelGGL((deft_stage2_many<D, 1, HOLES>), dim3(rows), dim3(64), 0, stream, a2.q_head, Hq, a2.inv_Hq, ints, a2);
    else if (rows > 1024 || T.max_parts <= 2 * 16)
        hipLaunchKernelGGL((deft_stage2_many<D, 2, HOLES>), dim3(rows), dim3(128), 0, stream, a2.q_head, Hq, a2.inv_Hq, ints, a2);
    else
        hipLaunchKernelGGL((deft_stage2_many<D, 4, HOLES>), dim3(rows), dim3(256), 0, stream, a2.q_head, Hq, a2.inv_Hq, ints, a2);
    return hip_ok(hipGetLastError(), "deft_stage2 launch");
}

// Everything the two stages share: argument checks, the schedule, the workspace carve-up.
struct Call {
    const deft::Schedule *S = nullptr;
    const uint8_t *img = nullptr;
    float *acc = nullptr, *pm = nullptr, *pl = nullptr;
    float *marks = nullptr;  // null: the workspace has no room for them
    float c = 0.f;
    hipStream_t stream = nullptr;
};

// The tasks of a whole call.  Chunks are cut anew into as many runs as the KV heads of the first upload ask for; with fewer heads
// they would leave most of the chip idle (12345 tokens under 26 queries x 4 heads, uploaded for 32 KV heads and called with two:
// 22 workgroups, 98 as planned).
const deft::TaskSet &whole_call(const Call &call, int32_t Hkv, int32_t d) {
    return d == 128 && Hkv == call.S->Hkv && call.S->recut.n_items > 0 ? call.S->recut : call.S->fused;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

int prepare(const deft_plan_t *plan, const void *dev_image, int32_t Hq, int32_t Hkv, int32_t d, float scale,
            void *workspace, size_t workspace_bytes, void *stream, Call &call) {
    if (!plan || !dev_image || !workspace) return DEFT_EINVAL;
    if (Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0 || (d != 64 && d != 128)) return DEFT_EINVAL;
    if (!aligned16(workspace) || !aligned16(dev_image)) return DEFT_EINVAL;
    call.S = deft::find_schedule(plan, Hq / Hkv);
    if (!call.S) return DEFT_ENOTREADY;
    if (workspace_bytes < deft::partials_bytes(plan, Hq, d)) return DEFT_EWORKSPACE;
    const int32_t most = std::max(call.S->by_chunk.n_items, whole_call(call, Hkv, d).n_items);
    if ((int64_t)most * Hkv > INT32_MAX) return DEFT_EINVAL;  // grid sizes are 32-bit
    if ((int64_t)plan->nq * Hq > INT32_MAX) return DEFT_EINVAL;
    const size_t rows = (size_t)plan->n_slots() * (size_t)Hq;
    call.img = static_cast<const uint8_t *>(dev_image);
    call.acc = static_cast<float *>(workspace);
    call.pm = call.acc + rows * (size_t)d;
    call.pl = call.pm + rows;
    call.marks = workspace_bytes < deft::workspace_bytes(plan, Hq, d) ? nullptr : call.pm + (2 * rows + 3) / 4 * 4;
    if (!(scale > 0.f)) scale = 1.0f / std::sqrt((float)d);
    call.c = scale * 1.4426950408889634f;  // log2(e)
    call.stream = reinterpret_cast<hipStream_t>(stream);
    return DEFT_OK;
}

void stage1_args(const Call &call, const void *q, const void *k, const void *v, int32_t Hq, int32_t Hkv, Stage1Args &a1) {
    const deft::Schedule &S = *call.S;
    auto at = [&](size_t off) { return reinterpret_cast<const int32_t *>(call.img + off); };
    a1.q = static_cast<const uint16_t *>(q);
    a1.k = static_cast<const uint16_t *>(k);
    a1.v = static_cast<const uint16_t *>(v);
    a1.part_acc = call.acc;
    a1.part_m = call.pm;
    a1.part_l = call.pl;
    a1.seg_tok_begin = at(S.off_seg_tok_begin);
    a1.seg_len = at(S.off_seg_len);
    a1.seg_qlo = at(S.off_seg_qlo);
    a1.seg_qhi = at(S.off_seg_qhi);
    a1.seg_off = at(S.off_seg_off);
    a1.q_order = at(S.off_q_order);
    a1.Hq = Hq;
    a1.Hkv = Hkv;
    a1.G = Hq / Hkv;
    a1.inv_G = inverse(a1.G);
    a1.table_len = S.table_len;
    a1.c = call.c;
}

void stage2_args(const deft_plan_t *plan, const Call &call, const deft::TaskSet &T, void *o, int32_t Hq, uint32_t flags, Stage2Args &a2) {
    auto at = [&](size_t off) { return reinterpret_cast<const int32_t *>(call.img + off); };
    a2.part_acc = call.acc;
    a2.part_m = call.pm;
    a2.part_l = call.pl;
    a2.q_head = at(T.off_q_head);
    a2.q_part_slot = at(T.off_q_part_slot);
    a2.out = o;
    a2.nq = plan->nq;
    a2.Hq = Hq;
    a2.head_ints = T.head_ints;
    a2.inv_Hq = inverse(Hq);
    a2.out_f32 = (flags == DEFT_OUT_F32);
    a2.c = call.c;
}

bool stage1_inputs_ok(const void *q, const void *k, const void *v) {
    return q && k && v && aligned16(q) && aligned16(k) && aligned16(v);
}

int run_stage1(const deft_plan_t *plan, const Call &call, const deft::TaskSet &T, const void *q, const void *k, const void *v, int32_t Hq,
               int32_t Hkv, int32_t d) {
    if (plan->n_chunks() == 0) return DEFT_OK;
    if (!stage1_inputs_ok(q, k, v)) return DEFT_EINVAL;
    CallArgs a{};
    stage1_args(call, q, k, v, Hq, Hkv, a.s1);
    const bool ok = d == 128 ? launch_stage1<128, false>(T, a, 0, call.img, call.stream)
                             : launch_stage1<64, false>(T, a, 0, call.img, call.stream);
    return ok ? DEFT_OK : DEFT_EHIP;
}

int run_stage2(const deft_plan_t *plan, const Call &call, const deft::TaskSet &T, void *o, int32_t Hq, int32_t d, uint32_t flags) {
    if (flags != DEFT_OUT_BF16 && flags != DEFT_OUT_F32) return DEFT_EINVAL;
    if (plan->nq == 0) return DEFT_OK;
    if (!o || !aligned16(o)) return DEFT_EINVAL;
    Stage2Args a2{};
    stage2_args(plan, call, T, o, Hq, flags, a2);
    // a stage 2 called apart may find slots that a whole call left empty
    const bool holes = &T == &call.S->by_chunk && whole_call(call, Hq / call.S->group, d).off_items != T.off_items;
    const bool ok = d == 128 ? (holes ? launch_stage2<128, true>(T, a2, call.stream) : launch_stage2<128, false>(T, a2, call.stream))
                             : (holes ? launch_stage2<64, true>(T, a2, call.stream) : launch_stage2<64, false>(T, a2, call.stream));
    return ok ? DEFT_OK : DEFT_EHIP;
}

// A number that no call of this process has had and that no memory is likely to hold.
uint64_t new_ticket() {
    static std::atomic<uint64_t> last{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() ^
                                      (uint64_t)reinterpret_cast<uintptr_t>(&hip_ok)};
    uint64_t x = last.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);  // splitmix64
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    x ^= x >> 31;
    return x ? x : 1;
}

// Both stages in one launch.
int run_call(const deft_plan_t *plan, const Call &call, const void *q, const void *k, const void *v, void *o, int32_t Hq,
             int32_t Hkv, int32_t d, uint32_t flags, int32_t polls) {
    if (!stage1_inputs_ok(q, k, v)) return DEFT_EINVAL;
    const deft::TaskSet &T = whole_call(call, Hkv, d);
    CallArgs a{};
    stage1_args(call, q, k, v, Hq, Hkv, a.s1);
    stage2_args(plan, call, T, o, Hq, flags, a.s2);
    a.s1.marks = call.marks;
    a.s1.ticket = new_ticket();
    a.s1.n_slots = plan->n_slots();
    a.polls = polls;
    const unsigned rows = (unsigned)plan->nq * (unsigned)Hq;
    const unsigned groups = std::min((rows + kWaves - 1) / kWaves, kReduceGroups);
    const bool ok = d == 128 ? launch_stage1<128, true>(T, a, groups, call.img, call.stream)
                             : launch_stage1<64, true>(T, a, groups, call.img, call.stream);
    return ok ? DEFT_OK : DEFT_EHIP;
}

// Whether what is enqueued on a stream now is recorded and run later, any number of times.  (The null stream's never is.)
bool is_captured(hipStream_t st) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (st && hipStreamIsCapturing(st, &capture) != hipSuccess) {
        (void)hipGetLastError();
        return true;  // nobody can tell: whatever suits both
    }
    return capture != hipStreamCaptureStatusNone;
}

// Which calls are made in one launch.  It saves the host 2 to 3 us and the GPU the microsecond between two kernels, but
// partial results cross the caches one by one, and the few waves that stage 2 has (reduce_rows) take some 2 us for every
// further batch of kReduceLoads loads.  With a row of the output to a wave: one batch where K and V are of a size that the
// host's work is a good part of the call, two where they are small.  With two rows: half a batch each.  Whole call, us, two
// launches -> one: one row of one batch, 0.4 MB 9.8 -> 6.8, 16 MB 9.8 -> 7.9, 33 MB 9.7 -> 9.2, 39 MB 12.3 -> 12.3, but 41 MB
// 13.0 -> 13.4; one of two, 6 MB 9.9 -> 8.5, 16 MB 9.9 -> 8.8, but 34 MB 9.7 -> 9.7, and earlier 38 MB 14.2 -> 15.1; two of half
// a batch, 0.6 MB 9.8 -> 8.8, 9 MB 9.9 -> 9.1, 2.4 MB 8.7 -> 9.0 where the host is quick, 9.9 -> 9.1 where it is not; two of
// one batch 8.8 -> 9.9, 10.0 -> 11.1, 10.1 -> 10.5 and 8.5 -> 11.0; three batches, 1.7 MB 11.4 -> 12.2, 5 MB 11.6 -> 13.0 or 10.1.
// A captured call takes two: its replays have no host to spare and the GPU is the slower for it (0.4 MB 6.4 -> 6.9, 16 MB 6.8 ->
// 7.5, 5 MB under 56 rows 7.5 -> 11.3), and their marks could hold the ticket from the replay before.
bool one_launch(const deft_plan_t *plan, const Call &call, int32_t Hq, int32_t Hkv, int32_t d) {
    constexpr int64_t kWavesOfRows = kWaves * kReduceGroups;
    const deft::TaskSet &T = whole_call(call, Hkv, d);
    if (!call.marks || plan->nq == 0 || T.n_items == 0) return false;
    const int64_t batch = d == 128 ? kReduceLoads * Stage2Row<128>::kRows : kReduceLoads * Stage2Row<64>::kRows;
    const int64_t rows = (int64_t)plan->nq * Hq, parts = T.max_parts, bytes = (int64_t)plan->n_flat * Hkv * d * 4;
    const bool pays = rows <= kWavesOfRows ? (parts <= batch && bytes <= (40 << 20)) || (parts <= 2 * batch && bytes <= (16 << 20))
                                           : rows <= 2 * kWavesOfRows && 2 * parts <= batch && bytes <= (16 << 20);
    return pays && !is_captured(call.stream);
}

// Pinned host staging for plan images: a ring of slots per device, allocated at the first upload on that
// device and kept until the process ends.  An image is copied into the next slot and fetched from there by a
// kernel on the stream, so deft_plan_upload neither waits for the stream nor depends on the plan staying
// alive.  A slot is reused only after its event has completed, which also is where a failure of the device is heard of.  The
// event is the fetch kernel's own end: recorded behind it, it would be a packet of its own that the queue stops at (4 us of a
// decode iteration of 147), and a fence for the host, which reads nothing, would be 1 us more.  Where memory
// or stream are not the current device's, the image is sent by a copy command with the event behind it.  In a stream that is
// being captured no slot is used (store_captured): replays would read it when it holds another plan's image.
constexpr int kStageSlots = 8;
constexpr size_t kStageSlotBytes = DEFT_STAGED_IMAGE_BYTES;
struct Staging {
    std::mutex mu;
    uint8_t *base = nullptr, *seen = nullptr;  // the slots, as the host and as the device addresses them
    hipEvent_t done[kStageSlots] = {};
    bool used[kStageSlots] = {};
    int next = 0;
};
Staging g_staging[64];

// Whether a kernel on this stream may be launched now and write there.  A copy command goes into any stream and reaches any
// memory; a kernel goes into a stream of the current device and reaches that device's memory: the memory of another one, or
// of the host, may not be mapped for it.
bool on_stream_device(const void *p, hipStream_t st, int dev) {
    hipPointerAttribute_t at{};
    hipDevice_t stream_dev = dev;
    if (hipPointerGetAttributes(&at, p) != hipSuccess || (st && hipStreamGetDevice(st, &stream_dev) != hipSuccess)) {
        (void)hipGetLastError();
        return false;
    }
    return at.type == hipMemoryTypeDevice && at.device == dev && stream_dev == dev;
}

// An image into a graph.
bool store_captured(void *dev_image, const uint8_t *src, size_t bytes, hipStream_t st) {
    const size_t words = bytes / 16;  // an image is a whole number of them
    for (size_t at = 0; at < words; at += kPartWords) {
        const uint32_t n = (uint32_t)std::min<size_t>(kPartWords, words - at);
        ImagePart part{};
        std::memcpy(part.word, src + 16 * at, 16 * n);
        hipLaunchKernelGGL(deft_store_part, dim3(1), dim3(256), 0, st, static_cast<u32x4 *>(dev_image) + at, n, part);
        if (!hip_ok(hipGetLastError(), "captured plan upload")) return false;
    }
    return true;
}

// Returns 1 when the image is on its way, 0 when the caller has to take the plain path
// (image larger than a slot, device index out of range), -1 on a runtime error.
int upload_staged(void *dev_image, const uint8_t *src, size_t bytes, hipStream_t st) {
    int dev = 0;
    if (bytes > kStageSlotBytes) return 0;
    if (!hip_ok(hipGetDevice(&dev), "hipGetDevice")) return -1;
    if (dev < 0 || dev >= 64) return 0;
    const bool fetch = on_stream_device(dev_image, st, dev);
    if (is_captured(st)) {
        if (!fetch) {
            g_hip_error = "captured plan upload: memory and stream have to be the current device's";
            return -1;
        }
        return store_captured(dev_image, src, bytes, st) ? 1 : -1;
    }
    Staging &g = g_staging[dev];
    std::lock_guard<std::mutex> lock(g.mu);
    if (!g.base) {
        void *p = nullptr, *seen = nullptr;
        if (!hip_ok(hipHostMalloc(&p, kStageSlots * kStageSlotBytes, hipHostMallocMapped | hipHostMallocCoherent), "pinned staging"))
            return -1;
        bool ok = hip_ok(hipHostGetDevicePointer(&seen, p, 0), "pinned staging");
        int made = 0;
        for (; ok && made < kStageSlots; ++made)
            if (!hip_ok(hipEventCreateWithFlags(&g.done[made], hipEventDisableTiming | hipEventDisableSystemFence), "staging event")) break;
        if (!ok || made < kStageSlots) {
            for (int j = 0; j < made; ++j) (void)hipEventDestroy(g.done[j]);
            (void)hipHostFree(p);
            return -1;
        }
        std::memset(p, 0, kStageSlots * kStageSlotBytes);  // (or the first image in each slot takes 10 us more, page by page)
        g.seen = static_cast<uint8_t *>(seen);
        g.base = static_cast<uint8_t *>(p);
    }
    const int i = g.next;
    g.next = (g.next + 1) % kStageSlots;
    if (g.used[i] && !hip_ok(hipEventSynchronize(g.done[i]), "staging slot")) return -1;
    uint8_t *slot = g.base + (size_t)i * kStageSlotBytes;
    std::memcpy(slot, src, bytes);
    if (!fetch) {
        if (!hip_ok(hipMemcpyAsync(dev_image, slot, bytes, hipMemcpyHostToDevice, st), "plan upload")) return -1;
        if (!hip_ok(hipEventRecord(g.done[i], st), "staging event record")) return -1;
    } else {
        const uint32_t words = (uint32_t)(bytes / 16);  // an image is a whole number of them
        hipExtLaunchKernelGGL(deft_fetch_image, dim3((words + kFetchThreads - 1) / kFetchThreads), dim3(kFetchThreads), 0, st, nullptr,
                              g.done[i], 0, reinterpret_cast<const u32x4 *>(g.seen + (size_t)i * kStageSlotBytes),
                              static_cast<u32x4 *>(dev_image), words);
        if (!hip_ok(hipGetLastError(), "plan upload")) return -1;
    }
    g.used[i] = true;
    return 1;
}

}  // namespace

extern "C" const char *deft_last_hip_error(void) { return g_hip_error.c_str(); }

extern "C" int deft_hbm_read_probe(const void *dev_buf, size_t bytes, void *dev_sink, void *stream) {
    if (!dev_buf || !dev_sink || bytes == 0 || (bytes & 15) || (reinterpret_cast<uintptr_t>(dev_buf) & 15)) return DEFT_EINVAL;
    const size_t n16 = bytes / 16;
    hipLaunchKernelGGL(deft_read_probe, dim3(kProbeGroups), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const u32x4 *>(dev_buf), n16, static_cast<uint32_t *>(dev_sink));
    return hip_ok(hipGetLastError(), "deft_read_probe launch") ? DEFT_OK : DEFT_EHIP;
}

extern "C" int deft_plan_upload(deft_plan_t *plan, int32_t Hq, int32_t Hkv, void *dev_image, size_t bytes, void *stream) {
    if (!plan || !dev_image || Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0) return DEFT_EINVAL;
    if (!aligned16(dev_image)) return DEFT_EINVAL;
    const deft::Schedule *S = nullptr;
    try {
        S = deft::get_schedule(plan, Hq / Hkv, Hkv);
    } catch (...) {
        return DEFT_ENOMEM;
    }
    if (bytes < S->bytes) return DEFT_EWORKSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int staged = upload_staged(dev_image, S->host_image.data(), S->bytes, st);
    if (staged < 0) return DEFT_EHIP;
    if (staged > 0) return DEFT_OK;
    // an image larger than a staging slot goes from the plan's own (pageable) copy, and the call waits for it
    if (!hip_ok(hipMemcpyAsync(dev_image, S->host_image.data(), S->bytes, hipMemcpyHostToDevice, st), "plan upload"))
        return DEFT_EHIP;
    if (!hip_ok(hipStreamSynchronize(st), "plan upload sync")) return DEFT_EHIP;
    return DEFT_OK;
}

extern "C" int deft_stage1_partial_attention(const deft_plan_t *plan, const void *dev_image, const void *q,
                                             const void *k, const void *v, int32_t Hq, int32_t Hkv, int32_t d,
                                             float scale, void *workspace, size_t workspace_bytes, void *stream) {
    Call call;
    int rc = prepare(plan, dev_image, Hq, Hkv, d, scale, workspace, workspace_bytes, stream, call);
    if (rc != DEFT_OK) return rc;
    return run_stage1(plan, call, call.S->by_chunk, q, k, v, Hq, Hkv, d);
}

extern "C" int deft_stage2_global_reduction(const deft_plan_t *plan, const void *dev_image, void *o, int32_t Hq,
                                            int32_t Hkv, int32_t d, float scale, uint32_t flags, void *workspace,
                                            size_t workspace_bytes, void *stream) {
    Call call;
    int rc = prepare(plan, dev_image, Hq, Hkv, d, scale, workspace, workspace_bytes, stream, call);
    if (rc != DEFT_OK) return rc;
    return run_stage2(plan, call, call.S->by_chunk, o, Hq, d, flags);
}

namespace {
int decode(const deft_plan_t *plan, const void *dev_image, const void *q, const void *k, const void *v, void *o, int32_t Hq, int32_t Hkv,
           int32_t d, float scale, uint32_t flags, void *workspace, size_t workspace_bytes, void *stream, int32_t polls) {
    Call call;
    int rc = prepare(plan, dev_image, Hq, Hkv, d, scale, workspace, workspace_bytes, stream, call);
    if (rc != DEFT_OK) return rc;
    // check both stages' arguments before launching anything
    if (flags != DEFT_OUT_BF16 && flags != DEFT_OUT_F32) return DEFT_EINVAL;
    if (plan->nq > 0 && (!o || !aligned16(o))) return DEFT_EINVAL;
    if (one_launch(plan, call, Hq, Hkv, d)) return run_call(plan, call, q, k, v, o, Hq, Hkv, d, flags, polls);
    rc = run_stage1(plan, call, whole_call(call, Hkv, d), q, k, v, Hq, Hkv, d);
    if (rc != DEFT_OK) return rc;
    return run_stage2(plan, call, whole_call(call, Hkv, d), o, Hq, d, flags);
}
}  // namespace

extern "C" int deft_tree_attn_decode(const deft_plan_t *plan, const void *dev_image, const void *q, const void *k,
                                     const void *v, void *o, int32_t Hq, int32_t Hkv, int32_t d, float scale,
                                     uint32_t flags, void *workspace, size_t workspace_bytes, void *stream) {
    return decode(plan, dev_image, q, k, v, o, Hq, Hkv, d, scale, flags, workspace, workspace_bytes, stream, kMarkPolls);
}

extern "C" int deft_decode_polls(const deft_plan_t *plan, const void *dev_image, const void *q, const void *k, const void *v, void *o,
                                 int32_t Hq, int32_t Hkv, int32_t d, float scale, uint32_t flags, void *workspace,
                                 size_t workspace_bytes, void *stream, int32_t polls) {
    if (polls < 1 || polls > kMarkPolls) return DEFT_EINVAL;
    return decode(plan, dev_image, q, k, v, o, Hq, Hkv, d, scale, flags, workspace, workspace_bytes, stream, polls);
}

namespace {

// Device address of `scratch` on the current device, looked up once per device.
std::mutex g_scratch_mu;
void *g_scratch_ptr[64] = {};

int static_scratch(void **out) {
    int dev = 0;
    if (!hip_ok(hipGetDevice(&dev), "hipGetDevice")) return DEFT_EHIP;
    if (dev < 0 || dev >= 64) return DEFT_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (!hip_ok(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "address of the static workspace")) return DEFT_EHIP;
        if (!p || !aligned16(p)) return DEFT_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return DEFT_OK;
}

}  // namespace

extern "C" int deft_tree_attn_decode_static(const deft_plan_t *plan, const void *dev_image, const void *q,
                                            const void *k, const void *v, void *o, int32_t Hq, int32_t Hkv, int32_t d,
                                            float scale, uint32_t flags, void *stream) {
    // size first: a plan whose partial results do not fit is refused before anything touches the device
    if (deft_workspace_bytes(plan, Hq, Hkv, d) == 0) return DEFT_EINVAL;
    if (deft::partials_bytes(plan, Hq, d) > (size_t)DEFT_STATIC_SCRATCH_BYTES) return DEFT_EWORKSPACE;
    void *ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc != DEFT_OK) return rc;
    // every (slot, head) stage 2 reads was written by stage 1 of the same call, so nothing has to be cleared
    return deft_tree_attn_decode(plan, dev_image, q, k, v, o, Hq, Hkv, d, scale, flags, ws, DEFT_STATIC_SCRATCH_BYTES,
                                 stream);
}
