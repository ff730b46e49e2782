// Backward kernels of gist-masked attention for gfx950 (bf16 MFMA, fp32 accumulation), no atomics.
//
// With P_ij = exp(scale S_ij - lse_i) on the visible pairs of Sec. 4.1, Eq. 3:
//   delta_i = dO_i . O_i                      dV_j = sum_i P_ij dO_i
//   dP_ij   = dO_i . V_j                      dS_ij = P_ij (dP_ij - delta_i)
//   dQ_i    = scale sum_j dS_ij K_j           dK_j = scale sum_i dS_ij Q_i   (summed over the q heads of a group)
//
// Launch sequence (all on the caller's stream):
//   1. dq_kernel            one workgroup per four units of 32 query rows of a head, same tile walk as the forward;
//                           leaves delta = rowsum(dO * O) and lse * log2(e) of its rows in the workspace
//   2. dkdv_kernel<GIST>    one workgroup per (compact gist tile, segment of query chunks): the pairs whose
//                           gist lies left of the query chunk's window phase; fp32 partials to the workspace
//   3. gist_reduce_kernel   sums the segments of a gist tile in a fixed order
//   4. dkdv_kernel<WINDOW>  one workgroup per contiguous 128-key tile: the pairs of the window phase; its
//                           epilogue adds the reduced gist-phase sums to the gist rows and writes dK, dV
// Short backwards run 2, 4 and 1 as one launch (bwd_joint_kernel) behind delta_kernel, which computes delta then, and 3
// behind it, where it writes the gist rows.  Backwards whose dQ is written over an input of the other phases, and stages
// launched one by one, start with delta_kernel too and end with 1.
// Every (query, key) pair is handled by exactly one of the two dkdv phases: a query chunk c (64 rows) sees
// the sinks and gists at positions < far(c) = floor(win_lo(64c) / 128) * 128 in the gist phase (win_lo = first
// position of a row's local window) and every key >= far(c) in the window phase.
//
// All contractions run on v_mfma_f32_16x16x32_bf16 (operand layouts in mfma_common.h); a wave always works on
// two 16-wide blocks at once so that every fragment read from LDS feeds two MFMAs.
// dkdv: a wave owns 32 keys as two 16-key blocks (a key is a column, spread over four lanes), K and V fragments
// stay in registers, Q / dO chunks are staged in LDS and read both row-wise (S = Q K^T, dP = dO V^T) and through
// transposing LDS reads (dV^T += dO^T P, dK^T += Q^T dS); the S/dP accumulators of the two 16-row halves of a
// query block are already the B operands of the last two.
// dq: forward-shaped; S^T = K Q^T and dP^T = V dO^T for the wave's two 16-row query blocks, dQ^T += K^T dS^T.
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "mfma_common.h"
#include "plan.h"

namespace unigist {
namespace {

constexpr int NT = 256;
constexpr int BNQ = kDqBn;  // keys per dq step
constexpr int PFS = 2, PFT = 2;  // dq: LDS fragment reads issued this many MFMA groups ahead (S/dP phase, dQ phase)
constexpr float kLog2e = 1.4426950408889634f;

// bits 0 .. n-1 set (none for n <= 0, all for n >= 32)
__device__ __forceinline__ unsigned below_bits(int n) { return n >= 32 ? ~0u : n <= 0 ? 0u : (1u << n) - 1u; }

// chunk steps (per kv head) of the gist phase of one sequence: every gist tile is walked by the chunks from the
// first one that has it left of its window phase to the last
long gist_chunk_steps(const AttnShape& s) {
    BwdPlan p;
    plan_counts(s, p, 32);
    long n = 0;
    for (int t = 0; t < p.n_gt; ++t) n += p.NC - first_chunk_with_more_far(s, p.NC, t * BNK);
    return n;
}

// Segment length (query chunks per gist-phase workgroup) for a launch with `steps` chunk steps in total over all
// (batch, kv head) pairs.  A workgroup of segc chunks walks segc * Hq/Hkv steps one after the other, so a launch that
// does not fill the chip's 512 workgroup slots (2 per CU) takes as long as its longest workgroup and wants short
// segments; a launch of many rounds wants long ones, whose fp32 partial sums (128 KB per workgroup at D = 128, written
// and read back once) are fewer.  Measured where the phases are launched apart (packs, and backwards beyond
// run_jointly's line), gist phase + reduction in us, segments of 2 / 4 / 8 / 16 / 32 chunks:
//   864 steps (2 x 2047 tokens, r 4, W 128)   58 /   62 /   92 /  152 /  248     (16 was the shortest before)
//   1392      (4096, W 512)                   83 /   76 /   95 /  152 /  278
//   5280      (8192, W 1024)                 220 /  219 /  198 /  207 /  279
//   10752     (8192, r 2, W 128)             441 /  433 /  361 /  356 /  375
//   23616     (16384, W 1024)                785 /  787 /  791 /  729 /  745
//   99600     (32768, W 1024)               2806 / 2816 / 2842 / 2833 / 2690
// The lines lie where neighbours cross: half a round of 512 such workgroups for the short ones, three quarters for
// 16, five rounds for 32.
int pick_segc(long steps) {
    const long slots = 512;
    if (steps >= slots * 32 * 5) return 32;
    if (steps >= slots * 16 * 3 / 4) return 16;
    if (steps >= slots * 8 / 2) return 8;
    return steps >= slots * 4 / 2 ? 4 : 2;
}
// The longest segments a launch takes for want of room.  A workspace for them is all that a call insists on: below the line
// of 32 it grows with the sequence, where the one for pick_segc's shrinks at each line (32/8 heads, W 512: 74 MB at 3520
// rows, 42 MB at 3521), and a buffer sized for the longest of a caller's sequences has to serve the shorter ones.
int roomiest_segc(long steps) { return std::max(pick_segc(steps), 16); }

long launch_steps(const AttnShape& s) { return gist_chunk_steps(s) * s.B * s.Hkv; }

// plan and workspace layout for segments of segc chunks, without the launch order
BwdPlan sized_plan(const AttnShape& s, int segc) {
    BwdPlan p;
    plan_counts(s, p, segc);
    plan_slots(s, p);
    const size_t a = 255;
    size_t off = ((size_t)s.B * s.Hq * s.L * sizeof(float) + a) & ~a;
    p.off_lse2 = off;  // lse * log2(e), written with delta by the leading dQ launch or the delta pass
    off += ((size_t)s.B * s.Hq * s.L * sizeof(float) + a) & ~a;
    p.off_part = off;  // one [2][D][BNK] fp32 block per (batch, kv head, segment, compact tile the segment reaches)
    off += (size_t)s.B * s.Hkv * p.slot0[p.nseg] * 2 * padded_head_dim(s.D) * BNK * sizeof(float);
    off = (off + a) & ~a;
    p.off_comp = off;  // their sums over the segments: one block per (batch, kv head, compact tile)
    off += (size_t)s.B * s.Hkv * p.n_gt * 2 * padded_head_dim(s.D) * BNK * sizeof(float);
    p.total = (off + a) & ~a;
    return p;
}

// Segment length for a joint launch (dense backwards up to run_jointly's line).  The other phases fill the slots that a few
// long units leave, so what limits the length is a unit itself, whose segc * Hq/Hkv steps run one after the other: it may take
// 1.6 times as long as all steps of the launch spread evenly over the chip's workgroup slots.  (The units come first, and
// in launches that small many of them walk only a part of their segment.)  A step of dQ, 64 keys, takes about 0.55 of a dK/dV
// step.  Whole backward, us, segments of 2 / 4 / 8 / 16 / 32 chunks; + = what the lines of pick_segc give, * = what is picked:
//   2 x 2047, 32/8 heads, W 128             136+ / 124  / 117* / 174  / 275
//   4096, W 512                             227  / 220+ / 205  / 203* / 319
//   3000, 16/16 heads, D 96, W 300           90  /  78+ /  70* /  68  /  81
//   6000, 8/1 heads, W 200                  151+* / 150 / 169  / 300  / 557
//   5000, 28/4 heads, r 2, 60 units         303  / 300  / 290+* / 310 / 539
//   3 x 2500, 16/4, D 64, 20 units           84  /  75+* / 80  / 122  / 192
//   8192, W 1024                            744  / 737  / 702+ / 682  / 669*
//   12000, 16/16, r 2, W 70                 968  / 962  / 968  / 826+ / 758*
//   20000, 8/1, D 64, W 1000                375  / 374  / 374+ / 373* / 452
// Sizes are asked for and refused by pick_segc, whose segments are never longer.
int pick_joint_segc(const AttnShape& s, long steps, int n_dq_wgs) {
    const long G = s.Hq / s.Hkv, NP = (long)s.B * s.Hkv, slots = 256 * (s.D <= 64 ? 3 : 2);
    const long reach = s.umode ? (s.W + 1L) * s.rp1 : s.W;  // rows that have a key in their window
    const double gist = (double)steps * G;
    const double window = (double)((s.L + BNK - 1) / BNK) * NP * G * (std::min((long)s.L, reach + BNK) / MQ);
    const double dq = (double)n_dq_wgs * (std::min((long)s.L, reach + kWaveRows) + s.L / s.rp1 / 2) / kDqBn;
    const double even = (gist + window + 0.55 * dq) / slots;
    int segc = pick_segc(steps);
    while (segc < 32 && 2 * segc * G <= 1.6 * even) segc *= 2;
    return segc;
}

// the plan of a launch whose workspace has `room` bytes: segments of segc chunks, or of the first doubling that fits
BwdPlan make_plan(const AttnShape& s, long steps, size_t room, int segc) {
    const int longest = std::max(segc, roomiest_segc(steps));
    BwdPlan p = sized_plan(s, segc);
    while (p.total > room && segc < longest) p = sized_plan(s, segc *= 2);
    plan_order(s, p);
    return p;
}

// ------------------------------------------------------------------ delta and lse * log2(e) in a pass of their own
// dO . O of eight columns; the columns are summed in this order and the eights in a tree wherever delta is computed, so that
// it is the same number to the last bit
__device__ __forceinline__ float dot8(const u32x4& a, const u32x4& b) {
    float acc = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        acc += __uint_as_float(a[t] << 16) * __uint_as_float(b[t] << 16);
        acc += __uint_as_float(a[t] & 0xffff0000u) * __uint_as_float(b[t] & 0xffff0000u);
    }
    return acc;
}

template <int D>
__global__ __launch_bounds__(NT) void delta_kernel(const bf16_t* __restrict__ out, const bf16_t* __restrict__ dout,
                                                  const float* __restrict__ lse, float* __restrict__ delta,
                                                  float* __restrict__ lse2, long nrows, int L, int qhs, int Hq,
                                                  long long q_bs, long long q_hs, int q_rs, int Dt) {
    constexpr int LPR = D / 8;  // lanes per row, 16 bytes each (Dt <= D elements per row in memory)
    const long row = (long)blockIdx.x * (NT / LPR) + threadIdx.x / LPR;  // dense: (b, h, i) -> (b Hq + h) L + i
    const int sub = threadIdx.x % LPR;
    const long grow = L == qhs ? row : (row / L) * qhs + row % L;        // the same row in the caller's tensors
    float acc = 0.f;
    if (row < nrows) {
        // element offset of the row in out / dout: dense, or with the caller's explicit strides (q_rs != 0)
        const long bh = row / L;
        const long eoff = q_rs ? (bh / Hq) * q_bs + (bh % Hq) * q_hs + (row % L) * (long)q_rs : grow * Dt;
        u32x4 a = {0u, 0u, 0u, 0u}, b = {0u, 0u, 0u, 0u};
        if (sub * 8 < Dt) {
            a = *(const u32x4*)(out + eoff + sub * 8);
            b = *(const u32x4*)(dout + eoff + sub * 8);
        }
        acc = dot8(a, b);
    }
    // reduce over the LPR lanes of a row (LPR is 8 or 16, rows are aligned to LPR lanes)
#pragma unroll
    for (int off = 1; off < LPR; off <<= 1) acc += __shfl_xor(acc, off, 64);
    if (row < nrows && sub == 0) {
        delta[row] = -acc;               // stored negated: the consumers add it (dK/dV: as the dP accumulator's start)
        lse2[row] = lse[grow] * kLog2e;  // the exponent base the dK/dV and dQ kernels subtract
    }
}

// Slots of a plan without a table (a document of a pack), one segment per lane: a count costs a few integer divisions,
// and added up one segment after the other, as each workgroup's first work, they held the reduction of five documents
// (32K tokens, 250 MB of partials) to 151 us; now 68 us.
struct SegSlots {
    int tiles, first;  // of segment `lane` (0 tiles from segment nseg on): compact tiles it reaches, its first slot
    int total;         // slots of the plan
};
__device__ __forceinline__ SegSlots wave_seg_slots(const AttnShape& s, const BwdPlan& pl, int lane) {
    static_assert(kMaxSegs <= 64, "a lane per segment");
    SegSlots r;
    r.tiles = lane < pl.nseg ? seg_tiles(s, pl, lane) : 0;
    int end = r.tiles;
#pragma unroll
    for (int off = 1; off < kMaxSegs; off <<= 1) {
        const int x = __shfl_up(end, off, 64);
        if (lane >= off) end += x;
    }
    r.first = end - r.tiles;
    r.total = __builtin_amdgcn_readlane(end, kMaxSegs - 1);
    return r;
}

// ------------------------------------------------------------------ 2./4. dK, dV
template <int D>
struct DkdvSmem {
    // the rows' lse * log2(e) and -delta first: with the two 64 KB of tiles in front of them their addresses would
    // not fit the 16-bit offset field of the LDS instructions and cost a vector instruction per read
    float lse2[2][MQ];
    float delta[2][MQ];
    // two stages of a 64-row Q chunk and dO chunk (rows unpadded, 16-byte chunks swizzled)
    char q[2][MQ * D * 2];
    char g[2][MQ * D * 2];
};

// GEN = false (here and in dq_kernel) is the layout without sinks and with the sliding window: the mask
// helpers then fold to their short forms at compile time.
// PACK = true (here and in dq_kernel): the launch covers the documents of a packed buffer (docs), s_arg is the shape
// of the whole pack, delta and lse2 have the layout of the caller's lse ([Hq, T]), and every document has its
// own run of slots in part and comp.
// QSTR = true: q and dout have the explicit strides of s_arg (q_bs, q_hs, q_rs) instead of the dense layout.  Tensors
// whose head dimension s.D is smaller than the D the kernel is built for (any multiple of 8) also come this way, with
// the strides of their dense layout: rows in memory are s.D elements long, LDS tiles and fragments have D columns,
// of which those from s.D on are zero in the K and V fragments (so they add nothing to S and dP) and are never stored.
template <int D, bool GIST, bool GEN, bool PACK, bool QSTR = false>
__global__ __launch_bounds__(NT, 2) void dkdv_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                    const bf16_t* __restrict__ v, const float* __restrict__ lse2,
                                                    const bf16_t* __restrict__ dout, const float* __restrict__ delta,
                                                    bf16_t* __restrict__ dk, bf16_t* __restrict__ dv,
                                                    float* __restrict__ part, const float* __restrict__ comp,
                                                    AttnShape s_arg, BwdPlan pl,
                                                    std::conditional_t<PACK, DocTab, NoDocs> docs) {
    constexpr bool JOINT = false;
    constexpr float* keep = nullptr;
    __shared__ __attribute__((aligned(1024))) DkdvSmem<D> sm;
    AttnShape s = s_arg;
    if constexpr (!GEN) {
        s.S = 0;
        s.umode = 0;
    }
    int n = blockIdx.x;
    if constexpr (PACK) {  // the document becomes the whole problem
        const int d = doc_of_block(docs, n);
        n -= docs.blk0[d];
        s = doc_view(s, docs.len[d]);
        plan_counts(s, pl, pl.segc);  // pl arrives with the launch's segment length only
        const size_t ro = (size_t)docs.c0[d] * (QSTR ? s.D : D);
        const size_t qro = QSTR ? (size_t)docs.c0[d] * s.q_rs : ro;
        q += qro;
        k += ro;
        v += ro;
        dout += qro;
        dk += ro;
        dv += ro;
        lse2 += docs.c0[d];
        delta += docs.c0[d];
        part += (size_t)docs.part0[d] * (2 * D * BNK);
        comp += (size_t)docs.comp0[d] * (2 * D * BNK);
    }
#include "dkdv_body.inc"
}

// ------------------------------------------------------------------ 3. sum the segments of each gist tile
// FINISH = false: the sums go to comp, and the window phase adds them to its own.  FINISH = true (after the joint
// launch): comp holds the window phase's sums of the gist rows; they are added and the rows of dk and dv written.
template <int D, bool FINISH>
__global__ __launch_bounds__(NT) void gist_reduce_kernel(const float* __restrict__ part, float* __restrict__ comp,
                                                        bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, BwdPlan pl,
                                                        AttnShape s) {
    // grid: x = slices of a tile's 2 D BNK floats (four per thread), y = tile, z = (b, hk).  The segments are
    // added in ascending order, so the result does not depend on the launch.
    constexpr int per_tile = 2 * D * BNK;
    static_assert(per_tile % (4 * NT) == 0, "whole workgroups");
    const int gt = blockIdx.y;
    const int idx = 4 * (blockIdx.x * NT + threadIdx.x);
    const int cf = first_chunk_with_more_far(s, pl.NC, gt * BNK);
    const float* pp = part + (size_t)blockIdx.z * pl.slot0[pl.nseg] * per_tile;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (cf < pl.NC)  // the tile has a slot in every segment from that of its first chunk on
#pragma unroll 4
        for (int sg = cf / pl.segc; sg < pl.nseg; ++sg) acc += *(const f32x4*)(pp + (size_t)(pl.slot0[sg] + gt) * per_tile + idx);
    float* cp = comp + ((size_t)blockIdx.z * pl.n_gt + gt) * per_tile + idx;
    if constexpr (FINISH) {
        const int e = gt * BNK + idx / (2 * D), col = idx % D;  // entry of the compact list; column of dK or dV
        if (e >= count_always(s, s.L) || col >= s.D) return;    // the last tile's missing entries; padding columns
        acc = *(const f32x4*)cp + acc;
        u32x2 r;
        r[0] = pack_bf16x2(acc[0], acc[1]);
        r[1] = pack_bf16x2(acc[2], acc[3]);
        bf16_t* o = idx % (2 * D) < D ? dk : dv;
        *(u32x2*)(o + ((size_t)blockIdx.z * s.kvhs + pos_of_always(s, e)) * s.D + col) = r;
    } else {
        *(f32x4*)cp = acc;
    }
}

// The same for a packed launch.  grid: x = slot of comp (a document's slots are its (kv head, gist tile) pairs,
// docs.blk0 holds the first slot of each document), y = slice of the slot's 2*D*BNK floats.
__global__ __launch_bounds__(NT) void gist_reduce_pack_kernel(const float* __restrict__ part, float* __restrict__ comp,
                                                             AttnShape s_arg, int per_tile, int segc, DocTab docs) {
    const int idx = 4 * (blockIdx.y * NT + threadIdx.x);
    if (idx >= per_tile) return;
    const int d = doc_of_block(docs, blockIdx.x);
    const int t = blockIdx.x - docs.blk0[d];  // (kv head) * n_gt + gist tile
    const AttnShape s = doc_view(s_arg, docs.len[d]);
    BwdPlan pl;
    plan_counts(s, pl, segc);
    const int gt = t % pl.n_gt;
    const int cf = first_chunk_with_more_far(s, pl.NC, gt * BNK);
    const SegSlots sl = wave_seg_slots(s, pl, threadIdx.x & 63);
    const float* pp = part + ((size_t)docs.part0[d] + (size_t)(t / pl.n_gt) * sl.total) * per_tile;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (cf < pl.NC)
        for (int sg = cf / pl.segc; sg < pl.nseg; sg += 4) {  // four loads in flight
            f32x4 x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                x[i] = *(const f32x4*)(pp + (size_t)(__builtin_amdgcn_readlane(sl.first, min(sg + i, pl.nseg - 1)) + gt) * per_tile + idx);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (sg + i < pl.nseg) acc += x[i];
        }
    *(f32x4*)(comp + ((size_t)docs.comp0[d] + t) * per_tile + idx) = acc;
}

// ------------------------------------------------------------------ 1. dQ
template <int D>
struct DqSmem {
    // two stages of a K tile and a V tile, rows unpadded, 16-byte chunks swizzled
    char k[2][BNQ * D * 2];
    char v[2][BNQ * D * 2];
};

// WITH_DELTA = true: the launch runs first and without a delta pass; a wave takes delta and lse * log2(e) of its rows from out
// and lse and leaves them in the workspace for the dK/dV phases.  The pass reads out and dout for that alone (2 x 268 MB at
// 32 heads x 32K x 128: 92 us of 8240 for forward and backward, 186 of 6990 for 4 x 16K at r 16); here dout is in registers
// already and a workgroup reads its 32 KB of out beside its q and dout.  Both together, pass + dQ / dQ with delta: 91 + 2534 /
// 2618 us at 32 x 32K x 128 (rows in registers cost dQ most of what the pass took), 4 x 16K forward and backward 6881 / 6788.
template <int D, bool GEN, bool PACK, bool QSTR = false, bool WITH_DELTA = false>
__global__ __launch_bounds__(NT, 2) void dq_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                  const bf16_t* __restrict__ v, const bf16_t* __restrict__ out,
                                                  const float* __restrict__ lse, float* lse2,
                                                  const bf16_t* __restrict__ dout, float* delta,
                                                  bf16_t* __restrict__ dq, AttnShape s_arg, int nq,
                                                  std::conditional_t<PACK, DocTab, NoDocs> docs) {
    __shared__ __attribute__((aligned(1024))) DqSmem<D> sm;
    AttnShape s = s_arg;
    if constexpr (!GEN) {
        s.S = 0;
        s.umode = 0;
    }
    int n = blockIdx.x;
    if constexpr (PACK) {
        const int d = doc_of_block(docs, n);
        n -= docs.blk0[d];
        s = doc_view(s, docs.len[d]);
        nq = row_units(s.L, s.Hq / s.Hkv).per;
        const size_t ro = (size_t)docs.c0[d] * (QSTR ? s.D : D);
        const size_t qro = QSTR ? (size_t)docs.c0[d] * s.q_rs : ro;
        q += qro;
        k += ro;
        v += ro;
        dout += qro;
        dq += qro;
        lse2 += docs.c0[d];
        delta += docs.c0[d];
        if constexpr (WITH_DELTA) {
            out += qro;
            lse += docs.c0[d];
        }
    }
#include "dq_body.inc"
}

// ------------------------------------------------------------------ 2., 4. and 1. in one launch
// The three heavy parts of a whole backward need nothing from each other (the window phase leaves its sums of the gist
// rows in comp for the reduction that follows), so they run as one launch: workgroups 0 .. n_gist-1 are the gist
// phase, the next n_win the window phase, the rest dQ, whose short walks come last.  What bounds a short backward is not
// the chip but the longest workgroup of each of its launches: alone, a phase of 2 x 2047 tokens leaves half of the 512
// workgroup slots empty.  Phases one by one / jointly (whole backward replayed from a graph, us, 32/8 heads unless noted):
//   1 head, 1024, D 64     36 /   18        1 x 8192           722 /  656
//   2 x 512                91 /   55        28/4 heads, 12000  762 /  655
//   2 x 2047              160 /  121        12288             1081 / 1038
//   2048, W 1024          238 /  187        4 x 4096, W 512    840 /  815
//   4096, W 512           258 /  201        16384             1981 / 1942
//   2 x 9000 (4512 dQ workgroups) 1604 / 1556    4 x 5000, r 8 (5024)  770 /  741    2 x 40000, 8/1 heads, r 8 (5000) 3244 / 3063
//   D 64: 24000, r 8 (6000) 1425 / 1392          8 x 3000 (6016) 415 / 411
// Further on the tails it fills are short, and phases that run side by side share the L2s of each other's streams: 24000 (6000)
// 3436 / 3454, 2 x 16384, r 8 (8192) 3030 / 3043, 32768 (8192) 6161 / 6331, at D = 64 3307 / 3381; without groups earlier: 30000,
// 16/16 heads (3760) 2707 / 2786.  So the lines lie at ten rounds of dQ workgroups with two per CU (D = 128), eight with three (D =
// 64), and without groups at six of either, where that was measured.
template <int D> bool run_jointly(long n_dq, int G) { return n_dq <= 256 * (D <= 64 ? 3 * (G > 1 ? 8 : 6) : 2 * (G > 1 ? 10 : 6)); }

// A dq that shares memory with q or dout, which its own workgroups have read before they write, is written too early for the
// other phases where dQ does not run last: such calls keep the launches apart, delta first and dQ last.  So do calls whose
// dq shares memory with out or lse, which the delta pass has read whole before anything is written.
bool dq_on_its_inputs(const bf16_t* q, const bf16_t* dout, const bf16_t* out, const float* lse, const bf16_t* dq, const AttnShape& s) {
    const long long rows = s.q_rs ? s.q_rs : s.D, heads = s.q_rs ? s.q_hs : (long long)s.qhs * s.D,
                    batches = s.q_rs ? s.q_bs : heads * s.Hq;
    const uintptr_t bytes = 2 * (uintptr_t)((s.B - 1) * batches + (s.Hq - 1) * heads + (s.L - 1) * rows + s.D);
    auto meets = [&](const void* x, uintptr_t n) { return (uintptr_t)x < (uintptr_t)dq + bytes && (uintptr_t)dq < (uintptr_t)x + n; };
    return meets(q, bytes) || meets(dout, bytes) || meets(out, bytes) || meets(lse, (uintptr_t)s.B * s.Hq * s.qhs * sizeof(float));
}

// The bodies are included and not called: as inlined functions of their own they left 4 to 8 VGPRs of all four instantiations
// at D = 128 in scratch, in the window phase a K fragment that was loaded again for every 32-row block, behind the next
// chunk's direct loads (whole backward, us, functions / includes: 2 x 2047 128 / 121, 8192 678 / 660, 2 x 9000 with 8/1 heads
// 574 / 524, 28/4 heads at D = 96 142 / 131).  Now one does, with two (general mask, dense tensors).
template <int D, bool GEN, bool QSTR>
__global__ __launch_bounds__(NT, 2) void bwd_joint_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                         const bf16_t* __restrict__ v, float* __restrict__ lse2,
                                                         const bf16_t* __restrict__ dout, float* __restrict__ delta,
                                                         bf16_t* __restrict__ dq, bf16_t* __restrict__ dk,
                                                         bf16_t* __restrict__ dv, float* __restrict__ part,
                                                         float* __restrict__ comp_, AttnShape s, BwdPlan pl, int n_gist,
                                                         int n_win, int nq) {
    static_assert(sizeof(DqSmem<D>) <= sizeof(DkdvSmem<D>), "one LDS block for both");
    __shared__ __attribute__((aligned(1024))) char smem[sizeof(DkdvSmem<D>)];
    constexpr bool JOINT = true, PACK = false, WITH_DELTA = false;
    const float* lse = nullptr;  // names that the bodies have for other launches
    const bf16_t* out = nullptr;
    float* keep = comp_;
    const float* comp = nullptr;
    if constexpr (!GEN) {
        s.S = 0;
        s.umode = 0;
    }
    if ((int)blockIdx.x < n_gist) {
        constexpr bool GIST = true;
        DkdvSmem<D>& sm = *(DkdvSmem<D>*)smem;
        const int n = blockIdx.x;
#include "dkdv_body.inc"
    } else if ((int)blockIdx.x < n_gist + n_win) {
        constexpr bool GIST = false;
        DkdvSmem<D>& sm = *(DkdvSmem<D>*)smem;
        const int n = blockIdx.x - n_gist;
#include "dkdv_body.inc"
    } else {
        DqSmem<D>& sm = *(DqSmem<D>*)smem;
        const int n = blockIdx.x - n_gist - n_win;
#include "dq_body.inc"
    }
}

template <int D>
hipError_t bwd_launch(const bf16_t* q, const bf16_t* k, const bf16_t* v, const bf16_t* out, const float* lse,
                      const bf16_t* dout, bf16_t* dq, bf16_t* dk, bf16_t* dv, char* ws, size_t room,
                      const AttnShape& s, unsigned stages, hipStream_t st) {
    const int nq = row_units(s.L, s.Hq / s.Hkv).per;
    const long nblk = (long)nq * s.Hkv * s.B;
    if (nblk > 0x7fffffffL) return hipErrorInvalidValue;
    const bool free_order = stages == UNIGIST_BWD_ALL && !dq_on_its_inputs(q, dout, out, lse, dq, s);
    const bool joint = free_order && run_jointly<D>(nblk, s.Hq / s.Hkv);
    const long steps = launch_steps(s);
    const BwdPlan pl = make_plan(s, steps, room, joint ? pick_joint_segc(s, steps, (int)nblk) : pick_segc(steps));
    const bool gen = s.S != 0 || s.umode != 0;
    const bool qstr = s.q_rs != 0;  // q, out, dout, dq with the caller's explicit strides
    float* delta = (float*)ws;
    float* lse2 = (float*)(ws + pl.off_lse2);
    float* part = (float*)(ws + pl.off_part);
    float* comp = (float*)(ws + pl.off_comp);
    hipError_t e;
    const dim3 reduce_grid((2 * D * BNK / 4) / NT, std::max(pl.n_gt, 1), s.B * s.Hkv);
    auto launch_dq = [&](auto with_delta) {
        constexpr bool WD = decltype(with_delta)::value;
        auto go = [&](auto kern) { kern<<<dim3((unsigned)nblk), NT, 0, st>>>(q, k, v, out, lse, lse2, dout, delta, dq, s, nq, NoDocs{}); };
        if (qstr) gen ? go(dq_kernel<D, true, false, true, WD>) : go(dq_kernel<D, false, false, true, WD>);
        else gen ? go(dq_kernel<D, true, false, false, WD>) : go(dq_kernel<D, false, false, false, WD>);
        return hipGetLastError();
    };
    if (free_order && !joint) {
        if ((e = launch_dq(std::true_type{})) != hipSuccess) return e;
    } else if (stages & UNIGIST_BWD_DELTA) {
        constexpr int rows_per_blk = NT / (D / 8);
        const long nrows = (long)s.B * s.Hq * s.L;
        delta_kernel<D><<<dim3((unsigned)((nrows + rows_per_blk - 1) / rows_per_blk)), NT, 0, st>>>(
            out, dout, lse, delta, lse2, nrows, s.L, s.qhs, s.Hq, s.q_bs, s.q_hs, s.q_rs, s.D);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const long n_gist = (long)pl.slot0[pl.nseg] * s.Hkv * s.B, n_win = (long)((s.L + BNK - 1) / BNK) * s.Hkv * s.B;
    if (joint) {
        auto go = [&](auto kern) {
            kern<<<dim3((unsigned)(n_gist + n_win + nblk)), NT, 0, st>>>(q, k, v, lse2, dout, delta, dq, dk, dv, part, comp, s,
                                                                       pl, (int)n_gist, (int)n_win, nq);
        };
        if (qstr) gen ? go(bwd_joint_kernel<D, true, true>) : go(bwd_joint_kernel<D, false, true>);
        else gen ? go(bwd_joint_kernel<D, true, false>) : go(bwd_joint_kernel<D, false, false>);
        if ((e = hipGetLastError()) != hipSuccess || pl.n_gt == 0) return e;
        gist_reduce_kernel<D, true><<<reduce_grid, NT, 0, st>>>(part, comp, dk, dv, pl, s);
        return hipGetLastError();
    }
    if (pl.n_gt > 0 && (stages & UNIGIST_BWD_DKDV_GIST)) {
        const dim3 grid((unsigned)n_gist);
        if (qstr) {
            if (gen) dkdv_kernel<D, true, true, false, true><<<grid, NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, pl, NoDocs{});
            else dkdv_kernel<D, true, false, false, true><<<grid, NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, pl, NoDocs{});
        } else if (gen) dkdv_kernel<D, true, true, false><<<grid, NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, pl, NoDocs{});
        else dkdv_kernel<D, true, false, false><<<grid, NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, pl, NoDocs{});
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (pl.n_gt > 0 && (stages & UNIGIST_BWD_GIST_REDUCE)) {
        gist_reduce_kernel<D, false><<<reduce_grid, NT, 0, st>>>(part, comp, dk, dv, pl, s);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (stages & UNIGIST_BWD_DKDV_WINDOW) {
        const dim3 grid((unsigned)n_win);
        if (qstr) {
            if (gen) dkdv_kernel<D, false, true, false, true><<<grid, NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, pl, NoDocs{});
            else dkdv_kernel<D, false, false, false, true><<<grid, NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, pl, NoDocs{});
        } else if (gen) dkdv_kernel<D, false, true, false><<<grid, NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, pl, NoDocs{});
        else dkdv_kernel<D, false, false, false><<<grid, NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, pl, NoDocs{});
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return (stages & UNIGIST_BWD_DQ) && !free_order ? launch_dq(std::false_type{}) : hipSuccess;
}

// ---- packed documents: the non-empty documents, longest first (their long tiles should not start last), and
// the slots each of them gets in the partial-sum arrays
struct PackPlan {
    std::vector<int> c0, len, part0, comp0;  // per document, in launch order
    int segc;                                // segment length asked of every document's plan
    size_t off_lse2, off_part, off_comp, total;
};

// the plan for segments of segc chunks; order = the non-empty documents, longest first
PackPlan sized_pack_plan(const AttnShape& s, const int* cu, const std::vector<int>& order, int segc) {
    PackPlan pp;
    pp.segc = segc;
    size_t nslot_part = 0, nslot_comp = 0;
    for (int d : order) {
        BwdPlan pl;
        plan_counts(doc_view(s, cu[d + 1] - cu[d]), pl, pp.segc);
        plan_slots(doc_view(s, cu[d + 1] - cu[d]), pl);
        pp.c0.push_back(cu[d]);
        pp.len.push_back(cu[d + 1] - cu[d]);
        pp.part0.push_back((int)nslot_part);
        pp.comp0.push_back((int)nslot_comp);
        nslot_part += (size_t)s.Hkv * pl.slot0[pl.nseg];
        nslot_comp += (size_t)s.Hkv * pl.n_gt;
    }
    const size_t a = 255, per_tile = (size_t)2 * padded_head_dim(s.D) * BNK * sizeof(float);
    size_t off = ((size_t)s.Hq * s.L * sizeof(float) + a) & ~a;  // delta, [Hq, T] like the caller's lse
    pp.off_lse2 = off;
    off += ((size_t)s.Hq * s.L * sizeof(float) + a) & ~a;
    pp.off_part = off;
    off += nslot_part * per_tile;
    pp.off_comp = off;
    off += nslot_comp * per_tile;
    pp.total = (off + a) & ~a;
    if (nslot_part > 0x7fffffffUL) pp.total = 0;  // slot numbers are kept in 32 bits
    return pp;
}

// the plan for a workspace of `room` bytes, like make_plan's (room 0: the least that a call insists on)
PackPlan make_pack_plan(const AttnShape& s, const int* cu, int ndocs, size_t room) {
    std::vector<int> order;
    for (int d = 0; d < ndocs; ++d)
        if (cu[d + 1] > cu[d]) order.push_back(d);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cu[a + 1] - cu[a] > cu[b + 1] - cu[b]; });
    long steps = 0;
    for (int d : order) steps += gist_chunk_steps(doc_view(s, cu[d + 1] - cu[d]));
    steps *= s.Hkv;
    int segc = room == 0 ? roomiest_segc(steps) : pick_segc(steps);
    PackPlan pp = sized_pack_plan(s, cu, order, segc);
    while (pp.total > room && segc < roomiest_segc(steps)) pp = sized_pack_plan(s, cu, order, segc *= 2);
    return pp;
}

template <int D>
hipError_t bwd_launch_pack(const bf16_t* q, const bf16_t* k, const bf16_t* v, const bf16_t* out, const float* lse,
                           const bf16_t* dout, bf16_t* dq, bf16_t* dk, bf16_t* dv, char* ws, size_t room, const AttnShape& s,
                           const int* cu, int ndocs, hipStream_t st) {
    const PackPlan pp = make_pack_plan(s, cu, ndocs, room);
    if (pp.total == 0) return hipErrorInvalidValue;
    float* delta = (float*)ws;
    float* lse2 = (float*)(ws + pp.off_lse2);
    float* part = (float*)(ws + pp.off_part);
    float* comp = (float*)(ws + pp.off_comp);
    hipError_t e;
    const bool free_order = !dq_on_its_inputs(q, dout, out, lse, dq, s);
    if (!free_order) {  // delta and lse2 of every row of the pack (a row's delta does not depend on its document)
        constexpr int rows_per_blk = NT / (D / 8);
        const long nrows = (long)s.Hq * s.L;
        delta_kernel<D><<<dim3((unsigned)((nrows + rows_per_blk - 1) / rows_per_blk)), NT, 0, st>>>(
            out, dout, lse, delta, lse2, nrows, s.L, s.qhs, s.Hq, 0, s.q_hs, s.q_rs, s.D);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const int nd = (int)pp.len.size();
    // one launch of each kernel per kMaxDocs documents; blocks(i) = workgroups (or slots) of document i
    auto for_chunks = [&](auto&& blocks, auto&& launch) -> hipError_t {
        for (int at = 0; at < nd; at += kMaxDocs) {
            DocTab t;
            memset(&t, 0, sizeof t);
            t.n = std::min(kMaxDocs, nd - at);
            long nblk = 0;
            for (int i = 0; i < t.n; ++i) {
                t.c0[i] = pp.c0[at + i];
                t.len[i] = pp.len[at + i];
                t.part0[i] = pp.part0[at + i];
                t.comp0[i] = pp.comp0[at + i];
                t.blk0[i] = (int)nblk;
                nblk += blocks(pp.len[at + i]);
                if (nblk > 0x7fffffffL) return hipErrorInvalidValue;
            }
            t.blk0[t.n] = (int)nblk;
            if (nblk == 0) continue;
            launch(t, (unsigned)nblk);
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
        return hipSuccess;
    };
    auto counts = [&](int len) {
        BwdPlan pl;
        plan_counts(doc_view(s, len), pl, pp.segc);
        plan_slots(doc_view(s, len), pl);
        return pl;
    };
    BwdPlan none = {};
    none.segc = pp.segc;
    const bool gen = s.S != 0 || s.umode != 0, qstr = s.q_rs != 0;
    auto launch_dq = [&](auto with_delta) {
        constexpr bool WD = decltype(with_delta)::value;
        return for_chunks([&](int len) { return (long)row_units(len, s.Hq / s.Hkv).per * s.Hkv; },
                          [&](const DocTab& t, unsigned nblk) {
                              auto go = [&](auto kern) { kern<<<dim3(nblk), NT, 0, st>>>(q, k, v, out, lse, lse2, dout, delta, dq, s, 0, t); };
                              if (qstr) gen ? go(dq_kernel<D, true, true, true, WD>) : go(dq_kernel<D, false, true, true, WD>);
                              else gen ? go(dq_kernel<D, true, true, false, WD>) : go(dq_kernel<D, false, true, false, WD>);
                          });
    };
    if (free_order && (e = launch_dq(std::true_type{})) != hipSuccess) return e;
    e = for_chunks([&](int len) { const BwdPlan pl = counts(len); return (long)pl.slot0[pl.nseg] * s.Hkv; },
                   [&](const DocTab& t, unsigned nblk) {
                       auto go = [&](auto kern) { kern<<<dim3(nblk), NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, none, t); };
                       if (qstr) gen ? go(dkdv_kernel<D, true, true, true, true>) : go(dkdv_kernel<D, true, false, true, true>);
                       else gen ? go(dkdv_kernel<D, true, true, true>) : go(dkdv_kernel<D, true, false, true>);
                   });
    if (e != hipSuccess) return e;
    constexpr int per_tile = 2 * D * BNK;
    e = for_chunks([&](int len) { return (long)counts(len).n_gt * s.Hkv; },
                   [&](const DocTab& t, unsigned nblk) {
                       gist_reduce_pack_kernel<<<dim3(nblk, (per_tile / 4 + NT - 1) / NT), NT, 0, st>>>(
                           part, comp, s, per_tile, pp.segc, t);
                   });
    if (e != hipSuccess) return e;
    e = for_chunks([&](int len) { return (long)((len + BNK - 1) / BNK) * s.Hkv; },
                   [&](const DocTab& t, unsigned nblk) {
                       auto go = [&](auto kern) { kern<<<dim3(nblk), NT, 0, st>>>(q, k, v, lse2, dout, delta, dk, dv, part, comp, s, none, t); };
                       if (qstr) gen ? go(dkdv_kernel<D, false, true, true, true>) : go(dkdv_kernel<D, false, false, true, true>);
                       else gen ? go(dkdv_kernel<D, false, true, true>) : go(dkdv_kernel<D, false, false, true>);
                   });
    if (e != hipSuccess) return e;
    return free_order ? hipSuccess : launch_dq(std::false_type{});
}

}  // namespace

size_t bwd_mfma_workspace(const AttnShape& s) { return sized_plan(s, pick_segc(launch_steps(s))).total; }
size_t bwd_mfma_least_workspace(const AttnShape& s) { return sized_plan(s, roomiest_segc(launch_steps(s))).total; }

BwdPlan make_bwd_plan(const AttnShape& s) {
    const long steps = launch_steps(s);
    return make_plan(s, steps, SIZE_MAX, pick_segc(steps));
}

size_t bwd_mfma_pack_workspace(const AttnShape& s, const int* cu, int ndocs) { return make_pack_plan(s, cu, ndocs, SIZE_MAX).total; }
size_t bwd_mfma_pack_least_workspace(const AttnShape& s, const int* cu, int ndocs) { return make_pack_plan(s, cu, ndocs, 0).total; }

// A head dimension below the one the kernels are built for goes through the instantiations for explicit strides of
// q, out, dout and dq, with the strides of the dense layout.
static AttnShape with_dense_strides_if_padded(AttnShape s) {
    if (s.D != padded_head_dim(s.D) && s.q_rs == 0) {
        s.q_rs = s.D;
        s.q_hs = (long long)s.qhs * s.D;
        s.q_bs = (long long)s.Hq * s.q_hs;
    }
    return s;
}

hipError_t launch_bwd_mfma_pack(const void* q, const void* k, const void* v, const void* out, const float* lse,
                                const void* dout, void* dq, void* dk, void* dv, void* ws, size_t room,
                                const AttnShape& s_in, const int* cu, int ndocs, hipStream_t st) {
    const AttnShape s = with_dense_strides_if_padded(s_in);
    if (s.D <= 64)
        return bwd_launch_pack<64>((const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, (const bf16_t*)out, lse,
                                   (const bf16_t*)dout, (bf16_t*)dq, (bf16_t*)dk, (bf16_t*)dv, (char*)ws, room, s, cu, ndocs, st);
    return bwd_launch_pack<128>((const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, (const bf16_t*)out, lse,
                                (const bf16_t*)dout, (bf16_t*)dq, (bf16_t*)dk, (bf16_t*)dv, (char*)ws, room, s, cu, ndocs, st);
}

hipError_t launch_bwd_mfma(const void* q, const void* k, const void* v, const void* out, const float* lse,
                           const void* dout, void* dq, void* dk, void* dv, void* ws, size_t room,
                           const AttnShape& s_in, unsigned stages, hipStream_t st) {
    const AttnShape s = with_dense_strides_if_padded(s_in);
    if (s.D <= 64)
        return bwd_launch<64>((const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, (const bf16_t*)out, lse,
                              (const bf16_t*)dout, (bf16_t*)dq, (bf16_t*)dk, (bf16_t*)dv, (char*)ws, room, s, stages, st);
    return bwd_launch<128>((const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, (const bf16_t*)out, lse,
                           (const bf16_t*)dout, (bf16_t*)dq, (bf16_t*)dk, (bf16_t*)dv, (char*)ws, room, s, stages, st);
}

}  // namespace unigist
