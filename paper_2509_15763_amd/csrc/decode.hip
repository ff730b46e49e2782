// Split-K decode over the compressed KV cache (Sec. 4.3 of the paper: after the raw
// tokens outside the window have been dropped, a new token attends to every cached
// key; the paper notes this is compatible with FlashDecoding-style split-K).
//
// The op streams K and V once from HBM: 4 flops per byte, so it is bandwidth bound.
// Three slice kernels share the workspace format and the combine kernel:
//   decode_split_mfma_kernel      bf16 queries, bf16 or E4M3 cache, query groups of up to 15 heads: contractions on
//                                 the matrix cores (described at the kernel);
//   decode_split_kernel           any dtype (the fp32 debug build) and any group size, plain vector arithmetic.
// Layout of the work of the vector kernel:
//   grid = (splits, kv heads or q heads, B), 256 threads.
//   A workgroup owns one contiguous slice of one sequence's keys for one kv head and
//   serves all G = Hq/Hkv query heads of that group from the same K/V bytes.
//   16 lanes share one key row (each holds D/16 contiguous elements, a 16-byte load
//   for bf16 D=128), so a wave covers 4 rows per load and the workgroup's 4 waves
//   cover 16 adjacent rows (4 KB contiguous for bf16 D=128).
//   Each 16-lane group keeps its own running (max, sum, acc) per query head; the 16
//   groups of a workgroup are merged through LDS and the slice's partial result goes
//   to the workspace as (m, l, acc[D]).  A second kernel merges the slices:
//   lse = ln sum_s l_s e^{m_s}, out = sum_s e^{m_s - m} acc_s / sum_s e^{m_s - m} l_s.
#include <algorithm>
#include <type_traits>

#include "mfma_common.h"

namespace unigist {
namespace {

constexpr int kThreads = 256;
constexpr int kLanesPerRow = 16;
constexpr int kRowsPerIter = kThreads / kLanesPerRow;  // 16
constexpr int kUnroll = 4;

template <typename T, int E> struct RowChunk;  // E contiguous elements of a row -> float[E]
template <int E> struct RowChunk<bf16_t, E> {
    static __device__ __forceinline__ void load(const bf16_t* p, float (&x)[E]) {
        if constexpr (E == 8) {
            u32x4 r = *(const u32x4*)p;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                x[2 * t] = __uint_as_float(r[t] << 16);
                x[2 * t + 1] = __uint_as_float(r[t] & 0xffff0000u);
            }
        } else {
            u32x2 r = *(const u32x2*)p;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                x[2 * t] = __uint_as_float(r[t] << 16);
                x[2 * t + 1] = __uint_as_float(r[t] & 0xffff0000u);
            }
        }
    }
};
template <int E> struct RowChunk<float, E> {
    static __device__ __forceinline__ void load(const float* p, float (&x)[E]) {
#pragma unroll
        for (int t = 0; t < E; t += 4) {
            f32x4 r = *(const f32x4*)(p + t);
            x[t] = r[0];
            x[t + 1] = r[1];
            x[t + 2] = r[2];
            x[t + 3] = r[3];
        }
    }
};

// E4M3 codes -> float, two per v_cvt_pk_f32_fp8
template <int E> struct RowChunk<fp8_t, E> {
    static __device__ __forceinline__ void load(const fp8_t* p, float (&x)[E]) {
        uint32_t r[E / 4];
        if constexpr (E == 8) {
            u32x2 t = *(const u32x2*)p;
            r[0] = t[0];
            r[1] = t[1];
        } else {
            r[0] = *(const uint32_t*)p;
        }
#pragma unroll
        for (int t = 0; t < E / 4; ++t) {
            f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)r[t], false);
            f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)r[t], true);
            x[4 * t] = lo[0];
            x[4 * t + 1] = lo[1];
            x[4 * t + 2] = hi[0];
            x[4 * t + 3] = hi[1];
        }
    }
};

// sum over the 16 lanes of a DPP row; every lane ends with the total
__device__ __forceinline__ float row16_sum(float x) {
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xf, 0xf, false));  // row_half_mirror
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xf, 0xf, false));  // row_mirror
    return x;
}

// workspace layout per (b, hq, split): [m, l, acc[D]] floats.
// TQ: type of the queries; T: type the cache is stored in.  A cache of E4M3 codes comes with one scale per kv
// head for K and for V (element = code * scale): the K scale is folded into the query, the V scale into the
// slice's partial result.
// D is the head dimension the kernel is built for (64 or 128), Dt <= D (a multiple of 8) the one of the tensors: rows in
// memory are Dt elements long and the lanes holding columns from Dt on work on zeros; the workspace keeps D columns.
template <typename TQ, typename T, int D, int G, int U>
__global__ __launch_bounds__(kThreads) void decode_split_kernel(const TQ* __restrict__ q, const T* __restrict__ kc,
                                                               const T* __restrict__ vc, const int* __restrict__ seqlens,
                                                               const float* __restrict__ k_scale,
                                                               const float* __restrict__ v_scale,
                                                               float* __restrict__ ws, int Hq, int Hkv, int Lk,
                                                               int nsplit, float scale, int Dt) {
    constexpr int E = D / kLanesPerRow;
    const int tid = threadIdx.x;
    const int sub = tid % kLanesPerRow;  // which D/16 chunk of a row
    const int grp = tid / kLanesPerRow;  // which of the 16 rows per iteration
    const int split = blockIdx.x, b = blockIdx.z;
    // G query heads share kv head hk; with G == 1 the grid runs over query heads
    const int hq0 = blockIdx.y * G;
    const int hk = hq0 / (Hq / Hkv);
    const int n = seqlens ? min(max(seqlens[b], 0), Lk) : Lk;  // never past the sequence's slab, whatever the caller wrote
    const int per = (((n + nsplit - 1) / nsplit) + kRowsPerIter - 1) / kRowsPerIter * kRowsPerIter;
    const int k0 = split * per;
    const int k1 = min(n, k0 + per);
    if (k0 >= k1) {  // a slice without keys
        if (tid < G) *(f32x2*)(ws + (((size_t)b * Hq + hq0 + tid) * nsplit + split) * (D + 2)) = f32x2{-INFINITY, 0.f};
        return;
    }

    float qr[G][E], acc[G][E], m[G], l[G];
    if (k_scale) scale *= k_scale[hk];
    const float vmul = v_scale ? v_scale[hk] : 1.f;
    const bool have = sub * E < Dt;  // does this lane's piece of a row exist?
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
        for (int e = 0; e < E; ++e) qr[g][e] = 0.f;
        if (have) RowChunk<TQ, E>::load(q + ((size_t)b * Hq + hq0 + g) * Dt + sub * E, qr[g]);
        m[g] = -INFINITY;
        l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            qr[g][e] *= scale;
            acc[g][e] = 0.f;
        }
    }
    const T* kb = kc + ((size_t)b * Hkv + hk) * Lk * Dt + (have ? sub * E : 0);  // a lane without a piece re-reads
    const T* vb = vc + ((size_t)b * Hkv + hk) * Lk * Dt + (have ? sub * E : 0);  // the first one; its q is zero

    for (int base = k0; base < k1; base += kRowsPerIter * U) {
        float kx[U][E], vx[U][E];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int row = base + u * kRowsPerIter + grp;
            ok[u] = row < k1;
            int rr = ok[u] ? row : k0;  // k0 < k1 <= n whenever this loop runs: always in bounds
            RowChunk<T, E>::load(kb + (size_t)rr * Dt, kx[u]);
            RowChunk<T, E>::load(vb + (size_t)rr * Dt, vx[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float s = 0.f;
#pragma unroll
                for (int e = 0; e < E; ++e) s += qr[g][e] * kx[u][e];
                s = row16_sum(s);
                if (ok[u]) {
                    if (s > m[g]) {
                        float a = __expf(m[g] - s);
                        l[g] *= a;
#pragma unroll
                        for (int e = 0; e < E; ++e) acc[g][e] *= a;
                        m[g] = s;
                    }
                    float p = __expf(s - m[g]);
                    l[g] += p;
#pragma unroll
                    for (int e = 0; e < E; ++e) acc[g][e] += p * vx[u][e];
                }
            }
        }
    }

    // merge the 16 row groups of the workgroup
    __shared__ float sm[G][kRowsPerIter];
    __shared__ float sl[G][kRowsPerIter];
    __shared__ float sacc[G][kRowsPerIter][D];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (sub == 0) {
            sm[g][grp] = m[g];
            sl[g][grp] = l[g];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) sacc[g][grp][sub * E + e] = acc[g][e];
    }
    __syncthreads();
    for (int idx = tid; idx < G * D; idx += kThreads) {
        const int g = idx / D, d = idx % D;
        float mm = -INFINITY;
#pragma unroll
        for (int t = 0; t < kRowsPerIter; ++t) mm = fmaxf(mm, sm[g][t]);
        float ll = 0.f, a = 0.f;
        if (mm > -INFINITY) {
#pragma unroll
            for (int t = 0; t < kRowsPerIter; ++t) {
                float w = __expf(sm[g][t] - mm);  // exp(-inf) = 0 for groups that saw no key
                ll += w * sl[g][t];
                a += w * sacc[g][t][d];
            }
        }
        float* o = ws + (((size_t)b * Hq + hq0 + g) * nsplit + split) * (D + 2);
        if (d == 0) {
            o[0] = mm;
            o[1] = ll;
        }
        o[2 + d] = a * vmul;
    }
}

// Merge of the slices of one (sequence, query head).  Both kernels are nothing but latency, and most of it the round trip to
// partials that other XCDs have just written, so all loads of a wave are in flight at once; a loop that first looks for
// the maximum and then sums pays two trips.  A slice without keys has m = -inf and leaves its accumulator unwritten: what
// is loaded of it may be anything, NaN included, and must not enter the sum.  A slice with keys enters it also with a
// weight that has underflowed to zero, so that its infinities and NaN reach the result as they would inside one slice.  A
// sequence of zero keys (outside the contract) gets the empty sum, not NaN; columns from Dt on are not in the tensors.

// Up to kFewSlices slices (N = 4 or 8 of them; five to eight slices, four waves / one, us: 1000 keys 8.5 / 8.0, 4 x 4000 ragged 15.9 /
// 15.4): a wave has them all in flight by itself.  Three more waves and their merge through LDS cost a batch
// that the slice kernel fills by itself 2.4 us (slice kernel + combine, us, four waves / one: 128 sequences of up to 500
// E4M3 rows at D = 64 17.7 / 15.1, 256 of 300 bf16 rows at D = 128 69.5 / 64.6, 32 of 1100 33.1 / 32.4).  With more
// slices the second trip costs more than that (24 slices 11.8 / 14.3).
constexpr int kFewSlices = 8;
template <typename T, int D, int N>
__global__ __launch_bounds__(64) void decode_combine_few_kernel(const float* __restrict__ ws, T* __restrict__ out,
                                                               float* __restrict__ lse, int nsplit, int Dt) {
    constexpr int C = D / 64;  // columns per lane
    const int bh = blockIdx.x, lane = threadIdx.x;
    const float* p = ws + (size_t)bh * nsplit * (D + 2);
    f32x2 ml[N];
    float x[N][C];
#pragma unroll
    for (int s = 0; s < N; ++s) {
        const float* ps = p + (size_t)min(s, nsplit - 1) * (D + 2);
        ml[s] = *(const f32x2*)ps;
#pragma unroll
        for (int c = 0; c < C; ++c) x[s][c] = ps[2 + 64 * c + lane];
    }
    float mm = -INFINITY, ll = 0.f, a[C];
#pragma unroll
    for (int s = 0; s < N; ++s) mm = fmaxf(mm, ml[s][0]);  // the last one again where there are fewer
#pragma unroll
    for (int c = 0; c < C; ++c) a[c] = 0.f;
#pragma unroll
    for (int s = 0; s < N; ++s)
        if (s < nsplit && ml[s][0] != -INFINITY) {
            const float w = __expf(ml[s][0] - mm);
            ll += w * ml[s][1];
#pragma unroll
            for (int c = 0; c < C; ++c) a[c] += w * x[s][c];
        }
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (64 * c + lane < Dt) Elem<T>::store(out + (size_t)bh * Dt + 64 * c + lane, mm == -INFINITY ? 0.f : a[c] / ll);
    if (lse && lane == 0) lse[bh] = mm == -INFINITY ? -INFINITY : mm + __logf(ll);
}

// More slices, up to 64: four waves, each taking every fourth slice (the accumulators of up to kBatch slices and, one slice
// per lane, the references of all are in flight).
// Slice kernel + this, us, against a combine kernel that loops over the slices twice: 8000 keys x 8 kv heads 27.6 -> 15.5,
// 20000 keys x 1 kv head 42.1 -> 17.6 (with the slice kernel as it now is 13.8 and 15.6).
template <typename T, int D>
__global__ __launch_bounds__(256) void decode_combine_kernel(const float* __restrict__ ws, T* __restrict__ out,
                                                            float* __restrict__ lse, int nsplit, int Dt) {
    constexpr int kWaves = 4, kBatch = 4, C = D / 64;  // C columns per lane
    const int bh = blockIdx.x, lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float* p = ws + (size_t)bh * nsplit * (D + 2);
    __shared__ float part[kWaves][D];
    const f32x2 ml = lane < nsplit ? *(const f32x2*)(p + (size_t)lane * (D + 2)) : f32x2{-INFINITY, 0.f};  // nsplit <= 64
    float x[kBatch][C];
    auto load = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int s = min(s0 + kWaves * i, nsplit - 1);
#pragma unroll
            for (int c = 0; c < C; ++c) x[i][c] = p[(size_t)s * (D + 2) + 2 + 64 * c + lane];
        }
    };
    load(w);
    const unsigned long long has_keys = __builtin_amdgcn_ballot_w64(ml[0] != -INFINITY);
    float mm = ml[0];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) mm = fmaxf(mm, __shfl_xor(mm, off, 64));
    const float wgt = ml[0] == -INFINITY ? 0.f : __expf(ml[0] - mm);
    float ll = wgt * ml[1];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) ll += __shfl_xor(ll, off, 64);
    float a[C];
#pragma unroll
    for (int c = 0; c < C; ++c) a[c] = 0.f;
    for (int s0 = w; s0 < nsplit; s0 += kWaves * kBatch) {
        if (s0 != w) load(s0);
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int s = s0 + kWaves * i;
            const float ws_ = __shfl(wgt, s < nsplit ? s : 0, 64);
            if (s < nsplit && (has_keys >> s & 1)) {
#pragma unroll
                for (int c = 0; c < C; ++c) a[c] += ws_ * x[i][c];
            }
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) part[w][64 * c + lane] = a[c];
    __syncthreads();
    const int d = threadIdx.x;
    if (d >= Dt) return;
    float r = 0.f;
    if (mm != -INFINITY) r = ((part[0][d] + part[1][d]) + (part[2][d] + part[3][d])) / ll;
    Elem<T>::store(out + (size_t)bh * Dt + d, r);
    if (lse && d == 0) lse[bh] = mm == -INFINITY ? -INFINITY : mm + __logf(ll);
}

template <typename T, int D>
hipError_t launch_combine(const float* ws, T* out, float* lse, int BH, int nsplit, int Dt, hipStream_t st) {
    if (nsplit <= 4) decode_combine_few_kernel<T, D, 4><<<BH, 64, 0, st>>>(ws, out, lse, nsplit, Dt);
    else if (nsplit <= kFewSlices) decode_combine_few_kernel<T, D, kFewSlices><<<BH, 64, 0, st>>>(ws, out, lse, nsplit, Dt);
    else decode_combine_kernel<T, D><<<BH, 256, 0, st>>>(ws, out, lse, nsplit, Dt);
    return hipGetLastError();
}

// where a launch of one slice per sequence writes its results
struct DecodeOut {
    bf16_t* out;
    float* lse;  // may be null
};

// ---------------------------------------------------------------------------------------------
// bf16 queries, cache in bf16 or as E4M3 codes, query groups of up to 15 heads per kv head: the contractions go to the matrix cores
// (v_mfma_f32_16x16x32_bf16; operand layouts in mfma_common.h), which are idle in this bandwidth-bound op, and the
// vector pipe is left with widening the codes (E4M3 values are exact in bf16; nothing to do for a bf16 cache) and a
// softmax over 16-key columns.
// A wave takes 32 keys per iteration, the workgroup's four waves 128:
//   S^T = K Q^T   A = K: lane (key r16, g4) holds D/4 elements of its key's row, eight per k-step (the contraction order is
//                 free as long as Q uses the same one).  bf16 (SEG64): load t takes the 16 bytes at 64 t + 16 g4, so the four
//                 lanes of a row read 64 contiguous bytes per instruction; with D/4 contiguous elements per lane every
//                 16 bytes of an instruction lay in another 64-byte segment, and the loads' address processing cost
//                 5 to 12 % (slice kernel + combine, us, 32/8 heads, D = 128: 1500 keys 9.3 -> 8.9, 4 x 1500 14.1 -> 12.4, 100 x
//                 3000 227 -> 215, 24 x 20000 ragged 218 -> 204; 64 x 17408, near the memory's rate, 752 -> 737; nothing at
//                 D = 64, where a row is 128 bytes).
//                 Rows of a head dimension below D end before the last loads, all of one t then, which repeat the row's start: 13 x 5437 keys at 72 of 128 columns 39.2 -> 46.4 us, at 96 47.1 -> 49.9.  Such rows
//                 keep D/4 contiguous elements per lane (SEG64 = false), where a lane of every load has none.
//                 E4M3: the lane's D/4 codes are two loads that the next lane continues; 64 t + 16 g4 gained nothing.
//                 B = Q^T: column = query head of the group (columns >= G are zero), in registers;
//   softmax       a head is a column spread over four lanes, each holding 4 of every 16 keys; its running
//                 reference is kept identical on the four lanes and raised lazily, the row sum is a per-lane partial;
//   O^T += V^T P^T  P in place as the B operand (slot 8 g4 + 4 kb + i = key 16 kb + 4 g4 + i); V^T through LDS: the
//                 wave widens its 32 V rows to bf16 into a private swizzled tile and reads it back transposed.
// The four waves' partial (m, l, O) are merged through LDS and written to the workspace like the other kernels'.
// AHEAD: the loads of the next 128 keys are issued before the work on these, into registers of their own.  Where one or two
// workgroups share a CU, an iteration is a round trip to memory and then the work, one after the other.  Slice kernel +
// combine, us, without / with: 8 x 12000 ragged 58.6 / 54.4, 16 x 9001 ragged E4M3 43.5 / 41.5, 13 x 5437 at D = 64 35.3 /
// 30.7, 12 x 30000 ragged E4M3, 8/1 heads, D = 64 20.8 / 16.6, 16 x 700 ragged E4M3 11.8 / 10.6.  It is left out where
// - a slice is one iteration (1500 keys, one sequence: 8.7 / 8.8), and
// - bf16 slabs at D = 128 without lengths, all of whose sequences are full, give more than 512 workgroups (64 x 17408 745 / 773) or are
//   longer than 10240 rows: 32 x 17408 380 / 397, 16 x 30000 323 / 327, 8 x 20000 114.3 /
//   115.6, 1 x 131072 94.7 / 95.9 (32 x 9000 200.6 / 197.9, 16 x 6000 71.9 / 71.5; rows of 96 columns gain longer: 10 x 30000, 16/4 heads
//   82.8 / 81.3).  With lengths it stays: they may all be equal, and then it costs 1 % of a long slab (48 x 17408, four slices 555.5 / 560.3)
//   and gains 1 to 6 % of a shorter one (64 x 9000 392 / 387, 100 x 1900 148 / 143), and where they are spread it gains more: 48 x 17408 348
//   / 332, 64 x 9000 253 / 232, 100 x 1900 84 / 81.  One long sequence among short ones gains (48 x 17408 133 / 114) but for short slabs of
//   many sequences, whose short ones load 128 keys too many (100 x 3000 34 / 40, 128 x 512 12.8 / 14.7).
// - more than 512 E4M3 workgroups at D = 128 (three fit a CU instead of four) have short slices: 64 ragged of up to 3000 51.0 / 52.2;
//   64 x 17408 386 / 378, 48 ragged x 20000 231 / 220.
// At D = 64 three bf16 or five E4M3 workgroups fit a CU with it: 64 x 17408 393 / 387, 48 ragged x 4000 49.4 / 47.6.
// Registers with bf16 at D = 128, where none are asked for: 224 and 36 accumulation registers with AHEAD, one workgroup per CU; 158
// and 32 without, two.  How many fit hardly matters with loads ahead: held to two per CU (224 in all), us, one / two: 64 x 17408 equal
// 745.6 / 747.5, spread 428.0 / 427.7, 24 x 17408 equal 289.3 / 289.5, 32 x 17408 spread 231.8 / 221.2, 100 x 3000 one full among eighths
// 40.0 / 42.0.  Three without AHEAD cost 2 to 4 % of a launch of few slices (us with / without: 4 x 1500 keys 12.9 / 12.5, 8000 14.6 /
// 14.0) and 1.5 % of 64 x 17408 (750 / 738).  With the 8-bit cache four are asked for without AHEAD (the compiler's own choice at D =
// 128, 130 VGPRs, allows three).
// DIRECT: a launch of one slice per sequence writes the result itself, as the merge of one slice would, and has no merge (us
// with / without: 120 keys x 8 kv heads 6.8 / 4.8, 100 x 16/4 heads x 200 at D = 64 8.8 / 6.4, 128 x 300 36.5 / 32.8, 128 x 3000
// 274 / 268).
template <int D, bool E4M3, bool SEG64, bool AHEAD, bool DIRECT>
__global__ __launch_bounds__(kThreads, E4M3 ? (AHEAD ? 3 : 4) : 1) void decode_split_mfma_kernel(const bf16_t* __restrict__ q,
                                                                         const uint8_t* __restrict__ kc,
                                                                         const uint8_t* __restrict__ vc,
                                                                         const int* __restrict__ seqlens,
                                                                         const float* __restrict__ k_scale,
                                                                         const float* __restrict__ v_scale,
                                                                         float* __restrict__ ws, int Hq, int Hkv, int Lk,
                                                                         int nsplit, float scale, int Dt,
                                                                         std::conditional_t<DIRECT, DecodeOut, NoDocs> res) {
    // Dt <= D: the head dimension of the tensors (rows of Dt elements in memory; a multiple of 8, of 16 for E4M3
    // codes); the K and Q columns from Dt on are zeros, the V columns from Dt on are never stored
    constexpr int KS = D / 32, DB = D / 16, CH = D / 8;  // k-steps, 16-row blocks of O^T, 16-byte chunks per bf16 row
    constexpr int EB = E4M3 ? 1 : 2;                     // bytes per cache element
    constexpr int BPL = D / 4;                           // K elements per lane and key
    constexpr int NKL = BPL * EB / 16;                   // 16-byte loads per lane and key for them
    constexpr int NLV = 32 * D * EB / 1024;              // 16-byte loads per lane for the wave's 32 V rows
    constexpr int LPR = D * EB / 16;                     // lanes per V row
    constexpr float kLog2e = 1.4426950408889634f;
    constexpr float kSlack = 8.f;                        // the reference is raised when a score exceeds it by 2^kSlack
    __shared__ __attribute__((aligned(1024))) char smem[4 * 32 * D * 2];  // per wave: 32 rows of D bf16

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int r16 = lane & 15, g4 = lane >> 4;
    const int G = Hq / Hkv;  // <= 15: the merge buffer below holds 4 G (D + 2) floats
    const int split = blockIdx.x, b = blockIdx.z, hk = blockIdx.y, hq0 = hk * G;
    const int n = seqlens ? min(max(seqlens[b], 0), Lk) : Lk;  // never past the sequence's slab, whatever the caller wrote
    const int per = (((n + nsplit - 1) / nsplit) + 127) / 128 * 128;
    const int k0 = split * per;
    const int k1 = min(n, k0 + per);
    if (k0 >= k1) {  // a slice without keys
        if constexpr (DIRECT) {
            for (int i = tid; i < G * Dt; i += kThreads) res.out[((size_t)b * Hq + hq0) * Dt + i] = 0;
            if (res.lse && tid < G) res.lse[(size_t)b * Hq + hq0 + tid] = -INFINITY;
        } else if (tid < G) {
            *(f32x2*)(ws + (((size_t)b * Hq + hq0 + tid) * nsplit + split) * (D + 2)) = f32x2{-INFINITY, 0.f};
        }
        return;
    }
    const float c = scale * (E4M3 ? k_scale[hk] : 1.f) * kLog2e;  // exp(x) = exp2(x log2 e); the K scale rides along

    // B operand Q^T: lane (column r16 = head of the group, g4) holds the eight elements of its head that K's k-step has
    bf16x8 qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        u32x4 z = {0u, 0u, 0u, 0u};
        const int e = SEG64 ? 32 * ks + 8 * g4 : BPL * g4 + 8 * ks;
        if (r16 < G && e < Dt) z = *(const u32x4*)(q + ((size_t)b * Hq + hq0 + r16) * Dt + e);
        qf[ks] = __builtin_bit_cast(bf16x8, z);
    }
    f32x4 o[DB];  // O^T: register i of o[db] is d = 16 db + 4 g4 + i, column = head r16
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = zero4();
    float m = -INFINITY, l = 0.f;

    const uint8_t* kb = kc + ((size_t)b * Hkv + hk) * Lk * (Dt * EB);
    const uint8_t* vb = vc + ((size_t)b * Hkv + hk) * Lk * (Dt * EB);
    const int row_bytes = Dt * EB;
    char* vt = smem + w * (32 * D * 2);
    int toff[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) toff[db] = tr16_lane_off16<CH>(db);
    // where this lane's V loads go in the tile: load j covers row (64 / LPR) j + lane / LPR and 16 bytes of it -- 16
    // codes, i.e. the bf16 chunks 2 (lane % LPR) and 2 (lane % LPR) + 1 of that row, or the bf16 chunk lane % LPR itself
    constexpr int NVW = E4M3 ? 2 : 1;
    int vwoff[NLV][NVW];
#pragma unroll
    for (int j = 0; j < NLV; ++j) {
        const int row = (64 / LPR) * j + lane / LPR;
#pragma unroll
        for (int t = 0; t < NVW; ++t)
            vwoff[j][t] = row * (CH * 16) + (((NVW * (lane % LPR) + t) ^ swz16<CH>(row)) << 4);
    }

    // ---- loads: K rows base + 16 kb + r16 (clamped into the slice: clamped keys are masked below), V rows likewise
    struct Tile {
        u32x4 kw[2][NKL], vw[NLV];
    };
    auto load = [&](Tile& x, int base) __attribute__((always_inline)) {
#pragma unroll
        for (int kb2 = 0; kb2 < 2; ++kb2) {
            const int row = min(base + 16 * kb2 + r16, k1 - 1);
#pragma unroll
            for (int t = 0; t < NKL; ++t) {
                const int o = SEG64 ? 64 * t + 16 * g4 : BPL * EB * g4 + 16 * t;  // a piece the rows do not have: the first one (its q is zero)
                x.kw[kb2][t] = *(const u32x4*)(kb + (size_t)row * row_bytes + (o < row_bytes ? o : 0));
            }
        }
#pragma unroll
        for (int j = 0; j < NLV; ++j) {
            const int row = min(base + (64 / LPR) * j + lane / LPR, k1 - 1);
            const int o = 16 * (lane % LPR);
            x.vw[j] = *(const u32x4*)(vb + (size_t)row * row_bytes + (o < row_bytes ? o : 0));
        }
    };
    auto step = [&](const Tile& x, int base) __attribute__((always_inline)) {
        const auto& kw = x.kw;
        const auto& vw = x.vw;
#include "decode_step.inc"
    };
    if constexpr (AHEAD) {
        Tile ta, tb;
        int base = k0 + 32 * w;
        if (base < k1) {
            load(ta, base);
            for (;;) {  // the loads behind the last keys repeat the last row: a branch around them would make the compiler wait for all
                load(tb, base + 128);
                step(ta, base);
                if ((base += 128) >= k1) break;
                load(ta, base + 128);
                step(tb, base);
                if ((base += 128) >= k1) break;
            }
        }
    } else {
        for (int base = k0 + 32 * w; base < k1; base += 128) {
            u32x4 kw[2][NKL], vw[NLV];
#pragma unroll
            for (int kb2 = 0; kb2 < 2; ++kb2) {
                const int row = min(base + 16 * kb2 + r16, k1 - 1);
#pragma unroll
                for (int t = 0; t < NKL; ++t) {
                    const int o = SEG64 ? 64 * t + 16 * g4 : BPL * EB * g4 + 16 * t;
                    kw[kb2][t] = *(const u32x4*)(kb + (size_t)row * row_bytes + (o < row_bytes ? o : 0));
                }
            }
#pragma unroll
            for (int j = 0; j < NLV; ++j) {
                const int row = min(base + (64 / LPR) * j + lane / LPR, k1 - 1);
                const int o = 16 * (lane % LPR);
                vw[j] = *(const u32x4*)(vb + (size_t)row * row_bytes + (o < row_bytes ? o : 0));
            }
#include "decode_step.inc"
        }
    }

    // ---- merge the four waves (the tiles are dead: their memory takes the partials)
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    __syncthreads();
    float* pm = (float*)smem;              // [4 waves][G]
    float* pl = pm + 4 * G;                // [4 waves][G]
    float* po = pl + 4 * G;                // [4 waves][G][D]
    if (r16 < G) {
        if (g4 == 0) {
            pm[w * G + r16] = m;
            pl[w * G + r16] = l;
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) po[((size_t)w * G + r16) * D + 16 * db + 4 * g4 + i] = o[db][i];
    }
    __syncthreads();
    const float vmul = E4M3 ? v_scale[hk] : 1.f;
    const float ln2 = 0.6931471805599453f;
    for (int idx = tid; idx < G * D; idx += kThreads) {
        const int g = idx / D, d = idx % D;
        float mm = -INFINITY;
#pragma unroll
        for (int t = 0; t < 4; ++t) mm = fmaxf(mm, pm[t * G + g]);
        float ll = 0.f, a = 0.f;
        if (mm > -INFINITY) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float wgt = __builtin_amdgcn_exp2f((pm[t * G + g] - mm) * c);  // exp2(-inf) = 0 for a wave that saw no key
                ll += wgt * pl[t * G + g];
                a += wgt * po[((size_t)t * G + g) * D + d];
            }
        }
        if constexpr (DIRECT) {
            const size_t row = (size_t)b * Hq + hq0 + g;
            const float mn = mm * c * ln2;
            if (d < Dt) Elem<bf16_t>::store(res.out + row * Dt + d, mn == -INFINITY ? 0.f : a * vmul / ll);
            if (d == 0 && res.lse) res.lse[row] = mn == -INFINITY ? -INFINITY : mn + __logf(ll);
            continue;
        }
        float* outp = ws + (((size_t)b * Hq + hq0 + g) * nsplit + split) * (D + 2);
        if (d == 0) {
            outp[0] = mm * c * ln2;  // the other kernels keep m in natural-log units of the scaled score
            outp[1] = ll;
        }
        outp[2 + d] = a * vmul;
    }
}

template <typename TQ, typename T, int D>
hipError_t decode_launch(const void* q, const void* kc, const void* vc, const float* k_scale, const float* v_scale,
                         void* out, float* lse, int B, int Hq, int Hkv, int Lk, const int* seqlens, int Dt, float* ws,
                         size_t room, hipStream_t st) {
    constexpr int U = kUnroll;
    constexpr unigist_dtype dt = std::is_same<TQ, float>::value ? UNIGIST_F32 : UNIGIST_BF16;
    const int nsplit = decode_num_splits(B, Hq, Hkv, Lk, Dt, dt, room, seqlens != nullptr);
    const float scale = 1.0f / sqrtf((float)Dt);
    if (decode_grouped(Hq, Hkv, dt) && Hq / Hkv == 4) {
        dim3 grid(nsplit, Hkv, B);
        decode_split_kernel<TQ, T, D, 4, U><<<grid, kThreads, 0, st>>>((const TQ*)q, (const T*)kc, (const T*)vc, seqlens,
                                                                       k_scale, v_scale, ws, Hq, Hkv, Lk, nsplit, scale, Dt);
    } else {
        dim3 grid(nsplit, Hq, B);
        decode_split_kernel<TQ, T, D, 1, U><<<grid, kThreads, 0, st>>>((const TQ*)q, (const T*)kc, (const T*)vc, seqlens,
                                                                       k_scale, v_scale, ws, Hq, Hkv, Lk, nsplit, scale, Dt);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_combine<TQ, D>(ws, (TQ*)out, lse, B * Hq, nsplit, Dt, st);
}

}  // namespace

// Does one workgroup serve all query heads of a kv head?  The matrix-core kernel takes groups of up to 15 heads
// (bf16 queries); the vector kernel, which the fp32 build uses, shares the K/V bytes for groups of 4 only.
bool decode_grouped(int Hq, int Hkv, unigist_dtype dt) {
    const int G = Hq / Hkv;
    return dt == UNIGIST_F32 ? G == 4 : G <= 15;
}

// Slices per sequence.  The slice kernel saturates HBM with one workgroup per CU, so the time of a launch goes
// with the number of rounds of 256 workgroups times the slice length: the split is chosen to fill whole rounds
// (a batch of 48 sequences x 8 kv heads = 384 workgroups would leave half of the second round idle), with a
// small price per slice for the partial results the combine kernel has to merge, and never slices shorter than
// 256 keys -- 128, one iteration of the kernel, where up to 64 (sequence, head) units leave most of the chip idle: both
// kernels for 1500 keys x 8 kv heads 10.5 -> 8.9 us, 300 keys 8.9 -> 7.6, 8 x 500 keys 11.1 -> 9.6.  Measured on batches of
// 1 to 256 sequences: one round is best up to 64 (sequence, head) units, two up to 256 units, four beyond.  A workspace too small for the shorter slices (whose size would otherwise fall where a batch
// passes 64 units, so that a loop that sized its buffer for 9 to 12 sequences could not run 8) is served with 256 keys.
namespace {
long decode_units(int B, int Hq, int Hkv, unigist_dtype dt) { return (long)B * (decode_grouped(Hq, Hkv, dt) ? Hkv : Hq); }

int best_splits(long units, int Lk, int min_keys) {
    const long target = units <= 64 ? 256 : units <= 256 ? 512 : 1024;
    long nmax = (target + units - 1) / units;
    if (nmax < 4) nmax = 4;
    if (nmax > 64) nmax = 64;
    const long cap = (Lk + min_keys - 1) / min_keys;
    if (nmax > cap) nmax = cap;
    if (nmax < 1) nmax = 1;
    int best = 1;
    double best_cost = 1e30;
    for (long n = 1; n <= nmax; ++n) {
        const long wgs = units * n;
        double cost = (double)((wgs + 255) / 256 * 256) / (double)wgs * (1.0 + 0.01 * (double)n);
        if (wgs < target) cost *= 1.05;
        if (cost < best_cost) {
            best_cost = cost;
            best = (int)n;
        }
    }
    return best;
}
int base_splits(long units, int Lk) { return best_splits(units, Lk, units <= 64 ? 128 : 256); }  // at least as many as with 256 keys

// One slice of the matrix-core kernel, which then writes the result itself, saves the merge and its launch, 2 to 4 us, and the
// partial results.  It pays up to three iterations, and longer where the (sequence, kv head) units fill the chip by themselves, the
// more so when they fill whole rounds of 256 workgroups (us, slices by the rule above / one; 32/8 heads: 8 units a sequence):
//   1 x 300  7.7 /  7.2    1 x 450   7.5 /  8.6    8 x 300 9.2 / 8.4     8 x 500  9.8 / 10.5    16 x 300 11.6 / 9.7   16 x 900 17.3 / 17.9
//   24 x 640 ragged 15.2 / 12.7    32 x 1000 29.1 / 26.9    32 x 2200 ragged 38.9 / 37.8     48 x 1500 58.5 / 59.6    48 x 2500 ragged 60 / 65
//   64 x 600 ragged 27.3 / 21.1    64 x 4000 189 / 181      100 x 1200 ragged 66.6 / 56.4    100 x 2500 189 / 195
//   E4M3: 32 x 500 15.0 / 10.8, 64 x 2000 56 / 50.5, 100 x 1200 ragged 38.0 / 33.5;  D = 64: 64 x 1500, 16/4 heads 24.0 / 21.0
// Ragged there: spread evenly from a sixteenth of Lk to Lk.  One full sequence among others of an eighth is walked by one workgroup per
// kv head, which shows where a slab has 2000 rows and more, and gains elsewhere (us, slices by the rule above / one, for all equal |
// spread | one full):
//   32 x 2048  51.8 / 47.0 | 39 / 33.4 | 23 / 25.5         64 x 1500  73.4 / 67.9 | 53 / 47 | 21.1 / 21.9
//   64 x 2048  98.3 / 92.1 | 68.8 / 63.4 | 24.6 / 28.0     64 x 2500  115 / 110 | 77.7 / 75.6 | 30.4 / 33.5
//   64 x 3000   136 / 132 | 89 / 88 | 32.7 / 39.2          64 x 4096   183 / 177 | 121 / 121 | 40.1 / 52.0
//   64 x 4096, D = 64  95 / 91 | 61 / 62 | 23 / 27          64 x 4096, E4M3  99.5 / 92 | 68 / 64 | 30.8 / 35.6
//   24 x 576   17.5 / 13.1 | 12.9 / 10.1 | 10.2 / 9.3      128 x 2048  184 / 179 | 123 / 114 | 48.0 / 40.1
// So bf16 rows of 128 columns with lengths stay one slice up to 2560 rows: further on the spread ones gain nothing and one full sequence
// loses 16 to 30 %.  D = 64 (where loads ahead made up for it: 27 before those too) and E4M3 keep the line that full sequences have.
// Sizes are asked for and refused by the slices of the other rules.
bool one_slice(long units, int Lk, bool wide_lengths) {
    const bool whole_rounds = (units + 255) / 256 * 256 <= units * 1.05;
    return Lk <= 384 || (units >= 128 && Lk <= (whole_rounds ? 8 : 3) * units && Lk <= (units > 512 ? 2048 : wide_lengths ? 2560 : 4096));
}

// Slices of a long bf16 slab (from 8192 rows) with lengths.  Lengths may differ, and then more slices let the workgroups of the longest
// sequences end less late; they may be equal as well, and then every round of workgroups costs 2 to 3 us and one that is not filled
// much more, while the launch has no tail to gain.  So: as many slices as fill one round of 512 workgroups up to
// 128 units, two up to 256, four beyond; or eight, where those fill rounds of 256 better.  Where the slices by the rule above fill
// their rounds already, they are two for one and six for two to four, whose rounds cost equal lengths 2 % at most; from 16384 rows of
// 128 columns on, where six cost 1 to 3 %, four for one or two, six for three, up to 4096 workgroups; below 16384 rows of
// 64 columns, where six cost 2 to 4 %, and beyond 512 units that do not fill their rounds, no more than those.  us, rule above without
// loads ahead / eight slices, or the most up to 4096 workgroups / this:
//                                   lengths all equal    spread from 1/16 to 1    one full, the others an eighth
//   12 x 17408 (5 / 8 / 8)           151 / 150 / 149      119 / 101 / 101           66 /  47 /  47
//   24 x 17408 (4 / 8 / 8)           281 / 288 / 288      196 / 172 / 172           83 /  62 /  62
//   18 x 17408 (3 / 8 / 7)           228 / 227 / 221      178 / 142 / 140           76 /  52 /  47
//   13 x 17408 (2 / 8 / 4)           155 / 173 / 160      136 / 105 / 100          123 /  48 /  59
//   10 x 30000 (3 / 8 / 6)           205 / 220 / 209      163 / 137 / 149          123 /  63 /  70
//   16 x 17408 (4 / 8 / 4)           198 / 202 / 199      130 / 120 / 124           80 /  55 /  69
//   32 x 17408 (2 / 8 / 4)           389 / 393 / 389      247 / 226 / 234          146 /  74 /  90
//   32 x 12000 (2 / 8 / 6)           267 / 269 / 268      185 / 157 / 158           89 /  51 /  48
//   64 x 9000 (2 / 8 / 6)            391 / 405 / 396      256 / 231 / 229          105 /  85 /  66
//   64 x 16000 (2 / 8 / 6)           687 / 703 / 692      431 / 391 / 388          187 / 114 / 123
//   16 x 12000 (4 / 8 / 6)           138 / 138 / 139       96 /  84 /  86           44 /  36 /  35
//   48 x 12000 (4 / 8 / 6)           394 / 401 / 400      251 / 229 / 226           87 /  72 /  65
//   85 x 9000, 16/4 (3 / 8 / 6)      264 / 273 / 266      186 / 160 / 159           61 /  58 /  41
//   64 x 17408, D 64 (2 / 8 / 6)     378 / 383 / 381      238 / 221 / 221          103 /  65 /  59
//   128 x 9000, D 64 (1 / 4 / 2)     389 / 400 / 388      258 / 231 / 234          105 /  59 /  70
//   64 x 17408 (2 / 8 / 4)           749 / 762 / 749      455 / 429 / 438          205 / 131 / 134
//   80 x 17408 (2 / 6 / 4)           966 / 972 / 961      606 / 520 / 533          229 / 148 / 154
//   100 x 30000, 8/1 (5 / 8 / 5)     271 / 299 / 272      178 / 166 / 167           81 /  64 /  72
// Equal lengths lose 2 % at most to the rule above but for 3 in few places (24 x 17408, where four slices would take 283, 175 and
// 75; 10 x 30000; 37 x 9000, 16/4 heads, D 64 65 / 67; 16 x 40000 432 / 450 / 452 on one card, 431 / 439 / 435 on another).
// rows: of 128 columns, a row of 64 being half of one
int uneven_splits(long units, int base, long rows) {
    auto fill = [&](int n, long round) { return (double)(units * n) / (double)((units * n + round - 1) / round * round); };
    if (units >= 512 || fill(base, 512) >= 0.95) {
        if (rows < 16384) {
            if (base == 1) return units <= 2048 ? 2 : 1;
            return base <= 4 && units <= 512 && rows >= 8192 ? 6 : base;
        }
        const long more = base < 3 ? 4 : base == 3 ? 6 : base;
        return std::max(base, (int)std::min(more, 4096 / units));
    }
    const int n = std::max(base, (int)((units <= 128 ? 512 : units <= 256 ? 1024 : 2048) / units));
    return units < 384 && fill(8, 256) > fill(n, 256) ? 8 : n;
}
}  // namespace

int decode_least_splits(int B, int Hq, int Hkv, int Lk, unigist_dtype dt) { return best_splits(decode_units(B, Hq, Hkv, dt), Lk, 256); }

// E4M3 codes, half the bytes, keep the slices by the general rule: eight cost equal lengths 2 to 4 % and do not reliably help spread
// ones (us, rule / eight: 64 x 17408 379 / 393 equal, 229 / 231 spread; 16 x 9001 56.0 / 57.4, 39.5 / 40.5; 48 x 20000 335 / 341, 213 /
// 203).  So do slabs without lengths, all of whose sequences are full.
//
// The additional slices are as many as `room` holds, and no more than the built-in scratch array holds where the slices by the rule
// above fit it: a call on that array and one on a workspace of the size asked for then sum alike, to the last bit.
int decode_num_splits(int B, int Hq, int Hkv, int Lk, int D, unigist_dtype dt, size_t room, bool lengths) {
    const long units = decode_units(B, Hq, Hkv, dt);
    const int base = base_splits(units, Lk);
    auto bytes = [&](int n) { return decode_split_bytes(B, Hq, n, D); };
    if (lengths && dt == UNIGIST_BF16 && decode_grouped(Hq, Hkv, dt) && Lk >= 8192 && units >= 64) {
        const int want = uneven_splits(units, base, (long)Lk * padded_head_dim(D) / 128);
        const size_t most = bytes(base) <= UNIGIST_DECODE_NOALLOC_SCRATCH_BYTES ? std::min(room, (size_t)UNIGIST_DECODE_NOALLOC_SCRATCH_BYTES) : room;
        for (int n = want; n > base; --n)
            if (bytes(n) <= most) return n;
    }
    return bytes(base) <= room ? base : decode_least_splits(B, Hq, Hkv, Lk, dt);
}

namespace {
// bf16 queries over a bf16 or E4M3 cache: the matrix-core kernel when the group fits its columns, else one
// workgroup per query head with the vector kernel
template <bool E4M3>
hipError_t decode_bf16q(const void* q, const void* kc, const void* vc, const float* k_scale, const float* v_scale, void* out,
                        float* lse, int B, int Hq, int Hkv, int Lk, const int* seqlens, int D, float* ws, size_t room, hipStream_t st) {
    if (!decode_grouped(Hq, Hkv, UNIGIST_BF16)) {
        using T = std::conditional_t<E4M3, fp8_t, bf16_t>;
        return D <= 64 ? decode_launch<bf16_t, T, 64>(q, kc, vc, k_scale, v_scale, out, lse, B, Hq, Hkv, Lk, seqlens, D, ws, room, st)
                       : decode_launch<bf16_t, T, 128>(q, kc, vc, k_scale, v_scale, out, lse, B, Hq, Hkv, Lk, seqlens, D, ws, room, st);
    }
    const int nsplit = one_slice(decode_units(B, Hq, Hkv, UNIGIST_BF16), Lk, seqlens && !E4M3 && D > 64) ? 1
                       : decode_num_splits(B, Hq, Hkv, Lk, D, E4M3 ? UNIGIST_E4M3 : UNIGIST_BF16, room, seqlens != nullptr);
    const float scale = 1.0f / sqrtf((float)D);
    const dim3 grid(nsplit, Hkv, B);
    const bool seg64 = D == padded_head_dim(D);
    const int slice = (Lk + nsplit - 1) / nsplit;  // see AHEAD at the kernel
    const bool two_per_cu = (long)B * Hkv * nsplit <= 512;
    const bool ahead = slice > 128 && (D <= 64 || (E4M3 ? two_per_cu || slice >= 4096 : seqlens || (two_per_cu && (!seg64 || Lk <= 10240))));
    auto pick = [&](auto ah, auto direct, auto res) {
        constexpr bool A = decltype(ah)::value, R = decltype(direct)::value;
        auto go = [&](auto kern) {
            kern<<<grid, kThreads, 0, st>>>((const bf16_t*)q, (const uint8_t*)kc, (const uint8_t*)vc, seqlens, k_scale, v_scale, ws, Hq,
                                            Hkv, Lk, nsplit, scale, D, res);
        };
        if (D <= 64) seg64 ? go(decode_split_mfma_kernel<64, E4M3, !E4M3, A, R>) : go(decode_split_mfma_kernel<64, E4M3, false, A, R>);
        else seg64 ? go(decode_split_mfma_kernel<128, E4M3, !E4M3, A, R>) : go(decode_split_mfma_kernel<128, E4M3, false, A, R>);
        return hipGetLastError();
    };
    const std::true_type yes;
    const std::false_type no;
    // A merge writes out and lse behind all reads of the slice kernel.  The direct write does not: where either lies on an input, the
    // merge stays, but for an out in q's very place, whose rows a workgroup has all read itself.
    const size_t q_bytes = (size_t)B * Hq * D * 2, slab_bytes = (size_t)B * Hkv * Lk * D * (E4M3 ? 1 : 2);
    auto on_inputs = [&](const void* dst, size_t bytes, bool own_rows) {
        auto meets = [&](const void* x, size_t n) { return dst && x && (uintptr_t)x < (uintptr_t)dst + bytes && (uintptr_t)dst < (uintptr_t)x + n; };
        return (!own_rows && meets(q, q_bytes)) || meets(kc, slab_bytes) || meets(vc, slab_bytes) || meets(seqlens, (size_t)B * sizeof(int)) ||
               meets(k_scale, (size_t)Hkv * sizeof(float)) || meets(v_scale, (size_t)Hkv * sizeof(float));
    };
    if (nsplit == 1 && !on_inputs(out, q_bytes, out == q) && !on_inputs(lse, (size_t)B * Hq * sizeof(float), false)) {
        const DecodeOut res{(bf16_t*)out, lse};
        return ahead ? pick(yes, yes, res) : pick(no, yes, res);
    }
    const hipError_t e = ahead ? pick(yes, no, NoDocs{}) : pick(no, no, NoDocs{});
    if (e != hipSuccess) return e;
    return D <= 64 ? launch_combine<bf16_t, 64>(ws, (bf16_t*)out, lse, B * Hq, nsplit, D, st)
                   : launch_combine<bf16_t, 128>(ws, (bf16_t*)out, lse, B * Hq, nsplit, D, st);
}
}  // namespace

hipError_t launch_decode(const void* q, const void* kc, const void* vc, void* out, float* lse, int B, int Hq,
                         int Hkv, int Lk, const int* seqlens, int D, unigist_dtype dt, float* ws, size_t room,
                         hipStream_t st) {
    if (dt == UNIGIST_F32)
        return D <= 64 ? decode_launch<float, float, 64>(q, kc, vc, nullptr, nullptr, out, lse, B, Hq, Hkv, Lk, seqlens, D, ws, room, st)
                       : decode_launch<float, float, 128>(q, kc, vc, nullptr, nullptr, out, lse, B, Hq, Hkv, Lk, seqlens, D, ws, room, st);
    return decode_bf16q<false>(q, kc, vc, nullptr, nullptr, out, lse, B, Hq, Hkv, Lk, seqlens, D, ws, room, st);
}

hipError_t launch_decode_fp8(const void* q, const void* kc, const void* vc, const float* k_scale, const float* v_scale,
                             void* out, float* lse, int B, int Hq, int Hkv, int Lk, const int* seqlens, int D,
                             float* ws, size_t room, hipStream_t st) {
    return decode_bf16q<true>(q, kc, vc, k_scale, v_scale, out, lse, B, Hq, Hkv, Lk, seqlens, D, ws, room, st);
}

// ---------------------------------------------------------------------------------------------
// Quantisation of new cache rows: y = e4m3(clamp(x / scale[head], -448, 448)), one correctly rounded binary32
// division per element, conversion by v_cvt_pk_fp8_f32 (round to nearest even).  16 elements per lane.
namespace {
template <typename T>
__global__ __launch_bounds__(256) void quantize_e4m3_kernel(const T* __restrict__ x, uint8_t* __restrict__ y,
                                                           const float* __restrict__ scale, int H, long per_head,
                                                           long nchunks) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= nchunks) return;
    const long e0 = idx * 16;
    const float c = scale[(e0 / per_head) % H];
    float f[2][8];
    RowChunk<T, 8>::load(x + e0, f[0]);
    RowChunk<T, 8>::load(x + e0 + 8, f[1]);
    u32x4 w;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float g[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float q = __fdiv_rn(f[t / 2][4 * (t % 2) + i], c);
            g[i] = q != q ? q : fminf(fmaxf(q, -448.f), 448.f);
        }
        int p = 0;
        p = __builtin_amdgcn_cvt_pk_fp8_f32(g[0], g[1], p, false);
        p = __builtin_amdgcn_cvt_pk_fp8_f32(g[2], g[3], p, true);
        w[t] = (uint32_t)p;
    }
    *(u32x4*)(y + e0) = w;
}
// E4M3 codes -> the same values in bf16 (exact: 3 mantissa bits, exponents well inside bf16's), 16 per lane.
// Lane idx covers the elements 16 idx .. 16 idx + 15 of the output, whose slabs hold `rows` of the input slab's `cap` rows.
__global__ __launch_bounds__(256) void widen_e4m3_kernel(const uint8_t* __restrict__ x, bf16_t* __restrict__ y,
                                                        long per_slab_out, long per_slab_in, long nchunks) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= nchunks) return;
    const long e0 = idx * 16;
    const long slab = e0 / per_slab_out, within = e0 % per_slab_out;
    const u32x4 w = *(const u32x4*)(x + slab * per_slab_in + within);
    u32x4 lo, hi;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[t], false), b = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[t], true);
        const uint32_t p0 = pack_bf16x2(a[0], a[1]), p1 = pack_bf16x2(b[0], b[1]);
        if (t < 2) {
            lo[2 * t] = p0;
            lo[2 * t + 1] = p1;
        } else {
            hi[2 * (t - 2)] = p0;
            hi[2 * (t - 2) + 1] = p1;
        }
    }
    *(u32x4*)(y + e0) = lo;
    *(u32x4*)(y + e0 + 8) = hi;
}
}  // namespace

hipError_t launch_widen_e4m3(const void* codes, void* y, int BH, int cap, int rows, int D, hipStream_t st) {
    const long per_out = (long)rows * D, per_in = (long)cap * D;
    const long nchunks = (long)BH * per_out / 16;
    if (nchunks <= 0) return hipSuccess;
    const long blocks = (nchunks + 255) / 256;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    widen_e4m3_kernel<<<dim3((unsigned)blocks), 256, 0, st>>>((const uint8_t*)codes, (bf16_t*)y, per_out, per_in, nchunks);
    return hipGetLastError();
}

hipError_t launch_quantize_e4m3(const void* x, void* y, const float* scale, int B, int H, int n, int D,
                                unigist_dtype dt_in, hipStream_t st) {
    const long per_head = (long)n * D;
    const long nchunks = (long)B * H * per_head / 16;
    if (nchunks <= 0) return hipSuccess;
    const long blocks = (nchunks + 255) / 256;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    if (dt_in == UNIGIST_F32)
        quantize_e4m3_kernel<float><<<dim3((unsigned)blocks), 256, 0, st>>>((const float*)x, (uint8_t*)y, scale, H, per_head, nchunks);
    else
        quantize_e4m3_kernel<bf16_t><<<dim3((unsigned)blocks), 256, 0, st>>>((const bf16_t*)x, (uint8_t*)y, scale, H, per_head, nchunks);
    return hipGetLastError();
}

}  // namespace unigist
