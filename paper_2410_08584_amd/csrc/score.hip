// Probe-token importance scores (supplementary Eq. (A); Eq. (6), Eq. (8);
// Algorithm 1 steps 2-4).  The m x n probe attention matrix is never stored:
//   pass 1  row statistics: for each (head, probe row) the sum of exp2 of the
//           masked, scaled logits over the chunk of keys a workgroup owns (one
//           number per row and chunk, or two where it is out of range);
//   pass 2  merges the numbers of its rows into one exponent offset per
//           row (in its prologue: no launch in between), recomputes the
//           logits, normalises them with that offset, sums them down the probe
//           rows and over the query heads of the group, and writes mass / rank.
// Both passes share one kernel body.  A workgroup owns a chunk of keys of one
// KV head and streams it through LDS in stages of 16 or 32 KiB, loaded straight from
// global memory (no staging registers), three stages ahead.  The work of a stage
// is a grid of 32-key x 32-probe tiles, one 32x32 MFMA accumulator each.  A
// wave owns one (query head, block of 32 probe rows) - its "task" - for the
// whole kernel: the probe rows' fragments stay in its registers, and the key
// fragments of a tile come from LDS.  With few tasks (one query head per KV
// head) several waves share a task and split the key blocks of a stage; more
// tasks are dealt to several workgroups in pass 1 (row_stats_plan), and taken in
// rounds, the chunk streamed once for each, in pass 2.
// Pass 1 computes K Q^T (lane = probe column: row statistics stay in the
// lane); pass 2 computes Q K^T (lane = key column: column sums stay in the
// lane, the tasks' sums of a stage meet in LDS and are added in task order, so
// the result does not depend on scheduling).
#include <algorithm>
#include <atomic>
#include <cfloat>
#include <type_traits>

#include "launch.h"
#include "ldsload.h"

namespace zipvl {

constexpr int kMaxGroup = 16;
constexpr int kSumStages = 8;               // stages whose scores are written at a time
constexpr int kStageBufs = 4;               // stage buffers in LDS: three stages are in flight while one is worked on

// What bounds it: long chunks of one query head per KV head memory; the others a chain (positions, probe rows and statistics, first keys: 4 to 7 of
// the 12 to 19 us of a launch) and then about 600 cycles a tile, products and vector work one after the other (done between the products of the
// next tile instead, as in the exact scores, a tile took 15 % longer: four waves a SIMD, a barrier every one to four tiles).  us, rows gathered by
// lanes behind three stages of keys, pairs of statistics, scores made by the last waves -> now: 40 heads, n = 4096, 64 recent and 64 random
// probes 37.2 -> 31.8; 28 on 4, n = 18432 35.0 -> 32.6; 32, n = 3072 19.7 -> 17.0; 32, n = 20000, m = 128 78.6 -> 67.5; 28 on 4, fp32, n = 12000,
// m = 128 224 -> 201; 4, fp32, d = 64, n = 576 14.4 -> 12.4; bound by memory, 40, n = 18432 67.4 -> 67.0; at d = 64 28 on 4, n = 2933,
// m = 128 22.3 -> 21.6, 4 x 32, n = 18432 112.5 -> 110.5, 32 on 2, n = 1000, m = 128 28.8 -> 28.6.
//
// NWV waves per workgroup.  16 waves (one workgroup per CU): stages of 32 KiB; 8 waves (two per CU): 16 KiB;
// never more than 128 keys (the column-sum buffers grow with the keys of a stage).
template <typename T, int D, int NWV>
struct ScoreCfg {
    static constexpr int E = Elem<T>::kBytes;
    static constexpr int CH = D / Elem<T>::kPerChunk;      // fragments per row per lane
    static constexpr int RB = D * E;                        // bytes per key row
    static constexpr int STG = NWV * 2048 < 128 * RB ? NWV * 2048 : 128 * RB;   // bytes per stage: two 1-KiB loads per wave, 128 keys at most
    static constexpr int SK = STG / RB;                     // keys per stage
    static constexpr int KBS = SK / 32;                     // 32-key blocks per stage
    static constexpr int NLD = STG / 1024 / NWV;            // 1-KiB loads per wave per stage
};

// The statistics of a row over some keys: the sum l of exp2(s c - e) about an offset e that is a whole number (the largest s c, rounded
// up), so that a change of offset scales l by a power of two and costs no rounding.  No key yet: l = 0, e = -FLT_MAX.
__device__ __forceinline__ void merge_stats(float& e, float& l, float e2, float l2) {
    const float E = fmaxf(e, e2);
    l = l * fast_exp2(e - E) + l2 * fast_exp2(e2 - E);
    e = E;
}
// A chunk's statistics of a row in one number, l 2^e, which fp32 holds exactly for offsets up to this and sums of 2^24 keys; beyond
// (and where l is no number) in two, -l and e.
constexpr float kWholeOffset = 100.f;

// PASS 1: partial[((b*Hq + head) * nsplit + chunk) * np + probe] = the sum over the chunk's keys of exp2(s c), or, where that is out of range
// (the sign tells), what is said above, the offset in a second plane of as many numbers
// PASS 2: mass / rank of the workgroup's keys; nsplit = chunks of pass 1
// np = probe rows rounded up to a multiple of 32 (NB blocks); rows beyond m are masked out.
// bpc = 32-key blocks per chunk of this pass; tpg = tasks per workgroup of pass 1, at most NWV.
// BY_STAGE (pass 2): scores are made stage by stage (scores_by_stage; known to the compiler: 2 to 3 % of short calls).
template <typename T, int D, int PASS, int NWV, bool BY_STAGE>
__global__ __launch_bounds__(64 * NWV, (Elem<T>::kBytes == 4 && D == 128 && NWV == 8) ? 2 : 4) void score_kernel(
    const T* __restrict__ Q, const T* __restrict__ K,
    int64_t qs0, int64_t qs1, int64_t qs2, int64_t ks0, int64_t ks1, int64_t ks2,
    ProbeList probes, int m, int NB, int n, int n_eff, float c, float* __restrict__ partial, int nsplit, int bpc, int tpg,
    float* __restrict__ mass, float* __restrict__ rank, int Hq, int Hkv, int kv_div)
{
    using C = ScoreCfg<T, D, NWV>;
    constexpr int CH = C::CH, RB = C::RB, SK = C::SK, KBS = C::KBS, NLD = C::NLD, kStageBytes = C::STG;
    constexpr int kThreads = 64 * NWV;
    extern __shared__ __attribute__((aligned(512))) char kstage[];   // kStageBufs stage buffers
    __shared__ __attribute__((aligned(16))) int sp[ZIPVL_MAX_PROBES];
    __shared__ float2 wstat[PASS == 1 ? NWV : 1][32];                // pass 1: per-wave row statistics
    __shared__ __attribute__((aligned(16))) float row_bias[PASS == 2 ? NWV : 1][32];
    __shared__ unsigned char marks[PASS == 2 ? NWV : 1][64];        // pass 2: which of a wave's 64 keys are probes
    __shared__ float keysum[PASS == 2 && !BY_STAGE ? (kSumStages - 1) * SK : 1];     // pass 2: sums of up to kSumStages - 1 stages
    __shared__ float colbuf[PASS == 2 ? 2 : 1][PASS == 2 ? NWV : 1][PASS == 2 ? SK : 1];

    const int G = Hq / Hkv, np = NB * 32;
    const int task0 = PASS == 1 ? blockIdx.z * tpg : 0;
    const int NT = PASS == 1 ? min(tpg, G * NB - task0) : G * NB;    // tasks of this workgroup
    const int u = blockIdx.y, b = u / Hkv, g = u - b * Hkv;
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);          // wave-uniform: everything derived from it lives in scalar registers
    const int nblk = ((PASS == 1 ? n_eff : n) + 31) >> 5;
    const int blk0 = blockIdx.x * bpc, blk1 = min(blk0 + bpc, nblk);
    if (blk0 >= blk1) return;
    const int S = (blk1 - blk0 + KBS - 1) / KBS;                     // stages of this chunk

    if (tid < ZIPVL_MAX_PROBES) sp[tid] = probes.pos[tid];           // -1 beyond m
    __syncthreads();

    // waves -> tasks.  Fewer tasks than waves: KS waves share a task and take the key blocks slot, slot + KS, ...
    const bool few = NT < NWV;
    const int KS = few ? NWV / NT : 1;
    const int rounds = PASS == 1 || few ? 1 : (NT + NWV - 1) / NWV;
    const int ts = few ? w % NT : w;                                 // task slot inside a round
    const int slot = few ? w / NT : 0;

    const char* Ku = reinterpret_cast<const char*>(K + b * ks0 + (g / kv_div) * ks1);   // kv_div > 1: every query head is its own unit
    const int row_stride = (int)ks2 * C::E;                          // bytes; a stage spans less than 2 GiB (checked on the host)
    const unsigned lds0 = lds_address(kstage);
    // where this lane's NLD 16-byte pieces of a stage come from: byte offset of (row inside the stage, chunk under the row swizzle)
    // (the loads of a wave are a multiple of 16 rows apart: one swizzle and one lane offset, the rest in the scalar base)
    constexpr int kLoadRows = NWV * 1024 / RB;
    static_assert(kLoadRows % 16 == 0, "one swizzle for all loads");
    const int ld_row = (w * 1024 + lane * 16) / RB;
    const int ld_off = ld_row * row_stride + ((((lane * 16) % RB >> 4) ^ k_row_swizzle<RB>(ld_row)) << 4);
    // Every wave issues exactly NLD loads per stage (pieces past the chunk's or the sequence's last row re-read
    // the stage's first row and are never used), so that "all but the newest p stages have landed" is a count.
    auto issue_stage = [&](int s) {
        const int row0 = (blk0 + s * KBS) * 32;
        const int rows = min(min(blk1 * 32, n) - row0, SK);           // rows of this stage that exist and belong to the chunk
        const char* gbase = Ku + (int64_t)row0 * row_stride;
        const unsigned dst = lds0 + (s % kStageBufs) * kStageBytes;
        if (rows == SK) {
#pragma unroll
            for (int q = 0; q < NLD; ++q) load_kib_to_lds(gbase + (int64_t)(q * kLoadRows) * row_stride, ld_off, dst + (q * NWV + w) * 1024);
        } else {
            int l = lane;                                            // derived again: nothing is carried for it
            asm volatile("" : "+v"(l));
            const int r0 = (w * 1024 + l * 16) / RB, off = r0 * row_stride + ((((l * 16) % RB >> 4) ^ k_row_swizzle<RB>(r0)) << 4);
#pragma unroll
            for (int q = 0; q < NLD; ++q) load_kib_to_lds(gbase, q * kLoadRows + r0 < rows ? q * kLoadRows * row_stride + off : 0, dst + (q * NWV + w) * 1024);
        }
    };
    // wait until at most `pending` stages (NLD loads each) of this wave are still on their way
    auto wait_stages = [&](int pending) {
        if (pending >= 2) __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * NLD));
        else if (pending == 1) __builtin_amdgcn_s_waitcnt(0x0F70 | NLD);
        else __builtin_amdgcn_s_waitcnt(0x0F70);
    };
    static_assert(2 * NLD < 16, "vmcnt immediate");

#pragma unroll 1
    for (int rd = 0; rd < rounds; ++rd) {
        const int task = rd * NWV + ts;
        const bool active = few ? w < NT * KS : task < NT;
        const int ntr = few ? NT : min(NWV, NT - rd * NWV);          // tasks of this round
        const int tk = PASS == 1 ? task0 + task : task;              // of the KV head's
        const int head = active ? tk / NB : 0, nb = active ? tk - (tk / NB) * NB : 0;
        const int bh = b * Hq + g * G + head;

        // chunk 2 cc + h of a row of the buffers, from where its chunk h is (rows are aligned to their size)
        using LdsFrag = const __attribute__((address_space(3))) uintx4*;
        auto fragment = [&](unsigned row, int cc) { return *(LdsFrag)(uintptr_t)(row ^ (32 * cc)); };
        if (rd) __syncthreads();                                     // the stage buffers of the previous round are free
        // This wave's probe rows: fragments of row nb*32 + i, held for the whole round.  Gathered lane by lane (a row each) a load touches 64
        // lines, and the 112 of a workgroup of 14 tasks kept the address unit busy for 3 us.  So they take the way of the keys: whole
        // rows to the end of the stage buffers, once for the waves of a task, and from there into registers.  The stages whose
        // buffers they leave free are on the way meanwhile.
        constexpr int kEnd = kStageBufs * kStageBytes;
        constexpr int kRows = NWV * 32 * RB <= kStageBufs * kStageBytes ? 32 : 16;       // rows of a task at a time
        static_assert(NWV * kRows * RB <= kStageBufs * kStageBytes, "room for the probe rows of all tasks of a round");
        const int rows_at = kEnd - (ts + 1) * kRows * RB;
        const int early = min(min(kStageBufs - 1, S), (kEnd - ntr * kRows * RB) / kStageBytes);
        const bool merges = PASS == 2 && active && slot == 0;
        const float* stats = partial + (int64_t)bh * nsplit * np + nb * 32;                     // wave-uniform base; the rest fits 32 bits (host check)
        // PASS 2: the statistics of a task's rows over pass 1's chunks, merged by one of its waves: lane = (4 rows, eighth of the chunks), 16
        // bytes a load, no more loads and sums than there are chunks for; as a rule plain sums.  (All 64 chunks' sums whatever their number, and four logarithms
        // by each of eight lanes: 32 on 2, d = 64, n = 577, m = 128 29.0 us, 28.45 so; fp32 at d = 128, where their zeros took the kernel past 128 registers, 8 heads,
        // n = 1500 24.3, 21.5.)
        auto merge_chunks = [&]() {
            int l = lane;
            asm volatile("" : "+v"(l));
            const int st_row = 4 * (l & 7), st_chunk = l >> 3;
            float L[4] = {0.f, 0.f, 0.f, 0.f}, E[4] = {0.f, 0.f, 0.f, 0.f};
            uint32_t signs = 0;
#pragma unroll 1
            for (int from = 0; from < nsplit; from += 64) {
                floatx4 v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (from + 8 * q < nsplit) v[q] = *reinterpret_cast<const floatx4*>(stats + min(from + st_chunk + 8 * q, nsplit - 1) * np + st_row);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    if (from + 8 * q >= nsplit) break;
                    const float there = from + st_chunk + 8 * q < nsplit ? 1.f : 0.f;
#pragma unroll
                    for (int r = 0; r < 4; ++r) L[r] = fmaf(v[q][r], there, L[r]);
                    signs |= __float_as_uint(v[q][0]) | __float_as_uint(v[q][1]);
                    signs |= __float_as_uint(v[q][2]) | __float_as_uint(v[q][3]);
                }
            }
            if (__any((int)signs < 0)) {
                const float* offsets = stats + (int64_t)gridDim.y * G * nsplit * np;
#pragma unroll
                for (int r = 0; r < 4; ++r) { L[r] = 0.f; E[r] = -FLT_MAX; }
#pragma unroll 1
                for (int s = st_chunk; s < nsplit; s += 8)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = stats[s * np + st_row + r];
                        if ((int)__float_as_uint(v) >= 0) merge_stats(E[r], L[r], v > 0.f ? 0.f : -FLT_MAX, v);
                        else merge_stats(E[r], L[r], offsets[s * np + st_row + r], -v);
                    }
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int x = 8; x <= 32; x *= 2) merge_stats(E[r], L[r], __shfl_xor(E[r], x), __shfl_xor(L[r], x));
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    L[r] += lane_moved<0x128, 0xF>(L[r], 0.f);                             // the other eight lanes of 16
                    const auto by16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(L[r]), __float_as_uint(L[r]), false, false);
                    L[r] = __uint_as_float(by16[0]) + __uint_as_float(by16[1]);
                    const auto by32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(L[r]), __float_as_uint(L[r]), false, false);
                    L[r] = __uint_as_float(by32[0]) + __uint_as_float(by32[1]);
                }
            }
            // every lane has the four rows' sums: one each for four of the eight lanes that share them
            const int row = st_row + st_chunk;
            const float sum = st_chunk == 0 ? L[0] : st_chunk == 1 ? L[1] : st_chunk == 2 ? L[2] : L[3], offset = st_chunk == 0 ? E[0] : st_chunk == 1 ? E[1] : st_chunk == 2 ? E[2] : E[3];
            if (st_chunk < 4) row_bias[ts][row] = (nb * 32 + row < m && sum > 0.f) ? offset + __log2f(sum) : INFINITY;
        };
        uintx4 qf[CH];
        auto request_stages = [&](int from, int to) {
            for (int s = from; s < to; ++s) issue_stage(s);
        };
        if constexpr (D == 64 && C::E == 2) {
            // rows of 128 bytes: four loads a wave, gathered behind the first stages (through LDS 32 heads on 8, n = 2933 14.4 -> 15.7 us, 4 x 32, n = 577 14.2 -> 14.9)
            request_stages(0, min(kStageBufs - 1, S));
            const T* qp = Q + b * qs0 + (int64_t)(g * G + head) * qs1 + (int64_t)sp[min(nb * 32 + i, m - 1)] * qs2 + h * Elem<T>::kPerFrag;
#pragma unroll
            for (int cc = 0; cc < CH; ++cc) qf[cc] = load16(qp + cc * Elem<T>::kPerChunk);
            if (merges) merge_chunks();
#pragma unroll
            for (int cc = 0; cc < CH; ++cc) asm volatile("" : "+v"(qf[cc]));      // here now, and not waited for in front of every tile
            if (PASS == 2) __syncthreads();
        } else {
#pragma unroll
        for (int r0 = 0; r0 < 32; r0 += kRows) {
            // (long chunks of few tasks: the keys first, they are what such a call waits for)
            if (r0 == 0 && early == kStageBufs - 1) request_stages(0, early);
            int l = lane;                                            // (through the empty asm: none of the addresses is kept from round to round)
            asm volatile("" : "+v"(l));
            if (active) {
                // lane: row l / (RB / 16) of each load's 1024 / RB, piece l % (RB / 16) under the swizzle
                const int lr = l * 16 / RB, lp = (l * 16 % RB >> 4), r1 = nb * 32 + r0 + lr;
                const char* Qh = reinterpret_cast<const char*>(Q + b * qs0 + (int64_t)(g * G + head) * qs1);
                const int64_t stride = qs2 * C::E;
                auto request = [&](auto narrow) {
                    for (int q = slot; q < kRows * RB / 1024; q += KS) {
                        const int r = q * (1024 / RB), prow = sp[min(r1 + r, m - 1)], piece = (lp ^ k_row_swizzle<RB>(r + lr)) << 4;
                        const unsigned dst = lds0 + rows_at + q * 1024;
                        if constexpr (decltype(narrow)::value) load_kib_to_lds(Qh, (int)(__umul24(prow, (unsigned)stride) + piece), dst);
                        else load_kib_to_lds_at(Qh + prow * stride + piece, dst);
                    }
                };
                if (stride < 1 << 24 && n * stride < (int64_t)1 << 32) request(std::true_type{});       // offsets of 32 bits: a sixth of the address arithmetic
                else request(std::false_type{});
            }
            if (r0 == 0 && early < kStageBufs - 1) request_stages(0, early);
            if (r0 == 0 && merges) merge_chunks();
            // all but the stages requested after them
            if (r0 == 0 && early == 1) __builtin_amdgcn_s_waitcnt(0x0F70 | NLD);
            else if (r0 == 0 && early == 2) __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * NLD));
            else __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            const int li = l & 31;
            const unsigned row = lds0 + rows_at + (kRows == 32 ? li : li & 15) * RB + (((l >> 5) ^ k_row_swizzle<RB>(li)) << 4);
            if (kRows == 32 || (li >> 4) == (r0 >> 4))
#pragma unroll
                for (int cc = 0; cc < CH; ++cc) qf[cc] = fragment(row, cc);
            if (r0 + kRows < 32 || early < min(kStageBufs - 1, S)) {
                __builtin_amdgcn_s_waitcnt(0xC07F);
                __syncthreads();                                     // every wave has read its rows
            }
        }
        request_stages(early, min(kStageBufs - 1, S));
        }
        const int Pm = sp[nb * 32 + i];                              // PASS 1: position of this lane's probe (-1: padding)
        // the first and last probe of this wave's block (sp ascends): its tiles up to the first need no mask, those past the
        // last are empty.  64 random probes put the first of all 128 near token 0, and every tile was masked.
        const int Pfirst = __builtin_amdgcn_readfirstlane(nb * 32 + 32 <= m ? sp[nb * 32] : -1);
        const int Plast = __builtin_amdgcn_readfirstlane(sp[min(nb * 32 + 31, m - 1)]);

        float e_run = -FLT_MAX, l_run = 0.f;                         // PASS 1
        // PASS 2: exponent offsets of this lane's probe rows nb*32 + acc_row(r, h); in LDS where registers are short
        constexpr bool kHeldBias = PASS == 2 && !(C::E == 4 && D == 128 && NWV == 16);
        float rb[16];
        auto load_bias = [&]() {
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const floatx4 v = *reinterpret_cast<const floatx4*>(&row_bias[ts][8 * a + 4 * h]);
                rb[4 * a] = v[0]; rb[4 * a + 1] = v[1]; rb[4 * a + 2] = v[2]; rb[4 * a + 3] = v[3];
            }
        };
        if (kHeldBias) load_bias();
        // PASS 2: the scores of a stage's keys, which every wave waits for at the next barrier: made by the last waves, or (BY_STAGE false) these add up
        // the tasks' sums only, and what makes scores of them is left for kSumStages stages at a time, to all waves.
        // The tasks' column sums, in task order.
        auto key_sum = [&](int s, int t) {
            const float* col = &colbuf[s & 1][0][t];
            float a = 0.f;
            for (int q = 0; q < ntr; q += 4) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = col[min(q + e, ntr - 1) * SK];
#pragma unroll
                for (int e = 0; e < 4; ++e) a += q + e < ntr ? v[e] : 0.f;
            }
            return a;
        };
        // by the workgroup's last threads (with more waves than tasks those waves are otherwise idle)
        auto sum_stage = [&](int s) {
            for (int t = kThreads - 1 - tid; t < SK; t += kThreads) keysum[(s % kSumStages) * SK + t] = key_sum(s, t);
        };
        // The scores of the keys of stages s0 .. s1 - 1; the last of them is still in the tasks' sums
        auto write_scores = [&](int s0, int s1) {
            const int row0 = (blk0 + s0 * KBS) * 32, last = (s1 - 1 - s0) * SK, keys = min(min(blk1 * 32, n) - row0, last + SK);
            for (int t0 = (NWV - 1 - w) * 64; t0 < keys; t0 += kThreads) {       // 64 keys of the wave
                const int t = t0 + lane, j = row0 + t;
                const bool mine = t < keys, seen = mine && j < n_eff;
                float a = 0.f;
                if (rd && seen) {                                    // tasks of earlier rounds
                    a = mass[(int64_t)u * n + j];
                    asm volatile("" : "+v"(a));                      // waited for here and not, with the stages in flight, on every path
                }
                if (seen) a += t < last ? keysum[t] : key_sum(s1 - 1, t - last);
                if (rd + 1 < rounds) {
                    if (mine) mass[(int64_t)u * n + j] = a;
                } else {
                    // Probes at or after j: m less those before it, of which two ballots count those before the 64 keys, and the others are marks
                    // among the keys (a bisection over the list in LDS is seven reads one after the other).
                    static_assert(ZIPVL_MAX_PROBES == 128, "two probes a lane");
                    const int j0 = row0 + t0;
                    int before = 0;
                    marks[w][lane] = 0;
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");       // other lanes' marks are neither before this nor behind the read below
#pragma unroll
                    for (int e = 0; e < ZIPVL_MAX_PROBES; e += 64) {
                        const int pos = e + lane < m ? sp[e + lane] - j0 : 64;
                        before += __popcll(__ballot(pos < 0));
                        if (pos >= 0 && pos < 64) marks[w][pos] = 1;
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    const uint64_t bits = __ballot(marks[w][lane]);
                    before += __builtin_amdgcn_mbcnt_hi((uint32_t)(bits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bits, 0));
                    const int cnt = m - before;
                    if (mine) {
                        mass[(int64_t)u * n + j] = a / (float)(G * m);
                        if (rank) rank[(int64_t)u * n + j] = cnt > 0 ? a / (float)(G * cnt) : 0.f;
                    }
                }
            }
        };
        const unsigned frag0 = lds0 + i * RB + ((h ^ k_row_swizzle<RB>(i)) << 4);
#pragma unroll 1
        for (int s = 0; s < S; ++s) {
            // stage s has landed (this wave's pieces, then everyone's); everyone is done with stage s - 1, whose
            // buffer takes stage s + kStageBufs - 1 and whose column sums are complete
            wait_stages(min(kStageBufs - 2, S - 1 - s));
            __syncthreads();
            if (s + kStageBufs - 1 < S) issue_stage(s + kStageBufs - 1);
            if (PASS == 2 && s > 0) {
                if (BY_STAGE || s % kSumStages == 0) write_scores(BY_STAGE ? s - 1 : s - kSumStages, s);
                else sum_stage(s - 1);
            }
            const int buf = s & 1;                                   // column-sum buffer of the stage
            const unsigned kb0 = frag0 + (s % kStageBufs) * kStageBytes;
            const int sblk = blk0 + s * KBS;                         // first key block of the stage
            if (active) {
#pragma unroll 1
                for (int kb = slot; kb < KBS && sblk + kb < blk1; kb += KS) {
                    const int jb = (sblk + kb) * 32;
                    if (jb > Plast) {                                // no probe row of the block sees these keys
                        if (PASS == 2 && h == 0) colbuf[buf][ts][kb * 32 + i] = 0.f;
                        continue;
                    }
                    const unsigned krow = kb0 + kb * 32 * RB;
                    auto kfrag = [&](int cc) { return fragment(krow, cc); };
                    floatx16 acc = {0};
                    // long chunks of few tasks are bound by memory, and faster where a wave with a tile waits for all stages on their way (40
                    // heads, n = 18432, m = 64 68.8 -> 67.4 us; at d = 64 4 x 32 heads 111.5 -> 118)
                    if (PASS == 1 && D == 128 && early == kStageBufs - 1 && S > 4 * (kStageBufs - 1)) __builtin_amdgcn_s_waitcnt(0x0F70);
                    // bf16: the fragments of the key block are read ahead of the products (four while 128 registers hold no more; two at
                    // a time: 14 heads on 2, n = 33000, m = 128 84.7 -> 80.3 us); an fp32 one feeds four products of 64 cycles
                    constexpr int kReads = C::E == 4 ? 1 : CH;
                    uintx4 kf[CH];
#pragma unroll
                    for (int cc = 0; cc < kReads; ++cc) kf[cc] = kfrag(cc);
                    if (C::E == 2) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int cc = 0; cc < CH; ++cc) {
                        if (cc + kReads < CH) kf[cc + kReads] = kfrag(cc + kReads);
                        acc = PASS == 1 ? mma_frag<T>(kf[cc], qf[cc], acc) : mma_frag<T>(qf[cc], kf[cc], acc);
                    }
                    const bool masked = jb + 31 > Pfirst;            // wave-uniform
                    if (PASS == 1) {
                        // acc[r]: key jb + acc_row(r, h), probe column nb*32 + i  (raw logit)
                        if (masked) {
                            const int own = Pm - jb - 4 * h;
#pragma unroll
                            for (int r = 0; r < 16; ++r)
                                if (acc_row(r, 0) > own) acc[r] = -INFINITY;
                        }
                        float mx = acc[0];
#pragma unroll
                        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, acc[r]);
                        const float e_new = fmaxf(e_run, ceilf(mx * c));     // a number also where the lane has seen no key yet: it adds zeros
                        float sum = l_run * fast_exp2(e_run - e_new);
#pragma unroll
                        for (int r = 0; r < 16; ++r) sum += fast_exp2(fmaf(acc[r], c, -e_new));
                        l_run = sum;
                        e_run = e_new;
                    } else {
                        // acc[r]: probe row nb*32 + acc_row(r, h), key column jb + i
                        if (!kHeldBias) load_bias();
                        float sum = 0.f;
                        if (masked) {
#pragma unroll
                            for (int a = 0; a < 4; ++a) {
                                const uintx4 pos = *reinterpret_cast<const uintx4*>(&sp[nb * 32 + 8 * a + 4 * h]);
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    const float pr = fast_exp2(fmaf(acc[4 * a + e], c, -rb[4 * a + e]));
                                    sum += jb + i > (int)pos[e] ? 0.f : pr;
                                }
                            }
                        } else {
#pragma unroll
                            for (int r = 0; r < 16; ++r) sum += fast_exp2(fmaf(acc[r], c, -rb[r]));
                        }
                        const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
                        if (h == 0) colbuf[buf][ts][kb * 32 + i] = __uint_as_float(halves[0]) + __uint_as_float(halves[1]);
                    }
                }
            }
        }
        if (PASS == 2) {
            __syncthreads();                                         // the last stage's column sums are in LDS
            write_scores(BY_STAGE ? S - 1 : (S - 1) / kSumStages * kSumStages, S);
        }

        if (PASS == 1) {
            // the two half-waves saw different keys of the same rows; waves that share a task saw different key blocks
            merge_stats(e_run, l_run, __shfl_xor(e_run, 32), __shfl_xor(l_run, 32));
            if (h == 0) wstat[w][i] = active ? make_float2(e_run, l_run) : make_float2(-FLT_MAX, 0.f);
            __syncthreads();
            for (int t = tid; t < ntr * 32; t += kThreads) {
                const int q = t >> 5, pc = t & 31;                   // task slot, probe row of its block
                float E = -FLT_MAX, L = 0.f;
                for (int sl = 0; sl < KS; ++sl) {
                    const float2 v = wstat[few ? sl * NT + q : q][pc];
                    merge_stats(E, L, v.x, v.y);
                }
                const int tk = task0 + rd * NWV + q, hd = tk / NB, nbk = tk - hd * NB;
                float* out = partial + ((int64_t)(b * Hq + g * G + hd) * nsplit + blockIdx.x) * np + nbk * 32 + pc;
                if (L == 0.f || (L > 0.f && fabsf(E) <= kWholeOffset)) {
                    *out = L > 0.f ? __builtin_amdgcn_ldexpf(L, (int)E) : 0.f;
                } else {
                    *out = __uint_as_float(__float_as_uint(L) | 0x80000000u);
                    out[(int64_t)gridDim.y * G * nsplit * np] = E;
                }
            }
        }
    }
}

// ---------------------------------------------------------------- host side
static int probe_rows(int m) { return (m + 31) / 32 * 32; }

// Workgroups that fit the chip at once with `waves` waves each (registers allow 16 waves per CU here).
static int resident_slots(int waves) {
    static std::atomic<int> cus{0};
    int c = cus.load();
    if (!c) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1) v = 256;
        cus = c = v;
    }
    return c * (16 / waves);
}

// 32-key blocks per chunk so that about `slots` workgroups cover `units` x nblk blocks
static int blocks_per_chunk(int nblk, int units, int slots) {
    const int chunks = std::max(1, std::min(nblk, slots / units));
    return (nblk + chunks - 1) / chunks;
}

size_t score_workspace_bytes(const zipvl_dims& d, int m) {
    // one pair (sum, offset; the offsets in a plane of their own) per head, probe row and pass-1 chunk; chunks per unit never exceed the resident slots
    const int max_chunks = std::max(1, resident_slots(8) / std::max(1, d.B * d.Hkv));
    return (size_t)d.B * d.Hq * max_chunks * probe_rows(m) * sizeof(float2);
}

// Pass 1: groups of tasks, a workgroup each, per KV head and chunk.  A task for each of the 8 waves, or half as many tasks
// and two waves for each: a chunk of as many workgroups is twice as long, so that pass 2 has half of the statistics to read and
// pass 1 reads K twice as often.  The two together, bytes per CU, decide (kKeyCost: a byte of K against one of the statistics, from
// where the two cost the same: 28 heads on 4, m = 64 n = 13000, 14 on 2 n = 33000).  us, all tasks of a KV head in one workgroup of 16 waves, in
// rounds of 16 where there are more -> 8 a workgroup, 4 a workgroup: 28 heads on 4, m = 64, n = 4096 22.4 -> 21.5, 20.0; n = 18432 37.3 -> 35.3, 36.4;
// m = 128 n = 4096 39.5 -> 30.3, 29.8; n = 18432 69.4 -> 62.1, 62.0; 32 on 2, n = 4096 40.8 -> 29.1, 26.7; 32 on 8, n = 4096 21.0 (8), 19.7.
// fp32 is bound by its products: there the tiles that the busiest SIMD takes decide first (7 of 8 waves with a task leave one SIMD with fewer),
// and chunks may be twice as many, taken in two turns, where one turn leaves slots empty (kTurnTiles: a turn costs 4.5 us at d = 64 and
// 10 at 128, as long as so many tiles).  28 heads on 4, m = 128, fp32, 16 waves in rounds, bytes
// alone -> so: batch 1 n = 33000 546, 554, 531; 3, n = 12000 572, 606, 566; 4, n = 12000 741, 764, 742; d = 64, batch 4, n = 25000 760, 802, 762.
constexpr double kKeyCost = 1.2;
constexpr int kTurnTiles = 5;

struct RowStatsPlan { int groups, bpc; };                        // groups of tasks, 32-key blocks of a chunk

static RowStatsPlan row_stats_plan(int NT, int units, int nblk, int row_bytes, int waves2, bool products) {
    const int full = (NT + 7) / 8, half = (NT + 3) / 4, slots = resident_slots(8), cus = resident_slots(16);
    auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    auto plan = [&](int groups, int turns) { return RowStatsPlan{groups, blocks_per_chunk(nblk, units * groups, turns * slots)}; };
    auto bytes = [&](const RowStatsPlan& p) {
        return kKeyCost * p.groups * units * nblk * 32.0 * row_bytes / cus + (double)ceil_div(nblk, p.bpc) * NT * 32 * sizeof(float) * (16 / waves2);
    };
    auto tiles = [&](const RowStatsPlan& p) {
        const int64_t tpg = ceil_div(NT, p.groups), shared = std::max<int64_t>(1, 8 / tpg), wgs = (int64_t)units * p.groups * ceil_div(nblk, p.bpc);
        const int64_t turns = ceil_div(wgs, slots);
        return turns * ceil_div(std::min<int64_t>(wgs, slots), cus) * ceil_div(tpg * shared, 4) * ceil_div(p.bpc, shared) + (turns - 1) * kTurnTiles;
    };
    RowStatsPlan best = plan(full, 1);
    auto look_at = [&](const RowStatsPlan& p) {
        const int64_t more = products ? tiles(p) - tiles(best) : 0;
        if (more < 0 || (more == 0 && bytes(p) < bytes(best))) best = p;
    };
    look_at(plan(half, 1));
    if (products && half > 1) look_at(plan(half, 2));            // (the workspace has room for slots / units chunks)
    return best;
}

template <typename T, int D, int PASS, int NWV, bool BY_STAGE = true>
static int reserve_lds() {
    static std::atomic<bool> done{false};                            // raising the dynamic-LDS cap is idempotent
    if (!done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&score_kernel<T, D, PASS, NWV, BY_STAGE>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kStageBufs * ScoreCfg<T, D, NWV>::STG) != hipSuccess)
            return set_error(ZIPVL_EHIP, "score: cannot reserve LDS for the key stages");
        done = true;
    }
    return ZIPVL_OK;
}

// Whether 8 waves make the scores of a chunk of `bpc` key blocks stage by stage (16 always do): where waves without a tile are there for it, and where the
// chunk has two stages at most.  us, eight stages at a time -> stage by stage: 28 heads on 4, n = 18432 32.4 -> 31.7,
// 32 on 2, d = 64, n = 1000, m = 128 29.8 -> 29.0; 8 waves, d = 64, 4 x 32 heads, n = 577 (2 stages) 14.5 -> 14.2; past the line 4 x 32 heads, n = 4096,
// m = 128 (16 stages) 62.4 -> 63.8, 32, d = 64, n = 8192 (4) 3 % slower.
static bool scores_by_stage(int NT, int key_blocks, int bpc) {
    const int last_slot = 7 / NT;                                    // of the last wave, if it has a task
    return (NT < 8 && (last_slot >= key_blocks || 8 > NT * (8 / NT))) || bpc <= 2 * key_blocks;
}

// NW2: waves per workgroup of pass 2 (pass 1: 8)
template <typename T, int D, int NW2>
static int launch_score_w(const void* Q, const void* K, const zipvl_dims& d, const ProbeList& pl, int m,
                          int n_eff, float scale, float* mass, float* rank, void* ws, int kv_div, hipStream_t st)
{
    const float c = scale * kLog2e;
    float* partial = (float*)ws;
    const int units = d.B * d.Hkv, NB = probe_rows(m) / 32, NT = d.Hq / d.Hkv * NB;
    constexpr size_t lds1 = (size_t)kStageBufs * ScoreCfg<T, D, 8>::STG, lds2 = (size_t)kStageBufs * ScoreCfg<T, D, NW2>::STG;
    int rc = reserve_lds<T, D, 1, 8>();
    if (rc) return rc;
    const int nblk1 = (n_eff + 31) / 32;
    const RowStatsPlan plan = row_stats_plan(NT, units, nblk1, D * (int)sizeof(T), NW2, Elem<T>::kBytes == 4);
    const int groups = plan.groups, tpg = (NT + groups - 1) / groups, bpc1 = plan.bpc, nsplit = (nblk1 + bpc1 - 1) / bpc1;
    const int nblk2 = (d.n + 31) / 32, bpc2 = blocks_per_chunk(nblk2, units, resident_slots(NW2)), chunks2 = (nblk2 + bpc2 - 1) / bpc2;
    {
        KernelTimer tm(ZIPVL_K_SCORE_ROWSTATS, st);
        hipLaunchKernelGGL((score_kernel<T, D, 1, 8, true>), dim3(nsplit, units, groups), dim3(512), lds1, st,
            (const T*)Q, (const T*)K, d.q_strides[0], d.q_strides[1], d.q_strides[2],
            d.k_strides[0], d.k_strides[1], d.k_strides[2], pl, m, NB, d.n, n_eff, c, partial, nsplit, bpc1, tpg,
            (float*)nullptr, (float*)nullptr, d.Hq, d.Hkv, kv_div);
    }
    rc = check_launch("score_rowstats");
    if (rc) return rc;
    auto pass2 = [&](auto by_stage) -> int {
        constexpr bool kByStage = decltype(by_stage)::value;
        rc = reserve_lds<T, D, 2, NW2, kByStage>();
        if (rc) return rc;
        KernelTimer tm(ZIPVL_K_SCORE_COLSUM, st);
        hipLaunchKernelGGL((score_kernel<T, D, 2, NW2, kByStage>), dim3(chunks2, units), dim3(64 * NW2), lds2, st,
            (const T*)Q, (const T*)K, d.q_strides[0], d.q_strides[1], d.q_strides[2],
            d.k_strides[0], d.k_strides[1], d.k_strides[2], pl, m, NB, d.n, n_eff, c, partial, nsplit, bpc2, NT,
            mass, rank, d.Hq, d.Hkv, kv_div);
        return check_launch("score_colsum");
    };
    if constexpr (NW2 == 8)
        if (!scores_by_stage(NT, ScoreCfg<T, D, NW2>::KBS, bpc2)) return pass2(std::false_type{});
    return pass2(std::true_type{});
}

template <typename T, int D>
static int launch_score_t(const void* Q, const void* K, const zipvl_dims& d, const ProbeList& pl, int m,
                          int n_eff, float scale, float* mass, float* rank, void* ws, int kv_div, hipStream_t st)
{
    const int NT = (d.Hq / d.Hkv) * (probe_rows(m) / 32);            // (head, probe block) tasks per unit
    if (NT > 8) return launch_score_w<T, D, 16>(Q, K, d, pl, m, n_eff, scale, mass, rank, ws, kv_div, st);
    return launch_score_w<T, D, 8>(Q, K, d, pl, m, n_eff, scale, mass, rank, ws, kv_div, st);
}

int launch_score(const void* Q, const void* K, const zipvl_dims& d0, const int32_t* probe_pos, int m,
                 float scale, int flags, float* mass, float* rank, void* ws, hipStream_t st)
{
    // one row of scores per query head: the same kernels on dims in which every query head is a unit of its own
    // that reads the K of the KV head it belongs to
    zipvl_dims d = d0;
    int kv_div = 1;
    if ((flags & ZIPVL_SCORE_PER_QHEAD) && d0.Hq != d0.Hkv) {
        kv_div = d0.Hq / d0.Hkv;
        d.Hkv = d0.Hq;
    }
    if (d0.Hq / d0.Hkv > kMaxGroup) return set_error(ZIPVL_ESHAPE, "score: Hq/Hkv = %d exceeds %d", d0.Hq / d0.Hkv, kMaxGroup);
    if (d.k_strides[2] * (d.dtype == ZIPVL_BF16 ? 2 : 4) > (1 << 22))       // 256 staged rows must span less than 2 GiB
        return set_error(ZIPVL_ESHAPE, "score: K token stride of %lld elements is too large", (long long)d.k_strides[2]);
    ProbeList pl;
    for (int t = 0; t < ZIPVL_MAX_PROBES; ++t) pl.pos[t] = t < m ? probe_pos[t] : -1;
    const int n_eff = probe_pos[m - 1] + 1;
    if (d.dtype == ZIPVL_BF16) {
        if (d.d == 128) return launch_score_t<__bf16, 128>(Q, K, d, pl, m, n_eff, scale, mass, rank, ws, kv_div, st);
        return launch_score_t<__bf16, 64>(Q, K, d, pl, m, n_eff, scale, mass, rank, ws, kv_div, st);
    }
    if (d.d == 128) return launch_score_t<float, 128>(Q, K, d, pl, m, n_eff, scale, mass, rank, ws, kv_div, st);
    return launch_score_t<float, 64>(Q, K, d, pl, m, n_eff, scale, mass, rank, ws, kv_div, st);
}

}  // namespace zipvl
