// Exact token scores from EVERY row of the attention matrix (Eq. (6) and Eq. (8)
// as written, before the probe approximation of the supplementary material): the
// accuracy reference for the probe scores.  A is never stored.  Two passes of one
// kernel body over the causal half of Q K^T:
//   pass 1  per query row, the exponent offset lse = log2(sum exp2(s c)) of its visible
//           logits (c = softmax scale * log2 e);
//   pass 2  per query head and key column, sum over the rows that see it of exp2(s c - lse);
//           a small kernel then averages the query heads of a group (fixed order) and writes
//           mass = a / n and rank = a / (n - j)  (every row at or after j counts in Eq. (8)).
// A workgroup keeps 32 or 64 rows per wave of one side in registers as MFMA fragments (queries in
// pass 1, keys in pass 2) and streams the other side through LDS in chunks of 64 rows, loaded
// straight from global memory, double buffered, one barrier per chunk.  The product is taken as
// (streamed rows) x (register rows)^T on 32x32 tiles, so a lane owns one register-side row of each
// 32 and its statistic (a running sum) never leaves the lane until the end.
#include <atomic>
#include <cfloat>
#include <numeric>
#include <type_traits>

#include "launch.h"
#include "ldsload.h"

namespace zipvl {

constexpr int kArChunk = 64;      // streamed rows per chunk
constexpr int kArWaves = 4;       // waves per workgroup; 8 (half the streaming traffic) gain 2 % at 28 heads x 18432 and lose 5-50 % where workgroups are few

// What bounds it: a 32x32x128 bf16 tile is 256 matrix cycles and, per lane, 16 x (fma + exp2 + add) (pass 1: + max), 290 to 340
// vector cycles that waves overlap with them; of large calls the power of the chip: at 58 % busy matrix cores the clock is 1.65 GHz.  So:
// staging that needs no registers, no barrier but one per 64 rows, no instruction that is not a tile's own (LDS addresses in the
// offset field of the reads, one lane offset for all loads of a chunk, the running maximum in the chain of a block's maxima), a
// block's products and the vector work of the block before written between each other (RG = 1 runs three waves a SIMD, short calls one), and
// for large calls 64 rows a wave: half the LDS reads per product.  28 heads on 4, n = 18432, d = 128, both passes, ms: 4.97 (staged through
// registers, 128-row blocks in no XCD order), 2.85 (90 vector instructions a tile and pass 1, part after part), 2.62 (68), 2.38 (the parts of an XCD
// in turns), 2.25 (64 rows a wave).  us, before these three -> now: 32 heads, n = 2933 136 -> 92, 8 heads, n = 6000 194 -> 135, 8 on 2, n = 6000, d = 64 161 -> 112,
// 4 x 40, n = 2000 256 -> 208.  Measured and not taken: three chunks in flight (52 KiB of LDS, 5 % slower), a lazily moved offset instead
// of the running maximum (4 % faster, other roundings), four waves a SIMD with that order (120 bytes of scratch a lane).
template <typename T, int D, int RG>
struct ArCfg {
    static constexpr int E = Elem<T>::kBytes;
    static constexpr int CH = D / Elem<T>::kPerChunk;       // fragments per row per lane
    static constexpr int RB = D * E;                         // bytes per row
    static constexpr int STG = kArChunk * RB;                // one chunk in LDS (rows unpadded, 16-byte pieces swizzled)
    static constexpr int NLD = STG / 1024 / kArWaves;        // 1-KiB loads per wave and chunk
    static constexpr int ROWS = 32 * RG * kArWaves;               // register-side rows per workgroup
    static constexpr size_t LDS = 2 * ((size_t)STG + kArWaves * kArChunk * sizeof(float));   // two chunks, and their rows' lse (one copy per wave)
};

// Which (head, block of register-side rows) a workgroup takes.  Workgroups go round-robin over the 8 XCDs; every XCD
// gets whole heads (or 1 / split of the blocks of one, where the heads do not divide by 8) so that the rows it streams
// stay in its own L2, the blocks with the most visible pairs of all its parts first: part after part, the heaviest block of the last one, a
// sixth of the launch, began when the others were done (28 heads on 4, n = 18432 18 % of the CU time idle, now 7).  Where an XCD has few workgroups, 32 rows
// a wave, every second 32 of them (it has 32 CUs) are turned, so that a CU gets heavy and light ones.  It is meant for those that start together, 96
// of an XCD in bf16 and 64 in fp32, and pays for half as many more, which follow where light ones end; the lines are measured.  us, in order -> so, by workgroups of an XCD: bf16, d = 128,
// 40 heads, n = 2500 (100) 88.8 -> 84.0, 32, n = 3500 (112) 123.9 -> 121.4, 32 on 8, n = 3800 (120) 144.8 -> 144.9, past it 32, n = 4096 (128) 158.9 -> 161.4,
// 40, n = 4090 (160) 188 -> 197; d = 64, 32 on 8, n = 4096 (128) 115 -> 108, 40, n = 4090 (160) 132 -> 128, 36 on 4, n = 4480 (158) as before; fp32, d = 64, 4 heads,
// n = 33 000 (129) 5140 -> 4282, 40, n = 4090 746 -> 730, d = 128, 8, n = 6000 (47) 992 -> 803, 40, n = 4090 1373 -> 1354.  Short chains lose (4 x 32 on 8, n = 1000 56.6 ->
// 58.5).  Grid: x = (block of the part, XCD), y = part of the XCD; neither dimension reaches the launch limits (2^32 threads,
// 65535) for any dims that are accepted.
template <typename T, int D> constexpr int kArTurned = Elem<T>::kBytes == 2 && D == 128 ? 120 : 160;      // workgroups of an XCD up to which
constexpr int kArTurnedBlocks = 16;                                                                       // blocks of a head from which
// Blocks of 128 rows of all heads, and rows of a head, from which a wave takes 64 rows (us, 32 rows -> 64): 8 on 2, n = 33000 (2064 blocks) 2225 -> 2084, 32 on 8,
// n = 8192 (2048) 563 -> 535, 4 x 40, n = 2800 (3520) 367 -> 361; past the lines 4 x 40, n = 2000 (2560) 204 -> 208, 4 heads, n = 33000,
// d = 64 (1032) 839 -> 962, 32, n = 2933 (736) 95 -> 112.
constexpr int kArWideBlocks = 2048, kArWideRows = 2560;

template <typename T, int D, int PASS, int RG>
__global__ __launch_bounds__(64 * kArWaves, Elem<T>::kBytes == 2 && RG == 1 ? 3 : 2) void allrows_pass_kernel(
    const T* __restrict__ R, int64_t rs0, int64_t rs1, int64_t rs2,     // register side: Q (pass 1) / K (pass 2)
    const T* __restrict__ S, int64_t ss0, int64_t ss1, int64_t ss2,     // streamed side: K (pass 1) / Q (pass 2)
    int n, float c, float* __restrict__ lse, float* __restrict__ colsum_out, int Hq, int G, int split,
    uint32_t inv_parts, uint32_t inv_split, uint32_t inv_hq, uint32_t inv_g)     // of the grid's y, split, Hq, G: places without divisions
{
    using C = ArCfg<T, D, RG>;
    constexpr int CH = C::CH, RB = C::RB, NLD = C::NLD, STG = C::STG;
    extern __shared__ __attribute__((aligned(16))) char smem[];          // two chunks, then (pass 2) 2 x kArWaves x kArChunk lse values
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (n + C::ROWS - 1) / C::ROWS;
    // the parts of an XCD take turns, block by block
    const int xcd_blocks = gridDim.x >> 3, total = xcd_blocks * gridDim.y;
    int turn = __builtin_amdgcn_readfirstlane(blockIdx.y * xcd_blocks + (blockIdx.x >> 3));
    if (RG == 1 && (turn & 32) && total <= kArTurned<T, D> && nblk >= kArTurnedBlocks) turn = (turn & ~31) + min(total - 1, turn | 31) - turn;
    const int rank = __builtin_amdgcn_readfirstlane(divided(turn, gridDim.y, inv_parts));                                       // scalar from here on
    const int part = __builtin_amdgcn_readfirstlane((blockIdx.x & 7) * gridDim.y + turn - rank * gridDim.y);      // split parts per head
    const int bh = __builtin_amdgcn_readfirstlane(divided(part, split, inv_split)), order = rank * split + part - bh * split;
    if (order >= nblk) return;
    const int b = __builtin_amdgcn_readfirstlane(divided(bh, Hq, inv_hq)), head = bh - b * Hq;
    const int g = __builtin_amdgcn_readfirstlane(divided(head, G, inv_g));
    // heavy blocks first: late queries in pass 1, early keys in pass 2
    const int row0 = (PASS == 1 ? nblk - 1 - order : order) * C::ROWS, wrow0 = row0 + 32 * RG * w;

    // streamed chunks: keys [0, last row] upwards in pass 1; query rows [first key, n) downwards in pass 2, so that the
    // workgroups of a head start on the same rows
    const int chunk_lo = PASS == 1 ? 0 : row0 / kArChunk;
    const int chunk_hi = PASS == 1 ? (min(n, row0 + C::ROWS) - 1) / kArChunk : (n - 1) / kArChunk;
    const int nchunk = chunk_hi - chunk_lo + 1;
    auto chunk_row = [&](int t) { return (PASS == 1 ? chunk_lo + t : chunk_hi - t) * kArChunk; };

    const char* Sb = reinterpret_cast<const char*>(S + b * ss0 + (int64_t)(PASS == 1 ? g : head) * ss1);
    const int64_t row_bytes = ss2 * C::E;
    const float* lse_h = lse + (int64_t)bh * n;
    const unsigned lds0 = lds_address(smem), lse0 = lds0 + 2 * STG;
    // This lane's pieces of a chunk: LDS byte o = row r, position p of the row; the piece's offset from the first row of its load.  Loads
    // whose rows are a multiple of 16 apart have the same swizzle: they share an offset and differ in the scalar base.
    constexpr int kRowsPerLoad = 1024 / RB, kLoadRows = kArWaves * kRowsPerLoad, kOffsets = kLoadRows % 16 == 0 ? 1 : 2;
    static_assert(kOffsets * kLoadRows % 16 == 0 && NLD % kOffsets == 0, "swizzles repeat");
    const bool narrow = row_bytes * kArChunk < (int64_t)1 << 31;        // a chunk's offsets fit 32 bits: row strides below 32 MiB
    unsigned ld_off[kOffsets];
#pragma unroll
    for (int q = 0; q < kOffsets; ++q) {
        const int r = w * kRowsPerLoad + lane * 16 / RB, p = (lane * 16 % RB) >> 4;
        ld_off[q] = (narrow ? (unsigned)(r * row_bytes) : 0u) + ((p ^ k_row_swizzle<RB>(q * kLoadRows + r)) << 4);
    }
    // Every wave issues the same number of loads for every chunk; rows past the end re-read the chunk's first one.  That form, and
    // the one for wide rows, derive what they need from the thread index (one load after the other, and with divisions for the workgroup's place: 8 heads on 2,
    // n = 300 19.1 us, 18.8 so, n = 130 16.0, 15.7; 15.0 when a call had no order written out and a third of the code).
    auto issue = [&](int t) {
        const int c0 = chunk_row(t), buf = (t & 1);
        const char* base = scalar_ptr(Sb + c0 * row_bytes);
        const unsigned dst = lds0 + buf * STG + w * 1024;
        const bool whole = c0 + kArChunk <= n;
        if (narrow && whole) {
#pragma unroll
            for (int q = 0; q < NLD; ++q) load_kib_to_lds(base + q * (kLoadRows * row_bytes), (int)ld_off[q % kOffsets], dst + q * kArWaves * 1024);
        } else {
            int l = lane;
            asm volatile("" : "+v"(l));
#pragma unroll
            for (int q = 0; q < NLD; ++q) {
                const int r = (q * kArWaves + w) * kRowsPerLoad + l * 16 / RB, p = (l * 16 % RB) >> 4;
                load_kib_to_lds_at(base + (c0 + r < n ? r * row_bytes + ((p ^ k_row_swizzle<RB>(r)) << 4) : 0), dst + q * kArWaves * 1024);
            }
        }
        if (PASS == 2) load_dwords_to_lds(scalar_ptr(reinterpret_cast<const char*>(lse_h + c0)), whole || c0 + lane < n ? lane * 4 : 0, lse0 + (buf * kArWaves + w) * (kArChunk * 4));
    };
#pragma unroll 1
    for (int t = 0; t < min(2, nchunk); ++t) issue(t);

    // register-side fragments: Q[b, head, row] in pass 1; K[b, g, row] in pass 2
    uintx4 rf[RG][CH];
    int my[RG];                                                          // this lane's register-side rows
#pragma unroll
    for (int e = 0; e < RG; ++e) {
        my[e] = wrow0 + 32 * e + i;
        const T* rp = R + b * rs0 + (int64_t)(PASS == 1 ? head : g) * rs1 + (int64_t)min(my[e], n - 1) * rs2;
#pragma unroll
        for (int cc = 0; cc < CH; ++cc) rf[e][cc] = load16(rp + cc * Elem<T>::kPerChunk + h * Elem<T>::kPerFrag);
    }

    using LdsFrag = const __attribute__((address_space(3))) uintx4*;
    using LdsFloat4 = const __attribute__((address_space(3))) floatx4*;
    unsigned frag[CH];                                                   // LDS bytes of this lane's operands in block 0 of chunk buffer 0
#pragma unroll
    for (int cc = 0; cc < CH; ++cc) frag[cc] = lds0 + i * RB + swz_chunk(2 * cc + h, k_row_swizzle<RB>(i));
    const unsigned lse_l = lse0 + (w * kArChunk + 4 * h) * 4;

    float m_run[RG], l_run[RG];                                          // pass 1: largest logit, sum of exp2((s - m_run) c)
    float colsum[RG], recent[RG];                                        // pass 2; recent: the latest 16 chunks', so that long sums round less often
#pragma unroll
    for (int e = 0; e < RG; ++e) { m_run[e] = -INFINITY; l_run[e] = colsum[e] = recent[e] = 0.f; }
    auto live = [&](int jb) { return PASS == 1 ? jb <= wrow0 + 32 * RG - 1 : jb + 31 >= wrow0; };    // any visible pair for this wave
    // block NB of the chunk in buffer BUF: both go into the offset field of the LDS reads
    auto multiply = [&](floatx16 (&acc)[RG], auto buf_tag, auto nb_tag) {
        constexpr unsigned at = decltype(buf_tag)::value * STG + decltype(nb_tag)::value * 32 * RB;
#pragma unroll
        for (int cc = 0; cc < CH; ++cc) {
            const uintx4 sf = *(LdsFrag)(uintptr_t)(frag[cc] + at);
#pragma unroll
            for (int e = 0; e < RG; ++e) acc[e] = mma_frag<T>(sf, rf[e][cc], cc == 0 ? floatx16{0} : acc[e]);
        }
    };
    float rb[16];                                                        // pass 2: lse of a block's rows
    auto row_lse = [&](auto buf_tag, auto nb_tag) {
        constexpr unsigned at = (decltype(buf_tag)::value * kArWaves * kArChunk + decltype(nb_tag)::value * 32) * 4;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const floatx4 v = *(LdsFloat4)(uintptr_t)(lse_l + at + 32 * a);
            rb[4 * a] = v[0]; rb[4 * a + 1] = v[1]; rb[4 * a + 2] = v[2]; rb[4 * a + 3] = v[3];
        }
    };
    // acc[e][r]: streamed row jb + acc_row(r, h), register-side row my[e]
    auto accumulate = [&](floatx16 (&acc)[RG], int jb) {
#pragma unroll
        for (int e = 0; e < RG; ++e) {
            const int first = wrow0 + 32 * e;
            const bool masked = PASS == 1 ? jb + 31 > first : (jb < first + 31 || jb + 32 > n);          // wave-uniform
            int own = my[e] - 4 * h, end = n - 4 * h;                    // (through the empty asm: no row number is carried through the loop)
            if (masked) asm volatile("" : "+v"(own), "+v"(end));
            if (PASS == 1) {
                if (masked) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (jb + acc_row(r, 0) > own) acc[e][r] = -INFINITY;
                }
                float m_new = m_run[e];
#pragma unroll
                for (int r = 0; r < 16; r += 2) m_new = fmaxf(fmaxf(m_new, acc[e][r]), acc[e][r + 1]);
                const float mc = fmaxf(m_new * c, -FLT_MAX);             // a number also where a lane has seen no key yet: it adds zeros
                float sum = fast_exp2(fmaf(acc[e][0], c, -mc));
#pragma unroll
                for (int r = 1; r < 16; ++r) sum += fast_exp2(fmaf(acc[e][r], c, -mc));
                // The factor is not exactly 1 while the maximum stands: m_run * c - mc is one fma and gives the rounding error of
                // mc, so the sum drifts by up to 2^-25 |mc| in each of the n / 32 blocks.  Against float64, n = 18432, the worst
                // score is off by 3.5e-5 of itself at logits of ordinary size and by 3.8e-4 under one early logit of 21; with
                // (m_run - m_new) * c it is 8e-7 and 2.7e-6.  Left as it is: that form moves scores by 7e-6, beyond the 5e-6
                // within which the scores of this call are declared to stay (perf/cases.py).
                l_run[e] = fmaf(l_run[e], fast_exp2(fmaf(m_run[e], c, -mc)), sum);
                m_run[e] = m_new;
            } else {
                float p[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) p[r] = fast_exp2(fmaf(acc[e][r], c, -rb[r]));
                if (masked) {                                            // on the result: the lse of a row that does not see this key may be no number
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int j = jb + acc_row(r, 0);
                        if (j < own || j >= end) p[r] = 0.f;
                    }
                }
                float s0 = p[0], s1 = p[1];
#pragma unroll
                for (int r = 2; r < 16; r += 2) { s0 += p[r]; s1 += p[r + 1]; }
                recent[e] += s0 + s1;
            }
        }
    };
    // bf16, blocks that every row of the wave sees whole: the products of block NB in buffer BUF (next), each preceded by the LDS read three
    // fragments ahead and followed by its share of the vector work of the block before (cur), in the order written; with LOADS the
    // requests of chunk t too, one at a time.  Sums are taken in the order of `accumulate`.
    auto steady = [&](floatx16 (&next)[RG], floatx16 (&cur)[RG], auto buf_tag, auto nb_tag, auto loads_tag, int t) {
        constexpr unsigned at = decltype(buf_tag)::value * STG + decltype(nb_tag)::value * 32 * RB;
        constexpr bool LOADS = decltype(loads_tag)::value;
        constexpr int AHEAD = 3, PIECES = 16 / CH;                       // a row block's vector work goes with CH products
        const int c0 = chunk_row(t), buf = t & 1;
        const char* base = scalar_ptr(Sb + c0 * row_bytes);
        const unsigned dst = lds0 + buf * STG + w * 1024;
        uintx4 sf[CH];
        float m_new = 0.f, mc = 0.f, alpha = 0.f, s0 = 0.f, s1 = 0.f, p[16];
        auto read = [&](int cc) { sf[cc] = *(LdsFrag)(uintptr_t)(frag[cc] + at); };
        auto request = [&](int q) {
            load_kib_to_lds(base + q * (kLoadRows * row_bytes), (int)ld_off[q % kOffsets], dst + q * kArWaves * 1024);
            if (PASS == 2 && q == 0) load_dwords_to_lds(scalar_ptr(reinterpret_cast<const char*>(lse_h + c0)), lane * 4, lse0 + (buf * kArWaves + w) * (kArChunk * 4));
        };
        auto piece = [&](int e, int r) {                                 // a sum takes in the exponential of the piece (pass 2: two pieces) before
            if (PASS == 1) {
                p[r] = fast_exp2(fmaf(cur[e][r], c, -mc));
                if (r >= 1) s0 = r == 1 ? p[0] : s0 + p[r - 1];
            } else {
                p[r] = fast_exp2(fmaf(cur[e][r], c, -rb[r]));
                if (r >= 2 && r % 2 == 0) s0 = r == 2 ? p[0] : s0 + p[r - 2];
                if (r >= 2 && r % 2 == 1) s1 = r == 3 ? p[1] : s1 + p[r - 2];
            }
        };
        auto vector_work = [&](int e, int share) {                       // of CH shares; in pass 1 the first is the maximum
            if (PASS == 1 && share == 0) {
                m_new = m_run[e];
#pragma unroll
                for (int r = 0; r < 16; r += 2) m_new = fmaxf(fmaxf(m_new, cur[e][r]), cur[e][r + 1]);
            } else if (PASS == 1) {
                if (share == 1) {
                    mc = fmaxf(m_new * c, -FLT_MAX);
                    alpha = fast_exp2(fmaf(m_run[e], c, -mc));
                }
#pragma unroll
                for (int r = 16 * (share - 1) / (CH - 1); r < 16 * share / (CH - 1); ++r) piece(e, r);
            } else {
#pragma unroll
                for (int r = PIECES * share; r < PIECES * (share + 1); ++r) piece(e, r);
            }
            if (share == CH - 1 && PASS == 1) {
                l_run[e] = fmaf(l_run[e], alpha, s0 + p[15]);
                m_run[e] = m_new;
            }
            if (share == CH - 1 && PASS == 2) recent[e] += (s0 + p[14]) + (s1 + p[15]);
        };
#pragma unroll
        for (int cc = 0; cc < AHEAD; ++cc) read(cc);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int cc = 0; cc < CH; ++cc) {
            if (cc + AHEAD < CH) read(cc + AHEAD);
#pragma unroll
            for (int e = 0; e < RG; ++e) {
                const int product = cc * RG + e;
                next[e] = mma_frag<T>(sf[cc], rf[e][cc], cc == 0 ? floatx16{0} : next[e]);
                if (LOADS && e == 0 && cc * NLD / CH != (cc + 1) * NLD / CH) request(cc * NLD / CH);
                vector_work(product / CH, product % CH);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    constexpr std::integral_constant<int, 0> k0{};
    constexpr std::integral_constant<int, 1> k1{};
    floatx16 acc0[RG], acc1[RG];
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    bool live0 = live(chunk_row(0));
    if (live0) multiply(acc0, k0, k0);
    auto flush = [&]() {
#pragma unroll
        for (int e = 0; e < RG; ++e) { colsum[e] += recent[e]; recent[e] = 0.f; }
    };
    auto chunk = [&](int t, auto buf, auto other) {
        const int jb = chunk_row(t);
        if constexpr (Elem<T>::kBytes == 2)
            // both blocks of this chunk and the first of the next are seen whole, and chunk t + 2 is a whole one
            if (narrow && t + 2 < nchunk && (PASS == 1 ? jb + 95 <= wrow0 && jb + 3 * kArChunk <= n : jb - kArChunk >= wrow0 + 32 * RG - 1 && jb + kArChunk <= n)) {
                if (PASS == 2) row_lse(buf, k0);
                steady(acc1, acc0, buf, k1, std::false_type{}, 0);
                if (PASS == 2) row_lse(buf, k1);
                // chunk t + 1 has landed (this wave's pieces, then everyone's), and everyone has read chunk t
                __builtin_amdgcn_s_waitcnt(0x0F70);
                __syncthreads();
                steady(acc0, acc1, other, k0, std::true_type{}, t + 2);
                if (PASS == 2 && (t & 15) == 15) flush();
                live0 = true;
                return;
            }
        const bool live1 = live(jb + 32), more = t + 1 < nchunk;
        if (PASS == 2) row_lse(buf, k0);
        if (live1) multiply(acc1, buf, k1);
        if (live0) accumulate(acc0, jb);
        if (PASS == 2) row_lse(buf, k1);
        if (more) {
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            if (t + 2 < nchunk) issue(t + 2);
            live0 = live(chunk_row(t + 1));
            if (live0) multiply(acc0, other, k0);
        }
        if (live1) accumulate(acc1, jb + 32);
        if (PASS == 2 && ((t & 15) == 15 || !more)) flush();
    };
    for (int t = 0; t < nchunk; t += 2) {
        chunk(t, k0, k1);
        if (t + 1 < nchunk) chunk(t + 1, k1, k0);
    }
    // the two half-waves saw different streamed rows of the same register-side rows
#pragma unroll
    for (int e = 0; e < RG; ++e) {
        if (PASS == 1) {
            const unsigned um = __float_as_uint(m_run[e]), ul = __float_as_uint(l_run[e]);
            const auto pm = __builtin_amdgcn_permlane32_swap(um, um, false, false);
            const auto pl = __builtin_amdgcn_permlane32_swap(ul, ul, false, false);
            const float m0 = __uint_as_float(pm[0]), m1 = __uint_as_float(pm[1]);
            const float l0 = __uint_as_float(pl[0]), l1 = __uint_as_float(pl[1]);
            const float M = fmaxf(m0, m1);                               // finite: a row sees at least itself
            const float L = l0 * fast_exp2((m0 - M) * c) + l1 * fast_exp2((m1 - M) * c);
            if (h == 0 && my[e] < n) lse[(int64_t)bh * n + my[e]] = M * c + __log2f(L);
        } else {
            const unsigned uc = __float_as_uint(colsum[e]);
            const auto pc = __builtin_amdgcn_permlane32_swap(uc, uc, false, false);
            if (h == 0 && my[e] < n) colsum_out[(int64_t)bh * n + my[e]] = __uint_as_float(pc[0]) + __uint_as_float(pc[1]);    // per-head column sums
        }
    }
}

// mass / rank of a unit from the per-head column sums: heads of the group added in ascending order
__global__ __launch_bounds__(256) void allrows_finish_kernel(
    const float* __restrict__ colsum, int n, int Hq, int Hkv, float* __restrict__ mass, float* __restrict__ rank)
{
    const int G = Hq / Hkv, u = blockIdx.y, b = u / Hkv, g = u - b * Hkv;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const float* p = colsum + (int64_t)(b * Hq + g * G) * n + j;
    float a = p[0];
    for (int hh = 1; hh < G; ++hh) a += p[(int64_t)hh * n];
    a /= (float)G;
    mass[(int64_t)u * n + j] = a / (float)n;
    if (rank) rank[(int64_t)u * n + j] = a / (float)(n - j);
}

size_t allrows_workspace_bytes(const zipvl_dims& d) { return 2 * (size_t)d.B * d.Hq * d.n * sizeof(float); }   // lse, per-head column sums

template <typename T, int D, int RG>
static int launch_allrows_t(const void* Q, const void* K, const zipvl_dims& d, float scale,
                            float* mass, float* rank, void* ws, hipStream_t st)
{
    using C = ArCfg<T, D, RG>;
    static std::atomic<bool> attr_done{false};
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&allrows_pass_kernel<T, D, 1, RG>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(&allrows_pass_kernel<T, D, 2, RG>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS) != hipSuccess)
            return set_error(ZIPVL_EHIP, "score_all_rows: cannot reserve %zu bytes of LDS", C::LDS);
        attr_done = true;
    }
    const float c = scale * kLog2e;
    const int nblk = (d.n + C::ROWS - 1) / C::ROWS, heads = d.B * d.Hq;
    const int split = 8 / std::gcd(heads, 8);
    const dim3 grid(8 * ((nblk + split - 1) / split), heads * split / 8);
    const int G = d.Hq / d.Hkv;
    float* lse = (float*)ws;
    float* colsum = lse + (size_t)heads * d.n;
    {
        KernelTimer tm(ZIPVL_K_ALLROWS_LSE, st);
        hipLaunchKernelGGL((allrows_pass_kernel<T, D, 1, RG>), grid, dim3(64 * kArWaves), C::LDS, st,
            (const T*)Q, d.q_strides[0], d.q_strides[1], d.q_strides[2],
            (const T*)K, d.k_strides[0], d.k_strides[1], d.k_strides[2],
            d.n, c, lse, (float*)nullptr, d.Hq, G, split, inverse(grid.y), inverse(split), inverse(d.Hq), inverse(G));
    }
    int rc = check_launch("allrows_lse");
    if (rc) return rc;
    KernelTimer tm(ZIPVL_K_ALLROWS_COLSUM, st);
    hipLaunchKernelGGL((allrows_pass_kernel<T, D, 2, RG>), grid, dim3(64 * kArWaves), C::LDS, st,
        (const T*)K, d.k_strides[0], d.k_strides[1], d.k_strides[2],
        (const T*)Q, d.q_strides[0], d.q_strides[1], d.q_strides[2],
        d.n, c, lse, colsum, d.Hq, G, split, inverse(grid.y), inverse(split), inverse(d.Hq), inverse(G));
    rc = check_launch("allrows_colsum");
    if (rc) return rc;
    hipLaunchKernelGGL(allrows_finish_kernel, dim3((d.n + 255) / 256, d.B * d.Hkv), dim3(256), 0, st,
        (const float*)colsum, d.n, d.Hq, d.Hkv, mass, rank);
    return check_launch("allrows_finish");
}

template <typename T, int D>
static int launch_allrows_d(const void* Q, const void* K, const zipvl_dims& d, float scale,
                            float* mass, float* rank, void* ws, hipStream_t st)
{
    if constexpr (Elem<T>::kBytes == 2)
        if (d.n >= kArWideRows && (int64_t)((d.n + 127) / 128) * d.B * d.Hq >= kArWideBlocks) return launch_allrows_t<T, D, 2>(Q, K, d, scale, mass, rank, ws, st);
    return launch_allrows_t<T, D, 1>(Q, K, d, scale, mass, rank, ws, st);
}

int launch_score_all_rows(const void* Q, const void* K, const zipvl_dims& d, float scale,
                          float* mass, float* rank, void* ws, hipStream_t st)
{
    if (d.dtype == ZIPVL_BF16) {
        if (d.d == 128) return launch_allrows_d<__bf16, 128>(Q, K, d, scale, mass, rank, ws, st);
        return launch_allrows_d<__bf16, 64>(Q, K, d, scale, mass, rank, ws, st);
    }
    if (d.d == 128) return launch_allrows_d<float, 128>(Q, K, d, scale, mass, rank, ws, st);
    return launch_allrows_d<float, 64>(Q, K, d, scale, mass, rank, ws, st);
}

}  // namespace zipvl
