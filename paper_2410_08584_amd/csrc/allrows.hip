// Exact token scores from EVERY row of the attention matrix (Eq. (6) and Eq. (8)
// as written, before the probe approximation of the supplementary material): the
// accuracy reference for the probe scores.  A is never stored.  Two passes of one
// kernel body over the causal half of Q K^T:
//   pass 1  per query row, the exponent offset lse = log2(sum exp2(s c)) of its visible
//           logits (c = softmax scale * log2 e);
//   pass 2  per query head and key column, sum over the rows that see it of exp2(s c - lse);
//           a small kernel then averages the query heads of a group (fixed order) and writes
//           mass = a / n and rank = a / (n - j)  (every row at or after j counts in Eq. (8)).
// A workgroup keeps 32 rows per wave of one side in registers as MFMA fragments (queries in
// pass 1, keys in pass 2) and streams the other side through LDS in chunks of 64 rows, loaded
// straight from global memory, double buffered, one barrier per chunk.  The product is taken as
// (streamed rows) x (register rows)^T on 32x32 tiles, so a lane owns one register-side row and
// its statistic (a running sum) never leaves the lane until the end.
#include <atomic>
#include <numeric>

#include "launch.h"
#include "ldsload.h"

namespace zipvl {

constexpr int kArChunk = 64;      // streamed rows per chunk
constexpr int kArWaves = 4;       // waves per workgroup; 8 (half the streaming traffic) gain 2 % at 28 heads x 18432 and lose 5-50 % where workgroups are few

// What bounds it: a 32x32x128 bf16 tile is 256 matrix cycles and, per lane, 16 x (fma + exp2 + add) (pass 1: + max),
// about 400 vector cycles, and waves overlap the two only in part.  So: staging that needs no registers (three to four
// waves per SIMD) and no barrier but one per 64 rows.  28 heads on 4, n = 18432, d = 128, both passes: 4.97 ms (staged through
// registers, 128-row blocks in no XCD order) -> 2.86 ms.  32 heads, n = 2933: 232 -> 138 us.  Measured and not taken: two row
// groups per wave (each fragment read from LDS feeds two MFMAs; same time, and 1.1-1.5 times slower below 2000
// workgroups), three chunks in flight (52 KiB of LDS, 5 % slower), MFMAs and exponentials interleaved by hand (3-8 %
// slower), a lazily moved offset instead of the running maximum (4 % faster, other roundings).
template <typename T, int D>
struct ArCfg {
    static constexpr int E = Elem<T>::kBytes;
    static constexpr int CH = D / Elem<T>::kPerChunk;       // fragments per row per lane
    static constexpr int RB = D * E;                         // bytes per row
    static constexpr int STG = kArChunk * RB;                // one chunk in LDS (rows unpadded, 16-byte pieces swizzled)
    static constexpr int NLD = STG / 1024 / kArWaves;        // 1-KiB loads per wave and chunk
    static constexpr int ROWS = 32 * kArWaves;               // register-side rows per workgroup
    static constexpr size_t LDS = 2 * ((size_t)STG + kArWaves * kArChunk * sizeof(float));   // two chunks, and their rows' lse (one copy per wave)
};

// Which (head, block of register-side rows) a workgroup takes.  Workgroups go round-robin over the 8 XCDs; every XCD
// gets whole heads (or 1 / split of the blocks of one, where the heads do not divide by 8) so that the rows it streams
// stay in its own L2, the blocks with the most visible pairs first.  Grid: x = (block of the part, XCD), y = part of the XCD;
// neither dimension reaches the launch limits (2^32 threads, 65535) for any dims that are accepted.

template <typename T, int D, int PASS>
__global__ __launch_bounds__(64 * kArWaves, Elem<T>::kBytes == 2 ? 3 : 2) void allrows_pass_kernel(
    const T* __restrict__ R, int64_t rs0, int64_t rs1, int64_t rs2,     // register side: Q (pass 1) / K (pass 2)
    const T* __restrict__ S, int64_t ss0, int64_t ss1, int64_t ss2,     // streamed side: K (pass 1) / Q (pass 2)
    int n, float c, float* __restrict__ lse, float* __restrict__ colsum_out, int Hq, int Hkv, int split)
{
    using C = ArCfg<T, D>;
    constexpr int CH = C::CH, RB = C::RB, NLD = C::NLD, STG = C::STG;
    extern __shared__ __attribute__((aligned(16))) char smem[];          // two chunks, then (pass 2) 2 x kArWaves x kArChunk lse values
    const int G = Hq / Hkv;
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (n + C::ROWS - 1) / C::ROWS;
    const int part = (blockIdx.x & 7) * gridDim.y + blockIdx.y;           // split parts per head
    const int order = __builtin_amdgcn_readfirstlane((blockIdx.x >> 3) * split + part % split);        // scalar from here on
    if (order >= nblk) return;
    const int bh = __builtin_amdgcn_readfirstlane(part / split), b = __builtin_amdgcn_readfirstlane(bh / Hq), head = bh - b * Hq;
    const int g = __builtin_amdgcn_readfirstlane(head / G);
    // heavy blocks first: late queries in pass 1, early keys in pass 2
    const int row0 = (PASS == 1 ? nblk - 1 - order : order) * C::ROWS, wrow0 = row0 + 32 * w;

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
    // this lane's pieces of a chunk: LDS byte o = row r, position p of the row; the piece's offset from the chunk's first row
    const int row_l = lane * 16 / RB;                                    // + (q kArWaves + w) kRowsPerLoad for load q
    constexpr int kRowsPerLoad = 1024 / RB;
    const bool narrow = row_bytes * kArChunk < (int64_t)1 << 31;        // a chunk's offsets fit 32 bits: row strides below 32 MiB
    unsigned ld_off[NLD];
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
        const int r = (q * kArWaves + w) * kRowsPerLoad + row_l, p = (lane * 16 % RB) >> 4;
        ld_off[q] = (narrow ? (unsigned)(r * row_bytes) : 0u) + ((p ^ k_row_swizzle<RB>(r)) << 4);
    }
    // Every wave issues the same number of loads for every chunk; rows past the end re-read the chunk's first one.
    auto issue = [&](int t) {
        const int c0 = chunk_row(t), buf = (t & 1);
        const char* base = scalar_ptr(Sb + c0 * row_bytes);
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const unsigned dst = lds0 + buf * STG + (q * kArWaves + w) * 1024;
            const int r = (q * kArWaves + w) * kRowsPerLoad + row_l;
            if (narrow) load_kib_to_lds(base, c0 + r < n ? (int)ld_off[q] : 0, dst);
            else load_kib_to_lds_at(base + (c0 + r < n ? r * row_bytes + ld_off[q] : 0), dst);
        }
        if (PASS == 2) load_dwords_to_lds(scalar_ptr(reinterpret_cast<const char*>(lse_h + c0)), c0 + lane < n ? lane * 4 : 0, lse0 + (buf * kArWaves + w) * (kArChunk * 4));
    };
#pragma unroll 1
    for (int t = 0; t < min(2, nchunk); ++t) issue(t);

    // register-side fragments: Q[b, head, row] in pass 1; K[b, g, row] in pass 2
    uintx4 rf[CH];
    const int my = wrow0 + i;                                            // this lane's register-side row
    {
        const T* rp = R + b * rs0 + (int64_t)(PASS == 1 ? head : g) * rs1 + (int64_t)min(my, n - 1) * rs2;
#pragma unroll
        for (int cc = 0; cc < CH; ++cc) rf[cc] = load16(rp + cc * Elem<T>::kPerChunk + h * Elem<T>::kPerFrag);
    }

    float m_run = -INFINITY, l_run = 0.f;                                // pass 1: largest logit, sum of exp2((s - m_run) c)
    float colsum = 0.f, recent = 0.f;                                    // pass 2; recent: the latest 16 chunks', so that long sums round less often
    auto live = [&](int jb) { return PASS == 1 ? jb <= wrow0 + 31 : jb + 31 >= wrow0; };    // any visible pair for this wave
    auto multiply = [&](floatx16& acc, int t, int nb) {
        const char* row = smem + (t & 1) * STG + (nb * 32 + i) * RB;
        acc = floatx16{0};
#pragma unroll
        for (int cc = 0; cc < CH; ++cc) {
            const uintx4 sf = *reinterpret_cast<const uintx4*>(row + swz_chunk(2 * cc + h, k_row_swizzle<RB>(i)));
            acc = mma_frag<T>(sf, rf[cc], acc);
        }
    };
    auto row_lse = [&](float (&rb)[16], int t, int nb) {                 // pass 2: lse of the block's rows
        const float* lp = reinterpret_cast<const float*>(smem + 2 * STG) + ((t & 1) * kArWaves + w) * kArChunk + nb * 32 + 4 * h;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const floatx4 v = *reinterpret_cast<const floatx4*>(lp + 8 * a);
            rb[4 * a] = v[0]; rb[4 * a + 1] = v[1]; rb[4 * a + 2] = v[2]; rb[4 * a + 3] = v[3];
        }
    };
    // acc[r]: streamed row jb + acc_row(r, h), register-side row `my`
    auto accumulate = [&](floatx16& acc, const float (&rb)[16], int jb) {
        const bool masked = PASS == 1 ? jb + 31 > wrow0 : (jb < wrow0 + 31 || jb + 32 > n);      // wave-uniform
        if (PASS == 1) {
            if (masked) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (jb + acc_row(r, h) > my) acc[r] = -INFINITY;
            }
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc[r]);
            if (mx > -INFINITY) {
                const float m_new = fmaxf(m_run, mx), mc = m_new * c;
                float sum = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) sum += fast_exp2(fmaf(acc[r], c, -mc));
                // The factor is not exactly 1 while the maximum stands: m_run * c - mc is one fma and gives the rounding error of
                // mc, so the sum drifts by up to 2^-25 |mc| in each of the n / 32 blocks.  Against float64, n = 18432, the worst
                // score is off by 3.5e-5 of itself at logits of ordinary size and by 3.8e-4 under one early logit of 21; with
                // (m_run - m_new) * c it is 8e-7 and 2.7e-6.  Left as it is: that form moves scores by 7e-6, beyond the 5e-6
                // within which the scores of this call are declared to stay (perf/cases.py).
                l_run = l_run * fast_exp2(m_run * c - mc) + sum;
                m_run = m_new;
            }
        } else {
            float p[16], s0 = 0.f, s1 = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) p[r] = fast_exp2(fmaf(acc[r], c, -rb[r]));
            if (masked) {                                                // on the result: the lse of a row that does not see this key may be no number
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = jb + acc_row(r, h);
                    if (j < my || j >= n) p[r] = 0.f;
                }
            }
#pragma unroll
            for (int r = 0; r < 16; r += 2) { s0 += p[r]; s1 += p[r + 1]; }
            recent += s0 + s1;
        }
    };

    floatx16 acc0, acc1;
    float rb0[16], rb1[16];
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    bool live0 = live(chunk_row(0));
    if (live0) multiply(acc0, 0, 0);
    if (PASS == 2) row_lse(rb0, 0, 0);
    for (int t = 0; t < nchunk; ++t) {
        const int jb = chunk_row(t);
        const bool live1 = live(jb + 32), more = t + 1 < nchunk;
        if (live1) multiply(acc1, t, 1);
        if (live0) accumulate(acc0, rb0, jb);
        if (PASS == 2) row_lse(rb1, t, 1);
        if (more) {
            // chunk t + 1 has landed (this wave's pieces, then everyone's), and everyone has read chunk t
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            if (t + 2 < nchunk) issue(t + 2);
            live0 = live(chunk_row(t + 1));
            if (live0) multiply(acc0, t + 1, 0);
            if (PASS == 2) row_lse(rb0, t + 1, 0);
        }
        if (live1) accumulate(acc1, rb1, jb + 32);
        if (PASS == 2 && ((t & 15) == 15 || !more)) { colsum += recent; recent = 0.f; }
    }
    // the two half-waves saw different streamed rows of the same register-side row
    if (PASS == 1) {
        const unsigned um = __float_as_uint(m_run), ul = __float_as_uint(l_run);
        const auto pm = __builtin_amdgcn_permlane32_swap(um, um, false, false);
        const auto pl = __builtin_amdgcn_permlane32_swap(ul, ul, false, false);
        const float m0 = __uint_as_float(pm[0]), m1 = __uint_as_float(pm[1]);
        const float l0 = __uint_as_float(pl[0]), l1 = __uint_as_float(pl[1]);
        const float M = fmaxf(m0, m1);                                   // finite: a row sees at least itself
        const float L = l0 * fast_exp2((m0 - M) * c) + l1 * fast_exp2((m1 - M) * c);
        if (h == 0 && my < n) lse[(int64_t)bh * n + my] = M * c + __log2f(L);
    } else {
        const unsigned uc = __float_as_uint(colsum);
        const auto pc = __builtin_amdgcn_permlane32_swap(uc, uc, false, false);
        if (h == 0 && my < n) colsum_out[(int64_t)bh * n + my] = __uint_as_float(pc[0]) + __uint_as_float(pc[1]);    // per-head column sums
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

template <typename T, int D>
static int launch_allrows_t(const void* Q, const void* K, const zipvl_dims& d, float scale,
                            float* mass, float* rank, void* ws, hipStream_t st)
{
    using C = ArCfg<T, D>;
    static std::atomic<bool> attr_done{false};
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&allrows_pass_kernel<T, D, 1>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(&allrows_pass_kernel<T, D, 2>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS) != hipSuccess)
            return set_error(ZIPVL_EHIP, "score_all_rows: cannot reserve %zu bytes of LDS", C::LDS);
        attr_done = true;
    }
    const float c = scale * kLog2e;
    const int nblk = (d.n + C::ROWS - 1) / C::ROWS, heads = d.B * d.Hq;
    const int split = 8 / std::gcd(heads, 8);
    const dim3 grid(8 * ((nblk + split - 1) / split), heads * split / 8);
    float* lse = (float*)ws;
    float* colsum = lse + (size_t)heads * d.n;
    {
        KernelTimer tm(ZIPVL_K_ALLROWS_LSE, st);
        hipLaunchKernelGGL((allrows_pass_kernel<T, D, 1>), grid, dim3(64 * kArWaves), C::LDS, st,
            (const T*)Q, d.q_strides[0], d.q_strides[1], d.q_strides[2],
            (const T*)K, d.k_strides[0], d.k_strides[1], d.k_strides[2],
            d.n, c, lse, (float*)nullptr, d.Hq, d.Hkv, split);
    }
    int rc = check_launch("allrows_lse");
    if (rc) return rc;
    KernelTimer tm(ZIPVL_K_ALLROWS_COLSUM, st);
    hipLaunchKernelGGL((allrows_pass_kernel<T, D, 2>), grid, dim3(64 * kArWaves), C::LDS, st,
        (const T*)K, d.k_strides[0], d.k_strides[1], d.k_strides[2],
        (const T*)Q, d.q_strides[0], d.q_strides[1], d.q_strides[2],
        d.n, c, lse, colsum, d.Hq, d.Hkv, split);
    rc = check_launch("allrows_colsum");
    if (rc) return rc;
    hipLaunchKernelGGL(allrows_finish_kernel, dim3((d.n + 255) / 256, d.B * d.Hkv), dim3(256), 0, st,
        (const float*)colsum, d.n, d.Hq, d.Hkv, mass, rank);
    return check_launch("allrows_finish");
}

int launch_score_all_rows(const void* Q, const void* K, const zipvl_dims& d, float scale,
                          float* mass, float* rank, void* ws, hipStream_t st)
{
    if (d.dtype == ZIPVL_BF16) {
        if (d.d == 128) return launch_allrows_t<__bf16, 128>(Q, K, d, scale, mass, rank, ws, st);
        return launch_allrows_t<__bf16, 64>(Q, K, d, scale, mass, rank, ws, st);
    }
    if (d.d == 128) return launch_allrows_t<float, 128>(Q, K, d, scale, mass, rank, ws, st);
    return launch_allrows_t<float, 64>(Q, K, d, scale, mass, rank, ws, st);
}

}  // namespace zipvl
