// Attention over the kept tokens (Section 4.2; Algorithm 1, sparse-attention
// step; Eq. (2) restricted to the important set T).
//
// Two kernels:
//   pack   gathers K[T] and V[T] into the workspace, once per KV head, zero-filling
//          the ragged tail.  An evicted cache with contiguous rows is read in place and
//          nothing is packed at all (the P.V operand comes from row-major V tiles in LDS
//          through the transposing read).
//   flash  one workgroup = 128 kept queries of one query head (4 waves x 32
//          rows; 64 where there are few, two waves then share 32 rows and halve
//          the keys of every tile).  K / V tiles of 64 keys are loaded straight into LDS (double
//          buffered) and shared by the four waves.  S^T = K Q^T and O^T = V^T P^T
//          are taken on 32x32 MFMA tiles, so a lane owns one query column and the
//          softmax statistics are per-lane scalars.  The key loop is a pipeline
//          three tiles deep: a step multiplies P.V for tile t-1, takes the
//          exponentials of tile t and multiplies K Q^T for tile t+1, with the
//          instruction order of the steady state written out (operand reads a few
//          matrix instructions ahead, the vector work and the tile requests spread
//          between them); every tile has a whole step to arrive from memory.
//          The first pass over the keys uses no exponent offset at all (no running
//          maximum, no exchange between lanes, no rescaling): exp2 of the scaled
//          logits as they are.  That is exact as long as the row sums stay far
//          inside the fp32 range, which is checked at the end; a workgroup with a
//          row outside [2^-64, 2^64] repeats its tiles with running maxima.
//          Causality is the plain lower triangle in kept-token coordinates because
//          T is ascending.  Query rows are gathered by idx on load, output rows are
//          scattered by idx on store.  The zero rows of dropped tokens are written
//          by extra workgroups at the end of the same grid (one per head and span
//          of positions), which run in the slots the thinning end of the
//          attention work leaves idle.
//          fp32 rows are split into three bf16 planes on their way into LDS, and a product
//          is taken as six of planes (flash_queries_f32).
// The kept count k lives on the device: the grid covers the worst case (k = n),
// but every workgroup knows the tiles of the longest head, so that those without
// work stand at the end of the grid; heavy (late) query tiles are scheduled first,
// over all KV heads of a schedule group, because the longest workgroup (all k keys)
// lasts a large part of the whole launch.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "launch.h"
#include "ldsload.h"

namespace zipvl {

constexpr int kBN = 64;      // keys per tile
// Launch shape: 4 waves x 32 queries, or (launch_prefill_t) 2 x 32 queries x 2 key blocks.  Measured alternatives: 8 waves per
// workgroup (half the L2 -> LDS traffic per query) is 3 % slower; 64 queries per wave (half the LDS operand reads per
// MFMA) does not fit the register file with the S^T double buffer and spills.
constexpr int kFillSpan = 512;       // positions per workgroup that clears dropped output rows
// Every workgroup reads all kept counts of a call (64 a load) unless they are more than kScanSets; a call of up to kScanBlocks
// workgroups is on the chip at once in whatever order, and the reading costs it 0.3 us of 11.
constexpr int kScanSets = 512, kScanBlocks = 512;
// Workgroups of the grid above which a head gets fewer of them than it has tiles if all is kept (half at least; the others are
// taken in a second round).  us, a row for every tile -> so: 4 x 32 heads, n = 8192, a quarter kept 209 -> 204, half kept 611 -> 612;
// 2 x 32, n = 12000, 15 % kept 92.6 -> 90.4; with half as many workgroups 207, 639 and 89.9.
constexpr int kSecondRound = 4096;
// Rows of workgroups from which a group of a multiple of 8 heads of a set, each with its own K / V, is turned by a head every kTurnRows rows.
// Workgroups go to the 8 XCDs in turn, so that a head is one XCD's, and heads keep different numbers of tokens.  us, every row alike -> so:
// 15 % more and less than half kept, 2 x 4 heads, n = 28000 407 -> 370, 4 x 4, d = 64 504 -> 437, 32, n = 25000, 40 % 838 -> 793, 3 x 8, n = 25000, 40 %
// 613 -> 590; by a head every row 374, 460, 833, 644; short ones lose the rows of a head that share its K / V on the way: 4 x 32, n = 8192, a
// quarter 195 -> 214, 32, n = 2933 22 -> 25 by a head every row.
constexpr int kTurnFrom = 64, kTurnRows = 4;
constexpr float kLazyLog2 = 8.f;     // slack of the running softmax offset below the running maximum (log2 domain)
constexpr float kSumLow = 0x1p-64f, kSumHigh = 0x1p64f;   // row sums of the offset-free pass that need no second pass
// fp32 in planes: magnitudes (other than 0) of outputs, and of queries, outside which the tiles are repeated in fp32 products
constexpr float kOutLow = 0x1p-80f, kQueryLow = 0x1p-100f, kQueryHigh = 0x1p90f;
template <int D> constexpr int kPlanesLine = D == 64 ? 900 : 600;   // fp32: live tiles up to which a head's keys are split (splits_keys)
constexpr int kSchedAhead = 3;       // LDS operand reads in flight ahead of the consuming MFMA

// fp32 (flash_queries_f32): K and V as three bf16 planes each in LDS
template <int D, int KS>
struct SplitCfg {
    static constexpr int NW = KS == 4 ? 8 : 4;               // waves; 32 NW / KS queries
    static constexpr int TK = 32 * KS;                       // keys per tile: a 32-key block for every wave
    static constexpr int RB = 2 * D;                         // bytes per row of a plane
    static constexpr int PLANE = TK * RB;
    // Three planes of K and three of V, or (d = 128, KS > 1) three that K and V take in turns.  The pass in fp32 products has a tile
    // of K and one of V.
    static constexpr bool kShared = D == 128 && KS > 1;
    static constexpr int LDS_BYTES = kShared ? 2 * TK * D * 4 : 6 * PLANE;
    static_assert(KS == 1 || 64 * NW * D * 2 <= LDS_BYTES, "room for the sums of all waves");
    static_assert(!kShared || 3 * PLANE + 32 * NW / KS * RB <= LDS_BYTES, "room for a plane of Q");
    static constexpr int LPR = D / 8;                        // lanes per row when a tile is converted (8 elements each)
    static constexpr int RPP = 64 * NW / LPR, NP = TK / RPP;     // rows per pass of the workgroup, passes
    static constexpr int CH = D / 16, ODB = D / 32;
};

// NW = waves per workgroup, of 32 queries each: a workgroup covers 32 NW kept queries, its K / V^T tiles are
// fetched from L2 once per that many queries.
// KS = 2: two waves share 32 queries and take one 32-key block of every tile each (their sums meet at the end).
template <typename T, int D, int NW = 4, int KS = 1>
struct AttnCfg {
    static constexpr int E = Elem<T>::kBytes;
    static constexpr int BM = 32 * NW / KS;                  // queries per workgroup
    static constexpr int NBK = 2 / KS;                       // 32-key blocks of a tile per wave
    static constexpr int NT = 64 * NW;                       // threads per workgroup
    static constexpr int CH = D / Elem<T>::kPerChunk;       // Q/K fragments per row per lane
    static constexpr int ODB = D / 32;                       // 32-row blocks of O^T
    // LDS tiles are unpadded; the 16-byte chunks of a row are XOR-swizzled with the row index instead, so
    // that 16 consecutive rows read at the same logical chunk hit 16 different bank groups.
    static constexpr int KRB = D * E;                        // bytes per K row
    static constexpr int VRB = D * E;                        // bytes per V row
    static constexpr int TILE_BYTES = kBN * D * E;           // one K tile = one V tile
    static constexpr int NLD = TILE_BYTES / 1024 / NW;       // 1-KiB direct-to-LDS loads per wave per tile
    static constexpr int LDS_BYTES = E == 4 ? SplitCfg<D, KS>::LDS_BYTES : 4 * TILE_BYTES + 256 * NW;     // two K and two V buffers, positions of a wave's queries
    // two waves per SIMD (<= 256 registers, accumulators stay in VGPRs), three for fp32 at d = 64 in workgroups of four
    static constexpr int MIN_WGS = E == 4 ? (D == 64 && NW == 4 ? 3 : 2) : 8 / NW;
};

// ------------------------------------------------------------------ pack
template <typename T, int D>
__global__ __launch_bounds__(256) void pack_kv_kernel(
    const T* __restrict__ K, const T* __restrict__ V,
    int64_t ks0, int64_t ks1, int64_t ks2, int64_t vs0, int64_t vs1, int64_t vs2,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ kcnt,
    T* __restrict__ Kp, T* __restrict__ Vp, int n, int npad, int Hkv, int rows_are_kept, int skip_k, int skip_v, int t_per_batch)
{
    constexpr int EPF = Elem<T>::kPerFrag;
    constexpr int CPR = D / EPF, kPass = 256 / CPR, kPasses = kBN / kPass;
    const int u = blockIdx.y, b = u / Hkv, g = u - b * Hkv;
    const int t0 = blockIdx.x * kBN;
    const int ut = t_per_batch ? b : u;                   // row of idx / k that holds this unit's T
    int kk = kcnt ? kcnt[ut] : n;
    kk = max(0, min(kk, n));
    if (t0 >= kk) return;
    const T* Kb = K + b * ks0 + g * ks1;
    const T* Vb = V + b * vs0 + g * vs1;
    // Positions, then rows: all of a thread's are requested at once, as in compact_kv.  One after the other (each behind a branch on
    // whether it is packed at all): 4 x 32 heads on 8, bf16, d = 128, n = 1500, a tenth kept 23.1 us a call (20.6 so), fp32 60.4 (55.7).
    const int cc = threadIdx.x % CPR, r1 = t0 + threadIdx.x / CPR;
    int src[kPasses];
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
        const int row = min(r1 + p * kPass, kk - 1);
        src[p] = (idx && !rows_are_kept) ? idx[(int64_t)ut * n + row] : row;
    }
    uintx4 kr[kPasses] = {}, vr[kPasses] = {};
    if (!skip_k)
#pragma unroll
        for (int p = 0; p < kPasses; ++p) kr[p] = load16(Kb + (int64_t)src[p] * ks2 + cc * EPF);
    if (!skip_v)
#pragma unroll
        for (int p = 0; p < kPasses; ++p) vr[p] = load16(Vb + (int64_t)src[p] * vs2 + cc * EPF);
    const int64_t out = ((int64_t)u * npad + r1) * D + cc * EPF;
    if (!skip_k)
#pragma unroll
        for (int p = 0; p < kPasses; ++p) store16(Kp + out + p * kPass * D, r1 + p * kPass < kk ? kr[p] : uintx4{0, 0, 0, 0});   // rows past k are zero rows
    if (!skip_v)
#pragma unroll
        for (int p = 0; p < kPasses; ++p) store16(Vp + out + p * kPass * D, r1 + p * kPass < kk ? vr[p] : uintx4{0, 0, 0, 0});
}

// ------------------------------------------------------------------ flash
// One tile (TILE_BYTES contiguous in global memory) -> one LDS buffer, without passing through
// registers: every wave issues NLD loads of 1 KiB, lane L of a load writes LDS bytes [16 L, 16 L + 16)
// of that KiB, and picks the global chunk that belongs there under the row swizzle.


// per-lane source offsets for tile_to_lds (rows of RB bytes)
// Row swizzle of a row-major bf16 V tile (rows of RB bytes): the transposing read of a 16-lane group
// touches 4 consecutive keys x 4 consecutive 16-byte chunks, so the key index goes into chunk bits 2..3
// (one bit of it is already an address bit when two rows share a 256-byte bank period).
template <int RB>
__device__ __forceinline__ int v_row_swizzle(int row) { return ((row & 3) >> (RB == 128 ? 1 : 0)) << 2; }

template <int RB, int NW, int NLD, bool V = false>
__device__ __forceinline__ void lds_fill_offsets(int w, int lane, int (&off)[NLD]) {
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
        const int o = (q * NW + w) * 1024 + lane * 16;
        const int r = o / RB, p = (o % RB) >> 4;
        off[q] = r * RB + ((p ^ (V ? v_row_swizzle<RB>(r) : k_row_swizzle<RB>(r))) << 4);
    }
}

// Load q of a tile (see tile_to_lds).  When the NW KiB that the waves fetch together cover a whole number of
// swizzle periods (16 rows), a lane's offset inside every such group is the same: one register serves all
// loads and the group's offset goes into the scalar base address.
template <int RB, int NW> constexpr bool kOffsetsRepeat = (NW * 1024 / RB) % 16 == 0;

template <int RB, int NW, int NLD>
__device__ __forceinline__ void tile_load(const char* gtile, int q, const int (&off)[NLD], unsigned lds_dst) {
    if constexpr (kOffsetsRepeat<RB, NW>) load_kib_to_lds(gtile + q * NW * 1024, off[0], lds_dst);
    else load_kib_to_lds(gtile, off[q], lds_dst);
}
// the same for whole tiles, placed by data flow (load_kib_to_lds_pinned)
template <int RB, int NW, int NLD>
__device__ __forceinline__ void tile_load_pinned(const char* gtile, int q, const int (&off)[NLD], unsigned lds_dst, unsigned& pin) {
    if constexpr (kOffsetsRepeat<RB, NW>) load_kib_to_lds_pinned(gtile + q * NW * 1024, off[0], lds_dst, pin);
    else load_kib_to_lds_pinned(gtile, off[q], lds_dst, pin);
}

// Only the first `rows` rows of the tile may be read: fewer than kBN happens once per head, at its last tile, and the
// rows after them are then filled from the last one, chunk for chunk.  That form derives its offsets again from the
// thread index, so that the key loop carries nothing for it.
template <int RB, int NW, int NLD, bool V = false>
__device__ __forceinline__ void tile_to_lds(const char* gtile, unsigned lds_dst, const int (&off)[NLD], int rows) {
    if (rows >= kBN) {
#pragma unroll
        for (int q = 0; q < NLD; ++q) tile_load<RB, NW, NLD>(gtile, q, off, lds_dst + q * NW * 1024);
    } else {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
#pragma unroll 1
        for (int q = 0; q < NLD; ++q) {
            const int o = q * NW * 1024 + tid * 16, r = o / RB, p = (o % RB) >> 4;
            const int chunk = (p ^ (V ? v_row_swizzle<RB>(r) : k_row_swizzle<RB>(r))) << 4;
            load_kib_to_lds(gtile, min(r, rows - 1) * RB + chunk, lds_dst + q * NW * 1024);
        }
    }
}

// S^T = K Q^T for 32 keys (block blk of the 64-key tile in LDS buffer kb) and the wave's queries:
// acc[blk][r] = key 32*blk + acc_row(r, h), this lane's query.
template <typename T, int D, int NW, int KS>
__device__ __forceinline__ void qk_block(const char* kb, int blk, int i, int h, int sw,
                                         const uintx4 (&qf)[AttnCfg<T, D, NW, KS>::CH], floatx16 (&acc)[AttnCfg<T, D, NW, KS>::NBK]) {
    using C = AttnCfg<T, D, NW, KS>;
    floatx16 a = {0};
#pragma unroll
    for (int cc = 0; cc < C::CH; ++cc) {
        const uintx4 kf = *reinterpret_cast<const uintx4*>(kb + (blk * 32 + i) * C::KRB + swz_chunk(2 * cc + h, sw));
        a = mma_frag<T>(kf, qf[cc], a);
    }
    acc[blk] = a;
}

// O^T += V^T P^T for the 32 keys of half HALF: p[HALF] holds the probabilities of S^T block HALF.
template <typename T, int D, int NW, int KS> struct PV;

template <int D, int NW, int KS> struct PV<__bf16, D, NW, KS> {
    using C = AttnCfg<__bf16, D, NW, KS>;
    // p[blk][s2]: the probabilities of S^T block blk as P^T operand fragments.  Contraction slot t of
    // this lane <-> key 16*s2 + 8*(t/4) + 4*h + t%4 of the block = accumulator register 8*s2 + t.
    using Probs = uintx4[C::NBK][2];
    // The matching V^T operand (lane = channel 32 db + lane % 32, slots = those 8 keys) comes from the
    // row-major V tile through ds_read_b64_tr_b16: in every group of 16 lanes, lane 4e + q supplies the
    // address of 4 consecutive channels of key e, and lane l receives channel l of keys 0..3.  Two reads
    // (keys +0..3 and +8..11 relative to 16 s2 + 4 h) make one operand.  lane_off[db]: this lane's
    // supplier address inside a tile for channel block db (row swizzle included).
    __device__ static __forceinline__ void lane_offsets(int lane, int (&lane_off)[C::ODB]) {
        const int h = lane >> 5, grp = (lane >> 4) & 1, e = (lane >> 2) & 3, q = lane & 3;
        const int row = 4 * h + e;                           // key inside its group of 8 = swizzle of the row
#pragma unroll
        for (int db = 0; db < C::ODB; ++db)
            lane_off[db] = row * C::VRB + swz_chunk(4 * db + 2 * grp + (q >> 1), v_row_swizzle<C::VRB>(row)) + (q & 1) * 8;
    }
    template <int HALF>
    __device__ static __forceinline__ void run(const char* vb, const int (&lane_off)[C::ODB], const Probs& p,
                                               floatx16 (&o)[C::ODB]) {
        typedef short shortx4 __attribute__((ext_vector_type(4)));
        using lds_ptr = __attribute__((address_space(3))) shortx4*;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
#pragma unroll
            for (int db = 0; db < C::ODB; ++db) {
                const char* a0 = vb + lane_off[db] + (32 * HALF + 16 * s2) * C::VRB;
                const uintx2 lo = __builtin_bit_cast(uintx2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)a0));
                const uintx2 hi = __builtin_bit_cast(uintx2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(a0 + 8 * C::VRB)));
                const uintx4 vf = {lo[0], lo[1], hi[0], hi[1]};
                o[db] = mma_frag<__bf16>(vf, p[HALF][s2], o[db]);
            }
        }
    }
};

// The two half-waves (lanes l and l ^ 32) hold the two halves of each query's keys: combine a per-lane
// value across them with one register swap (no trip through LDS).
__device__ __forceinline__ float xhalf_max(float v) {
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);   // r[0] = lower halves twice, r[1] = upper halves twice
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float v) {
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <typename T> __device__ __forceinline__ void store_out4(T* dst, float a, float b, float c, float d);
template <> __device__ __forceinline__ void store_out4<float>(float* dst, float a, float b, float c, float d) {
    *reinterpret_cast<floatx4*>(dst) = floatx4{a, b, c, d};
}
template <> __device__ __forceinline__ void store_out4<__bf16>(__bf16* dst, float a, float b, float c, float d) {
    *reinterpret_cast<uintx2*>(dst) = uintx2{pack_bf16x2(a, b), pack_bf16x2(c, d)};
}

// The kept queries i0 ... i0 + BM - 1 of one head by one workgroup.  Q: rows of the head; Kp, Vp: rows of its unit; O: of the head.
template <typename T, int D, int NW, int KS>
__device__ __forceinline__ void flash_queries(const T* __restrict__ Q, int64_t qs2, const T* __restrict__ Kp, const T* __restrict__ Vp,
                                              const int32_t* __restrict__ tidx, T* __restrict__ O, int i0, int kk, int npad, float c,
                                              int out_compact, int k_in_place, int v_in_place)
{
    using C = AttnCfg<T, D, NW, KS>;
    constexpr int kBM = C::BM, kRW = 32;                     // queries per workgroup, queries per wave
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int tid = threadIdx.x;
    if constexpr (KS == 1) asm volatile("" : "+v"(tid));     // nothing of a lane is kept from one tile of queries for the next
    const int w = tid >> 6, lane = tid & 63, i = lane & 31, h = lane >> 5;
    // KS = 2: wave w has the queries of wave qw and key block kw of every tile
    const int qw = KS == 1 ? w : w % (NW / KS), kw = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(w / (NW / KS));
    floatx16 o[C::ODB];
    float m_run, l_run;

    const int ntiles = (min(i0 + kBM, kk) + kBN - 1) / kBN;
    const int wave_first_row = i0 + kRW * qw, wave_last_row = wave_first_row + kRW - 1;
    const int key_room = min(wave_last_row, kk - 1) - 32 * kw;
    // later tiles lie wholly in this wave's future
    const int my_tiles = KS == 1 ? min(ntiles, wave_last_row / kBN + 1) : key_room >= 0 ? min(ntiles, key_room / kBN + 1) : 0;
    const char* kg = reinterpret_cast<const char*>(Kp);   // row-major kept rows of this unit
    const char* vg = reinterpret_cast<const char*>(Vp);
    // An evicted cache that is read in place need not hold a row at or beyond k: the tile with row k - 1 is loaded as far
    // as that row (what stands for later rows is masked and weighs nothing).  Packed tiles are whole.  The steps that
    // request it run outside the steady state: at most 1 us of 289 at 128 heads x 8192 tokens.
    const int krows = k_in_place ? kk : npad, vrows = v_in_place ? kk : npad;
    const int whole_tiles = min(krows, vrows) / kBN;
    const int steady_end = ntiles <= whole_tiles ? ntiles : whole_tiles - 2;   // the steps before this request whole tiles only
    char* const Kb0 = smem;
    char* const Vb0 = smem + 2 * C::TILE_BYTES;
    const int sw = k_row_swizzle<C::KRB>(i);
    int koff[C::NLD], voff[C::NLD];
    lds_fill_offsets<C::KRB, NW, C::NLD>(w, lane, koff);
    lds_fill_offsets<C::VRB, NW, C::NLD, true>(w, lane, voff);
    int vlane[C::ODB];
    PV<T, D, NW, KS>::lane_offsets(lane, vlane);

    const unsigned klds = lds_address(Kb0) + w * 1024, vlds = lds_address(Vb0) + w * 1024;
    auto load_k = [&](int t, int buf) {
        tile_to_lds<C::KRB, NW, C::NLD>(kg + (int64_t)t * C::TILE_BYTES, klds + buf * C::TILE_BYTES, koff, krows - t * kBN);
    };
    auto load_v = [&](int t, int buf) {
        tile_to_lds<C::VRB, NW, C::NLD, true>(vg + (int64_t)t * C::TILE_BYTES, vlds + buf * C::TILE_BYTES, voff, vrows - t * kBN);
    };
    // Positions, then the first key tiles, then query rows, all straight into LDS: the rows wait for the positions only (a load into
    // registers would wait for the tiles too), and a load asks for whole rows (fragment by fragment, 16 bytes of a row a lane, a wave's
    // took the address unit 64 clocks a load).  KS = 2 without a set asks for the rows first, and takes them while the tiles are on their way
    // (KS = 1 so: 3 x 40 heads, n = 390 16.6 -> 17.3).  The rows lie where
    // V tiles go from the first step on, in the swizzle of K rows; KS = 2 leaves room there for the first V tile, asked for as early.  A workgroup of
    // 17 steps had its rows 3.2 us after it asked for tiles, 3.0 so; with the rows of the output (below), calls with their sets and caches,
    // us: 4 x 32 heads, a third kept, n = 4000 120 -> 115, 32, n = 2933 39.7 -> 38.6, 28 on 4, n = 18432, 39 % 358 -> 353, d = 64, 3 x 40, n = 8000, a fifth 109.5 -> 107.
    // Where the longest tile has few queries there is little to gather, and it ends the call: every token kept, us, fragment by fragment, behind all tiles and before the first
    // V tile, now: 4 heads, n = 583 12.8, 13.2, 12.9; 8, n = 1300 19.8, 20.1, 19.8; n = 900 16.0, 16.5, 16.2; full ones 4 x 4, n = 300 10.9, 10.6, 10.3, 28 on 4, n = 583 14.8, 14.3, 14.2.
    constexpr int kRowLanes = C::KRB / 16, kRowsAtOnce = 64 / kRowLanes, kQueryLoads = 32 / kRowsAtOnce;
    char* const held = smem + 4 * C::TILE_BYTES + w * 256;
    char* const rows_lds = KS == 1 ? Vb0 + w * 32 * C::KRB : Vb0 + C::TILE_BYTES + qw * 32 * C::KRB;     // KS = 2: two waves load the same bytes to the same place
    auto request_first_tiles = [&]() {
        load_k(0, 0);
        if (ntiles > 1) load_k(1, 1);
    };
    const int first = i0 + kRW * qw;
    auto request_rows = [&](auto position) {
#pragma unroll
        for (int q = 0; q < kQueryLoads; ++q) {
            const int r = q * kRowsAtOnce + lane / kRowLanes;
            load_kib_to_lds_at(reinterpret_cast<const char*>(Q + (int64_t)position(r) * qs2) + swz_chunk(lane % kRowLanes, k_row_swizzle<C::KRB>(r)),
                               lds_address(rows_lds) + q * 1024);
        }
    };
    if (tidx) load_dwords_to_lds(reinterpret_cast<const char*>(tidx), min(first + i, kk - 1) * 4, lds_address(held));
    else if (KS == 2) request_rows([&](int r) { return min(first + r, kk - 1); });
    request_first_tiles();
    if (!tidx && KS == 1) request_rows([&](int r) { return min(first + r, kk - 1); });
    if (tidx) {
        if (ntiles > 1) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * C::NLD) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(C::NLD) : "memory");
        request_rows([&](int r) { return *reinterpret_cast<const int*>(held + 4 * r); });
    }
    const int qrow = first + i;                              // kept-token coordinate of this lane's query
    uintx4 qf[C::CH];
    if constexpr (KS == 2) load_v(0, 0);
    if (KS == 2 && !tidx && ntiles > 1) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(3 * C::NLD) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(KS == 2 ? C::NLD : 0) : "memory");
#pragma unroll
    for (int cc = 0; cc < C::CH; ++cc) qf[cc] = *reinterpret_cast<const uintx4*>(rows_lds + i * C::KRB + swz_chunk(2 * cc + h, sw));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    // One pass over the key tiles.  SAFE = false: the exponent offset stays 0 (softmax is shift invariant, and
    // floating point keeps its relative precision at any magnitude), so there is no running maximum, no
    // exchange between lanes and no rescaling in the loop; valid as long as the row sums stay far inside the
    // fp32 range, which is checked afterwards.  SAFE = true: the offset follows the running maximum.
    auto pass = [&](auto safe_tag) {
    constexpr bool SAFE = decltype(safe_tag)::value;
    using Probs = typename PV<T, D, NW, KS>::Probs;
    m_run = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int db = 0; db < C::ODB; ++db) o[db] = floatx16{0};
    // Software pipeline over key tiles, three stages deep.  Step t runs, on the matrix cores, P.V of tile
    // t-1 (first half) and the S^T product of tile t+1 (second half), and on the vector ALU the
    // exponentials of tile t: the three work on different tiles, so nothing inside a step waits for
    // anything else inside it.  K tile t+2 is requested in the first half of step t and first read in the
    // second half of step t+1; V tile t+1 is requested in the second half of step t and first read at the
    // start of step t+2: every tile has a whole step to arrive.  Two barriers per step (middle and end),
    // each preceded by a wait that leaves this wave's two most recent tile requests outstanding.
    if constexpr (SAFE) request_first_tiles();                  // the first pass requested them before the query rows
    if constexpr (SAFE && KS == 2) load_v(0, 0);
    if constexpr (KS == 2) __builtin_amdgcn_s_waitcnt(0x0070 | C::NLD);
    else __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if constexpr (KS == 1) load_v(0, 0);
    floatx16 sa[C::NBK], sb[C::NBK];
    Probs pa, pb;
    qk_block<T, D, NW, KS>(Kb0 + kw * 32 * C::KRB, 0, i, h, sw, qf, sa);       // tile 0 is visible to every row
    if constexpr (KS == 1) qk_block<T, D, NW, KS>(Kb0, 1, i, h, sw, qf, sa);
    __syncthreads();                                         // step 0 overwrites K tile 0

    // wait until at most `pending` of this wave's tile requests (NLD loads each) are outstanding, and for its LDS reads
    auto wait_tiles = [&](int pending) {
        if (pending >= 2) __builtin_amdgcn_s_waitcnt(0x0070 | ((2 * C::NLD) & 15) | (((2 * C::NLD) >> 4) << 14));
        else __builtin_amdgcn_s_waitcnt(0x0070);
    };
    // The two halves of a steady-state step with the instruction order written
    // out.  Every matrix instruction is followed by its share of the half's vector work (16 pieces: two
    // products, two exponentials, a pack and a row-sum update per pair of keys) and preceded by the LDS reads
    // of the operand kSchedAhead matrix instructions ahead; nothing moves across the fences between them.
    // HALF 0: P.V of the previous tile (src = its V tile), exponentials of key block 0, requests for a K tile.
    // HALF 1: S^T of the next tile (src = its K tile), exponentials of key block 1, requests for a V tile.
    static_assert(Elem<T>::kBytes == 2, "the order below is for bf16");
    auto steady_half = [&](auto half_tag, const char* src, floatx16 (&sc)[C::NBK], floatx16 (&sn)[C::NBK], Probs& pp, Probs& pc,
                           float& sum, const char* gt, unsigned lt) {
        constexpr int HALF = decltype(half_tag)::value;
        constexpr int NM = (HALF == 0 ? 4 * C::ODB : 2 * C::CH) / KS;  // matrix instructions of the half
        constexpr int PPM = 16 / KS / NM;                           // vector pieces per matrix instruction
        constexpr int BLK = KS == 1 ? HALF : 0;                     // key block whose exponentials these are
        typedef short shortx4 __attribute__((ext_vector_type(4)));
        using lds_ptr = __attribute__((address_space(3))) shortx4*;
        uintx4 frag[NM];
        float pe[16];
        auto read = [&](int j) {
            if constexpr (HALF == 0) {
                const int hf = j / (2 * C::ODB), s2 = (j / C::ODB) & 1, db = j % C::ODB;
                const char* a0 = src + vlane[db] + (32 * hf + 16 * s2) * C::VRB;
                const uintx2 lo = __builtin_bit_cast(uintx2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)a0));
                const uintx2 hi = __builtin_bit_cast(uintx2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(a0 + 8 * C::VRB)));
                frag[j] = uintx4{lo[0], lo[1], hi[0], hi[1]};
            } else {
                const int blk = KS == 1 ? j & 1 : 0, cc = KS == 1 ? j >> 1 : j;
                frag[j] = *reinterpret_cast<const uintx4*>(src + (blk * 32 + i) * C::KRB + swz_chunk(2 * cc + h, sw));
            }
        };
        auto piece = [&](int q) {                                   // q = 0..15 (KS = 2: 0..7 and 8..15): half a pair of keys
            const int r = 2 * (q >> 1);
            if ((q & 1) == 0) {
                pe[r] = sc[BLK][r] * c;
                pe[r + 1] = sc[BLK][r + 1] * c;
                pe[r] = fast_exp2(pe[r]);
            } else {
                pe[r + 1] = fast_exp2(pe[r + 1]);
#pragma unroll
                for (int L = 0; L < C::NLD; ++L)
                    if (q - (KS == 2 ? 8 * HALF : 0) == ((((2 * L + 1) * 16 / KS) / (2 * C::NLD)) | 1)) {     // request L rides on this piece
                        unsigned pin = __float_as_uint(pe[r + 1]);
                        if constexpr (HALF == 0) tile_load_pinned<C::KRB, NW, C::NLD>(gt, L, koff, lt + L * NW * 1024, pin);
                        else tile_load_pinned<C::VRB, NW, C::NLD>(gt, L, voff, lt + L * NW * 1024, pin);
                        pe[r + 1] = __uint_as_float(pin);
                    }
                const uint32_t pk = pack_bf16x2(pe[r], pe[r + 1]);
                pc[BLK][r >> 3][(r & 7) >> 1] = pk;
                sum = add_bf16x2(pk, sum);
            }
        };
#pragma unroll
        for (int j = 0; j < kSchedAhead; ++j) read(j);
#pragma unroll
        for (int j = 0; j < NM; ++j) {
            if (j + kSchedAhead < NM) read(j + kSchedAhead);
            if constexpr (HALF == 0) {
                const int hf = j / (2 * C::ODB), s2 = (j / C::ODB) & 1, db = j % C::ODB;
                o[db] = mma_frag<__bf16>(frag[j], pp[hf][s2], o[db]);
            } else {
                const int blk = KS == 1 ? j & 1 : 0, cc = KS == 1 ? j >> 1 : j;
                sn[blk] = mma_frag<__bf16>(frag[j], qf[cc], cc == 0 ? floatx16{0} : sn[blk]);
            }
#pragma unroll
            for (int q = 0; q < PPM; ++q) piece((KS == 2 ? 8 * HALF : 0) + j * PPM + q);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto step = [&](int t, floatx16 (&sc)[C::NBK], floatx16 (&sn)[C::NBK], Probs& pp, Probs& pc) {
        // requests of this step: K tile t+2 into the buffer tile t has left (first half), V tile t+1 into the
        // one tile t-1 leaves at the middle barrier (second half).  In the steady state they are issued one
        // at a time, each tied to one exponential (a burst of them stalls every wave of the workgroup at the
        // address unit); elsewhere in one go.  Past the last tile the last tile is fetched again, unread.
        const int kt = min(t + 2, ntiles - 1), vt = min(t + 1, ntiles - 1);
        const char* kgt = kg + (int64_t)kt * C::TILE_BYTES;
        const char* vgt = vg + (int64_t)vt * C::TILE_BYTES;
        const unsigned kl = klds + (t & 1) * C::TILE_BYTES, vl = vlds + ((t + 1) & 1) * C::TILE_BYTES;
        const bool has_pv = t >= 1 && t - 1 < my_tiles, has_s = t < my_tiles, has_next = t + 1 < my_tiles;
        const char* kb = Kb0 + ((t + 1) & 1) * C::TILE_BYTES + kw * 32 * C::KRB;
        const char* vb = Vb0 + ((t + 1) & 1) * C::TILE_BYTES + kw * 32 * C::VRB;      // V tile t-1
        float mc = 0.f, sum = 0.f;
        if (has_s && t * kBN + (KS == 1 ? kBN : 32 * kw + 32) - 1 > wave_first_row) {       // tile touches the diagonal (wave-uniform)
#pragma unroll
            for (int blk = 0; blk < C::NBK; ++blk)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (t * kBN + 32 * (KS == 1 ? blk : kw) + acc_row(r, h) > qrow) sc[blk][r] = -INFINITY;
        }
        // Probabilities of this tile, packed once into P^T operand fragments; the row sums are taken over the values as rounded
        // to bf16, so that numerator and denominator of the output use the same weights.
        auto exps = [&](int blk) {
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float p0 = fast_exp2(SAFE ? fmaf(sc[blk][r], c, -mc) : sc[blk][r] * c);
                const float p1 = fast_exp2(SAFE ? fmaf(sc[blk][r + 1], c, -mc) : sc[blk][r + 1] * c);
                const uint32_t pk = pack_bf16x2(p0, p1);
                pc[blk][r >> 3][(r & 7) >> 1] = pk;
                sum = add_bf16x2(pk, sum);
            }
        };
        const bool steady = has_pv && has_next && t < steady_end && !SAFE;
        // ---- first half: P.V of tile t-1 | exponentials of key block 0 of tile t | requests for K tile t+2
        if (steady) {
            steady_half(std::integral_constant<int, 0>{}, vb, sc, sn, pp, pc, sum, kgt, kl);
        } else {
            load_k(kt, t & 1);
            if (has_pv) {
                PV<T, D, NW, KS>::template run<0>(vb, vlane, pp, o);
                if constexpr (KS == 1) PV<T, D, NW, KS>::template run<1>(vb, vlane, pp, o);
            }
            if (has_s) {
                if constexpr (SAFE) {
                    // raw-logit maxima; the softmax scale (c > 0, log2 domain) is folded into the exponent.  The
                    // offset follows the maximum lazily: it moves only when a logit exceeds it by more than
                    // kLazyLog2 in the log2 domain, so probabilities stay below 2^kLazyLog2 and the accumulators
                    // (which hold every tile up to t-1 by now) are rescaled rarely.  The first tile always moves
                    // it (offset -inf; key 0 is visible to every row, so the maximum is finite).
                    const float lazy = kLazyLog2 / c;
                    float mx = -INFINITY;
#pragma unroll
                    for (int blk = 0; blk < C::NBK; ++blk)
#pragma unroll
                        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[blk][r]);
                    mx = xhalf_max(mx);
                    const bool grow = mx > m_run + lazy;
                    const float m_new = grow ? mx : m_run;
                    mc = KS == 1 || m_new > -INFINITY ? m_new * c : 0.f;          // KS = 2: a wave's keys may all lie in a row's future
                    if (__any(grow)) {
                        const float alpha = KS == 1 || m_run > -INFINITY ? fast_exp2(m_run * c - mc) : 0.f;       // 1 where the maximum stayed
                        l_run *= alpha;
#pragma unroll
                        for (int db = 0; db < C::ODB; ++db)
#pragma unroll
                            for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
                        m_run = m_new;
                    }
                }
                exps(0);
            }
        }
        wait_tiles(2);                                        // K tile t+1 has landed (this wave's part)
        __syncthreads();
        // ---- second half: S^T of tile t+1 | exponentials of key block 1 of tile t | requests for V tile t+1
        if (steady) {
            steady_half(std::integral_constant<int, 1>{}, kb, sc, sn, pp, pc, sum, vgt, vl);
        } else {
            load_v(vt, (t + 1) & 1);
            if (has_next) {
                qk_block<T, D, NW, KS>(kb, 0, i, h, sw, qf, sn);
                if constexpr (KS == 1) qk_block<T, D, NW, KS>(kb, 1, i, h, sw, qf, sn);
            }
            if constexpr (KS == 1)
                if (has_s) exps(1);
        }
        if (has_s) l_run += sum;
        wait_tiles(2);                                        // V tile t has landed (this wave's part)
        __syncthreads();
    };
    // steps 0 .. ntiles: the last one only finishes P.V of the last tile
    for (int t = 0; t <= ntiles; t += 2) {
        step(t, sa, sb, pb, pa);
        if (t + 1 <= ntiles) step(t + 1, sb, sa, pa, pb);
    }
    __builtin_amdgcn_s_waitcnt(0);
    };
    pass(std::false_type{});
    // Output rows.  Everything the stores need is derived again from the thread index here (the empty asm
    // keeps the compiler from carrying row numbers and pointers through the key loop, where registers are
    // scarce).
    int tid_out = threadIdx.x;
    asm volatile("" : "+v"(tid_out));
    const int i_out = tid_out & 31, h_out = (tid_out >> 5) & 1;
    // KS = 2: a query's sums lie in two waves.  A per-lane value of the partner wave (same queries, other keys), through LDS: the
    // tile buffers are free once every wave has waited for its last requests.
    float* const meet = reinterpret_cast<float*>(smem);
    auto partner = [&](float v) {
        const int lane_out = tid_out & 63, w_all = tid_out >> 6;
        __syncthreads();
        meet[w_all * 64 + lane_out] = v;
        __syncthreads();
        return meet[((w_all + NW / KS) % NW) * 64 + lane_out];
    };
    if constexpr (KS == 2) l_run += partner(l_run);
    {
        // the offset-free pass stands if every row sum of the workgroup is finite and far from both ends of the
        // fp32 range (no exponential overflowed, the dominant terms did not underflow); otherwise the whole
        // workgroup repeats its tiles with running maxima
        const float l_tot = xhalf_sum(l_run);
        if (__syncthreads_or(qrow < kk && !(l_tot >= kSumLow && l_tot <= kSumHigh))) {      // rows past k are never stored
            pass(std::true_type{});
            if constexpr (KS == 1) __syncthreads();              // the last requests of all waves have landed
            if constexpr (KS == 2) {                             // to the larger of the two offsets (key 0 is visible to every row: finite)
                const float m_all = fmaxf(m_run, partner(m_run));
                const float a = m_run > -INFINITY ? fast_exp2((m_run - m_all) * c) : 0.f;
                l_run *= a;
#pragma unroll
                for (int db = 0; db < C::ODB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[db][r] *= a;
                l_run += partner(l_run);
            }
        }
    }
    // KS = 2: either wave keeps half of the channel blocks, o[0 .. ODB / 2), and hands over the others
    constexpr int kOut = C::ODB / KS;
    if constexpr (KS == 2) {
        const int w_all = tid_out >> 6, lane_out = tid_out & 63;
        if (kw) {
#pragma unroll
            for (int db = 0; db < kOut; ++db) {
                const floatx16 x = o[db];
                o[db] = o[db + kOut];
                o[db + kOut] = x;
            }
        }
        __syncthreads();
#pragma unroll
        for (int db = 0; db < kOut; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) meet[((w_all * kOut + db) * 16 + r) * 64 + lane_out] = o[db + kOut][r];
        __syncthreads();
        const int w2 = (w_all + NW / KS) % NW;
#pragma unroll
        for (int db = 0; db < kOut; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db][r] += meet[((w2 * kOut + db) * 16 + r) * 64 + lane_out];
    }

    // Rows leave through LDS (a wave's own part of the V buffers), 16 bytes a lane and whole rows a store: from the accumulators a lane has 8 bytes of
    // a row at a time, 32 rows a store.  A workgroup ended 2.9 us after its last step (stores included), 2.1 so.
    // Streaming where queries are many: rows that stay in the caches are written back under the next kernel's reads.  us, ordinary -> so: 4 x 32 heads, n = 4000,
    // 30 % 113.2 -> 111.7, 2 x 40, n = 6000 127.0 -> 125.8, scores to attention of 4 x 32, n = 8192, an eighth kept 235.0 -> 230.6; small outputs (KS = 2) 21.4 -> 21.5.
    constexpr int kOutBytes = D * Elem<T>::kBytes / KS, kOutLanes = kOutBytes / 16, kOutRows = 64 / kOutLanes;
    char* const mine = Vb0 + (tid_out >> 6) * 32 * kOutBytes;
    auto out_chunk = [](int row, int c) { return row * kOutBytes + ((c ^ (row / (256 / kOutBytes) & (kOutLanes - 1))) << 4); };
    const float inv = 1.f / xhalf_sum(l_run);
#pragma unroll
    for (int db = 0; db < kOut; ++db)
#pragma unroll
        for (int a = 0; a < 4; ++a)
            store_out4<T>(reinterpret_cast<T*>(mine + out_chunk(i_out, 4 * db + a) + 8 * h_out), o[db][4 * a] * inv, o[db][4 * a + 1] * inv,
                          o[db][4 * a + 2] * inv, o[db][4 * a + 3] * inv);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the rows below are other lanes' stores
    const int w_out = KS == 1 ? tid_out >> 6 : (tid_out >> 6) % (NW / KS), lane_row = (tid_out & 63) / kOutLanes, c_out = tid_out % kOutLanes;
    const char* const held_out = smem + 4 * C::TILE_BYTES + (tid_out >> 6) * 256;
#pragma unroll
    for (int q = 0; q < 32 / kOutRows; ++q) {
        const int r = q * kOutRows + lane_row, qr = i0 + kRW * w_out + r;
        const uintx4 x = *reinterpret_cast<const uintx4*>(mine + out_chunk(r, c_out));
        const int orow = out_compact || !tidx ? qr : *reinterpret_cast<const int*>(held_out + 4 * r);
        uintx4* const dst = reinterpret_cast<uintx4*>(O + (int64_t)orow * D + (KS == 2 ? kw * (D / 2) : 0) + c_out * 8);
        if (qr < kk) {
            if constexpr (KS == 1) __builtin_nontemporal_store(x, dst);
            else *dst = x;
        }
    }
}

// ---------------------------------------------------------------- fp32
// Eight fp32 values as three bf16 planes, x = hi + mid + lo (8 significant bits and a sign each, rounded to nearest, so
// that a plane holds at most 2^-9 of the one before): exactly from 2^-109 on; below, the last plane ends at bf16's smallest number and
// the sum is off by up to 2^-134.  An infinity, a NaN or a value that rounds to one leaves a NaN in mid or lo.
struct Planes { uintx4 hi, mid, lo; };
// The smallest magnitude other than 0 of some fp32 values, as 2 |x| - 1 of the bits: 0 is the largest of all.
struct Least {
    uint32_t key = ~0u;
    __device__ __forceinline__ void add(uint32_t x) { key = min(key, 2 * x - 1); }
    __device__ __forceinline__ bool below(float x) const { return key < 2 * __float_as_uint(x) - 1; }        // x > 0
};
// x - the low (high) half of a packed pair, in one instruction
// (the factors through a register: as a constant 0xBF800000 is taken for the float -1)
__device__ __forceinline__ float less_half(float x, uint32_t pair, uint32_t factors) {
    asm("" : "+s"(factors));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, factors), x, false);
}
__device__ __forceinline__ float less_low(float x, uint32_t pair) { return less_half(x, pair, 0x0000BF80u); }
__device__ __forceinline__ float less_high(float x, uint32_t pair) { return less_half(x, pair, 0xBF800000u); }
__device__ __forceinline__ Planes split8(const uintx4& a, const uintx4& b) {
    Planes s;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x0 = __uint_as_float(e < 2 ? a[2 * e] : b[2 * e - 4]), x1 = __uint_as_float(e < 2 ? a[2 * e + 1] : b[2 * e - 3]);
        const uint32_t hi = pack_bf16x2(x0, x1);
        const float r0 = less_low(x0, hi), r1 = less_high(x1, hi);
        const uint32_t mid = pack_bf16x2(r0, r1);
        s.hi[e] = hi;
        s.mid[e] = mid;
        s.lo[e] = pack_bf16x2(less_low(r0, mid), less_high(r1, mid));
    }
    return s;
}
// acc + a b in six products, the small ones first; what is left out (mid lo, lo mid, lo lo) is below 2^-26 of |a| |b|.
__device__ __forceinline__ floatx16 mma_planes(const Planes& a, const Planes& b, floatx16 acc) {
    acc = mma_frag<__bf16>(a.lo, b.hi, acc);
    acc = mma_frag<__bf16>(a.hi, b.lo, acc);
    acc = mma_frag<__bf16>(a.mid, b.mid, acc);
    acc = mma_frag<__bf16>(a.mid, b.hi, acc);
    acc = mma_frag<__bf16>(a.hi, b.mid, acc);
    return mma_frag<__bf16>(a.hi, b.hi, acc);
}

// flash_queries for fp32.  A product of fp32 numbers on the matrix cores takes 16 times as long as one of bf16; here it is six of bf16.
// K and V rows go through registers into LDS, split there by the workgroup once for all its waves (7 vector instructions for two elements,
// a quarter of the time of the products of a 32-key tile); the queries' planes stay in registers, the weights are split where they
// are taken.  Against 64 bits the outputs are nearer than with fp32 products (48 sums in a logit of d = 128 and not 64; 2-norm at 9000 rows
// 9.4e-7, was 1.14e-6; at 300 6.2e-7, was 7.5e-7).  That an input of the planes is off by up to 2^-134 where it is small is nothing beside outputs
// of 2^-80 and more and queries between 2^-100 and 2^90; outside of that (and where a sum is no number) the workgroup repeats its tiles in fp32
// products.  Bound: large calls by the rate of bf16 products (28 heads on 4, 4485 of 20 000 kept: 610 us,
// 1.08 PFLOP/s of them), small ones by the chain of a workgroup's tiles: split, product, weights, product, between barriers.  Next rows are
// requested after a tile's first product, where no operand of it waits for registers.  us, fp32 products -> so, every token kept: 28 heads on 4,
// n = 3000 601 -> 350; 14 on 2, n = 3000 321 -> 207; d = 64, 32 on 8, n = 2000 161 -> 107; 4 heads, n = 576 26.8 -> 19.0; a third kept,
// 32 heads, n = 2933 147 -> 76; 4485 of 20 000 1262 -> 607.
template <int D, int KS>
__device__ __forceinline__ void flash_queries_f32(const float* __restrict__ Q, int64_t qs2, const float* __restrict__ Kp, const float* __restrict__ Vp,
                                                  const int32_t* __restrict__ tidx, float* __restrict__ O, int i0, int kk, float c, int out_compact)
{
    using C = SplitCfg<D, KS>;
    constexpr int NW = C::NW, BM = 32 * NW / KS, TK = C::TK, RB = C::RB;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qw = KS == 1 ? w : w % (NW / KS), kw = KS == 1 ? 0 : w / (NW / KS);        // wave w has the queries of wave qw, key block kw
    const int ntiles = (min(i0 + BM, kk) + TK - 1) / TK;
    // Derived again wherever it is used (the empty asm): carried through the key loop these would go to scratch, and so would what is
    // kept from one tile of queries for the next.
    struct Lane { int tid, lane, i, h, qrow, crow, ccol; };  // crow, ccol: its row and 8 elements of every pass over a tile of rows
    auto this_lane = [&]() {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        return Lane{tid, tid & 63, tid & 31, (tid >> 5) & 1, i0 + 32 * qw + (tid & 31), tid / C::LPR, tid % C::LPR};
    };
    const int first_row = i0 + 32 * qw, last_row = min(first_row + 31, kk - 1);          // of the wave
    floatx16 o[C::ODB];
    float m_run = 0.f, l_run = 0.f;

    auto load_rows = [&](const float* base, int t, const Lane& L, uintx4 (&raw)[C::NP][2]) {      // rows at and past k repeat row k - 1 and are masked
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const float* src = base + (int64_t)min(t * TK + p * C::RPP + L.crow, kk - 1) * D + L.ccol * 8;
            raw[p][0] = load16(src);
            raw[p][1] = load16(src + 4);
        }
    };
    auto store_planes = [&](char* dst, const Lane& L, const uintx4 (&raw)[C::NP][2], auto swizzle) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const int r = p * C::RPP + L.crow;
            const Planes x = split8(raw[p][0], raw[p][1]);
            char* const a = dst + r * RB + swz_chunk(L.ccol, swizzle(r));
            store16(a, x.hi);
            store16(a + C::PLANE, x.mid);
            store16(a + 2 * C::PLANE, x.lo);
        }
    };
    char* const kpl = smem;
    char* const vpl = smem + (C::kShared ? 0 : 3 * C::PLANE);
    auto mask = [&](int jb, const Lane& L, floatx16& s) {
        if (jb + 31 > first_row) {                           // touches the diagonal (wave-uniform)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (jb + acc_row(r, L.h) > L.qrow) s[r] = -INFINITY;
        }
    };
    auto pass_planes = [&]() {                               // returns whether its queries are in range
        const Lane L = this_lane();
        const int lane = L.lane, i = L.i, h = L.h, qrow = L.qrow;
        uintx4 kr[C::NP][2], vr[C::NP][2];
        load_rows(Kp, 0, L, kr);
        if constexpr (!C::kShared) load_rows(Vp, 0, L, vr);
        Planes qf[C::CH];
        char* const qlo = smem + 3 * C::PLANE + qw * (C::CH * 1024) + lane * 16;     // kShared: the last plane of Q stands in LDS (32 registers)
        bool in_range;
        {
            Least least;
            float most = 0.f;
            const int qc = min(qrow, kk - 1), pos = tidx ? tidx[qc] : qc;
            const float* qp = Q + (int64_t)pos * qs2 + 8 * h;
#pragma unroll
            for (int cc = 0; cc < C::CH; ++cc) {
                const uintx4 q0 = load16(qp + 16 * cc), q1 = load16(qp + 16 * cc + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    least.add(q0[e]);
                    least.add(q1[e]);
                    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(most) : "v"(q0[e]), "v"(q1[e]));
                }
                asm volatile("" : "+v"(least.key), "+v"(most));      // now, not with all rows held for it: 248 bytes of scratch in the form of two kinds
                qf[cc] = split8(q0, q1);
                if constexpr (C::kShared) store16(qlo + cc * 1024, qf[cc].lo);       // both waves of the queries store the same
            }
            in_range = !__any(least.below(kQueryLow) || most >= kQueryHigh);
        }
#pragma unroll
        for (int db = 0; db < C::ODB; ++db) o[db] = floatx16{0};
        // V^T operands through the transposing read, as for bf16
        int vlane[C::ODB];
        {
            const int grp = (lane >> 4) & 1, e = (lane >> 2) & 3, q = lane & 3, row = 4 * h + e;
#pragma unroll
            for (int db = 0; db < C::ODB; ++db)
                vlane[db] = (32 * kw + row) * RB + swz_chunk(4 * db + 2 * grp + (q >> 1), v_row_swizzle<RB>(row)) + (q & 1) * 8;
        }
        const int krow = (32 * kw + i) * RB, sw = k_row_swizzle<RB>(i);
#pragma unroll 1
        for (int t = 0; t < ntiles; ++t) {
            if (t) __syncthreads();                          // everyone is done with tile t - 1
            store_planes(kpl, L, kr, [](int r) { return k_row_swizzle<RB>(r); });
            if constexpr (C::kShared) {
                load_rows(Vp, t, L, vr);
            } else {
                store_planes(vpl, L, vr, [](int r) { return v_row_swizzle<RB>(r); });
            }
            __syncthreads();
            const int jb = t * TK + 32 * kw;
            const bool live = jb <= last_row;                // wave-uniform: not all of the keys in the future
            floatx16 s = {0};
            if (live) {
#pragma unroll
                for (int cc = 0; cc < C::CH; ++cc) {
                    const char* a = kpl + krow + swz_chunk(2 * cc + h, sw);
                    if constexpr (C::kShared) qf[cc].lo = load16(qlo + cc * 1024);
                    s = mma_planes(Planes{load16(a), load16(a + C::PLANE), load16(a + 2 * C::PLANE)}, qf[cc], s);
                }
            }
            if constexpr (C::kShared) {
                __syncthreads();
                store_planes(vpl, L, vr, [](int r) { return v_row_swizzle<RB>(r); });
                load_rows(Kp, min(t + 1, ntiles - 1), L, kr);
                __syncthreads();
            } else {
                load_rows(Kp, min(t + 1, ntiles - 1), L, kr);
                load_rows(Vp, min(t + 1, ntiles - 1), L, vr);
            }
            if (!live) continue;
            mask(jb, L, s);
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = fast_exp2(s[r] * c);
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) sum += s[r];
            l_run += sum;
            typedef short shortx4 __attribute__((ext_vector_type(4)));
            using lds_ptr = __attribute__((address_space(3))) shortx4*;
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                uintx4 pa, pb;
#pragma unroll
                for (int e = 0; e < 4; ++e) { pa[e] = __float_as_uint(s[8 * s2 + e]); pb[e] = __float_as_uint(s[8 * s2 + 4 + e]); }
                const Planes pp = split8(pa, pb);
#pragma unroll
                for (int db = 0; db < C::ODB; ++db) {
                    auto operand = [&](int plane) {
                        const char* a = vpl + plane * C::PLANE + vlane[db] + 16 * s2 * RB;
                        const uintx2 lo = __builtin_bit_cast(uintx2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)a));
                        const uintx2 hi = __builtin_bit_cast(uintx2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(a + 8 * RB)));
                        return uintx4{lo[0], lo[1], hi[0], hi[1]};
                    };
                    o[db] = mma_planes(Planes{operand(0), operand(1), operand(2)}, pp, o[db]);
                }
            }
        }
        return in_range;
    };
    // The same in fp32 products, for what the planes do not hold: infinities, and what is small enough to be cut short.  maxima: the
    // offset follows the running maximum, for row sums near the ends of the fp32 range; otherwise it stays 0.
    auto pass_fp32 = [&](bool maxima) {
        const float lazy = maxima ? kLazyLog2 / c : INFINITY;
        const Lane L = this_lane();
        const int i = L.i, h = L.h, qrow = L.qrow, crow = L.crow, ccol = L.ccol;
        constexpr int FRB = 4 * D;
        char* const kt = smem;
        char* const vt = smem + TK * FRB;
        uintx4 qf[D / 8];
        {
            const int qc = min(qrow, kk - 1), pos = tidx ? tidx[qc] : qc;
            const float* qp = Q + (int64_t)pos * qs2 + 4 * h;
#pragma unroll
            for (int cc = 0; cc < D / 8; ++cc) qf[cc] = load16(qp + 8 * cc);
        }
#pragma unroll
        for (int db = 0; db < C::ODB; ++db) o[db] = floatx16{0};
        m_run = maxima ? -INFINITY : 0.f;
        l_run = 0.f;
#pragma unroll 1
        for (int t = 0; t < ntiles; ++t) {
            __syncthreads();
#pragma unroll
            for (int p = 0; p < C::NP; ++p) {
                const int r = p * C::RPP + crow, sw = k_row_swizzle<FRB>(r);
                const int64_t src = (int64_t)min(t * TK + r, kk - 1) * D + ccol * 8;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    store16(kt + r * FRB + swz_chunk(2 * ccol + e, sw), load16(Kp + src + 4 * e));
                    store16(vt + r * FRB + (2 * ccol + e) * 16, load16(Vp + src + 4 * e));
                }
            }
            __syncthreads();
            const int jb = t * TK + 32 * kw;
            if (jb > last_row) continue;
            floatx16 s = {0};
#pragma unroll
            for (int cc = 0; cc < D / 8; ++cc)
                s = mma_frag<float>(load16(kt + (32 * kw + i) * FRB + swz_chunk(2 * cc + h, k_row_swizzle<FRB>(i))), qf[cc], s);
            mask(jb, L, s);
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
            mx = xhalf_max(mx);
            const float m_new = mx > m_run + lazy ? mx : m_run, mc = m_new > -INFINITY ? m_new * c : 0.f;
            const float alpha = m_run > -INFINITY ? fast_exp2(m_run * c - mc) : 0.f;     // 1 where the maximum stayed
            if (__any(m_new != m_run)) {
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < C::ODB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
                m_run = m_new;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s[r] = fast_exp2(fmaf(s[r], c, -mc));
                l_run += s[r];
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float* v = reinterpret_cast<const float*>(vt + (32 * kw + acc_row(r, h)) * FRB) + i;
#pragma unroll
                for (int db = 0; db < C::ODB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[32 * db], s[r], o[db], 0, 0, 0);
            }
        }
    };

    // over the waves of a query (its keys lie in KS of them), through LDS; the same in all of them
    float* const meet = reinterpret_cast<float*>(smem);
    auto over_waves = [&](float v, auto f) {
        if constexpr (KS == 1) return v;
        const Lane L = this_lane();
        __syncthreads();
        meet[L.tid] = v;
        __syncthreads();
        v = meet[qw * 64 + L.lane];
#pragma unroll
        for (int x = 1; x < KS; ++x) v = f(v, meet[(qw + x * (NW / KS)) * 64 + L.lane]);
        return v;
    };
    auto plus = [](float x, float y) { return x + y; };
    const bool in_range = pass_planes();
    const Lane out = this_lane();
    const int lane = out.lane, h = out.h, qrow = out.qrow;
    l_run = over_waves(l_run, plus);
    float probe = 0.f;                                       // NaN if any of the sums is no finite number
    Least least;
#pragma unroll
    for (int db = 0; db < C::ODB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            probe = fmaf(o[db][r], 0.f, probe);
            least.add(__float_as_uint(o[db][r]));
        }
    const float l_once = xhalf_sum(l_run);
    const bool sums = l_once >= kSumLow && l_once <= kSumHigh && probe == 0.f;
    // outputs may be small because of V or of their weights, and one wave has a part of them
    const bool stands = sums && in_range && !least.below(kOutLow * fmaxf(l_once, 1.f));
    if (__syncthreads_or(qrow < kk && !stands)) {
        pass_fp32(__syncthreads_or(qrow < kk && !sums));
        if constexpr (KS > 1) {                              // to the largest of the offsets (key 0 is visible to every row: finite)
            const float m_all = over_waves(m_run, [](float x, float y) { return fmaxf(x, y); });
            const float a = m_run > -INFINITY ? fast_exp2((m_run - m_all) * c) : 0.f;
            l_run *= a;
#pragma unroll
            for (int db = 0; db < C::ODB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[db][r] *= a;
            l_run = over_waves(l_run, plus);
        }
    }
    if constexpr (KS > 1) {                                  // a wave stores the channels of 4 / KS of a block's four register groups
        __syncthreads();
#pragma unroll
        for (int db = 0; db < C::ODB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) meet[((w * C::ODB + db) * 16 + r) * 64 + lane] = o[db][r];
        __syncthreads();
    }
    const float inv = 1.f / xhalf_sum(l_run);
    if (qrow < kk) {
        const int orow = (out_compact || !tidx) ? qrow : tidx[qrow];
        float* op = O + (int64_t)orow * D + 4 * h;
#pragma unroll
        for (int db = 0; db < C::ODB; ++db)
#pragma unroll
            for (int a = 0; a < 4 / KS; ++a) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (KS == 1) {
                        v[e] = o[db][4 * a + e];
                    } else {
                        const float* x = meet + ((qw * C::ODB + db) * 16 + 4 * (kw * (4 / KS) + a) + e) * 64 + lane;
                        v[e] = x[0];
#pragma unroll
                        for (int y = 1; y < KS; ++y) v[e] += x[y * (NW / KS) * C::ODB * 1024];
                    }
                }
                store_out4<float>(op + 32 * db + 8 * (kw * (4 / KS) + a), v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv);
            }
    }
}

// ------------------------------------------------------------------ host
// Whether a head's queries are taken 64 at a time with the keys split over two waves, where both are possible (KS = 0): k kept
// tokens, BH heads alike, so many live tiles of 128.  bf16, d = 128, rows in place, us, 128 -> 64: k >= 1000: 448 live tiles (32 heads,
// k = 1759) 44 -> 42, 532 (28 on 4, k = 2346) 57.1 -> 57.4, 576 (2 x 32 on 8, k = 1100) 35 -> 43, 688 (8, k = 11000) 258 -> 268; shorter:
// 256 (4 x 32, k = 230) 14.7 -> 14.4, 252 (3 x 28 on 4, k = 300) 14.1 -> 12.9, 320 (2 x 32, k = 599) 22.1 -> 22.5, 384 (4 x 32, k = 300) 15.7 -> 18.6.
// fp32 (planes), every token kept: d = 128: 336 (2 x 28 on 4, k = 700) 71.9 -> 54.5, 480 (40, k = 1500) 159 -> 156, 512 (4 x 32 on 8, k = 400)
// 53 -> 52, 672 (28 on 4, k = 3000) 352 -> 369; d = 64: 512 (32 on 8, k = 2000) 116 -> 105, 896 (28 on 4, k = 4000) 317 -> 317, 728 (k = 3265 of 12 000) 223 -> 205; d = 128: 608 (32 on 8, k = 2400) 267 -> 267.
template <typename T, int D>
__device__ __forceinline__ bool splits_keys(int k, int BH) {
    const int line = Elem<T>::kBytes == 4 ? kPlanesLine<D> : k >= 1000 ? 512 : 288;
    return ((k + 127) >> 7) * BH <= line;
}

// Clears the rows of one head at the positions of [p0, p1), up to kFillSpan of them, that are not among its fk kept ones (ft,
// ascending).
template <typename T, int D, int NT>
__device__ __forceinline__ void clear_dropped(T* __restrict__ O, const int32_t* __restrict__ ft, int fk, int p0, int p1, int* kept) {
    const int tid = threadIdx.x, lane = tid & 63;
    for (int e = tid; e < kFillSpan; e += NT) kept[e] = 0;
    int lo = 0, len = fk;                                    // the first kept row at or after p0 is in [lo, lo + len]: 64 probes a round
    while (len > 0) {
        const int step = (len + 63) >> 6, blocks = (len + step - 1) / step;
        const bool below = lane < blocks && ft[lo + min((lane + 1) * step, len) - 1] < p0;
        const int cnt = __popcll(__ballot(below));           // blocks that end before p0
        lo += min(cnt * step, len);
        len = cnt == blocks ? 0 : min(step, len - cnt * step) - 1;
    }
    __syncthreads();
    for (int e = lo + tid; e < min(fk, lo + kFillSpan); e += NT) {
        const int pos = ft[e];
        if (pos < p1) kept[pos - p0] = 1;
    }
    __syncthreads();
    constexpr int CPR = D * Elem<T>::kBytes / 16;
    const uintx4 z = {0, 0, 0, 0};
    char* base = reinterpret_cast<char*>(O + (int64_t)p0 * D);
    for (int q = tid; q < (p1 - p0) * CPR; q += NT)
        // whole rows, written once and not read again by this path: streaming stores, so that they do not stay
        // behind as dirty lines in the last-level cache, to be written back under the next kernel's reads
        if (!kept[q / CPR]) __builtin_nontemporal_store(z, reinterpret_cast<uintx4*>(base + (int64_t)q * 16));
}

// kp, vp: of batch element, KV head.  slots: rows of attention workgroups in the grid, BH each; fill: workgroups after them that clear
// rows; scan: whether the kept counts are read for the longest head; ug: KV heads of a scheduling group, one more in the first `extra` ones.
template <typename T> struct FlashArgs {
    const T* Q; int64_t qs0, qs1, qs2;
    const T* Kp; int64_t kp0, kp1;
    const T* Vp; int64_t vp0, vp1;
    const int32_t* idx; const int32_t* kcnt;
    T* O;
    int n, npad, slots, fill, scan, ug, extra, G, BH, Hq, Hkv;
    float c;
    int out_compact, t_per_batch, k_in_place, v_in_place;
    uint32_t inv_larger, inv_smaller, inv_g, inv_hkv;        // of (ug + 1) G, ug G, G, Hkv
};

template <typename T, int D, int NW, int KS>
__global__ __launch_bounds__(64 * NW, (AttnCfg<T, D, NW, KS == 0 ? 2 : KS>::MIN_WGS)) void flash_kept_kernel(FlashArgs<T> args)
{
    using C = AttnCfg<T, D, NW, KS == 0 ? 2 : KS>;
    constexpr int kBM = C::BM;                               // queries per tile
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int block = blockIdx.x;
    // All arguments at once: the compiler would load each where it is first used, 0.2 us apart.
    auto fetch = [](const auto& a) {
        const FlashArgs<T> x = {a.Q, a.qs0, a.qs1, a.qs2, a.Kp, a.kp0, a.kp1, a.Vp, a.vp0, a.vp1, a.idx, a.kcnt, a.O, a.n, a.npad, a.slots, a.fill, a.scan,
                                a.ug, a.extra, a.G, a.BH, a.Hq, a.Hkv, a.c, a.out_compact, a.t_per_batch, a.k_in_place, a.v_in_place,
                                a.inv_larger, a.inv_smaller, a.inv_g, a.inv_hkv};
        asm volatile("" :: "s"(x.Q), "s"(x.qs0), "s"(x.qs1), "s"(x.qs2), "s"(x.Kp), "s"(x.kp0), "s"(x.kp1), "s"(x.Vp), "s"(x.vp0), "s"(x.vp1), "s"(x.idx),
                     "s"(x.kcnt), "s"(x.O), "s"(x.n), "s"(x.npad), "s"(x.fill), "s"(x.ug), "s"(x.extra), "s"(x.G), "s"(x.BH), "s"(x.Hq), "s"(x.Hkv), "s"(x.c),
                     "s"(x.out_compact), "s"(x.t_per_batch), "s"(x.k_in_place), "s"(x.v_in_place), "s"(x.inv_larger), "s"(x.inv_smaller), "s"(x.inv_g), "s"(x.inv_hkv));
        return x;
    };
    const FlashArgs<T> a0 = fetch(args);
    // The query tiles of the longest head.  k is on the device and the grid is for k = n, so that most workgroups of a sparse call have
    // nothing to do; dispatched among the others, in their order and 1.5 us each in a slot of the chip, they kept a fifth of the slots
    // empty (4 x 32 heads, n = 8192, a quarter kept).  With this every workgroup knows them, and they are the last of the grid.
    int lmax = (a0.n + kBM - 1) / kBM, lane_k = 0, lane_k2 = 0, sets = 0;
    if (a0.scan) {
        sets = a0.t_per_batch ? divided(divided(a0.BH, a0.G, a0.inv_g), a0.Hkv, a0.inv_hkv) : divided(a0.BH, a0.G, a0.inv_g);
        const int lane = threadIdx.x & 63;
        lane_k = a0.kcnt[min(lane, sets - 1)];
        lane_k2 = a0.kcnt[min(lane + 64, sets - 1)];
        int most = max(max(lane_k, lane_k2), 0);
        for (int x = lane + 128; x < sets; x += 64) most = max(most, a0.kcnt[x]);
        lmax = min(lmax, (wave_reduce(most, 0, [](int x, int y) { return max(x, y); }) + kBM - 1) / kBM);
    }
    const int rows = min(lmax, a0.slots);
    // Workgroup -> (group of KV heads, row, KV head in group, head of the KV head), in that order of significance; heavy (late) query
    // tiles first inside a group (scheduling_groups), so that the light tail of one overlaps the heavy start of the next.
    struct Place { int row, b, g, head, set; };
    auto place = [&](const FlashArgs<T>& a) {
        const int wide = a.extra * (a.ug + 1);                   // KV heads of the larger groups
        const bool large = block < wide * a.G * rows;
        const int from = large ? 0 : wide, size = a.ug + large, heads = size * a.G, past = block - from * a.G * rows;
        const uint32_t inv = large ? a.inv_larger : a.inv_smaller;
        const int line = divided(past, heads, inv);        // row, counted from the first of these groups
        const int group = (unsigned)line / (unsigned)rows, row = line - group * rows;
        int rr = past - line * heads;
        if (rows >= kTurnFrom && a.kcnt && a.G == 1 && heads % 8 == 0) {
            rr += row / kTurnRows;
            rr -= divided(rr, heads, inv) * heads;
        }
        const int j = divided(rr, a.G, a.inv_g), u = from + group * size + j, b = divided(u, a.Hkv, a.inv_hkv), g = u - b * a.Hkv;
        return Place{row, b, g, g * a.G + rr - j * a.G, a.t_per_batch ? b : u};
    };
    auto kept = [&](const FlashArgs<T>& a, int set) { return a.kcnt ? a.kcnt[set] : a.n; };
    auto tile = [&](const FlashArgs<T>& a, const Place& at, int kk, int round) {
        kk = max(0, min(kk, a.n));
        const int x = round * rows + (round & 1 ? rows - 1 - at.row : at.row);
        // KS = 0: heads that take 128 queries at a time have half as many tiles, and start with the last one
        const bool wide = KS == 1 || (KS == 0 && !splits_keys<T, D>(kk, a.BH));
        const int i0 = KS == 0 && wide ? ((kk + 2 * kBM - 1) / (2 * kBM) - 1 - x) * 2 * kBM : (lmax - 1 - x) * kBM;
        if (i0 < 0 || i0 >= kk) return;
        const int32_t* tidx = a.idx ? a.idx + (int64_t)at.set * a.n : nullptr;       // this unit's T
        const T* q = a.Q + at.b * a.qs0 + at.head * a.qs1;
        const T* kp = a.Kp + at.b * a.kp0 + at.g * a.kp1;
        const T* vp = a.Vp + at.b * a.vp0 + at.g * a.vp1;
        T* Oh = a.O + (int64_t)(at.b * a.Hq + at.head) * a.n * D;
        auto queries = [&](auto ks) {
            constexpr int S = decltype(ks)::value;
            if constexpr (Elem<T>::kBytes == 4) flash_queries_f32<D, S>(q, a.qs2, kp, vp, tidx, Oh, i0, kk, a.c, a.out_compact);
            else flash_queries<T, D, NW, S>(q, a.qs2, kp, vp, tidx, Oh, i0, kk, a.npad, a.c, a.out_compact, a.k_in_place, a.v_in_place);
        };
        if constexpr (KS != 0) queries(std::integral_constant<int, KS>{});
        else if (wide) queries(std::integral_constant<int, 1>{});
        else queries(std::integral_constant<int, 2>{});
    };
    if (block >= a0.BH * rows) {
        // Outputs of dropped tokens are zero rows.  The workgroups after the last attention workgroup
        // each clear the dropped rows of one head inside one span of kFillSpan positions; they are
        // dispatched last, into the slots that the light end of the attention work leaves idle.
        const int f = block - a0.BH * rows, s = f / a0.BH, bh = f - s * a0.BH;
        if (f >= a0.fill) return;
        const int b = bh / a0.Hq, set = a0.t_per_batch ? b : b * a0.Hkv + (bh - b * a0.Hq) / a0.G;
        clear_dropped<T, D, C::NT>(a0.O + (int64_t)bh * a0.n * D, a0.idx + (int64_t)set * a0.n, max(0, min(kept(a0, set), a0.n)),
                                   s * kFillSpan, min(a0.n, (s + 1) * kFillSpan), reinterpret_cast<int*>(smem));
        return;
    }
    const Place at0 = place(a0);
    const int k0 = at0.set < min(sets, 128) ? __builtin_amdgcn_readlane(at0.set < 64 ? lane_k : lane_k2, at0.set & 63) : kept(a0, at0.set);
    if constexpr (KS != 1) {
        tile(a0, at0, k0, 0);
    } else {
        // A workgroup of a grid that has fewer rows than tiles takes a second one, from the light end.  What a round needs is
        // read from the arguments and derived again (the empty asm): carried through the key loop it would take more scalar
        // registers than there are.
        using ArgPtr = const __attribute__((address_space(4))) FlashArgs<T>*;
        ArgPtr again = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
        FlashArgs<T> a = a0;
        Place at = at0;
        int k = k0;
#pragma unroll 1
        for (int round = 0;;) {
            tile(a, at, k, round);
            if (++round * rows >= lmax) break;
            __syncthreads();
            asm volatile("" : "+s"(block), "+s"(again));
            a = fetch(*again);
            at = place(a);
            k = kept(a, at.set);
        }
    }
}

size_t prefill_workspace_bytes(const zipvl_dims& d) {
    const int e = d.dtype == ZIPVL_BF16 ? 2 : 4;
    const size_t npad = ((size_t)d.n + kBN - 1) / kBN * kBN;
    return 2 * (size_t)d.B * d.Hkv * npad * d.d * e;
}

// Scheduling groups of KV heads: as near as their number comes to 20 heads of queries each, or to 800 tiles of 128
// for shorter sequences; 1280 of a set, of which some are live (800: 2 x 32 on 8, n = 3000, a third kept 41 us, so 36; 32 heads, n = 6000 55, 48;
// 4 x 8, n = 5000 59, 52; 2 x 32 on 8, n = 3000, 60 % kept 73, 74.5; 1600: 4 x 32, n = 8192 2 % slower, the others as with 1280).  Larger groups take K / V beyond what the caches hold at a time, smaller ones leave too few light tiles under
// the heavy ones of the next, and an uneven last one runs on alone.  us, groups by bytes of K / V (32 and 8 heads, 42 and 22, ...) -> so:
// every token kept, 40 heads, n = 4096 195 -> 172; a third kept, 4 x 32 on 8, n = 5000 120 -> 109; d = 64, 2 x 32, n = 6000 59 -> 54;
// 15 %, 40 heads, n = 16000 97 -> 88; 20 %, 4 x 4, n = 20000 110 -> 105.  fp32, six products for one, hides the loads: one
// group (40 heads, n = 4000 829 us, in two 898; a third of 4 x 32 heads, d = 64, n = 3000 113, in groups 125).
// One group of up to 40 heads (32 of a set) where the tiles are few.  us, in two -> one: every token kept, d = 64, 32 heads, n = 5000 132 -> 126; a quarter
// kept, 32 on 8, n = 8000 57.3 -> 52.1; past the lines: half kept, 32 on 8, n = 11 098 151 -> 161, 40, n = 6326 131 -> 138, 3 x 32 on 8, n = 2538 70 -> 75,
// every token kept, 2 x 32 on 8, n = 2239 96 -> 101.
// Every token kept and own K / V for every head: groups of a multiple of 8 heads within a factor of 2 of that: workgroups go to the 8 XCDs in turn,
// and a head's tiles then meet on one L2.  The nearest count (20, 20 and 20 heads) -> so: 40 heads, n = 15000 2056 -> 2020 us, 2 x 40, n = 9000
// 1549 -> 1499, 4 x 40, n = 4200 717 -> 699; of a set, whose heads keep different numbers: 2 x 40, half kept, n = 10 180 343 -> 360.
// Otherwise groups of one size where their number divides the KV heads within sqrt(2) of the wanted one, which some number always is; if not, sizes
// differ by one (one group -> two: every token kept, 37 heads, n = 9000 855 -> 767, 31, n = 14000 1672 -> 1476, 29, n = 9000 643 -> 594).
constexpr int64_t kOneGroup = 3600, kOneGroupOfSet = 2048;

template <typename T>
static int scheduling_groups(int units, int G, int tiles, bool set) {
    const int64_t heads = (int64_t)units * G;
    if (Elem<T>::kBytes == 4 || (heads <= (set ? 32 : 40) && heads * tiles <= (set ? kOneGroupOfSet : kOneGroup))) return 1;
    const double want = units * G / (double)std::max(20, (set ? 1280 : 800) / tiles);
    auto off = [&](int groups) { return std::max(groups / want, want / groups); };
    int whole = 0, equal = 1, any = 1;
    for (int groups = 1; groups <= units; ++groups) {
        if (off(groups) < off(any)) any = groups;
        if (units % groups) continue;
        if (off(groups) < off(equal)) equal = groups;
        if (!set && G == 1 && units / groups % 8 == 0 && off(groups) <= 2 && (!whole || off(groups) < off(whole))) whole = groups;
    }
    if (whole) return whole;
    return off(equal) <= 1.4143 ? equal : any;
}

template <typename T, int D, int NW, int KS>
static int launch_flash(const void* Q, const void* K, const zipvl_dims& d, const int32_t* idx, const int32_t* k,
                        float scale, int out_compact, int t_per_batch, int skip_k, int skip_v, const void* V, const T* Kp, const T* Vp, int npad, void* O, hipStream_t st)
{
    using C = AttnCfg<T, D, NW, KS == 0 ? 2 : KS>;
    static std::atomic<bool> attr_done{false};       // raising the dynamic-LDS cap is idempotent
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&flash_kept_kernel<T, D, NW, KS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES) != hipSuccess)
            return set_error(ZIPVL_EHIP, "sparse_prefill: cannot reserve %d bytes of LDS", C::LDS_BYTES);
        attr_done = true;
    }
    {
        KernelTimer tm(ZIPVL_K_FLASH_KEPT, st);
        const int BH = d.B * d.Hq;
        const int ntq = (d.n + C::BM - 1) / C::BM, G = d.Hq / d.Hkv;
        const int slots = KS == 1 && idx ? std::max((ntq + 1) / 2, std::min(ntq, (kSecondRound + BH - 1) / BH)) : ntq;
        const int64_t blocks = (int64_t)slots * BH;
        // full-size output of a sparse call: one more workgroup per (head, span of positions) clears dropped rows
        const int64_t fill = (!out_compact && idx) ? (int64_t)BH * ((d.n + kFillSpan - 1) / kFillSpan) : 0;
        const int units = d.B * d.Hkv, groups = scheduling_groups<T>(units, G, (d.n + 127) / 128, idx != nullptr);
        const int scan = k && blocks > kScanBlocks && (t_per_batch ? d.B : d.B * d.Hkv) <= kScanSets;
        if (blocks + fill > 0x7fffffffLL) return set_error(ZIPVL_ESHAPE, "sparse_prefill: %lld workgroups exceed the grid limit", (long long)(blocks + fill));
        hipLaunchKernelGGL((flash_kept_kernel<T, D, NW, KS>), dim3((unsigned)(blocks + fill)), dim3(C::NT),
            C::LDS_BYTES, st, FlashArgs<T>{(const T*)Q, d.q_strides[0], d.q_strides[1], d.q_strides[2],
                skip_k ? (const T*)K : Kp, skip_k ? d.k_strides[0] : (int64_t)d.Hkv * npad * D, skip_k ? d.k_strides[1] : (int64_t)npad * D,
                skip_v ? (const T*)V : Vp, skip_v ? d.v_strides[0] : (int64_t)d.Hkv * npad * D, skip_v ? d.v_strides[1] : (int64_t)npad * D,
                idx, k, (T*)O, d.n, npad, slots, (int)fill, scan, units / groups, units % groups, G, BH, d.Hq, d.Hkv, scale * kLog2e, out_compact, t_per_batch, skip_k, skip_v,
                inverse((units / groups + 1) * G), inverse(units / groups * G), inverse(G), inverse(d.Hkv)});
    }
    return check_launch("flash_kept");
}

template <typename T, int D>
static int launch_prefill_t(const void* Q, const void* K, const void* V, const zipvl_dims& d,
                            const int32_t* idx, const int32_t* k, float scale, int flags,
                            void* O, void* ws, hipStream_t st)
{
    const int npad = (d.n + kBN - 1) / kBN * kBN;
    const int units = d.B * d.Hkv;
    T* Kp = (T*)ws;
    T* Vp = Kp + (size_t)units * npad * D;
    const int out_compact = (flags & ZIPVL_OUT_COMPACT) ? 1 : 0;
    const int rows_are_kept = ((flags & ZIPVL_KV_ALREADY_COMPACT) || !idx) ? 1 : 0;      // row i of K, V is kept token i
    const int t_per_batch = (flags & ZIPVL_T_PER_BATCH) ? 1 : 0;

    // An evicted cache (or, with every token kept, K and V themselves) with contiguous rows is read in place, whatever its length:
    // no row at or beyond k is read.  All of 28 heads on 4, n = 18432: the copy took 15 us of 2200.  32 heads,
    // n = 2933: packing all of it took 8.5 us of 64; fp32, 4 heads, n = 576: the launch that transposed V 3.8 of 45.
    const int skip_k = (rows_are_kept && d.k_strides[2] == D) ? 1 : 0;
    const int skip_v = (rows_are_kept && d.v_strides[2] == D) ? 1 : 0;
    if (!(skip_k && skip_v)) {
        KernelTimer tm(ZIPVL_K_PACK_KV, st);
        hipLaunchKernelGGL((pack_kv_kernel<T, D>), dim3(npad / kBN, units), dim3(256), 0, st,
            (const T*)K, (const T*)V, d.k_strides[0], d.k_strides[1], d.k_strides[2],
            d.v_strides[0], d.v_strides[1], d.v_strides[2], idx, k, Kp, Vp, d.n, npad, d.Hkv, rows_are_kept, skip_k, skip_v, t_per_batch);
        int rc = check_launch("pack_kv");
        if (rc) return rc;
    }

    // A call with few query tiles lasts as long as the one with the most keys: about 1 us per 64 keys (a SIMD's products and
    // exponentials one after the other) while most CUs are idle.  Tiles of 64 queries whose waves split the keys put the same
    // work on twice the workgroups: half the work per step on every SIMD, and long tiles share a CU with short ones.  With
    // enough tiles to fill the chip it only doubles the K / V traffic per query.  The line (tiles of 128 queries), bf16, d = 128,
    // us, 128 -> 64: every token kept, 32 heads, n = 1500 (384 tiles) 42 -> 37, 28 heads on 4, n = 2933 (644) 74 -> 82; below
    // n = 1000 the chains are short: 3 x 28 heads on 4, n = 500 (336) 20.2 -> 21.6, 2 x 32 heads, n = 500 (256) 24 -> 22.
    // Of a set only some tiles are live, and k is on the device.  Up to twice the line, bf16 at d = 128 decides there, head by
    // head (splits_keys; the kernel of both needs no more registers than that of 128): 32 heads, n = 2933, a third kept 29.5 us (128)
    // and 22.0 (64), 22.0 so, all of a set kept 80, 91 and 79; 4 x 32 heads, n = 500, 60 % kept 15.4, 18.5 and 15.3, all 21.4, 27.1 and
    // 22.4.  At d = 64 it would take the kernel of 64 a third of its waves: with up to 60 % kept 64 is
    // faster or equal (2 x 32 heads, n = 960, 512 tiles 12.5 -> 11.4), with all of a set kept up to 17 % slower.
    const int64_t tiles = (int64_t)((d.n + 127) / 128) * d.B * d.Hq, line = d.n >= 1000 ? 384 : 256;
    auto launch = [&](auto waves, auto ks) {
        return launch_flash<T, D, decltype(waves)::value, decltype(ks)::value>(Q, K, d, idx, k, scale, out_compact, t_per_batch, skip_k, skip_v, V, Kp, Vp, npad, O, st);
    };
    constexpr std::integral_constant<int, 0> chosen{};
    constexpr std::integral_constant<int, 1> whole{};
    constexpr std::integral_constant<int, 2> half{};
    constexpr std::integral_constant<int, 4> four{};
    constexpr std::integral_constant<int, 8> eight{};
    // fp32.  Fewer tiles than CUs: eight waves on 64 queries, two for every SIMD of a CU that has only this workgroup, take four key blocks of a
    // tile.  us, 64 queries by four waves -> by eight: 8 on 2, n = 700, d = 128 (48 tiles) 42 -> 39, 8 heads, n = 2933, d = 64 (184) 93 -> 70, 4 heads,
    // n = 8000 (252) 485 -> 380, 32 on 8, n = 1100 (288) 80 -> 86, 2 x 32 on 8, n = 500, d = 64 (256) 21 -> 24.  Of a set half is taken to be
    // live; above, the form is chosen by what is (splits_keys), until a quarter kept is past that line too.
    if constexpr (Elem<T>::kBytes == 4) {
        const int64_t few = (d.n >= 1000 ? 256 : 128) * (idx ? 2 : 1);
        if (tiles <= few) return launch(eight, four);
        if (idx && tiles <= 4 * kPlanesLine<D>) return launch(four, chosen);
        return tiles <= kPlanesLine<D> ? launch(four, half) : launch(four, whole);
    } else {
        if constexpr (D == 128)
            if (tiles > line && tiles <= 2 * line && idx) return launch(four, chosen);
        return tiles <= line * (idx ? 2 : 1) ? launch(four, half) : launch(four, whole);
    }
}

int launch_sparse_prefill(const void* Q, const void* K, const void* V, const zipvl_dims& d,
                          const int32_t* idx, const int32_t* k, float scale, int flags,
                          void* O, void* ws, hipStream_t st)
{
    if (d.dtype == ZIPVL_BF16) {
        if (d.d == 128) return launch_prefill_t<__bf16, 128>(Q, K, V, d, idx, k, scale, flags, O, ws, st);
        return launch_prefill_t<__bf16, 64>(Q, K, V, d, idx, k, scale, flags, O, ws, st);
    }
    if (d.d == 128) return launch_prefill_t<float, 128>(Q, K, V, d, idx, k, scale, flags, O, ws, st);
    return launch_prefill_t<float, 64>(Q, K, V, d, idx, k, scale, flags, O, ws, st);
}

}  // namespace zipvl
