// gemm_small.hpp -- the contraction with small output tiles, for shapes that the 256 x 256 tiles leave mostly idle.
//
// A 256 x 256 tile is the right size when there are hundreds of them.  A decoding batch has one row of tiles (24 of them
// for a 6144-wide projection), every workgroup then multiplies 224 or more rows of padding, and the K-step or two that it
// has in flight are all that its CU asks of memory.  Here a tile is 32 to 128 rows by 64 to 256 columns, so that there is a
// workgroup for every CU; if there still is none, the contraction of a tile is cut into `nsplit` ranges.  The plans, and
// what each tile measured, are in splitk_plan.hpp.
//
// The workgroups of a divided tile leave their fp32 partials in the workspace, row-major [range][M][N], and end.  The epilogue program
// then runs in a second kernel (epi_rows.hpp) that adds the ranges up in order: parallel over rows and columns instead of
// one workgroup per tile, and ordered by the stream instead of by tickets, so that the partials travel as ordinary cached
// stores and loads.
//
// Mainloop: a ring of S stages in LDS filled by direct-to-LDS loads; a stage is 128 bytes of the contraction per row of a
// K-contiguous operand, or the same number of k-rows of an MN-contiguous one.  One barrier per stage, and the fragments of
// the next MFMA step are read while the current ones are multiplied.  The MFMA instructions and their order along K are those
// of the 256 x 256 tiles, so that an undivided launch gives the same sums, bit for bit, on any tile (8-bit: 16x16x128, which rounds
// otherwise, is within some 10 % of 32x32x64 either way).  Up to 64 rows the kernel is bound by HBM (28672 x 8192 bf16 weights
// against one row: 70.6 us, 6.7 TB/s; a large copy 5.2).  At 128 rows no unit is full: of the cycles in which a CU has a
// workgroup the matrix pipe is busy in 58 % (509 x 16384 x 2048 on 128 x 256) and LDS in 30 %, and 4 % of the wave-cycles wait on LDS.  What
// is left is that the waves of a workgroup read, wait at the stage's barrier and multiply in step.  Two groups of waves a phase apart, as on
// the large tiles, were slower (1426 -> 1666 cycles a stage: the eight fragment reads of a phase take longer than its 256 cycles of MFMA).
#pragma once
#include "gemm_kernel.hpp"
#include "splitk_plan.hpp"

namespace coda {

struct SmallParams {
    const unsigned char *A, *B;
    int64_t lda, ldb;        // row pitches in bytes
    int M, N, K;
    int tiles_m, tiles_n, nsplit;
    int chain;               // longest chain of fp32 additions, in stages
    int rot_cols;            // B K-contiguous: a tile starts at stage n0 / rot_cols of its range and wraps around; undivided also 0:
                             // at stage 0, ROT_XCD: where its 256 x 256 tile starts (see gemm_item_dl)
    float *part;             // [nsplit][M][N]
};

template <int BM_, int BN_, int WGM_, int WGN_, int S_, bool F8_>
struct SmallCfg {
    static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, BKB = 128, S = S_, NW = WGM * WGN, NT = NW * 64;
    static constexpr bool F8 = F8_, ONCE = false;
    static constexpr int ESZ = F8 ? 1 : 2, BK = BKB / ESZ;        // contraction elements per stage
    static constexpr int WTM = BM / WGM, WTN = BN / WGN;
    static constexpr int FR = F8 ? 32 : 16;                       // rows (columns) of an MFMA block
    static constexpr int A_BYTES = BM * BKB, B_BYTES = BN * BKB, STAGE = A_BYTES + B_BYTES, LDS = S * STAGE;
    static constexpr int LA = A_BYTES / 1024 / NW, LB = B_BYTES / 1024 / NW;   // wave-loads of 1 KB per wave and stage
    static_assert(A_BYTES % (1024 * NW) == 0 && B_BYTES % (1024 * NW) == 0, "every wave issues the same number of loads");
    static_assert(WTM % FR == 0 && WTN % FR == 0 && S >= 2 && LDS <= 160 * 1024, "LDS");
};

// The same tile with B fetched past the caches, where reads_once() says so
template <class C>
struct Once : C {
    static constexpr bool ONCE = true;
};
template <class C, bool BKC>
inline bool reads_once(const SmallParams &p, int ranges)
{
    return reads_once(p.M, p.N, p.K, C::F8, BKC, C::BM, ranges, p.ldb, (uint64_t)(uintptr_t)p.B);
}

// 8-bit k-rows of ROWS bytes: the eight k-rows of a transposing read of two adjacent chunks fall into different bank groups
template <int ROWS>
__device__ __forceinline__ int small_swz_f8(int c, int k)
{
    return c ^ (2 * (ROWS == 64 ? (k >> 2) & 1 : (ROWS == 128 ? (k >> 1) & 3 : k & 7)));
}

// Byte offset, from the tile's first element, of the 16-byte chunk that lane `lane` of wave-load j fetches, and in `ck` the
// chunk's first contraction index within the stage.  The LDS position is the lane's (direct-to-LDS); the swizzle that
// keeps the fragment reads free of bank conflicts is applied here, on the global side.  `valid`: rows (columns) of the
// operand tile that exist; positions past it fetch the last existing row (chunk) again and are masked where results are stored.
template <class C, bool KCONT, int ROWS>
__device__ __forceinline__ uint32_t small_goffset(int j, int lane, int64_t ldb, int valid, int &ck)
{
    if constexpr (KCONT) {                           // [rows][128 B]: chunk c of row r at c ^ (r & 7), 8-bit c ^ ((r >> 1) & 7)
        const int r = j * 8 + (lane >> 3), c = (lane & 7) ^ ((C::F8 ? r >> 1 : r) & 7);
        ck = c * (16 / C::ESZ);
        return (uint32_t)((int64_t)(r < valid ? r : valid - 1) * ldb + c * 16);
    } else if constexpr (!C::F8) {                   // [64][ROWS columns]: the granule swizzle of lds_mn
        constexpr int CPR = ROWS / 8;
        const int idx = j * 64 + lane, k = idx / CPR, pc = idx % CPR;
        const int col = ((((pc >> 1) ^ mn_swz(k)) & (ROWS / 16 - 1)) * 2 + (pc & 1)) * 8;
        ck = k;
        return (uint32_t)((int64_t)k * ldb + (col < valid ? col : valid - 8) * 2);
    } else {                                         // [128][ROWS columns]: chunk c of k-row k at small_swz_f8(c, k)
        constexpr int CPR = ROWS / 16;
        const int idx = j * 64 + lane, k = idx / CPR, c = small_swz_f8<ROWS>(idx % CPR, k);
        ck = k;
        return (uint32_t)((int64_t)k * ldb + (c * 16 < valid ? c * 16 : valid - 16));
    }
}

template <class C>
using SmallFrag = typename std::conditional<C::F8, i32x8, bf16x8>::type;
template <class C>
using SmallAcc = typename std::conditional<C::F8, Acc32<C>, Acc16<C>>::type;

// Fragment of C::FR rows (columns) from row0 on, step h (0 / 1) of the stage: bf16: lane -> row lane % 16, k = 32 h + 8 (lane / 16)
// .. + 7; 8-bit: row lane % 32, k = 64 h + 32 (lane / 32) .. + 31.
template <class C, bool KCONT, int ROWS>
__device__ __forceinline__ SmallFrag<C> small_frag(const unsigned char *tile, int row0, int lane, int h)
{
    if constexpr (C::F8 && KCONT) {
        return dl_frag_pair_f8(tile, row0, lane, h);
    } else if constexpr (C::F8) {
        // transposing reads as in dl_frag_mn_f8, eight k-rows each: the lane's four reads are its 32 consecutive k
        typedef int v2i __attribute__((ext_vector_type(2)));
        typedef __attribute__((address_space(3))) v2i lds_v2i;
        const int i = lane & 15, g = lane >> 4, k0 = 64 * h + 32 * (g >> 1) + (i >> 1);      // k0 & 7 is the same in all four reads
        const unsigned char *a = tile + k0 * ROWS + (small_swz_f8<ROWS>((row0 >> 4) + (g & 1), k0) << 4) + ((i & 1) << 3);
        const v2i r0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(a));
        const v2i r1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(a + 8 * ROWS));
        const v2i r2 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(a + 16 * ROWS));
        const v2i r3 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(a + 24 * ROWS));
        return i32x8{r0[0], r0[1], r1[0], r1[1], r2[0], r2[1], r3[0], r3[1]};
    } else if constexpr (KCONT) {
        return dl_frag16_pair(tile, row0, lane, h);
    } else {
        return dl_frag16<ROWS, false>(tile + h * 32 * ROWS * 2, row0, lane);
    }
}

// Workgroup -> (range, tile): every XCD gets a contiguous run of ids, ranges outermost, tiles in groups of eight tile rows
// walked column by column (tile_coords), so that the workgroups of an XCD share operand panels in its L2.
__device__ __host__ __forceinline__ void small_coords(int bid, int tiles_m, int tiles_n, int nsplit, int &tm, int &tn, int &split)
{
    const int tiles = tiles_m * tiles_n, nb = tiles * nsplit;
    const int x = bid & 7, q = bid >> 3, base = nb >> 3, rem = nb & 7;
    const int id = x * base + (x < rem ? x : rem) + q;
    split = id / tiles;
    const int t = id - split * tiles, grp = t / (8 * tiles_n), first = grp * 8;
    const int gm = tiles_m - first < 8 ? tiles_m - first : 8, in = t - grp * 8 * tiles_n;
    tm = first + in % gm;
    tn = in / gm;
}

template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// loads of `ahead` stages (at most MAX) may be in flight
template <int MAX, int L>
__device__ __forceinline__ void wait_stages(int ahead)
{
    if constexpr (MAX <= 0) wait_loads<0>();
    else if (ahead == MAX) wait_loads<MAX * L>();
    else wait_stages<MAX - 1, L>(ahead);
}

// The contraction of one tile over the stages [kbeg, kbeg + KT) (elements from kbeg * BK on, zeros past K), KT >= 1.
// On return no wave reads or fills the ring any more.
template <class C, bool AK, bool BKC, bool CHAINS>
__device__ __forceinline__ void small_contract(SmallAcc<C> &acc, const SmallParams &p, int m0, int n0, int kbeg, int rot0, int KT,
                                               unsigned char *smem)
{
    static_assert(AK || C::BM == 128, "an A whose rows are not contiguous in K is staged as 128-wide k-rows");
    constexpr int NB = C::WTM / C::FR, NU = C::WTN / C::FR, S = C::S, L = C::LA + C::LB;
    typedef typename std::conditional<C::F8, f32x16, f32x4>::type Block;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % C::WGM, wn = wave / C::WGM;
    acc_zero(acc);
    uint32_t offa[C::LA], offb[C::LB];
    int cka[C::LA], ckb[C::LB];
    const int valid_m = p.M - m0 < C::BM ? p.M - m0 : C::BM, valid_n = p.N - n0 < C::BN ? p.N - n0 : C::BN;
#pragma unroll
    for (int i = 0; i < C::LA; ++i) offa[i] = small_goffset<C, AK, C::BM>(wave * C::LA + i, lane, p.lda, valid_m, cka[i]);
#pragma unroll
    for (int i = 0; i < C::LB; ++i) offb[i] = small_goffset<C, BKC, C::BN>(wave * C::LB + i, lane, p.ldb, valid_n, ckb[i]);
    const int64_t stepa = AK ? (int64_t)C::BKB : C::BK * p.lda, stepb = BKC ? (int64_t)C::BKB : C::BK * p.ldb;
    const unsigned char *ga = p.A + (AK ? (int64_t)m0 * p.lda : (int64_t)m0 * C::ESZ) + kbeg * stepa;
    const unsigned char *gb = p.B + (BKC ? (int64_t)n0 * p.ldb : (int64_t)n0 * C::ESZ) + kbeg * stepb;
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    // The stage that reaches past K (the last one of the last range, if K is not a whole number of stages): a lane whose
    // chunk lies past K stores zeros at its LDS position instead of fetching.  Fewer loads than L may then be counted, so
    // from the issue of that stage on the waits are for everything.
    const bool ragged = (kbeg + KT) * C::BK > p.K;
    // B rows contiguous in K: the rows of a stage lie a whole row pitch apart, which for the usual widths is a multiple of
    // the memory channels' interleave, so workgroups that walk K in step would all pull on the same few channels.  Where
    // p.rot_cols says so, every column of tiles starts its range at another stage and wraps around (28672 x 4096 8-bit, one
    // row: 30 us against 27; 65536 x 4096 bf16, one row, undivided: 124 against 97).
    const int rot = __builtin_amdgcn_readfirstlane(BKC && !ragged ? rot0 % KT : 0);
    int next = rot;                                  // the next stage to fetch, and its slot
    uint32_t slot_in = 0;
    auto advance = [&]() {
        ++next;
        if (BKC) next = next == KT ? 0 : next;
        slot_in = slot_in + C::STAGE == C::LDS ? 0u : slot_in + C::STAGE;
    };
    auto load_b = [&](uint32_t off, const void *from, uint32_t to) {
        if constexpr (C::ONCE) dl_load16_once(off, from, to);
        else dl_load16(off, from, to);
    };
    // part q of Q of the stage's loads; the last part moves on to the next stage
    auto issue_part = [&](int q, int Q) {
        const unsigned char *sa = ga + (int64_t)next * stepa, *sb = gb + (int64_t)next * stepb;
        const uint32_t la = lds0 + slot_in + (uint32_t)(wave * C::LA * 1024), lb = lds0 + slot_in + (uint32_t)(C::A_BYTES + wave * C::LB * 1024);
#pragma unroll
        for (int i = 0; i < L; ++i) {
            if (i < q * L / Q || i >= (q + 1) * L / Q) continue;
            if (i < C::LA) dl_load16(offa[i < C::LA ? i : 0], sa, la + (uint32_t)(i * 1024));
            else load_b(offb[i < C::LA ? 0 : i - C::LA], sb, lb + (uint32_t)((i - C::LA) * 1024));
        }
        if (q == Q - 1) advance();
    };
    auto issue = [&]() { issue_part(0, 1); };
    auto issue_last = [&]() {                        // the stage that reaches past K
        const int have = p.K - (kbeg + KT - 1) * C::BK;
        const unsigned char *sa = ga + (int64_t)next * stepa, *sb = gb + (int64_t)next * stepb;
        unsigned char *slot = smem + slot_in + lane * 16;
#pragma unroll
        for (int i = 0; i < C::LA; ++i) {
            const int at = (wave * C::LA + i) * 1024;
            if (cka[i] < have) dl_load16(offa[i], sa, lds0 + slot_in + (uint32_t)at);
            else *reinterpret_cast<u32x4 *>(slot + at) = u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int i = 0; i < C::LB; ++i) {
            const int at = C::A_BYTES + (wave * C::LB + i) * 1024;
            if (ckb[i] < have) load_b(offb[i], sb, lds0 + slot_in + (uint32_t)at);
            else *reinterpret_cast<u32x4 *>(slot + at) = u32x4{0u, 0u, 0u, 0u};
        }
    };
    SmallFrag<C> fa[NB], fb[NU], ha[NB], hb[NU];     // fragments of a stage's first and second MFMA step
    uint32_t slot_out = 0;                           // the slot being read
    // part q of Q of a step's fragments
    auto read_part = [&](SmallFrag<C>(&fa)[NB], SmallFrag<C>(&fb)[NU], int h, int q, int Q) {
        const unsigned char *ta = smem + slot_out, *tb = ta + C::A_BYTES;
#pragma unroll
        for (int u = 0; u < NU; ++u)
            if (u >= q * NU / Q && u < (q + 1) * NU / Q) fb[u] = small_frag<C, BKC, C::BN>(tb, wn * C::WTN + u * C::FR, lane, h);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (i >= q * NB / Q && i < (q + 1) * NB / Q) fa[i] = small_frag<C, AK, C::BM>(ta, wm * C::WTM + i * C::FR, lane, h);
    };
    // One MFMA step on f*, a row of blocks at a time (8-bit: block by block, those take twice as long).  `beside(i, n)` issues part i
    // of n of the loads and fragment reads of the next step: behind row i where two waves share a SIMD in step, so that the
    // matrix pipe starts at once after a barrier and works while they are issued in its shadow (128x256: 509 x 16384 x 2048
    // 37.5 -> 34.7 us); ahead of the rows where a wave has its SIMD to itself or shares it with another workgroup's (1 x 6144 x
    // 2048 at 64x64: 12.8 us against 13.5).
    auto mma = [&](const SmallFrag<C>(&fa)[NB], const SmallFrag<C>(&fb)[NU], auto beside) {
        if (C::NW < 8) {
#pragma unroll
            for (int i = 0; i < NB; ++i) beside(i, NB);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if (C::NW >= 8 || i == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                if constexpr (C::F8)
                    acc.a[i][u] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[u], fa[i], acc.a[i][u], 0, 0, 0, 0, 0, 0);
                else
                    acc.a[i][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[u], fa[i], acc.a[i][u], 0, 0, 0);
                if (C::NW < 8 || !C::F8) continue;
                __builtin_amdgcn_sched_barrier(0);
                beside(i * NU + u, NB * NU);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (C::NW < 8 || C::F8) continue;
            __builtin_amdgcn_sched_barrier(0);
            beside(i, NB);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // Behind the wait for a stage's loads: this wave's own LDS reads so far have returned and its zero stores are done;
    // behind the barrier that, and the stage's arrival, hold for all waves: it may be read, the slot before it refilled.
    auto meet = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0), known to the compiler: its own waits below count from here
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };
    // Chains: the accumulators are added to `sum` and start again from zero every p.chain stages, so that a range that is longer
    // than the ones the shape had on shared 256 x 256 tiles is no less accurate (509 x 2048 x 8192 in four ranges against 64 bits:
    // 2.7e-7 in one chain each, 1.9e-7 in two, as in eight ranges).  Not in launches that nothing divides (2 to 3 % at
    // 128x256; 8-bit 1 %).
    Block sum[CHAINS ? NB : 1][CHAINS ? NU : 1];
    int chain = p.chain;
    if constexpr (CHAINS) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int u = 0; u < NU; ++u) sum[i][u] = Block{};
    }
    auto end_of_stage = [&]() {
        if constexpr (CHAINS)
            if (--chain == 0) {
                chain = p.chain;
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int u = 0; u < NU; ++u) {
                        sum[i][u] += acc.a[i][u];
                        acc.a[i][u] = Block{};
                    }
            }
    };
    auto next_slot = [&]() { slot_out = slot_out + C::STAGE == C::LDS ? 0u : slot_out + C::STAGE; };
    // Stage t, f* being read already; the reads of the next MFMA step are in flight under every step.  The last step of a stage
    // takes its next fragments from the next stage: that is where the stage's one barrier and the refill of its slot are.
    // `steady`: the refill exists and lies inside K, no stage in flight is the one past K.
    auto stage = [&](int t, bool steady) {
        mma(fa, fb, [&](int i, int n) { read_part(ha, hb, 1, i, n); });
        const bool more = steady || t + 1 < KT;      // there is a next stage to read
        bool fill = steady;                          // and one to fetch, in full
        if (steady) {
            wait_loads<(S - 2) * L>();
            meet();
            next_slot();
        } else if (more) {
            const int ahead = KT - 2 - t;            // stages behind t + 1
            if (ragged && ahead <= S - 1) wait_loads<0>();
            else if (ahead >= S - 2) wait_loads<(S - 2) * L>();
            else wait_stages<S - 3, L>(ahead);
            meet();
            next_slot();
            fill = t + S < KT;
            if (ragged && t + S == KT - 1) {
                issue_last();
                fill = false;
            }
        }
        mma(ha, hb, [&](int i, int n) {
            if (fill) issue_part(i, n);
            if (more) read_part(fa, fb, 0, i, n);
        });
        end_of_stage();
    };
#pragma unroll
    for (int t = 0; t < S; ++t)
        if (t < KT) {
            if (ragged && t == KT - 1) issue_last();
            else issue();
        }
    if (KT >= S && !(ragged && KT == S)) {
        wait_loads<(S - 1) * L>();
    } else {
        wait_loads<0>();
    }
    meet();
    read_part(fa, fb, 0, 0, 1);
    int t = 0;
    for (; t + S + (ragged ? 1 : 0) < KT; ++t) stage(t, true);
    for (; t < KT; ++t) stage(t, false);
    if constexpr (CHAINS) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int u = 0; u < NU; ++u) acc.a[i][u] = sum[i][u] + acc.a[i][u];
    }
    __syncthreads();
}

template <class C, bool AK, bool BKC>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2, 2), amdgpu_num_vgpr(256))) void gemm_small_partial(const SmallParams p)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[C::LDS];
    int tm, tn, split;
    small_coords((int)blockIdx.x, p.tiles_m, p.tiles_n, p.nsplit, tm, tn, split);
    const int stages = (p.K + C::BK - 1) / C::BK;
    const int k0 = __builtin_amdgcn_readfirstlane((int)((int64_t)split * stages / p.nsplit));
    const int k1 = __builtin_amdgcn_readfirstlane((int)((int64_t)(split + 1) * stages / p.nsplit));   // k1 > k0: nsplit <= stages
    SmallAcc<C> acc;
    const int m0 = tm * C::BM, n0 = tn * C::BN;
    small_contract<C, AK, BKC, true>(acc, p, m0, n0, k0, n0 / p.rot_cols, k1 - k0, smem);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int mw = m0 + wave % C::WGM * C::WTM, nw = n0 + wave / C::WGM * C::WTN;
    float *out = p.part + (int64_t)split * p.M * p.N;
    using ACC = SmallAcc<C>;
    constexpr int RB = C::WTN * 4, UB = 16 * ACC::LQ, LR = ACC::LR;
    if constexpr (C::F8 || C::BM == 128) {
        // straight from registers a lane and its partners would store 32 (8-bit) or 64 bytes of a row: rows of the wave's tile, 256 bytes of 128x256 and 128
        // of 128x128, by way of LDS (eight ranges of 256 x 1984 x 4336 8-bit: 17.2 us, from registers 18.9; bf16, contraction and epilogue, 128x128: 159 x 640 x
        // 10928 18.4 -> 17.4, 509 x 2048 x 8192 34.7 -> 34.3, of 28 shapes one 0.6 % slower; 128x256: 144 x 10144 x 3848 39.8 -> 37.5, 1000 x 2048 x 5632 39.8 -> 39.4)
        unsigned char *reg = smem + wave * LR * RB;
        const uint32_t ulane = Stage<RB>::template unit_lane<16, LR>(lane);
#pragma unroll
        for (int i = 0; i < ACC::NB; ++i) {
#pragma unroll
            for (int u = 0; u < ACC::NU; ++u)
                *reinterpret_cast<f32x4 *>(reg + Stage<RB>::template unit_addr<LR>(ulane, 0, u * UB)) = acc.get(i, u);
            stage_fence();
            stage_store<RB, LR, true, false>(reg, reinterpret_cast<unsigned char *>(out + (int64_t)(mw + i * LR) * p.N + nw), (int64_t)p.N * 4,
                                             p.M - mw - i * LR, (p.N - nw) * 4, lane);
            stage_fence();
        }
    } else {                                         // up to 64 rows, often few: one row 80.3 us a block, by way of LDS 80.5
        const int m = mw + (lane & 15), n = nw + (lane >> 4) * 4;
#pragma unroll
        for (int i = 0; i < ACC::NB; ++i)
#pragma unroll
            for (int u = 0; u < ACC::NU; ++u)
                if (m + i * 16 < p.M && n + u * 16 < p.N)
                    *reinterpret_cast<f32x4 *>(out + (int64_t)(m + i * 16) * p.N + n + u * 16) = acc.get(i, u);
    }
}

// The contraction of a whole tile, then the epilogue program of the large kernels on it.
template <class C>
struct SmallLds {
    static constexpr int RED = 2 * C::WGN * C::BM * 4, BYTES = C::LDS + RED;
    static_assert(BYTES <= 160 * 1024, "LDS");
};
template <class C, bool AK, bool BKC, int EPI, bool CHAINS>
__device__ __forceinline__ void small_tile(const GemmParams &g, const SmallParams &p, unsigned char *smem)
{
    static_assert(EPI != EPI_RMSNORM_BWD, "column partials are per 256 rows");
    int tm, tn, split;
    small_coords((int)blockIdx.x, p.tiles_m, p.tiles_n, 1, tm, tn, split);
    const int m0 = tm * C::BM, n0 = tn * C::BN;
    SmallAcc<C> acc;
    const int stages = (p.K + C::BK - 1) / C::BK;
    int rot0 = 0;
    if (BKC && p.rot_cols == ROT_XCD)
        rot0 = xcd_rotation(tile_xcd(m0 / 256, n0 / 256, (p.M + 255) / 256, (p.N + 255) / 256), 2 * stages) / 2;
    else if (BKC && p.rot_cols)
        rot0 = n0 / p.rot_cols;
    small_contract<C, AK, BKC, CHAINS>(acc, p, m0, n0, 0, rot0, stages, smem);
    float *red = reinterpret_cast<float *>(smem + C::LDS);
    if (C::BM < 128 || m0 + C::BM > p.M || n0 + C::BN > p.N)
        run_epilogue<C, SmallAcc<C>, EPI, true, C::LDS>(acc, g, m0, n0, tn, smem, red, (int)threadIdx.x);
    else
        run_epilogue<C, SmallAcc<C>, EPI, false, C::LDS>(acc, g, m0, n0, tn, smem, red, (int)threadIdx.x);
}

// The whole launch in one kernel.  The callers' row-reduction partials are per 256 columns, so programs with one take the 256-wide
// tiles.
template <class C, bool AK, bool BKC, int EPI, bool CHAINS>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2, 2), amdgpu_num_vgpr(256))) void gemm_small_direct(const GemmParams g, const SmallParams p)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[SmallLds<C>::BYTES];
    small_tile<C, AK, BKC, EPI, CHAINS>(g, p, smem);
}

// A division into one range (up to 64 rows, weights of 129 to 256 tiles of 128 columns) for a program without row reductions: nothing
// to add up, so no partials and no second kernel.  Bound by HBM: one row of 28672 x 4096 bf16 in 43.8 us with the launch (partials and a
// second kernel: 45.0), past the caches in 38.6, 6.1 TB/s.
template <class C, bool BKC, int EPI>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2, 2), amdgpu_num_vgpr(256))) void gemm_small_stream(const GemmParams g, const SmallParams p)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[SmallLds<C>::BYTES];
    small_tile<C, true, BKC, EPI, true>(g, p, smem);
}

}  // namespace coda
