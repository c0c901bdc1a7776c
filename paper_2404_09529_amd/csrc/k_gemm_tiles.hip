// Projection GEMMs on smaller output tiles than k_gemm_bf16.hip's 256 x 256: C[M, N] =
// A[M, K] B[N, K]^T (bf16, float32 accumulation) for batches whose 256 x 256 tiles are too few,
// or too badly divided, for the 256 CUs.
//
// What bounds it: each K-step of 64 moves (BM + BN) x 128 bytes into LDS for BM BN 128 flops, and
// a CU receives about 60 GB/s with warm weights, 30-50 in a call, whatever the tile and the ring depth (8 steps
// ahead are no faster than 4, and the kernel without its MFMAs takes the same time); lines that were in
// L2 before the launch reach it at 120-150 GB/s.  60-84% of its requests hit L2 (counters): an XCD
// misses a line about once, but its tiles walk K together and ask for the line in the same steps, so
// the hits seem to wait for that miss, and a CU's requests in flight over that latency to be its rate.
// So the time is bytes per CU: small tiles on all the CUs for a few hundred rows, larger ones as
// soon as they fill the CUs.
// Measured (us, 256 x 256 tiles -> the tile chosen): 344 rows, N 2048, K 5504: 109 -> 25 (64 x 64);
// 344 rows, N 11008, K 2048: 46 -> 33 (128 x 256); 150 rows, N 2048, K 5504: 111 -> 22 (32 x 64);
// 1309 rows, N 2048, K 5504: 110 -> 47 (128 x 128; 57-59 in an MLP call, whose activations were written
// just before and whose weights come from HBM); 512 rows, N 4096, K 14336: 259 -> 102 (128 x 64).
//
// One 256-thread workgroup (2 x 2 wavefronts) per tile, persistent: a workgroup's tiles form one
// stream of K-steps through an LDS ring of NS slots (A rows, then B rows of one step), filled
// with direct-to-LDS loads of whole 128-byte row segments, NS - 1 steps ahead; the loads of the
// next tile's first steps are in flight while a tile's epilogue runs.  Per step one barrier: a
// wavefront reads the second half's fragments while the first half's MFMAs run, waits for the
// next step's loads, and after the barrier refills the slot it has just finished reading.
//
// The sum of an output element runs over K in ascending 32-wide MFMA steps, exactly as in the
// 256 x 256 kernel, and the epilogue arithmetic is shared: results are bit-identical whichever
// tile computes them.
#include <algorithm>

#include "device.h"
#include "gemm_epilogue.h"
#include "gemm_tiles.h"
#include "kernels.h"

namespace {

constexpr int BK = 64, ROW_B = BK * 2, NT = 256;
constexpr int kListRows = 256;   // rows of one entry of a plan's row-tile list
// Buffer descriptor word 3 for raw (unstructured) 32-bit-offset loads on gfx9-family parts.
constexpr int kRsrcWord3 = 0x00020000;
// s_waitcnt immediate: vmcnt(n) and lgkmcnt(0), expcnt not waited for (gfx9 encoding).
constexpr int wait_vm_lgkm0(int n) { return ((n >> 4) << 14) | (n & 15) | 0x0070; }
typedef __attribute__((address_space(3))) void lds_void;

// LDS swizzle of 128-byte rows: 16-byte chunk c of row r at chunk c ^ swz(r).  A fragment read
// takes chunk 4 ks + l / 16 of rows l % 16, lanes i and i + 32 served together: 8 rows x chunks
// {c, c ^ 2} on distinct banks (the derivation stands in k_gemm_bf16.hip).
__device__ __forceinline__ int swz(int r) { return ((r >> 1) & 1) | (((r >> 3) & 1) << 1) | (r & 4); }

__device__ __forceinline__ void barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// Wavefront (wm, wn) of a tile holds MB x NB blocks of 16 x 16: activation rows
// wm 16 MB + 16 j + .., weight rows wn 16 NB + 16 i + .. of the tile's B rows in LDS order.
template <int BM_, int BN_, int NS_>
struct Geom {
    static constexpr int BM = BM_, BN = BN_, NS = NS_;
    static constexpr int MB = BM / 32, NB = BN / 32;
    static constexpr int A_LD = BM * ROW_B / 1024 / 4, B_LD = BN * ROW_B / 1024 / 4;   // 1 KB loads per wavefront
    static constexpr int STEP_LD = A_LD + B_LD;
    static constexpr int SLOT_B = (BM + BN) * ROW_B;
    static constexpr int LDS = NS * SLOT_B;
    static_assert(A_LD >= 1 && B_LD >= 1 && NS >= 3 && LDS <= 160 * 1024 && (NS - 1) * STEP_LD <= 63, "ring");
};

// Weight row of LDS row r of the tile whose first weight row is n0, relative to n0.  QKV: a
// wavefront holds the rotate-half partners (dims c and c + 64 of a head) of NB / 2 blocks, its
// blocks 0 .. NB / 2 - 1 being c's and the others the partners'; a 64-row tile is 32 dims of a
// head and their partners (n0 = the head's first row + 0 or 32), wider tiles are whole heads.
template <int EPI, class G>
__device__ __forceinline__ int b_row(int r) {
    if constexpr (EPI == ppk::kQkvRope) {
        constexpr int W = 16 * G::NB, H = W / 2;   // rows per wavefront, and of its lower half
        const int wn = r / W, x = r % W, part = x / H;
        if constexpr (W >= 128) return r;          // the wavefront is a whole head
        else return part * 64 + wn * H + x % H;
    } else {
        return r;
    }
}

// Where a kernel's results go beside C.
template <int EPI>
struct OutOf {
    using type = ppk::QkvOut;
};
template <>
struct OutOf<ppk::kLogits> {
    using type = LogitsOut;
};

// mt_first: index of the first entry of the row-tile list (or of the 256-row tiles of M) that
// this launch takes; n_mt entries from there.  Each is kListRows / BM row tiles; those of the
// batch's last entry that start past M are left out.  The (row tile, column tile) list goes
// column by column in groups of at most GM row tiles and is cut into 8 contiguous ranges, one
// per XCD (workgroup id mod 8): the tiles resident on an XCD form a compact block, and for
// batches of up to GM row tiles every weight row is read by one XCD only.
template <int EPI, int BM, int BN, int NS, int WGS>
__global__ __launch_bounds__(NT, WGS) void gemm_tiles_kernel(const bf16* __restrict__ A, int64_t lda,
                                                             const bf16* __restrict__ B, int64_t ldb,
                                                             void* __restrict__ Cv, int64_t ldc, int M, int N, int K,
                                                             const int32_t* __restrict__ mtile_m0, int mt_first,
                                                             int n_mt, typename OutOf<EPI>::type qo) {
    using G = Geom<BM, BN, NS>;
    constexpr int MB = G::MB, NB = G::NB;
    constexpr int SUB = kListRows / BM, GM = 2048 / BM;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    const int last0 = mtile_m0 ? mtile_m0[mt_first + n_mt - 1] : (mt_first + n_mt - 1) * kListRows;
    const int tiles_m = (n_mt - 1) * SUB + min(SUB, (M - last0 + BM - 1) / BM);
    const int tiles_n = EPI == ppk::kLogits ? (N + BN - 1) / BN : N / BN;   // (only the logits' N may be ragged)
    const int xcd = blockIdx.x & 7, slot0 = blockIdx.x >> 3, n_slots = gridDim.x >> 3;
    const int total = tiles_m * tiles_n, per = (total + 7) / 8;
    const int g_begin = xcd * per, n_local = min(per, total - g_begin);
    const int n_groups = (tiles_m + GM - 1) / GM, gm = (tiles_m + n_groups - 1) / n_groups;
    if (slot0 >= n_local) return;
    auto tile_m0n0 = [&](int local, int& m0, int& n0) {
        const int gi = g_begin + local;
        const int group = gi / (gm * tiles_n), within = gi - group * gm * tiles_n;
        const int first = group * gm, gsz = min(tiles_m - first, gm);
        const int mt = first + within % gsz, nt = within / gsz;
        const int entry = mt_first + mt / SUB;
        m0 = (mtile_m0 ? mtile_m0[entry] : entry * kListRows) + mt % SUB * BM;
        n0 = EPI == ppk::kQkvRope && BN == 64 ? nt / 2 * 128 + nt % 2 * 32 : nt * BN;
    };
    // this workgroup's K-steps (all of them but for kPartial's splits, blockIdx.y of gridDim.y)
    const int k_first = K / BK * blockIdx.y / gridDim.y, nk = K / BK * (blockIdx.y + 1) / gridDim.y - k_first;
    if constexpr (EPI == ppk::kPartial) Cv = static_cast<float*>(Cv) + int64_t(blockIdx.y) * M * ldc;

    // ---- direct global -> LDS loads: each fills 1 KB = 8 rows x 128 bytes of a slot, lane l
    // landing at physical chunk l % 8 of row l / 8 and fetching the logical chunk that the
    // swizzle puts there.  Rows of A past M are read as row M - 1: every load is in range, so
    // loads complete in the order they were issued.
    const int64_t lda2 = lda * 2, ldb2 = ldb * 2;
    const int lrow = lane >> 3;
    int voff_a[G::A_LD], voff_b[G::B_LD];
#pragma unroll
    for (int t = 0; t < G::B_LD; ++t) {
        const int r = 8 * (G::B_LD * wave + t) + lrow;
        voff_b[t] = static_cast<int>(b_row<EPI, G>(r) * ldb2) + 16 * ((lane & 7) ^ swz(r));
    }
    // load cursor: the K-step being requested, into slot l_slot; past the last one its loads go
    // through an empty descriptor (they read nothing and land in slots that are not read again)
    int l_local = slot0, l_kt = 0, l_slot = 0;
    __amdgpu_buffer_rsrc_t rsrc_a, rsrc_b;
    const __amdgpu_buffer_rsrc_t rsrc_0 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(A), 0, 0, kRsrcWord3);
    auto set_cursor_tile = [&]() {
        if (l_local < n_local) {
            int m0, n0;
            tile_m0n0(l_local, m0, n0);
            const int a_rows = min(M - m0, BM);
            constexpr int b_rows = EPI == ppk::kQkvRope && BN == 64 ? 96 : BN;
            rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(A + int64_t(m0) * lda), 0,
                                                       static_cast<int>(a_rows * lda2), kRsrcWord3);
            const int b_here = EPI == ppk::kLogits ? min(N - n0, b_rows) : b_rows;
            rsrc_b = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(B + int64_t(n0) * ldb), 0,
                                                       static_cast<int>(b_here * ldb2), kRsrcWord3);
            if constexpr (EPI == ppk::kLogits) {   // rows past the vocabulary read its last row
#pragma unroll
                for (int t = 0; t < G::B_LD; ++t) {
                    const int r = 8 * (G::B_LD * wave + t) + lrow;
                    voff_b[t] = static_cast<int>(min(r, b_here - 1) * ldb2) + 16 * ((lane & 7) ^ swz(r));
                }
            }
#pragma unroll
            for (int t = 0; t < G::A_LD; ++t) {
                const int r = 8 * (G::A_LD * wave + t) + lrow;
                voff_a[t] = static_cast<int>(min(r, a_rows - 1) * lda2) + 16 * ((lane & 7) ^ swz(r));
            }
        } else {
            rsrc_a = rsrc_0;
            rsrc_b = rsrc_0;
        }
    };
    set_cursor_tile();
    auto load = [&](int t) {   // t of the step's STEP_LD loads: A first
        const bool is_a = t < G::A_LD;
        char* dst = smem + l_slot * G::SLOT_B + (is_a ? (G::A_LD * wave + t) * 1024
                                                      : BM * ROW_B + (G::B_LD * wave + t - G::A_LD) * 1024);
        const int voff = is_a ? voff_a[is_a ? t : 0] : voff_b[is_a ? 0 : t - G::A_LD];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(is_a ? rsrc_a : rsrc_b, (lds_void*)dst, 16, voff, (k_first + l_kt) * ROW_B,
                                                 0, 0);
    };
    auto advance_cursor = [&]() {
        l_slot = l_slot == NS - 1 ? 0 : l_slot + 1;
        if (l_local >= n_local) return;
        if (++l_kt == nk) {
            l_kt = 0;
            l_local += n_slots;
            set_cursor_tile();
        }
    };

    const int wn = wave & 1, wm = wave >> 1;
    int a_lds[2], b_lds[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int phys = ((4 * ks + (lane >> 4)) ^ swz(lane & 15)) * 16;
        a_lds[ks] = (wm * 16 * MB + (lane & 15)) * ROW_B + phys;
        b_lds[ks] = (BM + wn * 16 * NB + (lane & 15)) * ROW_B + phys;
    }
    struct Frags { bf16x8 w[NB], a[MB]; };
    auto read_one = [&](int slot, int ks, int q, Frags& f) {   // w0, a0 .., w1 ..: as the MFMAs need them
        const char* base = smem + slot * G::SLOT_B;
        if (q == 0) f.w[0] = *reinterpret_cast<const bf16x8*>(base + b_lds[ks]);
        else if (q <= MB) f.a[q - 1] = *reinterpret_cast<const bf16x8*>(base + a_lds[ks] + (q - 1) * 16 * ROW_B);
        else f.w[q - MB] = *reinterpret_cast<const bf16x8*>(base + b_lds[ks] + (q - MB) * 16 * ROW_B);
    };

    // ---- prologue: the first NS steps requested, the first one awaited
#pragma unroll
    for (int p = 0; p < NS; ++p) {
#pragma unroll
        for (int t = 0; t < G::STEP_LD; ++t) load(t);
        advance_cursor();
    }
    if (l_local < n_local) __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0((NS - 1) * G::STEP_LD));
    else __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
    barrier();
    Frags F0, F1;
    int c_slot = 0, c_local = slot0;
#pragma unroll
    for (int q = 0; q < NB + MB; ++q) read_one(0, 0, q, F0);

    while (true) {
        f32x4 acc[NB][MB];
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j) acc[i][j] = f32x4{};
        // the MFMAs on `cur` with the next half's fragment reads (and, in the second half, the
        // loads of the step that refills the slot just read) spread between them
        auto half = [&](const Frags& cur, Frags& nxt, int slot, int ks, bool refill) {
            constexpr int MF = NB * MB, RD = NB + MB;
#pragma unroll
            for (int m = 0; m < MF; ++m) {
                const int i = m / MB, j = m % MB;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur.w[i], cur.a[j], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = m * RD / MF; q < (m + 1) * RD / MF; ++q) read_one(slot, ks, q, nxt);
                if (refill) {
#pragma unroll
                    for (int t = m * G::STEP_LD / MF; t < (m + 1) * G::STEP_LD / MF; ++t) load(t);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        for (int kt = 0; kt < nk; ++kt) {
            const int n_slot = c_slot == NS - 1 ? 0 : c_slot + 1;
            half(F0, F1, c_slot, 1, false);
            // the next step is in when at most the NS - 2 steps requested after it are pending
            // (everything, once the last steps' loads are dead)
            if (l_local < n_local) __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0((NS - 2) * G::STEP_LD));
            else __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
            barrier();
            half(F1, F0, n_slot, 0, true);
            advance_cursor();
            c_slot = n_slot;
        }
        int m0, n0;
        tile_m0n0(c_local, m0, n0);
        if constexpr (EPI == ppk::kLogits)
            epilogue_logits<MB>(acc, M, m0 + wm * 16 * MB, n0 + wn * 16 * NB, lane, qo);
        else
            epilogue_direct<EPI, NB, MB>(acc, Cv, ldc, M, m0 + wm * 16 * MB, n0, wn, lane, qo);
        c_local += n_slots;
        if (c_local >= n_local) break;
    }
    __builtin_amdgcn_s_waitcnt(0);   // no load may still be writing LDS when the workgroup ends
}

// TILE: index into kTileRows / kTileCols; NS ring slots, WGS workgroups per CU.
template <int EPI, int TILE, int NS, int WGS>
void launch(const ppk::GemmArgs& g, int mt_first, int n_mt, int n_cu, hipStream_t s, int splits,
            const typename OutOf<EPI>::type& out) {
    constexpr int BM = ppk::kTileRows[TILE], BN = ppk::kTileCols[TILE];
    using G = Geom<BM, BN, NS>;
    static_assert(WGS * G::LDS <= 160 * 1024, "LDS of a CU's workgroups");
    static const bool attr = [] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tiles_kernel<EPI, BM, BN, NS, WGS>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS);
        return true;
    }();
    (void)attr;
    const int64_t tiles = int64_t(n_mt) * (kListRows / BM) * ((g.N + BN - 1) / BN);   // at least the kernel's count
    const int64_t grid = 8 * std::min<int64_t>((tiles + 7) / 8, WGS * (n_cu / 8));
    gemm_tiles_kernel<EPI, BM, BN, NS, WGS><<<dim3(static_cast<unsigned>(grid), splits), NT, G::LDS, s>>>(
        static_cast<const bf16*>(g.A), g.lda, static_cast<const bf16*>(g.B), g.ldb, g.C, g.ldc, g.M, g.N, g.K, g.mtile_m0,
        mt_first, n_mt, out);
}

template <int EPI>
void launch_tile(int tile, const ppk::GemmArgs& g, int mt_first, int n_mt, int n_cu, hipStream_t s, int splits) {
    switch (tile) {
        case 0: return launch<EPI, 0, 6, 2>(g, mt_first, n_mt, n_cu, s, splits, g.qkv);
        case 1: return launch<EPI, 1, 5, 2>(g, mt_first, n_mt, n_cu, s, splits, g.qkv);
        case 2: return launch<EPI, 2, 3, 2>(g, mt_first, n_mt, n_cu, s, splits, g.qkv);
        case 3: return launch<EPI, 3, 5, 1>(g, mt_first, n_mt, n_cu, s, splits, g.qkv);
        default: return launch<EPI, 4, 3, 1>(g, mt_first, n_mt, n_cu, s, splits, g.qkv);
    }
}

}  // namespace

namespace ppk {

void gemm_tiles(int epi, int tile, const GemmArgs& g, int mt_first, int n_mt, int n_cu, hipStream_t s, int splits) {
    switch (epi) {
        case kStore: return launch_tile<kStore>(tile, g, mt_first, n_mt, n_cu, s, splits);
        case kResidual: return launch_tile<kResidual>(tile, g, mt_first, n_mt, n_cu, s, splits);
        case kSwiGLU: return launch_tile<kSwiGLU>(tile, g, mt_first, n_mt, n_cu, s, splits);
        case kPartial: return launch_tile<kPartial>(tile, g, mt_first, n_mt, n_cu, s, splits);
        default: return launch_tile<kQkvRope>(tile, g, mt_first, n_mt, n_cu, s, splits);
    }
}

void lm_head_tiles(const void* hl, int k, const void* W, int V, int d, float* logits, void* part, int n_blocks,
                   hipStream_t s) {
    const LogitsOut out{logits, static_cast<ArgMax*>(part), V, n_blocks,
                        V % 4 == 0 && reinterpret_cast<uintptr_t>(logits) % 16 == 0};
    launch<kLogits, 4, 3, 1>(GemmArgs{hl, d, W, d, nullptr, 0, k, V, d, nullptr, QkvOut{}}, 0, (k + kListRows - 1) / kListRows,
                             cu_count(), s, 1, out);
}

}  // namespace ppk
