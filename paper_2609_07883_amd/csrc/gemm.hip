// bf16 GEMM out = A W^T on gfx950 matrix cores, with fused epilogues.
//
// A [m][k] and W [n][k] are both k-contiguous.  Three kernels:
//   tile_kernel    BM x BN output tiles staged through LDS, for everything
//                  but the smallest batches; k may be split across
//                  work-groups, whose fp32 partial sums a second kernel adds
//                  before it applies the same epilogue;
//   stream_kernel  weight streaming of wide gate/up projections for up to 8
//                  rows, with the RMSNorm before them folded in;
//   narrow_kernel  weight streaming of the other projections for a few rows,
//                  k split over the waves of one work-group.
//
// Two epilogues need two W rows of one output in the same lane: SwiGLU (a gate
// row and its up row) and QKV (dims i and i + hd/2 of a head, a RoPE pair).
// The kernels choose which W rows feed which MFMA rows so that the two sit in
// one lane (stream_kernel: in lanes 32 apart).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace slw {
namespace {

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// Head-local order of 32-dim blocks for hd = 128: B blocks 0,1,2,3 hold dims
// blocks 0,2,1,3 (the map is its own inverse).  hd = 64 needs no reordering.
__device__ __forceinline__ int qkv_dim(int cw, int hd) {
    if (hd != 128) return cw;
    const int b = cw >> 5;
    return ((((b & 1) << 1) | (b >> 1)) << 5) | (cw & 31);
}

// Rotate (x0, x1) = dims (d0, d0 + hd/2) of head hg of row `row` by the
// iteration's table (q and k heads; v heads are not rotated) and store; k and
// v also go to their KV page at slot[row].
__device__ __forceinline__ void qkv_store(const GemmArgs& g, int row, int hg, int d0, float x0, float x1) {
    const int d1 = d0 + g.hd / 2, slot = hg < g.hq ? 0 : g.slot[row];
    bf16* out = static_cast<bf16*>(g.out) + static_cast<size_t>(row) * g.ldo + hg * g.hd;
    if (hg < g.hq + g.hkv) {
        const float2 cs = g.rope_cs[row * (g.hd / 2) + d0];
        const float y0 = x0 * cs.x - x1 * cs.y;
        const float y1 = x1 * cs.x + x0 * cs.y;
        x0 = y0;
        x1 = y1;
    }
    const bf16 b0 = f2bf(x0), b1 = f2bf(x1);
    out[d0] = b0;
    out[d1] = b1;
    if (hg < g.hq) return;
    const size_t blk = slot >> 4, t = slot & 15;
    if (hg < g.hq + g.hkv) {
        bf16* pg = static_cast<bf16*>(g.k_pool) + (blk * g.hkv + (hg - g.hq)) * g.hd * 16;
        pg[(d0 >> 5) * 512 + t * 32 + (d0 & 31)] = b0;
        pg[(d1 >> 5) * 512 + t * 32 + (d1 & 31)] = b1;
    } else {
        bf16* pg = static_cast<bf16*>(g.v_pool) + (blk * g.hkv + (hg - g.hq - g.hkv)) * g.hd * 16;
        pg[d0 * 16 + t] = b0;
        pg[d1 * 16 + t] = b1;
    }
}

// Tile (tm, tn) at position t of the grouped tile order: group_m tile rows
// at a time, column by column within a group, so that tiles that run
// together share A rows and B columns.  With at most 16 tile rows a group
// spans them all: each weight panel is then streamed into an L2 once for
// every row tile.
__device__ __forceinline__ void tile_coords(int t, int nt_m, int nt_n, int& tm, int& tn) {
    const int GROUP_M = nt_m <= 16 ? nt_m : 8;
    const int per_group = GROUP_M * nt_n;
    const int first_m = (t / per_group) * GROUP_M;
    const int gsize = min(nt_m - first_m, GROUP_M);
    const int in_group = t % per_group;
    tm = first_m + in_group % gsize;
    tn = in_group / gsize;
}

__device__ __forceinline__ void tile_of(int pid, int nt_m, int nt_n, int& tm, int& tn) {
    tile_coords(xcd_order(pid, nt_m * nt_n), nt_m, nt_n, tm, tn);
}

// Wait until at most n vector-memory operations of this wave are
// outstanding (gfx9 s_waitcnt encoding, other counters left alone).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// Wait until at most N LDS operations of this wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
    static_assert(N >= 0 && N < 16, "lgkmcnt range");
    __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}

// Direct global->LDS load of 16 bytes per lane from base + off (base is
// wave-uniform): lane l's bytes land at lds + 16 l (lds is wave-uniform).
// Issued as assembly so that the compiler, which cannot tell which LDS buffer
// such a load writes, does not make every later LDS read wait for all of
// them; the main loop waits for them itself.  M0 is a reserved register that
// the compiler sets right before each instruction that reads it; no
// compiler-generated code in these kernels uses it, so the value left there
// is never relied on.
__device__ __forceinline__ void load_lds16(const void* base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds) : "memory");
}

// Workgroup barrier with no memory fence: the asm statement's memory clobber
// keeps the compiler from moving LDS or global accesses across it, and the
// waits it needs are issued explicitly before it.
__device__ __forceinline__ void barrier_only() { asm volatile("s_barrier" ::: "memory"); }

// ---------------------------------------------------------------------------
// Tile kernel.  Eight waves (WAVES_M x WAVES_N) compute a BM x BN tile with
// 16 x 16 x 32 MFMAs, weights as the A operand; k advances 64 at a time
// through two LDS buffers per operand.
//
// What bounds it: at the largest tile the chip runs into its power limit (the
// matrix cores are busy 72% of the cycles, and on all-zero operands the same
// kernel is 1.27 x faster: gate/up of the 8B layer at 4096 rows 661 -> 520 us,
// 1455 -> 1850 TFLOP/s), so the design saves energy per product as much as it
// hides latency: 16 x 16 x 32 MFMAs touch the accumulators half as often per
// product as 32 x 32 x 16 (+9% at 4096 x 28672 x 4096), every operand byte is
// read from LDS once per k step, and no register staging is used.
//
// Schedule.  A wave's tile is cut into four quadrants: its A rows in two
// halves (A0, A1), its B columns in two halves.  A k step runs four phases,
// one quadrant each, in the order A0 Bf, A0 Bs, A1 Bs, A1 Bf (first and second
// B half swap roles every step), so that each half is read from LDS once per
// step, one phase ahead of the MFMAs that need it:
//   phase 0 reads Bs(t), phase 1 A1(t), phase 2 A0(t+1), phase 3 Bf(t+1).
// A half's LDS region is free one phase after the phase that read it, and is
// refilled then with the same half of step t + 2 by direct global->LDS loads
// (phase 0 issues A0, phase 1 Bf, phase 2 Bs, phase 3 A1): each load has five
// phases to land, where a ring of whole steps drained its queue once a step.
// A phase ends on counted waits (this wave's reads of the phase before are
// done; its loads of the half read next have landed) and a bare barrier that
// makes both true for all waves.  LDS reads and loads are spread between the
// MFMAs of a phase, in an order pinned by scheduling barriers: issued together
// at its start, the loads of eight waves held up every wave's MFMAs (3-5%).
//
// Measured against the 256 x 256 two-buffer ring with 32 x 32 x 16 MFMAs that
// it replaced (8B layer, three weight sets in turn): gate/up 470 -> 374 us at
// 2080 rows (1040 -> 1306 TFLOP/s), 165 -> 98 at 512; down 286 -> 225 at
// 2080; qkv 138 -> 86 at 2080; output 109 -> 69 at 2080.
//
// LDS rows hold 64 bf16 (128 bytes, one cache line per load); the 16-byte
// chunk c of row r is stored at c ^ ((r >> 1) & 7), so that the rows read by
// eight consecutive lanes hit distinct banks.
//
// Column order.  MFMA row 4 g + e of the wave's B tile j (lane group g,
// element e of its result) takes the W row that gives a lane consecutive
// output columns over its tiles: 8 HB of them (16 at BN 256), or for the
// paired epilogues 4 HB outputs with both members of each pair, so every
// epilogue access is 8 or 16 bytes wide.
// ---------------------------------------------------------------------------
template <int BM_, int BN_, int WAVES_M_, int WAVES_N_>
struct Tile {
    static constexpr int BM = BM_, BN = BN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
    static constexpr int NW = WAVES_M * WAVES_N, THREADS = NW * 64;
    static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    // 16-row tiles of a wave's A halves, 16-column tiles of each B half
    static constexpr int HA = WM / 16, HA0 = (HA + 1) / 2, HA1 = HA - HA0, HB = WN / 32;
    // 1 KB loads (8 LDS rows) that fill each half, and how many of them a wave
    // issues; where the waves do not divide them, some piece is loaded twice
    // (the same bytes to the same place), so that every wave counts the same
    static constexpr int GA0 = WAVES_M * HA0 * 2, GA1 = WAVES_M * HA1 * 2, GB = WAVES_N * HB * 2;
    static constexpr int LA0 = (GA0 + NW - 1) / NW, LA1 = (GA1 + NW - 1) / NW, LB = (GB + NW - 1) / NW;
    static constexpr int LALL = LA0 + LA1 + 2 * LB;  // loads of a step
    static constexpr int ABUF = BM * 128, BBUF = BN * 128, LDS = 2 * (ABUF + BBUF);
    // two work-groups share a CU (four waves per SIMD, 128 registers) where LDS
    // and registers allow it
    static constexpr bool TWO = 2 * LDS <= 160 * 1024 && HA * 2 * HB * 4 + HA * 8 + HB * 16 <= 96;
    static_assert(BM % (16 * WAVES_M) == 0 && BN % (32 * WAVES_N) == 0 && HA >= 2, "whole MFMA tiles in every half");
    static_assert(LALL + LA0 + LB < 64, "vmcnt range");
};

// First W row of the lane's outputs and, for the paired epilogues, the row of
// their partners: lane group g of wave column wn of the tile at column n0.
template <int EPI, class T>
__device__ __forceinline__ void lane_cols(const GemmArgs& g, int n0, int wn, int grp, int& c0, int& c1) {
    if (EPI == EPI_SWIGLU) {
        c0 = (n0 >> 1) + wn * (T::WN / 2) + grp * 4 * T::HB;
        c1 = c0 + (g.n >> 1);
    } else if (EPI == EPI_QKV) {
        const int p = (n0 >> 1) + wn * (T::WN / 2) + grp * 4 * T::HB, half = g.hd >> 1;
        c0 = (p / half) * g.hd + p % half;
        c1 = c0 + half;
    } else {
        c0 = n0 + wn * T::WN + grp * 8 * T::HB;
        c1 = c0 + 4 * T::HB;
    }
}

// NV consecutive bf16 (4 or 8) at dst.
template <int NV>
__device__ __forceinline__ void store_bf16(bf16* dst, const bf16 (&v)[NV]) {
    if constexpr (NV == 8)
        *reinterpret_cast<bf16x8*>(dst) = bf16x8{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
    else
        *reinterpret_cast<bf16x4*>(dst) = bf16x4{v[0], v[1], v[2], v[3]};
}

// Epilogue of a wave's tile.  acc[i][j]: row 16 i + lane % 16, B tile j (HB
// tiles of the first half, then HB of the second), columns as in lane_cols.
// Rows past m are not stored; their table and residual reads are clamped to
// row m - 1.  Reads of a few row groups come before any of their stores: the
// compiler cannot tell that the stores do not alias them, so interleaved
// they would each wait out a memory round trip.
template <class T, int EPI, bool SPLIT>
__device__ __forceinline__ void tile_store(const GemmArgs& g, int m0, int n0, int wm, int wn, int lane,
                                           float* __restrict__ partial, const f32x4 (&acc)[T::HA][2 * T::HB]) {
    constexpr int HA = T::HA, HB = T::HB, NV = 4 * HB;
    const int rbase = m0 + wm * T::WM + (lane & 15);
    int c0, c1;
    lane_cols<EPI, T>(g, n0, wn, lane >> 4, c0, c1);
    if constexpr (SPLIT) {  // partial sums [m][n], W row order
#pragma unroll
        for (int i = 0; i < HA; ++i) {
            const int row = rbase + i * 16;
            if (row >= g.m) continue;
            float* p = partial + static_cast<size_t>(row) * g.n;
#pragma unroll
            for (int j = 0; j < HB; ++j) {
                *reinterpret_cast<f32x4*>(p + c0 + 4 * j) = acc[i][j];
                *reinterpret_cast<f32x4*>(p + c1 + 4 * j) = acc[i][HB + j];
            }
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int i = 0; i < HA; ++i) {
            const int row = rbase + i * 16;
            if (row >= g.m) continue;
            bf16 o[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) o[v] = f2bf(silu(acc[i][v / 4][v % 4]) * acc[i][HB + v / 4][v % 4]);
            store_bf16<NV>(static_cast<bf16*>(g.out) + static_cast<size_t>(row) * g.ldo + c0, o);
        }
    } else if constexpr (EPI == EPI_QKV) {
        const int half = g.hd >> 1, hg = c0 / g.hd, d0 = c0 % g.hd, d1 = d0 + half;
        const bool rot = hg < g.hq + g.hkv, paged = hg >= g.hq;
        constexpr int IC = 2;  // row groups whose tables are read at once
#pragma unroll
        for (int i0 = 0; i0 < HA; i0 += IC) {
            f32x4 cs[IC][2 * HB];  // (cos, sin) of the lane's NV dims
            int sl[IC];
#pragma unroll
            for (int i = 0; i < IC; ++i) {
                const int row = min(rbase + (i0 + i) * 16, g.m - 1);
                const f32x4* src = reinterpret_cast<const f32x4*>(g.rope_cs + static_cast<size_t>(row) * half + d0);
#pragma unroll
                for (int j = 0; j < 2 * HB; ++j) cs[i][j] = rot ? src[j] : f32x4{1.f, 0.f, 1.f, 0.f};
                sl[i] = paged ? g.slot[row] : 0;
            }
#pragma unroll
            for (int i = 0; i < IC; ++i) {
                const int row = rbase + (i0 + i) * 16;
                if (i0 + i >= HA || row >= g.m) continue;
                bf16 y0[NV], y1[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const float x0 = acc[i0 + i][v / 4][v % 4], x1 = acc[i0 + i][HB + v / 4][v % 4];
                    const float co = cs[i][v / 2][2 * (v & 1)], si = cs[i][v / 2][2 * (v & 1) + 1];
                    y0[v] = f2bf(rot ? x0 * co - x1 * si : x0);
                    y1[v] = f2bf(rot ? x1 * co + x0 * si : x1);
                }
                bf16* out = static_cast<bf16*>(g.out) + static_cast<size_t>(row) * g.ldo;
                store_bf16<NV>(out + c0, y0);
                store_bf16<NV>(out + c1, y1);
                if (!paged) continue;
                const size_t blk = sl[i] >> 4, t = sl[i] & 15;
                if (rot) {
                    bf16* pg = static_cast<bf16*>(g.k_pool) + (blk * g.hkv + (hg - g.hq)) * g.hd * 16 + t * 32;
                    store_bf16<NV>(pg + (d0 >> 5) * 512 + (d0 & 31), y0);
                    store_bf16<NV>(pg + (d1 >> 5) * 512 + (d1 & 31), y1);
                } else {
                    // dim-major page: consecutive rows of a chunk are consecutive
                    // tokens, so 16 lanes write one 32-byte row of the page
                    bf16* pg = static_cast<bf16*>(g.v_pool) + (blk * g.hkv + (hg - g.hq - g.hkv)) * g.hd * 16 + t;
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        pg[(d0 + v) * 16] = y0[v];
                        pg[(d1 + v) * 16] = y1[v];
                    }
                }
            }
        }
    } else {
        constexpr int IC = HA < 4 ? HA : 4;  // row groups whose residual is read at once
#pragma unroll
        for (int i0 = 0; i0 < HA; i0 += IC) {
            f32x4 r[IC][2 * HB];
#pragma unroll
            for (int i = 0; i < IC; ++i) {
                const size_t o = static_cast<size_t>(min(rbase + (i0 + i) * 16, g.m - 1)) * g.ldo + c0;
#pragma unroll
                for (int j = 0; j < 2 * HB; j += 2) {
                    if constexpr (EPI == EPI_RESID_F32OUT) {
                        const bf16x8 b = *reinterpret_cast<const bf16x8*>(static_cast<const bf16*>(g.resid) + o + 4 * j);
#pragma unroll
                        for (int e = 0; e < 8; ++e) r[i][j + e / 4][e % 4] = bf2f(b[e]);
                    } else {
                        const f32x4* src = reinterpret_cast<const f32x4*>(static_cast<const float*>(g.resid) + o + 4 * j);
                        r[i][j] = src[0];
                        r[i][j + 1] = src[1];
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < IC; ++i) {
                const int row = rbase + (i0 + i) * 16;
                if (i0 + i >= HA || row >= g.m) continue;
                const size_t o = static_cast<size_t>(row) * g.ldo + c0;
#pragma unroll
                for (int j = 0; j < 2 * HB; j += 2) {
                    const f32x4 a = acc[i0 + i][j] + r[i][j], b = acc[i0 + i][j + 1] + r[i][j + 1];
                    if constexpr (EPI == EPI_RESID_F32OUT) {
                        f32x4* dst = reinterpret_cast<f32x4*>(static_cast<float*>(g.out) + o + 4 * j);
                        dst[0] = a;
                        dst[1] = b;
                    } else {
                        const bf16 v[8] = {f2bf(a[0]), f2bf(a[1]), f2bf(a[2]), f2bf(a[3]),
                                           f2bf(b[0]), f2bf(b[1]), f2bf(b[2]), f2bf(b[3])};
                        store_bf16<8>(static_cast<bf16*>(g.out) + o + 4 * j, v);
                    }
                }
            }
        }
    }
}

// Grid (tiles, splits); blockIdx.y takes k_per_split of the k range.
template <class T, int EPI, bool SPLIT>
__global__ __launch_bounds__(T::THREADS, T::TWO ? T::NW / 2 : T::NW / 4) void tile_kernel(GemmArgs g,
                                                                                        float* __restrict__ partial,
                                                                                        int k_per_split) {
    constexpr int HA = T::HA, HA0 = T::HA0, HA1 = T::HA1, HB = T::HB, NW = T::NW, ABUF = T::ABUF, BBUF = T::BBUF;
    constexpr int LA0 = T::LA0, LA1 = T::LA1, LB = T::LB, LALL = T::LALL;
    constexpr int RA0 = HA0 * 2, RA1 = HA1 * 2, RB = HB * 2;  // LDS reads of each half per step
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    // A buffers of even and odd steps, then the B buffers
    __shared__ __attribute__((aligned(1024))) char smem[T::LDS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int wm = wave / T::WAVES_N, wn = wave % T::WAVES_N;
    int tm, tn;
    tile_of(blockIdx.x, (g.m + T::BM - 1) / T::BM, g.n / T::BN, tm, tn);
    const int m0 = tm * T::BM, n0 = tn * T::BN;
    const int nk = k_per_split / 64;
    const uint32_t lds0 =
        __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(&smem[0])));

    // Loads: lane l brings chunk (l % 8) ^ swizzle of row l / 8 of its piece.
    // Wave-uniform 64-bit bases (one per B half: a pair's rows may be far
    // apart) plus 32-bit lane offsets within the tile's rows.  Rows past m
    // read row m - 1: they only feed output rows that are never stored.
    const size_t k0 = static_cast<size_t>(blockIdx.y) * k_per_split;
    const char* Ab = static_cast<const char*>(g.a) + (static_cast<size_t>(m0) * g.lda + k0) * 2;
    int c00, c01;
    lane_cols<EPI, T>(g, n0, 0, 0, c00, c01);
    const char* Wb[2];
    Wb[0] = static_cast<const char*>(g.w) + (static_cast<size_t>(c00) * g.k + k0) * 2;
    Wb[1] = static_cast<const char*>(g.w) + (static_cast<size_t>(c01) * g.k + k0) * 2;
    uint32_t oA0[LA0], oA1[LA1], oB[2][LB], dA0[LA0], dA1[LA1], dB[2][LB];
    const int r_in = lane >> 3;
    auto chunk = [&](int row) { return ((lane & 7) ^ ((row >> 1) & 7)) * 16; };
    auto set_a = [&](int tiles, int first, int pieces, int i, uint32_t& off, uint32_t& dst) {
        const int piece = (wave + i * NW) % pieces, per = tiles * 2;
        const int r0 = (piece / per) * T::WM + first * 16 + (piece % per) * 8, row = r0 + r_in;
        off = static_cast<uint32_t>(min(row, g.m - 1 - m0)) * static_cast<uint32_t>(g.lda * 2) + chunk(row);
        dst = lds0 + r0 * 128;
    };
    auto set_b = [&](int h, int i) {
        const int piece = (wave + i * NW) % T::GB, w = piece / (HB * 2), p0 = (piece % (HB * 2)) * 8;
        const int r0 = w * T::WN + h * HB * 16 + p0, rh = p0 + r_in;  // first LDS row; row in the half
        int a0, a1;  // rh = 16 j + 4 grp + e
        lane_cols<EPI, T>(g, n0, w, (rh >> 2) & 3, a0, a1);
        const int wrow = (h ? a1 - c01 : a0 - c00) + 4 * (rh >> 4) + (rh & 3);
        oB[h][i] = static_cast<uint32_t>(wrow) * static_cast<uint32_t>(g.k * 2) + chunk(r0 + r_in);
        dB[h][i] = lds0 + 2 * ABUF + r0 * 128;
    };
#pragma unroll
    for (int i = 0; i < LA0; ++i) set_a(HA0, 0, T::GA0, i, oA0[i], dA0[i]);
#pragma unroll
    for (int i = 0; i < LA1; ++i) set_a(HA1, HA0, T::GA1, i, oA1[i], dA1[i]);
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        set_b(0, i);
        set_b(1, i);
    }
    auto ldA0 = [&](int x, int t, int par) { load_lds16(Ab + static_cast<size_t>(t) * 128, oA0[x], dA0[x] + par * ABUF); };
    auto ldA1 = [&](int x, int t, int par) { load_lds16(Ab + static_cast<size_t>(t) * 128, oA1[x], dA1[x] + par * ABUF); };
    auto ldB = [&](int h, int x, int t, int par) {
        load_lds16(Wb[h] + static_cast<size_t>(t) * 128, oB[h][x], dB[h][x] + par * BBUF);
    };

    // LDS reads: slice s (32 of the step's 64 k), chunk 4 s + lane / 16 of row lane % 16
    const char* aF[2];
    const char* bF[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int r = lane & 15, at = ((4 * s + (lane >> 4)) ^ ((r >> 1) & 7)) << 4;
        aF[s] = smem + (wm * T::WM + r) * 128 + at;
        bF[s] = smem + 2 * ABUF + (wn * T::WN + r) * 128 + at;
    }
    bf16x8 fa0[HA0][2], fa1[HA1][2], fb[2][HB][2];
    f32x4 acc[HA][2 * HB];
#pragma unroll
    for (int i = 0; i < HA; ++i)
#pragma unroll
        for (int j = 0; j < 2 * HB; ++j) acc[i][j] = f32x4{};
    auto rA0 = [&](int x, int par) {
        fa0[x % HA0][x / HA0] = *reinterpret_cast<const bf16x8*>(aF[x / HA0] + par * ABUF + (x % HA0) * 2048);
    };
    auto rA1 = [&](int x, int par) {
        fa1[x % HA1][x / HA1] = *reinterpret_cast<const bf16x8*>(aF[x / HA1] + par * ABUF + (HA0 + x % HA1) * 2048);
    };
    auto rB = [&](auto h_c, int x, int par) {
        constexpr int h = decltype(h_c)::value;
        fb[h][x % HB][x / HB] = *reinterpret_cast<const bf16x8*>(bF[x / HB] + par * BBUF + (h * HB + x % HB) * 2048);
    };
    // MFMA x of quadrant (A half, B half), slice by slice
    auto mma = [&](auto ah_c, auto bh_c, int x) {
        constexpr int ah = decltype(ah_c)::value, bh = decltype(bh_c)::value, per = (ah ? HA1 : HA0) * HB;
        const int s = x / per, i = (x % per) / HB, j = x % HB;
        if constexpr (ah) acc[HA0 + i][bh * HB + j] = mfma16(fb[bh][j][s], fa1[i][s], acc[HA0 + i][bh * HB + j]);
        else acc[i][bh * HB + j] = mfma16(fb[bh][j][s], fa0[i][s], acc[i][bh * HB + j]);
    };
    // The MFMAs of a quadrant with NR LDS reads and NL loads spread between them.
    auto quadrant = [&](auto ah, auto bh, auto nr_c, auto nl_c, auto rd, auto ld) {
        constexpr int NM = (decltype(ah)::value ? HA1 : HA0) * HB * 2, NR = decltype(nr_c)::value, NL = decltype(nl_c)::value;
#pragma unroll
        for (int x = 0; x < NM; ++x) {
            constexpr int MAX = 16;
#pragma unroll
            for (int r = 0; r < MAX; ++r)
                if (r < NR && r >= (NR * x + NM - 1) / NM && r < (NR * (x + 1) + NM - 1) / NM) rd(r);
            mma(ah, bh, x);
#pragma unroll
            for (int l = 0; l < MAX; ++l)
                if (l < NL && l >= (NL * x + NM - 1) / NM && l < (NL * (x + 1) + NM - 1) / NM) ld(l);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // End of a phase: at most NLDS of this wave's LDS reads (those of this phase)
    // and NV of its loads (those younger than the half read next) are left.
    auto phase_end = [&](auto nv_c, auto nlds_c) {
        wait_lgkmcnt<decltype(nlds_c)::value>();
        wait_vmcnt<decltype(nv_c)::value>();
        barrier_only();
    };
    // One k step of parity PAR (its buffers, and the B half that comes first).
    // MODE 0: loads of step t + 2 are issued; 1: the step before the last; 2: the last.
    auto step = [&](auto par_c, auto mode_c, int t) {
        constexpr int PAR = decltype(par_c)::value, MODE = decltype(mode_c)::value;
        constexpr bool L = MODE == 0, R = MODE != 2;
        using F = std::integral_constant<int, PAR>;
        using S = std::integral_constant<int, 1 - PAR>;
        quadrant(I0{}, F{}, std::integral_constant<int, RB>{}, std::integral_constant<int, L ? LA0 : 0>{},
                 [&](int x) { rB(S{}, x, PAR); }, [&](int x) { ldA0(x, t + 2, PAR); });
        phase_end(std::integral_constant<int, L ? LALL + LA0 : R ? LALL : 0>{}, std::integral_constant<int, RB>{});
        quadrant(I0{}, S{}, std::integral_constant<int, RA1>{}, std::integral_constant<int, L ? LB : 0>{},
                 [&](int x) { rA1(x, PAR); }, [&](int x) { ldB(PAR, x, t + 2, PAR); });
        phase_end(std::integral_constant<int, L ? LALL + LB : R ? LALL - LA0 : 0>{}, std::integral_constant<int, RA1>{});
        quadrant(I1{}, S{}, std::integral_constant<int, R ? RA0 : 0>{}, std::integral_constant<int, L ? LB : 0>{},
                 [&](int x) { rA0(x, 1 - PAR); }, [&](int x) { ldB(1 - PAR, x, t + 2, PAR); });
        if (R) phase_end(std::integral_constant<int, L ? LALL + LB : LB + LA1>{}, std::integral_constant<int, RA0>{});
        quadrant(I1{}, F{}, std::integral_constant<int, R ? RB : 0>{}, std::integral_constant<int, L ? LA1 : 0>{},
                 [&](int x) { rB(S{}, x, 1 - PAR); }, [&](int x) { ldA1(x, t + 2, PAR); });
        if (R) phase_end(std::integral_constant<int, L ? LALL + LA1 : LA1>{}, std::integral_constant<int, RB>{});
    };
    // Loads of the first two steps, in the order the phases read them; the
    // first halves of step 0 are read here.  (A range of one step loads it twice.)
    auto prologue = [&](auto p_c) {
        constexpr int P = decltype(p_c)::value;
        auto whole = [&](int t, int par) {
#pragma unroll
            for (int x = 0; x < LA0; ++x) ldA0(x, t, par);
#pragma unroll
            for (int x = 0; x < LB; ++x) ldB(par, x, t, par);
#pragma unroll
            for (int x = 0; x < LB; ++x) ldB(1 - par, x, t, par);
#pragma unroll
            for (int x = 0; x < LA1; ++x) ldA1(x, t, par);
        };
        whole(0, P);
        whole(min(1, nk - 1), 1 - P);
        wait_vmcnt<LALL + LA1>();
        barrier_only();
#pragma unroll
        for (int x = 0; x < RA0; ++x) rA0(x, P);
#pragma unroll
        for (int x = 0; x < RB; ++x) rB(std::integral_constant<int, P>{}, x, P);
        wait_lgkmcnt<0>();
        barrier_only();
    };
    // The last step has parity 1.
    int t = 0;
    if (nk & 1) {
        prologue(I1{});
        if (nk > 1) {
            step(I1{}, I0{}, 0);
            t = 1;
        }
    } else {
        prologue(I0{});
    }
    if (nk > 1) {
        for (; t + 2 < nk; t += 2) {
            step(I0{}, I0{}, t);
            step(I1{}, I0{}, t + 1);
        }
        step(I0{}, I1{}, t);
    }
    step(I1{}, I2{}, nk - 1);
    tile_store<T, EPI, SPLIT>(g, m0, n0, wm, wn, lane,
                              SPLIT ? partial + static_cast<size_t>(blockIdx.y) * g.m * g.n : nullptr, acc);
}

// Sum split-K partials [splits][m][n] (W row order) and apply the epilogue:
// four outputs (or pairs) per thread.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs g, const float* __restrict__ part, int splits) {
    constexpr bool PAIR = EPI == EPI_QKV || EPI == EPI_SWIGLU;
    const size_t slab = static_cast<size_t>(g.m) * g.n;
    const size_t idx = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
    const int per_row = (PAIR ? g.n / 2 : g.n) / 4;
    if (idx >= static_cast<size_t>(g.m) * per_row) return;
    const int row = static_cast<int>(idx / per_row), c = static_cast<int>(idx % per_row) * 4;
    const int half = g.hd >> 1;
    int c0 = c, c1 = 0;  // W rows of the four outputs and of their partners
    if (EPI == EPI_SWIGLU) c1 = c + (g.n >> 1);
    if (EPI == EPI_QKV) {
        c0 = (c / half) * g.hd + c % half;
        c1 = c0 + half;
    }
    const float* p = part + static_cast<size_t>(row) * g.n;
    f32x4 a = {}, b = {};
    for (int z = 0; z < splits; ++z) {
        a += *reinterpret_cast<const f32x4*>(p + z * slab + c0);
        if (PAIR) b += *reinterpret_cast<const f32x4*>(p + z * slab + c1);
    }
    if constexpr (EPI == EPI_QKV) {
#pragma unroll
        for (int e = 0; e < 4; ++e) qkv_store(g, row, c / half, c % half + e, a[e], b[e]);
        return;
    }
    const size_t o = static_cast<size_t>(row) * g.ldo + c;
    if constexpr (EPI == EPI_SWIGLU) {
        const bf16 v[4] = {f2bf(silu(a[0]) * b[0]), f2bf(silu(a[1]) * b[1]), f2bf(silu(a[2]) * b[2]),
                           f2bf(silu(a[3]) * b[3])};
        store_bf16<4>(static_cast<bf16*>(g.out) + o, v);
    } else if constexpr (EPI == EPI_RESID_F32OUT) {
        const bf16x4 r = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(g.resid) + o);
        *reinterpret_cast<f32x4*>(static_cast<float*>(g.out) + o) = a + f32x4{bf2f(r[0]), bf2f(r[1]), bf2f(r[2]), bf2f(r[3])};
    } else if constexpr (EPI == EPI_RESID_F32IN) {
        a += *reinterpret_cast<const f32x4*>(static_cast<const float*>(g.resid) + o);
        const bf16 v[4] = {f2bf(a[0]), f2bf(a[1]), f2bf(a[2]), f2bf(a[3])};
        store_bf16<4>(static_cast<bf16*>(g.out) + o, v);
    }
}

// W row feeding B column c (c = n0 + tile row).
template <int EPI>
__device__ __forceinline__ int w_row(const GemmArgs& g, int c) {
    if (EPI == EPI_SWIGLU) {
        const int sub = c >> 5, f = g.n >> 1;
        const int col = (sub >> 1) * 32 + (c & 31);
        return (sub & 1) ? f + col : col;
    }
    if (EPI == EPI_QKV) {
        const int cw = c % g.hd;
        return c - cw + qkv_dim(cw, g.hd);
    }
    return c;
}

// ---------------------------------------------------------------------------
// Weight-streaming gate/up GEMM for up to 8 rows, with the RMSNorm before it
// folded in.
//
// Bound by the weights' way from HBM: a CU draws about 23 KB/us, so all 256
// have to draw evenly and without a pause.  A work-group of eight waves takes
// a run of units of 16 W rows (eight gate rows and their up rows) one after the
// other, each wave an eighth of k; its loads run R slices of 32 k ahead (1 KB
// each) across unit boundaries, so the stream never drains.  The wave's
// activations for all rows stay in registers (they are the same for every
// unit); a unit's eight partial sums meet in one of two LDS buffers, and the
// waves take turns to add them and store, while the others stream on.
//
// g.a holds the rows before the RMSNorm in fp32, and each work-group
// normalises them itself while its first weights are on their way: the same
// arithmetic as the RMSNorm kernel, whose launch (4 us) is saved.  Every
// work-group reads all rows, which is what limits it to few of them.
//
// 8B layer, norm included, against the RMSNorm kernel and a weight-streaming
// kernel of 448 work-groups: 50.1 -> 46 us at 1 row (235 MB: 5.1 TB/s), 52.9 ->
// 50 at 8; at 16 rows 58 against 49 for RMSNorm and the tile kernel.  The same
// for the qkv projection lost at every row count (19.5 against 18.9 us at 1 row,
// 24 against 21 at 8): two units a CU do not pay for the rows' read.  Rows past
// 6144 do not fit the registers in fp32 and are read twice.
// ---------------------------------------------------------------------------
constexpr int kStreamMaxRows = 8;
// slices in flight per wave, a divisor of the slices of a unit (14 against 7 of 14
// and 28: 2-3% of a layer; longer ones than these gained nothing)
constexpr int stream_ring(int ns) {
    for (int r : {8, 10, 9, 14, 11, 13, 6})
        if (ns % r == 0) return r;
    return ns;
}

// A wave takes NS slices of 32 k, NS even, from 4 to 32: k = 256 NS, or with
// TAIL any k of at most that and more than 256 (NS - 2), whose last one or two
// slices are missing from some waves: those read another slice in their place
// and multiply zeros.
template <int NS, bool TAIL>
__global__ __launch_bounds__(512, 2) void stream_kernel(GemmArgs g, NormArgs norm, int units, int per_wg) {
    constexpr int R = stream_ring(NS);
    static_assert(NS % R == 0, "a unit is whole turns of the ring");
    __shared__ f32x4 red[2][8][64];
    __shared__ float ssq[8][16];
    const int lane = threadIdx.x & 63, ks = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int j = lane & 15, grp = lane >> 4;
    const int u0 = blockIdx.x * per_wg, u1 = min(u0 + per_wg, units);
    const int slices = g.k / 32, own = TAIL ? slices / 8 + (ks < slices % 8) : NS;
    const int kbeg = (TAIL ? ks * (slices / 8) + min(ks, slices % 8) : ks * NS) * 32 + 8 * grp;
    auto off = [&](int s) { return 32 * (TAIL && s >= NS - 2 ? min(s, own - 1) : s); };
    auto missing = [&](int s) { return TAIL && s >= NS - 2 && s >= own; };
    // W row of this lane in unit u: rows 0 .. 7 of the MFMA take gate rows 8 u .. 8 u + 7, rows 8 .. 15 their up rows
    auto wptr = [&](int u) {
        const int row = 8 * u + (j & 7) + (j >> 3) * (g.n >> 1);
        return static_cast<const bf16*>(g.w) + static_cast<size_t>(row) * g.k + kbeg;
    };
    bf16x8 wf[R];
    const bf16* wp = wptr(u0);
#pragma unroll
    for (int s = 0; s < R; ++s) wf[s] = *reinterpret_cast<const bf16x8*>(wp + off(s));

    // activations: row j (rows past m repeat row m - 1; their results are never
    // stored), read once and normalised in registers
    bf16x8 af[NS];
    {
        // rows of up to 6144 stay in registers between the sum of squares and
        // the scaling; longer ones are read twice
        constexpr bool KEEP = NS <= 24;
        const float* src = static_cast<const float*>(g.a) + static_cast<size_t>(min(j, g.m - 1)) * g.lda + kbeg;
        auto half = [&](int s, int h) { return *reinterpret_cast<const f32x4*>(src + off(s) + 4 * h); };
        f32x4 raw[KEEP ? NS : 1][2];
        float ss = 0.f;
        if constexpr (KEEP) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                raw[s][0] = half(s, 0);
                raw[s][1] = half(s, 1);
            }
        }
        auto x = [&](int s, int h) {
            if constexpr (KEEP) return raw[s][h];
            else return half(s, h);
        };
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x4 v = x(s, h);
                if (missing(s)) v = f32x4{};
#pragma unroll
                for (int e = 0; e < 4; ++e) ss += v[e] * v[e];
            }
            if (!KEEP && s % 8 == 7) __builtin_amdgcn_sched_barrier(0);  // else all reads are issued at once, and spill
        }
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (grp == 0) ssq[ks][j] = ss;
        wait_lgkmcnt<0>();
        barrier_only();
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) tot += ssq[w][j];
        const float inv = 1.0f / sqrtf(tot / static_cast<float>(g.k) + norm.eps);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const bf16x8 gain = *reinterpret_cast<const bf16x8*>(static_cast<const bf16*>(norm.gain) + kbeg + off(s));
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 v = x(s, h);
#pragma unroll
                for (int e = 0; e < 4; ++e) af[s][4 * h + e] = f2bf(v[e] * inv * bf2f(gain[4 * h + e]));
            }
            if (missing(s)) af[s] = bf16x8{};
            if (!KEEP && s % 8 == 7) __builtin_amdgcn_sched_barrier(0);
        }
    }

    // One unit; with MORE, the loads of the next one follow on.
    auto unit = [&](int u, auto more_c) {
        constexpr bool MORE = decltype(more_c)::value;
        const bf16* wn = MORE ? wptr(u + 1) : nullptr;
        f32x4 acc = {};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            // both factors of a missing slice are zero: the other slice's weights may not be finite
            acc = mfma16(missing(s) ? bf16x8{} : wf[s % R], af[s], acc);
            if (s + R < NS) wf[s % R] = *reinterpret_cast<const bf16x8*>(wp + off(s + R));
            else if (MORE) wf[s % R] = *reinterpret_cast<const bf16x8*>(wn + off(s + R - NS));
        }
        wp = wn;
        const int b = (u - u0) & 1;
        red[b][ks][lane] = acc;
        // no wait for the loads in flight: only the sums have to be there
        wait_lgkmcnt<0>();
        barrier_only();
        if (((u - u0) & 7) != ks) return;
        f32x4 v = red[b][0][lane];
#pragma unroll
        for (int w = 1; w < 8; ++w) v += red[b][w][lane];
        // lane groups 0, 1 hold the gates of outputs 8 u + 4 grp + e of row j, the lanes 32 on their ups
        f32x4 up;
#pragma unroll
        for (int e = 0; e < 4; ++e) up[e] = __shfl_xor(v[e], 32, 64);
        if (grp >= 2 || j >= g.m) return;
        const bf16 o[4] = {f2bf(silu(v[0]) * up[0]), f2bf(silu(v[1]) * up[1]), f2bf(silu(v[2]) * up[2]),
                           f2bf(silu(v[3]) * up[3])};
        store_bf16<4>(static_cast<bf16*>(g.out) + static_cast<size_t>(j) * g.ldo + 8 * u + 4 * grp, o);
    };
    for (int u = u0; u + 1 < u1; ++u) unit(u, std::integral_constant<bool, true>{});
    unit(u1 - 1, std::integral_constant<bool, false>{});
}

// Narrow GEMM for m <= 32 rows (decode-sized batches): a work-group of KS
// waves owns 16 output columns (CG == 1) or a RoPE / SwiGLU pair of 16-column
// groups 32 apart (CG == 2) and all m rows; each wave takes K / KS of the k
// range, so every weight byte is read once, and the waves' sums are added in
// LDS before the fused epilogue: no split of k across work-groups, no second
// kernel.  16 x 16 x 32 MFMAs with the weights as the A operand: a 64-lane
// operand load reads 64 contiguous bytes of each of 16 weight rows (16 cache
// lines, against 32 for a 32-row operand).  Four k slices of 32 are kept in
// flight per wave in a ring of registers.
constexpr int kNarrowMaxWaves = 8;
template <int T, int CG, int EPI>
__global__ __launch_bounds__(64 * kNarrowMaxWaves) void narrow_kernel(GemmArgs g, int ks_count) {
    constexpr int R = 4;  // slices in flight
    __shared__ f32x4 red[kNarrowMaxWaves][CG * T][64];
    const int lane = threadIdx.x & 63, ks = threadIdx.x >> 6;
    const int j = lane & 15, grp = lane >> 4;
    // first column of each group: CG == 2 takes 16 columns of a 64-column
    // tile and their partners 32 further on
    int col0[CG];
    if constexpr (CG == 2) {
        const int tile64 = (blockIdx.x >> 1) * 64, half = (blockIdx.x & 1) * 16;
        col0[0] = tile64 + half;
        col0[1] = tile64 + 32 + half;
    } else {
        col0[0] = blockIdx.x * 16;
    }
    const int k_wave = g.k / ks_count;
    const int kbeg = ks * k_wave + 8 * grp;
    const int nslice = k_wave / 32;
    const bf16* W = static_cast<const bf16*>(g.w);
    const bf16* A = static_cast<const bf16*>(g.a);
    const bf16* wp[CG];
#pragma unroll
    for (int c = 0; c < CG; ++c) wp[c] = W + static_cast<size_t>(w_row<EPI>(g, col0[c] + j)) * g.k + kbeg;
    const bf16* ap[T];
#pragma unroll
    for (int t = 0; t < T; ++t)  // rows past m read row m - 1; their results are never stored
        ap[t] = A + static_cast<size_t>(min(t * 16 + j, g.m - 1)) * g.lda + kbeg;

    bf16x8 wf[R][CG], af[R][T];
    auto load = [&](int sl, int b) {
#pragma unroll
        for (int c = 0; c < CG; ++c) wf[b][c] = *reinterpret_cast<const bf16x8*>(wp[c] + 32 * sl);
#pragma unroll
        for (int t = 0; t < T; ++t) af[b][t] = *reinterpret_cast<const bf16x8*>(ap[t] + 32 * sl);
    };
    f32x4 acc[CG][T];
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int t = 0; t < T; ++t) acc[c][t] = f32x4{};
#pragma unroll
    for (int b = 0; b < R; ++b)
        if (b < nslice) load(b, b);
    for (int s0 = 0; s0 < nslice; s0 += R) {
#pragma unroll
        for (int b = 0; b < R; ++b) {
            if (s0 + b < nslice) {
#pragma unroll
                for (int c = 0; c < CG; ++c)
#pragma unroll
                    for (int t = 0; t < T; ++t) acc[c][t] = mfma16(wf[b][c], af[b][t], acc[c][t]);
                if (s0 + b + R < nslice) load(s0 + b + R, b);
            }
        }
    }

    // Sum over the waves; wave t then stores token group t.
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int t = 0; t < T; ++t) red[ks][c * T + t][lane] = acc[c][t];
    __syncthreads();
    if (ks >= T) return;
    const int t = ks;
    f32x4 v[CG];
#pragma unroll
    for (int c = 0; c < CG; ++c) {
        v[c] = red[0][c * T + t][lane];
        for (int w = 1; w < ks_count; ++w) v[c] += red[w][c * T + t][lane];
    }
    const int row = t * 16 + j;
    if (row >= g.m) return;
    // element e of a lane: column col0[c] + 4 grp + e of row `row`
    if constexpr (EPI == EPI_QKV) {
        const int tile64 = col0[0] - (blockIdx.x & 1) * 16;
        const int hg = tile64 / g.hd, d0 = ((tile64 % g.hd) / 64) * 32 + (col0[0] - tile64) + 4 * grp;
#pragma unroll
        for (int e = 0; e < 4; ++e) qkv_store(g, row, hg, d0 + e, v[0][e], v[CG - 1][e]);
    } else if constexpr (EPI == EPI_SWIGLU) {
        const int tile64 = col0[0] - (blockIdx.x & 1) * 16;
        bf16* out = static_cast<bf16*>(g.out) + static_cast<size_t>(row) * g.ldo + (tile64 >> 1) +
                    (col0[0] - tile64) + 4 * grp;
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = f2bf(silu(v[0][e]) * v[CG - 1][e]);
        *reinterpret_cast<bf16x4*>(out) = o;
    } else {
        const size_t o = static_cast<size_t>(row) * g.ldo + col0[0] + 4 * grp;
        if constexpr (EPI == EPI_RESID_F32OUT) {
            const bf16x4 rb = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(g.resid) + o);
            *reinterpret_cast<f32x4*>(static_cast<float*>(g.out) + o) =
                v[0] + f32x4{bf2f(rb[0]), bf2f(rb[1]), bf2f(rb[2]), bf2f(rb[3])};
        } else {
            const f32x4 r = *reinterpret_cast<const f32x4*>(static_cast<const float*>(g.resid) + o) + v[0];
            *reinterpret_cast<bf16x4*>(static_cast<bf16*>(g.out) + o) = bf16x4{f2bf(r[0]), f2bf(r[1]), f2bf(r[2]), f2bf(r[3])};
        }
    }
}

// Tile configurations: rows, columns, work-groups that share a CU, and the
// planner's time per 64-deep k step of one work-group (us).
struct TileCfg {
    int bm, bn, per_cu;
    float step_us;
};
constexpr TileCfg kCfgs[] = {{256, 256, 1, 1.253f}, {224, 256, 1, 1.108f}, {192, 256, 1, 0.990f}, {160, 256, 1, 0.874f},
                             {256, 128, 1, 0.715f}, {192, 128, 1, 0.628f}, {160, 128, 2, 0.519f}, {128, 128, 2, 0.460f},
                             {96, 128, 2, 0.435f},  {64, 128, 2, 0.396f}};
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);
constexpr int kCus = 256;
constexpr int kMaxSplits = 8;

template <class T, int EPI>
void launch_tile(const GemmArgs& g, const GemmPlan& p, float* part, hipStream_t s) {
    const dim3 grid(((g.m + T::BM - 1) / T::BM) * (g.n / T::BN), p.splits);
    if (p.splits == 1) {
        tile_kernel<T, EPI, false><<<grid, T::THREADS, 0, s>>>(g, nullptr, g.k);
        return;
    }
    tile_kernel<T, EPI, true><<<grid, T::THREADS, 0, s>>>(g, part, g.k / p.splits);
    const size_t work = static_cast<size_t>(g.m) * (EPI == EPI_QKV || EPI == EPI_SWIGLU ? g.n / 8 : g.n / 4);
    splitk_reduce_kernel<EPI><<<static_cast<unsigned>((work + 255) / 256), 256, 0, s>>>(g, part, p.splits);
}

template <class T>
void launch_cfg(const GemmArgs& g, const GemmPlan& p, void* partial, hipStream_t s) {
    float* part = static_cast<float*>(partial);
    switch (g.epi) {
        case EPI_RESID_F32OUT: launch_tile<T, EPI_RESID_F32OUT>(g, p, part, s); break;
        case EPI_RESID_F32IN: launch_tile<T, EPI_RESID_F32IN>(g, p, part, s); break;
        case EPI_SWIGLU: launch_tile<T, EPI_SWIGLU>(g, p, part, s); break;
        default: launch_tile<T, EPI_QKV>(g, p, part, s); break;
    }
}

template <int NS>
void launch_stream_ns(const GemmArgs& g, const NormArgs& norm, hipStream_t s) {
    const int units = g.n / 16, per = (units + kCus - 1) / kCus, wgs = (units + per - 1) / per;
    if (g.k == 256 * NS) stream_kernel<NS, false><<<wgs, 512, 0, s>>>(g, norm, units, per);
    else stream_kernel<NS, true><<<wgs, 512, 0, s>>>(g, norm, units, per);
}

void launch_stream(const GemmArgs& g, const NormArgs& norm, hipStream_t s) {
    switch ((g.k + 511) / 512) {  // stream_shape_ok
        case 2: launch_stream_ns<4>(g, norm, s); break;
        case 3: launch_stream_ns<6>(g, norm, s); break;
        case 4: launch_stream_ns<8>(g, norm, s); break;
        case 5: launch_stream_ns<10>(g, norm, s); break;
        case 6: launch_stream_ns<12>(g, norm, s); break;
        case 7: launch_stream_ns<14>(g, norm, s); break;
        case 8: launch_stream_ns<16>(g, norm, s); break;
        case 9: launch_stream_ns<18>(g, norm, s); break;
        case 10: launch_stream_ns<20>(g, norm, s); break;
        case 11: launch_stream_ns<22>(g, norm, s); break;
        case 12: launch_stream_ns<24>(g, norm, s); break;
        case 13: launch_stream_ns<26>(g, norm, s); break;
        case 14: launch_stream_ns<28>(g, norm, s); break;
        case 15: launch_stream_ns<30>(g, norm, s); break;
        default: launch_stream_ns<32>(g, norm, s); break;
    }
}

template <int T, int CG, int EPI>
void launch_narrow_epi(const GemmArgs& g, const GemmPlan& p, hipStream_t s) {
    narrow_kernel<T, CG, EPI><<<g.n / (16 * CG), 64 * p.ks, 0, s>>>(g, p.ks);
}

template <int T>
void launch_narrow(const GemmArgs& g, const GemmPlan& p, hipStream_t s) {
    switch (g.epi) {
        case EPI_RESID_F32OUT: launch_narrow_epi<T, 1, EPI_RESID_F32OUT>(g, p, s); break;
        case EPI_RESID_F32IN: launch_narrow_epi<T, 1, EPI_RESID_F32IN>(g, p, s); break;
        case EPI_SWIGLU: launch_narrow_epi<T, 2, EPI_SWIGLU>(g, p, s); break;
        default: launch_narrow_epi<T, 2, EPI_QKV>(g, p, s); break;
    }
}

// Predicted time (us) of a tile configuration with a k split: rounds of
// work-groups over the CUs, each a fixed cost (fill of the LDS buffers,
// epilogue, which grows with the tile) plus its k steps; where two work-groups
// share a CU, a round of both takes about twice as long as one alone.  Against
// that stands the time to stream the weights and to bring every tile's panels
// from L2 (smooth maximum; its rates are free parameters of the fit, above what
// a plain read reaches: 5.7-5.9 TB/s, 23 KB/us and CU); a split adds its
// reduction's launch and traffic.  Rows count in blocks of 32 (every tile's row
// granularity), so that row counts of one block share a plan.  The constants are
// a fit to 4200 timings (ten shapes, 16 to 4104 rows, all configurations,
// splits 1 to 8; activations in cache, weights cycled through 700 MB so that
// none are: a layer finds them so, and fitted to weights in the last-level cache
// the rule picked tiles 20-40% slower for the output and qkv projections at 288
// rows): median error below 1%, 90% within -11% and +13%; the configuration it
// picks is on average 0.8% slower than the fastest one measured, 18% at worst.
// `tiles`: of the configuration, `inv`: 1 / splits.  A configuration that cannot
// come below `limit` is not priced to the end: every iteration prices some 60.
float predict_us(const TileCfg& c, int tiles, int splits, float inv, int m32, int n, int k, float limit) {
    const int wgs = tiles * splits;
    const float nk = static_cast<float>(k / 64) * inv;
    const float fixed = 4.18f + 2.66f * (c.bm * c.bn) / 65536.f;
    const float one = fixed + nk * c.step_us, both = fixed + 1.91f * nk * c.step_us;
    const int full = c.per_cu == 2 ? wgs / (2 * kCus) : wgs / kCus, rem = wgs - full * kCus * c.per_cu;
    float t = full * (c.per_cu == 2 ? both : one);
    if (rem) t += c.per_cu == 2 && rem > kCus ? both : one;
    const float reduce = splits > 1 ? 2.18f + 8.f * splits * m32 * n / 4.68e6f : 0.f;
    if (t + reduce >= limit) return limit;
    const float rate = std::min(6.73e6f, 32.0e3f * std::min(wgs, kCus));
    const float mem = 2.f * n * k / rate + 0.2f + 2.f * wgs * (c.bm + c.bn) * (static_cast<float>(k) * inv) / 40.59e6f;
    if (mem + reduce >= limit) return limit;
    const float t2 = t * t, m2 = mem * mem;
    return 0.91f + std::sqrt(std::sqrt(t2 * t2 + m2 * m2)) + reduce;
}

// Whether a gate/up projection of up to 8 rows streams its weights.  Multiples
// of 1024 from 2048 to 6144 do at any width.  Other k do where the tile kernel
// stands badly: below 2048, and at widths whose 128-column tiles fill half of its
// second round of work-groups or less; towards that end rows that have to be read
// twice stay below 5.  Norm and gate/up stages, tile kernel / streamed, us at 1
// and 8 rows: k 3584, n 37888: 71 / 59, 71 / 63; k 6656, n 37888: 125 / 101, 126
// / 111; k 7168, n 40960: 134 / 117, 134 / 126; k 1024, n 16384: 20 / 17, 20 / 17;
// k 6912, n 49152, the whole layer at 1 and 8 rows: 249 / 245, 277 / 282; and
// outside, where it can lose: k 7168, n 28672: 79 / 91, 79 / 99.
bool stream_shape_ok(int m, int n, int k) {
    if (m > kStreamMaxRows || k % 64 || k < 1024 || k > 8192) return false;
    if (k % 1024 == 0 && k >= 2048 && k <= 6144) return true;
    const int tiles = n / 128;
    if (2 * tiles > 3 * kCus || (8 * tiles > 11 * kCus && k > 6144 && m > 4)) return false;
    return k < 2048 || tiles > kCus;
}

}  // namespace

// Wide gate/up projections of up to 8 rows take the weight-streaming kernel with
// the norm folded in, where their shape suits it.
// The narrow kernel takes qkv- and down-like projections up to 8 rows and the
// output projection up to 24 (8B layer, against the tile kernel, us at 1 / 8 /
// 24 rows: output 8.4 / 9.2 / 12.4 against 11.6 / 12.1 / 12.4; down 21.6 /
// 25.8 at 1 / 8 rows against 25.5 / 26.0, 31.5 against 26.3 at 16; qkv 14.2 /
// 15.4 against 14.0 / 14.7 and no reduction launch), and all 32 rows it has
// where the tile kernel's few work-groups would need a split of k and its
// reduction (a layer at 25 / 32 rows, tile kernel against narrow: d_model 1024,
// FFN 4096: 59.6 / 59.4 against 54.6 / 56.4 us; d_model 3072, output only:
// 96.9 / 97.9 against 95.8 / 97.6).  Larger row counts, where each of its
// work-groups re-reads all activation rows, take the tile kernel with the
// configuration and split that predict_us ranks first.  n must be a multiple
// of 128 and k of 64; a split keeps at least 512 of k.
GemmPlan plan_gemm(int m, int n, int k, bool swiglu) {
    const bool wide = n >= 16384, qkv_like = n >= 6144 && !wide;
    if (swiglu && wide && stream_shape_ok(m, n, k)) return plan_with_cfg(kStreamCfg, 1, m, n, k);
    const int narrow_rows = qkv_like || k >= 8192 ? 8 : n <= 3072 && k >= 1024 ? 32 : 24;
    if (!wide && m <= narrow_rows) return plan_with_cfg(kNarrowCfg, 1, m, n, k);
    int cfg = kNumCfgs - 1, splits = 1;
    const int m32 = (m + 31) / 32 * 32;
    float best = HUGE_VALF;
    for (int c = 0; c < kNumCfgs; ++c) {
        if (n % kCfgs[c].bn) continue;
        const int tiles = ((m32 + kCfgs[c].bm - 1) / kCfgs[c].bm) * (n / kCfgs[c].bn);
        float inv = 1.f;
        for (int sp = 1; sp <= kMaxSplits && (sp == 1 || (k % (64 * sp) == 0 && k / sp >= 512)); sp *= 2, inv *= 0.5f) {
            const float t = predict_us(kCfgs[c], tiles, sp, inv, m32, n, k, best);
            if (t < best) {
                best = t;
                cfg = c;
                splits = sp;
            }
        }
    }
    return plan_with_cfg(cfg, splits, m, n, k);
}

GemmPlan plan_with_cfg(int cfg, int splits, int m, int n, int k) {
    GemmPlan p{};
    p.cfg = cfg;
    p.splits = 1;
    if (cfg == kNarrowCfg) {
        // waves per work-group: each takes a whole number of 32-wide k slices
        int ks = 8;
        while (ks > 1 && k % (32 * ks)) ks /= 2;
        p.ks = ks;
        p.bm = m <= 16 ? 16 : 32;
        p.bn = 16;
        return p;
    }
    if (cfg == kStreamCfg) {
        p.bm = kStreamMaxRows;
        p.bn = 16;
        return p;
    }
    p.bm = kCfgs[cfg].bm;
    p.bn = kCfgs[cfg].bn;
    p.splits = splits;
    p.partial_bytes = splits > 1 ? static_cast<size_t>(splits) * m * n * sizeof(float) : 0;
    return p;
}

bool gemm_plan_ok(const GemmPlan& p, int m, int n, int k, bool swiglu) {
    if (p.cfg == kNarrowCfg)  // paired epilogues need 64-column tiles
        return m <= 32 && n % 64 == 0 && p.ks >= 1 && p.ks <= kNarrowMaxWaves && k % (32 * p.ks) == 0;
    if (p.cfg == kStreamCfg) return swiglu && n % 16 == 0 && stream_shape_ok(m, n, k);
    return p.cfg >= 0 && p.cfg < kNumCfgs && n % p.bn == 0 && k % (p.splits * 64) == 0;
}

void launch_gemm(const GemmArgs& g, const GemmPlan& p, void* partial, size_t partial_bytes, hipStream_t s,
                 const NormArgs& norm) {
    if (g.m <= 0) return;
    const size_t row_bytes = static_cast<size_t>(p.splits) * g.n * sizeof(float);
    if (p.splits > 1 && g.m * row_bytes > partial_bytes) {
        // whole tile rows to a block where one fits; no result depends on the
        // rows beside it
        int rows = static_cast<int>(partial_bytes / row_bytes);
        if (rows > p.bm) rows -= rows % p.bm;
        const bool out_f32 = g.epi == EPI_RESID_F32OUT, resid_f32 = g.epi == EPI_RESID_F32IN;
        for (int r = 0; r < g.m; r += rows) {
            GemmArgs b = g;
            const size_t o = static_cast<size_t>(r) * g.ldo;
            b.m = std::min(rows, g.m - r);
            b.a = static_cast<const char*>(g.a) + static_cast<size_t>(r) * g.lda * 2;
            b.out = static_cast<char*>(g.out) + o * (out_f32 ? 4 : 2);
            if (g.resid) b.resid = static_cast<const char*>(g.resid) + o * (resid_f32 ? 4 : 2);
            if (g.epi == EPI_QKV) {
                b.rope_cs = g.rope_cs + static_cast<size_t>(r) * (g.hd / 2);
                b.slot = g.slot + r;
            }
            launch_gemm(b, p, partial, partial_bytes, s);
        }
        return;
    }
    if (p.cfg == kNarrowCfg) {  // plans cover m <= 32
        if (g.m <= 16) launch_narrow<1>(g, p, s);
        else launch_narrow<2>(g, p, s);
        return;
    }
    if (p.cfg == kStreamCfg) {
        launch_stream(g, norm, s);
        return;
    }
    switch (p.cfg) {  // kCfgs order
        case 0: launch_cfg<Tile<256, 256, 2, 4>>(g, p, partial, s); break;
        case 1: launch_cfg<Tile<224, 256, 2, 4>>(g, p, partial, s); break;
        case 2: launch_cfg<Tile<192, 256, 2, 4>>(g, p, partial, s); break;
        case 3: launch_cfg<Tile<160, 256, 2, 4>>(g, p, partial, s); break;
        case 4: launch_cfg<Tile<256, 128, 4, 2>>(g, p, partial, s); break;
        case 5: launch_cfg<Tile<192, 128, 2, 4>>(g, p, partial, s); break;
        case 6: launch_cfg<Tile<160, 128, 2, 4>>(g, p, partial, s); break;
        case 7: launch_cfg<Tile<128, 128, 2, 4>>(g, p, partial, s); break;
        case 8: launch_cfg<Tile<96, 128, 2, 4>>(g, p, partial, s); break;
        default: launch_cfg<Tile<64, 128, 2, 4>>(g, p, partial, s); break;
    }
}

}  // namespace slw
