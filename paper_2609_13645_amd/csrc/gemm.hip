// bf16 GEMM on gfx950 MFMA, fp32 accumulation.
//
// Every projection of the layer is one of three products (App. C: the
// backward of each GEMM is one data-gradient and one weight-gradient
// product): y = x W^T (both operands K-contiguous), dX = dY W (W is
// N-contiguous) and dW += dY^T X (both operands M/N-contiguous, reduction
// over tokens). Three pipelines share tile order, operand layouts and epilogue
// stores:
//
//  * ring_kernel (every layout; the large tiles): v_mfma_f32_16x16x32_bf16
//    over a ring of four 32-deep LDS stages, one MFMA k-step per stage. The
//    barrier that publishes stage s + 1 sits two MFMAs into stage s; after it
//    the fragment reads of stage s + 1 and the DMA of stage s + 4 (into the
//    slot stage s has just released) are spread evenly over the stage's
//    MFMAs, so neither the LDS nor the texture unit sees a burst. Fragment
//    reads are inline asm with explicit lgkmcnt waits: the compiler cannot
//    tell the transposing reads apart from the DMA writes and would otherwise
//    wait for every outstanding DMA before each of them. The 16x16x32 shape
//    does the work of 32x32x16 at the same rate per cycle with less power,
//    which keeps the clock higher under load.
//  * wave_kernel (every layout; 64 x 64 tiles, for products of few tiles): the
//    waves of a workgroup split the reduction, each with a ring of its own.
//  * gemm_kernel (K-contiguous 128 x 128): v_mfma_f32_32x32x16
//    over a block tile BM x BN x 64 double-buffered in LDS, one barrier per
//    k-step placed before the step's last 16-deep slice; the barrier also
//    frees the current buffer, which is refilled at once with the step after
//    next.
//  * Tiles are filled by buffer_load ... lds (global to LDS without
//    registers); out-of-range chunks read as zeros through the buffer
//    descriptor's range check, so ragged edges need no branches.
//  * A K-contiguous operand tile keeps 128-byte rows (eight 16-byte chunks,
//    chunk c of row r at c ^ ((r ^ (r >> 3)) & 7)) in gemm_kernel and 64-byte
//    rows (chunk c of row r at c ^ ((r >> 1) & 3)) in a ring stage; either
//    way the eight lanes a 16-byte read serves per cycle cover a 128-byte
//    bank window once (no bank conflicts). Each MFMA operand is one 16-byte
//    LDS read. An operand contiguous along M / N is
//    stored as it lies in HBM (chunks XOR-swizzled per k-row) and read with
//    gfx950's ds_read_b64_tr_b16 transpose reads, so dgrad and wgrad need no
//    transpose pass.
//  * The MFMA computes D = Btile * Atile^T, i.e. C transposed, so each lane's
//    four consecutive accumulator rows are four consecutive n of one row m of
//    C: the epilogue writes 16-byte fp32 vectors, and in the ring kernel
//    lanes l and l ^ 16 swap halves so that each writes eight consecutive
//    bf16 (one 16-byte store). The AdamW epilogues of the grouped
//    weight gradients stage the fp32 tile through the free stage ring and
//    stream it by rows through the optimizer state (adam_tile).
//  * Workgroups are dispatched round-robin over the 8 XCDs; the tile order is
//    remapped so each XCD works on a contiguous, M-grouped band of tiles and
//    reuses operands in its own L2.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace forge {
namespace {

constexpr int BK = 64;
constexpr int CHUNKS = BK / 8;  // 16-byte chunks per LDS tile row
constexpr int GROUP_M = 8;
constexpr int NUM_XCD = 8;

__device__ __forceinline__ int wave_incl_scan_int(int v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(v, d, 64);
    if ((int)(threadIdx.x & 63) >= d) v += u;
  }
  return v;
}
__device__ __forceinline__ int wave_sum_int(int v) { return __shfl(wave_incl_scan_int(v), 63, 64); }

__device__ __forceinline__ int swz(int row, int c) {
  return row * CHUNKS + (c ^ ((row ^ (row >> 3)) & 7));
}

// ---- buffer resources ------------------------------------------------------
// Raw buffer loads return zero for an offset past num_records, so every
// out-of-range chunk (ragged M/N edge, K tail) is fetched as zeros without a
// branch: the address of a chunk that is out of range is set to kOOB.
constexpr uint32_t kOOB = 0x80000000u;
constexpr uint32_t kRecords = 0x7FFFFFF0u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)kRecords,
                                           0x00020000);
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// ---- K-contiguous source: global -> LDS directly (no register staging) ----
// Each wave-wide buffer_load_dwordx4 ... lds writes 1 KB of LDS: 8 tile rows
// of 128 bytes, lane l landing at byte 16*l. Lane l therefore fetches the
// logical chunk that the swizzle places at physical slot l % 8 of row l / 8.
template <int ROWS, int NW>
struct KcLoader {
  static constexpr int PER = ROWS / 8 / NW;
  static_assert(PER * 8 * NW == ROWS, "tile rows must split over waves");
  __device__ __forceinline__ void load(const bf16_t* __restrict__ src, long ld, int row0,
                                       int rows_lim, int k0, int K, uint4* lds, int wave,
                                       int lane) const {
    const __amdgpu_buffer_rsrc_t r = rsrc(src + (long)row0 * ld + k0);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int blk = i * NW + wave;
      const int row = blk * 8 + (lane >> 3);
      const int c = (lane & 7) ^ ((row ^ (row >> 3)) & 7);
      const bool ok = (row0 + row < rows_lim) && (k0 + c * 8 < K);
      const uint32_t off = ok ? (uint32_t)(((long)row * ld + c * 8) * 2) : kOOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)(lds + blk * 64), 16, off, 0, 0, 0);
    }
  }
};

// Fragment of rows base..base+31 (the lane's row is base + lane % 32) over
// k-slice kk: eight consecutive k starting at kk*16 + 8*(lane / 32).
__device__ __forceinline__ bf16x8_t frag(const uint4* tile, int base, int kk, int lane) {
  return __builtin_bit_cast(bf16x8_t, tile[swz(base + (lane & 31), kk * 2 + (lane >> 5))]);
}

// ---- epilogue: four consecutive n of row m ---------------------------------
// fp32 C (and the C it accumulates into) goes through nontemporal accesses: a
// round of 256 x 256 tiles writes about as much C per XCD as the XCD's L2
// holds, and ordinary stores would evict the operand rows that the next tiles
// read there. bf16 pieces of 8 bytes stay ordinary stores (streaming stores
// that small are slower than the eviction they avoid).
template <int EPI>
__device__ __forceinline__ void store4(const GemmArgs& p, int m, int n, const float* vin) {
  if (m >= p.M) return;
  const bool full = (n + 3 < p.N);
  const float v[4] = {vin[0] * p.alpha, vin[1] * p.alpha, vin[2] * p.alpha, vin[3] * p.alpha};
  if (EPI == kStoreBF16 || EPI == kResidBF16) {
    bf16_t* C = reinterpret_cast<bf16_t*>(p.C) + (long)m * p.ldc + n;
    float x[4] = {v[0], v[1], v[2], v[3]};
    if (EPI == kResidBF16) {
      const bf16_t* R = p.R + (long)m * p.ldr + n;
      if (full) {
        const uint2 r = *reinterpret_cast<const uint2*>(R);
        x[0] += lo_f(r.x); x[1] += hi_f(r.x); x[2] += lo_f(r.y); x[3] += hi_f(r.y);
      } else {
        for (int e = 0; e < 4; ++e)
          if (n + e < p.N) x[e] += bf2f(R[e]);
      }
    }
    if (full) {
      *reinterpret_cast<uint2*>(C) = make_uint2(pack2(x[0], x[1]), pack2(x[2], x[3]));
    } else {
      for (int e = 0; e < 4; ++e)
        if (n + e < p.N) C[e] = f2bf(x[e]);
    }
  } else {
    float* C = reinterpret_cast<float*>(p.C) + (long)m * p.ldc + n;
    if (full) {
      f32x4_t o = {v[0], v[1], v[2], v[3]};
      if (EPI == kAccF32) o += __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(C));
      __builtin_nontemporal_store(o, reinterpret_cast<f32x4_t*>(C));
    } else {
      for (int e = 0; e < 4; ++e)
        if (n + e < p.N) C[e] = (EPI == kAccF32 ? C[e] : 0.0f) + v[e];
    }
  }
}

// ---- epilogue of a 32x32 block: lane holds C[m][n..n+3] for 4 groups ------
template <int EPI, int FN, int FM>
__device__ __forceinline__ void store_tile(const GemmArgs& p, const f32x16_t (&acc)[FN][FM],
                                           int mw, int nw, int lane) {
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) {
      const int m = mw + j * 32 + (lane & 31);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n = nw + i * 32 + g * 8 + (lane >> 5) * 4;
        float v[4] = {acc[i][j][g * 4 + 0], acc[i][j][g * 4 + 1], acc[i][j][g * 4 + 2],
                      acc[i][j][g * 4 + 3]};
        store4<EPI>(p, m, n, v);
      }
    }
}

// Tile of this workgroup (tm, tn) and the group-adjusted arguments; false
// when the workgroup has no tile (M-grouped launches over-provision).
template <int BM, int BN, int EPI, int GROUP, int LA = kMC, int LB = kMC>
__device__ __forceinline__ bool tile_setup(GemmArgs& p, int& tm, int& tn) {
  if (GROUP == 0) {
    // ---- tile order: XCD-contiguous bands, GROUP_M rows of tiles per band ----
    const int tiles_m = (p.M + BM - 1) / BM;
    const int tiles_n = (p.N + BN - 1) / BN;
    const int nb = gridDim.x;
    const int bid = blockIdx.x;
    const int nb8 = nb - nb % NUM_XCD;
    const int pid = bid < nb8 ? (bid % NUM_XCD) * (nb8 / NUM_XCD) + bid / NUM_XCD : bid;
    const int in_group = GROUP_M * tiles_n;
    const int first_m = (pid / in_group) * GROUP_M;
    const int gsize = min(tiles_m - first_m, GROUP_M);
    tm = first_m + (pid % in_group) % gsize;
    tn = (pid % in_group) / gsize;
  } else if (GROUP == 1) {
    // M-grouped. The grid is an upper bound (host does not know the group
    // sizes); the real tiles are counted from the device offsets and dealt
    // to the 8 XCDs (workgroup b runs on XCD b % 8) as balanced contiguous
    // ranges. Within a range, group by group, n-tile major with the group's
    // m-tiles consecutive: a B_e column block is reused from L2 by all of the
    // group's m-tiles, an A row block by neighbouring n-tiles.
    const int tiles_n = (p.N + BN - 1) / BN;
    // group sizes in m-tiles, 64 groups per wave-wide step (one coalesced
    // load, a lane per group, prefix sums across the wave)
    const int ln = threadIdx.x & 63;
    int total = 0;
    for (int base = 0; base < p.groups; base += 64) {
      const int g = base + ln;
      const int mt = g < p.groups ? (p.g_off[g + 1] - p.g_off[g] + BM - 1) / BM : 0;
      total += wave_sum_int(mt);
    }
    const int real = total * tiles_n;
    const int per = (real + NUM_XCD - 1) / NUM_XCD;
    const int li = blockIdx.x / NUM_XCD;
    const int pid = (blockIdx.x % NUM_XCD) * per + li;
    if (li >= per || pid >= real) return false;
    int e = 0, acc = 0, mte = 1;
    for (int base = 0; base < p.groups; base += 64) {
      const int g = base + ln;
      const int mt = g < p.groups ? (p.g_off[g + 1] - p.g_off[g] + BM - 1) / BM : 0;
      const int incl = wave_incl_scan_int(mt * tiles_n);
      const int excl = incl - mt * tiles_n;
      const uint64_t hit = __ballot(mt > 0 && pid >= acc + excl && pid < acc + incl);
      if (hit) {
        const int l = __ffsll((unsigned long long)hit) - 1;
        e = base + l;
        mte = __shfl(mt, l, 64);
        acc += __shfl(excl, l, 64);
        break;
      }
      acc += __shfl(incl, 63, 64);
    }
    e = __builtin_amdgcn_readfirstlane(e);
    mte = __builtin_amdgcn_readfirstlane(mte);
    acc = __builtin_amdgcn_readfirstlane(acc);
    tm = (pid - acc) % mte;
    tn = (pid - acc) / mte;
    const long r0 = p.g_off[e];
    p.M = p.g_off[e + 1] - p.g_off[e];
    p.A += r0 * p.lda;  // K-contiguous A: group rows are row blocks
    p.B += (long)e * p.strideB;
    p.C = (char*)p.C + r0 * p.ldc * (EPI == kStoreBF16 || EPI == kResidBF16 ? 2 : 4);
    if (EPI == kResidBF16) p.R += r0 * p.ldr;
  } else if (GROUP == 4) {
    // the last, partial round of a product of 2BN-wide tiles: full tile
    // p.tile_base + i of the band order above runs as two BN-wide halves
    // (workgroups 2i and 2i + 1 after the same XCD remapping), so the round
    // fills twice as many CUs with half as much work each
    const int tiles_m = (p.M + BM - 1) / BM;
    const int tiles_n = (p.N + 2 * BN - 1) / (2 * BN);
    const int nb = gridDim.x, bid = blockIdx.x;
    const int nb8 = nb - nb % NUM_XCD;
    const int ph = bid < nb8 ? (bid % NUM_XCD) * (nb8 / NUM_XCD) + bid / NUM_XCD : bid;
    const int pid = p.tile_base + ph / 2;
    const int in_group = GROUP_M * tiles_n;
    const int first_m = (pid / in_group) * GROUP_M;
    const int gsize = min(tiles_m - first_m, GROUP_M);
    tm = first_m + (pid % in_group) % gsize;
    tn = 2 * ((pid % in_group) / gsize) + (ph & 1);
  } else if (GROUP == 3) {
    // uniform split of the reduction: split e covers k rows [e * ks, e * ks + ks)
    // (ks = p.strideB) and stores its partial product to C + e * strideC
    const int tiles_m = (p.M + BM - 1) / BM;
    const int tiles_n = (p.N + BN - 1) / BN;
    const int nb = gridDim.x, bid = blockIdx.x;
    const int nb8 = nb - nb % NUM_XCD;
    const int pid = bid < nb8 ? (bid % NUM_XCD) * (nb8 / NUM_XCD) + bid / NUM_XCD : bid;
    const int e = pid / (tiles_m * tiles_n);
    const int t = pid % (tiles_m * tiles_n);
    const int in_group = GROUP_M * tiles_n;
    const int first_m = (t / in_group) * GROUP_M;
    const int gsize = min(tiles_m - first_m, GROUP_M);
    tm = first_m + (t % in_group) % gsize;
    tn = (t % in_group) / gsize;
    const long k0 = (long)e * p.strideB;
    p.K = (int)min((long)p.K - k0, p.strideB);
    p.A += LA == kKC ? k0 : k0 * p.lda;
    p.B += LB == kKC ? k0 : k0 * p.ldb;
    p.C = (char*)p.C + (long)e * p.strideC * 4;
  } else {
    // K-grouped: one (m, n) tile grid per group, reduction over the group's
    // rows; XCD-contiguous ranges of tiles, group by group
    const int tiles_m = (p.M + BM - 1) / BM;
    const int tiles_n = (p.N + BN - 1) / BN;
    const int nb = gridDim.x, bid = blockIdx.x;
    const int nb8 = nb - nb % NUM_XCD;
    const int pid = bid < nb8 ? (bid % NUM_XCD) * (nb8 / NUM_XCD) + bid / NUM_XCD : bid;
    const int e = pid / (tiles_m * tiles_n);
    const int t = pid % (tiles_m * tiles_n);
    tm = t / tiles_n;
    tn = t % tiles_n;
    const long r0 = p.g_off[e];
    p.K = p.g_off[e + 1] - p.g_off[e];
    p.A += r0 * p.lda;  // both operands M/N-contiguous: group rows are k rows
    p.B += r0 * p.ldb;
    p.C = (char*)p.C + (long)e * p.strideC * 4;
    if (EPI == kStoreF32Adam || EPI == kAccF32Adam) {
      const long off = (long)e * p.strideC;
      p.o_master += off;
      p.o_m += off;
      p.o_v += off;
      p.o_param += off;
    }
  }
  return true;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int LA, int LB, int EPI, int GROUP = 0>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64, 1) void gemm_kernel(GemmArgs p) {
  static_assert(LA == kKC && LB == kKC, "the double-buffered kernel takes K-contiguous operands");
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int FM = WM / 32, FN = WN / 32;
  static_assert(FM * 32 == WM && FN * 32 == WN, "wave tile must be a multiple of 32");
  constexpr int A_ELEMS = BM * CHUNKS, B_ELEMS = BN * CHUNKS;
  __shared__ uint4 lds[2][A_ELEMS + B_ELEMS];

  int tm, tn;
  if (!tile_setup<BM, BN, EPI, GROUP, LA, LB>(p, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;
  constexpr int NW = WAVES_M * WAVES_N;

  KcLoader<BM, NW> la;
  KcLoader<BN, NW> lb;

  f32x16_t acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // ---- main loop: the barrier that publishes tile t+1 sits before the last
  // 16-deep k-slice of tile t, so every wave leaves it with that slice's
  // MFMAs to issue while the first fragments of tile t+1 are read; right
  // after it, tile t+2 is loaded into tile t's buffer.
  const int nk = (p.K + BK - 1) / BK;
  constexpr int KS = BK / 16;
  la.load(p.A, p.lda, m0, p.M, 0, p.K, lds[0], wave, lane);
  lb.load(p.B, p.ldb, n0, p.N, 0, p.K, lds[0] + A_ELEMS, wave, lane);
  __syncthreads();
  bf16x8_t fa[2][FN], fb[2][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i) fa[0][i] = frag(lds[0] + A_ELEMS, wn * WN + i * 32, 0, lane);
#pragma unroll
  for (int j = 0; j < FM; ++j) fb[0][j] = frag(lds[0], wm * WM + j * 32, 0, lane);
  // tile 1 into the second buffer (past the end: zeros into an unused buffer)
  la.load(p.A, p.lda, m0, p.M, BK, p.K, lds[1], wave, lane);
  lb.load(p.B, p.ldb, n0, p.N, BK, p.K, lds[1] + A_ELEMS, wave, lane);

  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    const uint4* At = lds[cur];
    const uint4* Bt = lds[cur] + A_ELEMS;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const int cb = kk & 1, nx = cb ^ 1;
      if (kk + 1 < KS) {
#pragma unroll
        for (int i = 0; i < FN; ++i) fa[nx][i] = frag(Bt, wn * WN + i * 32, kk + 1, lane);
#pragma unroll
        for (int j = 0; j < FM; ++j) fb[nx][j] = frag(At, wm * WM + j * 32, kk + 1, lane);
      } else {
        // publish tile t+1: this wave's DMA has landed and its reads of tile
        // t are complete; after the barrier every wave's are
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_s_barrier();
        const uint4* An = lds[cur ^ 1];
        const uint4* Bn = lds[cur ^ 1] + A_ELEMS;
#pragma unroll
        for (int i = 0; i < FN; ++i) fa[nx][i] = frag(Bn, wn * WN + i * 32, 0, lane);
#pragma unroll
        for (int j = 0; j < FM; ++j) fb[nx][j] = frag(An, wm * WM + j * 32, 0, lane);
        // every wave's reads of tile t are complete: its buffer takes tile
        // t+2 (all zeros past the end)
        la.load(p.A, p.lda, m0, p.M, (kt + 2) * BK, p.K, lds[cur], wave, lane);
        lb.load(p.B, p.ldb, n0, p.N, (kt + 2) * BK, p.K, lds[cur] + A_ELEMS, wave, lane);
      }
#pragma unroll
      for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cb][i], fb[cb][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  __builtin_amdgcn_s_waitcnt(0);  // the last (all-zero) tile loads land before exit
  store_tile<EPI, FN, FM>(p, acc, m0 + wm * WM, n0 + wn * WN, lane);
}

// ---- ring pipeline: four 32-deep stages, 16x16x32 MFMAs ---------------------
// Stage slot = A part then B part. K-contiguous operand: ROWS rows of four
// 16-byte chunks (k 0..31), chunk c of row r at c ^ ((r >> 1) & 3).
// M/N-contiguous operand: 32 k-rows of ROWS elements, 16-byte chunk c of
// k-row k at c ^ ((k & 3) << 2) ^ (((k >> 3) & 1) << 1). A fragment read
// touches k-rows {0..3} and {8..11} (or their +4 / +16 shifts) in one
// half-wave; the two XOR terms put those eight rows' 32-byte pieces on
// distinct banks.
constexpr int SK = 32;

template <int ROWS, int NW>
struct RingPart {
  static constexpr int ELEMS = ROWS * 4;         // 16-byte chunks per stage
  static constexpr int PER = ROWS * 4 / 64 / NW;  // DMA instructions per wave per stage
  static_assert(PER * 64 * NW == ROWS * 4, "stage tile must split over the waves");
};

// K-contiguous stage: 64-byte rows (four 16-byte chunks), two rows per 128-byte
// bank window. A ds_read_b128 serves eight lanes per cycle, here eight
// consecutive rows at one logical chunk: XOR-ing the chunk with (row / 2) % 4
// puts the four rows of each parity on four different slots, so the eight
// reads cover the window once (keying on row / 4 left two rows per slot, a
// two-way conflict on every fragment read).
__device__ __forceinline__ int kc_swz(int row) { return (row >> 1) & 3; }
__device__ __forceinline__ int kc4(int row, int c) { return row * 4 + (c ^ kc_swz(row)); }

// M/N-contiguous stage of ROWS elements per k-row (see above). 64-element rows
// are 128 bytes, two to a 256-byte bank window: the four k-rows of one parity
// (k = 0, 2, 8, 10 and their shifts) take the four 32-byte pieces of a row.
template <int ROWS>
__device__ __forceinline__ int mc_swz(int k) {
  static_assert(ROWS >= 64, "the swizzle needs at least eight chunks per k-row");
  return ROWS >= 128 ? ((k & 3) << 2) ^ (((k >> 3) & 1) << 1)
                     : (((k >> 1) & 1) << 1) | (((k >> 3) & 1) << 2);
}

template <int ROWS>
__device__ __forceinline__ int mc_ring_elem(int k, int m) {
  return k * ROWS + (((m >> 3) ^ mc_swz<ROWS>(k)) << 3) + (m & 7);
}

__device__ __forceinline__ uint32_t lds_addr(const void* ptr) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)ptr;
}

// DMA instruction i (of RingPart::PER) of this wave for one operand of a stage.
template <int ROWS, int NW, int LAYOUT>
__device__ __forceinline__ void ring_dma(int i, const bf16_t* __restrict__ src, long ld, int row0,
                                         int rows_lim, int k0, int K, uint4* part, int wave,
                                         int lane) {
  const int blk = i * NW + wave;  // 1 KB block of the stage's part
  if (LAYOUT == kKC) {
    const __amdgpu_buffer_rsrc_t r = rsrc(src + (long)row0 * ld + k0);
    const int row = blk * 16 + (lane >> 2);
    const int c = (lane & 3) ^ kc_swz(row);
    const bool ok = (row0 + row < rows_lim) && (k0 + c * 8 < K);
    const uint32_t off = ok ? (uint32_t)(((long)row * ld + c * 8) * 2) : kOOB;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)(part + blk * 64), 16, off, 0, 0, 0);
  } else {
    constexpr int LPR = ROWS / 8;  // lanes per k-row
    constexpr int RPI = 64 / LPR;  // k-rows per instruction
    const __amdgpu_buffer_rsrc_t r = rsrc(src + (long)k0 * ld + row0);
    const int k = blk * RPI + lane / LPR;
    const int c = (lane % LPR) ^ mc_swz<ROWS>(k);
    const bool ok = (k0 + k < K) && (row0 + c * 8 < rows_lim);
    const uint32_t off = ok ? (uint32_t)(((long)k * ld + c * 8) * 2) : kOOB;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)(part + blk * 64), 16, off, 0, 0, 0);
  }
}

// 16x16x32 operand of rows base..base+15 over a whole stage: the lane holds
// row base + lane % 16, k = 8 (lane / 16) .. + 7. Issued as asm (not tracked
// by the compiler: ring_fence waits for it). M/N-contiguous: two transposing
// reads, lane 4r + j of each 16-lane group pointing at k-row r, elements
// 4j..4j+3 of a 4 x 16 block.
template <int LAYOUT, int ROWS>
__device__ __forceinline__ bf16x8_t ring_frag(const uint4* part, int base, int lane) {
  if (LAYOUT == kKC) {
    const uint32_t a = lds_addr(part + kc4(base + (lane & 15), lane >> 4));
    uint4 r;
    asm volatile("ds_read_b128 %0, %1" : "=v"(r) : "v"(a) : "memory");
    return __builtin_bit_cast(bf16x8_t, r);
  } else {
    const uint16_t* t = reinterpret_cast<const uint16_t*>(part);
    const int g = lane >> 4, i = lane & 15;
    const int m = base + 4 * (i & 3);
    const int k = g * 8 + (i >> 2);
    const uint32_t a0 = lds_addr(t + mc_ring_elem<ROWS>(k, m));
    const uint32_t a1 = lds_addr(t + mc_ring_elem<ROWS>(k + 4, m));
    uint2 lo, hi;
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(lo) : "v"(a0) : "memory");
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(hi) : "v"(a1) : "memory");
    return __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
  }
}

// Wait for every outstanding LDS read; the fragments count as rewritten here,
// so nothing that uses (or reuses the registers of) them moves above the wait.
template <int FN, int FM>
__device__ __forceinline__ void ring_fence(bf16x8_t (&fa)[FN], bf16x8_t (&fb)[FM]) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int i = 0; i < FN; ++i) asm volatile("" : "+v"(fa[i]));
#pragma unroll
  for (int j = 0; j < FM; ++j) asm volatile("" : "+v"(fb[j]));
}

// At most N DMA instructions of this wave still outstanding.
template <int N>
__device__ __forceinline__ void wait_dma() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// ---- bf16 epilogue: eight consecutive n of row m ---------------------------
// A full piece is one 16-byte store, streaming (nontemporal, see store4) or
// ordinary: 64 contiguous bytes per row and instruction, and where these are
// whole 64-byte lines streaming stores keep the XCD's L2 for the operand rows.
// Rows that do not start on a line straddle two in every instruction; streamed,
// each half goes to memory by itself, while ordinary stores meet in L2. N 6120
// (2144 x 6120 x 208, K-contiguous) streamed 29.1 us, ordinary 18.0; N 6144
// streamed 14.6, ordinary 16.5.
template <int EPI, bool STREAM>
__device__ __forceinline__ void store8_bf16(const GemmArgs& p, int m, int n, float* x) {
  if (m >= p.M) return;
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] *= p.alpha;
  bf16_t* C = reinterpret_cast<bf16_t*>(p.C) + (long)m * p.ldc + n;
  const bool full = (n + 7 < p.N);
  if (EPI == kResidBF16) {
    const bf16_t* R = p.R + (long)m * p.ldr + n;
    if (full) {
      float r[8];
      unpack8(*reinterpret_cast<const uint4*>(R), r);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] += r[e];
    } else {
      for (int e = 0; e < 8; ++e)
        if (n + e < p.N) x[e] += bf2f(R[e]);
    }
  }
  if (full) {
    const f32x4_t v = __builtin_bit_cast(f32x4_t, pack8(x));
    if (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<f32x4_t*>(C));
    else *reinterpret_cast<f32x4_t*>(C) = v;
  } else {
    for (int e = 0; e < 8; ++e)
      if (n + e < p.N) C[e] = f2bf(x[e]);
  }
}

// ---- epilogue of 16x16 blocks: lane holds C[m][n..n+3] ---------------------
// bf16 output: lanes l and l ^ 16 swap halves of two neighbouring blocks so
// that each lane holds eight consecutive n, and a row takes 64 contiguous
// bytes per store instruction.
// AdamW epilogue of C[m][n..n+3] (kStoreF32Adam / kAccF32Adam): the weight
// gradient g (acc, or C + acc, rounded as the plain fp32 epilogues round it)
// is stored to C, then the same elements of the optimizer state are updated
// exactly as the standalone AdamW kernel does (adam1; sc = lr, 1 / bc1,
// 1 / bc2, clip). Every stream is touched once: nontemporal accesses.
struct AdamPiece {
  f32x4_t g, w, m1, m2;
};

template <int EPI>
__device__ __forceinline__ void adam_load(const GemmArgs& p, int m, int n, const float* v,
                                          AdamPiece& a) {
  a.g = f32x4_t{v[0] * p.alpha, v[1] * p.alpha, v[2] * p.alpha, v[3] * p.alpha};
  if (m >= p.M || n + 3 >= p.N) return;  // ragged pieces: adam_store, element by element
  const long i = (long)m * p.ldc + n;
  if (EPI == kAccF32Adam)
    a.g += __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>((float*)p.C + i));
  a.w = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(p.o_master + i));
  a.m1 = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(p.o_m + i));
  a.m2 = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(p.o_v + i));
}

template <int EPI>
__device__ __forceinline__ void adam_store(const GemmArgs& p, const float* sc, int m, int n,
                                           AdamPiece& a) {
  if (m >= p.M) return;
  const long i = (long)m * p.ldc + n;
  float* C = reinterpret_cast<float*>(p.C) + i;
  if (n + 3 < p.N) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float we = a.w[e], me = a.m1[e], ve = a.m2[e];
      adam1(we, me, ve, a.g[e], p.o_b1, p.o_b2, p.o_eps, p.o_wd, sc[0], sc[1], sc[2], sc[3]);
      a.w[e] = we;
      a.m1[e] = me;
      a.m2[e] = ve;
    }
    __builtin_nontemporal_store(a.g, reinterpret_cast<f32x4_t*>(C));
    __builtin_nontemporal_store(a.w, reinterpret_cast<f32x4_t*>(p.o_master + i));
    __builtin_nontemporal_store(a.m1, reinterpret_cast<f32x4_t*>(p.o_m + i));
    __builtin_nontemporal_store(a.m2, reinterpret_cast<f32x4_t*>(p.o_v + i));
    const u32x2_t pb = {pack2(a.w[0], a.w[1]), pack2(a.w[2], a.w[3])};
    __builtin_nontemporal_store(pb, reinterpret_cast<u32x2_t*>(p.o_param + i));
  } else {
    for (int e = 0; e < 4; ++e)
      if (n + e < p.N) {
        const float g = (EPI == kAccF32Adam ? C[e] : 0.0f) + a.g[e];
        C[e] = g;
        float we = p.o_master[i + e], me = p.o_m[i + e], ve = p.o_v[i + e];
        adam1(we, me, ve, g, p.o_b1, p.o_b2, p.o_eps, p.o_wd, sc[0], sc[1], sc[2], sc[3]);
        p.o_master[i + e] = we;
        p.o_m[i + e] = me;
        p.o_v[i + e] = ve;
        p.o_param[i + e] = f2bf(we);
      }
  }
}

// LINES: choose streaming or ordinary stores by the rows of C (else streaming).
// Once for the tile: a branch at every piece costs 1.4 us of 15. Four-wave tiles
// stream always: with both forms the compiler copies their accumulators around
// (128 x 128, K 2048: 66 -> 76 us).
template <int EPI, bool LINES, int FN, int FM>
__device__ __forceinline__ void store_tile16(const GemmArgs& p, const f32x4_t (&acc)[FN][FM],
                                             int mw, int nw, int lane) {
  if constexpr (EPI == kStoreBF16 || EPI == kResidBF16) {
    static_assert(FN % 2 == 0, "bf16 epilogue pairs neighbouring n-blocks");
    const int g = lane >> 4;
    const bool even = (g & 1) == 0;
    auto store = [&](auto STREAM) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < FN; i += 2)
#pragma unroll
        for (int j = 0; j < FM; ++j) {
          const int m = mw + j * 16 + (lane & 15);
          float x[8];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float send = even ? acc[i + 1][j][e] : acc[i][j][e];
            const float recv = __shfl_xor(send, 16);
            x[e] = even ? acc[i][j][e] : recv;
            x[4 + e] = even ? recv : acc[i + 1][j][e];
          }
          const int n = nw + (even ? i * 16 + g * 4 : (i + 1) * 16 + (g - 1) * 4);
          store8_bf16<EPI, decltype(STREAM)::value>(p, m, n, x);
        }
    };
    if (!LINES || ((reinterpret_cast<uintptr_t>(p.C) | (uintptr_t)(p.ldc * 2)) & 63) == 0)
      store(std::true_type());
    else
      store(std::false_type());
  } else {
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int j = 0; j < FM; ++j) {
        const int m = mw + j * 16 + (lane & 15);
        const int n = nw + i * 16 + (lane >> 4) * 4;
        const float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
        store4<EPI>(p, m, n, v);
      }
  }
}

// AdamW epilogue of a whole tile (kStoreF32Adam / kAccF32Adam), through LDS:
// the tile goes to the stage ring (free after the loop) as fp32, half of its
// rows at a time, and comes back row by row, so that each wave streams whole
// tile rows (1 KB per instruction for 256 columns) through the update's
// streams (C, master, m and v in; those and the bf16 parameter out) instead
// of 64-byte pieces of 16 rows, with the loads of U rows issued together.
// Chunks are XOR-swizzled by row so that the column writes of 16 rows and
// the row reads are both free of bank conflicts.
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int FN, int FM>
__device__ __forceinline__ void adam_tile(const GemmArgs& p, const f32x4_t (&acc)[FN][FM],
                                          float* lds, int m0, int n0, int wm, int wn, int wave,
                                          int lane) {
  constexpr int NW = WAVES_M * WAVES_N, WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int HR = BM / 2;            // rows per half
  constexpr int CPR = BN / 4;           // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;         // rows per wave instruction
  constexpr int IT = HR / (NW * RPI);   // row groups per wave and half
  constexpr int U = IT >= 4 ? 4 : IT;   // row groups loaded together
  static_assert(CPR <= 64 && 64 % CPR == 0 && CPR >= 16, "row must split over a wave");
  static_assert(IT * NW * RPI == HR && IT % U == 0, "half tile must split over the waves");
  static_assert(HR % WM == 0, "a wave's rows lie in one half");
  const float sc[4] = {p.o_sc[0], 1.0f / p.o_sc[1], 1.0f / p.o_sc[2], p.o_sc[3]};
  const int c = lane % CPR;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    __syncthreads();  // the ring (or the previous half) is no longer read
    if ((wm * WM) / HR == h) {
#pragma unroll
      for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) {
          const int ml = wm * WM + j * 16 + (lane & 15) - h * HR;
          const int cw = (wn * WN + i * 16 + (lane >> 4) * 4) / 4;
          *reinterpret_cast<f32x4_t*>(lds + ml * BN + ((cw ^ (ml & 15)) * 4)) = acc[i][j];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it0 = 0; it0 < IT; it0 += U) {
      AdamPiece a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = (wave + (it0 + u) * NW) * RPI + lane / CPR;
        const f32x4_t g = *reinterpret_cast<const f32x4_t*>(lds + r * BN + ((c ^ (r & 15)) * 4));
        const float v[4] = {g[0], g[1], g[2], g[3]};
        adam_load<EPI>(p, m0 + h * HR + r, n0 + c * 4, v, a[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = (wave + (it0 + u) * NW) * RPI + lane / CPR;
        adam_store<EPI>(p, sc, m0 + h * HR + r, n0 + c * 4, a[u]);
      }
    }
  }
}

// Each stage is one 16x16x32 k-step. Its fragments were read during the
// previous stage (double-buffered registers); BAR_AT MFMAs into the stage the
// wave waits for its own DMA of the next stage and meets the others at the
// barrier, after which the next stage is readable and the slot of this stage
// (every wave has fenced its reads) takes the stage four ahead. The NF
// fragment reads of the next stage and the D DMA instructions of the stage
// four ahead are then spread evenly over the MFMAs up to TAIL before the end,
// reads and DMAs interleaved in proportion, so that neither the LDS nor the
// texture unit sees a burst.
template <int BM, int BN, int WAVES_M, int WAVES_N, int LA, int LB, int EPI, int GROUP = 0,
          int TAIL = 4>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64, 1) void ring_kernel(GemmArgs p) {
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int FM = WM / 16, FN = WN / 16;
  static_assert(FM * 16 == WM && FN * 16 == WN, "wave tile must be a multiple of 16");
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int AE = RingPart<BM, NW>::ELEMS, BE = RingPart<BN, NW>::ELEMS;
  constexpr int DA = RingPart<BM, NW>::PER, DB = RingPart<BN, NW>::PER;
  constexpr int D = DA + DB;  // DMA instructions per wave per stage
  constexpr int NF = FN + FM, NM = FN * FM;
  constexpr int SLOT = AE + BE;
  constexpr int BAR_AT = 2;   // MFMAs of a stage issued before its barrier
  constexpr int E = NF + D;   // memory instructions spread over a stage
  constexpr int W = NM - BAR_AT - TAIL;
  static_assert(W > 0, "wave tile too small for the barrier placement and tail");
  __shared__ uint4 lds[4 * SLOT];

  int tm, tn;
  if (!tile_setup<BM, BN, EPI, GROUP, LA, LB>(p, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;

  f32x4_t acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.0f;
  const int nst = (p.K + SK - 1) / SK;

  // DMA instruction d (0..D-1) of stage st into slot st % 4 (zeros past K)
  auto dma = [&](int st, int d) {
    uint4* slot = lds + (st & 3) * SLOT;
    if (d < DA) ring_dma<BM, NW, LA>(d, p.A, p.lda, m0, p.M, st * SK, p.K, slot, wave, lane);
    else ring_dma<BN, NW, LB>(d - DA, p.B, p.ldb, n0, p.N, st * SK, p.K, slot + AE, wave, lane);
  };
  // fragment f (B fragments first, then A) of stage st
  auto read = [&](bf16x8_t* fa_, bf16x8_t* fb_, int st, int f) {
    const uint4* slot = lds + (st & 3) * SLOT;
    if (f < FN) fa_[f] = ring_frag<LB, BN>(slot + AE, wn * WN + f * 16, lane);
    else fb_[f - FN] = ring_frag<LA, BM>(slot, wm * WM + (f - FN) * 16, lane);
  };

  // prologue: stages 0..3 in flight; publish stage 0; its fragments
#pragma unroll
  for (int st = 0; st < 4; ++st)
#pragma unroll
    for (int d = 0; d < D; ++d) dma(st, d);
  wait_dma<3 * D>();
  __builtin_amdgcn_s_barrier();
  bf16x8_t fa[2][FN], fb[2][FM];
#pragma unroll
  for (int f = 0; f < NF; ++f) read(fa[0], fb[0], 0, f);

  // two stages per iteration, so that the fragment buffers are fixed; past
  // the last stage the ring holds zeros (an odd stage count runs one stage
  // of zeros)
  for (int st = 0; st < nst; st += 2) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int s = st + h;
      bf16x8_t* ca = fa[h];
      bf16x8_t* cb = fb[h];
      bf16x8_t* na = fa[h ^ 1];
      bf16x8_t* nb = fb[h ^ 1];
      ring_fence<FN, FM>(fa[h], fb[h]);
      __builtin_amdgcn_sched_barrier(0);
      int fr = 0, dm = 0;
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        const int i = q / FM, j = q % FM;
        if (q == BAR_AT) {
          // this wave's part of stage s + 1 has landed (s + 2 and s + 3 may
          // still be in flight)
          wait_dma<2 * D>();
          __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
        }
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ca[i], cb[j], acc[i][j], 0, 0, 0);
        if (q >= BAR_AT) {
          // memory instructions due by the end of MFMA q: event e is a read
          // when the read count steps between e and e + 1
          const int due = q - BAR_AT + 1 >= W ? E : ((q - BAR_AT + 1) * E) / W;
#pragma unroll
          for (int t = 0; t < (E + W - 1) / W + 1; ++t) {
            if (fr + dm < due) {
              const int e = fr + dm;
              const bool is_read = ((e + 1) * NF) / E > (e * NF) / E;
              if ((is_read && fr < NF) || dm >= D) read(na, nb, s + 1, fr++);
              else dma(s + 4, dm++);
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // every DMA has landed and every LDS read returned before the registers of
  // the last (unused) fragments are reused and before the workgroup exits
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  ring_fence<FN, FM>(fa[0], fb[0]);
  if constexpr (EPI == kStoreF32Adam || EPI == kAccF32Adam) {
    static_assert(BM / 2 * BN <= 4 * SLOT * 4, "half a tile must fit the stage ring");
    adam_tile<BM, BN, WAVES_M, WAVES_N, EPI, FN, FM>(p, acc, reinterpret_cast<float*>(lds), m0,
                                                      n0, wm, wn, wave, lane);
  } else {
    store_tile16<EPI, NW == 8, FN, FM>(p, acc, m0 + wm * WM, n0 + wn * WN, lane);
  }
}

// ---- small products: the reduction split over the waves of a workgroup ------
// A product of few output tiles leaves most CUs idle on large tiles, and on
// small ones each workgroup is a chain of short k-steps whose latency (DMA,
// LDS read, barrier) nothing hides. Here every wave owns the whole BM x BN
// tile and takes the 32-deep stages wave, wave + NW, ...: each streams its
// stages through a ring of its own (R slots of LDS), so the loop has no
// barrier, the waves of a SIMD hide each other's latency, and the serial chain
// is NW times shorter. At the end the NW partial tiles are added through LDS
// in wave order (deterministic) and each thread stores eight consecutive n.
// Four waves and two slots (64 KB of LDS): two workgroups share a CU; eight
// waves, or four with four slots, measured the same or slower (1000 x 1024 x
// 3072 data gradient: 12.7 us, 13.1, 13.2; 128 x 128 tiles 40.7). Bound by the
// latency of the chain up to one workgroup per CU (128 x 256 x 1376: 6.9 us
// against 21 on 128 x 128 tiles), beyond that by the L2 -> LDS stream of the
// small tiles (2048^3: 30 us, 128 x 128 tiles 25-26). Ordinary stores: the next
// kernel reads a result this small from L2.
template <int EPI>
__device__ __forceinline__ void store8_cached(const GemmArgs& p, int m, int n, float* x) {
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] *= p.alpha;
  const bool full = n + 7 < p.N;
  if (EPI == kStoreBF16 || EPI == kResidBF16) {
    bf16_t* C = reinterpret_cast<bf16_t*>(p.C) + (long)m * p.ldc + n;
    const bf16_t* R = p.R + (long)m * p.ldr + n;
    if (full) {
      if (EPI == kResidBF16) {
        float r[8];
        unpack8(*reinterpret_cast<const uint4*>(R), r);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] += r[e];
      }
      *reinterpret_cast<uint4*>(C) = pack8(x);
    } else {
      for (int e = 0; e < 8; ++e)
        if (n + e < p.N) C[e] = f2bf(EPI == kResidBF16 ? x[e] + bf2f(R[e]) : x[e]);
    }
  } else {
    float* C = reinterpret_cast<float*>(p.C) + (long)m * p.ldc + n;
    if (full) {
      float4* C4 = reinterpret_cast<float4*>(C);
      float4 a = make_float4(x[0], x[1], x[2], x[3]), b = make_float4(x[4], x[5], x[6], x[7]);
      if (EPI == kAccF32) {
        const float4 c = C4[0], d = C4[1];
        a = make_float4(a.x + c.x, a.y + c.y, a.z + c.z, a.w + c.w);
        b = make_float4(b.x + d.x, b.y + d.y, b.z + d.z, b.w + d.w);
      }
      C4[0] = a;
      C4[1] = b;
    } else {
      for (int e = 0; e < 8; ++e)
        if (n + e < p.N) C[e] = (EPI == kAccF32 ? C[e] : 0.0f) + x[e];
    }
  }
}

template <int BM, int BN, int NW, int R, int LA, int LB, int EPI, int GROUP>
__global__ __launch_bounds__(NW * 64) void wave_kernel(GemmArgs p) {
  constexpr int FM = BM / 16, FN = BN / 16, NM = FM * FN;
  constexpr int AE = RingPart<BM, 1>::ELEMS, BE = RingPart<BN, 1>::ELEMS, SLOT = AE + BE;
  constexpr int DA = RingPart<BM, 1>::PER, DB = RingPart<BN, 1>::PER, D = DA + DB;
  constexpr int CPR = BN / 4;       // fp32 chunks of 16 bytes per tile row
  constexpr int RED = BM * CPR;     // chunks of one wave's partial tile
  constexpr int LDS = NW * (R * SLOT > RED ? R * SLOT : RED);
  static_assert(R * D < 64 && LDS * 16 <= 160 * 1024, "ring depth");
  __shared__ uint4 lds[LDS];

  int tm, tn;
  if (!tile_setup<BM, BN, EPI, GROUP, LA, LB>(p, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint4* ring = lds + wave * R * SLOT;

  f32x4_t acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.0f;
  const int nst = (p.K + SK - 1) / SK;
  const int cnt = nst > wave ? (nst - wave + NW - 1) / NW : 0;

  // stage i of this wave (stage wave + i NW of the tile) into slot u; zeros
  // past K
  auto dma = [&](int i, int u) __attribute__((always_inline)) {
    const int k0 = (wave + i * NW) * SK;
    uint4* slot = ring + u * SLOT;
#pragma unroll
    for (int d = 0; d < DA; ++d)
      ring_dma<BM, 1, LA>(d, p.A, p.lda, m0, p.M, k0, p.K, slot, 0, lane);
#pragma unroll
    for (int d = 0; d < DB; ++d)
      ring_dma<BN, 1, LB>(d, p.B, p.ldb, n0, p.N, k0, p.K, slot + AE, 0, lane);
  };
  auto read = [&](bf16x8_t (&fa)[FN], bf16x8_t (&fb)[FM], int u) __attribute__((always_inline)) {
    const uint4* slot = ring + u * SLOT;
#pragma unroll
    for (int i = 0; i < FN; ++i) fa[i] = ring_frag<LB, BN>(slot + AE, i * 16, lane);
#pragma unroll
    for (int j = 0; j < FM; ++j) fb[j] = ring_frag<LA, BM>(slot, j * 16, lane);
  };

  if (cnt > 0) {
    // the loop runs R stages at a time, so that slots and fragment buffers are
    // fixed; stages past the last are zeros. Each step: the stage's fragments
    // (read during the previous step) arrive, its slot takes the stage R ahead,
    // half of its MFMAs, then the next stage's DMA has landed and its
    // fragments are read under the other half.
    static_assert(R % 2 == 0, "fragment buffers alternate");
#pragma unroll
    for (int u = 0; u < R; ++u) dma(u, u);
    bf16x8_t fa[2][FN], fb[2][FM];
    wait_dma<(R - 1) * D>();
    read(fa[0], fb[0], 0);
    for (int i = 0; i < cnt; i += R) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        constexpr int H = NM / 2;
        const int h = u & 1;
        ring_fence<FN, FM>(fa[h], fb[h]);
        __builtin_amdgcn_sched_barrier(0);
        dma(i + u + R, u);
#pragma unroll
        for (int q = 0; q < NM; ++q) {
          if (q == H) {
            __builtin_amdgcn_sched_barrier(0);
            wait_dma<(R - 1) * D>();
            read(fa[h ^ 1], fb[h ^ 1], (u + 1) % R);
            __builtin_amdgcn_sched_barrier(0);
          }
          acc[q / FM][q % FM] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              fa[h][q / FM], fb[h][q % FM], acc[q / FM][q % FM], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // the (unused) last reads and DMA land before their registers and slots
    // are reused
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    ring_fence<FN, FM>(fa[0], fb[0]);
  }
  __syncthreads();
  // partial tiles to LDS: row m of wave w holds its chunks XOR-ed with m % 16
  // (16 rows of one chunk, and the chunks of two rows, cover all banks)
  f32x4_t* red = reinterpret_cast<f32x4_t*>(lds);
  constexpr int XM = CPR >= 16 ? 15 : CPR - 1;
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) {
      const int m = j * 16 + (lane & 15), c = i * 4 + (lane >> 4);
      red[wave * RED + m * CPR + (c ^ (m & XM))] = acc[i][j];
    }
  __syncthreads();
  constexpr int ITEMS = BM * BN / 8;
  for (int t = threadIdx.x; t < ITEMS; t += NW * 64) {
    const int m = t / (BN / 8), c = (t % (BN / 8)) * 2;
    const f32x4_t* r = red + m * CPR;
    f32x4_t a = r[c ^ (m & XM)], b = r[(c + 1) ^ (m & XM)];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      a += r[w * RED + (c ^ (m & XM))];
      b += r[w * RED + ((c + 1) ^ (m & XM))];
    }
    float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    if (m0 + m < p.M && n0 + c * 4 < p.N) store8_cached<EPI>(p, m0 + m, n0 + c * 4, x);
  }
}

// The ring pipeline runs every tile except the K-contiguous 128 x 128 one, which
// runs on the double-buffered kernel.
template <int BM, int BN, int WAVES_M, int WAVES_N, int LA, int LB, int EPI, int GROUP>
void launch_kernel(const GemmArgs& a, long grid, hipStream_t s) {
  constexpr bool kBuffered = LA == kKC && LB == kKC && GROUP == 0 && BM == 128 && BN == 128;
  if constexpr (kBuffered)
    hipLaunchKernelGGL((gemm_kernel<BM, BN, WAVES_M, WAVES_N, LA, LB, EPI, GROUP>),
                       dim3((unsigned)grid), dim3(WAVES_M * WAVES_N * 64), 0, s, a);
  else
    hipLaunchKernelGGL((ring_kernel<BM, BN, WAVES_M, WAVES_N, LA, LB, EPI, GROUP>),
                       dim3((unsigned)grid), dim3(WAVES_M * WAVES_N * 64), 0, s, a);
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int LA, int LB, int EPI>
hipError_t launch(const GemmArgs& a, hipStream_t s) {
  const long tiles = (long)((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  launch_kernel<BM, BN, WAVES_M, WAVES_N, LA, LB, EPI, 0>(a, tiles, s);
  return hipGetLastError();
}

// M-grouped: at most M / BM + groups m-tiles exist, whatever the group sizes.
// Real tiles <= (M / BM + groups) * tiles_n; rounded up so that every XCD's
// share of the workgroups covers ceil(real / 8) tiles.
template <int BM, int BN>
long grouped_m_grid(const GemmArgs& a) {
  const long mt = a.M / BM + a.groups;
  return ((mt * ((a.N + BN - 1) / BN) + NUM_XCD - 1) / NUM_XCD + 1) * NUM_XCD;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int LB, int EPI>
hipError_t launch_grouped_m(const GemmArgs& a, hipStream_t s) {
  launch_kernel<BM, BN, WAVES_M, WAVES_N, kKC, LB, EPI, 1>(a, grouped_m_grid<BM, BN>(a), s);
  return hipGetLastError();
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI>
hipError_t launch_grouped_k(const GemmArgs& a, hipStream_t s) {
  const long tiles = (long)a.groups * ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  launch_kernel<BM, BN, WAVES_M, WAVES_N, kMC, kMC, EPI, 2>(a, tiles, s);
  return hipGetLastError();
}

// C (op)= the sum of S fp32 partial products part[e][m][n] (leading dimension
// ldp, `stride` apart) in split order, with the epilogue of the product they
// are parts of; eight consecutive n per thread. HBM-bound: S partials read
// once, C written once.
template <int EPI>
__global__ __launch_bounds__(256) void split_reduce_k(GemmArgs p, const float* __restrict__ part,
                                                      int S, long stride, int ldp) {
  const int nq = ldp / 8;
  const long q = (long)blockIdx.x * 256 + threadIdx.x;
  if (q >= (long)p.M * nq) return;
  const int m = (int)(q / nq), n = (int)(q % nq) * 8;
  const float* src = part + (long)m * ldp + n;
  f32x4_t a = *reinterpret_cast<const f32x4_t*>(src);
  f32x4_t b = *reinterpret_cast<const f32x4_t*>(src + 4);
#pragma unroll 4
  for (int e = 1; e < S; ++e) {
    a += *reinterpret_cast<const f32x4_t*>(src + e * stride);
    b += *reinterpret_cast<const f32x4_t*>(src + e * stride + 4);
  }
  float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  store8_cached<EPI>(p, m, n, x);
}

constexpr int kCUs = 256;

// ---- choice of the tile ------------------------------------------------------
// Four tile shapes cover everything below a chip full of 256 x 256 tiles:
// 256 x 256, 128 x 256 and 128 x 128 with the waves side by side in the tile,
// 64 x 64 with the waves splitting the reduction (wave_kernel). None wins
// everywhere: a large tile reads the least per FLOP and leaves CUs idle when
// there are few of them, a small one the reverse. The choice is the smallest
// estimate of
//   fixed + round * (rounds - 1) + K * (per_k + full_k * share of CUs busy) * rounds
// microseconds, rounds counted over the tiles resident at once (`slots`: two
// workgroups of the four-wave tiles share a CU; a last round that gives every
// CU at most one of them costs `half`; one that gives some two costs a whole one,
// except with both operands K-contiguous at 128 x 128, whose kernel's cost rises
// evenly: with K 4096 45 us at 256 tiles, 50 at 288, 53 at 320, 60 at 384,
// and 51, 52, 54, 57 on 128 x 256. Over products of 257 to 511 tiles of 128 x 128
// the picks are 3.5 % from the fastest tile with the even rise and 3.7 % without
// (120 products, 6 of them then slower than one 256 x 128 launch); in the data
// gradient 11 % with it and 0.2 % without (20), in the weight gradient 9.8 and
// 6.6 % (72)). The constants are a fit (10-15 % rms)
// to 130 products, M, N in 64..16384, K in 64..16384, all layouts, timed on
// every tile: the pick is on average 2 % slower than the fastest tile, and
// 1.47 times as fast as one threshold on the number of tiles (256 x 256 from
// 256 tiles, then 256 x 128, else 128 x 128). The round of 64 x 64 tiles is set by
// reductions below 320 (1792 x 1800 x 40, data gradient, 841 tiles: 10.8 us, 8.3 on
// 128 x 128). E.g. (M, N, K) = (1000, 1024,
// 3072), data gradient: 12.7 us on 64 x 64, 40.7 on 128 x 128; (2048, 2048,
// 3072): 38 on 128 x 256, 41 on 128 x 128, 60 on 256 x 256.
enum Tile { kT256, kT128x256, kT128, kT64, kTiles };
constexpr int kTileM[kTiles] = {256, 128, 128, 64}, kTileN[kTiles] = {256, 256, 128, 64};
struct TileCost {
  double fixed, per_k, full_k;
};
constexpr int kSlots[kTiles] = {256, 256, 512, 512};
constexpr double kHalfRound[kTiles] = {1.0, 1.0, 0.55, 0.52}, kRound[kTiles] = {8.0, 5.0, 6.0, 2.5};
// [layout: (KC, KC), (KC, MC), (MC, MC)][tile]
constexpr TileCost kCost[3][kTiles] = {
    {{10.0, .0150, .0120}, {6.0, .0092, .0068}, {4.3, .0110, .0070}, {3.7, .0037, .0040}},
    {{10.0, .0155, .0100}, {6.5, .0093, .0055}, {6.0, .0175, .0010}, {3.7, .0043, .0042}},
    {{10.5, .0168, .0094}, {6.5, .0108, .0040}, {4.5, .0150, .0010}, {5.0, .0066, .0024}}};

long tile_count(int t, long M, long N) {
  return ((M + kTileM[t] - 1) / kTileM[t]) * ((N + kTileN[t] - 1) / kTileN[t]);
}

double tile_cost(int layout, int t, long tiles, long K) {
  const TileCost& c = kCost[layout][t];
  const long full = tiles / kSlots[t], rem = tiles % kSlots[t];
  const double half = kHalfRound[t];
  const double part = rem == 0      ? 0.0
                      : rem <= kCUs ? half
                      : t == kT128 && layout == 0
                          ? half + (1.0 - half) * (double)(rem - kCUs) / kCUs
                          : 1.0;
  const double busy = (double)(tiles < kCUs ? tiles : kCUs) / kCUs;
  return c.fixed + kRound[t] * (double)(full + (rem > 0) - 1) +
         (double)K * (c.per_k + c.full_k * busy) * ((double)full + part);
}

// A product may also split its reduction over S times as many workgroups
// (caller's scratch: fp32 partials, then one pass that adds them in split
// order), as long as the workgroups still fit one round: S partial tiles
// cost their own traffic, so more rounds never paid. Measured, data gradient
// (2048, 2048, 16384): 256 x 256 tiles 279 us on 64 CUs, 124 split four ways
// (128 x 128 tiles unsplit: 200); weight gradient (4096, 1024, 16384): 308,
// 129 (169).
constexpr int kMaxSplit = 16;
constexpr int kMinSplitK = 128;
double reduce_cost(long S, long M, long N) { return 3.0 + (double)(S * M * N) * 8.0 / 5.5e6; }

struct Plan {
  Tile tile;
  int splits;
  long ks;  // reduction length of a split (the last one may be shorter)
};

long split_len(long K, int S) { return ((K + S - 1) / S + BK - 1) / BK * BK; }
long partial_ld(long N) { return (N + 7) / 8 * 8; }
size_t partial_bytes(int S, long M, long N) {
  return S > 1 ? (size_t)S * (size_t)M * (size_t)partial_ld(N) * 4 : 0;
}

// scratch: bytes there are for partial tiles
Plan pick_plan(int layout, long M, long N, long K, size_t scratch) {
  Plan best = {kT256, 1, K};
  // From a chip of well filled 256 x 256 tiles up no other tile is better on
  // average (192 to 640 rows or columns: 0.84 to 1.5 times the estimate's pick;
  // 8192 x 1536 x 1536 has 192 tiles: 36.9 us, 128 x 128 46.8, 128 x 256 50.1).
  // With M or N of at most 128, or just above 256, half of each tile and more is
  // padding: 64 x 75072 x 368, data gradient, 24.2 us, 17.0 on the pick; 264 x
  // 98624 x 432 59 and 46; at 136 and 9/16 filled the two are level.
  const long big = tile_count(kT256, M, N);
  if (big >= kCUs && (double)M * (double)N > big * (65536.0 * 9 / 16)) return best;
  double cost = 1e30;
  long tiles[kTiles];
  for (int t = 0; t < kTiles; ++t) {
    tiles[t] = t == kT256 ? big : tile_count(t, M, N);
    const double c = tile_cost(layout, t, tiles[t], K);
    if (c < cost) {
      cost = c;
      best = {(Tile)t, 1, K};
    }
  }
  for (int t = 0; t < kTiles; ++t) {
    const int most = (int)std::min<long>(std::min<long>(kMaxSplit, kCUs / tiles[t]), K / kMinSplitK);
    const TileCost& tc = kCost[layout][t];
    for (int S = 2; S <= most; ++S) {
      // Partials of S splits alone, and of more, cost too much; or with a round of
      // the shorter reduction. (A layer call plans each of its products twice: a
      // small layer's take 0.6 us instead of 1.9.)
      const double extra = reduce_cost(S, M, N);
      if (tc.fixed + extra >= cost || partial_bytes(S, M, N) > scratch) break;
      if (tc.fixed + extra + (double)(K / S) * tc.per_k * 0.5 >= cost) continue;
      const long ks = split_len(K, S);
      if ((K + ks - 1) / ks != S) continue;  // the last split would be empty
      const double c = tile_cost(layout, t, tiles[t] * S, ks) + extra;
      if (c < cost) {
        cost = c;
        best = {(Tile)t, S, ks};
      }
    }
  }
  return best;
}

constexpr int layout_id(int la, int lb) { return la == kMC ? 2 : (lb == kMC ? 1 : 0); }

template <int LA, int LB, int EPI, int GROUP>
void launch_wave(const GemmArgs& a, long grid, hipStream_t s) {
  hipLaunchKernelGGL((wave_kernel<64, 64, 4, 2, LA, LB, EPI, GROUP>), dim3((unsigned)grid),
                     dim3(256), 0, s, a);
}

template <int LA, int LB, int EPI>
hipError_t launch_split(const GemmArgs& a, const Plan& pl, float* part, hipStream_t s) {
  GemmArgs p = a;
  const long ldp = partial_ld(a.N), stride = (long)a.M * ldp;
  p.C = part;
  p.ldc = ldp;
  p.alpha = 1.0f;
  p.strideB = pl.ks;
  p.strideC = stride;
  const long grid = tile_count(pl.tile, a.M, a.N) * pl.splits;
  switch (pl.tile) {
    case kT64: launch_wave<LA, LB, kStoreF32, 3>(p, grid, s); break;
    case kT128: launch_kernel<128, 128, 2, 2, LA, LB, kStoreF32, 3>(p, grid, s); break;
    case kT128x256: launch_kernel<128, 256, 2, 4, LA, LB, kStoreF32, 3>(p, grid, s); break;
    default: launch_kernel<256, 256, 2, 4, LA, LB, kStoreF32, 3>(p, grid, s); break;
  }
  const long items = (long)a.M * (ldp / 8);
  hipLaunchKernelGGL(split_reduce_k<EPI>, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s,
                     a, part, pl.splits, stride, (int)ldp);
  return hipGetLastError();
}

template <int LA, int LB, int EPI>
hipError_t dispatch_tiles(const GemmArgs& a, hipStream_t s, float* part, size_t part_bytes) {
  const long big = tile_count(kT256, a.M, a.N);
  const Plan pl = pick_plan(layout_id(LA, LB), a.M, a.N, a.K, part ? part_bytes : 0);
  if (pl.splits > 1) return launch_split<LA, LB, EPI>(a, pl, part, s);
  const Tile t = pl.tile;
  if (t == kT64) {
    launch_wave<LA, LB, EPI, 0>(a, tile_count(kT64, a.M, a.N), s);
    return hipGetLastError();
  }
  if (t == kT128) return launch<128, 128, 2, 2, LA, LB, EPI>(a, s);
  if (t == kT128x256) return launch<128, 256, 2, 4, LA, LB, EPI>(a, s);
  if constexpr (LA == kKC && LB == kKC) {
    const long tail = big % kCUs;
    if (big > kCUs && tail <= kCUs / 2 && tail > 0) {
      // whole rounds of 256 x 256 tiles, then the last half-empty round's
      // tiles as 256 x 128 halves, twice as many workgroups; only products
      // with both operands K-contiguous (the forward ones, which run alone
      // on the chip; a product that shares the chip with a side stream
      // leaves its partial round to that stream's work)
      launch_kernel<256, 256, 2, 4, LA, LB, EPI, 0>(a, big - tail, s);
      GemmArgs b = a;
      b.tile_base = (int)(big - tail);
      launch_kernel<256, 128, 2, 4, LA, LB, EPI, 4>(b, 2 * tail, s);
      return hipGetLastError();
    }
  }
  // 128 x 64 wave tiles (2 x 4 waves, two per SIMD): in a data gradient (B
  // M/N-contiguous, read with the slower transposing reads) they put the
  // transposing reads on the narrow side of the wave tile, half as many per
  // stage as with 64 x 128; the other products measured no slower (slightly
  // faster)
  return launch<256, 256, 2, 4, LA, LB, EPI>(a, s);
}

}  // namespace

namespace {
// Tile of a product over row groups, from the same estimates. The host knows
// the rows' upper bound, not the groups' sizes: a group of r rows is taken to
// have r / BM + 1/2 m-tiles, at least one. The smaller tile has to win by 5 %
// (groups of about 400 rows estimate alike and run better on 256 rows), and
// 64 x 64 tiles are for launches of at most two rounds (beyond, every tile
// streams its own weights). Measured, rows per group x groups, forward
// gate/up: 100 x 160 (N 1024, K 2048) 186 us on 256 x 256, 170 on 128 x 256,
// 234 on 64 x 64; 75 x 8 (2048, 1024) 30, 19, 13.5; 1024 x 64 (2816, 2048)
// 1000, 1027, 1575.
Tile pick_grouped_tile(int layout, long rows, long groups, long N, long K) {
  Tile best = kT256;
  double cost = 1e30;
  for (const Tile t : {kT256, kT128x256, kT64}) {
    const double per = (double)rows / (double)groups / kTileM[t] + 0.5;
    const long tiles = (long)((per < 1.0 ? 1.0 : per) * (double)groups) *
                       ((N + kTileN[t] - 1) / kTileN[t]);
    if (t == kT64 && tiles > 2 * kSlots[kT64]) continue;
    const double c = tile_cost(layout, t, tiles, K);
    if (c < 0.95 * cost) {
      cost = c;
      best = t;
    }
  }
  return best;
}

template <int LB>
hipError_t launch_grouped_rows(const GemmArgs& a, hipStream_t s) {
  switch (pick_grouped_tile(layout_id(kKC, LB), a.M, a.groups, a.N, a.K)) {
    case kT64:
      launch_wave<kKC, LB, kStoreBF16, 1>(a, grouped_m_grid<64, 64>(a), s);
      return hipGetLastError();
    case kT128x256: return launch_grouped_m<128, 256, 2, 4, LB, kStoreBF16>(a, s);
    default: break;
  }
  // the transposing reads of an M/N-contiguous weight on the narrow side of
  // the wave tile (128 x 64 waves), as in the ungrouped data gradient
  if constexpr (LB == kKC) return launch_grouped_m<256, 256, 4, 2, LB, kStoreBF16>(a, s);
  else return launch_grouped_m<256, 256, 2, 4, LB, kStoreBF16>(a, s);
}

}  // namespace

hipError_t gemm_grouped_m(GemmLayout lb, GemmEpilogue epi, const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0 || a.groups <= 0) return hipSuccess;
  if (lb == kKC && epi == kStoreBF16) return launch_grouped_rows<kKC>(a, s);
  if (lb == kMC && epi == kStoreBF16) return launch_grouped_rows<kMC>(a, s);
  return hipErrorInvalidValue;
}

// 128 x 64 waves: as fast as 64 x 128 with the AdamW epilogue (its streams bound
// it) and 2-10 % faster without (64 groups of 1024 rows, 2816 x 2048: 1004 us
// against 1018; 160 of 100, 1024 x 2048: 332 against 370). For groups of about
// 100 rows 128 x 128 tiles are 12 % faster alone (294 us), but their many small
// workgroups hold up the kernels beside them: layer 2034 -> 2118 us.
hipError_t gemm_grouped_k(GemmEpilogue epi, const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0 || a.groups <= 0) return hipSuccess;
  if (epi == kAccF32) return launch_grouped_k<256, 256, 2, 4, kAccF32>(a, s);
  if (epi == kStoreF32) return launch_grouped_k<256, 256, 2, 4, kStoreF32>(a, s);
  if (epi == kAccF32Adam) return launch_grouped_k<256, 256, 2, 4, kAccF32Adam>(a, s);
  if (epi == kStoreF32Adam) return launch_grouped_k<256, 256, 2, 4, kStoreF32Adam>(a, s);
  return hipErrorInvalidValue;
}

GemmPlan gemm_plan(GemmLayout la, GemmLayout lb, long M, long N, long K, size_t part_bytes) {
  const Plan pl = pick_plan(layout_id(la, lb), M, N, K, part_bytes);
  return {kTileM[pl.tile], kTileN[pl.tile], pl.splits, partial_bytes(pl.splits, M, N)};
}

GemmPlan gemm_grouped_m_plan(GemmLayout lb, long rows, long groups, long N, long K) {
  const Tile t = pick_grouped_tile(layout_id(kKC, lb), rows, groups, N, K);
  return {kTileM[t], kTileN[t], 1, 0};
}

size_t gemm_split_bytes(GemmLayout la, GemmLayout lb, long M, long N, long K) {
  return M <= 0 || N <= 0 ? 0 : gemm_plan(la, lb, M, N, K, SIZE_MAX).bytes;
}

hipError_t gemm(GemmLayout la, GemmLayout lb, GemmEpilogue epi, const GemmArgs& a, hipStream_t s,
                float* part, size_t part_bytes) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (la == kKC && lb == kKC) {
    switch (epi) {
      case kStoreBF16: return dispatch_tiles<kKC, kKC, kStoreBF16>(a, s, part, part_bytes);
      case kResidBF16: return dispatch_tiles<kKC, kKC, kResidBF16>(a, s, part, part_bytes);
      case kAccF32: return dispatch_tiles<kKC, kKC, kAccF32>(a, s, part, part_bytes);
      case kStoreF32: return dispatch_tiles<kKC, kKC, kStoreF32>(a, s, part, part_bytes);
      default: break;
    }
  } else if (la == kKC && lb == kMC) {
    switch (epi) {
      case kStoreBF16: return dispatch_tiles<kKC, kMC, kStoreBF16>(a, s, part, part_bytes);
      case kResidBF16: return dispatch_tiles<kKC, kMC, kResidBF16>(a, s, part, part_bytes);
      default: break;
    }
  } else if (la == kMC && lb == kMC) {
    switch (epi) {
      case kAccF32: return dispatch_tiles<kMC, kMC, kAccF32>(a, s, part, part_bytes);
      case kStoreF32: return dispatch_tiles<kMC, kMC, kStoreF32>(a, s, part, part_bytes);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace forge
