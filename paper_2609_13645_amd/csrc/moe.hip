// Routed mixture-of-experts pieces of the layer (the sparse model of App. B,
// Table "H100 architecture configurations": routed experts with top-k
// selection), dropless: every token goes to its top_k experts.
//
//  * route: one wave per token, lane l holds the fp32 logits of experts
//    l, l + 64, l + 128, l + 192 (E <= 256): softmax over all experts, then
//    top_k rounds of wave argmax on a total order of the logits (numeric
//    order, -0 equal to +0, NaN below -inf; ties to the lower expert id), so
//    every index lies in [0, E) whatever the logits hold. Gates are the
//    softmax probabilities of the chosen experts (no renormalisation).
//  * permutation: a counting sort that is deterministic by construction:
//    per-block expert histograms, then each block adds up the histograms
//    itself (the whole scan, in one launch) and assigns ranks in flat
//    (token, slot) order with wave ballots, so the order is expert-major,
//    token ascending, slot ascending.
//  * gather / combine / their backward move whole bf16 rows with 16-byte
//    vectors; every sum over the k slots of a token runs in slot order.
//  * the load-balance auxiliary loss alpha * E * sum_e f_e P_e and its
//    gradient through the softmax (f_e = count_e / (T k) is a constant);
//    the column sums behind P_e are per-block partials of the sort's blocks,
//    added in a fixed order by its second launch.
#include "common.h"
#include "kernels.h"

namespace forge {
namespace {

constexpr int kSortTokens = 128;  // tokens per counting-sort block, at least
constexpr int kSortBlocks = 512;  // counting-sort blocks, at most
constexpr int kMaxE = 256;        // experts (four per lane of a wave)

// ------------------------------------------------------------- routing ----
// Order key of a logit for the top-k choice: larger key = preferred. The
// integer image of the float is monotone in its value; -0 is first made +0
// (they compare equal), NaN gets the lowest key of all, 1, and 0 stands for an
// expert that is taken or absent (-inf, the lowest number, has 0x007FFFFF).
__device__ __forceinline__ uint32_t order_key(float f) {
  if (f == 0.0f) f = 0.0f;
  const int b = __float_as_int(f);
  const uint32_t key = (uint32_t)(b >= 0 ? b : (b ^ 0x7FFFFFFF)) ^ 0x80000000u;
  return f != f ? 1u : key;
}
// Largest value of the wave, uniform: a DPP reduction into lane 63 (row
// shifts, then the rows' last lanes broadcast; lanes without a source take
// the identity 0).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t max_dpp(uint32_t v) {
  const uint32_t w = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
  return w > v ? w : v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max_dpp<0x111, 0xF>(v);  // row_shr 1, 2, 4, 8
  v = max_dpp<0x112, 0xF>(v);
  v = max_dpp<0x114, 0xF>(v);
  v = max_dpp<0x118, 0xF>(v);
  v = max_dpp<0x142, 0xA>(v);  // row_bcast 15 into rows 1 and 3
  v = max_dpp<0x143, 0xC>(v);  // row_bcast 31 into rows 2 and 3
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// NS: expert slots per lane (E <= 64 NS). Latency-bound, one wave per token:
// each of the k rounds is one DPP maximum of 32-bit keys and a ballot that
// finds its lowest expert (64-bit keys through LDS shuffles before: 8192
// tokens, 64 experts, top 8 in 15 us).
template <int NS>
__global__ __launch_bounds__(256) void route_k(const float* __restrict__ logits, int T, int E,
                                               int k, int32_t* __restrict__ idx,
                                               float* __restrict__ gates,
                                               float* __restrict__ probs) {
  const int lane = threadIdx.x & 63;
  const long t = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  float l[NS], p[NS];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int e = lane + 64 * i;
    l[i] = e < E ? logits[t * E + e] : -INFINITY;
    mx = fmaxf(mx, l[i]);
  }
  mx = wave_max(mx);
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int e = lane + 64 * i;
    p[i] = e < E ? __expf(l[i] - mx) : 0.0f;
    sum += p[i];
  }
  sum = wave_sum(sum);
  uint32_t key[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int e = lane + 64 * i;
    p[i] /= sum;
    if (e < E) probs[t * E + e] = p[i];
    key[i] = e < E ? order_key(l[i]) : 0u;
  }
  // lane j % 64 keeps choice j; every 64 choices (and the last ones) are
  // stored together
  int my_e = 0;
  float my_g = 0.0f;
  for (int j = 0; j < k; ++j) {
    uint32_t best = key[0];
#pragma unroll
    for (int i = 1; i < NS; ++i) best = key[i] > best ? key[i] : best;
    best = wave_max_u32(best);
    // k <= E, so a real candidate is left in every round; the lowest slot
    // (then lane) that holds the key is the lowest expert id
    int e = 0;
    float g = 0.0f;
    bool found = false;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const uint64_t hit = __ballot(key[i] == best);
      if (!found && hit) {
        found = true;
        const int o = __ffsll((unsigned long long)hit) - 1;
        e = o + 64 * i;
        g = __builtin_bit_cast(
            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, p[i]), o));
        if (lane == o) key[i] = 0u;
      }
    }
    if (lane == (j & 63)) {
      my_e = e;
      my_g = g;
    }
    if ((j & 63) == 63 || j == k - 1) {
      const int j0 = j & ~63;
      if (lane <= (j & 63)) {
        idx[t * k + j0 + lane] = my_e;
        gates[t * k + j0 + lane] = my_g;
      }
    }
  }
}

// Per-block expert histogram of the flat (token, slot) entries of `tok`
// tokens (entries outside [0, E) are not counted) and, with probs, the block's
// column sums of the router probabilities, colsum[block][e]: 256 / E groups of
// threads sum interleaved tokens, the groups in order.
__global__ __launch_bounds__(256) void sort_count_k(const int32_t* __restrict__ idx, int T, int E,
                                                    int k, int tok,
                                                    int32_t* __restrict__ block_counts,
                                                    const float* __restrict__ probs,
                                                    float* __restrict__ colsum) {
  __shared__ int hist[kMaxE];
  __shared__ float part[256];
  hist[threadIdx.x] = 0;
  __syncthreads();
  const long t0 = (long)blockIdx.x * tok;
  const long t1 = min((long)T, t0 + tok);
  for (long f = t0 * k + threadIdx.x; f < t1 * k; f += blockDim.x) {
    const int e = idx[f];
    if ((unsigned)e < (unsigned)E) atomicAdd(&hist[e], 1);
  }
  if (probs) {
    const int groups = 256 / E, grp = threadIdx.x / E, e = threadIdx.x % E;
    float sum = 0.0f;
    if (grp < groups) {
#pragma unroll 8
      for (long t = t0 + grp; t < t1; t += groups) sum += probs[t * E + e];
    }
    part[threadIdx.x] = sum;
    __syncthreads();
    if (threadIdx.x < E) {
      for (int gq = 1; gq < groups; ++gq) sum += part[gq * E + threadIdx.x];
      colsum[(long)blockIdx.x * E + threadIdx.x] = sum;
    }
  }
  __syncthreads();
  if (threadIdx.x < E) block_counts[(long)blockIdx.x * E + threadIdx.x] = hist[threadIdx.x];
}

// Scan and scatter. Every block adds up the nblk histograms itself (coalesced,
// all loads in flight; at most kSortBlocks of them, from L2), which takes the
// place of a one-block scan launch between the two kernels (16 us at 64 blocks
// of 64 experts, a chain of dependent loads); block 0 writes counts and
// offsets (and, with colsum, adds the load-balance loss to aux). Then eight
// waves share the block's entries in flat order: each counts its own, the
// waves' bases follow in wave order, and each walks its entries 64 at a time:
// the lanes holding the same expert are found with one ballot per bit of the
// expert id (E <= 256: eight bits), so each lane's rank among the earlier
// lanes of its expert is a popcount, and the group's lowest lane advances the
// expert's running position. Entries outside [0, E) are skipped.
// perm[pos] = flat entry, pos_of[flat entry] = pos.
constexpr int kScatterWaves = 8;
__global__ __launch_bounds__(64 * kScatterWaves) void sort_scatter_k(
    const int32_t* __restrict__ idx, int T, int E, int k, int tok, int nblk,
    const int32_t* __restrict__ block_counts, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int32_t* __restrict__ pos_of,
    const float* __restrict__ colsum, float alpha, float* __restrict__ aux) {
  constexpr int NT = 64 * kScatterWaves;
  __shared__ int tot[NT], pre[NT], off[kMaxE];
  __shared__ int run[kScatterWaves][kMaxE];
  __shared__ float fpart[NT];
  __shared__ float term[kScatterWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int groups = NT / E, grp = tid / E, ge = tid % E;
  const int me = blockIdx.x;
  int all = 0, before = 0;
  if (grp < groups) {
#pragma unroll 8
    for (int b = grp; b < nblk; b += groups) {
      const int c = block_counts[(long)b * E + ge];
      all += c;
      before += b < me ? c : 0;
    }
  }
  tot[tid] = all;
  pre[tid] = before;
  for (int i = tid; i < kScatterWaves * kMaxE; i += NT) (&run[0][0])[i] = 0;
  __syncthreads();
  if (tid < E) {
    for (int gq = 1; gq < groups; ++gq) {
      all += tot[gq * E + tid];
      before += pre[gq * E + tid];
    }
  }
  __syncthreads();
  if (tid < kMaxE) {
    tot[tid] = tid < E ? all : 0;
    pre[tid] = before;
  }
  // each wave's own histogram (entries of a wave: whole rounds of 64)
  const long f0 = (long)me * tok * k, f1 = min((long)T * k, f0 + (long)tok * k);
  const long per = ((f1 - f0 + kScatterWaves * 64 - 1) / (kScatterWaves * 64)) * 64;
  const long w0 = min(f1, f0 + wave * per), w1 = min(f1, w0 + per);
  for (long f = w0 + lane; f < w1; f += 64) {
    const int e = idx[f];
    if ((unsigned)e < (unsigned)E) atomicAdd(&run[wave][e], 1);
  }
  __syncthreads();
  if (wave == 0) {  // exclusive scan over the experts, four to a lane
    int c[4], s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      c[i] = tot[lane * 4 + i];
      s += c[i];
    }
    int incl = s;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int u = __shfl_up(incl, d, 64);
      if (lane >= d) incl += u;
    }
    int at = incl - s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      off[lane * 4 + i] = at;
      at += c[i];
    }
  }
  __syncthreads();
  if (tid < E) {
    int at = off[tid] + pre[tid];
#pragma unroll
    for (int w = 0; w < kScatterWaves; ++w) {
      const int n = run[w][tid];
      run[w][tid] = at;
      at += n;
    }
    if (me == 0) {
      counts[tid] = tot[tid];
      offsets[tid] = off[tid];
      if (tid == E - 1) offsets[E] = off[tid] + tot[tid];
    }
  }
  __syncthreads();
  int* mine = run[wave];
  const uint64_t below = (1ull << lane) - 1ull;
  for (long base = w0; base < w1; base += 64) {
    const long f = base + lane;
    const int raw = f < w1 ? idx[f] : -1;
    const bool ok = (unsigned)raw < (unsigned)E;
    const int e = ok ? raw : 0;
    uint64_t same = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint64_t ones = __ballot(ok && ((e >> b) & 1));
      same &= ((e >> b) & 1) ? ones : ~ones;
    }
    const int pos = mine[e] + __popcll(same & below);  // every lane reads before any update
    __builtin_amdgcn_wave_barrier();
    if (ok) {
      perm[pos] = (int32_t)f;
      pos_of[f] = pos;
      if ((same & below) == 0) mine[e] += __popcll(same);
    }
    __builtin_amdgcn_wave_barrier();
  }
  // aux += alpha E sum_e f_e P_e with P_e = sum_t p[t, e] / T
  if (me == 0 && colsum) {
    float c = 0.0f;
    if (grp < groups) {
#pragma unroll 8
      for (int b = grp; b < nblk; b += groups) c += colsum[(long)b * E + ge];
    }
    fpart[tid] = c;
    __syncthreads();
    if (tid < E)
      for (int gq = 1; gq < groups; ++gq) c += fpart[gq * E + tid];
    const float fe = tid < E ? (float)tot[tid] / ((float)T * k) : 0.0f;
    const float w = wave_sum(tid < E ? fe * c : 0.0f);
    if (lane == 0) term[wave] = w;
    __syncthreads();
    if (tid == 0)
      aux[0] += alpha * (float)E * ((term[0] + term[1]) + (term[2] + term[3])) / (float)T;
  }
}

// xs[pos] = b[perm[pos] / k]; one thread per 8 elements.
__global__ __launch_bounds__(256) void gather_k(const bf16_t* __restrict__ b,
                                                const int32_t* __restrict__ perm, long rows, int h,
                                                int k, bf16_t* __restrict__ xs) {
  const int cpr = h / 8;
  const long id = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= rows * cpr) return;
  const long r = id / cpr;
  const int c = (int)(id % cpr);
  const long t = perm[r] / k;
  reinterpret_cast<uint4*>(xs + r * h)[c] = reinterpret_cast<const uint4*>(b + t * h)[c];
}

// out[t] = h1[t] + scale * sum_j gate[t, j] * ys[pos_of[t k + j]] (fp32,
// slot order; scale: the branch scale of muP, 1 otherwise).
__global__ __launch_bounds__(256) void combine_k(const bf16_t* __restrict__ ys,
                                                 const float* __restrict__ gates,
                                                 const int32_t* __restrict__ pos_of,
                                                 const bf16_t* __restrict__ h1, long T, int h,
                                                 int k, float scale, bf16_t* __restrict__ out) {
  const int cpr = h / 8;
  const long id = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= T * cpr) return;
  const long t = id / cpr;
  const int c = (int)(id % cpr);
  float acc[8] = {};
#pragma unroll 4
  for (int j = 0; j < k; ++j) {
    const float g = gates[t * k + j];
    float y[8];
    unpack8(reinterpret_cast<const uint4*>(ys + (long)pos_of[t * k + j] * h)[c], y);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += g * y[e];
  }
  float r[8];
  unpack8(reinterpret_cast<const uint4*>(h1 + t * h)[c], r);
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] += scale * acc[e];
  reinterpret_cast<uint4*>(out + t * h)[c] = pack8(r);
}

// Backward of combine for one token per block: dgate[t, j] = scale dy_t .
// ys_row and dys_row = scale gate[t, j] dy_t. k <= 16.
__global__ __launch_bounds__(256) void combine_bwd_k(const bf16_t* __restrict__ ys,
                                                     const float* __restrict__ gates,
                                                     const int32_t* __restrict__ pos_of,
                                                     const bf16_t* __restrict__ dy, int h, int k,
                                                     float scale, float* __restrict__ dgate,
                                                     bf16_t* __restrict__ dys) {
  __shared__ float red[4][16];
  const long t = blockIdx.x;
  const int cpr = h / 8;
  float dot[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) dot[j] = 0.0f;
  for (int c = threadIdx.x; c < cpr; c += blockDim.x) {
    float d[8];
    unpack8(reinterpret_cast<const uint4*>(dy + t * h)[c], d);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (j < k) {
        const long row = pos_of[t * k + j];
        float y[8], o[8];
        unpack8(reinterpret_cast<const uint4*>(ys + row * h)[c], y);
        const float g = scale * gates[t * k + j];
        float s = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          s += d[e] * y[e];
          o[e] = g * d[e];
        }
        dot[j] += s;
        reinterpret_cast<uint4*>(dys + row * h)[c] = pack8(o);
      }
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    if (j < k) {
      const float s = wave_sum(dot[j]);
      if (lane == 0) red[wave][j] = s;
    }
  }
  __syncthreads();
  if (threadIdx.x < k) {
    const int j = threadIdx.x;
    dgate[t * k + j] = scale * ((red[0][j] + red[1][j]) + (red[2][j] + red[3][j]));
  }
}

// db_s[t] = sum_j dxs[pos_of[t k + j]] (fp32 in slot order, one rounding).
__global__ __launch_bounds__(256) void scatter_back_k(const bf16_t* __restrict__ dxs,
                                                      const int32_t* __restrict__ pos_of, long T,
                                                      int h, int k, bf16_t* __restrict__ db) {
  const int cpr = h / 8;
  const long id = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= T * cpr) return;
  const long t = id / cpr;
  const int c = (int)(id % cpr);
  float acc[8] = {};
#pragma unroll 4
  for (int j = 0; j < k; ++j) {
    float y[8];
    unpack8(reinterpret_cast<const uint4*>(dxs + (long)pos_of[t * k + j] * h)[c], y);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += y[e];
  }
  reinterpret_cast<uint4*>(db + t * h)[c] = pack8(acc);
}

// dl[t, e] = p (dp - sum_e p dp) with dp = dgate on chosen experts plus the
// aux term alpha E f_e / T on every expert; written as bf16 for the router
// data / weight gradient products. One wave per token, lane l holding
// experts l + 64 i; lane j loads choice j, and the choices are then read from
// its registers (k <= 64).
template <int NS>
__global__ __launch_bounds__(256) void router_bwd_k(const float* __restrict__ probs,
                                                    const int32_t* __restrict__ idx,
                                                    const float* __restrict__ dgate,
                                                    const int32_t* __restrict__ counts, int T,
                                                    int E, int k, float alpha,
                                                    bf16_t* __restrict__ dl) {
  const int lane = threadIdx.x & 63;
  const long t = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const int my_e = lane < k ? idx[t * k + lane] : -1;
  const int my_d = lane < k ? __float_as_int(dgate[t * k + lane]) : 0;
  float p[NS], dp[NS];
  float part = 0.0f;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int e = lane + 64 * i;
    p[i] = e < E ? probs[t * E + e] : 0.0f;
    dp[i] = e < E ? alpha * (float)E * ((float)counts[e] / ((float)T * k)) / (float)T : 0.0f;
  }
  for (int j = 0; j < k; ++j) {
    const int e = __builtin_amdgcn_readlane(my_e, j);
    const float d = __int_as_float(__builtin_amdgcn_readlane(my_d, j));
#pragma unroll
    for (int i = 0; i < NS; ++i) dp[i] += lane + 64 * i == e ? d : 0.0f;
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) part += p[i] * dp[i];
  const float dot = wave_sum(part);
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int e = lane + 64 * i;
    if (e < E) dl[t * E + e] = f2bf(p[i] * (dp[i] - dot));
  }
}

inline unsigned nblocks(long work, int threads) { return (unsigned)((work + threads - 1) / threads); }

}  // namespace

namespace {
// tokens of a counting-sort block: every block reads every block's histogram,
// so their number is bounded
int sort_tokens(int T) {
  const long most = (long)kSortTokens * kSortBlocks;
  return kSortTokens * (int)(((long)T + most - 1) / most);
}
}  // namespace

int moe_sort_blocks(int T) {
  const int tok = sort_tokens(T);
  return (int)(((long)T + tok - 1) / tok);
}

hipError_t moe_route(const float* logits, int T, int E, int k, int32_t* idx, float* gates,
                     float* probs, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const dim3 grid(nblocks(T, 4)), block(256);
  if (E <= 64) hipLaunchKernelGGL(route_k<1>, grid, block, 0, s, logits, T, E, k, idx, gates, probs);
  else if (E <= 128) hipLaunchKernelGGL(route_k<2>, grid, block, 0, s, logits, T, E, k, idx, gates, probs);
  else if (E <= 192) hipLaunchKernelGGL(route_k<3>, grid, block, 0, s, logits, T, E, k, idx, gates, probs);
  else hipLaunchKernelGGL(route_k<4>, grid, block, 0, s, logits, T, E, k, idx, gates, probs);
  return hipGetLastError();
}

hipError_t moe_sort(const int32_t* idx, int T, int E, int k, int32_t* block_counts,
                    int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* pos_of,
                    hipStream_t s, const float* probs, float alpha, float* colsum, float* aux) {
  if (T <= 0) return hipSuccess;
  const int nb = moe_sort_blocks(T), tok = sort_tokens(T);
  if (!aux) probs = colsum = nullptr;
  hipLaunchKernelGGL(sort_count_k, dim3(nb), dim3(256), 0, s, idx, T, E, k, tok, block_counts,
                     probs, colsum);
  hipLaunchKernelGGL(sort_scatter_k, dim3(nb), dim3(64 * kScatterWaves), 0, s, idx, T, E, k, tok,
                     nb, block_counts, counts, offsets, perm, pos_of, colsum, alpha, aux);
  return hipGetLastError();
}

hipError_t moe_gather(const uint16_t* b, const int32_t* perm, long rows, int h, int k,
                      uint16_t* xs, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(gather_k, dim3(nblocks(rows * (h / 8), 256)), dim3(256), 0, s, b, perm, rows, h, k, xs);
  return hipGetLastError();
}

hipError_t moe_combine(const uint16_t* ys, const float* gates, const int32_t* pos_of,
                       const uint16_t* h1, long T, int h, int k, float scale, uint16_t* out,
                       hipStream_t s) {
  if (T <= 0) return hipSuccess;
  hipLaunchKernelGGL(combine_k, dim3(nblocks(T * (h / 8), 256)), dim3(256), 0, s, ys, gates, pos_of, h1, T, h, k, scale, out);
  return hipGetLastError();
}

hipError_t moe_combine_bwd(const uint16_t* ys, const float* gates, const int32_t* pos_of,
                           const uint16_t* dy, long T, int h, int k, float scale, float* dgate,
                           uint16_t* dys, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  hipLaunchKernelGGL(combine_bwd_k, dim3((unsigned)T), dim3(256), 0, s, ys, gates, pos_of, dy, h, k, scale, dgate, dys);
  return hipGetLastError();
}

hipError_t moe_scatter_back(const uint16_t* dxs, const int32_t* pos_of, long T, int h, int k,
                            uint16_t* db, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  hipLaunchKernelGGL(scatter_back_k, dim3(nblocks(T * (h / 8), 256)), dim3(256), 0, s, dxs, pos_of, T, h, k, db);
  return hipGetLastError();
}

hipError_t moe_router_bwd(const float* probs, const int32_t* idx, const float* dgate,
                          const int32_t* counts, int T, int E, int k, float alpha, uint16_t* dl,
                          hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const dim3 grid(nblocks(T, 4)), block(256);
#define FORGE_ROUTER_BWD(NS) \
  hipLaunchKernelGGL(router_bwd_k<NS>, grid, block, 0, s, probs, idx, dgate, counts, T, E, k, alpha, dl)
  if (E <= 64) FORGE_ROUTER_BWD(1);
  else if (E <= 128) FORGE_ROUTER_BWD(2);
  else if (E <= 192) FORGE_ROUTER_BWD(3);
  else FORGE_ROUTER_BWD(4);
#undef FORGE_ROUTER_BWD
  return hipGetLastError();
}

}  // namespace forge
