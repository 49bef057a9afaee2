// k_select.hip -- keep / drop partition of PruneKV (Algorithm 1, Step 1 and
// Step 3): one ranking per (layer, sequence, kv head) ordered by score
// descending then token index ascending; the first k tokens are kept, the next
// n_surv - k are dropped (their values get fused), the rest are discarded.
//
// One workgroup per unit (256 to 1024 threads, by the longest sequence); each
// thread holds a contiguous run of up to PER scores in registers.  Scores are
// non-negative fp32, so their bit patterns order like the values.  The k-th
// and n_surv-th largest bit patterns are found exactly by a most-significant-
// digit radix select over the 31 value bits (digits of 11, 10 and 10 bits,
// both cuts in the same passes): the keys that still match a cut's prefix are
// counted by digit in an LDS histogram, and two waves scan the histograms for
// the bin holding the wanted rank.  Ties at a threshold go to the lowest
// indices, and one block-wide prefix sum (DPP wave scans) gives every thread
// the places of its kept and dropped tokens, in ascending token order.
//
// A chain of LDS round trips and barriers bounds it, so the digits are wide
// (three passes; the first one's 11 bits also spread the scores, which share
// few exponents, over several times more bins than 8 bits do), all histograms
// are cleared while the scores are on their way, and the ties still wanted
// and the dropped tokens' places follow from the passes and the one scan.
// Against digits of 8, 8, 8 and 7 bits in a histogram a wave and two scans
// (stage times, 5 us of them the timing's own): 512 keys 10.2 -> 8.5 us, 3136
// 14.2 -> 11.0, 12544 22.4 -> 18.0, eight sequences of 14k to 23k (672 units)
// 102 -> 79.
#include "vc_device.h"
#include "vc_internal.h"

namespace vc {

namespace {

// Exclusive prefix over the block of four counters per thread.
template <int kWaves>
__device__ __forceinline__ void block_scan4(const uint32_t v[4], uint32_t excl[4], uint32_t (*wt)[kWaves]) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint32_t inc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    inc[c] = wave_incl_scan(v[c]);
    if (lane == 63) wt[c][w] = inc[c];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    uint32_t before = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) before += q < w ? wt[c][q] : 0u;
    excl[c] = before + inc[c] - v[c];
  }
}

// The bin, in descending order, that holds rank r (1-based) among the
// histogram's 64 PER bins, and the rank within it; (0, 0) for r = 0.  Whole
// wave: lane l sums bins PER l .. PER l + PER - 1 of the descending order, then
// the hit lane's bins are spread over the lanes.
template <int PER>
__device__ __forceinline__ void find_bin(const uint32_t *hist, uint32_t r, uint32_t *res) {
  constexpr int kBins = 64 * PER;
  const int lane = threadIdx.x & 63;
  uint32_t tot = 0u;
#pragma unroll
  for (int i = 0; i < PER; i += 4) {
    const u32x4 h = *reinterpret_cast<const u32x4 *>(hist + kBins - PER * (lane + 1) + i);
    tot += (h.x + h.y) + (h.z + h.w);
  }
  const uint32_t incl = wave_incl_scan(tot);
  const uint64_t hit = __builtin_amdgcn_ballot_w64(r > 0 && incl - tot < r && r <= incl);
  uint32_t dg = 0u, nr = 0u;
  if (hit) {
    const int src = __builtin_ctzll(hit);
    const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(incl - tot), src);
    const int bin = kBins - 1 - PER * src - lane;  // descending within the lane's bins
    const uint32_t h = lane < PER ? hist[max(bin, 0)] : 0u;
    const uint32_t in2 = wave_incl_scan(h) + before;
    const uint64_t hit2 = __builtin_amdgcn_ballot_w64(in2 - h < r && r <= in2);
    const int src2 = __builtin_ctzll(hit2);
    dg = (uint32_t)(kBins - 1 - PER * src - src2);
    nr = r - (uint32_t)__builtin_amdgcn_readlane((int)(in2 - h), src2);
  }
  if (lane == 0) {
    res[0] = dg;
    res[1] = nr;
  }
}

// One radix pass for both cuts over the digit of `64 PERB`-bin histograms at
// bit `sh`.  On entry pre[c] holds the cut's value bits above the digit and
// rank[c] the wanted rank (1-based, descending) among the keys sharing them;
// on exit the digit is fixed and the rank is relative to it.  A rank of 0
// (nothing wanted) stays 0.  While both cuts share their prefix (always in
// the first pass), one histogram serves both.  hist: zeroed.
template <int PERB, int PER>
__device__ __forceinline__ void radix_pass(const uint32_t (&key)[PER], int cnt, int sh, uint32_t (&pre)[2],
                                           uint32_t (&rank)[2], uint32_t *hist, uint32_t (*res)[2]) {
  constexpr int kBins = 64 * PERB;
  const int w = threadIdx.x >> 6;
  const uint32_t p0 = pre[0] / kBins >> sh, p1 = pre[1] / kBins >> sh;
  const bool same = p0 == p1;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (i < cnt) {
      const uint32_t hi = key[i] / kBins >> sh, dg = (key[i] >> sh) & (kBins - 1);
      if (hi == p0) atomicAdd(&hist[dg], 1u);
      if (!same && hi == p1) atomicAdd(&hist[kBins + dg], 1u);
    }
  }
  __syncthreads();
  if (w < 2) find_bin<PERB>(hist + (same || w == 0 ? 0 : kBins), w ? rank[1] : rank[0], res[w]);
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    pre[c] |= res[c][0] << sh;
    rank[c] = res[c][1];
  }
}

template <int kThreads, int PER>
__global__ __launch_bounds__(kThreads) void k_select(PrunePlan p) {
  constexpr int kWaves = kThreads / 64;
  // Digit counts: 2048 bins of the first pass, two times 1024 (a cut each) of
  // the second and of the third.
  constexpr int kHist = 2048 * 3;
  __shared__ __attribute__((aligned(16))) uint32_t hist[kHist];
  __shared__ uint32_t res[3][2][2];  // per pass and cut: digit, rank within it
  __shared__ uint32_t wt[4][kWaves];

  const int u = blockIdx.x;  // ((l * B) + b) * Hkv + g, l < h
  const int g = u % p.Hkv;
  const int b = (u / p.Hkv) % p.B;
  const int l = u / (p.Hkv * p.B);
  // Every parameter of the unit, output pointers included, in one batch of
  // loads.  There is no early exit: a unit with n_surv = 0 (k = 0) finds no
  // kept or dropped token below and writes nothing, and without the branch
  // the loads are not deferred behind the first one.
  const int nsv = ldg(p.ns + b * p.L + l);
  const int n = ldg(p.nb + b);
  const int k = ldg(p.kk + b * p.L + l);
  const int64_t toff = ldg(p.toff + b);
  const uint64_t idx_base = ldg(p.lp + LP_IDX * p.L + l), drop_base = ldg(p.lp + LP_DROP * p.L + l);
  const int job = ldg(&p.funit[max(min(u, p.nfrec - 1), 0)].job);  // (not used without kept tokens)
  const int64_t orow = ldg(p.orow + l * (p.B + 1) + b), drow = ldg(p.drow + l * (p.B + 1) + b);
  const int r = nsv - k;

  const float *S = p.mode ? p.gs + toff
                          : p.S + (int64_t)l * p.Ntot * p.Hkv + toff * p.Hkv + (int64_t)g * n;
  const int tid = threadIdx.x;
  const int per = (n + kThreads - 1) / kThreads;  // <= PER
  const int v0 = tid * per;
  const int cnt = max(0, min(per, n - v0));

  // Bit patterns of non-negative floats order like the values.  A set sign
  // bit (only possible from non-finite inputs) is mapped to the top of the
  // 31-bit range so every count below stays consistent.  Slots past the
  // thread's run hold 0 and are never counted.
  uint32_t key[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const uint32_t x = (i < cnt) ? __float_as_uint(ldg(S + v0 + i)) : 0u;
    key[i] = (x & 0x80000000u) ? 0x7FFFFFFFu : x;
  }

  for (int i = 4 * tid; i < kHist; i += 4 * kThreads) *reinterpret_cast<u32x4 *>(hist + i) = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();

  // Thresholds: the k-th and n_surv-th largest bit patterns (none wanted:
  // above every key).
  uint32_t pre[2] = {0u, 0u}, rank[2] = {(uint32_t)k, (uint32_t)nsv};
  radix_pass<32, PER>(key, cnt, 20, pre, rank, hist, res[0]);
  radix_pass<16, PER>(key, cnt, 10, pre, rank, hist + 2048, res[1]);
  radix_pass<16, PER>(key, cnt, 0, pre, rank, hist + 4096, res[2]);
  const uint32_t tk = k > 0 ? pre[0] : 0xFFFFFFFFu, ts = nsv > 0 ? pre[1] : 0xFFFFFFFFu;

  // Counts above and at each threshold; ties fill in ascending index order.
  uint32_t c4[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (i < cnt) {
      c4[0] += key[i] > tk;
      c4[1] += key[i] == tk;
      c4[2] += key[i] > ts;
      c4[3] += key[i] == ts;
    }
  uint32_t ex[4];
  block_scan4<kWaves>(c4, ex, wt);
  // The ranks within the thresholds are the ties wanted.  The kept tokens are
  // among the survivors, so the dropped ones before a thread are the
  // difference of both counts.
  const uint32_t need_k = rank[0], need_s = rank[1];
  uint32_t ek = ex[1], es = ex[3];
  uint32_t pk = ex[0] + min(ek, need_k), pd = ex[2] + min(es, need_s) - pk;

  int32_t *idx = reinterpret_cast<int32_t *>(idx_base) + orow + (int64_t)g * k;
  int32_t *drop = reinterpret_cast<int32_t *>(drop_base) + drow + (int64_t)g * r;
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (i < cnt) {
      const uint32_t x = key[i];
      const bool kp = x > tk || (x == tk && ek < need_k);
      const bool sv = x > ts || (x == ts && es < need_s);
      ek += x == tk;
      es += x == ts;
      if (kp) {
        if (pk < (uint32_t)k) {
          stg(idx + pk, (int32_t)(v0 + i));
          // The first kept token of a fusion job: dropped tokens before it.
          if (pk % kFuseRows == 0) stg(p.jstart + job + pk / kFuseRows, (int32_t)pd);
        }
        ++pk;
      } else if (sv) {
        if (pd < (uint32_t)r) stg(drop + pd, (int32_t)(v0 + i));
        ++pd;
      }
    }
}

}  // namespace

hipError_t launch_select(const PrunePlan &p, hipStream_t st) {
  const uint32_t grid = (uint32_t)p.h * p.B * p.Hkv;
  if (grid == 0) return hipSuccess;
  // 256 threads hold up to 8 scores each, then 512 and 1024 threads up to 16,
  // then 1024 threads up to 32.  Fewer scores per thread shorten each radix
  // pass; more waves lengthen the barriers and the scan, and leave fewer units
  // room on a CU.  Stage times in us (84 units a sequence) with 256, 512 and
  // 1024 threads: 512 keys 9.0, 10.2, 10.5; 1568 11.1, 11.2, 11.7; 2048 11.9,
  // 11.5, 11.7; eight sequences of 1500 15.2, 17.0, 29.8; 3136 14.3, 12.9, 13.3;
  // eight of 3136 20.8, 20.5, 33.4; 6000 (512, 1024) 16.3, 15.5; 8192 20.2, 19.2.
  if (p.nmax <= 256 * 8)
    hipLaunchKernelGGL((k_select<256, 8>), dim3(grid), dim3(256), 0, st, p);
  else if (p.nmax <= 512 * 16)
    hipLaunchKernelGGL((k_select<512, 16>), dim3(grid), dim3(512), 0, st, p);
  else if (p.nmax <= 1024 * 16)
    hipLaunchKernelGGL((k_select<1024, 16>), dim3(grid), dim3(1024), 0, st, p);
  else
    hipLaunchKernelGGL((k_select<1024, 32>), dim3(grid), dim3(1024), 0, st, p);
  return hipGetLastError();
}

}  // namespace vc
