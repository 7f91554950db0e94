// K4: partial (max, sum-exp) records over the draft logits of each request's root row, the
//     input of the draft top-1 confidence p_draft(top1) of Sec. 3.3, Eq. (2).
#pragma once

#include "k_common.h"

namespace asv {

constexpr int kConfPerLane = 32;
constexpr int kConfChunk = kConfPerLane * kWave;   // draft logits per record, one wave each
constexpr int kConfWaves = 4;                      // records per workgroup

struct ConfArgs {
  int N, V;
  const int32_t* req_offsets;
  const float* q;       // draft logits [N][V]
  float* part_m;
  float* part_s;
  int n_conf;           // records per request
  int n_shares;         // shares of the launch (0: none): K1's tile t takes share t
};

__host__ __device__ __forceinline__ int conf_shares(int n_conf) {   // workgroups per request
  return (n_conf + kConfWaves - 1) / kConfWaves;
}

// Share i of a launch: wave w reduces chunk 4 (i mod shares) + w of request i / shares to one (max,
// sum of exp(q - max)) record in one pass: each lane issues its loads (entry lo + 64 k + lane,
// coalesced) before using any, then reduces them in registers. Entries past V read as -inf and
// add nothing. An out-of-range root (malformed offsets, reported by K3) yields an empty record
// and reads nothing. The three parts may lie apart, so that other work covers the loads.
struct ConfShare {
  int b, ch, root, lo, hi;
  bool mine;            // the wave has a record to write
  float x[kConfPerLane];

  __device__ __forceinline__ void begin(const ConfArgs& a, int i, int wave) {
    const int shares = conf_shares(a.n_conf);
    b = i / shares;
    ch = (i % shares) * kConfWaves + wave;
    mine = i < a.n_shares && ch < a.n_conf;
    if (!mine) return;
    root = a.req_offsets[b];
    lo = ch * kConfChunk;
    hi = min(lo + kConfChunk, a.V);
  }
  __device__ __forceinline__ bool readable(const ConfArgs& a) const {
    return root >= 0 && root < a.N;
  }
  __device__ __forceinline__ void load(const ConfArgs& a, int lane) {
    if (!mine || !readable(a)) return;
    const float* row = a.q + (size_t)root * a.V;
#pragma unroll
    for (int k = 0; k < kConfPerLane; ++k) x[k] = row[min(lo + k * kWave + lane, hi - 1)];
  }
  __device__ __forceinline__ void finish(const ConfArgs& a, int lane) {
    if (!mine) return;
    float m = kNegInf, s = 0.f;
    if (readable(a)) {
      m = __builtin_nanf("");    // fmaxf takes the other one: stays when all entries are no numbers
#pragma unroll
      for (int k = 0; k < kConfPerLane; ++k) {
        x[k] = lo + k * kWave + lane < hi ? x[k] : kNegInf;
        m = fmaxf(m, x[k]);
      }
      if (m != kNegInf) {
        const float mb = m * kLog2e;
#pragma unroll
        for (int k = 0; k < kConfPerLane; ++k) s += exp2_rel(fmaf(x[k], kLog2e, -mb));
      }
    }
    const Rec r = rec_wave_reduce_dpp(Rec{m, s, 0});   // all -inf: m = -inf, s = 0
    if (lane == 0) {
      a.part_m[(size_t)b * a.n_conf + ch] = r.m;
      a.part_s[(size_t)b * a.n_conf + ch] = r.s;
    }
  }
};

// A launch of its own, one workgroup per share.
__global__ __launch_bounds__(kConfWaves * kWave)
void k_draft_conf_partial(ConfArgs a) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  ConfShare c;
  c.begin(a, blockIdx.y * gridDim.x + blockIdx.x, wave);
  c.load(a, lane);
  c.finish(a, lane);
}

}  // namespace asv
