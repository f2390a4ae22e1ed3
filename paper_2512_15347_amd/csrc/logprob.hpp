// Where the log-probability of a step goes and how it follows from the sum of its squared noise (the policy of paper Eq. 19).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace pg {

struct LogProb { float* logp; float* hist; float* sum; double log_norm; };
// logp[r] = -1/2 s - d (ln C + 1/2 ln 2 pi); history and running sum by original id
__device__ __forceinline__ void finish_logprob(const LogProb& o, int r, int id, double s) {
  const float lp = (float)(-0.5 * s - o.log_norm);
  if (o.logp) o.logp[r] = lp;
  if (o.hist) o.hist[id] = lp;
  if (o.sum) o.sum[id] += lp;
}

}  // namespace pg
