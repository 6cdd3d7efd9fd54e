// TEST INFRASTRUCTURE ONLY: where the kernels put and find the saved working
// sets, formed from the packed model as env_rollout_keep, env_recompute and
// env_rollout_grad form them, checked against the env's own block of the buffer.
#include "host_common.h"
extern "C" {
// Returns the number of envs whose accesses leave their block (the first one's
// index in *bad), or -1 if the model is refused.  total: floats of the buffer.
long long kw_check(const sim_model_desc* d, long long* total, long long* bad) {
  Host h;
  if (!make(d, h)) return -1;
  *total = h.P.seg_total;
  *bad = -1;
  const DevModel& M = h.M;
  long long n_bad = 0, end = 0;
  for (int e = 0; e < d->n_envs; ++e) {
    const Env F = make_env(M, e, nullptr, M.n_iters, false), A = make_env(M, e, nullptr, M.n_iters, true);
    const long long base = (long long)A.seg_base(), next = e + 1 < d->n_envs
        ? (long long)make_env(M, e + 1, nullptr, M.n_iters, true).seg_base() : h.P.seg_total;
    const long long stride = dump_stride_of(A.lay.total_fwd, M.n_iters, A.nslot, A.nb);
    const long long hist = A.lay.total_fwd, tail = hist + align4(M.n_iters * A.nslot);
    const long long steps = M.dump == DUMP_TRAJECTORY ? A.T : M.ckpt_every;
    bool ok = base == end && base <= next && base % 4 == 0 && stride % 4 == 0;
    // forward and reverse kernels agree on the layout
    ok = ok && F.lay.total_fwd == A.lay.total_fwd && F.lay.total_fwd % 4 == 0 && F.seg_off == A.seg_off;
    // a step's parts in order, its history and its tail inside the stride
    ok = ok && hist + (long long)M.n_iters * A.nslot <= tail && tail + 3LL * A.nb <= stride;
    // the records of the last joint and of the last contact a lane can hold
    ok = ok && A.jr * A.nj + 4LL * A.ccap <= A.nslot;
    // the last step, and in trajectory mode the loss body's final state after it
    ok = ok && base + steps * stride + (M.dump == DUMP_TRAJECTORY ? 18 : 0) <= next;
    // every checkpoint-to-checkpoint segment of the env
    for (int t0 = 0; t0 < A.T; t0 += M.ckpt_every) {
      const int t1 = std::min(A.T, t0 + M.ckpt_every);
      for (int t : {t0, t1 - 1}) {
        const long long at = base + (M.dump == DUMP_TRAJECTORY ? t : t - t0) * stride;
        for (int it : {0, M.n_iters - 1})
          ok = ok && (M.n_iters == 0 || at + hist + (long long)(it + 1) * A.nslot <= next) && at + stride <= next;
      }
    }
    if (!ok) {
      if (n_bad == 0) *bad = e;
      ++n_bad;
    }
    end = next;
  }
  return n_bad;
}
}
