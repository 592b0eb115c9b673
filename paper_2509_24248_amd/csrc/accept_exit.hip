// Stages 4 and 5 of the round (Alg. 1): greedy acceptance of the draft block against the
// target's argmax tokens, smoothing of the three exit signals (Appendix, EWMA with
// alpha = 0.1, or one of the appendix's other smoothers), the stop thresholds (Appendix, "Stop Threshold") and the step-split gate
// with truncation (Sec. 3.3 "Stopping Conditions").  One wave per sequence: the work is
// a few dozen integer operations, so the kernel costs one launch and nothing else, which
// is the point the paper makes against probing-based exits.
#include "common.hpp"
#include "kernels.hpp"

namespace sx {

namespace {

__device__ __forceinline__ bool in_sorted(const int32_t* a, int n, int32_t key) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    const int32_t v = a[mid];
    if (v == key) return true;
    if (v < key) lo = mid + 1; else hi = mid;
  }
  return false;
}

// Lane c holds node c of the block (n_q <= 64); everything a sequence needs is requested at once, and the walk along
// the tree, the gate and the cut run on shuffles and ballots.  (One thread per sequence, which followed the tree
// through memory, took 10.9 us for a 16-node tree: each step waits for the load of the one before.  This takes 2.8 us.)
__global__ __launch_bounds__(64) void k_accept_exit(const ExitArgs a) {
  const int b = blockIdx.x;
  const int lane = threadIdx.x;
  const int n = a.n_q;
  const bool node_ok = lane < n;
  const size_t at = static_cast<size_t>(b) * n + (node_ok ? lane : 0);
  const int32_t tok = a.block_tok[at], am = a.target_argmax[at];
  const int par = a.parent ? a.parent[at] : lane - 1;
  const int j = lane < 3 ? lane : 2;                  // signal of this lane (lanes from 3 on repeat the last one)
  const float sig = a.sig[b * 3 + j];
  float x = a.ewma[b * 3 + j];
  const int n_obs = a.n_obs[b], L = a.ctx_len[b];
  int thinking = a.is_thinking[b];
  // membership of every node's token in the split set: one set entry per lane, or a search for large sets
  int32_t split_entry = 0;
  if (a.S <= 64 && lane < a.S) split_entry = a.split_tok[lane];

  // ---- smoothing (Appendix, "Signal Smoothing"); the first observation seeds x
  //  EWMA       x_t = alpha s_t + (1 - alpha) x_{t-1}
  //  window     mean of the last n = min(N, observations) values, kept in a ring of N
  //  momentum   latest value + mean of the n-1 differences between the last n values; the
  //             differences telescope to (latest - oldest of the ring) / (n - 1)
  //  paragraph  mean of the values since the last paragraph end: a compensated running sum
  //             (words 0, 1 of the signal's row) and a count (word 2 of row 0)
  float* hist = a.smooth_state ? a.smooth_state + static_cast<size_t>(b) * kSmoothWords : nullptr;
  if (thinking && lane < 3) {
    const int seen = max(n_obs, 0);        // caller-owned state: a negative count must not reach the ring index
    const int N = a.window;
    const int cnt = min(seen + 1, N);
    const float s = sig;
    float* h = hist + 16 * j;
    if (a.smoother == 0) {
      x = seen == 0 ? s : fmaf(1.0f - a.alpha, x, __fmul_rn(a.alpha, s));
    } else if (a.smoother == 1) {
      x = s;
    } else if (a.smoother == 2 || a.smoother == 3) {
      h[seen % N] = s;
      const float oldest = h[(seen + 1 - cnt) % N];
      if (a.smoother == 2) {
        float sum = 0.f;
        for (int i = seen + 1 - cnt; i <= seen; ++i) sum += h[i % N];
        x = sum / static_cast<float>(cnt);
      } else {
        x = cnt == 1 ? s : s + (s - oldest) / static_cast<float>(cnt - 1);
      }
    } else {
      const int par_count = __float_as_int(hist[2]) + 1;
      // Kahan step: the mean of a long paragraph keeps full float accuracy
      const float y = s - h[1];
      const float t = __fadd_rn(h[0], y);
      h[1] = __fsub_rn(__fsub_rn(t, h[0]), y);
      h[0] = t;
      x = t / static_cast<float>(par_count);
      if (lane == 0) hist[2] = __int_as_float(par_count);
    }
    a.ewma[b * 3 + j] = x;
    if (lane == 0) a.n_obs[b] = seen + 1;
  }
  const float x0 = __shfl(x, 0, 64), x1 = __shfl(x, 1, 64), x2 = __shfl(x, 2, 64);

  // ---- acceptance: follow matching children from the root; lane i of `path` holds the i-th accepted node
  int cur = 0, len = 0, path = -1;
  while (true) {
    const int32_t want = __shfl(am, cur, 64);
    const uint64_t kids = __builtin_amdgcn_ballot_w64(node_ok && lane > cur && par == cur && tok == want);
    if (!kids) break;
    cur = __ffsll(static_cast<unsigned long long>(kids)) - 1;
    if (lane == len) path = cur;
    ++len;
  }
  int32_t t_rec = __shfl(am, cur, 64);

  // ---- exit gate
  bool pass = true;
  if (a.signal_mask & 1u) pass = pass && (x0 > a.thr_conf);
  if (a.signal_mask & 2u) pass = pass && (x1 > a.thr_prog);
  if (a.signal_mask & 4u) pass = pass && (x2 < a.thr_rem);
  int flag = 0;
  if (thinking && (pass || a.smoother == 4)) {
    bool in_set = false;
    if (a.S <= 64) {
      for (int i = 0; i < a.S; ++i) in_set |= tok == __shfl(split_entry, i, 64);
    } else {
      in_set = in_sorted(a.split_tok, a.S, tok);
    }
    const uint64_t split_nodes = __builtin_amdgcn_ballot_w64(node_ok && in_set);
    const uint64_t hits = __builtin_amdgcn_ballot_w64(lane < len && (split_nodes >> path & 1));
    int cut = -1;  // number of accepted drafts kept when the exit fires
    if (a.check_root && (split_nodes & 1)) cut = 0;
    if (hits && (a.split_pick != 0 || cut < 0))
      cut = a.split_pick == 0 ? __ffsll(static_cast<unsigned long long>(hits)) : 64 - __clzll(static_cast<long long>(hits));
    if (cut >= 0 && !pass) {
      // a step-split token was accepted but the sequence goes on thinking: its paragraph ends
      if (lane < 3) { hist[16 * lane] = 0.f; hist[16 * lane + 1] = 0.f; }
      if (lane == 0) hist[2] = __int_as_float(0);
    } else if (cut >= 0) {
      len = cut;
      cur = len ? __shfl(path, len - 1, 64) : 0;
      t_rec = a.stop_think_token;
      thinking = 0;
      flag = 1;
    }
  }
  if (node_ok) a.accept_path[static_cast<size_t>(b) * n + lane] = lane < len ? path : -1;
  if (lane == 0) {
    if (flag) a.is_thinking[b] = 0;
    a.accept_len[b] = len;
    a.recover_tok[b] = t_rec;
    a.last_node[b] = cur;
    a.exit_flag[b] = flag;
    a.new_ctx_len[b] = L + 1 + len;
  }
}

}  // namespace

hipError_t launch_accept_exit(const ExitArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_accept_exit, dim3(a.B), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace sx
