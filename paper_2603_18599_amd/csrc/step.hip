// Step bookkeeping kernels: state initialisation, KV commit (moving an accepted sibling's
// key/value row) and the state update after verification. Everything stays
// in device memory; the host only enqueues.
#include "device.h"
#include "forward.h"
#include "step.h"

namespace sjd {

// Placeholders of the first window: uniform over the support (stream tag 6,
// trial 0, step word 0xFFFFFFFF, row = window index), the row end token at
// forced positions; no draft distributions, no siblings.
__global__ void k_state_init(DevState* st, const int32_t* prompt, int n_p, const int32_t* uncond, int n_u, int L,
                             int V, int vis_lo, int eol, int row_len, uint64_t seed) {
  const int i = threadIdx.x;
  if (i == 0) {
    st->n = n_p - 1;
    st->pending = prompt[n_p - 1];
    st->pending_u = uncond ? uncond[n_u - 1] : prompt[n_p - 1];
    st->delta_u = uncond ? n_u - n_p : 0;
    st->pad2[0] = st->pad2[1] = 0;
    st->n_s = L;
    st->D_in = 0;
    st->n_q = 0;
    st->g0 = 0;
    st->q_off = 0;
    st->pad = 0;
    for (int t = 0; t < 8; ++t) st->meta[t] = 0;
  }
  if (i < 64) {
    st->sib[i] = -1;
    st->tok[i] = -1;
    int t = -1;
    if (i < L) {
      const bool forced = row_len > 0 && (i % (row_len + 1)) == row_len;
      if (forced) {
        t = eol;
      } else {
        const Stream is(seed, kTagInit, 0, (uint32_t)i, 0u, 0xFFFFFFFFu);
        t = vis_lo + (int)(((uint64_t)is.word(0) * (uint64_t)V) >> 32);
      }
    }
    st->spine[i] = t;
  }
}

// The end of a step, one launch for the KV commit and the state update (4 us
// each on their own): the commit reads the window's cached rows and spine length
// as they were when the window was built (win), not the state that the update
// rewrites beside it; the outcome words it reads (meta[1], meta[5]) stay.
// grid (layers, Hkv, caches + 1), block hd. z < caches, KV commit of cache z: an
// accepted sibling's (meta[5] = k >= 2 at first rejected row r) key and value
// move from cache position n + n_s + r(K-1) + k-2 to n + r + 1. Cache z is the one
// at c + z * sstride; without guidance it is image z's, with guidance caches 2b
// and 2b + 1 are image b's text and unconditional streams (the latter's positions
// shifted by the image's delta_u). z = caches: state update and outputs, an image
// per workgroup in turn; host_n[b] (pinned host memory) receives the image's
// cached rows after the step.
__global__ __launch_bounds__(128) void k_step_end(DevState* st, const Window* win, KvPlanes c, int Hkv, int hd,
                                                  int cap, int K, int guided, int32_t* out_meta, int32_t* out_tok,
                                                  int32_t* out_next, int L, int B, int32_t* host_n) {
  const int z = blockIdx.z, j = threadIdx.x;
  if (z + 1 < (int)gridDim.z) {
    const int b = guided ? z >> 1 : z;
    const DevState* s = st + b;
    const int acc_k = s->meta[5];
    if (acc_k < 2) return;
    c.kc += z * c.sstride;
    c.kc_lo += z * c.sstride;
    c.vt += z * c.sstride;
    c.vt_lo += z * c.sstride;
    const int n = win->n[b] + (guided && (z & 1) ? s->delta_u : 0), r = s->meta[1];
    const int src = n + win->n_s[b] + r * (K - 1) + (acc_k - 2);
    const int dst = n + r + 1;
    const size_t base = ((size_t)blockIdx.x * Hkv + blockIdx.y) * cap * hd;
    const size_t ks = base + kv_key_off(src, j, hd), kd = base + kv_key_off(dst, j, hd);
    const size_t vs = base + kv_val_off(src, j, hd), vd = base + kv_val_off(dst, j, hd);
    c.kc[kd] = c.kc[ks];
    c.kc_lo[kd] = c.kc_lo[ks];
    c.vt[vd] = c.vt[vs];
    c.vt_lo[vd] = c.vt_lo[vs];
    return;
  }
  for (int b = blockIdx.x + gridDim.x * blockIdx.y; b < B; b += gridDim.x * gridDim.y) {
    DevState* s = st + b;
    // (no thread writes a word that another one reads here: meta[0..6], tok and
    // spine stay, and n is rewritten by the thread that reads it)
    const int n_c = s->meta[0];
    if (out_tok && j < L) out_tok[L * b + j] = s->tok[j];
    if (out_next && j < L) out_next[L * b + j] = s->spine[j];
    if (out_meta && j < 7) out_meta[8 * b + j] = s->meta[j];
    if (j == 7) {
      const int n_new = s->n + (n_c > 0 ? n_c : 0);
      if (out_meta) out_meta[8 * b + 7] = n_new;
      if (host_n) host_n[b] = n_new;
      if (n_c > 0) {
        s->pending = s->tok[n_c - 1];
        s->pending_u = s->tok[n_c - 1];
        s->n = n_new;
        s->n_s = s->meta[3];
        s->D_in = s->meta[2];
        s->n_q = s->meta[4];
        s->g0 = s->meta[6];
        s->q_off = n_c;
        s->meta[7] = n_new;
      }
    }
  }
}

// Caller-supplied drafts of the next step: a plain chain (no drafting
// siblings) whose row j carries tok[j]; with has_q, row j's draft
// distribution is row j of the draft logits (q_off 0), otherwise no row has
// one and every row draws from its own distribution.
__global__ void k_set_drafts(DevState* st, const int32_t* tok, int L, int has_q) {
  const int j = threadIdx.x;
  if (j < L) st->spine[j] = tok[j];
  if (j == 0) {
    st->n_s = L;
    st->D_in = 0;
    st->n_q = has_q ? L : 0;
    st->q_off = 0;
  }
}

// SJD_CHECK_FINITE: counts the NaN and +inf entries of p[0 .. n) into *cnt
// (-inf marks an excluded token and is allowed).
__global__ void k_zero1(int32_t* cnt) { *cnt = 0; }
__global__ __launch_bounds__(256) void k_count_nonfinite(const float* p, size_t n, int32_t* cnt) {
  int bad = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const float v = p[i];
    bad += (v != v) || (v == INFINITY);
  }
  const int tot = wave_sum_i(bad);
  if ((threadIdx.x & (kWave - 1)) == 0 && tot) atomicAdd(cnt, tot);
}

hipError_t launch_count_nonfinite(const float* p, size_t n, int32_t* cnt, bool reset, hipStream_t s) {
  if (reset) hipLaunchKernelGGL(k_zero1, dim3(1), dim3(1), 0, s, cnt);
  if (n > 0) {
    size_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_count_nonfinite, dim3((unsigned)blocks), dim3(256), 0, s, p, n, cnt);
  }
  return hipGetLastError();
}

hipError_t launch_set_drafts(DevState* st, const int32_t* tok, int L, bool has_q, hipStream_t s) {
  if (L < 1 || L > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_set_drafts, dim3(1), dim3(64), 0, s, st, tok, L, has_q ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_state_init(DevState* st, const int32_t* prompt, int n_p, const int32_t* uncond, int n_u, int L,
                             int V, int vis_lo, int eol, int row_len, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL(k_state_init, dim3(1), dim3(64), 0, s, st, prompt, n_p, uncond, n_u, L, V, vis_lo, eol, row_len,
                     seed);
  return hipGetLastError();
}
hipError_t launch_step_end(DevState* st, const Window* win, const KvPlanes& c, int layers, int Hkv, int hd, int cap,
                           int K, int ncache, bool guided, int32_t* out_meta, int32_t* out_tok, int32_t* out_next,
                           int L, int B, int32_t* host_n, hipStream_t s) {
  if (hd > 128 || hd < 64 || L > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_step_end, dim3(layers, Hkv, ncache + 1), dim3(hd), 0, s, st, win, c, Hkv, hd, cap, K,
                     guided ? 1 : 0, out_meta, out_tok, out_next, L, B, host_n);
  return hipGetLastError();
}

}  // namespace sjd
