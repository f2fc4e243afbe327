// Small kernels of the window forward: window rows and embedding, RMSNorm, rotary
// embedding with the key/value cache write, and weight conversion.
#include <type_traits>

#include "device.h"
#include "forward.h"

namespace sjd {

// acc[0..C) += sum_s of C consecutive floats of S partial planes, in plane
// order. The planes were written moments ago by workgroups on every XCD, so
// each load is a far-memory round trip: the loads of G planes are issued at
// once (planes past S re-read the last plane and are not added).
template <int G, int C>
SJD_DEV void add_planes(float (&acc)[C], const float* p, int S, size_t plane) {
  float4 a[G][C / 4];
#pragma unroll
  for (int s = 0; s < G; ++s)
#pragma unroll
    for (int i = 0; i < C / 4; ++i) a[s][i] = *(const float4*)(p + (size_t)(s < S ? s : S - 1) * plane + 4 * i);
#pragma unroll
  for (int s = 0; s < G; ++s)
    if (s < S) {
#pragma unroll
      for (int i = 0; i < C / 4; ++i) {
        acc[4 * i] += a[s][i].x;
        acc[4 * i + 1] += a[s][i].y;
        acc[4 * i + 2] += a[s][i].z;
        acc[4 * i + 3] += a[s][i].w;
      }
    }
}

// Kernels that write tiled activations give each wave 8 rows x 8 C columns:
// lane = (row % 8) * 8 + column / C. With C = 8 a wave reads 256 contiguous bytes
// of each row and writes whole 128-byte lines (8 rows x 16 bytes) of the tile;
// C = 4 spreads narrow matrices over twice the waves (two of them share a
// line): at d = 1024 and 22 planes C = 8 took 5.2 us where C = 4 takes 4.2. Whole
// forwards of two images, C = 8 -> 4 in the norm at 256 waves (d = 2048, 12 layers)
// 1245 -> 1229 us, at 384 (d = 3072, 8 layers) 1102 -> 1090; one 8B image of 6 layers
// (256) 736 -> 731; the 7B shape 734 either way.
constexpr int kNarrowWaves = 512;  // C = 4 where C = 8 would give fewer waves

// x += sum_s part[s] (split-K partial planes of the projection that feeds
// the residual, fixed order), y = x * g as tiled activations, ss[m][c] = sum
// of x^2 over the 256 elements of chunk c, each four of them in order and then
// by a butterfly over the 64 fours (narrow models: the fours themselves, [m][64
// chunks]). grid (chunks, rows / 8), 32 / C waves.
template <int G, int C>
__global__ __launch_bounds__(2048 / C) void k_resid_norm(float* x, const float* part, int S, size_t plane,
                                                         const uint16_t* g, int M, int d, uint16_t* y, int mtiles,
                                                         float* ss, float* fours) {
  __shared__ float four[8][kWave];
  const int c = blockIdx.x, wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  const int m = blockIdx.y * 8 + (lane >> 3), i0 = c * 256 + wave * 8 * C + (lane & 7) * C;
  float sq[C / 4] = {};
  if (m < M && i0 < d) {  // d is a multiple of 64: a lane's columns are all in range
    float* xr = x + (size_t)m * d + i0;
    float v[C];
    uint16_t gg[C];
#pragma unroll
    for (int i = 0; i < C / 4; ++i) {
      *(float4*)&v[4 * i] = *(const float4*)(xr + 4 * i);
      *(ushort4*)&gg[4 * i] = *(const ushort4*)(g + i0 + 4 * i);
    }
    if (S > 0) {
      add_planes<G, C>(v, part + (size_t)m * d + i0, S, plane);
#pragma unroll
      for (int i = 0; i < C / 4; ++i) *(float4*)(xr + 4 * i) = *(const float4*)&v[4 * i];
    }
#pragma unroll
    for (int i = 0; i < C / 4; ++i)
      sq[i] = v[4 * i] * v[4 * i] + v[4 * i + 1] * v[4 * i + 1] + v[4 * i + 2] * v[4 * i + 2] +
              v[4 * i + 3] * v[4 * i + 3];
#pragma unroll
    for (int e = 0; e < C; ++e) v[e] *= bf16_to_f32(gg[e]);
    store_act<C>(y + act_off(m, i0, mtiles), v);
  }
  if (fours) {  // uniform over the grid
    if (m < M && i0 < d)
#pragma unroll
      for (int i = 0; i < C / 4; ++i) fours[(size_t)m * gridDim.x * 64 + (i0 >> 2) + i] = sq[i];
    return;
  }
#pragma unroll
  for (int i = 0; i < C / 4; ++i) four[lane >> 3][(wave * 8 + (lane & 7)) * (C / 4) + i] = sq[i];
  __syncthreads();
  constexpr int RW = C / 4;  // rows per wave
#pragma unroll
  for (int r = RW * wave; r < RW * wave + RW; ++r) {
    const float ssq = wave_sum(four[r][lane]);
    const int row = blockIdx.y * 8 + r;
    if (lane == 0 && row < M) ss[(size_t)row * gridDim.x + c] = ssq;
  }
}

hipError_t launch_resid_norm(float* x, const float* part, int S, size_t plane, const uint16_t* g, int M, int d,
                             uint16_t* y, int mtiles, float* ss, float* fours, hipStream_t s) {
  if (S < 0 || S > kGemmMaxSplits || M > 32 * mtiles) return hipErrorInvalidValue;
  const dim3 grid(norm_chunks(d), (M + 7) / 8);
  auto go = [&](auto c) {
    constexpr int C = decltype(c)::value;
    const auto k = S <= 4    ? k_resid_norm<4, C>
                   : S <= 8  ? k_resid_norm<8, C>
                   : S <= 16 ? k_resid_norm<16, C>
                             : k_resid_norm<kGemmMaxSplits, C>;
    hipLaunchKernelGGL(k, grid, dim3(2048 / C), 0, s, x, part, S, plane, g, M, d, y, mtiles, ss, fours);
  };
  if ((d / 64) * ((M + 7) / 8) < kNarrowWaves) go(std::integral_constant<int, 4>{});
  else go(std::integral_constant<int, 8>{});
  return hipGetLastError();
}

// Window layout (Sec. 3.3: L verified positions per forward; Sec. 4.1: K
// candidates at each of the first D positions after a rejection): slot 0 holds
// the pending token (last committed, not yet cached) at position n; slot i, 1 <=
// i < n_s, holds spine draft i-1 at n + i; slot n_s + d(K-1) + k-2 holds sibling
// k of depth d at n + 1 + d and sees slots 0..d and itself. A missing sibling
// slot is fed token vis_lo.
SJD_DEV void window_row(const WindowIn& in, int a, int& tok, int& pos, uint64_t& anc) {
  if (!in.st) {  // prefill: a causal chain
    tok = in.prompt[in.start + a];
    pos = in.start + a;
    const int r = a & 63;  // within its 64-row part (see launch_attention)
    anc = r == 63 ? ~0ull : ((1ull << (r + 1)) - 1ull);
    return;
  }
  const Streams& sm = in.sm;
  const bool multi = sm.mode != kStreamsOne;
  const int z = multi ? a >> 5 : 0;      // stream of this row
  const int loc = multi ? (a & 31) : a;  // window row within its stream
  if (loc >= in.L) {  // padding row of a multi-stream window: never read, never cached
    tok = in.vis_lo;
    pos = in.st->n;
    anc = 0ull;
    return;
  }
  // batched: stream z is image z; guided: streams 2b, 2b + 1 are image b
  const DevState* d = multi ? in.st + stream_image(sm, z) : in.st;
  const bool unc = multi && stream_uncond(sm, z);
  const int n = d->n, n_s = d->n_s;
  // both words that the row may need, loaded before n_s is known
  const int chain = loc == 0 ? (unc ? d->pending_u : d->pending) : d->spine[loc - 1];
  if (loc < n_s) {
    tok = chain;
    pos = n + loc;
    anc = loc == 63 ? ~0ull : ((1ull << (loc + 1)) - 1ull);
  } else {
    const int t = loc - n_s, dd = t / (in.K - 1), k = t % (in.K - 1);
    const int y = d->sib[dd * (in.K - 1) + k];
    tok = y >= 0 ? y : in.vis_lo;
    pos = n + 1 + dd;
    anc = ((1ull << (dd + 1)) - 1ull) | (1ull << loc);
  }
  if (unc) pos += d->delta_u;
}

// One launch for what were three (window build, embedding gather, first norm),
// each of which took 4-5 us of the step for a few hundred KB: the rows' tokens
// are a few words of cached state, so every workgroup derives its own. grid
// (256-column chunks, rows / 8), four waves of 8 rows x 64 columns. Token ids
// come from callers (prompts, drafts): none is used as an index unchecked.
__global__ __launch_bounds__(256) void k_window_in(WindowIn a) {
  __shared__ float four[8][kWave];
  const int c = blockIdx.x, wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  const int m = blockIdx.y * 8 + (lane >> 3), i0 = c * 256 + wave * 64 + (lane & 7) * 8;
  if (a.st && c == 0 && blockIdx.y == 0 && threadIdx.x < kMaxStreams) {
    const int images = a.sm.mode == kStreamsOne ? 1 : a.sm.guided ? a.sm.nz / 2 : a.sm.nz;
    if ((int)threadIdx.x < images) {
      a.win->n[threadIdx.x] = a.st[threadIdx.x].n;
      a.win->n_s[threadIdx.x] = a.st[threadIdx.x].n_s;
    }
  }
  float s0 = 0.0f, s1 = 0.0f;
  if (m < a.M) {
    int tok, pos;
    uint64_t anc;
    window_row(a, m, tok, pos, anc);
    if (c == 0 && wave == 0 && (lane & 7) == 0) {
      a.win->tok[m] = tok;
      a.win->pos[m] = pos;
      a.win->anc[m] = anc;
    }
    tok = (tok >= 0 && tok < a.vocab) ? tok : a.vis_lo;
    if (i0 < a.d) {  // d is a multiple of 64: a lane's 8 columns are all in range
      const uint4 u = *(const uint4*)(a.E + (size_t)tok * a.d + i0), gu = *(const uint4*)(a.g + i0);
      const uint32_t uw[4] = {u.x, u.y, u.z, u.w}, gw[4] = {gu.x, gu.y, gu.z, gu.w};
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(e & 1 ? uw[e >> 1] & 0xFFFF0000u : uw[e >> 1] << 16);
      float* xr = a.x + (size_t)m * a.d + i0;
      *(float4*)xr = make_float4(v[0], v[1], v[2], v[3]);
      *(float4*)(xr + 4) = make_float4(v[4], v[5], v[6], v[7]);
      s0 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
      s1 = v[4] * v[4] + v[5] * v[5] + v[6] * v[6] + v[7] * v[7];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] *= __uint_as_float(e & 1 ? gw[e >> 1] & 0xFFFF0000u : gw[e >> 1] << 16);
      store_act<8>(a.y + act_off(m, i0, a.mtiles), v);
      if (a.fours) *(float2*)(a.fours + (size_t)m * gridDim.x * 64 + (i0 >> 2)) = make_float2(s0, s1);
    }
  }
  if (a.fours) return;  // uniform over the grid
  *(float2*)&four[lane >> 3][wave * 16 + (lane & 7) * 2] = make_float2(s0, s1);
  __syncthreads();
#pragma unroll
  for (int r = 2 * wave; r < 2 * wave + 2; ++r) {
    const float ssq = wave_sum(four[r][lane]);
    const int row = blockIdx.y * 8 + r;
    if (lane == 0 && row < a.M) a.ss[(size_t)row * gridDim.x + c] = ssq;
  }
}

hipError_t launch_window_in(const WindowIn& a, hipStream_t s) {
  const bool multi = a.sm.mode != kStreamsOne;
  if (a.M < 1 || a.M > kWinRows || a.M > 32 * a.mtiles || a.vis_lo < 0 || a.vis_lo >= a.vocab || (!a.st && !a.prompt) ||
      (multi && (a.sm.nz < 1 || a.sm.nz > kMaxStreams || a.L > 32)) || (!multi && a.st && a.M > 64))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_window_in, dim3(norm_chunks(a.d), (a.M + 7) / 8), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Rotate-half rotary embedding (pair i with i + hd/2 at angle pos * theta^(-2i/hd),
// table rope[pos][i] = (cos, sin)), then: q -> q planes, k and v -> cache
// position n + m (tiled layout), all as hi / lo bf16 planes. Two-stream
// windows: row m is slot m & 31 of stream m >> 5, cached at that stream's
// own position in its own cache; padding rows get a zero q and no cache write.
// grid (H + 2 * Hkv, M), block hd / 2. Head-major: workgroups are dealt to
// the XCDs round-robin by launch index, so (with H + 2 Hkv a multiple of 8)
// every row of one head runs on one XCD. A cache tile interleaves the rows
// of 8 positions in each 16-byte chunk, and its lines then fill in one L2
// instead of leaving as partial lines from eight (the row-major grid wrote
// 5.8 MB per launch for about 1.5 MB of data, and the step took 60 us longer).
template <int SMAX>
__global__ void k_rope_kv(const float* qkv, int S, size_t plane, const Window* win, const int32_t* n_dev, int n_host,
                          int H, int Hkv, int hd, const float2* rope, KvPlanes o, int cap, Streams sm) {
  const int m = blockIdx.y, hh = blockIdx.x, i = threadIdx.x;
  const int half = hd / 2;
  const bool two = sm.mode != kStreamsOne;
  const int z = two ? m >> 5 : 0;
  const int loc = two ? (m & 31) : m;
  if (two && loc >= sm.L) {
    if (hh < H) {
      const size_t off = (size_t)m * H * hd + (size_t)hh * hd;
      o.q[off + i] = o.q_lo[off + i] = o.q[off + i + half] = o.q_lo[off + i + half] = 0;
    }
    return;
  }
  const int n = stream_rows(sm, n_dev ? *n_dev : n_host, z);
  const int row = n + loc;
  if (z) {
    o.kc += z * o.sstride;
    o.kc_lo += z * o.sstride;
    o.vt += z * o.sstride;
    o.vt_lo += z * o.sstride;
  }
  const int ld = (H + 2 * Hkv) * hd;
  const float* src = qkv + (size_t)m * ld + (size_t)hh * hd;
  // all plane loads in flight at once (see add_planes)
  float pa[SMAX], pb[SMAX];
#pragma unroll
  for (int s = 0; s < SMAX; ++s) {
    const size_t so = (size_t)(s < S ? s : S - 1) * plane;
    pa[s] = src[so + i];
    pb[s] = src[so + i + half];
  }
  float a = 0.0f, b = 0.0f;
#pragma unroll
  for (int s = 0; s < SMAX; ++s)
    if (s < S) {
      a += pa[s];
      b += pb[s];
    }
  if (hh < H + Hkv) {
    const float2 cs = rope[(size_t)win->pos[m] * half + i];
    float o0, o1;
    rotate_pair(a, b, cs, o0, o1);
    if (hh < H) {
      const size_t off = (size_t)m * H * hd + (size_t)hh * hd;
      split_bf16(o0, o.q[off + i], o.q_lo[off + i]);
      split_bf16(o1, o.q[off + i + half], o.q_lo[off + i + half]);
    } else {
      const size_t base = (size_t)(hh - H) * cap * hd;
      const size_t k0 = base + kv_key_off(row, i, hd), k1 = base + kv_key_off(row, i + half, hd);
      split_bf16(o0, o.kc[k0], o.kc_lo[k0]);
      split_bf16(o1, o.kc[k1], o.kc_lo[k1]);
    }
  } else {
    const size_t base = (size_t)(hh - H - Hkv) * cap * hd;
    const size_t v0 = base + kv_val_off(row, i, hd), v1 = base + kv_val_off(row, i + half, hd);
    split_bf16(a, o.vt[v0], o.vt_lo[v0]);
    split_bf16(b, o.vt[v1], o.vt_lo[v1]);
  }
}

hipError_t launch_rope_kv(const float* qkv, int S, size_t plane, const Window* win, const int32_t* n_dev, int n_host,
                          int M, int H, int Hkv, int hd, const float2* rope, const KvPlanes& o, int cap,
                          const Streams& sm, hipStream_t s) {
  const dim3 grid(H + 2 * Hkv, M), block(hd / 2);
  if (S < 1) return hipErrorInvalidValue;
  if (S <= 4)
    hipLaunchKernelGGL(k_rope_kv<4>, grid, block, 0, s, qkv, S, plane, win, n_dev, n_host, H, Hkv, hd, rope, o, cap, sm);
  else if (S <= 8)
    hipLaunchKernelGGL(k_rope_kv<8>, grid, block, 0, s, qkv, S, plane, win, n_dev, n_host, H, Hkv, hd, rope, o, cap, sm);
  else if (S <= 16)
    hipLaunchKernelGGL(k_rope_kv<16>, grid, block, 0, s, qkv, S, plane, win, n_dev, n_host, H, Hkv, hd, rope, o, cap,
                       sm);
  else if (S <= kGemmMaxSplits)
    hipLaunchKernelGGL(k_rope_kv<kGemmMaxSplits>, grid, block, 0, s, qkv, S, plane, win, n_dev, n_host, H, Hkv, hd,
                       rope, o, cap, sm);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// h[m][n] = silu(g) * u with g, u the plane sums of columns n and F + n, as
// tiled activations. grid (F / 8C, rows / 8), one wave.
template <int G, int C>
__global__ __launch_bounds__(64) void k_swiglu(const float* P, int S, size_t plane, int M, int F, uint16_t* h,
                                               int mtiles) {
  const int lane = threadIdx.x;
  const int m = blockIdx.y * 8 + (lane >> 3), n0 = blockIdx.x * 8 * C + (lane & 7) * C;
  if (m >= M) return;
  const float* pg = P + (size_t)m * 2 * F + n0;
  float gs[C] = {}, us[C] = {};
  add_planes<G, C>(gs, pg, S, plane);
  add_planes<G, C>(us, pg + F, S, plane);
#pragma unroll
  for (int e = 0; e < C; ++e) gs[e] = gs[e] / (1.0f + expf(-gs[e])) * us[e];
  store_act<C>(h + act_off(m, n0, mtiles), gs);
}

hipError_t launch_swiglu(const float* P, int S, size_t plane, int M, int F, uint16_t* h, int mtiles, hipStream_t s) {
  if (S < 1 || S > kGemmMaxSplits || M > 32 * mtiles) return hipErrorInvalidValue;
  auto go = [&](auto c) {
    constexpr int C = decltype(c)::value;
    const auto k = S <= 2    ? k_swiglu<2, C>
                   : S <= 4  ? k_swiglu<4, C>
                   : S <= 8  ? k_swiglu<8, C>
                   : S <= 16 ? k_swiglu<16, C>
                             : k_swiglu<kGemmMaxSplits, C>;
    hipLaunchKernelGGL(k, dim3(F / (8 * C), (M + 7) / 8), dim3(64), 0, s, P, S, plane, M, F, h, mtiles);
  };
  if ((F / 64) * ((M + 7) / 8) < kNarrowWaves) go(std::integral_constant<int, 4>{});
  else go(std::integral_constant<int, 8>{});
  return hipGetLastError();
}

// one thread per 8-element chunk of the tiled layout
__global__ void k_tile_weights(const void* src, int is_f32, size_t row0, int N, int K, uint16_t* dst,
                               int nblk_total, int nb0, int pair) {
  const size_t T = (size_t)K / 64;
  const size_t nchunks = (size_t)N / 32 * T * 256;
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < nchunks; q += (size_t)gridDim.x * blockDim.x) {
    const size_t tile = q / 256, within = q % 256;
    const int i = (int)(within / 64), l = (int)(within % 64);
    const size_t nb = tile / T, kb = tile % T;
    const size_t row = row0 + nb * 32 + (size_t)(l % 32);
    const size_t col = kb * 64 + (size_t)(l / 32) * 32 + (size_t)i * 8;
    uint16_t v[8];
    if (is_f32) {
      const float* p = (const float*)src + row * (size_t)K + col;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = f32_to_bf16(p[e]);
    } else {
      const uint16_t* p = (const uint16_t*)src + row * (size_t)K + col;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = p[e];
    }
    const int r = (int)nb * 32 + l % 32;
    size_t ob = nb;
    int ol = l;
    if (pair > 0) {
      const int j = r % pair;
      ob = (size_t)(r / pair) * (pair / 32) + (j % (pair / 2)) / 16;
      ol = (l & 32) + j % 16 + (j >= pair / 2 ? 16 : 0);
    } else if (pair < 0) {
      ob = (size_t)(r / 16);
      ol = (l & 32) + r % 16 + (pair == -2 ? 16 : 0);
    }
    uint16_t* d = dst + ((kb * nblk_total + nb0 + ob) * 256 + (size_t)i * 64 + ol) * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = v[e];
  }
}

hipError_t launch_tile_weights(const void* src, int is_f32, size_t row0, int N, int K, uint16_t* dst,
                               int nblk_total, int nb0, int pair, hipStream_t s) {
  if (pair > 0 && (pair % 32 || N % pair)) return hipErrorInvalidValue;
  size_t n = (size_t)N / 32 * (K / 64) * 256;
  size_t blocks = (n + 255) / 256;
  if (blocks > 65535 * 8) blocks = 65535 * 8;
  hipLaunchKernelGGL(k_tile_weights, dim3((unsigned)blocks), dim3(256), 0, s, src, is_f32, row0, N, K, dst,
                     nblk_total, nb0, pair);
  return hipGetLastError();
}

__global__ void k_f32_to_bf16(const float* src, uint16_t* dst, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = f32_to_bf16(src[i]);
}

hipError_t launch_f32_to_bf16(const float* src, uint16_t* dst, size_t n, hipStream_t s) {
  size_t blocks = (n + 255) / 256;
  if (blocks > 65535 * 4) blocks = 65535 * 4;
  hipLaunchKernelGGL(k_f32_to_bf16, dim3((unsigned)blocks), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}

}  // namespace sjd
