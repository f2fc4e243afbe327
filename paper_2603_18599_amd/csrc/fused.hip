// Projections of narrow models as one kernel each: GEMM, the sum over its K
// splits and the kernel that would consume the planes (rotary embedding with the
// cache write, residual + RMSNorm, SwiGLU).
//
// A narrow model's step (d = 1024: 25 MB of weights per layer, 256: 1.3 MB) is
// bound by launches and by the far-memory round trips between them, not by
// bytes: ten kernels per layer at 5-8 us each, of which launch and first access
// are 3-4. Here a workgroup owns one 32-column block over the whole of K: wave w
// takes the k range that split w of the plan has, the waves' accumulators meet
// in LDS, and the planes are summed there in split order, so no partial plane
// goes through memory and the result has the same bits as the split kernels'.
// The price is that each workgroup reads the whole activation (128 bytes per
// k and row tile, against 64 of weights), which wide models cannot pay: at d =
// 4096 the same structure ran at 2.6-3.1 TB/s on the O and down projections
// (12.5 and 28.8 us, where the split kernels take 11 and 20 and their consumers 3).
// Measured (d = 1024, 32 rows, us): QKV 8.2 for 7.5 + 4.6 (GEMM + rotary), O 7.0
// for 6.3 + 4.9, gate | up 8.6 for 8.4 + 4.8; with the one-kernel attention (8.8
// for 5.2 + 4.8) a 12-layer step at short caches 643 -> 590 us, the start of an
// image (prompt 64, 8 steps) 6.87 -> 5.65 ms; d = 256, 2 layers, 16 steps 2.16 ->
// 1.43 ms.
// A second row tile reads the weights again, from the caches; it pays all the same.
// Forwards at 200 cached rows, split kernels -> fused: mid shape (12 layers) 32 rows
// 635 -> 531 us, 64 768 -> 637, 96 868 -> 782, 128 1018 -> 851; d = 512 (12 layers) 555 -> 370
// and at 128 rows 868 -> 419; d = 1024 with an FFN of 4096 (6 layers) 340 -> 256 and 544 ->
// 453. Prompts of 500 (128-row windows): mid 3841 -> 3190, d = 512 3320 -> 1610.
// Columns whose results meet in one epilogue share a block: block b of the q,
// k, v rows holds 16 dims of a head and the 16 they rotate with, block b of gate |
// up holds 16 gate columns and the same 16 of up.
// RMSNorm: the residual epilogue leaves the sum of squares of each four columns
// ("fours"); the consumer adds them in the order the split path's norm does
// (butterfly over the 64 fours of a 256-column chunk, then chunk by chunk).
#include "device.h"
#include "forward.h"

namespace sjd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

SJD_DEV bf16x8 fused_bf16x8(const u32x4& u) { return __builtin_bit_cast(bf16x8, u); }

constexpr int kFusedWaves = 8;
constexpr int kRedLd = 36;  // LDS row stride of a plane's 32 x 32 block (16-byte aligned rows)

template <int MAXS>
struct FusedSmem {
  float red[MAXS][32][kRedLd];
  float chunk[32][kFusedMaxChunks];
  float inv[32];
};

// EPI: which epilogue. grid (column blocks, 32-row tiles): a second row tile reads
// the weights again, from the caches. The S splits go to min(S, 8) waves in turn;
// a wave runs its splits' k-steps as one sequence with RING of them in registers
// (a step is 12 KB, and the chain of far-memory loads is what a step costs), and
// leaves each split's accumulator in LDS when it ends. Everything the epilogue
// reads from memory is loaded ahead of the weights.
template <int EPI, int MAXS, int RING>
__global__ __launch_bounds__(kFusedWaves * kWave) void k_gemm_fused(FusedArgs a) {
  __shared__ FusedSmem<MAXS> sm;
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
  const int half = lane >> 5;
  const int nb = blockIdx.x, nblk = gridDim.x, m0 = blockIdx.y * 32;
  const int T = a.K / 64;
  const int NW = a.S < kFusedWaves ? a.S : kFusedWaves;

  // norm scale: (row, chunk) pairs, one per thread (at most 32 kFusedMaxChunks =
  // 128 of them, and four waves at least)
  constexpr bool kNorm = EPI != kFusedResid;
  const int npairs = kNorm ? 32 * a.nch : 0;
  float4 f4[16];
  if (kNorm && tid < npairs) {
    const float4* q = (const float4*)(a.fours + ((size_t)m0 * a.nch + tid) * 64);
#pragma unroll
    for (int i = 0; i < 16; ++i) f4[i] = q[i];
  }
  // epilogue thread: row of the tile, four columns (or two pairs)
  const int row = (tid & 255) >> 3, cq = tid & 7, m = m0 + row;
  const bool ep = tid < 256 && m < a.M;
  const int mr = m < a.M ? m : m0;  // a row that exists
  float4 xv = make_float4(0.f, 0.f, 0.f, 0.f);
  ushort4 gg = make_ushort4(0, 0, 0, 0);
  float* xr = nullptr;
  int pos = 0, krow = 0, z = 0;
  bool pad = false;
  const int hd2 = a.hd / 2, per = a.hd / 32;
  const int hh = EPI == kFusedRope ? nb / per : 0, i0 = EPI == kFusedRope ? (nb % per) * 16 + 2 * cq : 0;
  if constexpr (EPI == kFusedResid) {
    xr = a.x + (size_t)mr * a.N + nb * 32 + cq * 4;
    xv = *(const float4*)xr;
    gg = *(const ushort4*)(a.g + nb * 32 + cq * 4);
  } else if constexpr (EPI == kFusedRope) {
    const bool two = a.st.mode != kStreamsOne;
    const int loc = two ? (mr & 31) : mr;
    z = two ? mr >> 5 : 0;
    pad = two && loc >= a.st.L;
    pos = a.win->pos[mr];
    krow = stream_rows(a.st, a.n_dev ? *a.n_dev : a.n_host, z) + loc;
  }

  const uint16_t* wp = a.W + (size_t)nb * 2048 + (size_t)lane * 8;
  const size_t wstep = (size_t)nblk * 2048;
  const uint16_t* ap = a.A + (size_t)blockIdx.y * 4096 + (size_t)lane * 8;
  const size_t astep = (size_t)a.mtiles * 4096;
  u32x4 w[RING][4], x[RING][2][4];
  auto issue = [&](int st, int slot) {
    const uint16_t* pw = wp + (size_t)st * wstep;
    const uint16_t* pa = ap + (size_t)st * astep;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[slot][i] = *(const u32x4*)(pw + i * 512);
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[slot][p][i] = *(const u32x4*)(pa + p * kActLo + i * 512);
  };
  // the k-steps of this wave's splits wave, wave + NW, ... in turn; `end`: the
  // first step past the current split (empty splits are skipped)
  struct Cursor {
    int sp, st, end;
  };
  auto first = [&](int sp) {
    Cursor c{sp, 0, 0};
    for (; c.sp < a.S; c.sp += NW) {
      c.st = (int)((long)T * c.sp / a.S);
      c.end = (int)((long)T * (c.sp + 1) / a.S);
      if (c.st < c.end) break;
    }
    return c;
  };
  auto next = [&](Cursor c) { return c.st + 1 < c.end ? Cursor{c.sp, c.st + 1, c.end} : first(c.sp + NW); };
  Cursor cur = first(wave < NW ? wave : a.S), ahead = cur;
#pragma unroll
  for (int t = 0; t < RING; ++t)
    if (ahead.sp < a.S) {
      issue(ahead.st, t);
      ahead = next(ahead);
    }
  float2 cs[2];
  if constexpr (EPI == kFusedRope) {
#pragma unroll
    for (int e = 0; e < 2; ++e) cs[e] = a.rope[(size_t)pos * hd2 + i0 + e];
  }

  if constexpr (kNorm) {  // (while the operands are in flight)
    if (tid < npairs) {
      float v[64];
#pragma unroll
      for (int i = 0; i < 16; ++i) *(float4*)&v[4 * i] = f4[i];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int l = 0; l < o; ++l) v[l] += v[l + o];
      sm.chunk[tid / a.nch][tid % a.nch] = v[0];
    }
  }
  if (T < a.S) {  // empty splits: zero planes
    for (int i = tid; i < a.S * 32 * kRedLd; i += blockDim.x) (&sm.red[0][0][0])[i] = 0.0f;
    __syncthreads();
  }

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  while (cur.sp < a.S) {
#pragma unroll
    for (int u = 0; u < RING; ++u) {
      if (cur.sp < a.S) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fused_bf16x8(x[u][0][i]), fused_bf16x8(w[u][i]), acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fused_bf16x8(x[u][1][i]), fused_bf16x8(w[u][i]), acc, 0, 0, 0);
        }
        if (ahead.sp < a.S) {
          issue(ahead.st, u);
          ahead = next(ahead);
        }
        if (cur.st + 1 == cur.end) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            sm.red[cur.sp][8 * (r >> 2) + 4 * half + (r & 3)][lane & 31] = acc[r];
            acc[r] = 0.0f;
          }
        }
        cur = next(cur);
      }
    }
  }
  __syncthreads();
  if constexpr (kNorm) {
    if (tid < 32) {
      float ssum = 0.0f;
      for (int c = 0; c < a.nch; ++c) ssum += sm.chunk[tid][c];
      sm.inv[tid] = rsqrtf(ssum * a.inv_d + a.eps);
    }
    __syncthreads();
  }
  if (!ep) return;

  // plane value: accumulator times the norm scale, rounded before it is added
  // (the split path stores it in between)
  auto scaled = [&](float r) -> float {
#pragma clang fp contract(off)
    return r * sm.inv[row];
  };
  if constexpr (EPI == kFusedResid) {
    const int n0 = nb * 32 + cq * 4;
    for (int s = 0; s < a.S; ++s) {
      const float4 p = *(const float4*)&sm.red[s][row][cq * 4];
      xv.x += p.x;
      xv.y += p.y;
      xv.z += p.z;
      xv.w += p.w;
    }
    *(float4*)xr = xv;
    a.fours_out[(size_t)m * a.nch_out * 64 + (n0 >> 2)] = xv.x * xv.x + xv.y * xv.y + xv.z * xv.z + xv.w * xv.w;
    const float v[4] = {xv.x * bf16_to_f32(gg.x), xv.y * bf16_to_f32(gg.y), xv.z * bf16_to_f32(gg.z),
                        xv.w * bf16_to_f32(gg.w)};
    store_act<4>(a.y + act_off(m, n0, a.mtiles), v);
    return;
  }
  // columns 2 cq, 2 cq + 1 of the block's first 16 (p) and of its last 16 (q)
  float p[2] = {}, q[2] = {};
  for (int s = 0; s < a.S; ++s) {
    const float2 u = *(const float2*)&sm.red[s][row][2 * cq], v = *(const float2*)&sm.red[s][row][16 + 2 * cq];
    p[0] += scaled(u.x);
    p[1] += scaled(u.y);
    q[0] += scaled(v.x);
    q[1] += scaled(v.y);
  }
  auto pk = [](const uint16_t (&u)[2]) { return (uint32_t)u[0] | ((uint32_t)u[1] << 16); };
  uint16_t h0[2], l0[2], h1[2], l1[2];
  if constexpr (EPI == kFusedSwiglu) {
#pragma unroll
    for (int e = 0; e < 2; ++e) split_bf16(p[e] / (1.0f + expf(-p[e])) * q[e], h0[e], l0[e]);
    uint16_t* y = a.y + act_off(m, nb * 16 + 2 * cq, a.mtiles);
    *(uint32_t*)y = pk(h0);
    *(uint32_t*)(y + kActLo) = pk(l0);
  } else {
    // pairs (i, i + hd / 2), i = i0 + e, of head hh (see k_rope_kv)
    const size_t qo = (size_t)m * a.H * a.hd + (size_t)hh * a.hd + i0;
    if (pad) {
      if (hh < a.H)
        *(uint32_t*)(a.kv.q + qo) = *(uint32_t*)(a.kv.q_lo + qo) = *(uint32_t*)(a.kv.q + qo + hd2) =
            *(uint32_t*)(a.kv.q_lo + qo + hd2) = 0u;
      return;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float o0 = p[e], o1 = q[e];
      if (hh < a.H + a.Hkv) rotate_pair(p[e], q[e], cs[e], o0, o1);
      split_bf16(o0, h0[e], l0[e]);
      split_bf16(o1, h1[e], l1[e]);
    }
    const size_t so = (size_t)z * a.kv.sstride;
    if (hh < a.H) {
      *(uint32_t*)(a.kv.q + qo) = pk(h0);
      *(uint32_t*)(a.kv.q_lo + qo) = pk(l0);
      *(uint32_t*)(a.kv.q + qo + hd2) = pk(h1);
      *(uint32_t*)(a.kv.q_lo + qo + hd2) = pk(l1);
    } else if (hh < a.H + a.Hkv) {
      const size_t base = so + (size_t)(hh - a.H) * a.cap * a.hd;
      const size_t k0 = base + kv_key_off(krow, i0, a.hd), k1 = base + kv_key_off(krow, i0 + hd2, a.hd);
      *(uint32_t*)(a.kv.kc + k0) = pk(h0);
      *(uint32_t*)(a.kv.kc_lo + k0) = pk(l0);
      *(uint32_t*)(a.kv.kc + k1) = pk(h1);
      *(uint32_t*)(a.kv.kc_lo + k1) = pk(l1);
    } else {
      const size_t base = so + (size_t)(hh - a.H - a.Hkv) * a.cap * a.hd;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const size_t v0 = base + kv_val_off(krow, i0 + e, a.hd), v1 = base + kv_val_off(krow, i0 + e + hd2, a.hd);
        a.kv.vt[v0] = h0[e];
        a.kv.vt_lo[v0] = l0[e];
        a.kv.vt[v1] = h1[e];
        a.kv.vt_lo[v1] = l1[e];
      }
    }
  }
}

namespace {
template <int EPI>
hipError_t launch_epi(const FusedArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)(a.N / 32), (unsigned)((a.M + 31) / 32));
  // at least four waves: the epilogue takes 256 threads
  const dim3 block((unsigned)((a.S < 4 ? 4 : a.S < kFusedWaves ? a.S : kFusedWaves) * kWave));
  constexpr int RING = EPI == kFusedResid ? 4 : 3;
  if (a.S <= 8) hipLaunchKernelGGL((k_gemm_fused<EPI, 8, RING>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_gemm_fused<EPI, kGemmMaxSplits, RING>), grid, block, 0, s, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_gemm_fused(int epi, const FusedArgs& a, hipStream_t s) {
  if (a.M < 1 || a.M > 32 * kMaxStreams || a.M > 32 * a.mtiles || a.N % 32 || a.K % 64 || a.S < 1 ||
      a.S > kGemmMaxSplits)
    return hipErrorInvalidValue;
  if (epi == kFusedResid) {
    if (a.nch_out > kFusedMaxChunks) return hipErrorInvalidValue;
    return launch_epi<kFusedResid>(a, s);
  }
  if (a.nch < 1 || a.nch > kFusedMaxChunks) return hipErrorInvalidValue;
  if (epi == kFusedSwiglu) return launch_epi<kFusedSwiglu>(a, s);
  if (epi == kFusedRope && a.hd % 32 == 0) return launch_epi<kFusedRope>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace sjd
