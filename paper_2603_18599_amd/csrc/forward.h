// Internal interface of the window-forward kernels (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sjd {

constexpr int kGemmMaxSplits = 32;
constexpr int kFusedMaxChunks = 4;  // narrow models (fused.hip): 256-column norm chunks, d <= 1024

// Weights are repacked at init into 32-row x 64-column tiles (4 KB, bf16):
// tile (nb, kb) of a [N][K] matrix starts at element (kb * (N/32) + nb) *
// 2048 and holds, for i = 0..3 and lane l = 0..63, the 8 elements of row
// nb*32 + l%32, columns kb*64 + (l/32)*32 + i*8 .. +8 at (i*64 + l) * 8. A wave
// then reads one tile as four contiguous 1 KB loads, and the tiles that the
// column blocks read at the same k-step are adjacent (one contiguous stripe
// per k-step instead of tiles a whole row block apart, which measurably
// streams faster). Matrices that share an input (q, k, v; gate, up) are
// tiled as row blocks of one [N][K].
//
// Activations that enter a GEMM are stored the same way: tile (kb, mt), rows
// [32 mt, 32 mt + 32) x columns [64 kb, 64 kb + 64), holds its hi plane and then
// its lo plane (kActLo = 2048 elements each, the order above), at element (kb * mtiles +
// mt) * 4096 (mtiles = the buffer's row tiles). A wave stages 1 KB of it with
// one contiguous load; from row-major planes the same load touched 64 separate
// 16-byte pieces and kept the address unit busy four times as long, which at
// 64 and 128 rows was what the GEMM waited for.
__host__ __device__ inline size_t act_off(int m, int k, int mtiles) {
  const int lane = (m & 31) + (k & 32), i = (k & 31) >> 3;
  return ((size_t)(k >> 6) * mtiles + (m >> 5)) * 4096 + (size_t)(i * 64 + lane) * 8 + (k & 7);
}
inline size_t act_elems(int K, int mtiles) { return (size_t)(K / 64) * mtiles * 4096; }

struct GemmArgs {
  const uint16_t* A;   // activations as two bf16 planes (A = hi + lo), tiled as
  int mtiles;          // above (rows >= M of a started tile may hold anything)
  int M;               // 1..128
  const uint16_t* W;   // tiled weights [N][K]
  int N, K;            // N multiple of 32, K multiple of 64
  int S;               // workgroups along K = fp32 partial planes (1..kGemmMaxSplits)
  float* out;          // plane sp at out + sp * plane, row stride ldo
  size_t plane;
  int ldo;
  // optional RMS scale of row m (fused RMSNorm): rsqrt(sum_c ss[m * ss_n + c] *
  // inv_d + eps) multiplies the row of the product before the store
  const float* ss;
  int ss_n;
  const float* fours;  // or (ss NULL, narrow models): sums of squares of each four columns, [row][ss_n * 64]
  float inv_d, eps;
  // guided head (M > 32 only): for each image b (product rows [64 b, 64 b +
  // 64)), output row 32 b + m (m < cfg_rows) is u + cfg_w (c - u) with c =
  // product row 64 b + m, u = product row 64 b + 32 + m
  int cfg_rows;
  float cfg_w;
  // 8 column blocks per workgroup (else 4): half the activation loads per weight
  // byte; the grid is N / 256 column groups x S. (launch_gemm runs it 6 wide at up
  // to 64 rows where 8 would leave compute units idle; the width does not change a
  // result.)
  int wide;
  int ncu;  // the device's compute units
  // What padded k-steps take for weights, beside their zero activation tile: both
  // must be finite for such a step to add nothing, and the activation buffers hold
  // whatever earlier windows left in rows that this one does not write.
  const uint16_t* zeros;
};
// All lanes read the same 16 bytes at each of a tile's four offsets, and the zeros lie
// behind the activations, in pages that the kernel reads anyway. A whole tile of them
// in the library's own data cost 0.25 us a launch (mid shape, start of an image, us:
// 5134, four lines of it 5096; with 48-slot windows, 6 layers: 2111, behind the
// activations 2105; 7B forward of 6 layers 733, four lines 723).
constexpr int kZeroTile = 3 * 512 + 8;

// splits for about target_wgs workgroups of 4 (or, wide, 8) column blocks
int gemm_splits(int N, int K, int target_wgs, bool wide);
hipError_t launch_gemm(const GemmArgs& g, hipStream_t s);

// Repacks rows [row0, row0 + N) of a row-major [*][K] bf16 (or fp32, then
// rounded to nearest even) matrix into the tile layout above. Plain (pair 0):
// row blocks [nb0, nb0 + N/32) of a tiled matrix of nblk_total row blocks at
// dst. Paired, for the projections of narrow models (fused.hip):
//  - pair > 0 (q, k, v; pair = hd): row r of head r / hd, dim j = r % hd, goes to
//    row block nb0 + r / hd * (hd / 32) + (j % (hd / 2)) / 16, row j % 16, + 16 for
//    the upper half of the dims;
//  - pair < 0 (-1 gate, -2 up): row r goes to row block nb0 + r / 16, row r % 16, +
//    16 for up.
hipError_t launch_tile_weights(const void* src, int is_f32, size_t row0, int N, int K, uint16_t* dst,
                               int nblk_total, int nb0, int pair, hipStream_t s);

// Window description in device memory (written by the window builder).
// Row a's ancestors: bit i = row base + i of its own stream (base 0 for
// one stream, 32 z for stream z), a row itself included.
constexpr int kWinRows = 128;
struct Window {
  int32_t tok[kWinRows];
  int32_t pos[kWinRows];
  uint64_t anc[kWinRows];
  int32_t n[4], n_s[4];  // per image: cached rows and spine rows when the window was built
};

// Device-resident decoding state of one context.
struct DevState {
  int32_t n;        // cached rows
  int32_t pending;  // last committed token (slot 0)
  int32_t n_s, D_in, n_q, g0, q_off, pad;
  int32_t spine[64];
  int32_t sib[64];  // [D][K-1]
  int32_t meta[8];  // last step's outcome
  int32_t tok[64];  // last step's committed tokens
  int32_t pending_u;  // guided contexts: pending token of the unconditional stream
  int32_t delta_u;    // guided contexts: unconditional-stream position minus text-stream position
  int32_t pad2[2];
};

// A window forward runs one stream (rows [0, M)) or nz <= 4 streams of L <=
// 32 rows each: stream z at rows [32 z, 32 z + L), the other rows padding
// (never cached, never read). Each stream has its own key/value cache
// (stream z's at the stream-0 cache + z * sstride) and its own positions:
//  - batched: stream z is image z, with its own decoder state;
//  - guided (classifier-free guidance): streams come in pairs per image,
//    2b the text stream and 2b + 1 the unconditional stream, which is fed
//    the same window tokens (its own first pending token) at positions
//    shifted by the image's delta_u.
enum { kStreamsOne = 0, kStreamsMulti = 1 };
constexpr int kMaxStreams = 4;
struct Streams {
  int mode;            // kStreams*
  int L;               // window rows per stream (multi)
  int nz;              // streams (multi)
  int guided;          // multi: (text, unconditional) stream pairs
  const DevState* st;  // multi: decoder state of image 0 (image b at st + b)
};
__device__ inline int stream_image(const Streams& sm, int z) { return sm.guided ? z >> 1 : z; }
__device__ inline bool stream_uncond(const Streams& sm, int z) { return sm.guided && (z & 1); }
// cached rows before the window of stream z (one stream: n0)
__device__ inline int stream_rows(const Streams& sm, int n0, int z) {
  if (sm.mode == kStreamsOne) return n0;
  const DevState& d = sm.st[stream_image(sm, z)];
  return d.n + (stream_uncond(sm, z) ? d.delta_u : 0);
}

// Key / value cache layout. Per layer and kv head, positions are grouped in
// tiles of 32 (32 * hd elements each) stored in the register order of the
// attention MFMAs, so that every load of a tile is a contiguous 1 KB per
// wave: key (position p, dim j) is element (t * 64 + lane) * 8 + e of tile
// p / 32, with lane = swap23(p % 32) + 32 * (j / (hd / 2)), t = (j % (hd / 2)) / 8,
// e = j % 8 (swap23 exchanges bits 2 and 3: the key-row order of the score
// MFMA); value (p, j) is element ((j / 32) * 2 + i / 16) * 512 + lane * 8 + i % 8
// with i = p % 32, lane = j % 32 + 32 * ((i / 8) % 2) (the transposed-value
// operand of the output MFMA).
__host__ __device__ inline int swap23(int i) { return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1); }
__host__ __device__ inline size_t kv_key_off(int p, int j, int hd) {
  const int i = p & 31, h2 = hd / 2;
  const int lane = swap23(i) + 32 * (j / h2), t = (j % h2) >> 3;
  return (size_t)(p >> 5) * 32 * hd + (size_t)(t * 64 + lane) * 8 + (j & 7);
}
__host__ __device__ inline size_t kv_val_off(int p, int j, int hd) {
  const int i = p & 31;
  const int lane = (j & 31) + 32 * ((i >> 3) & 1);
  return (size_t)(p >> 5) * 32 * hd + (size_t)(((j >> 5) * 2 + (i >> 4)) * 64 + lane) * 8 + (i & 7);
}

struct AttnArgs {
  // every tensor below is a pair of bf16 planes (value = hi + lo)
  const uint16_t* q;     // [Mpad][H * hd], rotated
  const uint16_t* q_lo;
  const uint16_t* kc;    // [Hkv][cap * hd] key cache of this layer (tiled, see above)
  const uint16_t* kc_lo;
  const uint16_t* vt;    // [Hkv][cap * hd] value cache of this layer (tiled)
  const uint16_t* vt_lo;
  size_t sstride;        // multi-stream windows: stream z's caches are these + z * sstride
  Streams st;
  const Window* win;
  const int32_t* n_dev;  // cached rows before the window (device scalar), or NULL -> n_host
  int n_host;
  int M, H, Hkv, cap;
  float scale;
  float* ws_o;           // [H][nsplit_max][128][hd] partial outputs (per query slot)
  float* ws_ml;          // [H][nsplit_max][128][2]  partial max (log2 domain) and sum
  int nsplit_max;
  uint16_t* out;         // tiled activations (act_off), `mtiles` row tiles
  int mtiles;
  int whole;             // one kernel, where it can hold the cache (64-dim heads, kWholeChunks)
  int qparts;            // workgroups per key / value head, each taking H / Hkv / qparts query heads
};
constexpr int kAttnChunk = 128;  // keys per workgroup (4 waves x 32)
// k_attn_whole: chunks that its shared memory holds (no more than kCombGroup, whose
// order of sums it keeps). On the capacity, which no fill exceeds: what a captured
// launch holds is right for every later fill.
constexpr int kWholeChunks = 4;
hipError_t launch_attention(const AttnArgs& a, int hd, hipStream_t s);

// elementwise kernels
// A window's rows and their embedding, ready for the first layer: window tokens,
// positions and ancestors (from the decoder state, or from a prompt), x = E[tok]
// (ids outside [0, vocab) read as vis_lo), y = x * g as tiled activations and the
// norm's sums of squares (chunks ss, or for narrow models fours).
struct WindowIn {
  const DevState* st;     // state of image 0, or NULL:
  const int32_t* prompt;  //   rows are prompt[start ..) at positions start ..
  int start;
  int M, L, K, vis_lo;
  Streams sm;
  Window* win;
  const uint16_t* E;
  int d, vocab;
  float* x;
  const uint16_t* g;
  uint16_t* y;
  int mtiles;
  float* ss;
  float* fours;
};
hipError_t launch_window_in(const WindowIn& a, hipStream_t s);
// RMSNorm split in two: x += sum of S fp32 partial planes (fixed order; S
// may be 0), y = x * g as tiled activations (mtiles row tiles) and the sums of
// squares of x over 256-element chunks, ss[m][c] (c < norm_chunks(d)); the GEMM
// that consumes y applies the row scale 1 / sqrt(mean(x^2) + eps). With fours
// (narrow models) the sums of each four columns go there instead.
inline int norm_chunks(int d) { return (d + 255) / 256; }
hipError_t launch_resid_norm(float* x, const float* part, int S, size_t plane, const uint16_t* g, int M, int d,
                             uint16_t* y, int mtiles, float* ss, float* fours, hipStream_t s);
// rotary embedding of q and k, key row and transposed value column into the caches
struct KvPlanes {
  uint16_t *q, *q_lo, *kc, *kc_lo, *vt, *vt_lo;
  size_t sstride;  // multi-stream windows: stream z's caches are kc.. + z * sstride
};
// qkv: S fp32 partial planes [S][plane] summed in order
hipError_t launch_rope_kv(const float* qkv, int S, size_t plane, const Window* win, const int32_t* n_dev, int n_host,
                          int M, int H, int Hkv, int hd, const float2* rope, const KvPlanes& o, int cap,
                          const Streams& st, hipStream_t s);
// h = silu(gate) * up as tiled activations, gate = sum of the S fp32 partial
// planes at columns [0, F), up = at columns [F, 2F) (row stride 2F)
hipError_t launch_swiglu(const float* P, int S, size_t plane, int M, int F, uint16_t* h, int mtiles, hipStream_t s);
hipError_t launch_f32_to_bf16(const float* src, uint16_t* dst, size_t n, hipStream_t s);

// ---- narrow models (fused.hip): one kernel per projection
enum { kFusedRope = 0, kFusedResid = 1, kFusedSwiglu = 2 };
struct FusedArgs {
  const uint16_t* A;  // tiled activations, mtiles row tiles
  int mtiles, M;
  const uint16_t* W;  // tiled weights (q, k, v and gate | up paired)
  int N, K, S;        // S: the plan's split of K, which sets the summation order
  // norm scale of the input (Rope, Swiglu): sums of squares of each four
  // columns, [rows][nch * 64]
  const float* fours;
  int nch;
  float inv_d, eps;
  // Resid: x += product; y = x * g as tiled activations, fours of x
  float* x;
  const uint16_t* g;
  uint16_t* y;  // (Swiglu: the output)
  float* fours_out;
  int nch_out;
  // Rope
  const Window* win;
  const int32_t* n_dev;
  int n_host, H, Hkv, hd, cap;
  const float2* rope;
  KvPlanes kv;
  Streams st;
};
hipError_t launch_gemm_fused(int epi, const FusedArgs& a, hipStream_t s);

}  // namespace sjd
