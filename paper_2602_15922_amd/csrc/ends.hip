// The two ends of a step as one kernel each for gfx950: patch and action embedding into the
// fp32 residual, and the head (LayerNorm, modulation, the two output projections, the
// unpatchify) out of it.  Both are bound by the residual's bytes: 4 d per row, once each way.
#include "common.h"
#include "kernels.h"

namespace wam {
int cu_count();
namespace {

typedef float f32x4m __attribute__((ext_vector_type(4)));
WAM_DEV f32x4m mfma16(bf16x8 a, bf16x8 b, f32x4m c) {
  // 16x16x32 bf16.  Lane l: A[m = l % 16][k = 8 (l / 16) ..], B[k likewise][n = l % 16],
  // register r of D: [m = 4 (l / 16) + r][n = l % 16]
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------------
// Embedding: x[b][row][:] = feat(row) . W^T + bias, feat the 1x2x2 patch of a video token
// (W = w_patch, features (c, ph, pw)) or the features of an action token (w_ain).  A
// wavefront keeps the W rows of 64 columns as MFMA operands (a load of 32 different rows takes
// a cycle per lane in the address path, so they are read once) and walks tiles of 32 tokens,
// the patch gathered straight from the latents: a lane's token's (pw) pairs are 4-byte loads,
// consecutive tokens consecutive.  A lane of the product has one column of 16 tokens, so
// every store instruction writes two whole 128-byte lines.  Bound by the 4 d bytes written
// per row: at 3152 x 5120 the patchify, the two products and their launches took 34 us in the
// present GEMM tiles, this kernel 19 (3.4 TB/s).
// ---------------------------------------------------------------------------------
constexpr int EMB_COLS = 256;  // columns per workgroup, 64 per wavefront

template <int KS>  // MFMA k-steps of 16 that hold the features
__global__ __launch_bounds__(256) void embed_kernel(const EmbedArgs a, int tiles) {
  if (skip_step(a.skip)) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l32 = lane & 31, hh = lane >> 5;
  const int Hg = a.Hl >> 1, Wg = a.Wl >> 1, Lv = a.F * Hg * Wg, L = Lv + a.A;
  const int vt = (Lv + 31) >> 5, at = (a.A + 31) >> 5;  // token tiles of a sample
  const int ncol = a.d / EMB_COLS, step = gridDim.x / ncol;
  const int n0 = (blockIdx.x % ncol) * EMB_COLS + w * 64 + l32;
  bf16x8 wf[2][KS];
  float bn[2] = {0.f, 0.f};
  int have = -1;  // the kind whose W rows are loaded: 0 action, 1 video
  for (int t = blockIdx.x / ncol; t < tiles; t += step) {
    const int b = t / (vt + at), j = t % (vt + at);
    const bool video = j < vt;
    const int first = video ? 32 * j : 32 * (j - vt), count = video ? Lv : a.A;
    const int tok = first + l32 < count ? first + l32 : count - 1;
    const int K = video ? 4 * a.C : a.act_dim;
    if (have != (int)video) {
      have = video;
      const bf16* W = static_cast<const bf16*>(video ? a.w_patch : a.w_ain) + 8 * hh;
      const float* bias = video ? a.b_patch : a.b_ain;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          if (16 * ks < K) wf[c][ks] = load_bf16x8(W + (int64_t)(n0 + 32 * c) * K + 16 * ks);
        bn[c] = bias ? bias[n0 + 32 * c] : 0.f;
      }
    }
    bf16x8 f[KS];
    if (video) {
      const int s = tok % Wg, r = (tok / Wg) % Hg, fr = tok / (Wg * Hg);
      const bf16* z = static_cast<const bf16*>(a.z) + (((int64_t)b * a.C * a.F + fr) * a.Hl + 2 * r) * a.Wl + 2 * s;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        // features 16 ks + 8 hh .. + 7: channels c0 and c0 + 1, rows ph, pairs pw
        const int c0 = 4 * ks + 2 * hh;
        if (16 * ks < K) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const bf16x2 p = *reinterpret_cast<const bf16x2*>(z + ((int64_t)(c0 + (q >> 1)) * a.F * a.Hl + (q & 1)) * a.Wl);
            f[ks][2 * q] = p[0];
            f[ks][2 * q + 1] = p[1];
          }
        }
      }
    } else {
      const bf16* src = static_cast<const bf16*>(a.act) + ((int64_t)b * a.A + tok) * a.act_dim + 8 * hh;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        if (16 * ks < K) f[ks] = load_bf16x8(src + 16 * ks);
    }
    float* x = a.x + ((int64_t)b * L + (video ? 0 : Lv) + first + 4 * hh) * a.d + n0;
    const bool full = first + 32 <= count;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      f32x16 acc = f32x16{};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        if (16 * ks < K) acc = mfma32(f[ks], wf[c][ks], acc);
      if (full) {
#pragma unroll
        for (int r = 0; r < 16; ++r) x[(int64_t)(8 * (r >> 2) + (r & 3)) * a.d + 32 * c] = acc[r] + bn[c];
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (first + 8 * (r >> 2) + 4 * hh + (r & 3) < count)
            x[(int64_t)(8 * (r >> 2) + (r & 3)) * a.d + 32 * c] = acc[r] + bn[c];
      }
    }
  }
}

// ---------------------------------------------------------------------------------
// Head: h = bf16(LN(x)(1 + scale) + shift), v = h W^T + bias (W = w_hv for video rows, w_ha for
// action rows), the video features put back as pixels.  A workgroup of 8 wavefronts takes 16
// rows of one kind, two per wavefront, held in registers between the mean, variance and
// output passes, so x is read once.  The product runs over chunks of 256 columns with one
// barrier each: h of the chunk goes to LDS, its 64 rows of W come by direct loads into a ring of
// three stages, and wavefronts 0 to 3 multiply 16 outputs each (16x16x32 MFMA).  Every sum is
// taken in the order of the general path, so the velocities are bit for bit those of the modulated
// LayerNorm, the GEMM's fp32 epilogue and the unpatchify: a lane holds the columns it holds in
// the LayerNorm of that width (V8: 8 consecutive ones, 512 per step of the row, which are
// two chunks of h), and one wavefront runs an output's whole K.  (W straight from
// L2 into MFMA operands, 16 rows of 64 bytes per load, takes a cycle per lane in the address
// path: 44 us at 3152 x 5120, 55 with 8 rows per workgroup.)  Bound by the 4 d bytes read per
// row, then by the W reads (640 KB per workgroup at 64 bytes per cycle): the LayerNorm (a
// bf16 h written and read again), the products of 64 and 16 columns and the unpatchify took
// 53 us there in the present GEMM tiles (117 in 128-row tiles), this kernel 26.
// ---------------------------------------------------------------------------------
constexpr int HEAD_ROWS = 16, HEAD_CH = 256, HEAD_N = 64, HEAD_STAGES = 3, HEAD_HBUFS = 3;
constexpr int HEAD_WSTAGE = HEAD_N * HEAD_CH * 2, HEAD_HBUF = HEAD_ROWS * HEAD_CH * 2;  // bytes

typedef __attribute__((address_space(3))) void lds_void;

// 16-byte chunk c of row r of a W or h chunk (512-byte rows: unswizzled, the 16 rows a
// fragment read touches would share their banks)
WAM_DEV int head_swz(int r, int c) { return r * (HEAD_CH * 2) + ((c ^ (r & 15)) << 4); }

// NV: float4s of a row per lane = chunks of 256 columns (at least d / 256); V8: d a multiple of 512
template <int NV, bool V8>
__global__ __launch_bounds__(512, 2) void head_kernel(const HeadArgs a) {
  // W ring, h buffers, then the folded modulation P = 1 + scale and Q = shift; one array, so
  // that the compiler does not hold LDS reads back for the direct loads in flight
  constexpr int HS = HEAD_STAGES * HEAD_WSTAGE, PQ = HS + HEAD_HBUFS * HEAD_HBUF;
  __shared__ __attribute__((aligned(16))) char smem[PQ + 2 * NV * HEAD_CH * 4];
  if (skip_step(a.skip)) return;
  const int lane = threadIdx.x & 63, l16 = lane & 15, q4 = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int Hg = a.Hl >> 1, Wg = a.Wl >> 1, Lv = a.F * Hg * Wg, L = Lv + a.A, d = a.d, nv = d >> 8;
  const int vt = (Lv + HEAD_ROWS - 1) / HEAD_ROWS, at = (a.A + HEAD_ROWS - 1) / HEAD_ROWS;
  const int b = blockIdx.x / (vt + at), j = blockIdx.x % (vt + at);
  const bool video = j < vt;
  const int first = HEAD_ROWS * (video ? j : j - vt), count = video ? Lv : a.A;
  const int N = video ? 4 * a.C : a.act_dim;
  const float* x = a.x + ((int64_t)b * L + (video ? 0 : Lv)) * d;
  f32x4 v[2][NV];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int row = first + 2 * w + r < count ? first + 2 * w + r : count - 1;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (i < nv) {
        const int col = V8 ? ((i >> 1) * 64 + lane) * 8 + (i & 1) * 4 : (i * 64 + lane) * 4;
        v[r][i] = *reinterpret_cast<const f32x4*>(x + (int64_t)row * d + col);
      }
  }
  float* P = reinterpret_cast<float*>(smem + PQ);
  float* Q = P + d;
  {
    const float* ev = a.e + (int64_t)b * d + (video ? 0 : a.e_alt);
    for (int c = threadIdx.x * 4; c < d; c += 2048) {
      const f32x4 one = {1.f, 1.f, 1.f, 1.f};
      *reinterpret_cast<f32x4*>(Q + c) = *reinterpret_cast<const f32x4*>(a.mod2 + c) + *reinterpret_cast<const f32x4*>(ev + c);
      *reinterpret_cast<f32x4*>(P + c) =
          one + (*reinterpret_cast<const f32x4*>(a.mod2 + d + c) + *reinterpret_cast<const f32x4*>(ev + c));
    }
  }
  // W loads: unit u = (4 w + i) * 64 + lane of a chunk is row u / 32, physical 16-byte chunk u % 32
  // (rows past N re-read the last one; their columns are never stored)
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(video ? a.w_hv : a.w_ha), (short)0, 0x7fffffff, 0x00020000);
  int woff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int u = (4 * w + i) * 64 + lane, n = u >> 5, c = (u & 31) ^ (n & 15);
    woff[i] = 2 * ((n < N ? n : N - 1) * d + 8 * c);
  }
  auto fetch = [&](int c) {  // chunk c into stage c % 3; past the end the last one again (never read)
    const int cc = c < nv ? c : nv - 1;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void*)(smem + (c % HEAD_STAGES) * HEAD_WSTAGE + (4 * w + i) * 1024),
                                               16, woff[i], cc * HEAD_CH * 2, 0, 0);
  };
  float mean[2], rstd[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (i < nv) s += (v[r][i][0] + v[r][i][1]) + (v[r][i][2] + v[r][i][3]);
    mean[r] = wave_sum(s) / (float)d;
  }
  fetch(0);
  fetch(1);
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (i < nv) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float t = v[r][i][e] - mean[r];
          q += t * t;
        }
      }
    rstd[r] = rsqrtf(wave_sum(q) / (float)d + a.eps);
  }
  f32x4m acc = {0.f, 0.f, 0.f, 0.f};  // of outputs 16 w .. 16 w + 15 (wavefronts 0 to 3)
  const bool mul = 16 * w < N;
  __syncthreads();  // P and Q
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    if (c < nv) {
      if (!V8 || c % 2 == 0) {
        // this lane's columns of chunk c, or of chunks c (lanes 0 to 31) and c + 1 (the others)
        constexpr int E = V8 ? 2 : 1;  // float4s
        const int col = V8 ? HEAD_CH * c + 8 * lane : HEAD_CH * c + 4 * lane;
        const int buf = V8 && lane >= 32 ? (c + 1) % HEAD_HBUFS : c % HEAD_HBUFS;
        char* hb = smem + HS + buf * HEAD_HBUF;
        bf16 o[2][4 * E];
#pragma unroll
        for (int f = 0; f < E; ++f) {
          const f32x4 pp = *reinterpret_cast<const f32x4*>(P + col + 4 * f);
          const f32x4 qq = *reinterpret_cast<const f32x4*>(Q + col + 4 * f);
#pragma unroll
          for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[r][4 * f + e] = (bf16)((v[r][c + f][e] - mean[r]) * rstd[r] * pp[e] + qq[e]);
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          if constexpr (V8) {
            bf16x8 t;
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = o[r][e];
            *reinterpret_cast<bf16x8*>(hb + head_swz(2 * w + r, lane & 31)) = t;
          } else {
            bf16x4 t;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = o[r][e];
            *reinterpret_cast<bf16x4*>(hb + head_swz(2 * w + r, lane >> 1) + 8 * (lane & 1)) = t;
          }
        }
      }
      // h written, this wavefront's part of W's chunk c landed (chunk c + 1 may be in flight);
      // past the barrier both are everyone's, and the stage and the h buffer of chunk c - 1 are free
      __builtin_amdgcn_s_waitcnt(4 | (7 << 4) | (0 << 8));  // vmcnt(4), lgkmcnt(0)
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      fetch(c + 2);
      if (mul) {
        const char* hb = smem + HS + (c % HEAD_HBUFS) * HEAD_HBUF;
        const char* ws = smem + (c % HEAD_STAGES) * HEAD_WSTAGE;
#pragma unroll
        for (int ks = 0; ks < HEAD_CH / 32; ++ks)
          acc = mfma16(*reinterpret_cast<const bf16x8*>(hb + head_swz(l16, 4 * ks + q4)),
                       *reinterpret_cast<const bf16x8*>(ws + head_swz(16 * w + l16, 4 * ks + q4)), acc);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0);  // the ring's last loads land before its LDS is reused
  __syncthreads();
  float* red = reinterpret_cast<float*>(smem);  // [16 rows][64]
  if (mul)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[(4 * q4 + r) * HEAD_N + 16 * w + l16] = acc[r];
  __syncthreads();
  const float* bias = video ? a.b_hv : a.b_ha;
  for (int o = threadIdx.x; o < HEAD_ROWS * N; o += 512) {
    // video: two pixels of each of the 16 tokens, then the next (channel, row) pair, so that
    // neighbouring lanes write neighbouring pixels
    int m, n;
    if (video) {
      m = (o >> 1) & 15;
      n = 2 * (o >> 5) + (o & 1);
    } else {
      m = o / N;
      n = o - m * N;
    }
    if (first + m >= count) continue;
    const float s = red[m * HEAD_N + n] + (bias ? bias[n] : 0.f);
    const int tok = first + m;
    if (video) {
      const int sx = tok % Wg, r = (tok / Wg) % Hg, fr = tok / (Wg * Hg);
      const int ch = n >> 2, ph = (n >> 1) & 1, pw = n & 1;
      a.v_video[((((int64_t)b * a.C + ch) * a.F + fr) * a.Hl + 2 * r + ph) * a.Wl + 2 * sx + pw] = s;
    } else {
      a.v_action[((int64_t)b * a.A + tok) * a.act_dim + n] = s;
    }
  }
}

}  // namespace

hipError_t launch_embed(const EmbedArgs& a, hipStream_t s) {
  const int Lv = a.F * (a.Hl / 2) * (a.Wl / 2), ncol = a.d / EMB_COLS;
  const int tiles = a.B * ((Lv + 31) / 32 + (a.A + 31) / 32);
  // about four workgroups per CU, so that one's gather runs beside another's stores
  const int per_col = 4 * cu_count() / ncol > 0 ? 4 * cu_count() / ncol : 1;
  const dim3 grid((unsigned)(ncol * (tiles < per_col ? tiles : per_col))), block(256);
  const int K = 4 * a.C > a.act_dim ? 4 * a.C : a.act_dim;
  if (K <= 64) hipLaunchKernelGGL(embed_kernel<4>, grid, block, 0, s, a, tiles);
  else hipLaunchKernelGGL(embed_kernel<8>, grid, block, 0, s, a, tiles);
  return hipGetLastError();
}

hipError_t launch_head(const HeadArgs& a, hipStream_t s) {
  const int Lv = a.F * (a.Hl / 2) * (a.Wl / 2);
  const dim3 grid((unsigned)(a.B * ((Lv + HEAD_ROWS - 1) / HEAD_ROWS + (a.A + HEAD_ROWS - 1) / HEAD_ROWS))), block(512);
  const int nv = a.d / 256;
  if (nv % 2 == 0) {
    if (nv <= 4) hipLaunchKernelGGL((head_kernel<4, true>), grid, block, 0, s, a);
    else if (nv <= 12) hipLaunchKernelGGL((head_kernel<12, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((head_kernel<20, true>), grid, block, 0, s, a);
  } else {
    if (nv <= 3) hipLaunchKernelGGL((head_kernel<3, false>), grid, block, 0, s, a);
    else if (nv <= 11) hipLaunchKernelGGL((head_kernel<11, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((head_kernel<19, false>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace wam
