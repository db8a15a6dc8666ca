// Patch Selection Module forward pass: a small pre-norm transformer encoder
// over the text query's token embeddings, then a single-headed cross-attention
// of N learnable latent queries (one per camera view) over the encoded tokens
// and one linear head per view, giving the view logits that the patch
// selection fuses with its lexical scores.
//
// The module is tiny (d = 256, 4 layers, 128 tokens at the benchmark shape),
// so a forward is a chain of short launches: what a launch costs is its
// dependent round trips to memory, not its arithmetic, and beyond a few
// hundred rows the cache traffic of its tiles.
//   - psm_gemm_kernel: bf16 MFMA (v_mfma_f32_16x16x32_bf16) on A [M, K] times
//     W^T, W [N, K] fp32 from the parameter vector. A workgroup asks for its
//     whole first tile at once in whole rows, rounds it to bf16 on the way to
//     LDS and multiplies from there; A is bf16 or the LayerNorm of fp32 rows.
//   - self-attention: the library's prefill attention kernel, non-causal.
//   - psm_head_kernel: the cross-attention and the heads (7 us for one query;
//     forming the K and V rows and attending to them took 16 + 18.6 us). The latent side is
//     folded first, by a few workgroups beside the first layer's GEMMs
//     (psm_fold): with q_v = W_cq lat_v + b_cq, a token's logit is
//     x_t . (W_ck^T q_v) and its share of the view's output x_t . (W_cv^T w_v)
//     (w_v the head's weights), each plus a constant, so no K or V rows are
//     ever formed.
#include "common.hpp"
#include "launch.hpp"

namespace litevlm {
namespace {

typedef uint32_t psm_u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t psm_u32x4 __attribute__((ext_vector_type(4)));

// Exact-erf GELU, x * erfc(-x/sqrt(2)) / 2, branch-free: with z = |x|/sqrt(2) and
// t = 1/(1 + 0.4 z), erfc(z) = t exp(-z^2) P(t), P of degree 8 fitted to
// erfc(z) exp(z^2) / t over all z >= 0 (least squares reweighted towards equal
// relative error: 1.3e-7). Negative x needs no cancelling 1 + erf: the absolute
// error is 3.9e-7 at most, that of 0.5 x (1 + erf) in fp32 4.5e-7.
__device__ __forceinline__ float gelu_erf(float x) {
  const float z = fabsf(x) * 0.7071067811865476f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.4f, z, 1.f));
  float P = 0.050258949398994446f;
  P = fmaf(P, t, -0.18288986384868622f);
  P = fmaf(P, t, 0.16906839609146118f);
  P = fmaf(P, t, -0.005594694521278143f);
  P = fmaf(P, t, 0.14142614603042603f);
  P = fmaf(P, t, 0.16854313015937805f);
  P = fmaf(P, t, 0.20784257352352142f);
  P = fmaf(P, t, 0.22566960752010345f);
  P = fmaf(P, t, 0.22567586600780487f);
  const float e = 0.5f * t * P * __builtin_amdgcn_exp2f(-z * z * kLog2e);  // erfc(z) / 2
  return x * (x > 0.f ? 1.f - e : e);
}

// Two fp32 values to packed bf16 (round to nearest even).
__device__ __forceinline__ uint32_t psm_pk(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)lo, (__bf16)hi});
}

enum { kOutBf16 = 0, kOutGelu = 1, kOutResid = 2 };

// The latent side of the cross-attention, folded by the workgroups past the
// GEMM's own: stage 1 forms q_v, g_v = W_cv^T w_v and cst_v = w_v . b_cv +
// b_head_v, stage 2 (a later launch) u_v = W_ck^T q_v. All fp32. (An infinite
// head weight leaves NaN in g_v, so in the view's logit, where z first and w_v
// after would leave an infinity.)
struct PsmFold {
  int stage, d, n_views;  // stage 0: nothing
  const float *lat, *w_cq, *b_cq, *w_ck, *b_ck, *w_cv, *b_cv, *w_hd, *b_hd;
  float *qv, *u, *g, *cst;  // [N, d], [N, d], [N, d], [N]
};

// Workgroups of a stage: q_v takes four rows of W_cq each, the column sums 32 columns each.
__host__ __device__ constexpr int psm_fold_blocks(int stage, int d) {
  return stage == 0 ? 0 : (stage == 1 ? d / 4 + d / 32 : d / 32);
}
constexpr int kFoldViews = 8;  // views of one pass
constexpr int kFoldLds = (kFoldViews * 512 + 4 * kFoldViews * 32) * 4;

__device__ __forceinline__ float psm_wave_sum(float x) { return sum_xor32(sum_xor16(row16_sum(x))); }

// out[v][c] = sum_j w[v][j] W[j][c] for 32 columns c: thread (float4 piece tid
// % 8 of the columns, rows j = tid/8 mod 32), its W pieces all requested at
// once, the views' w rows in LDS; sums over the wave's eight row groups by
// lane exchanges, over the waves through LDS in wave order.
template <int D>
__device__ void psm_fold_cols(const float* __restrict__ W, const float* __restrict__ w, float* __restrict__ out, int c0,
                              int n_views, float* lds) {
  constexpr int NJ = D / 32;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, c4 = tid & 7, jg = tid >> 3;
  float* red = lds + kFoldViews * 512;
  float4 x[NJ];
#pragma unroll
  for (int i = 0; i < NJ; ++i) x[i] = *reinterpret_cast<const float4*>(W + (size_t)(jg + 32 * i) * D + c0 + 4 * c4);
  for (int v0 = 0; v0 < n_views; v0 += kFoldViews) {
    const int nv = min(kFoldViews, n_views - v0);
    for (int i = tid; i < nv * D; i += 256) lds[i] = w[(size_t)v0 * D + i];
    __syncthreads();
    for (int v = 0; v < nv; ++v) {
      float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int i = 0; i < NJ; ++i) {
        const float f = lds[v * D + jg + 32 * i];
        s = make_float4(fmaf(f, x[i].x, s.x), fmaf(f, x[i].y, s.y), fmaf(f, x[i].z, s.z), fmaf(f, x[i].w, s.w));
      }
      s = make_float4(s.x + dpp<0x128>(s.x), s.y + dpp<0x128>(s.y), s.z + dpp<0x128>(s.z), s.w + dpp<0x128>(s.w));  // row_ror:8
      s = make_float4(sum_xor32(sum_xor16(s.x)), sum_xor32(sum_xor16(s.y)), sum_xor32(sum_xor16(s.z)),
                      sum_xor32(sum_xor16(s.w)));
      if (lane < 8) *reinterpret_cast<float4*>(red + (v * 4 + wv) * 32 + 4 * c4) = s;
    }
    __syncthreads();
    if (tid < 32 * nv) {
      const int v = tid >> 5, c = tid & 31;
      out[(size_t)(v0 + v) * D + c0 + c] =
          ((red[v * 128 + c] + red[v * 128 + 32 + c]) + red[v * 128 + 64 + c]) + red[v * 128 + 96 + c];
    }
    __syncthreads();
  }
}

template <int D>
__device__ void psm_fold(const PsmFold& f, int blk, float* lds) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (f.stage == 2) {
    psm_fold_cols<D>(f.w_ck, f.qv, f.u, 32 * blk, f.n_views, lds);
    return;
  }
  if (blk >= D / 4) {
    psm_fold_cols<D>(f.w_cv, f.w_hd, f.g, 32 * (blk - D / 4), f.n_views, lds);
    return;
  }
  // q_v[j] for row j = 4*blk + w of W_cq
  constexpr int P = D / 256;  // float4 pieces per lane
  const int j = 4 * blk + w;
  float4 x[P];
#pragma unroll
  for (int i = 0; i < P; ++i) x[i] = reinterpret_cast<const float4*>(f.w_cq + (size_t)j * D)[lane + 64 * i];
  for (int v0 = 0; v0 < f.n_views; v0 += 8) {  // eight latents in flight
    float s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float4* l4 = reinterpret_cast<const float4*>(f.lat + (size_t)min(v0 + e, f.n_views - 1) * D) + lane;
      s[e] = 0.f;
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const float4 l = l4[64 * i];
        s[e] = fmaf(x[i].x, l.x, fmaf(x[i].y, l.y, fmaf(x[i].z, l.z, fmaf(x[i].w, l.w, s[e]))));
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float t = psm_wave_sum(s[e]);
      if (lane == 0 && v0 + e < f.n_views) f.qv[(size_t)(v0 + e) * D + j] = t + f.b_cq[j];
    }
  }
  // cst_v: view v by wave v % 4 of workgroup v / 4 (of at most 16)
  const int v = 4 * blk + w;
  if (v < f.n_views) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
      s = fmaf(f.w_hd[(size_t)v * D + lane + 64 * i], f.b_cv[lane + 64 * i], s);
      // b_ck adds a constant to every token's logit, which the softmax cancels
      // unless it is no number or infinite
      s = fmaf(0.f, f.b_ck[lane + 64 * i], s);
    }
    s = psm_wave_sum(s);
    if (lane == 0) f.cst[v] = s + f.b_hd[v];
  }
}

struct PsmGemm {
  const uint16_t* x;   // bf16 A [M, K], or
  const float* src;    // fp32 rows [M, K] to be normalised with gain g, bias bt
  const float *g, *bt;
  const float *W, *bias;  // [N, K], [N]
  int M, N, K;
  uint16_t *o0, *o1, *o2;  // bf16 outputs
  float* h;                // fp32 residual stream
  const float* rsrc;       // what the residual is added to (may be h itself)
  int32_t* cu;             // row offsets to write (first launch), or NULL
  int B, T;
  int mt, nt, per_xcd;     // tiles, and items per XCD
  PsmFold fold;
};

// out = A W^T + bias for one BM x BN output tile per workgroup: NW waves as 2 x
// NW/2, each its share of the tile in 16 x 16 MFMA blocks. KG = 2: two such wave
// groups take alternate chunks of the k range, their sums added through LDS.
//
// Bound by latency at a few hundred rows: one query (128 rows, d 256) takes 4.5
// to 6.5 us a launch, of which the arithmetic is under 0.1 us. What this form
// replaced read operands of 32 rows x 32 bytes an instruction in four dependent
// steps, the norm's statistics before them (QKV 9.3 us, up 9.9 us; batch 8:
// 21 and 32 us).
//
// LND = 0: A is bf16 x [M, K], staged in chunks beside W's. LND = d = K: A is
// the LayerNorm (eps 1e-5) of the fp32 rows src, formed once into an LDS panel
// of whole rows; 16 lanes hold a row in registers, so the mean and the squared
// deviations are two register passes. A chunk is 8192 values of W (KC columns,
// 32 KB fp32): each thread asks for 128 bytes of it in 16-byte pieces, whole
// rows to a wave, two chunks ahead of use. The chunk is rounded to bf16 into
// LDS rows whose 16-byte pieces are XOR-swizzled, so that the operand reads
// (16 rows x 1 piece) are conflict-free.
//
// The products are formed transposed (W rows as the A operand), so a lane ends
// with four consecutive output columns of one row.
//
// Modes: kOutBf16 to o0, o1, o2 (equal thirds of N); kOutGelu bf16 gelu(.) to
// o0; kOutResid h = rsrc + (.).
template <int MODE, int LND, int BM, int BN, int NW, int KG>
__global__ __launch_bounds__(64 * NW * KG, 2) void psm_gemm_kernel(PsmGemm p) {
  constexpr int KC = 8192 / BN;                 // columns per chunk
  constexpr int NPW = KC / 8;                   // 16-byte pieces per staged W (and bf16 A) row
  constexpr int ARB = LND ? 2 * LND : 2 * KC;   // bytes per LDS row of A
  constexpr int NPA = ARB / 16;
  constexpr int AB = BM * ARB, WB = BN * 2 * KC;
  constexpr int NT = 64 * NW;                   // threads of a k group
  constexpr int WM = BM / 2, WN = BN / (NW / 2);  // a wave's tile
  constexpr int FM = WM / 16, FN = WN / 16;     // 16 x 16 blocks per wave
  constexpr int WL = 2048 / NT;                 // 16-byte loads of W per thread and chunk
  constexpr int AL = LND ? 1 : BM * KC / 8 / NT;  // 16-byte loads of bf16 A per thread and chunk
  static_assert(LND || BM * KC % (8 * NT) == 0, "the bf16 chunk splits over the threads");
  constexpr int GB = AB + WB;  // LDS bytes per k group
  static_assert(LND == 0 || KG == 1, "the panel serves one k group");
  static_assert(KG == 1 || FM * FN * 16 * NT <= GB, "a group's accumulators fit its chunk buffers");
  __shared__ __attribute__((aligned(1024))) uint8_t lds_all[KG * GB];
  const int tid = threadIdx.x % NT, lane = tid & 63;
  const int kg = __builtin_amdgcn_readfirstlane(threadIdx.x / NT), w = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint8_t* lds = lds_all + kg * GB;
  uint8_t* wl = lds + AB;
  // an XCD takes a contiguous range of items: whole column tiles, whose W rows
  // all their row tiles then find in one L2
  const int n_items = p.mt * p.nt;
  if ((int)blockIdx.x >= 8 * p.per_xcd) {
    static_assert(GB >= kFoldLds, "the fold's rows and partial sums fit");
    if (threadIdx.x >= 256) return;
    if (p.fold.d == 512) psm_fold<512>(p.fold, blockIdx.x - 8 * p.per_xcd, reinterpret_cast<float*>(lds));
    else psm_fold<256>(p.fold, blockIdx.x - 8 * p.per_xcd, reinterpret_cast<float*>(lds));
    return;
  }
  const int item = (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
  if (p.cu && blockIdx.x == 0)
    for (int t = tid; t <= p.B; t += NT) p.cu[t] = t * p.T;
  if (item >= n_items) return;
  const int m0 = (item % p.mt) * BM, n0 = (item / p.mt) * BN;
  const int K = p.K, nch = (K + KC * KG - 1) / (KC * KG);  // chunks per k group: KG*c + kg
  auto swz_w = [](int row) { return NPW >= 16 ? row & 15 : (row >> 1) & (NPW - 1); };
  auto swz_a = [](int row) { return NPA >= 16 ? row & 15 : (row >> 1) & (NPA - 1); };

  // ---- chunk loads into registers: W (fp32) and, without the panel, A (bf16)
  float4 wr[2][WL];
  psm_u32x4 ar[2][AL];
  auto load_chunk = [&](int c, float4 (&wd)[WL], psm_u32x4 (&ad)[AL]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int q = tid + NT * i, row = q / (KC / 4), col = (KG * c + kg) * KC + (q % (KC / 4)) * 4;
      // columns past K (a last chunk cut short) are zero
      wd[i] = col < K ? *reinterpret_cast<const float4*>(p.W + (size_t)(n0 + row) * K + col) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if constexpr (LND == 0) {
#pragma unroll
      for (int i = 0; i < AL; ++i) {
        const int q = tid + NT * i, row = q / NPW, col = (KG * c + kg) * KC + (q % NPW) * 8;
        ad[i] = col < K ? *reinterpret_cast<const psm_u32x4*>(p.x + (size_t)min(m0 + row, p.M - 1) * K + col) : psm_u32x4{0, 0, 0, 0};
      }
    }
  };
  auto store_chunk = [&](const float4 (&wd)[WL], const psm_u32x4 (&ad)[AL]) __attribute__((always_inline)) {
    if constexpr (LND == 0) {
#pragma unroll
      for (int i = 0; i < AL; ++i) {
        const int q = tid + NT * i, row = q / NPW, pc = q % NPW;
        *reinterpret_cast<psm_u32x4*>(lds + row * ARB + ((pc ^ swz_a(row)) * 16)) = ad[i];
      }
    }
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int q = tid + NT * i, row = q / (KC / 4), c4 = q % (KC / 4);
      const psm_u32x2 v = {psm_pk(wd[i].x, wd[i].y), psm_pk(wd[i].z, wd[i].w)};
      *reinterpret_cast<psm_u32x2*>(wl + row * (2 * KC) + (((c4 >> 1) ^ swz_w(row)) * 16) + (c4 & 1) * 8) = v;
    }
  };

  if constexpr (LND != 0) {
    // ---- the normalised rows: row 4*NW*it + 4*w + lane/16, lane li of its 16
    // holding columns 4*(li + 16*j) .. +3
    constexpr int J = LND / 64, IT = BM / (4 * NW);
    const int li = lane & 15, r4 = 4 * w + (lane >> 4);
    auto load_row = [&](int it, float4 (&x)[J]) __attribute__((always_inline)) {
      const float4* xr = reinterpret_cast<const float4*>(p.src + (size_t)min(m0 + 4 * NW * it + r4, p.M - 1) * LND) + li;
#pragma unroll
      for (int j = 0; j < J; ++j) x[j] = xr[16 * j];
    };
    constexpr int XD = IT < 4 * 256 / LND ? IT : 4 * 256 / LND;  // rows in flight per lane
    float4 x[XD][J], gg[J], bb[J];
#pragma unroll
    for (int it = 0; it < XD; ++it) load_row(it, x[it]);
#pragma unroll
    for (int j = 0; j < J; ++j) {
      gg[j] = reinterpret_cast<const float4*>(p.g)[li + 16 * j];
      bb[j] = reinterpret_cast<const float4*>(p.bt)[li + 16 * j];
    }
    load_chunk(0, wr[0], ar[0]);
    auto norm_row = [&](int it, const float4 (&x)[J]) __attribute__((always_inline)) {
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < J; ++j) s += (x[j].x + x[j].y) + (x[j].z + x[j].w);
      const float mu = row16_sum(s) * (1.f / LND);
      float v = 0.f;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const float a = x[j].x - mu, b = x[j].y - mu, c = x[j].z - mu, e = x[j].w - mu;
        v = fmaf(a, a, fmaf(b, b, fmaf(c, c, fmaf(e, e, v))));
      }
      const float rstd = 1.f / sqrtf(row16_sum(v) * (1.f / LND) + 1e-5f);
      const int row = 4 * NW * it + r4;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int c4 = li + 16 * j;
        const psm_u32x2 y = {psm_pk(fmaf((x[j].x - mu) * rstd, gg[j].x, bb[j].x), fmaf((x[j].y - mu) * rstd, gg[j].y, bb[j].y)),
                             psm_pk(fmaf((x[j].z - mu) * rstd, gg[j].z, bb[j].z), fmaf((x[j].w - mu) * rstd, gg[j].w, bb[j].w))};
        *reinterpret_cast<psm_u32x2*>(lds + row * ARB + (((c4 >> 1) ^ swz_a(row)) * 16) + (c4 & 1) * 8) = y;
      }
    };
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      norm_row(it, x[it % XD]);
      if (it + XD < IT) load_row(it + XD, x[it % XD]);
    }
  } else {
    load_chunk(0, wr[0], ar[0]);
  }
  if (nch > 1) load_chunk(1, wr[1], ar[1]);

  const int wm = w & 1, wn = w >> 1;  // the wave's tile
  const int l16 = lane & 15, kq = lane >> 4;
  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto chunk = [&](int c, float4 (&wd)[WL], psm_u32x4 (&ad)[AL]) __attribute__((always_inline)) {
    store_chunk(wd, ad);
    __syncthreads();
    if (c + 2 < nch) load_chunk(c + 2, wd, ad);
#pragma unroll
    for (int ks = 0; ks < KC / 32; ++ks) {
      const int pw = 4 * ks + kq, pa = (LND ? c * (KC / 8) : 0) + pw;
      if (LND == 0 || c * KC + 32 * ks < LND) {
        bf16x8 a[FM], b[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const int row = wm * WM + 16 * i + l16;
          a[i] = *reinterpret_cast<const bf16x8*>(lds + row * ARB + ((pa ^ swz_a(row)) * 16));
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int row = wn * WN + 16 * j + l16;
          b[j] = *reinterpret_cast<const bf16x8*>(wl + row * (2 * KC) + ((pw ^ swz_w(row)) * 16));
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
      }
    }
    __syncthreads();
  };
  // what the epilogue reads is asked for now, with the first chunks
  float4 bc[FN], rs[MODE == kOutResid ? FM : 1][FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int n = n0 + wn * WN + 16 * j + 4 * kq;
    bc[j] = *reinterpret_cast<const float4*>(p.bias + n);
    if constexpr (MODE == kOutResid) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
        rs[i][j] = *reinterpret_cast<const float4*>(
            p.rsrc + (size_t)min(m0 + wm * WM + 16 * i + l16, p.M - 1) * p.N + n);
    }
  }
  for (int c = 0; c < nch; c += 2) {
    chunk(c, wr[0], ar[0]);
    if (c + 1 < nch) chunk(c + 1, wr[1], ar[1]);
  }

  if constexpr (KG > 1) {
    // the k groups' sums, added in group order (the last chunk's reads are done)
    if (kg > 0) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) *reinterpret_cast<f32x4*>(lds + ((i * FN + j) * NT + tid) * 16) = acc[i][j];
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int x = 1; x < KG; ++x)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] += *reinterpret_cast<const f32x4*>(lds_all + x * GB + ((i * FN + j) * NT + tid) * 16);
  }

  // ---- lane: row l16 of block i, columns 4*kq .. +3 of block j
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int n = n0 + wn * WN + 16 * j + 4 * kq;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int row = m0 + wm * WM + 16 * i + l16;
      if (row >= p.M) continue;
      float v[4] = {acc[i][j][0] + bc[j].x, acc[i][j][1] + bc[j].y, acc[i][j][2] + bc[j].z, acc[i][j][3] + bc[j].w};
      if constexpr (MODE == kOutResid) {
        const float4 r = rs[i][j];
        *reinterpret_cast<float4*>(p.h + (size_t)row * p.N + n) = make_float4(r.x + v[0], r.y + v[1], r.z + v[2], r.w + v[3]);
      } else {
        int ld = p.N, col = n;
        uint16_t* o = p.o0;
        if constexpr (MODE == kOutBf16) {
          ld = p.N / 3;
          const int sp = n / ld;
          col = n - sp * ld;
          o = sp == 0 ? p.o0 : (sp == 1 ? p.o1 : p.o2);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
        }
        *reinterpret_cast<psm_u32x2*>(o + (size_t)row * ld + col) = psm_u32x2{psm_pk(v[0], v[1]), psm_pk(v[2], v[3])};
      }
    }
  }
}

// View logits of views VPW*blockIdx.x .. and sample blockIdx.y from the folded
// latents: with x_t the final LayerNorm of token t, logit_v = sum_t
// softmax_t(x_t . u_v / sqrt(d)) (x_t . g_v) + cst_v (a constant in the softmax
// argument cancels). 16 lanes take a token row (NG rows at a time), hold it in
// registers and keep a running softmax of their rows; the gain and bias of the
// norm are folded into the lane's share of u and g first. fp32 throughout.
constexpr int psm_head_threads(int D) { return D == 512 ? 512 : 1024; }  // what the registers allow
template <int D>
__global__ __launch_bounds__(psm_head_threads(D)) void psm_head_kernel(const float* __restrict__ h, const float* __restrict__ gf,
                                                        const float* __restrict__ bf, const float* __restrict__ u,
                                                        const float* __restrict__ g, const float* __restrict__ cst,
                                                        float* __restrict__ logit, int T, int n_views) {
  constexpr int J = D / 64, VPW = 512 / D;  // float4 pieces per lane; views per workgroup
  constexpr int NG = psm_head_threads(D) / 16;
  __shared__ float part[3][VPW][NG];
  const int tid = threadIdx.x, li = tid & 15, grp = tid >> 4, b = blockIdx.y, v0 = blockIdx.x * VPW;
  const float4* hb = reinterpret_cast<const float4*>(h + (size_t)b * T * D) + li;
  auto load_row = [&](int t, float4 (&x)[J]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < J; ++j) x[j] = hb[(size_t)min(t, T - 1) * (D / 4) + 16 * j];
  };
  float4 x[J], nx[J], uu[VPW][J], gg[VPW][J];
  load_row(grp, x);
  float cg[VPW];
#pragma unroll
  for (int v = 0; v < VPW; ++v) {
    const int vv = min(v0 + v, n_views - 1);
    cg[v] = 0.f;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const float4 w = reinterpret_cast<const float4*>(gf)[li + 16 * j], o = reinterpret_cast<const float4*>(bf)[li + 16 * j];
      const float4 a = reinterpret_cast<const float4*>(u + (size_t)vv * D)[li + 16 * j];
      const float4 c = reinterpret_cast<const float4*>(g + (size_t)vv * D)[li + 16 * j];
      uu[v][j] = make_float4(a.x * w.x, a.y * w.y, a.z * w.z, a.w * w.w);
      gg[v][j] = make_float4(c.x * w.x, c.y * w.y, c.z * w.z, c.w * w.w);
      cg[v] = fmaf(c.x, o.x, fmaf(c.y, o.y, fmaf(c.z, o.z, fmaf(c.w, o.w, cg[v]))));
    }
    cg[v] = row16_sum(cg[v]);
  }
  const float scale = kLog2e / sqrtf((float)D);
  float m[VPW], l[VPW], z[VPW];
#pragma unroll
  for (int v = 0; v < VPW; ++v) {
    m[v] = -INFINITY;
    l[v] = 0.f;
    z[v] = 0.f;
  }
  for (int t = grp; t < T; t += NG) {
    if (t + NG < T) load_row(t + NG, nx);
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < J; ++j) s += (x[j].x + x[j].y) + (x[j].z + x[j].w);
    const float mu = row16_sum(s) * (1.f / D);
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      x[j] = make_float4(x[j].x - mu, x[j].y - mu, x[j].z - mu, x[j].w - mu);
      q = fmaf(x[j].x, x[j].x, fmaf(x[j].y, x[j].y, fmaf(x[j].z, x[j].z, fmaf(x[j].w, x[j].w, q))));
    }
    const float rstd = 1.f / sqrtf(row16_sum(q) * (1.f / D) + 1e-5f);
#pragma unroll
    for (int v = 0; v < VPW; ++v) {
      float a = 0.f, c = 0.f;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        a = fmaf(x[j].x, uu[v][j].x, fmaf(x[j].y, uu[v][j].y, fmaf(x[j].z, uu[v][j].z, fmaf(x[j].w, uu[v][j].w, a))));
        c = fmaf(x[j].x, gg[v][j].x, fmaf(x[j].y, gg[v][j].y, fmaf(x[j].z, gg[v][j].z, fmaf(x[j].w, gg[v][j].w, c))));
      }
      a = row16_sum(a) * rstd * scale;
      c = row16_sum(c) * rstd;
      // a row at -inf has no weight, before the first finite one too
      const float mn = fmaxf(m[v], a), ms = mn == -INFINITY ? 0.f : mn;
      const float al = __builtin_amdgcn_exp2f(m[v] - ms), e = __builtin_amdgcn_exp2f(a - ms);  // first row: al = exp2(-inf) = 0
      l[v] = fmaf(l[v], al, e);
      z[v] = fmaf(z[v], al, e * c);
      m[v] = mn;
    }
#pragma unroll
    for (int j = 0; j < J; ++j) x[j] = nx[j];
  }
#pragma unroll
  for (int v = 0; v < VPW; ++v)
    if (li == 0) {
      part[0][v][grp] = m[v];
      part[1][v][grp] = l[v];
      part[2][v][grp] = z[v];
    }
  __syncthreads();
  // wave v merges the groups of view v (a group without a row: max -inf, sums 0)
  const int v = tid >> 6, lane = tid & 63, gl = min(lane, NG - 1);
  if (v >= VPW || v0 + v >= n_views) return;
  const float mm = lane < NG ? part[0][v][gl] : -INFINITY;
  float mx = mm;
#pragma unroll
  for (int i = 1; i < kWave; i <<= 1) mx = wave_max_xor(mx, i);
  const float wgt = __builtin_amdgcn_exp2f(mm - mx);
  const float ls = psm_wave_sum(part[1][v][gl] * wgt), zs = psm_wave_sum(part[2][v][gl] * wgt);
  float cgv = cg[0];
#pragma unroll
  for (int i = 1; i < VPW; ++i) cgv = v == i ? cg[i] : cgv;
  if (lane == 0) logit[(size_t)b * n_views + v0 + v] = zs / ls + (cgv + cst[v0 + v]);
}

template <int MODE, int LND, int BM, int BN, int NW, int KG>
void gemm_launch(PsmGemm& p, hipStream_t s) {
  p.mt = (p.M + BM - 1) / BM;
  p.nt = p.N / BN;
  p.per_xcd = (p.mt * p.nt + 7) / 8;
  const int grid = 8 * p.per_xcd + psm_fold_blocks(p.fold.stage, p.fold.d);
  hipLaunchKernelGGL((psm_gemm_kernel<MODE, LND, BM, BN, NW, KG>), dim3(grid), dim3(64 * NW * KG), 0, s, p);
}

// Tile by the number of workgroups it gives (256 CUs). A 32 x 32 tile is one
// round trip of loads per workgroup, the shortest launch while the grid is
// small; past 192 tiles of 64 x 64 their halved cache traffic wins (batch 8 of
// 128 tokens, d 256: QKV 6.4 against 8.0 us, up 7.9 against 11.0 us), with eight
// waves to share a tile's loads and norm (four: 7.1 and 8.8 us). From 512 tiles
// of 64 x 128 on, bandwidth counts and four waves of 32 x 64 read LDS least
// (3200 x 2048 x 512: 36 us, 64 x 64 tiles 49 us, eight waves 51 us); without
// the norm four waves serve 64 x 64 too (3200 x 512 x 2048: 18.4 against 23.4).
// Around the line of 192 (whole forwards, 4 layers, with 32 x 32 tiles on both
// sides / as here / from 96 tiles on): 8 x 96 rows, d 256, up at 192 tiles 136 / 133
// / 129 us; 8 x 128, QKV at 192 149 / 139 / 139; 4 x 112, d 512, QKV at 168 189 / 173
// / 163; 8 x 192, d 256, output and down projection at 96 174 / 165 / 184; 4 x 192, d
// 512, the same at 96 249 / 232 / 262. The GEMMs with the norm would gain from a
// lower line, those without lose more by it.
// A long k range on few 32 x 32 tiles is shared by two wave groups, so that
// all of it is in flight at once (128 x 256 x 1024: 6.3 against 7.0 us).
template <int MODE, int LND>
void gemm(PsmGemm& p, hipStream_t s) {
  auto tiles = [&](int bm, int bn) { return (long long)((p.M + bm - 1) / bm) * (p.N / bn); };
  if (p.N % 128 == 0 && tiles(64, 128) >= 512) gemm_launch<MODE, LND, 64, 128, 4, 1>(p, s);
  else if (tiles(64, 64) >= 192) gemm_launch<MODE, LND, 64, 64, LND ? 8 : 4, 1>(p, s);
  else if (LND == 0 && p.K >= 512 && tiles(32, 32) < 256) gemm_launch<MODE, LND, 32, 32, 4, LND ? 1 : 2>(p, s);
  else gemm_launch<MODE, LND, 32, 32, 4, 1>(p, s);
}

template <int D>
hipError_t run(const PsmArgs& a, hipStream_t s) {
  const PsmLayout L = psm_layout(a.B, a.T, a.d, a.d_ff, a.n_views, a.n_layers);
  const int M = a.B * a.T, d = a.d, dff = a.d_ff, B = a.B, T = a.T;
  uint8_t* ws = static_cast<uint8_t*>(a.workspace);
  float* h = reinterpret_cast<float*>(ws + L.h_off);
  uint16_t* q = reinterpret_cast<uint16_t*>(ws + L.q_off);
  uint16_t* k = reinterpret_cast<uint16_t*>(ws + L.k_off);
  uint16_t* v = reinterpret_cast<uint16_t*>(ws + L.v_off);
  uint16_t* att = reinterpret_cast<uint16_t*>(ws + L.att_off);
  uint16_t* ff = reinterpret_cast<uint16_t*>(ws + L.ff_off);
  int32_t* cu = reinterpret_cast<int32_t*>(ws + L.cu_off);
  const float* P = a.params;
  const float* fp = P + (size_t)a.n_layers * L.layer_params;
  const float* lnf_g = fp;
  const float* lnf_b = lnf_g + d;
  PsmFold fold;
  fold.d = d;
  fold.n_views = a.n_views;
  fold.lat = lnf_b + d;
  fold.w_cq = fold.lat + (size_t)a.n_views * d;
  fold.b_cq = fold.w_cq + (size_t)d * d;
  fold.w_ck = fold.b_cq + d;
  fold.b_ck = fold.w_ck + (size_t)d * d;
  fold.w_cv = fold.b_ck + d;
  fold.b_cv = fold.w_cv + (size_t)d * d;
  fold.w_hd = fold.b_cv + d;
  fold.b_hd = fold.w_hd + (size_t)a.n_views * d;
  fold.qv = reinterpret_cast<float*>(ws + L.fold_off);
  fold.u = fold.qv + (size_t)a.n_views * d;
  fold.g = fold.u + (size_t)a.n_views * d;
  fold.cst = fold.g + (size_t)a.n_views * d;
  for (int i = 0; i < a.n_layers; ++i) {
    const float* lp = P + (size_t)i * L.layer_params;
    const float* ln1_g = lp;
    const float* ln1_b = ln1_g + d;
    const float* w_qkv = ln1_b + d;
    const float* b_qkv = w_qkv + (size_t)3 * d * d;
    const float* w_o = b_qkv + 3 * d;
    const float* b_o = w_o + (size_t)d * d;
    const float* ln2_g = b_o + d;
    const float* ln2_b = ln2_g + d;
    const float* w_up = ln2_b + d;
    const float* b_up = w_up + (size_t)dff * d;
    const float* w_dn = b_up + dff;
    const float* b_dn = w_dn + (size_t)d * dff;
    auto args = [&](const float* W, const float* bias, int N, int K, int stage) {
      PsmGemm p{};
      p.W = W;
      p.bias = bias;
      p.M = M;
      p.N = N;
      p.K = K;
      p.fold = fold;
      p.fold.stage = stage;
      return p;
    };
    // the first layer reads the embeddings; its first residual add seeds h
    PsmGemm p1 = args(w_qkv, b_qkv, 3 * d, d, i == 0 ? 1 : 0);
    p1.src = i == 0 ? a.emb : h;
    p1.g = ln1_g;
    p1.bt = ln1_b;
    p1.o0 = q;
    p1.o1 = k;
    p1.o2 = v;
    p1.cu = i == 0 ? cu : nullptr;
    p1.B = B;
    p1.T = T;
    gemm<kOutBf16, D>(p1, s);
    AttnArgs at;
    at.in_dtype = LITEVLM_BF16;
    at.out_dtype = LITEVLM_BF16;
    at.B = B;
    at.Hq = a.n_heads;
    at.Hkv = a.n_heads;
    at.D = d / a.n_heads;
    at.max_seqlen = T;
    at.causal = 0;
    at.q = q;
    at.k = k;
    at.v = v;
    at.cu_seqlens = cu;
    at.logit_scale_log2 = (float)(1.4426950408889634 / sqrt((double)at.D));
    at.out_scale = 1.f;
    at.o = att;
    const hipError_t e = launch_prefill_attn(at, s);
    if (e != hipSuccess) return e;
    PsmGemm p2 = args(w_o, b_o, d, d, i == 0 ? 2 : 0);
    p2.x = att;
    p2.h = h;
    p2.rsrc = i == 0 ? a.emb : h;
    gemm<kOutResid, 0>(p2, s);
    PsmGemm p3 = args(w_up, b_up, dff, d, 0);
    p3.src = h;
    p3.g = ln2_g;
    p3.bt = ln2_b;
    p3.o0 = ff;
    gemm<kOutGelu, D>(p3, s);
    PsmGemm p4 = args(w_dn, b_dn, d, dff, 0);
    p4.x = ff;
    p4.h = h;
    p4.rsrc = h;
    gemm<kOutResid, 0>(p4, s);
  }
  constexpr int VPW = 512 / D;
  hipLaunchKernelGGL((psm_head_kernel<D>), dim3((a.n_views + VPW - 1) / VPW, B),
                     dim3(psm_head_threads(D)), 0, s, h, lnf_g, lnf_b,
                     fold.u, fold.g, fold.cst, a.view_logit, T, a.n_views);
  return hipGetLastError();
}

}  // namespace

PsmLayout psm_layout(int B, int T, int d, int d_ff, int n_views, int n_layers) {
  PsmLayout L;
  L.layer_params = (size_t)4 * d + (size_t)3 * d * d + 3 * d + (size_t)d * d + d + (size_t)d_ff * d + d_ff +
                   (size_t)d * d_ff + d;
  L.params = (size_t)n_layers * L.layer_params + 2 * (size_t)d + (size_t)n_views * d + 3 * ((size_t)d * d + d) +
             (size_t)n_views * d + n_views;
  const size_t M = (size_t)B * T;
  auto a256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
  size_t off = 0;
  L.h_off = off;
  off = a256(off + M * d * 4);
  L.q_off = off;
  off = a256(off + M * d * 2);
  L.k_off = off;
  off = a256(off + M * d * 2);
  L.v_off = off;
  off = a256(off + M * d * 2);
  L.att_off = off;
  off = a256(off + M * d * 2);
  L.ff_off = off;
  off = a256(off + M * d_ff * 2);
  L.cu_off = off;
  off = a256(off + (size_t)(B + 1) * 4);
  // the folded latents of up to LITEVLM_MAX_VIEWS views (the size is asked for
  // without their number): q_v, u_v, g_v [d] and one constant each
  L.fold_off = off;
  off = a256(off + (size_t)LITEVLM_MAX_VIEWS * (3 * (size_t)d + 1) * 4);
  L.total = off;
  return L;
}

hipError_t launch_psm_forward(const PsmArgs& a, hipStream_t stream) {
  return a.d == 512 ? run<512>(a, stream) : run<256>(a, stream);
}

}  // namespace litevlm
