// Token Selection Module front end: the scoring queries and keys of the
// standalone first decoder layer, from the layer's input hidden states.
//
//   k[b, j]   = rope(r_j * x[b, j] W_k'^T, pos_j)   for every kept token j
//   q[b, t]   = rope(r_t * x[b, t] W_q'^T, pos_t)   for the text tokens t
//   r_j       = 1 / sqrt(mean_c x[b, j, c]^2 + eps)  (RMS normalisation)
//   pos_j     = number of kept tokens before j (positions of the patch-selected sequence)
//
// W' carries the normalisation gain (W'[n, c] = W[n, c] * gamma[c],
// tsm_fold_gain_kernel), so the projection is a plain bf16 GEMM on MFMA with
// fp32 accumulation, and the RMS factor and the rotary embedding are applied
// in its epilogue:
//   - the sum of squares of each row comes from the A operands the waves
//     already hold for the MFMAs (no second pass over x);
//   - a wave owns two column blocks that are rotary partners (elements d and
//     d + D/2 of one head), so the rotation is lane-local in the accumulators.
//
// Bound: MFMA in principle (about 730 flop per HBM byte), in fact the copies of
// the tiles from L2: without them the loop of the 256 x 256 tile takes 0.88 us a
// 64-column stage, its MFMA time, with them 1.5 us. So a tile is as large as it can
// be without a further round of the chip (the rule at the launch; eight prompts
// take 128 x 256), and its rows are staged in whole 128-byte lines (64 columns; with
// half lines the 128 x 128 tile took 430 against 394 us at batch 8).
// A workgroup is 4 waves (2 x 2), one wave per SIMD for the large tiles with the
// accumulators in the AGPRs; a wave's share of the tile is then so large (128 x
// 128 of the 256 x 256) that its LDS reads stay below the LDS rate. Global -> LDS
// copies are buffer loads (no vector arithmetic, half the address traffic) spread
// over the MFMAs. Two wave groups in turns on a SIMD (8 waves, one reading LDS
// while the other multiplies) took 380 us at batch 8 where one takes 361, both in
// 256 x 256 tiles.
//
// Epilogue: the rotation angle is reduced to [-1/2, 1/2] turns in double and
// taken by the hardware sine and cosine (which work in turns), and the rotated
// tile is staged through the free ring as bf16 rows so that it leaves in
// 16-byte stores of whole rows; the accumulators hold one feature per lane.
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace litevlm {
namespace {

constexpr int kNW = 4, kTh = 64 * kNW;

// Workgroup tile MT rows x NT features over 4 waves (2 x 2), staged KT columns of
// the model width at a time in a ring of R stages.
template <int MT, int NT, int KT, int R_>
struct TsmTile {
  static constexpr int R = R_;
  static constexpr int kPieces = KT / 8;  // 16-byte pieces per staged row
  static constexpr int kRowB = KT * 2;    // bytes per staged row
  static constexpr int kAB = MT * kRowB;  // A tile bytes per stage
  static constexpr int kBB = NT * kRowB;  // B tile bytes per stage
  static constexpr int kStageB = kAB + kBB;
  static constexpr int kRingB = R * kStageB;
  static constexpr int kLdsB = kRingB + MT * 4 /* row factors */ + MT * 4 /* positions */ + 128 /* reductions */ +
                               MT /* keep flags */;
  static constexpr int kWgPerCu = 2 * kLdsB <= 160 * 1024 ? 2 : 1;
  static constexpr int kRB = MT / 64;   // 32-row blocks per wave
  static constexpr int kCBW = NT / 64;  // 32-feature blocks per wave
  static_assert(kRB % 2 == 0 && (kCBW == 2 || kCBW == 4), "tile shape");
  static_assert(kLdsB <= 160 * 1024, "LDS of a workgroup");
};

struct TsmParams {
  const uint8_t* x;     // bf16 [B, S, Dm]
  const uint8_t* keep;  // uint8 [B, S] or NULL
  const uint8_t* wq;    // bf16 [Hq*D, Dm]
  const uint8_t* wk;    // bf16 [Hkv*D, Dm]
  uint16_t* q;          // bf16 [B, S, Hq, D]
  uint16_t* k;          // bf16 [B, S, Hkv, D]
  int B, S, V_full, Dm, Hq, Hkv;
  int mk, nk, mq, nq, gk, gq;           // gk, gq: key and query row tiles (B*mk, B*mq)
  int turn;                             // key row tiles dealt in turn to each XCD
  float eps;
  double log2_theta;
};

template <int N>
__device__ __forceinline__ void vm_wait() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// XOR swizzle of a staged row's pieces. The LDS serves a 16-byte read for 16
// lanes per cycle across 64 banks (256 bytes, 16 / PIECES staged rows): the 16
// consecutive rows such a group reads must put their pieces in distinct 16-byte
// bank slots.
template <int PIECES>
__device__ __forceinline__ int swz(int row) { return PIECES == 4 ? (row >> 2) & 3 : (row >> 1) & 7; }

// Workgroup barrier that waits only for this wave's LDS operations: the
// __syncthreads fence would also wait for every direct copy still in flight,
// which would drain the ring each stage.
__device__ __forceinline__ void ring_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef short s16x4v __attribute__((ext_vector_type(4)));

// Sum of the bytes of x plus c.
__device__ __forceinline__ uint32_t sum_bytes(uint32_t x, uint32_t c) { return __builtin_amdgcn_sad_u8(x, 0u, c); }

template <int D, int MT, int NT, int KT, int R>
__global__ __launch_bounds__(kTh, (TsmTile<MT, NT, KT, R>::kWgPerCu)) void tsm_proj_kernel(TsmParams p) {
  using Tl = TsmTile<MT, NT, KT, R>;
  constexpr int kPieces = Tl::kPieces, kRowB = Tl::kRowB;
  constexpr int kMT = MT, kNT = NT, kAB = Tl::kAB, kBB = Tl::kBB, kStageB = Tl::kStageB, kRingB = Tl::kRingB;
  constexpr int NW = kNW, NWR = 2;
  constexpr int PB = D / 64;     // column-block distance of rotary partners
  constexpr int RB = Tl::kRB;    // 32-row blocks per wave
  constexpr int CBW = Tl::kCBW;  // 32-column blocks per wave
  __shared__ __attribute__((aligned(1024))) uint8_t lds[Tl::kLdsB];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // ---- work item: a key row tile with one of its feature tiles, or a query row
  // tile with one of its. The first 8*turn key row tiles go to the XCDs in turn,
  // each with all its feature tiles (they share its rows of x in that L2); the other
  // items follow in contiguous ranges, equal to within one item.
  bool isq = false;
  int b, mt, nt;
  {
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3, nturn = p.turn * p.nk;
    int grp;
    if (j < nturn) {
      grp = x + 8 * (j / p.nk);
      nt = j % p.nk;
    } else {
      const int nkey = (p.gk - 8 * p.turn) * p.nk, total = nkey + p.gq * p.nq;
      const int i0 = (int)(((int64_t)x * total) >> 3), i1 = (int)(((int64_t)(x + 1) * total) >> 3);
      int item = i0 + j - nturn;
      if (item >= i1) return;
      isq = item >= nkey;
      if (isq) item -= nkey;
      const int per = isq ? p.nq : p.nk;
      grp = item / per;
      nt = item - grp * per;
      if (!isq) grp += 8 * p.turn;
    }
    const int mm = isq ? p.mq : p.mk;
    b = grp / mm;
    mt = grp - b * mm;
  }
  const int row0 = (isq ? p.V_full : 0) + mt * kMT;  // first row of the tile within the sample
  const int nrows = min(kMT, p.S - row0);
  const int n0 = nt * kNT;
  const uint8_t* W = isq ? p.wq : p.wk;
  const int H = isq ? p.Hq : p.Hkv;
  const int Dm = p.Dm;

  float* rs = reinterpret_cast<float*>(lds + kRingB);
  int* pos = reinterpret_cast<int*>(lds + kRingB + kMT * 4);
  int* red = reinterpret_cast<int*>(lds + kRingB + kMT * 8);
  uint8_t* kflag = lds + kRingB + kMT * 8 + 128;

  const int wr = w % NWR, wc = w / NWR, hl = lane >> 5, l32 = lane & 31;

  // ---- copies of a stage (fixed per-lane sources): copy j of a wave fills LDS
  // pieces (w + 4j)*64 + lane of the A (resp. B) tile
  constexpr int CA = kAB / (1024 * NW), CB = kBB / (1024 * NW), CS = CA + CB;  // copies per thread and stage
  static_assert(CA % 2 == 0 && CB % 2 == 0 && CS * (R - 1) <= 63, "copies in halves, vmcnt range");
  const uint8_t* xt = p.x + ((size_t)b * p.S + row0) * Dm * 2;  // the tile's first row
  const uint8_t* wt = W + (size_t)n0 * Dm * 2;                  // the tile's first feature
  uint32_t asrc[CA], bsrc[CB];
#pragma unroll
  for (int j = 0; j < CA; ++j) {
    const int slot = (w + NW * j) * 64 + lane;
    const int row = slot / kPieces, logical = (slot % kPieces) ^ swz<kPieces>(row);
    asrc[j] = (uint32_t)(min(row, nrows - 1) * Dm + logical * 8) * 2;  // < 256 * 65536 * 2
  }
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    const int slot = (w + NW * j) * 64 + lane;
    const int row = slot / kPieces, logical = (slot % kPieces) ^ swz<kPieces>(row);
    bsrc[j] = (uint32_t)(row * Dm + logical * 8) * 2;
  }
  const uint32_t lds_w = __builtin_amdgcn_readfirstlane((uint32_t)w * 1024u);
  const int nK = Dm / KT;
  // copies of stage s (past the end, the last stage's again, into bytes that
  // nothing reads: the loop stays one block of code) in two halves
  auto copy_half = [&](int s, uint32_t slot, int half) __attribute__((always_inline)) {
    const int col = min(s, nK - 1) * kRowB;
    uint8_t* st = lds + slot + lds_w;
#pragma unroll
    for (int j = half * CA / 2; j < (half + 1) * CA / 2; ++j)
      copy16_to_lds(xt, (uint32_t)(nrows * Dm * 2), asrc[j], col, st + NW * j * 1024);
#pragma unroll
    for (int j = half * CB / 2; j < (half + 1) * CB / 2; ++j)
      copy16_to_lds(wt, (uint32_t)(kNT * Dm * 2), bsrc[j], col, st + kAB + NW * j * 1024);
  };
  // the first stages are in flight while the positions are counted
#pragma unroll
  for (int s = 0; s < R; ++s) {
    copy_half(s, s * kStageB, 0);
    if (s < R - 1) copy_half(s, s * kStageB, 1);
  }

  // ---- positions of the tile's rows in the patch-selected sequence
  {
    const uint8_t* kr = p.keep ? p.keep + (size_t)b * p.S : nullptr;
    // kept rows before the tile, 16 bytes a load between an unaligned head and tail
    int cnt = 0;
    if (kr) {
      const int head = min(row0, (int)((16 - (reinterpret_cast<uintptr_t>(kr) & 15)) & 15));
      const int n16 = (row0 - head) / 16, tail = head + 16 * n16;
      const uint4* k16 = reinterpret_cast<const uint4*>(kr + head);
      uint32_t c = 0;
      if (tid < head) c += kr[tid];
      if (tid < row0 - tail) c += kr[tail + tid];
      for (int j = tid; j < n16; j += kTh) {
        const uint4 u = k16[j];
        c = sum_bytes(u.w, sum_bytes(u.z, sum_bytes(u.y, sum_bytes(u.x, c))));
      }
      cnt = (int)c;
    }
#pragma unroll
    for (int x = 1; x < kWave; x <<= 1) cnt += __shfl_xor(cnt, x, kWave);
    if (lane == 0) red[w] = cnt;
    __syncthreads();
    int base = row0;
    if (kr) {
      base = 0;
      for (int x = 0; x < NW; ++x) base += red[x];
    }
    for (int t0 = 0; t0 < kMT; t0 += kTh) {
      const int t = t0 + tid;
      int f = 0;
      if (t < nrows) f = kr ? kr[row0 + t] : 1;
      int incl = f;
#pragma unroll
      for (int x = 1; x < kWave; x <<= 1) {
        const int y = __shfl_up(incl, x, kWave);
        if (lane >= x) incl += y;
      }
      __syncthreads();
      if (lane == kWave - 1) red[NW + w] = incl;
      __syncthreads();
      int before = t0 == 0 ? 0 : red[2 * NW];  // kept rows of the earlier chunks
      for (int x = 0; x < w; ++x) before += red[NW + x];
      if (t < kMT) {
        pos[t] = base + before + (incl - f);
        kflag[t] = (uint8_t)f;
      }
      __syncthreads();
      if (tid == 0) {
        int c = t0 == 0 ? 0 : red[2 * NW];
        for (int x = 0; x < NW; ++x) c += red[NW + x];
        red[2 * NW] = c;
      }
    }
  }

  // ---- a key tile whose rows are all dropped tokens produces nothing: the
  // keys of dropped views are never scored
  if (!isq && p.keep) {
    __syncthreads();
    if (red[2 * NW] == 0) {
      vm_wait<0>();  // the copies into LDS land before the workgroup ends
      return;
    }
  }

  // ---- operand offsets: row (or feature) l32 of a 32-row block, piece 2*ks + hl
  constexpr int KS = KT / 16;  // k16 steps per stage
  uint32_t off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) off[ks] = l32 * kRowB + (((2 * ks + hl) ^ swz<kPieces>(l32)) * 16);
  // this wave's column blocks: rotary partners (blocks PB apart) always together
  int cbl[CBW];
  if constexpr (CBW == 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) cbl[i] = 4 * wc + i;
  } else {  // two waves share a 128-feature span: blocks {c0, c0 + PB}
    cbl[0] = (D == 128) ? wc : 2 * wc;
    cbl[1] = cbl[0] + PB;
  }
  // The two waves of a row half take its 32-row blocks in another order (the second
  // begins with the upper half), so that each sums the squares of its own first
  // RB / 2 blocks without a branch.
  constexpr int HB = RB / 2;
  auto row_block = [&](int rb) { return wr * RB + (rb < HB ? rb + wc * HB : rb - wc * HB); };
  const uint32_t a_lo = __builtin_amdgcn_readfirstlane((uint32_t)row_block(0) * 32u * kRowB);
  const uint32_t a_hi = __builtin_amdgcn_readfirstlane((uint32_t)row_block(HB) * 32u * kRowB);
  const uint32_t b0 = __builtin_amdgcn_readfirstlane((uint32_t)(kAB + cbl[0] * 32 * kRowB));
  constexpr int kCStep = (CBW == 2 ? PB : 1) * 32 * kRowB;  // bytes between the wave's column blocks

  f32x16 acc[RB][CBW];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int c = 0; c < CBW; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[rb][c][r] = 0.f;
  float ssq[HB][2];
#pragma unroll
  for (int rb = 0; rb < HB; ++rb) ssq[rb][0] = ssq[rb][1] = 0.f;

  // One wave per SIMD. The operands of a k16 step are read while the step before
  // it multiplies. One barrier a stage, before its last step: by then every wave
  // holds its last operands of the stage, so its slot is free, and the next
  // stage has landed, so its first operands can be read. A stage's copies are
  // spread over the MFMAs of the two steps after its slot became free, R - 1
  // stages ahead (issued together they hold up the MFMAs).
  bf16x8 a[2][RB], bo[2][CBW];
  auto read_step = [&](int set, uint32_t slot, int ks) __attribute__((always_inline)) {
    const uint8_t* st = lds + slot + off[ks];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      a[set][rb] = *reinterpret_cast<const bf16x8*>(st + (rb < HB ? a_lo : a_hi) + (rb % HB) * 32 * kRowB);
#pragma unroll
    for (int c = 0; c < CBW; ++c) bo[set][c] = *reinterpret_cast<const bf16x8*>(st + b0 + c * kCStep);
  };
  auto multiply = [&](int set) __attribute__((always_inline)) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
      for (int c = 0; c < CBW; ++c)
        acc[rb][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[set][rb], bo[set][c], acc[rb][c], 0, 0, 0);
      // Row sums of squares of the A operands, two vector instructions per MFMA
      // (they run beside it; the packed bf16 dot does not: 0.4 us a 64-column
      // stage of the 256 x 256 tile)
      if (rb < HB) {
        const u32x4v u = __builtin_bit_cast(u32x4v, a[set][rb]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = __uint_as_float(u[e] << 16), hi = __uint_as_float(u[e] & 0xFFFF0000u);
          ssq[rb][0] = fmaf(lo, lo, ssq[rb][0]);
          ssq[rb][1] = fmaf(hi, hi, ssq[rb][1]);
        }
      }
    }
  };
  // MFMAs with the next step's LDS reads and the copies spread among them
  auto interleave = [&]() __attribute__((always_inline)) {
    constexpr int NM = RB * CBW;
#pragma unroll
    for (int i = 0; i < NM / 4; ++i) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  vm_wait<0>();
  ring_barrier();
  read_step(0, 0, 0);
  uint32_t slot = 0, prev = (R - 1) * kStageB;  // slots of stages s and s - 1
  for (int s = 0; s < nK; ++s) {
    const uint32_t next = slot == (R - 1) * kStageB ? 0 : slot + kStageB;
    copy_half(s + R - 1, prev, 1);
#pragma unroll
    for (int ks = 0; ks + 1 < KS; ++ks) {
      read_step((ks + 1) & 1, slot, ks + 1);
      multiply(ks & 1);
      interleave();
    }
    vm_wait<(R - 2) * CS>();  // stage s + 1 has landed: R - 2 stages were issued after it
    ring_barrier();
    copy_half(s + R, slot, 0);
    read_step(0, next, 0);  // past the last stage: bytes of another slot, not used
    multiply(1);
    interleave();
    prev = slot;
    slot = next;
  }
  vm_wait<0>();  // the epilogue writes the ring

  // ---- epilogue: RMS factor per row, rotary embedding, bf16 store
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < HB; ++rb) {
    const float tot = sum_xor32(ssq[rb][0] + ssq[rb][1]);
    if (hl == 0) rs[32 * row_block(rb) + l32] = 1.f / sqrtf(tot / (float)Dm + p.eps);
  }
  __syncthreads();
  // The rotated tile goes through the (now free) ring as bf16 rows of kNT
  // features, 16-byte pieces XOR-swizzled by row, and leaves it in 16-byte
  // stores of whole rows (the accumulators hold one feature per lane).
  static_assert(kMT * kNT * 2 <= kRingB, "output tile exceeds the ring");
  constexpr int kOutRowB = kNT * 2;
  auto out_slot = [&](int row, int col) {
    return row * kOutRowB + ((((col * 2) >> 4) ^ (row & 7)) << 4) + ((col * 2) & 15);
  };
  // Rows 4q .. 4q+3 of one column per lane, as 4-byte stores of two columns: the
  // even lane of a pair takes rows 4q and 4q+2 of both, the odd lane the others.
  const uint32_t pick = (lane & 1) ? 0x03020706u : 0x05040100u;
  auto put4 = [&](int row4, int col, const float (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
      typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
      const uint32_t own = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)v[e], (__bf16)v[e + 1]});
      const uint32_t nb = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0xB1, 0xF, 0xF, false);  // lane ^ 1
      *reinterpret_cast<uint32_t*>(lds + out_slot(row4 + e + (lane & 1), col & ~1)) =
          __builtin_amdgcn_perm(nb, own, pick);
    }
  };
  // sine and cosine of pos * theta^(-2d/D): the angle in turns, reduced to
  // [-1/2, 1/2] in double; the hardware sine and cosine take turns
  auto sincos_turns = [](double t, float& sn, float& cs) __attribute__((always_inline)) {
    t -= rint(t);
    sn = __builtin_amdgcn_sinf((float)t);
    cs = __builtin_amdgcn_cosf((float)t);
  };
  // rotary pairs of this wave's column list: slots c (a first-half block) and
  // cp (its partner, PB blocks on)
  auto rotate_pair = [&](auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value;
    constexpr int c = CBW == 2 ? 0 : (D == 128 ? i : 2 * i);
    constexpr int cp = CBW == 2 ? 1 : c + PB;
    const int col = 32 * cbl[c] + l32;  // tile feature of the first-half element; its partner is D/2 on
    const int d = (32 * cbl[c]) % D + l32;  // element of the first half of its head (d < D/2)
    const double turns_per_pos = exp2(-(2.0 * d / D) * p.log2_theta) * 0.15915494309189535;  // / (2 pi)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row4 = 32 * row_block(rb) + 8 * q + 4 * hl;  // acc_row(4q .. 4q+3, hl)
        const f32x4 f = *reinterpret_cast<const f32x4*>(rs + row4);
        const i32x4 ps = *reinterpret_cast<const i32x4*>(pos + row4);
        float sn[4], cs[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) sincos_turns((double)ps[e] * turns_per_pos, sn[e], cs[e]);
        float y1[4], y2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x1 = acc[rb][c][4 * q + e] * f[e], x2 = acc[rb][cp][4 * q + e] * f[e];
          y1[e] = x1 * cs[e] - x2 * sn[e];
          y2[e] = x2 * cs[e] + x1 * sn[e];
        }
        put4(row4, col, y1);
        put4(row4, col + D / 2, y2);
      }
  };
  rotate_pair(std::integral_constant<int, 0>{});
  if constexpr (CBW == 4) rotate_pair(std::integral_constant<int, 1>{});
  __syncthreads();
  // rows of the tile that exist and are kept (queries: every text row)
  uint16_t* out = isq ? p.q : p.k;
  constexpr int kPiecesPerRow = kOutRowB / 16;
#pragma unroll
  for (int j = 0; j < kMT * kPiecesPerRow / kTh; ++j) {
    const int q = tid + kTh * j;
    const int row = q / kPiecesPerRow, pc = q % kPiecesPerRow;
    if (row < nrows && (isq || kflag[row])) {
      const u32x4v v = *reinterpret_cast<const u32x4v*>(lds + row * kOutRowB + ((pc ^ (row & 7)) << 4));
      *reinterpret_cast<u32x4v*>(out + ((size_t)b * p.S + row0 + row) * H * D + n0 + 8 * pc) = v;
    }
  }
}

// w_out[n, c] = bf16(w[n, c] * gamma[c]): the RMS normalisation gain folded
// into the projection that follows it (done once per set of weights).
__global__ __launch_bounds__(256) void tsm_fold_gain_kernel(const uint16_t* __restrict__ w,
                                                            const float* __restrict__ gamma,
                                                            uint16_t* __restrict__ w_out, int64_t rows, int cols) {
  const int64_t n = rows * cols;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    w_out[i] = f32_to_bf16_bits(bf16_bits_to_f32(w[i]) * gamma[i % cols]);
}

}  // namespace

hipError_t launch_tsm_qk(const TsmArgs& a, hipStream_t stream) {
  TsmParams p;
  p.x = static_cast<const uint8_t*>(a.hidden);
  p.keep = a.token_keep;
  p.wq = static_cast<const uint8_t*>(a.w_q);
  p.wk = static_cast<const uint8_t*>(a.w_k);
  p.q = static_cast<uint16_t*>(a.q);
  p.k = static_cast<uint16_t*>(a.k);
  p.B = a.B;
  p.S = a.S;
  p.V_full = a.V_full;
  p.Dm = a.Dm;
  p.Hq = a.Hq;
  p.Hkv = a.Hkv;
  p.eps = a.eps;
  p.log2_theta = log2((double)a.rope_theta);
  const int T = a.S - a.V_full;
  // A dropped view is a run of row tiles whose workgroups end at once. Dealt in
  // turn the runs spread over the XCDs, where contiguous ranges leave the XCDs
  // that hold them idle (eight prompts of 6 x 1024 visual and 120 text tokens, 0-4
  // views dropped: 410 -> 347 us; one, 3 dropped: 60 -> 51 us). Finding the working
  // tiles from the mask in every workgroup deals them exactly, but costs each 2.3
  // us before its first copy: 356 us for the eight, 54 for the one. It pays only
  // where a tile more or less decides about a round of the chip (five prompts, 32/8
  // heads of 64, width 1024, 3 of 30 views dropped: 56 against 65 us). Below four
  // tiles an XCD the ranges are as good (318 tokens, batch 4: 24.6 against 26.1 us).
  auto setup = [&](int MT, int NT) {
    p.mk = (a.S + MT - 1) / MT;
    p.nk = a.Hkv * a.D / NT;
    p.mq = (T + MT - 1) / MT;
    p.nq = a.Hq * a.D / NT;
    p.gk = a.B * p.mk;
    p.gq = a.B * p.mq;
    p.turn = a.token_keep && p.gk >= 32 ? p.gk / 8 : 0;
    const int64_t rest = (int64_t)(p.gk - 8 * p.turn) * p.nk + (int64_t)p.gq * p.nq;
    return dim3((unsigned)(8 * ((int64_t)p.turn * p.nk + (rest + 7) / 8)));
  };
  // Workgroups of a tile shape with every view kept (the host does not know the mask).
  auto items = [&](int MT, int NT) {
    return (int64_t)a.B * (((a.S + MT - 1) / MT) * (int64_t)(a.Hkv * a.D / NT) + ((T + MT - 1) / MT) * (int64_t)(a.Hq * a.D / NT));
  };
  const bool wide = (a.Hkv * a.D) % 256 == 0 && (a.Hq * a.D) % 256 == 0;
  auto launch = [&](auto kern, int MT, int NT) {
    const dim3 grid = setup(MT, NT);
    hipLaunchKernelGGL(kern, grid, dim3(kTh), 0, stream, p);
  };
#define LITEVLM_TSM(MT, NT, KT, R)                                           \
  (a.D == 128 ? launch(tsm_proj_kernel<128, MT, NT, KT, R>, MT, NT) \
              : launch(tsm_proj_kernel<64, MT, NT, KT, R>, MT, NT))
  // One 128 x 128 tile per CU or fewer: the smallest tile's K loop is the
  // shortest chain, in 32-column stages four deep (1536 visual tokens, 32/8 heads,
  // width 4096: 41 us against 54 in 128 x 256 tiles; 392 tokens, 16/8 heads,
  // width 2048: 23 against 32). Else 256-feature tiles where the heads divide so,
  // of 256 rows where these take no more rounds of the chip at twice the time each
  // (against 128 rows, views dropped: two prompts of 6144 visual tokens 102 and 112
  // us, four 207 and 179, eight 426 and 339; one, all kept, 94 and 59).
  if (items(128, 128) <= 256) LITEVLM_TSM(128, 128, 32, 4);
  else if (!wide) LITEVLM_TSM(256, 128, 64, 3);
  else if (2 * ((items(256, 256) + 255) / 256) <= (items(128, 256) + 255) / 256) LITEVLM_TSM(256, 256, 64, 2);
  else LITEVLM_TSM(128, 256, 64, 3);
#undef LITEVLM_TSM
  return hipGetLastError();
}

hipError_t launch_tsm_fold_gain(const void* w, const float* gamma, void* w_out, int rows, int cols,
                                hipStream_t stream) {
  const int64_t n = (int64_t)rows * cols;
  const int64_t blocks = (n + 255) / 256;
  const dim3 grid((unsigned)(blocks < 4096 ? blocks : 4096));
  hipLaunchKernelGGL(tsm_fold_gain_kernel, grid, dim3(256), 0, stream, static_cast<const uint16_t*>(w), gamma,
                     static_cast<uint16_t*>(w_out), (int64_t)rows, cols);
  return hipGetLastError();
}

}  // namespace litevlm
