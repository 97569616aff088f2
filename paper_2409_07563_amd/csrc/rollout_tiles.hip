// Step (a2) for the bicycle with an MLP residual (x_{t+1} = RK4 / Euler step
// + dt g([x_t; v_t])), and the checkpointing forward of the adjoint.
//
// A wave owns a tile of 16 samples.  The MLP runs on the matrix cores over
// the tile (mlp.h); every lane group g = lane / 16 carries a full copy of its
// sample's state, so the bicycle step and the cost run lane-locally, and the
// MLP input and output need only register selects and four-lane gathers.
// The nominal controls are staged in LDS.
//
// Checkpoints (optional): the state and the compensation terms of the
// positions at t = 0, c, 2c, ... are stored as ckpt[s][7][ldk], so the
// adjoint can rebuild each segment bit for bit.
#include <algorithm>
#include <type_traits>

#include "mlp.h"
#include "rollout.h"

namespace mppi {

constexpr int kTile = 16;
constexpr int kCkptWords = 7;
constexpr int kCus = 256;
// One-wave tiles share a workgroup from more than two tiles per CU on: the
// dispatcher places single waves by the SIMDs' turn, which after another launch
// puts two on one SIMD and none on the next (H = 64, T = 100, 4 tiles per CU, the
// rollout inside an iteration: 464 us; four waves of a workgroup get a SIMD each:
// 246, as alone).
constexpr int kTilesPerGroup = 4;

// BF: the MLP's products on bfloat16 operands (mlp::WeightsBf)
template <int MT, int INTEG, class Cost, bool FAST, bool BF>
__global__ __launch_bounds__(kWave * kTilesPerGroup) void rollout_tile_kernel(
    DevParams p, const float* __restrict__ x0, const float* __restrict__ u,
    const float* __restrict__ eps, int64_t ldk, int K, int T, float* __restrict__ S,
    float* __restrict__ ckpt, int ckpt_every) {
  using Model = Bicycle<FAST>;
  constexpr int N = Model::N, M = Model::M;
  extern __shared__ float4 lds[];
  const float* lds_u = stage_rollout_lds<Cost>(p, u, T * M, lds);
  const int lane = threadIdx.x % kWave, n = lane % kTile, g = lane / kTile;
  const int tile = __builtin_amdgcn_readfirstlane(
      static_cast<int>((blockIdx.x * blockDim.x + threadIdx.x) / kWave));
  if (tile * kTile >= K) return;  // the whole wave; no barrier follows
  const int k = tile * kTile + n;
  const bool live = k < K;
  const bool plain = k < p.n_plain;  // drawn around u (else around zero)
  // v = mean u + eps: an unconditional load and one FMA (mean u + eps is
  // exactly u + eps for mean = 1), no branch around the load of u
  const float mean = plain ? 1.0f : 0.0f;
  // lanes past K recompute sample K-1 (they take part in the MFMAs) and store nothing
  const float* e = eps + (live ? k : K - 1);
  std::conditional_t<BF, mlp::WeightsBf<MT ? MT : 1>, mlp::Weights<MT ? MT : 1>> W;
  if constexpr (MT > 0) {
    if constexpr (BF) W.load(p.mlp_bf, p.mlp, lane);
    else W.load(p.mlp, lane);
  }
  float x[N], comp[N];
#pragma unroll
  for (int i = 0; i < N; ++i) { x[i] = x0[i]; comp[i] = 0.0f; }
  typename Cost::State cs;
  Cost::init(cs, x, p, lds);
  float sum = 0.0f, sum_c = 0.0f;
  int next_ckpt = 0;
  float* ck = ckpt ? ckpt + k : nullptr;
  float rn[N];  // the reference of the coming step
  Cost::template fetch<N>(p, 0, rn);
  noise_steps<M, 8>(e, ldk, T, [&](int t, const float* nz, int) {
    float r[N];
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = rn[i];
    Cost::template fetch<N>(p, min(t + 1, T - 1), rn);
    float v[M];
#pragma unroll
    for (int j = 0; j < M; ++j) v[j] = mean * lds_u[t * M + j] + nz[j];
    if (ck && t == next_ckpt) {
      if (g == 0 && live) {
#pragma unroll
        for (int i = 0; i < N; ++i) ck[i * ldk] = x[i];
        ck[5 * ldk] = comp[0];
        ck[6 * ldk] = comp[1];
      }
      ck += kCkptWords * ldk;
      next_ckpt += ckpt_every;
    }
    if constexpr (MT > 0) {
      float res[N];
      mlp::residual<MT>(W, x, v, g, n, res);
      residual_step<FAST, INTEG>(x, v, comp, p, res);
    } else {
      step<Model, INTEG>(x, v, comp, p);
    }
    float l = Cost::template running_at<N, M>(x, v, r, p);
    if (p.importance && plain) l += is_term<M>(p, t, v, lds_u + t * M);
    if (p.cosines) l += inflation(p);
    const float y = l - sum_c;
    const float s = sum + y;
    sum_c = (s - sum) - y;
    sum = s;
  });
  sum = sum + (terminal_cost<Cost, N>(x, T, p, lds, cs) - sum_c);
  if (g == 0 && live) S[k] = __builtin_isfinite(sum) ? sum : __builtin_inff();
}

// The same rollout with a tile's work divided over the waves of one workgroup
// (H = 16 MT hidden units, SW = 2 or 4).  The step x' = F(x, v) + dt g(x, v)
// evaluates both terms at the state before the step, so they run side by side:
//   MLP wave w (SW of them) takes the M-tiles w MT/SW .. of both hidden layers
//   and the same K-tiles of the output layer;
//   the bicycle wave forms the RK4 (or Euler) increment;
//   the cost wave charges the step before: running cost, checkpoint, sum.
// Per step:
//   the MLP waves write their h1 tiles to LDS;                        barrier
//   the MLP waves take layer 2 over all of h1 and write their output
//   partials (BF: their h2 tiles), the bicycle wave its increment;    barrier
//   every wave adds the two and has the new state.
// A step is one dependent chain (the matrix cores' accumulations, the
// activations, two exchanges), and at K = 8192 a CU holds two tiles, so the
// length of the chain and the busiest SIMD bound the kernel: a binary32 MFMA
// keeps its SIMD's vector unit from issuing, and the bicycle's and the cost's
// arithmetic must not pile up on one SIMD.  Eight waves are launched for SW = 4
// (two per SIMD), of which two stay besides the MLP's four, on different SIMDs.
// Which two alternates between workgroups i and i + 256, the pair that a CU
// holds: where both start on the same SIMD their helpers sit on four.  The
// hardware chooses where a workgroup starts, so that is not assured.
// K = 8192, T = 100, us, against a form that repeated the bicycle step after the
// MLP and handed the state back through a third barrier: H = 64 175 -> 137 (one
// tile per CU, K = 4096: 126 -> 84), BF 111 -> 89; H = 32 140 -> 90, BF 98 -> 69.
// The matrix cores alone take 59 us at H = 64, and a binary32 MFMA and the vector
// unit of a SIMD do not overlap (measured), which leaves about 100 us as the
// floor of this arithmetic.
//
// The lanes of a wave hold the state as the next layer consumes it: lane group
// g needs x_g and (group 0) x_4, so the output layer's rows are laid out to give
// group g output g in accumulator register 0 and output 4 in register 1 (a lane
// reads another lane's row of the weight pack; the products are the same), and
// no value crosses lane groups.  In BF the input operand wants the whole state
// in lane group 0, so every MLP wave forms all outputs (over every K-block in
// order) and one v_permlane16_swap brings output 4 from group 1 to group 0.
//
// Every accumulation runs in the one-wave kernel's order and the increment and
// the step's last additions round as there (bicycle_increment, add_residual),
// so the results are bitwise the same (tested).  Each role runs its own step
// loop with the same two barriers per step; the role is a scalar, so a wave
// only ever meets its own role's barriers, T times two of them.
constexpr int split_launch_waves(int SW) { return SW == 4 ? 8 : SW + 2; }

template <int MT, int SW, int INTEG, class Cost, bool FAST, bool BF = false>
__global__ __launch_bounds__(kWave * split_launch_waves(SW)) void rollout_tile_split_kernel(
    DevParams p, const float* __restrict__ x0, const float* __restrict__ u,
    const float* __restrict__ eps, int64_t ldk, int K, int T, float* __restrict__ S,
    float* __restrict__ ckpt, int ckpt_every) {
  static_assert(MT % SW == 0 && MT % 2 == 0, "tiles per wave, whole K-blocks");
  constexpr int TW = MT / SW;  // M-tiles per wave
  constexpr int N = 5, M = 2;
  constexpr int kOut = 12;  // floats per sample of an output partial (16-byte rows, no bank conflicts)
  using f4 = mlp::f4;
  using P = mlp::Pack<MT>;
  using tile_t = std::conditional_t<BF, mlp::bf4, f4>;  // BF: rounded by the wave that formed it
  __shared__ tile_t xh[MT][kWave];           // h1 tiles
  __shared__ tile_t xg[BF ? MT : 1][kWave];  // BF: h2 tiles
  // output partials 0..4 per K-tile, read four at a time
  __shared__ alignas(sizeof(f4)) float xo[BF ? 1 : MT][kTile][kOut];
  static_assert(sizeof(float) * kOut % sizeof(f4) == 0, "a sample's row starts aligned");
  __shared__ float xq[kTile][8];             // the bicycle's increment
  extern __shared__ float4 lds[];
  const float* lds_u = stage_rollout_lds<Cost>(p, u, T * M, lds);
  const int lane = threadIdx.x % kWave;
  const int turn = static_cast<int>(blockIdx.x / kCus) & 1;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) ^ (SW == 2 ? 2 * turn : 0);
  const int n = lane % kTile, g = lane / kTile;
  const int k = blockIdx.x * kTile + n;
  const bool live = k < K;
  const bool plain = k < p.n_plain;  // drawn around u (else around zero)
  // v = mean u + eps: an unconditional load and one FMA (mean u + eps is
  // exactly u + eps for mean = 1), no branch around the load of u
  const float mean = plain ? 1.0f : 0.0f;
  const float* e = eps + (live ? k : K - 1);

  if (w >= SW) {  // a helper wave
    const int bicycle = SW == 4 ? SW + turn : SW, cost = SW == 4 ? SW + turn + 2 : SW + 1;
    if (w != bicycle && w != cost) return;
    float x[N], comp[N];
#pragma unroll
    for (int i = 0; i < N; ++i) { x[i] = x0[i]; comp[i] = 0.0f; }
    mlp::WeightsBf<MT> WB;  // BF: the output rows
    if constexpr (BF) WB.load(p.mlp_bf, p.mlp, lane);
    // the state after the step, from the MLP's outputs and the increment q
    auto finish = [&](const float* q) {
      float res[N];
      if constexpr (BF) {
        f4 o = WB.b3();
#pragma unroll
        for (int kb = 0; kb < mlp::PackBf<MT>::KB; ++kb)
          o = mlp::mfma_bf(WB.w3(kb), mlp::kblock_join(xg[2 * kb][lane], xg[2 * kb + 1][lane]), o);
        mlp::broadcast5(o, n, res);
      } else {
        f4 o = *reinterpret_cast<const f4*>(&xo[0][n][0]);
        res[4] = xo[0][n][4];
#pragma unroll
        for (int tt = 1; tt < MT; ++tt) {
          o += *reinterpret_cast<const f4*>(&xo[tt][n][0]);
          res[4] += xo[tt][n][4];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) res[i] = o[i];
      }
      add_residual<INTEG>(x, comp, q, res, p);
    };
    if (w == bicycle) {
      noise_steps<M, 8>(e, ldk, T, [&](int t, const float* nz, int) {
        float v[M], q[N];
#pragma unroll
        for (int j = 0; j < M; ++j) v[j] = mean * lds_u[t * M + j] + nz[j];
        if constexpr (INTEG == kRK4) {
          bicycle_increment_rows<FAST>(x, v, g, p, q, [] { __syncthreads(); });
        } else {
          __syncthreads();
          bicycle_increment<FAST, INTEG>(x, v, p, q);
        }
        if (g == 0) {
#pragma unroll
          for (int i = 0; i < N; ++i) xq[n][i] = q[i];
        }
        __syncthreads();
        finish(q);
      });
      return;
    }
    typename Cost::State cs;
    Cost::init(cs, x, p, lds);
    float sum = 0.0f, sum_c = 0.0f;
    int next_ckpt = 0;
    float* ck = ckpt ? ckpt + k : nullptr;
    float vp[M] = {0.0f, 0.0f};  // the control of the step before
    float rn[N];                 // the reference of the step to be charged next
    Cost::template fetch<N>(p, 0, rn);
    auto charge = [&](int t) {   // the running cost of step t at x_{t+1}
      float l = Cost::template running_at<N, M>(x, vp, rn, p);
      Cost::template fetch<N>(p, min(t + 1, T - 1), rn);
      if (p.importance && plain) l += is_term<M>(p, t, vp, lds_u + t * M);
      if (p.cosines) l += inflation(p);
      const float y = l - sum_c;
      const float s = sum + y;
      sum_c = (s - sum) - y;
      sum = s;
    };
    noise_steps<M, 8>(e, ldk, T, [&](int t, const float* nz, int) {
      if (t > 0) charge(t - 1);
      __syncthreads();
      if (ck && t == next_ckpt) {
        if (g == 0 && live) {
#pragma unroll
          for (int i = 0; i < N; ++i) ck[i * ldk] = x[i];
          ck[5 * ldk] = comp[0];
          ck[6 * ldk] = comp[1];
        }
        ck += kCkptWords * ldk;
        next_ckpt += ckpt_every;
      }
#pragma unroll
      for (int j = 0; j < M; ++j) vp[j] = mean * lds_u[t * M + j] + nz[j];
      __syncthreads();
      float q[N];
#pragma unroll
      for (int i = 0; i < N; ++i) q[i] = xq[n][i];
      finish(q);
    });
    charge(T - 1);
    sum = sum + (terminal_cost<Cost, N>(x, T, p, lds, cs) - sum_c);
    if (g == 0 && live) S[k] = __builtin_isfinite(sum) ? sum : __builtin_inff();
    return;
  }

  // an MLP wave: its operands (tiles q0 .. q0 + TW - 1)
  const int q0 = w * TW;
  const float* pk = p.mlp + lane;
  auto at = [&](int row) { return pk[row * kWave]; };
  f4 b1[TW], b2[TW];
#pragma unroll
  for (int q = 0; q < TW; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      b1[q][i] = at(P::kB1 + 4 * (q0 + q) + i);
      b2[q][i] = at(P::kB2 + 4 * (q0 + q) + i);
    }
  if constexpr (BF) {
    using PB = mlp::PackBf<MT>;
    constexpr int KB = PB::KB;
    mlp::WeightsBf<MT> W;  // the output rows; the own tiles' rows below
    W.load(p.mlp_bf, p.mlp, lane);
    mlp::bf8 v1[TW], v2[TW][KB];
#pragma unroll
    for (int q = 0; q < TW; ++q) {
      const uint4* bp = p.mlp_bf + lane;
      v1[q] = __builtin_bit_cast(mlp::bf8, bp[(PB::kW1 + q0 + q) * kWave]);
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        v2[q][kb] = __builtin_bit_cast(mlp::bf8, bp[(PB::kW2 + (q0 + q) * KB + kb) * kWave]);
    }
    // lane group 0 carries the state (the others' copies are never used)
    float x[N], comp[N];
#pragma unroll
    for (int i = 0; i < N; ++i) { x[i] = x0[i]; comp[i] = 0.0f; }
    float un[M] = {lds_u[0], lds_u[1]};  // u of the coming step, read a step ahead
    noise_steps<M, 8>(e, ldk, T, [&](int t, const float* nz, int) {
      float v[M];
#pragma unroll
      for (int j = 0; j < M; ++j) v[j] = mean * un[j] + nz[j];
      const mlp::bf8 zb = mlp::input_operand_bf(x, v, g);
#pragma unroll
      for (int q = 0; q < TW; ++q)
        xh[q0 + q][lane] = mlp::kblock_half(mlp::tanh4(mlp::mfma_bf(v1[q], zb, b1[q])));
      __syncthreads();
      mlp::bf8 hb[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        hb[kb] = mlp::kblock_join(xh[2 * kb][lane], xh[2 * kb + 1][lane]);
      const int t1 = min(t + 1, T - 1);
#pragma unroll
      for (int j = 0; j < M; ++j) un[j] = lds_u[t1 * M + j];
      f4 acc[TW];
#pragma unroll
      for (int q = 0; q < TW; ++q) {
        acc[q] = b2[q];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) acc[q] = mlp::mfma_bf(v2[q][kb], hb[kb], acc[q]);
        xg[q0 + q][lane] = mlp::kblock_half(mlp::tanh4(acc[q]));
      }
      __syncthreads();
      float qi[N], res[N];
#pragma unroll
      for (int i = 0; i < N; ++i) qi[i] = xq[n][i];
      f4 o = W.b3();
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        o = mlp::mfma_bf(W.w3(kb), mlp::kblock_join(xg[2 * kb][lane], xg[2 * kb + 1][lane]), o);
#pragma unroll
      for (int i = 0; i < 4; ++i) res[i] = o[i];
      const uint32_t o0 = __float_as_uint(o[0]);
      res[4] = __uint_as_float(__builtin_amdgcn_permlane16_swap(o0, o0, false, false)[1]);
      add_residual<INTEG>(x, comp, qi, res, p);
    });
  } else {
    float w1[TW][2], w2[TW][MT][4], w3[TW][4];
    f4 b3[TW];
    // output row m of the accumulator takes output m / 4 (m = 0 mod 4), output
    // 4 (m = 1 mod 4) or the pack's padding row
    const int m3 = (n & 3) == 0 ? n / 4 : (n & 3) == 1 ? 4 : 15;
    const float* pk3 = p.mlp + kTile * g + m3;
#pragma unroll
    for (int q = 0; q < TW; ++q) {
      const int t = q0 + q;
      w1[q][0] = at(P::kW1 + 2 * t);
      w1[q][1] = at(P::kW1 + 2 * t + 1);
#pragma unroll
      for (int tt = 0; tt < MT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) w2[q][tt][i] = at(P::kW2 + (t * MT + tt) * 4 + i);
#pragma unroll
      for (int i = 0; i < 4; ++i) w3[q][i] = pk3[(P::kW3 + 4 * t + i) * kWave];
      b3[q] = f4{0.0f, 0.0f, 0.0f, 0.0f};
      if (t == 0) {
        b3[q][0] = p.mlp[(P::kB3 + g) * kWave];       // output g
        b3[q][1] = p.mlp[P::kB3 * kWave + kTile];     // output 4
      }
    }
    // x_g (with its compensation: positions only), x_4 and the control that
    // the lane group's input slots take
    float xa = x0[g], xb = x0[4], ca = 0.0f;
    const int j = g == 2 ? 1 : 0;
    const float h = inc_scale<INTEG>(p);
    float un = lds_u[j];  // u of the coming step, read a step ahead
    noise_steps<1, 8>(e + j * ldk, M * ldk, T, [&](int t, const float* nz, int) {
      const float v = mean * un + nz[0];
      const float z1 = g == 0 ? xb : g == 3 ? 0.0f : v;
#pragma unroll
      for (int q = 0; q < TW; ++q)
        xh[q0 + q][lane] = mlp::tanh4(mlp::mfma(w1[q][1], z1, mlp::mfma(w1[q][0], xa, b1[q])));
      __syncthreads();
      // every read is requested before the first product (the compiler would
      // fetch the later tiles in the middle of the chain)
      f4 h1[MT], acc[TW];
#pragma unroll
      for (int tt = 0; tt < MT; ++tt) h1[tt] = xh[tt][lane];
      un = lds_u[min(t + 1, T - 1) * M + j];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < TW; ++q) acc[q] = b2[q];
#pragma unroll
      for (int tt = 0; tt < MT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int q = 0; q < TW; ++q) acc[q] = mlp::mfma(w2[q][tt][i], h1[tt][i], acc[q]);
#pragma unroll
      for (int q = 0; q < TW; ++q) {
        const f4 h2 = mlp::tanh4(acc[q]);
        __builtin_amdgcn_sched_barrier(0);  // the four activations side by side, then the products
        f4 part = b3[q];
#pragma unroll
        for (int i = 0; i < 4; ++i) part = mlp::mfma(w3[q][i], h2[i], part);
        xo[q0 + q][n][g] = part[0];
        if (g == 0) xo[q0 + q][n][4] = part[1];
      }
      __syncthreads();
      float ra = xo[0][n][g], rb = xo[0][n][4];
#pragma unroll
      for (int tt = 1; tt < MT; ++tt) {
        ra += xo[tt][n][g];
        rb += xo[tt][n][4];
      }
      const float qa = xq[n][g], qb = xq[n][4];
      {
#pragma clang fp contract(off)
        // add_residual for components g and 4
        const float ia = g < 3 ? __builtin_fmaf(p.dt, ra, qa) : __builtin_fmaf(h, qa, p.dt * ra);
        const float y = ia - ca;
        const float s = xa + y;
        ca = g < 2 ? (s - xa) - y : 0.0f;
        xa = s;
        xb = xb + __builtin_fmaf(h, qb, p.dt * rb);
      }
    });
  }
}

namespace {

using TileFn = void (*)(DevParams, const float*, const float*, const float*, int64_t, int, int,
                        float*, float*, int);

template <int MT, int INTEG, bool FAST, bool BF>
TileFn pick_cost(uint32_t cost) {
  if (cost == MPPI_COST_TRACK) return rollout_tile_kernel<MT, INTEG, CostTrack, FAST, BF>;
  if (cost == MPPI_COST_QUADRATIC) return rollout_tile_kernel<MT, INTEG, CostQuadratic, FAST, BF>;
  return nullptr;
}

template <int MT, bool BF = false>
TileFn pick_tile(uint32_t integrator, uint32_t cost, bool accurate) {
  if (integrator == MPPI_INT_RK4)
    return accurate ? pick_cost<MT, kRK4, false, BF>(cost) : pick_cost<MT, kRK4, true, BF>(cost);
  if (integrator == MPPI_INT_EULER)
    return accurate ? pick_cost<MT, kEuler, false, BF>(cost)
                    : pick_cost<MT, kEuler, true, BF>(cost);
  return nullptr;
}

template <int MT, int SW, int INTEG, bool FAST, bool BF>
TileFn pick_split_cost(uint32_t cost) {
  if (cost == MPPI_COST_TRACK) return rollout_tile_split_kernel<MT, SW, INTEG, CostTrack, FAST, BF>;
  if (cost == MPPI_COST_QUADRATIC)
    return rollout_tile_split_kernel<MT, SW, INTEG, CostQuadratic, FAST, BF>;
  return nullptr;
}

template <int MT, int SW, bool BF>
TileFn pick_split_bf(uint32_t integrator, uint32_t cost, bool accurate) {
  if (integrator == MPPI_INT_RK4)
    return accurate ? pick_split_cost<MT, SW, kRK4, false, BF>(cost)
                    : pick_split_cost<MT, SW, kRK4, true, BF>(cost);
  if (integrator == MPPI_INT_EULER)
    return accurate ? pick_split_cost<MT, SW, kEuler, false, BF>(cost)
                    : pick_split_cost<MT, SW, kEuler, true, BF>(cost);
  return nullptr;
}

template <int MT, int SW>
TileFn pick_split(uint32_t integrator, uint32_t cost, bool accurate, bool bf) {
  return bf ? pick_split_bf<MT, SW, true>(integrator, cost, accurate)
            : pick_split_bf<MT, SW, false>(integrator, cost, accurate);
}

TileFn select_tile(uint32_t dynamics, uint32_t integrator, uint32_t cost, bool accurate,
                   int hidden, bool bf = false) {
  if (dynamics == MPPI_DYN_BICYCLE) return pick_tile<0>(integrator, cost, accurate);
  if (dynamics != MPPI_DYN_BICYCLE_MLP) return nullptr;
  switch (hidden) {
    case 16: return bf ? pick_tile<1, true>(integrator, cost, accurate)
                       : pick_tile<1>(integrator, cost, accurate);
    case 32: return bf ? pick_tile<2, true>(integrator, cost, accurate)
                       : pick_tile<2>(integrator, cost, accurate);
    case 64: return bf ? pick_tile<4, true>(integrator, cost, accurate)
                       : pick_tile<4>(integrator, cost, accurate);
    default: return nullptr;
  }
}

}  // namespace

bool rollout_tiles_supported(uint32_t dynamics, uint32_t integrator, uint32_t cost, int hidden) {
  return select_tile(dynamics, integrator, cost, false, hidden) != nullptr;
}

namespace {

// How many of the first tiles run one wave each; the split form takes the rest
// (the costs are the same bit for bit).  A split tile's time adds up over the
// tiles of a CU, while four one-wave tiles run side by side on its SIMDs: with H = 64
// a round of four per CU is the faster so, and what is left over is split while that
// is short.  With H = 32 two or three one-wave tiles share a SIMD at little cost,
// so all tiles or none.  An iteration, T = 100, us, split | one wave:
//   H = 64, 1 to 4 tiles per CU (K 4096 each): 90 145 215 294 | 250 256 260 263;
//     5, 6, 8: 388 437 578 | 469 470 475, a round and the rest split 354 403 470
//   H = 64, bfloat16: 66 100 143 203 | 126 132 137 137; 5, 6, 8: 252 283 362 |
//     234 235 238, a round and the rest split 208 236 237 (T = 30, 6: 83 and 87)
//   H = 32, 1 to 12: 69 100 132 144 194 229 260 292 323 351 378 409 |
//     135 139 144 144 231 231 233 235 330 332 335 336
//   H = 32, bfloat16: 61 78 97 107 146 167 188 208 230 250 271 291 |
//     90 95 99 100 154 154 156 157 215 217 220 221
int one_wave_tiles(int hidden, int waves, bool bf, int tiles) {
  if (waves == 1) return tiles;
  if (hidden == 64 && waves == 4) {
    constexpr int kRound = 4 * kCus;
    const int rest = tiles % kRound;
    const int limit = !bf ? 3 : tiles < kRound ? 2 : 1;  // tiles per CU
    return rest > limit * kCus ? tiles : tiles - rest;
  }
  if (hidden == 32) {
    const int per_cu = (tiles + kCus - 1) / kCus;
    const bool one_over = per_cu % 4 == 1 && per_cu < (bf ? 8 : 12);
    return per_cu >= 4 && !one_over ? tiles : 0;
  }
  return 0;
}

}  // namespace

hipError_t launch_rollout_tiles(uint32_t dynamics, uint32_t integrator, uint32_t cost,
                                bool accurate_trig, const DevParams& p, const float* d_x0,
                                const float* d_u, const float* d_eps, int64_t ldk, int K, int T,
                                float* d_S, float* d_ckpt, int ckpt_every, hipStream_t stream,
                                int waves) {
  // the split forms: H = 32 over 2 waves; H = 64 over 2 or 4 waves
  const bool mlp = dynamics == MPPI_DYN_BICYCLE_MLP;
  const bool bf = mlp && p.mlp_bf != nullptr;  // BF16 products
  const TileFn one = select_tile(dynamics, integrator, cost, accurate_trig, p.mlp_hidden, bf);
  TileFn split = nullptr;
  if (mlp && p.mlp_hidden == 64 && waves == 4) split = pick_split<4, 4>(integrator, cost, accurate_trig, bf);
  else if (mlp && p.mlp_hidden == 64 && waves == 2) split = pick_split<4, 2>(integrator, cost, accurate_trig, bf);
  else if (mlp && p.mlp_hidden == 32 && waves == 2) split = pick_split<2, 2>(integrator, cost, accurate_trig, bf);
  if (!one || (waves != 1 && !split) || (d_ckpt && ckpt_every < 1)) return hipErrorInvalidValue;
  const size_t lds = sizeof(float) * static_cast<size_t>(T) * 2;
  // the tiles first .. first + count - 1 in workgroups of `threads` threads for
  // `per` tiles each
  auto launch = [&](TileFn fn, int first, int count, int per, int threads) -> hipError_t {
    if (count < 1) return hipSuccess;
    if (lds > 48 * 1024) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                         static_cast<int>(lds));
      if (e != hipSuccess) return e;
    }
    const int k0 = first * kTile;
    DevParams q = p;
    q.n_plain = p.n_plain - k0;
    hipLaunchKernelGGL(fn, dim3(static_cast<unsigned>((count + per - 1) / per)), dim3(threads), lds,
                       stream, q, d_x0, d_u, d_eps + k0, ldk, std::min(K - k0, count * kTile), T,
                       d_S + k0, d_ckpt ? d_ckpt + k0 : nullptr, ckpt_every);
    return hipGetLastError();
  };
  const int tiles = (K + kTile - 1) / kTile;
  const int n1 = one_wave_tiles(p.mlp_hidden, waves, bf, tiles);
  const int per = n1 > 2 * kCus ? kTilesPerGroup : 1;
  const hipError_t e = launch(one, 0, n1, per, kWave * per);
  // the split forms' helper waves come on top of the MLP's
  return e == hipSuccess ? launch(split, n1, tiles - n1, 1, kWave * split_launch_waves(waves)) : e;
}

}  // namespace mppi
