// fp32-storage matrix-core kernels of the SwitchHead layer (arXiv 2312.07987): the projections of Sec. 2.1 - 2.2, their
// data and weight gradients, and the attention of Sec. 2.1 with its backward pass.  fp32 operands, fp32 accumulation:
// v_mfma_f32_16x16x4_f32 is an fp32 fused multiply-add chain, so nothing is rounded that the plain kernels (simt.hip)
// would keep.
//
// Layouts of v_mfma_f32_16x16x4_f32 (lane = 16*g + r, g in 0..3):
//   A operand: A[row r][k = g]     B operand: B[k = g][col r]     D register v: D[row 4g + v][col r]
// The reduction index is taken in the order k = 16 c + 4 g + t (t = the instruction, 0..3): a lane's operands of four
// consecutive instructions are then 16 contiguous bytes of a row stored k-contiguous.
//
// The matrix pipe does 256 fp32 flop per clock and CU (157 TFLOP/s), a sixteenth of its bf16 rate, so a 64-row tile with
// one 16-row strip per wave needs only a third of the LDS bandwidth; what these shapes need instead is many resident
// work-groups (four per CU and more) to hide the load latency behind, hence the small tiles.
// Measured for a training step of the 47M-parameter layer (d_model 412, 2 heads of 76, 5 experts, 3 active) over 16 x 256 tokens:
// 2263 us on the vector kernels of simt.hip, 398 us here; value experts 110 -> 27 us (63 TFLOP/s: 390 tiles for 256 CUs, a second
// tile on half of them), output experts with their zero fill 188 -> 45, weight gradients 550 -> 89, attention forward 188 -> 17
// and backward 391 -> 37.  A toy layer (128 tokens, d_model 64) is launches and latency: 415 -> 70 us.
#include "common.h"
#include "mfma_util.h"

namespace sh {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma_16x16x4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// VEC consecutive floats, zeros where not `ok`
template <int VEC>
struct FVec;
template <>
struct FVec<4> {
  typedef f32x4 type;
};
template <>
struct FVec<1> {
  typedef float type;
};

// ----------------------------------------------------------------------------------------
// Row GEMM: 64 x (16 NJ) tile, wave w owns rows 16 w .. 16 w + 15, K step 32.  Two LDS stages (one barrier per step) and two
// register sets: a step's loads have two steps to arrive.  The loads carry no conditions (a test around a load makes the
// compiler wait for all of them at the join): a row past the end repeats the tile's first row, a column or reduction index
// past the end repeats index 0, and what must not count is replaced by zero on its way into LDS.
// VEC: floats per global load (1 where a row is no multiple of 16 bytes).
// ----------------------------------------------------------------------------------------
static constexpr int FBM = 64, FBK = 32, FLDA = FBK + 4;   // row stride 36 words: the 16 rows of a 16-byte read hit 64 banks

// SEG: one output element from the segments whose gate is not zero, up to the first NaN
template <bool BNT>
__device__ __forceinline__ float f32_selected_sum(const RowGemmArgs& a, const float* gates, int row, int n) {
  float s = 0.f;
  for (int q = 0; q < a.nseg && s == s; ++q) {
    const SegDesc& d = a.segd[q];
    const float gt = d.gcol >= 0 ? gates[d.gcol] : 1.f;
    if (gt == 0.f) continue;
    const int K = d.klen ? d.klen : a.K;
    const float* Ap = (const float*)d.A + (long)row * (d.klen ? d.lda : a.lda);
    const float* Bp = (const float*)d.B + (BNT ? (long)n * (d.klen ? d.sbn : a.sbn) : (long)n);
    for (int k = 0; k < K; ++k) s = fmaf(Ap[k] * gt, Bp[BNT ? (long)k : (long)k * a.sbk], s);
  }
  return s;
}

template <int NJ, int VEC, bool BNT, bool SEG>
__global__ __launch_bounds__(256) void f32_row_gemm_kernel(RowGemmArgs a) {
  constexpr int BN = 16 * NJ;
  constexpr int LDB = BNT ? FLDA : BN + 4;   // n-contiguous: rows 4 g + t of a read lie 16 banks apart
  typedef typename FVec<VEC>::type vec_t;
  __shared__ __attribute__((aligned(16))) float As_[2][FBM * FLDA];
  __shared__ __attribute__((aligned(16))) float Bs_[2][BNT ? BN * FLDA : FBK * (BN + 4)];
  __shared__ int ids[FBM];
  __shared__ float gsc[FBM];
  __shared__ float gts[SEG ? FBM * F32_MAX_SEGD : 1];   // the tile's dense gates, [row][head * experts + expert]
  __shared__ int again;                                 // SEG: an element of the tile is NaN

  const int h = blockIdx.z, n0 = blockIdx.y * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  int e = 0, row0, rows;
  if (a.perm) {
    if (!find_tile_wave(a.offsets + (long)h * (a.E + 1), a.E, FBM, blockIdx.x, lane, e, row0, rows)) return;
  } else {
    row0 = blockIdx.x * FBM;
    rows = a.M - row0 < FBM ? a.M - row0 : FBM;
  }
  const bool second = a.hsplit > 0 && h >= a.hsplit;
  const int hh = second ? h - a.hsplit : h;
  if (tid < FBM) {
    const int t = min(tid, rows - 1);
    const int id = a.perm ? a.perm[(long)h * a.M + row0 + t] : row0 + t;
    ids[tid] = id;
    gsc[tid] = a.gate ? a.gate[(long)h * a.gate_hstride + id] : 1.f;
  }
  if constexpr (SEG) {
    if (tid == 0) again = 0;
    if (a.gidx) {
      const int HE = a.gheads * a.experts;
      for (int t = tid; t < FBM * HE; t += 256) gts[(t / HE) * F32_MAX_SEGD + t % HE] = 0.f;
      __syncthreads();
      for (int t = tid; t < rows * a.gheads * a.gk; t += 256) {
        const int j = t % a.gk, row = t / a.gk % rows, hd = t / (a.gk * rows);
        const long o = ((long)hd * a.M + row0 + row) * a.gk + j;
        gts[row * F32_MAX_SEGD + hd * a.experts + a.gidx[o]] = a.ggate[o];
      }
    }
  }
  __syncthreads();

  const float* A = (const float*)a.A + (long)hh * a.a_hoff;
  const float* B = (const float*)(second ? a.B2 : a.B) + (long)hh * a.b_hstride + (long)e * a.b_estride;
  const int Nc = a.Nc;

  constexpr int A_CPR = FBK / VEC, A_N = FBM * A_CPR / 256;
  constexpr int B_CPR = BNT ? A_CPR : BN / VEC, B_TOT = FBK * BN / VEC, B_N = (B_TOT + 255) / 256;
  int a_row[A_N];   // operand row of each of the thread's pieces
#pragma unroll
  for (int i = 0; i < A_N; ++i) a_row[i] = ids[(tid + i * 256) / A_CPR] / a.a_div;
  struct Step {
    vec_t ra[A_N], rb[B_N];
    int gcol, K, k0;   // the step's segment: gate column, length; its first reduction index
  };
  int seg = 0, k0 = 0;   // the step that is requested next
  const int nseg = SEG ? a.nseg : 1;
  int steps = 0;
  if constexpr (SEG) {
    for (int t = 0; t < nseg; ++t) steps += ((a.segd[t].klen ? a.segd[t].klen : a.K) + FBK - 1) / FBK;
  } else {
    steps = (a.K + FBK - 1) / FBK;
  }
  auto load = [&](Step& st) {
    const float *Ap = A, *Bp = B;
    int lda = (int)a.lda, sbn = a.sbn, K = a.K;
    st.gcol = -1;
    bool odd = false;   // a segment of its own stride (a router's matrix): rows of any length and alignment
    if constexpr (SEG) {
      const SegDesc& d = a.segd[min(seg, nseg - 1)];   // (requests past the last step repeat the last segment)
      Ap = (const float*)d.A;
      Bp = (const float*)d.B;
      st.gcol = d.gcol;
      if (d.klen) {
        K = d.klen, lda = d.lda, sbn = d.sbn;
        odd = VEC == 4 && BNT;
      }
    }
    st.K = K;
    st.k0 = k0;
#pragma unroll
    for (int i = 0; i < A_N; ++i) {
      const int kk = k0 + ((tid + i * 256) % A_CPR) * VEC;
      st.ra[i] = *(const vec_t*)(Ap + (long)a_row[i] * lda + (kk < K ? kk : 0));
    }
    if constexpr (SEG && BNT && VEC == 4) {
      if (odd) {   // uniform
#pragma unroll
        for (int i = 0; i < B_N; ++i) {
          const int c = tid + i * 256, n = n0 + c / B_CPR, kk = k0 + (c % B_CPR) * 4;
#pragma unroll
          for (int t = 0; t < 4; ++t) st.rb[i][t] = Bp[(long)(n < Nc ? n : 0) * sbn + (kk + t < K ? kk + t : 0)];
        }
      }
    }
    if (!odd) {
#pragma unroll
      for (int i = 0; i < B_N; ++i) {
        const int c = tid + i * 256;
        if constexpr (BNT) {
          const int n = n0 + c / B_CPR, kk = k0 + (c % B_CPR) * VEC;
          st.rb[i] = *(const vec_t*)(Bp + (long)(n < Nc ? n : 0) * sbn + (kk < K ? kk : 0));
        } else {
          const int kk = k0 + c / B_CPR, n = n0 + (c % B_CPR) * VEC;
          st.rb[i] = *(const vec_t*)(Bp + (long)(kk < K ? kk : 0) * a.sbk + (n < Nc ? n : 0));
        }
      }
    }
    k0 += FBK;
    if (k0 >= K) {
      k0 = 0;
      ++seg;
    }
  };
  auto store = [&](const Step& st, int stage) {
#pragma unroll
    for (int i = 0; i < A_N; ++i) {
      const int c = tid + i * 256, kk = st.k0 + (c % A_CPR) * VEC;
      vec_t v = st.ra[i];
      if constexpr (SEG) {
        if (st.gcol >= 0) v *= gts[c / A_CPR * F32_MAX_SEGD + st.gcol];
      }
      if constexpr (VEC == 4) {
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = kk + t < st.K ? v[t] : 0.f;
      } else {
        v = kk < st.K ? v : 0.f;
      }
      *(vec_t*)&As_[stage][(c / A_CPR) * FLDA + (c % A_CPR) * VEC] = v;
    }
#pragma unroll
    for (int i = 0; i < B_N; ++i) {
      const int c = tid + i * 256;
      if (B_TOT % 256 == 0 || c < B_TOT) *(vec_t*)&Bs_[stage][(c / B_CPR) * LDB + (c % B_CPR) * VEC] = st.rb[i];
    }
    // What B holds past the end of the reduction is a repeat; it becomes zero as well (an infinity times the zero of A is NaN).  A
    // thread's own pieces, after they are stored: selecting on the way, as A does, costs every step.  (SEG computes NaNs again.)
    if (!SEG && st.k0 + FBK > st.K) {   // uniform
#pragma unroll
      for (int i = 0; i < B_N; ++i) {
        const int c = tid + i * 256;
        if (B_TOT % 256 != 0 && c >= B_TOT) continue;
#pragma unroll
        for (int t = 0; t < VEC; ++t)
          if (st.k0 + (BNT ? (c % B_CPR) * VEC + t : c / B_CPR) >= st.K) Bs_[stage][(c / B_CPR) * LDB + (c % B_CPR) * VEC + t] = 0.f;
      }
    }
  };

  f32x4 acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = f32x4{};
  auto compute = [&](int stage, int len) {
    const float *As = As_[stage], *Bs = Bs_[stage];
#pragma unroll
    for (int c = 0; c < FBK; c += 16) {
      if (c && c >= len) break;   // uniform: the second half of a segment's last step may hold nothing
      const f32x4 fa = *(const f32x4*)&As[(wave * 16 + r) * FLDA + c + 4 * g];
      f32x4 fb[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if constexpr (BNT)
          fb[j] = *(const f32x4*)&Bs[(j * 16 + r) * LDB + c + 4 * g];
        else
#pragma unroll
          for (int t = 0; t < 4; ++t) fb[j][t] = Bs[(c + 4 * g + t) * LDB + j * 16 + r];
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[j] = mfma_16x16x4(fa[t], fb[j][t], acc[j]);
    }
  };
  Step s0, s1;
  load(s0);
  load(s1);
  for (int it = 0; it < steps; it += 2) {
    store(s0, 0);
    const int l0 = s0.K - s0.k0;
    __syncthreads();
    load(s0);
    compute(0, l0);
    if (it + 1 == steps) break;
    store(s1, 1);
    const int l1 = s1.K - s1.k0;
    __syncthreads();
    load(s1);
    compute(1, l1);
  }

  float* C = (float*)(second ? a.C2 : a.C) + (long)hh * a.c_hoff;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = wave * 16 + 4 * g + v;
    if (row >= rows) continue;
    const float sc = gsc[row];
    float* crow = C + (long)(ids[row] / a.c_div) * a.ldc;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = n0 + j * 16 + r;
      if (n >= Nc) continue;
      if (a.mode == ATOMIC_F32)
        atomicAdd(crow + n, acc[j][v] * sc);
      else
        crow[n] = acc[j][v] * sc;
    }
  }
  if constexpr (SEG) {
    // An expert that a token did not select is multiplied by zero, which must not let its infinities and NaNs through: elements that
    // came out as NaN are computed once more from the selected experts alone, up to the first NaN that is really theirs.
    bool nan = false;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int j = 0; j < NJ; ++j) nan |= acc[j][v] != acc[j][v];
    if (__ballot(nan) && lane == 0) again = 1;
    __syncthreads();
    if (!again) return;
    for (int t = tid; t < rows * BN; t += 256) {
      const int row = t / BN, n = n0 + t % BN;
      if (n >= Nc) continue;
      float* o = C + (long)(row0 + row) * a.ldc + n;
      if (*o == *o) continue;
      *o = f32_selected_sum<BNT>(a, gts + row * F32_MAX_SEGD, row0 + row, n);
    }
  }
}

// ----------------------------------------------------------------------------------------
// The same products for launches of few tiles: 16 x 32 tiles, the reduction split over eight waves.  A 64 x 64 tile keeps one CU's matrix
// pipe for 1024 cycles per 32 reduction indices, so a launch of a few of them takes its whole reduction times that while most
// of the chip is idle.  Here a wave takes every eighth piece of 16 indices, its operands come straight from memory in fragment order, four
// pieces a trip, and the partial sums meet in LDS and are added in wave order.
// The line, launches of 128 tiles of 64 rows: a training step with the small tiles up to 0 / 32 / 128 / 256 of them, us: toy layer (d_model 64, 2
// heads of 32) over 128 tokens 91 / 71 / 70 / 70; 47M layer over 128 tokens 212 / 121 / 121 / 121, 512 tokens 235 / 224 / 160 / 159, 2048 tokens
// 268 / 268 / 264 / 296; 262M layer over 128 tokens 468 / 303 / 272 / 272, 512 tokens 549 / 549 / 483 / 498.
// A second line, small_tiles_pay(), where the small tiles are many and their reduction is short, or their scalar loads run along the columns of B.
static constexpr int F32_SMALL_TILES = 128;
static constexpr int FSM_M = 16, FSM_N = 32, FSM_W = 8, FSM_U = 4;

template <int VEC, bool BNT, bool SEG>
__global__ __launch_bounds__(64 * FSM_W) void f32_small_gemm_kernel(RowGemmArgs a) {
  __shared__ float part[FSM_W][FSM_M][FSM_N + 1];
  __shared__ int ids[FSM_M];
  __shared__ float gsc[FSM_M];
  __shared__ float gts[SEG ? FSM_M * F32_MAX_SEGD : 1];   // the tile's dense gates, [row][head * experts + expert]
  __shared__ SegDesc descs[SEG ? F32_MAX_SEGD : 1];
  const int h = blockIdx.z, n0 = blockIdx.y * FSM_N;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  int e = 0, row0, rows;
  if (a.perm) {
    if (!find_tile_wave(a.offsets + (long)h * (a.E + 1), a.E, FSM_M, blockIdx.x, lane, e, row0, rows)) return;
  } else {
    row0 = blockIdx.x * FSM_M;
    rows = a.M - row0 < FSM_M ? a.M - row0 : FSM_M;
  }
  const bool second = a.hsplit > 0 && h >= a.hsplit;
  const int hh = second ? h - a.hsplit : h;
  // (a row past the end repeats the last one; nothing of it is stored)
  const int id = a.perm ? a.perm[(long)h * a.M + row0 + min(r, rows - 1)] : row0 + min(r, rows - 1);
  if (tid < FSM_M) {
    ids[tid] = id;
    gsc[tid] = a.gate ? a.gate[(long)h * a.gate_hstride + id] : 1.f;
  }
  if constexpr (SEG) {
    if (tid < a.nseg) descs[tid] = a.segd[tid];
    if (a.gidx) {
      for (int t = tid; t < FSM_M * F32_MAX_SEGD; t += 64 * FSM_W) gts[t] = 0.f;
      __syncthreads();
      for (int t = tid; t < FSM_M * a.gheads * a.gk; t += 64 * FSM_W) {
        const int row = t % FSM_M, hd = t / FSM_M / a.gk, j = t / FSM_M % a.gk;
        if (row < rows) {
          const long o = ((long)hd * a.M + row0 + row) * a.gk + j;
          gts[row * F32_MAX_SEGD + hd * a.experts + a.gidx[o]] = a.ggate[o];
        }
      }
    }
  }
  __syncthreads();

  const float* A = (const float*)a.A + (long)hh * a.a_hoff;
  const float* B = (const float*)(second ? a.B2 : a.B) + (long)hh * a.b_hstride + (long)e * a.b_estride;
  const int nseg = SEG ? a.nseg : 1, regular = SEG ? nseg - a.seg_own : 1, Nc = a.Nc;
  const int cps = (a.K + 15) / 16, cps_own = SEG ? (descs[nseg - 1].klen + 15) / 16 : 0;   // pieces of a segment
  const unsigned inv = div_magic(cps);
  const int pieces = regular * cps + (nseg - regular) * cps_own;
  const long arow = id / a.a_div;
  f32x4 acc[2] = {f32x4{}, f32x4{}};
  for (int c0 = wave; c0 < pieces; c0 += FSM_W * FSM_U) {
    f32x4 fa[FSM_U], fb[FSM_U][2];
#pragma unroll
    for (int u = 0; u < FSM_U; ++u) {
      const int c = min(c0 + u * FSM_W, pieces - 1);   // (a piece past the last: loaded, not used)
      const float *Ap = A, *Bp = B;
      int lda = (int)a.lda, sbn = a.sbn, K = a.K, k0 = c * 16, gcol = -1;
      bool own = false;
      if constexpr (SEG) {
        const int c1 = c - regular * cps;
        const int seg = c1 < 0 ? div_by(c, inv) : regular + (cps_own > 1 ? c1 / cps_own : c1);
        k0 = (c1 < 0 ? c - seg * cps : c1 - (seg - regular) * cps_own) * 16;
        const SegDesc d = descs[seg];
        Ap = (const float*)d.A;
        Bp = (const float*)d.B;
        gcol = d.gcol;
        if (d.klen) K = d.klen, lda = d.lda, sbn = d.sbn, own = true;
      }
      const int kk = k0 + 4 * g;
      auto quad = [&](const float* row, bool vec) {   // row[kk .. kk + 3], zeros from K on
        f32x4 v;
        if (VEC == 4 && vec) {
          v = *(const f32x4*)(row + (kk < K ? kk : 0));
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = row[kk + t < K ? kk + t : 0];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = kk + t < K ? v[t] : 0.f;
        return v;
      };
      fa[u] = quad(Ap + arow * lda, true);
      if (SEG && gcol >= 0) fa[u] *= gts[r * F32_MAX_SEGD + gcol];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int n = n0 + 16 * j + r, nn = n < Nc ? n : 0;   // (a column past the last repeats the first; not stored)
        if constexpr (BNT) {
          fb[u][j] = quad(Bp + (long)nn * sbn, !own);
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float v = Bp[(long)(kk + t < K ? kk + t : 0) * a.sbk + nn];
            fb[u][j][t] = kk + t < K ? v : 0.f;
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < FSM_U; ++u)
      if (c0 + u * FSM_W < pieces) {   // uniform in the wave
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[j] = mfma_16x16x4(fa[u][t], fb[u][j][t], acc[j]);
      }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wave][4 * g + v][16 * j + r] = acc[j][v];
  __syncthreads();
  const int row = tid / FSM_N, n = n0 + tid % FSM_N;   // an output element per thread
  if (row >= rows || n >= Nc) return;
  float s = part[0][row][tid % FSM_N];
#pragma unroll
  for (int w = 1; w < FSM_W; ++w) s += part[w][row][tid % FSM_N];
  if constexpr (SEG) {
    // (zero times an infinity or NaN of an expert that the token did not select: once more from the selected experts alone, as above)
    if (s != s) s = f32_selected_sum<BNT>(a, gts + row * F32_MAX_SEGD, row0 + row, n);
  }
  s *= gsc[row];
  float* C = (float*)(second ? a.C2 : a.C) + (long)hh * a.c_hoff + (long)(ids[row] / a.c_div) * a.ldc + n;
  if (a.mode == ATOMIC_F32)
    atomicAdd(C, s);
  else
    *C = s;
}

// 16-byte loads of both operands are possible
static bool f32_vec4(const RowGemmArgs& a) {
  auto al = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  bool ok = a.lda % 4 == 0 && a.a_hoff % 4 == 0 && a.K % 4 == 0 && a.b_hstride % 4 == 0 && a.b_estride % 4 == 0;
  ok = ok && (a.sbk == 1 ? a.sbn % 4 == 0 : (a.sbk % 4 == 0 && a.Nc % 4 == 0));
  if (a.seg_mode == 3) {
    for (int s = 0; s < a.nseg; ++s)
      ok = ok && al(a.segd[s].A) && (a.segd[s].klen ? a.segd[s].lda % 4 == 0 : al(a.segd[s].B));
  } else {
    ok = ok && al(a.A) && al(a.B) && (a.hsplit == 0 || al(a.B2));
  }
  return ok;
}

bool f32_row_gemm_supported(const RowGemmArgs& a) {
  if (a.sbk != 1 && a.sbn != 1) return false;
  if (a.seg_mode != 0 && a.seg_mode != 3) return false;
  if (a.seg_mode == 3 && (a.nseg < 1 || a.nseg > F32_MAX_SEGD || a.heads != 1 || a.perm || a.a_div != 1)) return false;
  if (a.seg_mode == 3 && a.gidx && a.gheads * a.experts > F32_MAX_SEGD) return false;
  return a.E <= 128;   // the tile lookup covers 128 groups
}

template <int NJ, int VEC>
static void launch_f32_rg(const RowGemmArgs& a, hipStream_t s) {
  dim3 g((a.M + FBM - 1) / FBM + (a.perm ? a.E : 0), (a.Nc + 16 * NJ - 1) / (16 * NJ), a.heads);
  if (a.seg_mode == 3) {
    if (a.sbk == 1)
      f32_row_gemm_kernel<NJ, VEC, true, true><<<g, 256, 0, s>>>(a);
    else
      f32_row_gemm_kernel<NJ, VEC, false, true><<<g, 256, 0, s>>>(a);
  } else if (a.sbk == 1) {
    f32_row_gemm_kernel<NJ, VEC, true, false><<<g, 256, 0, s>>>(a);
  } else {
    f32_row_gemm_kernel<NJ, VEC, false, false><<<g, 256, 0, s>>>(a);
  }
}

// columns per tile: the width that pads the output least (a head of 76 takes one tile of 80, of 128 two of 64)
static int f32_nj(int cols) {
  if (cols <= 32) return 2;
  const int w4 = (cols + 63) / 64 * 64, w5 = (cols + 79) / 80 * 80;
  return w5 < w4 ? 5 : 4;
}

template <int VEC>
static void launch_f32_small(const RowGemmArgs& a, hipStream_t s) {
  const dim3 g((a.M + FSM_M - 1) / FSM_M + (a.perm ? a.E : 0), (a.Nc + FSM_N - 1) / FSM_N, a.heads);
  if (a.seg_mode == 3)
    a.sbk == 1 ? f32_small_gemm_kernel<VEC, true, true><<<g, 64 * FSM_W, 0, s>>>(a) : f32_small_gemm_kernel<VEC, false, true><<<g, 64 * FSM_W, 0, s>>>(a);
  else
    a.sbk == 1 ? f32_small_gemm_kernel<VEC, true, false><<<g, 64 * FSM_W, 0, s>>>(a) : f32_small_gemm_kernel<VEC, false, false><<<g, 64 * FSM_W, 0, s>>>(a);
}

// A work-group costs as much as 190 of its reduction indices before it begins, and a launch of large tiles little more than its
// reduction.  One launch, us, large tiles / small ones, work-groups of the latter and K: 1500 sorted rows of 4 heads of 48 7.4 / 12.2 (772, K 128),
// 1874 of 3 heads of 42 8.8 / 15.1 (717, 128), but 1107 rows of 4 heads of 76 18.7 / 11.3 (840, 412).  Rows of B along the
// reduction that cannot be read 16 bytes at a time are 32 scattered lines an instruction: 2018 sorted rows of 3 heads of 36 32.7 / 51.5 (777, 1030), 155 of
// 10 heads of 128 33.7 / 52.0 (500, 1030).  Of 3964 launches up to the first line 172 that come here are slower by more than 3 per cent, 322 us in all, and
// the others 60000 us faster; by the first line alone 245 were slower, 670 us.
static bool small_tiles_pay(const RowGemmArgs& a, bool v4) {
  const long wgs = (long)((a.M + FSM_M - 1) / FSM_M + (a.perm ? a.E / 2 : 0)) * ((a.Nc + FSM_N - 1) / FSM_N) * a.heads;
  const long K = a.seg_mode == 3 ? (long)(a.nseg - a.seg_own) * a.K + (a.seg_own ? (long)a.seg_own * a.segd[a.nseg - 1].klen : 0) : a.K;
  return !v4 && a.sbk == 1 ? wgs * (190 + K) <= 520 * (30 + K) : wgs * (190 + K) <= 1400 * (40 + K);
}

void launch_f32_row_gemm(const RowGemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.Nc <= 0) return;
  const bool v4 = f32_vec4(a);
  const int nj = f32_nj(a.Nc);
  const long tiles = (long)((a.M + FBM - 1) / FBM + (a.perm ? a.E / 2 : 0)) * ((a.Nc + 16 * nj - 1) / (16 * nj)) * a.heads;
  if (tiles <= F32_SMALL_TILES && small_tiles_pay(a, v4)) return v4 ? launch_f32_small<4>(a, s) : launch_f32_small<1>(a, s);
  switch (f32_nj(a.Nc) * 2 + (v4 ? 1 : 0)) {
    case 5: return launch_f32_rg<2, 4>(a, s);
    case 4: return launch_f32_rg<2, 1>(a, s);
    case 9: return launch_f32_rg<4, 4>(a, s);
    case 8: return launch_f32_rg<4, 1>(a, s);
    case 11: return launch_f32_rg<5, 4>(a, s);
    default: return launch_f32_rg<5, 1>(a, s);
  }
}

// ----------------------------------------------------------------------------------------
// Weight gradients dW[i][j] = sum_rows gate * A[row][i] * Bm[row][j], up to F32_WG_MAX of them in one launch (all of a
// backward pass's are independent of each other once the attention backward is done, and one launch of many small
// work-groups fills the chip where each alone would not).  64 x (16 NJ) output tile, 32 rows per step; both operand tiles
// lie [row][feature] in LDS as they do in memory.  A problem whose groups all fit into one chunk is stored; of the others every
// chunk stores its partial sum and f32_wgrad_reduce_kernel adds the chunks in order (fp32 atomic adds into zeroed outputs took
// 122 + 8 us instead of 85 for the four gradients of a 412-wide layer with 2 x 76 columns, 5 experts and 4096 tokens: the
// matrix pipe alone needs 35).
// ----------------------------------------------------------------------------------------
static constexpr int FWG_MAX_CHUNK = 768;

template <int NJ, int VEC>
__device__ __forceinline__ void f32_wgrad_body(const F32Wgrad& p, int blk, float* As, float* Bs, int* ids_a, int* ids_b, float* gsc) {
  constexpr int BM = 64, BN = 16 * NJ, LDA = BM + 4, LDB = BN + 4;
  typedef typename FVec<VEC>::type vec_t;
  const WgradArgs& a = p.w;
  const int ti = (a.Ka + BM - 1) / BM, tj = (a.Kb + BN - 1) / BN;
  const int tile = blk % (ti * tj), unit = blk / (ti * tj);
  int h, e = 0, row0 = 0, rows;
  if (p.nch == 1) {   // one chunk per group; an empty group stores its zeros
    h = unit / a.E;
    e = unit % a.E;
    rows = a.M;
    if (a.perm) {
      const int* off = a.offsets + (long)h * (a.E + 1);
      row0 = off[e];
      rows = off[e + 1] - row0;
    }
  } else {            // the unit-th chunk among those of the head's groups
    h = unit / p.slots;
    if (a.perm) {
      if (!find_tile_wave(a.offsets + (long)h * (a.E + 1), a.E, a.chunk, unit % p.slots, threadIdx.x & 63, e, row0, rows)) return;
    } else {
      row0 = unit % p.slots * a.chunk;
      rows = min(a.M - row0, a.chunk);
    }
  }
  const int which = a.hsplit > 0 ? h / a.hsplit : 0, hh = a.hsplit > 0 ? h % a.hsplit : h;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  for (int t = tid; t < rows; t += 256) {
    const int id = a.perm ? a.perm[(long)h * a.M + row0 + t] : row0 + t;
    ids_a[t] = id / a.a_div;
    ids_b[t] = id / a.b_div;
    gsc[t] = a.gate ? a.gate[(long)h * a.gate_hstride + id] : 1.f;
  }
  __syncthreads();
  const int i0 = (tile / tj) * BM, j0 = (tile % tj) * BN;
  const float* A = (const float*)a.A + (long)hh * a.a_hoff;
  const float* Bm = (const float*)(which ? a.Bm2 : a.Bm) + (long)hh * a.b_hoff;
  constexpr int A_CPR = BM / VEC, B_CPR = BN / VEC, A_N = 32 * A_CPR / 256, B_TOT = 32 * B_CPR, B_N = (B_TOT + 255) / 256;
  struct Step {
    vec_t ra[A_N], rb[B_N];
  };
  // unconditional loads, as in the row GEMM: rows past the chunk repeat its last row, features past the end feature 0
  auto load = [&](Step& st, int r0) {
#pragma unroll
    for (int i = 0; i < A_N; ++i) {
      const int c = tid + i * 256, rr = min(r0 + c / A_CPR, rows - 1), f = i0 + (c % A_CPR) * VEC;
      st.ra[i] = *(const vec_t*)(A + (long)ids_a[rr] * a.lda + (f < a.Ka ? f : 0));
    }
#pragma unroll
    for (int i = 0; i < B_N; ++i) {
      const int c = tid + i * 256, rr = min(r0 + c / B_CPR, rows - 1), f = j0 + (c % B_CPR) * VEC;
      st.rb[i] = *(const vec_t*)(Bm + (long)ids_b[rr] * a.ldb + (f < a.Kb ? f : 0));
    }
  };
  // the gate goes to one side, rows past the chunk become zeros on both (features past the end reach only results
  // that are not stored)
  auto store = [&](const Step& st, int stage, int r0) {
#pragma unroll
    for (int i = 0; i < A_N; ++i) {
      const int c = tid + i * 256, rr = r0 + c / A_CPR;
      vec_t v = st.ra[i] * gsc[min(rr, rows - 1)];
      if (rr >= rows) v = vec_t{};
      *(vec_t*)&As[stage * 32 * LDA + (c / A_CPR) * LDA + (c % A_CPR) * VEC] = v;
    }
#pragma unroll
    for (int i = 0; i < B_N; ++i) {
      const int c = tid + i * 256;
      if (B_TOT % 256 == 0 || c < B_TOT) *(vec_t*)&Bs[stage * 32 * LDB + (c / B_CPR) * LDB + (c % B_CPR) * VEC] = st.rb[i];
    }
    if (r0 + 32 > rows) {   // uniform; a thread's own pieces, as in the row GEMM
#pragma unroll
      for (int i = 0; i < B_N; ++i) {
        const int c = tid + i * 256;
        if ((B_TOT % 256 == 0 || c < B_TOT) && r0 + c / B_CPR >= rows)
          *(vec_t*)&Bs[stage * 32 * LDB + (c / B_CPR) * LDB + (c % B_CPR) * VEC] = vec_t{};
      }
    }
  };
  f32x4 acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = f32x4{};
  auto compute = [&](int stage) {
    const float *Ap = As + stage * 32 * LDA, *Bp = Bs + stage * 32 * LDB;
#pragma unroll
    for (int c = 0; c < 32; c += 16)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int k = c + 4 * g + t;
        const float fa = Ap[k * LDA + wave * 16 + r];
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[j] = mfma_16x16x4(fa, Bp[k * LDB + j * 16 + r], acc[j]);
      }
  };
  if (rows > 0) {
    Step s0, s1;
    load(s0, 0);
    load(s1, 32);
    for (int r0 = 0; r0 < rows; r0 += 64) {
      store(s0, 0, r0);
      __syncthreads();
      load(s0, r0 + 64);
      compute(0);
      if (r0 + 32 >= rows) break;
      store(s1, 1, r0 + 32);
      __syncthreads();
      load(s1, r0 + 96);
      compute(1);
    }
  }
  const int jmax = a.kb_store ? a.kb_store : a.Kb;
  float* out = (which ? a.dW2 : a.dW) + (long)hh * a.w_hstride + (long)e * a.w_estride;
  int ld = a.swa;
  if (p.nch > 1 && !p.add) {
    out = a.partial + (long)unit * a.Ka * jmax;
    ld = p.transposed ? a.Ka : jmax;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int ii = i0 + wave * 16 + 4 * g + v;
    if (ii >= a.Ka) continue;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int jj = j0 + j * 16 + r;
      if (jj >= jmax) continue;
      float* o = out + (p.transposed ? (long)jj * ld + ii : (long)ii * ld + jj);
      if (p.add)
        atomicAdd(o, acc[j][v]);
      else
        *o = acc[j][v];
    }
  }
}

// out[group] = the sum of its chunks' partial sums, in chunk order; one output element per thread, blockIdx.y = problem
__global__ __launch_bounds__(256) void f32_wgrad_reduce_kernel(F32WgradList l) {
  const F32Wgrad& p = l.p[blockIdx.y];
  const WgradArgs& a = p.w;
  if (p.nch == 1 || p.add) return;
  const int jmax = a.kb_store ? a.kb_store : a.Kb, per = a.Ka * jmax;
  const int nb = (per + 255) / 256;
  const int grp = blockIdx.x / nb, i = (blockIdx.x % nb) * 256 + threadIdx.x;
  if (grp >= a.heads * a.E) return;
  const int h = grp / a.E, e = grp % a.E;
  int first = 0, n = p.slots;
  if (a.perm) {
    const int* off = a.offsets + (long)h * (a.E + 1);
    for (int q = 0; q < e; ++q) first += (off[q + 1] - off[q] + a.chunk - 1) / a.chunk;
    n = (off[e + 1] - off[e] + a.chunk - 1) / a.chunk;
  }
  if (i >= per) return;
  const float* P = a.partial + ((long)h * p.slots + first) * per + i;
  float s = 0.f;
  for (int c = 0; c < n; ++c) s += P[(long)c * per];
  const int which = a.hsplit > 0 ? h / a.hsplit : 0, hh = a.hsplit > 0 ? h % a.hsplit : h;
  const int w = p.transposed ? a.Ka : jmax;   // the output's row length
  (which ? a.dW2 : a.dW)[(long)hh * a.w_hstride + (long)e * a.w_estride + (long)(i / w) * a.swa + i % w] = s;
}

template <int VEC>
__global__ __launch_bounds__(256) void f32_wgrad_kernel(F32WgradList l) {
  __shared__ __attribute__((aligned(16))) float As[2 * 32 * 68];
  __shared__ __attribute__((aligned(16))) float Bs[2 * 32 * 84];
  __shared__ int ids_a[FWG_MAX_CHUNK], ids_b[FWG_MAX_CHUNK];
  __shared__ float gsc[FWG_MAX_CHUNK];
  int q = 0, blk = blockIdx.x;
  while (q + 1 < l.n && blk >= l.p[q].blocks) blk -= l.p[q++].blocks;
  const F32Wgrad& p = l.p[q];
  if (p.nj == 5)
    f32_wgrad_body<5, VEC>(p, blk, As, Bs, ids_a, ids_b, gsc);
  else if (p.nj == 4)
    f32_wgrad_body<4, VEC>(p, blk, As, Bs, ids_a, ids_b, gsc);
  else
    f32_wgrad_body<2, VEC>(p, blk, As, Bs, ids_a, ids_b, gsc);
}

// Rows per chunk and the tile of one problem.  A group of at most 256 rows is one chunk, longer ones are cut.
void f32_wgrad_plan(F32Wgrad& p) {
  WgradArgs& a = p.w;
  // the narrower feature side takes the 16 NJ columns of the tile, padded less than the 64 of the other
  p.transposed = 0;
  if (a.Kb > a.Ka && a.kb_store == 0 && a.hsplit == 0) {
    const WgradArgs b = a;
    a.A = b.Bm, a.lda = b.ldb, a.a_hoff = b.b_hoff, a.Ka = b.Kb, a.a_div = b.b_div;
    a.Bm = b.A, a.ldb = b.lda, a.b_hoff = b.a_hoff, a.Kb = b.Ka, a.b_div = b.a_div;
    p.transposed = 1;
  }
  p.nj = f32_nj(a.Kb);
  const int rows = a.perm ? a.max_group_rows : a.M;
  const int tiles = ((a.Ka + 63) / 64) * ((a.Kb + 16 * p.nj - 1) / (16 * p.nj));
  if (rows <= 256) {
    a.chunk = (rows + 31) / 32 * 32;
  } else {
    // about 512 work-groups for the problem (two per CU): a group's expected rows are M / E
    const long units = 512 / tiles > 0 ? 512 / tiles : 1;
    long c = ((long)a.heads * a.M + units - 1) / units;
    c = (c + 31) / 32 * 32;
    a.chunk = (int)(c < 128 ? 128 : c > FWG_MAX_CHUNK ? FWG_MAX_CHUNK : c);
  }
  p.nch = (rows + a.chunk - 1) / a.chunk;
  p.slots = p.nch == 1 ? a.E : a.perm ? a.M / a.chunk + a.E : p.nch;   // per head: chunks, rounded up in every group
  p.blocks = tiles * p.slots * a.heads;
  p.partial_floats = p.nch == 1 ? 0 : (size_t)p.slots * a.heads * a.Ka * (a.kb_store ? a.kb_store : a.Kb);
}

void launch_f32_wgrad(const F32WgradList& l, hipStream_t s) {
  long blocks = 0, red = 0;
  bool v4 = true;
  for (int i = 0; i < l.n; ++i) {
    const WgradArgs& a = l.p[i].w;
    blocks += l.p[i].blocks;
    if (l.p[i].nch > 1 && !l.p[i].add) {
      const long nb = (long)(((long)a.Ka * (a.kb_store ? a.kb_store : a.Kb) + 255) / 256) * a.heads * a.E;
      red = nb > red ? nb : red;
    }
    auto al = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
    v4 = v4 && al(a.A) && al(a.Bm) && (a.hsplit == 0 || al(a.Bm2)) && a.lda % 4 == 0 && a.ldb % 4 == 0 && a.a_hoff % 4 == 0 &&
         a.b_hoff % 4 == 0 && a.Ka % 4 == 0 && a.Kb % 4 == 0;
  }
  if (!blocks) return;
  if (v4)
    f32_wgrad_kernel<4><<<(unsigned)blocks, 256, 0, s>>>(l);
  else
    f32_wgrad_kernel<1><<<(unsigned)blocks, 256, 0, s>>>(l);
  if (red) f32_wgrad_reduce_kernel<<<dim3((unsigned)red, l.n), 256, 0, s>>>(l);
}

// ----------------------------------------------------------------------------------------
// Attention.  A work-group owns 32 rows of one side (queries: forward, dQ; keys: dK, dV) and walks tiles of KT rows of the
// other in LDS; wave w owns 16 of the 32 and takes half of each tile's 16-row blocks (w >> 1), the two halves are merged
// through LDS at the end.  Scores are computed with the owned side in the columns of the result, S^T[key][query] (S[query][key]
// for dK / dV), so that register v of the result, row 4 g + v, is directly the B operand of the second product when its
// reduction index is taken in the order {4 g + v}.  Bound by the matrix pipe (5 k cycles per 16 owned rows and 64 rows of the
// other side at a head width of 80) and, at the sequence counts of small models, by how few work-groups there are: hence 32
// owned rows with the tile's blocks split, not 64.
// ----------------------------------------------------------------------------------------
template <int DH>
__host__ __device__ constexpr int f32_attn_kt() {
  return DH > 128 ? 32 : 64;
}

// NROWS rows of dh floats on their way into LDS [row][DH + 4]: load() requests them (16-byte rows: v4), store() writes them;
// columns past dh and rows outside lo .. hi - 1 zero.  Rows that no owned row sees stay out that way: a probability of zero
// would turn an infinity or a NaN of theirs into a NaN.
template <int DH, int NROWS>
struct F32Tile {
  static constexpr int LD = DH + 4, CPR = DH / 4, N = NROWS * CPR / 256;
  f32x4 v[N];
  const float* src;
  int valid;
  __device__ __forceinline__ void load(const float* s, long rs, int valid_rows, int dh, bool v4, int tid) {
    src = s;
    valid = valid_rows;
    if (!v4 || valid_rows <= 0) return;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int c = tid + i * 256, d = (c % CPR) * 4;
      v[i] = *(const f32x4*)(s + (long)min(c / CPR, valid_rows - 1) * rs + (d < dh ? d : 0));
    }
  }
  __device__ __forceinline__ void store(float* dst, long rs, int dh, bool v4, int tid, int lo, int hi) const {
    if (v4) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int c = tid + i * 256, d = (c % CPR) * 4;
        *(f32x4*)&dst[(c / CPR) * LD + d] = d < dh ? v[i] : f32x4{};
      }
      if (lo > 0 || hi < NROWS) {   // uniform; a thread's own pieces
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const int c = tid + i * 256, row = c / CPR;
          if (row < lo || row >= hi) *(f32x4*)&dst[row * LD + (c % CPR) * 4] = f32x4{};
        }
      }
    } else {
      for (int c = tid; c < NROWS * DH; c += 256) {
        const int row = c / DH, d = c % DH;
        dst[row * LD + d] = d < dh && row >= lo && row < hi ? src[(long)min(row, valid - 1) * rs + d] : 0.f;
      }
    }
  }
};

// operand fragments of one row: element [c][t] = row[16 c + 4 g + t]
template <int NC>
__device__ __forceinline__ void f32_row_frags(f32x4 (&f)[NC], const float* row, int g, int dh, bool ok) {
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int d = 16 * c + 4 * g + t;
      f[c][t] = ok && d < dh ? row[d] : 0.f;
    }
}

template <int NC>
__device__ __forceinline__ f32x4 f32_dot_block(const float* tile, int ld, int row, int g, const f32x4 (&f)[NC]) {
  f32x4 s = f32x4{};
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const f32x4 fa = *(const f32x4*)&tile[row * ld + 16 * c + 4 * g];
#pragma unroll
    for (int t = 0; t < 4; ++t) s = mfma_16x16x4(fa[t], f[c][t], s);
  }
  return s;
}

// acc[c][d = 16 c + 4 g + v][col r] += sum over the 16 rows of the block of tile[row][d] * p[row][col]
template <int NC>
__device__ __forceinline__ void f32_acc_block(f32x4 (&acc)[NC], const float* tile, int ld, int row0, int r, int g, f32x4 p) {
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = mfma_16x16x4(tile[(row0 + 4 * g + v) * ld + 16 * c + r], p[v], acc[c]);
}

template <int NC>
__device__ __forceinline__ void f32_store_cols(float* row, const f32x4 (&acc)[NC], float mul, int g, int dh) {
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (16 * c + 4 * g + v < dh) row[16 * c + 4 * g + v] = acc[c][v] * mul;
}

// the upper pair of waves parks its accumulators, the lower pair adds them
template <int NC>
__device__ __forceinline__ void f32_park(float* park, const f32x4 (&acc)[NC], int lane) {
#pragma unroll
  for (int c = 0; c < NC; ++c) *(f32x4*)&park[(c * 64 + lane) * 4] = acc[c];
}
template <int NC>
__device__ __forceinline__ void f32_unpark(f32x4 (&acc)[NC], const float* park, int lane, float f0, float f1) {
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = acc[c] * f0 + *(const f32x4*)&park[(c * 64 + lane) * 4] * f1;
}

template <int DH>
__global__ __launch_bounds__(256) void f32_attn_fwd_kernel(AttnArgs a, int v4, int rank0) {
  constexpr int KT = f32_attn_kt<DH>(), LD = DH + 4, NC = DH / 16, NB = KT / 32;   // NB: the wave's blocks of a tile
  extern __shared__ __attribute__((aligned(16))) float fl[];
  float *Ks = fl, *Vs = fl + KT * LD;
  const int T = a.T, dh = a.dh, Tq = a.Tq > 0 ? a.Tq : T, off = T - Tq;
  const int nt = (Tq + 31) / 32, pair = blockIdx.y * gridDim.x + blockIdx.x;
  if (pair >= a.B * a.H) return;
  const int tile = nt - 1 - rank0 - (int)blockIdx.z;   // under a causal mask the long tiles come first
  const int b = pair / a.H, h = pair % a.H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
  const int kb0 = (wave >> 1) * NB;
  const long rs = (long)a.H * dh;
  const float* Q = (const float*)a.Q + (long)b * Tq * rs + (long)h * dh;
  const float* K = (const float*)a.K + (long)b * T * rs + (long)h * dh;
  const float* V = (const float*)a.V + (long)b * T * rs + (long)h * dh;
  const int q0 = tile * 32, q = q0 + (wave & 1) * 16 + r;
  F32Tile<DH, KT> tk, tv;
  tk.load(K, rs, T, dh, v4, tid);
  tv.load(V, rs, T, dh, v4, tid);
  f32x4 qf[NC], o[NC];
  f32_row_frags<NC>(qf, Q + (long)q * rs, g, dh, q < Tq);
#pragma unroll
  for (int c = 0; c < NC; ++c) o[c] = f32x4{};
  float m = -INFINITY, l = 0.f;
  const float sc = a.scale * 1.44269504088896340736f;   // logits in log2 units
  const int kend = a.causal ? min(T, min(q0 + 32, Tq) + off) : T;
  const int last = a.causal ? min(T - 1, q + off) : T - 1;   // this lane's last visible key
  for (int k0 = 0; k0 < kend; k0 += KT) {
    __syncthreads();
    tk.store(Ks, rs, dh, v4, tid, 0, kend - k0);
    tv.store(Vs, rs, dh, v4, tid, 0, kend - k0);
    __syncthreads();
    if (k0 + KT < kend) {
      tk.load(K + (long)(k0 + KT) * rs, rs, T - k0 - KT, dh, v4, tid);
      tv.load(V + (long)(k0 + KT) * rs, rs, T - k0 - KT, dh, v4, tid);
    }
    f32x4 s[NB];
    float mt = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < NB; ++kb) {
      s[kb] = f32_dot_block<NC>(Ks, LD, (kb0 + kb) * 16 + r, g, qf);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        s[kb][v] = k0 + (kb0 + kb) * 16 + 4 * g + v <= last ? s[kb][v] * sc : -INFINITY;
        mt = fmaxf(mt, s[kb][v]);
      }
    }
    mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
    const float mn = fmaxf(m, mt), mb = mn == -INFINITY ? 0.f : mn;   // (no key seen yet: a half tile wholly masked)
    const float alpha = __builtin_amdgcn_exp2f(m - mb);
    m = mn;
    float ps = 0.f;
#pragma unroll
    for (int kb = 0; kb < NB; ++kb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        s[kb][v] = __builtin_amdgcn_exp2f(s[kb][v] - mb);
        ps += s[kb][v];
      }
    l = l * alpha + ps;
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] *= alpha;
#pragma unroll
    for (int kb = 0; kb < NB; ++kb) f32_acc_block<NC>(o, Vs, LD, (kb0 + kb) * 16, r, g, s[kb]);
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  __syncthreads();   // the tiles are dead
  float* park = fl + (wave & 1) * (NC * 256 + 128);
  if (wave >= 2) {
    f32_park<NC>(park, o, lane);
    park[NC * 256 + lane] = m;
    park[NC * 256 + 64 + lane] = l;
  }
  __syncthreads();
  if (wave >= 2) return;
  // the upper half may have seen no key (m = -inf, factor 0); the lower one always has (key 0)
  const float m1 = park[NC * 256 + lane], l1 = park[NC * 256 + 64 + lane], mn = fmaxf(m, m1);
  const float f0 = __builtin_amdgcn_exp2f(m - mn), f1 = __builtin_amdgcn_exp2f(m1 - mn);
  f32_unpark<NC>(o, park, lane, f0, f1);
  l = l * f0 + l1 * f1;
  if (q < Tq) {
    f32_store_cols<NC>((float*)a.O + (long)b * Tq * rs + (long)h * dh + (long)q * rs, o, 1.f / l, g, dh);
    if (g == 0) a.lse[((long)b * a.H + h) * Tq + q] = (mn + log2f(l)) * 0.69314718055994530942f;
  }
}

// Backward, one launch: the first blocks own 32 queries each (dQ), the rest 32 keys (dK, dV); neither needs the other.
template <int DH>
__global__ __launch_bounds__(256) void f32_attn_bwd_kernel(AttnBwdArgs a, int v4, int rank0) {
  constexpr int KT = f32_attn_kt<DH>(), LD = DH + 4, NC = DH / 16, NB = KT / 32;
  extern __shared__ __attribute__((aligned(16))) float fl[];
  float *t0 = fl, *t1 = fl + KT * LD, *ls = t1 + KT * LD, *dl = ls + KT;
  const int T = a.T, dh = a.dh, Tq = a.Tq > 0 ? a.Tq : T, off = T - Tq;
  const int nq = (Tq + 31) / 32, rank = rank0 + (int)blockIdx.z, pair = blockIdx.y * gridDim.x + blockIdx.x;
  if (pair >= a.B * a.H) return;
  const int b = pair / a.H, h = pair % a.H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
  const int b0 = (wave >> 1) * NB, own = (wave & 1) * 16 + r;
  const long rs = (long)a.H * dh;
  const long kbase = (long)b * T * rs + (long)h * dh, qbase = (long)b * Tq * rs + (long)h * dh;
  const float *Q = (const float*)a.Q + qbase, *dO = (const float*)a.dO + qbase;
  const float *K = (const float*)a.K + kbase, *V = (const float*)a.V + kbase;
  const float* lse = a.lse + ((long)b * a.H + h) * Tq;
  const float* delta = a.delta + (long)b * Tq * a.H + h;
  const float sc = a.scale * 1.44269504088896340736f;
  F32Tile<DH, KT> ta, tb;
  if (rank < nq) {
    const int q0 = (nq - 1 - rank) * 32, q = q0 + own;
    ta.load(K, rs, T, dh, v4, tid);
    tb.load(V, rs, T, dh, v4, tid);
    f32x4 qf[NC], gf[NC], acc[NC];
    f32_row_frags<NC>(qf, Q + (long)q * rs, g, dh, q < Tq);
    f32_row_frags<NC>(gf, dO + (long)q * rs, g, dh, q < Tq);
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = f32x4{};
    const float L = q < Tq ? lse[q] * 1.44269504088896340736f : 0.f, D = q < Tq ? delta[(long)q * a.H] : 0.f;
    const int kend = a.causal ? min(T, min(q0 + 32, Tq) + off) : T;
    const int last = a.causal ? min(T - 1, q + off) : T - 1;
    for (int k0 = 0; k0 < kend; k0 += KT) {
      __syncthreads();
      ta.store(t0, rs, dh, v4, tid, 0, kend - k0);
      tb.store(t1, rs, dh, v4, tid, 0, kend - k0);
      __syncthreads();
      if (k0 + KT < kend) {
        ta.load(K + (long)(k0 + KT) * rs, rs, T - k0 - KT, dh, v4, tid);
        tb.load(V + (long)(k0 + KT) * rs, rs, T - k0 - KT, dh, v4, tid);
      }
#pragma unroll
      for (int kb = b0; kb < b0 + NB; ++kb) {
        f32x4 s = f32_dot_block<NC>(t0, LD, kb * 16 + r, g, qf);
        const f32x4 dp = f32_dot_block<NC>(t1, LD, kb * 16 + r, g, gf);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[v], sc, -L));
          s[v] = k0 + kb * 16 + 4 * g + v <= last ? p * (dp[v] - D) : 0.f;
        }
        f32_acc_block<NC>(acc, t0, LD, kb * 16, r, g, s);
      }
    }
    __syncthreads();
    float* park = fl + (wave & 1) * NC * 256;
    if (wave >= 2) f32_park<NC>(park, acc, lane);
    __syncthreads();
    if (wave >= 2) return;
    f32_unpark<NC>(acc, park, lane, 1.f, 1.f);
    if (q < Tq) f32_store_cols<NC>((float*)a.dQ + qbase + (long)q * rs, acc, a.scale, g, dh);
    return;
  }
  const int u0 = (rank - nq) * 32, u = u0 + own;
  f32x4 kf[NC], vf[NC], ak[NC], av[NC];
  f32_row_frags<NC>(kf, K + (long)u * rs, g, dh, u < T);
  f32_row_frags<NC>(vf, V + (long)u * rs, g, dh, u < T);
#pragma unroll
  for (int c = 0; c < NC; ++c) ak[c] = av[c] = f32x4{};
  const int qfirst = a.causal ? max(u0 - off, 0) : 0, qbeg = qfirst / KT * KT;   // the first query that sees an owned key
  float nl = 0.f, nd = 0.f;
  auto request = [&](int qt) {
    ta.load(Q + (long)qt * rs, rs, Tq - qt, dh, v4, tid);
    tb.load(dO + (long)qt * rs, rs, Tq - qt, dh, v4, tid);
    const int q = min(qt + (tid & (KT - 1)), Tq - 1);
    nl = lse[q];
    nd = delta[(long)q * a.H];
  };
  if (qbeg < Tq) request(qbeg);
  for (int qt = qbeg; qt < Tq; qt += KT) {
    __syncthreads();
    ta.store(t0, rs, dh, v4, tid, qfirst - qt, Tq - qt);
    tb.store(t1, rs, dh, v4, tid, qfirst - qt, Tq - qt);
    if (tid < KT) {
      ls[tid] = nl * 1.44269504088896340736f;
      dl[tid] = nd;
    }
    __syncthreads();
    if (qt + KT < Tq) request(qt + KT);
#pragma unroll
    for (int qb = b0; qb < b0 + NB; ++qb) {
      f32x4 s = f32_dot_block<NC>(t0, LD, qb * 16 + r, g, kf);
      f32x4 dp = f32_dot_block<NC>(t1, LD, qb * 16 + r, g, vf);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ql = qb * 16 + 4 * g + v, q = qt + ql;
        const bool vis = q < Tq && u < T && (!a.causal || u <= q + off);
        const float p = vis ? __builtin_amdgcn_exp2f(fmaf(s[v], sc, -ls[ql])) : 0.f;
        s[v] = p;
        dp[v] = vis ? p * (dp[v] - dl[ql]) : 0.f;
      }
      f32_acc_block<NC>(av, t1, LD, qb * 16, r, g, s);
      f32_acc_block<NC>(ak, t0, LD, qb * 16, r, g, dp);
    }
  }
  __syncthreads();
  float* park = fl + (wave & 1) * NC * 512;
  if (wave >= 2) {
    f32_park<NC>(park, ak, lane);
    f32_park<NC>(park + NC * 256, av, lane);
  }
  __syncthreads();
  if (wave >= 2 || u >= T) return;
  f32_unpark<NC>(ak, park, lane, 1.f, 1.f);
  f32_unpark<NC>(av, park + NC * 256, lane, 1.f, 1.f);
  f32_store_cols<NC>((float*)a.dK + kbase + (long)u * rs, ak, a.scale, g, dh);
  f32_store_cols<NC>((float*)a.dV + kbase + (long)u * rs, av, 1.f, g, dh);
}

template <int DH>
static void launch_f32_attn_dh(const AttnArgs* f, const AttnBwdArgs* bw, hipStream_t s) {
  constexpr int KT = f32_attn_kt<DH>();
  const size_t lds = sizeof(float) * (size_t)(2 * KT * (DH + 4) + 2 * KT);
  auto al = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  const int B = f ? f->B : bw->B, H = f ? f->H : bw->H, T = f ? f->T : bw->T, tq = f ? f->Tq : bw->Tq, Tq = tq > 0 ? tq : T;
  const int ranks = (Tq + 31) / 32 + (f ? 0 : (T + 31) / 32);
  // a dimension of the grid holds less than 2^32 threads, y and z at most 65535 blocks; any B, H and T get through
  const unsigned P = (unsigned)B * (unsigned)H, px = P < (1u << 22) ? P : 1u << 22, py = (P + px - 1) / px;
  if (f) {
    const int v4 = f->dh % 4 == 0 && al(f->K) && al(f->V);
    if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)f32_attn_fwd_kernel<DH>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    for (int r0 = 0; r0 < ranks; r0 += 65535) f32_attn_fwd_kernel<DH><<<dim3(px, py, min(ranks - r0, 65535)), 256, lds, s>>>(*f, v4, r0);
  } else {
    const int v4 = bw->dh % 4 == 0 && al(bw->K) && al(bw->V) && al(bw->Q) && al(bw->dO);
    if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)f32_attn_bwd_kernel<DH>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    for (int r0 = 0; r0 < ranks; r0 += 65535) f32_attn_bwd_kernel<DH><<<dim3(px, py, min(ranks - r0, 65535)), 256, lds, s>>>(*bw, v4, r0);
  }
}

static void dispatch_f32_attn(int dh, const AttnArgs* f, const AttnBwdArgs* bw, hipStream_t s) {
  if (dh <= 32)
    launch_f32_attn_dh<32>(f, bw, s);
  else if (dh <= 64)
    launch_f32_attn_dh<64>(f, bw, s);
  else if (dh <= 80)
    launch_f32_attn_dh<80>(f, bw, s);
  else if (dh <= 128)
    launch_f32_attn_dh<128>(f, bw, s);
  else if (dh <= 192)
    launch_f32_attn_dh<192>(f, bw, s);
  else
    launch_f32_attn_dh<256>(f, bw, s);
}
void launch_f32_attn_fwd(const AttnArgs& a, hipStream_t s) { dispatch_f32_attn(a.dh, &a, nullptr, s); }
void launch_f32_attn_bwd(const AttnBwdArgs& a, hipStream_t s) { dispatch_f32_attn(a.dh, nullptr, &a, s); }

}  // namespace sh
