// Router of the SwitchHead layer (arXiv 2312.07987, Sec. 2.2: s = sigmoid(x W), argtopk)
// and the expert-sorted permutation of the token->expert assignments (the "sorting and
// top-k steps" of Sec. 3.6 "Shared Selection").
//
//   select    z = x W (+ b) in fp64, summed over i = 0..d_model-1 in that order with one
//             accumulator per logit, so the selection is a fixed function of the stored inputs
//             (products of bf16/fp32 inputs are exact in fp64); per (side, head, token) k passes of
//             "largest remaining logit, lowest index on ties"; gate = sigmoid(logit); expert counts
//             of the work-group's tokens
//   scan      exclusive scan over (expert major, token block minor), done by every scatter block for
//             itself where the table of counts is small; counts are [side, head][bin][token block]
//   scatter   stable placement: rank inside the block from ballots + popcounts, so
//             no atomics decide an order and the result is deterministic
#include "common.h"
#include "mfma_util.h"

namespace sh {

static constexpr int RT_TOK = 32;    // tokens per work-group of either router, and per block of counts
static constexpr int RT_KC = 64;     // d_model chunk staged in LDS
static constexpr int RB = 256;       // tokens per block of the scatter kernels

int router_blocks(int N) { return (N + RB - 1) / RB; }
int router_count_blocks(int N) { return (N + RT_TOK - 1) / RT_TOK; }

// Logits, selection and expert counts in one launch.  A work-group takes 32 tokens of one side (and as many whole heads as
// 64 logit columns hold): 8 threads per token, each with every eighth column, so a thread runs CPT fp64 chains over the
// features.  x and W go through LDS as fp32 in slabs of RT_KC features, the next slab waits in registers.  Bound by the
// latency of the slab loads and by the fp64 chains (one accumulator per logit, so a logit is d_model dependent FMAs); the
// earlier form (64 tokens, 16 columns per thread, 32 features per barrier pair, selection and histogram in a second launch,
// tables scanned in a third) took 156 us for 4096 tokens of d_model 412 with 2 x 10 columns, most of its threads on padding.
template <typename T, int CPT>
__global__ __launch_bounds__(256) void router_select_kernel(const T* __restrict__ x, const T* __restrict__ W0,
                                                            const T* __restrict__ W1, const float* __restrict__ b0,
                                                            const float* __restrict__ b1, int* __restrict__ idx,
                                                            float* __restrict__ gate, int* __restrict__ cnt, int N, int dm,
                                                            int H, int E, int k, int hpb, int ncb) {
  constexpr int NC = 8 * CPT;   // columns held in LDS
  constexpr int LX = RT_KC + 1;
  __shared__ float xs[RT_TOK * LX];
  __shared__ float ws[RT_KC * NC];
  __shared__ double z[RT_TOK][NC + 1];
  __shared__ int cn[NC];
  const int side = blockIdx.y, HE = H * E;
  const int h0 = blockIdx.z * hpb, nh = min(hpb, H - h0), ncols = nh * E, col0 = h0 * E;
  const T* W = side ? W1 : W0;
  const float* b = side ? b1 : b0;
  const int tok0 = blockIdx.x * RT_TOK;
  const int tid = threadIdx.x, tok = tid & (RT_TOK - 1), cg = tid / RT_TOK;
  constexpr int XN = RT_TOK * RT_KC / 256, WN = (RT_KC * NC + 255) / 256;
  T rx[XN], rw[WN];
  // (an index past the end loads element 0 and is replaced by zero in put(): no branch around a load)
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < XN; ++i) {
      const int t = tid + i * 256, n = tok0 + t / RT_KC, kk = k0 + t % RT_KC;
      rx[i] = x[n < N && kk < dm ? (long)n * dm + kk : 0];
    }
#pragma unroll
    for (int i = 0; i < WN; ++i) {
      const int t = tid + i * 256, kk = k0 + t / NC, c = t % NC;
      rw[i] = W[kk < dm && c < ncols ? (long)kk * HE + col0 + c : 0];
    }
  };
  auto put = [&](int k0) {
#pragma unroll
    for (int i = 0; i < XN; ++i) {
      const int t = tid + i * 256, n = tok0 + t / RT_KC, kk = k0 + t % RT_KC;
      xs[(t / RT_KC) * LX + t % RT_KC] = n < N && kk < dm ? ld(&rx[i], 0) : 0.f;
    }
#pragma unroll
    for (int i = 0; i < WN; ++i) {
      const int t = tid + i * 256, kk = k0 + t / NC, c = t % NC;
      if (t < RT_KC * NC) ws[t] = kk < dm && c < ncols ? ld(&rw[i], 0) : 0.f;
    }
  };
  double acc[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) acc[c] = 0.0;
  fetch(0);
  for (int k0 = 0; k0 < dm; k0 += RT_KC) {
    put(k0);
    __syncthreads();
    if (k0 + RT_KC < dm) fetch(k0 + RT_KC);
    // strictly ascending feature index; the zero padding beyond d_model adds exact zeros
#pragma unroll 8
    for (int i = 0; i < RT_KC; ++i) {
      const double xv = (double)xs[tok * LX + i];
#pragma unroll
      for (int c = 0; c < CPT; ++c) acc[c] = fma(xv, (double)ws[i * NC + cg + 8 * c], acc[c]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int col = cg + 8 * c;
    if (col < ncols) z[tok][col] = acc[c] + (b ? (double)b[col0 + col] : 0.0);
  }
  if (tid < NC) cn[tid] = 0;
  __syncthreads();
  for (int item = tid; item < RT_TOK * nh; item += 256) {
    const int t = item % RT_TOK, h = item / RT_TOK, n = tok0 + t;
    if (n >= N) continue;
    const double* zt = &z[t][h * E];
    unsigned long long sel = 0ull;
    const long o = ((long)(side * H + h0 + h) * N + n) * k;
    for (int j = 0; j < k; ++j) {
      int best = -1;
      double bv = 0.0;
      for (int e = 0; e < E; ++e) {
        if ((sel >> e) & 1ull) continue;
        const double v = zt[e];
        if (best < 0 || v > bv) {  // strict: the lower index keeps a tie
          best = e;
          bv = v;
        }
      }
      sel |= 1ull << best;
      idx[o + j] = best;
      gate[o + j] = (float)(1.0 / (1.0 + exp(-bv)));
      atomicAdd(&cn[h * E + best], 1);
    }
  }
  __syncthreads();
  for (int c = tid; c < ncols; c += 256) cnt[((long)(side * H + h0) * E + c) * ncb + blockIdx.x] = cn[c];
}

// sum over the 16 lanes of a row (rotations inside the row)
__device__ __forceinline__ int row_sum(int v) {
  v += __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, false);
  v += __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, false);
  v += __builtin_amdgcn_mov_dpp(v, 0x122, 0xf, 0xf, false);
  return v + __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, false);
}

// Starts of the bins in LDS: sbase[bin] becomes the first position of bin `bin` for token block blockIdx.x.
//   in: sbase[bin] the bin's count in the token blocks before this one, sbase[128 + bin] in all.  Token block 0 also writes
// offsets[0..nbins].  Called by all RB threads (at most 128 bins); barriers on both sides.
__device__ __forceinline__ void add_bin_starts(int* __restrict__ offsets, int nbins, int* __restrict__ sbase /* LDS [2 * 128] */) {
  const int* tot = sbase + 128;
  const int lane = threadIdx.x & 63;
  __syncthreads();
  if (threadIdx.x < 64) {   // exclusive sum over the bins
    const int v0 = lane < nbins ? tot[lane] : 0, v1 = lane + 64 < nbins ? tot[lane + 64] : 0;
    int p0 = v0, p1 = v1;
    for (int o = 1; o < 64 && o < nbins; o <<= 1) {
      const int u0 = __shfl_up(p0, o, 64), u1 = __shfl_up(p1, o, 64);
      if (lane >= o) {
        p0 += u0;
        p1 += u1;
      }
    }
    const int first_half = __shfl(p0, min(nbins, 64) - 1, 64);
    p1 += first_half;
    const int sum = nbins > 64 ? __shfl(p1, nbins - 65, 64) : first_half;
    if (lane < nbins) sbase[lane] += p0 - v0;
    if (lane + 64 < nbins) sbase[lane + 64] += p1 - v1;
    if (blockIdx.x == 0) {
      if (lane < nbins) offsets[lane] = p0 - v0;
      if (lane + 64 < nbins) offsets[lane + 64] = p1 - v1;
      if (lane == 0) offsets[nbins] = sum;
    }
  }
  __syncthreads();
}

// The same from the raw counts cnt[bin][count block] (for tables small enough that every block can read them whole): this token block
// holds the count blocks from blockIdx.x * per on.  16 lanes per bin, sixteen loads in flight.
__device__ __forceinline__ void block_bases(const int* __restrict__ cnt, int* __restrict__ offsets, int nbins, int ncb, int per,
                                            int* __restrict__ sbase) {
  const int first = blockIdx.x * per;
  const int lane = threadIdx.x & 63;
  int* tot = sbase + 128;
  for (int e0 = 0; e0 < nbins; e0 += RB / 16) {
    const int e = e0 + (threadIdx.x >> 4);
    const int* c = cnt + (long)min(e, nbins - 1) * ncb;
    int all = 0, pre = 0;
    for (int b0 = lane & 15; b0 - (lane & 15) < ncb; b0 += 256) {
      int v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = c[min(b0 + 16 * u, ncb - 1)];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int b = b0 + 16 * u;
        all += b < ncb ? v[u] : 0;
        pre += b < first ? v[u] : 0;   // (first < ncb)
      }
    }
    all = row_sum(all);
    pre = row_sum(pre);
    if ((lane & 15) == 0 && e < nbins) {
      tot[e] = all;
      sbase[e] = pre;
    }
  }
  add_bin_starts(offsets, nbins, sbase);
}

// ... and from the sums that scan_kernel left
__device__ __forceinline__ void stored_bases(const int* __restrict__ cnt, int* __restrict__ offsets, int nbins, int ncb, int per,
                                             int* __restrict__ sbase) {
  const int first = blockIdx.x * per;
  for (int e = threadIdx.x; e < nbins; e += RB) {
    const int* c = cnt + (long)e * ncb;
    sbase[128 + e] = c[0];
    sbase[e] = first ? c[first] : 0;
  }
  add_bin_starts(offsets, nbins, sbase);
}

// The waves' counts of a token block become their first positions.  base[e]: the block's.  Called by all threads; barriers
// on both sides.
template <int BINS>
__device__ __forceinline__ void wave_bases(int (&wcnt)[RB / 64][BINS], const int* base, int nbins) {
  __syncthreads();
  for (int e = threadIdx.x; e < nbins; e += RB) {
    int run = base[e];
#pragma unroll
    for (int w = 0; w < RB / 64; ++w) {
      const int v = wcnt[w][e];
      wcnt[w][e] = run;
      run += v;
    }
  }
  __syncthreads();
}

__global__ void dense_routing_kernel(int* idx, float* gate, int* perm, int* offsets, int n0, int n1, int H, int* setperm, float* gsort,
                                     int* setoff, int* setexp) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int side = blockIdx.y, N = side ? n1 : n0;
  const long at = (long)side * H * n0 + i;
  if (i < (long)H * N) {
    const int n = (int)(i % N);
    idx[at] = 0;
    gate[at] = 1.0f;
    perm[at] = n;
    if (setperm) {
      setperm[at] = n;
      gsort[at] = 1.0f;
    }
  }
  if (i < H) {
    const long o = (side * (long)H + i) * 2;
    offsets[o] = 0;
    offsets[o + 1] = N;
    if (setperm) {
      setoff[o] = 0;
      setoff[o + 1] = N;
    }
  }
  if (setperm && i == 0) setexp[0] = 0;
}

__global__ __launch_bounds__(256) void copy_list_kernel(CopyList l) {
  const unsigned* src = (const unsigned*)l.src[blockIdx.y];
  unsigned* dst = (unsigned*)l.dst[blockIdx.y];
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < l.count[blockIdx.y]; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

void launch_copy_list(const CopyList& l, hipStream_t s) {
  size_t mx = 0;
  for (int i = 0; i < l.n; ++i) mx = l.count[i] > mx ? l.count[i] : mx;
  if (!mx) return;
  const size_t b = (mx + 255) / 256;
  copy_list_kernel<<<dim3((unsigned)(b < 256 ? b : 256), l.n), 256, 0, s>>>(l);
}

// ----------------------------------------------------------------------------------------
// Two-stage router for bf16 storage, one launch: logits on the matrix cores, selection, fp64 recheck of doubtful decisions,
// block counts of both sorts, dense gate rows.
//
// Stage 1: a matrix instruction sums 32 exact bf16 x bf16 products in fp32, the two results of a K step of 64 are added in fp32, the K
// steps in fp64.  The distance from the canonical fp64 logit is bounded by
//   bound = 4 * KS * 2^-24 * |x_n|_2 * max_c |W[:,c]|_2  (+ 1e-13 relative for the fp64 adds),  KS = 33,
// a Cauchy-Schwarz bound on sum_i |x_i w_i| times the fp32 error of a 32-term sum and one addition, with a factor 4 of slack for the
// adder tree of the matrix core.  If every gap between consecutive sorted logits down to the (k+1)-th exceeds 2*bound, the ordered
// top-k list is provably the one the fp64 logits give.  Otherwise (a fraction of a percent, and every exact tie) stage 2
// re-evaluates the E logits in fp64 and selects from those.
//
// Stage 2 adds the products in a fixed blocked order (a lane takes a feature of each K step, then a butterfly, then the waves), the same
// for identical columns.  That is not the canonical order (one accumulator, i = 0 .. d_model-1 ascending, bias last), but both are fp64
// sums of the same exact products, so each lies within d_model * 2^-53 * sum|x_i w_i| of the true value and the two differ by
// at most twice that.  `reorder` is an upper bound of that difference (Cauchy-Schwarz, with slack): logits of the head that
// the blocked sum puts further apart are ordered the same way by the canonical sum.  If some pair is closer (every
// exact tie is), the canonical sums themselves are evaluated, an expert per lane, and the selection is made from them: the indices
// are those of the canonical logits in every case.
//
// A work-group takes 32 tokens of one side, its eight waves every eighth K step of 64.  A wave asks for everything it needs of S
// steps before it waits: its tokens' features go straight into operand fragments (16 rows of 64 contiguous bytes an instruction),
// the router's rows, contiguous in memory, through the wave's own corner of LDS, from where transposing reads make the other
// operand.  The norms of the bound are summed from the fragments (two products an instruction), the K steps' sums meet in LDS.
// Bound by one trip to memory and the chain of short steps behind it (25000 cycles for a tile, two or four tiles on a CU at a time), for many
// tokens by those tiles' vector instructions.  Router and sorts, us between events, against four launches (router packed and copied out as columns;
// logits on 64 x 64 tiles of the row GEMM, 20 of 64 columns used, and a recheck of one entry per wave; histogram; scan and scatter):
// d_model 1024, 2 x 20 columns, 100 tokens 45 -> 21, 6300 tokens 54 -> 27, 16384 tokens 53 -> 40; d_model 412, 2 x 10 columns, 16384
// tokens 49 -> 30; 2 x 32 columns, 16384 tokens 73 -> 52; 8000 cached and 8 query rows, with the copy of the latter, 54 -> 23.
// An entry whose logits tie takes one wave d_model / 16 trips to memory more, and the others wait for that wave at the barrier of the next
// entry but one: 16384 tokens of which 2 % are zeros 5.4 -> 3.9 ms, half of them 34 -> 12 ms.
// ----------------------------------------------------------------------------------------
struct RouterTileArgs {
  const unsigned short* x;
  const unsigned short* W[2];
  const float* b[2];
  int* idx;          // [side][H][N][k]
  float* gate;
  int* cnt;          // [side][H][E][count block]
  float* gtab;       // [side][N[0]][H*E] or NULL
  int* setid;        // NULL: no set tables
  float* gset;
  int* setexp;
  int* setcnt;       // [side][H][nsets][count block]
  unsigned short* xq;   // side 1's rows of x, packed, are written here (NULL: the sides share their tokens)
  int N[2], ncb[2], sides;
  int dm, H, E, k, nsets;
  int T, Tq;         // side 1 with tokens of its own: the last Tq of every T rows of x
};

constexpr int binom(int n, int r) {   // n < 64, results below 2^31 / n as far as they are used
  if (r < 0 || r > n) return 0;
  int v = 1;
  for (int i = 1; i <= r; ++i) v = v * (n - r + i) / i;
  return v;
}
struct BinomTable {
  int v[32][8];   // v[e][p] = C(e, p + 1)
  constexpr BinomTable() : v() {
    for (int e = 0; e < 32; ++e)
      for (int p = 0; p < 8; ++p) v[e][p] = binom(e, p + 1);
  }
};
__device__ const BinomTable binom_table = BinomTable();

// the ascending experts of every set (combinadic unranking), for the kernels that follow
__device__ __forceinline__ void write_set_experts(int* __restrict__ setexp, int nsets, int E, int k) {
  if ((int)threadIdx.x >= nsets) return;
  int rank = threadIdx.x;
  for (int p = k - 1; p >= 0; --p) {
    int x = p;
    while (x + 1 < E && binom(x + 1, p + 1) <= rank) ++x;
    rank -= binom(x, p + 1);
    setexp[threadIdx.x * 8 + p] = x;
  }
}

// sum of the squares of two bf16, added to s
__device__ __forceinline__ float sumsq2(unsigned w, float s) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const bf16x2_t v = __builtin_bit_cast(bf16x2_t, w);
  return __builtin_amdgcn_fdot2_f32_bf16(v, v, s, false);
}

__device__ __forceinline__ double bf16_to_f64(unsigned short v) { return (double)__uint_as_float((unsigned)v << 16); }

// k passes of "largest remaining logit, the lowest index on ties"
__device__ __forceinline__ void select_serial(const double* z, unsigned char* sel_out, int E, int k) {
  unsigned sel = 0;
  for (int j = 0; j < k; ++j) {
    int best = -1;
    double bv = 0.0;
    for (int e = 0; e < E; ++e) {
      if ((sel >> e) & 1u) continue;
      const double v = z[e];
      if (best < 0 || v > bv) {
        best = e;
        bv = v;
      }
    }
    sel |= 1u << best;
    sel_out[j] = (unsigned char)best;
  }
}

// The selection of one (token, head) from its fp64 logits z[0..E-1], by one wave.  xrow: the token's features; w: the head's first
// column (rows HE apart).
__device__ __forceinline__ void recheck_select(const unsigned short* __restrict__ xrow, const unsigned short* __restrict__ w, const float* __restrict__ bh,
                                               double* z, unsigned char* sel_out, int dm, int HE, int E, int k, int lane, double reorder) {
  bool close = false;
  if (E <= 8) {   // a lane per pair; the rank of an expert is the number of those that go before it
    const int e = lane >> 3, f = lane & 7;
    const double ze = z[min(e, E - 1)], zf = z[min(f, E - 1)];
    const bool pair = e < E && f < E && e != f;
    close = pair && !(fabs(ze - zf) > reorder);
    const unsigned long long before = __ballot(pair && zf > ze);
    if (!__ballot(close)) {
      const int rank = __popcll((before >> (8 * (lane & 7))) & 0xffull);
      if (lane < E && rank < k) sel_out[rank] = (unsigned char)lane;
      return;
    }
  } else {   // a lane per expert
    const double ze = z[min(lane, E - 1)];
    int rank = 0;
    for (int f0 = 0; f0 < E; f0 += 8) {
#pragma unroll
      for (int f = f0; f < f0 + 8; ++f) {
        const double zf = z[min(f, E - 1)];
        close = close || (f < E && f != lane && !(fabs(ze - zf) > reorder));
        rank += f < E && zf > ze;
      }
    }
    close = close && lane < E;
    if (!__ballot(close)) {
      if (lane < E && rank < k) sel_out[rank] = (unsigned char)lane;
      return;
    }
  }
  // the canonical sums, an expert per lane
  const int e = min(lane, E - 1);
  double acc = 0.0;
  for (int i0 = 0; i0 < dm; i0 += 16) {
    unsigned short xv[16], wv[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const unsigned i = min(i0 + j, dm - 1);
      xv[j] = xrow[i];
      wv[j] = w[i * (unsigned)HE + e];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const double next = fma(bf16_to_f64(xv[j]), bf16_to_f64(wv[j]), acc);
      acc = i0 + j < dm ? next : acc;
    }
  }
  wave_order();
  if (lane < E) z[lane] = acc + (bh ? (double)bh[lane] : 0.0);
  wave_order();
  if (lane == 0) select_serial(z, sel_out, E, k);
}

// VEC: bf16 elements of x per load (d_model a multiple of 8 or of 4).  S: K steps of a wave per trip (2: one trip, d_model at most 1024).  P: 8-byte pieces of a K step's
// router rows per lane (16 * H*E pieces).  CB: blocks of 16 logit columns.  WG: work-groups per CU.
template <int VEC, int S, int P, int CB, int WG>
__global__ __launch_bounds__(512, 2 * WG) void router_tile_kernel(RouterTileArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ int bt[32 * 8];            // binom_table
  __shared__ int cn[32], cns[384];      // counts of the tile's tokens per (head, expert) and per (head, set); H*E <= 32, at most 128 sets a head
  __shared__ unsigned char sidx[1024];  // [head][token][k] selected experts
  __shared__ float gd[RT_TOK * 32];     // [token][H*E] dense gates
  __shared__ unsigned short flist[1024];
  __shared__ float rsp[8][32], wsp[8][32], rs[32], w2[32];
  __shared__ double part[2][8][32];
  __shared__ int nflag;
  const int H = a.H, E = a.E, k = a.k, HE = H * E, dm = a.dm;
  int side, tile;
  if (a.xq) {   // two token sets: the tiles of one behind those of the other
    side = (int)blockIdx.x >= a.ncb[0];
    tile = (int)blockIdx.x - (side ? a.ncb[0] : 0);
  } else if (a.sides == 2) {   // both sides' tiles of the same tokens run on the same XCD (work-groups are dealt round-robin)
    side = ((int)blockIdx.x >> 3) & 1;
    tile = ((int)blockIdx.x >> 4) * 8 + ((int)blockIdx.x & 7);
  } else {
    side = 0;
    tile = blockIdx.x;
  }
  if (blockIdx.x == gridDim.x - 1) {   // one work-group more, for the table that no tile owns
    if (a.setid) write_set_experts(a.setexp, a.nsets, E, k);
    return;
  }
  if (tile >= a.ncb[side]) return;
  const int N = a.N[side], tok0 = tile * RT_TOK;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
  const bool own = side && a.xq;
  auto row_of = [&](int n) { return own ? (long)(n / a.Tq) * a.T + (a.T - a.Tq) + n % a.Tq : (long)n; };
  // a row past the end repeats the last one; nothing of it is kept
  const unsigned short* xp[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) xp[i] = a.x + row_of(min(tok0 + 16 * i + r, N - 1)) * dm;
  const unsigned short* W = a.W[side];
  const int total = dm * HE;

  const int ZS = HE | 1;   // row stride of the sums: odd, so that a column's rows lie in different banks
  // the wave's corner of LDS: its router rows of a K step, [column block][64][16], then its sums, [K step][32 tokens][ZS]
  const int corner = max(CB * 64 * 16 * 2, (S * 32 * ZS * 4 + 15) / 16 * 16);
  unsigned short* wl = (unsigned short*)(lds + wave * corner);
  float xs[2] = {0.f, 0.f}, ws[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) ws[c] = 0.f;
  double z[2] = {0.0, 0.0};   // the logits of token tid % 32, columns tid / 32 and 16 more
  // where a lane's pieces go: their first element's row and column
  const unsigned inv = div_magic(HE);
  int krc[P];   // row * 32 + column
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const int row = div_by(4 * (lane + 64 * i), inv);
    krc[i] = row * 32 + 4 * (lane + 64 * i) - row * HE;
  }
  // a K step's router rows into the wave's corner of LDS (the area is the wave's own, and a wave's LDS operations keep their order)
  auto stage = [&](unsigned short* dst, const uint2 (&v)[P]) {
    auto at = [&](int row, int c) { return dst + ((c >> 4) * 64 + row) * 16 + (c & 15); };
    wave_order();
    if (HE % 4 == 0) {
#pragma unroll
      for (int i = 0; i < P; ++i)
        if (lane + 64 * i < 16 * HE) *(uint2*)at(krc[i] >> 5, krc[i] & 31) = v[i];
    } else if (HE % 2 == 0) {
#pragma unroll
      for (int i = 0; i < P; ++i)
        if (lane + 64 * i < 16 * HE) {
          int at0 = krc[i];
          asm("" : "+v"(at0));   // (or the compiler computes this layout's addresses ahead of the loop in every layout)
          const int row = at0 >> 5, c = at0 & 31;
          const bool next = c + 2 >= HE;
          *(unsigned*)at(row, c) = v[i].x;
          *(unsigned*)at(row + next, c + 2 - (next ? HE : 0)) = v[i].y;
        }
    } else {
#pragma unroll
      for (int i = 0; i < P; ++i)
        if (lane + 64 * i < 16 * HE) {
          const unsigned short u[4] = {(unsigned short)v[i].x, (unsigned short)(v[i].x >> 16), (unsigned short)v[i].y, (unsigned short)(v[i].y >> 16)};
          int at0 = krc[i];
          asm("" : "+v"(at0));
          int row = at0 >> 5, c = at0 & 31;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            *at(row, c) = u[t];
            if (++c == HE) ++row, c = 0;
          }
        }
    }
    wave_order();
  };
  for (int kb = 0; kb < dm; kb += 512 * S) {
    uint2 wv[S][P], xa[S][2][2][2];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int k0 = kb + (s * 8 + wave) * 64;
#pragma unroll
      for (int i = 0; i < P; ++i) wv[s][i] = *(const uint2*)(W + min(k0 * HE + 4 * (lane + 64 * i), total - 4));
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int kk = k0 + 32 * j + 8 * g;
          if constexpr (VEC == 8) {
            const uint4 v = *(const uint4*)(xp[i] + min(kk, dm - 8));
            xa[s][i][j][0] = make_uint2(v.x, v.y);
            xa[s][i][j][1] = make_uint2(v.z, v.w);
          } else {
            xa[s][i][j][0] = *(const uint2*)(xp[i] + min(kk, dm - 4));
            xa[s][i][j][1] = *(const uint2*)(xp[i] + min(kk + 4, dm - 4));
          }
        }
    }
    if (kb == 0 && tid < 256) bt[tid] = (&binom_table.v[0][0])[tid];
    f32x4 sum[S][2][CB];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int k0 = kb + (s * 8 + wave) * 64;
      if (k0 + 64 > dm) {       // (uniform in the wave) what lies past the last feature counts as zero on both sides
#pragma unroll
        for (int i = 0; i < P; ++i)
          if (k0 * HE + 4 * (lane + 64 * i) >= total) wv[s][i] = make_uint2(0, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int kk = k0 + 32 * j + 8 * g;
            if (kk >= dm) xa[s][i][j][0] = make_uint2(0, 0);
            if (kk + 4 >= dm) xa[s][i][j][1] = make_uint2(0, 0);
          }
      }
      stage(wl, wv[s]);
      if (own) {   // the packed copy of the query tokens' rows
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int kk = k0 + 32 * j + 8 * g;
            unsigned short* q = a.xq + (long)(tok0 + 16 * i + r) * dm + kk;
            if (tok0 + 16 * i + r < N && kk < dm) *(uint2*)q = xa[s][i][j][0];
            if (tok0 + 16 * i + r < N && kk + 4 < dm) *(uint2*)(q + 4) = xa[s][i][j][1];
          }
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        // (columns past the last hold whatever LDS held: they only reach results that are never read)
        bf16x8 fb[CB], fa[2];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
          const unsigned short* p = wl + (c * 64 + 32 * j + 8 * g + (r >> 2)) * 16 + (r & 3) * 4;
          union {
            s16x4 h[2];
            bf16x8 v;
            uint4 w;
          } u;
          u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p));
          u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p + 4 * 16));
          fb[c] = u.v;
          ws[c] = sumsq2(u.w.x, sumsq2(u.w.y, sumsq2(u.w.z, sumsq2(u.w.w, ws[c]))));
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const uint2 lo = xa[s][i][j][0], hi = xa[s][i][j][1];
          xs[i] = sumsq2(lo.x, sumsq2(lo.y, sumsq2(hi.x, sumsq2(hi.y, xs[i]))));
          fa[i] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int c = 0; c < CB; ++c) {
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            const f32x4 m = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[c], zero, 0, 0, 0);
            sum[s][i][c] = j ? sum[s][i][c] + m : m;
          }
      }
    }
    wave_order();
    float* part = (float*)wl;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int c = 0; c < CB; ++c)
        if (16 * c + r < HE)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) part[(s * 32 + 16 * i + 4 * g + q) * ZS + 16 * c + r] = sum[s][i][c][q];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if ((tid >> 5) + 16 * u < HE) {
        const float* p = (const float*)lds + (tid & 31) * ZS + (tid >> 5) + 16 * u;
#pragma unroll
        for (int w = 0; w < 8; ++w)
#pragma unroll
          for (int s = 0; s < S; ++s) z[u] += (double)p[w * (corner / 4) + s * 32 * ZS];
      }
    if constexpr (S == 2) break;   // the host's promise: dm <= 1024 (a loop that the compiler sees costs 100 spilled registers)
    if (kb + 512 * S < dm) __syncthreads();
  }

#pragma unroll
  for (int i = 0; i < 2; ++i) {
    xs[i] += __shfl_xor(xs[i], 16, 64);
    xs[i] += __shfl_xor(xs[i], 32, 64);
    if (g == 0) rsp[wave][16 * i + r] = xs[i];
  }
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    ws[c] += __shfl_xor(ws[c], 16, 64);
    ws[c] += __shfl_xor(ws[c], 32, 64);
    if (g == 0) wsp[wave][16 * c + r] = ws[c];
  }
  if (tid < 32) cn[tid] = 0;
  if (tid == 0) nflag = 0;
  for (int t = tid; t < RT_TOK * HE; t += 512) gd[t] = 0.f;
  if (a.setid)
    for (int t = tid; t < H * a.nsets; t += 512) cns[t] = 0;
  __syncthreads();
  double* zp = (double*)lds;   // logits [32 tokens][ZS]
  const float* b = a.b[side];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int c = (tid >> 5) + 16 * u;
    if (c < HE) zp[(tid & 31) * ZS + c] = z[u] + (b ? (double)b[c] : 0.0);
  }
  if (tid < 32) {
    float v = rsp[0][tid];
#pragma unroll
    for (int w = 1; w < 8; ++w) v += rsp[w][tid];
    rs[tid] = v;
  } else if (tid >= 64 && tid < 64 + HE) {   // squared column norms
    float v = wsp[0][tid - 64];
#pragma unroll
    for (int w = 1; w < 8; ++w) v += wsp[w][tid - 64];
    w2[tid - 64] = v;
  }
  __syncthreads();

  // ---- first-stage selection, an item per (head, token) ----------------------------------
  const int items = RT_TOK * H;
  for (int it = tid; it < items; it += 512) {
    const int h = it / RT_TOK, t = it % RT_TOK;
    if (tok0 + t >= N) continue;
    const double* zi = zp + t * ZS + h * E;
    float wn = 0.f;   // largest squared column norm of the head
    for (int e = 0; e < E; ++e) {
      const float v = w2[h * E + e];
      wn = v > wn || v != v ? v : wn;   // (a NaN stays: nothing of that head counts as decided)
    }
    const double bound0 = 4.0 * 33 * 5.9604645e-8 * (double)(sqrtf(rs[t]) * 1.0001f) * (double)(sqrtf(wn) * 1.0001f);
    bool flag = false;
    if (E <= 8) {
      // every pair in registers; decided: no other logit close to a selected one, and every logit finite (with a NaN the pairs are no
      // order: 1, NaN, 2 gives every expert rank 1, and nothing would be written for rank 0)
      double v[8];
      int rank[8], near[8];
      double top = 0.0, finite = 0.0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] = zi[min(e, E - 1)];
        top = fmax(top, fabs(v[e]));
        finite = fma(v[e], 0.0, finite);   // stays 0, or a NaN from the first infinity or NaN on
        rank[e] = near[e] = 0;
      }
      flag = finite != 0.0;   // (the second stage writes every place)
      const double gap = 2.0 * (bound0 + 1e-13 * (top + 1.0));
#pragma unroll
      for (int e = 1; e < 8; ++e)
        if (e < E) {
#pragma unroll
          for (int f = 0; f < e; ++f) {
            const double d = v[e] - v[f];
            const int c = !(fabs(d) > gap), later = d > 0.0;
            rank[f] += later;
            rank[e] += 1 - later;
            near[e] |= c;
            near[f] |= c;
          }
        }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (e < E && rank[e] < k) {
          sidx[it * k + rank[e]] = (unsigned char)e;
          flag = flag || near[e];
        }
    } else {
      unsigned sel = 0;
      double prev = 0.0, bprev = 0.0;
      const int passes = k < E ? k + 1 : k;
      for (int j = 0; j < passes; ++j) {
        int best = -1;
        double bv = 0.0;
        for (int e = 0; e < E; ++e) {
          if ((sel >> e) & 1u) continue;
          const double v = zi[e];
          if (best < 0 || v > bv) {
            best = e;
            bv = v;
          }
        }
        const double bb = bound0 + 1e-13 * (fabs(bv) + 1.0);
        if (j > 0 && !(prev - bv > bprev + bb)) flag = true;
        prev = bv;
        bprev = bb;
        sel |= 1u << best;
        if (j < k) sidx[it * k + j] = (unsigned char)best;
      }
    }
    if (flag) flist[atomicAdd(&nflag, 1)] = (unsigned short)it;
  }
  __syncthreads();
  const int nf = nflag;
  if (nf) {
    // Second stage: the waves share an entry's K steps, the next wave in turn adds up their parts and selects while the others
    // go on (two sets of parts, one barrier each).  A lane takes one of 8, 16 or 32 columns and every 8th, 4th or 2nd row, so the router's
    // rows are staged once, however many experts there are.  (A lane per row with eight columns at a time, staged again for every eight: router
    // and sorts, us, 16384 tokens of d_model 1024, 3 heads, 4 of 10 experts 121 -> 80, 1 head, 2 of 31 143 -> 82; 298 tokens of d_model 2048, 8 of 31 273 -> 117.)
    unsigned short* w2l = (unsigned short*)(zp + (32 * ZS + 1) / 2 * 2) + wave * (CB * 64 * 16);   // behind the logits
    const int cbits = E <= 8 ? 3 : E <= 16 ? 4 : 5, nr = 1 << cbits, step = 64 >> cbits, r0 = lane >> cbits;
    int buf = 0;
    for (int f = 0; f < nf; ++f, buf ^= 1) {
      const int it = flist[f], h = it / RT_TOK, t = it % RT_TOK;
      const unsigned short* xrow = a.x + row_of(tok0 + t) * dm;
      double* zi = zp + t * ZS + h * E;
      const int c = h * E + min(lane & (nr - 1), E - 1);
      const unsigned short* wc = w2l + ((c >> 4) * 64 + r0) * 16 + (c & 15);
      double acc = 0.0;
      for (int kb = wave * 64; kb < dm; kb += 1024) {
        uint2 wv[2][P];
        unsigned short xv[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const int k0 = kb + 512 * s;
#pragma unroll
          for (int i = 0; i < P; ++i) wv[s][i] = *(const uint2*)(W + min(k0 * HE + 4 * (lane + 64 * i), total - 4));
          xv[s] = xrow[min(k0 + lane, dm - 1)];
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const int rows = dm - (kb + 512 * s);
          if (rows <= 0) break;   // uniform
          stage(w2l, wv[s]);
          for (int j0 = 0; j0 < nr; j0 += 8) {   // rows r0, r0 + step, ...
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int row = (j0 + j) * step;
              const double next = fma(bf16_to_f64((unsigned short)__shfl((int)xv[s], r0 + row, 64)), bf16_to_f64(wc[row * 16]), acc);
              acc = r0 + row < rows ? next : acc;
            }
          }
        }
      }
      // the same tree over the row groups for every column
      for (int o = 32; o >= nr; o >>= 1) acc += __shfl_xor(acc, o, 64);
      if (lane < E) part[buf][wave][lane] = acc;
      __syncthreads();
      if (wave == f % 8) {
        if (lane < E) {
          double v = part[buf][0][lane];
#pragma unroll
          for (int w = 1; w < 8; ++w) v += part[buf][w][lane];
          zi[lane] = v + (b ? (double)b[h * E + lane] : 0.0);
        }
        wave_order();
        // twice d_model * 2^-53 * |x| * max|w|, doubled again for the rounding of the norms themselves
        float wn = 0.f;
        for (int e = 0; e < E; ++e) wn = fmaxf(wn, w2[h * E + e]);
        const double reorder = 4.0 * (double)dm * 1.1102230246251565e-16 * (double)sqrtf(rs[t]) * (double)sqrtf(wn);
        recheck_select(xrow, W + h * E, b ? b + h * E : nullptr, zi, sidx + it * k, dm, HE, E, k, lane, reorder);
      }
    }
    __syncthreads();
  }

  // ---- gates, tables, counts ---------------------------------------------------------------
  const long out0 = (long)side * H * a.N[0];
  for (int u = tid; u < items * k; u += 512) {
    const int it = u / k, h = it / RT_TOK, t = it % RT_TOK;
    if (tok0 + t >= N) continue;
    const int c = h * E + sidx[u];
    const float gv = (float)(1.0 / (1.0 + exp(-zp[t * ZS + c])));
    gd[t * HE + c] = gv;
    const long o = (out0 + (long)h * N + tok0) * k + (u - h * RT_TOK * k);
    a.idx[o] = c - h * E;
    a.gate[o] = gv;
    atomicAdd(&cn[c], 1);
  }
  __syncthreads();
  if (a.setid) {
    for (int it = tid; it < items; it += 512) {
      const int h = it / RT_TOK, t = it % RT_TOK;
      if (tok0 + t >= N) continue;
      unsigned sel = 0;
      for (int j = 0; j < k; ++j) sel |= 1u << sidx[it * k + j];
      const long o = out0 + (long)h * N + tok0 + t;
      int sid = 0;
      for (int p = 0; p < k; ++p) {   // ascending experts
        const int e = __builtin_ctz(sel);
        sel &= sel - 1;
        sid += bt[e * 8 + p];
        a.gset[o * k + p] = gd[t * HE + h * E + e];
      }
      a.setid[o] = sid;
      atomicAdd(&cns[h * a.nsets + sid], 1);
    }
    __syncthreads();
    for (int c = tid; c < H * a.nsets; c += 512) a.setcnt[(long)side * H * a.nsets * a.ncb[0] + (long)c * a.ncb[side] + tile] = cns[c];
  }
  // (side 1's counts start where they would with N[0] tokens)
  for (int c = tid; c < HE; c += 512) a.cnt[(long)side * HE * a.ncb[0] + (long)c * a.ncb[side] + tile] = cn[c];
  if (a.gtab) {
    float* out = a.gtab + ((long)side * a.N[0] + tok0) * HE;
    const int cnt = min(RT_TOK, N - tok0) * HE;
    for (int u = tid; u < cnt; u += 512) out[u] = gd[u];
  }
}

// Wp[side][i][c] = W_side[i][c] for c < HE, 0 for HE <= c < HEp (rows padded to 16 bytes)
__global__ void pack_router_kernel(const bf16_t* __restrict__ W0, const bf16_t* __restrict__ W1, bf16_t* __restrict__ Wp,
                                   int dm, int HE, int HEp, int sides) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  long tot = (long)sides * dm * HEp;
  if (i >= tot) return;
  int c = (int)(i % HEp);
  long r = i / HEp;
  int side = (int)(r / dm);
  long row = r % dm;
  const bf16_t* W = side ? W1 : W0;
  bf16_t v;
  v.v = 0;
  if (c < HE) v = W[row * HE + c];
  Wp[i] = v;
}

void launch_pack_router(const void* W0, const void* W1, void* Wp, int dm, int HE, int HEp, int sides, hipStream_t s) {
  const long tot = (long)sides * dm * HEp;
  pack_router_kernel<<<(unsigned)((tot + 255) / 256), 256, 0, s>>>((const bf16_t*)W0, (const bf16_t*)W1, (bf16_t*)Wp, dm, HE, HEp, sides);
}

// Dense gate table for the gated-concatenation GEMMs: gtab[side][n][h*E + e] = the gate of expert e of head h
// for token n if the token selected it (Sec. 2.2: e in E^h), else 0.  One thread per (side, head, token).
__global__ __launch_bounds__(256) void gate_table_kernel(const int* __restrict__ idx, const float* __restrict__ gate,
                                                         float* __restrict__ gtab, int N, int H, int E, int k, long side_stride_in,
                                                         long side_stride_out) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  const int h = blockIdx.y, side = blockIdx.z;
  if (n >= N) return;
  float* out = gtab + side * side_stride_out + ((long)n * H + h) * E;
  for (int e = 0; e < E; ++e) out[e] = 0.f;
  const long o = side * side_stride_in + ((long)h * N + n) * k;
  for (int j = 0; j < k; ++j) out[idx[o + j]] = gate[o + j];
}

void launch_gate_table(const int* idx, const float* gate, float* gtab, int N, int H, int E, int k, int sides, long side_stride_in,
                       hipStream_t s) {
  dim3 g((N + 255) / 256, H, sides);
  gate_table_kernel<<<g, 256, 0, s>>>(idx, gate, gtab, N, H, E, k, side_stride_in, (long)N * H * E);
}

bool router_hybrid_supported(const RouterArgs& a) {
  return a.bf16 && a.dm % 4 == 0 && ((uintptr_t)a.x % 16) == 0 && ((uintptr_t)a.W[0] % 8) == 0 && ((uintptr_t)a.W[1] % 8) == 0 && a.H * a.E <= 32 &&
         (long)a.dm * a.H * a.E < (1l << 30);
}

template <typename T>
static void launch_router_select(const RouterArgs& a, hipStream_t s) {
  const int hpb = 64 / a.E < a.H ? 64 / a.E : a.H;   // whole heads per work-group
  const int ncb = router_count_blocks(a.N), cpt = (hpb * a.E + 7) / 8;
  const dim3 g(ncb, a.sides, (a.H + hpb - 1) / hpb);
  auto kern = cpt <= 1 ? router_select_kernel<T, 1> : cpt <= 2 ? router_select_kernel<T, 2> : cpt <= 4 ? router_select_kernel<T, 4> : router_select_kernel<T, 8>;
  kern<<<g, 256, 0, s>>>((const T*)a.x, (const T*)a.W[0], (const T*)a.W[1], a.b[0], a.b[1], a.idx, a.gate, a.blockcnt, a.N, a.dm,
                         a.H, a.E, a.k, hpb, ncb);
}

// ----------------------------------------------------------------------------------------
// Expert-SET sorting.  A token's k experts of one head form one of C(E,k) sets; tokens that
// share a set share all k weight matrices, so the k gate-weighted products of Sec. 2.2's
// output equation can be summed inside one matrix-core accumulator.  Set id = rank of the
// ascending combination (combinatorial number system), tokens are counting-sorted by it.
// ----------------------------------------------------------------------------------------
// Set ids, gates in ascending-expert order and counts from the top-k tables (routers other than the two-stage one, which
// writes them itself)
__global__ __launch_bounds__(RB) void set_hist_kernel(const int* __restrict__ idx, const float* __restrict__ gate,
                                                      int* __restrict__ setid, float* __restrict__ gset,
                                                      int* __restrict__ setexp, int* __restrict__ blockcnt, int N, int k,
                                                      int E, int nsets, int nblk) {
  __shared__ int cnt[128];
  const int sh_ = blockIdx.y;
  const int n = blockIdx.x * RB + threadIdx.x;
  const bool valid = n < N;
  if (threadIdx.x < 128) cnt[threadIdx.x] = 0;
  if (blockIdx.x == 0 && blockIdx.y == 0) write_set_experts(setexp, nsets, E, k);
  __syncthreads();
  if (valid) {
    int e[8];
    float g[8];
    const long o = ((long)sh_ * N + n) * k;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      e[j] = j < k ? idx[o + j] : 0x7fffffff;
      g[j] = j < k ? gate[o + j] : 0.f;
    }
    // ascending experts (k <= 8: odd-even transposition sort with static indexing)
#pragma unroll
    for (int pass = 0; pass < 8; ++pass)
#pragma unroll
      for (int j = pass & 1; j + 1 < 8; j += 2)
        if (e[j] > e[j + 1]) {
          int te = e[j];
          e[j] = e[j + 1];
          e[j + 1] = te;
          float tg = g[j];
          g[j] = g[j + 1];
          g[j + 1] = tg;
        }
    int sid = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j < k) {
        sid += binom(e[j], j + 1);
        gset[o + j] = g[j];
      }
    setid[(long)sh_ * N + n] = sid;
    atomicAdd(&cnt[sid], 1);
  }
  __syncthreads();
  if (threadIdx.x < nsets) blockcnt[((long)sh_ * nsets + threadIdx.x) * nblk + blockIdx.x] = cnt[threadIdx.x];
}

// The sorts of up to two sides (with tokens of their own or the same ones) from the tables and counts the routers leave: side s's
// tables start where they would if side 0 had N[0] tokens before them.  The expert sort and the set sort of a side have blocks of their own.
struct SortArgs {
  const int* idx;
  int *cnt, *perm, *offsets;   // cnt: [side][H][E][ncb]
  SetSortArgs t;               // t.setid NULL: no set tables; t.blockcnt: [side][H][nsets][ncb]
  int N[2], ncb[2], H, E, k, sides;
  int per;                     // count blocks per block of RB tokens
  int experts;                 // 0: the sets alone
};
// LOCAL: the block finds its first positions from the raw counts, else from their sums (scan_kernel).  Everything a block reads is requested before it
// waits: one trip to memory.
template <bool LOCAL>
__device__ __forceinline__ void sort_body(const SortArgs& a) {
  __shared__ int sb[2 * 128];
  __shared__ int wcnt[RB / 64][128];
  const int side = blockIdx.z % a.sides, sets = (int)blockIdx.z >= a.sides || !a.experts;
  const int h = blockIdx.y, N = a.N[side], ncb = a.ncb[side], first = blockIdx.x * a.per, k = a.k;
  if (first >= ncb) return;
  const long at = (long)side * a.H * a.N[0] + (long)h * N, sh_ = side * a.H + h;
  const int nbins = sets ? a.t.nsets : a.E;
  const int* c = (sets ? a.t.blockcnt : a.cnt) + ((long)side * a.H * a.ncb[0] + (long)h * ncb) * nbins;
  int* offsets = sets ? a.t.setoff + sh_ * (nbins + 1) : a.offsets + sh_ * (nbins + 1);
  const int n = blockIdx.x * RB + threadIdx.x, nc = min(n, N - 1);
  const bool valid = n < N;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long lt = (1ull << lane) - 1ull;
  if (sets) {
    const int sid = a.t.setid[at + nc];
    float gv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) gv[j] = a.t.gset[(at + nc) * k + min(j, k - 1)];
    for (int t = threadIdx.x; t < RB / 64 * 128; t += RB) (&wcnt[0][0])[t] = 0;
    LOCAL ? block_bases(c, offsets, nbins, ncb, a.per, sb) : stored_bases(c, offsets, nbins, ncb, a.per, sb);
    // the rank among the wave's tokens of the same set: the lanes whose set id agrees with one's own in every bit
    unsigned long long same = __ballot(valid);
    for (int bit = 0; (1 << bit) < nbins; ++bit) {
      const unsigned long long bal = __ballot((sid >> bit) & 1);
      same &= (sid >> bit) & 1 ? bal : ~bal;
    }
    const int rk = __popcll(same & lt);
    if (valid && rk == 0) wcnt[wave][sid] = __popcll(same);
    wave_bases(wcnt, sb, nbins);
    if (!valid) return;
    const int pos = rk + wcnt[wave][sid];
    a.t.setperm[at + pos] = n;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j < k) a.t.gsort[(at + pos) * k + j] = gv[j];
    return;
  }
  int ej[8], rk[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) ej[j] = a.idx[(at + nc) * k + min(j, k - 1)];
  LOCAL ? block_bases(c, offsets, nbins, ncb, a.per, sb) : stored_bases(c, offsets, nbins, ncb, a.per, sb);
  unsigned long long sel = 0ull;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (!valid || j >= k) ej[j] = -1;
    rk[j] = 0;
    if (ej[j] >= 0) sel |= 1ull << ej[j];
  }
  for (int e = 0; e < nbins; ++e) {
    const unsigned long long bal = __ballot((sel >> e) & 1ull);
    const int r = __popcll(bal & lt);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (ej[j] == e) rk[j] = r;
    if (lane == 0) wcnt[wave][e] = __popcll(bal);
  }
  wave_bases(wcnt, sb, nbins);
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (ej[j] >= 0) a.perm[at * k + rk[j] + wcnt[wave][ej[j]]] = n * k + j;
}
__global__ __launch_bounds__(RB) void scan_scatter_kernel(SortArgs a) { sort_body<true>(a); }
__global__ __launch_bounds__(RB) void scatter_kernel(SortArgs a) { sort_body<false>(a); }
// Running sums of the counts of a bin, a wave per bin of either table: the count of every block becomes the sum of those before it.  The first place,
// where that is 0, takes the sum of all.
// (A work-group per (side, head) and table for all of its bins, 64 counts a step: router and sorts of 3 x 126 sets, 16384 tokens 245 -> 81 us, 104000
// 1361 -> 333; 3 x 70 sets, 32768 tokens 261 -> 77; fp32, 64 experts, 65536 tokens 483 -> 161.)
__global__ __launch_bounds__(256) void scan_kernel(SortArgs a) {
  const int side = blockIdx.y, h = blockIdx.x, ncb = a.ncb[side], lane = threadIdx.x & 63;
  const int bin = blockIdx.z * 4 + (threadIdx.x >> 6), ne = a.experts ? a.E : 0;
  if (bin >= ne + a.t.nsets) return;
  const long at = (long)side * a.H * a.ncb[0] + (long)h * ncb;
  int* c = bin < ne ? a.cnt + at * a.E + (long)bin * ncb : a.t.blockcnt + at * a.t.nsets + (long)(bin - ne) * ncb;
  int run = 0;
  for (int b0 = 0; b0 < ncb; b0 += 64 * 16) {
    const int b = b0 + lane * 16;
    int v[16], sum = 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = c[min(b + u, ncb - 1)];
#pragma unroll
    for (int u = 0; u < 16; ++u) sum += b + u < ncb ? v[u] : 0;
    int inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o, 64);
      if (lane >= o) inc += t;
    }
    int pre = run + inc - sum;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if (b + u < ncb && b + u > 0) c[b + u] = pre;
      pre += v[u];
    }
    run += __shfl(inc, 63, 64);
  }
  if (lane == 0) c[0] = run;
}

// Short tables are scanned by every scatter block for itself, one launch instead of two.  A block takes a trip to memory for 256 counts of
// 16 bins, one after the other, and all blocks' trips share the caches: both sums have a line.  Router and sorts, us, by every block / scanned first: bf16,
// 16 to 64 features, two sides, 2 sets, one head, 49152 tokens (6 trips, 768 blocks) 41.7 / 44.2, 65536 (8, 1024) 53.4 / 53.7, 131072 107 / 94; 3 heads, 24576
// (3, 1152) 29.4 / 30.8, 32768 (4, 1536) 37.8 / 36.8, 131072 172 / 103; 3 x 10 sets, 24576 39.4 / 40.0, 32768 47.0 / 45.8; 3 x 28 sets, 16384 (4, 768)
// 34.1 / 35.4, 24576 (6, 1152) 47.9 / 46.6; 70 sets, 8192 (5, 128) 24.0 / 24.8, 12288 (10, 192) 27.8 / 26.0; 126 sets, 2048 (8, 32)
// 28.2 / 26.6; fp32, 2 x 16 experts, 49152 (6, 768) 46.0 / 49.0, 65536 (8, 1024) 59.1 / 59.6; 2 x 64, 8192 (4, 128) 65.6 / 66.2, 16384 (8, 256) 90.4 / 90.7.
static void launch_sort(const SortArgs& a, hipStream_t s) {
  const int nmax = a.sides > 1 && a.N[1] > a.N[0] ? a.N[1] : a.N[0];
  const int tables = (a.experts ? 1 : 0) + (a.t.setid ? 1 : 0);
  const dim3 g(router_blocks(nmax), a.H, a.sides * tables);
  const long bins = a.t.setid && a.t.nsets > a.E ? a.t.nsets : a.E;
  const int ncb = a.sides > 1 && a.ncb[1] > a.ncb[0] ? a.ncb[1] : a.ncb[0];
  const long trips = (bins + 15) / 16 * ((ncb + 255) / 256), blocks = (long)g.x * g.y * g.z;
  if (trips <= 7 && trips * blocks <= 5500) {
    scan_scatter_kernel<<<g, RB, 0, s>>>(a);
    return;
  }
  scan_kernel<<<dim3(a.H, a.sides, ((a.experts ? a.E : 0) + a.t.nsets + 3) / 4), 256, 0, s>>>(a);
  scatter_kernel<<<g, RB, 0, s>>>(a);
}

static SortArgs sort_args(const RouterArgs& a) {
  SortArgs d{};
  d.idx = a.idx;
  d.cnt = a.blockcnt;
  d.perm = a.perm;
  d.offsets = a.offsets;
  d.N[0] = a.N;
  d.N[1] = a.Nq > 0 ? a.Nq : a.N;
  for (int i = 0; i < 2; ++i) d.ncb[i] = router_count_blocks(d.N[i]);
  d.H = a.H;
  d.E = a.E;
  d.k = a.k;
  d.sides = a.sides;
  d.per = RB / RT_TOK;
  d.experts = 1;
  return d;
}

void launch_router(const RouterArgs& a, hipStream_t s) {
  if (a.bf16)
    launch_router_select<bf16_t>(a, s);
  else
    launch_router_select<float>(a, s);
  launch_sort(sort_args(a), s);
}

void launch_set_sort(const SetSortArgs& a, hipStream_t s) {
  const int nblk = router_blocks(a.N);
  dim3 g(nblk, a.sides * a.H);
  set_hist_kernel<<<g, RB, 0, s>>>(a.idx, a.gate, a.setid, a.gset, a.setexp, a.blockcnt, a.N, a.k, a.E, a.nsets, nblk);
  SortArgs d{};
  d.t = a;
  d.N[0] = d.N[1] = a.N;
  d.ncb[0] = d.ncb[1] = nblk;
  d.H = a.H;
  d.E = a.E;
  d.k = a.k;
  d.sides = a.sides;
  d.per = 1;
  launch_sort(d, s);
}

void launch_dense_routing(int* idx, float* gate, int* perm, int* offsets, int n0, int n1, int H, const SetSortArgs* t, hipStream_t s) {
  const long tot = (long)H * (n0 > n1 ? n0 : n1);
  dense_routing_kernel<<<dim3((unsigned)((tot + 255) / 256), 2), 256, 0, s>>>(idx, gate, perm, offsets, n0, n1, H, t ? t->setperm : nullptr,
                                                                              t ? t->gsort : nullptr, t ? t->setoff : nullptr, t ? t->setexp : nullptr);
}

template <int VEC, int S, int P, int CB>
static void launch_router_tiles(const RouterTileArgs& t, int blocks, hipStream_t s) {
  const size_t ZS = (t.H * t.E) | 1, wl = CB * 64 * 16 * 2, sums = (S * 32 * ZS * 4 + 15) / 16 * 16;
  const size_t first = 8 * (wl > sums ? wl : sums), second = (32 * ZS + 1) / 2 * 2 * 8 + 8 * wl;   // (the logits, then the second stage's router rows)
  const size_t lds = first > second ? first : second;   // at most 43008 bytes (20 columns, two steps), with the static part below 64 KB
  if constexpr (S == 1 && CB == 1) {
    // More than two tiles for each CU: three at a time, in 80 registers (six or seven spilled).  Forward calls, us, two / three: d_model 64, 2 x 2
    // columns, 8192 tokens (512 tiles) 44.3 / 44.4, 10240 49.5 / 47.4, 32768 63.9 / 59.8; d_model 412, 2 x 10 columns, 8192 78.4 /
    // 78.6, 10240 89.6 / 85.8, 16384 112.4 / 109.9, 32768 177.4 / 170.4.  Two steps a trip lose: d_model 1024, 2 x 10 columns, 32768 277 / 281.
    if (blocks > 512) {
      router_tile_kernel<VEC, S, P, CB, 3><<<blocks + 1, 512, lds, s>>>(t);
      return;
    }
  }
  router_tile_kernel<VEC, S, P, CB, 2><<<blocks + 1, 512, lds, s>>>(t);
}
template <int VEC, int S>
static void launch_router_tiles(const RouterTileArgs& t, int blocks, hipStream_t s) {
  const int HE = t.H * t.E;
  if (HE <= 12) return launch_router_tiles<VEC, S, 3, 1>(t, blocks, s);
  if (HE <= 16) return launch_router_tiles<VEC, S, 4, 1>(t, blocks, s);
  if (HE <= 20) return launch_router_tiles<VEC, S, 5, 2>(t, blocks, s);
  launch_router_tiles<VEC, 1, 8, 2>(t, blocks, s);   // (two would need the LDS of two work-groups)
}

void launch_router_hybrid(const RouterArgs& a, hipStream_t s) {
  RouterTileArgs t{};
  t.x = (const unsigned short*)a.x;
  SortArgs d = sort_args(a);
  for (int i = 0; i < 2; ++i) {
    t.W[i] = (const unsigned short*)a.W[a.shared ? 0 : i];
    t.b[i] = a.b[i];
    t.N[i] = d.N[i];
    t.ncb[i] = d.ncb[i];
  }
  t.idx = a.idx;
  t.gate = a.gate;
  t.cnt = a.blockcnt;
  t.gtab = a.gtab;
  if (a.sets) {
    d.t = *a.sets;
    t.setid = a.sets->setid;
    t.gset = a.sets->gset;
    t.setexp = a.sets->setexp;
    t.setcnt = a.sets->blockcnt;
    t.nsets = a.sets->nsets;
  }
  t.sides = a.sides;
  t.dm = a.dm;
  t.H = a.H;
  t.E = a.E;
  t.k = a.k;
  if (a.Nq > 0) {
    t.xq = (unsigned short*)a.xq;
    t.T = a.T;
    t.Tq = a.Tq;
  }
  const int blocks = a.Nq > 0 ? t.ncb[0] + t.ncb[1] : a.sides == 2 ? (t.ncb[0] + 7) / 8 * 16 : t.ncb[0];
  const bool two = a.dm > 512 && a.dm <= 1024;
  if (a.dm % 8 == 0)
    two ? launch_router_tiles<8, 2>(t, blocks, s) : launch_router_tiles<8, 1>(t, blocks, s);
  else
    two ? launch_router_tiles<4, 2>(t, blocks, s) : launch_router_tiles<4, 1>(t, blocks, s);
  launch_sort(d, s);
}

}  // namespace sh
