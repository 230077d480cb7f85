// Every weight gradient of a backward pass in one launch (arXiv 2312.07987, Sec. 2.1 - 2.2, chain rule): output and value
// experts, queries and keys (dense or experts), routers.  dW_g[i, j] = sum over the rows of group g of g * A[row, i] * B[row, j]
// on v_mfma_f32_32x32x16_bf16, output tiles of 128 x 256 or 256 x 128 features with two work-groups per CU, both operands
// staged [row][feature] and read with transposing LDS loads.
//
// The work is a list of items (problem, output tile, group), each of ceil(group rows / 64) units.  An item is cut into equal parts of
// at most L units, one work-group each; L is chosen by every wave from the group sizes on the device, as a rule the smallest length
// for which the parts of all items fit onto the chip at once (512 work-groups), so that a skewed routing is balanced like an even one.
// The parts leave partial tiles that wgrad_list_reduce_kernel adds in part order (a fixed order: the gradients are bit-reproducible).
//
// Why one launch: launched one by one (chunks of <= 2048 rows, about 480 work-groups each) every launch had its own prologue
// (offsets -> row ids -> gates -> first tiles, four dependent trips to memory that all work-groups make together), its own
// ragged last round and its own partial sums and reduction.
// Why this order (problem, output tile, part, group): work-groups of one XCD then walk the same columns of the same tokens side
// by side, for different experts and heads, and meet in its L2.  Equal shares of the unit list that start anywhere inside
// an item (no rounding up to whole parts, at most one cut per share) lose that: 255 us against 176 at B = 32, T = 512,
// d_model 1024, 4 heads of 128, E = 5, k = 3, where 1.7 GB of operand tiles then come from beyond the L2.  Three launches and three
// reductions of that shape took 73 + 72 + 54 + 46 us; this launch and its reduction take 176 + 21 (events around each).
#include "common.h"
#include "mfma_util.h"

namespace sh {

namespace {

constexpr int WL_UNIT = 64;        // rows per unit (two K steps)
constexpr int WL_SLOT = 256 * 128; // floats of a partial tile, in register order
constexpr int WL_MIN_PART = 2;     // units
constexpr int WL_BLOCKS = 512;     // two work-groups on each of 256 CUs
constexpr int WL_PLAN = 64;        // floats in front of the slots: the cut, for the reduction
constexpr int WL_OVERHEAD = 10;    // what a part costs beside its units
// Where the items alone nearly fill the chip, a second round of half-sized parts is better than a few work-groups in one.
__host__ __device__ constexpr int max_parts(int items) { return items > WL_BLOCKS * 7 / 8 ? items + 2 * WL_BLOCKS : WL_BLOCKS; }
constexpr int WL_SUB = 2048;       // rows whose ids and gates LDS holds at a time

template <int WM_, int WN_, int MI_, int NJ_>
struct WlCfg {
  static constexpr int WM = WM_, WN = WN_, MI = MI_, NJ = NJ_, BK = 32;
  static constexpr int BM = WM * MI * 32, BN = WN * NJ * 32;
  static constexpr int LDA = BM + 32, LDB = BN + 32;   // row strides 16 banks (mod 64) apart
  static constexpr int STAGE_ELEMS = BK * (LDA + LDB);
  static constexpr int ROW_CAP = WL_SUB + 4 * BK;      // the row tables reach past the rows as far as the prefetch does
  static constexpr size_t lds_bytes() { return (size_t)2 * STAGE_ELEMS * 2 + (size_t)ROW_CAP * 8; }
};
typedef WlCfg<1, 4, 4, 2> WlWide;   // 128 x 256, wave tile 128 x 64
typedef WlCfg<4, 1, 2, 4> WlTall;   // 256 x 128, wave tile 64 x 128
static_assert(WlWide::BM * WlWide::BN == WL_SLOT && WlTall::BM * WlTall::BN == WL_SLOT && WlWide::lds_bytes() == WlTall::lds_bytes(), "one slot size");

// How the items are cut, derived by every wave (lane g holds group g of every problem).
struct WlMap {
  int gu[WGRAD_LIST_MAX];      // units of the lane's group
  int first[WGRAD_LIST_MAX];   // first row of the lane's group in the sorted order
  int rows[WGRAD_LIST_MAX];
  int tot[WGRAD_LIST_MAX];     // parts of all groups, per output tile (uniform)
  int total;                   // parts in all
  int len;                     // L: units of the longest part allowed
};

__device__ __forceinline__ int parts_of(int units, int len) { return (units + len - 1) / len; }

__device__ __forceinline__ int wave_scan(int v, int lane) {   // inclusive
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  return v;
}

// first row and row count of the lane's group
__device__ __forceinline__ void group_rows(const WgradItem& a, int lane, int& first, int& rows) {
  const int grp = min(lane, a.heads * a.E - 1);
  first = 0;
  rows = a.M;
  if (a.perm) {
    const int* off = a.offsets + (long)(grp / a.E) * (a.E + 1) + grp % a.E;
    first = off[0];
    rows = off[1] - first;
  }
  if (lane != grp) rows = 0;
}

__device__ __forceinline__ void make_map(const WgradList& l, int lane, WlMap& m) {
#pragma unroll
  for (int p = 0; p < WGRAD_LIST_MAX; ++p) {
    m.first[p] = m.rows[p] = 0;
    if (p < l.n) group_rows(l.p[p], lane, m.first[p], m.rows[p]);
  }
  int all = 0;
#pragma unroll
  for (int p = 0; p < WGRAD_LIST_MAX; ++p) {
    m.gu[p] = (m.rows[p] + WL_UNIT - 1) / WL_UNIT;
    if (p < l.n) all += m.gu[p] * l.p[p].ntile;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) all += __shfl_xor(all, d, 64);
  // Lane j tries a length: 0.2 .. 0.95 of an even share L0 (several rounds), then L0 .. 3 L0 in steps of about 4 %.  Estimated time
  // in units: one round takes its longest part, several take the mean load and half a part of raggedness at the end; WL_OVERHEAD
  // is a part's prologue and partial sum.
  const int cap = max_parts(l.items);
  const int len0 = max(WL_MIN_PART, (all + WL_BLOCKS - 1) / WL_BLOCKS);
  const int len = lane < 16 ? max(WL_MIN_PART, (len0 * (lane + 4)) / 20) : len0 + (lane - 16) * (len0 / 24 + 1);
  const unsigned inv = div_magic(len);
  int tot[WGRAD_LIST_MAX], sum = 0;
#pragma unroll
  for (int p = 0; p < WGRAD_LIST_MAX; ++p) {
    tot[p] = 0;
    if (p < l.n) {
      const WgradItem& a = l.p[p];
      const int G = a.heads * a.E, n = a.perm ? G : 1;   // (without a permutation all groups are alike)
      for (int i = 0; i < n; ++i) tot[p] += div_by(__builtin_amdgcn_readlane(m.gu[p], i) + len - 1, inv);
      if (!a.perm) tot[p] *= G;
      sum += tot[p] * a.ntile;
    }
  }
  float cost = sum <= WL_BLOCKS ? (float)(len + WL_OVERHEAD)
                                : (float)(all + sum * WL_OVERHEAD) * (1.f / WL_BLOCKS) + 0.5f * (float)(len + WL_OVERHEAD);
  if (sum > cap) cost = 3e38f;
  float best = cost;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) best = fminf(best, __shfl_xor(best, d, 64));
  const bool fit = __ballot(cost < 3e38f) != 0;   // else nothing is cut.  (A ballot: the compiler has to see that all of this is uniform)
  const int pick = __builtin_ctzll(__ballot(cost == best));
  m.len = fit ? __builtin_amdgcn_readlane(len, pick) : 1 << 29;
  m.total = 0;
#pragma unroll
  for (int p = 0; p < WGRAD_LIST_MAX; ++p) {
    m.tot[p] = fit ? __builtin_amdgcn_readlane(tot[p], pick) : __popcll(__ballot(m.gu[p] > 0));
    if (p < l.n) m.total += m.tot[p] * l.p[p].ntile;
  }
}

__device__ __forceinline__ void store_dw(const WgradItem& a, int h, int e, int i, int j, float v) {
  float* out = a.dW;
  if (a.col_split > 0 && j >= a.col_split) {   // the right-hand block of columns has its own output
    j -= a.col_split;
    out = a.dW2;
  }
  if (i < a.Ka && j < a.kb_store && out) out[(long)h * a.w_hstride + (long)e * a.w_estride + (long)i * a.swa + j] = v;
}

// One part: `nrows` rows from sorted position row0 on of group (h, e), output tile at (i0, j0).  GATE: 0 none, 1 on the rows of A,
// 2 on the rows of B (the narrower side of the tile).  The sum goes to a slot in register order.
// What bounds the loop: a step of 32 rows is 16 MFMAs per wave (512 cycles of the matrix pipe) beside 48 KB of fragment reads and
// 24 KB of stores per work-group on the LDS pipe (1150 cycles for the CU's two work-groups against 1024 of MFMA).
// Rows past the part repeat its last row and are zeroed on their way into LDS, so no load carries a condition and the wait
// before a step is staged names exactly that step's loads; feature pieces past Ka / Kb repeat the last piece and only reach
// output elements that are never stored.
// HALF: rows of 8 but not 16 bytes in pieces of 16 bytes, half the loads, row lookups and stores of pieces of 8; the last piece of a row is
// read 8 bytes early and moved into place on its way into LDS.  All gradients of 4 heads of 100, d_model 1024, us: 1000 tokens 28.9 ->
// 27.6, 4000 54.0 -> 50.4, 24000 255 -> 211; 2 heads of 76, d_model 412, 16000 tokens 57.7 -> 53.6.  (Operands 4 wide keep pieces of 8.)
template <class Cfg, int VEC, int GATE, bool HALF>
__device__ __forceinline__ void wgrad_part(const WgradItem& a, int h, int e, int row0, int nrows, int i0, int j0, float4* slot,
                                            unsigned short* smem) {
  constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = Cfg::BK, MI = Cfg::MI, NJ = Cfg::NJ;
  constexpr int LDA = Cfg::LDA, LDB = Cfg::LDB;
  typedef typename Chunk<VEC>::type chunk_t;
  int* ids = (int*)(smem + 2 * Cfg::STAGE_ELEMS);
  float* gsc = (float*)(ids + Cfg::ROW_CAP);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int A_CPR = BM / VEC, B_CPR = BN / VEC;
  constexpr int A_N = BK * A_CPR / 256, B_N = BK * B_CPR / 256;
  // two register sets: a step's rows are requested two steps before they are multiplied
  chunk_t ra0[A_N], rb0[B_N], ra1[A_N], rb1[B_N];
  const char* Ab = (const char*)((const unsigned short*)a.A + (long)h * a.a_hoff);
  const char* Bb = (const char*)((const unsigned short*)a.B + (long)h * a.b_hoff);
  const unsigned lda2 = (unsigned)a.lda * 2, ldb2 = (unsigned)a.ldb * 2;
  const unsigned col_a2 = (unsigned)min(i0 + (tid % A_CPR) * VEC, a.Ka - VEC) * 2;
  const unsigned col_b2 = (unsigned)min(j0 + (tid % B_CPR) * VEC, a.Kb - VEC) * 2;
  const bool half_a = HALF && i0 + (tid % A_CPR) * VEC + 8 > a.Ka, half_b = HALF && j0 + (tid % B_CPR) * VEC + 8 > a.Kb;
  auto load_global = [&](chunk_t (&ra)[A_N], chunk_t (&rb)[B_N], int r0) {
    const int* ia = ids + r0 + tid / A_CPR;
    const int* ib = ids + r0 + tid / B_CPR;
#pragma unroll
    for (int i = 0; i < A_N; ++i) ra[i] = load_piece<VEC, HALF>((const unsigned short*)(Ab + (__umul24((unsigned)ia[i * (256 / A_CPR)], lda2) + col_a2)));
#pragma unroll
    for (int i = 0; i < B_N; ++i) rb[i] = load_piece<VEC, HALF>((const unsigned short*)(Bb + (__umul24((unsigned)ib[i * (256 / B_CPR)], ldb2) + col_b2)));
  };
  const int wm = (wave / Cfg::WN) * (MI * 32), wn = (wave % Cfg::WN) * (NJ * 32);
  const int r = lane & 31, g = lane >> 5;
  f32x16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
  auto compute = [&](int stage) {
    const unsigned short* As = smem + stage * Cfg::STAGE_ELEMS;
    const unsigned short* Bs = As + BK * LDA;
#pragma unroll
    for (int kk = 0; kk < BK; kk += 16) {
      bf16x8 fa[MI], fb[NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[i] = frag_transposed(As, LDA, kk + 8 * g, wm + i * 32, lane);
#pragma unroll
      for (int j = 0; j < NJ; ++j) fb[j] = frag_transposed(Bs, LDB, kk + 8 * g, wn + j * 32, lane);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
  };

  for (int s0 = 0; s0 < nrows; s0 += WL_SUB) {
    const int rows = min(nrows - s0, WL_SUB);
    __syncthreads();   // the tables and stages of what was computed before are read to the end
    {
      // all of a thread's ids are requested before it waits for one, and likewise the gates
      constexpr int PR = WL_SUB / 256;
      int idv[PR];
      float gv[PR];
      if (a.perm) {
        const int* pp = a.perm + (long)h * a.M + row0 + s0;
#pragma unroll
        for (int i = 0; i < PR; ++i) idv[i] = pp[min(tid + 256 * i, rows - 1)];
      } else {
#pragma unroll
        for (int i = 0; i < PR; ++i) idv[i] = row0 + s0 + min(tid + 256 * i, rows - 1);
      }
      if (GATE && a.gate) {
        const float* gp = a.gate + (long)h * a.gate_hstride;
#pragma unroll
        for (int i = 0; i < PR; ++i) gv[i] = gp[idv[i]];
      } else {
#pragma unroll
        for (int i = 0; i < PR; ++i) gv[i] = 1.f;
      }
#pragma unroll
      for (int i = 0; i < PR; ++i) {
        const int t = tid + 256 * i;
        if (t < rows) {
          ids[t] = div_by(idv[i], div_magic(a.div));
          gsc[t] = gv[i];
        }
      }
      __syncthreads();
      const int last = ids[rows - 1];
      for (int t = rows + tid; t < rows + 4 * BK && t < Cfg::ROW_CAP; t += 256) {
        gsc[t] = 0.f;
        ids[t] = last;
      }
      __syncthreads();
    }
    auto store_lds = [&](int stage, const chunk_t (&ra)[A_N], const chunk_t (&rb)[B_N], int r0) {
      unsigned short* As = smem + stage * Cfg::STAGE_ELEMS;
      unsigned short* Bs = As + BK * LDA;
      const float* ga = gsc + r0 + tid / A_CPR;
      const float* gb = gsc + r0 + tid / B_CPR;
#pragma unroll
      for (int i = 0; i < A_N; ++i) {
        chunk_t v = half_a ? second_half(ra[i]) : ra[i];
        if (GATE == 1) v = scale_chunk(v, ga[i * (256 / A_CPR)]);
        *(chunk_t*)(&As[(tid / A_CPR + i * (256 / A_CPR)) * LDA + (tid % A_CPR) * VEC]) = v;
      }
      if (r0 + BK <= rows) {   // uniform: every row of the step counts
#pragma unroll
        for (int i = 0; i < B_N; ++i) {
          chunk_t v = half_b ? second_half(rb[i]) : rb[i];
          if (GATE == 2) v = scale_chunk(v, gb[i * (256 / B_CPR)]);
          *(chunk_t*)(&Bs[(tid / B_CPR + i * (256 / B_CPR)) * LDB + (tid % B_CPR) * VEC]) = v;
        }
      } else {
#pragma unroll
        for (int i = 0; i < B_N; ++i) {
          const int rr = tid / B_CPR + i * (256 / B_CPR);
          chunk_t v = half_b ? second_half(rb[i]) : rb[i];
          if (GATE == 2) v = scale_chunk(v, gb[i * (256 / B_CPR)]);
          *(chunk_t*)(&Bs[rr * LDB + (tid % B_CPR) * VEC]) = r0 + rr < rows ? v : zero_chunk<VEC>();
        }
      }
    };
    // the loop body is two steps, straight-line: an odd step count is rounded up
    const int nk2 = ((rows + BK - 1) / BK + 1) & ~1;
    load_global(ra0, rb0, 0);
    load_global(ra1, rb1, BK);
    store_lds(0, ra0, rb0, 0);
    __syncthreads();
    for (int kt = 0; kt < nk2; kt += 2) {
      load_global(ra0, rb0, (kt + 2) * BK);
      compute(0);
      store_lds(1, ra1, rb1, (kt + 1) * BK);
      __syncthreads();
      load_global(ra1, rb1, (kt + 3) * BK);
      compute(1);
      store_lds(0, ra0, rb0, (kt + 2) * BK);
      __syncthreads();
    }
  }

  // 32 x 32 blocks past the last feature are neither stored nor added up
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (i0 + wm + i * 32 >= a.Ka || j0 + wn + j * 32 >= a.Kb) continue;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        slot[((i * NJ + j) * 4 + q4) * 256 + tid] = make_float4(acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]);
    }
}

}  // namespace

template <int VEC, bool HALF>
__global__ __launch_bounds__(256, 2) void mfma_wgrad_list_kernel(WgradList l) {
  extern __shared__ __attribute__((aligned(16))) unsigned short smem[];
  const int lane = threadIdx.x & 63;
  int prob = 0, tile = 0, grp = 0, parts = 0, part = 0, slot = 0, units = 0, row0 = 0, rows = 0;
  {
    WlMap m;
    make_map(l, lane, m);
    if (blockIdx.x == 0 && threadIdx.x == 0) {   // for the reduction
      int* plan = (int*)l.partial;
      plan[WGRAD_LIST_MAX] = m.len;
#pragma unroll
      for (int p = 0; p < WGRAD_LIST_MAX; ++p) plan[p] = m.tot[p];
    }
    // an XCD (work-group ids x, x + 8, ...) takes a contiguous eighth of the list
    const int share = (m.total + 7) / 8;
    int idx = (int)(blockIdx.x & 7) * share + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= share || idx >= m.total) return;
    bool found = false;
#pragma unroll
    for (int p = 0; p < WGRAD_LIST_MAX; ++p) {
      if (p < l.n && !found) {
        const int span = m.tot[p] * l.p[p].ntile;
        if (idx < span) {
          found = true;
          prob = p;
          tile = idx / m.tot[p];
          int rem = idx % m.tot[p];
          const int np = parts_of(m.gu[p], m.len);
          unsigned long long mask = 0;
          for (part = 0;; ++part) {
            mask = __ballot(np > part);
            const int cnt = __popcll(mask);
            if (rem < cnt) break;
            rem -= cnt;
          }
          for (; rem > 0; --rem) mask &= mask - 1;   // drop the groups before it
          grp = __builtin_ctzll(mask);
          const int incl = wave_scan(np, lane);
          parts = __builtin_amdgcn_readlane(np, grp);
          slot += tile * m.tot[p] + __builtin_amdgcn_readlane(incl, grp) - parts + part;
          units = __builtin_amdgcn_readlane(m.gu[p], grp);
          row0 = __builtin_amdgcn_readlane(m.first[p], grp);
          rows = __builtin_amdgcn_readlane(m.rows[p], grp);
        } else {
          idx -= span;
          slot += span;
        }
      }
    }
  }
  const WgradItem& a = l.p[prob];
  const int h = grp / a.E, e = grp % a.E, ti = tile / a.tj, tj = tile % a.tj;
  const int u0 = (int)((long)units * part / parts), u1 = (int)((long)units * (part + 1) / parts);
  const int nrows = min(rows, u1 * WL_UNIT) - u0 * WL_UNIT;
  row0 += u0 * WL_UNIT;
  float4* out = (float4*)(l.partial + WL_PLAN + (long)slot * WL_SLOT);
  if (a.wide)
    wgrad_part<WlWide, VEC, 1, HALF>(a, h, e, row0, nrows, ti * WlWide::BM, tj * WlWide::BN, out, smem);
  else if (a.gate)
    wgrad_part<WlTall, VEC, 2, HALF>(a, h, e, row0, nrows, ti * WlTall::BM, tj * WlTall::BN, out, smem);
  else
    wgrad_part<WlTall, VEC, 0, HALF>(a, h, e, row0, nrows, ti * WlTall::BM, tj * WlTall::BN, out, smem);
}

// Adds the parts of the items, in order; empty groups get zeros.  Block (item, 32 x 32 block of the wave tile).
// The blocks past the last item add the routers' bias gradients, one wave per column (block sums lane by lane, then a butterfly).
__global__ __launch_bounds__(256) void wgrad_list_reduce_kernel(WgradList l) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int item = blockIdx.x, prob = 0;
  if (item >= l.items) {
    const int col = (item - l.items) * 32 + blockIdx.y * 4 + wave;
    if (col >= l.db_sides * l.db_HE) return;
    const int side = col / l.db_HE, c = col % l.db_HE;
    float* db = side ? l.db1 : l.db0;
    if (!db) return;
    const float* p = l.dbpart + ((long)(side * (l.db_HE / l.db_E) + c / l.db_E) * l.db_nblk) * l.db_E + c % l.db_E;
    float s = 0.f;
    for (int b = lane; b < l.db_nblk; b += 64) s += p[(long)b * l.db_E];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) db[c] = s;
    return;
  }
  // the part length and the parts per tile are the ones the weight-gradient launch left; the item's own group sizes give the rest
  const int* plan = (const int*)l.partial;
  const int len = plan[WGRAD_LIST_MAX];
  int slot = 0;
  for (; prob < l.n; ++prob) {
    const int cnt = l.p[prob].heads * l.p[prob].E * l.p[prob].ntile;
    if (item < cnt) break;
    item -= cnt;
    slot += plan[prob] * l.p[prob].ntile;
  }
  const WgradItem& a = l.p[prob];
  const int G = a.heads * a.E, grp = item % G, tile = item / G, h = grp / a.E, e = grp % a.E;
  int first, rows;
  group_rows(a, lane, first, rows);
  const int np = parts_of((rows + WL_UNIT - 1) / WL_UNIT, len), incl = wave_scan(np, lane);
  const int parts = __builtin_amdgcn_readlane(np, grp);
  slot += tile * plan[prob] + __builtin_amdgcn_readlane(incl, grp) - parts;
  const int MI = a.wide ? WlWide::MI : WlTall::MI, NJ = a.wide ? WlWide::NJ : WlTall::NJ, WN = a.wide ? WlWide::WN : WlTall::WN;
  const int bi = blockIdx.y / NJ, bj = blockIdx.y % NJ;
  const int i0 = (tile / a.tj) * (a.wide ? WlWide::BM : WlTall::BM) + (wave / WN) * (MI * 32) + bi * 32;
  const int j0 = (tile % a.tj) * (a.wide ? WlWide::BN : WlTall::BN) + (wave % WN) * (NJ * 32) + bj * 32;
  if (i0 >= a.Ka || j0 >= a.Kb) return;
  float4 s[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) s[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  const float4* P = (const float4*)(l.partial + WL_PLAN + (long)slot * WL_SLOT) + (blockIdx.y * 4) * 256 + tid;
  for (int w = 0; w < parts; ++w) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = P[(long)w * (WL_SLOT / 4) + q * 256];
      s[q].x += v.x;
      s[q].y += v.y;
      s[q].z += v.z;
      s[q].w += v.w;
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = i0 + 8 * q + 4 * (lane >> 5), j = j0 + (lane & 31);
    store_dw(a, h, e, i, j, s[q].x);
    store_dw(a, h, e, i + 1, j, s[q].y);
    store_dw(a, h, e, i + 2, j, s[q].z);
    store_dw(a, h, e, i + 3, j, s[q].w);
  }
}

static bool wl_aligned(const void* p, size_t b) { return ((uintptr_t)p % b) == 0; }

void wgrad_list_add(WgradList& l, const WgradArgs& w) {
  if (l.n >= WGRAD_LIST_MAX) {
    l.n = WGRAD_LIST_MAX + 1;   // refused by wgrad_list_supported
    return;
  }
  WgradItem& a = l.p[l.n++];
  a.perm = w.perm;
  a.offsets = w.offsets;
  a.gate = w.gate;
  a.gate_hstride = w.gate_hstride;
  a.heads = w.heads;
  a.E = w.E;
  a.M = w.M;
  a.div = w.a_div;
  a.A = w.A;
  a.lda = w.lda;
  a.a_hoff = w.a_hoff;
  a.Ka = w.Ka;
  a.B = w.Bm;
  a.ldb = w.ldb;
  a.b_hoff = w.b_hoff;
  a.Kb = w.Kb;
  a.dW = w.dW;
  a.w_hstride = w.w_hstride;
  a.w_estride = w.w_estride;
  a.swa = w.swa;
  a.kb_store = w.kb_store ? w.kb_store : w.Kb;
  a.col_split = w.col_split;
  a.dW2 = w.dW2;
  // the tile shape that covers the output with fewer tiles; a tie goes along the longer side.  (The wide tile scales its A side,
  // the tall one its B side, so the 128 features of the tile are the ones that are scaled.)
  auto tiles = [&](int bm, int bn) { return ((a.Ka + bm - 1) / bm) * ((a.Kb + bn - 1) / bn); };
  const int tw = tiles(128, 256), tt = tiles(256, 128);
  a.wide = tw < tt || (tw == tt && a.Ka < a.Kb);
  a.tj = (a.Kb + (a.wide ? 255 : 127)) / (a.wide ? 256 : 128);
  a.ntile = a.wide ? tw : tt;
  l.items += a.ntile * a.heads * a.E;
}

static int list_blocks(const WgradList& l) { return (max_parts(l.items) + 7) / 8 * 8; }

size_t wgrad_list_partial_floats(const WgradList& l) {
  if (l.n > WGRAD_LIST_MAX) return 0;
  // no part of a cut item is shorter than WL_MIN_PART / 2 units
  long parts = l.items;
  for (int p = 0; p < l.n; ++p) parts += (long)l.p[p].heads * l.p[p].M / (WL_UNIT * WL_MIN_PART) * l.p[p].ntile;
  return (size_t)(parts < max_parts(l.items) ? parts : max_parts(l.items)) * WL_SLOT + WL_PLAN;
}

static int list_vec(const WgradList& l) {
  for (int vec = 8; vec >= 4; vec -= 4) {
    const size_t b = vec * 2;
    bool ok = true;
    for (int p = 0; p < l.n; ++p) {
      const WgradItem& a = l.p[p];
      ok = ok && wl_aligned(a.A, b) && wl_aligned(a.B, b) && a.lda % vec == 0 && a.a_hoff % vec == 0 && a.ldb % vec == 0 && a.b_hoff % vec == 0 &&
           a.Ka % vec == 0 && a.Kb % vec == 0;
    }
    if (ok) return vec;
  }
  return 0;
}

bool wgrad_list_supported(const WgradList& l) {
  if (l.n < 1 || l.n > WGRAD_LIST_MAX || !list_vec(l)) return false;
  long units = 0, longest = 0;
  for (int p = 0; p < l.n; ++p) {
    const WgradItem& a = l.p[p];
    // a lane per group; rows and strides below 2^24 and operands below 4 GiB (32-bit byte offsets made by a 24-bit multiply)
    const size_t op_rows = ((size_t)a.M + a.div - 1) / a.div, ldmax = (size_t)(a.lda > a.ldb ? a.lda : a.ldb);
    if (a.heads * a.E > 64 || a.M < 1 || !a.dW) return false;
    if (op_rows >= ((size_t)1 << 24) || ldmax * 2 >= ((size_t)1 << 24) || op_rows * ldmax * 2 >= ((size_t)1 << 32)) return false;
    if (!a.perm && a.div != 1) return false;
    if (a.perm && (size_t)a.M * a.div >= ((size_t)1 << 32)) return false;   // the reciprocal division of the ids
    units += ((long)a.heads * a.M / WL_UNIT + (long)a.heads * a.E) * a.ntile;
    if (a.M / WL_UNIT + 1 > longest) longest = a.M / WL_UNIT + 1;
  }
  // the reciprocal divisions by the tried part lengths (at most about three even shares)
  const long len = 4 * (units / WL_BLOCKS) + 256;
  return (longest + len) * len < (1l << 32);
}

void launch_wgrad_list(const WgradList& l, hipStream_t s) {
  const int nb = list_blocks(l);
  const size_t lds = WlTall::lds_bytes();
  bool half = list_vec(l) == 4;
  for (int p = 0; p < l.n; ++p) half = half && l.p[p].Ka >= 8 && l.p[p].Kb >= 8;
  auto kern = half ? mfma_wgrad_list_kernel<8, true> : list_vec(l) == 8 ? mfma_wgrad_list_kernel<8, false> : mfma_wgrad_list_kernel<4, false>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  kern<<<nb, 256, lds, s>>>(l);
  prof_mark(s, "bwd.wgrad_reduce");
  const int dbx = l.dbpart ? (l.db_sides * l.db_HE + 31) / 32 : 0;
  wgrad_list_reduce_kernel<<<dim3(l.items + dbx, 8), 256, 0, s>>>(l);
}

}  // namespace sh
