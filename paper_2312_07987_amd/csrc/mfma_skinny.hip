// Row GEMM of the SwitchHead projections (arXiv 2312.07987, Sec. 2.1 - 2.2: queries, keys, value experts) for calls of a few rows:
// one short prompt, the queries of a decoding step.  On the 128 x 128 tiles such a call has 8 to 20 work-groups whose K loop waits
// for memory at every step (K = 1024: sixteen round trips, 19 us for 100 rows whatever the width).  Here a work-group makes a
// 32 x 32 tile, its four waves take a quarter of the reduction each, and a wave requests everything it needs of up to 256
// reduction indices (32 x 256 of A straight into operand fragments, 256 x 32 of B) before it waits: one round trip per 1024.  The four
// partial sums meet in LDS and are added in wave order.
// 100 rows of d_model 1024, 4 heads of 128 (events around each): queries and keys 21 -> 10 us, value experts (5 experts, 3 active)
// 22 -> 15; the whole call 110 -> 92.  The line, on its safe side: 768 tiles are three for each CU, two of them resident.  A launch of 128 x 128
// tiles takes its sixteen trips whatever its size; in us, those / these: 608 tiles 21.7 / 15.2 and 800 21.5 / 17.9 (queries and
// keys, whole tiles), 680 22.3 / 20.6, 928 23.3 / 23.5, 980 22.5 / 22.0, 1280 22.2 / 26.6 (value experts, partly filled).
#include "common.h"
#include "mfma_util.h"

namespace sh {

namespace {
constexpr int SK_T = 32;      // tile rows and columns
constexpr int SK_KW = 256;    // reduction indices a wave holds at a time
constexpr int SK_MAX_TILES = 768;
}  // namespace

__global__ __launch_bounds__(256, 2) void skinny_row_gemm_kernel(RowGemmArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned short bs[4][SK_KW * SK_T];   // rows 64 bytes apart: the transposing reads' four rows lie
                                                                               // in four different quarters of the banks
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, g = lane >> 5;
  const int ncol = (a.Nc + SK_T - 1) / SK_T;
  const int grp = blockIdx.y / ncol, n0 = (blockIdx.y % ncol) * SK_T;
  const int h = grp / a.E, e = grp % a.E;
  int first = 0, end = a.M;
  if (a.perm) {
    first = a.offsets[(long)h * (a.E + 1) + e];
    end = a.offsets[(long)h * (a.E + 1) + e + 1];
  }
  const int row0 = first + blockIdx.x * SK_T;
  if (row0 >= end) return;
  const int rows = end - row0 < SK_T ? end - row0 : SK_T;
  const bool second = a.hsplit > 0 && h >= a.hsplit;
  const int hh = second ? h - a.hsplit : h;
  const unsigned short* B = (const unsigned short*)(second ? a.B2 : a.B) + (long)hh * a.b_hstride + (long)e * a.b_estride;

  // a row past the end repeats the tile's last one, an index past K or a column past Nc repeats the last piece; B's become zeros on
  // their way into LDS, A's meet those zeros (so they have to be finite: they are zeroed as well)
  const int rr = r < rows ? r : rows - 1;
  const int id = a.perm ? a.perm[(long)h * a.M + row0 + rr] : row0 + rr;
  const unsigned short* Arow = (const unsigned short*)a.A + (long)div_by(id, div_magic(a.a_div)) * a.lda + (long)hh * a.a_hoff;
  const int per = ((a.K + 3) / 4 + 15) / 16 * 16;   // a wave's share of the reduction
  const int kbeg = wave * per, kend = min(a.K, kbeg + per);
  const int bc = n0 + (lane & 3) * 8, bcol = min(bc, a.Nc - 8);
  f32x16 acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.f;
  for (int k0 = kbeg; k0 < kend; k0 += SK_KW) {
    uint4 rb[16];
    bf16x8 fa[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) rb[i] = *(const uint4*)(B + (long)min(k0 + (lane >> 2) + 16 * i, a.K - 1) * a.sbk + bcol);
#pragma unroll
    for (int i = 0; i < 16; ++i) fa[i] = *(const bf16x8*)(Arow + min(k0 + 16 * i + 8 * g, a.K - 8));
    wave_order();   // (the area is the wave's own and a wave's LDS operations keep their order)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int k = k0 + (lane >> 2) + 16 * i;
      *(uint4*)(&bs[wave][((lane >> 2) + 16 * i) * SK_T + (lane & 3) * 8]) = k < kend && bc < a.Nc ? rb[i] : make_uint4(0, 0, 0, 0);
    }
    wave_order();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (k0 + 16 * i < kend) {   // uniform
        const bf16x8 z = {};
        const bf16x8 f = k0 + 16 * i + 8 * g < a.K ? fa[i] : z;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, frag_transposed(bs[wave], SK_T, 16 * i + 8 * g, 0, lane), acc, 0, 0, 0);
      }
    }
    wave_order();
  }
  __syncthreads();
  float* part = (float*)&bs[0][0];   // [4][32][32]
#pragma unroll
  for (int q = 0; q < 16; ++q) part[(wave * SK_T + 8 * (q >> 2) + 4 * g + (q & 3)) * SK_T + r] = acc[q];
  __syncthreads();
  const int row = tid >> 3, c = (tid & 7) * 4;
  if (row >= rows || n0 + c >= a.Nc) return;
  float4 s = *(const float4*)(&part[row * SK_T + c]);
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    const float4 v = *(const float4*)(&part[(w * SK_T + row) * SK_T + c]);
    s.x += v.x;
    s.y += v.y;
    s.z += v.z;
    s.w += v.w;
  }
  const int oid = a.perm ? a.perm[(long)h * a.M + row0 + row] : row0 + row;
  unsigned short* C = (unsigned short*)(second ? a.C2 : a.C) + (long)div_by(oid, div_magic(a.c_div)) * a.ldc + (long)hh * a.c_hoff + n0 + c;
  *(uint2*)C = make_uint2(pack_bf16x2(s.x, s.y), pack_bf16x2(s.z, s.w));
}

// ----------------------------------------------------------------------------------------
// Output experts of calls of a few rows: y[n] = sum over every (head, expert) segment of gate * ctx[n, h] W_O[h, e] in one accumulator
// (segment mode 3, gates from the top-k tables).  32 x 32 tiles, token-ordered rows, the reduction shared out among the waves in pieces
// of a head and 64 indices.  A piece's product is an fp32 accumulator of its own that the gates multiply on its way into the sum: nothing
// is rounded before the end, and what an expert gives a token that did not select it (an infinity, a NaN) is left out.  By expert sets the same
// call was a launch of 128 x 128 tiles over the k selected experts of each head, a bf16 partial sum per head, and another launch to add
// them; by expert-sorted rows fp32 atomics, with launches to clear the accumulator and to cast it.
// ----------------------------------------------------------------------------------------
template <int VEC>
__device__ __forceinline__ uint4 sk_load8(const unsigned short* row, int k, int end) {   // row[k .. k + 7], zeros from `end` on (end >= VEC)
  if constexpr (VEC == 8) {
    const uint4 v = *(const uint4*)(row + min(k, end - 8));
    return k < end ? v : make_uint4(0, 0, 0, 0);
  } else {
    const uint2 lo = *(const uint2*)(row + min(k, end - 4)), hi = *(const uint2*)(row + min(k + 4, end - 4));
    return make_uint4(k < end ? lo.x : 0, k < end ? lo.y : 0, k + 4 < end ? hi.x : 0, k + 4 < end ? hi.y : 0);
  }
}

constexpr int SK_W = 8, SK_UK = 64, SK_EB = 5;   // waves; reduction indices and experts of a wave's item
// A wave's item: a head, 64 of its reduction indices (`per` pieces), up to SK_EB of its experts (fewer where there would be idle waves): eb
// experts, split items for all of them.
struct SkItems {
  int split, eb;
};
__host__ __device__ inline SkItems sk_items(int H, int E, int per) {
  const int most = (E + SK_EB - 1) / SK_EB, wide = SK_W / (H * per) < E ? SK_W / (H * per) : E;
  const int split = most > wide ? most : wide, eb = (E + split - 1) / split;
  return {(E + eb - 1) / eb, eb};
}

template <int VEC>
__global__ __launch_bounds__(512, 1) void skinny_concat_kernel(RowGemmArgs a) {
  constexpr int W = SK_W, UK = SK_UK, EB = SK_EB;
  __shared__ __attribute__((aligned(16))) unsigned short bs[W][UK * SK_T];   // then the partial sums [W][32][32] fp32
  __shared__ __attribute__((aligned(16))) float gts[MAX_SEGD * SK_T];   // the tile's gates [head * experts + expert][row], -1: not selected
  __shared__ SegDesc descs[MAX_SEGD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, g = lane >> 5;
  const int row0 = blockIdx.x * SK_T, n0 = blockIdx.y * SK_T;
  const int rows = min(a.M - row0, SK_T);
  if (tid < a.nseg) descs[tid] = a.segd[tid];
  for (int t = tid; t < a.nseg * SK_T; t += 512) gts[t] = a.gidx ? -1.f : 1.f;   // (no tables: every segment counts)
  __syncthreads();
  if (a.gidx) {
    for (int t = tid; t < SK_T * a.gheads * a.gk; t += 512) {
      const int row = t % SK_T, j = t / SK_T % a.gk, h = t / SK_T / a.gk;
      if (row < rows) {
        const long o = ((long)h * a.M + row0 + row) * a.gk + j;
        gts[(h * a.experts + a.gidx[o]) * SK_T + row] = a.ggate[o];
      }
    }
    __syncthreads();
  }
  // The head's read-out is loaded once for an item's experts; everything of an item is requested before the wave waits.
  const int H = a.gheads, E = a.experts, ups = (a.K + UK - 1) / UK;
  const SkItems items = sk_items(H, E, ups);
  const int split = items.split, eb = items.eb;
  const long arow = (long)(row0 + min(r, rows - 1)) * a.lda;   // (a row past the end repeats the last one; not stored)
  f32x16 acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.f;
  for (int it = wave; it < H * ups * split; it += W) {
    const int h = it / (ups * split), k0 = it / split % ups * UK, e0 = it % split * eb, ne = min(eb, E - e0);
    const unsigned short* Ap = (const unsigned short*)descs[h * E].A + arow;
    uint4 rb[EB][4], fa[4];
#pragma unroll
    for (int u = 0; u < EB; ++u)
      if (u < ne) {   // uniform
        const unsigned short* Bp = (const unsigned short*)descs[h * E + e0 + u].B;
#pragma unroll
        for (int i = 0; i < 4; ++i) rb[u][i] = sk_load8<VEC>(Bp + (long)min(k0 + (lane >> 2) + 16 * i, a.K - 1) * a.sbk, n0 + (lane & 3) * 8, a.Nc);
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[i] = sk_load8<VEC>(Ap, k0 + 16 * i + 8 * g, a.K);
#pragma unroll
    for (int u = 0; u < EB; ++u)
      if (u < ne) {
        f32x16 prod;
#pragma unroll
        for (int q = 0; q < 16; ++q) prod[q] = 0.f;
        wave_order();   // (the area is the wave's own and a wave's LDS operations keep their order)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *(uint4*)(&bs[wave][((lane >> 2) + 16 * i) * SK_T + (lane & 3) * 8]) = k0 + (lane >> 2) + 16 * i < a.K ? rb[u][i] : make_uint4(0, 0, 0, 0);
        wave_order();
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (k0 + 16 * i < a.K)   // uniform
            prod = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[i]), frag_transposed(bs[wave], SK_T, 16 * i + 8 * g, 0, lane), prod, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 gt = *(const f32x4*)(&gts[(h * E + e0 + u) * SK_T + 8 * i + 4 * g]);
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[4 * i + q] = gt[q] < 0.f ? acc[4 * i + q] : fmaf(gt[q], prod[4 * i + q], acc[4 * i + q]);
        }
      }
  }
  __syncthreads();
  float* part = (float*)&bs[0][0];   // [W][32][32]
#pragma unroll
  for (int q = 0; q < 16; ++q) part[(wave * SK_T + 8 * (q >> 2) + 4 * g + (q & 3)) * SK_T + r] = acc[q];
  __syncthreads();
  const int row = tid >> 4, c = (tid & 15) * 2, n = n0 + c;
  if (row >= rows || n >= a.Nc) return;
  float s[2] = {0.f, 0.f};
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const float2 v = *(const float2*)(&part[(w * SK_T + row) * SK_T + c]);
    s[0] = w ? s[0] + v.x : v.x;
    s[1] = w ? s[1] + v.y : v.y;
  }
  *(unsigned*)((unsigned short*)a.C + (long)(row0 + row) * a.ldc + n) = pack_bf16x2(s[0], s[1]);
}

static bool sk_aligned(const void* p) { return ((uintptr_t)p % 16) == 0; }

// A launch of at most SK_MAX_TILES tiles of 32 x 32 (expected: a sorted group's rows are counted together), three for each CU; 16-byte
// pieces of A and B, whole pieces of 8 columns.
bool skinny_row_gemm_supported(const RowGemmArgs& a) {
  if (a.seg_mode != 0 || a.gate || a.mode != STORE_T || a.sbn != 1 || a.sbk < a.Nc) return false;
  if (a.M < 1 || a.K < 8 || a.K % 8 != 0 || a.Nc < 8 || a.Nc % 8 != 0) return false;
  if (!sk_aligned(a.A) || !sk_aligned(a.B) || !sk_aligned(a.C) || (a.hsplit > 0 && !(sk_aligned(a.B2) && sk_aligned(a.C2)))) return false;
  if (a.lda % 8 || a.a_hoff % 8 || a.sbk % 8 || a.b_hstride % 8 || a.b_estride % 8 || a.ldc % 4 || a.c_hoff % 4) return false;
  if ((long)a.M * (a.a_div > a.c_div ? a.a_div : a.c_div) >= (1L << 32)) return false;
  const long cols = (a.Nc + SK_T - 1) / SK_T, groups = (long)a.heads * a.E;
  const long rows = a.perm ? ((long)a.heads * a.M / SK_T + groups) : groups * ((a.M + SK_T - 1) / SK_T);
  return rows * cols <= SK_MAX_TILES && groups * cols <= 65535;
}

void launch_skinny_row_gemm(const RowGemmArgs& a, hipStream_t s) {
  const int group_rows = a.perm && a.max_group_rows > 0 ? a.max_group_rows : a.M;
  const dim3 g((group_rows + SK_T - 1) / SK_T, a.heads * a.E * ((a.Nc + SK_T - 1) / SK_T));
  skinny_row_gemm_kernel<<<g, 256, 0, s>>>(a);
}

static int sk_concat_vec(const RowGemmArgs& a) {
  for (int vec = 8; vec >= 4; vec -= 4) {
    auto al = [&](const void* p) { return ((uintptr_t)p % (2 * vec)) == 0; };
    bool ok = a.K >= vec && a.Nc >= vec && a.K % vec == 0 && a.Nc % vec == 0 && a.lda % vec == 0 && a.sbk % vec == 0 && ((uintptr_t)a.C % 4) == 0 && a.ldc % 2 == 0;
    for (int p = 0; ok && p < a.nseg; ++p) ok = al(a.segd[p].A) && al(a.segd[p].B);
    if (ok) return vec;
  }
  return 0;
}

// Every expert is multiplied, selected or not, so the line compares what the two ways take, in us (the weights of both sums are fitted to
// 6000 calls that ran both ways, 1 to 4096 rows of 64 to 2048 columns, 1 to 10 heads of 16 to 256, up to 64 experts):
//   here: 0.8 for an expert that a wave multiplies, 2 for a round of 256 tiles;
//   expert sets (`sets`): 3.1, with more than one head 5.6 for the sum of the heads, and 0.7 for 64 indices of a selected expert;
//   expert-sorted rows (more sets than the tables hold, or rows that make none): 5.7 for the launches that clear and cast, 0.034 for a
//   tile of 128 rows and columns (few rows are nearly all tiles of a few rows each).
// The whole forward call, us, the other path / here.  Sets: 4 heads of 128, 5 of 5 experts, d_model 1024, 173 tokens 77.7 / 71.6; 2 heads of 96, 5 of 5,
// d_model 412, 256 tokens 69.5 / 56.8; 10 heads of 96, 3 of 5, 6 tokens of 412 138.9 / 147.1; 2 heads of 160, 1 of 32, 58 tokens of 768
// 189.7 / 217.1; one head of 128, 2 of 5, 119 tokens of 1024 45.6 / 42.9.  Sorted rows: 4 heads of 112, 8 of 16, 205 tokens of 1024 299.7 / 267.3,
// but 8 heads of 256, 1 of 4, 17 tokens of 100 52.3 / 71.0; 2 heads of 76, 5 of 32, 40 tokens of 64 68.4 / 81.3.
// Of 5000 other calls 47 that come here lose more than 2 per cent, 98 us in all, for 21000 us that the rest gain (a line in the products alone: one
// in fifteen lost, 1887 us on the 6000).
bool skinny_concat_supported(const RowGemmArgs& a, bool sets) {
  if (a.seg_mode != 3 || a.perm || a.heads != 1 || a.E != 1 || a.mode != STORE_T || a.sbn != 1 || a.M < 1 || a.gtab || a.seg_q) return false;
  // (segment h * experts + e: expert e of head h, the head's read-out the same for all of them)
  if (a.nseg < 1 || a.nseg > MAX_SEGD || a.gheads * a.experts != a.nseg) return false;
  const long tiles = (long)((a.M + SK_T - 1) / SK_T) * ((a.Nc + SK_T - 1) / SK_T);
  if (tiles > 512 || sk_concat_vec(a) == 0) return false;
  const int H = a.gheads, E = a.experts, per = (a.K + SK_UK - 1) / SK_UK;
  const SkItems it = sk_items(H, E, per);
  const long rounds = (tiles + 255) / 256, slots = (long)a.M * a.gk;
  const double here = 0.8 * rounds * ((H * per * it.split + SK_W - 1) / SK_W) * it.eb + 2.0 * rounds + 0.5;
  const double sorted_tiles = H * ((slots < E ? slots : E) + slots / 128.0) * ((a.Nc + 127) / 128);
  return here <= (sets ? (H > 1 ? 5.6 : 3.1) + 0.7 * a.gk * per : 5.7 + 0.034 * sorted_tiles);
}

void launch_skinny_concat(const RowGemmArgs& a, hipStream_t s) {
  const dim3 g((a.M + SK_T - 1) / SK_T, (a.Nc + SK_T - 1) / SK_T);
  if (sk_concat_vec(a) == 8)
    skinny_concat_kernel<8><<<g, 512, 0, s>>>(a);
  else
    skinny_concat_kernel<4><<<g, 512, 0, s>>>(a);
}

}  // namespace sh
