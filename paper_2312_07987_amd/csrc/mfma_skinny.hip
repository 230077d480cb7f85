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

}  // namespace sh
