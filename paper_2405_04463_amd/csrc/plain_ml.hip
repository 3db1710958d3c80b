// plain_ml.hip -- the mask overlap for the setting with masks in plain
// (Sec. 4.3, Alg. 2): the parties know every mask, so ml = |m' AND M| with
// m' the rotated query mask (Sec. 3) is a public integer that each party
// computes for itself; only the code dot is secret-shared.
//
// ml is a matrix product over 12,800 bits, taken on the matrix cores in FP4
// (E2M1): a 0/1 bit is one 4-bit operand element, f32 sums of at most 12,800
// ones are exact.  Query rotations are applied once per row by
// rotate_masks_kernel, so the main kernel reads plain packed rows.
#include "device.h"
#include "launch.h"

namespace imc {

struct RotMaskArgs {
  const uint64_t* masks;   // [q][200]
  uint64_t* out;           // [q*r][200]
  uint64_t q;
  int32_t r;
  int8_t rot[IMC_MAX_ROT_DEV];
};

// Word w of row qi*r + ri = bits 64w .. 64w+63 of rot_s(m_qi), s = rot[ri]:
// bit i of the rotated mask is bit rot_src(i, s) of the mask.  Columns are 4
// bits and angular rows 200 columns, so a word's 16 columns are at most three
// runs that are contiguous in the mask too (the word may cross into the next
// angular row, and the source may wrap): each is one shift of two words.
__global__ void __launch_bounds__(256) rotate_masks_kernel(RotMaskArgs a) {
  const uint64_t t = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const uint64_t rows = a.q * uint64_t(a.r);
  if (t >= rows * kWords) return;
  const uint64_t row = t / kWords;
  const int w = int(t % kWords);
  const uint64_t* m = a.masks + (row / uint64_t(a.r)) * kWords;
  const int s = a.rot[row % uint64_t(a.r)];
  constexpr int kCols = kRowLen / 4;
  uint64_t v = 0;
  for (int c = 0; c < 16;) {
    const int dst = 16 * w + c, arow = dst / kCols, dcol = dst - arow * kCols;
    int scol = dcol - s;
    scol += scol < 0 ? kCols : 0;
    scol -= scol >= kCols ? kCols : 0;
    const int len = min(min(16 - c, kCols - dcol), kCols - scol);
    const int bit = 4 * (arow * kCols + scol), off = bit & 63;
    uint64_t x = m[bit >> 6] >> off;
    if (off + 4 * len > 64) x |= m[(bit >> 6) + 1] << (64 - off);
    if (len < 16) x &= (1ull << (4 * len)) - 1;
    v |= x << (4 * c);
    c += len;
  }
  a.out[row * kWords + w] = v;
}

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i_a8 __attribute__((ext_vector_type(4), aligned(8)));   // masks are 8-byte aligned

constexpr int kMlT = 128;   // rows and entries of a tile

struct MlArgs {
  const uint64_t* rm;      // [rows][200] rotated query masks
  const uint64_t* dm;      // [n][200] database masks
  uint16_t* ml;            // [rows][ld]
  uint64_t rows, n, ld;
  uint32_t mt, nt;         // row tiles, entry tiles
};

// Bit J of every 4-bit group of w as FP4 elements: codes 1, 2, 4 are 0.5, 1
// and 2; bit 3 (the sign's place) is moved to code 4.
template <int J>
__device__ __forceinline__ v8i ml_elems(v4i w) {
  v8i o;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[i] = J == 3 ? (w[i] >> 1) & 0x44444444 : w[i] & (0x11111111 << J);
    o[i + 4] = 0;   // the upper half of the operand is not read in FP4
  }
  return o;
}

// The 16 x 16 block sums of bit J of 128 bit groups: 4 x 4 blocks of a wave.
template <int J>
__device__ __forceinline__ void ml_mfma(v4f (&acc)[4][4], const v4i (&x)[4], const v4i (&y)[4]) {
  // E8M0 scales that make every element's value 1: 2, 1, 1/2, 1/2
  constexpr int kScale = J == 0 ? int(0x80808080u) : J == 1 ? 0x7f7f7f7f : 0x7e7e7e7e;
  constexpr int kFp4 = 4;
  v8i b[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) b[j] = ml_elems<J>(y[j]);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const v8i a = ml_elems<J>(x[i]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      acc[i][j] =
          __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b[j], acc[i][j], kFp4, kFp4, 0, kScale, 0, kScale);
  }
}

// Workgroup tile 128 rows x 128 entries, four waves of 64 x 64.  A lane holds
// 16 bytes (128 bits) of a mask at a time, loaded straight from memory: the
// 16 lanes x 4 groups of a fragment are 16 masks x 64 contiguous bytes.  The
// order of the bits within k does not matter as long as both operands share
// it, so the four MFMAs of a 16-byte piece take bits 0, 1, 2 and 3 of its
// 4-bit groups: one AND per operand register, no unpacking.  Consecutive
// workgroups of one XCD walk the row tiles of one entry tile.  Bound by issue:
// 160 ANDs and 64 MFMAs of 16 cycles a piece (1,984 rows x 300,000 entries: MFMA
// pipes 0.60 busy at 2.1 GHz).  1,984 rows x 65,536 entries 3,170 -> 575 us
// (popcounts on the vector ALUs before); 31 rows x 1,000 entries 91 -> 26.  Without the scheduling fences the compiler moves the next
// piece's loads behind the MFMAs: 710 us, 850 without unrolling.
__global__ void __launch_bounds__(256) plain_ml_kernel(MlArgs a) {
  const uint32_t i = blockIdx.x, xcd = i & 7, s8 = i >> 3;
  const uint32_t u = s8 % a.mt, tt = (s8 / a.mt) * 8 + xcd;
  if (tt >= a.nt) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t r0 = uint64_t(u) * kMlT + (wave >> 1) * 64, e0 = uint64_t(tt) * kMlT + (wave & 1) * 64;
  if (r0 >= a.rows || e0 >= a.n) return;
  const int8_t* xp[4];
  const int8_t* yp[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint64_t r = min(r0 + 16 * j + (lane & 15), a.rows - 1), e = min(e0 + 16 * j + (lane & 15), a.n - 1);
    xp[j] = reinterpret_cast<const int8_t*>(a.rm + r * kWords) + (lane >> 4) * 16;
    yp[j] = reinterpret_cast<const int8_t*>(a.dm + e * kWords) + (lane >> 4) * 16;
  }
  v4f acc[4][4];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) acc[x][y] = v4f{0, 0, 0, 0};

  constexpr int kIters = kWords / 8;   // 25 pieces of 64 bytes a mask
  v4i x[4], y[4], nx[4], ny[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    nx[j] = *reinterpret_cast<const v4i_a8*>(xp[j]);
    ny[j] = *reinterpret_cast<const v4i_a8*>(yp[j]);
  }
#pragma unroll 5
  for (int k = 0; k < kIters; ++k) {
    const int next = min(k + 1, kIters - 1) * 64;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = nx[j];
      y[j] = ny[j];
      nx[j] = *reinterpret_cast<const v4i_a8*>(xp[j] + next);
      ny[j] = *reinterpret_cast<const v4i_a8*>(yp[j] + next);
    }
    __builtin_amdgcn_sched_barrier(0);
    ml_mfma<0>(acc, x, y);
    __builtin_amdgcn_sched_barrier(0);
    ml_mfma<1>(acc, x, y);
    __builtin_amdgcn_sched_barrier(0);
    ml_mfma<2>(acc, x, y);
    __builtin_amdgcn_sched_barrier(0);
    ml_mfma<3>(acc, x, y);
  }
  // 16 x 16 block: lane l holds column l % 16, register v row 4 (l / 16) + v
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint64_t row = r0 + 16 * p + 4 * (lane >> 4) + v;
      if (row >= a.rows) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint64_t e = e0 + 16 * q + (lane & 15);
        if (e < a.n) a.ml[row * a.ld + e] = uint16_t(acc[p][q][v]);
      }
    }
}

hipError_t launch_rotate_masks(const uint64_t* masks, uint64_t q, const imc_ids_dev& ids, uint64_t* out,
                               hipStream_t s) {
  const uint64_t threads = q * uint64_t(ids.r) * kWords;
  if (threads == 0) return hipSuccess;
  RotMaskArgs a;
  a.masks = masks;
  a.out = out;
  a.q = q;
  a.r = ids.r;
  for (int i = 0; i < IMC_MAX_ROT_DEV; ++i) a.rot[i] = i < ids.r ? ids.rot[i] : 0;
  if (!fits_grid(threads, 256)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(rotate_masks_kernel, dim3(unsigned((threads + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_plain_ml(const uint64_t* row_masks, uint64_t rows, const uint64_t* db_masks, uint64_t n,
                           uint16_t* ml, uint64_t ld, hipStream_t s) {
  if (rows == 0 || n == 0) return hipSuccess;
  MlArgs a;
  a.rm = row_masks;
  a.dm = db_masks;
  a.ml = ml;
  a.rows = rows;
  a.n = n;
  a.ld = ld;
  a.mt = uint32_t((rows + kMlT - 1) / kMlT);
  a.nt = uint32_t((n + kMlT - 1) / kMlT);
  const uint64_t groups = uint64_t((a.nt + 7) / 8) * 8 * a.mt;
  if (groups > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(plain_ml_kernel, dim3(unsigned(groups)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace imc
