// dot.hip -- party-local dot products of the shared protocol (Alg. 3, the
// code and mask inner products; App. C: two plain dot products per MPC dot
// product) as i8 MFMA with i32 accumulation over balanced byte limbs.
//
// v = lo + 256 hi (mod 2^16), lo, hi signed bytes.  For u, v in Z_2^16:
//   u v = lo_u lo_v + 256 (lo_u hi_v + hi_u lo_v)  (mod 2^16)
// (the hi*hi term carries 2^16 and vanishes), so each output needs
// acc0 = sum lo lo and acc1 = sum (lo hi + hi lo): three MFMA streams into two
// accumulators.  |acc0| <= 25600 * 2^14 < 2^31 and |acc1| <= 2 * 25600 * 2^14
// < 2^31, so no accumulator wraps.
#include <hip/hip_ext.h>

#include "device.h"
#include "launch.h"

namespace imc {


// ---------------------------------------------------------------------------
// Rotation expand: query operand rows (row-major, unrotated) -> rotated rows
// in the MFMA-native tiled layout [row-block][plane 4][k-chunk 1600][32][16 B].
// ---------------------------------------------------------------------------
struct Rot {
  int8_t s[IMC_MAX_ROT_DEV];
};

template <int K>
__global__ void __launch_bounds__(256) expand_kernel(const int8_t* __restrict__ qop, const uint32_t* __restrict__ qidx,
                                                     uint32_t q, uint32_t r, Rot rot, uint32_t rows_pad,
                                                     int8_t* __restrict__ a) {
  using G = Geo<K>;
  uint64_t t = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  uint64_t total = uint64_t(rows_pad) * kPlanes * G::kChunks;
  if (t >= total) return;
  uint32_t slot = uint32_t(t % 32);
  uint64_t rest = t / 32;
  uint32_t kc = uint32_t(rest % G::kChunks);
  rest /= G::kChunks;
  uint32_t plane = uint32_t(rest % kPlanes);
  uint32_t rb = uint32_t(rest / kPlanes);
  uint32_t row = rb * 32 + slot;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row < q * r) {
    uint32_t qi = row / r, ri = row % r;
    if (qidx) qi = qidx[qi];
    int s = rot.s[ri];
    uint32_t k0 = kc * 16;
    uint32_t h = k0 / kCodeBits, i0 = k0 - h * kCodeBits;
    uint32_t rrow = i0 / kRowLen, w0 = i0 - rrow * kRowLen;
    const int8_t* src = qop + uint64_t(qi) * G::kQopRowBytes + uint64_t(plane) * G::kK + h * kCodeBits + rrow * kRowLen;
    uint32_t wv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int w = int(w0) + 4 * j - 4 * s;
      w = (w % kRowLen + kRowLen) % kRowLen;
      wv[j] = *reinterpret_cast<const uint32_t*>(src + w);
    }
    v = make_uint4(wv[0], wv[1], wv[2], wv[3]);
  }
  *reinterpret_cast<uint4*>(a + uint64_t(rb) * G::kBlockBytes + uint64_t(plane) * G::kPlaneBlockBytes + uint64_t(kc) * 512 +
                            slot * 16) = v;
}

// Same, with an explicit row table (query index, rotation) per row: rows of
// many uneven batches expanded into one operand.  A row whose query index is
// out of range becomes a zero row.
template <int K>
__global__ void __launch_bounds__(256) expand_rows_kernel(const int8_t* __restrict__ qop, uint32_t q,
                                                          const imc_row* __restrict__ rows, uint32_t nrows,
                                                          uint32_t rows_pad, int8_t* __restrict__ a) {
  using G = Geo<K>;
  uint64_t t = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  uint64_t total = uint64_t(rows_pad) * kPlanes * G::kChunks;
  if (t >= total) return;
  uint32_t slot = uint32_t(t % 32);
  uint64_t rest = t / 32;
  uint32_t kc = uint32_t(rest % G::kChunks);
  rest /= G::kChunks;
  uint32_t plane = uint32_t(rest % kPlanes);
  uint32_t rb = uint32_t(rest / kPlanes);
  uint32_t row = rb * 32 + slot;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row < nrows && rows[row].query_index < q) {
    const uint32_t qi = rows[row].query_index;
    const int s = rows[row].rot % kRowLen;
    uint32_t k0 = kc * 16;
    uint32_t h = k0 / kCodeBits, i0 = k0 - h * kCodeBits;
    uint32_t rrow = i0 / kRowLen, w0 = i0 - rrow * kRowLen;
    const int8_t* src = qop + uint64_t(qi) * G::kQopRowBytes + uint64_t(plane) * G::kK + h * kCodeBits + rrow * kRowLen;
    uint32_t wv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int w = int(w0) + 4 * j - 4 * s;
      w = (w % kRowLen + kRowLen) % kRowLen;
      wv[j] = *reinterpret_cast<const uint32_t*>(src + w);
    }
    v = make_uint4(wv[0], wv[1], wv[2], wv[3]);
  }
  *reinterpret_cast<uint4*>(a + uint64_t(rb) * G::kBlockBytes + uint64_t(plane) * G::kPlaneBlockBytes + uint64_t(kc) * 512 +
                            slot * 16) = v;
}

// ---------------------------------------------------------------------------
// dot kernel.  Workgroup tile BM rows x BN entries, WAVES_M x WAVES_N waves of
// (32 WM) x (32 WN) outputs (WM x WN MFMA 32x32x32 blocks, two accumulators
// each).  Per K-step (32 bytes of k per plane) the workgroup stages its
// operand slices in LDS once -- A: BM/32 row-blocks, B: BN/32 entry-blocks,
// each 2 planes x 2 k-chunks x 32 slots x 16 B, i.e. exactly the tiled HBM
// layout -- so fragment reads are 1 KB contiguous per wave.  Three LDS stages
// and NSETS register sets keep the global loads NSETS + 2 steps ahead and the
// fragment reads one step ahead of the MFMAs.  blockIdx.z = 0
// code, 1 mask.
// ---------------------------------------------------------------------------
struct DotArgs {
  const int8_t* a;       // rotated query operand, tiled, rows_pad rows
  const int8_t* b;       // party's database region
  uint16_t* out[2];      // code, mask: [rows][ld]
  uint64_t ld;
  uint32_t rows;         // q * r
  uint32_t a_blocks;     // row-blocks present in a
  uint64_t b_block0;     // first database block (first_entry_id / 32)
  uint64_t b_blocks;     // database blocks holding columns [0, n)
  uint64_t n;            // columns
  uint32_t mt, nt;       // tiles along rows / columns
  uint32_t persistent;   // grid smaller than the tile count: loop over tiles
  uint32_t splits, steps_per;   // SPLIT: workgroups per tile, K-steps of each
  uint32_t* part;        // SPLIT: u32 [vec][split][rows][n]
};

template <int WM, int WN, int WAVES_M, int WAVES_N>
struct DotCfg {
  static constexpr int kBM = 32 * WM * WAVES_M, kBN = 32 * WN * WAVES_N;
  static constexpr int kThreads = 64 * WAVES_M * WAVES_N;
  static constexpr int kABlk = kBM / 32, kBBlk = kBN / 32;
  static constexpr int kChunksPerStep = (kABlk + kBBlk) * 2 * 2 * 32;   // 16-byte chunks
  static constexpr int kPerThread = kChunksPerStep / kThreads;
  static constexpr int kStageBytes = kChunksPerStep * 16;
  static_assert(kChunksPerStep % kThreads == 0, "chunks must divide evenly");
};

template <int K, int WM, int WN, int WAVES_M, int WAVES_N, int NSETS, bool SPLIT = false>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) dot_kernel(DotArgs args) {
  using C = DotCfg<WM, WN, WAVES_M, WAVES_N>;
  using G = Geo<K>;
  extern __shared__ __align__(16) int8_t lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int vec = blockIdx.z;
  // XCD-aware order: workgroup i runs on XCD i % 8; the workgroups one XCD
  // holds at a time are all row tiles of a few column tiles, so each database
  // slice is fetched from HBM once and served to them from that XCD's L2.
  // With a persistent grid (args.persistent) each workgroup walks its XCD's
  // tile sequence with stride gridDim.x / 8; otherwise one tile per workgroup.
  const uint32_t i = blockIdx.x;
  const uint32_t xcd = i & 7;
  // SPLIT: (column tile, part of the K loop) pairs take the place of column tiles.
  const uint32_t ntp = SPLIT ? args.nt * args.splits : args.nt;
  const uint32_t s_end = ((ntp + 7) / 8) * args.mt;
  const uint32_t s_step = args.persistent ? (gridDim.x >> 3) : s_end;
  for (uint32_t s = i >> 3; s < s_end; s += s_step) {
  const uint32_t u = s % args.mt, tg = s / args.mt;
  const uint32_t tp = tg * 8 + xcd;
  if (tp >= ntp) continue;
  const uint32_t t = SPLIT ? tp / args.splits : tp, part = SPLIT ? tp % args.splits : 0;

  // Global source of each 16-byte chunk this thread stages per K-step.
  // Chunk c: block (A row-blocks first, then B entry-blocks), plane, k-chunk, slot.
  const int8_t* src[C::kPerThread];
#pragma unroll
  for (int j = 0; j < C::kPerThread; ++j) {
    const int c = tid + j * C::kThreads;
    const int blk = c >> 7, rem = c & 127;
    const int plane = rem >> 6, kcl = (rem >> 5) & 1, slot = rem & 31;
    const int8_t* base;
    if (blk < C::kABlk) {
      uint32_t rb = u * C::kABlk + blk;
      rb = rb < args.a_blocks ? rb : args.a_blocks - 1;
      base = args.a + size_t(rb) * G::kBlockBytes;
    } else {
      uint64_t cb = uint64_t(t) * C::kBBlk + (blk - C::kABlk);
      cb = cb < args.b_blocks ? cb : args.b_blocks - 1;
      base = args.b + size_t(args.b_block0 + cb) * G::kBlockBytes;
    }
    src[j] = base + size_t(2 * vec + plane) * G::kPlaneBlockBytes + size_t(kcl) * 512 + slot * 16;
  }

  v16i acc0[WM][WN], acc1[WM][WN];
#pragma unroll
  for (int x = 0; x < WM; ++x)
#pragma unroll
    for (int y = 0; y < WN; ++y)
#pragma unroll
      for (int e = 0; e < 16; ++e) { acc0[x][y][e] = 0; acc1[x][y][e] = 0; }

  constexpr int kSteps = G::kChunks / 2;   // steps of 32 bytes of k
  static_assert(kSteps % NSETS == 0, "the K loop is unrolled by NSETS");
  const int k_b = SPLIT ? int(part * args.steps_per) : 0;
  const int k_e = SPLIT ? min(k_b + int(args.steps_per), kSteps) : kSteps;
  v4i rs[NSETS][C::kPerThread];
#define IMC_GLOAD(R, KS)                                                              \
  _Pragma("unroll") for (int c_ = 0; c_ < C::kPerThread; ++c_)                        \
      R[c_] = *reinterpret_cast<const v4i*>(src[c_] + size_t(2 * (KS)) * 512);
#define IMC_LSTORE(R, STAGE)                                                          \
  _Pragma("unroll") for (int c_ = 0; c_ < C::kPerThread; ++c_)                        \
      *reinterpret_cast<v4i*>(lds + (STAGE) * C::kStageBytes + (tid + c_ * C::kThreads) * 16) = R[c_];
#define IMC_FRAGS(ALO, AHI, BLO, BHI, STAGE)                                          \
  {                                                                                   \
    const int8_t* st_ = lds + (STAGE) * C::kStageBytes;                               \
    _Pragma("unroll") for (int x_ = 0; x_ < WM; ++x_) {                               \
      const int8_t* p_ = st_ + (wm * WM + x_) * 2048 + lane * 16;                     \
      ALO[x_] = *reinterpret_cast<const v4i*>(p_);                                    \
      AHI[x_] = *reinterpret_cast<const v4i*>(p_ + 1024);                             \
    }                                                                                 \
    _Pragma("unroll") for (int y_ = 0; y_ < WN; ++y_) {                               \
      const int8_t* p_ = st_ + (C::kABlk + wn * WN + y_) * 2048 + lane * 16;          \
      BLO[y_] = *reinterpret_cast<const v4i*>(p_);                                    \
      BHI[y_] = *reinterpret_cast<const v4i*>(p_ + 1024);                             \
    }                                                                                 \
  }

  // Pipeline over three LDS stages: step j is global-loaded NSETS iterations
  // ahead into register set (j - 2) % NSETS, written to stage j % 3 two
  // iterations ahead, and its fragments are read from LDS one iteration ahead,
  // while the MFMAs of the current step run.  Iteration k overwrites stage
  // (k + 2) % 3, last read at iteration k - 2.  Indices past the last step
  // are clamped (redundant reloads instead of branches keep the sets in VGPRs).
  v4i falo[WM], fahi[WM], fblo[WN], fbhi[WN];     // fragments of the current step
  v4i nalo[WM], nahi[WM], nblo[WN], nbhi[WN];     // fragments of the next step
  {
    v4i r0[C::kPerThread];
    IMC_GLOAD(r0, k_b)
    IMC_LSTORE(r0, k_b % 3)
    IMC_GLOAD(r0, k_b + 1)
    IMC_LSTORE(r0, (k_b + 1) % 3)
  }
#pragma unroll
  for (int set = 0; set < NSETS; ++set) { IMC_GLOAD(rs[set], min(k_b + set + 2, k_e - 1)) }
  __syncthreads();
  IMC_FRAGS(falo, fahi, fblo, fbhi, k_b % 3)
  for (int k0 = k_b; k0 < k_e; k0 += NSETS) {
#pragma unroll
    for (int uu = 0; uu < NSETS; ++uu) {
      const int k = k0 + uu;
      IMC_FRAGS(nalo, nahi, nblo, nbhi, (k + 1) % 3)
#pragma unroll
      for (int x = 0; x < WM; ++x)
#pragma unroll
        for (int y = 0; y < WN; ++y) {
          acc0[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(falo[x], fblo[y], acc0[x][y], 0, 0, 0);
          acc1[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(falo[x], fbhi[y], acc1[x][y], 0, 0, 0);
          acc1[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fahi[x], fblo[y], acc1[x][y], 0, 0, 0);
        }
      IMC_LSTORE(rs[uu], (k + 2) % 3)             // step k + 2
      __syncthreads();
      IMC_GLOAD(rs[uu], min(k + 2 + NSETS, k_e - 1))
#pragma unroll
      for (int x = 0; x < WM; ++x) { falo[x] = nalo[x]; fahi[x] = nahi[x]; }
#pragma unroll
      for (int y = 0; y < WN; ++y) { fblo[y] = nblo[y]; fbhi[y] = nbhi[y]; }
    }
  }
#undef IMC_FRAGS
#undef IMC_GLOAD
#undef IMC_LSTORE

  // Epilogue: 32x32 block, lane l holds column l%32, register e holds row
  // 8*(e/4) + 4*(l/32) + e%4.
  uint16_t* out = args.out[vec];
#pragma unroll
  for (int x = 0; x < WM; ++x)
#pragma unroll
    for (int y = 0; y < WN; ++y) {
      const uint64_t col = uint64_t(t) * C::kBN + (wn * WN + y) * 32 + (lane & 31);
      if (col >= args.n) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t row = u * C::kBM + (wm * WM + x) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (row < args.rows) {
          const uint32_t z = uint32_t(acc0[x][y][e]) + (uint32_t(acc1[x][y][e]) << 8);
          if (SPLIT)
            args.part[((uint64_t(vec) * args.splits + part) * args.rows + row) * args.n + col] = z;
          else
            out[uint64_t(row) * args.ld + col] = uint16_t(z);
        }
      }
    }
  __syncthreads();   // the next tile's prologue reuses the LDS stages
  }
}

// ---------------------------------------------------------------------------
// Tiles of 64 NX rows x 128 entries on 16 x 16 x 64 MFMAs: 8 waves of 16 NX x
// 64, a K-step of 64 bytes of k per plane (two of the layout's half-steps),
// staged as 1 KB fragments [16 rows or entries][plane][16-byte piece 4][16]
// through three LDS stages of 24 (two workgroups a CU) to 48 KB.
//
// What bounds it: the database stream up to 64 rows (5.7 - 6.2 TB/s), above
// power (a register-only loop of this MFMA on random bytes runs at 4.0 POP/s,
// of the 32 x 32 x 32 one at 3.35).  us against 65,536 entries, dot_kernel's
// tiles of 32 x 32 x 32 MFMAs (64, 128 and 256 rows) / these: 64 rows 1,175 /
// 1,172, 65 rows 1,625 / 1,305, 100 1,683 / 1,440, 128 1,720 / 1,507, 192 2,582 / 1,860, 256 2,644
// / 2,290, 512 4,944 / 4,120 (3.1 POP/s), 768 7,340 / 6,245; 270 rows x 5,000
// entries 495 / 407.  One register set of loads in flight instead of two: 1 -
// 2 % slower.
constexpr int wide_stage(int nx) { return (64 * nx + 128) * 128; }

template <int K, int NX, bool SPLIT = false>
__global__ void __launch_bounds__(512, NX == 1 ? 4 : 1) dot_wide_kernel(DotArgs args) {
  using G = Geo<K>;
  constexpr int kStage = wide_stage(NX), kUnits = 2 + NX;
  extern __shared__ __align__(16) int8_t lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int vec = blockIdx.z;
  // the order of dot_kernel
  const uint32_t i = blockIdx.x;
  const uint32_t xcd = i & 7;
  const uint32_t ntp = SPLIT ? args.nt * args.splits : args.nt;
  const uint32_t s_end = ((ntp + 7) / 8) * args.mt;
  const uint32_t s_step = args.persistent ? (gridDim.x >> 3) : s_end;
  for (uint32_t s = i >> 3; s < s_end; s += s_step) {
  const uint32_t u = s % args.mt, tg = s / args.mt;
  const uint32_t tp = tg * 8 + xcd;
  if (tp >= ntp) continue;
  const uint32_t t = SPLIT ? tp / args.splits : tp, part = SPLIT ? tp % args.splits : 0;

  // A wave copies one plane of one half-step of NX 32-row blocks and two
  // 32-entry blocks, a lane a 16-byte piece of each.
  const int half = wave & 1, plane = (wave >> 1) & 1, slot = lane & 31;
  const int8_t* src[kUnits];
#pragma unroll
  for (int j = 0; j < kUnits; ++j) {
    const int blk = (wave >> 2) + 2 * j;
    const int8_t* base;
    if (j < NX) {
      const uint32_t rb = min(u * (2 * NX) + blk, args.a_blocks - 1);
      base = args.a + size_t(rb) * G::kBlockBytes;
    } else {
      const uint64_t cb = min(uint64_t(t) * 4 + (blk - 2 * NX), args.b_blocks - 1);
      base = args.b + size_t(args.b_block0 + cb) * G::kBlockBytes;
    }
    src[j] = base + size_t(2 * vec + plane) * G::kPlaneBlockBytes + half * 1024 + lane * 16;
  }
  const uint32_t dst = uint32_t(((wave >> 2) * 2 + (slot >> 4)) * 2048 + plane * 1024 +
                                (half * 2 + (lane >> 5)) * 256 + (slot & 15) * 16);

  v4i acc0[NX][4], acc1[NX][4];
#pragma unroll
  for (int e = 0; e < 4 * NX; ++e) acc0[e >> 2][e & 3] = acc1[e >> 2][e & 3] = v4i{0, 0, 0, 0};

  constexpr int kSteps = G::kChunks / 4;
  static_assert(kSteps % 2 == 0, "two K-steps per turn of the loop");
  const int k_b = SPLIT ? int(part * args.steps_per) : 0;
  const int k_e = SPLIT ? min(k_b + int(args.steps_per), kSteps) : kSteps;
  v4i rs[2][kUnits];
#define IMC_GLOAD(SET, C, STEP) \
  rs[SET][C] = *reinterpret_cast<const v4i*>(src[C] + size_t(min((STEP), k_e - 1)) * 2048);
#define IMC_LSTORE(SET, C, ST) *reinterpret_cast<v4i*>(lds + ((ST) + dst + (C) * 8192)) = rs[SET][C];
  v4i al[NX], ah[NX], fbl[2], fbh[2];
#define IMC_AFRAG(X, ST)                                                              \
  al[X] = *reinterpret_cast<const v4i*>(lds + ((ST) + wm * (2048 * NX) + (X) * 2048 + lane * 16)); \
  ah[X] = *reinterpret_cast<const v4i*>(lds + ((ST) + wm * (2048 * NX) + (X) * 2048 + 1024 + lane * 16));
#define IMC_BFRAG(Y, ST)                                                              \
  fbl[(Y) & 1] = *reinterpret_cast<const v4i*>(lds + ((ST) + 8192 * NX + wn * 8192 + (Y) * 2048 + lane * 16)); \
  fbh[(Y) & 1] = *reinterpret_cast<const v4i*>(lds + ((ST) + 8192 * NX + wn * 8192 + (Y) * 2048 + 1024 + lane * 16));

  // Pipeline: step j's bytes are loaded in step j - 4, written to LDS
  // stage j % 3 in step j - 2 and read in step j, the query fragments and the
  // first 16 entries' in the step before it.  The stage written in a step was
  // last read in the step before.
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int c = 0; c < kUnits; ++c) { IMC_GLOAD(0, c, k_b + h) }
#pragma unroll
    for (int c = 0; c < kUnits; ++c) { IMC_LSTORE(0, c, h * kStage) }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < kUnits; ++c) { IMC_GLOAD(h, c, k_b + 2 + h) }
  __syncthreads();
  uint32_t st0 = 0, st1 = kStage, st2 = 2 * kStage;      // stages of steps j, j + 1, j + 2
  // a wave whose rows are all past the last row only stages operands (not in
  // 256-row tiles, where a second loop costs 2 - 3 %)
  const bool live = NX == 4 || u * (64 * NX) + wm * (16 * NX) < args.rows;
  if (!live) {
    for (int k0 = k_b; k0 < k_e; k0 += 2) {
#pragma unroll
      for (int uu = 0; uu < 2; ++uu) {
#pragma unroll
        for (int c = 0; c < kUnits; ++c) {
          IMC_LSTORE(uu, c, st2)
          IMC_GLOAD(uu, c, k0 + uu + 4)
        }
        __syncthreads();
        const uint32_t st = st0;
        st0 = st1;
        st1 = st2;
        st2 = st;
      }
    }
  } else {
#pragma unroll
    for (int x = 0; x < NX; ++x) { IMC_AFRAG(x, 0) }
    IMC_BFRAG(0, 0)
    for (int k0 = k_b; k0 < k_e; k0 += 2) {
#pragma unroll
      for (int uu = 0; uu < 2; ++uu) {
        const int k = k0 + uu;
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          __builtin_amdgcn_sched_barrier(0);
          IMC_BFRAG((y + 1) & 3, y == 3 ? st1 : st0)
#pragma unroll
          for (int x2 = 0; x2 < NX; x2 += 2) {
#pragma unroll
            for (int e = 0; e < 6; ++e) {
              // two row blocks together: their high-limb products last
              const int x = x2 + (e < 4 ? e >> 1 : e & 1);
              if (x >= NX) continue;
              if (e >= 4)
                acc1[x][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah[x], fbl[y & 1], acc1[x][y], 0, 0, 0);
              else if (e & 1)
                acc0[x][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al[x], fbl[y & 1], acc0[x][y], 0, 0, 0);
              else
                acc1[x][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al[x], fbh[y & 1], acc1[x][y], 0, 0, 0);
            }
            if (y == 3) {
              IMC_AFRAG(x2, st1)
              if constexpr (NX > 1)
                if (x2 + 1 < NX) { IMC_AFRAG(x2 + 1, st1) }
            }
          }
          if (y < 3) {
#pragma unroll
            for (int c = 2 * y; c < min(2 * y + 2, kUnits); ++c) {
              IMC_LSTORE(uu, c, st2)
              IMC_GLOAD(uu, c, k + 4)
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        const uint32_t st = st0;
        st0 = st1;
        st1 = st2;
        st2 = st;
      }
    }
  }
#undef IMC_GLOAD
#undef IMC_LSTORE
#undef IMC_AFRAG
#undef IMC_BFRAG

  // 16 x 16 block: lane l holds column l % 16, register e row 4 (l / 16) + e
  uint16_t* out = args.out[vec];
#pragma unroll
  for (int x = 0; x < NX; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const uint64_t col = uint64_t(t) * 128 + wn * 64 + y * 16 + (lane & 15);
      if (col >= args.n) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t row = u * (64 * NX) + (wm * NX + x) * 16 + 4 * (lane >> 4) + e;
        if (row < args.rows) {
          const uint32_t z = uint32_t(acc0[x][y][e]) + (uint32_t(acc1[x][y][e]) << 8);
          if (SPLIT)
            args.part[((uint64_t(vec) * args.splits + part) * args.rows + row) * args.n + col] = z;
          else
            out[uint64_t(row) * args.ld + col] = uint16_t(z);
        }
      }
    }
  __syncthreads();   // the next tile's prologue reuses the LDS stages
  }
}

hipError_t launch_expand(const int8_t* qop, const uint32_t* qidx, uint32_t q, uint32_t r, const int8_t* rot, int8_t* a,
                         uint32_t rows_pad, hipStream_t s, bool galois) {
  Rot rr;
  for (int i = 0; i < IMC_MAX_ROT_DEV; ++i) rr.s[i] = i < int(r) ? rot[i] : 0;
  const uint64_t chunks = galois ? Geo<kKGalois>::kChunks : Geo<kK>::kChunks;
  const uint64_t total = uint64_t(rows_pad) * kPlanes * chunks;
  if (!fits_grid(total, 256)) return hipErrorInvalidValue;
  const dim3 grid(unsigned((total + 255) / 256));
  if (galois)
    hipLaunchKernelGGL(expand_kernel<kKGalois>, grid, dim3(256), 0, s, qop, qidx, q, r, rr, rows_pad, a);
  else
    hipLaunchKernelGGL(expand_kernel<kK>, grid, dim3(256), 0, s, qop, qidx, q, r, rr, rows_pad, a);
  return hipGetLastError();
}

// Adds the parts of a split K loop: u32 [vec][split][rows][n] -> u16 [rows][ld] per vector.
__global__ void __launch_bounds__(256) reduce_parts_kernel(const uint32_t* __restrict__ part, uint32_t splits,
                                                           uint64_t count, uint64_t n, uint16_t* code, uint16_t* mask,
                                                           uint64_t ld) {
  const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint32_t* p = part + uint64_t(blockIdx.z) * splits * count + i;
  uint32_t z = 0;
#pragma unroll 4
  for (uint32_t k = 0; k < splits; ++k) z += p[k * count];
  (blockIdx.z ? mask : code)[i / n * ld + i % n] = uint16_t(z);
}

hipError_t launch_reduce_parts(const DotScratch& scratch, uint32_t splits, uint64_t rows, uint64_t n, uint16_t* code,
                               uint16_t* mask, uint64_t ld, hipStream_t s) {
  const uint64_t count = rows * n;
  if (!fits_grid(count, 256)) return hipErrorInvalidValue;
  // The launch records the event itself: 64 queries x 31 rotations x 64 entries
  // take 43.5 us with it and without one (2 us more where each call is waited
  // for), 45.2 with a record of its own, 45.5 with a system-scope fence.
  const uint32_t* part = scratch.part;
  void* args[] = {&part, &splits, const_cast<uint64_t*>(&count), &n, &code, &mask, &ld};
  return hipExtLaunchKernel(reinterpret_cast<const void*>(reduce_parts_kernel),
                            dim3(unsigned((count + 255) / 256), 1, mask ? 2 : 1), dim3(256), args, 0, s, nullptr,
                            scratch.done, 0);
}

// One launch of a kernel, whole or split, of bm x bn tiles.
using DotKernel = void (*)(DotArgs);
static hipError_t launch_tiles(DotKernel kern, DotKernel split, uint32_t bm, uint32_t bn, uint32_t threads, size_t lds,
                               uint32_t steps, uint32_t piece, DotArgs d, uint32_t rows, uint64_t n, hipStream_t s,
                               bool persistent, const DotScratch& scratch, uint32_t per_cu) {
  d.mt = (rows + bm - 1) / bm;
  d.nt = uint32_t((n + bn - 1) / bn);
  const uint32_t ntg = (d.nt + 7) / 8;
  if (uint64_t(ntg) * 8 * d.mt > 0x7FFFFFFFull) return hipErrorInvalidValue;
  uint32_t blocks = ntg * 8 * d.mt;
  d.persistent = 0;
  if (persistent) {
    // one resident workgroup per CU (two waves per SIMD)
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const uint32_t want = uint32_t(((cus + 7) / 8) * 8);
    if (want < blocks) {
      blocks = want;
      d.persistent = 1;
    }
  }
  const dim3 grid(blocks, 1, d.out[1] ? 2 : 1);   // z: code, mask (no mask dot when masks are public)
  // Split the K loop while CUs are left over, in pieces of `piece` steps (whole
  // turns of the loop): a call of few tiles takes as long as one workgroup's
  // loop.  1 row x 100 entries 428 -> 18 us, 33 rows x 5,000 entries 448 -> 139.
  const uint32_t pieces = steps / piece;
  const uint32_t splits =
      dot_splits(uint64_t(d.mt) * d.nt * grid.z, per_cu, pieces, uint64_t(rows) * n * grid.z, scratch);
  if (splits > 1) {
    d.steps_per = (pieces + splits - 1) / splits * piece;
    d.splits = (steps + d.steps_per - 1) / d.steps_per;
    d.part = scratch.part;
    d.persistent = 0;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(split),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e == hipSuccess) e = scratch.begin(s);
    if (e != hipSuccess) return e;
    const uint32_t ntp = (d.nt * d.splits + 7) / 8 * 8;
    hipLaunchKernelGGL(split, dim3(ntp * d.mt, 1, grid.z), dim3(threads), lds, s, d);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_reduce_parts(scratch, d.splits, rows, n, d.out[0], d.out[1], d.ld, s);
  }
  d.splits = d.steps_per = 0;
  d.part = nullptr;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, grid, dim3(threads), lds, s, d);
  return hipGetLastError();
}

template <int K, int WM, int WN, int WAVES_M, int WAVES_N, int NSETS>
static hipError_t launch_dot_cfg(const DotArgs& d, uint32_t rows, uint64_t n, hipStream_t s, bool persistent,
                                 const DotScratch& scratch) {
  using C = DotCfg<WM, WN, WAVES_M, WAVES_N>;
  static_assert(10 % NSETS == 0, "a piece is whole unrolled iterations");
  return launch_tiles(dot_kernel<K, WM, WN, WAVES_M, WAVES_N, NSETS>,
                      dot_kernel<K, WM, WN, WAVES_M, WAVES_N, NSETS, true>, C::kBM, C::kBN, C::kThreads,
                      3 * size_t(C::kStageBytes), Geo<K>::kChunks / 2, 10, d, rows, n, s, persistent, scratch, 1);
}

template <int K, int NX>
static hipError_t launch_dot_wide(const DotArgs& d, uint32_t rows, uint64_t n, hipStream_t s, bool persistent,
                                  const DotScratch& scratch) {
  return launch_tiles(dot_wide_kernel<K, NX>, dot_wide_kernel<K, NX, true>, 64 * NX, 128, 512,
                      3 * size_t(wide_stage(NX)), Geo<K>::kChunks / 4, 10, d, rows, n, s, persistent, scratch,
                      NX == 1 ? 2 : 1);
}

hipError_t launch_expand_rows(const int8_t* qop, uint32_t q, const imc_row* rows, uint32_t nrows, int8_t* a,
                              uint32_t rows_pad, hipStream_t s, bool galois) {
  const uint64_t chunks = galois ? Geo<kKGalois>::kChunks : Geo<kK>::kChunks;
  const uint64_t total = uint64_t(rows_pad) * kPlanes * chunks;
  if (!fits_grid(total, 256)) return hipErrorInvalidValue;
  const dim3 grid(unsigned((total + 255) / 256));
  if (galois)
    hipLaunchKernelGGL(expand_rows_kernel<kKGalois>, grid, dim3(256), 0, s, qop, q, rows, nrows, rows_pad, a);
  else
    hipLaunchKernelGGL(expand_rows_kernel<kK>, grid, dim3(256), 0, s, qop, q, rows, nrows, rows_pad, a);
  return hipGetLastError();
}

template <int K>
static hipError_t launch_dot_k(DotArgs d, uint32_t rows, uint64_t n, hipStream_t s, int variant,
                               const DotScratch& scratch) {
  const bool persistent = (variant & IMC_DOT_PERSISTENT) != 0;
  switch (variant & 0xF) {
    case 2: return launch_dot_cfg<K, 2, 2, 2, 2, 2>(d, rows, n, s, persistent, scratch);    // 128 x 128, 4 waves of 64 x 64
    case 3: return launch_dot_cfg<K, 2, 2, 4, 2, 1>(d, rows, n, s, persistent, scratch);    // 256 x 128, loads 3 steps ahead
    default: break;
  }
  // Few rows: the database stream bounds the call, and a tile of more rows
  // spends its steps on empty ones.  us against 65,536 entries, 256-row / these
  // tiles: 1 row 2,158 / 1,075, 64 rows 2,484 / 1,172, 65 rows 2,190 / 1,305, 128
  // rows 2,290 / 1,507, 150 rows 2,140 / 1,860; 200 rows 2,165 (192-row tiles
  // would be two).
  if (!persistent && rows <= 64) return launch_dot_wide<K, 1>(d, rows, n, s, false, scratch);
  if (!persistent && rows <= 128) return launch_dot_wide<K, 2>(d, rows, n, s, false, scratch);
  if (!persistent && rows <= 192) return launch_dot_wide<K, 3>(d, rows, n, s, false, scratch);
  // Up to 128 rows past the last whole 256-row tile go in a launch of those
  // tiles, once there is a tile for every CU (fewer split their loop).  us, one
  // launch / two, with 256-row tiles as they were: 320 rows x 65,536 entries
  // 4,675 / 3,797, 384 x 30,001 2,321 / 2,014, 260 x 20,000 1,563 / 1,479.
  const uint32_t whole = rows / 256 * 256, rest = rows - whole;
  const uint64_t tiles = (n + 127) / 128 * (rows / 256) * (d.out[1] ? 2 : 1);
  if (!persistent && whole != 0 && rest != 0 && rest <= 128 && tiles >= uint64_t(scratch.cus)) {
    d.rows = whole;
    const hipError_t e = launch_dot_wide<K, 4>(d, whole, n, s, false, scratch);
    if (e != hipSuccess) return e;
    d.a += size_t(whole / 32) * Geo<K>::kBlockBytes;
    d.a_blocks -= whole / 32;
    d.rows = rest;
    for (uint16_t*& o : d.out)
      if (o) o += uint64_t(whole) * d.ld;
    return rest <= 64 ? launch_dot_wide<K, 1>(d, rest, n, s, false, scratch)
                      : launch_dot_wide<K, 2>(d, rest, n, s, false, scratch);
  }
  return launch_dot_wide<K, 4>(d, rows, n, s, persistent, scratch);
}

hipError_t launch_dot(const int8_t* a, uint32_t rows, uint32_t a_blocks, const int8_t* b, uint64_t first_entry,
                      uint64_t n, uint16_t* code, uint16_t* mask, uint64_t ld, hipStream_t s, int variant,
                      bool galois, const DotScratch& scratch) {
  if (rows == 0 || n == 0) return hipSuccess;
  DotArgs d;
  d.a = a;
  d.b = b;
  d.out[0] = code;
  d.out[1] = mask;
  d.ld = ld;
  d.rows = rows;
  d.a_blocks = a_blocks;
  d.b_block0 = first_entry / 32;
  d.b_blocks = (n + 31) / 32;
  d.n = n;
  return galois ? launch_dot_k<kKGalois>(d, rows, n, s, variant, scratch)
                : launch_dot_k<kK>(d, rows, n, s, variant, scratch);
}

}  // namespace imc
