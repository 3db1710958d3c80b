// rot_dot.hip -- rotation-aware variant of the party-local dot products
// (Alg. 3; App. C).  Same arithmetic as the expanded kernel (balanced byte
// limbs, i8 MFMA with i32 accumulation, three products into two
// accumulators); the query rotations (Sec. 3: circular shifts of the
// angular axis, party-local because sharing is elementwise) are applied
// while reading the query operand from LDS instead of being materialised.
#include <algorithm>

#include "device.h"
#include "launch.h"

namespace imc {

// ---------------------------------------------------------------------------
// Rotation-aware dot kernel.  Rows are (query, rotation) pairs, so a 256-row
// tile holds only ceil(256/R) + 1 distinct queries.  The K loop walks the 32
// angular-row segments of 800 bytes (16 rows x 2 halves); for each segment the
// workgroup keeps every tile query's bytes of that segment in LDS with 64
// bytes of circular padding on both sides (928 B per plane), and a lane reads
// its rotated fragment directly: rotation s shifts the segment by 4s bytes,
// so the 16 bytes at (32t + 16g - 4s) are four aligned dword reads.  Only the
// database operand streams through LDS per K-step.  Query segments are loaded
// into registers one segment ahead and written into the other of two LDS
// buffers half-way through the current segment.
//
// What bounds it: power (and up to 64 rows, memory).  On random bytes a
// register-only loop of 16 x 16 x 64 MFMAs runs at 4.0 POP/s on this part, one
// of 32 x 32 x 32 at 3.35; 64 queries of 31 rotations against 300,000 entries run
// at 2.0 GHz with the MFMA pipes 0.64 busy and the LDS 0.49, a fifth of that bank
// conflicts of the rotated query reads.  One party's dots against 65,536 entries,
// ms, with 32 x 32 x 32 MFMAs and 64 rows per wave at any row count / as it
// stands: 1 query of 31 rotations 1.15 / 1.08 (6.2 GB/ms), 12 of 15: 2.03 / 1.78,
// 40 of 15: 5.90 / 5.34, 70 of 15: 9.56 / 8.67, 64 of 24: 12.2 / 11.3.
// Scheduling groups that spread the LDS reads over the MFMAs, and slot strides
// that keep two queries' rows in different banks, change nothing.  The next
// step's query fragments are read under the last two of its four groups of
// MFMAs: all of them under the last one left a launch of one tile per CU waiting
// at the barrier (19 queries of 13 rotations x 64 entries, 256-row tiles: 409 us,
// then 391; 40 of 15 x 65,536, on one box: 5.48 ms, then 5.34).
// ---------------------------------------------------------------------------
struct RotDotArgs {
  const int8_t* qop;     // unrotated query operand, row-major [q][plane 4][K]
  const uint32_t* qidx;  // optional: query i of the call is operand row qidx[i]
  const int8_t* b;       // party's database region
  uint16_t* out[2];
  uint64_t ld;
  uint32_t rows, q, r;
  uint64_t b_block0, b_blocks, n;
  uint32_t mt, nt;
  uint32_t lead;         // row tiles that share their column tiles' order; the last one follows if it is not of them
  uint32_t tile_m;       // rows of a tile: kRotM, fewer where a launch has few tiles
  uint32_t max_q;        // query slots per tile (LDS sizing)
  uint32_t splits, seg_per;   // split launches: workgroups per tile, segments of each
  uint32_t* part;        // split launches: u32 [vec][split][rows][n]
  int8_t rot[IMC_MAX_ROT_DEV];
};

// Waits and barriers with explicit counts (the kernels below keep copies and
// reads in flight across them).
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  // gfx9 s_waitcnt: vmcnt bits 3:0 and 15:14, expcnt 6:4 (7 = no wait), lgkmcnt 11:8 (15 = no wait)
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Wait for every outstanding LDS read (and nothing else).
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (0 << 8));
}

__device__ __forceinline__ void bar() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void copy16(const int8_t* g, int8_t* l) {
  __builtin_amdgcn_global_load_lds(static_cast<const void*>(g), (__attribute__((address_space(3))) void*)(l), 16, 0,
                                   0);
}

// What one output tile of the rotation-aware kernel reads and writes: the
// call's (or group's) unrotated query operand, its rotation list, the
// database region and the output plane of vector `vec`.
struct RotTile {
  const int8_t* qop;
  const uint32_t* qidx;
  const int8_t* b;
  uint16_t* out;
  const int8_t* rot;
  uint64_t ld, b_block0, b_blocks, n;
  uint32_t rows, r, max_q, tile_m;
  int seg_begin, seg_end;      // SPLIT: the tile's share of the angular-row segments
  uint32_t* part;              // SPLIT: where its sums go, u32 [rows][n]
};

// One 256 x 128 output tile (row tile u, column tile t) of vector `vec`,
// the whole K loop (SPLIT: some of its segments) and the epilogue: 8 waves of
// 64 x 64.  LDS: 3 database stages, then the two query segment buffers of
// max_q slots.
//
// A K-step is two of the 32-byte database steps (64 bytes of k), one
// 16 x 16 x 64 MFMA for each product of 16 rows and 16 entries.  A segment is
// 25 of the half-steps, so every second segment starts with the second half of
// a K-step: each lane takes its half's query bytes from the buffer and offset
// of that half's segment.
constexpr int kRotM = 256, kRotN = 128, kRotThreads = 512;
constexpr int kRotStage = kRotN * 128;                         // one K-step: 2 limbs x 64 B per entry
constexpr int kSegSteps = kRowLen / 32;                        // 25 half-steps per segment

template <int K, int ACH, int NX, bool SPLIT>
__device__ __forceinline__ void rot_dot_rows(const RotTile& args, uint32_t u, uint32_t t, int vec, int8_t* lds) {
  using G = Geo<K>;
  constexpr int kHalves = G::kChunks / 2;                      // 800 or 400
  static_assert(kHalves % 4 == 0, "two K-steps per turn of the loop");
  int8_t* ast = lds + 3 * kRotStage;                           // 2 A segment buffers
  const uint32_t abuf = args.max_q * 2 * kSegBytes;            // bytes per A buffer

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  const uint32_t m0 = u * args.tile_m;
  const uint32_t q_lo = m0 / args.r;
  const uint32_t last_row = min(m0 + args.tile_m, args.rows) - 1;
  const uint32_t nq = last_row / args.r - q_lo + 1;            // <= max_q

  const int seg_b = SPLIT ? args.seg_begin : 0, seg_e = SPLIT ? args.seg_end : kHalves / kSegSteps;
  const int k_b = seg_b * kSegSteps, k_e = seg_e * kSegSteps;  // in half-steps
  // a split part's last turn may reach past its end: zeros there
  const int steps = SPLIT ? (k_e - k_b + 3) / 4 * 2 : kHalves / 2;

  // Per-lane A fragment offsets (bytes into an A buffer) for its four 16-row blocks.
  int a_off[NX];
#pragma unroll
  for (int x = 0; x < NX; ++x) {
    const uint32_t row = m0 + (wm * NX + x) * 16 + (lane & 15);
    int slot = 0, sft = 0;
    if (row < args.rows) {
      slot = int(row / args.r - q_lo);
      sft = 4 * args.rot[row % args.r];
    }
    a_off[x] = slot * 2 * kSegBytes + kSegPad - sft + 16 * ((lane >> 4) & 1);
  }
  const bool second = (lane & 32) != 0;                        // this lane's half of a K-step

  // B staging: a wave copies one limb of one half-step, two 32-entry blocks
  const int b_half = wave & 1, b_limb = (wave >> 1) & 1;
  const int8_t* bsrc[2];
  uint32_t bdst[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int blk = (wave >> 2) + 2 * j, slot = lane & 31;
    uint64_t cb = uint64_t(t) * (kRotN / 32) + blk;
    cb = cb < args.b_blocks ? cb : args.b_blocks - 1;
    bsrc[j] = args.b + size_t(args.b_block0 + cb) * G::kBlockBytes + size_t(2 * vec + b_limb) * G::kPlaneBlockBytes +
              lane * 16;
    bdst[j] = uint32_t(((blk * 2 + (slot >> 4)) * 2 + b_limb) * 1024 + (b_half * 2 + (lane >> 5)) * 256 +
                       (slot & 15) * 16);
  }
  // A staging: chunk c of a segment buffer = (query slot, plane, 16-byte piece).
  const int a_chunks = int(nq) * 2 * kSegChunks;
  const int8_t* asrc[ACH];
  int adst[ACH];
#pragma unroll
  for (int j = 0; j < ACH; ++j) {
    int c = tid + j * kRotThreads;
    const bool ok = c < a_chunks;
    c = ok ? c : 0;
    const int qs = c / (2 * kSegChunks), rem = c % (2 * kSegChunks);
    const int pl = rem / kSegChunks, piece = rem % kSegChunks;
    const int src_off = ((piece * 16 - kSegPad) % kRowLen + kRowLen) % kRowLen;   // circular
    const uint32_t qrow = args.qidx ? args.qidx[q_lo + qs] : q_lo + qs;
    asrc[j] = args.qop + size_t(qrow) * G::kQopRowBytes + size_t(2 * vec + pl) * G::kK + src_off;
    adst[j] = ok ? (qs * 2 * kSegBytes + pl * kSegBytes + piece * 16) : -1;
  }

  v4i acc0[NX][4], acc1[NX][4];
#pragma unroll
  for (int i = 0; i < 4 * NX; ++i) acc0[i >> 2][i & 3] = acc1[i >> 2][i & 3] = v4i{0, 0, 0, 0};

  v4i rs[2][2];     // database bytes in flight: step j in set j % 2
  v4i ra[ACH];
#define IMC_BLOAD(SET, STEP)                                                          \
  {                                                                                   \
    const int k_ = min(k_b + 2 * (STEP) + b_half, k_e - 1);                           \
    _Pragma("unroll") for (int c_ = 0; c_ < 2; ++c_)                                  \
        rs[SET][c_] = *reinterpret_cast<const v4i*>(bsrc[c_] + size_t(k_) * 1024);    \
  }
#define IMC_BSTORE(SET, STEP, ST)                                                     \
  _Pragma("unroll") for (int c_ = 0; c_ < 2; ++c_) {                                  \
    v4i v_ = rs[SET][c_];                                                             \
    if (SPLIT && k_b + 2 * (STEP) + b_half >= k_e) v_ = v4i{0, 0, 0, 0};              \
    *reinterpret_cast<v4i*>(lds + ((ST) + bdst[c_])) = v_;                            \
  }
#define IMC_ALOAD(SEG)                                                                \
  _Pragma("unroll") for (int c_ = 0; c_ < ACH; ++c_)                                  \
      ra[c_] = *reinterpret_cast<const v4i*>(asrc[c_] + size_t(SEG) * kRowLen);
#define IMC_ASTORE(BUF)                                                               \
  _Pragma("unroll") for (int c_ = 0; c_ < ACH; ++c_)                                  \
      if (adst[c_] >= 0) *reinterpret_cast<v4i*>(ast + (BUF) * abuf + adst[c_]) = ra[c_];

  // Pipeline: step j's database bytes are loaded in step j - 4, written to
  // LDS stage j % 3 in step j - 2 and read in step j (the first 16 entries'
  // and the query fragments in the step before it).  The stage written in a
  // step was last read in the step before.
  v4i al[NX], ah[NX], fbl[2], fbh[2];
  // byte offset, in the query buffers, of this lane's half of K-step STEP
  const auto a_step = [&](int step) __attribute__((always_inline)) {
    const int k0 = min(k_b + 2 * step, k_e - 1), k1 = min(k_b + 2 * step + 1, k_e - 1);
    const int s0 = k0 / kSegSteps, s1 = k1 / kSegSteps;
    const uint32_t o0 = (s0 & 1) * abuf + 32 * (k0 - s0 * kSegSteps);
    const uint32_t o1 = (s1 & 1) * abuf + 32 * (k1 - s1 * kSegSteps);
    return second ? o1 : o0;
  };
#define IMC_AFRAG(LO, HI, X, OFF)                                                     \
  {                                                                                   \
    const int32_t* pl_ = reinterpret_cast<const int32_t*>(ast + ((OFF) + a_off[X]));  \
    const int32_t* ph_ = pl_ + kSegBytes / 4;                                         \
    LO[X] = v4i{pl_[0], pl_[1], pl_[2], pl_[3]};                                      \
    HI[X] = v4i{ph_[0], ph_[1], ph_[2], ph_[3]};                                      \
  }
#define IMC_BFRAG(Y, ST)                                                              \
  fbl[(Y) & 1] = *reinterpret_cast<const v4i*>(lds + ((ST) + wn * 8192 + (Y) * 2048 + lane * 16)); \
  fbh[(Y) & 1] = *reinterpret_cast<const v4i*>(lds + ((ST) + wn * 8192 + (Y) * 2048 + 1024 + lane * 16));

  IMC_ALOAD(seg_b)
  IMC_ASTORE(seg_b & 1)
  IMC_BLOAD(0, 0)
  IMC_BLOAD(1, 1)
  IMC_BSTORE(0, 0, 0)
  IMC_BSTORE(1, 1, kRotStage)
  IMC_BLOAD(0, 2)
  IMC_BLOAD(1, 3)
  IMC_ALOAD(min(seg_b + 1, seg_e - 1))
  __syncthreads();
  // a wave whose rows are all past the last row (the partial last row tile)
  // only stages operands for the others: no fragment reads, no MFMAs
  const bool live = m0 + uint32_t(wm * NX * 16) < args.rows;
  uint32_t st0 = 0, st1 = kRotStage, st2 = 2 * kRotStage;      // stages of steps j, j + 1, j + 2
  // the next segment's query bytes go to the other A buffer (last read at the
  // end of the previous segment) in the middle of this one
#define IMC_TURN(STEP)                                                                \
  {                                                                                   \
    const int k_ = k_b + 2 * (STEP), seg_ = k_ / kSegSteps;                           \
    if (((k_ - seg_ * kSegSteps + 1) >> 1) == 6 && seg_ + 1 < seg_e) {                \
      IMC_ASTORE((seg_ + 1) & 1)                                                      \
      IMC_ALOAD(min(seg_ + 2, seg_e - 1))                                             \
    }                                                                                 \
    __syncthreads();                                                                  \
    const uint32_t st_ = st0;                                                         \
    st0 = st1;                                                                        \
    st1 = st2;                                                                        \
    st2 = st_;                                                                        \
  }
  if (!live) {
    for (int j0 = 0; j0 < steps; j0 += 2) {
#pragma unroll
      for (int uu = 0; uu < 2; ++uu) {
        IMC_BSTORE(uu, j0 + uu + 2, st2)
        IMC_BLOAD(uu, j0 + uu + 4)
        IMC_TURN(j0 + uu)
      }
    }
  } else {
    {
      const uint32_t o = a_step(0);
#pragma unroll
      for (int x = 0; x < NX; ++x) { IMC_AFRAG(al, ah, x, o) }
      IMC_BFRAG(0, 0)
    }
    for (int j0 = 0; j0 < steps; j0 += 2) {
#pragma unroll
      for (int uu = 0; uu < 2; ++uu) {
        const int j = j0 + uu;
        const uint32_t a_next = a_step(j + 1);
        v4i nl[NX], nh[NX];
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          __builtin_amdgcn_sched_barrier(0);
          IMC_BFRAG((y + 1) & 3, y == 3 ? st1 : st0)
          if (y >= 2) {
#pragma unroll
            for (int x = (y - 2) * NX / 2; x < (y - 1) * NX / 2; ++x) { IMC_AFRAG(nl, nh, x, a_next) }
          }
#pragma unroll
          for (int x2 = 0; x2 < NX; x2 += 2)
#pragma unroll
            for (int i = 0; i < 6; ++i) {
              // two row blocks together: their high-limb products last
              const int x = x2 + (i < 4 ? i >> 1 : i & 1);
              if (x >= NX) continue;
              if (i >= 4)
                acc1[x][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah[x], fbl[y & 1], acc1[x][y], 0, 0, 0);
              else if (i & 1)
                acc0[x][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al[x], fbl[y & 1], acc0[x][y], 0, 0, 0);
              else
                acc1[x][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al[x], fbh[y & 1], acc1[x][y], 0, 0, 0);
            }
          if (y == 0) {
            IMC_BSTORE(uu, j + 2, st2)
            IMC_BLOAD(uu, j + 4)
          }
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int x = 0; x < NX; ++x) { al[x] = nl[x]; ah[x] = nh[x]; }
        IMC_TURN(j)
      }
    }
  }
#undef IMC_TURN
#undef IMC_AFRAG
#undef IMC_BFRAG
#undef IMC_BLOAD
#undef IMC_BSTORE
#undef IMC_ALOAD
#undef IMC_ASTORE

  // 16 x 16 block: lane l holds column l % 16, register e row 4 (l / 16) + e
  uint16_t* out = args.out;
#pragma unroll
  for (int x = 0; x < NX; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const uint64_t col = uint64_t(t) * kRotN + wn * 64 + y * 16 + (lane & 15);
      if (col >= args.n) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t row = m0 + (wm * NX + x) * 16 + 4 * (lane >> 4) + e;
        if (row < args.rows) {
          const uint32_t z = uint32_t(acc0[x][y][e]) + (uint32_t(acc1[x][y][e]) << 8);
          if (SPLIT)
            args.part[uint64_t(row) * args.n + col] = z;
          else
            out[uint64_t(row) * args.ld + col] = uint16_t(z);
        }
      }
    }
}

// A last row tile of few rows spreads them over all the waves, 16, 32 or 48
// each: with 64 a wave, a tile of 31 rows is one live wave pair on two of the
// four SIMDs.  us, 64 rows a wave / spread, 65,536 entries: 1 query of 31
// rotations 1,299 / 1,079, 4 of 15: 1,199 / 1,138, 12 of 15: 1,930 / 1,847.
// Where a launch has fewer tiles than CUs (rot_tile_rows), its tiles are of 64,
// 128 or 192 rows: a call whose loop is not split (captured, another
// stream, groups) takes as long as one tile.  us, 256-row tiles / these: 64
// queries of 31 x 64 entries 385 / 258, 19 of 13 x 64: 408 / 200, 8 of 31 x 2,000:
// 384 / 195, 12 of 15 x 8,000: 333 / 306; groups of 20 queries of 13 and 3 of 22
// x 5,000 entries 439 / 328.
template <int K, int ACH, bool SPLIT = false>
__device__ __forceinline__ void rot_dot_tile(const RotTile& args, uint32_t u, uint32_t t, int vec, int8_t* lds) {
  const uint32_t rows = min(args.rows - u * args.tile_m, args.tile_m);
  if (rows > 192)
    rot_dot_rows<K, ACH, 4, SPLIT>(args, u, t, vec, lds);
  else if (rows > 128)
    rot_dot_rows<K, ACH, 3, SPLIT>(args, u, t, vec, lds);
  else if (rows > 64)
    rot_dot_rows<K, ACH, 2, SPLIT>(args, u, t, vec, lds);
  else
    rot_dot_rows<K, ACH, 1, SPLIT>(args, u, t, vec, lds);
}

// One launch per call: workgroup i is output tile (u, t) in an XCD-aware
// order (consecutive workgroups go to the 8 XCDs in turn; each XCD walks
// every row tile of its column tiles, so a column tile's database bytes are
// read into one XCD's L2).
template <int K, int ACH>
__global__ void __launch_bounds__(kRotThreads) rot_dot_kernel(RotDotArgs args) {
  extern __shared__ __align__(16) int8_t lds[];
  const int vec = blockIdx.z;
  const uint32_t i = blockIdx.x;
  const uint32_t first = (args.nt + 7) / 8 * 8 * args.lead;    // workgroups of the leading row tiles
  uint32_t u = args.lead, t = i - first;
  if (i < first) {
    const uint32_t xcd = i & 7, s8 = i >> 3;
    u = s8 % args.lead;
    t = s8 / args.lead * 8 + xcd;
  }
  if (t >= args.nt) return;
  const RotTile tile{args.qop, args.qidx, args.b, args.out[vec], args.rot, args.ld, args.b_block0, args.b_blocks,
                     args.n, args.rows, args.r, args.max_q, args.tile_m, 0, 0, nullptr};
  rot_dot_tile<K, ACH>(tile, u, t, vec, lds);
}

// The same with a tile's segments split over args.splits workgroups, for
// calls with fewer tiles than CUs: their time is that of one workgroup's
// serial K loop, 0.5 us a step with up to 64 rows and 1.0 with all 256 (400
// steps), at whatever size.  Each part's sums go to scratch as u32 and
// reduce_parts_kernel adds them.  31 rows x 1,000 entries: 209 -> 25 us;
// 1,984 rows x 64 entries: 394 -> 43 us; 93 rows x 4,000: 244 -> 90.
template <int K, int ACH>
__global__ void __launch_bounds__(kRotThreads) rot_dot_split_kernel(RotDotArgs args) {
  using G = Geo<K>;
  extern __shared__ __align__(16) int8_t lds[];
  const int vec = blockIdx.z;
  // (column tile, part) pairs take the place of column tiles in the XCD-aware order
  const uint32_t i = blockIdx.x;
  const uint32_t xcd = i & 7, s8 = i >> 3;
  const uint32_t u = s8 % args.mt, tp = (s8 / args.mt) * 8 + xcd;
  if (tp >= args.nt * args.splits) return;
  const uint32_t t = tp / args.splits, part = tp % args.splits;
  constexpr int kSegs = G::kChunks / 2 / kSegSteps;
  const RotTile tile{args.qop, args.qidx, args.b, nullptr, args.rot, args.ld, args.b_block0, args.b_blocks,
                     args.n, args.rows, args.r, args.max_q, args.tile_m, int(part * args.seg_per),
                     min(int((part + 1) * args.seg_per), kSegs),
                     args.part + (uint64_t(vec) * args.splits + part) * args.rows * args.n};
  rot_dot_tile<K, ACH, true>(tile, u, t, vec, lds);
}

// ---------------------------------------------------------------------------
// Several query groups in one launch (uneven batches: each group is the
// queries of one rotation list, e.g. the batches checked at 31 rotations and
// those at 15).  Group g owns global tiles [tile0, tile0 + 8 * ntg * mt) and
// maps them to its (row tile, column tile) pairs exactly as one launch of
// rot_dot_kernel would, so every group keeps the XCD-aware order.  With a
// persistent grid (a multiple of 8 workgroups, fewer than the tiles) each
// workgroup walks tiles i, i + grid, ...: the same residue mod 8, so the
// same XCD, as a one-tile-per-workgroup launch would give them.
// ---------------------------------------------------------------------------
constexpr int kMaxDotGroups = IMC_MAX_DOT_GROUPS;
struct RotGroup {
  const int8_t* qop;
  uint16_t* out[2];
  uint32_t rows, r, mt, tile0;
  int8_t rot[IMC_MAX_ROT_DEV];
};
struct RotGroupsArgs {
  const int8_t* b;
  uint64_t ld, b_block0, b_blocks, n;
  uint32_t nt, ntiles, ngroups, max_q, tile_m;
  RotGroup g[kMaxDotGroups];
};

template <int K, int ACH>
__global__ void __launch_bounds__(kRotThreads) rot_dot_groups_kernel(RotGroupsArgs args) {
  extern __shared__ __align__(16) int8_t lds[];
  const int vec = blockIdx.z;
  bool first = true;
  for (uint32_t i = blockIdx.x; i < args.ntiles; i += gridDim.x) {
    uint32_t gi = 0;
    while (gi + 1 < args.ngroups && i >= args.g[gi + 1].tile0) ++gi;
    const RotGroup& grp = args.g[gi];
    const uint32_t li = i - grp.tile0;
    const uint32_t xcd = li & 7, s8 = li >> 3;
    const uint32_t u = s8 % grp.mt, tg = s8 / grp.mt;
    const uint32_t t = tg * 8 + xcd;
    if (t >= args.nt) continue;
    // the previous tile's last fragment reads end before this tile's prologue
    // overwrites the LDS stages
    if (!first) __syncthreads();
    first = false;
    const RotTile tile{grp.qop, nullptr, args.b, grp.out[vec], grp.rot, args.ld, args.b_block0, args.b_blocks,
                       args.n, grp.rows, grp.r, args.max_q, args.tile_m, 0, 0, nullptr};
    rot_dot_tile<K, ACH>(tile, u, t, vec, lds);
  }
}

// The query slots of a 256-row tile (ceil(256 / r) + 1 of them) must fit the
// A staging of the configuration: 3 chunks per thread up to 13 queries (r >= 22),
// 5 up to 22 queries (r >= 13, default configuration only).
bool rot_dot_applies(uint32_t r, int kind) { return kind == 0 ? r >= 13 : r >= 22; }

// ---------------------------------------------------------------------------
// The same rotation-aware tiling with the database fragments loaded by every
// wave straight from HBM (through its L1/L2) into registers D K-steps ahead:
// a fragment is 1 KB contiguous in the tiled layout, and the WAVES_M waves
// that share a column block hit the same lines.  Only the query segments go
// through LDS, so there is no per-step barrier: two per 25-step segment,
// around the store of the next segment into the other A buffer.
// ---------------------------------------------------------------------------
template <int K, int WM, int WN, int WAVES_M, int WAVES_N, int D, int ACH>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) rot_dot_gb_kernel(RotDotArgs args) {
  using G = Geo<K>;
  constexpr int kBM = 32 * WM * WAVES_M, kBN = 32 * WN * WAVES_N;
  constexpr int kThreads = 64 * WAVES_M * WAVES_N;
  constexpr int kBBlk = kBN / 32;
  extern __shared__ __align__(16) int8_t lds[];
  int8_t* ast = lds;                                           // 2 A segment buffers
  const uint32_t abuf = args.max_q * 2 * kSegBytes;            // bytes per A buffer

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int vec = blockIdx.z;
  const uint32_t i = blockIdx.x;
  const uint32_t xcd = i & 7, s8 = i >> 3;
  const uint32_t u = s8 % args.mt, tg = s8 / args.mt;
  const uint32_t t = tg * 8 + xcd;
  if (t >= args.nt) return;

  const uint32_t m0 = u * kBM;
  const uint32_t q_lo = m0 / args.r;
  const uint32_t last_row = min(m0 + kBM, args.rows) - 1;
  const uint32_t nq = last_row / args.r - q_lo + 1;            // <= max_q

  int a_off[WM];
#pragma unroll
  for (int x = 0; x < WM; ++x) {
    const uint32_t row = m0 + (wm * WM + x) * 32 + (lane & 31);
    int slot = 0, sft = 0;
    if (row < args.rows) {
      slot = int(row / args.r - q_lo);
      sft = 4 * args.rot[row % args.r];
    }
    a_off[x] = slot * 2 * kSegBytes + kSegPad - sft + 16 * (lane >> 5);
  }

  // This lane's 16 bytes of the lo-plane fragment of each of the wave's column
  // blocks at K-step 0; step k adds 1 KB, the hi plane one plane block.
  const int8_t* bfr[WN];
#pragma unroll
  for (int y = 0; y < WN; ++y) {
    uint64_t cb = uint64_t(t) * kBBlk + wn * WN + y;
    cb = cb < args.b_blocks ? cb : args.b_blocks - 1;
    bfr[y] = args.b + size_t(args.b_block0 + cb) * G::kBlockBytes + size_t(2 * vec) * G::kPlaneBlockBytes + lane * 16;
  }
  const int a_chunks = int(nq) * 2 * kSegChunks;
  const int8_t* asrc[ACH];
  int adst[ACH];
#pragma unroll
  for (int j = 0; j < ACH; ++j) {
    int c = tid + j * kThreads;
    const bool ok = c < a_chunks;
    c = ok ? c : 0;
    const int qs = c / (2 * kSegChunks), rem = c % (2 * kSegChunks);
    const int pl = rem / kSegChunks, piece = rem % kSegChunks;
    const int src_off = ((piece * 16 - kSegPad) % kRowLen + kRowLen) % kRowLen;   // circular
    const uint32_t qrow = args.qidx ? args.qidx[q_lo + qs] : q_lo + qs;
    asrc[j] = args.qop + size_t(qrow) * G::kQopRowBytes + size_t(2 * vec + pl) * G::kK + src_off;
    adst[j] = ok ? (qs * 2 * kSegBytes + pl * kSegBytes + piece * 16) : -1;
  }

  v16i acc0[WM][WN], acc1[WM][WN];
#pragma unroll
  for (int x = 0; x < WM; ++x)
#pragma unroll
    for (int y = 0; y < WN; ++y)
#pragma unroll
      for (int e = 0; e < 16; ++e) { acc0[x][y][e] = 0; acc1[x][y][e] = 0; }

  constexpr int kSteps = G::kChunks / 2;        // 800 or 400
  constexpr int kSegSteps = kRowLen / 32;       // 25 K-steps per segment
  static_assert(kSteps % D == 0, "the K loop is unrolled by D");
  v4i bl[D][WN], bh[D][WN];                     // database fragments, set = step % D
  v4i ra[ACH];

#define IMC_BLOAD(SET, KS)                                                            \
  _Pragma("unroll") for (int y_ = 0; y_ < WN; ++y_) {                                 \
    const int8_t* p_ = bfr[y_] + size_t(KS) * 1024;                                   \
    bl[SET][y_] = *reinterpret_cast<const v4i*>(p_);                                  \
    bh[SET][y_] = *reinterpret_cast<const v4i*>(p_ + G::kPlaneBlockBytes);            \
  }
#define IMC_ALOAD(SEG)                                                                \
  _Pragma("unroll") for (int c_ = 0; c_ < ACH; ++c_)                                  \
      ra[c_] = *reinterpret_cast<const v4i*>(asrc[c_] + size_t(SEG) * kRowLen);
#define IMC_ASTORE(BUF)                                                               \
  _Pragma("unroll") for (int c_ = 0; c_ < ACH; ++c_)                                  \
      if (adst[c_] >= 0) *reinterpret_cast<v4i*>(ast + (BUF) * abuf + adst[c_]) = ra[c_];
#define IMC_AFRAGS(ALO, AHI, K)                                                       \
  {                                                                                   \
    const int kk_ = (K);                                                              \
    const int seg_ = kk_ / kSegSteps, ts_ = kk_ - seg_ * kSegSteps;                   \
    const int8_t* sa_ = ast + (seg_ & 1) * abuf + 32 * ts_;                           \
    _Pragma("unroll") for (int x_ = 0; x_ < WM; ++x_) {                               \
      const int32_t* pa_ = reinterpret_cast<const int32_t*>(sa_ + a_off[x_]);         \
      const int32_t* ph_ = reinterpret_cast<const int32_t*>(sa_ + a_off[x_] + kSegBytes); \
      ALO[x_] = v4i{pa_[0], pa_[1], pa_[2], pa_[3]};                                  \
      AHI[x_] = v4i{ph_[0], ph_[1], ph_[2], ph_[3]};                                  \
    }                                                                                 \
  }

  // prologue: A segment 0 in buffer 0, segment 1 in registers; database
  // fragments of steps 0 .. D-1 in flight
  IMC_ALOAD(0)
  IMC_ASTORE(0)
  IMC_ALOAD(1)
#pragma unroll
  for (int set = 0; set < D; ++set) { IMC_BLOAD(set, set) }
  __syncthreads();
  v4i falo[WM], fahi[WM], nalo[WM], nahi[WM];
  IMC_AFRAGS(falo, fahi, 0)

  // One K-step: the next step's A fragments are read first (pinned ahead of
  // the MFMAs, so they complete under them), then the MFMAs of this step,
  // then the database fragments of step k + D are requested into the set
  // this step consumed.  Two A register sets alternate (the loop is unrolled
  // by D, which is even).
#define IMC_GSTEP(CUR, NXT, UU)                                                       \
  {                                                                                   \
    const int k_ = k0 + (UU);                                                         \
    const int seg_ = k_ / kSegSteps, ts_ = k_ - seg_ * kSegSteps;                     \
    wait_lds(); /* this step's A fragments, read during the previous step */          \
    if (ts_ == kSegSteps / 2 && seg_ + 1 < kSteps / kSegSteps) {                      \
      /* every wave is past its last read of the other A buffer (segment seg-1): */   \
      /* store segment seg+1 there and make it visible before the segment ends */     \
      __syncthreads();                                                                \
      IMC_ASTORE((seg_ + 1) & 1)                                                      \
      __syncthreads();                                                                \
      IMC_ALOAD(min(seg_ + 2, kSteps / kSegSteps - 1))                                \
    }                                                                                 \
    IMC_AFRAGS(NXT##alo, NXT##ahi, min(k_ + 1, kSteps - 1))                            \
    __builtin_amdgcn_sched_barrier(0);                                                \
    _Pragma("unroll") for (int x = 0; x < WM; ++x)                                    \
    _Pragma("unroll") for (int y = 0; y < WN; ++y) {                                  \
      acc0[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(CUR##alo[x], bl[UU][y], acc0[x][y], 0, 0, 0); \
      acc1[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(CUR##alo[x], bh[UU][y], acc1[x][y], 0, 0, 0); \
      acc1[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(CUR##ahi[x], bl[UU][y], acc1[x][y], 0, 0, 0); \
    }                                                                                 \
    IMC_BLOAD(UU, min(k_ + D, kSteps - 1))                                            \
  }
  static_assert(D % 2 == 0, "A register sets alternate");
  for (int k0 = 0; k0 < kSteps; k0 += D) {
#pragma unroll
    for (int h = 0; h < D; h += 2) {
      IMC_GSTEP(f, n, h)
      IMC_GSTEP(n, f, h + 1)
    }
  }
#undef IMC_GSTEP
#undef IMC_AFRAGS
#undef IMC_BLOAD
#undef IMC_ALOAD
#undef IMC_ASTORE

  uint16_t* out = args.out[vec];
#pragma unroll
  for (int x = 0; x < WM; ++x)
#pragma unroll
    for (int y = 0; y < WN; ++y) {
      const uint64_t col = uint64_t(t) * kBN + (wn * WN + y) * 32 + (lane & 31);
      if (col >= args.n) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t row = m0 + (wm * WM + x) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (row < args.rows) {
          const uint32_t z = uint32_t(acc0[x][y][e]) + (uint32_t(acc1[x][y][e]) << 8);
          out[uint64_t(row) * args.ld + col] = uint16_t(z);
        }
      }
    }
}

// ---------------------------------------------------------------------------
// The same rotation-aware tiling with the operands copied HBM -> LDS by the
// load units themselves (global_load_lds_dwordx4): no staging registers and
// no LDS store instructions, so the database stream can run S - 3 K-steps
// ahead through S LDS stages.  Each wave issues an identical sequence of
// copies (one per K-step for the database, ACH per query segment, inactive
// lanes copying a valid source into the buffer's unused tail), so a per-wave
// vmcnt wait of S - 3 guarantees that the copy of step k + 2 has landed
// before the barrier that precedes its fragment reads.  The barriers are
// bare s_barrier instructions: a workgroup fence would wait for every
// outstanding copy.
// ---------------------------------------------------------------------------

template <int K, int WM, int WN, int WAVES_M, int WAVES_N, int S, int ACH>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) rot_dot_dma_kernel(RotDotArgs args) {
  using G = Geo<K>;
  constexpr int kBM = 32 * WM * WAVES_M, kBN = 32 * WN * WAVES_N;
  constexpr int kThreads = 64 * WAVES_M * WAVES_N;
  constexpr int kBBlk = kBN / 32;
  constexpr int kBChunks = kBBlk * 2 * 2 * 32;                 // per K-step
  constexpr int kBPerThread = kBChunks / kThreads;
  constexpr int kBStage = kBChunks * 16;
  constexpr int kABuf = ACH * kThreads * 16;                   // A buffer incl. the unused tail
  static_assert(kBChunks % kThreads == 0, "B chunks must divide evenly");
  static_assert(S >= 4, "at least one copy in flight beyond the two read-ahead stages");
  // the wait for step k + 2 must also cover the query segment copied at mid-segment
  static_assert(S <= 12, "query segment copy must precede the copy waited for at the segment end");
  extern __shared__ __align__(16) int8_t lds[];
  int8_t* bst = lds;                                           // S B stages
  int8_t* ast = lds + S * kBStage;                             // 2 A segment buffers

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int vec = blockIdx.z;
  const uint32_t i = blockIdx.x;
  const uint32_t xcd = i & 7, s8 = i >> 3;
  const uint32_t u = s8 % args.mt, tg = s8 / args.mt;
  const uint32_t t = tg * 8 + xcd;
  if (t >= args.nt) return;

  const uint32_t m0 = u * kBM;
  const uint32_t q_lo = m0 / args.r;
  const uint32_t last_row = min(m0 + kBM, args.rows) - 1;
  const uint32_t nq = last_row / args.r - q_lo + 1;            // <= max_q

  int a_off[WM];
#pragma unroll
  for (int x = 0; x < WM; ++x) {
    const uint32_t row = m0 + (wm * WM + x) * 32 + (lane & 31);
    int slot = 0, sft = 0;
    if (row < args.rows) {
      slot = int(row / args.r - q_lo);
      sft = 4 * args.rot[row % args.r];
    }
    a_off[x] = slot * 2 * kSegBytes + kSegPad - sft + 16 * (lane >> 5);
  }

  const int8_t* bsrc[kBPerThread];
#pragma unroll
  for (int j = 0; j < kBPerThread; ++j) {
    const int c = tid + j * kThreads;
    const int blk = c >> 7, rem = c & 127;
    const int plane = rem >> 6, kcl = (rem >> 5) & 1, slot = rem & 31;
    uint64_t cb = uint64_t(t) * kBBlk + blk;
    cb = cb < args.b_blocks ? cb : args.b_blocks - 1;
    bsrc[j] = args.b + size_t(args.b_block0 + cb) * G::kBlockBytes + size_t(2 * vec + plane) * G::kPlaneBlockBytes +
              size_t(kcl) * 512 + slot * 16;
  }
  // A chunk c of a segment buffer = (query slot, plane, 16-byte piece) lands at
  // byte 16 c; chunks past the tile's queries copy piece 0 of slot 0.
  const int a_chunks = int(nq) * 2 * kSegChunks;
  const int8_t* asrc[ACH];
#pragma unroll
  for (int j = 0; j < ACH; ++j) {
    int c = tid + j * kThreads;
    c = c < a_chunks ? c : 0;
    const int qs = c / (2 * kSegChunks), rem = c % (2 * kSegChunks);
    const int pl = rem / kSegChunks, piece = rem % kSegChunks;
    const int src_off = ((piece * 16 - kSegPad) % kRowLen + kRowLen) % kRowLen;   // circular
    const uint32_t qrow = args.qidx ? args.qidx[q_lo + qs] : q_lo + qs;
    asrc[j] = args.qop + size_t(qrow) * G::kQopRowBytes + size_t(2 * vec + pl) * G::kK + src_off;
  }

  v16i acc0[WM][WN], acc1[WM][WN];
#pragma unroll
  for (int x = 0; x < WM; ++x)
#pragma unroll
    for (int y = 0; y < WN; ++y)
#pragma unroll
      for (int e = 0; e < 16; ++e) { acc0[x][y][e] = 0; acc1[x][y][e] = 0; }

  constexpr int kSteps = G::kChunks / 2;        // 800 or 400
  constexpr int kSegSteps = kRowLen / 32;    // 25 K-steps per segment
  constexpr int kSegs = kSteps / kSegSteps;  // 32 or 16

  // wave-uniform LDS bases of this wave's copies
  const int wbase = wave * 64 * 16;
#define IMC_BCOPY(KS)                                                                 \
  {                                                                                   \
    const int ks_ = (KS);                                                             \
    _Pragma("unroll") for (int c_ = 0; c_ < kBPerThread; ++c_)                        \
      copy16(bsrc[c_] + size_t(2 * ks_) * 512,                                        \
             bst + (ks_ % S) * kBStage + c_ * kThreads * 16 + wbase);                 \
  }
#define IMC_ACOPY(SEG, BUF)                                                           \
  _Pragma("unroll") for (int c_ = 0; c_ < ACH; ++c_)                                  \
    copy16(asrc[c_] + size_t(SEG) * kRowLen, ast + (BUF) * kABuf + c_ * kThreads * 16 + wbase);

  v4i falo[WM], fahi[WM], fblo[WN], fbhi[WN];
  v4i nalo[WM], nahi[WM], nblo[WN], nbhi[WN];
#define IMC_FRAGS(ALO, AHI, BLO, BHI, K)                                              \
  {                                                                                   \
    const int kk_ = (K);                                                              \
    const int seg_ = kk_ / kSegSteps, ts_ = kk_ - seg_ * kSegSteps;                   \
    const int8_t* sb_ = bst + (kk_ % S) * kBStage;                                    \
    const int8_t* sa_ = ast + (seg_ & 1) * kABuf + 32 * ts_;                          \
    _Pragma("unroll") for (int x_ = 0; x_ < WM; ++x_) {                               \
      const int32_t* pa_ = reinterpret_cast<const int32_t*>(sa_ + a_off[x_]);         \
      const int32_t* ph_ = reinterpret_cast<const int32_t*>(sa_ + a_off[x_] + kSegBytes); \
      ALO[x_] = v4i{pa_[0], pa_[1], pa_[2], pa_[3]};                                  \
      AHI[x_] = v4i{ph_[0], ph_[1], ph_[2], ph_[3]};                                  \
    }                                                                                 \
    _Pragma("unroll") for (int y_ = 0; y_ < WN; ++y_) {                               \
      const int8_t* pb_ = sb_ + (wn * WN + y_) * 2048 + lane * 16;                    \
      BLO[y_] = *reinterpret_cast<const v4i*>(pb_);                                   \
      BHI[y_] = *reinterpret_cast<const v4i*>(pb_ + 1024);                            \
    }                                                                                 \
  }

  // prologue: A segment 0, B steps 0 .. S - 2; all landed before the first reads
  IMC_ACOPY(0, 0)
#pragma unroll
  for (int j = 0; j < S - 1; ++j) IMC_BCOPY(j)
  wait_vm<0>();
  bar();
  IMC_FRAGS(falo, fahi, fblo, fbhi, 0)

  // One K-step: copies for later steps, the next step's fragment reads (issued
  // before the MFMAs so that they complete under them), the MFMAs, then the
  // wait for the copy of step k + 2 and the barrier.  Unrolled by two so the
  // current / next fragment registers alternate without moves.
#define IMC_STEP(CUR, NXT, K)                                                         \
  {                                                                                   \
    const int k_ = (K);                                                               \
    const int seg_ = k_ / kSegSteps, ts_ = k_ - seg_ * kSegSteps;                     \
    wait_lds(); /* this step's fragments, read during the previous step */            \
    if (ts_ == kSegSteps / 2 && seg_ + 1 < kSegs) IMC_ACOPY(seg_ + 1, (seg_ + 1) & 1) \
    const bool more_ = k_ + S - 1 < kSteps;                                           \
    if (more_) IMC_BCOPY(k_ + S - 1)                                                  \
    IMC_FRAGS(NXT##alo, NXT##ahi, NXT##blo, NXT##bhi, min(k_ + 1, kSteps - 1))         \
    __builtin_amdgcn_sched_barrier(0);                                                \
    _Pragma("unroll") for (int x = 0; x < WM; ++x)                                    \
    _Pragma("unroll") for (int y = 0; y < WN; ++y) {                                  \
      acc0[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(CUR##alo[x], CUR##blo[y], acc0[x][y], 0, 0, 0); \
      acc1[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(CUR##alo[x], CUR##bhi[y], acc1[x][y], 0, 0, 0); \
      acc1[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(CUR##ahi[x], CUR##blo[y], acc1[x][y], 0, 0, 0); \
    }                                                                                 \
    if (more_)                                                                        \
      wait_vm<S - 3>();                                                               \
    else                                                                              \
      wait_vm<0>();                                                                   \
    bar();                                                                            \
  }
  static_assert(kSteps % 2 == 0, "the K loop is unrolled by two");
  for (int k = 0; k < kSteps; k += 2) {
    IMC_STEP(f, n, k)
    IMC_STEP(n, f, k + 1)
  }
#undef IMC_STEP
  wait_vm<0>();
#undef IMC_FRAGS
#undef IMC_BCOPY
#undef IMC_ACOPY

  uint16_t* out = args.out[vec];
#pragma unroll
  for (int x = 0; x < WM; ++x)
#pragma unroll
    for (int y = 0; y < WN; ++y) {
      const uint64_t col = uint64_t(t) * kBN + (wn * WN + y) * 32 + (lane & 31);
      if (col >= args.n) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t row = m0 + (wm * WM + x) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (row < args.rows) {
          const uint32_t z = uint32_t(acc0[x][y][e]) + (uint32_t(acc1[x][y][e]) << 8);
          out[uint64_t(row) * args.ld + col] = uint16_t(z);
        }
      }
    }
}

template <int K, int ACH>
static hipError_t launch_rot_cfg(const int8_t* qop, const uint32_t* qidx, uint32_t q, uint32_t r, const int8_t* rot,
                                 const int8_t* b,
                                 uint64_t first_entry, uint64_t n, uint16_t* code, uint16_t* mask, uint64_t ld,
                                 hipStream_t s, const DotScratch& scratch) {
  constexpr int kBM = kRotM, kBN = kRotN, kThreads = kRotThreads;
  const uint32_t rows = q * r;
  if (rows == 0 || n == 0) return hipSuccess;
  if (r < 13) return hipErrorInvalidValue;
  RotDotArgs d;
  d.qop = qop;
  d.qidx = qidx;
  d.b = b;
  d.out[0] = code;
  d.out[1] = mask;
  d.ld = ld;
  d.rows = rows;
  d.q = q;
  d.r = r;
  d.b_block0 = first_entry / 32;
  d.b_blocks = (n + 31) / 32;
  d.n = n;
  d.nt = uint32_t((n + kBN - 1) / kBN);
  constexpr uint32_t kSegs = Geo<K>::kChunks / 2 / kSegSteps;
  static_assert(kSegs == rot_segs(K == kKGalois), "the plan's parts are the launch's");
  const uint32_t vecs = mask ? 2 : 1;
  const uint32_t splits = rot_splits(rows, n, vecs, dot_room(scratch, K == kKGalois));
  d.seg_per = (kSegs + splits - 1) / splits;
  d.splits = (kSegs + d.seg_per - 1) / d.seg_per;
  d.tile_m = d.splits > 1 ? kBM : rot_tile_rows(rows, d.nt, vecs, scratch.cus);
  d.mt = (rows + d.tile_m - 1) / d.tile_m;
  d.max_q = (d.tile_m + r - 1) / r + 1;
  if (int(d.max_q) * 2 * kSegChunks > ACH * kThreads) return hipErrorInvalidValue;
  for (int i = 0; i < IMC_MAX_ROT_DEV; ++i) d.rot[i] = i < int(r) ? rot[i] : 0;
  const uint32_t ntg = (d.nt + 7) / 8;
  if (uint64_t(ntg) * 8 * d.mt > 0x7FFFFFFFull) return hipErrorInvalidValue;
  const dim3 grid(ntg * 8 * d.mt, 1, vecs);   // z: code, mask
  const size_t lds = 3 * size_t(kRotStage) + 2 * size_t(d.max_q) * 2 * kSegBytes;
  if (d.splits > 1) {
    d.part = scratch.part;
    auto kern = rot_dot_split_kernel<K, ACH>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e == hipSuccess) e = scratch.begin(s);
    if (e != hipSuccess) return e;
    const uint32_t ntp = (d.nt * d.splits + 7) / 8 * 8;
    hipLaunchKernelGGL(kern, dim3(ntp * d.mt, 1, grid.z), dim3(kThreads), lds, s, d);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_reduce_parts(scratch, d.splits, rows, n, code, mask, ld, s);
  }
  d.part = nullptr;
  d.lead = d.tile_m < kRotM ? d.mt : rot_lead_tiles(rows, uint64_t(d.mt) * d.nt * vecs, scratch.cus);
  auto kern = rot_dot_kernel<K, ACH>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, grid, dim3(kThreads), lds, s, d);
  return hipGetLastError();
}

template <int K>
static hipError_t launch_rot_dma(const int8_t* qop, const uint32_t* qidx, uint32_t q, uint32_t r, const int8_t* rot,
                                 const int8_t* b,
                                 uint64_t first_entry, uint64_t n, uint16_t* code, uint16_t* mask, uint64_t ld,
                                 hipStream_t s) {
  constexpr int WM = 2, WN = 2, WAVES_M = 4, WAVES_N = 2, S = 8, ACH = 3;
  constexpr int kBM = 32 * WM * WAVES_M, kBN = 32 * WN * WAVES_N, kThreads = 64 * WAVES_M * WAVES_N;
  const uint32_t rows = q * r;
  if (rows == 0 || n == 0) return hipSuccess;
  if (r < 13) return hipErrorInvalidValue;
  RotDotArgs d;
  d.qop = qop;
  d.qidx = qidx;
  d.b = b;
  d.out[0] = code;
  d.out[1] = mask;
  d.ld = ld;
  d.rows = rows;
  d.q = q;
  d.r = r;
  d.b_block0 = first_entry / 32;
  d.b_blocks = (n + 31) / 32;
  d.n = n;
  d.mt = (rows + kBM - 1) / kBM;
  d.nt = uint32_t((n + kBN - 1) / kBN);
  d.max_q = (kBM + r - 1) / r + 1;
  if (int(d.max_q) * 2 * kSegChunks > ACH * kThreads) return hipErrorInvalidValue;
  for (int i = 0; i < IMC_MAX_ROT_DEV; ++i) d.rot[i] = i < int(r) ? rot[i] : 0;
  const uint32_t ntg = (d.nt + 7) / 8;
  if (uint64_t(ntg) * 8 * d.mt > 0x7FFFFFFFull) return hipErrorInvalidValue;
  const dim3 grid(ntg * 8 * d.mt, 1, mask ? 2 : 1);   // z: code, mask
  const size_t lds = size_t(S) * (kBN / 32) * 2 * 2 * 32 * 16 + 2 * size_t(ACH) * kThreads * 16;
  auto kern = rot_dot_dma_kernel<K, WM, WN, WAVES_M, WAVES_N, S, ACH>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, grid, dim3(kThreads), lds, s, d);
  return hipGetLastError();
}

template <int K, int WM, int WN, int WAVES_M, int WAVES_N, int D, int ACH>
static hipError_t launch_rot_gb(const int8_t* qop, const uint32_t* qidx, uint32_t q, uint32_t r, const int8_t* rot,
                                 const int8_t* b,
                                uint64_t first_entry, uint64_t n, uint16_t* code, uint16_t* mask, uint64_t ld,
                                hipStream_t s) {
  constexpr int kBM = 32 * WM * WAVES_M, kBN = 32 * WN * WAVES_N, kThreads = 64 * WAVES_M * WAVES_N;
  const uint32_t rows = q * r;
  if (rows == 0 || n == 0) return hipSuccess;
  if (r < 13) return hipErrorInvalidValue;
  RotDotArgs d;
  d.qop = qop;
  d.qidx = qidx;
  d.b = b;
  d.out[0] = code;
  d.out[1] = mask;
  d.ld = ld;
  d.rows = rows;
  d.q = q;
  d.r = r;
  d.b_block0 = first_entry / 32;
  d.b_blocks = (n + 31) / 32;
  d.n = n;
  d.mt = (rows + kBM - 1) / kBM;
  d.nt = uint32_t((n + kBN - 1) / kBN);
  d.max_q = (kBM + r - 1) / r + 1;
  if (int(d.max_q) * 2 * kSegChunks > ACH * kThreads) return hipErrorInvalidValue;
  for (int i = 0; i < IMC_MAX_ROT_DEV; ++i) d.rot[i] = i < int(r) ? rot[i] : 0;
  const uint32_t ntg = (d.nt + 7) / 8;
  if (uint64_t(ntg) * 8 * d.mt > 0x7FFFFFFFull) return hipErrorInvalidValue;
  const dim3 grid(ntg * 8 * d.mt, 1, mask ? 2 : 1);   // z: code, mask
  const size_t lds = 2 * size_t(d.max_q) * 2 * kSegBytes;
  auto kern = rot_dot_gb_kernel<K, WM, WN, WAVES_M, WAVES_N, D, ACH>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, grid, dim3(kThreads), lds, s, d);
  return hipGetLastError();
}

template <int K, int ACH>
static hipError_t launch_rot_groups_cfg(const DotGroup* groups, uint32_t ngroups, const int8_t* b,
                                        uint64_t first_entry, uint64_t n, uint64_t ld, bool persistent,
                                        hipStream_t s, int cus) {
  constexpr int kBN = kRotN, kThreads = kRotThreads;
  RotGroupsArgs d;
  d.b = b;
  d.ld = ld;
  d.b_block0 = first_entry / 32;
  d.b_blocks = (n + 31) / 32;
  d.n = n;
  d.nt = uint32_t((n + kBN - 1) / kBN);
  const uint64_t ntg = (d.nt + 7) / 8;
  d.tile_m = 64;
  for (; d.tile_m < kRotM; d.tile_m += 64) {   // as rot_tile_rows, over all groups
    uint64_t all = 0;
    uint32_t vecs = 1;
    for (uint32_t gi = 0; gi < ngroups; ++gi) {
      all += rot_tiles(uint64_t(groups[gi].q) * groups[gi].r, d.tile_m);
      if (groups[gi].mask) vecs = 2;
    }
    if (one_round(all, d.nt, vecs, cus)) break;
  }
  uint64_t tiles = 0;
  uint32_t max_q = 0, used = 0;
  bool mask = false;
  for (uint32_t gi = 0; gi < ngroups; ++gi) {
    const DotGroup& g = groups[gi];
    const uint32_t rows = g.q * g.r;
    if (rows == 0) continue;
    RotGroup& o = d.g[used++];
    o.qop = g.qop;
    o.out[0] = g.code;
    o.out[1] = g.mask;
    mask = g.mask != nullptr;
    o.rows = rows;
    o.r = g.r;
    o.mt = (rows + d.tile_m - 1) / d.tile_m;
    o.tile0 = uint32_t(tiles);
    for (int j = 0; j < IMC_MAX_ROT_DEV; ++j) o.rot[j] = j < int(g.r) ? g.rot[j] : 0;
    max_q = std::max(max_q, (d.tile_m + g.r - 1) / g.r + 1);
    tiles += ntg * 8 * o.mt;
    if (tiles > 0x7FFFFFFFull) return hipErrorInvalidValue;
  }
  if (used == 0 || n == 0) return hipSuccess;
  if (int(max_q) * 2 * kSegChunks > ACH * kThreads) return hipErrorInvalidValue;
  d.ngroups = used;
  d.ntiles = uint32_t(tiles);
  d.max_q = max_q;
  const size_t lds = 3 * size_t(kRotStage) + 2 * size_t(max_q) * 2 * kSegBytes;
  auto kern = rot_dot_groups_kernel<K, ACH>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e != hipSuccess) return e;
  uint32_t grid = d.ntiles;
  if (persistent) {
    // one workgroup per CU (the LDS of a tile allows no second one), a
    // multiple of the 8 XCDs
    const uint32_t g8 = (uint32_t(cus) + 7) / 8 * 8;
    grid = std::min<uint32_t>(grid, g8);
  }
  hipLaunchKernelGGL(kern, dim3(grid, 1, mask ? 2 : 1), dim3(kThreads), lds, s, d);
  return hipGetLastError();
}

hipError_t launch_rot_dot_groups(const DotGroup* groups, uint32_t ngroups, const int8_t* b, uint64_t first_entry,
                                 uint64_t n, uint64_t ld, bool persistent, hipStream_t s, bool galois, int cus) {
  if (cus <= 0 || ngroups > uint32_t(kMaxDotGroups)) return hipErrorInvalidValue;
  uint32_t rmin = 32;
  for (uint32_t gi = 0; gi < ngroups; ++gi) {
    if (groups[gi].q == 0) continue;
    if (groups[gi].r < 13) return hipErrorInvalidValue;
    rmin = std::min(rmin, groups[gi].r);
  }
  // the staging of the fewest rotations (the most query slots) sizes the launch
  if (galois)
    return rmin >= 22 ? launch_rot_groups_cfg<kKGalois, 3>(groups, ngroups, b, first_entry, n, ld, persistent, s, cus)
                      : launch_rot_groups_cfg<kKGalois, 5>(groups, ngroups, b, first_entry, n, ld, persistent, s, cus);
  return rmin >= 22 ? launch_rot_groups_cfg<kK, 3>(groups, ngroups, b, first_entry, n, ld, persistent, s, cus)
                    : launch_rot_groups_cfg<kK, 5>(groups, ngroups, b, first_entry, n, ld, persistent, s, cus);
}

hipError_t launch_rot_dot(const RotCall& c, hipStream_t s, int kind, bool galois, const DotScratch& scratch) {
  // 0: 8 waves of 64 x 64, loads 4 steps of 64 bytes ahead; 2: HBM -> LDS copies, 8
  // stages; 3: database fragments straight into registers
  if (galois) {
    switch (kind) {
      case 2: return launch_rot_dma<kKGalois>(c.qop, c.qidx, c.q, c.r, c.rot, c.b, c.first_entry, c.n, c.code, c.mask, c.ld, s);
      case 3: return launch_rot_gb<kKGalois, 2, 2, 4, 2, 4, 3>(c.qop, c.qidx, c.q, c.r, c.rot, c.b, c.first_entry, c.n, c.code, c.mask, c.ld, s);
      default:
        if (c.r >= 22) return launch_rot_cfg<kKGalois, 3>(c.qop, c.qidx, c.q, c.r, c.rot, c.b, c.first_entry, c.n, c.code, c.mask, c.ld, s, scratch);
        return launch_rot_cfg<kKGalois, 5>(c.qop, c.qidx, c.q, c.r, c.rot, c.b, c.first_entry, c.n, c.code, c.mask, c.ld, s, scratch);
    }
  }
  switch (kind) {
    case 2: return launch_rot_dma<kK>(c.qop, c.qidx, c.q, c.r, c.rot, c.b, c.first_entry, c.n, c.code, c.mask, c.ld, s);
    case 3: return launch_rot_gb<kK, 2, 2, 4, 2, 4, 3>(c.qop, c.qidx, c.q, c.r, c.rot, c.b, c.first_entry, c.n, c.code, c.mask, c.ld, s);
    default:
      if (c.r >= 22) return launch_rot_cfg<kK, 3>(c.qop, c.qidx, c.q, c.r, c.rot, c.b, c.first_entry, c.n, c.code, c.mask, c.ld, s, scratch);
      return launch_rot_cfg<kK, 5>(c.qop, c.qidx, c.q, c.r, c.rot, c.b, c.first_entry, c.n, c.code, c.mask, c.ld, s, scratch);
  }
}

}  // namespace imc
