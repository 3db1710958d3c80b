// pair_dot.hip -- party-local dot products (Alg. 3; App. C) of consecutive
// rotations, with a quarter of the ring multiplications taken out and most
// query fragments kept in registers.
//
// The r products of one query with one entry are a Toeplitz matrix-vector
// product along the angular axis: out(s) = sum_c x[c - s] y[c] over the 200
// columns c of each angular row (each column 4 elements; Sec. 3's rotations).
// Taking the columns in blocks of 8 as (c, c + 4) and the rotations in pairs
// (s, s + 4), with D[c] = x[c + 4] - x[c]:
//   P        = sum x[c - s]     (y[c] + y[c + 4])
//   out(s)   = P + sum D[c - s]     y[c + 4]
//   out(s+4) = P - sum D[c - s - 4] y[c]
// (c over the first 4 columns of each block of 8): three products over half
// the columns instead of two over all of them, exact in Z_2^16.  Sums and
// differences are formed mod 2^16 and split into balanced byte limbs again,
// so the limb products and accumulator bounds are those of dot.hip.
//
// Rotation index 8a + b (+ 4): the 16 bytes of x that rotation (a, b) reads
// at block g are those that (a - 1, b) read at block g - 1.  A wave therefore
// keeps the four a's in separate 16-row MFMA blocks (rows: 4 queries x 4 b's)
// and a query fragment read from LDS once serves them in four consecutive
// K-steps out of registers.
//
// What bounds it: power and issue, not memory.  A register-only loop of
// v_mfma_i32_32x32x32_i8 on random bytes runs at 3.35 POP/s on this part and
// one of v_mfma_i32_16x16x64_i8 at 4.0 (5.0 on zeros): random operands pull
// the clock down to 1.7 - 2.0 GHz, the 16 x 16 x 64 shape less.  One party's
// dots of 64 queries x 31 rotations against 65,536 entries: 15.8 ms with
// rot_dot.hip's kernel, 12.9 with this scheme on 32 x 32 x 32 MFMAs, 11.2 as
// it stands.  Against 300,000 entries: MFMA pipes 0.70 busy at 1.8 GHz, 69.7 GB
// read (each product streams its half of the database tile).  Without any
// staging the loops take 8.5 ms of the 11.2.
#include <utility>

#include "device.h"
#include "launch.h"

namespace imc {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

struct PairDotArgs {
  const int8_t* qop;     // unrotated query operand, row-major [q][plane 4][K]
  const uint32_t* qidx;  // optional: query i of the call is operand row qidx[i]
  const int8_t* b;       // party's database region
  uint16_t* out[2];
  uint64_t ld;
  uint32_t q, r;
  int32_t s0;            // first rotation of the consecutive list
  uint64_t b_block0, b_blocks, n;
  uint32_t mt, nt;
};

// Tile: 16 queries (256 rotation pairs) x 128 entries, 8 waves of 4 queries
// (64 pairs) x 64 entries; waves 0-3 also stage the database, 4-7 the queries.  A K-step is one block of 8 columns of four
// angular rows (64 bytes of k, one angular row per 16-lane group of the
// 16 x 16 x 64 MFMA), a segment the 25 blocks of four angular rows.
constexpr int kPairQ = 16, kPairN = 128, kPairThreads = 512;
constexpr int kStagers = 256;                     // threads of each staging role
constexpr int kPairT = 25;
constexpr int kPairRows = kPairQ * 4;             // (query, angular row) rows of a segment in LDS
// A segment's query bytes pass through LDS in two windows of its blocks:
// [-3, 11] (the a's of block 0 start at block -3) and [12, 24].  Pieces of 16
// bytes per row: 32 bytes per block, 28 more for the four b's and the
// fragment's own length, the start rounded down to 16.  A row holds the low
// limbs, then the high ones, then 16 bytes: an odd number of pieces, which
// puts a fragment read's 16 rows into distinct banks.
constexpr int kWin0 = 31, kWin1 = 27;
constexpr int kWin0Row = (2 * kWin0 + 1) * 16, kWin1Row = (2 * kWin1 + 1) * 16;
constexpr int kWin0Bytes = kPairRows * kWin0Row, kWin1Bytes = kPairRows * kWin1Row;
constexpr int kPairStage = kPairN * 128;          // one K-step of the database: 2 limbs x 4 rows x 16 B per entry
constexpr int kPairLds = 2 * kPairStage + kWin0Bytes + kWin1Bytes;
static_assert(kPairLds <= 160 * 1024, "one workgroup's LDS");

// a + b or a - b of four Z_2^16 values held as balanced byte limbs.
template <bool SUB>
__device__ __forceinline__ void limb_addsub(uint32_t la, uint32_t ha, uint32_t lb, uint32_t hb, uint32_t& lo,
                                            uint32_t& hi) {
  la ^= 0x80808080u;   // value + 0x80 = 256 hi + (lo ^ 0x80)
  lb ^= 0x80808080u;
  const u16x2 a0 = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(ha, la, 0x05010400u));
  const u16x2 a1 = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(ha, la, 0x07030602u));
  const u16x2 b0 = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(hb, lb, 0x05010400u));
  const u16x2 b1 = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(hb, lb, 0x07030602u));
  const u16x2 c = {0x80, 0x80};
  // result + 0x80 per 16 bits: its high byte is the high limb, its low byte
  // the low limb with the top bit flipped
  const uint32_t t0 = __builtin_bit_cast(uint32_t, u16x2(SUB ? a0 - b0 + c : a0 + b0 - c));
  const uint32_t t1 = __builtin_bit_cast(uint32_t, u16x2(SUB ? a1 - b1 + c : a1 + b1 - c));
  lo = __builtin_amdgcn_perm(t1, t0, 0x06040200u) ^ 0x80808080u;
  hi = __builtin_amdgcn_perm(t1, t0, 0x07050301u);
}

// The value that lane l + 1 holds (0 in lane 63).
__device__ __forceinline__ uint32_t next_lane(int v) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, v, 0x130 /* wave_shl:1 */, 0xf, 0xf, false));
}

template <typename F, int... T>
__device__ __forceinline__ void for_each_step(const F& step, std::integer_sequence<int, T...>) {
  (step(std::integral_constant<int, T>{}), ...);
}

// The three products in turn.  PH 0: x against y[c] + y[c + 4]; 1: D against
// y[c + 4]; 2: D (4 columns earlier) against y[c].
template <int PH, int K, bool LIVE, bool DBS>
__device__ __forceinline__ void pair_phase(const PairDotArgs& args, const int8_t* __restrict__ bbase, uint32_t u,
                                           uint64_t blk0, int vec, int8_t* lds, v4i (&acc0)[4][4],
                                           v4i (&acc1)[4][4]) {
  using G = Geo<K>;
  constexpr int kT = kPairT, kSegs = K / (4 * kRowLen), kSteps = kSegs * kT;
  const int tid = threadIdx.x & (kStagers - 1);
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  // first byte of window 0 within an angular row (window 1: 480 later)
  const int start0 = (-96 - 4 * (args.s0 + 3) - (PH == 2 ? 16 : 0)) & ~15;

  // Database staging.  Sum: two items (block, row, slot), both limbs of both
  // chunks; else four items (block, limb, row, slot) of one chunk.  Unit j, in
  // stage j % 2, holds what step j reads from LDS: its own entries except
  // each wave's first 16, and those of step j + 1 (read a block ahead).
  constexpr int kB = PH == 0 ? 2 : 4;
  uint32_t bsrc[kB];
  uint32_t bdst[kB];
  bool lead[kB];
#pragma unroll
  for (int j = 0; j < kB; ++j) {
    const int c = tid + j * kStagers;
    const int blk = PH == 0 ? c >> 7 : c >> 8, limb = PH == 0 ? 0 : (c >> 7) & 1;
    const int h = (c >> 5) & 3, slot = c & 31;
    lead[j] = (blk & 1) == 0 && slot < 16;
    const uint64_t cb = min(blk0 + blk, args.b_blocks - 1);
    bsrc[j] = uint32_t(cb - blk0) * uint32_t(G::kBlockBytes) + uint32_t(limb) * uint32_t(G::kPlaneBlockBytes) +
              h * 25600 + slot * 16 + (PH == 1 ? 512 : 0);
    bdst[j] = uint32_t(((blk * 2 + (slot >> 4)) * 2 + limb) * 1024 + h * 256 + (slot & 15) * 16);
  }
  constexpr int kRs = PH == 0 ? 8 : 4;
  v4i rs[5][kRs];

  // step k's block: segment k / 25 (four angular rows of 25,600 bytes), block k % 25
  const auto step_off = [](int k) {
    k = max(0, min(k, kSteps - 1));
    return uint32_t(k) * 1024u + uint32_t(k / kT) * 76800u;
  };
#define IMC_BLOAD(J, SET, UNIT)                                                                  \
  {                                                                                              \
    const uint32_t o0_ = step_off(UNIT), o1_ = step_off((UNIT) + 1);                             \
    const uint32_t x_ = bsrc[J] + (lead[J] ? o1_ : o0_);                                         \
    if constexpr (PH == 0) {                                                                     \
      rs[SET][4 * (J)] = *reinterpret_cast<const v4i*>(bbase + x_);                              \
      rs[SET][4 * (J) + 1] = *reinterpret_cast<const v4i*>(bbase + 512 + x_);                    \
      rs[SET][4 * (J) + 2] = *reinterpret_cast<const v4i*>(bbase + G::kPlaneBlockBytes + x_);    \
      rs[SET][4 * (J) + 3] = *reinterpret_cast<const v4i*>(bbase + (G::kPlaneBlockBytes + 512) + x_); \
    } else {                                                                                     \
      rs[SET][J] = *reinterpret_cast<const v4i*>(bbase + x_);                                    \
    }                                                                                            \
  }
#define IMC_BSTORE(J, SET, ST)                                                                   \
  if constexpr (PH == 0) {                                                                       \
    const v4i* r_ = &rs[SET][4 * (J)];                                                           \
    v4i lo_, hi_;                                                                                \
    _Pragma("unroll") for (int w_ = 0; w_ < 4; ++w_) {                                           \
      uint32_t l_, h_;                                                                           \
      limb_addsub<false>(r_[0][w_], r_[2][w_], r_[1][w_], r_[3][w_], l_, h_);                    \
      lo_[w_] = int(l_);                                                                         \
      hi_[w_] = int(h_);                                                                         \
    }                                                                                            \
    *reinterpret_cast<v4i*>(lds + ((ST) + bdst[J])) = lo_;                                       \
    *reinterpret_cast<v4i*>(lds + ((ST) + bdst[J] + 1024)) = hi_;                                \
  } else {                                                                                       \
    *reinterpret_cast<v4i*>(lds + ((ST) + bdst[J])) = rs[SET][J];                                \
  }

  // Query staging: a part is eight (query, angular row) rows of a window, two
  // per staging wave, a lane per 16-byte piece (the last lanes of a row stage
  // nothing).  D's piece is the next lane's piece of x minus this one.  A
  // wave's rows of all parts are the same angular rows, so a part's address is
  // a scalar plus a lane offset that never changes.
  constexpr int kParts = kPairRows / 8;
  const int st_h = (wave & 1) * 2 + (lane >> 5), st_pc = lane & 31;
  uint32_t st_src[2];
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    int o = start0 + 480 * w + 16 * st_pc;
    o += o < 0 ? kRowLen : 0;
    o -= o >= kRowLen ? kRowLen : 0;
    st_src[w] = uint32_t(st_h * kRowLen + o);
  }
  const uint32_t st_row = ((wave >> 1) & 1) * 4 + st_h;   // row of part 0
  uint32_t st_dst0 = uint32_t(2 * kPairStage) + st_row * kWin0Row + 16 * st_pc;
  uint32_t st_dst1 = uint32_t(2 * kPairStage + kWin0Bytes) + st_row * kWin1Row + 16 * st_pc;
  v4i ra[2];
#define IMC_ALOAD(R, W, PART, SEG)                                                               \
  {                                                                                              \
    const uint32_t qi_ = min(u * kPairQ + 2 * (PART) + ((wave >> 1) & 1), args.q - 1);           \
    const uint32_t qr_ = args.qidx ? args.qidx[qi_] : qi_;                                       \
    const int8_t* src_ = args.qop + size_t(qr_) * G::kQopRowBytes +                              \
                         (size_t(2 * vec) * K + size_t(4 * (SEG)) * kRowLen);                    \
    R[0] = *reinterpret_cast<const v4i*>(src_ + st_src[W]);                                      \
    R[1] = *reinterpret_cast<const v4i*>(src_ + K + st_src[W]);                                  \
  }
#define IMC_ASTORE(R, W, PART)                                                                   \
  {                                                                                              \
    v4i lo_ = R[0], hi_ = R[1];                                                                  \
    if (PH != 0) {                                                                               \
      _Pragma("unroll") for (int w_ = 0; w_ < 4; ++w_) {                                         \
        uint32_t l_, h_;                                                                         \
        limb_addsub<true>(next_lane(R[0][w_]), next_lane(R[1][w_]), R[0][w_], R[1][w_], l_, h_); \
        lo_[w_] = int(l_);                                                                       \
        hi_[w_] = int(h_);                                                                       \
      }                                                                                          \
    }                                                                                            \
    if (st_pc < ((W) ? kWin1 : kWin0)) {                                                         \
      int8_t* d_ = lds + ((W) ? st_dst1 + 8 * (PART)*kWin1Row : st_dst0 + 8 * (PART)*kWin0Row);  \
      *reinterpret_cast<v4i*>(d_) = lo_;                                                         \
      *reinterpret_cast<v4i*>(d_ + ((W) ? kWin1 : kWin0) * 16) = hi_;                            \
    }                                                                                            \
  }

  // this lane's query fragment: row (query, angular row), rotation index b.
  // LDS offsets of its blocks -3 and 12; opaque, so that every read is one of
  // them plus an immediate offset.
  const int a_in = -4 * (args.s0 + (lane & 3)) - (PH == 2 ? 16 : 0) - start0 - 96;   // in [0, 28)
  const int a_row = wm * 16 + ((lane >> 2) & 3) * 4 + (lane >> 4);
  uint32_t a_win0 = uint32_t(2 * kPairStage + a_row * kWin0Row + a_in);
  uint32_t a_win1 = uint32_t(2 * kPairStage + kWin0Bytes + a_row * kWin1Row + a_in);
  uint32_t b_off = uint32_t(wn * 8192 + lane * 16);
  asm volatile("" : "+v"(a_win0), "+v"(a_win1), "+v"(b_off));

  // F[g mod 5]: query fragments of block g; FB[y mod 2]: database fragments
  // of the wave's 16 entries y of four
  v4i flo[5], fhi[5], fbl[2], fbh[2];
#define IMC_AFRAG(GB)                                                                            \
  {                                                                                              \
    const int32_t* pl_ = reinterpret_cast<const int32_t*>(                                       \
        lds + ((GB) < 12 ? a_win0 + 32 * ((GB) + 3) : a_win1 + 32 * ((GB)-12)));                 \
    const int32_t* ph_ = pl_ + ((GB) < 12 ? kWin0 : kWin1) * 4;                                  \
    flo[((GB) + 5) % 5] = v4i{pl_[0], pl_[1], pl_[2], pl_[3]};                                   \
    fhi[((GB) + 5) % 5] = v4i{ph_[0], ph_[1], ph_[2], ph_[3]};                                   \
  }
#define IMC_BFRAG(Y, ST)                                                                         \
  fbl[(Y) & 1] = *reinterpret_cast<const v4i*>(lds + ((ST) + b_off + (Y) * 2048));               \
  fbh[(Y) & 1] = *reinterpret_cast<const v4i*>(lds + ((ST) + b_off + (Y) * 2048 + 1024));

#define IMC_SGB(MASK, N) __builtin_amdgcn_sched_group_barrier(MASK, N, 0);

  // prologue: window 0 of segment 0; database units -1 (its part of step 0) and 0
  if constexpr (DBS) {
#pragma unroll
    for (int j = 0; j < kB; ++j) {
      IMC_BLOAD(j, 4, -1)
      IMC_BLOAD(j, 0, 0)
    }
#pragma unroll
    for (int j = 0; j < kB; ++j) {
      IMC_BSTORE(j, 4, uint32_t(kPairStage))
      IMC_BSTORE(j, 0, 0u)
      IMC_BLOAD(j, 1, 1)
    }
  } else {
    v4i pa[4][2];
#pragma unroll
    for (int h = 0; h < kParts; h += 4) {
#pragma unroll
      for (int p = 0; p < 4; ++p) { IMC_ALOAD(pa[p], 0, h + p, 0) }
#pragma unroll
      for (int p = 0; p < 4; ++p) { IMC_ASTORE(pa[p], 0, h + p) }
    }
    IMC_ALOAD(ra, 1, 0, 0)
  }
  __syncthreads();
  if (LIVE) {
    IMC_BFRAG(0, uint32_t(kPairStage))
#pragma unroll
    for (int g = -3; g <= 0; ++g) { IMC_AFRAG(g) }
  }
  __syncthreads();

  for (int seg = 0; seg < kSegs; ++seg) {
    // 25 is odd: the parity of t that goes with a stage swaps with every segment
    const uint32_t st_even = (seg & 1) * kPairStage;
    const uint32_t st_odd = kPairStage - st_even;
    const bool more = seg + 1 < kSegs;
    const int k0 = seg * kT, seg_next = min(seg + 1, kSegs - 1);
#pragma unroll
    for (int j = 0; j < kB; ++j) asm volatile("" : "+v"(bsrc[j]), "+v"(bdst[j]));
    // the 25 steps written out: every ring index below is a constant
    const auto step = [&](auto tc) __attribute__((always_inline)) {
      constexpr int t = decltype(tc)::value;
      const uint32_t st_read = (t & 1) ? st_odd : st_even, st_write = (t & 1) ? st_even : st_odd;
      // Query windows: window 1 of this segment (read from step 11 on) is
      // stored in steps 2 .. 9, window 0 of the next one (read at step 24,
      // this one's last at step 10) in steps 14 .. 21; a part is loaded when
      // the one before it is stored.
      constexpr bool staged = !DBS && ((t >= 2 && t < 10) || (t >= 14 && t < 22));
      // 4 x 12 MFMAs, one group for each 16 of the wave's entries.  Each group
      // first reads the next group's database fragments; the third reads the
      // next step's query fragments; the first and third hold the staging of
      // the database, the first that of the queries, a step after its loads.
      const auto group = [&](auto yc) __attribute__((always_inline)) {
        constexpr int y = decltype(yc)::value;
        if (y == 0) __builtin_amdgcn_sched_barrier(0);
        if constexpr (LIVE) {
          IMC_BFRAG((y + 1) & 3, st_read)
          if constexpr (y == 2 && t + 1 < kT) { IMC_AFRAG(t + 1) }
#pragma unroll
          for (int a2 = 2; a2 >= 0; a2 -= 2) {
#pragma unroll
            for (int i = 0; i < 6; ++i) {
              // two a's together: their high-limb products last
              const int a = a2 + 1 - (i < 4 ? i >> 1 : i & 1), f = (t - a + 5) % 5;
              if (i >= 4)
                acc1[a][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fhi[f], fbl[y & 1], acc1[a][y], 0, 0, 0);
              else if (i & 1)
                acc0[a][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(flo[f], fbl[y & 1], acc0[a][y], 0, 0, 0);
              else
                acc1[a][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(flo[f], fbh[y & 1], acc1[a][y], 0, 0, 0);
            }
          }
        }
        if constexpr (DBS && (y & 1) == 0) {
#pragma unroll
          for (int j = 0; j < kB / 2; ++j) {
            IMC_BSTORE(j + y / 2 * (kB / 2), (t + 1) % 5, st_write)
          }
#pragma unroll
          for (int j = 0; j < kB / 2; ++j) {
            IMC_BLOAD(j + y / 2 * (kB / 2), (t + 2) % 5, k0 + t + 2)
          }
        }
        if constexpr (staged && y == 0) {
          constexpr int p = t < 10 ? t - 2 : t - 14;
          if constexpr (t < 10) {
            IMC_ASTORE(ra, 1, p)
            if constexpr (p + 1 < kParts) {
              IMC_ALOAD(ra, 1, p + 1, seg)
            } else {
              IMC_ALOAD(ra, 0, 0, seg_next)
            }
          } else {
            IMC_ASTORE(ra, 0, p)
            if constexpr (p + 1 < kParts) {
              IMC_ALOAD(ra, 0, p + 1, seg_next)
            } else {
              IMC_ALOAD(ra, 1, 0, seg_next)
            }
          }
        }
        if constexpr (LIVE) {
          IMC_SGB(0x008, 1) IMC_SGB(0x100, 1) IMC_SGB(0x008, 1) IMC_SGB(0x100, 1)
          if constexpr (y == 2 && !DBS) {
            IMC_SGB(0x008, 1) IMC_SGB(0x100, 1) IMC_SGB(0x008, 1) IMC_SGB(0x100, 1)
            IMC_SGB(0x008, 1) IMC_SGB(0x100, 1) IMC_SGB(0x008, 1) IMC_SGB(0x100, 1) IMC_SGB(0x008, 6)
          } else if constexpr (DBS && PH == 0 && (y & 1) == 0) {
#pragma unroll
            for (int i = 0; i < 9; ++i) { IMC_SGB(0x008, 1) IMC_SGB(0x002, 6) }
            IMC_SGB(0x200, 2) IMC_SGB(0x008, 1) IMC_SGB(0x020, 4)
          } else if constexpr (DBS && (y & 1) == 0) {
            IMC_SGB(0x008, 2) IMC_SGB(0x200, 1) IMC_SGB(0x008, 1) IMC_SGB(0x200, 1) IMC_SGB(0x008, 2)
            IMC_SGB(0x020, 1) IMC_SGB(0x008, 2) IMC_SGB(0x020, 1) IMC_SGB(0x008, 3)
          } else if constexpr (staged && y == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) { IMC_SGB(0x008, 1) IMC_SGB(0x002, 8) }
            IMC_SGB(0x200, 1) IMC_SGB(0x008, 1) IMC_SGB(0x200, 1) IMC_SGB(0x008, 1) IMC_SGB(0x020, 2)
          } else {
            IMC_SGB(0x008, 10)
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      group(std::integral_constant<int, 0>{});
      group(std::integral_constant<int, 1>{});
      group(std::integral_constant<int, 2>{});
      group(std::integral_constant<int, 3>{});
      if (t == kT - 1 && LIVE && more) {
#pragma unroll
        for (int g = -3; g <= 0; ++g) { IMC_AFRAG(g) }
      }
      __syncthreads();
    };
    for_each_step(step, std::make_integer_sequence<int, kT>{});
  }
#undef IMC_SGB
#undef IMC_BLOAD
#undef IMC_BSTORE
#undef IMC_ALOAD
#undef IMC_ASTORE
#undef IMC_AFRAG
#undef IMC_BFRAG
}

// Folds the accumulators to Z_2^16 and writes them: MODE 0 keeps P in the
// rows of s + 4, 1 writes the rows of s, 2 takes the third product from P.
// 16 x 16 block: lane l holds column l % 16, register e row 4 (l / 16) + e,
// i.e. query l / 16 and b = e.
template <int MODE>
__device__ __forceinline__ void pair_out(const PairDotArgs& args, uint32_t u, uint32_t t_col, int vec,
                                         const v4i (&acc0)[4][4], const v4i (&acc1)[4][4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t qi = u * kPairQ + (wave >> 1) * 4 + (lane >> 4);
  if (qi >= args.q) return;
  const uint64_t col0 = uint64_t(t_col) * kPairN + (wave & 1) * 64 + (lane & 15);
  uint16_t* out = args.out[vec] + uint64_t(qi) * args.r * args.ld + col0;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t ri = 8 * a + e + (MODE == 1 ? 0 : 4);
      if (ri >= args.r) continue;
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        if (col0 + 16 * y >= args.n) continue;
        uint16_t* p = out + ri * args.ld + 16 * y;
        const uint32_t z = uint32_t(acc0[a][y][e]) + (uint32_t(acc1[a][y][e]) << 8);
        *p = MODE == 2 ? uint16_t(*p - z) : uint16_t(z);
      }
    }
}

// The three products of a tile, as a wave of one staging role runs them.
template <int K, bool LIVE, bool DBS>
__device__ __forceinline__ void pair_tile(const PairDotArgs& args, const int8_t* __restrict__ bbase, uint32_t u,
                                          uint32_t t_col, int vec, int8_t* lds) {
  const uint64_t blk0 = uint64_t(t_col) * (kPairN / 32);
  v4i acc0[4][4], acc1[4][4];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc0[i >> 2][i & 3] = acc1[i >> 2][i & 3] = v4i{0, 0, 0, 0};
  pair_phase<0, K, LIVE, DBS>(args, bbase, u, blk0, vec, lds, acc0, acc1);
  if (LIVE) pair_out<0>(args, u, t_col, vec, acc0, acc1);
  pair_phase<1, K, LIVE, DBS>(args, bbase, u, blk0, vec, lds, acc0, acc1);
  if (LIVE) pair_out<1>(args, u, t_col, vec, acc0, acc1);
#pragma unroll
  for (int i = 0; i < 16; ++i) acc0[i >> 2][i & 3] = acc1[i >> 2][i & 3] = v4i{0, 0, 0, 0};
  pair_phase<2, K, LIVE, DBS>(args, bbase, u, blk0, vec, lds, acc0, acc1);
  if (LIVE) pair_out<2>(args, u, t_col, vec, acc0, acc1);
}

template <int K>
__global__ void __launch_bounds__(kPairThreads) pair_dot_kernel(PairDotArgs args) {
  using G = Geo<K>;
  extern __shared__ __align__(16) int8_t lds[];
  const int vec = blockIdx.z;
  // XCD-aware order: every query tile of a column tile runs on one XCD
  const uint32_t i = blockIdx.x, xcd = i & 7, s8 = i >> 3;
  const uint32_t u = s8 % args.mt, t_col = (s8 / args.mt) * 8 + xcd;
  if (t_col >= args.nt) return;
  const int8_t* bbase = args.b + size_t(args.b_block0 + uint64_t(t_col) * (kPairN / 32)) * G::kBlockBytes +
                        size_t(2 * vec) * G::kPlaneBlockBytes;
  // a wave whose queries are all past the last one only stages operands
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool live = u * kPairQ + (wave >> 1) * 4 < args.q;
  if (wave < 4) {
    if (live)
      pair_tile<K, true, true>(args, bbase, u, t_col, vec, lds);
    else
      pair_tile<K, false, true>(args, bbase, u, t_col, vec, lds);
  } else {
    if (live)
      pair_tile<K, true, false>(args, bbase, u, t_col, vec, lds);
    else
      pair_tile<K, false, false>(args, bbase, u, t_col, vec, lds);
  }
}

template <int K>
static hipError_t launch_pair_k(PairDotArgs d, bool mask, hipStream_t s) {
  d.mt = (d.q + kPairQ - 1) / kPairQ;
  d.nt = uint32_t((d.n + kPairN - 1) / kPairN);
  const uint64_t groups = uint64_t((d.nt + 7) / 8) * 8 * d.mt;
  if (groups > 0x7FFFFFFFull) return hipErrorInvalidValue;
  auto kern = pair_dot_kernel<K>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kPairLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(unsigned(groups), 1, mask ? 2 : 1), dim3(kPairThreads), kPairLds, s, d);
  return hipGetLastError();
}

static hipError_t launch_pair(const RotCall& c, hipStream_t s, bool galois) {
  PairDotArgs d;
  d.qop = c.qop;
  d.qidx = c.qidx;
  d.b = c.b;
  d.out[0] = c.code;
  d.out[1] = c.mask;
  d.ld = c.ld;
  d.q = c.q;
  d.r = c.r;
  d.s0 = c.rot[0];
  d.b_block0 = c.first_entry / 32;
  d.b_blocks = (c.n + 31) / 32;
  d.n = c.n;
  d.mt = d.nt = 0;
  return galois ? launch_pair_k<kKGalois>(d, c.mask != nullptr, s) : launch_pair_k<kK>(d, c.mask != nullptr, s);
}

// The call's columns from `from` on.
static RotCall columns_from(RotCall c, uint64_t from) {
  c.first_entry += from;
  c.n -= from;
  c.code += from;
  if (c.mask) c.mask += from;
  return c;
}

static hipError_t launch_rot_rounds(const RotCall& c, hipStream_t s, bool galois, const DotScratch& scratch) {
  RotCall first = c;
  first.n = rot_first_cols(c.q, c.r, c.n, c.mask ? 2 : 1, dot_room(scratch, galois));
  const hipError_t e = launch_rot_dot(first, s, 0, galois, scratch);
  return e != hipSuccess || first.n == c.n ? e : launch_rot_dot(columns_from(c, first.n), s, 0, galois, scratch);
}

hipError_t launch_rotations(const RotCall& c, hipStream_t s, bool galois, const DotScratch& scratch) {
  if (c.q == 0 || c.n == 0) return hipSuccess;
  const RotPlan p = rot_plan(c.q, c.r, c.rot, c.n, c.mask ? 2 : 1, dot_room(scratch, galois));
  if (p.n == 0) return launch_rot_rounds(c, s, galois, scratch);
  RotCall main = c;
  main.q = p.q;
  const RotCall right = columns_from(main, p.n);
  main.n = p.n;
  hipError_t e = launch_pair(main, s, galois);
  if (e == hipSuccess && right.n) e = launch_rot_rounds(right, s, galois, scratch);
  if (e == hipSuccess && p.q < c.q) {
    RotCall below = c;
    below.q = c.q - p.q;
    if (c.qidx)
      below.qidx += p.q;
    else
      below.qop += size_t(p.q) * (galois ? Geo<kKGalois>::kQopRowBytes : Geo<kK>::kQopRowBytes);
    const uint64_t off = uint64_t(p.q) * c.r * c.ld;
    below.code += off;
    if (below.mask) below.mask += off;
    e = launch_rot_rounds(below, s, galois, scratch);
  }
  return e;
}

}  // namespace imc
