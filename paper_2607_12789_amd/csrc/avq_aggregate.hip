// Per-codeword counts and value sums, Eq. (aggregates), with the Alg. 1
// convention that a parent row covers its whole cell and a child row the keys
// that moved to it; and the same pass with the child compare of Alg. 1 in it.
//
// A family is a parent and its Ch children (Ch = 0, a flat codebook: 16, 8, 4,
// 2 or 1 consecutive parents, see flat_shift). One workgroup owns one (batch,
// head) and a range of F families and is the only writer of their rows, so
// there are no float atomics and no partial results in HBM. The workgroup
//   1. scans the head's codes once: every wave compacts the keys of the range
//      into a private list in LDS, then counts them per family (integer LDS
//      atomics on full waves);
//   2. gives every family with keys whole groups of 32 slots in a key list and
//      scatters the keys into their family's slots;
//   3. deals the groups to its waves in equal contiguous runs. For a group
//      of 32 keys of one family a wave reads the 32 value rows (FUSED: and
//      the 32 key rows, whose child compare, avq_child.hpp, tells each key's
//      row), and adds them with matrix products: sums^T += onehot . V, where
//      row x of the 16 x 32 one-hot operand has a 1 for every key of row x
//      and row 8 a 1 for every key (the whole cell). Products with 0 and 1
//      are exact, the sums are fp32, and the same product with a column of
//      ones gives the counts. So the keys of a family need no order, the rows
//      of K and V arrive together, and a key costs one MFMA column instead of
//      an unpack and an add per value;
//   4. a wave that holds all of a family's groups writes its rows; the parts
//      of a family that spans waves meet in LDS, added in wave order by the
//      wave that holds the family's first group.
// The next group's rows are requested as soon as a group's registers are
// consumed, so a wave always has 8 (FUSED: 16 at d = 128) row loads in flight.
//
// The key list takes the LDS that is left. A range with more keys takes its
// families in batches that fit, and a single family that does not fit takes
// its keys in segments of the head, with the sums kept in registers from one
// to the next.
//
// What bounds it: at large sizes HBM (each value and key row is read once),
// at small ones the chain of phases of one workgroup; with few keys per family
// (about 16 and less) a wave's stores: the wait for the next group's rows is
// one for the family's stores as well. The precompute (parent assignment +
// fused pass), bf16, us, one row of a family after the other by vector adds ->
// by these products: B = 2, H = 16, N = 16384, d = 128, M0 = 256, Ch = 8: 104 ->
// 96 (the pass itself reads K and V at about 4.7 TB/s once it streams); B = 1,
// H = 16, N = 65536, M0 = 512: 282 -> 261; B = 8, H = 12, N = 4096, d = 64, M0 =
// 256: 89 -> 58; B = 4, H = 12, N = 1024, d = 64, M0 = 64: 35 -> 17. Aggregation
// with sums, fp32, d = 128, 96 x 512 families, N = 1500, Ch = 8: 128 -> 152.
//
// Packed aggregates (avq_packed.hpp): the mean value (sum / count) of every
// code rounded to the input type, in octets of 8 codes laid out as the
// attention kernel's MFMA operands, [octet][d][8], with n and ln n per code.
// Rows 0 .. 7 of an accumulator tile are one child octet (Ch = 16: tile 1 the
// second; flat: rows 0 .. 7 and 8 .. 15 are two parent octets).
#include "avq_child.hpp"
#include "avq_common.hpp"
#include "avq_launch.hpp"
#include "avq_packed.hpp"

#include <algorithm>
#include <type_traits>

namespace avq {

constexpr int kMaxFamilies = 64;  // families per workgroup, at most: one per lane
constexpr int kGroup = 32;        // keys per group

enum AggMode {
  kAggCodes,  // codes given, Ch >= 1
  kAggFlat,   // codes given, Ch = 0: families of 16 parents
  kAggFlatFew,  // the same with fewer parents per family
  kAggFused,  // parent indices given; the child compare writes the codes
};

struct FusedArgs {
  const void* K;   // [B][H][N][d]
  const void* Cp;  // [H][M0][d]
  const void* Cc;  // [H][M0][Ch][d]
  int32_t* code_idx;  // out: [B][H][N]
  int H;
};

// NT: accumulator tiles (and candidate tiles) per family, 1 for Ch <= 8, 2 for
// Ch = 16.
template <typename T, int D, int NT, int MODE, bool SMALL>
struct AggCfg {
  static constexpr bool kB = Elem<T>::kBf16;
  static constexpr bool kFlat = MODE == kAggFlat || MODE == kAggFlatFew;
  static constexpr bool kFused = MODE == kAggFused;
  // SMALL: 4 workgroups of 4 waves per CU (2 where the registers or the LDS
  // hold no more), whose phases overlap, instead of one of up to 16 waves (see
  // kSmallKeys). Otherwise as many waves
  // as the registers (16: 128 per lane, 12: 168, 8: 256) and the LDS (flat at
  // d = 128: 8) allow; the fused bf16 pass at d = 128 spills with 168
  // registers and is faster with 8 waves (c4 precompute 104 -> 96 us).
  static constexpr int kPerCU = SMALL ? (kB && D == 64 ? 4 : 2) : 1;
  static constexpr int kWaves =
      SMALL      ? 4
      : D == 128 ? (kFlat || kFused || NT == 2 ? 8 : kB ? 16 : 12)
                 : (NT == 2 ? (kFused && !kB ? 8 : 12) : kFused && !kB ? 12 : 16);
  static constexpr int kLds = 160 * 1024 / kPerCU;  // of one workgroup
  static constexpr int kThreads = kWaves * kWave;
  static constexpr int CT = D / 16;            // 16-column tiles
  static constexpr int ROWS = kFlat ? 16 : NT == 2 ? 17 : 9;  // rows held of a family
  static constexpr int OCTS = kFlat ? 2 : 1;  // octets written at a time
  static constexpr int OCT_BYTES = 8 * D * (int)sizeof(T);
  // LDS: the fixed tables, one partial slot and one staging area per wave,
  // the parent means of the range, then the key list
  struct Tables {
    int hist[kMaxFamilies];        // keys per family
    int gstart[kMaxFamilies + 1];  // first group of each family of the batch
    int cursor[kMaxFamilies];      // keys scattered so far
    int spilled;                   // some wave's private list was too short
    float cell[kMaxFamilies];      // cell sizes (n of the parents)
    // row bits of the group's keys, read as 16-byte vectors
    alignas(16) uint16_t onehot[kWaves][NT][kGroup];
  };
  static constexpr int al16(int x) { return (x + 15) / 16 * 16; }
  static constexpr int OFF_SLOT = al16((int)sizeof(Tables));
  static constexpr int SLOT_BYTES = al16(ROWS * D * 4 + ROWS * 4);
  static constexpr int OFF_STAGE = OFF_SLOT + kWaves * SLOT_BYTES;
  static constexpr int STAGE_BYTES = OCTS * OCT_BYTES;
  static constexpr int OFF_PMEAN = OFF_STAGE + kWaves * STAGE_BYTES;
  static constexpr int off_list(int F) {
    return OFF_PMEAN + (kFlat ? 0 : F * D * (int)sizeof(T));
  }
  // while the codes are scanned, the slots, staging areas and parent means
  // hold one private key list per wave
  static constexpr int priv_cap(int F) {
    return (off_list(F) - OFF_SLOT) / (4 * kWaves) / 16 * 16;
  }
  static_assert(OFF_PMEAN + (kFlat ? 0 : kMaxFamilies * D * (int)sizeof(T)) +
                        4 * kGroup * kMaxFamilies <= kLds,
                "a key list of one group per family fits the LDS");
};

// Families of a flat codebook, of 2^rsh parents each: whole octets, as many as
// hold the M0 parents (the padding octets after them belong to none).
constexpr int flat_families(int M0, int rsh) {
  return rsh >= 3 ? (M0 + (1 << rsh) - 1) >> rsh : (M0 + 7) / 8 << (3 - rsh);
}

// log2 of the parents per family of a flat codebook: 16, as many as a product
// has rows, or fewer where that leaves CUs without a workgroup and the keys
// are more than a few; the most that give every one of `workgroups` a family.
// Aggregation in us, 16 parents / the chosen number: bf16, 1 head x 256 parents,
// N = 2^20, d = 128: 1000 / 222; 4 x 128, N = 65536: 57.3 / 31.0; 32 x 64, N = 8192,
// d = 64: 20.8 / 14.0; 1 x 8, N = 65536, d = 64: 262 / 50; fp32, 4 x 128, N = 65536, d =
// 128: 158.7 / 43.4; but 8 x 500, N = 300, d = 128: 6.0 / 6.4 (8 parents; 16 taken).
constexpr int flat_shift(long long BH, int N, int M0, long long workgroups) {
  int rsh = 4;
  if (N > 512)
    while (rsh > 0 && BH * flat_families(M0, rsh) < workgroups) --rsh;
  return rsh;
}

// A value row piece of one lane: 16 bytes (bf16 at d = 64: 8), at the
// lane's columns; column col(t, c) belongs to column tile t.
template <typename T, int D>
struct ValRow {
  static constexpr int W = D * (int)sizeof(T) / 64;  // 32-bit words per lane
  static constexpr int CPW = W > 4 ? 4 : W;          // ... of one load
  uint32_t w[W];
  __device__ __forceinline__ void load(const T* row, int c) {
    const unsigned char* p = reinterpret_cast<const unsigned char*>(row);
#pragma unroll
    for (int i = 0; i < W / CPW; ++i) {
      if constexpr (CPW == 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(p + 256 * i + 16 * c);
        w[4 * i] = v.x;
        w[4 * i + 1] = v.y;
        w[4 * i + 2] = v.z;
        w[4 * i + 3] = v.w;
      } else {
        const uint2 v = *reinterpret_cast<const uint2*>(p + 8 * c);
        w[0] = v.x;
        w[1] = v.y;
      }
    }
  }
  // the same from a head's base and a 32-bit byte offset (bf16: a head is
  // below 4 GiB), so that the base stays in scalar registers
  __device__ __forceinline__ void load_key(const T* head, uint32_t key, int c) {
    if constexpr (sizeof(T) == 2) {
      const uint32_t off = key * (uint32_t)(D * sizeof(T));
      load(reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(head) + (size_t)(off + (uint32_t)(4 * CPW * c))), 0);
    } else {
      load(head + (size_t)key * D, c);
    }
  }
  // first column of the lane's run of consecutive columns, tiles t .. t + RUN - 1
  static constexpr int RUN = CPW * 4 / (int)sizeof(T);
  static __device__ __forceinline__ int col(int t, int c) {
    return (t / RUN) * 16 * RUN + RUN * c + t % RUN;
  }
};

template <typename T, int D, int NT, int MODE, bool SMALL>
__global__ __launch_bounds__((AggCfg<T, D, NT, MODE, SMALL>::kThreads))
__attribute__((amdgpu_waves_per_eu(AggCfg<T, D, NT, MODE, SMALL>::kWaves *
                                   AggCfg<T, D, NT, MODE, SMALL>::kPerCU / 4)))
void aggregate_kernel(
    const T* __restrict__ V, const int32_t* __restrict__ code_idx, float* __restrict__ Vbar,
    int32_t* __restrict__ counts, unsigned char* __restrict__ packed, int N, int M0, int Ch,
    int F, int ranges, int cap, int rsh, FusedArgs fa) {
  using Cfg = AggCfg<T, D, NT, MODE, SMALL>;
  constexpr bool kB = Cfg::kB, kFlat = Cfg::kFlat, kFused = Cfg::kFused;
  constexpr int W = Cfg::kWaves, CT = Cfg::CT, ROWS = Cfg::ROWS;
  using VR = ValRow<T, D>;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  typename Cfg::Tables& L = *reinterpret_cast<typename Cfg::Tables*>(lds_raw);
  T* pmean = reinterpret_cast<T*>(lds_raw + Cfg::OFF_PMEAN);  // [F][D]
  uint32_t* list = reinterpret_cast<uint32_t*>(lds_raw + Cfg::off_list(F));

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const int g = lane / 16, c = lane % 16;
  const int blk = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = blk / ranges;
  const PackedLayout PL = packed_layout(M0, Ch, D, (int)sizeof(T));
  if constexpr (MODE != kAggFlatFew) rsh = 4;
  const int R = 1 << rsh;  // flat: parents per family
  const int n_fam = kFlat ? flat_families(M0, rsh) : M0;
  const int p0 = (blk % ranges) * F;
  const int nfam = min(F, n_fam - p0);
  const int Mtot = M0 * (1 + Ch);
  const int ch_shift = kFlat ? 0 : 31 - __builtin_clz(Ch);  // Ch is a power of two
  const int32_t* codes = code_idx + (size_t)bh * N;  // FUSED: parent indices
  const T* vhead = V + (size_t)bh * N * D;
  const T* khead = static_cast<const T*>(fa.K) + (kFused ? (size_t)bh * N * D : 0);
  const int h = kFused ? bh % fa.H : 0;

  // (family of this range, row) of a code: false if it belongs to another
  // range. Rows: 0 the parent stays, 1 + x child x; flat: the parent's row.
  auto locate = [&](int code, int& f, int& row) {
    row = 0;
    if constexpr (kFused) {
      f = code - p0;
    } else if constexpr (kFlat) {
      f = (code >> rsh) - p0;
      row = code & (R - 1);
      if (code >= M0) f = -1;
    } else {
      const int x = code - M0;
      f = (x < 0 ? code : x >> ch_shift) - p0;
      row = x < 0 ? 0 : 1 + (x & (Ch - 1));
      if (code >= Mtot) f = -1;
    }
    return (unsigned)f < (unsigned)nfam && code >= 0;
  };
  // f(key, code) for the keys [k0, k1): 8 codes in flight per lane
  auto scan = [&](int k0, int k1, auto&& f) {
    constexpr int kStep = 8;
    for (int b = k0 + tid; b < k1; b += kStep * Cfg::kThreads) {
      int cd[kStep];
#pragma unroll
      for (int i = 0; i < kStep; ++i) {
        const int j = b + i * Cfg::kThreads;
        cd[i] = j < k1 ? codes[j] : -1;
      }
#pragma unroll
      for (int i = 0; i < kStep; ++i) f(b + i * Cfg::kThreads, cd[i]);
    }
  };

  // ---- 1. the range's keys, and keys per family ---------------------------
  // Each wave compacts the keys of this range among its share of the codes
  // into a private list (key in 21 bits, row in 5, family in 6; a ballot and
  // one LDS write per 64 codes), then counts and scatters from there: the LDS
  // atomics run on full waves of the range's keys, not on the few lanes per 64
  // codes that hold one. A wave whose share does not fit its list leaves the
  // scan to the general path below, as do heads of more than 2^21 keys and
  // ranges that need several batches (the lists do not outlive the first).
  constexpr int kKeyBits = 21;
  uint32_t* priv = reinterpret_cast<uint32_t*>(lds_raw + Cfg::OFF_SLOT) + wave * Cfg::priv_cap(F);
  const int priv_cap = Cfg::priv_cap(F);
  int n_priv = 0;  // wave-uniform
  const bool try_priv = N <= 1 << kKeyBits;
  if (tid < kMaxFamilies) {
    L.hist[tid] = 0;
    L.cursor[tid] = 0;
  }
  if (tid == 0) L.spilled = 0;
  if (try_priv) {
    auto take = [&](int key, int code) {
      int f, row;
      const bool in = locate(code, f, row);
      const unsigned long long mk = __ballot(in);
      const int pos = n_priv + bits_below(mk);
      if (in && pos < priv_cap)
        priv[pos] = (uint32_t)key | (uint32_t)row << kKeyBits | (uint32_t)f << (kKeyBits + 5);
      n_priv += __popcll(mk);
    };
    // a block of 512 keys per wave and step, the next one's codes in flight
    constexpr int kPer = 8, kBlock = kPer * kWave;
    const int stride = W * kBlock;
    int nx[kPer];
    if (N % 4 == 0) {  // the head's codes are 16-byte aligned: four per load
      auto fetch = [&](int b) {
#pragma unroll
        for (int i = 0; i < kPer / 4; ++i) {
          const int j = b + 4 * kWave * i + 4 * lane;
          const int4 v = j < N ? *reinterpret_cast<const int4*>(codes + j) : int4{-1, -1, -1, -1};
          nx[4 * i] = v.x;
          nx[4 * i + 1] = v.y;
          nx[4 * i + 2] = v.z;
          nx[4 * i + 3] = v.w;
        }
      };
      fetch(wave * kBlock);
      for (int b = wave * kBlock; b < N; b += stride) {
        int cd[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) cd[i] = nx[i];
        if (b + stride < N) fetch(b + stride);
#pragma unroll
        for (int i = 0; i < kPer; ++i) take(b + 4 * kWave * (i / 4) + 4 * lane + i % 4, cd[i]);
      }
    } else {
      auto fetch = [&](int b) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
          const int j = b + kWave * i + lane;
          nx[i] = j < N ? codes[j] : -1;
        }
      };
      fetch(wave * kBlock);
      for (int b = wave * kBlock; b < N; b += stride) {
        int cd[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) cd[i] = nx[i];
        if (b + stride < N) fetch(b + stride);
#pragma unroll
        for (int i = 0; i < kPer; ++i) take(b + kWave * i + lane, cd[i]);
      }
    }
  }
  __syncthreads();
  if (n_priv > priv_cap || !try_priv) {
    if (lane == 0) L.spilled = 1;
  } else {
    for (int e = lane; e < n_priv; e += kWave) atomicAdd(&L.hist[priv[e] >> (kKeyBits + 5)], 1);
  }
  __syncthreads();
  const bool spilled = L.spilled != 0;
  if (spilled) {
    __syncthreads();
    if (tid < kMaxFamilies) L.hist[tid] = 0;
    __syncthreads();
    scan(0, N, [&](int, int code) {
      int f, row;
      if (locate(code, f, row)) atomicAdd(&L.hist[f], 1);
    });
    __syncthreads();
  }

  // The lane index through an empty asm statement: the addresses formed from
  // it are computed where they are used, not hoisted out of the group loop and
  // held (or spilled) through it.
  auto hidden = [](int x) {
    asm volatile("" : "+v"(x));
    return x;
  };

  // a wave's LDS writes are read by its other lanes: LDS operations of one
  // wave complete in order
  auto wave_lds_fence = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  // ---- a family's sums ---------------------------------------------------
  // acc[nt][t][r]: row 4 g + r of tile nt at column VR::col(t, c); an[nt][r]
  // the row's count
  f32x4 acc[NT][CT], an[NT];
  auto zero_acc = [&]() {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      an[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < CT; ++t) acc[nt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  // held row x of tile nt: its index among ROWS, or -1
  auto held = [&](int nt, int x) {
    if constexpr (kFlat) return x;
    return nt == 0 ? (x <= 8 ? x : -1) : (x < 8 ? 9 + x : -1);
  };
  auto slot_sum = [&](int w) { return reinterpret_cast<float*>(lds_raw + Cfg::OFF_SLOT + w * Cfg::SLOT_BYTES); };
  auto store_slot = [&]() {
    const int lq = hidden(lane), g = lq / 16, c = lq % 16;
    float* s = slot_sum(wave);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int x = held(nt, 4 * g + r);
        if (x < 0) continue;
#pragma unroll
        for (int t = 0; t < CT; t += 4)
          *reinterpret_cast<f32x4*>(&s[x * D + VR::col(t, c)]) =
              f32x4{acc[nt][t][r], acc[nt][t + 1][r], acc[nt][t + 2][r], acc[nt][t + 3][r]};
        if (c == 0) s[ROWS * D + x] = an[nt][r];
      }
  };
  auto add_slot = [&](int w) {
    const int lq = hidden(lane), g = lq / 16, c = lq % 16;
    const float* s = slot_sum(w);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int x = held(nt, 4 * g + r);
        if (x < 0) continue;
#pragma unroll
        for (int t = 0; t < CT; t += 4) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(&s[x * D + VR::col(t, c)]);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[nt][t + i][r] += v[i];
        }
        an[nt][r] += s[ROWS * D + x];
      }
  };

  float* vb = Vbar ? Vbar + (size_t)bh * Mtot * D : nullptr;
  unsigned char* pk = packed ? packed + (size_t)bh * PL.bytes : nullptr;
  T* means = reinterpret_cast<T*>(pk);
  float* info = reinterpret_cast<float*>(pk + PL.info_off);
  int32_t* nb = counts + (size_t)bh * Mtot;
  constexpr float kNegInf = -__builtin_inff();
  constexpr float kLn2 = 0.6931471805599453f;
  auto ln_n = [&](float n) { return n > 0.f ? log2_hw(n) * kLn2 : kNegInf; };
  // writes every row of family f: sums, counts, its octets with their counts;
  // the parent's mean and cell size go to LDS
  auto write_family = [&](int f) {
    const int lq = hidden(lane), g = lq / 16, c = lq % 16;
    const int p = p0 + f;
    unsigned char* st = lds_raw + Cfg::OFF_STAGE + wave * Cfg::STAGE_BYTES;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      // the code of row x, or -1
      auto code_of = [&](int x) {
        if constexpr (kFlat) return x < R && R * p + x < M0 ? R * p + x : -1;
        return x < 8 ? (8 * nt + x < Ch ? M0 + p * Ch + 8 * nt + x : -1) : (x == 8 && nt == 0 ? p : -1);
      };
      float inv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int code = code_of(4 * g + r);
        const float n = an[nt][r];
        inv[r] = n > 0.f ? 1.f / n : 0.f;
        if (code >= 0) {
          if (c == 0) nb[code] = (int)n;
          if (vb) {
#pragma unroll
            for (int t = 0; t < CT; t += 4)
              *reinterpret_cast<f32x4*>(&vb[(size_t)code * D + VR::col(t, c)]) =
                  f32x4{acc[nt][t][r], acc[nt][t + 1][r], acc[nt][t + 2][r], acc[nt][t + 3][r]};
          }
        }
      }
      if (!pk) continue;
      if (!kFlat && nt == 0 && g == 2) {  // row 8: the parent
#pragma unroll
        for (int t = 0; t < CT; ++t) pmean[f * D + VR::col(t, c)] = (T)(acc[0][t][0] * inv[0]);
        if (c == 0) L.cell[f] = an[0][0];
      }
      // rows 0..7 (flat: and 8..15) through the staging area, so that each
      // store is 16 consecutive bytes per lane over the whole octet. 16-byte
      // units are XOR-swizzled so that the lanes' columns hit distinct banks.
      // (flat families of fewer than 8 parents: parts of an octet, stored as they
      // lie)
      constexpr int kUnits = Cfg::OCT_BYTES / 16;  // per octet
      auto swz = [&](int u) { return u ^ ((u >> 3) & 7); };
      const bool part = MODE == kAggFlatFew && R < 8;
      const bool mine = kFlat ? 4 * g < R : g < 2;  // rows of the octets
      const int oct = kFlat ? g / 2 : 0;  // octet of the staging area
      const int o0 = kFlat ? R * p / 8 : PL.PO + p * PL.CO + nt;  // the family's first
      const int q0 = part ? R * p % 8 : 4 * (g & 1);  // the lane's first slot in the octet
      if (mine) {
        unsigned char* so = st + oct * Cfg::OCT_BYTES;
#pragma unroll
        for (int t = 0; t < CT; ++t) {
          const int col = VR::col(t, c);
          using V4 = typename std::conditional<kB, bf16x4, f32x4>::type;
          const V4 o = {(T)(acc[nt][t][0] * inv[0]), (T)(acc[nt][t][1] * inv[1]),
                        (T)(acc[nt][t][2] * inv[2]), (T)(acc[nt][t][3] * inv[3])};
          if (part) {
            T* dst = means + ((size_t)o0 * D + col) * 8 + q0;
            if (R == 4) {
              *reinterpret_cast<V4*>(dst) = o;
            } else {
              dst[0] = o[0];
              if (R == 2) dst[1] = o[1];
            }
          } else if constexpr (kB) {
            *reinterpret_cast<V4*>(so + 16 * swz(col) + 2 * q0) = o;
          } else {
            *reinterpret_cast<V4*>(so + 16 * swz(2 * col + q0 / 4)) = o;
          }
        }
        if (c == 0) {
          float* io = &info[(size_t)(o0 + oct) * 16 + q0];
          f32x4 n4, l4;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            n4[r] = an[nt][r];
            l4[r] = ln_n(an[nt][r]);
          }
          if (!kFlat || R >= 4) {
            *reinterpret_cast<f32x4*>(io) = n4;
            *reinterpret_cast<f32x4*>(io + 8) = l4;
          } else {
#pragma unroll
            for (int r = 0; r < 2; ++r)
              if (r < R) {
                io[r] = n4[r];
                io[8 + r] = l4[r];
              }
          }
        }
      }
      if (part) continue;
      wave_lds_fence();
      constexpr int kOcts = kFlat ? 2 : 1;
#pragma unroll
      for (int i = 0; i < kOcts * kUnits / kWave; ++i) {
        const int u = lq + kWave * i;
        if (kFlat && u / kUnits * 8 >= R) break;  // wave-uniform
        const uint4 v = *reinterpret_cast<const uint4*>(st + (u / kUnits) * Cfg::OCT_BYTES + 16 * swz(u % kUnits));
        *reinterpret_cast<uint4*>(reinterpret_cast<unsigned char*>(means) +
                                  (size_t)(o0 + u / kUnits) * Cfg::OCT_BYTES + 16 * (u % kUnits)) = v;
      }
      wave_lds_fence();
    }
  };

  // ---- 2. and 3. in batches of families that fit the key list ------------
  for (int f0 = 0; f0 < nfam;) {
    // families f0 .. f1 - 1, groups for those with keys. Every wave finds the
    // same plan.
    int f1;
    bool giant;
    unsigned long long filled;  // families with keys
    {
      const int n = lane >= f0 && lane < nfam ? L.hist[lane] : 0;
      const int ng = (n + kGroup - 1) / kGroup;
      const int incl = wave_incl_scan(ng);
      if (lane < nfam) L.gstart[lane] = incl - ng;
      if (lane == nfam - 1) L.gstart[nfam] = incl;
      const int fit = __popcll(__ballot(lane >= f0 && lane < nfam && incl * kGroup <= cap));
      f1 = f0 + max(1, fit);
      // a family past the list: segments of the head that fit whatever they hold
      giant = fit == 0;
      filled = __ballot(lane >= f0 && lane < f1 && n > 0);
    }
    wave_lds_fence();
    // the family of group x (one of families f0 .. f1 - 1), the same in every lane
    auto family_of = [&](int x) {
      return (int)__builtin_ctzll(__ballot(lane >= f0 && lane < f1 && L.gstart[lane + 1] > x));
    };
    const bool from_priv = !spilled && f1 == nfam && f0 == 0 && !giant;
    zero_acc();
    for (int s0 = 0; s0 < N; s0 += giant ? cap : N) {
      const int s1 = giant ? min(N, s0 + cap) : N;
      // key k of a group lies in slot 8 (k % 4) + k / 4: lane group g reads
      // slots 8 g .. 8 g + 7, i.e. keys g, 4 + g, 8 + g, ...
      auto put = [&](int f, int key, int row) {
        const int k = atomicAdd(&L.cursor[f], 1);
        const int slot = L.gstart[f] * kGroup + (k & ~31) + (k & 3) * 8 + ((k & 31) >> 2);
        list[slot] = (uint32_t)key | (kFused ? 0u : (uint32_t)row << 24);
      };
      if (from_priv) {
        for (int e = lane; e < n_priv; e += kWave) {
          const uint32_t x = priv[e];
          put(x >> (kKeyBits + 5), x & ((1u << kKeyBits) - 1), (x >> kKeyBits) & 31u);
        }
      } else {
        scan(s0, s1, [&](int key, int code) {
          int f, row;
          if (locate(code, f, row) && f >= f0 && f < f1) put(f, key, row);
        });
      }
      __syncthreads();
      const int seg_n = L.cursor[f0];  // giant: keys of this segment
      const int NG = giant ? (seg_n + kGroup - 1) / kGroup : L.gstart[f1];
      const int gb = (int)((long long)NG * wave / W), ge = (int)((long long)NG * (wave + 1) / W);

      if (gb < ge) {
        using CTile = ChildTile<T, D, NT>;
        constexpr int KQ = CTile::KQ;
        using Frag = typename CTile::Frag;
        Frag kf[kFused ? 2 : 1][KQ];   // key rows: two tiles of 16 keys
        Frag cf[kFused ? NT : 1][KQ];  // the family's candidate rows
        f32x4 cn[kFused ? NT : 1];
        VR vr[8];
        uint32_t ent[8];    // list entries 8 g .. 8 g + 7 (key, row)
        uint32_t kent[2];   // FUSED: entries of compare columns c
        int f = giant ? f0 : family_of(gb);
        int n = 0;  // keys of the current group
        auto group_n = [&](int ff, int it) {
          const int tot = giant ? seg_n : L.hist[ff];
          return min(kGroup, tot - kGroup * (it - (giant ? 0 : L.gstart[ff])));
        };
        // list entries of group it (n keys): slots past n repeat the group's
        // first key (no group: key 0)
        auto read_entries = [&](int it, int nk) {
          const uint4* q = reinterpret_cast<const uint4*>(&list[it * kGroup + 8 * g]);
          const uint4 a = q[0], b = q[1];
          ent[0] = a.x;
          ent[1] = a.y;
          ent[2] = a.z;
          ent[3] = a.w;
          ent[4] = b.x;
          ent[5] = b.y;
          ent[6] = b.z;
          ent[7] = b.w;
          if constexpr (kFused) {
#pragma unroll
            for (int t = 0; t < 2; ++t) kent[t] = list[it * kGroup + 8 * (c / 4) + c % 4 + 4 * t];
          }
          if (nk < kGroup) {
            const uint32_t e0 = nk > 0 ? __builtin_amdgcn_readfirstlane(ent[0]) : 0u;
#pragma unroll
            for (int j = 0; j < 8; ++j) ent[j] = 4 * j + g < nk ? ent[j] : e0;
            if constexpr (kFused) {
#pragma unroll
              for (int t = 0; t < 2; ++t) kent[t] = 4 * (c % 4 + 4 * t) + c / 4 < nk ? kent[t] : e0;
            }
          }
        };
        auto load_k = [&]() {
          if constexpr (kFused) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              if constexpr (kB) {  // as ValRow::load_key
                const uint32_t off = kent[t] * (uint32_t)(D * sizeof(T)) + 16u * g;
                child_key<T, D, NT>(reinterpret_cast<const T*>(
                                        reinterpret_cast<const unsigned char*>(khead) + (size_t)off),
                                    0, kf[t]);
              } else {
                child_key<T, D, NT>(khead + (size_t)kent[t] * D, g, kf[t]);
              }
            }
          }
        };
        auto load_v = [&]() {
#pragma unroll
          for (int j = 0; j < 8; ++j) vr[j].load_key(vhead, ent[j] & 0xFFFFFFu, c);
        };
        auto load_rows = [&](int ff) {
          if constexpr (kFused)
            child_rows_load<T, D, NT>(static_cast<const T*>(fa.Cp), static_cast<const T*>(fa.Cc),
                                      h, M0, Ch, p0 + ff, g, c, cf);
        };
        n = group_n(f, gb);
        read_entries(gb, n);
        load_rows(f);
        load_k();
        load_v();
        bool fresh = true;              // candidate rows just loaded
        bool whole = giant ? false : L.gstart[f] >= gb;  // the family began in this run

        for (int it = gb; it < ge; ++it) {
          const bool last = !giant && L.gstart[f + 1] == it + 1;  // of the family
          const bool more = it + 1 < ge;
          // the next group's family, past those without keys
          const int fn = !last ? f : more ? __builtin_ctzll(filled & (~1ull << f)) : f1;
          // the 32 keys' row bits, two per word: bit x is accumulator row x
          uint32_t oh[NT][4];
          uint32_t kcur[2] = {0, 0};
          int rk[2] = {0, 0};
          if constexpr (kFused) {
            if (fresh) child_rows_finish<T, D, NT>(g, cf, cn);
            rk[0] = child_pick<T, D, NT>(cf, cn, kf[0], Ch, g, c);
            if (n > 16) rk[1] = child_pick<T, D, NT>(cf, cn, kf[1], Ch, g, c);
            if (g == 0) {
#pragma unroll
              for (int t = 0; t < 2; ++t) {
                const bool valid = 4 * (c % 4 + 4 * t) + c / 4 < n;
                const uint32_t bits = (1u << rk[t]) >> 1;  // children; none if it stays
                const int slot = 8 * (c / 4) + c % 4 + 4 * t;
                L.onehot[wave][0][slot] = (uint16_t)(valid ? (bits & 0xFFu) | 0x100u : 0u);
                if constexpr (NT == 2) L.onehot[wave][1][slot] = (uint16_t)(valid ? bits >> 8 : 0u);
                kcur[t] = valid ? kent[t] : 0xFFFFFFFFu;
              }
            }
            wave_lds_fence();
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
              const uint4 q = *reinterpret_cast<const uint4*>(&L.onehot[wave][nt][8 * g]);
              oh[nt][0] = q.x;
              oh[nt][1] = q.y;
              oh[nt][2] = q.z;
              oh[nt][3] = q.w;
            }
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              uint32_t w0[NT], w1[NT];
              auto bits_of = [&](int j, uint32_t (&w)[NT]) {
                const bool valid = 4 * j + g < n;
                const uint32_t row = ent[j] >> 24;
                if constexpr (kFlat) {
                  w[0] = valid ? 1u << row : 0u;
                } else {
                  const uint32_t b = (1u << row) >> 1;
                  w[0] = valid ? (b & 0xFFu) | 0x100u : 0u;
                  if constexpr (NT == 2) w[1] = valid ? b >> 8 : 0u;
                }
              };
              bits_of(2 * q, w0);
              bits_of(2 * q + 1, w1);
#pragma unroll
              for (int nt = 0; nt < NT; ++nt) oh[nt][q] = w0[nt] | (w1[nt] << 16);
            }
          }
          // the next group: its entries, and (FUSED) its candidate and key rows
          const int nn = more ? group_n(giant ? f : fn, it + 1) : 0;
          const int itn = more ? it + 1 : it;
          read_entries(itn, nn);
          if constexpr (kFused) {
            __builtin_amdgcn_sched_barrier(0);
            if (last && more) load_rows(fn);
            load_k();
            __builtin_amdgcn_sched_barrier(0);
            if (g == 0) {
#pragma unroll
              for (int t = 0; t < 2; ++t) {
                if (kcur[t] == 0xFFFFFFFFu) continue;
                const int p = p0 + f;
                fa.code_idx[(size_t)bh * N + kcur[t]] = rk[t] > 0 ? M0 + p * Ch + rk[t] - 1 : p;
              }
            }
          }
          // sums^T += onehot . V. Every group has keys; the branch keeps the block
          // apart (without it the compiler takes 4 registers more, spilled in the
          // fp32 pass at d = 128)
          if (n > 0) {
            // the one-hot rows as a bf16 operand; their product with ones is the
            // counts (exact, and for fp32 one product instead of eight)
            bf16x8 a[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
              uint32_t w[4];
#pragma unroll
              for (int q = 0; q < 4; ++q)  // bit c of both halves, as bf16 ones
                w[q] = __umul24((oh[nt][q] >> c) & 0x00010001u, 0x3F80u);
              __builtin_memcpy(&a[nt], w, 16);
            }
            if constexpr (kB) {
#pragma unroll
              for (int t = 0; t < CT; ++t) {
                uint32_t w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)  // keys 2q, 2q + 1 at the lane's column t
                  w[q] = __builtin_amdgcn_perm(vr[2 * q + 1].w[t / 2], vr[2 * q].w[t / 2],
                                               t % 2 ? 0x07060302u : 0x05040100u);
                bf16x8 b;
                __builtin_memcpy(&b, w, 16);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[nt][t] = mfma_bf16(a[nt], b, acc[nt][t]);
              }
            }
            const bf16x8 ones = {(bf16)1.f, (bf16)1.f, (bf16)1.f, (bf16)1.f,
                                 (bf16)1.f, (bf16)1.f, (bf16)1.f, (bf16)1.f};
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) an[nt] = mfma_bf16(a[nt], ones, an[nt]);
            if constexpr (!kB) {
              // step j adds keys 4 j .. 4 j + 3: none past the group's n keys (a
              // family of a few keys is mostly padding)
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                if (4 * j >= n) break;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                  const float x = (float)((oh[nt][j / 2] >> (c + 16 * (j % 2))) & 1u);
#pragma unroll
                  for (int t = 0; t < CT; ++t)
                    acc[nt][t] = mfma_f32(x, __uint_as_float(vr[j].w[t]), acc[nt][t]);
                }
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          load_v();
          __builtin_amdgcn_sched_barrier(0);
          if (last) {
            if (whole) write_family(f);
            else store_slot();
            zero_acc();
            whole = true;
          }
          fresh = last;
          f = fn;
          n = nn;
        }
        // a family that goes on in the next wave's run, begun in an earlier
        // one's: its part goes to the slot too (giant: after the last segment)
        if (!giant && f < f1 && !whole && L.gstart[f + 1] > ge) store_slot();
      }
      if (giant) {
        __syncthreads();
        if (tid == 0) L.cursor[f0] = 0;
        __syncthreads();
      }
    }
    if (giant) {
      if (wave > 0) store_slot();
      __syncthreads();
      if (wave == 0) {
        for (int w = 1; w < W; ++w) add_slot(w);
        write_family(f0);
      }
      __syncthreads();
    } else {
      __syncthreads();
      // the wave that holds the first, but not the last, group of a family
      const int NG = L.gstart[f1];
      auto run_end = [&](int w) { return (int)((long long)NG * (w + 1) / W); };
      const int gb = (int)((long long)NG * wave / W), ge = run_end(wave);
      if (gb < ge) {
        const int f = family_of(ge - 1);
        if (L.gstart[f + 1] > ge && L.gstart[f] >= gb) {
          for (int w = wave + 1; w < W; ++w) {
            if (run_end(w) > run_end(w - 1)) add_slot(w);
            if (run_end(w) >= L.gstart[f + 1]) break;
          }
          write_family(f);
        }
      }
      if (tid < kMaxFamilies) L.cursor[tid] = 0;  // for the next batch
      __syncthreads();
    }
    f0 = f1;
  }

  // ---- families without keys ------------------------------------------------
  // writes family f without keys: zeros alone, so no group's chain of loads,
  // products and stages is spent on it. Heads of few keys are mostly such
  // families. Aggregation or fused pass with it in us, a group of padding for
  // each / so: bf16, d = 128, 375 heads x 256 families, N = 25: 196 / 100; 147 x
  // 512, Ch = 16, N = 181: 397 / 283; 95 x 512, Ch = 8, N = 403: 175 / 135; fp32, d
  // = 128, 475 x 256, N = 1: 534 / 234.
  auto write_empty = [&](int f) {
    const int lane = hidden(tid % kWave), p = p0 + f;
    const uint32_t z = hidden(0);
    // n16 16-byte units of zeros
    auto zeros = [&](void* dst, int n16) {
      for (int i = lane; i < n16; i += kWave) static_cast<uint4*>(dst)[i] = uint4{z, z, z, z};
    };
    // rows of sums and counts: the parent and its children (flat: R parents)
    auto rows = [&](int code, int n) {
      if (lane < n) nb[code + lane] = z;
      if (vb) zeros(vb + (size_t)code * D, n * D / 4);
    };
    if constexpr (kFlat) {
      rows(R * p, min(R, M0 - R * p));
    } else {
      rows(p, 1);
      rows(M0 + p * Ch, Ch);
    }
    if (!pk) return;
    // n slots of octet o from slot q0 on, or (n a multiple of 8) whole octets
    auto slots = [&](int o, int q0, int n) {
      if (n % 8 == 0) {
        zeros(means + (size_t)o * D * 8, n / 8 * Cfg::OCT_BYTES / 16);
      } else {
        for (int i = lane; i < D * n; i += kWave)
          means[((size_t)o * D + i / n) * 8 + q0 + i % n] = T(__uint_as_float(z));
      }
      if (lane < n) {
        float* io = &info[(size_t)(o + lane / 8) * 16 + q0 + lane % 8];
        io[0] = __uint_as_float(z);
        io[8] = kNegInf;
      }
    };
    if constexpr (kFlat) {
      slots(R * p / 8, R * p % 8, R);
    } else {
      slots(PL.PO + p * PL.CO, 0, 8 * PL.CO);
      for (int i = lane; i < D; i += kWave) pmean[f * D + i] = T(__uint_as_float(z));
      if (lane == 0) L.cell[f] = __uint_as_float(z);
    }
  };
  {
    unsigned long long empty = __ballot(lane < nfam && L.hist[lane] == 0);
    if (empty != 0) {  // the same in every wave
      for (int i = 0; empty != 0; ++i, empty &= empty - 1)
        if (i % W == wave) write_empty(__builtin_ctzll(empty));
      __syncthreads();
    }
  }

  // ---- parent octets (flat: written above, but for the padding) ------------
  if (!pk) return;
  if constexpr (kFlat) {
    if (p0 + nfam == n_fam) {
      const int o0 = n_fam * R / 8;
      uint4* pad = reinterpret_cast<uint4*>(means + (size_t)o0 * D * 8);
      for (int i = tid; i < (PL.PO - o0) * Cfg::OCT_BYTES / 16; i += Cfg::kThreads) pad[i] = uint4{0, 0, 0, 0};
      for (int i = tid; i < (PL.PO - o0) * 16; i += Cfg::kThreads)
        info[(size_t)o0 * 16 + i] = i % 16 < 8 ? 0.f : kNegInf;
    }
  } else {
    const int p_end = p0 + nfam >= M0 ? 8 * PL.PO : p0 + nfam;  // the last range: the padding too
    if (F % 8 == 0) {
      const int o0 = p0 / 8;
      for (int i = tid; i < (p_end / 8 - o0) * D; i += Cfg::kThreads) {
        const int o = i / D, d = i % D;
        T v[8];
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) v[sl] = 8 * o + sl < nfam ? pmean[(8 * o + sl) * D + d] : T(0.f);
        uint4* dst = reinterpret_cast<uint4*>(means + ((size_t)(o0 + o) * D + d) * 8);
#pragma unroll
        for (int q = 0; q < (int)sizeof(T) / 2; ++q) {
          uint4 x;
          __builtin_memcpy(&x, reinterpret_cast<const unsigned char*>(v) + 16 * q, 16);
          dst[q] = x;
        }
      }
    } else {  // part of an octet: this range's slots
      for (int i = tid; i < (p_end - p0) * D; i += Cfg::kThreads) {
        const int q = i / D, d = i % D, p = p0 + q;
        means[((size_t)(p / 8) * D + d) * 8 + p % 8] = q < nfam ? pmean[q * D + d] : T(0.f);
      }
    }
    for (int q = tid; q < p_end - p0; q += Cfg::kThreads) {
      const int p = p0 + q;
      const float n = q < nfam ? L.cell[q] : 0.f;
      info[(size_t)(p / 8) * 16 + p % 8] = n;
      info[(size_t)(p / 8) * 16 + 8 + p % 8] = ln_n(n);
    }
  }
  if (p0 == 0) {  // the empty octet
    for (int i = tid; i < D * 8; i += Cfg::kThreads) means[(size_t)PL.zero_oct * D * 8 + i] = T(0.f);
    if (tid < 16) info[(size_t)PL.zero_oct * 16 + tid] = tid < 8 ? 0.f : kNegInf;
  }
}

// Families per workgroup: the fewest that let all workgroups run at once
// (slots of them), so that no CU is left with a second, partial round; with
// more families than kMaxFamilies times that, the fewest whole rounds. Fewer
// families per workgroup cost scanning (every workgroup scans all codes of
// its head) and a second round, more leave CUs idle. Precompute in us: 48
// heads of 64 families (N = 1024, d = 64, 1024 slots): 2 families 21.1, 4
// 17.3, 8 18.0, 16 21.9 (4 taken); 32 heads of 256 (N = 16384, d = 128, 256 slots):
// 16 104, 32 96, 64 123 (32 taken); 96 heads of 256 (N = 4096, 1024 slots), keys even
// / on few codes: 26 60.4 / 90.9, 32 57.7 / 113.1 (26 taken). Whole octets of
// parents (a multiple of 8) save the parts of an octet at the end, but over 22
// shapes they were 0.95 to 1.24 of the time, mostly more.
inline int families_per_workgroup(long long BH, int n_fam, long long slots) {
  const long long least = (n_fam + kMaxFamilies - 1) / kMaxFamilies;  // ranges per head
  const long long rounds = std::max(1LL, (least * BH + slots - 1) / slots);
  const long long ranges = rounds * slots / BH;  // at least `least`
  return (int)((n_fam + ranges - 1) / ranges);
}

template <typename T, int D, int NT, int MODE, bool SMALL>
hipError_t launch_aggregate_cfg(int BH, int N, int M0, int Ch, const void* V,
                                const int32_t* code_idx, float* Vbar, int32_t* counts,
                                void* packed, const FusedArgs& fa, hipStream_t stream) {
  using Cfg = AggCfg<T, D, NT, MODE, SMALL>;
  DeviceInfo dev;
  hipError_t e = device_info(&dev);
  if (e != hipSuccess) return e;
  const long long cus = dev.cus > 1 ? dev.cus : 1;
  const int rsh = Cfg::kFlat ? flat_shift(BH, N, M0, cus * std::min(Cfg::kPerCU, 2)) : 4;
  if constexpr (MODE == kAggFlat) {
    if (rsh < 4)
      return launch_aggregate_cfg<T, D, NT, kAggFlatFew, SMALL>(BH, N, M0, Ch, V, code_idx, Vbar,
                                                                counts, packed, fa, stream);
  }
  const int n_fam = Cfg::kFlat ? flat_families(M0, rsh) : M0;
  const int F = families_per_workgroup(BH, n_fam, cus * Cfg::kPerCU);
  const int ranges = (n_fam + F - 1) / F;
  const long long grid = (long long)BH * ranges;
  if (grid > 0x7fffffff) return hipErrorInvalidConfiguration;
  // the key list takes the rest of the LDS that one workgroup may use, and
  // no more than the head's keys with every family's last group padded
  const int room = (std::min(dev.lds_max, Cfg::kLds) - Cfg::off_list(F)) / (4 * kGroup) * kGroup;
  const long long most = ((long long)N + (long long)F * kGroup + kGroup - 1) / kGroup * kGroup;
  const int cap = (int)std::min<long long>(room, most);
  if (cap < F * kGroup) return hipErrorInvalidConfiguration;
  const int lds = Cfg::off_list(F) + 4 * cap;
  constexpr int slot = 64 + ((((Elem<T>::kBf16 ? 0 : 1) * 2 + (D == 128 ? 1 : 0)) * 2 + (NT - 1)) * 4 + MODE) +
                       (SMALL ? 64 : 0);
  e = ensure_dynamic_lds((const void*)aggregate_kernel<T, D, NT, MODE, SMALL>, lds, slot);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((aggregate_kernel<T, D, NT, MODE, SMALL>), dim3((unsigned)grid),
                     dim3(Cfg::kThreads), lds, stream, static_cast<const T*>(V), code_idx, Vbar,
                     counts, static_cast<unsigned char*>(packed), N, M0, Ch, F, ranges, cap, rsh, fa);
  return hipGetLastError();
}

// Ch <= 8 with few keys per head: SMALL. Their rows stream for a few us only,
// so a workgroup's chain of phases sets the time unless several workgroups
// per CU overlap theirs; with more keys the scan of all codes by more
// workgroups costs what that gains. bf16 at d = 64 (4 workgroups per CU) below
// 16384 keys. Precompute, SMALL / one 16-wave workgroup per CU, us: 96 heads x
// 256 families, N = 4096: 57.7 / 71.9; 48 x 256, N = 2048: 29.0 / 36.4; 48 x 64,
// N = 16384: 63.7 / 64.9; 16 x 256, N = 16384: 39.2 / 38.2; 4 x 128, N = 65536:
// 47.7 / 39.0. The others (2 per CU) below 1024. Aggregation, SMALL / one per
// CU, us: bf16, d = 128, 300 heads x 100 families, N = 512: 46.6 / 66.2; 48 x 64,
// N = 1024: 0.99 to 1.10 of one per CU's time; 16 x 256, N = 16384: 1.13; 64 x
// 128, N = 4096 (precompute): 52.4 / 52.7; fp32, d = 64, 1000 x 16, N = 130: 0.57;
// 300 x 100, N = 512: 38.0 / 65.5. (fp32 flat codebooks of
// 8192 keys gain 3 to 10%, but lose up to 1.9 times where one family holds most of
// the keys: 4 waves' fp32 products.)
template <typename T, int D>
constexpr int kSmallKeys = Elem<T>::kBf16 && D == 64 ? 16384 : 1024;

// Beyond that limit, up to 2048 keys, SMALL too where one workgroup per CU takes
// more than one round (the chain of phases once per round): aggregation with sums,
// SMALL / one per CU: 300 heads x 64 families, N = 2000, fp32, d = 64 0.89, d = 128
// 0.95; 214 x 256, N = 1040, Ch = 8, fp32 0.90 and 0.92, bf16, d = 128 0.97 (the fused
// pass 0.88); 96 x 512, N = 1500 0.92 to 1.02; but 96 x 256, N = 4096, skewed keys up
// to 1.19. And not for an fp32 flat codebook at d = 128 of fewer families of 16
// parents than CUs and more than 512 keys, where one skewed family is 4 waves'
// products: 26 x 64 parents, N = 872, skewed 1.21, even 1.06; 48 x 64, N = 800
// 1.19, 1.11; 64 x 32, N = 1000 1.20, 0.88; against 96 x 512, N = 700 0.99, 0.85.
template <typename T, int D, int MODE>
constexpr bool small_workgroups(long long BH, int N, int M0, long long cus) {
  constexpr bool kFlat = MODE == kAggFlat || MODE == kAggFlatFew;
  const int n_fam = kFlat ? flat_families(M0, 4) : M0;
  if (kFlat && !Elem<T>::kBf16 && D == 128 && N > 512 && BH * n_fam <= cus) return false;
  if (N < kSmallKeys<T, D>) return true;
  return N < 2048 && BH * ((n_fam + kMaxFamilies - 1) / kMaxFamilies) > cus;
}

template <typename T, int D, int NT, int MODE>
hipError_t launch_aggregate_nt(int BH, int N, int M0, int Ch, const void* V,
                               const int32_t* code_idx, float* Vbar, int32_t* counts,
                               void* packed, const FusedArgs& fa, hipStream_t stream) {
  if constexpr (NT == 1) {
    DeviceInfo dev;
    const hipError_t e = device_info(&dev);
    if (e != hipSuccess) return e;
    if (small_workgroups<T, D, MODE>(BH, N, M0, dev.cus > 1 ? dev.cus : 1))
      return launch_aggregate_cfg<T, D, NT, MODE, true>(BH, N, M0, Ch, V, code_idx, Vbar, counts,
                                                        packed, fa, stream);
  }
  return launch_aggregate_cfg<T, D, NT, MODE, false>(BH, N, M0, Ch, V, code_idx, Vbar, counts,
                                                     packed, fa, stream);
}

template <typename T, int D>
hipError_t launch_aggregate_d(int BH, int N, int M0, int Ch, const void* V,
                              const int32_t* code_idx, float* Vbar, int32_t* counts,
                              void* packed, hipStream_t stream) {
  const FusedArgs none{};
  if (Ch == 0)
    return launch_aggregate_nt<T, D, 1, kAggFlat>(BH, N, M0, Ch, V, code_idx, Vbar, counts,
                                                   packed, none, stream);
  if (Ch <= 8)
    return launch_aggregate_nt<T, D, 1, kAggCodes>(BH, N, M0, Ch, V, code_idx, Vbar, counts,
                                                    packed, none, stream);
  if (Ch <= 16)
    return launch_aggregate_nt<T, D, 2, kAggCodes>(BH, N, M0, Ch, V, code_idx, Vbar, counts,
                                                    packed, none, stream);
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_aggregate(int BH, int N, int d, int M0, int Ch, const void* V,
                            const int32_t* code_idx, float* Vbar, int32_t* counts, void* packed,
                            hipStream_t stream) {
  if (d == 64)
    return launch_aggregate_d<T, 64>(BH, N, M0, Ch, V, code_idx, Vbar, counts, packed, stream);
  if (d == 128)
    return launch_aggregate_d<T, 128>(BH, N, M0, Ch, V, code_idx, Vbar, counts, packed, stream);
  return hipErrorInvalidValue;
}

// Alg. 1 in two launches: the parent assignment (it reads K once and writes
// parent_idx), then the fused child compare + aggregation. Ch = 0 (the parent
// is the code) and fp32 with Ch = 16 at d = 128 (the candidate rows, the sums
// and the key and value rows of a group pass the 256 registers of a lane)
// take the assignment and then the plain aggregation.
template <typename T, int D>
hipError_t launch_assign_aggregate_d(int BH, int H, int N, int M0, int Ch, const void* K,
                                     const void* V, const void* Cp, const void* Cc,
                                     int32_t* parent_idx, int32_t* code_idx, float* Vbar,
                                     int32_t* counts, void* packed, hipStream_t stream) {
  constexpr bool kWide = Elem<T>::kBf16 || D == 64;  // Ch = 16 fused
  const bool fused = Ch >= 1 && (Ch <= 8 || kWide);
  hipError_t e = launch_assign<T, D>(BH, H, N, M0, Ch, K, Cp, Cc, parent_idx, code_idx, !fused, stream);
  if (e != hipSuccess) return e;
  if (!fused)
    return launch_aggregate_d<T, D>(BH, N, M0, Ch, V, code_idx, Vbar, counts, packed, stream);
  const FusedArgs fa{K, Cp, Cc, code_idx, H};
  if (Ch <= 8)
    return launch_aggregate_nt<T, D, 1, kAggFused>(BH, N, M0, Ch, V, parent_idx, Vbar, counts,
                                                    packed, fa, stream);
  if constexpr (kWide)
    return launch_aggregate_nt<T, D, 2, kAggFused>(BH, N, M0, Ch, V, parent_idx, Vbar, counts,
                                                    packed, fa, stream);
  return hipErrorInvalidValue;  // not reached
}

template <typename T>
hipError_t launch_assign_aggregate(int BH, int H, int N, int d, int M0, int Ch, const void* K,
                                   const void* V, const void* Cp, const void* Cc,
                                   int32_t* parent_idx, int32_t* code_idx, float* Vbar,
                                   int32_t* counts, void* packed, hipStream_t stream) {
  if (d == 64)
    return launch_assign_aggregate_d<T, 64>(BH, H, N, M0, Ch, K, V, Cp, Cc, parent_idx, code_idx,
                                            Vbar, counts, packed, stream);
  if (d == 128)
    return launch_assign_aggregate_d<T, 128>(BH, H, N, M0, Ch, K, V, Cp, Cc, parent_idx, code_idx,
                                             Vbar, counts, packed, stream);
  return hipErrorInvalidValue;
}

template hipError_t launch_aggregate<bf16>(int, int, int, int, int, const void*, const int32_t*,
                                           float*, int32_t*, void*, hipStream_t);
template hipError_t launch_aggregate<float>(int, int, int, int, int, const void*, const int32_t*,
                                            float*, int32_t*, void*, hipStream_t);
template hipError_t launch_assign_aggregate<bf16>(int, int, int, int, int, int, const void*,
                                                  const void*, const void*, const void*,
                                                  int32_t*, int32_t*, float*, int32_t*, void*,
                                                  hipStream_t);
template hipError_t launch_assign_aggregate<float>(int, int, int, int, int, int, const void*,
                                                   const void*, const void*, const void*,
                                                   int32_t*, int32_t*, float*, int32_t*, void*,
                                                   hipStream_t);

}  // namespace avq
