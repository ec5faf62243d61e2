// fp32 path of the grouped Fisher Gram, H[k] (+)= X^T Diag(s[:,k]) X on upper-triangle
// tiles (GuidedQuant, Algorithm 1, line 4).
//
// The products run on the bf16 matrix cores at fp32 accuracy: both fp32 operands, s * x (one fp32 rounding)
// and x, are split into three bf16 terms (24 mantissa bits, exact), and of the nine term products the six
// that matter are summed in fp32 (hi*hi, hi*mid, mid*hi, hi*lo, lo*hi, mid*mid; the others are below 2^-24
// of the product).  A step of 16 tokens of a 32 x 32 block is six bf16 instructions of 32 cycles instead of
// eight fp32 ones of 64: 2.7 times fewer matrix-core cycles.  Accumulators are flushed into a second-level
// sum every 2048 tokens to keep fp32 accumulation error well below the 1e-5 parity bar at large n.
//
// The split does not carry infinities (inf - inf) and overflows at the top of the range, so every kernel
// watches the largest operand it has split; where that is beyond kSplitMax the tile is computed again by the
// fp32 matrix instruction (v_mfma_f32_32x32x2_f32), which also sees NaN and infinity as fp32 arithmetic does.
//
// Two kernels share this arithmetic:
//   fisher_gram_f32_tile_kernel   256 x 128 tile per workgroup, operands split once and shared through LDS
//   fisher_gram_f32_block_kernel  32 x 32 tile per workgroup, the tokens dealt out to its 16 waves
#include <utility>

#include "gq_internal.hpp"

namespace gq {
namespace {

// f(0), f(1), ..., f(N - 1) with compile-time arguments
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

constexpr int kTile = 128;          // output tile edge
constexpr int kStep = 16;           // tokens per LDS stage
constexpr int kPitch = kTile + 32;  // floats; +32 keeps the two token rows of one MFMA read on disjoint banks
constexpr int kFlush = 2048 / kStep;
constexpr float kSplitMax = 3.0e38f;    // operands up to here split into finite bf16 terms

// Two fp32 values as three dwords of bf16 pairs (round to nearest even each): x = hi + mid + lo.
__device__ inline void split3_pair(float x0, float x1, unsigned& hi, unsigned& mid, unsigned& lo) {
  f32x2 v = {x0, x1};
  hi = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
  v[0] = x0 - __builtin_bit_cast(float, hi << 16);
  v[1] = x1 - __builtin_bit_cast(float, hi & 0xffff0000u);
  mid = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
  v[0] -= __builtin_bit_cast(float, mid << 16);
  v[1] -= __builtin_bit_cast(float, mid & 0xffff0000u);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
// the six term products (row term, column term), smallest first
__device__ constexpr int kProdA[6] = {0, 2, 1, 0, 1, 0}, kProdB[6] = {2, 0, 1, 1, 0, 0};

__device__ inline f32x4 load_row4(const float* __restrict__ X, int64_t ld, int64_t n, int64_t d, int64_t i,
                                  int64_t c) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (i < n) {
    const float* p = X + i * ld + c;
    if (c + 4 <= d) {
      v = *reinterpret_cast<const f32x4*>(p);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < d) v[e] = p[e];
    }
  }
  return v;
}

// The 128 x 128 tile at (a0, b0) by the fp32 matrix instruction: acc + tot is the result.  The operands are
// staged through LDS exactly as they lie in memory ([token][column]), the row operand times s[token, k].
__device__ __forceinline__ void tile_in_fp32(char* smem, const float* __restrict__ X, int64_t n, int64_t d, int64_t ld,
                                          const float* __restrict__ s, int G, int k, int64_t a0, int64_t b0,
                                          f32x16 (&acc)[2][2], f32x16 (&tot)[2][2]) {
  float (*As)[kStep][kPitch] = reinterpret_cast<float (*)[kStep][kPitch]>(smem);
  float (*Bs)[kStep][kPitch] = reinterpret_cast<float (*)[kStep][kPitch]>(smem + 2 * kStep * kPitch * 4);
  const int tid = threadIdx.x;
  const int lane = tid % kWave, wave = tid / kWave;
  const int wm = wave / 2, wn = wave % 2;  // wave's 64x64 quadrant

  // staging assignment: 16 rows x 32 float4 per operand = 512 float4, two per thread
  const int lrow = tid / 32;        // 0..7 (and +8)
  const int lcol = (tid % 32) * 4;  // column inside the tile

#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc[x][y][r] = 0.f; tot[x][y][r] = 0.f; }

  const int64_t steps = (n + kStep - 1) / kStep;
  f32x4 ra[2], rb[2];
  float rs[2];
  auto fetch = [&](int64_t step) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t i = step * kStep + lrow + 8 * h;
      ra[h] = load_row4(X, ld, n, d, i, a0 + lcol);
      rb[h] = load_row4(X, ld, n, d, i, b0 + lcol);
      rs[h] = (i < n) ? s[i * G + k] : 0.f;
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f32x4 sa = {ra[h][0] * rs[h], ra[h][1] * rs[h], ra[h][2] * rs[h], ra[h][3] * rs[h]};
      *reinterpret_cast<f32x4*>(&As[buf][lrow + 8 * h][lcol]) = sa;
      *reinterpret_cast<f32x4*>(&Bs[buf][lrow + 8 * h][lcol]) = rb[h];
    }
  };

  fetch(0);
  stash(0);
  __syncthreads();
  for (int64_t step = 0; step < steps; ++step) {
    const int buf = (int)(step & 1);
    if (step + 1 < steps) fetch(step + 1);
#pragma unroll
    for (int kk = 0; kk < kStep; kk += 2) {
      float av[2], bv[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) av[x] = As[buf][kk + lane / 32][wm * 64 + x * 32 + lane % 32];
#pragma unroll
      for (int y = 0; y < 2; ++y) bv[y] = Bs[buf][kk + lane / 32][wn * 64 + y * 32 + lane % 32];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[x], bv[y], acc[x][y], 0, 0, 0);
    }
    if ((step + 1) % kFlush == 0) {
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          tot[x][y] += acc[x][y];
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
        }
    }
    if (step + 1 < steps) stash(buf ^ 1);
    __syncthreads();
  }
}

// One 32 x 32 block of accumulators into H: register r of lane l holds row 8*(r/4)+4*(l/32)+(r%4), column l%32.
// The old values are read together, from addresses clamped into the upper triangle; only the stores are masked.
__device__ __forceinline__ void store_block(float* __restrict__ Hk, int64_t d, int64_t row0, int64_t col,
                                            const float (&v)[16], int accumulate) {
  float old[16];
  if (accumulate) {
    const int64_t cc = col < d ? col : d - 1;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t row = row0 + 8 * (r / 4) + (r % 4);
      old[r] = Hk[(row < cc ? row : cc) * d + cc];
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) old[r] = 0.f;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t row = row0 + 8 * (r / 4) + (r % 4);
    if (col < d && row <= col) Hk[row * d + col] = accumulate ? v[r] + old[r] : v[r];
  }
}

// One workgroup (4 waves, 2x2, one per SIMD) owns a 256 x 128 output tile of one group, every wave 128 x 64 of it,
// and walks over the tokens in stages of 16.  Staging transposes: a wave takes one octet of the stage's tokens and
// 128 row columns (a lane two neighbouring ones: eight 8-byte loads) and 64 column columns (eight 4-byte loads);
// the lane splits its 24 values pair by pair along the tokens, so that the eight tokens of a column and term are
// 16 bytes in the order the matrix instruction wants, and stores them as
//   stage buffer [row operand: term][octet][column ^ ((column >> 4) & 1)], [column operand: term][octet][column]
// (the XOR keeps the stores of every second column as free of bank conflicts as the fragment reads of 32
// consecutive ones).  Every value is split once per workgroup instead of once per wave that uses it: 3.4 vector
// instructions per matrix instruction, 0.375 LDS reads.
// Pipeline: the values of a stage are requested four stages ahead into two sets of registers that alternate, split
// and stored two stages ahead into a ring of three buffers, and its fragments replace those of the stage before in
// the same registers, each behind the last product that needs the old one.  One barrier per stage.
// Bound by the issue of one wave per SIMD (vector instructions, LDS accesses and loads share it with the matrix
// instructions) at the clock the chip holds: 1.1 us per stage of 48 matrix instructions.  Measured against the fp32
// matrix instruction on 128 x 128 tiles: X[12001,2501], G = 4 4.60 -> 1.88 ms; X[16384,4096], G = 4 12.1 -> 7.1 ms
// (155 TFLOP/s, 0.93 PFLOP/s of bf16 products).  128 x 128 tiles with two workgroups per compute unit: 2.09 and 7.0.
constexpr int kBufferWord3 = 0x00020000;             // raw buffer, 32-bit elements
constexpr int kRowsT = 2 * kTile;                    // rows of the output tile (256); kTile columns
constexpr int kTermA = 2 * kRowsT * 16;              // bytes of one term of the row operand (two octets): 8 KiB
constexpr int kTermB = 2 * kTile * 16;               // of the column operand: 4 KiB
constexpr int kBufBytes = 3 * (kTermA + kTermB);     // 36 KiB
constexpr int kBuffers = 3;
static_assert(kFlush % 2 == 0, "stages go in pairs");
static_assert(kBuffers * kBufBytes >= 4 * kStep * kPitch * 4, "the fp32 loop's staging fits");
__global__ __launch_bounds__(256, 1) void fisher_gram_f32_tile_kernel(const float* __restrict__ X, int64_t n, int64_t d,
                                                                      int64_t ld, const float* __restrict__ s, int G,
                                                                      float* __restrict__ H, int accumulate) {
  __shared__ __attribute__((aligned(16))) char smem[kBuffers * kBufBytes];

  // The groups of a tile read the same columns of X and neighbouring tiles share panels: workgroup ids are
  // dealt round-robin to the 8 XCDs, so every XCD gets one contiguous eighth of the (tile, group) list.
  // Tile column J holds the row blocks 0 .. J / 2 (row block I meets it on or above the diagonal iff 2 I <= J).
  int k, I, J;
  {
    const int64_t total = gridDim.x, id = blockIdx.x;
    const int64_t x = id % 8, idx = id / 8, q = total / 8, r = total % 8;
    const int64_t w = x * q + (x < r ? x : r) + idx;
    k = (int)(w % G);
    int i, j;
    const int64_t t = w / G;                         // pairs of tile columns 2 j, 2 j + 1 hold 2 (j + 1) tiles
    tri_decode(t / 2, i, j);
    const int64_t off = t - (int64_t)j * (j + 1);    // 0 .. 2 j + 1
    I = (int)(off / 2);
    J = 2 * j + (int)(off % 2);
    k = __builtin_amdgcn_readfirstlane(k);           // uniform anyway; now the compiler knows (tri_decode is vector code)
    I = __builtin_amdgcn_readfirstlane(I);
    J = __builtin_amdgcn_readfirstlane(J);
  }
  const int64_t a0 = (int64_t)I * kRowsT, b0 = (int64_t)J * kTile;
  if (b0 >= d) return;                               // the whole workgroup: the last pair may have one tile column only

  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wm = wave / 2, wn = wave % 2;            // the wave's 128 x 64 part of the tile

  // staging: tokens 8 oct .. 8 oct + 7 of a stage, columns 128 part + 2 lane and + 1 of the rows' 256,
  // column 64 part + lane of the columns' 128
  const int part = wave / 2, oct = wave % 2;
  const int64_t ca_in = a0 + 128 * part + 2 * lane, cb_in = b0 + 64 * part + lane;
  const int64_t ca = ca_in < d ? ca_in : (d - 1) / 2 * 2;    // past the matrix: any column inside (ld is a multiple of 4)
  const int64_t cb = cb_in < d ? cb_in : d - 1;
  const unsigned vo_a = (unsigned)(ca * 4), vo_b = (unsigned)(cb * 4);   // bytes; d < 2^29
  const bool second_in = ca + 1 < d;
  unsigned wpos[3];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int col = 128 * part + 2 * lane + e;
    wpos[e] = (unsigned)(oct * (kRowsT * 16) + (col ^ ((col >> 4) & 1)) * 16);
  }
  wpos[2] = (unsigned)(3 * kTermA + oct * (kTile * 16) + (64 * part + lane) * 16);
  const int64_t steps = (n + kStep - 1) / kStep;
  // All loads are buffer loads: the base of a stage and the token's distance from it are scalar, the lane adds its
  // column.  (The weights are the same for all lanes, but vector loads: scalar ones return in any order.)
  const unsigned row_bytes = (unsigned)(ld * 4), w_bytes = (unsigned)G * 4u;   // 7 * ld * 4 < 2^32 (the launcher sees to it)
  struct Raw {
    f32x2 a[8];
    float b[8], sv[8];
    int in;                                                  // tokens of the octet that exist
  };
  Raw set0, set1;
  __amdgpu_buffer_rsrc_t xr, wr;
  int in_next = 0;
  // fetch_from(step), then fetch_a, fetch_w and fetch_b: the values of a stage; past the last stage that one again, all of
  // it with weight 0
  auto fetch_from = [&](int64_t step) {
    const int64_t i0 = (step < steps ? step : steps - 1) * kStep + 8 * oct;
    const int64_t ib = i0 < n ? i0 : n - 1;                  // tokens past the end: an earlier one, with weight 0 (zero_past)
    in_next = step < steps ? (int)(n - i0 < 8 ? n - i0 : 8) : 0;
    xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(X + ib * ld), 0, -1, kBufferWord3);
    wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(s + ib * G + k), 0, -1, kBufferWord3);
  };
  auto fetch_a = [&](Raw& f, int t) {                        // row columns of token t
    const unsigned tt = t < in_next ? (unsigned)t : 0u;
    f.a[t] = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(xr, vo_a, tt * row_bytes, 0));
  };
  auto fetch_w = [&](Raw& f, int t) {
    const unsigned tt = t < in_next ? (unsigned)t : 0u;
    f.sv[t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wr, 0, tt * w_bytes, 0));
  };
  auto fetch_b = [&](Raw& f, int t) {
    const unsigned tt = t < in_next ? (unsigned)t : 0u;
    f.b[t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, vo_b, tt * row_bytes, 0));
    if (t == 7) f.in = in_next;
  };
  auto zero_past = [&](Raw& f) {
    if (f.in < 8) {                                          // uniform, from the last stage on
#pragma unroll
      for (int t = 0; t < 8; ++t)
        if (t >= f.in) {
          f.sv[t] = 0.f;
          f.b[t] = 0.f;
        }
    }
  };
  float most[3] = {0.f, 0.f, 0.f};                           // largest magnitude split, per column of the lane
  u32x4 term[3];
  // The splitting of a stage in 44 parts of three or four vector instructions each, one behind every matrix
  // instruction: the wave issues in order, so a longer stretch between two matrix instructions would leave the
  // matrix core idle.  Parts 4 p .. 4 p + 3 (p < 8) split tokens 2 (p % 4) and + 1 of the lane's row column p / 4,
  // parts 32 + 3 p .. + 2 tokens 2 p and + 1 of its column column.  (The empty asm statements keep each part where
  // it is written.)
  float v0 = 0.f, v1 = 0.f, w0 = 0.f, w1 = 0.f;
  auto upper = [](unsigned u) { return __builtin_bit_cast(float, u & 0xffff0000u); };
  auto lower = [](unsigned u) { return __builtin_bit_cast(float, u << 16); };
  auto pack = [&]() {
    const f32x2 v = {v0, v1};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
  };
  auto split_part = [&](const Raw& f, int g) {
    const bool rows = g < 32;
    const int p = rows ? g / 4 : (g - 32) / 3, q = rows ? g % 4 : (g - 32) % 3;
    const int e = rows ? p / 4 : 2, t = 2 * (p % 4);
    if (q == 0) {
      v0 = rows ? f.a[t][e % 2] * f.sv[t] : f.b[t];
      v1 = rows ? f.a[t + 1][e % 2] * f.sv[t + 1] : f.b[t + 1];
      most[e] = fmaxf(fmaxf(most[e], fabsf(v0)), fabsf(v1));
      term[0][t / 2] = pack();
      asm volatile("" : "+v"(v0), "+v"(v1), "+v"(most[e]));
      if (!rows) {
        w0 = lower(term[0][t / 2]);
        w1 = upper(term[0][t / 2]);
        asm volatile("" : "+v"(w0), "+v"(w1));
      }
    } else if (rows && q == 1) {
      v0 -= lower(term[0][t / 2]);
      v1 -= upper(term[0][t / 2]);
      asm volatile("" : "+v"(v0), "+v"(v1));
    } else if (rows && q == 2) {
      term[1][t / 2] = pack();
      w0 = lower(term[1][t / 2]);
      w1 = upper(term[1][t / 2]);
      asm volatile("" : "+v"(w0), "+v"(w1));
    } else if (!rows && q == 1) {
      v0 -= w0;
      v1 -= w1;
      term[1][t / 2] = pack();
      w0 = lower(term[1][t / 2]);
      asm volatile("" : "+v"(v0), "+v"(v1), "+v"(w0));
    } else {
      v0 -= w0;
      v1 -= rows ? w1 : upper(term[1][t / 2]);
      unsigned lo = pack();
      asm volatile("" : "+v"(lo));
      term[2][t / 2] = lo;
    }
  };
  auto store_term = [&](int e, int u, unsigned buf) {
    *reinterpret_cast<u32x4*>(&smem[buf + u * (e < 2 ? kTermA : kTermB) + wpos[e]]) = term[u];
  };

  // fragments: column l % 32 of a 32-column block, octet l / 32
  const int lcol = lane % 32;
  const unsigned fpos_a = (unsigned)((lane / 32) * (kRowsT * 16) + (wm * 128 + (lcol ^ ((lcol >> 4) & 1))) * 16);
  const unsigned fpos_b = (unsigned)(3 * kTermA + (lane / 32) * (kTile * 16) + (wn * 64 + lcol) * 16);
  bf16x8 fa[4][3], fb[2][3];
  auto read_a = [&](unsigned buf, int u, int x) {
    fa[x][u] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(&smem[buf + fpos_a + u * kTermA + x * 512]));
  };
  auto read_b = [&](unsigned buf, int u, int y) {
    fb[y][u] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(&smem[buf + fpos_b + u * kTermB + y * 512]));
  };

  f32x16 acc[4][2], tot[4][2];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc[x][y][r] = 0.f; tot[x][y][r] = 0.f; }

  auto fetch_all = [&](Raw& f, int64_t step) {
    fetch_from(step);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      fetch_a(f, t);
      fetch_w(f, t);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) fetch_b(f, t);
  };
  auto split_all = [&](Raw& f, unsigned buf) {
    zero_past(f);
    static_for<44>([&](auto g_c) {
      constexpr int g = g_c;
      split_part(f, g);
      if (g == 15 || g == 31 || g == 43) {
#pragma unroll
        for (int u = 0; u < 3; ++u) store_term(g / 16, u, buf);
      }
    });
  };
  fetch_all(set0, 0);
  fetch_all(set1, 1);
  split_all(set0, 0);
  fetch_all(set0, 2);
  split_all(set1, kBufBytes);
  fetch_all(set1, 3);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 3; ++u) {
#pragma unroll
    for (int x = 0; x < 4; ++x) read_a(0, u, x);
#pragma unroll
    for (int y = 0; y < 2; ++y) read_b(0, u, y);
  }
  unsigned nxt = kBufBytes, fill = 2 * kBufBytes;            // buffers of the next stage and of the one after it
  // One stage: multiplies the fragments in registers; splits the values in `f` (two stages ahead) into buffer
  // `fill` and requests the ones four stages ahead into `f`; reads the next stage's fragments.
  auto stage = [&](Raw& f, int64_t step) {
    // (row term, column term) of the six products: mid*mid first, whose operands were read first
    constexpr int kTa[6] = {1, 0, 2, 0, 1, 0}, kTb[6] = {1, 2, 0, 1, 0, 0};
    zero_past(f);
    fetch_from(step + 4);
    __builtin_amdgcn_sched_barrier(0);
    static_for<48>([&](auto i_c) {
      constexpr int i = i_c;
      const int pr = i / 8, x = (i / 2) % 4, y = i % 2;
      acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[x][kTa[pr]], fb[y][kTb[pr]], acc[x][y], 0, 0, 0);
      // (a term is stored before the next column's first parts overwrite it)
      if (i >= 16 && i < 19) store_term(0, i - 16, fill);
      if (i >= 32 && i < 35) store_term(1, i - 32, fill);
      if (i >= 44 && i < 47) store_term(2, i - 44, fill);
      if (i < 44) split_part(f, i);
      if (i >= 18 && i < 34) {                               // tokens whose values have just been used
        const int t = 2 * ((i - 18) / 4) + i % 2;
        if ((i - 18) % 4 < 2) fetch_a(f, t);
        else fetch_w(f, t);
      }
      if (i >= 34 && i < 46 && (i - 34) % 3 < 2) fetch_b(f, 2 * ((i - 34) / 3) + (i - 34) % 3);
      if (i == 16 || i == 17) read_b(nxt, 2, i - 16);
      if (i >= 24 && i < 28) read_a(nxt, 2, i - 24);
      if (i == 35 || i == 36) read_b(nxt, 1, i - 35);
      if (i >= 40 && i < 44) read_a(nxt, 1, i - 40);
      if (i == 44) read_a(nxt, 0, 0);
      if (i == 45) read_a(nxt, 0, 1);
      if (i == 46) read_a(nxt, 0, 2);
      if (i == 47) {
        read_a(nxt, 0, 3);
        read_b(nxt, 0, 0);
        read_b(nxt, 0, 1);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    const unsigned done = nxt == 0 ? 2 * kBufBytes : nxt - kBufBytes;   // this stage's buffer
    nxt = fill;
    fill = done;
    // LDS operations of a wave finish in order: with at most the four reads issued after its last store still
    // under way, everything this wave has stored is there.
    asm volatile("s_waitcnt lgkmcnt(4)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  for (int64_t step0 = 0; step0 < steps; step0 += kFlush) {
    const int64_t end = step0 + kFlush < steps ? step0 + kFlush : steps;
    for (int64_t step = step0; step < end; step += 2) {      // (an odd number of stages: one more, of zeros)
      stage(set0, step);
      stage(set1, step + 1);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        tot[x][y] += acc[x][y];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
      }
  }
  __syncthreads();
  float* Hk = H + (int64_t)k * d * d;
  const bool beyond = most[0] > kSplitMax || (second_in && most[1] > kSplitMax) || most[2] > kSplitMax;
  if (__syncthreads_or(beyond)) {                            // the whole tile again, in fp32, half by half
    for (int h = 0; h < 2; ++h) {
      f32x16 a2[2][2], t2[2][2];
      tile_in_fp32(smem, X, n, d, ld, s, G, k, a0 + h * kTile, b0, a2, t2);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          float v[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) v[r] = t2[x][y][r] + a2[x][y][r];
          store_block(Hk, d, a0 + h * kTile + wm * 64 + x * 32 + 4 * (lane / 32), b0 + wn * 64 + y * 32 + lane % 32, v,
                      accumulate);
        }
    }
    return;
  }
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = tot[x][y][r];
      store_block(Hk, d, a0 + wm * 128 + x * 32 + 4 * (lane / 32), b0 + wn * 64 + y * 32 + lane % 32, v, accumulate);
    }
}

// Problems with too few large tiles for the chip: one 32 x 32 tile of one group per workgroup, its 16 waves take
// the tokens in turn, 16 at a time.  A wave loads its operands straight into the fragment layout (lane -> column l % 32, tokens 8 (l / 32)
// .. + 7: eight 4-byte loads per operand, a 128-byte line per token row), splits them in registers and needs no
// LDS and no barrier until the end, when the 16 partial tiles are added in wave order through LDS.
// Large tiles from this many on.  Measured (us, this kernel / the tile kernel; n, d, G): 24 tiles 130 / 304
// (4096, 512, 4), 72 tiles 717 / 602 (8192, 2048, 1), 80 tiles 372 / 308 (4096, 1024, 4), 84 tiles 220 / 161
// (2048, 1536, 2); by its time per tile the lines cross at about 64.
constexpr int64_t kLargeTiles = 64;
constexpr int kSmallTile = 32, kSmallWaves = 16;
__global__ __launch_bounds__(kSmallWaves * kWave) void fisher_gram_f32_block_kernel(
    const float* __restrict__ X, int64_t n, int64_t d, int64_t ld, const float* __restrict__ s, int G,
    float* __restrict__ H, int accumulate) {
  __shared__ float part[kSmallWaves][kSmallTile * kSmallTile];
  int ti, tj;
  tri_decode((int64_t)(blockIdx.x / (unsigned)G), ti, tj);
  const int k = (int)(blockIdx.x % (unsigned)G);
  const int64_t a0 = (int64_t)ti * kSmallTile, b0 = (int64_t)tj * kSmallTile;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int oct = lane / 32;
  const int64_t ca = a0 + lane % 32 < d ? a0 + lane % 32 : d - 1, cb = b0 + lane % 32 < d ? b0 + lane % 32 : d - 1;
  const int64_t steps = (n + kStep - 1) / kStep;

  f32x16 acc, tot;
#pragma unroll
  for (int r = 0; r < 16; ++r) { acc[r] = 0.f; tot[r] = 0.f; }
  float ra[8], rb[8], rs[8], most = 0.f;
  auto fetch = [&](int64_t step) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int64_t i = step * kStep + 8 * oct + t, ic = i < n ? i : n - 1;
      ra[t] = X[ic * ld + ca];
      rb[t] = X[ic * ld + cb];
      rs[t] = s[ic * G + k];
    }
  };
  int done = 0;
  if (wave < steps) fetch(wave);
  for (int64_t step = wave; step < steps; step += kSmallWaves) {
    u32x4 at[3], bt[3];
    float va[8], vb[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const bool in = step * kStep + 8 * oct + t < n;
      va[t] = in ? ra[t] * rs[t] : 0.f;
      vb[t] = in ? rb[t] : 0.f;
    }
    if (step + kSmallWaves < steps) fetch(step + kSmallWaves);
#pragma unroll
    for (int t = 0; t < 8; t += 2) {
      most = fmaxf(fmaxf(most, fabsf(va[t])), fabsf(va[t + 1]));
      most = fmaxf(fmaxf(most, fabsf(vb[t])), fabsf(vb[t + 1]));
      unsigned h, m, l;
      split3_pair(va[t], va[t + 1], h, m, l);
      at[0][t / 2] = h;
      at[1][t / 2] = m;
      at[2][t / 2] = l;
      split3_pair(vb[t], vb[t + 1], h, m, l);
      bt[0][t / 2] = h;
      bt[1][t / 2] = m;
      bt[2][t / 2] = l;
    }
#pragma unroll
    for (int pr = 0; pr < 6; ++pr)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, at[kProdA[pr]]),
                                                    __builtin_bit_cast(bf16x8, bt[kProdB[pr]]), acc, 0, 0, 0);
    if (++done % kFlush == 0) {
      tot += acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    }
  }
  if (__any(most > kSplitMax)) {                             // uniform per wave: this wave's tokens again, in fp32
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[r] = 0.f; tot[r] = 0.f; }
    for (int64_t step = wave; step < steps; step += kSmallWaves) {
      for (int t = 0; t < kStep; t += 2) {
        const int64_t i = step * kStep + t + oct, ic = i < n ? i : n - 1;
        const float a = i < n ? X[ic * ld + ca] * s[ic * G + k] : 0.f, b = i < n ? X[ic * ld + cb] : 0.f;
        tot = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, tot, 0, 0, 0);
      }
    }
  }
  // register r of lane l holds row 8*(r/4)+4*(l/32)+(r%4), column l%32
#pragma unroll
  for (int r = 0; r < 16; ++r)
    part[wave][(8 * (r / 4) + 4 * (lane / 32) + (r % 4)) * kSmallTile + lane % 32] = tot[r] + acc[r];
  __syncthreads();
  const int e = threadIdx.x;                                 // one entry of the tile per thread
  const int64_t row = a0 + e / kSmallTile, col = b0 + e % kSmallTile;
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < kSmallWaves; ++w) v += part[w][e];
  if (col < d && row <= col) {
    float* p = H + ((int64_t)k * d + row) * d + col;
    *p = accumulate ? *p + v : v;
  }
}

}  // namespace

hipError_t launch_fisher_gram_f32(const float* X, int64_t n, int64_t d_in, int64_t ld, const float* s, int G,
                                  float* H, bool accumulate, hipStream_t st) {
  // tiles of 256 x 128 as the tile kernel counts them: pairs of tile columns
  const int64_t pairs = (d_in + 2 * kTile - 1) / (2 * kTile), large = pairs * (pairs + 1) * G;
  const int acc = accumulate ? 1 : 0;
  if (large >= kLargeTiles && ld < (int64_t)1 << 27) {
    fisher_gram_f32_tile_kernel<<<dim3((unsigned)large), dim3(256), 0, st>>>(X, n, d_in, ld, s, G, H, acc);
  } else {
    const int64_t T32 = (d_in + kSmallTile - 1) / kSmallTile;
    fisher_gram_f32_block_kernel<<<dim3((unsigned)(tri_count(T32) * G)), dim3(kSmallWaves * kWave), 0, st>>>(X, n, d_in, ld,
                                                                                                         s, G, H, acc);
  }
  return hipGetLastError();
}

}  // namespace gq
