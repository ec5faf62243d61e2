// Closed-form codebook update of LNQ for fixed assignments (Section 4.2, Eq. "conti-sol";
// Algorithm 2, lines 4 and 14), against the group Hessians:
//     c^(j) = (P^T H P + lam I)^-1 P^T H w_j,      P[i][q] = 1 if Q[j][i] == q else 0.
//
// With E_j = P^T (one-hot rows, one per grid point) the two small quantities of a channel are
//     T_j = E_j H            [m, d_in]      (row q: the sum of the rows of H assigned to q)
//     A_j[q][q'] = sum_{i : Q[j][i] == q'} T_j[q][i],      b_j[q] = sum_i T_j[q][i] * w_j[i].
// T for all channels of a group is ONE contraction (d_out/G * m rows) x d_in x d_in on the 8-bit integer
// matrix cores, which run twice the bf16 rate: the one-hot operand is exact in a byte, and every row of H is
// held in fixed point, 30 bits below the power of two above its largest entry, as four signed 8-bit digits:
//     H[i][i'] = 2^(e_i - 30) * (d3 * 2^24 + d2 * 2^16 + d1 * 2^8 + d0).
// The integer sums are exact; what is rounded is H itself, by at most 2^-31 of its row's power of two (an entry
// within a factor 64 of the largest is exact), and T once, to fp32.  (Three bf16 terms, as before: products
// exact, but every addition rounded to fp32; half again as many matrix-core cycles, 6 bytes instead of 4.)
// The one-hot operand never exists in memory: a lane's four code bytes become four operand bytes with ONE byte
// permutation (the codes select from an 8-byte table that holds a 1 at the row's grid point), so only H travels
// from L2 to LDS.  T never exists in memory
// either: a workgroup bins every 256 x 128 tile of it into its share of A and b while the
// tile is still on chip (through LDS; A by one more one-hot product on the bf16 matrix cores, b by
// a plain dot, both in a fixed order) and carries the sums over the column tiles it works
// through; what leaves the kernel is one partial [m][m + 1] system per channel and chunk of
// column tiles.  A second kernel adds the partial
// systems in chunk order and solves the m x m system in fp64 by Gauss-Jordan elimination
// with partial pivoting.
#include "gq_internal.hpp"

namespace gq {
namespace {

constexpr int kRows = 256;                           // rows (channel, grid point) of T per workgroup
constexpr int kCols = 128;                           // columns of T (= rows of H) per workgroup
constexpr int kK = 128;                              // contraction elements per stage (a byte each)
constexpr int kDTile = kCols * kK;                   // one staged digit of H (16 KiB)
constexpr int kHStage = 2 * kDTile;                  // the two digits of a sweep: 32 KiB
constexpr int kMaxCodeRows = 64;                     // rows of codes per workgroup at most (channels x code planes)
constexpr int kQStage = kMaxCodeRows * kK;           // their codes for one stage (8 KiB)
constexpr int kRing = 4;                             // stages: the one in use, the next one (already there), two on their way
constexpr int kLoadsPerStage = 5;                    // per wave: 4 pieces of H, 1 of the codes
constexpr int kBits = 30;                            // fraction bits of H relative to its row's power of two
constexpr int64_t kMaxSweep = 32768;                 // contraction elements whose integer sums fit 32 bits for certain:
                                                     // |d1 * 2^8 + d0| <= 32896 each
constexpr unsigned kPadCode = 12;                    // selects a zero byte in a byte permutation; no grid point has it
constexpr unsigned kNoLevel = 0x7E7E7E7Eu;           // a grid point no code has (rows past the tile's channels)
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

// The codes with the row pitch of the staged operands, one row per plane of eight grid points: Qp[j][p][i] =
// Q[j][i] - 8 p where that is a grid point's place within plane p (0 .. 7), else the pad code; four codes per thread.
__device__ __forceinline__ void pad_codes(int64_t t, const unsigned char* __restrict__ Q, int64_t d, int64_t ldp,
                                          int64_t d_out, int n_levels, int planes, unsigned char* __restrict__ Qp) {
  const int64_t j = 4 * t / ldp, i = 4 * t - j * ldp;        // ldp is a multiple of 128
  if (j >= d_out) return;
  unsigned c[4];
  if (d % 4 == 0 && (reinterpret_cast<uintptr_t>(Q) & 3) == 0) {   // uniform: rows of Q start at multiples of four bytes
    const unsigned w = i < d ? *reinterpret_cast<const unsigned*>(Q + j * d + i) : 0xffffffffu;
#pragma unroll
    for (int e = 0; e < 4; ++e) c[e] = (w >> (8 * e)) & 0xffu;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) c[e] = i + e < d ? Q[j * d + i + e] : 0xffu;
  }
  for (int p = 0; p < planes; ++p) {
    unsigned w = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w |= (c[e] < (unsigned)n_levels && c[e] / 8 == (unsigned)p ? c[e] % 8 : kPadCode) << (8 * e);
    *reinterpret_cast<unsigned*>(Qp + (j * planes + p) * ldp + i) = w;
  }
}

// The largest |H[k][i][i']| of every row i of the full symmetric matrix, from its upper triangle, as float bits, which
// order like the numbers; infinities and NaN come out on top.  Up to kPartTiles tiles per row every 64 x 64 tile writes
// what it found, most_part[k][tile][row], and the splitting kernel puts them together; beyond, they meet in most[k][row]
// by atomic maxima (whose order does not matter), cleared before by the launch that pads the codes.
// The first n_max workgroups do that, a tile on or above the diagonal each; the others pad codes.
constexpr int kPartTiles = 16;
__global__ __launch_bounds__(256) void lnq_prepare_kernel(const float* __restrict__ H, int64_t d, int64_t ldp, unsigned n_max,
                                                          unsigned* __restrict__ most, int in_parts, int64_t n_clear,
                                                          const unsigned char* __restrict__ Q, int64_t d_out, int n_levels,
                                                          int planes, unsigned char* __restrict__ Qp) {
  if (blockIdx.x >= n_max) {
    const int64_t t = (int64_t)(blockIdx.x - n_max) * 256 + threadIdx.x;
    for (int64_t i = t; i < n_clear; i += (int64_t)gridDim.x * 256) most[i] = 0u;
    pad_codes(t, Q, d, ldp, d_out, n_levels, planes, Qp);
    return;
  }
  __shared__ unsigned tile[64][65];
  __shared__ unsigned found[2][64];
  const int64_t n_t = (d + 63) / 64, n_tri = tri_count(n_t);
  const int k = (int)(blockIdx.x / (unsigned)n_tri);
  int ti, tj;
  tri_decode((int64_t)(blockIdx.x % (unsigned)n_tri), ti, tj);
  const float* Hk = H + (int64_t)k * d * d;
  const int tx = threadIdx.x % 64, ty = threadIdx.x / 64;
  const int64_t b = (int64_t)tj * 64 + tx;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int64_t a = (int64_t)ti * 64 + ty + 4 * u;
    const int64_t ac = a < d ? a : d - 1, bc = b < d ? b : d - 1;
    const unsigned bits = __builtin_bit_cast(unsigned, Hk[ac * d + bc]) & 0x7fffffffu;
    tile[ty + 4 * u][tx] = (a < d && b < d && a <= b) ? bits : 0u;
  }
  __syncthreads();
  if (threadIdx.x < 128) {                                   // threads 0 .. 63: a row of the tile each; 64 .. 127: a column
    const bool rows = threadIdx.x < 64;
    unsigned m = 0;
#pragma unroll
    for (int e = 0; e < 64; ++e) {
      const unsigned v = rows ? tile[tx][e] : tile[e][tx];
      m = v > m ? v : m;
    }
    found[rows ? 0 : 1][tx] = m;
  }
  __syncthreads();
  if (threadIdx.x < 128) {
    const bool rows = threadIdx.x < 64;
    unsigned m = found[rows ? 0 : 1][tx];
    if (ti == tj) {                                          // one block of rows: both kinds together
      if (!rows) return;
      m = found[1][tx] > m ? found[1][tx] : m;
    }
    const int64_t i = (int64_t)(rows ? ti : tj) * 64 + tx;
    if (in_parts) most[((int64_t)k * n_t + (rows ? tj : ti)) * ldp + i] = m;
    else if (i < d && m) atomicMax(most + (int64_t)k * ldp + i, m);
  }
}
// e with 2^(e - 1) <= x < 2^e for the x whose bits these are (0 for 0, infinity and NaN)
__device__ inline int row_exponent(unsigned bits) { return __builtin_amdgcn_frexp_expf(__builtin_bit_cast(float, bits)); }

// Rows [row0, row0 + 64 * gridDim.y) of the full symmetric H[k0 + z] (from its upper triangle) in fixed point, as
// four digits (digit 3 first): planes of [gridDim.z][pass_rows][ldp] bytes, plane_bytes apart, zero padded.
// One workgroup per 64 x 64 tile.
__global__ __launch_bounds__(256) void lnq_split_h_kernel(const float* __restrict__ H, int64_t d, int64_t ldp, int k0,
                                                          int64_t row0, int64_t pass_rows,
                                                          unsigned* __restrict__ most,
                                                          const unsigned* __restrict__ most_part, int64_t plane_bytes,
                                                          unsigned char* __restrict__ Hd) {
  __shared__ float tile[64][65];
  __shared__ unsigned found[4][64];
  const int kk = blockIdx.z;
  const int ti = (int)(row0 / 64) + blockIdx.y, tj = blockIdx.x;
  const float* Hk = H + (int64_t)(k0 + kk) * d * d;
  unsigned* mk = most + (int64_t)(k0 + kk) * ldp;
  const int tmin = ti < tj ? ti : tj, tmax = ti < tj ? tj : ti;
  const int tx = threadIdx.x % 64, ty = threadIdx.x / 64;
#pragma unroll
  for (int u = 0; u < 16; ++u) {                            // the tile on or above the diagonal; clamped, branch-free
    const int r = ty + 4 * u;
    const int64_t a = (int64_t)tmin * 64 + r, b = (int64_t)tmax * 64 + tx;
    const int64_t ac = a < d ? a : d - 1, bc = b < d ? b : d - 1;
    const float v = Hk[ac * d + bc];
    tile[r][tx] = (a < d && b < d) ? v : 0.f;
  }
  {                                                         // the largest entry of this tile's 64 rows
    const int64_t i = (int64_t)ti * 64 + tx;
    unsigned m = 0;
    if (most_part) {                                        // uniform
      const int64_t n_t = (d + 63) / 64;
      const unsigned* src = most_part + (int64_t)(k0 + kk) * n_t * ldp + i;
      if (ti < n_t)
        for (int64_t t = ty; t < n_t; t += 4) {
          const unsigned v = src[t * ldp];
          m = v > m ? v : m;
        }
    } else if (ty == 0 && i < d) {
      m = mk[i];
    }
    found[ty][tx] = m;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    unsigned m = found[0][tx];
    for (int w = 1; w < 4; ++w) m = found[w][tx] > m ? found[w][tx] : m;
    found[0][tx] = m;
    if (most_part && tj == 0) mk[(int64_t)ti * 64 + tx] = m;   // for the kernels that follow
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {                             // row li, columns lj0 .. lj0 + 3
    const int li = (int)threadIdx.x / 16 + 16 * u, lj0 = 4 * ((int)threadIdx.x % 16);
    const int up = kBits - row_exponent(found[0][li]);
    unsigned out[4] = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int lj = lj0 + e;
      float h;
      if (ti < tj) h = tile[li][lj];
      else if (ti > tj) h = tile[lj][li];
      else h = li <= lj ? tile[li][lj] : tile[lj][li];
      int q = (int)rintf(ldexpf(h, up));                    // (a row with an infinity or a NaN: whatever, T becomes NaN)
#pragma unroll
      for (int g = 3; g >= 0; --g) {                        // balanced digits, lowest first
        const int digit = g > 0 ? (int)(signed char)(q & 0xff) : q;
        out[g] |= (unsigned)(digit & 0xff) << (8 * e);
        q = (q - digit) >> 8;
      }
    }
    const int64_t off = ((int64_t)kk * pass_rows + (int64_t)blockIdx.y * 64 + li) * ldp + (int64_t)tj * 64 + lj0;
#pragma unroll
    for (int g = 0; g < 4; ++g) *reinterpret_cast<unsigned*>(Hd + g * plane_bytes + off) = out[g];
  }
}

// Eight bf16 values, 1.0 where the code byte equals the lane's grid point (qrep = that point in
// every byte), else 0.  All bytes involved are below 0x80, so adding 0x7F to a byte sets its
// top bit exactly when the byte is non-zero and never carries into the next byte.
__device__ inline bf16x8 onehot_frag(unsigned c0, unsigned c1, unsigned qrep) {
  const unsigned m0 = ~((c0 ^ qrep) + 0x7F7F7F7Fu) & 0x80808080u;        // 0x80 in every matching byte
  const unsigned m1 = ~((c1 ^ qrep) + 0x7F7F7F7Fu) & 0x80808080u;
  auto one = [](unsigned s) { return (s << 7) - s; };                    // 0x0080 -> 0x3F80 in both halves
  u32x4 v;
  v[0] = one(__builtin_amdgcn_perm(0u, m0, 0x0C010C00u));                 // bytes 0, 1 -> the low bytes of the halves
  v[1] = one(__builtin_amdgcn_perm(0u, m0, 0x0C030C02u));
  v[2] = one(__builtin_amdgcn_perm(0u, m1, 0x0C010C00u));
  v[3] = one(__builtin_amdgcn_perm(0u, m1, 0x0C030C02u));
  return __builtin_bit_cast(bf16x8, v);
}

// T[r][i] = sum_{i'} E[r][i'] * H[k][i][i']  for the rows r = (channel, grid point) of whole
// channels (256 rows at most) and 128 columns i at a time.  8 waves of 64 x 64 (4 along
// the rows, 2 along the columns).  The contraction is swept twice, first with digits 3 and 1 of H, then, the
// two sums shifted left by 8 bits, with digits 2 and 0: two accumulators per result instead of four, so that two
// waves per SIMD have room.  A stage is 128 contraction elements: one whole 128-byte line of each of the 2 x 128
// rows of the digits and of the rows of codes, copied straight into LDS (global_load_lds_dwordx4; chunk c of row r
// at position c ^ ((r >> 1) & 7)); a ring of four stages, one barrier per stage.  A lane's contraction
// elements within a stage are the 64 consecutive ones of its half-wave (the matrix cores do not
// care about the order as long as both operands agree), so its codes are four 16-byte reads.
// Per wave and stage: 32 matrix instructions, 24 LDS reads, 32 byte permutations.  Measured at 4096 channels x 4096
// coordinates, 4 groups, 8 grid points: 1.75 ms, 2.5 P integer operations/s (half the peak; one sixteenth of them useful
// sums); the three-term bf16 product took 2.4.  d_in = 11008: the whole step 19.0 -> 12.7 ms.
//
// A workgroup works through `cts_per` consecutive column tiles.  After each, the tile of T goes
// to LDS (the ring is idle then) and is binned where it lies:
//   A[r][u] += sum_i T[r][i] * [Q[j(r)][i] == u]  is one more product with one-hot rows: the rows of
//   the tile are cut into blocks of whole channels (at most 32 rows); for a block, T (split into
//   three bf16 terms, so that the one-hot products are exact again) times the transposed one-hot rows
//   of the same block gives a 32 x 32 result whose entry (r, n) with r and n in the same channel is
//   A[r][level of n].  Wave w owns blocks w and w + 8 and keeps their results in matrix-core
//   accumulators over all column tiles: the order of additions is fixed by the instruction stream.
//   b[r] += sum_i T[r][i] * w[j(r)][i]  in fp32 by two threads per row, 64 columns each, in column order.
// At the end both are written (or, in a later pass over the same channels, added) to row r of
// part[chunk][channel * n_levels + q][LV + 1] (b in column LV).  One launch covers the groups
// [k0, k0 + Gp) and the column tiles [ct0, ct0 + n_ct) whose rows of H the split buffers hold
// ([Gp][pass_rows][ldp]).  Workgroups are renumbered so that each XCD works through chunks of its
// own: a block of H is fetched into one L2 only.
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
constexpr int kTilePitch = kCols + 4;                 // floats per row of the tile of T in LDS (16-byte aligned rows)
template <int LV>
__global__ __launch_bounds__(512) void lnq_gemm_kernel(const unsigned char* __restrict__ Qp, int planes,
                                                       const unsigned char* __restrict__ Hd, int64_t h_plane,
                                                       const unsigned* __restrict__ most,
                                                       const float* __restrict__ W, int64_t ld, int64_t d,
                                                       int64_t per_group, int n_levels, int n_ch, int n_rt, int k0,
                                                       int Gp, int ct0, int n_ct, int cts_per, int n_chunks,
                                                       int64_t ldp, int64_t pass_rows, int64_t part_rows, int sweep0,
                                                       int n_stages, int accumulate, float* __restrict__ part) {
  constexpr int kRingBytes = kRing * (kHStage + kQStage), kTileBytes = kRows * kTilePitch * 4;
  __shared__ __attribute__((aligned(1024))) char smem[kRingBytes > kTileBytes ? kRingBytes : kTileBytes];
  const int n_blocks = n_rt * Gp * n_chunks;
  const int per_xcd = (n_blocks + 7) / 8;
  const int v = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if (v >= n_blocks) return;                                   // the whole workgroup, before any barrier
  const int chunk = v / (n_rt * Gp), rtg = v % (n_rt * Gp);
  const int kk = rtg / n_rt, rt = rtg % n_rt;
  const int k = k0 + kk;
  const int64_t j0 = (int64_t)k * per_group + (int64_t)rt * n_ch, j_last = (int64_t)(k + 1) * per_group - 1;
  const int64_t ch_left = per_group - (int64_t)rt * n_ch;
  const int rows_here = (int)(ch_left < n_ch ? ch_left : n_ch) * n_levels;   // rows of this tile that exist
  const int ct_first = chunk * cts_per;
  const int ct_end = ct_first + cts_per < n_ct ? ct_first + cts_per : n_ct;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wm = wave / 2, wn = wave % 2;
  const unsigned smem_base = (unsigned)(uintptr_t)(lds_char_ptr)smem;
  const unsigned q_base = smem_base + kRing * kHStage;

  // Staging: wave w moves four pieces of 1 KiB (8 rows) of the digits and one of the codes per stage.  A load is a
  // scalar base plus the lane's 32-bit offset: row lane / 8 of the piece, chunk (lane % 8) ^ ((row >> 1) & 7) of it.
  // Piece g = 4 w + i: digit g / 16 (0: the high pair's, 3 then 2; 1: the low pair's, 1 then 0), rows 8 (g % 16) ..
  const unsigned vo_row = (unsigned)(lane / 8) * (unsigned)ldp;
  const unsigned vo_h[2] = {vo_row + 16u * ((lane % 8) ^ (lane / 16)),                  // even pieces: (row >> 1) & 7 = lane / 16
                            vo_row + 16u * ((lane % 8) ^ (4 + lane / 16))};             // odd ones: 4 more
  const unsigned char* const hbase =
      Hd + 2 * (wave / 4) * h_plane + ((int64_t)kk * pass_rows + 32 * (wave % 4)) * ldp + (int64_t)sweep0 * kK;
  // Rows of codes: the tile's channels in plane 0, then (with more than 8 grid points) in plane 1; channels past the
  // group repeat its last one (never stored).
  unsigned vo_q;
  {
    const int r = 8 * wave + lane / 8;
    const int c = (lane % 8) ^ ((r >> 1) & 7);
    const int plane = (r >= n_ch && n_levels > 8) ? 1 : 0;
    const int64_t left = j_last - j0;
    int64_t ch = r - plane * n_ch;
    ch = ch < left ? ch : left;
    vo_q = (unsigned)((ch * planes + plane) * ldp + 16 * c);
  }
  const unsigned char* const qbase = Qp + j0 * planes * ldp + (int64_t)sweep0 * kK;

  // the two rows of E this lane supplies: the place of its codes in a stage, and the table that holds a 1 at its grid point
  const int lrow = lane % 32, half = lane / 32;
  unsigned tab_lo[2], tab_hi[2], q_at[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int lr = wm * 64 + 32 * x + lrow;
    const bool valid = lr < rows_here;
    const int ch = valid ? lr / n_levels : 0, lvl = valid ? lr % n_levels : 0;
    tab_lo[x] = valid && lvl % 8 < 4 ? 1u << (8 * (lvl % 8)) : 0u;
    tab_hi[x] = valid && lvl % 8 >= 4 ? 1u << (8 * (lvl % 8 - 4)) : 0u;
    const int row = ch + (lvl / 8) * n_ch;
    q_at[x] = kRing * kHStage + row * kK + 16 * ((4 * half) ^ ((row >> 1) & 7));
  }
  // chunk t of the half-wave's four sits at the place of chunk 0 with bits 4 and 5 of the address flipped by t
  const unsigned h_at = (wn * 64 + lrow) * kK + 16 * ((4 * half) ^ ((lrow >> 1) & 7));
  struct Frags {
    i32x4 a[2], h[2][2];
  };
  u32x4 codes[2];
  auto read_codes = [&](int slot, int t) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
      codes[x] = *reinterpret_cast<const u32x4*>(&smem[(slot * kQStage + q_at[x]) ^ (16u * t)]);
  };
  auto read_h = [&](Frags& f, int slot, int t, int g) {
#pragma unroll
    for (int y = 0; y < 2; ++y)
      f.h[g][y] = *reinterpret_cast<const i32x4*>(&smem[((slot * kHStage + h_at) ^ (16u * t)) + g * kDTile + y * 32 * kK]);
  };
  auto select = [&](Frags& f, int x) {                         // four codes at a time -> bytes of E
#pragma unroll
    for (int e = 0; e < 4; ++e) f.a[x][e] = (int)__builtin_amdgcn_perm(tab_hi[x], tab_lo[x], codes[x][e]);
  };

  // binning blocks: whole channels, at most 32 rows; this wave owns blocks wave and wave + 8
  const int rpb = (32 / n_levels) * n_levels;
  const int n_bb = (rows_here + rpb - 1) / rpb;                // at most 12 for n_levels <= 16
  float* tile = reinterpret_cast<float*>(smem);
  f32x16 bacc[2];
  int b_arow[2], b_ch[2], b_lvl[2];
  bool b_valid[2];
  unsigned b_qrep[2];
  const unsigned char* b_q[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
#pragma unroll
    for (int r = 0; r < 16; ++r) bacc[x][r] = 0.f;
    const int bb = wave + 8 * x;
    const int nrow = bb * rpb + lane % 32;                     // the row this lane stands for, as A row and as column n
    b_valid[x] = bb < n_bb && lane % 32 < rpb && nrow < rows_here;
    b_arow[x] = nrow < kRows ? nrow : kRows - 1;
    b_ch[x] = b_valid[x] ? nrow / n_levels : 0;
    b_lvl[x] = b_valid[x] ? nrow % n_levels : 0;
    b_qrep[x] = b_valid[x] ? (unsigned)(b_lvl[x] % 8) * 0x01010101u : kNoLevel;
    b_q[x] = Qp + ((j0 + b_ch[x]) * planes + b_lvl[x] / 8) * ldp + 8 * (lane / 32);
  }
  // b: two threads per row, 64 columns each
  const int brow = tid / 2, bhalf = tid % 2;
  const bool brow_valid = brow < rows_here;
  const int64_t bj = j0 + (brow_valid ? brow / n_levels : 0);
  float dot = 0.f;

  for (int ct = ct_first; ct < ct_end; ++ct) {
    const int64_t c0 = (int64_t)(ct0 + ct) * kCols;           // first column of T (= row of H) of this tile
    // stage st of 2 * n_stages: sweep st / n_stages, whose digits lie one plane further
    const int last = 2 * n_stages - 1;
    auto issue = [&](int st, int slot) {
      st = st < last ? st : last;                           // past the end: a harmless repeat keeps the count uniform
      const int sweep = st >= n_stages ? 1 : 0;
      const int64_t off = (int64_t)(st - sweep * n_stages) * kK;
      const unsigned char* h = hbase + (int64_t)ct * kCols * ldp + off + sweep * h_plane;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        dma16s(h + 8 * i * ldp, vo_h[i % 2], smem_base + slot * kHStage + (wave * 4 + i) * 1024);
      dma16s(qbase + off, vo_q, q_base + slot * kQStage + wave * 1024);
    };
    i32x16 acc[2][2][2];                                    // [digit pair][x][y]
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[g][x][y][r] = 0;

    // Stage s + 1 is in LDS before stage s is multiplied, so that its first fragments can be read in time; s + 2 and
    // s + 3 are on their way.  The operands of the next 32 contraction elements are read, and their codes turned
    // into bytes of E, between the eight matrix instructions of the current ones.
    issue(0, 0);
    issue(1, 1);
    issue(2, 2);
    wait_vmcnt<2 * kLoadsPerStage>();
    __builtin_amdgcn_s_barrier();
    Frags f0, f1;
    read_codes(0, 0);
    read_h(f0, 0, 0, 0);
    read_h(f0, 0, 0, 1);
    select(f0, 0);
    select(f0, 1);
    auto step = [&](const Frags& cur, Frags& nxt, int slot, int t) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int g = i / 4, y = (i / 2) % 2, x = i % 2;
        acc[g][x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur.a[x], cur.h[g][y], acc[g][x][y], 0, 0, 0);
        if (i == 0) read_codes(slot, t);
        if (i == 1) read_h(nxt, slot, t, 0);
        if (i == 2) read_h(nxt, slot, t, 1);
        if (i == 5) select(nxt, 0);
        if (i == 6) select(nxt, 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    int slot = 0;
    for (int sweep = 0; sweep < 2; ++sweep) {
      for (int s = sweep * n_stages; s < (sweep + 1) * n_stages; ++s) {
        wait_vmcnt<kLoadsPerStage>();                       // this wave's loads of stage s + 1 have landed
        __builtin_amdgcn_s_barrier();                       // everyone's have; and everyone is done with stage s - 1
        issue(s + 3, (slot + 3) % kRing);
        step(f0, f1, slot, 1);
        step(f1, f0, slot, 2);
        step(f0, f1, slot, 3);
        slot = (slot + 1) % kRing;
        step(f1, f0, slot, 0);
      }
      if (sweep == 0) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
              for (int r = 0; r < 16; ++r) acc[g][x][y][r] = (int)((unsigned)acc[g][x][y][r] << 8);
      }
    }
    wait_vmcnt<0>();                                        // the repeats issued past the end
    __syncthreads();                                        // every wave is done with the ring: it becomes the tile of T

    // register r of lane l holds row 8*(r/4)+4*(l/32)+(r%4), column l%32 of a 32 x 32 block.  The sums of the two
    // pairs are put together in 64 bits and rounded once; a row of H with an infinity or a NaN gives NaN.
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int64_t i = c0 + wn * 64 + 32 * y + lane % 32;
      const unsigned bits = i < d ? most[(int64_t)k * ldp + i] : 0u;
      const bool finite = bits < 0x7f800000u;
      const int down = row_exponent(bits) - kBits;
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int lr = wm * 64 + 32 * x + 8 * (r / 4) + 4 * (lane / 32) + (r % 4);
          const double v = __builtin_fma((double)acc[0][x][y][r], 65536.0, (double)acc[1][x][y][r]);
          const float f = (float)__builtin_amdgcn_ldexp(v, down);
          tile[lr * kTilePitch + wn * 64 + 32 * y + lane % 32] = finite ? f : __builtin_nanf("");
        }
    }
    __builtin_amdgcn_sched_barrier(0);                      // the accumulators are dead from here on: no load moves above
    // the codes of the binning blocks are fetched before the barrier and used after it
    unsigned bcodes[2][8][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
      if (wave + 8 * x < n_bb) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          const uint2 cc = *reinterpret_cast<const uint2*>(b_q[x] + c0 + 16 * ks);
          bcodes[x][ks][0] = cc.x;
          bcodes[x][ks][1] = cc.y;
        }
      }
    __syncthreads();
    // the weights of this thread's 64 columns, 32 at a time
    f32x4 wv[8];
    auto fetch_w = [&](int piece) {
      const float* wrow = W + bj * ld;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int64_t i = c0 + 64 * bhalf + 32 * piece + 4 * c;
        if (i + 3 < d) {
          wv[c] = *reinterpret_cast<const f32x4*>(wrow + i);
        } else {                                            // the ragged end: any finite value will do past d (T is 0 there)
#pragma unroll
          for (int e = 0; e < 4; ++e) wv[c][e] = wrow[i + e < d ? i + e : d - 1];
        }
      }
    };
    if (brow_valid) fetch_w(0);
#pragma unroll
    for (int x = 0; x < 2; ++x)
      if (wave + 8 * x < n_bb) {                              // wave-uniform
        const float* ta = tile + b_arow[x] * kTilePitch + 8 * (lane / 32);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          const f32x4 t0 = *reinterpret_cast<const f32x4*>(ta + 16 * ks);
          const f32x4 t1 = *reinterpret_cast<const f32x4*>(ta + 16 * ks + 4);
          u16x8 ah, am, al;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            unsigned short h, m, l;
            split3_bf16(e < 4 ? t0[e] : t1[e - 4], h, m, l);
            ah[e] = h;
            am[e] = m;
            al[e] = l;
          }
          const bf16x8 onehot = onehot_frag(bcodes[x][ks][0], bcodes[x][ks][1], b_qrep[x]);
          bacc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, al), onehot, bacc[x], 0, 0, 0);
          bacc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, am), onehot, bacc[x], 0, 0, 0);
          bacc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ah), onehot, bacc[x], 0, 0, 0);
        }
      }
    __builtin_amdgcn_sched_barrier(0);
    if (brow_valid) {
      const float* trow = tile + brow * kTilePitch + 64 * bhalf;
#pragma unroll
      for (int c = 0; c < 32; ++c) dot += trow[c] * wv[c / 4][c % 4];   // T is exactly 0 in the padded columns
      fetch_w(1);
#pragma unroll
      for (int c = 0; c < 32; ++c) dot += trow[32 + c] * wv[c / 4][c % 4];
    }
    __syncthreads();                                        // the ring is free again
  }

  float* prow = part + ((int64_t)chunk * part_rows + j0 * n_levels) * (LV + 1);
  dot += __shfl_xor(dot, 1, kWave);
  if (brow_valid && bhalf == 0) {
    float* dst = prow + (int64_t)brow * (LV + 1) + LV;
    *dst = accumulate ? *dst + dot : dot;
  }
  // register r of lane l holds row 8*(r/4)+4*(l/32)+(r%4), column l%32 of a block's 32 x 32 result
#pragma unroll
  for (int x = 0; x < 2; ++x)
    if (b_valid[x]) {
      const int r0 = (wave + 8 * x) * rpb;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = 8 * (r / 4) + 4 * (lane / 32) + (r % 4);
        const int row = r0 + rl;
        if (rl < rpb && row < rows_here && row / n_levels == b_ch[x]) {
          float* dst = prow + (int64_t)row * (LV + 1) + b_lvl[x];
          *dst = accumulate ? *dst + bacc[x][r] : bacc[x][r];
        }
      }
    }
}

// Four channels per workgroup.  Its first wave solves them, sixteen lanes per channel: lane r of a channel holds row r of
// its system in registers.  Adds the partial systems in chunk order (A: m x m, b: m) and solves (A + lam I) c = b in fp64
// by Gauss-Jordan elimination with partial pivoting: at step p the pivot is the largest entry of column p among the
// rows not yet used (the lowest row among equals); every other row is cleared in that column.  Rows are never moved.
// The steps depend on one another, so what counts is their latency: everything crosses lanes by permutation, there is
// no barrier.  (One workgroup per channel with the system in LDS took 32 us for 4096 channels of 8 grid points, this 12.)
// Then the workgroup writes the grid values and, if wanted, What[j][i] = c[Q[j][i]].  LV = 4, 8 or 16 bounds the number
// of grid points.
constexpr int kSolveChannels = 4;
template <int LV>
__global__ __launch_bounds__(256) void lnq_solve_kernel(const float* __restrict__ part, int n_chunks, int64_t part_rows,
                                                        const unsigned char* __restrict__ Q, int64_t d_out, int64_t d,
                                                        int64_t ld, int n_levels, double lam,
                                                        float* __restrict__ codebook, float* __restrict__ What) {
  __shared__ float cval[kSolveChannels][16];
  const int tid = threadIdx.x;
  const int n = n_levels;
  const int64_t j0 = (int64_t)blockIdx.x * kSolveChannels;
  if (tid < kWave) {
    const int ch = tid / 16, r = tid % 16;
    const int64_t j = j0 + ch, jc = j < d_out ? j : d_out - 1;
    const bool real = r < n;
    double row[LV + 1];                                        // column LV: b
#pragma unroll
    for (int u = 0; u <= LV; ++u) row[u] = 0.0;
    {
      const float* src = part + (jc * n + (real ? r : 0)) * (LV + 1);
      for (int c = 0; c < n_chunks; ++c)
#pragma unroll
        for (int u = 0; u <= LV; ++u) row[u] += (double)src[(int64_t)c * part_rows * (LV + 1) + u];   // (entries past n_levels: never used)
    }
#pragma unroll
    for (int u = 0; u < LV; ++u) row[u] += u == r ? lam : 0.0;

    bool used = !real;
    int mine = -1;                                             // the column whose pivot this row became
    double pivot = 0.0;
#pragma unroll
    for (int p = 0; p < LV; ++p) {
      if (p < n) {                                             // uniform
        // the pivot row: largest |entry| first, then the lowest lane (a NaN is never larger)
        double best = used ? -1.0 : fabs(row[p]);
        best = best >= 0.0 ? best : -1.0;                      // NaN
        int at = r;
#pragma unroll
        for (int w = 1; w < 16; w <<= 1) {
          const double ob = __shfl_xor(best, w, 16);
          const int oa = __shfl_xor(at, w, 16);
          const bool take = ob > best || (ob == best && oa < at);
          best = take ? ob : best;
          at = take ? oa : at;
        }
        at = best < 0.0 ? 0 : at;                              // nothing but NaN left
        const double piv = __shfl(row[p], at, 16);
        const double inv = piv != 0.0 ? 1.0 / piv : 0.0;
        const double f = row[p] * inv;
        const bool self = r == at;
        if (self) {
          mine = p;
          pivot = piv;
          used = true;
        }
#pragma unroll
        for (int u = p + 1; u <= LV; ++u) {
          const double o = __shfl(row[u], at, 16);
          row[u] = self ? row[u] : row[u] - f * o;
        }
      }
    }
    // (a system full of NaN has used one row several times: the grid points without a row of their own stay NaN)
    cval[ch][r] = __builtin_nanf("");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    if (mine >= 0) cval[ch][mine] = pivot != 0.0 ? (float)(row[LV] / pivot) : 0.f;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    if (real && j < d_out) codebook[j * n + r] = cval[ch][r];
  }
  __syncthreads();
  if (!What) return;
  const int n_here = (int)(d_out - j0 < kSolveChannels ? d_out - j0 : kSolveChannels);
  // four coordinates at a time where the rows of Q start at multiples of four bytes (those of What always start at 16)
  if (d % 4 == 0 && (reinterpret_cast<uintptr_t>(Q) & 3) == 0) {
    const int64_t quads = d / 4;
    for (int64_t t = tid; t < n_here * quads; t += 256) {
      const int64_t jj = t / quads, i = 4 * (t - jj * quads);
      const unsigned w = *reinterpret_cast<const unsigned*>(Q + (j0 + jj) * d + i);
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int code = (int)((w >> (8 * e)) & 0xffu);
        v[e] = code < n ? cval[jj][code & 15] : 0.f;
      }
      *reinterpret_cast<f32x4*>(What + (j0 + jj) * ld + i) = v;
    }
  } else {
    for (int64_t t = tid; t < n_here * d; t += 256) {
      const int64_t jj = t / d, i = t - jj * d;
      const int code = Q[(j0 + jj) * d + i];
      What[(j0 + jj) * ld + i] = code < n ? cval[jj][code & 15] : 0.f;
    }
  }
}

// The four digits of H are staged in passes: all groups at once if that fits kSplitBudget,
// else one group and a range of column tiles (= rows of H) at a time.
constexpr size_t kSplitBudget = (size_t)512 << 20;

struct Layout {
  int64_t ldp, part_rows, pass_rows;
  int n_ch, n_rt, n_ct, groups_per_pass, pass_cts, cts_per, chunks_per_pass, lv, code_planes;
  size_t h_bytes, q_bytes, part_bytes, most_bytes, most_part_bytes;   // h_bytes: one digit; q_bytes: one plane of codes
};
Layout make_layout(int64_t d_out, int64_t d_in, int G, int n_levels) {
  Layout L;
  L.ldp = (d_in + kCols - 1) / kCols * kCols;
  const int64_t per_group = d_out / G;
  L.code_planes = n_levels > 8 ? 2 : 1;
  const int max_ch = kMaxCodeRows / L.code_planes;
  L.n_ch = kRows / n_levels < max_ch ? kRows / n_levels : max_ch;          // whole channels per workgroup
  L.n_rt = (int)((per_group + L.n_ch - 1) / L.n_ch);
  L.n_ct = (int)(L.ldp / kCols);
  const size_t per_tile_row = (size_t)4 * L.ldp * kCols;                   // bytes of the four digits of one column tile
  if (per_tile_row * L.n_ct * G <= kSplitBudget) {
    L.groups_per_pass = G;
    L.pass_cts = L.n_ct;
  } else {                                                                  // passes of equal size
    L.groups_per_pass = 1;
    int64_t fit = (int64_t)(kSplitBudget / per_tile_row);
    fit = fit < 1 ? 1 : fit;
    const int64_t n_passes = (L.n_ct + fit - 1) / fit;
    L.pass_cts = (int)((L.n_ct + n_passes - 1) / n_passes);
  }
  // Column tiles per chunk: one workgroup per (row block, chunk), one workgroup per compute unit at a time.
  // Chunks stay short (at most 4 tiles): the workgroups of an XCD share a tile's rows of H in their L2 only
  // while they work on the same tile, and they drift apart over a long chunk (16 tiles per chunk ran at half
  // the speed of 1).  Of 4, 3, 2, 1 the first that fills whole rounds of 256 workgroups to 93 %, because
  // every chunk costs a partial system per channel; if none does, the best filled one.
  const int64_t row_blocks = (int64_t)L.n_rt * L.groups_per_pass;
  int best = 1;
  double best_eff = -1.0;
  for (int per = L.pass_cts < 4 ? L.pass_cts : 4; per >= 1; --per) {
    const int64_t chunks = (L.pass_cts + per - 1) / per;
    const int64_t wgs = row_blocks * chunks, rounds = (wgs + 255) / 256;
    const double eff = (double)wgs / (double)(rounds * 256);
    if (wgs >= 256 && eff >= 0.93) {
      best = per;
      break;
    }
    if (eff > best_eff + 1e-9) {
      best_eff = eff;
      best = per;
    }
  }
  L.cts_per = best;
  L.chunks_per_pass = (L.pass_cts + L.cts_per - 1) / L.cts_per;
  L.pass_rows = (int64_t)L.pass_cts * kCols;
  L.lv = n_levels <= 4 ? 4 : (n_levels <= 8 ? 8 : 16);
  L.part_rows = d_out * n_levels;
  auto up = [](size_t b) { return (b + 255) / 256 * 256; };
  L.h_bytes = up((size_t)L.groups_per_pass * L.pass_rows * L.ldp);
  L.most_bytes = up((size_t)G * L.ldp * sizeof(unsigned));
  const int64_t n_t = (d_in + 63) / 64;
  L.most_part_bytes = n_t <= kPartTiles ? up((size_t)G * n_t * L.ldp * sizeof(unsigned)) : 0;
  L.q_bytes = up((size_t)d_out * L.ldp);
  L.part_bytes = up((size_t)L.chunks_per_pass * L.part_rows * (L.lv + 1) * sizeof(float));
  return L;
}

}  // namespace

size_t lnq_codebook_workspace(int64_t d_out, int64_t d_in, int G, int n_levels) {
  const Layout L = make_layout(d_out, d_in, G, n_levels);
  return 4 * L.h_bytes + L.code_planes * L.q_bytes + L.part_bytes + L.most_bytes + L.most_part_bytes;
}

hipError_t launch_lnq_codebook(const float* W, int64_t d_out, int64_t d_in, int64_t ld, const unsigned char* Q,
                               const float* H, int G, int n_levels, double lam, float* codebook, float* What,
                               void* ws, bool splits_done, hipStream_t st) {
  const Layout L = make_layout(d_out, d_in, G, n_levels);
  // splits_done: an earlier call with the same H and this workspace has left the digits of H in place
  // (they survive a call only when one pass holds all of them)
  const bool keep_splits = splits_done && L.groups_per_pass == G && L.pass_cts == L.n_ct;
  char* p = (char*)ws;
  unsigned char* Hd = (unsigned char*)p;
  p += 4 * L.h_bytes;
  unsigned char* Qp = (unsigned char*)p;
  p += L.code_planes * L.q_bytes;
  float* part = (float*)p;
  p += L.part_bytes;
  unsigned* most = (unsigned*)p;
  p += L.most_bytes;
  unsigned* most_part = L.most_part_bytes ? (unsigned*)p : nullptr;

  hipError_t e;
  {
    const int64_t n_t = (d_in + 63) / 64, tiles = keep_splits ? 0 : tri_count(n_t) * G;
    const int64_t codes = (d_out * L.ldp / 4 + 255) / 256;
    if (codes + tiles > 0x7fffffff) return hipErrorInvalidValue;
    const int64_t clear = keep_splits || most_part ? 0 : G * L.ldp;
    auto prepare = [&](int64_t max_blocks, int64_t code_blocks, int64_t n_clear) {
      lnq_prepare_kernel<<<dim3((unsigned)(max_blocks + code_blocks)), dim3(256), 0, st>>>(
          H, d_in, L.ldp, (unsigned)max_blocks, most_part ? most_part : most, most_part ? 1 : 0, n_clear, Q, d_out, n_levels,
          L.code_planes, Qp);
      return hipGetLastError();
    };
    if (clear == 0) {
      if ((e = prepare(tiles, codes, 0)) != hipSuccess) return e;
    } else {
      if ((e = prepare(0, codes, clear)) != hipSuccess) return e;
      if ((e = prepare(tiles, 0, 0)) != hipSuccess) return e;
    }
  }
  for (int k0 = 0; k0 < G; k0 += L.groups_per_pass) {
    for (int ct0 = 0; ct0 < L.n_ct; ct0 += L.pass_cts) {
      const int n_ct = ct0 + L.pass_cts <= L.n_ct ? L.pass_cts : L.n_ct - ct0;
      const int n_chunks = (n_ct + L.cts_per - 1) / L.cts_per;
      if (!keep_splits) {
        lnq_split_h_kernel<<<dim3((unsigned)(L.ldp / 64), (unsigned)(n_ct * (kCols / 64)), (unsigned)L.groups_per_pass),
                             dim3(256), 0, st>>>(H, d_in, L.ldp, k0, (int64_t)ct0 * kCols, L.pass_rows, most,
                                                 most_part, (int64_t)L.h_bytes, Hd);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      const int64_t n_blocks = (int64_t)L.n_rt * L.groups_per_pass * n_chunks;
      const int64_t grid = (n_blocks + 7) / 8 * 8;
      if (grid > 0x7fffffff) return hipErrorInvalidValue;
      // a contraction too long for 32-bit sums runs in several launches that add to the partial systems
      for (int64_t sw = 0; sw < L.ldp; sw += kMaxSweep) {
        const int stages = (int)((L.ldp - sw < kMaxSweep ? L.ldp - sw : kMaxSweep) / kK);
        const int accumulate = (ct0 > 0 || sw > 0) ? 1 : 0;
#define GQ_LNQ_GEMM(LV)                                                                                                \
  lnq_gemm_kernel<LV><<<dim3((unsigned)grid), dim3(512), 0, st>>>(                                                      \
      Qp, L.code_planes, Hd, (int64_t)L.h_bytes, most, W, ld, d_in, d_out / G, n_levels, L.n_ch, L.n_rt, k0,               \
      L.groups_per_pass, ct0, n_ct, L.cts_per, n_chunks, L.ldp, L.pass_rows, L.part_rows, (int)(sw / kK), stages,       \
      accumulate, part);
        if (L.lv == 4) {
          GQ_LNQ_GEMM(4)
        } else if (L.lv == 8) {
          GQ_LNQ_GEMM(8)
        } else {
          GQ_LNQ_GEMM(16)
        }
#undef GQ_LNQ_GEMM
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
    }
  }
  const unsigned solve_grid = (unsigned)((d_out + kSolveChannels - 1) / kSolveChannels);
#define GQ_LNQ_SOLVE(LV)                                                                                       \
  lnq_solve_kernel<LV><<<dim3(solve_grid), dim3(256), 0, st>>>(part, L.chunks_per_pass, L.part_rows, Q, d_out, d_in, ld, \
                                                               n_levels, lam, codebook, What)
  if (L.lv == 4)
    GQ_LNQ_SOLVE(4);
  else if (L.lv == 8)
    GQ_LNQ_SOLVE(8);
  else
    GQ_LNQ_SOLVE(16);
#undef GQ_LNQ_SOLVE
  return hipGetLastError();
}

}  // namespace gq
