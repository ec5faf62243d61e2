// GuidedQuant layer objective (Eq. "ours2", Section 3.2):
//   obj_row[j] = delta_j^T H[k(j)] delta_j,  delta_j = W[j,:] - What[j,:],  obj[k] = sum_{j in J_k} obj_row[j].
//
// The contraction Y = Delta_k H_k (2 d_out d_in^2 flop) runs on the bf16 matrix cores at
// fp32-grade accuracy by splitting both operands into two bf16 terms, x = hi + lo with
// hi = bf16(x), lo = bf16(x - hi) (together 16 mantissa bits), and summing the three products
// hi*hi + hi*lo + lo*hi in fp32 accumulators (the dropped lo*lo term is below 2^-16 relative).
// Only the upper triangle of H is read.  In tile terms
//   delta^T H delta = 2 * sum_{ta < tb} delta_a^T H[ta,tb] delta_b + sum_tb delta_b^T H[tb,tb] delta_b,
// so a workgroup that owns 256 channels (rows j) and a pair of 128-wide column tiles
// (tb = 2P, 2P+1) contracts over a < (2P+2)*128; the accumulators of a column tile are doubled
// once the contraction reaches that tile's diagonal block (everything before it lies strictly
// above the diagonal), the first tile of the pair reads zeros past its diagonal block, and the
// workgroup finishes with partial[P][j] = sum_b Y[j,b] * delta[j,b] in fp32.
//
// Kernels: (1) split delta into hi/lo bf16; (2) split H into hi/lo bf16, TRANSPOSED
// (Hs[k][b][a] = H[k][a][b] for a <= b, the diagonal 128-tiles completed to full squares), so
// that both MFMA operands run along the contraction index a; both are written in the order the
// MFMA kernel consumes them: one contiguous 4 KiB block per (128-row tile, 16 contraction
// elements), already in the swizzled LDS layout, so staging is a linear copy of whole cache
// lines; (3) the MFMA kernel; (4) a two-step reduction that adds the partials of a row in fixed
// order (fp32 obj_row) and the rows of a group in fp64 (obj).  Everything is deterministic.
// A call that does not want obj_row takes a cheaper way to obj, further down.
#include <type_traits>

#include "gq_internal.hpp"

namespace gq {
namespace {

constexpr int kTile = 128;            // rows of a staged tile (channels j, or columns b of H)
constexpr int kKS = 16;               // contraction elements per LDS stage (one MFMA deep)
constexpr int kRowBytes = kKS * 2;    // a staged tile row: two 16-byte chunks
constexpr int kTileBytes = kTile * kRowBytes;       // 4 KiB
constexpr int kStageTiles = 8;                      // {Dh, Dl} x 2 row blocks, {Hh, Hl} x 2 column tiles
constexpr int kStageBytes = kStageTiles * kTileBytes;   // 32 KiB
constexpr int kStages = 5;                          // ring depth: 160 KiB, all of a CU
constexpr int kLoadsPerStage = kTileBytes / 1024;   // 1 KiB direct loads per wave and stage (wave w fills tile w)
constexpr int kPairStages = 2 * kTile / kKS;        // stages per pair of 128-tiles along the contraction (16)
constexpr int kOrderP = 4, kOrderR = 8;             // workgroups are ordered in blocks of 4 tile pairs x 8 row blocks
constexpr int kTileElems = kTile * kKS;             // bf16 elements of one staged tile

// Element offset, inside a staged tile, of contraction element e (0..15) of row r (0..127): a row
// is two 16-byte chunks, and rows 8..15 of every 16 keep them swapped, so that the 16-byte
// fragment reads of 16 consecutive rows fall into 16 different bank groups.
__host__ __device__ inline int tile_pos(int r, int e) { return r * kKS + ((((e >> 3) ^ (r >> 3)) & 1) << 3) + (e & 7); }

// Staged tiles of delta: block (k, rb) holds channels k*m + rb*128 + r, r < 128 (zero past the
// end of the group), stage st the contraction elements 16 st .. 16 st + 15 (zero past d):
//   Dh/Dl[((k*n_rb + rb) * n_st + st) * kTileElems + tile_pos(r, e)].
// One workgroup turns 128 rows x 64 contraction elements (four stages) through LDS: a wave
// reads 256 contiguous bytes of a row of W and of What, and writes 1 KiB contiguous.
__global__ __launch_bounds__(256) void split_delta_kernel(const float* __restrict__ W, const float* __restrict__ What,
                                                          int64_t d_out, int64_t d, int64_t ld, int G, int n_rb,
                                                          int64_t n_st, unsigned short* __restrict__ Dh,
                                                          unsigned short* __restrict__ Dl) {
  __shared__ float tile[kTile][64 + 1];
  const int64_t blk = blockIdx.y;
  const int k = (int)(blk / n_rb), rb = (int)(blk % n_rb);
  const int64_t m = d_out / G;
  const int64_t j0 = (int64_t)k * m + (int64_t)rb * kTile, j_end = (int64_t)(k + 1) * m;
  const int64_t a0 = (int64_t)blockIdx.x * 64;
  const int t = threadIdx.x;
  // branch-free (clamped addresses, values selected afterwards) so that all 32 x 2 loads of a thread are in flight together
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const int idx = t + 256 * i;
    const int r = idx / 64, ac = idx % 64;
    const int64_t j = j0 + r, a = a0 + ac;
    const int64_t jc = j < j_end ? j : j_end - 1, acl = a < d ? a : d - 1;
    const float v = W[jc * ld + acl] - What[jc * ld + acl];
    tile[r][ac] = (j < j_end && a < d) ? v : 0.f;
  }
  __syncthreads();
  const int r = t / 2, c = t % 2;
#pragma unroll
  for (int i = 0; i < 4; ++i) {                             // stage i of the block
    u32x4 h4, l4;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      unsigned short h0, l0, h1, l1;
      split_bf16(tile[r][16 * i + 8 * c + e], h0, l0);
      split_bf16(tile[r][16 * i + 8 * c + e + 1], h1, l1);
      h4[e / 2] = (unsigned)h0 | ((unsigned)h1 << 16);
      l4[e / 2] = (unsigned)l0 | ((unsigned)l1 << 16);
    }
    const int64_t st = a0 / kKS + i;
    const int64_t off = (blk * n_st + st) * kTileElems + tile_pos(r, 8 * c);
    *reinterpret_cast<u32x4*>(Dh + off) = h4;
    *reinterpret_cast<u32x4*>(Dl + off) = l4;
  }
}

// Staged tiles of the transposed H: column tile tb holds columns b = 128 tb + r as its rows,
// stage st the contraction elements a = 16 st .. 16 st + 15, for st < 16 (tb / 2 + 1):
//   Hh/Hl[k][(tb * n_st + st) * kTileElems + tile_pos(r, e)] = hi/lo of H[k][a][b]  (a <= b),
// of H[k][b][a] below the diagonal of the diagonal 128-tile, 0 past d; an even tile tb also
// gets eight stages of zeros after its diagonal block.  One workgroup turns a
// block of 64 a x 128 b (four stages) through LDS: coalesced reads along b, 1 KiB contiguous
// writes per wave.
__global__ __launch_bounds__(256) void split_h_kernel(const float* __restrict__ H, int64_t d, int64_t ldp, int64_t n_st,
                                                      unsigned short* __restrict__ Hh,
                                                      unsigned short* __restrict__ Hl) {
  __shared__ float tile[64][kTile + 1];
  const int k = blockIdx.y;
  const float* Hk = H + (int64_t)k * d * d;
  unsigned short* Hhk = Hh + (int64_t)k * ldp * ldp;
  unsigned short* Hlk = Hl + (int64_t)k * ldp * ldp;
  // 128-tiles (ta, tb) with ta/2 <= tb/2: the tile below the diagonal of a pair (ta = tb + 1) is
  // written as zeros, the MFMA kernel runs both column tiles of a pair over the same range
  int ta, tb;
  {
    int pa, pb;
    tri_decode(blockIdx.x / 8, pa, pb);
    const int sub = (blockIdx.x / 2) % 4;
    ta = 2 * pa + (sub & 1);
    tb = 2 * pb + (sub >> 1);
  }
  const int64_t a0 = (int64_t)ta * kTile + 64 * (blockIdx.x % 2), b0 = (int64_t)tb * kTile;
  const int t = threadIdx.x;
  // branch-free inside (clamped addresses, values selected afterwards): all 32 loads of a thread in flight together
  if (ta <= tb) {                                           // uniform; the tile below a pair's diagonal is all zeros
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      const int idx = t + 256 * i;
      const int ar = idx / kTile, bc = idx % kTile;
      const int64_t a = a0 + ar, b = b0 + bc;
      const int64_t lo = a < b ? a : b, hi = a < b ? b : a;   // below the diagonal of a diagonal tile: the mirror image
      const int64_t lc = lo < d ? lo : d - 1, hc = hi < d ? hi : d - 1;
      const float v = Hk[lc * d + hc];
      tile[ar][bc] = (hi < d) ? v : 0.f;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 32; ++i) tile[(t + 256 * i) / kTile][(t + 256 * i) % kTile] = 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {                             // stage i of the block; thread: row t/2, chunk t%2
    const int r = t / 2, c = t % 2;
    u32x4 h4, l4;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      unsigned short h0, l0, h1, l1;
      split_bf16(tile[16 * i + 8 * c + e][r], h0, l0);
      split_bf16(tile[16 * i + 8 * c + e + 1][r], h1, l1);
      h4[e / 2] = (unsigned)h0 | ((unsigned)h1 << 16);
      l4[e / 2] = (unsigned)l0 | ((unsigned)l1 << 16);
    }
    const int64_t st = a0 / kKS + i;
    const int64_t off = ((int64_t)tb * n_st + st) * kTileElems + tile_pos(r, 8 * c);
    *reinterpret_cast<u32x4*>(Hhk + off) = h4;
    *reinterpret_cast<u32x4*>(Hlk + off) = l4;
  }
}

// Y tile [256 j][256 b] for one pair P of column tiles, on bf16 MFMA with split operands, then
// the row dot.  8 waves: wave (wm, wn) owns rows 64 wm .. 64 wm + 63 and column tile 2P + wn.
//
// Staging.  The eight operand tiles of a stage (128 rows x 16 contraction elements each, 4 KiB
// contiguous in the split arrays and already in LDS order) go from global memory straight into
// LDS (global_load_lds_dwordx4: wave w copies tile w with four 1 KiB loads), kStages - 1 stages
// ahead of their use, tracked by an explicit vmcnt wait and one workgroup barrier per stage.
__global__ __launch_bounds__(512) void objective_mfma_kernel(const unsigned short* __restrict__ Dh,
                                                             const unsigned short* __restrict__ Dl,
                                                             const unsigned short* __restrict__ Hh,
                                                             const unsigned short* __restrict__ Hl,
                                                             const float* __restrict__ W, const float* __restrict__ What,
                                                             int64_t d_out, int64_t d, int64_t ld, int64_t ldp, int G,
                                                             int n_pairs, int n_rb2, int chunk, int n_slots,
                                                             int deal, float* __restrict__ partial) {
  __shared__ __attribute__((aligned(1024))) char smem[kStages * kStageBytes];
  // (the row-sum exchange at the end reuses the staging memory, after a barrier)

  // Work order.  Workgroup ids are dealt round-robin to the 8 XCDs (each with its own L2), so
  // the id is first remapped to give every XCD one contiguous stretch of the logical order.
  // That order walks, per group, blocks of kOrderP tile pairs x kOrderR row blocks (heavy pairs
  // first): the workgroups resident on an XCD then share both their H tiles and their delta
  // tiles through its L2.
  // The contraction of pair P (P + 1 pair blocks of 16 stages) is cut into slots of at most
  // `chunk` pair blocks: workgroups of similar length keep pace with their neighbours (and keep
  // sharing tiles), and small problems still give every CU several workgroups; slot 0 is the
  // last (diagonal) part of the heaviest pair.
  int k, sl, rb2;
  {
    constexpr int kXcd = 8, kDeal = kOrderP * kOrderR;      // 32: what the 32 CUs of an XCD run at a time
    const int64_t total = gridDim.x, id = blockIdx.x;
    const int64_t x = id % kXcd, idx = id / kXcd, q = total / kXcd, r = total % kXcd;
    // Large grids (`deal`): stretches of 32 consecutive workgroups of the logical order go to the XCDs in
    // turn; the order is heavy first, so every XCD gets the same share of the work and runs one stretch
    // (one block of pairs x row blocks) at a time.  Small grids: one contiguous stretch per XCD.
    const int64_t dealt = total / (kXcd * kDeal) * (kXcd * kDeal);
    const int64_t logical = !deal ? x * q + (x < r ? x : r) + idx
                                  : (id < dealt ? ((idx / kDeal) * kXcd + x) * kDeal + idx % kDeal : id);
    const int64_t per_group = (int64_t)n_slots * n_rb2;
    k = (int)(logical / per_group);
    int64_t rem = logical - (int64_t)k * per_group;
    // bands of kOrderP slots; the first band holds the remainder
    const int n_bands = (n_slots + kOrderP - 1) / kOrderP;
    const int first_w = n_slots - (n_bands - 1) * kOrderP;
    int band, pw;
    if (rem < (int64_t)first_w * n_rb2) {
      band = 0;
      pw = first_w;
    } else {
      rem -= (int64_t)first_w * n_rb2;
      band = 1 + (int)(rem / ((int64_t)kOrderP * n_rb2));
      rem = rem % ((int64_t)kOrderP * n_rb2);
      pw = kOrderP;
    }
    const int s_lo = band == 0 ? 0 : first_w + (band - 1) * kOrderP;   // first slot of the band
    const int rblk = (int)(rem / ((int64_t)pw * kOrderR));
    const int off = (int)(rem % ((int64_t)pw * kOrderR));
    const int rw = (n_rb2 - rblk * kOrderR) < kOrderR ? (n_rb2 - rblk * kOrderR) : kOrderR;
    sl = s_lo + off / rw;
    rb2 = rblk * kOrderR + off % rw;
  }
  // slot -> (pair, part): pairs from the heaviest down, the parts of a pair from its diagonal end down
  int P = n_pairs - 1, part;
  {
    int rem = sl;
    while (rem >= (P + chunk) / chunk) {                   // number of parts of pair P = ceil((P + 1) / chunk)
      rem -= (P + chunk) / chunk;
      --P;
    }
    part = (P + chunk) / chunk - 1 - rem;
  }
  const int pb_begin = part * chunk;                                        // first pair block of this part
  const bool last_part = (part + 1) * chunk >= P + 1;                       // it ends with the diagonal pair block
  const int64_t m = d_out / G;
  const int64_t j0 = (int64_t)k * m + (int64_t)rb2 * 2 * kTile;   // first channel of this block
  const int64_t j_end = (int64_t)(k + 1) * m;                     // rows >= j_end belong to another group
  const int64_t b0 = (int64_t)P * 2 * kTile;

  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wm = wave / 2, wn = wave % 2;

  // ---- this wave's share of the staging: tile `wave` of every stage, 16 bytes per lane -------
  const int64_t n_st = ldp / kKS;
  const unsigned short* gp[kLoadsPerStage];
  {
    const int which = (wave % 4) / 2;                       // row block / column tile of the pair
    const unsigned short* src =
        wave < 4 ? (wave % 2 == 0 ? Dh : Dl) + (((int64_t)k * n_rb2 + rb2) * 2 + which) * n_st * kTileElems
                 : (wave % 2 == 0 ? Hh : Hl) + (int64_t)k * ldp * ldp + ((int64_t)P * 2 + which) * n_st * kTileElems;
#pragma unroll
    for (int i = 0; i < kLoadsPerStage; ++i) gp[i] = src + (int64_t)pb_begin * kPairStages * kTileElems + i * 512 + lane * 8;
  }
  const unsigned smem_base = (unsigned)(uintptr_t)(lds_char_ptr)smem;
  // Requests the next stage of the contraction into ring slot `slot`; `advance` is false once
  // the last stage has been requested (later calls fetch it again into a free slot, which
  // keeps the number of loads in flight, and with it the vmcnt arithmetic, constant).
  auto issue = [&](int slot, bool advance) {
    const int step_elems = advance ? kTileElems : 0;
#pragma unroll
    for (int i = 0; i < kLoadsPerStage; ++i) {
      dma16(gp[i], smem_base + slot * kStageBytes + wave * kTileBytes + i * 1024);
      gp[i] += step_elems;
    }
  };

  // ---- fragment addresses: row l % 32 of a 32-row block, chunk l / 32 -----------------------
  const int lrow = lane % 32;
  const int frag_off = lrow * kRowBytes + (((lane / 32) ^ ((lrow >> 3) & 1)) * 16);
  const int a_off = (wm / 2) * 2 * kTileBytes + (wm % 2) * 64 * kRowBytes + frag_off;   // Dh tile; Dl follows it
  const int b_off = (4 + 2 * wn) * kTileBytes + frag_off;                               // Hh tile; Hl follows it
  auto frag = [&](int slot, int off) -> bf16x8 {
    const u32x4 v = *reinterpret_cast<const u32x4*>(&smem[slot * kStageBytes + off]);
    return __builtin_bit_cast(bf16x8, v);
  };

  f32x16 acc[2][4];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;

  // Fragments of one stage: rows of delta (hi, lo) and of the transposed H tile (hi, lo).
  struct Frags {
    bf16x8 ah[2], al[2], bh[4], bl[4];
  };
  // The three products of the two 32 x 32 blocks of column block y, interleaved so that
  // consecutive MFMAs never update the same accumulator.
  auto mma = [&](const Frags& f, int y) {
    acc[0][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.al[0], f.bh[y], acc[0][y], 0, 0, 0);
    acc[1][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.al[1], f.bh[y], acc[1][y], 0, 0, 0);
    acc[0][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[0], f.bl[y], acc[0][y], 0, 0, 0);
    acc[1][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[1], f.bl[y], acc[1][y], 0, 0, 0);
    acc[0][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[0], f.bh[y], acc[0][y], 0, 0, 0);
    acc[1][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[1], f.bh[y], acc[1][y], 0, 0, 0);
  };
  auto read_a = [&](Frags& f, int slot, int x) {
    f.ah[x] = frag(slot, a_off + x * 32 * kRowBytes);
    f.al[x] = frag(slot, a_off + kTileBytes + x * 32 * kRowBytes);
  };
  auto read_b = [&](Frags& f, int slot, int y) {
    f.bh[y] = frag(slot, b_off + y * 32 * kRowBytes);
    f.bl[y] = frag(slot, b_off + kTileBytes + y * 32 * kRowBytes);
  };
  auto read_all = [&](Frags& f, int slot) {
#pragma unroll
    for (int x = 0; x < 2; ++x) read_a(f, slot, x);
#pragma unroll
    for (int y = 0; y < 4; ++y) read_b(f, slot, y);
  };
  auto twice = [&]() {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y) acc[x][y] *= 2.f;
  };

  // Every kernel argument the epilogue needs is pulled into registers here: a scalar load left
  // pending across the loops would turn the partial LDS-counter waits inside them into full ones.
  asm volatile("" ::"s"(partial), "s"(W), "s"(What), "s"(ld), "s"(d), "s"(d_out), "s"(j_end));

  const int stages = (last_part ? P + 1 : (part + 1) * chunk) * kPairStages;   // end of this part; it has >= 16 stages
#pragma unroll
  for (int t = 0; t < kStages - 1; ++t) issue(t, true);
  int slot_next = 1, slot_fill = kStages - 1;               // ring slots of stage it + 1 and of stage it - 1

  // One step: the MFMAs of stage `it` run on fragments read during the previous step, while
  // the fragments of stage it + 1 are read and stage it + kStages - 1 is requested.  The step
  // is branch-free (past the end it reads a stale slot and requests the last stage again).
  // All eight waves leave the barrier together, so every wave first queues MFMAs and then
  // slips its loads and LDS reads in between groups of six MFMAs, in the order in which the
  // next step consumes them: the matrix pipe has work while the LDS serves the reads, and at
  // most 12 LDS reads are in flight (the counter that tracks them has 4 bits).
  auto fence = [&]() { __builtin_amdgcn_sched_barrier(0); };
  auto step = [&](const Frags& cur, Frags& nxt, int it) {
    wait_vmcnt<(kStages - 3) * kLoadsPerStage>();   // this wave's loads of stage it + 1 have landed
    // everyone's have; and everyone has issued the MFMAs of stage it - 1, so its slot is free
    __builtin_amdgcn_s_barrier();
    fence();
    mma(cur, 0);
    fence();
    issue(slot_fill, it + kStages < stages);
    read_a(nxt, slot_next, 0);
    read_a(nxt, slot_next, 1);
    fence();
    mma(cur, 1);
    fence();
    read_b(nxt, slot_next, 0);
    read_b(nxt, slot_next, 1);
    fence();
    mma(cur, 2);
    fence();
    read_b(nxt, slot_next, 2);
    read_b(nxt, slot_next, 3);
    fence();
    mma(cur, 3);
    fence();
    slot_fill = slot_fill + 1 == kStages ? 0 : slot_fill + 1;
    slot_next = slot_next + 1 == kStages ? 0 : slot_next + 1;
  };

  Frags f0, f1;
  wait_vmcnt<(kStages - 2) * kLoadsPerStage>();
  __builtin_amdgcn_s_barrier();
  read_all(f0, 0);
  int it = pb_begin * kPairStages;
  const int diag0 = P * kPairStages, diag1 = diag0 + kPairStages / 2;
  const int upper_end = last_part ? diag0 : stages;
  for (; it < upper_end; it += 2) {      // strictly above the diagonal for both column tiles
    step(f0, f1, it);
    step(f1, f0, it + 1);
  }
  // what came before counts twice (its mirror image is never visited)
  if (!last_part || (wn == 0 && P > 0)) twice();
  if (last_part) {
    for (; it < diag1; it += 2) {        // diagonal block of the first tile, still above the second's
      step(f0, f1, it);
      step(f1, f0, it + 1);
    }
    if (wn == 1) twice();
    for (; it < stages; it += 2) {       // diagonal block of the second tile (zeros for the first)
      step(f0, f1, it);
      step(f1, f0, it + 1);
    }
  }
  wait_vmcnt<0>();   // the repeated requests of the last stage
  __syncthreads();   // the ring is idle: `red` may reuse it

  // Row dot with delta[j, b] (fp32).  Register r of lane l holds row 8*(r/4)+4*(l/32)+(r%4),
  // column l%32 of a 32 x 32 block.  Branch-free: addresses are clamped into the matrix, which
  // is harmless because Y is exactly 0 in columns b >= d (the padded rows of the transposed H
  // are zeros) and rows j >= j_end are dropped at the final store.
  float v[2][16];
  {
    const int64_t bl = b0 + wn * kTile + lane % 32;
    int64_t bcol[4];
#pragma unroll
    for (int y = 0; y < 4; ++y) bcol[y] = (bl + 32 * y) < d ? (bl + 32 * y) : d - 1;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        int64_t j = j0 + wm * 64 + x * 32 + 8 * (r / 4) + 4 * (lane / 32) + (r % 4);
        j = j < j_end ? j : j_end - 1;
        float t = 0.f;
#pragma unroll
        for (int y = 0; y < 4; ++y) t += acc[x][y][r] * (W[j * ld + bcol[y]] - What[j * ld + bcol[y]]);
        v[x][r] = t;
      }
  }
  // Sum over the 32 lanes of each half-wave, for all 32 rows at once: every lane parks its 32
  // values as a column of a 32 x 32 array (pitch 33 floats), then adds up one row of it.
  constexpr int kPitch = 33;
  float* park = reinterpret_cast<float*>(&smem[0]) + (wave * 2 + lane / 32) * 32 * kPitch;
  float (*red)[2 * kTile] = reinterpret_cast<float (*)[2 * kTile]>(&smem[8 * 2 * 32 * kPitch * sizeof(float)]);
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int r = 0; r < 16; ++r) park[(x * 16 + r) * kPitch + lane % 32] = v[x][r];
  float sum = 0.f;   // no barrier: a wave reads back only what it wrote itself, and its LDS accesses stay in order
#pragma unroll
  for (int c = 0; c < 32; ++c) sum += park[(lane % 32) * kPitch + c];
  {
    const int xr = lane % 32;   // this lane now owns block x = xr / 16, register r = xr % 16 of its half-wave
    red[wn][wm * 64 + (xr / 16) * 32 + 8 * ((xr % 16) / 4) + 4 * (lane / 32) + (xr % 4)] = sum;
  }
  __syncthreads();
  if (tid < 2 * kTile) {
    const int64_t j = j0 + tid;
    if (j < j_end) partial[(int64_t)sl * d_out + j] = red[0][tid] + red[1][tid];
  }
}

// obj_row[j] = sum_tb partial[tb][j] (fixed order) for 256 rows per workgroup, and the fp64 sum
// of those rows (fixed tree) into block_sum[k][block].
__global__ __launch_bounds__(256) void objective_rows_kernel(const float* __restrict__ partial, int64_t d_out, int G,
                                                             int n_tb, float* __restrict__ obj_row,
                                                             double* __restrict__ block_sum) {
  __shared__ double red[256];
  const int k = blockIdx.y;
  const int64_t m = d_out / G;
  const int64_t jj = (int64_t)blockIdx.x * 256 + threadIdx.x;
  double acc = 0.0;
  if (jj < m) {
    const int64_t j = (int64_t)k * m + jj;
    // the partials are added in the order tb = 0, 1, ...; eight loads at a time are in flight (a loop of one load
    // and one add per turn waits for every load in turn)
    float v = 0.f;
    int tb = 0;
    for (; tb + 8 <= n_tb; tb += 8) {
      float p[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) p[u] = partial[(int64_t)(tb + u) * d_out + j];
#pragma unroll
      for (int u = 0; u < 8; ++u) v += p[u];
    }
    for (; tb < n_tb; ++tb) v += partial[(int64_t)tb * d_out + j];
    if (obj_row) obj_row[j] = v;
    acc = (double)v;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) block_sum[(int64_t)k * gridDim.x + blockIdx.x] = red[0];
}

// obj[k] = sum of the group's block sums, in block order.
__global__ void objective_groups_kernel(const double* __restrict__ block_sum, int n_blocks, double* __restrict__ obj) {
  const int k = blockIdx.x;
  if (threadIdx.x != 0) return;
  double acc = 0.0;
  for (int b = 0; b < n_blocks; ++b) acc += block_sum[(int64_t)k * n_blocks + b];
  obj[k] = acc;
}

// ---- without the per-channel terms ---------------------------------------------------------------
// obj[k] = sum_{a,b} H[k][a][b] M[a][b],  M = Delta_k^T Delta_k  (d_in x d_in, contraction over the group's channels):
// the same number of products as Delta_k H_k on the upper triangle, but H is an operand of the last multiplication only:
// it is read once, as it is, instead of being split and staged, and every tile of M takes the same time.  M never
// leaves the chip: a workgroup forms 256 x 256 of it (one pair of 256-blocks on or above the diagonal) on the bf16
// matrix cores from delta split in two terms, hi*hi + hi*lo + lo*hi, and sums H[a][b] * M[a][b] in fp64, twice, above
// the diagonal.  The diagonal of M, sums of squares in which neither the dropped lo*lo nor the rounding of a long fp32 sum
// on the matrix cores would average out (measured: obj off by 1e-8 per 16 channels), comes from the split, in fp64.
// The sum is linear in M, so the channels of a tile may be cut into parts: each part adds its own.
// Measured at W[4096,4096], G = 4: 233 us a call, 311 us by the kernels above; W[512,256], G = 2: 26 and 45 us; W[7,4000],
// G = 7: 73 and 187 us.  The error against 64 bits is smaller too (3e-8 and 6e-7 of obj at the first).
// What bounds it: 3 * d_out d_in^2 multiply-adds, 190 us of the 233, 1.15 PFLOP/s where this card's bf16 library product
// reaches 1.29; the split moves 192 MB in 47 us.

// Staged tiles of delta, contraction = channels: block (k, cb) holds coordinates cb*128 + r, r < 128 (zero past d), stage
// st the channels 16 st .. 16 st + 15 of the group (zero past its end):
//   Dh/Dl[((k*n_cb + cb) * n_st + st) * kTileElems + tile_pos(r, e)].
// One workgroup turns 64 channels x 64 coordinates (four stages) through LDS, and leaves each coordinate's sum of squares
// in squares[(k * j_blocks + block of channels) * ldp + a] and the bits of its largest |delta| in largest[k][..] (an
// infinity or a NaN counts as larger than any number).
__global__ __launch_bounds__(256) void split_delta_t_kernel(const float* __restrict__ W, const float* __restrict__ What,
                                                            int64_t d_out, int64_t d, int64_t ld, int G, int n_cb,
                                                            int64_t n_st, unsigned short* __restrict__ Dh,
                                                            unsigned short* __restrict__ Dl,
                                                            unsigned* __restrict__ largest,
                                                            double* __restrict__ squares) {
  __shared__ float tile[64][64 + 1];
  __shared__ double sq[4][64];
  __shared__ unsigned wave_largest[4];
  const int64_t j_blocks = n_st / 4, k = blockIdx.x / j_blocks;
  const int64_t m = d_out / G;
  const int64_t j0 = blockIdx.x % j_blocks * 64, a0 = (int64_t)blockIdx.y * 64;   // channels of the group, coordinates
  const int tx = threadIdx.x % 64, ty = threadIdx.x / 64;
  // branch-free (clamped addresses, values selected afterwards) so that all loads of a thread are in flight together
  unsigned most = 0;
  double sum = 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int64_t jj = j0 + ty + 4 * u, a = a0 + tx;
    const int64_t j = k * m + (jj < m ? jj : m - 1), ac = a < d ? a : d - 1;
    const float v = W[j * ld + ac] - What[j * ld + ac];
    const float kept = (jj < m && a < d) ? v : 0.f;
    const unsigned bits = __builtin_bit_cast(unsigned, kept) & 0x7fffffffu;
    most = bits > most ? bits : most;
    sum += (double)kept * (double)kept;
    tile[ty + 4 * u][tx] = kept;
  }
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) {
    const unsigned other = __shfl_xor(most, w, kWave);
    most = other > most ? other : most;
  }
  if (tx == 0) wave_largest[ty] = most;
  sq[ty][tx] = sum;
  __syncthreads();
  if (ty == 1) squares[(k * j_blocks + j0 / 64) * n_cb * kTile + a0 + tx] = (sq[0][tx] + sq[1][tx]) + (sq[2][tx] + sq[3][tx]);
  if (threadIdx.x == 0) {
    most = wave_largest[0];
    for (int w = 1; w < 4; ++w) most = wave_largest[w] > most ? wave_largest[w] : most;
    largest[(k * j_blocks + j0 / 64) * gridDim.y + blockIdx.y] = most;
  }
  const int r = (int)(a0 % kTile) + tx;                       // this thread: coordinate tx, stage ty of the block's four
  const int64_t off = ((k * n_cb + a0 / kTile) * n_st + j0 / kKS + ty) * kTileElems;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    u32x4 h4, l4;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      unsigned short h0, l0, h1, l1;
      split_bf16(tile[16 * ty + 8 * c + e][tx], h0, l0);
      split_bf16(tile[16 * ty + 8 * c + e + 1][tx], h1, l1);
      h4[e / 2] = (unsigned)h0 | ((unsigned)h1 << 16);
      l4[e / 2] = (unsigned)l0 | ((unsigned)l1 << 16);
    }
    *reinterpret_cast<u32x4*>(Dh + off + tile_pos(r, 8 * c)) = h4;
    *reinterpret_cast<u32x4*>(Dl + off + tile_pos(r, 8 * c)) = l4;
  }
}

// Products of two deltas have to stay within fp32: where the largest |delta| of a group is outside [2^-40, 2^40) its terms
// are brought to 1 .. 2 by a power of two here, which the sum takes out again.  Otherwise (practically always) there is
// nothing to do: 32 workgroups per group read the maxima and end.
__global__ __launch_bounds__(256) void scale_delta_kernel(unsigned short* __restrict__ Dh, unsigned short* __restrict__ Dl,
                                                          const unsigned* __restrict__ largest, int64_t n_largest,
                                                          int64_t group_elems, int* __restrict__ exponent) {
  __shared__ unsigned red[256];
  const int64_t k = blockIdx.x / 32, part = blockIdx.x % 32;
  unsigned most = 0;
  for (int64_t i = threadIdx.x; i < n_largest; i += 256) {
    const unsigned v = largest[k * n_largest + i];
    most = v > most ? v : most;
  }
  red[threadIdx.x] = most;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = red[threadIdx.x] > red[threadIdx.x + w] ? red[threadIdx.x] : red[threadIdx.x + w];
    __syncthreads();
  }
  most = red[0];
  int e = (int)(most >> 23) - 127;                            // -127 for denormal numbers and 0
  if (most == 0 || most >= 0x7f800000u || (e >= -40 && e < 40)) e = 0;
  if (part == 0 && threadIdx.x == 0) exponent[k] = e;
  if (e == 0) return;
  for (int64_t i = part * 256 + threadIdx.x; i < group_elems; i += 32 * 256) {
    unsigned short* const terms[2] = {Dh + k * group_elems + i, Dl + k * group_elems + i};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float v = ldexpf(__builtin_bit_cast(float, (unsigned)*terms[t] << 16), -e);
      *terms[t] = (unsigned short)(__builtin_bit_cast(unsigned, v) >> 16);
    }
  }
}

// The tiles of all groups, n_tri per group, are dealt out to kUnits workgroups, one per compute unit: whole tiles while
// there is one for each (the workgroups of an XCD then walk neighbouring tiles side by side and share their panels in
// L2), and of the rest every workgroup takes the same number of quads (four stages, 64 channels), across tiles.
// Measured at W[4096,4096], G = 4, 544 tiles, 2.1 per workgroup: one workgroup per tile 263 us, so 190 us.
constexpr int kUnits = 256;
struct Deal {
  int64_t rounds, quads_left;
  int quads;                                                  // per tile
};
__host__ __device__ inline Deal deal(int64_t tiles, int64_t n_st) {
  return {tiles / kUnits, tiles % kUnits * (n_st / 4), (int)(n_st / 4)};
}
// Does workgroup w take part of a tile t, t0 <= t < t1?
__device__ inline bool deal_meets(const Deal& D, int w, int64_t t0, int64_t t1) {
  int64_t t = t0 > w ? w + (t0 - w + kUnits - 1) / kUnits * kUnits : w;
  if (t < t1 && t < D.rounds * kUnits) return true;
  t = D.rounds * kUnits;
  const int64_t q0 = D.quads_left * w / kUnits, q1 = D.quads_left * (w + 1) / kUnits;
  return q0 < q1 && t + q0 / D.quads < t1 && t + (q1 - 1) / D.quads >= t0;
}

// One tile (pa, pb) of M after the other, each over some of its stages, and its sum against H.  Staging, fragments and the
// order of the inner loop are those of objective_mfma_kernel: 8 waves, wave (wm, wn) owns rows 64 wm .. + 63 and columns
// 128 wn .. + 127.  The first stages of the next tile are requested before H is read.
__global__ __launch_bounds__(512) void objective_gram_kernel(const unsigned short* __restrict__ Dh,
                                                             const unsigned short* __restrict__ Dl,
                                                             const float* __restrict__ H, int64_t d, int G, int n_pairs,
                                                             int64_t n_st, const double* __restrict__ squares,
                                                             const int* __restrict__ exponent,
                                                             double* __restrict__ partial) {
  __shared__ __attribute__((aligned(1024))) char smem[kStages * kStageBytes];
  const int unit = (int)(blockIdx.x % 8) * (kUnits / 8) + (int)(blockIdx.x / 8);   // neighbours on one XCD
  const int64_t n_tri = tri_count(n_pairs);
  const Deal D = deal(n_tri * G, n_st);
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wm = wave / 2, wn = wave % 2;

  struct Piece {
    int k, pa, pb, s0, count;                                 // stages s0 .. s0 + count - 1 of tile (pa, pb) of group k
  };
  int64_t round = 0, quad = D.quads_left * unit / kUnits;
  const int64_t quad_end = D.quads_left * (unit + 1) / kUnits;
  auto next_piece = [&](Piece& p) -> bool {
    unsigned tile;
    if (round < D.rounds) {
      tile = (unsigned)(round++ * kUnits + unit);
      p.s0 = 0;
      p.count = (int)n_st;
    } else if (quad < quad_end) {
      tile = (unsigned)(D.rounds * kUnits + quad / D.quads);
      const int q0 = (int)(quad % D.quads), q1 = quad_end - quad < D.quads - q0 ? q0 + (int)(quad_end - quad) : D.quads;
      p.s0 = 4 * q0;
      p.count = 4 * (q1 - q0);
      quad += q1 - q0;
    } else {
      return false;
    }
    p.k = __builtin_amdgcn_readfirstlane((int)(tile / (unsigned)n_tri));
    int pa, pb;
    tri_decode(tile % (unsigned)n_tri, pa, pb);
    p.pa = __builtin_amdgcn_readfirstlane(pa);
    p.pb = __builtin_amdgcn_readfirstlane(pb);
    return true;
  };

  const unsigned short* gp[kLoadsPerStage];
  const unsigned smem_base = (unsigned)(uintptr_t)(lds_char_ptr)smem;
  auto issue = [&](int slot, bool advance) {
    const int step_elems = advance ? kTileElems : 0;
#pragma unroll
    for (int i = 0; i < kLoadsPerStage; ++i) {
      dma16(gp[i], smem_base + slot * kStageBytes + wave * kTileBytes + i * 1024);
      gp[i] += step_elems;
    }
  };
  const int lrow = lane % 32;
  const int frag_off = lrow * kRowBytes + (((lane / 32) ^ ((lrow >> 3) & 1)) * 16);
  const int a_off = (wm / 2) * 2 * kTileBytes + (wm % 2) * 64 * kRowBytes + frag_off;
  const int b_off = (4 + 2 * wn) * kTileBytes + frag_off;
  auto frag = [&](int slot, int off) -> bf16x8 {
    const u32x4 v = *reinterpret_cast<const u32x4*>(&smem[slot * kStageBytes + off]);
    return __builtin_bit_cast(bf16x8, v);
  };
  f32x16 acc[2][4];
  struct Frags {
    bf16x8 ah[2], al[2], bh[4], bl[4];
  };
  auto mma = [&](const Frags& f, int y) {
    acc[0][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.al[0], f.bh[y], acc[0][y], 0, 0, 0);
    acc[1][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.al[1], f.bh[y], acc[1][y], 0, 0, 0);
    acc[0][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[0], f.bl[y], acc[0][y], 0, 0, 0);
    acc[1][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[1], f.bl[y], acc[1][y], 0, 0, 0);
    acc[0][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[0], f.bh[y], acc[0][y], 0, 0, 0);
    acc[1][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[1], f.bh[y], acc[1][y], 0, 0, 0);
  };
  auto read_a = [&](Frags& f, int slot, int x) {
    f.ah[x] = frag(slot, a_off + x * 32 * kRowBytes);
    f.al[x] = frag(slot, a_off + kTileBytes + x * 32 * kRowBytes);
  };
  auto read_b = [&](Frags& f, int slot, int y) {
    f.bh[y] = frag(slot, b_off + y * 32 * kRowBytes);
    f.bl[y] = frag(slot, b_off + kTileBytes + y * 32 * kRowBytes);
  };
  asm volatile("" ::"s"(partial), "s"(H), "s"(d), "s"(squares), "s"(exponent));   // no scalar load pending across the loop

  int slot_next, slot_fill;
  auto request = [&](const Piece& p) {                          // its first stages (the last one again if there are fewer)
    const int cb = 2 * (wave < 4 ? p.pa : p.pb) + (wave % 4) / 2;
    const unsigned short* src = (wave % 2 == 0 ? Dh : Dl) + (((int64_t)p.k * n_pairs * 2 + cb) * n_st + p.s0) * kTileElems;
#pragma unroll
    for (int i = 0; i < kLoadsPerStage; ++i) gp[i] = src + i * 512 + lane * 8;
#pragma unroll
    for (int t = 0; t < kStages - 1; ++t) issue(t, t + 1 < p.count);
  };
  auto fence = [&]() { __builtin_amdgcn_sched_barrier(0); };
  auto step = [&](const Frags& cur, Frags& nxt, int it, int count) {
    wait_vmcnt<(kStages - 3) * kLoadsPerStage>();
    __builtin_amdgcn_s_barrier();
    fence();
    mma(cur, 0);
    fence();
    issue(slot_fill, it + kStages < count);
    read_a(nxt, slot_next, 0);
    read_a(nxt, slot_next, 1);
    fence();
    mma(cur, 1);
    fence();
    read_b(nxt, slot_next, 0);
    read_b(nxt, slot_next, 1);
    fence();
    mma(cur, 2);
    fence();
    read_b(nxt, slot_next, 2);
    read_b(nxt, slot_next, 3);
    fence();
    mma(cur, 3);
    fence();
    slot_fill = slot_fill + 1 == kStages ? 0 : slot_fill + 1;
    slot_next = slot_next + 1 == kStages ? 0 : slot_next + 1;
  };
  Piece p, next;
  if (!next_piece(p)) return;                                 // uniform: fewer quads than workgroups
  request(p);
  double sum = 0.0;
  for (bool more = true; more; p = next) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
    slot_next = 1;
    slot_fill = kStages - 1;
    Frags f0, f1;
    wait_vmcnt<(kStages - 2) * kLoadsPerStage>();
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int x = 0; x < 2; ++x) read_a(f0, 0, x);
#pragma unroll
    for (int y = 0; y < 4; ++y) read_b(f0, 0, y);
    for (int it = 0; it < p.count; it += 2) {
      step(f0, f1, it, p.count);
      step(f1, f0, it + 1, p.count);
    }
    wait_vmcnt<0>();
    __syncthreads();                                          // the ring is idle
    more = next_piece(next);
    if (more) request(next);                                  // uniform

    // Register r of lane l holds row 8*(r/4)+4*(l/32)+(r%4), column l%32 of a 32 x 32 block.  H is read through a buffer
    // over the rows of this tile (256 rows of 4 d bytes: below 2^32): rows past d, and lanes whose column is past d, read 0.
    // What lies below the diagonal may hold anything: it is dropped, not multiplied by 0.
    const int64_t row0 = (int64_t)p.pa * 2 * kTile, rows = d - row0 < 2 * kTile ? d - row0 : 2 * kTile;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(H + (int64_t)p.k * d * d + row0 * d), 0,
                                                        (int)(unsigned)(rows * d * 4), 0x00020000);
    const unsigned pitch = (unsigned)d * 4u;
    const int la = wm * 64 + 4 * (lane / 32), lb = wn * kTile + lane % 32;   // within the tile
    double tile_sum = 0.0;
    const int last_b = lb + (p.pa == p.pb ? 0 : 2 * kTile);         // entry (ra, cb) is above the diagonal if ra < cb here
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int64_t b = (int64_t)p.pb * 2 * kTile + lb + 32 * y;
      const unsigned off = b < d ? (unsigned)la * pitch + (unsigned)b * 4u : 0xC0000000u;
      float h[2][16];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          h[x][r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                  rsrc, (int)(off + (unsigned)(32 * x + 8 * (r / 4) + r % 4) * pitch), 0, 0));
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float above = la + 32 * x + 8 * (r / 4) + r % 4 < last_b + 32 * y ? h[x][r] : 0.f;
          tile_sum = __builtin_fma((double)acc[x][y][r], (double)above, tile_sum);
        }
      asm volatile("" : "+v"(tile_sum));                      // 32 entries at a time: the sum is not put off
      __builtin_amdgcn_sched_barrier(0);
    }
    sum += tile_sum + tile_sum;                                 // H[a][b] and its mirror image
    if (p.pa == p.pb && tid < rows) {
      const int64_t ldp = (int64_t)n_pairs * 2 * kTile, b0 = p.s0 / 4, b1 = b0 + p.count / 4;
      const double* sq = squares + ((int64_t)p.k * (n_st / 4) + b0) * ldp + row0 + tid;
      double t = 0.0;
      for (int64_t i = b0; i < b1; ++i, sq += ldp) t += *sq;
      sum += ldexp(t, -2 * exponent[p.k]) * (double)H[((int64_t)p.k * d + row0 + tid) * d + row0 + tid];
    }

    if (!more || next.k != p.k) {                             // uniform
#pragma unroll
      for (int w = 32; w > 0; w >>= 1) sum += __shfl_xor(sum, w, kWave);
      double* red = reinterpret_cast<double*>(smem + (kStages - 1) * kStageBytes);   // the slot that is not requested yet
      if (lane == 0) red[wave] = sum;
      __syncthreads();
      if (tid == 0) {
        double t = 0.0;
        for (int w = 0; w < 8; ++w) t += red[w];
        partial[(int64_t)p.k * kUnits + unit] = t;
      }
      __syncthreads();
      wait_vmcnt<0>();                                        // the store: what counts requests counts nothing else
      sum = 0.0;
    }
  }
}

// obj[k] = the sum of the workgroups' partial sums, those that met the group, in a fixed tree.
__global__ __launch_bounds__(kUnits) void objective_sum_kernel(const double* __restrict__ partial, int64_t n_tri, int64_t n_st,
                                                               const int* __restrict__ exponent, double* __restrict__ obj) {
  __shared__ double red[kUnits];
  const int64_t k = blockIdx.x;
  const int w = threadIdx.x;
  red[w] = deal_meets(deal(n_tri * gridDim.x, n_st), w, k * n_tri, (k + 1) * n_tri) ? partial[k * kUnits + w] : 0.0;
  __syncthreads();
  for (int half = kUnits / 2; half > 0; half >>= 1) {
    if (w < half) red[w] += red[w + half];
    __syncthreads();
  }
  if (w == 0) obj[k] = ldexp(red[0], 2 * exponent[k]);
}

struct GramLayout {
  int64_t n_pairs, n_st;
  int64_t n_largest;                                          // maxima per group
  size_t delta_bytes, partial_bytes, largest_bytes, exponent_bytes, squares_bytes;   // delta_bytes: one of the hi/lo arrays
};
GramLayout make_gram_layout(int64_t d_out, int64_t d_in, int G) {
  GramLayout L;
  L.n_pairs = (d_in + 2 * kTile - 1) / (2 * kTile);
  L.n_st = (d_out / G + 63) / 64 * 4;
  L.delta_bytes = ((size_t)((int64_t)G * L.n_pairs * 2 * L.n_st * kTileElems) * 2 + 255) / 256 * 256;
  L.partial_bytes = ((size_t)kUnits * (size_t)G * sizeof(double) + 255) / 256 * 256;
  L.n_largest = L.n_st / 4 * 4 * L.n_pairs;
  L.largest_bytes = ((size_t)(L.n_largest * G) * sizeof(unsigned) + 255) / 256 * 256;
  L.squares_bytes = (size_t)(L.n_st / 4 * L.n_pairs * 2 * kTile * G) * sizeof(double);
  L.exponent_bytes = ((size_t)G * sizeof(int) + 255) / 256 * 256;
  return L;
}

struct Layout {
  int64_t ldp, n_pairs, n_rb2;
  int chunk, n_slots, deal;                     // pair blocks per workgroup, workgroups per (group, row block), XCD mapping
  int64_t n_blocks;                             // 256-row blocks per group in the final reduction
  size_t partial_bytes, sums_bytes, delta_bytes, h_bytes;   // delta_bytes / h_bytes: one of the hi/lo arrays
};
Layout make_layout(int64_t d_out, int64_t d_in, int G) {
  Layout L;
  L.n_pairs = (d_in + 2 * kTile - 1) / (2 * kTile);
  L.ldp = L.n_pairs * 2 * kTile;                // contraction length padded to whole tile pairs
  L.n_rb2 = (d_out / G + 2 * kTile - 1) / (2 * kTile);
  // Slots of at most `chunk` pair blocks (measured on MI355X over the 7B ... 70B shapes, chunk 1 ... 32, both
  // mappings): grids of a thousand workgroups and more run fastest with 12 and stretches dealt to the XCDs in
  // turn (the order is heavy first; a contiguous eighth per XCD leaves the XCD with the heavy pairs up to 30 %
  // behind); small grids (a few workgroups per CU) with three tenths of the pairs per slot and one contiguous
  // stretch per XCD.
  auto slots_with = [&](int64_t c) {
    int64_t n = 0;
    for (int64_t P = 0; P < L.n_pairs; ++P) n += (P + c) / c;
    return n;
  };
  L.chunk = (int)(L.n_pairs < 12 ? L.n_pairs : 12);
  L.deal = slots_with(L.chunk) * L.n_rb2 * G >= 1024 ? 1 : 0;
  if (!L.deal) {
    L.chunk = (int)((3 * L.n_pairs + 9) / 10);
    if (L.chunk < 2) L.chunk = (int)(L.n_pairs < 2 ? L.n_pairs : 2);
  }
  L.n_slots = 0;
  for (int64_t P = 0; P < L.n_pairs; ++P) L.n_slots += (int)((P + L.chunk) / L.chunk);
  L.partial_bytes = ((size_t)((int64_t)L.n_slots * d_out) * sizeof(float) + 255) / 256 * 256;
  L.n_blocks = (d_out / G + 255) / 256;
  L.sums_bytes = ((size_t)(L.n_blocks * G) * sizeof(double) + 255) / 256 * 256;
  L.delta_bytes = ((size_t)((int64_t)G * L.n_rb2 * 2 * kTile * L.ldp) * 2 + 255) / 256 * 256;
  L.h_bytes = ((size_t)((int64_t)G * L.ldp * L.ldp) * 2 + 255) / 256 * 256;
  return L;
}

}  // namespace

size_t objective_workspace(int64_t d_out, int64_t d_in, int G) {
  const Layout L = make_layout(d_out, d_in, G);
  const GramLayout M = make_gram_layout(d_out, d_in, G);       // whether the per-channel terms are wanted is not known here
  const size_t rows = L.partial_bytes + L.sums_bytes + 2 * L.delta_bytes + 2 * L.h_bytes;
  const size_t sums = M.partial_bytes + M.largest_bytes + M.exponent_bytes + M.squares_bytes + 2 * M.delta_bytes;
  return rows > sums ? rows : sums;
}

hipError_t launch_objective(const float* W, const float* What, int64_t d_out, int64_t d_in, int64_t ld,
                            const float* H, int G, double* obj, float* obj_row, void* ws, hipStream_t st) {
  char* p = (char*)ws;
  if (!obj_row) {
    const GramLayout M = make_gram_layout(d_out, d_in, G);
    double* sums = (double*)p;
    unsigned* largest = (unsigned*)(p + M.partial_bytes);
    int* exponent = (int*)((char*)largest + M.largest_bytes);
    double* squares = (double*)((char*)exponent + M.exponent_bytes);
    unsigned short* Dh = (unsigned short*)((char*)squares + M.squares_bytes);
    unsigned short* Dl = (unsigned short*)((char*)Dh + M.delta_bytes);
    const int n_cb = 2 * (int)M.n_pairs;
    hipError_t e;
    split_delta_t_kernel<<<dim3((unsigned)(M.n_st / 4 * G), (unsigned)(2 * n_cb)), dim3(256), 0, st>>>(
        W, What, d_out, d_in, ld, G, n_cb, M.n_st, Dh, Dl, largest, squares);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    scale_delta_kernel<<<dim3((unsigned)(32 * G)), dim3(256), 0, st>>>(Dh, Dl, largest, M.n_largest,
                                                                       n_cb * M.n_st * kTileElems, exponent);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    objective_gram_kernel<<<dim3(kUnits), dim3(512), 0, st>>>(Dh, Dl, H, d_in, G, (int)M.n_pairs, M.n_st, squares, exponent,
                                                              sums);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    objective_sum_kernel<<<dim3((unsigned)G), dim3(256), 0, st>>>(sums, tri_count(M.n_pairs), M.n_st, exponent, obj);
    return hipGetLastError();
  }
  const Layout L = make_layout(d_out, d_in, G);
  float* partial = (float*)p;
  p += L.partial_bytes;
  double* block_sum = (double*)p;
  p += L.sums_bytes;
  unsigned short* Dh = (unsigned short*)p;
  p += L.delta_bytes;
  unsigned short* Dl = (unsigned short*)p;
  p += L.delta_bytes;
  unsigned short* Hh = (unsigned short*)p;
  p += L.h_bytes;
  unsigned short* Hl = (unsigned short*)p;

  const int n_pairs = (int)L.n_pairs, n_rb2 = (int)L.n_rb2;
  hipError_t e;
  const int64_t n_st = L.ldp / kKS;
  split_delta_kernel<<<dim3((unsigned)(n_st / 4), (unsigned)(G * n_rb2 * 2)), dim3(256), 0, st>>>(W, What, d_out, d_in, ld, G,
                                                                                                 n_rb2 * 2, n_st, Dh, Dl);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  split_h_kernel<<<dim3((unsigned)(8 * tri_count(n_pairs)), (unsigned)G), dim3(256), 0, st>>>(H, d_in, L.ldp, n_st, Hh, Hl);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  objective_mfma_kernel<<<dim3((unsigned)((int64_t)L.n_slots * n_rb2 * G)), dim3(512), 0, st>>>(
      Dh, Dl, Hh, Hl, W, What, d_out, d_in, ld, L.ldp, G, n_pairs, n_rb2, L.chunk, L.n_slots, L.deal, partial);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  objective_rows_kernel<<<dim3((unsigned)L.n_blocks, (unsigned)G), dim3(256), 0, st>>>(partial, d_out, G, L.n_slots, obj_row,
                                                                                       block_sum);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  objective_groups_kernel<<<dim3((unsigned)G), dim3(64), 0, st>>>(block_sum, (int)L.n_blocks, obj);
  return hipGetLastError();
}

}  // namespace gq
