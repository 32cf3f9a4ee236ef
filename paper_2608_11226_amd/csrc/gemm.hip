// Projection GEMMs: y[m][n] = sum_k X[m][k] * W[n][k], fp32 accumulation.
//
// bf16 path (CDNA4 MFMA, v_mfma_f32_16x16x32_bf16).  Both operands live in
// HBM in MFMA operand order, so every global load is a fully coalesced
// 16-byte-per-lane read:
//   W (A operand): fragments of 16 weight rows x 32 k (64 lanes x 8, lane =
//                  row%16 + 16*((k%32)/8)), the four fragments of 4
//                  consecutive row blocks adjacent at each k-step (wfrag) --
//                  written once at synthesis;
//   X (B operand): tiles of 32 k x 16 activation rows, [K/32][M/16][64][8],
//                  lane = m%16 + 16*((k%32)/8) -- written by the producing
//                  kernel (norm, SwiGLU, attention).
// Weights are read exactly once per step, with non-temporal loads (keeping
// them out of the caches leaves room for the activations).
//
// k_gemm_ring (decode, M <= 64 rows): a workgroup owns NBW 16-row weight
// blocks and one K split; its one or two waves each take a share of the split.
// Weight and activation fragments stream through a D-deep register ring with
// no LDS and no barriers; every load is unconditional (addresses clamped into
// range, surplus steps masked at the MFMA), so the compiler keeps D - 1 ring
// stages in flight instead of draining the load queue at every step.  X is
// read from L2 by every wave, which costs M/(16 NBW) of the weight bytes in L2
// traffic and nothing in HBM.  Two waves add their sums through LDS once, at
// the end.  With several K splits each writes a partial [split][M][N] that
// the consumer sums in split order.  The SwiGLU variant (gate/up, one split) finishes in
// registers: gate row i and up row i are adjacent weight rows, so the lane
// that holds one also holds the other, and h goes straight to the down
// projection's operand layout.
//
// Gate/up with SwiGLU at decode batches whose weight blocks give every CU 4 to 10 of them (7B) takes a
// balanced grid instead: one workgroup of two waves per CU, the blocks shared out evenly (BAL below); so
// does the LM head, with four one-wave workgroups per CU.
//
// k_gemm_pp (prefill and decode batches of more than 64 rows): eight waves in two groups that take turns
// between LDS reads and MFMAs, both operands through an LDS ring filled by direct loads; tile and K splits
// chosen per shape (details at the kernel and at tile_plan).
//
// k_gemm_q4 (decode with int4 layer weights, M <= 64): weights as 4-bit codes
// in groups of 128 inputs with an fp32 scale and a zero point per row and
// group; the group's scale multiplies its integer dot product in fp32, so the
// weights are never rounded.  The codes enter the MFMA as exact bf16 integers
// (128 + q); a workgroup of eight waves shares each group's activation
// fragments and their sums through LDS.  Larger batches with int4 weights
// write a projection's integers q - z (exact in bf16) into fragments first and take k_gemm_pp on those,
// which scales every group's sum in fp32.
//
// fp32 path: fp32 MFMAs over row-major X and W (the fp32 path exists for exact
// parity on small models).
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace rollout {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

// k_gemm_pp: batches of more than 64 rows.  A workgroup of eight waves owns TN = NB * WN weight blocks (16 rows
// each) x TM = MBW * WM activation blocks; wave (wn, wm) multiplies NB of the weight blocks with MBW of the
// activation blocks (NB x MBW MFMA tiles in registers).  Each k-step's TN + TM fragments (1 KB each) go from
// global memory straight into LDS (dma_lds16: both operands are stored fragment by fragment, so a transfer
// is one contiguous KB and an LDS read is conflict-free) through a ring of NS k-steps, NS - 1 in flight.
//
// The two waves of every SIMD take turns: waves 0..3 and waves 4..7 run the same two phases per k-step, one
// phase apart -- memory (read the step's NB + MBW fragments from LDS, wait for the next step's transfers) and
// multiply (NB * MBW MFMAs) -- with a barrier between phases, so the matrix pipe of a SIMD always has one
// wave's MFMAs while the other wave's LDS reads and transfers run beside them.  (Waves of a workgroup are
// placed on the SIMDs in turn; another placement costs time, not correctness.)  With eight waves in step
// instead, the same tile, ring and fragments take 5 to 15% longer, also with the next step's fragments read
// into a second register set during the MFMAs.
//
// Phases and slots: barrier b0 follows the prologue; group 0 multiplies step s between barriers 2 s + 1 and
// 2 s + 2, group 1 between 2 s + 2 and 2 s + 3, and each reads step s from LDS in the phase before.  In that phase,
// behind its reads, a wave refills the slot of step s - 1 (with step s + NS - 1): both groups' reads of step s - 1 ended
// at a barrier before it.  Before the barrier that ends its reads of step s a wave waits until its own
// transfers of step s + 1 have landed, so the step is whole when group 0 comes to read it.  (Refilling a phase
// later leaves one step less in flight: 0.5% slower over two bf16 layers and 8 to 10% in int4 form, whose ring is
// short for its k-steps; two k-steps a phase, with half the barriers, measured the same.)
//
// Why: the previous kernels (a 256 x 128 tile of four waves with weights in a register ring; for 129..256 rows
// weights staged through registers and LDS by four waves) ran at the rate a CU fetches its operands or at
// one wave's latency per k-step.  us before -> now (sum of its partials' reads included), PFLOP/s now:
//   2,048 rows: 7B gate/up 479-553 -> 405-414 (1.36), 7B QKV 119 -> 61, O 75 -> 57, down 258 -> 210
//   4,096 rows: 14B gate/up 1,000 -> 819-829 (1.41), 14B O 235 -> 181, down 566 -> 413, 72B gate/up 3,150 -> 2,690 (1.48)
//   512 rows:   7B QKV 64 -> 31, down 95 -> 73, gate/up 147 -> 102;  256 rows: 7B gate/up 109 -> 71,
//   14B gate/up 88 -> 85, head 424 -> 367;  128 rows: 14B gate/up 84 -> 62, 7B down 45 -> 38, 7B head 248 -> 234
// All sums are bit-equal to the previous kernels' at equal splits (k order).
//
// rep: every output row is written rep times, to rows rep * m .. rep * m + rep - 1 (the LM head after a prefill: a
// prompt's logits for each member of its group).  rep 0: the product is added to the output instead (O and down
// projections of one split add to the residual stream: the norm that follows then reads the stream alone, not
// the stream and a partial, with the same sums; 4,096 x 5,120: norm 70 -> 50 us, the GEMM 281 -> 294).
//
// Q4 (int4 weights): W holds the integers q - z, exact in bf16 (k_dequant_q4), and Ws the fp32 scale of every
// (16-row block, 128-input group, row).  A group's four k-steps sum into P, and acc += s * P in fp32 while the
// wave reads the next step's fragments, so the weights are never rounded and the vector work runs beside the
// other group's MFMAs.  The tile's scales of a group ride in the ring as one more fragment per k-step.  Half
// of the previous form's MFMAs (two GEMMs over bf16 hi + lo tiles of the dequantised weight) and half of its
// dequantised bytes; needs twice the accumulators, so wave tiles stay at 20 MFMA tiles.
template <int NB, int MBW, int WN, int WM, int NS, bool SWI, bool Q4>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_pp(const bf16x8_t* __restrict__ XF, const bf16x8_t* __restrict__ W, const floatx4_t* __restrict__ Ws,
               float* __restrict__ out, int M, int N, int K, int kslice, int Nt, uint16_t* __restrict__ h, int rep) {
  constexpr int TN = NB * WN, TM = MBW * WM, FR = TN + TM + (Q4 ? 1 : 0);
  constexpr int PER = (FR + 7) / 8;  // fragments a wave transfers per k-step (surplus ones repeat the last)
  static_assert(WN * WM == 8 && NS >= 3, "eight waves; a slot is read, one lands, one is refilled");
  static_assert(!Q4 || (NS % 4 == 0 && TN <= 16), "a group is four unrolled k-steps; its scales fit one fragment");
  __shared__ bf16x8_t ls[NS][FR][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nbt = N >> 4, kbt = K >> 5, Mb = (M + 15) >> 4;
  const int Mt = (Mb + TM - 1) / TM, tiles = Mt * Nt;
  // XCD-aware order (workgroup b runs on XCD b % 8): each XCD takes a contiguous range of tiles, M fastest, so
  // the M tiles of one N tile share its weights through one L2
  const int x = blockIdx.x & 7, t0 = (int)((long long)x * tiles / 8), t1 = (int)((long long)(x + 1) * tiles / 8);
  const int tile = t0 + (int)(blockIdx.x >> 3);
  if (tile >= t1) return;
  const int nt = tile / Mt, mb0 = tile % Mt * TM;
  const int wb0 = (int)((long long)nt * nbt / Nt), wbc = (int)((long long)(nt + 1) * nbt / Nt) - wb0;  // wbc <= TN
  const int kb0 = (int)blockIdx.y * (kslice >> 5);
  const int nk = min(kbt, kb0 + (kslice >> 5)) - kb0;
  const int wn = wave % WN, wm = wave / WN;
  floatx4_t acc[NB][MBW];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < MBW; ++i) acc[j][i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // the wave's fragments of a k-step (blocks past the tile's or the matrix's repeat the last one)
  const char* fb[PER];
  uint32_t fs[PER];  // bytes from one k-step to the next
  const uint32_t soff = Q4 ? (uint32_t)min(lane >> 2, wbc - 1) * (uint32_t)(kbt >> 2) * 64 + (lane & 3) * 16 : 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int f = min(PER * wave + i, FR - 1);
    if (f < TN) {
      const int nb = wb0 + min(f, wbc - 1);
      fb[i] = (const char*)(W + wfrag(nb, kb0, nbt, kbt) * 64);
      fs[i] = wgroup_blocks(nb, nbt) * 1024;
    } else if (f < TN + TM) {
      fb[i] = (const char*)(XF + ((size_t)kb0 * Mb + min(mb0 + f - TN, Mb - 1)) * 64);
      fs[i] = (uint32_t)Mb * 1024;
    } else {  // scales: 64 bytes per (block, group); lane = 4 * block + four rows
      fb[i] = (const char*)(Ws + ((size_t)wb0 * (kbt >> 2) + (kb0 >> 2)) * 4);
      fs[i] = 64;
    }
  }
  // transfers of k-step st, called for 0, 1, 2, ... in turn (the addresses move on by themselves; steps past the
  // last repeat it into slots that are not read again)
  auto transfer = [&](int slot, int st) {
    const bool on = st + 1 < nk;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int f = min(PER * wave + i, FR - 1);
      const bool scales = Q4 && f == FR - 1;
      dma_lds16_at(fb[i], scales ? soff : lane * 16, &ls[slot][f][0]);
      fb[i] += on && (!scales || (st & 3) == 3) ? fs[i] : 0;
    }
  };
  floatx4_t P[Q4 ? NB : 1][Q4 ? MBW : 1];
  if constexpr (Q4) {  // the first k-step scales a group of zeros
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int i = 0; i < MBW; ++i) P[j][i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
  floatx4_t sc[Q4 ? NB : 1];
  if constexpr (Q4) {
#pragma unroll
    for (int j = 0; j < NB; ++j) sc[j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
  auto read_scales = [&](int slot) {  // of the group that k-step's slot belongs to
#pragma unroll
    for (int j = 0; j < NB; ++j)
      sc[j] = reinterpret_cast<const floatx4_t*>(&ls[slot][FR - 1][0])[(wn * NB + j) * 4 + (lane >> 4)];
  };
  auto scale_tile = [&](int j, int i) {  // acc += s * P
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[j][i][r] = fmaf(sc[j][r], P[j][i][r], acc[j][i][r]);
  };
  if (nk > 0) {
    bf16x8_t wf[NB], xf[MBW];
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) transfer(s, s);
    dma_wait_barrier<(NS - 2) * PER>();
    if (wave >= 4) phase_barrier();  // the second group runs one phase behind
    for (int s0 = 0; s0 < nk; s0 += NS) {
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const int st = s0 + u;
        if (st < nk) {
#pragma unroll
          for (int j = 0; j < NB; ++j) wf[j] = ls[u][wn * NB + j][lane];
#pragma unroll
          for (int i = 0; i < MBW; ++i) xf[i] = ls[u][TN + wm * MBW + i][lane];
          transfer((u + NS - 1) % NS, st + NS - 1);  // behind the reads; the slot of step st - 1
          if (Q4 && u % 4 == 3) read_scales(u);  // of the group that ends here, for the next step's FMAs
          dma_wait_barrier<(NS - 2) * PER>();
          __builtin_amdgcn_s_setprio(1);
          if constexpr (Q4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < MBW; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
              if (Q4 && u % 4 == 0) scale_tile(j, i);
              if constexpr (Q4)
                P[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    wf[j], xf[i], u % 4 == 0 ? floatx4_t{0.f, 0.f, 0.f, 0.f} : P[j][i], 0, 0, 0);
              else
                acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], xf[i], acc[j][i], 0, 0, 0);
            }
          if (Q4 && u % 4 == 0) {  // the last group's scaling stays between this step's MFMAs, four FMAs a tile
#pragma unroll
            for (int i = 0; i < MBW; ++i)
#pragma unroll
              for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(acc[j][i]));
#pragma unroll
            for (int t = 0; t < NB * MBW; ++t) {
              __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
          }
          __builtin_amdgcn_s_setprio(0);
          __builtin_amdgcn_sched_barrier(0);  // the MFMAs stay in their phase
          phase_barrier();
        }
      }
    }
    if (wave < 4) phase_barrier();  // as many barriers as the second group
    if constexpr (Q4) {  // the last group
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < MBW; ++i) scale_tile(j, i);
    }
    dma_wait();                     // no transfer outlives the workgroup's LDS
  }
  // D layout of the 16x16 MFMA: lane holds rows 4*(lane/16)+r (weight rows n) of column lane%16 (row m of X)
  float* o = out + (size_t)blockIdx.y * M * N;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if (wn * NB + j >= wbc) continue;
    const int n = (wb0 + wn * NB + j) * 16 + 4 * (lane >> 4);
    if (!SWI && rep == 0) {  // add to the output: a block's loads go out together
      floatx4_t t[MBW];
#pragma unroll
      for (int i = 0; i < MBW; ++i) {
        const int m = min((mb0 + wm * MBW + i) * 16 + (lane & 15), M - 1);
        t[i] = *reinterpret_cast<const floatx4_t*>(o + (size_t)m * N + n);
      }
#pragma unroll
      for (int i = 0; i < MBW; ++i) {
        const int m = (mb0 + wm * MBW + i) * 16 + (lane & 15);
        if (m < M) *reinterpret_cast<floatx4_t*>(o + (size_t)m * N + n) = t[i] + acc[j][i];
      }
      continue;
    }
#pragma unroll
    for (int i = 0; i < MBW; ++i) {
      const int m = (mb0 + wm * MBW + i) * 16 + (lane & 15);
      if (m >= M) continue;
      if constexpr (SWI) {
        // rows n, n+1 are (gate, up) of output f = n/2; rows n+2, n+3 of output f + 1
        const float g0 = acc[j][i][0], u0 = acc[j][i][1], g1 = acc[j][i][2], u1 = acc[j][i][3];
        const float h0 = g0 / (1.0f + expf(-g0)) * u0, h1 = g1 / (1.0f + expf(-g1)) * u1;
        *reinterpret_cast<uint32_t*>(h + xoff(h, m, n >> 1, N >> 1, Mb)) = pack_bf16x2(h0, h1);
      } else {
        const float4 v = make_float4(acc[j][i][0], acc[j][i][1], acc[j][i][2], acc[j][i][3]);
        for (int c = 0; c < rep; ++c) *reinterpret_cast<float4*>(o + ((size_t)m * rep + c) * N + n) = v;
      }
    }
  }
}

// MB = ceil(M/16) row blocks of X; NBW weight blocks per wave; D ring stages; KW waves per workgroup, which
// split the workgroup's K slice between them and add their sums through LDS (in wave order) before the
// epilogue, so a workgroup writes one partial however many waves it has.
// BAL: the grid's workgroups share the N/16 weight blocks out evenly, floor(nbt / grid) or one more each
// (at most NBW), so that a grid of one workgroup per CU gives every CU the same work; otherwise workgroup x
// owns blocks NBW x .. NBW x + NBW - 1.  A workgroup with fewer than NBW blocks loads its last block again
// for the missing ones (a cache hit) and stores nothing for them.
template <int MB, int NBW, int D, bool SWI, int KW, bool BAL = false>
__global__ __launch_bounds__(64 * KW) void k_gemm_ring(const bf16x8_t* __restrict__ XF, const bf16x8_t* __restrict__ W,
                                                       float* __restrict__ out, int M, int N, int K, int kslice,
                                                       uint16_t* __restrict__ h, int rep) {
  if constexpr (!SWI) asm volatile("" ::"s"(rep));  // here, with the other arguments, and not behind the sums
  const int lane = threadIdx.x & 63;
  const int wave = KW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  const int nbt = N >> 4, kbt = K >> 5;
  int nb0, nbc;  // the workgroup's first weight block and its block count (>= 1)
  if constexpr (BAL) {
    nb0 = (int)((long long)blockIdx.x * nbt / gridDim.x);
    nbc = (int)((long long)(blockIdx.x + 1) * nbt / gridDim.x) - nb0;
  } else {
    nb0 = blockIdx.x * NBW;
    nbc = min(NBW, nbt - nb0);
  }
  const int kw0 = (int)blockIdx.y * (kslice >> 5);         // the workgroup's first k-step
  const int nkw = min(kbt, kw0 + (kslice >> 5)) - kw0;    // and its k-steps (none in a surplus split)
  const int per = (nkw + KW - 1) / KW;
  const int kb0 = kw0 + wave * per;
  const int nk = min(kw0 + nkw, kb0 + per) - kb0;         // this wave's k-steps; an empty share adds zeros
  if constexpr (KW == 1) {
    if (nk <= 0) {  // an empty K split contributes zeros
      if constexpr (!SWI) {
        for (int j = 0; j < nbc; ++j)
          for (int m = lane & 15; m < M; m += 16)
            *reinterpret_cast<float4*>(out + ((size_t)blockIdx.y * M + m) * N + (nb0 + j) * 16 + 4 * (lane >> 4)) =
                make_float4(0.f, 0.f, 0.f, 0.f);
      }
      return;
    }
  }
  floatx4_t acc[NBW][MB];
#pragma unroll
  for (int j = 0; j < NBW; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[j][mb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  if (nk > 0) {
    const bf16x8_t* wp[NBW];
    int ws[NBW];  // k-step stride of each block's fragments
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
      const int nb = nb0 + min(j, nbc - 1);
      wp[j] = W + wfrag(nb, kb0, nbt, kbt) * 64 + lane;
      ws[j] = wgroup_blocks(nb, nbt) * 64;
    }
    const bf16x8_t* xp = XF + (size_t)kb0 * MB * 64 + lane;
    bf16x8_t wr[D][NBW], xr[D][MB];
    // ring stage d holds k-step min(i, nk - 1); steps past nk reload the last one and are not used
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const size_t kk = (size_t)min(d, nk - 1);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) xr[d][mb] = xp[(kk * MB + mb) * 64];
#pragma unroll
      for (int j = 0; j < NBW; ++j) wr[d][j] = __builtin_nontemporal_load(wp[j] + kk * ws[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int i = 0; i < nk; i += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (i + d < nk) {
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < NBW; ++j)
              acc[j][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[d][j], xr[d][mb], acc[j][mb], 0, 0, 0);
        }
        const size_t kk = (size_t)min(i + d + D, nk - 1);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) xr[d][mb] = xp[(kk * MB + mb) * 64];
#pragma unroll
        for (int j = 0; j < NBW; ++j) wr[d][j] = __builtin_nontemporal_load(wp[j] + kk * ws[j]);
        // keeps the ring order through scheduling, so each stage waits only for its own loads
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if constexpr (KW > 1) {
    // weight block j is finished by wave j % KW; the other waves hand it their sums through LDS
    static_assert(NBW % KW == 0, "weight blocks are shared out evenly");
    __shared__ floatx4_t red[KW - 1][NBW][MB][64];
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
      const int o = j % KW;
      if (wave != o) {
        const int sl = wave < o ? wave : wave - 1;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) red[sl][j][mb][lane] = acc[j][mb];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
      const int o = j % KW;
      if (wave == o) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          floatx4_t t = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int w = 0; w < KW; ++w) t += (w == o) ? acc[j][mb] : red[w < o ? w : w - 1][j][mb][lane];
          acc[j][mb] = t;
        }
      }
    }
  }
  // D layout of the 16x16 MFMA: lane holds rows 4*(lane/16)+r (weight rows n) of column lane%16 (row m of X)
  // The copies (rep) outside, one run of stores each: with a loop over them behind every store, and rep loaded there,
  // launches that write one took longer (64 rows, 768 outputs over 256 inputs 7.2 -> 6.75 us, 256 over 256 6.4 -> 5.95).
  int c = 0;
  do {
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
      if (j % KW != wave || j >= nbc) continue;
      const int n = (nb0 + j) * 16 + 4 * (lane >> 4);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int m = mb * 16 + (lane & 15);
        if (m >= M) continue;
        if constexpr (SWI) {
          // rows n, n+1 are (gate, up) of output f = n/2; rows n+2, n+3 of output f + 1
          const float g0 = acc[j][mb][0], u0 = acc[j][mb][1], g1 = acc[j][mb][2], u1 = acc[j][mb][3];
          const float h0 = g0 / (1.0f + expf(-g0)) * u0, h1 = g1 / (1.0f + expf(-g1)) * u1;
          *reinterpret_cast<uint32_t*>(h + xoff(h, m, n >> 1, N >> 1, MB)) = pack_bf16x2(h0, h1);
        } else {
          float* o = out + (size_t)blockIdx.y * M * N;
          *reinterpret_cast<float4*>(o + ((size_t)m * rep + c) * N + n) =
              make_float4(acc[j][mb][0], acc[j][mb][1], acc[j][mb][2], acc[j][mb][3]);
        }
      }
    }
  } while (!SWI && ++c < rep);
}

// int4 weights (format in synth.hip: codes [N/16][K/128][64][4 words] in AWQ nibble order, then fp32
// scales and uint8 zeros [N/16][K/128][16]), scaled per group: for a 128-input group g of row n,
//   y[m] += s[n,g] * sum_k (q[n,k] - z[n,g]) x[m,k].
// A code q enters the MFMA as the exact bf16 integer 128 + q (the nibble in the mantissa of 128: one
// shift and one and-or per pair of codes), so a group's MFMA partial is P = sum_k (128 + q) x.
// All-ones MFMAs give X = sum_k x[m,k] once per workgroup, and the group's
// scaling adds s * (P - (128 + z) * X) to the fp32 accumulator.  The weights are never rounded.
__device__ __forceinline__ bf16x8_t q4_operand(uint32_t w, uint32_t magic) {  // magic: 0x43004300
  u32x4_t d;
  d[0] = (w & 0x000F000Fu) | magic;
  d[1] = ((w >> 4) & 0x000F000Fu) | magic;
  d[2] = ((w >> 8) & 0x000F000Fu) | magic;
  d[3] = ((w >> 12) & 0x000F000Fu) | magic;
  return __builtin_bit_cast(bf16x8_t, d);
}

// A workgroup of eight waves owns 16 / KS weight blocks, two per wave: with KS = 2 the waves are two sets that
// take the two halves of the workgroup's groups (their sums meet in LDS at the end).  A set's activation fragments,
// codes, scales and zeros of a group come straight into LDS (dma_lds16_at) through a ring of NS groups, NS - 1
// in flight, and one barrier per group; a wave forms one row block's activation sums (with KS = 1, of half the
// k-steps).  A group is scaled between the first MFMAs of the next one, so that the vector work of the codes and of the
// scaling runs beside MFMAs.
//
// Bound at 64 rows: LDS (sixteen activation fragments per wave and group) and the transfers, half of whose bytes are
// activations out of L2: without any arithmetic the transfers alone take 60 of gate/up's 79 us.  Weights of four waves
// in registers, activations through registers into LDS (the form before) -> now, us at 64 rows:
//   72B (8,192 / 29,568) gate/up 91.6 -> 79.2, O and down 41.1 -> 30.5, QKV 25.6 -> 20.9
// and per layer, all kernels: 72B 1 row 161 -> 142, 32 rows 197 -> 158; 14B 104 -> 75, 126 -> 91; 7B 86 -> 77, 105 -> 93.
// Measured and not better: two halves of the waves that take turns at LDS and MFMAs (79 and 32 us), four waves of
// four blocks each (111 us: half the LDS reads, but one wave a SIMD hides nothing).
template <int MB, int KS, int NS, bool SWI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_q4(
    const bf16x8_t* __restrict__ XF, const u32x4_t* __restrict__ Wq, const floatx4_t* __restrict__ Ws,
    const uint32_t* __restrict__ Wz, float* __restrict__ out, int M, int N, int K, int kslice,
    uint16_t* __restrict__ h) {
  constexpr int WS = 8 / KS, TN = 2 * WS;   // waves and weight blocks of a set
  constexpr int XFR = 4 * MB, FR = XFR + TN + 2;  // fragments of a group: activations, codes, scales, zeros
  constexpr int SP = WS / 4;  // shares of the k-steps in the activation sums
  constexpr int PX = (XFR + 2 + WS - 1) / WS, PER = PX + 2;  // transfers of a wave per group, its two blocks' codes last
  __shared__ u32x4_t ls[NS][KS][FR][64];
  __shared__ float xsl[2][KS][SP][MB][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int set = wave / WS, w = wave % WS;
  const int nb0 = blockIdx.x * TN + 2 * w;  // the wave's blocks
  const int nbt = N >> 4, gbt = K >> 7;
  const int kg0 = (int)blockIdx.y * (kslice >> 7);
  const int ng = min(gbt, kg0 + (kslice >> 7)) - kg0;
  if (ng <= 0) {  // an empty K split contributes zeros
    if constexpr (!SWI) {
      if (set == 0)
        for (int j = 0; j < 2 && nb0 + j < nbt; ++j)
          for (int m = lane & 15; m < M; m += 16)
            *reinterpret_cast<float4*>(out + ((size_t)blockIdx.y * M + m) * N + (nb0 + j) * 16 + 4 * (lane >> 4)) =
                make_float4(0.f, 0.f, 0.f, 0.f);
    }
    return;
  }
  const int steps = (ng + KS - 1) / KS;             // both sets take as many barriers
  const int cnt = set ? ng - steps : steps;         // groups of this set, from g0 (a set without any loads group kg0's)
  const int g0 = cnt > 0 ? kg0 + set * steps : kg0;
  for (int i = tid; i < 2 * KS * SP * MB * 16; i += 512) (&xsl[0][0][0][0][0])[i] = 0.f;
  const char* fb[PER];
  uint32_t fo[PER], fs[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int f = min(PX * w + i, XFR + 1);
    fo[i] = lane * 16;
    if (i >= PX) {
      fb[i] = (const char*)(Wq + ((size_t)min(nb0 + i - PX, nbt - 1) * gbt + g0) * 64);
      fs[i] = 1024;
    } else if (f < XFR) {
      fb[i] = (const char*)(XF + ((size_t)g0 * XFR + f) * 64);
      fs[i] = XFR * 1024;
    } else {  // scales: 64 bytes a block, lane = 4 * block + four rows; zeros: 16 bytes a block, lane = block
      const int left = nbt - 1 - (int)blockIdx.x * TN;  // the last block
      const size_t it = (size_t)blockIdx.x * TN * gbt + g0;
      const bool zero = f > XFR;
      fb[i] = zero ? (const char*)Wz + it * 16 : (const char*)Ws + it * 64;
      fs[i] = zero ? 16 : 64;
      fo[i] = zero ? min(min(lane, TN - 1), left) * gbt * 16
                   : min(min(lane >> 2, TN - 1), left) * gbt * 64 + (lane & 3) * 16;
    }
  }
  // transfers of group st, called for 0, 1, 2, ... in turn (groups past the last repeat it, never read)
  auto transfer = [&](int slot, int st) {
    const bool on = st + 1 < cnt;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int f = i >= PX ? XFR + 2 * w + (i - PX) : min(PX * w + i, XFR + 1);
      dma_lds16_at(fb[i], fo[i], &ls[slot][set][i < PX && f >= XFR ? f + TN : f][0]);
      fb[i] += on ? fs[i] : 0;
    }
  };
  bf16x8_t ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = __builtin_bit_cast(__bf16, (uint16_t)0x3F80);
  uint32_t magic = 0x43004300u;
  asm("" : "+v"(magic));  // in a vector register: an and-or may read only one scalar
  const floatx4_t zf = floatx4_t{0.f, 0.f, 0.f, 0.f};
  floatx4_t acc[2][MB], P[2][MB], sc[2], of[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    sc[j] = of[j] = zf;  // the first group scales a group of zeros
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[j][mb] = P[j][mb] = zf;
  }
  const int ws = min(w & 3, MB - 1);
  float xs[MB];
  auto scale_tile = [&](int j, int mb) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      acc[j][mb][r] = fmaf(sc[j][r], fmaf(-of[j][r], xs[mb], P[j][mb][r]), acc[j][mb][r]);
  };
  auto read_sums = [&](int st) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      xs[mb] = xsl[st & 1][set][0][mb][lane & 15];
      if (SP == 2) xs[mb] += xsl[st & 1][set][SP - 1][mb][lane & 15];
    }
  };
#pragma unroll
  for (int st = 0; st < NS - 1; ++st) transfer(st, st);
  dma_wait_barrier<(NS - 2) * PER>();
  for (int s0 = 0; s0 < steps; s0 += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int st = s0 + u;
      if (st < steps) {
        if (st < cnt) {
          const auto& l = ls[u][set];
          u32x4_t c[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) c[j] = l[XFR + 2 * w + j][lane];
          bf16x8_t xf[4][MB];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) xf[0][mb] = __builtin_bit_cast(bf16x8_t, l[mb][lane]);
          read_sums(st + 1);  // of the group before
#pragma unroll
          for (int t = 1; t < 4; ++t)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) xf[t][mb] = __builtin_bit_cast(bf16x8_t, l[t * MB + mb][lane]);
          // activation sums: a wave's row block (of those past the last the last again), its share of the k-steps
          u32x4_t xq[4 / SP];
#pragma unroll
          for (int t = 0; t < 4 / SP; ++t) xq[t] = l[(SP * t + (w >> 2)) * MB + ws][lane];
          transfer((u + NS - 1) % NS, st + NS - 1);  // the slot of the group before
          __builtin_amdgcn_sched_barrier(0);  // the reads go out first
          floatx4_t sum = zf;
          bf16x8_t a[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) a[j] = q4_operand(c[j][0], magic);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            bf16x8_t an[2] = {a[0], a[1]};
            if (t < 3)
#pragma unroll
              for (int j = 0; j < 2; ++j) an[j] = q4_operand(c[j][t + 1], magic);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
              for (int j = 0; j < 2; ++j) {
                if (t == 0) {
                  scale_tile(j, mb);
                  asm volatile("" : "+v"(acc[j][mb]));  // here, not after the group's MFMAs
                }
                P[j][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j], xf[t][mb], t ? P[j][mb] : zf, 0, 0, 0);
              }
            if (t >= 4 - 4 / SP || SP == 1)
              sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  ones, __builtin_bit_cast(bf16x8_t, xq[SP == 1 ? t : t - 2]), sum, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 2; ++j) a[j] = an[j];
#pragma unroll
            for (int i = 0; i < 2 * MB; ++i) {
              if (t == 0) __builtin_amdgcn_sched_group_barrier(2, 10, 0);
              __builtin_amdgcn_sched_group_barrier(8, 1, 0);
              if (t) __builtin_amdgcn_sched_group_barrier(2, 2, 0);
            }
          }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            sc[j] = __builtin_bit_cast(floatx4_t, l[XFR + TN][4 * (2 * w + j) + (lane >> 4)]);
            const uint32_t z = reinterpret_cast<const uint32_t*>(&l[XFR + TN + 1][2 * w + j])[lane >> 4];
#pragma unroll
            for (int r = 0; r < 4; ++r)  // 128 + z: byte r of z in the mantissa of 128
              of[j][r] = __uint_as_float(__builtin_amdgcn_perm(0x43u, z, 0x04000C0Cu | (uint32_t)r << 16));
          }
          if (lane < 16) xsl[st & 1][set][w >> 2][ws][lane] = sum[0];
        }
        dma_wait_barrier<(NS - 2) * PER>();
      }
    }
  }
  read_sums(cnt + 1);  // the last group
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) scale_tile(j, mb);
  dma_wait();  // no transfer may still be on its way into LDS when it is used again or given back
  if constexpr (KS == 2) {  // set i keeps its waves' block i and takes the other set's sums of it
    floatx4_t(*red)[WS][MB][64] = reinterpret_cast<floatx4_t(*)[WS][MB][64]>(&ls[0][0][0][0]);
    __syncthreads();
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const floatx4_t a0 = acc[0][mb], a1 = acc[1][mb];
      red[set][w][mb][lane] = set ? a0 : a1;
    }
    __syncthreads();
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const floatx4_t o = red[1 - set][w][mb][lane];
      if (set)
        acc[1][mb] = o + acc[1][mb];
      else
        acc[0][mb] += o;
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (nb0 + j >= nbt || (KS == 2 && j != set)) continue;
    const int n = (nb0 + j) * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int m = mb * 16 + (lane & 15);
      if (m >= M) continue;
      if constexpr (SWI) {
        const float g0 = acc[j][mb][0], u0 = acc[j][mb][1], g1 = acc[j][mb][2], u1 = acc[j][mb][3];
        const float h0 = g0 / (1.0f + expf(-g0)) * u0, h1 = g1 / (1.0f + expf(-g1)) * u1;
        *reinterpret_cast<uint32_t*>(h + xoff(h, m, n >> 1, N >> 1, MB)) = pack_bf16x2(h0, h1);
      } else {
        float* o = out + (size_t)blockIdx.y * M * N;
        *reinterpret_cast<float4*>(o + (size_t)m * N + n) =
            make_float4(acc[j][mb][0], acc[j][mb][1], acc[j][mb][2], acc[j][mb][3]);
      }
    }
  }
}

// fp32 path, v_mfma_f32_16x16x4_f32 (fp32 products and sums): a workgroup of four waves owns MT x NT tiles of 16
// rows x 16 outputs, and the waves share out K in runs of 16 (their sums meet in LDS in wave order).  Lane (r, g)
// = (lane % 16, lane / 16) loads four consecutive k of row r at 4 g by one 16-byte load of each operand; four
// MFMAs then take element e of both, i.e. k = 4 g + e of every lane group, so the loads need no rearranging and
// nothing passes through LDS on the way in.  A wave's loads of U runs go out together (indices clamped, surplus
// runs not multiplied): at the small fp32 models' sizes a launch is a few round trips, not bandwidth.  8 rows: 128
// outputs over K = 512 12.1 -> 3.8 us, 1,024 over 128 5.9 -> 3.9 us against an LDS-tiled kernel of one output a thread
// that waited for memory and two barriers every 32 k.
template <int MT, int NT>
__global__ __launch_bounds__(256) void k_gemm_f32(const float* __restrict__ X, int ldx, const float* __restrict__ W,
                                                  float* __restrict__ out, int M, int N, int K, int rep) {
  constexpr int U = MT * NT > 1 ? 4 : 8;
  __shared__ floatx4_t red[3][MT][NT][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * (16 * NT), m0 = blockIdx.y * (16 * MT);
  const int runs = K >> 4, per = (runs + 3) / 4;
  const int c0 = wave * per, c1 = min(runs, c0 + per);
  const float* wp[NT];
  const float* xp[MT];
#pragma unroll
  for (int j = 0; j < NT; ++j) wp[j] = W + (size_t)min(n0 + 16 * j + r, N - 1) * K + 4 * g;
#pragma unroll
  for (int i = 0; i < MT; ++i) xp[i] = X + (size_t)min(m0 + 16 * i + r, M - 1) * ldx + 4 * g;
  floatx4_t acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  for (int c = c0; c < c1; c += U) {
    floatx4_t w[U][NT], x[U][MT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(c + u, c1 - 1) * 16;
#pragma unroll
      for (int j = 0; j < NT; ++j) w[u][j] = *reinterpret_cast<const floatx4_t*>(wp[j] + k);
#pragma unroll
      for (int i = 0; i < MT; ++i) x[u][i] = *reinterpret_cast<const floatx4_t*>(xp[i] + k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u < c1) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][j][e], x[u][i][e], acc[i][j], 0, 0, 0);
      }
  }
  if (wave > 0) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) red[wave - 1][i][j][lane] = acc[i][j];
  }
  __syncthreads();
  if (wave > 0) return;
  // D layout: lane holds outputs 4 g .. + 3 of row r
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const floatx4_t v = ((acc[i][j] + red[0][i][j][lane]) + red[1][i][j][lane]) + red[2][i][j][lane];
      const int m = m0 + 16 * i + r, n = n0 + 16 * j + 4 * g;
      if (m < M && n < N)
        for (int c = 0; c < rep; ++c) *reinterpret_cast<floatx4_t*>(out + ((size_t)m * rep + c) * N + n) = v;
    }
}

int kslice_for(int K, int splits) {
  const int per = (K + splits - 1) / splits;
  return (per + 31) / 32 * 32;
}

// Compute units of the current device (looked up once per device).
int device_cus() {
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// Tiles of k_gemm_pp (weight blocks x activation blocks), with the time of one k-step when every CU runs one
// (us, fitted over 1-8 splits of the 7B, 14B and 72B projections at 72 to 4,096 rows).
struct Tile {
  int tn, tm;
  float step;
};
enum { T_10x8, T_16x8, T_8x16, T_10x16, T_16x16, T_20x16, kTiles };
constexpr Tile kTile[kTiles] = {{10, 8, 0.305f}, {16, 8, 0.373f}, {8, 16, 0.383f}, {10, 16, 0.468f}, {16, 16, 0.679f}, {20, 16, 0.827f}};

struct TilePlan {
  int tile, splits, nt;  // nt: N tiles (they share the weight blocks out evenly)
};

// K slice of one split (int4: whole groups of 128 inputs)
int tile_kslice(int K, int splits, bool q4) { return q4 ? (kslice_for(K, splits) + 127) / 128 * 128 : kslice_for(K, splits); }

// Tile and K splits of a batch of more than 64 rows: the least of (rounds of one workgroup per CU x k-steps x
// the tile's step time + about 6 us a round, against the weights' stream, + what the partials cost to write
// and read).  A round's last workgroups leave CUs idle, so the tile that divides a shape evenly wins (4,096 x
// 5,120 rows: 16 x 16 tiles of 20 x 16 blocks are one round of 256, 16 x 20 of 16 x 16 two; 172 against 235 us).
// Over 162 (projection, rows) pairs the choice is on average 1.5% above the best of all tiles and splits.
// Which tiles are looked at: up to 128 rows those with one 128-row activation tile (two to four times fewer
// multiplications of padding rows); up to 256 rows the wide ones only where K is not split, since with several
// splits their few workgroups do not fill the chip, and the smallest for short K (256 rows of a 256-wide model, eight
// k-steps: 59.8 us a two-layer step with 8 x 16 tiles, 54.8 with 10 x 8; at 7B to 72B widths the cost never takes it
// for gate/up or head).  Up to 384 rows a third 128-row tile wastes less than a
// second 256-row one (300 rows, 72B gate/up 344 against 384 us).
// int4 weights take the tiles of at most 20 MFMA tiles a wave, and K slices of whole groups.
TilePlan tile_plan(int M, int N, int K, int smin, int smax, bool q4 = false) {
  const int nbt = N / 16, mb = (M + 15) / 16, cus = device_cus(), per_xcd = std::max(1, cus / 8);
  const bool single = smax == 1;
  TilePlan best{T_8x16, 1, 0};  // no candidate: refused by launch_pp
  float best_cost = 3e38f;
  for (int t = 0; t < kTiles; ++t) {
    bool look;
    if (M <= 128) look = t == T_10x8 || (t == T_16x8 && single);
    else if (M <= 256) look = single ? t == T_10x8 || t >= T_8x16 : (t == T_10x8 || t == T_8x16);
    else look = t >= T_8x16 || (t == T_16x8 && (M <= 384 || q4));
    if (!look || (q4 && t >= T_16x16)) continue;
    const Tile& T = kTile[t];
    const int mt = (mb + T.tm - 1) / T.tm, need = (nbt + T.tn - 1) / T.tn;
    for (int s = smin; s <= smax; ++s) {
      const int ks = tile_kslice(K, s, q4);
      if ((K + ks - 1) / ks != s) continue;
      const int nk = ks / 32;
      const float stream = (float)N * K * 2 / 5.45e6f;
      const float part = single ? 0.f : 1.6f * s * (float)M * N * 4 / 4.5e6f;
      auto cost = [&](int nt) {
        const int rounds = ((mt * nt + 7) / 8 * s + per_xcd - 1) / per_xcd;
        const float step = std::max(T.step, (float)nbt / nt * 1024 / 41e3f / mt);
        const float tm = rounds * (nk * step + 6.f);
        return std::cbrt(tm * tm * tm + stream * stream * stream) + part;
      };
      const float c = cost(need);
      if (c < best_cost) {
        best_cost = c;
        best = {t, s, need};
      }
      // one activation tile of 128 rows: bound by the weights' stream, so every CU of the last round gets a share
      const int rounds = ((mt * need + 7) / 8 * s + per_xcd - 1) / per_xcd;
      const int spread = std::min(nbt, rounds * cus / s);
      if (T.tm == 8 && mt == 1 && spread > need) {
        const float cs = cost(spread);
        if (cs <= best_cost) {
          best_cost = cs;
          best = {t, s, spread};
        }
      }
    }
  }
  return best;
}

template <int NB, int MBW, int WN, int WM, int NS, bool SWI, bool Q4>
hipError_t launch_pp(hipStream_t s, const TilePlan& p, const bf16x8_t* x, const bf16x8_t* w, const floatx4_t* ws,
                     float* out, int M, int N, int K, uint16_t* h, int rep) {
  // every N tile has a block and holds all of its blocks
  if (p.nt < 1 || p.nt > N / 16 || (N / 16 + p.nt - 1) / p.nt > NB * WN) return hipErrorInvalidValue;
  const int mt = ((M + 15) / 16 + MBW * WM - 1) / (MBW * WM);
  const dim3 grid((unsigned)(mt * p.nt + 7) / 8 * 8, p.splits);
  hipLaunchKernelGGL((k_gemm_pp<NB, MBW, WN, WM, NS, SWI, Q4>), grid, dim3(512), 0, s, x, w, ws, out, M, N, K,
                     tile_kslice(K, p.splits, Q4), p.nt, h, rep);
  return hipGetLastError();
}

// LDS of a tile: NS x (TN + TM) KB (int4 one more fragment), at most 160
template <bool SWI>
hipError_t launch_tile(hipStream_t s, const bf16x8_t* x, const bf16x8_t* w, float* out, int M, int N, int K, int splits,
                       uint16_t* h, int rep) {
  const TilePlan p = tile_plan(M, N, K, splits, splits);
  switch (p.tile) {
    case T_10x8: return launch_pp<5, 2, 2, 4, 5, SWI, false>(s, p, x, w, nullptr, out, M, N, K, h, rep);
    case T_16x8: return launch_pp<4, 4, 4, 2, 4, SWI, false>(s, p, x, w, nullptr, out, M, N, K, h, rep);
    case T_8x16: return launch_pp<4, 4, 2, 4, 4, SWI, false>(s, p, x, w, nullptr, out, M, N, K, h, rep);
    case T_10x16: return launch_pp<5, 4, 2, 4, 4, SWI, false>(s, p, x, w, nullptr, out, M, N, K, h, rep);
    case T_16x16: return launch_pp<4, 8, 4, 2, 4, SWI, false>(s, p, x, w, nullptr, out, M, N, K, h, rep);
    default: return launch_pp<5, 8, 4, 2, 4, SWI, false>(s, p, x, w, nullptr, out, M, N, K, h, rep);
  }
}

template <bool SWI>
hipError_t launch_tile_q4(hipStream_t s, const bf16x8_t* x, const bf16x8_t* w, const floatx4_t* ws, float* out, int M,
                          int N, int K, int splits, uint16_t* h, int rep) {
  const TilePlan p = tile_plan(M, N, K, splits, splits, true);
  switch (p.tile) {
    case T_10x8: return launch_pp<5, 2, 2, 4, 4, SWI, true>(s, p, x, w, ws, out, M, N, K, h, rep);
    case T_16x8: return launch_pp<4, 4, 4, 2, 4, SWI, true>(s, p, x, w, ws, out, M, N, K, h, rep);
    case T_10x16: return launch_pp<5, 4, 2, 4, 4, SWI, true>(s, p, x, w, ws, out, M, N, K, h, rep);
    default: return launch_pp<4, 4, 2, 4, 4, SWI, true>(s, p, x, w, ws, out, M, N, K, h, rep);
  }
}

// Ring kernel shape of the split projections (QKV, O, down at M <= 64).  Workgroups of 4 or 8 weight
// blocks, K split just far enough that the grid fills 80% of the CUs with at most one workgroup per CU: a
// CU's streaming rate bounds these kernels, so a second workgroup on some CUs sets the time, while every
// further split adds a partial for the consumer to sum.  Four-block workgroups are taken when their grid fills at least 80% of the CUs with K
// slices of at most 4096 (their activation reads per weight byte are twice those of eight blocks, which
// costs more than it saves on long K slices); their waves split the K slice four ways while each keeps at
// least 6 k-steps, else two.  Eight-block workgroups run two waves (one when the grid already holds two
// workgroups per CU).  A sweep over blocks per wave (2, 4, 8), waves per workgroup (1, 2, 4) and 1-16
// splits at M = 64 (GEMM time plus reading the partials) puts the optimum at this rule for the 7B and
// 72B QKV, O and down shapes (7B O 10.3 -> 9.3 us with 4 instead of 7 partials, QKV 11.4 -> 10.5 us with
// 3 instead of 7, 72B O 28.1 -> 26.1 us with 2 instead of 4; the two down projections keep 8 blocks), and
// the whole 7B rollout confirms it against the neighbouring shapes of each projection.
// Gate/up with SwiGLU (one split) and the LM head take the balanced grids below.
constexpr int kRingMaxRows = 64;
constexpr int kRingTargetWaves = 512;
int ring_groups(int N, int nbw) { return (N / 16 + nbw - 1) / nbw; }
bool ring_four_blocks(int N, int K, int splits) {
  const int g = ring_groups(N, 4) * splits, cus = device_cus();
  return g <= cus && 5 * g >= 4 * cus && kslice_for(K, splits) <= 4096;
}
int ring_splits(int N, int K, int max_splits) {
  const int cus = device_cus();
  const int smax = std::max(1, std::min(max_splits, K / 256));
  // the fewest splits that bring a grid of g workgroups to 80% of the CUs, never past one per CU
  auto pick = [&](int g) {
    int s = (4 * cus + 5 * g - 1) / (5 * g);
    if (s * g > cus) s = cus / g;
    s = std::max(1, std::min(smax, s));
    const int ks = kslice_for(K, s);
    return (K + ks - 1) / ks;
  };
  const int s4 = pick(ring_groups(N, 4));
  if (ring_four_blocks(N, K, s4)) return s4;
  return pick(ring_groups(N, 8));
}
// waves per workgroup of a split projection's ring kernel with nbw blocks
int ring_split_waves(int N, int K, int nbw, int splits) {
  if (nbw == 4) return kslice_for(K, splits) / 32 / 4 >= 6 ? 4 : 2;
  return ring_groups(N, nbw) * splits < 2 * device_cus() ? 2 : 1;
}
int ring_waves_per_group(int N, int nbw, int splits) {
  return ring_groups(N, nbw) * splits < kRingTargetWaves ? 2 : 1;
}

template <int NBW, bool SWI, int KW>
void launch_ring_kw(hipStream_t s, const bf16x8_t* x, const bf16x8_t* w, float* out, int M, int N, int K,
                    int splits, uint16_t* h, int rep) {
  const int kslice = kslice_for(K, splits);
  const dim3 grid(ring_groups(N, NBW), splits), block(64 * KW);
  switch ((M + 15) / 16) {
    case 1: hipLaunchKernelGGL((k_gemm_ring<1, NBW, 2, SWI, KW>), grid, block, 0, s, x, w, out, M, N, K, kslice, h, rep); break;
    case 2: hipLaunchKernelGGL((k_gemm_ring<2, NBW, 2, SWI, KW>), grid, block, 0, s, x, w, out, M, N, K, kslice, h, rep); break;
    case 3: hipLaunchKernelGGL((k_gemm_ring<3, NBW, 2, SWI, KW>), grid, block, 0, s, x, w, out, M, N, K, kslice, h, rep); break;
    default: hipLaunchKernelGGL((k_gemm_ring<4, NBW, 2, SWI, KW>), grid, block, 0, s, x, w, out, M, N, K, kslice, h, rep); break;
  }
}

// Gate/up with SwiGLU at decode batches, balanced: one workgroup of two waves per CU (the two waves split
// K and add their sums through LDS), the weight blocks shared out evenly, floor(nbt / CUs) or one more per
// workgroup.  The one-wave-per-four-blocks grid (7B: 592 waves) leaves 80 CUs with three waves and 176
// with two, and a CU's streaming rate, not HBM, bounds these kernels: the CUs with three waves set the
// time (7B gate/up 52.8 -> 50.0 us in isolation).  Taken when every CU gets between 4 and kBalNBW blocks.
// The same balance for single-split projections of many blocks (the LM head): four one-wave workgroups per
// CU, each with floor(nbt / grid) or one more of the blocks (7B: 9 or 10 instead of 1188 eight-block
// workgroups, 4.6 per CU; LM head 199.7 -> 180.4 us in isolation).
// Gate/up with more than kBalNBW blocks per CU (72B: 3,696 blocks, 14.4 per CU) takes two one-wave
// workgroups per CU with up to kBal2NBW blocks each, every wave streaming its blocks over the whole K:
// the one-wave-per-four-blocks grid put four workgroups on 156 CUs and three on 100 (72B rollout 2,176 ->
// 2,284 tokens/s; two two-wave workgroups per CU 2,264, four one-wave workgroups per CU 2,146).
constexpr int kBalNBW = 10;
constexpr int kBal2NBW = 8;
constexpr int kBalWavesPerCU = 4;
bool use_balanced_swiglu(int M, int N) {
  const int nbt = N / 16, cus = device_cus();
  return M <= kRingMaxRows && nbt >= 4 * cus && nbt <= kBalNBW * cus;
}
bool use_balanced_swiglu_wide(int M, int N) {
  const int nbt = N / 16, cus = device_cus();
  return M <= kRingMaxRows && nbt > kBalNBW * cus && nbt <= 2 * kBal2NBW * cus;
}
bool use_balanced_single(int M, int N, int splits) {
  const int nbt = N / 16, g = kBalWavesPerCU * device_cus();
  return M <= kRingMaxRows && splits == 1 && nbt >= 4 * g && nbt <= kBalNBW * g;
}

template <bool SWI, int KW, int NBW = kBalNBW>
hipError_t launch_ring_balanced(hipStream_t s, const bf16x8_t* x, const bf16x8_t* w, float* out, int M, int N, int K,
                                int groups, uint16_t* h, int rep) {
  const int kslice = kslice_for(K, 1);
  const dim3 grid(groups, 1), block(64 * KW);
  switch ((M + 15) / 16) {
    case 1: hipLaunchKernelGGL((k_gemm_ring<1, NBW, 2, SWI, KW, true>), grid, block, 0, s, x, w, out, M, N, K, kslice, h, rep); break;
    case 2: hipLaunchKernelGGL((k_gemm_ring<2, NBW, 2, SWI, KW, true>), grid, block, 0, s, x, w, out, M, N, K, kslice, h, rep); break;
    case 3: hipLaunchKernelGGL((k_gemm_ring<3, NBW, 2, SWI, KW, true>), grid, block, 0, s, x, w, out, M, N, K, kslice, h, rep); break;
    default: hipLaunchKernelGGL((k_gemm_ring<4, NBW, 2, SWI, KW, true>), grid, block, 0, s, x, w, out, M, N, K, kslice, h, rep); break;
  }
  return hipGetLastError();
}

template <int NBW, bool SWI>
hipError_t launch_ring(hipStream_t s, const bf16x8_t* x, const bf16x8_t* w, float* out, int M, int N, int K,
                       int splits, uint16_t* h) {
  if (ring_waves_per_group(N, NBW, splits) == 2)
    launch_ring_kw<NBW, SWI, 2>(s, x, w, out, M, N, K, splits, h, 1);
  else
    launch_ring_kw<NBW, SWI, 1>(s, x, w, out, M, N, K, splits, h, 1);
  return hipGetLastError();
}

// A split projection (no SwiGLU) on the ring kernel, shaped by ring_four_blocks / ring_split_waves.  Any
// shape gives the same partials; the split count is the caller's.
hipError_t launch_ring_split(hipStream_t s, const bf16x8_t* x, const bf16x8_t* w, float* out, int M, int N, int K,
                             int splits, int rep) {
  if (ring_four_blocks(N, K, splits)) {
    if (ring_split_waves(N, K, 4, splits) == 4)
      launch_ring_kw<4, false, 4>(s, x, w, out, M, N, K, splits, nullptr, rep);
    else
      launch_ring_kw<4, false, 2>(s, x, w, out, M, N, K, splits, nullptr, rep);
  } else if (ring_split_waves(N, K, 8, splits) == 2) {
    launch_ring_kw<8, false, 2>(s, x, w, out, M, N, K, splits, nullptr, rep);
  } else {
    launch_ring_kw<8, false, 1>(s, x, w, out, M, N, K, splits, nullptr, rep);
  }
  return hipGetLastError();
}

// int4 ring: K slices in whole 128-wide groups
int kslice_q4(int K, int splits) {
  const int per = (K + splits - 1) / splits;
  return (per + 127) / 128 * 128;
}

template <int MB, int KS, int NS, bool SWI>
void launch_q4_mb(hipStream_t s, const bf16x8_t* x, const void* w, float* out, int M, int N, int K, int splits,
                  uint16_t* h) {
  const int kslice = kslice_q4(K, splits);
  const dim3 grid((N / 16 + 16 / KS - 1) / (16 / KS), splits);
  const char* base = (const char*)w;
  const u32x4_t* wq = (const u32x4_t*)base;
  const floatx4_t* ws = (const floatx4_t*)(base + q4_code_bytes(N, K));
  const uint32_t* wz = (const uint32_t*)(base + q4_code_bytes(N, K) + (size_t)N * (K / 128) * 4);
  hipLaunchKernelGGL((k_gemm_q4<MB, KS, NS, SWI>), grid, dim3(512), 0, s, x, wq, ws, wz, out, M, N, K, kslice, h);
}

// One set of waves where the gate/up matrix has the blocks for 80% of the CUs at 16 each (72B: 231 workgroups in one
// wave of the grid, against 462 of two sets); two sets below that and for the split projections, which need the
// workgroups.  LDS: NS x KS x (4 MB + 16 / KS + 2) KB and the sums, at most 160.
template <bool SWI>
hipError_t launch_q4(hipStream_t s, const bf16x8_t* x, const void* w, float* out, int M, int N, int K, int splits,
                     uint16_t* h) {
  if constexpr (SWI) {
    if (5 * ((N / 16 + 15) / 16) >= 4 * device_cus()) {
      switch ((M + 15) / 16) {
        case 1: launch_q4_mb<1, 1, 6, SWI>(s, x, w, out, M, N, K, splits, h); break;
        case 2: launch_q4_mb<2, 1, 5, SWI>(s, x, w, out, M, N, K, splits, h); break;
        case 3: launch_q4_mb<3, 1, 5, SWI>(s, x, w, out, M, N, K, splits, h); break;
        default: launch_q4_mb<4, 1, 4, SWI>(s, x, w, out, M, N, K, splits, h); break;
      }
      return hipGetLastError();
    }
  }
  switch ((M + 15) / 16) {
    case 1: launch_q4_mb<1, 2, 5, SWI>(s, x, w, out, M, N, K, splits, h); break;
    case 2: launch_q4_mb<2, 2, 4, SWI>(s, x, w, out, M, N, K, splits, h); break;
    case 3: launch_q4_mb<3, 2, 3, SWI>(s, x, w, out, M, N, K, splits, h); break;
    default: launch_q4_mb<4, 2, 3, SWI>(s, x, w, out, M, N, K, splits, h); break;
  }
  return hipGetLastError();
}

}  // namespace

int gemm_splits_q4(int M, int N, int K, int max_splits) {
  if (max_splits <= 1) return 1;
  if (M > kRingMaxRows) return tile_plan(M, N, K, 1, std::max(1, std::min(max_splits, K / 256)), true).splits;
  const int groups = (N / 16 + 7) / 8;  // workgroups per K split
  // as for the bf16 split projections: the fewest splits that fill 80% of the CUs, at most one workgroup
  // per CU (72B: QKV 3, O and down 4 instead of 7-8 splits at two workgroups per CU; 72B int4 rollout +1%)
  const int cus = device_cus();
  int s = (4 * cus + 5 * groups - 1) / (5 * groups);
  if (s * groups > cus) s = cus / groups;
  s = std::min(s, std::max(1, K / 256));
  s = std::max(1, std::min(s, max_splits));
  const int ks = kslice_q4(K, s);
  return (K + ks - 1) / ks;
}

// W: the packed matrix (its scales are read from there); Wi: its integers q - z (launch_dequant_q4)
hipError_t launch_gemm_q4_tile(hipStream_t s, const void* X, const void* W, const void* Wi, float* out, int M, int N,
                               int K, int splits, int rep) {
  if (M <= 0) return hipSuccess;
  if (M <= kRingMaxRows || N % 16 || K % 128 || splits < 1 || rep < 0 || rep > 1 || (rep == 0 && splits > 1))
    return hipErrorInvalidValue;
  return launch_tile_q4<false>(s, (const bf16x8_t*)X, (const bf16x8_t*)Wi,
                               (const floatx4_t*)((const char*)W + q4_code_bytes(N, K)), out, M, N, K, splits, nullptr, rep);
}

hipError_t launch_gemm_swiglu_q4_tile(hipStream_t s, const void* X, const void* W, const void* Wi, int M, int N, int K,
                                      void* h) {
  if (M <= 0) return hipSuccess;
  if (M <= kRingMaxRows || N % 32 || K % 128) return hipErrorInvalidValue;
  return launch_tile_q4<true>(s, (const bf16x8_t*)X, (const bf16x8_t*)Wi,
                              (const floatx4_t*)((const char*)W + q4_code_bytes(N, K)), nullptr, M, N, K, 1, (uint16_t*)h, 1);
}

hipError_t launch_gemm_q4(hipStream_t s, const void* X, const void* W, float* out, int M, int N, int K, int splits) {
  if (M <= 0) return hipSuccess;
  if (M > kRingMaxRows || N % 16 || K % 128 || splits < 1) return hipErrorInvalidValue;
  return launch_q4<false>(s, (const bf16x8_t*)X, W, out, M, N, K, splits, nullptr);
}

hipError_t launch_gemm_swiglu_q4(hipStream_t s, const void* X, const void* W, int M, int N, int K, void* h) {
  if (M <= 0) return hipSuccess;
  if (M > kSwigluMaxRows || M > kRingMaxRows || N % 16 || K % 128) return hipErrorInvalidValue;
  return launch_q4<true>(s, (const bf16x8_t*)X, W, nullptr, M, N, K, 1, (uint16_t*)h);
}

int gemm_splits(int dtype, int M, int N, int K, int max_splits) {
  if (dtype != ROLLOUT_DTYPE_BF16 || max_splits <= 1) return 1;
  if (M <= kRingMaxRows) return ring_splits(N, K, max_splits);
  return tile_plan(M, N, K, 1, std::max(1, std::min(max_splits, K / 256))).splits;
}

bool gemm_adds(int dtype, int M, int splits) {
  return dtype == ROLLOUT_DTYPE_BF16 && M > kRingMaxRows && splits == 1;
}

hipError_t launch_gemm(hipStream_t s, int dtype, const void* X, int ldx, const void* W, float* out, int M, int N,
                       int K, int splits, int rep) {
  if (M <= 0) return hipSuccess;
  // adding is k_gemm_pp's only (see gemm_adds)
  if (rep < 0 || (rep != 1 && splits > 1) || (rep == 0 && !gemm_adds(dtype, M, splits))) return hipErrorInvalidValue;
  if (dtype != ROLLOUT_DTYPE_BF16) {
    if (N % 16 || K % 16 || ldx % 4) return hipErrorInvalidValue;
    // four tiles a workgroup once that leaves two workgroups per CU: half the operand reads per product
    const dim3 big((N + 31) / 32, (M + 31) / 32), small(N / 16, (M + 15) / 16);
    if ((size_t)big.x * big.y >= 2 * (size_t)device_cus())
      hipLaunchKernelGGL((k_gemm_f32<2, 2>), big, dim3(256), 0, s, (const float*)X, ldx, (const float*)W, out, M, N, K,
                         rep);
    else
      hipLaunchKernelGGL((k_gemm_f32<1, 1>), small, dim3(256), 0, s, (const float*)X, ldx, (const float*)W, out, M, N,
                         K, rep);
    return hipGetLastError();
  }
  if (N % 16 || K % 32) return hipErrorInvalidValue;
  const bf16x8_t* x = (const bf16x8_t*)X;
  const bf16x8_t* w = (const bf16x8_t*)W;
  if (M <= kRingMaxRows) {
    if (use_balanced_single(M, N, splits))
      return launch_ring_balanced<false, 1>(s, x, w, out, M, N, K, kBalWavesPerCU * device_cus(), nullptr, rep);
    return launch_ring_split(s, x, w, out, M, N, K, splits, rep);
  }
  return launch_tile<false>(s, x, w, out, M, N, K, splits, nullptr, rep);
}

hipError_t launch_gemm_swiglu(hipStream_t s, const void* X, const void* W, int M, int N, int K, void* h) {
  if (M <= 0) return hipSuccess;
  if (N % 32 || K % 32) return hipErrorInvalidValue;
  if (M > kRingMaxRows)  // larger batches: the same epilogue on k_gemm_pp, one K split
    return launch_tile<true>(s, (const bf16x8_t*)X, (const bf16x8_t*)W, nullptr, M, N, K, 1, (uint16_t*)h, 1);
  if (use_balanced_swiglu(M, N))
    return launch_ring_balanced<true, 2>(s, (const bf16x8_t*)X, (const bf16x8_t*)W, nullptr, M, N, K, device_cus(),
                                         (uint16_t*)h, 1);
  if (use_balanced_swiglu_wide(M, N))
    return launch_ring_balanced<true, 1, kBal2NBW>(s, (const bf16x8_t*)X, (const bf16x8_t*)W, nullptr, M, N, K,
                                                   2 * device_cus(), (uint16_t*)h, 1);
  return launch_ring<4, true>(s, (const bf16x8_t*)X, (const bf16x8_t*)W, nullptr, M, N, K, 1, (uint16_t*)h);
}

}  // namespace rollout
