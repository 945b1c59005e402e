// Self-attention of the chunk's queries over the rolling key/value window
// (current chunk plus the kept past chunks), softmax(q k^T / sqrt(d)) v per
// head, no mask.  Keys of all visible chunks are contiguous rows [0, Lk) of
// the per-head cache, so the kernel sees one key range.
//
// bf16 path (flash-style, one pass over the keys): the queries arrive scaled
// by log2(e) / sqrt(d), so probabilities are 2^score.
//   * workgroup = 256 queries of one head, one workgroup per CU;
//   * per 64-key tile, S^T = K Q^T on v_mfma_f32_32x32x16_bf16 (keys on the
//     MFMA rows, queries on the columns), so each lane holds the scores of
//     ONE query: its row sum (and running maximum) are lane-local except one
//     exchange with the partner lane (lane ^ 32);
//   * O^T += V^T P^T on the same MFMA: the V cache is stored transposed
//     ([d][keys]) so a lane's 8-key operand is one 16-byte LDS read, and the K
//     tile rows are permuted in LDS so that the score registers of each lane
//     are exactly the 8 consecutive keys the P operand needs (no shuffles);
//   * K and V^T tiles sit in LDS rings filled by LDS-DMA; the softmax
//     denominator sums the bf16 probabilities that the P.V product consumes;
//     accumulation is float.
// Two kernels: attn_bounded_kernel where the RMSNorm gains bound the scores
// (no running maximum) and its wider waves pay (attention_bounded,
// attention_wide_waves), attn_bf16_kernel otherwise.
// fp32 path: one workgroup per (query, head), plain online softmax.
#include "xc_internal.h"
#include "xc_rules.h"

#include <math.h>

namespace xc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// MFMA row R of a 32-key M-tile -> key offset within the 64-key tile.
//   R = g*8 + hh*4 + r  ->  key = mt*32 + (g/2)*16 + hh*8 + (g%2)*4 + r
__device__ __forceinline__ int key_of_row(int mt, int R) {
  const int g = R >> 3, hh = (R >> 2) & 1, r = R & 3;
  return mt * 32 + (g >> 1) * 16 + hh * 8 + (g & 1) * 4 + r;
}
// inverse: key offset (0..63) -> LDS row holding it
__device__ __forceinline__ int row_of_key(int key) {
  const int mt = key >> 5, k = key & 31;
  const int g = ((k >> 4) << 1) | ((k >> 2) & 1), hh = (k >> 3) & 1, r = k & 3;
  return mt * 32 + g * 8 + hh * 4 + r;
}

// vmcnt(0), the other counters left alone (gfx9 encoding)
#define XC_WAIT_VMCNT0() __builtin_amdgcn_s_waitcnt(0x3f70)
// One 16-byte chunk per lane, global -> LDS (lane l lands at byte 16 l of the
// wave's 1 KB block), from byte off (unsigned, per lane) past the wave-uniform
// base.  A buffer load and not a global one: global LDS loads are FLAT
// instructions, and while one is in flight the compiler turns every wait for
// an LDS read into lgkmcnt(0); behind a buffer load the reads stay counted,
// so a wave keeps several fragments in flight.
__device__ __forceinline__ void dma16(const char* base, unsigned off, bf16* lds_block) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), (short)0, -1, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, lds_block, 16, (int)off, 0, 0, 0);
}
// workgroup barrier that leaves this wave's LDS reads in flight
__device__ __forceinline__ void tile_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

constexpr int kXcds = 8;
constexpr int kWaves = 8;            // waves per attention workgroup
constexpr int kQT = 32 * kWaves;     // queries per attention workgroup
constexpr int kBWaves = kQT / 64;    // waves of the bounded kernel's workgroup

// Workspace floats of one (item, key split) piece: the piece's output
// normalised by its own softmax sum, bf16 [kQT][D], then its running max and
// sum, float [kQT] each.
__host__ __device__ constexpr long long piece_floats(int D) { return (long long)kQT * D / 2 + 2 * kQT; }

__device__ __forceinline__ float partner_max(float x) {
  // max(x, x of lane ^ 32): v_permlane32_swap exchanges the two half-waves
  // (a VALU operation, no LDS round trip)
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float partner_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Work distribution.  An item is (head, 256-query tile); its key tiles are
// split into S equal chunks, S chosen by the launcher so that the units
// (item, chunk) fill whole rounds of resident workgroups (one per CU).  Units
// are ordered [head][chunk][query tile] and dealt to the 8 XCDs (each with
// its own L2) in contiguous ranges (workgroups are dispatched round-robin
// over the XCDs, so workgroup b takes unit (b mod 8) * per_xcd + b / 8): the
// workgroups resident on one XCD then stream the same key/value chunk of one
// head at about the same time.  With S = 1 a unit writes the normalised
// output; otherwise it leaves its own normalised output with its running max
// and sum in the workspace and the merge kernel combines the S pieces of each
// item.
//
// attn_bf16_kernel, any scores (online softmax): 8 waves of 32 queries, two
// per SIMD.  Software pipeline, per wave and key tile j:
//   S(j+1) = K(j+1) Q^T on the MFMA pipe, while the VALU runs the softmax of
//   S(j); then O^T += V(j)^T P(j)^T.  K runs one tile ahead of V in LDS:
//   iteration j reads K(j+1) and V(j) and refills K(j+2) and V(j+1).
template <int D>
__global__ __launch_bounds__(64 * kWaves, 1) void attn_bf16_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ Kc,
                                                           const bf16* __restrict__ Vt, bf16* __restrict__ O, int L,
                                                           int Mpad, int Lcap, int Lk, int H, int n_qt, int n_split,
                                                           float* __restrict__ ws, const int* __restrict__ flag) {
  if (flag != nullptr && *flag) return;
  constexpr int KCH = D / 8;                // 16-byte chunks per key row
  constexpr int KCG = KCH / 8;              // groups of 8 chunks per K row
  constexpr int KB = 8 * KCG / kWaves;      // K DMA blocks per wave and tile
  constexpr int VB = D / 8 / kWaves;        // V^T DMA blocks per wave and tile
  static_assert(KB >= 1 && VB >= 1, "staging layout");
  constexpr int DT = D / 32;                // 32-row output tiles (head dims)
  // (both kernels) K and V^T tiles go global -> LDS by DMA, in 1 KB
  // blocks of 8 rows x 8 sixteen-byte chunks: row r, chunk c sits in block
  // (r / 8, c / 8) at slot ((c % 8) ^ (r / 8 % 2)) * 8 + r % 8.  A DMA
  // instruction fills one block (each lane fetches the chunk its slot holds:
  // 128-byte row segments), the 16 rows a quarter-wave reads at one chunk
  // fall in 16 distinct 16-byte bank groups without padding, and every
  // fragment address is a per-lane base plus a compile-time offset.
  // Four separate arrays: the compiler then tells a DMA into one buffer from
  // fragment reads of the other and does not wait for the DMA before them
  __shared__ __attribute__((aligned(1024))) bf16 sK0[64 * D];
  __shared__ __attribute__((aligned(1024))) bf16 sK1[64 * D];
  __shared__ __attribute__((aligned(1024))) bf16 sV0[D * 64];
  __shared__ __attribute__((aligned(1024))) bf16 sV1[D * 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hi = lane >> 5, lo = lane & 31;
  const int C = H * D;
  const int NT = (Lk + 63) / 64;
  const int units = H * n_split * n_qt;
  const int per_xcd = (units + kXcds - 1) / kXcds;
  const int unit = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (unit >= units) return;
  const int h = unit / (n_split * n_qt);
  const int rem = unit - h * n_split * n_qt;
  const int kc = rem / n_qt, qt = rem - kc * n_qt;
  const int k0 = (int)((long long)kc * NT / n_split), k1 = (int)((long long)(kc + 1) * NT / n_split);
  const int q0 = qt * kQT + wave * 32;
  // Waves whose 32 queries all lie past L (in a ragged last query tile) have
  // nothing to compute: they only stage their share of the K / V^T tiles, in
  // a loop of their own with the same barriers (a branch inside the shared
  // loop instead costs the other waves registers).
  const bool live = __builtin_amdgcn_readfirstlane(q0) < L;

  // source byte offsets (within a tile) of the blocks this wave fills: lane l
  // lands at slot l, i.e. row 8 rg + l % 8 and chunk 8 cg + ((l / 8) ^ (rg & 1));
  // LDS row R of a K tile holds key key_of_row(R / 32, R % 32)
  unsigned kg[KB], vg[VB];
#pragma unroll
  for (int i = 0; i < KB; ++i) {
    const int B = wave + kWaves * i, rg = B / KCG, cg = B % KCG;
    const int R = rg * 8 + (lane & 7), c = cg * 8 + ((lane >> 3) ^ (rg & 1));
    kg[i] = (key_of_row(R >> 5, R & 31) * D + c * 8) * 2;
  }
#pragma unroll
  for (int i = 0; i < VB; ++i) {
    const int rg = wave + kWaves * i;
    const int d = rg * 8 + (lane & 7), c = (lane >> 3) ^ (rg & 1);
    vg[i] = ((unsigned)d * Lcap + c * 8) * 2;
  }
  const int sw = hi ^ ((lo >> 3) & 1);
  const int k_frag = (lo >> 3) * KCG * 1024 + sw * 128 + (lo & 7) * 16;  // bytes
  const int v_frag = (lo >> 3) * 1024 + sw * 128 + (lo & 7) * 16;        // bytes
  {
    bf16x8 qf[D / 16];
    {
      const bf16* qrow = Q + ((long long)h * Mpad + q0 + lo) * D + hi * 8;
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16);
    }
    // staging sources: a wave-uniform per-head base plus 32-bit per-thread
    // byte offsets (the tile advance is a scalar add on the base)
    const char* Kh = reinterpret_cast<const char*>(Kc + (long long)h * Lcap * D);
    const char* Vh = reinterpret_cast<const char*>(Vt + (long long)h * D * Lcap);

    f32x16 oacc[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    auto dma_k = [&](int j, int buf) __attribute__((always_inline)) {
      const char* base = Kh + (long long)j * 64 * D * 2;
#pragma unroll
      for (int i = 0; i < KB; ++i)
        dma16(base, kg[i], (buf ? sK1 : sK0) + (wave + kWaves * i) * 512);
    };
    auto dma_v = [&](int j, int buf) __attribute__((always_inline)) {
      const char* base = Vh + (long long)j * 64 * 2;
#pragma unroll
      for (int i = 0; i < VB; ++i)
        dma16(base, vg[i], (buf ? sV1 : sV0) + (wave + kWaves * i) * 512);
    };
    auto qk = [&](f32x16* sacc, int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[mt][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          const bf16x8 a = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(buf ? sK1 : sK0) + k_frag +
                                                            mt * 4 * KCG * 1024 + (ks >> 2) * 1024 + (ks & 3) * 256);
          sacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], sacc[mt], 0, 0, 0);
        }
    };
    // keys past the window (last tile only) get -inf scores
    auto mask = [&](f32x16* sacc, int j) __attribute__((always_inline)) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = j * 64 + key_of_row(mt, (i >> 2) * 8 + hi * 4 + (i & 3));
          if (key >= Lk) sacc[mt][i] = -INFINITY;
        }
    };
    auto tile_max = [&](const f32x16* sacc) __attribute__((always_inline)) {
      float mx = -INFINITY;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sacc[mt][i]);
      return partner_max(mx);
    };
    // probabilities of one score tile against the settled running max m_run
    // (scores are in log2 units): p = 2^(s - m)
    auto probs = [&](f32x16* sacc, bf16x8* pb) __attribute__((always_inline)) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) sacc[mt][i] = __builtin_amdgcn_exp2f(sacc[mt][i] - m_run);
#pragma unroll
      for (int kv = 0; kv < 4; ++kv)
#pragma unroll
        for (int i = 0; i < 8; ++i) pb[kv][i] = (bf16)sacc[kv >> 1][(kv & 1) * 8 + i];
      const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
      float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
      for (int kv = 0; kv < 4; ++kv) {
        ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[kv], pb[kv], 0, 1), ones, ps0, false);
        ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[kv], pb[kv], 2, 3), ones, ps1, false);
        ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[kv], pb[kv], 4, 5), ones, ps0, false);
        ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[kv], pb[kv], 6, 7), ones, ps1, false);
      }
      l_run += ps0 + ps1;
    };
    auto pv = [&](const bf16x8* pb, int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int kv = 0; kv < 4; ++kv)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const bf16x8 a = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(buf ? sV1 : sV0) + v_frag +
                                                            dt * 4096 + kv * 256);
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[kv], oacc[dt], 0, 0, 0);
        }
    };
    // The running max moves only when a tile's max exceeds it by more than
    // 8 (p then stays <= 2^8 in between, harmless for the float sums and
    // the bf16 probabilities); the rescale then also covers the tile just
    // added.
    auto update_max = [&](float mx) __attribute__((always_inline)) {
      if (mx > m_run + 8.0f) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - mx);
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
        m_run = mx;
      }
    };

    // prologue: K(k0), V(k0), K(k0+1) in LDS; S(k0) and its max
    dma_k(k0, 0);
    dma_v(k0, 0);
    if (k0 + 1 < k1) dma_k(k0 + 1, 1);
    XC_WAIT_VMCNT0();
    __syncthreads();
    if (!live) {
      __syncthreads();
      for (int j = k0; j < k1; ++j) {
        // the buffers iteration j of the compute loop refills
        const int odd = (j - k0) & 1;
        if (j + 2 < k1) dma_k(j + 2, odd);
        if (j + 1 < k1) dma_v(j + 1, 1 - odd);
        XC_WAIT_VMCNT0();
        __syncthreads();
      }
      return;
    }
    f32x16 sa[2], sb[2];
    qk(sa, 0);
    if (k0 == NT - 1) mask(sa, k0);
    m_run = tile_max(sa);
    __syncthreads();  // the first iteration refills K buffer 0, which S(k0) just read

    // Iteration j (local index jj = j - k0; scur = S(j), its max already in m_run):
    //   the DMA refills K(j+2) -> K buffer vb_cur and V(j+1) -> V buffer kb_next
    //   (both last read in iteration j - 1) are issued first and land during
    //   region 1: S(j+1) MFMAs from K buffer kb_next  ||  probabilities of S(j)
    //   region 2: PV(j) MFMAs from V buffer vb_cur     ||  max of S(j+1)
    //   then the (rare) rescale, the wait for this wave's DMA and the barrier.
    // The steady-state loop calls it with constant buffer arguments and no
    // mask: no branch inside.
    auto iter = [&](int j, f32x16* scur, f32x16* snext, int kb_next, int vb_cur, bool has_next, bool mask_next,
                    bool peeled = true) __attribute__((always_inline)) {
      const bool more_k = j + 2 < k1;
      if (more_k) dma_k(j + 2, vb_cur);
      if (has_next) dma_v(j + 1, kb_next);
      if (has_next) qk(snext, kb_next);
      // the peeled iterations keep the steps apart (overlapped, they spill)
      if (peeled) __builtin_amdgcn_sched_barrier(0);
      bf16x8 pb[4];
      probs(scur, pb);
      if (peeled) __builtin_amdgcn_sched_barrier(0);
      pv(pb, vb_cur);
      if (has_next) {
        if (mask_next) mask(snext, j + 1);
        update_max(tile_max(snext));
      }
      XC_WAIT_VMCNT0();
      __syncthreads();
    };
    const int n = k1 - k0;
    const int n_reg = n > 2 ? n - 2 : 0;  // iterations whose next tile is not the segment's last
    int jj = 0;
    for (; jj + 1 < n_reg; jj += 2) {
      iter(k0 + jj, sa, sb, 1, 0, true, false, false);
      iter(k0 + jj + 1, sb, sa, 0, 1, true, false, false);
    }
    if (jj < n_reg) {
      iter(k0 + jj, sa, sb, 1, 0, true, false, false);
      ++jj;
    }
    // the last two iterations: the next tile may be the masked global last
    // one, then there is no next tile
    const bool mask_last = (Lk & 63) != 0 && k1 == NT;
    if ((jj & 1) == 0) {
      if (jj + 1 < n) {
        iter(k0 + jj, sa, sb, 1, 0, true, mask_last);
        iter(k0 + jj + 1, sb, sa, 0, 1, false, false);
      } else {
        iter(k0 + jj, sa, sb, 1, 0, false, false);
      }
    } else {
      if (jj + 1 < n) {
        iter(k0 + jj, sb, sa, 0, 1, true, mask_last);
        iter(k0 + jj + 1, sa, sb, 1, 0, false, false);
      } else {
        iter(k0 + jj, sb, sa, 0, 1, false, false);
      }
    }

    const float l_tot = partner_sum(l_run);
    const int q = q0 + lo;
    if (n_split == 1) {
      // whole item in this unit: normalised output
      const float inv = 1.0f / l_tot;
      if (q < L) {
        bf16* orow = O + (long long)q * C + h * D;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int dd = dt * 32 + g * 8 + hi * 4;
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            bf16x4 o4;
#pragma unroll
            for (int r = 0; r < 4; ++r) o4[r] = (bf16)(oacc[dt][g * 4 + r] * inv);
            *reinterpret_cast<bf16x4*>(orow + dd) = o4;
          }
      }
    } else {
      // partial piece (see piece_floats)
      const int item = h * n_qt + qt;
      float* wo = ws + ((long long)item * n_split + kc) * piece_floats(D);
      bf16* wob = reinterpret_cast<bf16*>(wo);
      const int ql = wave * 32 + lo;
      const float inv = 1.0f / l_tot;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int dd = dt * 32 + g * 8 + hi * 4;
          typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
          bf16x4 o4;
#pragma unroll
          for (int r = 0; r < 4; ++r) o4[r] = (bf16)(oacc[dt][g * 4 + r] * inv);
          *reinterpret_cast<bf16x4*>(wob + ql * D + dd) = o4;
        }
      if (hi == 0) {
        wo[kQT * D / 2 + ql] = m_run;
        wo[kQT * D / 2 + kQT + ql] = l_tot;
      }
    }
  }
}

// Attention whose scores are bounded (attention_bounded).  2^s then needs no
// running maximum: the output accumulators are touched by nothing but MFMAs
// and sit in AGPRs, and a wave has registers for 64 queries.  A workgroup is
// 4 waves (one per SIMD); the two 32-query groups of a wave share every K /
// V^T fragment, which halves the LDS reads per MFMA of 32-query waves.
//
// One wave per SIMD hides nothing behind another wave, so the key loop fixes
// its own order: a step (half a tile, 32 keys) is 8 + 8 slots (d = 128) of
// one fragment read, two MFMAs and 1/16 of the exponentials.  Step i runs
// S(i+1) = K Q^T, O += V^T P(i-1) and P(i) = 2^S(i) side by side: none of the
// three waits for another.  What fits in the shadow of an MFMA was measured
// (one wave, cycles per 32-cycle MFMA + instructions): one v_exp 32.4, two
// 32.5, six v_add 33; one v_dot2_f32_bf16 49, it shares the matrix unit - so
// the row sums unpack the bf16 probabilities and add (4 instructions per
// pair) instead of one dot product.
//
// Measured at 7020 queries, 21060 keys, 12 heads of 128 (main kernel + merge,
// interleaved runs): running maximum, 32-query waves 829 us; the same without
// the maximum 852; this kernel with both exponentials before one MFMA and dot
// products 783, one exponential per MFMA 769 (739 on another box), adds
// instead of dot products 727 there.  Counters: the matrix units are busy 64%
// of the cycles at 1.83 GHz; a loop of nothing but MFMAs holds 1.77 GHz.  So the
// clock is near what the chip's power allows, and 36% of the cycles are idle
// for the matrix units: the instructions between the MFMAs, and each tile's wait
// for all of its DMA.  How they share these cycles was not measured.
//
// The MFMAs are asm statements because the compiler otherwise keeps S in
// AGPRs and copies it out for the exponentials.  It does not see them as
// MFMAs, so the wait states around them are written here.  In the key loop
// the slots' scheduling barriers keep the distances: between the last MFMA on
// a score tile and its first exponential lie the 16 MFMAs (8 at d = 64) of
// P V with their VALU work, between a probability and its MFMA the slots of
// K Q^T.  Everywhere else settle() comes between an MFMA and the VALU reads
// of its result, ready() and pin() between VALU writes and an MFMA that reads
// them; each ties the registers it stands for, because the scheduler moves
// register arithmetic freely past a wait that names none.
template <int D>
__global__ __launch_bounds__(64 * kBWaves, 1) void attn_bounded_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ Kc,
                                                              const bf16* __restrict__ Vt, bf16* __restrict__ O, int L,
                                                              int Mpad, int Lcap, int Lk, int H, int n_qt, int n_split,
                                                              float* __restrict__ ws, const int* __restrict__ flag) {
  if (flag != nullptr && *flag) return;
  constexpr int KCG = D / 64;               // groups of 8 sixteen-byte chunks per key row
  constexpr int NW = kBWaves;
  constexpr int KB = 8 * KCG / NW;          // K DMA blocks per wave and tile
  constexpr int VB = D / 8 / NW;            // V^T DMA blocks per wave and tile
  constexpr int DT = D / 32;
  constexpr int KS = D / 16;
  __shared__ __attribute__((aligned(1024))) bf16 sK0[64 * D];
  __shared__ __attribute__((aligned(1024))) bf16 sK1[64 * D];
  __shared__ __attribute__((aligned(1024))) bf16 sK2[64 * D];
  __shared__ __attribute__((aligned(1024))) bf16 sV0[D * 64];
  __shared__ __attribute__((aligned(1024))) bf16 sV1[D * 64];
  __shared__ __attribute__((aligned(1024))) bf16 sV2[D * 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hi = lane >> 5, lo = lane & 31;
  const int NT = (Lk + 63) / 64;
  const int units = H * n_split * n_qt;
  const int per_xcd = (units + kXcds - 1) / kXcds;
  const int unit = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (unit >= units) return;
  const int h = unit / (n_split * n_qt);
  const int rem = unit - h * n_split * n_qt;
  const int kc = rem / n_qt, qt = rem - kc * n_qt;
  const int k0 = (int)((long long)kc * NT / n_split), k1 = (int)((long long)(kc + 1) * NT / n_split);
  const int q0 = qt * kQT + wave * 64;
  const bool live = __builtin_amdgcn_readfirstlane(q0) < L;

  unsigned kg[KB], vg[VB];
#pragma unroll
  for (int i = 0; i < KB; ++i) {
    const int B = wave + NW * i, rg = B / KCG, cg = B % KCG;
    const int R = rg * 8 + (lane & 7), c = cg * 8 + ((lane >> 3) ^ (rg & 1));
    kg[i] = (key_of_row(R >> 5, R & 31) * D + c * 8) * 2;
  }
#pragma unroll
  for (int i = 0; i < VB; ++i) {
    const int rg = wave + NW * i;
    const int d = rg * 8 + (lane & 7), c = (lane >> 3) ^ (rg & 1);
    vg[i] = ((unsigned)d * Lcap + c * 8) * 2;
  }
  const int sw = hi ^ ((lo >> 3) & 1);
  const int k_frag = (lo >> 3) * KCG * 1024 + sw * 128 + (lo & 7) * 16;  // bytes
  const int v_frag = (lo >> 3) * 1024 + sw * 128 + (lo & 7) * 16;        // bytes
  const char* Kh = reinterpret_cast<const char*>(Kc + (long long)h * Lcap * D);
  const char* Vh = reinterpret_cast<const char*>(Vt + (long long)h * D * Lcap);
  auto dma_k = [&](int j, bf16* dst) __attribute__((always_inline)) {
    const char* base = Kh + (long long)j * 64 * D * 2;
#pragma unroll
    for (int i = 0; i < KB; ++i) dma16(base, kg[i], dst + (wave + NW * i) * 512);
  };
  auto dma_v = [&](int j, bf16* dst) __attribute__((always_inline)) {
    const char* base = Vh + (long long)j * 64 * 2;
#pragma unroll
    for (int i = 0; i < VB; ++i) dma16(base, vg[i], dst + (wave + NW * i) * 512);
  };
  const int jl = k1 - 1;  // the segment's last tile
  dma_k(k0, sK0);
  dma_v(k0, sV0);
  dma_k(min(k0 + 1, jl), sK1);
  XC_WAIT_VMCNT0();
  tile_barrier();
  if (!live) {
    for (int j = k0; j < jl; j += 3) {
      dma_k(min(j + 2, jl), sK2);
      dma_v(min(j + 1, jl), sV1);
      XC_WAIT_VMCNT0();
      tile_barrier();
      if (j + 1 >= jl) break;
      dma_k(min(j + 3, jl), sK0);
      dma_v(min(j + 2, jl), sV2);
      XC_WAIT_VMCNT0();
      tile_barrier();
      if (j + 2 >= jl) break;
      dma_k(min(j + 4, jl), sK1);
      dma_v(min(j + 3, jl), sV0);
      XC_WAIT_VMCNT0();
      tile_barrier();
    }
    return;
  }

  bf16x8 qf[2][KS];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const bf16* qrow = Q + ((long long)h * Mpad + q0 + g * 32 + lo) * D + hi * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[g][ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16);
  }
  f32x16 oacc[2][DT];
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[g][i][r] = 0.f;
  float l_run[2][2] = {{0.f, 0.f}, {0.f, 0.f}};

  auto k_read = [&](const bf16* kt, int mt, int ks) __attribute__((always_inline)) {
    return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(kt) + k_frag + mt * 4 * KCG * 1024 +
                                            (ks >> 2) * 1024 + (ks & 3) * 256);
  };
  auto v_read = [&](const bf16* vt, int mt, int i) __attribute__((always_inline)) {  // i = kv * DT + dt
    return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(vt) + v_frag + (i % DT) * 4096 +
                                            (mt * 2 + i / DT) * 256);
  };
  auto mask = [&](f32x16 (&s)[2], int j, int mt) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int key = j * 64 + key_of_row(mt, (i >> 2) * 8 + hi * 4 + (i & 3));
#pragma unroll
      for (int g = 0; g < 2; ++g)
        if (key >= Lk) s[g][i] = -INFINITY;
    }
  };
  // probabilities of score pair p of the half (g = p / 8, scores 2 (p % 8), + 1)
  auto pack_pair = [&](float e0, float e1, u32x4 (&pk)[2][2], int p) __attribute__((always_inline)) {
    const int g = p >> 3, e = (p & 7) * 2;
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 f = {e0, e1};
    const bf16x2 b = __builtin_convertvector(f, bf16x2);
    const unsigned w = __builtin_bit_cast(unsigned, b);
    pk[g][e >> 3][(e & 7) >> 1] = w;
    l_run[g][0] += __uint_as_float(w << 16);
    l_run[g][1] += __uint_as_float(w & 0xffff0000u);
  };
  auto score_exp = [&](const f32x16 (&s)[2], int p, int k) __attribute__((always_inline)) {
    return __builtin_amdgcn_exp2f(s[p >> 3][(p & 7) * 2 + k]);
  };
  constexpr int NS = KS + 2 * DT;  // slots: one fragment, two MFMAs each
  constexpr int PF = 4;            // fragment reads in flight
  constexpr int PPS = 16 / NS;     // score pairs per slot
  bf16x8 fr[PF];

  // Half-tile step: S' = K Q^T (slots 0 .. KS-1), O += V^T P (the others) and
  // the probabilities of S into pn, spread over the slots.  nk: the next
  // step's K tile and half (its first PF fragments are read here).
  auto step = [&](const bf16* kt, int kmt, const bf16* vt, int vmt, const bf16* nkt, int nkmt, f32x16 (&sn)[2],
                  const f32x16 (&sc)[2], const u32x4 (&pc)[2][2], u32x4 (&pn)[2][2], bool with_pv, auto&& extra)
      __attribute__((always_inline)) {
    float e0 = 0.f, e1 = 0.f;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const bf16x8 a = fr[i % PF];
      const int n = i + PF;
      if (n < KS) fr[i % PF] = k_read(kt, kmt, n);
      else if (n < NS) { if (with_pv) fr[i % PF] = v_read(vt, vmt, n - KS); }
      else fr[i % PF] = k_read(nkt, nkmt, n - NS);
      extra(i);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        if (i < KS) {
          if (i == 0)
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(sn[g]) : "v"(a), "v"(qf[g][0]));
          else
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(sn[g]) : "v"(a), "v"(qf[g][i]));
        } else if (with_pv) {
          asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0"
                       : "+a"(oacc[g][(i - KS) % DT])
                       : "v"(a), "v"(pc[g][(i - KS) / DT]));
        }
        // in the MFMA's shadow: its share of the exponentials, and the pair
        // whose exponentials were taken before it
        if (PPS >= 2) {
          const int p = i * 2 + g;
          if (p > 0) pack_pair(e0, e1, pn, p - 1);
          e0 = score_exp(sc, p, 0);
          e1 = score_exp(sc, p, 1);
        } else if (g == 0) {
          if (i > 0) pack_pair(e0, e1, pn, i - 1);
          e0 = score_exp(sc, i, 0);
        } else {
          e1 = score_exp(sc, i, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    pack_pair(e0, e1, pn, 15);
  };
  auto none = [](int) __attribute__((always_inline)) {};
  // MFMA results that VALU instructions read need up to 19 wait states after
  // the last MFMA; the compiler does not see the MFMAs in the asm
  auto settle = [&](f32x16 (&s)[2]) __attribute__((always_inline)) {
    asm volatile("s_nop 15\n s_nop 7" : "+v"(s[0]), "+v"(s[1]));
  };
  // ... registers that VALU instructions wrote need 2 before an MFMA reads them
  auto ready = [&](u32x4 (&pk)[2][2]) __attribute__((always_inline)) {
    asm volatile("s_nop 3" : "+v"(pk[0][0]), "+v"(pk[0][1]), "+v"(pk[1][0]), "+v"(pk[1][1]));
  };
  // ... and register copies of the accumulators, where the compiler makes
  // any, must not directly precede an MFMA that accumulates on them
  auto pin = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int i = 0; i < DT; ++i) asm volatile("s_nop 3" : "+a"(oacc[g][i]));
  };

  f32x16 sa[2], sb[2];
  u32x4 pa[2][2], pb[2][2];
  // step 2j:   P(2j), O += V(j-1, half 1) P(2j-1), S(2j+1) = K(j, half 1) Q^T
  // step 2j+1: P(2j+1), O += V(j, half 0) P(2j),   S(2j+2) = K(j+1, half 0) Q^T
  auto iter = [&](int j, const bf16* kcur, const bf16* knext, const bf16* vprev, const bf16* vcur, bf16* kdst, bf16* vdst,
                  bool first) __attribute__((always_inline)) {
    const char* kbase = Kh + (long long)min(j + 2, jl) * 64 * D * 2;
    const char* vbase = Vh + (long long)min(j + 1, jl) * 64 * 2;
    auto dma = [&](int i) __attribute__((always_inline)) {
      if (i < KB) dma16(kbase, kg[i], kdst + (wave + NW * i) * 512);
      else if (i < KB + VB) dma16(vbase, vg[i - KB], vdst + (wave + NW * (i - KB)) * 512);
    };
    step(kcur, 1, vprev, 1, knext, 0, sb, sa, pb, pa, !first, dma);
    if (first) pin(), settle(sb);
    step(knext, 0, vcur, 0, knext, 1, sa, sb, pa, pb, true, none);
    XC_WAIT_VMCNT0();
    tile_barrier();
  };
  auto pv_half = [&](const u32x4 (&pc)[2][2], const bf16* vt, int mt) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2 * DT; ++i) {
      const bf16x8 a = v_read(vt, mt, i);
#pragma unroll
      for (int g = 0; g < 2; ++g)
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(oacc[g][i % DT]) : "v"(a), "v"(pc[g][i / DT]));
    }
  };
  auto qk_half = [&](f32x16 (&sn)[2], const bf16* kt, int mt) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const bf16x8 a = k_read(kt, mt, i);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        if (i == 0)
          asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(sn[g]) : "v"(a), "v"(qf[g][0]));
        else
          asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(sn[g]) : "v"(a), "v"(qf[g][i]));
      }
    }
    settle(sn);
  };
  auto probs = [&](const f32x16 (&s)[2], u32x4 (&pk)[2][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 16; ++p) pack_pair(score_exp(s, p, 0), score_exp(s, p, 1), pk, p);
  };
  pin();
  qk_half(sa, sK0, 0);
  const bf16 *kt = sK0, *kn = sK1, *kf = sK2;  // tiles j, j + 1 and the slot of j + 2
  const bf16 *vp = sV2, *vt = sV0, *vf = sV1;  // tiles j - 1, j and the slot of j + 1
  if (k0 < jl) {
#pragma unroll
    for (int i = 0; i < PF; ++i) fr[i] = k_read(sK0, 1, i);
    iter(k0, sK0, sK1, sV2, sV0, sK2, sV1, true);
    int j = k0 + 1;
    for (; j + 3 <= jl; j += 3) {
      iter(j, sK1, sK2, sV0, sV1, sK0, sV2, false);
      iter(j + 1, sK2, sK0, sV1, sV2, sK1, sV0, false);
      iter(j + 2, sK0, sK1, sV2, sV0, sK2, sV1, false);
    }
    kt = sK1, kn = sK2, kf = sK0;
    vp = sV0, vt = sV1, vf = sV2;
    for (; j < jl; ++j) {
      iter(j, kt, kn, vp, vt, const_cast<bf16*>(kf), const_cast<bf16*>(vf), false);
      const bf16* t = kt;
      kt = kn, kn = kf, kf = t;
      t = vp;
      vp = vt, vt = vf, vf = t;
    }
  }
  // the last tile, its keys past the window masked
  mask(sa, jl, 0);
  probs(sa, pa);
  if (k0 < jl) {
    pin();
    ready(pb);
    pv_half(pb, vp, 1);
  }
  qk_half(sb, kt, 1);
  mask(sb, jl, 1);
  probs(sb, pb);
  pin();
  ready(pa);
  ready(pb);
  pv_half(pa, vt, 0);
  pv_half(pb, vt, 1);
  asm volatile("s_nop 15\n s_nop 7");
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int i = 0; i < DT; ++i) asm volatile("" : "+a"(oacc[g][i]));

  const int C = H * D;
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const float l_tot = partner_sum(l_run[g][0] + l_run[g][1]);
    const float inv = 1.0f / l_tot;
    const int q = q0 + g * 32 + lo, ql = wave * 64 + g * 32 + lo;
    float* wo = ws + ((long long)(h * n_qt + qt) * n_split + kc) * piece_floats(D);
    bf16* row = n_split == 1 ? O + (long long)q * C + h * D : reinterpret_cast<bf16*>(wo) + ql * D;
    if (n_split > 1 || q < L) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
          bf16x4 o4;
#pragma unroll
          for (int r = 0; r < 4; ++r) o4[r] = (bf16)(oacc[g][dt][gg * 4 + r] * inv);
          *reinterpret_cast<bf16x4*>(row + dt * 32 + gg * 8 + hi * 4) = o4;
        }
    }
    if (n_split > 1 && hi == 0) {
      wo[kQT * D / 2 + ql] = 0.f;
      wo[kQT * D / 2 + kQT + ql] = l_tot;
    }
  }
}

// Combines the S pieces of each item in a fixed order (deterministic):
// O = sum_p w_p l_p Ohat_p / sum_p w_p l_p, w_p = 2^(m_p - M),
// M = max_p m_p, Ohat_p the piece's normalised output.
// A thread owns one query and 16 consecutive head dims.  It is a chain of
// memory latencies, so loads are issued together: the statistics of all
// pieces (SB >= S a compile-time bound; pieces past S repeat the last one) and
// the outputs of up to 5 pieces at a time.  Attention of 768 tokens, 8 heads
// of 64, 3072 keys in 10 pieces: 23.7 us with one piece after another, 19.3.
template <int D, int SB>
__global__ __launch_bounds__(256) void attn_merge_kernel(bf16* __restrict__ O, int L, int H, int n_qt, int n_split,
                                                         const float* __restrict__ ws,
                                                         const int* __restrict__ flag) {
  if (flag != nullptr && *flag) return;
  constexpr int TPQ = D / 16;  // threads per query
  constexpr int QPB = 256 / TPQ;  // queries per workgroup
  const int blocks_per_item = kQT / QPB;
  const int item = blockIdx.x / blocks_per_item;
  const int ql = (blockIdx.x % blocks_per_item) * QPB + threadIdx.x / TPQ;
  const int d0 = (threadIdx.x % TPQ) * 16;
  const int h = item / n_qt, qt = item - h * n_qt;
  const int q = qt * kQT + ql;
  if (q >= L) return;
  const long long stride = piece_floats(D);
  const float* base = ws + (long long)item * n_split * stride;
  float m[SB], l[SB];
#pragma unroll
  for (int p = 0; p < SB; ++p) {
    const float* pp = base + min(p, n_split - 1) * stride;
    m[p] = pp[kQT * D / 2 + ql];
    l[p] = pp[kQT * D / 2 + kQT + ql];
  }
  constexpr int CH = SB < 5 ? SB : 5;
  float M = m[0], den = 0.f, acc[16];
#pragma unroll
  for (int p = 1; p < SB; ++p) M = fmaxf(M, m[p]);
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
  for (int c = 0; c < SB; c += CH) {
    if (c >= n_split) break;
    bf16x8 v[CH][2];
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      const float* pp = base + min(c + k, n_split - 1) * stride;
      const bf16x8* src = reinterpret_cast<const bf16x8*>(reinterpret_cast<const bf16*>(pp) + ql * D + d0);
      v[k][0] = src[0];
      v[k][1] = src[1];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      if (c + k >= SB) break;
      const float w = c + k < n_split ? __builtin_amdgcn_exp2f(m[c + k] - M) * l[c + k] : 0.f;
      den += w;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        acc[i] += w * (float)v[k][0][i];
        acc[8 + i] += w * (float)v[k][1][i];
      }
    }
  }
  const float inv = 1.0f / den;
  bf16x8 o0, o1;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    o0[i] = (bf16)(acc[i] * inv);
    o1[i] = (bf16)(acc[8 + i] * inv);
  }
  bf16* orow = O + (long long)q * H * D + h * D + d0;
  *reinterpret_cast<bf16x8*>(orow) = o0;
  *reinterpret_cast<bf16x8*>(orow + 8) = o1;
}

template <int D>
void launch_merge(bf16* o, int L, int H, int n_qt, int n_split, const float* ws, const int* flag, hipStream_t st) {
  const int grid = H * n_qt * (kQT / (256 / (D / 16)));
  if (n_split <= 2) attn_merge_kernel<D, 2><<<grid, 256, 0, st>>>(o, L, H, n_qt, n_split, ws, flag);
  else if (n_split == 3) attn_merge_kernel<D, 3><<<grid, 256, 0, st>>>(o, L, H, n_qt, n_split, ws, flag);
  else if (n_split <= 5) attn_merge_kernel<D, 5><<<grid, 256, 0, st>>>(o, L, H, n_qt, n_split, ws, flag);
  else if (n_split <= 10) attn_merge_kernel<D, 10><<<grid, 256, 0, st>>>(o, L, H, n_qt, n_split, ws, flag);
  else attn_merge_kernel<D, 16><<<grid, 256, 0, st>>>(o, L, H, n_qt, n_split, ws, flag);
}

// float32: one workgroup per (query, head), its NW waves take 64-key chunks in
// turn with an online softmax each and merge at the end.  Bound by latency, so
// a lane's row of K (QK: one key per lane) and of V^T (PV: one head dim per
// lane) are read as 16-byte loads in flight together where VEC (D % 4 == 0);
// the scalar form takes any D <= 128.  64 queries, 128 keys, 4 heads of 32:
// 17.8 us with one wave and scalar loads, 5.8 so.  One wave alone (at most 64
// keys) has many queries to serve and little to do for each: it keeps to 64
// registers (eight waves a SIMD), loads rows by four chunks whatever their
// number and merges nothing.  2000 queries, 16 heads of 16: 1 / 7 / 64 keys 22.3 /
// 25.5 / 40.9 us without these, 17.3 / 18.4 / 41.2 with (16.2 / 21.3 / 80 in scalar loads).
template <bool VEC, int NW>
__global__ __launch_bounds__(64 * NW, NW == 1 ? 8 : 4) void attn_f32_kernel(const float* __restrict__ Q, const float* __restrict__ Kc,
                                                       const float* __restrict__ Vt, float* __restrict__ O, int L,
                                                       int Mpad, int Lcap, int Lk, int H, int D, float scale,
                                                       const int* __restrict__ flag) {
  if (flag != nullptr && *flag) return;
  __shared__ __attribute__((aligned(16))) float sq[128];
  __shared__ __attribute__((aligned(16))) float sp[NW][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = blockIdx.x, h = blockIdx.y;
  for (int i = threadIdx.x; i < D; i += 64 * NW) sq[i] = Q[((long long)h * Mpad + q) * D + i];
  __syncthreads();
  const float* Kh = Kc + (long long)h * Lcap * D;
  const float* Vh = Vt + (long long)h * D * Lcap;
  float m = -INFINITY, l = 0.f, o0 = 0.f, o1 = 0.f;
  for (int k0 = wave * 64; k0 < Lk; k0 += 64 * NW) {
    const int key = k0 + lane;
    float s = -INFINITY;
    if (key < Lk) {
      float acc = 0.f;
      if constexpr (VEC) {
        const float4* kr = reinterpret_cast<const float4*>(Kh + (long long)key * D);
        const float4* qr = reinterpret_cast<const float4*>(sq);
        const int n4 = D / 4;
        auto dot = [&](float4 qv, float4 kv) __attribute__((always_inline)) {
          acc += qv.x * kv.x + qv.y * kv.y + qv.z * kv.z + qv.w * kv.w;
        };
        if constexpr (NW == 1) {
          for (int i = 0; i < n4; i += 4) {  // past the row: its last chunk, not added
            float4 kv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) kv[u] = kr[min(i + u, n4 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (i + u < n4) dot(qr[i + u], kv[u]);
          }
        } else {
#pragma unroll 8
          for (int i = 0; i < n4; ++i) dot(qr[i], kr[i]);
        }
      } else {
        for (int i = 0; i < D; ++i) acc += sq[i] * Kh[(long long)key * D + i];
      }
      s = acc * scale;
    }
    float mx = s;
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    const float m_new = fmaxf(m, mx);
    const float alpha = expf(m - m_new);
    const float p = key < Lk ? expf(s - m_new) : 0.f;
    float ps = p;
    for (int off = 32; off > 0; off >>= 1) ps += __shfl_xor(ps, off, 64);
    l = l * alpha + ps;
    o0 *= alpha;
    o1 *= alpha;
    sp[wave][lane] = p;
    // the wave's own lanes read the probabilities: LDS operations of one wave
    // complete in order, the fence keeps the compiler from reordering them
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int nk = min(64, Lk - k0);
    auto pv = [&](int d, float o) __attribute__((always_inline)) {
      const float* vr = Vh + (long long)d * Lcap + k0;
      int jj = 0;
      if constexpr (VEC) {
        // rows of V^T are whole 64-key chunks: one wave's last keys in one load too
        const int n4 = nk & ~3;
        float4 last = {};
        if constexpr (NW == 1) last = *reinterpret_cast<const float4*>(vr + min(n4, 60));
#pragma unroll (NW == 1 ? 2 : 4)
        for (; jj < n4; jj += 4) {
          const float4 vv = *reinterpret_cast<const float4*>(vr + jj);
          const float4 pp = *reinterpret_cast<const float4*>(&sp[wave][jj]);
          o += pp.x * vv.x + pp.y * vv.y + pp.z * vv.z + pp.w * vv.w;
        }
        if constexpr (NW == 1) {
          if (jj < nk) o += sp[wave][jj] * last.x;
          if (jj + 1 < nk) o += sp[wave][jj + 1] * last.y;
          if (jj + 2 < nk) o += sp[wave][jj + 2] * last.z;
          return o;
        }
      }
      for (; jj < nk; ++jj) o += sp[wave][jj] * vr[jj];
      return o;
    };
    if (lane < D) o0 = pv(lane, o0);
    if (lane + 64 < D) o1 = pv(lane + 64, o1);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    m = m_new;
  }
  float* orow = O + (long long)q * H * D + h * D;
  if constexpr (NW == 1) {  // nothing to merge
    if (lane < D) orow[lane] = o0 / l;
    if (lane + 64 < D) orow[lane + 64] = o1 / l;
  } else {
    __shared__ float sm[NW], sl[NW], so[NW][128];
    if (lane == 0) {
      sm[wave] = m;
      sl[wave] = l;
    }
    so[wave][lane] = o0;
    so[wave][lane + 64] = o1;
    __syncthreads();
    // waves that saw no key have m = -inf and weight 0 (wave 0 always saw one)
    float M = sm[0], w[NW], den = 0.f;
#pragma unroll
    for (int i = 1; i < NW; ++i) M = fmaxf(M, sm[i]);
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      w[i] = i * 64 < Lk ? expf(sm[i] - M) : 0.f;
      den += w[i] * sl[i];
    }
    for (int d = threadIdx.x; d < D; d += 64 * NW) {
      float o = 0.f;
#pragma unroll
      for (int i = 0; i < NW; ++i)
        if (i * 64 < Lk) o += w[i] * so[i][d];
      orow[d] = o / den;
    }
  }
}

}  // namespace

int resident_attention_groups() {
  static int groups[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 512;
  if (groups[dev] == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    groups[dev] = cus;
  }
  return groups[dev];
}

// Key splits per item, among those whose partials fit in cap_floats workspace
// floats (one needs none).
int attention_splits(int L, int Lk, int H, int D, size_t cap_floats) {
  const long long items = (long long)H * ((L + kQT - 1) / kQT);
  const long long most = (long long)(cap_floats / ((size_t)items * (size_t)piece_floats(D)));
  return attention_split_count(items, (Lk + 63) / 64, resident_attention_groups(), most);
}

size_t attention_workspace_floats(int L, int Lk, int H, int D) {
  const int s = attention_splits(L, Lk, H, D, SIZE_MAX);
  if (s == 1) return 0;
  return (size_t)H * ((L + kQT - 1) / kQT) * s * (size_t)piece_floats(D);
}

// bounded: no running maximum (the limits and their reasons:
// attention_bounded); otherwise the running-maximum kernel keeps p <= 2^8
// whatever the scores.  At the shape above, in turn on one card: 810 us against 751
// bounded (24 heads of 64: 1017 and 825).
//
// bf16 requirements (checked by the caller): D in {64, 128}; Q has Mpad >=
// roundup(L, 256) rows per head; the caches have Lcap >= roundup(Lk, 64) rows,
// Lcap a multiple of 8 (16-byte aligned V^T rows for the DMA), 16-byte
// aligned bases, and keys past Lk that hold finite values; ws holds ws_floats floats (the key
// split is limited to what fits: attention_workspace_floats(L, Lk, H, D)
// floats allow the unconstrained choice).
void launch_attention(int dtype, const void* q, const void* kc, const void* vt, void* o, float* ws, size_t ws_floats,
                      int L, int Mpad, int Lcap, int Lk, int H, int D, bool bounded, const int* flag, hipStream_t st) {
  if (dtype == 1) {
    const int n_qt = (L + kQT - 1) / kQT;
    const int n_split = attention_splits(L, Lk, H, D, ws != nullptr ? ws_floats : 0);
    const int units = H * n_split * n_qt;
    const int grid = (units + kXcds - 1) / kXcds * kXcds;
    const bool wide = bounded && attention_wide_waves(L, Lk, D, (long long)H * n_qt, resident_attention_groups());
#define XC_ATTN(DD)                                                                                                \
  do {                                                                                                             \
    if (wide)                                                                                                      \
      attn_bounded_kernel<DD><<<grid, 64 * kBWaves, 0, st>>>((const bf16*)q, (const bf16*)kc, (const bf16*)vt,     \
                                                             (bf16*)o, L, Mpad, Lcap, Lk, H, n_qt, n_split, ws,    \
                                                             flag);                                                \
    else                                                                                                           \
      attn_bf16_kernel<DD><<<grid, 64 * kWaves, 0, st>>>((const bf16*)q, (const bf16*)kc, (const bf16*)vt,         \
                                                         (bf16*)o, L, Mpad, Lcap, Lk, H, n_qt, n_split, ws, flag); \
    if (n_split > 1) launch_merge<DD>((bf16*)o, L, H, n_qt, n_split, ws, flag, st);                                \
  } while (0)
    if (D == 128)
      XC_ATTN(128);
    else
      XC_ATTN(64);
#undef XC_ATTN
  } else {
    dim3 grid(L, H);
    const float scale = 1.0f / sqrtf((float)D);
#define XC_ATTN_F32(VEC, NW)                                                                                  \
  attn_f32_kernel<VEC, NW><<<grid, 64 * NW, 0, st>>>((const float*)q, (const float*)kc, (const float*)vt,      \
                                                     (float*)o, L, Mpad, Lcap, Lk, H, D, scale, flag)
    // Lcap is a multiple of 64: with D % 4 == 0 every row of either cache is 16-byte aligned
    const int waves = attention_f32_waves(Lk);
    if (D % 4 == 0) {
      if (waves == 1) XC_ATTN_F32(true, 1);
      else if (waves == 2) XC_ATTN_F32(true, 2);
      else XC_ATTN_F32(true, 4);
    } else {
      if (waves == 1) XC_ATTN_F32(false, 1);
      else if (waves == 2) XC_ATTN_F32(false, 2);
      else XC_ATTN_F32(false, 4);
    }
#undef XC_ATTN_F32
  }
}

}  // namespace xc
