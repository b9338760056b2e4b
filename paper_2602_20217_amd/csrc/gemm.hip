// Matrix products of the decoder sublayers.
//
// bf16 weights are stored in a tile layout that matches the B-operand registers
// of v_mfma_f32_16x16x32_bf16: a 16 (rows of W) x 32 (k) tile is 1 KiB and lane
// l holds row l%16, k = 8(l/16)..8(l/16)+7 at byte offset 16 l.  One 64-lane
// load therefore reads one contiguous KiB of HBM.
//
// Skinny path (M <= 16 rows: decode, draft, verify): the batch-1 decode step
// is HBM-bound, so every weight byte is read once.  Activations enter as two
// bf16 planes hi + lo so the product keeps ~16 mantissa bits of the float32
// activations; the 16 rows of the matrix instruction hold the hi planes of
// up to 8 activation rows in rows 0..7 and their lo planes in rows 8..15, so
// one instruction per weight fragment serves 8 rows (two for 9..16 rows, one
// per group of 8), and the two planes' sums are added in the epilogue.  K is
// split over the waves of a workgroup and reduced in LDS in a fixed order, so
// a row's result does not depend on how many rows are in the batch: a verify
// row and the decode step at the same position produce identical bits.
//
// Batched path (rows of the selection DP and of prefill): single bf16
// activations in the weights' tile layout, both operands staged through LDS by
// direct global-to-LDS loads of whole 1 KiB tiles; workgroup tiles of 128 x 128
// to 256 x 256, eight waves in two groups that alternate between matrix
// instructions and operand traffic.  The K sum is cut into parts by the sizes
// alone; the parts run in workgroups of their own or one after the other in one,
// and are added in order either way.
#include "ks_internal.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace ks {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline bf16x8 ld_frag(const bf16_t* p) {
  return __builtin_bit_cast(bf16x8, *(const u32x4*)p);
}
__device__ inline bf16x8 ld_frag_nt(const bf16_t* p) {
  return __builtin_bit_cast(bf16x8, __builtin_nontemporal_load((const u32x4*)p));
}
__device__ inline bf16x8 zero_frag() {
  u32x4 z = {0u, 0u, 0u, 0u};
  return __builtin_bit_cast(bf16x8, z);
}
__device__ inline float silu_mul(float g, float u) { return g / (1.0f + __expf(-g)) * u; }
__device__ inline void store_split(bf16_t* hi, bf16_t* lo, size_t off, float a) {
  bf16_t h = f2bf(a);
  hi[off] = h;
  if (lo) lo[off] = f2bf(a - bf2f(h));
}

// ------------------------------------------------------------------ skinny
// RMSNorm rides on the producers of the residual stream: the residual
// epilogue (and the embedding) writes x * gain of the next normed product as
// hi + lo bf16 planes together with sums of x^2 per 16-column tile.  AN = 1
// products read those planes like any activation and scale row m by
// 1/sqrt(sum/K + eps) at the end; the 256 tile sums of a row are added by one
// wave in a fixed order, whatever the row count.
template <int NB, int NW, int CH, int MINB, int EPI, int AN, int A1, int MH>
__global__ __launch_bounds__(NW * 64, MINB) void k_gemm_skinny(
    int M, int N, int K, const bf16_t* __restrict__ Ahi, const bf16_t* __restrict__ Alo,
    int lda, const bf16_t* __restrict__ Wp, float* out, int ldo, const float* res, int ldres,
    bf16_t* ohi, bf16_t* olo, int ldact, const float* __restrict__ ssq_in, int nssq, float eps,
    const float* __restrict__ next_gain, bf16_t* nhi, bf16_t* nlo, int ldn, float* next_ssq,
    QkvEpi qe) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KT = K >> 5;
  const int NT = N >> 4;
  const int nt0 = blockIdx.x * NB;
  const int kb = (wave * KT) / NW;
  const int ke = ((wave + 1) * KT) / NW;
  // matrix row of this lane: plane (0 hi, 1 lo) of activation row 8 h + (slot & 7)
  const int slot = lane & 15;
  const int plane = slot >> 3;
  const int kg = lane >> 4;

  static_assert(NB * 256 <= NW * 64, "one epilogue element per thread");
  static_assert(MH == 1 || (MH == 2 && A1 == 0), "one-row staging serves one group of 8 rows");
  // epilogue element of this thread: tile et, row group eh, hi-plane MFMA lane
  // el (its lo-plane partner is el + 32), accumulator register ev (row em,
  // column en)
  const int et = threadIdx.x >> 8, eh = (threadIdx.x >> 7) & 1, ev = threadIdx.x & 3;
  const int el = (threadIdx.x >> 2) & 31;
  const int em = 8 * eh + 4 * (el >> 4) + ev;
  const int en = (nt0 + et) * 16 + (el & 15);
  const bool eact = threadIdx.x < NB * 256 && eh < MH && em < M && nt0 + et < NT;

  // Epilogue operands that do not depend on the product are requested before
  // the weight stream, so that their memory latency overlaps it instead of
  // trailing every workgroup: the RMSNorm tile sums of this wave's first NPRE
  // rows (UPRE per lane), the residual and next-norm gain of the thread's
  // element, the position of its row.
  // (read unconditionally at clamped, valid indices; entries past M or nssq
  // are dropped when the sums are formed)
  constexpr int NPRE = AN ? (NW >= 16 ? 1 : 2) : 1;
  constexpr int UPRE = 4;
  float pre[NPRE][UPRE];
  if (AN) {
#pragma unroll
    for (int q = 0; q < NPRE; ++q) {
      const int m = min(wave + q * NW, M - 1);
#pragma unroll
      for (int u = 0; u < UPRE; ++u)
        pre[q][u] = ssq_in[(size_t)m * nssq + min(lane + 64 * u, nssq - 1)];
    }
  }
  float e_res = 0.f, e_gain = 0.f;
  int e_pos = 0;
  if (EPI == EPI_RESID && eact) {
    e_res = res[(size_t)em * ldres + en];
    if (next_gain) e_gain = next_gain[en];
  }
  if (EPI == EPI_QKV && eact) e_pos = qe.pos[em];

  // One-row products (A1 > 0, decode and draft steps): the activation row
  // (hi and lo planes) is staged in LDS once per workgroup, so the k loop's
  // only global loads are the weight fragments.  Loaded per k step, the
  // activation fragments are one of every two load instructions (for one row,
  // 8 lanes of each plane fetch the same 16 bytes), and the address unit's
  // time for them delays the weight stream's start.  The
  // matrix instructions see the same operand values either way, so the result
  // bits do not depend on the path.  A1 = 16-byte pieces per thread and plane
  // (the launcher takes the least with 64 NW A1 >= K / 8).
  extern __shared__ __align__(16) uint4 s_act[];  // A1: hi plane [K / 8], then lo plane
  constexpr int A1PT = A1 > 0 ? A1 : 1;
  const int n16 = K >> 3;
  uint4 av[2][A1PT];
  if constexpr (A1 != 0) {
    // unconditional loads at clamped indices, so the wait before the LDS
    // store counts only the weight loads issued after them
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
      for (int q = 0; q < A1PT; ++q) {
        const int i = threadIdx.x + q * NW * 64;
        av[pl][q] = ((const uint4*)(pl ? Alo : Ahi))[i < n16 ? i : n16 - 1];
      }
  }

  f32x4 acc[MH][NB];
#pragma unroll
  for (int h = 0; h < MH; ++h)
#pragma unroll
    for (int t = 0; t < NB; ++t) acc[h][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Lanes of rows past M read row 0: their products land in result rows that
  // are never stored (an MFMA result row depends only on its own A row).
  const bf16_t* ap[MH];
#pragma unroll
  for (int h = 0; h < MH; ++h) {
    const int r = 8 * h + (slot & 7);
    ap[h] = (plane ? Alo : Ahi) + (size_t)(r < M ? r : 0) * lda + kg * 8;
  }
  const bf16_t* wb[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    int nt = nt0 + t < NT ? nt0 + t : NT - 1;
    wb[t] = Wp + (size_t)nt * KT * 512 + lane * 8;
  }
  // The wave's k steps [kb, ke) run in full chunks of CH through two register
  // stages: the weight and activation fragments of chunk c + 1 are requested
  // before the matrix instructions of chunk c, so every wave keeps a chunk in
  // flight while it computes (branch-free chunk code, so the compiler counts
  // the loads in flight exactly); the last (ke - kb) % CH steps follow one by
  // one.  The order of the matrix instructions (k ascending, row groups in
  // order) is that of a plain loop.
  bf16x8 w0[NB][CH], x0[MH][CH];
  bf16x8 w1[NB][CH], x1[MH][CH];
  auto fetch = [&](int kc, bf16x8 (&w)[NB][CH], bf16x8 (&x)[MH][CH]) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
#pragma unroll
      for (int t = 0; t < NB; ++t) w[t][u] = ld_frag_nt(wb[t] + (size_t)(kc + u) * 512);
      if constexpr (A1 == 0) {
#pragma unroll
        for (int h = 0; h < MH; ++h) x[h][u] = ld_frag(ap[h] + (kc + u) * 32);
      }
    }
  };
  // A1: lane (slot, kg) takes k = 32 step + 8 kg .. + 7 of its plane of row 0
  // from LDS
  auto act_lds = [&](int k) {
    return __builtin_bit_cast(bf16x8, s_act[plane * n16 + 4 * k + kg]);
  };
  auto compute = [&](int kc, bf16x8 (&w)[NB][CH], bf16x8 (&x)[MH][CH]) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
#pragma unroll
      for (int h = 0; h < MH; ++h) {
        const bf16x8 a = A1 ? act_lds(kc + u) : x[h][u];
#pragma unroll
        for (int t = 0; t < NB; ++t)
          acc[h][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w[t][u], acc[h][t], 0, 0, 0);
      }
    }
  };
  const int nfull = (ke - kb) / CH;  // wave-uniform
  auto ck = [&](int c) { return kb + c * CH; };  // the wave's c-th full chunk
  if constexpr (A1 != 0) {
    // Two chunks in flight from the start (the launcher gives every wave at
    // least two): both are requested before the wait for the row, so the
    // stream does not pause while the row lands in LDS; then chunk c + 2 is
    // requested after chunk c's matrix instructions.
    fetch(ck(0), w0, x0);
    fetch(ck(1), w1, x1);
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
      for (int q = 0; q < A1PT; ++q) {
        const int i = threadIdx.x + q * NW * 64;
        if (i < n16) s_act[pl * n16 + i] = av[pl][q];
      }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's LDS writes are done
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
    int c = 0;
    for (; c + 3 < nfull; c += 2) {  // chunks c and c + 1 are in flight
      compute(ck(c), w0, x0);
      fetch(ck(c + 2), w0, x0);
      compute(ck(c + 1), w1, x1);
      fetch(ck(c + 3), w1, x1);
    }
    compute(ck(c), w0, x0);
    if (c + 2 < nfull) {
      fetch(ck(c + 2), w0, x0);
      compute(ck(c + 1), w1, x1);
      compute(ck(c + 2), w0, x0);
    } else {
      compute(ck(c + 1), w1, x1);
    }
  } else {
    if (nfull > 0) fetch(ck(0), w0, x0);
    int c = 0;
    for (; c + 2 < nfull; c += 2) {  // chunk c is in stage 0 and in flight
      fetch(ck(c + 1), w1, x1);
      compute(ck(c), w0, x0);
      fetch(ck(c + 2), w0, x0);
      compute(ck(c + 1), w1, x1);
    }
    if (c + 1 < nfull) {
      fetch(ck(c + 1), w1, x1);
      compute(ck(c), w0, x0);
      compute(ck(c + 1), w1, x1);
    } else if (c < nfull) {
      compute(ck(c), w0, x0);
    }
  }
  for (int k = kb + nfull * CH; k < ke; ++k) {
    bf16x8 b[NB];
#pragma unroll
    for (int t = 0; t < NB; ++t) b[t] = ld_frag_nt(wb[t] + (size_t)k * 512);
#pragma unroll
    for (int h = 0; h < MH; ++h) {
      const bf16x8 a = A1 ? act_lds(k) : ld_frag(ap[h] + k * 32);
#pragma unroll
      for (int t = 0; t < NB; ++t)
        acc[h][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[t], acc[h][t], 0, 0, 0);
    }
  }

  __shared__ f32x4 red[NW][NB][MH][64];
  __shared__ float s_rs[AN ? 16 : 1];
#pragma unroll
  for (int h = 0; h < MH; ++h)
#pragma unroll
    for (int t = 0; t < NB; ++t) red[wave][t][h][lane] = acc[h][t];
  // the product at (tile t, row group h, hi-plane lane l, register v): the
  // waves' hi-plane partials in wave order, plus their lo-plane partials in
  // wave order
  auto rsum = [&](int t, int h, int l, int v) {
    float a = 0.f, b = 0.f;
    for (int w = 0; w < NW; ++w) {
      a += red[w][t][h][l][v];
      b += red[w][t][h][l + 32][v];
    }
    return a + b;
  };
  if (AN) {
    // row sums in the order of a sequential sum over j = lane, lane + 64, ...,
    // then a butterfly
    auto finish = [&](int m, float t) {
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) t += __shfl_xor(t, o);
      if (lane == 0) s_rs[m] = 1.0f / sqrtf(t / (float)K + eps);
    };
#pragma unroll
    for (int q = 0; q < NPRE; ++q) {
      const int m = wave + q * NW;
      if (m < M) {
        float t = 0.f;
#pragma unroll
        for (int u = 0; u < UPRE; ++u)
          if (lane + 64 * u < nssq) t += pre[q][u];
        for (int j = lane + 64 * UPRE; j < nssq; j += 64) t += ssq_in[(size_t)m * nssq + j];
        finish(m, t);
      }
    }
    for (int m = wave + NPRE * NW; m < M; m += NW) {
      float t = 0.f;
      for (int j = lane; j < nssq; j += 64) t += ssq_in[(size_t)m * nssq + j];
      finish(m, t);
    }
  }
  __syncthreads();

  if (EPI == EPI_SWIGLU || EPI == EPI_QKV) {
    // tile rows 0..7 pair with rows 8..15 (gate/up, or rotary pairs)
    if (eact && (el & 15) < 8) {
      float g = rsum(et, eh, el, ev), u = rsum(et, eh, el + 8, ev);
      if (AN) {
        g *= s_rs[em];
        u *= s_rs[em];
      }
      if (EPI == EPI_SWIGLU) {
        const int c = (nt0 + et) * 8 + (el & 15);
        store_split(ohi, olo, (size_t)em * ldact + c, silu_mul(g, u));
      } else {
        const int tph = qe.hd >> 4, half = qe.hd >> 1;
        const int hh = (nt0 + et) / tph;
        const int f = 8 * ((nt0 + et) % tph) + (el & 15);
        const int p = e_pos;
        if (hh < qe.hq + qe.hkv) {
          const float2 cs = *(const float2*)&qe.rope_cs[((size_t)p * half + f) * 2];
          const float y0 = g * cs.x - u * cs.y;
          const float y1 = u * cs.x + g * cs.y;
          if (hh < qe.hq) {
            float* q = qe.q_out + ((size_t)em * qe.hq + hh) * qe.hd;
            q[f] = y0;
            q[f + half] = y1;
          } else {
            bf16_t* k = qe.kc + ((size_t)(hh - qe.hq) * qe.n_max + p) * qe.hd;
            k[f] = f2bf(y0);
            k[f + half] = f2bf(y1);
          }
        } else {
          bf16_t* vv = qe.vc + ((size_t)(hh - qe.hq - qe.hkv) * qe.n_max + p) * qe.hd;
          vv[f] = f2bf(g);
          vv[f + half] = f2bf(u);
        }
      }
    }
  } else {
    // thread < 256 owns (row em, column el % 16): in a wave the 16 columns of
    // a row sit on lane bits 2..5, so the tile's sum of squares for the next
    // norm is a 4-step butterfly
    static_assert(EPI != EPI_RESID || NB == 1, "next-norm sums assume one tile per block");
    const bool nn = EPI == EPI_RESID && next_gain != nullptr;
    if (threadIdx.x < NB * 256) {
      float s = 0.f;
      if (eact) {
        s = rsum(et, eh, el, ev);
        if (AN) s *= s_rs[em];
        if (EPI == EPI_RESID) s += e_res;
        out[(size_t)em * ldo + en] = s;
      }
      if (nn) {
        float sq = s * s;
        if (eact) store_split(nhi, nlo, (size_t)em * ldn + en, s * e_gain);
        sq += __shfl_xor(sq, 4);
        sq += __shfl_xor(sq, 8);
        sq += __shfl_xor(sq, 16);
        sq += __shfl_xor(sq, 32);
        if (eact && (el & 15) == 0) next_ssq[(size_t)em * NT + nt0 + et] = sq;
      }
    }
  }
}

template <int NB, int NW, int CH, int MINB, int AN, int A1, int MH>
static void launch_skinny_a1(const GemmArgs& g, hipStream_t st) {
  const int NT = g.N / 16;
  const bf16_t* Ahi = (const bf16_t*)g.A.hi;
  const bf16_t* Alo = (const bf16_t*)g.A.lo;
  const bf16_t* W = (const bf16_t*)g.W;
  dim3 grid((NT + NB - 1) / NB), block(NW * 64);
  const size_t lds = A1 ? (size_t)g.K * 4 : 0;  // hi and lo planes of the row
#define KS_SKINNY(E, OH, OL, OLD)                                                               \
  KS_LAUNCH((k_gemm_skinny<NB, NW, CH, MINB, E, AN, A1, MH>), grid, block, lds, st, g.M, g.N,   \
            g.K, Ahi, Alo, g.A.ld, W, g.out, g.ldo, g.res, g.ldres, OH, OL, OLD,                \
            g.ssq_in, g.nssq, g.eps, g.next_gain, (bf16_t*)g.next_act.hi,                       \
            (bf16_t*)g.next_act.lo, g.next_act.ld, g.next_ssq, g.qe)
  if (g.epi == EPI_SWIGLU)
    KS_SKINNY(EPI_SWIGLU, (bf16_t*)g.act_out.hi, (bf16_t*)g.act_out.lo, g.act_out.ld);
  else if (g.epi == EPI_QKV)
    KS_SKINNY(EPI_QKV, nullptr, nullptr, 0);
  else if (g.epi == EPI_RESID) {
    if constexpr (NB == 1) KS_SKINNY(EPI_RESID, nullptr, nullptr, 0);
  }
  else
    KS_SKINNY(EPI_STORE, nullptr, nullptr, 0);
#undef KS_SKINNY
}

template <int NB, int NW, int CH, int MINB, int AN, int STAGE>
static void launch_skinny_an(const GemmArgs& g, hipStream_t st) {
  // one row and a shape that gains from it (STAGE): the activation row from
  // LDS (hi + lo planes, 4 K bytes; 16-byte aligned planes, at most four
  // pieces per thread and plane, every wave at least two full chunks)
  const int pieces = g.K / 8, per = 64 * NW;
  const bool a1 = STAGE && g.M == 1 && g.K % 8 == 0 && (size_t)g.K * 4 <= 64 * 1024 &&
                  4 * per >= pieces && (g.K / 32) / NW >= 2 * CH &&
                  (((uintptr_t)g.A.hi | (uintptr_t)g.A.lo) & 15) == 0;
  if (!a1 && g.M > 8) launch_skinny_a1<NB, NW, CH, MINB, AN, 0, 2>(g, st);
  else if (!a1) launch_skinny_a1<NB, NW, CH, MINB, AN, 0, 1>(g, st);
  else if (per >= pieces) launch_skinny_a1<NB, NW, CH, MINB, AN, 1, 1>(g, st);
  else if (2 * per >= pieces) launch_skinny_a1<NB, NW, CH, MINB, AN, 2, 1>(g, st);
  else launch_skinny_a1<NB, NW, CH, MINB, AN, 4, 1>(g, st);
}

template <int NB, int NW, int CH, int MINB, int STAGE>
static void launch_skinny(const GemmArgs& g, hipStream_t st) {
  if (g.ssq_in) launch_skinny_an<NB, NW, CH, MINB, 1, STAGE>(g, st);
  else launch_skinny_an<NB, NW, CH, MINB, 0, STAGE>(g, st);
}

static int compute_units() {
  static std::atomic<int> cached[16];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n <= 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0)
      n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Vocabulary head on 4 to 8 rows: the arithmetic of k_gemm_skinny<1, 8, 4, ..>
// (EPI_STORE, AN = 1, same waves, k order and sums: the same bits) with workgroups
// that stay and walk the weight tiles blockIdx.x, + gridDim.x, ...  With one tile
// per workgroup every one of the 8016 (128256 rows) reads its rows' activation
// fragments again, as many bytes as its weights at 7 rows, and pays a start and an
// end; here a wave keeps the fragments of its KS k steps in registers for all its
// tiles, and the next tile's weights are requested before the current one's matrix
// instructions.  The tile's partial sums meet in one of two LDS buffers, so one
// barrier per tile orders both, and it waits for LDS only.
// Bound by the weight stream.  Final norm, head and argmax of the 128256-row head:
// 4 / 5 / 8 rows 186 / 198 / 237 -> 180 / 185 / 190 us (one row 172); up to 3 rows
// one tile per workgroup is the faster (2 rows: 172 against 181 us).
template <int KS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_head(
    int M, int N, int K, const bf16_t* __restrict__ Ahi, const bf16_t* __restrict__ Alo, int lda,
    const bf16_t* __restrict__ Wp, float* __restrict__ out, int ldo,
    const float* __restrict__ ssq_in, int nssq, float eps) {
  constexpr int NW = 8;
  __shared__ f32x4 red[2][NW][64];
  __shared__ float s_rs[8];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KT = K >> 5, NT = N >> 4;
  const int slot = lane & 15, plane = slot >> 3, kg = lane >> 4;
  const int r = (slot & 7) < M ? slot & 7 : 0;
  const bf16_t* wb = Wp + (size_t)wave * KS * 512 + lane * 8;
  bf16x8 x[KS], w[2][KS];
  auto fetch = [&](int nt, bf16x8 (&f)[KS]) {
#pragma unroll
    for (int u = 0; u < KS; ++u) f[u] = ld_frag_nt(wb + ((size_t)nt * KT + u) * 512);
  };
  int nt = blockIdx.x;
  fetch(nt, w[0]);
  {
    const bf16_t* ap = (plane ? Alo : Ahi) + (size_t)r * lda + (wave * KS) * 32 + kg * 8;
#pragma unroll
    for (int u = 0; u < KS; ++u) x[u] = ld_frag(ap + u * 32);
  }
  if (wave < M) {  // row sums as in k_gemm_skinny
    float t = 0.f;
    for (int j = lane; j < nssq; j += 64) t += ssq_in[(size_t)wave * nssq + j];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) t += __shfl_xor(t, o);
    if (lane == 0) s_rs[wave] = 1.0f / sqrtf(t / (float)K + eps);
  }
  // output of this thread: row em, column el % 16 of the tile
  const int el = (threadIdx.x >> 2) & 31, ev = threadIdx.x & 3;
  const int em = 4 * (el >> 4) + ev;
  const bool eact = threadIdx.x < 128 && em < M;
  auto tile = [&](auto buf_) {
    constexpr int buf = decltype(buf_)::value;
    const int next = nt + gridDim.x;
    if (next < NT) fetch(next, w[buf ^ 1]);
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < KS; ++u)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[u], w[buf][u], acc, 0, 0, 0);
    red[buf][wave][lane] = acc;
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's LDS accesses are done
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
    if (eact) {
      float a = 0.f, b = 0.f;
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        a += red[buf][q][el][ev];
        b += red[buf][q][el + 32][ev];
      }
      out[(size_t)em * ldo + nt * 16 + (el & 15)] = (a + b) * s_rs[em];
    }
    nt = next;
    return next < NT;
  };
  while (tile(std::integral_constant<int, 0>{}) && tile(std::integral_constant<int, 1>{})) {
  }
}

template <int KS>
static void launch_head(const GemmArgs& g, hipStream_t st) {
  KS_LAUNCH(k_gemm_head<KS>, dim3(std::min(g.N / 16, compute_units())), dim3(512), 0, st, g.M, g.N,
            g.K, (const bf16_t*)g.A.hi, (const bf16_t*)g.A.lo, g.A.ld, (const bf16_t*)g.W, g.out,
            g.ldo, g.ssq_in, g.nssq, g.eps);
}

// Launch shape by matrix shape; the row count picks only between forms that give
// a row the same bits (staging of a single row, one or two groups of 8 rows,
// k_gemm_head for 4 to 8 rows of a vocabulary; 9 to 16 rows of one keep a tile per
// workgroup, as k_gemm_head's registers hold one group).  Measured on MI355X with the Llama-8B shapes (cold weights; 4/8/16 waves, 1/2/4-deep
// pipelined chunks, workgroups per CU forced by the register budget, staging
// on or off): gate/up one tile per 4-wave workgroup, 2-deep chunks; the long-K
// down projection and the square O projection 16 waves, 4-deep; the vocabulary
// head and the q/k/v projection 8 waves, 4-deep; every shape but the head with the
// one-row activation staged in LDS and two chunks per wave in flight from the start
// (8K decode step 3.22 -> 3.09 ms against per-step activation loads).  The head's
// 8016 workgroups pay the staging each: 180 us with it, 171.5 without.
// (output tiles per workgroup, waves, k steps per chunk, workgroups per CU
// the register budget must allow, one-row activation staged in LDS)
#ifndef KS_SK_GU
#define KS_SK_GU 1, 4, 2, 1, 1
#endif
#ifndef KS_SK_DOWN
#define KS_SK_DOWN 1, 16, 4, 1, 1
#endif
#ifndef KS_SK_HEAD
#define KS_SK_HEAD 1, 8, 4, 1, 0
#endif
#ifndef KS_SK_SQ
#define KS_SK_SQ 1, 16, 4, 1, 1
#endif
#ifndef KS_SK_WIDE
#define KS_SK_WIDE 1, 8, 4, 1, 1
#endif
void gemm_bf16_skinny(const GemmArgs& g, hipStream_t st) {
  if (g.epi == EPI_SWIGLU) launch_skinny<KS_SK_GU>(g, st);
  else if (g.K >= 8192) launch_skinny<KS_SK_DOWN>(g, st);
  else if (g.N >= 65536 && g.M >= 4 && g.M <= 8 && g.ssq_in && g.epi == EPI_STORE &&
           g.K % 1024 == 0 && g.K <= 4096) {
    switch (g.K / 1024) {  // k steps per wave: K / 256
      case 1: launch_head<4>(g, st); break;
      case 2: launch_head<8>(g, st); break;
      case 3: launch_head<12>(g, st); break;
      default: launch_head<16>(g, st); break;
    }
  } else if (g.N >= 65536) launch_skinny<KS_SK_HEAD>(g, st);
  else if (g.N <= 4096) launch_skinny<KS_SK_SQ>(g, st);
  else launch_skinny<KS_SK_WIDE>(g, st);
}

// ----------------------------------------------------------------- batched
__device__ constexpr int vmcnt_imm(int n) {
  // s_waitcnt immediate: vmcnt = n, expcnt and lgkmcnt not waited for
  return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14);
}

// Batched rows (prefill chunks, selection DP).  Workgroup tile 64 RI x
// 64 (C0 + C1), eight waves (2 x 4).  A k step of 64 is four blocks in LDS, made
// of 1 KiB operand tiles (16 rows x 32 k) in MFMA register order as they lie in
// memory: the two row halves of A (2 RI row tiles each) and two column parts of
// W (4 C0 and 4 C1 column tiles); wave (wm, wn) owns RI row tiles of each A half
// and C0 + C1 column tiles, so its tile is four quadrants of 2 RI C matrix
// instructions per step.  Both steps of a two-stage ring are in use; a block is
// refilled with step k + 2 as soon as its last reader of step k is past, so
// loads run six phases ahead and no wait ever drains them.
//
// A step is four phases: [read the quadrant's new operands, request one block of
// step k + 2, wait for those reads and for the block needed next; barrier;
// matrix instructions; barrier].  The four waves of the upper row half (one
// per SIMD) run one segment ahead of the other four, so on every SIMD one wave
// issues matrix instructions while the other moves operands.
//   phase 0: reads A half 0 of step k        requests W part 0   A0 W0
//   phase 1: reads W part 1                  requests A half 0   A0 W1
//   phase 2: reads A half 1                  requests W part 1   A1 W1
//   phase 3: reads W part 0 of step k + 1    requests A half 1   A1 W0
// A block's refill is requested at least two segments after its reads in the
// leading group and one after those in the trailing group, which waited for
// them before the barrier in between.  Tiles past the last re-read the last
// one (valid addresses, never used), so the count of loads in flight is the
// same in every phase.  The W fragment is the first operand: a lane then holds
// four consecutive columns of one row.
//
// A result is the sum, in order, of P partial sums over the parts
// [p KT / P, (p + 1) KT / P) of the 32-wide k tiles, k ascending inside a part
// (P from gemm_parts).  SPLIT: one workgroup per part stores its float32 sums to
// part[p][M][N] for k_splitk_reduce.  FOLD: the workgroup walks all parts and
// adds each to a second set of accumulators where it ends, with no break in the
// stream of loads.  Tile shape and mode change no bit of the result.
//
// What bounds it: operand traffic into LDS, then the matrix units' clock.  At
// 4096 rows of the gate/up shape (256 x 256 tiles, seven full rounds) it takes
// 645 us = 1.49 PFLOP/s; without its loads 529-564 us.  With A row-major (each
// load 16 rows x 64 bytes) the same kernel took 701 us; 128 x 256 tiles in a
// three-stage ring with one barrier per step took 975 us row-major, 819 us in
// operand tiles.  At 512 and 1225 rows: 150 -> 101 us and 321 -> 244-273 us.
enum { MODE_ONE = 0, MODE_SPLIT = 1, MODE_FOLD = 2 };
template <int EPI, int MODE, int RI, int C0, int C1>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_wide(
    int M, int N, int K, const bf16_t* __restrict__ A, const bf16_t* __restrict__ Wp, float* out,
    int ldo, const float* res, int ldres, bf16_t* ohi, int okt, int MB, int NB, int P, int vec,
    float* __restrict__ part) {
  constexpr int GM = 8;  // row tiles that share column tiles (4, 8, 16: within 2%)
  constexpr int CT = C0 + C1;
  constexpr int NA = RI > 2 ? 2 : 1, N0 = C0, N1 = C1;  // loads of a wave per block
  constexpr int NS = 2 * NA + N0 + N1;                   // and per step
  constexpr int EA = 4 * RI * 512;                       // elements of an A block
  constexpr int E0 = 8 * C0 * 512, E1 = 8 * C1 * 512;
  constexpr int OA[2] = {0, EA}, OW[2] = {2 * EA, 2 * EA + E0};
  __shared__ __align__(16) bf16_t Sg[2][2 * EA + E0 + E1];  // by step parity
  const int KT = K >> 5, NT = N >> 4, MT = (M + 15) >> 4;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  // logical id: consecutive on one XCD (blocks are dealt round-robin over 8);
  // GM row tiles by all column tiles in turn, so the tiles that run together on
  // an XCD share rows and columns
  const int nblk = gridDim.x;
  int lb = blockIdx.x;
  if ((nblk & 7) == 0) lb = (lb & 7) * (nblk >> 3) + (lb >> 3);
  const int ks = MODE == MODE_SPLIT ? lb / (MB * NB) : 0;
  lb -= ks * (MB * NB);
  const int grp = lb / (GM * NB), gm = min(GM, MB - grp * GM);
  lb -= grp * GM * NB;
  const int mb = grp * GM + lb % gm, nb = lb / gm;
  const int mt0 = mb * 4 * RI, nt0 = nb * 4 * CT;
  // 32-wide k tiles [kb, kb + nkt) in nk steps of two (the last may hold one)
  const int kb = MODE == MODE_SPLIT ? (ks * KT) / P : 0;
  const int nkt = (MODE == MODE_SPLIT ? ((ks + 1) * KT) / P : KT) - kb;
  const int nk = (nkt + 1) >> 1;

  // pieces (1 KiB operand tiles) of this wave: of a two-load block tile `wave`,
  // both k tiles; of a one-load block tile wave / 2, k tile wave % 2 (a block of
  // 6 row tiles: two waves repeat the last tile)
  const char* ab = (const char*)(A + ((size_t)mt0 * KT + kb) * 512);
  const char* wb = (const char*)(Wp + ((size_t)nt0 * KT + kb) * 512);
  const int ta = NA == 2 ? min(wave, 2 * RI - 1) : wave >> 1;
  const int t0 = N0 == 2 ? wave : wave >> 1, t1 = N1 == 2 ? wave : wave >> 1;
  uint32_t ofs[4];
  ofs[0] = (uint32_t)min(ta, MT - 1 - mt0) * KT * 1024;
  ofs[1] = (uint32_t)min(2 * RI + ta, MT - 1 - mt0) * KT * 1024;
  ofs[2] = (uint32_t)min(t0, NT - 1 - nt0) * KT * 1024;
  ofs[3] = (uint32_t)min(4 * C0 + t1, NT - 1 - nt0) * KT * 1024;
  auto ask = [&](int k, auto blk_) {  // request block A0, A1, W0, W1 (0..3) of step k
    constexpr int blk = decltype(blk_)::value;
    constexpr int n = blk < 2 ? NA : (blk == 2 ? N0 : N1);
    const int tile = blk < 2 ? ta : (blk == 2 ? t0 : t1);
    bf16_t* dst = &Sg[k & 1][(blk < 2 ? OA[blk & 1] : OW[blk & 1]) +
                             (n == 2 ? 2 * tile : wave) * 512];
#pragma unroll
    for (int kt = 0; kt < n; ++kt)
      __builtin_amdgcn_global_load_lds(
          (const void*)((blk < 2 ? ab : wb) +
                        (size_t)min(2 * k + (n == 2 ? kt : wave & 1), nkt - 1) * 1024 + ofs[blk] +
                        lane * 16),
          (__attribute__((address_space(3))) void*)(dst + kt * 512), 16, 0, 0);
  };
  typedef std::integral_constant<int, 0> A0;
  typedef std::integral_constant<int, 1> A1;
  typedef std::integral_constant<int, 2> W0;
  typedef std::integral_constant<int, 3> W1;
  bf16x8 a[RI][2], w0[2][C0][2], w1[C1][2];
  auto rd_a = [&](int k, int h) {
    const bf16_t* s = &Sg[k & 1][OA[h] + wm * RI * 1024 + lane * 8];
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) a[i][kt] = ld_frag(s + (2 * i + kt) * 512);
  };
  auto rd_w0 = [&](int k, bf16x8 (&w)[C0][2]) {
    const bf16_t* s = &Sg[k & 1][OW[0] + wn * C0 * 1024 + lane * 8];
#pragma unroll
    for (int t = 0; t < C0; ++t)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) w[t][kt] = ld_frag(s + (2 * t + kt) * 512);
  };
  auto rd_w1 = [&](int k) {
    const bf16_t* s = &Sg[k & 1][OW[1] + wn * C1 * 1024 + lane * 8];
#pragma unroll
    for (int t = 0; t < C1; ++t)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) w1[t][kt] = ld_frag(s + (2 * t + kt) * 512);
  };
  f32x4 acc[2][RI][CT];  // [row half][row tile][column tile, part 0 first]
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int t = 0; t < CT; ++t) acc[h][i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 tot[MODE == MODE_FOLD ? 2 : 1][MODE == MODE_FOLD ? RI : 1][MODE == MODE_FOLD ? CT : 1];
  if constexpr (MODE == MODE_FOLD) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int t = 0; t < CT; ++t) tot[h][i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto barrier = [] {
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // the phase's wait (its LDS reads are in, all but the newest loads have
  // landed), barrier, matrix instructions, barrier
  // fold: -1 no part ends in this step, 0 / 1 before its first / second k tile
  auto mma = [&](auto hm_, auto wait_, auto part_, auto& w, bool second, int fold) {
    constexpr int hm = decltype(hm_)::value, c0 = decltype(part_)::value ? C0 : 0;
    constexpr int C = decltype(part_)::value ? C1 : C0, n = decltype(wait_)::value;
    auto ktile = [&](int kt) {
      if (MODE == MODE_FOLD && fold == kt) {
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
          for (int t = 0; t < C; ++t) {
            tot[hm][i][c0 + t] += acc[hm][i][c0 + t];
            acc[hm][i][c0 + t] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
      }
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int t = 0; t < C; ++t)
          acc[hm][i][c0 + t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][kt], a[i][kt],
                                                                       acc[hm][i][c0 + t], 0, 0, 0);
    };
    __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | ((n >> 4) << 14));
    barrier();
    __builtin_amdgcn_s_setprio(1);
    ktile(0);
    if (second) ktile(1);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    barrier();
  };
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    ask(k, W0{});
    ask(k, A0{});
    ask(k, W1{});
    ask(k, A1{});
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(NS));
  barrier();
  rd_w0(0, w0[0]);
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  barrier();
  if (wm) barrier();
  int ending = 0, ends = MODE == MODE_FOLD ? KT / P : 0;  // the part whose end is next
  auto step = [&](int k, auto par) {
    constexpr int p = decltype(par)::value;
    std::integral_constant<int, NS + NA + N0> wait0;
    std::integral_constant<int, NS + NA + N1> wait1;
    std::integral_constant<int, 0> I0;
    std::integral_constant<int, 1> I1;
    const bool second = 2 * k + 1 < nkt;
    const int fold = MODE == MODE_FOLD && (ends >> 1) == k ? ends & 1 : -1;
    if (fold >= 0) {
      ++ending;
      ends = ((ending + 1) * KT) / P;  // the last part's end is past the last step
    }
    rd_a(k, 0);
    ask(k + 2, W0{});
    mma(I0, wait0, I0, w0[p], second, fold);
    rd_w1(k);
    ask(k + 2, A0{});
    mma(I0, wait0, I1, w1, second, fold);
    rd_a(k, 1);
    ask(k + 2, W1{});
    mma(I1, wait1, I1, w1, second, fold);
    rd_w0(k + 1, w0[p ^ 1]);
    ask(k + 2, A1{});
    mma(I1, wait1, I0, w0[p], second, fold);
  };
  for (int k = 0; k < nk; k += 2) {
    step(k, std::integral_constant<int, 0>{});
    if (k + 1 < nk) step(k + 1, std::integral_constant<int, 1>{});
  }
  if (!wm) barrier();
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // the re-read steps have landed too

  if constexpr (MODE == MODE_FOLD) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[h][i][t] = tot[h][i][t] + acc[h][i][t];
  }
  float* pk = part + (size_t)ks * M * N;
  auto put = [&](float* dst, f32x4 v) {  // vec: dst is 16-byte aligned
    if (vec) {
      *(f32x4*)dst = v;
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) dst[u] = v[u];
    }
  };
#pragma unroll
  for (int hm = 0; hm < 2; ++hm)
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const int mt = mt0 + (2 * hm + wm) * RI + i;
      const int m = mt * 16 + (lane & 15);
      if (m >= M) continue;
      if (EPI == EPI_SWIGLU) {
        // rows 0..7 of a W tile are gates (lanes 0..31), 8..15 ups (lanes
        // 32..63): exchanging halves between two tiles gives every lane four
        // gates and their ups (of a single tile: the lower lanes)
        auto store = [&](int nt, bool ok, f32x4 x, f32x4 y) {
          float s4[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[v]),
                                                             __float_as_uint(y[v]), false, false);
            s4[v] = silu_mul(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
          }
          if (!ok) return;
          const int c = nt * 8 + 4 * ((lane >> 4) & 1);
          *(uint2*)(ohi + act_off(m, c, okt)) =
              make_uint2((uint32_t)f2bf(s4[0]) | ((uint32_t)f2bf(s4[1]) << 16),
                         (uint32_t)f2bf(s4[2]) | ((uint32_t)f2bf(s4[3]) << 16));
        };
        auto part_out = [&](int ntp, auto c0_, auto n_) {
          constexpr int c0 = decltype(c0_)::value, n = decltype(n_)::value;
          if constexpr (n == 2) {
            const int nt = ntp + (lane >> 5);
            store(nt, nt < NT, acc[hm][i][c0], acc[hm][i][c0 + 1]);
          } else {
            store(ntp, lane < 32 && ntp < NT, acc[hm][i][c0], acc[hm][i][c0]);
          }
        };
        part_out(nt0 + wn * C0, std::integral_constant<int, 0>{}, std::integral_constant<int, C0>{});
        part_out(nt0 + 4 * C0 + wn * C1, std::integral_constant<int, C0>{},
                 std::integral_constant<int, C1>{});
      } else {
#pragma unroll
        for (int t = 0; t < CT; ++t) {
          const int nt = nt0 + (t < C0 ? wn * C0 + t : 4 * C0 + wn * C1 + t - C0);
          if (nt >= NT) continue;
          const int n = nt * 16 + 4 * (lane >> 4);
          f32x4 v = acc[hm][i][t];
          if (MODE == MODE_SPLIT) {
            *(f32x4*)(pk + (size_t)m * N + n) = v;
          } else {
            if (EPI == EPI_RESID) {
              const float* r = res + (size_t)m * ldres + n;
              if (vec) {
                v = *(const f32x4*)r + v;
              } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = r[u] + v[u];
              }
            }
            put(out + (size_t)m * ldo + n, v);
          }
        }
      }
    }
}

// four floats at any float's address (callers' logits and rows)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// out[m][n] = (res[m][n] +) sum over ks in order of part[ks][m][n]; N % 4 == 0
template <int EPI>
__global__ __launch_bounds__(256) void k_splitk_reduce(int M, int N, int SK,
                                                       const float* __restrict__ part,
                                                       float* out, int ldo, const float* res,
                                                       int ldres) {
  const size_t i4 = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int n4 = N >> 2;
  if (i4 >= (size_t)M * n4) return;
  const int m = (int)(i4 / n4), n = (int)(i4 % n4) * 4;
  f32x4 s = *(const f32x4*)&part[(size_t)m * N + n];
  for (int k = 1; k < SK; ++k) s += *(const f32x4*)&part[((size_t)k * M + m) * N + n];
  if (EPI == EPI_RESID) s = *(const f32x4_any*)&res[(size_t)m * ldres + n] + s;
  *(f32x4_any*)&out[(size_t)m * ldo + n] = s;
}

// Parts of the K sum of a product over `rows` rows (see k_gemm_wide).  They set
// the result's bits, so they follow the sizes alone and are kept apart from the
// tile shape and from how many rows a launch holds: a prefill pass over several
// chunks, or another tile, gives the bits of one chunk at a time.  The rule stands
// for these bits and not for speed: it splits K while the rows leave CUs idle, by
// the costs of a kernel of 128 x 256 tiles, two workgroups per CU and three ring
// stages, that k_gemm_wide has replaced (us per 32-wide k step with a CU alone and
// shared, per split launch, and bytes per us).  Counts by k_gemm_wide's own costs
// would take 12.0 ms instead of 12.5 for 8192 tokens in chunks of 512 through two
// layers, and 5% off a selection, at other bits: decisions of a selection that hang
// on near ties move with them.
static int gemm_parts(const GemmArgs& g) {
  constexpr double T_ALONE = 0.57, T_SHARED = 0.97, T_LAUNCH = 3.0, BYTES_PER_US = 4.5e6;
  if (g.epi == EPI_SWIGLU || !g.part) return 1;
  const int rows = g.part_rows ? g.part_rows : g.M, KT = g.K / 32;
  const int tiles = ((rows + 127) / 128) * ((g.N / 16 + 15) / 16);
  const int cus = compute_units();
  const int resident = 2 * cus;
  double best = 0.0;
  int best_sk = 1;
  for (int sk = 1; sk <= 8; ++sk) {
    if (sk > 1 && ((size_t)sk * rows * g.N * 4 > g.part_bytes || KT / sk < 8)) break;
    const int steps = (KT + sk - 1) / sk;
    double t = 0.0;
    for (long left = (long)tiles * sk; left > 0; left -= resident)
      t += steps * (std::min<long>(left, resident) > cus ? T_SHARED : T_ALONE);
    if (sk > 1) t += T_LAUNCH + (sk + 2.0) * rows * (double)g.N * 4.0 / BYTES_PER_US;
    if (sk == 1 || t < best) {
      best = t;
      best_sk = sk;
    }
  }
  return best_sk;
}

// Tile shapes of k_gemm_wide and their cost on MI355X, fitted to 11 row counts
// (100..4096) x the four Llama-8B product shapes x every split factor: us per
// k step of 64 while more than one workgroup per CU (at most 80 KiB of LDS) or
// every CU is busy (full) and in a last round of at most one workgroup per CU
// (alone), and us per round.  A launch costs WIDE_LAUNCH, a split WIDE_SPLIT and
// P + 2 float32 planes at WIDE_BYTES per us: above the memory's rate, as the
// partials (at most 128 MiB) are summed out of the last-level cache.  One row tile
// whose weights stream through that cache (WIDE_LLC) evicts them and pays MEM_SPLIT
// and MEM_BYTES.  Folding the parts in the workgroup costs no traffic but needs a
// second set of accumulators, so only the 128 x 256 tile does it.  The split's costs
// are fitted to 310 split products (17..1200 rows, 4096..200064 columns, K 1024..8192),
// where the pick is within 0.7% of the best form on average and 8% at worst; with
// the memory's rate for all of them it folded too soon (1.4% and 17%), with the
// cache's too late (1.5% and 16%).  512 rows by 6144 columns of 2048 (the head call)
// 66.7 -> 59.2 us, 1200 by 4096 of 4096 118 -> 105; both sublayers on 700 / 1152 /
// 1390 candidate rows 468 -> 449 / 684 -> 622 / 836 -> 774 us (Qwen, Qwen, Llama).
struct WideShape {
  int ri, c0, c1;
  double full, alone, round;
};
static constexpr WideShape WIDE[] = {
    {2, 1, 1, 0.916, 0.609, 0.67},
    {2, 2, 2, 0.844, 0.675, 2.27},
    {3, 2, 2, 1.100, 0.836, 3.35},
    {4, 2, 2, 1.375, 1.023, 4.55},
};
struct WidePick {
  int shape, mode;
};
static WidePick wide_pick(const GemmArgs& g, int P) {
  constexpr double WIDE_LAUNCH = 4.8, WIDE_SPLIT = 1.0, WIDE_BYTES = 10e6;
  constexpr double MEM_SPLIT = 2.2, MEM_BYTES = 4.9e6;
  constexpr size_t WIDE_LLC = (size_t)256 << 20;
  const bool cached = g.M > 128 || (size_t)g.N * g.K * 2 <= WIDE_LLC;
  const int cus = compute_units();
  WidePick best{-1, MODE_ONE};
  // One row tile by more than a round of 128 x 128 tiles (a vocabulary): bound by
  // the weight stream, which the costs above do not hold.  Two workgroups per CU
  // that start and end apart keep it going, if their last round puts no more than
  // one on a CU or, as the second round, nearly fills it: final norm, head and argmax
  // of 17 / 64 / 96 / 128 rows 229 / 239 / 250 / 263 us at 128256 columns of 4096
  // (1002 tiles) against 233 / 250 / 260 / 272 in 128 x 256 tiles; 96 rows by 151936
  // columns (1187 tiles) 293 against 320.  With half to 4/5 of a round left (100352
  // to 110592 columns) or in later rounds (180224, 256000) some CUs stream two tiles
  // and others one: 5 to 10% and 1 to 5% the other way.
  if (P == 1 && g.M <= 128) {
    const int tiles = (g.N / 16 + 7) / 8, last = (tiles - 1) % (2 * cus) + 1;
    if (tiles > 2 * cus && (last <= cus || (tiles < 4 * cus && 5 * last >= 8 * cus)))
      return WidePick{0, MODE_ONE};
  }
  double tb = 0.0;
  for (int i = 0; i < 4; ++i) {
    const WideShape& w = WIDE[i];
    const long tiles = (long)((g.M + 64 * w.ri - 1) / (64 * w.ri)) *
                       ((g.N / 16 + 4 * (w.c0 + w.c1) - 1) / (4 * (w.c0 + w.c1)));
    const int resident = cus * (16 * w.ri + 16 * (w.c0 + w.c1) <= 80 ? 2 : 1);
    for (int mode = P > 1 ? MODE_SPLIT : MODE_ONE; mode <= (P > 1 ? MODE_FOLD : MODE_ONE); ++mode) {
      if (mode == MODE_SPLIT && (size_t)P * g.M * g.N * 4 > g.part_bytes) continue;
      if (mode == MODE_FOLD && i != 1) continue;
      const int steps = ((mode == MODE_SPLIT ? (g.K / 32 + P - 1) / P : g.K / 32) + 1) / 2;
      double t = WIDE_LAUNCH;
      for (long left = mode == MODE_SPLIT ? tiles * P : tiles; left > 0; left -= resident)
        t += w.round + steps * (left >= resident || left > cus ? w.full : w.alone);
      if (mode == MODE_SPLIT)
        t += (cached ? WIDE_SPLIT : MEM_SPLIT) +
             (P + 2.0) * g.M * (double)g.N * 4.0 / (cached ? WIDE_BYTES : MEM_BYTES);
      if (best.shape < 0 || t < tb) {
        tb = t;
        best = WidePick{i, mode};
      }
    }
  }
  return best;
}

template <int EPI, int MODE, int RI, int C0, int C1>
static void launch_wide(const GemmArgs& g, int P, hipStream_t st) {
  const int MB = (g.M + 64 * RI - 1) / (64 * RI);
  const int NB = (g.N / 16 + 4 * (C0 + C1) - 1) / (4 * (C0 + C1));
  const dim3 grid((unsigned)MB * NB * (MODE == MODE_SPLIT ? P : 1));
  // outputs and residuals of any float alignment (callers' logits and rows)
  const int vec = (((uintptr_t)g.out | (uintptr_t)g.res) & 15) == 0 && g.ldo % 4 == 0 &&
                  g.ldres % 4 == 0;
  KS_LAUNCH((k_gemm_wide<EPI, MODE, RI, C0, C1>), grid, dim3(512), 0, st, g.M, g.N, g.K,
            (const bf16_t*)g.A.hi, (const bf16_t*)g.W, g.out, g.ldo, g.res, g.ldres,
            (bf16_t*)g.act_out.hi, g.act_out.kt, MB, NB, P, vec, g.part);
}

template <int EPI>
static void launch_epi(const GemmArgs& g, hipStream_t st) {
  const int P = gemm_parts(g);
  const WidePick w = wide_pick(g, P);
  if constexpr (EPI != EPI_SWIGLU) {
    if (w.mode == MODE_FOLD) return launch_wide<EPI, MODE_FOLD, 2, 2, 2>(g, P, st);
    if (w.mode == MODE_SPLIT) {
      switch (w.shape) {
        case 0: launch_wide<EPI, MODE_SPLIT, 2, 1, 1>(g, P, st); break;
        case 1: launch_wide<EPI, MODE_SPLIT, 2, 2, 2>(g, P, st); break;
        case 2: launch_wide<EPI, MODE_SPLIT, 3, 2, 2>(g, P, st); break;
        default: launch_wide<EPI, MODE_SPLIT, 4, 2, 2>(g, P, st); break;
      }
      const size_t n4 = (size_t)g.M * (g.N / 4);
      KS_LAUNCH(k_splitk_reduce<EPI>, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, g.M,
                g.N, P, g.part, g.out, g.ldo, g.res, g.ldres);
      return;
    }
  }
  switch (w.shape) {
    case 0: launch_wide<EPI, MODE_ONE, 2, 1, 1>(g, P, st); break;
    case 1: launch_wide<EPI, MODE_ONE, 2, 2, 2>(g, P, st); break;
    case 2: launch_wide<EPI, MODE_ONE, 3, 2, 2>(g, P, st); break;
    default: launch_wide<EPI, MODE_ONE, 4, 2, 2>(g, P, st); break;
  }
}

void gemm_bf16_tiled(const GemmArgs& g, hipStream_t st) {
  if (g.epi == EPI_SWIGLU) launch_epi<EPI_SWIGLU>(g, st);
  else if (g.epi == EPI_RESID) launch_epi<EPI_RESID>(g, st);
  else launch_epi<EPI_STORE>(g, st);
}

// --------------------------------------------------------------------- f32
// float32 models: 16 x 16 outputs per workgroup of eight waves, on the float32
// matrix instruction (16x16x4, float32 products and sums).  Wave w takes the
// 16-wide k groups [w KG / 8, (w + 1) KG / 8), four instructions per group, and
// the eight partial sums are added in wave order, so a row's result does not
// depend on the other rows.  Both operands go straight to registers: lane
// (j, g) loads k 16 s + 4 g .. + 3 of row j, and instruction e of a group takes
// element e of every lane.  These products are bound by latency: at 5 rows the
// down projection of the tiny decoder (K = 1024, 16 workgroups) spent 31 us in 64
// dependent rounds of load, barrier and 16 multiply-adds; now all of a wave's
// loads are in flight together: 5 us (gate/up 12 -> 5, q/k/v 9.4 -> 4).
// vec: the weights are 16-byte aligned.
// EPI_SWIGLU: W is [gate rows; up rows], Nout = N/2 outputs.  Nout % 16 == 0,
// K % 16 == 0.
constexpr int F32_NW = 8;
template <int EPI>
__global__ __launch_bounds__(64 * F32_NW) void k_gemm_f32(int M, int Nout, int K,
                                                          const float* __restrict__ A, int lda,
                                                          const float* __restrict__ W, float* out,
                                                          int ldo, const float* res, int ldres,
                                                          float* aout, int ldact, int vec) {
  constexpr int NW = F32_NW, U = 4, NP = EPI == EPI_SWIGLU ? 2 : 1;
  __shared__ f32x4 red[NP][NW][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
  const int KG = K >> 4;
  const int kb = (wave * KG) / NW, ke = ((wave + 1) * KG) / NW;
  const float* src[1 + NP];  // row m0 + j of A (clamped: rows past M are not stored), of W
  src[0] = A + (size_t)min(m0 + j, M - 1) * lda + 4 * g;
#pragma unroll
  for (int p = 0; p < NP; ++p) src[1 + p] = W + (size_t)(p * Nout + n0 + j) * K + 4 * g;
  auto load = [&](const float* p) {
    if (vec) return *(const f32x4*)p;
    return f32x4{p[0], p[1], p[2], p[3]};
  };
  f32x4 acc[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) acc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k = kb; k < ke; k += U) {
    f32x4 x[1 + NP][U];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int p = 0; p <= NP; ++p) x[p][u] = load(src[p] + 16 * min(k + u, ke - 1));
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + u < ke) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int p = 0; p < NP; ++p)
            acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0][u][e], x[1 + p][u][e], acc[p], 0, 0, 0);
      }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) red[p][wave][lane] = acc[p];
  __syncthreads();
  // thread: lane l, register v of the result tile (row 4 (l / 16) + v, column l % 16)
  const int l = threadIdx.x >> 2, v = threadIdx.x & 3;
  const int m = m0 + 4 * (l >> 4) + v, n = n0 + (l & 15);
  if (l >= 64 || m >= M) return;
  float s[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    s[p] = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) s[p] += red[p][w][l][v];
  }
  if (EPI == EPI_SWIGLU) {
    aout[(size_t)m * ldact + n] = silu_mul(s[0], s[NP - 1]);
  } else {
    if (EPI == EPI_RESID) s[0] += res[(size_t)m * ldres + n];
    out[(size_t)m * ldo + n] = s[0];
  }
}

void gemm_f32(const GemmArgs& g, hipStream_t st) {
  const int Nout = g.epi == EPI_SWIGLU ? g.N / 2 : g.N;
  const dim3 grid(Nout / 16, (g.M + 15) / 16), block(64 * F32_NW);
  const float* A = (const float*)g.A.hi;
  const float* W = (const float*)g.W;
  const int vec = (((uintptr_t)A | (uintptr_t)W) & 15) == 0 && g.A.ld % 4 == 0;
  if (g.epi == EPI_SWIGLU)
    KS_LAUNCH(k_gemm_f32<EPI_SWIGLU>, grid, block, 0, st, g.M, Nout, g.K, A, g.A.ld, W, g.out,
              g.ldo, g.res, g.ldres, (float*)g.act_out.hi, g.act_out.ld, vec);
  else if (g.epi == EPI_RESID)
    KS_LAUNCH(k_gemm_f32<EPI_RESID>, grid, block, 0, st, g.M, Nout, g.K, A, g.A.ld, W, g.out,
              g.ldo, g.res, g.ldres, nullptr, 0, vec);
  else
    KS_LAUNCH(k_gemm_f32<EPI_STORE>, grid, block, 0, st, g.M, Nout, g.K, A, g.A.ld, W, g.out,
              g.ldo, g.res, g.ldres, nullptr, 0, vec);
}

// ----------------------------------------------------------------- packing
// One thread per 8-element (16-byte) fragment of the destination.
// mode 0: plain; 1: gate/up 8 + 8 interleave; 2: q/k/v heads of hd rows with
// tile t of a head holding rows 8t..8t+7 and hd/2 + 8t..hd/2 + 8t + 7
__global__ void k_pack(const bf16_t* __restrict__ src0, const bf16_t* __restrict__ src1,
                       bf16_t* __restrict__ dst, int N, int K, int mode, int hd) {
  const size_t f = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int KT = K >> 5;
  const size_t nfrag = (size_t)N * K / 8;
  if (f >= nfrag) return;
  const int l = (int)(f & 63);
  const size_t tile = f >> 6;
  const int kt = (int)(tile % KT);
  const int nt = (int)(tile / KT);
  const bf16_t* src = src0;
  int row = nt * 16 + (l & 15);
  if (mode == 1) {  // tile t: gate rows 8t..8t+7, then up rows 8t..8t+7
    src = (l & 8) ? src1 : src0;
    row = nt * 8 + (l & 7);
  } else if (mode == 2) {
    const int tph = hd / 16, h = nt / tph, t = nt % tph;
    row = h * hd + 8 * t + (l & 7) + (hd / 2) * ((l >> 3) & 1);
  }
  const u32x4 v = *(const u32x4*)(src + (size_t)row * K + kt * 32 + (l >> 4) * 8);
  *(u32x4*)(dst + f * 8) = v;
}

void pack_matrix_bf16(const bf16_t* src, bf16_t* dst, int N, int K, hipStream_t st) {
  const size_t nfrag = (size_t)N * K / 8;
  KS_LAUNCH(k_pack, dim3((unsigned)((nfrag + 255) / 256)), dim3(256), 0, st, src,
            nullptr, dst, N, K, 0, 0);
}

void pack_qkv_bf16(const bf16_t* src, bf16_t* dst, int heads, int hd, int d, hipStream_t st) {
  const size_t nfrag = (size_t)heads * hd * d / 8;
  KS_LAUNCH(k_pack, dim3((unsigned)((nfrag + 255) / 256)), dim3(256), 0, st, src,
            nullptr, dst, heads * hd, d, 2, hd);
}

void pack_gate_up_bf16(const bf16_t* gate, const bf16_t* up, bf16_t* dst, int ffn, int d,
                       hipStream_t st) {
  const size_t nfrag = (size_t)2 * ffn * d / 8;
  KS_LAUNCH(k_pack, dim3((unsigned)((nfrag + 255) / 256)), dim3(256), 0, st, gate, up,
            dst, 2 * ffn, d, 1, 0);
}

}  // namespace ks
