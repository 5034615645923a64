// Projections of 17 to 64 rows: one row tile of MG = 4 16-row groups, a workgroup
// per 64, 128 or 256 output columns, eight waves as WM (rows) x WN (columns).
//
// What bounds it: the weight stream, and what a compute unit takes in.  Each
// workgroup reads its weight columns once from memory and the whole of X from
// the L2, so it moves MG + columns / 16 KiB per K step at about 40-45 GB/s; a
// layout is good when the launch is one full round of compute units and that
// sum is small (plan_tiled).  Against k_gemm's staged layout (X through LDS by
// a ninth wave, weights in registers, K split over the waves of a workgroup):
//  * both operands are copied straight into LDS, kLead chunks of two K steps
//    ahead and by all eight waves, so the stream runs at the depth of the LDS
//    ring whatever the registers hold, and no wave is set aside to load;
//  * the copies are issued from asm: tracked loads into LDS would be drained
//    before every LDS read.  They write no registers.  Loads complete in issue
//    order, so a wave knows its copies of a chunk have landed when no more are
//    outstanding than it has issued since; the barrier then hands the chunk
//    to all waves;
//  * every wave multiplies the whole K range of its own tiles: no reduction
//    across waves and no second pass over LDS; even and odd K steps are summed
//    apart, so a sum is no longer than one of the staged layout's, where two
//    waves halve K (float32 sums of 37 rows, K of 4096, relative distance from
//    a 64-bit product: 4.0e-7 in one sum, 2.7e-7 in two and in the staged
//    layout; no time difference);
//  * the fragments of the next half step are read while the current one
//    multiplies, also across the barrier.
// Measured (cold weights, us, staged -> here): gate/up 28672 x 4096 at 64 rows
// 47.4 -> 39.5, 37 rows 44.6 -> 38.3; 16384 x 3072 at 64 rows 20.1 -> 18.9;
// down 4096 x 14336 at 37 rows 25.0 -> 20.8; a head of 32000 x 4096 at 37 rows
// 62.3 -> 42.7.  A pure read of 28672 x 4096 takes 37.5.  At 65 to 128 rows (8
// row groups) the same kernel was no faster (gate/up 53.7 against 51.8, head of
// 128256 x 4096 204 against 198 in the pass), so they keep the staged layout.
#include <algorithm>
#include <climits>

#include <hip/hip_ext.h>

#include "dev.hpp"
#include "gemm.hpp"
#include "gemm_epi.hpp"

namespace vsk {

// 16 bytes per lane from base + voff (bytes) into LDS at lds + 16 * lane.  (M0,
// which takes the LDS address, is a register the compiler never allocates and
// uses for nothing else here.)
template <bool NT>
__device__ __forceinline__ void lds_copy16(const void* base, uint32_t voff, uint32_t lds) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :
                 : "v"(voff), "s"(base), "s"(lds)
                 : "memory");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff), "s"(base), "s"(lds)
                 : "memory");
}

constexpr int kChunk = 2;  // K steps per chunk (every K here is a multiple of 64)
// Chunks of a tile's fragments held in LDS: at most 144 KiB, at most four
constexpr int tiled_buffers(int mg, int tn) {
  const int fit = 144 / (kChunk * (mg + tn));
  return fit < 4 ? fit : 4;
}

template <int WM, int MG, int NT, int EPI>
__global__ __launch_bounds__(512, 2) void k_gemm_tiled(GemmArgs a) {
  constexpr int WN = 8 / WM;
  constexpr int TN = WN * NT;              // column tiles of the macro tile
  constexpr int MGW = MG / WM;             // row groups of a wave
  constexpr int kBuf = tiled_buffers(MG, TN);
  constexpr int kLead = kBuf - 1;          // chunks copied ahead
  constexpr int kStep = MG + TN;           // 1 KiB fragments per K step
  constexpr int kPieces = kChunk * kStep;  // and per chunk
  constexpr int kCopies = kPieces / 8;     // copies per wave and chunk
  constexpr int XB = MGW / 2;              // row groups of a half step
  static_assert(kPieces % 8 == 0 && MG % WM == 0 && MGW % 2 == 0, "pieces and row groups in equal shares");
  static_assert(kBuf >= 2 && (kLead - 1) * kCopies <= 63, "outstanding loads beyond the wait counter");
  extern __shared__ __align__(16) unsigned char smem[];  // [kBuf][kChunk][MG X pieces, TN W pieces][1 KiB]
  __shared__ float s_amv[EPI == EPI_LOGITS ? WN : 1][MG][16];
  __shared__ int s_ami[EPI == EPI_LOGITS ? WN : 1][MG][16];
  __shared__ double s_ss[EPI == EPI_RESID ? WN : 1][MG][16];

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = w % WN, wm = w / WN;
  const int ng = blockIdx.x, ks = blockIdx.y;
  const int Rv = a.count != nullptr ? min(a.R, *a.count) : a.R;
  if (Rv <= 0) return;  // (uniform) an empty cohort
  const int n_tiles = a.N >> 4;
  const bool split_out = EPI == EPI_RESID && a.ypart != nullptr;
  const int nt0 = (ng * WN + wn) * NT;
  const int gw = wm * MGW;  // this wave's first row group
  const int rsub = lane & 15;
  const int nq = 4 * (lane >> 4);

  // K steps [k_lo, k_hi): every split is a whole number of chunks
  const int kc = (a.Kt / kChunk + gridDim.y - 1) / gridDim.y * kChunk;
  const int k_lo = ks * kc, k_hi = min(a.Kt, k_lo + kc);
  const int n_chunks = (k_hi - k_lo) / kChunk;

  // one sum per step of a chunk, added at the end (the head's logits, rounded
  // to bf16, keep one: so they had in the staged layout)
  constexpr int kSums = EPI == EPI_LOGITS ? 1 : kChunk;
  f32x4 sums[kSums][NT][MGW];
#pragma unroll
  for (int st = 0; st < kSums; ++st)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int g = 0; g < MGW; ++g) sums[st][j][g] = f32x4{0.f, 0.f, 0.f, 0.f};

  // This wave's copies of chunk c: pieces w, w + 8, ...; in each K step X
  // pieces first, then W.  Row groups and column tiles past the end copy a
  // valid one (their sums are never stored), chunks past the last one copy
  // the last.
  const uint32_t lds0 =
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)smem));
  auto copy = [&](int c) {
    const int kt = k_lo + min(c, n_chunks - 1) * kChunk;
    const uint32_t dst = lds0 + static_cast<uint32_t>((c % kBuf) * kPieces + w) * 1024;
    const uint32_t voff = static_cast<uint32_t>(lane) * 16;
#pragma unroll
    for (int p = 0; p < kCopies; ++p) {
      const int pc = w + 8 * p;
      const int st = pc / kStep, q = pc % kStep;
      if (q < MG)
        lds_copy16<false>(a.X + (static_cast<size_t>(kt + st) * a.Rg + min(q, a.Rg - 1)) * 64, voff, dst + p * 8192);
      else
        lds_copy16<true>(
            a.W + (static_cast<size_t>(min(ng * TN + q - MG, n_tiles - 1)) * w_stride(a.Kt) + kt + st) * 64, voff,
            dst + p * 8192);
    }
  };
  // wait until this wave's copies of all but the newest kLead - 1 chunks have landed
  auto wait_copies = [&]() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kLead - 1) * kCopies) : "memory");
  };
  const u32x4* xs = reinterpret_cast<const u32x4*>(smem) + wm * MGW * 64 + lane;
  const u32x4* ws = reinterpret_cast<const u32x4*>(smem) + (MG + wn * NT) * 64 + lane;
  u32x4 xa[XB], xb[XB], wa[NT], wb[NT];
  // X fragments of the first (h = 0) or second half of a step's row groups
  auto xread = [&](u32x4 (&r)[XB], int c, int st, auto h_c) {
    constexpr int h = decltype(h_c)::value;
    const u32x4* p = xs + ((c % kBuf) * kPieces + st * kStep + h * XB) * 64;
#pragma unroll
    for (int g = 0; g < XB; ++g) r[g] = p[g * 64];
  };
  auto wread = [&](u32x4 (&r)[NT], int c, int st) {
    const u32x4* p = ws + ((c % kBuf) * kPieces + st * kStep) * 64;
#pragma unroll
    for (int j = 0; j < NT; ++j) r[j] = p[j * 64];
  };
  auto mma = [&](f32x4 (&acc)[NT][MGW], const u32x4 (&fw)[NT], const u32x4 (&r)[XB], auto h_c) {
    constexpr int h = decltype(h_c)::value;
#pragma unroll
    for (int g = 0; g < XB; ++g)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[j][h * XB + g] = mfma_16x16x32(fw[j], r[g], acc[j][h * XB + g]);
  };
  constexpr auto kH0 = std::integral_constant<int, 0>{};
  constexpr auto kH1 = std::integral_constant<int, 1>{};

#pragma unroll
  for (int i = 0; i < kLead; ++i) copy(i);
  wait_copies();  // chunk 0 has landed
  barrier_no_fence();
  wread(wa, 0, 0);
  xread(xa, 0, 0, kH0);

  // one K step: the second half's fragments are read while the first half
  // multiplies, the next step's first half while the second does; in a
  // chunk's last step the barrier between them publishes the next chunk and
  // frees this one's buffer (every wave's reads of it are done), which the
  // copy at the start of the next chunk then fills
  auto kstep = [&](int c, auto st_c, u32x4 (&wc)[NT], u32x4 (&wnx)[NT]) {
    constexpr int st = decltype(st_c)::value;
    if (st == 0) copy(c + kLead);
    xread(xb, c, st, kH1);
    __builtin_amdgcn_sched_barrier(0);
    mma(sums[st % kSums], wc, xa, kH0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (st == kChunk - 1) {
      wait_copies();
      barrier_after_lds_reads();
      wread(wnx, c + 1, 0);
      xread(xa, c + 1, 0, kH0);
    } else {
      wread(wnx, c, st + 1);
      xread(xa, c, st + 1, kH0);
    }
    __builtin_amdgcn_sched_barrier(0);
    mma(sums[st % kSums], wc, xb, kH1);
    __builtin_amdgcn_sched_barrier(0);
  };
  static_assert(kChunk == 2, "two weight fragment sets, one per step of a chunk");
  for (int c = 0; c < n_chunks; ++c) {
    kstep(c, kH0, wa, wb);
    kstep(c, kH1, wb, wa);
  }
  // the copies past the last step must land before the workgroup ends
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  f32x4 (&acc)[NT][MGW] = sums[0];
  if constexpr (kSums > 1) {
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int g = 0; g < MGW; ++g) acc[j][g] += sums[1][j][g];
  }

  // ---- epilogues
  if constexpr (EPI == EPI_RESID) {
    if (split_out) {
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int g = 0; g < MGW; ++g) {
          const int row = 16 * (gw + g) + rsub;
          if (nt0 + j >= n_tiles || row >= Rv) continue;
          const int n0 = 16 * (nt0 + j) + nq;
          *reinterpret_cast<f32x4*>(a.ypart + (static_cast<size_t>(ks) * a.R + row) * a.N + n0) = acc[j][g];
        }
      return;
    }
    // x += y; this workgroup's share of sum x^2 per row.  A row group's
    // residual is loaded one group ahead of its use.
    float4 xv[2][NT];
    auto xload = [&](float4 (&r)[NT], int g) {
      const int row = 16 * (gw + g) + rsub;
#pragma unroll
      for (int j = 0; j < NT; ++j)
        r[j] = (nt0 + j < n_tiles && row < Rv)
                   ? *reinterpret_cast<const float4*>(a.x + static_cast<size_t>(row) * a.N + 16 * (nt0 + j) + nq)
                   : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    xload(xv[0], 0);
#pragma unroll
    for (int g = 0; g < MGW; ++g) {
      if (g + 1 < MGW) xload(xv[(g + 1) & 1], g + 1);
      const int row = 16 * (gw + g) + rsub;
      double ss = 0.0;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if (nt0 + j >= n_tiles || row >= Rv) continue;
        float4 v = xv[g & 1][j];
        v.x += acc[j][g][0];
        v.y += acc[j][g][1];
        v.z += acc[j][g][2];
        v.w += acc[j][g][3];
        *reinterpret_cast<float4*>(a.x + static_cast<size_t>(row) * a.N + 16 * (nt0 + j) + nq) = v;
        ss += static_cast<double>(v.x) * v.x + static_cast<double>(v.y) * v.y + static_cast<double>(v.z) * v.z +
              static_cast<double>(v.w) * v.w;
      }
      // the four lane groups hold the same row
      ss += __shfl_xor(ss, 16, 64);
      ss += __shfl_xor(ss, 32, 64);
      if (lane < 16) s_ss[wn][wm * MGW + g][lane] = ss;
    }
    if (a.ssq_out != nullptr) {
      __syncthreads();
      for (int i = threadIdx.x; i < MG * 16; i += 512) {
        const int g = i >> 4, l = i & 15;
        double ss = s_ss[0][g][l];
#pragma unroll
        for (int w2 = 1; w2 < WN; ++w2) ss += s_ss[w2][g][l];
        const int row = 16 * g + l;
        if (row < Rv) a.ssq_out[static_cast<size_t>(row) * gridDim.x + ng] = ss;  // [row][workgroup]
      }
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if (nt0 + j >= n_tiles) continue;
      const int u = 4 * (nt0 + j) + (lane >> 4);  // output columns 2u, 2u+1
#pragma unroll
      for (int g = 0; g < MGW; ++g) {
        const int row = 16 * (gw + g) + rsub;
        if (row >= Rv) continue;
        const float a0 = silu_f(acc[j][g][0]) * acc[j][g][2];
        const float a1 = silu_f(acc[j][g][1]) * acc[j][g][3];
        *reinterpret_cast<uint32_t*>(a.out + frag_index(row, 2 * u, a.out_Rg)) = pack_bf2(a0, a1);
      }
    }
  } else if constexpr (EPI == EPI_QKV) {
    const int half = a.hd >> 1;
    int q_slot[MGW], q_pos[MGW];
#pragma unroll
    for (int g = 0; g < MGW; ++g) {
      const int row = 16 * (gw + g) + rsub;
      q_slot[g] = row < Rv ? a.slot[row] : 0;
      q_pos[g] = row < Rv ? a.pos[row] : 0;
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if (nt0 + j >= n_tiles) continue;
      const int n0 = 16 * (nt0 + j) + nq;
      const int j0 = (n0 % a.hd) >> 1;
      const bool rot = n0 < a.Nq + a.Nkv;
      // the rotary factors of all the wave's rows before the first store
      float4 cs[MGW];
#pragma unroll
      for (int g = 0; g < MGW; ++g)
        cs[g] = rot ? *reinterpret_cast<const float4*>(a.rope + static_cast<size_t>(q_pos[g]) * half + j0)
                    : make_float4(1.f, 0.f, 1.f, 0.f);
#pragma unroll
      for (int g = 0; g < MGW; ++g) {
        const int row = 16 * (gw + g) + rsub;
        if (row >= Rv) continue;
        qkv_store(a, row, n0, acc[j][g], q_slot[g], make_float2(cs[g].x, cs[g].y), make_float2(cs[g].z, cs[g].w));
      }
    }
  } else if constexpr (EPI == EPI_LOGITS) {
#pragma unroll
    for (int g = 0; g < MGW; ++g) {
      const int row = 16 * (gw + g) + rsub;
      float bv = -INFINITY;
      int bi = INT_MAX;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if (nt0 + j >= n_tiles || row >= Rv) continue;
        const int n0 = 16 * (nt0 + j) + nq;
        const f32x4 v = acc[j][g];
        uint2 packed;
        packed.x = pack_bf2(v[0], v[1]);
        packed.y = pack_bf2(v[2], v[3]);
        *reinterpret_cast<uint2*>(a.out + static_cast<size_t>(row) * a.N + n0) = packed;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (!(v[r] != v[r])) am_merge(bv, bi, v[r], n0 + r);
      }
#pragma unroll
      for (int m = 16; m <= 32; m <<= 1) {  // lanes l, l^16, l^32, l^48 hold the same row
        const float v2 = shfl_xor(bv, m);
        const int i2 = shfl_xor(bi, m);
        am_merge(bv, bi, v2, i2);
      }
      if (lane < 16) {
        s_amv[wn][wm * MGW + g][lane] = bv;
        s_ami[wn][wm * MGW + g][lane] = bi;
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < MG * 16; i += 512) {
      const int g = i >> 4, l = i & 15;
      float bv = s_amv[0][g][l];
      int bi = s_ami[0][g][l];
#pragma unroll
      for (int w2 = 1; w2 < WN; ++w2) am_merge(bv, bi, s_amv[w2][g][l], s_ami[w2][g][l]);
      const int row = 16 * g + l;
      if (row < Rv) {
        a.am_val[static_cast<size_t>(ng) * a.R + row] = bv;
        a.am_idx[static_cast<size_t>(ng) * a.R + row] = bi;
      }
    }
  }
}

template <int WM, int MG, int NT, int EPI>
static hipError_t launch_tiled_cfg(const GemmArgs& a, int ksplit, hipStream_t s, const LaunchEvents& ev) {
  constexpr int TN = 8 / WM * NT;
  const dim3 grid((a.N / 16 + TN - 1) / TN, ksplit), block(512);
  constexpr size_t smem = static_cast<size_t>(tiled_buffers(MG, TN)) * kChunk * (MG + TN) * 1024;
  // with the static arrays this can be more than 64 KiB of LDS: allow it once
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_tiled<WM, MG, NT, EPI>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem));
  if (attr != hipSuccess) return attr;
  if (ev.start != nullptr || ev.stop != nullptr)  // events bound to this dispatch
    hipExtLaunchKernelGGL((k_gemm_tiled<WM, MG, NT, EPI>), grid, block, static_cast<uint32_t>(smem), s, ev.start,
                          ev.stop, 0u, a);
  else
    hipLaunchKernelGGL((k_gemm_tiled<WM, MG, NT, EPI>), grid, block, smem, s, a);
  return hipGetLastError();
}

// 64 columns: 2 x 4 waves of one column tile; 128 and 256: the eight waves
// side by side with one and two
template <int EPI>
static hipError_t launch_tiled_epi(const GemmArgs& a, const GemmPlan& p, hipStream_t s, const LaunchEvents& ev) {
  if (a.Kt % kChunk != 0 || a.Rg > kTiledGroups || p.mg != kTiledGroups) return hipErrorInvalidValue;
  switch (p.nt * p.wn) {
    case 4: return launch_tiled_cfg<2, kTiledGroups, 1, EPI>(a, p.ksplit, s, ev);
    case 8: return launch_tiled_cfg<1, kTiledGroups, 1, EPI>(a, p.ksplit, s, ev);
    case 16:
      if constexpr (EPI != EPI_RESID) return launch_tiled_cfg<1, kTiledGroups, 2, EPI>(a, p.ksplit, s, ev);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_tiled(const GemmArgs& a, const GemmPlan& p, int epi, hipStream_t s, const LaunchEvents& ev) {
  switch (epi) {
    case EPI_RESID: return launch_tiled_epi<EPI_RESID>(a, p, s, ev);
    case EPI_QKV: return launch_tiled_epi<EPI_QKV>(a, p, s, ev);
    case EPI_SWIGLU: return launch_tiled_epi<EPI_SWIGLU>(a, p, s, ev);
    default: return launch_tiled_epi<EPI_LOGITS>(a, p, s, ev);
  }
}

GemmPlan plan_tiled(int N, int K, int R, int epi, int target) {
  const int Kt = K / 32;
  GemmPlan best;
  double best_cost = 0;
  for (const int tn : {4, 8, 16}) {  // 64, 128, 256 columns
    if (tn == 16 && epi == EPI_RESID) break;
    GemmPlan p;
    p.tiled = true;
    p.mg = kTiledGroups;
    p.wn = tn == 4 ? 4 : 8;
    p.nt = tn / p.wn;
    p.n_groups = (N / 16 + tn - 1) / tn;
    if (epi == EPI_RESID && target > 0) {
      // as many K splits as keep the launch within the target, K / splits at
      // least eight steps, every split a whole number of chunks (the last one
      // what is left)
      const int want = std::clamp(target / p.n_groups, 1, std::min(kMaxResidSplits, std::max(1, Kt / 8)));
      const int kc = (Kt / kChunk + want - 1) / want * kChunk;
      p.ksplit = (Kt + kc - 1) / kc;
    }
    const int rounds = (p.n_groups * p.ksplit + kComputeUnits - 1) / kComputeUnits;
    const double steps = static_cast<double>(Kt) / p.ksplit;
    // KiB through a compute unit, and the splits' products, written here and
    // read again by the kernel that adds them (a split of 64 x 5120 sums costs
    // as much as 66 KiB through every unit)
    const double cost = rounds * steps * (p.mg + tn) + (p.ksplit > 1 ? 2e-4 * p.ksplit * R * N : 0.0);
    if (best_cost == 0 || cost < best_cost) {
      best = p;
      best_cost = cost;
    }
  }
  return best;
}

}  // namespace vsk
