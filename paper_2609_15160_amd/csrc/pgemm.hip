// MFMA GEMM of the bf16 models' prefill projections: out = A W^T on the rows
// [0, *nact) of one loop (every sequence's gathered tokens, compact).
//
// A comes as bf16 operand rows that the producing kernel wrote: one bf16 part
// per activation (prefill_act_bf16), or the hi and lo parts side by side,
// [row][K / 32][hi 32 | lo 32] (operand_off in kernels.h), one product per
// part, so that an activation enters with about 16 significant bits.  A K
// step of 32 is then one 128-byte line per row.  W is the fragment-ordered
// copy (launch_wfrag): 16 columns x one K step are one contiguous kilobyte.
//
// Both operands go from global memory straight into LDS (global_load_lds:
// no registers, no conversions, no LDS stores), the wave's 64 lanes filling
// one kilobyte per instruction, through NST stages of KSUB K steps each, one
// wait and one barrier per stage.  A rows are XOR-swizzled by 16-byte chunk
// (the 16 rows of a fragment read hit distinct banks); W blocks are read back
// as they lie, 64 lanes one kilobyte.
//
// NORM: the operand rows hold the residual x and the product is taken with
// RMSNorm(x): (x / rms) W^T = (x W^T) / rms.  The residual projections write x
// as the next operand and each row's sum of squares in parts of 32 columns
// (ssq), so no kernel normalises rows in between.
//
// The host does not know a loop's active rows, so the workgroups read the
// count and take the tile shape from it (pick_shape), and a persistent grid
// walks the tiles.
#include <initializer_list>

#include "kernels.h"

namespace tlf {

namespace {

__device__ __forceinline__ void transpose4(float& v0, float& v1, float& v2, float& v3, int t) {
  // 4 x 4 transpose inside each group of four lanes: lane t of the group holds
  // (row r, column t) on entry and (row t, column r) on return
  float a = (t & 1) ? v0 : v1, b = (t & 1) ? v2 : v3;
  a = shfl_xor(a, 1);
  b = shfl_xor(b, 1);
  if (t & 1) { v0 = a; v2 = b; } else { v1 = a; v3 = b; }
  a = (t & 2) ? v0 : v2;
  b = (t & 2) ? v1 : v3;
  a = shfl_xor(a, 2);
  b = shfl_xor(b, 2);
  if (t & 2) { v0 = a; v1 = b; } else { v2 = a; v3 = b; }
}

__device__ __forceinline__ unsigned lds_addr(const void* p) {
  return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// 16 bytes per lane from global memory into 64 consecutive 16-byte LDS chunks
// from byte `lds` (wave-uniform, in M0).  Assembly, so that the compiler does
// not wait for every such load before the next LDS read; counts toward vmcnt.
// A scalar write of M0 needs one wait state before a load into LDS; the
// compiler, which writes M0 right before the text, inserts it for its own
// instructions only, so the s_nop is part of the text.
__device__ __forceinline__ void load_lds16(const void* g, unsigned lds) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "{m0}"(lds) : "memory");
}
__device__ __forceinline__ void load_lds4(const void* g, unsigned lds) {  // 4 bytes per lane
  asm volatile("s_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(g), "{m0}"(lds) : "memory");
}
// At most N of this wave's vector-memory operations outstanding and its LDS
// reads done, then the barrier.
template <int N> __device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// BM x BN output tile of WM x WN waves, KSUB K steps of 32 per stage, NST
// stages; WK groups of such waves share a stage's K steps (their partial tiles
// are added in LDS after the last stage, in a fixed order).
template <int BM_, int BN_, int WM_, int WN_, int WK_, int KSUB_, int NST_> struct PShape {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, WK = WK_, KSUB = KSUB_, NST = NST_;
};

template <typename SH, int P> struct PLds {
  static constexpr int A = SH::KSUB * SH::BM * 32 * P;  // elements of one stage's A
  static constexpr int B = SH::KSUB * SH::BN * 32;
  static constexpr int STAGE = A + B;
  static constexpr int ELEMS = SH::NST * STAGE;
};

// Outstanding loads that may remain when `left` later stages are in flight.
template <int LPT> __device__ __forceinline__ void wait_stages(int left) {
  if (left >= 2) wait_barrier<2 * LPT>();
  else if (left == 1) wait_barrier<LPT>();
  else wait_barrier<0>();
}

template <typename SH, int P, int AK, int EK, bool NORM>
__device__ __forceinline__ void pgemm_tile(const GemmArgs& g, int r0, int n0, int nact, bf16* lds, int* src_s,
                                           int64_t* kv_s, int* mod_s, float* inv_s) {
  using M = Mfma<bf16>;
  using L = PLds<SH, P>;
  constexpr int BM = SH::BM, BN = SH::BN, WN = SH::WN, WK = SH::WK, KSUB = SH::KSUB, NST = SH::NST;
  constexpr int NTH = SH::WM * WN * WK * kWave;
  constexpr int MT = BM / SH::WM / 16, NT = BN / WN / 16;
  constexpr int CPR = 4 * P;                       // 16-byte chunks of a row per K step
  constexpr int ACH = BM * CPR * KSUB / NTH;       // A chunks per thread and stage
  constexpr int BCH = BN * 4 * KSUB / NTH;
  constexpr int LPT = ACH + BCH;
  static_assert(ACH >= 1 && BM * CPR * KSUB % NTH == 0 && BCH >= 1 && BN * 4 * KSUB % NTH == 0, "chunks");
  static_assert(2 * LPT < 64 && NST >= 2 && NST <= 4, "vmcnt");
  static_assert(KSUB % WK == 0 && (WK - 1) * BM * BN * 2 <= L::ELEMS, "K groups");
  static_assert(MT >= 1 && NT >= 1 && (EK != E_SWIGLU || NT % 2 == 0), "wave tile");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wk = wave / (SH::WM * WN), wmn = wave % (SH::WM * WN), wm = wmn / WN, wn = wmn % WN;
  const int wbase = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
  const int S = g.K / 32, KT = S / KSUB;  // whole stages: kStageK

  auto key = [](int row) { return P == 2 ? (row >> 1) & 7 : (row >> 2) & 3; };

  // W chunk c of a thread: chunk q = tid + c NTH of the stage, block (q / 64)
  // = 16 columns of one K step, lane q % 64 of the fragment
  const bf16* b_src[BCH];
  constexpr int CB = BN / 16;  // column blocks
#pragma unroll
  for (int c = 0; c < BCH; ++c) {
    const int blk = (wbase + c * NTH) / kWave;  // wave-uniform
    const int ks = blk / CB, cb = blk % CB;
    if (g.Wf) {
      const int nb = min((n0 >> 4) + cb, (g.N >> 4) - 1);
      b_src[c] = reinterpret_cast<const bf16*>(g.Wf) + ((int64_t)(nb * S + ks) * kWave + lane) * 8;
    } else {
      const int n = min(n0 + cb * 16 + (lane & 15), g.w_rows - 1);
      b_src[c] = reinterpret_cast<const bf16*>(g.W) + (int64_t)n * g.K + ks * 32 + (lane >> 4) * 8;
    }
  }
  const int bstep = (g.Wf ? kWave * 8 : 32) * KSUB;
  auto issue_b = [&](int kt, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < BCH; ++c)
      load_lds16(b_src[c] + (int64_t)kt * bstep, lds_addr(lds + st * L::STAGE + L::A + (c * NTH + wbase) * 8));
  };
  // A chunk q = tid + c NTH: K step q / (BM CPR), row (q / CPR) % BM, LDS place
  // q % CPR, which holds the row's chunk place ^ key(row).  Rows past the
  // count read the last active row (never stored).  The row sources and the
  // epilogue's row tables are requested first, then the weights of the first
  // stages, which do not depend on them: one round trip for both.
  int a_row[ACH];
#pragma unroll
  for (int c = 0; c < ACH; ++c) {
    const int r = min(r0 + (tid + c * NTH) / CPR % BM, nact - 1);
    a_row[c] = AK == A_SRC ? row_src(g.rm, r) : r;
  }
  // NORM: TPR threads of a row read its sums of squares
  constexpr int TPR = NTH / BM, SQ = kNormMaxWidth / 128 / TPR;
  int sq_row = 0;
  if constexpr (NORM) sq_row = row_src(g.rm, min(r0 + tid / TPR, nact - 1));
  // the epilogue's row tables go straight into LDS as well (rows past the
  // count hold some other row's entry; the epilogue tests the row)
  if constexpr (EK == E_RESID) {
    if (g.rm.src && wbase < BM)
      load_lds4(g.rm.src + min(r0 + tid, g.rm.rows - 1), lds_addr(src_s + wbase));
  }
  if constexpr (EK == E_QKV) {
#pragma unroll
    for (int c = 0; c < (2 * BM + NTH - 1) / NTH; ++c) {
      const int wb = wbase + c * NTH;  // two words of each entry
      if (wb < 2 * BM)
        load_lds4(reinterpret_cast<const int32_t*>(g.kv.slot_base + min(r0 + ((wb + lane) >> 1), g.rm.rows - 1)) + (lane & 1),
                  lds_addr(reinterpret_cast<int32_t*>(kv_s) + wb));
    }
  }
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < KT) issue_b(t, t);
  const bf16* a_src[ACH];
#pragma unroll
  for (int c = 0; c < ACH; ++c) {
    const int q = tid + c * NTH, ks = q / (BM * CPR), row = (q / CPR) % BM, pl = q % CPR;
    a_src[c] = g.A16 + (int64_t)a_row[c] * (P * g.K) + ks * 32 * P + ((pl ^ key(row)) * 8);
  }
  if constexpr (EK == E_RESID) {
    if (g.mod_a && tid < BM) {
      const int tr = min(r0 + tid, nact - 1);
      mod_s[tid] = (g.mod_depth[g.mod_by_src ? row_src(g.rm, tr) : tr] - 1) * g.mod_ld;
    }
  }
  auto issue_a = [&](int kt, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < ACH; ++c)
      load_lds16(a_src[c] + (int64_t)kt * (32 * P * KSUB), lds_addr(lds + st * L::STAGE + (c * NTH + wbase) * 8));
  };
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < KT) issue_a(t, t);

  float4 sq[NORM ? SQ : 1];
  if constexpr (NORM) {
    const float4* sp = reinterpret_cast<const float4*>(g.ssq + (int64_t)sq_row * (g.K / 32));
#pragma unroll
    for (int k = 0; k < SQ; ++k) {
      const int q = tid % TPR + k * TPR, n = g.K / 128;
      const float4 v = sp[min(q, n - 1)];
      const float m = q < n ? 1.f : 0.f;
      sq[k] = make_float4(v.x * m, v.y * m, v.z * m, v.w * m);
    }
  }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int frow = lane & 15, quad = lane >> 4;
  auto multiply = [&](int st) __attribute__((always_inline)) {
    const bf16* As = lds + st * L::STAGE;
    const bf16* Bs = As + L::A;
#pragma unroll
    for (int kq = 0; kq < KSUB / WK; ++kq) {
      const int ks = kq * WK + wk;
      bf16x8 af[P][MT], bfr[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j) bfr[j] = M::load(Bs + ((ks * CB + wn * NT + j) * kWave + lane) * 8);
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          const int row = wm * MT * 16 + i * 16 + frow;
          af[p][i] = M::load(As + ((ks * BM + row) * CPR + ((p * 4 + quad) ^ key(row))) * 8);
        }
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j) acc[i][j] = M::mma(af[p][i], bfr[j], acc[i][j]);
    }
  };
  // stage kt + NST - 1 is fetched into the place that stage kt - 1 used,
  // after the barrier that ends every wave's reads of it
  int st = 0;
  for (int kt = 0; kt < KT; ++kt) {
    // outstanding after stage kt: the first stages' weights all went out ahead
    // of their A chunks, so of a first stage only the A chunks count
    const int later = min(NST - 2, KT - 1 - kt);        // stages issued after kt
    const int first = min(later, max(0, NST - 2 - kt));  // of them, first stages
    if (first == 2) wait_barrier<2 * ACH>();
    else if (first == 1 && later == 2) wait_barrier<ACH + LPT>();
    else if (first == 1) wait_barrier<ACH>();
    else wait_stages<LPT>(later);
    if (kt + NST - 1 < KT) {
      const int sn = st == 0 ? NST - 1 : st - 1;
      issue_b(kt + NST - 1, sn);
      issue_a(kt + NST - 1, sn);
    }
    multiply(st);
    st = st == NST - 1 ? 0 : st + 1;
  }
  if constexpr (NORM) {
    float c = 0.f;
#pragma unroll
    for (int k = 0; k < SQ; ++k) c += sq[k].x + sq[k].y + (sq[k].z + sq[k].w);
#pragma unroll
    for (int o = 1; o < TPR; o <<= 1) c += shfl_xor(c, o);
    if (tid % TPR == 0) inv_s[tid / TPR] = rsqrtf(c / (float)g.K + g.eps);
  }
  __syncthreads();
  if constexpr (WK > 1) {
    // the stages are free: groups 1 .. WK - 1 hand their tiles to group 0
    float* part = reinterpret_cast<float*>(lds);
    constexpr int PT = MT * NT * 4 * kWave;  // floats of one wave's tile
    if (wk > 0) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          *reinterpret_cast<f32x4*>(part + ((wk - 1) * SH::WM * WN + wmn) * PT + ((i * NT + j) * kWave + lane) * 4) = acc[i][j];
    }
    __syncthreads();
    if (wk > 0) return;
#pragma unroll
    for (int k = 1; k < WK; ++k)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] += *reinterpret_cast<const f32x4*>(part + ((k - 1) * SH::WM * WN + wmn) * PT + ((i * NT + j) * kWave + lane) * 4);
  }

  const int col16 = lane & 15, t = col16 & 3;
  if constexpr (NORM) {  // accumulator rows 4 quad + r: scaled by 1 / rms
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float inv = inv_s[wm * MT * 16 + i * 16 + quad * 4 + r];
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j][r] *= inv;
      }
  }
  if constexpr (EK == E_QKV) {
    // q to its buffer; k and v into the cache pages.  A 16-column tile lies
    // in one of q, k and v.  q and k tiles go through an in-group 4 x 4
    // transpose, after which lane t holds four consecutive columns of row
    // 4 quad + t: one 16-byte q store, or one 8-byte k store.  A v tile keeps
    // the lane's column: when its four rows are consecutive slots of one page
    // from a multiple of 4 (a fresh prefill), their values of that dimension
    // are one aligned run in the V block.
    bf16* pool = reinterpret_cast<bf16*>(g.kv.c.pool);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int nt = n0 + wn * NT * 16 + j * 16;
      if (nt >= g.N) continue;
      const int part = nt < g.d ? 0 : nt < 2 * g.d ? 1 : 2;
      const int w0 = nt - part * g.d, h = w0 / g.kv.c.D, e0 = w0 - h * g.kv.c.D;
      const int64_t kvb = part == 2 ? v_block(g.kv.c, g.kv.layer, h) : k_block(g.kv.c, g.kv.layer, h);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int rl0 = wm * MT * 16 + i * 16 + quad * 4;
        if (part < 2) {
          float v0 = acc[i][j][0], v1 = acc[i][j][1], v2 = acc[i][j][2], v3 = acc[i][j][3];
          transpose4(v0, v1, v2, v3, t);
          const int rl = rl0 + t, cw = col16 & ~3;
          if (part == 0) {
            if (r0 + rl < nact) {
              const int64_t qo = (int64_t)(r0 + rl) * g.ldo + nt + cw;
              if (P == 1 && g.q16) {  // scaled and rounded to bf16 as the attention would on loading q
                const float sc = g.q_scale;
                *reinterpret_cast<uint2*>(g.q16 + qo) =
                    make_uint2(pack_bf16x2(v0 * sc, v1 * sc), pack_bf16x2(v2 * sc, v3 * sc));
              } else {
                *reinterpret_cast<float4*>(g.out + qo) = make_float4(v0, v1, v2, v3);
              }
            }
          } else {
            const int64_t base = r0 + rl < nact ? kv_s[rl] : -1;
            if (base >= 0) {
              const int slot = (int)(base & (kPage - 1));
              *reinterpret_cast<uint2*>(pool + (base - slot) + kvb + k_frag_off<bf16>(slot, e0 + cw)) =
                  make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
            }
          }
          continue;
        }
        const int e = e0 + col16;
        const int64_t b0 = kv_s[rl0];
        if (r0 + rl0 + 3 < nact && b0 >= 0 && (b0 & 3) == 0 && kv_s[rl0 + 1] == b0 + 1 && kv_s[rl0 + 2] == b0 + 2 && kv_s[rl0 + 3] == b0 + 3) {
          const int slot = (int)(b0 & (kPage - 1));
          *reinterpret_cast<uint2*>(pool + (b0 - slot) + kvb + v_frag_off(slot, e, g.kv.c.D)) =
              make_uint2(pack_bf16x2(acc[i][j][0], acc[i][j][1]), pack_bf16x2(acc[i][j][2], acc[i][j][3]));
          continue;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t base = kv_s[rl0 + r];
          if (r0 + rl0 + r >= nact || base < 0) continue;
          const int slot = (int)(base & (kPage - 1));
          pool[base - slot + kvb + v_frag_off(slot, e, g.kv.c.D)] = (bf16)acc[i][j][r];
        }
      }
    }
  } else if constexpr (EK == E_RESID) {
    // x[src(r)] += result: the residual values of a few column tiles are
    // loaded together; inactive rows and columns past N read in bounds and store nothing
    auto residual = [&](auto gate_c) __attribute__((always_inline)) {
      constexpr bool kGate = decltype(gate_c)::value;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int rl = wm * MT * 16 + i * 16 + quad * 4 + t;
        const int src = r0 + rl < nact ? (g.rm.src ? src_s[rl] : r0 + rl) : -1;
        const int64_t xo = (int64_t)(src < 0 ? 0 : src) * g.ldo;
        float sq = 0.f;  // of the wave's columns of the row, this lane's
        constexpr int JN = kGate || NT < 4 ? 2 : 4;  // column tiles in hand: more would spill
#pragma unroll
        for (int j0 = 0; j0 < NT; j0 += JN) {
          float4 xv[JN], gv[kGate ? JN : 1];
#pragma unroll
          for (int j = 0; j < JN; ++j) {
            const int nb = min(n0 + (wn * NT + j0 + j) * 16 + (col16 & ~3), g.N - 4);
            xv[j] = *reinterpret_cast<const float4*>(g.out + xo + nb);
            if constexpr (kGate) gv[j] = *reinterpret_cast<const float4*>(g.mod_a + mod_s[rl] + nb);
          }
#pragma unroll
          for (int j = 0; j < JN; ++j) {
            f32x4 v = acc[i][j0 + j];
            float v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];
            transpose4(v0, v1, v2, v3, t);
            if constexpr (kGate) { v0 *= 1.f + gv[j].x; v1 *= 1.f + gv[j].y; v2 *= 1.f + gv[j].z; v3 *= 1.f + gv[j].w; }
            const int nb = n0 + (wn * NT + j0 + j) * 16 + (col16 & ~3);
            if (src >= 0 && nb < g.N) {
              const float4 x = make_float4(xv[j].x + v0, xv[j].y + v1, xv[j].z + v2, xv[j].w + v3);
              *reinterpret_cast<float4*>(g.out + xo + nb) = x;
              if (g.out16) {  // the next projection's operand
                store_operand4<P>(g.out16, src, nb, g.N, x);
                sq = fmaf(x.w, x.w, fmaf(x.z, x.z, fmaf(x.y, x.y, fmaf(x.x, x.x, sq))));
              }
            }
          }
        }
        if (g.out16) {
          // the four lanes that share the row; the sum goes to the first of the
          // wave's parts of 32 columns, zeros to the others
          sq += shfl_xor(sq, 4);
          sq += shfl_xor(sq, 8);
          const int part = (n0 >> 5) + wn * (NT / 2) + (col16 >> 2);
          if (src >= 0 && (col16 >> 2) < NT / 2 && part < g.N / 32)
            g.ssq[(int64_t)src * (g.N / 32) + part] = col16 < 4 ? sq : 0.f;
        }
      }
    };
    if (g.mod_a) residual(std::true_type{});
    else residual(std::false_type{});
  } else if constexpr (EK == E_SWIGLU) {
    // gate columns j, up columns j + 1 of the same 16 hidden units; silu(g) =
    // g / (1 + e^-g) with the hardware reciprocal (within an ulp of the division)
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int rl = wm * MT * 16 + i * 16 + quad * 4 + t;
#pragma unroll
      for (int j = 0; j < NT; j += 2) {
        float h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float gt = acc[i][j][r], up = acc[i][j + 1][r];
          h[r] = gt * __builtin_amdgcn_rcpf(1.f + __expf(-gt)) * up;
        }
        transpose4(h[0], h[1], h[2], h[3], t);
        const int n = n0 + wn * NT * 16 + j * 16;  // first gate column of the group
        const int unit = (n >> 5) * 16 + (col16 & ~3);
        if (r0 + rl < nact && unit < g.F)
          store_operand4<P>(g.out16, r0 + rl, unit, g.F, make_float4(h[0], h[1], h[2], h[3]));
      }
    }
  } else {
    static_assert(EK == E_LOGITS, "epilogue");
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int rl = wm * MT * 16 + i * 16 + quad * 4 + t;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        float v0 = acc[i][j][0], v1 = acc[i][j][1], v2 = acc[i][j][2], v3 = acc[i][j][3];
        transpose4(v0, v1, v2, v3, t);
        const int nb = n0 + wn * NT * 16 + j * 16 + (col16 & ~3);
        if (r0 + rl >= nact) continue;
        float* o = g.out + (int64_t)(g.out_row_off + r0 + rl) * g.ldo + nb;
        if (nb + 4 <= g.N && g.ldo % 4 == 0) {
          *reinterpret_cast<float4*>(o) = make_float4(v0, v1, v2, v3);
        } else {
          if (nb < g.N) o[0] = v0;
          if (nb + 1 < g.N) o[1] = v1;
          if (nb + 2 < g.N) o[2] = v2;
          if (nb + 3 < g.N) o[3] = v3;
        }
      }
    }
  }
}

// Tile shapes (rows x columns): large for many rows, middle and small ones so
// that a loop with few active rows still spreads over the device.
template <int P> using PLarge = PShape<128, 256, 2, 2, 1, 1, P == 2 ? 2 : 3>;
template <int P> using PWide = PShape<128, 128, 2, 2, 1, 1, P == 2 ? 3 : 4>;
using PMid = PShape<64, 128, 2, 2, 1, 1, 4>;
using PSmall = PShape<32, 64, 1, 2, 2, 2, 3>;
using PTiny = PShape<32, 32, 1, 1, 4, 4, 3>;

// K must be whole stages of the shape with the most K steps per stage: the
// shape is chosen on the device, and a tile runs K / (32 KSUB) whole stages.
constexpr int max_ksub(std::initializer_list<int> l) {
  int m = 0;
  for (int k : l) m = k > m ? k : m;
  return m;
}
constexpr int kStageK = 32 * max_ksub({PLarge<1>::KSUB, PLarge<2>::KSUB, PWide<1>::KSUB, PWide<2>::KSUB, PMid::KSUB,
                                       PSmall::KSUB, PTiny::KSUB});
static_assert(kStageK % (32 * PSmall::KSUB) == 0 && kStageK % (32 * PTiny::KSUB) == 0, "whole stages of every shape");

// Workgroup L runs on XCD L % 8, and each XCD has its own L2.  Up to 3072
// columns the tiles are dealt to the XCDs as rectangles: RX groups of row
// tiles times CX = 8 / RX groups of column tiles, so that an XCD reads 1 / RX
// of A and 1 / CX of W; of the four splits the one with the fewest rounds,
// then the least bytes per XCD.  Against tiles in plain order (two parts): 8192
// x 768 x 2048 81 -> 55 us (64 x 128 tiles), 16384 x 2304 x 768 116 -> 103 us
// (128 x 256).  With more columns (gate/up, LM head) the plain order, which
// gives each XCD a subset of the columns, is the faster one for many rows
// (16384 x 4096 x 768 158 against 174 us) and equal for few.
template <typename SH, int P, int AK, int EK, bool NORM>
__device__ __forceinline__ void walk_tiles(const GemmArgs& g, int nact, bf16* lds, int* src_s, int64_t* kv_s, int* mod_s,
                                           float* inv_s) {
  const int tn = (g.N + SH::BN - 1) / SH::BN, tm = (nact + SH::BM - 1) / SH::BM;
  int first = (int)blockIdx.x, stride = (int)gridDim.x, rb = 0, cb = 0, nc = tn, tiles = tm * tn;
  if (g.N <= 3072 && stride % 8 == 0) {
    stride >>= 3;
    const int x = first & 7;
    first >>= 3;
    const float inv = 1.f / (float)stride;
    int l = -1, rounds = 0;
    int64_t bytes = 0;
#pragma unroll
    for (int k = 0; k <= 3; ++k) {  // RX = 1 << k
      const int mr = (tm + (1 << k) - 1) >> k, mc = (tn + (8 >> k) - 1) >> (3 - k), rd = (int)((float)(mr * mc - 1) * inv);  // rounds - 1
      const int64_t by = (int64_t)mr * SH::BM * P + (int64_t)mc * SH::BN;
      if (l < 0 || rd < rounds || (rd == rounds && by < bytes)) { l = k; rounds = rd; bytes = by; }
    }
    const int rx = x & ((1 << l) - 1), cx = x >> l;
    rb = tm * rx >> l;
    cb = tn * cx >> (3 - l);
    nc = (tn * (cx + 1) >> (3 - l)) - cb;
    tiles = ((tm * (rx + 1) >> l) - rb) * nc;
  }
  for (int k = first; k < tiles; k += stride) {
    pgemm_tile<SH, P, AK, EK, NORM>(g, (rb + k / nc) * SH::BM, (cb + k % nc) * SH::BN, nact, lds, src_s, kv_s, mod_s, inv_s);
    __syncthreads();  // the next tile overwrites the stages and the row tables
  }
}

template <int P, int AK, int EK, bool NORM>
__global__ __launch_bounds__(256, 2) void k_pgemm(GemmArgs g) {
  constexpr int E1 = PLds<PLarge<P>, P>::ELEMS, E2 = PLds<PWide<P>, P>::ELEMS, E3 = PLds<PTiny, P>::ELEMS;
  constexpr int E = E1 > E2 ? (E1 > E3 ? E1 : E3) : (E2 > E3 ? E2 : E3);
  static_assert(PLds<PMid, P>::ELEMS <= E && PLds<PSmall, P>::ELEMS <= E, "LDS");
  __shared__ __align__(16) bf16 lds[E];
  __shared__ int src_s[EK == E_RESID ? 128 : 1];
  __shared__ int64_t kv_s[EK == E_QKV ? 128 : 1];
  __shared__ int mod_s[EK == E_RESID ? 128 : 1];
  __shared__ float inv_s[NORM ? 128 : 1];  // 1 / rms of the tile's rows
  const int nact = g.rm.nact ? min(*g.rm.nact, g.rm.rows) : g.rm.rows;
  if (nact <= 0) return;
  int pick = 4;
  for (int i = 0; i < kShapeRuns; ++i) {  // uniform
    if (nact <= g.shapes.run[i] >> 3) {
      pick = g.shapes.run[i] & 7;
      break;
    }
  }
  if (pick == 4) walk_tiles<PLarge<P>, P, AK, EK, NORM>(g, nact, lds, src_s, kv_s, mod_s, inv_s);
  else if (pick == 3) walk_tiles<PWide<P>, P, AK, EK, NORM>(g, nact, lds, src_s, kv_s, mod_s, inv_s);
  else if (pick == 2) walk_tiles<PMid, P, AK, EK, NORM>(g, nact, lds, src_s, kv_s, mod_s, inv_s);
  else if (pick == 1) walk_tiles<PSmall, P, AK, EK, NORM>(g, nact, lds, src_s, kv_s, mod_s, inv_s);
  else walk_tiles<PTiny, P, AK, EK, NORM>(g, nact, lds, src_s, kv_s, mod_s, inv_s);
}

template <int P>
hipError_t launch_parts(const GemmArgs& a, AKind ak, EKind ek, bool norm, int cus, hipStream_t s) {
  // no more workgroups than the smallest tiles of every row
  const int64_t most = ((int64_t)((a.rm.rows + 31) / 32) * ((a.N + 31) / 32) + 7) / 8 * 8;
  const int grid = (int)(most < 2 * cus ? most : 2 * cus);
#define TLF_PG(AKV, EKV, NORMV) hipLaunchKernelGGL((k_pgemm<P, AKV, EKV, NORMV>), dim3(grid), dim3(256), 0, s, a)
  if (ak == A_SRC && ek == E_QKV) {
    if (norm) TLF_PG(A_SRC, E_QKV, true);
    else TLF_PG(A_SRC, E_QKV, false);
  } else if (ak == A_SRC && ek == E_SWIGLU) {
    if (norm) TLF_PG(A_SRC, E_SWIGLU, true);
    else TLF_PG(A_SRC, E_SWIGLU, false);
  } else if (ak == A_CMP && ek == E_RESID && !norm) {
    TLF_PG(A_CMP, E_RESID, false);
  } else if (P == 2 && ak == A_SRC && ek == E_LOGITS) {
    if (norm) TLF_PG(A_SRC, E_LOGITS, true);
    else TLF_PG(A_SRC, E_LOGITS, false);
  } else {
    return hipErrorInvalidValue;
  }
#undef TLF_PG
  return hipGetLastError();
}

// Estimated time of `tiles` tiles on `cus` compute units, two workgroups each
// (nanoseconds): per round a start and an epilogue (`base`, half hidden by the
// neighbour workgroup from the second round on), per K step t1 with one and t2
// with two workgroups on a compute unit.
int64_t tile_time(int64_t tiles, int cus, int steps, int t1, int t2, int base) {
  const int64_t full = tiles / (2 * cus), rem = tiles - full * 2 * cus, rounds = full + (rem > 0);
  return steps * (full * t2 + (rem == 0 ? 0 : rem <= cus ? t1 : t2)) + base + (rounds - 1) * base / 2;
}

}  // namespace

hipError_t launch_pgemm(const GemmArgs& a, AKind ak, EKind ek, bool norm, int parts, int cus, hipStream_t s) {
  if (!a.A16 || a.K <= 0 || a.K % kStageK != 0 || (a.N % 4 != 0 && ek != E_LOGITS) || cus <= 0) return hipErrorInvalidValue;
  if (a.rm.rows <= 0 || a.N <= 0) return hipSuccess;
  if (norm && (!a.ssq || a.K > kNormMaxWidth || a.K % 128 != 0)) return hipErrorInvalidValue;
  if (ek == E_RESID && a.out16 && (!a.ssq || a.mod_a || a.N % 32 != 0)) return hipErrorInvalidValue;
  if (a.mod_g) return hipErrorInvalidValue;  // the operand scale is applied where the rows are written
  if (a.Wf && a.N % 16 != 0) return hipErrorInvalidValue;
  // the QKV epilogue takes each 16-column tile as wholly q, k or v
  if (ek == E_QKV && (a.d % 16 != 0 || a.ldo % 4 != 0 || a.kv.c.D % 16 != 0 || !a.Wf)) return hipErrorInvalidValue;
  if (ek == E_RESID && (a.ldo % 4 != 0 || (a.mod_a && a.mod_ld % 4 != 0) || !a.Wf)) return hipErrorInvalidValue;
  // gate and up columns are interleaved in the fragment-ordered copy only
  if (ek == E_SWIGLU && (a.F % 32 != 0 || !a.Wf || !a.out16)) return hipErrorInvalidValue;
  return parts == 2 ? launch_parts<2>(a, ak, ek, norm, cus, s) : launch_parts<1>(a, ak, ek, norm, cus, s);
}

// The rule was fitted to every shape timed at K 768 to 2816, N 768 to 5632 and
// 16 to 32768 rows; ns per K step with one and two workgroups per compute unit:
//            32 x 32    32 x 64    64 x 128    128 x 128   128 x 256
//   2 parts  75, 200    112, 240   295, 460    475, 800    750, 1450
//   1 part   54, 120    91, 160    220, 340    310, 540    480, 900
//   base     4100       4200       4600        6000        9000
// e.g. 1000 rows x 768 x 2048 in two parts: 20, 16, 25, 40 and 61 us; 16384 x
// 2304 x 768: -, 208, 122, 112 and 103 us.  A run changes shape only for a
// gain of 2%.
PgemmShapes pgemm_shapes(int N, int K, int parts, int cus, int max_rows) {
  static const int bm[5] = {32, 32, 64, 128, 128}, bn[5] = {32, 64, 128, 128, 256};
  static const int t1[2][5] = {{54, 91, 220, 310, 480}, {75, 112, 295, 475, 750}};
  static const int t2[2][5] = {{120, 160, 340, 540, 900}, {200, 240, 460, 800, 1450}};
  static const int base[5] = {4100, 4200, 4600, 6000, 9000};
  PgemmShapes out;
  int runs = 0, cur = 0;
  const int step = max_rows > 65536 ? (max_rows + 4095) / 4096 : 16;
  for (int n = step; runs < kShapeRuns - 1; n += step) {
    const int rows = n < max_rows ? n : max_rows;
    int64_t t[5];
    int best = 0;
    for (int s = 0; s < 5; ++s) {
      t[s] = tile_time((int64_t)((rows + bm[s] - 1) / bm[s]) * ((N + bn[s] - 1) / bn[s]), cus, K / 32, t1[parts - 1][s],
                       t2[parts - 1][s], base[s]);
      if (t[s] < t[best]) best = s;
    }
    if (n == step) {
      cur = best;
    } else if (best != cur && t[best] * 102 < t[cur] * 100) {
      out.run[runs++] = (n - step) << 3 | cur;
      cur = best;
    }
    if (n >= max_rows) break;
  }
  for (; runs < kShapeRuns; ++runs) out.run[runs] = INT32_MAX - 7 + cur;  // every row count
  return out;
}

}  // namespace tlf
