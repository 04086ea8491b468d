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
// The host does not know a loop's active rows, so the workgroups read the
// count and take the tile shape from it (pick_shape), and a persistent grid
// walks the tiles.
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
__device__ __forceinline__ void load_lds16(const void* g, unsigned lds) {
  asm volatile("global_load_lds_dwordx4 %0, off" ::"v"(g), "{m0}"(lds) : "memory");
}
// At most N of this wave's vector-memory operations outstanding and its LDS
// reads done, then the barrier.
template <int N> __device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// BM x BN output tile of WM x WN waves, KSUB K steps of 32 per stage, NST stages.
template <int BM_, int BN_, int WM_, int WN_, int KSUB_, int NST_> struct PShape {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KSUB = KSUB_, NST = NST_;
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

template <typename SH, int P, int AK, int EK>
__device__ __forceinline__ void pgemm_tile(const GemmArgs& g, int r0, int n0, int nact, bf16* lds, int* src_s,
                                           int64_t* kv_s, int* mod_s) {
  using M = Mfma<bf16>;
  using L = PLds<SH, P>;
  constexpr int BM = SH::BM, BN = SH::BN, WN = SH::WN, KSUB = SH::KSUB, NST = SH::NST;
  constexpr int NTH = SH::WM * SH::WN * kWave;
  constexpr int MT = BM / SH::WM / 16, NT = BN / WN / 16;
  constexpr int CPR = 4 * P;                       // 16-byte chunks of a row per K step
  constexpr int ACH = BM * CPR * KSUB / NTH;       // A chunks per thread and stage
  constexpr int BCH = BN * 4 * KSUB / NTH;
  constexpr int LPT = ACH + BCH;
  static_assert(ACH >= 1 && BM * CPR * KSUB % NTH == 0 && BCH >= 1 && BN * 4 * KSUB % NTH == 0, "chunks");
  static_assert(2 * LPT < 64 && NST >= 2 && NST <= 4, "vmcnt");
  static_assert(MT >= 1 && NT >= 1 && (EK != E_SWIGLU || NT % 2 == 0), "wave tile");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int wbase = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
  const int S = g.K / 32, KT = S / KSUB;  // the launcher checks K % (32 KSUB) == 0

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
  const int tr = min(r0 + tid % BM, nact - 1);
  int t_src = 0;
  int64_t t_kv = -1;
  if constexpr (EK == E_RESID) t_src = row_src(g.rm, tr);
  if constexpr (EK == E_QKV) t_kv = g.kv.slot_base[tr];
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < KT) issue_b(t, t);
  const bf16* a_src[ACH];
#pragma unroll
  for (int c = 0; c < ACH; ++c) {
    const int q = tid + c * NTH, ks = q / (BM * CPR), row = (q / CPR) % BM, pl = q % CPR;
    a_src[c] = g.A16 + (int64_t)a_row[c] * (P * g.K) + ks * 32 * P + ((pl ^ key(row)) * 8);
  }
  if (tid < BM) {
    const bool act = r0 + tid < nact;
    if constexpr (EK == E_RESID) {
      src_s[tid] = act ? t_src : -1;
      if (g.mod_a) mod_s[tid] = (g.mod_depth[g.mod_by_src ? t_src : tr] - 1) * g.mod_ld;
    }
    if constexpr (EK == E_QKV) kv_s[tid] = act ? t_kv : -1;
  }
  auto issue_a = [&](int kt, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < ACH; ++c)
      load_lds16(a_src[c] + (int64_t)kt * (32 * P * KSUB), lds_addr(lds + st * L::STAGE + (c * NTH + wbase) * 8));
  };
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < KT) issue_a(t, t);

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
    for (int ks = 0; ks < KSUB; ++ks) {
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
  __syncthreads();  // (also: the row tables are written)

  const int col16 = lane & 15, t = col16 & 3;
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
            const int64_t base = kv_s[rl];
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
        if (b0 >= 0 && (b0 & 3) == 0 && kv_s[rl0 + 1] == b0 + 1 && kv_s[rl0 + 2] == b0 + 2 && kv_s[rl0 + 3] == b0 + 3) {
          const int slot = (int)(b0 & (kPage - 1));
          *reinterpret_cast<uint2*>(pool + (b0 - slot) + kvb + v_frag_off(slot, e, g.kv.c.D)) =
              make_uint2(pack_bf16x2(acc[i][j][0], acc[i][j][1]), pack_bf16x2(acc[i][j][2], acc[i][j][3]));
          continue;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t base = kv_s[rl0 + r];
          if (base < 0) continue;
          const int slot = (int)(base & (kPage - 1));
          pool[base - slot + kvb + v_frag_off(slot, e, g.kv.c.D)] = (bf16)acc[i][j][r];
        }
      }
    }
  } else if constexpr (EK == E_RESID) {
    // x[src(r)] += result: the residual values of up to four column tiles are
    // loaded together; inactive rows and columns past N read in bounds and store nothing
    auto residual = [&](auto gate_c) __attribute__((always_inline)) {
      constexpr bool kGate = decltype(gate_c)::value;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int rl = wm * MT * 16 + i * 16 + quad * 4 + t;
        const int src = src_s[rl];
        const int64_t xo = (int64_t)(src < 0 ? 0 : src) * g.ldo;
        constexpr int JN = NT < 4 ? NT : 4;  // columns in hand: more would spill
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
            if (src >= 0 && nb < g.N)
              *reinterpret_cast<float4*>(g.out + xo + nb) =
                  make_float4(xv[j].x + v0, xv[j].y + v1, xv[j].z + v2, xv[j].w + v3);
          }
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
template <int P> using PLarge = PShape<128, 256, 2, 2, 1, P == 2 ? 2 : 3>;
using PMid = PShape<64, 128, 2, 2, 1, 4>;
using PSmall = PShape<32, 64, 1, 4, 2, 3>;
using PSmallGate = PShape<32, 64, 2, 2, 2, 3>;  // gate/up: a wave needs column pairs

// Shape with the least estimated time on `cus` compute units, two workgroups
// each: cycles per K step of a round with two and with one workgroup per
// compute unit.
__device__ __forceinline__ int round_cost(int tiles, int cus, int two, int one) {
  const int full = tiles / (2 * cus), rem = tiles - full * 2 * cus;
  return full * two + (rem == 0 ? 0 : rem <= cus ? one : two);
}
template <int P> __device__ __forceinline__ int pick_shape(int nact, int N, int cus) {
  const int large = ((nact + 127) >> 7) * ((N + 255) >> 8), mid = ((nact + 63) >> 6) * ((N + 127) >> 7),
            small = ((nact + 31) >> 5) * ((N + 63) >> 6);
  const int cl = round_cost(large, cus, P == 2 ? 2300 : 1300, P == 2 ? 1600 : 1000);
  const int cm = round_cost(mid, cus, P == 2 ? 800 : 550, P == 2 ? 550 : 400);
  const int cs = round_cost(small, cus, P == 2 ? 320 : 260, P == 2 ? 240 : 200);
  if (cl <= cm && cl <= cs) return 2;
  return cm <= cs ? 1 : 0;
}

template <typename SH, int P, int AK, int EK>
__device__ __forceinline__ void walk_tiles(const GemmArgs& g, int nact, bf16* lds, int* src_s, int64_t* kv_s, int* mod_s) {
  const int tn = (g.N + SH::BN - 1) / SH::BN, tiles = (nact + SH::BM - 1) / SH::BM * tn;
  const int G = (int)gridDim.x, L = (int)blockIdx.x;
  for (int base = 0; base < tiles; base += G) {
    // workgroup L runs on XCD L % 8.  With at most four column tiles a round's
    // tiles go to the XCDs as contiguous runs (each L2 holds a few row tiles),
    // else in plain order, which gives each XCD a subset of the weight columns.
    const int n = min(tiles - base, G);
    if (L >= n) break;
    int k = L;
    if (tn <= 4) {
      const int x = L & 7, per = n >> 3, rem = n & 7;
      k = x * per + min(x, rem) + (L >> 3);
    }
    const int tl = base + k;
    pgemm_tile<SH, P, AK, EK>(g, tl / tn * SH::BM, tl % tn * SH::BN, nact, lds, src_s, kv_s, mod_s);
    __syncthreads();  // the next tile overwrites the stages and the row tables
  }
}

template <int P, int AK, int EK>
__global__ __launch_bounds__(256, 2) void k_pgemm(GemmArgs g, int cus, int shape) {
  using PS = std::conditional_t<EK == E_SWIGLU, PSmallGate, PSmall>;
  constexpr int E1 = PLds<PLarge<P>, P>::ELEMS, E2 = PLds<PMid, P>::ELEMS, E3 = PLds<PS, P>::ELEMS;
  constexpr int E = E1 > E2 ? (E1 > E3 ? E1 : E3) : (E2 > E3 ? E2 : E3);
  __shared__ __align__(16) bf16 lds[E];
  __shared__ int src_s[EK == E_RESID ? 128 : 1];
  __shared__ int64_t kv_s[EK == E_QKV ? 128 : 1];
  __shared__ int mod_s[EK == E_RESID ? 128 : 1];
  const int nact = g.rm.nact ? min(*g.rm.nact, g.rm.rows) : g.rm.rows;
  if (nact <= 0) return;
  const int pick = shape >= 0 ? shape : pick_shape<P>(nact, g.N, cus);
  if (pick == 2) walk_tiles<PLarge<P>, P, AK, EK>(g, nact, lds, src_s, kv_s, mod_s);
  else if (pick == 1) walk_tiles<PMid, P, AK, EK>(g, nact, lds, src_s, kv_s, mod_s);
  else walk_tiles<PS, P, AK, EK>(g, nact, lds, src_s, kv_s, mod_s);
}

template <int P>
hipError_t launch_parts(const GemmArgs& a, AKind ak, EKind ek, int cus, hipStream_t s) {
  // no more workgroups than the smallest tiles of every row
  const int64_t most = (int64_t)((a.rm.rows + 31) / 32) * ((a.N + 63) / 64);
  const int grid = (int)(most < 2 * cus ? most : 2 * cus);
#define TLF_PG(AKV, EKV) hipLaunchKernelGGL((k_pgemm<P, AKV, EKV>), dim3(grid), dim3(256), 0, s, a, cus, -1)
  if (ak == A_SRC && ek == E_QKV) TLF_PG(A_SRC, E_QKV);
  else if (ak == A_SRC && ek == E_SWIGLU) TLF_PG(A_SRC, E_SWIGLU);
  else if (ak == A_CMP && ek == E_RESID) TLF_PG(A_CMP, E_RESID);
  else if (P == 2 && ak == A_SRC && ek == E_LOGITS) TLF_PG(A_SRC, E_LOGITS);
  else return hipErrorInvalidValue;
#undef TLF_PG
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pgemm(const GemmArgs& a, AKind ak, EKind ek, int parts, int cus, hipStream_t s) {
  if (!a.A16 || a.K <= 0 || a.K % 64 != 0 || (a.N % 4 != 0 && ek != E_LOGITS) || cus <= 0) return hipErrorInvalidValue;
  if (a.rm.rows <= 0 || a.N <= 0) return hipSuccess;
  if (a.mod_g) return hipErrorInvalidValue;  // the operand scale is applied where the rows are written
  if (a.Wf && a.N % 16 != 0) return hipErrorInvalidValue;
  // the QKV epilogue takes each 16-column tile as wholly q, k or v
  if (ek == E_QKV && (a.d % 16 != 0 || a.ldo % 4 != 0 || a.kv.c.D % 16 != 0 || !a.Wf)) return hipErrorInvalidValue;
  if (ek == E_RESID && (a.ldo % 4 != 0 || (a.mod_a && a.mod_ld % 4 != 0) || !a.Wf)) return hipErrorInvalidValue;
  // gate and up columns are interleaved in the fragment-ordered copy only
  if (ek == E_SWIGLU && (a.F % 32 != 0 || !a.Wf || !a.out16)) return hipErrorInvalidValue;
  return parts == 2 ? launch_parts<2>(a, ak, ek, cus, s) : launch_parts<1>(a, ak, ek, cus, s);
}

}  // namespace tlf
