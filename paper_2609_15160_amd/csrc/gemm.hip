// MFMA GEMM with float32 rows: the prefill projections and LM head of float32
// models, the MLP router's hidden layer of a prefill, and the decode LM head
// of a large batch (pgemm.hip holds the bf16 models' prefill projections).
//
// out = A W^T on the active rows of a row map, with W [N][K] row-major
// (linear-layer layout) in the storage dtype and A float32, either the
// normalised residual rows y[src(r)] (A_SRC) or compact rows buf[r] (A_CMP).
// With bf16 weights every A tile is split into bf16 hi and lo parts in LDS
// and each product runs once per part, so the activations keep about 16
// significant bits; the weights are exact in bf16.
// Epilogues:
//   E_QKV:     q to a buffer; k, v appended to the loop's cache pages (Eq. 11)
//   E_RESID:   x[src(r)] += result (residual of the attention/FFN branch)
//   E_SWIGLU:  act = silu(gate) * up, gate/up columns interleaved in 16-column
//              groups so every wave holds matching pairs
//   E_LOGITS:  float logits plus a packed (value, -index) greedy key per 64 columns;
//              compact rows (A_CMP, the decode LM head) go to row src(r)
//   E_HIDDEN:  silu(result + bias), the MLP router's hidden layer
//
// Tiling: 256 threads = 4 waves in a 2 x 2 grid, a 128 x 256 output tile
// per workgroup (64 x 128 per wave; 128 x 128 when there are few row tiles).
// K advances 32 elements per tile through two LDS stages, the next tile's
// global loads in flight while the current one is multiplied, then converted
// and stored to the other stage (one barrier per tile).  LDS rows are
// XOR-swizzled by 16-byte chunk instead of padded, so two workgroups fit on
// a compute unit.
#include "kernels.h"

namespace tlf {

namespace {

// Each wave kGemmMT x NT MFMA tiles of 16 x 16 (64 rows x 128 or 64
// columns), K kGemmBK at a time.
constexpr int kGemmMT = 4, kGemmBK = 32;

__device__ __forceinline__ unsigned int ordered_bits(float v) {
  unsigned int u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// 4 x 4 transpose inside each group of four lanes: lane t of the group holds
// v[r] = (row r, column t) of a 4 x 4 block on entry and (row t, column r) on
// return, so an accumulator tile's four consecutive columns of one row meet
// in one lane (one 16-byte access instead of four 4-byte ones).
__device__ __forceinline__ void transpose4(float& v0, float& v1, float& v2, float& v3, int t) {
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

// 16-byte chunk c of LDS row `row` is stored at chunk c ^ key(row): the 16
// rows that one MFMA fragment read touches land in distinct banks without
// padding (bf16 rows of 32 elements hold 4 chunks, float rows 8).
template <typename T> __device__ __forceinline__ int swz(int row, int c) {
  if constexpr (sizeof(T) == 2) return c ^ ((row >> 2) & 3);
  else return c ^ (row & 7);
}

// MOD: the A rows are scaled by (1 + gamma) of their AdaLN modulation rows.
// NORM: A holds residual rows x and the product is taken with RMSNorm(x): the
// sum of squares of each row is accumulated from the A chunks as they pass
// and the output row is scaled by 1 / rms, since (x / rms) W^T = (x W^T) / rms.
// MT x NT: each wave's 16 x 16 MFMA tiles; BK: K elements per LDS stage.
// The LDS comes in as pointers: with the arrays named here the compiler works
// out each fragment's LDS address again in every K tile (18 more vector
// instructions of 426 in float32): float32 prefills of 40 x 60 tokens, d = 256,
// took 2094 against 2028 us, of 2 x 300, d = 512, 3633 against 3505.
template <typename T, int MT, int NT, int BK, int AK, int EK, bool MOD, bool NORM>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, const int r0, const int n0, void* as_lds, void* bs_lds,
                                          int* row_src_s, int* row_mod_s, float* row_inv_s, int64_t* kv_base) {
  constexpr int NTH = 256;                           // 2 x 2 waves
  constexpr int BM = 2 * MT * 16, BN = 2 * NT * 16;
  constexpr bool kBf16 = sizeof(T) == 2;             // bf16 weights: A converted to bf16 in LDS
  constexpr int NST = 2;                             // LDS stages
  constexpr int NA = kBf16 ? 2 : 1;                  // operand parts of A (hi, lo)
  constexpr int CE = 16 / (int)sizeof(T);            // storage elements per 16-byte chunk
  constexpr int WCR = BK / CE;                       // weight chunks per row per K tile
  constexpr int ACR = BK / 4;                        // A chunks (4 floats) per row per K tile
  using M = Mfma<T>;
  constexpr int KS = M::KS, EPL = M::EPL;
  constexpr int ACH = BM * ACR / NTH;                // A chunks per thread
  constexpr int BCH = BN * WCR / NTH;                // B chunks per thread
  static_assert(ACH >= 1 && BM * ACR % NTH == 0, "A tile split");
  static_assert(BCH >= 1 && BN * WCR % NTH == 0, "B tile split");
  static_assert(BK % KS == 0 && (KS * (int)sizeof(T)) % 16 == 0 || EPL == 1, "K tile");

  // the workgroup's LDS: operand stages, and per tile row its source row,
  // modulation row offset (AdaLN, 0 without), 1 / rms and cache slot
  auto& As = *reinterpret_cast<T (*)[NST][NA][BM * BK]>(as_lds);
  auto& Bs = *reinterpret_cast<T (*)[NST][BN * BK]>(bs_lds);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  // decode: a tile whose first row has exited is empty (rows are depth-sorted)
  if (g.rm.nact && r0 >= *g.rm.nact) return;
  // W row of output column n (clamped; columns >= N are never stored)
  auto w_row = [&](int n) -> int {
    int wr = n;
    if constexpr (EK == E_SWIGLU) {
      const int grp = n >> 5, w = n & 31;
      wr = (w < 16) ? grp * 16 + w : g.F + grp * 16 + (w - 16);
    }
    return wr < g.w_rows ? wr : g.w_rows - 1;
  };

  float4 ra[ACH];
  float4 rg[MOD ? ACH : 1];  // gamma of the A chunks in flight
  V16<T> rb[BCH];
  const float* A = reinterpret_cast<const float*>(g.A);
  const T* W = reinterpret_cast<const T*>(g.W);
  const int KT = g.K / BK;

  // chunk u of thread t: A row (t + NTH u) / ACR, floats 4 ((t + NTH u) % ACR)
  // .. + 3; W row (t + NTH u) / WCR, chunk (t + NTH u) % WCR
  auto load_b = [&](int kt) {
    const int kk = kt * BK;
#pragma unroll
    for (int c = 0; c < BCH; ++c) {
      const int ch = tid + c * NTH, row = ch / WCR, col = (ch % WCR) * CE;
      rb[c] = ld16(W + (int64_t)w_row(n0 + row) * g.K + kk + col);
    }
  };
  auto load_a = [&](int kt) {
    const int kk = kt * BK;
#pragma unroll
    for (int c = 0; c < ACH; ++c) {
      const int ch = tid + c * NTH, row = ch / ACR, col = (ch % ACR) * 4;
      const int s = row_src_s[row];
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f), gm = v;
      if (s >= 0) {
        const int64_t ar = (AK == A_SRC) ? (int64_t)s : (int64_t)(r0 + row);
        // fragment order (bf16 MFMA): the four floats lie in one run of EPL = 8
        v = *reinterpret_cast<const float4*>(A + (g.a_frag ? frag_index<T>((int)ar, kk + col, g.K)
                                                            : ar * g.lda + kk + col));
        if constexpr (MOD) gm = *reinterpret_cast<const float4*>(g.mod_g + row_mod_s[row] + kk + col);
      }
      ra[c] = v;
      if constexpr (MOD) rg[c] = gm;
    }
  };
  // NORM: this thread's rows are tid / ACR + c * (NTH / ACR), c < ACH
  float ssq[NORM ? ACH : 1];
#pragma unroll
  for (int c = 0; c < (NORM ? ACH : 1); ++c) ssq[c] = 0.f;
  auto store_tiles = [&](int st) {
#pragma unroll
    for (int c = 0; c < ACH; ++c) {
      const int ch = tid + c * NTH, row = ch / ACR, f = ch % ACR;  // floats 4f .. 4f + 3 of the row
      float4 av = ra[c];
      if constexpr (NORM) ssq[c] += av.x * av.x + av.y * av.y + av.z * av.z + av.w * av.w;
      if constexpr (MOD)
        av = make_float4(av.x * (1.f + rg[c].x), av.y * (1.f + rg[c].y), av.z * (1.f + rg[c].z),
                         av.w * (1.f + rg[c].w));
      const int e = 4 * f;  // first element: chunk e / CE, offset e % CE
      T* dst = &As[st][0][row * BK + swz<T>(row, e / CE) * CE + e % CE];
      if constexpr (kBf16) {
        uint2 hi, lo;
        split4(av, hi, lo);
        *reinterpret_cast<uint2*>(dst) = hi;
        *reinterpret_cast<uint2*>(dst + BM * BK) = lo;  // As[st][1]
      } else {
        *reinterpret_cast<float4*>(dst) = av;
      }
    }
#pragma unroll
    for (int c = 0; c < BCH; ++c) {
      const int ch = tid + c * NTH, row = ch / WCR, cc = ch % WCR;
      st16(&Bs[st][row * BK + swz<T>(row, cc) * CE], rb[c]);
    }
  };

  // the weight tile does not depend on which rows are active: it goes out first
  load_b(0);

  // thread t < BM resolves row r0 + t.  Its source row (and for QKV its
  // cache slot, consumed by the epilogue) is loaded together with the
  // activity test: both are in bounds for every row of the grid and are used
  // only for active rows.
  int my_src = -1;
  int64_t my_kv = -1;
  if (tid < BM) {
    const int r = r0 + tid, rc = min(r, g.rm.rows - 1);
    const int src = row_src(g.rm, rc);
    if constexpr (EK == E_QKV) my_kv = g.kv.slot_base[rc];
    const bool act = row_active(g.rm, r);
    my_src = act ? src : -1;
    row_src_s[tid] = my_src;
    row_mod_s[tid] = (g.mod_depth && my_src >= 0)
                         ? (g.mod_depth[g.mod_by_src ? my_src : r] - 1) * g.mod_ld : 0;
  }
  if (!__syncthreads_or(my_src >= 0)) return;
  load_a(0);

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int frow = lane & 15, quad = lane >> 4;
  auto multiply = [&](int st) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < BK / KS; ++ks) {
      const int k0 = ks * KS + quad * EPL;  // the lane's first element of this K step
      typename M::frag af[NA][MT], bfr[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int row = wm * MT * 16 + i * 16 + frow;
        const int off = row * BK + swz<T>(row, k0 / CE) * CE + k0 % CE;
#pragma unroll
        for (int a = 0; a < NA; ++a) af[a][i] = M::load(&As[st][a][off]);
      }
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int row = wn * NT * 16 + j * 16 + frow;
        bfr[j] = M::load(&Bs[st][row * BK + swz<T>(row, k0 / CE) * CE + k0 % CE]);
      }
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j) acc[i][j] = M::mma(af[a][i], bfr[j], acc[i][j]);
    }
  };
  // double-buffered LDS: tile kt + 1 loads into registers while tile kt is
  // multiplied, then goes to the other stage; one barrier per tile
  store_tiles(0);
  __syncthreads();
  for (int kt = 0; kt < KT; ++kt) {
    const int st = kt & 1;
    if (kt + 1 < KT) {
      load_b(kt + 1);
      load_a(kt + 1);
    }
    multiply(st);
    if (kt + 1 < KT) store_tiles(st ^ 1);
    __syncthreads();
  }
  if constexpr (EK == E_QKV) {
    if (tid < BM) kv_base[tid] = my_src >= 0 ? my_kv : -1;
    __syncthreads();
  }
  if constexpr (NORM) {
    static_assert(NTH % ACR == 0 && ACR <= kWave, "rows of the A chunks");
    // the ACR threads of a row are consecutive lanes of one wave
#pragma unroll
    for (int c = 0; c < ACH; ++c) {
      float t = ssq[c];
#pragma unroll
      for (int o = 1; o < ACR; o <<= 1) t += shfl_xor(t, o);
      if (tid % ACR == 0) row_inv_s[tid / ACR + c * (NTH / ACR)] = rsqrtf(t / (float)g.K + g.eps);
    }
    __syncthreads();
  }

  const int col16 = lane & 15;
  if constexpr (EK == E_QKV) {
    // q to its buffer; k and v into the cache pages (float32 models).  A
    // 16-column tile lies in one of q, k and v (d is a multiple of 16).  A q
    // tile goes through an in-group 4 x 4 transpose, after which lane t holds
    // four consecutive columns of row 4 quad + t: one 16-byte store.  k and v
    // tiles keep the lane's column: when the four rows of a v tile are
    // consecutive slots of one page from a multiple of 4 (a fresh prefill),
    // their values of that dimension are one aligned run in the V block and go
    // out as one store; otherwise element by element.  The tile's part, head
    // and first dimension are resolved once per tile.
    static_assert(sizeof(T) == 4, "bf16 models: pgemm.hip");
    T* pool = reinterpret_cast<T*>(g.kv.c.pool);
    const int t = col16 & 3;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      // the 16-column tile's first column (wave-uniform), its part (0: q,
      // 1: k, 2: v), head and first dimension: one division per tile
      const int nt = n0 + wn * NT * 16 + j * 16;
      if (nt >= g.N) continue;
      const int part = nt < g.d ? 0 : nt < 2 * g.d ? 1 : 2;
      const int w0 = nt - part * g.d, h = w0 / g.kv.c.D, e0 = w0 - h * g.kv.c.D;
      const int64_t kvb = part == 2 ? v_block(g.kv.c, g.kv.layer, h) : k_block(g.kv.c, g.kv.layer, h);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int rl0 = wm * MT * 16 + i * 16 + quad * 4;
        if (part == 0) {
          float v0 = acc[i][j][0], v1 = acc[i][j][1], v2 = acc[i][j][2], v3 = acc[i][j][3];
          transpose4(v0, v1, v2, v3, t);
          const int rl = rl0 + t, cw = col16 & ~3;  // the lane's first column in the tile
          if (row_src_s[rl] >= 0) {
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(g.out) + (int64_t)(r0 + rl) * g.ldo + nt + cw) =
                make_float4(v0, v1, v2, v3);
          }
          continue;
        }
        const int e = e0 + col16;
        const int64_t b0 = kv_base[rl0];
        const bool run4 = part == 2 && b0 >= 0 && (b0 & 3) == 0 && kv_base[rl0 + 1] == b0 + 1 &&
                          kv_base[rl0 + 2] == b0 + 2 && kv_base[rl0 + 3] == b0 + 3;
        if (run4) {
          const int slot = (int)(b0 & (kPage - 1));
          T* dst = pool + (b0 - slot) + kvb + v_frag_off(slot, e, g.kv.c.D);
          *reinterpret_cast<float4*>(dst) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
          continue;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t base = kv_base[rl0 + r];
          if (base < 0) continue;
          const int slot = (int)(base & (kPage - 1));
          const int64_t page = base - slot;
          const float v = acc[i][j][r];
          if (part == 1)
            pool[page + kvb + k_frag_off<T>(slot, e)] = from_f<T>(v);
          else
            pool[page + kvb + v_frag_off(slot, e, g.kv.c.D)] = from_f<T>(v);
        }
      }
    }
    return;
  }
  if constexpr (EK == E_RESID || EK == E_SWIGLU) {
    // lane t = col16 % 4 of each group of four writes row 4 quad + t of the
    // group's four columns (SwiGLU: four consecutive hidden units) as one
    // 16-byte access (the launcher checks that the widths allow it)
    const int t = col16 & 3;
    if constexpr (EK == E_RESID) {
      // The residual values of one row fragment (NT float4 per lane) are
      // loaded together, so the epilogue waits once per fragment instead of
      // once per 16 x 16 tile.  Inactive rows and columns past N read row 0
      // or the last four columns (in bounds) and store nothing.  With the
      // AdaLN gate (1 + alpha) per column, its values are loaded with them.
      float* out = reinterpret_cast<float*>(g.out);
      auto residual = [&](auto gate_c) __attribute__((always_inline)) {
        constexpr bool kGate = decltype(gate_c)::value;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          const int rl = wm * MT * 16 + i * 16 + quad * 4 + t;
          const int src = row_src_s[rl];
          const int64_t xo = (int64_t)(src < 0 ? 0 : src) * g.ldo;
          float4 xv[NT], gv[kGate ? NT : 1];
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            const int nb = min(n0 + wn * NT * 16 + j * 16 + (col16 & ~3), g.N - 4);
            xv[j] = *reinterpret_cast<const float4*>(out + xo + nb);
            if constexpr (kGate) gv[j] = *reinterpret_cast<const float4*>(g.mod_a + row_mod_s[rl] + nb);
          }
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            float v0 = acc[i][j][0], v1 = acc[i][j][1], v2 = acc[i][j][2], v3 = acc[i][j][3];
            transpose4(v0, v1, v2, v3, t);
            if constexpr (kGate) { v0 *= 1.f + gv[j].x; v1 *= 1.f + gv[j].y; v2 *= 1.f + gv[j].z; v3 *= 1.f + gv[j].w; }
            const int nb = n0 + wn * NT * 16 + j * 16 + (col16 & ~3);
            if (src >= 0 && nb < g.N)
              *reinterpret_cast<float4*>(out + xo + nb) =
                  make_float4(xv[j].x + v0, xv[j].y + v1, xv[j].z + v2, xv[j].w + v3);
          }
        }
      };
      if (g.mod_a) residual(std::true_type{});
      else residual(std::false_type{});
      return;
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int rl = wm * MT * 16 + i * 16 + quad * 4 + t;
      const int src = row_src_s[rl];
      if constexpr (EK == E_SWIGLU) {
#pragma unroll
        for (int j = 0; j < NT; j += 2) {
          // gate columns j, up columns j + 1 of the same 16 hidden units;
          // silu(g) = g / (1 + e^-g) with the hardware reciprocal (within an
          // ulp of the division, which took ~10 instructions per unit while
          // every workgroup of the round was in its epilogue)
          float h[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float gt = acc[i][j][r], up = acc[i][j + 1][r];
            h[r] = gt * __builtin_amdgcn_rcpf(1.f + __expf(-gt)) * up;
          }
          transpose4(h[0], h[1], h[2], h[3], t);
          const int n = n0 + wn * NT * 16 + j * 16;  // first gate column of the group
          const int unit = (n >> 5) * 16 + (col16 & ~3);
          if (src < 0 || unit >= g.F) continue;
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(g.out) + (int64_t)(r0 + rl) * g.ldo + unit) =
              make_float4(h[0], h[1], h[2], h[3]);
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rl = wm * MT * 16 + i * 16 + quad * 4 + r;
      const int src = row_src_s[rl];
      const int rg = r0 + rl;
      const float rs = NORM ? row_inv_s[rl] : 1.f;
      if constexpr (EK == E_LOGITS) {
        static_assert(NT * 16 % 64 == 0, "whole greedy key groups per wave");
        // compact rows (A_CMP) write their logits to row src(r), the sequence's
        const int orow = AK == A_CMP ? src : g.out_row_off + rg;
#pragma unroll
        for (int j0 = 0; j0 < NT; j0 += 4) {  // one key group: 4 x 16 columns
          unsigned long long best = 0ull;
#pragma unroll
          for (int j = j0; j < j0 + 4; ++j) {
            const int n = n0 + wn * NT * 16 + j * 16 + col16;
            const float v = acc[i][j][r] * rs;
            if (src >= 0 && n < g.N) {
              reinterpret_cast<float*>(g.out)[(int64_t)orow * g.ldo + n] = v;
              const unsigned long long key =
                  ((unsigned long long)ordered_bits(v) << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)n);
              best = key > best ? key : best;
            }
          }
          if (g.argmax_keys) {
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) {
              const unsigned long long other = shfl_xor(best, o);
              best = other > best ? other : best;
            }
            if (col16 == 0 && src >= 0 && best != 0ull)
              g.argmax_keys[(int64_t)orow * g.key_groups + (n0 + wn * NT * 16 + j0 * 16) / 64] = best;
          }
        }
      } else if constexpr (EK == E_HIDDEN) {  // the other epilogues return above
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const int n = n0 + wn * NT * 16 + j * 16 + col16;
          if (src < 0 || n >= g.N) continue;
          const float u = acc[i][j][r] + g.bias[n];
          g.out[(int64_t)rg * g.ldo + n] = u / (1.f + __expf(-u));
        }
      }
    }
  }
}

template <typename T, int MT, int NT, int BK, int AK, int EK, bool MOD, bool NORM>
__global__ __launch_bounds__(256, 2) void k_gemm(GemmArgs g) {
  constexpr int BM = 2 * MT * 16, BN = 2 * NT * 16;
  __shared__ __align__(16) T As[2][sizeof(T) == 2 ? 2 : 1][BM * BK];
  __shared__ __align__(16) T Bs[2][BN * BK];
  __shared__ int row_src_s[BM];
  __shared__ int row_mod_s[BM];
  __shared__ float row_inv_s[NORM ? BM : 1];
  __shared__ int64_t kv_base[EK == E_QKV ? BM : 1];
  gemm_tile<T, MT, NT, BK, AK, EK, MOD, NORM>(g, blockIdx.y * BM, blockIdx.x * BN, As, Bs, row_src_s, row_mod_s,
                                              row_inv_s, kv_base);
}

template <typename T, int MT, int NT>
hipError_t launch_tiles(const GemmArgs& a, AKind ak, EKind ek, bool norm, hipStream_t s) {
  constexpr int BM = 2 * MT * 16, BN = 2 * NT * 16;
  const dim3 grid((a.N + BN - 1) / BN, (a.rm.rows + BM - 1) / BM);
  if (grid.x == 0 || grid.y == 0) return hipSuccess;
  const bool mod = a.mod_g != nullptr;
#define TLF_GEMM_CASE(AKV, EKV, MODV, NORMV)                                                                        \
  if (ak == AKV && ek == EKV && mod == MODV && norm == NORMV) {                                                     \
    hipLaunchKernelGGL((k_gemm<T, MT, NT, kGemmBK, AKV, EKV, MODV, NORMV>), grid, dim3(256), 0, s, a);              \
    return hipGetLastError();                                                                                       \
  }
  if constexpr (sizeof(T) == 4) {  // bf16 models' prefill projections: launch_pgemm
    TLF_GEMM_CASE(A_SRC, E_QKV, false, false)
    TLF_GEMM_CASE(A_SRC, E_QKV, true, false)
    TLF_GEMM_CASE(A_SRC, E_SWIGLU, false, false)
    TLF_GEMM_CASE(A_SRC, E_SWIGLU, true, false)
    TLF_GEMM_CASE(A_CMP, E_RESID, false, false)
    TLF_GEMM_CASE(A_SRC, E_LOGITS, false, false)
  }
  TLF_GEMM_CASE(A_CMP, E_LOGITS, false, true)
  TLF_GEMM_CASE(A_CMP, E_HIDDEN, false, false)
#undef TLF_GEMM_CASE
  return hipErrorInvalidValue;
}

}  // namespace

template <typename T>
hipError_t launch_gemm(const GemmArgs& a, AKind ak, EKind ek, bool norm, hipStream_t s) {
  if (a.K % kGemmBK != 0) return hipErrorInvalidValue;
  // float A in fragment order: bf16 weights (8 consecutive k per run), compact rows
  if (a.a_frag && (sizeof(T) != 2 || ak != A_CMP)) return hipErrorInvalidValue;
  // the QKV epilogue takes each 16-column tile as wholly q, k or v
  if (ek == E_QKV && (a.d % 16 != 0 || a.ldo % 4 != 0 || a.kv.c.D % 16 != 0)) return hipErrorInvalidValue;
  // the residual and SwiGLU epilogues write four consecutive columns at once
  if ((ek == E_RESID && (a.N % 4 != 0 || a.ldo % 4 != 0 || (a.mod_a && a.mod_ld % 4 != 0))) ||
      (ek == E_SWIGLU && (a.F % 4 != 0 || a.ldo % 4 != 0)))
    return hipErrorInvalidValue;
  // a few row tiles (the decode LM head) take 128-column tiles so the grid
  // still holds about two workgroups per compute unit; prefill takes 256
  const int row_tiles = (a.rm.rows + 2 * kGemmMT * 16 - 1) / (2 * kGemmMT * 16);
  if (row_tiles <= 4) return launch_tiles<T, kGemmMT, 4>(a, ak, ek, norm, s);
  return launch_tiles<T, kGemmMT, 8>(a, ak, ek, norm, s);
}

template hipError_t launch_gemm<float>(const GemmArgs&, AKind, EKind, bool, hipStream_t);
template hipError_t launch_gemm<bf16>(const GemmArgs&, AKind, EKind, bool, hipStream_t);

}  // namespace tlf
