// Look-ahead forward of chunkwise triadic linear attention on gfx950 (bf16
// operands, K >= 64, E >= 4): the prep kernel with the cross-chunk tiles, and the
// recurrent forward.  See tla_la.hpp for the algebra.
// Part of tla_fwd.hip, which alone includes it: one translation unit, and so one
// code object, for the training and the inference forward.
#pragma once
#include "tla_la.hpp"

namespace tla {

// ------------------------------------------------------------------- prep
// One workgroup per (head, chunk).  As k_prep (in-chunk cumulative log-gates
// in fp64, coefficient vectors, decayed Grams, M, Tu by the blocked inverse),
// with every C x C tile formed transposed on the matrix cores (A: the rows of
// the columns' side), so that an accumulator is already the A operand that
// the recurrences read and leaves as whole 16-byte pieces without a shared
// copy, and with the tiles G between this chunk and the one before.
template <int KD, int C, int E>
struct LaPrepSmem {
  static constexpr int KP = KD + 8;  // 16-byte rows, conflict-free 16-byte fragment reads
  static constexpr int CP = C + 4;
  static constexpr int NT = C / 16;
  union U {
    struct { bf16_t sQ[C][KP]; bf16_t sK[C][KP]; } qk;
    struct { float X[C][CP]; float Y[NT > 1 ? NT - 1 : 1][16][17]; } inv;
  };
  alignas(16) U u;
  alignas(16) float L[C][CP];  // diag(beta)(A_kk o R), strictly lower (the upper part is not formed)
  alignas(16) float q2[C][E];
  alignas(16) float k2[C][E];
  alignas(16) double G[C][E];  // in-chunk cumulative log-gates
  alignas(16) float cp[C][E];  // c of the chunk before: k2 gamma^C / gamma
  alignas(16) float beta[C];
};

// Eight waves for E <= 8 (two workgroups a CU, 128 registers a lane), four above.
template <int E> constexpr int la_prep_waves() { return E <= 8 ? 8 : 4; }

// Eight values (two fragments) as a (hi, lo) operand: the parts are FR elements apart.
__device__ __forceinline__ void store_op(bf16_t* dst, f32x4 x0, f32x4 x1) {
  bf16x4 h0, l0, h1, l1;
  split_frag(x0, h0, l0);
  split_frag(x1, h1, l1);
  gstore_b128(dst, __builtin_bit_cast(u32x4, __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7)));
  gstore_b128(dst + 512, __builtin_bit_cast(u32x4, __builtin_shufflevector(l0, l1, 0, 1, 2, 3, 4, 5, 6, 7)));
}

template <int KD, int C, int E>
__global__ __launch_bounds__(la_prep_waves<E>() * 64, E <= 8 ? 4 : 2) void k_prep_la(Shape s, FwdIn in, PrepBufs p) {
  typedef bf16_t T;
  constexpr int NW = la_prep_waves<E>(), NTHR = NW * 64;
  constexpr int NT = C / 16, NP = NT / 2;
  constexpr int E4 = (E + 3) & ~3;
  constexpr int KB = KD / 32;
  typedef LaPrepSmem<KD, C, E> Sm;
  typedef LaOps<KD, C> OT;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Sm& sm = *reinterpret_cast<Sm*>(smem_raw);

  const int ch = blockIdx.x;
  const int head = ch / s.Nc, ci = ch % s.Nc;
  const int b = head / s.H, h = head % s.H;
  const int t0 = ci * C;
  const int tid = threadIdx.x;
  const size_t tok0 = seq_begin(s, b);
  s.T = seq_len(s, b);
  if (t0 >= s.T) return;  // past the end of a shorter packed sequence
  const int w = wave_id(), l = lane_id(), g = l >> 4, n = l & 15;
  const size_t krs = (size_t)s.H * KD;
  const T* Qg = (const T*)in.q + (tok0 * s.H + h) * KD;
  const T* Kg = (const T*)in.k + (tok0 * s.H + h) * KD;
  const size_t eoff = (tok0 * s.H + h) * E, erow = (size_t)s.H * E;
  const bool prev = ci > 0;  // the chunk before is a whole one
  // G couples the retrieval of this chunk to the chunk before (GDN)
  const bool need_g = prev && s.variant == 1;

  // ---- every global load of the phase before the first of the stores
  constexpr int NQE = (C * E + NTHR - 1) / NTHR;
  constexpr int IT = (C * KD / 8 + NTHR - 1) / NTHR;
  constexpr int NGE = (E + NW - 1) / NW;
  float q2v[NQE], k2v[NQE], bv = 0.f, k2p[NGE];
  Raw8<T> qv[IT], kv[IT];
  double gv[NGE], gp[NGE];
#pragma unroll
  for (int i = 0; i < NQE; ++i) {
    const int idx = min(tid + NTHR * i, C * E - 1), r = idx / E, e = idx % E;
    const size_t off = eoff + (size_t)min(t0 + r, s.T - 1) * erow + e;
    q2v[i] = ld_f((const T*)in.q2 + off);
    k2v[i] = ld_f((const T*)in.k2 + off);
  }
  if (tid < C) {
    const int t = min(t0 + tid, s.T - 1);
    bv = in.beta ? in.beta[(tok0 + t) * s.H + h] : 1.f;
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int idx = min(tid + NTHR * it, C * KD / 8 - 1);
    const int r = idx / (KD / 8), c8 = idx % (KD / 8);
    const size_t off = (size_t)min(t0 + r, s.T - 1) * krs + 8 * c8;
    qv[it] = load8(Qg + off);
    kv[it] = load8(Kg + off);
  }
  const int tp = need_g ? t0 - C : t0;  // first position of the chunk before (or, not needed, of this one)
#pragma unroll
  for (int i = 0; i < NGE; ++i) {
    const int e = min(w + NW * i, E - 1);
    gv[i] = (double)in.g[eoff + (size_t)min(t0 + l, s.T - 1) * erow + e];
    const size_t offp = eoff + (size_t)min(tp + min(l, C - 1), s.T - 1) * erow + e;
    gp[i] = (double)in.g[offp];
    k2p[i] = ld_f((const T*)in.k2 + offp);
  }
  // ---- the stores
#pragma unroll
  for (int i = 0; i < NQE; ++i) {
    const int idx = tid + NTHR * i, r = idx / E, e = idx % E;
    if (idx >= C * E) continue;
    const bool ok = t0 + r < s.T;
    sm.q2[r][e] = ok ? q2v[i] : 0.f;
    sm.k2[r][e] = ok ? k2v[i] : 0.f;
  }
  if (tid < C) sm.beta[tid] = (t0 + tid < s.T) ? bv : 0.f;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int idx = tid + NTHR * it;
    if (idx >= C * KD / 8) continue;
    const int r = idx / (KD / 8), c8 = idx % (KD / 8);
    const bool ok = t0 + r < s.T;
    *(Raw8<T>*)&sm.u.qk.sQ[r][8 * c8] = ok ? qv[it] : zero_raw8<T>();
    *(Raw8<T>*)&sm.u.qk.sK[r][8 * c8] = ok ? kv[it] : zero_raw8<T>();
  }
  // G: inclusive cumulative sum over the chunk in fp64 (one wave per slice,
  // lane r holds row r), and c of the chunk before from its own sums
#pragma unroll
  for (int i = 0; i < NGE; ++i) {
    const int e = w + NW * i;
    if (e >= E) continue;  // wave-uniform
    double x = (l < C && t0 + l < s.T) ? gv[i] : 0.0;
    double y = (l < C) ? gp[i] : 0.0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double xo = __shfl_up(x, off, 64), yo = __shfl_up(y, off, 64);
      if (l >= off) {
        x += xo;
        y += yo;
      }
    }
    const double yC = __shfl(y, C - 1, 64);
    if (l < C) {
      sm.G[l][e] = x;
      sm.cp[l][e] = k2p[i] * exp_nonpos((float)(yC - y));
    }
  }
  __syncthreads();

  // K rows of the chunk before for the wave's first pair of cross-chunk tiles,
  // in flight under the Grams
  Raw8<T> kp[2][KB];
  auto load_prev = [&](int pp) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        kp[hh][kb] = load8(Kg + (size_t)min(tp + 16 * (2 * pp + hh) + n, s.T - 1) * krs + 32 * kb + 8 * g);
  };
  load_prev(w % NP);

  // ---- coefficient vectors a = k2 gamma, b = q2 gamma, c = k2 gamma^C / gamma; gamma^C
  float* coef = p.coef + (size_t)ch * 3 * E * C;
  for (int idx = tid; idx < E * C / 4; idx += NTHR) {
    const int e = idx / (C / 4), r0 = 4 * (idx % (C / 4));
    const double GC = sm.G[C - 1][e];
    f32x4 a, bq, c;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const double G = sm.G[r0 + j][e];
      const float gam = exp_nonpos((float)G);
      a[j] = sm.k2[r0 + j][e] * gam;
      bq[j] = sm.q2[r0 + j][e] * gam;
      c[j] = sm.k2[r0 + j][e] * exp_nonpos((float)(GC - G));
    }
    gstore_b128(coef + (0 * E + e) * C + r0, __builtin_bit_cast(u32x4, a));
    gstore_b128(coef + (1 * E + e) * C + r0, __builtin_bit_cast(u32x4, bq));
    gstore_b128(coef + (2 * E + e) * C + r0, __builtin_bit_cast(u32x4, c));
  }
  if (tid < E4) p.gC[(size_t)ch * E4 + tid] = (tid < E) ? exp_nonpos((float)sm.G[C - 1][tid]) : 0.f;

  auto qrow8 = [&](int r, int col) -> Raw8<T> { return *(const Raw8<T>*)&sm.u.qk.sQ[r][col]; };
  auto krow8 = [&](int r, int col) -> Raw8<T> { return *(const Raw8<T>*)&sm.u.qk.sK[r][col]; };
  T* ops = (T*)p.ops + (size_t)ch * OT::STRIDE;

  // ---- M and L: operand (rt, pp) is the tile pair (rt, 2 pp), (rt, 2 pp + 1);
  // lane (g, n) holds row r = 16 rt + n, columns 16 st + 4 g + j
  for (int pair = w; pair < OT::NTRI; pair += NW) {
    int rt = 0;
    while (OT::tri(rt + 1, 0) <= pair) ++rt;
    const int pp = pair - OT::tri(rt, 0);
    const int r = 16 * rt + n;
    f32x4 mv[2];
    const float br = sm.beta[r];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int st = 2 * pp + hh;
      mv[hh] = zero4();
      if (st > rt) continue;  // wave-uniform
      f32x4 aq = zero4(), ak = zero4();
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const int col = 32 * kb + 8 * g;
        const Raw8<T> ka = krow8(16 * st + n, col);
        mma8(aq, ka, qrow8(r, col));
        mma8(ak, ka, krow8(r, col));
      }
      f32x4 lv;
      if (st < rt) {
        // every pair of the tile has the tile's last column m between c and r:
        // Gamma = exp(G_r - G_m) exp(G_m - G_c), both exponents non-positive, and
        // the sum over slices is a product on the fp32 MFMA (four slices a
        // step): E / 2 exponentials a lane instead of 4 E
        f32x4 rq = zero4(), rk = zero4();
        const int m = 16 * st + 15, cn = 16 * st + n;
#pragma unroll
        for (int q = 0; q < E / 4; ++q) {
          const int e = 4 * q + g;
          const double Gm = sm.G[m][e];
          const float u = exp_nonpos((float)(sm.G[r][e] - Gm));
          const float v = sm.k2[cn][e] * exp_nonpos((float)(Gm - sm.G[cn][e]));
          rq = __builtin_amdgcn_mfma_f32_16x16x4f32(v, sm.q2[r][e] * u, rq, 0, 0, 0);
          rk = __builtin_amdgcn_mfma_f32_16x16x4f32(v, sm.k2[r][e] * u, rk, 0, 0, 0);
        }
        mv[hh] = aq * rq;
        lv = br * ak * rk;
      } else {
        double Gr[E];
        float q2r[E], k2r[E];
        lds_row<E>(Gr, &sm.G[r][0]);
        lds_row<E>(q2r, &sm.q2[r][0]);
        lds_row<E>(k2r, &sm.k2[r][0]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = 16 * st + 4 * g + j;
          double Gc[E];
          float k2c[E];
          lds_row<E>(Gc, &sm.G[c][0]);
          lds_row<E>(k2c, &sm.k2[c][0]);
          float rq = 0.f, rk = 0.f;
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const float d = exp_nonpos((float)(Gr[e] - Gc[e])) * k2c[e];
            rq += q2r[e] * d;
            rk += k2r[e] * d;
          }
          mv[hh][j] = (c <= r) ? aq[j] * rq : 0.f;
          lv[j] = (c < r) ? br * ak[j] * rk : 0.f;
        }
      }
      *(f32x4*)&sm.L[r][16 * st + 4 * g] = lv;
    }
    store_op(ops + OT::M + (size_t)pair * 2 * OT::FR + 8 * l, mv[0], mv[1]);
  }
  // ---- G: K rows of the chunk before from global memory, the rank-E
  // factor sum_e a_e c_e^T on the fp32 MFMA (four slices a step)
  if (need_g) {
    for (int pair = w; pair < NT * NP; pair += NW) {
      const int rt = pair / NP, pp = pair % NP;
      static_assert(NW % NP == 0, "every pair of a wave has the same columns");
      // a_e of row r, slice 4 q + g
      auto av = [&](int r, int q) {
        return sm.k2[r][4 * q + g] * exp_nonpos((float)sm.G[r][4 * q + g]);
      };
      // rows r of this chunk (tile rt), columns s of the one before (tiles 2 pp, 2 pp + 1)
      f32x4 x[2];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        f32x4 ak = zero4(), rr = zero4();
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) mma8(ak, kp[hh][kb], krow8(16 * rt + n, 32 * kb + 8 * g));
#pragma unroll
        for (int q = 0; q < E / 4; ++q)
          rr = __builtin_amdgcn_mfma_f32_16x16x4f32(sm.cp[16 * (2 * pp + hh) + n][4 * q + g],
                                                    av(16 * rt + n, q), rr, 0, 0, 0);
        x[hh] = ak * rr;
      }
      store_op(ops + OT::G + (size_t)OT::full(rt, pp) * 2 * OT::FR + 8 * l, x[0], x[1]);
    }
  }
  // ---- K^T, read out of the staged rows column-wise
  for (int idx = tid; idx < KD * C / 8; idx += NTHR) {
    int R, c8;
    SwzTile<T, KD, C>::logical(idx, R, c8);
    const int key = la_key(R);
    uint32_t wd[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p0 = 8 * c8 + 2 * i;
      const uint16_t v0 = sm.u.qk.sK[p0][key], v1 = sm.u.qk.sK[p0 + 1][key];
      wd[i] = (uint32_t)v0 | ((uint32_t)v1 << 16);
    }
    gstore_b128(ops + OT::Kt + (size_t)8 * idx, u32x4{wd[0], wd[1], wd[2], wd[3]});
  }
  if (s.variant != 1) return;
  __syncthreads();

  // ---- Tu = (I + L)^{-1} diag(beta), blocked unit-lower inverse in fp32
  unit_lower_inverse<C, NTHR>([&](int r, int c) { return sm.L[r][c]; }, &sm.u.inv.X[0][0], Sm::CP,
                              &sm.u.inv.Y[0][0][0]);
  for (int pair = w; pair < OT::NTRI; pair += NW) {
    int rt = 0;
    while (OT::tri(rt + 1, 0) <= pair) ++rt;
    const int c = 32 * (pair - OT::tri(rt, 0)) + 4 * g;
    const float* src = &sm.u.inv.X[16 * rt + n][c];
    store_op(ops + OT::Tu + (size_t)pair * 2 * OT::FR + 8 * l, *(const f32x4*)src * *(const f32x4*)&sm.beta[c],
             *(const f32x4*)(src + 16) * *(const f32x4*)&sm.beta[c + 16]);
  }
}

// ---------------------------------------------------------------- forward
// One workgroup per (head, value tile), sequential over chunks, eight waves in
// two roles.  Waves 0..3 (state waves) own the fp32 state and run
// S_{c+1} = gamma^C S_c + K_c^T diag(c) U_c; they also issue and await the
// copies into shared memory.  Waves 4..7 (row waves; wave 4 + w shares a SIMD
// with state wave w) own row tile w of the chunk: from the bf16 copy of S_c in
// shared memory they form, in one pass over it, their rows of the retrieval
// of chunk c + 1 and of the output of chunk c, then X = V - W and
// U_{c+1} = Tu X, and store the outputs.  Two barriers a step:
//   B0 .. B1  state: the update's first half   row: O_c, X_{c+1}
//   B1 .. B0  state: second half, copy of S    row: U_{c+1}, stores
// (GDN's last step has no B1: nothing is written to shared memory after it.)
// A row tile's partial sums over slices stay in registers (no exchange), and
// the row waves read K, Q, M, G and Tu straight from global memory into
// registers, each a whole step ahead, in operand order.
//
// State tiles are 32 keys x 32 columns (v_mfma_f32_32x32x16_bf16: one wave
// issues those back to back at 97% of the matrix rate, 16x16x32 ones at 59%).
// The 32 columns are a "unit": two slices of 16 value columns, or with PK four
// slices of 8, which halves a workgroup's work and doubles the workgroups.
// Row waves work on 16x16x32 products formed transposed (rows: columns of the
// state, columns: chunk rows): a lane then holds one chunk row, so that its
// coefficient of a slice is one word, and four adjacent value columns, so that
// rows of X, U and O leave as they are; the (hi, lo) rows of X and U are
// kept row-major and come back as operands through transposing reads.  (Row
// tiles of K stacked on Q in 32-row products were slower: 32 lines a load.)
//
// With two row tiles (C = 32) a tile has two row waves, one for K's rows (X, U)
// and one for Q's (outputs): with both sides in one wave and two waves idle an
// instance took 160-180 registers, one workgroup a CU, and calls of many
// sequences were slower than before the look-ahead (GDN K64 E8, whole forwards,
// kernel whose W waits for the update / one wave a tile / two waves a tile: B32
// H16 T512 268 / 326 / 243 us, B64 H16 T64 93 / 123 / 92 us, B1 H8 T4096 262 /
// 180 / 155 us; K128 E8 B64 H16 T64 292 / 313 / 261 us).
//
// Measured (kernel alone, MI355X, before / after: the kernel whose W waits for
// the update): GDN B1 H16 T65536 E16 3.85 / 2.95 ms, GDN B1 H16 T777 E8 58 /
// 36 us, sGLA B4 H8 T4096 E8 177 / 124-129 us.  A GDN step takes 6.8 k cycles,
// 5.2 k without its memory operations.  Counters (GDN B4 H8 T4096 E8, 180 us; in
// brackets B1 H16 T65536 E16): matrix cores busy 34% (36%) of the cycles, shared
// memory active 33% (40%) with 0.19 (0.27) conflict cycles each, waves waiting
// 25% (25%) of their time: bound by the chain of a step through its two barriers,
// not by one unit.
//
// GDN: every LA_SYNC-th chunk forms its W from its own start state instead (two
// more barriers): a sequence cut there and resumed from the handed-on fp32
// state then repeats the uncut one bit for bit (elsewhere the two differ by
// where the state's bf16 operand copy was rounded: 4e-5 of the outputs at E = 8,
// cut at 512 of 812 tokens).  sGLA, whose U needs no state, repeats it at every
// chunk boundary.
constexpr int LA_SYNC = 16;

template <int KD, int C, int E, bool PK>
struct LaFwdSmem {
  static constexpr int NT = C / 16, NP = NT / 2, KB = KD / 16;
  static constexpr int SPU = PK ? 4 : 2, UE = E / SPU;  // slices in a unit, units
  static constexpr int E4 = (E + 3) & ~3;
  alignas(16) bf16x8 sop[UE][KB][64];  // copy of S_c: [unit][16-key block][lane]
  SwzTile<bf16_t, KD, C> Kt[2];
  alignas(16) float ca[2][E][C];      // a_e (chunk c + 1)
  alignas(16) float cbc[2][2][E][C];  // b_e, c_e (chunk c)
  alignas(16) float gC[2][E4 < 64 ? 64 : E4];
  alignas(16) float beta[2][C];
  alignas(16) bf16_t V[2][C][16];
  alignas(16) float Uf[C][16];       // U_c
  alignas(16) bf16_t Uo[2][C][16];   // U_c as (hi, lo)
  alignas(16) bf16_t Xo[2][C][16];   // X_{c+1} likewise
};

template <int KD, int C, int E, bool PK, bool GDN>
__global__ __launch_bounds__(512, C == 32 ? 4 : 2) void k_fwd_la(Shape s, FwdIn in, PrepBufs p, void* out,
                                                   float* s_final) {
  typedef bf16_t T;
  typedef LaFwdSmem<KD, C, E, PK> Sm;
  typedef LaOps<KD, C> OT;
  constexpr int NT = Sm::NT, NP = Sm::NP, KB = Sm::KB, UE = Sm::UE, SPU = Sm::SPU, E4 = Sm::E4;
  constexpr int VW = PK ? 8 : 16, KT = KD / 32;
  constexpr int NKT = UE * KT / 4;  // state tiles of a state wave
  static_assert(UE >= 1 && (UE * KT) % 4 == 0 && (NKT <= KT) && (NT == 2 || NT == 4),
                "one unit per state wave, one row tile per row wave");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Sm& sm = *reinterpret_cast<Sm*>(smem_raw);

  const int wv = wave_id(), w = wv & 3, l = lane_id(), g = l >> 4, n = l & 15;
  const int hf = l >> 5, nn = l & 31;
  const int V = s.V;
  int head, vt;
  xcd_map(blockIdx.x, s.NH, V / VW, head, vt);
  const int b = head / s.H, h = head % s.H;
  const int v0 = vt * VW;
  const int vc = nn & (VW - 1);                            // this lane's value column
  auto slc = [&](int u) { return SPU * u + nn / VW; };     // and slice in unit u
  const size_t tok0 = seq_begin(s, b);
  s.T = __builtin_amdgcn_readfirstlane(seq_len(s, b));  // this sequence's length from here on
  const int nc = (s.T + C - 1) / C;    // its chunks (s.Nc: the per-head stride)
  const size_t ch0 = (size_t)head * s.Nc;
  const T* opsg = (const T*)p.ops + ch0 * OT::STRIDE;
  // chunks whose U is formed from their own start state (GDN; sGLA's U needs
  // no state): the first, and every SYNC-th
  auto direct = [](int c) { return GDN ? c % LA_SYNC == 0 : c == 0; };

  if (wv < 4) {
    // ================================================= state waves
    // S[i]: key tile kt0 + i (rows in the order of la_key) of unit un
    const int un = w * NKT / KT, kt0 = w * NKT % KT, e = slc(un);
    f32x16 S[NKT];
    auto state_ptr = [&](auto* base, int i, int a) {  // keys of registers 4 a .. 4 a + 3
      return base + (((size_t)head * E + e) * KD + 32 * (kt0 + i) + la_key(8 * a + 4 * hf)) * V + v0 + vc;
    };
    auto put_sop = [&]() {
#pragma unroll
      for (int i = 0; i < NKT; ++i)
#pragma unroll
        for (int k = 0; k < 2; ++k) sm.sop[un][2 * (kt0 + i) + k][l] = half_op(S[i], k);
    };
    const T* Vg = (const T*)in.v + (tok0 * s.H + h) * (size_t)V + v0;
    const size_t vrs = (size_t)s.H * V;
    const bool sbeta = !GDN && in.beta != nullptr;
    const float* bg = sbeta ? in.beta + tok0 * s.H + h : nullptr;
    const uint32_t off16 = 16 * l;
    // NB bytes (a multiple of 1 KiB), pieces dealt to the waves starting at wave W0
    auto lin = [&](auto nb, int w0, void* dst, const void* src) {
      constexpr int NK = decltype(nb)::value / 1024;
#pragma unroll
      for (int i = 0; i < (NK + 3) / 4; ++i) {
        const int k = 4 * i + ((w + w0) & 3);
        if (NK % 4 == 0 || k < NK) dma_kib((char*)dst + 1024 * k, (const char*)src + 1024 * k, off16);
      }
    };
    // V rows of chunk c (rows past T read row T - 1), 16-byte pieces; PK: the
    // eight columns fill both halves of each row
    auto dma_v = [&](int c) {
      constexpr int VL = C * 2 / 4;
      const int q = w * VL + l, r = q >> 1, last = s.T - 1 - c * C;
      const uint32_t off = (uint32_t)(2 * (size_t)min(r, last) * vrs) + (PK ? 0 : 16 * (q & 1));
      if (l < VL) lds_dma<16>(uniform_ptr(Vg + (size_t)c * C * vrs), off, lds_addr(&sm.V[c & 1][0][0]) + 16 * w * VL);
    };
    auto dma_beta = [&](int c) {
      constexpr int BL = C / 4;
      const int last = s.T - 1 - c * C;
      const uint32_t off = (uint32_t)(4 * (size_t)min(w * BL + l, last) * s.H);
      if (l < BL) lds_dma<4>(uniform_ptr(bg + (size_t)c * C * s.H), off, lds_addr(&sm.beta[c & 1][0]) + 4 * w * BL);
    };
    auto dma_a = [&](int c) {
      if constexpr (GDN)
        lin(std::integral_constant<int, E * C * 4>{}, 0, &sm.ca[c & 1][0][0], p.coef + (ch0 + c) * 3 * E * C);
      dma_v(c);
      if (sbeta) dma_beta(c);
    };
    auto dma_k = [&](int c) {
      lin(std::integral_constant<int, KD * C * 2>{}, 0, sm.Kt[c & 1].d, opsg + c * OT::STRIDE + OT::Kt);
      lin(std::integral_constant<int, 2 * E * C * 4>{}, 0, &sm.cbc[c & 1][0][0][0],
          p.coef + (ch0 + c) * 3 * E * C + E * C);
      if (w == 3 && l < E4) lds_dma<4>(uniform_ptr(p.gC + (ch0 + c) * E4), 4 * l, lds_addr(&sm.gC[c & 1][0]));
    };
    // The first copies go out before the initial state is read (one memory latency
    // for both) where that is faster.  After / before, whole calls: GDN K64 E16 B64
    // H16 T64 217 / 211 us, B1 H8 T4096 152 / 150, the forward kernel of K128 E16
    // B64 H16 T64 with an initial state 726 / 712; but sGLA K128 E8 B64 H16 T64 224 /
    // 238 and GDN at C = 32 (K128 E8 B64 H16 T64) 231 / 240.
    constexpr bool COPIES_FIRST = GDN && NT == 4;
    auto copies = [&]() {
      if (nc == 0) return;
      dma_a(0);
      dma_k(0);
      if (nc > 1) dma_a(1);
    };
    if constexpr (COPIES_FIRST) copies();
#pragma unroll
    for (int i = 0; i < NKT; ++i) {
      S[i] = zero16();
      if (in.s0) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int j = 0; j < 4; ++j) S[i][4 * a + j] = state_ptr(in.s0, i, a)[(size_t)j * V];
      }
    }
    if (nc > 0) {
      put_sop();
      if constexpr (!COPIES_FIRST) copies();
      wait_vmcnt<0>();
    }
    for (int c = 0; c < nc; ++c) {
      block_sync();  // B0
      if (direct(c)) {
        block_sync();  // the row waves' X_c
        block_sync();  // and U_c, from S_c itself
      }
      if (c + 1 < nc) dma_k(c + 1);
      if (c + 2 < nc) dma_a(c + 2);
      // diag(c_e) U: this lane's column, positions 16 pb + 8 hf + 0..7
      bf16x8 Uh[NT], Ul[NT];
#pragma unroll
      for (int pb = 0; pb < NT; ++pb) {
        bf16x4 h[2], lo[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int r0 = 16 * pb + 8 * hf + 4 * k;
          const f32x4 u = {sm.Uf[r0][n], sm.Uf[r0 + 1][n], sm.Uf[r0 + 2][n], sm.Uf[r0 + 3][n]};
          split_frag(u * *(const f32x4*)&sm.cbc[c & 1][1][e][r0], h[k], lo[k]);
        }
        Uh[pb] = join8(h[0], h[1]);
        Ul[pb] = join8(lo[0], lo[1]);
      }
      const float gc = sm.gC[c & 1][e];
#pragma unroll
      for (int i = 0; i < NKT; ++i) S[i] *= gc;
#pragma unroll
      for (int pb = 0; pb < NT; ++pb) {
        bf16x8 a[NKT];
#pragma unroll
        for (int i = 0; i < NKT; ++i) a[i] = *(const bf16x8*)sm.Kt[c & 1].at(32 * (kt0 + i) + nn, 16 * pb + 8 * hf);
#pragma unroll
        for (int i = 0; i < NKT; ++i) S[i] = mma_32(a[i], Uh[pb], S[i]);
#pragma unroll
        for (int i = 0; i < NKT; ++i) S[i] = mma_32(a[i], Ul[pb], S[i]);
        // B1: the row waves are done with the copy of S_c
        if (pb == NT / 2 - 1 && (!GDN || c + 1 < nc)) block_sync();
      }
      if (c + 1 < nc) put_sop();
      wait_vmcnt<0>();  // the copies issued at the top of the step
    }
    wait_vmcnt<0>();
    if (s_final) {
#pragma unroll
      for (int i = 0; i < NKT; ++i)
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int j = 0; j < 4; ++j) state_ptr(s_final, i, a)[(size_t)j * V] = S[i][4 * a + j];
    }
  } else {
    // ================================================= row waves
    if (nc == 0) return;
    const int rt = w & (NT - 1);  // the wave's row tile
    const int pw = rt >> 1;       // last operand of its rows in a triangular matrix
    if constexpr (!GDN) {
      if (!in.beta)
        for (int r = threadIdx.x - 256; r < 2 * C; r += 256) (&sm.beta[0][0])[r] = 1.f;
    }
    bf16x8 mo[NP][2], go[NP][2], to[NP][2];
    auto load_tri = [&](bf16x8(&x)[NP][2], size_t mat, int c) {
      const T* src = opsg + (size_t)min(c, nc - 1) * OT::STRIDE + mat + (size_t)OT::tri(rt, 0) * 2 * OT::FR + 8 * l;
#pragma unroll
      for (int pp = 0; pp < NP; ++pp)
        if (pp <= pw) {
          x[pp][0] = *(const bf16x8*)(src + (2 * pp) * OT::FR);
          x[pp][1] = *(const bf16x8*)(src + (2 * pp + 1) * OT::FR);
        }
    };
    auto load_full = [&](bf16x8(&x)[NP][2], size_t mat, int c) {
      const T* src = opsg + (size_t)min(c, nc - 1) * OT::STRIDE + mat + (size_t)OT::full(rt, 0) * 2 * OT::FR + 8 * l;
#pragma unroll
      for (int pp = 0; pp < NP; ++pp) {
        x[pp][0] = *(const bf16x8*)(src + (2 * pp) * OT::FR);
        x[pp][1] = *(const bf16x8*)(src + (2 * pp + 1) * OT::FR);
      }
    };
    // The rows of the state pass: rows 16 rt + n of K (chunk ck) and Q (chunk
    // cq), 32-key operands.  Chunks are clamped to the last one, rows to the
    // last position (loaded, never used).
    constexpr int NX = KB / 2;
    bf16x8 kf[GDN ? NX : 1], qf[NX];
    auto x_ptr = [&](const void* base, int c) {
      return (const T*)base + ((tok0 + min(min(c, nc - 1) * C + 16 * rt + n, s.T - 1)) * s.H + h) * KD + 8 * g;
    };
    auto load_k = [&](int c) {
      const T* kr = x_ptr(in.k, c);
#pragma unroll
      for (int k = 0; k < NX; ++k)
        if constexpr (GDN) kf[k] = *(const bf16x8*)(kr + 32 * k);
    };
    auto load_q = [&](int c) {
      const T* qr = x_ptr(in.q, c);
#pragma unroll
      for (int k = 0; k < NX; ++k) qf[k] = *(const bf16x8*)(qr + 32 * k);
    };
    // block k (32 keys) of half unit u (16 columns: one slice, or with PK two)
    auto s_op = [&](int u, int k) {
      return sm.sop[u >> 1][2 * k + (g >> 1)][32 * (g & 1) + 16 * (u & 1) + n];
    };
    auto cslc = [&](int u) { return PK ? 2 * u + (g >> 1) : u; };  // slice of this lane's columns in half unit u
    // a 32-position operand (transposed) of a row-major (hi, lo) tile
    auto row_op = [&](const bf16_t(*x)[16], int pp) {
      const int q = (l >> 2) & 3, c4 = 4 * (l & 3);
      return join8(lds_read_tr16(&x[32 * pp + 4 * g + q][c4]), lds_read_tr16(&x[32 * pp + 16 + 4 * g + q][c4]));
    };
    // B (A hi + A lo)^T-style product without lo lo, one 32-deep step
    auto mma3 = [](f32x4& acc, const bf16x8(&a)[2], bf16x8 bh, bf16x8 bl) {
      acc = mma_16(bh, a[0], acc);
      acc = mma_16(bl, a[0], acc);
      acc = mma_16(bh, a[1], acc);
    };
    const int row = 16 * rt + n;  // this lane's row of a chunk
    // four values of the lane's row as a (hi, lo) row-major tile
    auto put_rows = [&](bf16_t(*dst)[C][16], f32x4 x) {
      bf16x4 hi, lo;
      split_frag(x, hi, lo);
      *(bf16x4*)&dst[0][row][4 * g] = hi;
      *(bf16x4*)&dst[1][row][4 * g] = lo;
    };
    auto v_row = [&](int c) {
      const f32x4 x = bf16x4_to_f(*(const bf16x4*)&sm.V[c & 1][row][4 * g]);
      return c * C + row < s.T ? x : zero4();
    };
    auto put_x = [&](int c, f32x4 x) { put_rows(sm.Xo, c * C + row < s.T ? x : zero4()); };
    auto put_u = [&](f32x4 u) {
      *(f32x4*)&sm.Uf[row][4 * g] = u;
      put_rows(sm.Uo, u);
    };
    // U of chunk c: Tu X (GDN) or diag(beta) V (sGLA)
    auto form_u = [&](int c) {
      f32x4 u = zero4();
      if constexpr (GDN) {
#pragma unroll
        for (int pp = 0; pp < NP; ++pp)
          if (pp <= pw) mma3(u, to[pp], row_op(sm.Xo[0], pp), row_op(sm.Xo[1], pp));
      } else {
        u = v_row(c) * sm.beta[c & 1][row];
      }
      return u;
    };
    // Sums over slices run over the even and over the odd slices and add the
    // two: with PK they lie in the two lane halves of a half unit, else in NS = 2
    // sums.  One order for both widths, so that the width, which goes by the
    // heads of the whole call, does not reach the results: a sequence gives the
    // same bits alone and among others.
    constexpr int NS = PK ? 1 : 2;
    struct Sum { f32x4 p[NS]; };
    auto zero_sum = [] {
      Sum x;
#pragma unroll
      for (int i = 0; i < NS; ++i) x.p[i] = zero4();
      return x;
    };
    auto total = [](const Sum& x) {
      if constexpr (PK) {
        f32x4 r;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t b = __float_as_uint(x.p[0][j]);
          const auto y = __builtin_amdgcn_permlane32_swap(b, b, false, false);
          r[j] = __uint_as_float(y[0]) + __uint_as_float(y[1]);
        }
        return r;
      } else {
        return x.p[0] + x.p[1];
      }
    };

    // The row waves' steps: KS forms X and U of the row tile, QS its outputs.
    auto run = [&](auto ks_c, auto qs_c) {
      constexpr bool KS = decltype(ks_c)::value, QS = decltype(qs_c)::value;
      if constexpr (KS && GDN) load_k(0);
      if constexpr (QS) load_q(0);
      if constexpr (KS && GDN) load_tri(to, OT::Tu, 0);
      if constexpr (QS) load_tri(mo, OT::M, 0);
      // One step.  GDN: the last chunk's (LAST), which forms nothing of a next
      // chunk, is a copy of its own.  Done like the others it cost calls of many
      // short sequences a third product and the wait for rows never used (whole
      // forwards, B64 H16 T64 K128, before the look-ahead / with that / now: E8
      // 256 / 290 / 260 us, E4 183 / 216 / 183, E16 549 / 593 / 535); skipped by a
      // branch inside the loop's step, the loads in flight have to arrive at every
      // join (10-30% slower at all lengths).
      auto step = [&](auto last_c, int c) {
        constexpr bool LAST = decltype(last_c)::value;
        block_sync();  // B0: the copy of S_c (and, unless direct, U_c) is there
        if (direct(c)) {
          if constexpr (KS && GDN) {  // X_c = V_c - sum_e diag(a_e) K_c S_c
            Sum ws = zero_sum();
#pragma unroll
            for (int u = 0; u < 2 * UE; ++u) {
              f32x4 P = zero4();
#pragma unroll
              for (int k = 0; k < NX; ++k) P = mma_16(s_op(u, k), kf[k], P);
              ws.p[u % NS] += sm.ca[c & 1][cslc(u)][row] * P;
            }
            put_x(c, v_row(c) - total(ws));
            if constexpr (!LAST) {
              load_k(c + 1);  // (Q_c is there)
              load_full(go, OT::G, c + 1);
            }
          }
          block_sync();
          if constexpr (KS) {
            put_u(form_u(c));
            if constexpr (GDN && !LAST) load_tri(to, OT::Tu, c + 1);
          }
          block_sync();
        }
        const bool more = GDN ? !LAST : c + 1 < nc;
        const bool ahead = more && !direct(c + 1);  // X_{c+1}, U_{c+1} are formed in this step
        constexpr bool DK = KS && GDN && !LAST;
        f32x4 o = zero4(), x = zero4();
        if constexpr (DK || QS) {
#pragma unroll
          for (int pp = 0; pp < NP; ++pp) {
            const bf16x8 uh = row_op(sm.Uo[0], pp), ul = row_op(sm.Uo[1], pp);
            if constexpr (DK) mma3(x, go[pp], uh, ul);
            if (QS && pp <= pw) mma3(o, mo[pp], uh, ul);
          }
          if constexpr (QS && !LAST) load_tri(mo, OT::M, c + 1);
          if constexpr (DK) load_full(go, OT::G, c + 2);
          // K_{c+1} S_c and Q_c S_c, all half units, one pass over the copy of S_c
          f32x4 Pk[DK ? 2 * UE : 1], Pq[QS ? 2 * UE : 1];
#pragma unroll
          for (int u = 0; u < 2 * UE; ++u) {
            if constexpr (QS) Pq[u] = zero4();
            if constexpr (DK) Pk[u] = zero4();
          }
          const T* kr = x_ptr(in.k, ahead ? c + 2 : c + 1);
          const T* qr = x_ptr(in.q, c + 1);
#pragma unroll
          for (int k = 0; k < NX; ++k) {
#pragma unroll
            for (int u = 0; u < 2 * UE; ++u) {
              const bf16x8 sb = s_op(u, k);
              if constexpr (QS) Pq[u] = mma_16(sb, qf[k], Pq[u]);
              if constexpr (DK) Pk[u] = mma_16(sb, kf[k], Pk[u]);
            }
            // done with this key block: the next step's rows
            if constexpr (QS && !LAST) qf[k] = *(const bf16x8*)(qr + 32 * k);
            if constexpr (DK) kf[k] = *(const bf16x8*)(kr + 32 * k);
          }
          Sum os = zero_sum(), ws = zero_sum();
#pragma unroll
          for (int u = 0; u < 2 * UE; ++u) {
            const int e = cslc(u);
            if constexpr (QS) os.p[u % NS] += sm.cbc[c & 1][0][e][row] * Pq[u];
            if constexpr (DK) ws.p[u % NS] += (sm.gC[c & 1][e] * sm.ca[(c + 1) & 1][e][row]) * Pk[u];
          }
          if constexpr (DK)
            if (ahead) put_x(c + 1, v_row(c + 1) - (total(ws) + x));
          if constexpr (QS) o += total(os);
        }
        if constexpr (!LAST) block_sync();  // B1: X_{c+1}; every row wave is done with U_c and the copy of S_c
        if constexpr (KS) {
          if (ahead || (!GDN && more)) {
            put_u(form_u(c + 1));
            if constexpr (GDN) load_tri(to, OT::Tu, c + 2);
          }
        }
        if constexpr (QS) {
          const int t = c * C + row;
          if (t < s.T && (!PK || g < 2)) {
            const size_t off = ((tok0 + t) * s.H + h) * (size_t)V + v0 + 4 * g;
            if (s.out_bf16)
              __builtin_nontemporal_store(__builtin_bit_cast(u32x2, cvt_frag<T>(o)), (u32x2*)((T*)out + off));
            else
              __builtin_nontemporal_store(__builtin_bit_cast(u32x4, o), (u32x4*)((float*)out + off));
          }
        }
      };
      for (int c = 0; c < nc - GDN; ++c) step(std::false_type{}, c);
      if constexpr (GDN) step(std::true_type{}, nc - 1);
    };
    if constexpr (NT == 4) {
      run(std::true_type{}, std::true_type{});
    } else {  // two waves a row tile, one side each
      if (w < NT)
        run(std::false_type{}, std::true_type{});
      else
        run(std::true_type{}, std::false_type{});
    }
  }
}

// ---------------------------------------------------------------- launchers
template <auto K>
static void lds_limit(size_t smem) {
  static bool set = false;
  if (!set) {
    (void)hipFuncSetAttribute((const void*)K, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    set = true;
  }
}

template <int KD, int C, int E>
static hipError_t prep_la(const Shape& s, const FwdIn& in, const PrepBufs& p, hipStream_t st) {
  static_assert(LaOps<KD, C>::STRIDE <= OpTiles<bf16_t, KD, C>::STRIDE, "the tiles fit the workspace");
  const size_t smem = sizeof(LaPrepSmem<KD, C, E>);
  lds_limit<k_prep_la<KD, C, E>>(smem);
  hipLaunchKernelGGL((k_prep_la<KD, C, E>), dim3(s.NH * s.Nc), dim3(la_prep_waves<E>() * 64), smem, st, s,
                     in, p);
  return hipGetLastError();
}

template <int KD, int C, int E, bool PK, bool GDN>
static hipError_t fwd_la2(const Shape& s, const FwdIn& in, const PrepBufs& p, void* o, float* s_final,
                          hipStream_t st) {
  const size_t smem = sizeof(LaFwdSmem<KD, C, E, PK>);
  static_assert(sizeof(LaFwdSmem<KD, C, E, PK>) <= 160 * 1024, "shared-memory plan");
  lds_limit<k_fwd_la<KD, C, E, PK, GDN>>(smem);
  hipLaunchKernelGGL((k_fwd_la<KD, C, E, PK, GDN>), dim3(s.NH * (s.V / (PK ? 8 : 16))), dim3(512),
                     smem, st, s, in, p, o, s_final);
  return hipGetLastError();
}

template <int KD, int C, int E>
static hipError_t fwd_la(const Shape& s, const FwdIn& in, const PrepBufs& p, void* o, float* s_final,
                         hipStream_t st) {
  auto go = [&](auto pk) {
    constexpr bool PK = decltype(pk)::value;
    return s.variant == 1 ? fwd_la2<KD, C, E, PK, true>(s, in, p, o, s_final, st)
                          : fwd_la2<KD, C, E, PK, false>(s, in, p, o, s_final, st);
  };
  if constexpr (E >= 16) {  // four slices a unit: the state of a wave fits its registers only so
    return go(std::true_type{});
  } else {
    // 8-column workgroups while 16-column ones would leave half of the 256 CUs
    // idle: 36 against 41 us for GDN at B1 H16 T777 E8 (256 or 128 workgroups);
    // whole forwards at E = 4: sGLA B1 H4 T65536 1.45 against 1.59 ms, GDN
    // there 2.28 against 2.32 ms, sGLA B2 H8 T2048 60 against 63 us
    if (s.NH * (s.V / 16) <= 128) return go(std::true_type{});
    return go(std::false_type{});
  }
}

// The instances, in one list: fields of s, CALL(K, C, E).
#define TLA_LA_FOR_EACH(CALL)                                \
  if (s.K == 64 && s.C == 32 && s.E == 8) return CALL(64, 32, 8);    \
  if (s.K == 64 && s.C == 64 && s.E == 16) return CALL(64, 64, 16);  \
  if (s.K == 128 && s.C == 64 && s.E == 4) return CALL(128, 64, 4);  \
  if (s.K == 128 && s.C == 64 && s.E == 8) return CALL(128, 64, 8);  \
  if (s.K == 128 && s.C == 64 && s.E == 16) return CALL(128, 64, 16); \
  if (s.K == 128 && s.C == 32 && s.E == 8) return CALL(128, 32, 8);

bool la_instance(const Shape& s) {
  if (!s.in_bf16) return false;
#define CALL_I(KD_, C_, E_) true
  TLA_LA_FOR_EACH(CALL_I)
#undef CALL_I
  return false;
}

hipError_t launch_prep_la(const Shape& s, const FwdIn& in, const PrepBufs& p, hipStream_t st) {
#define CALL_P(KD_, C_, E_) prep_la<KD_, C_, E_>(s, in, p, st)
  TLA_LA_FOR_EACH(CALL_P)
#undef CALL_P
  return hipErrorInvalidValue;
}

hipError_t launch_fwd_la(const Shape& s, const FwdIn& in, const PrepBufs& p, void* o, float* s_final,
                         hipStream_t st) {
#define CALL_F(KD_, C_, E_) fwd_la<KD_, C_, E_>(s, in, p, o, s_final, st)
  TLA_LA_FOR_EACH(CALL_F)
#undef CALL_F
  return hipErrorInvalidValue;
}

}  // namespace tla
