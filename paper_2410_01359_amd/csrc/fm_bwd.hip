// Backward pass (Algorithm 2) for gfx950, as two kernels:
//
//   dq_kernel     row-parallel loop over query blocks i, run first: its prologue is Algorithm 2's D
//                 pre-pass, D_i = sum_c dO_ic O_ic (left in the workspace for the other loop); then
//                 S, P = exp(S - L), dP, dS per tile and dQ_i += dS K_j, accumulated in registers in a
//                 fixed order.
//   dkdv_kernel   column-parallel loop over key blocks j: recompute S and
//                 P = exp(S - L), dV_j += P^T dO_i, dP = dO_i V_j^T,
//                 dS = P o (dP - D_i), dK_j += dS^T Q_i           (Algorithm 2 main loop)
//
// Algorithm 2 adds every tile's dS K_j into dQ_i in HBM from the column-parallel
// loop.  On this chip fp32 atomic adds sustain about 1.4 TB/s, which would cap
// the backward far below the matrix-core rate, so dQ gets its own row-parallel
// pass instead (two extra products per tile, no atomics, bit-reproducible).
#include "fm_common.h"
#include "fm_interval.h"
#include "fm_kernels.h"

namespace fm {

// ---------------------------------------------------------------------------
// dQ: row-parallel, same transposed-score layout as the forward kernel.
// ---------------------------------------------------------------------------
// S: groups of waves that share a unit's key tiles, each tile of the list belongs to one group (2: direct units only).
// WR: waves of a group, 32 rows each.  DIRECT: direct units, whose tiles have 64 keys at either d (short lists).
template <int D, int S = 1, int WR = 4, bool DIRECT = false>
struct DqCfg {
  static constexpr int KT = DIRECT ? 64 : fm_dq_bc(D);
  static constexpr int BR = 32 * WR;
  static constexpr int THREADS = 64 * S * WR;
  using L = TileLayout<D>;
  static constexpr int K_BYTES = KT * L::RS;
  static constexpr int V_BYTES = KT * L::RS;
  static constexpr int BND_BYTES = 4 * KT * 4;
  static constexpr int STAGE = K_BYTES + V_BYTES + BND_BYTES;
  static constexpr int LIST_CAP = 1024;
  static constexpr int CNT_OFF = LIST_CAP * 4;
  static constexpr int STAGE_OFF = CNT_OFF + 256;   // stages start at multiples of 256 bytes (see the operand reads)
  static constexpr int LDS_BYTES = STAGE_OFF + 2 * S * STAGE;   // two stages of S tiles each
  static_assert(STAGE % 256 == 0 && STAGE_OFF % 256 == 0 && K_BYTES % 256 == 0, "XOR after add");
};

// RAGGED: see the forward kernel -- loops at the padded length, clamped tile copies, guarded stores.
template <int D, bool RAGGED, bool GEN, int S, int WR, bool DIRECT>
__device__ __forceinline__ void dq_body(const FmBwdKernelArgs<GEN>& a) {
  using C = DqCfg<D, S, WR, DIRECT>;
  constexpr int NTC = WR == 4 ? 1 : S;    // tiles per step that a wave takes part in copying (see the forward)
  constexpr int KT = C::KT, NKB = KT / 32, NDB = D / 16, NKK = D / 32;
  extern __shared__ __attribute__((aligned(256))) char smem[];   // the operand reads rely on the alignment

  const int t_r = ((RAGGED ? a.N : a.Np) + C::BR - 1) / C::BR;
  i32x4 rec = {-1, 0, 0, 0};
  int bh, i_blk;   // batch row and head, row block
  if (!DIRECT) {
    rec = queue_take(a.queue_dq, (int*)(smem + C::CNT_OFF) + 8);
    if (rec[0] < 0) return;
    bh = rec[0] / t_r;
    i_blk = rec[0] - bh * t_r;
  } else {
    args_at_once(a.order, a.q, a.lts, a.lte, a.uts, a.ute, a.N, a.Np, a.H);
    const FmDirectUnit u = fm_direct_unit<GEN>(a.order, (int)blockIdx.x);
    if (u.block < 0) return;
    bh = GEN ? u.slice * (int)a.order.group.n + u.member : u.slice;
    i_blk = t_r - 1 - u.block;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int quad = lane >> 4, c = lane & 15;   // see mfma16
  const int N = a.Np, H = a.H;            // padded length: what the loops and tables see
  const int Nr = RAGGED ? a.N : a.Np;     // rows the tensors really have
  const int t_c = N / KT;
  const int j_lo = DIRECT ? 0 : rec[1], j_hi = DIRECT ? t_c : rec[2];
  const int b = bh / H;
  const int q0 = i_blk * C::BR;
  const int wrow = S == 1 ? wave : wave % WR, grp = S == 1 ? 0 : wave / WR;
  const int cwave = S * WR == 4 ? wave : wave % 4, sub0 = WR == 4 ? grp : 0;
  const int qw0 = q0 + wrow * 32;
  const int row[2] = {qw0 + c, qw0 + 16 + c};  // this lane's query rows

  const int h = bh - b * H, hk = GEN ? h / (H / a.Hk) : h, Hk = GEN ? a.Hk : H;
  const __bf16* qp = slice_ptr<D, GEN>(a.q, a.sq, b, h, H, Nr);
  const __bf16* kp = slice_ptr<D, GEN>(a.k, a.sk, b, hk, Hk, Nr);
  const __bf16* vp = slice_ptr<D, GEN>(a.v, a.sv, b, hk, Hk, Nr);
  const __bf16* dop = slice_ptr<D, GEN>(a.dout, a.sdo, b, h, H, Nr);
  const int q_rs = row_stride<D, GEN>(a.sq), k_rs = row_stride<D, GEN>(a.sk), v_rs = row_stride<D, GEN>(a.sv);
  const int do_rs = row_stride<D, GEN>(a.sdo);
  const int* table = a.minmax_dq + (size_t)b * 8 * t_c;
  // The four bound slices of a partially masked tile (KT ints each, one after the other in LDS) are copied by the
  // first BND_WAVES waves, 1 KB each: a lane moves 16 bytes of vector (64 * cwave + lane) / (KT / 4).
  constexpr int BND_LPV = KT / 4, BND_WAVES = 4 * BND_LPV / 64;
  const int* my_bvec;
  {
    const int which = (64 * cwave + lane) / BND_LPV;
    const int* p = a.lts;
    if (which == 1) p = a.lte;
    if (which == 2) p = a.uts;
    if (which == 3) p = a.ute;
    my_bvec = p + (size_t)b * Nr + (lane % BND_LPV) * 4;
  }
  // RAGGED: rows of the bound vectors are 4-byte aligned only and the last key block reaches past their end:
  // wave w copies one vector's slice, 4 bytes per lane
  const int* wave_bvec = (cwave == 0 ? a.lts : cwave == 1 ? a.lte : cwave == 2 ? a.uts : a.ute) + (size_t)b * Nr;
  CopyLanes<D> copy_lanes, copy_lanes_v_;
  copy_lanes.init(lane, 2 * k_rs);
  if (GEN) copy_lanes_v_.init(lane, 2 * v_rs);
  const CopyLanes<D>& copy_lanes_v = GEN ? copy_lanes_v_ : copy_lanes;
  const char* const kp_wave = CopyLanes<D>::wave_base(kp, cwave, 2 * k_rs);
  const char* const vp_wave = CopyLanes<D>::wave_base(vp, cwave, 2 * v_rs);

  int* list = (int*)smem;
  const int* bnd_rows[4] = {a.lts + (size_t)b * Nr, a.lte + (size_t)b * Nr, a.uts + (size_t)b * Nr, a.ute + (size_t)b * Nr};
  // Where one pass covers all key blocks, their bounds are requested ahead of the rows and classified while those are in
  // flight.  With more passes it would be one more round trip: two are requested together then.
  DirectPass<RAGGED, T_FULLY, WR, S * WR> first;
  static_assert(first.BLOCKS <= C::LIST_CAP, "a pass fits the list");
  const bool one_pass = DIRECT && t_c <= first.BLOCKS;
  if (one_pass) {
    first.load(bnd_rows, Nr, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  // Q and dO fragments (B operands): lane holds elements 32 kk + 8 quad ..+7 of its rows.
  bf16x8 qreg[2][NKK], doreg[2][NKK];
  size_t row_ld[2];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    row_ld[qb] = RAGGED ? min(row[qb], Nr - 1) : row[qb];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      qreg[qb][kk] = *(const bf16x8*)(qp + row_ld[qb] * q_rs + kk * 32 + 8 * quad);
      doreg[qb][kk] = *(const bf16x8*)(dop + row_ld[qb] * do_rs + kk * 32 + 8 * quad);
    }
  }
  // Algorithm 2's D pre-pass, folded into this loop's prologue (the dO fragments are at hand; the O
  // fragments are loaded in the same layout): D_i = sum_c dO_ic O_ic of this lane's rows, a partial sum
  // per lane and the sum over the four lanes that hold a row.  -D and the log2-domain
  // lse (+inf for a row with no visible key and for padding rows, so that P = 0 there) also go to the
  // workspace, where the dK/dV loop, which runs after this one, picks them up per tile.
  float lse2[2], dneg[2] = {0.f, 0.f};
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) lse2[qb] = !RAGGED || row[qb] < Nr ? a.lse[(size_t)bh * Nr + row[qb]] : -INFINITY;
  {
    const __bf16* outp = slice_ptr<D, GEN>(a.out, a.so, b, h, H, Nr);
    const int o_rs = row_stride<D, GEN>(a.so);
    bf16x8 oreg[2][NKK];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) oreg[qb][kk] = *(const bf16x8*)(outp + row_ld[qb] * o_rs + kk * 32 + 8 * quad);
    if (one_pass) {
      __builtin_amdgcn_sched_barrier(0);   // behind the requests for the rows
      first.classify(Nr, 0, 0, t_c, q0, min(q0 + C::BR, Nr), list);
    }
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e) dneg[qb] -= (float)oreg[qb][kk][e] * (float)doreg[qb][kk][e];
      dneg[qb] = quad_sum(dneg[qb]);
      if (RAGGED && row[qb] >= Nr) dneg[qb] = 0.f;
      lse2[qb] = (lse2[qb] == -INFINITY) ? INFINITY : lse2[qb] * kLog2e;
    }
  }
  if (quad < 2 && grp == 0) {
    a.dvec[(size_t)bh * N + qw0 + lane] = quad ? dneg[1] : dneg[0];
    a.lse2[(size_t)bh * N + qw0 + lane] = quad ? lse2[1] : lse2[0];
  }
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      settle(qreg[qb][kk]);
      settle(doreg[qb][kk]);
    }
    settle(lse2[qb]);
    settle(dneg[qb]);
  }

  f32x4 dqacc[NDB][2];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
      for (int r = 0; r < 4; ++r) dqacc[db][qb][r] = 0.f;

  int* wave_cnt = (int*)(smem + C::CNT_OFF);
  const float sc = a.scale * kLog2e;
  // lane-dependent LDS offsets inside a tile: operand rows (16 rows, a whole panel) and transpose reads (4 rows and 32
  // bytes of the panel to every 16 lanes)
  const int a_base = C::L::off(c, 16 * quad);
  const int t_base = C::L::off(4 * quad + (c >> 2), 8 * (c & 3));

#define FM_LOAD_TILE(ENTRY, BUF, SUB)                                                          \
  {                                                                                            \
    const int j_ = entry_block(ENTRY, chunk);                                                  \
    char* st_ = smem + C::STAGE_OFF + ((BUF) * S + (SUB)) * C::STAGE;                          \
    _Pragma("unroll") for (int sub = 0; sub < KT / 64; ++sub) {   /* 64 keys per copy call */  \
      const int r_ = j_ * KT + sub * 64;                                                       \
      char* ks_ = st_ + sub * 64 * C::L::RS;                                                   \
      if (RAGGED && r_ + 64 > Nr) {                                                            \
        tile_load_async_clamped<D>(kp, r_, Nr, ks_, cwave, lane, 2 * k_rs);                     \
        tile_load_async_clamped<D>(vp, r_, Nr, ks_ + C::K_BYTES, cwave, lane, 2 * v_rs);        \
      } else {                                                                                 \
        tile_load_async<D>(kp_wave + (size_t)(2 * r_) * k_rs, copy_lanes, ks_, cwave);          \
        tile_load_async<D>(vp_wave + (size_t)(2 * r_) * v_rs, copy_lanes_v, ks_ + C::K_BYTES, cwave); \
      }                                                                                        \
    }                                                                                          \
    if (entry_tile_class(ENTRY) == T_PARTIAL) {                                                \
      const unsigned bnd_ = lds_address(st_ + C::K_BYTES + C::V_BYTES);                        \
      if (RAGGED) {                                                                            \
        _Pragma("unroll") for (int sub = 0; sub < KT / 64; ++sub)                              \
          async_copy4(bound_or_pad(wave_bvec, cwave, j_ * KT + sub * 64 + lane, Nr), bnd_ + cwave * (KT * 4) + sub * 256); \
      } else if (cwave < BND_WAVES) {                                                           \
        async_copy16(my_bvec + j_ * KT, bnd_ + cwave * 1024);                                   \
      }                                                                                        \
    }                                                                                          \
  }

  // only the key blocks [j_lo, j_hi) can be live for this row block (found by the work pre-pass)
  for (int chunk = j_lo; chunk < j_hi; chunk += C::LIST_CAP) {
    const int chunk_end = min(chunk + C::LIST_CAP, j_hi), r1 = min(q0 + C::BR, Nr);
    int n_live;
    if constexpr (!DIRECT) {
      n_live = build_live_key_blocks<T_FULLY>(table, t_c, chunk, chunk_end, q0, r1, C::BR / 4, list, wave_cnt);
    } else {
      n_live = build_live_key_blocks_direct<RAGGED, T_FULLY, WR, S * WR>(one_pass, bnd_rows, Nr, chunk, chunk_end, q0, r1, list, wave_cnt);
    }
    if (n_live == 0) continue;
    // the entries of tiles t and t + 1 travel in scalar registers; the one that joins them at the next tile is
    // read from the list at the top of a tile and picked up behind the tile's barrier, so that no tile starts by
    // waiting for LDS
    int entry_s[NTC], next_entry_s[NTC];   // one per group of waves
#pragma unroll
    for (int s_ = 0; s_ < NTC; ++s_) {
      entry_s[s_] = __builtin_amdgcn_readfirstlane(list[min(sub0 + s_, n_live - 1)]);
      next_entry_s[s_] = __builtin_amdgcn_readfirstlane(list[min(S + sub0 + s_, n_live - 1)]);
      if (S == 1 || sub0 + s_ < n_live) FM_LOAD_TILE(entry_s[s_], 0, sub0 + s_);
    }
    async_wait<0>();
    barrier_nofence();

    const int n_steps = (n_live + S - 1) / S;
    for (int t = 0; t < n_steps; ++t) {
      int v_after[NTC];
#pragma unroll
      for (int s_ = 0; s_ < NTC; ++s_) v_after[s_] = list[min(S * (t + 2) + sub0 + s_, n_live - 1)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s_ = 0; s_ < NTC; ++s_)
        if (S * (t + 1) + sub0 + s_ < n_live) FM_LOAD_TILE(next_entry_s[s_], (t + 1) & 1, sub0 + s_);

      const char* st = smem + C::STAGE_OFF + ((t & 1) * S + grp) * C::STAGE;
      const int* bnd = (const int*)(st + C::K_BYTES + C::V_BYTES);

      const int entry = NTC == 1 || grp == 0 ? entry_s[0] : entry_s[NTC - 1];
      // Equation 4 on this wave's own rows; a group without a tile in the last step has nothing to do
      const int wcls = S == 1 || S * t + grp < n_live ? entry_wave_class(entry, wrow) : T_FULLY;
      if (wcls != T_FULLY) {
        const unsigned a_s = lds_address(st) + (unsigned)a_base, t_s = lds_address(st) + (unsigned)t_base;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
          // S^T = K Q^T, then dP^T = V dO^T, for 32 keys x 32 queries: NS steps of one operand from LDS (16 keys) and two
          // MFMAs (16 queries each); the operand of a step is fetched RS steps ahead into a small register ring.  The S
          // chain goes first, so that the exponentials P = exp(S - L) can ride along with the dP chain.  Of either, the
          // first 16 keys are complete halfway.
          f32x4 sacc[2][2], dpacc[2][2];   // [16 keys][16 queries]: keys 4 quad + r, query c
          constexpr int NH = 2 * NKK, NS = 2 * NH, RS = 3, NT = NDB, RT = 3;
          constexpr int EXPS = (16 + NH - 2) / (NH - 1);   // exponentials next to each of the last NH - 1 dP steps
          auto s_operand = [&](int n) __attribute__((always_inline)) {
            return lds_read_row16(a_s + (n >= NH ? C::K_BYTES : 0) + (kb * 32 + 16 * (n % NH / NKK)) * C::L::RS + n % NKK * 1024);
          };
          auto t_operand = [&](int n) __attribute__((always_inline)) {
            const unsigned at = C::L::add_col(t_s, n * 32) + kb * 32 * C::L::RS;
            return cat4(lds_read_tr16_at(at), lds_read_tr16_at(at + 16 * C::L::RS));
          };
          auto s_step = [&](int n, bf16x8 x) __attribute__((always_inline)) {
            const int ks = n % NH / NKK, kk = n % NKK;
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
              if (n < NH) sacc[ks][qb] = mfma16(x, qreg[qb][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sacc[ks][qb]);
              // the dP accumulator starts from -D of the row, so it ends as dP - D
              else dpacc[ks][qb] = mfma16(x, doreg[qb][kk], kk == 0 ? f32x4{dneg[qb], dneg[qb], dneg[qb], dneg[qb]} : dpacc[ks][qb]);
            }
          };
          bf16x8 ring[RS];
#pragma unroll
          for (int n = 0; n < RS; ++n) {
            ring[n] = s_operand(n);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int n = 0; n <= NH; ++n) {   // the S chain and the first dP step
            s_step(n, ring[n % RS]);
            if (n + RS < NS) ring[n % RS] = s_operand(n + RS);
            __builtin_amdgcn_sched_barrier(0);
          }
          if (wcls & T_PARTIAL) {
            // which pairs the workgroup's tile needs (1 = LT, 2 = UT, 3 = both): a pair that is not needed masks
            // no element of the tile, and most partially masked tiles need only one
            const int need = entry_need_pairs(entry);
            // Where one comparison per pair decides (5, 6, 7, see entry_mask_mode): half the bounds and compares.  Training
            // step: documents, d = 128 N = 4099 343 -> 329 us, N = 1000 79.6 -> 78.6; d = 64 N = 4099 215.7 -> 205.4, N = 1000
            // 55.4 -> 54.0, N = 8192 614 -> 607.  dQ loop in the queued units over full blocks at d = 128 (which had no register left
            // for it before the 16x16x32 products): shared questions 2048 83.3 -> 80.1 us, documents 8192 330 -> 323, 16384 918 -> 911.
            const int mode = entry_mask_mode(entry);
            auto bounds = [&](int which, int ks) __attribute__((always_inline)) {   // of this lane's keys
              return *(const i32x4*)(bnd + which * KT + kb * 32 + 16 * ks + 4 * quad);
            };
            auto hide = [&](int ks, auto hit) __attribute__((always_inline)) {   // hit(row, key): whether the element is masked
#pragma unroll
              for (int qb = 0; qb < 2; ++qb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                  if (hit(row[qb], r)) sacc[ks][qb][r] = -INFINITY;
            };
            if (mode & 4) {
              if (mode == 7) {
                const i32x4 bl[2] = {bounds(0, 0), bounds(0, 1)}, bv[2] = {bounds(3, 0), bounds(3, 1)};
                __builtin_amdgcn_sched_barrier(0);   // all in flight together
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) hide(ks, [&](int i, int r) { return (i >= bl[ks][r]) | (i < bv[ks][r]); });
              } else if (mode == 5) {
                const i32x4 bl[2] = {bounds(0, 0), bounds(0, 1)};
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                  for (int qb = 0; qb < 2; ++qb) hide4(sacc[ks][qb], 0, [&](int r) { return row[qb] >= bl[ks][r]; });
              } else {
                const i32x4 bv[2] = {bounds(3, 0), bounds(3, 1)};
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                  for (int qb = 0; qb < 2; ++qb) hide4(sacc[ks][qb], 0, [&](int r) { return row[qb] < bv[ks][r]; });
              }
            } else if (need == 3) {
#pragma unroll
              for (int ks = 0; ks < 2; ++ks) {
                const i32x4 bl = bounds(0, ks), be = bounds(1, ks), bu = bounds(2, ks), bv = bounds(3, ks);
                hide(ks, [&](int i, int r) { return ((i >= bl[r]) & (i < be[r])) | ((i >= bu[r]) & (i < bv[r])); });
              }
            } else {
              const int lo = need == 2 ? 2 : 0;   // the one pair that is needed
              const i32x4 bs[2] = {bounds(lo, 0), bounds(lo, 1)}, be[2] = {bounds(lo + 1, 0), bounds(lo + 1, 1)};
#pragma unroll
              for (int ks = 0; ks < 2; ++ks) hide(ks, [&](int i, int r) { return (i >= bs[ks][r]) & (i < be[ks][r]); });
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          auto ds_elem = [&](int e) __attribute__((always_inline)) { sacc[e / 8][e / 4 % 2][e % 4] *= dpacc[e / 8][e / 4 % 2][e % 4]; };
          bf16x8 dsb[2];
#pragma unroll
          for (int n = NH + 1; n < NS; ++n) {   // the rest of the dP chain, P = exp(S - L) beside it
            s_step(n, ring[n % RS]);
            if (n + RS < NS) ring[n % RS] = s_operand(n + RS);
#pragma unroll
            for (int e = (n - NH - 1) * EXPS; e < (n - NH) * EXPS && e < 16; ++e)
              sacc[e / 8][e / 4 % 2][e % 4] = fast_exp2(__builtin_fmaf(sacc[e / 8][e / 4 % 2][e % 4], sc, -lse2[e / 4 % 2]));
            // dS = P o (dP - D) of the first 16 keys beside the last steps
            constexpr int DS_FROM = NS - 3;
            if (NKK > 2 && n >= DS_FROM) {
#pragma unroll
              for (int e = (n - DS_FROM) * 3; e < (n - DS_FROM + 1) * 3 && e < 8; ++e) ds_elem(e);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          // K^T operands of the dQ product do not depend on dS: fetch the first ones now
          bf16x8 tring[RT];
#pragma unroll
          for (int n = 0; n < RT; ++n) tring[n] = t_operand(n);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = NKK > 2 ? 8 : 0; e < 16; ++e) ds_elem(e);
#pragma unroll
          for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int e = 0; e < 8; ++e) dsb[qb][e] = (__bf16)sacc[e / 4][qb][e % 4];
          __builtin_amdgcn_sched_barrier(0);
          // dQ^T += K^T dS^T, a step is 16 columns of d: element t of a lane's operands is key 4 quad + t of the first
          // (t < 4) or second 16 keys
#pragma unroll
          for (int n = 0; n < NT; ++n) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) dqacc[n][qb] = mfma16(tring[n % RT], dsb[qb], dqacc[n][qb]);
            if (n + RT < NT) tring[n % RT] = t_operand(n + RT);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }

      async_wait<0>();   // the next tile has landed ...
      barrier_nofence(); // ... for every wave, and every wave is done reading this one
#pragma unroll
      for (int s_ = 0; s_ < NTC; ++s_) {
        entry_s[s_] = next_entry_s[s_];
        next_entry_s[s_] = __builtin_amdgcn_readfirstlane(v_after[s_]);
      }
    }
    __syncthreads();     // the list is rebuilt by the next pass
  }
#undef FM_LOAD_TILE

  __bf16* dqp = (__bf16*)slice_ptr<D, GEN>(a.dq, a.sdq, b, h, H, Nr);
  const int dq_rs = row_stride<D, GEN>(a.sdq);
  // every wave is past its last tile and nothing is in flight into the stages (the barrier that ends a
  // pass over the list): their first bytes serve as the waves' store staging
  using RSt = RowStage<D>;
  static_assert(4 * RSt::BYTES <= 2 * S * C::STAGE, "store staging fits the stages");
  if (S == 2) {
    // the second group hands its sums to the first through LDS
    static_assert(S == 1 || 4 * RSt::BYTES + WR * 64 * 8 * NDB * 4 <= 2 * S * C::STAGE, "exchange fits the stages");
    float* const part = (float*)(smem + C::STAGE_OFF + 4 * RSt::BYTES) + wrow * (64 * 8 * NDB) + lane * 4;
    if (grp == 1) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) *(f32x4*)(part + (db * 2 + qb) * 256) = dqacc[db][qb];
    }
    barrier_nofence();
    if (grp == 1) return;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        const f32x4 o = *(const f32x4*)(part + (db * 2 + qb) * 256);
#pragma unroll
        for (int r = 0; r < 4; ++r) dqacc[db][qb][r] += o[r];
      }
  }
  char* stage = smem + C::STAGE_OFF + wave * RSt::BYTES;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      bf16x4 o4;
#pragma unroll
      for (int r = 0; r < 4; ++r) o4[r] = (__bf16)(dqacc[db][qb][r] * a.scale);
      RSt::put(stage, 16 * qb + c, 16 * db + 4 * quad, o4);
    }
  RSt::flush(stage, dqp + (size_t)qw0 * dq_rs, dq_rs, lane, RAGGED ? min(32, Nr - qw0) : 32);
}

// ---------------------------------------------------------------------------
// dK, dV: column-parallel.  A workgroup owns FM_DKDV_BC = 128 keys (32 per
// wave, K and V fragments resident in registers) and walks the row blocks of
// FM_DKDV_BR = 64 queries that are not fully masked for its keys.  Scores are
// NOT transposed here (S = Q K^T): every lane then holds one KEY column, so the
// four bounds of that key sit in four registers for the whole kernel and P^T,
// dS^T are already A operands of dV += P^T dO and dK += dS^T Q.
//
// One wave per SIMD at d = 128 (the accumulators alone take 128 registers; at d = 64 they take 64 and
// two workgroups share a CU), so the overlap of matrix and vector work is arranged inside the wave: a 64-row tile
// is two 32-row blocks, and the instruction stream is
//   S0,dP0 | S1,dP1 with the exp/dS arithmetic of block 0 between the MFMAs |
//   dV,dK of block 0 with the arithmetic of block 1 between the MFMAs | dV,dK of block 1
// with every LDS operand fetched a fixed number of steps ahead of its MFMA.
// Scheduling fences pin that order.
// ---------------------------------------------------------------------------
// S: groups of waves that share a unit's row tiles (1: units of 128 keys; 2: direct units of 64 keys, each tile of the
// list belongs to one pair of waves)
template <int D, int S = 1>
struct DkdvCfg {
  static constexpr int QT = FM_DKDV_BR;    // query rows per step
  static constexpr int BC = FM_DKDV_BC / S;   // keys per workgroup
  using L = TileLayout<D>;
  static constexpr int Q_BYTES = QT * L::RS;
  static constexpr int DO_BYTES = QT * L::RS;
  static constexpr int VEC_BYTES = 2 * QT * 4;  // lse (log2 domain, +inf for dead rows) and D of the rows
  static constexpr int STAGE = Q_BYTES + DO_BYTES + VEC_BYTES;
  static constexpr int LIST_CAP = 2048;
  // The last entry is repeated behind the list, so that the loops read on without a bound: a step reads up to AHEAD steps further.
  static constexpr int LIST_PAD = 64;
  static constexpr int CNT_OFF = (LIST_CAP + LIST_PAD) * 4;
  static constexpr int STAGE_OFF = CNT_OFF + 256;   // stages start at multiples of 256 bytes (dkdv_operand)
  // A copy's trip to L2 or HBM is longer than a tile's math, so it has two tiles' time.  Two workgroups per CU (d = 64): a
  // tile is copied three ahead, behind the workgroup step near a tile's end.  One (d = 128): two ahead, in the first steps
  // of a tile, which carry no vector work; the stage it goes into held the tile two back, which every wave had left when it
  // took the last workgroup step, so four stages need no barrier in front of the copies.  A unit then starts with two
  // tiles' copies instead of three and does not end with a wait for copies issued in its last steps: backward, d =
  // 128, three / two ahead: prefix 4096 of 32768 12325 / 12230 us, documents in 8192 730 / 718, causal 4096 478 / 473,
  // window 1024 at 32768 1034 / 1028, skewed documents at 131072 7693 / 7630; at d = 64, where the
  // other workgroup covers both, 0.5 % slower.  S = 2 has the four stages as two
  // pairs: a step's two tiles are copied while the step before them runs.
  static constexpr int NSTAGE = 4, AHEAD = S == 2 ? 1 : D == 128 ? 2 : 3;   // AHEAD in steps
  static constexpr int LDS_BYTES = STAGE_OFF + NSTAGE * STAGE;
  // async copy instructions one wave issues per tile: COPIES for its quarter of Q and dO plus
  // one for its quarter of the lse / D slice.  Every wave issues the same number for every
  // tile, so "tile landed" is a constant outstanding-copy count.
  static constexpr int COPIES = 2 * CopyLanes<D>::NINST;
  static constexpr int NC = COPIES + 1;
  // MFMA operand fetch distance in steps; divides the steps per tile, so ring slots line up across tiles
  static constexpr int RD = 8;
  // One workgroup per CU: nothing else hides the start of a unit, so workgroups go on from unit to unit and fetch the
  // next record early (d = 128, two rows of 8192 tokens in 11 documents: whole step 2 % faster than a workgroup per
  // unit).  With two on a CU the early draws of all workgroups only meet on the queue counters: a workgroup per unit
  // is faster from 1024 units of 3 to 8 tiles (65.9 -> 42.9 us) to 4096 units of 64 (557 -> 549 us).
  static constexpr bool PERSISTENT = D == 128;
  static constexpr int PER_CU = fm_dkdv_per_cu(D);   // workgroups of 128-key units on a compute unit
};

// lse / D slice of a tile in LDS: wave w copies rows 16w..16w+15 as 128 contiguous bytes,
// 64 bytes of lse then 64 bytes of D.  Float offset of row r (r % 4 == 0 for the 16-byte reads):
__device__ __forceinline__ constexpr int dkdv_vec_off(int r, bool d_part) {
  return (r >> 4) * 32 + (d_part ? 16 : 0) + (r & 15);
}

#define FM_FENCE() __builtin_amdgcn_sched_barrier(0)
// Steps between the last MFMA of a block's S / dP chains and the first vector instruction that reads their
// result: with none, that instruction waits out the MFMA's passes with the wave idle (one wave per SIMD).
#ifndef FM_DKDV_VSHIFT
#define FM_DKDV_VSHIFT 1
#endif

// exp / dS arithmetic of elements [e0, e0 + cnt) of one 32x32 block held in the
// MFMA output layout: register r is query row 8*(r/4) + 4*g + r%4 of the block.
// The exp / dS arithmetic of one score element, cut into three stages that the
// tile loop issues in three consecutive steps, so that a step never holds two
// dependent vector instructions of the same element (one wave per SIMD: nothing
// else hides the latency of v_exp_f32 and of the AGPR reads):
//   A: t = s*sc - lse2     B: p = exp2(t)     C: p = 0 where masked, dS = p * (dP - D)
// (dP - D comes straight out of the MFMA: its accumulator starts from the -D values of the rows)
// Register r of a block is query row 8*(r/4) + 4*g + r%4.
// The element mask of a lane's key is two row intervals: a 32-row block's are formed as a word with a bit per row
// (interval_rows) beside the first block's score MFMAs, which no other vector work rides along with, and an element's bit,
// spread over a word, is ANDed to its P.  Two instructions per element and 42 per tile, where comparing the row with both
// intervals and selecting took six: a partially masked tile had 530 instead of 619 instructions (417 instead of 506 at
// d = 64; 422 and 308 without mask; now 504 and 402, 398 and 297 without, branches counted).  Training step, both sides: eleven documents in 8192 tokens, 64 slices, d = 128 1050 ->
// 1030 us, five in 1000, 32 slices 86.7 -> 81.5; window 1024, N = 32768 1458 -> 1443.
__device__ __forceinline__ void dkdv_stage_a(const f32x16& s, const f32x16& dp, float (&t)[16], float (&u)[16],
                                             const f32x4 (&l4)[4], int e0, int cnt, float sc) {
#pragma unroll
  for (int r = e0; r < e0 + cnt; ++r) {
    t[r] = __builtin_fmaf(s[r], sc, -l4[r >> 2][r & 3]);
    u[r] = dp[r];   // dP - D: the dP accumulator was started from -D
  }
}

// What the tail of a tile's stream does for the tiles that follow it.
template <int S>
struct DkdvAhead {
  unsigned nqs;           // LDS address of the stage of the next list entry (its Q tile; dO follows), for the operand prefetch
  int v_copy[S];          // list entry (still in a vector register) of the tile AHEAD steps ahead, to be copied
                          // (S = 2: of the next step's two tiles)
  const char* q_base;     // global Q / dO of this (batch, head), already advanced to this wave's 16-row block
  const char* do_base;    // of a tile, and this lane's lse2 / D source
  const float* vec_src;
  int q_rs2, do_rs2;      // bytes between consecutive rows of Q / dO in global memory
  unsigned lds_copy;      // LDS address of the stage that receives the (first) copy
  int n_real, lane;       // ragged sequences: rows the tensors really have, and this thread's lane
  CopyLanes<128> lanes;   // per-lane source offsets of the copy instructions of Q (the first D/32 entries are used)
  CopyLanes<128> lanes_do;   // ... and of dO
  int wave;
};

// Copy number K (of NC) of the tile whose 64-row base offsets are given.  RAGGED: a tile that
// reaches past the last real row (i_copy is its index) clamps every lane's source row instead.
template <int D, int K, bool RAGGED, int S>
__device__ __forceinline__ void dkdv_issue_copy(const DkdvAhead<S>& ah, const char* q_src, const char* do_src,
                                                const float* vec_src, unsigned lds_stage, int i_copy) {
  using C = DkdvCfg<D>;
  constexpr int HALF = C::COPIES / 2;
  constexpr int WB = 16 * C::L::RS;   // bytes of a wave's 16-row block
  if (RAGGED && K < C::COPIES && (i_copy + 1) * C::QT > ah.n_real) {
    constexpr int I = K % HALF;
    const int grow = min(i_copy * C::QT + ah.wave * 16 + ah.lane / 4, ah.n_real - 1);
    const char* base = (K < HALF ? ah.q_base : ah.do_base) + CopyLanes<D>::BIAS;
    const long long rel = (long long)(grow - ah.wave * 16) * (K < HALF ? ah.q_rs2 : ah.do_rs2);   // the bases are this wave's
    const char* src = base + rel + CopyLanes<D>::source_col(ah.lane, I);
    async_copy16(src, lds_stage + (K < HALF ? 0 : C::Q_BYTES) + ah.wave * WB + I * 1024);
    return;
  }
  if (K < HALF) {
    if (K == 0 || RAGGED) async_window(lds_stage + ah.wave * WB);
    async_copy16_window<(K % HALF) * 1024>(q_src, ah.lanes.v[K % HALF]);
  } else if (K < C::COPIES) {
    if (K == HALF || RAGGED) async_window(lds_stage + C::Q_BYTES + ah.wave * WB);
    async_copy16_window<(K % HALF) * 1024>(do_src, ah.lanes_do.v[K % HALF]);
  } else {
    async_copy16_lanes8(vec_src, lds_stage + C::Q_BYTES + C::DO_BYTES + ah.wave * 128);
  }
}

// Order of the 2*NKK score MFMAs of one 32-row block (step y): the S chain leads by NKK/2
// steps, so the -D values the dP chain starts from have time to arrive from LDS:
//   y < H: S   |   H <= y < 3H: dP, S alternating   |   y >= 3H: dP          (H = NKK / 2)
template <int D>
__device__ __forceinline__ constexpr bool dkdv_is_s(int y) {
  constexpr int H = D / 32;
  return y < H || (y < 3 * H && ((y - H) & 1));
}
template <int D>
__device__ __forceinline__ constexpr int dkdv_kk(int y) {
  constexpr int H = D / 32;
  if (y < H) return y;
  if (y < 3 * H) return ((y - H) & 1) ? H + (y - H - 1) / 2 : (y - H) / 2;
  return H + (y - 3 * H);
}

// Per-lane LDS addresses of a list entry's stage: the stage's address plus the lane-dependent part of
// the three read patterns (row reads; transpose reads of rows 0-7 and 8-15 of a 16-row group).  Further columns,
// rows and the dO tile are immediate offsets, but for every second column group of the row reads, 32 bytes further
// on, which is an XOR (TileLayout::add_col): stage addresses are multiples of 256 bytes, so the sum keeps the lane
// part's low byte.
struct DkdvBases {
  unsigned a, t0, t1;
};
__device__ __forceinline__ DkdvBases dkdv_bases(unsigned s, int a_base, int t_base0, int t_base1) {
  return DkdvBases{s + (unsigned)a_base, s + (unsigned)t_base0, s + (unsigned)t_base1};
}
// LDS operand of step x of the list entry whose stage addresses are bs (Q tile, dO tile right behind it)
template <int D>
__device__ __forceinline__ bf16x8 dkdv_operand(const DkdvBases& bs, int x) {
  using L = TileLayout<D>;
  constexpr int NKK = D / 16, NDB = D / 32, NST = 2 * NKK;
  constexpr unsigned DO = DkdvCfg<D>::Q_BYTES;
  static_assert(DkdvCfg<D>::STAGE % 256 == 0 && DkdvCfg<D>::STAGE_OFF % 256 == 0 && DO % 256 == 0, "XOR after add");
  if (x < 2 * NST) {             // row reads: Q or dO rows of block x / NST as MFMA A operand
    const int qb = x / NST;
    const unsigned tile = dkdv_is_s<D>(x % NST) ? 0u : DO;
    return lds_read_row16(L::add_col(bs.a, dkdv_kk<D>(x % NST) * 32) + tile + qb * 32 * L::RS);
  }
  // transpose reads: dO (even step, dV) or Q (odd step, dK) as MFMA B operand
  const int u = x - 2 * NST, qb = u / NST, w = u % NST, h = w / (2 * NDB), db = (w % (2 * NDB)) / 2;
  const unsigned rows = ((u & 1) ? 0u : DO) + (qb * 32 + 16 * h) * L::RS;
  return cat4(lds_read_tr16_at(L::add_col(bs.t0, db * 64) + rows), lds_read_tr16_at(L::add_col(bs.t1, db * 64) + rows));
}

// The workgroup-level step that every wave takes once per list entry, in the middle of the
// entry's stream : wait for this wave's part of the
// NEXT entry's tile, meet the other waves (so the next tile is complete in LDS and nobody
// still reads the previous one), then the caller refills the previous tile's stage.
template <int D>
__device__ __forceinline__ void dkdv_sync() {
  async_wait<DkdvCfg<D>::NC>();   // copies complete in order: only the tile after the next may be in flight
  // The operand ring has reads of this entry's and the next entry's stages in flight here.  The stage
  // refilled after the barrier is the PREVIOUS entry's: its last read fed an MFMA a whole tile of
  // steps ago, in program order, so it has long returned.
  barrier_reads_in_flight();
}

// One 64-row tile = two 32-row blocks.  The tile's 8*NKK MFMAs form one stream
//   [S0 | dP0 | S1 | dP1 | dV,dK of block 0 | dV,dK of block 1]      (NKK = D/16 MFMAs per bar, 2*NKK for dV,dK)
// each taking one operand from LDS (a 128-bit row read for the first four
// groups, a transpose read for the rest) that is fetched RD steps ahead into a
// small register ring.  The exp / dS arithmetic of block 0 is spread over the
// steps of S1 and dP1, that of block 1 over the dV,dK steps of block 0, so the
// vector work always has matrix work in flight beside it.  The stream runs on
// into the next list entry: the copies of the tile AHEAD entries ahead go out one
// per step, near its end the wave takes the workgroup step (dkdv_sync), and its last RD operand fetches already read the next entry's tile, so
// the MFMA pipe does not drain between tiles.  On entry `op` holds the operands
// of steps 0..RD-1 of this tile, on exit those of the next one.
//
// S = 2 (two stages per group of waves instead of four): the stage that the next step's tiles are copied into is the
// previous step's, so the copies go out at the start of the stream, behind a barrier that every wave reaches with its
// previous tile used up, and a second barrier, in front of the first operand fetch from the next tile, publishes them.
template <int D, bool MASK, bool RAGGED, int S>
__device__ __forceinline__ void dkdv_tile(unsigned qs, const DkdvAhead<S>& ah,
                                          bf16x8 (&op)[DkdvCfg<D>::RD], const bf16x8 (&kreg)[D / 16],
                                          const bf16x8 (&vreg)[D / 16], f32x16 (&dkacc)[D / 32],
                                          f32x16 (&dvacc)[D / 32], int a_base, int t_base0, int t_base1, int r0,
                                          int g, float sc, int s_a, unsigned len_a, int s_b, unsigned len_b) {
  using C = DkdvCfg<D>;
  constexpr int NKK = D / 16, NDB = D / 32;
  constexpr int NST = 2 * NKK;     // MFMAs per block and product pair
  constexpr int EPS = 16 / NST;    // elements handled next to one MFMA (D = 128: 1, D = 64: 2)
  constexpr int NX = 4 * NST;      // MFMAs per tile
  constexpr int RD = C::RD;
  constexpr bool BEHIND = S == 1 && C::AHEAD == 3;       // the copies are issued behind the workgroup sync
  constexpr int XS = NX - (BEHIND && C::NC > RD ? C::NC : RD);   // step of the workgroup sync
  constexpr int XC = BEHIND ? XS : S == 2 ? 0 : RD;      // first of the steps that issue the copies, one each
  static_assert(NX % RD == 0 && XS > 0 && (BEHIND || XC + S * C::NC <= XS), "ring layout");
  const f32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  const unsigned vec_s = qs + C::Q_BYTES + C::DO_BYTES + 16 * g;   // lse and -D of row 4 g
  const DkdvBases bs_cur = dkdv_bases(qs, a_base, t_base0, t_base1);
  const DkdvBases bs_next = dkdv_bases(ah.nqs, a_base, t_base0, t_base1);

  f32x16 sb[2], pb[2];             // S then P, dP then dS, of the two blocks
  bf16x8 pa[2][2], dsa[2][2];      // bf16 P^T and dS^T, [block][16-row half]
  f32x4 l4[2][4];                  // lse (log2 domain) of the blocks' rows, fetched one group of 4 rows ahead
  float tq[2][16], uq[2][16];      // per element: exponent then P, and dP - D then dS
  unsigned seen[2], hidden = 0;    // rows of the blocks that this lane's key is seen by, a bit each (see interval_rows)
  int keep[2];                     // the bit of an element, spread over a word
  auto vec_group = [&](int qb, int grp) __attribute__((always_inline)) {
    l4[qb][grp] = *(FM_LDS const f32x4*)(size_t)(vec_s + 4 * dkdv_vec_off(qb * 32 + 8 * grp, false));
  };
  const char* q_src = nullptr;
  const char* do_src = nullptr;
  const float* vec_src = nullptr;
  unsigned lds_stage = 0;
  int i_copy = 0;

#pragma unroll
  for (int x = 0; x < NX; ++x) {
    // --- the MFMA of this step
    if (x < 2 * NST) {
      const int qb = x / NST, y = x % NST, kk = dkdv_kk<D>(y);   // two independent accumulation chains
      if (y == 0) {   // the dP accumulator starts from -D of the block's rows (register r: row 8*(r/4) + 4*g + r%4)
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
          const f32x4 dn = *(FM_LDS const f32x4*)(size_t)(vec_s + 4 * dkdv_vec_off(qb * 32 + 8 * grp, true));
#pragma unroll
          for (int i = 0; i < 4; ++i) pb[qb][4 * grp + i] = dn[i];
        }
      }
      if (dkdv_is_s<D>(y))
        sb[qb] = mfma32(op[x % RD], kreg[kk], kk == 0 ? zero : sb[qb]);
      else
        pb[qb] = mfma32(op[x % RD], vreg[kk], pb[qb]);
    } else {
      const int u = x - 2 * NST, qb = u / NST, w = u % NST, h = w / (2 * NDB), db = (w % (2 * NDB)) / 2;
      if (D == 64) {
        // d = 64: the accumulators are half as many and two workgroups share a CU (two waves per SIMD,
        // 256 registers each), so they stay ordinary compiler-managed registers
        if (u & 1)
          dkacc[db] = mfma32(op[x % RD], dsa[qb][h], dkacc[db]);
        else
          dvacc[db] = mfma32(op[x % RD], pa[qb][h], dvacc[db]);
      } else if (u & 1) {
        // dsa[qb][h] / pa[qb][h] were converted several steps ago (the vector work of a block ends before the
        // block's dV, dK steps begin), which is the distance that mfma32_acc asks for
        mfma32_acc(dkacc[db], op[x % RD], dsa[qb][h]);
      } else {
        mfma32_acc(dvacc[db], op[x % RD], pa[qb][h]);
      }
    }
    // --- the workgroup step(s) and the copies behind it
    if (S == 2 && x == 0) barrier_reads_in_flight();   // the operands in flight are this tile's
    if (x == XS) {
      if (S == 2) {
        async_wait<0>();
        barrier_reads_in_flight();
      } else {
        dkdv_sync<D>();
      }
    }
    if (x >= XC && x < XC + S * C::NC) {
      const int sub = (x - XC) / C::NC;
      if ((x - XC) % C::NC == 0) {
        i_copy = __builtin_amdgcn_readfirstlane(ah.v_copy[sub]) & 0xFFFFFF;
        q_src = ah.q_base + (size_t)i_copy * C::QT * ah.q_rs2;
        do_src = ah.do_base + (size_t)i_copy * C::QT * ah.do_rs2;
        vec_src = ah.vec_src + i_copy * C::QT;
        lds_stage = ah.lds_copy + sub * C::STAGE;
      }
      switch ((x - XC) % C::NC) {
        case 0: dkdv_issue_copy<D, 0, RAGGED>(ah, q_src, do_src, vec_src, lds_stage, i_copy); break;
        case 1: dkdv_issue_copy<D, 1, RAGGED>(ah, q_src, do_src, vec_src, lds_stage, i_copy); break;
        case 2: dkdv_issue_copy<D, 2, RAGGED>(ah, q_src, do_src, vec_src, lds_stage, i_copy); break;
        case 3: dkdv_issue_copy<D, 3, RAGGED>(ah, q_src, do_src, vec_src, lds_stage, i_copy); break;
        case 4: dkdv_issue_copy<D, 4, RAGGED>(ah, q_src, do_src, vec_src, lds_stage, i_copy); break;
        case 5: dkdv_issue_copy<D, 5, RAGGED>(ah, q_src, do_src, vec_src, lds_stage, i_copy); break;
        case 6: dkdv_issue_copy<D, 6, RAGGED>(ah, q_src, do_src, vec_src, lds_stage, i_copy); break;
        case 7: dkdv_issue_copy<D, 7, RAGGED>(ah, q_src, do_src, vec_src, lds_stage, i_copy); break;
        default: dkdv_issue_copy<D, 8, RAGGED>(ah, q_src, do_src, vec_src, lds_stage, i_copy); break;
      }
    }
    // --- fetch the operand of step x + RD (of the next tile once this one is used up)
    if (x + RD < NX)
      op[x % RD] = dkdv_operand<D>(bs_cur, x + RD);
    else
      op[x % RD] = dkdv_operand<D>(bs_next, x + RD - NX);
    // --- vector work riding along.  Vector step j handles EPS elements of
    //     block j / NST: stage A at x, stage B one step later, stage C two steps later
    //     (j = x - NST - FM_DKDV_VSHIFT - stage).
    if (x == NST - 1) vec_group(0, 0);
    if (MASK && x >= NST - 8 && x < NST && x % 2 == 0) {   // no other vector work here: one interval of one block at a time
      const int qb = (x - NST + 8) / 4, row = r0 + 32 * qb + 4 * g;
      if (x % 4 == 0) hidden = interval_rows(interval_offset(row, s_a), len_a);
      else seen[qb] = ~(hidden | interval_rows(interval_offset(row, s_b), len_b));
    }
#pragma unroll
    for (int stage = 2; stage >= 0; --stage) {
      const int j = x - NST - FM_DKDV_VSHIFT - stage;
      if (j >= 0 && j < 2 * NST) {
        const int qb = j / NST, e0 = (j % NST) * EPS;
        if (stage == 0) {
          if (e0 % 4 == 0 && e0 / 4 + 1 < 4) vec_group(qb, e0 / 4 + 1);
          if (qb == 0 && e0 + EPS == 16) vec_group(1, 0);
          dkdv_stage_a(sb[qb], pb[qb], tq[qb], uq[qb], l4[qb], e0, EPS, sc);
        } else if (stage == 1) {
#pragma unroll
          for (int r = e0; r < e0 + EPS; ++r) {
            tq[qb][r] = fast_exp2(tq[qb][r]);
            if (MASK) {
              keep[r % 2] = __builtin_amdgcn_sbfe((int)seen[qb], 8 * (r / 4) + r % 4, 1);
              asm("" : "+v"(keep[r % 2]));   // or the compiler turns it and the AND below into bit test, compare, select
            }
          }
        } else {
#pragma unroll
          for (int r = e0; r < e0 + EPS; ++r) {
            if (MASK) tq[qb][r] = __builtin_bit_cast(float, __builtin_bit_cast(int, tq[qb][r]) & keep[r % 2]);
            uq[qb][r] *= tq[qb][r];
          }
          if ((e0 + EPS) % 8 == 0) {   // a 16-row half of P^T and dS^T is complete: convert it to bf16 operands
            const int hh = (e0 + EPS) / 8 - 1;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              pa[qb][hh][e] = (__bf16)tq[qb][8 * hh + e];
              dsa[qb][hh][e] = (__bf16)uq[qb][8 * hh + e];
            }
            if (D == 128) {
              // here and not just in front of the MFMAs that read them, where ragged lengths' branches let the compiler
              // sink the conversions to: closer than mfma32_acc allows
              settle(pa[qb][hh]);
              settle(dsa[qb][hh]);
            }
          }
        }
      }
    }
    FM_FENCE();
  }
}

// RAGGED: see the forward kernel -- loops at the padded length, clamped tile copies and fragment
// loads, guarded stores; the padding rows carry lse = +inf (P = 0), and a lane past the last key works on a
// copy of that key and stores nothing.
// GEN: tensors with caller-given strides; a workgroup then owns 128 keys of one K/V head and
// walks the query heads that share it one after the other (same list of live row blocks: the
// mask does not depend on the head), accumulating dK and dV over all of them.
template <int D, bool RAGGED, bool GEN, int S, bool DIRECT>
__device__ __forceinline__ void dkdv_body(const FmBwdKernelArgs<GEN>& a) {
  using C = DkdvCfg<D, S>;
  constexpr int QT = C::QT, NDB = D / 32, NKK = D / 16;
  static_assert(QT == 64, "the tile loop is written for two 32-row blocks per tile");
  extern __shared__ __attribute__((aligned(256))) char smem[];   // dkdv_operand relies on the alignment

  // hand-off words of the unit queue: int 8 = slot of the first take, ints 12..15 = record of the next unit
  int* qwords = (int*)(smem + C::CNT_OFF);
  i32x4 rec = {-1, 0, 0, 0};
  FmDirectUnit direct = {};
  if (!DIRECT) {
    rec = queue_take(a.queue_dkdv, qwords + 8);
  } else {
    args_at_once(a.order, a.k, a.lts, a.lte, a.uts, a.ute, a.N, a.Np, a.H);
    direct = fm_direct_unit<false>(a.order, (int)blockIdx.x);
    rec[0] = direct.block;
    rec[2] = (a.N + QT - 1) / QT;   // every row block may be live
  }
  if (rec[0] < 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, c = lane & 31;
  const int N = a.Np, H = a.H;            // padded length: what the loops and tables see
  const int Hk = GEN ? a.Hk : H, G = GEN ? H / Hk : 1;   // K/V heads, query heads per K/V head
  const int Nr = RAGGED ? a.N : a.Np;     // rows the tensors really have
  const int t_c = (Nr + C::BC - 1) / C::BC;
  constexpr int WK = 4 / S;               // waves that share the unit's keys, 32 each
  const int wkey = S == 1 ? wave : wave % WK, grp = S == 1 ? 0 : wave / WK;
  const int q_rs = row_stride<D, GEN>(a.sq), k_rs = row_stride<D, GEN>(a.sk), v_rs = row_stride<D, GEN>(a.sv);
  const int do_rs = row_stride<D, GEN>(a.sdo);
  int* list = (int*)smem;
  int* wave_cnt = (int*)(smem + C::CNT_OFF);
  const float sc = a.scale * kLog2e;
  // lane-dependent LDS offsets inside a tile (row block 0, first column group)
  const int i16 = lane & 15, half = (lane >> 4) & 1;
  const int a_base = C::L::off(c, 16 * g);
  const int t_base0 = C::L::off(4 * g + (i16 >> 2), (16 * half + 4 * (i16 & 3)) * 2);
  const int t_base1 = C::L::off(4 * g + (i16 >> 2) + 8, (16 * half + 4 * (i16 & 3)) * 2);
  CopyLanes<D> copy_lanes, copy_lanes_do_;
  copy_lanes.init(lane, 2 * q_rs);
  if (GEN) copy_lanes_do_.init(lane, 2 * do_rs);
  const CopyLanes<D>& copy_lanes_do = GEN ? copy_lanes_do_ : copy_lanes;
  const unsigned lds_ring = lds_address(smem) + C::STAGE_OFF;

  DkdvAhead<S> ah;
  ah.q_rs2 = 2 * q_rs;
  ah.do_rs2 = 2 * do_rs;
#pragma unroll
  for (int s = 0; s < CopyLanes<D>::NINST; ++s) {
    ah.lanes.v[s] = copy_lanes.v[s];
    ah.lanes_do.v[s] = copy_lanes_do.v[s];
  }
  ah.wave = wave;
  ah.n_real = Nr;
  ah.lane = lane;
  bf16x8 op[C::RD];

  // One pass of the tile loop over list entries [T0, T1) with the element mask compiled in or
  // out.  Tiles that need no element mask are listed first and run through the mask-free
  // instantiation, partially masked ones (for the workgroup's 128 keys) through the other;
  // keeping the two instantiations in separate loops keeps the 128 accumulator registers where
  // they are (merged into one loop, the compiler shuffled all of them every tile; a third loop for
  // tiles that need only one of the two intervals made it spill inside the mask-free one).
  // Entries past the end of the list repeat the last one: the copies and operand
  // fetches made for them are never used, and every entry costs the same number of copies.
  // S = 2: t counts steps of two tiles, of which this wave's group takes one.
  // A step's list entries are read without a bound and its stages follow from the last step's: 394 instead of 407 instructions
  // a tile at d = 128 (branches not counted), dK/dV prefix 32768 6775 -> 6703 us, documents at 131072 4225 -> 4173, answers 16384 1190 -> 1175.
#define FM_TILE_LOOP(T0, T1, MASK)                                                                     \
  for (int t = (T0); t < (T1); ++t) {                                                                  \
    const int v_next = list[S * (t + 1) + grp];                                                        \
    constexpr int AHEAD = C::AHEAD;   /* steps between a tile and the one copied beside it */            \
    _Pragma("unroll") for (int s_ = 0; s_ < S; ++s_) ah.v_copy[s_] = list[S * (t + AHEAD) + s_];       \
    ah.nqs = st_next;                                                                                  \
    const unsigned st_after = stage_after(st_next);                                                    \
    ah.lds_copy = S == 2 ? st_next - grp * C::STAGE : AHEAD == 2 ? st_after : stage_after(st_after);    \
    const int r0 = (e_cur & 0xFFFFFF) * QT;                                                            \
    dkdv_tile<D, MASK, RAGGED, S>(st_cur, ah, op, kreg, vreg, dkacc, dvacc, \
                         a_base, t_base0, t_base1, r0, g, sc, b_lts, len_lt, b_uts, len_ut);           \
    e_cur = __builtin_amdgcn_readfirstlane(v_next);                                                    \
    st_cur = st_next;                                                                                  \
    st_next = st_after;                                                                                \
  }

  // the first unit's min/max values (Section 4.2's table); the later units' arrive with their records
  MinMax8 gmm;
  if (!DIRECT) {
    const int bh0 = rec[0] / t_c;
    gmm = load_minmax(a.minmax_dkdv + (size_t)(bh0 / Hk) * 8 * t_c, t_c, rec[0] - bh0 * t_c);
    // into scalar registers here, once: left in vector registers, every unit's list build would wait for
    // "these loads" again, i.e. for everything the workgroup has in flight, the previous unit's result
    // stores included
#pragma unroll
    for (int e = 0; e < 8; ++e) gmm.v[e] = __builtin_amdgcn_readfirstlane(gmm.v[e]);
  }

  const bool one_round = DIRECT || !C::PERSISTENT || a.queue_dkdv.first == a.queue_dkdv.tickets;   // a workgroup per unit
  // A workgroup works units off until the queues are empty: the launch holds as many workgroups as the
  // chip runs at once, and the next unit's ticket, record and min/max values are fetched while the first
  // tile copies of the current unit are in flight.
  while (true) {
  const int unit = rec[0], i_lo = rec[1], i_hi = rec[2];
  const int bh = DIRECT ? direct.slice : unit / t_c, j_blk = DIRECT ? direct.block : unit - bh * t_c;
  const int b = bh / Hk, hk = bh - b * Hk;   // bh counts K/V heads
  const int k0 = j_blk * C::BC;
  const int kw0 = k0 + wkey * 32;
  const int key = kw0 + c;  // this lane's key column
  const int key_ld = RAGGED ? min(key, Nr - 1) : key;

  const __bf16* kp = slice_ptr<D, GEN>(a.k, a.sk, b, hk, Hk, Nr);
  const __bf16* vp = slice_ptr<D, GEN>(a.v, a.sv, b, hk, Hk, Nr);

  // Lanes past the last key work on a copy of it, its bounds like its K and V: what they sum is stored nowhere, and
  // the columns that do not exist keep no tile of a direct unit alive (as columns that mask every row they left every
  // row block partially masked).
  const size_t bnd = (size_t)b * Nr + key_ld;
  int b_lts = a.lts[bnd], b_lte = a.lte[bnd], b_uts = a.uts[bnd], b_ute = a.ute[bnd];
  // Requested first: a direct unit's list is built from them, and loads return in order.  Training step, d = 128, N = 512
  // 35.0 -> 33.9 us, N = 1500 window 200 55.1 -> 54.1, causal 2048, 24 slices 199.2 -> 196.9; d = 64 0.3 to 1.3 %.
  __builtin_amdgcn_sched_barrier(0);
  // K and V fragments of this wave's 32 keys (B operands of S = Q K^T, dP = dO V^T), which like the four
  // bounds of this lane's key stay in registers (Algorithm 2 loads them once per key
  // block).  They are only waited for after the first tile copies have been issued.
  bf16x8 kreg[NKK], vreg[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    kreg[kk] = *(const bf16x8*)(kp + (size_t)key_ld * k_rs + kk * 16 + 8 * g);
    vreg[kk] = *(const bf16x8*)(vp + (size_t)key_ld * v_rs + kk * 16 + 8 * g);
  }

  if (DIRECT) {   // the unit's min/max values from its own keys' bounds: over the wave's 32 keys, then over the waves
    const int own[4] = {b_lts, b_lte, b_uts, b_ute};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int mx = row16_max(own[e]), mn = row16_min(own[e]);
      gmm.v[2 * e] = max(mx, __shfl_xor(mx, 16, 64));
      gmm.v[2 * e + 1] = min(mn, __shfl_xor(mn, 16, 64));
    }
    if (lane == 0 && grp == 0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) qwords[32 + 8 * wkey + e] = gmm.v[e];
    }
    barrier_nofence();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      int x = qwords[32 + e];
#pragma unroll
      for (int w = 1; w < WK; ++w) x = e & 1 ? min(x, qwords[32 + 8 * w + e]) : max(x, qwords[32 + 8 * w + e]);
      gmm.v[e] = __builtin_amdgcn_readfirstlane(x);
    }
  }

  f32x16 dkacc[NDB], dvacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      dkacc[db][r] = 0.f;
      dvacc[db][r] = 0.f;
    }
  bool drawn = one_round;   // the next unit's ticket has been drawn (uniform over the workgroup), or there is none

  // only the row blocks [i_lo, i_hi) can be live for this key block (found by the work pre-pass)
  for (int chunk = i_lo; chunk < i_hi; chunk += C::LIST_CAP) {
    int n_plain = 0;
    const int n_live = build_live_row_blocks(gmm, Nr, QT, chunk, min(chunk + C::LIST_CAP, i_hi), list, wave_cnt, n_plain);
    if (n_live == 0) continue;
    // behind the list, from its own end on (read in the loops, behind the barrier in front of them)
    if (tid < S * (C::AHEAD + 1)) list[n_live + tid] = list[n_live - 1];
    static_assert(S * (C::AHEAD + 1) <= C::LIST_PAD, "what the loops read past the end");
    // the query heads that share this K/V head, one after the other (one pass if there is no sharing)
    for (int hq = 0; hq < (GEN ? G : 1); ++hq) {
    const int h = hk * G + hq;
    const __bf16* qp = slice_ptr<D, GEN>(a.q, a.sq, b, h, H, Nr);
    const __bf16* dop = slice_ptr<D, GEN>(a.dout, a.sdo, b, h, H, Nr);
    // every wave copies its 16 rows of a tile's lse and D slices with lanes 0..7:
    // lanes 0-3 lse, lanes 4-7 D, 16 bytes each
    const float* my_vec = ((lane & 4) ? a.dvec : a.lse2) + (size_t)(b * H + h) * N + wave * 16 + (lane & 3) * 4;
    ah.q_base = CopyLanes<D>::wave_base(qp, wave, ah.q_rs2);
    ah.do_base = CopyLanes<D>::wave_base(dop, wave, ah.do_rs2);
    ah.vec_src = my_vec;
    // prologue: copies of the tiles of the first AHEAD steps, then the first tile's first operands
    constexpr int FIRST = S * C::AHEAD;
#pragma unroll
    for (int p = 0; p < FIRST; ++p) {
      const int i_p = __builtin_amdgcn_readfirstlane(list[min(p, n_live - 1)]) & 0xFFFFFF;
      const char* st_ = smem + C::STAGE_OFF + p * C::STAGE;
      if (RAGGED && (i_p + 1) * QT > Nr) {
        tile_load_async_clamped<D>(qp, i_p * QT, Nr, st_, wave, lane, 2 * q_rs);
        tile_load_async_clamped<D>(dop, i_p * QT, Nr, st_ + C::Q_BYTES, wave, lane, 2 * do_rs);
      } else {
        tile_load_async<D>(ah.q_base + (size_t)i_p * QT * ah.q_rs2, copy_lanes, st_, wave);
        tile_load_async<D>(ah.do_base + (size_t)i_p * QT * ah.do_rs2, copy_lanes_do, st_ + C::Q_BYTES, wave);
      }
      async_copy16_lanes8(my_vec + i_p * QT, lds_address(st_ + C::Q_BYTES + C::DO_BYTES) + wave * 128);
    }
    // the next unit's ticket and record, while these copies are in flight
    if (!DIRECT && !drawn) {
      if (wave == 0) queue_prefetch_key_block(a.queue_dkdv, qwords + 12, a.minmax_dkdv, t_c, Hk);
      drawn = true;
    }
    // The fragment and bound loads must be complete, and known complete to the compiler, before
    // the tile loops: a compiler-inserted wait for them inside a loop would also drain the
    // copies in flight there.  (No-op after the first chunk.)
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      settle(kreg[kk]);
      settle(vreg[kk]);
    }
    settle(b_lts);
    settle(b_lte);
    settle(b_uts);
    settle(b_ute);
    // lengths of the key's two masked row intervals, for the element mask's compare
    const unsigned len_lt = interval_length(b_lts, b_lte), len_ut = interval_length(b_uts, b_ute);
    async_wait<S == 2 ? 0 : (C::AHEAD - 1) * C::NC>();
    barrier_nofence();
    int e_cur = __builtin_amdgcn_readfirstlane(list[min(grp, n_live - 1)]);
    // this group's stages of this step and the next
    auto stage_after = [&](unsigned st) __attribute__((always_inline)) {   // the one S further on in the ring
      const unsigned x = st + S * C::STAGE;
      return x >= lds_ring + C::NSTAGE * C::STAGE ? x - C::NSTAGE * C::STAGE : x;
    };
    unsigned st_cur = lds_ring + grp * C::STAGE, st_next = stage_after(st_cur);
#pragma unroll
    for (int x = 0; x < C::RD; ++x)
      op[x] = dkdv_operand<D>(dkdv_bases(st_cur, a_base, t_base0, t_base1), x);
    // this group's tiles: entries grp, grp + S, ... (the clamp is for a group without any)
    const int own_plain = (max(n_plain - grp, 0) + S - 1) / S, own_live = (max(n_live - grp, 0) + S - 1) / S;
    FM_TILE_LOOP(0, own_plain, false)
    FM_TILE_LOOP(own_plain, own_live, true)
    if (S == 2 && own_live < (n_live + S - 1) / S) {   // the last step has no tile for this group: its barriers
      barrier_reads_in_flight();
      async_wait<0>();
      barrier_reads_in_flight();
    }
    mfma_acc_drain();  // dkacc / dvacc are read by ordinary code after the loops over heads and chunks
    async_wait<0>();   // the copies made for entries past the end must not outlive the list / the workgroup
    __syncthreads();   // the ring is refilled by the next head, the list rebuilt by the next chunk
    }  // query heads
  }
  if (!DIRECT && !drawn) {   // a unit without a live tile: nothing was in flight to hide the draw behind
    if (wave == 0) queue_prefetch_key_block(a.queue_dkdv, qwords + 12, a.minmax_dkdv, t_c, Hk);
  }

  // accumulators (dK^T, dV^T): register r of block db holds [d = db*32 + 8*(r/4) + 4*g + r%4][key kw0 + c].
  // Nothing is in flight into the ring here and every wave is past its last tile (the barrier that ends the
  // loop over heads and chunks), so the ring's first bytes serve as the waves' store staging.
  __bf16* dkp = (__bf16*)slice_ptr<D, GEN>(a.dk, a.sdk, b, hk, Hk, Nr);
  __bf16* dvp_out = (__bf16*)slice_ptr<D, GEN>(a.dv, a.sdv, b, hk, Hk, Nr);
  const int dk_rs = row_stride<D, GEN>(a.sdk), dv_rs = row_stride<D, GEN>(a.sdv);
  if constexpr (S == 2) {
    // The two groups' sums of the same keys meet in LDS: the first group finishes dK, the second dV.
    using RSt = RowStage<D>;
    static_assert(4 * RSt::BYTES + 4 * 64 * 16 * NDB * 4 <= C::NSTAGE * C::STAGE, "exchange fits the ring");
    char* stage = smem + C::STAGE_OFF + wave * RSt::BYTES;
    float* const exchange = (float*)(smem + C::STAGE_OFF + 4 * RSt::BYTES) + lane * 4;
    constexpr int PER_WAVE = 64 * 16 * NDB;
    auto give = [&](const f32x16(&acc)[NDB]) __attribute__((always_inline)) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *(f32x4*)(exchange + wave * PER_WAVE + (db * 4 + q) * 256) =
              f32x4{acc[db][4 * q], acc[db][4 * q + 1], acc[db][4 * q + 2], acc[db][4 * q + 3]};
    };
    auto finish = [&](const f32x16(&acc)[NDB], float factor, __bf16* rows, int rs) __attribute__((always_inline)) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 o = *(const f32x4*)(exchange + (wave ^ WK) * PER_WAVE + (db * 4 + q) * 256);
          bf16x4 x4;
#pragma unroll
          for (int e = 0; e < 4; ++e) x4[e] = (__bf16)((acc[db][4 * q + e] + o[e]) * factor);
          RSt::put(stage, c, g, db, q, x4);
        }
      RSt::flush(stage, rows + (size_t)kw0 * rs, rs, lane, RAGGED ? min(32, Nr - kw0) : 32);
    };
    if (grp == 0) give(dvacc);
    else give(dkacc);
    barrier_nofence();
    if (grp == 0) finish(dkacc, a.scale, dkp, dk_rs);
    else finish(dvacc, 1.f, dvp_out, dv_rs);
    return;   // one unit per workgroup
  } else {
    using RSt = RowStage<D>;
    static_assert(8 * RSt::BYTES <= C::NSTAGE * C::STAGE, "store staging fits the ring");
    char* stage_k = smem + C::STAGE_OFF + (2 * wave) * RSt::BYTES;
    char* stage_v = stage_k + RSt::BYTES;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        bf16x4 k4, v4;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          k4[e] = (__bf16)(dkacc[db][4 * q + e] * a.scale);
          v4[e] = (__bf16)dvacc[db][4 * q + e];
        }
        RSt::put(stage_k, c, g, db, q, k4);
        RSt::put(stage_v, c, g, db, q, v4);
      }
    const int n_rows = RAGGED ? min(32, Nr - kw0) : 32;
    RSt::flush(stage_k, dkp + (size_t)kw0 * dk_rs, dk_rs, lane, n_rows);
    RSt::flush(stage_v, dvp_out + (size_t)kw0 * dv_rs, dv_rs, lane, n_rows);
  }
  if (one_round) break;
  __syncthreads();                       // the next record is in LDS (written before the tile loops, or just above)
  rec = queue_next_record(qwords + 12);
  if (rec[0] < 0) break;
#pragma unroll
  for (int e = 0; e < 8; ++e) gmm.v[e] = __builtin_amdgcn_readfirstlane(qwords[16 + e]);
  __syncthreads();                       // everyone has read it before the next unit's draw overwrites it
  }
#undef FM_TILE_LOOP
}

template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(256, FM_DQ_PER_CU) void dq_kernel(FmBwdKernelArgs<GEN> a) {
  dq_body<D, RAGGED, GEN, 1, 4, false>(a);
}
template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(256, fm_dkdv_per_cu(D)) void dkdv_kernel(FmBwdKernelArgs<GEN> a) {
  dkdv_body<D, RAGGED, GEN, 1, false>(a);
}
// Direct units.  LDS for two tiles per step leaves one workgroup per compute unit at d = 128, two at d = 64.
template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(256, FM_DQ_PER_CU) void single_dq_kernel(FmBwdKernelArgs<GEN> a) {
  dq_body<D, RAGGED, GEN, 1, 4, true>(a);
}
template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void direct_dq_kernel(FmBwdKernelArgs<GEN> a) {
  dq_body<D, RAGGED, GEN, 2, 2, true>(a);
}
template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(512, 1) void wide_dq_kernel(FmBwdKernelArgs<GEN> a) {
  dq_body<D, RAGGED, GEN, 2, 4, true>(a);
}
template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(256, fm_dkdv_per_cu(D)) void single_dkdv_kernel(FmBwdKernelArgs<GEN> a) {
  dkdv_body<D, RAGGED, GEN, 1, true>(a);
}
template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(256, fm_dkdv_per_cu(D)) void direct_dkdv_kernel(FmBwdKernelArgs<GEN> a) {
  dkdv_body<D, RAGGED, GEN, 2, true>(a);
}

}  // namespace fm

using namespace fm;

template <int D, bool RAGGED, bool GEN, FmUnits U>
struct DqLaunch {
  using C = DqCfg<D, fm_groups(U), fm_group_waves(U), U != FM_QUEUED>;
  static constexpr auto kernel() {
    if constexpr (U == FM_QUEUED) return dq_kernel<D, RAGGED, GEN>;
    else if constexpr (U == FM_DIRECT) return single_dq_kernel<D, RAGGED, GEN>;
    else if constexpr (U == FM_DIRECT_HALVED) return direct_dq_kernel<D, RAGGED, GEN>;
    else return wide_dq_kernel<D, RAGGED, GEN>;
  }
  static FmLdsLimit lds() { return {(const void*)kernel(), C::LDS_BYTES}; }
};

template <int D, bool RAGGED, bool GEN, FmUnits U>
static hipError_t launch_dq_s(const FmBwdArgs& a, hipStream_t stream) {
  using L = DqLaunch<D, RAGGED, GEN, U>;
  using C = typename L::C;
  auto args = fm_kernel_args<GEN>(a);
  const int blocks = (a.N + C::BR - 1) / C::BR;
  if (U == FM_QUEUED) args.queue_dq = fm_queue_for_launch(a.queue_dq, FM_DQ_PER_CU);
  else args.order = fm_direct_order(a.B * a.Hk, a.H / a.Hk, blocks, a.B * a.H * blocks <= fm_compute_units());
  const int grid = U == FM_QUEUED ? fm_launch_grid(args.queue_dq) : fm_direct_grid(args.order);
  hipLaunchKernelGGL(L::kernel(), dim3(grid), dim3(C::THREADS), C::LDS_BYTES, stream, args);
  return hipGetLastError();
}

template <int D, bool RAGGED, bool GEN>
static hipError_t launch_dq_t(const FmBwdArgs& a, hipStream_t stream) {
  static bool allowed[FM_MAX_DEVICES] = {};
  if (hipError_t e = fm_allow_lds({DqLaunch<D, RAGGED, GEN, FM_QUEUED>::lds(),
                                   DqLaunch<D, RAGGED, GEN, FM_DIRECT>::lds(),
                                   DqLaunch<D, RAGGED, GEN, FM_DIRECT_HALVED>::lds(),
                                   DqLaunch<D, RAGGED, GEN, D == 128 ? FM_DIRECT_PAIRED : FM_QUEUED>::lds()},
                                  allowed);
      e != hipSuccess)
    return e;
  switch (a.units_dq) {
    case FM_DIRECT: return launch_dq_s<D, RAGGED, GEN, FM_DIRECT>(a, stream);
    case FM_DIRECT_HALVED: return launch_dq_s<D, RAGGED, GEN, FM_DIRECT_HALVED>(a, stream);
    case FM_DIRECT_PAIRED:
      if constexpr (D == 128) return launch_dq_s<D, RAGGED, GEN, FM_DIRECT_PAIRED>(a, stream);
    default: return launch_dq_s<D, RAGGED, GEN, FM_QUEUED>(a, stream);
  }
}

template <int D>
static hipError_t launch_dq_d(const FmBwdArgs& a, hipStream_t stream) {
  const bool ragged = a.Np != a.N;
  if (a.general) return ragged ? launch_dq_t<D, true, true>(a, stream) : launch_dq_t<D, false, true>(a, stream);
  return ragged ? launch_dq_t<D, true, false>(a, stream) : launch_dq_t<D, false, false>(a, stream);
}

hipError_t fm_launch_bwd_dq(const FmBwdArgs& a, hipStream_t stream) {
  return a.d == 128 ? launch_dq_d<128>(a, stream) : launch_dq_d<64>(a, stream);
}

template <int D, bool RAGGED, bool GEN, FmUnits U>
struct DkdvLaunch {
  using C = DkdvCfg<D, fm_groups(U)>;
  static constexpr auto kernel() {
    if constexpr (U == FM_QUEUED) return dkdv_kernel<D, RAGGED, GEN>;
    else if constexpr (U == FM_DIRECT) return single_dkdv_kernel<D, RAGGED, GEN>;
    else return direct_dkdv_kernel<D, RAGGED, GEN>;
  }
  static FmLdsLimit lds() { return {(const void*)kernel(), C::LDS_BYTES}; }
};

template <int D, bool RAGGED, bool GEN, FmUnits U>
static hipError_t launch_dkdv_s(const FmBwdArgs& a, hipStream_t stream) {
  using L = DkdvLaunch<D, RAGGED, GEN, U>;
  using C = typename L::C;
  auto args = fm_kernel_args<GEN>(a);
  const int blocks = (a.N + C::BC - 1) / C::BC;
  if (U == FM_QUEUED) args.queue_dkdv = fm_queue_for_launch(a.queue_dkdv, C::PER_CU);
  else args.order = fm_direct_order(a.B * a.Hk, 1, blocks, a.B * a.Hk * blocks <= fm_compute_units());
  const int grid = U != FM_QUEUED   ? fm_direct_grid(args.order)
                   : C::PERSISTENT ? fm_persistent_grid(args.queue_dkdv)
                                   : fm_launch_grid(args.queue_dkdv);
  hipLaunchKernelGGL(L::kernel(), dim3(grid), dim3(256), C::LDS_BYTES, stream, args);
  return hipGetLastError();
}

template <int D, bool RAGGED, bool GEN>
static hipError_t launch_dkdv_t(const FmBwdArgs& a, hipStream_t stream) {
  static bool allowed[FM_MAX_DEVICES] = {};
  if (hipError_t e = fm_allow_lds({DkdvLaunch<D, RAGGED, GEN, FM_QUEUED>::lds(),
                                   DkdvLaunch<D, RAGGED, GEN, FM_DIRECT>::lds(),
                                   DkdvLaunch<D, RAGGED, GEN, FM_DIRECT_HALVED>::lds()},
                                  allowed);
      e != hipSuccess)
    return e;
  switch (a.units_dkdv) {
    case FM_DIRECT: return launch_dkdv_s<D, RAGGED, GEN, FM_DIRECT>(a, stream);
    case FM_DIRECT_HALVED: return launch_dkdv_s<D, RAGGED, GEN, FM_DIRECT_HALVED>(a, stream);
    default: return launch_dkdv_s<D, RAGGED, GEN, FM_QUEUED>(a, stream);
  }
}

template <int D>
static hipError_t launch_dkdv_d(const FmBwdArgs& a, hipStream_t stream) {
  const bool ragged = a.Np != a.N;
  if (a.general) return ragged ? launch_dkdv_t<D, true, true>(a, stream) : launch_dkdv_t<D, false, true>(a, stream);
  return ragged ? launch_dkdv_t<D, true, false>(a, stream) : launch_dkdv_t<D, false, false>(a, stream);
}

hipError_t fm_launch_bwd_dkdv(const FmBwdArgs& a, hipStream_t stream) {
  return a.d == 128 ? launch_dkdv_d<128>(a, stream) : launch_dkdv_d<64>(a, stream);
}
