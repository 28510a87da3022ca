#pragma once
// Backward attention, dQ part (gfx950), query-major.
//
// Same work items and schedule as the fused forward: one workgroup takes a
// tile of query tokens of one piece for `heads_per_tile` query heads of one
// KV head, and walks the received key range (no mask) and then the local key
// range (intra-document causal). Key/value tiles of 64 keys are
// double-buffered in LDS (asynchronous HBM-to-LDS copies) and shared by the
// waves, i.e. by the heads of the group. Per tile, with a query per lane:
//   S^T = K Q^T, dP^T = V dO^T      Q and dO held in registers;
//   P = exp(S - LSE), dS = P (dP - D)  LSE and D are per-lane scalars;
//   dQ^T += K^T dS^T                 K^T read from LDS with transpose reads.
// dQ is produced whole by the workgroup that owns the query rows, so it is
// written once, without atomics, and is deterministic. Recomputing S and dP
// here costs two extra products per key tile compared with accumulating dQ
// inside the key-major kernel, but removes that kernel's dQ traffic and
// frees the registers and LDS that limit its occupancy.
#include "common.hpp"
#include "launch.hpp"

#include <type_traits>

namespace fck {

template <int D>
struct DqLds {
  static constexpr uint32_t bytes = 4 * 64 * D * 2;
};

// One workgroup's query tile (workgroup index b); smem: DqLds<D>::bytes of
// shared memory. HOLD: sixteen registers hold -D for dP's accumulators.
template <int D, int HPW, bool HOLD>
__device__ __forceinline__ void dq_tile(const DqParams& p, int b, char* smem) {
  constexpr int BN = 64;
  constexpr int RPW = 32 / HPW;  // query rows per wave and head
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr uint32_t TILE = BN * D * 2;  // bytes of one K or V tile
  // LDS: K0 | V0 | K1 | V1 (double buffer); the loop is unrolled by two so
  // every read names its buffer with a compile-time offset
  static_assert(4 * TILE == DqLds<D>::bytes, "LDS layout");

  const int lane = threadIdx.x & 63, wave = wave_id();
  const int half = lane >> 5;
  const int kvh = b % p.hkv;
  const int rest = b / p.hkv;
  const int hc = rest % p.head_chunks;
  const int32_t* it = p.items + 8 * (rest / p.head_chunks);
  const int q0 = it[0], q1 = it[1], r0 = it[2], r1 = it[3], l0 = it[4], l1 = it[5];
  const int ldiag = it[6];

  // lane -> (query row, head) as in the forward: RPW rows of each of the
  // HPW heads per wave; a wave with no row skips the products
  const int l31 = lane & 31;
  const int h = kvh * p.group + hc * HPW + l31 / RPW;
  const int qrow = q0 + wave * RPW + l31 % RPW;
  const bool qvalid = qrow < q1;
  const bool active = q0 + wave * RPW < q1;  // wave-uniform
  const float sl2 = p.scale * kLog2e;

  const int n_r = (r1 - r0 + BN - 1) / BN;
  const int n_t = n_r + (l1 - l0 + BN - 1) / BN;

  const TileLoader<D, BN> ld(p.hkv * D);
  auto fetch = [&](int j, uint32_t kofs) {
    const bool rs = j < n_r;
    const int k0 = rs ? r0 + j * BN : l0 + (j - n_r) * BN;
    const int hi = rs ? r1 : l1;
    const size_t base = (size_t(k0) * p.hkv + kvh) * D;
    ld.load_at(lds_addr(smem) + kofs, (rs ? p.k_recv : p.k_loc) + base, hi - k0);
    ld.load_at(lds_addr(smem) + kofs + TILE, (rs ? p.v_recv : p.v_loc) + base, hi - k0);
  };

  // the workgroup's Q and dO rows through LDS first (Q over the second K/V
  // buffer, dO over the first), then key tile 0
  const int h0 = kvh * p.group + hc * HPW;
  load_pairs<D, RPW>(lds_addr(smem) + 2 * TILE, p.q, q0, q1, p.hq, h0);
  load_pairs<D, RPW>(lds_addr(smem), p.dout, q0, q1, p.hq, h0);

  bf16x8 qreg[KS], oreg[KS];
  float lse2 = 0.f, ndel = 0.f;
  if (qvalid) {
    lse2 = p.lse[(size_t)h * p.t_q + qrow] * kLog2e;
    ndel = -p.delta[(size_t)h * p.t_q + qrow];
  }

  // per-lane LDS byte offsets: K/V rows for k-step ks, and the two transpose
  // reads of K^T block db
  uint32_t pr[KS], pt[DB][2];
  {
    const int rb = row_base<D>(0, lane), tb = tr_base<D>(lane);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) pr[ks] = 2u * uint32_t(rb ^ (ks << 4));
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      pt[db][0] = 2u * uint32_t(tb ^ (db << 5));
      pt[db][1] = 2u * uint32_t((tb ^ ((db << 5) | 16)) + 8 * D);
    }
  }

  f32x16 dq[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) dq[db] = zero16();
  wait_async();
  __syncthreads();
  if (active) {
    const int qb = row_base<D>(32 * wave, lane);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qreg[ks] = lds_b128(smem, 2u * uint32_t(qb ^ (ks << 4)), 2 * TILE);
      oreg[ks] = lds_b128(smem, 2u * uint32_t(qb ^ (ks << 4)), 0);
    }
  }
  __syncthreads();  // every wave holds its rows before tile 0 overwrites them
  if (n_t > 0) fetch(0, 0);
  wait_async();
  __syncthreads();

  // One key tile. Its MFMAs run as one software pipeline of slots:
  //   S^T, keys 0-31; S^T, keys 32-63 (with P of keys 0-31); dP^T, keys 0-31
  //   (with P of keys 32-63); dP^T, keys 32-63 (with dS of keys 0-31);
  //   dQ^T += K^T dS^T over keys 0-31 (with dS of keys 32-63), then 32-63.
  // Each slot issues the LDS reads of the slot two ahead, its MFMA and its
  // share of the vector work, which runs while the MFMA does; a scheduling
  // barrier after each slot keeps this order.
  constexpr int NS = 4 * KS + 4 * DB;        // slots per tile
  constexpr int EP = 16 / KS, EQ = 8 / DB;   // elements per slot (P, dS)
  constexpr int INIT0 = KS - 2, INIT1 = HOLD ? KS - 1 : 3 * KS - 2;  // of dP, see below
  auto step = [&](int j, auto buf) {
    constexpr uint32_t KO = decltype(buf)::value * 2 * TILE, VO = KO + TILE;
    if (j + 1 < n_t) fetch(j + 1, 2 * TILE - KO);
    const bool rs = j < n_r;
    const int k0 = rs ? r0 + j * BN : l0 + (j - n_r) * BN;
    const int hi = rs ? r1 : l1;
    if (active) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) pr[ks] = opaque(pr[ks]);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        pt[db][0] = opaque(pt[db][0]);
        pt[db][1] = opaque(pt[db][1]);
      }
      // key k0 + 4*half + c (c = 32*mb + 8*(i/4) + i%4 for register i) is seen
      // iff c < rel: keys past the range, and later keys on diagonal tiles,
      // give P = 0. Only edge tiles (diagonal, or running past the range)
      // mask, in one branch before each half's dS.
      const bool diag = !rs && k0 >= ldiag;
      const int rel = (diag ? min(hi, qrow + 1) : hi) - k0 - 4 * half;
      const bool edge = diag || k0 + BN > hi;

      f32x16 s[2] = {zero16(), zero16()}, dp[2];
      bf16x8 ring[3], sb[4];
      auto rd = [&](int n) {
        bf16x8& a = ring[n % 3];
        if (n < 4 * KS) {  // K rows (S) or V rows (dP)
          const int ks = n % KS, mb = (n / KS) & 1;
          a = lds_b128(smem, pr[ks], (n < 2 * KS ? KO : VO) + mb * 64 * D);
        } else {  // K^T for dQ
          const int u = n - 4 * KS, kk = u / DB, db = u % DB;
          const uint32_t ro = KO + kk * 32 * D;
          a = cat8(lds_tr(smem, pt[db][0], ro), lds_tr(smem, pt[db][1], ro));
        }
      };
      auto pexp = [&](int mb, int i) {
        s[mb][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[mb][i], sl2, -lse2));
      };
      auto mask = [&](int mb) {
        if (edge) {
#pragma unroll
          for (int i = 0; i < 16; ++i)
            s[mb][i] = 32 * mb + 8 * (i >> 2) + (i & 3) < rel ? s[mb][i] : 0.f;
        }
      };
      // dP's accumulators start from -D, as in the dK/dV workgroups (whose dS
      // has the same bits). With HOLD (head dim 64) sixteen registers hold it
      // for the first MFMA; at 128 there is no room for them, and the
      // accumulators are set: the first 32 keys' beside the first S products,
      // which have no other vector work, the others' two slots before they are
      // read (set together with the first, sixteen registers live through eight
      // more slots cost the grid a spill; either is as fast). Two registers per
      // move, named here (the compiler would write two moves); volatile, so that
      // they stay slots ahead of the MFMA that reads them. Layer of 16/8 heads of 64 over 32K
      // tokens: 349 -> 342 us (120 instead of 152 vector instructions beside 24
      // MFMAs); at 128, within noise.
      auto dp_init = [&](int mb) {
        if constexpr (HOLD) {
#pragma unroll
          for (int i = 0; i < 16; ++i) dp[mb][i] = ndel;
        } else {
          typedef uint64_t u64x8 __attribute__((ext_vector_type(8)));
          const uint32_t x = __builtin_bit_cast(uint32_t, ndel);
          u64x8 y;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            uint64_t r;
            asm volatile("v_mov_b64 %0, %1" : "=v"(r) : "v"(uint64_t(x) << 32 | x));
            y[i] = r;
          }
          dp[mb] = __builtin_bit_cast(f32x16, y);
        }
      };
      auto dsv = [&](int mb, int i) { dp[mb][i] *= s[mb][i]; };
      rd(0);
      rd(1);
      static_for<0, NS>([&](auto nc) {
        constexpr int n = decltype(nc)::value;
        if (n + 2 < NS) rd(n + 2);
        const bf16x8& a = ring[n % 3];
        if (n < 2 * KS) {
          const int ks = n % KS, mb = n / KS;
          s[mb] = mfma32(a, qreg[ks], s[mb]);
          if (n == INIT0) dp_init(0);
          if (n == INIT1) dp_init(1);
          if (mb == 1)
#pragma unroll
            for (int e = ks * EP; e < (ks + 1) * EP; ++e) pexp(0, e);
        } else if (n < 4 * KS) {
          const int ks = n % KS, mb = (n - 2 * KS) / KS;
          dp[mb] = mfma32(a, oreg[ks], dp[mb]);
          if (n == INIT1) dp_init(1);
          if (mb == 1 && ks == 0) mask(0);
          if (mb == 0) {
#pragma unroll
            for (int e = ks * EP; e < (ks + 1) * EP; ++e) pexp(1, e);
          } else {
#pragma unroll
            for (int e = ks * EP; e < (ks + 1) * EP; ++e) dsv(0, e);
            if ((ks + 1) * EP == 8) sb[0] = pack8(dp[0], 0);
            if ((ks + 1) * EP == 16) sb[1] = pack8(dp[0], 8);
          }
        } else {
          const int u = n - 4 * KS, kk = u / DB, db = u % DB;
          dq[db] = mfma32(a, sb[kk], dq[db]);
          if (u == 0) mask(1);
          if (u < 2 * DB) {
#pragma unroll
            for (int e = u * EQ; e < (u + 1) * EQ; ++e) dsv(1, e);
            if ((u + 1) * EQ == 8) sb[2] = pack8(dp[1], 0);
            if ((u + 1) * EQ == 16) sb[3] = pack8(dp[1], 8);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    wait_async();
    __syncthreads();
  };
  for (int j = 0; j < n_t; j += 2) {
    step(j, std::integral_constant<int, 0>());
    if (j + 1 < n_t) step(j + 1, std::integral_constant<int, 1>());
  }

  // a part of a split key range: the unscaled sums go to the part's slot, in
  // register order (1 KiB per store instruction), and are added up by
  // dq_combine_kernel
  if (p.part && it[7] >= 0) {
    if (active) {
      const size_t slot = (size_t(it[7]) * p.head_chunks + hc) * p.hkv + kvh;
      float* const sl = p.part + (slot * 4 + wave) * (32 * D) + 4 * lane;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 v;
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) v[jj] = dq[db][4 * g + jj];
          *reinterpret_cast<f32x4*>(sl + 256 * (4 * db + g)) = v;
        }
    }
    return;
  }

  // dQ rows out through this wave's share of the (now free) K/V buffers,
  // 1 KiB per store instruction
  store_rows<D, RPW>(
      smem + size_t(wave) * (32 * D * 4), active,
      [&](int db, int g) {
        f32x4 v;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) v[jj] = p.scale * dq[db][4 * g + jj];
        return v;
      },
      q0 + wave * RPW, q1, p.hq, kvh * p.group + hc * HPW, p.dq, nullptr);
}

// dQ of a query tile whose key range was split: the parts' slots added in
// slot order (key order), scaled and stored. A workgroup takes one wave's 32
// rows, a quarter of the columns per wave and four slots in flight at once, so
// that few tiles still spread over the chip: bound by the latency of its reads.
template <int D, int HPW>
__global__ __launch_bounds__(256) void dq_combine_kernel(DqParams p) {
  constexpr int RPW = 32 / HPW, KW = D / 32;  // KW: 16-byte pieces per lane
  __shared__ __attribute__((aligned(16))) float st[32 * D];
  const int lane = threadIdx.x & 63;
  const int qw = blockIdx.x & 3, b = blockIdx.x >> 2;  // the rows' wave, the tile
  const int kvh = b % p.hkv, rest = b / p.hkv, hc = rest % p.head_chunks;
  const int32_t* e = p.comb + 8 * (rest / p.head_chunks);
  const int q0 = e[0], q1 = e[1], first = e[2], n = e[3];
  if (q0 + qw * RPW >= q1) return;
  auto read = [&](f32x4 (&x)[KW], int s) {
    const size_t slot = (size_t(first + s) * p.head_chunks + hc) * p.hkv + kvh;
    const float* const o = p.part + (slot * 4 + qw) * (32 * D) + 256 * KW * wave_id() + 4 * lane;
#pragma unroll
    for (int k = 0; k < KW; ++k) x[k] = *reinterpret_cast<const f32x4*>(o + 256 * k);
  };
  f32x4 acc[KW], x[4][KW];
  auto add = [&](const f32x4 (&y)[KW]) {
#pragma unroll
    for (int k = 0; k < KW; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[k][j] += y[k][j];
  };
  read(acc, 0);
  for (int s = 1; s < n; s += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) read(x[u], min(s + u, n - 1));
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s + u < n) add(x[u]);
  }
  store_rows_shared<D, RPW>(
      st,
      [&](int k) {
        f32x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = p.scale * acc[k][j];
        return v;
      },
      q0 + qw * RPW, q1, p.hq, kvh * p.group + hc * HPW, p.dq, nullptr);
}

template <int D>
static hipError_t launch_dq_combine_d(const DqParams& p, int hpw, hipStream_t s) {
  const dim3 grid(unsigned(p.n_comb) * p.hkv * p.head_chunks * 4), block(256);
  switch (hpw) {
    case 1: hipLaunchKernelGGL((dq_combine_kernel<D, 1>), grid, block, 0, s, p); break;
    case 2: hipLaunchKernelGGL((dq_combine_kernel<D, 2>), grid, block, 0, s, p); break;
    case 4: hipLaunchKernelGGL((dq_combine_kernel<D, 4>), grid, block, 0, s, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace fck
