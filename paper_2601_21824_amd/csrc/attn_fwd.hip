// attn_fwd.hip -- attention forward producing O (bf16) and L = logsumexp (fp32),
// the inputs Algorithm 1 takes.
//
// One workgroup = 4 waves, each with QG groups of 32 query rows; K and V
// arrive in tiles of KT rows by direct global->LDS copies.  The work runs in
// units of 32 keys.  Per wave and unit: S^T = K Q^T on bf16 MFMA 32x32x16 (the
// C layout then holds one query per lane, so row maxima and sums are in-lane up
// to one swap of the lane halves), online softmax in the log2 domain, O^T += V^T P^T
// with P^T fed to the MFMA straight from registers and V^T read from the
// row-major tile by transposed LDS reads.  Deterministic: every reduction is
// inside one wave in a fixed order.
//
// What bounds it: matrix instructions (4 N^2 d FLOP) and, next to them, the
// softmax's VALU work (fused multiply-add, exp, sum, half a max and half a
// conversion per score), which a wave can only overlap with its own MFMAs where
// it stands between two of them (one MFMA hid 6 VALU instructions of its wave in
// a probe).  So the loop is software-pipelined: while unit u's scores go through
// exp, the matrix cores compute unit u+1's scores; while O^T of unit u is summed,
// the VALU adds unit u's row sum and takes unit u+1's maximum; and every MFMA
// is followed by its share of that work.  Two waves per SIMD fill each other's
// waits.  Long calls run at the power limit: 64 heads of 8192 causal at d = 128
// keep the matrix cores busy for 47% of 1.91 GHz, 8 of 32768 full at d = 256 for 43% of 2.24.
//
// Measured (us, in turn on one card, before -> now; before: 64-key steps staged
// through registers, no overlap of scores, softmax and O): 64 heads of 8192 at d = 128
// causal 2494 -> 1183 (441 -> 929 TFLOP/s); 32 heads full 1639 -> 1077; 64 heads
// of 8192 at d = 64 full 1991 -> 1208, causal 1492 -> 697; 8 heads of 16384 at
// d = 256 full 4625 -> 2254; 1024 heads of 512 at d = 128 causal 263 -> 163.  Cards
// differ by 5%.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "bwd_common.h"
#include "lds_layout.h"

namespace dash {

template <int D, int KT, int VBUF>
struct FwdSmem {
  __bf16 k[2][KT * D];
  __bf16 v[VBUF][KT * D];
};

// x of the two lane halves: lo = x of lane l % 32, hi = x of lane l % 32 + 32.
// v_permlane32_swap exchanges the upper half of one register with the lower
// half of another; the s_nop covers the wait it needs after a VALU write of
// its operands (the compiler does not see into the asm).
__device__ inline void halves(float x, float& lo, float& hi) {
  lo = hi = x;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
}
__device__ inline float half_max(float x) {
  float a, b;
  halves(x, a, b);
  return fmaxf(a, b);
}
__device__ inline float half_sum(float x) {
  float a, b;
  halves(x, a, b);
  return a + b;
}

// The score MFMA of head dim 256, with Q held in AGPRs: O^T fills half of the
// VGPRs there, and the compiler, which builds both operands of an MFMA in VGPRs,
// would copy Q out of the AGPRs for every unit (64 reads).  The compiler does not
// see an MFMA here, so its wait states are the caller's: K comes from LDS and
// Q is loaded once, so no VALU instruction writes an operand right before; a read
// of s by another instruction needs score_settle first.
template <bool FIRST>
__device__ inline void mfma32_qa(bf16x8 k, bf16x8 q, f32x16& s) {
  if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(k), "a"(q));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(k), "a"(q));
}
// 20 wait states: more than any MFMA's result takes
__device__ inline void score_settle(f32x16& s) { asm volatile("s_nop 15\n\ts_nop 3" : "+v"(s)); }

__device__ inline float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

__device__ inline bf16x8 lds_b128(uint32_t at) {
  return *(const __attribute__((address_space(3))) bf16x8*)(at);
}
__device__ inline u32x2 lds_tr(uint32_t at) {
  typedef short s16x4 __attribute__((__vector_size__(8)));
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at)));
}

// A wave's rows whose running maximum (log2 domain) is this far from 0, or -inf
// after the first unit, go through far_rows.
constexpr float kFarMax = 1048576.f;

// Rows row0 .. row0 + 31 by one wave from global memory, for rows the pipelined loop
// cannot do: it takes S c2 - m in one fused operation, which for the largest
// score is not 0 but the error of m's own rounding, up to 2^-24 |m|, and 2^that
// overflows from |m| = 2^31 on (keys taken out by an added -1e30, for a row that
// has seen no other yet); and it takes -inf less -inf after 32 keys that all score
// -inf.  Here S c2 is rounded as m was, so that the largest score gives
// P = 1, and keys that score -inf have P = 0 (a row of nothing else: O NaN, L -inf).
// Not tuned, and small: 64 columns of O a pass, each pass with its own scores, V's
// operands gathered two bytes at a time, nothing kept in registers through the
// loop for it (O of 256 columns at once cost the loop of d = 256 3-6%).  Its rows
// cost 2 (d = 64) to 7 (d = 256) times the loop's; taking m off inside the loop
// instead, where it is far, cost every call 2-7%.
template <int D>
__device__ void far_rows(const FwdArgs& a, int bh, int row0) {
  const int l = fresh_lane();
  const int N = a.n, g = l >> 5, lc = l & 31, qrow = row0 + lc;
  const float c2 = a.scale * kLog2e;
  const size_t head = (size_t)bh * N * D;
  const uint32_t hbytes = (uint32_t)((size_t)N * D * 2);
  const auto rq = make_rsrc((const __bf16*)a.q + head, hbytes);
  const auto rk = make_rsrc((const __bf16*)a.k + head, hbytes);
  const auto rv = make_rsrc((const __bf16*)a.v + head, hbytes);
  const auto ro = make_rsrc((__bf16*)a.o + head, hbytes);
  const int end = a.causal ? min(N, row0 + 32) : N;
#pragma clang loop unroll(disable)
  for (int d0 = 0; d0 < D; d0 += 64) {
    f32x16 o[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) o[0][r] = o[1][r] = 0.f;
    float m = -INFINITY, sum = 0.f;
#pragma clang loop unroll(disable)
    for (int k0 = 0; k0 < end; k0 += 32) {
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma clang loop unroll(disable)
      for (int c = 0; c < D; c += 16)
        s = mfma32(as_bf16x8(ld16(rk, (uint32_t)((k0 + lc) * D + c + 8 * g) * 2)),
                   as_bf16x8(ld16(rq, (uint32_t)(qrow * D + c + 8 * g) * 2)), s);
      // element r: key k0 + 8(r/4) + 4g + r%4, query qrow
      const int lim = (a.causal ? min(N - 1, qrow) : N - 1) - k0 - 4 * g;
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float x = s[r] * c2;
        asm("" : "+v"(x));  // rounded: not to be fused with the difference
        s[r] = 8 * (r >> 2) + (r & 3) > lim ? -INFINITY : x;
        mx = fmaxf(mx, s[r]);
      }
      const float mnew = fmaxf(m, half_max(mx));
      const float mm = mnew == -INFINITY ? 0.f : mnew;
      const float alpha = __builtin_amdgcn_exp2f(m - mm);
      m = mnew;
      float rs = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) rs += s[r] = __builtin_amdgcn_exp2f(s[r] - mm);
      sum = sum * alpha + half_sum(rs);
#pragma unroll
      for (int db = 0; db < 2; ++db) {
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          unsigned e[8];
#pragma unroll
          for (int i = 0; i < 8; ++i)
            e[i] = ld2(rv, (uint32_t)((k0 + 16 * h + 8 * (i >> 2) + 4 * g + (i & 3)) * D + d0 + 32 * db + lc) * 2);
          const u32x4 v = {e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16};
          o[db] = mfma32(as_bf16x8(v), pack8(s, 8 * h), o[db]);
        }
      }
    }
    const float inv = 1.f / sum;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        const u32x2 t = {pack_bf16(o[db][4 * rb] * inv, o[db][4 * rb + 1] * inv),
                         pack_bf16(o[db][4 * rb + 2] * inv, o[db][4 * rb + 3] * inv)};
        st8(ro, (uint32_t)(qrow * D + d0 + 32 * db + 8 * rb + 4 * g) * 2, t);
      }
    if (d0 == 0 && g == 0)
      st4f(make_rsrc(a.lse + (size_t)bh * N, (uint32_t)N * 4), (uint32_t)qrow * 4, (m + __log2f(sum)) * kLn2);
  }
}

template <int D, int QG, int WPS>
__global__ __launch_bounds__(256, WPS) void attn_fwd_kernel(FwdArgs a) {
  constexpr int KT = D == 256 ? 32 : 64;  // keys per tile
  constexpr int NU = KT / 32;             // units per tile
  constexpr int KS = D / 16;              // k-steps over d
  constexpr int NDB = D / 32;             // 32-row blocks of d in O^T
  constexpr int NP = 2 * NDB;             // PV steps per unit
  constexpr int CPR = D / 8;              // 16-byte chunks per row
  constexpr int PARTS = KT * CPR / 256;   // direct copies per thread for one tile
  constexpr int VBUF = NU == 1 ? 4 : 3;
  constexpr int TILE = KT * D * 2;        // bytes
  constexpr int QROWS = 128 * QG;
  constexpr bool kQAgpr = D == 256;
  __shared__ __attribute__((aligned(1024))) FwdSmem<D, KT, VBUF> sm;

  const int tid = threadIdx.x, l = tid & 63, g = l >> 5, lc = l & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.n;
  const int nqb = (N + QROWS - 1) / QROWS;
  // Workgroup -> (head, query block).  Consecutive workgroups go to the 8
  // XCDs in turn; each XCD takes a contiguous run of the head-major order, so
  // that the workgroups sharing an XCD's L2 read the same K and V.
  const int items = nqb * a.bh;
  const int per = (items + 7) >> 3;
  const int item = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || item >= items) return;
  const int bh = item / nqb;
  int qb_i = item % nqb;
  // causal: the longest query blocks (last rows) first; where a run ends inside
  // a head, long and short ones alternate instead so that every run holds the
  // same work
  if (a.causal) qb_i = (a.bh & 7) == 0 ? nqb - 1 - qb_i : (qb_i & 1) ? qb_i >> 1 : nqb - 1 - (qb_i >> 1);
  const int q0 = qb_i * QROWS, q0w = q0 + 32 * QG * w;
  const size_t head = (size_t)bh * N * D;
  const uint32_t hbytes = (uint32_t)((size_t)N * D * 2);
  const auto rq = make_rsrc((const __bf16*)a.q + head, hbytes);
  const auto rk = make_rsrc((const __bf16*)a.k + head, hbytes);
  const auto rv = make_rsrc((const __bf16*)a.v + head, hbytes);
  const float c2 = a.scale * kLog2e;

  // ---- tiles: K into k[t % 2], V into v[t % VBUF]
  const uint32_t k_lds = lds_base(&sm.k[0][0]), v_lds = lds_base(&sm.v[0][0]);
  auto load_tile = [&](int t) {
    const int r = tid / CPR;
    const uint32_t kb = k_lds + (uint32_t)(t & 1) * TILE + 1024u * w;
    const uint32_t vb = v_lds + (uint32_t)(t % VBUF) * TILE + 1024u * w;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
      const int row = r + p * (256 / CPR);
      const int c = (tid % CPR) ^ tile_swz<D>(row);
      dma16_pair(rk, rv, kb + 4096u * p, vb + 4096u * p, (uint32_t)((t * KT + row) * D + 8 * c) * 2, 0);
    }
  };
  const int kv_end = a.causal ? min(N, q0 + QROWS) : N;
  const int nt = (kv_end + KT - 1) / KT;                                // tiles of the workgroup
  // units of this wave (rows past N: one, which nothing reads)
  const int nu = q0w >= N ? 1 : ((a.causal ? min(N, q0w + 32 * QG) : N) + 31) / 32;
  load_tile(0);

  // Q of this wave's rows: the B operand of S^T
  bf16x8 qreg[QG][KS];
#pragma unroll
  for (int qg = 0; qg < QG; ++qg)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qreg[qg][ks] = as_bf16x8(ld16(rq, (uint32_t)((q0w + 32 * qg + lc) * D + 16 * ks + 8 * g) * 2));

  f32x16 oacc[QG][NDB];
#pragma unroll
  for (int qg = 0; qg < QG; ++qg)
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[qg][db][r] = 0.f;
  float m[QG], lsum[QG], mx[QG];
#pragma unroll
  for (int qg = 0; qg < QG; ++qg) m[qg] = -INFINITY, lsum[qg] = 0.f;

  // Lane bases of the operand reads.  K rows: lane l reads row 32 uu + l%32,
  // chunk (2 ks + l/32) ^ swz(l%32); V^T: rows 16 half + 4 (l/32) + (l%16)/4
  // (and 8 below), columns 32 db + 16 ((l/16)%2) + 4 (l%4).  The swizzle only
  // depends on the lane, so the step enters as an XOR of the chunk bits.
  const uint32_t k_lane = (uint32_t)(lc * D * 2 + ((g ^ tile_swz<D>(lc)) << 4));
  const int L16 = l & 15, nh = (l >> 4) & 1;
  const int vrow = 4 * g + (L16 >> 2);
  auto v_lane = [&](int e) {
    const int row = vrow + 8 * e;
    return (uint32_t)(row * D * 2 + (((2 * nh + ((L16 & 3) >> 1)) ^ tile_swz<D>(row)) << 4) + ((L16 & 1) << 3));
  };
  const uint32_t v_lane0 = v_lane(0), v_lane1 = v_lane(1);

  // K and V operand addresses of the current tiles, one register per XOR value
  // (moved once per tile); units and row halves are instruction offsets.
  uint32_t ka[KS], va[2][NDB];
  auto k_tile = [&](int t) {
    const uint32_t base = k_lds + (uint32_t)(t & 1) * TILE;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      ka[ks] = base + (k_lane ^ (uint32_t)(ks << 5));
      asm volatile("" : "+v"(ka[ks]));  // not to be rebuilt at each read
    }
  };
  auto v_tile = [&](uint32_t base) {
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      va[0][db] = base + (v_lane0 ^ (uint32_t)(db << 6));
      va[1][db] = base + (v_lane1 ^ (uint32_t)(db << 6));
      asm volatile("" : "+v"(va[0][db]), "+v"(va[1][db]));
    }
  };
  auto v_base = [&](int t) { return v_lds + (uint32_t)(t % VBUF) * TILE; };

  constexpr int KRING = 4, VRING = 4;
  bf16x8 kr[KRING], vr[VRING];
  auto rd_k = [&](int uu, int ks) { kr[ks % KRING] = lds_b128(ka[ks] + (uint32_t)(uu * 32 * D * 2)); };
  auto rd_v = [&](int uu, int p) {  // operand p: half p / NDB of the unit's keys, d block p % NDB
    const uint32_t at = (uint32_t)((32 * uu + 16 * (p / NDB)) * D * 2);
    vr[p % VRING] = as_bf16x8(lds_tr(va[0][p % NDB] + at), lds_tr(va[1][p % NDB] + at));
  };

  f32x16 s[2][QG];  // scores (then P) of the current unit and the next one
  u32x4 pb[QG][2];  // P^T of the current unit, packed
  float rs[QG];

  // exp slot i of KS for group qg: P = 2^(S c2 - m) of 16 / KS elements; the
  // elements of the slot before are packed by twos (a slot late: a conversion
  // right behind its exponential would wait for it).  The empty asm keeps the
  // exponentials here, beside the score MFMAs (the compiler would sink them
  // into phase B, where P is used).
  auto pack_pair = [&](f32x16(&sc)[QG], int qg, int r) {  // elements r, r + 1
    unsigned x = pack_bf16(sc[qg][r], sc[qg][r + 1]);
    asm volatile("" : "+v"(x));
    pb[qg][r >> 3][(r & 7) >> 1] = x;
  };
  auto exp_slot = [&](f32x16(&sc)[QG], int qg, int i) {
    constexpr int E = 16 / KS;
#pragma unroll
    for (int r = i * E; r < (i + 1) * E; ++r) sc[qg][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[qg][r], c2, -m[qg]));
#pragma unroll
    for (int r = i * E - E; r < i * E; ++r)
      if (r > 0 && (r & 1)) pack_pair(sc, qg, r - 1);
    if (i == KS - 1)
#pragma unroll
      for (int r = i * E; r < 16; ++r)
        if (r & 1) pack_pair(sc, qg, r - 1);
  };
  // S^T of unit uu of the current K tile (K operands 0 .. KRING-2 already
  // requested).  A wave's VALU work overlaps its MFMAs only where it stands
  // between two of them, so every MFMA is followed by its share.
  auto qk = [&](f32x16(&sn)[QG], int uu, auto&& extra) {
#pragma unroll
    for (int qg = 0; qg < QG; ++qg)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if constexpr (!kQAgpr) sn[qg][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + KRING - 1 < KS) rd_k(uu, ks + KRING - 1);
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!kQAgpr) sn[qg] = mfma32(kr[ks % KRING], qreg[qg][ks], sn[qg]);
        else if (ks == 0) mfma32_qa<true>(kr[0], qreg[qg][0], sn[qg]);
        else mfma32_qa<false>(kr[ks % KRING], qreg[qg][ks], sn[qg]);
        __builtin_amdgcn_sched_barrier(0);
        extra(ks, qg);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // O^T += V^T P^T of unit uu of the current V tile (V operands 0 .. VRING-2 already requested)
  auto pv = [&](int uu, auto&& extra) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p + VRING - 1 < NP) rd_v(uu, p + VRING - 1);
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) {
        __builtin_amdgcn_sched_barrier(0);
        oacc[qg][p % NDB] = mfma32(vr[p % VRING], __builtin_bit_cast(bf16x8, pb[qg][p / NDB]), oacc[qg][p % NDB]);
        __builtin_amdgcn_sched_barrier(0);
        extra(p, qg);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto pre_k = [&](int uu) {
#pragma unroll
    for (int ks = 0; ks < KRING - 1; ++ks) rd_k(uu, ks);
  };
  auto pre_v = [&](int uu) {
#pragma unroll
    for (int p = 0; p < VRING - 1; ++p) rd_v(uu, p);
  };
  // element (qg, r) of unit u <-> key 32u + 8(r/4) + 4g + r%4, query q0w + 32qg + lc
  auto mask = [&](f32x16(&sc)[QG], int u) {
    if (!(32 * u + 32 > N || (a.causal && 32 * u + 31 > q0w))) return;
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) {
      if constexpr (kQAgpr) score_settle(sc[qg]);
      const int lim = (a.causal ? min(N - 1, q0w + 32 * qg + lc) : N - 1) - 32 * u - 4 * g;  // last visible key
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + (r & 3) > lim) sc[qg][r] = -INFINITY;
    }
  };
  // Maximum of a unit's scores in 4 pieces.  The first two elements are
  // compared in plain code: the compiler waits for the score MFMAs there (or
  // score_settle does), before the asm of max3 (which it does not see into) reads the others.
  auto max_piece = [&](f32x16(&sc)[QG], int qg, int i) {
    if (i == 0) {
      if constexpr (kQAgpr) score_settle(sc[qg]);
      mx[qg] = fmaxf(sc[qg][14], sc[qg][15]);
      mx[qg] = max3(mx[qg], sc[qg][0], sc[qg][1]);
    } else {
#pragma unroll
      for (int r = 4 * i - 2; r < 4 * i + 2; r += 2) mx[qg] = max3(mx[qg], sc[qg][r], sc[qg][r + 1]);
    }
    if (i == 3) mx[qg] = half_max(mx[qg]) * c2;
  };
  // row sum of a unit's P (this lane half) in 4 pieces, added to the running sum
  auto sum_piece = [&](f32x16(&sc)[QG], int qg, int i) {
    const float q = (sc[qg][4 * i] + sc[qg][4 * i + 1]) + (sc[qg][4 * i + 2] + sc[qg][4 * i + 3]);
    rs[qg] = i == 0 ? q : rs[qg] + q;
    if (i == 3) lsum[qg] += rs[qg];
  };
  // The running maximum of a row moves whenever a unit exceeds it, and O^T is
  // rescaled then (skipped when no row of the wave moves).  Moving it only
  // after a rise by 2^8, as fp32 sums would allow, saves 4-6% of the time but
  // costs accuracy: with the row's maximum at exactly 1 the large P lie just
  // below a power of two, where bf16 is most precise (O's error against 64
  // bits at N = 8192, d = 128, causal: 2.06e-3, and 2.15e-3 with lazy moves).
  auto rescale = [&]() {
    bool any = false;
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) any |= mx[qg] > m[qg];
    if (!__any(any)) return;
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) {
      const bool need = mx[qg] > m[qg];
      const float alpha = need ? __builtin_amdgcn_exp2f(m[qg] - mx[qg]) : 1.f;
      m[qg] = need ? mx[qg] : m[qg];
      lsum[qg] *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[qg][db][r] *= alpha;
    }
  };

  // The pipeline.  Steady state of unit u (its scores masked and their maximum
  // taken): phase A computes unit u+1's scores beside unit u's exp; phase B
  // sums O^T of unit u beside unit u's row sum and unit u+1's maximum.
  // Tile t is published (its copies waited for, then a barrier) half a unit
  // before its first scores are computed, after every wave has read tile
  // t - 1's K for the last time; then tile t+1 is requested into the buffers
  // that nobody reads any more.
  auto publish = [&](int t) {
    if (t >= nt) return;
    vm_wait<0>();
    __syncthreads();
    if (t + 1 < nt) load_tile(t + 1);
  };
  // phase B's VALU work: 8 QG pieces spread over its NP QG slots
  auto b_slot = [&](f32x16(&sc)[QG], f32x16(&sn)[QG], int slot, bool next) {
#pragma unroll
    for (int j = 0; j < 8 * QG; ++j) {
      if (j * NP / 8 != slot) continue;
      if (j < 4 * QG) sum_piece(sc, j >> 2, j & 3);
      else if (next) max_piece(sn, (j - 4 * QG) >> 2, j & 3);
    }
  };
  int published = 0;  // tiles 0 .. published have been published
  // one steady unit: u = its index, uu = its place in a pair of units
  auto steady = [&](int u, auto uu_c, f32x16(&sc)[QG], f32x16(&sn)[QG]) {
    constexpr int uu = decltype(uu_c)::value;
    // phase A: scores of unit u+1 (K operands requested) beside exp of unit u
    if (NU == 1 || uu == 0) v_tile(v_base(u / NU));
    qk(sn, NU == 1 ? 0 : uu ^ 1, [&](int ks, int qg) {
      exp_slot(sc, qg, ks);
      if (qg == QG - 1 && ks >= KS - VRING + 1) rd_v(NU == 1 ? 0 : uu, ks - (KS - VRING + 1));
    });
    mask(sn, u + 1);
    if (NU == 1 || uu == 0) {
      published = NU == 1 ? u + 2 : u / NU + 1;
      publish(published);
      k_tile(published);
    }
    // phase B: O^T of unit u beside its row sum and unit u+1's maximum
    pv(NU == 1 ? 0 : uu, [&](int p, int qg) {
      b_slot(sc, sn, p * QG + qg, true);
      if (qg == QG - 1 && p >= NP - KRING + 1) rd_k(NU == 1 ? 0 : uu, p - (NP - KRING + 1));
    });
    rescale();
  };

  // ---- first unit: scores, maximum
  publish(0);
  k_tile(0);
  pre_k(0);
  qk(s[0], 0, [](int, int) {});
  mask(s[0], 0);
#pragma unroll
  for (int qg = 0; qg < QG; ++qg)
#pragma unroll
    for (int i = 0; i < 4; ++i) max_piece(s[0], qg, i);
  rescale();
  // a row's maximum only rises: where it starts and where it ends say whether it
  // was ever far from 0 (a row of NaN scores is done as any other)
  bool far = false;
#pragma unroll
  for (int qg = 0; qg < QG; ++qg) far |= !(m[qg] > -kFarMax) && mx[qg] == mx[qg];
  const bool far_first = __any(far);
  if (NU == 1) {
    published = 1;
    publish(1);
    k_tile(1);
    pre_k(0);
  } else {
    pre_k(1);
  }

  int u = 0;
  using E_ = std::integral_constant<int, 0>;
  using O_ = std::integral_constant<int, 1>;
  for (; u + 2 < nu; u += 2) {
    steady(u, E_{}, s[0], s[1]);
    steady(u + 1, O_{}, s[1], s[0]);
  }
  if (u + 1 < nu) {
    steady(u, E_{}, s[0], s[1]);
    ++u;
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) s[0][qg] = s[1][qg];
  }
  // ---- last unit of this wave
  v_tile(v_base(u / NU) + (NU == 1 ? 0 : (uint32_t)(u & 1) * (32 * D * 2)));
  pre_v(0);
#pragma unroll
  for (int i = 0; i < KS; ++i)
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) exp_slot(s[0], qg, i);
  pv(0, [&](int p, int qg) { b_slot(s[0], s[0], p * QG + qg, false); });
  // the other waves' remaining tiles
  for (int t = published + 1; t < nt; ++t) publish(t);

#pragma unroll
  for (int qg = 0; qg < QG; ++qg) far = (qg > 0 && far) || m[qg] >= kFarMax;
  if (far_first || __any(far)) {
    for (int qg = 0; qg < QG; ++qg)
      if (q0w + 32 * qg < N) far_rows<D>(a, bh, q0w + 32 * qg);
    return;
  }

  // oacc[qg][db][r] <-> d = 32db + 8(r/4) + 4g + r%4, query q0w + 32qg + lc
  const auto ro = make_rsrc((__bf16*)a.o + head, hbytes);
  const auto rl = make_rsrc(a.lse + (size_t)bh * N, (uint32_t)N * 4);
#pragma unroll
  for (int qg = 0; qg < QG; ++qg) {
    const int qrow = q0w + 32 * qg + lc;
    const float sum = half_sum(lsum[qg]);
    const float inv = 1.f / sum;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        const f32x16& o = oacc[qg][db];
        u32x2 t = {pack_bf16(o[4 * rb] * inv, o[4 * rb + 1] * inv), pack_bf16(o[4 * rb + 2] * inv, o[4 * rb + 3] * inv)};
        st8(ro, (uint32_t)(qrow * D + 32 * db + 8 * rb + 4 * g) * 2, t);
      }
    if (g == 0) st4f(rl, (uint32_t)qrow * 4, (m[qg] + __log2f(sum)) * kLn2);
  }
}

template <int D, int QG, int WPS>
void launch_fwd(const FwdArgs& a, hipStream_t stream) {
  const long items = (long)((a.n + 128 * QG - 1) / (128 * QG)) * a.bh;
  hipLaunchKernelGGL((attn_fwd_kernel<D, QG, WPS>), dim3((unsigned)((items + 7) / 8 * 8)), dim3(256), 0, stream, a);
}

hipError_t launch_attn_fwd(const FwdArgs& a, int d, hipStream_t stream) {
  // Two query groups per wave halve the LDS reads per MFMA, but need 256-row
  // workgroups enough for two per CU, and under a causal mask leave half of a
  // diagonal workgroup's waves waiting.  At d = 64, full mask, 512 to 4096
  // such workgroups: 0-11% faster (16 heads of 8192: 291 against 322 us), with
  // 256 and fewer 1-33% slower, causal 3-34% slower below N = 16384.  A head of at most 128 rows
  // leaves two of the four waves without any: 600 heads of 100 13.8 us against
  // 9.1, 2048 of 128 34.2 against 29.7, 8192 of 33 61.8 against 37.1.  At d = 128 two
  // groups leave room for one wave per SIMD only: -13% to +4% at 512 workgroups
  // and more, so it is not built.
  const long wide = (long)((a.n + 255) / 256) * a.bh;
  if (d == 64) {
    if (!a.causal && a.n > 128 && wide >= 512) launch_fwd<64, 2, 2>(a, stream);
    else launch_fwd<64, 1, 3>(a, stream);
  } else if (d == 128) {
    launch_fwd<128, 1, 2>(a, stream);
  } else {
    launch_fwd<256, 1, 1>(a, stream);
  }
  return hipGetLastError();
}

}  // namespace dash
