// Phase-2 partial attention for a few dozen query tokens (Algorithm 1, Phase 2:
// the query encoding, and a host's partials of a short query).
//
// Rows.  As in decode.hip the query rows that read one KV head (token t, head
// kvh*group + h -> row t*group + h) form 32-row tiles of 32 / group tokens.  A
// wave holds RT tiles at once, so that a K/V step feeds RT * 32 rows; the
// attention kernel's workgroup would compute 64 rows of every head whatever
// the number of tokens.
//
// Work.  A workgroup is four waves, one per SIMD (the RT accumulators take
// the registers of two): NG groups of RT row tiles times KS = 4 / NG key
// sets, all of one key range of one (shard, KV head).  Key set s takes the
// 32-key steps s, s + KS, ... of the range.  The NG waves of a key set share
// its K and V steps: each moves its part of a step into one of ST LDS stages
// by loads that write LDS directly, ST - 1 steps ahead.  The key sets are
// merged through LDS at the end, so that a range leaves one (o, lse) partial.
// The generation shard of a query step (see decode.hip) rides in the same
// launch: its ranges have workgroups of their own or follow a shard's range.
//
// Step.  S^T = K Q^T with K rows and Q rows from LDS, P in the B layout of the
// PV product because LDS row r of a K step holds key swap_bits23(r); O^T += V^T
// P^T with V read transposed.  Rows sit in LDS with their 16-byte chunks
// permuted by the row, which keeps the reads free of bank conflicts.
//
// Softmax.  Log2 domain.  The fast pass takes every row's weights against its
// maximum over the wave's first step, so that a step is straight-line code;
// a workgroup that finds a sum above 2^88 (a later score far above the
// reference) repeats its range with a reference that is raised, O and the
// sums rescaled, as the scores grow.  P enters PV rounded to bf16, O is
// divided by the sum of those rounded weights, the LSE uses the fp32 sum.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "tiles.hpp"

namespace {

constexpr int PK_WAVES = 4;
constexpr int PK_KEYS = 32;  // keys per step
constexpr float PK_SLACK = 8.0f;  // log2 slack before the reference is raised

struct PackedArgs {
  const uint16_t* Q;  // bf16 [Tq, Hq, D]
  const uint16_t* K;  // bf16 [n_shards, S, Hkv, D]
  const uint16_t* V;
  int Tq, Hq, Hkv, group;
  int n_shards;
  int64_t S;
  int nparts;         // key ranges per shard (one workgroup each)
  int part_len;       // keys per range
  const uint16_t* Kg; // generation shard, bf16 [G + Tq, Hkv, D] (gen_parts > 0)
  const uint16_t* Vg;
  int G;
  int gen_parts;      // its key ranges (0: no generation shard)
  int gen_part_len;
  int gen_own;        // its ranges have workgroups of their own, after the shards'
  int tile_tokens;    // tokens per 32-row tile, 32 / group
  float scale_log2;
  float* O;           // [n_shards * nparts + gen_parts, Tq, Hq, D]
  float* lse;         // [n_shards * nparts + gen_parts, Hq, Tq]
};

// LDS: the rows of Q, then ST stages of one K and one V step per key set; at
// the end the key sets' states on their way to be merged.
template <int D, int RT, int NG>
struct PkLds {
  static constexpr int KS = PK_WAVES / NG;
  static constexpr int ST = NG == 1 ? 2 : 3;
  static constexpr int STEP = PK_KEYS * D * 2;  // bytes of a K or V step
  static constexpr int Q_BYTES = NG * RT * 32 * D * 2;
  static constexpr int LOOP = Q_BYTES + ST * KS * 2 * STEP;
  // a state is RT * D / 32 units of 16 registers and three values per tile;
  // a wave hands over the units that the other key sets of its group own
  static constexpr int UNITS = RT * (D / 32);
  static constexpr int UNIT_BYTES = 16 * 64 * 4;
  static constexpr int GIVEN = UNITS / KS * (KS - 1);
  static constexpr int SUMS = PK_WAVES * GIVEN * UNIT_BYTES;  // offset of m, l, lr
  static constexpr int MERGE = SUMS + PK_WAVES * RT * 3 * 64 * 4;
  static constexpr int BYTES = LOOP > MERGE ? LOOP : MERGE;
};

template <int D, int RT, int NG>
__global__ __launch_bounds__(64 * PK_WAVES) __attribute__((amdgpu_waves_per_eu(1, 1)))
void packed_attn_kernel(PackedArgs a) {
  using L = PkLds<D, RT, NG>;
  constexpr int KS = L::KS, ST = L::ST;
  constexpr int CPR = D / 8;       // 16-byte chunks per row
  constexpr int DS = D / 16;       // k-steps of S
  constexpr int DT = D / 32;       // 32-row tiles of O^T
  constexpr int SEGS = L::STEP / 1024 / NG;  // 1 KiB load segments of a step per wave
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave % NG, ks = wave / NG;
  const int l32 = lane & 31;
  const int g = lane >> 5;
  // workgroup -> (KV head, key range); the generation shard's ranges are
  // dealt to the first ranges of a head, or have workgroups of their own
  const int kvh = blockIdx.x % a.Hkv;
  const int z = blockIdx.x / a.Hkv;  // partial of this range
  const int tok0 = grp * RT * a.tile_tokens;  // first token of the wave's tiles
  const float c2 = a.scale_log2;
  const uint32_t row_bytes = (uint32_t)(a.Hkv * D * 2);
  const uint32_t head_off = (uint32_t)(kvh * D * 2);

  // This lane's query row of tile t: token, head, and whether it is live.
  const int tl = l32 / a.group;
  const int head = kvh * a.group + (l32 - tl * a.group);
  auto token = [&](int t) { return tok0 + t * a.tile_tokens + tl; };
  auto live = [&](int t) { return tl < a.tile_tokens && token(t) < a.Tq; };

  // ---- steps -------------------------------------------------------------
  // Chunk c of LDS row r (Q and K) sits at chunk position c ^ swz(r): 16
  // consecutive rows' chunks of one column fall in different banks.
  auto swz = [](int r) { return CPR == 16 ? (r & 15) : ((r >> 1) & 7); };
  // Keys [begin, end) of one key array, in steps of KS * 32; the last may lie
  // past the end for some key sets (loads re-read the first key; masked).
  struct Span {
    const uint16_t *k, *v;
    uint32_t bytes;
    int begin, end, nsteps;
  };
  auto make_span = [&](const uint16_t* Kz, const uint16_t* Vz, int64_t rows, int begin, int end) {
    return Span{Kz, Vz, (uint32_t)(rows * a.Hkv * D * 2), begin, end,
                max(0, (end - begin + KS * PK_KEYS - 1) / (KS * PK_KEYS))};
  };
  const int n_ranges = a.n_shards * a.nparts;
  Span span[2];
  {
    const bool has = z < n_ranges;
    const int shard = has ? z / a.nparts : 0;
    const int begin = (z - shard * a.nparts) * a.part_len;
    const int64_t off = shard * a.S * a.Hkv * D;
    span[0] = make_span(a.K + off, a.V + off, a.S, begin,
                        has ? (int)min((int64_t)begin + a.part_len, a.S) : begin);
    const int gi = a.gen_own ? z - n_ranges : z;  // range of the generation shard
    const bool has_gen = gi >= 0 && gi < a.gen_parts;
    const int gb = has_gen ? gi * a.gen_part_len : 0;
    span[1] = make_span(a.Kg, a.Vg, (int64_t)a.G + a.Tq, gb,
                        has_gen ? min(gb + a.gen_part_len, a.G + a.Tq) : 0);
  }
  // steps 0 .. n0 - 1 are the shard's, then the generation shard's
  const int n0 = span[0].nsteps, nsteps = n0 + span[1].nsteps;
  auto key0 = [&](int j) {
    return (j < n0 ? span[0].begin + j * KS * PK_KEYS : span[1].begin + (j - n0) * KS * PK_KEYS) +
           ks * PK_KEYS;
  };
  lds_u8* const stages = (lds_u8*)smem + L::Q_BYTES + ks * 2 * L::STEP;
  auto stage_of = [&](int j) { return stages + (j % ST) * (KS * 2 * L::STEP); };
  // this wave's segments of K and V step j
  auto issue = [&](int j) {
    const bool gen = j >= n0;
    const uint32_t bytes = gen ? span[1].bytes : span[0].bytes;
    const int begin = gen ? span[1].begin : span[0].begin, end = gen ? span[1].end : span[0].end;
    const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(gen ? span[1].k : span[0].k), (short)0, (int)bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(gen ? span[1].v : span[0].v), (short)0, (int)bytes, kBufferFlags);
    const uint32_t st =
        __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)stage_of(j)) + grp * 1024;
    const int k0 = key0(j);
#pragma unroll
    for (int i = 0; i < SEGS; ++i) {
      const int slot = (i * NG + grp) * 64 + lane;
      const int r = slot / CPR, c = slot % CPR;
      int kk = k0 + swap_bits23(r), kv = k0 + r;
      kk = kk < end ? kk : begin;
      kv = kv < end ? kv : begin;
      lds_dma16(kr, (uint32_t)kk * row_bytes + head_off + (uint32_t)(c ^ swz(r)) * 16u,
                st + i * NG * 1024);
      lds_dma16(vr, (uint32_t)kv * row_bytes + head_off + (uint32_t)(c ^ v_swizzle<D>(r)) * 16u,
                st + L::STEP + i * NG * 1024);
    }
  };

  // ---- Q rows into LDS: packed row (token, head) r of the workgroup ---------
  {
    constexpr int ROWS = NG * RT * 32;
    for (int i = threadIdx.x; i < ROWS * CPR; i += 64 * PK_WAVES) {
      const int r = i / CPR, c = i % CPR;
      const int rt = r & 31, rl = rt / a.group;
      const int tok = (r >> 5) * a.tile_tokens + rl;
      const int h = kvh * a.group + (rt - rl * a.group);
      u32x4 v = {0u, 0u, 0u, 0u};
      if (rl < a.tile_tokens && tok < a.Tq)
        v = *reinterpret_cast<const u32x4*>(a.Q + ((int64_t)tok * a.Hq + h) * D + 8 * c);
      *reinterpret_cast<u32x4*>(smem + (r * CPR + (c ^ swz(r))) * 16) = v;
    }
  }
  // Chunk 2s + g of row l32: the fragments of S (K as A, Q as B operand).
  uint32_t frag_off[DS];
#pragma unroll
  for (int s = 0; s < DS; ++s) frag_off[s] = (l32 * CPR + ((2 * s + g) ^ swz(l32))) * 16;
  auto frag = [&](const lds_u8* rows, int s) {
    return *reinterpret_cast<const lds_bf16x8*>(rows + frag_off[s]);
  };
  const lds_u8* const q_lds = (lds_u8*)smem + grp * RT * 32 * D * 2;
  auto q_frag = [&](int t, int s) { return frag(q_lds + t * 32 * D * 2, s); };
  uint32_t vtr_base[DT];
  v_tr_base<D>(lane, vtr_base);
  auto v_frag = [&](const lds_u8* sV, int c, int e) -> bf16x8 {
    return v_tr_read<D>(sV + vtr_base[e] + (16 * c) * (2 * D));
  };

  f32x16 acc[RT][DT];
  float m_run[RT], l_run[RT], lr_run[RT];

  // EXACT = false: every row's reference is its maximum over the wave's first
  // step.  EXACT = true: the reference is raised, with O and the sums rescaled,
  // when a step's maximum exceeds it by more than 2^8; a row that has seen no
  // key keeps -inf.
  auto run_pass = [&](auto exact_tag) {
    constexpr bool EXACT = decltype(exact_tag)::value;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
#pragma unroll
      for (int e = 0; e < DT; ++e) acc[t][e] = f32x16{};
      m_run[t] = -INFINITY;
      l_run[t] = lr_run[t] = 0.f;
    }
      // K fragments of step j, and S^T of tile t against them
      auto k_frags = [&](int j, bf16x8 (&kf)[DS]) {
        const lds_u8* sK = stage_of(j);
#pragma unroll
        for (int s = 0; s < DS; ++s) kf[s] = frag(sK, s);
      };
      auto scores = [&](const bf16x8 (&kf)[DS], int t) {
        f32x16 S = f32x16{};
#pragma unroll
        for (int s = 0; s < DS; ++s)
          S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], q_frag(t, s), S, 0, 0, 0);
        return S;
      };
      // weights of scores 2i, 2i + 1 of tile t
      auto weigh = [&](const f32x16& S, int t, int i, float m_use, bf16x2 (&P)[8]) {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        f32x2 p;
        p[0] = __builtin_amdgcn_exp2f(__builtin_fmaf(S[2 * i], c2, -m_use));
        p[1] = __builtin_amdgcn_exp2f(__builtin_fmaf(S[2 * i + 1], c2, -m_use));
        l_run[t] += p[0];
        l_run[t] += p[1];
        P[i] = __builtin_convertvector(p, bf16x2);
        lr_run[t] = __builtin_amdgcn_fdot2_f32_bf16(P[i], kOnes2, lr_run[t], false);
        // the sums are formed here: left to itself the compiler keeps every
        // weight and adds them up after the step
        asm volatile("" : "+v"(l_run[t]), "+v"(lr_run[t]));
      };
      auto p_frag = [&](const bf16x2 (&P)[8], int c) {
        return bf16x8{P[4 * c][0], P[4 * c][1], P[4 * c + 1][0], P[4 * c + 1][1],
                      P[4 * c + 2][0], P[4 * c + 2][1], P[4 * c + 3][0], P[4 * c + 3][1]};
      };
      auto v_frags = [&](int j, bf16x8 (&vf)[2][DT]) {
        const lds_u8* sV = stage_of(j) + L::STEP;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int e = 0; e < DT; ++e) vf[c][e] = v_frag(sV, c, e);
      };
      // Keys past the range's end weigh zero, in the generation shard those
      // after the row's own token too.
      auto mask = [&](int j, int t, f32x16& S) {
        const int vis_end =
            j < n0 ? span[0].end : min(span[1].end, a.G + token(t) + 1);
        const int k0 = key0(j);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = 8 * (v >> 2) + 4 * g + (v & 3);
          if (k0 + swap_bits23(row) >= vis_end) S[v] = -INFINITY;
        }
      };
      auto row_max = [&](const f32x16& S) {
        float mx = S[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, S[v]);
        return fmaxf(mx, __shfl_xor(mx, 32, 64)) * c2;
      };
      // Step j is in LDS for the waves of its key set, and everyone is done
      // with step j - 1, whose stage step j + ST - 1 takes.  A key set of one
      // wave needs no barrier (the first step's makes Q visible).
      auto arrive = [&](int j) {
        __builtin_amdgcn_sched_barrier(0);
        if (ST > 2 && j + 1 < nsteps)
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * SEGS) : "memory");
        else
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (NG > 1 || j == 0) __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
      };
      // the stages are free: a pass ends with a barrier
#pragma unroll
      for (int j = 0; j < ST - 1; ++j)
        if (j < nsteps) issue(j);
      // A step that needs no mask: the weights of tile t - 1 are formed between
      // the matrix instructions of tile t's scores, those of the last tile
      // between tile 0's PV products, the loads issued between the others.
      // (The fences keep that order.)
      auto step = [&](int j) {
        constexpr int QD = 4;  // Q fragments read ahead
        bf16x8 kf[DS], vf[2 * DT], ring[QD];
        bf16x2 P[RT][8];
        f32x16 S[2];
        const lds_u8* const sV = stage_of(j) + L::STEP;
        auto q_at = [&](int n) { return q_frag(n / DS, n % DS); };
        k_frags(j, kf);
#pragma unroll
        for (int n = 0; n < QD; ++n) ring[n] = q_at(n);
        if (j + ST - 1 < nsteps) issue(j + ST - 1);
        __builtin_amdgcn_sched_barrier(0);
        S[0] = f32x16{};
#pragma unroll
        for (int i = 0; i < DS; ++i) {
          S[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], ring[i % QD], S[0], 0, 0, 0);
          if (i + QD < RT * DS) ring[i % QD] = q_at(i + QD);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int t = 1; t <= RT; ++t) {
          f32x16 Sn = f32x16{};
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            if (t < RT && i < DS) {
              const int n = t * DS + i;
              Sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], ring[n % QD], Sn, 0, 0, 0);
              if (n + QD < RT * DS) ring[n % QD] = q_at(n + QD);
              // the last tile frees the K fragments one by one
              if (t == RT - 1) vf[i] = v_frag(sV, i / DT, i % DT);
            } else if (t == RT && i < 2 * DT) {
              const int c = i / DT, e = i % DT;
              acc[0][e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i], p_frag(P[0], c), acc[0][e],
                                                                  0, 0, 0);
            }
            weigh(S[(t - 1) & 1], t - 1, i, m_run[t - 1], P[t - 1]);
            __builtin_amdgcn_sched_barrier(0);
          }
          S[t & 1] = Sn;
        }
#pragma unroll
        for (int t = 1; t < RT; ++t)
#pragma unroll
          for (int i = 0; i < 2 * DT; ++i)
            acc[t][i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i], p_frag(P[t], i / DT),
                                                                     acc[t][i % DT], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      };
      // Any step, one tile after the other.
      auto step_edge = [&](int j) {
        bf16x8 kf[DS], vf[2][DT];
        bf16x2 P[RT][8];
        if (j + ST - 1 < nsteps) issue(j + ST - 1);
        k_frags(j, kf);
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          f32x16 S = scores(kf, t);
          mask(j, t, S);
          if (EXACT) {
            const float mx = row_max(S);
            if (__any(mx > m_run[t] + PK_SLACK)) {
              const float m_new = mx > m_run[t] + PK_SLACK ? mx : m_run[t];
              const float alpha =
                  m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run[t] - m_new);
#pragma unroll
              for (int e = 0; e < DT; ++e) acc[t][e] *= alpha;
              l_run[t] *= alpha;
              lr_run[t] *= alpha;
              m_run[t] = m_new;
            }
          }
          // a row that has seen no key yet takes its weights against 0, so
          // that they come out 0
          const float m_use = EXACT && m_run[t] == -INFINITY ? 0.f : m_run[t];
#pragma unroll
          for (int i = 0; i < 8; ++i) weigh(S, t, i, m_use, P[t]);
          __builtin_amdgcn_sched_barrier(0);
        }
        v_frags(j, vf);
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
          for (int i = 0; i < 2 * DT; ++i) {
            const int c = i / DT, e = i % DT;
            acc[t][e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[c][e], p_frag(P[t], c), acc[t][e],
                                                                0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
      };
      arrive(0);
      int j = 0;
      if (!EXACT) {
        // the references, then all steps of the shard but the last unmasked
        bf16x8 kf[DS];
        k_frags(0, kf);
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          f32x16 S = scores(kf, t);
          mask(0, t, S);
          m_run[t] = row_max(S);
          __builtin_amdgcn_sched_barrier(0);
        }
        for (; j + 1 < n0; ++j) {
          step(j);
          arrive(j + 1);
        }
      }
      for (; j < nsteps; ++j) {
        step_edge(j);
        if (j + 1 < nsteps) arrive(j + 1);
      }
      __syncthreads();
  };
  // Every weight is at most the sum, so a sum below 2^88 bounds them all; a
  // workgroup with a larger one runs the exact pass, as does one that has no
  // step of a shard for every wave to take its references from.
  bool redo = span[0].end - span[0].begin <= (KS - 1) * PK_KEYS;
  if (!redo) {
    run_pass(std::false_type{});
    bool over = false;
#pragma unroll
    for (int t = 0; t < RT; ++t) over |= !(lr_run[t] <= 0x1p88f);
    int* const flag = reinterpret_cast<int*>(smem + L::Q_BYTES);  // of each wave
    if (lane == 0) flag[wave] = 0;
    if (__any(over) && lane == 0) flag[wave] = 1;
    __syncthreads();
    for (int w = 0; w < PK_WAVES; ++w) redo |= flag[w] != 0;
    __syncthreads();
  }
  if (redo) run_pass(std::true_type{});

  // ---- merge of the key sets ------------------------------------------------
  // Unit u = t * DT + e of a group's state (registers acc[t][e]) is merged,
  // normalised and written by key set u % KS; the others hand it over.
  {
    float* const units = reinterpret_cast<float*>(smem) + lane * 4;
    float* const sums = reinterpret_cast<float*>(smem + L::SUMS) + lane;
    auto unit_at = [&](int src, int u) {  // unit u, handed over by key set src
      const int owner = u % KS;
      const int i = (u / KS) * (KS - 1) + (owner < src ? owner : owner - 1);
      return units + ((src * NG + grp) * L::GIVEN + i) * (L::UNIT_BYTES / 4);
    };
    auto sum_at = [&](int src, int t, int k) {
      return sums + (((src * NG + grp) * RT + t) * 3 + k) * 64;
    };
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      // each row's two lanes hold the sums of half its keys
      l_run[t] += __shfl_xor(l_run[t], 32, 64);
      lr_run[t] += __shfl_xor(lr_run[t], 32, 64);
      *sum_at(ks, t, 0) = m_run[t];
      *sum_at(ks, t, 1) = l_run[t];
      *sum_at(ks, t, 2) = lr_run[t];
#pragma unroll
      for (int e = 0; e < DT; ++e) {
        __builtin_amdgcn_sched_barrier(0);
        if ((t * DT + e) % KS == ks) continue;
        float* const dst = unit_at(ks, t * DT + e);
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          *reinterpret_cast<f32x4*>(dst + q4 * 256) =
              f32x4{acc[t][e][4 * q4], acc[t][e][4 * q4 + 1], acc[t][e][4 * q4 + 2],
                    acc[t][e][4 * q4 + 3]};
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      float m = -INFINITY, l = 0.f, lr = 0.f, w[KS];
#pragma unroll
      for (int k = 0; k < KS; ++k) m = fmaxf(m, *sum_at(k, t, 0));
      const float use = m == -INFINITY ? 0.f : m;
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        w[k] = __builtin_amdgcn_exp2f(*sum_at(k, t, 0) - use);
        l += w[k] * *sum_at(k, t, 1);
        lr += w[k] * *sum_at(k, t, 2);
      }
      const float inv = lr > 0.f ? 1.f / lr : 0.f;
      const float w_own = __builtin_amdgcn_exp2f(m_run[t] - use) * inv;
      const int tok = token(t);
#pragma unroll
      for (int e = 0; e < DT; ++e) {
        if ((t * DT + e) % KS != ks) continue;
        f32x16 o = acc[t][e] * w_own;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
          __builtin_amdgcn_sched_barrier(0);
          if (k == ks) continue;
          const float* const src = unit_at(k, t * DT + e);
          const float wk = w[k] * inv;
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(src + q4 * 256);
#pragma unroll
            for (int i = 0; i < 4; ++i) o[4 * q4 + i] += x[i] * wk;
          }
        }
        if (live(t)) {
          float* const dst = a.O + (int64_t)z * a.Tq * a.Hq * D + ((int64_t)tok * a.Hq + head) * D;
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
            *reinterpret_cast<f32x4*>(dst + e * 32 + 8 * q4 + 4 * g) =
                f32x4{o[4 * q4], o[4 * q4 + 1], o[4 * q4 + 2], o[4 * q4 + 3]};
        }
      }
      if (ks == 0 && g == 0 && live(t))
        a.lse[(int64_t)z * a.Hq * a.Tq + (int64_t)head * a.Tq + tok] =
            l > 0.f ? (m + __log2f(l)) * 0.69314718055994531f : -INFINITY;
    }
  }
}

template <int D, int RT, int NG>
int launch_packed_impl(const PackedArgs& a, int64_t nwg, hipStream_t stream) {
  constexpr int lds = PkLds<D, RT, NG>::BYTES;
  static_assert(lds <= PULSAR_LDS_BYTES, "one workgroup per compute unit");
  const auto kern = packed_attn_kernel<D, RT, NG>;
  if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) !=
      hipSuccess)
    return PULSAR_EHIP;
  hipLaunchKernelGGL(kern, dim3((unsigned)nwg), dim3(64 * PK_WAVES), lds, stream, a);
  return hipGetLastError() == hipSuccess ? PULSAR_OK : PULSAR_EHIP;
}

template <int D>
int launch_packed_d(const PackedArgs& a, int tiles, int64_t nwg, hipStream_t stream) {
  switch (tiles) {
    case 1:
    case 2: return launch_packed_impl<D, 2, 1>(a, nwg, stream);
    case 3:
    case 4: return launch_packed_impl<D, 2, 2>(a, nwg, stream);
    case 5:
    case 6:
      if constexpr (D == 64) return launch_packed_impl<D, 3, 2>(a, nwg, stream);
      else return PULSAR_EUNSUPPORTED;
    default: return PULSAR_EUNSUPPORTED;
  }
}

}  // namespace

// Up to four row tiles at d = 128 and six at d = 64, where the step of a wave
// holds two (three) tiles.  At 8 shards of 4096 keys, 32 / 8 heads of 128, the
// attention kernel against this one, launches and merge: 2 tiles 47.5 / 31.0
// us, 4 tiles 50.0 / 38.5 us (16 x 8192 keys: 138 / 104 and 144 / 121 us); with
// three tiles per wave 5 tiles take 52.8 / 56 us, 6 tiles at 16 x 8192 keys
// 160 / 168 us: their accumulators fill the registers.  At d = 64, 5 x 3000
// keys of 16 heads, 2 tiles: 46.5 / 19.2 us; 16 x 2000, 16 / 8 heads, 4 tiles:
// 38.4 / 27.9 us; a query step of 6 tiles, 16 / 4 heads, 8 x 4096 keys 33.5 /
// 25.4, 16 / 16 heads, 16 x 8192 185 / 181 (partials alone: packed_partial in
// api.hip).
int packed_tokens(int Hq, int Hkv, int d) {
  const int group = Hq / Hkv, tiles = d == 64 ? 6 : 4;
  return (d == 64 || d == 128) && group >= 1 && group <= 32 ? tiles * (32 / group) : 0;
}

bool packed_applies(int Tq, int Hq, int Hkv, int d) {
  return Tq >= 1 && Tq <= packed_tokens(Hq, Hkv, d);
}

// Keys per range when S keys are cut into nparts ranges of whole steps of all
// four waves.
static int packed_part_len(int64_t S, int nparts) {
  const int64_t len = (S + nparts - 1) / nparts;
  constexpr int unit = PK_KEYS * PK_WAVES;
  return (int)((len + unit - 1) / unit * unit);
}

// Key ranges per shard: the most that still give one workgroup per compute
// unit in one round, at least min_keys keys each.
int packed_parts(int n_shards, int64_t S, int Hkv, int min_keys) {
  if (S <= 0 || n_shards <= 0 || Hkv <= 0) return 1;
  const int64_t wgs = (int64_t)n_shards * Hkv;
  const int64_t np = std::max<int64_t>(
      std::min<int64_t>(256 / wgs, (S + min_keys - 1) / min_keys), 1);
  return packed_ranges(S, (int)np);
}

// The ranges that `nparts` come to in whole steps.
int packed_ranges(int64_t S, int nparts) {
  const int64_t len = packed_part_len(S, nparts);
  return (int)((S + len - 1) / len);
}

// Row tiles of a KV head.
int packed_tiles(int Tq, int group) {
  const int tokens = 32 / group;
  return (Tq + tokens - 1) / tokens;
}

// Key ranges per shard of a call that merges them in a launch of its own: the
// number with the least of a workgroup's steps, the launch (2.7 us) and the
// partials' bytes (0.63 us a MB, written and merged), or one.  128 keys take
// 0.86, 1.6 and 2.2 us for up to two, four and six tiles at d 64, 1.4 and 2.5 us
// for up to two and four at d 128 (fitted to 3400 times of 612 shapes with up to
// 64 ranges, within 3 % on average).  16 tokens of 4 heads over 32 x 300 keys, 4
// KV heads of 64: 8.1 us in one range a shard, 11.8 in two; over 5 x 3000 keys
// 24.3 in one, 13.3 in eight.
int packed_shard_parts(int n_shards, int Tq, int64_t S, int Hq, int Hkv, int d) {
  const int most = packed_parts(n_shards, S, Hkv);
  if (most == 1) return 1;
  constexpr int unit = PK_KEYS * PK_WAVES;
  const int tiles = packed_tiles(Tq, Hq / Hkv);
  const double step = d == 64 ? (tiles <= 2 ? 0.86 : tiles <= 4 ? 1.6 : 2.2) : tiles <= 2 ? 1.4 : 2.5;
  const double mb = 0.63e-6 * n_shards * Tq * Hq * (d + 1) * 4;  // of one range a shard, in us
  const double best = std::sqrt(step * (double)S / unit / mb);
  const int np = packed_ranges(S, (int)std::min<double>(std::max(best + 0.5, 2.0), most));
  const auto steps = [&](int parts) { return step * packed_part_len(S, parts) / unit; };
  return steps(np) + 2.7 + mb * np < steps(1) ? np : 1;
}

int64_t packed_ranges_most(int n_shards, int64_t S, int Hkv, int min_keys) {
  if (S <= 0 || n_shards <= 0) return std::max(n_shards, 0);
  return std::min<int64_t>(n_shards * ((S + min_keys - 1) / min_keys),
                           std::max(256 / Hkv, n_shards));
}

int launch_packed(const uint16_t* q, const uint16_t* K, const uint16_t* V, int n_shards, int Tq,
                  int64_t S, int Hq, int Hkv, int d, float scale, float* o, float* lse,
                  int nparts, hipStream_t stream, const DecodeGen* gen) {
  PackedArgs a{};
  a.Q = q;
  a.K = K;
  a.V = V;
  a.Tq = Tq;
  a.Hq = Hq;
  a.Hkv = Hkv;
  a.group = Hq / Hkv;
  if (!packed_applies(Tq, Hq, Hkv, d)) return PULSAR_EUNSUPPORTED;
  a.n_shards = n_shards;
  a.S = S;
  a.nparts = nparts;
  a.part_len = packed_part_len(S, nparts);
  a.tile_tokens = 32 / a.group;
  if (gen != nullptr && gen->nparts > 0) {
    a.Kg = gen->K;
    a.Vg = gen->V;
    a.G = (int)gen->G;
    a.gen_parts = gen->nparts;
    a.gen_part_len = packed_part_len(gen->G + Tq, gen->nparts);
    a.gen_own = gen->own;
  }
  a.scale_log2 = scale * 1.4426950408889634f;
  a.O = o;
  a.lse = lse;
  const int64_t ranges = (int64_t)n_shards * nparts;
  if (!a.gen_own && a.gen_parts > ranges) return PULSAR_EINVAL;
  const int64_t nwg = Hkv * (ranges + (a.gen_own ? a.gen_parts : 0));
  if (nwg == 0) return PULSAR_OK;
  if (nwg > 0x7fffffff) return PULSAR_EUNSUPPORTED;
  const int tiles = packed_tiles(Tq, a.group);
  return d == 128 ? launch_packed_d<128>(a, tiles, nwg, stream)
                  : launch_packed_d<64>(a, tiles, nwg, stream);
}
