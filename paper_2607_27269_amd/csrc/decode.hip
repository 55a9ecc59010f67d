// Decoding with the reconstructed MLA block in absorbed form (one query token per sequence).
//
// The cache keeps, per token, the latent c^KV_j and the rotated positional key k^PE_j
// (Eq. 5; the [c^KV | k^PE] rows the student forward produces).  With a single positional
// key (G_r = 1) every head attends against the same cache row [c_j ; k^PE_j]: head i uses
// the absorbed query [W_UK[g]^T q^nope_i ; q^rope_i] and its output is W_UV[g] applied to
// the attention-weighted latent (g = i / (H / G_kv)).  So decoding is multi-query attention
// with key width r_kv + d_rope, value width r_kv (the latent itself) and all H heads in one
// MFMA column block, followed by a per-group projection.
//
// Kernels (three launches: with short caches the launches are most of the time):
// * absorb_kernel: the absorbed queries [B][HP][DK] bf16 (heads padded to HP = 32k; padding
//   rows hold what scratch held before: a product column each, which has no say in the ballot
//   over the columns and is not stored), the latent part as one matrix-core product per KV group.
// * decode_attn_kernel: split-K over the cache (flash-decoding).  A workgroup (4 waves)
//   owns one (sequence, key chunk, block of 32 heads).  Key tiles of 32 rows are copied
//   straight into LDS in a ring of three stages (two tiles in flight).  The
//   tile's S^T = K Q^T (key in the MFMA row, head in the column, so each lane owns one
//   head's online-softmax state) is split over the 4 waves along the key width: each wave
//   multiplies a quarter of the 16-wide K steps (its absorbed-query fragments held in
//   registers) and the partial products are summed through
//   LDS in wave order, so every wave holds the same S^T (the same values in every wave).
//   Each wave then updates O^T += V^T P^T for its quarter of the latent width; V^T is the
//   tile's latent columns read with the transposing LDS read.  Partial (max, sum,
//   unnormalised output) per split.
// * decode_finish_kernel: merges the splits of 8 sequences of a head and applies W_UV on the
//   matrix cores.
#include <mutex>

#include "attn_common.h"
#include "kernels.h"
#include "mfma.h"
#include "mla_recon.h"

namespace mla {

// Scratch of the allocation-free decoding entry point (mla_recon_decode_noalloc): a
// file-scope device array, one copy per GPU, held until the process ends.  Host code never
// passes the array's name to a kernel (on the host it is only a stand-in symbol): it uses
// the per-device address hipGetSymbolAddress returns, obtained once per device with that
// device current.
constexpr size_t DECODE_SCRATCH_BYTES = MLA_DECODE_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) char scratch[DECODE_SCRATCH_BYTES];

constexpr int SCRATCH_MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[SCRATCH_MAX_DEVICES];

size_t decode_scratch_bytes() { return DECODE_SCRATCH_BYTES; }

hipError_t decode_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

namespace {

constexpr int DEC_KT = 32;     // keys per tile
constexpr int DEC_WAVES = 4;
constexpr float DEC_SLACK = 8.f;  // log2 units the running reference max may lag

struct DecodeDev {
  const bf16_t* qabs;   // [B][HP][DK]
  const bf16_t* cache;  // [B][Lmax][ldc]
  int64_t seq_stride;   // Lmax * ldc
  int ldc;              // row stride of the cache (elements)
  const int32_t* len;   // [B]
  int Lmax, H, HP, nsplit, chunk;
  float sl2;            // softmax scale * log2(e)
  float* part_o;        // [B][nsplit][HP][DVL]
  float* part_ml;       // [B][nsplit][HP][2]
};

// The absorbed queries of the heads of group g = blockIdx.z: row r = (b, j) of the
// B hpg rows is head i = g hpg + j of sequence b; qabs[b][i][c] = sum_d q[b][i][d] W_UK[g][d][c]
// for c < rkv, then the rotary part copied.  A workgroup (two wavefronts) makes 32 rows x 64
// columns; W_UK's 64 columns are staged in LDS as they lie ([d][c]) and read transposed
// (MFMA row = c), the query rows come straight from memory (MFMA column = row), so that a
// lane ends with 4 consecutive c of its row: 8-byte stores.  Bound by latency (W_UK is 1 MB at
// H = 32, r_kv = 512; one round of small workgroups), fp32 accumulation.  Measured with the
// rotary copy: 64 sequences 26 -> 9.0 us, one sequence 13.6 -> 4.1 us (a vector-ALU product and
// a copy launch before).
constexpr int ABS_LD = 96;  // LDS row stride: 4 rows of a transposing read on distinct banks
constexpr int ABS_DN = 192;
__global__ __launch_bounds__(128) void absorb_kernel(const bf16_t* __restrict__ q,
                                                     const bf16_t* __restrict__ Wuk,
                                                     bf16_t* __restrict__ qabs, int B, int H, int HP,
                                                     int hpg, int dn, int dr, int rkv) {
  __shared__ __attribute__((aligned(16))) bf16_t Ws[ABS_DN * ABS_LD];
  const int g = blockIdx.z, c0 = 64 * blockIdx.x, r0 = 32 * blockIdx.y;
  const int DK = rkv + dr, dq = dn + dr, tid = threadIdx.x;
  const int lane = tid & 63, wave = wave_id(), half = lane >> 5, col = lane & 31;
  const int dnp = (dn + 15) & ~15;  // d rounded up to the K step, zero filled
  const bf16_t* Wg = Wuk + (int64_t)g * dn * rkv + c0;
  if ((uintptr_t)Wuk % 16 == 0) {  // uniform
    for (int e = tid; e < dnp * 8; e += 128) {
      const int d = e >> 3, c = 8 * (e & 7);
      *(u32x4*)(Ws + d * ABS_LD + c) = d < dn ? *(const u32x4*)(Wg + (int64_t)d * rkv + c) : u32x4{0u, 0u, 0u, 0u};
    }
  } else {
    for (int e = tid; e < dnp * 64; e += 128) {
      const int d = e >> 6, c = e & 63;
      Ws[d * ABS_LD + c] = d < dn ? Wg[(int64_t)d * rkv + c] : (bf16_t)0;
    }
  }
  const int rows = B * hpg, rr = r0 + col, rc = min(rr, rows - 1);
  const int64_t bi = (int64_t)(rc / hpg) * H + g * hpg + rc % hpg;           // row of q
  const int64_t qi = (int64_t)(rc / hpg) * HP + g * hpg + rc % hpg;          // row of qabs
  const bf16_t* qp = q + bi * dq + 8 * half;
  bf16x8 qf[ABS_DN / 16];  // this lane's row, asked for before the staging's barrier
#pragma unroll
  for (int kk = 0; kk < ABS_DN / 16; ++kk) {
    u32x4 w = {0u, 0u, 0u, 0u};
    if (16 * kk + 8 * half < dn) w = *(const u32x4*)(qp + 16 * kk);
    qf[kk] = __builtin_bit_cast(bf16x8, w);
  }
  if (blockIdx.x == 0 && wave == 0 && rr < rows)  // rotary part: dr elements, half a row per lane
    for (int c = 8 * half; c < dr; c += 16)
      *(u32x4*)(qabs + qi * DK + rkv + c) = *(const u32x4*)(q + bi * dq + dn + c);
  __syncthreads();
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
  for (int kk = 0; kk < ABS_DN / 16; ++kk)
    if (16 * kk < dnp)  // uniform
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          lds_operand_tr(Ws, ABS_LD, 32 * wave, 16 * kk + 8 * half, 16 * kk + 8 * half + 4), qf[kk], acc,
          0, 0, 0);
  if (rr >= rows) return;
  bf16_t* out = qabs + qi * DK + c0 + 32 * wave + 4 * half;
#pragma unroll
  for (int e4 = 0; e4 < 4; ++e4)
    *(u32x2*)(out + 8 * e4) = u32x2{pack2bf(acc[4 * e4], acc[4 * e4 + 1]), pack2bf(acc[4 * e4 + 2], acc[4 * e4 + 3])};
}

template <int DK, int DVL>
__global__ __launch_bounds__(64 * DEC_WAVES) void decode_attn_kernel(DecodeDev a) {
  constexpr int LDK = attn::ld_of(DK);        // padded rows: conflict-free operand reads
  constexpr int NKK = DK / 16;
  constexpr int QMAX = (NKK + DEC_WAVES - 1) / DEC_WAVES;  // K steps per wave, at most
  constexpr int WV = DVL / DEC_WAVES;         // latent rows per wave
  constexpr int NCV = WV / 32;
  constexpr int NST = 3;                      // key-tile ring: two tiles in flight
  static_assert(DK % 16 == 0 && WV % 32 == 0, "decode shape");
  using KT = DmaTile<DEC_KT, DK, LDK, DEC_WAVES, true>;
  constexpr int D = KT::PER;                  // copies per wave per tile
  __shared__ __attribute__((aligned(1024))) bf16_t Ks[NST][KT::ALLOC];
  // partial S^T of each wave: [wave][e / 4][lane][4] (16-byte accesses, conflict-free)
  __shared__ __attribute__((aligned(16))) float Sp[DEC_WAVES][4][64][4];

  const int split = blockIdx.x, b = blockIdx.y, h0 = 32 * blockIdx.z;
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int half = lane >> 5, col = lane & 31;
  const int len = min(max(a.len[b], 0), a.Lmax);
  const int kbeg = split * a.chunk;
  const int kend = min(len, kbeg + a.chunk);
  const int64_t pbase = ((int64_t)b * a.nsplit + split) * a.HP + h0;
  // this wave's share of the K steps
  const int kk0 = wave * NKK / DEC_WAVES, kk1 = (wave + 1) * NKK / DEC_WAVES;

  const bf16_t* cs = a.cache + (int64_t)b * a.seq_stride;
  KT kt_copy;
  kt_copy.init();
  // key tile t into stage t % NST; rows past the chunk end repeat its last row (finite,
  // and given no weight below)
  auto issue = [&](int t) {
    const int k0 = kbeg + t * DEC_KT;
    if (k0 + DEC_KT <= kend) {  // full tile: uniform row base plus 32-bit lane offsets
      kt_copy.issue_s(Ks[t % NST], cs + (int64_t)k0 * a.ldc,
                      [&](int r, int c) { return r * a.ldc + c; });
    } else {
      kt_copy.issue(Ks[t % NST], [&](int r, int c) {
        return cs + (int64_t)min(k0 + r, kend - 1) * a.ldc + c;
      });
    }
  };
  const int ntile = kend > kbeg ? (kend - kbeg + DEC_KT - 1) / DEC_KT : 0;
  if (ntile > 0) issue(0);
  if (ntile > 1) issue(1);
  // this lane's head as B-operand fragments for the wave's K steps (head h0 + col,
  // k = 16 kk + 8 half + 0..7)
  bf16x8 qf[QMAX];
  {
    const bf16_t* qsrc = a.qabs + ((int64_t)b * a.HP + h0 + col) * DK + 8 * half;
#pragma unroll
    for (int j = 0; j < QMAX; ++j)
      qf[j] = kk0 + j < kk1 ? *(const bf16x8*)(qsrc + 16 * (kk0 + j)) : bf16x8{};
  }
  wait_vm<0>();
#pragma unroll
  for (int j = 0; j < QMAX; ++j) asm volatile("" : "+v"(qf[j]));
  __syncthreads();

  f32x16 acc[NCV];
#pragma unroll
  for (int c = 0; c < NCV; ++c)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[c][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  // lanes whose column has a head: the others must not move the reference of these, or their
  // roundings would depend on what scratch held before (reading a head's row there instead
  // measured 0.6% slower at 64 x 4096 rows)
  const uint64_t heads = __ballot(h0 + col < a.H);

  for (int t = 0; t < ntile; ++t) {
    const bf16_t* kt = Ks[t % NST];
    const int k0 = kbeg + t * DEC_KT;
    // the stage of tile t - 1 is free: every wave passed the barrier that ended it
    if (t + 2 < ntile) issue(t + 2);
    // S^T (32 keys x 32 heads): key = MFMA row, head = column (this lane's head: col);
    // this wave's K steps, then the four partial products summed in wave order
    f32x16 s;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int j = 0; j < QMAX; ++j)
      if (kk0 + j < kk1)
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            *(const bf16x8*)(kt + col * LDK + 16 * (kk0 + j) + 8 * half), qf[j], s, 0, 0, 0);
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4)
      *(f32x4*)Sp[wave][e4][lane] = f32x4{s[4 * e4], s[4 * e4 + 1], s[4 * e4 + 2], s[4 * e4 + 3]};
    lds_barrier();
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      f32x4 u = *(const f32x4*)Sp[0][e4][lane];
#pragma unroll
      for (int w2 = 1; w2 < DEC_WAVES; ++w2) u += *(const f32x4*)Sp[w2][e4][lane];
#pragma unroll
      for (int r = 0; r < 4; ++r) s[4 * e4 + r] = u[r];
    }
    // keys past the chunk end (last tile only; a real branch): no weight
    if (k0 + DEC_KT > kend) {
      asm volatile("");
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (k0 + 8 * (e >> 2) + 4 * half + (e & 3) >= kend) s[e] = -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[e]);
    mx = pair_max32(mx) * a.sl2;
    // lazy rescale: the reference max moves only when a block max exceeds it by more than
    // DEC_SLACK (so P <= 2^DEC_SLACK); one decision for all heads of the block,
    // wave-uniform, and the same in every wave (same S^T)
    if ((__ballot(mx > m_run + DEC_SLACK) & heads) != 0) {
      const float m_new = fmaxf(m_run, mx);
      const float corr = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));
      m_run = m_new;
      l_run *= corr;
#pragma unroll
      for (int c = 0; c < NCV; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[c][e] *= corr;
    }
    const float m_use = m_run == -INFINITY ? 0.f : m_run;
    // P^T as the B operand of O^T = V^T P^T (K-step u: keys 16u + {4h'..4h'+3, 8+4h'..})
    bf16x8 pf[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      u32x4 w;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * u + 2 * q], a.sl2, -m_use));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * u + 2 * q + 1], a.sl2, -m_use));
        l_run += p0 + p1;
        w[q] = pack2bf(p0, p1);
      }
      pf[u] = __builtin_bit_cast(bf16x8, w);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int klo = 16 * u + 4 * half;
#pragma unroll
      for (int c = 0; c < NCV; ++c)
        acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            lds_operand_tr(kt, LDK, wave * WV + 32 * c, klo, klo + 8), pf[u], acc[c], 0, 0, 0);
    }
    // tile t + 1 has landed (tile t + 2's copies may still fly) and every wave is done with
    // tile t and the partial sums
    if (t + 2 < ntile) wait_vm<D>();
    else wait_vm<0>();
    lds_barrier();
  }

  // partial state of this split: lane (head col, half) holds rows
  // wave WV + 32 c + 8 (e / 4) + 4 half + e % 4 of the unnormalised latent output
  const float l = pair_sum32(l_run);
  if (h0 + col >= a.H) return;  // a column without a head
  const int64_t hrow = pbase + col;
  if (wave == 0 && half == 0) {
    a.part_ml[2 * hrow] = m_run;
    a.part_ml[2 * hrow + 1] = l;
  }
  float* po = a.part_o + hrow * DVL + wave * WV + 4 * half;
#pragma unroll
  for (int c = 0; c < NCV; ++c)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *(f32x4*)(po + 32 * c + 8 * g) =
          f32x4{acc[c][4 * g], acc[c][4 * g + 1], acc[c][4 * g + 2], acc[c][4 * g + 3]};
}

// The splits of a (sequence, head) merged, then W_UV: lat[d] = sum_s o_s[d] 2^(m_s - M) /
// sum_s l_s 2^(m_s - M), rounded to bf16, and o[b][i][e] = sum_d W_UV[g][e][d] lat[d].  A
// workgroup owns head i and FIN_RB sequences.  Its wavefronts first ask for their W_UV rows
// (kept in registers: the merge hides their latency), then the maxima and sums of the splits
// go over the lanes of a wavefront per sequence, and DVL / 4 threads (each four columns) times
// 1024 / DVL slots (each every so-many-th split) sum the partials, slots in order.  The product
// runs on 16 x 16 x 32 steps with W_UV in the MFMA row.  Bound by latency; the merge reads
// the partials once.  Measured: one sequence of 6000 rows (47 splits) 49 -> 9.6 us, 64 of
// 4096 rows 19.6 -> 12.2 us (a merge that walked the splits one by one in every thread, and a
// launch for the product, before).
constexpr int FIN_RB = 8;
template <int DVL, int DV>
__global__ __launch_bounds__(256) void decode_finish_kernel(const float* __restrict__ part_o,
                                                            const float* __restrict__ part_ml,
                                                            const bf16_t* __restrict__ Wuv,
                                                            bf16_t* __restrict__ o, int B, int H, int HP,
                                                            int nsplit, int hpg) {
  constexpr int NCG = DVL / 4, NSLOT = 256 / NCG, NK = DVL / 32, NT = DV / 64, LDL = DVL + 8;
  __shared__ float red[FIN_RB][NSLOT][DVL];
  __shared__ __attribute__((aligned(16))) bf16_t lat[FIN_RB * LDL];
  __shared__ float sM[FIN_RB], sInv[FIN_RB];
  const int i = blockIdx.x, b0 = FIN_RB * blockIdx.y, nb = min(FIN_RB, B - b0);
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  // W_UV rows 16 (NT wave + t) + lane % 16, k = 32 kk + 8 (lane / 16) + 0..7
  bf16x8 wf[NT][NK];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const bf16_t* wp = Wuv + ((int64_t)(i / hpg) * DV + 16 * (NT * wave + t) + (lane & 15)) * DVL + 8 * (lane >> 4);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) wf[t][kk] = *(const bf16x8*)(wp + 32 * kk);
  }
  // maxima and sums, a wavefront per FIN_RB / 4 sequences side by side; a lane takes every
  // 64th split (its running sum rescaled as its maximum grows)
  {
    float M[FIN_RB / 4], L[FIN_RB / 4];
#pragma unroll
    for (int u = 0; u < FIN_RB / 4; ++u) {
      M[u] = -INFINITY;
      L[u] = 0.f;
    }
    for (int sp = lane; sp < nsplit; sp += 64) {
#pragma unroll
      for (int u = 0; u < FIN_RB / 4; ++u) {
        const int bb = min(wave + 4 * u, nb - 1);
        const f32x2 ml = *(const f32x2*)(part_ml + 2 * (((int64_t)(b0 + bb) * nsplit + sp) * HP + i));
        if (ml[0] != -INFINITY) {
          const float m1 = fmaxf(M[u], ml[0]);
          L[u] = L[u] * __builtin_amdgcn_exp2f(M[u] - m1) + ml[1] * __builtin_amdgcn_exp2f(ml[0] - m1);
          M[u] = m1;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < FIN_RB / 4; ++u) {
      const float Mw = warp_max(M[u]);
      const float Lw = warp_sum(M[u] == -INFINITY ? L[u] : L[u] * __builtin_amdgcn_exp2f(M[u] - Mw));
      if (lane == 0 && wave + 4 * u < nb) {
        sM[wave + 4 * u] = Mw;
        sInv[wave + 4 * u] = Lw > 0.f ? 1.f / Lw : 0.f;
      }
    }
  }
  __syncthreads();
  const int cg = tid % NCG, slot = tid / NCG;
  const float* pol = part_o + 4 * cg;
  if (nsplit <= 8 * NSLOT) {
    // few splits: the sequences' loads of one split together
    f32x4 v[FIN_RB];
#pragma unroll
    for (int bb = 0; bb < FIN_RB; ++bb) v[bb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int sp = slot; sp < nsplit; sp += NSLOT) {
      f32x4 x[FIN_RB];
      float m[FIN_RB];
#pragma unroll
      for (int bb = 0; bb < FIN_RB; ++bb) {
        const int64_t rw = ((int64_t)(b0 + min(bb, nb - 1)) * nsplit + sp) * HP + i;
        x[bb] = *(const f32x4*)(pol + rw * DVL);
        m[bb] = part_ml[2 * rw];
      }
#pragma unroll
      for (int bb = 0; bb < FIN_RB; ++bb)
        if (m[bb] != -INFINITY)  // (an empty split adds nothing)
          v[bb] += x[bb] * __builtin_amdgcn_exp2f(m[bb] - sM[min(bb, nb - 1)]);
    }
#pragma unroll
    for (int bb = 0; bb < FIN_RB; ++bb) *(f32x4*)&red[bb][slot][4 * cg] = v[bb];
  } else {
    // many splits: eight of a sequence's together
    for (int bb = 0; bb < nb; ++bb) {
      const int64_t row0 = (int64_t)(b0 + bb) * nsplit * HP + i;
      const float M = sM[bb];
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      for (int s0 = slot; s0 < nsplit; s0 += 8 * NSLOT) {
        f32x4 x[8];
        float m[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int64_t rw = row0 + (int64_t)HP * min(s0 + u * NSLOT, nsplit - 1);
          x[u] = *(const f32x4*)(pol + rw * DVL);
          m[u] = part_ml[2 * rw];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (m[u] != -INFINITY && s0 + u * NSLOT < nsplit) v += x[u] * __builtin_amdgcn_exp2f(m[u] - M);
      }
      *(f32x4*)&red[bb][slot][4 * cg] = v;
    }
  }
  __syncthreads();
  for (int e = tid; e < nb * NCG; e += 256) {
    const int bb = e / NCG, c = 4 * (e % NCG);
    f32x4 v = *(const f32x4*)&red[bb][0][c];
#pragma unroll
    for (int sl = 1; sl < NSLOT; ++sl) v += *(const f32x4*)&red[bb][sl][c];
    v *= sInv[bb];
    *(u32x2*)(lat + bb * LDL + c) = u32x2{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])};
  }
  __syncthreads();
  const int n = lane & 15;  // MFMA column: sequence b0 + n
  const bf16_t* lp = lat + min(n, nb - 1) * LDL + 8 * (lane >> 4);
  f32x4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const bf16x8 lf = *(const bf16x8*)(lp + 32 * kk);
#pragma unroll
    for (int t = 0; t < NT; ++t)
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[t][kk], lf, acc[t], 0, 0, 0);
  }
  if (n >= nb) return;
  // rows 4 (lane / 16) + 0..3 of each 16-row tile
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    bf16_t* op = o + ((int64_t)(b0 + n) * H + i) * DV + 16 * (NT * wave + t) + 4 * (lane >> 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) op[k] = f2bf(acc[t][k]);
  }
}

// o[r][i][e] = sum_c W_UV[g dv + e][c] lat[r][i][c] (g = i / hpg) on the matrix cores: a
// workgroup owns 32 rows of one head, each of its DV / 32 wavefronts 32 of the head's dv
// outputs; both operands are K-contiguous rows read straight from memory (16 bytes per
// lane per K step; the workgroup's wavefronts share the latent rows through L1), fp32
// accumulation over the r_kv latent dims.  bf16 output.
template <int DV>
__global__ __launch_bounds__(64 * (DV / 32)) void uv_mfma_kernel(const bf16_t* __restrict__ lat,
                                                                  const bf16_t* __restrict__ Wuv,
                                                                  bf16_t* __restrict__ o, int rows,
                                                                  int H, int rkv, int hpg) {
  const int i = blockIdx.y, r0 = 32 * blockIdx.x;
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int half = lane >> 5, col = lane & 31;
  const int r = min(r0 + col, rows - 1);
  const bf16_t* ap = lat + ((int64_t)r * H + i) * rkv + 8 * half;
  const bf16_t* bp = Wuv + ((int64_t)(i / hpg) * DV + 32 * wave + col) * rkv + 8 * half;
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  for (int k = 0; k < rkv; k += 16)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(ap + k), *(const bf16x8*)(bp + k),
                                                  acc, 0, 0, 0);
  // acc: row r0 + 8 (e / 4) + 4 half + e % 4, output column 32 wave + col
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int rr = r0 + 8 * (e >> 2) + 4 * half + (e & 3);
    if (rr < rows) o[((int64_t)rr * H + i) * DV + 32 * wave + col] = f2bf(acc[e]);
  }
}

#define MLA_DECODE_SHAPES(X) X(576, 512) X(288, 256) X(160, 128)

int decode_chunk(int Lmax, int B) {
  // at least 4 tiles per workgroup, and no more workgroups than one round on the CUs (one
  // workgroup per CU): long streams per workgroup keep its copy ring full
  int chunk = DEC_KT * 4;
  while ((int64_t)B * ((Lmax + chunk - 1) / chunk) > 256 && chunk < (1 << 20)) chunk *= 2;
  return chunk;
}

}  // namespace

bool decode_supported(int DK, int DVL) {
#define X(a_, b_) if (DK == a_ && DVL == b_) return true;
  MLA_DECODE_SHAPES(X)
#undef X
  return false;
}

// (The last term, a latent per sequence and head, is used by nothing since the merge and W_UV
// share a launch.  It stays: callers keep workspaces of this size, the call without a workspace
// holds it against its static buffer, and what that refused it refuses still.)
size_t decode_ws_bytes(int B, int H, int DK, int DVL, int Lmax) {
  const int HP = (H + 31) / 32 * 32;
  const int nsplit = (Lmax + decode_chunk(Lmax, B) - 1) / decode_chunk(Lmax, B);
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  return al((size_t)B * HP * DK * 2) + al((size_t)B * nsplit * HP * DVL * 4) +
         al((size_t)B * nsplit * HP * 2 * 4) + al((size_t)B * H * DVL * 2);
}

hipError_t decode_attention(const Decode& d, hipStream_t s) {
  const int DK = d.rkv + d.dr, DVL = d.rkv;
  if (!decode_supported(DK, DVL)) return hipErrorInvalidValue;
  const int HP = (d.H + 31) / 32 * 32;
  const int chunk = decode_chunk(d.Lmax, d.B);
  const int nsplit = (d.Lmax + chunk - 1) / chunk;
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  char* w = (char*)d.ws;
  bf16_t* qabs = (bf16_t*)w;
  w += al((size_t)d.B * HP * DK * 2);
  float* part_o = (float*)w;
  w += al((size_t)d.B * nsplit * HP * DVL * 4);
  float* part_ml = (float*)w;
  w += al((size_t)d.B * nsplit * HP * 2 * 4);

  const int G = d.H / d.hpg;
  if (d.dn > ABS_DN || d.rkv % 64) return hipErrorInvalidValue;
  prof_begin(KC_ELEM, s);
  absorb_kernel<<<dim3(d.rkv / 64, (d.B * d.hpg + 31) / 32, G), 128, 0, s>>>(
      (const bf16_t*)d.q, (const bf16_t*)d.Wuk, qabs, d.B, d.H, HP, d.hpg, d.dn, d.dr, d.rkv);
  prof_end(KC_ELEM, s, 2.0 * d.B * d.H * d.dn * d.rkv, (double)d.B * d.H * (DK + d.dn + d.dr) * 2,
           KLABEL("absorb_kernel"));

  DecodeDev a;
  a.qabs = qabs; a.cache = (const bf16_t*)d.cache; a.ldc = d.ldc;
  a.seq_stride = (int64_t)d.Lmax * d.ldc; a.len = d.len; a.Lmax = d.Lmax; a.H = d.H; a.HP = HP;
  a.nsplit = nsplit; a.chunk = chunk; a.sl2 = d.scale * attn::LOG2E;
  a.part_o = part_o; a.part_ml = part_ml;
  const dim3 grid(nsplit, d.B, HP / 32);
  // algorithmic work at full cache lengths: the cache rows once, 2 (DK + DVL) flops per
  // (head, key)
  prof_begin(KC_ATTN_FWD, s);
#define X(a_, b_) \
  if (DK == a_ && DVL == b_) decode_attn_kernel<a_, b_><<<grid, 64 * DEC_WAVES, 0, s>>>(a);
  MLA_DECODE_SHAPES(X)
#undef X
  prof_end(KC_ATTN_FWD, s, 2.0 * d.B * d.H * (double)d.Lmax * (DK + DVL),
           (double)d.B * d.Lmax * DK * 2, KLABEL("decode_attn_kernel"));
  const double fbytes = (double)d.B * nsplit * d.H * (DVL + 2) * 4 + (double)d.B * d.H * d.dv * 2;
  const dim3 fgrid(d.H, (d.B + FIN_RB - 1) / FIN_RB);
  prof_begin(KC_ELEM, s);
#define X(a_, b_)                                                                                  \
  if (DK == a_ && DVL == b_) {                                                                     \
    if (d.dv == 128)                                                                               \
      decode_finish_kernel<b_, 128><<<fgrid, 256, 0, s>>>(part_o, part_ml, (const bf16_t*)d.Wuv,   \
                                                          (bf16_t*)d.o, d.B, d.H, HP, nsplit, d.hpg); \
    else if (d.dv == 64)                                                                           \
      decode_finish_kernel<b_, 64><<<fgrid, 256, 0, s>>>(part_o, part_ml, (const bf16_t*)d.Wuv,    \
                                                         (bf16_t*)d.o, d.B, d.H, HP, nsplit, d.hpg); \
    else                                                                                           \
      return hipErrorInvalidValue;                                                                 \
  }
  MLA_DECODE_SHAPES(X)
#undef X
  prof_end(KC_ELEM, s, 2.0 * d.B * d.H * d.dv * d.rkv, fbytes, KLABEL("decode_finish_kernel"));
  return hipGetLastError();
}

hipError_t uv_project(const void* lat, const void* Wuv, void* o, int rows, int H, int rkv, int hpg,
                      int dv, hipStream_t s) {
  // o = W_UV[g] lat per head (matrix cores)
  prof_begin(KC_ELEM, s);
  const dim3 grid((rows + 31) / 32, H);
  if (dv == 128)
    uv_mfma_kernel<128><<<grid, 256, 0, s>>>((const bf16_t*)lat, (const bf16_t*)Wuv, (bf16_t*)o, rows,
                                             H, rkv, hpg);
  else if (dv == 64)
    uv_mfma_kernel<64><<<grid, 128, 0, s>>>((const bf16_t*)lat, (const bf16_t*)Wuv, (bf16_t*)o, rows,
                                            H, rkv, hpg);
  else
    return hipErrorInvalidValue;
  prof_end(KC_ELEM, s, 2.0 * rows * H * dv * rkv,
           (double)rows * H * (dv + rkv) * 2 + (double)H / hpg * dv * rkv * 2, KLABEL("uv_mfma_kernel"));
  return hipGetLastError();
}

// One wavefront per cache row: 16 bytes of the latent per lane (rkv <= 512).  Reads the
// latents once; rows are rewritten only where they are not finite.  Finite latents can have
// values beyond bf16 (a cache row past the tokens in use may hold anything): where a latent
// reaches 2^64 the row's values are read too.  (Below that it would take weights of 2^55: a
// sum has at most 512 terms.)
__global__ __launch_bounds__(256) void prefill_guard_kernel(const bf16_t* __restrict__ cache,
                                                            int64_t rows, int rkv, int dr,
                                                            bf16_t* __restrict__ keys, int nk,
                                                            int copy_pe, bf16_t* __restrict__ v,
                                                            int nv, bf16_t* __restrict__ lat_copy) {
  const int64_t row = (int64_t)blockIdx.x * 4 + wave_id();
  if (row >= rows) return;
  const int lane = threadIdx.x & 63;
  const bf16_t* src = cache + row * (rkv + dr);
  const bool in = 8 * lane < rkv;
  u32x4 w = {0u, 0u, 0u, 0u};
  if (in) w = *(const u32x4*)(src + 8 * lane);
  uint32_t top = 0u;  // the lane's largest exponent field, in place of the upper half's
#pragma unroll
  for (int q = 0; q < 4; ++q) top = max(top, max(w[q] << 16 & 0x7f800000u, w[q] & 0x7f800000u));
  bool any = __ballot(top == 0x7f800000u) != 0;  // wave-uniform
  if (!any && v && __ballot(top >= (127u + 64u) << 23) != 0) {
    bool bad = false;
    for (int c = lane; c < nv; c += 64) bad |= (v[row * nv + c] & 0x7f80u) == 0x7f80u;
    any = __ballot(bad) != 0;
  }
  if (lat_copy && in) *(u32x4*)(lat_copy + row * rkv + 8 * lane) = any ? u32x4{0u, 0u, 0u, 0u} : w;
  if (copy_pe)
    for (int c = lane; c < nk; c += 64) keys[row * nk + c] = any ? (bf16_t)0x7fc0 : src[rkv + c];
  if (!any) return;
  if (!copy_pe)
    for (int c = lane; c < nk; c += 64) keys[row * nk + c] = (bf16_t)0x7fc0;
  if (v)
    for (int c = lane; c < nv; c += 64) v[row * nv + c] = (bf16_t)0;
}

hipError_t prefill_guard(const void* cache, int64_t rows, int rkv, int dr, void* keys, int nk,
                         bool copy_pe, void* v, int nv, void* lat_copy, hipStream_t s) {
  if (rkv > 512 || rkv % 8 || (copy_pe && nk != dr)) return hipErrorInvalidValue;
  prof_begin(KC_ELEM, s);
  prefill_guard_kernel<<<(unsigned)((rows + 3) / 4), 256, 0, s>>>(
      (const bf16_t*)cache, rows, rkv, dr, (bf16_t*)keys, nk, copy_pe ? 1 : 0, (bf16_t*)v, nv,
      (bf16_t*)lat_copy);
  prof_end(KC_ELEM, s, 0.0, (double)rows * rkv * 2.0 * (lat_copy ? 2.0 : 1.0), KLABEL("prefill_guard_kernel"));
  return hipGetLastError();
}

}  // namespace mla
