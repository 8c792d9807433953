// Grouped expert FFN with the weights stationary in registers, for bf16 at
// d_h 128 and d_ff 128 where the experts see enough slots.
//
// One workgroup of four wavefronts (two workgroups per CU) holds ONE expert's
// weights in its registers and streams the expert's clustered slots past
// them, a tile of 64 per step in two blocks of 32:
//
//   GEMM1  wavefront w owns d_ff rows 32 w .. 32 w + 31 of W1 and W3 (64
//          registers): A = W1_w X^T, B = W3_w X^T for 32 slots, the X
//          fragments read from LDS by every wavefront;
//   h      silu(A) * B (or gelu(A)) rounded to bf16, in LDS;
//   GEMM2  wavefront w contracts h with d_h rows 32 w .. + 31 of W2 (32
//          registers); the outputs are stored from the registers.
//
// Sub-step j runs GEMM1 of block j, the activation of block j - 1 and GEMM2
// of block j - 3 interleaved instruction by instruction, so that the vector
// ALU has work at every MFMA (measured on this chip: two wavefronts per SIMD
// sustain one 32x32x16 MFMA, four vector and 1.3 transcendental operations
// per 40 cycles when they alternate, and hardly overlap when one wavefront
// has only MFMAs and the other only vector work to issue).  One barrier per
// step (two sub-steps) hands h over; X rows are gathered by LDS DMA a step
// ahead.
//
// What bounds it: memory and issue together.  At 16384 tokens, 16 heads, 256
// experts, k 16 a launch takes 468 us and moves 2.42 GB by the counters (the
// gathered rows, 0.4 GB of weights, 1.07 GB of outputs), 5.2 TB/s where the
// combine's plain read reaches 6; the matrix cores are busy 42% of it, with 9
// vector operations per MFMA, and no LDS bank conflicts.  Streaming the weights
// through LDS instead (ffn_q32_kernel: an expert's weights once per 256 slots,
// a barrier and a DMA wait per 24 MFMAs) takes 619 us there; a barrier per
// sub-step with the outputs staged in LDS and stored as whole rows took 8% more
// than one barrier per step with stores of 64-byte pieces.  (At d_ff 256, with eight wavefronts and
// 16-row GEMM2 tiles, the same scheme measured no better than ffn_q32_kernel,
// which stays there.)
#include <math.h>
#include <stddef.h>

#include <type_traits>

#include "device_common.hpp"
#include "ffn_common.hpp"
#include "launch.hpp"

namespace mhl {
namespace {

// slot / k for slots below 2^31 and 1 <= k <= 32: with S = 31 + ceil(log2 k)
// and m = ceil(2^S / k) < 2^32, floor(slot m / 2^S) is exact (see div_magic);
// taken as the high word of (2 slot) m, shifted by S - 31 = ceil(log2 k).
struct SlotDiv {
  uint32_t m;
  int shift;
};
__device__ __forceinline__ uint32_t slot_token(uint32_t slot, SlotDiv d) {
  return __umulhi(slot << 1, d.m) >> d.shift;
}

struct Ws {
  static constexpr int DH = 128, DFF = 128;
  static constexpr int NW = 4, THREADS = NW * kWave;
  static constexpr int SB = 32;                        // slots per block
  static constexpr int ROW = 256;                      // bytes of an X row
  static constexpr int BLK = SB * ROW;                 // X or h of a block
  static constexpr int NSL = 8;                        // ring of slot lists
  static constexpr int STAGE = 2048;                   // a wavefront's LDS to turn weights in
  static constexpr int X_OFF = 0;                      // X of two tiles: [slot][unit ^ slot]
  static constexpr int H_OFF = X_OFF + 4 * BLK;        // h of four blocks: [16-byte unit][slot]
  static constexpr int S_OFF = H_OFF + 4 * BLK;
  static constexpr int T_OFF = S_OFF + NSL * 2 * SB * 4;
  static constexpr int TOTAL = T_OFF + NW * STAGE;
  static constexpr int RPW = 2 * SB / NW, NDMA = RPW / 4;  // X rows, DMA instructions per wavefront
  static constexpr int BLOCKS = 2;                     // workgroups per CU
  static_assert(kWsTileRows == 2 * SB && TOTAL * BLOCKS <= 160 * 1024, "LDS");
};

template <bool GELU>
__global__ __launch_bounds__(Ws::THREADS, Ws::BLOCKS) void ffn_ws_kernel(
    const uint16_t* __restrict__ X, const int32_t* __restrict__ perm,
    const TileInfo* __restrict__ tiles, const int32_t* __restrict__ shares,
    const uint16_t* __restrict__ W1, const uint16_t* __restrict__ W3,
    const uint16_t* __restrict__ W2, int64_t T, int Nh, int Ne, int k,
    uint16_t* __restrict__ yslot) {
  using L = Ws;
  constexpr int DH = L::DH, DFF = L::DFF;
  __shared__ __attribute__((aligned(16))) uint8_t smem[L::TOTAL];

  // A contiguous share of the tiles per workgroup (ws_shares_at), the shares
  // of one accelerator die next to each other (neighbours split an expert and
  // read its weights through one L2).
  const int me = (int)(blockIdx.x % kXcds) * (kWsGrid / kXcds) + (int)(blockIdx.x / kXcds);
  const int b0 = shares[me], b1 = shares[me + 1];
  if (b0 >= b1) return;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid & (kWave - 1);
  const int g = lane >> 5, c = lane & 31;  // MFMA operand: row or column c, K half g
  // A copy of the lane number that the compiler cannot hoist what is computed
  // from: keeps rarely used addresses out of the registers of the main loop.
  auto here = [&]() {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  const DivMagic kmag = div_magic(k);
  const SlotDiv kdiv{(uint32_t)kmag.m, kmag.shift - 31};
  constexpr int64_t WEXP = (int64_t)DFF * DH;

  // X fragments: slot c of the block, 16-byte unit 2 s + g, XOR-swizzled by
  // the row.  h: unit u of slot m at (32 u + m) 16 bytes.  hrd: the lane's
  // GEMM2 fragment of K step 0; hwr: the unit of d_ff rows 32 wave + 8 g.
  uint32_t off[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) off[s] = c * L::ROW + 16 * ((2 * s + g) ^ (c & 15));
  const uint32_t hrd = g * 512 + c * 16;
  const uint32_t hwr = (4 * wave + g) * 512 + c * 16;

  // The slot ids of a tile's 64 rows (rows past its end: its last one) by LDS
  // DMA, one instruction of one wavefront.  (Buffer and not global LDS DMA,
  // here and below: the compiler takes the latter for a flat access that
  // also counts as an LDS operation, and turns every later wait for an LDS
  // fragment into lgkmcnt(0).)
  const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int32_t*>(perm), 0, (int)(uint32_t)(T * k * Nh * 4), 0x00020000);
  const uint32_t head_slots = (uint32_t)(T * k);
  auto dma_slots = [&](const TileInfo& t, int n) {
    const int row = t.row_begin + here();
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        prs, (__attribute__((address_space(3))) void*)(smem + L::S_OFF + (n & (L::NSL - 1)) * 256),
        4, ((uint32_t)t.head * head_slots + (uint32_t)(row < t.row_end ? row : t.row_end - 1)) * 4,
        0, 0, 0);
  };
  auto slot_at = [&](int n, int row) {
    return *reinterpret_cast<const int*>(smem + L::S_OFF + (n & (L::NSL - 1)) * 256 + row * 4);
  };
  // X rows of a tile: DMA instruction d of the wavefront fills rows RPW wave
  // + 4 d + [0, 4) (lane / 16), physical unit lane % 16.
  auto row_slots = [&](int n, int* s) {
    const int row = L::RPW * wave + (here() >> 4);
#pragma unroll
    for (int d = 0; d < L::NDMA; ++d) s[d] = slot_at(n, row + 4 * d);
  };
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(X), 0, (int)(uint32_t)(T * Nh * (DH * 2)), 0x00020000);
  auto dma_x = [&](const TileInfo& t, const int* s, uint32_t xbase) {
    const int l = here(), row = L::RPW * wave + (l >> 4), r = l & 15;
#pragma unroll
    for (int d = 0; d < L::NDMA; ++d) {
      const uint32_t th = slot_token((uint32_t)s[d], kdiv) * (uint32_t)Nh + (uint32_t)t.head;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          xrs,
          (__attribute__((address_space(3))) void*)(smem + xbase + (L::RPW * wave + 4 * d) * L::ROW),
          16, th * (DH * 2) + 16 * (r ^ ((row + 4 * d) & 15)), 0, 0, 0);
    }
  };

  // Weights.  The wavefront's 32 rows of W1, W3 or W2 are loaded coalesced,
  // 16 rows x 64 bytes per instruction (lane: row lane / 4, unit lane % 4),
  // into the registers that will hold them, and turned into MFMA fragments
  // (lane: row c, unit 2 s + g) through 2 KiB of LDS of the wavefront's own,
  // [row][4 units] with the units XORed by bits 2-3 of the row (both sides
  // free of bank conflicts).  Loaded straight into fragments, an instruction
  // touches 32 cache lines and uses 32 bytes of each: an expert's weights
  // then took several microseconds more.
  u32x4 w1[8], w3[GELU ? 1 : 8], w2[8];
  auto load_w = [&](u32x4* w, const uint16_t* base) {
    const int l = here();
    const uint16_t* p = base + (l >> 2) * DH + 8 * (l & 3);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      w[i] = *reinterpret_cast<const u32x4*>(p + (i & 1) * 16 * DH + (i >> 1) * 32);
  };
  auto turn_w = [&](u32x4* w) {
    uint8_t* st = smem + L::T_OFF + wave * L::STAGE;
    const int l = here(), g = l >> 5, c = l & 31;
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        *reinterpret_cast<u32x4*>(st + (16 * j + (l >> 2)) * 64 + 16 * ((l & 3) ^ ((l >> 4) & 3))) =
            w[i + j];
      wave_lds_order();
#pragma unroll
      for (int j = 0; j < 2; ++j)
        w[i + j] = *reinterpret_cast<const u32x4*>(st + c * 64 + 16 * ((2 * j + g) ^ ((c >> 2) & 3)));
      wave_lds_order();
    }
  };
  auto expert_off = [&](const TileInfo& t) { return ((int64_t)t.head * Ne + t.expert) * WEXP; };
  auto weights13 = [&](const TileInfo& t) {
    const int64_t o = expert_off(t) + (int64_t)(32 * wave) * DH;
    load_w(w1, W1 + o);
    if constexpr (!GELU) load_w(w3, W3 + o);
    turn_w(w1);
    if constexpr (!GELU) turn_w(w3);
  };
  auto weights2 = [&](const TileInfo& t) {
    load_w(w2, W2 + expert_off(t) + (int64_t)(32 * wave) * DFF);
    turn_w(w2);
  };
  f32x16 A[2], B[2];        // GEMM1 of blocks of either parity
  f32x16 y;                 // GEMM2
  float u[8];
  uint32_t pk[4], ey[8];
  u32x4 xr[2], hr[2];       // fragments, two K steps ahead

  // Activation op o of block parity P: for each half hh of the 16
  // accumulator elements, stage-major, then 4 packs, and 2 swaps (lanes c
  // and c + 32 trade halves: 8 consecutive d_ff rows per lane) with one
  // 16-byte LDS write of h at hbase.
  constexpr int NE = GELU ? 8 : 48;
  constexpr int NHALF = NE + 4 + 2;
  constexpr int NACT = 2 * NHALF;
  auto act = [&](auto Pc, auto Oc, uint32_t hbase) {
    constexpr int hh = decltype(Oc)::value / NHALF, o = decltype(Oc)::value % NHALF;
    const f32x16& a = A[decltype(Pc)::value];
    const f32x16& b = B[decltype(Pc)::value];
    if constexpr (o < NE) {
      constexpr int v = o % 8, e = 8 * hh + v, st = o / 8;
      if constexpr (GELU) u[v] = gelu_logistic(a[e]);
      else if constexpr (st == 0) u[v] = -1.4426950408889634f * a[e];
      else if constexpr (st == 1) u[v] = __builtin_amdgcn_exp2f(u[v]);
      else if constexpr (st == 2) u[v] = 1.0f + u[v];
      else if constexpr (st == 3) u[v] = __builtin_amdgcn_rcpf(u[v]);
      else if constexpr (st == 4) u[v] = a[e] * u[v];
      else u[v] = u[v] * b[e];
    } else if constexpr (o < NE + 4) {
      constexpr int p = o - NE;
      pk[p] = pack_bf16x2(u[2 * p], u[2 * p + 1]);
    } else {
      constexpr int w = o - NE - 4;
      const auto x = permlane32_swap(pk[w], pk[2 + w]);
      pk[w] = x[0];
      pk[2 + w] = x[1];
      if constexpr (w == 1)
        *reinterpret_cast<u32x4*>(smem + hbase + hwr + hh * 1024) = u32x4{pk[0], pk[1], pk[2], pk[3]};
    }
  };

  // Outputs: packed before the next GEMM2 overwrites y; after 4 lane swaps (c
  // and c + 32) and 4 more (c and c + 16) ey[0..3] are 16 bytes of slot r =
  // lane % 16 and ey[4..7] of slot 16 + r, lane row q = lane / 16 having unit
  // 2 (q % 2) + q / 2 of the wavefront's 64 bytes, so that a store covers 64
  // contiguous bytes of 16 rows (32 bytes of 32 rows before the last swaps).
  // Rows past the tile's end repeat its last one, bit for bit.
  auto pack_y = [&]() {
#pragma unroll
    for (int i = 0; i < 8; ++i) ey[i] = pack_bf16x2(y[2 * i], y[2 * i + 1]);
  };
  auto store_y = [&](const TileInfo& t, int n, int blk) {
#pragma unroll
    for (int h = 0; h < 8; h += 4)
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const auto x = permlane32_swap(ey[h + w], ey[h + 2 + w]);
        ey[h + w] = x[0];
        ey[h + 2 + w] = x[1];
      }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const auto x = __builtin_amdgcn_permlane16_swap(ey[w], ey[4 + w], false, false);
      ey[w] = x[0];
      ey[4 + w] = x[1];
    }
    if (blk == 1 && t.row_end - t.row_begin <= 32) return;  // a block without rows
    const int l = here(), q = l >> 4, r = l & 15;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t slot = (uint32_t)slot_at(n, 32 * blk + 16 * i + r);
      const uint32_t tok = slot_token(slot, kdiv);
      const uint32_t o = (tok * (uint32_t)Nh + (uint32_t)t.head) * (uint32_t)k + (slot - tok * (uint32_t)k);
      *reinterpret_cast<u32x4*>(yslot + (uint64_t)o * DH + 32 * wave + 16 * (q & 1) + 8 * (q >> 1)) =
          u32x4{ey[4 * i], ey[4 * i + 1], ey[4 * i + 2], ey[4 * i + 3]};
    }
  };

  auto xfrag = [&](uint32_t base, int s) {
    return *reinterpret_cast<const u32x4*>(smem + (base + off[s]));
  };
  auto hfrag = [&](uint32_t base, int s) {
    return *reinterpret_cast<const u32x4*>(smem + base + hrd + 1024 * s);
  };
  auto gemm1 = [&](auto Pc, auto Sc, auto MATc, const u32x4& f) {
    constexpr int P = decltype(Pc)::value, s = decltype(Sc)::value;
    if constexpr (decltype(MATc)::value == 0)
      A[P] = mfma32_bf16(as_bf16x8(w1[s]), as_bf16x8(f), s == 0 ? zero16() : A[P]);
    else
      B[P] = mfma32_bf16(as_bf16x8(w3[s]), as_bf16x8(f), s == 0 ? zero16() : B[P]);
  };
  auto gemm2 = [&](auto Sc, const u32x4& f) {
    constexpr int s = decltype(Sc)::value;
    y = mfma32_bf16(as_bf16x8(w2[s]), as_bf16x8(f), s == 0 ? zero16() : y);
  };

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  // The full sub-step of parity P: GEMM1 of the block at xb, the activation
  // of the previous block into h at hw, GEMM2 of the block with h at hb; the
  // previous GEMM2's outputs are packed after the first MFMA; hook(s) runs
  // after K step s.  The wavefronts' priority falls as a step proceeds, so that
  // of the two on a SIMD the one behind catches up (the scheduler would serve
  // the older one first and leave the other to run alone; 5% of the kernel).
  auto sub_full = [&](auto Pc, uint32_t xb, uint32_t hb, uint32_t hw, auto&& hook) {
    using O = std::integral_constant<int, 1 - decltype(Pc)::value>;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      xr[s] = xfrag(xb, s);
      hr[s] = hfrag(hb, s);
    }
    constexpr int NM = GELU ? 2 : 3;  // MFMAs per K step
    auto ops = [&](auto Sc, auto Ic) {
      constexpr int i = decltype(Sc)::value * NM + decltype(Ic)::value;
      static_for<i * NACT / (8 * NM), (i + 1) * NACT / (8 * NM)>([&](auto o) { act(O{}, o, hw); });
      __builtin_amdgcn_sched_barrier(0);
    };
    static_for<0, 8>([&](auto Sc) {
      constexpr int s = decltype(Sc)::value;
      if constexpr (s % 4 == 0) __builtin_amdgcn_s_setprio(3 - 2 * decltype(Pc)::value - s / 4);
      gemm1(Pc, Sc, I0{}, xr[s % 2]);
      if constexpr (s == 0) pack_y();
      ops(Sc, I0{});
      if constexpr (!GELU) {
        gemm1(Pc, Sc, I1{}, xr[s % 2]);
        ops(Sc, I1{});
      }
      if constexpr (s + 2 < 8) xr[s % 2] = xfrag(xb, s + 2);
      gemm2(Sc, hr[s % 2]);
      if constexpr (s + 2 < 8) hr[s % 2] = hfrag(hb, s + 2);
      ops(Sc, std::integral_constant<int, NM - 1>{});
      hook(Sc);
    });
  };

  // A tile descriptor by a vector load (lane l reads word l % 4), read back
  // into scalars later: scalar loads return out of order with the LDS reads,
  // so one in flight would turn every wait for a fragment into a wait for
  // all of them.
  static_assert(sizeof(TileInfo) == 16 && offsetof(TileInfo, row_begin) == 4, "tile words");
  auto tile_load = [&](int b) {
    return reinterpret_cast<const int32_t*>(tiles + (b < b1 ? b : b1 - 1))[here() & 3];
  };
  auto tile_read = [&](int v) {
    return TileInfo{__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 1),
                    __builtin_amdgcn_readlane(v, 2), __builtin_amdgcn_readlane(v, 3)};
  };
  auto other = [](const TileInfo& p, const TileInfo& o) {
    return p.expert != o.expert || p.head != o.head;
  };

  // Prologue: the first tiles' slots, rows and weights.
  auto tile_at = [&](int b) { return tiles[b < b1 ? b : b1 - 1]; };
  TileInfo t0 = tile_at(b0), t1 = tile_at(b0 + 1), t2 = tile_at(b0 + 2);  // tiles t .. t + 2
  TileInfo p1 = t0, p2 = t0;                                              // t - 1 and t - 2
  if (wave == 0) dma_slots(t0, 0);
  if (wave == 1) dma_slots(t1, 1);
  weights2(t0);
  weights13(t0);
  barrier_vm<0>();
  {
    int s[L::NDMA];
    row_slots(0, s);
    dma_x(t0, s, L::X_OFF);
  }
  barrier_vm<0>();

  // Step t (n = t - b0): blocks 2 n (rows 0-31 of tile t) and 2 n + 1.  X of
  // tile t in buffer n % 2, h of block j in place j % 4, slots of tile t in
  // list n % 8.  GEMM2 runs on blocks 2 n - 3 (tile t - 2) and 2 n - 2 (tile t
  // - 1); the outputs of tile t - 2 are packed and stored.  Two steps past the
  // last tile drain it.
  auto step = [&](int t, auto FULLc) {
    constexpr bool FULL = decltype(FULLc)::value;
    const int n = t - b0;
    const uint32_t x0 = L::X_OFF + (n & 1) * 2 * L::BLK;         // blocks 2 n, 2 n + 1
    const uint32_t x1 = L::X_OFF + ((n & 1) ^ 1) * 2 * L::BLK;   // the next tile's
    const uint32_t he = L::H_OFF + (n & 1) * 2 * L::BLK;         // places of blocks 2 n, 2 n + 1
    const uint32_t ho = L::H_OFF + ((n & 1) ^ 1) * 2 * L::BLK;   // of blocks 2 n - 2, 2 n - 1
    int tv = 0, sl[L::NDMA];

    // Another expert's W1 and W3 (its W2 in mid-step, before GEMM2 reaches
    // its first block).
    if ((FULL || (n > 0 && t < b1)) && other(t0, p1)) weights13(t0);
    const bool sw2 = (FULL || (n >= 2 && t <= b1)) && other(p1, p2);
    // Loads for later steps: the next tile's rows, the slots of the one after
    // it, the descriptor of the third.  (Touching its weights ahead, for them
    // to wait in L2, changed nothing.)
    auto load_next = [&]() {
      dma_x(t1, sl, x1);
      if (wave == 0) dma_slots(t2, n + 2);
      tv = tile_load(t + 3);
    };
    if constexpr (FULL) {
      sub_full(I0{}, x0, he + L::BLK, ho + L::BLK, [&](auto Sc) {
        constexpr int s = decltype(Sc)::value;
        if constexpr (s == 0) row_slots(n + 1, sl);
        if constexpr (s == 2) load_next();
        if constexpr (s == 4) store_y(p2, n - 2, 0);
      });
      if (sw2) weights2(p1);
      sub_full(I1{}, x0 + L::BLK, ho, he, [&](auto Sc) {
        if constexpr (decltype(Sc)::value == 4) store_y(p2, n - 2, 1);
      });
    } else {
      // The same, part by part and each only where its block exists.
      const bool live = t < b1;
      if (live) {
        row_slots(n + 1, sl);
        load_next();
      }
      auto part = [&](auto Pc, bool ac, bool g2, uint32_t xb, uint32_t hb, uint32_t hw) {
        constexpr int P = decltype(Pc)::value;
        if (n >= 2) {
          pack_y();
          store_y(p2, n - 2, P);
        }
        if (live)
          static_for<0, 8>([&](auto Sc) {
            const u32x4 f = xfrag(xb, decltype(Sc)::value);
            gemm1(Pc, Sc, I0{}, f);
            if constexpr (!GELU) gemm1(Pc, Sc, I1{}, f);
          });
        if (ac)
          static_for<0, NACT>([&](auto o) { act(std::integral_constant<int, 1 - P>{}, o, hw); });
        if (g2) static_for<0, 8>([&](auto Sc) { gemm2(Sc, hfrag(hb, decltype(Sc)::value)); });
      };
      part(I0{}, n >= 1 && t <= b1, n >= 2, x0, he + L::BLK, ho + L::BLK);
      if (sw2) weights2(p1);
      part(I1{}, live, n >= 1 && t <= b1, x0 + L::BLK, ho, he);
    }
    barrier_vm<0>();
    p2 = p1;
    p1 = t0;
    t0 = t1;
    t1 = t2;
    t2 = tile_read(tv);
  };
  for (int t = b0;;) {
    for (; t >= b0 + 2 && t < b1; ++t) step(t, std::true_type{});
    if (t == b1 + 2) break;
    step(t++, std::false_type{});
  }
  // no LDS DMA left in flight when the wavefront ends
  __builtin_amdgcn_s_waitcnt(0x0F70);
}

}  // namespace

hipError_t launch_ffn_ws(const void* X, const int32_t* perm, const TileInfo* tiles,
                         const int32_t* head_base, const void* W1, const void* W3,
                         const void* W2, int64_t T, int Nh, int Ne, int k, void* yslot,
                         hipStream_t s) {
  static_assert(kWsGrid == 256 * Ws::BLOCKS, "every workgroup resident");
  const dim3 grid(kWsGrid), block(Ws::THREADS);
  const int32_t* shares = head_base + Nh + 1;
  if (W3 != nullptr)
    hipLaunchKernelGGL((ffn_ws_kernel<false>), grid, block, 0, s, (const uint16_t*)X, perm, tiles,
                       shares, (const uint16_t*)W1, (const uint16_t*)W3, (const uint16_t*)W2, T,
                       Nh, Ne, k, (uint16_t*)yslot);
  else
    hipLaunchKernelGGL((ffn_ws_kernel<true>), grid, block, 0, s, (const uint16_t*)X, perm, tiles,
                       shares, (const uint16_t*)W1, (const uint16_t*)W1, (const uint16_t*)W2, T,
                       Nh, Ne, k, (uint16_t*)yslot);
  return hipGetLastError();
}

}  // namespace mhl
