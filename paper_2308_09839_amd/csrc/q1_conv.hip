// BF16 matrix-core kernels of the learned preconditioner's network: 3x3x3
// convolution forward, its adjoint in the data (backward-data) and its
// gradient in the weights (backward-weight), all with FP32 accumulation on
// v_mfma_f32_16x16x32_bf16, plus the elementwise kernels around them
// (pooling, upsampling adjoints, ReLU masks, the 1x1 head, the loss, Adam,
// weight packing).
//
// Tensors are channel-last with a zero halo (PGrid): 8 channels of one voxel
// are one 16-byte load and every tap of an output tile is in memory, so the
// inner loops have no bounds tests.  A convolution is the implicit GEMM
// Y^T (Cout x V) = Wp (Cout x K) * X^T (K x V) with K = 27 taps x Cin in
// groups of 8 channels: group g = tap * Cin/8 + cg.  The 16x16x32 instruction
// takes, per lane l, 8 consecutive K of row l%16 of the first operand and 8
// consecutive K of column l%16 of the second, K-block l/16; so each lane
// reads one group (16 bytes) of the packed weights for its output channel and
// one group of the shifted input voxel for its voxel, at an address that it
// holds in a register per K-step.  The result holds 4 consecutive output
// channels of one voxel per lane.  A wavefront owns two 8-voxel rows (16 voxels,
// the columns of an instruction) in each of a tile's 4 z-slices.
//
// Backward-data is the same kernel: the adjoint of a 3x3x3 correlation is
// the correlation with the tap-reversed kernel and transposed channel blocks,
// so only the weight packing differs.  Backward-weight contracts over voxels
// (K = 32 voxels per instruction), with the gradient block as the first operand
// (rows = output channels) and the shifted input as the second (columns = input
// channels), both transposed on the way out of LDS; a workgroup keeps all 27
// taps' accumulators and writes one partial sum per chunk of voxels, which a
// second kernel adds in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "q1_conv.hpp"
#include "q1_internal.hpp"

namespace q1 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(unsigned short u) { return __uint_as_float(unsigned(u) << 16); }
__device__ __forceinline__ unsigned short f2bf(float f) {
  return __builtin_bit_cast(unsigned short, static_cast<__bf16>(f));
}
__device__ __forceinline__ bf16x8 ld8(const bf16 *p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(p));
}

// ---- convolution forward / backward-data ---------------------------------------
//
// A workgroup of four wavefronts computes 8 x 8 x 4 voxel tiles, marching in z, for
// 16 output channels; a wavefront owns two rows of a tile (columns of the
// instruction: 8 x 2 voxels) and its four slices.  The input channels are taken in
// chunks of CC (16, or 8 for an 8-channel input): the chunk's 10 x 10 x 6 halo tile
// (zero outside the padded grid) is staged in LDS once, and all 27 taps of the
// chunk read their shifted voxels from there, so each input voxel is loaded from
// memory once per chunk instead of once per tap; the chunk's weights of the block's
// 16 output channels are staged beside it (once per workgroup when there is one
// chunk), so the K loop issues no global loads.  The next chunk's loads are in
// flight, in registers, while a chunk is computed.  K is ordered chunk-major: chunk
// cc, then tap, then the 8-channel half h of the chunk; each chunk's 27 (CC/8)
// groups are padded to whole K-steps of 4 groups with zero weights (k_pack_* write
// the matching layout).
//
// The K loop is unrolled: a K-step's lane address is one of KSC registers set up
// once (which of the step's taps a lane reads depends on its K-block only) plus an
// immediate offset, so a step is five 16-byte LDS reads, issued one step ahead, and
// four matrix instructions, with no index arithmetic.
//
// LDS banks: a 16-byte read serves lanes {0-3, 12-15, 20-23, 24-27}, then {4-11,
// 16-19, 28-31}, then the same of the upper half in one pass over the 256 B of the
// banks each (found from conflict counts).  So that neither group repeats a bank,
// the halves of a voxel lie in planes a multiple of 256 B apart, 8 voxels of a row
// contiguous in each, and a wavefront's two rows are w and w + 4: 640 B = 128 B
// modulo 256.  Rows 2w and 2w + 1 of interleaved halves kept the LDS busy 1.7 times
// as long.
//
// What bounds it: the LDS reads (1.25 KB per matrix instruction) on the finest
// level, the halo tiles' traffic and FP32 stores elsewhere.  68^3, ten layers:
// batch 1 136 us, batch 4 316 us forward and 353 us backward-data; before (index
// arithmetic in the loop, conflicts, one tile per workgroup, tiles dealt round the
// XCDs so that no L2 saw a neighbour's halo) 200, 500 and 485 us.  Measured and
// dropped: 32 output channels per wavefront (within 5% either way), 2 and 8
// slices per tile.

constexpr int kTX = 8, kTY = 8, kTZ = 4;     // output tile of a workgroup
constexpr int kHX = kTX + 2, kHY = kTY + 2;  // its halo tile

template <int CC>  // staged channels
__global__ __launch_bounds__(256, 3) void k_conv_fwd(ConvArgs a, int nseg) {
  constexpr int TZ = kTZ, HG = CC / 8;      // slices; 8-channel groups per voxel and chunk
  constexpr int NR = kHY * (TZ + 2);        // x rows of the halo tile
  constexpr int HV = kHX * NR;              // voxels
  constexpr int HP = (HV + 15) & ~15;       // voxels of a half's plane (whole 256 B)
  constexpr int KSC = (27 * HG + 3) / 4;    // K-steps per chunk
  constexpr int IPR = kHX * HG;             // 16-byte staging items per row
  constexpr int RPP = 256 / IPR;            // rows per staging pass (the threads past them idle)
  constexpr int PASSES = (NR + RPP - 1) / RPP;
  constexpr int NW = KSC * 4 * 16;          // 16-byte weight items per chunk
  constexpr int WITEMS = (NW + 255) / 256;  // per thread
  __shared__ __align__(16) bf16 sx[HP * CC];  // [h][voxel][8]
  __shared__ __align__(16) bf16 sw[NW * 8];   // the chunk's weights [ks][kg][row][8]
  const PGrid g = a.g;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int TX = (g.W + kTX - 1) / kTX, TY = (g.H + kTY - 1) / kTY, TZn = (g.D + TZ - 1) / TZ;
  const int nrg = a.cout / 16;
  // each XCD takes a contiguous range of the tiles, whose halos then share its L2
  unsigned t = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int rg = int(t % unsigned(nrg));
  t /= unsigned(nrg);
  const int tx = int(t % unsigned(TX));
  t /= unsigned(TX);
  const int ty = int(t % unsigned(TY));
  t /= unsigned(TY);
  const int seg = int(t % unsigned(nseg));
  const int b = int(t / unsigned(nseg));
  if (b >= g.B) return;
  const int x0 = tx * kTX, y0 = ty * kTY;  // logical origin; halo (0,0,0) is padded voxel
                                           // (z0, y0, x0)
  // z tiles [t0, t1): the first TZn % nseg segments have one tile more
  const int tq = TZn / nseg, tr = TZn - tq * nseg;
  const int t0 = tq * seg + min(seg, tr), t1 = t0 + tq + (seg < tr ? 1 : 0);
  const int kg = lane >> 4, j = lane & 15;
  const int vx = j & 7, vy = w + 4 * (j >> 3);  // in the tile

  // this thread's staging items: 8 channels (half h) of voxel hx of rows r0, r0 + RPP, ...
  // of the halo tile; voxels outside the padded grid read the first voxel of their
  // slice's halo, which is zero
  const int64_t plane = int64_t(g.Hp) * g.Wp;
  const bf16 *xb = a.x + (int64_t(b) * g.Dp + int64_t(t0) * TZ) * plane * a.cin;
  const int r0 = tid / IPR, hx = (tid - r0 * IPR) / HG, h = tid % HG;
  unsigned xo[PASSES];  // voxel offsets from slice z0
#pragma unroll
  for (int k = 0; k < PASSES; ++k) {
    const int r = min(r0 + k * RPP, NR - 1), hz = r / kHY, py = y0 + r - hz * kHY;
    xo[k] = x0 + hx < g.Wp && py < g.Hp ? unsigned((hz * g.Hp + py) * g.Wp + x0 + hx) : 0u;
  }
  bf16 *sxw = sx + (h * HP + r0 * kHX + hx) * 8;
  const bool stager = tid < RPP * IPR;
  const bf16 *wb = a.wp + (rg * 16 + size_t(tid / 16) * a.cout + tid % 16) * 8;
  u16x8 xs[PASSES], ws[WITEMS];
  auto load_x = [&](const bf16 *x) {
#pragma unroll
    for (int k = 0; k < PASSES; ++k)
      xs[k] = *reinterpret_cast<const u16x8 *>(x + uint64_t(xo[k]) * unsigned(a.cin));
  };
  auto load_w = [&](int cc) {
#pragma unroll
    for (int k = 0; k < WITEMS; ++k) {  // [q][row] of this row group, q = ks * 4 + kg
      const int q = NW % 256 == 0 || k < WITEMS - 1 || tid < NW % 256 ? k * 16 : 0;
      ws[k] = *reinterpret_cast<const u16x8 *>(wb + size_t(cc * KSC * 4 + q) * a.cout * 8);
    }
  };
  // lane address of K-step ks: group G = 4 ks + kg is (tap, h); padding groups (zero
  // weights) read the centre tap
  int ax[KSC];
#pragma unroll
  for (int ks = 0; ks < KSC; ++ks) {
    int off[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int G = 4 * ks + q, tap = G < 27 * HG ? G / HG : 13, hh = G < 27 * HG ? G % HG : 0;
      off[q] = hh * HP + ((tap / 9) * kHY + (tap / 3) % 3) * kHX + tap % 3;
    }
    const int o = kg < 2 ? (kg == 0 ? off[0] : off[1]) : (kg == 2 ? off[2] : off[3]);
    ax[ks] = (o + vy * kHX + vx) * 8;
  }
  const bf16 *swl = sw + (kg * 16 + j) * 8;

  // this lane's outputs: channels c + i of voxel (x, y, z0 + zb)
  const int ox = x0 + vx, oy = y0 + vy, c = rg * 16 + kg * 4;
  const bool inside = ox < g.W && oy < g.H;
  int64_t vox = g.at(b, t0 * TZ, inside ? oy : 0, inside ? ox : 0);
  float bias[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) bias[i] = a.bias ? a.bias[c + i] : 0.f;
  f32x4 acc[TZ];
  const int nchunk = a.cin / CC;
  // outputs of z tile tz from the accumulators
  auto store = [&](int tz) {
    const int z0 = tz * TZ;
    const int nz = inside ? min(TZ, g.D - z0) : 0;
#pragma unroll
    for (int zb = 0; zb < TZ; ++zb) {
      if (zb >= nz) break;
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = acc[zb][i] + bias[i];
      if (a.relu)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
      if (a.mask.p) {
        const ushort4 m =
            *reinterpret_cast<const ushort4 *>(a.mask.p + vox * a.mask.cs + a.mask.co + c);
        if (!(bf2f(m.x) > 0.f)) v[0] = 0.f;
        if (!(bf2f(m.y) > 0.f)) v[1] = 0.f;
        if (!(bf2f(m.z) > 0.f)) v[2] = 0.f;
        if (!(bf2f(m.w) > 0.f)) v[3] = 0.f;
      }
      if (a.out.p) {
        const ushort4 o{f2bf(v[0]), f2bf(v[1]), f2bf(v[2]), f2bf(v[3])};
        if (!a.out_up) {
          *reinterpret_cast<ushort4 *>(a.out.p + vox * a.out.cs + a.out.co + c) = o;
        } else {
          const PGrid f = g.twice();
          bf16 *p = a.out.p + f.at(b, 2 * (z0 + zb), 2 * oy, 2 * ox) * a.out.cs + a.out.co + c;
#pragma unroll
          for (int k = 0; k < 8; ++k)
            *reinterpret_cast<ushort4 *>(
                p + ((int64_t(k >> 2) * f.Hp + ((k >> 1) & 1)) * f.Wp + (k & 1)) * a.out.cs) = o;
        }
      }
      if (a.o32) {
        const float4 o{v[0], v[1], v[2], v[3]};
        if (a.split == 0)
          *reinterpret_cast<float4 *>(a.o32 + vox * a.cout + c) = o;
        else if (c < a.split)
          *reinterpret_cast<float4 *>(a.o32 + vox * a.split + c) = o;
        else
          *reinterpret_cast<float4 *>(a.o32b + vox * (a.cout - a.split) + (c - a.split)) = o;
      }
      vox += plane;
    }
  };
  load_w(0);
  load_x(xb + h * 8);
  int cc = 0, done = -1;  // done: a finished tile whose outputs are still in acc
  for (int tz = t0; tz < t1;) {
    if (done >= 0 || cc) __syncthreads();  // the previous chunk's reads are done
    if (nchunk > 1 || tz == t0)
#pragma unroll
      for (int k = 0; k < WITEMS; ++k)
        if (NW % 256 == 0 || k < WITEMS - 1 || tid < NW % 256)
          *reinterpret_cast<u16x8 *>(sw + (k * 256 + tid) * 8) = ws[k];
#pragma unroll
    for (int k = 0; k < PASSES; ++k)
      if (stager && (NR % RPP == 0 || k < PASSES - 1 || r0 + k * RPP < NR))
        *reinterpret_cast<u16x8 *>(sxw + k * RPP * kHX * 8) = xs[k];
    __syncthreads();
    // The finished tile's stores go out here, before the next loads: loads and
    // stores complete in order on one counter, so a store issued after the loads
    // would have to land before the next staging, with no work to cover it.
    if (done >= 0) store(done);
    done = -1;
    const bool first = cc == 0;
    if (++cc == nchunk) {
      done = tz++;
      cc = 0;
      xb += TZ * plane * a.cin;
    }
    if (tz < t1) {  // the next chunk, or the next tile's first
      if (nchunk > 1) load_w(cc);
      load_x(xb + cc * CC + h * 8);
    }
    if (first)
#pragma unroll
      for (int zb = 0; zb < TZ; ++zb) acc[zb] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 wv[2], xv[2][TZ];  // operands, read one K-step ahead of their use
    auto read = [&](int ks) {
      wv[ks & 1] = *reinterpret_cast<const bf16x8 *>(swl + ks * 4 * 16 * 8);
#pragma unroll
      for (int zb = 0; zb < TZ; ++zb)
        xv[ks & 1][zb] = *reinterpret_cast<const bf16x8 *>(sx + ax[ks] + zb * kHX * kHY * 8);
    };
    read(0);
#pragma unroll
    for (int ks = 0; ks < KSC; ++ks) {
      if (ks + 1 < KSC) read(ks + 1);
#pragma unroll
      for (int zb = 0; zb < TZ; ++zb)
        acc[zb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[ks & 1], xv[ks & 1][zb], acc[zb],
                                                          0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (done >= 0) store(done);
}

// ---- convolution backward-weight ---------------------------------------------------
//
// dW[t][ci][co] = sum_v x[v + d_t][ci] gy[v][co]: a matrix product that contracts
// over voxels, while the tensors are channel-last.  A workgroup owns one block of
// 16 output x 16 input channels (a unit) and one chunk of the voxels: a run of at
// most kWP pieces of 4 x-consecutive voxels of the (y, x) plane (rows rounded up
// to whole pieces; the round-up region reads zeros), marched through a segment of
// z.  Each slice's run (x with its one-voxel y and x halo, gy without) is copied
// to LDS with 16-byte direct loads, 32 bytes per voxel, and read back as matrix
// operands with the transposing LDS read: a 16-lane group's ds_read_tr16_b64
// returns, per lane, one channel of 4 consecutive voxels, so a tap's shift in x is
// an address offset of 32 bytes and no element is moved by vector instructions.
// A wave holds its gy operands of the last three slices in registers, so each x
// operand (one per (dy, dx)) is read once and feeds the three taps in z: 9 + 1 LDS
// operand reads for 27 matrix instructions.  The four waves' accumulators are
// added in a fixed order at the end, giving one partial per chunk.
//
// What bounds it: at 16 channels (the finest level) the copies of x and gy, which
// a workgroup waits for between slices (two workgroups per compute unit, 238
// VGPRs, so one copies while the other computes); at 32 and more channels the LDS
// operand reads (0.37 KB per matrix instruction and wave).  68^3, batch 4, the ten
// layers of the network: 0.27 ms (0.6 PFLOP/s at the 48 -> 16 and 96 -> 32
// channel layers: 68 and 54 us), against 2.79 ms for per-element gathers (216
// two-byte loads per 32 voxels and lane).

constexpr int kWKS = 3;               // 32-voxel K-steps per wave and slice
constexpr int kWP = 4 * kWKS * 8;     // pieces of a chunk's run: 4 waves
constexpr int kWZero = 256;           // bytes of zeros that absent pieces read
constexpr int kWAcc = 27 * 64 * 16;   // bytes of one wave's accumulators

typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 ld_tr(const char *lds0, const char *lds1) {
  using L = __attribute__((address_space(3))) s16x4;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((L *)(lds0));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((L *)(lds1));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// 16 bytes per lane from src to lds + 16 lane (lds uniform over the wave)
__device__ __forceinline__ void load_lds16(const void *src, char *lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src),
                                   (__attribute__((address_space(3))) void *)(lds), 16, 0, 0);
}

__global__ __launch_bounds__(256, 2) void k_conv_wgrad(ConvWArgs a, WgradPlan pl) {
  extern __shared__ __align__(16) char smem[];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nrb = a.cout >> 4, ncb = (a.cin + 15) >> 4, units = nrb * ncb;
  // each XCD takes a contiguous range of the blocks: the units of one chunk and
  // neighbouring runs read the same lines of x and gy through one L2
  const int nblk = a.nchunks * units, per = (nblk + 7) >> 3;
  const int lb = int(blockIdx.x & 7) * per + int(blockIdx.x >> 3);
  if (int(blockIdx.x >> 3) >= per || lb >= nblk) return;
  const PGrid g = a.g;
  const int unit = lb % units, ch = lb / units;
  const int rbo = unit % nrb, cbi = unit / nrb;
  const int PW = (g.W + 3) >> 2;  // pieces per row
  const int64_t np_all = int64_t(g.H) * PW, plane = int64_t(g.Hp) * g.Wp;
  // LDS: x (pl.S positions between the staged rows of dy = -1, 0, 1; one contiguous
  // range when that is the row pitch), then gy, then zeros
  char *sx = smem, *sg = smem + pl.gy_off, *sz = smem + pl.zero_off;
  if (threadIdx.x < kWZero / 16)
    reinterpret_cast<uint4 *>(sz)[threadIdx.x] = uint4{0, 0, 0, 0};
  const int kg = lane >> 4, i16 = lane & 15;
  const int sub = (i16 >> 2) * 32 + (i16 & 3) * 8;
  f32x4 acc[27], accb = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 27; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 G[3][kWKS];  // gy operands of this slice and the two before it
  u16x8 one;
#pragma unroll
  for (int i = 0; i < 8; ++i) one[i] = 0x3f80;
  const int64_t i0 = pl.items * ch / a.nchunks, i1 = pl.items * (ch + 1) / a.nchunks;
  for (int64_t item = i0; item < i1; ++item) {
    const int run = int(item % pl.nruns), zs = int((item / pl.nruns) % pl.nzseg);
    const int b = int(item / (int64_t(pl.nruns) * pl.nzseg));
    const int z0 = int(int64_t(g.D) * zs / pl.nzseg), z1 = int(int64_t(g.D) * (zs + 1) / pl.nzseg);
    const int nz = z1 - z0;
    const int64_t q0 = np_all * run / pl.nruns, q1 = np_all * (run + 1) / pl.nruns;
    const int np = int(q1 - q0);  // <= kWP
    // padded in-plane position of a piece's first voxel
    auto pos = [&](int64_t q) { return (q / PW + 1) * g.Wp + 4 * (q % PW) + 1; };
    const int64_t p0 = pos(q0);
    const int last = int(pos(q1 - 1) - p0);  // relative position of the last piece
    const int nx = 2 * (pl.S == g.Wp ? last + 2 * g.Wp + 6 : 3 * pl.S), ng = 2 * (last + 4);
    // this lane's operand addresses: read r of K-step ks takes piece (w kWKS + ks) 8 + 4 r + kg
    int ox[kWKS][2], og[kWKS][2];
    int stride[kWKS][2];  // bytes between the rows of dy (0 in the zeros)
#pragma unroll
    for (int ks = 0; ks < kWKS; ++ks)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int q = (w * kWKS + ks) * 8 + 4 * r + kg;
        const bool in = q < np;
        const int rel = in ? int(pos(q0 + q) - p0) : 0;
        ox[ks][r] = (in ? rel * 32 : pl.zero_off) + sub;
        og[ks][r] = (in ? pl.gy_off + rel * 32 : pl.zero_off) + sub;
        stride[ks][r] = in ? pl.S * 32 : 0;
      }
    for (int s = 0; s < nz + 2; ++s) {
      __syncthreads();  // the previous slice's reads are done
      {
        const bf16 *src = a.x + ((int64_t(b) * g.Dp + z0 + s) * plane + p0 - g.Wp - 1) * a.cin;
        const int c0 = cbi * 16;
        for (int k = w * 64; k < nx; k += 256) {
          const int it = min(k + lane, nx - 1);
          const int p = it >> 1;
          int gp = p;
          if (pl.S != g.Wp) gp = (p / pl.S) * g.Wp + min(p % pl.S, last + 5);
          int c = c0 + (it & 1) * 8;
          c = c < a.cin ? c : c0;  // columns past cin are computed but not stored
          load_lds16(src + int64_t(gp) * a.cin + c, sx + k * 16);
        }
      }
      if (s < nz) {
        const bf16 *src = a.gy + ((int64_t(b) * g.Dp + z0 + s + 1) * plane + p0) * a.cout + rbo * 16;
        for (int k = w * 64; k < ng; k += 256) {
          const int it = min(k + lane, ng - 1);
          load_lds16(src + int64_t(it >> 1) * a.cout + (it & 1) * 8, sg + k * 16);
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the direct loads to LDS have landed
      __syncthreads();
#pragma unroll
      for (int ks = 0; ks < kWKS; ++ks) {
        if (s < nz) G[0][ks] = ld_tr(smem + og[ks][0], smem + og[ks][1]);
        bf16x8 X[9];
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
          const char *x0 = smem + ox[ks][0] + dy * stride[ks][0];
          const char *x1 = smem + ox[ks][1] + dy * stride[ks][1];
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) X[dy * 3 + dx] = ld_tr(x0 + dx * 32, x1 + dx * 32);
        }
        // slice s of x is tap dz of gy slice s - dz
        if (s < nz) {
          if (cbi == 0)
            accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(G[0][ks], __builtin_bit_cast(bf16x8, one),
                                                           accb, 0, 0, 0);
#pragma unroll
          for (int t = 0; t < 9; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(G[0][ks], X[t], acc[t], 0, 0, 0);
        }
        if (s >= 1 && s <= nz)
#pragma unroll
          for (int t = 0; t < 9; ++t)
            acc[9 + t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(G[1][ks], X[t], acc[9 + t], 0, 0, 0);
        if (s >= 2)
#pragma unroll
          for (int t = 0; t < 9; ++t)
            acc[18 + t] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(G[2][ks], X[t], acc[18 + t], 0, 0, 0);
        G[2][ks] = G[1][ks];
        G[1][ks] = G[0][ks];
      }
    }
  }
  // (w0 + w2) + (w1 + w3) through two LDS areas, the bias sums beside them
  f32x4 *red = reinterpret_cast<f32x4 *>(smem);
  f32x4 *redb = reinterpret_cast<f32x4 *>(smem + 2 * kWAcc);
  __syncthreads();
  if (w >= 2) {
#pragma unroll
    for (int t = 0; t < 27; ++t) red[((w - 2) * 27 + t) * 64 + lane] = acc[t];
    redb[(w - 2) * 64 + lane] = accb;
  }
  __syncthreads();
  if (w < 2) {
#pragma unroll
    for (int t = 0; t < 27; ++t) acc[t] += red[(w * 27 + t) * 64 + lane];
    accb += redb[w * 64 + lane];
  }
  __syncthreads();
  if (w == 1) {
#pragma unroll
    for (int t = 0; t < 27; ++t) red[t * 64 + lane] = acc[t];
    redb[lane] = accb;
  }
  __syncthreads();
  if (w != 0) return;
#pragma unroll
  for (int t = 0; t < 27; ++t) acc[t] += red[t * 64 + lane];
  accb += redb[lane];
  // rows = output channels rbo*16 + 4*kg + i, column = input channel ci
  const int ci = cbi * 16 + i16;
  const size_t nk = size_t(27) * a.cin_real * a.cout + a.cout;
  float *p = a.part + ch * nk + rbo * 16 + kg * 4;
  if (ci < a.cin_real) {
#pragma unroll
    for (int t = 0; t < 27; ++t)
      *reinterpret_cast<f32x4 *>(p + (size_t(t) * a.cin_real + ci) * a.cout) = acc[t];
  }
  if (cbi == 0 && i16 == 0)
    *reinterpret_cast<f32x4 *>(p + size_t(27) * a.cin_real * a.cout) = accb;
}

// The parts [nparts][n] (weights, then the bias) added in a fixed order: the
// block's wave w takes parts w, w + 16, ... of 64 consecutive entries, eight
// loads in flight, and the 16 wave sums are added in wave order.  k < nw goes to
// gw, the rest to gb.  One launch; its time is one pass over the parts.
__global__ __launch_bounds__(1024) void k_wgrad_sum(const float *__restrict__ part, int nparts,
                                                    int64_t n, int64_t nw, float *__restrict__ gw,
                                                    float *__restrict__ gb) {
  constexpr int NW = 16, U = 8;
  __shared__ float sh[NW][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t k = int64_t(blockIdx.x) * 64 + lane;
  const int64_t kc = k < n ? k : n - 1;
  float s = 0.f;
  for (int c = w; c < nparts; c += NW * U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = part[int64_t(min(c + u * NW, nparts - 1)) * n + kc];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u * NW < nparts) s += v[u];
  }
  sh[w][lane] = s;
  __syncthreads();
  if (w != 0 || k >= n) return;
  float t = sh[0][lane];
#pragma unroll
  for (int i = 1; i < NW; ++i) t += sh[i][lane];
  if (k < nw)
    gw[k] = t;
  else
    gb[k - nw] = t;
}

// Fixed-order sums over parts: out[k] = sum_c part[c * n + k], in two stages.
// Stage 1: block (kb, grp) adds the parts of group grp (kGrp consecutive parts)
// for 64 consecutive k, its four wavefronts taking every fourth part, and
// writes the group sum over the group's first part (read by no other block).
// Stage 2 adds the group sums the same way.
constexpr int kGrp = 64;

__device__ __forceinline__ float sum4_fixed(float (&sh)[4][64], int lane, float v, int w) {
  sh[w][lane] = v;
  __syncthreads();
  return (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
}

__global__ __launch_bounds__(256) void k_sum_parts_grp(float *__restrict__ part, int nparts,
                                                       int64_t n) {
  __shared__ float sh[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t k = int64_t(blockIdx.x) * 64 + lane;
  const int c0 = blockIdx.y * kGrp, c1 = min(nparts, c0 + kGrp);
  float s = 0.f;
  if (k < n)
    for (int c = c0 + w; c < c1; c += 4) s += part[c * n + k];
  const float t = sum4_fixed(sh, lane, s, w);
  if (w == 0 && k < n) part[c0 * n + k] = t;
}

__global__ __launch_bounds__(256) void k_sum_groups(const float *__restrict__ part, int nparts,
                                                    int64_t n, float *__restrict__ out) {
  __shared__ float sh[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t k = int64_t(blockIdx.x) * 64 + lane;
  float s = 0.f;
  if (k < n)
    for (int c = w * kGrp; c < nparts; c += 4 * kGrp) s += part[c * n + k];
  const float t = sum4_fixed(sh, lane, s, w);
  if (w == 0 && k < n) out[k] = t;
}

// out = fixed-order sum of the nparts partial vectors of length n (part is overwritten)
static int sum_parts(float *part, int nparts, int64_t n, float *out, hipStream_t s) {
  const unsigned kb = unsigned((n + 63) / 64), ng = unsigned((nparts + kGrp - 1) / kGrp);
  hipLaunchKernelGGL(k_sum_parts_grp, dim3(kb, ng), dim3(256), 0, s, part, nparts, n);
  hipLaunchKernelGGL(k_sum_groups, dim3(kb), dim3(256), 0, s, part, nparts, n, out);
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

// ---- weight packing ----------------------------------------------------------------------

// The chunk-major K order of k_conv_fwd for an input of cin channels: global
// group q = (cc * KSC + ks) * 4 + kg; within the chunk G = 4 ks + kg, tap =
// G / HG, half h = G % HG (channel cc CC + 8 h + jj); G >= 27 HG is padding.
struct KOrder {
  int CC, HG, KSC;
  __host__ __device__ explicit KOrder(int cin)
      : CC(cin < 16 ? 8 : 16), HG(cin < 16 ? 1 : 2), KSC((27 * (cin < 16 ? 1 : 2) + 3) / 4) {}
  // tap (27 = padding) and first channel of group q
  __host__ __device__ void group(int q, int &tap, int &c) const {
    const int cc = q / (4 * KSC), G = q - cc * 4 * KSC;
    tap = G < 27 * HG ? G / HG : 27;
    c = cc * CC + (G - (G / HG) * HG) * 8;
  }
};

int conv_ksteps(int cin) {
  const KOrder k(cin);
  return (cin / k.CC) * k.KSC;
}

// One launch packs the weights of up to kMaxPack convolutions (a network's forward and
// backward-data forms: a launch each had cost 3.7 us, 20 times).  Forward:
// wp[q][co][jj] = W[tap][c + jj][co] for group q = (tap, c) of the chunk-major order
// over cin_pad channels; zero for padding groups and channels past cin_real; W is
// [27][cin_real][cout] FP32.  Backward-data: the correlation with reversed taps and
// swapped channels over an input of cout channels (the forward's outputs), output ci:
// wq[q][ci][jj] = W[26 - tap][ci][c + jj].
__global__ __launch_bounds__(256) void k_pack(PackJobs jobs) {
  int n = 0;
  while (n + 1 < jobs.n && blockIdx.x >= jobs.j[n + 1].block0) ++n;
  const PackJob &p = jobs.j[n];
  const int rows = p.bwd ? p.cin_real : p.cout;
  const unsigned i = (blockIdx.x - p.block0) * 256 + threadIdx.x;
  if (i >= unsigned(p.groups) * rows * 8) return;
  const int jj = int(i & 7);
  const int row = int((i >> 3) % unsigned(rows)), q = int((i >> 3) / unsigned(rows));
  int tap, c;
  KOrder(p.bwd ? p.cout : p.cin_pad).group(q, tap, c);
  c += jj;
  float v = 0.f;
  if (tap < 27) {
    if (p.bwd)
      v = p.W[(size_t(26 - tap) * p.cin_real + row) * p.cout + c];
    else if (c < p.cin_real)
      v = p.W[(size_t(tap) * p.cin_real + c) * p.cout + row];
  }
  p.out[i] = f2bf(v);
}

// ---- layout changes, pooling, upsampling adjoints, masks ------------------------------

// A block per x row (b, z, y) of the grid: the row's index is split by scalar
// divisions once per block, the threads take its 8-channel items (16-byte loads and
// stores).  Per-element 64-bit divisions had bound these kernels: 68^3 batch 4, the
// 16-channel adjoint of the pooling 61 us, 29 so, of which its 160 MB take most.
struct Row {
  int b, z, y;
  __device__ Row(const PGrid &g, unsigned r) {
    const unsigned q = r / unsigned(g.H);
    y = int(r - q * unsigned(g.H));
    b = int(q / unsigned(g.D));
    z = int(q - unsigned(b) * unsigned(g.D));
  }
};
// the rows of a block: its own index, then every gridDim.x-th (grids are capped)
#define Q1_FOR_ROWS(row, rows) \
  for (unsigned row = blockIdx.x; row < (rows); row += gridDim.x)

struct F8 {
  float v[8];
};
__device__ __forceinline__ F8 ldf8(const float *p) {
  F8 r;
  *reinterpret_cast<float4 *>(r.v) = *reinterpret_cast<const float4 *>(p);
  *reinterpret_cast<float4 *>(r.v + 4) = *reinterpret_cast<const float4 *>(p + 4);
  return r;
}
__device__ __forceinline__ u16x8 ldu8(const bf16 *p) { return *reinterpret_cast<const u16x8 *>(p); }

// Item i of a flat sweep over voxels x C8 items: the voxel's coordinates and the item
// (32-bit divisions while the sweep is that short).  For rows too short to fill a
// block: a row of 68 items per block took 6.2 us at 68^3 where this takes 5.2.
struct Item {
  int b, z, y, x, c;
  __device__ Item(uint64_t i, uint64_t n, unsigned C8, const PGrid &g) {
    uint64_t v;
    if (n >> 32) {
      v = i / C8;
      c = int(i - v * C8) * 8;
    } else {
      const unsigned u = unsigned(i) / C8;
      c = int(unsigned(i) - u * C8) * 8;
      v = u;
    }
    const unsigned w = unsigned(v), q = w / unsigned(g.W), p = q / unsigned(g.H);
    x = int(w - q * unsigned(g.W));
    y = int(q - p * unsigned(g.H));
    b = int(p / unsigned(g.D));
    z = int(p - unsigned(b) * unsigned(g.D));
  }
};

// padded concatenation of unpadded a (half grid when up_a) and b (either may be
// aligned to one element only: ALIGNED says whether both allow 16-byte loads)
template <bool ALIGNED>
__global__ void k_gather_padded(const bf16 *__restrict__ a, int ca, int up_a,
                                const bf16 *__restrict__ b, int cb, PGrid g,
                                bf16 *__restrict__ out, uint64_t n) {
  const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Item e(i, n, unsigned(ca + cb) >> 3, g);
  const bf16 *src;
  if (e.c < ca) {
    const int64_t v = up_a ? ((int64_t(e.b) * (g.D / 2) + (e.z >> 1)) * (g.H / 2) + (e.y >> 1)) *
                                     (g.W / 2) + (e.x >> 1)
                           : ((int64_t(e.b) * g.D + e.z) * g.H + e.y) * g.W + e.x;
    src = a + v * ca + e.c;
  } else {
    src = b + (((int64_t(e.b) * g.D + e.z) * g.H + e.y) * g.W + e.x) * cb + (e.c - ca);
  }
  u16x8 v;
  if constexpr (ALIGNED) {
    v = ldu8(src);
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = src[k];
  }
  *reinterpret_cast<u16x8 *>(out + g.at(e.b, e.z, e.y, e.x) * (ca + cb) + e.c) = v;
}

// C a multiple of 8; out (the caller's) aligned to one float only
__global__ void k_unpad_f32(const float *__restrict__ in, PGrid g, int C, float *__restrict__ out,
                            unsigned rows) {
  Q1_FOR_ROWS(row, rows) {
    const Row r(g, row);
    const float *p = in + g.at(r.b, r.z, r.y, 0) * C;
    float *o = out + ((int64_t(r.b) * g.D + r.z) * g.H + r.y) * g.W * C;
    const int64_t n = int64_t(g.W) * C;
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) o[i] = p[i];
  }
}

// 2x2x2 average pooling of a channel window into a padded coarse tensor [C]
__global__ void k_pool2(Slice in, PGrid f, int C, bf16 *__restrict__ out, uint64_t n) {
  const PGrid g = f.half();
  const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Item e(i, n, unsigned(C) >> 3, g);
  const bf16 *p = in.p + f.at(e.b, 2 * e.z, 2 * e.y, 2 * e.x) * in.cs + in.co + e.c;
  u16x8 v[8], w;
#pragma unroll
  for (int k = 0; k < 8; ++k)
    v[k] = ldu8(p + ((int64_t(k >> 2) * f.Hp + ((k >> 1) & 1)) * f.Wp + (k & 1)) * in.cs);
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) s += bf2f(v[k][c]);
    w[c] = f2bf(s * 0.125f);
  }
  *reinterpret_cast<u16x8 *>(out + g.at(e.b, e.z, e.y, e.x) * C + e.c) = w;
}

// coarse gpre = (sum of the 8 children of gup) * (mask > 0); gup FP32 padded fine [C];
// the mask is the coarse activation, stored upsampled (read at the first child)
__global__ void k_up_adjoint_mask(const float *__restrict__ gup, Slice mask, PGrid g, int C,
                                  bf16 *__restrict__ out, unsigned rows) {
  const PGrid f = g.twice();
  Q1_FOR_ROWS(row, rows) {
    const Row r(g, row);
    const unsigned C8 = unsigned(C) >> 3;
    bf16 *o = out + g.at(r.b, r.z, r.y, 0) * C;
    for (unsigned i = threadIdx.x; i < unsigned(g.W) * C8; i += blockDim.x) {
      const unsigned x = i / C8;
      const int c0 = int(i - x * C8) * 8;
      const int64_t v = f.at(r.b, 2 * r.z, 2 * r.y, 2 * int(x));
      const u16x8 m = ldu8(mask.p + v * mask.cs + mask.co + c0);
      F8 ch[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        ch[k] = ldf8(gup + (v + (int64_t(k >> 2) * f.Hp + ((k >> 1) & 1)) * f.Wp + (k & 1)) * C + c0);
      u16x8 w;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) s += ch[k].v[c];
        w[c] = f2bf(bf2f(m[c]) > 0.f ? s : 0.f);
      }
      *reinterpret_cast<u16x8 *>(o + int64_t(i) * 8) = w;
    }
  }
}

// fine gpre = (gskip + gp[parent] / 8) * (mask > 0), all padded
__global__ void k_pool_adjoint_add_mask(const float *__restrict__ gskip,
                                        const float *__restrict__ gp, Slice mask, PGrid f, int C,
                                        bf16 *__restrict__ out, unsigned rows) {
  const PGrid g = f.half();
  Q1_FOR_ROWS(row, rows) {
    const Row r(f, row);
    const unsigned C8 = unsigned(C) >> 3;
    const int64_t v0 = f.at(r.b, r.z, r.y, 0), p0 = g.at(r.b, r.z >> 1, r.y >> 1, 0);
    for (unsigned i = threadIdx.x; i < unsigned(f.W) * C8; i += blockDim.x) {
      const unsigned x = i / C8;
      const int c0 = int(i - x * C8) * 8;
      const F8 a = ldf8(gskip + v0 * C + int64_t(i) * 8), p = ldf8(gp + (p0 + (x >> 1)) * C + c0);
      const u16x8 m = ldu8(mask.p + (v0 + x) * mask.cs + mask.co + c0);
      u16x8 w;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const float s = a.v[c] + 0.125f * p.v[c];
        w[c] = f2bf(bf2f(m[c]) > 0.f ? s : 0.f);
      }
      *reinterpret_cast<u16x8 *>(out + v0 * C + int64_t(i) * 8) = w;
    }
  }
}

// ---- head, loss -------------------------------------------------------------------------

// padded voxel of logical voxel i (32-bit divisions: a grid that fits the memory has
// fewer than 2^32 voxels)
__device__ __forceinline__ int64_t padded_voxel(unsigned i, const PGrid &g) {
  const unsigned q = i / unsigned(g.W), p = q / unsigned(g.H), b = p / unsigned(g.D);
  return g.at(int(b), int(p - b * unsigned(g.D)), int(q - p * unsigned(g.H)),
              int(i - q * unsigned(g.W)));
}

// out[b][z][y][x] (unpadded) = sum_c t[v][c] wh[c] + bh, t padded [16]
__global__ void k_head_fwd(const bf16 *__restrict__ t, PGrid g, unsigned nv,
                           const float *__restrict__ wh, float *__restrict__ out) {
  constexpr int C = 16;
  const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nv) return;
  const bf16 *tv = t + padded_voxel(i, g) * C;
  const u16x8 lo = ldu8(tv), hi = ldu8(tv + 8);
  float s = wh[C];
#pragma unroll
  for (int c = 0; c < C; ++c) s += bf2f(c < 8 ? lo[c] : hi[c - 8]) * wh[c];
  out[i] = s;
}

constexpr int kHB = 256;  // threads per block of the head / loss reductions

// gpre[v][c] = dout[v] wh[c] (t[v][c] > 0); per-block partials of
// dL/dwh[c] = sum_v dout[v] t[v][c] and dL/dbh = sum_v dout[v]
__global__ __launch_bounds__(kHB) void k_head_bwd(const float *__restrict__ dout,
                                                 const bf16 *__restrict__ t, PGrid g, unsigned nv,
                                                 const float *__restrict__ wh,
                                                 bf16 *__restrict__ gpre,
                                                 float *__restrict__ part /*[nblk][17]*/) {
  constexpr int C = 16;
  __shared__ float sh[C + 1][kHB / 64];
  float acc[C + 1];
#pragma unroll
  for (int c = 0; c <= C; ++c) acc[c] = 0.f;
  const unsigned step = gridDim.x * kHB;
  for (uint64_t j = blockIdx.x * kHB + threadIdx.x; j < nv; j += step) {
    const unsigned i = unsigned(j);
    const int64_t v = padded_voxel(i, g) * C;
    const float d = dout[i];
    const u16x8 in[2] = {ldu8(t + v), ldu8(t + v + 8)};
    acc[C] += d;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u16x8 o;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int c = 8 * h + k;
        const float tv = bf2f(in[h][k]);
        acc[c] += d * tv;
        o[k] = f2bf(tv > 0.f ? d * wh[c] : 0.f);
      }
      *reinterpret_cast<u16x8 *>(gpre + v + 8 * h) = o;
    }
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c <= C; ++c) {
    float s = acc[c];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) sh[c][w] = s;
  }
  __syncthreads();
  if (threadIdx.x <= C) {
    float s = 0.f;
    for (int k = 0; k < kHB / 64; ++k) s += sh[threadIdx.x][k];
    part[blockIdx.x * (C + 1) + threadIdx.x] = s;
  }
}

// per-block partials of sum(weight) and sum(weight (out - target)^2)
__global__ __launch_bounds__(kHB) void k_mse_partials(const float *__restrict__ out,
                                                     const float *__restrict__ tgt,
                                                     const float *__restrict__ wgt, int64_t n,
                                                     double *__restrict__ part) {
  __shared__ double sh[2][kHB / 64];
  double a = 0.0, s = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * kHB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kHB) {
    const double d = double(out[i]) - double(tgt[i]);
    a += wgt[i];
    s += double(wgt[i]) * d * d;
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o);
    s += __shfl_xor(s, o);
  }
  if (lane == 0) {
    sh[0][w] = a;
    sh[1][w] = s;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double r = 0.0;
    for (int k = 0; k < kHB / 64; ++k) r += sh[threadIdx.x][k];
    part[blockIdx.x * 2 + threadIdx.x] = r;
  }
}

// dout = 2 weight (out - target) / sum(weight); loss = sum(w d^2) / sum(w)
__global__ __launch_bounds__(kHB) void k_mse_grad(const float *__restrict__ out,
                                                 const float *__restrict__ tgt,
                                                 const float *__restrict__ wgt, int64_t n,
                                                 const double *__restrict__ part, int nparts,
                                                 float *__restrict__ dout,
                                                 float *__restrict__ loss) {
  // the sums of the parts, in the same fixed order in every block: thread t adds parts
  // t, t + 256, ..., then the tree (one thread adding all of them took 80 us)
  __shared__ double sh[2][kHB / 64];
  double den = 0.0, num = 0.0;
  for (int k = threadIdx.x; k < nparts; k += kHB) {
    den += part[2 * k];
    num += part[2 * k + 1];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    den += __shfl_xor(den, o);
    num += __shfl_xor(num, o);
  }
  if ((threadIdx.x & 63) == 0) {
    sh[0][threadIdx.x >> 6] = den;
    sh[1][threadIdx.x >> 6] = num;
  }
  __syncthreads();
  den = num = 0.0;
  for (int k = 0; k < kHB / 64; ++k) {
    den += sh[0][k];
    num += sh[1][k];
  }
  const float scale = den > 0.0 ? float(2.0 / den) : 0.f;
  for (int64_t i = int64_t(blockIdx.x) * kHB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kHB)
    dout[i] = scale * wgt[i] * (out[i] - tgt[i]);
  if (blockIdx.x == 0 && threadIdx.x == 0 && loss) *loss = den > 0.0 ? float(num / den) : 0.f;
}

// ---- Adam --------------------------------------------------------------------------------

__global__ void k_adam(float *__restrict__ th, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                       float c1, float c2) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ---- host launchers ---------------------------------------------------------------------

static inline dim3 g1(int64_t n, int bs = 256) { return dim3(unsigned((n + bs - 1) / bs)); }
static inline unsigned logical(const PGrid &g) { return unsigned(g.B) * g.D * g.H * g.W; }
// a block per x row of `items` 8-channel items
static inline unsigned nrows(const PGrid &g) { return unsigned(g.B) * g.D * g.H; }
static inline dim3 rows_of(const PGrid &g) { return dim3(std::min(nrows(g), 1u << 22)); }
static inline dim3 row_threads(int items) {
  return dim3(unsigned(std::min(256, (items + 63) / 64 * 64)));
}

int conv_forward(const ConvArgs &a, hipStream_t s) {
  Q1_CHECK(a.cin % 8 == 0 && a.cin >= 8 && (a.cin == 8 || a.cin % 16 == 0) && a.cin <= 96,
           Q1_EUNSUPPORTED, "conv: %d input channels", a.cin);
  Q1_CHECK(a.nchunks == conv_ksteps(a.cin), Q1_EINVAL, "conv: %d K-steps for %d channels",
           a.nchunks, a.cin);
  Q1_CHECK(a.cout % 16 == 0 && a.cout >= 16 && a.cout <= 96, Q1_EUNSUPPORTED,
           "conv: %d output channels (16, 32, 48, 64, 96)", a.cout);
  // z segments: about 2,048 workgroups (three to a compute unit run at once; fewer,
  // longer marches save weight loads and index set-up but leave uneven last rounds:
  // batch 4 at 68^3 670 us of convolutions against 723 with 768 workgroups and 744
  // with one tile each)
  const int64_t cols = int64_t(a.g.B) * ((a.g.H + kTY - 1) / kTY) *
                       ((a.g.W + kTX - 1) / kTX) * (a.cout / 16);
  const int nzt = (a.g.D + kTZ - 1) / kTZ;
  const int nseg = int(std::min<int64_t>(nzt, (2048 + cols - 1) / cols));
  const dim3 blocks(unsigned((cols * nseg + 7) / 8 * 8));
  if (a.cin == 8)
    hipLaunchKernelGGL(k_conv_fwd<8>, blocks, dim3(256), 0, s, a, nseg);
  else
    hipLaunchKernelGGL(k_conv_fwd<16>, blocks, dim3(256), 0, s, a, nseg);
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

// The chunks of the weight gradient: runs of at most kWP pieces cover the plane; z
// is cut into segments so that units x runs x segments is about kWBlocks
// workgroups (two per compute unit; each further segment loads two halo slices of
// x again).  A chunk is one (run, segment, sample) item, or several when that
// would give more than 4 kWBlocks workgroups.
constexpr int kWBlocks = 512;

static WgradPlan wgrad_plan(const ConvWArgs &a) {
  WgradPlan pl;
  const PGrid &g = a.g;
  const int PW = (g.W + 3) / 4, units = (a.cout / 16) * ((a.cin + 15) / 16);
  const int64_t np = int64_t(g.H) * PW;
  pl.nruns = (np + kWP - 1) / kWP;
  const int64_t per_z = units * pl.nruns * g.B;
  pl.nzseg = int(std::max<int64_t>(1, std::min<int64_t>(g.D, kWBlocks / per_z)));
  pl.items = pl.nruns * pl.nzseg * g.B;
  pl.nchunks = int(std::min<int64_t>(pl.items, std::max(1, 4 * kWBlocks / units)));
  // the longest run: n pieces, crossing at most (n - 1 + PW - 1) / PW row ends
  const int n = int((np + pl.nruns - 1) / pl.nruns);
  const int last = 4 * (n - 1) + (n + PW - 2) / PW * (g.Wp - 4 * PW);
  pl.S = std::min(g.Wp, last + 6);
  const int xpos = pl.S == g.Wp ? last + 2 * g.Wp + 6 : 3 * pl.S;
  const auto up = [](int v) { return (v + 1023) & ~1023; };  // whole 64-lane loads
  pl.gy_off = up(xpos * 32);
  pl.zero_off = pl.gy_off + up((last + 4) * 32);
  pl.lds = std::max(pl.zero_off + kWZero, 2 * kWAcc + 2 * 1024);
  return pl;
}

size_t wgrad_part_floats(const ConvWArgs &a) {
  return size_t(wgrad_plan(a).nchunks) * (size_t(27) * a.cin_real + 1) * a.cout;
}

int conv_wgrad(ConvWArgs a, float *gw, float *gb, hipStream_t s) {
  const WgradPlan pl = wgrad_plan(a);
  a.nchunks = pl.nchunks;
  const int nblk = pl.nchunks * (a.cout / 16) * ((a.cin + 15) / 16);
  hipLaunchKernelGGL(k_conv_wgrad, dim3(unsigned((nblk + 7) / 8 * 8)), dim3(256), pl.lds, s, a, pl);
  Q1_HIP(hipGetLastError());
  const int64_t nw = int64_t(27) * a.cin_real * a.cout, n = nw + a.cout;
  hipLaunchKernelGGL(k_wgrad_sum, dim3(unsigned((n + 63) / 64)), dim3(1024), 0, s, a.part,
                     a.nchunks, n, nw, gw, gb);
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

void PackJobs::add(const float *W, int cin_real, int cin_pad, int cout, bool bwd, bf16 *out) {
  PackJob &p = j[n++];
  p = PackJob{W, out, cin_real, cin_pad, cout, 4 * conv_ksteps(bwd ? cout : cin_pad), bwd, blocks};
  blocks += (unsigned(p.groups) * (bwd ? cin_real : cout) * 8 + 255) / 256;
}

int pack_weights(const PackJobs &jobs, hipStream_t s) {
  hipLaunchKernelGGL(k_pack, dim3(jobs.blocks), dim3(256), 0, s, jobs);
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

int gather_padded(const bf16 *a, int ca, int up_a, const bf16 *b, int cb, const PGrid &g, bf16 *out,
                  hipStream_t s) {
  const bool aligned = (reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) % 16 == 0;
  const uint64_t n = uint64_t(logical(g)) * ((ca + cb) / 8);
  hipLaunchKernelGGL((aligned ? k_gather_padded<true> : k_gather_padded<false>), g1(n), dim3(256),
                     0, s, a, ca, up_a, b, cb, g, out, n);
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

int unpad_f32(const float *in, const PGrid &g, int C, float *out, hipStream_t s) {
  hipLaunchKernelGGL(k_unpad_f32, rows_of(g), row_threads(g.W * C), 0, s, in, g, C, out,
                     nrows(g));
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

int pool2(Slice in, const PGrid &fine, int C, bf16 *out, hipStream_t s) {
  const uint64_t n = uint64_t(logical(fine.half())) * (C / 8);
  hipLaunchKernelGGL(k_pool2, g1(n), dim3(256), 0, s, in, fine, C, out, n);
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

int up_adjoint_mask(const float *gup, Slice mask_fine, const PGrid &coarse, int C, bf16 *out,
                    hipStream_t s) {
  hipLaunchKernelGGL(k_up_adjoint_mask, rows_of(coarse), row_threads(coarse.W * C / 8), 0, s, gup,
                     mask_fine, coarse, C, out, nrows(coarse));
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

int pool_adjoint_add_mask(const float *gskip, const float *gp, Slice mask, const PGrid &fine, int C,
                          bf16 *out, hipStream_t s) {
  hipLaunchKernelGGL(k_pool_adjoint_add_mask, rows_of(fine), row_threads(fine.W * C / 8), 0, s,
                     gskip, gp, mask, fine, C, out, nrows(fine));
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

int head_forward(const bf16 *t, const PGrid &g, const float *wh, float *out, hipStream_t s) {
  hipLaunchKernelGGL(k_head_fwd, g1(logical(g)), dim3(256), 0, s, t, g, logical(g), wh, out);
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

int head_backward(const float *dout, const bf16 *t, const PGrid &g, const float *wh, bf16 *gpre,
                  float *part, int nblk, float *gwh, hipStream_t s) {
  hipLaunchKernelGGL(k_head_bwd, dim3(nblk), dim3(kHB), 0, s, dout, t, g, logical(g), wh, gpre,
                     part);
  Q1_HIP(hipGetLastError());
  return sum_parts(part, nblk, int64_t(17), gwh, s);
}

int mse(const float *out, const float *tgt, const float *wgt, int64_t n, double *part, int nblk,
        float *dout, float *loss, hipStream_t s) {
  hipLaunchKernelGGL(k_mse_partials, dim3(nblk), dim3(kHB), 0, s, out, tgt, wgt, n, part);
  hipLaunchKernelGGL(k_mse_grad, dim3(nblk), dim3(kHB), 0, s, out, tgt, wgt, n, part, nblk, dout,
                     loss);
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

int adam(float *th, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2,
         float eps, int step, hipStream_t s) {
  const float c1 = 1.f - std::pow(b1, float(step)), c2 = 1.f - std::pow(b2, float(step));
  hipLaunchKernelGGL(k_adam, g1(n), dim3(256), 0, s, th, g, m, v, n, lr, b1, b2, eps, c1, c2);
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

}  // namespace q1
