// wave_kernels_block.hip -- the sweep of small grids: one TW x TY x ZC block of
// points per workgroup, all of its operands requested at once (paper Eq. 2-3
// and the damping layer of Sec. III-B; the per-point arithmetic is
// wave_point.h's, operand for operand).
//
// What bounds a small grid is latency: a workgroup of the streaming kernel
// works through its 32 planes one after the other, 0.5 us each whatever the
// grid (three planes of loads in flight against 1.5 us of memory latency),
// on a chip that a few hundred workgroups do not fill (64^3: 24 workgroups,
// 22.5 us a step).  Here a workgroup requests the u values of its block with
// all halos, u^{n-1}, vp and phi together, waits once, stages the centre
// planes in LDS with one barrier and computes ZC planes from registers and LDS.
// The z halo is read (ZC + 8) / ZC times, which the XCD's L2 absorbs: its
// blocks are neighbours.  The data fit the memory-side cache and are kept there
// (plain loads, stores written through), and odd steps walk the blocks
// backwards, so that a grid a little larger than that cache finds the part
// touched last.  One step of this kernel also adds the sources and samples
// the receivers of the step before, which saves the second launch.
//
// us per step with a source and a receiver line, before (64 x 8 streaming
// tiles) -> now: 64^3 22.5 -> 4.0, 128^3 23.4 -> 9.2, 160^3 29.5 -> 14.5, 192^3 35.9
// -> 24.5, 256^3 65.0 -> 55 (20-cell layer; 16 at 64^3); 256^3 without a layer 50.1
// -> 40 (7.2 TB/s of its algorithmic bytes on a zero field; a copy inside that
// cache moves 8.3).  bf16 with two points per lane: 128^3 23.5 -> 7.4, 256^3 57 ->
// 42.
//
// What bounds it now: up to about 96^3 the launch itself (2.5 us) and one pass of
// memory latency; above, vector instructions in the layer and traffic to the
// memory-side cache outside it (160^3: the vector units are busy 63 % of the
// time).  Outside the z caps eta is the same in every plane of a block, so its
// float64 sum, both denominators and their reciprocals are formed once per lane,
// and the divisions continue from the reciprocals (div_by_rcp): 52 instead of 68
// vector instructions per layer point.  Measured, us per step: float32 192^3
// 25.9 -> 25.3, bf16 256^3 49.6 -> 46.7, stochastic bf16 256^3 55.7 -> 51.4.
//
// 4 x 4 rows and planes: 8 x 8 blocks read less halo, but hold more registers
// with the layer's operands and leave fewer, longer workgroups (160^3 20.5).
// Without a layer the registers are not short and 8 x 8 wins on larger grids.
// Lanes laid out as 32 columns x 2 rows in tiles that hold an x wall, which pays
// in the streaming kernel, does not here (192^3 23.0 either way).  All tiles 32
// wide (32 x 8 x 4) pay where 64-wide ones leave lanes idle: narrow_blocks.
#include <algorithm>

#include "wave_internal.h"
#include "wave_pair.h"
#include "wave_point.h"

namespace wave {
namespace {

typedef const double __attribute__((address_space(4))) BCDouble;
typedef const float __attribute__((address_space(4))) BCFloat;

// Staged planes of a block.  yz: the centre planes with their y halo, rows of
// 64 floats, so that one base register and the 64-float strides of ds_read2st64
// reach every y neighbour of every plane (also for 32-wide tiles: packed rows cost
// 22 registers of addresses, 160^3 15.5 -> 16.4 us); xr: each row with its x halo,
// the planes of a row back to back.
template <int TW, int TY, int ZC>
struct BlockLds {
  float xr[TY][ZC][TW + 2 * kR];
  float yz[ZC][TY + 2 * kR][kTX];
};

// Where a block lies: its first point, its planes [zb, zb + nzb) with nzb <= ZC.
struct BlockAt {
  int x0, y0, zb, nzb;
};

// One wavefront's row of the block, or two rows of a 32-wide one.  EM as in the
// streaming kernel: 0 no layer point, 1 eta array, 2 tables, and 3 tables outside
// the z caps, where the profile's z term is 0 and eta is the same in every plane.
// FULL: the block has all ZC planes.  NTP: the state is larger than the memory-side
// cache, and all but u^n goes around it.
template <class S, int TW, int TY, int ZC, int EM, bool FULL, bool NTP>
__device__ __forceinline__ void block_rows(const SweepArgs& a, const StepIO& io,
                                           BlockLds<TW, TY, ZC>& sm, const BlockAt& b, bool lay) {
  using T = typename S::T;
  constexpr int NT = TW * TY;
  constexpr int NYH = (2 * kR + TY - 1) / TY;  // y-halo cells per lane and plane
  constexpr int NXE = 2 * kR * TY * ZC;        // x-halo cells of the block
  constexpr int NXH = (NXE + NT - 1) / NT;
  constexpr uint32_t ES = sizeof(T);
  constexpr int kBst = NTP ? kSt : kStThrough;
  constexpr bool LAYER = EM != 0;
  constexpr bool EARR = EM == 1;
  static_assert((2 * kR) % TY == 0 && NT % 64 == 0, "whole y-halo rows per pass");
  static_assert(ZC % 2 == 0, "planes in pairs");

  const int tid = threadIdx.x;
  // column and row in the tile; 64-wide rows are wavefronts
  const int col = tid & (TW - 1);
  const int row = TW == 64 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid / TW;
  const int x = b.x0 + col, y = b.y0 + row;
  const int nzb = FULL ? ZC : b.nzb;
  // window index of plane k of the block (past a partial block's end: its last)
  auto pl = [&](int k) -> uint32_t { return (uint32_t)(kR + (FULL ? k : min(k, nzb - 1))); };
  const int64_t Q = a.plane;
  const int P = a.pitch;
  const uint32_t pe = (uint32_t)Q * ES, p4 = (uint32_t)Q * 4u;
  // window: planes zb-4 .. zb+nzb+3 from row -4, as in the streaming kernel;
  // offsets at kOOB read 0 and store nothing (ghosts, lanes past the grid)
  const int64_t w0 = (int64_t)(b.zb - kR) * Q - (int64_t)kR * P;
  const uint32_t nwin = (uint32_t)(nzb + 2 * kR);
  const auto ru = rsrc_at(static_cast<const T*>(a.cur) + w0, nwin * pe);
  const auto rn = rsrc_at(static_cast<T*>(a.nxt) + w0, nwin * pe);
  const auto rv = rsrc_at(a.vp + w0, nwin * p4);
  const auto rph = rsrc_at(LAYER ? (const void*)(a.phi + w0) : nullptr, LAYER ? nwin * p4 : 0u);
  const auto ret = rsrc_at(EARR ? (const void*)(a.eta + w0) : nullptr, EARR ? nwin * p4 : 0u);
  const bool valid = x < a.nx && y < a.ny;
  const uint32_t ro = (uint32_t)((y + kR) * P + x);
  const uint32_t vo = valid ? ro * ES : kOOB, vo4 = valid ? ro * 4u : kOOB;
  const uint32_t fo = LAYER && lay ? vo4 : kOOB;  // phi and eta: layer points only

  // sources of this step in the wavefront's rows
  constexpr int RW = 64 / TW;
  const int yw = TW == 64 ? y : __builtin_amdgcn_readfirstlane(y);
  uint32_t smask = 0;
#pragma unroll
  for (int s = 0; s < kStepSrc; ++s)
    if (io.sy[s] >= yw && io.sy[s] < yw + RW && io.sz[s] >= b.zb && io.sz[s] < b.zb + nzb &&
        io.sx[s] >= b.x0 && io.sx[s] < b.x0 + TW)
      smask |= 1u << s;

  // every load of the block: first what the staged planes hold, then the rest
  float q[ZC + 2 * kR], hy[NYH][ZC], hx[NXH], vv[ZC], pv[ZC], ph[ZC];
#pragma unroll
  for (int k = 0; k < ZC; ++k)
    q[kR + k] = S::bld(ru, vo, (uint32_t)(FULL ? kR + k : min(kR + k, nzb + 2 * kR - 1)) * pe);
#pragma unroll
  for (int i = 0; i < NYH; ++i) {
    const int hr = row + i * TY;  // halo row
    const int gy = hr < kR ? b.y0 - kR + hr : b.y0 + TY + (hr - kR);
    const uint32_t ho =
        gy >= 0 && gy < a.ny && x < a.nx ? (uint32_t)((gy + kR) * P + x) * ES : kOOB;
#pragma unroll
    for (int k = 0; k < ZC; ++k) hy[i][k] = S::bld(ru, ho, pl(k) * pe);
  }
#pragma unroll
  for (int i = 0; i < NXH; ++i) {
    const int e = tid + i * NT;
    const int cc = e & (2 * kR - 1), rr = (e / (2 * kR)) % TY, k = e / (2 * kR * TY);
    const int gx = cc < kR ? b.x0 - kR + cc : b.x0 + TW + (cc - kR), gy = b.y0 + rr;
    const bool in = k < nzb && gx >= 0 && gx < a.nx && gy < a.ny;
    hx[i] = S::bld(ru, in ? (uint32_t)((gy + kR) * P + gx) * ES + (uint32_t)(kR + k) * pe : kOOB, 0u);
  }
#pragma unroll
  for (int j = 0; j < kR; ++j) {
    q[j] = S::bld(ru, vo, (uint32_t)j * pe);
    q[kR + ZC + j] =
        S::bld(ru, vo, (uint32_t)(FULL ? kR + ZC + j : min(kR + ZC + j, nzb + 2 * kR - 1)) * pe);
  }
#pragma unroll
  for (int k = 0; k < ZC; ++k) {
    vv[k] = NTP ? bld1_f32(rv, vo4, pl(k) * p4) : bld_f32(rv, vo4, pl(k) * p4);
    pv[k] = NTP ? S::bld1(rn, vo, pl(k) * pe) : S::bld(rn, vo, pl(k) * pe);
    if (LAYER) ph[k] = bld_f32(rph, fo, pl(k) * p4);
  }
  float er[ZC + 2], ex0[ZC], ex1[ZC], ey0[ZC], ey1[ZC];
  double tsc = 0.0, tz[ZC];
  float dqx = 0.0f, dqy = 0.0f, dz[ZC];
  if (EM >= 2) {
    const double* tx = a.etab + 1;
    const double* ty = tx + a.nx + 2;
    const BCDouble* tzt = (const BCDouble*)(ty + a.ny + 2) + b.zb;
    const BCFloat* dqzt = (const BCFloat*)(a.etq + a.nx + a.ny) + b.zb;
    const int xc = min(x, a.nx - 1), yc = min(y, a.ny - 1);
    tsc = tx[xc] + ty[yc];
    dqx = a.etq[xc];
    dqy = a.etq[a.nx + yc];
#pragma unroll
    for (int k = 0; k < ZC; ++k) {
      if (EM == 2) tz[k] = tzt[pl(k) - kR];
      dz[k] = dqzt[pl(k) - kR];
    }
  }
  if (EARR) {
    const uint32_t rb4 = (uint32_t)P * 4u;
#pragma unroll
    for (int k = 0; k < ZC; ++k) {
      ex0[k] = bld_f32(ret, fo - 4u, pl(k) * p4);
      ex1[k] = bld_f32(ret, fo + 4u, pl(k) * p4);
      ey0[k] = bld_f32(ret, fo - rb4, pl(k) * p4);
      ey1[k] = bld_f32(ret, fo + rb4, pl(k) * p4);
    }
#pragma unroll
    for (int k = 0; k < ZC + 2; ++k)
      er[k] = bld_f32(ret, fo, (uint32_t)(kR - 1 + (FULL ? k : min(k, nzb + 1))) * p4);
  }

  // stage the centre planes with their x and y halos; one barrier
#pragma unroll
  for (int k = 0; k < ZC; ++k) {
    sm.yz[k][kR + row][col] = q[kR + k];
    sm.xr[row][k][kR + col] = q[kR + k];
#pragma unroll
    for (int i = 0; i < NYH; ++i) {
      const int hr = row + i * TY;
      sm.yz[k][hr < kR ? hr : TY + hr][col] = hy[i][k];
    }
  }
#pragma unroll
  for (int i = 0; i < NXH; ++i) {
    const int e = tid + i * NT;
    const int cc = e & (2 * kR - 1), rr = (e / (2 * kR)) % TY, k = e / (2 * kR * TY);
    if (NXE % NT == 0 || e < NXE) sm.xr[rr][k][cc < kR ? cc : TW + cc] = hx[i];
  }
  __syncthreads();

  // the x rows' base in a register of its own: the reads then fit the 8-bit
  // offsets of ds_read2 without an address add each
  int xbase = (row * ZC) * (TW + 2 * kR) + kR + col;
  asm volatile("" : "+v"(xbase));
  float res[ZC], et[ZC], n1[ZC], n2[ZC];
  if (EM == 3) et[0] = lay ? (float)(a.dt * tsc) : 0.0f;
#pragma unroll
  for (int k = 0; k < ZC; ++k) {
    const float* xr = &sm.xr[0][0][0] + xbase + k * (TW + 2 * kR);
    const float* yr = &sm.yz[k][kR + row][col];
    const float c = q[kR + k];
    float lap = a.c[0] * c;
#pragma unroll
    for (int m = 1; m <= kR; ++m) lap = __builtin_fmaf(a.c[m], xr[m] + xr[-m], lap);
#pragma unroll
    for (int m = 1; m <= kR; ++m)
      lap = __builtin_fmaf(a.c[4 + m], yr[m * kTX] + yr[-m * kTX], lap);
#pragma unroll
    for (int m = 1; m <= kR; ++m)
      lap = __builtin_fmaf(a.c[8 + m], q[kR + k + m] + q[kR + k - m], lap);
    lap = __builtin_fmaf(a.ce, c, lap);
    if (LAYER) {
      float gx, gy, gz;
      if (EARR) {
        et[k] = er[k + 1];
        gx = (ex1[k] - ex0[k]) * a.q[0];
        gy = (ey1[k] - ey0[k]) * a.q[1];
        gz = (er[k + 2] - er[k]) * a.q[2];
      } else {
        if (EM == 2) et[k] = lay ? (float)(a.dt * (tsc + tz[k])) : 0.0f;
        gx = dqx;
        gy = dqy;
        gz = dz[k];
      }
      // outside the layer eta and phi read 0 and the store of phi is dropped
      n1[k] = layer_num(c, pv[k], vv[k], lap, et[EM == 3 ? 0 : k], ph[k]);
      n2[k] = phi_num(ph[k], gx, xr[1] - xr[-1], gy, yr[kTX] - yr[-kTX], gz,
                      q[kR + k + 1] - q[kR + k - 1]);
    } else {
      res[k] = upd_inner(c, pv[k], vv[k], lap);
    }
  }
  if (LAYER) {
    // Zeros count as small, so ahead of the wavefront, where all is zero, the plain
    // divisions run; such steps are not the slower ones (us per step of shots from rest
    // and in flight: 192^3 21.9 and 24.7, 256^3 54.3 and 54.9, bf16 160^3 15.0 and 14.7).
    float least = __builtin_fminf(__builtin_fabsf(n1[0]), __builtin_fabsf(n2[0]));
#pragma unroll
    for (int k = 1; k < ZC; ++k)
      least = __builtin_fminf(least, __builtin_fminf(__builtin_fabsf(n1[k]), __builtin_fabsf(n2[k])));
    if (__any(lay && least < kDivMin)) {
#pragma unroll
      for (int k = 0; k < ZC; ++k) {
        const float e = et[EM == 3 ? 0 : k];
        n1[k] = n1[k] / layer_den(e);
        n2[k] = n2[k] / phi_den(e);
      }
    } else {
      float r1 = 0.0f, r2 = 0.0f;
#pragma unroll
      for (int k = 0; k < ZC; ++k) {
        const float e = et[EM == 3 ? 0 : k], d1 = layer_den(e), d2 = phi_den(e);
        if (EM != 3 || k == 0) {
          r1 = rcp_of(d1);
          r2 = rcp_of(d2);
        }
        n1[k] = div_by_rcp(n1[k], d1, r1);
        n2[k] = div_by_rcp(n2[k], d2, r2);
      }
    }
#pragma unroll
    for (int k = 0; k < ZC; ++k) {
      res[k] = q[kR + k] + n1[k];
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(n2[k]), rph,
                                            (int)(FULL || k < nzb ? fo : kOOB), (int)(pl(k) * p4), kStThrough);
    }
  }

  // to the storage type, then the sources of this step (Alg. 1), added to
  // the stored value in list order; planes past the block store nothing
  const uint32_t srkey = S::kSR ? pcg_hash((uint32_t)a.step) : 0u;
  T ev[ZC];
  if constexpr (S::kSR) {
    // The two lanes of an x pair take their bits from one word: the even one forms
    // it for the even planes, the odd one for the odd planes, and they swap.  Every
    // lane of the wavefront is active here.  Half the hashes: us per step, 96^3 7.2
    // -> 6.8, 192^3 24.3 -> 23.4, 256x240x256 46.2 -> 45.6, 256^3 without a layer
    // 37.2 -> 35.9.
    const bool odd = x & 1;
#pragma unroll
    for (int k = 0; k < ZC; k += 2) {
      const uint32_t own = sr_word(srkey, a.nx, a.ny, x, y, b.zb + k + (odd ? 1 : 0));
      const uint32_t other = __builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);
      ev[k] = f32_to_bf16_sr(res[k], odd ? other >> 16 : own);
      ev[k + 1] = f32_to_bf16_sr(res[k + 1], odd ? own >> 16 : other);
    }
  } else {
#pragma unroll
    for (int k = 0; k < ZC; ++k) ev[k] = S::enc(res[k]);
  }
  if (smask) {
#pragma unroll
    for (int s = 0; s < kStepSrc; ++s) {
      if (!(smask >> s & 1)) continue;
#pragma unroll
      for (int k = 0; k < ZC; ++k)
        if (io.sz[s] == b.zb + k && io.sx[s] == x && (TW == 64 || io.sy[s] == y))
          ev[k] = S::enc(__builtin_fmaf(vv[k], io.sw[s], S::cvt(ev[k])));
    }
  }
#pragma unroll
  for (int k = 0; k < ZC; ++k) {
    const int so = (int)(pl(k) * pe), vk = (int)(FULL || k < nzb ? vo : kOOB);
    if constexpr (sizeof(T) == 4)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, ev[k]), rn, vk, so, kBst);
    else
      __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, ev[k]), rn, vk, so, kBst);
  }
}

// The 64 x 8 x 4 block with two x-adjacent points per lane: a wavefront owns two
// rows of 32 pairs.  For 16-bit storage, whose one-point loads and stores move 2
// bytes per lane: half the memory and LDS instructions of the 4 x 4 block
// (f16 333 x 256 x 272, 20-cell layer, 73 -> 66 us per step; bf16 256^3 50 -> 42).
// float32 gains nothing (192^3 24.3 -> 27.4: 109 registers, 4 wavefronts per SIMD),
// and stochastic rounding spills.  EM 0, 2 or 3.
constexpr int kDY = 8, kDZ = 4;
struct DuoLds {
  float xr[kDY][kDZ][kTX + 2 * kR];
  float yz[kDZ][kDY + 2 * kR][kTX];
};

template <class S, int EM, bool FULL>
__device__ __forceinline__ void duo_rows(const SweepArgs& a, const StepIO& io, DuoLds& sm,
                                         const BlockAt& b, const bool (&lay)[2]) {
  using T = typename S::T;
  using IO = PairIO<S>;
  constexpr int NT = 32 * kDY;
  constexpr int NXE = kR * kDY * kDZ;  // x-halo pairs of the block
  constexpr uint32_t ES = sizeof(T);
  constexpr bool LAYER = EM != 0;
  constexpr int ZC = kDZ;
  static_assert(2 * kR * (kTX / 2) == NT && NXE <= NT, "one y-halo pair per thread and plane");
  static_assert(sizeof(T) == 2 && !S::kSR && (EM == 0 || EM >= 2), "what duo_t launches");

  const int tid = threadIdx.x;
  const int col = 2 * (tid & 31), row = tid >> 5;
  const int x = b.x0 + col, y = b.y0 + row;
  const int nzb = FULL ? ZC : b.nzb;
  auto pl = [&](int k) -> uint32_t { return (uint32_t)(kR + (FULL ? k : min(k, nzb - 1))); };
  const int64_t Q = a.plane;
  const int P = a.pitch;
  const uint32_t pe = (uint32_t)Q * ES, p4 = (uint32_t)Q * 4u;
  const int64_t w0 = (int64_t)(b.zb - kR) * Q - (int64_t)kR * P;
  const uint32_t nwin = (uint32_t)(nzb + 2 * kR);
  const auto ru = rsrc_at(static_cast<const T*>(a.cur) + w0, nwin * pe);
  const auto rn = rsrc_at(static_cast<T*>(a.nxt) + w0, nwin * pe);
  const auto rv = rsrc_at(a.vp + w0, nwin * p4);
  const auto rph = rsrc_at(LAYER ? (const void*)(a.phi + w0) : nullptr, LAYER ? nwin * p4 : 0u);
  // a pair past the grid touches nothing; one whose second point is the first
  // ghost column stores that point's 0
  const bool valid = x < a.nx && y < a.ny, valid1 = x + 1 < a.nx;
  const uint32_t ro = (uint32_t)((y + kR) * P + x);
  const uint32_t vo = valid ? ro * ES : kOOB, vo4 = valid ? ro * 4u : kOOB;
  const uint32_t fo = LAYER && (lay[0] || lay[1]) ? vo4 : kOOB;

  uint32_t smask = 0;
#pragma unroll
  for (int s = 0; s < kStepSrc; ++s)
    if (io.sz[s] >= b.zb && io.sz[s] < b.zb + nzb && io.sy[s] >= b.y0 && io.sy[s] < b.y0 + kDY &&
        io.sx[s] >= b.x0 && io.sx[s] < b.x0 + kTX)
      smask |= 1u << s;

  f32x2 q[ZC + 2 * kR], hy[ZC], hx, vv[ZC], pv[ZC], ph[ZC];
#pragma unroll
  for (int k = 0; k < ZC; ++k)
    q[kR + k] = IO::ld(ru, vo, (uint32_t)(FULL ? kR + k : min(kR + k, nzb + 2 * kR - 1)) * pe);
  const int gy = row < kR ? b.y0 - kR + row : b.y0 + kDY + (row - kR);  // halo row
  const uint32_t ho = gy >= 0 && gy < a.ny && x < a.nx ? (uint32_t)((gy + kR) * P + x) * ES : kOOB;
#pragma unroll
  for (int k = 0; k < ZC; ++k) hy[k] = IO::ld(ru, ho, pl(k) * pe);
  const int hp = tid & 3, hr = (tid >> 2) % kDY, hk = tid / (4 * kDY);
  const int gx = hp < 2 ? b.x0 - kR + 2 * hp : b.x0 + kTX + 2 * (hp - 2);
  const bool hin = hk < nzb && gx >= 0 && gx < a.nx && b.y0 + hr < a.ny;
  hx = IO::ld(ru, hin ? (uint32_t)((b.y0 + hr + kR) * P + gx) * ES + (uint32_t)(kR + hk) * pe : kOOB, 0u);
#pragma unroll
  for (int j = 0; j < kR; ++j) {
    q[j] = IO::ld(ru, vo, (uint32_t)j * pe);
    q[kR + ZC + j] =
        IO::ld(ru, vo, (uint32_t)(FULL ? kR + ZC + j : min(kR + ZC + j, nzb + 2 * kR - 1)) * pe);
  }
#pragma unroll
  for (int k = 0; k < ZC; ++k) {
    vv[k] = ld_f32x2(rv, vo4, pl(k) * p4, false);
    pv[k] = IO::ld(rn, vo, pl(k) * pe);
    if (LAYER) ph[k] = ld_f32x2(rph, fo, pl(k) * p4, false);
  }
  double tsc[2] = {0.0, 0.0}, tz[ZC];
  float dqx[2] = {0.0f, 0.0f}, dqy = 0.0f, dz[ZC];
  if (LAYER) {
    const double* tx = a.etab + 1;
    const double* ty = tx + a.nx + 2;
    const BCDouble* tzt = (const BCDouble*)(ty + a.ny + 2) + b.zb;
    const BCFloat* dqzt = (const BCFloat*)(a.etq + a.nx + a.ny) + b.zb;
    const int xc = min(x, a.nx - 1), xd = min(x + 1, a.nx - 1), yc = min(y, a.ny - 1);
    tsc[0] = tx[xc] + ty[yc];
    tsc[1] = tx[xd] + ty[yc];
    dqx[0] = a.etq[xc];
    dqx[1] = a.etq[xd];
    dqy = a.etq[a.nx + yc];
#pragma unroll
    for (int k = 0; k < ZC; ++k) {
      if (EM == 2) tz[k] = tzt[pl(k) - kR];
      dz[k] = dqzt[pl(k) - kR];
    }
  }

  const int hrow = row < kR ? row : kDY + row;
#pragma unroll
  for (int k = 0; k < ZC; ++k) {
    *reinterpret_cast<f32x2*>(&sm.yz[k][kR + row][col]) = q[kR + k];
    *reinterpret_cast<f32x2*>(&sm.xr[row][k][kR + col]) = q[kR + k];
    *reinterpret_cast<f32x2*>(&sm.yz[k][hrow][col]) = hy[k];
  }
  if (tid < NXE) *reinterpret_cast<f32x2*>(&sm.xr[hr][hk][hp < 2 ? 2 * hp : kTX + 2 * hp]) = hx;
  __syncthreads();

  // the x rows' base in a register of its own: the reads then fit the 8-bit
  // offsets of ds_read2 without an address add each
  int xbase = (row * ZC) * (kTX + 2 * kR) + kR + col;
  asm volatile("" : "+v"(xbase));
  float res[ZC][2], et[ZC][2], n2[ZC][2];
  if (EM == 3)
#pragma unroll
    for (int i = 0; i < 2; ++i) et[0][i] = lay[i] ? (float)(a.dt * tsc[i]) : 0.0f;
#pragma unroll
  for (int k = 0; k < ZC; ++k) {
    const float* xr = &sm.xr[0][0][0] + xbase + k * (kTX + 2 * kR);
    const float* yr = &sm.yz[k][kR + row][col];
    const f32x2 cc = q[kR + k];
    const f32x2 a4 = *reinterpret_cast<const f32x2*>(xr - 4), a2 = *reinterpret_cast<const f32x2*>(xr - 2);
    const f32x2 b2 = *reinterpret_cast<const f32x2*>(xr + 2), b4 = *reinterpret_cast<const f32x2*>(xr + 4);
    const float xv[10] = {a4[0], a4[1], a2[0], a2[1], cc[0], cc[1], b2[0], b2[1], b4[0], b4[1]};
    f32x2 ym[kR], yp[kR];
#pragma unroll
    for (int m = 1; m <= kR; ++m) {
      ym[m - 1] = *reinterpret_cast<const f32x2*>(yr - m * kTX);
      yp[m - 1] = *reinterpret_cast<const f32x2*>(yr + m * kTX);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float c = cc[i];
      float lap = a.c[0] * c;
#pragma unroll
      for (int m = 1; m <= kR; ++m) lap = __builtin_fmaf(a.c[m], xv[4 + i + m] + xv[4 + i - m], lap);
#pragma unroll
      for (int m = 1; m <= kR; ++m) lap = __builtin_fmaf(a.c[4 + m], yp[m - 1][i] + ym[m - 1][i], lap);
#pragma unroll
      for (int m = 1; m <= kR; ++m)
        lap = __builtin_fmaf(a.c[8 + m], q[kR + k + m][i] + q[kR + k - m][i], lap);
      lap = __builtin_fmaf(a.ce, c, lap);
      if (LAYER) {
        // a pair's inner point: eta and phi count as 0, phi is written back
        if (EM == 2) et[k][i] = lay[i] ? (float)(a.dt * (tsc[i] + tz[k])) : 0.0f;
        const float phv = lay[i] ? ph[k][i] : 0.0f;
        res[k][i] = layer_num(c, pv[k][i], vv[k][i], lap, et[EM == 3 ? 0 : k][i], phv);
        n2[k][i] = phi_num(phv, dqx[i], xv[5 + i] - xv[3 + i], dqy, yp[0][i] - ym[0][i], dz[k],
                           q[kR + k + 1][i] - q[kR + k - 1][i]);
      } else {
        res[k][i] = upd_inner(c, pv[k][i], vv[k][i], lap);
      }
    }
  }
  if (LAYER) {
    bool small = false;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float least = __builtin_fminf(__builtin_fabsf(res[0][i]), __builtin_fabsf(n2[0][i]));
#pragma unroll
      for (int k = 1; k < ZC; ++k)
        least = __builtin_fminf(least, __builtin_fminf(__builtin_fabsf(res[k][i]), __builtin_fabsf(n2[k][i])));
      small = small || (lay[i] && least < kDivMin);
    }
    const bool exact = __any(small);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (exact) {
#pragma unroll
        for (int k = 0; k < ZC; ++k) {
          const float e = et[EM == 3 ? 0 : k][i];
          res[k][i] = res[k][i] / layer_den(e);
          n2[k][i] = n2[k][i] / phi_den(e);
        }
      } else {
        float r1 = 0.0f, r2 = 0.0f;
#pragma unroll
        for (int k = 0; k < ZC; ++k) {
          const float e = et[EM == 3 ? 0 : k][i], d1 = layer_den(e), d2 = phi_den(e);
          if (EM != 3 || k == 0) {
            r1 = rcp_of(d1);
            r2 = rcp_of(d2);
          }
          res[k][i] = div_by_rcp(res[k][i], d1, r1);
          n2[k][i] = div_by_rcp(n2[k][i], d2, r2);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < ZC; ++k) {
      res[k][0] = q[kR + k][0] + res[k][0];
      res[k][1] = q[kR + k][1] + res[k][1];
      __builtin_amdgcn_raw_buffer_store_b64(
          u32x2{__float_as_uint(lay[0] ? n2[k][0] : ph[k][0]), __float_as_uint(lay[1] ? n2[k][1] : ph[k][1])},
          rph, (int)(FULL || k < nzb ? fo : kOOB), (int)(pl(k) * p4), kStThrough);
    }
  }

  T ev[ZC][2];
#pragma unroll
  for (int k = 0; k < ZC; ++k) {
    ev[k][0] = S::enc(res[k][0]);
    ev[k][1] = S::enc(res[k][1]);
  }
  if (smask) {
#pragma unroll
    for (int s = 0; s < kStepSrc; ++s) {
      if (!(smask >> s & 1)) continue;
#pragma unroll
      for (int k = 0; k < ZC; ++k)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (io.sz[s] == b.zb + k && io.sy[s] == y && io.sx[s] == x + i)
            ev[k][i] = S::enc(__builtin_fmaf(vv[k][i], io.sw[s], S::cvt(ev[k][i])));
    }
  }
#pragma unroll
  for (int k = 0; k < ZC; ++k) {
    const int so = (int)(pl(k) * pe), vk = (int)(FULL || k < nzb ? vo : kOOB);
    const T e1 = valid1 ? ev[k][1] : (T)0;
    __builtin_amdgcn_raw_buffer_store_b32(
        (uint32_t)__builtin_bit_cast(uint16_t, ev[k][0]) | ((uint32_t)__builtin_bit_cast(uint16_t, e1) << 16),
        rn, vk, so, kStThrough);
  }
}

__device__ __forceinline__ int div_by(int n, int d, uint32_t m) {
  return d == 1 ? n : (int)__umulhi((uint32_t)n, m);
}

// Tile and layer of block `at` of XCD xcd; false: padding.  An XCD takes one
// slab of tile rows through the layers of blocks, so neighbouring blocks read
// their halos from one L2 (8 % faster at 256^3 than a contiguous run of layers
// per XCD).  Where the tile rows do not divide by 8 the slabs differ by a row;
// in the upper half of the layers every XCD takes the next one's, which evens
// them out.  Few tile rows do not make 8 slabs of about one size, and leave XCDs
// idle: there each takes a run of consecutive rows of blocks (block_grid).
__device__ __forceinline__ bool block_at(const BlockGrid& g, int xcd, int at, int* tx, int* ty,
                                         int* zl) {
  const int t2 = div_by(at, g.tiles_x, g.mx);
  *tx = at - t2 * g.tiles_x;
  const int r = t2 + xcd * g.run;
  *zl = div_by(r, g.slab, g.mrow);
  *ty = r - *zl * g.slab;
  if (g.run) return *zl < g.layers;
  const int k = (xcd + (*zl >= g.half ? 1 : 0)) & 7;
  *ty += k * g.tiles_y >> 3;
  return *ty < ((k + 1) * g.tiles_y >> 3);
}

// Block `at` of XCD xcd.  LM: the layer's update, 0 damping off, 1 eta array,
// 2 tables.
template <class S, int TW, int TY, int ZC, int LM, bool NTP>
__device__ __forceinline__ void block_sweep(const SweepArgs& a, const StepIO& io,
                                            BlockLds<TW, TY, ZC>& sm, const BlockGrid& g, int xcd,
                                            int at) {
  int tx, ty, zl;
  if (!block_at(g, xcd, at, &tx, &ty, &zl)) return;
  constexpr bool damp = LM != 0;
  static_assert(!(NTP && damp), "larger states with a layer run the streaming kernels");
  const ChunkInfo c = chunk_of(zl, a.nz, a.w, ZC, damp);
  BlockAt b;
  b.x0 = tx * TW;
  b.y0 = ty * TY;
  b.zb = c.zb;
  b.nzb = c.ze - c.zb;
  const int x = b.x0 + (int)(threadIdx.x & (TW - 1));
  const int y = b.y0 + (TW == 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)
                                 : (int)threadIdx.x / TW);
  const bool lay = damp && x < a.nx && y < a.ny &&
                   (c.cap || x < a.w || x >= a.nx - a.w || y < a.w || y >= a.ny - a.w);
  const bool none = LM == 0 || !__any(lay);
  if (b.nzb == ZC) {
    if (none)
      block_rows<S, TW, TY, ZC, 0, true, NTP>(a, io, sm, b, false);
    else if (LM == 2 && !c.cap)
      block_rows<S, TW, TY, ZC, 3, true, NTP>(a, io, sm, b, lay);
    else
      block_rows<S, TW, TY, ZC, LM, true, NTP>(a, io, sm, b, lay);
  } else {
    if (none)
      block_rows<S, TW, TY, ZC, 0, false, NTP>(a, io, sm, b, false);
    else
      block_rows<S, TW, TY, ZC, LM, false, NTP>(a, io, sm, b, lay);
  }
}

// The same for blocks with two points per lane.
template <class S, int LM>
__device__ __forceinline__ void duo_sweep(const SweepArgs& a, const StepIO& io, DuoLds& sm,
                                          const BlockGrid& g, int xcd, int at) {
  int tx, ty, zl;
  if (!block_at(g, xcd, at, &tx, &ty, &zl)) return;
  constexpr bool damp = LM != 0;
  const ChunkInfo c = chunk_of(zl, a.nz, a.w, kDZ, damp);
  BlockAt b;
  b.x0 = tx * kTX;
  b.y0 = ty * kDY;
  b.zb = c.zb;
  b.nzb = c.ze - c.zb;
  const int y = b.y0 + (int)(threadIdx.x >> 5);
  bool lay[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int x = b.x0 + 2 * (int)(threadIdx.x & 31) + i;
    lay[i] = damp && x < a.nx && y < a.ny &&
             (c.cap || x < a.w || x >= a.nx - a.w || y < a.w || y >= a.ny - a.w);
  }
  const bool none = LM == 0 || !__any(lay[0] || lay[1]);
  if (b.nzb == kDZ) {
    if (none)
      duo_rows<S, 0, true>(a, io, sm, b, lay);
    else if (LM == 2 && !c.cap)
      duo_rows<S, 3, true>(a, io, sm, b, lay);
    else
      duo_rows<S, LM, true>(a, io, sm, b, lay);
  } else {
    if (none)
      duo_rows<S, 0, false>(a, io, sm, b, lay);
    else
      duo_rows<S, LM, false>(a, io, sm, b, lay);
  }
}

// Requests every 64-byte line of the kernel's arguments at its start, in one wait.
// Each step's arguments are new to the scalar cache; read where they are first
// used, their lines arrive one after the other, which a small grid has nothing to
// hide behind.  us per step: 64^3 4.5 -> 4.1, 70x45x37 4.85 -> 4.35, 96^3 6.6 ->
// 6.0, 128^3 9.8 -> 9.2, 176x144x160 16.8 -> 16.3; from 256^3 on no difference.
__device__ __forceinline__ void touch_args(const SweepArgs& a, const StepIO& io, const BlockGrid& g) {
  asm volatile("" ::"s"(a.nx), "s"(a.etab), "s"(io.sz[3]), "s"(g.per_xcd), "s"(a.step));
}

template <class S, int LM>
__global__ __launch_bounds__(256, 4) void k_sweep_duo(SweepArgs a, StepIO io, BlockGrid g) {
  __shared__ __attribute__((aligned(16))) DuoLds sm;
  touch_args(a, io, g);
  const int slot = blockIdx.x >> 3;
  if (slot >= g.per_xcd) {
    record_row<S>(a, io, (blockIdx.x - 8 * g.per_xcd) * 256 + threadIdx.x);
    return;
  }
  duo_sweep<S, LM>(a, io, sm, g, blockIdx.x & 7, (a.step & 1) ? g.per_xcd - 1 - slot : slot);
}

template <class S, int TW, int TY, int ZC, int LM, bool NTP>
__global__ __launch_bounds__(TW * TY, 4) void k_sweep_block(SweepArgs a, StepIO io, BlockGrid g) {
  __shared__ BlockLds<TW, TY, ZC> sm;
  touch_args(a, io, g);
  const int slot = blockIdx.x >> 3;
  if (slot >= g.per_xcd) {  // receivers of u^n, the last step's field
    record_row<S>(a, io, (blockIdx.x - 8 * g.per_xcd) * TW * TY + threadIdx.x);
    return;
  }
  // Odd steps walk the blocks backwards: what a step touched last is still in
  // the memory-side cache when the next one starts (256^3: 60.7 -> 51.6 us).
  block_sweep<S, TW, TY, ZC, LM, NTP>(a, io, sm, g, blockIdx.x & 7,
                                      (a.step & 1) ? g.per_xcd - 1 - slot : slot);
}

union WideOrNarrow {
  BlockLds<64, 4, 4> wide;
  BlockLds<32, 8, 4> narrow;
};

// Several members of a batch in one launch.  The sweep's arguments come from
// the batch's table, everything that changes from step to step by value.
template <class S, int LM, bool DUO>
__global__ __launch_bounds__(256, 4) void k_sweep_block_batch(const BatchShot* __restrict__ shots,
                                                              BlockBatch bb) {
  __shared__ __attribute__((aligned(16))) std::conditional_t<DUO, DuoLds, WideOrNarrow> sm;
  const int bid = (int)order_block(blockIdx.x, gridDim.x, bb.back);
  int m = 0;
  for (int i = 1; i < bb.n; ++i)
    if (bid >= bb.begin[i]) m = i;
  const BlockBatch::Member& e = bb.m[m];
  SweepArgs a = shots[m].sa;
  a.cur = shots[m].u[e.cur];
  a.nxt = shots[m].u[e.cur ^ 1];
  a.step = e.step;
  const int local = bid - bb.begin[m];
  if ((local >> 3) >= e.g.per_xcd) {
    record_row<S>(a, e.io, (local - 8 * e.g.per_xcd) * 256 + threadIdx.x);
    return;
  }
  if constexpr (DUO)
    duo_sweep<S, LM>(a, e.io, sm, e.g, local & 7, local >> 3);
  else if (e.g.narrow)
    block_sweep<S, 32, 8, 4, LM, false>(a, e.io, sm.narrow, e.g, local & 7, local >> 3);
  else
    block_sweep<S, 64, 4, 4, LM, false>(a, e.io, sm.wide, e.g, local & 7, local >> 3);
}

// Receivers of the last step of a run, one workgroup per member; the members'
// states in the table are those at its start.
template <class S>
__global__ __launch_bounds__(256) void k_record_last(const BatchShot* __restrict__ shots,
                                                     const BatchState* __restrict__ state) {
  using T = typename S::T;
  const BatchShot& b = shots[blockIdx.x];
  const BatchState& st = state[blockIdx.x];
  if (b.target < 1) return;
  const T* u = static_cast<const T*>(b.u[st.cur ^ (b.target & 1)]);
  double* row = b.inj.traces + (int64_t)(st.trace_row + b.target - 1) * b.inj.nrec;
  for (int r = threadIdx.x; r < b.inj.nrec; r += blockDim.x) row[r] = (double)S::ld(u, b.inj.rec_off[r]);
}

// 4 x 4 blocks are 64 points wide, or 32 x 8 where that saves a sixth of the lanes
// or more: with 1, 3 or 5 tiles of 32 columns (1..32, 65..96 and 129..160 points in x)
// 64-wide tiles leave a half tile idle.  us per step, 64 -> 32 wide: 70x45x37 5.05 -> 4.85,
// 96^3 7.05 -> 6.6 (no layer 5.9 -> 5.3), 160^3 16.8 -> 15.6 (no layer 12.8 -> 11.3),
// 160^3 in f16 16.7 -> 14.3 and stochastic bf16 18.0 -> 16.4.  With 7 tiles the
// saving no longer decides (224^3 37.4..39.9 -> 38.3..39.4), and where it saves none,
// 32-wide tiles read more x halo (176x144x160 16.6 -> 17.5, 256^3 55 -> 56.4).  Up to
// 32 points half of every wavefront was idle: 9 x 1420 x 1173 316 -> 224 (64 x 8
// streaming tiles 288), 32 x 753 x 622 84 -> 59, 30 x 100 x 100 5.1 -> 4.4 and bf16 5.1
// -> 4.6; below 64^2 rows a launch is too short to gain (bf16 32^3 3.9 -> 4.3).
bool narrow_blocks(const SweepArgs& a) {
  const int tiles = cdiv(a.nx, 32);
  return tiles == 3 || tiles == 5 || (tiles == 1 && (int64_t)a.ny * a.nz >= 4096);
}

// A launch holds less than 2^32 threads; a sixteenth of them is left for receivers.
constexpr int64_t kLaunchThreads = 0xf0000000LL;

// false: the grid does not fit the index arithmetic or one launch.
bool block_grid(const SweepArgs& a, int tw, int ty, int zc, BlockGrid* g) {
  g->tiles_x = cdiv(a.nx, tw);
  g->tiles_y = cdiv(a.ny, ty);
  g->slab = cdiv(g->tiles_y, 8);
  const int layers = chunk_count(a.nz, a.w, zc, a.damping != 0);
  g->half = cdiv(layers, 2);
  // Runs where slabs load the busiest XCD by more than 8 % more; us per step, slabs ->
  // runs, with the loads' ratio: 8 x 4 bf16 2939 x 5 x 2041 398 -> 123 (4.0), 774 x 72 x
  // 537 109 -> 83 (1.33); 4 x 4 float32 1039 x 20 x 721 80 -> 49 (1.6), 70x45x37 4.3 ->
  // 4.0 (1.22); 8 x 8 without a layer 500 x 200 x 500 146 -> 146, bf16 112 -> 99 (1.12).
  // Also where slabs of a few rows share little: blocks of 4 rows up to 160 rows of
  // points (580 x 64 x 403 58 -> 48, 96^3 5.9 -> 5.4, 300 x 160 x 200 35.7 -> 34.9; 376 x
  // 152 x 261 47.8 -> 48.1), of 8 x 4 up to 112 (670 x 96 x 465 84 -> 79, 621 x 112 x 431
  // 81 -> 77; 600 x 120 x 416 79.5 -> 80).  Elsewhere slabs: 8 x 8 948 x 64 x 658 110.1 ->
  // 110.8 and 512^3 358 -> 401, 4 x 4 192^3 with an eta array 28.7 -> 29.1 and 256^3 54.4
  // -> 63.8, 8 x 4 256^3 42.4 -> 43.4.
  const int64_t rows = (int64_t)g->tiles_y * layers;
  auto slab_rows = [&](int k) { return ((k + 1) * g->tiles_y >> 3) - (k * g->tiles_y >> 3); };
  int64_t most = 0;
  for (int k = 0; k < 8; ++k)
    most = std::max(most, (int64_t)g->half * slab_rows(k) + (int64_t)(layers - g->half) * slab_rows((k + 1) & 7));
  const int64_t run = (rows + 7) / 8;
  const bool runs = 25 * most > 27 * run || (zc == 4 && a.ny <= (tw == kTX && ty == kDY ? 112 : 160));
  const int64_t n = g->tiles_x * (runs ? run : (int64_t)g->slab * layers);
  if ((int64_t)(zc + 2 * kR) * a.plane * 4 > kWindowMax ||
      n * std::max(g->tiles_x, g->slab) >= (int64_t(1) << 32) ||
      8 * n * (tw == kTX && ty == kDY && zc == kDZ ? 256 : tw * ty) > kLaunchThreads ||
      (runs && 8 * run * g->tiles_y >= (int64_t(1) << 32)))  // rows of blocks by layers
    return false;
  g->run = runs ? (int32_t)run : 0;
  g->layers = layers;
  if (runs) g->slab = g->tiles_y;
  g->per_xcd = (int)n;
  auto magic = [](int d) { return (uint32_t)(0xffffffffu / (uint32_t)d + 1u); };
  g->mx = magic(g->tiles_x);
  g->mrow = magic(g->slab);
  g->narrow = tw == 32;
  return true;
}

bool block_grid_44(const SweepArgs& a, BlockGrid* g) {
  return narrow_blocks(a) ? block_grid(a, 32, 8, 4, g) : block_grid(a, kTX, 4, 4, g);
}

template <class S, int TW, int TY, int ZC, int LM, bool NTP>
hipError_t block_t(const SweepArgs& a, const StepIO& io, hipStream_t st) {
  BlockGrid g;
  if (!block_grid(a, TW, TY, ZC, &g)) return hipErrorInvalidValue;
  const int rec = io.nrec > 0 ? cdiv(io.nrec, TW * TY) : 0;
  const dim3 grid((unsigned)(8 * g.per_xcd + rec)), blk(TW * TY);
  hipLaunchKernelGGL((k_sweep_block<S, TW, TY, ZC, LM, NTP>), grid, blk, 0, st, a, io, g);
  return hipGetLastError();
}

template <class S, int LM>
hipError_t duo_t(const SweepArgs& a, const StepIO& io, hipStream_t st) {
  BlockGrid g;
  if (!block_grid(a, kTX, kDY, kDZ, &g)) return hipErrorInvalidValue;
  const int rec = io.nrec > 0 ? cdiv(io.nrec, 256) : 0;
  hipLaunchKernelGGL((k_sweep_duo<S, LM>), dim3((unsigned)(8 * g.per_xcd + rec)), dim3(256), 0, st, a, io, g);
  return hipGetLastError();
}

template <class S>
hipError_t block_s(const SweepArgs& a, const StepIO& io, int ty, int zc, bool nt, hipStream_t st) {
  if (ty == 4 && zc == 4) {
    if (narrow_blocks(a))
      return a.eta       ? block_t<S, 32, 8, 4, 1, false>(a, io, st)
             : a.damping ? block_t<S, 32, 8, 4, 2, false>(a, io, st)
                         : block_t<S, 32, 8, 4, 0, false>(a, io, st);
    return a.eta       ? block_t<S, 64, 4, 4, 1, false>(a, io, st)
           : a.damping ? block_t<S, 64, 4, 4, 2, false>(a, io, st)
                       : block_t<S, 64, 4, 4, 0, false>(a, io, st);
  }
  if constexpr (sizeof(typename S::T) == 2 && !S::kSR) {
    if (ty == kDY && zc == kDZ && !a.eta) return a.damping ? duo_t<S, 2>(a, io, st) : duo_t<S, 0>(a, io, st);
  }
  if constexpr (!S::kSR) {
    if (ty == 8 && zc == 8 && !a.damping)
      return nt ? block_t<S, 64, 8, 8, 0, true>(a, io, st) : block_t<S, 64, 8, 8, 0, false>(a, io, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool block_config_supported(int ty, int zc, const SweepArgs& a, int storage) {
  const bool cfg = (ty == 4 && zc == 4) ||
                   (ty == kDY && zc == kDZ && !a.eta && (storage == 1 || storage == 2)) ||
                   (ty == 8 && zc == 8 && !a.damping && storage != 3);
  BlockGrid g;
  return cfg && (ty == 4 ? block_grid_44(a, &g) : block_grid(a, kTX, ty, zc, &g));
}

int64_t sweep_footprint(int nx, int ny, int nz, int w, bool damping, bool eta_array, int es) {
  const int64_t pts = (int64_t)nx * ny * nz;
  const int64_t inner = (int64_t)(nx - 2 * w) * (ny - 2 * w) * (nz - 2 * w);
  return pts * (2 * es + 4 + (eta_array ? 4 : 0)) + (damping ? (pts - inner) * 4 : 0);
}

void block_default(const SweepArgs& a, int storage, int* ty, int* zc) {
  const int es = storage == 0 ? 4 : 2;
  const int64_t bytes =
      sweep_footprint(a.nx, a.ny, a.nz, a.w, a.damping != 0, a.eta != nullptr, es);
  *ty = *zc = 0;
  // one plane past whole layers of 8 costs as much as 8 (us per step against the
  // streaming tiles: float32 2529 x 1756 x 9 181 / 170, 1840 x 1278 x 17 157 / 145, 1321
  // x 917 x 33 132 / 128, 1185 x 823 x 41 127 / 128, and of less state 1380 x 958 x 17
  // 84 / 81, 1138 x 790 x 25 77 / 80; bf16 3098 x 2151 x 9 206 / 193, 2254 x 1565 x 17
  // 166 / 169; four planes past, float32 2104 x 1461 x 13, 136 / 151)
  const bool one_more = a.nz % 8 == 1 && a.nz > 1 &&
                        a.nz < (es == 2 ? 16 : bytes > 280 * 1000000LL ? 40 : 24);
  const bool duo = es == 2 && storage != 3 && !a.eta && bytes > 10 * 1000000LL &&
                   bytes <= (a.damping ? 360 : 280) * 1000000LL;
  if (duo) {
    *ty = kDY;
    *zc = kDZ;
  } else if (!a.damping && storage != 3 && bytes > 240 * 1000000LL) {
    if (!one_more) *ty = *zc = 8;
  } else if (bytes <= 280 * 1000000LL) {
    *ty = *zc = 4;
  }
  if (*ty && !block_config_supported(*ty, *zc, a, storage)) *ty = *zc = 0;
}

hipError_t launch_sweep_block(const SweepArgs& a, const StepIO& io, int storage, int ty, int zc,
                              hipStream_t s) {
  // past 400 MB (no layer: one array set of u, u_prev and vp) the cache holds
  // too little of the state to be worth the traffic: 8 x 8 blocks without a
  // layer run 320x304x288 (336 MB) in 71.0 us plain and 72.0 around it, 384^3
  // (680 MB) in 149 and 137
  const bool nt = sweep_footprint(a.nx, a.ny, a.nz, a.w, a.damping != 0, a.eta != nullptr,
                                  storage == 0 ? 4 : 2) > 400 * 1000000LL;
  switch (storage) {
    case 0: return block_s<StF32>(a, io, ty, zc, nt, s);
    case 1: return block_s<StBF16>(a, io, ty, zc, nt, s);
    case 2: return block_s<StF16>(a, io, ty, zc, nt, s);
    case 3: return block_s<StBF16SR>(a, io, ty, zc, nt, s);
  }
  return hipErrorInvalidValue;
}

int block_batch_grid(const SweepArgs& a, bool duo, int nrec, BlockGrid* g) {
  if (!(duo ? block_grid(a, kTX, kDY, kDZ, g) : block_grid_44(a, g))) return 0;
  return 8 * (g->per_xcd + cdiv(cdiv(nrec, 256), 8));
}

template <class S>
hipError_t block_batch_s(const BatchShot* shots, const BlockBatch& bb, int lm, bool duo,
                         hipStream_t st) {
  const dim3 grid((unsigned)bb.begin[bb.n]);
  if constexpr (sizeof(typename S::T) == 2 && !S::kSR) {
    if (duo) {
      if (lm == 0)
        hipLaunchKernelGGL((k_sweep_block_batch<S, 0, true>), grid, dim3(256), 0, st, shots, bb);
      else
        hipLaunchKernelGGL((k_sweep_block_batch<S, 2, true>), grid, dim3(256), 0, st, shots, bb);
      return hipGetLastError();
    }
  }
  if (lm == 0)
    hipLaunchKernelGGL((k_sweep_block_batch<S, 0, false>), grid, dim3(256), 0, st, shots, bb);
  else if (lm == 1)
    hipLaunchKernelGGL((k_sweep_block_batch<S, 1, false>), grid, dim3(256), 0, st, shots, bb);
  else
    hipLaunchKernelGGL((k_sweep_block_batch<S, 2, false>), grid, dim3(256), 0, st, shots, bb);
  return hipGetLastError();
}

hipError_t launch_sweep_block_batch(const BatchShot* shots, const BlockBatch& bb, int storage,
                                    int lm, bool duo, hipStream_t s) {
  if (bb.n < 1 || bb.n > kBlockMembers || bb.begin[bb.n] < 1 ||
      (duo && (lm == 1 || storage == 0 || storage == 3)))
    return hipErrorInvalidValue;
  switch (storage) {
    case 0: return block_batch_s<StF32>(shots, bb, lm, duo, s);
    case 1: return block_batch_s<StBF16>(shots, bb, lm, duo, s);
    case 2: return block_batch_s<StF16>(shots, bb, lm, duo, s);
    case 3: return block_batch_s<StBF16SR>(shots, bb, lm, duo, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_record_last(const BatchShot* shots, const BatchState* state, int n, int storage,
                              hipStream_t s) {
  const dim3 grid((unsigned)n);
  switch (storage) {
    case 0: hipLaunchKernelGGL(k_record_last<StF32>, grid, dim3(256), 0, s, shots, state); break;
    case 1:
    case 3: hipLaunchKernelGGL(k_record_last<StBF16>, grid, dim3(256), 0, s, shots, state); break;
    case 2: hipLaunchKernelGGL(k_record_last<StF16>, grid, dim3(256), 0, s, shots, state); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace wave
