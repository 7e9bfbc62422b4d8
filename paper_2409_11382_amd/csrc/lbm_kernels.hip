// HIP kernels of the batched Biot LBM engine for gfx950 (CDNA4, 64-wide waves).
//
// Elastic sweep ("tile sweep"): a 256-thread block owns a tile of 60 x 12
// output cells of one level of one problem.  Its 64 lanes cover 64 adjacent
// columns (the 60 outputs and two halo columns on each side); each wave owns
// two pairs of rows of the 16-row region (12 outputs and two halo rows above
// and below), so every load of the block is issued at once.
//   phase 1: populations of the region (plus the prolongated coarse correction)
//            and D(g) (eq. LBM:divergence) into LDS;
//   phase 2: self-force (eq. MG:selfdependence) and collision (Algorithm 2,
//            Tables 2-3) of the 14 collision rows into LDS;
//   phase 3: pull-stream with every boundary rule of Sec. 3.6, then the mode's
//            output: under-relaxed update (eq. MG:smoother), the application
//            itself, or residual and 2x2 full-sum restriction
//            (eqs. LBM:residual, MG:restriction) with FP64 norm partials.
// The flow step uses the same tiling with a one-row halo.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lbm_engine.h"

namespace biot {

// Direction tables as compile-time functions: every caller indexes them with
// an unrolled loop counter, so all population indices fold to constants.
__device__ constexpr int cx8(int q) { return q == 0 || q == 4 || q == 7 ? 1 : (q == 2 || q == 5 || q == 6 ? -1 : 0); }
__device__ constexpr int cy8(int q) { return q == 1 || q == 4 || q == 5 ? 1 : (q == 3 || q == 6 || q == 7 ? -1 : 0); }
__device__ constexpr int opp8(int q) { return q < 4 ? (q + 2) % 4 : 4 + (q - 2) % 4; }
__device__ constexpr int mx8(int q) {  // (-cx, cy)
  return q == 0 ? 2 : q == 2 ? 0 : q == 4 ? 5 : q == 5 ? 4 : q == 6 ? 7 : q == 7 ? 6 : q;
}
__device__ constexpr int my8(int q) {  // (cx, -cy)
  return q == 1 ? 3 : q == 3 ? 1 : q == 4 ? 7 : q == 7 ? 4 : q == 5 ? 6 : q == 6 ? 5 : q;
}
__device__ constexpr int cx9(int i) { return i == 1 || i == 5 || i == 8 ? 1 : (i == 3 || i == 6 || i == 7 ? -1 : 0); }
__device__ constexpr int cy9(int i) { return i == 2 || i == 5 || i == 6 ? 1 : (i == 4 || i == 7 || i == 8 ? -1 : 0); }
__device__ constexpr int opp9(int i) { return i == 0 ? 0 : (i < 5 ? 1 + (i + 1) % 4 : 5 + (i - 3) % 4); }
__device__ constexpr int mx9(int i) {
  return i == 1 ? 3 : i == 3 ? 1 : i == 5 ? 6 : i == 6 ? 5 : i == 7 ? 8 : i == 8 ? 7 : i;
}
__device__ constexpr int my9(int i) {
  return i == 2 ? 4 : i == 4 ? 2 : i == 5 ? 8 : i == 8 ? 5 : i == 6 ? 7 : i == 7 ? 6 : i;
}
__device__ constexpr double w9(int i) { return i == 0 ? 4.0 / 9 : (i < 5 ? 1.0 / 9 : 1.0 / 36); }

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// launches of the adaptive schedule: skip when a stop flag is set, or (need)
// run only when the step before stopped normally
__device__ __forceinline__ bool gated_off(const int* skip, const int* need) {
  return (skip && *skip) || (need && *need != 1);
}

// ======================================================================
// elastic tile sweep
// ======================================================================
template <typename T, typename Tc, int MODE, bool SHIFT>
__global__ __launch_bounds__(256) void k_tsweep(SweepL a) {
  if (gated_off(a.skip, a.need)) return;  // uniform over the grid
  constexpr int TY = kTileY;     // output rows
  constexpr int RR = TY + 4;     // region rows (two halo rows each side)
  constexpr int CR = TY + 2;     // collision rows
  constexpr int NK = RR / 4;     // rows owned by each wave (two pairs)
  __shared__ T sD[RR][kWave];
  __shared__ T sS[8][CR][kWave];
  // shifted storage: the displacement reference, two FP64 planes or (in the
  // same bytes) two FP32 planes
  __shared__ std::conditional_t<SHIFT, double, T> sEd[SHIFT ? 2 : 1][SHIFT ? CR : 1][kWave];
  float (*sEf)[SHIFT ? CR : 1][kWave] = reinterpret_cast<float (*)[SHIFT ? CR : 1][kWave]>(sEd);
  __shared__ double sRed[8];

  const int2 te = a.tiles[blockIdx.x];
  const ProbD& P = a.probs[te.x];
  const int l = P.L - a.depth;
  const LevelD& V = P.lv[l];
  const int nx = V.nx, ny = V.ny, pitch = V.pitch;
  const int64_t plane = V.plane;
  const int tx = te.y % V.tiles_x, ty = te.y / V.tiles_x;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int x = tx * kTileX - kHalo + lane;
  const int y0 = ty * TY;
  const bool perx = P.el[kLeft] == kElPeriodic, pery = P.el[kBottom] == kElPeriodic;
  const bool col_ok = x >= -kHalo && x < nx + kHalo;
  const int gx = col_ok ? ghost_map(x, nx, perx) : 0;
  const bool out_lane = lane >= kHalo && lane < kWave - kHalo && x < nx;
  const T* gin = a.in_sel == 2 ? nullptr : (const T*)(a.in_sel ? V.gB : V.gA);
  T* gout = (T*)(a.out_sel ? V.gB : V.gA);
  const T* rr = (const T*)V.r;
  const bool fine = a.depth == 0;
  const T* Ft = fine ? (const T*)P.Ft : nullptr;
  const bool pro = a.prolong && l > 1;
  const Tc* ec = pro ? (const Tc*)P.lv[l - 1].gA : nullptr;
  const int cpitch = l > 1 ? P.lv[l - 1].pitch : 0;
  const int64_t cplane = l > 1 ? P.lv[l - 1].plane : 0;
  Tc* rc = (MODE == kRestrict && l > 1) ? (Tc*)P.lv[l - 1].r : nullptr;
  const void* eref = SHIFT ? (a.eref_in ? P.eref2 : P.eref) : nullptr;
  const bool r64 = P.ref64 != 0;  // reference precision (uniform)
  ElConst<T> k;
  k.om_s = T(P.om_s);
  k.om_d = T(P.om_d);
  k.beta22 = T(P.beta22);
  k.kD = T(P.kD);
  k.cstar = T(P.cstar);
  k.gamma = T(P.gamma);
  // lagged self-force (Algorithm 1 read with eq. source:implicit): the
  // divergence of the previous pseudo-time step comes from dlag[lag_rd]; the
  // input's own goes to the other plane for the next application
  const T* dlag_in = (MODE == kSmooth && a.lag == 2) ? (const T*)P.dlag[a.lag_rd] : nullptr;
  T* dlag_out = (MODE == kSmooth && a.lag != 0) ? (T*)P.dlag[a.lag == 1 ? 0 : 1 - a.lag_rd] : nullptr;

  T G[NK][8], Rv[NK][8], Fx[NK], Fy[NK];

  // ---- phase 1: load the region, D(g)
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const int j = 2 * (w + 4 * (kk >> 1)) + (kk & 1);
    const int y = y0 - kHalo + j;
    const bool ok = col_ok && y >= -kHalo && y < ny + kHalo;
    const int gy = ok ? ghost_map(y, ny, pery) : 0;
    const int64_t idx = (int64_t)gy * pitch + gx;
#pragma unroll
    for (int q = 0; q < 8; ++q) G[kk][q] = (ok && gin) ? gin[q * plane + idx] : T(0);
    if (ok && pro) {
      const int64_t cidx = (int64_t)(gy >> 1) * cpitch + (gx >> 1);
#pragma unroll
      for (int q = 0; q < 8; ++q) G[kk][q] += T(ec[q * cplane + cidx]);
    }
    if (dlag_in)
      sD[j][lane] = ok ? dlag_in[idx] : T(0);
    else
      sD[j][lane] = k.kD * el_ms(G[kk]);
    const bool crow = j >= 1 && j < CR + 1;
#pragma unroll
    for (int q = 0; q < 8; ++q) Rv[kk][q] = (ok && crow && rr) ? rr[q * plane + idx] : T(0);
    Fx[kk] = (ok && crow && Ft) ? Ft[idx] : T(0);
    Fy[kk] = (ok && crow && Ft) ? Ft[plane + idx] : T(0);
    if (SHIFT && crow) {
      if (r64) {
        sEd[0][j - 1][lane] = ok ? ((const double*)eref)[idx] : 0.0;
        sEd[1][j - 1][lane] = ok ? ((const double*)eref)[plane + idx] : 0.0;
      } else {
        sEf[0][j - 1][lane] = ok ? ((const float*)eref)[idx] : 0.f;
        sEf[1][j - 1][lane] = ok ? ((const float*)eref)[plane + idx] : 0.f;
      }
    }
  }
  __syncthreads();

  // ---- phase 2: self-force and collision of the collision rows
  const int lm = clampi(lane - 1, 0, kWave - 1), lp = clampi(lane + 1, 0, kWave - 1);
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const int j = 2 * (w + 4 * (kk >> 1)) + (kk & 1);
    if (j >= 1 && j < CR + 1) {
      T v[3][3] = {{sD[j - 1][lm], sD[j - 1][lane], sD[j - 1][lp]},
                   {sD[j][lm], sD[j][lane], sD[j][lp]},
                   {sD[j + 1][lm], sD[j + 1][lane], sD[j + 1][lp]}};
      T gx_, gy_;
      grad_c(v, gx_, gy_);
      T u[8], s[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) u[q] = G[kk][q] - Rv[kk][q];
      el_collide(u, Fx[kk] + k.cstar * gx_, Fy[kk] + k.cstar * gy_, k, s);
#pragma unroll
      for (int q = 0; q < 8; ++q) sS[q][j - 1][lane] = s[q];
    }
  }
  __syncthreads();

  // ---- phase 3: pull-stream, boundary rules, output
  const T gam = k.gamma, omg = T(1) - k.gamma;
  double acc_r = 0.0, acc_g = 0.0;
  T racc[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) racc[q] = T(0);
  const bool wl = out_lane && x == 0 && !perx;
  const bool wr = out_lane && x == nx - 1 && !perx;
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const int j = 2 * (w + 4 * (kk >> 1)) + (kk & 1);
    if (j < 2 || j >= TY + 2) continue;   // wave-uniform
    const int y = y0 + j - 2;
    const bool valid = out_lane && y < ny;
    const int c = j - 1;                  // collision row index of row j
    const int lc = valid ? lane : 2;      // keep LDS indices in range on idle lanes
    T gi[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) gi[q] = sS[q][c - cy8(q)][lc - cx8(q)];
    double ex = 0.0, ey = 0.0;
    if (SHIFT && r64) {  // reference differences in FP64, rounded once
      ex = sEd[0][c][lc];
      ey = sEd[1][c][lc];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        gi[q] += T(el_geq<double>(q, sEd[0][c - cy8(q)][lc - cx8(q)] - ex, sEd[1][c - cy8(q)][lc - cx8(q)] - ey));
    } else if (SHIFT) {
      const float exf = sEf[0][c][lc], eyf = sEf[1][c][lc];
      ex = exf;
      ey = eyf;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        gi[q] += T(el_geq<float>(q, sEf[0][c - cy8(q)][lc - cx8(q)] - exf, sEf[1][c - cy8(q)][lc - cx8(q)] - eyf));
    }
    // wall rules against the reference: FP64 with FP64 references, else in
    // the population precision. Mirror rules take the source's reference
    // (population qm) minus this cell's (population qq); bounce-back rules
    // twice this cell's.
    auto mirror = [&](int qm, int qq, int cc, int ll) -> T {
      if constexpr (SHIFT) {
        if (r64) return T(el_geq<double>(qm, sEd[0][cc][ll], sEd[1][cc][ll]) - el_geq<double>(qq, ex, ey));
        return el_geq<T>(qm, T(sEf[0][cc][ll]), T(sEf[1][cc][ll])) - el_geq<T>(qq, T(ex), T(ey));
      }
      return T(0);
    };
    auto twice_own = [&](int qq) -> T {
      return r64 ? T(2.0 * el_geq<double>(qq, ex, ey)) : T(2) * el_geq<T>(qq, T(ex), T(ey));
    };
    const bool wb = valid && y == 0 && !pery;
    const bool wt = valid && y == ny - 1 && !pery;
    if (wl || wr || wb || wt) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int cx = cx8(q), cy = cy8(q);
        const bool ox = (cx > 0 && wl) || (cx < 0 && wr);
        const bool oy = (cy > 0 && wb) || (cy < 0 && wt);
        if (!(ox || oy)) continue;
        const int elx = cx > 0 ? P.el[kLeft] : P.el[kRight];
        const int ely = cy > 0 ? P.el[kBottom] : P.el[kTop];
        T v = T(0);
        bool usex = false, half = false;
        if (ox && oy) {
          if (elx == kElSymmetry && ely == kElSymmetry) {
            // corner between two mirrors: diagonal bounce-back
            v = sS[opp8(q)][c][lc];
            if (SHIFT) v -= twice_own(q);
          } else {
            usex = ely == kElSymmetry;
            half = true;
          }
        } else if (ox) {
          usex = true;
          if (elx == kElSymmetry) {  // mirror image: own column, row y - cy
            v = sS[mx8(q)][c - cy][lc];
            if (SHIFT) v += mirror(mx8(q), q, c - cy, lc);
          } else {
            half = true;
          }
        } else {
          if (ely == kElSymmetry) {  // mirror image: column x - cx, own row
            v = sS[my8(q)][c][lc - cx];
            if (SHIFT) v += mirror(my8(q), q, c, lc - cx);
          } else {
            half = true;
          }
        }
        if (half) {  // halfway rules at the cell itself
          const int type = usex ? elx : ely;
          const double* bc = fine ? (usex ? (cx > 0 ? P.elbc[kLeft] : P.elbc[kRight])
                                          : (cy > 0 ? P.elbc[kBottom] : P.elbc[kTop]))
                                  : nullptr;
          const int bidx = usex ? y : x;
          const double add = bc ? bc[8 * bidx + q] : 0.0;
          const T o = sS[opp8(q)][c][lc];
          if (type == kElDirichlet) {
            if (SHIFT && r64)  // the wall term and the reference's share in FP64, rounded once
              v = o + T(add - 2.0 * el_geq<double>(q, ex, ey));
            else
              v = o + T(add) - (SHIFT ? twice_own(q) : T(0));
          } else {
            v = -o + T(add);  // traction
          }
        }
        gi[q] = v;
      }
    }
    if (a.partials && valid) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const double rho = double(G[kk][q]) - double(gi[q]);
        double gf = double(G[kk][q]);
        if (SHIFT) gf += el_geq<double>(q, ex, ey);
        acc_r += rho * rho;
        acc_g += gf * gf;
      }
    }
    const int64_t oidx = (int64_t)y * pitch + x;
    if (MODE == kSmooth) {
      if (valid) {
#pragma unroll
        for (int q = 0; q < 8; ++q) gout[q * plane + oidx] = omg * G[kk][q] + gam * gi[q];
        if (dlag_out) dlag_out[oidx] = k.kD * el_ms(G[kk]);
      }
    } else if (MODE == kApply) {
      if (valid) {
#pragma unroll
        for (int q = 0; q < 8; ++q) gout[q * plane + oidx] = gi[q];
      }
    } else {
      // residual, summed over lane pairs (x, x+1) and over the row pair
      T rx[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const T rho = valid ? G[kk][q] - gi[q] : T(0);
        rx[q] = rho + from_right(rho);
      }
      if ((kk & 1) == 0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) racc[q] = rx[q];
      } else if (valid && (x & 1) == 0 && rc) {
        const int64_t cidx = (int64_t)(y >> 1) * cpitch + (x >> 1);
#pragma unroll
        for (int q = 0; q < 8; ++q) rc[q * cplane + cidx] = Tc(racc[q] + rx[q]);
      }
    }
  }
  if (a.partials) {
    acc_r = wave_sum(acc_r);
    acc_g = wave_sum(acc_g);
    if (lane == 0) {
      sRed[2 * w] = acc_r;
      sRed[2 * w + 1] = acc_g;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      P.partials[2 * te.y] = (sRed[0] + sRed[2]) + (sRed[4] + sRed[6]);
      P.partials[2 * te.y + 1] = (sRed[1] + sRed[3]) + (sRed[5] + sRed[7]);
    }
  }
}

template <typename T, typename Tc, int MODE, bool SHIFT>
hipError_t launch_tsweep(const SweepL& a, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_tsweep<T, Tc, MODE, SHIFT>), dim3(ntiles), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ======================================================================
// several applications in one launch
// ======================================================================
// Same arithmetic as APPS k_tsweep smoothing launches, followed (RES) by the
// residual/restriction launch on their result.  The tile loads a 64-column
// region with a halo of H = 2 A, A = APPS + RES (64 - 2H output columns,
// NW NK - 2H output rows); each wave keeps its NK rows in registers across the
// applications, whose valid region shrinks by 2 per application (D and
// collision need one neighbour, the pull one more).
// Walls: these launches are bound by one block's chain of dependent phases on
// depths of few cells, and nearly every block there holds a wall.  So the
// rules cost no branch, barrier or global load inside an application: the
// divergence's ghost is the wall cell itself (an index), a wall population is
// read from its mirror image or its opposite by a selected LDS offset, the
// reference's share joins the correction that every pull adds anyway, and the
// halfway rules' data wait in LDS.  Branches per lane over the wall types, a
// ghost-row pass behind its own barrier and loads of the data in every
// application cost 12 to 20% of a launch on depths of few cells.
// Launches in FP32 shifted (FP64), us: four applications at 64^2 11.2 (12.3),
// with the restriction 12.8 (14.9); pairs at 512^2 13.9 (17.5), with the
// restriction 18.5 (22.9); at 1024^2 33.8 (43.6) and 48.0 (74.0); at 2048^2 105
// and 164, the pair at 3.4 TB/s of HBM and half of the vector issue: two blocks
// a CU do not cover each other's loads and barriers fully.
// R64: shifted storage whose references may be FP64 (FP64 populations, or a
// problem above the size where FP32 references lose accuracy); without it the
// reference arithmetic is FP32 only.
// WIDE: planes of 4 GiB and more (finest level only), whose cells lie beyond a
// 32-bit byte offset: a wave's row, which is one row there, joins the scalar
// base, and the lane's offset lies within it.  32768 x 16384 cells in FP32
// shifted: 13.6 ms a pair; 21.0 with 64-bit offsets per lane, whose registers
// leave one block on a CU.
template <typename T, typename Tc, bool FINE, bool SHIFT, int APPS, bool RES, bool ALT, bool R64, bool WIDE = false>
__global__ __launch_bounds__((kWave * sweepn_waves<T, SHIFT, APPS + RES, ALT>())) void k_tsweep2(SweepL a) {
  if (gated_off(a.skip, a.need)) return;  // uniform over the grid
  constexpr int A = APPS + (RES ? 1 : 0);
  constexpr int NW = sweepn_waves<T, SHIFT, A, ALT>();
  constexpr int NK = sweepn_rows<T, SHIFT, A, ALT>();
  constexpr int H = 2 * A;         // halo
  constexpr int RX = sweepn_cols<A, ALT>();  // region columns
  constexpr int S = kWave / RX;    // rows per wave and row index kk
  constexpr int RR = NW * NK * S;  // region rows
  constexpr int TY = RR - 2 * H;   // output rows
  constexpr int TXO = RX - 2 * H;
  __shared__ T sD[RR][RX];
  __shared__ T sS[8][RR - 2][RX];
  // shifted storage: the displacement reference, two FP64 planes (ex, ey) or,
  // in the same bytes, four FP32 planes (ex, ey, ex + ey, ey - ex)
  __shared__ std::conditional_t<SHIFT, double, T> sEd[SHIFT ? 2 : 1][SHIFT ? RR : 1][RX];
  float (*sEf)[SHIFT ? RR : 1][RX] = reinterpret_cast<float (*)[SHIFT ? RR : 1][RX]>(sEd);
  __shared__ double sRed[2 * NW];
  // data of the halfway rules (finest level): the three populations entering
  // through the bottom and the top at each region column, and through the left
  // and the right at each region row
  using BcT = std::conditional_t<R64, double, T>;
  __shared__ BcT sBy[2][3][FINE ? RX : 1];
  __shared__ BcT sBx[2][3][FINE ? RR : 1];
  constexpr int PS = (RR - 2) * RX;  // plane stride of sS
  static_assert(!WIDE || (FINE && S == 1), "a wave holds one row of the finest level");

  const int2 te = a.tiles[blockIdx.x];
  // the entry names the level too: one dependent descriptor load less (1.5 us of
  // a 512^2 step)
  const ProbD& P = a.probs[te.x & ((1 << kTileLevelShift) - 1)];
  const int l = te.x >> kTileLevelShift;
  const LevelD& V = P.lv[l];
  const int nx = V.nx, ny = V.ny, pitch = V.pitch;
  const int64_t plane = V.plane;
  const int sh = V.tile_shift[A];  // tile column and row packed by the host: no division here
  const int tx = te.y & ((1 << sh) - 1), ty = te.y >> sh;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int col = lane & (RX - 1), sub = lane / RX;  // a wave holds S rows of RX cells
  const int x = tx * TXO - H + col;
  const int y0 = ty * TY;
  const bool perx = P.el[kLeft] == kElPeriodic, pery = P.el[kBottom] == kElPeriodic;
  // ghosts: periodic copies; beyond a wall any cell (no valid cell reads them:
  // the wall cells' stencils stop at the wall, see the rules below)
  const int gx = perx ? wrap_index(x, nx, RX) : clampi(x, 0, nx - 1);
  const bool xreal = x >= -H && x < nx + H && (perx || (x >= 0 && x < nx));
  const bool zero_in = a.in_sel == 2;
  const GPtr<T> gin = gptr<T>(a.in_sel ? V.gB : V.gA), gout = gptr<T>(a.out_sel ? V.gB : V.gA);
  const bool pro = a.prolong && l > 1;
  const LevelD& C = P.lv[l > 1 ? l - 1 : l];  // the coarser level
  const int cpitch = C.pitch;
  const int64_t cplane = C.plane;
  const GPtr<Tc> cr = gptr<Tc>(C.r);  // read before any store: a scalar load
  const void* eref = SHIFT ? (a.eref_in ? P.eref2 : P.eref) : nullptr;
  const bool r64 = R64 && P.ref64 != 0;  // reference precision (uniform)
  ElConst<T> k;
  k.om_s = T(P.om_s);
  k.om_d = T(P.om_d);
  k.beta22 = T(P.beta22);
  k.kD = T(P.kD);
  k.cstar = T(P.cstar);
  k.gamma = T(P.gamma);

  T G[NK][8];
  T Rv[FINE ? 1 : NK][8];
  T Fx[FINE ? NK : 1], Fy[FINE ? NK : 1];

  // ---- load the region: every lane loads, from 32-bit byte offsets.  With each
  // load in a branch of its own, a 64-bit address per lane and ghosts and tiles
  // found by integer division, the chain before the first application is 650
  // instructions, in this form 400, and a launch about 8% shorter at every size.
  // The loads of every row are issued before the first value is used: the
  // reference's way to LDS and the coarse correction would make each row wait
  // for its own (5% of a pair)
  uint32_t off[NK], coff[NK];  // byte offset of the row's cell in a plane, of its coarse cell in a coarse plane
  int64_t row[WIDE ? NK : 1];  // WIDE: the row's first cell, and off counts from there
  auto at = [&](auto base, int kk) {
    if constexpr (WIDE)
      return base + row[kk];
    else
      return base;
  };
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const int j = (w + NW * kk) * S + sub;
    const int y = y0 - H + j;
    const int gy = pery ? wrap_index(y, ny, RR) : clampi(y, 0, ny - 1);
    if constexpr (WIDE) row[kk] = (int64_t)__builtin_amdgcn_readfirstlane(gy) * pitch;
    off[kk] = ((WIDE ? 0u : (uint32_t)gy * (uint32_t)pitch) + (uint32_t)gx) * (uint32_t)sizeof(T);
    coff[kk] = ((uint32_t)(gy >> 1) * (uint32_t)cpitch + (uint32_t)(gx >> 1)) * (uint32_t)sizeof(Tc);
  }
  double e64[R64 ? NK : 1][2];
  float e32[SHIFT ? NK : 1][2];
  // row by row in FP32 (2048^2 pairs 104.6 us, plane by plane 107.0), plane by
  // plane in FP64 (1024^2 43.8, row by row 44.5)
  constexpr bool ROWS = sizeof(T) == 4;
  if (!ROWS) {
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        G[kk][q] = zero_in ? T(0) : gload(at(gin + q * plane, kk), off[kk]);
        if (!FINE) Rv[FINE ? 0 : kk][q] = gload(gptr<T>(V.r) + q * plane, off[kk]);
      }
  }
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    if (ROWS) {
#pragma unroll
      for (int q = 0; q < 8; ++q) G[kk][q] = T(0);
      if (!zero_in) {
#pragma unroll
        for (int q = 0; q < 8; ++q) G[kk][q] = gload(at(gin + q * plane, kk), off[kk]);
      }
    }
    if (FINE) {
      const GPtr<T> Ft = gptr<T>(P.Ft);
      Fx[FINE ? kk : 0] = gload(at(Ft, kk), off[kk]);
      Fy[FINE ? kk : 0] = gload(at(Ft + plane, kk), off[kk]);
    } else if (ROWS) {
      const GPtr<T> rr = gptr<T>(V.r);
#pragma unroll
      for (int q = 0; q < 8; ++q) Rv[FINE ? 0 : kk][q] = gload(rr + q * plane, off[kk]);
    }
    const uint32_t cell = off[kk] / (uint32_t)sizeof(T);
    if (R64 && r64) {
      const GPtr<double> e = gptr<double>(eref);
      e64[R64 ? kk : 0][0] = gload(at(e, kk), cell * 8u);
      e64[R64 ? kk : 0][1] = gload(at(e + plane, kk), cell * 8u);
    } else if (SHIFT) {
      const GPtr<float> e = gptr<float>(eref);
      e32[SHIFT ? kk : 0][0] = gload(at(e, kk), cell * 4u);
      e32[SHIFT ? kk : 0][1] = gload(at(e + plane, kk), cell * 4u);
    }
  }
  if (pro) {
    const GPtr<Tc> ec = gptr<Tc>(C.gA);
    Tc E[NK][8];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int q = 0; q < 8; ++q) E[kk][q] = gload(ec + q * cplane, coff[kk]);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int q = 0; q < 8; ++q) G[kk][q] += T(E[kk][q]);
  }
  if (SHIFT) {
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const int j = (w + NW * kk) * S + sub;
      if (r64) {
        sEd[0][j][col] = e64[R64 ? kk : 0][0];
        sEd[1][j][col] = e64[R64 ? kk : 0][1];
      } else {
        const float ex = e32[SHIFT ? kk : 0][0], ey = e32[SHIFT ? kk : 0][1];
        sEf[0][j][col] = ex;
        sEf[1][j][col] = ey;
        sEf[2][j][col] = ex + ey;
        sEf[3][j][col] = ey - ex;
      }
    }
  }

  // does the pull region (columns and rows [2, RX - 2) x [2, RR - 2)) hold a
  // wall cell?  Tiles that hold none skip every boundary rule.
  const int xa = tx * TXO - H + 2, xb = xa + RX - 5, ya = y0 - H + 2, yb = ya + RR - 5;
  const bool atL = !perx && xa <= 0 && xb >= 0, atR = !perx && xa <= nx - 1 && xb >= nx - 1;
  const bool atB = !pery && ya <= 0 && yb >= 0, atT = !pery && ya <= ny - 1 && yb >= ny - 1;
  const bool bnd = atL || atR || atB || atT;
  // a collided row beside the bottom or top wall (its divergence has a ghost)
  const bool dwall = !pery && (y0 - H + 1 <= 0 || y0 - H + RR - 2 >= ny - 1);
  // wall rules by side (uniform): symmetry walls mirror, the others take a
  // halfway rule at the cell itself (Dirichlet bounces back, traction
  // anti-bounces back) with the wall's data
  const int elL = P.el[kLeft], elR = P.el[kRight], elB = P.el[kBottom], elT = P.el[kTop];
  const bool symL = elL == kElSymmetry, symR = elR == kElSymmetry, symB = elB == kElSymmetry, symT = elT == kElSymmetry;
  const bool half = (atL && !symL) || (atR && !symR) || (atB && !symB) || (atT && !symT);
  if (FINE && half) {
    for (int i = threadIdx.x; i < 6 * RX + 6 * RR; i += kWave * NW) {
      const bool isy = i < 6 * RX;
      const int e = isy ? i : i - 6 * RX, n = isy ? RX : RR;
      const int sd = e / (3 * n), m = e / n % 3, at = e % n;  // side, population of the side, column or row
      // populations entering: bottom 1 4 5, top 3 6 7, left 0 4 7, right 2 5 6
      const int q = isy ? (sd ? (m == 0 ? 3 : m + 5) : (m == 0 ? 1 : m + 3))
                        : (sd ? (m == 0 ? 2 : m + 4) : (m == 0 ? 0 : 3 * m + 1));
      const double* bc = P.elbc[isy ? (sd ? kTop : kBottom) : (sd ? kRight : kLeft)];
      const int z = (isy ? tx * TXO : y0) - H + at, nz = isy ? nx : ny;
      const bool pz = isy ? perx : pery;
      const bool on = bc && (pz ? z >= -H && z < nz + H : z >= 0 && z < nz);
      const BcT v = on ? BcT(bc[8 * (int64_t)ghost_map(z, nz, pz) + q]) : BcT(0);
      if (isy)
        sBy[sd][m][FINE ? at : 0] = v;
      else
        sBx[sd][m][FINE ? at : 0] = v;
    }
  }

  const T gam = k.gamma, omg = T(1) - k.gamma;
  const double inv_gam = 1.0 / P.gamma;
  // columns of the divergence's neighbours; at a wall the ghost holds the even
  // reflection, which is the wall cell itself
  const int lm = (!perx && x == 0) ? col : clampi(col - 1, 0, RX - 1);
  const int lp = (!perx && x == nx - 1) ? col : clampi(col + 1, 0, RX - 1);
  double acc_r = 0.0, acc_g = 0.0;
  // shifted storage: the pull's correction per direction, the source's
  // reference minus this cell's in the rest equilibrium of the population
  // (el_geq); constant during the launch, formed in the first application
  T Cr[SHIFT ? NK : 1][8];

#pragma unroll
  for (int app = 0; app < A; ++app) {
    const int e = 2 * app;  // rows / columns [e, RR - e) hold a valid iterate
    // smoothing applications stream gamma times the post-collision
    // populations, so the blend (1 - gamma) g + gamma g_in is one FMA; the
    // residual application streams them unscaled
    const bool resid = RES && app == A - 1;
    const T sc = resid ? T(1) : gam;
    // ---- D(g)
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const int j = (w + NW * kk) * S + sub;
      if (j >= e && j < RR - e) sD[j][col] = k.kD * el_ms(G[kk]);
    }
    __syncthreads();
    // ---- self-force and collision
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const int j = (w + NW * kk) * S + sub;
      if (j >= e + 1 && j < RR - e - 1) {
        T v[3][3] = {{T(0), T(0), T(0)}, {sD[j][lm], T(0), sD[j][lp]}, {T(0), T(0), T(0)}};  // the centre is not used
        if (!dwall) {
          v[0][0] = sD[j - 1][lm], v[0][1] = sD[j - 1][col], v[0][2] = sD[j - 1][lp];
          v[2][0] = sD[j + 1][lm], v[2][1] = sD[j + 1][col], v[2][2] = sD[j + 1][lp];
        } else {
          const int y = y0 - H + j;
          const int jm = (!pery && y == 0) ? j : j - 1, jp = (!pery && y == ny - 1) ? j : j + 1;
          v[0][0] = sD[jm][lm], v[0][1] = sD[jm][col], v[0][2] = sD[jm][lp];
          v[2][0] = sD[jp][lm], v[2][1] = sD[jp][col], v[2][2] = sD[jp][lp];
        }
        T gx_, gy_;
        grad_c(v, gx_, gy_);
        T u[8], s8[8];
        T fx = k.cstar * gx_, fy = k.cstar * gy_;
        if (FINE) {
          fx += Fx[kk];
          fy += Fy[kk];
#pragma unroll
          for (int q = 0; q < 8; ++q) u[q] = G[kk][q];
        } else {
#pragma unroll
          for (int q = 0; q < 8; ++q) u[q] = G[kk][q] - Rv[kk][q];
        }
        el_collide(u, fx, fy, k, s8, sc);
#pragma unroll
        for (int q = 0; q < 8; ++q) sS[q][j - 1][col] = s8[q];
      }
    }
    __syncthreads();
    // ---- pull-stream with the boundary rules, under-relaxation
    const bool pl = col >= e + 2 && col < RX - e - 2;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const int j = (w + NW * kk) * S + sub;
      if (j < e + 2 || j >= RR - e - 2) continue;  // uniform over each row of a wave
      const int y = y0 - H + j;
      const int c = j - 1;
      const int lc = pl ? col : 4;  // keep LDS indices in range on idle lanes
      bool wl = false, wr = false, wb = false, wt = false;
      if (bnd) {
        const bool yreal = pery ? (y >= -H && y < ny + H) : (y >= 0 && y < ny);
        const bool real = pl && xreal && yreal;
        wl = real && !perx && x == 0;
        wr = real && !perx && x == nx - 1;
        wb = real && !pery && y == 0;
        wt = real && !pery && y == ny - 1;
      }
      // the value a population arrives from: the neighbour's, at a symmetry
      // wall the mirror image (own column or row), at a halfway rule and where
      // two walls meet this cell's opposite population
      T gi[8];
      const T* sp = &sS[0][c][lc];
      if (!bnd) {
#pragma unroll
        for (int q = 0; q < 8; ++q) gi[q] = sp[q * PS - cy8(q) * RX - cx8(q)];
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int cx = cx8(q), cy = cy8(q), back = opp8(q) * PS;
          int off = q * PS - cy * RX - cx;
          const int offx = (cx > 0 ? symL : symR) ? mx8(q) * PS - cy * RX : back;
          const int offy = (cy > 0 ? symB : symT) ? my8(q) * PS - cx : back;
          const bool ox = cx > 0 ? wl : wr, oy = cy > 0 ? wb : wt;
          if (cx != 0 && cy != 0)
            off = ox ? (oy ? back : offx) : (oy ? offy : off);
          else
            off = cx != 0 ? (ox ? offx : off) : (oy ? offy : off);
          gi[q] = sp[off];
        }
      }
      // own reference, read from LDS where a rule needs it (FP64 registers
      // per row would cost occupancy)
      auto own_x = [&]() { return r64 ? sEd[0][j][col] : double(sEf[0][j][col]); };
      auto own_y = [&]() { return r64 ? sEd[1][j][col] : double(sEf[1][j][col]); };
      if (SHIFT) {
        if (app == 0 && r64) {  // rows and columns pulled later are a subset
          // reference differences in FP64, rounded once
          const double ex = sEd[0][j][col], ey = sEd[1][j][col];
          const double sp = ex + ey, sm = ey - ex;
          const double third = 1.0 / 3.0, twelfth = 1.0 / 12.0;
          Cr[kk][0] = T(third * (sEd[0][j][lc - 1] - ex));
          Cr[kk][1] = T(third * (sEd[1][j - 1][lc] - ey));
          Cr[kk][2] = T(-third * (sEd[0][j][lc + 1] - ex));
          Cr[kk][3] = T(-third * (sEd[1][j + 1][lc] - ey));
          Cr[kk][4] = T(twelfth * ((sEd[0][j - 1][lc - 1] + sEd[1][j - 1][lc - 1]) - sp));
          Cr[kk][5] = T(twelfth * ((sEd[1][j - 1][lc + 1] - sEd[0][j - 1][lc + 1]) - sm));
          Cr[kk][6] = T(-twelfth * ((sEd[0][j + 1][lc + 1] + sEd[1][j + 1][lc + 1]) - sp));
          Cr[kk][7] = T(-twelfth * ((sEd[1][j + 1][lc - 1] - sEd[0][j + 1][lc - 1]) - sm));
        } else if (app == 0) {  // FP32 reference
          const float exf = sEf[0][j][col], eyf = sEf[1][j][col];
          const float sp = exf + eyf, sm = eyf - exf;
          const float third = 1.0f / 3.0f, twelfth = 1.0f / 12.0f;
          Cr[kk][0] = T(third * (sEf[0][j][lc - 1] - exf));
          Cr[kk][1] = T(third * (sEf[1][j - 1][lc] - eyf));
          Cr[kk][2] = T(-third * (sEf[0][j][lc + 1] - exf));
          Cr[kk][3] = T(-third * (sEf[1][j + 1][lc] - eyf));
          Cr[kk][4] = T(twelfth * (sEf[2][j - 1][lc - 1] - sp));
          Cr[kk][5] = T(twelfth * (sEf[3][j - 1][lc + 1] - sm));
          Cr[kk][6] = T(-twelfth * (sEf[2][j + 1][lc + 1] - sp));
          Cr[kk][7] = T(-twelfth * (sEf[3][j + 1][lc - 1] - sm));
        }
        if (app == 0 && bnd && (wl || wr || wb || wt)) {
          // wall populations: the source's reference in the population it is
          // read from minus this cell's (mirrors flip the component normal to
          // the wall, a halfway rule both), a halfway rule's data, and no
          // reference at all in a traction rule; once per launch
          using Rf = std::conditional_t<R64, double, float>;
          auto rx = [&](int jj, int ll) { return r64 ? Rf(sEd[0][jj][ll]) : Rf(sEf[0][jj][ll]); };
          auto ry = [&](int jj, int ll) { return r64 ? Rf(sEd[1][jj][ll]) : Rf(sEf[1][jj][ll]); };
          const Rf ex = rx(j, lc), ey = ry(j, lc);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const int cx = cx8(q), cy = cy8(q);
            const bool ox = (cx > 0 && wl) || (cx < 0 && wr), oy = (cy > 0 && wb) || (cy < 0 && wt);
            if (!(ox || oy)) continue;
            const bool hx = ox && !(cx > 0 ? symL : symR), hy = oy && !(cy > 0 ? symB : symT);
            if (hx || hy) {
              const int type = hy ? (cy > 0 ? elB : elT) : (cx > 0 ? elL : elR);
              const int my_ = cy > 0 ? (q == 1 ? 0 : q - 3) : (q == 3 ? 0 : q - 5);
              const int mx_ = cx > 0 ? (q == 0 ? 0 : (q - 1) / 3) : (q == 2 ? 0 : q - 4);
              const Rf add = FINE ? Rf(hy ? sBy[cy > 0 ? 0 : 1][cy != 0 ? my_ : 0][FINE ? lc : 0]
                                          : sBx[cx > 0 ? 0 : 1][cx != 0 ? mx_ : 0][FINE ? j : 0])
                                  : Rf(0);
              Cr[kk][q] = T(type == kElDirichlet ? add - Rf(2) * el_geq<Rf>(q, ex, ey) : add);
            } else {
              const int jj = oy ? j : j - cy, ll = ox ? lc : lc - cx;
              const Rf sx = rx(jj, ll), sy = ry(jj, ll);
              Cr[kk][q] = T(el_geq<Rf>(q, ox ? -sx : sx, oy ? -sy : sy) - el_geq<Rf>(q, ex, ey));
            }
          }
        }
      }
      if (half) {
        // the halfway rules' sign and (unshifted storage) data; where two
        // walls meet the bottom or top wall's rule wins, unless it mirrors
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int cx = cx8(q), cy = cy8(q);
          const bool hx = (cx > 0 && wl && !symL) || (cx < 0 && wr && !symR);
          const bool hy = (cy > 0 && wb && !symB) || (cy < 0 && wt && !symT);
          const bool neg = hy ? (cy > 0 ? elB : elT) == kElTraction : (hx && (cx > 0 ? elL : elR) == kElTraction);
          gi[q] = neg ? -gi[q] : gi[q];
          if (FINE && !SHIFT) {
            const int my_ = cy > 0 ? (q == 1 ? 0 : q - 3) : (q == 3 ? 0 : q - 5);
            const int mx_ = cx > 0 ? (q == 0 ? 0 : (q - 1) / 3) : (q == 2 ? 0 : q - 4);
            T add = T(0);
            if (cx != 0) add = hx ? T(sBx[cx > 0 ? 0 : 1][cx != 0 ? mx_ : 0][FINE ? j : 0]) : add;
            if (cy != 0) add = hy ? T(sBy[cy > 0 ? 0 : 1][cy != 0 ? my_ : 0][FINE ? lc : 0]) : add;
            gi[q] += sc * add;
          }
        }
      }
      if (SHIFT) {
#pragma unroll
        for (int q = 0; q < 8; ++q) gi[q] += sc * Cr[kk][q];
      }
      const bool out = pl && x >= 0 && x < nx && y >= 0 && y < ny && col >= H && col < RX - H &&
                       j >= H && j < RR - H;
      if (a.partials == 2 && app == 0 && out) {
        // the adaptive stopping test's norms of the launch's input, the
        // iterate the cycle starts from: ||g - S(g)||^2 and ||g||^2
        const double ex = SHIFT ? own_x() : 0.0, ey = SHIFT ? own_y() : 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const double rho = double(G[kk][q]) - double(gi[q]) * inv_gam;
          double gf = double(G[kk][q]);
          if (SHIFT) gf += el_geq<double>(q, ex, ey);
          acc_r += rho * rho;
          acc_g += gf * gf;
        }
      }
      if (RES && app == A - 1) {
        // residual of the smoothed iterate, summed over lane pairs (x, x + 1)
        // (both lanes of a pair lie in one row);
        // the row pairs are summed through LDS below
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const T rho = out ? G[kk][q] - gi[q] : T(0);
          G[kk][q] = rho + from_right(rho);
        }
      } else if (RES && app == A - 2) {
#pragma unroll
        for (int q = 0; q < 8; ++q) G[kk][q] = omg * G[kk][q] + gi[q];
        if (out) {
#pragma unroll
          for (int q = 0; q < 8; ++q) gstore(at(gout + q * plane, kk), off[kk], G[kk][q]);
        }
      } else if (!RES && app == A - 1) {
        if (a.partials == 1 && out) {
          const double ex = SHIFT ? own_x() : 0.0, ey = SHIFT ? own_y() : 0.0;
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const double rho = double(G[kk][q]) - double(gi[q]) * inv_gam;
            double gf = double(G[kk][q]);
            if (SHIFT) gf += el_geq<double>(q, ex, ey);
            acc_r += rho * rho;
            acc_g += gf * gf;
          }
        }
        if (out) {
          T gn[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) gn[q] = omg * G[kk][q] + gi[q];
          if (SHIFT && a.rebase_out) {
            // the re-basing kernel's step on this output: its displacement
            // moves into the reference, which goes to the other buffer
            const T m10 = (gn[0] - gn[2]) + (gn[4] - gn[5]) + (gn[7] - gn[6]);
            const T m01 = (gn[1] - gn[3]) + (gn[4] + gn[5]) - (gn[6] + gn[7]);
#pragma unroll
            for (int q = 0; q < 8; ++q) gn[q] -= el_geq<T>(q, m10, m01);
            void* eo = a.eref_in ? P.eref : P.eref2;
            const double ex = own_x(), ey = own_y();
            const uint32_t cell = off[kk] / (uint32_t)sizeof(T);
            if (r64) {
              gstore(at(gptr<double>(eo), kk), cell * 8u, ex + double(m10));
              gstore(at(gptr<double>(eo) + plane, kk), cell * 8u, ey + double(m01));
            } else {
              gstore(at(gptr<float>(eo), kk), cell * 4u, float(ex) + float(m10));
              gstore(at(gptr<float>(eo) + plane, kk), cell * 4u, float(ey) + float(m01));
            }
          }
#pragma unroll
          for (int q = 0; q < 8; ++q) gstore(at(gout + q * plane, kk), off[kk], gn[q]);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) G[kk][q] = omg * G[kk][q] + gi[q];
      }
    }
  }
  if (RES) {
    // row pairs (y, y + 1) of the lane-pair sums, through LDS
    __syncthreads();  // every pull has read sS
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const int j = (w + NW * kk) * S + sub;
      if (j >= H && j < RR - H) {
#pragma unroll
        for (int q = 0; q < 8; ++q) sS[q][j][col] = G[kk][q];
      }
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const int j = (w + NW * kk) * S + sub;
      const int y = y0 - H + j;
      if (l > 1 && j >= H && j < RR - H && (y & 1) == 0 && y < ny && col >= H && col < RX - H && x >= 0 &&
          x < nx && (x & 1) == 0) {
        const uint32_t co = ((uint32_t)(y >> 1) * (uint32_t)cpitch + (uint32_t)(x >> 1)) * (uint32_t)sizeof(Tc);
#pragma unroll
        for (int q = 0; q < 8; ++q) gstore(cr + q * cplane, co, Tc(sS[q][j][col] + sS[q][j + 1][col]));
      }
    }
  }
  if (a.partials) {
    acc_r = wave_sum(acc_r);
    acc_g = wave_sum(acc_g);
    if (lane == 0) {
      sRed[2 * w] = acc_r;
      sRed[2 * w + 1] = acc_g;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      double r = 0.0, g = 0.0;
#pragma unroll
      for (int v = 0; v < NW; ++v) {
        r += sRed[2 * v];
        g += sRed[2 * v + 1];
      }
      const int t = ty * V.tiles_xn[A] + tx;
      P.partials2[2 * t] = r;
      P.partials2[2 * t + 1] = g;
    }
  }
}

template <typename T, typename Tc, bool FINE, bool SHIFT, int APPS, bool RES, bool ALT>
hipError_t launch_tsweep2(const SweepL& a, int ntiles, bool ref64, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  const dim3 block(kWave * sweepn_waves<T, SHIFT, APPS + (RES ? 1 : 0), ALT>());
  constexpr bool dbl = std::is_same<T, double>::value;
  if constexpr (SHIFT && !dbl) {
    if (ref64)
      hipLaunchKernelGGL((k_tsweep2<T, Tc, FINE, SHIFT, APPS, RES, ALT, true>), dim3(ntiles), block, 0, s, a);
    else
      hipLaunchKernelGGL((k_tsweep2<T, Tc, FINE, SHIFT, APPS, RES, ALT, false>), dim3(ntiles), block, 0, s, a);
  } else {
    hipLaunchKernelGGL((k_tsweep2<T, Tc, FINE, SHIFT, APPS, RES, ALT, SHIFT && dbl>), dim3(ntiles), block, 0, s, a);
  }
  return hipGetLastError();
}

template <typename T, typename Tc, bool SHIFT, bool RES>
hipError_t launch_tsweep2_wide(const SweepL& a, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  const dim3 block(kWave * sweepn_waves<T, SHIFT, 2 + (RES ? 1 : 0), false>());
  hipLaunchKernelGGL((k_tsweep2<T, Tc, true, SHIFT, 2, RES, false, SHIFT, true>), dim3(ntiles), block, 0, s, a);
  return hipGetLastError();
}

// fixed-order FP64 sum of the finest level's norm partials of problem pid and
// what follows from it, by the first 256 threads of a block (all take part in
// the barriers)
__device__ __forceinline__ void finalize_norms(const ProbL& a, int pid, double* sr, double* sg) {
  const ProbD& P = a.probs[pid];
  double r = 0.0, g = 0.0;
  const int n = a.fused == 2 ? P.ntiles_test : (a.fused ? P.ntiles_fine2 : P.ntiles_fine);
  const double2* part = (const double2*)(a.fused ? P.partials2 : P.partials);
  // each thread sums the pairs k = t, t + 256, ... in that order; eight loads
  // are in flight at a time (an absent pair adds +0, which leaves the sums of
  // squares unchanged)
  for (int k0 = threadIdx.x; k0 < n && threadIdx.x < 256; k0 += 8 * 256) {
    double2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + 256 * u;
      v[u] = k < n ? part[k] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      r += v[u].x;
      g += v[u].y;
    }
  }
  if (threadIdx.x < 256) {
    sr[threadIdx.x] = r;
    sg[threadIdx.x] = g;
  }
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      sr[threadIdx.x] += sr[threadIdx.x + o];
      sg[threadIdx.x] += sg[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    P.norm2[0] = sr[0];
    P.norm2[1] = sg[0];
    // divergence: a non-finite norm, or (at the end of a fixed-cycle step)
    // ||g|| grown above 1e8 times the largest of its first kGrowthWindow
    // non-zero step-end values since the initial conditions.  The window
    // keeps a first value at rounding level (loads that cancel at t = 0)
    // from becoming the reference.
    if (!isfinite(sr[0]) || !isfinite(sg[0])) P.flags[0] = 1;
    if (a.advance && isfinite(sg[0]) && sg[0] > 0.0) {
      double* gr = P.gref;
      if (gr[1] < kGrowthWindow) {
        gr[0] = fmax(gr[0], sg[0]);
        gr[1] += 1.0;
      } else if (sg[0] > 1e16 * gr[0]) {
        P.flags[0] = 1;
      }
    }
    if (a.div && P.flags[0]) a.div[pid] = 1;
    if (a.advance) *P.phase += 1;
    if (a.decide && !P.ad[0]) {
      // the host's stopping test of the adaptive schedule, in the same FP64
      // steps: stop, or count the cycle that follows
      const double nr = sqrt(sr[0]), ng = sqrt(sg[0]);
      P.ad_ratio[0] = ng > 0 ? nr / ng : 0.0;
      if (!isfinite(nr) || !isfinite(ng))
        P.ad[0] = 2;
      else if (nr <= a.tol * ng || P.ad[1] >= a.ne_max)
        P.ad[0] = 1;
      else
        P.ad[1] += 1;
    }
  }
}

// ======================================================================
// flow step: D^n, centred coupling source (eq. source:implicit), pressure
// (eq. pressure), SRT collision with source (eqs. pressure:collision,
// pressure:collision:source), pull-stream and boundary rules; then, by the
// last block of a problem to end, the step's norms and counter (a.finish)
// ======================================================================
// Bound by memory on large grids and by one block's chain of loads on small
// ones: every load of both rows of a lane is issued before the first use, from
// offsets without branches (ghost cells are copies: an index), and 8 waves of
// 2 rows keep more loads in flight than 4 of 4.  Types of wall cells are read in
// tiles that hold a wall.  64^2 11.7 us, 512^2 16.7, 2048^2 132 (144 bytes per
// cell, 4.6 TB/s), 1024^2 in FP64 55; with 4 waves of 4 rows and a launch of its
// own for the norms 20, 23.6, 149 and 66.
template <typename T, bool SHIFT>
__global__ __launch_bounds__((kWave * kFlowWaves)) void k_tflow(CellL a) {
  if (gated_off(a.skip, a.need)) return;  // uniform over the grid
  constexpr int NW = kFlowWaves, NK = kFlowRows;
  constexpr int RR = NW * NK;                // one halo row each side
  constexpr int TY = kFlowTileY;
  using Off = uint64_t;  // offsets of 32 bits are no faster here
  __shared__ T sF[9][RR][kWave];
  __shared__ double sPd[SHIFT ? RR : 1][kWave];  // pressure reference, FP64 or FP32 (same bytes)
  float (*sPf)[kWave] = reinterpret_cast<float (*)[kWave]>(sPd);

  const int2 te = a.tiles[blockIdx.x];
  const ProbD& P = a.probs[te.x];
  const LevelD& V = P.lv[P.L];
  const int nx = V.nx, ny = V.ny, pitch = V.pitch;
  const int64_t plane = V.plane;
  const int sh = V.tile_shift[1];
  const int tx = te.y & ((1 << sh) - 1), ty = te.y >> sh;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int x = tx * kFlowTileX - 1 + lane;
  const int y0 = ty * TY;
  const int n = *P.phase;
  const GPtr<T> fin = gptr<T>(P.f[n & 1]), fout = gptr<T>(P.f[(n + 1) & 1]), g = gptr<T>(V.gA);
  const GPtr<double> D1 = gptr<double>(P.D[(n + 2) % 3]), D2 = gptr<double>(P.D[(n + 1) % 3]);
  const GPtr<double> Dn = gptr<double>(P.D[n % 3]), pout = gptr<double>(P.pout);
  const GPtr<double> src = gptr<double>(P.src), omf = gptr<double>(P.omf);
  const bool has_src = P.src != nullptr, has_omf = P.omf != nullptr;
  const bool perx = P.fper[0] != 0, pery = P.fper[1] != 0;
  const int gx = perx ? wrap_index(x, nx, kWave) : clampi(x, 0, nx - 1);
  const bool out_lane = lane >= 1 && lane < kWave - 1 && x < nx;
  const void* pref = SHIFT ? P.pref[n & 1] : nullptr;
  void* pref_next = SHIFT ? P.pref[(n + 1) & 1] : nullptr;
  const bool r64 = P.ref64 != 0;

  T f[NK][9], gg[NK][8];
  double d1[NK], d2[NK], sc[NK], om_[NK], pr[NK];
  Off cell[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const int y = y0 - 1 + w + NW * kk;
    const int gy = pery ? wrap_index(y, ny, RR) : clampi(y, 0, ny - 1);
    cell[kk] = (Off)gy * (Off)pitch + (Off)gx;
#pragma unroll
    for (int i = 0; i < 9; ++i) f[kk][i] = gload(fin + i * plane, cell[kk] * (Off)sizeof(T));
#pragma unroll
    for (int q = 0; q < 8; ++q) gg[kk][q] = gload(g + q * plane, cell[kk] * (Off)sizeof(T));
    d1[kk] = gload(D1, cell[kk] * 8);
    d2[kk] = gload(D2, cell[kk] * 8);
    sc[kk] = has_src ? gload(src, cell[kk] * 8) : 0.0;
    om_[kk] = has_omf ? gload(omf, cell[kk] * 8) : P.omf_u;
    pr[kk] = !SHIFT ? 0.0
                    : (r64 ? gload(gptr<double>(pref), cell[kk] * 8) : double(gload(gptr<float>(pref), cell[kk] * 4)));
  }
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const int j = w + NW * kk;
    const double dn = P.kD * double(el_ms(gg[kk]));
    double sv = -P.alpha_h * ((1.0 - P.r) * (d1[kk] - d2[kk]) + P.r * (dn - d1[kk]));
    if (has_src) sv += sc[kk];
    const T s = T(sv), om = T(om_[kk]);
    T p = T(0);
#pragma unroll
    for (int i = 0; i < 9; ++i) p += f[kk][i];
    if (out_lane && j >= 1 && j <= TY && y0 - 1 + j < ny) {
      gstore(Dn, cell[kk] * 8, dn);
      gstore(pout, cell[kk] * 8, double(p) + 0.5 * sv + pr[kk]);
    }
    p += T(0.5) * s;
    const T so = (T(1) - T(0.5) * om) * s;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const T wi = T(w9(i));
      sF[i][j][lane] = f[kk][i] - om * (f[kk][i] - wi * p) + wi * so;
    }
    if (SHIFT) {
      if (r64)
        sPd[j][lane] = pr[kk];
      else
        sPf[j][lane] = float(pr[kk]);
    }
  }
  __syncthreads();

  // does the tile hold a wall cell?
  const bool bnd = (!perx && (tx == 0 || (tx + 1) * kFlowTileX >= nx)) || (!pery && (ty == 0 || y0 + TY >= ny));
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const int j = w + NW * kk;
    if (j < 1 || j > TY) continue;
    const int y = y0 - 1 + j;
    const bool valid = out_lane && y < ny;
    if (!valid) continue;
    T fo[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) fo[i] = sF[i][j - cy9(i)][lane - cx9(i)];
    double p0 = 0.0;
    if (SHIFT && r64) {  // reference differences in FP64, rounded once
      p0 = sPd[j][lane];
#pragma unroll
      for (int i = 1; i < 9; ++i) fo[i] += T(w9(i) * (sPd[j - cy9(i)][lane - cx9(i)] - p0));
    } else if (SHIFT) {
      const float p0f = sPf[j][lane];
      p0 = p0f;
#pragma unroll
      for (int i = 1; i < 9; ++i) fo[i] += T(float(w9(i)) * (sPf[j - cy9(i)][lane - cx9(i)] - p0f));
    }
    auto pn = [&](int jj, int ll) { return r64 ? sPd[jj][ll] : double(sPf[jj][ll]); };
    int tL = kFlPeriodic, tR = kFlPeriodic, tB = kFlPeriodic, tT = kFlPeriodic;
    if (bnd) {
      tL = P.ftype[kLeft][y], tR = P.ftype[kRight][y];
      tB = P.ftype[kBottom][x], tT = P.ftype[kTop][x];
    }
    const bool wl = x == 0 && tL != kFlPeriodic;
    const bool wr = x == nx - 1 && tR != kFlPeriodic;
    const bool wb = y == 0 && tB != kFlPeriodic;
    const bool wt = y == ny - 1 && tT != kFlPeriodic;
    if (wl || wr || wb || wt) {
#pragma unroll
      for (int i = 1; i < 9; ++i) {
        const int cx = cx9(i), cy = cy9(i);
        const bool ox = (cx > 0 && wl) || (cx < 0 && wr);
        const bool oy = (cy > 0 && wb) || (cy < 0 && wt);
        if (!(ox || oy)) continue;
        const int tx_ = cx > 0 ? tL : tR;
        const int ty_ = cy > 0 ? tB : tT;
        T v = T(0);
        bool usex = false, half = false;
        if (ox && oy) {
          if (tx_ == kFlSymmetry && ty_ == kFlSymmetry) {
            v = sF[opp9(i)][j][lane];
          } else {
            usex = ty_ == kFlSymmetry;
            half = true;
          }
        } else if (ox) {
          usex = true;
          if (tx_ == kFlSymmetry) {
            v = sF[mx9(i)][j - cy][lane];
            if (SHIFT) v += T(w9(i) * (pn(j - cy, lane) - p0));
          } else {
            half = true;
          }
        } else {
          if (ty_ == kFlSymmetry) {
            v = sF[my9(i)][j][lane - cx];
            if (SHIFT) v += T(w9(i) * (pn(j, lane - cx) - p0));
          } else {
            half = true;
          }
        }
        if (half) {
          const int type = usex ? tx_ : ty_;
          const T o = sF[opp9(i)][j][lane];
          if (type == kFlNoflow) {
            v = o;  // eq. BC:noFlow
          } else {  // eq. BC:pressure
            const double* bc = usex ? (cx > 0 ? P.flbc[kLeft] : P.flbc[kRight])
                                    : (cy > 0 ? P.flbc[kBottom] : P.flbc[kTop]);
            const int bidx = usex ? y : x;
            const double add = bc ? bc[9 * bidx + i] : 0.0;
            v = -o + T(SHIFT ? add - 2.0 * w9(i) * p0 : add);  // one rounding
          }
        }
        fo[i] = v;
      }
    }
    const Off idx = (Off)y * (Off)pitch + (Off)x;
    if (SHIFT) {
      // the next step's re-base of the pressure: its zeroth moment moves into
      // the reference, written to the other buffer (neighbours of this launch
      // still read this step's)
      T pl = T(0);
#pragma unroll
      for (int i = 0; i < 9; ++i) pl += fo[i];
#pragma unroll
      for (int i = 0; i < 9; ++i) fo[i] -= T(w9(i)) * pl;
      if (r64)
        gstore(gptr<double>(pref_next), idx * 8, p0 + double(pl));
      else
        gstore(gptr<float>(pref_next), idx * 4, float(p0) + float(pl));
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) gstore(fout + i * plane, idx * (Off)sizeof(T), fo[i]);
  }

  // the last block of the problem to end: every other has read the step
  // counter, and the norms' partials come from an earlier launch
  if (a.finish) {
    __shared__ int last;
    __syncthreads();  // sF is free
    if (threadIdx.x == 0) {
      const int blocks = V.tiles_xn[1] * ((ny + TY - 1) / TY);
      last = atomicAdd(P.arrived, 1) == blocks - 1;
    }
    __syncthreads();
    if (last) {
      if (threadIdx.x == 0) *P.arrived = 0;
      if (a.finish == 1) {
        ProbL p{};
        p.probs = a.probs;
        p.fused = a.fused;
        p.advance = 1;
        p.div = a.div;
        double* sr = reinterpret_cast<double*>(&sF[0][0][0]);
        finalize_norms(p, te.x, sr, sr + 256);
      } else if (threadIdx.x == 0) {
        *P.phase += 1;
      }
    }
  }
}


template <typename T, bool SHIFT>
hipError_t launch_tflow(const CellL& a, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_tflow<T, SHIFT>), dim3(ntiles), dim3(kWave * kFlowWaves), 0, s, a);
  return hipGetLastError();
}

// ======================================================================
// per-cell kernels over the finest level (64 x 4 cells per block)
// ======================================================================
struct CellPos {
  int x, y;
  bool in;
};
__device__ __forceinline__ CellPos cell_pos(const LevelD& V, int b) {
  const int cbx = (V.nx + kCellBX - 1) / kCellBX;
  CellPos c;
  c.x = (b % cbx) * kCellBX + (int)(threadIdx.x & 63);
  c.y = (b / cbx) * kCellBY + (int)(threadIdx.x >> 6);
  c.in = c.x < V.nx && c.y < V.ny;
  return c;
}

// explicit force of the step: Ft = h^2 c0 f - alpha h grad p with the
// first-moment gradient (eq. pressure:gradient) or the central difference of
// p (eq. pressure:gradient:alternative), and the explicit part of the centred
// source.  A block of 64 x 4 cells first stages the inputs that the central
// differences take from the 3 x 3 neighbourhood, for its 66 x 6 region: st,
// the source's explicit part (FP64 D fields), and with CENTRAL the sum of the
// populations plus the pressure reference.  Each is formed once per cell.
constexpr int kFRX = kCellBX + 2, kFRY = kCellBY + 2;

template <typename T, bool CENTRAL>
__device__ __forceinline__ void force_stage(const ProbD& P, const LevelD& V, int b, int n, double (*sst)[kFRX],
                                            double (*sp)[kFRX]) {
  const int cbx = (V.nx + kCellBX - 1) / kCellBX;
  const int x0 = (b % cbx) * kCellBX - 1, y0 = (b / cbx) * kCellBY - 1;
  const double* D1 = P.D[(n + 2) % 3];
  const double* D2 = P.D[(n + 1) % 3];
  const T* f = (const T*)P.f[n & 1];
  const void* pref = P.pref[n & 1];
  const bool r64 = P.ref64 != 0;
  const bool perx = P.el[kLeft] == kElPeriodic, pery = P.el[kBottom] == kElPeriodic;
  for (int r = threadIdx.x; r < kFRX * kFRY; r += blockDim.x) {
    const int rx = r % kFRX, ry = r / kFRX;
    const int x = x0 + rx, y = y0 + ry;
    if (x > V.nx || y > V.ny) continue;  // no cell of the grid reads farther
    const int xs = ghost_map(x, V.nx, perx), ys = ghost_map(y, V.ny, pery);
    const int64_t k = (int64_t)ys * V.pitch + xs;
    const double d1 = D1[k], d2 = D2[k];
    double v = -P.alpha_h * ((1.0 - P.r) * (d1 - d2) - P.r * d1);
    if (P.src) v += P.src[k];
    sst[ry][rx] = v;
    if (CENTRAL) {
      // shifted storage holds f - w p_ref, whose sum lacks p_ref
      double sum = pref ? (r64 ? ((const double*)pref)[k] : double(((const float*)pref)[k])) : 0.0;
#pragma unroll
      for (int i = 0; i < 9; ++i) sum += double(f[i * V.plane + k]);
      sp[ry][rx] = sum;
    }
  }
}

// the 3 x 3 neighbourhood of this thread's cell in a staged plane
__device__ __forceinline__ void force_gather(const double (*s)[kFRX], double v[3][3]) {
  const int lx = threadIdx.x % kCellBX, ly = threadIdx.x / kCellBX;
#pragma unroll
  for (int dy = 0; dy < 3; ++dy)
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) v[dy][dx] = s[ly + dy][lx + dx];
}

// Ft from the gradients of the source part (gx, gy) and of p (px, py)
template <typename T>
__device__ __forceinline__ void force_write(const ProbD& P, const LevelD& V, const CellPos& c, double gx, double gy,
                                            double px, double py) {
  const int64_t idx = (int64_t)c.y * V.pitch + c.x;
  double Fx = -P.alpha * P.h * (px + 0.5 * gx);
  double Fy = -P.alpha * P.h * (py + 0.5 * gy);
  if (P.fbody) {
    Fx += P.fbody[idx];
    Fy += P.fbody[V.plane + idx];
  }
  T* Ft = (T*)P.Ft;
  Ft[idx] = T(Fx);
  Ft[V.plane + idx] = T(Fy);
}

// first-moment gradient (eq. pressure:gradient) from the first moments of the
// cell's own populations
__device__ __forceinline__ void force_moments(const ProbD& P, const LevelD& V, const CellPos& c, double jx,
                                              double jy, double& px, double& py) {
  const int64_t idx = (int64_t)c.y * V.pitch + c.x;
  const double om = P.omf ? P.omf[idx] : P.omf_u;
  px = -3.0 * om * jx;
  py = -3.0 * om * jy;
}

// the force of this thread's cell from the staged planes: the source part's
// gradient, and the pressure gradient (central: from the staged pressure;
// else from the first moments of the cell's own populations)
template <typename T>
__device__ __forceinline__ void force_finish(const ProbD& P, const LevelD& V, const CellPos& c, int n, bool central,
                                             const double (*sst)[kFRX], const double (*sp)[kFRX]) {
  double v[3][3], gx, gy, px, py;
  force_gather(sst, v);
  grad_c(v, gx, gy);
  if (central) {
    force_gather(sp, v);
    grad_c(v, px, py);  // gradient of p without its source part
  } else {
    const T* f = (const T*)P.f[n & 1];
    const int64_t idx = (int64_t)c.y * V.pitch + c.x;
    double jx = 0.0, jy = 0.0;
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      const double fv = double(f[i * V.plane + idx]);
      jx += fv * cx9(i);
      jy += fv * cy9(i);
    }
    force_moments(P, V, c, jx, jy, px, py);
  }
  force_write<T>(P, V, c, gx, gy, px, py);
}

template <typename T>
__global__ __launch_bounds__(256) void k_force(CellL a) {
  if (gated_off(a.skip, a.need)) return;  // uniform over the grid
  __shared__ double sst[kFRY][kFRX];
  __shared__ double sp[kFRY][kFRX];
  const int2 te = a.tiles[blockIdx.x];
  const ProbD& P = a.probs[te.x];
  const LevelD& V = P.lv[P.L];
  const int n = *P.phase;
  const bool central = P.grad_central != 0;  // one problem per block
  if (central)
    force_stage<T, true>(P, V, te.y, n, sst, sp);
  else
    force_stage<T, false>(P, V, te.y, n, sst, sp);
  __syncthreads();
  const CellPos c = cell_pos(V, te.y);
  if (!c.in) return;
  force_finish<T>(P, V, c, n, central, sst, sp);
}

// initial conditions (eqs. ICs, ICs:moments with p = 0 and eta = 0 at t = 0)
template <typename T>
__global__ __launch_bounds__(256) void k_init(CellL a) {
  const int2 te = a.tiles[blockIdx.x];
  const ProbD& P = a.probs[te.x];
  const LevelD& V = P.lv[P.L];
  if (te.y == 0 && threadIdx.x == 0) {
    *P.phase = 0;
    P.flags[0] = 0;
    *P.arrived = 0;
    P.gref[0] = 0.0;
    P.gref[1] = 0.0;
  }
  const CellPos c = cell_pos(V, te.y);
  if (!c.in) return;
  const int64_t idx = (int64_t)c.y * V.pitch + c.x;
  const double s = P.src ? P.src[idx] : 0.0;
  T* f0 = (T*)P.f[0];
  T* f1 = (T*)P.f[1];
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    f0[i * V.plane + idx] = T(-0.5 * w9(i) * s);
    f1[i * V.plane + idx] = T(0);
  }
  const double Fx = P.fbody ? P.fbody[idx] : 0.0, Fy = P.fbody ? P.fbody[V.plane + idx] : 0.0;
  // the force the extraction adds back (eta = m10 + F/2 = 0 at t = 0); every
  // step recomputes it
  ((T*)P.Ft)[idx] = T(Fx);
  ((T*)P.Ft)[V.plane + idx] = T(Fy);
  // moments m10 = -F/2, m12 = -F/6 (x), m01 = -F/2, m21 = -F/6 (y); others 0
  const double A = -0.5 * Fx, B = -0.5 * Fy, Pm = -Fx / 6.0, Q = -Fy / 6.0;
  double g[8];
  g[0] = 0.5 * (A - Pm);
  g[2] = -0.5 * (A - Pm);
  g[1] = 0.5 * (B - Q);
  g[3] = -0.5 * (B - Q);
  g[4] = 0.25 * (Pm + Q);
  g[5] = 0.25 * (Q - Pm);
  g[6] = -0.25 * (Pm + Q);
  g[7] = 0.25 * (Pm - Q);
  T* gA = (T*)V.gA;
#pragma unroll
  for (int q = 0; q < 8; ++q) gA[q * V.plane + idx] = T(g[q]);
  for (int k = 0; k < 3; ++k) P.D[k][idx] = 0.0;
  if (P.eref && P.ref64) {
    ((double*)P.eref)[idx] = 0.0;
    ((double*)P.eref)[V.plane + idx] = 0.0;
    ((double*)P.pref[0])[idx] = 0.0;
    ((double*)P.pref[1])[idx] = 0.0;
  } else if (P.eref) {
    ((float*)P.eref)[idx] = 0.f;
    ((float*)P.eref)[V.plane + idx] = 0.f;
    ((float*)P.pref[0])[idx] = 0.f;
    ((float*)P.pref[1])[idx] = 0.f;
  }
  P.pout[idx] = 0.0;
}

// re-basing of the shifted storage: move the per-cell displacement reference
// to the current displacement so the stored offsets stay small (the pressure
// is re-based by the flow step that writes the populations).  FORCE: the
// step's explicit force in the same pass; it reads the populations and the
// pressure reference, which this kernel leaves alone, so the central gradient
// may read any neighbour.
template <typename T, bool FORCE>
__global__ __launch_bounds__(256) void k_rebase(CellL a) {
  if (gated_off(a.skip, a.need)) return;  // uniform over the grid
  __shared__ double sst[FORCE ? kFRY : 1][kFRX];
  __shared__ double sp[FORCE ? kFRY : 1][kFRX];
  const int2 te = a.tiles[blockIdx.x];
  const ProbD& P = a.probs[te.x];
  const LevelD& V = P.lv[P.L];
  const int n = FORCE ? *P.phase : 0;
  const bool central = FORCE && P.grad_central != 0;  // one problem per block
  if (FORCE) {
    if (central)
      force_stage<T, true>(P, V, te.y, n, sst, sp);
    else
      force_stage<T, false>(P, V, te.y, n, sst, sp);
    __syncthreads();
  }
  const CellPos c = cell_pos(V, te.y);
  if (!c.in) return;
  const int64_t idx = (int64_t)c.y * V.pitch + c.x;
  T* g = (T*)V.gA;
  T u[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) u[q] = g[q * V.plane + idx];
  const T m10 = (u[0] - u[2]) + (u[4] - u[5]) + (u[7] - u[6]);
  const T m01 = (u[1] - u[3]) + (u[4] + u[5]) - (u[6] + u[7]);
#pragma unroll
  for (int q = 0; q < 8; ++q) g[q * V.plane + idx] = u[q] - el_geq<T>(q, m10, m01);
  if (P.ref64) {
    double* eref = (double*)P.eref;
    eref[idx] += double(m10);
    eref[V.plane + idx] += double(m01);
  } else {
    float* eref = (float*)P.eref;
    eref[idx] += float(m10);
    eref[V.plane + idx] += float(m01);
  }
  if (FORCE) force_finish<T>(P, V, c, n, central, sst, sp);
}

// displacement, pressure and stress of the current populations (eqs.
// displacement, moments:bared; stress in physical units) for rows row0 ..
// row0 + rows - 1, as dense planes.  The output may be host memory that the
// device maps: the link to the host then bounds the launch, and writing there
// leaves out a copy.  D of a block's 66 x 6 region is formed once per cell.
template <typename T, bool SHIFT>
__global__ __launch_bounds__(256) void k_extract(ExtractL a) {
  __shared__ double sD[kFRY][kFRX];
  const ProbD& P = *a.prob;
  const LevelD& V = P.lv[P.L];
  const T* g = (const T*)V.gA;
  const bool perx = P.el[kLeft] == kElPeriodic, pery = P.el[kBottom] == kElPeriodic;
  const int cbx = (V.nx + kCellBX - 1) / kCellBX;
  const int x0 = (int)(blockIdx.x % cbx) * kCellBX, y0 = a.row0 + (int)(blockIdx.x / cbx) * kCellBY;
  for (int r = threadIdx.x; r < kFRX * kFRY; r += blockDim.x) {
    const int rx = r % kFRX, ry = r / kFRX;
    const int x = x0 - 1 + rx, y = y0 - 1 + ry;
    if (x > V.nx || y > V.ny) continue;  // no cell of the grid reads farther
    const int64_t k = (int64_t)ghost_map(y, V.ny, pery) * V.pitch + ghost_map(x, V.nx, perx);
    T u[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) u[q] = g[q * V.plane + k];
    sD[ry][rx] = P.kD * double(el_ms(u));
  }
  __syncthreads();
  if (a.flags && blockIdx.x == 0 && threadIdx.x == 0) a.flags[1] = P.flags[0];
  const int x = x0 + (int)(threadIdx.x % kCellBX), row = y0 - a.row0 + (int)(threadIdx.x / kCellBX);
  const int y = a.row0 + row;
  if (x >= V.nx || row >= a.rows || y >= V.ny) return;
  double D[3][3], gx, gy;
  force_gather(sD, D);
  grad_c(D, gx, gy);
  const int64_t idx = (int64_t)y * V.pitch + x;
  double u[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) u[q] = double(g[q * V.plane + idx]);
  const T* Ft = (const T*)P.Ft;
  const double Fx = double(Ft[idx]) + P.cstar * gx, Fy = double(Ft[V.plane + idx]) + P.cstar * gy;
  double m10 = (u[0] - u[2]) + (u[4] - u[5]) + (u[7] - u[6]);
  double m01 = (u[1] - u[3]) + (u[4] + u[5]) - (u[6] + u[7]);
  const double m11 = (u[4] - u[5]) + (u[6] - u[7]);
  const double ms = ((u[0] + u[2]) + (u[1] + u[3])) + 2.0 * ((u[4] + u[5]) + (u[6] + u[7]));
  const double md = (u[0] + u[2]) - (u[1] + u[3]);
  if (SHIFT) {
    m10 += P.ref64 ? ((const double*)P.eref)[idx] : double(((const float*)P.eref)[idx]);
    m01 += P.ref64 ? ((const double*)P.eref)[V.plane + idx] : double(((const float*)P.eref)[V.plane + idx]);
  }
  const int64_t o = (int64_t)row * V.nx + x, N = a.stride;
  const double ex = m10 + 0.5 * Fx, ey = m01 + 0.5 * Fy;
  a.eta[o] = ex;
  a.eta[N + o] = ey;
  const double bs = P.b_s * ms, bd = P.b_d * md, b11 = P.b_d * m11;
  a.sig[o] = -0.5 * (bs + bd) * P.inv_c0h;
  a.sig[N + o] = -b11 * P.inv_c0h;
  a.sig[2 * N + o] = -0.5 * (bs - bd) * P.inv_c0h;
  if (a.p) a.p[o] = P.pout[idx] / a.c0;
  if (a.flags && !(isfinite(ex) && isfinite(ey))) a.flags[0] = 1;
}

template <typename T>
hipError_t launch_force(const CellL& a, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_force<T>), dim3(ntiles), dim3(256), 0, s, a);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_init(const CellL& a, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_init<T>), dim3(ntiles), dim3(256), 0, s, a);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_rebase(const CellL& a, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_rebase<T, false>), dim3(ntiles), dim3(256), 0, s, a);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_rebase_force(const CellL& a, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_rebase<T, true>), dim3(ntiles), dim3(256), 0, s, a);
  return hipGetLastError();
}
template <typename T, bool SHIFT>
hipError_t launch_extract(const ExtractL& a, int nx, hipStream_t s) {
  const int blocks = ((nx + kCellBX - 1) / kCellBX) * ((a.rows + kCellBY - 1) / kCellBY);
  if (blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_extract<T, SHIFT>), dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ======================================================================
// coarse tail of the multigrid recursion: one workgroup per problem runs
// Algorithm 4 on all levels from L - depth down to the coarsest.  Every cell
// of a level is owned by one thread (at most 4 per thread), which keeps the
// level's iterate and right-hand side in registers across its sweeps; D(g)
// and the post-collision populations live in LDS.  Global memory (L2-resident
// at these sizes) is touched only between levels: right-hand sides going
// down, iterates kept for the ascent and the coarse correction coming up.
// Coarse levels carry homogeneous boundary data and no explicit force.
// ======================================================================
// Every homogeneous rule of a coarse level gives the population q arriving at
// (x, y) as plus or minus one post-collision value of the level: interior and
// periodic pulls, mirror images at symmetry walls, bounce-back (Dirichlet) and
// anti-bounce-back (traction).  The code returned is that value's index in sG
// (q-major: q * ps + y * nx + x) with bit 15 set for a minus sign.
__device__ __forceinline__ uint32_t tail_pull_code(const int q, int x, int y, int nx, int ny, const int* el, int ps) {
  const int cx = cx8(q), cy = cy8(q);
  int sx = x - cx, sy = y - cy;
  const bool perx = el[kLeft] == kElPeriodic, pery = el[kBottom] == kElPeriodic;
  bool ox = sx < 0 || sx >= nx, oy = sy < 0 || sy >= ny;
  if (ox && perx) {
    sx = (sx + nx) % nx;
    ox = false;
  }
  if (oy && pery) {
    sy = (sy + ny) % ny;
    oy = false;
  }
  if (!ox && !oy) return (uint32_t)(q * ps + sy * nx + sx);
  const int elx = cx > 0 ? el[kLeft] : el[kRight];
  const int ely = cy > 0 ? el[kBottom] : el[kTop];
  bool usex;
  if (ox && oy) {
    if (elx == kElSymmetry && ely == kElSymmetry) return (uint32_t)(opp8(q) * ps + y * nx + x);
    usex = ely == kElSymmetry;
  } else if (ox) {
    if (elx == kElSymmetry) return (uint32_t)(mx8(q) * ps + sy * nx + x);
    usex = true;
  } else {
    if (ely == kElSymmetry) return (uint32_t)(my8(q) * ps + y * nx + sx);
    usex = false;
  }
  const uint32_t o = (uint32_t)(opp8(q) * ps + y * nx + x);
  return (usex ? elx : ely) == kElDirichlet ? o : (o | 0x8000u);
}

// per-cell gather tables of a level: the 8 neighbours of the D(g) stencil
// (mirror ghosts at walls) and the 8 populations pulled, as 16-bit byte offsets
// into the level's planes in LDS (planes of `ps` cells of sz bytes), ready as
// LDS addresses.  An offset is a multiple of 4, so the two low bits of a word of
// pulls hold the signs of its lower and upper one (anti-bounce-back).
struct TailTab {
  uint32_t dn[4], pl[4];
  bool neg;  // a pull of this wave changes sign (tail_tab_signs)
};

__device__ __forceinline__ TailTab tail_table(const int* el, int c, int nx, int ny, uint32_t sz, uint32_t ps) {
  TailTab tb;
  const int x = c % nx, y = c / nx;
  const bool perx = el[kLeft] == kElPeriodic, pery = el[kBottom] == kElPeriodic;
  uint32_t d[8];
  int k = 0;
#pragma unroll
  for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx)
      if (dx != 0 || dy != 0) d[k++] = sz * (uint32_t)(ghost_map(y + dy, ny, pery) * nx + ghost_map(x + dx, nx, perx));
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    tb.dn[j] = d[2 * j] | (d[2 * j + 1] << 16);
    const uint32_t lo = tail_pull_code(2 * j, x, y, nx, ny, el, ps), hi = tail_pull_code(2 * j + 1, x, y, nx, ny, el, ps);
    tb.pl[j] = (lo & 0x7fffu) * sz | (lo >> 15) | (hi >> 15) << 1 | ((hi & 0x7fffu) * sz) << 16;
  }
  tb.neg = false;
  return tb;
}
__device__ __forceinline__ void tail_tab_signs(TailTab& tb) {
  tb.neg = __any(((tb.pl[0] | tb.pl[1] | tb.pl[2] | tb.pl[3]) & 3u) != 0);
}

__device__ __forceinline__ uint32_t lo16(uint32_t w) { return w & 0xffffu; }
__device__ __forceinline__ uint32_t hi16(uint32_t w) { return w >> 16; }
template <typename T> __device__ __forceinline__ T tail_at(const T* base, uint32_t off) {
  return *(const T*)((const char*)base + off);
}
// population q as pulled through the table
template <typename T> __device__ __forceinline__ T tail_pull(const TailTab& tb, const T* sG, int q) {
  const uint32_t w = tb.pl[q >> 1];
  T v = tail_at(sG, (q & 1) ? hi16(w) : w & 0xfffcu);
  if (tb.neg) {
    const uint32_t flip = (q & 1) ? (w << 30) & 0x80000000u : w << 31;
    if constexpr (sizeof(T) == 8)
      v = __builtin_bit_cast(T, __builtin_bit_cast(uint64_t, v) ^ (uint64_t)flip << 32);
    else
      v = __builtin_bit_cast(T, __builtin_bit_cast(uint32_t, v) ^ flip);
  }
  return v;
}
// central gradient of D at this thread's cell
template <typename T> __device__ __forceinline__ void tail_grad(const TailTab& tb, const T* sD, T& gx, T& gy) {
  T v[3][3];
  v[0][0] = tail_at(sD, lo16(tb.dn[0]));
  v[0][1] = tail_at(sD, hi16(tb.dn[0]));
  v[0][2] = tail_at(sD, lo16(tb.dn[1]));
  v[1][0] = tail_at(sD, hi16(tb.dn[1]));
  v[1][2] = tail_at(sD, lo16(tb.dn[2]));
  v[2][0] = tail_at(sD, hi16(tb.dn[2]));
  v[2][1] = tail_at(sD, lo16(tb.dn[3]));
  v[2][2] = tail_at(sD, hi16(tb.dn[3]));
  v[1][1] = T(0);  // the centred gradient does not use the centre
  grad_c(v, gx, gy);
}

template <typename T>
__device__ __forceinline__ ElConst<T> tail_consts(const ProbD& P) {
  ElConst<T> k;
  k.om_s = T(P.om_s);
  k.om_d = T(P.om_d);
  k.beta22 = T(P.beta22);
  k.kD = T(P.kD);
  k.cstar = T(P.cstar);
  k.gamma = T(P.gamma);
  return k;
}

// a level of one wave needs no barrier between its own LDS writes and reads
// (in FP32 1.2 us of a tail; in FP64 it gained nothing)
template <typename T> __device__ __forceinline__ void tail_sync(int n) {
  if (sizeof(T) == 8 || __builtin_expect(n > kWave, 1)) {  // uniform
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// one application of S on a whole level held by the workgroup: thread c owns
// cell c; G (iterate) and R (right-hand side) in registers, gathers through the
// level's tables.  blend: G <- (1 - gamma) G + gamma S(G); otherwise
// G <- G - S(G) (residual).  Two barriers; sD and sG may be reused right after
// the return.  sG's planes have PS cells whatever the level, so that planes and
// tables are LDS addresses as they stand (50 of a sweep's 170 vector
// instructions were address arithmetic and unpacking, 1.5 us of an FP64 tail).
template <typename T, int PS = kTailThreads>
__device__ __forceinline__ void tail_relax(const ElConst<T>& k, int n, const TailTab& tb, T (&G)[1][8],
                                           const T (&R)[1][8], T* sD, T* sG, bool blend) {
  const int c = threadIdx.x;
  if (c < n) sD[c] = k.kD * el_ms(G[0]);
  tail_sync<T>(n);
  if (c < n) {
    T gx_, gy_;
    tail_grad(tb, sD, gx_, gy_);
    T u[8], s8[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) u[q] = G[0][q] - R[0][q];
    // a blending sweep streams gamma times the post-collision populations
    el_collide(u, k.cstar * gx_, k.cstar * gy_, k, s8, blend ? k.gamma : T(1));
#pragma unroll
    for (int q = 0; q < 8; ++q) sG[q * PS + c] = s8[q];
  }
  tail_sync<T>(n);
  const T omg = T(1) - k.gamma;
  if (c < n) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const T gi = tail_pull(tb, sG, q);
      G[0][q] = blend ? omg * G[0][q] + gi : G[0][q] - gi;
    }
  }
}

// the first smoothing application of a zero iterate: D(g) = 0, so the
// collision of -R needs no neighbour.  One barrier; sG is read until the next.
template <typename T>
__device__ __forceinline__ void tail_first(const ElConst<T>& k, int n, const TailTab& tb, T (&G)[1][8],
                                           const T (&R)[1][8], T* sG) {
  const int c = threadIdx.x;
  if (c < n) {
    T u[8], s8[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) u[q] = -R[0][q];
    el_collide(u, T(0), T(0), k, s8, k.gamma);
#pragma unroll
    for (int q = 0; q < 8; ++q) sG[q * kTailThreads + c] = s8[q];
  }
  tail_sync<T>(n);
  if (c < n) {
#pragma unroll
    for (int q = 0; q < 8; ++q) G[0][q] = tail_pull(tb, sG, q);
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) G[0][q] = T(0);
  }
}

// the gather tables of level l (built once at setup by k_tail_tables)
// (threads without a cell take the last one's)
__device__ __forceinline__ void tail_tab_load(const ProbD& P, int l, int c, TailTab& tb) {
  const uint4* t = (const uint4*)(P.ttab + 8 * (size_t)P.lv[l].toff) + 2 * min(c, P.lv[l].nx * P.lv[l].ny - 1);
  const uint4 a = t[0], b = t[1];
  tb.dn[0] = a.x;
  tb.dn[1] = a.y;
  tb.dn[2] = a.z;
  tb.dn[3] = a.w;
  tb.pl[0] = b.x;
  tb.pl[1] = b.y;
  tb.pl[2] = b.z;
  tb.pl[3] = b.w;
  tb.neg = false;
}

__global__ __launch_bounds__(kTailThreads) void k_tail_tables(int4 el4, int nx, int ny, int sz, uint32_t* out) {
  const int c = threadIdx.x;
  if (c >= nx * ny) return;
  const int el[4] = {el4.x, el4.y, el4.z, el4.w};
  const TailTab tb = tail_table(el, c, nx, ny, (uint32_t)sz, kTailThreads);
  uint4* o = (uint4*)(out + 8 * c);
  o[0] = make_uint4(tb.dn[0], tb.dn[1], tb.dn[2], tb.dn[3]);
  o[1] = make_uint4(tb.pl[0], tb.pl[1], tb.pl[2], tb.pl[3]);
}

hipError_t launch_tail_tables(const int* el, int nx, int ny, int sz, uint32_t* out, hipStream_t s) {
  if (nx * ny > kTailThreads) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_tail_tables, dim3(1), dim3(kTailThreads), 0, s, make_int4(el[0], el[1], el[2], el[3]), nx, ny,
                     sz, out);
  return hipGetLastError();
}

// row of cell c < 1024 in a level of nx columns, inv = ceil(2^20 / nx): exact,
// since c (inv nx - 2^20) < 1024 nx and the quotient's fraction is below
// 1 - 1/nx
__device__ __forceinline__ int tail_row(int c, uint32_t inv) { return (int)(((uint32_t)c * inv) >> 20); }

// one thread, one cell (c < n): the 8 planes of a level buffer (waves without
// a cell load nothing)
template <typename T>
__device__ __forceinline__ void tail_load1(const LevelD& V, const void* buf, int c, T (&A)[1][8]) {
#pragma unroll
  for (int q = 0; q < 8; ++q) A[0][q] = T(0);
  if (c >= V.nx * V.ny) return;
  const int y = tail_row(c, V.inv_nx);
  const uint32_t off = (uint32_t)(y * (V.pitch - V.nx) + c) * (uint32_t)sizeof(T);
  const GPtr<T> p = gptr<T>(buf);
#pragma unroll
  for (int q = 0; q < 8; ++q) A[0][q] = gload(p + q * V.plane, off);
}

template <typename T>
__device__ __forceinline__ void tail_store1(const LevelD& V, void* buf, int c, const T (&A)[1][8]) {
  if (c >= V.nx * V.ny) return;
  const int y = tail_row(c, V.inv_nx);
  const uint32_t off = (uint32_t)(y * (V.pitch - V.nx) + c) * (uint32_t)sizeof(T);
  const GPtr<T> p = gptr<T>(buf);
#pragma unroll
  for (int q = 0; q < 8; ++q) gstore(p + q * V.plane, off, A[0][q]);
}

template <typename T>
__device__ __forceinline__ void tail_zero(T (&A)[1][8]) {
#pragma unroll
  for (int q = 0; q < 8; ++q) A[0][q] = T(0);
}

// ---- the smallest levels as one matrix.  A V-cycle from a zero iterate on
// levels of at most kTailDenseCells cells is a fixed linear map of its
// right-hand side, and its 17 sweeps of one wave each (two levels, K = 4) are
// a chain of about 12 us, while the map's 128 x 128 matrix is read in under
// one.  It is formed once per problem in FP64 (k_tail_matrix) and applied in
// FP64 to the right-hand side as the sweeps would receive it.
constexpr int kTailPart = 8;  // threads per row of the matrix

// G = V-cycle on levels l..1 (at most kTailDenseCells cells each) from zero
// with the right-hand side R, in FP64 registers; rows of the recursion are
// kept in `keep` (LDS), 16 planes per level
__device__ __forceinline__ void tail_small(const ProbD& P, int top, int K, const double (&R0)[1][8], double (&G)[1][8],
                                           double* keep, double* lds) {
  const int c = threadIdx.x;
  const ElConst<double> k = tail_consts<double>(P);
  TailTab tb{};
  double R[1][8];
#pragma unroll
  for (int q = 0; q < 8; ++q) R[0][q] = R0[0][q];
  constexpr int N = kTailDenseCells;
  auto table = [&](int l) {
    if (c < P.lv[l].nx * P.lv[l].ny) tb = tail_table(P.el, c, P.lv[l].nx, P.lv[l].ny, sizeof(double), N);
    tail_tab_signs(tb);
  };
  for (int l = top; l >= 1; --l) {
    const LevelD& V = P.lv[l];
    const int nx = V.nx, n = nx * V.ny;
    double *sD = lds, *sG = lds + N;
    table(l);
    tail_zero(G);
    const int sweeps = l > 1 ? K : P.csweeps;
    for (int s = 0; s < sweeps; ++s) tail_relax<double, N>(k, n, tb, G, R, sD, sG, true);
    if (l == 1) break;
    if (c < n) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        keep[(16 * l + q) * N + c] = G[0][q];
        keep[(16 * l + 8 + q) * N + c] = R[0][q];
      }
    }
    tail_relax<double, N>(k, n, tb, G, R, sD, sG, false);
    __syncthreads();
    if (c < n) {
#pragma unroll
      for (int q = 0; q < 8; ++q) sG[q * N + c] = G[0][q];
    }
    __syncthreads();
    const LevelD& C = P.lv[l - 1];
    const int cnx = C.nx, f0 = 2 * c + 2 * cnx * tail_row(c, C.inv_nx), f1 = f0 + nx;
#pragma unroll
    for (int q = 0; q < 8; ++q)
      R[0][q] = c < cnx * C.ny ? (sG[q * N + f0] + sG[q * N + f0 + 1]) + (sG[q * N + f1] + sG[q * N + f1 + 1]) : 0.0;
    __syncthreads();
  }
  for (int l = 2; l <= top; ++l) {
    const LevelD& V = P.lv[l];
    const int nx = V.nx, n = nx * V.ny, cnx = nx / 2, cn = cnx * (V.ny / 2);
    double *sD = lds, *sG = lds + N;
    __syncthreads();
    if (c < cn) {
#pragma unroll
      for (int q = 0; q < 8; ++q) sG[q * N + c] = G[0][q];
    }
    __syncthreads();
    const int y = tail_row(c, V.inv_nx), ci = (y >> 1) * cnx + ((c - y * nx) >> 1);
    if (c < n) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        G[0][q] = keep[(16 * l + q) * N + c] + sG[q * N + ci];
        R[0][q] = keep[(16 * l + 8 + q) * N + c];
      }
    }
    __syncthreads();
    table(l);
    for (int s = 0; s < K; ++s) tail_relax<double, N>(k, n, tb, G, R, sD, sG, true);
  }
}

// one block per unit right-hand side: column b = q n + c of the matrix, stored
// so that thread t of the tail reads its entries k at out[k 1024 + t]
__global__ __launch_bounds__(kWave) void k_tail_matrix(ProbD P, int top, int K, double* out) {
  constexpr int N = kTailDenseCells;
  __shared__ double lds[9 * N], keep[16 * (kTailDenseLevels + 1) * N];
  const int c = threadIdx.x, n = P.lv[top].nx * P.lv[top].ny, b = blockIdx.x;
  double R[1][8], G[1][8];
#pragma unroll
  for (int q = 0; q < 8; ++q) R[0][q] = (q * n + c == b && c < n) ? 1.0 : 0.0;
  tail_small(P, top, K, R, G, keep, lds);
  if (c < n) {
#pragma unroll
    for (int q = 0; q < 8; ++q) out[(b / kTailPart) * kTailThreads + (q * n + c) * kTailPart + b % kTailPart] = G[0][q];
  }
}

hipError_t launch_tail_matrix(const ProbD& P, int top, int K, double* out, hipStream_t s) {
  const int n = P.lv[top].nx * P.lv[top].ny;
  if (top < 1 || top > kTailDenseLevels || n > kTailDenseCells) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_tail_matrix, dim3(8 * n), dim3(kWave), 0, s, P, top, K, out);
  return hipGetLastError();
}

// the matrix times the right-hand side R of level P.tml (thread c: cell c),
// left in LDS as plane q of cell c at lds + (1 + q) 1024 in type TT
constexpr int kTailM = 8 * kTailDenseCells / kTailPart;  // entries per thread
__device__ __forceinline__ void tail_dense_load(const ProbD& P, double (&m)[kTailM]) {
  const int n8 = 8 * P.lv[P.tml].nx * P.lv[P.tml].ny;
  const GPtr<double> M = gptr<double>(P.tmat);
#pragma unroll
  for (int k = 0; k < kTailM; ++k)
    m[k] = k * kTailPart < n8 ? gload(M + k * kTailThreads, (uint32_t)threadIdx.x * 8u) : 0.0;
}
template <typename TR, typename TT>
__device__ __forceinline__ void tail_dense(const ProbD& P, const TR (&R)[1][8], const double (&m)[kTailM], char* lds) {
  const int t = threadIdx.x, n = P.lv[P.tml].nx * P.lv[P.tml].ny, n8 = 8 * n;
  double* r = (double*)lds;
  if (t < n) {
#pragma unroll
    for (int q = 0; q < 8; ++q) r[q * n + t] = double(R[0][q]);
  }
  __syncthreads();
  const int part = t % kTailPart, o = t / kTailPart, q0 = o / n;
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < kTailM; ++k)
    if (k * kTailPart < n8) acc += m[k] * r[k * kTailPart + part];
#pragma unroll
  for (int w = 1; w < kTailPart; w *= 2) acc += __shfl_xor(acc, w, kWave);
  __syncthreads();  // every thread has read r
  if (part == 0 && o < n8) ((TT*)lds)[(1 + q0) * kTailThreads + (o - q0 * n)] = TT(acc);
  __syncthreads();
}

// The tail is one workgroup's chain.  From 32^2 on it takes 29 us in FP32 and 38
// to 41 in FP64, about half of them its sweeps, the rest the way between levels.
// Level descriptors are read as constant memory, whose loads need not follow
// every store and barrier anew: in k_tail_full, 50 cycles of an 8 x 128 column,
// 1.69 ms in FP64 (2.07 without) and 1.42 in FP32 (1.81).
// Algorithm 4 on levels lt..1 of one problem; levels >= 2 are stored as T,
// level 1 as T1.  Thread c owns cell c of every level.  Going down, the
// restricted residual of a level stays in the registers of the thread that
// owns the coarse cell (and is kept in the level's right-hand-side buffer for
// the way up); going up, the coarse correction passes through LDS and each
// level's stored iterate and right-hand side are fetched one level ahead.
// Levels P.tml..1 (0: none) are the matrix.
template <typename T, typename T1>
__device__ __forceinline__ void tail_run(const ProbD& P, int lt, int K, char* lds) {
  const int c = threadIdx.x;
  constexpr bool kPrefetch = sizeof(T) == 4;  // FP64 lacks the registers
  T R[1][8], G[1][8];
  T1 R1[1][8], G1[1][8];
  const int lm = P.tml;  // the turn: the matrix, or level 1's sweeps
  const int low = lm > 0 ? lm : 1;
  const ElConst<T> k = tail_consts<T>(P);
  // gather tables: tb for the level being swept, tn fetched one level ahead
  // (order of use: lt, ..., 2, 1, 2, ..., lt)
  TailTab tb, tn;
  if (kPrefetch && lt > lm) tail_tab_load(P, lt, c, tn);
  if (lt >= 2)
    tail_load1<T>(P.lv[lt], P.lv[lt].r, c, R);
  else
    tail_load1<T1>(P.lv[1], P.lv[1].r, c, R1);
  // the matrix (read cold at the turn it takes 4.4 us): in FP32
  // fetched before the sweeps of the level above, in FP64, which lacks the
  // registers, brought into this XCD's L2 behind the first sweeps, a word of
  // each 128-byte line
  double m[kTailM];
  const bool warm = !kPrefetch && lm > 0 && lt > lm && c * 128 < P.lv[lm].nx * P.lv[lm].ny * kTailThreads * 8;
  const int line = warm ? gload(gptr<int>(P.tmat), (uint32_t)c * 128u) : 0;
  // ---- descent: K pre-smoothing sweeps from zero, residual, restriction
  for (int l = lt; l > low; --l) {
    const LevelD& V = P.lv[l];
    const int nx = V.nx, ny = V.ny, n = nx * ny;
    T* sD = (T*)lds;
    T* sG = sD + kTailThreads;
    if (kPrefetch) {
      tb = tn;
      tail_tab_signs(tb);
      if (l - 1 > lm) tail_tab_load(P, l - 1, c, tn);
    } else {
      tail_tab_load(P, l, c, tb);
      tail_tab_signs(tb);
    }
    if (kPrefetch && lm > 0 && l == low + 1) tail_dense_load(P, m);
    tail_first<T>(k, n, tb, G, R, sG);
    for (int s = 1; s < K; ++s) tail_relax<T>(k, n, tb, G, R, sD, sG, true);
    if (!kPrefetch && l == lt) asm volatile("" ::"v"(line));  // loaded
    tail_store1<T>(V, V.gA, c, G);
    tail_relax<T>(k, n, tb, G, R, sD, sG, false);
    __syncthreads();  // every pull has read sG
    if (c < n) {
#pragma unroll
      for (int q = 0; q < 8; ++q) sG[q * kTailThreads + c] = G[0][q];
    }
    __syncthreads();
    const LevelD& C = P.lv[l - 1];
    const int cnx = nx / 2, cn = cnx * (ny / 2);
    T sum[8];
    if (c < cn) {
      // fine cell (2 X, 2 Y) of coarse cell (X, Y) = c
      const int f0 = 2 * c + 2 * cnx * tail_row(c, C.inv_nx), f1 = f0 + nx;
#pragma unroll
      for (int q = 0; q < 8; ++q) sum[q] = (sG[q * kTailThreads + f0] + sG[q * kTailThreads + f0 + 1]) + (sG[q * kTailThreads + f1] + sG[q * kTailThreads + f1 + 1]);
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) sum[q] = T(0);
    }
    if (l - 1 >= 2) {
#pragma unroll
      for (int q = 0; q < 8; ++q) R[0][q] = sum[q];
      if (l - 1 > lm) tail_store1<T>(C, C.r, c, R);
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) R1[0][q] = T1(sum[q]);
      if (lm == 0) tail_store1<T1>(C, C.r, c, R1);
    }
    __syncthreads();  // sG is reused by the next level
  }
  // prefetch the next level's stored iterate and right-hand side for the way up
  // (in FP64 later levels' registers are not there during the sweeps: their
  // loads follow the sweeps of the level below)
  T Gn[1][8], Rn[1][8];
  if (lt > low) {
    tail_load1<T>(P.lv[low + 1], P.lv[low + 1].gA, c, Gn);
    tail_load1<T>(P.lv[low + 1], P.lv[low + 1].r, c, Rn);
  }
  if (lm == 0) {
    // ---- coarsest level: its smoothing sweeps (2K unless set) from zero
    const LevelD& V = P.lv[1];
    const int n = V.nx * V.ny;
    T1* sD = (T1*)lds;
    T1* sG = sD + kTailThreads;
    const ElConst<T1> k1 = tail_consts<T1>(P);
    if (kPrefetch)
      tb = tn;
    else
      tail_tab_load(P, 1, c, tb);
    tail_tab_signs(tb);
    if (kPrefetch && lt >= 2) tail_tab_load(P, 2, c, tn);
    tail_first<T1>(k1, n, tb, G1, R1, sG);
    for (int s = 1; s < P.csweeps; ++s) tail_relax<T1>(k1, n, tb, G1, R1, sD, sG, true);
    tail_store1<T1>(V, V.gA, c, G1);
    __syncthreads();  // every pull has read sG
    if (c < n) {
#pragma unroll
      for (int q = 0; q < 8; ++q) sG[q * kTailThreads + c] = G1[0][q];
    }
    __syncthreads();
  } else {
    if (kPrefetch && lt > lm) tail_tab_load(P, lm + 1, c, tn);
    if (!kPrefetch || lt == lm) tail_dense_load(P, m);
    if (lm == 1)
      tail_dense<T1, T1>(P, R1, m, lds);
    else
      tail_dense<T, T>(P, R, m, lds);
    if (lt == lm) {  // the matrix is the whole tail
      const LevelD& V = P.lv[lm];
      const int n = V.nx * V.ny;
      if (lm == 1) {
        if (c < n) {
#pragma unroll
          for (int q = 0; q < 8; ++q) G1[0][q] = ((const T1*)lds)[(1 + q) * kTailThreads + c];
        }
        tail_store1<T1>(V, V.gA, c, G1);
      } else {
        if (c < n) {
#pragma unroll
          for (int q = 0; q < 8; ++q) G[0][q] = ((const T*)lds)[(1 + q) * kTailThreads + c];
        }
        tail_store1<T>(V, V.gA, c, G);
      }
    }
  }
  // ---- ascent: iterate plus injected coarse correction, K post-smoothing
  // sweeps; the coarse level's result sits in LDS after its sD plane
  for (int l = low + 1; l <= lt; ++l) {
    const LevelD& V = P.lv[l];
    const int nx = V.nx, ny = V.ny, n = nx * ny;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      G[0][q] = Gn[0][q];
      R[0][q] = Rn[0][q];
    }
    if (c < n) {
      const int y = tail_row(c, V.inv_nx), ci = (y >> 1) * (nx / 2) + ((c - y * nx) >> 1);
      if (l == 2) {
        const T1* ex = (const T1*)lds + kTailThreads;
#pragma unroll
        for (int q = 0; q < 8; ++q) G[0][q] += T(ex[q * kTailThreads + ci]);
      } else {
        const T* ex = (const T*)lds + kTailThreads;
#pragma unroll
        for (int q = 0; q < 8; ++q) G[0][q] += ex[q * kTailThreads + ci];
      }
    }
    if (kPrefetch && l + 1 <= lt) {
      tail_load1<T>(P.lv[l + 1], P.lv[l + 1].gA, c, Gn);
      tail_load1<T>(P.lv[l + 1], P.lv[l + 1].r, c, Rn);
    }
    __syncthreads();  // the sweeps' sD overlaps the coarse result just read
    T* sD = (T*)lds;
    T* sG = sD + kTailThreads;
    if (kPrefetch) {
      tb = tn;
      tail_tab_signs(tb);
      if (l + 1 <= lt) tail_tab_load(P, l + 1, c, tn);
    } else {
      tail_tab_load(P, l, c, tb);
      tail_tab_signs(tb);
    }
    for (int s = 0; s < K; ++s) tail_relax<T>(k, n, tb, G, R, sD, sG, true);
    if (l == lt) {
      tail_store1<T>(V, V.gA, c, G);
    } else {
      if (!kPrefetch) {
        tail_load1<T>(P.lv[l + 1], P.lv[l + 1].gA, c, Gn);
        tail_load1<T>(P.lv[l + 1], P.lv[l + 1].r, c, Rn);
      }
      __syncthreads();  // every pull has read sG
      if (c < n) {
#pragma unroll
        for (int q = 0; q < 8; ++q) sG[q * kTailThreads + c] = G[0][q];
      }
      __syncthreads();
    }
  }
}

// ---- cycle-shaped tail: W- and F-visits, and visits that continue from the
// top level's stored iterate.  The recursion of the cycle runs as a loop over
// an explicit per-level stack whose entries are the same for every thread, so
// every barrier is reached by the whole workgroup.  Between levels a thread
// passes only its own cells through global memory (iterate in buffer A,
// right-hand side in r); the coarse correction that finer cells read from
// other threads passes through LDS, as in tail_run.

// the coarse result handed to the finer level: plane q of cell c at
// lds + (1 + q) 1024 in the level's type
template <typename TT>
__device__ __forceinline__ void tail_hand_up(char* lds, int n, const TT (&G)[1][8]) {
  const int c = threadIdx.x;
  TT* sG = (TT*)lds + kTailThreads;
  __syncthreads();  // every pull of the last sweep has read sG
  if (c < n) {
#pragma unroll
    for (int q = 0; q < 8; ++q) sG[q * kTailThreads + c] = G[0][q];
  }
  __syncthreads();
}

// the residual G of level l >= 2 (one cell per thread) summed over 2 x 2
// blocks into level l - 1's right-hand side (type T, or T1 for level 1),
// through LDS; the LDS may be reused after the return
template <typename T, typename T1>
__device__ __forceinline__ void tail_restrict(const ProbD& P, int l, const T (&G)[1][8], char* lds) {
  const int c = threadIdx.x;
  const LevelD& V = P.lv[l];
  const int nx = V.nx, ny = V.ny, n = nx * ny;
  T* sG = (T*)lds + kTailThreads;
  __syncthreads();  // every pull of the residual sweep has read sG
  if (c < n) {
#pragma unroll
    for (int q = 0; q < 8; ++q) sG[q * kTailThreads + c] = G[0][q];
  }
  __syncthreads();
  const LevelD& C = P.lv[l - 1];
  const int cnx = nx / 2, cn = cnx * (ny / 2);
  T sum[8];
  if (c < cn) {
    const int f0 = 2 * c + 2 * cnx * tail_row(c, C.inv_nx), f1 = f0 + nx;  // fine cell (2 X, 2 Y) of (X, Y) = c
#pragma unroll
    for (int q = 0; q < 8; ++q) sum[q] = (sG[q * kTailThreads + f0] + sG[q * kTailThreads + f0 + 1]) + (sG[q * kTailThreads + f1] + sG[q * kTailThreads + f1 + 1]);
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) sum[q] = T(0);
  }
  if (l - 1 >= 2) {
    T Rc[1][8];
#pragma unroll
    for (int q = 0; q < 8; ++q) Rc[0][q] = sum[q];
    tail_store1<T>(C, C.r, c, Rc);
  } else {
    T1 Rc[1][8];
#pragma unroll
    for (int q = 0; q < 8; ++q) Rc[0][q] = T1(sum[q]);
    tail_store1<T1>(C, C.r, c, Rc);
  }
  __syncthreads();  // sG is reused by the next level
}

// pre-smoothing of level l >= 2 (K sweeps from zero or from buffer A), the
// iterate stored to A, the residual restricted into level l - 1's r
template <typename T, typename T1>
__device__ __forceinline__ void tail_pre(const ProbD& P, int l, int K, bool zero, char* lds) {
  const int c = threadIdx.x;
  const LevelD& V = P.lv[l];
  const int nx = V.nx, ny = V.ny, n = nx * ny;
  T* sD = (T*)lds;
  T* sG = sD + kTailThreads;
  const ElConst<T> k = tail_consts<T>(P);
  TailTab tb;
  T G[1][8], R[1][8];
  tail_tab_load(P, l, c, tb);
  tail_tab_signs(tb);
  tail_load1<T>(V, V.r, c, R);
  if (zero)
    tail_zero(G);
  else
    tail_load1<T>(V, V.gA, c, G);
  for (int s = 0; s < K; ++s) tail_relax<T>(k, n, tb, G, R, sD, sG, true);
  tail_store1<T>(V, V.gA, c, G);
  tail_relax<T>(k, n, tb, G, R, sD, sG, false);
  tail_restrict<T, T1>(P, l, G, lds);
}

// the coarsest level: its sweeps (2K unless the problem sets another count)
// from zero or from buffer A, stored to A and handed up through LDS
template <typename T1>
__device__ __forceinline__ void tail_coarsest(const ProbD& P, int K, bool zero, char* lds) {
  const int c = threadIdx.x;
  const LevelD& V = P.lv[1];
  const int n = V.nx * V.ny;
  T1* sD = (T1*)lds;
  T1* sG = sD + kTailThreads;
  const ElConst<T1> k = tail_consts<T1>(P);
  TailTab tb;
  T1 G[1][8], R[1][8];
  tail_tab_load(P, 1, c, tb);
  tail_tab_signs(tb);
  tail_load1<T1>(V, V.r, c, R);
  if (zero)
    tail_zero(G);
  else
    tail_load1<T1>(V, V.gA, c, G);
  for (int s = 0; s < P.csweeps; ++s) tail_relax<T1>(k, n, tb, G, R, sD, sG, true);
  tail_store1<T1>(V, V.gA, c, G);
  tail_hand_up<T1>(lds, n, G);
}

// post-smoothing of level l >= 2: its stored iterate plus the injected coarse
// correction (in LDS, type TC), K sweeps, stored to A and handed up
template <typename T, typename TC>
__device__ __forceinline__ void tail_post(const ProbD& P, int l, int K, char* lds) {
  const int c = threadIdx.x;
  const LevelD& V = P.lv[l];
  const int nx = V.nx, ny = V.ny, n = nx * ny;
  TailTab tb;
  T G[1][8], R[1][8];
  tail_tab_load(P, l, c, tb);
  tail_tab_signs(tb);
  tail_load1<T>(V, V.gA, c, G);
  tail_load1<T>(V, V.r, c, R);
  if (c < n) {
    const int y = tail_row(c, V.inv_nx), ci = (y >> 1) * (nx / 2) + ((c - y * nx) >> 1);
    const TC* ex = (const TC*)lds + kTailThreads;
#pragma unroll
    for (int q = 0; q < 8; ++q) G[0][q] += T(ex[q * kTailThreads + ci]);
  }
  __syncthreads();  // the sweeps' sD overlaps the coarse result just read
  T* sD = (T*)lds;
  T* sG = sD + kTailThreads;
  const ElConst<T> k = tail_consts<T>(P);
  for (int s = 0; s < K; ++s) tail_relax<T>(k, n, tb, G, R, sD, sG, true);
  tail_store1<T>(V, V.gA, c, G);
  tail_hand_up<T>(lds, n, G);
}

// one visit of shape `shape` of levels lt..1: V one coarse visit, W two
// W-visits, F an F-visit then a V-visit; every coarse visit after the first
// continues from the coarse level's stored iterate
template <typename T, typename T1>
__device__ __forceinline__ void tail_run_shaped(const ProbD& P, int lt, int K, int shape, bool zero, char* lds) {
  // per level: the shape of its current visit (2 bits at 2 l) and whether a
  // second coarse visit is still to start (bit l); uniform over the workgroup
  uint32_t shp = uint32_t(shape) << (2 * lt), second = 0;
  auto shape_of = [&](int lv) { return int((shp >> (2 * lv)) & 3u); };
  auto set_shape = [&](int lv, int v) { shp = (shp & ~(3u << (2 * lv))) | (uint32_t(v) << (2 * lv)); };
  int l = lt;
  bool z = zero, entering = true;
  for (;;) {
    if (entering) {
      if (l == 1) {
        tail_coarsest<T1>(P, K, z, lds);
        if (lt == 1) break;
        l = 2;
        entering = false;
        continue;
      }
      tail_pre<T, T1>(P, l, K, z, lds);
      const int sh = shape_of(l);
      if (sh != 0) second |= 1u << l;  // W and F visit the coarser level twice
      set_shape(l - 1, sh);            // the first visit: W-, F- or V-visit as this one
      --l;
      z = true;
      continue;
    }
    // back on level l from a visit of level l - 1
    if (second & (1u << l)) {
      second &= ~(1u << l);
      set_shape(l - 1, shape_of(l) == 1 ? 1 : 0);  // W: another W-visit; F: a V-visit
      --l;
      z = false;  // continuing from the first visit's iterate
      entering = true;
      continue;
    }
    if (l == 2)
      tail_post<T, T1>(P, l, K, lds);
    else
      tail_post<T, T>(P, l, K, lds);
    if (l == lt) break;
    ++l;
  }
}

// ---- whole-problem tail: the finest level too, for problems of at most
// one workgroup's cells.  Its sweeps add the explicit force to the
// self-force and its wall terms (per cell and population, scaled like the
// post-collision populations) to the pulled values; R = 0 there.

// the finest level's force of this thread's cell, and its wall terms in LDS
// (thread c's own entries q kTailThreads + c; read by the waves that hold a
// wall cell alone)
template <typename T>
struct TailFine {
  T Fx, Fy;
  const T* add;
  bool wall;  // uniform over the wave
};

// one application of S on the finest level held by the workgroup (one cell
// per thread): as tail_relax with the force and wall terms f.
// mode 1: G <- (1 - gamma) G + gamma S(G); 0: G <- G - S(G); 3 (the
// measuring sweep): G <- (1 - gamma) G + gamma S(G) from the unscaled S(G),
// adding ||G - S(G)||^2 and ||G||^2 of the cell to (mr, mg) in FP64
template <typename T>
__device__ __forceinline__ void tail_relax_fine(const ElConst<T>& k, int n, const TailTab& tb, T (&G)[1][8],
                                                const TailFine<T>& f, T* sD, T* sG, int mode,
                                                double* mr = nullptr, double* mg = nullptr) {
  const int c = threadIdx.x;
  const bool blend = mode == 1;
  if (c < n) sD[c] = k.kD * el_ms(G[0]);
  __syncthreads();
  const T sc = blend ? k.gamma : T(1);
  if (c < n) {
    T gx_, gy_;
    tail_grad(tb, sD, gx_, gy_);
    T u[8], s8[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) u[q] = G[0][q];
    el_collide(u, k.cstar * gx_ + f.Fx, k.cstar * gy_ + f.Fy, k, s8, sc);
#pragma unroll
    for (int q = 0; q < 8; ++q) sG[q * kTailThreads + c] = s8[q];
  }
  __syncthreads();
  const T omg = T(1) - k.gamma;
  if (c < n) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      T gi = tail_pull(tb, sG, q);
      if (f.wall) gi += sc * f.add[q * kTailThreads + c];
      if (mode == 3) {
        const double rho = double(G[0][q]) - double(gi);
        *mr += rho * rho;
        *mg += double(G[0][q]) * double(G[0][q]);
        G[0][q] = omg * G[0][q] + k.gamma * gi;
      } else {
        G[0][q] = blend ? omg * G[0][q] + gi : G[0][q] - gi;
      }
    }
  }
}

// the finest level's force and wall terms, loaded into LDS once per launch
// (every phase of every cycle uses them; registers held across the phases
// would spill): 8 planes of wall terms, then the force's two.  A serial chain
// of sweeps bounds the launch (loads in each phase cost 7% of it)
template <typename T>
__device__ __forceinline__ bool tail_fine_load(const ProbD& P, const LevelD& V, T* sF) {
  const int c = threadIdx.x;
  bool wall = false;
  if (c < V.nx * V.ny) {
    const int64_t idx = (int64_t)tail_row(c, V.inv_nx) * (V.pitch - V.nx) + c;
    const T* F = (const T*)P.Ft;
    const T* ad = (const T*)P.addt;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const T v = ad[q * V.plane + idx];
      wall = wall || v != T(0);
      sF[q * kTailThreads + c] = v;
    }
    sF[8 * kTailThreads + c] = F[idx];
    sF[9 * kTailThreads + c] = F[V.plane + idx];
  }
  return __any(wall);
}
template <typename T>
__device__ __forceinline__ TailFine<T> tail_fine_terms(const T* sF, bool wall) {
  const int c = threadIdx.x;
  return {sF[8 * kTailThreads + c], sF[9 * kTailThreads + c], sF, wall};
}

// pre-smoothing of the finest level L from buffer A or B (npre sweeps), the
// iterate stored to A, the residual restricted into level L - 1's r
template <typename T, typename T1>
__device__ __forceinline__ void tail_fine_pre_g(const ProbD& P, int L, int npre, T (&G)[1][8], char* lds, const T* sF,
                                                bool wall) {
  const int c = threadIdx.x;
  const LevelD& V = P.lv[L];
  const int nx = V.nx, ny = V.ny, n = nx * ny;
  T* sD = (T*)lds;
  T* sG = sD + kTailThreads;
  const ElConst<T> k = tail_consts<T>(P);
  TailTab tb;
  tail_tab_load(P, L, c, tb);
  tail_tab_signs(tb);
  const TailFine<T> f = tail_fine_terms<T>(sF, wall);
  for (int s = 0; s < npre; ++s) tail_relax_fine<T>(k, n, tb, G, f, sD, sG, 1);
  tail_store1<T>(V, V.gA, c, G);
  tail_relax_fine<T>(k, n, tb, G, f, sD, sG, 0);
  tail_restrict<T, T1>(P, L, G, lds);
}

// post-smoothing of the finest level: its stored iterate plus the injected
// coarse correction (in LDS, type TC), K sweeps, stored to A
template <typename T, typename TC>
__device__ __forceinline__ void tail_fine_post(const ProbD& P, int L, int K, char* lds, const T* sF, bool wall) {
  const int c = threadIdx.x;
  const LevelD& V = P.lv[L];
  const int nx = V.nx, ny = V.ny, n = nx * ny;
  TailTab tb;
  T G[1][8];
  tail_tab_load(P, L, c, tb);
  tail_tab_signs(tb);
  tail_load1<T>(V, V.gA, c, G);
  if (c < n) {
    const int y = tail_row(c, V.inv_nx), ci = (y >> 1) * (nx / 2) + ((c - y * nx) >> 1);
    const TC* ex = (const TC*)lds + kTailThreads;
#pragma unroll
    for (int q = 0; q < 8; ++q) G[0][q] += T(ex[q * kTailThreads + ci]);
  }
  __syncthreads();  // the sweeps' sD overlaps the coarse result just read
  T* sD = (T*)lds;
  T* sG = sD + kTailThreads;
  const ElConst<T> k = tail_consts<T>(P);
  const TailFine<T> f = tail_fine_terms<T>(sF, wall);
  for (int s = 0; s < K; ++s) tail_relax_fine<T>(k, n, tb, G, f, sD, sG, 1);
  tail_store1<T>(V, V.gA, c, G);
}

// the stopping test's state of the in-kernel adaptive loop, in LDS past the
// levels' kTailLdsBytes
struct TailFullState {
  double ratio, rr, gg;
  int stopped, count;
};
// (levels, the test's state, the finest level's terms: 156 of 160 KiB in FP64)
template <typename T> constexpr int tail_full_lds() { return kTailLdsBytes + 64 + 10 * kTailThreads * (int)sizeof(T); }
static_assert(tail_full_lds<double>() <= 160 * 1024, "one workgroup's LDS");
static_assert(sizeof(TailFullState) <= 64, "state fits its LDS slot");

// one cycle of the whole problem: pre-smoothing from buffer A or B, the
// coarse correction (one visit, or two for W (W, W) and F (F, V)), the
// post-smoothing into A
template <typename T>
__device__ __forceinline__ void tail_full_cycle(const ProbD& P, const TailL& a, int npre, T (&G)[1][8], char* lds,
                                                const T* sF, bool wall) {
  const int L = P.L;
  tail_fine_pre_g<T, double>(P, L, npre, G, lds, sF, wall);
  const int visits = a.shape != 0 ? 2 : 1;
  for (int v = 0; v < visits; ++v)  // one call site: one inlined copy of the recursion
    tail_run_shaped<T, double>(P, L - 1, a.K, v == 0 ? a.shape : (a.shape == 1 ? 1 : 0), v == 0, lds);
  if (L == 2)
    tail_fine_post<T, double>(P, L, a.K, lds, sF, wall);
  else
    tail_fine_post<T, T>(P, L, a.K, lds, sF, wall);
}

// the measuring sweep of the adaptive schedule on the finest level: one
// smoothing application of the iterate in A (its result, which the next
// cycle continues from, left in G), with the FP64 squares ||g - S(g)||^2 and
// ||g||^2 summed over the level in a fixed order (lanes, then waves)
template <typename T>
__device__ __forceinline__ void tail_measure(const ProbD& P, char* lds, T (&G)[1][8], double& rr, double& gg, const T* sF,
                                             bool wall) {
  const int c = threadIdx.x;
  const LevelD& V = P.lv[P.L];
  const int n = V.nx * V.ny;
  T* sD = (T*)lds;
  T* sG = sD + kTailThreads;
  const ElConst<T> k = tail_consts<T>(P);
  TailTab tb;
  tail_tab_load(P, P.L, c, tb);
  tail_tab_signs(tb);
  tail_load1<T>(V, V.gA, c, G);
  double r = 0.0, g = 0.0;
  tail_relax_fine<T>(k, n, tb, G, tail_fine_terms<T>(sF, wall), sD, sG, 3, &r, &g);
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    r += __shfl_down(r, o, kWave);
    g += __shfl_down(g, o, kWave);
  }
  __syncthreads();  // every pull has read sG: reuse the LDS for the sums
  double* sw = (double*)lds;
  const int w = c / kWave, nw = kTailThreads / kWave;
  if (c % kWave == 0) {
    sw[w] = r;
    sw[nw + w] = g;
  }
  __syncthreads();
  rr = 0.0;
  gg = 0.0;
  if (c == 0)
    for (int v = 0; v < nw; ++v) {
      rr += sw[v];
      gg += sw[nw + v];
    }
}

template <typename T>
__global__ __launch_bounds__(kTailThreads) void k_tail_full(TailL a) {
  if (gated_off(a.skip, a.need)) return;  // uniform over the grid
  extern __shared__ char lds[];
  const ProbD& P = constant(a.probs + a.pids[2 * blockIdx.x]);  // (problem, 0) entries
  const int L = P.L;
  if (L < 2 || L - 1 > kTailMaxLevel || !P.addt) return;  // uniform; the host never asks for it
  // without the loop: one cycle from buffer fine_in with fine_pre
  // pre-smoothing sweeps.  With it: all cycles of the step, the first from A
  // unconditionally, each later one after the measuring sweep and the
  // stopping test, which thread 0 takes in the FP64 steps of the tile
  // schedule's test and hands to every thread; at most ne_max + 1 passes (the
  // test stops at ne_max cycles).  The test's state sits in LDS past what the
  // levels use (registers held across the cycles would spill) and is stored
  // once at the end.  One call site of the cycle: one inlined copy.
  TailFullState* st = (TailFullState*)(lds + kTailLdsBytes);
  if (a.loop && threadIdx.x == 0) {
    st->stopped = P.ad[0];
    st->count = P.ad[1];
    st->ratio = 0.0;
    st->rr = 0.0;
    st->gg = 0.0;
  }
  T* sF = (T*)(lds + kTailLdsBytes + 64);
  const bool wall = tail_fine_load<T>(P, P.lv[L], sF);
  T G[1][8];
  tail_load1<T>(P.lv[L], (!a.loop && a.fine_in) ? P.lv[L].gB : P.lv[L].gA, threadIdx.x, G);
  int npre = a.loop ? a.K : a.fine_pre;
  for (int pass = 0; pass <= a.ne_max; ++pass) {
    tail_full_cycle<T>(P, a, npre, G, lds, sF, wall);
    if (!a.loop) break;
    double rr, gg;
    tail_measure<T>(P, lds, G, rr, gg, sF, wall);
    if (threadIdx.x == 0) {
      st->rr = rr;
      st->gg = gg;
      if (!isfinite(rr) || !isfinite(gg)) P.flags[0] = 1;
      if (!st->stopped) {
        const double nr = sqrt(rr), ng = sqrt(gg);
        st->ratio = ng > 0 ? nr / ng : 0.0;
        if (!isfinite(nr) || !isfinite(ng))
          st->stopped = 2;
        else if (nr <= a.tol * ng || st->count >= a.ne_max)
          st->stopped = 1;
        else
          st->count += 1;
      }
    }
    __syncthreads();
    const bool stop = st->stopped != 0;
    __syncthreads();  // the LDS is reused by the next cycle
    if (stop) break;
    npre = a.K - 1;
  }
  if (a.loop && threadIdx.x == 0) {
    P.norm2[0] = st->rr;
    P.norm2[1] = st->gg;
    P.ad_ratio[0] = st->ratio;
    P.ad[1] = st->count;
    P.ad[0] = st->stopped;
  }
}

template <typename T>
__global__ __launch_bounds__(kTailThreads) void k_tail_shaped(TailL a) {
  if (gated_off(a.skip, a.need)) return;  // uniform over the grid
  extern __shared__ char lds[];
  const ProbD& P = constant(a.probs + a.pids[2 * blockIdx.x]);  // (problem, 0) entries
  const int lt = P.L - a.depth;
  if (lt < 1 || lt > kTailMaxLevel) return;  // uniform; the host never asks for it
  tail_run_shaped<T, double>(P, lt, a.K, a.shape, a.from_zero != 0, lds);
}

template <typename T>
__global__ __launch_bounds__(kTailThreads) void k_tail(TailL a) {
  if (gated_off(a.skip, a.need)) return;  // uniform over the grid
  extern __shared__ char lds[];
  // (problem, depth) entries: with a.depth < 0 each problem's tail starts at
  // the entry's depth, else at the launch's
  const ProbD& P = constant(a.probs + a.pids[2 * blockIdx.x]);
  tail_run<T, double>(P, P.L - (a.depth < 0 ? a.pids[2 * blockIdx.x + 1] : a.depth), a.K, lds);
}

hipError_t launch_tail(const TailL& a, int nprobs, bool dbl, hipStream_t s) {
  if (nprobs <= 0) return hipSuccess;
  static bool attr = false;
  if (!attr) {
    const void* ks[6] = {(const void*)k_tail<float>,        (const void*)k_tail<double>,
                         (const void*)k_tail_shaped<float>, (const void*)k_tail_shaped<double>,
                         (const void*)k_tail_full<float>,   (const void*)k_tail_full<double>};
    for (int i = 0; i < 6; ++i) {
      const hipError_t e = hipFuncSetAttribute(ks[i], hipFuncAttributeMaxDynamicSharedMemorySize,
                                               i == 4 ? tail_full_lds<float>() : (i == 5 ? tail_full_lds<double>() : kTailLdsBytes));
      if (e != hipSuccess) return e;
    }
    attr = true;
  }
  // the V-cycle from a zero iterate (the time step's own visit) takes the
  // prefetching kernel; other shapes and continued visits the shaped one
  const bool shaped = a.shape != 0 || !a.from_zero;
  if (a.full && dbl)
    hipLaunchKernelGGL(k_tail_full<double>, dim3(nprobs), dim3(kTailThreads), tail_full_lds<double>(), s, a);
  else if (a.full)
    hipLaunchKernelGGL(k_tail_full<float>, dim3(nprobs), dim3(kTailThreads), tail_full_lds<float>(), s, a);
  else if (shaped && dbl)
    hipLaunchKernelGGL(k_tail_shaped<double>, dim3(nprobs), dim3(kTailThreads), kTailLdsBytes, s, a);
  else if (shaped)
    hipLaunchKernelGGL(k_tail_shaped<float>, dim3(nprobs), dim3(kTailThreads), kTailLdsBytes, s, a);
  else if (dbl)
    hipLaunchKernelGGL(k_tail<double>, dim3(nprobs), dim3(kTailThreads), kTailLdsBytes, s, a);
  else
    hipLaunchKernelGGL(k_tail<float>, dim3(nprobs), dim3(kTailThreads), kTailLdsBytes, s, a);
  return hipGetLastError();
}

// ======================================================================
// per-problem kernels
// ======================================================================
__global__ __launch_bounds__(256) void k_finalize(ProbL a) {
  if (gated_off(a.skip, a.need)) return;  // uniform over the grid
  __shared__ double sr[256], sg[256];
  finalize_norms(a, a.pids[blockIdx.x], sr, sg);
}

__global__ __launch_bounds__(256) void k_copy(uint4* dst, const uint4* src, size_t n16) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n16; k += stride) dst[k] = src[k];
}

__global__ __launch_bounds__(256) void k_zero(uint4* dst, size_t n16) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n16; k += stride) dst[k] = make_uint4(0, 0, 0, 0);
}

__global__ void k_ad_reset(ProbL a) {
  if (gated_off(a.skip, a.need)) return;
  if (threadIdx.x == 0) {
    const ProbD& P = a.probs[a.pids[0]];
    P.ad[0] = 0;
    P.ad[1] = 1;  // the first cycle runs unconditionally
  }
}

hipError_t launch_ad_reset(const ProbL& a, hipStream_t s) {
  hipLaunchKernelGGL(k_ad_reset, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_finalize(const ProbL& a, int nprobs, hipStream_t s) {
  if (nprobs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_finalize, dim3(nprobs), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const size_t n16 = bytes / 16;
  int blocks = (int)((n16 + 255) / 256);
  if (blocks > 8192) blocks = 8192;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_copy, dim3(blocks), dim3(256), 0, s, (uint4*)dst, (const uint4*)src, n16);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* dst, size_t bytes, hipStream_t s) {
  const size_t n16 = bytes / 16;
  int blocks = (int)((n16 + 255) / 256);
  if (blocks > 8192) blocks = 8192;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_zero, dim3(blocks), dim3(256), 0, s, (uint4*)dst, n16);
  return hipGetLastError();
}

// ---------------------------------------------------------- instantiations
#define BIOT_SWEEP(T, Tc)                                                                        \
  template hipError_t launch_tsweep<T, Tc, kSmooth, false>(const SweepL&, int, hipStream_t);     \
  template hipError_t launch_tsweep<T, Tc, kRestrict, false>(const SweepL&, int, hipStream_t);   \
  template hipError_t launch_tsweep<T, Tc, kApply, false>(const SweepL&, int, hipStream_t);      \
  template hipError_t launch_tsweep<T, Tc, kSmooth, true>(const SweepL&, int, hipStream_t);      \
  template hipError_t launch_tsweep<T, Tc, kRestrict, true>(const SweepL&, int, hipStream_t);    \
  template hipError_t launch_tsweep<T, Tc, kApply, true>(const SweepL&, int, hipStream_t);
BIOT_SWEEP(float, float)
BIOT_SWEEP(float, double)
BIOT_SWEEP(double, double)
#undef BIOT_SWEEP
#define BIOT_SWEEPN_ALT(T, Tc, ALT)                                                                    \
  template hipError_t launch_tsweep2<T, Tc, true, true, 2, false, ALT>(const SweepL&, int, bool, hipStream_t);  \
  template hipError_t launch_tsweep2<T, Tc, true, false, 2, false, ALT>(const SweepL&, int, bool, hipStream_t); \
  template hipError_t launch_tsweep2<T, Tc, true, true, 2, true, ALT>(const SweepL&, int, bool, hipStream_t);   \
  template hipError_t launch_tsweep2<T, Tc, true, false, 2, true, ALT>(const SweepL&, int, bool, hipStream_t);  \
  template hipError_t launch_tsweep2<T, Tc, false, false, 2, false, ALT>(const SweepL&, int, bool, hipStream_t); \
  template hipError_t launch_tsweep2<T, Tc, false, false, 2, true, ALT>(const SweepL&, int, bool, hipStream_t);  \
  template hipError_t launch_tsweep2<T, Tc, false, false, 4, true, ALT>(const SweepL&, int, bool, hipStream_t);  \
  template hipError_t launch_tsweep2<T, Tc, true, false, 4, true, ALT>(const SweepL&, int, bool, hipStream_t);  \
  template hipError_t launch_tsweep2<T, Tc, false, false, 4, false, ALT>(const SweepL&, int, bool, hipStream_t); \
  template hipError_t launch_tsweep2<T, Tc, true, false, 4, false, ALT>(const SweepL&, int, bool, hipStream_t);
#define BIOT_SWEEPN(T, Tc)                                                                            \
  BIOT_SWEEPN_ALT(T, Tc, false)                                                                       \
  BIOT_SWEEPN_ALT(T, Tc, true)
BIOT_SWEEPN(float, float)
BIOT_SWEEPN(float, double)
BIOT_SWEEPN(double, double)
#undef BIOT_SWEEPN
#undef BIOT_SWEEPN_ALT
#define BIOT_SWEEPN_WIDE(T, Tc)                                                            \
  template hipError_t launch_tsweep2_wide<T, Tc, false, false>(const SweepL&, int, hipStream_t); \
  template hipError_t launch_tsweep2_wide<T, Tc, false, true>(const SweepL&, int, hipStream_t);  \
  template hipError_t launch_tsweep2_wide<T, Tc, true, false>(const SweepL&, int, hipStream_t);  \
  template hipError_t launch_tsweep2_wide<T, Tc, true, true>(const SweepL&, int, hipStream_t);
BIOT_SWEEPN_WIDE(float, float)
BIOT_SWEEPN_WIDE(float, double)
BIOT_SWEEPN_WIDE(double, double)
#undef BIOT_SWEEPN_WIDE
template hipError_t launch_tsweep2<float, float, true, true, 4, false>(const SweepL&, int, bool, hipStream_t);
template hipError_t launch_tsweep2<float, float, true, true, 4, true>(const SweepL&, int, bool, hipStream_t);
template hipError_t launch_tsweep2<float, double, true, true, 4, false>(const SweepL&, int, bool, hipStream_t);
template hipError_t launch_tsweep2<float, double, true, true, 4, true>(const SweepL&, int, bool, hipStream_t);
template hipError_t launch_tsweep2<float, float, true, true, 4, false, true>(const SweepL&, int, bool, hipStream_t);
template hipError_t launch_tsweep2<float, double, true, true, 4, false, true>(const SweepL&, int, bool, hipStream_t);
template hipError_t launch_tsweep2<float, float, true, true, 4, true, true>(const SweepL&, int, bool, hipStream_t);
template hipError_t launch_tsweep2<float, double, true, true, 4, true, true>(const SweepL&, int, bool, hipStream_t);
// FP64 shifted storage has no LDS room for four applications; the schedule
// never asks for them (these stubs keep the dispatch table complete)
template <>
hipError_t launch_tsweep2<double, double, true, true, 4, false>(const SweepL&, int, bool, hipStream_t) {
  return hipErrorInvalidConfiguration;
}
template <>
hipError_t launch_tsweep2<double, double, true, true, 4, true>(const SweepL&, int, bool, hipStream_t) {
  return hipErrorInvalidConfiguration;
}
template <>
hipError_t launch_tsweep2<double, double, true, true, 4, false, true>(const SweepL&, int, bool, hipStream_t) {
  return hipErrorInvalidConfiguration;
}
template <>
hipError_t launch_tsweep2<double, double, true, true, 4, true, true>(const SweepL&, int, bool, hipStream_t) {
  return hipErrorInvalidConfiguration;
}
template hipError_t launch_tflow<float, false>(const CellL&, int, hipStream_t);
template hipError_t launch_tflow<float, true>(const CellL&, int, hipStream_t);
template hipError_t launch_tflow<double, false>(const CellL&, int, hipStream_t);
template hipError_t launch_tflow<double, true>(const CellL&, int, hipStream_t);
template hipError_t launch_force<float>(const CellL&, int, hipStream_t);
template hipError_t launch_force<double>(const CellL&, int, hipStream_t);
template hipError_t launch_init<float>(const CellL&, int, hipStream_t);
template hipError_t launch_init<double>(const CellL&, int, hipStream_t);
template hipError_t launch_rebase<float>(const CellL&, int, hipStream_t);
template hipError_t launch_rebase<double>(const CellL&, int, hipStream_t);
template hipError_t launch_rebase_force<float>(const CellL&, int, hipStream_t);
template hipError_t launch_rebase_force<double>(const CellL&, int, hipStream_t);
template hipError_t launch_extract<float, false>(const ExtractL&, int, hipStream_t);
template hipError_t launch_extract<float, true>(const ExtractL&, int, hipStream_t);
template hipError_t launch_extract<double, false>(const ExtractL&, int, hipStream_t);
template hipError_t launch_extract<double, true>(const ExtractL&, int, hipStream_t);

}  // namespace biot
