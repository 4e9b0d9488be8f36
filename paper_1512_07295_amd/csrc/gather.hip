// Adjoint gather of the P(k) gradient (the transpose of the deposit, Sec. 2.3
// kernels differentiated): every particle reads its stencils on the grids of
// its set.
//
// What bounds it (gfx950): cache lines per load instruction, and the latency
// of the loads with few waves.  So a stencil's cells along z are read as one
// row (16-byte loads, both components of a complex grid), not cell by cell;
// PCS particles are split over four lanes, one x plane each (order 6: two
// lanes), which brings 32 B x 4 rows x 2 grids of one lane in flight at 90
// VGPRs; the rows of a pair's two grids are read in turn, since they mostly
// share cache lines.  PCS pair, one thread per particle reading cells -> now:
// 128^3 particles on 256^3 in lattice order 0.213 -> 0.140 ms, in random
// order 1.40 -> 1.12 (grids one after the other: 0.120 and 1.47), 64^3 on
// 240^3 46 -> 37 us, on 100^3 32 -> 25, on 64^3 25 -> 25; order 6 0.87 ->
// 0.49 ms, 3 94 -> 88 us, 2 37 -> 36 us, eight grids on 200^3 91 -> 61 us.
#include "particles.hpp"

namespace fsest {

// ------------------------------------------------------------------ adjoint gather
// dL/dx_{j,alpha} = -(N/L) sum_a sum_{g in stencil_a} G_a(g) W'(s_alpha) prod_{beta != alpha} W(s_beta)
// where G_a = dL/drho_a sits in the grid buffer with the deposit's layout.
// IL: 0 one grid, 1 the interlaced pair, 2 the g.ng grids of interlace codes 2
// and 3 (grid gi: shift mask grid_mask(code, gi), component gi % 2 of slab
// gi / 2 of its set)
typedef float f4_t __attribute__((ext_vector_type(4), aligned(4)));
typedef float f2_t __attribute__((ext_vector_type(2), aligned(4)));

// K consecutive floats in as few loads as there are
template <int K>
__device__ __forceinline__ void load_row(const float* __restrict__ p, float (&v)[K]) {
  constexpr int K4 = K / 4 * 4;
#pragma unroll
  for (int i = 0; i < K4; i += 4) {
    const f4_t r = *(const f4_t*)(p + i);
    v[i] = r.x, v[i + 1] = r.y, v[i + 2] = r.z, v[i + 3] = r.w;
  }
  if constexpr (K - K4 >= 2) {
    const f2_t r = *(const f2_t*)(p + K4);
    v[K4] = r.x, v[K4 + 1] = r.y;
  }
  if constexpr (K % 2) v[K - 1] = p[K - 1];
}

// lanes that share a particle, its x planes split evenly: one where the
// stencil is short (order 2: 36 us with one lane, 40 with two) or odd
template <int P>
__host__ __device__ constexpr int gather_lanes() { return P == 4 ? 4 : P == 6 ? 2 : 1; }

// order 3: 128 VGPRs instead of 132, four waves per SIMD instead of three
// (pair of 256^3 grids 97 -> 88 us)
template <int P, int IL, typename TP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(P == 3 ? 4 : 1))) void k_gather_grad(const TP* __restrict__ pos, int64_t n_total,
                                                     const int64_t* __restrict__ offsets,
                                                     const float* __restrict__ grid, Geom g,
                                                     const float* __restrict__ w,
                                                     TP* __restrict__ grad) {
  constexpr int G = gather_lanes<P>();
  constexpr int PPL = P / G;     // x planes per lane
  constexpr int W = 64 / G;      // particles per wave
  constexpr int S = IL ? 2 : 1;  // floats per cell
  const int lane = threadIdx.x & 63;
  const int part = lane / W;     // which of the particle's lanes
  const int64_t j = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * W + lane % W;
  const bool valid = j < n_total;
  const int64_t jj = valid ? j : n_total - 1;
  double x, y, z;
  load_pos(pos, jj, x, y, z);
  const int mock = mock_of(offsets, g.batch, jj);
  const int n = g.n;
  const double u[3] = {grid_coord(x, g.box, g.inv), grid_coord(y, g.box, g.inv),
                       grid_coord(z, g.box, g.inv)};
  float gx = 0.0f, gy = 0.0f, gz = 0.0f;
  const int pitch = IL ? 2 * g.nz : n;
  // the pair's two grids lie in the same complex elements: row by row
  // together, so that the second grid's rows are still in the cache
  constexpr int H = IL ? 2 : 1;
  const int nslab = IL == 2 ? g.npair : 1;
#pragma unroll 1
  for (int sl = 0; sl < nslab; ++sl) {
    const int slab = mock * nslab + sl;
    int cy[H][P], cz[H][P];
    float wy[H][P], wz[H][P], dy[H][P], dz[H][P];
    // this lane's planes
    const float* plane[H][PPL];
    float wx[H][PPL], dx[H][PPL];
    bool wraps = false;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int mk = (IL == 2) ? grid_mask(g.code, 2 * sl + h) : (h ? 7 : 0);
      int c[P];
      float wt[P], d[P];
      const double ux = u[0] + ((mk & 1) ? 0.5 : 0.0);
      const double uy = u[1] + ((mk & 2) ? 0.5 : 0.0);
      const double uz = u[2] + ((mk & 4) ? 0.5 : 0.0);
      stencil_1d<P>(ux, n, c, wt);
      stencil_1d_deriv<P>(ux, d);
      stencil_1d<P>(uy, n, cy[h], wy[h]);
      stencil_1d_deriv<P>(uy, dy[h]);
      stencil_1d<P>(uz, n, cz[h], wz[h]);
      stencil_1d_deriv<P>(uz, dz[h]);
      wraps |= P > 1 && cz[h][0] > n - P;
#pragma unroll
      for (int i = 0; i < PPL; ++i) {
        int cx = c[i];
        wx[h][i] = wt[i];
        dx[h][i] = d[i];
#pragma unroll
        for (int k = 1; k < G; ++k) {
          cx = part == k ? c[k * PPL + i] : cx;
          wx[h][i] = part == k ? wt[k * PPL + i] : wx[h][i];
          dx[h][i] = part == k ? d[k * PPL + i] : dx[h][i];
        }
        // float offsets: a complex grid holds grid h as component h of each
        // complex element, a packed real grid two reals per element
        plane[h][i] = grid + 2 * (((int64_t)slab * n + cx) * g.ps);
      }
    }
    auto row = [&](int h, int i, int b, const float (&v)[S * P]) __attribute__((always_inline)) {
      float t = 0.0f, r = 0.0f;
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const float e = v[S * q + h];
        t = __builtin_fmaf(wz[h][q], e, t);
        r = __builtin_fmaf(dz[h][q], e, r);
      }
      gx = __builtin_fmaf(dx[h][i] * wy[h][b], t, gx);
      gy = __builtin_fmaf(wx[h][i] * dy[h][b], t, gy);
      gz = __builtin_fmaf(wx[h][i] * wy[h][b], r, gz);
    };
    if (!wraps) {
#pragma unroll
      for (int i = 0; i < PPL; ++i)
#pragma unroll
        for (int b = 0; b < P; ++b)
#pragma unroll
          for (int h = 0; h < H; ++h) {
            float v[S * P];
            load_row<S * P>(plane[h][i] + cy[h][b] * pitch + S * cz[h][0], v);
            row(h, i, b, v);
          }
    } else {  // a stencil passes the end of the axis
#pragma unroll
      for (int i = 0; i < PPL; ++i)
#pragma unroll
        for (int b = 0; b < P; ++b)
#pragma unroll
          for (int h = 0; h < H; ++h) {
            float v[S * P];
#pragma unroll
            for (int q = 0; q < P; ++q) v[S * q + h] = plane[h][i][cy[h][b] * pitch + S * cz[h][q] + h];
            row(h, i, b, v);
          }
    }
  }
#pragma unroll
  for (int m = W; m < 64; m *= 2) {
    gx += __shfl_xor(gx, m);
    gy += __shfl_xor(gy, m);
    gz += __shfl_xor(gz, m);
  }
  if (!valid || (G > 1 && part != 0)) return;
  // a particle of mass w_j deposits w_j times the kernel
  const double sc = -(double)n / g.box * (w ? (double)w[j] : 1.0);
  grad[3 * j + 0] = (TP)(sc * gx);
  grad[3 * j + 1] = (TP)(sc * gy);
  grad[3 * j + 2] = (TP)(sc * gz);
}

template <int P, int IL>
static void gather_t(const Geom& g, const void* pos, est_dtype dt, const int64_t* offsets,
                     int64_t n_total, const float* w, const Buffers& b, void* grad, hipStream_t s) {
  constexpr int per = 256 / gather_lanes<P>();  // particles per workgroup
  const unsigned blocks = (unsigned)((n_total + per - 1) / per);
  if (dt == EST_F32)
    hipLaunchKernelGGL((k_gather_grad<P, IL, float>), dim3(blocks), dim3(256), 0, s,
                       (const float*)pos, n_total, offsets, (const float*)b.grid, g, w, (float*)grad);
  else
    hipLaunchKernelGGL((k_gather_grad<P, IL, double>), dim3(blocks), dim3(256), 0, s,
                       (const double*)pos, n_total, offsets, (const float*)b.grid, g, w,
                       (double*)grad);
}

template <int P>
static void dispatch_gather(const Geom& g, const void* pos, est_dtype dt, const int64_t* offsets,
                            int64_t n_total, const float* w, const Buffers& b, void* grad,
                            hipStream_t s) {
  if (g.code >= 2) gather_t<P, 2>(g, pos, dt, offsets, n_total, w, b, grad, s);
  else if (g.code == 1) gather_t<P, 1>(g, pos, dt, offsets, n_total, w, b, grad, s);
  else gather_t<P, 0>(g, pos, dt, offsets, n_total, w, b, grad, s);
}

hipError_t launch_gather_grad(const Geom& g, const void* pos, est_dtype dt, const int64_t* offsets,
                              int64_t n_total, const float* w, const Buffers& b, void* grad,
                              hipStream_t s) {
  switch (g.order) {
    case 1: dispatch_gather<1>(g, pos, dt, offsets, n_total, w, b, grad, s); break;
    case 2: dispatch_gather<2>(g, pos, dt, offsets, n_total, w, b, grad, s); break;
    case 3: dispatch_gather<3>(g, pos, dt, offsets, n_total, w, b, grad, s); break;
    case 4: dispatch_gather<4>(g, pos, dt, offsets, n_total, w, b, grad, s); break;
    case 5: dispatch_gather<5>(g, pos, dt, offsets, n_total, w, b, grad, s); break;
    default: dispatch_gather<6>(g, pos, dt, offsets, n_total, w, b, grad, s); break;
  }
  return hipGetLastError();
}

}  // namespace fsest
