// Window sums of the forward transform (Algorithm 2.1 step 3) on the matrix
// cores: float32, d = 2, tile edge 16, m >= 5.
//
// f_n = sum_i a_n[i] sum_c b_n[c] G[i][c] over the padded tile of the node's
// tile (P = 16 + 2m rows and columns). Sixteen nodes at a time, the inner sum
// is a product of a block of 16 rows of G with the 16 columns b_n,
//     H[i][n] = sum_c G[i][c] b_n[c],
// whose inner dimension runs over the padded columns, four per
// v_mfma_f32_16x16x4f32 (P / 4 steps, real and imaginary part). The nodes of a
// tile are sorted by row at plan time, so sixteen consecutive nodes span few
// rows and one block of 16 rows usually covers all their windows (2m + rows
// spanned <= 16; two blocks otherwise). Lane (q, n) of the result holds rows
// 4q .. 4q + 3 for node n, multiplies them by its row factors, and the four
// lanes of a node are summed.
//
// The window factors are evaluated per call, lane (k, n) polynomials
// k, k + 4, ... at node n's two offsets, and go through rows of LDS that are
// zero outside the window: the factor of padded column c is read at
// c - l1 - 1 whatever the node's column, without a bounds test.
//
// Bound: the float32 matrix operations (2 P / 4 per 16 nodes) and the vector
// work take turns (no cycle with both busy, by the counters), and together
// they are about two thirds of the kernel. The lane-per-node form it replaced
// reads (2m)^2 cells per node from LDS and evaluates the window again for
// every right-hand side; here a work-group keeps NR tiles in LDS and one
// evaluation serves all of them. Spiral of 131072 nodes, M = 256, m = 6, 32
// right-hand sides: 217 -> 129 us; polar set of 262144 nodes, one, in the traces
// 15.6 -> 15.5 (forward) and 17.0 -> 16.6 (refinement).
#include "spread_common.hpp"

namespace nfft {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kInterpT = 16;
constexpr int kInterpWaves = 4;
// narrower windows leave too much of the 16 x P block unused: at m = 4 the
// lane-per-node kernel takes as long or less (polar set of 262144 nodes, M =
// 256, whole transform: 22.2 against 22.7 us; at m = 6 28.0 against 25.6, at
// m = 8 34.3 against 29.4; 8 right-hand sides of the spiral at m = 4: 57.1
// against 59.1)
constexpr int kInterpMinM = 5;

template <int MW, int NR>
struct InterpShape {
  static constexpr int P = kInterpT + 2 * MW;
  static constexpr int KS = (P + 3) / 4;  // steps of four columns
  // row stride of the tile in LDS: covers the steps, and 2 mod 4 complex
  // cells, so that 16 rows x 2 columns (half a wave's 8-byte reads) lie in
  // different banks
  static constexpr int PS = (4 * KS + 1) / 4 * 4 + 2;
  // factor rows: cell p of node n's window (-1: the closed edge) at
  // n * FS + FO + p, zeros between the windows of neighbouring rows. A row or
  // column of the tile is at most 16 cells before and 31 after a node's
  // first window cell: 34 leaves at least 16 zeros on either side of a window
  // of 2m + 1 <= 17, and equal cells of 16 nodes and two neighbouring cells
  // lie in 32 different banks
  static constexpr int FS = 34;
  static constexpr int FO = 16;
  static constexpr int FN = 16 * FS + 16;  // columns, one wave
  // rows: the same, or for four right-hand sides and m <= 6 only a zero on
  // either side of the window with the cell clamped, which lets four
  // work-groups instead of three into a compute unit's LDS (spiral of 131072
  // nodes, 32 right-hand sides, m = 6: whole transform 163.8 -> 157.9 us; for
  // one right-hand side the clamps cost 1 to 2 %)
  static constexpr bool compact = NR == 4 && MW <= 6;
  static constexpr int RS = compact ? 2 * MW + 3 : FS;
  static constexpr int RO = compact ? 2 : FO;
  static constexpr int RN = compact ? (16 * RS + 3) / 4 * 4 : FN;
  static constexpr size_t tile = (size_t)P * PS * sizeof(float2);
  static constexpr size_t factors = (size_t)kInterpWaves * (FN + RN) * sizeof(float);
};

}  // namespace

template <int MW, int NR>
__global__ __launch_bounds__(64 * kInterpWaves) void interp_mma_kernel(InterpArgs<float> a, int nrhs) {
  using S = InterpShape<MW, NR>;
  using R = float;
  typedef v4f v4;
  constexpr int K2 = 2 * MW;
  constexpr int P = S::P, PS = S::PS, KS = S::KS, FS = S::FS, FN = S::FN, RN = S::RN;
  constexpr int NP = (K2 + 3) / 4;  // polynomials per lane
  constexpr int DEG = PolyDeg<R>::value;
  constexpr int NT = 64 * kInterpWaves;
  static_assert(PS >= 4 * KS, "operand reads stay in the row");
  static_assert(NR == 1 || NR % 2 == 0, "right-hand sides are reduced in pairs");
  extern __shared__ double lds_d[];
  cplx<R>* tiles = reinterpret_cast<cplx<R>*>(lds_d);                 // [NR][P][PS]
  R* fac = reinterpret_cast<R*>(tiles + (size_t)NR * P * PS);         // [wave][FN + RN]

  const int item = blockIdx.x;
  const int rhs0 = blockIdx.y * NR;
  const int nr = nrhs - rhs0 < NR ? nrhs - rhs0 : NR;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int q = lane >> 4;  // column of a step (operands), row quarter (result)
  const int n = lane & 15;  // row (first operand), node
  const int Ms = a.g.Ms;
  const int64_t N = a.g.N;
  const int4 it = reinterpret_cast<const int4*>(a.items)[item];
  const int start = it.x, cnt = it.y, bin = it.z;
  if (cnt == 0) return;
  const int org0 = (bin / a.g.nb) * kInterpT - MW;
  const int org1 = (bin % a.g.nb) * kInterpT - MW;

  // node data of a group of 16: 32-bit offsets from the item's first node,
  // past the last node the last one again
  const int ng = (cnt + 15) >> 4;
  struct Node {
    uint32_t L;
    R x0, x1;
    int j;
  };
  auto load_node = [&](int g) {
    const uint32_t i = (uint32_t)(16 * g + n < cnt ? 16 * g + n : cnt - 1);
    Node v;
    v.L = at(a.loc + start, i);
    v.x0 = at(a.frac + start, i);
    v.x1 = at(a.frac + N + start, i);
    v.j = at(a.perm + start, i);
    return v;
  };
  int g = wave;
  Node nd = load_node(g);  // in flight during the tile load

  R cf[NP][DEG + 1];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int p = q + 4 * i < K2 ? q + 4 * i : K2 - 1;
#pragma unroll
    for (int t = 0; t <= DEG; ++t) cf[i][t] = a.coef[p * (DEG + 1) + t];
  }

  // the padded tiles; the tile edge divides M_sigma, so one wrap each way is
  // enough. Columns past P have zero factors, and the tiles past the last
  // right-hand side are not used: both hold other cells of the grid.
#pragma unroll (NR > 4 ? 1 : 4)
  for (int i = tid; i < P * PS; i += NT) {
    const int r = i / PS, c = i - r * PS;
    int s0 = org0 + r, s1 = org1 + c;
    s0 = s0 < 0 ? s0 + Ms : (s0 >= Ms ? s0 - Ms : s0);
    s1 = s1 < 0 ? s1 + Ms : (s1 >= Ms ? s1 - Ms : s1);
    const cplx<R>* src = a.grid + rhs0 * a.grid_rs + (int64_t)s0 * Ms + s1;
    cplx<R> v[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) v[t] = src[(NR > 1 ? min(t, nr - 1) : 0) * a.grid_rs];
#pragma unroll
    for (int t = 0; t < NR; ++t) tiles[t * (P * PS) + i] = v[t];
  }
  for (int i = tid; i < kInterpWaves * (FN + RN) / 4; i += NT)
    reinterpret_cast<v4*>(fac)[i] = v4{(R)0, (R)0, (R)0, (R)0};
  R* f1 = fac + wave * (FN + RN) + n * FS + S::FO;       // column factors of node n
  R* f0 = fac + wave * (FN + RN) + FN + n * S::RS + S::RO;  // row factors
  __syncthreads();

  const R edge = a.edge;
  // the coefficients have arrived: a wait for them inside the loop would wait
  // for the loads and stores of the groups, too
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int t = 0; t <= DEG; ++t) asm volatile("" : "+v"(cf[i][t]));
  asm volatile("" : "+v"(nd.L), "+v"(nd.x0), "+v"(nd.x1), "+v"(nd.j));
  for (; g < ng; g += kInterpWaves) {
    const bool valid = 16 * g + n < cnt;
    const int jn = nd.j;
    const uint32_t L = nd.L;
    const int l0 = (int)(L & kLocMask), l1 = (int)((L >> kLocBits) & kLocMask);
    const R y0 = (R)2 * nd.x0 - (R)1, y1 = (R)2 * nd.x1 - (R)1;
    // rows: from the first node's first row (its closed-edge row only if a
    // node of the group lies on a grid line) to the last node's last
    const int rmin = __builtin_amdgcn_readfirstlane(l0);
    const int rmax = __builtin_amdgcn_readlane(l0, 15);
    const int r0 = rmin + (__builtin_amdgcn_ballot_w64((L >> kEdgeShift) & 1u) ? 0 : 1);
    // the first right-hand side's operands; rows past the tile have zero
    // factors, so any row of the tile will do for them
    auto row_of = [&](int rb) { return tiles + min(rb + n, P - 1) * PS + q; };
    cplx<R> gv[2][KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) gv[0][s] = row_of(r0)[4 * s];
    // lane quarters 0 and 1 write the outputs of two right-hand sides
    const int64_t o = rhs0 * a.f_rs + (q & 1) * a.f_rs + jn;
    cplx<R> sub[NR > 1 ? NR / 2 : 1];
    if (a.sub) {
#pragma unroll
      for (int t = 0; t < NR; t += 2)
        if (valid && t + q < (NR > 1 ? nr : 1) && q < 2) sub[t / 2] = a.sub[o + t * a.f_rs];
    }
    nd = load_node(g + kInterpWaves);  // the next group's

    wave_lds_fence();  // the previous group's factors are read
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int p = q + 4 * i;
      const R h0 = horner<R>(cf[i], y0);
      const R h1 = horner<R>(cf[i], y1);
      if (4 * i + 3 < K2 || p < K2) {
        f0[p] = h0;
        f1[p] = h1;
      }
    }
    if (q < 2) (q ? f1 : f0)[-1] = (L >> (kEdgeShift + q)) & 1u ? edge : (R)0;
    wave_lds_fence();

    R b[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) b[s] = f1[4 * s + q - l1 - 1];
    R sx[NR], sy[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) sx[t] = sy[t] = (R)0;
    for (int rb = r0;;) {
      R ra[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int c = rb + 4 * q + v - l0 - 1;
        ra[v] = f0[S::compact ? min(max(c, -2), K2) : c];
      }
      const cplx<R>* tr = row_of(rb);
      // the operands of one right-hand side are read while the products of
      // the one before run
#pragma unroll
      for (int t = 0; t < NR; ++t) {
        if (NR == 1 || t < nr) {
          if (t + 1 < NR) {
#pragma unroll
            for (int s = 0; s < KS; ++s) gv[(t + 1) & 1][s] = tr[(t + 1) * (P * PS) + 4 * s];
          }
          v4 hr = {(R)0, (R)0, (R)0, (R)0}, hi = hr;
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            hr = __builtin_amdgcn_mfma_f32_16x16x4f32(gv[t & 1][s].x, b[s], hr, 0, 0, 0);
            hi = __builtin_amdgcn_mfma_f32_16x16x4f32(gv[t & 1][s].y, b[s], hi, 0, 0, 0);
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            sx[t] += hr[v] * ra[v];
            sy[t] += hi[v] * ra[v];
          }
        }
      }
      rb += 16;
      if (rb > rmax + K2) break;
#pragma unroll
      for (int s = 0; s < KS; ++s) gv[0][s] = row_of(rb)[4 * s];
    }
    // the next group's data have arrived: a wait for them after the stores
    // below would wait for the stores, too
    asm volatile("" : "+v"(nd.L), "+v"(nd.x0), "+v"(nd.x1), "+v"(nd.j));
    // sums over the four lanes of a node, two right-hand sides at a time:
    // lane quarters 0 .. 3 get Re t, Re t + 1, Im t, Im t + 1, and the lower
    // half of the wave both parts
#pragma unroll
    for (int t = 0; t < NR; t += 2) {
      const R v0 = sum32(sx[t], sy[t]);
      const R v1 = NR > 1 ? sum32(sx[t + (NR > 1)], sy[t + (NR > 1)]) : v0;
      const R re = sum16(v0, v1);
      const R im = upper(re);
      if (valid && q < 2 && t + q < (NR > 1 ? nr : 1)) {
        const cplx<R> v = a.sub ? mkc<R>(sub[t / 2].x - re, sub[t / 2].y - im) : mkc<R>(re, im);
        a.f[o + t * a.f_rs] = v;
      }
    }
  }
}

bool interp_mma_supported(int d, int T, bool f64, int m) {
  return d == 2 && T == kInterpT && !f64 && m >= kInterpMinM && m <= 8;
}

template <int MW, int NR>
static hipError_t interp_mma_nr(const InterpArgs<float>& a, int nrhs, hipStream_t s) {
  using S = InterpShape<MW, NR>;
  hipLaunchKernelGGL((interp_mma_kernel<MW, NR>), dim3(a.nitems, (nrhs + NR - 1) / NR),
                     dim3(64 * kInterpWaves), NR * S::tile + S::factors, s, a, nrhs);
  return hipGetLastError();
}

// Several right-hand sides share the window and the node data of a work-group
// where that leaves three work-groups per compute unit; with fewer, a work-group
// is one chain of its right-hand sides and one each is faster. Whole transforms
// (graph replays), lane-per-node kernel > one > two > four a work-group, in us:
// m = 8, 8192 uniform nodes, M = 32, 5 of them 15.8 > 14.1 > 16.7 > 21.2 (39 items);
// m = 6, 65536, M = 128, 8 of them 43.3 > 36.3 > 33.9 > 32.6 (377 items). Of 2988
// sets, m = 5 .. 8, 1 to 32 of them, 4 are slower than with the lane-per-node
// kernel by more than 2 %, with 512 instead of 768 13, with 1024 8. By eight instead of
// four, 32 of them on the spiral of 131072 nodes, M = 256, m = 6, took 133 against
// 134 us. At m = 5 one a work-group is as fast as the lane-per-node kernel, or up
// to 8 % slower, on less than 3000 items of 64 nodes or more (131072 spiral
// nodes, M = 128, 15.3 > 16.6), else up to 1.2 times as fast.
int interp_mma_rhs(int m, int64_t N, int nitems, int nrhs) {
  for (int nr = 4; nr > 1; nr /= 2)
    if (2 * nrhs > nr && (int64_t)nitems * ((nrhs + nr - 1) / nr) >= 768) return nr;
  return m == kInterpMinM && nitems < 3000 && N >= 64 * (int64_t)nitems ? 0 : 1;
}

template <int MW>
static hipError_t interp_mma_m(const InterpArgs<float>& a, int nrhs, hipStream_t s) {
  switch (interp_mma_rhs(MW, a.g.N, a.nitems, nrhs)) {
    case 4: return interp_mma_nr<MW, 4>(a, nrhs, s);
    case 2: return interp_mma_nr<MW, 2>(a, nrhs, s);
    default: return interp_mma_nr<MW, 1>(a, nrhs, s);
  }
}

hipError_t launch_interp_mma(const InterpArgs<float>& a, int nrhs, hipStream_t s) {
  if (!interp_mma_supported(a.g.d, a.g.T, false, a.g.m) || !a.items) return hipErrorInvalidValue;
  if (a.nitems == 0) return hipSuccess;
  switch (a.g.m) {
    case 5: return interp_mma_m<5>(a, nrhs, s);
    case 6: return interp_mma_m<6>(a, nrhs, s);
    case 7: return interp_mma_m<7>(a, nrhs, s);
    case 8: return interp_mma_m<8>(a, nrhs, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nfft
