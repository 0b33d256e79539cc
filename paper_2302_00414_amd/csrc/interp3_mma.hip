// Window sums of the forward transform (Algorithm 2.1 step 3) on the matrix
// cores: float32, d = 3, tile edge 8, m = 4.
//
// f_n = sum_i a_n[i] sum_r b_n[r] sum_c e_n[c] G[i][r][c] over the padded tile
// of the node's tile (P = 8 + 2m <= 16 cells per dimension). Sixteen nodes at a
// time, the innermost sum over one plane i is a product of the plane's rows
// with the 16 columns e_n,
//     H[r][n] = sum_c G[i][r][c] e_n[c],
// P / 4 steps of v_mfma_f32_16x16x4f32 for the real and the imaginary part.
// Lane (q, n) of the result holds rows 4q .. 4q + 3 for node n, multiplies them
// by its row factors b_n and the sum by a_n[i]; the four lanes of a node are
// summed at the end. The nodes of a tile are sorted by their dimension-0 cell
// at plan time, so sixteen of them need few planes more than 2m.
//
// The window factors are evaluated per call, lane (k, n) polynomials k, k + 4
// at node n's three offsets, and go through rows of LDS that are zero outside
// the window (as in the d = 2 kernel).
//
// Bound: matrix and vector work, which take turns: about 9 planes x (8 matrix
// operations of 32 cycles and 12 vector instructions) per 16 nodes. The
// lane-per-node kernel reads (2m)^3 cells a node from LDS, at 2 to 3 times the
// conflict-free time as the nodes of a wave lie anywhere in the tile: jittered
// set of 524288 nodes, M = 64, 134 -> 60 us (the matrix operations alone 32 us).
// At m = 3 the two take turns (whole transform of 524288 uniform nodes 82 us
// lane per node, 88 here; of 20000 at M = 32, 28 and 25), at m = 2 the cells
// are few: m = 4 only (166 -> 100 us, 33.5 -> 25.7).
#include "spread_common.hpp"

namespace nfft {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int k3T = 8;
constexpr int k3Waves = 4;
// factor rows: cell p of node n's window (-1: the closed edge) at n * k3FS +
// k3FO + p. A plane, row or column is at most 8 cells before and 14 after a
// node's first window cell; 18: the window cells of the next row start past
// that, and equal cells of 16 nodes and two neighbouring cells lie in 32
// different banks.
constexpr int k3FS = 18;
constexpr int k3FO = 8;
constexpr int k3FN = 16 * k3FS + 16;

template <int MW>
struct Interp3Shape {
  static constexpr int P = k3T + 2 * MW;
  static constexpr int KS = (P + 3) / 4;
  // row stride: 2 mod 4 complex cells (16 rows x 2 columns in different banks)
  static constexpr int PS = 4 * KS + 2;
  static constexpr size_t bytes =
      (size_t)P * P * PS * sizeof(float2) + (size_t)k3Waves * 3 * k3FN * sizeof(float);
};

}  // namespace

template <int MW>
__global__ __launch_bounds__(64 * k3Waves) void interp3_mma_kernel(InterpArgs<float> a) {
  using S = Interp3Shape<MW>;
  constexpr int K2 = 2 * MW;
  constexpr int P = S::P, KS = S::KS, PS = S::PS;
  constexpr int NP = (K2 + 3) / 4;  // polynomials per lane
  constexpr int DEG = PolyDeg<float>::value;
  constexpr int NT = 64 * k3Waves;
  static_assert(P <= 16 && K2 >= 4, "a plane is one block of 16 rows");
  extern __shared__ double lds_d[];
  float2* tile = reinterpret_cast<float2*>(lds_d);           // [P][P][PS]
  float* fac = reinterpret_cast<float*>(tile + P * P * PS);  // [wave][3][k3FN]

  const int4 it = reinterpret_cast<const int4*>(a.items)[blockIdx.x];
  const int start = it.x, cnt = it.y;
  if (cnt == 0) return;
  const int rhs = blockIdx.y;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int q = lane >> 4;  // column of a step (operands), row quarter (result)
  const int n = lane & 15;  // row (first operand), node
  const int Ms = a.g.Ms, nb = a.g.nb;
  const int64_t N = a.g.N;
  const int org2 = (it.z % nb) * k3T - MW;
  const int org1 = (it.z / nb % nb) * k3T - MW;
  const int org0 = (it.z / (nb * nb)) * k3T - MW;

  const int ng = (cnt + 15) >> 4;
  struct Node {
    uint32_t L;
    float x[3];
    int j;
  };
  auto load_node = [&](int g) {
    const uint32_t i = (uint32_t)(16 * g + n < cnt ? 16 * g + n : cnt - 1);
    Node v;
    v.L = at(a.loc + start, i);
#pragma unroll
    for (int t = 0; t < 3; ++t) v.x[t] = at(a.frac + t * N + start, i);
    v.j = at(a.perm + start, i);
    return v;
  };
  int g = wave;
  Node nd = load_node(g);  // in flight during the tile load

  float cf[NP][DEG + 1];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int p = q + 4 * i < K2 ? q + 4 * i : K2 - 1;
#pragma unroll
    for (int t = 0; t <= DEG; ++t) cf[i][t] = a.coef[p * (DEG + 1) + t];
  }

  // the padded tile plane by plane, thread (r, c) its row r, column c; the tile
  // edge divides M_sigma, so one wrap each way is enough. Columns past P have
  // zero factors and hold other cells.
  {
    auto wrap = [&](int s) { return s < 0 ? s + Ms : (s >= Ms ? s - Ms : s); };
    const int r = tid >> 4, c = tid & 15;
    const float2* src = a.grid + rhs * a.grid_rs + (int64_t)wrap(org1 + r) * Ms + wrap(org2 + c);
    float2* dst = tile + r * PS + c;
    const int64_t plane = (int64_t)Ms * Ms;
    float2 v[P];
#pragma unroll
    for (int pl = 0; pl < P; ++pl) v[pl] = src[wrap(org0 + pl) * plane];
    if (P == 16 || r < P)
#pragma unroll
      for (int pl = 0; pl < P; ++pl) dst[pl * (P * PS)] = v[pl];
  }
  for (int i = tid; i < k3Waves * 3 * k3FN / 4; i += NT)
    reinterpret_cast<v4f*>(fac)[i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  float* f0 = fac + (wave * 3) * k3FN + n * k3FS + k3FO;
  float* f1 = f0 + k3FN;
  float* f2 = f1 + k3FN;
  __syncthreads();

  const float edge = a.edge;
  // the coefficients and the first nodes have arrived: a wait for them inside
  // the loop would wait for the loads and stores of the groups, too
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int t = 0; t <= DEG; ++t) asm volatile("" : "+v"(cf[i][t]));
  asm volatile("" : "+v"(nd.L), "+v"(nd.x[0]), "+v"(nd.x[1]), "+v"(nd.x[2]), "+v"(nd.j));
  const float2* rowp = tile + (n < P ? n : P - 1) * PS + q;
  for (; g < ng; g += k3Waves) {
    const bool valid = 16 * g + n < cnt;
    const int64_t o = rhs * a.f_rs + nd.j;
    const uint32_t L = nd.L;
    const int l0 = (int)(L & kLocMask), l1 = (int)((L >> kLocBits) & kLocMask);
    const int l2 = (int)((L >> (2 * kLocBits)) & kLocMask);
    const float y0 = 2.0f * nd.x[0] - 1.0f, y1 = 2.0f * nd.x[1] - 1.0f, y2 = 2.0f * nd.x[2] - 1.0f;
    // planes: from the first node's first (its closed-edge plane only if a
    // node of the group lies on a grid plane) to the last node's last
    const int p0 = __builtin_amdgcn_readfirstlane(l0) +
                   (__builtin_amdgcn_ballot_w64((L >> kEdgeShift) & 1u) ? 0 : 1);
    const int p1 = __builtin_amdgcn_readlane(l0, 15) + K2;
    float2 gv[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) gv[s] = rowp[p0 * (P * PS) + 4 * s];
    float2 sub = make_float2(0.0f, 0.0f);
    if (a.sub && valid && q == 0) sub = a.sub[o];
    nd = load_node(g + k3Waves);  // the next group's

    wave_lds_fence();  // the previous group's factors are read
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int p = q + 4 * i;
      const float h0 = horner<float>(cf[i], y0);
      const float h1 = horner<float>(cf[i], y1);
      const float h2 = horner<float>(cf[i], y2);
      if (4 * i + 3 < K2 || p < K2) {
        f0[p] = h0;
        f1[p] = h1;
        f2[p] = h2;
      }
    }
    if (q < 3) f0[q * k3FN - 1] = (L >> (kEdgeShift + q)) & 1u ? edge : 0.0f;
    wave_lds_fence();

    float b[KS], rb[4];
#pragma unroll
    for (int s = 0; s < KS; ++s) b[s] = f2[4 * s + q - l2 - 1];
#pragma unroll
    for (int v = 0; v < 4; ++v) rb[v] = f1[4 * q + v - l1 - 1];
    float sx = 0.0f, sy = 0.0f;
    const float* fa = f0 - l0 - 1;
#pragma unroll 2
    for (int p = p0; p <= p1; ++p) {
      float2 gc[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) gc[s] = gv[s];
      const float ra = fa[p];
      // the next plane's operands (past the last: the last again)
      const float2* nx = rowp + (p < p1 ? p + 1 : p1) * (P * PS);
#pragma unroll
      for (int s = 0; s < KS; ++s) gv[s] = nx[4 * s];
      v4f hr = {0.0f, 0.0f, 0.0f, 0.0f}, hi = hr;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        hr = __builtin_amdgcn_mfma_f32_16x16x4f32(gc[s].x, b[s], hr, 0, 0, 0);
        hi = __builtin_amdgcn_mfma_f32_16x16x4f32(gc[s].y, b[s], hi, 0, 0, 0);
      }
      float tx = hr[0] * rb[0], ty = hi[0] * rb[0];
#pragma unroll
      for (int v = 1; v < 4; ++v) {
        tx += hr[v] * rb[v];
        ty += hi[v] * rb[v];
      }
      sx += tx * ra;
      sy += ty * ra;
    }
    // the next group's data have arrived: a wait for them after the store
    // below would wait for the store, too
    asm volatile("" : "+v"(nd.L), "+v"(nd.x[0]), "+v"(nd.x[1]), "+v"(nd.x[2]), "+v"(nd.j));
    const float v = sum32(sx, sy);  // lower half of the wave Re, upper half Im
    const float re = sum16(v, v);
    const float im = upper(re);
    if (valid && q == 0)
      a.f[o] = a.sub ? make_float2(sub.x - re, sub.y - im) : make_float2(re, im);
  }
}

bool interp3_mma_supported(int d, int T, bool f64, int m) {
  return d == 3 && T == k3T && !f64 && m == 4;
}

hipError_t launch_interp3_mma(const InterpArgs<float>& a, int nrhs, hipStream_t s) {
  if (!interp3_mma_supported(a.g.d, a.g.T, false, a.g.m) || !a.items) return hipErrorInvalidValue;
  if (a.nitems == 0) return hipSuccess;
  hipLaunchKernelGGL((interp3_mma_kernel<4>), dim3(a.nitems, nrhs), dim3(64 * k3Waves),
                     Interp3Shape<4>::bytes, s, a);
  return hipGetLastError();
}

}  // namespace nfft
