// Spreading for d = 3 on the matrix cores, float32 and float64 (Algorithm
// 2.4 step 1 with the weights of (3.7)), tile edge 8 and 2m <= 8, so that
// plane i0 of the padded tile of a work item (P = 8 + 2m <= 16 cells per
// dimension) is one 16 x 16 block (rows i1, columns i2) of
// v_mfma_f32_16x16x4f32 (float64: v_mfma_f64_16x16x4f64) accumulators, real and
// imaginary part.
//
// A node at tile-local cell (l0, l1, l2) reaches the padded cells
// (l0 + 1 + p0, l1 + 1 + p1, l2 + 1 + p2), p_t < 2m, with the window factors
// a(p0) b(p1) e(p2), and on a grid plane of dimension t also the closed-edge
// cell l_t of that dimension. For one plane the update is
//     G[i0][i1][i2] += sum_n (b_n[i1] c_n) (a_n[i0] e_n[i2]),   c_n = w_n f_n,
// a product whose inner dimension runs over the nodes, four at a time.
//
// Four waves share the nodes of an item, 64 at a time: each evaluates the
// window of 16 of them and writes the factors to LDS, a row of 16 padded cells
// per node and dimension, zero where the window does not reach; then wave w
// takes all groups of four through the planes i0 = w mod 4 (two of the 2m that
// a node reaches, at m = 4). The rows being zero outside the windows, a group
// may hold any nodes; they are sorted by l0 at plan time, so that a group
// reaches few planes more than 2m. No cell is summed by two waves and the order
// of every sum is fixed. The padded tile is written out like the other
// kernels' (the split-tile sums and the first FFT pass merge the tiles).
//
// Bound: matrix and vector work, which take turns: 16 matrix operations per
// group of four nodes (m = 4; a quarter of their products is inside the
// windows) and about 65 vector instructions, half of them the staging. A form
// with one wave per item, which formed its operands per group and held all
// planes, took 68.5 us on the jittered set of 524288 nodes at M = 64, m = 4
// (62.7 here), in float64 151 (113 here). Reading the next group's operands a
// group ahead costs more in moves than it hides (108 against 100 us for the
// transform of as many uniform nodes); two groups a step against one 99.7 and
// 100.1, against four 98.4.
#include "spread_common.hpp"

namespace nfft {

namespace {

template <typename R> struct Mma3T;
template <> struct Mma3T<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mfma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // row of element v of lane quarter q
  static __device__ __forceinline__ int row(int q, int v) { return 4 * q + v; }
};
template <> struct Mma3T<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mfma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int q, int v) { return 4 * v + q; }
};

constexpr int k3MmaT = 8;
constexpr int k3Chunk = 64;           // nodes staged at a time
constexpr int k3Rows = k3Chunk + 4;   // the last group may look past the last node
constexpr int k3RowFS = 48;           // a (16), b (16), e (16)

}  // namespace

template <typename R, int MW>
__global__ __launch_bounds__(256) void spread3_mma_kernel(SpreadArgs<R> a) {
  using M3 = Mma3T<R>;
  typedef typename M3::v4 v4;
  constexpr int K2 = 2 * MW;
  constexpr int P = k3MmaT + K2;
  constexpr int NK = (P + 3) / 4;  // planes of a wave: w + 4 k
  constexpr int DEG = PolyDeg<R>::value;
  constexpr int FS = k3RowFS, NN = k3Chunk;
  constexpr int UG = 2;  // groups per step
  static_assert(P <= 16, "a plane of the padded tile is one 16 x 16 block");
  __shared__ R tab[k3Rows * FS];
  __shared__ cplx<R> ct[k3Rows];

  const int item = blockIdx.x;
  const int rhs = blockIdx.y;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int kq = lane >> 4;  // node of a group; accumulator row quarter
  const int j = lane & 15;   // pair and dimension (staging); row i1 (A), column i2 (B)
  const int64_t N = a.g.N;
  const int start = a.item_start[item];
  const int cnt = a.item_count[item];
  const R edge = a.edge;
  const cplx<R>* f = a.f + rhs * a.f_rs;

  // Staging. The window is even: the polynomial of cell 2m - 1 - p is that of
  // cell p at -y. Of a node's 16 lanes, lane 4 t + p evaluates the sums of the
  // odd terms and of the even terms from y^2 on of polynomial p < m at the
  // node's offset in dimension t < 3, from them both cells, and writes two of
  // the zeros around the window; lanes with p >= m write four zeros. The last
  // two steps are Horner's, so that c_0, the largest term, enters in one
  // rounding: float32 error of whole transforms over that of one plain Horner
  // chain a cell 0.99 to 1.01, with c_0 inside the even terms' chain 1.00 to
  // 1.06 (m = 3 most). Cell c of the window is padded cell l + 1 + c; cells
  // 2m .. 15 go round to the padded cells outside it, cell 15 being the closed
  // edge l.
  const int dim = j >> 2 < 3 ? j >> 2 : 2, jj = j & 3;
  const bool stages = j < 12;
  const int c1 = jj < MW ? jj : 4 * MW + 4 * (jj - MW);
  const int c2 = jj < MW ? K2 - 1 - jj : c1 + 1;
  const int c3 = jj < MW ? K2 + 2 * jj : c1 + 2;
  const int c4 = c3 + 1;
  const uint32_t em = jj == 3 ? 1u << (kEdgeShift + dim) : 0u;  // its c4 is cell 15
  const R* pcf = a.coef + (jj < MW ? jj : 0) * (DEG + 1);
  R ce[DEG / 2 + 1], co[DEG / 2];
#pragma unroll
  for (int t = 0; t <= DEG / 2; ++t) ce[t] = pcf[2 * t];
#pragma unroll
  for (int t = 0; t < DEG / 2; ++t) co[t] = pcf[2 * t + 1];
#pragma unroll
  for (int t = 0; t <= DEG / 2; ++t) ce[t] = jj < MW ? ce[t] : (R)0;
#pragma unroll
  for (int t = 0; t < DEG / 2; ++t) co[t] = jj < MW ? co[t] : (R)0;

  // node data of a chunk, in registers one chunk ahead: cell word and one
  // offset of the four nodes whose factors this lane evaluates, the cell word
  // of node `lane`, and (wave 0) weight, sample and index of node `lane`. Nodes
  // past the item's last are its neighbours' or the arrays' padding: their c is
  // taken as zero.
  uint32_t Ln[4], Lb;
  R xn[4];
  cplx<R> wv = mkc<R>(0, 0), fv = wv;
  int jn = 0;
  const uint32_t* loc = a.loc + start;
  const R* fr = a.frac + start + dim * N + kq;
  auto load_chunk = [&](int b0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      Ln[t] = (loc + b0 + 16 * wave + 4 * t)[kq];
      xn[t] = (fr + b0 + 16 * wave + 4 * t)[0];
    }
    Lb = (loc + b0)[lane];
    if (wave == 0) {
      wv = (a.w + start + b0)[lane];
      fv = f[jn];
      jn = (a.perm + start + b0 + NN)[lane];
    }
  };
  if (wave == 0) jn = (a.perm + start)[lane];
  load_chunk(0);

  // the rows past a chunk are read by its last group: any finite value will do
  for (int i = tid; i < (k3Rows - NN) * FS; i += 256) tab[NN * FS + i] = (R)0;

  v4 acc[NK][2];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    acc[k][0] = v4{(R)0, (R)0, (R)0, (R)0};
    acc[k][1] = acc[k][0];
  }
  const R* opb = tab + kq * FS + 16 + j;  // b row; e row 16 further; a row's plane 4 k: below
  const R* opa = tab + kq * FS + wave;
  const cplx<R>* opc = ct + kq;

  for (int b0 = 0; b0 < cnt; b0 += NN) {
    const int nb = cnt - b0 < NN ? cnt - b0 : NN;
    if (b0) __syncthreads();  // the previous chunk is consumed
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t L = Ln[t];
      const R y = (R)2 * xn[t] - (R)1;
      const R y2 = y * y;
      R ev = ce[DEG / 2], od = co[DEG / 2 - 1];
#pragma unroll
      for (int q = DEG / 2 - 1; q >= 1; --q) ev = ev * y2 + ce[q];
#pragma unroll
      for (int q = DEG / 2 - 2; q >= 0; --q) od = od * y2 + co[q];
      const R v1 = ce[0] + y * (od + y * ev), v2 = ce[0] - y * (od - y * ev);
      const int l1 = (int)((L >> (kLocBits * dim)) & kLocMask) + 1;
      R* row = tab + (16 * wave + 4 * t + kq) * FS + 16 * dim;
      if (stages) {
        row[(l1 + c1) & 15] = v1;
        row[(l1 + c2) & 15] = v2;
        row[(l1 + c3) & 15] = (R)0;
        row[(l1 + c4) & 15] = L & em ? edge : (R)0;
      }
    }
    if (wave == 0)
      ct[lane] = mkc<R>(wv.x * fv.x - wv.y * fv.y, wv.x * fv.y + wv.y * fv.x);
    // planes of lane's group of four that this wave owns, as bits k: from the
    // group's first plane (a closed edge's if it has one; the nodes are sorted
    // by l0, but one on a grid plane may begin before its predecessors) to its
    // last node's last
    int mask;
    {
      const int l0 = (int)(Lb & kLocMask);
      int first = lane < nb ? l0 + ((Lb >> kEdgeShift) & 1u ? 0 : 1) : P;
      int last = lane < nb ? l0 + K2 : -1;
      first = min(first, __shfl_xor(first, 1));
      first = min(first, __shfl_xor(first, 2));
      last = max(last, __shfl_xor(last, 1));
      last = max(last, __shfl_xor(last, 2));
      const int k0 = (max(first - wave, 0) + 3) >> 2;
      const int k1 = (last - wave) >> 2;  // -1 before this wave's first plane
      mask = ((1 << (k1 + 1)) - 1) & ~((1 << k0) - 1);
    }
    __syncthreads();
    if (b0 + NN < cnt) load_chunk(b0 + NN);

    const R* pb = opb;
    const R* pa = opa;
    const cplx<R>* pc = opc;
    auto group = [&](int n, int u, bool part) {
      const R b = pb[4 * u * FS], e = pb[4 * u * FS + 16];
      cplx<R> c = pc[4 * u];
      R an[NK];
#pragma unroll
      for (int k = 0; k < NK; ++k) an[k] = pa[4 * u * FS + 4 * k];
      if (part) c = kq < nb - n ? c : mkc<R>(0, 0);
      const R br = b * c.x, bi = b * c.y;
      const int m = __builtin_amdgcn_readlane(mask, n);
#pragma unroll
      for (int k = 0; k < NK; ++k)
        if (m >> k & 1) {
          const R ae = an[k] * e;
          acc[k][0] = M3::mfma(br, ae, acc[k][0]);
          acc[k][1] = M3::mfma(bi, ae, acc[k][1]);
        }
    };
    int n = 0;
    for (; n + UG * 4 <= nb; n += UG * 4, pb += UG * 4 * FS, pa += UG * 4 * FS, pc += UG * 4)
#pragma unroll
      for (int u = 0; u < UG; ++u) group(n + 4 * u, u, false);
    for (; n < nb; n += 4, pb += 4 * FS, pa += 4 * FS, pc += 4) group(n, 0, n + 4 > nb);
  }

  // element v of lane l: row i1, column i2 = l & 15
  const int slot = a.item_slot[item];
  constexpr int Ptot = P * P * P;
  cplx<R>* out = slot < 0 ? a.tilep + rhs * a.tile_rs + (int64_t)a.item_bin[item] * Ptot
                          : a.itemp + rhs * a.item_rs + (int64_t)slot * Ptot;
#pragma unroll
  for (int k = 0; k < NK; ++k)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i0 = wave + 4 * k, i1 = M3::row(kq, v);
      if (i0 < P && i1 < P && j < P)
        out[(i0 * P + i1) * P + j] = mkc<R>(acc[k][0][v], acc[k][1][v]);
    }
}

bool spread3_mma_supported(int d, int T, bool f64, int m) {
  (void)f64;  // float32 and float64
  return d == 3 && T == k3MmaT && m >= 1 && k3MmaT + 2 * m <= 16;
}

// The default spread mode takes this kernel for m >= 2 (whole transforms of
// uniform nodes at M = 64, 0.1 to 400 a tile, LDS accumulation > this kernel, in
// us; 409, 8192, 131072 and 1638400 nodes: float32, m = 2 35.4 > 34.6, 44.8 >
// 45.3, 58.6 > 51.2, 273 > 172; m = 3 39.7 > 38.6, 54.9 > 49.8, 75.8 > 57.7, 428 >
// 244; m = 4 48.2 > 45.5, 73.6 > 59.6, 99.5 > 69.3, 592 > 297; float64, m = 2
// 57.9 > 57.2, 77.8 > 74.0, 87.7 > 84.2, 408 > 326; m = 3 69.4 > 67.6, 98.4 >
// 87.0, 122 > 101, 706 > 460; smaller grids alike). The one exception: at m = 2 in
// float32 a device full of items of a few nodes each, where its fixed share of
// an item shows (three right-hand sides, 8192 nodes 90.3 > 93.7, 32768, eight a
// tile, 99.3 > 102.0; one, 131072, 32 a tile, 58.6 > 51.2). At m = 1 a node
// updates 8 cells and either may be the faster one.
bool spread3_mma_preferred(int d, int T, bool f64, int m, int64_t N, int nrhs,
                           const ItemShape& items) {
  if (m == 2 && !f64 && (int64_t)items.n * nrhs >= 2048 && N < 16 * (int64_t)items.n)
    return false;
  return m >= 2 && spread3_mma_supported(d, T, f64, m);
}

// the kernel's staging arrays (static LDS)
size_t spread3_mma_lds_bytes(bool f64) {
  return (size_t)k3Rows * (k3RowFS + 2) * (f64 ? sizeof(double) : sizeof(float));
}

template <typename R>
hipError_t launch_spread3_mma(const SpreadArgs<R>& a, int nrhs, hipStream_t s) {
  if (!spread3_mma_supported(a.g.d, a.g.T, !std::is_same<R, float>::value, a.g.m))
    return hipErrorInvalidValue;
  if (a.g.nsub == 0) return hipSuccess;
  const dim3 grid(a.g.nsub, nrhs);
  switch (a.g.m) {
    case 1: hipLaunchKernelGGL((spread3_mma_kernel<R, 1>), grid, dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL((spread3_mma_kernel<R, 2>), grid, dim3(256), 0, s, a); break;
    case 3: hipLaunchKernelGGL((spread3_mma_kernel<R, 3>), grid, dim3(256), 0, s, a); break;
    case 4: hipLaunchKernelGGL((spread3_mma_kernel<R, 4>), grid, dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template hipError_t launch_spread3_mma<float>(const SpreadArgs<float>&, int, hipStream_t);
template hipError_t launch_spread3_mma<double>(const SpreadArgs<double>&, int, hipStream_t);

}  // namespace nfft
