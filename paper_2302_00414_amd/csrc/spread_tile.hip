// Spreading for d = 2, tile edge 16, on the matrix cores (float32 and
// float64, m <= 8; Algorithm 2.4 step 1 with the weights of (3.7)).
//
// A node at tile-local cell (l0, l1) reaches the padded rows l0 .. l0 + 2m of
// its tile's padded tile (P = 16 + 2m rows and columns): row l0 only if it
// lies on a grid line (closed edge), rows l0 + 1 .. l0 + 2m with the window
// factors a_0 .. a_{2m-1}; the same holds for the columns with b_0 ... The
// nodes of a work item come sorted by row. RB consecutive tile rows (a band,
// RB + 2m <= 16) reach 16 padded rows, so any four nodes of a band update
//     G[i][c] += sum_n A_n[i] B_n[c] c_n,   c_n = w_n f_n,
// a product whose inner dimension runs over the nodes: v_mfma_*_16x16x4 with
// A_n[i] c_n and B_n[c] as operands. The 16 accumulator rows are slots, slot
// s holding the padded row congruent to s modulo 16: after the last node of a
// band its RB rows are complete, go to the tile in LDS and make room for the
// rows 16 further down.
//
// Four waves share the nodes of an item, 64 at a time (NS = 4: sixteen waves,
// 256 at a time, of which four go on to the sums): each evaluates the window
// of 16 of them (lane (k, p) polynomial p at node k's two offsets) and
// writes the factors to LDS in operand order: entry i of a node's A row is
// the factor of slot i, entries of its two B rows those of padded columns i
// and 16 + i, zero where the window does not reach. Then every wave owns one
// column block and one part (real or imaginary) of the sums and takes all
// groups of four through it: two operand reads, one product with c_n and one
// matrix operation per group and right-hand side, without selects or lane
// exchanges, all reads free of bank conflicts. No cell is summed by two
// waves, so there is nothing to merge and the order of every sum is fixed; in
// float32 the runs of a chunk are added in float64. Several right-hand sides
// of a call (NR) share the factors.
//
// For m = 8 the 16 window rows fill the slots: a band is one row, whose slot
// is taken out before the row's nodes (its next user is 16 rows down), and
// the closed-edge row is summed by vector operations beside it.
//
// Bound: matrix and vector work, which take turns (no cycle with both busy by
// the counters): per group of four nodes 4 matrix operations (64 cycles each in
// float64, 32 in float32) and 60 to 100 vector instructions, half of them the
// staging. Linogram below at m = 8: 58 and 87 of 214 us, polar set at m = 6 in
// float64 7.0 and 7.7 of 27, the rest waits of short chains. Against mode 7's other shape
// (every wave its own padded tile of a quarter of the groups, summed in LDS
// at the end), polar set of 262144 nodes, M = 256, float64, whole transforms:
// m = 3 43.7 -> 34.3 us, m = 6 50.5 -> 40.0, m = 7 67.7 -> 49.3; float32,
// m = 6 30.7 -> 32.6, m = 7 36.3 -> 33.5; 1000003 uniform nodes, M = 512,
// m = 6: float64 141 -> 108 us, float32 76.6 -> 69.6. Against the LDS
// accumulation (mode 1): linogram of 2097152 nodes, M = 512, m = 8, float64
// 541 -> 247 us; 40321 nodes, M = 128, m = 6, 11 right-hand sides, float32
// 71 -> 43 us. Summing the split tiles here (the last work-group of a tile to
// arrive) instead of in a kernel of its own took 36.5 against 32.6 us.
#include "spread_common.hpp"

namespace nfft {

namespace {

template <typename R> struct TileMma;
template <> struct TileMma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mfma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // slot of operand row i: lane quarter q holds slots 4q .. 4q + 3 of the
  // result in both types
  static __device__ __forceinline__ int slot(int i) { return i; }
};
template <> struct TileMma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mfma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int slot(int i) { return ((i & 3) << 2) | (i >> 2); }
};

constexpr int kTileT = 16;
constexpr int kTileChunk = 64;             // nodes of a sub-chunk: 16 per staging wave
// factor rows beyond a chunk: its last group may look past its nodes. With
// eight of them a float64 work-group at m = 6 does not fit four times into a
// compute unit's LDS (polar set of 262144 nodes: 33.8 against 27.5 us).
constexpr int kTilePast = 4;
constexpr int kTileFS = 48;                // A (16), B of columns 0..15, B of columns 16..31

template <typename R, int MW, int NR, int NS>
struct TileLds {
  static constexpr int P = kTileT + 2 * MW;
  static constexpr int rows = NS * kTileChunk + kTilePast;
  static constexpr size_t tab = (size_t)rows * kTileFS * sizeof(R);
  static constexpr size_t c = (size_t)2 * NR * rows * sizeof(R);
  static constexpr size_t edge = MW == 8 ? rows * sizeof(R) : 0;
  static constexpr size_t tiles = (size_t)NR * P * P * sizeof(cplx<R>);
  static constexpr size_t bytes = tiles + tab + c + edge;
};

}  // namespace

template <typename R, int MW, int NR, int NS>
__global__ __launch_bounds__(256 * NS) void spread_tile_kernel(SpreadArgs<R> a, int nrhs) {
  using M4 = TileMma<R>;
  typedef typename M4::v4 v4;
  constexpr int K2 = 2 * MW;
  constexpr int P = kTileT + K2;
  constexpr int DEG = PolyDeg<R>::value;
  constexpr int FS = kTileFS, NN = NS * kTileChunk, NRow = TileLds<R, MW, NR, NS>::rows;
  constexpr int NT = 256 * NS;
  constexpr int RB = MW <= 4 ? 8 : MW <= 6 ? 4 : MW == 7 ? 2 : 1;  // rows of a band
  constexpr int NBAND = kTileT / RB;
  constexpr bool F32 = std::is_same<R, float>::value;
  constexpr int NA = F32 ? 4 : 1;
  constexpr int RUN = 4 * NA;  // groups of a run
  constexpr bool FULL = K2 == 16;  // the window rows fill the slots
  static_assert(FULL || RB + K2 <= 16, "the rows of a band's nodes fit in 16 slots");
  static_assert(NR <= 2, "wave r loads right-hand side r");
  extern __shared__ double lds_d[];
  cplx<R>* tiles = reinterpret_cast<cplx<R>*>(lds_d);        // [NR][P][P]
  R* tab = reinterpret_cast<R*>(tiles + NR * P * P);         // [NRow][FS]
  R* ct = tab + NRow * FS;                              // [part][NR][NRow]
  R* et = ct + 2 * NR * NRow;                           // [NRow] closed-edge factor (m = 8)

  const int item = blockIdx.x;
  const int rhs0 = blockIdx.y * NR;
  const int nr = nrhs - rhs0 < NR ? nrhs - rhs0 : NR;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int kq = lane >> 4;  // node of a group; slots 4 kq .. 4 kq + 3 of the result
  const int j = lane & 15;   // polynomial and dimension (staging); operand row or column
  const int sub = wave >> 2;  // sub-chunk this wave stages; those of the first take the sums
  const int blk = wave & 1, part = (wave >> 1) & 1;
  const int64_t N = a.g.N;
  const int start = a.item_start[item];
  const int cnt = a.item_count[item];
  const R edge = a.edge;

  // node data of a chunk, in registers one chunk ahead: cell word and one
  // offset of the four nodes whose factors this lane evaluates, the cell words
  // of node `lane` of every sub-chunk, and (wave r of a sub-chunk's) weight,
  // sample and index of its node `lane` for right-hand side r
  uint32_t Ln[4], Lb[NS] = {};
  R xn[4];
  cplx<R> wv = mkc<R>(0, 0), fv = wv;
  int jn = 0;
  const uint32_t* loc = a.loc + start;
  const int dim = j >> 3, jj = j & 7;
  const R* fr = a.frac + start + (dim ? N : 0) + kq;
  const int cr = wave & 3, cn = 64 * sub + lane;
  const bool cw = cr < nr;
  const cplx<R>* f = a.f + (rhs0 + (cw ? cr : 0)) * a.f_rs;
  // Nodes past the item's last are its neighbours' or the arrays' padding:
  // their cell words are not counted and their c is taken as zero.
  auto load_chunk = [&](int b0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      Ln[t] = (loc + b0 + 16 * wave + 4 * t)[kq];
      xn[t] = (fr + b0 + 16 * wave + 4 * t)[0];
    }
    if (sub == 0)
#pragma unroll
      for (int u = 0; u < NS; ++u) Lb[u] = (loc + b0 + 64 * u)[lane];
    if (cw) {
      wv = (a.w + start + b0)[cn];
      fv = f[jn];
      jn = (a.perm + start + b0 + NN)[cn];
    }
  };
  if (cw) jn = (a.perm + start)[cn];

  // The window is even: the polynomial of cell 2m - 1 - p is that of cell p
  // at -y. Lane p < m of a node's 16 evaluates the sums of the odd terms and of
  // the even terms from y^2 on of polynomial p at the node's row offset, and
  // from them both cells, lane 8 + p at its column offset. The last two steps
  // are Horner's, so that c_0, the largest term, enters in one rounding: float32
  // errors of whole transforms over the LDS kernel's 0.94 to 1.01, with the
  // even part closed before the odd one is added 0.94 to 1.02. The entries past
  // the window (its cells 2m .. 15: zeros and, as cell 15, the closed edge) fall
  // to the lanes p >= m.
  R ce[DEG / 2 + 1], co[DEG / 2];
  const R* pcf = a.coef + (jj < MW ? jj : 0) * (DEG + 1);
#pragma unroll
  for (int t = 0; t <= DEG / 2; ++t) ce[t] = pcf[2 * t];
#pragma unroll
  for (int t = 0; t < DEG / 2; ++t) co[t] = pcf[2 * t + 1];
#pragma unroll
  for (int t = 0; t <= DEG / 2; ++t) ce[t] = jj < MW ? ce[t] : (R)0;
#pragma unroll
  for (int t = 0; t < DEG / 2; ++t) co[t] = jj < MW ? co[t] : (R)0;
  const int c1 = jj < MW ? jj : MW + jj;               // this lane's two cells
  const int c2 = jj < MW ? K2 - 1 - jj : jj == 7 ? -1 : 8 + jj;
  const int pm = dim ? 31 : 15;  // entry of padded row or column i: i & pm
  // lane whose second cell is the closed edge (m < 8), or whose column 16
  // before its second cell is (m = 8: cell 15 is column l1 + 16)
  const uint32_t em = jj == (FULL ? 0 : 7) && (dim || !FULL) ? 1u << (kEdgeShift + dim) : 0u;
  load_chunk(0);

  // rows past the last node of a first, short chunk are read by its last
  // group: any finite value will do (their c is taken as zero)
  {
    const int z0 = cnt < NN ? cnt : NN;
    for (int i = tid; i < (NRow - NN) * FS; i += NT) tab[z0 * FS + i] = (R)0;
  }

  // float32: a cell's sum is formed in runs of about RUN groups, in NA
  // interleaved parts, which are added in float64: error against float64 over
  // the LDS kernel's 0.94 to 1.01; with runs of twice the groups, their parts
  // added in float32, 1.02 to 1.06
  v4 acc[NA][NR];
  double big[F32 ? NR : 1][4];
  R er[NR], pend[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
#pragma unroll
    for (int u = 0; u < NA; ++u) acc[u][r] = v4{(R)0, (R)0, (R)0, (R)0};
    if constexpr (F32)
#pragma unroll
      for (int v = 0; v < 4; ++v) big[r][v] = 0.0;
    er[r] = pend[r] = (R)0;
  }
  auto fold = [&](int r, auto vc) {
    constexpr int v = decltype(vc)::value;
    if constexpr (F32) {
      double s = (double)acc[0][r][v] + (double)acc[1][r][v];
      if constexpr (NA == 4) s += (double)acc[2][r][v] + (double)acc[3][r][v];
      big[r][v] += s;
#pragma unroll
      for (int u = 0; u < NA; ++u) acc[u][r][v] = 0.0f;
    }
  };
  auto fold_all = [&]() {
#pragma unroll
    for (int r = 0; r < NR; ++r) static_for<0, 4>([&](auto vc) { fold(r, vc); });
  };
  // element v of the (folded) sums, and its clearing in the lanes with `in`
  auto total = [&](int r, int v) {
    if constexpr (F32)
      return (R)big[r][v];
    else
      return acc[0][r][v];
  };
  auto clear = [&](bool in, int r, int v) {
    if constexpr (F32)
      big[r][v] = in ? 0.0 : big[r][v];
    else
      acc[0][r][v] = in ? (R)0 : acc[0][r][v];
  };
  const int col = 16 * blk + j;
  const R* opA = tab + kq * FS + M4::slot(j);
  const R* opB = tab + kq * FS + 16 + 16 * blk + j;
  const R* opC = ct + part * NR * NRow + kq;
  R* out_lds = reinterpret_cast<R*>(tiles) + part;  // part of cell i at 2 i
  bool edges = false;

  // slots of band b (its rows are complete): to the tile, cleared. For bands
  // of less than four rows the element is a uniform branch.
  auto take_v = [&](bool in, auto vc) {
    constexpr int v = decltype(vc)::value;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      fold(r, vc);
      if constexpr (FULL) {
        pend[r] = total(r, v);
      } else {
        if (in && col < P) out_lds[2 * ((r * P + 4 * kq + v) * P + col)] = total(r, v);
      }
      clear(in, r, v);
    }
  };
  auto take = [&](int b) {
    if constexpr (RB >= 4) {
      const bool in = kq / (RB / 4) == b;
      static_for<0, 4>([&](auto vc) { take_v(in, vc); });
    } else {
      const bool in = kq == b * RB / 4;
      static_for<0, 4 / RB>([&](auto gc) {
        constexpr int g = decltype(gc)::value;
        if (b % (4 / RB) == g)
          static_for<g * RB, g * RB + RB>([&](auto vc) { take_v(in, vc); });
      });
    }
  };
  // m = 8: row b, taken out before its nodes, with its nodes' closed-edge sums
  auto put_row = [&](int b) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      R v = pend[r];
      if (edges) {
        R s = er[r];
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        v += edge * s;
        er[r] = (R)0;
      }
      if (kq == b >> 2) out_lds[2 * ((r * P + b) * P + col)] = v;
    }
    edges = false;
  };

  int band = 0, run = 0;
  if constexpr (FULL) take(0);
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
      const R v1 = ce[0] + y * (od + y * ev);
      R v2 = ce[0] - y * (od - y * ev);
      const int l = (int)((L >> (kLocBits * dim)) & kLocMask);
      const int t1 = (l + 1 + c1) & pm, t2 = (l + 1 + c2) & pm;
      const R ed = L & em ? edge : (R)0;
      if constexpr (!FULL) v2 += ed;  // zero in the edge's lane
      R* row = tab + (16 * wave + 4 * t + kq) * FS + 16 * dim;
      row[t1] = v1;
      row[t2] = v2;
      if (dim) {
        // the same column of the other block
        row[t1 ^ 16] = (R)0;
        row[t2 ^ 16] = FULL ? ed : (R)0;
      }
      if constexpr (FULL)
        if (j == 0) et[16 * wave + 4 * t + kq] = (L >> kEdgeShift) & 1u ? (R)1 : (R)0;
    }
    if (cw) {
      ct[cr * NRow + cn] = wv.x * fv.x - wv.y * fv.y;
      ct[(NR + cr) * NRow + cn] = wv.x * fv.y + wv.y * fv.x;
    }
    int mb[NS];  // bands
    bool any_edge = false;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const bool valid = 64 * u + lane < nb;
      mb[u] = valid ? (int)(Lb[u] & kLocMask) / RB : NBAND;
      if constexpr (FULL)
        any_edge |= __builtin_amdgcn_ballot_w64(valid && ((Lb[u] >> kEdgeShift) & 1u)) != 0;
    }
    const bool has_edge = FULL && any_edge;
    __syncthreads();
    if (b0 + NN < cnt) load_chunk(b0 + NN);
    if (sub) continue;
    for (int n = 0; n < nb;) {
      // the band's end: nodes are sorted by row
      int e = 0;
#pragma unroll
      for (int u = 0; u < NS; ++u)
        e += __builtin_popcountll(__builtin_amdgcn_ballot_w64(mb[u] <= band));
      // whole groups, four at a time
      for (; n + 16 <= e; n += 16) {
        R A[4], B[4], c[4][NR];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          A[u] = opA[(n + 4 * u) * FS];
          B[u] = opB[(n + 4 * u) * FS];
#pragma unroll
          for (int r = 0; r < NR; ++r) c[u][r] = opC[r * NRow + n + 4 * u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int r = 0; r < NR; ++r)
            acc[u % NA][r] = M4::mfma(A[u] * c[u][r], B[u], acc[u % NA][r]);
        if constexpr (F32 && NS > 1)
          if ((run += 4) >= RUN) {
            fold_all();
            run = 0;
          }
        if constexpr (FULL)
          if (has_edge) {
            edges = true;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const R eb = et[n + 4 * u + kq] * B[u];
#pragma unroll
              for (int r = 0; r < NR; ++r) er[r] += eb * c[u][r];
            }
          }
      }
      // the rest of the band in this chunk; its parts from `first` on
      auto rest = [&](auto fc) {
        constexpr int first = decltype(fc)::value;
#pragma unroll
        for (int u = 0; u < 4; ++u, n += 4) {
          if (n >= e) break;
          const bool in = kq < e - n;
          const R A = opA[n * FS], B = opB[n * FS];
          R c[NR];
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            c[r] = opC[r * NRow + n];
            c[r] = in ? c[r] : (R)0;
            v4& p = acc[(first + u) % NA][r];
            p = M4::mfma(A * c[r], B, p);
          }
          if constexpr (FULL)
            if (has_edge) {
              edges = true;
              const R eb = in ? et[n + kq] * B : (R)0;
#pragma unroll
              for (int r = 0; r < NR; ++r) er[r] += eb * c[r];
            }
        }
      };
      if constexpr (FULL && F32) {  // a row has few groups: every second one starts at part 2
        if (band & 1)
          rest(std::integral_constant<int, 2>{});
        else
          rest(std::integral_constant<int, 0>{});
      } else {
        rest(std::integral_constant<int, 0>{});
      }
      n = e;
      if (n < nb) {  // the band is complete: further nodes lie below it
        if constexpr (FULL) {
          put_row(band);
          take(band + 1);
        } else {
          take(band);
        }
        ++band;
        if (RB >= 4) run = 0;  // the band's end has added every run
      }
    }
    if constexpr (NS == 1) run += nb / 4;
    if (F32 && run >= RUN) {
      fold_all();
      run = 0;
    }
  }
  if (sub == 0) {
    for (; band < NBAND; ++band) {
      if constexpr (FULL) {
        put_row(band);
        if (band + 1 < NBAND) take(band + 1);
      } else {
        take(band);
      }
    }
    fold_all();
    // padded rows 16 .. P - 1: slot s holds row 16 + s
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 16 + 4 * kq + v;
      if (row < P && col < P)
#pragma unroll
        for (int r = 0; r < NR; ++r) out_lds[2 * ((r * P + row) * P + col)] = total(r, v);
    }
  }
  __syncthreads();

  const int slot = a.item_slot[item];
  cplx<R>* out = slot < 0 ? a.tilep + (int64_t)a.item_bin[item] * (P * P)
                          : a.itemp + (int64_t)slot * (P * P);
  const int64_t rs = slot < 0 ? a.tile_rs : a.item_rs;
  constexpr int VW = 16 / sizeof(R);  // 16-byte copies
  for (int r = 0; r < nr; ++r) {
    const float4* src = reinterpret_cast<const float4*>(tiles + r * P * P);
    float4* dst = reinterpret_cast<float4*>(out + (rhs0 + r) * rs);
    for (int i = tid; i < 2 * P * P / VW; i += NT) dst[i] = src[i];
  }
}

bool spread_tile_supported(int d, int T, int m) {
  return d == 2 && T == kTileT && m >= 1 && m <= 8;
}

// The default spread mode's choice. Its lines are from whole transforms (graph
// replays) of uniform, polar and spiral sets, M = 16 .. 512, 1 to 512 nodes a
// tile, 1, 2 and 11 right-hand sides; times in us, LDS kernel > this one.
//
// Items: joining up to two saves the sum of split tiles, but doubles the chain
// of chunks that a work-group takes one after the other (float64, m = 6: 6 us, m
// = 8: 8). With few work-groups it pays while the chain grows by one chunk, in
// float32 (sixteen staging waves up to m = 7) by two (float64, m = 6, 16 tiles of
// 256 uniform nodes 20.4 -> 18.8, of 512 20.4 -> 26.8; float32, 371 a tile
// 17.2 -> 16.7). Where the default items are about one work-group per compute
// unit or more and the joined ones are at most that, also with longer chains
// (256 tiles, half the nodes in half of them, longest 351 26.2 -> 23.4, 492 25.9 ->
// 26.5; all alike, 503 30.6 -> 26.8), with the device full of joined items always
// (4096 tiles of 256 127 -> 99.5). Tiles that stay split: from three default
// items per compute unit on (m = 8: 130464 polar nodes on 224 tiles 37.4 -> 38.5,
// 261936 on 856 55.2 -> 55.4, 2097152 uniform ones on 4096 284 -> 233).
//
// Kernel: while the LDS kernel has up to two work-groups per compute unit
// (float64 at m = 8: 300), the longest item is the time of either kernel, with
// more of them the mean item.
// float64, few: m = 3, longest 217 15.1 > 16.0, 256 19.2 > 19.4, 289 (joined)
// 19.0 > 17.5; m = 4, 148 14.2 > 14.5, 217 16.3 > 16.2; m = 6, 71 13.1 > 13.7,
// 104 14.5 > 14.0; m = 8, 256 on a spiral 26.7 > 27.4 and on uniform nodes 27.2 >
// 24.5: the LDS kernel but for joined items (298 on a spiral 26.2 > 27.1, 296 on
// uniform nodes 26.8 > 23.3). Many: m = 3, mean 192 76.6 > 79.1, 256 (joined)
// 107 > 92.8; m = 4, 64 25.0 > 25.6, 96 28.1 > 27.9; m = 6, 22 48.6 > 51.6, 64
// 63.0 > 59.4; m = 8, 96 94.7 > 95.5, 128 116 > 103. At m <= 2 about even at best
// (joined, mean 256, m = 2 36.6 > 34.3 and 88.9 > 91.7): the LDS kernel.
// float32, few: m = 4, longest 13 11.3 > 10.9, m = 2, 13 10.7 > 10.8, 104 13.4 >
// 12.4; m = 8, 223 on a spiral 23.2 > 24.7, 256 27.2 > 26.5 but on other spirals
// 0.98 of the LDS kernel: left to that. Many: m = 2, mean 192 23.3 > 24.1, 256
// (joined) 31.3 > 27.0; m = 3, 22 17.3 > 18.1, 64 19.2 > 19.4 and, on 4096 tiles,
// 45.5 > 41.7; m = 4, 22 18.3 > 18.6 and 42.4 > 37.9; m = 8, 45 29.5 > 28.4.
TileChoice spread_tile_choice(bool f64, int m, int64_t N, int nrhs, const ItemShape& items,
                              const ItemShape& joined) {
  const int64_t wgs = (int64_t)items.n * nrhs;
  bool join = false;
  if (joined.n > 0) {
    const int pairs = (nrhs + 1) / 2;  // as the launch below groups them
    const int64_t groups = (int64_t)joined.n * pairs >= 512 ? pairs : nrhs;
    const bool dense = N * groups >= 3 * 256 * 256;
    const bool quick = !f64 && m <= 7;
    int chain = quick ? 400 : 320;
    if (wgs >= 240) chain = quick && wgs <= 768 ? 512 : 400;
    if (wgs >= 360 && 3 * N >= 2 * (int64_t)joined.longest * joined.n) chain = 512;
    if (joined.n * groups >= 1024 || dense) chain = 512;
    join = joined.split ? dense : joined.longest <= chain;
  }
  const ItemShape& it = join ? joined : items;
  const TileChoice tile = join ? TileChoice::kJoined : TileChoice::kItems;
  // from which longest or mean item on, by m; X: not at all
  constexpr int X = 1 << 30;
  if (wgs <= (f64 && m == 8 ? 300 : 512)) {
    static const int longest64[9] = {X, X, X, 256, 160, 160, 100, 100, X};
    static const int longest32[9] = {X, 128, 128, 0, 0, 0, 0, 0, X};
    if (f64 && m == 8) return join ? tile : TileChoice::kLds;
    return it.longest >= (f64 ? longest64 : longest32)[m] ? tile : TileChoice::kLds;
  }
  static const int mean64[9] = {X, X, X, 200, 110, 110, 64, 64, 110};
  static const int mean32[9] = {X, 200, 200, 64, 0, 0, 0, 0, 64};
  int64_t mean = (f64 ? mean64 : mean32)[m];
  // with tiles still split the sum of their slots takes the gain up to denser
  // sets (m = 2, mean 264 29.7 > 30.5, 342 47.9 > 41.5)
  if (m <= 2 && it.split) mean = m == 2 && !f64 && wgs >= 1280 ? 300 : X;
  return N >= mean * it.n ? tile : TileChoice::kLds;
}

size_t spread_tile_lds_bytes(int m, bool f64) {
  // one right-hand side; float32 at m <= 7 in its largest form
  const size_t P = kTileT + 2 * m, rb = f64 ? 8 : 4;
  const size_t ns = f64 || m == 8 ? 1 : 4;
  return P * P * 2 * rb + (ns * kTileChunk + kTilePast) * (kTileFS + 3) * rb;
}

template <typename R, int MW, int NR, int NS>
static hipError_t spread_tile_nr(const SpreadArgs<R>& a, int nrhs, hipStream_t s) {
  hipLaunchKernelGGL((spread_tile_kernel<R, MW, NR, NS>), dim3(a.g.nsub, (nrhs + NR - 1) / NR),
                     dim3(256 * NS), (TileLds<R, MW, NR, NS>::bytes), s, a, nrhs);
  return hipGetLastError();
}

// Two right-hand sides per work-group where that leaves two work-groups per
// compute unit: one evaluation of the window serves both. Four took, spiral of
// 40321 nodes, M = 128, m = 6, 11 right-hand sides, float32, with the two parts
// that fit in their registers, 57.4 against 52.0 us.
template <typename R, int MW>
static hipError_t spread_tile_m(const SpreadArgs<R>& a, int nrhs, hipStream_t s) {
  if (nrhs > 1 && (int64_t)a.g.nsub * ((nrhs + 1) / 2) >= 512)
    return spread_tile_nr<R, MW, 2, 1>(a, nrhs, s);
  // At most one work-group per compute unit, of several chunks: nothing covers
  // the waits of a chunk's staging, so 16 waves stage four chunks at a time
  // (float32, whole transforms, against one at a time: 20001 nodes, M = 32,
  // m = 4, 23.7 -> 21.2 us; 40321, M = 128, m = 6, 16.9 -> 16.0). Not at m = 8
  // (140000, M = 128: 32.1 -> 32.8), nor in float64, whose products cover them
  // (4096, M = 32, m = 4: 18.4 -> 19.0).
  if constexpr (std::is_same<R, float>::value && MW <= 7)
    if ((int64_t)a.g.nsub * nrhs <= 256 && a.g.N > (int64_t)kTileChunk * a.g.nsub)
      return spread_tile_nr<R, MW, 1, 4>(a, nrhs, s);
  return spread_tile_nr<R, MW, 1, 1>(a, nrhs, s);
}

template <typename R>
hipError_t launch_spread_tile(const SpreadArgs<R>& a, int nrhs, hipStream_t s) {
  if (!spread_tile_supported(a.g.d, a.g.T, a.g.m)) return hipErrorInvalidValue;
  if (a.g.nsub == 0) return hipSuccess;
  switch (a.g.m) {
    case 1: return spread_tile_m<R, 1>(a, nrhs, s);
    case 2: return spread_tile_m<R, 2>(a, nrhs, s);
    case 3: return spread_tile_m<R, 3>(a, nrhs, s);
    case 4: return spread_tile_m<R, 4>(a, nrhs, s);
    case 5: return spread_tile_m<R, 5>(a, nrhs, s);
    case 6: return spread_tile_m<R, 6>(a, nrhs, s);
    case 7: return spread_tile_m<R, 7>(a, nrhs, s);
    case 8: return spread_tile_m<R, 8>(a, nrhs, s);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_spread_tile<float>(const SpreadArgs<float>&, int, hipStream_t);
template hipError_t launch_spread_tile<double>(const SpreadArgs<double>&, int, hipStream_t);

}  // namespace nfft
