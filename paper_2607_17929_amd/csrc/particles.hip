// Particle kernels: ingest, CIC deposit, gather + kick + drift, counting sort by cell.
//
// The particle store (arrays of records, kernels.h) is kept sorted by mesh cell in row-major order
// key = (iz n + iy) n + ix, so that the particles of one x-row of cells are
// contiguous and ordered along x, as in the paper's particle handler
// (Sec. 2.1).  cell_start[key] .. cell_start[key + 1] is the range of a cell.
#include <type_traits>

#include "kernels.h"

namespace gpm {

__device__ __forceinline__ void cell_of(double x, int n, int& i, double& f) {
  // n is a power of two, so x * n is exact in FP64
  const double s = x * (double)n;
  const double fl = floor(s);
  f = s - fl;
  i = ((int)fl) & (n - 1);
}

__device__ __forceinline__ double wrap01(double x) {
  double y = x - floor(x);
  return (y >= 1.0) ? 0.0 : y;
}

__device__ __forceinline__ uint32_t cell_key(double x, double y, double z, int n) {
  int ix, iy, iz;
  double f;
  cell_of(x, n, ix, f);
  cell_of(y, n, iy, f);
  cell_of(z, n, iz, f);
  return ((uint32_t)iz * (uint32_t)n + (uint32_t)iy) * (uint32_t)n + (uint32_t)ix;
}

// ---------------------------------------------------------------------------
// ingest: [n][3] inputs -> store, wrap, validate, rank within the cell
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void ingest_kernel(const double* pos, const T* u, const uint32_t* ids, long np,
                                                     Particles<T> out, int nmesh, uint32_t* rank, uint32_t* cnt,
                                                     int* err) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  const V3<double> pi = *reinterpret_cast<const V3<double>*>(pos + 3 * i);
  const V3<T> ui = *reinterpret_cast<const V3<T>*>(u + 3 * i);
  double x = pi.x, y = pi.y, z = pi.z;
  T ux = ui.x, uy = ui.y, uz = ui.z;
  if (!(isfinite(x) && isfinite(y) && isfinite(z) && isfinite(ux) && isfinite(uy) && isfinite(uz))) {
    atomicOr(err, 1);
    x = y = z = 0.0;
    ux = uy = uz = (T)0;
  }
  x = wrap01(x); y = wrap01(y); z = wrap01(z);
  uint32_t id = ids ? ids[i] : (uint32_t)i;
  if ((long)id >= np) {
    atomicOr(err, 2);
    id = 0;
  }
  store_particle(out, i, Particle<T>{x, y, z, ux, uy, uz, id});
  const uint32_t k = cell_key(x, y, z, nmesh);
  rank[i] = atomicAdd(&cnt[k], 1u);
}

template <typename T>
void launch_ingest(const double* pos_aos, const T* u_aos, const uint32_t* ids, long n, Particles<T> out, int nmesh,
                   uint32_t* rank, uint32_t* cnt, int* err, hipStream_t st) {
  hipLaunchKernelGGL((ingest_kernel<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, pos_aos, u_aos, ids, n,
                     out, nmesh, rank, cnt, err);
}

// ---------------------------------------------------------------------------
// CIC deposit without atomics, streamed along z.  A workgroup owns a column of
// TX x TY vertices (x, y) over zb vertex planes and walks the cell planes
// z0 - 1 .. z0 + zb - 1 in order.  The particles of one cell plane that touch
// the column -- TY + 1 cell rows, each the halo cell x0 - 1 and the cells
// x0 .. x0 + TX - 1, i.e. two contiguous ranges of the cell-sorted store -- are
// staged in LDS (cell fractions, energy, momentum and the stresses u_i u_j / e),
// and each thread, owning one vertex column, sums the contributions of the
// particles of its 4 cells of the plane in one loop over both cell rows:
// weight (1 - f_z) to the vertex on the plane's lower face, f_z to the one on
// its upper face.  A vertex plane is complete after the cell planes below and
// above it and is stored then, so every cell plane is read once per column.
// While a plane is summed, the particles of the next plane are being loaded
// into registers and the cell offsets of the plane after the next one too (row
// offsets of the staged lists are scanned in LDS, three planes in flight).
// Only cell_start and the particle arrays are read; each vertex is written once.
// ---------------------------------------------------------------------------
// Workgroups of 256 threads and 32 x 8 vertex columns, on the largest meshes 128 threads and 32 x 4 (clustered: 512^3
// 5.18 ms against 5.79, FP64 5.96 against 6.55, 1024^3 with 512^3 particles 16.5 against 18.0; at 128^3 and 256^3 they
// take 0.39 against 0.37 and 0.45 against 0.44 ms): one column a thread.
__host__ __device__ constexpr int dep_nt(int n) { return n >= 512 ? 128 : 256; }
// staged particles per chunk: a plane of mean density fits one (33 x 9 or 33 x 5 cells), in FP64 with three waves a SIMD
template <typename T, int NT> constexpr int dep_cap() { return sizeof(T) == 4 ? 2 * NT : 3 * NT / 2; }
// Vertex planes per workgroup: 16, and fewer where that leaves fewer than DEP_WAVES waves (four rounds of 16 on
// every CU): a 32^3 mesh in 16-plane columns is 8 workgroups that walk 17 cell planes each (59 us; 13 us with
// single planes), a clustered 128^3 mesh 512 of them (0.42 ms; 0.38 with the 2 planes taken here).
constexpr int DEP_ZB = 16, DEP_WAVES = 16384;
// A cell of this many particles or more is summed by the whole wave on the matrix cores (crowded_cell below): in the
// lane loop its n particles cost a lane of each of 4 vertex columns 45 n instructions while 60 others wait, here
// n / 4 matrix products and about 100 instructions (FP64, cells of up to 690: 256^3 clustered deposit 1.45 -> 1.05 ms).
// The FP32 stress-energy stays in the lane loop: its stresses are FP32 sums that run through the particles in the
// store's order, and in any other order or width a run's last bits change (clustered 512^3 5.18 ms, on the matrix
// cores 4.32; 256^3 1.13 and 0.79, 128^3 0.38 and 0.22; eight lanes to a vertex, which keep the order, 5.24, 1.25, 0.45).
constexpr uint32_t DEP_CROWD = 12;

__host__ __device__ constexpr int dep_tx(int n) { return n >= 32 ? 32 : 16; }

// exclusive prefix of c over the first wave's lanes (R <= 64 rows): off[0] = 0, off[r + 1] = sum_{q <= r} c_q
template <int R>
__device__ __forceinline__ void wave_row_offsets(uint32_t c, uint32_t* off) {
  const int lane = threadIdx.x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = __shfl_up(c, d);
    if (lane >= d) c += t;
  }
  if (lane < R) off[lane + 1] = c;
  if (lane == 0) off[0] = 0;
}

// largest r in [0, R) with off[r] <= i, for a non-decreasing off with off[0] = 0 <= i (R <= 64)
template <int R>
__device__ __forceinline__ int row_of(const uint32_t* off, uint32_t i) {
  int lo = 0;
#pragma unroll
  for (int step = 32; step > 0; step >>= 1)
    if (step < R && lo + step < R && off[lo + step] <= i) lo += step;
  return lo;
}

typedef double v4d __attribute__((ext_vector_type(4)));

template <typename T, int NC, bool REL, int TX, int DEP_NT>
__global__ __launch_bounds__(DEP_NT, sizeof(T) == 4 ? 4 : 3) void deposit_kernel(Particles<T> p, const uint32_t* __restrict__ cell_start, int n,
                                                         int zb, T a, double a64, T w, double wd, int accumulate,
                                                         T* __restrict__ dep, double* __restrict__ esum,
                                                         const float* __restrict__ vals) {
  constexpr int TY = DEP_NT / TX, ROWS = TY + 1, RW = TX + 3;  // raw offsets per row: halo start/end, x0 .. x0 + TX
  constexpr int CAP = dep_cap<T, DEP_NT>(), SPT = (CAP + DEP_NT - 1) / DEP_NT;
  constexpr int NQ = (ROWS * RW + DEP_NT - 1) / DEP_NT;
  constexpr int N4 = NC < 4 ? NC : 4, N6 = NC > 4 ? NC - 4 : 1;
  constexpr int WX = TX >= 16 ? 16 : TX, WY = 64 / WX;         // a wave's vertex columns: WX x WY
  static_assert(ROWS <= 64 && TX % WX == 0 && TY % WY == 0, "tile shape");
  // (a count takes so little that the test for crowded cells costs more)
  constexpr bool CROWD = NC == 3 || (NC > 4 && sizeof(T) == 8);
  constexpr bool VEC = NC == 3;               // sums of W v for the 3-vectors vals[id] instead of the stress-energy
  constexpr int C4 = NC > 1 ? CAP : 1, C6 = NC > 4 ? CAP : 1;
  __shared__ V4<T> sfr[CAP];                  // f_x, f_y, f_z, -
  __shared__ V4<T> sq[C4], ss[C6];            // (e, u_x, u_y, u_z), (u_x u_x, u_x u_y, u_x u_z, u_y u_y) / e
  __shared__ T ss2[C6][2];                    // (u_y u_z, u_z u_z) / e
  __shared__ uint32_t raw[3][ROWS][RW];       // cell offsets of the planes in flight (plane mod 3)
  __shared__ uint32_t roff[3][ROWS + 1];      // staged offset of each row
  __shared__ double red[DEP_NT / 64];
  __shared__ double scr[CROWD ? DEP_NT / 64 : 1][8][NC];  // corner sums of a crowded cell
  const int m = n - 1;
  int bx, by, bz;
  xcd_block3(bx, by, bz);
  const int x0 = bx * TX, y0 = by * TY, zs = bz * zb;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // waves of WX x WY vertex columns (the clustered occupancy is less uneven over squarer patches)
  const int lvx = (wave % (TX / WX)) * WX + lane % WX, lvy = (wave / (TX / WX)) * WY + lane / WX;
  const long nn = (long)n * n, n3 = nn * n;

  // the thread index as a value of this place: with ten quantities, what is formed from it is formed again in
  // every plane instead of being kept in registers through all of them (the sums and the prefetch fill the
  // 128 registers of four waves a SIMD; a few spilled ones cost 8 to 20 % of the kernel's time)
  auto here = [&]() {
    int t = tid;
    if constexpr (NC > 4) asm volatile("" : "+v"(t));
    return t;
  };
  // raw cell offsets of cell plane cz: row r is cell row y0 - 1 + r; entry 0/1 = start/end of the
  // halo cell x0 - 1, entry 2 + j = start of cell x0 + j (j = 0 .. TX)
  auto load_raw = [&](int cz, uint32_t* v) {
    const int t0 = here();
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const int q = t0 + k * DEP_NT;
      if (q < ROWS * RW) {
        const int r = q / RW, j = q - r * RW;
        const uint32_t rb = ((uint32_t)(cz & m) * (uint32_t)n + (uint32_t)((y0 - 1 + r) & m)) * (uint32_t)n;
        const uint32_t hc = rb + (uint32_t)((x0 - 1) & m);
        v[k] = cell_start[j == 0 ? hc : (j == 1 ? hc + 1 : rb + x0 + (j - 2))];
      }
    }
  };
  auto store_raw = [&](int b, const uint32_t* v) {
    const int t0 = here();
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const int q = t0 + k * DEP_NT;
      if (q < ROWS * RW) raw[b][q / RW][q % RW] = v[k];
    }
  };
  // staged offsets of the rows of the plane in buffer b (first wave)
  auto scan_rows = [&](int b) {
    if (tid < 64) {
      uint32_t c = 0;
      if (tid < ROWS) c = (raw[b][tid][1] - raw[b][tid][0]) + (raw[b][tid][2 + TX] - raw[b][tid][2]);
      wave_row_offsets<ROWS>(c, roff[b]);
    }
  };
  // global index of staged particle i of the plane in buffer b; own: in a cell of this column
  auto source_of = [&](int b, uint32_t i, bool& own) {
    const int r = row_of<ROWS + 1>(roff[b], i);
    const uint32_t k = i - roff[b][r];
    const uint32_t hs = raw[b][r][0], hn = raw[b][r][1] - hs;
    own = r > 0 && k >= hn;
    return k < hn ? hs + k : raw[b][r][2] + (k - hn);
  };
  using Held = std::conditional_t<(NC > 4), Loaded<T>, Particle<T>>;
  auto load_part = [&](uint32_t g, Held& d) {
    if constexpr (NC > 4) {
      load_raw_state(p, g, d);
    } else {
      load_pos(p, g, d);
    }
    if constexpr (VEC) {
      const long id = load_id(p, g);
      d.ux = vals[3 * id]; d.uy = vals[3 * id + 1]; d.uz = vals[3 * id + 2];
    }
  };
  double e_own = 0.0;
  auto stage = [&](uint32_t l, const Held& held, bool own) {
    Particle<T> d;
    if constexpr (NC > 4) d = unpacked(held);
    else d = held;
    const double sx = d.x * (double)n, sy = d.y * (double)n, sz = d.z * (double)n;
    V4<T> fr;
    fr.x = (T)(sx - floor(sx));
    fr.y = (T)(sy - floor(sy));
    fr.z = (T)(sz - floor(sz));
    fr.w = (T)0;
    sfr[l] = fr;
    if constexpr (VEC) {
      sq[l] = V4<T>{d.ux, d.uy, d.uz, (T)0};
    } else if constexpr (NC > 1) {
      const T vx = d.ux, vy = d.uy, vz = d.uz;
      const T u2 = vx * vx + vy * vy + vz * vz;
      const T e = REL ? sqrt(a * a + u2) : a;
      const T ie = rcp(e);
      V4<T> q, t;
      q.x = e; q.y = vx; q.z = vy; q.w = vz;
      const T ix = vx * ie, iy = vy * ie;
      t.x = ix * vx; t.y = ix * vy; t.z = ix * vz; t.w = iy * vy;
      sq[l] = q;
      ss[l] = t;
      ss2[l][0] = iy * vz;
      ss2[l][1] = vz * ie * vz;
      // FP64 sum over the particles of this column's own cells (the homogeneous source of phi is its
      // small difference from the background, so e is formed from the momenta in FP64 here)
      if (own) {
        const double dx = vx, dy = vy, dz = vz;
        e_own += REL ? sqrt(a64 * a64 + dx * dx + dy * dy + dz * dz) : a64;
      }
    }
  };

  // sums of the vertex on the current plane's lower face (lo) and upper face (hi): n00 and n0i in FP64
  // (each product w q in T), the stresses in T.  The lagged time derivative of phi is the change
  // between two solves, which would otherwise carry the independent rounding of two FP32 sums over a
  // crowded cell amplified by |phi| / |phi_n - phi_{n-1}|.
  double lo4[N4], hi4[N4];
  T lo6[N6], hi6[N6];
#pragma unroll
  for (int c = 0; c < N4; ++c) lo4[c] = hi4[c] = 0.0;
#pragma unroll
  for (int c = 0; c < N6; ++c) lo6[c] = hi6[c] = (T)0;

  // The 8 corner sums of one crowded cell's n staged particles from b0 on, by the whole wave on the
  // matrix cores: a 16x16x4 FP64 product of corner weights (rows) and quantities (columns) over the
  // particles, four to an instruction; lane l feeds row and column l % 16 of particle l / 16.  The sums
  // go through the wave's scratch to the lanes of the cell's 4 vertex columns (cell c, row r of the tile).
  auto crowded_cell = [&](uint32_t b0, uint32_t n, int c, int r) {
    const int mcol = here() & 15, mk4 = (here() & 63) >> 4;
    const T* qbase = nullptr;  // quantity mcol of staged particle 0 and its stride
    int qstride = 4;
    if constexpr (NC > 1) {
      qbase = reinterpret_cast<const T*>(NC < 4 || mcol < 4 ? sq : ss) + (mcol & 3);
      if (NC > 8 && mcol >= 8) { qbase = &ss2[0][mcol & 1]; qstride = 2; }
    }
    v4d acc = {0.0, 0.0, 0.0, 0.0};
    for (uint32_t k0 = 0; k0 < n; k0 += 4) {
      const uint32_t k = k0 + mk4;
      const uint32_t l = b0 + min(k, n - 1);  // (beyond the last particle: zeros, its own values may be infinite)
      const V4<T> fr = sfr[l];
      const T wx = (mcol & 1) ? fr.x : (T)1 - fr.x;
      const T wxy = wx * ((mcol & 2) ? fr.y : (T)1 - fr.y);
      const T wh = wxy * fr.z;
      const T w8 = (k < n && mcol < 8) ? ((mcol & 4) ? wh : wxy - wh) : (T)0;
      T q = a;
      if constexpr (NC > 1) q = qbase[l * qstride];
      if (k >= n) q = (T)0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)w8, (double)q, acc, 0, 0, 0);
    }
    // rows l / 16 (lower face) and 4 + l / 16 (upper face) of column l % 16
    if (mcol < NC) {
      scr[wave][mk4][mcol] = acc[0];
      scr[wave][4 + mk4][mcol] = acc[1];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const uint32_t ox = (uint32_t)(c - lvx), oy = (uint32_t)(r - lvy);
    if (ox <= 1u && oy <= 1u) {
      const int xy = (int)((1u - ox) + 2u * (1u - oy));
#pragma unroll
      for (int q = 0; q < N4; ++q) { lo4[q] += scr[wave][xy][q]; hi4[q] += scr[wave][4 + xy][q]; }
#pragma unroll
      for (int q = 4; q < NC; ++q) { lo6[q - 4] += (T)scr[wave][xy][q]; hi6[q - 4] += (T)scr[wave][4 + xy][q]; }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };

  // sum the staged particles [c0, c1) of the plane in buffer b: the thread's cells are, in the cell
  // rows lvy (below the vertex: weight f_y) and lvy + 1 (1 - f_y), the local cells lvx (x0 + lvx - 1,
  // weight f_x) and lvx + 1 (1 - f_x), one contiguous staged range per row.  Cells of DEP_CROWD
  // particles or more are left to the wave (crowded_cell): one of them would hold up 63 other lanes.
  auto accumulate_chunk = [&](int b, uint32_t c0, uint32_t c1) {
    uint32_t beg[2], spl[2], end[2];
#pragma unroll
    for (int dy = 0; dy < 2; ++dy) {
      const int r = lvy + dy;
      const uint32_t* rr = raw[b][r];
      const uint32_t hn = rr[1] - rr[0], m0 = rr[2], ro = roff[b][r];
      const uint32_t s0 = ro + (lvx == 0 ? 0u : hn + (rr[1 + lvx] - m0));
      const uint32_t s1 = ro + hn + (rr[2 + lvx] - m0);
      const uint32_t s2 = ro + hn + (rr[3 + lvx] - m0);
      const uint32_t bb = max(s0, c0), ee = max(min(s2, c1), bb);
      beg[dy] = bb - c0;
      end[dy] = ee - c0;
      spl[dy] = (CROWD ? min(max(s1, bb), ee) : max(s1, c0)) - c0;
    }
    if constexpr (CROWD) {
      const uint32_t most = max(max(spl[0] - beg[0], end[0] - spl[0]), max(spl[1] - beg[1], end[1] - spl[1]));
      if (__ballot(most >= DEP_CROWD)) {
        // the wave's crowded cells: each lane answers for the cell below and left of its vertex, the
        // lanes at the patch's upper edges for the cells beyond them too
        const bool ex = lane % WX == WX - 1, ey = lane / WX == WY - 1;
#pragma unroll 1
        for (int q = 0; q < 4; ++q) {
          const bool right = q & 1, up = q >> 1;
          const uint32_t lb = up ? +beg[1] : +beg[0], lm = up ? +spl[1] : +spl[0], le = up ? +end[1] : +end[0];
          const uint32_t cb = right ? +lm : +lb, cn = (right ? +le : +lm) - cb;
          uint64_t m = __ballot((!right || ex) && (!up || ey) && cn >= DEP_CROWD);
          while (m) {
            const int src = __builtin_ctzll(m);
            m &= m - 1;
            crowded_cell(__builtin_amdgcn_readlane(cb, src), __builtin_amdgcn_readlane(cn, src),
                         (wave % (TX / WX)) * WX + src % WX + (q & 1), (wave / (TX / WX)) * WY + src / WX + (q >> 1));
          }
        }
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
          if (spl[dy] - beg[dy] >= DEP_CROWD) beg[dy] = spl[dy];
          if (end[dy] - spl[dy] >= DEP_CROWD) end[dy] = spl[dy];
        }
      }
    }
    const uint32_t len[2] = {end[0] - beg[0], end[1] - beg[1]};
    const uint32_t tot = len[0] + len[1];
    for (uint32_t j = 0; j < tot; ++j) {
      const bool r1 = j >= len[0];
      const uint32_t l = r1 ? beg[1] + (j - len[0]) : beg[0] + j;
      const V4<T> fr = sfr[l];
      const T wx = l < (r1 ? spl[1] : spl[0]) ? fr.x : (T)1 - fr.x;
      const T wy = r1 ? (T)1 - fr.y : fr.y;
      const T wxy = wx * wy;
      // f_z and (1 - f_z) shares (the roundings of wl and of the stresses' sums are written out: runs repeat by them)
      const T wh = wxy * fr.z, wl = fma(wx, wy, -wh);
      if constexpr (NC == 1) {
        lo4[0] += (double)(wl * a);
        hi4[0] += (double)(wh * a);
      } else if constexpr (VEC) {
        const V4<T> q = sq[l];
        const double dl = (double)wl, dh = (double)wh;
        lo4[0] = fma(dl, (double)q.x, lo4[0]); lo4[1] = fma(dl, (double)q.y, lo4[1]); lo4[2] = fma(dl, (double)q.z, lo4[2]);
        hi4[0] = fma(dh, (double)q.x, hi4[0]); hi4[1] = fma(dh, (double)q.y, hi4[1]); hi4[2] = fma(dh, (double)q.z, hi4[2]);
      } else {
        const V4<T> q = sq[l], t = ss[l];
        const T t4 = ss2[l][0], t5 = ss2[l][1];
        const double dl = (double)wl, dh = (double)wh;
        const double q0 = (double)q.x, q1 = (double)q.y, q2 = (double)q.z, q3 = (double)q.w;
        lo4[0] = fma(dl, q0, lo4[0]); lo4[1] = fma(dl, q1, lo4[1]);
        lo4[2] = fma(dl, q2, lo4[2]); lo4[3] = fma(dl, q3, lo4[3]);
        hi4[0] = fma(dh, q0, hi4[0]); hi4[1] = fma(dh, q1, hi4[1]);
        hi4[2] = fma(dh, q2, hi4[2]); hi4[3] = fma(dh, q3, hi4[3]);
        lo6[0] = fma(wl, t.x, lo6[0]); lo6[1] = fma(wl, t.y, lo6[1]); lo6[2] = fma(wl, t.z, lo6[2]);
        lo6[3] = fma(wl, t.w, lo6[3]); lo6[4] = fma(wl, t4, lo6[4]); lo6[5] = fma(wl, t5, lo6[5]);
        hi6[0] = fma(wh, t.x, hi6[0]); hi6[1] = fma(wh, t.y, hi6[1]); hi6[2] = fma(wh, t.z, hi6[2]);
        hi6[3] = fma(wh, t.w, hi6[3]); hi6[4] = fma(wh, t4, hi6[4]); hi6[5] = fma(wh, t5, hi6[5]);
      }
    }
  };

  // prologue: offsets of the first three planes, row offsets of the first two, the first plane's
  // particles in flight
  {
    uint32_t v[NQ];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      if (q <= zb) {
        load_raw(zs - 1 + q, v);
        store_raw(q, v);
      }
    }
  }
  __syncthreads();
  scan_rows(0);
  scan_rows(1);
  __syncthreads();
  Held pr[SPT];
  bool pown[SPT];
  {
    const uint32_t lim = min(roff[0][ROWS], (uint32_t)CAP);
#pragma unroll
    for (int s2 = 0; s2 < SPT; ++s2) {
      const uint32_t i = tid + s2 * DEP_NT;
      if (i < lim) {
        bool own;
        load_part(source_of(0, i, own), pr[s2]);
      }
      pown[s2] = false;  // the first plane is below the column's own cells
    }
  }
  uint32_t rnext[NQ];
  for (int P = 0; P <= zb; ++P) {
    const int b = P % 3, b1 = (P + 1) % 3, b2 = (P + 2) % 3;
    const int cz = zs - 1 + P;
    const uint32_t total = roff[b][ROWS];
    // 1. the prefetched first chunk of this plane into LDS
    {
      const uint32_t lim = min(total, (uint32_t)CAP), t0 = here();
#pragma unroll
      for (int s2 = 0; s2 < SPT; ++s2) {
        const uint32_t i = t0 + s2 * DEP_NT;
        if (i < lim) stage(i, pr[s2], pown[s2]);
      }
    }
    __syncthreads();
    // 2. requests for the next planes: particles of plane P + 1, cell offsets of plane P + 3
    if (P + 1 <= zb) {
      const uint32_t lim = min(roff[b1][ROWS], (uint32_t)CAP), t1 = here();
#pragma unroll
      for (int s2 = 0; s2 < SPT; ++s2) {
        const uint32_t i = t1 + s2 * DEP_NT;
        pown[s2] = false;
        if (i < lim) load_part(source_of(b1, i, pown[s2]), pr[s2]);
      }
    }
    if (P + 3 <= zb) load_raw(cz + 3, rnext);
    // 3. sum this plane: (1 - f_z) to vertex plane cz, f_z to vertex plane cz + 1 (the first plane's
    //    lower-face sums and the last plane's upper-face sums belong to other columns and are dropped)
    for (uint32_t c0 = 0;;) {
      accumulate_chunk(b, c0, min(total, c0 + (uint32_t)CAP));
      c0 += CAP;
      if (c0 >= total) break;
      // a crowded plane: further chunks loaded and summed in turn
      const uint32_t c1 = min(total, c0 + (uint32_t)CAP);
      __syncthreads();
#pragma unroll
      for (int s2 = 0; s2 < SPT; ++s2) {
        const uint32_t i = c0 + here() + s2 * DEP_NT;
        if (i < c1) {
          bool own;
          Held d;
          load_part(source_of(b, i, own), d);
          stage(i - c0, d, own && P > 0);
        }
      }
      __syncthreads();
    }
    // 4. vertex plane cz is complete: store it and move the upper-face sums down
    if (P > 0) {
      const long o = ((long)cz * n + (y0 + lvy)) * n + (x0 + lvx);
      if constexpr (VEC) {
        // bfloat16 [vertex][16], channels 3 .. 15 zero: the closure's output gradient
        uint4* o16 = reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(dep) + o * 16);
        o16[0] = make_uint4((uint32_t)f2bf((float)lo4[0]) | ((uint32_t)f2bf((float)lo4[1]) << 16),
                            (uint32_t)f2bf((float)lo4[2]), 0u, 0u);
        o16[1] = make_uint4(0u, 0u, 0u, 0u);
      } else if (accumulate) {
        // a further species: its sums, weighted by its particle mass over the first species', are added
#pragma unroll
        for (int c = 0; c < N4; ++c) dep[c * n3 + o] = (T)((double)dep[c * n3 + o] + wd * lo4[c]);
#pragma unroll
        for (int c = 4; c < NC; ++c) dep[c * n3 + o] += w * lo6[c - 4];
      } else {
#pragma unroll
        for (int c = 0; c < N4; ++c) dep[c * n3 + o] = (T)lo4[c];
#pragma unroll
        for (int c = 4; c < NC; ++c) dep[c * n3 + o] = lo6[c - 4];
      }
    }
#pragma unroll
    for (int c = 0; c < N4; ++c) { lo4[c] = hi4[c]; hi4[c] = 0.0; }
#pragma unroll
    for (int c = 0; c < N6; ++c) { lo6[c] = hi6[c]; hi6[c] = (T)0; }
    __syncthreads();
    // 5. row offsets of plane P + 2; the cell offsets of plane P + 3 replace this plane's
    if (P + 2 <= zb) scan_rows(b2);
    if (P + 3 <= zb) store_raw(b, rnext);
  }
  if (esum) {
    // fixed-order reduction: within each wave, then the waves' sums in order
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) e_own += __shfl_down(e_own, d);
    if (lane == 0) red[wave] = e_own;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
#pragma unroll
      for (int w2 = 0; w2 < DEP_NT / 64; ++w2) t += red[w2];
      esum[(bz * gridDim.y + by) * gridDim.x + bx] = wd * t;
    }
  }
}

static int dep_zb(int n) {
  const long waves = (long)n * n / 64;  // of one layer of columns
  int zb = n < DEP_ZB ? n : DEP_ZB;
  while (zb > 1 && waves * (n / zb) < DEP_WAVES) zb /= 2;
  return zb;
}

int deposit_blocks(int n) {
  const int tx = dep_tx(n), ty = dep_nt(n) / tx;
  return (n / tx) * (n / ty) * (n / dep_zb(n));
}

template <typename T, int NC, bool REL, int TX, int NT>
static void launch_deposit_shape(const Particles<T>& p, const uint32_t* cell_start, int n, double a, double weight,
                                 bool accumulate, T* dep, double* esum_part, const float* vals, hipStream_t st) {
  const int zb = dep_zb(n);
  hipLaunchKernelGGL((deposit_kernel<T, NC, REL, TX, NT>), dim3(n / TX, n / (NT / TX), n / zb), dim3(NT), 0, st, p,
                     cell_start, n, zb, (T)a, a, (T)weight, weight, accumulate ? 1 : 0, dep, esum_part, vals);
}

template <typename T, int NC, bool REL>
static void launch_deposit_nc(const Particles<T>& p, const uint32_t* cell_start, int n, double a, double weight,
                              bool accumulate, T* dep, double* esum_part, const float* vals, hipStream_t st) {
  if (NC > 1 && dep_nt(n) == 128)
    launch_deposit_shape<T, NC, REL, 32, 128>(p, cell_start, n, a, weight, accumulate, dep, esum_part, vals, st);
  else if (dep_tx(n) == 32)
    launch_deposit_shape<T, NC, REL, 32, 256>(p, cell_start, n, a, weight, accumulate, dep, esum_part, vals, st);
  else
    launch_deposit_shape<T, NC, REL, 16, 256>(p, cell_start, n, a, weight, accumulate, dep, esum_part, vals, st);
}

template <typename T>
void launch_deposit(const Particles<T>& p, const uint32_t* cell_start, int n, int ncomp, bool relativistic, double a,
                    double weight, bool accumulate, T* dep, double* esum_part, hipStream_t st) {
  if (ncomp == 1)
    launch_deposit_nc<T, 1, false>(p, cell_start, n, a, weight, accumulate, dep, nullptr, nullptr, st);
  else if (relativistic)
    launch_deposit_nc<T, 10, true>(p, cell_start, n, a, weight, accumulate, dep, esum_part, nullptr, st);
  else
    launch_deposit_nc<T, 10, false>(p, cell_start, n, a, weight, accumulate, dep, esum_part, nullptr, st);
}

// Adjoint of the CIC gather of three fields: the sums over particles of W vals[id] as bfloat16
// [vertex][16], channels 3 .. 15 zero.  (By FP32 atomics into three fields and a conversion pass: 1.85 ms at 128^3 with crowded cells.)
template <typename T>
void launch_deposit_vectors(const Particles<T>& p, const uint32_t* cell_start, int n, const float* vals, uint16_t* out,
                            hipStream_t st) {
  launch_deposit_nc<T, 3, false>(p, cell_start, n, 0.0, 1.0, false, reinterpret_cast<T*>(out), nullptr, vals, st);
}

// ---------------------------------------------------------------------------
// gather + kick + drift + rank in the new cell.  A workgroup takes the particles of a
// TX x TY x TZ block of cells (TY*TZ contiguous row ranges of the sorted
// store) and first copies the fields it needs -- the block's vertices plus a
// margin of one below and two above, enough for the centred differences at
// the 8 corners of every cell -- into LDS.  Each particle then interpolates
// phi, chi, B and their centred-difference gradients from LDS (the CIC
// interpolation of the vertex gradients, written out per corner), kicks, drifts
// and takes its rank inside its new cell (the sort recomputes the cell from
// the stored position).
// ---------------------------------------------------------------------------
// Blocks are TX x TY x TZ cells with TX = 32 (16 on a 16^3 mesh): rows of 32 cells keep the
// row segments of the particle records at whole 128-byte lines more often.  FP32: 32x4x8
// cells (the field tile is 2.6 values per cell of the block) and 512 threads, or 256 with two
// fields or one where a block holds fewer than 512 particles on average (256^3 scalar with 128^3 particles: 0.179 ->
// 0.155 ms; with a particle per cell the kick gains 6 % too, but the sort that follows loses as much, its ranks being
// drawn in a more mixed order), on meshes large enough to fill the chip with them (64^3: 18 -> 24 us).
// Blocks of 2048 cells and 1024 threads (5.4 ms) or of 512 or 256 cells (4.97 - 5.15 ms) are slower.
// FP64: 32x2x4 cells and 256 threads: its registers allow 12 waves per CU, three such workgroups (measured at 512^3:
// 8.5 ms against 9.6 ms for 32x4x8 with 512 threads, whose 108 KB tile holds one per CU).
template <typename T> struct KdShape { static constexpr int TY = 4, TZ = 8, WPE = 4; };
template <> struct KdShape<double> { static constexpr int TY = 2, TZ = 4, WPE = 3; };
template <typename T, int TX> struct KdTile {
  static constexpr int GX = TX + 3, GY = KdShape<T>::TY + 3, GZ = KdShape<T>::TZ + 3, G = GX * GY * GZ;
};

// W fields of the tile side by side per vertex: one LDS read of up to 16 bytes brings all of them at an immediate
// offset from the particle's corner (field after field the FP32 kernel with five fields had 107 LDS reads and 126
// integer additions, now 60 and 49; kick at 512^3: 4.65 -> 4.03 ms on the grid, 4.85 -> 4.4 - 4.8 clustered; FP64 at
// 256^3 1.08 -> 0.98).
template <typename T, int W> struct alignas(W * sizeof(T)) FieldVec { T f[W]; };

// Values v and gradients g[c] of W fields at a particle.  f: the tile with x stride 1, y stride GX, z stride GX*GY, at the
// vertex one below the particle's cell in every axis
template <typename T, int W, int GX, int GY>
__device__ __forceinline__ void gather_lds(const FieldVec<T, W>* __restrict__ f, const T* wx, const T* wy, const T* wz,
                                           T half_n, T* v, T (*g)[3]) {
  // The order of the sums is that of the corners.  The outer vertices of a direction are asked for while the previous
  // ones are summed; the empty asm keeps the compiler from asking for all 32 vertices first (236 registers in FP32
  // where 128 let four waves share a SIMD).
  constexpr int SY = GX, SZ = GX * GY;
  FieldVec<T, W> in[2][2][2];  // the corners of the particle's cell
#pragma unroll
  for (int cz = 0; cz < 2; ++cz)
#pragma unroll
    for (int cy = 0; cy < 2; ++cy)
#pragma unroll
      for (int cx = 0; cx < 2; ++cx) in[cz][cy][cx] = f[(cz + 1) * SZ + (cy + 1) * SY + (cx + 1)];
#pragma unroll
  for (int c = 0; c < W; ++c) v[c] = g[c][0] = g[c][1] = g[c][2] = (T)0;
  FieldVec<T, W> out[2][2][2];
  auto load = [&](int k) {
    const int cz = k / 3, d = k % 3;
#pragma unroll
    for (int cy = 0; cy < 2; ++cy)
#pragma unroll
      for (int cx = 0; cx < 2; ++cx)
        out[k & 1][cy][cx] =
            f[(d == 2 ? 3 * cz : cz + 1) * SZ + (d == 1 ? 3 * cy : cy + 1) * SY + (d == 0 ? 3 * cx : cx + 1)];
  };
  load(0);
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const int cz = k / 3, d = k % 3;
    if (k < 5) load(k + 1);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int cy = 0; cy < 2; ++cy)
#pragma unroll
      for (int cx = 0; cx < 2; ++cx) {
        const T w = wx[cx] * wy[cy] * wz[cz];
        const bool up = d == 0 ? cx : (d == 1 ? cy : cz);
        const FieldVec<T, W> i = d == 0 ? in[cz][cy][1 - cx] : (d == 1 ? in[cz][1 - cy][cx] : in[1 - cz][cy][cx]);
        const FieldVec<T, W> o = out[k & 1][cy][cx];
#pragma unroll
        for (int c = 0; c < W; ++c) {
          if (d == 0) v[c] += w * in[cz][cy][cx].f[c];
          g[c][d] += w * (up ? o.f[c] - i.f[c] : i.f[c] - o.f[c]);
        }
      }
#pragma unroll
    for (int c = 0; c < W; ++c) asm volatile("" : "+v"(v[c]), "+v"(g[c][d]) : : "memory");
  }
#pragma unroll
  for (int c = 0; c < W; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) g[c][d] *= half_n;
}

// Rank of a particle among those that reach the same cell.  The store is
// sorted by cell and few particles change cell in a step, so equal keys mostly
// sit in consecutive lanes: each such run of the wave takes its slots with one
// atomicAdd of its length (one per run instead of one per particle, which
// serialises on the counter of a crowded cell).  Call with the active lanes in
// lockstep; every key gets a distinct rank in [0, final count of its cell).
__device__ __forceinline__ uint32_t rank_in_cell(uint32_t* cnt, uint32_t k) {
  const int lane = (int)__lane_id();
  const uint64_t act = __ballot(1);
  const uint32_t kp = __shfl_up(k, 1);
  const bool joins_prev = lane > 0 && ((act >> (lane - 1)) & 1ull) && kp == k;
  const uint64_t heads = __ballot(!joins_prev);
  const uint64_t upto = (2ull << lane) - 1ull;  // lanes 0 .. lane (all ones for lane 63)
  const int head = 63 - __clzll((long long)(heads & upto));
  const uint64_t after = (heads | ~act) & ~upto;  // run boundaries above this lane
  const int next = after ? __ffsll((long long)after) - 1 : 64;
  uint32_t base = 0;
  if (head == lane) base = atomicAdd(&cnt[k], (uint32_t)(next - head));
  base = __shfl(base, head);
  return base + (uint32_t)(lane - head);
}

template <typename T, int MODE, int TX, int KD_NT>
__global__ __launch_bounds__(KD_NT, KdShape<T>::WPE) void kick_drift_kernel(Particles<T> p,
                                                                    const uint32_t* __restrict__ cell_start, int n,
                                                                    GatherArgs<T> ga, uint32_t* rank, uint32_t* cnt,
                                                                    int* err) {
  constexpr int KD_TY = KdShape<T>::TY, KD_TZ = KdShape<T>::TZ;
  constexpr int NF = MODE == MODE_FULL ? 5 : (MODE == MODE_SCALAR ? 2 : 1);
  constexpr int NR = KD_TY * KD_TZ;                   // particle rows of the block
  constexpr int KD_GX = KdTile<T, TX>::GX, KD_GY = KdTile<T, TX>::GY, KD_G = KdTile<T, TX>::G;
  constexpr int NTL = (KD_G + KD_NT - 1) / KD_NT;     // tile entries per thread and field
  static_assert(NR <= 64, "row scan in one wave");
  // fields per vertex of the first tile, and of the others
  constexpr int WA = NF == 5 ? (sizeof(T) == 4 ? 4 : 2) : NF, WB = NF == 5 && sizeof(T) == 8 ? 2 : 0, WC = NF - WA - WB;
  __shared__ FieldVec<T, WA> tile_a[KD_G];
  __shared__ FieldVec<T, WB ? WB : 1> tile_b[WB ? KD_G : 1];
  __shared__ T tile_c[WC ? KD_G : 1];
  __shared__ uint32_t rbeg[NR], roff[NR + 1];
  const int m = n - 1;
  int bx, by, bz;
  xcd_block3(bx, by, bz);
  const int x0 = bx * TX, y0 = by * KD_TY, z0 = bz * KD_TZ;
  const int tid = threadIdx.x;
  const long nn = (long)n * n;
  // field tile with periodic wrap: local (gx, gy, gz) <-> global (x0 - 1 + gx, ...), x fastest;
  // every read of the thread is issued before the first is used
  const T* src[5] = {ga.phi, ga.chi, ga.bx, ga.by, ga.bz};
  T tv[NF][NTL];
#pragma unroll
  for (int k = 0; k < NTL; ++k) {
    const int q = tid + k * KD_NT;
    if (q < KD_G) {
      const int gx = q % KD_GX, row = q / KD_GX;
      const int gy = row % KD_GY, gz = row / KD_GY;
      const long o = (long)((z0 - 1 + gz) & m) * nn + (long)((y0 - 1 + gy) & m) * n + ((x0 - 1 + gx) & m);
#pragma unroll
      for (int f = 0; f < NF; ++f) tv[f][k] = src[f][o];
    }
  }
  // particle rows of the block: start of each row in the sorted store and the prefix of their lengths
  if (tid < 64) {
    uint32_t c = 0;
    if (tid < NR) {
      const int ly = tid % KD_TY, lz = tid / KD_TY;
      const long rb = ((long)(z0 + lz) * n + (y0 + ly)) * n;
      const uint32_t b = cell_start[rb + x0], e = cell_start[rb + x0 + TX];
      rbeg[tid] = b;
      c = e - b;
    }
    wave_row_offsets<NR>(c, roff);
  }
#pragma unroll
  for (int k = 0; k < NTL; ++k) {
    const int q = tid + k * KD_NT;
    if (q < KD_G) {
      FieldVec<T, WA> va;
#pragma unroll
      for (int f = 0; f < WA; ++f) va.f[f] = tv[f][k];
      tile_a[q] = va;
      if constexpr (WB > 0) {
        FieldVec<T, WB> vb;
#pragma unroll
        for (int f = 0; f < WB; ++f) vb.f[f] = tv[WA + f][k];
        tile_b[q] = vb;
      }
      if constexpr (WC > 0) tile_c[q] = tv[NF - 1][k];
    }
  }
  __syncthreads();
  const uint32_t total = roff[NR];
  const T hn = (T)(0.5 * n);
  const T dt = (T)ga.dtau;
  const T a = (T)ga.a, ah = (T)ga.a_half;
  // each thread takes particles tid, tid + KD_NT, ...; the next one's state is read while the
  // current one is processed
  uint32_t pin = 0;
  Loaded<T> next = {};
  auto load_next = [&](uint32_t i) {
    const int r = row_of<NR>(roff, i);
    pin = rbeg[r] + (i - roff[r]);
    load_raw_state(p, pin, next);
  };
  if ((uint32_t)tid < total) load_next(tid);
  for (uint32_t i = tid; i < total; i += KD_NT) {
    const uint32_t pi = pin;
    const Particle<T> now = unpacked(next);
    double x = now.x, y = now.y, z = now.z;
    T ux = now.ux, uy = now.uy, uz = now.uz;
    if (i + KD_NT < total) load_next(i + KD_NT);
    int ix, iy, iz;
    double fxd, fyd, fzd;
    cell_of(x, n, ix, fxd);
    cell_of(y, n, iy, fyd);
    cell_of(z, n, iz, fzd);
    const T wx[2] = {(T)1 - (T)fxd, (T)fxd}, wy[2] = {(T)1 - (T)fyd, (T)fyd}, wz[2] = {(T)1 - (T)fzd, (T)fzd};
    const int lx = ix - x0, ly = iy - y0, lz = iz - z0;  // in [0, T*) by construction of the rows
    const int corner = (lz * KD_GY + ly) * KD_GX + lx;
    T fv[NF], gf[NF][3];
    gather_lds<T, WA, KD_GX, KD_GY>(tile_a + corner, wx, wy, wz, hn, fv, gf);
    if constexpr (WB > 0) gather_lds<T, WB, KD_GX, KD_GY>(tile_b + corner, wx, wy, wz, hn, fv + WA, gf + WA);
    if constexpr (WC > 0)
      gather_lds<T, 1, KD_GX, KD_GY>(reinterpret_cast<const FieldVec<T, 1>*>(tile_c) + corner, wx, wy, wz, hn, fv + NF - 1,
                                     gf + NF - 1);
    const T phi_p = fv[0];
    T* gphi = gf[0];
    if (ga.corr) {
      // learned closure: CIC-interpolated correction to grad phi
      const long n3 = nn * n;
      const int xs[2] = {ix, (ix + 1) & m}, ys[2] = {iy, (iy + 1) & m}, zs[2] = {iz, (iz + 1) & m};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float* g = ga.corr + c * n3;
        T acc = 0;
#pragma unroll
        for (int a2 = 0; a2 < 2; ++a2)
#pragma unroll
          for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
            for (int d2 = 0; d2 < 2; ++d2)
              acc += wz[a2] * wy[b2] * wx[d2] * (T)g[zs[a2] * nn + (long)ys[b2] * n + xs[d2]];
        gphi[c] += acc;
      }
    }
    T vx, vy, vz;
    if constexpr (MODE == MODE_NEWTONIAN) {
      ux -= dt * a * gphi[0];
      uy -= dt * a * gphi[1];
      uz -= dt * a * gphi[2];
      const T ia = rcp(ah);
      vx = ux * ia; vy = uy * ia; vz = uz * ia;
    } else {
      const T chi_p = fv[1];
      const T* gchi = gf[1];
      // (the roundings of the squares are written out: which products the compiler fuses otherwise depends on how the
      // momentum was loaded, and a hot particle's last bits with it)
      const T u2 = fma(uz, uz, fma(uy, uy, ux * ux));
      const T ie = rsqrt_(a * a + u2);
      const T e = (a * a + u2) * ie;
      const T cphi = -(a * a + (T)2 * u2) * ie;
      T fx = cphi * gphi[0] + e * gchi[0];
      T fy = cphi * gphi[1] + e * gchi[1];
      T fz = cphi * gphi[2] + e * gchi[2];
      T B[3] = {0, 0, 0};
      if constexpr (MODE == MODE_FULL) {
        const T(*gb)[3] = gf + 2;  // gb[j][i] = d_i B_j
        B[0] = fv[2]; B[1] = fv[3]; B[2] = fv[4];
        fx -= ux * gb[0][0] + uy * gb[1][0] + uz * gb[2][0];
        fy -= ux * gb[0][1] + uy * gb[1][1] + uz * gb[2][1];
        fz -= ux * gb[0][2] + uy * gb[1][2] + uz * gb[2][2];
      }
      ux += dt * fx;
      uy += dt * fy;
      uz += dt * fz;
      const T v2 = fma(uz, uz, fma(ux, ux, uy * uy));
      const T eh2 = ah * ah + v2;
      const T ieh = rsqrt_(eh2);
      const T fac = ((T)1 + ((T)3 - v2 * ieh * ieh) * phi_p - chi_p) * ieh;
      vx = ux * fac + B[0];
      vy = uy * fac + B[1];
      vz = uz * fac + B[2];
    }
    x += ga.dtau * (double)vx;
    y += ga.dtau * (double)vy;
    z += ga.dtau * (double)vz;
    if (!(isfinite(x) && isfinite(y) && isfinite(z))) {
      atomicOr(err, 1);
      x = y = z = 0.0;
    }
    x = wrap01(x); y = wrap01(y); z = wrap01(z);
    store_state(p, pi, Particle<T>{x, y, z, ux, uy, uz, 0u});
    rank[pi] = rank_in_cell(cnt, cell_key(x, y, z, n));
  }
}

template <typename T, int TX, int NT, int NT_FULL>
static void launch_kick_drift_tx(const Particles<T>& p, int n, const uint32_t* cell_start, const GatherArgs<T>& g,
                                 uint32_t* rank, uint32_t* cnt, int* err, hipStream_t st) {
  dim3 grid(n / TX, n / KdShape<T>::TY, n / KdShape<T>::TZ);
  if (g.mode == MODE_NEWTONIAN)
    hipLaunchKernelGGL((kick_drift_kernel<T, MODE_NEWTONIAN, TX, NT>), grid, dim3(NT), 0, st, p, cell_start, n, g, rank,
                       cnt, err);
  else if (g.mode == MODE_SCALAR)
    hipLaunchKernelGGL((kick_drift_kernel<T, MODE_SCALAR, TX, NT>), grid, dim3(NT), 0, st, p, cell_start, n, g, rank,
                       cnt, err);
  else
    hipLaunchKernelGGL((kick_drift_kernel<T, MODE_FULL, TX, NT_FULL>), grid, dim3(NT_FULL), 0, st, p, cell_start, n, g,
                       rank, cnt, err);
}

template <typename T>
void launch_kick_drift(const Particles<T>& p, long np, int n, const uint32_t* cell_start, const GatherArgs<T>& g,
                       uint32_t* rank, uint32_t* cnt, int* err, hipStream_t st) {
  constexpr int NT = sizeof(T) == 4 ? 512 : 256;
  if (n >= 128 && 2 * np <= (long)n * n * n)
    launch_kick_drift_tx<T, 32, 256, NT>(p, n, cell_start, g, rank, cnt, err, st);
  else if (n >= 32)
    launch_kick_drift_tx<T, 32, NT, NT>(p, n, cell_start, g, rank, cnt, err, st);
  else
    launch_kick_drift_tx<T, 16, NT, NT>(p, n, cell_start, g, rank, cnt, err, st);
}

// ---------------------------------------------------------------------------
// exclusive scan of the per-cell counts -> cell_start (n^3 + 1 entries);
// the counts are reset to zero for the next histogram (by the scan or by the scatter that follows it).
// ---------------------------------------------------------------------------
constexpr int SCAN_NT = 256, SCAN_PER = 16, SCAN_CHUNK = SCAN_NT * SCAN_PER;

size_t scan_block_sums_count(long ncell) { return (size_t)((ncell + SCAN_CHUNK - 1) / SCAN_CHUNK); }

// block sums; the order inside a block does not matter, so loads are striped (coalesced)
__global__ __launch_bounds__(SCAN_NT) void scan_reduce_kernel(const uint32_t* cnt, long ncell, uint32_t* bsum) {
  __shared__ uint32_t red[SCAN_NT];
  const long base = (long)blockIdx.x * SCAN_CHUNK + threadIdx.x;
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < SCAN_PER; ++j) {
    const long i = base + (long)j * SCAN_NT;
    if (i < ncell) s += cnt[i];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = SCAN_NT / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}

// single workgroup: exclusive scan of the block sums in place
__global__ __launch_bounds__(1024) void scan_blocks_kernel(uint32_t* bsum, long nb) {
  __shared__ uint32_t part[1024];
  const long per = (nb + 1023) / 1024;
  const long b0 = threadIdx.x * per;
  uint32_t s = 0;
  for (long j = 0; j < per; ++j)
    if (b0 + j < nb) s += bsum[b0 + j];
  part[threadIdx.x] = s;
  __syncthreads();
  // Hillis-Steele inclusive scan of the 1024 partial sums
  for (int off = 1; off < 1024; off <<= 1) {
    const uint32_t v = (threadIdx.x >= (unsigned)off) ? part[threadIdx.x - off] : 0u;
    __syncthreads();
    part[threadIdx.x] += v;
    __syncthreads();
  }
  uint32_t run = (threadIdx.x == 0) ? 0u : part[threadIdx.x - 1];
  for (long j = 0; j < per; ++j) {
    if (b0 + j < nb) {
      const uint32_t v = bsum[b0 + j];
      bsum[b0 + j] = run;
      run += v;
    }
  }
}

// Where the chunk's offset comes from: the scanned block sums, the block sums before it (added up here, one launch
// less), or the counts before it themselves (two launches less; the counts are then reset by the scatter, after
// every chunk has read them).
enum { SCAN_OFFSETS = 0, SCAN_SUMS = 1, SCAN_COUNTS = 2 };

// exclusive scan of one chunk: striped coalesced loads into LDS, per-thread scan of 16
// consecutive values (padded LDS rows), block scan of the thread totals, striped stores
template <int FROM>
__global__ __launch_bounds__(SCAN_NT) void scan_apply_kernel(uint32_t* cnt, long ncell, const uint32_t* boff,
                                                             uint32_t* cell_start) {
  constexpr int PAD = SCAN_PER + 1;
  __shared__ uint32_t buf[SCAN_NT * PAD];
  __shared__ uint32_t part[SCAN_NT / 64], before[SCAN_NT / 64];
  const long base = (long)blockIdx.x * SCAN_CHUNK;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  uint32_t pre = 0;
  if constexpr (FROM == SCAN_SUMS) {
    for (int i = t; i < (int)blockIdx.x; i += SCAN_NT) pre += boff[i];
  } else if constexpr (FROM == SCAN_COUNTS) {
    const uint4* c4 = reinterpret_cast<const uint4*>(cnt);  // whole chunks, 16-byte aligned
#pragma unroll 4
    for (int i = t; i < (int)base / 4; i += SCAN_NT) {
      const uint4 v = c4[i];
      pre += v.x + v.y + v.z + v.w;
    }
  }
#pragma unroll
  for (int j = 0; j < SCAN_PER; ++j) {
    const int q = t + j * SCAN_NT;  // element of the chunk
    const long i = base + q;
    buf[(q / SCAN_PER) * PAD + q % SCAN_PER] = (i < ncell) ? cnt[i] : 0u;
    if (FROM != SCAN_COUNTS && i < ncell) cnt[i] = 0u;
  }
  __syncthreads();
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < SCAN_PER; ++j) s += buf[t * PAD + j];
  // inclusive scan of the thread totals within the wave, then the waves' totals in order
  uint32_t inc = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t v = __shfl_up(inc, d);
    if (lane >= d) inc += v;
  }
  if (lane == 63) part[wave] = inc;
  if constexpr (FROM != SCAN_OFFSETS) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) pre += __shfl_down(pre, d);
    if (lane == 0) before[wave] = pre;
  }
  __syncthreads();
  uint32_t run = inc - s, total = 0, first = FROM == SCAN_OFFSETS ? boff[blockIdx.x] : 0u;
#pragma unroll
  for (int w = 0; w < SCAN_NT / 64; ++w) {
    if (w < wave) run += part[w];
    total += part[w];
    if (FROM != SCAN_OFFSETS) first += before[w];
  }
  run += first;
#pragma unroll
  for (int j = 0; j < SCAN_PER; ++j) {
    const uint32_t v = buf[t * PAD + j];
    buf[t * PAD + j] = run;
    run += v;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < SCAN_PER; ++j) {
    const int q = t + j * SCAN_NT;
    const long i = base + q;
    if (i < ncell) cell_start[i] = buf[(q / SCAN_PER) * PAD + q % SCAN_PER];
  }
  // the last block also writes the total at cell_start[ncell]
  if (base + SCAN_CHUNK >= ncell && t == 0) cell_start[ncell] = first + total;
}

// The lines of the rule: 32^3 (8 chunks, one launch of 6 us for three of 6 + 3 + 6), 256^3 (4096 chunks: adding up
// the block sums costs 2 us, the launch between cost 4); at 512^3 every chunk would read 128 KB of block sums.
static bool scan_from_counts(long ncell) { return scan_block_sums_count(ncell) <= 8; }

void launch_scan(uint32_t* cnt, uint32_t* cell_start, long ncell, uint32_t* block_sums, hipStream_t st) {
  const long nb = (long)scan_block_sums_count(ncell);
  const dim3 grid((unsigned)nb), block(SCAN_NT);
  if (scan_from_counts(ncell)) {
    hipLaunchKernelGGL(scan_apply_kernel<SCAN_COUNTS>, grid, block, 0, st, cnt, ncell, block_sums, cell_start);
    return;
  }
  hipLaunchKernelGGL(scan_reduce_kernel, grid, block, 0, st, cnt, ncell, block_sums);
  if (nb <= 4096) {
    hipLaunchKernelGGL(scan_apply_kernel<SCAN_SUMS>, grid, block, 0, st, cnt, ncell, block_sums, cell_start);
    return;
  }
  hipLaunchKernelGGL(scan_blocks_kernel, dim3(1), dim3(1024), 0, st, block_sums, nb);
  hipLaunchKernelGGL(scan_apply_kernel<SCAN_OFFSETS>, grid, block, 0, st, cnt, ncell, block_sums, cell_start);
}

// ---------------------------------------------------------------------------
// scatter into the other buffer at cell_start[cell] + rank; the cell is
// recomputed from the stored position exactly as the kick/drift computed it.
// Bound by the scattered stores, 16 + 16 + 4 + 4 bytes apart by particles that left their neighbours
// (512^3 FP32: 3.3 ms for 84 bytes each, 3.4 TB/s; a stream of the same bytes takes 2.6).
// One particle per thread: two or four in flight gain nothing (3.92, 4.07 and 4.11 ms).
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void scatter_kernel(Particles<T> s, Particles<T> d, long np, int nmesh,
                                                      const uint32_t* __restrict__ rank,
                                                      const uint32_t* __restrict__ cell_start, uint32_t* cnt,
                                                      int nreset) {
  // counts left standing by the scan
  for (int c = (int)(blockIdx.x * 256 + threadIdx.x); c < nreset; c += (int)(gridDim.x * 256)) cnt[c] = 0u;
  const long i = (long)xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (i >= np) return;
  const uint32_t r = rank[i];
  Particle<T> v;
  load_particle(s, i, v);
  store_particle(d, (long)cell_start[cell_key(v.x, v.y, v.z, nmesh)] + r, v);
}

template <typename T>
void launch_scatter(const Particles<T>& src, Particles<T> dst, long np, int nmesh, const uint32_t* rank,
                    const uint32_t* cell_start, uint32_t* cnt, hipStream_t st) {
  const long ncell = (long)nmesh * nmesh * nmesh;
  const int nreset = scan_from_counts(ncell) ? (int)ncell : 0;
  hipLaunchKernelGGL((scatter_kernel<T>), dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, src, dst,
                     np, nmesh, rank, cell_start, cnt, nreset);
}

// ---------------------------------------------------------------------------
// deterministic order inside each cell: after the counting sort the particles of
// a cell sit in the order in which atomic counters handed out their ranks; this
// pass moves each particle to cell_start[cell] + (number of particles of its cell
// with a smaller identifier), so the store -- and every sum over it -- no longer
// depends on that order (identifiers are unique)
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void order_by_id_kernel(Particles<T> s, Particles<T> d, long np, int nmesh,
                                                          const uint32_t* __restrict__ cell_start) {
  const long i = (long)xcd_remap(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (i >= np) return;
  Particle<T> v;
  load_particle(s, i, v);
  const uint32_t k = cell_key(v.x, v.y, v.z, nmesh);
  const uint32_t b = cell_start[k], e = cell_start[k + 1];
  uint32_t r = 0;
  for (uint32_t j = b; j < e; ++j) r += load_id(s, j) < v.id ? 1u : 0u;
  store_particle(d, (long)b + r, v);
}

template <typename T>
void launch_order_by_id(const Particles<T>& src, Particles<T> dst, long np, int nmesh, const uint32_t* cell_start,
                        hipStream_t st) {
  hipLaunchKernelGGL((order_by_id_kernel<T>), dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, src, dst, np, nmesh,
                     cell_start);
}

// ---------------------------------------------------------------------------
// consistency check of a restored store (checkpoint bodies are not trusted):
// cell_start[0] = 0, cell_start[n^3] = np, non-decreasing; every particle has
// finite momenta, a position in [0, 1), an identifier < np, and sits inside the
// range of the cell its position falls in.  Any failure sets bit 4 of err.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void check_offsets_kernel(const uint32_t* cell_start, long ncell, long np, int* err) {
  const long c = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c > ncell) return;
  bool bad = false;
  if (c == 0) bad = cell_start[0] != 0u;
  if (c == ncell) bad = bad || (long)cell_start[ncell] != np;
  if (c < ncell) bad = bad || cell_start[c] > cell_start[c + 1];
  if (bad) atomicOr(err, 4);
}

template <typename T>
__global__ __launch_bounds__(256) void check_store_kernel(Particles<T> p, long np, int nmesh,
                                                          const uint32_t* cell_start, int* err) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  Particle<T> v;
  load_particle(p, i, v);
  const double x = v.x, y = v.y, z = v.z;
  bool ok = isfinite(v.ux) && isfinite(v.uy) && isfinite(v.uz);
  ok = ok && x >= 0.0 && x < 1.0 && y >= 0.0 && y < 1.0 && z >= 0.0 && z < 1.0;  // false for NaN
  ok = ok && (long)v.id < np;
  if (ok) {
    const uint32_t k = cell_key(x, y, z, nmesh);
    ok = (long)cell_start[k] <= i && i < (long)cell_start[k + 1];
  }
  if (!ok) atomicOr(err, 4);
}

template <typename T>
void launch_check_store(const Particles<T>& p, long np, int nmesh, const uint32_t* cell_start, int* err,
                        hipStream_t st) {
  const long ncell = (long)nmesh * nmesh * nmesh;
  hipLaunchKernelGGL(check_offsets_kernel, dim3((unsigned)((ncell + 1 + 255) / 256)), dim3(256), 0, st, cell_start,
                     ncell, np, err);
  hipLaunchKernelGGL((check_store_kernel<T>), dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, p, np, nmesh,
                     cell_start, err);
}

// ---------------------------------------------------------------------------
// the store as separate arrays and back (checkpoints)
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void unpack_kernel(Particles<T> p, long n, double* pos, T* mom, uint32_t* ids, long gap) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  const long sp = n + gap / (long)sizeof(double), sm = n + gap / (long)sizeof(T);
  if (i < gap / (long)sizeof(T)) {
    mom[n + i] = mom[sm + n + i] = (T)0;
    if (i < gap / (long)sizeof(double)) pos[n + i] = pos[sp + n + i] = 0.0;
  }
  if (i >= n) return;
  Particle<T> v;
  load_particle(p, i, v);
  pos[i] = v.x; pos[sp + i] = v.y; pos[2 * sp + i] = v.z;
  mom[i] = v.ux; mom[sm + i] = v.uy; mom[2 * sm + i] = v.uz;
  ids[i] = v.id;
}

template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(const double* pos, const T* mom, const uint32_t* ids, long n, long gap,
                                                   Particles<T> p) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const long sp = n + gap / (long)sizeof(double), sm = n + gap / (long)sizeof(T);
  store_particle(p, i, Particle<T>{pos[i], pos[sp + i], pos[2 * sp + i], mom[i], mom[sm + i], mom[2 * sm + i], ids[i]});
}

template <typename T>
void launch_unpack(const Particles<T>& p, long n, double* pos, T* mom, uint32_t* ids, long gap, hipStream_t st) {
  const long m = n > gap ? n : gap;
  hipLaunchKernelGGL((unpack_kernel<T>), dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, p, n, pos, mom, ids, gap);
}

template <typename T>
void launch_pack(const double* pos, const T* mom, const uint32_t* ids, long n, long gap, const Particles<T>& p,
                 hipStream_t st) {
  hipLaunchKernelGGL((pack_kernel<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, pos, mom, ids, n, gap, p);
}

// ---------------------------------------------------------------------------
// export in identifier order as [n][3] arrays
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void export_kernel(Particles<T> p, long np, double* pos, T* u, uint32_t* ids) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  Particle<T> v;
  load_particle(p, i, v);
  const long d = v.id;
  if (pos) *reinterpret_cast<V3<double>*>(pos + 3 * d) = V3<double>{v.x, v.y, v.z};
  if (u) *reinterpret_cast<V3<T>*>(u + 3 * d) = V3<T>{v.ux, v.uy, v.uz};
  if (ids) ids[d] = (uint32_t)d;
}

template <typename T>
void launch_export(const Particles<T>& p, long np, double* pos_aos, T* u_aos, uint32_t* ids, hipStream_t st) {
  hipLaunchKernelGGL((export_kernel<T>), dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, p, np, pos_aos, u_aos,
                     ids);
}

// ---------------------------------------------------------------------------
// FP64 sums of the three momentum components (diagnostics): the records that hold them read once, block after block of
// the store and the blocks' sums in order.  Bound by its bytes (512^3 FP32: 2.7 GB, pm_diagnostics 0.55 ms; with three
// passes over single components 1.68 ms, and 1.37 when they were arrays of their own).
// ---------------------------------------------------------------------------
constexpr int MOM_BLOCKS = MOMENTUM_SCRATCH / 3;

// the sums of the workgroup's 256 threads in thread 0, in a fixed order
__device__ __forceinline__ void block_sum3(double* s) {
  __shared__ double red[3][4];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) s[d] += __shfl_down(s[d], w);
    if ((threadIdx.x & 63) == 0) red[d][threadIdx.x >> 6] = s[d];
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < 3; ++d) s[d] = ((red[d][0] + red[d][1]) + red[d][2]) + red[d][3];
}

template <typename T>
__global__ __launch_bounds__(256) void momentum_partial_kernel(Particles<T> p, long np, double* __restrict__ part) {
  const long per = (np + gridDim.x - 1) / gridDim.x;
  const long b = (long)blockIdx.x * per, e = min(np, b + per);
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll 4
  for (long i = b + threadIdx.x; i < e; i += 256) {
    if constexpr (sizeof(T) == 4) {
      s[0] += (double)p.b[i].ux; s[1] += (double)p.b[i].uy; s[2] += (double)p.c[i].uz;
    } else {
      s[0] += p.b[i].ux; s[1] += p.c[i].uy; s[2] += p.c[i].uz;
    }
  }
  block_sum3(s);
  if (threadIdx.x == 0)
    for (int d = 0; d < 3; ++d) part[d * gridDim.x + blockIdx.x] = s[d];
}

__global__ __launch_bounds__(256) void momentum_final_kernel(const double* __restrict__ part, int nb, double* out) {
  double s[3] = {0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < nb; i += 256)
    for (int d = 0; d < 3; ++d) s[d] += part[d * nb + i];
  block_sum3(s);
  if (threadIdx.x == 0)
    for (int d = 0; d < 3; ++d) out[d] = s[d];
}

template <typename T>
void launch_sum_momentum(const Particles<T>& p, long np, double* out, double* scratch, hipStream_t st) {
  const int nb = (int)min((long)MOM_BLOCKS, (np + 1023) / 1024);
  hipLaunchKernelGGL((momentum_partial_kernel<T>), dim3(nb), dim3(256), 0, st, p, np, scratch);
  hipLaunchKernelGGL(momentum_final_kernel, dim3(1), dim3(256), 0, st, scratch, nb, out);
}

#define GPM_INST(T)                                                                                                   \
  template void launch_ingest<T>(const double*, const T*, const uint32_t*, long, Particles<T>, int, uint32_t*,         \
                                 uint32_t*, int*, hipStream_t);                                                        \
  template void launch_deposit<T>(const Particles<T>&, const uint32_t*, int, int, bool, double, double, bool, T*,     \
                                  double*, hipStream_t);                                                              \
  template void launch_kick_drift<T>(const Particles<T>&, long, int, const uint32_t*, const GatherArgs<T>&, uint32_t*, \
                                     uint32_t*, int*, hipStream_t);                                                    \
  template void launch_scatter<T>(const Particles<T>&, Particles<T>, long, int, const uint32_t*, const uint32_t*,      \
                                  uint32_t*, hipStream_t);                                                                        \
  template void launch_unpack<T>(const Particles<T>&, long, double*, T*, uint32_t*, long, hipStream_t);               \
  template void launch_pack<T>(const double*, const T*, const uint32_t*, long, long, const Particles<T>&, hipStream_t); \
  template void launch_deposit_vectors<T>(const Particles<T>&, const uint32_t*, int, const float*, uint16_t*,         \
                                          hipStream_t);                                                               \
  template void launch_export<T>(const Particles<T>&, long, double*, T*, uint32_t*, hipStream_t);                      \
  template void launch_sum_momentum<T>(const Particles<T>&, long, double*, double*, hipStream_t);                     \
  template void launch_check_store<T>(const Particles<T>&, long, int, const uint32_t*, int*, hipStream_t);            \
  template void launch_order_by_id<T>(const Particles<T>&, Particles<T>, long, int, const uint32_t*, hipStream_t);
GPM_INST(float)
GPM_INST(double)

}  // namespace gpm
