// Reciprocal-space sums over the MM charges on a regular mesh.
//
// The two sums of the long-range part that run over every (k, MM charge) pair,
//   S_MM(k) = sum_i q_i e^{i k.R_i}              (structure factor)
//   V(R_i)  = Re sum_k W(k) e^{-i k.R_i}, grad V (potential of the QM multipoles)
// (paper: SI, multipolar Ewald, long-range tensors) are nonuniform discrete
// Fourier transforms of types 1 and 2.  Evaluated densely they cost 4 and 8
// flops per (k, charge), 12 (2m+1)^3/2 per charge: 0.7 Mflop at |n| <= 24.
// Here each charge is spread to 16^3 mesh points with a separable compact
// kernel, the mesh is transformed to the wanted k with three small dense
// contractions, one per axis, and the kernel's own transform is divided out
// (folded into the contraction tables); the adjoint runs the same steps
// backwards and reads each charge's 16^3 points with the kernel and its
// derivative.  The method is the nonuniform FFT of Dutt and Rokhlin with the
// Kaiser-Bessel kernel (Jackson et al. 1991; error analysis in Barnett,
// Magland and af Klinteberg 2019).
//
// Precision: kernel width w = 16 points and beta = 42.5.  A wave number n = u N
// is contaminated by its alias at N - n, relative to itself by
//   exp(-[S(u) - S(1 - u)]),  S(v) = sqrt(max(0, beta^2 - (pi w v)^2)),
// below 1e-17 for u < 0.15 (the gradient needs beta this large: the kernel's
// derivative jumps by beta^2 / (2 I0(beta)) at the edge of the support) and
// rising towards the band edge, where the Ewald weight
// exp(-k^2 / 4 alpha^2) = exp(-A (n/m)^2), A = (pi m / (alpha L))^2, outweighs
// it.  N is chosen so that the product stays below 1e-14 at the worst n
// (mesh_damping gives the smallest A for which it does); a call with less
// damping takes the dense sums.  Few wave numbers come near that one, and the
// outputs' errors stay those of the dense sums, 4e-16 to 1e-14: they are the same
// to a digit with 1e-16 (a fifth more points per axis), while 7e-13 at the worst n
// raises the MM gradient's from 5e-16 to 2e-14 (35 000 charges at kmax 24).
// Everything is FP64.
//
// Measured against the dense sums (both directions, kernels alone): 16 frames of
// 100 000 charges at kmax 32 41 ms dense, 3.4 ms here (meshes of 96^3); 64 frames of 5000
// to 30 000 at kmax 20 8.3 and 2.4 ms (64^3); one frame of 35 000 at kmax 24 440 and
// 150 us (80^3).
//
// The charges are taken to be spread over the box.  Where many share a few
// tiles the time is that of the fullest ones: 35 000 charges all within 20 A of one point
// of a 70 A box take 1.5 times as long as dense sums.
//
// Real basis.  The mesh is real, so every contraction runs over the real
// functions cos(2 pi n x/L), n = 0..m, and sin(2 pi n x/L), n = 1..m of each
// axis (index n for cos, m + n for sin; padded to a multiple of 16 with zero
// rows).  T[a][b][c] = sum over the mesh of the product of basis functions a
// (x), b (y), c (z), and the four k = (nx, +-ny, +-nz) of the half space are
// sums of eight T.
#include <math.h>

#include <algorithm>
#include <vector>

#include "ewald_internal.h"
#include "lanes.h"

namespace mpe {

#define DEV __device__ __forceinline__

static constexpr double kPiM = 3.14159265358979323846;

typedef double v4d __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4f64: D(16x16) += A(16x4) B(4x16).  A[i][k] sits in lane
// i + 16k, B[k][j] in lane j + 16k, and element r of D in lane l is D[l/16 + 4r][l%16].
DEV v4d mfma(double a, double b, v4d c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

DEV int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// What the mesh kernels need of a frame, through the scalar cache (the
// descriptors do not change while a kernel runs).
struct MeshFrame {
  double box[3], inv_box[3];
  int nm, moff;
};

DEV MeshFrame mesh_frame(const FrameArg& fa, int f) {
  typedef const __attribute__((address_space(4))) FrameDev ConstFrame;
  MeshFrame r;
  if (fa.frames) {
    ConstFrame* p = (ConstFrame*)(uintptr_t)fa.frames + f;
    for (int a = 0; a < 3; a++) {
      r.box[a] = p->box[a];
      r.inv_box[a] = p->inv_box[a];
    }
    r.nm = p->nm;
    r.moff = p->moff;
  } else {
    for (int a = 0; a < 3; a++) {
      r.box[a] = fa.f0.box[a];
      r.inv_box[a] = fa.f0.inv_box[a];
    }
    r.nm = fa.f0.nm;
    r.moff = fa.f0.moff;
  }
  return r;
}

DEV void lds_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Consecutive blocks go to the 8 XCDs in turn; give each XCD a contiguous run
// of work items instead, so that neighbouring tiles share its L2.
DEV int xcd_order(int bid, int n) {
  const int per = n / 8;
  return bid < 8 * per ? (bid & 7) * per + (bid >> 3) : bid;
}

// Mesh cell i in [0, N) and offset t in [0, 1) of a wrapped coordinate x in
// [0, L): x N / L = i + t, t to an absolute 1e-16 (the division's remainder
// is added back).  A NaN coordinate lands in cell 0 with t = NaN.
DEV void mesh_cell(double x, double L, int N, int& i, double& t) {
  const double f = x / L, r = fma(-f, L, x) / L;
  const double u = f * (double)N;
  i = u >= 0.0 ? (u < (double)(N - 1) ? (int)u : N - 1) : 0;
  t = fma(f, (double)N, -(double)i) + (double)N * r;
}

// ------------------------------------------------------------------ counting sort into bins of 4^3 mesh cells
// Bin index with x fastest, so that the bins of a row of neighbouring x are
// contiguous in the sorted order.
DEV int mesh_bin(const Mesh& m, int ix, int iy, int iz) { return ((iz >> 2) * m.nb[1] + (iy >> 2)) * m.nb[0] + (ix >> 2); }

// one atom per thread: its bin, and its rank among the bin's atoms (arrival order)
__global__ __launch_bounds__(256) void k_mesh_count(Mesh m, FrameArg fa, const double* __restrict__ mm4, int cap_mm,
                                                    int* __restrict__ cnt, int2* __restrict__ slot) {
  const int f = blockIdx.y;
  const MeshFrame fr = mesh_frame(fa, f);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= fr.nm) return;
  const int row = fr.moff + i;
  int c[3];
  double t;
  for (int a = 0; a < 3; a++) mesh_cell(mm4[(size_t)a * cap_mm + row], fr.box[a], m.N[a], c[a], t);
  const int bin = mesh_bin(m, c[0], c[1], c[2]);
  slot[row] = make_int2(bin, atomicAdd(&cnt[(size_t)f * m.nbt + bin], 1));
}

// one block per frame: exclusive scan of the bin counts (nbt + 1 entries); the
// counts are cleared for the next call
__global__ __launch_bounds__(1024) void k_mesh_scan(Mesh m, int* __restrict__ cnt, int* __restrict__ start) {
  __shared__ int part[16];
  int* __restrict__ c = cnt + (size_t)blockIdx.x * m.nbt;
  int* __restrict__ st = start + (size_t)blockIdx.x * (m.nbt + 1);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int carry = 0;
  for (int base = 0; base < m.nbt; base += 4096) {  // nbt is a multiple of 4: four bins per thread and round
    const int b = base + 4 * tid;
    int4 v = make_int4(0, 0, 0, 0);
    if (b < m.nbt) {
      v = *(const int4*)(c + b);
      *(int4*)(c + b) = make_int4(0, 0, 0, 0);
    }
    const int s = v.x + v.y + v.z + v.w;
    int inc = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(inc, o, 64);
      if (lane >= o) inc += u;
    }
    if (lane == 63) part[wave] = inc;
    __syncthreads();
    int off = carry;
#pragma unroll
    for (int k = 0; k < 16; k++) {
      const int pk = part[k];
      if (k < wave) off += pk;
      carry += pk;
    }
    const int e = off + inc - s;
    if (b < m.nbt) {
      st[b] = e;
      st[b + 1] = e + v.x;
      st[b + 2] = e + v.x + v.y;
      st[b + 3] = e + v.x + v.y + v.z;
    }
    __syncthreads();  // part is reused
  }
  if (tid == 0) st[m.nbt] = carry;
}

// Deterministic plans: the arrival order of a bin's atoms depends on the
// atomics, so the bin's members are listed first and each atom's rank becomes
// the number of members with a lower index.
__global__ __launch_bounds__(256) void k_mesh_list(Mesh m, FrameArg fa, const int* __restrict__ start,
                                                   const int2* __restrict__ slot, int* __restrict__ perm) {
  const int f = blockIdx.y;
  const MeshFrame fr = mesh_frame(fa, f);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= fr.nm) return;
  const int2 s = slot[fr.moff + i];
  perm[fr.moff + start[(size_t)f * (m.nbt + 1) + s.x] + s.y] = i;
}

__global__ __launch_bounds__(256) void k_mesh_rank(Mesh m, FrameArg fa, const int* __restrict__ start,
                                                   const int* __restrict__ perm, int2* __restrict__ slot) {
  const int f = blockIdx.y;
  const MeshFrame fr = mesh_frame(fa, f);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= fr.nm) return;
  const int bin = slot[fr.moff + i].x;
  const int* st = start + (size_t)f * (m.nbt + 1) + bin;
  int rank = 0;
  for (int p = st[0]; p < st[1]; p++) rank += perm[fr.moff + p] < i ? 1 : 0;
  slot[fr.moff + i].y = rank;
}

// Sorted records: the kernel values of the atom's 16 mesh points per axis
// (taps, one axis per blockIdx.z; the x ones times its charge), its cell and
// row, and its offsets.  Tap j of an axis, at mesh point i - 7 + j, is a
// polynomial of degree 19 in s = 2t - 1 whose even and odd parts
// E(s^2) + s O(s^2) also give tap 15 - j (the kernel is even).  The taps go through
// LDS, so that eight lanes write an atom's 128 bytes of an axis (16 frames of 100 000 charges
// 266 us with a thread per atom writing them, 204 so, 3.4 TB/s).
__global__ __launch_bounds__(256) void k_mesh_sort(Mesh m, FrameArg fa, const double* __restrict__ mm4, int cap_mm,
                                                   const int* __restrict__ start, const int2* __restrict__ slot,
                                                   const double* __restrict__ poly, double* __restrict__ taps,
                                                   double4* __restrict__ off, int2* __restrict__ cell) {
  const int f = blockIdx.y, ax = blockIdx.z;
  const MeshFrame fr = mesh_frame(fa, f);
  if (blockIdx.x * 256 >= fr.nm) return;
  __shared__ double tap[256][17];
  __shared__ int place[256];
  const int tid = threadIdx.x, last = min(256, fr.nm - (int)blockIdx.x * 256) - 1;
  const int row = fr.moff + blockIdx.x * 256 + min(tid, last);
  const int2 sl = slot[row];
  const size_t p = (size_t)fr.moff + start[(size_t)f * (m.nbt + 1) + sl.x] + sl.y;
  const double L = ax == 0 ? fr.box[0] : ax == 1 ? fr.box[1] : fr.box[2];
  const int N = ax == 0 ? m.N[0] : ax == 1 ? m.N[1] : m.N[2];
  int c;
  double t, q = 1.0;
  mesh_cell(mm4[(size_t)ax * cap_mm + row], L, N, c, t);
  const double s = 2.0 * t - 1.0, s2 = s * s;
  if (ax == 0 && tid <= last) {
    int cy, cz;
    double ty, tz;
    mesh_cell(mm4[(size_t)cap_mm + row], fr.box[1], m.N[1], cy, ty);
    mesh_cell(mm4[(size_t)2 * cap_mm + row], fr.box[2], m.N[2], cz, tz);
    off[p] = make_double4(s, 2.0 * ty - 1.0, 2.0 * tz - 1.0, 0.0);
    cell[p] = make_int2(c | cy << 10 | cz << 20, row);
    q = mm4[(size_t)3 * cap_mm + row];
  }
#pragma unroll
  for (int j = 0; j < 8; j++) {
    double e = poly[j * kMeshPoly + kMeshPoly - 2], o = poly[j * kMeshPoly + kMeshPoly - 1];
#pragma unroll
    for (int k = kMeshPoly - 4; k >= 0; k -= 2) {
      e = fma(e, s2, poly[j * kMeshPoly + k]);
      o = fma(o, s2, poly[j * kMeshPoly + k + 1]);
    }
    tap[tid][j] = q * fma(o, s, e);
    tap[tid][15 - j] = q * fma(-o, s, e);
  }
  place[tid] = (int)p;
  __syncthreads();
  // eight lanes write an atom's 128 bytes
#pragma unroll
  for (int k = 0; k < 8; k++) {
    const int a = 32 * k + (tid >> 3), j = 2 * (tid & 7);
    if (a <= last) *(double2*)(taps + (size_t)place[a] * 48 + ax * 16 + j) = make_double2(tap[a][j], tap[a][j + 1]);
  }
}

// ------------------------------------------------------------------ spreading
// mesh[x][y][z] = sum_i q_i phi_x phi_y phi_z, gathered per output tile so that
// no atomics are needed and the sum's order is that of the sorted atoms.  A
// block owns a 16 x 8 x 16 tile, each of its four waves a 16 x 4 x 8 part as
// two matrix-core accumulators: D[x][yz] += A[x][atom] B[atom][yz], four atoms
// per instruction, A = q phi_x and B = phi_y phi_z.  The atoms of the bins
// around the tile are staged in LDS 32 at a time with zeros on both sides of
// their taps, so that a point off the support reads a zero without a test
// (the next 32 are on their way from memory meanwhile); each wave lists the
// atoms whose 16^3 points meet its part, with the three LDS byte addresses of
// its first point.  The products phi_y phi_z of a step are formed before it, so
// that its two matrix instructions follow each other.  A 4 x 4 part has less work
// outside the support (31 19 19 / 16^3 = 2.7 times the useful multiply-adds,
// 3.3 here) but twice the x reads.  In batches matrix cores and LDS are each busy
// about half the time; 27 KB of LDS and 80 registers let six blocks share a CU and
// cover each other's staging: 16 frames of 100 000 charges on a 112^3 mesh 1.67 ms with
// chunks of 64 and three blocks, 1.37 ms so (matrix instructions alone 0.59 ms), 1.30 on
// the 96^3 that these plans take; 64 frames of 5000 to 30 000 on 80^3 1.13 -> 0.90 ms, on
// 64^3 0.82.  Where the tiles are too few for six blocks per CU, KS shares of the atoms
// per block (each with its own staging, summed in LDS at the end): one frame of 35 000
// on 80^3 (250 tiles) 75 us with one share, 54 with two, 44 with four, on 96^3 (432) 60,
// 49 and 53; one of 19 200 on 64^3 (128) 81, 58 and 47 us.  A single frame waits for its own
// staging: matrix cores and LDS 30% busy at 80^3.
// A staged atom: [15 zeros | x taps | 15 zeros | y taps | 7 zeros | z taps], each
// run of zeros (and the next atom's first one) padding the taps on both sides;
// an odd number of doubles for the LDS banks.
static constexpr int kSpreadX = 15, kSpreadY = kSpreadX + 16 + 15, kSpreadZ = kSpreadY + 16 + 7;
static constexpr int kSpreadAtom = kSpreadZ + 16;
static constexpr int kSpreadTail = 16;                                  // zeros after the last atom
static constexpr int kSpreadChunk = 32;                                  // atoms staged at a time
static constexpr int kSpreadRows = 48;                                  // rows of bins around a tile

template <int KS>
__global__ __launch_bounds__(256 * KS, KS == 4 ? 4 : 6) void k_mesh_spread(Mesh m, FrameArg fa, int tx, int ty, int tz,
                                                     const int* __restrict__ start, const double* __restrict__ taps,
                                                     const int2* __restrict__ cell, double* __restrict__ mesh) {
  __shared__ double staged[KS][kSpreadChunk * kSpreadAtom + kSpreadTail];
  __shared__ int cells[KS][kSpreadChunk];
  __shared__ int sources[KS][256];
  __shared__ int2 list[4 * KS][kSpreadChunk + 12];
  __shared__ int row_off[kSpreadRows + 1], row_s0[kSpreadRows], row_l0[kSpreadRows], row_s1[kSpreadRows];
  const int f = blockIdx.y;
  const MeshFrame fr = mesh_frame(fa, f);
  const int nt = tx * ty * tz;
  const int bid = xcd_order(blockIdx.x, nt);
  const int bz = bid / (tx * ty), by = (bid - bz * tx * ty) / tx, bx = bid - (bz * ty + by) * tx;
  const int X0 = 16 * bx, Y0 = 8 * by, Z0 = 16 * bz;
  const int share = KS == 1 ? 0 : uni((int)(threadIdx.x >> 8)), tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
  double* tp = staged[share];
  int *pk = cells[share], *src = sources[share];
  const int* __restrict__ st = start + (size_t)f * (m.nbt + 1);
  // the rows of bins (6 in y, 8 in z; 8 bins along x, in two runs where they
  // wrap) whose atoms can reach the tile
  if (threadIdx.x < 64) {
    int s0 = 0, l0 = 0, s1 = 0, len = 0;
    if (lane < kSpreadRows) {
      int ry = (Y0 >> 2) - 2 + lane % 6, rz = (Z0 >> 2) - 2 + lane / 6;
      ry += ry < 0 ? m.nb[1] : ry >= m.nb[1] ? -m.nb[1] : 0;
      rz += rz < 0 ? m.nb[2] : rz >= m.nb[2] ? -m.nb[2] : 0;
      const int base = (rz * m.nb[1] + ry) * m.nb[0];
      int c0 = (X0 >> 2) - 2;
      if (c0 < 0) c0 += m.nb[0];
      const int c1 = c0 + 8;
      s0 = st[base + c0];
      l0 = st[base + min(c1, m.nb[0])] - s0;
      len = l0;
      if (c1 > m.nb[0]) {
        s1 = st[base];
        len += st[base + c1 - m.nb[0]] - s1;
      }
    }
    int inc = len;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(inc, o, 64);
      if (lane >= o) inc += u;
    }
    if (lane < kSpreadRows) {
      row_off[lane + 1] = inc;
      row_s0[lane] = s0;
      row_l0[lane] = l0;
      row_s1[lane] = s1;
    }
    if (lane == 0) row_off[0] = 0;
  }
  for (int e = tid; e < kSpreadChunk * kSpreadAtom + kSpreadTail; e += 256) tp[e] = 0.0;
  __syncthreads();
  // chunk q holds the atoms q, q + chunks, q + 2 chunks, ...: a sample of the whole
  // neighbourhood, so that the four parts get about as many atoms of it each; the
  // block's shares take the chunks in turn
  const int all = uni(row_off[kSpreadRows]), chunks = (all + kSpreadChunk - 1) / kSpreadChunk;
  const int rounds = (chunks + KS - 1) / KS;
  const int least = all / max(chunks, 1), more = all - least * chunks;
  auto held = [&](int t) {  // atoms in this share's chunk t
    const int q = share + KS * t;
    return q < chunks ? least + (q < more) : 0;
  };
  const int oy = 4 * (wave & 1), oz = 8 * (wave >> 1);
  const int li = lane & 15, lk = lane >> 4;
  // this lane's point relative to the wave's first one, in bytes
  const int xq = 8 * li, yq = 8 * (li >> 2), zq = 8 * (li & 3);
  v4d acc[2];
  acc[0] = acc[1] = v4d{0.0, 0.0, 0.0, 0.0};
  // sorted positions of the atoms of 8 chunks from t, one per thread: the last
  // row that starts at or before the atom
  auto locate = [&](int t) {
    const int q = share + KS * (t + (tid >> 5)), j = q + (tid & 31) * chunks;
    if (q < chunks && j < all) {
      int lo = 0, hi = kSpreadRows - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (row_off[mid] <= j) lo = mid; else hi = mid - 1;
      }
      const int e = j - row_off[lo];
      src[tid] = e < row_l0[lo] ? row_s0[lo] + e : row_s1[lo] + e - row_l0[lo];
    }
  };
  // staging: eight threads per atom load its taps (16 bytes each per axis)
  const int sa = tid >> 3, sp = tid & 7;
  double2 vx, vy, vz;
  int c;
  auto load = [&](int t) {
    if (sa < held(t)) {
      const size_t p = (size_t)fr.moff + src[(t & 7) * kSpreadChunk + sa];
      const double2* __restrict__ from = (const double2*)(taps + p * 48) + sp;
      vx = from[0];
      vy = from[8];
      vz = from[16];
      if (sp == 0) c = cell[p].x;
    }
  };
  if (rounds > 0) {
    locate(0);
    __syncthreads();
    load(0);
  }
  for (int t = 0; t < rounds; t++) {
    const int n = held(t);
    if (sa < n) {
      double* d = tp + sa * kSpreadAtom + 2 * sp;
      d[kSpreadX] = vx.x;
      d[kSpreadX + 1] = vx.y;
      d[kSpreadY] = vy.x;
      d[kSpreadY + 1] = vy.y;
      d[kSpreadZ] = vz.x;
      d[kSpreadZ + 1] = vz.y;
      if (sp == 0) {
        // mesh cell of the atom relative to the tile, biased by 9
        int rx = (c & 1023) - X0, ry = ((c >> 10) & 1023) - Y0, rz = ((c >> 20) & 1023) - Z0;
        rx += rx < -8 ? m.N[0] : rx >= m.N[0] - 8 ? -m.N[0] : 0;
        ry += ry < -8 ? m.N[1] : ry >= m.N[1] - 8 ? -m.N[1] : 0;
        rz += rz < -8 ? m.N[2] : rz >= m.N[2] - 8 ? -m.N[2] : 0;
        pk[sa] = (min(rx, 60) + 9) | (min(ry, 60) + 9) << 8 | (min(rz, 60) + 9) << 16;
      }
    }
    __syncthreads();
    if (((t + 1) & 7) == 0 && t + 1 < rounds) {  // block-uniform
      locate(t + 1);  // (the positions of the previous chunks were read before the barrier)
      __syncthreads();
    }
    if (t + 1 < rounds) load(t + 1);
    {
      bool hit = false;
      int2 ad = make_int2(0, 0);  // byte addresses of its first point: x | y << 16, z
      if (lane < n) {
        const int e = pk[lane];
        // first mesh point of the atom relative to the wave's part
        const int rx = (e & 255) - 16, ry = ((e >> 8) & 255) - 16 - oy, rz = ((e >> 16) & 255) - 16 - oz;
        hit = rx <= 15 && ry >= -15 && ry <= 3 && rz >= -15 && rz <= 7;
        // tap j of an axis sits at its first tap + j; the part's first point reads tap -r
        const int b = 8 * lane * kSpreadAtom;
        ad = make_int2((b + 8 * (kSpreadX - rx)) | (b + 8 * (kSpreadY - ry)) << 16, b + 8 * (kSpreadZ - rz));
      }
      const unsigned long long mask = __ballot(hit);
      const int cnt = (int)__popcll(mask);
      int2* lw = list[4 * share + wave];
      if (hit) lw[__popcll(mask & ((1ull << lane) - 1ull))] = ad;
      // padding to whole steps and for the reads ahead: the zeros at the end
      constexpr int kNone = 8 * kSpreadChunk * kSpreadAtom;
      static_assert(kNone + 8 * kSpreadTail <= 32768, "16-bit addresses");
      if (lane < 12) lw[cnt + lane] = make_int2(kNone | kNone << 16, kNone);
      lds_wave_sync();
      // four atoms per step: the operands of the next step are read and the list
      // entries of the one after while this step is contracted
      const char* __restrict__ tb = (const char*)tp;
      auto at = [&](int byte, int u) { return ((const double*)(tb + byte))[u]; };
      int2 e = lw[lk];
      double x = at((e.x & 0xffff) + xq, 0), p0, p1;
      {
        const double y = at((e.x >> 16) + yq, 0);
        p0 = y * at(e.y + zq, 0);
        p1 = y * at(e.y + zq, 4);
      }
      e = lw[4 + lk];
      for (int s = 0; s < cnt; s += 4) {
        const double nx = at((e.x & 0xffff) + xq, 0), ny = at((e.x >> 16) + yq, 0), nz0 = at(e.y + zq, 0), nz1 = at(e.y + zq, 4);
        e = lw[s + 8 + lk];
        __builtin_amdgcn_sched_barrier(0);
        acc[0] = mfma(x, p0, acc[0]);
        acc[1] = mfma(x, p1, acc[1]);
        __builtin_amdgcn_sched_barrier(0);
        x = nx;
        p0 = ny * nz0;
        p1 = ny * nz1;
      }
    }
    __syncthreads();  // the staged atoms are replaced
  }
  if (KS > 1) {  // the shares' sums (the staged atoms have been read)
    if (share > 0)
#pragma unroll
      for (int r = 0; r < 8; r++) tp[r * 256 + tid] = acc[r & 1][r >> 1];
    __syncthreads();
    if (share > 0) return;
#pragma unroll
    for (int h = 1; h < KS; h++)
#pragma unroll
      for (int r = 0; r < 8; r++) acc[r & 1][r >> 1] += staged[h][r * 256 + tid];
  }
  double* __restrict__ o = mesh + (((size_t)f * m.N[0] + X0) * m.N[1] + Y0 + oy + (li >> 2)) * m.N[2] + Z0 + oz + (li & 3);
  const size_t plane = (size_t)m.N[1] * m.N[2];
#pragma unroll
  for (int r = 0; r < 4; r++)
#pragma unroll
    for (int u = 0; u < 2; u++) o[(size_t)(lk + 4 * r) * plane + 4 * u] = acc[u][r];
}

// ------------------------------------------------------------------ axis contractions
// out[b][M][n] = sum_k tab[M][k] in[b][k][n] on the matrix cores: tab in A
// fragment order [M tile][K step][64 lanes]; one 16 x 32 output part per wave
// (the table fragment serves two column tiles), K in chunks of four steps
// whose loads are issued before the previous chunk is contracted.  The parts of
// all b lie in the grid's x: b runs over frames times x planes along y, more than
// the 65 536 that y takes from 1366 frames on a mesh of 48 planes.
__global__ __launch_bounds__(256) void k_mesh_left(const double* __restrict__ tab, const double* __restrict__ in,
                                                   double* __restrict__ out, int m_tiles, int K, int cols, int batch) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int c_pairs = (cols + 31) / 32, per = m_tiles * c_pairs;
  const int part = blockIdx.x * 4 + uni((int)(threadIdx.x >> 6));
  const int b = part / per, unit = part - b * per;
  if (b >= batch) return;
  const int cp = unit / m_tiles, mt = unit - cp * m_tiles;
  const double* __restrict__ src = in + (size_t)b * K * cols;
  const int c0 = 32 * cp + li, c1 = min(c0 + 16, cols - 16 + li);
  const double* __restrict__ ta = tab + (size_t)mt * (K / 4) * 64 + lane;
  const double* __restrict__ p0 = src + (size_t)lk * cols + c0;
  const double* __restrict__ p1 = src + (size_t)lk * cols + c1;
  const size_t rs = (size_t)4 * cols;
  v4d acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
  double a[4], x[4], y[4];
#pragma unroll
  for (int u = 0; u < 4; u++) {
    a[u] = ta[u * 64];
    x[u] = p0[u * rs];
    y[u] = p1[u * rs];
  }
  for (int k = 16; k <= K; k += 16) {
    double an[4], xn[4], yn[4];
    const int kn = k < K ? k : 0;  // the last round reloads the first chunk (unused)
#pragma unroll
    for (int u = 0; u < 4; u++) {
      an[u] = ta[(kn / 4 + u) * 64];
      xn[u] = p0[(kn / 4 + u) * rs];
      yn[u] = p1[(kn / 4 + u) * rs];
    }
#pragma unroll
    for (int u = 0; u < 4; u++) {
      acc0 = mfma(a[u], x[u], acc0);
      acc1 = mfma(a[u], y[u], acc1);
    }
#pragma unroll
    for (int u = 0; u < 4; u++) {
      a[u] = an[u];
      x[u] = xn[u];
      y[u] = yn[u];
    }
  }
  double* __restrict__ o = out + ((size_t)b * m_tiles * 16 + mt * 16 + lk) * cols;
#pragma unroll
  for (int r = 0; r < 4; r++) {
    o[(size_t)4 * r * cols + c0] = acc0[r];
    if (c0 + 16 < cols) o[(size_t)4 * r * cols + c0 + 16] = acc1[r];
  }
}

// out[row][n] = sum_k in[row][k] tab[k][n]: rows contiguous in k, tab in B
// fragment order [column tile][chunk of 16 k][4 steps][64 lanes], step u of a
// chunk taking k = 16 chunk + 4 (lane / 16) + u so that a lane's four A values
// are 32 contiguous bytes; a 32 x 32 output part per wave.
__global__ __launch_bounds__(256) void k_mesh_right(const double* __restrict__ tab, const double* __restrict__ in,
                                                    double* __restrict__ out, int rows, int K, int cols) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int c_tiles = cols / 16, c_pairs = (c_tiles + 1) / 2;
  const int unit = blockIdx.x * 4 + uni((int)(threadIdx.x >> 6));
  if (unit >= (rows / 32) * c_pairs) return;
  const int rt = unit / c_pairs, cp = unit - rt * c_pairs;
  const int t0 = 2 * cp, t1 = min(t0 + 1, c_tiles - 1);
  const double* __restrict__ src = in + (size_t)blockIdx.y * rows * K;
  const double* __restrict__ pa = src + (size_t)(32 * rt + li) * K + 4 * lk;
  const double* __restrict__ pb = pa + (size_t)16 * K;
  const double* __restrict__ q0 = tab + (size_t)t0 * K * 16 + lane;
  const double* __restrict__ q1 = tab + (size_t)t1 * K * 16 + lane;
  v4d acc[2][2];
#pragma unroll
  for (int u = 0; u < 2; u++)
#pragma unroll
    for (int v = 0; v < 2; v++) acc[u][v] = v4d{0.0, 0.0, 0.0, 0.0};
  double a[2][4], b[2][4];
  auto load = [&](int k, double (&ar)[2][4], double (&br)[2][4]) {
    *(double2*)&ar[0][0] = *(const double2*)(pa + k);
    *(double2*)&ar[0][2] = *(const double2*)(pa + k + 2);
    *(double2*)&ar[1][0] = *(const double2*)(pb + k);
    *(double2*)&ar[1][2] = *(const double2*)(pb + k + 2);
#pragma unroll
    for (int u = 0; u < 4; u++) {
      br[0][u] = q0[(size_t)(k * 16) + u * 64];
      br[1][u] = q1[(size_t)(k * 16) + u * 64];
    }
  };
  load(0, a, b);
  for (int k = 16; k <= K; k += 16) {
    double an[2][4], bn[2][4];
    load(k < K ? k : 0, an, bn);
#pragma unroll
    for (int u = 0; u < 4; u++) {
      acc[0][0] = mfma(a[0][u], b[0][u], acc[0][0]);
      acc[0][1] = mfma(a[0][u], b[1][u], acc[0][1]);
      acc[1][0] = mfma(a[1][u], b[0][u], acc[1][0]);
      acc[1][1] = mfma(a[1][u], b[1][u], acc[1][1]);
    }
#pragma unroll
    for (int u = 0; u < 4; u++)
#pragma unroll
      for (int v = 0; v < 2; v++) {
        a[v][u] = an[v][u];
        b[v][u] = bn[v][u];
      }
  }
  double* __restrict__ o = out + ((size_t)blockIdx.y * rows + 32 * rt + lk) * cols + li;
#pragma unroll
  for (int v = 0; v < 2; v++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      o[(size_t)(16 * v + 4 * r) * cols + 16 * t0] = acc[v][0][r];
      if (t0 + 1 < c_tiles) o[(size_t)(16 * v + 4 * r) * cols + 16 * (t0 + 1)] = acc[v][1][r];
    }
}

// ------------------------------------------------------------------ real basis <-> half space
// Thread = (nx, |ny|, |nz|).  S(nx, s ny, t nz) = sum q (cx + i sx)(cy + i s sy)(cz + i t sz).
struct Mode {
  int nx, ny, nz;
  bool in;
};

DEV Mode mesh_mode(const Mesh& m) {
  const int nz1 = m.m[2] + 1, ny1 = m.m[1] + 1;
  const int e = blockIdx.x * 256 + threadIdx.x;
  Mode o;
  o.nz = e % nz1;
  o.ny = (e / nz1) % ny1;
  o.nx = e / (nz1 * ny1);
  o.in = o.nx <= m.m[0];
  return o;
}

// index of basis function cos (s = 0) or sin (s = 1) of wave number n; sin 0 is absent
DEV int basis(int n, int s, int m) { return s ? m + n : n; }

__global__ __launch_bounds__(256) void k_mesh_smm(Mesh m, int KF, const double* __restrict__ T,
                                                  double2* __restrict__ smm, size_t smm_stride) {
  const int f = blockIdx.y;
  const Mode o = mesh_mode(m);
  if (!o.in) return;
  const double* __restrict__ t = T + (size_t)f * m.C[0] * m.C[1] * m.C[2];
  double v[2][2][2];
#pragma unroll
  for (int u = 0; u < 8; u++) {
    const int a = u >> 2, b = (u >> 1) & 1, c = u & 1;
    const bool have = (!a || o.nx > 0) && (!b || o.ny > 0) && (!c || o.nz > 0);
    v[a][b][c] = have ? t[((size_t)basis(o.nx, a, m.m[0]) * m.C[1] + basis(o.ny, b, m.m[1])) * m.C[2] +
                          basis(o.nz, c, m.m[2])]
                      : 0.0;
  }
  const int NY = 2 * m.m[1] + 1, NZ = 2 * m.m[2] + 1;
  double2* __restrict__ out = smm + (size_t)f * smm_stride;
#pragma unroll
  for (int u = 0; u < 4; u++) {
    const int sy = u >> 1, sz = u & 1;
    if ((sy && o.ny == 0) || (sz && o.nz == 0)) continue;
    const double s = sy ? -1.0 : 1.0, tt = sz ? -1.0 : 1.0;
    const double re = v[0][0][0] - s * tt * v[0][1][1] - s * v[1][1][0] - tt * v[1][0][1];
    const double im = v[1][0][0] + s * v[0][1][0] + tt * v[0][0][1] - s * tt * v[1][1][1];
    out[((size_t)o.nx * NY + (sy ? -o.ny : o.ny) + m.m[1]) * NZ + (sz ? -o.nz : o.nz) + m.m[2]] = make_double2(re, im);
  }
}

// Re[W e^{-i(nx x + s ny y + t nz z)}] summed over the four signs, on the real basis
__global__ __launch_bounds__(256) void k_mesh_wk(Mesh m, int KF, const double2* __restrict__ wk,
                                                 double* __restrict__ U) {
  const int f = blockIdx.y;
  const Mode o = mesh_mode(m);
  if (!o.in) return;
  const int NY = 2 * m.m[1] + 1, NZ = 2 * m.m[2] + 1;
  const double2* __restrict__ w = wk + (size_t)f * KF;
  double v[2][2][2] = {};
#pragma unroll
  for (int u = 0; u < 4; u++) {
    const int sy = u >> 1, sz = u & 1;
    if ((sy && o.ny == 0) || (sz && o.nz == 0)) continue;
    const double s = sy ? -1.0 : 1.0, tt = sz ? -1.0 : 1.0;
    const double2 W = w[((size_t)o.nx * NY + (sy ? -o.ny : o.ny) + m.m[1]) * NZ + (sz ? -o.nz : o.nz) + m.m[2]];
    v[0][0][0] += W.x;
    v[0][1][1] -= s * tt * W.x;
    v[1][1][0] -= s * W.x;
    v[1][0][1] -= tt * W.x;
    v[1][0][0] += W.y;
    v[0][1][0] += s * W.y;
    v[0][0][1] += tt * W.y;
    v[1][1][1] -= s * tt * W.y;
  }
  double* __restrict__ t = U + (size_t)f * m.C[0] * m.C[1] * m.C[2];
#pragma unroll
  for (int u = 0; u < 8; u++) {
    const int a = u >> 2, b = (u >> 1) & 1, c = u & 1;
    if ((!a || o.nx > 0) && (!b || o.ny > 0) && (!c || o.nz > 0))
      t[((size_t)basis(o.nx, a, m.m[0]) * m.C[1] + basis(o.ny, b, m.m[1])) * m.C[2] + basis(o.nz, c, m.m[2])] = v[a][b][c];
  }
}

// ------------------------------------------------------------------ reading the mesh at the charges
// A block (one per CU) marches along x through columns of 8 x 16 mesh cells in
// y and z, four cells (one bin) per step.  A step's atoms read 19 x 23 x 31 mesh
// points; the planes live in a ring in LDS, so that a step loads only the four
// planes it adds (24 KB per 512 cells; a tile of 1024 cells by itself reads
// 135 KB).  27 planes let waves drift one step apart: a wave that enters step k
// adds its share of the planes of step k + 1 (loaded into registers during step
// k - 1) and counts itself in, then takes atoms, which the waves claim one after
// another; it enters k + 1 once all waves have counted in for k.  A wave's share
// of the planes of k + 1 replaces planes last read in step k - 2, which every
// wave has left when it counts in for k - 1.
//
// A wave takes one atom at a time: lanes 0..47 evaluate the 48 taps and their
// derivatives from polynomials kept in registers; then lanes hold 16 z points
// x 4 y points (y in four rounds) and the x points come one after another,
// their two factors read from the lanes into scalar registers.  Each lane sums
// its column over x with both (128 multiply-adds for the atom's 4096 points),
// then the y and z factors give potential and gradient, reduced over the wave.
// The 4096 reads per atom bound it: 32 KB per atom from LDS at 128 bytes per
// cycle and CU.  Three waves per SIMD with the reads of one x point ahead cover
// each other's start and end of an atom.
// Measured against tiles of 8 x 8 x 16 cells, each staged whole, dealt to the
// waves in turn: 16 frames of 100 000 charges on a 112^3 mesh 1.45 -> 1.38 ms (the
// LDS reads alone 0.85 ms), 64 frames of 5000 to 30 000 on 80^3 1.62 -> 1.09 ms,
// one of 35 000 on 96^3 54 -> 50 us.  On the 96^3, 64^3 and 80^3 that these plans take
// 1.23 ms, 0.90 ms and 42 us; with 8 waves 1.50, 1.07 and 47, with 16 (registers short)
// 1.22, 0.93 and 50.
static constexpr int kGatherY = 8, kGatherZ = 16;                        // cells of a column
static constexpr int kGatherWY = kGatherY + 15, kGatherWZ = kGatherZ + 15;  // points of a plane
static constexpr int kGatherWindow = 4 + 15;                             // planes a step reads
static constexpr int kGatherRing = kGatherWindow + 8;                    // planes kept
static constexpr int kGatherPlane = kGatherWY * kGatherWZ;
static constexpr int kGatherBlocks = 256;                                // one per CU
static constexpr int kGatherWaves = 12;
static constexpr int kGatherGroups = 4 * kGatherWaves;                   // rows loaded at a time, 16 lanes each
static constexpr int kGatherFill = (kGatherWindow * kGatherWY + kGatherGroups - 1) / kGatherGroups;
static constexpr int kGatherAdd = (4 * kGatherWY + kGatherGroups - 1) / kGatherGroups;

typedef double v2d __attribute__((ext_vector_type(2)));

// value of a double in lane `l` (wave-uniform result)
DEV double lane_value(double v, int l) {
  const unsigned long long b = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)(b & 0xffffffffu), l);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// A step's atoms among the sorted ones: lane r < 8 holds the first atom (s0)
// and the running count (exc) of bin row r (2 in y, 4 in z).
struct GatherStep {
  int s0, exc, total;
};

__global__ __launch_bounds__(64 * kGatherWaves) void k_mesh_gather(Mesh m, FrameArg fa, int ty, int tz, int parts,
                                                      const int* __restrict__ start, const double* __restrict__ poly,
                                                      const double4* __restrict__ off, const int2* __restrict__ cell,
                                                      const double* __restrict__ mesh, double* __restrict__ fpart) {
  __shared__ double ring[kGatherRing * kGatherPlane];
  __shared__ double2 tv[kGatherWaves][32];
  __shared__ int counted, claimed;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int lz = lane & 15, ly = lane >> 4;
  const int grp = tid >> 4, zp = 2 * (tid & 15);
  double c[kMeshPoly];
  {
    const double* __restrict__ pc = poly + (lz < 8 ? lz : 15 - lz) * kMeshPoly;
#pragma unroll
    for (int k = 0; k < kMeshPoly; k++) c[k] = (k & 1) && lz >= 8 ? -pc[k] : pc[k];
  }
  const int ax = min(ly, 2);

  // Segments: column u / parts of a frame, part u % parts of its steps.  The
  // 8 XCDs (blocks go to them in turn) take contiguous eighths of each frame's
  // segments, another eighth from frame to frame (frames come largest first).
  const int per = parts * ty * tz, xcd = blockIdx.x & 7;
  int i = blockIdx.x >> 3;  // the block's place in its XCD's list
  for (int f = 0; f < fa.n_frames; f++) {
    const int e = (xcd + f) & 7, u0 = (int)((long)per * e / 8), u1 = (int)((long)per * (e + 1) / 8);
    for (; i < u1 - u0; i += gridDim.x >> 3) {
      const int u = u0 + i, part = u % parts, col = u / parts;
      const int by = col % ty, bz = col / ty;
      const int Y0 = kGatherY * by, Z0 = kGatherZ * bz - 8;  // the first column in z wraps
      const int b0 = m.nb[0] * part / parts, len = m.nb[0] * (part + 1) / parts - b0, X0 = 4 * b0;
      const MeshFrame fr = mesh_frame(fa, f);
      const double* __restrict__ src = mesh + (size_t)f * m.N[0] * m.N[1] * m.N[2];
      const int* __restrict__ st = start + (size_t)f * (m.nbt + 1);

      auto rows_of = [&](int k) {  // first and last + 1 atom of the step's bin row `lane`
        int2 r = make_int2(0, 0);
        if (lane < 8) {
          int rz = (Z0 >> 2) + (lane >> 1);
          rz += rz < 0 ? m.nb[2] : 0;
          const int* __restrict__ p = st + (rz * m.nb[1] + (Y0 >> 2) + (lane & 1)) * m.nb[0] + b0 + k;
          r = make_int2(p[0], p[1]);
        }
        return r;
      };
      auto count = [&](int2 r) {
        const int n = r.y - r.x;
        int inc = n;
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
          const int v = __shfl_up(inc, o, 64);
          if (lane >= o) inc += v;
        }
        return GatherStep{r.x, lane < 8 ? inc - n : 0x7fffffff, (int)__builtin_amdgcn_readlane(inc, 7)};
      };
      // points zp - 1 and zp (of 31; point 0 pairs with one outside) of row y of plane p
      int gz = Z0 - 8 + zp;
      gz += gz < 0 ? m.N[2] : gz >= m.N[2] ? -m.N[2] : 0;
      auto load = [&](int p, int y) {
        int gx = X0 - 7 + p, gy = Y0 - 7 + y;
        gx += gx < 0 ? m.N[0] : gx >= m.N[0] ? -m.N[0] : 0;
        gy += gy < 0 ? m.N[1] : gy >= m.N[1] ? -m.N[1] : 0;
        return *(const v2d*)(src + (size_t)((gx * m.N[1] + gy) * m.N[2] + gz));
      };
      auto put = [&](int slot, int y, v2d v) {
        double* d = ring + slot * kGatherPlane + y * kGatherWZ + zp - 1;
        if (zp) d[0] = v.x;
        d[1] = v.y;
      };

      __syncthreads();  // the previous segment has been read
      if (tid == 0) counted = claimed = 0;
      {
        v2d v[kGatherFill];
#pragma unroll
        for (int t = 0; t < kGatherFill; t++) {
          const int r = min(grp + kGatherGroups * t, kGatherWindow * kGatherWY - 1), p = r / kGatherWY;
          v[t] = load(p, r - p * kGatherWY);
        }
#pragma unroll
        for (int t = 0; t < kGatherFill; t++) {
          const int r = grp + kGatherGroups * t, p = r / kGatherWY;
          if (r < kGatherWindow * kGatherWY) put(p, r - p * kGatherWY, v[t]);
        }
      }
      v2d add[kGatherAdd];
      auto load_step = [&](int k) {  // the planes step k adds
#pragma unroll
        for (int t = 0; t < kGatherAdd; t++) {
          const int r = min(grp + kGatherGroups * t, 4 * kGatherWY - 1), p = r / kGatherWY;
          add[t] = load(kGatherWindow - 4 + 4 * k + p, r - p * kGatherWY);
        }
      };
      auto put_step = [&](int k) {
        const int s = (kGatherWindow - 4 + 4 * k) % kGatherRing;
#pragma unroll
        for (int t = 0; t < kGatherAdd; t++) {
          const int r = grp + kGatherGroups * t, p = r / kGatherWY;
          if (r < 4 * kGatherWY) put(s + p >= kGatherRing ? s + p - kGatherRing : s + p, r - p * kGatherWY, add[t]);
        }
      };

      // Waves claim the segment's atoms in order, each claim on its way while
      // the wave works on the atoms claimed before.  The claim `j` counts from the
      // first atom of step kf.
      int kf = 0, base = 0, next = 0;
      GatherStep g = count(rows_of(0));
      int2 ahead = rows_of(min(1, len - 1));
      auto claim = [&]() {
        next = 0;
        if (lane == 0) next = __hip_atomic_fetch_add(&claimed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      };
      // an atom's step (len: no more atoms), its offset along the lane's axis, its cell and its row
      struct Atom {
        double s;
        int k, cx, row;
      };
      auto fetch = [&]() {
        Atom a{};
        const int j = uni(next);
        while (j - base >= g.total && kf < len) {
          base += g.total;
          kf++;
          g = count(ahead);
          ahead = rows_of(min(kf + 1, len - 1));
        }
        a.k = kf;
        if (kf < len) {
          claim();
          const int jf = j - base;
          const int row = (int)__popcll(__ballot(g.exc <= jf)) - 1;  // the bin row that holds the atom
          const int p = fr.moff + __builtin_amdgcn_readlane(g.s0, row) + jf - __builtin_amdgcn_readlane(g.exc, row);
          a.s = ((const double*)(off + p))[ax];
          const int2 ce = cell[p];
          a.cx = ce.x;
          a.row = ce.y;
        }
        return a;
      };
      // group ly ends with the potential (0) or a gradient component (per mesh cell -> per length)
      const double scale = ly == 0   ? 1.0
                           : ly == 1 ? m.N[0] * fr.inv_box[0]
                           : ly == 2 ? m.N[1] * fr.inv_box[1]
                                     : m.N[2] * fr.inv_box[2];
      auto evaluate = [&](const Atom& at) {
        const double s = at.s;
        double pv = c[kMeshPoly - 1], pd = 0.0;
#pragma unroll
        for (int k = kMeshPoly - 2; k >= 0; k--) {
          pd = fma(pd, s, pv);
          pv = fma(pv, s, c[k]);
        }
        pd *= 2.0;  // d/dt
        if (lane >= 16 && lane < 48) tv[wave][lane - 16] = make_double2(pv, pd);
        const int cx = uni(at.cx);
        int dz = (cx >> 20 & 1023) - Z0;
        dz -= dz >= m.N[2] ? m.N[2] : 0;
        const double* w0 = ring + ((cx >> 10 & 1023) - Y0 + ly) * kGatherWZ + dz + lz;
        const int slot = ((cx & 1023) - X0) % kGatherRing;  // of the atom's first plane
        auto plane = [&](int x) { return w0 + (slot + x >= kGatherRing ? slot + x - kGatherRing : slot + x) * kGatherPlane; };
        // the reads of the next x point are issued ahead of the multiply-adds of this one
        double A[4] = {0.0, 0.0, 0.0, 0.0}, D[4] = {0.0, 0.0, 0.0, 0.0}, w[2][4];
        const double* wp = plane(0);
#pragma unroll
        for (int q = 0; q < 4; q++) w[0][q] = wp[4 * q * kGatherWZ];
#pragma unroll
        for (int x = 0; x < 16; x++) {
          if (x < 15) {
            wp = plane(x + 1);
#pragma unroll
            for (int q = 0; q < 4; q++) w[(x + 1) & 1][q] = wp[4 * q * kGatherWZ];
          }
          __builtin_amdgcn_sched_barrier(0);
          const double xv = lane_value(pv, x), xd = lane_value(pd, x);
#pragma unroll
          for (int q = 0; q < 4; q++) {
            A[q] = fma(xv, w[x & 1][q], A[q]);
            D[q] = fma(xd, w[x & 1][q], D[q]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        lds_wave_sync();
        double u0 = 0.0, u1 = 0.0, u2 = 0.0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const double2 y = tv[wave][ly + 4 * q];
          u0 = fma(y.x, A[q], u0);
          u1 = fma(y.x, D[q], u1);
          u2 = fma(y.y, A[q], u2);
        }
        const double2 z = tv[wave][16 + lz];
        lds_wave_sync();  // the taps are replaced for the next atom
        const double o0 = u0 * z.x, o1 = u1 * z.x, o2 = u2 * z.x, o3 = u0 * z.y;
        // four sums over 64 lanes: row ly of 16 lanes ends with o<ly>
        const double a = row_sum(fold16(fold32(o0, o2), fold32(o1, o3)));
        if (lz == 0) fpart[(size_t)at.row * 4 + ly] = a * scale;
      };

      if (len > 1) load_step(1);
      __syncthreads();
      claim();
      Atom a0 = fetch(), a1 = fetch();
      auto enter = [&](int k) {
        // every wave counts in once per step, whether it has atoms or not, and
        // waits only for counts of the step before: all of them come
        if (k > 0)
          while (__hip_atomic_load(&counted, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < k * kGatherWaves)
            __builtin_amdgcn_s_sleep(1);
        if (k + 1 < len) {
          put_step(k + 1);
          // the count releases the points written, and the reads of the steps before, of all lanes of the wave
          if (lane == 0) __hip_atomic_fetch_add(&counted, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (k + 2 < len) load_step(k + 2);
        }
      };
      enter(0);
      int k = 0;
      while (true) {
        const int until = min(a0.k, len - 1);
        while (k < until) enter(++k);
        if (a0.k >= len) break;
        const Atom a = a0;
        a0 = a1;
        a1 = fetch();
        evaluate(a);
      }
    }
    i -= u1 - u0;
  }
}

// ------------------------------------------------------------------ launchers
static hipError_t left(const double* tab, const double* in, double* out, int m, int K, int cols, int batch,
                       hipStream_t s) {
  // (below 2^24: each writes at least 256 numbers of the mesh workspace, which is held to kMeshMaxBytes)
  const int parts = (m / 16) * ((cols + 31) / 32) * batch;
  hipLaunchKernelGGL(k_mesh_left, dim3((parts + 3) / 4), dim3(256), 0, s, tab, in, out, m / 16, K, cols, batch);
  return hipGetLastError();
}

static hipError_t right(const double* tab, const double* in, double* out, int rows, int K, int cols, int batch,
                        hipStream_t s) {
  const int units = (rows / 32) * ((cols / 16 + 1) / 2);
  hipLaunchKernelGGL(k_mesh_right, dim3((units + 3) / 4, batch), dim3(256), 0, s, tab, in, out, rows, K, cols);
  return hipGetLastError();
}

#define MCHK(x)                            \
  do {                                     \
    const hipError_t e_ = (x);             \
    if (e_ != hipSuccess) return e_;       \
  } while (0)

hipError_t launch_mesh_sort(const Mesh& m, const FrameArg& fa, int max_nm, int cap_mm, Work& w, hipStream_t s) {
  if (max_nm > 0) {
    const dim3 grid((max_nm + 255) / 256, fa.n_frames);
    hipLaunchKernelGGL(k_mesh_count, grid, dim3(256), 0, s, m, fa, w.mm4, cap_mm, w.mesh_cnt, w.mesh_slot);
    MCHK(hipGetLastError());
  }
  hipLaunchKernelGGL(k_mesh_scan, dim3(fa.n_frames), dim3(1024), 0, s, m, w.mesh_cnt, w.mesh_start);
  MCHK(hipGetLastError());
  if (max_nm == 0) return hipSuccess;
  const dim3 grid((max_nm + 255) / 256, fa.n_frames);
  if (w.mesh_perm) {
    hipLaunchKernelGGL(k_mesh_list, grid, dim3(256), 0, s, m, fa, w.mesh_start, w.mesh_slot, w.mesh_perm);
    MCHK(hipGetLastError());
    hipLaunchKernelGGL(k_mesh_rank, grid, dim3(256), 0, s, m, fa, w.mesh_start, w.mesh_perm, w.mesh_slot);
    MCHK(hipGetLastError());
  }
  hipLaunchKernelGGL(k_mesh_sort, dim3(grid.x, grid.y, 3), dim3(256), 0, s, m, fa, w.mm4, cap_mm, w.mesh_start,
                     w.mesh_slot, w.mesh_poly, w.mesh_taps, w.mesh_off, w.mesh_cell);
  return hipGetLastError();
}

// shares of a tile's atoms: as many as the 24 waves of each CU hold at once
// (times of each beside the kernel)
int mesh_shares(const Mesh& m, int n_frames) {
  const long tiles = (long)(m.N[0] / 16) * (m.N[1] / 8) * (m.N[2] / 16) * n_frames;
  return tiles <= 256 ? 4 : tiles <= 768 ? 2 : 1;
}

// a tile meets the atoms of 32 x 24 x 32 cells
double mesh_spread_rounds(const Mesh& m, int n_frames, double n) {
  const double cells = (double)m.N[0] * m.N[1] * m.N[2];
  return n * (32.0 * 24.0 * 32.0) / cells / (kSpreadChunk * mesh_shares(m, n_frames));
}

hipError_t launch_mesh_sfac(const Mesh& m, const FrameArg& fa, Work& w, hipStream_t s) {
  const int F = fa.n_frames;
  const int tx = m.N[0] / 16, ty = m.N[1] / 8, tz = m.N[2] / 16;
  const int shares = mesh_shares(m, F);
#define SPREAD(KS)                                                                                               \
  hipLaunchKernelGGL(k_mesh_spread<KS>, dim3(tx * ty * tz, F), dim3(256 * KS), 0, s, m, fa, tx, ty, tz,          \
                     w.mesh_start, w.mesh_taps, w.mesh_cell, w.mesh_q)
  if (shares == 4)
    SPREAD(4);
  else if (shares == 2)
    SPREAD(2);
  else
    SPREAD(1);
#undef SPREAD
  MCHK(hipGetLastError());
  MCHK(right(w.mesh_tab[2], w.mesh_q, w.mesh_h, m.N[0] * m.N[1], m.N[2], m.C[2], F, s));
  MCHK(left(w.mesh_tab[1], w.mesh_h, w.mesh_g, m.C[1], m.N[1], m.C[2], F * m.N[0], s));
  return left(w.mesh_tab[0], w.mesh_g, w.mesh_t, m.C[0], m.N[0], m.C[1] * m.C[2], F, s);
}

hipError_t launch_mesh_smm(const Mesh& m, const Grid& g, const FrameArg& fa, double2* smm, size_t smm_stride, Work& w,
                           hipStream_t s) {
  const int n = (m.m[0] + 1) * (m.m[1] + 1) * (m.m[2] + 1);
  hipLaunchKernelGGL(k_mesh_smm, dim3((n + 255) / 256, fa.n_frames), dim3(256), 0, s, m, g.KF, w.mesh_t, smm,
                     smm_stride);
  return hipGetLastError();
}

hipError_t launch_mesh_force(const Mesh& m, const Grid& g, const FrameArg& fa, int max_nm, Work& w, hipStream_t s) {
  if (max_nm == 0) return hipSuccess;
  const int F = fa.n_frames;
  const int n = (m.m[0] + 1) * (m.m[1] + 1) * (m.m[2] + 1);
  hipLaunchKernelGGL(k_mesh_wk, dim3((n + 255) / 256, F), dim3(256), 0, s, m, g.KF, w.wk, w.mesh_bt);
  MCHK(hipGetLastError());
  MCHK(left(w.mesh_btab[0], w.mesh_bt, w.mesh_bg, m.N[0], m.C[0], m.C[1] * m.C[2], F, s));
  MCHK(left(w.mesh_btab[1], w.mesh_bg, w.mesh_bh, m.N[1], m.C[1], m.C[2], F * m.N[0], s));
  MCHK(right(w.mesh_btab[2], w.mesh_bh, w.mesh_v, m.N[0] * m.N[1], m.C[2], m.N[2], F, s));
  // Parts of a column's steps: the blocks' largest share, a segment's start
  // counted as 1.5 steps.
  const int ty = m.N[1] / kGatherY, tz = m.N[2] / kGatherZ;
  int parts = 1;
  double least = 1e300;
  for (int p = 1; p <= m.nb[0]; p++) {
    const long units = (long)p * ty * tz * F;
    const double cost = (double)((units + kGatherBlocks - 1) / kGatherBlocks) * ((m.nb[0] + p - 1) / p + 1.5);
    if (cost < least) {
      least = cost;
      parts = p;
    }
  }
  const int blocks = (int)std::min((long)kGatherBlocks, ((long)parts * ty * tz * F + 7) / 8 * 8);
  hipLaunchKernelGGL(k_mesh_gather, dim3(blocks), dim3(64 * kGatherWaves), 0, s, m, fa, ty, tz, parts, w.mesh_start,
                     w.mesh_poly, w.mesh_off, w.mesh_cell, w.mesh_v, w.fpart);
  return hipGetLastError();
}

// ------------------------------------------------------------------ tables (host)
static constexpr double kMeshBeta = 42.5;
static constexpr int kMeshWidth = 16;

// Smallest damping A at the band edge of |n| <= m on N points for which the
// aliasing, weighted with exp(-A (n/m)^2), stays below 1e-14 at every n.
double mesh_damping(int N, int m) {
  const double pw = kPiM * kMeshWidth, need = 32.2;  // -ln 1e-14
  auto S = [&](double v) { return sqrt(std::max(0.0, kMeshBeta * kMeshBeta - pw * pw * v * v)); };
  double A = 0.0;
  for (int n = 1; n <= m; n++) {
    const double u = (double)n / N, lack = need - (S(u) - S(1.0 - u));
    if (lack > 0.0) A = std::max(A, lack * m * (double)m / ((double)n * n));
  }
  return A;
}

// The smallest N (a multiple of 16: tiles of the spreading and of the
// contractions; at least 48, so that a tile meets an atom's points once) that
// suits the damping A of the plan's box with a margin of 20% (boxes of other
// frames and later calls may be larger) and never relies on more than A = 21.
// From N = 6 m on hardly any damping is needed.
bool mesh_shape(const Grid& g, const double box[3], Mesh& m) {
  const int mm[3] = {g.mx, g.my, g.mz};
  for (int a = 0; a < 3; a++) {
    const double x = kPiM * mm[a] / (g.alpha * box[a]), A = std::min(0.8 * x * x, 21.0);
    int N = std::max(48, 16 * ((2 * mm[a] + 1 + 15) / 16));
    while (N < 6 * mm[a] && mesh_damping(N, mm[a]) > A) N += 16;
    m.m[a] = mm[a];
    m.N[a] = N;
    m.nb[a] = N / 4;
    m.C[a] = 16 * ((2 * mm[a] + 1 + 15) / 16);
    m.damping[a] = mesh_damping(N, mm[a]);
    if (N > 1008) return false;  // cells are stored in 10 bits per axis
  }
  m.nbt = m.nb[0] * m.nb[1] * m.nb[2];
  // one frame's mesh is addressed with 32-bit byte offsets
  return (size_t)m.N[0] * m.N[1] * m.N[2] * 8 < (size_t(1) << 31);
}

static long double bessel_i0(long double x) {
  const long double t = x * x / 4;
  long double s = 1, term = 1;
  for (int k = 1; k < 200 && term > s * 1e-22L; k++) {
    term *= t / ((long double)k * k);
    s += term;
  }
  return s;
}

void mesh_tables(const Mesh& m, std::vector<double>& poly, std::vector<double> (&fwd)[3],
                 std::vector<double> (&bwd)[3]) {
  const long double pi = acosl(-1.0L), beta = kMeshBeta, i0b = bessel_i0(beta);
  constexpr int w = kMeshWidth, P = kMeshPoly;
  // taps: Chebyshev interpolation in s, then powers of s
  long double ch[4 * P];  // cos(pi k / (2 P))
  for (int k = 0; k < 4 * P; k++) ch[k] = cosl(pi * k / (2 * P));
  poly.assign((size_t)8 * P, 0.0);
  for (int j = 0; j < 8; j++) {
    long double fv[P], c[P], p[P] = {0}, t0[P] = {0}, t1[P] = {0};
    for (int k = 0; k < P; k++) {
      const long double s = ch[2 * k + 1], x = ((j - 7) - (s + 1) / 2) * 2 / w, r2 = 1 - x * x;
      fv[k] = r2 > 0 ? bessel_i0(beta * sqrtl(r2)) / i0b : 1 / i0b;
    }
    for (int n = 0; n < P; n++) {
      c[n] = 0;
      for (int k = 0; k < P; k++) c[n] += fv[k] * ch[n * (2 * k + 1) % (4 * P)];
      c[n] *= (n ? 2.0L : 1.0L) / P;
    }
    t0[0] = 1;
    t1[1] = 1;
    for (int k = 0; k < P; k++) p[k] = c[0] * t0[k] + c[1] * t1[k];
    for (int n = 2; n < P; n++) {
      long double t2[P];
      for (int k = 0; k < P; k++) t2[k] = (k ? 2 * t1[k - 1] : 0) - t0[k];
      for (int k = 0; k < P; k++) {
        p[k] += c[n] * t2[k];
        t0[k] = t1[k];
        t1[k] = t2[k];
      }
    }
    for (int k = 0; k < P; k++) poly[(size_t)j * P + k] = (double)p[k];
  }
  for (int a = 0; a < 3; a++) {
    const int N = m.N[a], mm = m.m[a], C = m.C[a];
    std::vector<long double> cs(N);  // cos(2 pi l / N); N is a multiple of 4
    for (int l = 0; l < N; l++) cs[l] = cosl(2 * pi * l / N);
    // basis function c at mesh point l, divided by the kernel's transform
    std::vector<double> b((size_t)C * N, 0.0);
    for (int n = 0; n <= mm; n++) {
      const long double xi = pi * w * n / N, r = sqrtl(beta * beta - xi * xi);  // n/N < 1/2: xi < beta
      const long double dec = r * i0b / (w * sinhl(r));
      for (int l = 0; l < N; l++) {
        const int th = (int)((long)n * l % N);
        b[(size_t)n * N + l] = (double)(cs[th] * dec);
        if (n) b[(size_t)(mm + n) * N + l] = (double)(cs[(th + 3 * N / 4) % N] * dec);  // sin = cos(. - pi/2)
      }
    }
    fwd[a].resize((size_t)C * N);
    bwd[a].resize((size_t)C * N);
    auto left_order = [&](std::vector<double>& o, int M, int K, auto&& e) {
      for (int mt = 0; mt < M / 16; mt++)
        for (int st = 0; st < K / 4; st++)
          for (int l = 0; l < 64; l++) o[((size_t)mt * (K / 4) + st) * 64 + l] = e(16 * mt + (l & 15), 4 * st + (l >> 4));
    };
    auto right_order = [&](std::vector<double>& o, int K, int cols, auto&& e) {
      for (int ct = 0; ct < cols / 16; ct++)
        for (int ch = 0; ch < K / 16; ch++)
          for (int u = 0; u < 4; u++)
            for (int l = 0; l < 64; l++)
              o[(((size_t)ct * (K / 16) + ch) * 4 + u) * 64 + l] = e(16 * ch + 4 * (l >> 4) + u, 16 * ct + (l & 15));
    };
    if (a < 2) {
      left_order(fwd[a], C, N, [&](int i, int k) { return b[(size_t)i * N + k]; });
      left_order(bwd[a], N, C, [&](int i, int k) { return b[(size_t)k * N + i]; });
    } else {
      right_order(fwd[a], N, C, [&](int k, int j) { return b[(size_t)j * N + k]; });
      right_order(bwd[a], C, N, [&](int k, int j) { return b[(size_t)k * N + j]; });
    }
  }
}

}  // namespace mpe
