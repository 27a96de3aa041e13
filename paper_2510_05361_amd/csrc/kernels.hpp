// Device kernels of the MT-DAO hot path for CDNA4 (gfx950).
//
// All kernels are streaming, HBM-bound passes: the local step reads x, g,
// u^1..u^N, v once and writes x, u^1..u^N, v once per element (no MFMA:
// there is no contraction).  A lane owns V consecutive elements, so loads
// and stores are 16-byte vector accesses (8-byte for bf16 in the step) and a
// 64-lane wavefront moves 1 KiB per instruction; all loads of a tile are
// issued before any of them is consumed.  Rows are replica-major [K][P] and
// start at any element: vectors are aligned to their element only.  Three
// organisations:
//   - flat: the plain step takes the K P elements of each buffer as one
//     array, as the update is element-wise;
//   - one wavefront per replica (the fused step + sync, the mean, the
//     diagnostics and Algorithm 4's step for 1 < K <= 16): a workgroup of
//     K waves takes one piece of 64 V elements of every row, and values
//     that must be averaged meet in LDS;
//   - one thread per column of all K rows (the same for K = 1 and K > 16).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mtdao {

constexpr int kBlock = 256;
constexpr int kMaxN = 4;
constexpr int kMaxMeanStates = 2 + kMaxN;

enum Form { kAdam = 0, kAdopt = 1, kSgdm = 2 };
enum AdoptOrder { kPrev = 0, kCur = 1 };

// scalars, and vectors at addresses aligned to their element only
struct f32x1 { using type = float; };
struct f32x4 { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };
struct u16x1 { using type = uint16_t; };
struct u16x4 { typedef uint16_t type __attribute__((ext_vector_type(4), aligned(2))); };
struct u16x8 { typedef uint16_t type __attribute__((ext_vector_type(8), aligned(2))); };

template <bool B>
struct BoolC { static constexpr bool value = B; };

// ------------------------------------------------------------ conversions

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Round-to-nearest-even fp32 -> bf16 (NaN stays a quiet NaN).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// A wave-uniform value that no running kernel writes (a parameter table, the
// device-side step count, the clip factors of an earlier launch), read
// through the scalar cache: the load waits only on other scalar loads,
// never on the vector loads of the tile in flight.
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
  return *(const __attribute__((address_space(4))) T*)p;
}

// Uniform device pointers, in scalar registers from here on, all in one
// round of scalar loads (the address space goes with them: behind asm a
// plain pointer would be a flat one).
template <typename A, typename B, typename C, typename D>
__device__ __forceinline__ void in_sgprs(A*& a, B*& b, C*& c, D*& d) {
  typedef A __attribute__((address_space(1)))* GA;
  typedef B __attribute__((address_space(1)))* GB;
  typedef C __attribute__((address_space(1)))* GC;
  typedef D __attribute__((address_space(1)))* GD;
  GA qa = (GA)a;
  GB qb = (GB)b;
  GC qc = (GC)c;
  GD qd = (GD)d;
  asm volatile("" : "+s"(qa), "+s"(qb), "+s"(qc), "+s"(qd));
  a = (A*)qa;
  b = (B*)qb;
  c = (C*)qc;
  d = (D*)qd;
}

// --------------------------------------------------- vector load / store
//
// load_v<T, V>(p, e, out): V consecutive elements starting at element e,
// widened to fp32.  T = float, or uint16_t holding bf16 bit patterns.  V = 1
// (the end of a row), 4 or 8.

// (vector types go by alias: a deduced type would lose the alignment)
template <bool NT, typename VT>
__device__ __forceinline__ typename VT::type ld(const void* p) {
  if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const typename VT::type*>(p));
  else return *reinterpret_cast<const typename VT::type*>(p);
}

template <bool NT, typename VT>
__device__ __forceinline__ void st(void* p, typename VT::type v) {
  if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<typename VT::type*>(p));
  else *reinterpret_cast<typename VT::type*>(p) = v;
}

template <typename T, int V, bool NT>
__device__ __forceinline__ void load_v(const T* __restrict__ p, int64_t e, float (&o)[V]) {
  if constexpr (sizeof(T) == 4) {
    const float* q = reinterpret_cast<const float*>(p) + e;
    if constexpr (V == 1) {
      o[0] = ld<NT, f32x1>(q);
    } else {
#pragma unroll
      for (int k = 0; k < V / 4; ++k) {
        const f32x4::type a = ld<NT, f32x4>(q + 4 * k);
        o[4 * k + 0] = a.x; o[4 * k + 1] = a.y; o[4 * k + 2] = a.z; o[4 * k + 3] = a.w;
      }
    }
  } else {
    const uint16_t* q = reinterpret_cast<const uint16_t*>(p) + e;
    if constexpr (V == 1) {
      o[0] = bf16_to_f32(ld<NT, u16x1>(q));
    } else if constexpr (V == 4) {
      const u16x4::type a = ld<NT, u16x4>(q);
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = bf16_to_f32(a[k]);
    } else {
#pragma unroll
      for (int k = 0; k < V / 8; ++k) {
        const u16x8::type a = ld<NT, u16x8>(q + 8 * k);
#pragma unroll
        for (int t = 0; t < 8; ++t) o[8 * k + t] = bf16_to_f32(a[t]);
      }
    }
  }
}

template <typename T, int V, bool NT>
__device__ __forceinline__ void store_v(T* __restrict__ p, int64_t e, const float (&o)[V]) {
  if constexpr (sizeof(T) == 4) {
    float* q = reinterpret_cast<float*>(p) + e;
    if constexpr (V == 1) {
      st<NT, f32x1>(q, o[0]);
    } else {
#pragma unroll
      for (int k = 0; k < V / 4; ++k) {
        const f32x4::type a = {o[4 * k + 0], o[4 * k + 1], o[4 * k + 2], o[4 * k + 3]};
        st<NT, f32x4>(q + 4 * k, a);
      }
    }
  } else {
    uint16_t* q = reinterpret_cast<uint16_t*>(p) + e;
    if constexpr (V == 1) {
      st<NT, u16x1>(q, f32_to_bf16(o[0]));
    } else if constexpr (V == 4) {
      u16x4::type a;
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k] = f32_to_bf16(o[k]);
      st<NT, u16x4>(q, a);
    } else {
#pragma unroll
      for (int k = 0; k < V / 8; ++k) {
        u16x8::type a;
#pragma unroll
        for (int t = 0; t < 8; ++t) a[t] = f32_to_bf16(o[8 * k + t]);
        st<NT, u16x8>(q + 8 * k, a);
      }
    }
  }
}

// Accesses of up to V elements at base + o: all V as one vector access
// (FULL), or the first n < V element by element, zeros for the others (n < 0
// counts from the row's end, which lies past base: at least one element of
// the row follows base).  Loads beyond the row take its last element, so that
// they are all in flight: one after another behind their checks, the loads of
// the last piece made a short row's whole time (mean of 400,000 bf16 x 24
// replicas 20.5 us so, 10 us now).
// base is the same in every lane and o a 32-bit element offset, so an access
// takes a scalar base and one vector register: with a 64-bit element index
// per lane each stream held two registers of address from its load to its
// store.  Rows start at any element (row m at m P), so base + o is aligned
// to its element only; the hardware takes 16-byte accesses at any 4-byte
// (fp32) or 2-byte (bf16) address.
template <typename T>
__device__ __forceinline__ const T* at(const T* base, uint32_t o) {
  return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (uint32_t)(o * (uint32_t)sizeof(T)));
}

template <typename T>
__device__ __forceinline__ T* at(T* base, uint32_t o) {
  return reinterpret_cast<T*>(reinterpret_cast<char*>(base) + (uint32_t)(o * (uint32_t)sizeof(T)));
}

template <bool FULL, typename T, int V, bool NT>
__device__ __forceinline__ void load_n(const T* base, uint32_t o, int32_t n, float (&a)[V]) {
  if constexpr (FULL) {
    load_v<T, V, NT>(at(base, o), 0, a);
  } else {
    // a copy of o that the compiler cannot see through: an address that both
    // paths share would be formed before them in vector registers
    asm("" : "+v"(o));
    const uint32_t last = o + (uint32_t)n - 1;  // of the row
    float b[V][1];
#pragma unroll
    for (int t = 0; t < V; ++t) load_v<T, 1, false>(at(base, o + t < last ? o + t : last), 0, b[t]);
#pragma unroll
    for (int t = 0; t < V; ++t) a[t] = t < n ? b[t][0] : 0.0f;
  }
}

template <bool FULL, typename T, int V, bool NT>
__device__ __forceinline__ void store_n(T* base, uint32_t o, int32_t n, const float (&a)[V]) {
  if constexpr (FULL) {
    store_v<T, V, NT>(at(base, o), 0, a);
  } else {
    asm("" : "+v"(o));  // as in load_n
#pragma unroll
    for (int t = 0; t < V; ++t) {
      const float b[1] = {a[t]};
      if (t < n) store_v<T, 1, false>(at(base, o), t, b);
    }
  }
}

// Elements from `from` to the end of a row, as a 32-bit count (callers
// subtract lane offsets far below 2^30 from it).
__device__ __forceinline__ int32_t left_in_row(int64_t from, int64_t end) {
  const int64_t n = end - from;
  return n > (1 << 30) ? (1 << 30) : n < 0 ? 0 : (int32_t)n;
}

// Where a lane's V elements lie in a piece of which in_row >= V elements are
// in the row: lanes that reach past the row's end take its last V elements,
// which other lanes of the wave hold too.  All of them load before any
// stores, form the same values and store the same, so the last piece of a row
// runs as the others do.  (Element by element, in code of its own that only
// the last piece fetched, it made a short row's time: 100,000 bf16 x 24
// replicas, fused SGDM N = 1 24.3 us; mean of 400,000 bf16 x 24 20.5 us, now
// 7.7 us.)
template <int V>
__device__ __forceinline__ uint32_t slot_in_row(uint32_t o, int32_t in_row) {
  const uint32_t end = (uint32_t)in_row - V;
  return o < end ? o : end;
}

// ------------------------------------------------------ tile -> elements
//
// Workgroups are dispatched round-robin over the 8 XCDs, so with a plain
// tile sequence XCD i works on tiles i, i + 8, ...  The HBM rate of a
// streaming pass depends on how large a contiguous piece each XCD takes in
// turn: pieces of 512 B - 1 KiB per stream spread the XCDs' traffic over
// the memory channels best, 2 KiB pieces worst (about 10 % apart on MI355X
// for the same bytes).  tile_elem() therefore splits a tile of B*V*U
// elements into pieces of C elements and places piece j of tile t at piece
// index ((t / 8) * R + j) * 8 + t % 8 of the row (R = pieces per tile), so
// workgroups on one XCD still take one piece in eight and the pieces of a
// tile are 8 C elements apart.  C = 0 keeps the tile contiguous.  Every
// element of the row belongs to exactly one (tile, slot, thread) for
// tiles < tiles_for<B * V * U, C>(P); elements past P are skipped by the
// callers' bounds checks.
template <int T, int C>
__device__ __forceinline__ int64_t tile_elem(int64_t tile, int local) {
  if constexpr (C == 0) {
    return tile * (int64_t)T + local;
  } else {
    static_assert(T % C == 0, "a tile holds whole pieces");
    constexpr int R = T / C;
    const int64_t piece = ((tile >> 3) * R + local / C) * 8 + (tile & 7);
    return piece * C + local % C;
  }
}

// Number of tiles that cover a row of P elements under tile_elem<T, C>.
template <int T, int C>
__host__ __device__ constexpr int64_t tiles_for(int64_t P) {
  if constexpr (C == 0) {
    return (P + T - 1) / T;
  } else {
    const int64_t pieces = (P + C - 1) / C;
    const int64_t per8 = 8 * (int64_t)(T / C);  // pieces covered by 8 consecutive tiles
    return (pieces + per8 - 1) / per8 * 8;
  }
}

// The tile of this workgroup: tiles are numbered along x, then y, in
// dispatch order (a launch's x extent is limited to 2^32 threads).  One tile
// per workgroup and no loop over tiles: a loop makes the compiler keep every
// stream's base + lane offset in vector registers across it, in place of a
// scalar base and one offset.
__device__ __forceinline__ int64_t launch_tile() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

// ------------------------------------------------------ launch shapes

// Grid of kernels that take launch_tile(): tiles along x, then y, with the
// thread count of x below 2^32 for workgroups of up to 1024.  x is a
// multiple of 16 (or y is 1), so a tile's XCD (dispatch order mod 8) and its
// parity are those of its number, and beyond that rounding every workgroup
// has a tile.  (Whole rows of 2^21 workgroups left 23 % of those of 1.31B x 4
// empty, each with its place on a CU and its LDS: fused step with x due
// 40.3 ms, mean of one state 7.25 ms, against 36.7 and 6.4 ms.)
inline dim3 tile_grid(int64_t tiles, int32_t nz = 1) {
  const int64_t maxx = INT64_C(1) << 21;
  if (tiles < 1) tiles = 1;
  const int64_t y = (tiles + maxx - 1) / maxx;
  const int64_t x = y == 1 ? tiles : ((tiles + y - 1) / y + 15) / 16 * 16;
  return dim3((unsigned)x, (unsigned)y, (unsigned)nz);
}

// The piece of this workgroup in the wave-per-replica kernels, which take
// one piece of every row.  group = 1: pieces in order, so the XCDs take one
// in turn.  group = 8: each XCD takes 8 consecutive pieces with 8 workgroups
// that follow one another on it.  Rows that do not start on 128-byte lines
// share a line between neighbouring pieces; written from two XCDs' L2 caches
// each half goes to memory by itself, so such rows take group = 8
// (row_group; `bytes` of an element, 4 for the fused kernels, most of whose
// streams are fp32).  group = 1 -> 8 on the same buffers: fused Adam N = 2,
// K = 4, x due, 30M + 1 927 -> 858 us, 30M + 8 895 -> 841 us, 30M + 16
// 806 -> 794 us, 30M + 32 (whole lines) 749 -> 774 us; mean K = 4, bf16,
// 80M + 32 243 -> 225 us, fp32, 40M + 4 227 -> 209 us; K = 16, fp32, 40M + 32
// (whole lines) 888 -> 926 us.  Groups of 16 and 32 were equal to 8.  (The
// piece formed by shifts starts a workgroup's loads earlier and was slower:
// 98M x 3 1936 -> 2017 us, 25M x 3 484 -> 500 us.)  Pieces past the row have
// no elements.
__device__ __forceinline__ int64_t group_piece(int32_t group) {
  const int64_t t = launch_tile();
  if (group == 1) return t;
  return t / (8 * group) * (8 * group) + (t & 7) * group + (t >> 3) % group;
}
inline int32_t row_group(int64_t P, int bytes) { return P * bytes % 128 == 0 ? 1 : 8; }
inline dim3 group_grid(int64_t pieces, int32_t group, int32_t nz = 1) {
  const int64_t span = group == 1 ? 1 : 8 * group;
  return tile_grid((pieces + span - 1) / span * span, nz);
}

// Workgroups per CU of the streaming kernels.  Bytes in flight beyond what
// covers the HBM's latency only spread the accesses over more DRAM pages:
// about 40 KiB of loads per CU ran fastest for every mix of streams, against
// up to 192 KiB at full occupancy.  A launch limits the workgroups that a CU
// holds at once by asking for LDS it does not use: 160 KiB per CU, in units
// of 1280 bytes; the limit asks for 51 of them at most, which leaves two.
// Passes that load less than kResidentMin bytes hit the 256 MB MALL more than the
// HBM and keep every wave that the CUs hold (Adam N = 3, 4 replicas, limited
// against not: 88 MB 15.5 us against 15.1 us, 176 MB 29.3 us against
// 30.3 us, 352 MB 57.2 us against 59.2 us).
constexpr int64_t kResidentMin = INT64_C(64) << 20;
constexpr size_t resident_lds(int n) { return (size_t)(128 / n > 51 ? 51 : 128 / n) * 1280; }

// Workgroups per CU of the steps with one wave per replica, for `bytes`
// loaded per element.  Their barriers ask for more bytes in flight than the
// plain step, and the fewer streams a form has the more waves those take:
// from no limit at two 2-byte and one 4-byte stream (8 bytes) to 12 waves at
// six 4-byte ones (72 KiB of loads).  More also where every state is due
// (`many`: more than half; all stores wait for the exchange), where x takes
// the OuterOpt (`outer`, whose parameters are loaded with the tile) and where
// the clip norm has just left the gradients in the MALL (`clip`).  At least
// two workgroups, which K > 8 has by its size (one took 0.86 to 0.96 of the
// rate), unless their LDS does not allow it (more than 80 KiB each: six due
// states of 14 or more rows).  The table is the best of 2, 3, 4, 5, 6, 8, 10
// and 14 workgroups and no limit over K = 2, 3, 4, 5, 6, 8, seven forms, x or
// all states due, with clipping and without, 0.3 and 1.2 GB loaded, same
// buffers of an MI355X: within 1 % of each row's best on average, where one
// value per form was 1 to 4 % off and with clipping up to 17 % (SGDM N = 1
// fp32 K = 4 all due, clipped, 1.2 GB: 400 us at 18 waves, 348 us at 28; Adam
// N = 1 K = 4 408 us at 16, 349 us at 24; without clipping SGDM N = 2 K = 6
// three workgroups 361 us, two 347 us, K = 3 six 346 us, unlimited 352 us).
// Under the OuterOpt and K > 4 the waves are rounded up to a whole workgroup
// (Adam N = 1 K = 7, 1.2 GB: two 398 us, three 347 us; N = 2 K = 6
// 386 / 361 us).  12 waves against no limit: Adam N = 3 354M x 4 10.54 against
// 11.39 ms in one placement of the buffers, 9.94 against 9.93 ms in another.
constexpr int wave_resident(int K, int bytes, bool many = false, bool clip = false, bool outer = false) {
  int waves = 12;
  if (bytes <= 8) waves = 32;
  else if (bytes <= 10) waves = many && clip ? 28 : 24;
  else if (bytes <= 14) waves = many ? (clip ? 28 : 24) : clip ? 24 : outer ? 21 : 18;
  else if (bytes <= 16) waves = many ? (clip ? 24 : K > 5 ? 12 : 18) : clip ? 21 : outer ? 18 : 16;
  else if (bytes <= 22) waves = many && clip ? 18 : 14;
  else if (many && clip) waves = 16;
  if (outer && K > 4 && waves < 32) waves += K - 1;
  return waves / K > 2 ? waves / K : 2;
}

// The local step's workgroups for `bytes` loaded per element (four elements
// per lane): two waves each, for steps of the limit that are fine enough,
// and from six 4-byte streams on two workgroups of four waves (354M x 4
// Adam N = 3: 9.95 ms, against 10.29 ms with four of two waves).  At full
// occupancy -> limited, on the same buffers of an MI355X: 16.8M x 4 Adam
// N = 3 497 -> 457 us, 354M x 4 11.02 -> 10.09 ms; 124M x 8 ADOPT N = 2 in
// bf16 4.97 -> 4.58 ms; 124M x 16 SGDM N = 2 9.28 -> 8.59 ms; 60M x 2 Adam
// N = 1 564 -> 505 us.
struct StepLaunch {
  int threads;   // of a workgroup
  int resident;  // workgroups per CU
  int bytes;     // loaded per element
};
constexpr StepLaunch step_launch(int bytes) {
  if (bytes > 20) return {256, 2, bytes};
  return {128, (40 * 1024 / 2 + 128 * bytes) / (256 * bytes), bytes};
}

// ------------------------------------------------------------ OuterOpt

// Nesterov OuterOpt at an averaging event of x (xo == nullptr: plain
// averaging).  xo, mom: fp32 [P] outer parameters and outer momentum.
struct OuterParams {
  float* xo;
  float* mom;
  float lr;        // outer learning rate
  float mu;        // outer momentum
  int32_t update;  // 0: xo and mom are only read (the outer step of this s already ran)
};

// xbar (the workers' mean) becomes the value every worker restarts from:
// d = xo - xbar; mom = mu mom + d; xo = xo - lr (d + mu mom).
template <int V>
__device__ __forceinline__ void outer_step(const OuterParams& o, int64_t e, float (&xbar)[V]) {
#pragma clang fp contract(off)
  if (o.xo == nullptr || !o.update) return;
  float xo[V], b[V];
  load_v<float, V, false>(o.xo, e, xo);
  load_v<float, V, false>(o.mom, e, b);
#pragma unroll
  for (int t = 0; t < V; ++t) {
    const float d = xo[t] - xbar[t];
    b[t] = __builtin_fmaf(o.mu, b[t], d);
    xo[t] = __builtin_fmaf(-o.lr, __builtin_fmaf(o.mu, b[t], d), xo[t]);
    xbar[t] = xo[t];
  }
  store_v<float, V, false>(o.xo, e, xo);
  store_v<float, V, false>(o.mom, e, b);
}

// The same over the n elements of a row's last piece (FULL: all V).
template <bool FULL, int V>
__device__ __forceinline__ void outer_step_n(const OuterParams& o, int64_t e, int32_t n, float (&xbar)[V]) {
  if constexpr (FULL) {
    outer_step<V>(o, e, xbar);
  } else {
#pragma unroll
    for (int t = 0; t < V; ++t)
      if (t < n) {
        float a[1] = {xbar[t]};
        outer_step<1>(o, e + t, a);
        xbar[t] = a[0];
      }
  }
}

// The outer parameters and momentum of the elements that a thread averages,
// loaded with the tile: loaded after the mean, their latency was part of
// every workgroup's chain of barriers.  U elements per thread at most.
template <int U>
struct OuterAhead {
  float xo[U], mom[U];
};

// outer_step's update of element e with its inputs already loaded.
__device__ __forceinline__ float outer_element(const OuterParams& o, int64_t e, float xo, float mom, float xbar) {
#pragma clang fp contract(off)
  const float d = xo - xbar;
  const float b = __builtin_fmaf(o.mu, mom, d);
  xo = __builtin_fmaf(-o.lr, __builtin_fmaf(o.mu, b, d), xo);
  o.xo[e] = xo;
  o.mom[e] = b;
  return xo;
}

// ------------------------------------------------------------ local step

// The update count kept on the device for graph replay (the layout of
// mtdao_device_step): a launch at offset k after the last advance takes
// update s = s + k; k_device_step_add moves s on by a window of calls.
struct DeviceStep {
  int64_t s;
  int64_t reserved;
};

// b^s for s >= 0 by repeated squaring in plain IEEE double multiplies, so
// host and device code compute the same bits.
__host__ __device__ inline double pow_steps(double b, int64_t s) {
#pragma clang fp contract(off)
  double r = 1.0, a = b;
  while (s > 0) {
    if (s & 1) r = r * a;
    a = a * a;
    s >>= 1;
  }
  return r;
}

// Hyper-parameters the step-dependent scalars are formed from.
struct BiasCorrection {
  float beta[kMaxN];
  float omega[kMaxN];
  float beta2;
  int32_t n;
  int32_t on;  // Adam with bias correction
};

// w_j = omega_j / (1 - beta_j^s) and 1 / (1 - beta_2^s) (omega_j and 1
// without correction) in double, rounded once to fp32; the same code on
// the host (eager calls) and in the kernels (device-side s).
__host__ __device__ inline void step_scalars(const BiasCorrection& c, int64_t s, float* w, float* inv_bc2) {
#pragma clang fp contract(off)
  for (int j = 0; j < c.n; ++j)
    w[j] = (float)(c.on ? (double)c.omega[j] / (1.0 - pow_steps((double)c.beta[j], s)) : (double)c.omega[j]);
  *inv_bc2 = (float)(c.on ? 1.0 / (1.0 - pow_steps((double)c.beta2, s)) : 1.0);
}

__global__ __launch_bounds__(64) void k_device_step_set(DeviceStep* __restrict__ d, int64_t s) {
  if (threadIdx.x == 0) d->s = s;
}

__global__ __launch_bounds__(64) void k_device_step_add(DeviceStep* __restrict__ d, int64_t n) {
  if (threadIdx.x == 0) d->s = d->s + n;
}

// Per-launch scalars, prepared on the host in double and rounded to fp32.
struct StepParams {
  void* x;                 // [K][P] params (XT)
  const void* g;           // [K][P] gradients (GT)
  float* u[kMaxN];         // [K][P] first moments
  float* v;                // [K][P] second moment (Adam, ADOPT)
  const float* scale;      // [K] global-norm clip factors, or nullptr
  int64_t P;               // row length
  int64_t n;               // k_local_step: K P, elements of a state
  double rp;               // 1 / P
  int32_t replicas;        // K
  int32_t group;           // wave-per-replica kernels: group_piece
  float beta[kMaxN];       // beta_{1,j}
  float omb[kMaxN];        // 1 - beta_{1,j}
  float w[kMaxN];          // omega_j (times 1/(1 - beta_{1,j}^s) for bias-corrected Adam)
  float gw;                // 1 - sum_j omega_j: weight of the current gradient
  float beta2, omb2;       // beta_2, 1 - beta_2
  float inv_bc2;           // 1/(1 - beta_2^s) (Adam with bias correction), else 1
  float eps;
  float lr;                // eta_t
  float clip;              // ADOPT c_t (<= 0: no clamp)
  OuterParams outer;       // OuterOpt applied when x is averaged
  // device-side update number (graph replay): when dev is non-null the
  // update is s = dev->s + dev_k, and lr, clip, w and inv_bc2 are formed
  // from it: eta_t = lr_table[s - 1], c_t = clip_table[s - 1] (the last
  // entries beyond table_len; clip off without a table), corrections from bc
  const DeviceStep* dev;
  int64_t dev_k;
  const float* lr_table;
  const float* clip_table;
  int64_t table_len;
  BiasCorrection bc;
};

// The value that lane l (the same for the whole wave) holds, in a scalar
// register: the fp64 arithmetic below runs in the vector ALU, whose results
// would otherwise each hold a vector register for the rest of the kernel.
__device__ __forceinline__ float lane_value(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

// The launch's scalars: those of the argument block, or those of the
// device-side update number when it is given (every wave forms them).  Lane
// j forms the weight of moment j (lane n: 1 / (1 - beta_2^s)) with
// step_scalars' operations, and the results are read across: one power and
// one quotient per wave in place of n + 1 in turn.  Called where every lane
// of the wave is active.
__device__ __forceinline__ StepParams device_scalars(const StepParams& p0) {
#pragma clang fp contract(off)
  if (p0.dev == nullptr) return p0;
  StepParams p = p0;
  const int64_t s = load_uniform(&p0.dev->s) + p0.dev_k;
  const int64_t i = (s < p0.table_len ? s : p0.table_len) - 1;
  p.lr = load_uniform(p0.lr_table + i);
  p.clip = p0.clip_table != nullptr ? load_uniform(p0.clip_table + i) : 0.0f;
  const int lane = threadIdx.x & 63;
  float beta = p0.bc.beta2, omega = 1.0f;
#pragma unroll
  for (int j = 0; j < kMaxN; ++j) {
    float b = p0.bc.beta[j], o = p0.bc.omega[j];
    asm("" : "+s"(b), "+s"(o));  // selects of values: not a load from a selected address
    const bool mine = j < p0.bc.n && lane == j;
    beta = mine ? b : beta;
    omega = mine ? o : omega;
  }
  const float w = (float)(p0.bc.on ? (double)omega / (1.0 - pow_steps((double)beta, s)) : (double)omega);
#pragma unroll
  for (int j = 0; j < kMaxN; ++j)
    if (j < p0.bc.n) p.w[j] = lane_value(w, j);
  p.inv_bc2 = lane_value(w, p0.bc.n);
  return p;
}

// The update of one element of one replica (the loop body of Algorithm 1, 2
// or 3).  x, u[0..N), v hold the stored values on entry and the updated
// values on exit; graw is the stored gradient and sc the replica's clip
// factor.  Contraction is pinned (explicit fma, no implicit fusion) so
// every kernel that calls this computes bit-identical values.
template <int FORM, int N, int ORDER>
__device__ __forceinline__ void update_element(const StepParams& p, float sc, float graw, float& x,
                                               float (&u)[N], float& v) {
#pragma clang fp contract(off)
  if constexpr (FORM == kAdam) {
    const float gh = sc * graw;
    float num = p.gw * gh;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      u[j] = __builtin_fmaf(p.beta[j], u[j], p.omb[j] * gh);
      num = __builtin_fmaf(p.w[j], u[j], num);
    }
    v = __builtin_fmaf(p.beta2, v, p.omb2 * (gh * gh));
    const float den = __builtin_sqrtf(v * p.inv_bc2) + p.eps;
    x = __builtin_fmaf(-p.lr, num / den, x);
  } else if constexpr (FORM == kAdopt) {
    float gn;
    if constexpr (ORDER == kPrev) {
      gn = graw / (__builtin_sqrtf(v) + p.eps);
      v = __builtin_fmaf(p.beta2, v, p.omb2 * (graw * graw));
    } else {
      v = __builtin_fmaf(p.beta2, v, p.omb2 * (graw * graw));
      gn = graw / (__builtin_sqrtf(v) + p.eps);
    }
    if (p.clip > 0.0f) gn = gn > p.clip ? p.clip : (gn < -p.clip ? -p.clip : gn);
    float delta = p.gw * gn;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      u[j] = __builtin_fmaf(p.beta[j], u[j], p.omb[j] * gn);
      delta = __builtin_fmaf(p.w[j], u[j], delta);
    }
    x = __builtin_fmaf(-p.lr, delta, x);
  } else {
    const float gh = sc * graw;
    float delta = p.gw * gh;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      u[j] = __builtin_fmaf(p.beta[j], u[j], p.omb[j] * gh);
      delta = __builtin_fmaf(p.w[j], u[j], delta);
    }
    x = __builtin_fmaf(-p.lr, delta, x);
  }
}

// The row that holds element e of a [K][P] buffer taken as a flat array:
// e / P for 0 <= e < 2^40, rp = 1 / P in fp64.  e is exact
// in fp64 and the product is off by less than one, so one correction each
// way gives the quotient.
__device__ __forceinline__ int64_t row_of(int64_t e, int64_t P, double rp) {
  int64_t m = (int64_t)((double)e * rp);
  if (m * P > e) --m;
  if ((m + 1) * P <= e) ++m;
  return m;
}

// One update of all elements of all replicas (Algorithm 1, 2 or 3 body).
// The update is element-wise, so the [K][P] buffers are taken as flat arrays
// of n = K P elements: every access starts at a multiple of V elements from
// a 16-byte aligned base whatever P is, and only the clip factor needs the
// row of an element.
//   FORM       kAdam / kAdopt / kSgdm
//   N          number of first moments
//   XT, GT     storage of params / gradients (float or bf16)
//   V          elements per thread
//   NTM        bit 0: nontemporal loads, bit 1: nontemporal stores
//   ORDER      ADOPT normalisation order (kPrev: v from before this step)
//   ROWS       clip factors: kNoScale, kTwoRows (rows of at least a wave's
//              64 V elements, so a wave meets two rows at most) or kAnyRows
//   B          threads of a workgroup
// A wave's elements are one piece of the tile -> element map (tile_elem).
// The launch limits the workgroups that a CU holds at once (resident_lds in
// the host code): the HBM serves the fewest bytes that cover its latency
// faster than all that the CUs could keep in flight.
enum ScaleRows { kNoScale = 0, kTwoRows = 1, kAnyRows = 2 };

template <int FORM, int N, typename XT, typename GT, int V, int NTM, int ORDER, int ROWS, int B>
__global__ __launch_bounds__(B) void k_local_step(StepParams p0) {
  constexpr bool NTL = (NTM & 1) != 0, NTS = (NTM & 2) != 0;
  constexpr int C = 64 * V;

  XT* x = reinterpret_cast<XT*>(p0.x);
  const GT* g = reinterpret_cast<const GT*>(p0.g);
  float* u[kMaxN];
#pragma unroll
  for (int j = 0; j < kMaxN; ++j) u[j] = p0.u[j < N ? j : 0];
  float* v = FORM != kSgdm ? p0.v : p0.u[0];
  const int64_t total = p0.n;
  in_sgprs(x, g, u[0], v);
  if constexpr (N > 1) in_sgprs(u[1], u[2], u[3], v);

  const int64_t tile = launch_tile();
  // the tile's first element, and this thread's place after it
  const int64_t base = tile_elem<B * V, C>(tile, 0);
  const uint32_t o = (uint32_t)tile_elem<B * V, C>(0, (int)threadIdx.x * V);
  const int32_t ow = __builtin_amdgcn_readfirstlane((int32_t)o);
  const int32_t nw = left_in_row(base, total) - ow, n = left_in_row(base, total) - (int32_t)o;
  x += base;
  g += base;
#pragma unroll
  for (int j = 0; j < N; ++j) u[j] += base;
  if constexpr (FORM != kSgdm) v += base;
  // the wave's piece: whole (one uniform branch, so that the vector path has
  // no merges with the other between its loads and its stores), or the last
  // one of the buffers
  auto piece = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    float gv[V], xv[V], uv[N][V], vv[V];
    // issue every load of the tile before any arithmetic
    load_n<F, GT, V, NTL>(g, o, n, gv);
    load_n<F, XT, V, NTL>(x, o, n, xv);
#pragma unroll
    for (int j = 0; j < N; ++j) load_n<F, float, V, NTL>(u[j], o, n, uv[j]);
    if constexpr (FORM != kSgdm) load_n<F, float, V, NTL>(v, o, n, vv);
    // clip factors: s0 for the row of the wave's first element, s1 from
    // `left` elements after this thread's first, where the next row starts
    float s0 = 1.0f, s1 = 1.0f;
    int32_t left = V;
    if constexpr (ROWS == kTwoRows) {
      const int32_t m = __builtin_amdgcn_readfirstlane((int32_t)row_of(base + ow, p0.P, p0.rp));
      s0 = load_uniform(p0.scale + m);
      s1 = load_uniform(p0.scale + (m + 1 < p0.replicas ? m + 1 : m));
      left = left_in_row(base, (m + 1) * p0.P) - (int32_t)o;
    }
    // the step-dependent scalars after the loads are in flight (from the
    // device-side update number when there is one)
    const StepParams p = device_scalars(p0);
#pragma unroll
    for (int t = 0; t < V; ++t) {
      float uu[N];
#pragma unroll
      for (int j = 0; j < N; ++j) uu[j] = uv[j][t];
      float vt = (FORM != kSgdm) ? vv[t] : 0.0f;
      float sc = 1.0f;
      if constexpr (ROWS == kTwoRows) sc = t < left ? s0 : s1;
      if constexpr (ROWS == kAnyRows) sc = t < n ? p0.scale[row_of(base + o + t, p0.P, p0.rp)] : 1.0f;
      update_element<FORM, N, ORDER>(p, sc, gv[t], xv[t], uu, vt);
#pragma unroll
      for (int j = 0; j < N; ++j) uv[j][t] = uu[j];
      if constexpr (FORM != kSgdm) vv[t] = vt;
    }
    store_n<F, XT, V, NTS>(x, o, n, xv);
#pragma unroll
    for (int j = 0; j < N; ++j) store_n<F, float, V, NTS>(u[j], o, n, uv[j]);
    if constexpr (FORM != kSgdm) store_n<F, float, V, NTS>(v, o, n, vv);
  };
  if (nw >= C) piece(BoolC<true>{});
  else if (nw > 0) piece(BoolC<false>{});
}

// Value a state holds once stored: bf16 parameters are rounded.
template <typename T>
__device__ __forceinline__ float as_stored(float a) {
  if constexpr (sizeof(T) == 2) return bf16_to_f32(f32_to_bf16(a));
  else return a;
}

// The replica mean of one element, shared by every averaging kernel:
// S^0 + (sum_{m>=1} (S^m - S^0)) / K, the differences summed in fp64 in
// replica order and the result rounded to fp32 once.  (An fp32 running sum
// loses up to about (K - 1) 2^-24 of the rows' spread, which at large K is
// more than the mean itself carries when the rows nearly cancel.)  Identical
// rows give S^0 back exactly.  rk = 1 / K in fp64.
__device__ __forceinline__ void mean_add(double& d, float a, float s0) { d += (double)a - (double)s0; }
__device__ __forceinline__ float mean_of(float s0, double d, double rk) {
  return (float)__builtin_fma(d, rk, (double)s0);
}

// Local update of every replica followed by the replica mean of the states
// in `mask` (bit 0 = x, bit j = u^j, bit N+1 = v), in one pass.  A thread
// owns V columns of every replica: it updates replica 0..K-1 in order,
// stores the states that are not due, and accumulates the due ones as
// S^0 + (sum_{m>=1} (S^m - S^0)) / K from their stored values -- the same
// arithmetic, in the same order, as k_local_step followed by
// k_replica_mean, so both paths give bit-identical results -- then writes
// that mean to all K rows.  The separate mean pass (2 K sizeof(T) bytes
// per element per due state) disappears.
template <int FORM, int N, typename XT, typename GT, int V, int NTM, int ORDER>
__global__ __launch_bounds__(kBlock) void k_local_step_sync(StepParams p0, uint32_t mask, int32_t K) {
  const StepParams p = device_scalars(p0);
  constexpr bool NTL = (NTM & 1) != 0, NTS = (NTM & 2) != 0;
  const bool sync_x = (mask & 1u) != 0;
  bool sync_u[N];
#pragma unroll
  for (int j = 0; j < N; ++j) sync_u[j] = ((mask >> (j + 1)) & 1u) != 0;
  const bool sync_v = FORM != kSgdm && ((mask >> (N + 1)) & 1u) != 0;
  XT* __restrict__ x = reinterpret_cast<XT*>(p.x);
  const GT* __restrict__ g = reinterpret_cast<const GT*>(p.g);
  const double rk = 1.0 / (double)K;

  // a wave's elements are one piece of the tile
  const int64_t base = tile_elem<kBlock * V, 64 * V>(launch_tile(), 0);
  const uint32_t lane_o = (uint32_t)tile_elem<kBlock * V, 64 * V>(0, (int)threadIdx.x * V);
  const int32_t in_row = left_in_row(base, p.P);
  const int32_t n = in_row - (int32_t)lane_o, nw = __builtin_amdgcn_readfirstlane(n);
  auto piece = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    const uint32_t o = F ? slot_in_row<V>(lane_o, in_row) : lane_o;
    float x0[V], u0[N][V], v0[V];
    double dx[V], du[N][V], dv[V];
#pragma unroll
    for (int t = 0; t < V; ++t) {
      dx[t] = 0.0;
      dv[t] = 0.0;
#pragma unroll
      for (int j = 0; j < N; ++j) du[j][t] = 0.0;
    }
    for (int32_t m = 0; m < K; ++m) {
      const int64_t r = (int64_t)m * p.P + base;
      float gv[V], xv[V], uv[N][V], vv[V];
      load_n<F, GT, V, NTL>(g + r, o, n, gv);
      load_n<F, XT, V, NTL>(x + r, o, n, xv);
#pragma unroll
      for (int j = 0; j < N; ++j) load_n<F, float, V, NTL>(p.u[j] + r, o, n, uv[j]);
      if constexpr (FORM != kSgdm) load_n<F, float, V, NTL>(p.v + r, o, n, vv);
      const float sc = (FORM != kAdopt && p.scale != nullptr) ? load_uniform(p.scale + m) : 1.0f;
#pragma unroll
      for (int t = 0; t < V; ++t) {
        float uu[N];
#pragma unroll
        for (int j = 0; j < N; ++j) uu[j] = uv[j][t];
        float vt = (FORM != kSgdm) ? vv[t] : 0.0f;
        update_element<FORM, N, ORDER>(p, sc, gv[t], xv[t], uu, vt);
        xv[t] = as_stored<XT>(xv[t]);
#pragma unroll
        for (int j = 0; j < N; ++j) uv[j][t] = uu[j];
        vv[t] = vt;
      }
      // states not due: store now; due: accumulate the shifted sum
      if (sync_x) {
#pragma unroll
        for (int t = 0; t < V; ++t) {
          if (m == 0) x0[t] = xv[t];
          else mean_add(dx[t], xv[t], x0[t]);
        }
      } else {
        store_n<F, XT, V, NTS>(x + r, o, n, xv);
      }
#pragma unroll
      for (int j = 0; j < N; ++j) {
        if (sync_u[j]) {
#pragma unroll
          for (int t = 0; t < V; ++t) {
            if (m == 0) u0[j][t] = uv[j][t];
            else mean_add(du[j][t], uv[j][t], u0[j][t]);
          }
        } else {
          store_n<F, float, V, NTS>(p.u[j] + r, o, n, uv[j]);
        }
      }
      if constexpr (FORM != kSgdm) {
        if (sync_v) {
#pragma unroll
          for (int t = 0; t < V; ++t) {
            if (m == 0) v0[t] = vv[t];
            else mean_add(dv[t], vv[t], v0[t]);
          }
        } else {
          store_n<F, float, V, NTS>(p.v + r, o, n, vv);
        }
      }
    }
    // the means, written to every replica row
    if (sync_x) {
#pragma unroll
      for (int t = 0; t < V; ++t) x0[t] = mean_of(x0[t], dx[t], rk);
      outer_step_n<F, V>(p.outer, base + o, n, x0);
      for (int32_t m = 0; m < K; ++m) store_n<F, XT, V, NTS>(x + (int64_t)m * p.P + base, o, n, x0);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (!sync_u[j]) continue;
#pragma unroll
      for (int t = 0; t < V; ++t) u0[j][t] = mean_of(u0[j][t], du[j][t], rk);
      for (int32_t m = 0; m < K; ++m) store_n<F, float, V, NTS>(p.u[j] + (int64_t)m * p.P + base, o, n, u0[j]);
    }
    if constexpr (FORM != kSgdm) {
      if (sync_v) {
#pragma unroll
        for (int t = 0; t < V; ++t) v0[t] = mean_of(v0[t], dv[t], rk);
        for (int32_t m = 0; m < K; ++m) store_n<F, float, V, NTS>(p.v + (int64_t)m * p.P + base, o, n, v0);
      }
    }
  };
  if (nw >= V) piece(BoolC<true>{});
  else if (nw > 0) piece(BoolC<false>{});  // fewer elements than a slot
}

// The wave-per-replica kernels (1 < K <= kWaveMaxK): a workgroup of K waves
// (or K / R, R rows per wave) takes one piece of 64 V elements of every row,
// so every row has its own loads in flight, and values to be averaged meet
// in LDS as [K][64 V] floats in element order.
constexpr int kWaveMaxK = 16;
constexpr int kPieceMaxU = 2;  // elements of a 4-element-per-lane piece per thread at K = 2

// Averages `states` stages of E elements that lie back to back in LDS, each
// [K][E]: element c's mean, in replica order with mean_add and mean_of,
// replaces its row 0 value.  Threads take (stage, element) pairs in turn, so
// all waves of the workgroup share the work.  With `outer` (and `ahead`
// loaded by outer_ahead) stage 0 is x and takes the OuterOpt.
template <int E, int U>
__device__ __forceinline__ void average_stages(float* lds, int32_t K, int32_t states, int32_t in_row, double rk,
                                               const OuterParams& o, bool outer, const OuterAhead<U>& ahead,
                                               int64_t e0) {
  auto mean = [&](int32_t j) {
    float* q = lds + (j / E) * (K * E) + j % E;
    const float s0 = q[0];
    double d = 0.0;
#pragma unroll 4
    for (int32_t m = 1; m < K; ++m) mean_add(d, q[m * E], s0);
    return mean_of(s0, d, rk);
  };
  int32_t j = threadIdx.x;
  if (outer) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (j < E) {
        if (j < in_row) lds[j] = outer_element(o, e0 + j, ahead.xo[i], ahead.mom[i], mean(j));
        j += blockDim.x;
      }
    }
  }
  for (; j < states * E; j += blockDim.x)
    if (j % E < in_row) lds[(j / E) * (K * E) + j % E] = mean(j);
}

// The outer inputs of elements e0 + threadIdx.x, + blockDim.x, ... below E.
template <int E, int U>
__device__ __forceinline__ void outer_ahead(const OuterParams& o, int64_t e0, int32_t in_row, OuterAhead<U>& a) {
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const int32_t j = (int32_t)threadIdx.x + i * (int32_t)blockDim.x;
    if (j < E && j < in_row) {
      a.xo[i] = o.xo[e0 + j];
      a.mom[i] = o.mom[e0 + j];
    }
  }
}

// V floats at p in LDS, 16-byte aligned.
typedef float lds_f32x4 __attribute__((ext_vector_type(4)));
template <int V>
__device__ __forceinline__ void lds_put(float* p, const float (&a)[V]) {
#pragma unroll
  for (int k = 0; k < V / 4; ++k)
    reinterpret_cast<lds_f32x4*>(p)[k] = lds_f32x4{a[4 * k], a[4 * k + 1], a[4 * k + 2], a[4 * k + 3]};
}
template <int V>
__device__ __forceinline__ void lds_get(const float* p, float (&a)[V]) {
#pragma unroll
  for (int k = 0; k < V / 4; ++k) {
    const lds_f32x4 q = reinterpret_cast<const lds_f32x4*>(p)[k];
    a[4 * k] = q.x; a[4 * k + 1] = q.y; a[4 * k + 2] = q.z; a[4 * k + 3] = q.w;
  }
}

// The fused step + mean with one wavefront per replica (blockDim = 64 K):
// lane l of wave m updates elements [4 l, 4 l + 4) of its piece of row m
// exactly like the plain step.  States not due are stored at once; the due
// ones are staged in LDS together (dynamic LDS of K * 64 V floats per due
// state), averaged by all waves between two barriers, and every wave stores
// the means to its row.  Every thread reaches the barriers, also in the last
// piece of a row.
template <int FORM, int N, typename XT, typename GT, int V, int NTM, int ORDER>
__global__ __launch_bounds__(64 * kWaveMaxK) __attribute__((amdgpu_waves_per_eu(8)))
void k_local_step_sync_waves(StepParams p0, uint32_t mask, int32_t K) {
  constexpr bool NTL = (NTM & 1) != 0, NTS = (NTM & 2) != 0;
  constexpr int NS = 2 + N, E = 64 * V;  // x, u^1..u^N, v
  extern __shared__ __align__(16) float stage[];
  const int32_t m = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
  const int64_t e0 = group_piece(p0.group) * E, row = (int64_t)m * p0.P + e0;
  const uint32_t o = (threadIdx.x & 63) * V;
  const int32_t in_row = left_in_row(e0, p0.P), n = in_row - (int32_t)o;
  if (in_row == 0) return;  // a whole workgroup past the row
  XT* x = reinterpret_cast<XT*>(p0.x) + row;
  const GT* g = reinterpret_cast<const GT*>(p0.g) + row;
  float* u[N];
#pragma unroll
  for (int j = 0; j < N; ++j) u[j] = p0.u[j] + row;
  float* v = FORM != kSgdm ? p0.v + row : nullptr;

  auto piece = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    float gv[V], val[NS][V];  // x, u^j, v of this lane's elements
    load_n<F, GT, V, NTL>(g, o, n, gv);
    load_n<F, XT, V, NTL>(x, o, n, val[0]);
#pragma unroll
    for (int j = 0; j < N; ++j) load_n<F, float, V, NTL>(u[j], o, n, val[1 + j]);
    if constexpr (FORM != kSgdm) load_n<F, float, V, NTL>(v, o, n, val[NS - 1]);
    const bool outer = (mask & 1u) != 0 && p0.outer.xo != nullptr;
    OuterAhead<kPieceMaxU> ahead;
    if (outer) outer_ahead<E>(p0.outer, e0, in_row, ahead);
    const float sc = (FORM != kAdopt && p0.scale != nullptr) ? load_uniform(p0.scale + m) : 1.0f;
    // the step-dependent scalars after the loads are in flight
    const StepParams p = device_scalars(p0);
#pragma unroll
    for (int t = 0; t < V; ++t) {
      float uu[N];
#pragma unroll
      for (int j = 0; j < N; ++j) uu[j] = val[1 + j][t];
      float vt = (FORM != kSgdm) ? val[NS - 1][t] : 0.0f;
      update_element<FORM, N, ORDER>(p, sc, gv[t], val[0][t], uu, vt);
      val[0][t] = as_stored<XT>(val[0][t]);
#pragma unroll
      for (int j = 0; j < N; ++j) val[1 + j][t] = uu[j];
      val[NS - 1][t] = vt;
    }
    auto put = [&](int k, const float (&a)[V]) {
      if (k == 0) store_n<F, XT, V, NTS>(x, o, n, a);
      else if (k == NS - 1) store_n<F, float, V, NTS>(v, o, n, a);
      else store_n<F, float, V, NTS>(u[k - 1 < N ? k - 1 : 0], o, n, a);
    };
    int32_t due = 0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (FORM == kSgdm && k == NS - 1) continue;
      if ((mask >> k) & 1u) lds_put<V>(stage + (due++ * K + m) * E + o, val[k]);
      else put(k, val[k]);
    }
    __syncthreads();
    average_stages<E>(stage, K, due, in_row, 1.0 / (double)K, p0.outer, outer, ahead, e0);
    __syncthreads();
    due = 0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (FORM == kSgdm && k == NS - 1) continue;
      if (!((mask >> k) & 1u)) continue;
      float mean[V];
      lds_get<V>(stage + due++ * K * E + o, mean);
      put(k, mean);
    }
  };
  if (in_row >= E) piece(BoolC<true>{});
  else piece(BoolC<false>{});
}

// The same step with one exchange per due state: each is staged (column t of
// the piece at [t][lane]), averaged by waves t mod K and stored before the
// next is.  For K > 8 and row lengths that are a multiple of V, where the
// staging of all due states together ran slower: the two 16-wave workgroups
// of a CU cannot be fewer, and holding every state back until the one
// exchange bunches their stores (SGDM N = 2, K = 16, all due, 60M: 4.89 ms,
// staged together 4.96 ms; with x due, Adam N = 3, 20M: 2.70 against
// 2.75 ms).  Other lengths take the kernel above (16M + 1: 1.65 ms, against
// 2.72 ms for one element per lane).
template <int FORM, int N, typename XT, typename GT, int V, int NTM, int ORDER>
__global__ __launch_bounds__(64 * kWaveMaxK) __attribute__((amdgpu_waves_per_eu(8)))
void k_local_step_sync_waves_rounds(StepParams p0, uint32_t mask, int32_t K) {
  constexpr bool NTL = (NTM & 1) != 0, NTS = (NTM & 2) != 0;
  // The device-side update number's scalars take a few dozen fp64
  // operations.  Formed after a tile's loads are issued, their latency is
  // hidden, but their temporaries meet the loaded values: with six or more
  // streams loaded that exceeded the 64-register budget and spilled, so
  // those forms take them once per workgroup before any load.
  constexpr bool kEarly = 2 + N + (FORM != kSgdm ? 1 : 0) >= 6;
  const StepParams early = kEarly ? device_scalars(p0) : p0;
  constexpr int NS = 2 + N;  // x, u^1..u^N, v
  __shared__ float lds[kWaveMaxK][64 * V];
  const int32_t m = threadIdx.x >> 6, lane = threadIdx.x & 63;
  XT* __restrict__ x = reinterpret_cast<XT*>(p0.x);
  const GT* __restrict__ g = reinterpret_cast<const GT*>(p0.g);
  const double rk = 1.0 / (double)K;
  // m is the same in every lane of a wave: readfirstlane makes that visible
  const float sc =
      (FORM != kAdopt && p0.scale != nullptr) ? load_uniform(p0.scale + __builtin_amdgcn_readfirstlane(m)) : 1.0f;

  const int64_t tile = launch_tile();
  const int64_t e = tile * (int64_t)(64 * V) + (int64_t)lane * V;
  if (tile * (int64_t)(64 * V) >= p0.P) return;  // a whole workgroup past the row
  const bool in = e < p0.P;
  const int64_t r = (int64_t)m * p0.P + e;
  float val[NS][V];  // updated x, u^j, v of this lane's elements
  float gv[V], uv[N][V];
  if (in) {
    load_v<GT, V, NTL>(g, r, gv);
    load_v<XT, V, NTL>(x, r, val[0]);
#pragma unroll
    for (int j = 0; j < N; ++j) load_v<float, V, NTL>(p0.u[j], r, uv[j]);
    if constexpr (FORM != kSgdm) load_v<float, V, NTL>(p0.v, r, val[NS - 1]);
  }
  // the step-dependent scalars after the loads are in flight
  const StepParams p = kEarly ? early : device_scalars(p0);
  if (in) {
#pragma unroll
    for (int t = 0; t < V; ++t) {
      float uu[N];
#pragma unroll
      for (int j = 0; j < N; ++j) uu[j] = uv[j][t];
      float vt = (FORM != kSgdm) ? val[NS - 1][t] : 0.0f;
      update_element<FORM, N, ORDER>(p, sc, gv[t], val[0][t], uu, vt);
      val[0][t] = as_stored<XT>(val[0][t]);
#pragma unroll
      for (int j = 0; j < N; ++j) val[1 + j][t] = uu[j];
      val[NS - 1][t] = vt;
    }
  }
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    if (FORM == kSgdm && k == NS - 1) continue;
    const bool due = ((mask >> k) & 1u) != 0;
    if (!due) {
      if (!in) continue;
      if (k == 0) store_v<XT, V, NTS>(x, r, val[0]);
      else if (k == NS - 1) store_v<float, V, NTS>(p0.v, r, val[k]);
      else store_v<float, V, NTS>(p0.u[k - 1], r, val[k]);
      continue;
    }
#pragma unroll
    for (int t = 0; t < V; ++t) lds[m][t * 64 + lane] = val[k][t];
    __syncthreads();
    // column t (element e + t of every lane) is averaged by wave t mod K
    for (int t = m; in && t < V; t += K) {
      const float s0 = lds[0][t * 64 + lane];
      double d = 0.0;
#pragma unroll 4
      for (int32_t q = 1; q < K; ++q) mean_add(d, lds[q][t * 64 + lane], s0);
      lds[0][t * 64 + lane] = mean_of(s0, d, rk);
    }
    __syncthreads();
    if (k == 0 && p0.outer.xo != nullptr) {
      // run j of 64 consecutive elements to wave j mod K
      const int64_t e0 = tile * (int64_t)(64 * V);
      for (int j = m * 64 + lane; j < 64 * V; j += 64 * K) {
        if (e0 + j >= p0.P) continue;
        float a[1] = {lds[0][(j % V) * 64 + j / V]};
        outer_step<1>(p0.outer, e0 + j, a);
        lds[0][(j % V) * 64 + j / V] = a[0];
      }
      __syncthreads();
    }
    if (in) {
      float mean[V];
#pragma unroll
      for (int t = 0; t < V; ++t) mean[t] = lds[0][t * 64 + lane];
      if (k == 0) store_v<XT, V, NTS>(x, r, mean);
      else if (k == NS - 1) store_v<float, V, NTS>(p0.v, r, mean);
      else store_v<float, V, NTS>(p0.u[k - 1], r, mean);
    }
    __syncthreads();
  }
}

// Probabilistic SGDM variant (Algorithm 4): the first moments due in mask
// are averaged over the replicas BEFORE the update direction uses them, so
// every replica steps with the averaged momentum; x is updated and, when
// bit 0 is set, averaged as in k_local_step_sync.  Two passes per column:
// pass 1 updates every replica's moments and stores the ones not due (the
// same thread reloads them in pass 2) and the means of the due ones; pass 2
// forms each replica's direction and updates x.
template <int N, typename XT, typename GT, int V, int NTM>
__global__ __launch_bounds__(kBlock) void k_sgdm_averaged_momenta(StepParams p0, uint32_t mask, int32_t K) {
#pragma clang fp contract(off)
  const StepParams p = device_scalars(p0);
  constexpr bool NTL = (NTM & 1) != 0, NTS = (NTM & 2) != 0;
  const bool sync_x = (mask & 1u) != 0;
  bool sync_u[N];
#pragma unroll
  for (int j = 0; j < N; ++j) sync_u[j] = ((mask >> (j + 1)) & 1u) != 0;
  XT* __restrict__ x = reinterpret_cast<XT*>(p.x);
  const GT* __restrict__ g = reinterpret_cast<const GT*>(p.g);
  const double rk = 1.0 / (double)K;

  // a wave's elements are one piece of the tile
  const int64_t base = tile_elem<kBlock * V, 64 * V>(launch_tile(), 0);
  const uint32_t lane_o = (uint32_t)tile_elem<kBlock * V, 64 * V>(0, (int)threadIdx.x * V);
  const int32_t in_row = left_in_row(base, p.P);
  const int32_t n = in_row - (int32_t)lane_o, nw = __builtin_amdgcn_readfirstlane(n);
  auto piece = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    const uint32_t o = F ? slot_in_row<V>(lane_o, in_row) : lane_o;
    // pass 1: u^j of every replica; due ones become their replica mean
    float u0[N][V];
    double du[N][V];
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
      for (int t = 0; t < V; ++t) du[j][t] = 0.0;
    for (int32_t m = 0; m < K; ++m) {
      const int64_t r = (int64_t)m * p.P + base;
      float gv[V], uv[N][V];
      load_n<F, GT, V, NTL>(g + r, o, n, gv);
#pragma unroll
      for (int j = 0; j < N; ++j) load_n<F, float, V, NTL>(p.u[j] + r, o, n, uv[j]);
      const float sc = p.scale != nullptr ? load_uniform(p.scale + m) : 1.0f;
#pragma unroll
      for (int t = 0; t < V; ++t) {
        const float gh = sc * gv[t];
#pragma unroll
        for (int j = 0; j < N; ++j) uv[j][t] = __builtin_fmaf(p.beta[j], uv[j][t], p.omb[j] * gh);
      }
#pragma unroll
      for (int j = 0; j < N; ++j) {
        if (sync_u[j]) {
#pragma unroll
          for (int t = 0; t < V; ++t) {
            if (m == 0) u0[j][t] = uv[j][t];
            else mean_add(du[j][t], uv[j][t], u0[j][t]);
          }
        } else {
          store_n<F, float, V, false>(p.u[j] + r, o, n, uv[j]);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (!sync_u[j]) continue;
#pragma unroll
      for (int t = 0; t < V; ++t) u0[j][t] = mean_of(u0[j][t], du[j][t], rk);
      for (int32_t m = 0; m < K; ++m) store_n<F, float, V, NTS>(p.u[j] + (int64_t)m * p.P + base, o, n, u0[j]);
    }
    // pass 2: direction with the averaged (due) or local (not due) moments
    float x0[V];
    double dx[V];
#pragma unroll
    for (int t = 0; t < V; ++t) dx[t] = 0.0;
    for (int32_t m = 0; m < K; ++m) {
      const int64_t r = (int64_t)m * p.P + base;
      float gv[V], xv[V], uv[N][V];
      load_n<F, GT, V, NTL>(g + r, o, n, gv);
      load_n<F, XT, V, NTL>(x + r, o, n, xv);
#pragma unroll
      for (int j = 0; j < N; ++j) {
        if (sync_u[j]) {
#pragma unroll
          for (int t = 0; t < V; ++t) uv[j][t] = u0[j][t];
        } else {
          load_n<F, float, V, false>(p.u[j] + r, o, n, uv[j]);
        }
      }
      const float sc = p.scale != nullptr ? load_uniform(p.scale + m) : 1.0f;
#pragma unroll
      for (int t = 0; t < V; ++t) {
        const float gh = sc * gv[t];
        float delta = p.gw * gh;
#pragma unroll
        for (int j = 0; j < N; ++j) delta = __builtin_fmaf(p.w[j], uv[j][t], delta);
        xv[t] = as_stored<XT>(__builtin_fmaf(-p.lr, delta, xv[t]));
      }
      if (sync_x) {
#pragma unroll
        for (int t = 0; t < V; ++t) {
          if (m == 0) x0[t] = xv[t];
          else mean_add(dx[t], xv[t], x0[t]);
        }
      } else {
        store_n<F, XT, V, NTS>(x + r, o, n, xv);
      }
    }
    if (sync_x) {
#pragma unroll
      for (int t = 0; t < V; ++t) x0[t] = mean_of(x0[t], dx[t], rk);
      for (int32_t m = 0; m < K; ++m) store_n<F, XT, V, NTS>(x + (int64_t)m * p.P + base, o, n, x0);
    }
  };
  if (nw >= V) piece(BoolC<true>{});
  else if (nw > 0) piece(BoolC<false>{});  // fewer elements than a slot
}

// The same step with one wavefront per replica (blockDim = 64 K,
// 1 < K <= kWaveMaxK), in one pass: wave m loads g, x and every u^j of
// replica m once and updates its moments; the due ones are staged in LDS
// together, averaged and read back by every wave before the direction uses
// them; x is updated and, when due, averaged the same way.  The values equal
// k_sgdm_averaged_momenta's bit for bit; that kernel re-reads g (and the
// moments not due) in its second pass.  Dynamic LDS of K * 64 V floats per
// due moment (and at least one such stage).
template <int N, typename XT, typename GT, int V, int NTM>
__global__ __launch_bounds__(64 * kWaveMaxK) __attribute__((amdgpu_waves_per_eu(8)))
void k_sgdm_averaged_momenta_waves(StepParams p0, uint32_t mask, int32_t K) {
#pragma clang fp contract(off)
  constexpr bool NTL = (NTM & 1) != 0, NTS = (NTM & 2) != 0;
  constexpr int E = 64 * V;
  extern __shared__ __align__(16) float stage[];
  const int32_t m = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
  const int64_t e0 = group_piece(p0.group) * E, row = (int64_t)m * p0.P + e0;
  const uint32_t o = (threadIdx.x & 63) * V;
  const int32_t in_row = left_in_row(e0, p0.P), n = in_row - (int32_t)o;
  if (in_row == 0) return;  // a whole workgroup past the row
  XT* x = reinterpret_cast<XT*>(p0.x) + row;
  const GT* g = reinterpret_cast<const GT*>(p0.g) + row;
  const double rk = 1.0 / (double)K;

  auto piece = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    float gv[V], xv[V], uv[N][V];
    load_n<F, GT, V, NTL>(g, o, n, gv);
#pragma unroll
    for (int j = 0; j < N; ++j) load_n<F, float, V, NTL>(p0.u[j] + row, o, n, uv[j]);
    load_n<F, XT, V, NTL>(x, o, n, xv);
    const float sc = p0.scale != nullptr ? load_uniform(p0.scale + m) : 1.0f;
    const StepParams p = device_scalars(p0);
    const OuterAhead<1> none{};
#pragma unroll
    for (int t = 0; t < V; ++t) {
      const float gh = sc * gv[t];
#pragma unroll
      for (int j = 0; j < N; ++j) uv[j][t] = __builtin_fmaf(p.beta[j], uv[j][t], p.omb[j] * gh);
    }
    int32_t due = 0;
#pragma unroll
    for (int j = 0; j < N; ++j)
      if ((mask >> (j + 1)) & 1u) lds_put<V>(stage + (due++ * K + m) * E + o, uv[j]);
    __syncthreads();
    average_stages<E>(stage, K, due, in_row, rk, p0.outer, false, none, e0);
    __syncthreads();
    due = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if ((mask >> (j + 1)) & 1u) lds_get<V>(stage + due++ * K * E + o, uv[j]);
      store_n<F, float, V, NTS>(p0.u[j] + row, o, n, uv[j]);
    }
#pragma unroll
    for (int t = 0; t < V; ++t) {
      const float gh = sc * gv[t];
      float delta = p.gw * gh;
#pragma unroll
      for (int j = 0; j < N; ++j) delta = __builtin_fmaf(p.w[j], uv[j][t], delta);
      xv[t] = as_stored<XT>(__builtin_fmaf(-p.lr, delta, xv[t]));
    }
    if (mask & 1u) {
      __syncthreads();  // every wave has read the moments' means
      lds_put<V>(stage + m * E + o, xv);
      __syncthreads();
      average_stages<E>(stage, K, 1, in_row, rk, p0.outer, false, none, e0);
      __syncthreads();
      lds_get<V>(stage + o, xv);
    }
    store_n<F, XT, V, NTS>(x, o, n, xv);
  };
  if (in_row >= E) piece(BoolC<true>{});
  else piece(BoolC<false>{});
}

// The same with one exchange per due state, for row lengths that are a
// multiple of V and K > 8, as in k_local_step_sync_waves_rounds (16.8M x 16,
// N = 2, all due: 1349 us, staged together 1371 us), or K > 4 and 8 bytes
// loaded per element (N = 1, bf16 parameters and gradients, 1.2 GB loaded:
// K = 5 341 us, staged together 360 us; K = 7 353 / 365 us, clipped 387 /
// 406 us; K = 8 equal).
template <int N, typename XT, typename GT, int V, int NTM>
__global__ __launch_bounds__(64 * kWaveMaxK) __attribute__((amdgpu_waves_per_eu(8)))
void k_sgdm_averaged_momenta_waves_rounds(StepParams p0, uint32_t mask, int32_t K) {
#pragma clang fp contract(off)
  const StepParams p = device_scalars(p0);
  constexpr bool NTL = (NTM & 1) != 0, NTS = (NTM & 2) != 0;
  __shared__ float lds[kWaveMaxK][64 * V];
  const int32_t m = threadIdx.x >> 6, lane = threadIdx.x & 63;
  XT* __restrict__ x = reinterpret_cast<XT*>(p.x);
  const GT* __restrict__ g = reinterpret_cast<const GT*>(p.g);
  const double rk = 1.0 / (double)K;
  const float sc = p.scale != nullptr ? load_uniform(p.scale + __builtin_amdgcn_readfirstlane(m)) : 1.0f;

  // the mean over the replicas of val (this wave's row values), through
  // LDS, written back into val
  auto average = [&](float (&val)[V], bool in) {
#pragma unroll
    for (int t = 0; t < V; ++t) lds[m][t * 64 + lane] = val[t];
    __syncthreads();
    for (int t = m; in && t < V; t += K) {
      const float s0 = lds[0][t * 64 + lane];
      double d = 0.0;
#pragma unroll 4
      for (int32_t q = 1; q < K; ++q) mean_add(d, lds[q][t * 64 + lane], s0);
      lds[0][t * 64 + lane] = mean_of(s0, d, rk);
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < V; ++t) val[t] = lds[0][t * 64 + lane];
    __syncthreads();
  };

  const int64_t tile = launch_tile();
  const int64_t e = tile * (int64_t)(64 * V) + (int64_t)lane * V;
  if (tile * (int64_t)(64 * V) >= p.P) return;  // a whole workgroup past the row
  const bool in = e < p.P;
  const int64_t r = (int64_t)m * p.P + e;
  float gv[V], xv[V], uv[N][V];
#pragma unroll
  for (int t = 0; t < V; ++t) gv[t] = xv[t] = 0.0f;
#pragma unroll
  for (int j = 0; j < N; ++j)
#pragma unroll
    for (int t = 0; t < V; ++t) uv[j][t] = 0.0f;
  if (in) {
    load_v<GT, V, NTL>(g, r, gv);
    load_v<XT, V, NTL>(x, r, xv);
#pragma unroll
    for (int j = 0; j < N; ++j) load_v<float, V, NTL>(p.u[j], r, uv[j]);
  }
#pragma unroll
  for (int t = 0; t < V; ++t) {
    const float gh = sc * gv[t];
#pragma unroll
    for (int j = 0; j < N; ++j) uv[j][t] = __builtin_fmaf(p.beta[j], uv[j][t], p.omb[j] * gh);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    if ((mask >> (j + 1)) & 1u) average(uv[j], in);
    if (in) store_v<float, V, NTS>(p.u[j], r, uv[j]);
  }
#pragma unroll
  for (int t = 0; t < V; ++t) {
    const float gh = sc * gv[t];
    float delta = p.gw * gh;
#pragma unroll
    for (int j = 0; j < N; ++j) delta = __builtin_fmaf(p.w[j], uv[j][t], delta);
    xv[t] = as_stored<XT>(__builtin_fmaf(-p.lr, delta, xv[t]));
  }
  if (mask & 1u) average(xv, in);
  if (in) store_v<XT, V, NTS>(x, r, xv);
}

// ADOPT's first update with the previous-v order: v = g^2, nothing else,
// over the n = K P elements as flat arrays.
template <typename GT, int V>
__global__ __launch_bounds__(kBlock) void k_adopt_init_v(const void* gp, float* vp, int64_t total) {
  const int64_t base = launch_tile() * (kBlock * V);
  const uint32_t o = threadIdx.x * V;
  const int32_t n = left_in_row(base, total) - (int32_t)o;
  const GT* g = reinterpret_cast<const GT*>(gp) + base;
  float a[V];
  auto piece = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    load_n<F, GT, V, false>(g, o, n, a);
#pragma unroll
    for (int t = 0; t < V; ++t) a[t] = a[t] * a[t];
    store_n<F, float, V, false>(vp + base, o, n, a);
  };
  if (n >= V) piece(BoolC<true>{});
  else if (n > 0) piece(BoolC<false>{});
}

// --------------------------------------------------------- replica mean

struct MeanParams {
  void* state[kMaxMeanStates];  // [K][P] buffers of one storage type
  int64_t P;
  int64_t tiles;                // k_replica_mean_stats: workgroups
  double rk;                    // k_replica_mean_waves: 1 / K
  int32_t K;
  int32_t group;                // group_piece
  int32_t outer_state;          // index of x in state[] when OuterOpt applies, else -1
  OuterParams outer;
};

// E_m[S] for the state blockIdx.z: every element becomes
// S^0 + (sum_{m>=1} (S^m - S^0)) / K (mean_of) and is stored to all K rows.
// Each thread reads the K rows of its own columns, R at a time, and writes
// them back, so the in-place update has no cross-thread hazard.
template <typename T, int V, bool NT, int R>
__global__ __launch_bounds__(kBlock) void k_replica_mean(MeanParams p) {
  T* s = reinterpret_cast<T*>(p.state[blockIdx.z]);
  const double rk = 1.0 / (double)p.K;
  // a wave's elements are one piece of the tile
  const int64_t base = tile_elem<kBlock * V, 64 * V>(launch_tile(), 0);
  const uint32_t lane_o = (uint32_t)tile_elem<kBlock * V, 64 * V>(0, (int)threadIdx.x * V);
  const int32_t in_row = left_in_row(base, p.P);
  const int32_t n = in_row - (int32_t)lane_o, nw = __builtin_amdgcn_readfirstlane(n);
  auto piece = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    const uint32_t o = F ? slot_in_row<V>(lane_o, in_row) : lane_o;
    float s0[V], q[V];
    double d[V];
    load_n<F, T, V, NT>(s + base, o, n, s0);
#pragma unroll
    for (int t = 0; t < V; ++t) d[t] = 0.0;
    int32_t m = 1;
    for (; m + R <= p.K; m += R) {
      float r[R][V];
#pragma unroll
      for (int i = 0; i < R; ++i) load_n<F, T, V, NT>(s + (int64_t)(m + i) * p.P + base, o, n, r[i]);
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int t = 0; t < V; ++t) mean_add(d[t], r[i][t], s0[t]);
    }
    for (; m < p.K; ++m) {
      load_n<F, T, V, NT>(s + (int64_t)m * p.P + base, o, n, q);
#pragma unroll
      for (int t = 0; t < V; ++t) mean_add(d[t], q[t], s0[t]);
    }
#pragma unroll
    for (int t = 0; t < V; ++t) s0[t] = mean_of(s0[t], d[t], rk);
    if ((int32_t)blockIdx.z == p.outer_state) outer_step_n<F, V>(p.outer, base + o, n, s0);
    for (m = 0; m < p.K; ++m) store_n<F, T, V, NT>(s + (int64_t)m * p.P + base, o, n, s0);
  };
  if (nw >= V) piece(BoolC<true>{});
  else if (nw > 0) piece(BoolC<false>{});  // fewer elements than a slot
}

// The same mean with whole waves per replica row (blockDim = 64 K / R,
// 1 < K <= kWaveMaxK, R | K; dynamic LDS of K * 64 * V floats): each
// workgroup takes one piece of 64 V consecutive elements (a 1 KiB access
// for fp32 and bf16 rows), wave w loads the pieces of rows w, w + W, ...,
// w + (R - 1) W (W = K / R waves), the K pieces meet in LDS, all waves share
// the means (mean_add / mean_of in replica order, so every element gets
// exactly the value k_replica_mean gives), the OuterOpt runs element by
// element on x (O: one of the launch's states takes it), and each wave stores
// the mean to its rows.  Each wave then issues R loads and R stores per
// piece, as a plain copy does; a thread that walks all K rows of its columns
// (k_replica_mean) ran the K = 4 mean at 74% of the HBM peak on MI355X, this
// kernel runs at 82% (1.31B x 4 fp32: 6.37 ms).  A wave has one access per
// piece in flight, so whatever stands between its load and its store costs
// bandwidth: with 1 / K divided or loaded between the barriers, the OuterOpt
// in the same code, a signed element count that was divided into stages, and
// the rows' sum unrolled by four (K = 4 has three to add) the same pass took
// 6.57 ms.
template <typename T, int V, bool NT, bool O, int R = 1>
__global__ __launch_bounds__(64 * kWaveMaxK / R) void k_replica_mean_waves(MeanParams p) {
  constexpr int E = 64 * V, U = kPieceMaxU * V / 4;
  extern __shared__ __align__(16) float stage[];
  const int32_t K = p.K, W = K / R, lane = threadIdx.x & 63;
  const int32_t w = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
  const int64_t e0 = group_piece(p.group) * E;
  const int32_t in_row = left_in_row(e0, p.P), n = in_row - lane * V;
  if (in_row == 0) return;  // a whole workgroup past the row
  T* s = reinterpret_cast<T*>(p.state[blockIdx.z]) + e0;
  const bool outer = O && (int32_t)blockIdx.z == p.outer_state;
  double rk = p.rk;
  asm("" : "+s"(rk));  // loaded here, not between the barriers

  auto piece = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    const uint32_t place = lane * V, o = F ? slot_in_row<V>(place, in_row) : place;  // in LDS, in the row
    float a[R][V];
#pragma unroll
    for (int r = 0; r < R; ++r) load_n<F, T, V, NT>(s + (int64_t)(w + r * W) * p.P, o, n, a[r]);
    OuterAhead<U> ahead;
    if (outer) outer_ahead<E>(p.outer, e0, in_row, ahead);
#pragma unroll
    for (int r = 0; r < R; ++r) lds_put<V>(stage + (w + r * W) * E + place, a[r]);
    __syncthreads();
    // run r of 64 elements to wave r mod W
    auto average = [&](uint32_t r, auto&& put) {
      const int32_t j = (int32_t)(r * 64) + lane;
      if (!F && j >= in_row) return;
      const float s0 = stage[j];
      double d = 0.0;
#pragma unroll 3
      for (int32_t q = 1; q < K; ++q) mean_add(d, stage[q * E + j], s0);
      stage[j] = put(j, mean_of(s0, d, rk));
    };
    if (outer) {
#pragma unroll
      for (int i = 0; i < U; ++i)
        if (w + i * W < E / 64)
          average(w + i * W, [&](int32_t j, float a) {
            return outer_element(p.outer, e0 + j, ahead.xo[i], ahead.mom[i], a);
          });
    } else {
      for (uint32_t r = w; r < E / 64; r += W) average(r, [](int32_t, float a) { return a; });
    }
    __syncthreads();
    float b[V];
    lds_get<V>(stage + place, b);
#pragma unroll
    for (int r = 0; r < R; ++r) store_n<F, T, V, NT>(s + (int64_t)(w + r * W) * p.P, o, n, b);
  };
  // the OuterOpt takes elements by their place in LDS: the row's last ones one by one
  if (in_row >= (outer ? E : V)) piece(BoolC<true>{});
  else piece(BoolC<false>{});
}

// ----------------------------------------------------- global-norm clip

// One 64-lane DPP move of a double (both halves), rows outside RowMask and
// lanes without a source read 0.
template <int Ctrl, int RowMask>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, Ctrl, RowMask, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), Ctrl, RowMask, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// Sum of a double over the 64 lanes of a wave, in a fixed order, returned
// as a wave-uniform value.  Quad permutes [1,0,3,2] and [2,3,0,1], the
// half-row mirror and the row mirror leave every lane with its 16-lane
// row's sum; the row-15 broadcast (rows 1 and 3) and the row-31 broadcast
// (rows 2 and 3) carry the lower rows' sums into row 3, and lane 63 holds
// the total.  DPP moves stay in the vector ALU: the xor-shuffle butterfly
// goes through ds_bpermute, two LDS permutes of 256 B per step for a
// double, and in the diagnostics kernel, which ends every workgroup with
// five such sums per wave, that LDS traffic cost more time than the
// workgroup's own data exchange.
__device__ __forceinline__ double wave_sum(double a) {
  a += dpp_f64<0xB1, 0xf>(a);   // quad_perm [1,0,3,2]
  a += dpp_f64<0x4E, 0xf>(a);   // quad_perm [2,3,0,1]
  a += dpp_f64<0x141, 0xf>(a);  // row_half_mirror
  a += dpp_f64<0x140, 0xf>(a);  // row_mirror
  a += dpp_f64<0x142, 0xa>(a);  // row_bcast:15 into rows 1, 3
  a += dpp_f64<0x143, 0xc>(a);  // row_bcast:31 into rows 2, 3
  const unsigned long long b = __builtin_bit_cast(unsigned long long, a);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, 63);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 63);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Partial sums of g^2 in fp64 for replica blockIdx.y; each block writes
// one partial (fixed order: deterministic for a fixed grid).  A tile issues
// its U loads back to back, so U vector loads per lane are in flight.  A
// tile's pieces are spread over 8 T elements, so the last eight tiles of a
// row, which are all tiles of a short one, reach past its end: there a lane
// whose slot does loads the row's last V elements instead and counts those
// that lie in its slot.
template <typename GT, int V, int U, int C>
__global__ __launch_bounds__(kBlock) void k_sumsq_partial(const void* gp, int64_t P, double* __restrict__ partials) {
  constexpr int T = kBlock * V * U;
  const int64_t base = tile_elem<T, C>(blockIdx.x, 0);
  const GT* __restrict__ g = reinterpret_cast<const GT*>(gp) + (int64_t)blockIdx.y * P + base;
  const int32_t in_row = left_in_row(base, P);
  const uint32_t last = (uint32_t)tile_elem<T, C>(0, ((U - 1) * kBlock + (kBlock - 1)) * V) + V;
  double acc = 0.0;
  auto offset = [](int k) { return (uint32_t)tile_elem<T, C>(0, (k * kBlock + (int)threadIdx.x) * V); };
  auto tile = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    float a[U][V];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const uint32_t o = offset(k), end = (uint32_t)in_row - V;
      load_n<true, GT, V, false>(g, F || o < end ? o : end, V, a[k]);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      // elements [V - n, V) of the load lie in the slot
      const int32_t n = F ? V : in_row - (int32_t)offset(k);
#pragma unroll
      for (int t = 0; t < V; ++t) {
        const double d = F || t >= V - n ? (double)a[k][t] : 0.0;
        acc = __builtin_fma(d, d, acc);
      }
    }
  };
  if (in_row >= (int32_t)last) {
    tile(BoolC<true>{});
  } else if (in_row >= V) {
    tile(BoolC<false>{});
  } else if (threadIdx.x == 0) {  // fewer elements than a slot
    for (int32_t t = 0; t < in_row; ++t) {
      float a[1];
      load_v<GT, 1, false>(g, t, a);
      const double d = (double)a[0];
      acc = __builtin_fma(d, d, acc);
    }
  }
  acc = wave_sum(acc);
  __shared__ double ws[kBlock / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) ws[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < kBlock / 64; ++i) t += ws[i];
    partials[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
  }
}

// scale[m] = min(1, rho / ||g^m||), 1 for a zero norm; one workgroup of
// kFinalizeBlock threads per replica sums that replica's nb partials in a
// fixed order (thread-strided, four independent accumulators per thread so
// four loads are in flight, then waves in order): deterministic for a given
// nb, and short next to the norm pass even with one partial per 4096
// elements.
constexpr int kFinalizeBlock = 1024;

__global__ __launch_bounds__(kFinalizeBlock) void k_clip_finalize(const double* __restrict__ partials, int32_t nb,
                                                                  double rho, float* __restrict__ scale) {
  const int32_t m = blockIdx.x;
  const double* __restrict__ q = partials + (int64_t)m * nb;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  int32_t i = threadIdx.x;
  for (; i + 3 * kFinalizeBlock < nb; i += 4 * kFinalizeBlock) {
    a0 += q[i];
    a1 += q[i + kFinalizeBlock];
    a2 += q[i + 2 * kFinalizeBlock];
    a3 += q[i + 3 * kFinalizeBlock];
  }
  for (; i < nb; i += kFinalizeBlock) a0 += q[i];
  double acc = wave_sum((a0 + a1) + (a2 + a3));
  __shared__ double ws[kFinalizeBlock / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) ws[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kFinalizeBlock / 64; ++w) t += ws[w];
    const double norm = __builtin_sqrt(t);
    double c = 1.0;
    if (norm > 0.0) {
      c = rho / norm;
      if (!(c < 1.0)) c = 1.0;
    }
    scale[m] = (float)c;
  }
}

// ------------------------------------------------ averaging diagnostics

constexpr int kStatsMaxK = 16;
constexpr int kStatsStride = 4 + 2 * kStatsMaxK;  // doubles per state (layout in mtdao.h)

// The replica mean of the wave-per-replica kernel (same pieces, same
// mean_add / mean_of order, same values) plus, from the values before
// averaging, the averaging diagnostics of state blockIdx.z: ||cbar||^2,
// sum_m ||c^m - cbar||^2, ||xo||^2, ||c^m||^2 and <c^m, cbar>, with
// c^m = S^m, or c^m = xo - x^m for x under a Nesterov OuterOpt.
// blockDim = 64 K (1 <= K <= kStatsMaxK), dynamic LDS of 2 K * 64 V floats.
// Workgroup b takes Q pieces of 64 V elements, pieces ((b / 8) Q + i) 8 +
// b mod 8 for i < Q: each XCD keeps one piece in eight, and as workgroups
// are dispatched in order the pieces in flight stay a compact window, as in
// the plain mean (a fixed grid of workgroups striding over the row scattered
// them and ran 30% slower).  The next piece's loads are issued before a
// piece's exchange, and consecutive pieces use two LDS buffers in turn, so a
// piece takes two barriers.  That the loads stay in flight over the exchange
// takes code without branches between them and their use (the last pieces of
// a row have code of their own) and slots kept as stored: with both kinds of
// piece and the conversion in one body the compiler waited for the next
// piece at once (fp32, 16M x 4 one state 127 us, now 113; 4M x 16 175 -> 122;
// bf16 92 -> 71 and 124 -> 78 us, at 78 registers against 56 now).  Each wave keeps fp64 sums for its own replica
// (wave 0 also those of cbar and xo).  Rows of whole 16-byte slots: a lane
// forms the V products of a piece in fp32 (one rounding each, about 6e-8
// relative) and adds their fp32 sum to the fp64 sums, which keeps the fp64
// work per element to a fraction of an operation.  Other rows (EACH) add
// every product, rounded to fp32, to the fp64 sums by itself.  The workgroup
// writes its kStatsSums(K) sums, contiguous, to
// partials[state][workgroup][sum]:
//   0 ||cbar||^2, 1 sum_m ||c^m - cbar||^2, 2 ||xo||^2,
//   3 + m ||c^m||^2, 3 + K + m <c^m, cbar>.
__host__ __device__ constexpr int kStatsSums(int K) { return 3 + 2 * K; }

// A 16-byte slot of a row as it is stored.
template <typename T>
struct Slot;
template <>
struct Slot<float> : f32x4 {};
template <>
struct Slot<uint16_t> : u16x8 {};
__device__ __forceinline__ float widen(float a) { return a; }
__device__ __forceinline__ float widen(uint16_t a) { return bf16_to_f32(a); }

template <typename T, int V, int Q, bool EACH, bool O>
__global__ __launch_bounds__(64 * kStatsMaxK) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 && O ? 7 : 8)))
void k_replica_mean_stats(MeanParams p, double* __restrict__ partials) {
  constexpr int E = 64 * V;
  extern __shared__ __align__(16) float stage[];  // [2][K][64 V]
  __shared__ double red[kStatsMaxK][5];
  const int32_t K = p.K, lane = threadIdx.x & 63;
  const int32_t m = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
  const int64_t block = launch_tile();
  if (block >= p.tiles) return;
  const bool outer = O && (int32_t)blockIdx.z == p.outer_state;
  const double rk = p.rk;
  T* row = reinterpret_cast<T*>(p.state[blockIdx.z]) + (int64_t)m * p.P;
  const uint32_t o = lane * V;
  double a_sq = 0.0, a_dot = 0.0, a_var = 0.0, a_mean = 0.0, a_ref = 0.0;
  auto first = [&](int i) { return (((block >> 3) * Q + i) * 8 + (block & 7)) * E; };
  // all Q pieces whole: one branch for the workgroup, so that a piece waits
  // for its own loads and leaves the next one's in flight
  auto pieces = [&](auto full) {
    constexpr bool F = decltype(full)::value;
    auto fetch = [&](int64_t e0) {
      const int32_t n = left_in_row(e0, p.P) - (int32_t)o;
      typename Slot<T>::type a = {};  // a piece past the row is not loaded
      if (F || n + (int32_t)o >= E) {
        a = ld<true, Slot<T>>(at((const T*)row + e0, o));
      } else if (e0 < p.P) {
        T b[V];
#pragma unroll
        for (int t = 0; t < V; ++t) b[t] = *at((const T*)row + e0, o + min(t, n - 1));
#pragma unroll
        for (int t = 0; t < V; ++t) a[t] = t < n ? b[t] : (T)0;
      }
      return a;
    };
    typename Slot<T>::type cur = fetch(first(0)), next = cur;
#pragma unroll 1
    for (int i = 0; i < Q; ++i) {
      const int64_t e0 = first(i);
      if (!F && e0 >= p.P) break;  // uniform over the workgroup
      const int32_t in_row = F ? E : left_in_row(e0, p.P), n = in_row - (int32_t)o;
      const bool whole = F || in_row >= E;
      float* buf = stage + (i & 1) * K * E;
      if (i + 1 < Q) next = fetch(first(i + 1));
      float a[V], xo[V];
      if (outer) {
        if (whole) load_n<true, float, V, false>(p.outer.xo + e0, o, n, xo);
        else load_n<false, float, V, false>(p.outer.xo + e0, o, n, xo);
      }
#pragma unroll
      for (int t = 0; t < V; ++t) a[t] = widen((T)cur[t]);
      lds_put<V>(buf + m * E + o, a);
      __syncthreads();
      average_stages<E>(buf, K, 1, in_row, rk, p.outer, false, OuterAhead<1>{}, e0);
      __syncthreads();
      float mean[V], out[V];
      lds_get<V>(buf + o, mean);
      if (outer) {
        __syncthreads();  // every wave has read the means before the outer step rewrites them
        if (p.outer.update)
          for (int32_t j = threadIdx.x; j < E; j += blockDim.x)
            if (j < in_row) buf[j] = outer_element(p.outer, e0 + j, p.outer.xo[e0 + j], p.outer.mom[e0 + j], buf[j]);
        __syncthreads();
        lds_get<V>(buf + o, out);
      } else {
#pragma unroll
        for (int t = 0; t < V; ++t) out[t] = mean[t];
      }
      // store first, then reduce the diagnostics while the stores drain
      if (whole) store_n<true, T, V, true>(row + e0, o, n, out);
      else store_n<false, T, V, true>(row + e0, o, n, out);
      // the terms of the piece's V elements (values, means and outer parameters
      // beyond the row are 0): each product rounded to fp32 once, then added to
      // the fp64 sums (EACH) or to an fp32 sum that joins them once per piece
      float f_sq = 0.0f, f_dot = 0.0f, f_var = 0.0f, f_mean = 0.0f, f_ref = 0.0f;
#pragma unroll
      for (int t = 0; t < V; ++t) {
        const float c0 = widen((T)cur[t]);
        const float cbar = outer ? xo[t] - mean[t] : mean[t];
        const float c = outer ? xo[t] - c0 : c0;
        const float dv = c0 - mean[t];  // c - cbar up to sign
        auto add = [&](double& sum, float& part, float y, float z) {
          if constexpr (EACH) sum += (double)(y * z);
          else part = __builtin_fmaf(y, z, part);
        };
        add(a_sq, f_sq, c, c);
        add(a_dot, f_dot, c, cbar);
        add(a_var, f_var, dv, dv);
        if (m == 0) {
          add(a_mean, f_mean, cbar, cbar);
          if (outer) add(a_ref, f_ref, xo[t], xo[t]);
        }
      }
      if constexpr (!EACH) {
        a_sq += (double)f_sq;
        a_dot += (double)f_dot;
        a_var += (double)f_var;
        if (m == 0) {
          a_mean += (double)f_mean;
          if (outer) a_ref += (double)f_ref;
        }
      }
      cur = next;
    }
  };
  if (first(Q - 1) + E <= p.P) pieces(BoolC<true>{});
  else pieces(BoolC<false>{});
  // the workgroup's sums, fixed order
  const double sq = wave_sum(a_sq), dot = wave_sum(a_dot), var = wave_sum(a_var);
  const double mn = wave_sum(a_mean), ref = wave_sum(a_ref);
  if (lane == 0) {
    red[m][0] = sq;
    red[m][1] = dot;
    red[m][2] = var;
    red[m][3] = mn;
    red[m][4] = ref;
  }
  __syncthreads();
  const int ns = kStatsSums(K);
  if ((int)threadIdx.x < ns) {
    const int k = threadIdx.x;
    double v = 0.0;
    if (k == 0) v = red[0][3];
    else if (k == 1) for (int32_t q = 0; q < K; ++q) v += red[q][2];
    else if (k == 2) v = red[0][4];
    else if (k < 3 + K) v = red[k - 3][0];
    else v = red[k - 3 - K][1];
    partials[((int64_t)blockIdx.z * p.tiles + block) * ns + k] = v;
  }
}

// Fixed-order reduction of the workgroup sums, in two levels: rows of
// ns = kStatsSums(K) sums, contiguous in memory.  Thread t adds sum t mod ns
// of rows t / ns, t / ns + G, ... (G rows per pass, so consecutive threads
// read consecutive sums), four rows in flight, and the G group totals are
// added in order.  (A thread that added whole rows waited for each of its ns
// loads in turn, and one workgroup per 8192 rows left most CUs idle.)
constexpr int kStatsMaxSums = 3 + 2 * kStatsMaxK;
constexpr int kStatsChunk = 256;    // rows of a first-level workgroup
constexpr int kStatsBlock = 512;

// Sum k of rows [lo, hi) of q (row r at q + r * stride) into tot[k], k < ns.
__device__ __forceinline__ void stats_sum_rows(const double* __restrict__ q, int64_t stride, int64_t lo, int64_t hi,
                                               int32_t ns, double* tot) {
  __shared__ double part[kStatsBlock];
  const int32_t G = kStatsBlock / ns, k = threadIdx.x % ns, first = threadIdx.x / ns;
  if (first < G) {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int64_t r = lo + first;
    for (; r + 3 * G < hi; r += 4 * G) {
      const double b0 = q[r * stride + k], b1 = q[(r + G) * stride + k];
      const double b2 = q[(r + 2 * G) * stride + k], b3 = q[(r + 3 * G) * stride + k];
      a0 += b0;
      a1 += b1;
      a2 += b2;
      a3 += b3;
    }
    for (; r < hi; r += G) a0 += q[r * stride + k];
    part[threadIdx.x] = (a0 + a1) + (a2 + a3);
  }
  __syncthreads();
  if ((int)threadIdx.x < ns) {
    double t = 0.0;
    for (int32_t i = 0; i < G; ++i) t += part[i * ns + threadIdx.x];
    tot[threadIdx.x] = t;
  }
  __syncthreads();
}

// Level 1: the sums of chunk blockIdx.x (kStatsChunk workgroup rows) of
// state blockIdx.y replace the chunk's first row.
__global__ __launch_bounds__(kStatsBlock) void k_stats_reduce(double* __restrict__ partials, int64_t nb, int32_t ns) {
  __shared__ double tot[kStatsMaxSums];
  double* q = partials + (int64_t)blockIdx.y * nb * ns;
  const int64_t lo = (int64_t)blockIdx.x * kStatsChunk;
  const int64_t hi = lo + kStatsChunk < nb ? lo + kStatsChunk : nb;
  stats_sum_rows(q, ns, lo, hi, ns, tot);
  if ((int)threadIdx.x < ns) q[lo * ns + threadIdx.x] = tot[threadIdx.x];
}

// Level 2: the chunk sums of state blockIdx.x into out in the layout of
// mtdao.h (kStatsStride doubles per state; slot 3 and the slots of workers
// m >= K are 0); the variance sum is divided by K.
__global__ __launch_bounds__(kStatsBlock) void k_stats_finalize(const double* __restrict__ partials, int64_t nb,
                                                                int32_t K, double* __restrict__ out) {
  __shared__ double tot[kStatsMaxSums];
  const int32_t state = blockIdx.x, ns = kStatsSums(K);
  stats_sum_rows(partials + (int64_t)state * nb * ns, (int64_t)kStatsChunk * ns, 0,
                 (nb + kStatsChunk - 1) / kStatsChunk, ns, tot);
  if (threadIdx.x < kStatsStride) {
    const int k = threadIdx.x;
    double t = 0.0;
    if (k < 3) t = tot[k];
    else if (k >= 4 && k < 4 + K) t = tot[3 + (k - 4)];
    else if (k >= 4 + kStatsMaxK && k < 4 + kStatsMaxK + K) t = tot[3 + K + (k - 4 - kStatsMaxK)];
    out[(int64_t)state * kStatsStride + k] = (k == 1) ? t / (double)K : t;
  }
}

// ------------------------------------------------------------ init

// Rows 1..K-1 of x <- row 0 (every worker starts from the same x_0).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_broadcast_row0(T* __restrict__ x, int64_t P, int32_t K) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < P; i += stride) {
    const T a = x[i];
    for (int32_t m = 1; m < K; ++m) x[(int64_t)m * P + i] = a;
  }
}

// xo[i] = x[0][i] widened to fp32 (the outer parameters start at x_0).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_row0_to_f32(const T* __restrict__ x, float* __restrict__ xo, int64_t P) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < P; i += stride) {
    if constexpr (sizeof(T) == 2) xo[i] = bf16_to_f32(x[i]);
    else xo[i] = x[i];
  }
}

__global__ __launch_bounds__(kBlock) void k_fill_zero(float* __restrict__ a, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) a[i] = 0.0f;
}

}  // namespace mtdao
